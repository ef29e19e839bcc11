"""The tuner's cache: a build with settings fixed by the caller leaves nothing
behind that an unrestricted build of the same graph would take, and both find
their own entry again."""
import pytest

import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fixed,field,value", [
    (dict(roots_in_flight=3), "roots_in_flight", 3),
    (dict(wg_size=1024), "wg_size", 1024),
    (dict(delta=123457), "delta", 123457),
    (dict(small=False), "small_trees", 0),
    (dict(early_term=False), None, None),
])
@pytest.mark.parametrize("prune", [-1, 64])
def test_fixed_settings_keep_to_themselves(fixed, field, value, prune):
    from paper_1907_00140_amd import chl
    # a graph of its own for every case: the cache lives as long as the process
    seed = 7000 + prune + sum(map(ord, str(fixed)))
    n, u, v, w = gg.random_edges(3000, 9000, 1, 100, seed)
    row, col, ww = gg.to_csr(n, u, v, w)
    order = gg.degree_rank(row, seed)

    def settings(**kw):
        L = chl.build(row, col, ww, order, prune_hubs=prune, **kw)
        st = L.stats()
        L.free()
        return st

    print("tune cache", fixed, prune, flush=True)
    a = settings(**fixed)
    assert a["tune_ms"] > 0 and (field is None or a[field] == value)
    free = settings()
    assert free["tune_ms"] > 0, "tuned by a restricted build"
    keys = ("roots_in_flight", "wg_size", "delta", "small_trees")
    for again, st in ((settings(), free), (settings(**fixed), a)):
        assert again["tune_ms"] == 0
        assert [again[k] for k in keys] == [st[k] for k in keys]
