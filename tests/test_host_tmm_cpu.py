"""Which thin-film queries are solved by kind, and in how many workgroups
(precision 0 double, 1 mixed, 2 single; the stand-in GPU has 256 CUs)."""
import pytest

from tests.host_only import run

FULL = 2 * 256 * 256                                         # queries of two workgroups a CU


@pytest.mark.parametrize("precision,n_layers,silver,n,by_kind,blocks", [
    (1, 200, False, 2000, True, 8),                          # a query a lane, as in order
    (1, 8, True, 64, True, 1),
    (1, 2000, False, 100000, True, 391),
    (1, 200, True, FULL, True, 512),
    (1, 200, True, FULL + 1, True, 410),                     # 320 queries a workgroup
    (0, 200, False, FULL, False, 512),
    (0, 200, False, FULL + 1, True, 410),
    (0, 31, False, FULL + 1, False, 513),
    (0, 200, True, 300000, False, 1172),
    (2, 200, False, 300000, False, 1172)])
def test_rule_of_queries_by_kind(precision, n_layers, silver, n, by_kind, blocks):
    out = run(f"""
assert h.tmm({n_layers}, {silver}, {n}, {precision}) == 0, h.error()
k, = h.kernels('k_tmm_rt')
out['k'] = k[:3]
""")
    name, b, threads = out["k"]
    # mangled template arguments: precision, tables by value, by kind
    assert f"ILi{precision}ELb" in name
    assert (name.split("ELb")[2][0] == "1") == by_kind
    assert (b, threads) == (blocks, 256)
