"""Rates that bench.py reports per kernel: the passes after the decision run on
accepted attempts only, their mean time over all attempts does not go with the
bytes of one that ran (1.02 of the memory's peak at half the attempts)."""
import bench


def test_passes_after_the_decision_are_rated_by_their_counted_bytes():
    n, ms = 1000, 0.5
    kb = bench.kernel_bytes(4)
    timed = {k: {"avg_ms": ms, "count": 3} for k in kb}
    rates = bench.kernel_rates(kb, timed, {"lncc_bwd": 24 * n}, n)
    for k in ("update", "lncc_fwd"):
        assert rates[k]["achieved"] == round(kb[k] * n / (ms * 1e-3) / 1e9, 1)
    assert rates["lncc_bwd"]["achieved"] == round(24 * n / (ms * 1e-3) / 1e9, 1)
    assert rates["lncc_bwd"]["traffic"] == 24 * n
    for k in ("smooth", "decide"):
        assert "achieved" not in rates[k] and rates[k]["launches"] == 3
