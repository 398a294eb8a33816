"""The autotuner times every tile/map candidate, returns the fastest, caches
it, and never changes results (integer and Life bodies are tile-invariant)."""
import numpy as np
import pytest

import oracle
from gpu_helpers import dev, host, note, padded_ld
from paper_1609_01490_amd import inputs

pytestmark = pytest.mark.gpu


def _tm():
    from paper_1609_01490_amd import trimap
    return trimap


@pytest.mark.parametrize("workload,n,d", [(0, 4096, 0), (1, 2048, 0), (2, 2048, 0),
                                          (3, 700, 32), (4, 700, 32)])
def test_autotune_picks_the_fastest_candidate(workload, n, d, tmp_path):
    tm = _tm()
    tm.tune_cache_clear()
    note("autotune", workload, n, d)
    best, allc = tm.autotune(workload, n, d, reps=2, use_cache=False)
    assert allc, "no candidate timed"
    assert best["ms"] == min(c["ms"] for c in allc)
    assert all(c["ms"] > 0 for c in allc)
    maps = {c["map"] for c in allc}
    assert "lambda" in maps and "bb" in maps
    # a cached answer comes back unchanged without timing
    again, allc2 = tm.autotune(workload, n, d, reps=2, use_cache=True)
    assert again == best and allc2 == []
    # save / load round trip
    f = str(tmp_path / "tune.json")
    tm.tune_cache_save(f)
    tm.tune_cache_clear()
    tm.tune_cache_load(f)
    third, allc3 = tm.autotune(workload, n, d, reps=2, use_cache=True)
    assert allc3 == [] and third["tile"] == best["tile"] and third["map"] == best["map"]
    # the chosen (tile, map, flags) runs the body and gives the oracle's result
    note("autotune choice", workload, best)
    _check_choice(tm, workload, n, d, best)


def _check_choice(tm, workload, n, d, ch):
    import torch
    U = 2.0 ** -24
    if workload in (0, 1, 2):
        p = tm.Plan(n, ch["tile"], ch["map"], flags=ch["flags"])
    else:
        p = tm.Plan(n, ch["tile"], ch["map"], include_diag=False, flags=ch["flags"])
    if workload == 0:
        ld = padded_ld(n)
        a, X, Y, C0 = inputs.f32_elementwise(n, seed=31, ld=ld)
        c = dev(C0)
        p.elementwise(tm.OP_AXPYT_F32, dev(X), dev(Y), c, ld=ld, a=float(a))
        exp = C0.copy()
        oracle.c1(a, X, Y, exp, n=n)
        assert (host(c).view(np.uint32) == exp.view(np.uint32)).all()
    elif workload == 1:
        A, B, C0 = inputs.int_elementwise(n, seed=32)
        c = dev(C0)
        p.elementwise(tm.OP_XORMUL_I32, dev(A), dev(B), c, ld=n)
        exp = C0.copy()
        oracle.c0(A, B, exp)
        assert (host(c) == exp).all()
    elif workload == 2:
        steps = 21
        g = inputs.life(n, 0.3, seed=33, ld=padded_ld(n, 16))
        cur, nxt = dev(g), torch.zeros((n, g.shape[1]), dtype=torch.uint8, device="cuda")
        p.stencil(cur, nxt, steps)
        got = host(nxt if steps % 2 else cur)[:, :n]
        low = np.tril(np.ones((n, n), dtype=bool))
        assert (got[low] == oracle.gol(g, n, steps)[low]).all()
    else:
        mode = tm.EDM_FP32 if workload == 3 else tm.EDM_BF16X3
        X, _ = inputs.points(n, d, dup_frac=0.02, seed=34)
        out = torch.full((n * (n - 1) // 2,), -1.0, dtype=torch.float32, device="cuda")
        ws = None
        if mode != tm.EDM_FP32:
            ws = torch.empty(p.edm_workspace_size(d, mode), dtype=torch.uint8, device="cuda")
        p.edm(dev(X), out, mode=mode, ws=ws)
        got = host(out)
        e = oracle.edm_condensed(X)
        nz = e > 0
        rel = np.abs(got.astype(np.float64)[nz] - e[nz]) / e[nz]
        assert rel.max() <= ((d + 2) * U / 2 + U if mode == tm.EDM_FP32 else 1e-3)


@pytest.mark.parametrize("workload,n,d", [(0, 1000, 0), (0, 1024, 0), (1, 1000, 0), (1, 1024, 0),
                                          (2, 1000, 8), (3, 300, 32), (3, 300, 8)])
def test_autotune_times_no_launch_twice(workload, n, d):
    """Flags that a kernel ignores make no candidates of their own."""
    tm = _tm()
    tm.tune_cache_clear()
    note("autotune candidates", workload, n, d)
    _, allc = tm.autotune(workload, n, d, reps=1, use_cache=False)
    assert len({(c["tile"], c["map"], c["flags"]) for c in allc}) == len(allc)
    orders = tm.FLAG_XCD_SWIZZLE | tm.FLAG_ORDER_REVERSE | tm.FLAG_ORDER_PAIRS
    for tile in {c["tile"] for c in allc}:
        lam = [c["flags"] for c in allc if c["tile"] == tile and c["map"] == "lambda"]
        if workload == 2:
            temporal = [f for f in lam if f & tm.FLAG_LIFE_TEMPORAL]
            assert len(temporal) == {8: 0, 16: 3, 32: 3, 64: 1}[tile]
        elif workload == 3:
            assert lam == [0]
        else:
            plain = [f for f in lam if f & ~orders == 0]
            swizzled = n % 32 != 0 and (workload == 0 or tile < 32)
            assert len(plain) == (1 if swizzled else 5), tile
    tm.tune_cache_clear()
