"""GPU parity of the batched persistent queue: every instance of a batch
equals the oracle (Life bit-exact; distance map within the FP32 bound), and
the graph, stream and per-instance launch modes give identical bits."""
import numpy as np
import pytest

import oracle
from gpu_helpers import dev, host, note, padded_ld
from paper_1609_01490_amd import inputs

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def _tm():
    from paper_1609_01490_amd import trimap
    return trimap


def _make(tm, spec, d, steps, edm_tile, life_tile, seed, flags=0, all16=False):
    import torch
    kinds, ns, ds, host_in, A, B = [], [], [], [], [], []
    for k, (kind, n) in enumerate(spec):
        if kind == "edm":
            X, _ = inputs.points(n, d, dup_frac=0.0, seed=seed + k)
            host_in.append(X)
            A.append(dev(X))
            B.append(torch.full((n * (n - 1) // 2,), -1.0, dtype=torch.float32, device="cuda"))
            kinds.append(tm.KIND_EDM)
        else:
            # every other Life grid with rows padded to 16 bytes (the
            # bit-sliced body moves those rows as 16-byte vectors)
            ld = padded_ld(n, 16 if all16 or k % 4 == 1 else 4)
            g = inputs.life(n, 0.3, seed=seed + k, ld=ld)
            host_in.append(g)
            A.append(dev(g))
            B.append(torch.zeros_like(A[-1]))
            kinds.append(tm.KIND_LIFE)
        ns.append(n)
        ds.append(d)
    b = tm.Batch(kinds, ns, ds, edm_tile=edm_tile, life_tile=life_tile, life_steps=steps,
                 flags=flags)
    b.bind(A, B)
    return b, host_in, A, B


def _results(spec, A, B, steps):
    out = []
    for (kind, n), a, b in zip(spec, A, B):
        if kind == "edm":
            out.append(host(b))
        else:
            out.append(host(a if steps % 2 == 0 else b)[:, :n])
    return out


def _check_oracle(spec, host_in, res, d, steps):
    for (kind, n), x, r in zip(spec, host_in, res):
        if kind == "edm":
            if n < 2:
                continue
            e = oracle.edm_condensed(x)
            nz = e > 0
            rel = np.abs(r.astype(np.float64)[nz] - e[nz]) / e[nz]
            assert rel.max() <= (d + 2) * U / 2 + U, (n, rel.max())
        else:
            exp = oracle.gol(x, n, steps)
            low = np.tril(np.ones((n, n), dtype=bool))
            assert (r[low] == exp[low]).all(), n


@pytest.mark.parametrize("edm_tile,life_tile,flags,all16", [
    (16, 8, 0, False), (32, 16, 0, False), (32, 32, 0, False), (64, 64, 0, False),
    (32, 16, 32, False), (64, 64, 32, False), (64, 64, 32, True), (16, 64, 32, True)])
def test_batch_matches_oracle_and_modes(edm_tile, life_tile, flags, all16):
    """all16: every Life grid with 16-byte rows, so that tile 64 with several
    generations per node binds the bit-sliced kernel (one tile per wave)."""
    tm = _tm()
    rng = np.random.default_rng(edm_tile + life_tile)
    spec = [("edm" if k % 2 == 0 else "life", int(n)) for k, n in
            enumerate(rng.integers(2, 260, size=14))] + [("edm", 2), ("life", 1), ("life", 3),
                                                          ("life", 33 * 64 + 5), ("edm", 70),
                                                          ("life", 33 * 64 + 5)]
    d, steps = 32, 5
    outs = {}
    for how in (tm.BATCH_GRAPH, tm.BATCH_STREAM, tm.BATCH_PER_INSTANCE):
        note("batch", edm_tile, life_tile, flags, all16, how)
        b, host_in, A, B = _make(tm, spec, d, steps, edm_tile, life_tile, seed=70, flags=flags,
                                 all16=all16)
        b.launch(how)
        outs[how] = _results(spec, A, B, steps)
        if how == tm.BATCH_GRAPH:
            _check_oracle(spec, host_in, outs[how], d, steps)
    for how in (tm.BATCH_STREAM, tm.BATCH_PER_INSTANCE):
        for x, y in zip(outs[tm.BATCH_GRAPH], outs[how]):
            assert (x.view(np.uint8) == y.view(np.uint8)).all()


@pytest.mark.parametrize("life_tile,flags,all16", [(32, 0, False), (64, 32, True)])
@pytest.mark.parametrize("d", [31, 33, 100, 512, 513])
def test_batch_distance_dimensions(life_tile, flags, all16, d):
    """Distance tiles of 64 on both sides of the dimensions that take products
    (32 to 512), ragged ones among them: the FP32 bound, and the per-instance
    launches' bits.  19 generations: one node of windows."""
    tm = _tm()
    spec = [("edm", 65), ("life", 300), ("edm", 66), ("edm", 2), ("edm", 200), ("life", 70)]
    res = []
    for how in (tm.BATCH_GRAPH, tm.BATCH_PER_INSTANCE):
        note("batch dimensions", life_tile, flags, d, how)
        b, host_in, A, B = _make(tm, spec, d, 19, 64, life_tile, seed=95, flags=flags, all16=all16)
        b.launch(how)
        res.append(_results(spec, A, B, 19))
        _check_oracle(spec, host_in, res[-1], d, 19)
    for x, y in zip(*res):
        assert (x.view(np.uint8) == y.view(np.uint8)).all()


def test_batch_graph_replays():
    """The graph is replayed several times with eager work in between; every
    replay must give the same (oracle-checked) result."""
    import torch
    tm = _tm()
    spec = [("life", 100), ("edm", 90), ("life", 37), ("edm", 300), ("life", 250)]
    d, steps = 16, 4  # even: a Life grid holds the result and is re-run from there
    b, host_in, A, B = _make(tm, spec, d, steps, 32, 32, seed=90)
    ref = None
    state = [x.copy() for x in host_in]
    for rep in range(3):
        note("batch replay", rep)
        b.launch(tm.BATCH_GRAPH)
        torch.cuda.synchronize()
        _ = torch.ones(1000, device="cuda").sum().item()  # eager work between replays
        res = _results(spec, A, B, steps)
        # Life continues from where it stopped, distance maps are recomputed
        for k, (kind, n) in enumerate(spec):
            if kind == "life":
                state[k] = np.pad(oracle.gol(state[k], n, steps), ((0, 0), (0, state[k].shape[1] - n)))
        for (kind, n), x, s, r in zip(spec, host_in, state, res):
            if kind == "life":
                low = np.tril(np.ones((n, n), dtype=bool))
                assert (r[low] == s[:, :n][low]).all(), (rep, n)
        if ref is None:
            ref = [r for r, (kind, _) in zip(res, spec) if kind == "edm"]
        else:
            for x, y in zip(ref, [r for r, (kind, _) in zip(res, spec) if kind == "edm"]):
                assert (x == y).all()


def test_batch_plan_errors():
    tm = _tm()
    with pytest.raises(tm.TrimapError):
        tm.Batch([0, 1], [10, 10], [4, 4], edm_tile=8)
    with pytest.raises(tm.TrimapError):
        tm.Batch([0, 5], [10, 10], [4, 4])
    with pytest.raises(tm.TrimapError):
        tm.Batch([0], [10], [0])
    b = tm.Batch([0, 1], [10, 10], [4, 4])
    with pytest.raises(tm.TrimapError):
        b.launch(tm.BATCH_GRAPH)   # not bound


def test_batch_autotune_choice_is_valid_and_exact():
    tm = _tm()
    spec = [("edm", 120), ("life", 200), ("edm", 33), ("life", 64), ("life", 9)]
    d, steps = 16, 3
    import torch
    kinds, ns, ds, A, B = [], [], [], [], []
    for k, (kind, n) in enumerate(spec):
        if kind == "edm":
            X, _ = inputs.points(n, d, dup_frac=0.0, seed=200 + k)
            A.append(dev(X))
            B.append(torch.empty((n * (n - 1) // 2,), dtype=torch.float32, device="cuda"))
            kinds.append(tm.KIND_EDM)
        else:
            ld = padded_ld(n)
            A.append(dev(inputs.life(n, 0.3, seed=200 + k, ld=ld)))
            B.append(torch.zeros_like(A[-1]))
            kinds.append(tm.KIND_LIFE)
        ns.append(n)
        ds.append(d)
    note("batch autotune")
    te, tl, fl, ms = tm.batch_autotune(kinds, ns, ds, steps, A, B, reps=1)
    assert te in (16, 32, 64) and tl in (8, 16, 32, 64) and fl in (0, 32) and ms > 0
    # the chosen tiles give the oracle's results
    b, host_in, A2, B2 = _make(tm, spec, d, steps, te, tl, seed=300, flags=fl)
    b.launch(tm.BATCH_GRAPH)
    _check_oracle(spec, host_in, _results(spec, A2, B2, steps), d, steps)


@pytest.mark.parametrize("all16,nodes", [(True, 2), (False, 6)])
def test_batch_binding_picks_the_life_kernel(all16, nodes):
    """20 generations with tile 64 and temporal blocking: Life grids all with
    16-byte rows bind the bit-sliced kernel (up to 16 generations per node:
    2 nodes), otherwise the byte-sliced one (up to 4: 6 nodes); both equal
    the oracle."""
    tm = _tm()
    spec = [("life", 300), ("edm", 90), ("life", 2117), ("life", 65)]
    d, steps = 16, 20
    b, host_in, A, B = _make(tm, spec, d, steps, 32, 64, seed=81, flags=tm.FLAG_LIFE_TEMPORAL,
                             all16=all16)
    note("batch binding", all16)
    if not all16:
        assert any(a.stride(0) % 16 for a, (k, _) in zip(A, spec) if k == "life")
    assert b.info["graph_nodes"] == nodes
    b.launch(tm.BATCH_GRAPH)
    _check_oracle(spec, host_in, _results(spec, A, B, steps), d, steps)


@pytest.mark.slow
def test_batch_512_benchmark_shape_matches_oracle():
    """The 512-instance batch exactly as the benchmark builds and times it
    (inputs.batch_instances(): n log-uniform in [64, 8192], even index a
    distance map with d = 32, odd index Life for 20 generations with rows
    padded to 16 bytes; distance tile 64, Life tile 64 with temporal
    blocking, one graph launch).  Every distance instance is checked on
    whole sampled rows (the first, the last and two seeded random ones)
    within the FP32 bound, a seeded sample of 16 Life instances (always with
    the largest) on the whole grid, bit-exact; the per-instance launches give
    the same bits on that sample."""
    import concurrent.futures as cf
    import torch
    tm = _tm()
    d, steps = 32, 20
    spec = inputs.batch_instances()
    assert len(spec) == 512
    kinds, ns, ds, A, B, host_in = [], [], [], [], [], []
    for k, (kind, n) in enumerate(spec):
        seed = inputs.seed_for(4) * 1000 + k
        if kind == "edm":
            X, _ = inputs.points(n, d, dup_frac=0.0, seed=seed)
            host_in.append(X)
            A.append(dev(X))
            B.append(torch.full((n * (n - 1) // 2,), -1.0, dtype=torch.float32, device="cuda"))
            kinds.append(tm.KIND_EDM)
        else:
            g = inputs.life(n, 0.3, seed=seed, ld=padded_ld(n, 16))
            host_in.append(g)
            A.append(dev(g))
            B.append(torch.zeros_like(A[-1]))
            kinds.append(tm.KIND_LIFE)
        ns.append(n)
        ds.append(d)
    note("batch 512: inputs on the device")
    b = tm.Batch(kinds, ns, ds, edm_tile=64, life_tile=64, life_steps=steps,
                 flags=tm.FLAG_LIFE_TEMPORAL)
    b.bind(A, B)
    assert b.info["graph_nodes"] < steps  # temporally blocked nodes
    note("batch 512: graph launch")
    b.launch(tm.BATCH_GRAPH)
    torch.cuda.synchronize()

    rng = np.random.default_rng(512)
    life_idx = [k for k, (kind, _) in enumerate(spec) if kind == "life"]
    largest = max(life_idx, key=lambda k: spec[k][1])
    sample = sorted(set(rng.choice(life_idx, 15, replace=False).tolist()) | {largest})

    def life_result(k):
        n = spec[k][1]
        return host(A[k] if steps % 2 == 0 else B[k])[:, :n].copy()

    got_life = {k: life_result(k) for k in sample}
    edm_rows = {}
    for k, (kind, n) in enumerate(spec):
        if kind == "edm":
            rows = sorted({1, n - 1} | set(rng.integers(1, n, 2).tolist()))
            edm_rows[k] = (rows, [B[k][r * (r - 1) // 2: r * (r - 1) // 2 + r].cpu().numpy()
                                  for r in rows])
    note("batch 512: oracle")
    bound = (d + 2) * U / 2 + U
    for k, (rows, got) in edm_rows.items():
        for r, g, e in zip(rows, got, oracle.edm_rows(host_in[k], rows)):
            nz = e > 0
            rel = np.abs(g.astype(np.float64)[nz] - e[nz]) / e[nz]
            assert rel.size == 0 or rel.max() <= bound, (k, r, rel.max())

    def life_oracle(k):
        n = spec[k][1]
        return k, oracle.gol(host_in[k], n, steps)

    with cf.ThreadPoolExecutor(8) as ex:
        for k, exp in ex.map(life_oracle, sample):
            n = spec[k][1]
            low = np.tril(np.ones((n, n), dtype=bool))
            assert (got_life[k][low] == exp[low]).all(), (k, n)
            note("batch 512: life instance", k, n, "exact")

    # the same bodies launched per instance, from generation 0 again
    for k in life_idx:
        A[k].copy_(dev(host_in[k]))
        B[k].zero_()
    note("batch 512: per-instance launches")
    b.launch(tm.BATCH_PER_INSTANCE)
    torch.cuda.synchronize()
    for k in sample:
        assert (life_result(k) == got_life[k]).all(), k
    for k, (rows, got) in edm_rows.items():
        for r, g in zip(rows, got):
            assert (B[k][r * (r - 1) // 2: r * (r - 1) // 2 + r].cpu().numpy().view(np.uint32)
                    == g.view(np.uint32)).all(), (k, r)
    b.close()
    del A, B
    torch.cuda.empty_cache()
