"""GPU parity of the kernel that multiplies the binary planes as fp16 +-1 on the matrix cores (batches beyond what lookups
and 4-bit floats are the faster way for): at the edges of its row units (64 rows), K steps (128 columns) and tiles of one and two
sub-slabs, K groups of fewer steps than wavefronts, row ranges of several passes of one to three row units, several chains of
fp32 additions, every plane count, group class and scale layout, numbers that are not finite, the error of long rows, and in
a captured graph."""
import numpy as np
import pytest

import paper_2206_09557_amd as L
from oracle import bcq_oracle as O
from oracle import c_oracle
from paper_2206_09557_amd import synth

from gpu_util import Packed, check_parity, make_workspace, row_l1_bound, run

pytestmark = pytest.mark.gpu

MODES = {"greedy": L.LUTGEMM_Q_GREEDY, "greedy_z": L.LUTGEMM_Q_GREEDY_MEAN_OFFSET, "rtn": L.LUTGEMM_Q_UNIFORM_RTN}

# m, n, q, g, mode, batch, lutgemm_gemm with LUTGEMM_PATH_AUTO
CASES = [
    (1, 128, 7, 128, "greedy", 5, False),        # one row, one K step
    (63, 64, 1, 64, "greedy", 17, True),         # half a K step
    (64, 1024, 3, 128, "greedy", 32, True),      # exactly one row unit and one tile
    (65, 1160, 8, 0, "greedy", 31, False),       # a row more; row-wise scales on a length no step divides
    (130, 256, 2, 32, "rtn", 6, False),          # two K steps: wavefronts share out the row units as well
    (700, 480, 3, 32, "greedy_z", 9, False),     # four steps in one sub-slab, groups of 32
    (257, 1312, 4, 32, "greedy", 13, False),     # a last tile of one sub-slab after one of two, groups of 32
    (300, 2080, 6, 160, "rtn", 16, False),       # groups that straddle steps, the last step a quarter of one
    (200, 1344, 5, 64, "greedy_z", 7, False),    # two groups per step, the last step holds one of them
    (333, 4800, 2, 192, "rtn", 19, True),        # ... that straddle steps
    (5000, 640, 2, 64, "greedy", 20, True),      # one row unit per workgroup, then two in one pass
    (20000, 2048, 3, 128, "greedy", 18, True),
    (13000, 1024, 4, 128, "greedy_z", 24, True),
    (48, 65536, 3, 32, "greedy", 12, False),     # many K groups on one row unit
    (1000, 20480, 3, 256, "rtn", 30, True),
    (11000, 3200, 2, 128, "rtn", 17, False),     # in the place of two launches of the 4-bit-float kernel
    (901, 12416, 3, 128, "greedy_z", 20, False),
    (300, 20480, 6, 0, "greedy", 27, False),
    (65, 1088, 5, 64, "greedy", 6, True),        # up to sixteen vectors of the matrix-core path: many planes ...
    (50, 2176, 8, 128, "rtn", 16, True),
    (130, 1280, 7, 0, "greedy_z", 3, True),
    (8200, 16448, 1, 64, "greedy", 13, True),    # ... and large layers of long rows
]


@pytest.mark.parametrize("m,n,q,g,mode,batch,auto", CASES)
def test_edges_match_oracle(m, n, q, g, mode, batch, auto):
    flags = L.LUTGEMM_PATH_AUTO if auto else 0
    plan = L.lutgemm_plan_gemm(m, n, q, g, mode != "greedy", batch, flags)
    print(f"case f16 m={m} n={n} q={q} g={g} mode={mode} batch={batch} plan={plan}", flush=True)
    assert [k[:2] for k in plan] == [(L.LUTGEMM_KERNEL_FP16, batch)]
    if not auto and q <= 6 and (g == 0 or g % 128 == 0):                        # short chains of fp32 additions
        assert plan[0][3] * (q + (mode != "greedy")) <= 16
    W = synth.weights_fp16(m, n, seed=18000 + m + 7 * n + q)
    X = synth.activations_fp16(n, seed=18500 + m + n, batch=batch)
    X[:, ::97] *= np.float16(20.0)
    p = Packed.from_weights(W, q, g, MODES[mode])
    gg = n if g == 0 else g
    z = None if p.z is None else O.decode_z(p.z, m, n // gg)
    bound = row_l1_bound(O.decode_alpha(p.alpha, m, n // gg, q), z, gg)
    y_ref, _ = c_oracle.gemv_packed(p.bits, p.alpha, p.z, X, m, n, q, g)
    y = run(p, X, f32_out=True, auto=auto)
    for b in range(batch):
        check_parity(y[b], y_ref[b], X[b], bound, f32_out=True)
    np.testing.assert_array_equal(y.astype(np.float16), run(p, X, auto=auto))
    np.testing.assert_array_equal(run(p, X, f32_out=True, auto=auto), y)        # bitwise reproducible
    if mode == "rtn" and not auto:                                              # one scale per group: the same bits
        p.share()
        np.testing.assert_array_equal(run(p, X, f32_out=True, shared=True), y)


# lutgemm_gemm_mfma below three vectors, where a workspace holds the fewest K groups.
@pytest.mark.parametrize("m,n,q,g,batch", [(65, 1088, 5, 64, 1), (17, 20480, 8, 128, 1), (130, 9280, 6, 64, 2), (1, 1280, 7, 0, 2)])
def test_one_and_two_vectors(m, n, q, g, batch):
    p = Packed.from_weights(synth.weights_fp16(m, n, seed=18800 + n), q, g)
    X = synth.activations_fp16(n, seed=18801 + n, batch=batch)
    gg = n if g == 0 else g
    bound = row_l1_bound(O.decode_alpha(p.alpha, m, n // gg, q), None, gg)
    y_ref, _ = c_oracle.gemv_packed(p.bits, p.alpha, None, X, m, n, q, g)
    y = run(p, X, f32_out=True, mfma=True)
    for b in range(batch):
        check_parity(y[b], y_ref[b], X[b], bound, f32_out=True)
    np.testing.assert_array_equal(run(p, X, f32_out=True, mfma=True), y)


@pytest.mark.parametrize("m,n,q,g,batch", [(150, 2080, 2, 32, 9), (150, 1312, 7, 32 * 41, 6), (100, 3072, 5, 64, 32)])
def test_infinities_and_nans(m, n, q, g, batch):
    # They reach the rows of their own vector and no other; a scale that is not finite reaches its own row.
    W = synth.weights_fp16(m, n, seed=18900 + n)
    p = Packed.from_weights(W, q, g)
    X = synth.activations_fp16(n, seed=18901, batch=batch)
    clean = run(p, X, f32_out=True)
    assert np.isfinite(clean).all()
    X[0, 5] = np.inf
    X[1, n - 3] = np.nan
    y = run(p, X, f32_out=True)
    np.testing.assert_array_equal(y[2:], clean[2:])
    assert not np.isfinite(y[0]).any() and np.isnan(y[1]).all()
    X = synth.activations_fp16(n, seed=18901, batch=batch)
    alpha = O.decode_alpha(p.alpha, m, n // g, q).copy()
    alpha[0, 77, 0] = np.inf
    packed, _ = L.lutgemm_pack_scales(alpha, None, n, g)
    y = run(Packed(p.bits, packed, None, m, n, q, g), X, f32_out=True)
    assert not np.isfinite(y[:, 77]).any()
    np.testing.assert_array_equal(np.delete(y, 77, axis=1), np.delete(clean, 77, axis=1))


@pytest.mark.parametrize("q,g,batch", [(3, 32, 9), (8, 128, 32)])
def test_captured_and_replayed(q, g, batch):
    import torch
    m, n = 1500, 3072
    assert [k[0] for k in L.lutgemm_plan_gemm(m, n, q, g, False, batch)] == [L.LUTGEMM_KERNEL_FP16]
    p = Packed.from_weights(synth.weights_fp16(m, n, seed=18950), q, g)
    wsb = L.lutgemm_workspace_bytes(m, n, q, g, 8, batch)
    ws = make_workspace(wsb)
    d_x = torch.zeros((batch, n), dtype=torch.float16, device="cuda")
    d_y = torch.zeros((batch, m), dtype=torch.float32, device="cuda")

    def enqueue(stream):
        L.lutgemm_gemm(d_x, p.d_bits, p.d_alpha, None, d_y, q, g, 8, m, n, batch, L.LUTGEMM_Y_F32, ws, wsb, stream)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        enqueue(side.cuda_stream)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        enqueue(torch.cuda.current_stream().cuda_stream)
    for seed in range(3):
        x = synth.activations_fp16(n, seed=18960 + seed, batch=batch)
        d_x.copy_(torch.from_numpy(x))
        d_y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(d_y.cpu().numpy(), run(p, x, f32_out=True))


def _synthetic(m, n, q, g, with_z, seed, factor=0.5):
    """A layer packed without a quantiser: random keys, scales halving from plane to plane (or times `factor`), small
    offsets."""
    rng = np.random.default_rng(seed)
    gg = n if g == 0 else g
    bits = rng.integers(0, 256, L.lutgemm_bits_bytes(m, n, q), dtype=np.uint8)
    spread = 1.0 + 0.1 * rng.standard_normal((m, n // gg), dtype=np.float32).clip(-4, 4)
    alpha = np.stack([(0.016 * spread).astype(np.float16) * np.float16(factor ** k) for k in range(q)])
    z = (0.004 * rng.standard_normal((m, n // gg), dtype=np.float32)).astype(np.float16) if with_z else None
    alpha, z = L.lutgemm_pack_scales(alpha, z, n, gg)
    return Packed(bits, alpha, z, m, n, q, g)


# Long rows on few K groups: with all tiles of one in a single fp32 chain the error was up to 3.3e-7.  `additions`: the most
# that a wavefront makes one after the other there now.  Each rounds by 2.4e-8 of its sum (2^-24 of a number
# between two powers of two, spread evenly), and with scales that halve from plane to plane the sum has about its size from
# the first terms on: sqrt(additions) * 2.4e-8 for a chain, and as much for the sum of such chains.  What is left of short ones
# (the matrix instructions' own sums, the result) measured 4.5e-8.
@pytest.mark.parametrize("m,n,q,g,with_z,batch,auto,additions", [
    (16384, 22016, 3, 32, True, 8, False, 32), (16384, 8256, 6, 96, False, 9, False, 24), (16384, 12288, 4, 64, False, 16, False, 12),
    (12288, 12288, 2, 64, True, 32, False, 12), (16384, 15360, 8, 128, True, 8, False, 32), (7446, 27264, 7, 0, False, 8, False, 24),
    (7446, 27264, 7, 0, False, 24, True, 24), (8192, 22016, 4, 64, True, 32, True, 48), (7446, 27264, 7, 0, False, 8, True, 24),
])
def test_error_of_long_rows(m, n, q, g, with_z, batch, auto, additions):
    plan = L.lutgemm_plan_gemm(m, n, q, g, with_z, batch, L.LUTGEMM_PATH_AUTO if auto else 0)
    print(f"case f16 error m={m} n={n} q={q} g={g} z={with_z} batch={batch} auto={auto}: {plan}", flush=True)
    assert [k[:2] for k in plan] == [(L.LUTGEMM_KERNEL_FP16, batch)]
    p = _synthetic(m, n, q, g, with_z, seed=19000 + n)
    X = synth.activations_fp16(n, seed=19001 + n, batch=batch)
    rows = np.sort(np.random.default_rng(19002).choice(m, 300, replace=False))
    y_ref, _ = c_oracle.gemv_packed(p.bits, p.alpha, p.z, X, m, n, q, g, rows=rows)
    y = run(p, X, f32_out=True, auto=auto)[:, rows]
    error = np.linalg.norm(y - y_ref) / np.linalg.norm(y_ref)
    limit = np.sqrt(additions * 2.4e-8 ** 2 + 4.5e-8 ** 2)
    print(f"error {error:.2e} limit {limit:.2e}", flush=True)
    assert error <= limit


@pytest.mark.parametrize("m,n,q,g,with_z,batch,auto", [
    (70, 1152, 3, 128, False, 24, False), (70, 1152, 3, 128, True, 24, True), (70, 1088, 3, 64, False, 24, True), (70, 1096, 7, 0, False, 8, False),
    (70, 1088, 5, 64, False, 7, False), (70, 640, 3, 32, True, 9, False), (70, 1056, 2, 32, True, 9, False), (70, 200, 8, 40 * 5, True, 6, False),
])
def test_infinite_scale_of_the_last_group(m, n, q, g, with_z, batch, auto):
    # The last K step of a row has no columns for all its segments, and a K tile fewer steps than wavefronts: what has none
    # is zero whatever the scale.  Signs and activations are all positive.
    gg = g or n
    X = np.tile(np.float16([1.0 + 2.0 ** -10, 2.0 ** -17, 2.0 ** -24, 1.0]), (batch, n // 4))
    flags = L.LUTGEMM_PATH_AUTO if auto else 0
    assert [k[0] for k in L.lutgemm_plan_gemm(m, n, q, g, with_z, batch, flags)] == [L.LUTGEMM_KERNEL_FP16]
    for which in range(2 if with_z else 1):
        alpha = np.full((q, m, n // gg), 0.5, dtype=np.float16)
        z = np.full((m, n // gg), 0.25, dtype=np.float16) if with_z else None
        (z if which else alpha[q - 1])[[3, 67], -1] = np.inf
        pa, pz = L.lutgemm_pack_scales(alpha, z, n, gg)
        y = run(Packed(L.lutgemm_pack_planes(np.ones((q, m, n), dtype=np.int8)), pa, pz, m, n, q, g), X, f32_out=True, auto=auto)
        assert np.isposinf(y[:, [3, 67]]).all() and np.isfinite(np.delete(y, [3, 67], axis=1)).all()


# Row ranges of several passes.  m, n, q, g, offsets, batch, LUTGEMM_PATH_AUTO; then row units of a wavefront's pass, wavefronts'
# shares of the row units (of a K group with fewer K steps than wavefronts), passes of a workgroup, K groups and
# chains (one or several).
PASS_CASES = [
    (33300, 1088, 5, 64, False, 17, False, 1, 1, 3, 1, 2),
    (16470, 2176, 1, 32, True, 17, False, 1, 1, 2, 1, 2),
    (18422, 1152, 8, 128, True, 32, False, 1, 1, 2, 1, 2),
    (8597, 2336, 2, 32, False, 13, False, 1, 1, 2, 2, 1),
    (8446, 5184, 3, 192, True, 18, False, 1, 1, 2, 2, 2),
    (98351, 576, 1, 0, False, 24, False, 2, 1, 4, 1, 1),       # seven row units in passes of two
    (98780, 640, 1, 0, True, 18, True, 2, 1, 4, 1, 1),
    (65000, 896, 3, 128, True, 24, False, 2, 1, 2, 1, 1),
    (52206, 1216, 4, 64, False, 24, False, 2, 1, 2, 1, 2),
    (19589, 4288, 4, 64, False, 13, False, 2, 1, 2, 2, 2),
    (73527, 576, 1, 0, False, 18, False, 3, 1, 2, 1, 1),       # five in passes of three
    (97000, 896, 3, 128, False, 32, False, 3, 1, 2, 1, 1),
    (32810, 288, 1, 32, False, 9, False, 1, 2, 2, 1, 1),       # three in passes of two shares, ...
    (133654, 320, 1, 0, False, 17, False, 3, 2, 2, 1, 1),
    (66131, 192, 2, 64, True, 13, False, 1, 4, 2, 1, 1),
    (132915, 64, 1, 32, False, 17, False, 1, 8, 2, 1, 1),      # ... nine in passes of eight
    (138934, 32, 5, 32, True, 24, False, 1, 8, 2, 1, 1),
]


@pytest.mark.parametrize("m,n,q,g,with_z,batch,auto,tall,shares,passes,groups,chains", PASS_CASES)
def test_row_ranges_of_several_passes(m, n, q, g, with_z, batch, auto, tall, shares, passes, groups, chains):
    (kernel, vectors, kg, tiles, ranges, chain, rows), = L.lutgemm_plan_gemm(m, n, q, g, with_z, batch, L.LUTGEMM_PATH_AUTO if auto else 0)
    print(f"case f16 passes m={m} n={n} q={q} g={g} z={with_z} batch={batch}: {(kg, tiles, ranges, chain, rows)}", flush=True)
    blocks = -(-m // 64)
    units = -(-blocks // ranges)
    assert (kernel, vectors) == (L.LUTGEMM_KERNEL_FP16, batch) and rows == tall * shares and -(-units // rows) == passes
    assert shares == (1 if tiles > 1 or n > 512 else 8 // min(8, 1 << (-(-n // 128) - 1).bit_length()))
    assert (kg > 1) == (groups > 1) and (chain < tiles) == (chains > 1)
    p = _synthetic(m, n, q, g, with_z, seed=20000 + m, factor=2.0 if with_z else 0.5)
    X = synth.activations_fp16(n, seed=20001 + n, batch=batch)
    gg = n if g == 0 else g
    z = None if p.z is None else O.decode_z(p.z, m, n // gg)
    # where row units meet in the first two row ranges and the last, and others
    first = np.arange(0, min(2 * units, blocks) + 1) * 64
    check = np.concatenate([(first[:, None] + np.arange(-2, 2)).ravel(), np.arange(m - 130, m),
                            (m - 64 * np.arange(1, units + 1)[:, None] + np.arange(-2, 2)).ravel(),
                            np.random.default_rng(20002).integers(0, m, 150)])
    check = np.unique(check[(check >= 0) & (check < m)])
    bound = row_l1_bound(O.decode_alpha(p.alpha, m, n // gg, q), z, gg)[check]
    y_ref, _ = c_oracle.gemv_packed(p.bits, p.alpha, p.z, X, m, n, q, g, rows=check)
    y = run(p, X, f32_out=True, auto=auto)
    for b in range(batch):
        check_parity(y[b][check], y_ref[b], X[b], bound, f32_out=True)
    np.testing.assert_array_equal(y.astype(np.float16), run(p, X, auto=auto))
    np.testing.assert_array_equal(run(p, X, f32_out=True, auto=auto), y)
    if with_z and not auto:                                                     # one scale per group: the same bits
        p.share()
        np.testing.assert_array_equal(run(p, X, f32_out=True, shared=True), y)
