"""GPU parity of the kernel that multiplies the binary planes as 4-bit floats on the matrix cores
(two to sixteen activation vectors): at the edges of its row units (64 rows), K steps (128 columns), tiles
of one and two sub-slabs and vector counts, for every plane count it takes, all scale layouts, and
for activations its digits do not hold (infinities, NaNs) or hold only just (subnormals beside the
largest numbers); sums that go from the registers to y or to the workspace, and row ranges that are
worked through in several stretches, with and without infinities."""
import numpy as np
import pytest

import paper_2206_09557_amd as L
from oracle import bcq_oracle as O
from oracle import c_oracle
from paper_2206_09557_amd import synth

from gpu_util import Packed, check_parity, row_l1_bound, run

pytestmark = pytest.mark.gpu

MODES = {"greedy": L.LUTGEMM_Q_GREEDY, "greedy_z": L.LUTGEMM_Q_GREEDY_MEAN_OFFSET, "rtn": L.LUTGEMM_Q_UNIFORM_RTN}

# m, n, q, g, mode, batch.  One scale group per K step: 4, 2 and 1 operand rows per vector (batch <= 4, <= 8,
# <= 16), up to six planes; two groups per step (g = 64, 192): batch 5 to 8, up to four planes.
CASES = [
    (1, 128, 1, 128, "greedy", 3),           # one row, one K step, one plane
    (63, 256, 2, 128, "greedy_z", 4),
    (64, 1024, 3, 128, "greedy", 5),         # exactly one row unit and one tile
    (65, 1152, 3, 128, "rtn", 8),            # a row more, a last tile of one K step in one sub-slab
    (129, 1536, 4, 0, "greedy_z", 9),        # last tile with exactly 64 chunks: one sub-slab, four steps
    (257, 1544, 6, 0, "greedy", 16),         # ... and with 65: two sub-slabs, a step of 8 columns
    (300, 1032, 5, 0, "rtn", 2),             # row-wise scales on a length no step divides
    (256, 8, 3, 8, "greedy", 2),             # a single chunk
    (700, 2048, 6, 256, "greedy_z", 7),
    (333, 640, 4, 64, "rtn", 5),             # two groups per step
    (500, 2112, 3, 64, "greedy_z", 8),       # ... the last step holds one of them
    (130, 4224, 2, 192, "greedy", 13),       # ... groups that straddle steps, eight vectors and five
    (48, 65536, 3, 128, "greedy_z", 3),      # many K groups on one row unit
    (20000, 384, 2, 128, "greedy", 12),      # many row units on one K group
    (4100, 3072, 4, 128, "rtn", 19),         # sixteen vectors and three
]


@pytest.mark.parametrize("m,n,q,g,mode,batch", CASES)
def test_edges_match_oracle(m, n, q, g, mode, batch):
    print(f"case fp4 m={m} n={n} q={q} g={g} mode={mode} batch={batch}", flush=True)
    W = synth.weights_fp16(m, n, seed=16000 + m + 7 * n + q)
    X = synth.activations_fp16(n, seed=16500 + m + n, batch=batch)
    p = Packed.from_weights(W, q, g, MODES[mode])
    gg = n if g == 0 else g
    z = None if p.z is None else O.decode_z(p.z, m, n // gg)
    bound = row_l1_bound(O.decode_alpha(p.alpha, m, n // gg, q), z, gg)
    y_ref, _ = c_oracle.gemv_packed(p.bits, p.alpha, p.z, X, m, n, q, g)
    y = run(p, X, f32_out=True)
    for b in range(batch):
        check_parity(y[b], y_ref[b], X[b], bound, f32_out=True)
    np.testing.assert_array_equal(y.astype(np.float16), run(p, X))
    np.testing.assert_array_equal(run(p, X, f32_out=True), y)        # bitwise reproducible
    if mode == "rtn":                                                # one scale per group: the same bits
        p.share()
        np.testing.assert_array_equal(run(p, X, f32_out=True, shared=True), y)
    if gg % 64 == 0 and 3 <= batch <= 8 and q <= 4:                  # one kernel behind the three ways to ask
        np.testing.assert_array_equal(run(p, X, f32_out=True, auto=True), run(p, X, f32_out=True, mfma=True))


@pytest.mark.parametrize("g,batch,mode,shared", [(128, 4, "greedy", False), (128, 8, "greedy", False), (128, 16, "greedy", False),
                                                 (64, 8, "greedy", False), (128, 8, "greedy_z", False), (128, 8, "rtn", False),
                                                 (128, 8, "rtn", True)])
def test_wide_range_activations(g, batch, mode, shared):
    # Subnormals, ordinary numbers and the largest ones within one block of 32 columns.  A digit expansion
    # is off by at most 2^-29 of the block's largest magnitude per activation; everything else is exact or
    # an fp32 rounding, of which a sum of up to 12 steps of 3 planes and offsets, added up in 64 bits behind
    # that, has at most 24 in a row (8 chains of a step, 12 steps, 3 operand rows):
    # |error| <= (sum(alpha) + |z|) * (32 * 2^-29 * sum over blocks of the largest + 24 * 2^-24 * |x|_1).
    m, n, q = 200, 2048, 3
    W = synth.weights_fp16(m, n, seed=16900)
    p = Packed.from_weights(W, q, g, MODES[mode])
    if shared:
        p.share()
    X = synth.activations_fp16(n, seed=16901, batch=batch)
    X[:, ::5] = np.float16(6.0e-8)
    X[:, 1::37] *= np.float16(1000.0)
    X[0, 7::64] = np.float16(60000.0)
    X[1, :] = (np.arange(n) % 1024 + 1).astype(np.float16) * np.float16(2.0 ** -24)   # subnormals alone: exact digits
    X[2, 2::3] = 0
    y_ref, _ = c_oracle.gemv_packed(p.bits, p.alpha, p.z, X, m, n, q, g)
    y = run(p, X, f32_out=True, shared=shared).astype(np.float64)
    a = O.decode_alpha(p.alpha, m, n // g, q).astype(np.float64).sum(axis=0)
    if p.z is not None:
        a += np.abs(O.decode_z(p.z, m, n // g).astype(np.float64))
    a = a.max(axis=1)
    ax = np.abs(X.astype(np.float64))
    for b in range(batch):
        limit = a * (32 * 2.0 ** -29 * ax[b].reshape(-1, 32).max(axis=1).sum() + 24 * 2.0 ** -24 * ax[b].sum())
        assert (np.abs(y[b] - y_ref[b]) <= limit).all(), f"vector {b}: {np.abs(y[b] - y_ref[b]).max()} against {limit.min()}"


@pytest.mark.parametrize("n,g,batch,mode", [(2048, 128, 3, "greedy"), (1544, 0, 7, "greedy"), (16384, 128, 16, "greedy_z"), (640, 64, 6, "greedy")])
def test_infinities_and_nans(n, g, batch, mode):
    # They reach the rows of their own vector and no other: +-inf where all planes of the column (and a
    # second one's) agree in sign, else NaN; the other vectors' results stay what they are without them.
    m, q = 150, 2
    W = synth.weights_fp16(m, n, seed=17000 + n)
    p = Packed.from_weights(W, q, g, MODES[mode])
    B = L.lutgemm_unpack_bcq(p.bits, m, n, q).astype(np.float64)
    X = synth.activations_fp16(n, seed=17001, batch=batch)
    clean = run(p, X, f32_out=True)
    c0, c1 = 5, n - 3
    X[0, c0] = np.inf
    X[1, [c0, c1]] = [-np.inf, np.inf]
    X[2, c1] = np.nan
    y = run(p, X, f32_out=True)
    np.testing.assert_array_equal(y[3:], clean[3:])
    assert np.isnan(y[2]).all()
    gg = n if g == 0 else g
    z = np.zeros((m, n // gg)) if p.z is None else O.decode_z(p.z, m, n // gg).astype(np.float64)
    for v, cols in ((0, [c0]), (1, [c0, c1])):
        with np.errstate(invalid="ignore"):
            terms = [s * X[v, c].astype(np.float64) for c in cols for s in (B[0, :, c], B[1, :, c])]
            if p.z is not None:
                terms += [z[:, c // gg] * X[v, c].astype(np.float64) for c in cols]
            want = sum(terms)
        np.testing.assert_array_equal(np.isnan(y[v]), np.isnan(want))
        np.testing.assert_array_equal(y[v][~np.isnan(want)], want[~np.isnan(want)])
        assert np.isinf(y[v]).any() or (p.z is not None)


class _Probe:
    """A layer of one plane whose row r returns what the kernel makes of group r's activations: the scale is 1 for
    (row r, group r) and 0 elsewhere, all signs are +1 but that of column 2 of a group's chunks."""

    def __init__(self, g, groups=512):
        self.g, self.groups, n = g, groups, g * groups
        B = np.ones((1, groups, n), dtype=np.int8)
        B[:, :, 2::8] = -1
        alpha, _ = L.lutgemm_pack_scales(np.eye(groups, dtype=np.float16)[None], None, n, g)
        self.p = Packed(L.lutgemm_pack_planes(B), alpha, None, groups, n, 1, g)

    def __call__(self, values, batch, beside=0.0):
        """What `values` come out as, each in a group of its own whose chunk holds +-beside as well (added and
        taken away again)."""
        per_call = batch * self.groups
        v = np.zeros(-(-len(values) // per_call) * per_call, dtype=np.float16)
        v[:len(values)] = values
        out = []
        for part in v.reshape(-1, batch, self.groups):
            X = np.zeros((batch, self.groups, self.g), dtype=np.float16)
            at = 8 * (np.arange(self.groups) % (self.g // 8))       # every chunk of a group in turn
            for col, what in ((0, part), (1, beside), (2, beside)):
                X[:, np.arange(self.groups), at + col] = what
            out.append(run(self.p, X.reshape(batch, -1), f32_out=True))
        return np.concatenate([o.ravel() for o in out])[:len(values)]


def _finite_halves():
    v = np.arange(1 << 16, dtype=np.uint16).view(np.float16)
    return v[np.isfinite(v)]


ROWS_PER_VECTOR = [(128, 4), (128, 8), (128, 16), (64, 8)]     # 4, 2, 1 operand rows per vector; two groups per step


@pytest.mark.parametrize("g,batch", ROWS_PER_VECTOR)
def test_every_finite_activation_alone(g, batch):
    # The largest of its block of 32 columns: digits hold it bit for bit, and the sum has one term.
    v = _finite_halves()
    np.testing.assert_array_equal(_Probe(g)(v, batch), v.astype(np.float32))


@pytest.mark.parametrize("g,batch", ROWS_PER_VECTOR)
def test_activations_beside_the_largest_ones(g, batch):
    # The largest binade, where the first digit may round up to 2^16, which fp16 does not hold: what six digits
    # miss of a number (2^-29 of the power of two below the block's largest), the last bit of a
    # subnormal, and the rounding of the fp32 sum.
    probe, v = _Probe(g), _finite_halves()
    for beside in (63456.0, 63488.0, 64504.0, 65504.0):
        err = np.abs(probe(v, batch, beside).astype(np.float64) - v.astype(np.float64))
        limit = 2.0 ** -29 * 32768.0 + 2.0 ** -24 + 2.0 ** -23 * np.abs(v.astype(np.float64))
        assert (err <= limit).all(), f"beside {beside}: {v[err > limit][:4]} off by {err[err > limit][:4]}"


@pytest.mark.parametrize("g,batch", ROWS_PER_VECTOR)
def test_small_activations_beside_large_ones(g, batch):
    # Beside an activation of magnitude 2^e the digits hold a smaller one to 2^-29 of that power of two (and the
    # last bit of a subnormal in the largest binade): bit for bit down to 2^18 times smaller, where
    # only the rounding of the fp32 sum is left.
    probe, v = _Probe(g), _finite_halves()
    for beside in (2.0 ** -14, 1.5, 1000.0, 65504.0):
        w = v[np.abs(v.astype(np.float64)) <= beside]
        power = 2.0 ** np.floor(np.log2(beside))
        err = np.abs(probe(w, batch, beside).astype(np.float64) - w.astype(np.float64))
        limit = 2.0 ** -29 * power + (2.0 ** -24 if power == 32768.0 else 0.0) + 2.0 ** -23 * np.abs(w.astype(np.float64))
        assert (err <= limit).all(), f"beside {beside}: {w[err > limit][:4]} off by {err[err > limit][:4]}"


@pytest.mark.parametrize("batch", [4, 8, 16])
@pytest.mark.parametrize("period", [32, 64, 1024])
def test_error_with_large_outliers_is_no_larger_than_the_lookups(batch, period):
    # A few activations 2^14 times the others: digits cut off too early, or bits that an accumulator loses
    # where it enters a matrix instruction, show as an error above that of fp32 sums (1.3e-7 to 1.8e-7 here).
    m, n, q, g = 2048, 4096, 3, 128
    p = Packed.from_weights(synth.weights_fp16(m, n, seed=17100), q, g)
    X = synth.activations_fp16(n, seed=17101 + batch, batch=batch)
    X[:, ::period] *= np.float16(2.0 ** 13)
    y_ref, _ = c_oracle.gemv_packed(p.bits, p.alpha, p.z, X, m, n, q, g)

    def error(y):
        return np.linalg.norm(y - y_ref) / np.linalg.norm(y_ref)

    planes, lookups = error(run(p, X, f32_out=True)), error(np.stack([run(p, x, f32_out=True) for x in X]))
    assert planes <= lookups, f"{planes} against {lookups}"


@pytest.mark.parametrize("offsets", [False, True])
@pytest.mark.parametrize("batch", [4, 5, 8, 16])
@pytest.mark.parametrize("spread", [0, 3, 7])
def test_sum_of_a_step_is_its_nearest_number(batch, offsets, spread):
    # K steps of numbers that the first three digits hold, in one or two blocks of the largest magnitude and others
    # 2^spread times smaller (32 columns share a block scale: every other eight of 64).  The sum of two digits takes 24 bits at most (2^8 to 2^-8, and 7 more), the
    # third one's 19: both are exact, and added up they are rounded once, to the exact sum's nearest
    # fp32 number.  Where the third digit enters the accumulator of the other two its last bits are lost.
    # Row r returns K step r's sum (the offset term's: with no signs): it has scales of 1 there and of 0 elsewhere.
    steps, n = 256, 256 * 128
    rng = np.random.default_rng(19000 + 100 * spread + batch)
    signs = rng.choice(np.array([-1, 1], dtype=np.int8), (1, steps, n), p=[0.1, 0.9])
    ones = np.eye(steps, dtype=np.float16)
    alpha, z = L.lutgemm_pack_scales(np.zeros_like(ones)[None] if offsets else ones[None], ones if offsets else None, n, 128)
    p = Packed(L.lutgemm_pack_planes(signs), alpha, z, steps, n, 1, 128)
    assert [k[0] for k in L.lutgemm_plan_gemm(steps, n, 1, 128, offsets, batch)] == [L.LUTGEMM_KERNEL_FP4]
    x = rng.integers(1024, 2048, (batch, steps, 128)) / 1024.0 * 2.0 ** -rng.integers(0, 4, (batch, steps, 128))
    x[:, :, [0, 8, 64, 72]] = 1.0 + rng.integers(0, 1024, (batch, steps, 4)) / 1024.0     # a block's largest is 1 to 2, ...
    down = np.array([[0, 1, 1, 1], [0, 0, 1, 1]])[rng.integers(0, 2, (batch, steps))] * spread    # ... and so many powers of two less
    block = 2 * (np.arange(128) // 64) + np.arange(128) // 8 % 2
    x = x * rng.choice([-1.0, 1.0], x.shape, p=[0.1, 0.9]) * 2.0 ** -down[:, :, block]
    own = signs[0].reshape(steps, steps, 128)[np.arange(steps), np.arange(steps)].astype(np.float64)
    exact = (x if offsets else x * own).sum(axis=2)
    np.testing.assert_array_equal(run(p, x.reshape(batch, n).astype(np.float16), f32_out=True), exact.astype(np.float32))


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("g,batch", ROWS_PER_VECTOR)
@pytest.mark.parametrize("period", [32, 1024])
def test_error_of_large_offsets_with_large_outliers(g, batch, shared, period):
    # The same where the offsets are a thousand times the scales: the result is the offset term's, which has digits and
    # chains of its own.
    m, n, q = 1024, 4096, 3
    rng = np.random.default_rng(19200)
    step = (0.001 + 0.0002 * rng.random((m, n // g))).astype(np.float16)
    alpha = np.stack([step * np.float16(2 ** i) for i in range(q)])
    alpha, z = L.lutgemm_pack_scales(alpha, rng.standard_normal((m, n // g)).astype(np.float16), n, g)
    p = Packed(rng.integers(0, 256, L.lutgemm_bits_bytes(m, n, q), dtype=np.uint8), alpha, z, m, n, q, g).share()
    X = synth.activations_fp16(n, seed=19201 + batch, batch=batch)
    X[:, ::period] *= np.float16(2.0 ** 13)
    y_ref, _ = c_oracle.gemv_packed(p.bits, p.alpha, p.z, X, m, n, q, g)

    def error(y):
        return np.linalg.norm(y - y_ref) / np.linalg.norm(y_ref)

    planes = error(run(p, X, f32_out=True, shared=shared))
    lookups = error(np.stack([run(p, x, f32_out=True, shared=shared) for x in X]))
    assert planes <= lookups, f"{planes} against {lookups}"


@pytest.mark.parametrize("batch,g", [(3, 128), (7, 128), (13, 128), (6, 64)])
def test_infinite_scale_beside_infinite_activations(batch, g):
    # A row with an infinite scale is +inf for finite activations (signs and activations all positive, with
    # some in every digit), whatever other vectors of the call hold, +inf for a vector with +inf of its
    # own, and NaN for one with -inf.
    m, n, q = 70, 512, 3
    alpha = np.full((q, m, n // g), 0.5, dtype=np.float16)
    alpha[1, 3, 0] = np.inf
    packed, _ = L.lutgemm_pack_scales(alpha, None, n, g)
    p = Packed(L.lutgemm_pack_planes(np.ones((q, m, n), dtype=np.int8)), packed, None, m, n, q, g)
    X = np.tile(np.float16([1.0 + 2.0 ** -10, 2.0 ** -17, 2.0 ** -24, 1.0]), (batch, n // 4))
    clean = run(p, X, f32_out=True)
    assert np.isposinf(clean[:, 3]).all() and np.isfinite(np.delete(clean, 3, axis=1)).all()
    X[0, n - 5], X[1, n - 3] = -np.inf, np.inf
    y = run(p, X, f32_out=True)
    np.testing.assert_array_equal(y[2:], clean[2:])
    assert np.isposinf(y[1]).all()
    assert np.isnan(y[0, 3]) and np.isneginf(np.delete(y[0], 3)).all()


def _random_packed(m, n, q, g, seed):
    """A layer packed without a quantiser: random keys, scales of about 1 / 100."""
    rng = np.random.default_rng(seed)
    bits = rng.integers(0, 256, L.lutgemm_bits_bytes(m, n, q), dtype=np.uint8)
    alpha = (0.01 + 0.002 * rng.random(L.lutgemm_alpha_bytes(m, n, q, g) // 2)).astype(np.float16)
    return Packed(bits, alpha, None, m, n, q, g)


# m, n, q, g, batch, K groups (1 or several), how a row range is worked through: "direct" (a row unit's whole K
# group is one item: its sums go from the registers to y, or to the workspace where there are several K
# groups), "even" or "rest" (stretches, the last one full or not)
ROW_RANGE_CASES = [
    (1000, 128, 2, 128, 9, 1, "direct"), (977, 128, 3, 128, 6, 1, "direct"), (996, 128, 4, 0, 4, 1, "direct"),
    (1069, 128, 4, 64, 8, 1, "direct"),
    (17213, 1600, 4, 0, 12, 2, "direct"), (16506, 1600, 2, 0, 6, 2, "direct"), (17051, 1280, 4, 256, 3, 2, "direct"),
    (92109, 1600, 1, 0, 16, 1, "rest"), (91165, 1792, 1, 128, 16, 1, "even"), (142689, 3200, 1, 128, 8, 1, "rest"),
    (779, 125568, 1, 128, 16, 2, "rest"), (582, 120768, 1, 0, 16, 2, "even"), (4673, 79104, 1, 128, 8, 2, "rest"),
]


@pytest.mark.parametrize("m,n,q,g,batch,groups,kind", ROW_RANGE_CASES)
def test_row_ranges(m, n, q, g, batch, groups, kind):
    plan = L.lutgemm_plan_gemm(m, n, q, g, False, batch)
    print(f"case fp4 rows m={m} n={n} q={q} g={g} batch={batch}: {plan}", flush=True)
    (kernel, _, kg, steps, ranges, run_steps, stretch), = plan
    units = -(-(-(-m // 64)) // ranges)
    assert kernel == L.LUTGEMM_KERNEL_FP4 and (kg > 1) == (groups > 1)
    assert kind == ("direct" if run_steps >= steps else "even" if units % stretch == 0 else "rest")
    assert kind == "direct" or stretch < units
    p = _random_packed(m, n, q, g, seed=18000 + m)
    X = synth.activations_fp16(n, seed=18100 + n, batch=batch)
    gg = n if g == 0 else g
    rng = np.random.default_rng(18200)
    per_range = 64 * units
    rows = np.unique(np.concatenate([np.arange(min(m, 70)), np.arange(max(0, m - 70), m), rng.integers(0, m, 100),
                                     np.minimum(per_range + np.arange(-70, 70), m - 1),          # two ranges ...
                                     np.minimum(64 * stretch + np.arange(-70, 70), m - 1)]))     # ... and stretches meet
    rows = rows[rows >= 0]
    bound = row_l1_bound(O.decode_alpha(p.alpha, m, n // gg, q), None, gg)
    y_ref, _ = c_oracle.gemv_packed(p.bits, p.alpha, None, X, m, n, q, g, rows=rows)
    y = run(p, X, f32_out=True)
    for b in range(batch):
        check_parity(y[b][rows], y_ref[b], X[b], bound[rows], f32_out=True)
    np.testing.assert_array_equal(run(p, X, f32_out=True), y)
    np.testing.assert_array_equal(run(p, X), y.astype(np.float16))
    # infinities and NaNs of three vectors, in the first, the last and a middle column: +-inf in the rows where all
    # planes of the column agree in sign, else NaN, and the other vectors untouched
    special = X.copy()
    special[0, 0], special[1, n - 1], special[2, n // 2 + 1] = np.inf, -np.inf, np.nan
    B = L.lutgemm_unpack_bcq(p.bits, m, n, q)
    want = np.stack([B[:, :, 0], -B[:, :, n - 1]]).astype(np.float32).sum(axis=1) / q
    want = np.where(np.abs(want) == 1, np.copysign(np.float32(np.inf), want), np.float32(np.nan))
    del B
    for f32_out in (True, False):
        got, clean = run(p, special, f32_out=f32_out), y if f32_out else y.astype(np.float16)
        np.testing.assert_array_equal(got[3:], clean[3:])
        np.testing.assert_array_equal(got[:2], want.astype(got.dtype))
        assert np.isnan(got[2]).all()
