"""GPU parity of the one-vector kernel for group sizes that are an odd multiple of 8 columns (every
chunk may have a scale set of its own): single tiles and many, a one-sub-slab last tile behind
two-sub-slab tiles of the same K group, row ranges that need several stretches of LDS, every scale
layout, one plane and eight."""
import numpy as np
import pytest

import paper_2206_09557_amd as L
from oracle import bcq_oracle as O
from oracle import c_oracle
from paper_2206_09557_amd import synth
from paper_2206_09557_amd.lutgemm import lutgemm_plan_grid

from gpu_util import Packed, check_parity, row_l1_bound, run

pytestmark = pytest.mark.gpu

MODES = {"greedy": L.LUTGEMM_Q_GREEDY, "greedy_z": L.LUTGEMM_Q_GREEDY_MEAN_OFFSET, "rtn": L.LUTGEMM_Q_UNIFORM_RTN}

CASES = [
    (1, 8, 1, 8, "greedy"),                 # one row, one chunk
    (17, 72, 3, 24, "greedy_z"),            # one tile of one sub-slab: y written directly
    (33, 1000, 2, 40, "rtn"),               # ... of two
    (300, 1032, 8, 8, "greedy_z"),          # a last tile of one chunk
    (257, 1560, 5, 24, "rtn"),              # groups that straddle tiles
    (130, 5160, 4, 1720, "greedy"),         # groups longer than a tile
    (90, 2568, 6, 0, "greedy_z"),           # row-wise scales on an odd number of chunks
    (16, 262152, 1, 8, "greedy"),           # K groups of several tiles, the last of one chunk
    (40, 262152, 2, 8, "rtn"),
    # more items in a row range than LDS holds (no "rtn": some of 440,000 ranges of 8 weights are so narrow
    # that a 255th of them is a subnormal fp16, whose planes' scales are no exact doublings)
    (220000, 16, 8, 8, "greedy_z"),
    (220000, 8, 8, 8, "greedy"),
]


@pytest.mark.parametrize("m,n,q,g,mode", CASES)
def test_edges_match_oracle(m, n, q, g, mode):
    print(f"case chunk m={m} n={n} q={q} g={g} mode={mode}", flush=True)
    kg, tpg, rs = lutgemm_plan_grid(m, n, q, g, 1, 256)
    if n > 100000:
        assert tpg > 1                      # (else the case would not cover what it is for)
    if m > 100000:
        assert (m // 16) // rs * (q + (mode != "greedy")) > 400
    W = synth.weights_fp16(m, n, seed=17000 + m + 7 * n + q)
    x = synth.activations_fp16(n, seed=17500 + m + n, batch=1)
    p = Packed.from_weights(W, q, g, MODES[mode])
    gg = n if g == 0 else g
    z = None if p.z is None else O.decode_z(p.z, m, n // gg)
    bound = row_l1_bound(O.decode_alpha(p.alpha, m, n // gg, q), z, gg)
    y_ref, _ = c_oracle.gemv_packed(p.bits, p.alpha, p.z, x, m, n, q, g)
    y = run(p, x, f32_out=True)
    check_parity(np.ravel(y), np.ravel(y_ref), x[0], bound, f32_out=True)
    np.testing.assert_array_equal(run(p, x, f32_out=True), y)        # bitwise reproducible
    if mode == "rtn":
        p.share()
        np.testing.assert_array_equal(run(p, x, f32_out=True, shared=True), y)
