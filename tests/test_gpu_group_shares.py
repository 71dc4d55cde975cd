"""A group launch whose layers together are more than one round of workgroups deals one round out to
them: the outputs stay those of separate launches, bit for bit, and match the oracle, where the
shares are even, where a layer is too small or too large for its share, where a layer cannot
give up a row range, and for the most layers a group takes."""
import pytest

import paper_2206_09557_amd as L
from paper_2206_09557_amd import synth
from paper_2206_09557_amd.lutgemm import lutgemm_plan_grid

from gpu_util import Packed
from test_gpu_decoder_block import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes,q,g,mode", [
    ([(2800, 4096)] * 3, 2, 128, L.LUTGEMM_Q_GREEDY),                                   # even shares
    ([(16, 8192), (30000, 512), (2000, 4096)], 1, 64, L.LUTGEMM_Q_GREEDY),          # a small, a direct and an ordinary layer
    ([(24, 131072), (6000, 3072), (1800, 5120)], 1, 32, L.LUTGEMM_Q_GREEDY_MEAN_OFFSET),  # K groups of several tiles, one range
    ([(2201, 2048)] * 8, 2, 0, L.LUTGEMM_Q_UNIFORM_RTN),                                # eight layers, ragged rows
])
def test_one_round_for_all_layers(shapes, q, g, mode):
    print(f"case group shares shapes={shapes} q={q} g={g} mode={mode}", flush=True)
    planned = [lutgemm_plan_grid(m, n, q, g, 1, 256) for m, n in shapes]
    assert sum(kg * rs for kg, _, rs in planned) > 256
    layers, xs = [], []
    for li, (m, n) in enumerate(shapes):
        layers.append(Packed.from_weights(synth.weights_fp16(m, n, seed=18000 + 17 * li + m), q, g, mode))
        xs.append(synth.activations_fp16(n, seed=18500 + li + n))
    _check(layers, xs, q, g)
