"""A group launch whose layers together are more than one round of workgroups deals one round out to
them: the outputs stay those of separate launches, bit for bit, and match the oracle, where the
shares are even, where a layer is too small or too large for its share, where the layers keep their own
grids because a share would be too uneven, and for the most layers a group takes."""
import pytest

import paper_2206_09557_amd as L
from paper_2206_09557_amd import synth

from gpu_util import Packed
from test_gpu_decoder_block import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes,q,g,mode,dealt", [
    ([(2800, 4096)] * 3, 2, 128, L.LUTGEMM_Q_GREEDY, True),                             # even shares
    ([(16, 8192), (30000, 512), (2000, 4096)], 1, 64, L.LUTGEMM_Q_GREEDY, True),    # a small, a direct and an ordinary layer
    ([(24, 131072), (6000, 3072), (1800, 5120)], 1, 32, L.LUTGEMM_Q_GREEDY_MEAN_OFFSET, False),  # K groups of several tiles, one range
    ([(2201, 2048)] * 8, 2, 0, L.LUTGEMM_Q_UNIFORM_RTN, True),                          # eight layers, ragged rows
])
def test_one_round_for_all_layers(shapes, q, g, mode, dealt):
    print(f"case group shares shapes={shapes} q={q} g={g} mode={mode}", flush=True)
    alone = [L.lutgemm_plan_grid(m, n, q, g, 1)[::2] for m, n in shapes]
    group = L.lutgemm_plan_group(shapes, q, g)
    assert sum(kg * rs for kg, rs in alone) > 256
    assert (sum(kg * rs for kg, rs in group) <= 256) if dealt else (group == alone)
    assert [kg for kg, _ in group] == [kg for kg, _ in alone]
    layers, xs = [], []
    for li, (m, n) in enumerate(shapes):
        layers.append(Packed.from_weights(synth.weights_fp16(m, n, seed=18000 + 17 * li + m), q, g, mode))
        xs.append(synth.activations_fp16(n, seed=18500 + li + n))
    _check(layers, xs, q, g)
