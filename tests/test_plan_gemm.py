"""CPU-side checks of what lutgemm_gemm and lutgemm_gemv_group say that they launch (lutgemm_plan_gemm,
lutgemm_plan_group): the kernel a call gets, and that every planned grid covers the layer within the workspace and
the LDS it was sized for."""
import random
import time

import pytest

import paper_2206_09557_amd as L

FP4, FP16 = L.LUTGEMM_KERNEL_FP4, L.LUTGEMM_KERNEL_FP16
LDS = 160 * 1024


# Layers that the fp16 operands are faster on, and others of about their size that they are not.
@pytest.mark.parametrize("m,n,q,g,z,batch,kernel", [
    (12288, 49152, 3, 128, False, 16, FP16), (12288, 49152, 3, 128, False, 8, FP4),
    (12914, 37248, 3, 0, True, 16, FP16), (12914, 37248, 3, 0, True, 9, FP4),
    (8192, 22016, 4, 128, False, 16, FP4), (12288, 12288, 3, 128, False, 16, FP4),
    (704, 704, 4, 0, False, 12, FP16), (15466, 1024, 4, 128, False, 12, FP4),
    (1363, 320, 2, 0, False, 5, FP16), (720, 512, 3, 128, True, 5, FP4), (15263, 512, 4, 128, False, 5, FP4),
    (813, 640, 3, 0, True, 5, FP16), (107, 768, 5, 256, False, 8, FP4),
    (1607, 576, 4, 64, False, 8, FP16), (8192, 22016, 2, 64, False, 8, FP4),
    (2843, 4352, 2, 256, False, 12, FP16), (22812, 6144, 2, 256, False, 12, FP4),
    (100000, 16384, 3, 128, False, 16, FP4),     # (too tall for the fp16 kernel, which would refuse it)
    (131, 31232, 3, 512, False, 13, FP16), (837, 42752, 3, 128, True, 13, FP4),
    (8192, 8192, 6, 128, True, 16, FP4), (8192, 8192, 7, 128, True, 16, FP16),
    (49152, 12288, 3, 128, False, 32, FP16),
])
def test_matrix_core_path_takes_the_faster_kernel(m, n, q, g, z, batch, kernel):
    plan = L.lutgemm_plan_gemm(m, n, q, g, z, batch, L.LUTGEMM_PATH_AUTO, 256)
    assert [(p[0], p[1]) for p in plan] == [(kernel, batch)]


def test_kernels_of_a_batch():
    def kernels(m, n, q, g, batch, flags=0):
        return [p[:2] for p in L.lutgemm_plan_gemm(m, n, q, g, True, batch, flags, 256)]
    assert kernels(4096, 4096, 3, 128, 1) == [(1, 1)]
    assert kernels(4096, 4096, 3, 32, 7) == [(4, 4), (4, 3)]
    assert kernels(4096, 4096, 3, 32, 10) == [(4, 4), (4, 4), (2, 2)]
    assert kernels(4096, 4096, 7, 128, 5) == [(4, 4), (1, 1)]
    assert kernels(4096, 4096, 3, 64, 4) == [(4, 4)]
    assert kernels(4096, 4096, 3, 64, 13) == [(FP4, 8), (FP4, 5)]
    assert kernels(4096, 4096, 3, 128, 19) == [(FP4, 16), (FP4, 3)]
    assert kernels(4096, 4096, 3, 128, 8, L.LUTGEMM_ALPHA_SHARED | L.LUTGEMM_PATH_AUTO) == [(FP4, 8)]


def test_plans_cover_the_layer_within_workspace_and_lds():
    rng = random.Random(5)
    for _ in range(6000):
        q, g = rng.randint(1, 8), rng.choice([0, 0, 8, 32, 64, 128, 128, 256, 192])
        m = int(2 ** rng.uniform(0, 18))
        unit = g or 8
        n = unit * max(1, int(2 ** rng.uniform(3, 16.5) / unit))
        batch, z, flags = rng.randint(1, 32), rng.random() < 0.5, rng.choice([0, L.LUTGEMM_PATH_AUTO])
        plan = L.lutgemm_plan_gemm(m, n, q, g, z, batch, flags, 256)
        assert sum(p[1] for p in plan) == batch
        steps, tiles, blocks = -(-n // 128), -(-n // 1024), -(-m // 16)
        rows = 16 * (blocks + blocks % 2)
        for kernel, vectors, kg, per_group, ranges, run, stretch in plan:
            assert kg >= 1 and 1 <= ranges
            whole = {1: tiles, FP16: tiles, FP4: steps, 4: 4 * tiles}.get(kernel)
            if whole:
                assert kg * per_group >= whole > (kg - 1) * per_group
            if kernel == FP16 and kg > 1 and ranges > 256:    # refused (too tall for its arrival counters): no other way here
                assert m > 49152 and [p[0] for p in L.lutgemm_plan_gemm(m, n, q, g, z, batch, 0, 256)] != [FP4]
            elif kg > 1:
                assert ranges <= 256
                # the partial sums of the call's vectors lie behind one another in every K group
                assert 32768 + kg * batch * rows * 4 <= L.lutgemm_workspace_bytes(m, n, q, g, 8, batch)
            if kernel == FP4:
                units = -(-(-(-blocks // 4)) // ranges)
                items = -(-per_group // run)
                assert 1 <= run <= 12 and 1 <= stretch <= units
                lds = 96 + per_group * (vectors * 592 + 16) + (stretch * items * vectors * 256 if items > 1 else 0)
                assert lds <= LDS
                assert items > 1 or stretch == units


def test_plan_group_shares_one_round():
    alone = [L.lutgemm_plan_grid(5120, 5120, 4, 128, 1, 256)] * 3
    assert sum(kg * rs for kg, _, rs in alone) > 256
    shared = L.lutgemm_plan_group([(5120, 5120)] * 3, 4, 128, 256)
    assert [kg for kg, _ in shared] == [kg for kg, _, _ in alone]     # (the same sums)
    assert 200 < sum(kg * rs for kg, rs in shared) <= 256
    # one round already: every layer as it would be alone
    few = [(1024, 1024), (2048, 1024)]
    assert [(kg, rs) for kg, rs in L.lutgemm_plan_group(few, 3, 128, 256)] == \
        [L.lutgemm_plan_grid(m, n, 3, 128, 1, 256)[::2] for m, n in few]


# The fp16 kernel's offsets reach 2^30 activations.  What is left of a batch beyond them after some lookups would fit, but
# the kernel is launched for whole batches.
@pytest.mark.parametrize("q,g", [(3, 96), (7, 192), (5, 192)])
def test_batches_beyond_the_offsets_of_the_fp16_kernel(q, g):
    n = g * (2 ** 26 // g)
    assert [p[:2] for p in L.lutgemm_plan_gemm(16, n, q, g, False, 15, 0, 256)] == [(FP16, 15)]
    plan = L.lutgemm_plan_gemm(16, n, q, g, False, 17, 0, 256)
    assert sum(p[1] for p in plan) == 17 and FP16 not in [p[0] for p in plan]


def test_chains_of_the_fp16_kernel_are_bounded():
    # Additions of a wavefront one after the other in fp32, whose number the error grows with: one per plane and offset and
    # scale group of a K step, over the K tiles of a chain.  Within a tile they are what they are.
    rng = random.Random(6)
    seen = {True: 0, False: 0}
    for _ in range(6000):
        q, g, z = rng.randint(1, 8), rng.choice([0, 32, 32, 64, 64, 96, 128, 192, 256, 1024, 2048]), rng.random() < 0.5
        m = int(2 ** rng.uniform(5, 16))
        unit = g or 64
        n = unit * max(1, int(2 ** rng.uniform(6, 16) / unit))
        gg = g or n
        batch, auto = rng.randint(5, 32), rng.random() < 0.4
        for kernel, _, _, tiles, _, chain, rows in L.lutgemm_plan_gemm(m, n, q, g, z, batch, L.LUTGEMM_PATH_AUTO if auto else 0, 256):
            matrix = auto and gg % 64 == 0 and (batch >= 6 or (batch == 5 and m * n < 1 << 28))
            if kernel != FP16 or (matrix and batch <= 16 and chain == 0):      # (expanded from a table)
                continue
            per_step = 1 if gg == n or gg % 128 == 0 else 2 if gg % 64 == 0 else 4
            most = 32 if z and n > 4096 else 24 if n > 4096 else 16
            if matrix:
                most = 24 if gg >= 1024 else 48
            elif per_step == 1 and q <= 6:
                most = 16
            elif per_step == 2 and q <= 4:
                most = 12
            additions = per_step * (q + z)
            assert 1 <= chain <= tiles and (chain == 1 or chain * additions <= most), (m, n, q, g, z, batch, auto)
            assert rows >= 1 and (chain == tiles or rows <= 2)                 # (whose sums LDS has room for)
            seen[chain < tiles] += 1
    assert min(seen.values()) > 200


@pytest.mark.parametrize("m,n,q,g", [(3001, 5160, 5, 24), (8192, 8200, 3, 8), (3001, 5160, 5, 40), (4096, 528, 2, 24)])
def test_grid_of_one_vector_is_the_one_launched(m, n, q, g):
    # Groups with a scale set per chunk: the choice looks at the row length.
    launched, = L.lutgemm_plan_gemm(m, n, q, g, True, 1, 0, 256)
    for other in (8, 512, 520, 1 << 20):      # (whatever an earlier call has left on the stack)
        L.lutgemm_plan_group([(16, other)] * 8, q, 8, 256)
        L.lutgemm_plan_gemm(16, other, 1, 0, False, 1, 0, 256)
        assert L.lutgemm_plan_grid(m, n, q, g, 1, 256) == launched[2:5]


def test_long_rows_are_planned_in_no_time():
    # The grid of the fp16 kernel is chosen anew for every call: with every K group count looked at, 2^15 K tiles took 120 times
    # as long as eight, 150 us, more than the launch.
    def best(n):
        times = []
        for _ in range(30):
            start = time.perf_counter()
            plan = L.lutgemm_plan_gemm(16, n, 3, 32, False, 8, 0, 256)
            times.append(time.perf_counter() - start)
            assert plan[0][0] == FP16
        return min(times)
    assert best(1 << 25) < 8 * best(1 << 13)


@pytest.mark.parametrize("m,n,q,z,least", [(8192, 8192, 3, True, 9), (24576, 8192, 3, False, 10), (36864, 12288, 2, True, 10),
                                           (36864, 12288, 1, True, 11), (20480, 5120, 1, True, 11), (20480, 5120, 1, False, 9)])
def test_one_or_two_vectors_beyond_eight(m, n, q, z, least):
    # Groups of 64 columns: on large layers eight vectors as 4-bit floats and one or two by lookups are the faster way.
    for batch in range(9, 13):
        kernels = [p[0] for p in L.lutgemm_plan_gemm(m, n, q, 64, z, batch, 0, 256)]
        assert (kernels == [FP16]) == (batch >= least) and (kernels[0] == FP4) == (batch < least)
