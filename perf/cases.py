"""The calls that a program using this library makes, as cases that can be timed and checked.

A case is one call of a device entry point: a product of a packed layer with one activation
vector (decode, one sequence), with a small batch of them (decode of several sequences), or
several independent layers at once.  Weights are synthetic: key bytes are uniform (the signs of
a zero-mean weight matrix are), scales are those the greedy quantiser gives N(0, 0.02) weights
(each plane about half the one before, spread by some 10 % from group to group), offsets are
small, and for uniformly quantised weights plane i has 2^i times the scale of plane 0.
Activations are N(0, 1) in fp16 with a few channels ten to thirty times larger, as the hidden
states of large decoders have them.
"""
import math

import torch

import paper_2206_09557_amd as L

MU = 8


def listed():
    # Sizes are the layer shapes of the workload list (1024^2; OPT-13B, OPT-175B and LLaMA-65B
    # linear layers), plus one deliberately ragged layer.
    return [
        # the smallest call: launch and latency, hardly any bytes
        _case("gemv_1024", "gemv", [(1024, 1024)], 3, 128),
        # mid-sized decode step, four planes (OPT-13B attention input projection)
        _case("gemv_13b_qkv", "gemv", [(15360, 5120)], 4, 128),
        # the layers of the headline benchmark: the square one and the largest
        _case("gemv_175b_out", "gemv", [(12288, 12288)], 3, 128),
        _case("gemv_175b_fc1", "gemv", [(49152, 12288)], 3, 128),
        # uniformly quantised, with offsets, small groups, rows that are not whole tiles, fp32 result
        _case("gemv_65b_down_g32", "gemv", [(8192, 22016)], 3, 32, scales="offset", f32=True),
        # the same kind of weights with one stored scale per group
        _case("gemv_65b_qkv_shared", "gemv", [(24576, 8192)], 2, 64, scales="shared"),
        # row-wise scales through the entry point that takes no workspace
        _case("static_65b_out_rowwise", "static", [(8192, 8192)], 4, 0, scales="offset"),
        # nothing divides anything: odd rows, ragged last tile, groups of 24 columns, five planes
        _case("gemv_ragged_g24", "gemv", [(3001, 5160)], 5, 24, scales="offset", f32=True),
        # separately stored Q, K and V projections of one activation vector
        _case("group_13b_q_k_v", "group", [(5120, 5120)] * 3, 4, 128),
        # four sequences decoded together
        _case("gemm4_13b_fc1", "gemm", [(20480, 5120)], 4, 128, batch=4),
        # eight sequences, the library picks the path
        _case("auto8_175b_fc1", "auto", [(49152, 12288)], 3, 128, batch=8),
        # the largest batch the library takes
        _case("auto32_175b_fc1", "auto", [(49152, 12288)], 3, 128, batch=32),
    ]


def _case(name, entry, shapes, q, g, batch=1, scales="planes", f32=False):
    """entry: gemv / static / group (one vector), gemm (lookup path asked for), auto (the library
    picks), mfma (matrix cores asked for).  scales: "planes" (one per plane and group), "offset"
    (the same with offsets), "shared" (one per group, with offsets).  A case holds plain values
    only: the shapes of up to eight layers are written m0, n0, m1, n1, ..."""
    c = {"name": name} if name else {}
    c.update(entry=entry, count=len(shapes), q=q, g=g, batch=batch, scales=scales, f32=f32)
    for i, (m, n) in enumerate(shapes):
        c[f"m{i}"], c[f"n{i}"] = m, n
    return c


def _shapes(case):
    return [(case[f"m{i}"], case[f"n{i}"]) for i in range(case["count"])]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# weights x planes x passes over them: what the largest listed case costs, with a margin
_COST_CAP = 3.0 * 49152 * 12288 * 3


def draw(rng):
    while True:
        entry = rng.choices(["gemv", "static", "group", "gemm", "auto", "mfma"], [8, 1, 2, 4, 4, 1])[0]
        q = rng.choices(range(1, 9), [1, 4, 6, 5, 1, 1, 1, 1])[0]
        scales = rng.choices(["planes", "offset", "shared"], [5, 3, 2])[0]
        g = rng.choices([128, 64, 32, 0, 256, 192, 96, 16, 24, 8, 40], [12, 5, 5, 4, 2, 1, 1, 1, 1, 1, 1])[0]
        batch = 1 if entry in ("gemv", "static", "group") else _log_uniform(rng, 2, 32)
        if entry == "mfma":
            scales = "planes" if scales == "shared" else scales
            g = g if g in (128, 64, 0, 256, 192) else 128
        if entry == "group" and g in (24, 8, 40):     # not offered in a group
            g = 64
        count = rng.randint(2, 6) if entry == "group" else 1
        shapes = []
        for _ in range(count):
            m = _log_uniform(rng, 64, 50000)
            unit = 64 if g == 0 else g
            n = unit * max(1, round(_log_uniform(rng, 256, 50000) / unit))
            if g == 0 and entry not in ("mfma", "group") and rng.random() < 0.5:
                n += 8 * rng.randint(1, 7)            # row-wise scales on a length that no tile divides
            if rng.random() < 0.5:
                m = max(64, m // 16 * 16)
            shapes.append((m, n))
        weights = sum(m * n for m, n in shapes)
        passes = 1.0 if batch == 1 else 1.5 * math.ceil(batch / 4)
        if weights * q * passes > _COST_CAP or weights < 1 << 16:
            continue
        if entry == "static" and L.lutgemm_workspace_bytes(*shapes[0], q, g) > L.lutgemm_static_scratch_bytes():
            continue
        return _case(None, entry, shapes, q, g, batch, scales, rng.random() < 0.4)


# ---- synthetic layers -------------------------------------------------------------------

def _generator(seed, i):
    gen = torch.Generator(device="cuda")
    gen.manual_seed((seed * 1000003 + 7919 * i + 17) % (1 << 62))
    return gen


def _canonical(case, seed, i):
    """keys uint8 [q][m][n/8] (bit j of a byte: sign of column 8c + j), scales fp16 [q][m][n/g],
    offsets fp16 [m][n/g] or None, activations fp16 [batch][n]; from the seed alone."""
    m, n = _shapes(case)[i]
    q = case["q"]
    groups = n // (case["g"] or n)
    gen = _generator(seed, i)
    keys = torch.randint(0, 256, (q, m, n // 8), dtype=torch.uint8, device="cuda", generator=gen)
    spread = 1.0 + 0.1 * torch.randn((q, m, groups), device="cuda", generator=gen).clamp_(-4, 4)
    if case["scales"] == "planes":
        alpha = torch.empty_like(spread)
        for k in range(q):
            alpha[k] = 0.016 * 0.5 ** k * spread[k]
        alpha, z = alpha.half(), None
    else:
        # step of a uniform quantiser over +-3 standard deviations; plane k has 2^(k-1) steps
        step = (0.06 / (2 ** q - 1) * spread[0]).half().float()
        alpha = torch.stack([step * 2.0 ** k for k in range(q)]).half()
        alpha[1:] = torch.stack([alpha[0] * 2.0 ** k for k in range(1, q)]) if q > 1 else alpha[1:]
        z = (0.004 * torch.randn((m, groups), device="cuda", generator=gen)).half()
    x = torch.randn((case["batch"], n), device="cuda", generator=gen)
    loud = torch.randint(0, n, (max(1, n // 1024),), device="cuda", generator=gen)
    x[:, loud] *= 10 + 20 * torch.rand((1, loud.numel()), device="cuda", generator=gen)
    return keys, alpha, z, x.half()


def _pack_keys(keys):
    """The packed key layout that lutgemm.h specifies, on the device."""
    q, m, chunks = keys.shape
    blocks = (m + 15) // 16
    tiles = (chunks + 127) // 128
    parts = []
    last = chunks - 128 * (tiles - 1)
    for first, count, subs, have in ((0, tiles - 1, 2, 128), (tiles - 1, 1, 2 if last > 64 else 1, last)):
        if count == 0:
            continue
        t = torch.zeros((q, blocks * 16, count, subs * 64), dtype=torch.uint8, device=keys.device)
        t[:, :m, :, :have] = keys[:, :, 128 * first:128 * first + count * have].reshape(q, m, count, have)
        # [plane][block][k = row / 4][row % 4][tile][quad][slot of the quad][sub-slab]
        t = t.view(q, blocks, 4, 4, count, 16, 4, subs)
        out = torch.empty((count, blocks, q, subs, 16, 4, 4, 4), dtype=torch.uint8, device=keys.device)
        for k in range(4):      # lane k of a quad keeps slot c in dword (c - k) mod 4
            for c in range(4):
                out[:, :, :, :, :, k, (c - k) % 4, :] = t[:, :, k, :, :, :, c, :].permute(3, 1, 0, 5, 4, 2)
        parts.append(out.reshape(-1))
    return torch.cat(parts)


def _pack_rows(v):
    """fp16 [m][groups] -> [row block][group][16 rows], missing rows 0."""
    m, groups = v.shape
    blocks = (m + 15) // 16
    out = torch.zeros((blocks * 16, groups), dtype=torch.float16, device=v.device)
    out[:m] = v
    return out.view(blocks, 16, groups).permute(0, 2, 1).contiguous().view(-1)


def _pack_alpha(alpha):
    """fp16 [q][m][groups] -> [row block][group][row / 4][plane][row % 4], missing rows 0."""
    q, m, groups = alpha.shape
    blocks = (m + 15) // 16
    out = torch.zeros((q, blocks * 16, groups), dtype=torch.float16, device=alpha.device)
    out[:, :m] = alpha
    return out.view(q, blocks, 4, 4, groups).permute(1, 4, 2, 0, 3).contiguous().view(-1)


def prepare(case, seed):
    q, g, batch, shared = case["q"], case["g"], case["batch"], case["scales"] == "shared"
    shapes = _shapes(case)
    s = {"case": case, "x": [], "bits": [], "alpha": [], "z": [], "y": []}
    s["m"], s["n"] = [m for m, _ in shapes], [n for _, n in shapes]
    for i, (m, n) in enumerate(shapes):
        keys, alpha, z, x = _canonical(case, seed, i)
        s["bits"].append(_pack_keys(keys))
        s["alpha"].append(_pack_rows(alpha[0]) if shared else _pack_alpha(alpha))
        s["z"].append(None if z is None else _pack_rows(z))
        s["x"].append(x if case["entry"] in ("gemm", "auto", "mfma") else x[0])
        s["y"].append(torch.empty((batch, m) if s["x"][i].dim() == 2 else (m,),
                                  dtype=torch.float32 if case["f32"] else torch.float16, device="cuda"))
    s["flags"] = (L.LUTGEMM_Y_F32 if case["f32"] else L.LUTGEMM_Y_F16) | (L.LUTGEMM_ALPHA_SHARED if shared else 0) | \
                 (L.LUTGEMM_PATH_AUTO if case["entry"] == "auto" else 0)
    if case["entry"] == "group":
        s["ws_bytes"] = L.lutgemm_group_workspace_bytes(s["m"], s["n"], q, g)
    else:
        s["ws_bytes"] = L.lutgemm_workspace_bytes(*shapes[0], q, g, MU, batch)
    if case["entry"] != "static":
        s["ws"] = torch.empty(s["ws_bytes"], dtype=torch.uint8, device="cuda")
        L.lutgemm_workspace_init(s["ws"], s["ws_bytes"], torch.cuda.current_stream().cuda_stream)
    return s


def run(s):
    c = s["case"]
    q, g = c["q"], c["g"]
    stream = torch.cuda.current_stream().cuda_stream
    if c["entry"] == "group":
        z = None if s["z"][0] is None else s["z"]
        L.lutgemm_gemv_group(s["x"], s["bits"], s["alpha"], z, s["y"], s["m"], s["n"], q, g, MU, s["flags"], s["ws"],
                             s["ws_bytes"], stream)
        return s["y"]
    x, bits, alpha, z, y, m, n = (s[k][0] for k in ("x", "bits", "alpha", "z", "y", "m", "n"))
    if c["entry"] == "gemv":
        L.lutgemm_gemv(x, bits, alpha, z, y, q, g, MU, m, n, s["flags"], s["ws"], s["ws_bytes"], stream)
    elif c["entry"] == "static":
        L.lutgemm_gemv_static(x, bits, alpha, z, y, q, g, MU, m, n, s["flags"], stream)
    else:
        call = L.lutgemm_gemm_mfma if c["entry"] == "mfma" else L.lutgemm_gemm
        call(x, bits, alpha, z, y, q, g, MU, m, n, c["batch"], s["flags"], s["ws"], s["ws_bytes"], stream)
    return y


def work(case):
    """Packed planes, scales, offsets and activations read once, results written once; two
    operations per weight and activation vector."""
    size = flops = 0
    q, g, b = case["q"], case["g"], case["batch"]
    for m, n in _shapes(case):
        groups = n // (g or n)
        size += m * n * q // 8 + 2 * m * groups * (1 if case["scales"] == "shared" else q)
        size += (0 if case["scales"] == "planes" else 2 * m * groups) + 2 * b * n + (4 if case["f32"] else 2) * b * m
        flops += 2 * m * n * b
    return {"bytes": size, "flops": flops}


def tolerance(case):
    # fp32 result: fp16 inputs, fp32 sums; the paths' sums run in different orders and are up to
    # 2.3e-7 (largest difference 1.8e-6) from the 64-bit result.  fp16 result: one rounding to
    # 11 bits on top, 2.1e-4 and 4.9e-4.
    if case["f32"]:
        return {"rel": 1e-6, "max": 8e-6}
    return {"rel": 5e-4, "max": 1e-3}


def exact(case, seed):
    q, b = case["q"], case["batch"]
    out = []
    bit = torch.arange(8, dtype=torch.uint8, device="cuda")
    for i, (m, n) in enumerate(_shapes(case)):
        keys, alpha, z, x = _canonical(case, seed, i)
        g = case["g"] or n
        x64 = x.double()
        group_sums = x64.view(b, n // g, g).sum(2)
        y = torch.zeros((b, m), dtype=torch.float64, device="cuda")
        step = max(16, (1 << 26) // n)
        for r in range(0, m, step):
            e = min(m, r + step)
            w = torch.zeros((e - r, n // g, g), dtype=torch.float64, device="cuda")
            for k in range(q):
                sign = ((keys[k, r:e, :, None] >> bit) & 1).double().mul_(2).sub_(1).view(e - r, n // g, g)
                w += sign.mul_(alpha[k, r:e, :, None].double())
            y[:, r:e] = x64 @ w.view(e - r, n).t()
            if z is not None:
                y[:, r:e] += group_sums @ z[r:e].double().t()
        out.append(y if case["entry"] in ("gemm", "auto", "mfma") else y[0])
    return out if case["entry"] == "group" else out[0]
