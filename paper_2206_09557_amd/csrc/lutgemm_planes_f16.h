// Batches of up to thirty-two activation vectors with the binary planes on the matrix cores, weights as
// fp16 +-1 (part of lutgemm_device.hip; included there).
//
// What it computes is what the lookup kernels compute, plane by plane and group by group:
// y_r = sum_i alpha_i[r][G] * (B_i . x)_G + z[r][G] * (sum of x over G), with B_i . x on
// v_mfma_f32_32x32x16_f16: products +-x are exact, sums fp32.  Its time hardly depends on the number of vectors
// (the operand has thirty-two rows whatever it is; those beyond the last vector repeat it, and nobody reads what comes of
// them), so it is for batches that the lookups would take in several turns and the 4-bit-float kernel in two launches, or not
// at all; of the matrix-core path, which would else expand keys from a table, from one vector on.
//
// Weights.  A lane has 16 key bytes of a K step (128 columns) and row unit (64 rows) per plane, rows 4k..4k+3 of four
// chunks; a byte transpose and an exchange between lanes 16 apart make words of 32 weights of one row of
// them, so that the 64 rows are two tiles of 32 operand columns.  A shift, of two words in one 64-bit
// instruction, puts one bit of every nibble on its sign bit, an and-or makes +-1 as a 4-bit float of it, and one
// conversion makes two fp16 numbers of a byte of these: 23 vector instructions for 32 weights, where shifting and masking
// fp16 directly takes 31.  Product (w, e) of a step is 16 columns: groups of any multiple of 32 columns need no
// products beyond those of long groups, only more scalings (SB: scale groups per step).
//
// Work split.  A workgroup owns a row range and a K group.  It walks a row range in passes of T row units per wavefront:
// a pass goes through the K tiles of the group, each wavefront with one of a tile's eight K steps, and keeps its sums in
// registers, a chain of fp32 additions; at its end the wavefronts' sums are added through LDS, in their order and in 64 bits.
// Where a K group would be too long a chain for the error that its calls had before (the rule: F16Tiles), there are several,
// and their sums stay in LDS, in 64 bits.  Sums between
// K groups, where there are several, are the only ones that go through memory.  The activations of a tile come
// by way of the registers into one half of LDS while the other half is in use: one barrier per tile.  A plane's keys and scales
// give way to those of the next unit as soon as they are used up.  A pass of several row units shares the
// activations' turn and the barrier, as many as the accumulators leave registers for (f16_most_tall; several chains: two).
//
// What bounds it (MI355X, 49152 x 12288, q = 3, g = 128, 32 vectors, weights in no cache): 109 us (1.06 PFLOP/s; 108 to 116 on several devices), where the
// kernel before (+-1 from a table in LDS, half the vectors per product) took 167.  3456 matrix instructions per SIMD, 32
// cycles each, are 46 us at full clock; 9 vector instructions to each of them, four of these conversions, take 40 cycles
// of issue, of which the matrix instruction hides 24 or so.  The device also lowers its clock under this load: with
// weights and activations of zeros the same launch takes 84 us.  The products and the vector instructions that feed them are
// interleaved by hand, one product to a group of eight (left to the compiler: 116).  One row unit per pass 119,
// K groups of half the columns 115.
// Error against 64-bit sums (2-norm; N(0, 1) activations, one in 1024 columns ten to thirty times larger): 0.4 to 1.2e-7 over 246 drawn
// layers of all routes.
#pragma once

typedef _Float16 f16x8v __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef int i32x4w __attribute__((ext_vector_type(4)));

struct F16Params : Fp4Params {   // SPG: K steps of a K group, whole K tiles
  int blocks_per_group;          // blocks of 128 / SB columns in a scale group
  int group_step, block_step;    // scale groups, and blocks beyond them, of a K tile
  int tall;                      // row units of a wavefront's pass (the kernel's T)
  int waves_k_shift;             // log2 of the wavefronts among which the K steps of a row unit are dealt out: all eight, or,
                                 // where a K group has fewer steps, that many
  uint32_t set_magic;            // number / (16 * vectors) of up to 8 * 16 * vectors numbers: the upper half of their product with it
  int chain;                     // K tiles that a wavefront adds up one after the other in fp32 (several chains: T < 3)
};

constexpr int kF16Waves = 8;
constexpr int kF16StepBytes = 8192;                            // 32 vectors x 128 columns
constexpr int kF16StageBytes = kF16Waves * kF16StepBytes;      // a K tile, one step per wavefront
constexpr int kF16PartBytes = 32 * kFp4UnitRows * 4;           // a wavefront's sums of a row unit
static_assert(kF16Waves * kF16PartBytes <= kF16StageBytes, "the sums take the place of a tile's activations");
constexpr int kF16LdsBytes = 2 * kF16StageBytes;
constexpr int kF16RunningBytes = 32 * kFp4UnitRows * 8;        // ... and behind these, of a row unit, the 64-bit sums of its chains so far

// Keys, scales and offsets of a unit (row unit, K step) as a lane has them.
template <int Q, int ZM, int SB>
struct F16Unit {
  static constexpr int QA = ZM == 2 ? 1 : Q;
  u32x4 w[Q];
  u32x2 al[SB][QA];
  u32x2 zz[SB];
};

// Where a wavefront is: row unit, K tile of the K group, and the scale group of its K step.
struct F16Place {
  int ru, stage, group, block;   // ru: first of the T row units of a pass
};

// The lane's number, formed anew.
__device__ __forceinline__ int f16_lane_number() {
  int zero = 0;
  asm volatile("" : "+v"(zero));
  return (int)__builtin_amdgcn_mbcnt_hi(0xffffffffu, __builtin_amdgcn_mbcnt_lo(0xffffffffu, (uint32_t)zero));
}

// What a lane knows about its place.  Loads: lane = 32 s + 16 j + 4 r + k holds rows 4k..4k+3 of row block r, four
// chunks.  Products: lane = 32 h + column; columns are the rows of weights with bit 4 the parity of the row.
template <int SB>
struct F16Lane {
  int r, k, j, s;
  uint32_t key_off2, key_off1;    // the lane's 16 key bytes within a K step of a two- / one-sub-slab tile
  uint32_t sel_even, sel_odd;     // byte selectors of the second transpose step
};

template <int SB>
__device__ __forceinline__ F16Lane<SB> f16_lane(int lane) {
  F16Lane<SB> L;
  L.k = lane & 3;
  L.r = (lane >> 2) & 3;
  L.j = (lane >> 4) & 1;
  L.s = lane >> 5;
  const int sub = SB == 4 ? L.j : L.s, quad = SB == 4 ? L.s : L.j;
  L.key_off2 = (uint32_t)(sub * 1024 + (quad * 4 + L.k) * 16);
  L.key_off1 = (uint32_t)(((2 * L.j + L.s) * 4 + L.k) * 16);
  L.sel_even = 0;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const uint32_t s = (uint32_t)(c - L.k) & 3u;
    L.sel_even |= ((s & 2u ? 4u : 0u) + (s & 1u)) << (8 * c);
  }
  L.sel_odd = L.sel_even + 0x02020202u;
  return L;
}

// Addresses of a unit's keys, scales and offsets: a uniform part and the lane's.
template <int Q, int ZM, int SB>
struct F16Source {
  const uint8_t* keys;
  const char* alpha[SB];
  const char* z[SB];
  uint32_t key_off, alpha_off, z_off;
  int slab_row;
};

template <int Q, int ZM, int SB>
__device__ __forceinline__ F16Source<Q, ZM, SB> f16_source(const F16Params& p, const F16Lane<SB>& L, int step0, int wk, int ru, const F16Place& at) {
  F16Source<Q, ZM, SB> src;
  const int step = min(step0 + at.stage * kF16Waves + wk, p.steps - 1);
  const bool one = fp4_one_slab(p, step);
  src.slab_row = one ? 1024 : 2048;
  const int r_use = min(L.r, p.RB - 1 - 4 * ru);    // blocks past the end repeat the last one (their rows are never stored)
  src.key_off = (uint32_t)(r_use * Q * src.slab_row) + (one ? L.key_off1 : L.key_off2);
  src.keys = p.bits + (int64_t)(step >> 3) * p.RB * (Q * 2048) + (int64_t)ru * (4 * Q * src.slab_row) + (step & 7) * (one ? 256 : 128);
  const uint32_t row = (uint32_t)(r_use * p.NG);
  src.alpha_off = ZM == 2 ? row * 32u + L.k * 8u : row * (32u * Q) + L.k * (8u * Q);
  src.z_off = row * 32u + L.k * 8u;
#pragma unroll
  for (int s = 0; s < SB; ++s) {
    int g = at.group;
    if (SB > 1) g += p.blocks_per_group == 1 ? s : (at.block + s >= p.blocks_per_group ? 1 : 0);
    const int64_t pair = (int64_t)ru * 4 * p.NG + min(g, p.NG - 1);
    src.alpha[s] = reinterpret_cast<const char*>(p.alpha) + pair * (ZM == 2 ? 32 : 32 * Q);
    src.z[s] = reinterpret_cast<const char*>(p.z) + pair * 32;
  }
  return src;
}

template <int Q, int ZM, int SB>
__device__ __forceinline__ void f16_load_plane(F16Unit<Q, ZM, SB>& u, const F16Source<Q, ZM, SB>& src, int i) {
  u.w[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src.keys + i * src.slab_row + src.key_off));
  if (ZM != 2) {
#pragma unroll
    for (int s = 0; s < SB; ++s) u.al[s][i] = *reinterpret_cast<const u32x2*>(src.alpha[s] + src.alpha_off + i * 8);
  }
}
// What the planes of a unit share.
template <int Q, int ZM, int SB>
__device__ __forceinline__ void f16_load_shared(F16Unit<Q, ZM, SB>& u, const F16Source<Q, ZM, SB>& src) {
#pragma unroll
  for (int s = 0; s < SB; ++s) {
    if (ZM == 2) u.al[s][0] = *reinterpret_cast<const u32x2*>(src.alpha[s] + src.alpha_off);
    if (ZM != 0) u.zz[s] = *reinterpret_cast<const u32x2*>(src.z[s] + src.z_off);
  }
}

// Chunk of a K step that stands at product (region w, byte e) and half of K.
template <int SB>
__device__ __forceinline__ int f16_chunk(bool one, int w, int e, int half) {
  if (!one) return 8 * w + 2 * e + half;
  return SB == 4 ? 4 * (2 * w + (e >> 1)) + 2 * half + (e & 1) : 4 * (2 * w + half) + e;
}

// Byte e (a constant) of the four fp4 words of a row as eight fp16 numbers.
__device__ __forceinline__ f16x8v f16_weights(const uint32_t (&f4)[4], int e) {
  i32x4w b;
#pragma unroll
  for (int beta = 0; beta < 4; ++beta) {
    h16x2 h;
    if (e == 0) h = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(f4[beta], 1.0f, 0);
    if (e == 1) h = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(f4[beta], 1.0f, 1);
    if (e == 2) h = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(f4[beta], 1.0f, 2);
    if (e == 3) h = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(f4[beta], 1.0f, 3);
    b[beta] = __builtin_bit_cast(int, h);
  }
  return __builtin_bit_cast(f16x8v, b);
}

__device__ __forceinline__ void f16_swap16(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
__device__ __forceinline__ void f16_swap32(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}

template <int Q, int ZM, int SB, int T>
__global__ __launch_bounds__(kF16Waves * 64) void lutgemm_f16_kernel(F16Params p) {
  extern __shared__ __align__(16) char lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int kg = blockIdx.x, rs = blockIdx.y;
  const int step0 = kg * p.SPG, steps = min(p.SPG, p.steps - step0), stages = (steps + kF16Waves - 1) / kF16Waves;
  const int range0 = rs * p.range_base + min(rs, p.range_rem), range_units = p.range_base + (rs < p.range_rem ? 1 : 0);
  const int waves_k = 1 << p.waves_k_shift, wk = wave & (waves_k - 1), sets = kF16Waves >> p.waves_k_shift;
  const int pass_units = T * sets;
  const F16Lane<SB> L = f16_lane<SB>(lane);

  // ---- activations of a stage, one K tile, by way of the registers: a wavefront takes four vectors' part of every K
  // step, a lane one chunk of them.  A step lies in LDS as [product][half of K][vector]; the vectors of a piece of 512
  // bytes are exchanged by its number so that neither side meets in a bank.  Rows beyond the last vector repeat it.  Columns
  // beyond the last are the next vector's first ones, or, of the last vector, zeros (the buffer's bound holds for the whole offset, the
  // scalar part included): stage_body puts zeros in the place of either.
  const int xc = lane & 15, xvec = 4 * wave + (lane >> 4);
  const __amdgpu_buffer_rsrc_t xrsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<__half*>(p.x), 0, (int)((int64_t)p.vectors * p.n * 2), 0x00027000);
  const int x_off = (int)(((int64_t)min(xvec, p.vectors - 1) * p.n + xc * 8) * 2);
  auto fetch_x = [&](int stage, int i) {
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(xrsrc, x_off + i * 256, (step0 + stage * kF16Waves) * 256, 0));
  };
  auto place_x = [&](int stage, int turn) {   // of the first K step
    int piece = xc;
    if (fp4_one_slab(p, step0 + stage * kF16Waves))
      piece = SB == 4 ? (xc & 12) | (xc & 1) << 1 | (xc >> 1 & 1) : (xc & 8) | (xc & 3) << 1 | (xc >> 2 & 1);
    return (turn & 1) * kF16StageBytes + piece * 512 + ((xvec ^ piece) << 4);
  };
  auto store_x = [&](int at, int i, u32x4 x) {
    asm volatile("" : "+v"(x));   // (not to be waited for ahead of this)
    const u32x4 y = {__builtin_amdgcn_perm(x[2], x[0], 0x05040100u), __builtin_amdgcn_perm(x[2], x[0], 0x07060302u),
                     __builtin_amdgcn_perm(x[3], x[1], 0x05040100u), __builtin_amdgcn_perm(x[3], x[1], 0x07060302u)};
    *reinterpret_cast<u32x4*>(lds + at + i * kF16StepBytes) = y;
  };
  u32x4 xr[kF16Waves];
#pragma unroll
  for (int i = 0; i < kF16Waves; ++i) xr[i] = fetch_x(0, i);
  {
    const int to = place_x(0, 0);
#pragma unroll
    for (int i = 0; i < kF16Waves; ++i) store_x(to, i, xr[i]);
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---- the order of a workgroup's units: K tiles of a row unit, row unit after row unit
  const int first_block = (step0 + wk) * SB, first_group = first_block / p.blocks_per_group;
  const F16Place first = {range0, 0, first_group, first_block - first_group * p.blocks_per_group};
  auto advance = [&](F16Place& at) {
    if (at.stage + 1 < stages) {
      ++at.stage;
      at.group += p.group_step;
      at.block += p.block_step;
      if (at.block >= p.blocks_per_group) {
        at.block -= p.blocks_per_group;
        ++at.group;
      }
    } else {
      const int ru = at.ru + pass_units;
      at = first;
      at.ru = ru;
    }
  };
  // (Past the end of the range its last row unit again: the loads are unconditional.)
  auto source = [&](const F16Place& at, int t) {
    return f16_source<Q, ZM, SB>(p, L, step0, wk, min(at.ru + (wave >> p.waves_k_shift) * T + t, range0 + range_units - 1), at);
  };
  F16Place here = first, ahead = first;   // of the current stage and the next
  advance(ahead);
  F16Unit<Q, ZM, SB> u;
  {
    const F16Source<Q, ZM, SB> src = source(here, 0);
    __builtin_amdgcn_sched_barrier(0);
    f16_load_shared(u, src);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      __builtin_amdgcn_sched_barrier(0);   // (in the order of the loop, which the waits there count on)
      f16_load_plane(u, src, i);
    }
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---- key words of the next (plane, tile of 32 rows), made in pieces among the products of the current one
  const Fp4Weights kw = fp4_weights();
  const uint32_t al_shift = L.j ? 16u : 0u;
  uint32_t w0 = 0, w1 = 0, half_a = 0, half_b = 0;
  uint64_t next_words[4];
  auto select_halves = [&](bool one) {   // of the words that the two halves of the lanes exchange where SB == 4
    half_a = one ? 0x05040100u : 0x03020100u;
    half_b = one ? 0x07060302u : 0x07060504u;
  };
  auto expand_rows = [&](const u32x4& d, int tile) {
    const uint32_t x01 = __builtin_amdgcn_perm(d[1], d[0], tile ? 0x07030602u : 0x05010400u);
    const uint32_t x23 = __builtin_amdgcn_perm(d[3], d[2], tile ? 0x07030602u : 0x05010400u);
    w0 = __builtin_amdgcn_perm(x23, x01, L.sel_even);
    w1 = __builtin_amdgcn_perm(x23, x01, L.sel_odd);
  };
  auto expand_swap = [&]() {
    f16_swap16(w0, w1);
    if (SB == 4) {
      uint32_t p0 = __builtin_amdgcn_perm(w1, w0, half_a), p1 = __builtin_amdgcn_perm(w1, w0, half_b);
      f16_swap32(p0, p1);
      w0 = __builtin_amdgcn_perm(p1, p0, half_a);
      w1 = __builtin_amdgcn_perm(p1, p0, half_b);
    }
  };
  auto expand_bits = [&](int beta) {   // (what a shift of both words carries across stays clear of the sign bits)
    const uint64_t w = ((uint64_t)w1 << 32) | w0;
    uint64_t v = w;
    if (beta == 0) asm("v_lshlrev_b64 %0, 3, %1" : "=v"(v) : "v"(w));
    if (beta == 1) asm("v_lshlrev_b64 %0, 2, %1" : "=v"(v) : "v"(w));
    if (beta == 2) asm("v_lshlrev_b64 %0, 1, %1" : "=v"(v) : "v"(w));
    next_words[beta] = ((uint64_t)((((uint32_t)(v >> 32)) & kw.sign) | kw.one) << 32) | ((((uint32_t)v) & kw.sign) | kw.one);
  };
  auto operand = [&](const uint64_t (&words)[4], int w, int e) {
    uint32_t f4[4];
#pragma unroll
    for (int beta = 0; beta < 4; ++beta) f4[beta] = (uint32_t)(words[beta] >> (32 * w));
    return f16_weights(f4, e);
  };
  select_halves(fp4_one_slab(p, step0));
  expand_rows(u.w[0], 0);
  expand_swap();
#pragma unroll
  for (int beta = 0; beta < 4; ++beta) expand_bits(beta);
  f16x8v bnext = operand(next_words, 0, 0);

  f32x16 acc[T][2];
#pragma unroll
  for (int t = 0; t < T; ++t) acc[t][0] = acc[t][1] = f32x16{};
  f32x16 pend = {};       // sums of the last segment of products, and their scale
  float pend_al = 0.0f;

  // One unit: `u`, whose place is taken by the unit at `ahead`, plane after plane as it is used up.  turn: number of
  // the stage among all that the workgroup goes through.
  int turn = 0;
  auto stage_body = [&](int stage) {
    __syncthreads();
    const int x_stage = stage + 1 < stages ? stage + 1 : 0;
    const int x_to = place_x(x_stage, turn + 1);
    const int local = stage * kF16Waves + wk;
    // A scale or offset counts where its segment of the K step has columns: behind the last one sums are zero, which an
    // infinity would turn into a NaN.
    int scale_bits[SB];
#pragma unroll
    for (int s = 0; s < SB; ++s) scale_bits[s] = 16 * (step0 + local) + s * (16 / SB) < p.nchunks ? 16 : 0;
    f16x8v a[2][4];
    {
      const char* xs = lds + (turn & 1) * kF16StageBytes + wk * kF16StepBytes + L.s * 512;
#pragma unroll
      for (int b = 0; b < 8; ++b) a[b >> 2][b & 3] = *reinterpret_cast<const f16x8v*>(xs + b * 1024 + (((lane & 31) ^ (2 * b + L.s)) << 4));
      if (step0 + local >= p.steps - 1) {   // no columns beyond the last
        const int left = p.nchunks - 16 * (step0 + local);
        const bool one = fp4_one_slab(p, min(step0 + local, p.steps - 1));
#pragma unroll
        for (int b = 0; b < 8; ++b)
          if (f16_chunk<SB>(one, b >> 2, b & 3, L.s) >= left) a[b >> 2][b & 3] = f16x8v{};
      }
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const F16Source<Q, ZM, SB> src = t + 1 < T ? source(here, t + 1) : source(ahead, 0);
      __builtin_amdgcn_sched_barrier(0);
      uint32_t al[2][SB];   // scale of the lane's row in either tile (its 16 bits)
      auto take_scales = [&](int i) {
#pragma unroll
        for (int s = 0; s < SB; ++s) {
          al[0][s] = __builtin_amdgcn_ubfe(u.al[s][i].x, al_shift, scale_bits[s]);
          al[1][s] = __builtin_amdgcn_ubfe(u.al[s][i].y, al_shift, scale_bits[s]);
          asm volatile("" : "+v"(al[0][s]), "+v"(al[1][s]));   // (now: their place is asked for)
        }
      };
      if (ZM != 0) {
        uint32_t zz[2][SB];
#pragma unroll
        for (int s = 0; s < SB; ++s) {
          zz[0][s] = __builtin_amdgcn_ubfe(u.zz[s].x, al_shift, scale_bits[s]);
          zz[1][s] = __builtin_amdgcn_ubfe(u.zz[s].y, al_shift, scale_bits[s]);
          asm volatile("" : "+v"(zz[0][s]), "+v"(zz[1][s]));
        }
        if (ZM == 2) take_scales(0);
        f16_load_shared(u, src);
        const u32x4 ones = {0x3c003c00u, 0x3c003c00u, 0x3c003c00u, 0x3c003c00u};
#pragma unroll
        for (int s = 0; s < SB; ++s) {
          f32x16 sx = {};
#pragma unroll
          for (int b = s * (8 / SB); b < (s + 1) * (8 / SB); ++b)
            sx = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[b >> 2][b & 3], __builtin_bit_cast(f16x8v, ones), sx, 0, 0, 0);
#pragma unroll
          for (int tile = 0; tile < 2; ++tile) {
            const float zf = half_lo(zz[tile][s]);
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[t][tile][e] = fmaf(zf, sx[e], acc[t][tile][e]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int it = 0; it < 2 * Q; ++it) {
        __builtin_amdgcn_sched_barrier(0);
        const int i = it >> 1, tile = it & 1;
        uint64_t words[4];
#pragma unroll
        for (int beta = 0; beta < 4; ++beta) words[beta] = next_words[beta];
        if (SB == 4 && it == 2 * Q - 1 && t == T - 1) select_halves(fp4_one_slab(p, step0 + x_stage * kF16Waves));
        f32x16 s = {};
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          constexpr int kSeg = 8 / SB;       // products of a segment: those of one scale
          const int sg = b / kSeg, in = b % kSeg;
          const f16x8v bnow = bnext;
          s = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[b >> 2][b & 3], bnow, s, 0, 0, 0);
          bnext = b < 7 ? operand(words, (b + 1) >> 2, (b + 1) & 3) : operand(next_words, 0, 0);
          // the next words; a plane's keys make room for those of the unit ahead
          if (b == 0) {
            expand_rows(tile == 0 ? u.w[i] : u.w[i + 1 < Q ? i + 1 : 0], 1 - tile);
            if (tile == 0) {
              if (ZM != 2) take_scales(i);
              f16_load_plane(u, src, i);
            }
          }
          if (b == 1) expand_swap();
          if (b >= 1 && b <= 4) expand_bits(b - 1);
          // the next stage's activations, spread over this one's products
          if (b == 2 || b == 5) {
            constexpr int kIts = 2 * Q * T, kAhead = kIts < 4 ? kIts - 1 : (T > 1 || SB == 4 ? 2 : 3);
#pragma unroll
            for (int j = 0; j < kF16Waves; ++j) {
              const int from = j * (kIts - kAhead) / kF16Waves, to = from + kAhead;
              if (b == 2 && t * 2 * Q + it == from) xr[j] = fetch_x(x_stage, j);
              if (b == 5 && t * 2 * Q + it == to) store_x(x_to, j, xr[j]);
            }
          }
          // the sums of the segment before this one
          const int to_tile = sg > 0 ? tile : 1 - tile, to_t = sg > 0 || it > 0 ? t : (t > 0 ? t - 1 : T - 1);
          constexpr int kFrom[3][9] = {{0, 0, 0, 2, 4, 7, 10, 13, 16}, {0, 2, 6, 11, 16, 0, 0, 0, 0}, {0, 6, 16, 0, 0, 0, 0, 0, 0}};
          const int q0 = kFrom[SB >> 1][in], q1 = kFrom[SB >> 1][in + 1];
#pragma unroll
          for (int q = 0; q < 16; ++q)
            if (q >= q0 && q < q1) acc[to_t][to_tile][q] = fmaf(-pend_al, pend[q], acc[to_t][to_tile][q]);
          if (in == kSeg - 1) {
            pend = s;
            pend_al = half_lo(al[tile][sg]);
            if (ZM == 2) pend_al *= (float)(1 << i);   // exact: the per-plane layout's scale bit for bit
            s = f32x16{};
          }
          if (in == kSeg - 1) asm volatile("" : "+v"(acc[to_t][to_tile]));   // (the additions stay here: the compiler would put them off, and spill)
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    asm volatile("" : "+v"(bnext), "+v"(next_words[0]), "+v"(next_words[1]), "+v"(next_words[2]), "+v"(next_words[3]));
    here = ahead;
    advance(ahead);
    ++turn;
  };

  // ---- the end of a chain: the wavefronts' sums of a row unit, in their order, where the last stage's activations
  // were.  Sums of several chains meet in 64 bits, in a place of LDS that only the thread that adds them up knows.
  auto finish_chain = [&](int ru, bool first, bool last) {
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[T - 1][1][q] = fmaf(-pend_al, pend[q], acc[T - 1][1][q]);
    pend_al = 0.0f;
    pend = f32x16{};
    float* part = reinterpret_cast<float*>(lds + ((turn - 1) & 1) * kF16StageBytes);
    const int lane_again = f16_lane_number();   // (nothing of this is to stay in registers over the stages)
    const int tid = wave * 64 + lane_again;
    float* dst = part + wave * (kF16PartBytes / 4) + 4 * (lane_again & 15) + (lane_again >> 4 & 1) + (lane_again >> 5) * (4 * kFp4UnitRows);
#pragma unroll
    for (int t = 0; t < T; ++t) {
      __syncthreads();
#pragma unroll
      for (int tile = 0; tile < 2; ++tile) {
#pragma unroll
        for (int q = 0; q < 16; ++q)
          if (T > 2 || 8 * (q >> 2) < p.vectors) dst[(8 * (q >> 2) + (q & 3)) * kFp4UnitRows + 2 * tile] = acc[t][tile][q];
        acc[t][tile] = f32x16{};
      }
      __syncthreads();
      for (int i = tid; i < sets * p.vectors * 16; i += kF16Waves * 64) {   // (row unit, vector, four rows)
        const int set = (int)__umulhi((uint32_t)i, p.set_magic), vec = (i >> 4) - set * p.vectors, unit = ru + set * T + t;
        const int row = unit * kFp4UnitRows + 4 * (i & 15);
        if (unit >= range0 + range_units) continue;
        const f32x4* src = reinterpret_cast<const f32x4*>(part + (set << p.waves_k_shift) * (kF16PartBytes / 4) + vec * kFp4UnitRows) + (i & 15);
        f32x4 q[kF16Waves];
#pragma unroll
        for (int k = 0; k < kF16Waves; ++k) q[k] = src[min(k, waves_k - 1) * (kF16PartBytes / 16)];
        double sum[4] = {0.0, 0.0, 0.0, 0.0};   // few additions, and the last ones: 64 bits cost nothing here
#pragma unroll
        for (int k = 0; k < kF16Waves; ++k)
          if (k < waves_k) {
#pragma unroll
            for (int b = 0; b < 4; ++b) sum[b] += q[k][b];
          }
        if (T < 3 && !(first && last)) {   // (several K tiles, so one set: i < 512)
          double* running = reinterpret_cast<double*>(lds + kF16LdsBytes + t * kF16RunningBytes) + 4 * i;
          if (!first) {
#pragma unroll
            for (int b = 0; b < 4; ++b) sum[b] += running[b];
          }
          if (!last) {
#pragma unroll
            for (int b = 0; b < 4; ++b) running[b] = sum[b];
            continue;
          }
        }
        const float s[4] = {(float)sum[0], (float)sum[1], (float)sum[2], (float)sum[3]};
        if (p.KG == 1) {
          fp4_store_rows(p, vec, row, s);
        } else if (row < p.vec_stride) {
          float* q = p.partial + kg * p.kg_stride + vec * p.vec_stride + row;
          fp4_store_pair(q, s[0], s[1]);
          fp4_store_pair(q + 2, s[2], s[3]);
        }
      }
    }
  };

#pragma unroll 1
  for (int ru = range0; ru < range0 + range_units; ru += pass_units) {
#pragma unroll 1
    for (int stage = 0; stage < stages;) {
      const int first = stage, end = min(stage + p.chain, stages);
#pragma unroll 1
      for (; stage < end; ++stage) stage_body(stage);
      finish_chain(ru, first == 0, end == stages);
    }
  }
  if (p.KG == 1) return;

  // ---- K groups: the hand-off of finish_row_range.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  int* flag = reinterpret_cast<int*>(lds);
  const int lane_again = f16_lane_number();
  if (wave == 0 && lane_again == 0) {
    const bool all = __hip_atomic_fetch_add(p.counters + rs, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)(p.KG - 1);
    *flag = all ? 1 : 0;
    if (all) __hip_atomic_store(p.counters + rs, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // zero for the next call on this workspace
  }
  __syncthreads();
  if (*flag == 0) return;
  const int quads = (p.vectors + 3) / 4;
  for (int i = wave; i < range_units * quads; i += kF16Waves) {
    const int un = i / quads;
    fp4_add_groups(p, lane_again, range0 + un, i - un * quads);
  }
}
