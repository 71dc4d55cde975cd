// Two to sixteen activation vectors with the binary planes on the matrix cores, weights as
// 4-bit floats (part of lutgemm_device.hip; included there).
//
// What it computes is what the lookup kernels compute, plane by plane and group by group:
// y_r = sum_i alpha_i[r][G] * (B_i . x)_G + z[r][G] * (sum of x over G).  B_i . x runs on
// v_mfma_scale_f32_16x16x128_f8f6f4 with the weights +-1 as e2m1 and the activations as six e2m3
// numbers each:
//   * Weights.  A key dword (four chunks of one row after a byte transpose) holds eight weights
//     per bit position modulo 4.  A shift puts that bit of every nibble on its sign bit, one
//     and-or makes +-1 of it: 7 vector instructions for 32 weights.  +-1 in fp16 takes 16 at the
//     least, and the instruction covers 128 columns in the time the fp16 one covers 32.
//   * Activations.  Within the 32 columns that share a block scale of the instruction, x is
//     written as  2^e * sum_d a_d 32^-d  with balanced digits a_d that are multiples of 1/8 in
//     [-2, 2]: exact values of e2m3.  With U the power of two below the block's largest
//     magnitude, six digits end at 2^-28 U: an fp16 activation is exact unless it is more than 2^18
//     times smaller than U, and then it is wrong by at most 2^-29 U, a thirty-second part of
//     what an fp32 sum that holds the largest one resolves.  (Five digits, 2^-24 U, made the error
//     of a product up to twice that of the lookups where a few activations are 2^14 times the others.)
//     The digits of a vector are R rows of the operand, consecutive ones in a row, one instruction
//     each: up to 16 vectors (R = 1) take 6 instructions, up to 8 (R = 2) 3, up to 4 (R = 4, three
//     of the rows) 2.
//   * Sums of digit products of a block are small integers in units of the block scale and
//     exact inside the instruction; blocks whose scales differ by up to 2^14 add exactly (measured).
//     A chain's accumulator loses bits where it meets products that are much larger than it, or so
//     much smaller that the sum takes more than 24 bits: a row's two largest digits, whose sum takes
//     no more while the four block scales of a K step are within 2^7, and the others have chains
//     of their own, which meet in a rounded addition.  Error against 64-bit sums (2-norm,
//     8192 x 8192 to 4096 x 16384, q = 2 to 6, 2 to 16 vectors; N(0, 1) activations alone, with 30
//     times larger ones every 1024 columns, or 2^14 times larger ones every 32): 0.64e-7 to 1.0e-7;
//     six digits in one chain, the smallest first, 2.6e-7 at worst; lookups 0.84e-7 to 1.8e-7, fp16
//     matrix path 1.0e-7 to 3.0e-7.
//     Not taken, three digits (five to eight vectors) in one chain: the largest first 0.62 and 0.66e-7
//     for 0.64 and 0.72 of N(0, 1) activations (2048 x 16384, q = 2 at six vectors; 4096 x 8192, q = 3
//     at eight), but 0.73 and 0.77 for 0.67 and 0.75 with the 2^14 times larger ones; the smallest
//     first 1.84 and 1.56 there.  It would save 3 us of the 67 below.
//
// Work split.  A K step is 128 columns, a row unit four row blocks (64 rows), a unit the two
// together: per plane one 16-byte key load per lane and 4 x 6 / R instructions, number b of the 4
// taking row 4k + b of each of 16 (row block, k) pairs, so that no key has to move between
// lanes.  Where a K step touches SB = 2 scale groups, the 16 rows of the activation operand are
// (vector, group) pairs instead of vectors, each with zeros outside its group's columns.
// A workgroup owns a K group (consecutive K steps, whose activation digits it makes once and
// keeps in LDS) and a row range.  Its wavefronts draw items, a row unit by `run` K steps, from a
// queue.  Where an item is a row unit's whole K group its sums go from the registers to y (or to
// the workspace); else they go to LDS, where the items of a row are added in step order.  K groups
// are added by the last workgroup to arrive for a row range, in group order: the result does
// not depend on who computed what.
//
// What bounds it (MI355X, 49152 x 12288, q = 3, g = 128, weights in no cache; microseconds, before: lookups
// at 4 vectors, fp16 matrix cores beyond): 53 at 4 vectors (before 72), 67 at 8 (113), 102 at 16 (118).
// Up to four vectors mostly the weight stream (255 MB, 38 us at the 6.7 TB/s of a read loop), with
// 2 to 3 us until the digits stand and 2 to 8 for the hand-off around it.  At 16 the matrix and the
// vector units together: 5184 matrix instructions per SIMD (10 to 11 ns each with random operands, 7.4
// with zeros: 54 us) and 24,500 vector instructions, on two wavefronts that hide the one
// behind the other only in part; the hand-off, 3 MB of partial sums per K group, is most of the
// rest.  The second chain is 3 us of the 67, the sixth digit about 1 by difference; both are 9 of the 102.  Eight wavefronts at
// 256 registers: with twelve or sixteen the accumulators spill or it measured slower; both
// chains of a plane in flight together measured equal.
#pragma once

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2v __attribute__((ext_vector_type(2)));
typedef _Float16 h16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 h16x32 __attribute__((ext_vector_type(32)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));

struct Fp4Params {
  const __half* x;         // [vectors][n]
  const uint8_t* bits;     // packed
  const __half* alpha;     // packed, per plane or shared
  const __half* z;         // packed or null
  void* y;                 // [vectors][m], fp16 or fp32
  float* partial;          // [KG][vectors][vec_stride] when KG > 1
  uint32_t* counters;      // one per row range
  int64_t kg_stride;       // floats between the partials of consecutive K groups
  int64_t vec_stride;      // ... and of consecutive vectors (rows, padded to 32)
  int m, n, RB, NT, NG, g, nchunks;
  int steps;               // K steps of 128 columns
  int KG, SPG;             // K groups and K steps per group
  int run;                 // K steps of an item
  int stretch;             // row units per pass over the K group (bounds the partial sums in LDS)
  int row_splits;          // row ranges
  int range_base, range_rem;   // row units per row range, plus one for the first range_rem
  int vectors;             // at most 16 / (SB * R)
  int y_f32;
};

constexpr int kFp4Digits = 6;
constexpr int kFp4DigitBytes = 24;                        // 32 six-bit digits
constexpr int kFp4RowBytes = 4 * kFp4DigitBytes;          // one digit of a vector's K step: four 32-column blocks
constexpr int kFp4ScalesAt = kFp4Digits * kFp4RowBytes;   // one vector of a K step: the digits, ...
// ... then its four block scales.  592 bytes, 20 banks beyond a multiple of all 64, keep the 16 rows of an
// operand of sixteen vectors in different banks; with 576 (the scales elsewhere) they met in
// four (8192 x 8192, q = 6, 16 vectors 53 us instead of 30).
constexpr int kFp4VecBytes = kFp4ScalesAt + 16;
constexpr int kFp4UnitRows = 64;
// LDS: [24 zero bytes, queue, spare][one word per wavefront][digits and block scales][group numbers]
//      [partial sums: item, vector, row]
constexpr int kFp4FixedBytes = 32 + 64;

__host__ __device__ constexpr int fp4_step_bytes(int vectors) { return vectors * kFp4VecBytes + 16; }

__device__ __forceinline__ f32x4 fp4_mfma(const i32x8& a, const i32x8& b, const f32x4& c, int scale_a) {
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 2 /* A: e2m3 */, 4 /* B: e2m1 */, 0, scale_a, 0, 127);
}

// K steps in a tile of one sub-slab (the last tile of a row when it has at most 64 chunks) keep
// their four 32-column blocks in four quads; in the usual tile of two sub-slabs, in two quads of
// both sub-slabs.
__device__ __forceinline__ bool fp4_one_slab(const Fp4Params& p, int step) {
  const int kt = step >> 3;
  return kt == p.NT - 1 && p.nchunks - 128 * kt <= 64;
}

// Chunk that slot c of 32-column block kb of a K step stands for.
__device__ __forceinline__ int fp4_chunk(int step, bool one, int kb, int c) {
  return 16 * step + (one ? 4 * kb + c : 8 * (kb >> 1) + 2 * c + (kb & 1));
}

// A preparation task: one 32-column block of one vector.
struct Fp4Task {
  u32x4 xs[4];
  int v, local, kb;
};

__device__ __forceinline__ void fp4_fetch_task(Fp4Task& t, const Fp4Params& p, int index, int step0) {
  const int pair = index >> 2;          // (K step, vector)
  t.kb = index & 3;
  t.local = pair / p.vectors;
  t.v = pair - t.local * p.vectors;
  const int step = step0 + t.local;
  const bool one = fp4_one_slab(p, step);
  const u32x4* xv = reinterpret_cast<const u32x4*>(p.x + (int64_t)t.v * p.n);
#pragma unroll
  for (int c = 0; c < 4; ++c) t.xs[c] = xv[min(fp4_chunk(step, one, t.kb, c), p.nchunks - 1)];
}

// Digits of -x (a set key bit is expanded to -1) and block scale of a task into LDS.  Element
// 8 * beta + 2 * c + h of a block is column 4h + beta of its slot c: the order in which fp4_expand
// leaves the weights.  Returns whether the block holds an infinity or NaN; these count as zero
// here, see fp4_overlay_specials.
__device__ __forceinline__ bool fp4_make_digits(Fp4Task& t, const Fp4Params& p, char* lds, int step0, int digits_at) {
  const int step = step0 + t.local;
  const bool one = fp4_one_slab(p, step);
  uint32_t h[16];   // pairs of elements
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    if (fp4_chunk(step, one, t.kb, c) >= p.nchunks) t.xs[c] = u32x4{0u, 0u, 0u, 0u};
    t.xs[c] ^= 0x80008000u;
    h[c] = __builtin_amdgcn_perm(t.xs[c][2], t.xs[c][0], 0x05040100u);
    h[4 + c] = __builtin_amdgcn_perm(t.xs[c][2], t.xs[c][0], 0x07060302u);
    h[8 + c] = __builtin_amdgcn_perm(t.xs[c][3], t.xs[c][1], 0x05040100u);
    h[12 + c] = __builtin_amdgcn_perm(t.xs[c][3], t.xs[c][1], 0x07060302u);
  }
  u16x2 top2 = {0, 0};
#pragma unroll
  for (int e = 0; e < 16; ++e) top2 = __builtin_elementwise_max(top2, __builtin_bit_cast(u16x2, h[e] & 0x7fff7fffu));
  int top = max((int)top2.x, (int)top2.y);
  const bool special = top >= 0x7c00;
  if (special) {
    top = 0;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      if ((h[e] & 0x7c00u) == 0x7c00u) h[e] &= 0xffff0000u;
      if ((h[e] & 0x7c000000u) == 0x7c000000u) h[e] &= 0xffffu;
      top = max(top, max((int)(h[e] & 0x7fffu), (int)(h[e] >> 16 & 0x7fffu)));
    }
  }
  const int exponent = max(top >> 10, 1) + 112;   // biased as in fp32: |x| < 2^(exponent - 126)
  char* vec = lds + digits_at + (t.local * p.vectors + t.v) * kFp4VecBytes;
  *reinterpret_cast<int*>(vec + kFp4ScalesAt + t.kb * 4) = exponent;
  // In the largest binade a first digit of 2 is 2^16, which the remainder's fp16 does not hold: such
  // blocks are split as their halves.  (Lost with it: the last bit of subnormals, 2^-39 of the block's largest.)
  const bool halves = top >= 0x7800;
  if (halves) {
#pragma unroll
    for (int e = 0; e < 16; ++e) h[e] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(h16x2, h[e]) * (_Float16)0.5f);
  }
  const int first_unit = halves ? exponent - 1 : exponent;
  char* dst = vec + t.kb * kFp4DigitBytes;
#pragma unroll
  for (int d = 0; d < kFp4Digits; ++d) {
    const float unit = __builtin_bit_cast(float, (first_unit - 5 * d) << 23);
    u32x16 packed;
#pragma unroll
    for (int e = 0; e < 16; ++e) packed[e] = h[e];
    const auto q = __builtin_amdgcn_cvt_scalef32_pk32_fp6_f16(__builtin_bit_cast(h16x32, packed), unit);
    u32x2* out = reinterpret_cast<u32x2*>(dst + d * kFp4RowBytes);
    out[0] = u32x2{(uint32_t)q[0], (uint32_t)q[1]};
    out[1] = u32x2{(uint32_t)q[2], (uint32_t)q[3]};
    out[2] = u32x2{(uint32_t)q[4], (uint32_t)q[5]};
    if (d + 1 < kFp4Digits) {   // the remainder, exact
      const u32x16 back = __builtin_bit_cast(u32x16, __builtin_amdgcn_cvt_scalef32_pk32_f16_fp6(q, unit));
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const uint32_t b = back[e];
        h[e] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(h16x2, h[e]) - __builtin_bit_cast(h16x2, b));
      }
    }
  }
  return special;
}

// What a lane knows about its place in the operands.  Weight operand: lane = 16 * kb + 4 * r + k
// holds row block r of the unit, rows 4k..4k+3, 32-column block kb.  Activation operand: lane =
// 16 * kb + row.  Result: lane 16 * lg + column holds rows 4 * lg .. 4 * lg + 3.
template <int SB, int R>
struct Fp4Lane {
  int r, k, kb, lg, row;
  uint32_t key_off2, key_off1;      // the lane's 16 key bytes within a K step of a two- / one-sub-slab tile
  uint32_t sel_even, sel_odd;       // byte selectors of the second transpose step
  static constexpr int C = (kFp4Digits + R - 1) / R;   // digits of a row: consecutive ones, one per instruction
  uint32_t a_at;                    // LDS address of the lane's largest digit in the first step
  uint32_t a_step;                  // ... and per step (0: always the zero bytes)
  uint32_t a_next;                  // ... and per digit
  uint32_t s_at, s_minus;           // block scale in the first step, 5 * largest digit's number
};

template <int SB, int R>
__device__ __forceinline__ Fp4Lane<SB, R> fp4_lane(int lane, int vectors, int digits_at) {
  Fp4Lane<SB, R> L;
  L.row = lane & 15;
  L.k = lane & 3;
  L.r = (lane >> 2) & 3;
  L.kb = L.lg = lane >> 4;
  L.key_off2 = (uint32_t)((L.kb & 1) * 1024 + ((L.kb >> 1) * 4 + L.k) * 16);
  L.key_off1 = (uint32_t)((L.kb * 4 + L.k) * 16);
  L.sel_even = 0;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const uint32_t s = (uint32_t)(c - L.k) & 3u;
    L.sel_even |= ((s & 2u ? 4u : 0u) + (s & 1u)) << (8 * c);
  }
  L.sel_odd = L.sel_even + 0x02020202u;
  const int v = L.row / (SB * R), sb = (L.row / R) % SB, part = L.row % R;
  constexpr int C = Fp4Lane<SB, R>::C;
  static_assert(kFp4Digits % C == 0, "a row has all its digits or none");
  // SB == 2: blocks 0 and 1 are the first 64 columns.  R == 4: three rows have two digits each, the fourth none.
  const bool mine = v < vectors && part * C < kFp4Digits && (SB == 1 || (L.kb >> 1) == sb);
  L.s_at = (uint32_t)(digits_at + (v < vectors ? v : 0) * kFp4VecBytes + kFp4ScalesAt + L.kb * 4);
  L.s_minus = 5u * C * part;
  L.a_at = mine ? (uint32_t)(digits_at + v * kFp4VecBytes + part * C * kFp4RowBytes + L.kb * kFp4DigitBytes) : 0u;
  L.a_step = mine ? (uint32_t)(vectors * kFp4VecBytes) : 0u;
  L.a_next = mine ? (uint32_t)kFp4RowBytes : 0u;
  return L;
}

template <int Q, int ZM, int SB>
struct Fp4Unit {
  static constexpr int QA = ZM == 2 ? 1 : Q;
  u32x4 w[Q];         // key words
  u32x2 al[SB][QA];   // scales of rows 4k..4k+3
  u32x2 zz[SB];       // offsets
};

template <int Q, int ZM, int SB, int R>
__device__ __forceinline__ void fp4_load_unit(Fp4Unit<Q, ZM, SB>& u, const Fp4Params& p, const Fp4Lane<SB, R>& L, int ru, int step,
                                              const int* step_groups) {
  const int kt = step >> 3, J = step & 7;
  const bool one = fp4_one_slab(p, step);
  const int slab_row = one ? 1024 : 2048;              // bytes of one plane of a row block
  const int r_use = min(L.r, p.RB - 1 - 4 * ru);       // blocks past the end repeat the last one (their rows are never stored)
  const uint32_t off = (uint32_t)(r_use * Q * slab_row) + (one ? L.key_off1 : L.key_off2);
  const uint8_t* base = p.bits + (int64_t)kt * p.RB * (Q * 2048) + (int64_t)ru * (4 * Q * slab_row) + J * (one ? 256 : 128);
#pragma unroll
  for (int i = 0; i < Q; ++i) u.w[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + i * slab_row + off));
  const int64_t first = (int64_t)ru * 4 * p.NG;        // (row block, group) pairs in front of the unit's rows
  const char* ab = reinterpret_cast<const char*>(p.alpha) + first * (ZM == 2 ? 32 : 32 * Q);
  const char* zb = reinterpret_cast<const char*>(p.z) + first * 32;
#pragma unroll
  for (int s = 0; s < SB; ++s) {
    const uint32_t pair = (uint32_t)(r_use * p.NG + step_groups[s * (4 / SB)]);
    const uint32_t zo = pair * 32u + L.k * 8u;
    if (ZM == 2) {
      u.al[s][0] = *reinterpret_cast<const u32x2*>(ab + zo);
    } else {
      const uint32_t ao = pair * (32u * Q) + L.k * (8u * Q);
#pragma unroll
      for (int i = 0; i < Q; ++i) u.al[s][i] = *reinterpret_cast<const u32x2*>(ab + ao + i * 8);
    }
    if (ZM != 0) u.zz[s] = *reinterpret_cast<const u32x2*>(zb + zo);
  }
}

// The four key words of a lane (dword s: rows 4k..4k+3 of slot (s + k) mod 4) -> one word per row,
// slots in order.
template <int SB, int R>
__device__ __forceinline__ void fp4_rows(const u32x4& d, const Fp4Lane<SB, R>& L, uint32_t (&row)[4]) {
  const uint32_t lo01 = __builtin_amdgcn_perm(d[1], d[0], 0x05010400u), hi01 = __builtin_amdgcn_perm(d[1], d[0], 0x07030602u);
  const uint32_t lo23 = __builtin_amdgcn_perm(d[3], d[2], 0x05010400u), hi23 = __builtin_amdgcn_perm(d[3], d[2], 0x07030602u);
  row[0] = __builtin_amdgcn_perm(lo23, lo01, L.sel_even);
  row[1] = __builtin_amdgcn_perm(lo23, lo01, L.sel_odd);
  row[2] = __builtin_amdgcn_perm(hi23, hi01, L.sel_even);
  row[3] = __builtin_amdgcn_perm(hi23, hi01, L.sel_odd);
}

// 32 weights of a row: key bit set -> -1, clear -> +1.  v_and_or_b32 takes no literals, so the
// mask (scalar) and the exponent bits (vector: one scalar operand per instruction) have to live in
// registers, which the compiler has to be kept from undoing.
struct Fp4Weights {
  uint32_t sign, one;
};
__device__ __forceinline__ Fp4Weights fp4_weights() {
  Fp4Weights k = {0x88888888u, 0x22222222u};
  asm volatile("" : "+s"(k.sign), "+v"(k.one));
  return k;
}
__device__ __forceinline__ i32x8 fp4_expand(uint32_t row, const Fp4Weights& k) {
  i32x8 b = {};
#pragma unroll
  for (int beta = 0; beta < 4; ++beta) b[beta] = (int)(((row << (3 - beta)) & k.sign) | k.one);
  return b;
}

// Activation operand with the infinities and NaNs of a K step and nothing else, as e5m2 (the upper
// byte of an fp16 number; sign turned like the digits').
template <int SB, int R>
__device__ __forceinline__ i32x8 fp4_specials(const Fp4Params& p, const Fp4Lane<SB, R>& L, int step, bool one) {
  const int v = L.row / (SB * R), sb = (L.row / R) % SB;
  const unsigned short* xv = reinterpret_cast<const unsigned short*>(p.x) + (int64_t)min(v, p.vectors - 1) * p.n;
  i32x8 a = {};
#pragma unroll
  for (int w = 0; w < 8; ++w) {
    uint32_t packed = 0;
#pragma unroll 1
    for (int byte = 0; byte < 4; ++byte) {
      const int e = 4 * w + byte;
      // byte e of lane 16 * kb + row is column 64 * (e / 16) + 16 * kb + e % 16 of an 8-bit operand
      const int col = 64 * (e >> 4) + 16 * L.kb + (e & 15), kb4 = col >> 5, idx = col & 31;
      const int chunk = fp4_chunk(step, one, kb4, (idx >> 1) & 3), j = 4 * (idx & 1) + (idx >> 3);
      const bool mine = v < p.vectors && L.row % R == 0 && chunk < p.nchunks && ((chunk - 16 * step) >> 2) / (4 / SB) == sb;
      const uint32_t x = xv[(int64_t)min(chunk, p.nchunks - 1) * 8 + j];
      if (mine && (x & 0x7c00u) == 0x7c00u) packed |= (((x >> 8) ^ 0x80u) | ((x & 0x3ffu) ? 2u : 0u)) << (8 * byte);
    }
    a[w] = (int)packed;
  }
  return a;
}

// The lane's part of the activation operand for digit c of its row in a K step.
template <int SB, int R>
__device__ __forceinline__ i32x8 fp4_digit(const Fp4Lane<SB, R>& L, const char* lds, int local, int c) {
  const uint32_t at = L.a_at + (uint32_t)local * L.a_step + c * L.a_next;
  const u32x2* src = reinterpret_cast<const u32x2*>(lds + at);
  const u32x2 q0 = src[0], q1 = src[1], q2 = src[2];
  return i32x8{(int)q0.x, (int)q0.y, (int)q1.x, (int)q1.y, (int)q2.x, (int)q2.y, 0, 0};
}

// R == 4: the last of a vector's four rows has no digits; not even an infinite scale makes anything of it.
template <int R>
__device__ __forceinline__ constexpr bool fp4_empty_row(int e) { return (e % R) * ((kFp4Digits + R - 1) / R) >= kFp4Digits; }

// The block scale that goes with the lane's largest digit in a K step.
template <int SB, int R>
__device__ __forceinline__ int fp4_block_scale(const Fp4Params& p, const Fp4Lane<SB, R>& L, const char* lds, int local) {
  return *reinterpret_cast<const int*>(lds + L.s_at + (uint32_t)local * (uint32_t)(p.vectors * kFp4VecBytes)) - (int)L.s_minus;
}

// One unit into the sums: acc[b][e] is operand row 4 * lg + e, weight row 4k + b.  The unit's planes are
// added among themselves first: one addition per unit to the long sums, whose rounding is what the
// result's error is made of (49152 x 12288 at 16 vectors: 1.4e-7 without, see kFp4MaxRun).  The digits stay in
// registers for all planes where these have room, else they are read from LDS for every plane.
template <int Q, int ZM, int SB, int R>
__device__ __forceinline__ void fp4_compute(const Fp4Unit<Q, ZM, SB>& u, const Fp4Params& p, const Fp4Lane<SB, R>& L,
                                            const Fp4Weights& kw, const char* lds, int local, f32x4 (&acc)[4]) {
  constexpr int C = Fp4Lane<SB, R>::C;
  constexpr bool kHold = 6 * C + 2 * (4 * Q + SB * (2 * Q + (ZM != 0 ? 2 : 0))) <= 100;
  const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  const int scale = fp4_block_scale(p, L, lds, local);
  i32x8 held[kHold ? C : 1];
  if (kHold) {
#pragma unroll
    for (int c = C - 1; c >= 0; --c) held[kHold ? c : 0] = fp4_digit(L, lds, local, c);
  }
  auto digit = [&](int c) { return kHold ? held[kHold ? c : 0] : fp4_digit(L, lds, local, c); };
  // The two largest digits of a row, then the others (see the head of this file).
  constexpr int kHi = C < 2 ? C : 2, kChains = C > kHi ? 2 : 1;
  f32x4 sum[4] = {zero, zero, zero, zero};
  if (ZM != 0) {   // offset term of eq. 3: z times the sum of the activations
    const int m1 = (int)0xaaaaaaaa;
    const i32x8 w = {m1, m1, m1, m1, 0, 0, 0, 0};
#pragma unroll
    for (int h = kChains - 1; h >= 0; --h) {
      f32x4 sx = zero;
#pragma unroll
      for (int c = (h ? C : kHi) - 1; c >= (h ? kHi : 0); --c) sx = fp4_mfma(digit(c), w, sx, scale - 5 * c);
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (!fp4_empty_row<R>(e)) sum[b][e] = fmaf(half_of(u.zz[(e / R) % SB], b), sx[e], sum[b][e]);
    }
  }
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    __builtin_amdgcn_sched_barrier(0);   // one plane's expanded weights at a time
    uint32_t row[4];
    fp4_rows(u.w[i], L, row);
    i32x8 w[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) w[b] = fp4_expand(row[b], kw);
#pragma unroll
    for (int h = kChains - 1; h >= 0; --h) {
      f32x4 s[4] = {zero, zero, zero, zero};   // four independent chains
#pragma unroll
      for (int c = (h ? C : kHi) - 1; c >= (h ? kHi : 0); --c) {
        const i32x8 a = digit(c);
#pragma unroll
        for (int b = 0; b < 4; ++b) s[b] = fp4_mfma(a, w[b], s[b], scale - 5 * c);
      }
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (fp4_empty_row<R>(e)) continue;
          float al = half_of(u.al[(e / R) % SB][ZM == 2 ? 0 : i], b);
          if (ZM == 2) al *= (float)(1 << i);   // exact: the per-plane layout's scale bit for bit
          sum[b][e] = fmaf(al, s[b][e], sum[b][e]);
        }
      if (kChains > 1) {   // chain after chain: left alone, the compiler keeps all planes' products for later (and spills)
#pragma unroll
        for (int b = 0; b < 4; ++b) asm volatile("" : "+v"(sum[b]));
      }
    }
  }
#pragma unroll
  for (int b = 0; b < 4; ++b) acc[b] += sum[b];
}

// Four consecutive rows of one vector to y.
__device__ __forceinline__ void fp4_store_rows(const Fp4Params& p, int v, int row, const float (&s)[4]) {
  const int64_t at = (int64_t)v * p.m + row;
  if ((p.m & 3) == 0 && row + 4 <= p.m) {
    if (p.y_f32) {
      *reinterpret_cast<f32x4*>(static_cast<float*>(p.y) + at) = f32x4{s[0], s[1], s[2], s[3]};
    } else {   // nearest even (paper table 1: FP16 output)
      const __half h[4] = {__float2half_rn(s[0]), __float2half_rn(s[1]), __float2half_rn(s[2]), __float2half_rn(s[3])};
      *reinterpret_cast<u32x2*>(static_cast<__half*>(p.y) + at) = __builtin_bit_cast(u32x2, h);
    }
    return;
  }
#pragma unroll
  for (int b = 0; b < 4; ++b)
    if (row + b < p.m) {
      if (p.y_f32)
        static_cast<float*>(p.y)[at + b] = s[b];
      else
        static_cast<__half*>(p.y)[at + b] = __float2half_rn(s[b]);
    }
}

__device__ __forceinline__ void fp4_store_pair(float* p, float a, float b) {
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p), __builtin_bit_cast(uint64_t, f32x2v{a, b}), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ f32x2v fp4_load_pair(const float* p) {
  return __builtin_bit_cast(f32x2v, __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// A finished item: to LDS (`dst`: the item's place), or, where it is all there is of the row unit in
// this K group, to y or the workspace.
template <int SB, int R>
__device__ __forceinline__ void fp4_finish_item(const Fp4Params& p, const Fp4Lane<SB, R>& L, float* dst, int kg, int ru,
                                                f32x4 (&acc)[4]) {
  constexpr int P = SB * R;    // operand rows of a vector
  constexpr int NR = 4 / P;    // vectors of a lane
  const int row = ru * kFp4UnitRows + 4 * L.row;
#pragma unroll
  for (int c = 0; c < NR; ++c) {
    const int v = L.lg * NR + c;
    float s[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      if (P == 1) s[b] = acc[b][c];
      if (P == 2) s[b] = acc[b][2 * c + 1] + acc[b][2 * c];
      if (P == 4) s[b] = (acc[b][3] + acc[b][2]) + (acc[b][1] + acc[b][0]);
    }
    if (v < p.vectors) {
      if (dst) {
        *reinterpret_cast<f32x4*>(dst + v * kFp4UnitRows + 4 * L.row) = f32x4{s[0], s[1], s[2], s[3]};
      } else if (p.KG == 1) {
        fp4_store_rows(p, v, row, s);
      } else if (row < p.vec_stride) {
        float* q = p.partial + kg * p.kg_stride + v * p.vec_stride + row;
        fp4_store_pair(q, s[0], s[1]);
        fp4_store_pair(q + 2, s[2], s[3]);
      }
    }
  }
}

// The sum of the K groups, in group order, of vectors 4 * vq .. 4 * vq + 3 of a row unit.
__device__ __forceinline__ void fp4_add_groups(const Fp4Params& p, int lane, int ru, int vq) {
  const int row = ru * kFp4UnitRows + 4 * (lane & 15), v = 4 * vq + (lane >> 4);
  constexpr int kBatch = 8;   // K groups whose loads are in flight together
  if (row >= p.vec_stride || v >= p.vectors) return;
  const float* src = p.partial + v * p.vec_stride + row;
  double sum[4] = {0.0, 0.0, 0.0, 0.0};   // few additions, and the last ones: 64 bits cost nothing here
#pragma unroll 1
  for (int k0 = 0; k0 < p.KG; k0 += kBatch) {
    f32x2v t[kBatch][2];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const float* q = src + (int64_t)min(k0 + j, p.KG - 1) * p.kg_stride;
      t[j][0] = fp4_load_pair(q);
      t[j][1] = fp4_load_pair(q + 2);
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j)
      if (k0 + j < p.KG) {
        sum[0] += t[j][0].x;
        sum[1] += t[j][0].y;
        sum[2] += t[j][1].x;
        sum[3] += t[j][1].y;
      }
  }
  const float s[4] = {(float)sum[0], (float)sum[1], (float)sum[2], (float)sum[3]};
  fp4_store_rows(p, v, row, s);
}

// Items of a stretch of row units [ru0, ru0 + units): the wavefront's first is item number `wave`,
// whose first unit is in `ua`; the others come from the queue.
template <int Q, int ZM, int SB, int R>
__device__ __forceinline__ void fp4_items(const Fp4Params& p, const Fp4Lane<SB, R>& L, char* lds, float* part, int lane, int wave, int kg,
                                          int step0, int steps, int per_unit, uint32_t per_unit_magic, int ru0, int units, int groups_at,
                                          Fp4Unit<Q, ZM, SB>& ua) {
  int* queue = reinterpret_cast<int*>(lds + 24);
  const int* groups = reinterpret_cast<const int*>(lds + groups_at);
  const Fp4Weights kw = fp4_weights();
  const int items = units * per_unit;
  if (wave >= items) return;
  Fp4Unit<Q, ZM, SB> ub;
  auto unit_of = [&](int t) { return per_unit == 1 ? t : (int)__umulhi((uint32_t)t, per_unit_magic); };
  int item = wave, ru = unit_of(item), local = (item - ru * per_unit) * p.run, end = min(local + p.run, steps);
  f32x4 acc[4];
  auto clear = [&]() {
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  };
  // The read of lane 0's ticket follows the addition directly: left for later, the branch around the
  // addition would stand at the end of the loop, where the compiler may let the other lanes go
  // round without lane 0.
  auto draw = [&]() {
    int t = 0;
    if (lane == 0) t = __hip_atomic_fetch_add(queue, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    return __builtin_amdgcn_readfirstlane(t);
  };
  clear();
  // computes the unit in `now` while the next one is on its way to `next`; false: none left
  auto turn = [&](const Fp4Unit<Q, ZM, SB>& now, Fp4Unit<Q, ZM, SB>& next) {
    const bool last = local + 1 == end;
    int nitem = item, nru = ru, nlocal = local + 1;
    if (last) {
      nitem = draw();
      nru = unit_of(nitem);
      nlocal = (nitem - nru * per_unit) * p.run;
      if (nitem >= items) {   // past the end: this unit again, its lines are at hand (the loads stay unconditional)
        nru = ru;
        nlocal = local;
      }
    }
    fp4_load_unit(next, p, L, ru0 + nru, step0 + nlocal, groups + nlocal * 4);
    fp4_compute<Q, ZM, SB, R>(now, p, L, kw, lds, local, acc);
    if (last) {
      fp4_finish_item(p, L, per_unit > 1 ? part + item * p.vectors * kFp4UnitRows : nullptr, kg, ru0 + ru, acc);
      if (nitem >= items) return false;
      clear();
      end = min(nlocal + p.run, steps);
    }
    item = nitem;
    ru = nru;
    local = nlocal;
    return true;
  };
  while (turn(ua, ub) && turn(ub, ua)) {
  }
}

// Infinities and NaNs of the activations have no digits.  Where there are any, the sums are formed once more with
// their products among them, after the finite ones, and written over those of the (vector, row)
// pairs that they reach: those with a product that is not zero (of what is in the operand only the
// infinities and NaNs give one), whatever the scales are.  Rare, and not tuned: what is written is
// an infinity or NaN, so that one chain does for the digits.
template <int Q, int ZM, int SB, int R>
__device__ __forceinline__ void fp4_overlay_specials(const Fp4Params& p, const Fp4Lane<SB, R>& L, const char* lds, float* part, int wave,
                                                     int waves, int kg, int step0, int steps, int per_unit, int ru0, int units,
                                                     int groups_at) {
  constexpr int P = SB * R, NR = 4 / P;
  const int* groups = reinterpret_cast<const int*>(lds + groups_at);
  const Fp4Weights kw = fp4_weights();
#pragma unroll 1
  for (int u = wave; u < units; u += waves) {
    f32x4 acc[4];
    uint32_t reached = 0;   // bit 4 * b + c: vector c of the lane, row b
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
    for (int local = 0; local < steps; ++local) {
      const int step = step0 + local, rb = min(4 * (ru0 + u) + L.r, p.RB - 1);
      const bool one = fp4_one_slab(p, step);
      const int slab_row = one ? 1024 : 2048;
      const uint8_t* keys = p.bits + (int64_t)(step >> 3) * p.RB * (Q * 2048) + (int64_t)rb * (Q * slab_row) +
                            (step & 7) * (one ? 256 : 128) + (one ? L.key_off1 : L.key_off2);
      const i32x8 a = fp4_specials(p, L, step, one);
      const int scale = fp4_block_scale(p, L, lds, local);
#pragma unroll 1
      for (int t = (ZM != 0 ? -1 : 0); t < Q; ++t) {   // planes; -1: the offsets, a plane of +1
        uint32_t row[4] = {0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu};
        if (t >= 0) fp4_rows(*reinterpret_cast<const u32x4*>(keys + t * slab_row), L, row);
        f32x4 dot[4];
#pragma unroll
        for (int b = 0; b < 4; ++b)
          dot[b] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, fp4_expand(row[b], kw), f32x4{0.0f, 0.0f, 0.0f, 0.0f},
                                                                    1 /* A: e5m2 */, 4, 0, 127, 0, 127);
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (!(dot[b][e] == 0.0f)) reached |= 1u << (4 * b + e / P);
#pragma unroll 1
        for (int c = Fp4Lane<SB, R>::C - 1; c >= 0; --c) {
          const i32x8 digit = fp4_digit(L, lds, local, c);
#pragma unroll
          for (int b = 0; b < 4; ++b) dot[b] += fp4_mfma(digit, fp4_expand(row[b], kw), f32x4{0.0f, 0.0f, 0.0f, 0.0f}, scale - 5 * c);
        }
#pragma unroll
        for (int s = 0; s < SB; ++s) {
          const int64_t pair = (int64_t)rb * p.NG + groups[local * 4 + s * (4 / SB)];
          const u32x2 sc = *reinterpret_cast<const u32x2*>(
              t < 0 ? p.z + pair * 16 + L.k * 4 : (ZM == 2 ? p.alpha + pair * 16 + L.k * 4 : p.alpha + ((pair * 4 + L.k) * Q + t) * 4));
#pragma unroll
          for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              float al = half_of(sc, b);
              if (ZM == 2 && t >= 0) al *= (float)(1 << t);
              if ((e / R) % SB == s && !fp4_empty_row<R>(e)) acc[b][e] = fmaf(al, dot[b][e], acc[b][e]);
            }
        }
      }
    }
#pragma unroll
    for (int c = 0; c < NR; ++c)
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        float s = acc[b][c * P];
#pragma unroll
        for (int e = 1; e < P; ++e) s += acc[b][c * P + e];
        const int v = L.lg * NR + c, row = (ru0 + u) * kFp4UnitRows + 4 * L.row + b;
        if (v >= p.vectors || (reached >> (4 * b + c) & 1u) == 0u) continue;
        if (per_unit > 1)
          part[(u * per_unit * p.vectors + v) * kFp4UnitRows + 4 * L.row + b] = s;
        else if (p.KG > 1 && row < p.vec_stride)
          store_device_coherent(p.partial + kg * p.kg_stride + v * p.vec_stride + row, s);
        else if (p.KG == 1 && row < p.m && p.y_f32)
          static_cast<float*>(p.y)[(int64_t)v * p.m + row] = s;
        else if (p.KG == 1 && row < p.m)
          static_cast<__half*>(p.y)[(int64_t)v * p.m + row] = __float2half_rn(s);
      }
  }
}

// Longest item in K steps.  An item's sums are fp32 additions one after the other, everything behind
// them is added in 64 bits: 12 of them keep the error against a 64-bit product at 0.9e-7 (relative, 2-norm)
// where the lookup kernels have 1.0e-7; 39 gave 2.0e-7.
constexpr int kFp4MaxRun = 12;

constexpr int kFp4Waves = 8;   // per workgroup, and what a compute unit holds at 256 registers each

template <int Q, int ZM, int SB, int R>
__global__ __launch_bounds__(kFp4Waves * 64) void lutgemm_fp4_kernel(Fp4Params p) {
  extern __shared__ __align__(16) char lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  constexpr int waves = kFp4Waves;
  const int kg = blockIdx.x, rs = blockIdx.y;
  const int step0 = kg * p.SPG, steps = min(p.SPG, p.steps - step0);
  const int range0 = rs * p.range_base + min(rs, p.range_rem), range_units = p.range_base + (rs < p.range_rem ? 1 : 0);
  const int digits_at = kFp4FixedBytes, groups_at = digits_at + steps * p.vectors * kFp4VecBytes;
  float* part = reinterpret_cast<float*>(lds + groups_at + steps * 16);
  uint32_t* wave_flag = reinterpret_cast<uint32_t*>(lds + 32);
  const int per_unit = (steps + p.run - 1) / p.run;      // items of a row unit
  const uint32_t per_unit_magic = 0xffffffffu / (uint32_t)per_unit + 1u;   // t / per_unit, exact for the few thousand items there are
  const Fp4Lane<SB, R> L = fp4_lane<SB, R>(lane, p.vectors, digits_at);

  // ---- digits.  The activations are asked for first and waited for: asked for behind the first
  // unit's weights they would arrive behind them.
  const int tasks = steps * 4 * p.vectors;
  Fp4Task task;
  fp4_fetch_task(task, p, min((int)threadIdx.x, tasks - 1), step0);
  auto first_unit = [&](int ru0, int units, int& ru, int& local) {
    const int t = min(wave, units * per_unit - 1), u = per_unit == 1 ? t : (int)__umulhi((uint32_t)t, per_unit_magic);
    ru = ru0 + u;
    local = (t - u * per_unit) * p.run;
  };
  int ru, local;
  first_unit(range0, min(p.stretch, range_units), ru, local);
  int first_groups[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) first_groups[s] = min(((step0 + local) * 4 + s) * 32, p.n - 1) / p.g;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  Fp4Unit<Q, ZM, SB> ua;
  fp4_load_unit(ua, p, L, ru, step0 + local, first_groups);
  bool special = false;
  if ((int)threadIdx.x < tasks) special = fp4_make_digits(task, p, lds, step0, digits_at);
  for (int t = threadIdx.x + kFp4Waves * 64; t < tasks; t += kFp4Waves * 64) {
    fp4_fetch_task(task, p, t, step0);
    special |= fp4_make_digits(task, p, lds, step0, digits_at);
  }
  for (int t = threadIdx.x; t < steps * 4; t += kFp4Waves * 64)
    *reinterpret_cast<int*>(lds + groups_at + t * 4) = min((step0 * 4 + t) * 32, p.n - 1) / p.g;
  if (threadIdx.x < 6) *reinterpret_cast<uint32_t*>(lds + threadIdx.x * 4) = 0u;
  if (threadIdx.x == 6) *reinterpret_cast<int*>(lds + 24) = waves;
  const bool wave_special = __builtin_amdgcn_ballot_w64(special) != 0;
  if (lane == 0) wave_flag[wave] = wave_special ? 1u : 0u;
  __syncthreads();
  uint32_t any_special = 0;
  for (int w = 0; w < waves; ++w) any_special |= wave_flag[w];
  any_special = __builtin_amdgcn_readfirstlane(any_special);

  for (int ru0 = range0; ru0 < range0 + range_units; ru0 += p.stretch) {
    const int units = min(p.stretch, range0 + range_units - ru0);
    if (ru0 != range0) {   // a further stretch: queue and first unit anew (the partial sums have been read)
      if (threadIdx.x == 0) *reinterpret_cast<int*>(lds + 24) = waves;
      first_unit(ru0, units, ru, local);
      fp4_load_unit(ua, p, L, ru, step0 + local, reinterpret_cast<const int*>(lds + groups_at) + local * 4);
      __syncthreads();
    }
    fp4_items<Q, ZM, SB, R>(p, L, lds, part, lane, wave, kg, step0, steps, per_unit, per_unit_magic, ru0, units, groups_at, ua);
    if (any_special != 0u) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the finite sums are where they belong
      __syncthreads();
      int lane_again = lane;   // (nothing of this is to stay in registers over the items)
      asm volatile("" : "+v"(lane_again));
      const Fp4Lane<SB, R> again = fp4_lane<SB, R>(lane_again, p.vectors, digits_at);
      fp4_overlay_specials<Q, ZM, SB, R>(p, again, lds, part, wave, waves, kg, step0, steps, per_unit, ru0, units, groups_at);
    }
    if (per_unit > 1) {    // items of a row in step order
      __syncthreads();
      for (int t = threadIdx.x; t < units * p.vectors * 16; t += kFp4Waves * 64) {   // (row unit, vector, four rows)
        const int uv = t >> 4, u = uv / p.vectors, v = uv - u * p.vectors, row = (ru0 + u) * kFp4UnitRows + 4 * (t & 15);
        const f32x4* src = reinterpret_cast<const f32x4*>(part + (u * per_unit * p.vectors + v) * kFp4UnitRows) + (t & 15);
        double sum[4] = {0.0, 0.0, 0.0, 0.0};   // few additions, and the last ones: 64 bits cost nothing here
        for (int j = 0; j < per_unit; ++j) {
          const f32x4 q = src[j * p.vectors * (kFp4UnitRows / 4)];
#pragma unroll
          for (int b = 0; b < 4; ++b) sum[b] += q[b];
        }
        const float s[4] = {(float)sum[0], (float)sum[1], (float)sum[2], (float)sum[3]};
        if (p.KG == 1) {
          fp4_store_rows(p, v, row, s);
        } else if (row < p.vec_stride) {
          float* q = p.partial + kg * p.kg_stride + v * p.vec_stride + row;
          fp4_store_pair(q, s[0], s[1]);
          fp4_store_pair(q + 2, s[2], s[3]);
        }
      }
    }
    if (ru0 + p.stretch < range0 + range_units) __syncthreads();
  }
  if (p.KG == 1) return;

  // ---- K groups: the hand-off of finish_row_range.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const bool all = __hip_atomic_fetch_add(p.counters + rs, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)(p.KG - 1);
    wave_flag[0] = all ? 1u : 0u;
    if (all) __hip_atomic_store(p.counters + rs, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // zero for the next call on this workspace
  }
  __syncthreads();
  if (wave_flag[0] == 0u) return;
  const int quads = (p.vectors + 3) / 4;
  for (int t = wave; t < range_units * quads; t += waves) {
    const int u = t / quads;
    fp4_add_groups(p, lane, range0 + u, t - u * quads);
  }
}
