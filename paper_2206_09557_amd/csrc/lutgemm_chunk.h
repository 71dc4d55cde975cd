// One activation vector where every chunk of 8 columns may have a scale set of its own
// (g % 16 == 8; part of lutgemm_device.hip; included there).
//
// Here a lane needs 4 T scale sets for its dwords, so all planes of a unit together do not fit its
// registers.  The work is handed out in items of ONE part of a (K tile, row block) unit: a
// plane, or the offsets.  An item is one fetch of 4 T scale words and T key words per lane, and a
// wavefront has the next item's fetch in flight while it looks up the current one.
//   * The offsets are one more plane whose keys are all 0xff (that table entry is the sum of
//     the chunk's activations) and whose scales lie in the offset buffer.
//   * The sum of an item and row goes to a place of its own in LDS, where the tiles of a K
//     group add to it in order; the parts of a row are added in order at the end.  So the
//     result does not depend on which wavefront took what, and nothing goes through memory
//     between tiles.  A row range that has more items than places is walked in stretches.
//
// What bounds it: on small layers latency, a chain of activations -> tables -> fetch -> sum over the K
// groups; on large ones the stream, of which the scales are more than a third at g = 24.
// Measured (MI355X, weights in no cache; before: one plane fetched at a time by a wavefront that
// kept a whole unit, sums sent from tile to tile through memory): 3001 x 5160, q = 5, g = 24 with offsets
// 15.2 -> 10.2 us; 8192 x 8200, q = 4, g = 8 with offsets 52.5 -> 39.8; 49152 x 12288, q = 3, g = 24 87 -> 71
// (5.3 TB/s); 1000 x 1000, q = 4, g = 40 9.9 -> 6.3; 704 x 712, q = 1, g = 8 5.3 -> 5.0.
// Fifty random layers of 64 to 50000 rows and columns: 1.17 times as fast on average; slowest
// beside the old kernel are two planes with offsets at g = 40 (5200 x 13080 13.3 -> 13.8).
template <int T>
struct ChunkItem {
  u32x4 w[T];        // key words: dword s = four rows of slot 4j + (s + k) mod 4
  u32x2 al[4][T];    // fp16 scales of the lane's four rows per (dword, sub-slab)
};

template <int Q, int T, bool HAS_Z, bool SHARED>
__device__ __forceinline__ void load_chunk_item(ChunkItem<T>& u, const GemvParams& p, int64_t tile_base, int64_t group0,
                                                int rb, int part, int lane, const uint32_t (&rel)[4][T]) {
  const bool offsets = HAS_Z && part == Q;
  const int plane = offsets ? 0 : part;
  const char* bp = reinterpret_cast<const char*>(p.bits) + tile_base + ((int64_t)rb * Q + plane) * (T * 1024);
  const uint32_t lane_bytes = offsets ? 0u : (uint32_t)lane * 16u;   // (the keys of the offsets are not used: one address, no branch)
#pragma unroll
  for (int t = 0; t < T; ++t) u.w[t] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(bp + t * 1024 + lane_bytes));
  const uint32_t stride = SHARED || offsets ? 1u : (uint32_t)Q;      // values per (row, group) in the buffer
  const char* base = reinterpret_cast<const char*>(offsets ? p.z : p.alpha);
  base += (((int64_t)rb * p.NG + group0) * 4 * stride + (stride == 1u ? 0 : plane)) * 8;
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int t = 0; t < T; ++t) u.al[s][t] = *reinterpret_cast<const u32x2*>(base + __umul24(rel[s][t], stride));
}

// Look up, scale, add over the lanes, and put the 16 row sums into the item's place.
template <int Q, int T, bool HAS_Z, bool SHARED>
__device__ __forceinline__ void finish_chunk_item(const ChunkItem<T>& u, float* lut, int item, int part, int lane,
                                                  const uint32_t (&lane_base)[4], bool first_tile) {
  const bool offsets = HAS_Z && part == Q;
  float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if (offsets) {   // (wave-uniform) one lookup serves the four rows
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const float v = lds_f32(((uint32_t)t << 16) | 0xff00u | (lane_base[s] & 0xffu));
#pragma unroll
        for (int rho = 0; rho < 4; ++rho) acc[rho] = fmaf(half_of(u.al[s][t], rho), v, acc[rho]);
      }
  } else {
    const float factor = SHARED ? (float)(1 << part) : 1.0f;
#pragma unroll
    for (int rho = 0; rho < 4; ++rho) {
      const uint32_t sel_t[2] = {0x0c0c0000u | ((4u + rho) << 8), 0x0c010000u | ((4u + rho) << 8)};   // see accumulate_unit
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int t = 0; t < T; ++t) {
          const float v = lds_f32(__builtin_amdgcn_perm(u.w[t][s], lane_base[s], sel_t[t]));
          const float a = half_of(u.al[s][t], rho);
          acc[rho] = fmaf(SHARED ? a * factor : a, v, acc[rho]);
        }
    }
  }
  int row;
  const float sum = quad_rows_reduce(acc, lane, &row);
  if (lane < 16) {
    float* r = lut + kRunWord + item * 16 + row;
    *r = first_tile ? sum : *r + sum;
  }
}

// One workgroup, one K tile, row blocks [rb0, rb1) of a stretch.
template <int Q, int T, bool HAS_Z, bool SHARED>
__device__ __forceinline__ void chunk_tile_body(const GemvParams& p, float* lut, int kt, int rb0, int rb1, bool first_tile) {
  constexpr int kParts = Q + (HAS_Z ? 1 : 0);
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));   // (as in tile_body)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int chunks_in_tile = min(128, p.nchunks - 128 * kt);
  const int64_t tile_base = (int64_t)kt * p.RB * Q * 2048;
  const int n_items = (rb1 - rb0) * kParts;
  if (threadIdx.x == 0) reinterpret_cast<int*>(lut + kQueueWord)[0] = kWaves;   // items 0..kWaves-1 are taken

  // the start of a tile as in tile_body: half the wavefronts build, the others fetch
  const bool builder = wave >= kWaves / 2;
  const int slot0 = 2 * (wave & 7);
  u32x4 xr0 = {0u, 0u, 0u, 0u}, xr1 = {0u, 0u, 0u, 0u};
  if (builder) {
    xr0 = fetch_slot_x<T>(p, kt, chunks_in_tile, slot0, lane);
    xr1 = fetch_slot_x<T>(p, kt, chunks_in_tile, slot0 + 1, lane);
  }
  // Byte offset of the scale set of every (dword, sub-slab) from that of the tile's first
  // group, in a buffer of one value per (row, group); worked out while x is on its way.  The
  // groups within the tile by a reciprocal: at most 128, so the product is off by less than one
  // (2^-22 of it, and c's rounding does no more), which the comparison behind it corrects.
  const uint32_t g8 = (uint32_t)p.g >> 3, first_chunk = 128u * (uint32_t)kt;
  const uint32_t group0 = first_chunk / g8, into = first_chunk - group0 * g8;
  const float per_group = 1.0f / (float)g8;
  uint32_t rel[4][T];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int slot = (lane & ~3) | ((s + lane) & 3);
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const uint32_t c = into + (uint32_t)min(T * slot + t, chunks_in_tile - 1);
      uint32_t group = (uint32_t)((float)c * per_group);
      const int32_t rest = (int32_t)(c - group * g8);
      group += rest < 0 ? -1 : (rest >= (int32_t)g8 ? 1 : 0);
      rel[s][t] = (group * 4u + (uint32_t)(lane & 3)) * 8u;
    }
  }
  if (builder) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  auto load = [&](ChunkItem<T>& u, int item) {
    load_chunk_item<Q, T, HAS_Z, SHARED>(u, p, tile_base, group0, rb0 + item / kParts, item % kParts, lane, rel);
  };
  ChunkItem<T> a, b;
  int cur = wave;
  const int first = min(cur, n_items - 1);
  if (!builder) {
    load(a, first);
  } else {
    build_slot<T>(lut, chunks_in_tile, slot0, lane, xr0);
    build_slot<T>(lut, chunks_in_tile, slot0 + 1, lane, xr1);
  }
  __syncthreads();
  if (builder) load(a, first);
  uint32_t lane_base[4];
  float unused[4][T];
  lane_tables<T, false>(lane, lane_base, unused);
  auto finish = [&](const ChunkItem<T>& u, int item) {
    finish_chunk_item<Q, T, HAS_Z, SHARED>(u, lut, item, item % kParts, lane, lane_base, first_tile);
  };
  if (cur >= n_items) return;
  while (true) {   // two items a trip, so that the fetched registers are never moved
    const int next = next_unit(lut, lane);
    if (next >= n_items) {
      finish(a, cur);
      break;
    }
    load(b, next);
    __builtin_amdgcn_sched_barrier(0);
    finish(a, cur);
    cur = next_unit(lut, lane);
    if (cur >= n_items) {
      finish(b, next);
      break;
    }
    load(a, cur);
    __builtin_amdgcn_sched_barrier(0);
    finish(b, next);
  }
}

template <int Q, bool HAS_Z, bool SHARED>
__global__ __launch_bounds__(kThreads) void lutgemm_gemv_chunk_kernel(GemvParams p) {
  __shared__ float lut[kGemvLdsFloats];   // (the kernel's only LDS object: see gemv_workgroup)
  constexpr int kParts = Q + (HAS_Z ? 1 : 0), kStretch = kRunBlocks / kParts;
  const int kg = blockIdx.x, rs = blockIdx.y;
  int rb0, rb1;
  row_range(p, rs, &rb0, &rb1);
  float* partial = p.partial + (int64_t)kg * p.kg_stride;
  const bool direct = p.NT == 1;
  const int kt0 = kg * p.TPG, kt1 = min(kt0 + p.TPG, p.NT);
  for (int s0 = rb0; s0 < rb1; s0 += kStretch) {
    const int s1 = min(s0 + kStretch, rb1);
    for (int kt = kt0; kt < kt1; ++kt) {
      // every lookup of the previous tile is done before its tables and the queue are written again
      if (kt != kt0 || s0 != rb0) __syncthreads();
      if (min(128, p.nchunks - 128 * kt) > 64)
        chunk_tile_body<Q, 2, HAS_Z, SHARED>(p, lut, kt, s0, s1, kt == kt0);
      else
        chunk_tile_body<Q, 1, HAS_Z, SHARED>(p, lut, kt, s0, s1, kt == kt0);
    }
    __syncthreads();
    const int rows = (s1 - s0) * 16;
    for (int i = threadIdx.x; i < rows; i += kThreads) {
      const float* r = lut + kRunWord + (i >> 4) * (kParts * 16) + (i & 15);
      float sum = r[0];
#pragma unroll
      for (int part = 1; part < kParts; ++part) sum += r[part * 16];
      store_row_sum(p, partial, direct, s0 * 16 + i, sum);
    }
  }
  if (!direct) finish_row_range<1, (Q <= 4)>(p, lut, rs, rb0, rb1);
}
