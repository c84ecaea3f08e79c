// Sparse gradient (Alg. 1, sparse branch) of a small batch by array tile.
//
// The general pipeline (pss_sparse.hip) groups the lookups, sorts the chunk
// records fully by base and scans an ownership list: 26 launches, 140-150 us
// however small the batch.  Here:
//
//   records  the run sums of the pieces of the order by token (pss_pieces.hip): one
//            row of d floats per run and one (base, row * C + j) record per run and chunk
//   sort     one stable 8-bit radix pass by super tile (at most 255 of
//            2^shift elements, shift >= 12; positions without a record sort last)
//   count    (list) one workgroup per tile of 2^12 elements: the elements that the records
//            reaching the tile touch
//   apply    one workgroup per tile: the records reaching it are staged in
//            LDS, stably ordered by the range they begin in; lane groups, each
//            owning a range of the tile, add the parts of the chunks that
//            fall in their range to an LDS copy with plain read-add-writes;
//            then the tile's touched elements are written as (location,
//            value), or updated in place
//
// No float atomics: an element belongs to one lane group, which adds its
// records in their sorted order, so every sum is taken in a fixed order.
// Bound by the chain of launches and of dependent loads (times: see
// sparse_by_tile).  Letting every group scan all of a tile's records instead
// of two bins took the apply step from 31 to 38 us on the list of 26 x 4096
// lookups, 1024 threads per tile to 64 us.
#include "pss_launch.hpp"

namespace pss {

constexpr int kTileShift = 12;
constexpr uint32_t kTileLen = 1u << kTileShift;
constexpr int kTileThreads = 256;
constexpr int kTileStage = 4;  // records per thread staged together
constexpr uint32_t kTileWords = kTileLen / 32;  // bits of the touched elements
constexpr int kTileBatch = 8;                   // records a lane group requests together

// Smallest super tile (a power of two of whole tiles) of which at most 255
// cover the array: digit 255 is left to the positions without a record.
static int super_shift(uint32_t M) {
  int s = kTileShift;
  while (((M - 1) >> s) > 254) ++s;
  return s;
}

// starts[u] = first of the sorted records of super tile u (starts[256]: their
// number), by the workgroup, from the super tiles' record counts.
__device__ __forceinline__ void super_starts(uint32_t* starts, uint32_t* wsum,
                                             const uint32_t* __restrict__ totals) {
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & (kWave - 1);
  const uint32_t c = totals[tid];
  uint32_t incl = c;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const uint32_t y = __shfl_up(incl, off);
    if (lane >= off) incl += y;
  }
  if (lane == kWave - 1) wsum[wv] = incl;
  __syncthreads();
  uint32_t pre = 0;
#pragma unroll
  for (int v = 0; v < kTileThreads / kWave; ++v) pre += v < wv ? wsum[v] : 0u;
  starts[tid] = pre + incl - c;
  if (tid == kTileThreads - 1) starts[kTileThreads] = pre + incl;
  __syncthreads();
}

// Calls f(lo, hi) for every run of the sorted records that can reach tile x:
// those of its own super tile; of the one before when the tile is its first
// (a chunk is no longer than a tile, so it crosses at most one boundary); for
// tile 0 of the last two (chunks wrapping past M, the last super tile
// possibly shorter than a chunk).
template <typename F>
__device__ __forceinline__ void for_runs(const uint32_t x, const uint32_t M, const int shift,
                                         const uint32_t* starts, F f) {
  const uint32_t x0 = x << kTileShift;
  const uint32_t ns = ((M - 1) >> shift) + 1, u = x0 >> shift;
  const uint32_t lo0 = u >= 1 && (x0 & ((1u << shift) - 1)) == 0 ? u - 1 : u;
  f(starts[lo0], starts[u + 1]);
  if (x == 0 && ns >= 2) f(starts[ns >= 3 ? ns - 2 : ns - 1], starts[ns]);
}

// Sets the bits of the tile's elements that the chunk from `base` touches.
__device__ __forceinline__ void touch_bits(uint32_t* bits, uint32_t base, uint32_t x0,
                                           uint32_t len, uint32_t M, uint32_t Z) {
  auto span = [&](uint32_t lo, uint32_t hi) {  // [lo, hi) of the array; hi <= M < 2^31
    lo = lo > x0 ? lo - x0 : 0u;
    hi = hi > x0 ? (hi - x0 < len ? hi - x0 : len) : 0u;
    while (lo < hi) {
      const uint32_t end = (lo | 31u) + 1 < hi ? (lo | 31u) + 1 : hi;
      const uint32_t n = end - lo;
      atomicOr(&bits[lo >> 5], (n == 32 ? 0xffffffffu : (1u << n) - 1) << (lo & 31));
      lo = end;
    }
  };
  const uint32_t end = base + Z;  // < 2^32
  span(base, end < M ? end : M);
  if (end > M) span(0, end - M);
}

// counts[x] = elements of tile x that some record touches.
__global__ __launch_bounds__(kTileThreads) void tile_count_kernel(
    const uint32_t M, const uint32_t Z, const int shift, const uint32_t* __restrict__ keys,
    const uint32_t* __restrict__ totals, uint32_t* __restrict__ counts) {
  __shared__ uint32_t starts[kTileThreads + 1], wsum[kTileThreads / kWave];
  __shared__ uint32_t bits[kTileWords];
  __shared__ uint32_t sum;
  const int tid = threadIdx.x;
  const uint32_t x = blockIdx.x, x0 = x << kTileShift;
  const uint32_t len = M - x0 < kTileLen ? M - x0 : kTileLen;
  if (tid < static_cast<int>(kTileWords)) bits[tid] = 0;
  if (tid == 0) sum = 0;
  super_starts(starts, wsum, totals);
  for_runs(x, M, shift, starts, [&](uint32_t lo, uint32_t hi) {
    for (uint32_t r0 = lo; r0 < hi; r0 += kTileStage * kTileThreads) {
      uint32_t base[kTileStage];
#pragma unroll
      for (int v = 0; v < kTileStage; ++v) {
        const uint32_t r = r0 + v * kTileThreads + tid;
        base[v] = r < hi ? keys[r] : kNoChunk;
      }
#pragma unroll 1
      for (int v = 0; v < kTileStage; ++v) {
        uint32_t bv = base[0];
#pragma unroll
        for (int q = 1; q < kTileStage; ++q) bv = q == v ? base[q] : bv;
        if (bv != kNoChunk && chunk_reaches(bv, Z, M, x0, len)) touch_bits(bits, bv, x0, len, M, Z);
      }
    }
  });
  __syncthreads();
  if (tid < static_cast<int>(kTileWords)) atomicAdd(&sum, static_cast<uint32_t>(__popc(bits[tid])));
  __syncthreads();
  if (tid == 0) counts[x] = sum;
}

// What the apply step does with a tile: write the list (LIST), or update.
struct TileList {
  uint32_t* locations;
  float* values;
  int64_t capacity;
  int64_t* num_unique;
  const uint32_t* counts;
};

// A lane group of G lanes owns kRange consecutive elements of the tile, at least
// a chunk's length.  The records reaching the tile are staged in LDS ordered by
// the range their chunk begins in (bin 0: before the tile, or wrapping past
// M), stably, by counting: the records a group has to look at are then those
// of two neighbouring bins.
template <int G, bool LIST, typename WT, bool ADAGRAD>
__global__ __launch_bounds__(kTileThreads, 5) void tile_apply_kernel(
    const uint32_t M, const uint32_t Z, const int shift, const uint32_t* __restrict__ keys,
    const uint32_t* __restrict__ ids, const uint32_t* __restrict__ totals,
    const float* __restrict__ sums, const TileList list, WT* __restrict__ w,
    float* __restrict__ s, const float lr, const float eps) {
  constexpr int kGroups = kTileThreads / G;
  constexpr uint32_t kRange = kTileLen / kGroups;
  constexpr int kBins = kGroups + 1;
  constexpr int kBinBits = G == 8 ? 6 : G == 16 ? 5 : G == 32 ? 4 : 3;
  static_assert(kBins <= (1 << kBinBits) && kTileWords <= kTileThreads, "bins and words fit");
  constexpr int kRows = kTileStage * kTileThreads / kWave;  // wavefront-sized rows of a stage
  __shared__ __align__(16) float acc[kTileLen];
  __shared__ uint32_t starts[kTileThreads + 1];
  __shared__ uint32_t sbase[kTileStage * kTileThreads], sid[kTileStage * kTileThreads];
  __shared__ uint32_t cnt[kRows][kBins];
  __shared__ uint32_t first[kBins + 1];
  __shared__ uint32_t bits[LIST ? kTileWords : 1], wpre[LIST ? kTileWords : 1];
  __shared__ uint32_t wsum[kTileThreads / kWave];
  __shared__ uint32_t before;
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & (kWave - 1), gl = tid % G;
  const uint32_t x = blockIdx.x, x0 = x << kTileShift;
  const uint32_t len = M - x0 < kTileLen ? M - x0 : kTileLen;
  if (LIST && tid < static_cast<int>(kTileWords)) bits[tid] = 0;
  super_starts(starts, wsum, totals);
  const int grp = tid / G;
  const uint32_t q0 = static_cast<uint32_t>(grp) * kRange;  // the group's range, in the tile
  const uint32_t r0 = x0 + q0;
  const uint32_t rlen = q0 >= len ? 0u : (len - q0 < kRange ? len - q0 : kRange);
  float* mine = acc + q0;
  bool any = false;
  for_runs(x, M, shift, starts, [&](uint32_t lo, uint32_t hi) {
    for (uint32_t c0 = lo; c0 < hi; c0 += kTileStage * kTileThreads) {
      uint32_t base[kTileStage], id[kTileStage];
      int bin[kTileStage];
      uint32_t rank[kTileStage];
      bool some = false;
#pragma unroll
      for (int v = 0; v < kTileStage; ++v) {
        const uint32_t r = c0 + v * kTileThreads + tid;
        base[v] = r < hi ? keys[r] : kNoChunk;
        id[v] = r < hi ? ids[r] : 0u;
        bin[v] = -1;
        if (base[v] != kNoChunk && chunk_reaches(base[v], Z, M, x0, len)) {
          const uint32_t o = base[v] - x0;  // below len: begins in the tile
          bin[v] = o < len ? static_cast<int>(o / kRange) + 1 : 0;
        }
        some |= bin[v] >= 0;
      }
      if (!__syncthreads_or(some)) continue;  // (also: the previous stage has been read)
      if (!any)
        for (uint32_t q = tid; q < kTileLen / 4; q += kTileThreads)
          reinterpret_cast<float4*>(acc)[q] = float4{0.f, 0.f, 0.f, 0.f};
      any = true;  // the same for the whole workgroup
      for (int q = tid; q < kRows * kBins; q += kTileThreads) (&cnt[0][0])[q] = 0;
      __syncthreads();
#pragma unroll
      for (int v = 0; v < kTileStage; ++v) {
        const bool in = bin[v] >= 0;
        uint64_t eq = __ballot(in);
#pragma unroll
        for (int bit = 0; bit < kBinBits; ++bit) {
          const uint64_t m = __ballot((bin[v] >> bit) & 1);
          eq &= ((bin[v] >> bit) & 1) ? m : ~m;
        }
        rank[v] = static_cast<uint32_t>(__popcll(eq & ((1ull << lane) - 1)));
        if (in && rank[v] == 0) cnt[v * (kTileThreads / kWave) + wv][bin[v]] = __popcll(eq);
      }
      __syncthreads();
      if (tid < kBins) {  // rows of a bin, in order
        uint32_t run = 0;
#pragma unroll
        for (int q = 0; q < kRows; ++q) {
          const uint32_t c = cnt[q][tid];
          cnt[q][tid] = run;
          run += c;
        }
        first[tid + 1] = run;
        if (tid == 0) first[0] = 0;
      }
      __syncthreads();
      if (wv == 0) {  // bins in order (at most 33)
        uint32_t f = lane < kBins ? first[lane + 1] : 0u;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
          const uint32_t y = __shfl_up(f, off);
          if (lane >= off) f += y;
        }
        if (lane < kBins) first[lane + 1] = f;
      }
      __syncthreads();
      const uint32_t n = first[kBins];
#pragma unroll
      for (int v = 0; v < kTileStage; ++v) {
        if (bin[v] < 0) continue;
        const uint32_t at = first[bin[v]] + cnt[v * (kTileThreads / kWave) + wv][bin[v]] + rank[v];
        sbase[at] = base[v];
        sid[at] = id[v];
      }
      __syncthreads();
      if (LIST)
        for (uint32_t q = tid; q < n; q += kTileThreads) touch_bits(bits, sbase[q], x0, len, M, Z);
      // bins grp (chunks beginning in the range before) and grp + 1 (in this one)
      const uint32_t b0 = rlen ? first[grp] : 0u, b1 = rlen ? first[grp + 2] : 0u;
      for (uint32_t i0 = b0; __ballot(i0 < b1); i0 += kTileBatch) {
        uint32_t bs[kTileBatch], at[kTileBatch];
#pragma unroll
        for (int v = 0; v < kTileBatch; ++v) {
          const uint32_t q = i0 + v < b1 ? i0 + v : 0u;
          bs[v] = sbase[q];
          at[v] = sid[q] * Z;  // N * d < 2^32
        }
        for (uint32_t k0 = 0; k0 < Z; k0 += G) {
          const uint32_t k = k0 + gl;
          float x4[kTileBatch];
          uint32_t off[kTileBatch];
#pragma unroll
          for (int v = 0; v < kTileBatch; ++v) {
            uint32_t m = bs[v] + k;  // base < M and k < Z <= M: no overflow
            if (m >= M) m -= M;
            off[v] = i0 + v < b1 && k < Z ? m - r0 : 0xffffffffu;  // below rlen: in the range
            x4[v] = off[v] < rlen ? sums[static_cast<uint64_t>(at[v]) + k] : 0.f;
          }
#pragma unroll
          for (int v = 0; v < kTileBatch; ++v) {
            if (off[v] < rlen) mine[off[v]] += x4[v];
            // chunks of two records may overlap at other lanes' elements
            wave_lds_fence();
          }
        }
      }
    }
  });
  __syncthreads();
  if (LIST) {
    // output slots: the touched elements of earlier tiles, of earlier words
    uint32_t b = 0;
    for (uint32_t v = tid; v < x; v += kTileThreads) b += list.counts[v];
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) b += __shfl_xor(b, off);
    if (tid == 0) before = 0;
    __syncthreads();
    if (lane == 0 && b) atomicAdd(&before, b);
    const uint32_t pc = tid < static_cast<int>(kTileWords) ? __popc(bits[tid]) : 0u;
    uint32_t incl = pc;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const uint32_t y = __shfl_up(incl, off);
      if (lane >= off) incl += y;
    }
    if (lane == kWave - 1) wsum[wv] = incl;
    __syncthreads();
    uint32_t pre = 0;
    for (int w2 = 0; w2 < wv; ++w2) pre += wsum[w2];
    if (tid < static_cast<int>(kTileWords)) wpre[tid] = pre + incl - pc;
    __syncthreads();
    if (tid == kTileThreads - 1 && x == gridDim.x - 1)
      *list.num_unique = static_cast<int64_t>(before) + pre + incl;
  }
  if (!any) return;
  if (LIST) {
#pragma unroll 4
    for (uint32_t i = tid; i < len; i += kTileThreads) {
      const uint32_t word = bits[i >> 5], bit = i & 31;
      const int64_t k = static_cast<int64_t>(before) + wpre[i >> 5] +
                        __popc(word & ((1u << bit) - 1));
      if (((word >> bit) & 1u) && k < list.capacity) {
        list.locations[k] = x0 + i;
        list.values[k] = acc[i];
      }
    }
    return;
  }
  // kTileOpt elements per lane: weights and states of those with G != 0
  // requested before any is updated
  constexpr int kTileOpt = 8;
#pragma unroll 1
  for (uint32_t i0 = tid; i0 < len; i0 += kTileOpt * kTileThreads) {
    float g[kTileOpt], wo[kTileOpt], so[kTileOpt];
#pragma unroll
    for (int v = 0; v < kTileOpt; ++v) {
      const uint32_t i = i0 + v * kTileThreads;
      g[v] = i < len ? acc[i] : 0.f;
    }
#pragma unroll
    for (int v = 0; v < kTileOpt; ++v) {
      const int64_t m = static_cast<int64_t>(x0) + i0 + v * kTileThreads;
      wo[v] = g[v] != 0.f ? load_weight64(w, m) : 0.f;
      so[v] = ADAGRAD && g[v] != 0.f ? s[m] : 0.f;
    }
#pragma unroll
    for (int v = 0; v < kTileOpt; ++v)
      if (g[v] != 0.f)
        update_loaded<WT, ADAGRAD>(w, s, static_cast<int64_t>(x0) + i0 + v * kTileThreads, g[v],
                                   wo[v], so[v], lr, eps);
  }
}

static uint32_t tiles_of(const KParams& p) {
  return static_cast<uint32_t>((static_cast<uint64_t>(p.M) + kTileLen - 1) >> kTileShift);
}

// sums, the two record buffers, the radix scratch, the counts of the list,
// 1 / |bag| of a batch that is not one item per bag
size_t tile_workspace_bytes(const KParams& p, bool list) {
  const uint64_t n = static_cast<uint64_t>(p.N) * p.C;
  return static_cast<size_t>(p.N) * p.d * 4 + n * 16 + radix_scratch_bytes(static_cast<int64_t>(n)) +
         (list ? static_cast<size_t>(tiles_of(p)) * 4 : 0) +
         (p.mean && !keygen_counts(p) ? static_cast<size_t>(p.num_bags) * 4 : 0) + 7 * 256;
}

struct TileRecords {
  const float* sums;
  const uint32_t *keys, *ids, *totals;
  uint32_t* counts;
  int shift;
};

static hipError_t tile_records(const KParams& p, const void* indices, const void* offsets,
                               const void* grad, void* workspace, TileRecords* out,
                               hipStream_t stream) {
  const uint64_t n = static_cast<uint64_t>(p.N) * p.C;
  char* cur = static_cast<char*>(workspace);
  auto carve = [&](uint64_t words) {
    uint32_t* q = reinterpret_cast<uint32_t*>(cur);
    cur += (words * 4 + 255) & ~uint64_t(255);
    return q;
  };
  float* sums = reinterpret_cast<float*>(carve(static_cast<uint64_t>(p.N) * p.d));
  uint32_t *k0 = carve(n), *v0 = carve(n), *k1 = carve(n), *v1 = carve(n);
  uint32_t* scratch = reinterpret_cast<uint32_t*>(cur);
  cur += (radix_scratch_bytes(static_cast<int64_t>(n)) + 255) & ~size_t(255);
  // Lookups of a batch that is not one item per bag: their keys and rows in the
  // buffers that the radix pass writes later.
  hipError_t e = hipSuccess;
  GroupedPairs pairs;
  const bool keygen = !keygen_counts(p);
  if (keygen) {
    float* inv_len = nullptr;
    if (p.mean) inv_len = reinterpret_cast<float*>(carve(p.num_bags));
    e = launch_keygen(p, indices, offsets, k1, v1, inv_len, stream);
    pairs.keys = k1;
    pairs.rows = v1;
    pairs.inv_len = inv_len;
  }
  if (e == hipSuccess)
    e = launch_piece_records(sums, p, indices, offsets, keygen ? &pairs : nullptr, grad, k0, v0,
                             stream);
  if (e != hipSuccess) return e;
  const int shift = super_shift(p.M);
  e = radix_sort_pairs(k0, v0, k1, v1, static_cast<int64_t>(n), 8, scratch, stream, nullptr, false,
                       shift);
  *out = TileRecords{sums, k0, v0, radix_totals(scratch, static_cast<int64_t>(n)),
                     reinterpret_cast<uint32_t*>(cur), shift};  // counts: the list only
  return e;
}

template <bool LIST, typename WT, bool ADAGRAD>
static hipError_t launch_apply(const KParams& p, const TileRecords& r, const TileList& list, WT* w,
                               float* s, float lr, float eps, hipStream_t stream) {
  const dim3 grid(tiles_of(p)), block(kTileThreads);
  const auto kernel = p.Z <= 8    ? tile_apply_kernel<8, LIST, WT, ADAGRAD>
                      : p.Z <= 16 ? tile_apply_kernel<16, LIST, WT, ADAGRAD>
                      : p.Z <= 32 ? tile_apply_kernel<32, LIST, WT, ADAGRAD>
                                  : tile_apply_kernel<64, LIST, WT, ADAGRAD>;
  hipLaunchKernelGGL(kernel, grid, block, 0, stream, p.M, p.Z, r.shift, r.keys, r.ids, r.totals,
                     r.sums, list, w, s, lr, eps);
  return hipGetLastError();
}

hipError_t launch_gradient_tiles(const KParams& p, const void* indices, const void* offsets,
                                 const void* grad, void* workspace, uint32_t* locations,
                                 float* values, int64_t capacity, int64_t* num_unique,
                                 hipStream_t stream) {
  TileRecords r;
  hipError_t e = tile_records(p, indices, offsets, grad, workspace, &r, stream);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(tile_count_kernel, dim3(tiles_of(p)), dim3(kTileThreads), 0, stream, p.M, p.Z,
                     r.shift, r.keys, r.totals, r.counts);
  const TileList list{locations, values, capacity, num_unique, r.counts};
  return launch_apply<true, float, false>(p, r, list, nullptr, nullptr, 0.f, 0.f, stream);
}

hipError_t launch_update_tiles(const KParams& p, const void* indices, const void* offsets,
                               const void* grad, void* workspace, void* w, bool bf16, float* state,
                               float lr, float eps, hipStream_t stream) {
  TileRecords r;
  const hipError_t e = tile_records(p, indices, offsets, grad, workspace, &r, stream);
  if (e != hipSuccess) return e;
  const TileList none{};
  if (bf16) {
    uint16_t* wb = static_cast<uint16_t*>(w);
    return state ? launch_apply<false, uint16_t, true>(p, r, none, wb, state, lr, eps, stream)
                 : launch_apply<false, uint16_t, false>(p, r, none, wb, state, lr, eps, stream);
  }
  float* wf = static_cast<float*>(w);
  return state ? launch_apply<false, float, true>(p, r, none, wf, state, lr, eps, stream)
               : launch_apply<false, float, false>(p, r, none, wf, state, lr, eps, stream);
}

// Where it applies: batches whose general pipeline is a chain of launches
// (pieces_fit), chunks of at least 4 elements (a record with fewer
// leaves most of its lane group idle) that fit a lane group's range, an array
// of two whole tiles (a chunk that begins in tile 0 then does not wrap around
// into it: a record stands in one bin), few enough tiles (each
// costs a workgroup, and the list sums the counts of the tiles before) and
// few enough records per tile (one workgroup adds them).  Kernel time of the call, general / by tile:
// 8192 lookups, d = 64, Z = 16, 16 M elements 145 / 51 us; the list of 26 x 4096 Zipf lookups on 4 M
// elements 141 / 83 us (75 us with records of the batch's own order, whose sums lie up to 1.23 times
// farther from 64-bit ones), 10240 uniform ones with d = 128, Z = 32 on 1.28 M elements 137 / 55 us.
// The limits keep a margin to where the two meet (general / by tile, 8192 lookups, d = 64, Z = 16):
// list of 4096 tiles 139 / 67 us, 8192 137 / 104 us, 16384 135 / 188 us; update of 16384
// tiles 136 / 84 us, 32768 138 / 118 us, 60000 136 / 164 us; records per tile, 32768 lookups: update 512
// 129 / 59 us, 2048 122 / 72 us, 4096 123 / 95 us, 8192 124 / 144 us, the list of 106496 lookups 832
// 138 / 95 us, 3328 134 / 119 us, 6656 138 / 165 us (uniform addresses; a skewed batch has more in
// some tiles).
constexpr int64_t kTileMaxRecords = 1024;  // per tile
constexpr int64_t kTileMaxList = 4096, kTileMaxUpdate = 16384;  // tiles
bool sparse_by_tile(const KParams& p, bool list) {
  const int64_t tiles = tiles_of(p);
  return pieces_fit(p) && p.Z >= 4 && p.Z <= 1024 && p.M >= 2 * kTileLen &&
         tiles <= (list ? kTileMaxList : kTileMaxUpdate) &&
         p.N * static_cast<int64_t>(p.C) <= tiles * kTileMaxRecords;
}

}  // namespace pss
