// Forward of the PSS layer: hash -> chunk gather -> sum-pool (paper Sec. 2.4
// forward(i) = (S e_i)^T M with the ROBE-Z mapping of Sec. 2.5).
//
// Four kernels, all bound by the memory system (rows written, chunks
// gathered):
//   rows   one item per bag (as many items as bags): a wavefront takes a run
//          of consecutive bags of a table, a lane group holds one row;
//   bags   any other batch: a lane group pools one bag;
//   long   few long bags: a workgroup pools one bag;
//   tiled  one item per bag, at least 2^20 bags and an array beyond the
//          aggregate L2: a wavefront takes 64 bags, sorts their tokens and
//          gathers each distinct one once.
// Rows are written with non-temporal stores: the output stream must not
// evict the shared array from the L2s and the memory-side cache (plain
// stores: 254 against 173 us on 26 x 65536 rows of 512 bytes).
//
// Options: SIGN (template) multiplies each chunk by its sign factor and skips
// chunks of factor 0; mean pooling divides a finished row by the bag's item
// count; rows may be stored as bfloat16 (round to nearest even); indices and
// offsets may be int32.
#include "pss_launch.hpp"

namespace pss {

// The row kernels give each XCD a contiguous share of the batch (see
// xcd_block) whatever the array's size: its L2 then holds the hot tokens of
// about 1/kXcds of the tables (26 x 65536 one-hot rows, 10 MB array: 173 ->
// 169 us, 26 x 16384: 48.9 -> 45.4 us).
//
// Workgroups are dispatched round-robin over the chip's XCDs (workgroup b on
// XCD b mod kXcds), each with an L2 of its own.  grid.x is a multiple of
// kXcds; any other dispatch order only changes which L2 sees which part.
__device__ __forceinline__ uint64_t xcd_block() {
  return (blockIdx.x % kXcds) * static_cast<uint64_t>(gridDim.x / kXcds) + blockIdx.x / kXcds;
}

// Arrays beyond the chip's aggregate L2 (8 x 4 MiB): see tiled_applies.
constexpr uint64_t kL2Bytes = 32ull << 20;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));        // 4-byte aligned
typedef uint32_t u32x2u __attribute__((ext_vector_type(2), aligned(2)));     // 2-byte aligned

__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, int lane) {
  const uint32_t lo = readlane_u32(static_cast<uint32_t>(v), lane);
  const uint32_t hi = readlane_u32(static_cast<uint32_t>(v >> 32), lane);
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

// Cached loads of indices[e] / offsets[g] (wave-uniform choice of width): a
// line of indices serves several lane groups.
__device__ __forceinline__ uint32_t index_at(const void* idx, uint64_t e, uint32_t i32) {
  return i32 ? static_cast<uint32_t>(static_cast<const int32_t*>(idx)[e])
             : static_cast<uint32_t>(static_cast<const int64_t*>(idx)[e]);
}
__device__ __forceinline__ int64_t offset_at(const void* off, uint64_t g, uint32_t i32) {
  return i32 ? static_cast<int64_t>(static_cast<const int32_t*>(off)[g])
             : static_cast<const int64_t*>(off)[g];
}

// What the first kTouchBlocks workgroups (one per compute unit) read once before their
// own work, in whole 16-byte pieces lying inside it, at the streaming rate:
// later reads then find it in the memory-side cache.
//  index  the batch's index and offset arrays.  After a backward they lie
//         in HBM, where the index loads of the later wavefronts would queue
//         behind the write stream (26 x 65536 rows in a training step:
//         252 -> 176 us; 26 x 16384: 58.8 -> 46.6 us).  For batches of several
//         generations of workgroups.
//  bytes  the shared array, when it is larger than the L2s but fits the
//         memory-side cache beside other data and the batch gathers 8 times its size or
//         more.  Where other work has evicted it since its last use, each
//         of its lines would otherwise be fetched by a random read (128 MB
//         array, 26 x 262144 rows of 256 bytes: 970 -> 751 us, the training step
//         2156 -> 1932 us).  Where it has not (the same step over and over, nothing
//         else running), the pass costs 17 to 28 us of 1860.  Rows of 256 bytes, forward
//         without / with the pass, array evicted and still cached: 128 MB gathered
//         twice 194 / 166 and 115 / 132 us, 4 times 358 / 286 and 231 / 246 us, 8 times
//         580 / 502 and 439 / 455 us, 16 times 1011 / 939 and 862 / 874 us: from 8 times on what
//         it may cost is below 4%.  192 MB, 8 times 882 / 780 and 690 / 719 us; a 256 MB array
//         does not stay cached either way (1174 / 1037 and 1116 / 953 us) and is left to its
//         gathers: beside other data the pass would evict its own lines.
struct Touch {
  uint32_t index = 0;
  uint64_t bytes = 0;
};
constexpr uint32_t kTouchBlocks = 256;
constexpr uint64_t kTouchBags = 1ull << 18;
constexpr uint64_t kTouchMaxBytes = 192ull << 20;  // of the 256 MiB memory-side cache
__device__ __forceinline__ void touch_batch(const KParams& p, const void* __restrict__ w,
                                            const void* __restrict__ indices,
                                            const void* __restrict__ offsets,
                                            void* __restrict__ out, const Touch& touch) {
  if (blockIdx.x >= kTouchBlocks || blockIdx.y != 0) return;
  if (!touch.index && !touch.bytes) return;
  const uint64_t es = p.idx32 ? 4 : 8;
  uint32_t seen = 0;
  auto read = [&](const void* base, uint64_t bytes) {
    const uint64_t a0 = reinterpret_cast<uint64_t>(base);
    const uint64_t c_lo = (a0 + 15) / 16, c_end = (a0 + bytes) / 16;
    constexpr int kPieces = 8;  // requested before any is used (16 take the kernels past 64 VGPRs)
    const uint64_t blocks = gridDim.x < kTouchBlocks ? gridDim.x : kTouchBlocks;
    const uint64_t stride = blocks * kBlockThreads;
    for (uint64_t c0 = c_lo + static_cast<uint64_t>(blockIdx.x) * kBlockThreads + threadIdx.x;
         c0 < c_end; c0 += kPieces * stride) {
      uint4 v4[kPieces];
#pragma unroll
      for (int k = 0; k < kPieces; ++k) {
        const uint64_t c = c0 + k * stride;
        v4[k] = c < c_end ? *reinterpret_cast<const uint4*>(c * 16) : uint4{0u, 0u, 0u, 0u};
      }
#pragma unroll
      for (int k = 0; k < kPieces; ++k) seen ^= v4[k].x ^ v4[k].y ^ v4[k].z ^ v4[k].w;
    }
  };
  if (touch.index) {
    read(indices, static_cast<uint64_t>(p.N) * es);
    read(offsets, (p.num_bags + 1) * es);
  }
  if (touch.bytes) read(w, touch.bytes);
  // never true (N >= 0): keeps the loads
  if (seen == 0x9e3779b9u && p.N < 0) static_cast<uint32_t*>(out)[threadIdx.x] = seen;
}

// ---------------------------------------------------------------------------
// Rows and bags.  LPB lanes (a power of two) hold one pooled row, V
// consecutive elements per lane, so that a wavefront works on GP = 64 / LPB
// rows at once and one load per lane gathers a whole item.  V = 4 (one
// 16-byte load; 8 bytes of bfloat16) when the chunk size is a multiple of 4: a
// chunk then never splits a lane's elements.  V = 1 otherwise.  Wider rows
// are cut into slabs of LPB * V elements (blockIdx.y).
//
// The chunk entries (hashed base and sign) of the items in hand are
// evaluated once each, spread over the lanes, into a wave-private LDS table:
// the lanes that share a chunk would otherwise all repeat its modular
// reductions.
// ---------------------------------------------------------------------------

// Items a lane group of the bags kernel has in flight: 8 pieces of 16 bytes
// per lane keep it within 64 VGPRs, 8 wavefronts per SIMD.  16 in flight (half the
// wavefronts) gained 2% on bags of 20 items and lost 15% on shorter ones; 4
// lost 1% on the long bags.
template <int LPB> constexpr int bag_batch() { return LPB >= 8 ? 8 : 4; }
// Rows a lane group of the one-row-per-bag kernel holds: more wavefronts of
// fewer rows each hide the index load's latency better.  8 / 4 rows: 3328
// rows of 512 bytes 4.2 / 3.6 us, 26 x 2048 10.7 / 9.2 us, 26 x 65536 183 / 180 us a
// lookup pass, 401 / 398 us a training step.
constexpr int kRowBatch = 4;

template <int V> struct Piece;
template <> struct Piece<4> { typedef f32x4 type; };
template <> struct Piece<1> { typedef float type; };

template <bool SIGN>
__device__ __forceinline__ uint32_t entry_base(uint32_t ent) {
  return SIGN ? (ent != kSkip ? ent & 0x7fffffffu : 0u) : ent;
}

// Whether elements kk .. kk + V - 1 of the chunk of `ent` run past the end
// of the array in the middle of a lane's piece (a single element wraps as a
// whole).
template <int V, bool SIGN>
__device__ __forceinline__ bool splits(uint32_t ent, uint32_t kk, uint32_t M) {
  return V > 1 && entry_base<SIGN>(ent) + kk + (V - 1) >= M;  // < 2M <= 2^32
}

// Elements kk .. kk + V - 1 of the chunk of `ent`, widened, unsigned; the
// piece must not be split by the end of the array.
template <typename WT, int V, bool SIGN>
__device__ __forceinline__ typename Piece<V>::type gather(const WT* __restrict__ w, uint32_t ent,
                                                          uint32_t kk, uint32_t M) {
  const uint32_t base = entry_base<SIGN>(ent);
  if constexpr (V == 1) {
    return load_weight(w, wrap_add(base, kk, M));
  } else {
    const uint32_t m = SIGN && ent == kSkip ? 0u : base + kk;
    if constexpr (sizeof(WT) == 4) {
      return *reinterpret_cast<const f32x4u*>(reinterpret_cast<const float*>(w) + m);
    } else {
      const u32x2u b = *reinterpret_cast<const u32x2u*>(w + m);
      return f32x4{__uint_as_float(b.x << 16), __uint_as_float(b.x & 0xffff0000u),
                   __uint_as_float(b.y << 16), __uint_as_float(b.y & 0xffff0000u)};
    }
  }
}

// The same for any piece, element by element.
template <typename WT, int V, bool SIGN>
__device__ __forceinline__ typename Piece<V>::type gather_split(const WT* __restrict__ w,
                                                                uint32_t ent, uint32_t kk,
                                                                uint32_t M) {
  const uint32_t base = entry_base<SIGN>(ent);
  if constexpr (V == 1) {
    return load_weight(w, wrap_add(base, kk, M));
  } else {
    return f32x4{load_weight(w, wrap_add(base, kk, M)), load_weight(w, wrap_add(base, kk + 1, M)),
                 load_weight(w, wrap_add(base, kk + 2, M)), load_weight(w, wrap_add(base, kk + 3, M))};
  }
}

__device__ __forceinline__ float flip(float x, uint32_t neg) {
  return __uint_as_float(__float_as_uint(x) ^ neg);
}
template <bool SIGN>
__device__ __forceinline__ float sign_piece(float x, uint32_t ent) {
  if (!SIGN) return x;
  return ent == kSkip ? 0.f : flip(x, ent & 0x80000000u);
}
template <bool SIGN>
__device__ __forceinline__ f32x4 sign_piece(f32x4 x, uint32_t ent) {
  if (!SIGN) return x;
  if (ent == kSkip) return f32x4{0.f, 0.f, 0.f, 0.f};
  const uint32_t neg = ent & 0x80000000u;
  return f32x4{flip(x.x, neg), flip(x.y, neg), flip(x.z, neg), flip(x.w, neg)};
}

// Elements e .. of the output: float32, or bfloat16 rounded to nearest even.
__device__ __forceinline__ void store_piece(void* __restrict__ out, uint64_t e, float v,
                                            uint32_t bf16) {
  if (bf16)
    __builtin_nontemporal_store(f32_to_bf16_rne(v), static_cast<uint16_t*>(out) + e);
  else
    __builtin_nontemporal_store(v, static_cast<float*>(out) + e);
}
__device__ __forceinline__ void store_piece(void* __restrict__ out, uint64_t e, f32x4 v,
                                            uint32_t bf16) {
  if (bf16) {
    const u32x2u x = {static_cast<uint32_t>(f32_to_bf16_rne(v.x)) |
                          (static_cast<uint32_t>(f32_to_bf16_rne(v.y)) << 16),
                      static_cast<uint32_t>(f32_to_bf16_rne(v.z)) |
                          (static_cast<uint32_t>(f32_to_bf16_rne(v.w)) << 16)};
    __builtin_nontemporal_store(x, reinterpret_cast<u32x2u*>(static_cast<uint16_t*>(out) + e));
  } else {
    __builtin_nontemporal_store(v, reinterpret_cast<f32x4u*>(static_cast<float*>(out) + e));
  }
}

// The lane's elements of a row: dims c .. c + V - 1 of slab blockIdx.y, in
// chunk jc at offset kk; the slab meets the Cs chunks from j0 on (Cs <= LPB:
// every chunk holds at least V dims of it).
template <int V, int LPB>
struct RowLane {
  uint32_t c, kk, jc, j0, Cs;
  bool act;
  __device__ __forceinline__ RowLane(const KParams& p, int gl) {
    const uint32_t c0 = blockIdx.y * (LPB * V);
    c = c0 + static_cast<uint32_t>(gl) * V;
    act = c < p.d;
    j0 = c0 / p.Z;
    const uint32_t dend = p.d < c0 + LPB * V ? p.d : c0 + LPB * V;
    Cs = (dend - 1) / p.Z - j0 + 1;
    const uint32_t cc = act ? c : c0;
    jc = cc / p.Z;
    kk = cc - jc * p.Z;
  }
};

// Chunk entry of chunk j of the item with hash h.
template <bool SIGN>
__device__ __forceinline__ uint32_t item_entry(const KParams& p, uint32_t h, uint32_t j) {
  const uint32_t base = fast_mod(add_mod_p(h, chunk_step(p.a, j)), p.fm_c, p.M);
  if (!SIGN) return base;
  return chunk_entry<SIGN>(
      base, add_mod_p(sign_hash0(h, p.s_alpha, p.s_beta), chunk_step(p.a2, j)), p);
}

// Any batch: one lane group per bag, items in order.  Lane i < U of the
// group requests the index of item i of the next batch of U items while this
// one is gathered.  Measured against the tiled kernel that pooled a tile of
// 64 bags per wavefront before: 23101 bags of 9 items on average (d = 96, Z = 8,
// bfloat16) 111 -> 24 us (that kernel filled 361 wavefronts), 852 K bags of 20
// items (d = 64, Z = 16, 64 MB array) 889 -> 811 us: the rate of random
// 64-byte requests beyond the L2s.
template <typename WT, int V, int LPB, bool SIGN>
__global__ __launch_bounds__(kBlockThreads, 8) void forward_bags_kernel(
    const WT* __restrict__ w, const KParams p, const void* __restrict__ indices,
    const void* __restrict__ offsets, void* __restrict__ out, const uint64_t wave0,
    const KeygenOut kg) {
  constexpr int U = bag_batch<LPB>();
  constexpr int GP = kWave / LPB;
  static_assert(U <= LPB, "one lane per item of the batch");
  __shared__ uint32_t tab_all[kWavesPerBlock][GP * U * LPB];
  const int lane = threadIdx.x & (kWave - 1);
  const int grp = lane / LPB, gl = lane % LPB;
  const uint64_t wave = wave0 + xcd_block() * kWavesPerBlock + (threadIdx.x >> 6);
  if (wave * GP >= p.num_bags) return;  // whole wavefront
  uint32_t* tab = tab_all[threadIdx.x >> 6] + grp * U * LPB;
  const uint64_t g = wave * GP + grp;
  const bool live = g < p.num_bags;
  const RowLane<V, LPB> rl(p, gl);
  const uint32_t jl = rl.jc - rl.j0;
  int64_t e = 0, e1 = 0;
  uint32_t t = 0, b = 0;
  if (live) {
    e = offset_at(offsets, g, p.idx32);
    e1 = offset_at(offsets, g + 1, p.idx32);
    e = e < 0 ? 0 : (e > p.N ? p.N : e);
    e1 = e1 < 0 ? 0 : (e1 > p.N ? p.N : e1);
    if (e1 < e) e1 = e;
    t = static_cast<uint32_t>(g) / p.B;  // bags number fewer than 2^32
    b = static_cast<uint32_t>(g) - t * p.B;
  }
  const uint32_t tC = t * p.C;
  uint32_t left = static_cast<uint32_t>(e1 - e);  // N < 2^32
  const uint32_t len = left;
  // the lookups' keys and rows for the backward, when asked for
  const bool keys = kg.keys != nullptr && blockIdx.y == 0;
  const uint32_t row = b * p.T + t;
  if (keys && p.mean && gl == 0 && len) kg.inv_len[row] = 1.f / static_cast<float>(len);
  typename Piece<V>::type acc = {};
  uint32_t ix = 0;
  if (gl < U && static_cast<uint32_t>(gl) < left)
    ix = index_at(indices, static_cast<uint64_t>(e + gl), p.idx32);
  while (__ballot(left != 0)) {
    const uint32_t n = left < U ? left : U;
    const uint32_t h0 = item_hash(ix, tC, p.TC, p.a, p.b);
    if (gl < U && static_cast<uint32_t>(U + gl) < left)
      ix = index_at(indices, static_cast<uint64_t>(e + U + gl), p.idx32);
    if (keys && static_cast<uint32_t>(gl) < n) {
      kg.keys[e + gl] = h0;
      kg.rows[e + gl] = row;
    }
#pragma unroll 1
    for (uint32_t k0 = 0; __ballot(k0 < n * rl.Cs); k0 += LPB) {
      const uint32_t k = k0 + gl;
      const uint32_t i = k / rl.Cs, j = k - i * rl.Cs;
      const uint32_t h = __shfl(h0, grp * LPB + static_cast<int>(i < U ? i : 0u));
      if (k < n * rl.Cs) tab[k] = item_entry<SIGN>(p, h, rl.j0 + j);
    }
    wave_lds_fence();
    uint32_t ent[U];
    bool split = false;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // past the bag's end: its last item again (element 0 for an empty bag)
      const uint32_t uu = static_cast<uint32_t>(u) < n ? u : (n ? n - 1 : 0u);
      ent[u] = n ? tab[uu * rl.Cs + jl] : 0u;
      split |= n && splits<V, SIGN>(ent[u], rl.kk, p.M);
    }
    if (__ballot(split)) {  // a piece runs past the end of the array
#pragma unroll 1
      for (uint32_t u = 0; u < n; ++u) {
        const uint32_t en = tab[u * rl.Cs + jl];
        acc += sign_piece<SIGN>(gather_split<WT, V, SIGN>(w, en, rl.kk, p.M), en);
      }
    } else {
      typename Piece<V>::type v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = gather<WT, V, SIGN>(w, ent[u], n ? rl.kk : 0u, p.M);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (static_cast<uint32_t>(u) < n) acc += sign_piece<SIGN>(v[u], ent[u]);
    }
    wave_lds_fence();
    e += n;
    left -= n;
  }
  if (p.mean && len) acc /= static_cast<float>(len);
  if (live && rl.act)
    store_piece(out, static_cast<uint64_t>(b) * p.row_stride + static_cast<uint64_t>(t) * p.d + rl.c,
                acc, p.rows_bf16);
}

// Items [e0, e1) of a bag pooled by one lane group, AHEAD of them in flight,
// without the table.
template <typename WT, int V, int AHEAD, bool SIGN>
__device__ __forceinline__ typename Piece<V>::type pool_items(
    const WT* __restrict__ w, const KParams& p, const void* __restrict__ indices, const int64_t e0,
    const int64_t e1, const uint32_t t, const uint32_t kk, const uint32_t jc, const KeygenOut& kg,
    const bool keys, const uint32_t row) {
  typename Piece<V>::type acc = {};
#pragma unroll 1
  for (int64_t e = e0; e < e1; e += AHEAD) {
    uint32_t en[AHEAD];
    bool split = false;
#pragma unroll
    for (int q = 0; q < AHEAD; ++q)  // past the end: the last one again
      en[q] = index_at(indices, static_cast<uint64_t>(e + q < e1 ? e + q : e1 - 1), p.idx32);
#pragma unroll
    for (int q = 0; q < AHEAD; ++q) {
      const uint32_t h = item_hash(en[q], t * p.C, p.TC, p.a, p.b);
      if (keys && e + q < e1) {
        kg.keys[e + q] = h;
        kg.rows[e + q] = row;
      }
      en[q] = item_entry<SIGN>(p, h, jc);
      split |= splits<V, SIGN>(en[q], kk, p.M);
    }
    if (__ballot(split)) {
#pragma unroll 1
      for (int q = 0; q < AHEAD; ++q) {
        uint32_t ent = en[0];
#pragma unroll
        for (int r = 1; r < AHEAD; ++r) ent = r == q ? en[r] : ent;
        if (e + q < e1) acc += sign_piece<SIGN>(gather_split<WT, V, SIGN>(w, ent, kk, p.M), ent);
      }
    } else {
      typename Piece<V>::type v[AHEAD];
#pragma unroll
      for (int q = 0; q < AHEAD; ++q) v[q] = gather<WT, V, SIGN>(w, en[q], kk, p.M);
#pragma unroll
      for (int q = 0; q < AHEAD; ++q)
        if (e + q < e1) acc += sign_piece<SIGN>(v[q], en[q]);
    }
  }
  return acc;
}

__device__ __forceinline__ float shfl_xor_piece(float x, int m) { return __shfl_xor(x, m); }
__device__ __forceinline__ f32x4 shfl_xor_piece(f32x4 x, int m) {
  return f32x4{__shfl_xor(x.x, m), __shfl_xor(x.y, m), __shfl_xor(x.z, m), __shfl_xor(x.w, m)};
}

// Few long bags: a workgroup per bag (blockIdx.x; slab blockIdx.y), a share of its
// items to every lane group of its wavefronts.  One lane group per bag would be
// bound by its chain of index, hash and gather: a bag of 50000 items, d = 16 (Z = 4) 15.7 ms / 288 us
// (one lane group / this kernel), d = 128 (Z = 32) 7.4 / 1.2 ms; 64 bags of 400 items, d = 64
// 76 / 9.6 us.
template <typename WT, int V, int LPB, bool SIGN>
__global__ __launch_bounds__(kBlockThreads) void forward_long_kernel(
    const WT* __restrict__ w, const KParams p, const void* __restrict__ indices,
    const void* __restrict__ offsets, void* __restrict__ out, const KeygenOut kg) {
  constexpr int GP = kWave / LPB, kShares = kWavesPerBlock * GP;
  __shared__ __align__(16) float part[kWavesPerBlock][LPB * V];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & (kWave - 1);
  const int grp = wv * GP + lane / LPB, gl = lane % LPB;
  const uint32_t g = blockIdx.x, t = g / p.B, b = g - t * p.B, row = b * p.T + t;
  const RowLane<V, LPB> rl(p, gl);
  const bool keys = kg.keys != nullptr && blockIdx.y == 0;
  int64_t e0 = offset_at(offsets, g, p.idx32);
  int64_t e1 = offset_at(offsets, static_cast<uint64_t>(g) + 1, p.idx32);
  e0 = e0 < 0 ? 0 : (e0 > p.N ? p.N : e0);
  e1 = e1 < 0 ? 0 : (e1 > p.N ? p.N : e1);
  if (e1 < e0) e1 = e0;
  const int64_t share = (e1 - e0 + kShares - 1) / kShares;
  const int64_t i0 = e0 + grp * share, i1 = i0 + share < e1 ? i0 + share : e1;
  typename Piece<V>::type sum = pool_items<WT, V, 8, SIGN>(w, p, indices, i0, i1, t, rl.kk, rl.jc, kg,
                                                           keys && gl == 0, row);
#pragma unroll
  for (int off = LPB; off < kWave; off <<= 1) sum += shfl_xor_piece(sum, off);
  if (lane < LPB) *reinterpret_cast<typename Piece<V>::type*>(&part[wv][gl * V]) = sum;
  __syncthreads();
  const float n = static_cast<float>(e1 - e0);
  if (keys && p.mean && threadIdx.x == 0 && e1 > e0) kg.inv_len[row] = 1.f / n;
  if (threadIdx.x >= LPB || !rl.act) return;
  sum = typename Piece<V>::type{};
#pragma unroll
  for (int v = 0; v < kWavesPerBlock; ++v)
    sum += *reinterpret_cast<const typename Piece<V>::type*>(&part[v][gl * V]);
  if (p.mean && e1 > e0) sum /= n;
  store_piece(out, static_cast<uint64_t>(b) * p.row_stride + static_cast<uint64_t>(t) * p.d + rl.c, sum,
              p.rows_bf16);
}

// As many items as bags (N == T*B), usually one per bag: a wavefront takes NB = U * GP
// consecutive bags, a lane each for the index and item hash, then gathers and stores U
// pieces per lane.  A wavefront that meets a bag of another length or position, or a
// piece split by the end of the array, works bag by bag.
//
// This replaced a persistent kernel that wrote the output in row order, one
// wavefront per SIMD in groups of 32 steps: 3328 rows of 512 bytes 11.8 -> 3.6 us, 10240
// 13 -> 5 us, 26 x 2048 13.1 -> 9 us, 26 x 16384 50.7 -> 45.4 us, 26 x 65536
// 179 -> 170 us (187 -> 176 us in a training step); and the tiled kernel for d = 16 and
// 1024 rows 18.1 -> 4.0 us.  Writing the rows alone in table order takes 160-170 us at
// 26 x 65536 (5.1-5.4 TB/s); small batches are bound by the chain of
// index load, hash, gather and store.
template <typename WT, int V, int LPB, bool SIGN>
__global__ __launch_bounds__(kBlockThreads, 8) void forward_stream_kernel(
    const WT* __restrict__ w, const KParams p, const void* __restrict__ indices,
    const void* __restrict__ offsets, void* __restrict__ out, const uint64_t wave0,
    const Touch touch, const KeygenOut kg) {
  constexpr int U = kRowBatch;
  constexpr int GP = kWave / LPB;
  constexpr int NB = U * GP;
  static_assert(NB <= kWave, "one lane per bag");
  touch_batch(p, w, indices, offsets, out, touch);
  __shared__ uint32_t tab_all[kWavesPerBlock][NB * LPB];
  const int lane = threadIdx.x & (kWave - 1);
  const int grp = lane / LPB, gl = lane % LPB;
  const uint64_t wave = wave0 + xcd_block() * kWavesPerBlock + (threadIdx.x >> 6);
  const uint64_t q0 = wave * NB;
  if (q0 >= p.num_bags) return;  // whole wavefront
  uint32_t* tab = tab_all[threadIdx.x >> 6];
  const uint32_t nb = p.num_bags - q0 < NB ? static_cast<uint32_t>(p.num_bags - q0) : NB;
  const bool mine = static_cast<uint32_t>(lane) < nb;
  const uint32_t g = static_cast<uint32_t>(q0) + (mine ? lane : 0u);  // bags number below 2^32
  const uint32_t t = g / p.B, b = g - t * p.B;
  const int64_t o0 = offset_at(offsets, g, p.idx32);
  const int64_t o1 = offset_at(offsets, static_cast<uint64_t>(g) + 1, p.idx32);
  const uint32_t idx = index_at(indices, g, p.idx32);  // g < N
  const RowLane<V, LPB> rl(p, gl);
  const uint32_t jl = rl.jc - rl.j0;
  const uint32_t tC = t * p.C;
  const uint64_t ro = static_cast<uint64_t>(b) * p.row_stride + static_cast<uint64_t>(t) * p.d;
  const uint32_t h0 = item_hash(idx, tC, p.TC, p.a, p.b);
#pragma unroll 1
  for (uint32_t k0 = 0; k0 < nb * rl.Cs; k0 += kWave) {
    const uint32_t k = k0 + lane;
    const uint32_t i = k / rl.Cs, j = k - i * rl.Cs;
    const uint32_t h = __shfl(h0, static_cast<int>(i < NB ? i : 0u));
    if (k < nb * rl.Cs) tab[k] = item_entry<SIGN>(p, h, rl.j0 + j);
  }
  wave_lds_fence();
  uint32_t ent[U];
  bool odd = mine && !(o0 == static_cast<int64_t>(g) && o1 == static_cast<int64_t>(g) + 1);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t i = static_cast<uint32_t>(u * GP + grp);
    ent[u] = tab[(i < nb ? i : 0u) * rl.Cs + jl];
    odd |= splits<V, SIGN>(ent[u], rl.kk, p.M);
  }
  // the lookups' keys and rows for the backward, when asked for
  const bool keys = kg.keys != nullptr && blockIdx.y == 0;
  if (__ballot(odd)) {
#pragma unroll 1
    for (int u = 0; u < U; ++u) {
      const int i = u * GP + grp;
      const int64_t s0 = __shfl(o0, i), s1 = __shfl(o1, i);
      const uint32_t tCi = __shfl(tC, i);
      const uint64_t roi = __shfl(ro, i);
      const uint32_t row = __shfl(b * p.T + t, i);
      if (static_cast<uint32_t>(i) >= nb) continue;
      const int64_t f0 = s0 < 0 ? 0 : (s0 > p.N ? p.N : s0);
      int64_t f1 = s1 < 0 ? 0 : (s1 > p.N ? p.N : s1);
      if (f1 < f0) f1 = f0;
      typename Piece<V>::type acc = {};
#pragma unroll 1
      for (int64_t e = f0; e < f1; ++e) {
        const uint32_t h =
            item_hash(index_at(indices, static_cast<uint64_t>(e), p.idx32), tCi, p.TC, p.a, p.b);
        if (keys && gl == 0) {
          kg.keys[e] = h;
          kg.rows[e] = row;
        }
        const uint32_t en = item_entry<SIGN>(p, h, rl.jc);
        acc += sign_piece<SIGN>(gather_split<WT, V, SIGN>(w, en, rl.kk, p.M), en);
      }
      if (keys && p.mean && gl == 0 && f1 > f0)
        kg.inv_len[row] = 1.f / static_cast<float>(f1 - f0);
      if (p.mean && f1 > f0) acc /= static_cast<float>(f1 - f0);
      if (rl.act) store_piece(out, roi + rl.c, acc, p.rows_bf16);
    }
    return;
  }
  typename Piece<V>::type v[U];
#pragma unroll
  for (int u = 0; u < U; ++u) v[u] = gather<WT, V, SIGN>(w, ent[u], rl.kk, p.M);
  if (keys && mine) {
    const uint32_t row = b * p.T + t;
    kg.keys[g] = h0;
    kg.rows[g] = row;
    if (p.mean) kg.inv_len[row] = 1.f;
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = u * GP + grp;
    const uint64_t roi = __shfl(ro, i);
    if (static_cast<uint32_t>(i) < nb && rl.act)
      store_piece(out, roi + rl.c, sign_piece<SIGN>(v[u], ent[u]), p.rows_bf16);
  }
}

// ---------------------------------------------------------------------------
// Tiled: one wavefront per tile of 64 bags of one table.  Each lane evaluates
// the C <= kTabChunks chunk bases of one item of the current 64-item block into a
// wave-private LDS table and the gathers read their base from it.  U items
// are gathered before any is consumed, and all U gathers of a batch are
// issued before any store of that batch (on gfx9 stores and loads share one
// in-order wait counter).
// ---------------------------------------------------------------------------

// One-hot tile: item l of the tile is bag l.  The (h0, bag) pairs are sorted
// across the lanes; every run of equal h0 is one token, gathered once (U runs
// in flight) and stored to the rows of all its bags.
template <typename WT, int EPL, int U, bool SIGN>
__device__ __forceinline__ void forward_onehot_tile(
    const WT* __restrict__ w, const KParams& p, const Tile& tl, const void* __restrict__ indices,
    void* __restrict__ out, uint32_t* tab, int lane, uint32_t c0, const uint32_t* jj,
    const uint32_t* kk, const bool* act, uint32_t spec) {
  const int nb = tl.nb;
  uint32_t key = 0xffffffffu;  // empty lanes sort last
  uint32_t bag = static_cast<uint32_t>(lane);
  const bool hit = tl.E0 == static_cast<int64_t>(tl.g0);
  if (lane < nb) {
    const uint32_t i = hit ? spec : load_index(indices, tl.E0 + lane, p.idx32);
    key = item_hash(i, tl.tC, p.TC, p.a, p.b);
  }
  wave_sort_pairs(key, bag, lane);
  fill_base_table<SIGN>(tab, key, p, lane);
  const uint32_t prev = __shfl_up(key, 1);
  uint64_t starts = __ballot(lane < nb && (lane == 0 || prev != key));
  while (starts) {
    // next U runs: first positions pos[u], run u covers [pos[u], pos[u+1])
    int pos[U + 1];
#pragma unroll
    for (int u = 0; u <= U; ++u) {
      if (starts) {
        pos[u] = __builtin_ctzll(starts);
        if (u < U) starts &= starts - 1;
      } else {
        pos[u] = nb;
      }
    }
    float v[U][EPL];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int pu = pos[u] < nb ? pos[u] : pos[0];
#pragma unroll
      for (int r = 0; r < EPL; ++r) {
        const Elem el = elem_of<SIGN>(tab[pu * kTabStride + jj[r]], kk[r], p.M);
        const float x = load_weight(w, act[r] ? el.m : 0u);
        v[u][r] = SIGN ? apply_sign(x, el) : x;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      for (int q = pos[u]; q < pos[u + 1]; ++q) {
        const int b = static_cast<int>(readlane_u32(bag, q));
        const uint64_t ro = readlane_u64(tl.row_off, b) + c0 + lane;
#pragma unroll
        for (int r = 0; r < EPL; ++r)
          if (act[r]) store_piece(out, ro + kWave * r, v[u][r], p.rows_bf16);
      }
    }
  }
}

template <typename WT, int EPL, int U, bool SIGN>
__global__ __launch_bounds__(kBlockThreads) void forward_kernel(
    const WT* __restrict__ w, const KParams p, const void* __restrict__ indices,
    const void* __restrict__ offsets, void* __restrict__ out, const uint64_t wave0,
    const Touch touch) {
  touch_batch(p, w, indices, offsets, out, touch);
  const int lane = threadIdx.x & (kWave - 1);
  const uint64_t wave = wave0 + xcd_block() * kWavesPerBlock + (threadIdx.x >> 6);
  const uint64_t g0 = wave * kTileBags;
  if (g0 >= p.num_bags) return;
  const uint32_t c0 = blockIdx.y * (kWave * EPL);

  __shared__ uint32_t tab_all[kWavesPerBlock * kWave * kTabStride];
  uint32_t* tab = tab_all + (threadIdx.x >> 6) * kWave * kTabStride;

  uint32_t kk[EPL], jj[EPL];
  bool act[EPL];
#pragma unroll
  for (int r = 0; r < EPL; ++r) {
    const uint32_t c = c0 + lane + kWave * r;
    act[r] = c < p.d;
    const uint32_t cc = act[r] ? c : 0;
    jj[r] = cc / p.Z;
    kk[r] = cc - jj[r] * p.Z;
  }

  // One-hot batches: item g0 + lane is usually bag g0 + lane's item; its
  // index is requested together with the offsets.
  uint32_t spec = 0;
  if (static_cast<int64_t>(g0) + lane < p.N) spec = load_index(indices, g0 + lane, p.idx32);
  const Tile tl = load_tile(p, offsets, g0, lane);

  // One-hot tile (every bag exactly one item): gather each distinct token
  // of the tile once and store its row to every bag that reads it.
  if (__ballot(lane >= tl.nb || tl.len == 1) == ~0ull) {
    forward_onehot_tile<WT, EPL, U, SIGN>(w, p, tl, indices, out, tab, lane, c0, jj, kk, act, spec);
    return;
  }

  float acc[EPL];
#pragma unroll
  for (int r = 0; r < EPL; ++r) acc[r] = 0.f;
  int cur = -1;  // local bag being pooled (wave-uniform)

  auto store_row = [&](int bag, bool zero) {
    const uint64_t ro = readlane_u64(tl.row_off, bag) + c0 + lane;
    float div = 1.f;
    if (p.mean && !zero) div = static_cast<float>(readlane_u32(tl.len, bag));
#pragma unroll
    for (int r = 0; r < EPL; ++r) {
      if (act[r]) {
        const float x = zero ? 0.f : (p.mean ? acc[r] / div : acc[r]);
        store_piece(out, ro + kWave * r, x, p.rows_bf16);
      }
    }
  };

  for (int64_t blk = tl.E0; blk < tl.E1; blk += kWave) {
    const int64_t rem = tl.E1 - blk;
    const int n = rem < kWave ? static_cast<int>(rem) : kWave;
    const int64_t e = blk + lane;
    uint32_t idx = 0;
    if (lane < n) idx = load_index(indices, e, p.idx32);
    const int bag = bag_of_item(tl, e);
    const uint32_t tC = __shfl(tl.tC, bag);
    fill_base_table<SIGN>(tab, item_hash(idx, tC, p.TC, p.a, p.b), p, lane);

    for (int q = 0; q < n; q += U) {
      // Gather phase: straight-line, U items x EPL loads in flight.  Items
      // past the end of the block re-read the last item (clamped index) and
      // inactive dims read element 0, so no load sits behind a branch.
      float v[U][EPL];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int uu = q + u < n ? q + u : n - 1;
#pragma unroll
        for (int r = 0; r < EPL; ++r) {
          const uint32_t ent = tab[uu * kTabStride + jj[r]];
          const Elem el = elem_of<SIGN>(ent, kk[r], p.M);
          const float x = load_weight(w, act[r] ? el.m : 0u);
          v[u][r] = SIGN ? apply_sign(x, el) : x;
        }
      }
      // Pool phase: stores only here, after every gather of the batch was
      // issued (a store counts in the same wait counter as the gathers).
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (q + u < n) {
          const int bg = static_cast<int>(readlane_u32(static_cast<uint32_t>(bag), q + u));
          if (bg != cur) {
            if (cur >= 0) store_row(cur, false);
            for (int z = cur + 1; z < bg; ++z) store_row(z, true);
            cur = bg;
#pragma unroll
            for (int r = 0; r < EPL; ++r) acc[r] = 0.f;
          }
#pragma unroll
          for (int r = 0; r < EPL; ++r) acc[r] += v[u][r];
        }
      }
    }
  }
  if (cur >= 0) store_row(cur, false);
  for (int z = cur + 1; z < tl.nb; ++z) store_row(z, true);
}

// A grid dimension holds fewer than 2^32 work-items (a larger one is cut to
// its low 32 bits without an error, and rows stay unwritten): batches of more
// bags take several launches, of whole multiples of kXcds workgroups.
constexpr uint64_t kMaxBlocks = 0xffffffffull / kBlockThreads / kXcds * kXcds;

// launch(blocks, wave0, touch) for consecutive shares of `waves` wavefronts, of
// which the first also reads ahead; blocks is a multiple of kXcds (the extra
// workgroups of the last share lie past the last bag and exit at once).
template <typename F>
static hipError_t launch_shares(uint64_t waves, const Touch& touch, F launch) {
  const uint64_t all = (waves + kWavesPerBlock - 1) / kWavesPerBlock;
  for (uint64_t b0 = 0; b0 < all; b0 += kMaxBlocks) {
    const uint64_t n = all - b0 < kMaxBlocks ? all - b0 : kMaxBlocks;
    launch(static_cast<uint32_t>((n + kXcds - 1) / kXcds * kXcds), b0 * kWavesPerBlock,
           b0 == 0 ? touch : Touch{});
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

static bool one_per_bag(const KParams& p) { return static_cast<uint64_t>(p.N) == p.num_bags; }

template <typename WT, int EPL, int U, bool SIGN>
static hipError_t launch_tiled_t(const WT* w, const KParams& p, const void* indices,
                                 const void* offsets, void* out, hipStream_t stream,
                                 const Touch& touch) {
  const uint32_t slabs = (p.d + kWave * EPL - 1) / (kWave * EPL);
  return launch_shares((p.num_bags + kTileBags - 1) / kTileBags, touch,
                       [&](uint32_t blocks, uint64_t wave0, const Touch& t) {
    hipLaunchKernelGGL((forward_kernel<WT, EPL, U, SIGN>), dim3(blocks, slabs),
                       dim3(kBlockThreads), 0, stream, w, p, indices, offsets, out, wave0, t);
  });
}

template <typename WT, bool SIGN>
static hipError_t launch_tiled(const WT* w, const KParams& p, const void* indices,
                               const void* offsets, void* out, hipStream_t stream,
                               const Touch& touch) {
  if (p.d <= 64) return launch_tiled_t<WT, 1, 16, SIGN>(w, p, indices, offsets, out, stream, touch);
  if (p.d <= 128) return launch_tiled_t<WT, 2, 8, SIGN>(w, p, indices, offsets, out, stream, touch);
  if (p.d <= 256) return launch_tiled_t<WT, 4, 4, SIGN>(w, p, indices, offsets, out, stream, touch);
  return launch_tiled_t<WT, 8, 2, SIGN>(w, p, indices, offsets, out, stream, touch);
}

// Bags of 64 items or more on average, too few of them to fill the chip by lane groups (a
// wavefront of the bags kernel on every SIMD) or by workgroups.  Bags / long kernel, d = 16, Z = 4, 64
// items each: 64 bags 24.6 / 5.4 us, 4000 30 / 24 us, 8000 31 / 43 us; d = 128, Z = 32: 1000 bags
// 15.2 / 7.4 us, 2000 (1000 wavefronts) 16.3 / 10.3 us; from there on the bags kernel is bound by
// its gathers.
constexpr uint64_t kLongBagItems = 64, kLongBagWaves = 1024, kLongBagBlocks = 4096;
static bool few_long_bags(const KParams& p, uint64_t waves, uint32_t slabs) {
  return !one_per_bag(p) && waves < kLongBagWaves && p.num_bags * slabs <= kLongBagBlocks &&
         static_cast<uint64_t>(p.N) >= kLongBagItems * p.num_bags;
}

template <typename WT, int V, int LPB, bool SIGN>
static hipError_t launch_rows_t(const WT* w, const KParams& p, const void* indices,
                                const void* offsets, void* out, hipStream_t stream,
                               const Touch& touch, const KeygenOut& kg) {
  const uint64_t per_wave = (kWave / LPB) * (one_per_bag(p) ? kRowBatch : 1);
  const uint32_t slabs = (p.d + LPB * V - 1) / (LPB * V);
  if (few_long_bags(p, p.num_bags / per_wave * slabs, slabs)) {
    hipLaunchKernelGGL((forward_long_kernel<WT, V, LPB, SIGN>),
                       dim3(static_cast<uint32_t>(p.num_bags), slabs), dim3(kBlockThreads), 0, stream, w,
                       p, indices, offsets, out, kg);
    return hipGetLastError();
  }
  return launch_shares((p.num_bags + per_wave - 1) / per_wave, touch,
                       [&](uint32_t blocks, uint64_t wave0, const Touch& t) {
    if (one_per_bag(p))
      hipLaunchKernelGGL((forward_stream_kernel<WT, V, LPB, SIGN>), dim3(blocks, slabs),
                         dim3(kBlockThreads), 0, stream, w, p, indices, offsets, out, wave0, t, kg);
    else
      hipLaunchKernelGGL((forward_bags_kernel<WT, V, LPB, SIGN>), dim3(blocks, slabs),
                         dim3(kBlockThreads), 0, stream, w, p, indices, offsets, out, wave0, kg);
  });
}

template <typename WT, int V, bool SIGN>
static hipError_t launch_rows_v(const WT* w, const KParams& p, const void* indices,
                                const void* offsets, void* out, hipStream_t stream,
                               const Touch& touch, const KeygenOut& kg) {
  const uint32_t lanes = (p.d + V - 1) / V;
  if (lanes <= 4) return launch_rows_t<WT, V, 4, SIGN>(w, p, indices, offsets, out, stream, touch, kg);
  if (lanes <= 8) return launch_rows_t<WT, V, 8, SIGN>(w, p, indices, offsets, out, stream, touch, kg);
  if (lanes <= 16) return launch_rows_t<WT, V, 16, SIGN>(w, p, indices, offsets, out, stream, touch, kg);
  if (lanes <= 32) return launch_rows_t<WT, V, 32, SIGN>(w, p, indices, offsets, out, stream, touch, kg);
  return launch_rows_t<WT, V, 64, SIGN>(w, p, indices, offsets, out, stream, touch, kg);
}

// The tiled kernel is kept where gathering each distinct token of 64 bags
// once pays for its longer chain: one-hot batches of 2^20 bags or more on an
// array beyond the aggregate L2.  Measured on 26 tables of Zipf(1.2) tokens, d = Z =
// 128, 128 MB bfloat16 array, rows / tiled: 2048 samples 8.2 / 23.7 us, 16384
// 44.9 / 65.2 us, 65536 212 / 199 us, 262144 990 / 774 us.
template <typename WT>
static bool tiled_applies(const KParams& p) {
  return one_per_bag(p) && p.num_bags >= (1ull << 20) &&
         p.C <= static_cast<uint32_t>(kTabChunks) &&
         static_cast<uint64_t>(p.M) * sizeof(WT) > kL2Bytes;
}

template <typename WT, bool SIGN>
static hipError_t launch_fwd_s(const WT* w, const KParams& p, const void* indices,
                               const void* offsets, void* out, hipStream_t stream,
                               const Touch& touch, const KeygenOut& kg) {
  if (tiled_applies<WT>(p)) {
    if (kg.keys != nullptr) return hipErrorInvalidValue;  // it does not write them
    return launch_tiled<WT, SIGN>(w, p, indices, offsets, out, stream, touch);
  }
  if (p.Z % 4 == 0) return launch_rows_v<WT, 4, SIGN>(w, p, indices, offsets, out, stream, touch, kg);
  return launch_rows_v<WT, 1, SIGN>(w, p, indices, offsets, out, stream, touch, kg);
}

template <typename WT>
static hipError_t launch_fwd_w(const WT* w, const KParams& p, const void* indices,
                               const void* offsets, void* out, hipStream_t stream,
                               const Touch& touch, const KeygenOut& kg) {
  if (p.sign_mode) return launch_fwd_s<WT, true>(w, p, indices, offsets, out, stream, touch, kg);
  return launch_fwd_s<WT, false>(w, p, indices, offsets, out, stream, touch, kg);
}

hipError_t launch_forward(const void* w, bool bf16, const KParams& p, const void* indices,
                          const void* offsets, void* out, hipStream_t stream, bool batch_read,
                          const KeygenOut& kg) {
  // (bags of several items gain from neither: 26 x 32768 bags of 20 items 906 us
  // without, 911 us with the array read)
  Touch touch;
  touch.index = !batch_read && p.num_bags >= kTouchBags ? 1u : 0u;
  const uint64_t bytes = static_cast<uint64_t>(p.M) * (bf16 ? 2 : 4);
  const uint64_t gathered = static_cast<uint64_t>(p.N) * p.d * (bf16 ? 2 : 4);
  if (bytes > kL2Bytes && bytes <= kTouchMaxBytes && gathered >= 8 * bytes) touch.bytes = bytes;
  if (bf16)
    return launch_fwd_w(static_cast<const uint16_t*>(w), p, indices, offsets, out, stream, touch, kg);
  return launch_fwd_w(static_cast<const float*>(w), p, indices, offsets, out, stream, touch, kg);
}

}  // namespace pss
