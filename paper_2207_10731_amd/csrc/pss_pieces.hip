// Deposit by pieces: the SORTED backward of small batches in one kernel.
//
// The grouped deposit (radix sort of the lookups by token, then the reduce
// stage) is a chain of four or five launches.  Up to kPieceMaxItems lookups that chain, not
// the memory traffic, is most of the call's time.  Here a workgroup takes P
// consecutive lookups in the batch's own order (items of one table, usually), finds
// their bags, sorts them by item hash, sums the output-gradient rows of each
// token and adds each sum once at its hashed addresses.  A token is deposited
// once per piece that holds it instead of about once per batch: 1.6 times the
// deposits on 26 x 2048 Zipf(1.1) lookups in pieces of 256.
//
//   items   item -> (h0, row, 1/|bag|): its bag is the item's own position
//           in a one-hot piece, else found by a search over the offsets; or
//           read from a prepared keygen (keys, rows)
//   sort    by counting, 4 threads per pair
//   sum     groups of LPB lanes (lanes over the dims), each 16 (LPB = 64), 8
//           or 4 consecutive pairs of the merged order, all rows requested
//           before any is used; a run that goes on into the next group's
//           pairs is finished by the group where it began
//   deposit float atomics at the run's chunk entries (hashed once per pair
//           into LDS for C <= kTabChunks)
#include <hip/hip_ext.h>

#include "pss_keygen.hpp"
#include "pss_launch.hpp"

namespace pss {

// Largest g in [0, num_bags) with offsets[g] <= e (0 if none), by one
// wavefront: 64 probes per step.
template <bool I32>
__device__ __forceinline__ uint64_t bag_search(const void* __restrict__ offsets, uint64_t num_bags,
                                               int64_t e, int lane) {
  uint64_t lo = 0, hi = num_bags;
  while (hi - lo > 1) {
    const uint64_t step = (hi - lo + kWave - 1) / kWave;
    const uint64_t pos = lo + (static_cast<uint64_t>(lane) + 1) * step;
    const bool below = pos < hi && load_int<I32>(offsets, pos) <= e;
    const uint64_t n = static_cast<uint64_t>(__popcll(__ballot(below)));
    lo += n * step;
    hi = lo + step < hi ? lo + step : hi;
  }
  return lo;
}

// With REC nothing is deposited: the run that begins at merged position q
// becomes row p0 + q of dst (N x d floats, its sign factors applied), and every
// position and chunk j a record (rec_keys, rec_ids): the chunk's base and
// (p0 + q) * C + j, or kNoChunk where no run begins or the chunk is not read.
// Every sum is then taken in a fixed order.
constexpr uint32_t kNoChunk = 0xffffffffu;
template <int EPL, int LPB, int P, bool SIGN, bool I32, bool REC, typename GT>
__global__ __launch_bounds__(4 * P) void deposit_pieces_kernel(
    float* __restrict__ dst, const float scale, const KParams p, const void* __restrict__ indices,
    const void* __restrict__ offsets, const uint32_t* __restrict__ keys,
    const uint32_t* __restrict__ rows, const float* __restrict__ inv_len,
    const GT* __restrict__ grad, uint32_t* __restrict__ rec_keys, uint32_t* __restrict__ rec_ids) {
  constexpr int GP = kWave / LPB;           // lane groups of a wavefront
  constexpr int NG = 4 * P / kWave * GP;    // ... of the workgroup
  constexpr int S = P / NG;                 // pairs per group
  constexpr int U = EPL * S > 64 ? 64 / EPL : S;  // rows in flight
  static_assert(S * GP == 16 && (EPL == 1 || LPB == kWave), "whole rows per group");
  __shared__ __align__(16) uint32_t lk[P];
  __shared__ uint32_t lr[P], mk[P], mr[P];
  __shared__ float ll[P], ml[P];
  __shared__ int64_t st[P + 1];
  __shared__ uint64_t first_bag;
  __shared__ int irregular;
  __shared__ uint32_t tab[P * kTabChunks];
  __shared__ float headv[NG][EPL * LPB];
  __shared__ uint32_t through[NG];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & (kWave - 1);
  const int64_t p0 = static_cast<int64_t>(blockIdx.x) * P;
  const int cnt = p.N - p0 < P ? static_cast<int>(p.N - p0) : P;

  // items
  const int64_t e = p0 + tid;
  const bool mine = tid < cnt;
  uint32_t key = 0xffffffffu, row = 0;
  float il = 1.f;
  if (keys != nullptr) {
    if (mine) {
      key = keys[e];
      row = rows[e];
      // both come from a keygen; the clamps keep reads and ranks in bounds
      if (key >= kP) key = 0;
      if (row >= p.num_bags) row = 0;
      if (p.mean) il = inv_len[row];
    }
  } else {
    uint32_t ix = 0;
    if (mine) ix = static_cast<uint32_t>(load_int<I32>(indices, static_cast<uint64_t>(e)));
    // one item per bag: offsets[e] = e all over the piece (then e < num_bags)
    bool own = static_cast<uint64_t>(p.N) == p.num_bags;
    if (own && tid <= cnt) own = load_int<I32>(offsets, static_cast<uint64_t>(e)) == e;
    if (tid == 0) irregular = 0;
    __syncthreads();
    if (tid <= cnt && !own) irregular = 1;
    __syncthreads();
    uint64_t g = static_cast<uint64_t>(e);
    if (irregular) {
      if (w == 0) {
        const uint64_t g0 = bag_search<I32>(offsets, p.num_bags, p0, lane);
        if (lane == 0) first_bag = g0;
      }
      __syncthreads();
      const uint64_t g0 = first_bag;
      if (tid <= P) {
        const uint64_t q = g0 + tid < p.num_bags ? g0 + tid : p.num_bags;
        st[tid] = load_int<I32>(offsets, q);
      }
      __syncthreads();
      if (mine) {
        int64_t s0, s1;
        // the P bags from g0 on reach the piece's last item, unless many
        // of them are empty
        if (g0 + P >= p.num_bags || st[P] > p0 + cnt - 1) {
          const int nb = p.num_bags - g0 < P ? static_cast<int>(p.num_bags - g0) : P;
          int lo = 0;
          for (int step = P / 2; step >= 1; step >>= 1)
            if (lo + step < nb && st[lo + step] <= e) lo += step;
          g = g0 + lo;
          s0 = st[lo];
          s1 = st[lo + 1];
        } else {
          uint64_t lo = g0, hi = p.num_bags - 1;
          while (lo < hi) {
            const uint64_t mid = (lo + hi + 1) >> 1;
            if (load_int<I32>(offsets, mid) <= e) lo = mid; else hi = mid - 1;
          }
          g = lo;
          s0 = load_int<I32>(offsets, lo);
          s1 = load_int<I32>(offsets, lo + 1);
        }
        if (p.mean && s1 > s0) il = 1.f / static_cast<float>(s1 - s0);
      }
    }
    if (mine) {
      const uint32_t t = static_cast<uint32_t>(g) / p.B;  // bags number below 2^32
      const uint32_t b = static_cast<uint32_t>(g) - t * p.B;
      row = b * p.T + t;
      key = item_hash(ix, t * p.C, p.TC, p.a, p.b);
    }
  }

  // sort, by counting: 4 threads per pair each compare its key with a
  // quarter of the keys (equal keys keep their order).  Empty slots hold key
  // 0xffffffff, above any hash, and stay behind.
  if (tid < P) {
    lk[tid] = key;
    lr[tid] = row;
    ll[tid] = il;
  }
  __syncthreads();
  {
    const int i = tid >> 2, part = tid & 3;
    const uint32_t ki = lk[i];
    uint32_t before = 0;
    const uint4* quarter = reinterpret_cast<const uint4*>(lk + part * (P / 4));
#pragma unroll 4
    for (int v = 0; v < P / 16; ++v) {
      const uint4 k4 = quarter[v];
      const int j = part * (P / 4) + v * 4;
      before += k4.x < ki + (j < i ? 1u : 0u);
      before += k4.y < ki + (j + 1 < i ? 1u : 0u);
      before += k4.z < ki + (j + 2 < i ? 1u : 0u);
      before += k4.w < ki + (j + 3 < i ? 1u : 0u);
    }
    before += __shfl_xor(before, 1);
    before += __shfl_xor(before, 2);
    const uint32_t rank = i < cnt ? before : static_cast<uint32_t>(i);
    if (part == 0) {
      mk[rank] = ki;
      mr[rank] = lr[i];
      ml[rank] = ll[i];
    }
  }
  __syncthreads();

  // sum
  const int gl = lane % LPB;
  const int grp = w * GP + lane / LPB;
  const uint32_t c0 = blockIdx.y * (LPB * EPL);
  bool act[EPL];
  uint32_t cc[EPL];
#pragma unroll
  for (int r = 0; r < EPL; ++r) {
    const uint32_t c = c0 + gl + LPB * r;
    act[r] = c < p.d;
    cc[r] = act[r] ? c : 0u;
  }
  const int q0 = grp * S;
  const int nq = cnt - q0 < S ? (cnt > q0 ? cnt - q0 : 0) : S;
  // lane u < S of the group: pair q0 + u (past the end the last one again)
  const int base_lane = lane - gl;
  const int qu = q0 + (gl < nq ? gl : (nq ? nq - 1 : 0));
  const uint32_t wr = nq ? mr[qu] : 0u;
  const float wf = p.mean && nq ? ml[qu] : 1.f;
  // whether its run ends with it
  const uint64_t ends_all =
      __ballot(gl < nq && (qu + 1 >= cnt || mk[qu + 1] != mk[qu]));
  const uint32_t ends_mask = static_cast<uint32_t>(ends_all >> base_lane) & ((1u << S) - 1);
  float g[U][EPL];
  auto request = [&](int u0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t ru = LPB == kWave ? readlane_u32(wr, u0 + u) : __shfl(wr, base_lane + u0 + u);
      const GT* grow = grad + static_cast<uint64_t>(ru) * p.d;
#pragma unroll
      for (int r = 0; r < EPL; ++r) g[u][r] = load_row(grow, cc[r]);
    }
  };
  request(0);
  // chunk entries of every pair, while the rows are on their way
  const bool use_tab = p.C <= static_cast<uint32_t>(kTabChunks);
  if (REC && blockIdx.y == 0) {
    for (uint32_t k = tid; k < static_cast<uint32_t>(cnt) * p.C; k += 4 * P) {
      const uint32_t i = k / p.C, j = k - i * p.C;
      const uint32_t h = mk[i];
      uint32_t base = kNoChunk;
      if (i == 0 || mk[i - 1] != h) {
        const uint32_t ent = chunk_entry<SIGN>(
            fast_mod(add_mod_p(h, chunk_step(p.a, j)), p.fm_c, p.M),
            SIGN ? add_mod_p(sign_hash0(h, p.s_alpha, p.s_beta), chunk_step(p.a2, j)) : 0u, p);
        if (!SIGN || ent != kSkip) base = ent & 0x7fffffffu;
      }
      const uint64_t at = static_cast<uint64_t>(p0) * p.C + k;
      rec_keys[at] = base;
      rec_ids[at] = static_cast<uint32_t>(at);
    }
  }
  if (use_tab && (!REC || SIGN)) {
    for (uint32_t k = tid; k < static_cast<uint32_t>(cnt) * p.C; k += 4 * P) {
      const uint32_t i = k / p.C, j = k - i * p.C;
      const uint32_t h = mk[i];
      const uint32_t base = fast_mod(add_mod_p(h, chunk_step(p.a, j)), p.fm_c, p.M);
      tab[k] = SIGN ? chunk_entry<SIGN>(base, add_mod_p(sign_hash0(h, p.s_alpha, p.s_beta),
                                                        chunk_step(p.a2, j)), p)
                    : base;
    }
  }
  uint32_t jj[EPL], kk[EPL];
#pragma unroll
  for (int r = 0; r < EPL; ++r) {
    jj[r] = cc[r] / p.Z;
    kk[r] = cc[r] - jj[r] * p.Z;
  }
  __syncthreads();
  auto deposit = [&](const float* acc, int q) {
    if (REC && !SIGN) {
      float* row = dst + (static_cast<uint64_t>(p0) + q) * p.d;
#pragma unroll
      for (int r = 0; r < EPL; ++r)
        if (act[r]) row[cc[r]] = acc[r];
      return;
    }
    const uint32_t h = use_tab ? 0u : mk[q];
    const uint32_t h2 = SIGN && !use_tab ? sign_hash0(h, p.s_alpha, p.s_beta) : 0u;
#pragma unroll
    for (int r = 0; r < EPL; ++r) {
      if (!act[r]) continue;
      const uint32_t ent =
          use_tab ? tab[q * p.C + jj[r]]
                  : chunk_entry<SIGN>(fast_mod(add_mod_p(h, chunk_step(p.a, jj[r])), p.fm_c, p.M),
                                      add_mod_p(h2, SIGN ? chunk_step(p.a2, jj[r]) : 0u), p);
      const Elem el = elem_of<SIGN>(ent, kk[r], p.M);
      const float x = scale * acc[r];
      if (REC) {
        dst[(static_cast<uint64_t>(p0) + q) * p.d + cc[r]] = apply_sign(x, el);
        continue;
      }
      if (!SIGN || el.read) unsafeAtomicAdd(dst + el.m, SIGN ? apply_sign(x, el) : x);
    }
  };
  float acc[EPL];
#pragma unroll
  for (int r = 0; r < EPL; ++r) acc[r] = 0.f;
  // the group's first run began in an earlier group's pairs
  bool head = q0 > 0 && nq > 0 && mk[q0] == mk[q0 - 1];
  bool tail = false;  // its last run goes on in the next group's pairs
  int start = q0;     // where its current run begins
#pragma unroll 1
  for (int u0 = 0; u0 < S; u0 += U) {
    if (u0 > 0) request(u0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = q0 + u0 + u;
      if (u0 + u < nq) {
        const float f = __shfl(wf, base_lane + u0 + u);
#pragma unroll
        for (int r = 0; r < EPL; ++r) acc[r] += p.mean ? g[u][r] * f : g[u][r];
        const bool ends = (ends_mask >> (u0 + u)) & 1u;
        tail = !ends;
        if (ends) {
          if (head) {
#pragma unroll
            for (int r = 0; r < EPL; ++r) headv[grp][LPB * r + gl] = acc[r];
            head = false;
          } else {
            deposit(acc, start);
          }
          start = q + 1;
#pragma unroll
          for (int r = 0; r < EPL; ++r) acc[r] = 0.f;
        }
      }
    }
  }
  const bool thru = head && tail;  // all of its pairs lie inside one run
  if (thru) {
#pragma unroll
    for (int r = 0; r < EPL; ++r) headv[grp][LPB * r + gl] = acc[r];
  }
  if (gl == 0) through[grp] = thru ? 1u : 0u;
  __syncthreads();
  if (tail && !thru) {
    for (int k = grp + 1; k < NG; ++k) {
#pragma unroll
      for (int r = 0; r < EPL; ++r) acc[r] += headv[k][LPB * r + gl];
      if (!through[k]) break;
    }
    deposit(acc, start);
  }
}

// What a launch writes besides dst: nothing, or records.
struct PieceRecords {
  uint32_t* keys = nullptr;
  uint32_t* ids = nullptr;
};

template <int EPL, int LPB, int P, bool SIGN, bool REC, typename GT>
static hipError_t launch_pieces_t(float* dst, float scale, const KParams& p, const void* indices,
                                  const void* offsets, const GroupedPairs* pairs, const GT* grad,
                                  const PieceRecords& rec, hipStream_t stream) {
  const dim3 grid(static_cast<uint32_t>((p.N + P - 1) / P), (p.d + LPB * EPL - 1) / (LPB * EPL));
  const uint32_t* keys = pairs != nullptr ? pairs->keys : nullptr;
  const uint32_t* rows = pairs != nullptr ? pairs->rows : nullptr;
  const float* il = pairs != nullptr ? pairs->inv_len : nullptr;
  const dim3 block(4 * P);
  hipEvent_t before = nullptr, after = nullptr;
  if (!REC) reduce_events(&before, &after);
  const auto kernel = p.idx32 ? deposit_pieces_kernel<EPL, LPB, P, SIGN, true, REC, GT>
                              : deposit_pieces_kernel<EPL, LPB, P, SIGN, false, REC, GT>;
  if (before != nullptr)  // the timing hook: the dispatch records both events
    hipExtLaunchKernelGGL(kernel, grid, block, 0, stream, before, after, 0u, dst, scale, p, indices,
                          offsets, keys, rows, il, grad, rec.keys, rec.ids);
  else
    hipLaunchKernelGGL(kernel, grid, block, 0, stream, dst, scale, p, indices, offsets, keys, rows,
                       il, grad, rec.keys, rec.ids);
  return hipGetLastError();
}

// Pieces of 64 lookups while pieces of 256 would leave compute units idle:
// 10240 lookups 10.7 / 16 us (64 / 256), 13312 10.4 / 15 us, 53248 32.5 / 28 us (the
// shorter pieces make more deposits).
constexpr int64_t kSmallPieceItems = 1 << 15;

template <int EPL, int LPB, bool SIGN, bool REC, typename GT, typename... A>
static hipError_t launch_pieces_p(float* dst, float scale, const KParams& p, A... a) {
  if (p.N <= kSmallPieceItems) return launch_pieces_t<EPL, LPB, 64, SIGN, REC, GT>(dst, scale, p, a...);
  return launch_pieces_t<EPL, LPB, 256, SIGN, REC, GT>(dst, scale, p, a...);
}

template <bool SIGN, bool REC, typename GT, typename... A>
static hipError_t launch_pieces_s(float* dst, float scale, const KParams& p, A... a) {
  if (p.d <= 16) return launch_pieces_p<1, 16, SIGN, REC, GT>(dst, scale, p, a...);
  if (p.d <= 32) return launch_pieces_p<1, 32, SIGN, REC, GT>(dst, scale, p, a...);
  if (p.d <= 64) return launch_pieces_p<1, 64, SIGN, REC, GT>(dst, scale, p, a...);
  if (p.d <= 128) return launch_pieces_p<2, 64, SIGN, REC, GT>(dst, scale, p, a...);
  return launch_pieces_p<4, 64, SIGN, REC, GT>(dst, scale, p, a...);
}

template <bool REC, typename GT>
static hipError_t launch_pieces_g(float* dst, float scale, const KParams& p, const void* indices,
                                  const void* offsets, const GroupedPairs* pairs, const void* grad,
                                  const PieceRecords& rec, hipStream_t stream) {
  const GT* g = static_cast<const GT*>(grad);
  if (p.sign_mode)
    return launch_pieces_s<true, REC, GT>(dst, scale, p, indices, offsets, pairs, g, rec, stream);
  return launch_pieces_s<false, REC, GT>(dst, scale, p, indices, offsets, pairs, g, rec, stream);
}

hipError_t launch_deposit_pieces(float* dst, float scale, const KParams& p, const void* indices,
                                 const void* offsets, const GroupedPairs* pairs, const void* grad,
                                 hipStream_t stream) {
  if (p.N == 0) return hipSuccess;
  const PieceRecords none;
  if (p.rows_bf16)
    return launch_pieces_g<false, uint16_t>(dst, scale, p, indices, offsets, pairs, grad, none, stream);
  return launch_pieces_g<false, float>(dst, scale, p, indices, offsets, pairs, grad, none, stream);
}

hipError_t launch_piece_records(float* sums, const KParams& p, const void* indices,
                                const void* offsets, const void* grad, uint32_t* rec_keys,
                                uint32_t* rec_ids, hipStream_t stream) {
  const PieceRecords rec{rec_keys, rec_ids};
  if (p.rows_bf16)
    return launch_pieces_g<true, uint16_t>(sums, 1.f, p, indices, offsets, nullptr, grad, rec, stream);
  return launch_pieces_g<true, float>(sums, 1.f, p, indices, offsets, nullptr, grad, rec, stream);
}

// Where one kernel is the faster form.  It saves three or four launches (25
// to 30 us in a chain) and pays in deposits: each costs a 64-byte line
// update at the memory side, about 20 G/s, for every line of every chunk.  So
// the rule counts the lookups' chunk lines.  Pieces / grouped (kernel times, the
// latter without the gaps between its four kernels), 26 tables of Zipf(1.1)
// tokens, d = 128, Z = 32: 512 samples 10.4 / 33 us, 2048 28 / 36 us (0.64 M lines),
// 4096 46 / 46 us (1.3 M), 8192 85 / 64 us (2.6 M); 13 tables of 9-item bags, d = 96,
// Z = 8: 58 K lookups 49 / 62 us (1.0 M), 207 K 152 / 118 us (3.7 M).
//
// A frequent token is deposited once per piece, and every deposit rounds in 32
// bits at its element.  Relative distance from 64-bit sums, pieces against
// grouped, geometric mean over drawn shapes: up to 4096 lookups per
// table 0.85 (95 results), to 12000 0.97 (31), to 16384 1.31 (4) and beyond
// 1.17 (23); so tables of more lookups keep the grouped deposit.
constexpr int64_t kPieceMaxItems = 1 << 18;
constexpr int64_t kPieceMaxLines = 3 << 19;
constexpr int64_t kPieceTableItems = 12000;
bool deposits_by_piece(const KParams& p) {
  return p.N <= kPieceMaxItems &&
         p.N * static_cast<int64_t>(p.C) * (p.Z / 16 + 1) <= kPieceMaxLines &&
         static_cast<uint64_t>(p.N) * p.B <= kPieceTableItems * p.num_bags;
}

}  // namespace pss
