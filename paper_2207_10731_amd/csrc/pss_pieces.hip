// Deposit by pieces: the SORTED backward of small one-hot batches in one kernel.
//
// The grouped deposit (radix sort of the lookups by token, then the reduce
// stage) is a chain of four or five launches.  Up to kPieceMaxItems lookups that chain, not
// the memory traffic, is most of the call's time.  Here a workgroup finds by
// itself the lookups of one piece of the order by token (token_order), sorts them
// by item hash, sums the output-gradient rows of each token and adds each
// sum once at its hashed addresses.
//
//   order   lookups of the piece: see token_order
//   sort    by counting, 4 threads per pair
//   sum     groups of LPB lanes (lanes over the dims), each 16 (LPB = 64), 8
//           or 4 consecutive pairs of the merged order, all rows requested
//           before any is used; a run that goes on into the next group's
//           pairs is finished by the group where it began
//   deposit float atomics at the run's chunk entries (hashed once per pair
//           into LDS for C <= kTabChunks)
//
// Pieces of the batch's own order, each token deposited once per piece that holds
// it, need no order stage, but every deposit rounds in 32 bits at its element: the
// distance from 64-bit sums grew up to 1.5 times (2 tables of 3927
// Zipf lookups, d = 256, Z = 8).  In the order by token, with two chains of additions
// per run, it is at most 1.03 times the grouped deposit's, shape by shape, and 0.87
// times in the mean (69 results of drawn and skewed shapes, three seeds each).
#include <hip/hip_ext.h>

#include "pss_keygen.hpp"
#include "pss_launch.hpp"

namespace pss {

// The bag of lookup e: largest g with offsets[g] <= e.
template <bool I32>
__device__ __forceinline__ uint64_t bag_of(const KParams& p, const void* __restrict__ offsets,
                                           int64_t e) {
  uint64_t lo = 0, hi = p.num_bags - 1;
  while (lo < hi) {
    const uint64_t mid = (lo + hi + 1) >> 1;
    if (load_int<I32>(offsets, mid) <= e) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// The order by token: the batch is cut into regions of `len` consecutive lookups
// (whole tables), a region into `pieces` pieces of its lookups ordered by bins of
// the item hash, within a bin as in the batch.  Every workgroup counts its region's
// bins by itself (their keys stay in LDS), finds the piece's two cuts and collects
// the lookups between them: no sorted list is kept, and no launch is needed to make
// one.  A token is then deposited once, or once per piece of a bin that outgrows the
// slack below, as in the grouped deposit.  The cost grows with the region:
// see kPieceRegion.
//
// Nominal cuts lie piece_cut apart; a cut inside a bin of up to P - piece_cut lookups
// moves back to the bin's start, so that no small bin is divided, and a piece
// has at most P lookups.
struct Regions {
  uint32_t len, pieces;
};
constexpr int kTokenBins = 1024;
template <int P> constexpr uint32_t piece_cut() { return P - P / 8; }
__device__ __forceinline__ uint32_t token_bin(uint32_t key) { return (key * 0x9e3779b1u) >> 22; }

template <int P>
struct TokenOrder {
  static constexpr int kWaves = 4 * P / kWave;
  __align__(16) uint64_t pair[P];  // the piece's lookups, in any order: key << 32 | lookup
  uint32_t start[kTokenBins];      // counts, then first position of each bin
  uint32_t wsum[kWaves], part[2][kWaves];
  uint32_t cut[2], bin[2];         // the piece's cuts and the bins they divide
  uint32_t taken;
  int irregular;
};
constexpr uint32_t kNoBin = 0xffffffffu;

// Collects the lookups of workgroup blockIdx.x's piece in lds.pair, sets *p0 to its first
// position in the batch and returns their number (the same for the whole
// workgroup).  Which lookups they are depends on the batch alone.
template <int P, bool I32>
__device__ __forceinline__ int token_order(const KParams& p, const void* __restrict__ indices,
                                           const void* __restrict__ offsets,
                                           const uint32_t* __restrict__ keys, const Regions& regions,
                                           TokenOrder<P>& lds, uint32_t* p0, bool* searched) {
  constexpr int NT = 4 * P, NW = TokenOrder<P>::kWaves;
  constexpr uint32_t kCut = piece_cut<P>(), kSlack = P - kCut;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & (kWave - 1);
  const uint32_t region = blockIdx.x / regions.pieces, piece = blockIdx.x - region * regions.pieces;
  const uint32_t lo = region * regions.len;  // N < 2^32
  const uint32_t n = static_cast<uint32_t>(p.N) - lo < regions.len ? static_cast<uint32_t>(p.N) - lo
                                                                  : regions.len;
  const uint32_t q0 = piece * kCut, q1 = q0 + kCut < n ? q0 + kCut : n;  // nominal cuts
  if (q0 >= n) return 0;
  // a wavefront takes a contiguous part of the region, in whole wavefronts
  const uint32_t per_wave = ((n + NW - 1) / NW + kWave - 1) / kWave * kWave;
  const uint32_t i_lo = w * per_wave < n ? w * per_wave : n;
  const uint32_t i_hi = i_lo + per_wave < n ? i_lo + per_wave : n;
  extern __shared__ uint32_t region_keys[];  // n, kept between the passes
  bool search = false;  // bags are not one item each: found by a search
  for (;;) {
    for (int b = tid; b < kTokenBins; b += NT) lds.start[b] = 0;
    if (tid == 0) lds.irregular = 0;
    __syncthreads();
    // without keys: as many lookups as bags, one per bag unless an offset says
    // otherwise (then e < num_bags all over the region)
    const bool check = keys == nullptr && !search;
    bool odd = check && tid == 0 && load_int<I32>(offsets, lo + n) != lo + n;
    constexpr int kAhead = 8;  // requested together
    for (uint32_t i0 = i_lo; i0 < i_hi; i0 += kAhead * kWave) {
      uint32_t e[kAhead], k[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {  // (past the end: the last one again)
        const uint32_t i = i0 + u * kWave + lane;
        e[u] = lo + (i < i_hi ? i : i_hi - 1);
      }
      if (keys != nullptr) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) k[u] = keys[e[u]];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) k[u] = k[u] < kP ? k[u] : 0u;
      } else {
        uint32_t g[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          k[u] = static_cast<uint32_t>(load_int<I32>(indices, e[u]));
          g[u] = static_cast<uint32_t>(load_int<I32>(offsets, e[u]));  // at most N < 2^32
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) odd |= check && g[u] != e[u];
        if (search) {
#pragma unroll 1
          for (int u = 0; u < kAhead; ++u) {
            const uint32_t b = static_cast<uint32_t>(bag_of<I32>(p, offsets, e[0] + u * kWave));
#pragma unroll
            for (int v = 0; v < kAhead; ++v) g[v] = u == v ? b : g[v];
          }
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
          k[u] = item_hash(k[u], (search ? g[u] : e[u]) / p.B * p.C, p.TC, p.a, p.b);
      }
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const uint32_t i = i0 + u * kWave + lane;
        if (i >= i_hi) continue;
        region_keys[i] = k[u];
        atomicAdd(&lds.start[token_bin(k[u])], 1u);
      }
    }
    if (odd) lds.irregular = 1;
    __syncthreads();
    if (!lds.irregular) break;
    __syncthreads();
    search = true;
  }
  // positions of the bins, and the two cuts
  constexpr int kOwn = kTokenBins / NT;  // consecutive bins per thread
  uint32_t c[kOwn], sum = 0;
#pragma unroll
  for (int b = 0; b < kOwn; ++b) {
    c[b] = lds.start[tid * kOwn + b];
    sum += c[b];
  }
  uint32_t incl = sum;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const uint32_t y = __shfl_up(incl, off);
    if (lane >= off) incl += y;
  }
  if (lane == kWave - 1) lds.wsum[w] = incl;
  if (tid < 2) {
    lds.cut[tid] = tid ? q1 : q0;
    lds.bin[tid] = kNoBin;
  }
  if (tid == 2) lds.taken = 0;
  __syncthreads();
  uint32_t s = incl - sum;
#pragma unroll
  for (int v = 0; v < NW; ++v) s += v < w ? lds.wsum[v] : 0u;
#pragma unroll
  for (int b = 0; b < kOwn; ++b) {
    lds.start[tid * kOwn + b] = s;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const uint32_t q = x ? q1 : q0;
      if (s < q && q < s + c[b]) {  // the cut lies inside the bin
        if (c[b] <= kSlack) lds.cut[x] = s;
        else lds.bin[x] = tid * kOwn + b;
      }
    }
    s += c[b];
  }
  __syncthreads();
  const uint32_t c0 = lds.cut[0], c1 = lds.cut[1];
  const uint32_t b0 = lds.bin[0], b1 = lds.bin[1];
  // Slots: the lookups of whole bins as they come, then those of the divided
  // bins by their position.
  const uint32_t cnt = c1 - c0;
  const uint32_t s0 = b0 != kNoBin ? lds.start[b0] : 0u, s1 = b1 != kNoBin ? lds.start[b1] : 0u;
  uint32_t end0 = c0;  // of b0's part
  if (b0 != kNoBin) end0 = b0 == b1 || b0 + 1 == kTokenBins ? c1 : lds.start[b0 + 1];
  const uint32_t n0 = end0 - c0, n1 = b1 != kNoBin && b1 != b0 ? c1 - s1 : 0u;
  const uint32_t at0 = cnt - n0 - n1, at1 = cnt - n1;
  const uint64_t below = (1ull << lane) - 1;
  auto put = [&](uint32_t at, uint32_t k, uint32_t i) {
    if (at < P) lds.pair[at] = static_cast<uint64_t>(k) << 32 | (lo + i);
  };
  constexpr int kSteps = 4;  // looked up together
  for (uint32_t i0 = i_lo; i0 < i_hi; i0 += kSteps * kWave) {
    uint32_t k[kSteps], first[kSteps];
    bool take[kSteps];
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
      const uint32_t i = i0 + u * kWave + lane;
      k[u] = i < i_hi ? region_keys[i] : 0u;
    }
#pragma unroll
    for (int u = 0; u < kSteps; ++u) first[u] = lds.start[token_bin(k[u])];
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
      const uint32_t b = token_bin(k[u]);
      take[u] = i0 + u * kWave + lane < i_hi && first[u] >= c0 && first[u] < c1 && b != b0 && b != b1;
    }
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
      const uint64_t m = __ballot(take[u]);
      if (m == 0) continue;
      uint32_t base = 0;
      if (lane == 0) base = atomicAdd(&lds.taken, static_cast<uint32_t>(__popcll(m)));
      base = readlane_u32(base, 0);
      if (take[u]) put(base + __popcll(m & below), k[u], i0 + u * kWave + lane);
    }
  }
  if (n0 + n1 != 0) {  // ranks in the divided bins, in the batch's order
    auto each = [&](auto f) {
      for (uint32_t i0 = i_lo; i0 < i_hi; i0 += kWave) {
        const uint32_t i = i0 + lane;
        const uint32_t k = i < i_hi ? region_keys[i] : 0u;
        const uint32_t b = i >= i_hi ? kNoBin : token_bin(k);
        f(i, k, __ballot(n0 != 0 && b == b0), __ballot(n1 != 0 && b == b1));
      }
    };
    uint32_t rank0 = 0, rank1 = 0;
    each([&](uint32_t, uint32_t, uint64_t m0, uint64_t m1) {
      rank0 += __popcll(m0);
      rank1 += __popcll(m1);
    });
    if (lane == 0) {
      lds.part[0][w] = rank0;
      lds.part[1][w] = rank1;
    }
    __syncthreads();
    rank0 = rank1 = 0;
    for (int v = 0; v < w; ++v) {
      rank0 += lds.part[0][v];
      rank1 += lds.part[1][v];
    }
    each([&](uint32_t i, uint32_t k, uint64_t m0, uint64_t m1) {
      if ((m0 >> lane) & 1u) {
        const uint32_t pos = s0 + rank0 + __popcll(m0 & below);
        if (pos >= c0 && pos < end0) put(at0 + pos - c0, k, i);
      }
      if ((m1 >> lane) & 1u) {
        const uint32_t pos = s1 + rank1 + __popcll(m1 & below);
        if (pos < c1) put(at1 + pos - s1, k, i);
      }
      rank0 += __popcll(m0);
      rank1 += __popcll(m1);
    });
  }
  __syncthreads();
  *p0 = lo + c0;
  *searched = search;
  return cnt < P ? static_cast<int>(cnt) : P;
}

// With REC nothing is deposited: the run that begins at merged position q
// becomes row p0 + q of dst (N x d floats, its sign factors applied), and every
// position and chunk j a record (rec_keys, rec_ids): the chunk's base and
// (p0 + q) * C + j, or kNoChunk where no run begins or the chunk is not read.
// Every sum is then taken in a fixed order.
template <int EPL, int LPB, int P, bool SIGN, bool I32, bool REC, typename GT>
__global__ __launch_bounds__(4 * P) void deposit_pieces_kernel(
    float* __restrict__ dst, const float scale, const KParams p, const void* __restrict__ indices,
    const void* __restrict__ offsets, const uint32_t* __restrict__ keys,
    const uint32_t* __restrict__ rows, const float* __restrict__ inv_len,
    const GT* __restrict__ grad, uint32_t* __restrict__ rec_keys, uint32_t* __restrict__ rec_ids,
    const Regions regions) {
  constexpr int GP = kWave / LPB;           // lane groups of a wavefront
  constexpr int NG = 4 * P / kWave * GP;    // ... of the workgroup
  constexpr int S = P / NG;                 // pairs per group
  constexpr int U = EPL * S > 64 ? 64 / EPL : S;  // rows in flight
  static_assert(S * GP == 16 && (EPL == 1 || LPB == kWave), "whole rows per group");
  __shared__ uint32_t lr[P], mk[P], mr[P];
  __shared__ float ll[P], ml[P];
  __shared__ uint32_t tab[P * kTabChunks];
  __shared__ float headv[NG][EPL * LPB];
  __shared__ uint32_t through[NG];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & (kWave - 1);
  // the piece's lookups
  __shared__ TokenOrder<P> order;
  uint32_t p0 = 0;
  bool searched = false;
  const int cnt = token_order<P, I32>(p, indices, offsets, keys, regions, order, &p0, &searched);
  if (cnt == 0) return;  // whole workgroup
  // their pooled rows and 1/|bag|; empty slots sort last (no key is 0xffffffff)
  if (tid < P) {
    uint32_t row = 0;
    float il = 1.f;
    if (tid >= cnt) {
      order.pair[tid] = ~0ull;
    } else {
      uint32_t e = static_cast<uint32_t>(order.pair[tid]);
      if (e >= p.N) e = 0;  // (indices changed during the call)
      if (keys != nullptr) {
        row = rows[e];
        if (row >= p.num_bags) row = 0;  // from a keygen; the clamp keeps reads in bounds
        if (p.mean) il = inv_len[row];
      } else {
        uint32_t g = e;
        if (searched) {
          g = static_cast<uint32_t>(bag_of<I32>(p, offsets, e));
          const int64_t o0 = load_int<I32>(offsets, g);
          const int64_t o1 = load_int<I32>(offsets, static_cast<uint64_t>(g) + 1);
          if (p.mean && o1 > o0) il = 1.f / static_cast<float>(o1 - o0);
        }
        const uint32_t t = g / p.B, b = g - t * p.B;  // bags number below 2^32
        row = b * p.T + t;
      }
    }
    lr[tid] = row;
    ll[tid] = il;
  }
  __syncthreads();

  // sort by key and lookup, by counting: 4 threads per pair each compare it
  // with a quarter of the pairs
  {
    const int i = tid >> 2, part = tid & 3;
    const uint64_t ki = order.pair[i];
    uint32_t before = 0;
    const ulonglong2* quarter = reinterpret_cast<const ulonglong2*>(order.pair + part * (P / 4));
#pragma unroll 8
    for (int v = 0; v < P / 8; ++v) {
      const ulonglong2 k2 = quarter[v];
      before += k2.x < ki;
      before += k2.y < ki;
    }
    before += __shfl_xor(before, 1);
    before += __shfl_xor(before, 2);
    const uint32_t rank = i < cnt ? before : static_cast<uint32_t>(i);
    if (part == 0) {
      mk[rank] = static_cast<uint32_t>(ki >> 32);
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
  // two chains of additions per run (a 32-bit sum of n terms in one chain rounds
  // about as far off as sqrt(n / 2) last places)
  float acc[2][EPL] = {};
  // the group's first run began in an earlier group's pairs
  bool head = q0 > 0 && nq > 0 && mk[q0] == mk[q0 - 1];
  bool tail = false;  // its last run goes on in the next group's pairs
  int start = q0;     // where its current run begins
  float sum[EPL];
  auto run_sum = [&] {
#pragma unroll
    for (int r = 0; r < EPL; ++r) sum[r] = acc[0][r] + acc[1][r];
  };
#pragma unroll 1
  for (int u0 = 0; u0 < S; u0 += U) {
    if (u0 > 0) request(u0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = q0 + u0 + u;
      if (u0 + u < nq) {
        const float f = __shfl(wf, base_lane + u0 + u);
#pragma unroll
        for (int r = 0; r < EPL; ++r) acc[u & 1][r] += p.mean ? g[u][r] * f : g[u][r];
        const bool ends = (ends_mask >> (u0 + u)) & 1u;
        tail = !ends;
        if (ends) {
          run_sum();
          if (head) {
#pragma unroll
            for (int r = 0; r < EPL; ++r) headv[grp][LPB * r + gl] = sum[r];
            head = false;
          } else {
            deposit(sum, start);
          }
          start = q + 1;
#pragma unroll
          for (int r = 0; r < EPL; ++r) acc[0][r] = acc[1][r] = 0.f;
        }
      }
    }
  }
  run_sum();
  const bool thru = head && tail;  // all of its pairs lie inside one run
  if (thru) {
#pragma unroll
    for (int r = 0; r < EPL; ++r) headv[grp][LPB * r + gl] = sum[r];
  }
  if (gl == 0) through[grp] = thru ? 1u : 0u;
  __syncthreads();
  if (tail && !thru) {
    float odd[EPL] = {};
    for (int k = grp + 1; k < NG; k += 2) {
#pragma unroll
      for (int r = 0; r < EPL; ++r) odd[r] += headv[k][LPB * r + gl];
      if (!through[k] || k + 1 >= NG) break;
#pragma unroll
      for (int r = 0; r < EPL; ++r) sum[r] += headv[k + 1][LPB * r + gl];
      if (!through[k + 1]) break;
    }
#pragma unroll
    for (int r = 0; r < EPL; ++r) sum[r] += odd[r];
    deposit(sum, start);
  }
}

// Lookups of a region: one item per bag, whole tables of at least 1024 lookups together
// (smaller ones would leave the last piece of each mostly empty); else the whole
// batch, whose tables begin where only the device knows.
static uint32_t region_len(const KParams& p) {
  if (!keygen_counts(p)) return static_cast<uint32_t>(p.N);
  const uint64_t tables = (1024 + static_cast<uint64_t>(p.B) - 1) / p.B;
  return static_cast<uint32_t>(p.B * (tables < p.T ? tables : p.T));
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
  Regions regions;
  regions.len = region_len(p);
  regions.pieces = (regions.len + piece_cut<P>() - 1) / piece_cut<P>();
  const uint64_t count = (static_cast<uint64_t>(p.N) + regions.len - 1) / regions.len;
  const dim3 grid(static_cast<uint32_t>(count * regions.pieces), (p.d + LPB * EPL - 1) / (LPB * EPL));
  const uint32_t* keys = pairs != nullptr ? pairs->keys : nullptr;
  const uint32_t* rows = pairs != nullptr ? pairs->rows : nullptr;
  const float* il = pairs != nullptr ? pairs->inv_len : nullptr;
  const dim3 block(4 * P);
  const uint32_t lds = regions.len * 4;  // the region's keys
  hipEvent_t before = nullptr, after = nullptr;
  if (!REC) reduce_events(&before, &after);
  const auto kernel = p.idx32 ? deposit_pieces_kernel<EPL, LPB, P, SIGN, true, REC, GT>
                              : deposit_pieces_kernel<EPL, LPB, P, SIGN, false, REC, GT>;
  if (before != nullptr)  // the timing hook: the dispatch records both events
    hipExtLaunchKernelGGL(kernel, grid, block, lds, stream, before, after, 0u, dst, scale, p, indices,
                          offsets, keys, rows, il, grad, rec.keys, rec.ids, regions);
  else
    hipLaunchKernelGGL(kernel, grid, block, lds, stream, dst, scale, p, indices, offsets, keys, rows,
                       il, grad, rec.keys, rec.ids, regions);
  return hipGetLastError();
}

// Pieces of 64 lookups for short regions, of 128 for longer ones, whose scan fewer
// workgroups then repeat.  Backward, 64 / 128 (N lookups in regions of R): N = R = 1024 13.2 / 14.2 us,
// 26 x 1024 18.3 / 21.5 us, 26 x 2048 28.7 / 28.3 us, N = R = 4096 20.4 / 17.4 us, 13 x 4096
// 31.4 / 27.7 us.  256: N = R = 8192 step 30.1 us against 27.2 by 128, 26 x 2048 backward 35.7 us.
constexpr uint32_t kSmallPieceRegion = 1536;
template <int EPL, int LPB, bool SIGN, bool REC, typename GT, typename... A>
static hipError_t launch_pieces_p(float* dst, float scale, const KParams& p, A... a) {
  if (region_len(p) <= kSmallPieceRegion)
    return launch_pieces_t<EPL, LPB, 64, SIGN, REC, GT>(dst, scale, p, a...);
  return launch_pieces_t<EPL, LPB, 128, SIGN, REC, GT>(dst, scale, p, a...);
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
                                const void* offsets, const GroupedPairs* pairs, const void* grad,
                                uint32_t* rec_keys, uint32_t* rec_ids, hipStream_t stream) {
  const PieceRecords rec{rec_keys, rec_ids};
  if (p.rows_bf16)
    return launch_pieces_g<true, uint16_t>(sums, 1.f, p, indices, offsets, pairs, grad, rec, stream);
  return launch_pieces_g<true, float>(sums, 1.f, p, indices, offsets, pairs, grad, rec, stream);
}

// Where one kernel is the faster form of the deposit: one item per bag (the lookups of
// a table are then T*B / T consecutive ones, and need no keygen), up to 65536
// lookups, and regions for which the workgroups' scans (N / 112 of them, each of
// a region) cost less than the sort's launches.  Backward, pieces / grouped, uniform or
// Zipf(1.1) tokens of 10^7 rows, d = 128, Z = 32: 4 x 256 13.3 / 26 us, 26 x 512 13.8 / 27.8 us, 1 x
// 4096 17.6 / 27.4 us, 26 x 2048 29 / 35.5 us, 13 x 4096 27.9 / 34.2 us; 26 x 4096 52.1 / 52.1 us, of three tokens a
// table 34.2 / 26.1 us; bags of 9 to 10 items 35 to 37 us (with its keygen) against 32 to 35 us.
// Training steps: 1 x 8192 27.2 / 31.7 us, 2 x 8192 28.1 / 32.9 us, 4 x 8192 36.1 / 35.6 us, 1 x 12288 32.5 / 32.8 us,
// 1 x 16384 38.1 / 33.0 us, 6 x 10240 62.8 / 46.0 us.  Beyond 8192 lookups per table a token that
// fills its table would also be rounded more often than by the grouped deposit.
// A deposit costs a 64-byte line update at the memory side, about 20 G/s, for
// every line of every chunk: the third bound keeps that below the chain's time.
constexpr int64_t kPieceMaxItems = 1 << 16;
constexpr int64_t kPieceMaxLines = 3 << 19;
constexpr uint32_t kPieceRegion = 8192;
constexpr int64_t kPieceScans = 1 << 28;
bool deposits_by_piece(const KParams& p) {
  return p.N <= kPieceMaxItems && keygen_counts(p) && region_len(p) <= kPieceRegion &&
         p.N * region_len(p) <= kPieceScans &&
         p.N * static_cast<int64_t>(p.C) * (p.Z / 16 + 1) <= kPieceMaxLines;
}

// Records replace a longer chain (the sparse branch's 26 launches) and are worth
// longer regions: list of N = R lookups, d = 64, Z = 16, 4 M elements, by tile / general: 8192
// 49 / 123 us, 16384 62 / 126 us, 22500 in bags 75 / 132 us; 30000 124 / 128 us.
// The keys of a region (96 KB at most) share a workgroup's 160 KB of LDS with 24 KB.
constexpr int64_t kRecordItems = 1 << 18;
constexpr uint32_t kRecordRegion = 24576;
bool pieces_fit(const KParams& p) {
  return p.N <= kRecordItems && region_len(p) <= kRecordRegion;
}

}  // namespace pss
