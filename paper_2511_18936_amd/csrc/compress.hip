// Compress-append (Algorithm 1, the steps that project, append, evict and
// prune).
//
// Several new tokens per sequence: every vector leaving the ring is read before
// a new token overwrites its slot, by the same workgroup (short appends) or in
// an earlier launch.  One new token (a decode step): one launch, step_kernel,
// which evicts the slot's old vector before it writes the new one.
//   evict_kernel   one wave per ring vector that leaves the buffer: top-k of
//                  its stored values, packed into its page slot
//   insert_kernel  one workgroup per (sequence, kv head, role) and some pages:
//                  rotation x . P in float64 on MFMA, rounded once to the
//                  storage type; tokens still inside the buffer go to their
//                  ring slot, the others are pruned and packed at once
//   few_kernel     the same for few tokens of many (sequence, kv head, role): one
//                  wave per 8 tokens, float64 VALU
//   step_kernel    a decode step: one workgroup of four waves per (sequence,
//                  kv head, role), each wave a quarter of P's rows; the same
//                  rounding, ring write or pruning, and the eviction.  In
//                  swan_decode_step the key workgroup also rotates the step's
//                  queries of its kv head (q_hat for the attention that
//                  follows) with the same rows of P_QK
//
// Top-k (Sec. 4.3, ranking the stored values, ties to the lower index): each
// lane holds dims 2l and 2l+1; the key (|x| bits << 8) | (255 - dim) is unique
// and orders by magnitude, then by lower index.  A binary search over the key
// bits with wave ballots finds the k-th largest key; the selected entries are
// then numbered in ascending dim order with mbcnt and written to the page.
#include <limits.h>
#include <math.h>
#include <string.h>

#include <type_traits>

#include "swan_cache_ops.h"
#include "swan_device.h"

namespace swan {

// Write the top-k of a 128-vector of stored values (lane holds elements 2l,
// 2l+1) into page slot `slot` of the page at `page`, in page format F (the
// values as stored, or rounded to E4M3; the selection ranks the stored values).
template <typename F>
__device__ __forceinline__ void select_and_pack(typename Store<typename Fmt<F>::Elem>::Bits x0,
                                                typename Store<typename Fmt<F>::Elem>::Bits x1,
                                                int k, char* page, int slot, int lane) {
  using St = Store<typename Fmt<F>::Elem>;
  using Key = typename std::conditional<(St::kMagBits + 8 > 32), uint64_t, uint32_t>::type;
  constexpr int kKeyBits = St::kMagBits + 8;
  const Key key0 = ((Key)St::mag(x0) << 8) | (Key)(255 - 2 * lane);
  const Key key1 = ((Key)St::mag(x1) << 8) | (Key)(255 - (2 * lane + 1));
  Key thr = 0;
  for (int bit = kKeyBits - 1; bit >= 0; --bit) {
    const Key cand = thr | ((Key)1 << bit);
    const int cnt = __popcll(__ballot(key0 >= cand)) + __popcll(__ballot(key1 >= cand));
    if (cnt >= k) thr = cand;
  }
  const bool s0 = key0 >= thr;
  const bool s1 = key1 >= thr;
  const uint64_t m0 = __ballot(s0);
  const uint64_t m1 = __ballot(s1);
  const int e0 = popc_below(m0) + popc_below(m1);
  const int e1 = e0 + (s0 ? 1 : 0);
  constexpr int VB = Fmt<F>::kValBytes, CB = Fmt<F>::kChunkBytes, GV = CB / VB;
  const int kp = kpad_of(k);
  char* vals = page + slot * CB;
  char* idxs = page + (int64_t)kPage * kp * VB + slot * 8;
  auto put = [&](int e, typename St::Bits x) {
    char* dst = vals + (e / GV) * (kPage * CB) + (e % GV) * VB;
    if constexpr (std::is_same<F, E4M3V>::value)
      *(uint8_t*)dst = (uint8_t)f16_bits_to_e4m3(x);
    else
      *(typename St::Bits*)dst = x;
  };
  if (s0) {
    put(e0, x0);
    idxs[(e0 / 8) * 512 + (e0 % 8)] = (char)(2 * lane);
  }
  if (s1) {
    put(e1, x1);
    idxs[(e1 / 8) * 512 + (e1 % 8)] = (char)(2 * lane + 1);
  }
  // padding entries k .. kp-1: value +0 at the lowest unselected dims, so that
  // the indices of a token stay distinct
  const int npad = kp - k;
  if (npad > 0) {
    const uint64_t n0 = __ballot(!s0);
    const uint64_t n1 = __ballot(!s1);
    const int r0 = popc_below(n0) + popc_below(n1);
    const int r1 = r0 + (s0 ? 0 : 1);
    if (!s0 && r0 < npad) {
      const int e = k + r0;
      put(e, 0);
      idxs[(e / 8) * 512 + (e % 8)] = (char)(2 * lane);
    }
    if (!s1 && r1 < npad) {
      const int e = k + r1;
      put(e, 0);
      idxs[(e / 8) * 512 + (e % 8)] = (char)(2 * lane + 1);
    }
  }
}

__host__ __device__ __forceinline__ int evict_begin(int len_old, int bb) {
  return len_old > bb ? len_old - bb : 0;
}

// tokens that leave the ring in this call: positions [begin, end)
__host__ __device__ __forceinline__ int evict_end(int len_old, int n_new, int bb) {
  const int lim = len_old + n_new - bb;
  return len_old < lim ? len_old : lim;
}

template <typename F>
__global__ __launch_bounds__(64) void evict_kernel(CompressLaunch a) {
  using St = Store<typename Fmt<F>::Elem>;
  const int lane = threadIdx.x;
  int w = blockIdx.x;
  const int e = w % a.max_evict;
  w /= a.max_evict;
  const int role = w & 1;
  w >>= 1;
  const int h = w % a.Hkv;
  const int b = w / a.Hkv;
  const int len_old = a.tab.len[b];
  const int p0 = evict_begin(len_old, a.bb);
  const int p1 = evict_end(len_old, a.tab.nnew[b], a.bb);
  const int p = p0 + e;
  if (p >= p1) return;
  const typename St::Bits* ring =
      (const typename St::Bits*)(role ? a.v_ring : a.k_ring) +
      (((int64_t)b * a.Hkv + h) * a.bb + (p % a.bb)) * kD;
  const typename St::Bits x0 = ring[2 * lane];
  const typename St::Bits x1 = ring[2 * lane + 1];
  const int k = a.tab.kact[role][b];
  const int64_t pbytes = page_bytes_of(Fmt<F>::kValBytes, k);
  char* page = (char*)(role ? a.v_pages : a.k_pages) + a.tab.page_off[role][b] +
               ((int64_t)h * a.n_pages_cap + p / kPage) * pbytes;
  select_and_pack<F>(x0, x1, k, page, p % kPage, lane);
}

// ---------------------------------------------------------------------------
// several new tokens
// ---------------------------------------------------------------------------
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kInsWaves = 8;
constexpr int kXStride = kD + 4;  // LDS row of one token's 128 float32 values (+ pad)
constexpr int kIdxStride = kD + 8;  // LDS row of one token's kept dims (+ pad)

// sum over the 8 lanes of a token, in every lane (lanes xor 1, 2, then the
// mirror of the 8)
__device__ __forceinline__ int sum8(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);   // quad_perm 1 0 3 2
  v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);   // quad_perm 2 3 0 1
  v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false);  // row_half_mirror
  return v;
}
// sum over the lanes of the token below this one (sub: lane in the token)
__device__ __forceinline__ int below8(int v, int sub) {
  int y = v;
  const int a = __builtin_amdgcn_update_dpp(0, y, 0x111, 0xF, 0xF, false);  // row_shr 1
  y += sub >= 1 ? a : 0;
  const int b = __builtin_amdgcn_update_dpp(0, y, 0x112, 0xF, 0xF, false);
  y += sub >= 2 ? b : 0;
  const int c = __builtin_amdgcn_update_dpp(0, y, 0x114, 0xF, 0xF, false);
  y += sub >= 4 ? c : 0;
  return y - v;
}

// Eight lanes per token, 16 dims each (lane sub: dims 16 sub ..): the token's k
// kept pairs, ties to the lower dim, packed in ascending order into its LDS row
// (values, over the row itself, which the lanes have read by then) and `idx`
// (dims); entries k..kp-1 are the padding, value +0 at the lowest dims not kept.
// Lanes with on == false write nothing.
template <typename St>
__device__ __forceinline__ void select_rows(typename St::Bits* row, uint8_t* idx, int k, int kp,
                                            int sub, bool on) {
  using Bits = typename St::Bits;
  constexpr int W = (int)sizeof(Bits) * 16 / 4;  // this lane's words
  uint32_t w[W];
#pragma unroll
  for (int c = 0; c < W / 4; ++c) {
    const u32x4 v = *(const u32x4*)(row + 16 * sub + c * (16 / (int)sizeof(Bits)));
    w[4 * c] = v.x;
    w[4 * c + 1] = v.y;
    w[4 * c + 2] = v.z;
    w[4 * c + 3] = v.w;
  }
  // The k-th largest magnitude, from the top bit down, or as soon as a candidate
  // has exactly k magnitudes at or above it, that candidate: the same k are kept.
  // (The wave stops when its 8 tokens have: for float32 after about 20 of 31 bits.)
  uint32_t thr = 0u;
  bool open = true;
#pragma unroll 1
  for (int bit = St::kMagBits - 1; bit >= 0 && __ballot(open) != 0ull; --bit) {
    const uint32_t cand = thr | (1u << bit);
    int cnt = 0;
#pragma unroll
    for (int i = 0; i < W; ++i) {
      if constexpr (sizeof(Bits) == 2)  // two magnitudes per word: bits 15 and 31 stay when >=
        cnt += __popc((((w[i] & 0x7FFF7FFFu) | 0x80008000u) - cand * 0x10001u) & 0x80008000u);
      else
        cnt += (w[i] & 0x7FFFFFFFu) >= cand ? 1 : 0;
    }
    const int all = sum8(cnt);
    thr = open && all >= k ? cand : thr;
    open = open && all != k;
  }
  auto bits_of = [&](int i) -> uint32_t {
    if constexpr (sizeof(Bits) == 2) return (w[i >> 1] >> (16 * (i & 1))) & 0xFFFFu;
    else return w[i];
  };
  uint32_t gt = 0u, eq = 0u;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const uint32_t m = St::mag((Bits)bits_of(i));
    gt |= m > thr ? 1u << i : 0u;
    eq |= m == thr ? 1u << i : 0u;
  }
  const int ngt = sum8(__popc(gt)), neq = __popc(eq);
  int quota = k - ngt - below8(neq, sub);  // of this lane's ties, the lowest first
  quota = quota < 0 ? 0 : quota > neq ? neq : quota;
  while (__popc(eq) > quota) eq &= ~(0x80000000u >> __clz(eq));
  const uint32_t kept = gt | eq;
  int e = below8(__popc(kept), sub);
  const int r0 = 16 * sub - e;  // dims not kept below this lane's
  if (!on) return;
#pragma unroll
  for (int i = 0; i < 16; ++i)
    if ((kept >> i) & 1u) {
      row[e] = (Bits)bits_of(i);
      idx[e] = (uint8_t)(16 * sub + i);
      ++e;
    }
  if (kp > k) {  // uniform
    uint32_t rest = ~kept & 0xFFFFu;
    for (int r = r0; rest != 0u && r < kp - k; ++r) {
      idx[k + r] = (uint8_t)(16 * sub + __builtin_ctz(rest));
      rest &= rest - 1u;
    }
    if (sub < kp - k) row[k + sub] = 0;
  }
}

// The (sequence, kv head, role) and the group of a workgroup.  even: as many blocks in
// every sequence, grid (units, groups); else grid (all workgroups), the sequence with the
// most blocks first, its workgroups numbered together, group by group: tab.nsplit (what
// a decode call keeps there, an append has no use for) holds each one's first number
// times 64, plus the sequence.  So no number is left out and long and short do not alternate:
// workgroups go to the 8 XCDs, and in each to 4 shader engines, round-robin, and where
// every second one was short, or most had nothing to do, the others fell to the same few
// processors (us, float32: 4096 units x 512 tokens, 8 blocks and 1 in two groups side by
// side 3190, now 1750; 1024 units x 80, 64 and 16 in two groups 87, 61).
__device__ __forceinline__ void place(const CompressLaunch& a, bool even, int lane, int& b,
                                      int& h, int& role, int& grp) {
  const unsigned per_seq = 2 * a.Hkv, id = blockIdx.x;
  unsigned w;
  if (even) {
    b = (int)(id / per_seq);
    grp = (int)blockIdx.y;
    w = id - (unsigned)b * per_seq;
  } else {
    const bool upto = lane < a.B && ((uint32_t)a.tab.nsplit[lane] >> 6) <= id;
    const uint32_t at = (uint32_t)a.tab.nsplit[__popcll(__ballot(upto)) - 1];
    b = (int)(at & 63u);
    w = id - (at >> 6);
    grp = (int)(w / per_seq);
    w -= (unsigned)grp * per_seq;
  }
  role = (int)(w & 1);
  h = (int)(w >> 1);
}

// `blocks` blocks of `bt` positions per workgroup: 64 (pages), or, when no new
// token is pruned (every sequence's fit its buffer), 16, 32 or 64.  evict: the
// workgroup first prunes and packs the vectors that leave the buffer: all of its
// unit's (it has all of the unit's blocks), or, when none of the new tokens is
// pruned, those whose slots its own tokens take.  Wave w holds columns 16 w .. of P
// in registers for all of the workgroup's blocks.  Per block: the tokens' rows to
// LDS, x . P on v_mfma_f64_16x16x4 (32 per 16 tokens and 16 columns), the rounded
// rows to LDS, then the dense rows to the ring and the kept pairs, packed in LDS,
// to the page (a wave's store is 1 KiB contiguous).
//
// What bounds it: many tokens, the float64 MFMAs (64 cycles each; two workgroups
// share a compute unit, one's selection under the other's MFMAs); few, the chain
// of loads and barriers.
template <typename F>
__global__ __launch_bounds__(64 * kInsWaves) __attribute__((amdgpu_waves_per_eu(4)))
void insert_kernel(CompressLaunch a, bool even, int blocks, int bt, bool evict) {
  using T = typename Fmt<F>::Elem;
  using St = Store<T>;
  using Bits = typename St::Bits;
  constexpr int VB = Fmt<F>::kValBytes, CB = Fmt<F>::kChunkBytes;
  constexpr int EV = 16 / (int)sizeof(T);                     // elements per 16-byte load
  constexpr int RS = kD + 16 / (int)sizeof(T);                // LDS row of stored values
  __shared__ __attribute__((aligned(16))) float xs[kPage * kXStride];
  __shared__ __attribute__((aligned(16))) Bits rows[kPage * RS];  // as stored
  __shared__ __attribute__((aligned(16))) uint8_t idxs[kPage * kIdxStride];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 15, g = lane >> 4;
  int b, h, role, grp;
  place(a, even, lane, b, h, role, grp);
  const int nnew = a.tab.nnew[b];
  if (nnew == 0) return;  // uniform
  const int len_old = a.tab.len[b], len_new = len_old + nnew;
  // no new token is pruned when all fit the buffer: blocks then begin anywhere
  const bool fits = nnew <= a.bb;
  const int org = fits ? len_old : len_old & ~(kPage - 1);
  const int nblk = (len_new - org + bt - 1) / bt;
  if (!even && nblk > blocks) {  // the groups of a unit as long as each other
    const int ng = (nblk + blocks - 1) / blocks;
    blocks = (nblk + ng - 1) / ng;
  }
  const int blk0 = grp * blocks, blk1 = blk0 + blocks < nblk ? blk0 + blocks : nblk;
  if (blk0 >= blk1) return;  // uniform
  const T* x = (const T*)(role ? a.v_new : a.k_new) + ((int64_t)b * a.Hkv + h) * a.n_new * kD;
  const float* Prole = role ? a.P_vo : a.P_qk;
  // the k dims of an MFMA step in any order, the same for x and P: lane group g
  // takes dims 32 g + s in step s, so that a lane's x are contiguous
  float pr[32];
  if (Prole) {
    const float* P = Prole + (int64_t)h * kD * kD + (int64_t)(32 * g) * kD + 16 * wave + m;
#pragma unroll
    for (int s = 0; s < 32; ++s) pr[s] = P[s * kD];
  }
  const int k = a.tab.kact[role][b], kp = kpad_of(k);
  const int64_t pbytes = page_bytes_of(VB, k);
  char* pages = (char*)(role ? a.v_pages : a.k_pages) + a.tab.page_off[role][b] +
                (int64_t)h * a.n_pages_cap * pbytes;
  Bits* ring = (Bits*)(role ? a.v_ring : a.k_ring) + ((int64_t)b * a.Hkv + h) * a.bb * kD;
  if (evict) {
    int p0 = evict_begin(len_old, a.bb), p1 = evict_end(len_old, nnew, a.bb);
    if (fits) {
      const int q0 = org + blk0 * bt - a.bb, q1 = org + blk1 * bt - a.bb;
      p0 = p0 > q0 ? p0 : q0;
      p1 = p1 < q1 ? p1 : q1;
    }
    for (int p = p0 + wave; p < p1; p += kInsWaves) {
      const Bits* old = ring + (int64_t)(p % a.bb) * kD;
      const Bits o0 = old[2 * lane], o1 = old[2 * lane + 1];
      select_and_pack<F>(o0, o1, k, pages + (int64_t)(p / kPage) * pbytes, p % kPage, lane);
    }
  }
  const int first_dense = len_new - a.bb;  // positions from here on stay in the buffer
  for (int blk = blk0; blk < blk1; ++blk) {
    const int pos0 = org + blk * bt;
    const int lo = len_old > pos0 ? len_old - pos0 : 0;          // the block's new tokens
    const int hi = len_new - pos0 < bt ? len_new - pos0 : bt;
    for (int v = tid; v < bt * kD / EV; v += 64 * kInsWaves) {
      const int t = v / (kD / EV), c = v % (kD / EV);
      if (t < (lo & ~15) || t >= ((hi + 15) & ~15)) continue;
      u32x4 q = {0u, 0u, 0u, 0u};
      if (t >= lo && t < hi) q = *(const u32x4*)(x + (int64_t)(pos0 + t - len_old) * kD + c * EV);
      float4* dst = (float4*)(xs + t * kXStride + c * EV);
      if constexpr (sizeof(T) == 2) {
        dst[0] = make_float4(f16_bits_to_f32(q.x & 0xFFFFu), f16_bits_to_f32(q.x >> 16),
                             f16_bits_to_f32(q.y & 0xFFFFu), f16_bits_to_f32(q.y >> 16));
        dst[1] = make_float4(f16_bits_to_f32(q.z & 0xFFFFu), f16_bits_to_f32(q.z >> 16),
                             f16_bits_to_f32(q.w & 0xFFFFu), f16_bits_to_f32(q.w >> 16));
      } else {
        dst[0] = make_float4(__uint_as_float(q.x), __uint_as_float(q.y), __uint_as_float(q.z),
                             __uint_as_float(q.w));
      }
    }
    __syncthreads();  // the rows; the first time also the evictions' ring reads
    // 16 tokens at a time; result layout: register v of lane l is token 16 T + 4 v +
    // l / 16, dim 16 wave + l % 16
#pragma unroll 1
    for (int T = lo / 16; T < (hi + 15) / 16; ++T) {
      f64x4 acc = {0.0, 0.0, 0.0, 0.0};
      if (Prole) {
#pragma unroll
        for (int s4 = 0; s4 < 8; ++s4) {
          const float4 xv = *(const float4*)(xs + (16 * T + m) * kXStride + 32 * g + 4 * s4);
          const float xe[4] = {xv.x, xv.y, xv.z, xv.w};
#pragma unroll
          for (int i = 0; i < 4; ++i)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)xe[i], (double)pr[4 * s4 + i], acc,
                                                       0, 0, 0);
        }
      } else {  // values already in the rotated basis (P_VO absorbed into W_V)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          acc[v] = (double)xs[(16 * T + 4 * v + g) * kXStride + 16 * wave + m];
      }
      Bits y[4];
      bool nan = false;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if constexpr (sizeof(Bits) == 2) y[v] = f64_to_f16_bits_fast(acc[v]);
        else y[v] = St::from_f64(acc[v]);
        nan |= acc[v] != acc[v];
      }
      if constexpr (sizeof(Bits) == 2) {
        if (nan)
#pragma unroll
          for (int v = 0; v < 4; ++v) y[v] = one_nan(y[v]);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) rows[(16 * T + 4 * v + g) * RS + 16 * wave + m] = y[v];
    }
    __syncthreads();
    // dense tokens to the ring: slot pos % b
    const int dlo = first_dense > pos0 + lo ? first_dense - pos0 : lo;
    for (int v = tid + dlo * (kD / EV); v < hi * (kD / EV); v += 64 * kInsWaves) {
      const int t = v / (kD / EV), c = v % (kD / EV);
      *(u32x4*)(ring + (int64_t)((pos0 + t) % a.bb) * kD + c * EV) =
          *(const u32x4*)(rows + t * RS + c * EV);
    }
    // the others pruned: slots [lo, plo) of the block's page
    const int phi = first_dense - pos0 < hi ? first_dense - pos0 : hi;
    if (phi > lo) {  // uniform
      const int t = 8 * wave + (lane >> 3), sub = lane & 7;
      if (8 * wave < phi && 8 * wave + 8 > lo) {
        const bool on = t >= lo && t < phi;
        select_rows<St>(rows + t * RS, idxs + t * kIdxStride, k, kp, sub, on);
      }
      __syncthreads();
      char* page = pages + (int64_t)(pos0 / kPage) * pbytes;
      if (lane >= lo && lane < phi) {
        const char* row = (const char*)(rows + lane * RS);
        for (int c = wave; c < kp * VB / CB; c += kInsWaves) {
          const u32x4 v = *(const u32x4*)(row + 16 * c);
          if constexpr (std::is_same<F, E4M3V>::value) {
            uint32_t q[2] = {0u, 0u};
#pragma unroll
            for (int i = 0; i < 8; ++i)
              q[i >> 2] |= f16_bits_to_e4m3((v[i >> 1] >> (16 * (i & 1))) & 0xFFFFu)
                           << (8 * (i & 3));
            *(u32x2*)(page + c * (kPage * CB) + lane * CB) = u32x2{q[0], q[1]};
          } else {
            *(u32x4*)(page + c * (kPage * CB) + lane * CB) = v;
          }
        }
        char* ip = page + (int64_t)kPage * kp * VB;
        for (int c = wave; c < kp / 8; c += kInsWaves)
          *(u32x2*)(ip + c * 512 + lane * 8) = *(const u32x2*)(idxs + lane * kIdxStride + 8 * c);
      }
    }
    __syncthreads();  // the rows have been read
  }
}

// Few tokens of many units: one wave per kFewTokens of them, nothing shared, so that
// every unit's chain of loads is in flight at once where insert_kernel takes several
// rounds of workgroups of 8 waves.  Lane l rotates to dims 2 l and 2 l + 1, all 128
// rows of P in batches of 32.  evict: the wave has all of its unit's new tokens and
// first prunes and packs the vectors that leave the buffer (each lane reads the two
// elements it overwrites later).
constexpr int kFewTokens = 8;

template <typename F>
__global__ __launch_bounds__(64) void few_kernel(CompressLaunch a, bool even, bool evict) {
  using T = typename Fmt<F>::Elem;
  using St = Store<T>;
  __shared__ __attribute__((aligned(16))) double xs[kD][kFewTokens];
  const int lane = threadIdx.x;
  int b, h, role, grp;
  place(a, even, lane, b, h, role, grp);
  const int t0 = grp * kFewTokens;
  const int nnew = a.tab.nnew[b];
  if (t0 >= nnew) return;
  const int nt = nnew - t0 < kFewTokens ? nnew - t0 : kFewTokens;
  const T* x = (const T*)(role ? a.v_new : a.k_new) +
               (((int64_t)b * a.Hkv + h) * a.n_new + t0) * kD;
#pragma unroll
  for (int t = 0; t < kFewTokens; ++t) {
    double v0 = 0.0, v1 = 0.0;
    if (t < nt) {
      v0 = (double)(float)x[(int64_t)t * kD + 2 * lane];
      v1 = (double)(float)x[(int64_t)t * kD + 2 * lane + 1];
    }
    xs[2 * lane][t] = v0;
    xs[2 * lane + 1][t] = v1;
  }
  const int len_old = a.tab.len[b], len_new = len_old + nnew;
  const int k = a.tab.kact[role][b];
  const int64_t pbytes = page_bytes_of(Fmt<F>::kValBytes, k);
  char* pages = (char*)(role ? a.v_pages : a.k_pages) + a.tab.page_off[role][b] +
                (int64_t)h * a.n_pages_cap * pbytes;
  typename St::Bits* ring = (typename St::Bits*)(role ? a.v_ring : a.k_ring) +
                            ((int64_t)b * a.Hkv + h) * a.bb * kD;
  if (evict) {
    const int p1 = evict_end(len_old, nnew, a.bb);
    for (int p = evict_begin(len_old, a.bb); p < p1; ++p) {
      const typename St::Bits* old = ring + (int64_t)(p % a.bb) * kD;
      const typename St::Bits o0 = old[2 * lane], o1 = old[2 * lane + 1];
      select_and_pack<F>(o0, o1, k, pages + (int64_t)(p / kPage) * pbytes, p % kPage, lane);
    }
  }
  __syncthreads();  // xs
  double acc0[kFewTokens], acc1[kFewTokens];
  const float* Prole = role ? a.P_vo : a.P_qk;
  if (!Prole) {  // values already in the rotated basis (P_VO absorbed into W_V)
#pragma unroll
    for (int t = 0; t < kFewTokens; ++t) {
      acc0[t] = xs[2 * lane][t];
      acc1[t] = xs[2 * lane + 1][t];
    }
  } else {
    const float2* P = (const float2*)(Prole + (int64_t)h * kD * kD) + lane;
#pragma unroll
    for (int t = 0; t < kFewTokens; ++t) acc0[t] = acc1[t] = 0.0;
#pragma unroll 32
    for (int i = 0; i < kD; ++i) {
      const float2 pr = P[i * (kD / 2)];
      const double p0 = (double)pr.x, p1 = (double)pr.y;
#pragma unroll
      for (int t = 0; t < kFewTokens; ++t) {
        const double xv = xs[i][t];
        acc0[t] = fma(xv, p0, acc0[t]);
        acc1[t] = fma(xv, p1, acc1[t]);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < kFewTokens; ++t) {
    if (t >= nt) break;
    const typename St::Bits y0 = St::from_f64(acc0[t]);
    const typename St::Bits y1 = St::from_f64(acc1[t]);
    const int pos = len_old + t0 + t;
    if (pos >= len_new - a.bb) {  // stays dense: ring slot pos % b
      typename St::Bits* r = ring + (int64_t)(pos % a.bb) * kD;
      r[2 * lane] = y0;
      r[2 * lane + 1] = y1;
    } else {  // pruned on arrival
      select_and_pack<F>(y0, y1, k, pages + (int64_t)(pos / kPage) * pbytes, pos % kPage, lane);
    }
  }
}

// A decode step's append, one new token per sequence: one workgroup of four
// waves per (sequence, kv head, role).  Wave s rotates with rows 32 s .. 32 s
// + 31 of P, its 32 row loads issued together, so the rotation costs one
// memory latency rather than a wave's walk over all 128 rows; the four
// float64 partials meet in LDS as (s0 + s1) + (s2 + s3), and wave 0 rounds the
// sum once and writes the ring slot (or, with no buffer, prunes and packs the
// token), after it has pruned and packed the vector that leaves the buffer
// from that same slot.  QG > 0 (swan_decode_step): the key workgroup also
// rotates the QG query rows of its kv head, q_hat = q . P_QK[h] * qmult in
// float32, quarter s in wave s with even and odd rows in two accumulators
// that are added, the quarters meeting as (q0 + q1) + (q2 + q3): the order of
// qrot_kernel, so q_hat has the same bits as from that kernel.
template <typename F, int QG>
__global__ __launch_bounds__(256) void step_kernel(CompressLaunch a) {
  using T = typename Fmt<F>::Elem;
  using St = Store<T>;
  constexpr int NQ = QG > 0 ? QG : 1;
  __shared__ double xs[kD];
  __shared__ double part[4][kD];
  __shared__ float qs[NQ][kD];
  __shared__ float qpart[NQ][4][kD];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int w = blockIdx.x;
  const int role = w & 1;
  w >>= 1;
  const int h = w % a.Hkv;
  const int b = w / a.Hkv;
  if (a.tab.nnew[b] == 0) return;  // uniform over the workgroup
  const bool with_q = QG > 0 && role == 0;
  const T* x = (const T*)(role ? a.v_new : a.k_new) + ((int64_t)b * a.Hkv + h) * a.n_new * kD;
  const int64_t q0 = ((int64_t)b * a.Hq + (int64_t)h * NQ) * kD;  // first query row
  if (tid < kD) xs[tid] = (double)(float)x[tid];
  if (with_q)
    for (int i = tid; i < NQ * kD; i += 256) qs[i / kD][i % kD] = (float)((const T*)a.q)[q0 + i];
  const int len_old = a.tab.len[b];
  const int k = a.tab.kact[role][b];
  const int64_t pbytes = page_bytes_of(Fmt<F>::kValBytes, k);
  char* pages = (char*)(role ? a.v_pages : a.k_pages) + a.tab.page_off[role][b] +
                (int64_t)h * a.n_pages_cap * pbytes;
  typename St::Bits* ring = (typename St::Bits*)(role ? a.v_ring : a.k_ring) +
                            ((int64_t)b * a.Hkv + h) * a.bb * kD;
  const float* Prole = role ? a.P_vo : a.P_qk;
  float2 pr[32];
  if (Prole) {  // this wave's quarter of P: 32 rows in flight
    const float2* P = (const float2*)(Prole + (int64_t)h * kD * kD + (int64_t)(32 * wave) * kD) +
                      lane;
#pragma unroll
    for (int u = 0; u < 32; ++u) pr[u] = P[u * (kD / 2)];
  }
  // the vector that leaves the buffer (if any) sits in the ring slot the new
  // token takes: wave 0 prunes and packs it first (each lane reads the two
  // elements it overwrites below)
  const int p0 = evict_begin(len_old, a.bb);
  if (wave == 0 && p0 < evict_end(len_old, 1, a.bb)) {
    const typename St::Bits* old = ring + (int64_t)(p0 % a.bb) * kD;
    const typename St::Bits o0 = old[2 * lane];
    const typename St::Bits o1 = old[2 * lane + 1];
    select_and_pack<F>(o0, o1, k, pages + (int64_t)(p0 / kPage) * pbytes, p0 % kPage, lane);
  }
  __syncthreads();  // xs and qs
  if (Prole) {
    double acc0 = 0.0, acc1 = 0.0;
#pragma unroll
    for (int u = 0; u < 32; ++u) {
      const double xv = xs[32 * wave + u];
      acc0 = fma(xv, (double)pr[u].x, acc0);
      acc1 = fma(xv, (double)pr[u].y, acc1);
    }
    part[wave][2 * lane] = acc0;
    part[wave][2 * lane + 1] = acc1;
    if (with_q) {
#pragma unroll
      for (int g = 0; g < NQ; ++g) {
        float e0 = 0.f, o0 = 0.f, e1 = 0.f, o1 = 0.f;  // [even / odd rows][output 2 lane + 0 / 1]
#pragma unroll
        for (int u = 0; u < 32; u += 2) {
          e0 = fmaf(qs[g][32 * wave + u], pr[u].x, e0);
          o0 = fmaf(qs[g][32 * wave + u + 1], pr[u + 1].x, o0);
          e1 = fmaf(qs[g][32 * wave + u], pr[u].y, e1);
          o1 = fmaf(qs[g][32 * wave + u + 1], pr[u + 1].y, o1);
        }
        qpart[g][wave][2 * lane] = e0 + o0;
        qpart[g][wave][2 * lane + 1] = e1 + o1;
      }
    }
  }
  __syncthreads();  // the partials
  if (wave == 0) {
    double y0 = xs[2 * lane], y1 = xs[2 * lane + 1];  // values already rotated (P_VO absorbed)
    if (Prole) {
      y0 = (part[0][2 * lane] + part[1][2 * lane]) + (part[2][2 * lane] + part[3][2 * lane]);
      y1 = (part[0][2 * lane + 1] + part[1][2 * lane + 1]) +
           (part[2][2 * lane + 1] + part[3][2 * lane + 1]);
    }
    const typename St::Bits v0 = St::from_f64(y0);
    const typename St::Bits v1 = St::from_f64(y1);
    const int pos = len_old;
    if (a.bb > 0) {  // stays dense: ring slot pos % b
      typename St::Bits* r = ring + (int64_t)(pos % a.bb) * kD;
      r[2 * lane] = v0;
      r[2 * lane + 1] = v1;
    } else {  // no buffer: pruned on arrival
      select_and_pack<F>(v0, v1, k, pages + (int64_t)(pos / kPage) * pbytes, pos % kPage, lane);
    }
  } else if (wave == 1 && with_q) {
    for (int i = lane; i < NQ * kD; i += 64) {
      const int g = i / kD, j = i % kD;
      a.qhat[q0 + i] =
          ((qpart[g][0][j] + qpart[g][1][j]) + (qpart[g][2][j] + qpart[g][3][j])) * a.qmult;
    }
  }
}

// How an append of several tokens runs.
struct AppendPlan {
  int kernel;      // kAppend...
  int bt;          // positions per block
  int blocks;      // ... per workgroup of insert_kernel
  int groups;      // workgroups of insert or few_kernel per (kv head, role): the most of
                   // any sequence
  int64_t wgs;     // ... of all
  bool even;       // as many blocks in every sequence (and groups within a grid's limit);
                   // else the sequences with the most blocks first:
  uint32_t table[SWAN_MAX_BATCH];  // each one's first workgroup times 64, plus its number
  bool fused;      // that kernel evicts; else an eviction launch goes first
};

// What an append holds, over all sequences, kv heads and roles.
struct AppendWork {
  double blocks = 0, tiles = 0;     // insert_kernel's blocks and their tiles of 16 positions
  double pruning = 0, uneven = 0;   // blocks with tokens pruned; with cut 128-byte lines of 8
  double tokens = 0, waves = 0;     // few_kernel's waves
  double pruned = 0, evicted = 0;   // new tokens pruned on arrival, tokens leaving the buffer
  double evict_waves = 0;           // of an eviction launch
};

// Times of the two kernels in us, binary16 and float32: few_kernel's chain (per token
// that a wave selects, and per other token) and a round of 1024 waves; insert_kernel's
// and a round of 512 blocks, by what they do; the eviction in a launch of its own, and
// per 1024 waves of it.  Fitted to both kernels' times at 256 to 4096 units x 2 to 48
// tokens that fit the buffer, make others leave it, are pruned or both, from a page's
// start and within it: 1400 shapes in each type.
struct AppendCost {
  double few, few_selected, few_token, wave, wave_selected;
  double insert, block, tile, pruning, uneven, evicting, evicted;
  double launch, launch_evicted;
};
constexpr AppendCost kCostF16 = {7.9, 0.99, 0.67, 6.42, 0.22, 3.15, 2.24,
                                 4.13, 3.26, 0.66, 0.19, 0.19, 2.6, 0.68};
constexpr AppendCost kCostF32 = {8.2, 1.15, 0.27, 6.21, 0.37, 4.34, 2.35,
                                 4.12, 5.9, 2.17, 0.19, 0.39, 4.6, 1.02};

// Whether few_kernel takes the append and not insert_kernel as `pl` has it: the smaller
// of the times above.  No shape of the fit is slower by it than on the other kernel by
// more than 15 % (those between two numbers of rounds), nine in ten not at all.  Some
// (us, insert / few, units x tokens): binary16, fit, 1024 x 2 16 / 17, 2048 x 8 29 / 25,
// x 16 30 / 41, 4096 x 2 56 / 37; evicting 2048 x 2 32 / 23, x 8 35 / 32; pruned 512 x 2
// 13.6 / 16.7, 1152 x 16 29 / 38, 4096 x 2 85 / 37, x 20 118 / 107, x 24 115 / 121.
// float32: fit 4096 x 8 56 / 36, x 16 59 / 64; evicting 4096 x 8 83 / 57, x 16 111 /
// 129; pruned 4096 x 2 120 / 37, x 20 153 / 116, x 32 139 / 169.
static bool few_is_faster(const AppendWork& w, const AppendPlan& pl, bool f32, bool one_wave) {
  const AppendCost& c = f32 ? kCostF32 : kCostF16;
  const double launch =
      w.evict_waves > 0 ? c.launch + c.launch_evicted * w.evict_waves / 1024 : 0;
  const double selected = (w.pruned + (one_wave ? w.evicted : 0)) / w.waves;  // per wave
  const double others = w.tokens / w.waves - selected;
  const double few = c.few + c.few_selected * selected + c.few_token * (others > 0 ? others : 0) +
                     (c.wave + c.wave_selected * selected) * ceil(w.waves / 1024) +
                     (one_wave ? 0 : launch);
  const double a_block = c.block + (c.tile * w.tiles + c.pruning * w.pruning +
                                    c.uneven * w.uneven) / w.blocks +
                         (pl.fused && w.evicted > 0
                              ? c.evicting + c.evicted * w.evicted / w.blocks : 0);
  const double rounds = w.blocks / pl.wgs * ceil((double)pl.wgs / 512);
  const double insert = c.insert + a_block * (rounds + w.blocks / 512) / 2 +
                        (pl.fused ? 0 : launch);
  return 1.02 * few < insert;
}

// First position of a sequence's blocks: anywhere where no new token is pruned.
static int origin(const CompressLaunch& a, int b) {
  return a.tab.nnew[b] <= a.bb ? a.tab.len[b] : a.tab.len[b] & ~(kPage - 1);
}

// nblk: blocks of a unit of each sequence
static AppendWork append_work(const CompressLaunch& a, const int32_t* nblk) {
  AppendWork w;
  for (int b = 0; b < a.B; ++b) {
    const int len = a.tab.len[b], nnew = a.tab.nnew[b], org = origin(a, b);
    if (nnew == 0) continue;
    w.blocks += nblk[b];
    // blocks are multiples of 16 positions from org on
    w.tiles += (len + nnew - org + 15) / 16 - (len - org) / 16;
    w.tokens += nnew;
    w.waves += (nnew + kFewTokens - 1) / kFewTokens;
    const int evict = evict_end(len, nnew, a.bb) - evict_begin(len, a.bb);
    w.evicted += evict > 0 ? evict : 0;
    if (nnew <= a.bb) continue;
    const int end = len + nnew - a.bb;  // of the pruned positions
    w.pruned += nnew - a.bb;
    w.pruning += nblk[b];
    const int cut = (len % 8 != 0) + (end % 8 != 0);
    w.uneven += cut < nblk[b] ? cut : nblk[b];
  }
  w.evict_waves = (double)a.B * a.max_evict;
  double* all[] = {&w.blocks, &w.tiles, &w.pruning, &w.uneven, &w.tokens,
                   &w.waves, &w.pruned, &w.evicted, &w.evict_waves};
  for (double* v : all) *v *= 2 * a.Hkv;
  return w;
}

// The workgroups of pl, of nblk[b] blocks per unit, `blocks` per workgroup.
static void place_workgroups(const CompressLaunch& a, const int32_t* nblk, int blocks,
                             AppendPlan& pl) {
  int most = 0, least = INT_MAX;
  for (int b = 0; b < a.B; ++b) {
    most = nblk[b] > most ? nblk[b] : most;
    least = nblk[b] < least ? nblk[b] : least;
  }
  pl.groups = (most + blocks - 1) / blocks;
  pl.wgs = (int64_t)a.B * pl.groups * 2 * a.Hkv;
  pl.even = least == most && pl.groups <= 65535;
  if (pl.even) return;
  int order[SWAN_MAX_BATCH];
  for (int b = 0; b < a.B; ++b) {  // sorted in place, equal ones in their order
    int at = b;
    for (; at > 0 && nblk[order[at - 1]] < nblk[b]; --at) order[at] = order[at - 1];
    order[at] = b;
  }
  int64_t wgs = 0;
  for (int at = 0; at < a.B; ++at) {
    pl.table[at] = (uint32_t)wgs << 6 | (uint32_t)order[at];
    wgs += (int64_t)((nblk[order[at]] + blocks - 1) / blocks) * 2 * a.Hkv;
  }
  if (wgs <= UINT32_MAX >> 6) pl.wgs = wgs;
  else pl.even = true;  // (a grid that some workgroups leave at once)
}
static_assert(SWAN_MAX_BATCH <= 64, "the table's 6 bits, a ballot's lanes");

static AppendPlan plan_append(const CompressLaunch& a) {
  AppendPlan pl;
  pl.kernel = kAppendNone;
  const int units = a.B * a.Hkv * 2;
  bool fit = true;  // no new token is pruned
  int longest = 0, appending = 0;
  int64_t tokens = 0;  // of the appending sequences
  for (int b = 0; b < a.B; ++b) {
    fit = fit && a.tab.nnew[b] <= a.bb;
    longest = a.tab.nnew[b] > longest ? a.tab.nnew[b] : longest;
    tokens += a.tab.nnew[b];
    appending += a.tab.nnew[b] > 0;
  }
  if (longest == 0) return pl;
  // Positions per block: where no new token is pruned, so many that two
  // workgroups per compute unit share the tokens (8 sequences x 8 kv heads x 40
  // tokens: 12.4 us with blocks of 16, 16.2 with blocks of 64).
  int shift = 6;
  if (fit)
    while (shift > 4 && (int64_t)units * ((longest + (1 << (shift - 1)) - 1) >> (shift - 1)) <= 512)
      --shift;
  pl.bt = 1 << shift;
  int32_t nblk[SWAN_MAX_BATCH];  // blocks of a unit of each sequence
  int most = 0;
  int64_t total = 0;  // blocks of all
  for (int b = 0; b < a.B; ++b) {
    const int nnew = a.tab.nnew[b];
    nblk[b] = nnew ? (a.tab.len[b] + nnew - origin(a, b) + pl.bt - 1) >> shift : 0;
    most = nblk[b] > most ? nblk[b] : most;
    total += (int64_t)nblk[b] * 2 * a.Hkv;
  }
  // Blocks per workgroup: P's columns are loaded once for all of them (~2 us), so
  // many blocks go up to 8 to a workgroup, as long as the GPU keeps 4 rounds of
  // two workgroups per compute unit.  Where the units alone fill it, a few blocks
  // stay together, so that the eviction needs no launch of its own (on 1000 cached
  // tokens, us, eviction launch / this: 256 units x 100 tokens, buffer 64, 52 / 36,
  // float32 x 200 80 / 76, x 129, buffer 128, 69 / 72; 1024 units x 200, buffer 128,
  // 225 / 193; 128 units x 100, buffer 64, 31 / 36).
  int blocks = (int)(total / (256 * 2 * 4));
  blocks = blocks < 1 ? 1 : blocks > 8 ? 8 : blocks;
  if (a.max_evict > 0 && !fit && most <= 4 && units >= 256) blocks = most;
  pl.kernel = kAppendInsert;
  pl.blocks = blocks;
  place_workgroups(a, nblk, blocks, pl);
  pl.fused = fit || pl.groups == 1;
  // few_kernel: in the range of its fit, where both were measured (at 256 units it was
  // never the faster one), tokens on average
  if (appending * a.Hkv * 2 >= 512 && tokens <= (int64_t)48 * appending &&
      few_is_faster(append_work(a, nblk), pl, a.dtype == SWAN_F32, longest <= kFewTokens)) {
    pl.kernel = kAppendFew;
    pl.fused = longest <= kFewTokens;
    for (int b = 0; b < a.B; ++b) nblk[b] = (a.tab.nnew[b] + kFewTokens - 1) / kFewTokens;
    place_workgroups(a, nblk, 1, pl);
    return pl;
  }
  // Long appends of binary16 rows go to the prefill kernel: its rotation on int8 MFMA
  // has twice the rate of float64's, but a workgroup first makes P's digits and takes
  // 256 tokens at a time, and its grid has the longest sequence's workgroups for every
  // sequence.  Measured (one unit = a kv head's keys or values, us, insert / prefill),
  // all sequences with as many tokens: 16 units x 1024 19 / 29, 128 x 256 (512 blocks)
  // 31 / 29, 256 x 64 19 / 22, x 160 39 / 31, x 1024 207 / 115; 1024 x 96 87 / 77, x 128
  // 109 / 82, x 160 138 / 105, x 256 207 / 117; on 1000 cached tokens, 64 of them evicted,
  // 1024 x 96 114 / 117, x 128 139 / 126, x 160 167 / 133, 128 of them, x 128 138 / 152,
  // x 160 177 / 160.  Of different lengths (1024 units; one long sequence in so many):
  // 400 and 100 in 2 255 / 208; 256, 64 in 2 135 / 110, evicting 180 / 237; 700, 200 in 4
  // 303 / 213; 300, 20 in 8 68 / 164; 1000, 20 in 8 138 / 299; 1000, 100 in 4 276 / 326;
  // 2000, 100 in 8 295 / 370; 2000, 300 in 4 602 / 575; 4000, 100 in 8 479 / 441.  The
  // lengths are the sequences' own, not the rows' stride (64 tokens each in rows for 256:
  // 54 / 74).
  const double mean = (double)tokens / appending;
  const bool many = mean >= (longest >= kPrefillMinTokens ? kPrefillMinMeanLong : kPrefillMinMean);
  const bool alike = longest <= 2.25 * mean || mean >= kPrefillAnyMean;
  if (many && alike && total > kPrefillMinBlocks && a.dtype != SWAN_F32) {
    pl.kernel = kAppendPrefill;
    pl.fused = false;
  }
  return pl;
}

template <typename F>
static hipError_t launch_compress_t(const CompressLaunch& a) {
  const int units = a.B * a.Hkv * 2;
  if (a.n_new == 1) {  // a decode step: eviction and insertion in one launch
    const dim3 grid(units), block(256);
    switch (a.q ? a.Hq / a.Hkv : 0) {
      case 0:
        hipLaunchKernelGGL((step_kernel<F, 0>), grid, block, 0, a.stream, a);
        break;
      case 1:
        hipLaunchKernelGGL((step_kernel<F, 1>), grid, block, 0, a.stream, a);
        break;
      case 2:
        hipLaunchKernelGGL((step_kernel<F, 2>), grid, block, 0, a.stream, a);
        break;
      case 3:
        hipLaunchKernelGGL((step_kernel<F, 3>), grid, block, 0, a.stream, a);
        break;
      case 4:
        hipLaunchKernelGGL((step_kernel<F, 4>), grid, block, 0, a.stream, a);
        break;
      case 5:
        hipLaunchKernelGGL((step_kernel<F, 5>), grid, block, 0, a.stream, a);
        break;
      case 6:
        hipLaunchKernelGGL((step_kernel<F, 6>), grid, block, 0, a.stream, a);
        break;
      case 7:
        hipLaunchKernelGGL((step_kernel<F, 7>), grid, block, 0, a.stream, a);
        break;
      case 8:
        hipLaunchKernelGGL((step_kernel<F, 8>), grid, block, 0, a.stream, a);
        break;
      default:
        return hipErrorInvalidValue;  // the caller rotates more query heads per kv head itself
    }
    return hipGetLastError();
  }
  const AppendPlan pl = plan_append(a);
  if (pl.kernel == kAppendNone) return hipSuccess;
  if (a.max_evict > 0 && !pl.fused) {
    hipLaunchKernelGGL(evict_kernel<F>, dim3(units * a.max_evict), dim3(64), 0, a.stream, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (pl.kernel == kAppendPrefill) return launch_prefill(a);
  const bool evict = pl.fused && a.max_evict > 0;
  auto launch = [&](dim3 grid, const CompressLaunch& l) {
    if (pl.kernel == kAppendFew)
      hipLaunchKernelGGL(few_kernel<F>, grid, dim3(64), 0, a.stream, l, pl.even, evict);
    else
      hipLaunchKernelGGL(insert_kernel<F>, grid, dim3(64 * kInsWaves), 0, a.stream, l, pl.even,
                         pl.blocks, pl.bt, evict);
  };
  if (pl.even) {
    launch(dim3(units, pl.groups), a);
  } else {
    CompressLaunch l = a;
    memcpy(l.tab.nsplit, pl.table, sizeof(pl.table));
    launch(dim3((unsigned)pl.wgs), l);
  }
  return hipGetLastError();
}

hipError_t launch_compress(const CompressLaunch& a) {
  if (a.dtype == SWAN_F16) return launch_compress_t<_Float16>(a);
  if (a.dtype == SWAN_F16_E4M3) return launch_compress_t<E4M3V>(a);
  return launch_compress_t<float>(a);
}

}  // namespace swan

extern "C" int32_t swan_append_kernel(int32_t dtype, int32_t batch, int32_t n_kv_heads,
                                      int32_t buffer_tokens, const int32_t* seq_len_host,
                                      int32_t n_new, const int32_t* n_new_host) {
  if (!seq_len_host || batch < 1 || batch > SWAN_MAX_BATCH || n_new < 0) return -1;
  if (n_new == 1) return swan::kAppendStep;
  swan::CompressLaunch a = {};
  a.dtype = dtype;
  a.B = batch;
  a.Hkv = n_kv_heads;
  a.bb = buffer_tokens;
  a.n_new = n_new;
  for (int b = 0; b < batch; ++b) {
    a.tab.len[b] = seq_len_host[b];
    a.tab.nnew[b] = n_new_host ? n_new_host[b] : n_new;
    const int evict = swan::evict_end(a.tab.len[b], a.tab.nnew[b], a.bb) -
                      swan::evict_begin(a.tab.len[b], a.bb);
    a.max_evict = evict > a.max_evict ? evict : a.max_evict;
  }
  return swan::plan_append(a).kernel;
}
