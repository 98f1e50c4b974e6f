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
void insert_kernel(CompressLaunch a, int groups, int blocks, int bt, bool evict) {
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
  // Group-major: workgroups go to the 8 XCDs round-robin, so with a unit's groups side
  // by side and an even number of them, its short last group always fell to the same
  // XCDs (4096 units x 512 tokens, float32, 8 blocks and 1: 3.19 ms, 1.75 now).
  const int units = 2 * a.B * a.Hkv, grp = blockIdx.x / units;
  int w = blockIdx.x % units;
  const int role = w & 1;
  w >>= 1;
  const int h = w % a.Hkv;
  const int b = w / a.Hkv;
  const int nnew = a.tab.nnew[b];
  if (nnew == 0) return;  // uniform
  const int len_old = a.tab.len[b], len_new = len_old + nnew;
  // no new token is pruned when all fit the buffer: blocks then begin anywhere
  const bool fits = nnew <= a.bb;
  const int org = fits ? len_old : len_old & ~(kPage - 1);
  const int nblk = (len_new - org + bt - 1) / bt;
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
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        Bits y;
        if constexpr (sizeof(Bits) == 2) y = f64_to_f16_bits_fast(acc[v]);
        else y = St::from_f64(acc[v]);
        rows[(16 * T + 4 * v + g) * RS + 16 * wave + m] = y;
      }
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
__global__ __launch_bounds__(64) void few_kernel(CompressLaunch a, int groups, bool evict) {
  using T = typename Fmt<F>::Elem;
  using St = Store<T>;
  __shared__ __attribute__((aligned(16))) double xs[kD][kFewTokens];
  const int lane = threadIdx.x;
  const int units = 2 * a.B * a.Hkv, grp = blockIdx.x / units;  // as in insert_kernel
  int w = blockIdx.x % units;
  const int role = w & 1;
  w >>= 1;
  const int h = w % a.Hkv;
  const int b = w / a.Hkv;
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
  int groups;      // workgroups per (sequence, kv head, role) of insert or few_kernel
  bool fused;      // that kernel evicts; else an eviction launch goes first
};

// Blocks of an append of at most n tokens per unit from which few_kernel is faster than
// insert_kernel; fit: no new token is pruned, evict: some leave the buffer.  Measured
// (us, insert / few, units x tokens): binary16, fit, 1024 x 2 15.4 / 16.4, 1536 x 2
// 21.7 / 19.8, 1536 x 8 22.3 / 23.9, 2048 x 8 28.8 / 25.8, 4096 x 2 54 / 36; evicting
// 2048 x 2 32 / 23, x 8 36 / 33; pruned on arrival 512 x 2 13.5 / 16.8, 1024 x 2 24 /
// 18, x 8 22.7 / 25.4, 2048 x 8 42 / 32, x 16 59 / 50.  float32: fit 768 x 2 13.5 / 15.0,
// 1024 x 2 16.5 / 15.5, x 8 16.8 / 16.6; evicting 1024 x 4 20.6 / 22.7, 1536 x 4 29 / 28.5,
// 2048 x 8 45 / 39; pruned 512 x 2 18.5 / 17.2, 1024 x 8 30 / 27, 2048 x 2 63 / 24.
static int few_from(bool f32, bool fit, bool evict, int n) {
  if (fit) return !f32 ? 1000 + 100 * n : evict ? 600 + 130 * n : 1000;
  if (n <= kFewTokens) return f32 ? 300 + 60 * n : 500 + 100 * n;
  return f32 ? (evict ? 1200 : 700) : (evict ? 1500 : 1000);  // the eviction in a launch
}

static AppendPlan plan_append(const CompressLaunch& a) {
  AppendPlan pl = {kAppendNone, kPage, 1, 0, false};
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
  // Positions per block: where no new token is pruned, so many that two
  // workgroups per compute unit share the tokens (8 sequences x 8 kv heads x 40
  // tokens: 12.4 us with blocks of 16, 16.2 with blocks of 64).
  if (fit)
    while (pl.bt > 16 && (int64_t)units * ((longest + pl.bt / 2 - 1) / (pl.bt / 2)) <= 512)
      pl.bt /= 2;
  int most = 0;       // blocks of one unit
  int64_t total = 0;  // blocks of all
  int64_t waves = 0;  // few_kernel's for all
  for (int b = 0; b < a.B; ++b) {
    const int org = a.tab.nnew[b] <= a.bb ? a.tab.len[b] : a.tab.len[b] & ~(kPage - 1);
    const int n = a.tab.nnew[b] ? (a.tab.len[b] + a.tab.nnew[b] - org + pl.bt - 1) / pl.bt : 0;
    most = n > most ? n : most;
    total += (int64_t)n * 2 * a.Hkv;
    waves += (int64_t)((a.tab.nnew[b] + kFewTokens - 1) / kFewTokens) * 2 * a.Hkv;
  }
  if (most == 0) return pl;
  // Few tokens of many units.  A wave of few_kernel takes under half the time of a
  // block of 64 that is pruned, more than half of a short one that fits the buffer
  // (4096 units x 16 tokens, two waves each: pruned 112 us on insert_kernel, 85 on
  // few_kernel, x 24, three waves, 114 / 117; dense, 16: 55 / 70).
  if (waves <= (fit ? 1 : 2) * total &&
      total >= few_from(a.dtype == SWAN_F32, fit, a.max_evict > 0, longest)) {
    pl.kernel = kAppendFew;
    pl.groups = (longest + kFewTokens - 1) / kFewTokens;
    pl.fused = pl.groups == 1;
    return pl;
  }
  // Long appends of binary16 rows go to the prefill kernel: its rotation on int8
  // MFMA has twice the rate of float64's, but a workgroup first makes P's digits
  // and takes 256 tokens at a time.  Measured (one unit = a kv head's keys or
  // values, us, insert / prefill), all sequences with as many tokens: 16 units x
  // 1024 tokens 19 / 32, 128 x 256 (512 blocks) 29 / 28, 256 x 64 14 / 20, x 160
  // 46 / 28, x 1024 195 / 115, 1024 x 64 43 / 62, x 160 133 / 91, x 256 195 / 108;
  // on 1000 cached tokens, 64 of them evicted, 1024 x 96 110 / 117, x 128 131 / 125,
  // x 160 158 / 125.  Of different lengths (1024 units): 200 and 40 tokens in turn
  // 180 / 100; 300 for one sequence in 8, else 20: 79 / 166; 1000 for one in 8, else
  // 20: 471 / 306.  The lengths are the sequences' own, not the rows' stride (64
  // tokens each in rows for 256: 54 / 74).
  const bool many = longest >= kPrefillMinTokens || tokens >= (int64_t)kPrefillMinMean * appending;
  const bool prefill = many && total > kPrefillMinBlocks && a.dtype != SWAN_F32;
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
  pl.kernel = prefill ? kAppendPrefill : kAppendInsert;
  pl.blocks = blocks;
  pl.groups = (most + blocks - 1) / blocks;
  pl.fused = !prefill && (fit || pl.groups == 1);
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
  if (pl.kernel == kAppendFew) {
    hipLaunchKernelGGL(few_kernel<F>, dim3((int64_t)units * pl.groups), dim3(64), 0, a.stream, a,
                       pl.groups, pl.fused && a.max_evict > 0);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(insert_kernel<F>, dim3((int64_t)units * pl.groups), dim3(64 * kInsWaves), 0,
                     a.stream, a, pl.groups, pl.blocks, pl.bt, pl.fused && a.max_evict > 0);
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
