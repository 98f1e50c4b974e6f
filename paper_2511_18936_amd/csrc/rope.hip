// Rotary position embedding (RoPE) of the Llama models the paper evaluates,
// for the query and key rows of a layer before the SWAN rotation: the paper
// rotates post-RoPE queries and keys, which is why P_QK cannot be folded into
// W_Q / W_K (Sec. 4.2).  Dims j and j + 64 of a row at position pos rotate by
// the angle pos * base^(-2j/128) ("rotate half" pairing), computed in float64
// and rounded once to the storage type, so the rows are what the cache's exact
// rotation then sees.
#include "swan_cache_ops.h"
#include "swan_device.h"

namespace swan {

template <typename T>
__device__ __forceinline__ T rounded(double y) {
  if constexpr (sizeof(T) == 2) return __builtin_bit_cast(T, f64_to_f16_bits_fast(y));
  else return (T)y;
}

// y: rounded results of a pair with a NaN
template <typename T>
__device__ __forceinline__ void one_nan_of(T& y) {
  if constexpr (sizeof(T) == 2) y = __builtin_bit_cast(T, one_nan(__builtin_bit_cast(uint16_t, y)));
}

// One wave per (sequence, position) and `heads` of its heads.  base^(-2j/128) is
// computed once per wave, the sine and cosine once per position, for all of its
// heads.  Two heads at a time, lane l of a half wave holds the pairs (2 l, 2 l + 64),
// (2 l + 1, 2 l + 65) of its head's row (4-byte accesses for binary16).
//
// What bounds it: memory.  32 heads x 1999 positions, binary16: 46 us with pow and
// sincos for every row, 14.8 us now; 16 x 32 heads x 8192: 2.45, 0.62 ms.
template <typename T>
__global__ __launch_bounds__(256) void rope_kernel(RopeLaunch a, int heads, int chunks) {
  constexpr int E = 2;
  const int lane = threadIdx.x & 63;
  const int l = lane & 31, first = lane >> 5;
  const int wpb = blockDim.x >> 6;
  const int64_t waves = (int64_t)gridDim.x * wpb;
  const int64_t items = (int64_t)a.B * a.n * chunks;
  double freq[E];
#pragma unroll
  for (int e = 0; e < E; ++e) freq[e] = pow(a.base, -(2.0 * (E * l + e)) / kD);
  for (int64_t w = (int64_t)blockIdx.x * wpb + (threadIdx.x >> 6); w < items; w += waves) {
    const int chunk = (int)(w % chunks);
    const int64_t at = w / chunks;
    const int b = (int)(at / a.n), i = (int)(at % a.n);
    const double pos = (double)a.pos0[b] + (double)i;
    double s[E], c[E];
#pragma unroll
    for (int e = 0; e < E; ++e) sincos(pos * freq[e], &s[e], &c[e]);
    const int h1 = min(a.H, (chunk + 1) * heads);
#pragma unroll 4
    for (int h = chunk * heads + first; h < h1; h += E) {
      const int64_t off = (((int64_t)b * a.H + h) * a.n + i) * kD + E * l;
      struct alignas(E * sizeof(T)) Vec {
        T v[E];
      };
      const Vec lo = *(const Vec*)((const T*)a.x + off);
      const Vec hi = *(const Vec*)((const T*)a.x + off + kD / 2);
      Vec p, q;
      bool nan = false;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const double x0 = (double)(float)lo.v[e], x1 = (double)(float)hi.v[e];
        p.v[e] = rounded<T>(x0 * c[e] - x1 * s[e]);
        q.v[e] = rounded<T>(x1 * c[e] + x0 * s[e]);
        nan |= __builtin_isunordered((float)lo.v[e], (float)hi.v[e]);
      }
      if (nan)
#pragma unroll
        for (int e = 0; e < E; ++e) {
          one_nan_of(p.v[e]);
          one_nan_of(q.v[e]);
        }
      *(Vec*)((T*)a.y + off) = p;
      *(Vec*)((T*)a.y + off + kD / 2) = q;
    }
  }
}

// Few rows: lane l holds the pair (l, l + 64) of one head after another, half the chain
// of a lane with two pairs.  Grid (positions, chunks of heads, sequences).
//
// What bounds it: latency, the float64 pow and sincos (~300 instructions) after the
// launch; so the first row is loaded before them and the grid numbers the items.  With
// 64-bit divisions for that and the loads after the chain, float32 rows took 3.3 us
// for 8 heads x 1 position and 5.9 for 32 x 100, now 2.7 and 4.3; 8 x 1999, binary16,
// 8.2 and 6.1 (13.4 with pow and sincos for every row).
template <typename T>
__global__ __launch_bounds__(64) void rope_few_kernel(RopeLaunch a, int heads) {
  const int l = threadIdx.x, i = blockIdx.x, b = blockIdx.z;
  const int h0 = blockIdx.y * heads, h1 = min(a.H, h0 + heads);
  int64_t off = (((int64_t)b * a.H + h0) * a.n + i) * kD + l;
  T lo = ((const T*)a.x)[off], hi = ((const T*)a.x)[off + kD / 2];
  double s, c;
  sincos(((double)a.pos0[b] + (double)i) * pow(a.base, -(2.0 * l) / kD), &s, &c);
#pragma unroll 1
  for (int h = h0; h < h1; ++h) {
    const int64_t next = off + (h + 1 < h1 ? (int64_t)a.n * kD : 0);
    const double x0 = (double)(float)lo, x1 = (double)(float)hi;
    if (h + 1 < h1) {
      lo = ((const T*)a.x)[next];
      hi = ((const T*)a.x)[next + kD / 2];
    }
    T p = rounded<T>(x0 * c - x1 * s), q = rounded<T>(x1 * c + x0 * s);
    if (x0 != x0 || x1 != x1) {
      one_nan_of(p);
      one_nan_of(q);
    }
    ((T*)a.y)[off] = p;
    ((T*)a.y)[off + kD / 2] = q;
    off = next;
  }
}

template <typename T>
static hipError_t launch_rope_t(const RopeLaunch& a) {
  // Up to 4096 waves (4 per SIMD), so that pow and sincos are shared by as many
  // rows as the GPU's size allows.  Few rows (a decode step, or a few thousand
  // positions of few heads): the shorter chain, one wave per workgroup; more
  // rows: two heads at a time, few positions splitting their heads.
  const int64_t rows = (int64_t)a.B * a.n;
  if (rows * a.H <= 4 * 4096) {
    const int heads = (int)((rows * a.H + 4095) / 4096);  // 1 to 4
    const int chunks = (a.H + heads - 1) / heads;
    hipLaunchKernelGGL(rope_few_kernel<T>, dim3(a.n, chunks, a.B), dim3(64), 0, a.stream, a,
                       heads);
    return hipGetLastError();
  }
  const int64_t most = (a.H + 1) / 2;
  int64_t split = 4096 / rows;
  split = split < 1 ? 1 : split > most ? most : split;
  const int heads = (int)(((a.H + split - 1) / split + 1) / 2 * 2);
  const int chunks = (a.H + heads - 1) / heads;
  const int64_t items = rows * chunks;
  const dim3 grid((unsigned)((items < 4096 ? items + 3 : 4096) / 4));
  hipLaunchKernelGGL(rope_kernel<T>, grid, dim3(256), 0, a.stream, a, heads, chunks);
  return hipGetLastError();
}

hipError_t launch_rope(const RopeLaunch& a) {
  return a.dtype == SWAN_F32 ? launch_rope_t<float>(a) : launch_rope_t<_Float16>(a);
}

}  // namespace swan
