// Offline calibration (Sec. 4.1.2): the projection P is the right singular
// matrix of the joint matrix S, i.e. the eigenvector matrix of S^T S.  One call
// solves a batch of problems side by side (a layer has two per kv head).
//
//   gram_kernel    G = S^T S in float64 (products of float32 are exact in
//                  float64) on float64 MFMA: the three 64 x 64 quadrants of the
//                  upper triangle, the rows in up to kGramChunks chunks, one
//                  workgroup per quadrant and chunk
//   reduce_kernel  the chunks' partial sums, in order
//   qr_kernel      G = Q R by Householder reflections, one workgroup per problem;
//                  left out (Q = I) where the diagonal of G is graded
//   similar_kernel A = R Q = Q^T G Q, and Q, row by row: one step of the QR
//                  iteration, which orders the diagonal and takes most of the
//                  off-diagonal mass (without it a spectrum like that of keys, each
//                  value 0.94 of the last, took 16 sweeps; with it 7)
//   jacobi_kernel  parallel cyclic Jacobi in float64, one workgroup per problem:
//                  round-robin pairing, 64 disjoint rotations per round, 127
//                  rounds per sweep, until the off-diagonal mass is negligible
//                  (and one sweep more where the diagonal is graded); the
//                  rotations (one float each) are recorded, not applied to the
//                  eigenvectors
//   vector_kernel  the recorded rotations applied to Q: every row of the
//                  eigenvector matrix on its own, one wave per row
//   finish_kernel  columns ordered by eigenvalue (descending, stable), signs
//                  canonicalised (largest-magnitude entry positive, lowest row
//                  on ties), sigma = sqrt(lambda), P written in float32
//
// The Jacobi rounds are a serial chain on one compute unit and set the time.
// With the players of the round-robin moving over the matrix, a round walked
// its rows and columns in LDS and the eigenvectors in the workspace and took
// 5-6 us; now the players stay at fixed positions and the matrix moves: pair i
// sits at positions 2 i and 2 i + 1, a round reads each 2 x 2 block of the
// upper triangle once, rotates it from both sides and writes its elements where
// the next round's positions put them, in a second buffer, all addresses fixed
// for the whole solve: 1.03 us.  One head's 4096 rows: 1.44 ms (7 sweeps; 2.26
// ms and 16 sweeps without the QR step; 2.18 ms where the diagonal is graded), from
// 11.8 ms; a layer of 8 kv heads (16 problems of 5 k and 17 k rows, side by side
// instead of one after another): 2.2 ms (2.70 ms without the QR step), from 190 ms.
#include <type_traits>

#include "swan_cache_ops.h"
#include "swan_device.h"

namespace swan {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kPairs = kD / 2;
constexpr int kRounds = kD - 1;
constexpr int kOffBlocks = kPairs * (kPairs - 1) / 2;  // 2 x 2 blocks above the diagonal ones
constexpr int kQuad = 64 * 64;                         // elements of a quadrant

// ---------------------------------------------------------------------------
// Gram matrix.  Grid (3 quadrants, chunks, problems); a wave takes 32 x 32 of
// its quadrant, 4 rows of S per step.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int64_t chunk_rows_of(int64_t n_rows) {  // a multiple of a step's 16
  const int64_t r = ((n_rows + kGramChunks - 1) / kGramChunks + 15) / 16 * 16;
  return r < 256 ? 256 : r;
}

__global__ __launch_bounds__(256) void gram_kernel(CalibLaunch a) {
  const int quad = blockIdx.x, chunk = blockIdx.y, prob = blockIdx.z;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m = lane & 15, k = lane >> 4;
  const int i0 = (quad == 2 ? 64 : 0) + 32 * (wave >> 1);
  const int j0 = (quad == 0 ? 0 : 64) + 32 * (wave & 1);
  const float* S = a.rows + a.row0[prob] * kD;
  const int64_t n = a.n_rows[prob], chunk_rows = chunk_rows_of(n);
  const int64_t r0 = chunk * chunk_rows;
  if (r0 >= n) return;
  const int64_t r1 = r0 + chunk_rows < n ? r0 + chunk_rows : n;
  f64x4 acc[2][2] = {};
  float next[4][4];  // [step][i0, i0 + 16, j0, j0 + 16], 16 rows ahead
  auto load = [&](int64_t r) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int64_t row = r + 4 * s + k;
      const float* p = S + row * kD + m;
      const bool in = row < r1;
      next[s][0] = in ? p[i0] : 0.f;
      next[s][1] = in ? p[i0 + 16] : 0.f;
      next[s][2] = in ? p[j0] : 0.f;
      next[s][3] = in ? p[j0 + 16] : 0.f;
    }
  };
  load(r0);
  for (int64_t r = r0; r < r1; r += 16) {
    float x[4][4];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i) x[s][i] = next[s][i];
    load(r + 16);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)x[s][i], (double)x[s][2 + j],
                                                           acc[i][j], 0, 0, 0);
  }
  // register v of lane l: row 4 v + l / 16, column l % 16 of the 16 x 16 tile
  double* out = a.part + ((int64_t)(prob * kGramChunks + chunk) * 3 + quad) * kQuad;
  const int li = 32 * (wave >> 1), lj = 32 * (wave & 1);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        out[(li + 16 * i + 4 * v + k) * 64 + lj + 16 * j + m] = acc[i][j][v];
}

// grid (kD * kD / 256, problems): one element of the full matrix per thread
__global__ __launch_bounds__(256) void reduce_kernel(CalibLaunch a) {
  const int e = blockIdx.x * 256 + threadIdx.x, prob = blockIdx.y;
  int i = e / kD, j = e % kD;
  if (i > j) {
    const int t = i;
    i = j;
    j = t;
  }
  const int quad = j < 64 ? 0 : i < 64 ? 1 : 2;
  const double* p = a.part + ((int64_t)prob * kGramChunks * 3 + quad) * kQuad + (i & 63) * 64 +
                    (j & 63);
  const int64_t n = a.n_rows[prob], chunk_rows = chunk_rows_of(n);
  const int chunks = (int)((n + chunk_rows - 1) / chunk_rows);
  double sum = 0.0;
#pragma unroll 8
  for (int c = 0; c < chunks; ++c) sum += p[(int64_t)c * 3 * kQuad];
  a.gram[(int64_t)prob * kD * kD + e] = sum;
}

// ---------------------------------------------------------------------------
// One QR step
// ---------------------------------------------------------------------------
constexpr int kQrGroups = 8;                   // threads per column
constexpr int kQrRows = kD / kQrGroups;        // rows a thread holds

// Householder vectors of a problem (row k: vector k, zero below index k), then
// their factors 2 / v^T v, in the partials' place until the Jacobi rotations come
__device__ __forceinline__ double* reflectors(const CalibLaunch& a, int prob) {
  return a.part + (int64_t)prob * kCalibPart;
}

// Where the columns of S differ in scale (outlier or nearly dead channels), Jacobi
// on G keeps the small eigenvalues and their vectors to nearly the accuracy of the
// small columns; a Householder step mixes the rows and leaves an error of 1e-15 of
// the LARGEST eigenvalue.  Such a G goes to Jacobi as it is.  The line: smallest
// diagonal element below 1/64 of the largest.  Largest error of a column of the
// basis without / with the QR step (2048 rows, 16 of 128 channels scaled, float64
// model against a long double solution): scale 0.1 (diagonal 9e-3) 7e-12 / 7e-12,
// 0.03 4e-12 / 1e-11, 1e-3 2e-12 / 4e-9, 1e-6 1e-12 / 1e-6, 1e-8 4e-12 / 7e-5; a
// rotated spectrum, ungraded (0.19), 2e-9 / 5e-10.  P is written in float32.
constexpr double kGraded = 1.0 / 64.0;

// Thread (j, g) holds rows 16 g .. of column j in registers; LDS carries the
// column to eliminate (zero above the diagonal), its dot products with every
// column (its own square norm among them, so that a step has two barriers) and
// row k.  What is left below the diagonal by a skipped step stays in the matrix:
// Q^T G is what is written, whatever its zeros.  2.7 us a step, the chain of its
// two reductions (3.4 us with the matrix in LDS): 0.35 ms a problem, which saves nine
// sweeps of 0.13 ms on a spectrum like that of keys (16 to 7) and one on values over
// output weights (11 to 10): alone those lose 0.2 ms by it, beside the keys' problems
// of a layer, whose step takes that time anyway, they gain the sweep.
__global__ __launch_bounds__(1024) void qr_kernel(CalibLaunch a) {
  __shared__ __attribute__((aligned(16))) double xcol[2][kD];
  __shared__ double part[kQrGroups][kD];
  __shared__ double krow[kD];
  __shared__ double red[4];
  const int tid = threadIdx.x, prob = blockIdx.x;
  const int j = tid & (kD - 1), g = tid >> 7;
  double* G = a.gram + (int64_t)prob * kD * kD;
  double* V = reflectors(a, prob);
  double m[kQrRows];
#pragma unroll
  for (int r = 0; r < kQrRows; ++r) m[r] = G[(kQrRows * g + r) * kD + j];
  // columns of less than 1e-30 of the largest diagonal element are left alone (what
  // remains of a matrix of low rank; their squares would underflow step by step)
  double dm = tid < kD ? G[tid * kD + tid] : 0.0, dn = dm;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    dm = fmax(dm, __shfl_xor(dm, o, 64));
    dn = fmin(dn, __shfl_xor(dn, o, 64));
  }
  if ((tid & 63) == 0 && tid < kD) {
    red[tid >> 6] = dm;
    red[2 + (tid >> 6)] = dn;
  }
  if (j == 0)
#pragma unroll
    for (int r = 0; r < kQrRows; ++r) xcol[0][kQrRows * g + r] = m[r];
  __syncthreads();
  dm = fmax(red[0], red[1]);
  const int graded = __builtin_amdgcn_readfirstlane(fmin(red[2], red[3]) < kGraded * dm ? 1 : 0);
  if (tid == 0) a.graded[prob] = graded;
  if (graded) return;
  const double tiny = 1e-60 * dm * dm;
  for (int k = 0; k < kD - 1; ++k) {
    const double* xc = xcol[k & 1];
    double dot = 0.0;
#pragma unroll
    for (int r = 0; r < kQrRows; r += 2) {
      const double2 v = *(const double2*)&xc[kQrRows * g + r];
      dot = fma(v.x, m[r], dot);
      dot = fma(v.y, m[r + 1], dot);
    }
    part[g][j] = dot;
    const int kr = k - kQrRows * g;  // row k in this thread's rows, if it has it
    if (kr >= 0 && kr < kQrRows) {   // uniform over the wave
      double mk = m[0];
#pragma unroll
      for (int r = 1; r < kQrRows; ++r) mk = kr == r ? m[r] : mk;
      krow[j] = mk;
    }
    __syncthreads();
    double sk = 0.0, sj = 0.0;
#pragma unroll
    for (int q = 0; q < kQrGroups; ++q) {
      sk += part[q][k];
      sj += part[q][j];
    }
    const double xk = xc[k];
    const bool on = sk > xk * xk && sk > tiny;  // something below the diagonal (uniform)
    // square root and reciprocal by two Newton steps on the hardware's estimates:
    // every wave computes them, in a sixth of the library's instructions
    double rs = __builtin_amdgcn_rsq(on ? sk : 1.0);
#pragma unroll
    for (int i = 0; i < 2; ++i) rs = rs * fma(-0.5 * sk * rs, rs, 1.5);
    const double norm = sk * rs;
    const double alpha = xk >= 0.0 ? -norm : norm;
    const double den = fma(fabs(xk), norm, sk);
    double beta = __builtin_amdgcn_rcp(on ? den : 1.0);
#pragma unroll
    for (int i = 0; i < 2; ++i) beta = beta * fma(-den, beta, 2.0);
    beta = on ? beta : 0.0;
    // v = x - alpha e_k; the columns before k are done
    const double w = j >= k && on ? beta * (sj - alpha * krow[j]) : 0.0;
#pragma unroll
    for (int r = 0; r < kQrRows; r += 2) {
      const double2 x = *(const double2*)&xc[kQrRows * g + r];
      m[r] = fma(-(kr == r ? xk - alpha : x.x), w, m[r]);
      m[r + 1] = fma(-(kr == r + 1 ? xk - alpha : x.y), w, m[r + 1]);
    }
    if (on && j == k)
#pragma unroll
      for (int r = 0; r < kQrRows; ++r) m[r] = kr > r ? m[r] : kr == r ? alpha : 0.0;
    if (j == k + 1)
#pragma unroll
      for (int r = 0; r < kQrRows; ++r)
        xcol[(k + 1) & 1][kQrRows * g + r] = kr + 1 <= r ? m[r] : 0.0;
    if (tid < kD) V[k * kD + tid] = tid == k ? xk - alpha : xc[tid];
    if (tid == 0) V[kD * kD + k] = beta;
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < kQrRows; ++r) G[(kQrRows * g + r) * kD + j] = m[r];
}

// the sum of v over the wave, in every lane
__device__ __forceinline__ double wave_sum_f64(double v) {
  auto step = [](double x, auto ctrl, auto rows) {
    const int64_t b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, decltype(ctrl)::value,
                                               decltype(rows)::value, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), decltype(ctrl)::value,
                                               decltype(rows)::value, 0xF, false);
    return x + __longlong_as_double(((int64_t)hi << 32) | (uint32_t)lo);
  };
  v = step(v, std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xF>{});
  v = step(v, std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xF>{});
  v = step(v, std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xF>{});
  v = step(v, std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xF>{});
  v = step(v, std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xA>{});
  v = step(v, std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xC>{});
  const int64_t b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, 63);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
  return __longlong_as_double(((int64_t)hi << 32) | (uint32_t)lo);
}

// Row r < kD: row r of Q^T G times Q, in place; row kD + r: row r of Q.  One wave
// per row, lane l holds columns 2 l and 2 l + 1; grid (2 kD / 4, problems).
// Graded: no steps, so G stays as it is and Q = I.
__global__ __launch_bounds__(256) void similar_kernel(CalibLaunch a) {
  const int lane = threadIdx.x & 63, prob = blockIdx.y;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int r = row & (kD - 1);
  double2* out = (double2*)((row < kD ? a.gram : a.vecs) + (int64_t)prob * kD * kD + r * kD);
  const double* V = reflectors(a, prob);
  const double2* v = (const double2*)V + lane;
  double2 x = make_double2(r == 2 * lane ? 1.0 : 0.0, r == 2 * lane + 1 ? 1.0 : 0.0);
  const int steps = a.graded[prob] ? 0 : kD - 1;
  if (row < kD) x = out[lane];
  constexpr int kAhead = 4;
  double2 next[kAhead];
#pragma unroll
  for (int i = 0; i < kAhead; ++i) next[i] = v[i * kPairs];
  for (int k0 = 0; k0 < steps; k0 += kAhead) {
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      const int k = k0 + i;
      if (k >= kD - 1) break;  // uniform
      const double2 h = next[i];
      if (k + kAhead < kD - 1) next[i] = v[(k + kAhead) * kPairs];
      const double w = V[kD * kD + k] * wave_sum_f64(fma(x.x, h.x, x.y * h.y));
      x.x = fma(-w, h.x, x.x);
      x.y = fma(-w, h.y, x.y);
    }
  }
  out[lane] = x;
}

// ---------------------------------------------------------------------------
// Jacobi
// ---------------------------------------------------------------------------
// Position 2 i is the upper player of pair i, 2 i + 1 the lower one.  After a
// round every player but position 0 moves on along the circle: the upper ones
// to the next pair, the last upper one down, the lower ones back, the first
// lower one up; after 127 rounds all are back.
__device__ __forceinline__ int next_pos(int p) {
  const int i = p >> 1;
  if (p & 1) return i == 0 ? 2 : p - 2;
  return i == 0 ? 0 : i == kPairs - 1 ? p + 1 : p + 2;
}

// One buffer of the matrix in LDS: the blocks (i, j), i < j, row-major, their
// first rows (two doubles each), then their second rows; then per pair the
// diagonal block's three elements.
constexpr int kOffRow = kOffBlocks * 16;           // bytes of one row plane
constexpr int kDiagA = 2 * kOffRow;                // (2 i, 2 i)
constexpr int kDiagB = kDiagA + kPairs * 8;        // (2 i, 2 i + 1)
constexpr int kDiagD = kDiagB + kPairs * 8;        // (2 i + 1, 2 i + 1)
constexpr int kMatBytes = kDiagD + kPairs * 8;
constexpr int kJacobiLds = 2 * kMatBytes + kPairs * 16 + 32 * 8 + 16;

__device__ __forceinline__ int block_index(int i, int j) {  // i < j
  return i * (kPairs - 1) - i * (i - 1) / 2 + (j - i - 1);
}

// byte offset in a buffer of the element at positions (r, c)
__device__ __forceinline__ int elem_off(int r, int c) {
  if ((r >> 1) > (c >> 1)) {
    const int t = r;
    r = c;
    c = t;
  }
  const int i = r >> 1, j = c >> 1;
  if (i == j) return ((r & 1) != (c & 1) ? kDiagB : (r & 1) ? kDiagD : kDiagA) + 8 * i;
  return (r & 1) * kOffRow + block_index(i, j) * 16 + (c & 1) * 8;
}

// cos and sin of the rotation with tangent t, to float64: 1 / sqrt(1 + t^2) by
// two Newton steps on the hardware's estimate
__device__ __forceinline__ void rotation(float t, double& c, double& s) {
  const double td = (double)t;
  const double u = fma(td, td, 1.0);
  double r = __builtin_amdgcn_rsq(u);
#pragma unroll
  for (int i = 0; i < 2; ++i) r = r * fma(-0.5 * u * r, r, 1.5);
  c = r;
  s = td * r;
}

// What bounds it: LDS and latency.  A round moves 2 x 64 KiB of blocks and 64
// KiB of rotations through LDS (~1.6 k cycles) behind one wave's chain for the
// rotations (~0.5 k cycles); the rounds depend on each other.
__global__ __launch_bounds__(1024) void jacobi_kernel(CalibLaunch a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  double2* cs = (double2*)(lds + 2 * kMatBytes);
  double* red = (double*)(lds + 2 * kMatBytes + kPairs * 16);  // [2][16]
  int* flag = (int*)(red + 32);
  const int tid = threadIdx.x, prob = blockIdx.x;
  const double* G = a.gram + (int64_t)prob * kD * kD;
  float* rec = (float*)(a.part + (int64_t)prob * kGramChunks * 3 * kQuad);  // partials are done
  // the matrix scaled by a power of two so that its largest diagonal element is
  // near 1: squares of its elements then neither overflow nor, where they
  // matter, underflow
  double dm = tid < kD ? G[tid * kD + tid] : 0.0;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) dm = fmax(dm, __shfl_xor(dm, o, 64));
  if ((tid & 63) == 0 && tid < kD) red[tid >> 6] = dm;
  __syncthreads();
  dm = fmax(red[0], red[1]);
  int ex = 0;
  if (dm > 0.0) (void)__builtin_frexp(dm, &ex);
  __syncthreads();
  for (int e = tid; e < kD * kD; e += 1024) {
    const int r = e / kD, c = e % kD;
    if (r <= c) *(double*)(lds + elem_off(r, c)) = __builtin_ldexp(G[e], -ex);
  }
  // this thread's blocks (i, j) and, for each, where its four elements go
  int bi[2] = {0, 0}, bj[2] = {0, 0}, to[2][4] = {};
  const bool have[2] = {true, tid + 1024 < kOffBlocks};
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    if (!have[u]) continue;
    const int n = tid + 1024 * u;
    int i = 0;
    while (block_index(i + 1, i + 2) <= n && i + 2 < kPairs) ++i;
    const int j = n - block_index(i, i + 1) + i + 1;
    bi[u] = i;
    bj[u] = j;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      to[u][q] = elem_off(next_pos(2 * i + (q >> 1)), next_pos(2 * j + (q & 1)));
  }
  int dto[3] = {0, 0, 0};  // pair tid's diagonal block
  if (tid < kPairs) {
    const int p = next_pos(2 * tid), q = next_pos(2 * tid + 1);
    dto[0] = elem_off(p, p);
    dto[1] = elem_off(p, q);
    dto[2] = elem_off(q, q);
  }
  __syncthreads();
  int cur = 0, sweep = 0, done = 0;
  // Graded: when the test passes, the elements among the small columns may still be
  // large against those columns' own diagonal, and rotations by float32 tangents
  // take up to a sweep more than exact ones to clear them: 16 of 128 channels of a
  // rotated spectrum at 1e-4, 4e-7 off without one more sweep, 8e-10 with it.
  int extra = a.graded[prob];
  for (; sweep < kJacobiMaxSweeps; ++sweep) {
    // convergence test: off-diagonal Frobenius mass against the diagonal's
    const char* A = lds + cur * kMatBytes;
    double off = 0.0, dia = 0.0;
    for (int n = tid; n < 4 * kOffBlocks; n += 1024) {
      const double v = ((const double*)A)[n];
      off = fma(2.0 * v, v, off);
    }
    if (tid < kPairs) {
      const double x = *(const double*)(A + kDiagA + 8 * tid);
      const double y = *(const double*)(A + kDiagB + 8 * tid);
      const double z = *(const double*)(A + kDiagD + 8 * tid);
      off = fma(2.0 * y, y, off);
      dia = fma(x, x, z * z);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      off += __shfl_xor(off, o, 64);
      dia += __shfl_xor(dia, o, 64);
    }
    if ((tid & 63) == 0) {
      red[tid >> 6] = off;
      red[16 + (tid >> 6)] = dia;
    }
    __syncthreads();
    if (tid == 0) {
      double o = 0.0, d = 0.0;
      for (int w = 0; w < 16; ++w) {
        o += red[w];
        d += red[16 + w];
      }
      *flag = (o <= 1e-30 * d) ? 1 : 0;
    }
    __syncthreads();
    done |= *flag;
    if (done && extra-- <= 0) break;
    for (int r = 0; r < kRounds; ++r) {
      const char* src = lds + cur * kMatBytes;
      char* dst = lds + (cur ^ 1) * kMatBytes;
      double2 x[2], y[2];  // the blocks' rows, read while wave 0 finds the rotations
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (have[u]) {
          x[u] = *(const double2*)(src + (tid + 1024 * u) * 16);
          y[u] = *(const double2*)(src + kOffRow + (tid + 1024 * u) * 16);
        }
      if (tid < kPairs) {
        const double p = *(const double*)(src + kDiagA + 8 * tid);
        const double q = *(const double*)(src + kDiagB + 8 * tid);
        const double d = *(const double*)(src + kDiagD + 8 * tid);
        // t = tan of the angle that zeroes q, to about float32: a rotation need
        // not be exact (what it leaves of q the next sweeps take), it must only
        // be the same rotation in the matrix and in the eigenvectors
        float t = 0.f;
        const double w4 = 4.0 * q * q;
        if (w4 > 1e-290 && w4 > 4e-36 * fabs(p * d)) {
          const double h = d - p;
          const double w = fma(h, h, w4);
          const double root = w * __builtin_amdgcn_rsq(w);
          t = (float)(2.0 * q * __builtin_amdgcn_rcp(fabs(h) + root));
          t = h < 0.0 ? -t : t;
        }
        double c, s;
        rotation(t, c, s);
        cs[tid] = make_double2(c, s);
        rec[((int64_t)sweep * kRounds + r) * kPairs + tid] = t;
        const double u0 = c * p - s * q, u1 = s * p + c * q;
        const double w0 = c * q - s * d, w1 = s * q + c * d;
        *(double*)(dst + dto[0]) = c * u0 - s * w0;
        *(double*)(dst + dto[1]) = c * u1 - s * w1;
        *(double*)(dst + dto[2]) = s * u1 + c * w1;
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (have[u]) {
          const double2 ri = cs[bi[u]], rj = cs[bj[u]];
          const double u0 = rj.x * x[u].x - rj.y * x[u].y, u1 = rj.y * x[u].x + rj.x * x[u].y;
          const double w0 = rj.x * y[u].x - rj.y * y[u].y, w1 = rj.y * y[u].x + rj.x * y[u].y;
          *(double*)(dst + to[u][0]) = ri.x * u0 - ri.y * w0;
          *(double*)(dst + to[u][1]) = ri.x * u1 - ri.y * w1;
          *(double*)(dst + to[u][2]) = ri.y * u0 + ri.x * w0;
          *(double*)(dst + to[u][3]) = ri.y * u1 + ri.x * w1;
        }
      __syncthreads();
      cur ^= 1;
    }
  }
  // whole sweeps: position p holds column p again
  double* lam = a.lam + (int64_t)prob * kD;
  if (tid < kPairs) {
    const char* A = lds + cur * kMatBytes;
    lam[2 * tid] = __builtin_ldexp(*(const double*)(A + kDiagA + 8 * tid), ex);
    lam[2 * tid + 1] = __builtin_ldexp(*(const double*)(A + kDiagD + 8 * tid), ex);
  }
  if (tid == 0) {
    a.status[2 * prob] = done;
    a.status[2 * prob + 1] = sweep;
  }
}

// lane l: v of lane l - 1 (lane 0: first) / of lane l + 1 (lane 63: last)
template <int CTRL>
__device__ __forceinline__ double wave_shift(double edge, double v) {
  const int64_t e = __double_as_longlong(edge), b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp((int)e, (int)b, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(e >> 32), (int)(b >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double(((int64_t)hi << 32) | (uint32_t)lo);
}

// Row r of the eigenvector matrix: row r of Q times the recorded rotations.  One wave per row, lane i holds positions 2 i and 2 i + 1; the
// players' move is a shift by one lane.  Grid (rows / 4, problems).  A chain of
// ~20 instructions per round, the rotations read 8 rounds ahead.
__global__ __launch_bounds__(256) void vector_kernel(CalibLaunch a) {
  const int lane = threadIdx.x & 63, prob = blockIdx.y;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int rounds = a.status[2 * prob + 1] * kRounds;
  const float* rec = (const float*)(a.part + (int64_t)prob * kGramChunks * 3 * kQuad) + lane;
  double2* out = (double2*)(a.vecs + (int64_t)prob * kD * kD + (int64_t)row * kD);
  const double2 q = out[lane];
  double x = q.x, y = q.y;
  constexpr int kAhead = 8;
  float next[kAhead];
#pragma unroll
  for (int i = 0; i < kAhead; ++i) next[i] = i < rounds ? rec[i * kPairs] : 0.f;
  for (int r0 = 0; r0 < rounds; r0 += kAhead) {
    float t[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      t[i] = next[i];
      const int n = r0 + kAhead + i;
      next[i] = n < rounds ? rec[(int64_t)n * kPairs] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      if (r0 + i >= rounds) break;  // uniform
      double c, s;
      rotation(t[i], c, s);
      const double xr = c * x - s * y, yr = s * x + c * y;
      x = wave_shift<0x138>(xr, lane == 0 ? yr : xr);  // from lane l - 1; pair 0's lower one up
      y = wave_shift<0x130>(xr, yr);                   // from lane l + 1; the last upper one down
    }
  }
  out[lane] = make_double2(x, y);
}

// grid (kD, problems): column j of the eigenvectors, thread r its row r
__global__ __launch_bounds__(kD) void finish_kernel(CalibLaunch a) {
  __shared__ double bv[2];
  __shared__ int br[2], cnt[2];
  const int j = blockIdx.x, prob = blockIdx.y, r = threadIdx.x;
  const double* lam = a.lam + (int64_t)prob * kD;
  const double v = a.vecs[(int64_t)prob * kD * kD + r * kD + j];
  const double lj = lam[j], lr = lam[r];
  const uint64_t ahead = __ballot(lr > lj || (lr == lj && r < j));
  // the largest magnitude, the lowest row on ties
  double best = fabs(v);
  int arg = r;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const double ob = __shfl_xor(best, o, 64);
    const int oa = __shfl_xor(arg, o, 64);
    const bool take = ob > best || (ob == best && oa < arg);
    best = take ? ob : best;
    arg = take ? oa : arg;
  }
  if ((r & 63) == 0) {
    bv[r >> 6] = best;
    br[r >> 6] = arg;
    cnt[r >> 6] = __popcll(ahead);
  }
  __syncthreads();
  const int rank = cnt[0] + cnt[1];
  const int top = bv[1] > bv[0] ? br[1] : br[0];
  const double vt = a.vecs[(int64_t)prob * kD * kD + top * kD + j];
  a.P_out[(int64_t)prob * kD * kD + r * kD + rank] = (float)(vt < 0.0 ? -v : v);
  if (r == 0 && a.sigma_out)
    a.sigma_out[(int64_t)prob * kD + rank] = (float)sqrt(lj > 0.0 ? lj : 0.0);
}

hipError_t launch_calibrate(const CalibLaunch& a) {
  hipError_t e;
  hipLaunchKernelGGL(gram_kernel, dim3(3, kGramChunks, a.count), dim3(256), 0, a.stream, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(reduce_kernel, dim3(kD * kD / 256, a.count), dim3(256), 0, a.stream, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(qr_kernel, dim3(a.count), dim3(1024), 0, a.stream, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(similar_kernel, dim3(2 * kD / 4, a.count), dim3(256), 0, a.stream, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  e = hipFuncSetAttribute((const void*)jacobi_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                          kJacobiLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(jacobi_kernel, dim3(a.count), dim3(1024), kJacobiLds, a.stream, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(vector_kernel, dim3(kD / 4, a.count), dim3(256), 0, a.stream, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(finish_kernel, dim3(kD, a.count), dim3(kD), 0, a.stream, a);
  return hipGetLastError();
}

}  // namespace swan
