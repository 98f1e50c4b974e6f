// Compress-append of many tokens at once (prefill), fp16 storage (sparse
// values fp16 or E4M3).
//
// Same result as token-by-token Algorithm 1 (and as insert_kernel): each new
// key/value x is rotated, x_hat = x . P, and the exact x_hat is rounded once to
// fp16; tokens that stay in the buffer go to their ring slot, the others are
// pruned to their top-k magnitudes (ties: lower index) and packed.
//
// The rotation runs on int8 MFMA (v_mfma_i32_16x16x64_i8) with exact integer
// arithmetic.  Each token row is a fixed-point integer X (30 bits below a
// power of two above the row's largest magnitude) and P a fixed-point integer
// Y (38 bits below a power of two above its largest entry), each split into
// balanced base-256 digits (4 for X, 5 for Y, every digit in [-128, 127]).
// The digit products are accumulated exactly in int32, one accumulator per
// digit weight; the 17 digit pairs whose weight is within 5 digits of the top
// give x_hat up to a bounded remainder: the 3 dropped pairs (below 2^-38 of
// the two powers of two's product), plus the truncation of tiny entries of x
// (counted per row) or of P (bounded per column).  Each
// element is rounded to fp16 in two ways that must agree: both ends of its
// error interval (widened by the float64 and float32 roundings) are rounded
// through float32; about 6 elements in 10^4 disagree and get an exact
// certification in float64 (no fp16 rounding boundary within the bound of the
// computed value), and the few that fail that are recomputed in float64 from
// x and P.  Either way the stored value is the exact x_hat rounded once to
// fp16.
//
// A workgroup of 8 waves serves one (sequence, kv head, role): it first writes
// P's digits, in the MFMA operand layout, to LDS (80 KiB), then each wave
// handles units of 32 positions (half a page), two waves per SIMD:
//   rotation   two 16-token tiles: x digits in registers (the MFMA's B
//              operand, the unit's rows loaded one unit ahead), P digits read
//              from LDS one step ahead (its A operand); 8 output tiles of 2 x
//              34 MFMAs, each followed by its conversion: a lane holds 4
//              consecutive output dims of one token, so the token's error
//              terms are lane constants and the 4 values go to its LDS row in
//              one 8-byte write
//   selection  two lanes per token, 64 dims each: a radix select on bit planes
//              of the magnitudes finds the kept dims (a 128-bit mask; ties at
//              the k-th largest to the lower dim), the counts of the two lanes
//              added by a lane swap
//   output     the kept values, then their dims, are packed into the token's
//              LDS row 8 dims at a time with table lookups and v_perm, read back
//              in page chunks and stored (512 B contiguous per half wave); a
//              dense row goes to the ring
// What bounds it: the VALU work around the MFMAs (about 3 k instructions per
// unit, 5 cycles each for one wave) and the MFMAs (544, 16 cycles each), which
// one wave cannot overlap; so two waves share a SIMD (256 registers each, which
// is why a wave takes 32 positions and not 64).  Measured at 8 sequences x 32
// heads x 16384 tokens, k in {32, 48, 64, 96}: 2.40 ms, from 3.28 ms with one
// wave of 64 positions per SIMD; without the selection and output 1.88 ms.
// (32x32x32 MFMA tiles: 2.59 ms, their conversion does not fit between the
// MFMAs of the next tile; the output as a walk over the set bits: 2.51 ms.)
#include <type_traits>

#include "swan_cache_ops.h"
#include "swan_device.h"

namespace swan {

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kRowHalves = 136;        // LDS row of one token's 128 fp16 values (+ pad)
constexpr int kUnit = 32;              // positions a wave handles at a time (half a page)
constexpr int kPrefillWaves = 8;       // waves per workgroup, sharing P's digits
constexpr int kXcds = 8;               // MI355X: 8 XCDs, each with its own L2
constexpr int kCus = 256;              // MI355X: compute units, one workgroup each (LDS)
constexpr int kStageBytes = kUnit * kRowHalves * 2;  // the rows of one wave
// digit arithmetic of the rotation
constexpr int kXDigits = 4;                    // x: balanced base-256 digits
constexpr int kPDigits = 5;                    // P: balanced base-256 digits
constexpr int kXFix = 8 * kXDigits - 2;        // |X| < 2^30
constexpr int kPFix = 8 * kPDigits - 2;        // |Y| < 2^38
constexpr int kTopLevel = 5;                   // digit pairs (s, t) with s + t <= 5 ...
constexpr int kLevels = kTopLevel + 1;         // ... accumulated per weight s + t
// The 3 dropped pairs, (2,4) and (3,3) of weight 2^8 and (3,4) of weight 1 in
// units of the lowest digit product: each sums 128 products of at most 2^14.
constexpr double kDroppedUnits = (2.0 * 256.0 + 1.0) * 128.0 * 16384.0;
// the conversion keeps the level sums down to 2^16 of the lowest level, rounded
// to nearest: at most half of that, in the same units
constexpr double kLevelRounding = 32768.0 * 65536.0;
constexpr int kBDigBytes = 8 * 2 * kPDigits * 1024;   // [out tile][k step][digit][lane][16 B]
// LDS: P's digits, the waves' rows, the compaction tables (packed_values),
// the P bound of each column and a few words of reduction
constexpr int kTabOff = kBDigBytes + kPrefillWaves * kStageBytes;
constexpr int kTabBytes = 256 * (16 + 16 + 8);
constexpr int kPrefillLds = kTabOff + kTabBytes + 128 * 4 + 64;
static_assert(kPrefillLds <= 160 * 1024, "one workgroup per CU");
constexpr uint16_t kUncertain = 0xFFFFu;       // a NaN pattern: never a rounded x_hat

// One step of a 16x16 bit-matrix transpose applied to both 16-bit halves of
// 16 words at once (row i of each matrix = half of w[i], column b = bit b):
// the k x k off-diagonal blocks of every 2k x 2k block trade places.
template <int K>
__device__ __forceinline__ void transpose_step(uint32_t* w, uint32_t mask) {
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    if (i & K) continue;
    const uint32_t t = ((w[i] >> K) ^ w[i + K]) & mask;
    w[i + K] ^= t;
    w[i] ^= t << K;
  }
}

// Bits 0-15 of a bit-plane word stand for a chunk's even dims, bits 16-31 for
// its odd ones; this puts them in dim order (bit i = dim 32 c + i).
__device__ __forceinline__ uint32_t spread16(uint32_t x) {
  x = (x | (x << 8)) & 0x00FF00FFu;
  x = (x | (x << 4)) & 0x0F0F0F0Fu;
  x = (x | (x << 2)) & 0x33333333u;
  return (x | (x << 1)) & 0x55555555u;
}
__device__ __forceinline__ uint32_t dim_order(uint32_t w) {
  return spread16(w & 0xFFFFu) | (spread16(w >> 16) << 1);
}

// lo: x of the same lane in the lower half of the wave, hi: in the upper half
struct HalfPair {
  uint32_t lo, hi;
};
__device__ __forceinline__ HalfPair half_pair(uint32_t x) {
  const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return {r[0], r[1]};
}

// The k dims kept of a token's 128 fp16 magnitudes, two lanes per token: v
// holds this lane's 64 (two per dword; lanes 0-31 dims 0-63, lanes 32-63 dims
// 64-127), kept gets the mask of those 64, in dim order.  The k largest, ties at the
// k-th largest to the lower dim.  Radix select on bit planes: the magnitudes
// of each 32-element chunk c are transposed so that pl[b][c] holds bit b of
// each element (bits 0-15: the chunk's even elements, 16-31: its odd ones);
// from the top bit down, the candidates still equal to the threshold prefix
// are split by the next bit, and those above it are collected.
__device__ __forceinline__ void kept_dims(const uint32_t* v, int k, int half, uint32_t* kept) {
  uint32_t pl[15][2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    uint32_t w[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i] = v[16 * c + i] & 0x7FFF7FFFu;
    transpose_step<8>(w, 0x00FF00FFu);
    transpose_step<4>(w, 0x0F0F0F0Fu);
    transpose_step<2>(w, 0x33333333u);
    transpose_step<1>(w, 0x55555555u);
#pragma unroll
    for (int b = 0; b < 15; ++b) pl[b][c] = w[b];  // plane 15 (the sign) is zero
  }
  uint32_t eq[2] = {~0u, ~0u}, gt[2] = {0u, 0u};
  int ngt = 0;
#pragma unroll
  for (int b = 14; b >= 0; --b) {
    const uint32_t hi0 = eq[0] & pl[b][0], hi1 = eq[1] & pl[b][1];
    const HalfPair n = half_pair((uint32_t)(__popc(hi0) + __popc(hi1)));
    const int above = ngt + (int)(n.lo + n.hi);
    const bool one = above >= k;  // the k-th largest has this bit set
    const uint32_t m = one ? ~0u : 0u;
    ngt = one ? ngt : above;
    gt[0] |= hi0 & ~m;
    gt[1] |= hi1 & ~m;
    eq[0] &= ~(pl[b][0] ^ m);
    eq[1] &= ~(pl[b][1] ^ m);
  }
  // eq: the elements equal to the k-th largest; k - ngt of them are kept,
  // lowest dims first
  eq[0] = dim_order(eq[0]);
  eq[1] = dim_order(eq[1]);
  const HalfPair neq = half_pair((uint32_t)(__popc(eq[0]) + __popc(eq[1])));
  const int need_all = k - ngt;
  if ((int)(neq.lo + neq.hi) > need_all) {  // ties: keep the lowest of them
    int need = half ? max(need_all - (int)neq.lo, 0) : min(need_all, (int)neq.lo);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      uint32_t keep = 0u, rest = eq[c];
      while (need > 0 && rest != 0u) {
        keep |= rest & (0u - rest);
        rest &= rest - 1u;
        --need;
      }
      eq[c] = keep;
    }
  }
  kept[0] = dim_order(gt[0]) | eq[0];
  kept[1] = dim_order(gt[1]) | eq[1];
}

// The lowest set dim of the 128-bit mask (lo: dims 0-63, hi: 64-127), cleared;
// branch-free.
__device__ __forceinline__ uint32_t pop_lowest(uint64_t& lo, uint64_t& hi) {
  const bool in_lo = lo != 0ull;
  const uint64_t m = in_lo ? lo : hi;
  const uint32_t d = (uint32_t)__builtin_ctzll(m) + (in_lo ? 0u : 64u);
  const uint64_t rest = m & (m - 1ull);
  lo = in_lo ? rest : lo;
  hi = in_lo ? hi : rest;
  return d;
}

// Packing a token's kept values.  A group of 8 dims has 256 possible masks;
// three tables in LDS hold for each mask m
//   sel_lo, sel_hi [m][4]  v_perm selectors: dword i of the group's kept values,
//                          packed to the front in ascending order, is
//                          perm(values 0-3, sel_lo[i]) | perm(values 4-7,
//                          sel_hi[i]) (selector 12 gives a zero byte)
//   pos [m][8]             the kept dims of the group in ascending order
// so that packing takes the same few instructions per group of 8 whatever k is
// (a walk over the set bits took 17 per kept entry).
__device__ __forceinline__ void fill_tables(char* tab, int tid) {
  if (tid >= 256) return;
  uint32_t lo[4], hi[4], ps[2] = {0u, 0u};
#pragma unroll
  for (int i = 0; i < 4; ++i) lo[i] = hi[i] = 0x0C0C0C0Cu;
  uint32_t n = 0u;  // kept so far
#pragma unroll
  for (uint32_t d = 0; d < 8; ++d) {
    const bool on = (tid >> d) & 1;
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
      // half n & 1 of dword n >> 1 takes the two bytes of value d
      const bool here = on && (n >> 1) == i;
      const uint32_t sh = 16u * (n & 1u);
      const uint32_t two = ((2u * (d & 3u)) | ((2u * (d & 3u) + 1u) << 8)) << sh;
      const uint32_t clear = ~(0xFFFFu << sh);
      if (d < 4) lo[i] = here ? (lo[i] & clear) | two : lo[i];
      else hi[i] = here ? (hi[i] & clear) | two : hi[i];
    }
    ps[0] |= on && n < 4u ? d << (8u * n) : 0u;
    ps[1] |= on && n >= 4u ? d << (8u * (n - 4u)) : 0u;
    n += on ? 1u : 0u;
  }
  ((u32x4*)tab)[tid] = u32x4{lo[0], lo[1], lo[2], lo[3]};
  ((u32x4*)(tab + 4096))[tid] = u32x4{hi[0], hi[1], hi[2], hi[3]};
  ((u32x2*)(tab + 8192))[tid] = u32x2{ps[0], ps[1]};
}

// v_perm_b32: byte i of the result is byte sel_i of the 8 bytes {hi : lo}
__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) {
  return __builtin_amdgcn_perm(hi, lo, sel);
}

// LDS accesses of one wave run in program order; the compiler keeps them so
// across this point
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Two lanes per token (half 0: dims 0-63, half 1: dims 64-127): its page slot.
// v: this lane's 64 values, kept: the mask of its kept dims.  The kept values
// of all 128 dims are packed into the token's LDS row `row` (which v was read
// from), 8 dims at a time in ascending order, each group's write covering the
// unused rest of the one before; half 0's groups all go before half 1's.  The
// padding's zeros are put in their place one by one.  Then the row is read
// back chunk by chunk and stored, each half every other chunk, and the same is
// done for the indices (the padding's are the lowest dims not kept).  Lanes with store == false (tokens that have
// no slot here) write nothing to the page.
template <typename F>
__device__ __forceinline__ void store_slot(char* row, const char* tab, const uint32_t* v,
                                           const uint32_t* kept, int k, int kp, char* page,
                                           int slot, int half, bool store) {
  constexpr int VB = Fmt<F>::kValBytes;
  constexpr bool kE4M3 = std::is_same<F, E4M3V>::value;
  const int C = kp / 8;
  const HalfPair n2 = half_pair((uint32_t)(__popc(kept[0]) + __popc(kept[1])));
  const uint32_t first = half ? n2.lo : 0u;  // this lane's first entry
  u32x2 pos[8];
  uint32_t at[8];  // first entry of each group
  {
    u32x4 packed[8];
    uint32_t n = first;
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      const uint32_t m = (kept[g >> 2] >> (8 * (g & 3))) & 0xFFu;
      const u32x4 lo = *(const u32x4*)(tab + 16 * m);
      const u32x4 hi = *(const u32x4*)(tab + 4096 + 16 * m);
      const u32x2 ps = *(const u32x2*)(tab + 8192 + 8 * m);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        packed[g][i] = perm(v[4 * g + 1], v[4 * g], lo[i]) | perm(v[4 * g + 3], v[4 * g + 2], hi[i]);
      pos[g] = u32x2{ps.x + 0x08080808u * (uint32_t)g, ps.y + 0x08080808u * (uint32_t)g};
      at[g] = n;
      n += (uint32_t)__popc(m);
    }
    wave_lds_fence();  // v has been read
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      if (half == hh) {
#pragma unroll
        for (int g = 0; g < 8; ++g) __builtin_memcpy(row + 2 * at[g], &packed[g], 16);
      }
      wave_lds_fence();
    }
  }
  if (k < kp) {  // uniform
    for (int e = k; e < kp; ++e) ((uint16_t*)row)[e] = 0;
    wave_lds_fence();
  }
  for (int c = half; c < C; c += 2) {
    const u32x4 val = *(const u32x4*)(row + 16 * c);
    if constexpr (kE4M3) {
      uint32_t w[2] = {0u, 0u};
#pragma unroll
      for (int q = 0; q < 8; ++q)
        w[q >> 2] |= f16_bits_to_e4m3((val[q >> 1] >> (16 * (q & 1))) & 0xFFFFu) << (8 * (q & 3));
      if (store) *(u32x2*)(page + c * 512 + slot * 8) = u32x2{w[0], w[1]};
    } else {
      if (store) *(u32x4*)(page + c * 1024 + slot * 16) = val;
    }
  }
  wave_lds_fence();
  const uint32_t base = half ? 0x40404040u : 0u;
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    if (half == hh) {
#pragma unroll
      for (int g = 0; g < 8; ++g) {
        const u32x2 p = {pos[g].x + base, pos[g].y + base};
        __builtin_memcpy(row + at[g], &p, 8);
      }
    }
    wave_lds_fence();
  }
  if (k < kp) {  // uniform
    const HalfPair k0 = half_pair(kept[0]), k1 = half_pair(kept[1]);
    uint64_t flo = ~(k0.lo | ((uint64_t)k1.lo << 32)), fhi = ~(k0.hi | ((uint64_t)k1.hi << 32));
    for (int e = k; e < kp; ++e) row[e] = (char)pop_lowest(flo, fhi);  // both halves: the same
    wave_lds_fence();
  }
  char* ipage = page + 64 * kp * VB;
  for (int c = half; c < C; c += 2) {
    const u32x2 idx = *(const u32x2*)(row + 8 * c);
    if (store) *(u32x2*)(ipage + c * 512 + slot * 8) = idx;
  }
}

// The balanced base-256 digits of four fixed-point values, as four int8 words
// (digit 0 = the top one).  yb = X + 0x808080: its low three bytes are the low
// digits plus 128, its top byte the top digit (two's complement).
__device__ __forceinline__ void digit_words(uint32_t a, uint32_t b, uint32_t c, uint32_t d,
                                            uint32_t* w) {
  const uint32_t ab_lo = perm(b, a, 0x05010400u), ab_hi = perm(b, a, 0x07030602u);
  const uint32_t cd_lo = perm(d, c, 0x05010400u), cd_hi = perm(d, c, 0x07030602u);
  w[3] = perm(cd_lo, ab_lo, 0x05040100u) ^ 0x80808080u;
  w[2] = perm(cd_lo, ab_lo, 0x07060302u) ^ 0x80808080u;
  w[1] = perm(cd_hi, ab_hi, 0x05040100u) ^ 0x80808080u;
  w[0] = perm(cd_hi, ab_hi, 0x07060302u);
}

// fixed-point value of one fp16 element: trunc(x * 2^shift) + 0x808080, scale =
// 2^shift (the fma is one instruction with the fp16 operand, and exact)
__device__ __forceinline__ uint32_t fixed_biased(_Float16 x, float scale) {
  return (uint32_t)(int32_t)fmaf((float)x, scale, 0.f) + 0x00808080u;
}

// The fp16 rounding of a value y known to within E: y's own rounding when no
// fp16 rounding boundary lies within E of it, else kUncertain.  Branch-free:
// y is rounded to float32 with round-to-odd (round to nearest, then back
// toward zero and the last bit set when that was inexact), which keeps the
// information that the hardware float32 -> fp16 rounding needs to round y
// itself correctly; the distance to the boundary is measured in float64.
__device__ __forceinline__ uint32_t certified_f16(double y, double E) {
  const float yn = (float)y;
  const double back = (double)yn;
  const bool inexact = back != y;
  const bool away = fabs(back) > fabs(y);
  float y32 = __uint_as_float((__float_as_uint(yn) - (inexact && away ? 1u : 0u)) |
                              (inexact ? 1u : 0u));
  asm("" : "+v"(y32));  // two hardware conversions, not one software f64 -> f16
  const uint32_t hb = (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)y32);
  const uint32_t ex = (hb >> 10) & 31u;
  const double hd = (double)f16_bits_to_f32(hb);
  const double dist = fabs(y - hd);  // exact
  // half the spacing of fp16 values at hb on y's side: below a power of two the
  // spacing halves.  (E < half / 2 keeps the other side's boundary out of reach
  // too.)
  const double half = ex ? __builtin_ldexp(1.0, (int)ex - 26) : 0x1p-25;
  const bool below_pow2 = (hb & 0x3FFu) == 0u && ex > 1u && fabs(y) < fabs(hd);
  const double side = below_pow2 ? 0.5 * half : half;
  const bool ok = (ex != 31u) & (dist + E + fabs(y) * 0x1p-50 < side) & (E < 0.25 * half);
  return ok ? hb : kUncertain;
}

__device__ __forceinline__ double wave_sum_f64(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

template <typename F>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void prefill_kernel(CompressLaunch a, int units_per_wave) {
  constexpr int VB = Fmt<F>::kValBytes;
  extern __shared__ __attribute__((aligned(16))) char lds_all[];
  char* bdig = lds_all;
  char* tab = lds_all + kTabOff;                   // store_slot's tables
  float* colDY = (float*)(tab + kTabBytes);        // [128]
  float* wgred = colDY + 128;                      // [8]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  char* lds = lds_all + kBDigBytes + wave * kStageBytes;  // this wave's rows
  uint16_t* rows = (uint16_t*)lds;                        // [32 tokens][kRowHalves]
  const int m16 = lane & 15, g4 = lane >> 4;              // rotation
  const int tok = lane & 31, half = lane >> 5;            // output: two lanes per token
  // grid: (b, h, role, group of units)
  // Workgroups go to the 8 XCDs round-robin by id, so XCD id % 8 gets the
  // (head, role) pairs u = xcd, xcd + 8, ...: its L2 then holds 1/8 of the P
  // matrices instead of all of them.  Where the pairs are no multiple of 8, all of
  // them alternate (with pairs padded to one, 2 kv heads used half of the XCDs: 256
  // units x 160 tokens 53 us, 31 now).
  const int pairs = 2 * a.Hkv, across = pairs % kXcds ? pairs : kXcds;
  const int first = blockIdx.x % across;
  int w = blockIdx.x / across;
  const int ngrp = a.prefill_groups;
  const int grp = w % ngrp;
  w /= ngrp;
  const int b = w % a.B;
  const int u = first + across * (w / a.B);  // (head, role) pair
  const int h = u >> 1;
  const int role = u & 1;
  const int len_old = a.tab.len[b];
  const int nnew = a.tab.nnew[b];
  if (nnew <= 0) return;
  const int len_new = len_old + nnew;
  const int unit0 = len_old / kUnit;
  const int unit1 = (len_new - 1) / kUnit;  // inclusive
  const int wbeg = unit0 + grp * kPrefillWaves * units_per_wave;  // the workgroup's units
  if (wbeg > unit1) return;  // uniform

  const _Float16* x = (const _Float16*)(role ? a.v_new : a.k_new) +
                      ((int64_t)b * a.Hkv + h) * a.n_new * kD;
  // NULL P_vo: values already in the rotated basis, stored as given
  const float* Prole = role ? a.P_vo : a.P_qk;
  const float* P = Prole ? Prole + (int64_t)h * kD * kD : nullptr;

  // a wave's units: wbeg + wave, + 8, ... (neighbouring waves read neighbouring rows)
  const int bend = min(wbeg + kPrefillWaves * units_per_wave, unit1 + 1);

  // The x rows of a unit's two 16-token tiles (lane (m16, g4): token 16 T +
  // m16, dims 64 ks + 16 g4 + j), zero past the workgroup's units and the new
  // tokens.  They are loaded one unit ahead of their use.
  auto load_x = [&](int unit_, u32x4 (&xv)[2][2][2]) {
#pragma unroll
    for (int T = 0; T < 2; ++T) {
      const int t = unit_ * kUnit + 16 * T + m16 - len_old;
      if (unit_ < bend && t >= 0 && t < nnew) {
        const u32x4* src = (const u32x4*)(x + (int64_t)t * kD + 16 * g4);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          xv[T][ks][0] = src[8 * ks];
          xv[T][ks][1] = src[8 * ks + 1];
        }
      } else {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) xv[T][ks][0] = xv[T][ks][1] = u32x4{0u, 0u, 0u, 0u};
      }
    }
  };
  u32x4 xnext[2][2][2];
  if (P) load_x(wbeg + wave, xnext);

  // ---- P's digits (once per workgroup) ----
  fill_tables(tab, tid);
  int G = 0;         // Y = trunc(P * 2^G), |Y| < 2^38
  float pmax = 0.f;  // largest |P|
  if (P) {
    // vector v = tid + 512 r: 16 entries P[k][col], k = 64 ks + 16 g + j, the 16
    // bytes of lane (col % 16) + 16 g of the A operand of output tile col / 16,
    // step ks; read once, for the largest entry and for the digits
    float pv[2][16];
    float pm = 0.f;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int v = tid + 512 * r;
      const int n = v & 15, g = (v >> 4) & 3, ks = (v >> 6) & 1, o = v >> 7;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        pv[r][j] = P[(64 * ks + 16 * g + j) * kD + 16 * o + n];
        pm = fmaxf(pm, fabsf(pv[r][j]));
      }
    }
    pm = wave_max(pm);
    if (lane == 0) wgred[wave] = pm;
    if (tid < kD) colDY[tid] = 0.f;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPrefillWaves; ++i) pmax = fmaxf(pmax, wgred[i]);
    int pe = 0;
    if (pmax > 0.f) (void)__builtin_frexpf(pmax, &pe);  // pmax < 2^pe
    G = kPFix - pe;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int v = tid + 512 * r;
      const int n = v & 15, g = (v >> 4) & 3, ks = (v >> 6) & 1, o = v >> 7;
      uint32_t dw[kPDigits][4];
      float dy = 0.f;
#pragma unroll
      for (int j4 = 0; j4 < 4; ++j4) {
        uint32_t lo[4];   // the four low digits plus 128 each, lowest first
        uint32_t top = 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          // Y = yh 2^16 + yl, truncated toward zero in two exact steps of float32
          // (P 2^(G-16) is below 2^22 and has 24 bits; so has its fraction)
          const float f = __builtin_ldexpf(pv[r][4 * j4 + i], G - 16);
          const float fh = truncf(f);
          const float fl = (f - fh) * 65536.f;
          const float fli = truncf(fl);
          dy = fmaxf(dy, fabsf(fl - fli));  // exact, in units of 2^-G
          const int64_t yb = (int64_t)(int)fh * 65536 + (int)fli + 0x80808080ll;
          lo[i] = (uint32_t)yb;
          top |= ((uint32_t)(yb >> 32) & 0xFFu) << (8 * i);  // |top| <= 64
        }
        dw[0][j4] = top;
        const uint32_t ab_lo = perm(lo[1], lo[0], 0x05010400u);
        const uint32_t ab_hi = perm(lo[1], lo[0], 0x07030602u);
        const uint32_t cd_lo = perm(lo[3], lo[2], 0x05010400u);
        const uint32_t cd_hi = perm(lo[3], lo[2], 0x07030602u);
        dw[4][j4] = perm(cd_lo, ab_lo, 0x05040100u) ^ 0x80808080u;
        dw[3][j4] = perm(cd_lo, ab_lo, 0x07060302u) ^ 0x80808080u;
        dw[2][j4] = perm(cd_hi, ab_hi, 0x05040100u) ^ 0x80808080u;
        dw[1][j4] = perm(cd_hi, ab_hi, 0x07060302u) ^ 0x80808080u;
      }
#pragma unroll
      for (int t = 0; t < kPDigits; ++t)
        *(u32x4*)(bdig + ((o * 2 + ks) * kPDigits + t) * 1024 + (n + 16 * g) * 16) =
            u32x4{dw[t][0], dw[t][1], dw[t][2], dw[t][3]};
      // in units of 1: below the float32 range the bound is its smallest normal
      float dyf = __builtin_ldexpf(dy, -G);
      if (dy > 0.f) dyf = fmaxf(dyf, 0x1p-126f);
      atomicMax((unsigned int*)&colDY[16 * o + n], __float_as_uint(dyf));
    }
  }
  __syncthreads();

  const int k = a.tab.kact[role][b];
  const int kp = kpad_of(k);
  const int64_t pbytes = page_bytes_of(VB, k);
  char* pages = (char*)(role ? a.v_pages : a.k_pages) + a.tab.page_off[role][b] +
                (int64_t)h * a.n_pages_cap * pbytes;
  uint16_t* ring = (uint16_t*)(role ? a.v_ring : a.k_ring) + ((int64_t)b * a.Hkv + h) * a.bb * kD;

  for (int unit = wbeg + wave; unit < bend; unit += kPrefillWaves) {
    const int pos0 = unit * kUnit;
    bool uncertain = false;  // some element of the unit needs the float64 path
    if (P) {
      // ---- x digits ----
      i32x4 X[2][2][kXDigits];  // [tile][k step][digit]
      float Eb[2];              // the token's bound without the P term
      float Ey[2];              // factor of the column's P truncation term
      int sx[2];                // x_hat = (level sums / 2^16) * 2^sx
#pragma unroll
      for (int T = 0; T < 2; ++T) {
        const u32x4 (&xv)[2][2] = xnext[T];
        // the row's largest magnitude (fp16 bits), the sum of its magnitudes
        // and the smallest |x| - 1 (as 16-bit integers, so that 0 wraps to
        // the largest), two elements per instruction
        u16x2 mx2 = {0, 0}, tm2 = {0xFFFF, 0xFFFF};
        float l1 = 0.f;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
          for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const uint32_t wa = xv[ks][c][q] & 0x7FFF7FFFu;
              const u16x2 a2 = __builtin_bit_cast(u16x2, wa);
              mx2 = __builtin_elementwise_max(mx2, a2);
              tm2 = __builtin_elementwise_min(tm2, a2 - (u16x2){1, 1});
              l1 = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, wa), (f16x2){1, 1}, l1, false);
            }
        uint32_t mx = max((uint32_t)mx2.x, (uint32_t)mx2.y);
        uint32_t tm = min((uint32_t)tm2.x, (uint32_t)tm2.y);
        mx = max(mx, (uint32_t)__shfl_xor((int)mx, 16));
        mx = max(mx, (uint32_t)__shfl_xor((int)mx, 32));
        tm = min(tm, (uint32_t)__shfl_xor((int)tm, 16));
        tm = min(tm, (uint32_t)__shfl_xor((int)tm, 32));
        l1 += __shfl_xor(l1, 16);
        l1 += __shfl_xor(l1, 32);
        // max|x| < 2^e
        const int e = mx == 0u ? 0
                      : (mx >> 10) ? (int)(mx >> 10) - 14
                                   : 8 - __builtin_clz(mx);  // (32 - clz) - 24
        const float scale = __builtin_ldexpf(1.f, kXFix - e);
        // |x| >= 2^(e - 20) is exact in 30 bits below 2^e; each smaller nonzero
        // element is truncated by less than 2^(e - 30): count them (rare: only
        // when the smallest nonzero |x| is below thr).  thr: the fp16 bits of
        // 2^(e - 20), or 0 below the fp16 range (none truncated)
        const int te = e - kXFix + 10;
        const uint32_t thr = te >= -14 ? (uint32_t)(te + 15) << 10
                             : te >= -24 ? 1u << (te + 24) : 0u;
        int ntr = 0;
        if (__ballot(thr != 0u && tm < thr - 1u) != 0ull) {
#pragma unroll
          for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const uint32_t wv = xv[ks][c][q];
                ntr += ((wv & 0x7FFFu) - 1u < thr - 1u) ? 1 : 0;  // 0 < |x| < 2^(e - 20)
                ntr += (((wv >> 16) & 0x7FFFu) - 1u < thr - 1u) ? 1 : 0;
              }
          ntr += __shfl_xor(ntr, 16);
          ntr += __shfl_xor(ntr, 32);
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          uint32_t dg[kXDigits][4];
#pragma unroll
          for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int q2 = 0; q2 < 2; ++q2) {
              // values 8 c + 4 q2 .. + 3
              const uint32_t w0 = xv[ks][c][2 * q2], w1 = xv[ks][c][2 * q2 + 1];
              const f16x2 v01 = __builtin_bit_cast(f16x2, w0);
              const f16x2 v23 = __builtin_bit_cast(f16x2, w1);
              uint32_t wd[kXDigits];
              digit_words(fixed_biased(v01.x, scale), fixed_biased(v01.y, scale),
                          fixed_biased(v23.x, scale), fixed_biased(v23.y, scale), wd);
#pragma unroll
              for (int s = 0; s < kXDigits; ++s) dg[s][2 * c + q2] = wd[s];
            }
#pragma unroll
          for (int s = 0; s < kXDigits; ++s)
            X[T][ks][s] = i32x4{(int)dg[s][0], (int)dg[s][1], (int)dg[s][2], (int)dg[s][3]};
        }
        // the token's scale and bounds: a lane's results are of the token of its
        // own row.  (float32, rounded up: the factors 1 + 2^-15 leave room for
        // that rounding, for the float32 additions of l1 (128 terms) and for the
        // rounding of the float32 fma that combines them per element.)  A row
        // of zeros gives exact zeros.
        sx[T] = 32 + e - kXFix - G;
        Eb[T] = mx == 0u ? 0.f
                         : (float)((kDroppedUnits + kLevelRounding) *
                                       __builtin_ldexp(1.0, e - kXFix - G) +
                                   (double)ntr * (double)pmax * __builtin_ldexp(1.0, e - kXFix)) *
                               (1.0f + 0x1p-15f);
        Ey[T] = l1 * (1.0f + 0x1p-14f);  // sum |x_i|
      }
      // ---- MFMAs of 16 output dims, then their certified fp16 values to the
      //      rows.  Step j = 2 o + ks: output tile o, k step ks; the P digits of
      //      a step are read from LDS into registers one step ahead. ----
      auto load_p = [&](int j, i32x4 (&A)[kPDigits]) {
#pragma unroll
        for (int t = 0; t < kPDigits; ++t)
          A[t] = *(const i32x4*)(bdig + (j * kPDigits + t) * 1024 + lane * 16);
      };
      i32x4 Aq[2][kPDigits];
      load_p(0, Aq[0]);
#pragma unroll 1
      for (int o = 0; o < 8; ++o) {
        i32x4 acc[2][kLevels];
#pragma unroll
        for (int T = 0; T < 2; ++T)
#pragma unroll
          for (int l = 0; l < kLevels; ++l) {
            const int z = l == kTopLevel ? 0x8000 : 0;  // the last level's sum is rounded
            acc[T][l] = i32x4{z, z, z, z};
          }
        const float4 dyc = *(const float4*)&colDY[16 * o + 4 * g4];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          const int jn = 2 * o + ks + 1;
          load_p(jn < 16 ? jn : 0, Aq[ks ^ 1]);
          // the 17 digit pairs (s of x, t of P), s + t <= 5
#pragma unroll
          for (int s = 0; s < kXDigits; ++s)
#pragma unroll
            for (int t = 0; t < kPDigits; ++t)
              if (s + t <= kTopLevel) {
#pragma unroll
                for (int T = 0; T < 2; ++T)
                  acc[T][s + t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
                      Aq[ks][t], X[T][ks][s], acc[T][s + t], 0, 0, 0);
              }
        }
        // Result layout: register v of lane l is output dim 16 o + 4 (l / 16) + v
        // of token l % 16.  With C_l the sum of level l, H = sum_l C_l 256^(5 -
        // l) = (t01 2^16 + t23) 2^16 + t45, t01 = C_0 256 + C_1 etc. exact in
        // int32: a top digit of x or P lies in [-64, 64], so over 128 products
        // |C_0| <= 2^19, |C_1| <= 2^21, |C_2| <= 2^22, |C_3| <= 3 * 2^21, |C_4|
        // <= 7 * 2^20, |C_5| <= 3 * 2^21.
        //
        // Fast check, in float32: H / 2^16 rounded to an integer hi 2^16 + lo
        // (the 0x8000 in C_5 and the arithmetic shift round to nearest: at most
        // kLevelRounding off, in E), as y: float(hi) is exact below 2^24 and
        // otherwise within 2^-24 of it, the fma adds 2^-24 |y|, lo is exact.  Both ends of
        // [y - E1, y + E1], E1 = E + 3.25 * 2^-24 |y|, are rounded to float32
        // (another 2^-24) and that to fp16.  The margin covers the three
        // roundings, so the two bracket every value within E of x_hat; rounding
        // is monotone, so when they agree that is the fp16 rounding of x_hat.
        // The elements whose ends disagree (about 6 in 10^4) get the exact
        // certification.
        const float dycv[4] = {dyc.x, dyc.y, dyc.z, dyc.w};
        uint32_t open[2][2];  // [T][v / 2]: nonzero halves where the ends disagree
#pragma unroll
        for (int T = 0; T < 2; ++T) {
          u32x2 four;
#pragma unroll
          for (int vp = 0; vp < 2; ++vp) {
            f32x2 lo2, hi2;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
              const int v = 2 * vp + i;
              const int t01 = acc[T][0][v] * 256 + acc[T][1][v];
              const int t23 = acc[T][2][v] * 256 + acc[T][3][v];
              const int t45 = acc[T][4][v] * 256 + acc[T][5][v];
              const int t = t23 + (t45 >> 16);
              const float y = __builtin_ldexpf(
                  fmaf((float)(t01 + (t >> 16)), 65536.f, (float)((uint32_t)t & 0xFFFFu)), sx[T]);
              const float E1 = fmaf(fabsf(y), 0x1.ap-23f, fmaf(dycv[v], Ey[T], Eb[T]));
              lo2[i] = y - E1;
              hi2[i] = y + E1;
            }
            const uint32_t lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo2, f16x2));
            const uint32_t hi = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi2, f16x2));
            four[vp] = lo;
            open[T][vp] = lo ^ hi;
          }
          __builtin_memcpy(
              __builtin_assume_aligned(&rows[(16 * T + m16) * kRowHalves + 16 * o + 4 * g4], 8),
              &four, 8);
        }
        if (__ballot((open[0][0] | open[0][1] | open[1][0] | open[1][1]) != 0u) != 0ull) {
          // the exact certification of every open element, in float64 (exact
          // below 2^53, else within 2^-53 |H|)
#pragma unroll
          for (int T = 0; T < 2; ++T)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              if ((open[T][v >> 1] & (v & 1 ? 0xFFFF0000u : 0xFFFFu)) == 0u) continue;
              const int t01 = acc[T][0][v] * 256 + acc[T][1][v];
              const int t23 = acc[T][2][v] * 256 + acc[T][3][v];
              const int t45 = acc[T][4][v] * 256 + (acc[T][5][v] - 0x8000);
              const double H = fma(fma((double)t01, 65536.0, (double)t23), 65536.0, (double)t45);
              const double y = __builtin_ldexp(H, sx[T] - 16);
              const uint32_t hb = certified_f16(y, (double)fmaf(dycv[v], Ey[T], Eb[T]));
              uncertain |= hb == kUncertain;
              rows[(16 * T + m16) * kRowHalves + 16 * o + 4 * g4 + v] = (uint16_t)hb;
            }
        }
      }
    } else {
      // values given in the rotated basis: the rows are the input
      const int t = pos0 + tok - len_old;
      u32x4* dst = (u32x4*)(rows + tok * kRowHalves + 64 * half);
      if (t >= 0 && t < nnew) {
        const u32x4* src = (const u32x4*)(x + (int64_t)t * kD + 64 * half);
#pragma unroll
        for (int c = 0; c < 8; ++c) dst[c] = src[c];
      }
    }
    wave_lds_fence();
    if (__ballot(uncertain) != 0) {
      // The rare uncertain elements: x_hat in float64 over the input row and P,
      // rounded once.  The wave takes them one at a time, each lane summing the
      // products of two input dims.
      const int t = pos0 + tok - len_old;
      uint16_t* myrow = rows + tok * kRowHalves + 64 * half;
      uint32_t um[2] = {0u, 0u};  // this lane's uncertain dims (64 half + ...)
      if (t >= 0 && t < nnew)
        for (int j = 0; j < 64; ++j)
          if (myrow[j] == kUncertain) um[j >> 5] |= 1u << (j & 31);
      for (uint64_t act = __ballot((um[0] | um[1]) != 0u); act != 0u;
           act = __ballot((um[0] | um[1]) != 0u)) {
        const int L = __builtin_ctzll(act);
        const int jl = um[0] ? __builtin_ctz(um[0]) : um[1] ? 32 + __builtin_ctz(um[1]) : 0;
        const int j = __shfl(jl + 64 * half, L);
        const int tl = __shfl(t, L);
        const uint32_t xw = *(const uint32_t*)(x + (int64_t)tl * kD + 2 * lane);
        double part = (double)f16_bits_to_f32(xw & 0xFFFFu) * (double)P[(2 * lane) * kD + j];
        part = fma((double)f16_bits_to_f32(xw >> 16), (double)P[(2 * lane + 1) * kD + j], part);
        part = wave_sum_f64(part);
        if (lane == L) {
          myrow[jl] = f64_to_f16_bits(part);
          um[jl >> 5] &= ~(1u << (jl & 31));
        }
      }
      wave_lds_fence();
    }

    // the next unit's rows (here the registers of the rotation are free)
    if (P) load_x(unit + kPrefillWaves, xnext);

    // ---- two lanes per token ----
    const int pos = pos0 + tok;
    const int t = pos - len_old;
    const bool mine = t >= 0 && t < nnew;
    const bool dense = pos >= len_new - a.bb;
    const uint16_t* row = rows + tok * kRowHalves;
    if (mine && dense) {  // stays in the buffer: ring slot pos % b
      u32x4* dst = (u32x4*)(ring + (int64_t)(pos % a.bb) * kD + 64 * half);
#pragma unroll
      for (int c = 0; c < 8; ++c) dst[c] = ((const u32x4*)(row + 64 * half))[c];
    }
    if (__ballot(mine && !dense) != 0ull) {
      uint32_t v[32];
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const u32x4 c4 = ((const u32x4*)(row + 64 * half))[c];
        v[4 * c] = c4.x;
        v[4 * c + 1] = c4.y;
        v[4 * c + 2] = c4.z;
        v[4 * c + 3] = c4.w;
      }
      uint32_t kept[2];
      kept_dims(v, k, half, kept);
      store_slot<F>((char*)rows + tok * kRowHalves * 2, tab, v, kept, k, kp,
                    pages + (int64_t)(pos0 / kPage) * pbytes, (pos0 & (kPage - 1)) + tok, half,
                    mine && !dense);
    }
    wave_lds_fence();  // the rows are rewritten by the next unit
  }
}

// Units of 32 positions per wave: a workgroup's set-up (P's digits, ~4 us) is
// paid once for all of its waves' units, so long prompts take 16; but the GPU
// runs one workgroup per compute unit, so a batch that would leave it in fewer
// than 4 rounds of workgroups takes fewer units each, down to one: 1009 tokens on
// 8 kv heads took 30 us here (201 us with 8 blocks of 64 per wave; the insert
// kernel, which such a prompt goes to, takes 18 us).
static int units_per_wave(int64_t total_units) {
  int64_t n = total_units / ((int64_t)kCus * kPrefillWaves * 4);
  return n < 1 ? 1 : n > 16 ? 16 : (int)n;
}

template <typename F>
static hipError_t launch_prefill_f(const CompressLaunch& a, dim3 grid, int upw) {
  const hipError_t e = hipFuncSetAttribute((const void*)prefill_kernel<F>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kPrefillLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(prefill_kernel<F>, grid, dim3(64 * kPrefillWaves), kPrefillLds, a.stream, a,
                     upw);
  return hipGetLastError();
}

hipError_t launch_prefill(const CompressLaunch& in) {
  CompressLaunch a = in;
  int64_t total = 0;  // units of all sequences, heads and roles
  int most = 0;       // of one sequence's head and role
  for (int b = 0; b < a.B; ++b) {
    if (a.tab.nnew[b] <= 0) continue;
    const int n = (a.tab.len[b] + a.tab.nnew[b] - 1) / kUnit - a.tab.len[b] / kUnit + 1;
    total += (int64_t)n * 2 * a.Hkv;
    most = n > most ? n : most;
  }
  if (most == 0) return hipSuccess;
  const int upw = units_per_wave(total);
  a.prefill_groups = (most + kPrefillWaves * upw - 1) / (kPrefillWaves * upw);
  const dim3 grid((int64_t)2 * a.Hkv * a.B * a.prefill_groups);
  if (a.dtype == SWAN_F16_E4M3) return launch_prefill_f<E4M3V>(a, grid, upw);
  return launch_prefill_f<_Float16>(a, grid, upw);
}

}  // namespace swan
