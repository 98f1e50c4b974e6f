// Launchers of what runs beside the decode attention: append and prefill, change of k,
// RoPE, calibration.  A header of their own, so that the record of the attention's
// memory traffic, kept per state of its sources, outlives a change of these.
#pragma once

#include "swan_device.h"
#include "swan_internal.h"

namespace swan {

// f64_to_f16_bits_fast keeps a NaN's bits; f64_to_f16_bits has one NaN (and its sign).
// Of the former's result, so that a token's bytes do not depend on the kernel that
// stores it.  (Called where a NaN was seen: for every value it took RoPE 5 to 12 % more.)
__device__ __forceinline__ uint16_t one_nan(uint16_t h) {
  return (h & 0x7FFFu) > 0x7C00u ? (uint16_t)((h & 0x8000u) | 0x7E00u) : h;
}

struct CompressLaunch {
  const void* k_new;
  const void* v_new;
  const float* P_qk;
  const float* P_vo;
  void* k_pages;
  void* v_pages;
  void* k_ring;
  void* v_ring;
  int B, Hkv, bb, n_pages_cap, n_new;  // n_new: token stride of k_new / v_new
  int max_evict;  // largest per-sequence eviction count
  int prefill_groups;  // set by launch_prefill: workgroups per (sequence, head, role)
  int dtype;
  SeqTab tab;     // len = tokens cached before the call
  hipStream_t stream;
  // decode steps (n_new == 1) only: q != nullptr makes the key waves also
  // write q_hat = q . P_qk * qmult for the Hq / Hkv (at most kStepQG) query
  // heads of their kv head, q [B][Hq][128] storage type, qhat [B][Hq][128]
  const void* q = nullptr;
  float* qhat = nullptr;
  int Hq = 0;
  float qmult = 0.f;
};
constexpr int kStepQG = 8;
hipError_t launch_compress(const CompressLaunch& a);
// prefill path (fp16, many tokens): int8 MFMA rotation, two lanes per token's top-k
constexpr int kPrefillMinMean = 160;      // tokens per sequence that appends, on average,
constexpr int kPrefillMinMeanLong = 128;  // ... with one of
constexpr int kPrefillMinTokens = 256;
constexpr int kPrefillAnyMean = 512;      // ... from which lengths may differ as they like
constexpr int kPrefillMinBlocks = 512;  // of 64 positions, over all sequences, heads and roles
hipError_t launch_prefill(const CompressLaunch& a);
// what an append runs
enum AppendKernel { kAppendNone, kAppendStep, kAppendInsert, kAppendPrefill, kAppendFew };

// run-time change of k: one launch per role, over the role's page arrays
// (change_k.hip)
struct ChangeKLaunch {
  const char* src;  // the role's pages in the source cache
  char* dst;        // the role's pages in the destination cache
  int B, Hkv, bb, npc_src, npc_dst, max_pages, dtype;
  int32_t len[SWAN_MAX_BATCH];      // tokens cached
  int32_t k_src[SWAN_MAX_BATCH];    // the role's k in the source layout
  int32_t k_dst[SWAN_MAX_BATCH];    // the role's k in the destination layout
  int64_t off_src[SWAN_MAX_BATCH];  // byte offset of the sequence's first source page
  int64_t off_dst[SWAN_MAX_BATCH];  // byte offset of the sequence's first destination page
  int nsel;                         // set by launch_change_k: the sequences of one launch
  int32_t sel[SWAN_MAX_BATCH];
  hipStream_t stream;
};
hipError_t launch_change_k(const ChangeKLaunch& a);

// RoPE of query / key rows before the rotation (rope.hip)
struct RopeLaunch {
  const void* x;
  void* y;
  int B, H, n, dtype;
  int32_t pos0[SWAN_MAX_BATCH];  // position of each sequence's first row
  double base;
  hipStream_t stream;
};
hipError_t launch_rope(const RopeLaunch& a);

constexpr int kMaxCalib = 64;  // problems per launch
struct CalibLaunch {
  const float* rows;           // the problems' rows, 128 floats each
  int64_t row0[kMaxCalib];     // first row of each problem
  int64_t n_rows[kMaxCalib];
  int count;                   // problems solved side by side
  float* P_out;       // [count][128][128]
  float* sigma_out;   // [count][128] or null
  double* gram;       // [count][128][128]
  double* vecs;       // [count][128][128]
  double* lam;        // [count][128]
  double* part;       // [count][kGramChunks][3][64][64]; then the Jacobi rotations
  int32_t* status;    // [count][2]: converged, sweeps
  int32_t* graded;    // [count]: the diagonal of G is graded
  hipStream_t stream;
};
hipError_t launch_calibrate(const CalibLaunch& a);
constexpr int kJacobiMaxSweeps = 40;
constexpr int kGramChunks = 32;
// workspace per problem, in doubles: gram, vecs, lam, partials, status and graded
constexpr size_t kCalibPart = (size_t)kGramChunks * 3 * 64 * 64;
constexpr size_t kCalibWorkspace = sizeof(double) * (2 * kD * kD + kD + kCalibPart + 32);
static_assert(kCalibPart * sizeof(double) >=
                  (size_t)kJacobiMaxSweeps * (kD - 1) * (kD / 2) * sizeof(float) &&
                  kCalibPart >= (size_t)kD * kD + kD,
              "the reflectors, then the rotations, take the partials' place");

}  // namespace swan

// The AppendKernel of swan_compress_append with these arguments (-1: refused), for the
// tests that are written for one of them; host arithmetic only.
extern "C" int32_t swan_append_kernel(int32_t dtype, int32_t batch, int32_t n_kv_heads,
                                      int32_t buffer_tokens, const int32_t* seq_len_host,
                                      int32_t n_new, const int32_t* n_new_host);
