// What the reduction kernel and the expansion's prologue share: the term of an element, the order of the
// top-K list, and the partial results of a row that several workgroups reduce.
//
// A launch of few rows leaves most of the chip idle when a row belongs to one workgroup.  Such a row is cut
// into P parts, one workgroup each, that leave a partial result in the workspace: the K best of the part, the sum
// of the terms and its reference exponent.  The expansion kernel's prologue merges them (one wavefront a row, the
// parts' K best one candidate a lane, P K <= 64), so the split costs no launch of its own.
#pragma once

#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>

#include "expand_common.h"
#include "internal.h"

namespace caddtree {
namespace red {

constexpr float kLog2eHi = 0x1.715476p+0f;     // log2(e) rounded to fp32
constexpr float kLog2eLo = 0x1.4ae0c0p-26f;    // log2(e) - kLog2eHi, rounded to fp32
constexpr double kLog2eD = 0x1.71547652b82fep+0;
constexpr double kLn2D = 0x1.62e42fefa39efp-1;
constexpr float kNoExp = -1.0e30f;             // "no reference exponent yet"

__device__ __forceinline__ float term(float x, float r) {
  float a = fmaf(x, kLog2eHi, -r);
  a = fmaf(x, kLog2eLo, a);
  return __builtin_amdgcn_exp2f(a);
}

// (value, id) as one unsigned 64-bit key whose order is the top-K order: the value's bits mapped
// to an unsigned integer that grows with the value (-0 taken as +0, which compares equal to it),
// then INT_MAX - id (smaller ids first)
__device__ __forceinline__ uint64_t order_key(float v, int id) {
  uint32_t b = (uint32_t)__float_as_int(v);
  if (b == 0x80000000u) b = 0u;
  const uint32_t u = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
  return ((uint64_t)u << 32) | (uint32_t)(INT_MAX - id);
}
// A list's empty slot as candidate i of its row's parts: below every element, and distinct, so that the ranks are.
__device__ __forceinline__ uint64_t empty_key(int i) { return (uint64_t)(uint32_t)i; }
__device__ __forceinline__ int key_id(uint64_t k) { return (k >> 32) != 0 ? INT_MAX - (int)(uint32_t)k : INT_MAX; }

// One row's partial results, P parts (split_row_bytes(K, P) bytes a row)
struct PartRow {
  uint64_t* key;  // [P, K] the K best of each part, as keys
  double* sum;    // [P] sum of the part's terms, relative to r
  float* r;       // [P]
  float* v;       // [P, K] the values as read (the sign of a zero included)
};
__device__ __forceinline__ PartRow part_row(void* parts, int64_t row, int K, int P) {
  char* b = static_cast<char*>(parts) + row * (int64_t)split_row_bytes(K, P);
  PartRow p;
  p.key = reinterpret_cast<uint64_t*>(b);
  p.sum = reinterpret_cast<double*>(p.key + P * K);
  p.r = reinterpret_cast<float*>(p.sum + P);
  p.v = p.r + P;
  return p;
}

__device__ __forceinline__ double lse_of(double sum, float R) { return (double)R * kLn2D + log(sum); }

// A row's partial results as a wavefront holds them: lane i < P K one candidate, lane p < P a part's sum.
struct PartRegs {
  uint64_t key;
  double sum;
  float v, r;
  __device__ __forceinline__ void load(const PartRow& p, int K, int P, int lane) {
    const int i = lane < P * K ? lane : P * K - 1, q = lane < P ? lane : P - 1;
    key = p.key[i];
    v = p.v[i];
    sum = p.sum[q];
    r = p.r[q];
  }
};

// Merges a row's candidates: lane k < K gets the k-th best in v, id.  A candidate's rank among all of them is
// its lane (the keys are distinct).
__device__ __forceinline__ void merge_list(const PartRegs& m, int n, int lane, float& v, int& id) {
  const uint64_t key = lane < n ? m.key : 0ull;
  const uint32_t klo = (uint32_t)key, khi = (uint32_t)(key >> 32);
  int rank = lane < n ? 0 : 63;
#pragma unroll 8
  for (int j = 0; j < n; ++j) {
    const uint64_t kj = ((uint64_t)xp::rl_u(khi, j) << 32) | xp::rl_u(klo, j);
    rank += kj > key ? 1 : 0;
  }
  const int to = (rank < 63 ? rank : 63) * 4;
  v = __int_as_float(__builtin_amdgcn_ds_permute(to, __float_as_int(m.v)));
  id = __builtin_amdgcn_ds_permute(to, key_id(key));
}
// ... and its sum, in part order, the same in every lane
__device__ __forceinline__ void merge_sum(const PartRegs& m, int P, double& sum, float& R) {
  R = __uint_as_float(xp::rl_u(__float_as_uint(m.r), 0));
  for (int p = 1; p < P; ++p) R = fmaxf(R, __uint_as_float(xp::rl_u(__float_as_uint(m.r), p)));
  const double t = ldexp(m.sum, (int)fmaxf(m.r - R, -2000.f));
  sum = 0.0;
  for (int p = 0; p < P; ++p) sum += xp::rl_d(t, p);
}

}  // namespace red
}  // namespace caddtree
