// Stage 1: per (round, position) row, the full-vocabulary log-normaliser
// LSE = log sum_v exp(l_v) and the top-K tokens by (logit desc, id asc)
// (Sec. 3.2, eq. marginals; the Require line of Algorithm 1).
//
// One HBM pass per row.  The row's 16-byte aligned part is cut into `waves_per_row`
// contiguous segments, one wavefront each, all in one workgroup; the few elements
// before and after it (rows of a vocabulary or a stride that is no multiple of 16
// bytes start anywhere) are one more step of the last wavefront, one element a lane.
// (Element loads for every row off a 16-byte boundary took 181 us for 48 x 15 rows of
// 100003 bf16 logits; the vectors and the edge step 40, and 33 with the row-wide
// threshold.)
// A wavefront streams 16-byte loads (8 bf16 or 4 fp32 per lane, 1 KiB per wave per
// load) and keeps, per lane, an fp64 sum of 2^(x log2 e - r) where r is a wave-uniform
// integer exponent, a little below the running maximum's, that only grows: when it
// moves, the sums are rescaled by an exact power of two.  The exponent argument is
// formed with a two-part log2 e (two fmas), so the only per-term errors are the
// argument's rounding and the hardware exp2.
//
// Top-K: the wave keeps a sorted list of 16 slots in lanes 0..15 of its first
// DPP row.  An element is a candidate when it reaches the wave threshold (an initial
// lower bound, then the next value above the K-th slot's); the fast path is one
// compare of the lane's chunk maximum per 8 elements, and the rare path inserts
// candidates one at a time with a DPP row shift.  The initial bound is the K-th
// largest of the lanes' maxima over the first chunks of all of the row's wavefronts,
// which is <= the K-th largest element, so no top-K element is ever filtered out.
//
// At the end every wavefront replaces its listed terms' fp32 exp2 values (recomputed
// bit-identically from the exponent recorded at insertion) by fp64 values, which
// removes the error of the largest terms from the normaliser; the waves' lists are
// merged (each candidate, as a 64-bit key, is ranked against all of them in one pass),
// and wave 0 combines the per-wave sums.
//
// A row of a few rounds may be cut into parts of a workgroup each, which the expansion
// merges (reduce_merge.h).

#include <climits>
#include <cmath>

#include "expand_common.h"
#include "internal.h"
#include "reduce_merge.h"

namespace caddtree {
namespace {

using namespace red;

constexpr int kWave = 64;
constexpr int kMaxWaves = 8;                    // wavefronts per row
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Streaming 16-byte loads of a wavefront's segment, with the non-temporal hint (each byte of the logits is
// read once).  Buffer loads: the segment's base and size are scalars and the lane's offset never changes, so a
// load needs no vector address arithmetic, and a load past the segment's end returns zeros without touching
// memory, so the ring needs no branch or clamp at the end of a segment.  The hardware holds the sum of the lane's
// offset and the instruction's (12 bits) against the size; the scalar offset is no part of that check, so it
// stays 0 and a group of eight loads takes two descriptors, 4 KiB apart.
constexpr int kNonTemporal = 2;                 // the nt bit of a buffer load's cache policy
constexpr int kSpan = 4;                        // loads of 1 KiB that the instruction's offset reaches
struct Segment {
  const char* base;                             // the next group's first vector (wave-uniform)
  int64_t left;                                 // bytes from there to the segment's end
  // the bytes from `at` on
  __device__ __forceinline__ auto rsrc(int at) const {
    const int64_t n = left - at;
    const int64_t cut = n < 0 ? 0 : (n < (1 << 30) ? n : (1 << 30));   // a group is at most 8 KiB
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base) + at, 0, (int)cut, 0x00027000);
  }
};
template <typename R>
__device__ __forceinline__ uint4 span_load(R rsrc, int& lane_off, int k) {
  asm volatile("" : "+v"(lane_off));            // (no register is kept for its sums with the loads' places)
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane_off + k * (kWave * 16), 0, kNonTemporal);
  return make_uint4(v.x, v.y, v.z, v.w);
}
// load u of a group (u is known at compile time): vector u kWave + lane; lo and hi: the group's descriptors
template <typename R>
__device__ __forceinline__ uint4 stream_load(R lo, R hi, int& lane_off, int u) {
  return u < kSpan ? span_load(lo, lane_off, u) : span_load(hi, lane_off, u - kSpan);
}

template <typename T> struct Vec;
template <> struct Vec<float> { static constexpr int n = 4; };
template <> struct Vec<uint16_t> { static constexpr int n = 8; };

__device__ __forceinline__ float readlane_f(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ int readlane_i(int v, int l) { return __builtin_amdgcn_readlane(v, l); }

// lane k <- lane k-1 inside each row of 16 lanes; lane 0 of a row gets 0
__device__ __forceinline__ int shr1(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true); }
__device__ __forceinline__ float shr1f(float v) { return __int_as_float(shr1(__float_as_int(v))); }

// the maximum over the wave, wave-uniform: a DPP max-scan (row shifts, then row broadcasts; a lane
// with no source keeps its own value), whose last lane holds the total
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_keep(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, ROW_MASK, 0xF, false));
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_keep<0x111, 0xF>(v));
  v = fmaxf(v, dpp_keep<0x112, 0xF>(v));
  v = fmaxf(v, dpp_keep<0x114, 0xF>(v));
  v = fmaxf(v, dpp_keep<0x118, 0xF>(v));
  v = fmaxf(v, dpp_keep<0x142, 0xA>(v));
  v = fmaxf(v, dpp_keep<0x143, 0xC>(v));
  return readlane_f(v, kWave - 1);
}

// ---- the 16 largest of the wave's 64 values, for the initial threshold: each row of 16 lanes is sorted in
// descending order by a bitonic network, then rows are merged pairwise (the larger of a row and the other
// row reversed is a bitonic row of the 16 largest of both)
template <int CTRL>
__device__ __forceinline__ float dpp_row(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
// the value of lane ^ J, J < 16 (XOR 4 and 8: a permutation of the quad or row, then a half-row mirror)
template <int J>
__device__ __forceinline__ float row_xor(float v) {
  if constexpr (J == 1) return dpp_row<0xB1>(v);
  else if constexpr (J == 2) return dpp_row<0x4E>(v);
  else if constexpr (J == 4) return dpp_row<0x141>(dpp_row<0x1B>(v));
  else return dpp_row<0x141>(dpp_row<0x140>(v));
}
// one compare-exchange stage at distance J of blocks of KB lanes (KB = 16: every row descending)
template <int KB, int J>
__device__ __forceinline__ float row_stage(float v, int lane) {
  const float o = row_xor<J>(v);
  const bool keep_max = ((lane & J) == 0) == ((lane & KB & 15) == 0);
  return keep_max ? fmaxf(v, o) : fminf(v, o);
}
__device__ __forceinline__ float row_merge_sort(float v, int lane) {   // a bitonic row to descending order
  v = row_stage<16, 8>(v, lane);
  v = row_stage<16, 4>(v, lane);
  v = row_stage<16, 2>(v, lane);
  return row_stage<16, 1>(v, lane);
}
__device__ __forceinline__ float row_sort(float v, int lane) {
  v = row_stage<2, 1>(v, lane);
  v = row_stage<4, 2>(v, lane);
  v = row_stage<4, 1>(v, lane);
  v = row_stage<8, 4>(v, lane);
  v = row_stage<8, 2>(v, lane);
  v = row_stage<8, 1>(v, lane);
  return row_merge_sort(v, lane);
}
// the 16 largest of two descending rows, in descending order
__device__ __forceinline__ float row_merge(float a, float b, int lane) {
  return row_merge_sort(fmaxf(a, dpp_row<0x140>(b)), lane);
}
// the 16 largest of four descending rows (one per 16 lanes), in descending order in every row
__device__ __forceinline__ float merge_rows(float v, int lane) {
  v = row_merge(v, __shfl_xor(v, 16), lane);
  return row_merge(v, __shfl_xor(v, 32), lane);
}

// (v, id) goes before (w, wid) in the order value desc, id asc
__device__ __forceinline__ bool before(float v, int id, float w, int wid) {
  return v > w || (v == w && id < wid);
}

// The reference exponent for a running maximum of mx: terms of up to 2^4.  The hardware exp2's error is
// biased and grows with the size of its argument, so the reference sits a little below the maximum, nearer
// the terms that make up most of the sum of a flat row; the largest terms are recomputed in fp64 at the end.
// Normaliser against 64 bits, rms, with the reference 3, 4, 5 and 6 below: 1024 rows of 151936 bf16 normal logits
// 1.8e-8, 1.3e-8, 1.0e-8, 8.8e-9; 512 of 32024 1.2e-8, 9.1e-9, 1.2e-8, 1.9e-8; 1024 of 151936 of Gumbel noise over a
// temperature of 3 6.7e-9, 6.5e-9, 7.0e-9, 7.4e-9, over one of 0.3 5.0e-11, 4.0e-11, 3.6e-11, 3.2e-11.
__device__ __forceinline__ float ref_exp(float mx) { return ceilf(mx * kLog2eHi) - 4.0f; }

struct WaveState {
  double acc;     // per lane
  float r;        // wave-uniform reference exponent (integral value)
  float mx;       // wave-uniform running maximum
  float thr;      // wave-uniform: an element still to come is a candidate if it reaches this
  float lv;       // list slot (lanes 0..15): value, id, exponent at insertion
  int lid;
  float lr;
};

// the least value above v (+inf: NaN, which no value reaches)
__device__ __forceinline__ float next_up(float v) {
  const int b = __float_as_int(v);
  return __int_as_float(v == 0.f ? 1 : b + (b < 0 ? -1 : 1));
}

// Inserts an element.  A segment is read in the order of the ids, so once the list holds K elements those still
// to come enter only above the K-th value: values equal to it (a constant row, masked logits) are no candidates.
// (Compared with >=, each of them took a turn of the rare path's loop: 1024 rows of 151936 bf16 logits, all equal
// or all but five masked, 7750 us, now 54 and 51, against 57 of random ones.)
__device__ __forceinline__ void list_insert(WaveState& s, float v, int id, float r, int K) {
  const bool b = before(v, id, s.lv, s.lid);
  const float pv = shr1f(s.lv);
  const int pid = shr1(s.lid);
  const float pr = shr1f(s.lr);
  const int pb = shr1(b ? 1 : 0);
  if (b) {
    if (pb) { s.lv = pv; s.lid = pid; s.lr = pr; }
    else    { s.lv = v;  s.lid = id;  s.lr = r; }
  }
  if (readlane_i(s.lid, K - 1) != INT_MAX) s.thr = next_up(readlane_f(s.lv, K - 1));
}

// a value that 16 lanes reach: the least of the largest of 16 groups (lanes l, l + 16, l + 32, l + 48)
__device__ __forceinline__ float sixteenth(float v) {
  const unsigned b = __float_as_uint(v);
  const auto h = __builtin_amdgcn_permlane32_swap(b, b, false, false);   // the lower and the upper half, in both
  v = fmaxf(__uint_as_float(h[0]), __uint_as_float(h[1]));
  const unsigned c = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane16_swap(c, c, false, false);   // the even and the odd rows, in both
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  v = fminf(v, row_xor<1>(v));
  v = fminf(v, row_xor<2>(v));
  v = fminf(v, row_xor<4>(v));
  v = fminf(v, row_xor<8>(v));
  return readlane_f(v, 0);
}

// x[j] of a per-lane j: a tree of bit selects (a select between array elements would become an indexed
// access, which registers do not have)
template <int VEC>
__device__ __forceinline__ float pick(const float (&x)[VEC], int j) {
  uint32_t t[VEC];
#pragma unroll
  for (int i = 0; i < VEC; ++i) t[i] = __float_as_uint(x[i]);
#pragma unroll
  for (int w = 1; w < VEC; w <<= 1) {
    const uint32_t up = (j & w) ? ~0u : 0u;
#pragma unroll
    for (int i = 0; i + w < VEC; i += 2 * w) t[i] = (t[i + w] & up) | (t[i] & ~up);
  }
  return __uint_as_float(t[0]);
}

// the reference exponent after elements of up to cmax in each lane
__device__ __forceinline__ void move_reference(WaveState& s, float cmax) {
  if (__ballot(cmax > s.mx)) {
    const float m = wave_max(cmax);
    s.mx = m;
    const float nr = ref_exp(m);
    if (nr > s.r) {
      s.acc = ldexp(s.acc, (int)fmaxf(s.r - nr, -2000.f));
      s.r = nr;
    }
  }
}

// Rare path of a chunk: move the reference exponent, then insert candidates, in the order of their ids.
// x[j] of lane l is element base + l VEC + j of the row; lanes with ok unset hold none.
// The insertion stands in one loop over all (lane, j) candidates and not once per j: this path is
// inlined into every unrolled chunk, and the code of a row is fetched once per launch, so a short
// launch pays for its length (one copy per j: 62 KB of code, the size of the instruction
// cache).
// Where most lanes hold candidates (values that rise along the row), the threshold first rises to a value that 16
// of them reach; and each turn drops, in all lanes at once, the candidates that the threshold has passed.  (Rows
// of 151936 rising bf16 logits: 1858 us with a turn for each, now 66.)  A candidate that comes up when the
// threshold has passed it changes none of the K best.
template <int VEC>
__device__ __forceinline__ void rare(WaveState& s, const float (&x)[VEC], bool ok, float cmax,
                                     unsigned long long cands, int base, int K, int lane) {
  static_assert(CADDTREE_MAX_K <= 16, "16 elements reach the raised threshold");
  move_reference(s, cmax);
  // (a lane of NaN alone holds nothing)
  if (__builtin_expect(__popcll(cands) > 32, 0))
    s.thr = fmaxf(s.thr, sixteenth(ok ? fmaxf(cmax, -INFINITY) : -INFINITY));
  uint32_t cm = 0u;                            // bit j: x[j] is a candidate
#pragma unroll
  for (int j = 0; j < VEC; ++j) cm |= (ok && x[j] >= s.thr) ? 1u << j : 0u;
  unsigned long long m = __ballot(cm != 0u);
#pragma unroll 1
  while (m) {
    const int l = __builtin_ctzll(m);
    const int jl = __builtin_ctz(cm | 0x100u);   // this lane's next candidate
    const float xl = pick(x, jl);
    list_insert(s, readlane_f(xl, l), base + l * VEC + readlane_i(jl, l), s.r, K);
    if (lane == l || !(xl >= s.thr)) cm &= cm - 1u;
    m = __ballot(cm != 0u);
  }
}

// The elements outside the aligned part: at most one a lane (x; -inf in a lane without one).  Those before it
// come after it here, so a value equal to the K-th may still enter, by its id.
template <typename IdOf>
__device__ __forceinline__ void edge_step(WaveState& s, float x, bool ok, IdOf id_of, int K, int lane) {
  const float least = readlane_i(s.lid, K - 1) != INT_MAX ? readlane_f(s.lv, K - 1) : s.thr;
  unsigned long long m = __ballot(ok && x >= least);
  if (m) move_reference(s, x);
  while (m) {
    const int l = __builtin_ctzll(m);
    m &= m - 1;
    list_insert(s, readlane_f(x, l), id_of(l), s.r, K);
  }
  s.acc += ok ? (double)term(x, s.r) : 0.0;
}

// A chunk: one vector a lane, elements base + lane * VEC + j (a lane with ok unset holds -inf, whose
// terms are zero).  Every lane adds its terms pairwise in fp32 and the result once in
// fp64.  A lane whose elements include a candidate (the rare path), and every lane of the
// row's last, ragged chunk, then adds the fp64 difference between its terms summed one by
// one and that fp32 sum: its contribution is the fp64 sum of its fp32 terms.  So the
// correction of the listed terms at the end removes their whole error, and a short row
// is summed in fp64.
template <int VEC>
__device__ __forceinline__ void chunk(WaveState& s, const float (&x)[VEC], bool ok, bool ragged, int base, int K,
                                      int lane) {
  float cmax = x[0];
#pragma unroll
  for (int j = 1; j < VEC; ++j) cmax = fmaxf(cmax, x[j]);
  const bool cand = ok && cmax >= s.thr;
  const unsigned long long cands = __ballot(cand);
  const bool any = cands != 0;
  if (__builtin_expect(any, 0)) rare<VEC>(s, x, ok, cmax, cands, base, K, lane);
  float t[VEC], p[VEC];
#pragma unroll
  for (int j = 0; j < VEC; ++j) p[j] = t[j] = term(x[j], s.r);
#pragma unroll
  for (int w = 1; w < VEC; w <<= 1)
#pragma unroll
    for (int j = 0; j + w < VEC; j += 2 * w) p[j] += p[j + w];
  s.acc += (double)p[0];
  if (__builtin_expect(any || ragged, 0) && (cand || ragged)) {
    double e = 0.0;
#pragma unroll
    for (int j = 0; j < VEC; ++j) e += (double)t[j];
    s.acc += e - (double)p[0];
  }
}

__device__ __forceinline__ void unpack(const uint4& q, float (&x)[8]) {
  x[0] = __uint_as_float(q.x << 16); x[1] = __uint_as_float(q.x & 0xffff0000u);
  x[2] = __uint_as_float(q.y << 16); x[3] = __uint_as_float(q.y & 0xffff0000u);
  x[4] = __uint_as_float(q.z << 16); x[5] = __uint_as_float(q.z & 0xffff0000u);
  x[6] = __uint_as_float(q.w << 16); x[7] = __uint_as_float(q.w & 0xffff0000u);
}
__device__ __forceinline__ void unpack(const uint4& q, float (&x)[4]) {
  x[0] = __uint_as_float(q.x); x[1] = __uint_as_float(q.y);
  x[2] = __uint_as_float(q.z); x[3] = __uint_as_float(q.w);
}

__device__ __forceinline__ uint32_t raw_bits(const float* p) { return __float_as_uint(*p); }
__device__ __forceinline__ uint32_t raw_bits(const uint16_t* p) { return *p; }

// kUnroll: 16-byte loads in flight per lane (4 or 8); kS: wavefronts per row (1, 2, 4 or 8)
template <typename T, int kUnroll, int kS>
__global__ void __launch_bounds__(kWave * kMaxWaves)
reduce_topk_kernel(const T* __restrict__ logits, int64_t row_stride, int V, int K,
                   int32_t* __restrict__ out_ids, float* __restrict__ out_logit,
                   float* __restrict__ out_lq, double* __restrict__ out_lse, void* __restrict__ parts) {
  constexpr int VEC = Vec<T>::n;
  constexpr int CH = kWave * VEC;
  __shared__ float s_top[16 * kS];      // the waves' 16 largest lane maxima of the first group
  __shared__ double s_acc[kS];
  __shared__ float s_r[kS];
  __shared__ uint64_t s_key[16 * kS];   // the waves' K best as keys
  __shared__ float s_kv[16 * kS];       // ... their values as read (the sign of a zero included)
  __shared__ int s_sel[16];

  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  constexpr int S = kS;
  const int64_t row = blockIdx.x;
  const T* rowp = logits + row * row_stride;
  // the row's aligned part: nv vectors from element `head` on
  const int mis = (int)((reinterpret_cast<uintptr_t>(rowp) & 15u) / sizeof(T));
  const int head = mis == 0 ? 0 : (VEC - mis < V ? VEC - mis : V);
  const int nv = (V - head) / VEC;
  const int nch = (nv + kWave - 1) / kWave;
  const int P = (int)gridDim.y, part = (int)blockIdx.y;   // a row may be cut into P parts, one workgroup each
  const int c0 = (int)((int64_t)(part * S + wave) * nch / (P * S));
  const int c1 = (int)((int64_t)(part * S + wave + 1) * nch / (P * S));
  const int v1 = c1 * kWave < nv ? c1 * kWave : nv;   // the segment's vectors are c0 kWave .. v1 - 1

  WaveState s;
  s.acc = 0.0; s.r = kNoExp; s.mx = -INFINITY; s.thr = -INFINITY;
  s.lv = -INFINITY; s.lid = INT_MAX; s.lr = 0.f;

  // elements 0 .. head - 1 and head + nv VEC .. V - 1, fewer than 2 VEC in all: a step of the last
  // wavefront, loaded ahead of its stream
  const int gap = nv * VEC;
  const auto edge_id = [head, gap](int l) { return l < head ? l : gap + l; };
  const int edge = wave == S - 1 && part == P - 1 ? V - gap : 0;
  uint32_t edge_raw = 0u;
  if (lane < edge) edge_raw = raw_bits(rowp + edge_id(lane));

  int lane_off = lane * 16;
  Segment seg{reinterpret_cast<const char*>(rowp + head) + (int64_t)c0 * (kWave * 16),
              (int64_t)(v1 - c0 * kWave) * 16};
  int c = c0;
  uint4 q[kUnroll];
  {
    const auto lo = seg.rsrc(0), hi = seg.rsrc(kSpan * kWave * 16);
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) q[u] = stream_load(lo, hi, lane_off, u);
  }
  // The first group (all of a short segment) sets the reference exponent and the initial threshold: the
  // K-th largest over the row's wavefronts of each lane's maximum, so that K elements reach it.  Whatever
  // it lets through is inserted one by one, and each of the row's wavefronts fills a list of its own, so a
  // short segment spends more on its list than on its stream when the bound is loose: with the least of
  // K lane groups' maxima, each wavefront's own, 16 rows of 151936 bf16 took 28.4 us, with this one 17.1
  // (1024 rows: 58.0 and 53.7).
  {
    float g = -INFINITY;
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {   // unpacked twice: keeps the live registers to one chunk
      float x[VEC];
      unpack(q[u], x);
      float m = x[0];
#pragma unroll
      for (int j = 1; j < VEC; ++j) m = fmaxf(m, x[j]);
      g = (c0 + u) * kWave + lane < v1 ? fmaxf(g, m) : g;
    }
    float t = merge_rows(row_sort(g, lane), lane);
    s.mx = readlane_f(t, 0);
    if constexpr (S > 1) {
      if (lane < 16) s_top[wave * 16 + lane] = t;
      __syncthreads();
      if constexpr (S <= 4) {
        t = lane < S * 16 ? s_top[lane] : -INFINITY;
      } else {
        t = s_top[lane];
#pragma unroll
        for (int w = kWave; w < S * 16; w += kWave) t = row_merge(t, s_top[w + lane], lane);
      }
      t = merge_rows(t, lane);
    }
    s.thr = readlane_f(t, K - 1);
    // an element moves the reference only as a candidate, so the reference may not lie below the bound
    // (a segment that starts with masked logits)
    s.mx = fmaxf(s.mx, s.thr);
    s.r = fmaxf(ref_exp(s.mx), kNoExp);
  }
  if (c0 < c1) {
    // a ring of kUnroll loads in flight: each chunk's slot (the first group's too) is refilled with the
    // load kUnroll chunks ahead as soon as its registers are unpacked, before its arithmetic.  The last
    // group's loads run through the ring as well, zeros past the segment's end: a load that is waited for
    // alone costs its whole latency, which a short segment would pay up to kUnroll - 1 times
#pragma unroll 1
    for (; c + kUnroll < c1; c += kUnroll) {
      seg.base += kUnroll * kWave * 16;
      seg.left -= kUnroll * kWave * 16;
      const auto lo = seg.rsrc(0), hi = seg.rsrc(kSpan * kWave * 16);
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        float x[VEC];
        unpack(q[u], x);
        q[u] = stream_load(lo, hi, lane_off, u);
        chunk<VEC>(s, x, true, false, head + (c + u) * CH, K, lane);
      }
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      if (c + u < c1) {
        const bool ok = (c + u) * kWave + lane < v1;
        float x[VEC];
        unpack(q[u], x);
        const bool ragged = (c + u + 1) * kWave > v1;   // the row's last chunk, of fewer than kWave vectors
        if (ragged) {
#pragma unroll
          for (int j = 0; j < VEC; ++j) x[j] = ok ? x[j] : -INFINITY;
        }
        chunk<VEC>(s, x, ok, ragged, head + (c + u) * CH, K, lane);
      }
    }
  }
  if (edge > 0) {
    asm volatile("" : "+v"(edge_raw));     // the value is first wanted here: no wait for it before the stream
    const float x = __uint_as_float(sizeof(T) == 2 ? edge_raw << 16 : edge_raw);
    edge_step(s, lane < edge ? x : -INFINITY, lane < edge, edge_id, K, lane);
  }

  // The fp32 terms of the listed elements (the K best and what they displaced), recomputed bit for bit, are
  // replaced by fp64 values.  Every wavefront does so for its own list, at once and off wave 0's path: what the
  // merge leaves out is exact as well, and a sharp row's sum lies there (256 rows of 151936 bf16 of Gumbel noise over a
  // temperature of 0.3, K = 8: rms error 4.9e-11; 7.3e-10 with the row's K best alone).
  if (lane < 16 && s.lid != INT_MAX) {
    const double approx = ldexp((double)term(s.lv, s.lr), (int)fmaxf(s.lr - s.r, -2000.f));
    s.acc += exp2((double)s.lv * kLog2eD - (double)s.r) - approx;
  }
  // wave sum of the per-lane accumulators (fixed order: a DPP scan, the total in the last lane)
  const double acc = xp::rl_d(xp::wave_incl_scan(s.acc), kWave - 1);
  const int n = S * K;                    // candidates: every wave's K best, wave w's at w K .. w K + K - 1
  if (S > 1 && lane < K) {
    s_key[wave * K + lane] = order_key(s.lv, s.lid);
    s_kv[wave * K + lane] = s.lv;
  }
  if (lane == 0) { s_acc[wave] = acc; s_r[wave] = s.r; }
  if (wave == 0 && lane < K) s_sel[lane] = lane;   // a valid index in every slot, whatever the row holds
  __syncthreads();
  if (S > 1) {
    // One candidate a thread, over as many waves as that takes: its rank among all of them is its slot in
    // the merged list.  Real entries have distinct keys (ids are distinct); the padding of a segment with
    // fewer than K elements shares one key below every real one.  The row holds at least K elements, so
    // slots 0 .. K - 1 each receive exactly one candidate, a real one.
    // (Inserting the waves' lists one by one, as products S K above 64 did, is a chain of S K dependent
    // steps on one wave.)
    const int me = threadIdx.x;
    if (me < n) {
      const uint64_t key = s_key[me];
      int rank = 0;
#pragma unroll 4
      for (int j = 0; j < n; ++j) rank += s_key[j] > key ? 1 : 0;
      if (rank < K) s_sel[rank] = me;
    }
    if (n > kWave) __syncthreads();
  }
  if (wave != 0) return;
  if (S > 1 && lane < K) {
    const int src = s_sel[lane];
    s.lid = key_id(s_key[src]);
    s.lv = s_kv[src];
  }
  float R = s_r[0];
#pragma unroll
  for (int w = 1; w < S; ++w) R = fmaxf(R, s_r[w]);
  double sum = 0.0;
#pragma unroll
  for (int w = 0; w < S; ++w) sum += ldexp(s_acc[w], (int)fmaxf(s_r[w] - R, -2000.f));
  if (P > 1) {                             // a part's result, merged by the expansion
    const PartRow pr = part_row(parts, row, K, P);
    if (lane < K) {
      pr.key[part * K + lane] = s.lid != INT_MAX ? order_key(s.lv, s.lid) : empty_key(part * K + lane);
      pr.v[part * K + lane] = s.lv;
    }
    if (lane == 0) {
      pr.sum[part] = sum;
      pr.r[part] = R;
    }
    return;
  }
  const double lse = lse_of(sum, R);
  if (lane < K) {
    const int64_t o = row * K + lane;
    out_ids[o] = s.lid;
    out_logit[o] = s.lv;
    if (out_lq) out_lq[o] = (float)((double)s.lv - lse);
  }
  if (lane == 0) out_lse[row] = lse;
}

// The parts of a split reduction merged by a kernel of its own, a wavefront a row, before the expansions whose
// prologue does not (about 4 us, still less than the split saves).
constexpr int kMergeRows = 4;
__global__ void __launch_bounds__(kMergeRows * kWave) merge_kernel(MergeIn mg, int64_t rows, int K) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t row = (int64_t)blockIdx.x * kMergeRows + threadIdx.x / kWave;
  if (row >= rows) return;
  PartRegs m;
  m.load(part_row(mg.parts, row, K, mg.split), K, mg.split, lane);
  float v, R;
  int id;
  double sum;
  merge_list(m, mg.split * K, lane, v, id);
  merge_sum(m, mg.split, sum, R);
  const double lse = lse_of(sum, R);
  if (lane < K) {
    mg.ids[row * K + lane] = id;
    mg.logit[row * K + lane] = v;
    if (mg.lq) mg.lq[row * K + lane] = (float)((double)v - lse);
  }
  if (lane == 0) mg.lse[row] = lse;
}

template <typename T, int U, int S>
void launch_s(const ReduceArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL((reduce_topk_kernel<T, U, S>), dim3((unsigned)a.rows, (unsigned)a.split),
                     dim3((unsigned)(kWave * S)), 0, stream, static_cast<const T*>(a.logits), a.row_stride, a.V, a.K,
                     a.ids, a.logit, a.lq, a.lse, a.parts);
}

template <typename T, int U>
hipError_t launch_u(const ReduceArgs& a, hipStream_t stream) {
  switch (a.waves_per_row) {
    case 1: launch_s<T, U, 1>(a, stream); break;
    case 2: launch_s<T, U, 2>(a, stream); break;
    case 4: launch_s<T, U, 4>(a, stream); break;
    case 8: launch_s<T, U, 8>(a, stream); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename T>
hipError_t launch_t(const ReduceArgs& a, hipStream_t stream) {
  return a.unroll == 8 ? launch_u<T, 8>(a, stream) : launch_u<T, 4>(a, stream);
}

}  // namespace

// Launch shape, from sweeps of the shapes over 16 .. 22400 rows of 3000 .. 151936 logits (times in us).  `full` is
// the waves of a full chip at four per SIMD, 4096 on 256 compute units.
// - More rows than that: one wave per row, 8 loads in flight (8192 rows of 151936 fp32: 728, with 4 loads 735), but 4
//   for rows of at most 4 chunks (4 against 8 loads, 6400 bf16 rows of 2048: 16.9 and 17.6; of 2500, 5 chunks, 19.5 and
//   19.0, of 4096 25.4 and 21.9, of 32000 76.8 and 73.9) and from 4097 to 8191 fp32 rows (6400 of 4000: 24.3 and 24.9, of
//   32000 125 and 129, of 151936 582 and 595).
// - Else the most waves per row, up to 8, that keep `full` waves on the chip at once and leave a wave 3
//   chunks (64 rows of 16 chunks: 1 wave 19.0, 2 waves 15.5, 4 waves 14.7; 128 rows of 63: 32.1, 25.5, 20.0, and
//   8 waves 17.6).  16 waves are no better at any size (16 rows of 297 chunks 17.1, with 8 waves 16.6; 512
//   rows 37.1 and 28.7).
// - fp32 rows of 4 waves that leave no room for 8 (513 to 1024 rows) take 4 loads (against 8: 600 rows of 32000 18.7 and
//   20.3, 800 23.5 and 25.0, 1000 25.7 and 27.5, 1024 25.7 and 27.6; of 8000 9.8 and 9.9, 11.0 and 11.1, 11.2 and 11.6,
//   11.3 and 11.7; of 151936 59.2 and 61.6, 81.9 and 83.3, 90.8 and 92.5, 92.9 and 94.0).  With 8 waves neither is
//   better throughout (400 rows of 32000 14.4 and 13.9, of 8000 9.0 and 9.1), with fewer waves and in bf16 8 loads are as
//   good or better (1025 fp32 rows of 8000 12.7 and 12.0; 600 bf16 rows of 32000 18.0 and 16.5).
// - So few rows that compute units are left idle, where there is memory for partial results: up to 4 parts per
//   row, at most a compute unit's worth of parts each, and 4 chunks a wave (a build of 16 rows of 297 chunks:
//   25.6, in two parts 23.1, in four 20.9, in eight 22.9, since the merge grows with the parts; 128 rows: 28.1,
//   24.6, 26.1; 192 rows: 27.8, 30.2; 8 rows of 125 chunks: 16.0, 15.9, 15.7).
ReduceShape reduce_default_shape(int64_t rows, int32_t V, int32_t K, caddtree_dtype_t dtype, bool may_split,
                                 int32_t num_cu) {
  const int CH = kWave * (dtype == CADDTREE_BF16 ? 8 : 4);
  const int nch = (V + CH - 1) / CH;
  const int64_t full = 16 * (int64_t)num_cu;
  ReduceShape sh{1, 8, 1};
  if (rows > full) {
    if (nch <= 4 || (dtype == CADDTREE_F32 && rows < 2 * full)) sh.unroll = 4;
    return sh;
  }
  while (sh.waves < 8 && rows * sh.waves * 2 <= full && nch / (2 * sh.waves) >= 3) sh.waves *= 2;
  if (dtype == CADDTREE_F32 && sh.waves == 4 && rows * 8 > full) sh.unroll = 4;
  while (may_split && sh.split < 4 && rows * sh.split * 2 <= num_cu && 2 * sh.split * K <= kWave &&
         nch / (2 * sh.split * sh.waves) >= 4)
    sh.split *= 2;
  return sh;
}

hipError_t launch_reduce_topk(const ReduceArgs& a, caddtree_dtype_t dtype, hipStream_t stream) {
  if (a.rows == 0) return hipSuccess;
  return dtype == CADDTREE_BF16 ? launch_t<uint16_t>(a, stream) : launch_t<float>(a, stream);
}

hipError_t launch_merge(const MergeIn& mg, int64_t rows, int32_t K, hipStream_t stream) {
  if (rows == 0) return hipSuccess;
  hipLaunchKernelGGL(merge_kernel, dim3((unsigned)((rows + kMergeRows - 1) / kMergeRows)), dim3(kMergeRows * kWave), 0,
                     stream, mg, rows, K);
  return hipGetLastError();
}

}  // namespace caddtree
