// gfx950 kernels of the QODA hot path (arXiv 2505.14371): per-layer norms, stochastic quantization + code
// packing, fused decode + K-way mean + optimistic dual averaging update, and the histogram level fit.
//
// Execution shape of the norm and quantize passes: one workgroup = 256 threads = 4 wave64 = one tile of 16384
// coordinates of one (node, layer).  Wave w owns the 16 consecutive 256-coordinate blocks 16w..16w+15 of the tile; in a
// block, lane i owns coordinates 4i..4i+3 (one 128-bit load, 1 KB contiguous per wave).  Thread t = 64w+i is reduction
// slot t of the fixed-order fp64 sums.  The decode pass keeps the lane <-> coordinate mapping but runs in shorter
// workgroups (8, 4 or 2 blocks of an octet per wave, see k_decode).  The packed message is lane-local: the codes of the 32 coordinates a lane
// owns in 8 consecutive blocks (an octet) are shifted into C1 = 1 + b 32-bit words per lane, and word r of the
// 64 lanes is one contiguous 256-byte store.
//
// Arithmetic that feeds an integer decision (level index, rounding direction, packed bits, histogram bin) is
// written as single IEEE operations with contraction off, so that it has one well-defined result.

#include <string.h>

#include "qoda_choices.h"
#include "qoda_kernels.h"

namespace qoda {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));   // plain vector type: usable behind address-space pointers

__device__ __forceinline__ unsigned int f2u(float f) { return __float_as_uint(f); }
__device__ __forceinline__ float u2f(unsigned int u) { return __uint_as_float(u); }

constexpr float kFltMax = 3.402823466e+38f;
constexpr float kFltMin = 1.17549435e-38f;   // 2^-126, the smallest normal float

// Bits of the sticky device status word.
constexpr unsigned int kStatusNonFinite = 1u;   // a statistic is not a finite number in range
constexpr unsigned int kStatusTinyNorm = 2u;    // 0 < norm < 2^-126: 1/norm is not a float (the one case where the
                                                // quantizer of that vector is biased, Thm 5.1)

// largest float n >= 0 with n*n <= s (n*n is exact in fp64); 0 when s is not a finite number in range.
__device__ float sqrt_floor(double s) {
  const double lim = (double)kFltMax * (double)kFltMax;
  if (!(s >= 0.0) || !(s <= lim)) return 0.0f;
  const double r = sqrt(s);
  float n = (r >= (double)kFltMax) ? kFltMax : (float)r;
  for (int it = 0; it < 4 && (double)n * (double)n > s; ++it) n = u2f(f2u(n) - 1u);
  for (int it = 0; it < 4; ++it) {
    if (n == kFltMax) break;
    const float up = u2f(f2u(n) + 1u);
    if ((double)up * (double)up <= s) n = up; else break;
  }
  return n;
}

// largest finite float r >= 0 with x*r <= 1 (exact in fp64); 0 for x <= 0 or non-finite x.
__device__ float rcp_floor(float x) {
  if (!(x > 0.0f) || x > kFltMax) return 0.0f;
  float r = 1.0f / x;
  if (r > kFltMax) r = kFltMax;
  for (int it = 0; it < 4 && (double)x * (double)r > 1.0; ++it) r = u2f(f2u(r) - 1u);
  for (int it = 0; it < 4; ++it) {
    if (r == kFltMax) break;
    const float up = u2f(f2u(r) + 1u);
    if ((double)x * (double)up <= 1.0) r = up; else break;
  }
  return r;
}

// x minus one unit of the last place where m is negative.
__device__ __forceinline__ float step_down(float x, int m) { return u2f(f2u(x) + (unsigned int)(m >> 31)); }

// The same two functions for the per-bucket norms, where they run once per 128 coordinates and their cost shows:
// straight-line code for arguments in a comfortable range (sums of squares in [2^-200, 2^200]), the general
// routines otherwise.  Both return exactly what sqrt_floor / rcp_floor return: the definitions are by exact
// comparisons, and a value less than one unit of the last place off needs only one of them.  (Candidates from two units
// above, stepped down by three comparisons in fp64 each, and a correctly rounded root before them, took twice as long.)
__device__ __forceinline__ void norm_and_inverse(double s, float &n_out, float &r_out) {
  const long long bits = __double_as_longlong(s);
  const int e = (int)((bits >> 52) & 0x7FF) - 1023;
  if (e < -200 || e > 200) {   // zero, tiny, huge or not a number: the general path
    n_out = sqrt_floor(s);
    r_out = rcp_floor(n_out);
    return;
  }
  // s = sp * 4^k with sp in [1, 4)
  const int k = e >> 1;
  const double sp = __longlong_as_double(bits - ((long long)(2 * k) << 52));
  const float sf = (float)sp;                       // moves the root by up to 0.36 unit
  const float y = __builtin_amdgcn_rsqf(sf);        // 1/sqrt(sp) to a few units: one Newton step leaves rounding only
  const float n0 = sf * y;
  float n = __builtin_fmaf(__builtin_fmaf(-n0, n0, sf), 0.5f * y, n0);   // within 0.87 unit: it or the float below it
  const double nd = (double)n;
  n = step_down(n, (int)(__double_as_longlong(__builtin_fma(-nd, nd, sp)) >> 32));   // the fused operation has the exact sign
  const float q = __builtin_fmaf(__builtin_fmaf(-n, y, 1.0f), y, y);     // y is within a few units of 1/n too: 1/2 unit
  const float r = step_down(q, (int)f2u(__builtin_fmaf(-n, q, 1.0f)));
  n_out = u2f(f2u(n) + ((unsigned int)k << 23));    // times 2^k, 2^-k: exact, the results are normal numbers
  r_out = u2f(f2u(r) - ((unsigned int)k << 23));
}

// Lane i + H's value in the lanes i < H of a wave (in the others whatever comes): the step of a halving tree, in registers.  Through the
// shared memory's lane permutation a step takes about 100 cycles, and a short kernel has two to four trees of six steps in its chain:
// us a round of 2 x 512 entries, K = 4 13.9 -> 13.4, of 152 k entries with one norm per vector 23.3 -> 22.1.
template <int H>
__device__ __forceinline__ unsigned int lane_down(unsigned int v) {
  if constexpr (H == 32) return __builtin_amdgcn_permlane32_swap(v, v, false, false)[1];
  else if constexpr (H == 16) return __builtin_amdgcn_permlane16_swap(v, v, false, false)[1];
  else return (unsigned int)__builtin_amdgcn_update_dpp(0, (int)v, 0x100 + H, 0xF, 0xF, true);   // row_shl
}
template <int H>
__device__ __forceinline__ double lane_down(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  return __longlong_as_double((long long)((unsigned long long)lane_down<H>((unsigned int)(b >> 32)) << 32 | lane_down<H>((unsigned int)b)));
}

// The smallest of the lanes' values (never a NaN), valid in lane 0.
__device__ __forceinline__ double lane_least(double r) {
  r = fmin(r, lane_down<32>(r));
  r = fmin(r, lane_down<16>(r));
  r = fmin(r, lane_down<8>(r));
  r = fmin(r, lane_down<4>(r));
  r = fmin(r, lane_down<2>(r));
  return fmin(r, lane_down<1>(r));
}

// The halving tree's steps inside a wave, h = 32 .. 1: r[i] with r[i + h] for i < h.  The result is valid in lane 0.  SUM false: the maximum.
template <bool SUM>
__device__ __forceinline__ double lane_tree(double r) {
  const auto step = [&](double o) { r = SUM ? r + o : fmax(r, o); };
  step(lane_down<32>(r));
  step(lane_down<16>(r));
  step(lane_down<8>(r));
  step(lane_down<4>(r));
  step(lane_down<2>(r));
  step(lane_down<1>(r));
  return r;
}

// Fixed halving tree over the 256 slots: p[i] += p[i+h], h = 128 .. 1.  The two cross-wave steps are one pass
// through shared memory, the six in-wave steps are lane_tree's (lane i < h adds lane i + h, exactly the tree).
// The total is valid in thread 0 only.
__device__ double block_tree(double v, double *red) {
  const int t = threadIdx.x;
  red[t] = v;
  __syncthreads();
  double r = 0.0;
  if (t < 64) {
    r = (red[t] + red[t + 128]) + (red[t + 64] + red[t + 192]);
    r = lane_tree<true>(r);
  }
  __syncthreads();   // red may be reused by the caller
  return r;
}

// The same shape with the maximum instead of the sum (the order does not matter for a maximum; v >= 0, never NaN).
__device__ double block_max(double v, double *red) {
  const int t = threadIdx.x;
  red[t] = v;
  __syncthreads();
  double r = 0.0;
  if (t < 64) {
    r = fmax(fmax(red[t], red[t + 128]), fmax(red[t + 64], red[t + 192]));
    r = lane_tree<false>(r);
  }
  __syncthreads();
  return r;
}

// ----- the three kinds of norm: statistic -> finite?, norm, reciprocal, fit weight
__device__ __forceinline__ bool stat_finite(double s, int kind) {
  const double fm = (double)kFltMax;
  return (s >= 0.0) && (s <= (kind == kNormL2 ? fm * fm : fm));
}
__device__ __forceinline__ float norm_of(double s, int kind) {
  return kind == kNormL2 ? sqrt_floor(s) : __double2float_rn(s);
}
__device__ __forceinline__ double weight_of(double s, int kind) { return kind == kNormL2 ? s : s * s; }
// largest magnitude from the running maximum of magnitude bit patterns: an infinity or a NaN pattern gives +infinity
__device__ __forceinline__ float magnitude_from_bits(unsigned int mb) { return u2f(mb > 0x7F7FFFFFu ? 0x7F800000u : mb); }

// rcp_floor for a norm in a comfortable range by straight-line code (as in norm_and_inverse), the general routine
// otherwise: the same bits either way.
__device__ __forceinline__ float inverse_of(float n) {
  const int e = (int)((f2u(n) >> 23) & 0xFF) - 127;
  if (e < -100 || e > 100) return rcp_floor(n);
  const float y = __builtin_amdgcn_rcpf(n);
  const float q = __builtin_fmaf(__builtin_fmaf(-n, y, 1.0f), y, y);   // within 1/2 unit
  return step_down(q, (int)f2u(__builtin_fmaf(-n, q, 1.0f)));
}

// Norm and inverse of a statistic (0 where it is not finite), by straight-line code where that will do: the general routines are 0.5 us
// on the way of a short kernel.
__device__ __forceinline__ void stat_scale(double s, int kind, float &n, float &r) {
  n = 0.0f;
  r = 0.0f;
  if (!stat_finite(s, kind)) return;
  if (kind == kNormL2) {
    norm_and_inverse(s, n, r);
  } else {
    n = __double2float_rn(s);
    r = inverse_of(n);
  }
}

// Philox4x32-10 (Salmon et al., SC'11).
__device__ __forceinline__ void philox4x32_10(unsigned int c0, unsigned int c1, unsigned int c2, unsigned int c3,
                                               unsigned int k0, unsigned int k1, unsigned int out[4]) {
  constexpr unsigned long long M0 = 0xD2511F53ull, M1 = 0xCD9E8D57ull;
  constexpr unsigned int W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) { k0 += W0; k1 += W1; }
    const unsigned long long p0 = M0 * (unsigned long long)c0;
    const unsigned long long p1 = M1 * (unsigned long long)c2;
    const unsigned int n0 = __builtin_amdgcn_bitop3_b32((unsigned int)(p1 >> 32), c1, k0, 0x96);   // 3-input xor
    const unsigned int n1 = (unsigned int)p1;
    const unsigned int n2 = __builtin_amdgcn_bitop3_b32((unsigned int)(p0 >> 32), c3, k1, 0x96);
    const unsigned int n3 = (unsigned int)p0;
    c0 = n0; c1 = n1; c2 = n2; c3 = n3;
  }
  out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// Table entry of a value u in [0, 1], by its grid bin (bins: kGridPoints entries in shared memory, see build_tables): one
// 128-bit read gives {l_tau, 1/gap, l_tau+1, tau}, tau being that of the bin's lower edge.  (A table of tau by bin and one of
// {l_tau, 1/gap, l_tau+1} by tau are two reads one after the other; k_quantize has that form too, see QuantTables.)
__device__ __forceinline__ float4 bin_entry(const float4 *bins, float u) {
  return bins[__builtin_elementwise_sub_sat(f2u(u) >> 20, (unsigned int)kGridBase)];
}

// The grid bins' entries of a type into shared memory; where a lane may have to walk on from the entry of its bin (walk), also
// the entries by tau, the last one with the upper neighbour +infinity, which stops every walk.  256 threads or more; all loads
// are requested before the first is used (one after the other they cost a small launch 1 us).
__device__ __forceinline__ void load_tables(const Dev &a, int type, int S, int walk, float4 *bins, float4 *tab) {
  static_assert(kGridPoints == kThreads + 1 && kMaxPoints == kThreads, "one entry a thread, and one more");
  const v4f *src = reinterpret_cast<const v4f *>(a.bins + (size_t)type * kGridPoints);
  const float *lev = a.lev + (size_t)type * kMaxPoints, *rg = a.rgap + (size_t)type * kMaxPoints;
  const int t = threadIdx.x, j = min(t, kThreads - 1);
  const v4f v = src[j], last = src[kThreads];
  const float lj = lev[j], ln = lev[min(j + 1, kMaxPoints - 1)], rj = rg[j];
  if (t >= kThreads) return;
  *reinterpret_cast<v4f *>(&bins[t]) = v;
  if (t == 0) *reinterpret_cast<v4f *>(&bins[kThreads]) = last;
  if (walk && t < S) tab[t] = make_float4(lj, rj, t + 1 < S ? ln : __builtin_inff(), u2f((unsigned int)t));   // rgap is 0 from S-1 on
}

// What k_quantize finds a value's level with: {l_tau, 1/gap, l_tau+1} for the tau of its bin's lower edge, and the entries by tau to
// walk on from there (the last one with the upper neighbour +infinity, which stops every walk).
//   BINS   one 128-bit read from the table by grid bin, which has tau in its last word
//   !BINS  tau from a table of bytes by bits(u) >> 20, then the entry of tau: two reads one after the other
// quantize_bins says which, with the times.  The byte form keeps room for 256 entries at every width: with as many as there are levels
// the pass over 74 k tiles (8 levels, K = 8, previous message) takes 1024 to 1032 us instead of 993 to 1009, for the same instructions.
template <int C1, bool BINS>
struct QuantTables {
  float4 bins[BINS ? kGridPoints : 1];
  unsigned int lut[BINS ? 1 : kLutSize / 4];
  float4 tab[BINS ? 1 << (C1 - 1) : kMaxPoints];
};

// The lane's number in its wave, from no register that would have to be kept for it.
__device__ __forceinline__ int lane_id() { return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

// A value of lane bb of the lane's row of 16 lanes.
template <int BB>
__device__ __forceinline__ unsigned int row_lane(unsigned int v) {
  return (unsigned int)__builtin_amdgcn_mov_dpp((int)v, 0x150 + BB, 0xF, 0xF, true);   // row_newbcast
}
__device__ __forceinline__ unsigned int row_value(unsigned int v, int bb) {   // bb in 0..7, known where this is unrolled
  switch (bb) {
    case 0: return row_lane<0>(v);
    case 1: return row_lane<1>(v);
    case 2: return row_lane<2>(v);
    case 3: return row_lane<3>(v);
    case 4: return row_lane<4>(v);
    case 5: return row_lane<5>(v);
    case 6: return row_lane<6>(v);
    default: return row_lane<7>(v);
  }
}

// A neighbour's value inside a group of four lanes (quad permutation CTRL).
template <int CTRL>
__device__ __forceinline__ double quad_swap(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, true), hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, true);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned int)hi << 32) | (unsigned int)lo));
}

// Loads through pointers read from device tables: tell the compiler they point to global memory.
template <class T>
__device__ __forceinline__ const __attribute__((address_space(1))) T *as_global(const T *p) {
  return (const __attribute__((address_space(1))) T *)p;
}

// Four coordinates e..e+3 of a layer of d entries; entries past the end read as +0.
__device__ __forceinline__ void load4(const float *__restrict__ v, long long e, long long d, float x[4]) {
  const auto *g = as_global(v);
  if (e + 4 <= d) {
    // every big array here is streamed once per pass: nontemporal accesses measurably raise the read rate
    const v4f q = __builtin_nontemporal_load(reinterpret_cast<const __attribute__((address_space(1))) v4f *>(g + e));
    x[0] = q.x; x[1] = q.y; x[2] = q.z; x[3] = q.w;
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = (e + j < d) ? g[e + j] : 0.0f;
  }
}

__device__ __forceinline__ void store4(float *__restrict__ v, long long e, long long d, const float x[4]) {
  auto *g = (__attribute__((address_space(1))) float *)v;
  if (e + 4 <= d) {
    v4f q;
    q.x = x[0]; q.y = x[1]; q.z = x[2]; q.w = x[3];
    __builtin_nontemporal_store(q, reinterpret_cast<__attribute__((address_space(1))) v4f *>(g + e));
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (e + j < d) g[e + j] = x[j];
  }
}

// ---- packed lane records (message body).  A lane's 32 codes of an octet (8 blocks x 4 coordinates, code
// number jj = 4*block + component, C1 bits each: sign | index << 1) form a little-endian bit string kept in C1
// 32-bit registers.  jj is a compile-time constant wherever these are called (fully unrolled loops), so every
// shift below is an immediate.
template <int C1>
__device__ __forceinline__ void insert_code(unsigned int (&D)[C1], unsigned int code, int jj) {
  const int pos = C1 * jj, r = pos >> 5, sh = pos & 31;
  D[r] |= code << sh;
  if (sh + C1 > 32) D[r + 1] |= code >> (32 - sh);
}

template <int C1>
__device__ __forceinline__ unsigned int extract_code(const unsigned int (&D)[C1], int jj) {
  const int pos = C1 * jj, r = pos >> 5, sh = pos & 31;
  unsigned int v = D[r] >> sh;
  if (sh + C1 > 32) v |= D[r + 1] << (32 - sh);
  return v & ((1u << C1) - 1u);
}

// Byte offset (code * 4) of code jj into a table of floats: two instructions (shift or funnel shift, mask).
template <int C1, int N>
__device__ __forceinline__ unsigned int extract_off(const unsigned int (&D)[N], int jj) {
  const int pos = C1 * jj, r = pos >> 5, sh = pos & 31;
  unsigned int v;
  if (sh + C1 <= 32) v = (sh >= 2) ? (D[r] >> (sh - 2)) : (D[r] << (2 - sh));
  else v = __builtin_amdgcn_alignbit(D[r + 1], D[r], sh - 2);   // straddles two words; then sh >= 23
  return v & (((1u << C1) - 1u) << 2);
}

__device__ __forceinline__ float lds_float_at(const float *table, unsigned int byte_off) {
  return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(table) + byte_off);
}

// Shift a C1-word little-endian bit string right by 8*C1 bits (one block pair's worth of codes).
template <int C1>
__device__ __forceinline__ void shift_out_pair(unsigned int (&D)[C1]) {
  constexpr int wq = (8 * C1) >> 5, bq = (8 * C1) & 31;
#pragma unroll
  for (int r = 0; r < C1; ++r) {
    const unsigned int lo = (r + wq < C1) ? D[r + wq] : 0u;
    const unsigned int hi = (r + wq + 1 < C1) ? D[r + wq + 1] : 0u;
    D[r] = (bq == 0) ? lo : ((lo >> bq) | (hi << (32 - bq)));
  }
}

// The C1 record words of lane i of one octet: word r is the 32-bit word r*64 + i of the octet's 256*C1 bytes.
template <int C1>
__device__ __forceinline__ void load_record(const unsigned char *octet, int i, unsigned int (&D)[C1]) {
  const auto *g = reinterpret_cast<const __attribute__((address_space(1))) unsigned int *>(as_global(octet));
#pragma unroll
  for (int r = 0; r < C1; ++r) D[r] = __builtin_nontemporal_load(g + r * 64 + i);
}

template <int C1>
__device__ __forceinline__ void store_record(unsigned char *octet, int i, const unsigned int (&D)[C1]) {
  auto *g = (__attribute__((address_space(1))) unsigned int *)octet;
#pragma unroll
  for (int r = 0; r < C1; ++r) __builtin_nontemporal_store(D[r], g + r * 64 + i);
}

}  // namespace

// ------------------------------------------------------------------------------------------------ zero fill
__global__ void k_zero_u32(unsigned int *p, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = 0u;
}

// Bucket scope: the fit statistics of n (node, layer) pairs start from zero.
__device__ __forceinline__ void zero_stats(unsigned int *hist, double *stat, size_t pair) {
  unsigned long long *h = reinterpret_cast<unsigned long long *>(hist + pair * kHistBins);
  for (int j = threadIdx.x; j < kGridPoints; j += kThreads) h[j] = 0ull;
  if (threadIdx.x == 0) stat[pair] = 0.0;
}
__global__ void __launch_bounds__(kThreads) k_zero_stats(unsigned int *hist, double *stat) { zero_stats(hist, stat, blockIdx.x); }

// ------------------------------------------------------------------------------------------------ pass 1
// Sum of squares of one tile in fp64 (Sec. 2.2, L2 norm before the root), optionally with the histogram of the
// top 11 magnitude bits of every coordinate (the distribution estimate of Alg. 1 line 4).
template <bool HIST, int KIND>
__global__ void __launch_bounds__(kThreads) k_sumsq(Dev a) {
  __shared__ double red[kThreads];
  __shared__ unsigned int lh[HIST ? kHistBins : 1];
  // a workgroup takes up to kSuperTile consecutive tiles of one layer, so that the histogram is flushed to global
  // memory (integer atomics on a few hot addresses) once per run instead of once per tile; without a histogram most
  // launches take them one by one (see launch_sumsq_kind)
  int4 st;   // (layer, first chunk inside the layer, chunks)
  if (HIST || a.stiles != nullptr) {
    st = a.stiles[blockIdx.x];
  } else {
    const int2 tile = a.tiles[blockIdx.x];
    st = make_int4(tile.x, tile.y, 1, 0);
  }
  const int l = st.x;
  const int k = a.node0 + blockIdx.y;
  const int kr = k - a.row0;   // row of this node in the per-node scratch and pointer tables
  const LayerMeta m = a.meta[l];
  const float *__restrict__ v = a.grad[(size_t)kr * a.L + l];
  const int t = threadIdx.x;
  const int w = t >> 6, i = t & 63;
  if (HIST) {
    for (int b = t; b < kHistBins; b += kThreads) lh[b] = 0u;
    __syncthreads();
  }
  for (int cc = 0; cc < st.z; ++cc) {
    const int chunk = st.y + cc;
    const long long base = (long long)chunk * kChunkCoords + (long long)w * 16 * kBlockCoords + 4 * i;
    double acc = 0.0;
    unsigned int mb = 0u;   // KIND == kNormLinf: largest magnitude bit pattern
    if ((long long)(chunk + 1) * kChunkCoords <= m.d) {
      v4f q[16];
#pragma unroll
      for (int s = 0; s < 16; ++s)
        q[s] = __builtin_nontemporal_load(reinterpret_cast<const __attribute__((address_space(1))) v4f *>(
            as_global(v) + base + (long long)s * kBlockCoords));
#pragma unroll
      for (int s = 0; s < 16; ++s) {
        const float x[4] = {q[s].x, q[s].y, q[s].z, q[s].w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const double xd = (double)x[j];
          if (KIND == kNormL2) acc = __builtin_fma(xd, xd, acc);   // the product is exact in fp64, so this equals acc + xd*xd
          else if (KIND == kNormL1) acc = acc + fabs(xd);
          else mb = max(mb, f2u(x[j]) & 0x7FFFFFFFu);
          if (HIST) atomicAdd(&lh[(f2u(x[j]) & 0x7FFFFFFFu) >> 20], 1u);
        }
      }
    } else {
      for (int s = 0; s < 16; ++s) {
        const long long e = base + (long long)s * kBlockCoords;
        if (e >= m.d) break;
        float x[4];
        load4(v, e, m.d, x);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const double xd = (double)x[j];
          if (KIND == kNormL2) acc = __builtin_fma(xd, xd, acc);
          else if (KIND == kNormL1) acc = acc + fabs(xd);
          else mb = max(mb, f2u(x[j]) & 0x7FFFFFFFu);
          if (HIST && e + j < m.d) atomicAdd(&lh[(f2u(x[j]) & 0x7FFFFFFFu) >> 20], 1u);
        }
      }
    }
    const double total = (KIND == kNormLinf) ? block_max((double)magnitude_from_bits(mb), red) : block_tree(acc, red);
    if (t == 0) a.partial[(size_t)kr * a.G + m.first_chunk + chunk] = total;
  }
  if (HIST) {
    __syncthreads();
    unsigned int *gh = a.hist + ((size_t)k * a.L + l) * kHistBins;
    for (int b = t; b < kHistBins; b += kThreads) {
      const unsigned int c = lh[b];
      if (c) atomicAdd(&gh[b], c);
    }
  }
}

// Combine the tile sums of one (node, layer): slot j takes tiles j, j+256, ... in increasing order, then the
// halving tree; then norm = sqrt_floor(sum), inv = rcp_floor(norm).
__global__ void __launch_bounds__(kThreads) k_norm_finalize(Dev a) {
  __shared__ double red[kThreads];
  const int l = a.layers ? a.layers[blockIdx.x] : blockIdx.x;
  const int k = a.node0 + blockIdx.y - a.row0;   // row in the per-node scratch tables
  const LayerMeta m = a.meta[l];
  const double *p = a.partial + (size_t)k * a.G + m.first_chunk;
  double acc = 0.0;
  double s;
  if (a.kind == kNormLinf) {
    for (int c = threadIdx.x; c < m.nchunks; c += kThreads) acc = fmax(acc, p[c]);
    s = block_max(acc, red);
  } else {
    int c = threadIdx.x;
    for (; c + 7 * kThreads < m.nchunks; c += 8 * kThreads) {   // loads 8 at a time, sums in the slot's order
      double v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = p[c + q * kThreads];
#pragma unroll
      for (int q = 0; q < 8; ++q) acc = acc + v[q];
    }
    for (; c < m.nchunks; c += kThreads) acc = acc + p[c];
    s = block_tree(acc, red);
  }
  if (threadIdx.x == 0) {
    const bool finite = stat_finite(s, a.kind);
    float n, r;
    stat_scale(s, a.kind, n, r);
    const size_t idx = (size_t)k * a.L + l;
    a.sumsq[idx] = s;
    a.norm[idx] = n;
    a.inv[idx] = r;
    if (!finite) atomicOr(a.status, kStatusNonFinite);
    if (n > 0.0f && n < kFltMin) atomicOr(a.status, kStatusTinyNorm);
  }
}

// Whole-vector scope (the literal normalisation of Sec. 2.2 / Sec. 3.1): the L layer sums of a node are combined
// (slot j takes layers j, j+256, ... in increasing order, then the halving tree) and every layer of the node gets
// that sum, its root and the root's reciprocal.
__global__ void __launch_bounds__(kThreads) k_norm_vector(Dev a) {
  __shared__ double red[kThreads];
  __shared__ double tot[1];
  const int k = a.node0 + blockIdx.x - a.row0;   // row in the per-node scratch tables
  double acc = 0.0;
  double s;
  if (a.kind == kNormLinf) {
    for (int l = threadIdx.x; l < a.L; l += kThreads) acc = fmax(acc, a.sumsq[(size_t)k * a.L + l]);
    s = block_max(acc, red);
  } else {
    for (int l = threadIdx.x; l < a.L; l += kThreads) acc = acc + a.sumsq[(size_t)k * a.L + l];
    s = block_tree(acc, red);
  }
  if (threadIdx.x == 0) tot[0] = s;
  __syncthreads();
  const double total = tot[0];
  const bool finite = stat_finite(total, a.kind);
  float n, r;
  stat_scale(total, a.kind, n, r);
  for (int l = threadIdx.x; l < a.L; l += kThreads) {
    const size_t idx = (size_t)k * a.L + l;
    a.sumsq[idx] = total;
    a.norm[idx] = n;
    a.inv[idx] = r;
  }
  if (threadIdx.x == 0 && !finite) atomicOr(a.status, kStatusNonFinite);
  if (threadIdx.x == 0 && n > 0.0f && n < kFltMin) atomicOr(a.status, kStatusTinyNorm);
}

// ------------------------------------------------------------------------------------------------ pass 2
// Quantize + pack one tile (Sec. 3.1, Sec. 3.2) and accumulate the squared distance to the node's previous
// decoded message (the step-size term of eq. (general_stepsize)).
// Quantize the four coordinates a lane owns in one block (Sec. 3.1), append their codes to the record and add
// their squared distance to the previous decoded message (eq. (general_stepsize)).  jl0 = 0 or 4: position of
// the block inside its pair.
template <int C1, bool PREV, bool BINS>
__device__ __forceinline__ void quantize_block(const float (&x)[4], const unsigned int (&o)[4], int half, float inv,
                                               float norm, const QuantTables<C1, BINS> &T, bool walk,
                                               const float *tprev, unsigned int (&D)[C1], const unsigned int (&Dp)[C1],
                                               float &acc) {
  float u[4];
  float4 lv[4];   // {l_tau, 1/gap, l_tau+1, tau (BINS)}
  unsigned int tau[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    // min(|v| * inv, 1): the product is never negative or NaN for finite input, so the [0, 1] clamp of the
    // multiply instruction is the same thing
    u[j] = __builtin_amdgcn_fmed3f(fabsf(x[j]) * inv, 0.0f, 1.0f);
    if (BINS) lv[j] = bin_entry(T.bins, u[j]);
    else tau[j] = reinterpret_cast<const unsigned char *>(T.lut)[f2u(u[j]) >> 20];
  }
  if (!BINS) {
#pragma unroll
    for (int j = 0; j < 4; ++j) lv[j] = T.tab[tau[j]];
  }
  // A level inside a bin (walk; never the case for fitted levels, which sit on bin edges) makes some lanes walk on from the
  // entry of its lower edge.  At u = 1 the walk ends on the entry of the last level itself (xi = 0, never rounds up), which
  // yields the same code and value as tau = S-2 rounding up: there xi is 1 - 2^-23 at least, above every 16-bit draw.
  if (walk && __ballot((lv[0].z <= u[0]) | (lv[1].z <= u[1]) | (lv[2].z <= u[2]) | (lv[3].z <= u[3])) != 0ull) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (BINS) {
        while (lv[j].z <= u[j]) lv[j] = T.tab[f2u(lv[j].w) + 1u];
      } else {
        while (lv[j].z <= u[j]) { ++tau[j]; lv[j] = T.tab[tau[j]]; }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int jl = 4 * half + j;                       // position of the coordinate inside the pair
    const unsigned int w16 = half ? (o[j] >> 16) : (o[j] & 0xFFFFu);
    const float xi = (u[j] - lv[j].x) * lv[j].y;
    // (w16 + 0.5) < xi * 65536  <=>  w16 < xi * 65536 - 0.5 : the scaling by 2^16 is exact, and the subtraction
    // is exact whenever its result is not negative, so one fused operation decides the same.
    const bool up = (float)w16 < __builtin_fmaf(xi, 65536.0f, -0.5f);
    const unsigned int h = (BINS ? f2u(lv[j].w) : tau[j]) + (up ? 1u : 0u);
    // norm * l_h, the value the decoder will rebuild (the +inf of the last entry is never selected: there xi = 0)
    const float mag = norm * (up ? lv[j].z : lv[j].x);
    const float cur = __builtin_copysignf(mag, x[j]);
    insert_code<C1>(D, (h << 1) | (f2u(x[j]) >> 31), 24 + jl);
    float diff = cur;   // PREV == false: no node has a previous message (first round, or the rule of eq. (Alt))
    if (PREV) diff = cur - lds_float_at(tprev, extract_off<C1>(Dp, jl));   // table all zero for a node without one
    acc = __builtin_fmaf(diff, diff, acc);
  }
}

__device__ __forceinline__ void load_block_fast(const float *__restrict__ v, long long B, int i, float (&x)[4]) {
  const v4f q = __builtin_nontemporal_load(
      reinterpret_cast<const __attribute__((address_space(1))) v4f *>(as_global(v) + B * kBlockCoords + 4 * i));
  x[0] = q.x; x[1] = q.y; x[2] = q.z; x[3] = q.w;
}

// One octet (8 blocks = 2048 coordinates) of one (node, layer) for one wave: 4 block pairs, each with one
// generator call and 8 coordinates per lane.  The lane record is built as a shift register: every pair shifts it
// right by 8*C1 bits and writes its 8 codes into the top quarter, so that after four pairs pair 0 sits at bit 0;
// the previous message's record is consumed from the bottom the same way.  The pair loop is deliberately not
// unrolled: unrolled, the compiler interleaves the pairs and needs more than 256 registers.  The next pair's
// gradient values are requested before the current pair is processed.
// FAST: the whole octet lies inside the layer (no bounds checks anywhere).
template <int C1, bool FAST, bool PREV, bool BINS>
__device__ __forceinline__ void quantize_octet(const Dev &a, const LayerMeta &m, int l, int k, long long O,
                                               const float *__restrict__ v, unsigned char *body,
                                               const unsigned char *prevbody, float inv, float norm,
                                               const QuantTables<C1, BINS> &T, bool walk, const float *tprev, int i, float &acc) {
  const unsigned int k0 = (unsigned int)a.seed, k1 = (unsigned int)(a.seed >> 32);
  unsigned int D[C1], Dp[C1];
#pragma unroll
  for (int r = 0; r < C1; ++r) { D[r] = 0u; Dp[r] = 0u; }
  if (PREV && prevbody != nullptr) load_record<C1>(prevbody + O * 256 * C1, i, Dp);
  float xa[4] = {0.0f, 0.0f, 0.0f, 0.0f}, xb[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if (FAST) {
    load_block_fast(v, O * 8, i, xa);
    load_block_fast(v, O * 8 + 1, i, xb);
  }
#pragma unroll 1
  for (int pp = 0; pp < 4; ++pp) {
    const long long B0 = O * 8 + 2 * pp;   // block index inside the layer
    shift_out_pair<C1>(D);
    if (FAST || B0 < m.nblk) {
      float x0[4], x1[4];
      if (FAST) {
#pragma unroll
        for (int j = 0; j < 4; ++j) { x0[j] = xa[j]; x1[j] = xb[j]; }
        if (pp < 3) {
          load_block_fast(v, B0 + 2, i, xa);
          load_block_fast(v, B0 + 3, i, xb);
        }
      } else {
        load4(v, B0 * kBlockCoords + 4 * i, m.d, x0);
#pragma unroll
        for (int j = 0; j < 4; ++j) x1[j] = 0.0f;
        if (B0 + 1 < m.nblk) load4(v, (B0 + 1) * kBlockCoords + 4 * i, m.d, x1);
      }
      unsigned int o[4];
      philox4x32_10((unsigned int)((B0 >> 1) * 64 + i), (unsigned int)l, a.round, (unsigned int)k, k0, k1, o);
      quantize_block<C1, PREV, BINS>(x0, o, 0, inv, norm, T, walk, tprev, D, Dp, acc);
      // a block past the end of the layer is all padding: +0 inputs give code 0 and add nothing, as required
      quantize_block<C1, PREV, BINS>(x1, o, 1, inv, norm, T, walk, tprev, D, Dp, acc);
    }
    if (PREV) shift_out_pair<C1>(Dp);
  }
  store_record<C1>(body + O * 256 * C1, i, D);
}

template <int C1, bool PREV, bool BINS>
__device__ __forceinline__ void quantize_tile(const Dev &a, const LayerMeta &m, int l, int k, int chunk,
                                              const QuantTables<C1, BINS> &T, bool walk, const float *tprev, double *red) {
  const int t = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int i = t & 63;
  const int kr = k - a.row0;   // row of this node in the per-node scratch and pointer tables
  const float *__restrict__ v = a.grad[(size_t)kr * a.L + l];
  unsigned char *body = a.msg[kr] + m.body_off;
  const unsigned char *prevbody = (a.prev != nullptr && a.prev[kr] != nullptr) ? a.prev[kr] + m.body_off : nullptr;
  const float inv = a.inv[(size_t)kr * a.L + l];
  const float norm = a.norm[(size_t)kr * a.L + l];
  const long long noct = (m.nblk + 7) >> 3;
  float acc = 0.0f;   // this slot's squared differences: an fp32 fused multiply-add chain in increasing coordinate
  for (int oo = 0; oo < 2; ++oo) {
    const long long O = (long long)chunk * 8 + w * 2 + oo;   // octet index inside the layer
    if (O >= noct) break;
    if ((O + 1) * 2048 <= m.d)
      quantize_octet<C1, true, PREV, BINS>(a, m, l, k, O, v, body, prevbody, inv, norm, T, walk, tprev, i, acc);
    else
      quantize_octet<C1, false, PREV, BINS>(a, m, l, k, O, v, body, prevbody, inv, norm, T, walk, tprev, i, acc);
  }
  const double total = block_tree((double)acc, red);
  if (t == 0) a.dpartial[(size_t)kr * a.G + m.first_chunk + chunk] = total;
}

template <int C1, bool PREV, bool BINS>
__global__ void __launch_bounds__(kThreads) k_quantize(Dev a) {
  __shared__ QuantTables<C1, BINS> T;
  __shared__ float tprev[1 << C1];   // previous message's decode table indexed by code = sign | h << 1
  __shared__ double red[kThreads];
  const int2 tile = a.tiles[blockIdx.x];
  const int l = tile.x;
  const int k = a.node0 + blockIdx.y;
  const LayerMeta m = a.meta[l];
  if (m.planes != C1) return;   // layers of another code width are served by another instantiation
  const int t = threadIdx.x;
  const float *lev = a.lev + (size_t)m.type * kMaxPoints;
  const int kr = k - a.row0;
  const float norm = a.norm[(size_t)kr * a.L + l];
  const unsigned char *prevmsg = (a.prev != nullptr) ? a.prev[kr] : nullptr;
  // (without a previous message, 6 bits: the test of the flag would take the sixth wave of a SIMD, 82 registers instead of 80)
  const bool walk = (!BINS && !PREV && C1 == 6) || a.walk[m.type] != 0;
  if constexpr (BINS) {
    load_tables(a, m.type, m.S, walk, T.bins, T.tab);
  } else {
    const float *rg = a.rgap + (size_t)m.type * kMaxPoints;
    T.lut[t] = reinterpret_cast<const unsigned int *>(a.lut + (size_t)m.type * kLutSize)[t];
    if (t < m.S) T.tab[t] = make_float4(lev[t], rg[t], t + 1 < m.S ? lev[t + 1] : __builtin_inff(), 0.0f);
  }
  if (tile.y == 0) {   // message header of this layer: {norm, levels[S]} (Sec. 3.2: the norm in C_q = 32 bits)
    float *h = reinterpret_cast<float *>(a.msg[kr] + m.hdr_off);
    for (int j = t; j <= m.S; j += kThreads) h[j] = (j == 0) ? norm : lev[j - 1];
  }
  for (int c = t; c < (1 << m.planes); c += kThreads) {   // codes past S-1 decode as the last level
    float pv = 0.0f;
    if (prevmsg) {
      const float *hp = reinterpret_cast<const float *>(prevmsg + m.hdr_off);
      const float mag = hp[0] * hp[1 + min(c >> 1, m.S - 1)];
      pv = (c & 1) ? -mag : mag;
    }
    tprev[c] = pv;
  }
  __syncthreads();
  quantize_tile<C1, PREV, BINS>(a, m, l, k, tile.y, T, walk, tprev, red);
}

// ------------------------------------------------------------------------------------------------ octets in registers
// The quantizer for a wave that holds a whole octet (8 blocks = 2048 coordinates; 32 values a lane): the form with the
// fewest instructions.  Used where the pass is bound by the vector ALU or by latency and not, like k_quantize on large
// models, by the memory system's rate for its mix of loads and stores.

// Bits of word r of a record that hold the sign of a code (bit C1*jj of the little-endian string).
template <int C1>
constexpr unsigned int sign_bits(int r) {
  unsigned int m = 0u;
  for (int jj = 0; jj < 32; ++jj)
    if ((C1 * jj) >> 5 == r) m |= 1u << ((C1 * jj) & 31);
  return m;
}

// Append the codes of block bb (sign | index << 1, C1 bits each) to the record.  The codes of up to 32 bits are
// assembled from the last one down, two instructions each: index by shift-and-or, sign by a funnel shift out of the value.
template <int C1>
__device__ __forceinline__ void insert_block(unsigned int (&D)[C1], const unsigned int (&h)[4], const float *x, int bb) {
  constexpr int N = C1 <= 8 ? 4 : 2;   // codes per unit
#pragma unroll
  for (int q = 0; q < 4; q += N) {
    unsigned int F = 0u;
#pragma unroll
    for (int j = N - 1; j >= 0; --j) {
      F = (F << (C1 - 1)) | h[q + j];
      F = __builtin_amdgcn_alignbit(F, f2u(x[q + j]), 31);   // (F << 1) | sign
    }
    const int pos = C1 * (4 * bb + q), r = pos >> 5, sh = pos & 31;
    D[r] |= F << sh;
    if (sh + N * C1 > 32) D[r + 1] |= F >> (32 - sh);
  }
}

// Nothing of a block may be worked out before its turn or be left for later: with the blocks interleaved, or the
// differences computed where the sum needs them, the compiler keeps more than 200 registers.  The block's values pass
// through an empty statement that keeps its place.
__device__ __forceinline__ void pin_block(float *x) {
  asm volatile("" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]));
}

// One octet from registers.  x: the lane's 32 values in order (zeros past the end of the layer: they give code 0 and
// distance 0).  A block's four differences to the previous message (up to a sign that their square does not see) are
// given to done(bb, diff) as soon as they are known; it may put new values into the block's place in x.  pairs: how many
// of the four pairs of blocks to work on (the same for the wave).
// Tables: bins and tab as in load_tables; tprev[code] = value the previous message's code stands for.
// WALK: some level of the type lies inside a grid bin, so a lane may have to step on from the entry of its bin.
// Fitted levels sit on bin edges: then tau at the lower edge is tau.  (At u = 1 the walk ends on the entry of the last
// level, xi = 0; without it tau = S-2 and xi = 1 - 2^-23 at least, above every 16-bit draw: the same code.)
// sc: one set of scales (layer norms), or one per block (bucket norms; lane bb of the lane's row holds block bb's).
struct Scales { float inv, norm, pnorm; };

template <int C1, bool PREV, bool WALK, bool BUCKET, class Hist, class Done>
__device__ __forceinline__ void quantize_regs(float (&x)[32], unsigned int c0, unsigned int l, unsigned int round,
                                               unsigned int k, unsigned int k0, unsigned int k1, Scales sc,
                                               const float4 *bins, const float4 *tab, const float *tprev, unsigned int (&D)[C1],
                                               const unsigned int (&Dp)[C1], Hist &&hist, Done &&done, int pairs = 4) {
#pragma unroll
  for (int pp = 0; pp < 4; ++pp) {   // pairs of blocks: one generator call serves 8 coordinates of a lane
    if (pp >= pairs) break;
    asm volatile("" : "+v"(c0));
    unsigned int o[4];
    philox4x32_10(c0, l, round, k, k0, k1, o);
    c0 += 64u;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int bb = 2 * pp + half;
      float *xb = &x[4 * bb];
      pin_block(xb);
      const float bi = BUCKET ? u2f(row_value(f2u(sc.inv), bb)) : sc.inv;
      float u[4], mag[4];
      unsigned int h[4];
      float4 lv[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        // min(|v| * inv, 1): the product is never negative or NaN for finite input, so the [0, 1] clamp of the
        // multiply instruction is the same thing
        u[j] = __builtin_amdgcn_fmed3f(fabsf(xb[j]) * bi, 0.0f, 1.0f);
        lv[j] = bin_entry(bins, u[j]);
      }
      hist(xb, u, bb);
      if (WALK) {
        if (__ballot((lv[0].z <= u[0]) | (lv[1].z <= u[1]) | (lv[2].z <= u[2]) | (lv[3].z <= u[3])) != 0ull) {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            while (lv[j].z <= u[j]) lv[j] = tab[f2u(lv[j].w) + 1u];
        }
      }
      const float bn = BUCKET ? u2f(row_value(f2u(sc.norm), bb)) : sc.norm;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const unsigned int w16 = half ? (o[j] >> 16) : (o[j] & 0xFFFFu);
        const float xi = (u[j] - lv[j].x) * lv[j].y;
        // (w16 + 0.5) < xi * 65536  <=>  w16 < xi * 65536 - 0.5 : the scaling by 2^16 is exact, and the subtraction
        // is exact whenever its result is not negative, so one fused operation decides the same.
        const bool up = (float)w16 < __builtin_fmaf(xi, 65536.0f, -0.5f);
        h[j] = f2u(lv[j].w) + (up ? 1u : 0u);
        // norm * l_h, the value the decoder will rebuild (the last entry's upper neighbour is never selected: xi = 0)
        mag[j] = bn * (up ? lv[j].z : lv[j].x);
      }
      insert_block<C1>(D, h, xb, bb);
      if (PREV) {
        // +-mag - prev = +-(mag -+ prev): the value's sign, now in the record, is folded into the previous code's sign
        // (one operation per word), so that the table gives the previous value relative to it
        const float bp = BUCKET ? u2f(row_value(f2u(sc.pnorm), bb)) : 0.0f;
        unsigned int E[C1];
#pragma unroll
        for (int r = 0; r < C1; ++r) E[r] = __builtin_amdgcn_bitop3_b32(Dp[r], D[r], sign_bits<C1>(r), 0x78);   // a ^ (b & c)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float pl = lds_float_at(tprev, extract_off<C1>(E, 4 * bb + j));   // table all zero without a message
          mag[j] = mag[j] - (BUCKET ? bp * pl : pl);
        }
      }
      done(bb, mag);
#pragma unroll
      for (int r = 0; r < C1; ++r) asm volatile("" : "+v"(D[r]));
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

struct NoHist {
  __device__ __forceinline__ void operator()(const float *, const float (&)[4], int) const {}
};

// The lane's 32 coordinates of octet O of a layer of d entries (zeros past the end).  TOGETHER: the loads of a ragged last octet are all on
// their way at once too, where otherwise a block waits for the one before it; for k_quantize_held, where a group waits for its last
// tile.  (In the bucket quantizer it costs up to ten more spilled registers, in k_quantize_small five more registers.)
template <bool TOGETHER = false>
__device__ __forceinline__ void load_octet(const float *__restrict__ v, long long O, long long d, int i, float (&x)[32]) {
  const long long e0 = O * 2048 + 4 * i;
  if ((O + 1) * 2048 <= d) {
    v4f q[8];
#pragma unroll
    for (int bb = 0; bb < 8; ++bb)
      q[bb] = __builtin_nontemporal_load(reinterpret_cast<const __attribute__((address_space(1))) v4f *>(as_global(v) + e0 + bb * kBlockCoords));
#pragma unroll
    for (int bb = 0; bb < 8; ++bb) { x[4 * bb] = q[bb].x; x[4 * bb + 1] = q[bb].y; x[4 * bb + 2] = q[bb].z; x[4 * bb + 3] = q[bb].w; }
  } else if constexpr (TOGETHER) {
    // Lanes past the layer's end request its last whole quad again and drop it; the coordinates behind that quad are loaded by every lane.
    const auto *g = as_global(v) + O * 2048;
    const int n = (int)(d - O * 2048), whole = n & ~3;   // coordinates of the octet (1 at least), those in whole quads
    v4f q[8] = {};
    if (d >= 4) {
#pragma unroll
      for (int bb = 0; bb < 8; ++bb)
        q[bb] = __builtin_nontemporal_load(reinterpret_cast<const __attribute__((address_space(1))) v4f *>(g + min(bb * kBlockCoords + 4 * i, whole - 4)));
    }
    float p[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) p[j] = g[min(whole + j, n - 1)];
#pragma unroll
    for (int bb = 0; bb < 8; ++bb) {
      const int e = bb * kBlockCoords + 4 * i;
      const float y[4] = {q[bb].x, q[bb].y, q[bb].z, q[bb].w};
#pragma unroll
      for (int j = 0; j < 4; ++j) x[4 * bb + j] = e < whole ? y[j] : e + j < n && j < 3 ? p[j] : 0.0f;
    }
  } else {
#pragma unroll
    for (int bb = 0; bb < 8; ++bb) {
      float y[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      if (e0 + bb * kBlockCoords < d) load4(v, e0 + bb * kBlockCoords, d, y);
#pragma unroll
      for (int j = 0; j < 4; ++j) x[4 * bb + j] = y[j];
    }
  }
}

// Block bb of an octet that lies inside its layer; vo: the octet's first coordinate (the same for the wave).
__device__ __forceinline__ void load_block(const float *vo, int bb, unsigned int i, float *x) {
  const auto *g = reinterpret_cast<const __attribute__((address_space(1))) char *>(as_global(vo));
  const v4f q = __builtin_nontemporal_load(reinterpret_cast<const __attribute__((address_space(1))) v4f *>(g + (16u * i + 1024u * bb)));
  x[0] = q.x; x[1] = q.y; x[2] = q.z; x[3] = q.w;
}

// The tile sums of a run from its slots' fp32 chains: a wave takes every fourth tile, widens the 256 slots and combines
// them by the halving tree.
__device__ __forceinline__ void sum_tiles(const Dev &a, const float *chain, const LayerMeta &m, int4 st, int kr, int w, int i) {
  for (int cc = w; cc < st.z; cc += kThreads / 64) {
    const float *ch = chain + cc * kThreads;
    double r = ((double)ch[i] + (double)ch[i + 128]) + ((double)ch[i + 64] + (double)ch[i + 192]);
    r = lane_tree<true>(r);
    if (i == 0) a.dpartial[(size_t)kr * a.G + m.first_chunk + st.y + cc] = r;
  }
}

// ------------------------------------------------------------------------------------------------ small models
// Norms, quantization and the node's delta in one launch, for layer and vector scope.  A small model's pass is a chain of
// short kernels (norm pass, its combination, for vector scope a second combination, quantize, delta), each a few
// microseconds of launch and dependent loads around almost no work.  Here a workgroup of eight waves holds one tile in
// registers (an octet a wave), reduces its statistic, publishes it, waits for those of its group (the tiles of its layer;
// under vector scope all tiles of its node), combines them in the order that k_norm_finalize and k_norm_vector use, and
// quantizes what it holds: one read of the vectors.  The node's last workgroup to finish sums the squared distances.
//
// What the workgroups exchange are the values themselves: a statistic is stored as the complement of its bit pattern, so
// that the zeros left by the call before mean "not there yet" (no double that these sums produce has all bits set).  Every
// access to them is a device-scope atomic, so no cache keeps an old value; a value is all that a reader needs, so no fence
// goes with it.  Thread 0 of a workgroup makes both stores and then counts the workgroup in `finished`; who finds that all
// workgroups of a node have been counted waits until all their values are there, and clears: nothing but its zeros is written
// there after that, in this call.  (When each workgroup waited for its stores before it counted, 2 x 512 entries took 0.4 us more.)
// A group of one tile has nothing to exchange and waits for nothing; its tile's statistic is the layer's.
// Waiting ends: after `tries` looks a workgroup computes the missing statistics itself, one per turn, from the vectors, with
// the same operations in the same order, and keeps them to itself.
// Bound by latency: tile -> layer -> pointers -> values, the exchange, four pairs of blocks one after the other.  A quantize
// call, with the separate kernels / in one launch: 2 x 512 entries, K = 4 17.2 / 8.6 us, one tile, K = 1 17.0 / 10.1, 100 tiles,
// K = 5 33.7 / 21.1 (more where the rule stands, use_small).  Since then norms by straight-line code, trees in registers and no wait before
// the count have made rounds of up to 40 tiles 1.5 to 2.5 us faster.
__device__ __forceinline__ void publish(unsigned long long *p, double v) {
  __hip_atomic_store(p, ~(unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The tree's steps for one wave, from 256 slots in shared memory; the total is valid in lane 0.  SUM false: the maximum.
template <bool SUM>
__device__ __forceinline__ double wave_tree(const double *slot, int i) {
  double r = SUM ? (slot[i] + slot[i + 128]) + (slot[i + 64] + slot[i + 192])
                 : fmax(fmax(slot[i], slot[i + 128]), fmax(slot[i + 64], slot[i + 192]));
  return lane_tree<SUM>(r);
}

// A slot's statistic goes on through N more values.
template <int N>
__device__ __forceinline__ double add_terms(double acc, const float *x, int kind) {
  if (kind == kNormL2) {
#pragma unroll
    for (int j = 0; j < N; ++j) acc = __builtin_fma((double)x[j], (double)x[j], acc);
  } else if (kind == kNormL1) {
#pragma unroll
    for (int j = 0; j < N; ++j) acc = acc + fabs((double)x[j]);
  } else {
    unsigned int mb = 0u;
#pragma unroll
    for (int j = 0; j < N; ++j) mb = max(mb, f2u(x[j]) & 0x7FFFFFFFu);
    acc = fmax(acc, (double)magnitude_from_bits(mb));
  }
  return acc;
}

// The statistic of any tile, from memory: what its own workgroup publishes.  All threads of the workgroup call this, 256 at least, of which
// the first 256 work.
__device__ double tile_statistic(const float *__restrict__ v, long long d, int chunk, int kind, double *slot, int t) {
  __syncthreads();
  if (t < kThreads) {
    double acc = 0.0;
    const long long base = (long long)chunk * kChunkCoords + (long long)(t >> 6) * 16 * kBlockCoords + 4 * (t & 63);
#pragma unroll 1
    for (int s = 0; s < 16; ++s) {
      float x[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      if (base + s * kBlockCoords < d) load4(v, base + s * kBlockCoords, d, x);
      acc = add_terms<4>(acc, x, kind);
    }
    slot[t] = acc;
  }
  __syncthreads();
  return kind == kNormLinf ? wave_tree<false>(slot, t & 63) : wave_tree<true>(slot, t & 63);
}

template <int C1, bool PREV>
__global__ void __launch_bounds__(kSmallThreads) k_quantize_small(Dev a) {
  __shared__ float4 bins[kGridPoints];
  __shared__ float4 tab[1 << (C1 - 1)];
  __shared__ float tprev[1 << C1];      // previous message's decode table indexed by code = sign | h << 1
  __shared__ double slot[kThreads];
  __shared__ float chain[kThreads];
  __shared__ double group[kSmallGroup];   // the group's tile statistics
  __shared__ double layer[kSmallLayers];   // vector scope: the layers' sums
  __shared__ double total_stat[1];
  __shared__ float scale[2];
  __shared__ int missing[1];
  const int2 tile = a.tiles[blockIdx.x];
  const int l = tile.x;
  const int k = a.node0 + blockIdx.y;
  const LayerMeta m = a.meta[l];
  const int t = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int i = t & 63;
  const int kr = k - a.row0;   // row of this node in the per-node scratch and pointer tables
  const long long O = (long long)tile.y * 8 + w;   // octet index inside the layer
  const bool live = O < ((m.nblk + 7) >> 3);
  const unsigned char *prevmsg = (a.prev != nullptr) ? a.prev[kr] : nullptr;
  const float *__restrict__ v = a.grad[(size_t)kr * a.L + l];
  unsigned char *msg = a.msg[kr];
  float x[32];
  unsigned int D[C1], Dp[C1];
#pragma unroll
  for (int r = 0; r < C1; ++r) { D[r] = 0u; Dp[r] = 0u; }
  if (live) {
    load_octet(v, O, m.d, i, x);
    if (PREV && prevmsg != nullptr) load_record<C1>(prevmsg + m.body_off + O * 256 * C1, i, Dp);
  } else {
#pragma unroll
    for (int j = 0; j < 32; ++j) x[j] = 0.0f;
  }
  // tables that do not depend on the norm
  const float *lev = a.lev + (size_t)m.type * kMaxPoints;
  const int walk = a.walk[m.type];
  const float lj = t < m.S ? lev[t] : 0.0f;
  load_tables(a, m.type, m.S, walk, bins, tab);
  if (t < (1 << C1)) {   // codes past S-1 decode as the last level
    float pv = 0.0f;
    if (prevmsg) {
      const float *hp = reinterpret_cast<const float *>(prevmsg + m.hdr_off);
      const float mag = hp[0] * hp[1 + min(t >> 1, m.S - 1)];
      pv = (t & 1) ? -mag : mag;
    }
    tprev[t] = pv;
  }
  // the tile's statistic; a slot runs through the octets of a pair of waves, the odd one goes on from the even one's sum
  const int kind = a.kind;
  const int sl = (w >> 1) * 64 + i;
  double acc = 0.0;
  if (!(w & 1)) {
    if (live) acc = add_terms<32>(acc, x, kind);
    slot[sl] = acc;
  }
  __syncthreads();
  if ((w & 1) && live) slot[sl] = add_terms<32>(slot[sl], x, kind);
  __syncthreads();
  unsigned long long *stat = a.exch + (size_t)kr * exch_row(a.G);   // the node's statistics, then its squared distances
  unsigned long long *dist = stat + a.G;
  const bool vec = a.scope == kScopeVector;
  const int first = vec ? 0 : m.first_chunk, n = vec ? a.G : m.nchunks;   // the group
  const bool alone = !vec && n == 1;   // the tile's statistic is the layer's
  double own = 0.0;
  if (w == 0) {
    own = kind == kNormLinf ? wave_tree<false>(slot, i) : wave_tree<true>(slot, i);
    if (i == 0) publish(&stat[m.first_chunk + tile.y], own);   // (nobody else needs it where the tile is alone; see the end)
  }
  // the group's statistics; n <= kSmallGroup, one thread each
  bool have = t >= n;
  for (int tries = 0; !alone; ++tries) {
    if (!have && a.tries > 0) {
      const unsigned long long b = __hip_atomic_load(&stat[first + t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      have = b != 0ull;
      if (have) group[t] = __longlong_as_double((long long)~b);
    }
    if (__syncthreads_and(have)) break;
    if (tries < a.tries) continue;
    // some workgroup of the group is not running: its statistic is computed here, one tile per turn
    if (t == 0) missing[0] = 0x7FFFFFFF;
    __syncthreads();
    if (!have) atomicMin(&missing[0], t);
    __syncthreads();
    const int q = missing[0];
    const int2 mt = a.tiles[first + q];
    const double s = tile_statistic(a.grad[(size_t)kr * a.L + mt.x], a.meta[mt.x].d, mt.y, kind, slot, t);
    if (t == 0) group[q] = s;   // the same value that its own workgroup stores
    if (t == q) have = true;
  }
  // combine: slot j takes items j, j + 256, ... in increasing order, then the tree
  if (alone) {
  } else if (!vec) {
    if (t < kThreads) {
      double s = t < n ? group[t] : 0.0;
      if (t + kThreads < n) s = kind == kNormLinf ? fmax(s, group[t + kThreads]) : s + group[t + kThreads];
      slot[t] = s;
    }
  } else {
    for (int q = w; q < a.L; q += kSmallThreads / 64) {   // layer sums, a wave each
      const int f = a.meta[q].first_chunk, c = a.meta[q].nchunks;
      double p[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int j = i + 64 * r;
        p[r] = j < c ? group[f + j] : 0.0;
        if (j + kThreads < c) p[r] = kind == kNormLinf ? fmax(p[r], group[f + j + kThreads]) : p[r] + group[f + j + kThreads];
      }
      double s = kind == kNormLinf ? fmax(fmax(p[0], p[2]), fmax(p[1], p[3])) : (p[0] + p[2]) + (p[1] + p[3]);
      s = kind == kNormLinf ? lane_tree<false>(s) : lane_tree<true>(s);
      if (i == 0) {
        layer[q] = s;
        if (blockIdx.x == 0 && stat_finite(s, kind)) {   // a layer's own norm raises this flag under vector scope too
          const float nl = norm_of(s, kind);
          if (nl > 0.0f && nl < kFltMin) atomicOr(a.status, kStatusTinyNorm);
        }
      }
    }
    __syncthreads();
    if (t < kThreads) {
      double s = t < a.L ? layer[t] : 0.0;
      if (t + kThreads < a.L) s = kind == kNormLinf ? fmax(s, layer[t + kThreads]) : s + layer[t + kThreads];
      slot[t] = s;
    }
  }
  if (!alone) __syncthreads();
  if (w == 0) {
    const double s = alone ? own : kind == kNormLinf ? wave_tree<false>(slot, i) : wave_tree<true>(slot, i);
    if (i == 0) {
      const bool finite = stat_finite(s, kind);
      float nn, rr;
      stat_scale(s, kind, nn, rr);
      scale[0] = nn;
      scale[1] = rr;
      total_stat[0] = s;
      if (tile.y == 0) {   // one workgroup of the layer
        const size_t idx = (size_t)kr * a.L + l;
        a.sumsq[idx] = s;
        a.norm[idx] = nn;
        a.inv[idx] = rr;
        if (!finite) atomicOr(a.status, kStatusNonFinite);
        if (nn > 0.0f && nn < kFltMin) atomicOr(a.status, kStatusTinyNorm);
      }
    }
  }
  __syncthreads();
  const float norm = scale[0], inv = scale[1];
  if (tile.y == 0) {   // message header of this layer: {norm, levels[S]} (Sec. 3.2: the norm in C_q = 32 bits)
    float *h = reinterpret_cast<float *>(msg + m.hdr_off);
    if (t < m.S) h[1 + t] = lj;
    if (t == 0) h[0] = norm;
  }
  // layers without coordinates: statistics (under vector scope the node's) and header entries, a wave each
  for (int q = blockIdx.x * (kSmallThreads / 64) + w; q < a.n_empty; q += gridDim.x * (kSmallThreads / 64)) {
    const int e = a.empty_layers[q];
    const LayerMeta me = a.meta[e];
    const size_t idx = (size_t)kr * a.L + e;
    if (i == 0) {
      a.sumsq[idx] = vec ? total_stat[0] : 0.0;
      a.norm[idx] = vec ? norm : 0.0f;
      a.inv[idx] = vec ? inv : 0.0f;
    }
    float *h = reinterpret_cast<float *>(msg + me.hdr_off);
    for (int j = i; j <= me.S; j += 64) h[j] = (j == 0) ? (vec ? norm : 0.0f) : a.lev[(size_t)me.type * kMaxPoints + j - 1];
  }
  __syncthreads();
  float dacc = 0.0f;   // this slot's squared differences: an fp32 fused multiply-add chain in increasing coordinate
  if (live) {
    const unsigned int c0 = (unsigned int)(O * 256 + i);   // counter of the octet's first pair: 64 per 512 coordinates
    const unsigned int k0 = (unsigned int)a.seed, k1 = (unsigned int)(a.seed >> 32);
    const int pairs = (int)min(4ll, (m.nblk + 1 - O * 8) >> 1);   // the layer's; the others stay code 0, distance 0
    const auto keep = [&](int bb, float (&diff)[4]) {
      pin_block(diff);
#pragma unroll
      for (int j = 0; j < 4; ++j) x[4 * bb + j] = diff[j];
    };
    if (walk) quantize_regs<C1, PREV, true, false>(x, c0, l, a.round, k, k0, k1, Scales{inv, norm, 0.0f}, bins, tab, tprev, D, Dp, NoHist(), keep, pairs);
    else quantize_regs<C1, PREV, false, false>(x, c0, l, a.round, k, k0, k1, Scales{inv, norm, 0.0f}, bins, tab, tprev, D, Dp, NoHist(), keep, pairs);
    store_record<C1>(msg + m.body_off + O * 256 * C1, i, D);
    if (!(w & 1)) {
#pragma unroll
      for (int j = 0; j < 32; ++j) dacc = __builtin_fmaf(x[j], x[j], dacc);
    }
  }
  if (!(w & 1)) chain[sl] = dacc;
  __syncthreads();
  if (w & 1) {
    dacc = chain[sl];
    if (live) {
#pragma unroll
      for (int j = 0; j < 32; ++j) dacc = __builtin_fmaf(x[j], x[j], dacc);
    }
    slot[sl] = (double)dacc;
  }
  __syncthreads();
  if (w != 0) return;
  // the node's last workgroup sums the squared distances (slot j: tiles j, j + 256, ... of the node), in one wave
  const double total = wave_tree<true>(slot, i);
  unsigned int done = 0u;
  if (i == 0) {
    publish(&dist[m.first_chunk + tile.y], total);
    done = __hip_atomic_fetch_add(&a.finished[k], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (__builtin_amdgcn_readfirstlane(done) != (unsigned int)a.G - 1u) return;
  asm volatile("" : : : "memory");   // the distances are read after the count
  // Who has been counted has both stores on their way: they are waited for here, and nothing is stored to the area after that but
  // the zeros below.
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    double s = 0.0;
    for (int g = i + 64 * r; g < a.G; g += kThreads) {
      unsigned long long b, c;
      do {
        b = __hip_atomic_load(&dist[g], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        c = __hip_atomic_load(&stat[g], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } while (b == 0ull || c == 0ull);
      s = s + __longlong_as_double((long long)~b);
    }
    slot[i + 64 * r] = s;
  }
  const double delta = wave_tree<true>(slot, i);
  if (i == 0) {
    a.delta[k] = delta;
    __hip_atomic_store(&a.finished[k], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  for (int g = i; g < 2 * a.G; g += 64)   // for the next call; everybody has read them
    __hip_atomic_store(&stat[g], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------------------------------------------ held tiles
// Norms and quantization in one launch for models of any number of tiles, where their groups (a layer's tiles; under vector scope a
// node's) are small enough (held_tiles): one read of the vectors instead of two.  A workgroup of four waves holds its tile: of a wave's
// two octets the first in registers, the second in shared memory, where it goes without passing through registers.  With 32 KiB
// of data, tables of up to 7 KiB and 109 to 125 registers four workgroups fit a CU, 1024 tiles the device (three, 768 tiles, with
// 9-bit codes, whose tables are larger).  (k_quantize_small keeps a tile in the registers of eight waves: 512 tiles, all of a launch.)
// Bound by what a tile waits for: of the 20 us that a tile of a long launch is on the device (3112 tiles, groups of 389, 5-bit codes)
// it loads for 5.6, waits for its group for 10 and quantizes for 5.4; 1024 tiles pass in 17 us where groups are single tiles, in 21
// where they are 256 tiles, where the two reads of the separate kernels take 24.  So statistics and collecting go before
// quantizing (s_setprio: 11 k tiles 245 -> 232 us).  Tried without gain: every workgroup collects for itself (their looks
// slow the loads: 3112 tiles 78 -> 125 us); loads let in by a window of 256 to 640 tiles, or an octet at a time; 512 workgroups that
// stay, with the next tile's statistic out before the codes of this one (two workgroups a CU quantize at 2.8 us a tile instead of
// 2.1, and who collects holds up the rest: 106 us).
//
// Exchange: a tile's statistic and a layer's sum travel as the complement of their bit pattern, a pair {norm, inverse} as the
// complement of its two words: zero means "not there yet", and all of it is zero between calls (k_delta_finalize clears what the
// pass used).  The last tile of a layer collects the statistics of the layer's tiles and combines them (in the order of
// k_norm_finalize); under vector scope the last tile of the node then collects the sums of the layers (in the order of
// k_norm_vector).  The others look at one word.
// Workgroups start in the order of the table, so on an empty device all tiles of the oldest unfinished group are there or done.  Other
// streams' work may hold a part of the device, and then workgroups wait for such as cannot start before they end.  So every wait ends:
// who has looked `tries` times does the collecting work itself, and computes missing statistics from the vectors, one tile a turn and
// each workgroup another one.  Such a value is the one that its own workgroup stores, bit for bit, so it is published too, for all.
// (us beside a stream of elementwise additions; separate kernels / 1024 looks, the same tile in all workgroups, and as many looks again
// for every layer that is missing / 256, 64, 32 and 16 looks, shared out: one layer of 1024 tiles 101 / 1884 / 288, 153 to 165, 148, 147;
// a vector of 900 layers of a tile 104 / 461, one call 6973 / 112, 130 to 144, 152, 170; two layers of 400 tiles 91 / 71 / 71, 74, 71, 96; 8 vectors of
// 389 216 / 221 / 217, 218, 226, 271.  Alone 16 looks are too few: the vectors of 389 take 112 instead of 92.)
// All accesses to the area are device-scope atomics; nothing but the value that is read depends on them.
__device__ __forceinline__ unsigned long long look(const unsigned long long *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double published(unsigned long long b) { return __longlong_as_double((long long)~b); }
__device__ __forceinline__ void publish_scale(unsigned long long *p, float n, float r) {
  __hip_atomic_store(p, ~((unsigned long long)f2u(n) << 32 | f2u(r)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What the workgroups of one node share.
struct HeldNode {
  unsigned long long *stat;    // [G] statistics of the tiles
  unsigned long long *word;    // [G] at a layer's first tile: {norm, inverse} of the layer, under vector scope its sum
  unsigned long long *scale;   // vector scope: {norm, inverse} of the node
};

// Shared memory of the collecting work.
struct HeldShared {
  double *slot;     // [256]
  int *missing;
};

// The 256 slots of the workgroup by the tree; the total is valid in the first lane of the first wave.
__device__ __forceinline__ double held_tree(double v, int kind, double *slot) {
  __syncthreads();
  slot[threadIdx.x] = v;
  __syncthreads();
  if (threadIdx.x >= 64) return 0.0;
  return kind == kNormLinf ? wave_tree<false>(slot, threadIdx.x) : wave_tree<true>(slot, threadIdx.x);
}

constexpr int kNothing = 0x7FFFFFFF;

// One of the threads' indices (at least one has one; the others kNothing), which each workgroup takes in an order of its own, so that those
// that look for the same ones share them out.  (By rank, workgroup after workgroup: no faster beside other work, and 1 % slower without
// any, vectors of 389 79.4 instead of 78.1 us.)
__device__ __forceinline__ int pick_missing(int mine, int *missing) {
  const unsigned int order = ((unsigned int)mine * 0x9E3779B1u ^ blockIdx.x * 0x85EBCA77u) * 0xC2B2AE3Du;   // odd multipliers
  __syncthreads();
  if (threadIdx.x == 0) *missing = kNothing;
  __syncthreads();
  if (mine != kNothing) atomicMin(missing, (int)((order >> 1 & ~(unsigned int)(kThreads - 1)) | threadIdx.x));
  __syncthreads();
  const int first = *missing & (kThreads - 1);   // the thread
  __syncthreads();
  if (first == (int)threadIdx.x) *missing = mine;
  __syncthreads();
  return *missing;
}

// A store of the first thread is there for all threads of the workgroup that look after this.
__device__ __forceinline__ void settle() {
  asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
  __syncthreads();
}

// The statistic of layer m from those of its tiles; valid in thread 0.  All threads call this.  After `looks` looks the missing ones are
// computed here.
__device__ double collect_layer(const Dev &a, const LayerMeta &m, const float *v, const HeldNode &hn, const HeldShared &hs, int looks) {
  const int t = threadIdx.x, kind = a.kind;
  const unsigned long long *stat = hn.stat + m.first_chunk;
  constexpr int N = kHeldSlots / kThreads;
  unsigned long long got[N];
  for (int tries = 0;; ++tries) {
    int none = kNothing;   // the first of this thread's tiles whose statistic is not there
#pragma unroll
    for (int q = N - 1; q >= 0; --q) {
      const int j = t + q * kThreads;
      got[q] = 0ull;
      if (j < m.nchunks) {
        got[q] = look(&stat[j]);
        if (got[q] == 0ull) none = j;
      }
    }
    if (__syncthreads_and(none == kNothing)) break;
    if (tries < looks) continue;
    const int chunk = pick_missing(none, hs.missing);
    const double s = tile_statistic(v, m.d, chunk, kind, hs.slot, t);
    if (t == 0) publish(&hn.stat[m.first_chunk + chunk], s);
    settle();
  }
  double s = t < m.nchunks ? published(got[0]) : 0.0;
#pragma unroll
  for (int q = 1; q < N; ++q)
    if (t + q * kThreads < m.nchunks) s = kind == kNormLinf ? fmax(s, published(got[q])) : s + published(got[q]);
  return held_tree(s, kind, hs.slot);
}

// Vector scope: the node's statistic from those of its layers; valid in thread 0.  All threads call this.
__device__ double collect_node(const Dev &a, int kr, const HeldNode &hn, const HeldShared &hs, int looks) {
  const int t = threadIdx.x, kind = a.kind;
  double s = 0.0;
  for (int tries = 0;; ++tries) {
    int none = kNothing;
    s = 0.0;
    for (int q = t; q < a.L; q += kThreads) {
      double v = 0.0;
      if (a.meta[q].nchunks != 0) {
        const unsigned long long b = look(&hn.word[a.meta[q].first_chunk]);
        if (b == 0ull) none = min(none, q);
        else v = published(b);
      }
      s = kind == kNormLinf ? fmax(s, v) : s + v;
    }
    if (__syncthreads_and(none == kNothing)) break;
    if (tries < looks) continue;
    const int q = pick_missing(none, hs.missing);
    const LayerMeta m = a.meta[q];
    const double sum = collect_layer(a, m, a.grad[(size_t)kr * a.L + q], hn, hs, 0);
    if (t == 0) publish(&hn.word[m.first_chunk], sum);
    settle();
  }
  return held_tree(s, kind, hs.slot);
}

template <int C1, bool PREV>
__global__ void __launch_bounds__(kThreads, C1 == 9 ? 3 : 4) k_quantize_held(Dev a) {
  typedef __attribute__((address_space(3))) void *lds_ptr;
  constexpr int kTabBytes = 16 << (C1 - 1), kPrevBytes = PREV ? 4 << C1 : 0;
  __shared__ v4f hold[kThreads / 64][8][64];   // the waves' second octets
  __shared__ float4 bins[kGridPoints];
  // the slots of the sums, and between the norm and the distances the tables that would not fit beside them
  __shared__ __attribute__((aligned(16))) unsigned char area[kTabBytes + kPrevBytes > 8 * kThreads ? kTabBytes + kPrevBytes : 8 * kThreads];
  __shared__ float scale[2];
  __shared__ int flag[1];
  double *slot = reinterpret_cast<double *>(area);
  float4 *tab = reinterpret_cast<float4 *>(area);
  float *tprev = reinterpret_cast<float *>(area + kTabBytes);
  __builtin_amdgcn_s_setprio(3);
  const int2 tile = a.tiles[blockIdx.x];
  const int l = tile.x;
  const int k = a.node0 + blockIdx.y;
  const LayerMeta m = a.meta[l];
  if (m.planes != C1) return;   // layers of another code width are served by another instantiation
  const int t = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int i = t & 63;
  const int kr = k - a.row0;   // row of this node in the per-node scratch and pointer tables
  const long long noct = (m.nblk + 7) >> 3, O0 = (long long)tile.y * 8 + 2 * w;   // octets inside the layer
  const float *__restrict__ v = a.grad[(size_t)kr * a.L + l];
  unsigned char *msg = a.msg[kr];
  const unsigned char *prevmsg = (PREV && a.prev != nullptr) ? a.prev[kr] : nullptr;
  float x[32];
  if (O0 < noct) {
    load_octet<true>(v, O0, m.d, i, x);
  } else {
#pragma unroll
    for (int j = 0; j < 32; ++j) x[j] = 0.0f;
  }
  if (O0 + 1 < noct) {
    if ((O0 + 2) * 2048 <= m.d) {
      const auto *src = as_global(v) + (O0 + 1) * 2048 + 4 * i;
#pragma unroll
      for (int bb = 0; bb < 8; ++bb)   // 16 bytes a lane, nontemporal
        __builtin_amdgcn_global_load_lds(reinterpret_cast<const __attribute__((address_space(1))) void *>(src + bb * kBlockCoords),
                                         (lds_ptr)(void *)&hold[w][bb][0], 16, 0, 2);
    } else {
      // The layer's ragged last octet, its loads together too (when they were one after the other the group waited for this tile: 16
      // nodes of one layer of 350 tiles less 3 entries 161 -> 142 us, separate kernels 148; 12 k layers of a tile less 3 entries 233 -> 201).
      const auto *src = as_global(v) + (O0 + 1) * 2048;
      const int n = (int)(m.d - (O0 + 1) * 2048);
#pragma unroll
      for (int bb = 0; bb < 8; ++bb) {
        const int e = bb * kBlockCoords + 4 * i;
        if (e + 4 <= n) {
          __builtin_amdgcn_global_load_lds(reinterpret_cast<const __attribute__((address_space(1))) void *>(src + e),
                                           (lds_ptr)(void *)&hold[w][bb][0], 16, 0, 2);
        } else {
          v4f q = {0.0f, 0.0f, 0.0f, 0.0f};
          if (e < n) {
            q.x = src[e];
            if (e + 1 < n) q.y = src[e + 1];
            if (e + 2 < n) q.z = src[e + 2];
          }
          hold[w][bb][i] = q;
        }
      }
    }
  }
  // tables that do not depend on the norm: requested now, the ones that share the area of the slots stored later
  const float *lev = a.lev + (size_t)m.type * kMaxPoints, *rg = a.rgap + (size_t)m.type * kMaxPoints;
  const int walk = a.walk[m.type];
  const float lj = t < m.S ? lev[t] : 0.0f, ln = t + 1 < m.S ? lev[t + 1] : __builtin_inff(), rj = t < m.S ? rg[t] : 0.0f;
  float pl[2] = {0.0f, 0.0f};
  if (PREV && prevmsg) {
    const float *hp = reinterpret_cast<const float *>(prevmsg + m.hdr_off);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int c = t + q * kThreads;   // codes past S-1 decode as the last level
      if (c < (1 << C1)) {
        const float mag = hp[0] * hp[1 + min(c >> 1, m.S - 1)];
        pl[q] = (c & 1) ? -mag : mag;
      }
    }
  }
  {
    const v4f *src = reinterpret_cast<const v4f *>(a.bins + (size_t)m.type * kGridPoints);
    *reinterpret_cast<v4f *>(&bins[t]) = src[t];
    if (t == 0) *reinterpret_cast<v4f *>(&bins[kThreads]) = src[kThreads];
  }
  // the tile's statistic: a slot runs through the wave's two octets
  const int kind = a.kind;
  double own = 0.0;
  if (O0 < noct) own = add_terms<32>(own, x, kind);
  if (O0 + 1 < noct) {
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
#pragma unroll
    for (int bb = 0; bb < 8; ++bb) {
      const v4f q = hold[w][bb][i];
      const float y[4] = {q.x, q.y, q.z, q.w};
      own = add_terms<4>(own, y, kind);
    }
  }
  const HeldShared hs = {slot, flag};
  const bool vec = a.scope == kScopeVector;
  unsigned long long *row = a.exch + (size_t)kr * exch_row(a.G);
  const HeldNode hn = {row, row + a.G, row + 2 * (size_t)a.G};
  unsigned long long *word = vec ? hn.scale : &hn.word[m.first_chunk];   // of the group
  double s = held_tree(own, kind, slot);   // valid in thread 0, as all totals here
  if (m.nchunks > 1 && t == 0) publish(&hn.stat[m.first_chunk + tile.y], s);
  // collectors: the last tile of a layer, and under vector scope that of the last layer with coordinates
  bool collects = tile.y == m.nchunks - 1;
  if (collects) {
    if (m.nchunks > 1) s = collect_layer(a, m, v, hn, hs, a.tries);
    if (vec) {
      if (t == 0) {
        publish(&hn.word[m.first_chunk], s);
        float n, r;   // a layer's own norm raises this flag under vector scope too
        stat_scale(s, kind, n, r);
        if (n > 0.0f && n < kFltMin) atomicOr(a.status, kStatusTinyNorm);
      }
      collects = m.first_chunk + m.nchunks == a.G;
      if (collects) {
        settle();
        s = collect_node(a, kr, hn, hs, a.tries);
      }
    }
  }
  if (!collects) {
    if (t == 0) {
      unsigned long long b = 0ull;
      for (int tries = 0; tries < a.tries && b == 0ull; ++tries) {
        if (tries) __builtin_amdgcn_s_sleep(16);
        b = look(word);
      }
      scale[0] = u2f((unsigned int)(~b >> 32));
      scale[1] = u2f((unsigned int)~b);
      flag[0] = b != 0ull;
    }
    __syncthreads();
    if (flag[0] == 0) {   // no answer: the collecting work is done here as well, and its result is the group's
      s = vec ? collect_node(a, kr, hn, hs, 0) : collect_layer(a, m, v, hn, hs, 0);
      if (t == 0) {
        float n, r;
        stat_scale(s, kind, n, r);
        scale[0] = n;
        scale[1] = r;
        publish_scale(word, n, r);
      }
    }
  } else {
    if (t == 0) {
      float n, r;
      stat_scale(s, kind, n, r);
      scale[0] = n;
      scale[1] = r;
      if (vec || m.nchunks > 1) publish_scale(word, n, r);
      if (!stat_finite(s, kind)) atomicOr(a.status, kStatusNonFinite);
      if (n > 0.0f && n < kFltMin) atomicOr(a.status, kStatusTinyNorm);
      if (!vec) {
        const size_t idx = (size_t)kr * a.L + l;
        a.sumsq[idx] = s;
        a.norm[idx] = n;
        a.inv[idx] = r;
      } else {
        slot[0] = s;
      }
    }
    if (vec) {   // every layer of the node has its statistic, norm and inverse
      __syncthreads();
      for (int q = t; q < a.L; q += kThreads) {
        const size_t idx = (size_t)kr * a.L + q;
        a.sumsq[idx] = slot[0];
        a.norm[idx] = scale[0];
        a.inv[idx] = scale[1];
      }
    }
  }
  __syncthreads();   // scale is there, the slots are free
  const float norm = scale[0], inv = scale[1];
  if (t < m.S) tab[t] = make_float4(lj, rj, ln, u2f((unsigned int)t));   // the walk's entries, see load_tables
  if (PREV) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
      if (t + q * kThreads < (1 << C1)) tprev[t + q * kThreads] = pl[q];
  }
  if (tile.y == 0) {   // message header of this layer: {norm, levels[S]} (Sec. 3.2: the norm in C_q = 32 bits)
    float *h = reinterpret_cast<float *>(msg + m.hdr_off);
    if (t < m.S) h[1 + t] = lj;
    if (t == 0) h[0] = norm;
  }
  if (!vec) {   // layers without coordinates: their header entries are written by k_delta_finalize
    for (int q = blockIdx.x * kThreads + t; q < a.n_empty; q += gridDim.x * kThreads) {
      const size_t idx = (size_t)kr * a.L + a.empty_layers[q];
      a.sumsq[idx] = 0.0;
      a.norm[idx] = 0.0f;
      a.inv[idx] = 0.0f;
    }
  }
  __syncthreads();
  __builtin_amdgcn_s_setprio(0);
  float dacc = 0.0f;   // this slot's squared differences: an fp32 fused multiply-add chain in increasing coordinate
  const unsigned int k0 = (unsigned int)a.seed, k1 = (unsigned int)(a.seed >> 32);
  unsigned int Dp[C1];
#pragma unroll
  for (int r = 0; r < C1; ++r) Dp[r] = 0u;
#pragma unroll 1
  for (int oo = 0; oo < 2; ++oo) {
    const long long O = O0 + oo;
    if (O >= noct) break;
    unsigned int D[C1];
#pragma unroll
    for (int r = 0; r < C1; ++r) D[r] = 0u;
    if (PREV && prevmsg != nullptr) load_record<C1>(prevmsg + m.body_off + O * 256 * C1, i, Dp);
    const bool more = oo == 0 && O + 1 < noct;
    const auto done = [&](int bb, float (&diff)[4]) {
#pragma unroll
      for (int j = 0; j < 4; ++j) dacc = __builtin_fmaf(diff[j], diff[j], dacc);
      asm volatile("" : "+v"(dacc));
      if (more) {
        const v4f q = hold[w][bb][i];
        x[4 * bb] = q.x; x[4 * bb + 1] = q.y; x[4 * bb + 2] = q.z; x[4 * bb + 3] = q.w;
      }
    };
    const unsigned int c0 = (unsigned int)(O * 256 + i);   // counter of the octet's first pair: 64 per 512 coordinates
    const int pairs = (int)min(4ll, (m.nblk + 1 - O * 8) >> 1);   // the layer's; the others stay code 0, distance 0
    const Scales sc = {inv, norm, 0.0f};
    if (walk) quantize_regs<C1, PREV, true, false>(x, c0, l, a.round, k, k0, k1, sc, bins, tab, tprev, D, Dp, NoHist(), done, pairs);
    else quantize_regs<C1, PREV, false, false>(x, c0, l, a.round, k, k0, k1, sc, bins, tab, tprev, D, Dp, NoHist(), done, pairs);
    store_record<C1>(msg + m.body_off + O * 256 * C1, i, D);
  }
  __syncthreads();   // the tables are done with
  slot[t] = (double)dacc;
  __syncthreads();
  if (w != 0) return;
  const double total = wave_tree<true>(slot, i);
  if (i == 0) a.dpartial[(size_t)kr * a.G + m.first_chunk + tile.y] = total;
}

// ------------------------------------------------------------------------------------------------ bucket scope
// One norm per 128 consecutive coordinates (the experiments' setting, Sec. 7): the norms are computed by the wave
// that quantizes, from the registers that it then quantizes from, so the gradient is read once.
//
// Per-wave shared memory of the bucket-scope quantizer.
constexpr double kBucketRescueBelow = 7.888609052210118e-31;   // 2^-100

struct __attribute__((aligned(8))) BucketWave {
  // the lane's sum of its 4 squares (fp32 fused chain in coordinate order) for block bb, lane i, at index
  // 72*bb + i + i/8: one word of padding after every 8, so that the transposed read below (lane L reads the 8
  // consecutive entries 8L .. 8L+7, i.e. a stride of 9 words between lanes) spreads over all banks
  float psum[8 * 72];
  float norm[16];       // [8*half + block] of the current octet
  float inv[16];
  unsigned int wfix[16];   // fit statistics: integer weight of the bucket (0: gathers nothing)
};

// The sums of squares of the 16 buckets of one octet once more with exact fp64 squares (a lane's chain
// acc = fma((double)x, (double)x, acc), then the same tree): the path taken when a single-precision result is below
// 2^-100 or not finite.  The 8 x 64 lane sums go through the wave's shared memory four blocks at a time (as doubles they
// fill the area the single-precision pass used).  Every lane of the wave must call this; the result is the sum of
// the lane's own bucket.
__device__ __forceinline__ double bucket_sums_exact(const float (&x)[32], float *psum, int i) {
  double *dsum = reinterpret_cast<double *>(psum);
  const int q = i >> 2, r = i & 3;
  const int bb = q >> 1, hf = q & 1;
  double s = 0.0;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int b4 = 0; b4 < 4; ++b4) {
      double acc = 0.0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const double xd = (double)x[16 * half + 4 * b4 + j];
        acc = __builtin_fma(xd, xd, acc);
      }
      dsum[72 * b4 + i + (i >> 3)] = acc;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if ((bb >> 2) == half) {
      const double *p = &dsum[72 * (bb & 3) + 36 * hf + 9 * r];
      s = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
    }
  }
  s = s + quad_swap<0xB1>(s);
  s = s + quad_swap<0x4E>(s);
  return s;
}

// The fit's weighted grid histogram of a run, in shared memory: 32-bit adds, the weights (at most 2^30) cut into their
// low kHistLowBits bits and the rest, which is zero for most buckets of heavy-tailed vectors and then not added at all.
// A run has at most 4 * 16384 coordinates and a copy takes every kHistCopies-th lane's, so no cell overflows:
// 2^16 / 16 * (2^19 - 1) < 2^32 and 2^16 / 4 * 2^11 < 2^32.  Copies of a bin lie side by side: lanes that meet in a bin
// collide rarely.  An add of 64 lanes keeps the CU's shared memory busy for 6 cycles here, against 13 for the 64-bit adds
// of four copies that this replaces (10 for eight copies).
constexpr int kHistLowBits = 19;
constexpr int kHistCopies = 16, kHistHighCopies = 4;   // powers of two
constexpr int kHistFewCopies = 2;    // of the low cells, where a run is a single octet: 2^11 / 2 * (2^19 - 1) < 2^32
static_assert((long long)kQuantRun * kChunkCoords / kHistCopies * ((1 << kHistLowBits) - 1) < (1ll << 32), "low cells");

// Statistics of the 16 buckets of one octet (the lane's 32 values in x) -> norm, inv (shared memory) and the octet's
// norm trailer.
// A lane's four squares are an fp32 fused chain; lane L then finishes bucket q = L/4 (block q/2, half q%2): it adds 8
// consecutive lane sums, widened to fp64, by the in-order binary tree, then the four lanes of the quad combine
// (neighbour, then pair), which continues the same tree.
// A single-precision result below 2^-100 (squares may have vanished) or not finite (squares may have overflowed) is
// replaced by the exact one (bucket_sums_exact).
// ex: weight scale of the layer's type for the fit statistics (kTypeSkip: none); best: running maximum of the bit
// patterns of the lane's bucket sums.  Returns whether some weight of the octet has bits above kHistLowBits.
// sc, wfix: norm, inv and weight of the half's buckets, as quantize_regs takes them.
template <int KIND>
__device__ __forceinline__ bool bucket_norms(const Dev &a, const float (&x)[32], float *trailer, BucketWave &bw, int i, int ex,
                                             unsigned long long &best, Scales &sc, unsigned int &wfix) {
#pragma unroll
  for (int bb = 0; bb < 8; ++bb) {
    float acc = 0.0f;
    if (KIND == kNormL2) {
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = __builtin_fmaf(x[4 * bb + j], x[4 * bb + j], acc);
    } else if (KIND == kNormL1) {
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = acc + fabsf(x[4 * bb + j]);
    } else {
      unsigned int mb = 0u;
#pragma unroll
      for (int j = 0; j < 4; ++j) mb = max(mb, f2u(x[4 * bb + j]) & 0x7FFFFFFFu);
      acc = magnitude_from_bits(mb);
    }
    bw.psum[72 * bb + i + (i >> 3)] = acc;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const int q = i >> 2, r = i & 3;
  const int bb = q >> 1, hf = q & 1;
  const float *p = &bw.psum[72 * bb + 36 * hf + 9 * r];   // lanes 32*hf + 8*r .. +7 of block bb in the padded layout
  double s;
  if (KIND == kNormLinf) {
    const float mx = fmaxf(fmaxf(fmaxf(p[0], p[1]), fmaxf(p[2], p[3])), fmaxf(fmaxf(p[4], p[5]), fmaxf(p[6], p[7])));
    s = (double)mx;
    s = fmax(s, quad_swap<0xB1>(s));
    s = fmax(s, quad_swap<0x4E>(s));
  } else {
    s = (((double)p[0] + (double)p[1]) + ((double)p[2] + (double)p[3])) +
        (((double)p[4] + (double)p[5]) + ((double)p[6] + (double)p[7]));
    s = s + quad_swap<0xB1>(s);
    s = s + quad_swap<0x4E>(s);
  }
  if (KIND == kNormL2) {
    const bool redo = !(s >= kBucketRescueBelow) || !(s <= 1.7976931348623157e308);
    if (__ballot(redo) != 0ull) {   // rare: all lanes of the wave take the exact path together
      const double exact = bucket_sums_exact(x, bw.psum, i);
      if (redo) s = exact;
    }
  }
  const bool finite = stat_finite(s, KIND);
  float n = 0.0f, rinv = 0.0f;
  if (finite) {
    if (KIND == kNormL2) {
      norm_and_inverse(s, n, rinv);
    } else {
      n = __double2float_rn(s);
      rinv = inverse_of(n);
    }
  }
  if (!finite) atomicOr(a.status, kStatusNonFinite);
  if (n > 0.0f && n < kFltMin) atomicOr(a.status, kStatusTinyNorm);
  {
    const unsigned long long bits = finite ? (unsigned long long)__double_as_longlong(s) : 0x7FF0000000000000ull;
    best = bits > best ? bits : best;
  }
  unsigned int wf = 0u;
  if (ex != kTypeSkip && finite && rinv != 0.0f)
    wf = (unsigned int)fmin(floor(ldexp(weight_of(s, KIND), 23 - ex)), 1073741824.0);
  if (r == 0) {
    bw.norm[8 * hf + bb] = n;
    bw.inv[8 * hf + bb] = rinv;
    bw.wfix[8 * hf + bb] = wf;
    trailer[8 * hf + bb] = n;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const int at = 8 * (i >> 5) + (i & 7);
  sc.norm = bw.norm[at];
  sc.inv = bw.inv[at];
  wfix = bw.wfix[at];
  return __ballot(wf >> kHistLowBits) != 0ull;
}

struct BucketHist {
  unsigned int wfix;    // weights of the eight buckets of the lane's half: lane bb of a row holds block bb's
  unsigned int *lo, *hi;      // the lane's copies
  bool on;      // statistics are gathered (this and the next two: the same for the whole wave)
  bool high;    // some weight of the octet has bits above kHistLowBits
  bool plain;   // no such weight, and no coordinate of the octet is in raw magnitude bin 0
  __device__ __forceinline__ void operator()(const float *x, const float (&u)[4], int bb) const {
    if (!on) return;
    const unsigned int w = row_value(wfix, bb);
    if (plain) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        atomicAdd(&lo[__builtin_elementwise_sub_sat(f2u(u[j]) >> 20, (unsigned int)kGridBase) * kHistCopies], w);
      return;
    }
    if (w == 0u) return;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (fabsf(x[j]) < 0x1p-129f) continue;   // raw magnitude bin 0; also the +0 padding past the layer's end
      // u <= 1, so its bin never exceeds the last grid index: only the lower clamp is needed (saturating subtract)
      const unsigned int g = __builtin_elementwise_sub_sat(f2u(u[j]) >> 20, (unsigned int)kGridBase);
      atomicAdd(&lo[g * kHistCopies], w & ((1u << kHistLowBits) - 1u));
      if (high) atomicAdd(&hi[g * kHistHighCopies], w >> kHistLowBits);
    }
  }
};

// Bound by the vector ALU (35.7 instructions per coordinate) together with what its waves wait for: shared memory is busy 45 % of
// the time, and a wave spends 44 % of its own waiting for a value.  Up to 64 levels (codes of 7 bits) four waves a SIMD: 128
// registers and 37.9 to 39.4 KiB of shared memory a workgroup, of which the table by grid bin is 4 KiB; so a run has at most 4 tiles.
// With the previous message 6 registers are spilled at 32 levels and 8 at 64, and four waves are still the better choice: 64 levels,
// K = 8, statistics gathered, us with four waves / with three and nothing spilled: 100 tiles a node 32.6 / 38.4, 387 77.3 / 82.6, 1250
// 210 / 228, 9300 1404 / 1454; only launches of up to 400 tiles lose (20 tiles 20.1 / 19.4, 50 25.1 / 23.1).  Wider codes have larger
// tables, three workgroups a CU, and the compiler takes 141 to 157 registers.  What made it 151 M coordinates, K = 8, 8 levels 1345 -> 1252 us and 3112 tiles, 16 levels 87 -> 79 us: one 128-bit
// table read per coordinate instead of two reads one after the other; the buckets' scales in registers, broadcast along the rows
// of 16 lanes, instead of four reads per block; root and reciprocal with one exact test each; the previous record requested at
// the start of its octet instead of one ahead (128 registers without spills).  Entries requested a block ahead need 20 registers
// more: 2144 us.
// Layers of a block or two have a form of one pair of blocks, and runs of one octet fewer copies of the histogram.
template <int C1, bool PREV, int KIND>
__global__ void __launch_bounds__(kThreads, 4) k_quantize_b(Dev a) {
  __shared__ float4 bins[kGridPoints];
  __shared__ float4 tab[1 << (C1 - 1)];
  __shared__ float tprev[1 << C1];   // +-level of the previous message, indexed by code = sign | h << 1
  __shared__ float chain[kQuantRun * kThreads];   // the slots' squared distances, tile by tile
  __shared__ BucketWave bws[kThreads / 64];
  __shared__ unsigned int lo[kGridPoints * kHistCopies], hi[kGridPoints * kHistHighCopies];
  __shared__ unsigned long long wmax[kThreads / 64];
  constexpr long long OS = 256 * C1 + 64;   // bytes per octet: codes, then the 16 bucket norms
  // a workgroup takes a run of consecutive tiles of one layer: the tables are set up and the statistics flushed once
  // per run
  const int4 st = a.stiles[blockIdx.x];
  const int l = st.x;
  const int k = a.node0 + blockIdx.y;
  const LayerMeta m = a.meta[l];
  if (m.planes != C1) return;
  const int t = threadIdx.x;
  const float *lev = a.lev + (size_t)m.type * kMaxPoints;
  const int kr = k - a.row0;   // row in the pointer tables and in the per-tile scratch; the fit statistics use k
  const unsigned char *prevmsg = (a.prev != nullptr) ? a.prev[kr] : nullptr;
  const int ex = a.type_exp[m.type];
  const int walk = a.walk[m.type];
  load_tables(a, m.type, m.S, 1, bins, tab);   // the form for one pair of blocks walks, whatever the type
  if (st.y == 0) {   // header of this layer: the norm entry is unused under bucket scope
    float *h = reinterpret_cast<float *>(a.msg[kr] + m.hdr_off);
    for (int j = t; j <= m.S; j += kThreads) h[j] = (j == 0) ? 0.0f : lev[j - 1];
  }
  for (int c = t; c < (1 << C1); c += kThreads) {
    float pl = 0.0f;
    if (prevmsg) {
      const float *hp = reinterpret_cast<const float *>(prevmsg + m.hdr_off);
      const float lvl = hp[1 + min(c >> 1, m.S - 1)];
      pl = (c & 1) ? -lvl : lvl;
    }
    tprev[c] = pl;
  }
  // a run of one octet (a small layer) has so few adds that fewer copies, and less to clear and to flush, serve better
  const bool few = m.nblk - (long long)st.y * (kChunkCoords / kBlockCoords) <= 8;
  const int copies = few ? kHistFewCopies : kHistCopies;
  if (ex != kTypeSkip) {
    if (few) {
      for (int j = t; j < kGridPoints * kHistFewCopies; j += kThreads) lo[(j / kHistFewCopies) * kHistCopies + j % kHistFewCopies] = 0u;
    } else {
      for (int j = t; j < kGridPoints * kHistCopies; j += kThreads) lo[j] = 0u;
    }
    for (int j = t; j < kGridPoints * kHistHighCopies; j += kThreads) hi[j] = 0u;
  }
  __syncthreads();
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int i = t & 63;
  BucketWave &bw = bws[w];
  const float *__restrict__ v = a.grad[(size_t)kr * a.L + l];
  unsigned char *body = a.msg[kr] + m.body_off;
  const unsigned char *prevbody = prevmsg ? prevmsg + m.body_off : nullptr;
  const unsigned int k0 = (unsigned int)a.seed, k1 = (unsigned int)(a.seed >> 32);
  const long long noct = (m.nblk + 7) >> 3;
  unsigned long long best = 0ull;
  // The wave's octets of the run, one after the other: two of each tile.  The next octet's values are requested block by
  // block as the current one's are done with, into the same registers.
  const int n = 2 * st.z;
  float x[32], acc = 0.0f;
  unsigned int Dp[C1];
  float pn = 0.0f;
#pragma unroll
  for (int r = 0; r < C1; ++r) Dp[r] = 0u;
  const long long O0 = (long long)st.y * 8 + w * 2;
  if (O0 < noct) {
    load_octet(v, O0, m.d, i, x);
  }
#pragma unroll 1
  for (int q = 0; q < n; ++q) {
    const long long O = O0 + 8 * (q >> 1) + (q & 1), On = O0 + 8 * ((q + 1) >> 1) + ((q + 1) & 1);
    if (O < noct) {
      unsigned int D[C1];
#pragma unroll
      for (int r = 0; r < C1; ++r) D[r] = 0u;
      int i = t & 63;   // kept opaque: addresses derived from it are cheaper to form again than to hold through the loop
      asm volatile("" : "+v"(i));
      if (PREV && prevbody != nullptr) {   // requested here, used after the norms: a record held ahead would cost C1 registers
        load_record<C1>(prevbody + O * OS, i, Dp);
        pn = reinterpret_cast<const float *>(prevbody + O * OS + 256 * C1)[8 * (i >> 5) + (i & 7)];
      }
      Scales sc;
      unsigned int wfix;
      const bool high = bucket_norms<KIND>(a, x, reinterpret_cast<float *>(body + O * OS + 256 * C1), bw, i, ex, best, sc, wfix);
      sc.pnorm = pn;
      const bool more = q + 1 < n && On < noct;
      const bool full = more && (On + 1) * 2048 <= m.d;
      const float *vn = v + On * 2048;
      const auto done = [&](int bb, float (&diff)[4]) {
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = __builtin_fmaf(diff[j], diff[j], acc);
        asm volatile("" : "+v"(acc));
        if (full) load_block(vn, bb, i, &x[4 * bb]);
      };
      bool plain = false;
      if (ex != kTypeSkip) {
        float least = 3.402823466e+38f;
#pragma unroll
        for (int j = 0; j < 32; ++j) least = fminf(least, fabsf(x[j]));
        plain = !high && __ballot(least < 0x1p-129f) == 0ull;
      }
      const BucketHist hist = {wfix, lo + (i & (copies - 1)), hi + (i & (kHistHighCopies - 1)), ex != kTypeSkip, high, plain};
      const unsigned int c0 = (unsigned int)(O * 256 + i);
      if (m.nblk - O * 8 <= 2)   // one pair of blocks is all there is: the others would be worked on for nothing
        quantize_regs<C1, PREV, true, true>(x, c0, l, a.round, k, k0, k1, sc, bins, tab, tprev, D, Dp, hist, done, 1);
      else if (walk)
        quantize_regs<C1, PREV, true, true>(x, c0, l, a.round, k, k0, k1, sc, bins, tab, tprev, D, Dp, hist, done);
      else
        quantize_regs<C1, PREV, false, true>(x, c0, l, a.round, k, k0, k1, sc, bins, tab, tprev, D, Dp, hist, done);
      store_record<C1>(body + O * OS, i, D);
      if (more && !full) load_octet(v, On, m.d, i, x);   // the layer's ragged last octet
    }
    if (q & 1) {
      chain[(q >> 1) * kThreads + t] = acc;
      acc = 0.0f;
    }
  }
  __syncthreads();
  sum_tiles(a, chain, m, st, kr, w, i);
  // statistics of the run: largest bucket sum (bit pattern of a non-negative double) and the histogram
#pragma unroll
  for (int sh = 1; sh < 64; sh *= 2) {
    const unsigned long long other = __shfl_xor(best, sh, 64);
    best = other > best ? other : best;
  }
  if (i == 0) wmax[w] = best;
  __syncthreads();
  const size_t idx = (size_t)k * a.L + l;
  if (t == 0) {
    for (int q = 1; q < kThreads / 64; ++q) best = wmax[q] > best ? wmax[q] : best;
    if (best) atomicMax(reinterpret_cast<unsigned long long *>(a.sumsq) + idx, best);
  }
  if (ex != kTypeSkip) {
    unsigned long long *gh = reinterpret_cast<unsigned long long *>(a.hist + idx * kHistBins);
    for (int j = t; j < kGridPoints; j += kThreads) {
      unsigned long long c = 0ull, ch = 0ull;
      if (few) {
#pragma unroll
        for (int q = 0; q < kHistFewCopies; ++q) c += lo[j * kHistCopies + q];
      } else {
#pragma unroll
        for (int q = 0; q < kHistCopies; ++q) c += lo[j * kHistCopies + ((q + j) & (kHistCopies - 1))];
      }
#pragma unroll
      for (int q = 0; q < kHistHighCopies; ++q) ch += hi[j * kHistHighCopies + q];
      c += ch << kHistLowBits;
      if (c) atomicAdd(&gh[j], c);
    }
  }
}

// delta_k: slot j takes the node's tiles j, j+256, ... (all layers, in order), then the halving tree.
// Further workgroups clear what the next pass finds zero: under bucket scope, with a.hist_old, the statistics of the pass before; with
// a.clear_exch what the held tiles of this pass exchanged.
__global__ void __launch_bounds__(kThreads) k_delta_finalize(Dev a) {
  __shared__ double red[kThreads];
  const int k = a.node0 + blockIdx.x;
  const int kr = k - a.row0;   // row in the per-node scratch and pointer tables
  if (blockIdx.y != 0) {
    if (a.clear_exch) {
      unsigned long long *row = a.exch + (size_t)kr * exch_row(a.G);
      const size_t n = exch_row(a.G);
      for (size_t j = (blockIdx.y - 1) * (size_t)kThreads + threadIdx.x; j < n; j += a.clear_exch * (size_t)kThreads) row[j] = 0ull;
    } else {
      zero_stats(a.hist_old, a.sumsq_old, (size_t)k * a.L + blockIdx.y - 1);
    }
    return;
  }
  const double *p = a.dpartial + (size_t)kr * a.G;
  double acc = 0.0;
  // the loads of a slot are independent of its running sum: requested 16 at a time, added in the slot's order
  int g = threadIdx.x;
  for (; g + 15 * kThreads < a.G; g += 16 * kThreads) {
    double v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = p[g + q * kThreads];
#pragma unroll
    for (int q = 0; q < 16; ++q) acc = acc + v[q];
  }
  for (; g < a.G; g += kThreads) acc = acc + p[g];
  const double s = block_tree(acc, red);
  if (threadIdx.x == 0) a.delta[k] = s;
  // layers without coordinates have no tile: their header entries (norm 0, levels) are written here
  for (int q = 0; q < a.n_empty; ++q) {
    const LayerMeta m = a.meta[a.empty_layers[q]];
    float *h = reinterpret_cast<float *>(a.msg[kr] + m.hdr_off);
    const float *lev = a.lev + (size_t)m.type * kMaxPoints;
    const float n0 = (a.scope == kScopeBucket) ? 0.0f : a.norm[(size_t)kr * a.L + a.empty_layers[q]];
    for (int j = threadIdx.x; j <= m.S; j += kThreads) h[j] = (j == 0) ? n0 : lev[j - 1];
  }
}

// ------------------------------------------------------------------------------------------------ step
// eq. (general_stepsize): acc += (sum_k delta_k) / K^2 ; eta = gamma = (1 + acc)^(-1/2), taken as
// rcp_floor(sqrt_floor(1 + acc)).
__device__ __forceinline__ double sum_distances(const Dev &a) {
  double sum = a.delta[0];
  for (int k = 1; k < a.K; ++k) sum = sum + a.delta[k];
  return *a.acc + sum * a.invK2;
}
__device__ __forceinline__ float step_size(double acc) {
  float n, r;
  norm_and_inverse(1.0 + acc, n, r);   // 1 + acc is 1 at least, or not a number
  return r;
}
__device__ __forceinline__ void store_scalars(const Dev &a, double acc, float eta) {
  *a.acc = acc;
  a.eta[0] = eta;
  a.eta[1] = eta;
  if (a.eta_out) { a.eta_out[0] = eta; a.eta_out[1] = eta; }
}
__global__ void k_step_scalars(Dev a) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const double acc = sum_distances(a);
  store_scalars(a, acc, step_size(acc));
}

// eq. (Alt), Sec. 6: the rates for the update of this round from the sums over the rounds before it,
//   eta = (1 + lambda + mu)^(-1/2) as rcp_floor(sqrt_floor(.)),  gamma = (1 + lambda)^(q - 1/2),
// the power built from correctly rounded fp64 operations only: r_j = sqrt(r_{j-1}), r_0 = 1 + lambda, and
// (1 + lambda)^q = product of the r_j whose binary digit of q is set (j increasing).  Then lambda takes this
// round's sum_k ||Vhat_k||^2 / K^2 (the quantizer's distance output against an all-zero previous message).
__global__ void k_alt_scalars(Dev a) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const double lambda = a.alt_sums[0], mu = a.alt_sums[1];
  const float eta_prev = a.eta_out[0];
  const float eta = rcp_floor(sqrt_floor(1.0 + lambda + mu));
  const double base = 1.0 + lambda;
  double r = base, p = 1.0;
  for (int j = 1; j <= 32; ++j) {
    r = __dsqrt_rn(r);
    if ((a.q_digits >> (32 - j)) & 1u) p = p * r;
  }
  const float gamma = (float)__ddiv_rn(p, __dsqrt_rn(base));
  a.eta[0] = eta;
  a.eta[1] = gamma;
  a.eta[2] = eta_prev;
  a.eta_out[0] = eta;
  a.eta_out[1] = gamma;
  double sum = a.delta[0];
  for (int k = 1; k < a.K; ++k) sum = sum + a.delta[k];
  a.alt_sums[0] = lambda + sum * a.invK2;
}

// mu += ||X_t - X_{t+1}||^2: slot j takes the tiles j, j+256, ... (all layers, in order), then the halving tree.
__global__ void __launch_bounds__(kThreads) k_alt_finalize(Dev a) {
  __shared__ double red[kThreads];
  double acc = 0.0;
  int g = threadIdx.x;
  for (; g + 15 * kThreads < a.G; g += 16 * kThreads) {   // loads 16 at a time, sums in the slot's order
    double v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = a.dpartial[g + q * kThreads];
#pragma unroll
    for (int q = 0; q < 16; ++q) acc = acc + v[q];
  }
  for (; g < a.G; g += kThreads) acc = acc + a.dpartial[g];
  const double s = block_tree(acc, red);
  if (threadIdx.x == 0) a.alt_sums[1] = a.alt_sums[1] + s;
}

// DECODE + K-way mean (+ eq. (ODA) update unless MODE is kDecodeMean): one pass over Y, X_1 and the K messages.
// A wave takes NB = 8, 4 or 2 consecutive blocks of an octet: 4 * NB running sums per lane, the codes of K records, then the
// blocks of state.
// Under kDecodeUpdateAlt the lane also rebuilds X_t = X_1 + eta_prev * Y_t; its differences X_t - X_{t+1} go on the slot's chain
// (CHAIN) or are left in diffs.

// Words that hold 4*NB codes from any bit of a record where a part can start (a multiple of 4*NB*C1 bits).
template <int C1, int NB>
constexpr int part_words() {
  int most = 0;
  for (int part = 0; part < 8 / NB; ++part) {
    const int first = 4 * NB * C1 * part, end = first + 4 * NB * C1;
    const int words = (end + 31) / 32 - first / 32;
    most = words > most ? words : most;
  }
  return most;
}

// The record words of a lane that hold the codes of blocks NB*part .. of one octet (the last word again where a part needs
// fewer than the others).
template <int C1, int NB>
__device__ __forceinline__ void load_part(const unsigned char *octet, int part, int i, unsigned int (&D)[part_words<C1, NB>()]) {
  const auto *g = reinterpret_cast<const __attribute__((address_space(1))) unsigned int *>(as_global(octet));
  const int w0 = (4 * NB * C1 * part) >> 5;
#pragma unroll
  for (int r = 0; r < part_words<C1, NB>(); ++r) D[r] = __builtin_nontemporal_load(g + min(w0 + r, C1 - 1) * 64 + i);
}

// A part may start inside a word: its codes are moved to bit 0.
template <int C1, int NB>
__device__ __forceinline__ void align_part(unsigned int (&D)[part_words<C1, NB>()], int part) {
  if constexpr (4 * NB * C1 % 32 != 0) {
    constexpr int N = part_words<C1, NB>();
    const int sh = (4 * NB * C1 * part) & 31;
#pragma unroll
    for (int r = 0; r < N; ++r) D[r] = __builtin_amdgcn_alignbit(r + 1 < N ? D[r + 1] : 0u, D[r], sh);
  }
}

// The bucket norms a lane needs from one octet's trailer (its half's, blocks NB*part ..).
template <int NB>
__device__ __forceinline__ void load_bucket_norms(const unsigned char *trailer, int part, int i, float (&n)[NB]) {
  typedef float vec __attribute__((ext_vector_type(NB == 2 ? 2 : 4)));
  constexpr int V = NB == 2 ? 2 : 4;
  const auto *g = reinterpret_cast<const __attribute__((address_space(1))) vec *>(as_global(trailer)) + (8 / V) * (i >> 5) + part * (NB / V);
#pragma unroll
  for (int q = 0; q < NB / V; ++q) {
    const vec v = g[q];
#pragma unroll
    for (int j = 0; j < V; ++j) n[V * q + j] = v[j];
  }
}

// What a wave needs of one node's message: codes and, under bucket scope, norms.
template <int C1, int NB, bool BUCKET>
struct Part {
  unsigned int D[part_words<C1, NB>()];
  float n[BUCKET ? NB : 1];
  __device__ __forceinline__ void load(const unsigned char *octet, int part, int i) {
    load_part<C1, NB>(octet, part, i, D);
    if constexpr (BUCKET) load_bucket_norms<NB>(octet + 256 * C1, part, i, n);
  }
};

// The update of a few tiles requests its part of the state before the tables are set up: there is no other wave to fill the wait for it.
template <int MODE, int NB>
struct StatePart {
  static constexpr bool early = MODE == kDecodeUpdateScalars;
  float y[early ? 4 * NB : 1], x1[early ? 4 * NB : 1];
};

// EARLY: cur is node 0's part already, requested before the tables were set up.
template <int C1, int MODE, bool FAST, bool BUCKET, int NB, bool EARLY, bool CHAIN>
__device__ __forceinline__ void decode_part(const Dev &a, const LayerMeta &m, int l, long long O, int part, const float *T, int i,
                                            float eta, float gamma, float eta_prev, const StatePart<MODE, NB> &st, Part<C1, NB, BUCKET> cur,
                                            float (&diffs)[MODE == kDecodeUpdateAlt ? 4 * NB : 1], float &chain) {
  constexpr int TS = 1 << C1;   // table entries per node, indexed by code = sign | h << 1
  constexpr long long OS = 256 * C1 + (BUCKET ? 64 : 0);   // bytes per octet (bucket scope: codes + 16 norms)
  const long long boff = m.body_off + O * OS;
  float sum[4 * NB];
  if (!EARLY) cur.load(a.msgs_in[0] + boff, part, i);
  if constexpr (StatePart<MODE, NB>::early) {
    // few tiles: nothing else fills the wait for a node's part, so several are on their way (K = 4, us a round: 9 k entries 15.9 -> 15.2,
    // 152 k 19.4 -> 18.7)
    constexpr int N = 4;
    const auto take = [&](Part<C1, NB, BUCKET> &p, int k) {   // node k's part, which is here
      const float *Tk = T + k * TS;
      align_part<C1, NB>(p.D, part);
#pragma unroll
      for (int jj = 0; jj < 4 * NB; ++jj) {
        float val = lds_float_at(Tk, extract_off<C1>(p.D, jj));   // layer / vector scope: +-norm_k * level
        if (BUCKET) val = p.n[jj >> 2] * val;                     // bucket scope: the table holds +-level
        sum[jj] = (k == 0) ? val : sum[jj] + val;
      }
    };
    Part<C1, NB, BUCKET> ring[N];
    ring[0] = cur;
#pragma unroll
    for (int q = 1; q < N; ++q)
      if (q < a.K) ring[q].load(a.msgs_in[q] + boff, part, i);
    for (int k = 0; k < a.K; k += N) {
#pragma unroll
      for (int q = 0; q < N; ++q) {
        if (k + q >= a.K) break;
        take(ring[q], k + q);
        if (k + q + N < a.K) ring[q].load(a.msgs_in[k + q + N] + boff, part, i);
      }
    }
  } else {
    for (int k = 0; k < a.K; ++k) {   // cur: node k's, requested before; the next node's are requested now
      Part<C1, NB, BUCKET> nxt = {};
      if (k + 1 < a.K) nxt.load(a.msgs_in[k + 1] + boff, part, i);
      // (Written out: with the body shared with the loop above the compiler orders it otherwise, the mean of 151 M entries, K = 8
      // 198.6 -> 199.7 us.)
      const float *Tk = T + k * TS;
      align_part<C1, NB>(cur.D, part);
#pragma unroll
      for (int jj = 0; jj < 4 * NB; ++jj) {
        float val = lds_float_at(Tk, extract_off<C1>(cur.D, jj));
        if (BUCKET) val = cur.n[jj >> 2] * val;
        sum[jj] = (k == 0) ? val : sum[jj] + val;
      }
      cur = nxt;
    }
  }
  const int lane = CHAIN ? i : lane_id();   // i, which the loop above need not keep (with two octets a wave keeping it is cheaper)
#pragma unroll
  for (int bb = 0; bb < NB; ++bb) {
    const long long B = O * 8 + part * NB + bb;
    if (FAST || B < m.nblk) {
      const long long e = B * kBlockCoords + 4 * lane;
      const long long dlim = FAST ? e + 4 : m.d;   // FAST: the whole block is inside the layer
      float mean[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) mean[j] = sum[4 * bb + j] * a.invK;
      if (MODE == kDecodeMean) {
        store4(a.mean_out[l], e, dlim, mean);
      } else if (MODE == kDecodeExtrapolate) {   // out = x - gamma * mean (x in a.x1, out in a.x_half)
        float x[4], out[4];
        load4(a.x1[l], e, dlim, x);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float gm = gamma * mean[j];
          out[j] = x[j] - gm;
        }
        store4(a.x_half[l], e, dlim, out);
      } else {
        float y[4], x1[4], xn[4], xh[4];
        if constexpr (StatePart<MODE, NB>::early) {
#pragma unroll
          for (int j = 0; j < 4; ++j) { y[j] = st.y[4 * bb + j]; x1[j] = st.x1[4 * bb + j]; }
        } else {
          load4(a.y[l], e, dlim, y);      // coordinates past the end of the layer read as 0 and add nothing below
          load4(a.x1[l], e, dlim, x1);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float xt = 0.0f;
          if (MODE == kDecodeUpdateAlt) {
            const float ey_old = eta_prev * y[j];
            xt = x1[j] + ey_old;
          }
          y[j] = y[j] - mean[j];
          const float ey = eta * y[j];
          xn[j] = x1[j] + ey;
          const float gm = gamma * mean[j];
          xh[j] = xn[j] - gm;
          if (MODE == kDecodeUpdateAlt) {
            const float diff = xt - xn[j];
            if (CHAIN) chain = __builtin_fmaf(diff, diff, chain);
            else diffs[4 * bb + j] = diff;
          }
        }
        store4(a.y[l], e, dlim, y);
        store4(a.x_half[l], e, dlim, xh);
        if (a.x_next) store4(a.x_next[l], e, dlim, xn);
      }
    } else if (MODE == kDecodeUpdateAlt && !CHAIN) {
#pragma unroll
      for (int j = 0; j < 4; ++j) diffs[4 * bb + j] = 0.0f;
    }
  }
}

// The decode pass runs best in short workgroups (measured against one tile per workgroup of four waves with two octets
// each: 6 % faster at K = 8, 4 % at K = 16): a workgroup takes a few consecutive octets of a tile (kDecodeOctets), 8 / NB waves
// an octet.  How many blocks a wave takes is chosen by decode_blocks.  EARLY: node 0's part is requested before the tables are set
// up (parts of octets always; whole ones where mean_early says so).  Only the (Alt) variant keeps a workgroup to the tile: its
// squared-distance term is defined per slot and tile.  It has eight waves, where a slot's chain goes from the even wave of a pair to
// the odd one, or (NB = 16) four, each with two octets, one after the other; alt_blocks chooses.  Four waves a SIMD (128
// registers) are two tiles of eight waves on a CU: with one register more it is one, under bucket scope with 8 and 9 bits 11 k tiles,
// K = 4 791 and 813 us, now 643 and 672.
template <int C1, int MODE, bool BUCKET, int NB, bool EARLY>
__global__ void __launch_bounds__(NB > 8 ? kThreads : 2 * kThreads, MODE != kDecodeUpdateAlt ? 1 : (BUCKET && NB > 8) ? 3 : 4) k_decode(Dev a) {
  extern __shared__ float T[];   // [K][2^C1]: +-norm_k * level_h (bucket scope: +-level_h) from the K message headers
  constexpr bool ALT = MODE == kDecodeUpdateAlt;
  __shared__ double red[ALT ? kThreads : 1];
  const int noct_wg = (int)(blockDim.x >> 6) * NB / 8;   // octets of a workgroup
  const int parts = 8 / noct_wg;                         // workgroups per tile
  const int g = blockIdx.x / parts, part = blockIdx.x - g * parts;
  const int2 tile = a.tiles[g];
  const int l = tile.x;
  const LayerMeta m = a.meta[l];
  if (m.planes != C1) return;
  const int t = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int i = t & 63;
  constexpr int PB = NB < 8 ? NB : 8;   // blocks of a wave's part
  const int piece = w % (8 / PB);
  const long long O = (long long)tile.y * 8 + part * noct_wg + w * NB / 8, noct = (m.nblk + 7) >> 3;
  const bool live = O < noct;
  Part<C1, PB, BUCKET> first = {};
  if (EARLY && live) first.load(a.msgs_in[0] + m.body_off + O * (256 * C1 + (BUCKET ? 64 : 0)), piece, i);
  StatePart<MODE, PB> state;
  if constexpr (StatePart<MODE, PB>::early) {
#pragma unroll
    for (int bb = 0; bb < PB; ++bb) {
      const long long e = (O * 8 + piece * PB + bb) * kBlockCoords + 4 * i;
      float q[4] = {0.0f, 0.0f, 0.0f, 0.0f}, v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      if (e < m.d) {
        load4(a.y[l], e, m.d, q);
        load4(a.x1[l], e, m.d, v);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) { state.y[4 * bb + j] = q[j]; state.x1[4 * bb + j] = v[j]; }
    }
  }
  const int TS = 1 << C1;
  double new_acc = 0.0;
  if (MODE == kDecodeUpdateScalars) new_acc = sum_distances(a);   // every wave computes what k_step_scalars computes
  for (int idx = threadIdx.x; idx < a.K * TS; idx += blockDim.x) {
    const int k = idx / TS, c = idx - k * TS;
    const float *hp = reinterpret_cast<const float *>(a.msgs_in[k] + m.hdr_off);
    const float lvl = hp[1 + min(c >> 1, m.S - 1)];
    const float mag = BUCKET ? lvl : hp[0] * lvl;
    T[idx] = (c & 1) ? -mag : mag;
  }
  // The workgroup counted last in a.readers overwrites *a.acc (below).  So a workgroup may be counted only after each of
  // its waves has the old value in a register: the sum is complete here (the empty statement needs it), before the barrier,
  // and the count comes after the barrier.
  if (MODE == kDecodeUpdateScalars) asm volatile("" : "+v"(new_acc) : : "memory");
  __syncthreads();
  float eta = 0.0f, gamma = 0.0f, eta_prev = 0.0f;
  if (MODE == kDecodeUpdate || ALT) { eta = a.eta[0]; gamma = a.eta[1]; }
  unsigned int readers = 0u;
  if (MODE == kDecodeUpdateScalars) {
    if (t == 0) readers = __hip_atomic_fetch_add(a.readers, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    eta = gamma = step_size(new_acc);
  }
  if (ALT) eta_prev = a.eta[2];
  if (MODE == kDecodeExtrapolate) gamma = a.gamma_in[0];
  float diffs[ALT ? 4 * PB : 1], accx = 0.0f;
  if constexpr (NB > 8) {
    for (int oo = 0; oo < NB / 8; ++oo) {
      const long long Oc = O + oo;
      if (Oc >= noct) break;
      if ((Oc + 1) * 2048 <= m.d) decode_part<C1, MODE, true, BUCKET, PB, EARLY, true>(a, m, l, Oc, 0, T, i, eta, gamma, eta_prev, state, first, diffs, accx);
      else decode_part<C1, MODE, false, BUCKET, PB, EARLY, true>(a, m, l, Oc, 0, T, i, eta, gamma, eta_prev, state, first, diffs, accx);
    }
    const double total = block_tree((double)accx, red);
    if (t == 0) a.dpartial[g] = total;
  } else if (live) {
    if ((O + 1) * 2048 <= m.d) decode_part<C1, MODE, true, BUCKET, PB, EARLY, false>(a, m, l, O, piece, T, i, eta, gamma, eta_prev, state, first, diffs, accx);
    else decode_part<C1, MODE, false, BUCKET, PB, EARLY, false>(a, m, l, O, piece, T, i, eta, gamma, eta_prev, state, first, diffs, accx);
  }
  if (ALT && NB == 8) {
    // a slot's fp32 fused chain in increasing coordinate: even waves first
    float *chain = reinterpret_cast<float *>(red);
    const int sl = (w >> 1) * 64 + i;
    if (!(w & 1)) {
      if (live) {
#pragma unroll
        for (int j = 0; j < 4 * PB; ++j) accx = __builtin_fmaf(diffs[j], diffs[j], accx);
      }
      chain[sl] = accx;
    }
    __syncthreads();
    if (w & 1) {
      accx = chain[sl];
      if (live) {
#pragma unroll
        for (int j = 0; j < 4 * PB; ++j) accx = __builtin_fmaf(diffs[j], diffs[j], accx);
      }
    }
    __syncthreads();   // the chains' room becomes that of the 256 slots
    if (w & 1) red[sl] = (double)accx;
    __syncthreads();
    if (w == 0) {
      const double total = wave_tree<true>(red, i);
      if (i == 0) a.dpartial[g] = total;
    }
  }
  if (MODE == kDecodeUpdateScalars && t == 0 && readers == gridDim.x - 1u) {   // all waves of all workgroups have read *a.acc
    store_scalars(a, new_acc, eta);
    *a.readers = 0u;
  }
}

// ------------------------------------------------------------------------------------------------ code lengths
// Occurrences of every level index in the K messages, per type (the empirical p_j of Thm 5.3).  Every code of every
// octet is counted, padding included (index 0): the host subtracts the padding.  Each lane counts into its own column
// of a shared-memory table [index][lane], so no two lanes of a wave ever meet on an address.
template <int C1, bool BUCKET>
__global__ void __launch_bounds__(kThreads) k_index_hist(Dev a) {
  extern __shared__ unsigned int cnt[];   // [2^(C1-1)][64]
  constexpr int NI = 1 << (C1 - 1);
  constexpr long long OS = 256 * C1 + (BUCKET ? 64 : 0);
  const int4 st = a.stiles[blockIdx.x];   // a run of up to kSuperTile tiles of one layer: one flush per run
  const int l = st.x, k = blockIdx.y;
  const LayerMeta m = a.meta[l];
  if (m.planes != C1) return;
  const int t = threadIdx.x, w = t >> 6, i = t & 63;
  for (int q = t; q < NI * 64; q += kThreads) cnt[q] = 0u;
  __syncthreads();
  const long long noct = (m.nblk + 7) >> 3;
  for (int cc = 0; cc < st.z; ++cc)
    for (int oo = 0; oo < 2; ++oo) {
      const long long O = (long long)(st.y + cc) * 8 + w * 2 + oo;
      if (O >= noct) break;
      unsigned int D[C1];
      load_record<C1>(a.msgs_in[k] + m.body_off + O * OS, i, D);
#pragma unroll
      for (int jj = 0; jj < 32; ++jj) {
        const unsigned int h = extract_code<C1>(D, jj) >> 1;
        atomicAdd(&cnt[h * 64 + i], 1u);
      }
    }
  __syncthreads();
  for (int h = t; h < NI; h += kThreads) {
    unsigned long long sum = 0ull;
    for (int q = 0; q < 64; ++q) sum += cnt[h * 64 + ((q + h) & 63)];
    if (sum) atomicAdd(&a.index_counts[(size_t)m.type * 256 + h], sum);
  }
}

// ------------------------------------------------------------------------------------------------ level fit
// Largest squared norm of a type -> its binary exponent (fixed-point scale of the weights lambda_z).
__global__ void __launch_bounds__(kThreads) k_fit_typemax(Dev a) {
  __shared__ double red[kThreads];
  __shared__ int bad[1];
  const int mtype = blockIdx.x;
  if (threadIdx.x == 0) bad[0] = 0;
  for (int j = threadIdx.x; j < kGridPoints; j += kThreads) a.pooled[(size_t)mtype * kGridPoints + j] = 0ull;
  __syncthreads();
  double mx = 0.0;   // largest weight ||v||_q^2 of the type
  for (int idx = threadIdx.x; idx < a.K * a.L; idx += kThreads) {
    const int l = idx % a.L;
    if (a.meta[l].type != mtype) continue;
    const double s = a.sumsq[idx];
    if (!stat_finite(s, a.kind)) bad[0] = 1;
    else mx = fmax(mx, weight_of(s, a.kind));
  }
  red[threadIdx.x] = mx;
  __syncthreads();
  for (int h = kThreads / 2; h >= 1; h >>= 1) {
    if (threadIdx.x < h) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + h]);
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double smax = red[0];
    int ex = kTypeSkip;
    if (!bad[0] && smax > 0.0) ex = (int)((__double_as_longlong(smax) >> 52) & 0x7FF) - 1023;
    a.type_exp[mtype] = ex;
  }
}

// The weight of a vector in fixed point, exponent ex of its type.
__device__ __forceinline__ unsigned long long fit_weight(double stat, int kind, int ex) {
  return (unsigned long long)floor(ldexp(weight_of(stat, kind), 23 - ex));
}
// Grid index of the midpoint of a raw magnitude bin under the vector's normalisation.
__device__ __forceinline__ int raw_bin_to_grid(int b, float inv) {
  const float mid = u2f(((unsigned int)b << 20) | (1u << 19));
  const int j = (int)(f2u(fminf(mid * inv, 1.0f)) >> 20) - kGridBase;
  return max(0, min(j, kGridPoints - 1));
}
// A count of the accumulating histogram; it moves to the histogram of the last fit, and its cell is zero for the next one.
__device__ __forceinline__ void move_count(const Dev &a, size_t idx, int b, unsigned int c) {
  a.hist_last[idx * kHistBins + b] = c;
  if (c != 0u) a.hist[idx * kHistBins + b] = 0u;
}

// Re-bin one (node, layer) histogram onto the normalised grid with weight floor(||v||_q^2 * 2^(23 - exponent)).
__global__ void __launch_bounds__(kThreads) k_fit_pool(Dev a) {
  const int l = blockIdx.x, k = blockIdx.y;
  const LayerMeta m = a.meta[l];
  const size_t idx = (size_t)k * a.L + l;
  unsigned long long *W = a.pooled + (size_t)m.type * kGridPoints;
  const int ex = a.type_exp[m.type];
  const unsigned long long wfix = ex == kTypeSkip ? 0ull : fit_weight(a.sumsq[idx], a.kind, ex);
  const float inv = a.inv[idx];
  for (int b = threadIdx.x; b < kHistBins; b += kThreads) {
    const unsigned int c = a.hist[idx * kHistBins + b];
    move_count(a, idx, b, c);
    if (wfix != 0ull && inv != 0.0f && b != 0 && c != 0u) atomicAdd(&W[raw_bin_to_grid(b, inv)], wfix * (unsigned long long)c);
  }
}

// ---- level fit under bucket scope from given vectors: two passes over them (scale of the weights, then histogram).
// Statistic of the lane's bucket (half of block B) by the in-order binary tree, valid in all its 32 lanes.  Every lane
// of the wave must call this.
__device__ __forceinline__ double half_block_stat(const LayerMeta &m, const float *__restrict__ v, long long B, int i,
                                                  float (&x)[4], int kind) {
  const long long e = B * kBlockCoords + 4 * i;
#pragma unroll
  for (int j = 0; j < 4; ++j) x[j] = 0.0f;
  if (e < m.d) load4(v, e, m.d, x);
  if (kind == kNormLinf) {   // largest magnitude of the bucket
    unsigned int mb = 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j) mb = max(mb, f2u(x[j]) & 0x7FFFFFFFu);
    double s = (double)magnitude_from_bits(mb);
#pragma unroll
    for (int w = 1; w < 32; w *= 2) s = fmax(s, __shfl_xor(s, w, 64));
    return s;
  }
  float acc = 0.0f;
  if (kind == kNormL2) {
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = __builtin_fmaf(x[j], x[j], acc);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = acc + fabsf(x[j]);
  }
  double s = (double)acc;
#pragma unroll
  for (int w = 1; w < 32; w *= 2) s = s + __shfl_xor(s, w, 64);
  if (kind == kNormL2) {
    // below 2^-100 (squares may have vanished) or not finite (they may have overflowed): exact fp64 squares instead
    const bool redo = !(s >= kBucketRescueBelow) || !(s <= 1.7976931348623157e308);
    if (__ballot(redo) != 0ull) {
      double acc64 = 0.0;
#pragma unroll
      for (int j = 0; j < 4; ++j) acc64 = __builtin_fma((double)x[j], (double)x[j], acc64);
#pragma unroll
      for (int w = 1; w < 32; w *= 2) acc64 = acc64 + __shfl_xor(acc64, w, 64);
      if (redo) s = acc64;
    }
  }
  return s;
}

// Largest bucket statistic of every (node, layer), as the bit pattern of a non-negative double (ordered like
// an integer); one that is not a finite number in range leaves +infinity.  a.sumsq must be zero on entry.
__global__ void __launch_bounds__(kThreads) k_bucket_max(Dev a) {
  __shared__ unsigned long long wmax[kThreads / 64];
  const int4 st = a.stiles[blockIdx.x];
  const int l = st.x, k = blockIdx.y;
  const LayerMeta m = a.meta[l];
  const float *__restrict__ v = a.grad[(size_t)k * a.L + l];
  const int t = threadIdx.x, w = t >> 6, i = t & 63;
  unsigned long long best = 0ull;
  for (int cc = 0; cc < st.z; ++cc)
    for (int oo = 0; oo < 2; ++oo) {
      const long long O = (long long)(st.y + cc) * 8 + w * 2 + oo;
      for (int bb = 0; bb < 8; ++bb) {
        const long long B = O * 8 + bb;
        if (B >= m.nblk) break;   // the same for every lane of the wave
        float x[4];
        const double s = half_block_stat(m, v, B, i, x, a.kind);
        const bool finite = stat_finite(s, a.kind);
        const unsigned long long bits = finite ? (unsigned long long)__double_as_longlong(s) : 0x7FF0000000000000ull;
        best = bits > best ? bits : best;
      }
    }
  // both halves of the wave, then the four waves
  const unsigned long long other = __shfl_xor(best, 32, 64);
  best = other > best ? other : best;
  if (i == 0) wmax[w] = best;
  __syncthreads();
  if (t == 0) {
    for (int q = 1; q < kThreads / 64; ++q) best = wmax[q] > best ? wmax[q] : best;
    if (best) atomicMax(reinterpret_cast<unsigned long long *>(a.sumsq) + ((size_t)k * a.L + l), best);
  }
}

// Weighted histogram of the normalised magnitudes of the coordinates of every (node, layer) on the 257-point
// grid: weight floor(bucket sum * 2^(23 - exponent of the type)), integer adds, kept per (node, layer) in the first
// 257 64-bit words of its histogram area.
__global__ void __launch_bounds__(kThreads) k_bucket_hist(Dev a) {
  __shared__ unsigned long long lh[kGridPoints];
  const int4 st = a.stiles[blockIdx.x];
  const int l = st.x, k = blockIdx.y;
  const LayerMeta m = a.meta[l];
  const int ex = a.type_exp[m.type];
  if (ex == kTypeSkip) return;
  const float *__restrict__ v = a.grad[(size_t)k * a.L + l];
  const int t = threadIdx.x, w = t >> 6, i = t & 63;
  for (int j = t; j < kGridPoints; j += kThreads) lh[j] = 0ull;
  __syncthreads();
  for (int cc = 0; cc < st.z; ++cc)
    for (int oo = 0; oo < 2; ++oo) {
      const long long O = (long long)(st.y + cc) * 8 + w * 2 + oo;
      for (int bb = 0; bb < 8; ++bb) {
        const long long B = O * 8 + bb;
        if (B >= m.nblk) break;   // the same for every lane of the wave
        float x[4];
        const double s = half_block_stat(m, v, B, i, x, a.kind);
        const unsigned long long wfix = (unsigned long long)floor(ldexp(weight_of(s, a.kind), 23 - ex));
        const float inv = rcp_floor(norm_of(s, a.kind));
        if (wfix == 0ull || inv == 0.0f) continue;
        const long long e = B * kBlockCoords + 4 * i;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (e + j >= m.d || ((f2u(x[j]) & 0x7FFFFFFFu) >> 20) == 0u) continue;
          const float uc = fminf(fabsf(x[j]) * inv, 1.0f);
          int g = (int)(f2u(uc) >> 20) - kGridBase;
          g = max(0, min(g, kGridPoints - 1));
          atomicAdd(&lh[g], wfix);
        }
      }
    }
  __syncthreads();
  unsigned long long *gh = reinterpret_cast<unsigned long long *>(a.hist + ((size_t)k * a.L + l) * kHistBins);
  for (int j = t; j < kGridPoints; j += kThreads) {
    const unsigned long long c = lh[j];
    if (c) atomicAdd(&gh[j], c);
  }
}

// Pool the per-(node, layer) grid histograms of a type.
__global__ void __launch_bounds__(kThreads) k_fit_pool_b(Dev a) {
  const int l = blockIdx.x, k = blockIdx.y;
  const LayerMeta m = a.meta[l];
  if (a.type_exp[m.type] == kTypeSkip) return;
  const unsigned long long *gh = reinterpret_cast<const unsigned long long *>(a.hist + ((size_t)k * a.L + l) * kHistBins);
  unsigned long long *W = a.pooled + (size_t)m.type * kGridPoints;
  for (int j = threadIdx.x; j < kGridPoints; j += kThreads) {
    const unsigned long long c = gh[j];
    if (c) atomicAdd(&W[j], c);
  }
}

__device__ __forceinline__ float grid_value(int j) { return u2f((unsigned int)(j + kGridBase) << 20); }

// Search tables of one type from its levels (in shared memory; sgap: room for kMaxPoints): reciprocal gaps, tau of the lower edge of
// every bin of values whose top bits are the same, tau = the largest j <= S-2 with l_j <= edge (the levels increase, so that j is found
// by halving), and for every grid bin the entry {l_tau, 1/gap, l_tau+1, tau}.  Grid bin 0 also serves all values below it: its
// entry is that of tau = 0.
__device__ void build_tables(const Dev &a, int mtype, int S, const float *slev, float *sgap) {
  float *rg = a.rgap + (size_t)mtype * kMaxPoints;
  for (int j = threadIdx.x; j < kMaxPoints; j += (int)blockDim.x) {
    const float r = (j < S - 1) ? rcp_floor(slev[j + 1] - slev[j]) : 0.0f;
    rg[j] = r;
    sgap[j] = r;
  }
  // Does some interior level lie inside a bin, or not above the first one?  Then a lane may have to step on from the entry of
  // its bin.  (0 and 1 are edges.)
  int inside = 0;
  for (int j = threadIdx.x + 1; j <= S - 2; j += (int)blockDim.x)
    inside |= (f2u(slev[j]) & 0xFFFFFu) != 0u || f2u(slev[j]) <= (unsigned int)kGridBase << 20;
  const int walk = __syncthreads_or(inside);
  if (threadIdx.x == 0) a.walk[mtype] = walk;
  for (int q = threadIdx.x; q < kLutSize; q += (int)blockDim.x) {
    const float lo = u2f((unsigned int)min(q, kGridBase + kGridPoints - 1) << 20);   // the last bins are beyond 1
    int tau = 0;
    for (int n = S - 2; n > 0;) {   // the answer lies in tau .. tau + n
      const int h = (n + 1) >> 1;
      if (slev[tau + h] <= lo) { tau += h; n -= h; }
      else n = h - 1;
    }
    a.lut[(size_t)mtype * kLutSize + q] = (unsigned char)tau;
    const int g = q - kGridBase;
    if (g < 0 || g >= kGridPoints) continue;
    if (g == 0) tau = 0;
    a.bins[(size_t)mtype * kGridPoints + g] = make_float4(slev[tau], sgap[tau], slev[tau + 1], u2f((unsigned int)tau));
  }
}

__global__ void __launch_bounds__(kThreads) k_build_tables(Dev a, int mtype) {
  __shared__ float slev[kMaxPoints], sgap[kMaxPoints];
  const int S = a.type_points[mtype];
  for (int j = threadIdx.x; j < S; j += kThreads) slev[j] = a.lev[(size_t)mtype * kMaxPoints + j];
  __syncthreads();
  build_tables(a, mtype, S, slev, sgap);
}

// Exact minimisation of eq. (Qada2) over interior levels on the grid by dynamic programming; one workgroup per type.
// cost(a, b) = sum over bins i in [a, b) of W_i (g_b - mid_i)(mid_i - g_a), from prefix sums P0, P1, P2 of W, W*mid,
// W*mid^2 taken sequentially in increasing bin (fp64; the same operation order as the CPU oracle).
struct FitRow { double p0, p1, p2, g; };

__device__ __forceinline__ double fit_cost(const FitRow &ra, const FitRow &rb) {
  return ((ra.g + rb.g) * (rb.p1 - ra.p1) - (rb.p2 - ra.p2)) - (ra.g * rb.g) * (rb.p0 - ra.p0);
}

constexpr int kFitThreads = 1024;
static_assert(kHistBins == 2 * kFitThreads, "two raw bins a thread");
constexpr int kFitLdsPoints = 128;  // up to this many level points the back-pointers stay in shared memory
// The cost of a pair (a, b) does not depend on the stage, so every thread computes the costs of its pairs once and
// keeps them in registers.  Grid indices b (1..255, the only places an interior level can sit) go two by two: couple q has
// b = 2q-1 and 2q, whose candidates a = 0..2q-1 are cut into segments of kFitSeg, one thread per segment for both b -- 975
// threads, 2 * kFitSeg costs each.  A stage is then, per pair, half a shared-memory read, one addition, one comparison, one
// minimum and one select, and a second step in which four threads per b combine its segments in increasing a.
// Bound by one CU: a stage takes 1.6 us, of which 1.0 is the issue of 4 fp64 instructions per pair and, beside them, 16 cycles
// of shared memory per 128-bit read of a wave; the rest is the chain of the second step.  Segments are 144 bytes apart, so
// that the 15 of them start on different banks.  With one b a thread (40 candidates, twice the reads; segments 320 bytes apart,
// rows of the prefix sums 1280, which met on banks) the kernel took, with layers / gathered statistics: 4 levels 28.3 / 27.7
// us, now 19.5 / 18.0; 8 35.9 / 34.0, 27 / 24; 16 51.4 / 49.7, 39.8 / 37.2; 64 139 / 137, 119 / 114; 256 508 / 509, 447 / 433.
constexpr int kFitSeg = 18;
constexpr int kFitSegs = 15;        // segments of the last couple
constexpr int kFitGroup = kFitSeg / 2;   // couples kFitGroup*(g-1)+1 .. kFitGroup*g have g segments each
constexpr int kFitPad = 272;        // rows are read up to index 14 * 18 + 17
static_assert(kFitGroup * kFitSegs * (kFitSegs - 1) / 2 + 2 * kFitSegs <= kFitThreads - 32, "two b of 14 groups and the last two couples");

// SRC: where the pooled weights come from.
//   kFitPooled   k_fit_typemax and k_fit_pool have run
//   kFitLayers   layer scope, at most kFitLayerPairs (node, layer) pairs a type: the workgroup does for its type what
//                k_norm_finalize, k_fit_typemax and k_fit_pool do, and clears the histogram for the next fit.  Four launches
//                of 3 to 5 us less, 8 us more here: 6.3 M entries in 10 tensors, K = 8, 16 levels 183 -> 177.5 us per round.
//                Of this kernel's 40 us there: norms 4, pooling 4, the three running sums 3, pair costs 5, thirteen stages
//                20, last stage, backtrack and tables 4.
//   kFitBuckets  bucket scope, at most kFitBucketPairs: pools what the last quantize passes gathered and derives the next scale
template <int SRC>
__global__ void __launch_bounds__(kFitThreads) k_fit_dp(Dev a) {
  __shared__ __attribute__((aligned(16))) double D[2][kFitPad];
  __shared__ __attribute__((aligned(16))) double P[3][kFitPad], gv[kFitPad];   // by grid index: sums over the bins below it, its value
  __shared__ __attribute__((aligned(16))) double pbest[2 * kFitThreads - 64];   // the segments' minima for both b of their couple
  __shared__ unsigned char pj[2 * kFitThreads];   // ... and where in the segment they are taken
  __shared__ float slev[kMaxPoints];
  // back-pointers of the stages 2, 3, ..., when S is small enough; before the stages the pooled weights and the per-bin terms
  __shared__ __attribute__((aligned(16))) unsigned char sarg[(kFitLdsPoints - 2) * 256];
  unsigned long long *Ws = reinterpret_cast<unsigned long long *>(sarg);
  double (*wd)[kFitPad + 16] = reinterpret_cast<double (*)[kFitPad + 16]>(sarg + 8 * kFitPad);   // W, W*mid, (W*mid)*mid per bin
  static_assert(sizeof(sarg) >= 8 * kFitPad + 3 * 8 * (kFitPad + 16), "weights and terms share the back-pointers' space");
  __shared__ double stat[SRC == kFitPooled ? 1 : SRC == kFitLayers ? kFitLayerPairs : kFitBucketPairs];
  __shared__ float sinv[SRC == kFitLayers ? kFitLayerPairs : 1];
  __shared__ unsigned long long swgt[SRC == kFitLayers ? kFitLayerPairs : 1];
  const int mtype = blockIdx.x;
  const int S = a.type_points[mtype];
  const int t = threadIdx.x;
  if (SRC == kFitPooled) {
    if (a.type_exp[mtype] == kTypeSkip) return;   // all-zero or non-finite vectors: the type keeps its levels
  } else {
    const int f0 = a.type_first[mtype], nl = a.type_first[mtype + 1] - f0, P = a.K * nl;   // pair p: node p / nl
    const auto at = [&](int p) { return (size_t)(p / nl) * a.L + a.type_layers[f0 + p % nl].x; };
    unsigned int count[kFitLayerPairs][2];   // raw bins t and t + 1024 of the pairs: requested before the norms are worked out
    if (SRC == kFitLayers) {
#pragma unroll
      for (int q = 0; q < kFitLayerPairs; ++q) {
        const size_t idx = q < P ? at(q) : 0;
        count[q][0] = q < P ? a.hist[idx * kHistBins + t] : 0u;
        count[q][1] = q < P ? a.hist[idx * kHistBins + kFitThreads + t] : 0u;
      }
      // norms, a wave per pair: slot j takes a layer's tiles j, j + 256, ... in increasing order, then the tree; lane i has
      // the slots i, i + 64, i + 128, i + 192
      const int i = t & 63;
      for (int p = t >> 6; p < P; p += kFitThreads / 64) {
        const int3 lay = a.type_layers[f0 + p % nl];   // layer, first tile, tiles
        const int tiles = lay.z;
        const double *part = a.partial + (size_t)(p / nl) * a.G + lay.y;
        const bool sum = a.kind != kNormLinf;
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        int c = i;
        for (; c + 15 * 64 < tiles; c += 16 * 64) {   // loads 16 at a time, sums in the slots' order
          double v[16];
#pragma unroll
          for (int q = 0; q < 16; ++q) v[q] = part[c + 64 * q];
#pragma unroll
          for (int q = 0; q < 16; ++q) acc[q & 3] = sum ? acc[q & 3] + v[q] : fmax(acc[q & 3], v[q]);
        }
#pragma unroll
        for (int q = 0; q < 16; ++q)
          if (c + 64 * q < tiles) acc[q & 3] = sum ? acc[q & 3] + part[c + 64 * q] : fmax(acc[q & 3], part[c + 64 * q]);
        double s = sum ? (acc[0] + acc[2]) + (acc[1] + acc[3]) : fmax(fmax(acc[0], acc[2]), fmax(acc[1], acc[3]));
        s = sum ? lane_tree<true>(s) : lane_tree<false>(s);
        if (i == 0) {
          const bool finite = stat_finite(s, a.kind);
          float n, r;
          stat_scale(s, a.kind, n, r);
          const size_t idx = (size_t)(p / nl) * a.L + lay.x;
          a.sumsq[idx] = s;
          a.norm[idx] = n;
          a.inv[idx] = r;
          if (!finite) atomicOr(a.status, kStatusNonFinite);
          if (n > 0.0f && n < kFltMin) atomicOr(a.status, kStatusTinyNorm);
          stat[p] = s;
          sinv[p] = r;
        }
      }
    } else {
      for (int p = t; p < P; p += kFitThreads) stat[p] = a.sumsq[at(p)];
    }
    for (int j = t; j < kGridPoints; j += kFitThreads) Ws[j] = 0ull;
    const int was = SRC == kFitBuckets ? a.type_exp[mtype] : 0;   // the scale that the statistics were gathered under
    __syncthreads();
    // exponent of the type's largest weight
    double mx = 0.0;
    bool bad = false;
    for (int p = 0; p < P; ++p) {
      if (!stat_finite(stat[p], a.kind)) bad = true;
      else mx = fmax(mx, weight_of(stat[p], a.kind));
    }
    const int found = (!bad && mx > 0.0) ? (int)((__double_as_longlong(mx) >> 52) & 0x7FF) - 1023 : kTypeSkip;
    const int ex = SRC == kFitBuckets ? was : found;
    if (SRC == kFitLayers) {
      if (t < P) swgt[t] = ex == kTypeSkip || sinv[t] == 0.0f ? 0ull : fit_weight(stat[t], a.kind, ex);
      __syncthreads();
#pragma unroll
      for (int p = 0; p < kFitLayerPairs; ++p) {
        if (p >= P) break;
        const size_t idx = at(p);
        const unsigned long long wfix = swgt[p];
        const float inv = sinv[p];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int b = t + h * kFitThreads;
          const unsigned int c = count[p][h];
          move_count(a, idx, b, c);
          if (wfix != 0ull && b != 0 && c != 0u) atomicAdd(&Ws[raw_bin_to_grid(b, inv)], wfix * (unsigned long long)c);
        }
      }
    } else if (ex != kTypeSkip) {
      for (int e = t; e < P * kGridPoints; e += kFitThreads) {
        const int p = e / kGridPoints, j = e - p * kGridPoints;
        const size_t idx = at(p);
        const unsigned long long c = reinterpret_cast<const unsigned long long *>(a.hist + idx * kHistBins)[j];
        if (c) atomicAdd(&Ws[j], c);
      }
    }
    __syncthreads();
    if (t == 0) a.type_exp[mtype] = found;
    for (int j = t; j < kGridPoints; j += kFitThreads) a.pooled[(size_t)mtype * kGridPoints + j] = Ws[j];
    if (ex == kTypeSkip) return;   // all-zero or non-finite vectors: the type keeps its levels
  }
  const unsigned long long *W = SRC == kFitPooled ? a.pooled + (size_t)mtype * kGridPoints : Ws;
  const int last = kGridPoints - 1;
  const double inf = __longlong_as_double(0x7FF0000000000000ll);
  for (int j = t; j < kGridPoints; j += kFitThreads) {
    const double wj = (double)W[j];
    const double mid = (j == last) ? 1.0 : (double)u2f(((unsigned int)(j + kGridBase) << 20) | (1u << 19));
    const double wm = wj * mid;
    wd[0][j] = wj;
    wd[1][j] = wm;
    wd[2][j] = wm * mid;
    gv[j] = (double)grid_value(j);
  }
  for (int j = t; j < 2 * kFitPad; j += kFitThreads) D[0][j] = inf;   // both rows: index 0, index `last`, the padding
  __syncthreads();
  // the three running sums, bin after bin: a chain of 257 dependent additions; their operands are read 16 at a time, a batch
  // ahead, into two sets of registers by turns.  Three lanes of one wave: an access to shared memory takes its time however
  // few lanes make it (in three waves the sums took 4.1 us, in one 2.7).
  if (t < 3) {
    const double *src = wd[t];
    double *dst = P[t];
    constexpr int N = 16;
    double p = 0.0, x[N], y[N];
    dst[0] = 0.0;
#pragma unroll
    for (int q = 0; q < N; ++q) x[q] = src[q];
#pragma unroll 1
    for (int j = 0; j < 256; j += 2 * N) {
#pragma unroll
      for (int q = 0; q < N; ++q) y[q] = src[j + N + q];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < N; ++q) { p = p + x[q]; dst[j + q + 1] = p; }
#pragma unroll
      for (int q = 0; q < N; ++q) x[q] = src[j + 2 * N + q];   // the last time: bin 256, then padding
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < N; ++q) { p = p + y[q]; dst[j + N + q + 1] = p; }
    }
    dst[kGridPoints] = p + x[0];
  }
  __syncthreads();
  if (P[0][kGridPoints] == 0.0) return;   // no mass on the grid at all: the type keeps its levels
  const auto row_at = [&](int j) { return FitRow{P[0][j], P[1][j], P[2][j], gv[j]}; };
  short *arg = a.dp_arg + a.dp_arg_off[mtype];
  const bool lds_arg = S <= kFitLdsPoints;   // candidates a are at most 254: a byte each, 255 for "none"
  if (S > 2) {
    // level 1 at grid index b: cost of the bins below g_b against the levels 0 and g_b
    for (int b = t; b < kGridPoints; b += kFitThreads)
      D[1][b] = (b >= 1 && b <= last - (S - 2)) ? (gv[b] * P[1][b] - P[2][b]) : inf;
    // this thread's couple (0: no work) and segment
    int couple = 0, seg = 0;
    {
      int g = 1, base = 0;
      while (base + kFitGroup * g <= t) { base += kFitGroup * g; ++g; }
      const int o = t - base, w = (int)(((float)o + 0.5f) * (1.0f / (float)g));   // o / g: o < 9 * 15
      const int q = kFitGroup * (g - 1) + 1 + w;
      if (q <= 128) { couple = q; seg = o - w * g; }
    }
    const int a0 = seg * kFitSeg;
    double cost[2][kFitSeg];
    {
      const int b1 = max(2 * couple, 1);
      const FitRow r0 = row_at(b1 - 1), r1 = row_at(b1);
      FitRow nx = row_at(a0);
#pragma unroll
      for (int j = 0; j < kFitSeg; ++j) {
        const int aa = a0 + j;
        const FitRow ra = nx;
        if (j + 1 < kFitSeg) nx = row_at(aa + 1);   // a row ahead; up to index 269, beyond the grid: not used
        asm volatile("" : : : "memory");            // all rows in flight would not fit the registers
        cost[0][j] = fit_cost(ra, r0);
        cost[1][j] = fit_cost(ra, r1);
        if (!(aa < b1 - 1)) cost[0][j] = inf;       // +infinity never wins a comparison below
        if (!(aa < b1 && b1 < last)) cost[1][j] = inf;   // (b = 256 is no place for an interior level)
        asm volatile("" : "+v"(cost[0][j]), "+v"(cost[1][j]));
      }
    }
    // the second step's index b, and which of its segments: four threads per b, four segments each
    const int cb = 1 + (t >> 2), cq = (cb + 1) >> 1, cg = (cq + kFitGroup - 1) / kFitGroup;   // cb's couple, its segments
    const int cs = 4 * (t & 3), cn = cb < last ? cg : 0;
    const int cfirst = kFitGroup * (cg * (cg - 1) / 2) + (cq - 1 - kFitGroup * (cg - 1)) * cg + cs;   // the thread of this one's first
    __syncthreads();
    for (int s = 2; s <= S - 2; ++s) {
      // D of the previous stage is +infinity wherever level s-1 cannot sit (in particular below index s-1), so the
      // candidates need no range test: min over a of D[a] + cost(a, b), the smallest a on equal cost
      const double *Dp = D[(s - 1) & 1] + a0;
      double *Dc = D[s & 1];
      if (couple != 0) {
        double best0 = inf, best1 = inf;
        int j0 = 0, j1 = 0;
        constexpr int N = 6;   // values of D that are read together, a batch ahead
        double d[2][N];
#pragma unroll
        for (int q = 0; q < N; ++q) d[0][q] = Dp[q];
#pragma unroll
        for (int j = 0; j < kFitSeg; ++j) {
          if (j % N == 0) {
            asm volatile("" : : : "memory");
            if (j + N < kFitSeg) {
#pragma unroll
              for (int q = 0; q < N; ++q) d[(j / N + 1) & 1][q] = Dp[j + N + q];
            }
            asm volatile("" : : : "memory");
          }
          const double c0 = d[(j / N) & 1][j % N] + cost[0][j], c1 = d[(j / N) & 1][j % N] + cost[1][j];
          // never a NaN: costs and D are finite or +infinity
          j0 = (c0 < best0) ? j : j0;
          best0 = fmin(best0, c0);
          j1 = (c1 < best1) ? j : j1;
          best1 = fmin(best1, c1);
          asm volatile("" : "+v"(j0), "+v"(j1));   // left to itself the compiler keeps all comparisons for later
        }
        pbest[2 * t] = best0;
        pbest[2 * t + 1] = best1;
        *reinterpret_cast<unsigned short *>(&pj[2 * t]) = (unsigned short)(j0 | j1 << 8);
      }
      __syncthreads();
      {
        // a chain of dependent instructions: short rather than few
        double ov[4];
        int oa[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const bool have = cs + q < cn;
          const int e = have ? 2 * (cfirst + q) + 1 - (cb & 1) : 0;
          ov[q] = pbest[e];
          oa[q] = (cs + q) * kFitSeg + pj[e];
          if (!have) ov[q] = inf;
        }
        // later segments hold larger a: they win only with a smaller cost
        if (ov[1] < ov[0]) { ov[0] = ov[1]; oa[0] = oa[1]; }
        if (ov[3] < ov[2]) { ov[2] = ov[3]; oa[2] = oa[3]; }
        if (ov[2] < ov[0]) { ov[0] = ov[2]; oa[0] = oa[2]; }
        double best = ov[0], o = quad_swap<0xB1>(best);   // and so between the four threads
        int at = oa[0], ob = __builtin_amdgcn_mov_dpp(at, 0xB1, 0xF, 0xF, true);
        if (o < best) { best = o; at = ob; }
        o = quad_swap<0x4E>(best);
        ob = __builtin_amdgcn_mov_dpp(at, 0x4E, 0xF, 0xF, true);
        if (o < best) { best = o; at = ob; }
        if ((t & 3) == 0 && cb < last) {
          if (!(cb >= s && cb <= last - (S - 1 - s))) best = inf;   // level s cannot sit here
          Dc[cb] = best;
          if (lds_arg) sarg[(s - 2) * 256 + cb] = (unsigned char)(best < inf ? at : 255);
          else arg[(size_t)s * kGridPoints + cb] = (short)(best < inf ? at : -1);
        }
      }
      __syncthreads();
    }
  }
  if (t < 64) {   // one wave: the last level (1.0) sits at grid index `last`
    int b = 0;
    if (S > 2) {
      // the smallest cost over its candidates (ties: smallest index), four neighbours a lane
      const double *Dp = D[(S - 2) & 1];
      const FitRow rb = row_at(last);
      double best = inf;
      b = 0x7FFFFFFF;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int aa = 4 * t + q;
        if (aa >= S - 2 && aa <= last - 1) {
          const double c = Dp[aa] + fit_cost(row_at(aa), rb);
          if (c < best) { best = c; b = aa; }
        }
      }
      // the smallest of all lanes' minima, and the first lane that has it: lanes hold increasing indices
      const unsigned long long lo = (unsigned long long)__double_as_longlong(lane_least(best));
      const double least = __longlong_as_double((long long)((unsigned long long)(unsigned int)__builtin_amdgcn_readfirstlane((int)(lo >> 32)) << 32 |
                                                            (unsigned int)__builtin_amdgcn_readfirstlane((int)lo)));
      b = __builtin_amdgcn_readlane(b, __ffsll(__ballot(best == least)) - 1);
    }
    if (t == 0) {
      slev[0] = 0.0f;
      slev[S - 1] = 1.0f;
      for (int s = S - 2; s >= 1; --s) {
        b = max(1, min(b, last - 1));   // cannot trigger for finite costs; keeps a corrupted table in bounds
        slev[s] = grid_value(b);
        if (s >= 2) b = lds_arg ? (int)sarg[(s - 2) * 256 + b] : (int)arg[(size_t)s * kGridPoints + b];
      }
    }
  }
  __syncthreads();
  for (int j = t; j < S; j += kFitThreads) a.lev[(size_t)mtype * kMaxPoints + j] = slev[j];
  build_tables(a, mtype, S, slev, reinterpret_cast<float *>(pbest));   // the segments' minima are no longer needed
}

// ------------------------------------------------------------------------------------------------ calibration
// Plain 128-bit copy of n float4: the known-size kernel that hardware byte counters are calibrated against.
__global__ void __launch_bounds__(kThreads) k_copy_f4(const float4 *__restrict__ src, float4 *__restrict__ dst, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) dst[i] = src[i];
}

// Streaming with the access type of the three big kernels: a workgroup takes tiles of 64 KiB; every thread issues 16
// nontemporal 128-bit loads per tile (1 KiB contiguous per wave and load) and STORES nontemporal 128-bit stores of
// values derived from them.  STORES = 0 measures the read-only ceiling (the norm pass), 16 a copy, values between
// the read/write mixes of the quantize pass (about 2) and of the decode + update pass (about 9).
template <int STORES>
__global__ void __launch_bounds__(kThreads) k_stream(const float *__restrict__ src, float *__restrict__ dst, size_t tiles,
                                                     float *sink) {
  const int t = threadIdx.x;
  float keep = 0.0f;
  for (size_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const size_t base = tile * kChunkCoords + (size_t)(t >> 6) * 16 * kBlockCoords + 4 * (t & 63);
    v4f q[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      const auto *lp = reinterpret_cast<const __attribute__((address_space(1))) v4f *>(as_global(src) + base + (size_t)s * kBlockCoords);
      q[s] = __builtin_nontemporal_load(lp);
    }
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      if (s < STORES) {
        auto *sp = reinterpret_cast<__attribute__((address_space(1))) v4f *>((__attribute__((address_space(1))) float *)dst + base + (size_t)s * kBlockCoords);
        __builtin_nontemporal_store(q[s], sp);
      } else {
        keep += (q[s].x + q[s].y) + (q[s].z + q[s].w);
      }
    }
  }
  if (keep == 12345.678f) sink[0] = keep;   // keeps the loads alive; practically never true
}

// ------------------------------------------------------------------------------------------------ staging
// Small host arrays (pointer tables, level values) reach the device as kernel arguments and are written to their device
// table by the kernel itself: no staging buffer, no copy engine, no host memory that must outlive the call.
// A launch takes a full pack or, if that is enough, a short one: a launch more is 2.6 to 4.7 us on the stream, words that are not needed
// cost the host 0.1 us.  (One node's call, its pointers in one launch instead of three or
// four: 9 tensors of 16 k entries in all 19.6 -> 13.0 us, 193 tensors 21.4 -> 14.7, 179 tensors of 151 M entries 248 -> 244.)
constexpr int kPackWords = 896, kPackShort = 128;
template <int N>
struct WordPack { unsigned int w[N]; };

template <int N>
__global__ void __launch_bounds__(N) k_stage_words(unsigned int *dst, WordPack<N> pack, int n) {
  const int t = threadIdx.x;
  if (t < n) dst[t] = pack.w[t];
}

// ------------------------------------------------------------------------------------------------ launchers
// Words [q, q + n) of src, then those of tail.
template <int N>
static void stage_pack(unsigned int *dst, const unsigned int *src, size_t nsrc, const unsigned int *tail, size_t q, int n, hipStream_t s) {
  WordPack<N> pack;
  const size_t own = q < nsrc ? (nsrc - q < (size_t)n ? nsrc - q : (size_t)n) : 0;
  if (own) memcpy(pack.w, src + q, own * sizeof(unsigned int));
  if (own < (size_t)n) memcpy(pack.w + own, tail + (q + own - nsrc), ((size_t)n - own) * sizeof(unsigned int));
  memset(pack.w + n, 0, (size_t)(N - n) * sizeof(unsigned int));
  hipLaunchKernelGGL(k_stage_words<N>, dim3(1), dim3(N), 0, s, dst + q, pack, n);
}

static hipError_t stage_words(void *dst_dev, const void *src_host, size_t nsrc, const void *tail_host, size_t ntail, hipStream_t s) {
  const unsigned int *src = static_cast<const unsigned int *>(src_host), *tail = static_cast<const unsigned int *>(tail_host);
  unsigned int *dst = static_cast<unsigned int *>(dst_dev);
  for (size_t q = 0, n = nsrc + ntail; q < n; q += kPackWords) {
    const int m = (int)(n - q < (size_t)kPackWords ? n - q : (size_t)kPackWords);
    if (m <= kPackShort) stage_pack<kPackShort>(dst, src, nsrc, tail, q, m, s);
    else stage_pack<kPackWords>(dst, src, nsrc, tail, q, m, s);
  }
  return hipGetLastError();
}

hipError_t launch_stage_words(void *dst_dev, const void *src_host, size_t nwords, hipStream_t s) {
  return stage_words(dst_dev, src_host, nwords, nullptr, 0, s);
}

hipError_t launch_stage_pointers(void **dst_dev, const void *const *src_host, size_t n, hipStream_t s) {
  static_assert(sizeof(void *) == 2 * sizeof(unsigned int), "a pointer is two words");
  return launch_stage_words(dst_dev, src_host, 2 * n, s);
}

hipError_t launch_stage_node(void **dst_dev, const void *const *src_host, size_t n, const void *msg, const void *prev, hipStream_t s) {
  const void *const tail[2] = {msg, prev};
  return stage_words(dst_dev, src_host, 2 * n, tail, 4, s);
}

hipError_t launch_copy(const void *src, void *dst, size_t bytes, hipStream_t s) {
  const size_t n = bytes / 16;
  if (n == 0) return hipSuccess;
  const size_t want = (n + kThreads * 4 - 1) / (kThreads * 4);
  const unsigned int blocks = (unsigned int)(want < 1048576 ? want : 1048576);
  hipLaunchKernelGGL(k_copy_f4, dim3(blocks), dim3(kThreads), 0, s, reinterpret_cast<const float4 *>(src),
                     reinterpret_cast<float4 *>(dst), n);
  return hipGetLastError();
}

hipError_t launch_stream(const void *src, void *dst, size_t bytes, int stores, void *sink, hipStream_t s) {
  const size_t tiles = bytes / (4 * (size_t)kChunkCoords);
  if (tiles == 0) return hipSuccess;
  const dim3 grid((unsigned int)(tiles < 65536 ? tiles : 65536)), block(kThreads);
  const float *a = static_cast<const float *>(src);
  float *b = static_cast<float *>(dst), *k = static_cast<float *>(sink);
  switch (stores) {
    case 0: hipLaunchKernelGGL((k_stream<0>), grid, block, 0, s, a, b, tiles, k); break;
    case 1: hipLaunchKernelGGL((k_stream<1>), grid, block, 0, s, a, b, tiles, k); break;
    case 2: hipLaunchKernelGGL((k_stream<2>), grid, block, 0, s, a, b, tiles, k); break;
    case 4: hipLaunchKernelGGL((k_stream<4>), grid, block, 0, s, a, b, tiles, k); break;
    case 8: hipLaunchKernelGGL((k_stream<8>), grid, block, 0, s, a, b, tiles, k); break;
    case 16: hipLaunchKernelGGL((k_stream<16>), grid, block, 0, s, a, b, tiles, k); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_zero_stats(unsigned int *hist, double *stat, size_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_zero_stats, dim3((unsigned int)n), dim3(kThreads), 0, s, hist, stat);
  return hipGetLastError();
}

hipError_t launch_zero_u32(unsigned int *p, size_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const unsigned int blocks = (unsigned int)((n + 1023) / 1024 < 65535 ? (n + 1023) / 1024 : 65535);
  hipLaunchKernelGGL(k_zero_u32, dim3(blocks), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

template <int KIND>
static void launch_sumsq_kind(const Dev &a, bool with_hist, hipStream_t s) {
  const dim3 runs(a.GS, a.nnodes), tiles(a.NT, a.nnodes), block(kThreads);
  // Without a histogram nothing is kept per run, and single tiles are the most even load.  Only where they would fill the
  // device one and a half to two times (the second fill's waves come and go with too few loads in flight) fewer, longer
  // workgroups are a little faster.  us of the pass with runs / single tiles, K = 1 and K = 8: 512 tiles 20 / 10 and - ; 2048
  // 31 / 27; 2560 38 / 32 and 38 / 32; 2800 39 / 35 and 34 / 35; 3096 39 / 37 and 36 / 38; 3300 38 / 40 and 39 / 40; 3600 45 / 43
  // and 41 / 44; 3900 44 / 44 and 45 / 45; 4600 57 / 52 and 58 / 52; 8192 90 / 88 and 87 / 87; 32768 323 / 322.
  const long long n = (long long)a.NT * a.nnodes;
  const bool long_runs = a.stiles != nullptr && n > 4 * kTaperWorkgroups / 3 && n < 15 * kTaperWorkgroups / 8;
  if (with_hist) {
    hipLaunchKernelGGL((k_sumsq<true, KIND>), runs, block, 0, s, a);
  } else if (long_runs) {
    hipLaunchKernelGGL((k_sumsq<false, KIND>), runs, block, 0, s, a);
  } else {
    Dev b = a;
    b.stiles = nullptr;
    hipLaunchKernelGGL((k_sumsq<false, KIND>), tiles, block, 0, s, b);
  }
}

hipError_t launch_sumsq(const Dev &a, bool with_hist, hipStream_t s) {
  if (a.GS == 0 || a.nnodes == 0) return hipSuccess;
  if (a.kind == kNormL2) launch_sumsq_kind<kNormL2>(a, with_hist, s);
  else if (a.kind == kNormL1) launch_sumsq_kind<kNormL1>(a, with_hist, s);
  else launch_sumsq_kind<kNormLinf>(a, with_hist, s);
  return hipGetLastError();
}

hipError_t launch_norm_finalize(const Dev &a, hipStream_t s) {
  hipLaunchKernelGGL(k_norm_finalize, dim3(a.layers ? a.NL : a.L, a.nnodes), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

template <int C1, bool PREV>
static void launch_quantize_tables(const Dev &a, hipStream_t s) {
  constexpr bool bins = quantize_bins_width(PREV, C1), bytes = quantize_bytes_width(PREV, C1);
  static_assert(bins || bytes, "a form for every width");
  const dim3 grid(a.NT, a.nnodes), block(kThreads);
  if constexpr (bins) {
    if (!bytes || quantize_bins((long long)a.NT * a.nnodes, PREV, C1)) {
      hipLaunchKernelGGL((k_quantize<C1, PREV, true>), grid, block, 0, s, a);
      return;
    }
  }
  if constexpr (bytes) hipLaunchKernelGGL((k_quantize<C1, PREV, false>), grid, block, 0, s, a);
}

// planes_mask: bit p set when some layer has code width p (2..9); one launch per width present.
template <int C1>
static void launch_quantize_width(const Dev &a, hipStream_t s) {
  const dim3 block(kThreads);
  const bool prev = a.prev != nullptr;   // no node has a previous message: the kernels skip that half of the work
  if (a.scope == kScopeBucket) {
    const dim3 grid(a.GS, a.nnodes);   // runs of tiles
    if (a.kind == kNormL2) {
      if (prev) hipLaunchKernelGGL((k_quantize_b<C1, true, kNormL2>), grid, block, 0, s, a);
      else hipLaunchKernelGGL((k_quantize_b<C1, false, kNormL2>), grid, block, 0, s, a);
    } else if (a.kind == kNormL1) {
      if (prev) hipLaunchKernelGGL((k_quantize_b<C1, true, kNormL1>), grid, block, 0, s, a);
      else hipLaunchKernelGGL((k_quantize_b<C1, false, kNormL1>), grid, block, 0, s, a);
    } else {
      if (prev) hipLaunchKernelGGL((k_quantize_b<C1, true, kNormLinf>), grid, block, 0, s, a);
      else hipLaunchKernelGGL((k_quantize_b<C1, false, kNormLinf>), grid, block, 0, s, a);
    }
  } else {
    if (prev) launch_quantize_tables<C1, true>(a, s);
    else launch_quantize_tables<C1, false>(a, s);
  }
}

hipError_t launch_quantize(const Dev &a, unsigned int planes_mask, hipStream_t s) {
  if (a.NT == 0 || a.nnodes == 0) return hipSuccess;
  if (planes_mask & (1u << 2)) launch_quantize_width<2>(a, s);
  if (planes_mask & (1u << 3)) launch_quantize_width<3>(a, s);
  if (planes_mask & (1u << 4)) launch_quantize_width<4>(a, s);
  if (planes_mask & (1u << 5)) launch_quantize_width<5>(a, s);
  if (planes_mask & (1u << 6)) launch_quantize_width<6>(a, s);
  if (planes_mask & (1u << 7)) launch_quantize_width<7>(a, s);
  if (planes_mask & (1u << 8)) launch_quantize_width<8>(a, s);
  if (planes_mask & (1u << 9)) launch_quantize_width<9>(a, s);
  return hipGetLastError();
}

template <int C1>
static void launch_small_width(const Dev &a, hipStream_t s) {
  const dim3 grid(a.G, a.nnodes), block(kSmallThreads);
  if (a.prev != nullptr) hipLaunchKernelGGL((k_quantize_small<C1, true>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((k_quantize_small<C1, false>), grid, block, 0, s, a);
}

hipError_t launch_quantize_small(const Dev &a, unsigned int planes_mask, hipStream_t s) {
  switch (planes_mask) {   // one code width in the model
    case 1u << 2: launch_small_width<2>(a, s); break;
    case 1u << 3: launch_small_width<3>(a, s); break;
    case 1u << 4: launch_small_width<4>(a, s); break;
    case 1u << 5: launch_small_width<5>(a, s); break;
    case 1u << 6: launch_small_width<6>(a, s); break;
    case 1u << 7: launch_small_width<7>(a, s); break;
    case 1u << 8: launch_small_width<8>(a, s); break;
    case 1u << 9: launch_small_width<9>(a, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int C1>
static void launch_held_width(const Dev &a, hipStream_t s) {
  const dim3 grid(a.NT, a.nnodes), block(kThreads);
  if (a.prev != nullptr) hipLaunchKernelGGL((k_quantize_held<C1, true>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((k_quantize_held<C1, false>), grid, block, 0, s, a);
}

hipError_t launch_quantize_held(const Dev &a, unsigned int planes_mask, hipStream_t s) {
  if (a.NT == 0 || a.nnodes == 0) return hipSuccess;
  if (planes_mask & (1u << 2)) launch_held_width<2>(a, s);
  if (planes_mask & (1u << 3)) launch_held_width<3>(a, s);
  if (planes_mask & (1u << 4)) launch_held_width<4>(a, s);
  if (planes_mask & (1u << 5)) launch_held_width<5>(a, s);
  if (planes_mask & (1u << 6)) launch_held_width<6>(a, s);
  if (planes_mask & (1u << 7)) launch_held_width<7>(a, s);
  if (planes_mask & (1u << 8)) launch_held_width<8>(a, s);
  if (planes_mask & (1u << 9)) launch_held_width<9>(a, s);
  return hipGetLastError();
}

hipError_t launch_delta_finalize(const Dev &a, hipStream_t s) {
  // the layers go into grid.y: up to 65534 of them (the caller sees to it)
  const int more = a.clear_exch ? a.clear_exch : a.hist_old ? a.L : 0;
  hipLaunchKernelGGL(k_delta_finalize, dim3(a.nnodes, (unsigned int)(1 + more)), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_norm_vector(const Dev &a, hipStream_t s) {
  hipLaunchKernelGGL(k_norm_vector, dim3(a.nnodes), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_step_scalars(const Dev &a, hipStream_t s) {
  hipLaunchKernelGGL(k_step_scalars, dim3(1), dim3(64), 0, s, a);
  return hipGetLastError();
}

template <int C1, int MODE, bool BUCKET, int NB, bool EARLY>
static void launch_decode_blocks(const Dev &a, size_t lds_bytes, hipStream_t s) {
  // short workgroups: two octets, four where the K decode tables are large enough to limit the workgroups per CU
  const int oct = MODE == kDecodeUpdateAlt ? 8 : (lds_bytes > 8192 && NB > 2) ? 4 : kDecodeOctets;
  const dim3 grid((unsigned int)a.G * (8 / oct)), block(64 * oct * 8 / NB);
  hipLaunchKernelGGL((k_decode<C1, MODE, BUCKET, NB, EARLY>), grid, block, lds_bytes, s, a);
}

template <int C1, int MODE, bool BUCKET>
static void launch_decode_mode(const Dev &a, size_t lds_bytes, hipStream_t s) {
  if constexpr (MODE == kDecodeUpdateAlt) {
    if (alt_blocks(a.G, a.K, BUCKET, C1) == 16) launch_decode_blocks<C1, MODE, BUCKET, 16, false>(a, lds_bytes, s);
    else launch_decode_blocks<C1, MODE, BUCKET, 8, C1 <= 6>(a, lds_bytes, s);
  } else if constexpr (MODE == kDecodeUpdateScalars) {
    launch_decode_blocks<C1, MODE, BUCKET, 2, true>(a, lds_bytes, s);   // few tiles
  } else {
    switch (decode_blocks(a.G, a.K, MODE, BUCKET, C1)) {
      case 2: launch_decode_blocks<C1, MODE, BUCKET, 2, true>(a, lds_bytes, s); return;
      case 4: launch_decode_blocks<C1, MODE, BUCKET, 4, true>(a, lds_bytes, s); return;
    }
    if constexpr (MODE == kDecodeMean && mean_early(1, 1, BUCKET, C1)) {
      if (mean_early(a.G, a.K, BUCKET, C1)) { launch_decode_blocks<C1, MODE, BUCKET, 8, true>(a, lds_bytes, s); return; }
    }
    launch_decode_blocks<C1, MODE, BUCKET, 8, false>(a, lds_bytes, s);
  }
}

template <int C1, bool BUCKET>
static void launch_decode_scope(const Dev &a, int mode, size_t lds_bytes, hipStream_t s) {
  if (mode == kDecodeExtrapolate) launch_decode_mode<C1, kDecodeExtrapolate, BUCKET>(a, lds_bytes, s);
  else if (mode == kDecodeUpdateAlt) launch_decode_mode<C1, kDecodeUpdateAlt, BUCKET>(a, lds_bytes, s);
  else if (mode == kDecodeUpdate) launch_decode_mode<C1, kDecodeUpdate, BUCKET>(a, lds_bytes, s);
  else if (mode == kDecodeUpdateScalars) launch_decode_mode<C1, kDecodeUpdateScalars, BUCKET>(a, lds_bytes, s);
  else launch_decode_mode<C1, kDecodeMean, BUCKET>(a, lds_bytes, s);
}

template <int C1>
static void launch_decode_width(const Dev &a, int mode, size_t lds_bytes, hipStream_t s) {
  if (a.scope == kScopeBucket) launch_decode_scope<C1, true>(a, mode, lds_bytes, s);
  else launch_decode_scope<C1, false>(a, mode, lds_bytes, s);
}

hipError_t launch_decode(const Dev &a, int mode, unsigned int planes_mask, hipStream_t s) {
  if (a.G == 0) return hipSuccess;
  if (planes_mask & (1u << 2)) launch_decode_width<2>(a, mode, (size_t)a.K * 4 * sizeof(float), s);
  if (planes_mask & (1u << 3)) launch_decode_width<3>(a, mode, (size_t)a.K * 8 * sizeof(float), s);
  if (planes_mask & (1u << 4)) launch_decode_width<4>(a, mode, (size_t)a.K * 16 * sizeof(float), s);
  if (planes_mask & (1u << 5)) launch_decode_width<5>(a, mode, (size_t)a.K * 32 * sizeof(float), s);
  if (planes_mask & (1u << 6)) launch_decode_width<6>(a, mode, (size_t)a.K * 64 * sizeof(float), s);
  if (planes_mask & (1u << 7)) launch_decode_width<7>(a, mode, (size_t)a.K * 128 * sizeof(float), s);
  if (planes_mask & (1u << 8)) launch_decode_width<8>(a, mode, (size_t)a.K * 256 * sizeof(float), s);
  if (planes_mask & (1u << 9)) launch_decode_width<9>(a, mode, (size_t)a.K * 512 * sizeof(float), s);
  return hipGetLastError();
}

template <int C1>
static void launch_index_hist_width(const Dev &a, hipStream_t s) {
  const dim3 grid(a.GS, a.K), block(kThreads);
  const size_t lds = (size_t)(1 << (C1 - 1)) * 64 * sizeof(unsigned int);
  if (a.scope == kScopeBucket) hipLaunchKernelGGL((k_index_hist<C1, true>), grid, block, lds, s, a);
  else hipLaunchKernelGGL((k_index_hist<C1, false>), grid, block, lds, s, a);
}

hipError_t launch_index_hist(const Dev &a, unsigned int planes_mask, hipStream_t s) {
  if (a.G == 0) return hipSuccess;
  if (planes_mask & (1u << 2)) launch_index_hist_width<2>(a, s);
  if (planes_mask & (1u << 3)) launch_index_hist_width<3>(a, s);
  if (planes_mask & (1u << 4)) launch_index_hist_width<4>(a, s);
  if (planes_mask & (1u << 5)) launch_index_hist_width<5>(a, s);
  if (planes_mask & (1u << 6)) launch_index_hist_width<6>(a, s);
  if (planes_mask & (1u << 7)) launch_index_hist_width<7>(a, s);
  if (planes_mask & (1u << 8)) launch_index_hist_width<8>(a, s);
  if (planes_mask & (1u << 9)) launch_index_hist_width<9>(a, s);
  return hipGetLastError();
}

hipError_t launch_alt_scalars(const Dev &a, hipStream_t s) {
  hipLaunchKernelGGL(k_alt_scalars, dim3(1), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_alt_finalize(const Dev &a, hipStream_t s) {
  hipLaunchKernelGGL(k_alt_finalize, dim3(1), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_bucket_max(const Dev &a, hipStream_t s) {
  if (a.GS == 0) return hipSuccess;
  hipLaunchKernelGGL(k_bucket_max, dim3(a.GS, a.K), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_bucket_hist(const Dev &a, hipStream_t s) {
  if (a.GS == 0) return hipSuccess;
  hipLaunchKernelGGL(k_bucket_hist, dim3(a.GS, a.K), dim3(kThreads), 0, s, a);
  hipLaunchKernelGGL(k_fit_pool_b, dim3(a.L, a.K), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_fit_pool_b(const Dev &a, hipStream_t s) {
  hipLaunchKernelGGL(k_fit_pool_b, dim3(a.L, a.K), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_fit_typemax(const Dev &a, hipStream_t s) {
  hipLaunchKernelGGL(k_fit_typemax, dim3(a.M), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_fit_pool(const Dev &a, hipStream_t s) {
  hipLaunchKernelGGL(k_fit_pool, dim3(a.L, a.K), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_fit_dp(const Dev &a, int source, hipStream_t s) {
  const dim3 grid(a.M), block(kFitThreads);
  if (source == kFitLayers) hipLaunchKernelGGL((k_fit_dp<kFitLayers>), grid, block, 0, s, a);
  else if (source == kFitBuckets) hipLaunchKernelGGL((k_fit_dp<kFitBuckets>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((k_fit_dp<kFitPooled>), grid, block, 0, s, a);
  return hipGetLastError();
}

hipError_t launch_build_tables(const Dev &a, int type, hipStream_t s) {
  hipLaunchKernelGGL(k_build_tables, dim3(1), dim3(kThreads), 0, s, a, type);
  return hipGetLastError();
}

}  // namespace qoda
