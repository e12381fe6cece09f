// Offline calibration (Sec. 3.1 "Offline Channel Assignment Strategy";
// Def. 1, eq. quantization-threshold; Appendix C.2 "Derivations"): from
// calibration activations X [L, K] compute each channel's mean |X|, the
// stable ascending order sigma of those means, and the group sizes given by
// the thresholds
//   T(n) = 2^b * 2^(n-1) / q_max * max|X| / 254
// of E2M1 (n = 4) and the 6-bit format (n = 6).  A channel belongs to G4 when
// its mean is <= T(4), to G6 when it is <= T(6), else to G8; each count is
// rounded down to a multiple of 32, so channels only ever move to a wider
// group.
//
// Stream-ordered launches, deterministic for a given (L, K):
//   1. column sums: each workgroup adds |x| in fp64 over one 512-channel tile
//      and one fixed chunk of rows (HBM-bound, 2 bytes read per element) and
//      writes its partial sums and its largest |x|.  About one workgroup per
//      CU streams best: more concurrent row streams lose DRAM locality;
//   2. means: each channel adds its chunk partials in a fixed order, / L.  At
//      most sizes (see kFuseK) the rank workgroups do this for the channels that
//      they compare, again in each workgroup, which is less than a launch of its
//      own and the wait for it;
//   3. rank: workgroup (jb, sl) compares 256 channels with a 256-channel
//      slice of the means and stores, per channel, how many of them sort
//      before it under the strict order (mean, index); the workgroups of
//      slice 0 also evaluate the thresholds against the largest |x| and count
//      their channels' groups;
//   4. place: rank[j] = the sum of j's slice counts, sigma[rank[j]] = j, and
//      workgroup 0 sums the group counts into the split.
// Measured, whole call (us, separate means -> fused): 32768 x 4096 59.2 -> 54.7
// (column sums 41.5), 2048 x 4096 22.2 -> 18.8, 300 x 1024 21.8 -> 16.4, 32768 x
// 5120 73.3 -> 71.6, but 16384 x 14336 106 -> 120 and 2000 x 32768 114 -> 195
// (every mean formed K / 256 times).
// No atomics: every result is written by exactly one thread.
#include <mutex>

#include "kernels.hpp"

namespace mm {

// Workspace of mm_calibrate_no_alloc: every GPU the library runs on holds
// its own copy.  In host code this name is only a stand-in for the symbol
// (not a device address): kernels get the address calibrate_scratch()
// looked up.  No kernel reads a workspace byte before writing it, so the
// contents a previous call left need no clearing.
static __device__ __align__(256) uint8_t scratch[kCalibScratchBytes];

namespace {

constexpr int kSumWaves = 4;               // waves per column-sum workgroup
constexpr int kLaneCols = 8;               // channels per lane (one 16-byte load)
constexpr int kTileCols = 64 * kLaneCols;  // channels per column-sum workgroup
constexpr int kMeanChains = 16;            // partial sums of a mean (one chunk subset each)
constexpr int kRankThreads = 256;          // channels per rank workgroup
// Where the rank kernel forms the means: up to kFuseK channels, or up to kFuseFewK
// with at most kFuseFew row chunks (us, separate / fused: 1461 x 5696 26.9 / 27.4,
// 2046 x 6720 29.1 / 31.0, 1024 x 8192 25.3 / 29.6, but 601 x 5568 25.4 / 22.3, 716 x
// 6208 27.7 / 26.1, 83 x 7264 25.7 / 23.5); not at up to kSlowK channels with more
// than three chunks per chain, whose few threads would add them one after the
// other (9314 x 32 15.4 / 17.2, 7507 x 64 15.1 / 16.1; 7250 x 128 16.2 / 15.1).
constexpr int kFuseK = 5632, kFuseFewK = 7680, kFuseFew = 12, kSlowK = 64;
constexpr int kRankSlice = kCalibSlice;    // means compared per rank workgroup
constexpr uint32_t kF32Inf = 0x7F800000u;  // |x| fp32 patterns at or above this are Inf or NaN

// |x| of the two bf16 values in a 32-bit word, as fp32 bit patterns (a bf16
// is the top half of an fp32; clearing the sign bit gives |x|).  Their
// conversion to fp64 is exact: the kernels keep fp32 denormals (the default
// floating-point mode), so subnormal inputs are not flushed.
__device__ __forceinline__ void add_word(double* s, uint32_t& mx, uint32_t w) {
  const uint32_t lo = (w << 16) & 0x7FFF0000u, hi = w & 0x7FFF0000u;
  s[0] += (double)__uint_as_float(lo);
  s[1] += (double)__uint_as_float(hi);
  mx = max(mx, max(lo, hi));
}

// 16 bytes of X, non-temporal: every byte is read once, so its L2 lines go
// first (32768 x 14336: 191 -> 172 us for the whole call).
typedef unsigned int u32x4_nt __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load_x16(const uint16_t* p) {
  const u32x4_nt v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_nt*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ void add_row(double* s, uint32_t& mx, uint4 v) {
  add_word(s + 0, mx, v.x);
  add_word(s + 2, mx, v.y);
  add_word(s + 4, mx, v.z);
  add_word(s + 6, mx, v.w);
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  for (int o = 32; o > 0; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o));
  return v;
}

__device__ __forceinline__ int wave_sum(int v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// Largest |x| of the whole input (fp32 bit pattern), from the column-sum
// workgroups' maxima; every thread of the workgroup gets it, the first
// kRankThreads look for it.
__device__ uint32_t input_amax(const CalibArgs& a, uint32_t* lds4) {
  uint32_t m = 0u;
  if (threadIdx.x < kRankThreads)
    for (int i = threadIdx.x; i < a.nmax; i += kRankThreads) m = max(m, a.wgmax[i]);
  m = wave_max(m);
  if (threadIdx.x < kRankThreads && (threadIdx.x & 63) == 0) lds4[threadIdx.x >> 6] = m;
  __syncthreads();
  return max(max(lds4[0], lds4[1]), max(lds4[2], lds4[3]));
}

// Mean |x| of channel j: chain w adds the partials of chunks w, w + 16, ... in
// order, the chains are added in order.
__device__ __forceinline__ double channel_mean(const CalibArgs& a, int j) {
  const double* p = a.partial + j;
  double s[kMeanChains];
#pragma unroll
  for (int w = 0; w < kMeanChains; ++w) s[w] = w < a.nchunks ? p[(int64_t)w * a.K] : 0.0;
  for (int c0 = kMeanChains; c0 < a.nchunks; c0 += kMeanChains) {
    double v[kMeanChains];
#pragma unroll
    for (int w = 0; w < kMeanChains; ++w) v[w] = c0 + w < a.nchunks ? p[(int64_t)(c0 + w) * a.K] : 0.0;
#pragma unroll
    for (int w = 0; w < kMeanChains; ++w) s[w] += v[w];
  }
#pragma unroll
  for (int w = 1; w < kMeanChains; ++w) s[0] += s[w];
  return s[0] / (double)a.rows;
}

// How many of the n means in `tile` (channels base .. base+n-1, n a multiple
// of 32) sort before channel j with mean mj.  MODE 0: every tile channel
// has a larger index than j (ties do not count); MODE 1: every one has a
// smaller index (ties count); MODE 2: the slice holds j, jl = j - base.
template <int MODE>
__device__ __forceinline__ int count_before(const double* tile, int n, double mj, int jl) {
  int cnt = 0;
  for (int i0 = 0; i0 < n; i0 += 32) {
#pragma unroll
    for (int k = 0; k < 32; k += 2) {
      const double2 v = *reinterpret_cast<const double2*>(tile + i0 + k);
      if constexpr (MODE == 0) cnt += (v.x < mj) + (v.y < mj);
      else if constexpr (MODE == 1) cnt += (v.x <= mj) + (v.y <= mj);
      else  // bitwise, not short-circuit: no per-lane branches
        cnt += ((int)(v.x < mj) | ((int)(v.x == mj) & (int)(i0 + k < jl))) +
               ((int)(v.y < mj) | ((int)(v.y == mj) & (int)(i0 + k + 1 < jl)));
    }
  }
  return cnt;
}

__global__ __launch_bounds__(64 * kSumWaves) void colsum_kernel(CalibArgs a) {
  __shared__ double red[kSumWaves - 1][kLaneCols][64];
  __shared__ uint32_t wmax[kSumWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c0 = blockIdx.x * kTileCols + lane * kLaneCols;
  const int64_t r0 = (int64_t)blockIdx.y * a.chunk_rows;
  const int64_t r1 = min(a.rows, r0 + a.chunk_rows);
  double s[kLaneCols];
  for (int i = 0; i < kLaneCols; ++i) s[i] = 0.0;
  uint32_t mx = 0u;
  if (c0 < a.K) {
    // wave w adds rows r0 + w, r0 + w + 4, ... in increasing order
    const uint16_t* p = a.x + c0;
    int64_t r = r0 + wave;
    constexpr int U = 8;
    for (; r + (U - 1) * kSumWaves < r1; r += U * kSumWaves) {
      uint4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = load_x16(p + (r + u * kSumWaves) * a.ldx);
#pragma unroll
      for (int u = 0; u < U; ++u) add_row(s, mx, v[u]);
    }
    for (; r < r1; r += kSumWaves) add_row(s, mx, load_x16(p + r * a.ldx));
  }
  mx = wave_max(mx);
  if (lane == 0) wmax[wave] = mx;
  // fixed-order combine of the four waves' partial sums
  if (wave > 0)
    for (int i = 0; i < kLaneCols; ++i) red[wave - 1][i][lane] = s[i];
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t m = wmax[0];
    for (int w = 1; w < kSumWaves; ++w) m = max(m, wmax[w]);
    a.wgmax[blockIdx.y * gridDim.x + blockIdx.x] = m;
  }
  if (wave != 0 || c0 >= a.K) return;
  for (int w = 0; w < kSumWaves - 1; ++w)
    for (int i = 0; i < kLaneCols; ++i) s[i] += red[w][i][lane];
  double2* out = reinterpret_cast<double2*>(a.partial + (int64_t)blockIdx.y * a.K + c0);
  for (int i = 0; i < kLaneCols / 2; ++i) out[i] = make_double2(s[2 * i], s[2 * i + 1]);
}

__global__ __launch_bounds__(64 * kMeanChains) void mean_kernel(CalibArgs a) {
  __shared__ double red[kMeanChains][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;  // a wavefront per chain
  const int j = blockIdx.x * 64 + lane;
  double s = 0.0;
  if (j < a.K)
    for (int c = wave; c < a.nchunks; c += kMeanChains) s += a.partial[(int64_t)c * a.K + j];
  red[wave][lane] = s;
  __syncthreads();
  if (wave != 0 || j >= a.K) return;
  for (int w = 1; w < kMeanChains; ++w) s += red[w][lane];
  a.mean[j] = s / (double)a.rows;
}

// kParts: threads per channel, each comparing with its part of the slice (the
// chain of comparisons sets the kernel's length while there are few
// workgroups).  kFuse: form the means here.
template <int kParts, bool kFuse>
__global__ __launch_bounds__(kRankThreads * kParts) void rank_kernel(CalibArgs a) {
  static_assert(!kFuse || kParts >= 2, "part 0 forms the channels' means, part 1 the slice's");
  __shared__ __align__(16) double tile[kRankSlice];
  __shared__ double mean[kFuse ? kRankThreads : 1];
  __shared__ int part_cnt[kParts][kRankThreads];
  __shared__ uint32_t lds4[4];
  __shared__ int c4[4], c6[4];
  const int tl = threadIdx.x % kRankThreads, part = threadIdx.x / kRankThreads;
  const int jb = blockIdx.x * kRankThreads, j = jb + tl;
  const int base = blockIdx.y * kRankSlice;
  const int n = min(kRankSlice, a.K - base);
  double mj;
  if constexpr (kFuse) {
    if (part == 0) mean[tl] = j < a.K ? channel_mean(a, j) : 0.0;
    else if (part == 1 && tl < n) tile[tl] = channel_mean(a, base + tl);
    __syncthreads();
    mj = mean[tl];
  } else {
    mj = j < a.K ? a.mean[j] : 0.0;
    if (part == 0 && tl < n) tile[tl] = a.mean[base + tl];
    __syncthreads();
  }
  // this part's share of the slice, whole 32s (n is a multiple of 32)
  const int per = (n / 32 + kParts - 1) / kParts * 32;
  const int lo = min(n, part * per), m = min(n, lo + per) - lo;
  int cnt;
  if (jb + kRankThreads <= base) cnt = count_before<0>(tile + lo, m, mj, 0);  // uniform per workgroup
  else if (jb >= base + n) cnt = count_before<1>(tile + lo, m, mj, 0);
  else cnt = count_before<2>(tile + lo, m, mj, j - base - lo);
  if constexpr (kParts > 1) {
    part_cnt[part][tl] = cnt;
    __syncthreads();
#pragma unroll
    for (int p = 1; p < kParts; ++p) cnt += part_cnt[p][tl];  // (of use in part 0)
  }
  if (part == 0 && j < a.K) a.slice_counts[(int64_t)blockIdx.y * a.K + j] = cnt;
  if (blockIdx.y != 0) return;
  // group counts of this workgroup's channels (slice 0 only: once per channel)
  const uint32_t amax = input_amax(a, lds4);
  // thresholds, in the order of operations of their definition
  const double tx = (double)__uint_as_float(amax);
  const double t4 = 2.0 * 8.0 / 6.0 * (tx / 254.0);                                  // E2M1: b 1, q_max 6
  const double t6 = a.fp6_e2m3 ? 2.0 * 32.0 / 7.5 * (tx / 254.0)                     // E2M3: b 1, q_max 7.5
                               : 8.0 * 32.0 / 28.0 * (tx / 254.0);                   // E3M2: b 3, q_max 28
  const bool in4 = j < a.K && mj <= t4;
  const bool in6 = j < a.K && !in4 && mj <= t6;
  const int n4 = wave_sum(in4), n6 = wave_sum(in6);
  if (part == 0 && (threadIdx.x & 63) == 0) {
    c4[threadIdx.x >> 6] = n4;
    c6[threadIdx.x >> 6] = n6;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    a.counts[2 * blockIdx.x] = c4[0] + c4[1] + c4[2] + c4[3];
    a.counts[2 * blockIdx.x + 1] = c6[0] + c6[1] + c6[2] + c6[3];
  }
}

__global__ __launch_bounds__(kRankThreads) void place_kernel(CalibArgs a) {
  __shared__ uint32_t lds4[4];
  const bool finite = input_amax(a, lds4) < kF32Inf;
  const int j = blockIdx.x * kRankThreads + threadIdx.x;
  if (j < a.K) {
    const int nslices = (a.K + kRankSlice - 1) / kRankSlice;
    int rank = 0;
#pragma unroll 8
    for (int sl = 0; sl < nslices; ++sl) rank += a.slice_counts[(int64_t)sl * a.K + j];
    a.perm[finite ? rank : j] = j;
  }
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  if (!finite) {
    a.split[0] = a.split[1] = a.split[2] = -1;
    return;
  }
  int n4 = 0, n6 = 0;
  for (int b = 0; b < (int)gridDim.x; ++b) {
    n4 += a.counts[2 * b];
    n6 += a.counts[2 * b + 1];
  }
  const int p4 = n4 / 32 * 32, p46 = (n4 + n6) / 32 * 32;
  a.split[0] = p4;
  a.split[1] = p46 - p4;
  a.split[2] = a.K - p46;
}

}  // namespace

hipError_t calibrate_scratch(void** ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p || ((uintptr_t)p & 255u)) return hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

hipError_t launch_calibrate(const CalibArgs& a, hipStream_t stream) {
  const int tiles = (a.K + kTileCols - 1) / kTileCols;
  hipLaunchKernelGGL(colsum_kernel, dim3(tiles, a.nchunks), dim3(64 * kSumWaves), 0, stream, a);
  const dim3 ranks((a.K + kRankThreads - 1) / kRankThreads, (a.K + kRankSlice - 1) / kRankSlice);
  const bool slow = a.K <= kSlowK && a.nchunks > 3 * kMeanChains;
  if (!slow && a.K <= (a.nchunks <= kFuseFew ? kFuseFewK : kFuseK)) {
    hipLaunchKernelGGL((rank_kernel<4, true>), ranks, dim3(kRankThreads * 4), 0, stream, a);
  } else {
    hipLaunchKernelGGL(mean_kernel, dim3((a.K + 63) / 64), dim3(64 * kMeanChains), 0, stream, a);
    hipLaunchKernelGGL((rank_kernel<1, false>), ranks, dim3(kRankThreads), 0, stream, a);
  }
  hipLaunchKernelGGL(place_kernel, dim3((a.K + kRankThreads - 1) / kRankThreads), dim3(kRankThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace mm
