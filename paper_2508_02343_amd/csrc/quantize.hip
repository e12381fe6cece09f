// Fused reorder-and-quantize (MicroMix Sec. 3.2 "Quantization kernel",
// Fig. "micromix-design" b): one pass over bf16 rows that gathers channels by
// sigma (Sec. 3.1), takes each 32-channel block's shared E8M0 scale and writes
// E2M1 / E3M2 / E4M3 codes for the three groups (Sec. 2.1 MX rule), with the
// layer's RMSNorm in front where asked for (App. D.2).
//
// HBM-bound.  A workgroup stages a pass of RH rows in LDS, one thread per (row,
// 32-channel block), and several workgroups share a CU, so that one loads
// while another quantises:
//  - rows arrive with 16-byte coalesced loads (the only HBM read, four per
//    thread, all in flight at once, marked non-temporal as they are read once)
//    and go to LDS; the next pass's loads are issued before this one is
//    quantised;
//  - a pass of padding rows only loads nothing (their workgroups read the last
//    row over and over, up to 31 at a time: 1 x 20480 8.0 -> 6.7, 4 x 27648 9.9 ->
//    7.8 us);
//  - lanes run over the pass's rows first, so the lanes that store one
//    block's codes hold consecutive rows, whose codes are consecutive in the
//    packed layout (64-byte runs with four rows);
//  - each thread keeps its block's 32 sigma entries as byte offsets in a row,
//    two per register, and gathers with 32 LDS u16 reads; the block absmax is a
//    packed 16-bit max over the sign-cleared bf16 bits;
//  - the codes come from the gfx950 scaled conversions, which divide by the
//    E8M0 scale and round to nearest even (E2M1 and E4M3 two codes per
//    instruction, E3M2 one instruction per block giving the packed 24-byte bit
//    stream).  The E4M3 conversion does not saturate, so E4M3 inputs are first
//    clamped to 448 * scale, which is exact in bf16.
//
// With the RMSNorm, each thread also adds up the squares of the values it
// loads, in fp64 (exact squares, so no scaling is needed), before they go to
// LDS; the wavefronts' row sums meet in LDS under the same barrier as the
// rows, and every gathered element becomes bf16(gamma * bf16(x * r)) (fp32
// products, round to nearest even).  The weights sit in LDS in block order,
// four 16-byte pieces per block at (piece * nblk + block) * 16, so a
// wavefront's reads are conflict-free.
//
// Measured (us; before: a ring of LDS slots filled by producer wavefronts, one
// workgroup per CU, and for K > 8192 one row per workgroup at a time):
//   plain   8 x 4096   5.2 -> 3.7    2048 x 4096  9.3 ->  8.5   8192 x 5120   30.7 -> 25.1 (4.4 TB/s)
//         333 x 27648 19.4 -> 13.3   4096 x 14336 39.5 -> 34.0   5120 x 27648 170  -> 86
//   norm    8 x 4096   8.6 -> 5.2    2048 x 4096 13.8 -> 12.8   8192 x 5120   43.4 -> 40.9
//         512 x 4096   9.1 -> 6.5    4096 x 14336 73.3 -> 50.4   5120 x 27648 577  -> 113
// The plain kernel waits on memory (loads in flight only while a workgroup
// quantises, code stores in runs of a few rows); the norm's 540 VALU
// instructions per wavefront and pass, against 190, bound its large shapes.
// What spills costs more than what it saves: the norm variant fits 128 registers
// only because it gathers eight channels at a time (with 32 spilled registers
// 8192 x 5120 took 59 us, with 10, 44); with two and four rows per pass it still
// spills two.  Tried: two blocks per thread
// (34 us plain on 8192 x 5120), five wavefronts per SIMD (spills, 37 us).
#include "kernels.hpp"

namespace mm {
namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x32 __attribute__((ext_vector_type(32)));
typedef short i16x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef int i32x6 __attribute__((ext_vector_type(6)));
typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

typedef float f32x2 __attribute__((ext_vector_type(2)));

// LDS pointers built from 32-bit byte addresses (the base already added)
typedef const __attribute__((address_space(3))) uint16_t lds_u16_t;

__device__ __forceinline__ uint16_t lds_u16(uint32_t byte_addr) {
  return *reinterpret_cast<lds_u16_t*>((uintptr_t)byte_addr);
}

__device__ __forceinline__ uint32_t max_u16x2(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t,
                            __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}

__device__ __forceinline__ uint32_t min_u16x2(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t,
                            __builtin_elementwise_min(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}

// Zero codes and scale byte for block j of step `step` of row n (padding).
template <int G>
__device__ __forceinline__ void zero_block(const QuantArgs& a, int64_t step, int64_t gstep, int64_t n, int j) {
  uint8_t* dst = a.q[G] + code_offset<G>(step, a.rp, n, j);
  if constexpr (G == 0) {
    *reinterpret_cast<uint4*>(dst) = make_uint4(0u, 0u, 0u, 0u);
  } else if constexpr (G == 1) {
    uint2* d = reinterpret_cast<uint2*>(dst);
    d[0] = d[1] = d[2] = make_uint2(0u, 0u);
  } else {
    *reinterpret_cast<uint4*>(dst) = make_uint4(0u, 0u, 0u, 0u);
    *reinterpret_cast<uint4*>(dst + 512) = make_uint4(0u, 0u, 0u, 0u);
  }
  a.sc[(gstep * a.rp + n) * kStepBlocks + j] = 0;
}

template <int G>
__device__ __forceinline__ void zero_tail(const QuantArgs& a, int64_t step, int64_t gstep, int64_t n, int j) {
  for (int jj = j + 1; jj < kStepBlocks; ++jj) zero_block<G>(a, step, gstep, n, jj);
}

// Bytes from row 0's codes of a block to row n's, n a multiple of the rows per
// pass: whole row groups, then rows within one.
template <int G>
__device__ __forceinline__ int64_t row_offset(int64_t n) {
  return (n & ~(int64_t)(kRowGroup - 1)) * step_row_bytes(G) + (n & (kRowGroup - 1)) * (G == 1 ? 24 : 16);
}

// Quantise the 32 gathered channels d (bf16 pairs) of block b (local to its
// group) of row n = n0 + prow, n0 uniform over the workgroup; dst and sdst are
// the block's codes and scale byte of row prow.  Rows past a.rows are padding
// and quantise an all-zero block.  The thread that owns a group's last block
// also zeroes the padding blocks of that step.
__device__ __forceinline__ void encode_block(uint32_t (&d)[16], int group, bool last, const QuantArgs& a, int64_t n0,
                                             int prow, int b, int gstep0, uint8_t* dst, uint8_t* sdst) {
  const int64_t n = n0 + prow;
  const bool pad_row = n >= a.rows;
#pragma unroll
  for (int i = 0; i < 16; ++i) d[i] = pad_row ? 0u : d[i];

  // absmax: bf16 magnitudes compare as unsigned integers
  uint32_t m[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) m[i] = d[i] & 0x7FFF7FFFu;
#pragma unroll
  for (int i = 4; i < 16; ++i) m[i & 3] = max_u16x2(m[i & 3], d[i] & 0x7FFF7FFFu);
  m[0] = max_u16x2(max_u16x2(m[0], m[1]), max_u16x2(m[2], m[3]));
  const uint32_t amax = (m[0] & 0xFFFFu) > (m[0] >> 16) ? (m[0] & 0xFFFFu) : (m[0] >> 16);

  // Shared exponent e = floor(log2 amax) - emax, clamped below at -127: for
  // a bf16 amax with biased exponent E this is max(E - 127 - emax, -127); a
  // subnormal or zero amax (E = 0) lands on the clamp.  The E8M0 byte is e+127.
  const bool e2m3 = (a.fs & 1) != 0, e5m2 = (a.fs & 2) != 0;  // the alternative formats of groups 1 and 2
  const int emax = group == 0 ? 2 : (group == 1 ? (e2m3 ? 2 : 4) : (e5m2 ? 15 : 8));
  const int E = (int)(amax >> 7);
  const uint32_t sbyte = (uint32_t)(E - emax > 0 ? E - emax : 0);
  // the conversions read the scale's E8M0 exponent from an fp32 operand
  const float scale = __uint_as_float(sbyte << 23);

  const int64_t step = b >> 2;
  const int j = b & 3;
  const int64_t gstep = gstep0 + step;
  sdst[n0 * kStepBlocks] = (uint8_t)sbyte;
  if (group == 0) {
    uint32_t w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint32_t v = 0;
      v = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(v, __builtin_bit_cast(bf16x2, d[4 * q + 0]), scale, 0);
      v = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(v, __builtin_bit_cast(bf16x2, d[4 * q + 1]), scale, 1);
      v = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(v, __builtin_bit_cast(bf16x2, d[4 * q + 2]), scale, 2);
      v = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(v, __builtin_bit_cast(bf16x2, d[4 * q + 3]), scale, 3);
      w[q] = v;
    }
    *reinterpret_cast<uint4*>(dst + row_offset<0>(n0)) = make_uint4(w[0], w[1], w[2], w[3]);
    if (last) zero_tail<0>(a, step, gstep, n, j);
  } else if (group == 1) {
    u32x16 v;
    i32x6 c;
    if (e2m3) {
      // clamp the magnitudes to the largest E2M3 value, 7.5 * 2^e (exact in
      // bf16: biased exponent e + 129 = sbyte + 2, mantissa 0x70), keep the
      // signs; nothing then depends on how the conversion treats larger values
      const uint32_t lim = ((sbyte + 2u) << 7) | 0x70u;
      const uint32_t lim2 = lim | (lim << 16);
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = min_u16x2(d[i] & 0x7FFF7FFFu, lim2) | (d[i] & 0x80008000u);
      c = __builtin_amdgcn_cvt_scalef32_pk32_fp6_bf16(__builtin_bit_cast(bf16x32, v), scale);
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = d[i];
      c = __builtin_amdgcn_cvt_scalef32_pk32_bf6_bf16(__builtin_bit_cast(bf16x32, v), scale);
    }
    uint2* p = reinterpret_cast<uint2*>(dst + row_offset<1>(n0));
    p[0] = make_uint2((uint32_t)c[0], (uint32_t)c[1]);
    p[1] = make_uint2((uint32_t)c[2], (uint32_t)c[3]);
    p[2] = make_uint2((uint32_t)c[4], (uint32_t)c[5]);
    if (last) zero_tail<1>(a, step, gstep, n, j);
  } else {
    // the largest finite value times 2^e in bf16, mantissa 0x60 (1.75): E4M3
    // 448 (biased exponent e + 127 + 8 = sbyte + 8), E5M2 57344 (sbyte + 15)
    const uint32_t lim = ((sbyte + (e5m2 ? 15u : 8u)) << 7) | 0x60u;
    const uint32_t lim2 = lim | (lim << 16);
    uint32_t w[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      // clamp the magnitudes, keep the signs
      const uint32_t c0 = min_u16x2(d[2 * q] & 0x7FFF7FFFu, lim2) | (d[2 * q] & 0x80008000u);
      const uint32_t c1 = min_u16x2(d[2 * q + 1] & 0x7FFF7FFFu, lim2) | (d[2 * q + 1] & 0x80008000u);
      i16x2 v = {0, 0};
      if (e5m2) {
        v = __builtin_amdgcn_cvt_scalef32_pk_bf8_bf16(v, __builtin_bit_cast(bf16x2, c0), scale, false);
        v = __builtin_amdgcn_cvt_scalef32_pk_bf8_bf16(v, __builtin_bit_cast(bf16x2, c1), scale, true);
      } else {
        v = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(v, __builtin_bit_cast(bf16x2, c0), scale, false);
        v = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(v, __builtin_bit_cast(bf16x2, c1), scale, true);
      }
      w[q] = __builtin_bit_cast(uint32_t, v);
    }
    uint8_t* p = dst + row_offset<2>(n0);
    *reinterpret_cast<uint4*>(p) = make_uint4(w[0], w[1], w[2], w[3]);
    *reinterpret_cast<uint4*>(p + 512) = make_uint4(w[4], w[5], w[6], w[7]);
    if (last) zero_tail<2>(a, step, gstep, n, j);
  }
}

// base + one 16-bit half of w (one instruction; written out because the
// compiler would otherwise hoist the 32 halves, or their sums, out of the
// loop over the passes and spill).
template <int H>
__device__ __forceinline__ uint32_t add_word(uint32_t base, uint32_t w) {
  uint32_t r;
  if constexpr (H == 0)
    asm("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0"
        : "=v"(r)
        : "v"(base), "v"(w));
  else
    asm("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1"
        : "=v"(r)
        : "v"(base), "v"(w));
  return r;
}

// v + (v of another lane of the row of 16, chosen by the DPP control).
template <int CTRL>
__device__ __forceinline__ double add_dpp(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
  return v + __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Sum over the wavefront of each of N (1, 2 or 4) values per lane: lane l gets
// the sum of value l % N, in a fixed order.  The first steps, over lanes 1 and
// 2 apart, halve the values; the others rotate within rows of 16 lanes and
// swap rows, so nothing goes through LDS.
template <int N>
__device__ __forceinline__ double wave_sums(const double (&v)[N], int lane) {
  constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kRor4 = 0x124, kRor8 = 0x128;  // quad_perm / row_ror
  double t;
  if constexpr (N == 4) {
    // lane l keeps the values of its own parity of l / 2, then of l
    double k[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const double a = add_dpp<kXor2>(v[i]), b = add_dpp<kXor2>(v[i + 2]);
      k[i] = lane & 2 ? b : a;
    }
    const double a = add_dpp<kXor1>(k[0]), b = add_dpp<kXor1>(k[1]);
    t = lane & 1 ? b : a;
  } else if constexpr (N == 2) {
    const double a = add_dpp<kXor1>(v[0]), b = add_dpp<kXor1>(v[1]);
    t = add_dpp<kXor2>(lane & 1 ? b : a);
  } else {
    t = add_dpp<kXor2>(add_dpp<kXor1>(v[0]));
  }
  t = add_dpp<kRor8>(add_dpp<kRor4>(t));
  // rows of 16: swapping a copy's odd rows with another's even rows pairs
  // them up, then the halves
  uint64_t u = __builtin_bit_cast(uint64_t, t);
  const auto l16 = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
  const auto h16 = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
  t = __builtin_bit_cast(double, (uint64_t)h16[0] << 32 | l16[0]) + __builtin_bit_cast(double, (uint64_t)h16[1] << 32 | l16[1]);
  u = __builtin_bit_cast(uint64_t, t);
  const auto l32 = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)u, false, false);
  const auto h32 = __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
  return __builtin_bit_cast(double, (uint64_t)h32[0] << 32 | l32[0]) + __builtin_bit_cast(double, (uint64_t)h32[1] << 32 | l32[1]);
}

// fp32(1 / sqrt(m)), m > 0 and normal or infinite, evaluated in fp64: the
// hardware's reciprocal square root estimate and two Newton steps (relative
// error below 2^-51, as a square root and a division have) instead of their
// long expansions, which every thread of a row would run.  A row with an
// infinite element keeps the estimate's zero (the steps would give a NaN).
__device__ __forceinline__ float rsqrt_f64(double m) {
  double y = __builtin_amdgcn_rsq(m);
#pragma unroll
  for (int i = 0; i < 2; ++i) y = fma(y * 0.5, fma(-m * y, y, 1.0), y);
  return m == __builtin_inf() ? 0.0f : (float)y;
}

// 32-bit LDS addresses
template <typename T>
__device__ __forceinline__ T lds_load(uint32_t addr) {
  return *reinterpret_cast<const __attribute__((address_space(3))) T*>((uintptr_t)addr);
}
template <typename T>
__device__ __forceinline__ void lds_store(uint32_t addr, T v) {
  *reinterpret_cast<__attribute__((address_space(3))) T*>((uintptr_t)addr) = v;
}

}  // namespace

constexpr int kMaxThreads = 1024;

// Pass p covers rows p RH .. p RH + RH - 1 (padding rows included), thread t
// block t / RH of row t % RH; gridDim.x <= passes.  LDS: RH rows of 2 K + 16
// bytes (the padding shifts the banks of consecutive rows), then with the norm
// 2 K bytes of weights and RH fp64 sums per wavefront.
template <int RH, bool kNorm>
__global__ __launch_bounds__(kMaxThreads) void quantize_kernel(QuantArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint8_t stage[];
  static_assert(RH <= 4 || !kNorm, "a row sum's chunks belong to one row per load");
  const uint32_t lds0 = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint8_t*)stage;
  const int K = a.K, nblk = K >> 5;
  const int tid = threadIdx.x;
  const int n_act = RH * nblk;  // threads with a block
  const bool active = tid < n_act;
  const int t = active ? tid : 0;
  const int blk = t / RH, prow = t - blk * RH;
  const uint32_t row_stride = (uint32_t)(2 * K + 16);
  const uint32_t gam0 = lds0 + RH * row_stride;
  const uint32_t sums0 = gam0 + 2u * (uint32_t)K;

  // this workgroup's passes: workgroups are dealt to the 8 XCDs round-robin,
  // each XCD takes a contiguous range of passes, so the rows of one 32-row
  // group (which share cache lines in the packed layout) are written through
  // one XCD's L2
  const int64_t passes = (a.rp + RH - 1) / RH;
  int64_t q, q_end, stride;
  if (gridDim.x % 8 == 0) {
    const int x = blockIdx.x & 7;
    q = passes * x / 8 + (blockIdx.x >> 3);
    q_end = passes * (x + 1) / 8;
    stride = gridDim.x / 8;
  } else {
    q = blockIdx.x;
    q_end = passes;
    stride = gridDim.x;
  }
  if (q >= q_end) return;  // uniform over the workgroup

  // A pass has four 16-byte chunks per thread.  Chunk j: up to four rows, the
  // threads share a row's 4 / RH parts, so j alone gives row and part; above,
  // RH / 4 rows per j, row_in the thread's.
  constexpr int kParts = RH < 4 ? 4 / RH : 1, kRowsPer = RH < 4 ? 1 : RH / 4;
  const int row_in = RH > 4 ? t / (K >> 3) : 0;
  const int col = RH > 4 ? t - row_in * (K >> 3) : t;
  u32x4 buf[4] = {};
  auto load = [&](int64_t p) {
    if (p * RH >= a.rows) return;  // padding rows only
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int64_t row = p * RH + j / kParts * kRowsPer + row_in;
      row = row < a.rows ? row : a.rows - 1;  // (padding rows quantise zeros)
      const uint8_t* src = reinterpret_cast<const uint8_t*>(a.x + row * a.ldx + j % kParts * n_act * 8);
      buf[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src + (uint32_t)col * 16u));
    }
  };
  load(q);
  u32x4 gam[4 / RH + 1];
  if constexpr (kNorm)
#pragma unroll
    for (int j = 0; j < 4 / RH; ++j) gam[j] = *reinterpret_cast<const u32x4*>(a.gamma + (int64_t)(j * n_act + t) * 8);

  // sigma of the thread's block; an out-of-range entry (a caller error) is
  // clamped to stay inside the row
  uint32_t sig[16];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int4 v = *reinterpret_cast<const int4*>(a.perm + blk * 32 + 4 * k);
    const int p[4] = {v.x, v.y, v.z, v.w};
    uint32_t o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = 2u * (uint32_t)((unsigned)p[i] < (unsigned)K ? p[i] : 0);
    sig[2 * k] = o[0] | (o[1] << 16);
    sig[2 * k + 1] = o[2] | (o[3] << 16);
  }
  if constexpr (kNorm) {
    // the weights in block order, gathered by sigma from a copy of gamma that
    // takes the rows' place in LDS first (gathered from global memory, they
    // would wait for sigma and then for themselves: 2 us)
#pragma unroll
    for (int j = 0; j < 4 / RH; ++j)
      if (active) lds_store<u32x4>(lds0 + (uint32_t)(j * n_act + t) * 16u, gam[j]);
    // sixteen wavefronts' sums; those of wavefronts that are not there stay zero
    if (tid < kMaxThreads / 64 * RH) lds_store<double>(sums0 + (uint32_t)tid * 8u, 0.0);
    __syncthreads();
    if (active && prow == 0)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        u32x4 g;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t s = sig[4 * k + i];
          g[i] = lds_u16(add_word<0>(lds0, s)) | ((uint32_t)lds_u16(add_word<1>(lds0, s)) << 16);
        }
        lds_store<u32x4>(gam0 + (uint32_t)(k * nblk + blk) * 16u, g);
      }
    __syncthreads();
  }
  const int group = blk < a.nb[0] ? 0 : (blk < a.nb[0] + a.nb[1] ? 1 : 2);
  const int b = blk - (group >= 1 ? a.nb[0] : 0) - (group >= 2 ? a.nb[1] : 0);  // block within its group
  const int gstep0 = (group >= 1 ? a.steps[0] : 0) + (group >= 2 ? a.steps[1] : 0);
  const bool last = b == (group == 0 ? a.nb[0] : (group == 1 ? a.nb[1] : a.nb[2])) - 1;  // the group's last block

  // where the thread's codes and scale byte of the rows 32 i + prow start
  uint8_t* const dst = (group == 0 ? a.q[0] + code_offset<0>(b >> 2, a.rp, prow, b & 3)
                                   : (group == 1 ? a.q[1] + code_offset<1>(b >> 2, a.rp, prow, b & 3)
                                                 : a.q[2] + code_offset<2>(b >> 2, a.rp, prow, b & 3)));
  uint8_t* const sdst = a.sc + ((gstep0 + (b >> 2)) * a.rp + prow) * kStepBlocks + (b & 3);

  for (; q < q_end; q += stride) {
    if constexpr (kNorm) {
      double c[4] = {0.0, 0.0, 0.0, 0.0};  // of each chunk
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const double lo = (double)__uint_as_float(buf[j][k] << 16);
          const double hi = (double)__uint_as_float(buf[j][k] & 0xFFFF0000u);
          c[j] = fma(lo, lo, c[j]);
          c[j] = fma(hi, hi, c[j]);
        }
      double sq[RH];
      if constexpr (RH == 4) {
#pragma unroll
        for (int i = 0; i < 4; ++i) sq[i] = active ? c[i] : 0.0;
      } else if constexpr (RH == 2) {
        sq[0] = active ? c[0] + c[1] : 0.0;
        sq[1] = active ? c[2] + c[3] : 0.0;
      } else {
        sq[0] = active ? (c[0] + c[1]) + (c[2] + c[3]) : 0.0;
      }
      const int lane = tid & 63;
      const double s = wave_sums<RH>(sq, lane);
      if (lane < RH) lds_store<double>(sums0 + (uint32_t)((tid >> 6) * RH + lane) * 8u, s);
    }
    if (active)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        lds_store<u32x4>(lds0 + (uint32_t)(j / kParts * kRowsPer + row_in) * row_stride +
                             (uint32_t)(j % kParts * n_act + col) * 16u,
                         buf[j]);
    __syncthreads();
    if (q + stride < q_end) load(q + stride);
    float rn = 0.0f;
    if constexpr (kNorm) {
      double p[8];
#pragma unroll
      for (int w = 0; w < 8; ++w) p[w] = lds_load<double>(sums0 + (uint32_t)(w * RH + prow) * 8u);
      double s = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
      if (blockDim.x > 8 * 64) {
#pragma unroll
        for (int w = 0; w < 8; ++w) p[w] = lds_load<double>(sums0 + (uint32_t)((8 + w) * RH + prow) * 8u);
        s += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
      }
      rn = rsqrt_f64(fma(s, a.inv_k, (double)a.eps));
    }
    uint32_t base = lds0 + (uint32_t)prow * row_stride;
    asm volatile("" : "+v"(base));  // (see add_word)
    uint32_t d[16];
    if constexpr (kNorm) {
      // bf16(gamma * bf16(x * r)), fp32 products, each rounded to nearest even:
      // eight channels at a time, the next eight's reads in flight (more would
      // spill)
      uint16_t e[2][8];
      u32x4 gm[2];
      auto read = [&](int k) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          e[k & 1][2 * i] = lds_u16(add_word<0>(base, sig[4 * k + i]));
          e[k & 1][2 * i + 1] = lds_u16(add_word<1>(base, sig[4 * k + i]));
        }
        gm[k & 1] = lds_load<u32x4>(gam0 + (uint32_t)(k * nblk + blk) * 16u);
        __builtin_amdgcn_sched_barrier(0);
      };
      read(0);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (k < 3) read(k + 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t g = gm[k & 1][i];
          const f32x2 x = {__uint_as_float((uint32_t)e[k & 1][2 * i] << 16) * rn,
                           __uint_as_float((uint32_t)e[k & 1][2 * i + 1] << 16) * rn};
          const uint32_t y = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
          const f32x2 z = {__uint_as_float(y << 16) * __uint_as_float(g << 16),
                           __uint_as_float(y & 0xFFFF0000u) * __uint_as_float(g & 0xFFFF0000u)};
          d[4 * k + i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(z, bf16x2));
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h) {  // sixteen reads in flight at a time
        uint16_t e[16];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          e[2 * i] = lds_u16(add_word<0>(base, sig[8 * h + i]));
          e[2 * i + 1] = lds_u16(add_word<1>(base, sig[8 * h + i]));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          u16x2 v;
          v.x = e[2 * i];
          v.y = e[2 * i + 1];
          d[8 * h + i] = __builtin_bit_cast(uint32_t, v);
        }
      }
    }
    const int64_t row0 = q * RH;  // (a multiple of RH, so the pass lies in one row group)
    if (active && row0 + prow < a.rp) encode_block(d, group, last, a, row0, prow, b, gstep0, dst, sdst);
    __syncthreads();
  }
}

template <int RH, bool kNorm>
static hipError_t launch_rows(const QuantArgs& a, const Device& dev, hipStream_t stream) {
  static DeviceOnce once;
  constexpr int kLds = 160 * 1024;
  hipError_t e = allow_lds(once, dev, reinterpret_cast<const void*>(quantize_kernel<RH, kNorm>), kLds);
  if (e != hipSuccess) return e;
  const int waves = (RH * (a.K >> 5) + 63) / 64;
  const size_t lds = (size_t)RH * (2 * a.K + 16) + (kNorm ? 2 * (size_t)a.K + 8 * (kMaxThreads / 64) * RH : 0);
  if (64 * waves > kMaxThreads || lds > kLds) return hipErrorInvalidValue;  // cannot happen: see launch_quantize
  // as many workgroups as the chip holds at once (four wavefronts on each of a
  // CU's four SIMDs and 160 KB of LDS), so that each keeps its sigma for all of its
  // passes.  The wavefronts of a workgroup spread over the SIMDs evenly: of five,
  // two share one, and a third such workgroup finds no room (counted in, those
  // left over ran behind the others: 3144 x 5120 16.6 -> 13.2, with the norm 27.9 ->
  // 20.8; 28557 x 2272 48.8 -> 39.3 us).
  int64_t per = waves <= 4 ? 16 / waves : 4 / ((waves + 3) / 4);
  if (per * lds > kLds) per = kLds / lds;
  const int64_t passes = (a.rp + RH - 1) / RH, cap = per * dev.cus;
  hipLaunchKernelGGL((quantize_kernel<RH, kNorm>), dim3((unsigned)(passes < cap ? passes : cap)), dim3(64 * waves), lds,
                     stream, a);
  return hipGetLastError();
}

// Rows per pass.  As many as 1024 threads and a 64 KB of rows take (K <= 8192:
// 4, <= 16384: 2) for the longest runs of codes per store; fewer rows give more
// and smaller workgroups, which start and finish sooner, and win where there is
// little to stream.  Measured (us, 1 / 2 / 4 rows per pass): 128 x 4096 3.6 / 3.7
// / 4.3, 512 x 4096 4.7 / 4.5 / 5.0, 2048 x 4096 10.3 / 8.1 / 8.6, 4096 x 4096
// 15.4 / 12.8 / 13.4, 14336 x 4096 42.6 / 35.1 / 33.0, 8192 x 5120 34 / 26.3 /
// 26.1, with the norm 512 x 4096 7.6 / 6.5 / 8.0 and 4096 x 5120 25.2 / 24.7 / 24.9;
// below 2048 channels four rows are never slower (1000 x 608: 4.0 / 3.9 / 3.6),
// and up to 512 sixteen beat them without the norm (28672 x 512: 12.2 / 10.8).
// Above 8192 channels one row, as long as every row is in flight at once (256 x
// 14336 6.9 / 7.7, 384 x 14336 9.1 / 8.1).
// With the norm, whose arithmetic bounds the large sizes, four rows per pass can
// leave the CU with too few wavefronts: two workgroups of five (K 2080 .. 2560:
// two rows make five of three, 28557 x 2560 67.1 -> 65.3) or one of nine or ten
// (K 4128 .. 5120: one row makes five of three, 28557 x 5120 125 -> 118, 8192 x
// 5120 42.3 -> 40.9, but only from 4480 channels on, which fill most of their
// lanes: 28557 x 4160 112 -> 121).
hipError_t launch_quantize(const QuantArgs& a, const Device& dev, hipStream_t stream) {
  if (a.rows == 0) return hipSuccess;
  const bool norm = a.norm != 0;
  const int64_t n = a.rp * a.K;
  int rh = a.K <= 8192 ? 4 : (a.K <= 16384 ? 2 : 1);
  if (a.K >= 2048) {
    if (n < (1 << 20) || (a.K > 8192 && a.rp <= dev.cus)) rh = 1;
    else if (n < (24 << 20) && rh > 2) rh = 2;
    else if (norm && a.K > 2048 && a.K <= 2560) rh = 2;
    else if (norm && a.K >= 4480 && a.K <= 5120) rh = 1;
  } else if (a.K <= 512 && !norm) {
    rh = 16;
  }
  switch (rh) {
    case 1: return norm ? launch_rows<1, true>(a, dev, stream) : launch_rows<1, false>(a, dev, stream);
    case 2: return norm ? launch_rows<2, true>(a, dev, stream) : launch_rows<2, false>(a, dev, stream);
    case 4: return norm ? launch_rows<4, true>(a, dev, stream) : launch_rows<4, false>(a, dev, stream);
    default: return launch_rows<16, false>(a, dev, stream);
  }
}

}  // namespace mm
