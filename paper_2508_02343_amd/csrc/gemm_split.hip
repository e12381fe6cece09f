// Mixed MX GEMM for the shapes between decode and prefill (batched decode,
// prompt chunks, few weight rows): too many activation rows, or too few steps
// for its weight rows, for the decode kernel, too few output tiles for the
// LDS-tiled kernel to give every CU one.
//
// What bounds these shapes is how many CUs share the operand stream, and the
// latency and rate at which one CU takes it, so a workgroup covers a small
// output tile, 32 TN weight rows by 32 TM activation rows, and its eight
// wavefronts split the K loop instead of the tile: each accumulates the whole
// tile over its own layout steps, so every operand byte is loaded once per
// workgroup, straight from global memory into the MFMA registers (1 KB
// contiguous per load from the packed layout).  No LDS staging and no
// barrier inside the K loop: a wavefront waits for its own loads only, two
// stages (an E2M1 step, or half an E3M2 / E4M3 step) in flight each.  The
// fp32 partial sums are added through LDS in wavefront order and rounded to
// bf16 once (Sec. 3.2 "GEMM kernel").
//
// Measured (us, 75 / 18.75 / 6.25 % split, M x K x N, weights in rotation beyond
// the caches; before: the decode kernel up to 64 rows, the LDS-tiled one above):
//   32 x 4096 x 28672    18.2 -> 16.8    128 x 4096 x 6144     28.0 -> 9.2
//   64 x 4096 x 4096      6.9 ->  6.3    512 x 4096 x 4096     27.2 -> 12.5
//   64 x 14336 x 4096    15.3 -> 14.6    333 x 27648 x 5120   133   -> 54
// (the last takes 14 TB/s of operands from L2 into the CUs, with 140 MB of L2
// misses; its loads alone take two thirds of that time).  Tried, with the
// weights in the cache: four wavefronts with
// every wavefront walking all groups and rings of four stages (7.6 and 50.6 us
// on 128 x 4096 x 6144 and 333 x 27648 x 5120); a fragment's reload issued
// between the MFMAs (equal, and spills on the widest tile); non-temporal weight
// loads (slower where the weight is cached, equal where it is not).
//
// Every wavefront works on one group (E2M1, E3M2 or E4M3), the wavefronts
// shared out by the groups' bytes, so an output's summation order depends on
// the split and K only, not on the tile shape.
#include "gemm_common.hpp"
#include "gemm_route.hpp"

namespace mm {

namespace split {

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
// one 16-byte word per lane of a wavefront, padded so that the words of one
// output row (in different chunks) fall on different banks
constexpr int kChunkBytes = 64 * 16 + 16;

// A wave-uniform pointer, kept in SGPRs.
__device__ __forceinline__ const uint8_t* uni(const uint8_t* p) {
  const uint64_t v = (uint64_t)p;
  const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
  return (const uint8_t*)(lo | hi << 32);
}

// A wavefront's walk over its layout steps: where the tile's first row of the
// next step starts in both operands' codes and scales, the way to the step
// after it, and how many steps are left.
struct Walk {
  const uint8_t *w, *x, *sw, *sx;
  int64_t dw, dx, dsw, dsx;
  int left;
};

template <int G>
__device__ __forceinline__ Walk walk(const GemmArgs& a, int64_t n0, int64_t m0, int wv, int W, int n) {
  constexpr int RB = step_row_bytes(G);
  const int64_t gstep = wv + (G >= 1 ? a.steps[0] : 0) + (G >= 2 ? a.steps[1] : 0);
  Walk k;
  k.w = uni(a.w.q[G] + (wv * a.w.rp + n0) * RB);
  k.x = uni(a.x.q[G] + (wv * a.x.rp + m0) * RB);
  k.sw = uni(a.w.sc + (gstep * a.w.rp + n0) * kStepBlocks);
  k.sx = uni(a.x.sc + (gstep * a.x.rp + m0) * kStepBlocks);
  k.dw = W * a.w.rp * RB;
  k.dx = W * a.x.rp * RB;
  k.dsw = W * a.w.rp * kStepBlocks;
  k.dsx = W * a.x.rp * kStepBlocks;
  k.left = n;
  return k;
}

__device__ __forceinline__ void next_step(Walk& k) {
  k.w = uni(k.w + k.dw);
  k.x = uni(k.x + k.dx);
  k.sw = uni(k.sw + k.dsw);
  k.sx = uni(k.sx + k.dsx);
  --k.left;
}

// Buffer descriptors of one step's loads (a tile's rows of a step lie within
// 16 KB).  Past the wavefront's last step they are empty and the loads touch no
// memory and give zero, so the loops below issue the same loads for every
// stage, without branches, and the waits the compiler places leave exactly the
// younger stage in flight.
struct Desc {
  __amdgpu_buffer_rsrc_t w, x, sw, sx;
};
__device__ __forceinline__ __amdgpu_buffer_rsrc_t desc(const uint8_t* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p), 0, bytes, 0x00020000);
}
__device__ __forceinline__ Desc descs(const Walk& k) {
  const int bytes = k.left > 0 ? 0x7fffffff : 0;
  return Desc{desc(k.w, bytes), desc(k.x, bytes), desc(k.sw, bytes), desc(k.sx, bytes)};
}

// Half h of a layout step of group G (E2M1: the whole step, h = 0) for row
// group i of an operand: lane 32 g + r holds row r, as the 32 x 32 x 64 MFMA
// takes it (E2M1: dwords 0-3 the step's first 64 channels, 4-7 the second).
template <int G>
__device__ __forceinline__ v8i load_frag(__amdgpu_buffer_rsrc_t d, int i, int h, int lane) {
  const int g = lane >> 5, r = lane & 31;
  const int off = G == 1 ? g * 768 + r * 24 : g * 512 + r * 16;
  const int at = h * (G == 1 ? 1536 : 2048) + i * (kRowGroup * step_row_bytes(G));
  const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(d, off, at, 0);
  if constexpr (G == 1) {
    const u32x2 b = __builtin_amdgcn_raw_buffer_load_b64(d, off + 16, at, 0);
    return v8i{(int)a.x, (int)a.y, (int)a.z, (int)a.w, (int)b.x, (int)b.y, 0, 0};
  } else {
    const u32x4 b = __builtin_amdgcn_raw_buffer_load_b128(d, off + 1024, at, 0);
    return v8i{(int)a.x, (int)a.y, (int)a.z, (int)a.w, (int)b.x, (int)b.y, (int)b.z, (int)b.w};
  }
}

template <int TN, int TM>
using Acc = v16f[TN][TM];

template <int TN, int TM>
struct Stage {
  v8i w[TN], x[TM];
};

// The scale words (four E8M0 bytes per row) of a step.
template <int TN, int TM>
struct Scales {
  uint32_t w[TN], x[TM];
};

template <int G, int TN, int TM>
__device__ __forceinline__ void load_stage(Stage<TN, TM>& b, const Desc& d, int h, int lane) {
#pragma unroll
  for (int i = 0; i < TN; ++i) b.w[i] = load_frag<G>(d.w, i, h, lane);
#pragma unroll
  for (int j = 0; j < TM; ++j) b.x[j] = load_frag<G>(d.x, j, h, lane);
}

template <int TN, int TM>
__device__ __forceinline__ void load_scales(Scales<TN, TM>& s, const Desc& d, int lane) {
  const int off = (lane & 31) * kStepBlocks;
#pragma unroll
  for (int i = 0; i < TN; ++i) s.w[i] = __builtin_amdgcn_raw_buffer_load_b32(d.sw, off, i * kRowGroup * kStepBlocks, 0);
#pragma unroll
  for (int j = 0; j < TM; ++j) s.x[j] = __builtin_amdgcn_raw_buffer_load_b32(d.sx, off, j * kRowGroup * kStepBlocks, 0);
}

// Lane 32 g + r feeds the scale of block 2 h + g of its row, h the 64-channel
// half of the step: the word shifted down by 8 g, byte 2 h by op_sel.
template <int TN, int TM>
__device__ __forceinline__ void shift_scales(Scales<TN, TM>& s, int lane) {
  const int sh = (lane >> 5) * 8;
#pragma unroll
  for (int i = 0; i < TN; ++i) s.w[i] >>= sh;
#pragma unroll
  for (int j = 0; j < TM; ++j) s.x[j] >>= sh;
}

// The MFMAs of one 64-channel slice: fragment dwords 4 KK .. of E2M1, scale
// byte OP.
template <int G, int FS, int OP, int KK, int TN, int TM>
__device__ __forceinline__ void mfma_slice(Acc<TN, TM>& acc, const Stage<TN, TM>& b, const Scales<TN, TM>& s) {
  constexpr int fmt = group_fmt(G, FS);
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      const v8i& p = b.w[i];
      const v8i& q = b.x[j];
      const v8i pw = G == 0 ? v8i{p[4 * KK], p[4 * KK + 1], p[4 * KK + 2], p[4 * KK + 3], 0, 0, 0, 0} : p;
      const v8i qx = G == 0 ? v8i{q[4 * KK], q[4 * KK + 1], q[4 * KK + 2], q[4 * KK + 3], 0, 0, 0, 0} : q;
      acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(pw, qx, acc[i][j], fmt, fmt, OP, (int)s.w[i], OP,
                                                                  (int)s.x[j]);
    }
}

// A wavefront's E2M1 steps wv, wv + W, ...: two stages, each one step,
// reloaded as soon as its MFMAs are issued.  The last two are computed
// without loads behind them (with one step, or an odd number, the last stage
// is empty: zero codes).
template <int FS, int TN, int TM>
__device__ __forceinline__ void run_e2m1(Acc<TN, TM>& acc, const GemmArgs& a, int64_t n0, int64_t m0, int wv, int W,
                                         int lane) {
  const int n = (a.steps[0] - wv + W - 1) / W;
  if (n <= 0) return;
  Walk k = walk<0>(a, n0, m0, wv, W, n);
  Stage<TN, TM> b[2];
  Scales<TN, TM> s[2];
  auto load = [&](int d) {
    const Desc e = descs(k);
    load_scales(s[d], e, lane);
    load_stage<0>(b[d], e, 0, lane);
    next_step(k);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto compute = [&](int d) {
    shift_scales(s[d], lane);
    mfma_slice<0, FS, 0, 0>(acc, b[d], s[d]);
    mfma_slice<0, FS, 2, 1>(acc, b[d], s[d]);
    __builtin_amdgcn_sched_barrier(0);
  };
  load(0);
  load(1);
  for (int i = 2; i < n; i += 2) {
    compute(0);
    load(0);
    compute(1);
    load(1);
  }
  compute(0);
  compute(1);
}

// The same for the E3M2 / E4M3 steps, each two stages (its halves).
template <int G, int FS, int TN, int TM>
__device__ __forceinline__ void run_halves(Acc<TN, TM>& acc, const GemmArgs& a, int64_t n0, int64_t m0, int wv, int W,
                                           int lane) {
  const int n = (a.steps[G] - wv + W - 1) / W;
  if (n <= 0) return;
  Walk k = walk<G>(a, n0, m0, wv, W, n);
  Stage<TN, TM> b0, b1;
  Scales<TN, TM> s;
  Desc e = descs(k);
  load_scales(s, e, lane);
  load_stage<G>(b0, e, 0, lane);
  __builtin_amdgcn_sched_barrier(0);
  load_stage<G>(b1, e, 1, lane);
  __builtin_amdgcn_sched_barrier(0);
  for (int i = 1; i < n; ++i) {
    next_step(k);
    e = descs(k);
    Scales<TN, TM> c = s;
    shift_scales(c, lane);
    mfma_slice<G, FS, 0, 0>(acc, b0, c);
    __builtin_amdgcn_sched_barrier(0);
    load_scales(s, e, lane);
    load_stage<G>(b0, e, 0, lane);
    __builtin_amdgcn_sched_barrier(0);
    mfma_slice<G, FS, 2, 0>(acc, b1, c);
    __builtin_amdgcn_sched_barrier(0);
    load_stage<G>(b1, e, 1, lane);
    __builtin_amdgcn_sched_barrier(0);
  }
  shift_scales(s, lane);
  mfma_slice<G, FS, 0, 0>(acc, b0, s);
  __builtin_amdgcn_sched_barrier(0);
  mfma_slice<G, FS, 2, 0>(acc, b1, s);
}

// Activation fragments added up at a time: the LDS of eight wavefronts'
// partial sums of that many columns of the tile.
template <int TN, int TM>
__host__ __device__ constexpr int reduce_cols() {
  constexpr int most = 4 / TN;  // 133 KB
  return TM < most ? TM : most;
}
template <int TN, int TM>
__host__ __device__ constexpr int lds_bytes() {
  return kWaves * TN * reduce_cols<TN, TM>() * 4 * kChunkBytes;
}

}  // namespace split

using namespace split;

template <int TN, int TM, int FS>
__global__ __launch_bounds__(kThreads) void gemm_split_kernel(GemmArgs a, int tiles_n, int tiles_m, int w0, int w1,
                                                              int w2) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // workgroup -> tile: consecutive tiles per XCD (workgroups are dealt to the
  // 8 XCDs round-robin), activation tiles fastest, so the tiles that share a
  // weight panel run on one XCD
  const int nt = tiles_n * tiles_m;
  const int xcd = blockIdx.x & 7, k = blockIdx.x >> 3;
  const int per_x = nt >> 3, extra = nt & 7;
  const int id = xcd * per_x + (xcd < extra ? xcd : extra) + k;
  const int tn = id / tiles_m, tm = id - tn * tiles_m;
  // the last tile of each direction starts early enough to lie inside the
  // padded rows; the outputs it shares with the tile before are stored by that one
  const int64_t n_own = (int64_t)tn * (32 * TN), m_own = (int64_t)tm * (32 * TM);
  const int64_t n0 = n_own + 32 * TN <= a.w.rp ? n_own : a.w.rp - 32 * TN;
  const int64_t m0 = m_own + 32 * TM <= a.x.rp ? m_own : a.x.rp - 32 * TM;

  Acc<TN, TM> acc;
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;

  if (wave < w0) run_e2m1<FS, TN, TM>(acc, a, n0, m0, wave, w0, lane);
  else if (wave < w0 + w1) run_halves<1, FS, TN, TM>(acc, a, n0, m0, wave - w0, w1, lane);
  else if (wave < w0 + w1 + w2) run_halves<2, FS, TN, TM>(acc, a, n0, m0, wave - w0 - w1, w2, lane);

  // Partial sums through LDS, JC activation fragments at a time.  Wavefront
  // w's words of fragment (i, j): four chunks (registers 4h .. 4h+3), lane
  // 32 g + r holding output row r, columns 8 h + 4 g .. + 3 of the fragment.
  // A thread adds up two words, eight consecutive columns of one row, and
  // stores them as one 16-byte word; consecutive threads take one row's words.
  constexpr int JC = reduce_cols<TN, TM>();
  constexpr int kRowWords = 4 * TN;  // 16-byte output words per row of the tile
  const int64_t M = a.x.rows, N = a.w.rows;
#pragma unroll
  for (int j0 = 0; j0 < TM; j0 += JC) {
    if (j0) __syncthreads();
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int j = j0; j < j0 + JC && j < TM; ++j)
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          const int chunk = ((wave * TN + i) * JC + (j - j0)) * 4 + h;
          const v16f& c = acc[i][j];
          *reinterpret_cast<v4f*>(lds + chunk * kChunkBytes + lane * 16) =
              v4f{c[4 * h], c[4 * h + 1], c[4 * h + 2], c[4 * h + 3]};
        }
    __syncthreads();
    constexpr int kWords = 32 * JC * kRowWords;
#pragma unroll
    for (int e0 = 0; e0 < kWords; e0 += kThreads) {
      const int e = e0 + (int)threadIdx.x;
      if (kWords % kThreads != 0 && e >= kWords) break;
      const int row = e / kRowWords, word = e - row * kRowWords;
      const int i = word >> 2, h = word & 3, j = row >> 5, r = row & 31;
      const int64_t m = m0 + 32 * j0 + row, n = n0 + 8 * word;
      if (j0 + j >= TM || m < m_own || m >= M || n < n_own || n >= N) continue;
      v4f lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const uint8_t* p = lds + (((w * TN + i) * JC + j) * 4 + h) * kChunkBytes + r * 16;
        const v4f cl = *reinterpret_cast<const v4f*>(p), ch = *reinterpret_cast<const v4f*>(p + 32 * 16);
        lo = w == 0 ? cl : lo + cl;
        hi = w == 0 ? ch : hi + ch;
      }
      uint16_t* dst = a.y + m * a.ldy + n;
      const u32x4 v = {pack_bf16x2_rne(lo[0], lo[1]), pack_bf16x2_rne(lo[2], lo[3]), pack_bf16x2_rne(hi[0], hi[1]),
                       pack_bf16x2_rne(hi[2], hi[3])};
      if (n + 8 <= N) {
        *reinterpret_cast<u32x4*>(dst) = v;
      } else {
        for (int q = 0; q < (int)(N - n); ++q) dst[q] = (uint16_t)(v[q >> 1] >> (16 * (q & 1)));
      }
    }
  }
}

template <int TN, int TM, int FS>
static hipError_t launch_split_fs(const GemmArgs& a, const Device& dev, hipStream_t stream) {
  constexpr int lds = lds_bytes<TN, TM>();
  static DeviceOnce once;
  hipError_t e = allow_lds(once, dev, reinterpret_cast<const void*>(gemm_split_kernel<TN, TM, FS>), lds);
  if (e != hipSuccess) return e;
  const int64_t tn = (a.w.rows + 32 * TN - 1) / (32 * TN), tm = (a.x.rows + 32 * TM - 1) / (32 * TM);
  int w[3];
  share_waves(a.steps, kByteCost, kWaves, w);
  hipLaunchKernelGGL((gemm_split_kernel<TN, TM, FS>), dim3((unsigned)(tn * tm)), dim3(kThreads), lds, stream, a, (int)tn,
                     (int)tm, w[0], w[1], w[2]);
  return hipGetLastError();
}

// The format set is an instruction immediate: one kernel per set.
template <int TN, int TM>
static hipError_t launch_split(const GemmArgs& a, const Device& dev, hipStream_t stream) {
  switch (a.fs) {
    case 0: return launch_split_fs<TN, TM, 0>(a, dev, stream);
    case 1: return launch_split_fs<TN, TM, 1>(a, dev, stream);
    case 2: return launch_split_fs<TN, TM, 2>(a, dev, stream);
    case 3: return launch_split_fs<TN, TM, 3>(a, dev, stream);
  }
  return hipErrorInvalidValue;
}

template <int I>
static hipError_t launch_shape(const GemmArgs& a, const Device& dev, hipStream_t stream) {
  return launch_split<kSplitShapes[I].tn, kSplitShapes[I].tm>(a, dev, stream);
}

hipError_t launch_gemm_split(const GemmArgs& a, int shape, const Device& dev, hipStream_t stream) {
  switch (shape) {
    case 0: return launch_shape<0>(a, dev, stream);
    case 1: return launch_shape<1>(a, dev, stream);
    case 2: return launch_shape<2>(a, dev, stream);
    case 3: return launch_shape<3>(a, dev, stream);
    case 4: return launch_shape<4>(a, dev, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace mm
