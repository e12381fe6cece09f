// Mixed MX GEMM for prefill shapes (many activation rows): compute-bound on
// the block-scaled MFMA, so operand tiles are staged in LDS and reused by the
// whole workgroup.
//
// Workgroup tile: BN = 256 weight rows (output columns n) x BM = 256 or 128
// activation rows (output rows m).  Four wavefronts, one per SIMD, in a
// 2 x 2 grid; each owns a (BN/2) x (BM/2) block of 32 x 32 fp32 MFMA
// accumulators (128 x 128: 256 accumulator registers, in the AGPR half of
// the register file).  A wavefront reads TN + TM operand fragments per
// 64-channel slice for TN * TM MFMAs, half the LDS traffic per MFMA of
// 128 x 64 blocks.  The K loop visits the E2M1 group, then E3M2, then E4M3
// (Sec. 3.1 group order), all accumulating into the same registers
// (Sec. 3.2 "GEMM kernel": one fp32 accumulation, one bf16 rounding at the
// end).
//
// Memory pipeline (gfx950): the packed layout stores each 32-row group's
// layout step contiguously and block-major, so a tile's share of a step is
// a few contiguous runs; it goes straight from global memory into LDS with
// global_load_lds_dwordx4 (1 KB per wavefront instruction).  One ring of
// equal slots serves all three groups: a slot holds one "stage", an E2M1
// layout step (128 channels, two slices) or half an E3M2 / E4M3 step (64
// channels, one slice), plus the step's E8M0 scale words of every tile row.
// The ring runs on across group boundaries, so the next group's first
// stages are in flight while the current group finishes.
//
// Every loading wavefront issues the same number of loads for every stage: a
// quarter of the weight rows' codes, a quarter of the activation rows' and one
// scale load (a share with fewer pieces is completed by loading its last ones
// again, into the same LDS bytes with the same data).  The vmcnt wait for a
// stage is then one constant, and issuing the next stage is a cursor (base
// pointers, per-lane offsets fixed per group) instead of per-stage address
// arithmetic.  (With wavefronts 0-1 on the weight rows and 2-3 on half as many
// activation rows, the latter repeated half of their loads at 256 x 128.)
//
// 256 x 128: four more wavefronts, the producers, do the loading (produce).
// 256 x 256: the registers allow one wavefront per SIMD, which loads and
// multiplies; the K loop runs in segments whose refills stay in one group:
// inside a segment the cursor only adds a precomputed increment (no branch,
// its per-lane offsets untouched), and it is re-pointed between segments; with
// the group change tested every stage, the scalar bookkeeping of a stage
// outweighed its MFMAs (5-10 % slower).
//
// Per stage q: its MFMAs, each followed by its share of the other work: the
// loads that refill stage q's slot with stage q + slots (256 x 256), the LDS
// reads of stage q+1's operands, and shortly before the end one s_barrier
// behind waits for these reads and for stage q+2's loads (mfma_block).  The
// sched_barrier fences keep that order.  Workgroups are mapped to tiles
// XCD by XCD and in groups of weight tiles, so the tiles that run together
// on one XCD share its L2.
//
// Measured (us, M x K x N): without the producers and with the waits between
// the stages 2048 x 4096 x 4096 took 29.9 (with them 27.0), 1000 x 4096 x 5400 in
// E2M3 / E5M2 30.1 (26.6), 700 x 4096 x 14336 44.0 (39.4); the 256 x 256 tile
// 4096 x 4096 x 14336 150 (148.5), 8192 x 5120 x 27648 640 (636; with all-zero
// codes 507: power is a part of what bounds it).  Without loads and LDS reads,
// but with the launch, the set-up and the epilogue of every tile: 19.0 (2048 x
// 4096 x 4096, of which the K loop's MFMAs are 9-10), 430 (8192 x 5120 x 27648).
#include "gemm_common.hpp"

namespace mm {

namespace tiled {

constexpr int kLdsBytes = 160 * 1024;
constexpr int kWaves = 4;  // wavefronts with accumulators, one per SIMD

// A stage of group G: E2M1 one layout step (two 64-channel slices), E3M2 and
// E4M3 half a step (one slice).
__host__ __device__ constexpr int stage_slices(int G) { return G == 0 ? 2 : 1; }
// Bytes of one 32-row group's share of a stage.
__host__ __device__ constexpr int stage_grp_bytes(int G) { return G == 1 ? 1536 : 2048; }
// LDS read pattern of a group: 0 for the 2 KB row-group shares of E2M1 and
// E4M3 (their fragment reads are the same), 1 for the 1.5 KB ones of E3M2.
__host__ __device__ constexpr int pattern(int G) { return G == 1 ? 1 : 0; }

template <int BN, int BM>
struct Tile {
  static constexpr int WN = BN / 2, WM = BM / 2;    // a wavefront's block
  static constexpr int TN = WN / 32, TM = WM / 32;  // its 32-row fragments
  static constexpr int F = TN + TM;
  static constexpr int kRows = BN + BM;
  static constexpr int kScaleOff = kRows * 64;  // scale words follow the largest code payload (64 B per row)
  static constexpr int kSlotBytes = kScaleOff + kRows * kStepBlocks;
  // The 256 x 128 tile leaves each SIMD the registers of a second wavefront:
  // four producer wavefronts then issue the loads.  A load occupies the CU's
  // texture-address path for about 20 cycles, 560-600 cycles for a stage's 32
  // against 512 of its MFMAs, and a wavefront that issues both in order has its
  // MFMAs wait behind its loads (stage times on 2048 x 4096 x 4096: MFMAs
  // alone 275 ns, with the LDS reads 410, with the loads 390, with both 540).
  static constexpr bool kProducers = BM == 128;
  static constexpr int kThreads = 64 * kWaves * (kProducers ? 2 : 1);
  static constexpr int kSlots = kProducers ? 6 : 4;
  // a wavefront's loads of a stage: a quarter of each operand's codes, and a
  // scale load
  static constexpr int kLoadsW = BN / 64, kLoadsX = BM / 64;
  static constexpr int kCodeLoads = kLoadsW + kLoadsX, kLoads = kCodeLoads + 1;
  static_assert(BN == 256 && (BM == 256 || BM == 128), "tile shapes");
  static_assert(kSlots * kSlotBytes <= kLdsBytes, "the ring fits LDS");
  static_assert((kSlots - 1) * kLoads < 64, "vmcnt range");
};

// vmcnt-only wait (expcnt and lgkmcnt left at their maxima).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// lgkmcnt(0) only.
__device__ __forceinline__ void wait_lgkm0() { __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (3 << 14)); }

// Workgroup barrier that is also a compiler memory barrier but, unlike
// __syncthreads, adds no wait for loads in flight.
__device__ __forceinline__ void barrier() { asm volatile("s_barrier" ::: "memory"); }

// 32-bit LDS address of a pointer into dynamic shared memory.
__device__ __forceinline__ uint32_t lds_addr(const uint8_t* p) {
  return (uint32_t)(size_t)(const __attribute__((address_space(3))) uint8_t*)p;
}

template <typename T>
__device__ __forceinline__ T lds_read(uint32_t addr) {
  return *reinterpret_cast<const __attribute__((address_space(3))) T*>((uintptr_t)addr);
}

// Direct global -> LDS load (GLOBAL_LOAD_LDS_DWORDX4) with a wave-uniform
// 64-bit base in SGPRs and a 32-bit per-lane offset: lane i's 16 bytes land
// at M0 + 16 i (M0 is bound as an operand, so the compiler sets it).  Written
// as inline asm so that the compiler does not track the load (it would
// otherwise wait for every one of them before any LDS read it cannot prove
// disjoint); the ring relies on the explicit vmcnt waits.  The s_nop covers
// the wait state between writing M0 and the load reading it.
__device__ __forceinline__ void dma16_s(uint32_t voff, const void* sbase, uint32_t lds) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(voff), "s"(sbase), "{m0}"(lds) : "memory");
}

// The same for part of the lanes: the exec mask is narrowed inside the asm
// statement (and restored before it ends), so a partial load stays one
// straight-line instruction that the vmcnt bookkeeping counts once.
__device__ __forceinline__ void dma16_masked(uint32_t voff, const void* sbase, uint32_t lds, uint64_t mask) {
  uint64_t saved;
  asm volatile(
      "s_mov_b64 %0, exec\n\t"
      "s_mov_b64 exec, %4\n\t"
      "s_nop 1\n\t"
      "global_load_lds_dwordx4 %1, %2\n\t"
      "s_mov_b64 exec, %0"
      : "=&s"(saved)
      : "v"(voff), "s"(sbase), "{m0}"(lds), "s"(mask)
      : "memory");
}

// A wave-uniform value kept in SGPRs (the compiler is told it is uniform).
__device__ __forceinline__ uint32_t uni(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ const uint8_t* uni(const uint8_t* p) {
  const uint64_t v = (uint64_t)p;
  const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
  return (const uint8_t*)(lo | (hi << 32));
}

// Hide a value from loop-invariant code motion (hoisting every derived
// address out of the K loop would keep them all live across it).
template <typename V>
__device__ __forceinline__ V opaque_s(V v) {
  asm volatile("" : "+s"(v));
  return v;
}

// ---------------------------------------------------------------------------
// DMA cursor: where the next stage to issue comes from and goes to.
// ---------------------------------------------------------------------------

// One operand's codes: at the tile's first row per group, bytes between
// layout steps per group (padded rows x step row bytes), the last row group
// (relative to the tile) with rows, and the LDS offset of its part of a slot
// (2 KB and 1.5 KB row-group shares).
struct DmaCodes {
  const uint8_t *code0, *code1, *code2;
  int64_t rstride0, rstride1, rstride2;
  int last;
  uint32_t lds, lds6;
};

// Per-tile constants of this wavefront's loads.
struct DmaConst {
  DmaCodes w, x;
  const uint8_t* sc;       // this wavefront's operand scales at the tile's first row, layout step 0
  int64_t sstride;         // bytes between layout steps of the scales
  uint32_t soff;           // this lane's byte offset for the scale load
  uint32_t sdst;           // LDS offset of this wavefront's scale words in a slot
  uint64_t smask;          // lanes that take part in the scale load
  int wave;
};

// The state that advances stage by stage.
template <int NW, int NX>
struct DmaCursor {
  const uint8_t *bw, *bx;  // code bases of the next stage to issue
  const uint8_t* bs;       // scale base of the next stage to issue
  int u;                   // its half of the layout step (E3M2 / E4M3)
  // the step to the next stage inside a segment (see run_group): code and
  // scale base increments when u is 0 / 1, and whether u alternates
  int64_t winc0, winc1, xinc0, xinc1, sinc0, sinc1;
  int flip;
  uint32_t wdoff[NW], xdoff[NX];  // this lane's global byte offset for each code load of group g
  uint32_t wmo[NW], xmo[NX];      // LDS offset (in a slot) of each code load of group g
};

// Per-lane offsets of a wavefront's N loads of one operand's share of a group
// G stage (`rows` tile rows): its quarter, completed by repeating pieces (into
// the same LDS bytes with the same data) where the share has fewer.
template <int G, int N>
__device__ __forceinline__ void operand_offsets(const DmaCodes& k, int rows, int wave, uint32_t (&doff)[N],
                                                uint32_t (&mo)[N], int lane) {
  constexpr int GB = stage_grp_bytes(G);
  constexpr int RB = step_row_bytes(G);
  const int n = rows / kRowGroup * GB / 1024;  // 1 KB loads of the operand's share
#pragma unroll
  for (int p = 0; p < N; ++p) {
    int li = wave * n / 4 + p;  // load within the operand's share
    li = li < n ? li : n - 1;
    const int x = li * 1024 + lane * 16;  // this lane's byte within the share
    int grp = x / GB;
    const int within = x - grp * GB;
    grp = grp < k.last ? grp : k.last;  // row groups past the padded rows re-read the last one
    doff[p] = (uint32_t)(grp * kRowGroup * RB + within);
    mo[p] = uni((G == 1 ? k.lds6 : k.lds) + (uint32_t)li * 1024u);
  }
}

template <int BN, int BM>
using Cursor = DmaCursor<Tile<BN, BM>::kLoadsW, Tile<BN, BM>::kLoadsX>;

template <int G, int BN, int BM>
__device__ __forceinline__ void group_offsets(const DmaConst& k, Cursor<BN, BM>& cur, int lane) {
  operand_offsets<G, Tile<BN, BM>::kLoadsW>(k.w, BN, k.wave, cur.wdoff, cur.wmo, lane);
  operand_offsets<G, Tile<BN, BM>::kLoadsX>(k.x, BM, k.wave, cur.xdoff, cur.xmo, lane);
}

// Stage boundaries: group 0 is [0, q1), group 1 [q1, q2), group 2 [q2, Q);
// t1, t2 the first layout steps of groups 1 and 2 in the scale buffer.
struct Stages {
  int q1, q2, Q, t1, t2;
};

__device__ __forceinline__ int stage_group(const Stages& S, int q) { return q < S.q1 ? 0 : (q < S.q2 ? 1 : 2); }

// Point the cursor at the s-th stage of group G: its bases, the group's offsets
// and the increments to the stages after it.
template <int G, int BN, int BM>
__device__ __forceinline__ void cursor_group(const DmaConst& k, const Stages& S, Cursor<BN, BM>& cur, int s, int lane) {
  const int64_t ws = G == 0 ? k.w.rstride0 : (G == 1 ? k.w.rstride1 : k.w.rstride2);
  const int64_t xs = G == 0 ? k.x.rstride0 : (G == 1 ? k.x.rstride1 : k.x.rstride2);
  const int step = G == 0 ? s : s >> 1;
  const int u = G == 0 ? 0 : s & 1;
  const int64_t half = stage_grp_bytes(G);  // to the second half of a step (E3M2 / E4M3)
  cur.u = u;
  cur.bw = uni((G == 0 ? k.w.code0 : (G == 1 ? k.w.code1 : k.w.code2)) + step * ws + u * half);
  cur.bx = uni((G == 0 ? k.x.code0 : (G == 1 ? k.x.code1 : k.x.code2)) + step * xs + u * half);
  cur.bs = uni(k.sc + (int64_t)((G == 0 ? 0 : (G == 1 ? S.t1 : S.t2)) + step) * k.sstride);
  cur.winc0 = G == 0 ? ws : half;
  cur.winc1 = G == 0 ? ws : ws - half;
  cur.xinc0 = G == 0 ? xs : half;
  cur.xinc1 = G == 0 ? xs : xs - half;
  cur.sinc0 = G == 0 ? k.sstride : 0;
  cur.sinc1 = k.sstride;
  cur.flip = G == 0 ? 0 : 1;
  group_offsets<G, BN, BM>(k, cur, lane);
}

// Point the cursor at stage q.
template <int BN, int BM>
__device__ __forceinline__ void cursor_at(const DmaConst& k, const Stages& S, Cursor<BN, BM>& cur, int q, int lane) {
  if (q < S.q1)
    cursor_group<0, BN, BM>(k, S, cur, q, lane);
  else if (q < S.q2)
    cursor_group<1, BN, BM>(k, S, cur, q - S.q1, lane);
  else
    cursor_group<2, BN, BM>(k, S, cur, q - S.q2, lane);
}

// One stage on inside a group: no branch, the offsets untouched.
template <int NW, int NX>
__device__ __forceinline__ void cursor_step(DmaCursor<NW, NX>& cur) {
  cur.bw = uni(cur.bw + (cur.u ? cur.winc1 : cur.winc0));
  cur.bx = uni(cur.bx + (cur.u ? cur.xinc1 : cur.xinc0));
  cur.bs = uni(cur.bs + (cur.u ? cur.sinc1 : cur.sinc0));
  cur.u ^= cur.flip;
}

// Point the cursor at stage qr for a run of stages whose refills stay in
// qr's group (hold = true: every refill of the run is qr itself, the last
// stage).  Only here do the group's per-lane offsets change.
template <int BN, int BM>
__device__ __forceinline__ void cursor_segment(const DmaConst& k, const Stages& S, Cursor<BN, BM>& cur, int qr, bool hold,
                                               int lane) {
  cursor_at<BN, BM>(k, S, cur, qr, lane);
  if (hold) {
    cur.winc0 = cur.winc1 = cur.xinc0 = cur.xinc1 = cur.sinc0 = cur.sinc1 = 0;
    cur.flip = 0;
  }
}

// Load P of the stage the cursor points at, into the slot at LDS byte
// address st: the weight rows' codes, the activation rows', the scales.
template <int P, int BN, int BM>
__device__ __forceinline__ void issue_load(const DmaConst& k, const Cursor<BN, BM>& cur, uint32_t st) {
  using T = Tile<BN, BM>;
  if constexpr (P < T::kLoadsW)
    dma16_s(cur.wdoff[P], cur.bw, st + cur.wmo[P]);
  else if constexpr (P < T::kCodeLoads)
    dma16_s(cur.xdoff[P - T::kLoadsW], cur.bx, st + cur.xmo[P - T::kLoadsW]);
  else
    dma16_masked(k.soff, cur.bs, st + k.sdst, k.smask);
}

// ---------------------------------------------------------------------------
// Operands in registers and the MFMAs.
// ---------------------------------------------------------------------------

// Registers of one stage's operands, any group: TN weight then TM
// activation fragments of 8 dwords, and the raw scale words of their rows
// in the same order.  E2M1: dwords 0-3 hold the stage's first 64-channel
// slice and 4-7 its second; E3M2: dwords 0-5; E4M3: all 8.
template <int BN, int BM>
struct Ops {
  v8i f[Tile<BN, BM>::F];
  int s[Tile<BN, BM>::F];
};

// LDS byte addresses of one stage's reads for this lane.
struct OpsAddr {
  uint32_t w, x, sw, sx;
};

template <int PT, int BN, int BM>
__device__ __forceinline__ OpsAddr ops_addr(uint32_t st, int wn0, int wm0, int lane) {
  using T = Tile<BN, BM>;
  constexpr int GB = PT == 0 ? 2048 : 1536;
  constexpr int kWBytes = BN / kRowGroup * GB;
  const int g = lane >> 5, r = lane & 31;
  const int part = PT == 0 ? g * 512 + r * 16 : g * 768 + r * 24;
  OpsAddr ad;
  ad.w = st + wn0 / kRowGroup * GB + part;
  ad.x = st + kWBytes + wm0 / kRowGroup * GB + part;
  ad.sw = st + T::kScaleOff + (wn0 + r) * kStepBlocks;
  ad.sx = st + T::kScaleOff + (BN + wm0 + r) * kStepBlocks;
  return ad;
}

// This lane's fragment at LDS byte address p (block-major record).
// Pattern 0: lane 32 g + r reads 16 bytes of block g and 16 of block 2 + g
// (E2M1: block g of each slice; E4M3: channels 16g .. 16g+15 of each of the
// slice's two blocks).  Pattern 1 (E3M2): the 24 bytes of block g.
template <int PT>
__device__ __forceinline__ void read_frag(v8i& v, uint32_t p) {
  if constexpr (PT == 0) {
    const u32x4 lo = lds_read<u32x4>(p), hi = lds_read<u32x4>(p + 1024);
    v = v8i{(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
  } else {
    const u32x2 d0 = lds_read<u32x2>(p), d1 = lds_read<u32x2>(p + 8), d2 = lds_read<u32x2>(p + 16);
    v[0] = (int)d0.x;
    v[1] = (int)d0.y;
    v[2] = (int)d1.x;
    v[3] = (int)d1.y;
    v[4] = (int)d2.x;
    v[5] = (int)d2.y;
  }
}

// Read item I of a stage into o: the scale words of the weight rows and of
// the activation rows first (they are needed first), then weight fragments
// 0..TN-1 and activation fragments.
template <int PT, int I, int BN, int BM>
__device__ __forceinline__ void read_item(Ops<BN, BM>& o, const OpsAddr& ad) {
  using T = Tile<BN, BM>;
  constexpr int GB = PT == 0 ? 2048 : 1536;
  if constexpr (I < T::F) {
    if constexpr (I < T::TN) o.s[I] = lds_read<int>(ad.sw + I * kRowGroup * kStepBlocks);
    else o.s[I] = lds_read<int>(ad.sx + (I - T::TN) * kRowGroup * kStepBlocks);
  } else {
    constexpr int f = I - T::F;
    if constexpr (f < T::TN) read_frag<PT>(o.f[f], ad.w + f * GB);
    else read_frag<PT>(o.f[f], ad.x + (f - T::TN) * GB);
  }
}

template <int PT, int I0, int I1, int BN, int BM>
__device__ __forceinline__ void read_items(Ops<BN, BM>& o, const OpsAddr& ad) {
  if constexpr (I0 < I1) {
    read_item<PT, I0>(o, ad);
    read_items<PT, I0 + 1, I1>(o, ad);
  }
}

template <int BN, int BM>
using Acc = v16f[Tile<BN, BM>::TN][Tile<BN, BM>::TM];

// The MFMA operand of one slice of a fragment.
template <int G, int KK>
__device__ __forceinline__ v8i operand(const v8i& f) {
  if constexpr (G == 0) return KK == 0 ? v8i{f[0], f[1], f[2], f[3], 0, 0, 0, 0} : v8i{f[4], f[5], f[6], f[7], 0, 0, 0, 0};
  else if constexpr (G == 1) return v8i{f[0], f[1], f[2], f[3], f[4], f[5], 0, 0};
  else return f;
}

// Loads P0 .. P1-1 of the refill.
template <int P0, int P1, int BN, int BM>
__device__ __forceinline__ void issue_loads(const DmaConst& k, const Cursor<BN, BM>& cur, uint32_t st) {
  if constexpr (P0 < P1) {
    issue_load<P0, BN, BM>(k, cur, st);
    issue_loads<P0 + 1, P1, BN, BM>(k, cur, st);
  }
}

// Kernel-wide state of one tile.
template <int BN, int BM>
struct Ctx {
  DmaConst k;
  Stages S;
  uint32_t lds0;
  int wn0, wm0, lane;
};

// What moves on from stage to stage: the slot in use, the LDS addresses of the
// next stage's reads, the DMA cursor and the next stage's scale shift.
template <int BN, int BM>
struct Loop {
  uint32_t st;     // slot of the stage whose MFMAs run
  OpsAddr ad;      // reads of the stage after it
  Cursor<BN, BM> dma;
  int shift;       // 8 g, + 16 in the second half of an E3M2 / E4M3 step, of the stage after it
};

// Shift scale words F0 .. F1-1 down to what their lanes feed the MFMA.
template <int F0, int F1, int BN, int BM>
__device__ __forceinline__ void shift_scales(Ops<BN, BM>& o, int shift) {
#pragma unroll
  for (int f = F0; f < F1; ++f) o.s[f] = (int)((uint32_t)o.s[f] >> shift);
}

// The MFMAs of one group-G stage q (acc += W x X^T), in program order: E2M1
// runs its first slice over every accumulator, then its second (so no MFMA
// waits for the one before it).  Lane 32 g + r needs the scale of block
// 2 kk' + g of its row, kk' the slice's 64-channel position in the layout
// step: o.s holds the scale words shifted right by 8 g (+ 16 for the second
// half of an E3M2 / E4M3 step) and op_sel picks byte 2 kk (kk the slice
// within the stage).
//
// Everything else the stage does goes out behind one of its MFMAs, so that
// between two stages' MFMAs nothing is left to issue (with the cursor, the
// addresses, the scale shifts and the waits between the stages, the matrix
// cores idled for 200-400 cycles of each):
//  - the first three quarters (kR): the loads that refill stage q's slot and
//    the reads of stage q+1 (for the group's last stage they are of no use,
//    harmlessly, and the next group reads its first stage again);
//  - then the cursor's and the addresses' step to the next stage;
//  - three MFMAs before the end the synchronisation that the next stage
//    needs: this wavefront's reads of stage q+1 are done (its slot is
//    refilled next), its loads of stage q+2 have landed (every stage issues
//    kLoads, and the NS - 2 stages after q+2 may still be in flight), and so
//    for everyone at the barrier;
//  - behind the last two, stage q+1's scale shifts.
template <int G, int FS, int T, int BN, int BM>
__device__ __forceinline__ void mfma_block(const Ctx<BN, BM>& c, Acc<BN, BM>& acc, const Ops<BN, BM>& o,
                                           Ops<BN, BM>& nxt, Loop<BN, BM>& l) {
  using Ti = Tile<BN, BM>;
  constexpr int TN = Ti::TN, TM = Ti::TM, F = Ti::F, NS = Ti::kSlots;
  constexpr int kPer = TN * TM;
  constexpr int kM = stage_slices(G) * kPer;
  constexpr int kR = kM == 8 ? 4 : kM * 3 / 4, kS = kM - 3;
  if constexpr (T < kM) {
    constexpr int fmt = group_fmt(G, FS);
    constexpr int KK = T / kPer, i = (T % kPer) / TM, j = T % TM;
    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(operand<G, KK>(o.f[i]), operand<G, KK>(o.f[TN + j]),
                                                                acc[i][j], fmt, fmt, 2 * KK, o.s[i], 2 * KK, o.s[TN + j]);
    if constexpr (T < kR) {
      constexpr int kLoads = Ti::kLoads, kItems = 2 * F;
      if constexpr (!Ti::kProducers)
        issue_loads<(T * kLoads + kR - 1) / kR, ((T + 1) * kLoads + kR - 1) / kR, BN, BM>(c.k, l.dma, l.st);
      read_items<pattern(G), T * kItems / kR, (T + 1) * kItems / kR>(nxt, l.ad);
    }
    if constexpr (T == kR && !Ti::kProducers) cursor_step(l.dma);
    if constexpr (T == kR + 1) {
      const uint32_t st_end = c.lds0 + NS * Ti::kSlotBytes;
      l.st = uni(l.st + Ti::kSlotBytes < st_end ? l.st + Ti::kSlotBytes : c.lds0);
      const uint32_t after = l.st + Ti::kSlotBytes < st_end ? l.st + Ti::kSlotBytes : c.lds0;
      l.ad = ops_addr<pattern(G), BN, BM>(after, opaque_s(c.wn0), opaque_s(c.wm0), c.lane);
    }
    if constexpr (T == kS) {
      wait_lgkm0();
      if constexpr (!Ti::kProducers) wait_vmcnt<(NS - 2) * Ti::kLoads>();
      barrier();
    }
    if constexpr (T == kM - 2) shift_scales<0, F / 2>(nxt, l.shift);
    if constexpr (T == kM - 1) {
      shift_scales<F / 2, F>(nxt, l.shift);
      if constexpr (G >= 1) l.shift ^= 16;
    }
    __builtin_amdgcn_sched_barrier(0);
    mfma_block<G, FS, T + 1>(c, acc, o, nxt, l);
  }
}

// All stages of group G, two per iteration (the operand registers
// alternate).  On entry the group's first stage has landed for everyone and
// l.st is its slot; on exit the same holds for the next group's.  The first
// MFMAs need the second stage as well: it has landed behind the barrier in
// front of them.  The cursor is pointed while the first stage's reads run;
// behind the barrier it held a tile's first MFMAs back by 0.3-0.4 us (us, M x K
// x N: 768 x 128 x 22016 in E2M1 19.0 -> 18.0, 8192 x 128 x 28672 132.5 -> 127.5,
// 4096 x 4096 x 14336 149.4 -> 146.4).
template <int G, int FS, int BN, int BM>
__device__ __forceinline__ void run_group(const Ctx<BN, BM>& c, Acc<BN, BM>& acc, Loop<BN, BM>& l) {
  using T = Tile<BN, BM>;
  const int qb = G == 0 ? 0 : (G == 1 ? c.S.q1 : c.S.q2);
  const int qe = G == 0 ? c.S.q1 : (G == 1 ? c.S.q2 : c.S.Q);
  if (qb == qe) return;
  constexpr int NS = T::kSlots;
  const Stages& S = c.S;
  Ops<BN, BM> A, B;
  read_items<pattern(G), 0, 2 * T::F>(A, ops_addr<pattern(G), BN, BM>(l.st, c.wn0, c.wm0, c.lane));
  const uint32_t after = l.st + T::kSlotBytes < c.lds0 + NS * T::kSlotBytes ? l.st + T::kSlotBytes : c.lds0;
  l.ad = ops_addr<pattern(G), BN, BM>(after, c.wn0, c.wm0, c.lane);
  l.shift = 8 * (c.lane >> 5);
  // segments: runs of stages whose refills (stage q + NS, the last one
  // again past the end) stay in one group, so that inside a run the cursor
  // only steps; it is re-pointed between runs.  Points it at stage q's refill and
  // gives the run's end.
  auto segment = [&](int q) {
    const int qr = q + NS < S.Q ? q + NS : S.Q - 1;
    const bool hold = q + NS >= S.Q - 1;
    int e = qe;
    if (!hold) {
      const int gr = stage_group(S, qr);
      if (gr == 0 && S.q1 - NS < e) e = S.q1 - NS;
      if (gr <= 1 && S.q2 - NS < e) e = S.q2 - NS;
      if (S.Q - 1 - NS < e) e = S.Q - 1 - NS;
    }
    cursor_segment<BN, BM>(c.k, S, l.dma, qr, hold, c.lane);
    return e > q ? e : q + 1;
  };
  int e = qe;
  if constexpr (!T::kProducers) {
    e = segment(qb);  // (while the reads run)
    __builtin_amdgcn_sched_barrier(0);
  }
  shift_scales<0, T::F>(A, l.shift);
  if constexpr (G >= 1) l.shift ^= 16;
  wait_lgkm0();
  if constexpr (!T::kProducers) wait_vmcnt<(NS - 2) * T::kLoads>();  // (nothing to wait for but at the tile's start)
  barrier();  // everyone has read the first stage: its slot may be refilled
  if constexpr (T::kProducers) {
    int q = qb;
    for (; q + 1 < qe; q += 2) {
      mfma_block<G, FS, 0>(c, acc, A, B, l);
      mfma_block<G, FS, 0>(c, acc, B, A, l);
    }
    if (q < qe) mfma_block<G, FS, 0>(c, acc, A, B, l);
    return;
  }
  int q = qb;
  while (true) {
    for (; q + 1 < e; q += 2) {
      mfma_block<G, FS, 0>(c, acc, A, B, l);
      mfma_block<G, FS, 0>(c, acc, B, A, l);
    }
    if (q < e) {
      mfma_block<G, FS, 0>(c, acc, A, B, l);
      A = B;  // the next run starts from A
      ++q;
    }
    if (q >= qe) break;
    e = segment(q);
  }
}

// Fill the ring (issues past the last stage repeat it) and wait for the first
// stage.
template <int BN, int BM>
__device__ __forceinline__ void fill_ring(const Ctx<BN, BM>& c, Cursor<BN, BM>& cur) {
  using T = Tile<BN, BM>;
  for (int q = 0; q < T::kSlots; ++q) {
    const int qi = q < c.S.Q ? q : c.S.Q - 1;
    if (q == 0 || qi == c.S.q1 || qi == c.S.q2) cursor_at<BN, BM>(c.k, c.S, cur, qi, c.lane);
    issue_loads<0, T::kLoads, BN, BM>(c.k, cur, uni(c.lds0 + q * T::kSlotBytes));
    if (qi + 1 < c.S.Q) cursor_step(cur);
  }
  wait_vmcnt<(T::kSlots - 1) * T::kLoads>();
  barrier();
}

// A producer wavefront: after each barrier behind which a stage's slot is free
// (everyone has read the stage) the loads of the stage kSlots on, then its own
// loads of the stage two on have landed, and the barrier that says so.  The
// barriers are those of run_group.  The K loop starts behind the first kStart
// stages; the rest of the ring fills two stages at a time behind the first
// ones (filled whole at the start, it held the K loop back by 1 us).
template <int BN, int BM>
__device__ __forceinline__ void produce(const Ctx<BN, BM>& c) {
  using T = Tile<BN, BM>;
  constexpr int NS = T::kSlots, L = T::kLoads, kStart = 3;
  static_assert(NS == 2 * kStart, "three turns of two stages reach the steady distance");
  Cursor<BN, BM> cur;
  uint32_t st = c.lds0;
  int s = 0;  // next stage to issue (past the end the last one again)
  auto issue = [&]() {
    const int qi = s < c.S.Q ? s : c.S.Q - 1;
    if (s == 0 || qi == c.S.q1 || qi == c.S.q2) cursor_at<BN, BM>(c.k, c.S, cur, qi, c.lane);
    issue_loads<0, L, BN, BM>(c.k, cur, uni(st));
    if (qi + 1 < c.S.Q) cursor_step(cur);
    st = st + T::kSlotBytes < c.lds0 + NS * T::kSlotBytes ? st + T::kSlotBytes : c.lds0;
    ++s;
  };
  for (int k = 0; k < kStart; ++k) issue();
  wait_vmcnt<(kStart - 1) * L>();
  barrier();  // the first stage has landed
  wait_vmcnt<(kStart - 2) * L>();
  for (int q = 0; q < c.S.Q; ++q) {
    if (q == 0 || q == c.S.q1 || q == c.S.q2) barrier();  // a group's first stage has been read (and at 0 the second has landed)
    if (q < kStart) issue();  // into a slot that no stage has used yet, or one free since the last barrier
    issue();
    // stage q + 2 has landed: the stages issued after it may be in flight
    if (q == 0) wait_vmcnt<2 * L>();
    else if (q == 1) wait_vmcnt<3 * L>();
    else wait_vmcnt<(NS - 2) * L>();
    barrier();
  }
}

}  // namespace tiled

using namespace tiled;

template <int BN, int BM, int FS>
__global__ __launch_bounds__((Tile<BN, BM>::kThreads), 1) void gemm_tiled_kernel(GemmArgs a, int tiles_n, int tiles_m) {
  using T = Tile<BN, BM>;
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  constexpr int kGroupN = 4;  // weight tiles that share an XCD's L2 at a time

  // workgroup -> tile: consecutive tiles per XCD (workgroups are dealt to the
  // 8 XCDs round-robin), then groups of kGroupN weight tiles, activation
  // tiles fastest inside a group
  const int nt = tiles_n * tiles_m;
  const int wg = blockIdx.x;
  const int xcd = wg & 7, kq = wg >> 3;
  const int per_x = nt >> 3, extra = nt & 7;
  const int t = xcd * per_x + (xcd < extra ? xcd : extra) + kq;
  const int grp = t / (kGroupN * tiles_m);
  const int within = t - grp * kGroupN * tiles_m;
  const int gn = tiles_n - grp * kGroupN < kGroupN ? tiles_n - grp * kGroupN : kGroupN;
  const int tn = grp * kGroupN + within % gn;
  const int tm = within / gn;
  const int64_t n0 = (int64_t)tn * BN, m0 = (int64_t)tm * BM;

  Ctx<BN, BM> c;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform: keeps DMA setup scalar
  c.lane = threadIdx.x & 63;
  const int w4 = T::kProducers ? wave & 3 : wave;  // (producers: which quarter of the loads)
  c.wn0 = (w4 & 1) * T::WN;
  c.wm0 = (w4 >> 1) * T::WM;
  c.lds0 = lds_addr(lds);
  c.S.q1 = a.steps[0];
  c.S.q2 = c.S.q1 + 2 * a.steps[1];
  c.S.Q = c.S.q2 + 2 * a.steps[2];
  c.S.t1 = a.steps[0];
  c.S.t2 = a.steps[0] + a.steps[1];

  DmaConst& k = c.k;
  k.wave = w4;
  auto codes = [&](DmaCodes& d, const Operand& o, int64_t r0) {  // r0: the tile's first row (below its padded rows - 31)
    d.code0 = o.q[0] + r0 * step_row_bytes(0);
    d.code1 = o.q[1] + r0 * step_row_bytes(1);
    d.code2 = o.q[2] + r0 * step_row_bytes(2);
    d.rstride0 = o.rp * step_row_bytes(0);
    d.rstride1 = o.rp * step_row_bytes(1);
    d.rstride2 = o.rp * step_row_bytes(2);
    d.last = (int)(o.rp / kRowGroup - r0 / kRowGroup - 1);
  };
  codes(k.w, a.w, n0);
  codes(k.x, a.x, m0);
  k.w.lds = k.w.lds6 = 0;
  k.x.lds = BN / kRowGroup * 2048;
  k.x.lds6 = BN / kRowGroup * 1536;
  const int op = w4 >> 1, half = w4 & 1;  // of the scale load: wavefronts 0-1 the weight rows, 2-3 the activation rows
  const Operand& o = op ? a.x : a.w;
  const int64_t r0 = op ? m0 : n0;
  // scale words (4 bytes per row and step): one half of the operand's rows,
  // 4 rows per lane; rows past the padded rows re-read the last 4
  const int per = (op ? BM : BN) / 2;
  int64_t row = half * per + c.lane * 4;  // row within the tile
  row = r0 + row + 4 <= o.rp ? row : o.rp - 4 - r0;
  k.soff = (uint32_t)row * kStepBlocks;
  k.sdst = (uint32_t)(T::kScaleOff + (op ? BN * kStepBlocks : 0) + half * per * kStepBlocks);
  k.smask = per / 4 >= 64 ? ~0ull : ((1ull << (per / 4)) - 1);
  k.sc = o.sc + r0 * kStepBlocks;
  k.sstride = o.rp * kStepBlocks;

  Acc<BN, BM> acc;
#pragma unroll
  for (int i = 0; i < T::TN; ++i)
#pragma unroll
    for (int j = 0; j < T::TM; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;

  const bool producer = T::kProducers && wave >= kWaves;
  if (producer) {
    if constexpr (T::kProducers) produce(c);
  } else {
    // the K loop, group by group
    Loop<BN, BM> l;
    if constexpr (T::kProducers) barrier();  // the ring's first stage has landed
    else fill_ring(c, l.dma);
    l.st = uni(c.lds0);
    run_group<0, FS>(c, acc, l);
    run_group<1, FS>(c, acc, l);
    run_group<2, FS>(c, acc, l);
  }

  // Epilogue: every load and read of the ring is done (the last stages
  // issued repeats of the last one); the bf16 tile is assembled in LDS and
  // written out as whole rows, 16 bytes per lane, so every store fills full
  // cache lines.  Lane 32 g + r, register q holds output column
  // n = 8 (q/4) + 4 g + q%4 of its fragment and output row m = r.  Rows are
  // padded by 16 bytes: the fragment writes of 32 lanes (32 rows) then fall
  // on distinct banks.
  wait_vmcnt<0>();
  wait_lgkm0();
  barrier();
  constexpr int kRowStride = BN * 2 + 16;
  static_assert(BM * kRowStride <= kLdsBytes, "epilogue tile fits LDS");
  const int r = c.lane & 31, g = c.lane >> 5;
  if (!producer) {
#pragma unroll
    for (int i = 0; i < T::TN; ++i)
#pragma unroll
      for (int j = 0; j < T::TM; ++j) {
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          const uint32_t lo = pack_bf16x2_rne(acc[i][j][4 * h], acc[i][j][4 * h + 1]);
          const uint32_t hi = pack_bf16x2_rne(acc[i][j][4 * h + 2], acc[i][j][4 * h + 3]);
          const uint32_t at = c.lds0 + (c.wm0 + 32 * j + r) * kRowStride + (c.wn0 + 32 * i + 8 * h + 4 * g) * 2;
          *reinterpret_cast<__attribute__((address_space(3))) u32x2*>((uintptr_t)at) = u32x2{lo, hi};
        }
        // one accumulator tile at a time: keeps the VGPR copies of the
        // accumulators few
        __builtin_amdgcn_sched_barrier(0);
      }
  }
  __syncthreads();
  constexpr int kChunks = BN / 8;  // 16-byte chunks per row
  const int64_t M = a.x.rows, N = a.w.rows;
  for (int ch = threadIdx.x; ch < BM * kChunks; ch += T::kThreads) {
    const int rr = ch / kChunks, col = (ch - rr * kChunks) * 8;
    const int64_t m = m0 + rr, n = n0 + col;
    if (m >= M || n >= N) continue;
    const u32x4 v = lds_read<u32x4>(c.lds0 + rr * kRowStride + col * 2);
    uint16_t* dst = a.y + m * a.ldy + n;
    if (n + 8 <= N) {
      // streamed: the output is not read again here, and keeping it out of
      // the L2 leaves the operand panels of the tiles still running there
      __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(dst));
    } else {
      for (int e = 0; e < (int)(N - n); ++e) {
        const uint32_t wd = e < 2 ? v.x : (e < 4 ? v.y : (e < 6 ? v.z : v.w));
        dst[e] = (uint16_t)(wd >> (16 * (e & 1)));
      }
    }
  }
}

template <int BN, int BM, int FS>
static hipError_t launch_tile_fs(const GemmArgs& a, const Device& dev, hipStream_t stream) {
  static DeviceOnce once;
  hipError_t e = allow_lds(once, dev, reinterpret_cast<const void*>(gemm_tiled_kernel<BN, BM, FS>), kLdsBytes);
  if (e != hipSuccess) return e;
  const int tn = (int)((a.w.rows + BN - 1) / BN), tm = (int)((a.x.rows + BM - 1) / BM);
  hipLaunchKernelGGL((gemm_tiled_kernel<BN, BM, FS>), dim3((unsigned)(tn * tm)), dim3(Tile<BN, BM>::kThreads), kLdsBytes, stream, a,
                     tn, tm);
  return hipGetLastError();
}

// The format set is an instruction immediate: one kernel per set.
template <int BN, int BM>
static hipError_t launch_tile(const GemmArgs& a, const Device& dev, hipStream_t stream) {
  switch (a.fs) {
    case 0: return launch_tile_fs<BN, BM, 0>(a, dev, stream);
    case 1: return launch_tile_fs<BN, BM, 1>(a, dev, stream);
    case 2: return launch_tile_fs<BN, BM, 2>(a, dev, stream);
    case 3: return launch_tile_fs<BN, BM, 3>(a, dev, stream);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_tiled(const GemmArgs& a, bool square, const Device& dev, hipStream_t stream) {
  return square ? launch_tile<256, 256>(a, dev, stream) : launch_tile<256, 128>(a, dev, stream);
}

}  // namespace mm
