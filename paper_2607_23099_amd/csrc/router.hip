// Router of the MoE layer (Sec. II-A): gating logits x * Wg^T (+ bias), the k largest logits
// per token and the softmax over them.  Its cost belongs to the end-to-end layer the paper
// times inside one graph (Sec. V-C).
//
// Two kernels a call, both deterministic.  The logits (bf16 MFMA 32x32x16, fp32 partial sums [S][T][E] in
// the workspace) come from one of three:
//   k_router_logits<1, 4, 2>  few tokens: 32 tokens x 64 experts a block, whose 4 waves split the
//                             block's K range; the gate matrix is the traffic, so it is spread over
//                             many blocks.
//   k_router_logits_lds       from 8 tiles of 128 tokens on, up to 512 experts: 128 tokens x all
//                             experts a block, both operands through LDS rings.
//   k_router_logits<4, 2, 3>  many tokens and more experts: 128 tokens x 64 experts a block, two waves
//                             per 32-token slice along K, the gate tile shared through L1.
// Then k_router_topk_* sums the S partials in split order (a block per token when S is large, a wave per
// token otherwise), adds the bias, selects the top k with an order-preserving integer key (ties to the
// lower expert id) and writes ids and softmax gates.
#include <type_traits>

#include "common.h"
#include "device.h"

namespace damoe {
namespace {

constexpr int kTok = 32;           // tokens per wave tile (MFMA rows)
constexpr int kExpTile = 64;       // experts per block tile (two 32-wide MFMA blocks)
constexpr int kStepK = 64;         // k per step: 128 contiguous bytes of each row
constexpr int kTargetBlocks = 256; // blocks the few-token plan aims for (one per compute unit)
constexpr int kLdsMinTiles = 8;    // 128-token tiles from which the LDS kernel takes over

struct LogitsArgs {
  const uint16_t* x;   // [T][H]
  const uint16_t* wg;  // [E][H]
  float* part;         // [S][T][E]
  int32_t T, H, E, S;
  int32_t tiles_t, tiles_e, n_items, per_xcd;
};

struct TopkArgs {
  const float* part;   // [S][T][E]
  const float* bias;   // [E] or null
  float* logits;       // [T][E] or null
  int32_t* ids;        // [T][k]
  float* w;            // [T][k]
  int32_t T, E, k, S;
};

// WT waves along tokens (32 tokens each) x WK waves along K; NB register sets of operands
// (NB - 1 steps of loads in flight while one multiplies).
template <int WT, int WK, int NB>
__global__ __launch_bounds__(kWave * WT * WK) void k_router_logits(LogitsArgs a) {
  pin(a.x);
  pin(a.wg);
  pin(a.part);
  pin(a.T);
  pin(a.H);
  pin(a.E);
  pin(a.S);
  // Blocks b and b + 8 share an XCD (and its L2): give each XCD a contiguous run of items,
  // token tiles fastest, so the blocks reading one gate-matrix slice sit on one L2.
  const int b = blockIdx.x;
  const int item = (b & 7) * a.per_xcd + (b >> 3);
  if (item >= a.n_items) return;
  const int tt = item % a.tiles_t;
  const int et = (item / a.tiles_t) % a.tiles_e;
  const int s = item / (a.tiles_t * a.tiles_e);

  // The wave index is uniform within a wave; in a scalar register the K range and the
  // buffer offsets derived from it stay scalar (no per-lane loop around each buffer load).
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tw = wave % WT, kw = wave / WT;
  const int r = lane & 31, h = lane >> 5;
  const int t0 = tt * kTok * WT + tw * kTok;
  const int e0 = et * kExpTile;
  const uint32_t row_bytes = (uint32_t)a.H * 2u;

  const __amdgpu_buffer_rsrc_t rx = make_rsrc(a.x, (uint32_t)a.T * row_bytes);
  const __amdgpu_buffer_rsrc_t rw = make_rsrc(a.wg, (uint32_t)a.E * row_bytes);
  // Lane (r, h) feeds row r with bytes [64 h, 64 h + 64) of each 128-byte step; MFMA i takes
  // the i-th 16 bytes of both halves.  A and B use the same k assignment, so the sum over the
  // step's 64 k values is complete.
  const uint32_t vx = (t0 + r < a.T) ? (uint32_t)(t0 + r) * row_bytes + 64u * h : kOobOffset;
  uint32_t vw[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int e = e0 + 32 * c + r;
    vw[c] = (e < a.E) ? (uint32_t)e * row_bytes + 64u * h : kOobOffset;
  }

  const int steps = a.H / kStepK;
  const int G = a.S * WK, g = s * WK + kw;
  const int st0 = (int)((int64_t)g * steps / G), st1 = (int)((int64_t)(g + 1) * steps / G);

  floatx16 acc[2];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[c][i] = 0.0f;

  // A ring of NB register sets.  Loads beyond the last step re-read that step (in bounds,
  // unused).
  uint4 xa[NB][4], wb[NB][2][4];
  auto load = [&](int st, int buf) {
    const uint32_t soff = (uint32_t)min(st, st1 - 1) * (kStepK * 2);
#pragma unroll
    for (int i = 0; i < 4; ++i) xa[buf][i] = buf_load<uint4, 0>(rx, vx + 16u * i, soff);
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) wb[buf][c][i] = buf_load<uint4, 0>(rw, vw[c] + 16u * i, soff);
  };
  auto mul = [&](int buf) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int c = 0; c < 2; ++c) acc[c] = mfma32x32x16(xa[buf][i], wb[buf][c][i], acc[c]);
  };
  // Invariant at the top of each group: register set u holds step st + u for u < NB - 1.
  // Whole groups run without guards (one path, so the compiler's wait counts are exact); the
  // fewer than NB steps left over are then already in flight and only multiply.
  if (st0 < st1) {
#pragma unroll
    for (int i = 0; i < NB - 1; ++i) load(st0 + i, i);
    int st = st0;
    for (; st + NB <= st1; st += NB) {
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        // The scheduler would sink the prefetch below the multiplies; keep the issue order.
        load(st + u + NB - 1, (u + NB - 1) % NB);
        __builtin_amdgcn_sched_barrier(0);
        mul(u);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int u = 0; u < NB - 1; ++u)
      if (st + u < st1) mul(u);
  }

  // Output element (token 8 (q / 4) + 4 h + q % 4, expert 32 c + r) of accumulator register q.
  // With WK > 1 the K slices meet in LDS and the first slice's waves add them in slice order.
  float* out = a.part + (size_t)s * a.T * a.E;
  if constexpr (WK > 1) {
    __shared__ float red[WK - 1][WT * kTok][kExpTile + 1];
    if (kw > 0) {
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int q = 0; q < 16; ++q)
          red[kw - 1][tw * kTok + 8 * (q >> 2) + 4 * h + (q & 3)][32 * c + r] = acc[c][q];
    }
    __syncthreads();
    if (kw > 0) return;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int q = 0; q < 16; ++q)
#pragma unroll
        for (int w = 0; w < WK - 1; ++w)
          acc[c][q] += red[w][tw * kTok + 8 * (q >> 2) + 4 * h + (q & 3)][32 * c + r];
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int e = e0 + 32 * c + r;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int t = t0 + 8 * (q >> 2) + 4 * h + (q & 3);
      if (t < a.T && e < a.E) out[(size_t)t * a.E + e] = acc[c][q];
    }
  }
}

typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef uint32_t u32x4_r __attribute__((ext_vector_type(4)));

// 16 bytes per lane from a buffer straight into LDS at dst + 16 lane.
__device__ __forceinline__ void lds_move16(__amdgpu_buffer_rsrc_t r, lds_u8* dst, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)dst, 16, voff, soff, 0, 0);
}

// s_waitcnt vmcnt(VM), other counters left alone (gfx9 encoding).
template <int VM>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(VM >= 0 && VM < 64, "counter range");
  __builtin_amdgcn_s_waitcnt((VM & 15) | (7 << 4) | (15 << 8) | ((VM >> 4) << 14));
}

__device__ __forceinline__ uint4 lds_read16_r(const lds_u8* p) {
  return __builtin_bit_cast(uint4, *reinterpret_cast<const __attribute__((address_space(3))) u32x4_r*>(p));
}

// Many tokens: a block takes 128 tokens and all experts (NE blocks of 32, a quarter of them per
// wave) for one K range of the split, so every token row is read once per split and every gate
// row once per block.  Both operands of each 64-wide K step move into LDS rings with direct
// buffer -> LDS loads, whole 128-byte lines of 8 rows each, and are shared by the 4 waves.  Loaded
// straight into MFMA operands, the gate took 16 bytes of 32 lines an instruction, and the address
// path bounded the kernel (60 us at T = 8192, E = 256 for 12 us of MFMAs).  Waves 0 and 1 move the
// tokens and waves 2 and 3 the gate: each wave counts its own moves, so the token moves (from HBM) run
// further ahead than the gate's (from L2).
// The k assignment is k_router_logits' (lane (r, h): row r, bytes [64 h, 64 h + 64) of the step;
// MFMA i takes the i-th 16 bytes) for both operands.  In LDS a row's 16-byte chunk j sits in slot
// j ^ (row / 2 & 7): the 16 rows of one read phase hit distinct banks.  Per step a wave reads 16 KB of
// tokens and NE / 4 x 4 KB of gate for 4 NE MFMAs.
template <int NE>
struct RouterCfg {
  static constexpr int TB = 4;                            // 32-token blocks per tile
  static constexpr int NW = NE / 4;                       // 32-expert blocks per wave
  static constexpr uint32_t kTokStage = TB * 32 * 128;    // 16 KB
  static constexpr uint32_t kGateStage = NE * 32 * 128;   // 32 KB at E = 256
  static constexpr int NG = NE <= 8 ? 3 : 2;              // stages of the gate ring
  static constexpr int NT = NE <= 12 ? 4 : 2;             // stages of the token ring
  static constexpr uint32_t kGateOff = NT * kTokStage;
  static constexpr size_t kLds = kGateOff + NG * (size_t)kGateStage;
  static_assert(NE % 4 == 0 && kLds <= 160 * 1024, "LDS of one CU");
};

template <int NE>
__global__ __launch_bounds__(256) void k_router_logits_lds(LogitsArgs a) {
  using Cfg = RouterCfg<NE>;
  constexpr int NW = Cfg::NW, TB = Cfg::TB, NT = Cfg::NT, NG = Cfg::NG;
  constexpr int MT = TB * 32 / 8 / 2, MG = NE * 32 / 8 / 2;  // moves per step of a token / gate wave
  extern __shared__ __attribute__((aligned(1024))) uint8_t router_smem[];
  lds_u8* const lds = (lds_u8*)router_smem;
  pin(a.x);
  pin(a.wg);
  pin(a.part);
  pin(a.T);
  pin(a.H);
  pin(a.E);
  pin(a.S);
  const int b = blockIdx.x;
  const int item = (b & 7) * a.per_xcd + (b >> 3);
  if (item >= a.n_items) return;
  const int tt = item % a.tiles_t;
  const int s = item / a.tiles_t;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, h = lane >> 5;
  const int t0 = tt * TB * 32;
  const int e0 = wave * NW * 32;
  const uint32_t row_bytes = (uint32_t)a.H * 2u;
  const int steps = a.H / kStepK;
  const int st0 = (int)((int64_t)s * steps / a.S), n = (int)((int64_t)(s + 1) * steps / a.S) - st0;

  // Rows this wave moves: 8 per move, lane l row l / 8 of them, the chunk that belongs in slot
  // l % 8.  Rows past the last repeat it (their results are not stored).
  const bool tok = wave < 2;
  const int m0 = (wave & 1) * (tok ? MT : MG);  // first move
  constexpr int MM = MT > MG ? MT : MG;
  uint32_t vo[MM];
#pragma unroll
  for (int j = 0; j < MM; ++j) {
    const int row = 8 * (m0 + j) + (lane >> 3);
    const uint32_t chunk = (uint32_t)((lane & 7) ^ ((row >> 1) & 7));
    vo[j] = (uint32_t)(tok ? min(t0 + row, a.T - 1) : min(row, a.E - 1)) * row_bytes + chunk * 16u;
  }
  const void* const src = tok ? (const void*)a.x : (const void*)a.wg;
  const uint32_t src_bytes = (uint32_t)(tok ? a.T : a.E) * row_bytes;
  // Move i of step j (relative to st0); steps past the last go through an empty resource, which reads
  // no memory and keeps the counts of moves in flight.
  auto move_src = [&](int j, __amdgpu_buffer_rsrc_t& rs, uint32_t& soff) __attribute__((always_inline)) {
    rs = make_rsrc(src, j < n ? src_bytes : 0u);
    soff = j < n ? (uint32_t)(st0 + j) * (kStepK * 2) : 0u;
  };
  // This wave's ring: NT stages of tokens or NG of gate rows.
  const uint32_t ring0 = (tok ? 0u : Cfg::kGateOff) + (uint32_t)m0 * 1024u;
  const uint32_t ring_stage = tok ? Cfg::kTokStage : Cfg::kGateStage;
  const int ring_n = tok ? NT : NG;

  floatx16 acc[TB][NW];
#pragma unroll
  for (int tb = 0; tb < TB; ++tb)
#pragma unroll
    for (int c = 0; c < NW; ++c)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[tb][c][i] = 0.0f;

  // Step j: the moves of step j + NT - 1 (tokens) or j + NG - 1 (gate) into the buffer step j - 1 left,
  // the MFMAs of step j with each 16-byte chunk's operands read during the MFMAs of the one before (the
  // last chunk's MFMAs run in the next step), then a wait for this wave's moves of step j + 1 and its
  // LDS reads, and the barrier that publishes step j + 1 and frees step j's buffers.  With one wave per
  // SIMD nothing else fills the matrix cores while a wave issues moves and reads, so those are placed
  // between the MFMAs, one or two behind each (issued ahead of them in one piece, a step took 2680
  // cycles for 1024 of MFMAs).
  auto wait_next = [&]() __attribute__((always_inline)) {
    constexpr int VT = (NT - 2) * MT, VG = (NG - 2) * MG;
    static_assert(VT < 64 && VG < 64, "counter range");
    if (tok) wait_vmcnt<VT>();
    else wait_vmcnt<VG>();
  };
  struct Ops {
    uint4 v[TB + NW];
  };
  constexpr int NM = TB * NW, NR = TB + NW;  // MFMAs and reads of one chunk
  const uint32_t lx = (uint32_t)r * 128u, lsw = (uint32_t)((r >> 1) & 7);
  auto read1 = [&](const lds_u8* tc, const lds_u8* gc, int i, int k, Ops& o) __attribute__((always_inline)) {
    const uint32_t off = lx + (((4u * h + i) ^ lsw) << 4);
    o.v[k] = k < TB ? lds_read16_r(tc + off + k * 4096) : lds_read16_r(gc + off + (e0 + 32 * (k - TB)) * 128);
  };
  auto mul1 = [&](const Ops& o, int m) __attribute__((always_inline)) {
    const int tb = m / NW, c = m % NW;
    acc[tb][c] = mfma32x32x16(o.v[tb], o.v[TB + c], acc[tb][c]);
  };
  Ops A, B;
  int dst_i = ring_n - 1, t_i = 0, g_i = 0;  // ring slots of the moves' and the reads' buffers
  auto step = [&](lds_u8* __restrict__ dst, const lds_u8* __restrict__ tc, const lds_u8* __restrict__ gc, int j)
      __attribute__((always_inline)) {
    __amdgpu_buffer_rsrc_t rs;
    uint32_t soff;
    move_src(j + ring_n - 1, rs, soff);
    // Chunk 0's reads and the moves, between the last chunk's MFMAs of the step before.
    constexpr int MVS = (MM + NM - 1) / NM;  // moves behind each of them
#pragma unroll
    for (int k = 0; k < NR; ++k) read1(tc, gc, 0, k, A);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      if (j > 0) mul1(B, m);
#pragma unroll
      for (int i = m * MVS; i < (m + 1) * MVS; ++i)
        if (i < MT || (i < MG && !tok)) lds_move16(rs, dst + i * 1024, vo[i], soff);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 1; i < 4; ++i) {
      Ops& cur = i % 2 ? A : B;
      Ops& nxt = i % 2 ? B : A;
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        mul1(cur, m);
#pragma unroll
        for (int k = 0; k < NR; ++k)
          if (k * NM / NR == m) read1(tc, gc, i, k, nxt);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    wait_next();
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll 1
  for (int j = 0; j < ring_n - 1; ++j) {
    __amdgpu_buffer_rsrc_t rs;
    uint32_t soff;
    move_src(j, rs, soff);
#pragma unroll
    for (int i = 0; i < MM; ++i)
      if (i < MT || (i < MG && !tok)) lds_move16(rs, lds + ring0 + j * ring_stage + i * 1024, vo[i], soff);
  }
  wait_next();
  __syncthreads();
  for (int j = 0; j < n; ++j) {
    step(lds + ring0 + dst_i * ring_stage, lds + t_i * Cfg::kTokStage, lds + Cfg::kGateOff + g_i * Cfg::kGateStage, j);
    dst_i = dst_i + 1 == ring_n ? 0 : dst_i + 1;
    t_i = t_i + 1 == NT ? 0 : t_i + 1;
    g_i = g_i + 1 == NG ? 0 : g_i + 1;
  }
#pragma unroll
  for (int m = 0; m < NM; ++m) mul1(B, m);
  wait_vmcnt<0>();  // empty moves write LDS too: they must land before the workgroup ends

  // Accumulator register q of block (tb, c): token 32 tb + 8 (q / 4) + 4 h + q % 4, expert
  // e0 + 32 c + r.  The code runs once per wave, so its time is the instruction fetch: whole tiles
  // store with one scalar offset a row and no row check.
  float* out = a.part + ((size_t)s * a.T + t0) * a.E;
  const int rows = min(a.T - t0, TB * 32);
  const __amdgpu_buffer_rsrc_t ro = make_rsrc(out, (uint32_t)rows * (uint32_t)a.E * 4u);
#pragma unroll
  for (int c = 0; c < NW; ++c) {
    const int e = e0 + 32 * c + r;
    const uint32_t vo = e < a.E ? (uint32_t)(4 * h * a.E + e) * 4u : kOobOffset;
    if (rows == TB * 32) {
#pragma unroll
      for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int q = 0; q < 16; ++q)
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[tb][c][q]), ro, vo,
                                                (uint32_t)(32 * tb + 8 * (q >> 2) + (q & 3)) * (uint32_t)a.E * 4u, 0);
    } else {
#pragma unroll
      for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          const int t = 32 * tb + 8 * (q >> 2) + 4 * h + (q & 3);
          if (t < rows && e < a.E) out[(size_t)t * a.E + e] = acc[tb][c][q];
        }
    }
  }
}

// Order-preserving key of a float: larger float -> larger unsigned key; -0 is taken as +0.
__device__ __forceinline__ uint32_t float_key(float f) {
  uint32_t u = __float_as_uint(f);
  if (u == 0x80000000u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float key_float(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp0(uint32_t v) {
  // Lanes of rows outside ROW_MASK read 0, the identity of an unsigned max.
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, false);
}

// Unsigned max over the wave, returned to every lane: butterflies within quads, 8- and
// 16-lane mirrors, then row broadcasts into the last row and a read of lane 63.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  v = max(v, dpp0<0xB1, 0xF>(v));   // quad_perm [1,0,3,2]
  v = max(v, dpp0<0x4E, 0xF>(v));   // quad_perm [2,3,0,1]
  v = max(v, dpp0<0x141, 0xF>(v));  // row_half_mirror
  v = max(v, dpp0<0x140, 0xF>(v));  // row_mirror
  v = max(v, dpp0<0x142, 0xA>(v));  // row_bcast15: rows 1, 3 take rows 0, 2
  v = max(v, dpp0<0x143, 0xC>(v));  // row_bcast31: rows 2, 3 take row 1
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Top-k selection and gates of token t from the E logits the wave holds (expert lane + 64 j
// in v[j], bit j of `left` set where that expert exists).  Each round takes the largest key left, among
// equal keys the lowest expert id.
//   SORT: each lane first sorts its experts, by falling key and rising id, so a round looks at one value a
//   lane, and the winner's lane moves its list up.
//   Else a round scans every lane's values, and ballots find the winner (smallest j, then lowest lane).
// The sort costs NJ^2 / 2 exchanges of 64-bit keys, a round of the scan about 3 NJ operations, so the
// sort pays from k = NJ / 2 rounds on.  One token, call with scan / sort: E = 512, k = 2 8.3 / 10.2 us,
// k = 4 9.2 / 8.8, k = 16 13.7 / 11.2; E = 1024, k = 8 14.7 / 14.1; E = 64 (one value a lane) 8.5 / 8.7.
// The rounds are a loop, not unrolled: the kernel stays small, so a block's first instruction fetches
// are few.
template <int NJ, bool SORT>
__device__ __forceinline__ void select_topk(const float (&v)[NJ], uint32_t left, int lane, int t,
                                            const TopkArgs& a) {
  int32_t my_id = 0;
  uint32_t my_key = 0;
  if constexpr (SORT) {
    // Key in the high word, the id's complement in the low word; 0 where there is no expert (a NaN's
    // key may be 0, its low word is not).
    uint64_t c[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      c[j] = ((left >> j) & 1u) ? (uint64_t)float_key(v[j]) << 32 | (uint32_t)~(kWave * j + lane) : 0ull;
    // Odd-even transposition sort, falling.
#pragma unroll
    for (int p = 0; p < NJ; ++p)
#pragma unroll
      for (int j = p & 1; j + 1 < NJ; j += 2) {
        const bool sw = c[j + 1] > c[j];
        const uint64_t x = sw ? c[j + 1] : c[j], y = sw ? c[j] : c[j + 1];
        c[j] = x;
        c[j + 1] = y;
      }
#pragma unroll 1
    for (int r = 0; r < a.k; ++r) {
      const uint32_t key = (uint32_t)(c[0] >> 32), low = (uint32_t)c[0];
      const uint32_t m = wave_max_u32(key);
      const uint64_t hold = __ballot(key == m);
      uint32_t win = (uint32_t)__builtin_amdgcn_readlane((int)low, (int)__builtin_ctzll(hold));
      if (m == 0 || (hold & (hold - 1)) != 0) win = wave_max_u32(key == m ? low : 0u);  // ties
      if (lane == r) {
        my_id = (int32_t)~win;
        my_key = m;
      }
      if (low == win && key == m) {
#pragma unroll
        for (int j = 0; j + 1 < NJ; ++j) c[j] = c[j + 1];
        c[NJ - 1] = 0ull;
      }
    }
  } else {
    uint32_t key[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) key[j] = float_key(v[j]);
#pragma unroll 1
    for (int r = 0; r < a.k; ++r) {
      uint32_t m = 0;
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        if ((left >> j) & 1u) m = max(m, key[j]);
      m = wave_max_u32(m);
      int32_t e = -1;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if (e < 0) {
          const uint64_t hold = __ballot(((left >> j) & 1u) && key[j] == m);
          if (hold) e = kWave * j + (int32_t)__builtin_ctzll(hold);
        }
      }
      if ((e & (kWave - 1)) == lane) left &= ~(1u << (e / kWave));
      if (lane == r) {
        my_id = e;
        my_key = m;
      }
    }
  }
  const float top = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, key_float(my_key)), 0));
  const float ex = expf(key_float(my_key) - top);
  float z = 0.0f;
  for (int r = 0; r < a.k; ++r)
    z += __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, ex), r));
  if (lane < a.k) {
    a.ids[(size_t)t * a.k + lane] = my_id;
    a.w[(size_t)t * a.k + lane] = ex / z;
  }
}

// Few splits (many tokens): one wave per token sums its experts' S partials in split order.
// NJ = 64-expert groups held per lane (ceil(E / 64) rounded up to a power of two).
template <int NJ, bool SORT>
__global__ __launch_bounds__(256) void k_router_topk_wave(TopkArgs a) {
  pin(a.part);
  pin(a.bias);
  pin(a.logits);
  pin(a.ids);
  pin(a.w);
  pin(a.T);
  pin(a.E);
  pin(a.k);
  pin(a.S);
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= a.T) return;
  float v[NJ];
  uint32_t left = 0;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    v[j] = 0.0f;
    if (lane + kWave * j < a.E) left |= 1u << j;
  }
  const float* p = a.part + (size_t)t * a.E + lane;
  const size_t split = (size_t)a.T * a.E;
  // Four splits' loads in flight at a time, added in split order (above 512 experts there is one split,
  // rarely two).
  constexpr int B = NJ <= 8 ? 4 : 1;
#pragma unroll 1
  for (int s0 = 0; s0 < a.S; s0 += B) {
    float q[B][NJ];
#pragma unroll
    for (int u = 0; u < B; ++u)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        q[u][j] = (s0 + u < a.S && ((left >> j) & 1u)) ? p[(size_t)(s0 + u) * split + kWave * j] : 0.0f;
#pragma unroll
    for (int u = 0; u < B; ++u)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        if (s0 + u < a.S) v[j] += q[u][j];
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    if ((left >> j) & 1u) {
      const int e = lane + kWave * j;
      if (a.bias) v[j] += a.bias[e];
      if (a.logits) a.logits[(size_t)t * a.E + e] = v[j];
    }
  }
  select_topk<NJ, SORT>(v, left, lane, t, a);
}

// Many splits (few tokens): a block per token.  Each thread sums MB = NJ / 4 experts over the
// S partials in split order, 32 / MB splits' loads in flight at a time (with 64 / MB the whole sum of 28
// splits is one round trip, yet E = 384 and 512 ran 0.6-0.8 us slower); the logits meet in LDS and the
// first wave selects.
template <int NJ, bool SORT>
__global__ __launch_bounds__(256) void k_router_topk_block(TopkArgs a) {
  constexpr int MB = NJ >= 4 ? NJ / 4 : 1;
  constexpr int B = 32 / MB;
  __shared__ float lg[NJ * kWave];
  pin(a.part);
  pin(a.bias);
  pin(a.logits);
  pin(a.ids);
  pin(a.w);
  pin(a.T);
  pin(a.E);
  pin(a.k);
  pin(a.S);
  const int t = blockIdx.x;
  const float* p = a.part + (size_t)t * a.E + threadIdx.x;
  const size_t split = (size_t)a.T * a.E;
  float v[MB];
#pragma unroll
  for (int m = 0; m < MB; ++m) v[m] = 0.0f;
#pragma unroll 1
  for (int s0 = 0; s0 < a.S; s0 += B) {
    float q[B][MB];
#pragma unroll
    for (int u = 0; u < B; ++u)
#pragma unroll
      for (int m = 0; m < MB; ++m)
        q[u][m] = (s0 + u < a.S && (int)threadIdx.x + 256 * m < a.E) ? p[(size_t)(s0 + u) * split + 256 * m] : 0.0f;
#pragma unroll
    for (int u = 0; u < B; ++u)
#pragma unroll
      for (int m = 0; m < MB; ++m)
        if (s0 + u < a.S) v[m] += q[u][m];
  }
#pragma unroll
  for (int m = 0; m < MB; ++m) {
    const int e = threadIdx.x + 256 * m;
    if (e < a.E) {
      if (a.bias) v[m] += a.bias[e];
      if (a.logits) a.logits[(size_t)t * a.E + e] = v[m];
      lg[e] = v[m];
    }
  }
  __syncthreads();
  if (threadIdx.x >= kWave) return;
  const int lane = threadIdx.x;
  float w[NJ];
  uint32_t left = 0;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    w[j] = 0.0f;
    if (lane + kWave * j < a.E) {
      w[j] = lg[lane + kWave * j];
      left |= 1u << j;
    }
  }
  select_topk<NJ, SORT>(w, left, lane, t, a);
}

template <int NJ, bool SORT>
hipError_t launch_topk_as(const TopkArgs& ta, bool per_block, hipStream_t stream) {
  if (per_block)
    hipLaunchKernelGGL((k_router_topk_block<NJ, SORT>), dim3(ta.T), dim3(256), 0, stream, ta);
  else
    hipLaunchKernelGGL((k_router_topk_wave<NJ, SORT>), dim3((ta.T + 3) / 4), dim3(256), 0, stream, ta);
  return hipGetLastError();
}

template <int NJ>
hipError_t launch_topk(const TopkArgs& ta, bool per_block, hipStream_t stream) {
  if constexpr (NJ > 1) {
    if (2 * ta.k >= NJ) return launch_topk_as<NJ, true>(ta, per_block, stream);
  }
  return launch_topk_as<NJ, false>(ta, per_block, stream);
}

struct Plan {
  int wt, S, tiles_t, tiles_e, n_items, per_xcd;
  int ne;  // > 0: the LDS kernel with ne 32-expert blocks
};

// 32-expert blocks the LDS kernel holds for E experts (its instances), 0 if E is too large.
int lds_blocks(int32_t E) {
  const int nb = (E + 31) / 32;
  return nb <= 4 ? 4 : nb <= 8 ? 8 : nb <= 12 ? 12 : nb <= 16 ? 16 : 0;
}

Plan plan(int32_t T, int32_t H, int32_t E) {
  Plan p{};
  p.tiles_e = (E + kExpTile - 1) / kExpTile;
  const int steps = H / kStepK;
  const int big_tiles = (T + 4 * kTok - 1) / (4 * kTok);
  if (big_tiles >= kLdsMinTiles && lds_blocks(E) > 0) {
    // Many tokens: 128-token tiles over all experts, K split to fill the target grid.
    p.ne = lds_blocks(E);
    p.wt = 4;
    p.tiles_e = 1;
    p.tiles_t = big_tiles;
    p.S = std::max(1, std::min((kTargetBlocks + big_tiles - 1) / big_tiles, std::max(1, steps / 4)));
  } else if (big_tiles * p.tiles_e >= kTargetBlocks / 2) {
    p.wt = 4;
    p.S = 1;
    p.tiles_t = big_tiles;
  } else {
    p.wt = 1;
    p.tiles_t = (T + kTok - 1) / kTok;
    const int tiles = p.tiles_t * p.tiles_e;
    p.S = std::max(1, std::min((kTargetBlocks + tiles - 1) / tiles, steps / 4));
  }
  p.n_items = p.S * p.tiles_e * p.tiles_t;
  p.per_xcd = (p.n_items + 7) / 8;
  return p;
}

bool router_shape_ok(int32_t E, int32_t H, int32_t k) {
  return E >= 1 && E <= DAMOE_MAX_E && k >= 1 && k <= DAMOE_MAX_K && k <= E && H > 0;
}

size_t partial_bytes(int32_t T, int32_t H, int32_t E) {
  if (T <= 0) return 0;
  const Plan p = plan(T, H, E);
  return (size_t)p.S * T * E * sizeof(float);
}

}  // namespace

}  // namespace damoe

using namespace damoe;

extern "C" {

size_t damoe_router_workspace_size(int32_t E, int32_t H, int32_t T_max) {
  if (!router_shape_ok(E, H, 1) || H % kStepK || T_max < 0 || T_max > DAMOE_MAX_T) return 0;
  // The split count falls as T grows, so S * T is not monotone: take the largest over T <= T_max.
  // Above the point where a single split fills the target grid S is 1 and S * T = T.
  size_t best = partial_bytes(T_max, H, E);
  // Both split plans have S = 1 once T fills the target grid with 32-token (few-token plan)
  // or 128-token (LDS plan) tiles alone.
  const int32_t t_split = std::min<int32_t>(T_max, (kTargetBlocks + 1) * 4 * kTok);
  for (int32_t T = 1; T <= t_split; ++T) best = std::max(best, partial_bytes(T, H, E));
  return std::max<size_t>(256, (best + 255) / 256 * 256);
}

damoe_status damoe_router(const uint16_t* x, const uint16_t* wg, const float* bias, int32_t T, int32_t H,
                          int32_t E, int32_t k, float* logits, int32_t* topk_ids, float* topk_w, void* ws,
                          size_t ws_bytes, hipStream_t stream) {
  if (!router_shape_ok(E, H, k) || T < 0 || T > DAMOE_MAX_T) return DAMOE_ERR_INVALID_ARG;
  if (H % kStepK) return DAMOE_ERR_UNSUPPORTED;
  // 32-bit buffer offsets address the token and gate rows.
  if ((size_t)T * H * 2 >= ((size_t)1 << 31) || (size_t)E * H * 2 >= ((size_t)1 << 31))
    return DAMOE_ERR_UNSUPPORTED;
  if (T == 0) return DAMOE_OK;
  if (ws_bytes < partial_bytes(T, H, E)) return DAMOE_ERR_WORKSPACE;
  if (!x || !wg || !topk_ids || !topk_w || !ws) return DAMOE_ERR_INVALID_ARG;
  const Plan p = plan(T, H, E);
  if (p.ne > 0) {
    const damoe_status st = device_setup();  // the LDS kernels' limits
    if (st != DAMOE_OK) return st;
  }
  LogitsArgs la{x, wg, static_cast<float*>(ws), T, H, E, p.S, p.tiles_t, p.tiles_e, p.n_items, p.per_xcd};
  const dim3 grid(8 * p.per_xcd);
  if (p.ne > 0) {
    switch (p.ne) {
      case 4: hipLaunchKernelGGL(k_router_logits_lds<4>, grid, dim3(256), RouterCfg<4>::kLds, stream, la); break;
      case 8: hipLaunchKernelGGL(k_router_logits_lds<8>, grid, dim3(256), RouterCfg<8>::kLds, stream, la); break;
      case 12: hipLaunchKernelGGL(k_router_logits_lds<12>, grid, dim3(256), RouterCfg<12>::kLds, stream, la); break;
      default: hipLaunchKernelGGL(k_router_logits_lds<16>, grid, dim3(256), RouterCfg<16>::kLds, stream, la); break;
    }
  } else if (p.wt == 4) {
    hipLaunchKernelGGL((k_router_logits<4, 2, 3>), grid, dim3(512), 0, stream, la);
  } else {
    hipLaunchKernelGGL((k_router_logits<1, 4, 2>), grid, dim3(256), 0, stream, la);
  }
  if (hipGetLastError() != hipSuccess) return DAMOE_ERR_HIP;
  TopkArgs ta{static_cast<const float*>(ws), bias, logits, topk_ids, topk_w, T, E, k, p.S};
  // A block per token for many splits at few tokens; a wave per token otherwise (at thousands
  // of tokens a block each costs more in scheduling than a few partials per lane do).
  const bool per_block = p.S > 8 || (p.S > 2 && T <= 1024);
  const int groups = (E + kWave - 1) / kWave;
  const hipError_t e = groups <= 1   ? launch_topk<1>(ta, per_block, stream)
                       : groups <= 2 ? launch_topk<2>(ta, per_block, stream)
                       : groups <= 4 ? launch_topk<4>(ta, per_block, stream)
                       : groups <= 8 ? launch_topk<8>(ta, per_block, stream)
                                     : launch_topk<16>(ta, per_block, stream);
  return e == hipSuccess ? DAMOE_OK : DAMOE_ERR_HIP;
}

}  // extern "C"

namespace damoe {

// Dynamic LDS above 64 KB needs the per-kernel limit (set once per device).
hipError_t router_set_lds_limits() {
  struct Fn {
    const void* f;
    size_t lds;
  };
  const Fn fns[] = {{reinterpret_cast<const void*>(&k_router_logits_lds<4>), RouterCfg<4>::kLds},
                    {reinterpret_cast<const void*>(&k_router_logits_lds<8>), RouterCfg<8>::kLds},
                    {reinterpret_cast<const void*>(&k_router_logits_lds<12>), RouterCfg<12>::kLds},
                    {reinterpret_cast<const void*>(&k_router_logits_lds<16>), RouterCfg<16>::kLds}};
  for (const Fn& f : fns) {
    const hipError_t e = hipFuncSetAttribute(f.f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)f.lds);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace damoe
