// Big-tile class of the grouped expert GEMMs (a6, a7) for prefill-sized token counts, where the
// work is bound by the matrix cores rather than by the weight stream.  Fragment-packed weights;
// row-major ones take gemm_big_rm.hip.
//
// One workgroup of 4 waves per CU, one per SIMD.  A work item is (tile of up to 256 tokens of one
// expert, 256 weight rows): for GEMM1 the rows are 128 features of W1 (gate) and the same 128 of W3
// (up), for GEMM2 256 rows of W2.  h passes between the two stage-major ([I / 64][A][64] bf16), so
// that each of GEMM2's token moves reads whole contiguous rows of the tile.
//
// A wave owns 64 weight rows x all tokens of the tile: 2 x NN MFMA blocks of 32 x 32 (32x32x16 bf16,
// up to 256 fp32 accumulators per lane), NN the tile's 32-token blocks with valid rows.  Its weights
// stream from memory into registers, each fragment read by one wave only and, in fp8, decoded once;
// a ring of 2 or 4 K stages of 64 columns keeps 16 to 32 KB per wave in flight.  GEMM1 pairs 16 gate
// and 16 up rows in one 32-row operand, so gate and up of a feature meet in one lane.  The token
// rows, shared by the 4 waves, move into an LDS ring of 4 stages with direct buffer -> LDS loads, as
// 128-byte rows with XOR-swizzled 16-byte chunks; each operand read is one conflict-free 16-byte LDS
// read per lane that feeds two MFMAs (8 KB of LDS reads per 16 MFMAs; a 2 x 4 split over 8 waves with
// both operands in LDS read 12 KB and held two stages).
//
// What bounds it.  Full tiles: the card's power.  At 512 tokens per expert (DeepSeek-V3 shape, bf16,
// random data) the matrix cores are busy 72-74% of the cycles at a clock of 1.4 GHz; with all-zero
// tokens the same code runs at 1.95 GHz and 1480 TF/s instead of 1160.  Every byte moved costs there,
// so items are ordered for L2 reuse (big_order).  Short tiles: the weight stream (5.9-6.3 TB/s).
// Per layer call, before (8 waves, both operands in a two- or three-stage LDS ring) and now:
//   bf16, 512 tokens per expert:  GEMM1 6.94-7.12 -> 6.56-6.71 ms, GEMM2 3.87-4.08 -> 3.42-3.54 ms
//   bf16, 64 tokens per expert:   GEMM1 2.81-2.91 -> 2.41 ms
//   Kimi-K2 shape, T = 8192, alpha = 0.3:   GEMM1 5.6 -> 4.95-5.05 ms, GEMM2 2.84 -> 2.65-2.70 ms
//   DeepSeek-V3 fp8, T = 16384, alpha = 0.3: GEMM1 8.1 -> 7.2-7.4 ms
#include <type_traits>

#include "common.h"
#include "device.h"
#include "queue.h"

namespace damoe {
namespace {

constexpr int kBigBM = 256;    // tokens per tile
constexpr int kBigRows = 256;  // weight rows per item
constexpr uint32_t kMove = 1024;  // bytes of one token move: 64 lanes x 16
constexpr int kBigMaxSk = 128;    // fp8 scale columns per row held in LDS (K <= 16384)
constexpr int kBigThreads = 256;  // 4 waves
constexpr int kBigWaves = kBigThreads / 64;
constexpr int kBigMB = kBigRows / (32 * kBigWaves);  // 32-row weight blocks per wave

// Items of at most this many token blocks load weights with the nontemporal hint: most are an
// expert's only tile, which streams its weights once (a 4 GiB read runs at 7.1-7.3 TB/s with the
// hint, 6.0-6.3 without); an expert with further tiles keeps its weights cached for them.
constexpr int kBigNtMax = 4;
constexpr int kBigBK = 64;          // K columns per stage: a token row of a stage is one 128-byte line
constexpr uint32_t kBigRing = 128 * 1024;                      // LDS ring of token stages
constexpr uint32_t kBigScaleOff = kBigRing;                    // fp8: the item's two rows of block scales
constexpr uint32_t kBigSlotOff = kBigScaleOff + 2 * kBigMaxSk * 4;
constexpr uint32_t kBigOrderOff = kBigSlotOff + 16;            // uint16 tile order
constexpr size_t kBigLds = kBigOrderOff + 2 * kMaxSortedTiles;
static_assert(kBigLds <= 160 * 1024, "LDS of one CU");

// Per count NN of active token blocks of 32 (1 .. 8) of an item: token moves per wave and stage, token
// stages in the LDS ring (of 8, 16 or 32 KB each), and weight stages in the register ring (32 VGPRs
// a stage of bf16 weights, 16 of fp8).  Up to 4 blocks leave registers for 4 bf16 stages: those tiles
// are bound by the weight stream, their time is the bytes in flight over the memory latency.  Deeper
// rings of either kind spill, or need more than the 63 moves that the counter can tell apart.
template <bool FP8, int NN>
struct BigCfg {
  static constexpr int NTOK = NN <= 2 ? 2 : NN <= 4 ? 4 : 8;
  static constexpr uint32_t kTok = NTOK * kBigWaves * kMove;
  static constexpr int NT = 4;
  static constexpr int D = FP8 || NN <= 4 ? 4 : 2;
  static constexpr int NB = NN < 4 ? NN : 4;   // token blocks of one operand set
  static constexpr int NH = NN > 4 ? 2 : 1;    // operand sets per 16-column k-step
};

typedef __attribute__((address_space(3))) uint8_t lds_t;
typedef __attribute__((address_space(3))) float lds_f32;

__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t r, lds_t* dst, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)dst, 16, voff, soff, 0, 0);
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint4 lds_read16(const lds_t* p) {
  return __builtin_bit_cast(uint4, *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(p));
}

// s_waitcnt vmcnt(VM) lgkmcnt(LGKM) (gfx9 encoding; expcnt left alone).
template <int VM, int LGKM>
__device__ __forceinline__ void wait_cnt() {
  static_assert(VM >= 0 && VM < 64 && LGKM >= 0 && LGKM < 16, "counter range");
  __builtin_amdgcn_s_waitcnt((VM & 15) | (7 << 4) | (LGKM << 8) | ((VM >> 4) << 14));
}

// Tile order of a launch: by falling count of 32-token blocks, list order within a count (a stable
// counting sort, one per workgroup).  The items an XCD runs at one time then take equally long, so
// its workgroups stay at the same K stage and share its L2: the feature blocks of a tile its token
// rows, the tiles of an expert its weights.  In list order short and long tiles alternate, the
// workgroups drift apart and most reads miss.
__device__ __forceinline__ int big_class(int2 en) { return 8 - min(8, max(1, ((en.y >> 16) + 31) / 32)); }

__device__ __forceinline__ void big_order(const int2* __restrict__ ent, int n, lds_t* lds) {
  typedef __attribute__((address_space(3))) uint16_t lds_u16;
  typedef __attribute__((address_space(3))) uint32_t lds_u32;
  lds_u16* const order = reinterpret_cast<lds_u16*>(lds + kBigOrderOff);
  lds_u32* const cnt = reinterpret_cast<lds_u32*>(lds);  // [8 classes][threads], in the idle ring
  const int tid = threadIdx.x, per = (n + kBigThreads - 1) / kBigThreads;
  const int i0 = min(n, tid * per), i1 = min(n, i0 + per);
#pragma unroll
  for (int c = 0; c < 8; ++c) cnt[c * kBigThreads + tid] = 0;
  for (int i = i0; i < i1; ++i) ++cnt[big_class(ent[i]) * kBigThreads + tid];
  __syncthreads();
  // Exclusive prefix over (class, thread): 8 counts per thread, then across the threads.
  lds_u32* const part = cnt + 8 * kBigThreads;
  uint32_t v[8], sum = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    v[j] = cnt[8 * tid + j];
    sum += v[j];
  }
  part[tid] = sum;
  __syncthreads();
  uint32_t base = 0;
  for (int t = 0; t < tid; ++t) base += part[t];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    cnt[8 * tid + j] = base;
    base += v[j];
  }
  __syncthreads();
  for (int i = i0; i < i1; ++i) order[cnt[big_class(ent[i]) * kBigThreads + tid]++] = (uint16_t)i;
  __syncthreads();
}

// The kernel's arguments, read again from the argument segment by every item: held in registers over
// an item's K loop they spill, and the spilled registers' reloads land in the loop.
typedef const __attribute__((address_space(4))) GemmArgs* args_ptr;
__device__ __forceinline__ args_ptr item_args() {
  args_ptr p = (args_ptr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return p;
}

// mx: GEMM1 of the fp8-MFMA variant (fp8 weights only): h is rounded to bf16 as for the other
// variants, then quantised to e4m3 with one E8M0 scale per 32 features of a row, into out
// (codes [N / 64][A][64]) and o8s (scale words [N / 64][A][4]), the operand of its fp8-MFMA
// GEMM2, stored stage-major so that each of GEMM2's moves reads contiguous bytes.
// rowmajor_h: bf16 h as [A][N], for the deep-ring variant's GEMM2 (fp8 weights).
template <bool GLU, bool FP8>
__device__ __forceinline__ void big_body(const GemmArgs& ka, lds_t* lds, bool mx, bool rowmajor_h) {
  constexpr int FEAT = GLU ? kBigRows / 2 : kBigRows;  // output features per item
  constexpr int EB = FP8 ? 1 : 2;
  constexpr int BK = kBigBK;
  using WRaw = typename std::conditional<FP8, uint2, uint4>::type;
  typedef const __attribute__((address_space(1))) uint8_t* gptr;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t* __restrict__ list = ka.tiles.list[4];
  const int n_tiles = tile_count(list, ka);
  const int2* __restrict__ ent = reinterpret_cast<const int2*>(list + 2);
  const int n_fb = (ka.N + FEAT - 1) / FEAT;
  const int l32 = lane & 31, lh = lane >> 5;
  const bool sorted = GLU && sort_tiles(n_tiles, n_fb, (int)gridDim.x);
  const ItemMap map(n_tiles, n_fb, GLU && both_ends(n_tiles, n_fb, (int)gridDim.x, FP8));
  if (sorted) big_order(ent, n_tiles, lds);

  // Items come from the per-XCD work queues.  Thread 0 takes the tickets, one item ahead, and
  // hands each to the workgroup through an LDS word.
  QueueTaker taker(ka.ctrl);
  typedef volatile __attribute__((address_space(3))) int32_t lds_i32;
  lds_i32* const slot = reinterpret_cast<lds_i32*>(lds + kBigSlotOff);
  int next = 0;
  if (tid == 0) slot[0] = taker.take(map);
  __syncthreads();

  for (;;) {
    const int cur = __builtin_amdgcn_readfirstlane(slot[0]);
    __syncthreads();  // every wave has read the ticket before thread 0 may replace it
    if (cur < 0) break;
    if (tid == 0) next = taker.take(map);  // the next ticket, while this item runs
    int tile = 0, fb = 0;
    bool ok = map.item(cur >> 28, cur & 0x0FFFFFFF, n_tiles, tile, fb);
    if (ok && sorted) tile = reinterpret_cast<const __attribute__((address_space(3))) uint16_t*>(lds + kBigOrderOff)[tile];
    const int2 en = ok ? ent[tile] : make_int2(0, 0);
    const int p0 = __builtin_amdgcn_readfirstlane(en.x);
    const int e = __builtin_amdgcn_readfirstlane(en.y & 0xFFFF), rows = __builtin_amdgcn_readfirstlane(en.y >> 16);
    if (ok && (p0 < 0 || rows <= 0 || rows > kBigBM || p0 + rows > ka.A || e >= ka.E)) {
      if (tid == 0) atomicOr(&ka.ctrl[0], DAMOE_DEVERR_TILES);
      ok = false;
    }

    // One item whose valid rows fill NN token blocks of 32.
    auto run_item = [&](auto nn_c) __attribute__((always_inline)) {
    constexpr int NN = decltype(nn_c)::value;
    using Cfg = BigCfg<FP8, NN>;
    constexpr int NTOK = Cfg::NTOK, NT = Cfg::NT, D = Cfg::D, NB = Cfg::NB, NH = Cfg::NH;
    constexpr int NS = 4 * NH;  // operand sets per stage
    const args_ptr a = item_args();
    const int K = a->K, N = a->N, A = a->A;
    const int nst = K / BK;

    // Token moves of this wave (padding rows read as zero).  GEMM1 gathers rows perm[p] / k of
    // x; GEMM2 reads h stage-major ([K / BK][A][BK], as this kernel's GEMM1 writes it), whose
    // rows of one stage are contiguous, through a resource per stage over the tile's rows.
    // Move j carries rows 8 (NTOK wave + j) .. + 7 of the tile, 128 bytes each: lane l moves
    // row r = 8 (NTOK wave + j) + l / 8, its 16-byte chunk c = (l % 8) ^ ((r / 2) % 8), which
    // lands at slot l % 8 of the row.  The swizzle puts the 16 rows that one read phase of an
    // MFMA operand touches on 16 distinct bank groups.
    const uint32_t xbytes = (uint32_t)((size_t)(A / a->k) * K * 2);
    uint32_t xo[NTOK];
#pragma unroll
    for (int j = 0; j < NTOK; ++j) {
      const int r = 8 * (NTOK * wave + j) + (lane >> 3);
      const uint32_t cb = (uint32_t)(((lane & 7) ^ ((r >> 1) & 7)) * 16);
      if (r < rows) {
        xo[j] = GLU ? (uint32_t)(a->perm[p0 + r] / a->k) * (uint32_t)K * 2u + cb : (uint32_t)r * (BK * 2u) + cb;
      } else {
        xo[j] = kOobOffset;
      }
    }
    // Moves of stages past the last go through an empty resource: they read no memory, and the
    // counts of moves in flight stay the same.
    auto tok_src = [&](int st, uint32_t& soff) __attribute__((always_inline)) {
      const bool in = st < nst;
      const uint32_t s0 = in ? st : 0;
      soff = GLU ? s0 * (BK * 2u) : 0u;
      return GLU ? make_rsrc(a->x, in ? xbytes : 0u)
                 : make_rsrc(a->x + ((size_t)s0 * A + p0) * BK, in ? (uint32_t)rows * (BK * 2u) : 0u);
    };
    auto dma_tok = [&](int st, lds_t* sb) __attribute__((always_inline)) {
      uint32_t soff;
      const __amdgpu_buffer_rsrc_t rx = tok_src(st, soff);
#pragma unroll
      for (int j = 0; j < NTOK; ++j) dma16(rx, sb + (NTOK * wave + j) * kMove, xo[j], soff);
    };

    // Weight operand of this wave: 32 rows, lane l row l % 32, 8 columns 8 (l / 32) .. of a
    // 16-column k-step.  GEMM1, operand m: rows 0..15 are W1 features fb * 128 + 32 wave + 16 m ..,
    // rows 16..31 the same features of W3, so gate and up of a feature meet in one lane.  GEMM2:
    // W2 rows fb * 256 + 64 wave + 32 m ..; a last item of 128 rows repeats row blocks (never stored).
    const size_t slab = (size_t)N * K * EB;
    gptr wp[kBigMB], wps[kBigMB];
#pragma unroll
    for (int m = 0; m < kBigMB; ++m) {
      const uint32_t rb = GLU ? (uint32_t)(fb * 8 + wave * kBigMB + m)
                              : (uint32_t)min(fb * 16 + (wave * kBigMB + m) * 2 + (l32 >> 4), N / 16 - 1);
      const size_t woff = (size_t)e * slab + (size_t)rb * (K / 32) * (512 * EB) + ((l32 & 15) + 16 * lh) * 8 * EB;
      wp[m] = (gptr)((GLU && (l32 >> 4)) ? a->wb : a->wa) + woff;
    }
    constexpr uint32_t kWStage = 1024 * EB;  // bytes from one stage to the next
    WRaw wf[D][4][kBigMB];
    auto wstage = [&](int st) __attribute__((always_inline)) {
#pragma unroll
      for (int m = 0; m < kBigMB; ++m) wps[m] = wp[m] + (size_t)min(st, nst - 1) * kWStage;
    };
    auto wload = [&](int d, int ks) __attribute__((always_inline)) {
      typedef uint32_t vec __attribute__((ext_vector_type(sizeof(WRaw) / 4)));
      const uint32_t off = ((ks >> 1) * 512u + (ks & 1) * 256u) * EB;
#pragma unroll
      for (int m = 0; m < kBigMB; ++m) {
        const auto* q = reinterpret_cast<const __attribute__((address_space(1))) vec*>(wps[m] + off);
        if constexpr (NN <= kBigNtMax) wf[d][ks][m] = __builtin_bit_cast(WRaw, __builtin_nontemporal_load(q));
        else wf[d][ks][m] = __builtin_bit_cast(WRaw, *q);
      }
    };

    // fp8 block scales of the item's rows (a 128-row block per matrix of GEMM1, per half of
    // GEMM2), one per 128 columns, staged in LDS.
    lds_f32* const sc_lds = reinterpret_cast<lds_f32*>(lds + kBigScaleOff);
    if constexpr (FP8) {
      const int sk = K / 128;
      for (int i = tid; i < 2 * kBigMaxSk; i += kBigThreads) {
        const int m = i / kBigMaxSk, kb = i % kBigMaxSk;
        const int srow = GLU ? fb : min(fb * 2 + m, N / 128 - 1);
        if (kb < sk) sc_lds[i] = ((GLU && m) ? a->sb : a->sa)[((size_t)e * (N / 128) + srow) * sk + kb];
      }
    }
    const lds_f32* const sc_lane = sc_lds + (GLU ? (l32 >> 4) : (wave >> 1)) * kBigMaxSk;

    floatx16 acc[kBigMB][NN];
#pragma unroll
    for (int m = 0; m < kBigMB; ++m)
#pragma unroll
      for (int n = 0; n < NN; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[m][n][r] = 0.f;

    // Token operands: lane l takes row 32 n + l % 32 of token block n and the 8-column chunk
    // 2 ks + l / 32 of the stage, at its swizzled slot.  Set s of a stage is k-step s / NH, token
    // blocks 4 (s % NH) .. of it.
    uint4 tf[2][NB];
    auto read1 = [&](int s, const lds_t* tcur, int i, uint4 (&o)[NB]) __attribute__((always_inline)) {
      const int ks = s / NH, n0 = 4 * (s % NH);
      const lds_t* row = tcur + l32 * 128 + (((2 * ks + lh) ^ ((l32 >> 1) & 7)) << 4);
      if (i < NB && n0 + i < NN) o[i] = lds_read16(row + (n0 + i) * 4096);
    };
    uint4 wv[kBigMB];
    float sc = 0.f;
    auto conv = [&](int s, int d) __attribute__((always_inline)) {
      if (s % NH == 0) {
#pragma unroll
        for (int m = 0; m < kBigMB; ++m) {
          if constexpr (FP8) wv[m] = fp8x8_to_bf16x8(wf[d][s / NH][m], sc);
          else wv[m] = wf[d][s / NH][m];
        }
      }
    };
    constexpr int NMF = NB * kBigMB;  // MFMAs of a set (fewer in a last half set)
    auto mma1 = [&](int s, int i, const uint4 (&o)[NB]) __attribute__((always_inline)) {
      const int n = 4 * (s % NH) + i / kBigMB, m = i % kBigMB;
      if (n < NN) acc[m][n] = mfma32x32x16(wv[m], o[i / kBigMB], acc[m][n]);
    };

    // Software pipeline.  Iteration t (between barriers t - 1 and t): the DMA of the tokens of
    // stage t + NT - 1 into the buffer stage t - 1 left; operand reads of stage t, each set's
    // issued ahead of the MFMAs of the one before (the last set's MFMAs run in the next
    // iteration); each k-step's weight registers are loaded again, for stage t + D, after its last
    // MFMAs.  Then a wait for this wave's token moves of stage t + 1 and its LDS reads, and the
    // barrier that makes stage t + 1 visible to every wave and frees stage t's buffer.  Moves
    // complete in issue order: after those of stage t + 1 the wave issued the moves of NT - 2
    // stages and the loads of NT - 1 iterations (at the start of the item, those of D stages).
    // The count is right only while the compiler keeps every load in it: it removes loads that
    // nothing reads.  In the loop each feeds a later trip; the two iterations of a tail (`last`)
    // have none, their weights being in the ring, and wait by the token moves alone, which always
    // write LDS.  The barrier is a bare s_barrier: the counter waits before it are the ordering (a
    // fence would drain the moves still ahead).  `tdst` and `tcur` are distinct buffers, so the
    // compiler does not hold the reads behind the moves.
    constexpr int NW = 4 * kBigMB;  // weight loads of a stage
    constexpr int kAhead = (NT - 2) * NTOK + (NW * (NT - 1) < NW * (D + 1) - kBigMB ? NW * (NT - 1) : NW * (D + 1) - kBigMB);
    auto iter = [&](lds_t* __restrict__ tdst, const lds_t* __restrict__ tcur, int t, auto d_c, auto last_c)
        __attribute__((always_inline)) {
      constexpr int d = decltype(d_c)::value, dp = (d + D - 1) % D;
      constexpr bool last = decltype(last_c)::value;
      uint32_t soff;
      const __amdgpu_buffer_rsrc_t rx = tok_src(t + NT - 1, soff);
      float sc_next = 0.f;
      if constexpr (FP8) sc_next = sc_lane[(t * BK) >> 7];
      // Behind each MFMA of the set before: one operand read of this set, or moves of the stage ahead.
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int sp = s == 0 ? NS - 1 : s - 1;
        constexpr int MV = (NTOK + NMF - 1) / NMF;
        conv(sp, s == 0 ? dp : d);  // (of nothing in iteration 0)
#pragma unroll
        for (int i = 0; i < NMF; ++i) {
          if (s > 0 || t > 0) mma1(sp, i, tf[sp & 1]);
          read1(s, tcur, i, tf[s & 1]);
          if (s == 0) {
#pragma unroll
            for (int j = i * MV; j < (i + 1) * MV; ++j)
              if (j < NTOK) dma16(rx, tdst + (NTOK * wave + j) * kMove, xo[j], soff);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        if (s == 0) {
          if constexpr (!last) {
            wload(dp, 3);
            wstage(t + D);
          }
          sc = sc_next;
        } else if (s % NH == 0) {
          if constexpr (!last) wload(d, s / NH - 1);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      wait_cnt<last ? (NT - 2) * NTOK : kAhead, 0>();
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    };
    auto tbuf = [&](int i) __attribute__((always_inline)) { return lds + (uint32_t)(i % NT) * Cfg::kTok; };

#pragma unroll
    for (int i = 0; i < NT - 1; ++i) dma_tok(i, tbuf(i));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 0; d < D; ++d) {
      wstage(d);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        if (d < D - 1 || ks < 3) wload(d, ks);  // the last one in iteration 0
    }
    __builtin_amdgcn_sched_barrier(0);
    wait_cnt<(NT - 2) * NTOK + NW * D - kBigMB, 15>();  // this wave's stage-0 moves have landed
    __syncthreads();                              // ... and every wave's, and the scales
    int t = 0;
    auto trip = [&](auto cnt_c, auto last_c) __attribute__((always_inline)) {
      constexpr int CNT = decltype(cnt_c)::value;
      static_assert(CNT == 2 || CNT == 4, "iterations of a trip");
      iter(tbuf(t + NT - 1), tbuf(t), t, std::integral_constant<int, 0>{}, last_c);
      iter(tbuf(t + NT), tbuf(t + 1), t + 1, std::integral_constant<int, 1>{}, last_c);
      if constexpr (CNT >= 4) {
        iter(tbuf(t + NT + 1), tbuf(t + 2), t + 2, std::integral_constant<int, 2>{}, last_c);
        iter(tbuf(t + NT + 2), tbuf(t + 3), t + 3, std::integral_constant<int, 3>{}, last_c);
      }
      t += CNT;
    };
    // K is a multiple of 128 (512 with fp8 weights), so the stages are a multiple of 2 (8).
    while (t + D <= nst) trip(std::integral_constant<int, D>{}, std::false_type{});
    if (D == 4 && !FP8 && t < nst) {
      trip(std::integral_constant<int, 2>{}, std::true_type{});
      conv(NS - 1, 1);
    } else {
      conv(NS - 1, D - 1);
    }
#pragma unroll
    for (int i = 0; i < NMF; ++i) mma1(NS - 1, i, tf[1]);
    // Moves and loads past the last stage may still be in flight: drain before the next item's.
    wait_cnt<0, 0>();
    __syncthreads();

    // Epilogue from the accumulators: in block n lane l holds token 32 n + l % 32 and, in
    // registers 4 q .. 4 q + 3, weight rows 8 q + 4 (l / 32) .. + 3 of the wave's 32.  A swap of
    // the lane halves between the packed words of q and q + 1 leaves 8 consecutive features in
    // each lane: 8 (l / 32) .. + 7 of the 16.
    const args_ptr ae = item_args();
    const int Ne = ae->N, Ae = ae->A;
    void* const out = ae->out;
    // h: bytes from one position to the next, and from one 64-feature stage to the next.
    const size_t h_row = rowmajor_h ? (size_t)Ne * 2 : BK * 2, h_stage = rowmajor_h ? BK * 2 : (size_t)Ae * BK * 2;
    auto swap = [&](uint32_t& x, uint32_t& y) __attribute__((always_inline)) {
      const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
      x = r[0];
      y = r[1];
    };
    if constexpr (GLU) {
      float hv[kBigMB][8];
      auto swiglu = [&](int n) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < kBigMB; ++m)
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const float g = acc[m][n][j], u = acc[m][n][8 + j];
            hv[m][j] = g / (1.0f + __expf(-g)) * u;
          }
      };
      const int f0 = fb * FEAT + 32 * wave;  // the wave's 32 features
#pragma unroll
      for (int n = 0; n < NN; ++n) {
        const int i = 32 * n + l32;
        swiglu(n);
        if constexpr (FP8) {
          if (mx) {
            // The wave's 32 features of token i are an MX block: lane l and lane l ^ 32 hold them.
            float amax = 0.f;
#pragma unroll
            for (int m = 0; m < kBigMB; ++m)
#pragma unroll
              for (int j = 0; j < 8; ++j) {
                hv[m][j] = (float)(__bf16)hv[m][j];
                amax = fmaxf(amax, fabsf(hv[m][j]));
              }
            amax = fmaxf(amax, __shfl_xor(amax, 32));
            const uint32_t scb = mx_scale_byte(amax);
            const float inv = mx_inv_scale(scb);
            // Stage-major for GEMM2's 64-column stages: codes [N / 64][A][64], scale words
            // [N / 64][A][4] (byte (f0 / 32) % 2; bytes 2 and 3 unused).
            const size_t srow = (size_t)(f0 / 64) * Ae + (p0 + i);
#pragma unroll
            for (int m = 0; m < kBigMB; ++m) {
              uint32_t c0 = e4m3x4(hv[m][0] * inv, hv[m][1] * inv, hv[m][2] * inv, hv[m][3] * inv);
              uint32_t c1 = e4m3x4(hv[m][4] * inv, hv[m][5] * inv, hv[m][6] * inv, hv[m][7] * inv);
              swap(c0, c1);
              if (i < rows)
                *reinterpret_cast<uint2*>(reinterpret_cast<uint8_t*>(out) + srow * 64 + f0 % 64 + 16 * m + 8 * lh) =
                    make_uint2(c0, c1);
            }
            if (i < rows && lh == 0) ae->o8s[srow * 4 + (f0 / 32) % 2] = (uint8_t)scb;
            continue;
          }
        }
        // h stage-major for this kernel's GEMM2 (its stages of BK columns): [N / BK][A][BK].
#pragma unroll
        for (int m = 0; m < kBigMB; ++m) {
          uint4 pk = make_uint4(pack_bf16x2(hv[m][0], hv[m][1]), pack_bf16x2(hv[m][2], hv[m][3]),
                                pack_bf16x2(hv[m][4], hv[m][5]), pack_bf16x2(hv[m][6], hv[m][7]));
          swap(pk.x, pk.z);
          swap(pk.y, pk.w);
          if (i < rows)
            *reinterpret_cast<uint4*>(reinterpret_cast<uint8_t*>(out) + (size_t)(f0 / BK) * h_stage +
                                      (size_t)(p0 + i) * h_row + (f0 % BK + 16 * m + 8 * lh) * 2) = pk;
        }
      }
    } else {
#pragma unroll
      for (int n = 0; n < NN; ++n) {
        const int i = 32 * n + l32;
        uint16_t* orow = reinterpret_cast<uint16_t*>(out) + (size_t)(p0 + i) * Ne;
#pragma unroll
        for (int m = 0; m < kBigMB; ++m)
#pragma unroll
          for (int q = 0; q < 4; q += 2) {
            const floatx16& c = acc[m][n];
            uint4 pk = make_uint4(pack_bf16x2(c[4 * q], c[4 * q + 1]), pack_bf16x2(c[4 * q + 2], c[4 * q + 3]),
                                  pack_bf16x2(c[4 * q + 4], c[4 * q + 5]), pack_bf16x2(c[4 * q + 6], c[4 * q + 7]));
            swap(pk.x, pk.z);
            swap(pk.y, pk.w);
            const int f = fb * FEAT + (wave * kBigMB + m) * 32 + 8 * q + 8 * lh;
            if (i < rows && f < Ne) *reinterpret_cast<uint4*>(orow + f) = pk;
          }
      }
    }
    };  // run_item
    if (ok) {
      switch ((rows + 31) / 32) {
        case 1: run_item(std::integral_constant<int, 1>{}); break;
        case 2: run_item(std::integral_constant<int, 2>{}); break;
        case 3: run_item(std::integral_constant<int, 3>{}); break;
        case 4: run_item(std::integral_constant<int, 4>{}); break;
        case 5: run_item(std::integral_constant<int, 5>{}); break;
        case 6: run_item(std::integral_constant<int, 6>{}); break;
        case 7: run_item(std::integral_constant<int, 7>{}); break;
        default: run_item(std::integral_constant<int, 8>{}); break;
      }
    }
    // Every wave has read this item's ticket and its K loop has drained (or it had none).
    if (tid == 0) slot[0] = next;
    __syncthreads();
  }
  if (tid == 0) taker.finish();
}

template <bool GLU, bool FP8>
__global__ void __launch_bounds__(kBigThreads, 1) k_gemm_big(GemmArgs a) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t big_smem[];
  flag_stale_tiles(a);
  const int v = a.force_variant >= 0 ? a.force_variant : *a.variant_id;
  if (GLU && blockIdx.x == 0 && threadIdx.x == 0) a.ctrl[4] = v;
  if (!variant_admitted(v, a.force_variant, a.candidates)) {
    if (blockIdx.x == 0 && threadIdx.x == 0) atomicOr(&a.ctrl[0], DAMOE_DEVERR_VARIANT);
    return;
  }
  // This kernel runs the big-tile variant and, with fp8 weights, GEMM1 of both fp8-MFMA variants and
  // of the deep-ring variant.  The deep-ring kernel's own fp8 GEMM1 decoded each weight operand for
  // tiles of 64 tokens and padded them to 16: DeepSeek-V3 shape, T = 1024, alpha = 1, 1656 us against
  // 1408 us here; at 64 tokens an expert, its best case, 1483 against 1468 us.
  const bool mx = GLU && FP8 && (v == kBig8Variant || v == kDeep8Variant);
  const bool rowmajor_h = GLU && FP8 && v == kDeepVariant;
  if (v != kBigVariant && !mx && !rowmajor_h) return;  // the device chose another kernel class
  big_body<GLU, FP8>(a, (lds_t*)big_smem, mx, rowmajor_h);
}

template <bool GLU>
hipError_t launch_big_stage(const GemmArgs& a, int grid, hipStream_t stream) {
  if (a.fp8) hipLaunchKernelGGL((k_gemm_big<GLU, true>), dim3(grid), dim3(kBigThreads), kBigLds, stream, a);
  else hipLaunchKernelGGL((k_gemm_big<GLU, false>), dim3(grid), dim3(kBigThreads), kBigLds, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t big_set_lds_limits() {
  const void* fns[] = {
      reinterpret_cast<const void*>(&k_gemm_big<true, false>), reinterpret_cast<const void*>(&k_gemm_big<false, false>),
      reinterpret_cast<const void*>(&k_gemm_big<true, true>), reinterpret_cast<const void*>(&k_gemm_big<false, true>)};
  for (const void* f : fns) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kBigLds);
    if (e != hipSuccess) return e;
  }
  return big_rm_set_lds_limits();
}

// Row-major weights take the kernel that gathers them into LDS (k_gemm_big_rm, where both are measured).
hipError_t launch_big_gemm1(const GemmArgs& a, int grid, hipStream_t stream) {
  return a.packed ? launch_big_stage<true>(a, grid, stream) : launch_big_rm_gemm1(a, grid, stream);
}

hipError_t launch_big_gemm2(const GemmArgs& a, int grid, hipStream_t stream) {
  return a.packed ? launch_big_stage<false>(a, grid, stream) : launch_big_rm_gemm2(a, grid, stream);
}

}  // namespace damoe
