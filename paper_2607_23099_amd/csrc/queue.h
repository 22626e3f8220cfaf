// Per-XCD work queues of the large-tile grouped-GEMM kernels (tiled and big-tile classes).
//
// Workgroup b runs on XCD b % 8 (round-robin placement).  Items (token tile, feature block)
// are grouped in chunks of tg token tiles x fg feature blocks (tg * fg = the workgroups of one
// XCD), so one XCD's L2 is shared by tg token tiles and fg weight blocks instead of every token
// tile being spread over all XCDs.  The chunks form one work queue per XCD (chunk c in queue
// c % 8, in order), taken item by item through an atomic ticket: the items an XCD runs at one
// time are then always neighbours in chunk order, however far its workgroups drift apart (a
// fixed round-robin assignment let them drift whole chunks apart over the rounds, and the
// sharing with them).  A workgroup whose queue is empty takes items from the next XCDs' queues.
//
// The queue words are control words kQueueCtrl .. + kXcds (tickets, then the count of finished
// workgroups).  They are zero between launches: the routing kernel clears them and the last
// workgroup out of each launch returns them to zero.  Nothing waits on another workgroup: a
// take tries at most one ticket per queue once it is empty.
#pragma once

#include "common.h"

namespace damoe {

constexpr int kXcds = 8;

struct ItemMap {
  bool xcd, ends;
  int fg, tg, n_fg, nq, n_chunks;

  // both_ends: odd queues run their chunks from the last to the first.  For tiles sorted by length
  // only: half the XCDs then run long tiles (bound by the matrix cores) while the others run short
  // ones (bound by the weight stream).  In list order it would start the odd queues with the partial
  // last chunk and part the tiles of an expert.
  __device__ ItemMap(int n_tiles, int n_fb, bool both_ends = false)
      : ItemMap(n_tiles, n_fb, both_ends, (int)gridDim.x) {}
  __host__ __device__ ItemMap(int n_tiles, int n_fb, bool both_ends, int grid) : ends(both_ends) {
    const int per_xcd = grid / kXcds;
    xcd = grid % kXcds == 0 && per_xcd > 0;
    fg = n_fb % 4 == 0 ? 4 : n_fb % 2 == 0 ? 2 : 1;
    if (!xcd || fg > per_xcd) fg = 1;
    tg = xcd ? per_xcd / fg : 1;
    n_fg = n_fb / fg;
    nq = xcd ? kXcds : 1;
    n_chunks = (n_tiles + tg - 1) / tg * n_fg;
  }

  // Tickets of queue q: its chunks q, q + nq, ... times tg * fg items each.
  __host__ __device__ int queue_len(int q) const { return q < n_chunks ? ((n_chunks - 1 - q) / nq + 1) * (tg * fg) : 0; }

  // Item of ticket t of queue q; false for the slots past the last tile of a partial chunk.
  __host__ __device__ bool item(int q, int t, int n_tiles, int& tile, int& fb) const {
    int j = t / (tg * fg);
    if (ends && (q & 1)) j = (n_chunks - 1 - q) / nq - j;
    const int chunk = q + j * nq;
    const int local = t % (tg * fg);
    const int tgroup = chunk / n_fg;
    tile = tgroup * tg + local / fg;
    fb = (chunk - tgroup * n_fg) * fg + local % fg;
    return tile < n_tiles;
  }
};

// Whether a launch runs its tiles sorted by length: where a workgroup takes more than one item (before
// that the order changes nothing), up to the longest list whose order fits the LDS beside the rings.
// Longer lists run in list order from the first tile.
constexpr int kMaxSortedTiles = 8192;
__host__ __device__ inline bool sort_tiles(int n_tiles, int n_fb, int grid) {
  return n_tiles <= kMaxSortedTiles && n_tiles * n_fb > grid;
}
// Whether such a launch runs its odd queues from the short end: bf16 weights, from 7 items a workgroup on.
// Before that the long tiles that the odd queues start last stick out at the end, and fp8 weights, half
// the bytes, leave little to gain from short tiles beside long ones.  GEMM1 from both ends against from
// the long end only, DeepSeek-V3 shape, tiles of mixed length: fp8, 3 to 4 items a workgroup
// (T = 150-350, alpha = 0.04-0.06) 335-443 against 294-398 us, from 9 items on within 4% either way; bf16,
// 7 to 14 items 1-6% faster from both ends, below 7 items between 5% slower and 2% faster.
__host__ __device__ inline bool both_ends(int n_tiles, int n_fb, int grid, bool fp8) {
  return !fp8 && sort_tiles(n_tiles, n_fb, grid) && n_tiles * n_fb >= 7 * grid;
}

// Thread 0's side of the queues.  take() returns queue << 28 | ticket, or -1 once every queue
// is empty; the workgroup learns it through an LDS word (the kernels' item loops).  A
// workgroup's first ticket is fixed: ticket blockIdx.x / nq of its own queue, so that the
// first items spread over the workgroups in launch order, one per CU while there are fewer
// items than CUs (taken first-come, two could land on one CU and leave another idle); the
// counters hand out the tickets after those.
struct QueueTaker {
  uint32_t* qctrl;
  int qj = 0;          // queues found empty so far, own queue first
  bool first = true;

  __device__ explicit QueueTaker(int32_t* ctrl) : qctrl(reinterpret_cast<uint32_t*>(ctrl + kQueueCtrl)) {}

  __device__ int take(const ItemMap& m) {
    const int fixed = (int)gridDim.x / m.nq;  // tickets per queue taken as first tickets
    if (first) {
      first = false;
      const int q = (int)blockIdx.x % m.nq, t = (int)blockIdx.x / m.nq;
      if (t < m.queue_len(q)) return q << 28 | t;
    }
    while (qj < m.nq) {
      const int q = ((int)blockIdx.x + qj) % m.nq;
      const int t = fixed + (int)atomicAdd(qctrl + q, 1u);
      if (t < m.queue_len(q)) return q << 28 | t;
      ++qj;
    }
    return -1;
  }

  // After the workgroup's last take: the last workgroup out returns the words to zero (every
  // other workgroup has finished taking tickets, its last ticket returned before its count).
  __device__ void finish() {
    const uint32_t done = atomicAdd(qctrl + kXcds, 1u);
    if (done == gridDim.x - 1) {
      for (int x = 0; x <= kXcds; ++x) __hip_atomic_store(qctrl + x, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
};

}  // namespace damoe
