// Work queue of a persistent launch: the grid is one workgroup per CU (times the kernel's
// occupancy) and every workgroup takes (head, tile) items until none are left, instead of one
// workgroup per item.  Two things are gained over leaving the distribution to the hardware
// dispatcher.  (1) With one resident workgroup per CU, the dispatcher can only start the next
// workgroup after the previous one has gone; measured on the forward kernel that gap (dispatch
// plus prologue) is 14 us per workgroup, 3 % of the kernel.  (2) The dispatcher deals workgroups
// to the 8 XCDs round-robin, an equal share each, but under load the XCDs do not run at one
// clock (6 % apart in the same kernel), so the slowest XCD finishes late while the others idle.
// Here every XCD has its own list (the items of "its" heads, in the order decode_tile defines, so
// that the workgroups of an XCD still stream the same head's K/V through its L2 together), and a
// workgroup whose list is empty takes from whichever of the others still have entries (next_work).
//
// The counters of a launch (kQueueBytes, `AttnParams::q_counters`) are memory that belongs to
// that launch alone: the backward kernels take them from the caller's workspace, the forward from
// a pool of slots whose use the host tracks with events (attn_fwd_wide.hip).  They have to be zeros when the main
// kernel starts: the backward's are cleared by the call's first kernel (or, when a call runs single kernels, by a
// one-wave kernel in front of each), the forward's slots start out as zeros and are left so by every launch
// (queue_leave).
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>

#include "attn_common.hpp"
#include "launch.hpp"

namespace ie {

constexpr int kQueueBytes = 64;   // 8 list counters, one counter of workgroups that have left (queue_leave), padding

static __global__ void tile_queue_reset_kernel(unsigned int* counters) {
  if (threadIdx.x < kQueueBytes / 4) counters[threadIdx.x] = 0u;
}

// The XCD this wave runs on (0..7).
__device__ __forceinline__ uint32_t xcc_id() {
  uint32_t x;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(x));
  return x & 7u;
}

// A workgroup's queue state, in LDS.  (Held in registers through an item's main loop, or read from the kernel's arguments,
// which the compiler does ahead of the item loop, it would cost the kernels scalar registers that they do not have.)
struct QueueState {
  unsigned int* counters;
  uint32_t per;            // entries of a list
  uint32_t dealt;          // AttnParams::q_dealt
  uint32_t index;          // the workgroup's
  int lists;               // eight lists, or one
  int list;                // the list this workgroup draws from; kListNone before its first item
  int work;
};
constexpr int kListNone = -1;
constexpr unsigned int kNotClaimed = ~0u;

__device__ __forceinline__ void queue_init(const AttnParams& p, QueueState* s) {
  if (threadIdx.x == 0) {
    s->counters = p.q_counters;
    s->per = (uint32_t)(p.q_per_xcd > 0 ? p.q_per_xcd : p.q_total);
    s->dealt = p.q_dealt;
    s->index = blockIdx.x;
    s->lists = p.q_per_xcd > 0;
    s->list = kListNone;
  }
}

// (The counters' address comes out of LDS: said to be global memory, or the compiler waits for every LDS access with it; and
// opaque, or it takes the add for one that many lanes make, and waits for the first lane's result on the spot.)
typedef __attribute__((address_space(1))) unsigned int GlobalCounter;
__device__ __forceinline__ unsigned int queue_add(unsigned int* c) {
  asm volatile("" : "+v"(c));
  return __hip_atomic_fetch_add((GlobalCounter*)c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Claims the workgroup's next entry ahead of next_work(), from the list it draws from; called in front of an item's
// epilogue, whose stores hide the atomic's way to memory and back (0.8 us per item).  The result counts in thread 0 and
// goes to next_work() as `claimed`.  (Claimed any earlier, an entry would wait for its workgroup while others are idle.)
__device__ __forceinline__ unsigned int queue_claim(QueueState* s) {
  unsigned int c = 0;
  if (threadIdx.x == 0) c = queue_add(s->counters + s->list);
  return c;
}

// The next item of this launch for the calling workgroup, or -1 when all lists are empty.  All threads of the workgroup
// call it; on return everyone has left the previous item (its LDS is free) and sees the same result.  `claimed`: what
// queue_claim() returned for this call, or kNotClaimed.
// With q_dealt a workgroup's first item goes by its index, entry (index / 8) of list (index % 8), which is the XCD it runs
// on: the first round takes no atomic, and where several workgroups share a CU (indices a grid's 256 apart) one of them
// has heavy items and another light ones.
// A list that is found empty stays empty, and which of the others have entries left is read with one load of all
// eight counters, so that a workgroup that has run out of work leaves after one round trip to memory.  (Trying the lists
// one after the other, the workgroups of a launch spent up to 80 us on eight atomics each to one cache line: the pass of
// 640 short items in the backward's two queues, D = 64, 111-125 us against 28 us without queues.)
__device__ __forceinline__ int next_work(QueueState* s, unsigned int claimed) {
  if (threadIdx.x < 64) {   // one wave
    const bool lists = uniform((uint32_t)s->lists) != 0;
    const uint32_t per = uniform(s->per), all_dealt = uniform(s->dealt);
    // entries of list `x` that are dealt by index: its counter counts from there
    auto dealt = [&](int x) { return lists ? (all_dealt + 7u - (uint32_t)x) >> 3 : all_dealt; };
    int x = (int)uniform((uint32_t)s->list);
    const bool start = x == kListNone;
    uint32_t slot;
    if (start && all_dealt > 0) {
      const uint32_t index = uniform(s->index);
      x = lists ? (int)(index & 7) : 0;
      slot = lists ? index >> 3 : index;
    } else {
      if (start) x = lists ? (int)xcc_id() : 0;
      uint32_t c = uniform(claimed);
      if (c == kNotClaimed) {
        if (threadIdx.x == 0) c = queue_add(s->counters + x);
        c = uniform(c);
      }
      slot = c + dealt(x);
    }
    if (slot >= per && lists) {
      const int y = (x + (int)threadIdx.x) & 7;
      uint32_t c = per;
      if (threadIdx.x < 8) c = __hip_atomic_load((const GlobalCounter*)(s->counters + y), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      uint64_t open = __builtin_amdgcn_ballot_w64(threadIdx.x < 8 && c + dealt(y) < per);
      const int from = x;
      while (open != 0) {   // (at most eight trips)
        x = (from + __builtin_ctzll(open)) & 7;
        uint32_t t = 0;
        if (threadIdx.x == 0) t = queue_add(s->counters + x);
        slot = uniform(t) + dealt(x);
        if (slot < per) break;
        open &= open - 1;
      }
    }
    if (threadIdx.x == 0) {
      s->work = slot < per ? (int)(lists ? slot * 8u + (uint32_t)x : slot) : -1;
      s->list = x;
    }
  }
  __syncthreads();   // (the previous read of s->work lies in front of a barrier of the previous item)
  return (int)uniform((uint32_t)s->work);
}

// For launches whose counters are NOT cleared in front of them (the forward's slots, which start out as zeros): every
// workgroup calls this once, after its last next_work(); the last one to do so, which knows that nobody will touch the
// counters again, clears them for the slot's next launch.
__device__ __forceinline__ void queue_leave(QueueState* s_work) {
  if (threadIdx.x == 0) {
    unsigned int* c = s_work->counters;
    if (atomicAdd(c + 8, 1u) == gridDim.x - 1) {
#pragma unroll
      for (int i = 0; i < 9; ++i) __hip_atomic_store(c + i, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// Per kernel and device: the dynamic LDS limit is raised once, and the number of workgroups of `kernel`
// that fit on one CU together (registers, LDS; at least 1) is asked once.
struct KernelSetup { std::atomic<int> per_cu[kMaxDevices]; };
template <typename K>
static inline int kernel_setup(KernelSetup& ks, K kernel, int smem_bytes, int* per_cu, int threads = kThreads) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e);
  int n = dev < kMaxDevices ? ks.per_cu[dev].load(std::memory_order_acquire) : 0;
  if (n == 0) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, smem_bytes);
    if (e != hipSuccess) return hip_fail(e);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void*>(kernel), threads, (size_t)smem_bytes) != hipSuccess || n < 1) n = 1;
    if (dev < kMaxDevices) ks.per_cu[dev].store(n, std::memory_order_release);
  }
  *per_cu = n;
  return 0;
}

// Host side: fills the queue fields of `p` for `total` items (= tiles per head x B x heads) with the
// launch's own `counters` (device memory, kQueueBytes) and clears them on `st` (unless they are clear already).  Returns the grid size for
// `per_cu` resident workgroups per CU.  `deal`: the first items may go by workgroup index.
struct QueueLaunch { int grid; hipError_t err; };
static inline QueueLaunch tile_queue_prepare(AttnParams& p, unsigned int* counters, int64_t total, int heads, int per_cu, hipStream_t st,
                                             bool already_clear = false, bool deal = true) {
  QueueLaunch r{0, hipSuccess};
  const int cus = cu_count(&r.err);
  if (r.err != hipSuccess) return r;
  const int64_t nH = p.B * heads;
  p.q_counters = counters;
  p.q_total = (int32_t)total;
  p.q_per_xcd = (nH % 8 == 0) ? (int32_t)(total / 8) : 0;
  const int64_t want = (int64_t)cus * per_cu;
  r.grid = (int)(total < want ? total : want);
  // One list of more than two items per workgroup leaves the first round to the order of arrival too (start dealt : by
  // arrival, dQ 65536 x 4 4885 : 4818 us, dK/dV 131072 x 1 6918 : 6793, forward 65536 x 3 2666 : 2646, but forward 9000 x 20
  // 394 : 399; with two items or fewer dQ 16384 x 6 496 : 598).
  p.q_dealt = deal && (p.q_per_xcd > 0 || total <= 2 * want) ? (uint32_t)r.grid : 0u;
  // Head by head for the heavier 5/8 of a head's tiles, so that an XCD's workgroups share a head's rows in its L2; from the
  // heaviest tile of all heads down where a workgroup gets two items at most and the balance is what counts (dQ 4096 x 32
  // 196 : 168 us, dQ 1600 x 24 x 2 at head dimension 64 54 : 48, 4096 x 16 71 : 71; above it dK/dV 2048 x 40 94 : 100,
  // 2 x 4096 x 32 479 : 497, 32768 x 32 13.5 : 14.0 ms).
  p.q_heavy = total <= 2 * want ? 0 : p.tiles - p.tiles * 3 / 8;
  // (`already_clear`: a kernel in front of this launch on the same stream has cleared the counters)
  if (!already_clear) {
    tile_queue_reset_kernel<<<1, 64, 0, st>>>(counters);
    r.err = hipGetLastError();
  }
  return r;
}

}  // namespace ie
