// Device side of the persistent partitioned reduction (gfx950, wave64).
//
// One launch serves one epoch of a request.  The epoch's counters were
// cleared by the previous launch (two counter sets alternate by epoch
// parity), so no wavefront ever has to find out that it is the last one,
// and no other launch precedes the reduce kernel.  The worker is a workgroup
// of up to kMaxWavesPerGroup wavefronts that reduce the rows of one tile
// together (wavefront w of W takes every W-th row).  No worker ever waits
// for another, so the launch needs no co-residency and drains even if it is
// larger than the machine.  Wavefront 0 of the group drives the protocol; the
// group meets at one barrier per tile.  A worker loops:
//
//   1. take a global tile index t: its workgroup number the first time (no
//      atomic, so the launch does not start with a burst of atomics on one
//      address), then one atomic add per tile, issued before the current
//      tile is reduced so that its latency hides behind the tile;
//   2. wait until t is covered by the work queue.  While starved, the few
//      workers at the front of the claim order move newly readied partitions
//      into the queue: they read the host ready list (host-coherent memory,
//      written by pready) and this epoch's device ready ring (written by the
//      ready kernels), and whoever finds entries locks the queue with a
//      compare-and-swap on its state and appends each partition not yet
//      queued this epoch with the running total of its tiles.
//      Partitions are reduced in the order they became ready (the chunk
//      pipeline of Section 4.3: chunks proceed as soon as they can);
//   3. find the queue entry covering t (64 entries per wave-wide probe),
//      giving the partition and the tile inside it;
//   4. reduce the tile (rank order 0..P-1 per element), store the result;
//   5. publish: once the group's stores are in memory, add the tile to its
//      partition's done counter (finished tiles are published in batches, see
//      publish()); the worker that completes the partition stores the epoch
//      into its arrived flag in host-coherent memory (completion is signalled
//      only after every chunk of the partition has landed, Section 4.5).
//
// Exit: t >= total tiles.  A worker that starves past the deadline, or sees
// the host's abort word, records the reason (also in host memory, stamped
// with the epoch) and leaves; the others follow.  The host's wait returns
// when the done word carries the epoch, or an error is recorded (or the
// launch has failed).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "layout.hpp"

namespace pcoll {
namespace dev {

// ---------------------------------------------------------------- atomics
__device__ __forceinline__ uint32_t ld_acq_sys(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ uint32_t ld_rlx_sys(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ uint64_t ld_rlx_sys64(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ uint32_t ld_acq(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t ld_rlx(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t ld_acq64(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t ld_rlx64(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_rlx(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_rel(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_rlx64(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_rel64(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_rel_sys(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Pointer into the constant address space: uniform loads through it become
// scalar loads.  Only for tables no kernel writes during the launch.
template <class T>
using const_ptr = __attribute__((address_space(4))) const T*;

// ---------------------------------------------------------- wave helpers
__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }
__device__ __forceinline__ uint32_t uni(uint32_t v) {
  return __builtin_amdgcn_readfirstlane(v);
}
__device__ __forceinline__ uint64_t uni64(uint64_t v) {
  uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return ((uint64_t)hi << 32) | lo;
}
// Inclusive prefix sum over the wavefront (every lane active) in six DPP
// adds: within rows of 16 lanes, then across them.  (Through LDS shuffles
// each step waits for a round trip, and the queue is on the critical path.)
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x) {
  int v = (int)x;
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  // lane 15 of each row to the next one; lane 31 to the upper half
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
  return (uint32_t)v;
}
__device__ __forceinline__ uint32_t lane_value(uint32_t v, uint32_t lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)lane);
}

// ---------------------------------------------------------- the partitions
// Elements [off, off + len) of bucket `bucket`: the chunk rule, computed from
// the bucket's count and partition length, so that no table of partitions is
// read (a dependent load per tile and per queued partition).
struct Span {
  uint32_t bucket;
  uint64_t off, len;
};
__device__ __forceinline__ Span span_of(uint32_t k, uint32_t bucket,
                                        uint64_t count, uint64_t psize) {
  const uint64_t at = (uint64_t)k * psize;
  const uint64_t off = at < count ? at : count;
  const uint64_t left = count - off;
  return {bucket, off, left < psize ? left : psize};
}
// A wave-uniform partition: the bucket's numbers come from the arguments
// (one bucket) or by scalar loads.
__device__ __forceinline__ Span part_span(const ReduceArgs& a, uint32_t part) {
  if (a.bucket_parts == a.nparts_total)
    return span_of(part, 0u, a.count0, a.psize0);
  const uint32_t b = part / a.bucket_parts;
  const const_ptr<BucketDesc> bd = (const_ptr<BucketDesc>)(a.buckets) + b;
  return span_of(part - b * a.bucket_parts, b, bd->count, bd->psize);
}
// Rows of each lane's own partition.
__device__ __forceinline__ uint32_t part_rows(const ReduceArgs& a,
                                              uint32_t part) {
  Span s;
  if (a.bucket_parts == a.nparts_total) {
    s = span_of(part, 0u, a.count0, a.psize0);
  } else {
    const uint32_t b = part / a.bucket_parts;
    s = span_of(part - b * a.bucket_parts, b, a.buckets[b].count,
                a.buckets[b].psize);
  }
  return (uint32_t)((s.len + ((1ull << a.row_shift) - 1ull)) >> a.row_shift);
}

// ------------------------------------------------------------- the queue

// Appends the partitions held by the lanes with `valid` set, in lane order.
// Caller holds the ingest lock; qcount / qtiles / qrows are wave-uniform and
// updated in place.
//
// Tile count (guided self-scheduling, when `guide` f > 0): a partition
// whose first row has `rem` rows of the request from it to the end (itself
// included, partitions not yet queued counted too) is cut into tiles of
// about s = clamp(ceil(rem / (f G)), min_tile_rows, max_tile_rows) rows, G
// the workgroups of the launch: large tiles while much work remains, small
// ones near the end, so that workgroups run out of work at about the same
// time.  With f = 0 every tile has max_tile_rows rows.
//
// A partition is appended once per epoch, whatever the number of ready
// signals: queue_stamp() exchanges its queued stamp first and the append
// keeps it only if the stamp was not this epoch's already.  It issues
// nothing that waits, so the stamps of several chunks can be in flight
// together before their appends.  The host lists a partition once per epoch
// (it checks), so while no entry of the device ring has been queued this
// epoch (`alone`, under the lock), a host entry cannot be a duplicate: its
// stamp is stored and nothing is waited for.
struct Stamped {
  uint32_t part;
  uint32_t rows;   // rows of the partition (when valid)
  bool valid;
};

__device__ __forceinline__ Stamped queue_stamp(const ReduceArgs& a,
                                               uint32_t epoch, bool valid,
                                               uint32_t part, bool alone) {
  Stamped c{part, 0u, valid && part < a.nparts_total};
  uint32_t old = alone ? ~epoch : epoch;
  if (c.valid) {
    // the bucket's loads (batched requests) do not wait for the exchange
    c.rows = part_rows(a, part);
    if (alone)
      st_rlx(&a.queued[part], epoch);
    else
      old = __hip_atomic_exchange(&a.queued[part], epoch, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
  }
  c.valid = c.valid && old != epoch;
  return c;
}

// A worker's place in the queue: the entry `cursor` found last, its
// partition, and the tiles [prev_end, end) it covers (end = 0: none yet).
struct Place {
  uint32_t cursor, prev_end, part, end;
};

// `t`, `at`: the caller's own tile; if these entries cover it, `at` is set to
// its entry, which spares the caller the read of what it has just written.
__device__ __forceinline__ void queue_append(const ReduceArgs& a,
                                             const Stamped& c, uint32_t t,
                                             uint32_t& qcount,
                                             uint32_t& qtiles,
                                             uint64_t& qrows, Place& at) {
  const uint32_t lane = lane_id();
  const bool valid = c.valid;
  const uint32_t part = c.part;
  const uint32_t rows = valid ? c.rows : 0u;
  uint64_t s = a.max_tile_rows;
  if (a.guide) {
    const uint32_t rincl = wave_incl_scan(rows);
    const uint64_t before = qrows + (rincl - rows);
    const uint64_t rem = a.total_rows > before ? a.total_rows - before : rows;
    const uint64_t g = (uint64_t)a.guide * a.total_groups;
    s = (rem + g - 1) / g;
    if (s < a.min_tile_rows) s = a.min_tile_rows;
    if (s > a.max_tile_rows) s = a.max_tile_rows;
    qrows += lane_value(rincl, 63);
  }
  const uint32_t s32 = (uint32_t)s;  // at most max_tile_rows
  const uint32_t nt = valid ? (rows == 0u ? 1u : (rows + s32 - 1u) / s32) : 0u;
  const uint32_t incl = wave_incl_scan(nt);
  const uint64_t vm = __ballot(valid);
  const uint32_t rank = __popcll(vm & ((1ull << lane) - 1ull));
  const uint32_t slot = qcount + rank;
  if (valid && slot < a.nparts_total) {
    const uint64_t e = ((uint64_t)(qtiles + incl) << 32) | part;
    st_rlx64(reinterpret_cast<uint64_t*>(&a.queue[slot]), e);
    if (a.tile_counts) a.tile_counts[part] = nt;
  }
  const uint64_t past = __ballot(valid && qtiles + incl > t);
  if (past != 0 && t >= qtiles) {
    const uint32_t k = (uint32_t)(__ffsll((long long)past) - 1);
    at.cursor = qcount + (uint32_t)__popcll(vm & ((1ull << k) - 1ull));
    at.part = lane_value(part, k);
    at.end = qtiles + lane_value(incl, k);
    at.prev_end = at.end - lane_value(nt, k);
  }
  qcount += (uint32_t)__popcll(vm);
  qtiles += lane_value(incl, 63);
}

// Parts of the queue state.
__device__ __forceinline__ uint32_t q_entries(uint64_t qs) {
  return (uint32_t)((qs & ~(kQLocked | kQDevice)) >> 32);
}
__device__ __forceinline__ uint32_t q_tiles(uint64_t qs) {
  return (uint32_t)qs;
}

// Entries reserved in this epoch's device ready ring, from its word (which
// carries the epoch from the previous launch on; a word of another epoch
// counts as empty).
__device__ __forceinline__ uint32_t ring_entries(uint64_t w, uint32_t epoch) {
  w = uni64(w);
  return (uint32_t)(w >> 32) == epoch ? (uint32_t)w : 0u;
}
__device__ __forceinline__ uint64_t ring_word(const ReduceArgs& a,
                                              uint32_t epoch) {
  return ld_rlx64(&a.ring[epoch & 1u].reserve);
}

// The next 256 host ready entries from entry `at` on (64 per word of `w`),
// read in one bus round trip, and how many from the first on are this
// epoch's (lim[k] of chunk k, `total` in all): the list ends at the first
// entry of another epoch (not yet written).
struct HostWindow {
  uint64_t w[4];
  uint32_t lim[4];
  uint32_t total;
};
__device__ __forceinline__ HostWindow host_window(const ReduceArgs& a,
                                                  uint32_t epoch,
                                                  uint32_t at) {
  HostWindow h;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t i = at + 64u * k + lane_id();
    h.w[k] = i < a.nparts_total ? ld_rlx_sys64(&a.hlist[i]) : 0ull;
  }
  h.total = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint64_t bad = __ballot((uint32_t)(h.w[k] >> 32) != epoch);
    h.lim[k] = bad ? (uint32_t)(__ffsll((long long)bad) - 1) : 64u;
    if (h.total != 64u * k) h.lim[k] = 0u;
    h.total += h.lim[k];
  }
  return h;
}

// Moves newly readied partitions into the queue.  Returns true if it queued
// any tile, with the new queue state in qs_out (the caller's to use: it
// wrote the last entries and acquired the others).  Wave-wide.
//
// `qs` is the queue state as the caller has just read it (or knows it: zero
// at the start of an epoch).  The lists are read before the lock is taken: a
// read of host memory takes 1.2 us, and several workers have theirs in
// flight, so that an entry is seen soon after the host writes it.  The lock's compare-and-swap then expects `qs`: if it succeeds, nothing
// was queued in between, and the host entries read are still the next ones;
// if another worker was first, the entries it left are still good, and the
// compare-and-swap is repeated on the newer state.  (Once device ring entries
// were consumed, the consumed counts are in a word of their own, read again
// under the lock.)
//
// `probe`: a worker that has waited a while looks at one host entry first, so
// an epoch that waits for its producers keeps no wide bus reads in flight.
__device__ __forceinline__ bool try_ingest(const ReduceArgs& a, uint32_t epoch,
                                           uint64_t qs, bool probe,
                                           uint32_t t, uint64_t& qs_out,
                                           Place& at) {
  const uint32_t lane = lane_id();
  EpochCounters* c = a.ctr;
  if (qs & kQLocked) return false;
  const bool device = (qs & kQDevice) != 0;
  const uint64_t rw = ring_word(a, epoch);
  uint32_t hcons = q_entries(qs), dcons = 0;
  if (device) {
    const uint64_t used = uni64(ld_rlx64(&c->consumed));
    hcons = (uint32_t)used;
    dcons = (uint32_t)(used >> 32);
  }
  bool host = true;
  if (probe) {
    // both in flight; what the ring holds is taken without waiting for the
    // host list's round trips over the bus (the next look makes those)
    uint64_t head = 0;
    if (lane == 0 && hcons < a.nparts_total)
      head = ld_rlx_sys64(&a.hlist[hcons]);
    host = ring_entries(rw, epoch) <= dcons;
    if (host && (uint32_t)(uni64(head) >> 32) != epoch) return false;
  }
  // (past the list's end nothing is read)
  HostWindow h = host_window(a, epoch, host ? hcons : a.nparts_total);
  const uint32_t dr = ring_entries(rw, epoch);
  if (h.total == 0u && dr <= dcons) return false;

  uint32_t skip = 0;  // entries of the window that another worker has queued
  for (uint32_t tries = 0;; ++tries) {
    uint64_t seen = qs;
    if (lane == 0)
      __hip_atomic_compare_exchange_strong(
          &c->qstate, &seen, qs | kQLocked, __ATOMIC_RELAXED,
          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    seen = uni64(seen);
    if (seen == qs) break;
    for (; (seen & kQLocked) && tries < 4u; ++tries) {
      __builtin_amdgcn_s_sleep(2);
      seen = uni64(ld_rlx64(&c->qstate));
    }
    skip = q_entries(seen) - hcons;
    if ((seen & (kQLocked | kQDevice)) || device || skip >= h.total ||
        tries >= 4u)
      return false;
    qs = seen;
  }
  if (device) {
    const uint64_t used = uni64(ld_rlx64(&c->consumed));
    dcons = (uint32_t)(used >> 32);
    if ((uint32_t)used != hcons) {  // only duplicates, so qs is the same
      hcons = (uint32_t)used;
      h = host_window(a, epoch, host ? hcons : a.nparts_total);
    }
  }
  uint32_t qcount = q_entries(qs), qtiles = q_tiles(qs);
  uint64_t qrows = 0;
  if (a.guide) {
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    qrows = uni64(ld_rlx64(&c->queued_rows));
  }
  const uint32_t qtiles0 = qtiles;
  const auto state = [&] {
    return (dcons ? kQDevice : 0ull) | ((uint64_t)qcount << 32) | qtiles;
  };
  // publishes the counts so far, still holding the lock
  const auto publish_counts = [&] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    if (lane == 0) st_rlx64(&c->qstate, kQLocked | state());
  };

  // the host's entries, 256 per bus round trip; the counts are published
  // after every 64 that others follow, so that workers start on them
  for (;;) {
    // acquires the lock; and the host wrote its entries with release stores
    // after their partitions' data were in place
    if (h.total)
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");
    else
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    // stamps and buckets of every chunk in flight together
    Stamped st[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      st[k] = queue_stamp(a, epoch,
                          lane < h.lim[k] && 64u * k + lane >= skip,
                          (uint32_t)h.w[k], dcons == 0u);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (h.lim[k] == 0u) break;
      queue_append(a, st[k], t, qcount, qtiles, qrows, at);
      if (k == 3 || h.lim[k < 3 ? k + 1 : 3] != 0u) publish_counts();
    }
    hcons += h.total;
    skip = 0;
    if (h.total != 256u || hcons >= a.nparts_total) break;
    h = host_window(a, epoch, hcons);
    if (h.total == 0u) break;
  }

  // this epoch's device ready ring: entry c is slot c, stored as (epoch <<
  // 32) | part; stop at the first reserved entry whose writer has not
  // stored it yet (its slot still holds an older epoch's tag)
  const uint64_t* ring = a.dlist + (size_t)(epoch & 1u) * a.nparts_total;
  while (dcons < dr) {
    const uint32_t i = dcons + lane;
    const bool in = i < dr;
    uint64_t e = in ? ld_rlx64(&ring[i]) : 0ull;
    const bool ok = in && (uint32_t)(e >> 32) == epoch;
    const uint64_t pending = __ballot(in && !ok);
    const uint32_t lim =
        pending ? (uint32_t)(__ffsll((long long)pending) - 1) : 64u;
    // the producers of these partitions ended before their signals ran
    // (stream order), which made their stores visible device-wide;
    // acquire, so that no stale line of them is read from this XCD's caches
    if (__ballot(ok && lane < lim)) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE,
                                                            "agent");
    queue_append(a,
                 queue_stamp(a, epoch, ok && lane < lim, (uint32_t)e, false),
                 t, qcount, qtiles, qrows, at);
    const uint32_t avail = dr - dcons < 64u ? dr - dcons : 64u;
    dcons += lim < avail ? lim : avail;
    if (pending) break;
  }

  // one release for the entries, stamps and counters, then one store that
  // publishes the counts and gives the lock up
  if (lane == 0) {
    if (dcons) st_rlx64(&c->consumed, ((uint64_t)dcons << 32) | hcons);
    if (a.guide) st_rlx64(&c->queued_rows, qrows);
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  qs_out = state();
  if (lane == 0) st_rlx64(&c->qstate, qs_out);
  return qtiles != qtiles0;
}

// Records the first error of the epoch; the recording wavefront also
// publishes it to the host, stamped with the epoch.
__device__ __forceinline__ void set_error(const ReduceArgs& a, uint32_t code,
                                          uint32_t epoch) {
  if (lane_id() == 0) {
    uint32_t expect = 0;
    if (__hip_atomic_compare_exchange_strong(&a.ctr->error, &expect, code,
                                             __ATOMIC_RELAXED,
                                             __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT)) {
      __hip_atomic_store(&a.host->status, code, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_SYSTEM);
      st_rel_sys(&a.host->status_epoch, epoch);
    }
  }
}

enum WaitResult { kBail, kStop, kReady, kDrain };

// Waits until tile t is queued (kReady, with the queue state in qs_out).
// kDrain, with `pending` tiles unpublished: it would have to wait, and they
// must not sit behind the wait; the caller publishes them and calls again.
// kStop: every partition is queued and t is beyond the last tile.  kBail:
// give up (deadline, host abort, or another worker's error).  The few
// workers at the front of the claim order (t within 8 tiles of the queued
// total) poll the ready lists and the host's abort word; the rest re-read
// the device-side queue state at a slower pace, and after a long wait they
// also poll the lists now and then (see below).
__device__ __forceinline__ WaitResult wait_queued(const ReduceArgs& a,
                                                  uint32_t t, uint32_t epoch,
                                                  uint64_t t0, bool first,
                                                  bool pending,
                                                  uint64_t& qs_out,
                                                  Place& at) {
  // the queue state this worker acquired last: entries it covers are
  // already visible, so a tile inside it needs no new acquire; and once it
  // holds every partition there is no more to come
  if (q_tiles(qs_out) > t) return kReady;
  if (q_entries(qs_out) >= a.nparts_total) return kStop;
  for (uint32_t spins = 0;; ++spins) {
    uint64_t qs = 0;
    if (first && spins == 0u && t < 8u) {
      // an epoch starts with nothing queued: the first workers look at the
      // ready lists at once, worker t after t fifths of a microsecond, so
      // that the list is seen at a fine grain while the host's first
      // readiness calls arrive
      for (uint32_t k = 0; k < t; ++k) __builtin_amdgcn_s_sleep(7);
    } else {
      // polled relaxed; acquired (one fence) only once it covers t: an
      // acquire invalidates caches, which a waiting kernel should not keep
      // doing to the kernels that run beside it
      qs = uni64(ld_rlx64(&a.ctr->qstate));
    }
    const uint32_t qt = q_tiles(qs);
    if (qt > t) {
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      qs_out = qs;
      return kReady;
    }
    if (q_entries(qs) >= a.nparts_total) return kStop;
    if (pending) return kDrain;
    // The workers near the queue's end ingest.  So does, every 128th
    // poll, any worker that has waited 64 polls: a launch can have more
    // workgroups than fit on the device at once, and the tiles at the
    // queue's end may belong to workgroups that start only when resident
    // ones leave, so ingesting must not depend on them.  Those far from the
    // end read host memory (the ready list, the abort word) that rarely:
    // a read of host memory crosses the bus, and a few hundred waiting
    // workers that read it every few polls load the bus enough to slow
    // the dispatch of kernels on other streams (the producers an epoch
    // waits for).
    const bool near = t - qt < 8u;
    const bool stuck = spins >= 64u;
    const bool front = near || (stuck && (spins & 127u) == 0u);
    if (front && try_ingest(a, epoch, qs, spins >= 16u, t, qs_out, at)) {
      if (q_tiles(qs_out) > t) return kReady;
      continue;
    }
    if (uni(ld_rlx(&a.ctr->error)) != 0u) return kBail;
    if ((spins & 7u) == 7u) {
      const bool poll_abort = near || (stuck && (spins & 255u) == 255u);
      if (poll_abort && uni(ld_rlx_sys(&a.host->abort)) == epoch) {
        set_error(a, kStatusAborted, epoch);
        return kBail;
      }
      if (wall_clock64() - t0 > a.timeout_ticks) {
        set_error(a, kStatusTimeout, epoch);
        return kBail;
      }
    }
    if (near)
      __builtin_amdgcn_s_sleep(2);
    else
      __builtin_amdgcn_s_sleep(8);
  }
}

// Finds the queue entry covering tile t among entries [at.cursor, qcount).
// The place only moves forward, since a worker's claims increase; a tile in
// the same partition as the previous one needs no queue read.
__device__ __forceinline__ void locate(const ReduceArgs& a, uint32_t t,
                                       uint32_t qcount, Place& at) {
  const uint32_t lane = lane_id();
  if (t < at.end) return;  // t >= prev_end: claims increase
  for (;;) {
    const uint32_t i = at.cursor + lane;
    const uint64_t e =
        i < qcount
            ? ld_rlx64(reinterpret_cast<const uint64_t*>(&a.queue[i]))
            : ~0ull;
    const uint32_t ce = (uint32_t)(e >> 32);
    const uint64_t m = __ballot(ce > t);
    if (m) {
      const uint32_t k = (uint32_t)(__ffsll((long long)m) - 1);
      if (k != 0) at.prev_end = lane_value(ce, k - 1);
      at.cursor += k;
      at.part = lane_value((uint32_t)e, k);
      at.end = lane_value(ce, k);
      return;
    }
    at.prev_end = lane_value(ce, 63);
    at.cursor += 64;
  }
}

// Completion of finished tiles.  Publishing a tile means: its stores are
// visible device-wide, then the partition's done counter counts it; the
// worker whose count completes the partition stores the epoch into the
// host-visible arrived flag.  The stores go through to memory (st_row), so a
// wavefront that has waited for its own has nothing left to release.  A group
// keeps up to `publish_batch` finished tiles pending, its wavefronts running
// on into the next tiles with the stores still in flight; to publish, every
// wavefront waits for its stores once (kJobDrain), then one instruction counts
// the tiles, a lane for each partition among them.  It does so when the batch
// is full, before it waits for work (a partition is late by at most one batch
// of one group, and only while the kernel has a backlog of readied work).  A
// lane for each tile would put 64 atomics of every group on one counter where
// a partition is large, at 16 ns each: fp32, 8 ranks, 256 MiB each, 1 / 4 / 16
// partitions, kernel on a cold cache 480 / 450 / 436 us that way against 369 /
// 367 / 366 now (64 partitions 365 either way), 512 MiB in one partition 732.
//
// A group that runs out of work counts itself instead (retire): when the last
// one has, every tile of the epoch is final, and it stores the epoch into the
// host's done word.  That is one bus write, not one per partition (256
// partitions of a small message: 28 -> 19 us), and the host does not wait for
// the launch to retire and its end event to be processed.
//
// Measured: with ordinary stores, each publication wrote back the XCD's L2
// (0.2 us alone, and one after the other for the groups of an XCD; 256 groups
// publishing at the end cost 10 us, so the last tiles were left to the
// launch's end).  With the done word, an epoch of 4 KiB over 8 ranks takes
// 14.3 us of host time instead of 20.8, of 1 MiB over 4 ranks 16.5 instead of
// 21.1.  The launch itself ends later by what it now counts: kernel on a cold
// cache, 8 ranks, 2^10 elements in 4 partitions 8.1 -> 9.0 us, 2^22 32.6 ->
// 33.9 us, which is what a stream that waits for the epoch sees.
struct Pending {
  uint32_t part;
  uint32_t nt;
};

__device__ __forceinline__ void publish(const ReduceArgs& a,
                                        const Pending* pend, uint32_t& npend,
                                        uint32_t epoch) {
  if (npend == 0) return;
  const uint32_t l = lane_id();
  const bool in = l < npend;
  const uint32_t part = in ? pend[l].part : 0u;
  // a group's tiles of one partition follow each other: the first of them
  // counts them all
  const bool head = in && (l == 0u || pend[l - 1u].part != part);
  const uint64_t heads = __ballot(head);
  if (in && a.tile_hits)
    __hip_atomic_fetch_add(&a.tile_hits[part], 1u, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
  if (head) {
    const uint64_t later = heads & ~((2ull << l) - 1ull);
    const uint32_t n =
        (later ? (uint32_t)__ffsll((long long)later) - 1u : npend) - l;
    const uint32_t nt = pend[l].nt;
    // exactly one add completes a partition; one of one tile needs no count
    if (nt == 1u ||
        __hip_atomic_fetch_add(&a.done[part], n, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT) +
                n ==
            nt)
      __hip_atomic_store(&a.arrived[part], epoch, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_SYSTEM);
  }
  npend = 0;
}

// The group has run out of work, and its stores are in memory: its pending
// tiles need no counts of their own.
__device__ __forceinline__ void retire(const ReduceArgs& a,
                                       const Pending* pend, uint32_t npend,
                                       uint32_t epoch) {
  const uint32_t l = lane_id();
  if (a.tile_hits && l < npend)
    __hip_atomic_fetch_add(&a.tile_hits[pend[l].part], 1u, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
  if (l != 0) return;
  // a level of one member has nothing to count: a returning atomic, 0.3 us,
  // less with up to 16 workgroups, two with one
  const uint32_t set = blockIdx.x % kRetireSets;
  const uint32_t members = (a.total_groups - set + kRetireSets - 1) / kRetireSets;
  const uint32_t sets = min(a.total_groups, kRetireSets);
  const auto last = [&](uint32_t k, uint32_t of) {
    return of == 1u ||
           __hip_atomic_fetch_add(&a.ctr->retired[k].n, 1u, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT) +
                   1u ==
               of;
  };
  if (last(set, members) && last(kRetireSets, sets))
    __hip_atomic_store(&a.host->done, epoch, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

// The tile index after the first round: one relaxed atomic add by lane 0.
__device__ __forceinline__ uint32_t claim(const ReduceArgs& a) {
  uint32_t t = 0;
  if (lane_id() == 0)
    t = __hip_atomic_fetch_add(&a.ctr->claim, 1u, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT) +
        a.total_groups;
  return t;  // valid in lane 0; broadcast by the caller when needed
}

// What wavefront 0 hands the group: one tile, or
constexpr uint32_t kJobStop = ~0u;         // the end
constexpr uint32_t kJobDrain = ~0u - 1u;   // wait for your stores
constexpr uint32_t kJobRetire = ~0u - 2u;  // the same, and the end
struct TileJob {
  uint32_t part;  // global partition, or one of the above
  uint32_t lt;    // tile index within the partition
  uint32_t nt;    // tiles of the partition
};

// The epoch after e (the host's rule: epoch 0 is never used, so after
// 2^32 - 1 the count goes on at 2, which keeps the parity alternating).
__device__ __forceinline__ uint32_t next_epoch(uint32_t e) {
  return e + 1u == 0u ? 2u : e + 1u;
}

// Clears the counter set and done counters of the other epoch parity, for
// the next launch, and opens the other parity's device ready ring for the
// next epoch: the previous launch, which used them, has retired (the
// stream orders launches), and the next one starts only after this one.
// Every workgroup clears its share of the done counters; workgroup 0 the
// counter set and the ring's reservation word.  A device-side signal of an
// ended epoch that still tries to reserve in that ring then finds another
// epoch in the word and appends nothing.
__device__ __forceinline__ void clear_next_epoch(const ReduceArgs& args,
                                                 uint32_t epoch) {
  const uint32_t other = (epoch & 1u) ^ 1u;
  uint32_t* done = args.done + (size_t)other * args.nparts_total;
  for (uint32_t p = blockIdx.x * 64u + lane_id(); p < args.nparts_total;
       p += args.total_groups * 64u)
    st_rlx(&done[p], 0u);
  if (blockIdx.x == 0 && lane_id() == 0) {
    EpochCounters* c = args.ctr + other;
    st_rlx(&c->claim, 0u);
    st_rlx64(&c->qstate, 0ull);
    st_rlx64(&c->consumed, 0ull);
    st_rlx64(&c->queued_rows, 0ull);
    st_rlx(&c->error, 0u);
    for (uint32_t k = 0; k <= kRetireSets; ++k) st_rlx(&c->retired[k].n, 0u);
    st_rlx64(&args.ring[other].reserve, (uint64_t)next_epoch(epoch) << 32);
  }
}

// The worker loop of one workgroup.  Tile::run<P>(bucket, partition offset,
// partition length, tile index, tiles of the partition, interleave,
// wavefront, wavefronts) reduces this wavefront's rows of a tile.
template <class Tile, int P>
__device__ __forceinline__ void persistent_loop(const ReduceArgs& args) {
  // two jobs in turn: wavefront 0 writes the next one while others still
  // work on the last, so one barrier per tile is enough
  __shared__ TileJob jobs[2];
  __shared__ Pending pend[kMaxPublishBatch];
  const uint32_t wave = uni(threadIdx.x / 64u);
  const uint32_t nwaves = blockDim.x / 64u;
  // only wavefront 0 runs the protocol and needs the epoch.  A graph
  // replay reads it from host memory: the launch has no more workgroups
  // than tiles, every workgroup's first tile is its own number, so the
  // epoch cannot complete (and the host cannot store the next stamp)
  // before every workgroup has read this one
  uint32_t epoch = 0;
  if (wave == 0)
    epoch = args.epoch ? args.epoch : uni(ld_acq_sys(&args.host->epoch));
  ReduceArgs a = args;
  a.ctr = args.ctr + (epoch & 1u);
  a.done = args.done + (size_t)(epoch & 1u) * args.nparts_total;
  if (wave == 0) clear_next_epoch(args, epoch);
  const uint64_t t0 = wall_clock64();
  Place at{0u, 0u, 0u, 0u};
  uint32_t t = blockIdx.x;  // first round: tile = workgroup number
  uint32_t next = 0;
  uint64_t qs = 0;          // queue state last acquired (wavefront 0)
  uint32_t npend = 0;       // finished tiles not yet published (wavefront 0)
  uint32_t ntiles = 0;      // tiles reduced (wavefront 0, for the trace)
  uint64_t t_first = 0;     // when the first tile was queued (trace)
  bool first = true;
  if (wave == 1 && a.bucket_parts == a.nparts_total) {
    // one bucket: bring its pointers into the scalar cache while wavefront 0
    // waits for the queue
    const const_ptr<BucketDesc> bd = (const_ptr<BucketDesc>)(a.buckets);
    asm volatile("" ::"s"(bd->in[0]), "s"(bd->in[P - 1]), "s"(bd->out));
  }
  for (uint32_t turn = 0;; turn ^= 1u) {
    if (wave == 0) {
      TileJob j{kJobStop, 0u, 0u};
      const WaitResult w =
          npend >= a.publish_batch
              ? kDrain
              : wait_queued(a, t, epoch, t0, first, npend != 0u, qs, at);
      first = false;
      if (w == kReady) {
        if (a.trace && ntiles == 0) t_first = wall_clock64();
        locate(a, t, q_entries(qs), at);
        j.part = at.part;
        j.lt = t - at.prev_end;
        j.nt = at.end - at.prev_end;
        next = claim(a);  // in flight while the tile is reduced
      } else if (w != kBail) {
        j.part = w == kStop ? kJobRetire : kJobDrain;
      }
      if (a.trace && (w == kStop || w == kBail) && lane_id() == 0) {
        uint64_t* s = a.trace + (size_t)blockIdx.x * 4u;
        s[0] = t0;
        s[1] = t_first;
        s[2] = wall_clock64();
        s[3] = ntiles;
      }
      if (lane_id() == 0) jobs[turn] = j;
    }
    __syncthreads();
    const TileJob j = jobs[turn];
    if (j.part == kJobStop) break;
    if (j.part >= kJobRetire) {  // retire or drain
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      if (j.part == kJobRetire) {
        if (wave == 0) retire(a, pend, npend, epoch);
        break;
      }
      if (wave == 0) publish(a, pend, npend, epoch);
      continue;
    }
    // the bucket table is read-only for the whole launch: scalar loads
    const Span sp = part_span(a, j.part);
    const const_ptr<BucketDesc> bd =
        (const_ptr<BucketDesc>)(a.buckets) + sp.bucket;
    Tile::template run<P>(bd, sp.off, sp.len, j.lt, j.nt, a.interleave, wave,
                          nwaves);
    if (wave == 0) {
      if (lane_id() == 0) pend[npend] = Pending{j.part, j.nt};
      ++npend;
      ++ntiles;
      t = uni(next);
    }
  }
}

// ------------------------------------------------------ memory streaming
// 16-byte streaming access through the global address space (global_load /
// global_store with the nontemporal hint, never the generic flat path).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const u32x4* gload_ptr;
typedef __attribute__((address_space(1))) u32x4* gstore_ptr;
__device__ __forceinline__ uint4 ld_stream(const uint4* p) {
  const u32x4 v = __builtin_nontemporal_load((gload_ptr)(p));
  return make_uint4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void st_stream(uint4* p, uint4 v) {
  const u32x4 w = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(w, (gstore_ptr)(p));
}

// Lane's 16 bytes of the 1 KiB row at `row` (wave-uniform), through a buffer
// descriptor: the row's address stays in scalar registers.
__device__ __forceinline__ uint4 ld_row(const void* row, uint32_t lane) {
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(row), 0, 1024, 0x00027000);
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(
      rs, (int)(lane * 16u), 0, /* nt */ 2);
  return make_uint4(v[0], v[1], v[2], v[3]);
}

// Stores of a tile's results.  They go through to memory (the agent-scope
// bit beside the nontemporal hint) instead of staying dirty in this XCD's L2:
// once a wavefront has waited for them they are visible device-wide, and
// publishing a tile needs no release, which writes back the whole L2 (0.2 us
// alone, and one after the other for all workgroups of an XCD).  Whole cache
// lines either way, and the stream's rate is the same.
//
// Lane's 16 bytes of the 1 KiB row at `row` (wave-uniform).
__device__ __forceinline__ void st_row(void* row, uint32_t lane, uint4 v) {
  const u32x4 w = {v.x, v.y, v.z, v.w};
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(row, 0, 1024, 0x00027000);
  __builtin_amdgcn_raw_buffer_store_b128(w, rs, (int)(lane * 16u), 0,
                                         /* nt | sc1 */ 2 | 16);
}
// One scalar (the ragged ends, the block scales).
template <class T>
__device__ __forceinline__ void st_out(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Knuth's TwoSum: s = fl(a + b), e = a + b - s exactly.
__device__ __forceinline__ void two_sum(float a, float b, float& s, float& e) {
  s = a + b;
  float bv = s - a;
  float av = s - bv;
  e = (a - av) + (b - bv);
}

}  // namespace dev
}  // namespace pcoll
