// Slot-level replay of a finished plan under given kernel durations.
//
// Not a step of G10's planner: a small stand-in for the breakdown its simulator reports (stall
// time next to compute time, traffic per destination; evaluation Sections 7.2, 7.3, 7.6).  The
// model: kernels run in order; the eviction of a migration is issued when kernel
// `evict_after` has finished, its prefetch when the last absent kernel has finished (or at the
// earlier slot smart prefetching moved it to); every (destination, direction) pair is one
// channel that serves its transfers one after the other in the order they were issued (same
// instant: plan order), a transfer taking the plan's eviction / prefetch time; a prefetch does
// not start before its eviction is done; a kernel starts when the previous one has finished and
// every prefetch whose tensor it uses is done, and what it waits beyond the previous kernel's
// end is stall time.  Two iterations are replayed end to end with every migration in both (a
// weight evicted in the first comes back in the second); the second one is reported.
//
// On the device: every migration gives up to three events per iteration (eviction issued,
// prefetch issued, tensor used), keyed by (point before kernel j, kind, plan order) and put in
// order by the radix sort.  The replay itself is a chain - each completion time depends on the
// channel and on the stalls before it - and runs in one wavefront, 64 events at a time, one per
// lane.  What couples the channels is the delay of the kernels alone, and that changes only
// where a kernel waits: up to the next such event every channel is a queue of known requests,
// whose completion times come from running maxima.  So the walk takes a step per 64 events and one
// per wait instead of one per event (1240 of the waits of the stress trace follow from one another,
// whatever is walked at a time).  Bound by the latency of those steps.  Stress trace, 55 476 events with about
// 1400 waits: 14.4 ms with one event after the other; 4.2 with a scan of the steps x -> max(x + a, b) per channel
// in 64-bit integers and three dependent trips to memory before every 64 events; 2.6 with the lanes in the order of
// their channels, running maxima in doubles - one for both channels of a direction - and every trip a
// stage ahead.
// A result needed by a later event of the same 64, or of the next, is passed on through a
// register; older ones come from the result array.

#include "g10_plan_defs.h"

#include <stdlib.h>
#include <string.h>

using namespace g10;

namespace {

// Kinds of events in the order of one point; eviction and prefetch per destination (their channels are independent, so
// the order between the two does not matter).
enum { EV_OUT = 0, EV_IN = 2, EV_USE = 4, EV_NONE = 5, EV_BITS = 3 };

struct ReplayStats {
  u64 iter_ns, stall_ns, n_stalled, pad;
  u64 bytes[2], busy_out[2], busy_in[2];
};

// Keys of the events of migration i in both iterations: {point, kind | migration, iteration}; ~0 for events beyond the
// second iteration.  The events are written in the order of migration and iteration, and the sort is stable: so it goes by
// point and kind alone (for the migrations of the encoder trace two digits; with the low bits four, and three of them for
// the kind in three bits where two had done).
__global__ __launch_bounds__(G10_BLOCK) void k_rp_events(const g10_migration* __restrict__ rec, const uint2* __restrict__ rec_ab,
                                                        const u32* __restrict__ gained, u32 n, u32 K, u32 rbits,
                                                        u64* __restrict__ keys, ReplayStats* __restrict__ st) {
  __shared__ u64 tmp[G10_WAVES + 1];
  const u32 i = blockIdx.x * G10_BLOCK + threadIdx.x;
  u64 by[2] = {0, 0}, bo[2] = {0, 0}, bi[2] = {0, 0};
  if (i < n) {
    const g10_migration m = rec[i];
    const u32 b2 = rec_ab[i].y, R2 = m.next_use + (m.wraps ? K : 0u);
    const u32 kind[3] = {EV_OUT + m.dest, EV_IN + m.dest, EV_USE}, issue = b2 + 1 - (gained ? gained[i] : 0u);
    for (u32 c = 0; c < 2; ++c) {
      const u32 pt[3] = {m.evict_after + 1 + c * K, issue + c * K, R2 + c * K};
      for (u32 t = 0; t < 3; ++t)
        keys[(u64)6 * i + 3 * c + t] = pt[t] < 2 * K ? (((((u64)pt[t] << EV_BITS) | kind[t]) << (rbits + 1)) | ((u64)i << 1) | c) : NONE64;
    }
    by[m.dest] = m.size_bytes; bo[m.dest] = m.t_out_ns; bi[m.dest] = m.t_in_ns;
  }
  for (u32 d = 0; d < 2; ++d) {                       // traffic and channel time per destination
    const u64 a = block_sum(by[d], tmp), b = block_sum(bo[d], tmp), c = block_sum(bi[d], tmp);
    if (threadIdx.x == 0) {
      if (a) atomicAdd((unsigned long long*)&st->bytes[d], (unsigned long long)a);
      if (b) atomicAdd((unsigned long long*)&st->busy_out[d], (unsigned long long)b);
      if (c) atomicAdd((unsigned long long*)&st->busy_in[d], (unsigned long long)c);
    }
  }
}

// where the eviction and the prefetch of every (iteration, migration) stand in the sorted order
__global__ __launch_bounds__(G10_BLOCK) void k_rp_index(const u64* __restrict__ sorted, u32 ne, u32 n, u32 rbits,
                                                       u32* __restrict__ pos_of) {
  const u32 p = blockIdx.x * G10_BLOCK + threadIdx.x;
  if (p >= ne) return;
  const u64 k = sorted[p];
  if (k == NONE64) return;
  const u32 c = (u32)(k & 1ull), i = (u32)((k >> 1) & ((1ull << rbits) - 1ull)), t = (u32)((k >> (rbits + 1)) & ((1u << EV_BITS) - 1u));
  if (t != EV_USE) pos_of[(u64)((t >= EV_IN ? 2u : 0u) + c) * n + i] = p;
}

__device__ __forceinline__ u64 lane_get(u64 v, u32 l) {
  const u32 lo = (u32)__builtin_amdgcn_readlane((int)(u32)v, (int)l), hi = (u32)__builtin_amdgcn_readlane((int)(u32)(v >> 32), (int)l);
  return ((u64)hi << 32) | lo;
}
// lane l's v for every lane's own l (all lanes of the wavefront take part)
__device__ __forceinline__ u64 lane_any(u64 v, u32 l) {
  const u32 lo = (u32)__shfl((int)(u32)v, (int)l), hi = (u32)__shfl((int)(u32)(v >> 32), (int)l);
  return ((u64)hi << 32) | lo;
}

// One step of a channel queue, x -> max(x + a, b): the time the channel is free again after a transfer of
// length a that cannot end before b.  (0, 0) is the identity on times.
struct Queue {
  u64 a, b;
};
__device__ __forceinline__ Queue then(const Queue& f, const Queue& g) {      // f first
  const u64 x = f.b + g.a;
  return Queue{f.a + g.a, x > g.b ? x : g.b};
}
template <int CTRL, int ROW_MASK, int BANK_MASK>
__device__ __forceinline__ Queue queue_from(const Queue& f) {
  return Queue{dpp_move<CTRL, ROW_MASK, BANK_MASK>((u64)0, f.a), dpp_move<CTRL, ROW_MASK, BANK_MASK>((u64)0, f.b)};
}
// the steps of lanes 0 .. l one after the other, for every lane l
__device__ __forceinline__ Queue queue_scan(Queue f) {
  f = then(queue_from<0x111, 0xf, 0xf>(f), f);                 // row_shr:1, 2, 4, 8
  f = then(queue_from<0x112, 0xf, 0xf>(f), f);
  f = then(queue_from<0x114, 0xf, 0xf>(f), f);
  f = then(queue_from<0x118, 0xf, 0xf>(f), f);
  f = then(queue_from<0x142, 0xa, 0xf>(f), f);                 // lane 15 of rows 0 and 2 into rows 1 and 3
  f = then(queue_from<0x143, 0xc, 0xf>(f), f);                 // lane 31 into rows 2 and 3
  return f;
}

// The walk in whole numbers, for times over REPLAY_EXACT: an event per lane in the order of the events, a scan of the
// steps x -> max(x + a, b) per channel.
__global__ __launch_bounds__(G10_WAVE) void k_replay_long(const u64* __restrict__ sorted, u32 ne, const g10_migration* __restrict__ rec,
                                                    u32 n, u32 rbits, const u32* __restrict__ pos_of,
                                                    const u64* __restrict__ start, u32 K, u64 T, u64* __restrict__ res,
                                                    u64* __restrict__ late, ReplayStats* __restrict__ st) {
  const u32 lane = threadIdx.x;
  // the state of the walk; the same in every lane
  u64 delta = 0;                        // end of the previous kernel minus its end without any stall
  u64 delta_first = 0;                  // the same when the second iteration begins
  bool second = false;
  u64 ch_out[2] = {0, 0}, ch_in[2] = {0, 0};               // when each channel is free again
  u64 stall = 0, n_stalled = 0;
  u32 use_pt = NONE32, stalled_pt = NONE32;
  u64 delta_pt = 0;                     // delta when the uses of the current point began
  // One event per lane, gathered one step ahead of the walk: key, record fields, the point's time
  // without stalls, and the result the event waits for.  While batch b is walked the results of
  // the batches before b are in memory, so an older one is loaded here; one of batch b or of the
  // batch gathered itself is noted by its lane and read from a register during the walk.
  struct Ev { u64 tau, sp, pval; u32 type, i, pt, dest, pin, psrc; bool valid; };   // psrc 0: pval; 1: this batch; 2: the batch before
  auto gather = [&](u32 base, u32 done) -> Ev {           // results of positions < done are in memory
    Ev v;
    v.tau = 0; v.sp = 0; v.pval = 0; v.type = 3; v.i = 0; v.pt = 0; v.dest = 0; v.pin = 0; v.psrc = 0;
    const u32 p = base + lane;
    const u64 k = p < ne ? sorted[p] : NONE64;
    v.valid = k != NONE64;
    if (v.valid) {
      const u32 c = (u32)(k & 1ull);
      v.i = (u32)((k >> 1) & ((1ull << rbits) - 1ull));
      const u64 q = k >> (rbits + 1);
      const u32 kind = (u32)(q & ((1u << EV_BITS) - 1u));
      v.type = kind >= EV_USE ? 2u : kind >= EV_IN ? 1u : 0u; v.pt = (u32)(q >> EV_BITS);
      const g10_migration m = rec[v.i];
      v.dest = m.dest;
      v.tau = v.type == 0u ? m.t_out_ns : m.t_in_ns;
      v.sp = v.pt < K ? start[v.pt] : start[v.pt - K] + T;     // end of kernel pt - 1 without any stall
      if (v.type != 0u) {                                 // its eviction / its prefetch
        const u32 pp = pos_of[(u64)((v.type - 1) * 2 + c) * n + v.i];
        if (pp >= base) { v.psrc = 1; v.pin = pp - base; }
        else if (pp >= done) { v.psrc = 2; v.pin = pp - done; }
        else v.pval = res[pp];
      }
    }
    return v;
  };
  Ev nxt = gather(0, 0);
  u64 resv_prev = 0;                    // results of the batch before, one per lane
  for (u32 base = 0; base < ne; base += G10_WAVE) {
    const Ev cur = nxt;
    const u32 p = base + lane;
    const bool valid = cur.valid;
    const u32 type = cur.type, i = cur.i, pt = cur.pt, dest = cur.dest;
    const u64 tau = cur.tau, sp = cur.sp;
    if (base + G10_WAVE < ne) nxt = gather(base + G10_WAVE, base);   // in flight during the walk
    const u32 cnt = (u32)__popcll(__ballot(valid));             // the valid events come first
    u64 resv = 0, latev = 0;
    // ---- the walk: as many events at a time as no stall separates --------------------------
    // `delta` changes only where a kernel waits.  Up to the next wait every channel is a queue whose
    // requests are known, so the completion times of all remaining events come from one scan per
    // channel; the first use that finds its prefetch late ends the step: what lies behind it is
    // worked out again with the new delta.
    const u64 from_prev = lane_any(resv_prev, cur.pin);                     // (every lane takes part: a lane read must be active)
    const u64 pv = cur.psrc == 2 ? from_prev : cur.pval;                    // what the event waits for, if it is older than these 64
    const bool here = valid && cur.psrc == 1;                               // (else it is lane pin's result)
    const u64 use_m = __ballot(valid && type == 2u), second_m = __ballot(valid && pt >= K);
    const u64 out_m[2] = {__ballot(valid && type == 0u && dest == 0), __ballot(valid && type == 0u && dest == 1)};
    const u64 in_m[2] = {__ballot(valid && type == 1u && dest == 0), __ballot(valid && type == 1u && dest == 1)};
    u32 from = 0;
    while (from < cnt) {
      const bool open = valid && lane >= from;
      const u64 open_m = ~0ull << from;
      const u64 free_at = sp + delta;                                       // end of the previous kernel
      u64 t = resv;
#pragma unroll
      for (u32 d = 0; d < 2; ++d) {                                         // evictions
        if (!(out_m[d] & open_m)) continue;
        const bool mine = open && type == 0u && dest == d;
        const Queue q = queue_scan(Queue{mine ? tau : 0ull, mine ? free_at + tau : 0ull});
        const u64 x = ch_out[d] + q.a, y = x > q.b ? x : q.b;
        if (mine) t = y;
      }
      u64 w = pv;
      const u64 from_out = lane_any(t, cur.pin);
      if (here && type == 1u) w = from_out;
#pragma unroll
      for (u32 d = 0; d < 2; ++d) {                                         // prefetches, not before their evictions
        if (!(in_m[d] & open_m)) continue;
        const bool mine = open && type == 1u && dest == d;
        const u64 ready = free_at > w ? free_at : w;
        const Queue q = queue_scan(Queue{mine ? tau : 0ull, mine ? ready + tau : 0ull});
        const u64 x = ch_in[d] + q.a, y = x > q.b ? x : q.b;
        if (mine) t = y;
      }
      const u64 from_in = lane_any(t, cur.pin);
      if (here && type == 2u) w = from_in;
      const bool is_use = open && type == 2u;
      const u64 waits = __ballot(is_use && w > free_at);
      const u32 f = waits ? (u32)__builtin_ctzll(waits) : cnt - 1;          // the step ends with event f
      const u64 step_m = open_m & (f >= 63u ? ~0ull : (1ull << (f + 1)) - 1ull);
      if (!second && (second_m & step_m)) { second = true; delta_first = delta; }
      if ((step_m >> lane) & 1ull) {
        resv = t;
        // (the previous kernel's end, before any wait of this one)
        const u64 prev_end = sp + (pt == use_pt ? delta_pt : delta);
        if (is_use && pt >= K && w > prev_end) latev = w - prev_end;
      }
#pragma unroll
      for (u32 d = 0; d < 2; ++d) {                                         // the channels after event f
        const u64 om = out_m[d] & step_m, im = in_m[d] & step_m;
        if (om) ch_out[d] = lane_get(t, 63u - (u32)__builtin_clzll(om));
        if (im) ch_in[d] = lane_get(t, 63u - (u32)__builtin_clzll(im));
      }
      const u64 um = use_m & step_m;
      if (um) {
        const u32 upt = (u32)__builtin_amdgcn_readlane((int)pt, (int)(63u - (u32)__builtin_clzll(um)));
        if (upt != use_pt) { use_pt = upt; delta_pt = delta; }
      }
      if (waits) {                                              // the kernel waits for this prefetch
        const u64 pf = lane_get(w, f), spf = lane_get(sp, f);
        if (use_pt >= K) {
          stall += pf - (spf + delta);
          if (stalled_pt != use_pt) { stalled_pt = use_pt; n_stalled += 1; }
        }
        delta = pf - spf;
      }
      from = f + 1;
    }
    // ---- results out ---------------------------------------------------------------------
    if (valid && type != 2u) res[p] = resv;
    if (valid && type == 2u && pt >= K) late[i] = latev;
    resv_prev = resv;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);                              // the next gather may read what was just written
    if (cnt < G10_WAVE) break;
  }
  if (!second) delta_first = delta;
  if (lane == 0) {
    st->iter_ns = T + delta - delta_first;
    st->stall_ns = stall;
    st->n_stalled = n_stalled;
  }
}

// ---------------------------------------------------------------------------
// The walk.  Times in doubles, exact below 2^53: no time of the walk exceeds two iterations and every transfer one after
// the other, 2 T + 8 T of the plan (a channel's transfers fit the iteration they were planned for).
// ---------------------------------------------------------------------------
constexpr u64 REPLAY_EXACT = 1ull << 48;          // bound of 2 T + 8 T (with SEGMENT between the channels of a scan)
constexpr double SEGMENT = 0x1p50;

struct OpAddF {
  static __device__ __forceinline__ u64 f(u64 a, u64 b) {
    return (u64)__double_as_longlong(__longlong_as_double((long long)a) + __longlong_as_double((long long)b));
  }
};
// Running maximum of values that are not negative: lanes without a source give 0, and a maximum may meet a value twice,
// so the steps across rows need no mask and no identity of their own.
template <int CTRL>
__device__ __forceinline__ double max_from(double v) {
  const u64 x = (u64)__double_as_longlong(v);
  const u32 lo = (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)x, CTRL, 0xf, 0xf, true);
  const u32 hi = (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)(x >> 32), CTRL, 0xf, 0xf, true);
  return fmax(v, __longlong_as_double((long long)(((u64)hi << 32) | lo)));
}
__device__ __forceinline__ double scan_max(double v) {
  v = max_from<0x111>(v);                                        // row_shr:1, 2, 4, 8
  v = max_from<0x112>(v);
  v = max_from<0x114>(v);
  v = max_from<0x118>(v);
  v = max_from<0x142>(v);                                        // lane 15 of a row into the next row
  return max_from<0x143>(v);                                     // lane 31 into rows 2 and 3
}
__device__ __forceinline__ double scan_sum(double v) { return __longlong_as_double((long long)wave_scan_dpp<OpAddF>((u64)__double_as_longlong(v), (u64)0)); }
__device__ __forceinline__ double lane_getf(double v, u32 l) { return __longlong_as_double((long long)lane_get((u64)__double_as_longlong(v), l)); }
__device__ __forceinline__ double lane_anyf(double v, u32 l) { return __longlong_as_double((long long)lane_any((u64)__double_as_longlong(v), l)); }
__device__ __forceinline__ u32 to_lane(u32 v, u32 l) { return (u32)__builtin_amdgcn_ds_permute((int)(l << 2), (int)v); }   // (l: another one for every lane)
__device__ __forceinline__ double whole(u64 x) { return __fma_rn((double)(u32)(x >> 32), 4294967296.0, (double)(u32)x); }

__global__ __launch_bounds__(G10_WAVE) void k_replay(const u64* __restrict__ sorted, u32 ne, const g10_migration* __restrict__ rec,
                                                    u32 n, u32 rbits, const u32* __restrict__ pos_of,
                                                    const u64* __restrict__ start, u32 K, u64 T, u64* __restrict__ res,
                                                    u64* __restrict__ late, ReplayStats* __restrict__ st) {
  const u32 lane = threadIdx.x;
  const u64 below = (1ull << lane) - 1ull;
  // the state of the walk; the same in every lane
  double delta = 0;                     // end of the previous kernel minus its end without any stall
  double delta_first = 0;               // the same when the second iteration begins
  bool second = false;
  double free0 = 0, free1 = 0, free2 = 0, free3 = 0;       // when each channel is free again (out 0, 1, in 0, 1)
  double stall = 0;
  u64 n_stalled = 0;
  u32 use_pt = NONE32, stalled_pt = NONE32;
  double delta_pt = 0;                  // delta when the uses of the current point began

  // 64 events at a time, one per lane, the lanes in the order of their kinds: each channel's requests lie side by side, in
  // order.  They are fetched in stages, a stage a step of 64 ahead of the next, so that no trip to memory is waited for:
  // the keys; record, time of the point and where the event's predecessor stands; the predecessor's result.
  struct Keys { u64 k; u32 place, pos; };                  // place: the lane that the event of this position goes to; pos: the position of this lane's event
  // (loaded words stay as they come until a later stage uses them: a conversion beside the load would wait for it)
  struct Loads { u64 tau, sp; u32 kind, i, pt, pos, place, pred; };
  struct Ev { Loads l; u64 pval; u32 src, psrc; };         // psrc 0: pval; 1: lane src of these 64; 2: of the 64 before
  auto load_key = [&](u64 at) -> u64 { return at + lane < ne ? sorted[at + lane] : NONE64; };
  auto spread = [&](u64 k) -> Keys {
    const u32 kind = k == NONE64 ? (u32)EV_NONE : (u32)(k >> (rbits + 1)) & ((1u << EV_BITS) - 1u);
    Keys r;
    u32 at = 0;
    r.place = 0;
#pragma unroll
    for (u32 c = 0; c <= EV_NONE; ++c) {
      const u64 m = __ballot(kind == c);
      if (kind == c) r.place = at + (u32)__popcll(m & below);
      at += (u32)__popcll(m);
    }
    r.k = ((u64)to_lane((u32)(k >> 32), r.place) << 32) | to_lane((u32)k, r.place);
    r.pos = to_lane(lane, r.place);
    return r;
  };
  auto load_ops = [&](const Keys& q) -> Loads {
    Loads v;
    const bool valid = q.k != NONE64;
    const u64 x = q.k >> (rbits + 1);
    v.i = valid ? (u32)((q.k >> 1) & ((1ull << rbits) - 1ull)) : 0u;
    v.kind = valid ? (u32)(x & ((1u << EV_BITS) - 1u)) : (u32)EV_NONE;
    v.pt = valid ? (u32)(x >> EV_BITS) : 0u;
    v.pos = q.pos; v.place = q.place;
    v.tau = *(v.kind < EV_IN ? &rec[v.i].t_out_ns : &rec[v.i].t_in_ns);
    v.sp = start[v.pt < K ? v.pt : v.pt - K];
    v.pred = pos_of[(u64)((v.kind == EV_USE ? 2u : 0u) + (u32)(q.k & 1ull)) * n + v.i];   // its eviction / its prefetch (an eviction: not used)
    return v;
  };
  // (the events from `base` on; those before `done` have their results in memory, the ones between lie where place_prev says)
  auto load_pred = [&](const Loads& l, u32 base, u32 done, u32 place_prev) -> Ev {
    Ev v;
    v.l = l;
    const bool has = l.kind >= EV_IN && l.kind <= EV_USE;
    const u32 here = (u32)__shfl((int)l.place, (int)((l.pred - base) & 63u)), there = (u32)__shfl((int)place_prev, (int)((l.pred - done) & 63u));
    v.psrc = !has ? 0u : l.pred >= base ? 1u : l.pred >= done ? 2u : 0u;
    v.src = v.psrc == 1u ? here : there;
    v.pval = res[has && v.psrc == 0u ? l.pred : 0u];       // (the others: not used)
    return v;
  };
  Keys kq = spread(load_key(0));
  Loads lq = load_ops(kq);
  kq = spread(load_key(G10_WAVE));
  u64 kraw = load_key(2 * G10_WAVE);
  Ev nxt = load_pred(lq, 0, 0, 0);
  lq = load_ops(kq);
  double t_prev = 0;                    // results of the 64 before, one per lane
  for (u32 base = 0; base < ne; base += G10_WAVE) {
    const Ev cur = nxt;
    const u32 kind = cur.l.kind, pt = cur.l.pt, pos = cur.l.pos;
    const double tau = kind >= EV_USE ? 0.0 : whole(cur.l.tau), sp = whole(cur.l.sp + (pt < K ? 0ull : T));     // (sp: end of kernel pt - 1 without any stall)
    nxt = load_pred(lq, base + G10_WAVE, base, cur.l.place);
    lq = load_ops(spread(kraw));
    kraw = load_key((u64)base + 3 * G10_WAVE);
    const bool is_out = kind < EV_IN, is_in = kind >= EV_IN && kind < EV_USE, is_use = kind == EV_USE;
    const u64 use_m = __ballot(is_use), valid_m = __ballot(kind != EV_NONE);
    const u32 cnt = (u32)__popcll(valid_m);                     // the valid events come first
    const u64 out1_m = __ballot(kind == EV_OUT + 1), in0_m = __ballot(kind == EV_IN), in1_m = __ballot(kind == EV_IN + 1), out0_m = __ballot(kind == EV_OUT);
    // A channel that is free at x serves requests that are ready at r_1, r_2, .. and take tau_1, tau_2, ..: the k-th is done
    // at A_k + max(x, r_j - A_(j-1) for j <= k), A the sums of tau.  Those do not change while the delay does, so a step
    // of the walk is a running maximum for the evictions and one for the prefetches, both destinations in one
    // (SEGMENT apart).  Settled requests keep their maximum.
    const double sum = scan_sum(tau);
    const double before1 = out0_m ? lane_getf(sum, 63u - (u32)__builtin_clzll(out0_m)) : 0.0;
    const u64 o01 = out0_m | out1_m, in01 = in0_m | in1_m, o012 = o01 | in0_m;
    const double before2 = o01 ? lane_getf(sum, 63u - (u32)__builtin_clzll(o01)) : 0.0, before3 = o012 ? lane_getf(sum, 63u - (u32)__builtin_clzll(o012)) : 0.0;
    const double A = sum - (kind == EV_OUT ? 0.0 : kind == EV_OUT + 1 ? before1 : kind == EV_IN ? before2 : before3);
    const double free_c = kind == EV_OUT ? free0 : kind == EV_OUT + 1 ? free1 : kind == EV_IN ? free2 : free3;
    const double seg = (kind & 1u) ? 2.0 * SEGMENT : SEGMENT;    // (a request's ready time less the sums before it is above -SEGMENT)
    const double from_prev = lane_anyf(t_prev, cur.src);
    const bool here = cur.psrc == 1;
    const double pv = cur.psrc == 2 ? from_prev : whole(cur.pval);      // what the event waits for, if it is older than these 64
    const bool any_here_in = __any(here && is_in), any_here_use = __any(here && is_use);
    double M = 0, t = 0, latev = 0;                              // the request's maximum (`seg` up) and completion time
    u32 from = 0;                                                // events before this position are settled
    while (from < cnt) {
      const bool open = pos >= from;
      const double free_at = sp + delta;                         // end of the previous kernel
      const u64 open_m = __ballot(open);
      if (o01 & open_m) {                                        // evictions
        const double m = scan_max(is_out ? (open ? free_at + (seg - (A - tau)) : M) : 0.0);
        if (is_out) { M = m; const double y = m - seg; t = A + (y > free_c ? y : free_c); }
      }
      double w = pv;
      if (any_here_in) { const double x = lane_anyf(t, cur.src); if (here && is_in) w = x; }
      if (in01 & open_m) {                                       // prefetches, not before their evictions
        const double ready = free_at > w ? free_at : w;
        const double m = scan_max(is_in ? (open ? ready + (seg - (A - tau)) : M) : 0.0);
        if (is_in) { M = m; const double y = m - seg; t = A + (y > free_c ? y : free_c); }
      }
      if (any_here_use) { const double x = lane_anyf(t, cur.src); if (here && is_use) w = x; }
      const u64 waits = __ballot(is_use && open && w > free_at);
      const u32 fl = waits ? (u32)__builtin_ctzll(waits) : 0u;   // (the uses lie in their order)
      const u32 f = waits ? (u32)__builtin_amdgcn_readlane((int)pos, (int)fl) : cnt - 1;       // the step ends with event f
      const bool in_step = open && pos <= f && kind != EV_NONE;
      if (!second && __any(in_step && pt >= K)) { second = true; delta_first = delta; }
      if (is_use && in_step && pt >= K) {                        // lateness: beyond the previous kernel's end, before any wait of this one
        const double prev_end = sp + (pt == use_pt ? delta_pt : delta);
        latev = w > prev_end ? w - prev_end : 0.0;
      }
      const u64 um = use_m & __ballot(in_step);
      if (um) {
        const u32 upt = (u32)__builtin_amdgcn_readlane((int)pt, (int)(63u - (u32)__builtin_clzll(um)));
        if (upt != use_pt) { use_pt = upt; delta_pt = delta; }
      }
      if (waits) {                                               // the kernel waits for this prefetch
        const double pf = lane_getf(w, fl), spf = lane_getf(sp, fl);
        if (use_pt >= K) {
          stall += pf - (spf + delta);
          if (stalled_pt != use_pt) { stalled_pt = use_pt; n_stalled += 1; }
        }
        delta = pf - spf;
      }
      from = f + 1;
    }
    // ---- results out ---------------------------------------------------------------------
    if (out0_m) free0 = lane_getf(t, 63u - (u32)__builtin_clzll(out0_m));
    if (out1_m) free1 = lane_getf(t, 63u - (u32)__builtin_clzll(out1_m));
    if (in0_m) free2 = lane_getf(t, 63u - (u32)__builtin_clzll(in0_m));
    if (in1_m) free3 = lane_getf(t, 63u - (u32)__builtin_clzll(in1_m));
    if (is_out || is_in) res[base + pos] = (u64)t;
    if (is_use && pt >= K) late[cur.l.i] = (u64)latev;
    t_prev = t;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // the next loads find what was just written (in order)
    if (cnt < G10_WAVE) break;
  }
  if (!second) delta_first = delta;
  if (lane == 0) {
    st->iter_ns = T + (u64)(delta - delta_first);
    st->stall_ns = (u64)stall;
    st->n_stalled = n_stalled;
  }
}

}  // namespace

void replay_free(PlanWork* w) {
  mem_dev_free(w->rp_arena);
  w->rp_arena = nullptr; w->rp_cap = 0;
  free(w->h_rp_late); w->h_rp_late = nullptr;
}

// Do the keys of n migrations on K slots fit 64 bits?  (They do not from 2^28 migrations and 2^29 slots on: with its
// timelines and candidates such a plan takes more memory than a GPU has.)
bool replay_key_fits(u32 K, u32 n) { return bits_for(2ull * K) + EV_BITS + bits_for(n ? n - 1 : 0) + 1 <= 64; }

int replay_run(g10_plan_s* h, const u64* dur_ns, u32 eager, g10_replay_result* out) {
  PlanWork* w = h->work;
  if (!w || !w->planned) return G10_EINVAL;
  if (eager && !w->prefetched) return G10_EINVAL;
  hipStream_t s = h->stream;
  const u32 K = h->K, n = (u32)w->plan_n_mig;
  const u64 ne = (u64)6 * n;
  if (ne >= (1ull << 32) || !replay_key_fits(K, n)) return G10_EINVAL;
  // workspace of its own, sized for this plan's migrations
  if (!w->rp_arena || w->rp_cap < n) {
    G10_HIP(hipStreamSynchronize(s));
    replay_free(w);
    const u64 cap = n ? n : 1, ce = 6 * cap;
    const u64 he = radix_hist_elems(ce);
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off += (bytes + 255) & ~(size_t)255; return o; };
    const size_t o_keys = take(ce * 8), o_alt = take(ce * 8), o_res = take(ce * 8), o_late = take(cap * 8), o_pos = take(4 * cap * 4),
                 o_hist = take(he * 4), o_st = take(sizeof(ReplayStats)), o_dur = take((u64)K * 8),
                 o_start = take(((u64)K + 1) * 8), o_ts = take(scan_scratch_elems(K) * 8), o_tst = take(128);
    void* q = nullptr;
    G10_TRY(mem_dev_alloc(&q, off));
    char* b = (char*)q;
    w->rp_arena = q; w->rp_cap = (u32)cap;
    w->rp_keys = (u64*)(b + o_keys); w->rp_alt = (u64*)(b + o_alt); w->rp_res = (u64*)(b + o_res); w->rp_late = (u64*)(b + o_late);
    w->rp_pos = (u32*)(b + o_pos); w->rp_hist = (u32*)(b + o_hist); w->rp_stats = (void*)(b + o_st);
    w->rp_dur = (u64*)(b + o_dur); w->rp_start = (u64*)(b + o_start); w->rp_tscr = (u64*)(b + o_ts); w->rp_tstats = (void*)(b + o_tst);
    w->h_rp_late = (u64*)malloc(cap * 8);
    if (!w->h_rp_late) { replay_free(w); return G10_ENOMEM; }      // both or none: the next call must find the same state as the first
  }
  // the durations to replay with: the given ones, else the ones the plan was made for
  const u64* start = w->start;
  u64 T = w->T;
  if (dur_ns) {
    u64 check[16];
    G10_TRY(slot_times_begin(dur_ns, K, w->rp_dur, w->rp_start, w->rp_tscr, w->rp_tstats, check, s));
    G10_HIP(hipStreamSynchronize(s));
    G10_TRY(slot_times_end(check, &T));
    start = w->rp_start;
  }
  G10_HIP(hipEventRecord(w->ev[0], s));
  ReplayStats* st = (ReplayStats*)w->rp_stats;
  G10_HIP(hipMemsetAsync(st, 0, sizeof(ReplayStats), s));
  if (n) G10_HIP(hipMemsetAsync(w->rp_late, 0, (u64)n * 8, s));
  const u32 rbits = bits_for(n ? n - 1 : 0);
  u64 *keys = w->rp_keys, *alt = w->rp_alt;
  if (n) {
    hipLaunchKernelGGL(k_rp_events, dim3((n + G10_BLOCK - 1) / G10_BLOCK), dim3(G10_BLOCK), 0, s, (const g10_migration*)w->records,
                       (const uint2*)w->rec_ab, eager ? (const u32*)w->pf_gained : (const u32*)nullptr, n, K, rbits, keys, st);
    G10_HIP(hipGetLastError());
    G10_TRY(radix_sort_u64(&keys, &alt, ne, rbits + 1 + EV_BITS + bits_for(2ull * K), w->rp_hist, s, rbits + 1));
    hipLaunchKernelGGL(k_rp_index, dim3((u32)((ne + G10_BLOCK - 1) / G10_BLOCK)), dim3(G10_BLOCK), 0, s, (const u64*)keys, (u32)ne, n, rbits,
                       w->rp_pos);
    G10_HIP(hipGetLastError());
  }
  // (a channel's transfers fit the iteration that they were planned for, w->T; each is made twice)
  const bool exact = T < REPLAY_EXACT / 10 && w->T < REPLAY_EXACT / 10;
  hipLaunchKernelGGL((exact ? k_replay : k_replay_long), dim3(1), dim3(G10_WAVE), 0, s, (const u64*)keys, (u32)ne, (const g10_migration*)w->records, n, rbits,
                     (const u32*)w->rp_pos, start, K, T, w->rp_res, w->rp_late, st);
  G10_HIP(hipGetLastError());
  ReplayStats hs;
  G10_HIP(hipMemcpyAsync(&hs, st, sizeof hs, hipMemcpyDeviceToHost, s));
  if (n) G10_HIP(hipMemcpyAsync(w->h_rp_late, w->rp_late, (u64)n * 8, hipMemcpyDeviceToHost, s));
  G10_HIP(hipEventRecord(w->ev[1], s));
  G10_HIP(hipStreamSynchronize(s));
  float ms = 0.f;
  G10_HIP(hipEventElapsedTime(&ms, w->ev[0], w->ev[1]));
  memset(out, 0, sizeof *out);
  out->iter_ns = hs.iter_ns; out->planned_ns = T; out->stall_ns = hs.stall_ns; out->n_stalled = hs.n_stalled;
  for (int d = 0; d < 2; ++d) { out->bytes[d] = hs.bytes[d]; out->busy_out_ns[d] = hs.busy_out[d]; out->busy_in_ns[d] = hs.busy_in[d]; }
  out->n_migrations = n; out->late_ns = w->h_rp_late; out->ms = ms;
  return G10_OK;
}
