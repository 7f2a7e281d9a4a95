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
// whatever is walked at a time).  Bound by the latency of those steps, which one wavefront issues an instruction after the
// other.  Stress trace, 55 476 events with about 3000 waits in both iterations: 14.4 ms with one event after the other; 4.2
// with a scan of the steps x -> max(x + a, b) per channel in 64-bit integers and three dependent trips to memory before
// every 64 events; 2.4 with the lanes in the order of their channels, running maxima in doubles and every trip a stage ahead;
// 1.6 with all that an event needs worked out beforehand, in parallel (k_rp_expand), and loaded four steps ahead; 1.35 with
// one running maximum for all four channels and a third of the instructions per wait (540 cycles, and 1080 per 64 events).
// A result needed by a later event of the same 64 is passed on through a register, of the next 192 through LDS; older ones
// come from the result array.

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

// The lanes of 64 neighbouring events in the order of their kinds: the lane that this lane's event goes to.  Each channel's
// requests lie side by side then, in order, and the uses behind them.
__device__ __forceinline__ u32 place_of(u32 kind) {
  const u64 below = (1ull << lane_id()) - 1ull;
  u32 at = 0, place = 0;
#pragma unroll
  for (u32 c = 0; c <= EV_NONE; ++c) {
    const u64 m = __ballot(kind == c);
    if (kind == c) place = at + (u32)__popcll(m & below);
    at += (u32)__popcll(m);
  }
  return place;
}
__device__ __forceinline__ u32 kind_of(u64 k, u32 rbits) { return k == NONE64 ? (u32)EV_NONE : (u32)(k >> (rbits + 1)) & ((1u << EV_BITS) - 1u); }

// where the eviction and the prefetch of every (iteration, migration) stand in the sorted order (by_lane: the place in their 64)
__global__ __launch_bounds__(G10_BLOCK) void k_rp_index(const u64* __restrict__ sorted, u32 ne, u32 n, u32 rbits, u32 by_lane,
                                                       u32* __restrict__ pos_of) {
  const u32 p = blockIdx.x * G10_BLOCK + threadIdx.x;
  const u64 k = p < ne ? sorted[p] : NONE64;
  const u32 t = kind_of(k, rbits), place = place_of(t);
  if (t >= EV_USE) return;
  const u32 c = (u32)(k & 1ull), i = (u32)((k >> 1) & ((1ull << rbits) - 1ull));
  pos_of[(u64)((t >= EV_IN ? 2u : 0u) + c) * n + i] = by_lane ? (p & ~63u) + place : p;
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
// (no NaN is compared: fmax() would cost an instruction more per operand, in case it were a signalling one)
__device__ __forceinline__ double larger(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
template <int CTRL>
__device__ __forceinline__ double max_from(double v) {
  const u64 x = (u64)__double_as_longlong(v);
  const u32 lo = (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)x, CTRL, 0xf, 0xf, true);
  const u32 hi = (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)(x >> 32), CTRL, 0xf, 0xf, true);
  const double o = __longlong_as_double((long long)(((u64)hi << 32) | lo));
  return larger(v, o);
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
// (at: four times the lane)
__device__ __forceinline__ double lane_at(double v, u32 at) {
  const u64 x = (u64)__double_as_longlong(v);
  const u32 lo = (u32)__builtin_amdgcn_ds_bpermute((int)at, (int)(u32)x), hi = (u32)__builtin_amdgcn_ds_bpermute((int)at, (int)(u32)(x >> 32));
  return __longlong_as_double((long long)(((u64)hi << 32) | lo));
}
__device__ __forceinline__ u32 to_lane(u32 v, u32 l) { return (u32)__builtin_amdgcn_ds_permute((int)(l << 2), (int)v); }   // (l: another one for every lane)
__device__ __forceinline__ double whole(u64 x) { return __fma_rn((double)(u32)(x >> 32), 4294967296.0, (double)(u32)x); }

// What the walk needs of an event, worked out for all events at once, a wavefront per 64 events and in the order of their
// lanes: a walk that gathered keys, records, times and predecessors itself waited for them at every 64.
struct Walk {
  double* sp;        // end of the kernel before the event's point without any stall
  double* A;         // transfer times of its channel's requests among the 64, up to and with this one
  double* off;       // what is added to the time it is ready to find the running maximum: its segment less the requests before it
  uint2* ev;         // W_* below; migration
  u32* pred;         // place of its eviction / its prefetch, NONE32 if it waits for none
};
enum : u32 {         // ev.x: kind in the lowest bits, then
  W_POS = 3,         // where the event stands among the 64 (6 bits)
  W_FIRST = 9,       // a use: the lane of the first use at its point among the 64 (6 bits)
  W_CONT = 1u << 15, // ... and that point has uses among the 64 before
  W_SECOND = 1u << 16              // in the second iteration
};
constexpr u32 WALK_STAGES = 4;                    // steps of 64 between an event's loads and its use
constexpr u32 WALK_PAD = 2 * WALK_STAGES * 64;    // events (of no kind) behind the last: what is loaded ahead of the walk
u64 walk_events(u64 ne) { return (ne + 64 * WALK_STAGES - 1) / (64 * WALK_STAGES) * (64 * WALK_STAGES) + WALK_PAD; }

__global__ __launch_bounds__(G10_BLOCK) void k_rp_expand(const u64* __restrict__ sorted, u32 ne, u32 np, const g10_migration* __restrict__ rec, u32 n,
                                                        u32 rbits, const u32* __restrict__ pos_of, const u64* __restrict__ start, u32 K, u64 T, Walk w) {
  const u32 p = blockIdx.x * G10_BLOCK + threadIdx.x, lane = lane_id(), base = p & ~63u;
  if (base >= np) return;
  const u64 k0 = p < ne ? sorted[p] : NONE64;
  const u32 place = place_of(kind_of(k0, rbits));
  const u64 k = ((u64)to_lane((u32)(k0 >> 32), place) << 32) | to_lane((u32)k0, place);
  const u32 pos = to_lane(lane, place), kind = kind_of(k, rbits);
  const bool valid = kind != EV_NONE;
  const u32 i = valid ? (u32)((k >> 1) & ((1ull << rbits) - 1ull)) : 0u, pt = valid ? (u32)(k >> (rbits + 1 + EV_BITS)) : 0u;
  double tau = 0, sp = 0;
  u32 pred = NONE32;
  if (valid) {
    if (kind < EV_USE) tau = whole(kind < EV_IN ? rec[i].t_out_ns : rec[i].t_in_ns);
    sp = whole(pt < K ? start[pt] : start[pt - K] + T);
    if (kind >= EV_IN) pred = pos_of[(u64)((kind == EV_USE ? 2u : 0u) + (u32)(k & 1ull)) * n + i];
  }
  // sums of the transfer times per channel
  const double sum = scan_sum(tau);
  double before = 0;
#pragma unroll
  for (u32 c = EV_OUT; c < EV_USE; ++c) {
    const u64 m = __ballot(kind == c);
    const double x = m ? lane_getf(sum - tau, (u32)__builtin_ctzll(m)) : 0.0;
    if (kind == c) before = x;
  }
  const double A = sum - before;
  // the uses by point: they lie in the order of their points
  const u64 use_m = __ballot(kind == EV_USE);
  const u32 pt_left = (u32)__shfl_up((int)pt, 1);
  const u64 heads = __ballot(kind == EV_USE && (!((use_m << 1) >> lane & 1ull) || pt_left != pt));
  const u64 mine = heads & (((1ull << lane) - 1ull) | (1ull << lane));
  const u32 first = kind == EV_USE ? 63u - (u32)__builtin_clzll(mine) : 0u;
  // (uses at one point are neighbours in the sorted order: the point goes on if the event before these 64 is one of its uses)
  bool cont = false;
  if (base && use_m) {
    const u64 kp = sorted[base - 1];
    cont = kind == EV_USE && first == (u32)__builtin_ctzll(use_m) && kind_of(kp, rbits) == EV_USE && (u32)(kp >> (rbits + 1 + EV_BITS)) == pt;
  }
  w.sp[p] = sp; w.A[p] = A; w.off[p] = (double)(kind + 1u) * SEGMENT - (A - tau);
  w.ev[p] = make_uint2(kind | (pos << W_POS) | (first << W_FIRST) | (cont ? W_CONT : 0u) | (pt >= K ? W_SECOND : 0u), i);
  w.pred[p] = pred;
}

__global__ __launch_bounds__(G10_WAVE) void k_replay(Walk w, u32 steps, u64 T, double* __restrict__ res, u64* __restrict__ late,
                                                    ReplayStats* __restrict__ st) {
  // results of the last steps (those before have come back from memory when they are needed)
  __shared__ double recent[WALK_STAGES * 64];
  const u32 lane = threadIdx.x;
  const u64 below = (1ull << lane) - 1ull;
  // the state of the walk; the same in every lane
  double delta = 0;                     // end of the previous kernel minus its end without any stall
  double delta_first = 0;               // the same when the second iteration begins
  bool second = false;
  double free0 = 0, free1 = 0, free2 = 0, free3 = 0;       // when each channel is free again (out 0, 1, in 0, 1)
  double delta_pt = 0;                  // delta when the uses of the last point began
  bool stalled_pt = false;              // ... and whether its kernel has waited
  double stall = 0;                     // of this lane's events
  u32 n_stalled = 0;

  // An event's own values are loaded WALK_STAGES steps ahead, its predecessor's place as many steps before that, so
  // that the predecessor's result - if it was stored by then - comes with the values.
  double r_sp[WALK_STAGES], r_A[WALK_STAGES], r_off[WALK_STAGES], r_val[WALK_STAGES];
  uint2 r_ev[WALK_STAGES];
  u32 r_pred[WALK_STAGES], ahead[WALK_STAGES];
#pragma unroll
  for (u32 q = 0; q < WALK_STAGES; ++q) {
    const u32 p = q * 64u + lane;
    r_sp[q] = w.sp[p]; r_A[q] = w.A[p]; r_off[q] = w.off[p]; r_ev[q] = w.ev[p]; r_pred[q] = w.pred[p];
    r_val[q] = 0;                       // (no result is in memory yet)
    ahead[q] = w.pred[p + WALK_STAGES * 64u];
  }
  for (u32 step0 = 0; step0 < steps; step0 += WALK_STAGES) {
#pragma unroll
    for (u32 q = 0; q < WALK_STAGES; ++q) {
      const u32 base = (step0 + q) * 64u;
      const double sp = r_sp[q], A = r_A[q], off = r_off[q];
      const u32 ev = r_ev[q].x, mig = r_ev[q].y, kind = ev & 7u, pos = (ev >> W_POS) & 63u, pred = r_pred[q];
      const bool has = pred != NONE32, here = has && pred >= base;
      // what it waits for: in memory when its values were loaded, one of the steps since, or of these 64
      double pv = !has ? 0.0 : pred + WALK_STAGES * 64u < base + 64u ? r_val[q] : recent[pred % (WALK_STAGES * 64u)];
      if (here) pv = 0;
      const bool is_in = kind >= EV_IN && kind < EV_USE, is_use = kind == EV_USE;
      const u64 m0 = ballot(kind == EV_OUT), m1 = ballot(kind == EV_OUT + 1), m2 = ballot(kind == EV_IN), m3 = ballot(kind == EV_IN + 1),
                use_m = ballot(is_use), second_m = ballot((ev & W_SECOND) != 0);
      const u64 in_here = ballot(here && is_in), use_here = ballot(here && is_use);
      const u32 src = (pred & 63u) << 2;
      // A channel that is free at x serves requests that are ready at r_1, r_2, .. and take tau_1, tau_2, ..: the k-th is done
      // at A_k + max(x, r_j - A_(j-1) for j <= k), A the sums of tau.  Those do not change while the delay does, so a step
      // of the walk is one running maximum for all four channels, SEGMENT apart (two, where a prefetch's eviction is among
      // the 64).  A settled event keeps the end of the kernel before it, and so its maximum.
      const double As = A - (double)(kind + 1u) * SEGMENT;
      const double served = A + (kind == EV_OUT ? free0 : kind == EV_OUT + 1 ? free1 : kind == EV_IN ? free2 : free3);
      double win = is_in ? pv : 0.0, wuse = is_use ? pv : 0.0;     // what a prefetch, a use waits for
      double free_at = sp + delta, t;                              // end of the previous kernel
      u64 waited = 0;
      while (true) {
        if (in_here) {
          const double out = lane_at(larger(scan_max(free_at + off) + As, served), src);
          if (here && is_in) win = out;
        }
        t = larger(scan_max(larger(win, free_at) + off) + As, served);
        if (use_here) { const double x = lane_at(t, src); if (here && is_use) wuse = x; }
        const u64 waits = ballot(wuse > free_at) & ~waited;
        if (!waits) break;
        const u32 fl = (u32)__builtin_ctzll(waits);                // the kernel waits for this prefetch (the uses lie in their order)
        waited |= 1ull << fl;
        delta = lane_getf(wuse - sp, fl);
        const double next = sp + delta;
        if (pos > (u32)__builtin_amdgcn_readlane((int)pos, (int)fl)) free_at = next;     // (the events behind it)
      }
      const double dl = free_at - sp;                              // the delay when the event was settled
      if (!second && second_m) {
        // (the first event of the second iteration: all behind it are of it too)
        second = true;
        const u32 cnt = (u32)__popcll(m0 | m1 | m2 | m3 | use_m);
        delta_first = lane_getf(dl, (u32)__builtin_ctzll(ballot(pos == cnt - (u32)__popcll(second_m))));
      }
      if (use_m) {
        const u32 first = (ev >> W_FIRST) & 63u;
        double began = lane_at(dl, first << 2);                    // the delay when the uses of its point began
        if (ev & W_CONT) began = delta_pt;
        if (is_use && (ev & W_SECOND)) { const double e = sp + began; late[mig] = wuse > e ? (u64)(wuse - e) : 0ull; }
        const u32 last = 63u - (u32)__builtin_clzll(use_m);
        delta_pt = lane_getf(began, last);
        const u32 ev_last = (u32)__builtin_amdgcn_readlane((int)ev, (int)last);
        const u64 of_last = ~0ull << ((ev_last >> W_FIRST) & 63u);
        // points whose kernels waited, counted at the first use that did
        const u64 w2 = waited & second_m;
        if (w2) {
          const bool is = (w2 >> lane) & 1ull;
          if (is) stall += wuse - free_at;
          n_stalled += (u32)__popcll(ballot(is && !(w2 & below & (~0ull << first)) && !((ev & W_CONT) && stalled_pt)));
        }
        stalled_pt = (w2 & of_last) != 0 || ((ev_last & W_CONT) && stalled_pt);
      }
      if (m0) free0 = lane_getf(t, 63u - (u32)__builtin_clzll(m0));
      if (m1) free1 = lane_getf(t, 63u - (u32)__builtin_clzll(m1));
      if (m2) free2 = lane_getf(t, 63u - (u32)__builtin_clzll(m2));
      if (m3) free3 = lane_getf(t, 63u - (u32)__builtin_clzll(m3));
      res[base + lane] = t;
      recent[(base + lane) % (WALK_STAGES * 64u)] = t;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");       // the next loads find what was just written (in order)
      // the step that takes these registers next
      const u32 p = base + WALK_STAGES * 64u + lane, pn = ahead[q];
      r_sp[q] = w.sp[p]; r_A[q] = w.A[p]; r_off[q] = w.off[p]; r_ev[q] = w.ev[p]; r_pred[q] = pn;
      r_val[q] = res[pn < base + 64u ? pn : 0u];                   // (the others: not used)
      ahead[q] = w.pred[p + WALK_STAGES * 64u];
    }
  }
  if (!second) delta_first = delta;
  stall = lane_getf(scan_sum(stall), 63u);
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
    const u64 cap = n ? n : 1, ce = 6 * cap, cp = walk_events(ce);
    const u64 he = radix_hist_elems(ce);
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off += (bytes + 255) & ~(size_t)255; return o; };
    const size_t o_keys = take(ce * 8), o_alt = take(ce * 8), o_res = take(cp * 8), o_late = take(cap * 8), o_pos = take(4 * cap * 4),
                 o_hist = take(he * 4), o_st = take(sizeof(ReplayStats)), o_dur = take((u64)K * 8),
                 o_start = take(((u64)K + 1) * 8), o_ts = take(scan_scratch_elems(K) * 8), o_tst = take(128),
                 o_sp = take(cp * 8), o_A = take(cp * 8), o_off = take(cp * 8), o_ev = take(cp * 8), o_pred = take(cp * 4);
    void* q = nullptr;
    G10_TRY(mem_dev_alloc(&q, off));
    char* b = (char*)q;
    w->rp_arena = q; w->rp_cap = (u32)cap;
    w->rp_keys = (u64*)(b + o_keys); w->rp_alt = (u64*)(b + o_alt); w->rp_res = (u64*)(b + o_res); w->rp_late = (u64*)(b + o_late);
    w->rp_pos = (u32*)(b + o_pos); w->rp_hist = (u32*)(b + o_hist); w->rp_stats = (void*)(b + o_st);
    w->rp_dur = (u64*)(b + o_dur); w->rp_start = (u64*)(b + o_start); w->rp_tscr = (u64*)(b + o_ts); w->rp_tstats = (void*)(b + o_tst);
    w->rp_sp = (double*)(b + o_sp); w->rp_A = (double*)(b + o_A); w->rp_off = (double*)(b + o_off); w->rp_ev = (uint2*)(b + o_ev);
    w->rp_pred = (u32*)(b + o_pred);
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
  // (a channel's transfers fit the iteration that they were planned for, w->T; each is made twice)
  const bool exact = T < REPLAY_EXACT / 10 && w->T < REPLAY_EXACT / 10 && walk_events(ne) < (1ull << 32);
  if (n) {
    hipLaunchKernelGGL(k_rp_events, dim3((n + G10_BLOCK - 1) / G10_BLOCK), dim3(G10_BLOCK), 0, s, (const g10_migration*)w->records,
                       (const uint2*)w->rec_ab, eager ? (const u32*)w->pf_gained : (const u32*)nullptr, n, K, rbits, keys, st);
    G10_HIP(hipGetLastError());
    G10_TRY(radix_sort_u64(&keys, &alt, ne, rbits + 1 + EV_BITS + bits_for(2ull * K), w->rp_hist, s, rbits + 1));
    hipLaunchKernelGGL(k_rp_index, dim3((u32)((ne + G10_BLOCK - 1) / G10_BLOCK)), dim3(G10_BLOCK), 0, s, (const u64*)keys, (u32)ne, n, rbits,
                       exact ? 1u : 0u, w->rp_pos);
    G10_HIP(hipGetLastError());
  }
  if (exact) {
    const u32 np = (u32)walk_events(ne);
    const Walk wk = {w->rp_sp, w->rp_A, w->rp_off, w->rp_ev, w->rp_pred};
    hipLaunchKernelGGL(k_rp_expand, dim3((np + G10_BLOCK - 1) / G10_BLOCK), dim3(G10_BLOCK), 0, s, (const u64*)keys, (u32)ne, np,
                       (const g10_migration*)w->records, n, rbits, (const u32*)w->rp_pos, start, K, T, wk);
    G10_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_replay, dim3(1), dim3(G10_WAVE), 0, s, wk, (np - WALK_PAD) / 64u, T, (double*)w->rp_res, w->rp_late, st);
  } else
    hipLaunchKernelGGL(k_replay_long, dim3(1), dim3(G10_WAVE), 0, s, (const u64*)keys, (u32)ne, (const g10_migration*)w->records, n, rbits,
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
