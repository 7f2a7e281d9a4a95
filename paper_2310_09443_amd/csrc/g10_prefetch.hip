// Smart tensor prefetching (G10, Section 4.4) on a finished plan.
//
// The evicted periods are visited in the order of their latest safe prefetch
// time; each prefetch moves back, in whole kernel slots and not past the first
// absent slot, to the earliest slot from which every slot up to the old
// prefetch can hold the tensor (pressure + size <= capacity); the pressure of
// the slots gained rises by the tensor's size.  Every step depends on the
// pressure the earlier ones left, so this is a serial chain like the eviction
// loop: one wavefront walks it (a workgroup sets the timeline up and finishes
// it), the pressure in HBM / L2, per chunk a lazy add and the chunk maximum in
// LDS.  The search asks the chunk maxima which chunk can hold the last slot
// that cannot take the tensor and scans only that chunk; the update adds
// lazily to whole chunks and slot by slot at the ends.

#include "g10_plan_defs.h"

#include <stdlib.h>
#include <string.h>

using namespace g10;

namespace {

__global__ __launch_bounds__(G10_BLOCK) void k_pf_keys(const g10_migration* __restrict__ rec, u32 n, const u64* __restrict__ start,
                                                      u32 K, u64 T, u64* __restrict__ keys, u32* __restrict__ order) {
  const u32 i = blockIdx.x * G10_BLOCK + threadIdx.x;
  if (i >= n) return;
  const u64 t_use = start[rec[i].next_use] + (rec[i].wraps ? T : 0ull);
  keys[i] = t_use - rec[i].t_in_ns;              // latest safe prefetch time
  order[i] = i;
}

__device__ __forceinline__ u64 lane_value64(u64 v, u32 l) {      // lane l's v (l the same in the whole wavefront)
  const u32 lo = (u32)__builtin_amdgcn_readlane((int)(u32)v, (int)l), hi = (u32)__builtin_amdgcn_readlane((int)(u32)(v >> 32), (int)l);
  return ((u64)hi << 32) | lo;
}

// largest value over the lanes: the upper halves first, then the lower ones of the lanes that have it (a maximum of 64-bit
// values in one go compares and selects at every step of the reduction)
__device__ __forceinline__ u64 wave_max64(u64 v) {
  const u32 hi = (u32)(v >> 32), top = wave_max(hi);
  return ((u64)top << 32) | wave_max(hi == top ? (u32)v : 0u);
}

struct PfShared {
  u64 n_moved, slots;
};

// ONE: a chunk is one strip of 256 slots (timelines of up to 131 072 slots).  E holds nch chunks, zeros behind slot K - 1.
template <bool ONE>
__global__ __launch_bounds__(WG) void k_eager(const g10_migration* __restrict__ rec, const uint2* __restrict__ rec_ab,
                                             const u32* __restrict__ order, u32 n, u64* __restrict__ E, u32 K, u32 nch,
                                             u32 spt, u32 shift_ch, u64 cap, u32* __restrict__ gained,
                                             u32* __restrict__ last, u64* __restrict__ stats) {
  extern __shared__ __align__(16) unsigned char smem[];
  u64* cmax = (u64*)smem;                          // [nch] largest pressure of the chunk (lazy add included)
  u64* ladd = cmax + nch;                          // [nch] added to every slot of the chunk, not yet in E
  PfShared* S = (PfShared*)(ladd + nch);
  const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, CH = 1u << shift_ch, strips = ONE ? 1u : spt;

  for (u32 c = wave; c < nch; c += WG_WAVES) {           // chunk maxima; the slots behind the timeline's end
    u64 m = 0;
    for (u32 st = 0; st < strips; ++st) {
      const u32 j0 = c * CH + st * 256u + lane * 4u;
#pragma unroll
      for (u32 i = 0; i < 4; ++i) {
        if (j0 + i < K) { const u64 x = E[j0 + i]; m = x > m ? x : m; }
        else E[j0 + i] = 0;
      }
    }
    m = wave_max64(m);
    if (lane == 0) { cmax[c] = m; ladd[c] = 0; }
  }
  if (tid == 0) { S->n_moved = 0; S->slots = 0; }
  __syncthreads();

  // The chain itself runs in the first wavefront alone: every step waits for the one before, and one wavefront
  // needs no barrier between them (the others wait at the barrier below; they set up and finish the timeline).
  // Most prefetches cannot move at all: the slot just before them cannot take the tensor.  That test needs the pressure
  // of one slot; so 64 records are tested at once, one per lane, those before the first that passes are done - nothing
  // gained -, only that one takes the search, and the ones behind it are tested again with what its move adds to their
  // slots (kept in the lanes, not loaded anew).  (The records of the next 64 are on their way meanwhile.)
  // A move is bound by the instructions of the one wavefront, which it issues one after the other, and by a trip to L2: the
  // chunk at the end of the window is asked for first, the highest chunk that may refuse as soon as the chunk maxima name it;
  // both come whole, and are written back from those registers, without a wait - the accesses of one wavefront are served
  // in order.  The chunks between them take a lazy add.  (Stress trace, 1226 moves: 6.2 ms with a trip for the test, one or
  // more for the search, one per cut chunk and one for the stores to arrive; 3.3 with one trip, 6600 cycles a
  // move, and a maximum of 64-bit values over the lanes for the search and for each cut chunk; 2.15 now.)
  if (wave == 0) {
    u64 n_moved = 0, slots = 0;
    // (the next 64 records and the numbers of those behind them; past the end the last one again)
    auto number = [&](u32 at) -> u32 { return order[at < n ? at : n - 1u]; };
    u32 nr = 0, nr2 = 0, na = 0, nb = 0;
    u64 nsz = 0;
    if (n) { nr = number(lane); nr2 = number(64u + lane); nsz = rec[nr].size_bytes; const uint2 ab = rec_ab[nr]; na = ab.x; nb = ab.y; }
    u32 it = 0;                                    // first record of the next 64
    struct Strip { u64 x[4]; };                    // a strip of 256 slots of a chunk, 64 apart in a lane
    auto load_strip = [&](u32 c, u32 st) -> Strip {
      Strip v;
      const u64* at = E + (c * CH + st * 256u + lane);
#pragma unroll
      for (u32 i = 0; i < 4; ++i) v.x[i] = at[i * 64u];
      return v;
    };
    while (it < n) {
      // ---- the next 64 records -----------------------------------------------------------------------------------
      const u32 cnt = n - it < 64u ? n - it : 64u;
      const u32 cr = nr, ca = na, cb = nb, cbb = cb >= K ? cb - K : cb;      // this lane's record: its number, absent window, last absent slot
      const u64 csz = nsz, climit = cap - csz;     // (a slot holds the tensor iff its pressure is not above this; a tensor above the capacity never moves)
      u64 val = E[cbb] + ladd[cbb >> shift_ch];    // pressure of the last absent slot
      u32 cg = 0;                                  // slots gained
      u64 todo = ballot(lane < cnt && csz <= cap); // lanes whose record is not done yet
      it += cnt;
      nr = nr2; nsz = rec[nr].size_bytes;
      { const uint2 ab = rec_ab[nr]; na = ab.x; nb = ab.y; }
      nr2 = number(it + 64u + lane);
      while (true) {
        todo &= ballot(val <= climit);             // (the pressure only rises: a record that cannot move now does not move)
        if (!todo) break;
        const u32 f = (u32)__builtin_ctzll(todo);  // the records before it stay where they are
        todo &= todo - 1;
        const u32 a = (u32)__builtin_amdgcn_readlane((int)ca, (int)f), b = (u32)__builtin_amdgcn_readlane((int)cb, (int)f), bb = b >= K ? b - K : b;
        const u64 s = lane_value64(csz, f), lim = cap - s;
        const u32 c_end = bb >> shift_ch;          // the chunk at the end of the window
        Strip v_end = {}, v_hit = {};
        if (ONE) v_end = load_strip(c_end, 0);

        // the earliest slot from which every slot up to b can hold the tensor: one past the last slot of [a, b]
        // that cannot.  The window in pieces of chunks, from its end back - the part in the second iteration, then the one in
        // the first -, a piece per lane: the chunk maxima say which piece may hold that slot, and that piece is scanned.
        const u32 n2 = b >= K ? c_end + 1u - ((a > K ? a - K : 0u) >> shift_ch) : 0u;     // pieces of the second iteration
        const u32 t1 = (b < K ? b : K - 1u) >> shift_ch, n1 = a < K ? t1 + 1u - (a >> shift_ch) : 0u;      // last chunk, pieces of the first
        auto chunk_of = [&](u32 t) -> u32 { return t < n2 ? c_end - t : t1 + n2 - t; };
        u32 p = a, c_hit = NONE32, t0 = 0, pieces = n1 + n2;                // (pieces from the end down to the one of p)
        while (t0 < n1 + n2) {
          const u32 t = t0 + lane;
          const u64 hits = ballot(t < n1 + n2 && cmax[t < n1 + n2 ? chunk_of(t) : 0u] > lim);
          if (!hits) { t0 += 64u; continue; }
          const u32 th = t0 + (u32)__builtin_ctzll(hits), c = chunk_of(th), second = th < n2 ? K : 0u;
          const u32 lo = c * CH + second > a ? c * CH + second : a, end_ = c * CH + CH < K ? c * CH + CH : K;
          const u32 hi = end_ - 1u + second < b ? end_ - 1u + second : b;
          const u64 lz = uniform(ladd[c]), limz = lim - lz;
          u32 best = 0;                            // doubled coordinate + 1 of the last refusing slot of the piece
          for (u32 st = strips; st-- > 0 && !best;) {
            const u32 j0 = c * CH + st * 256u + second;
            u64 m[4];
            auto refusing = [&](const Strip& v) {
#pragma unroll
              for (u32 i = 0; i < 4; ++i) m[i] = ballot(j0 + lane + i * 64u - lo <= hi - lo && (v.x[i] > limz || lz > lim));
            };
            if (ONE && c == c_end) refusing(v_end);        // (a copy of it would be waited for before the other load is made)
            else { v_hit = load_strip(c, st); c_hit = c; refusing(v_hit); }
            if (m[3]) best = j0 + 256u - (u32)__builtin_clzll(m[3]);
            else if (m[2]) best = j0 + 192u - (u32)__builtin_clzll(m[2]);
            else if (m[1]) best = j0 + 128u - (u32)__builtin_clzll(m[1]);
            else if (m[0]) best = j0 + 64u - (u32)__builtin_clzll(m[0]);
          }
          if (best) { p = best; pieces = best > hi ? th : th + 1u; break; }      // (one past the piece's end: the piece is not gained)
          t0 = th + 1u;
        }
        const u32 g = b + 1 - p;                   // (one at least: slot b can hold it)
        if (lane == f) cg = g;
        // ---- the slots gained take the tensor ----------------------------------------------------------------------
        n_moved += 1; slots += g;
        // (slots in [p, b]: both less K where it lies in the second iteration, or all but the (b - K, p) between)
        const bool both = p < K && b >= K;
        const u32 rlo = both ? b - K + 1u : p >= K ? p - K : p, rn = both ? p - rlo : b - p + 1u;
        if ((cbb - rlo < rn) != both) val += s;
        // the pieces between the first and the last lie inside the window
        for (u32 t = 1u + lane; t + 1u < pieces; t += 64u) { const u32 c = chunk_of(t); ladd[c] += s; cmax[c] += s; }
        // those two, slot by slot (one chunk, where the window goes around)
        const u32 c_low = chunk_of(pieces - 1u);
        if (ONE) {
          const u64 lz0 = ladd[c_end], lz1 = ladd[c_low];
          const u32 j0 = c_end * 256u + lane, j1 = c_low * 256u + lane;
          if (c_low != c_hit) v_hit = load_strip(c_low, 0);
          u64 m0 = 0, m1 = 0;
#pragma unroll
          for (u32 i = 0; i < 4; ++i) {
            const u32 j = j0 + i * 64u;
            if ((j - rlo < rn) != both && j < K) { v_end.x[i] += s; E[j] = v_end.x[i]; }
            m0 = v_end.x[i] > m0 ? v_end.x[i] : m0;
          }
          if (c_low != c_end) {
#pragma unroll
            for (u32 i = 0; i < 4; ++i) {
              const u32 j = j1 + i * 64u;
              if ((j - rlo < rn) != both && j < K) { v_hit.x[i] += s; E[j] = v_hit.x[i]; }
              m1 = v_hit.x[i] > m1 ? v_hit.x[i] : m1;
            }
            m1 = wave_max64(m1) + lz1;
            if (lane == 0) cmax[c_low] = m1;
          }
          m0 = wave_max64(m0) + lz0;
          if (lane == 0) cmax[c_end] = m0;
        } else {
#pragma unroll 1
          for (u32 w = 0; w < (c_low != c_end ? 2u : 1u); ++w) {
            const u32 c = w ? c_low : c_end;
            u64 m = 0;
            for (u32 st = 0; st < strips; ++st) {
              const u32 j0 = c * CH + st * 256u + lane;
              Strip v = load_strip(c, st);
#pragma unroll
              for (u32 i = 0; i < 4; ++i) {
                const u32 j = j0 + i * 64u;
                if ((j - rlo < rn) != both && j < K) { v.x[i] += s; E[j] = v.x[i]; }
                m = v.x[i] > m ? v.x[i] : m;
              }
            }
            m = wave_max64(m) + ladd[c];
            if (lane == 0) cmax[c] = m;
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the next loads find what was just written (in order)
      }
      if (lane < cnt) {
        gained[cr] = cg;
        const u32 nl = cb - cg;                    // last absent slot left (one before a if none)
        last[cr] = nl >= K ? nl - K : nl;
      }
    }
    if (lane == 0) { S->n_moved = n_moved; S->slots = slots; }
  }
  __syncthreads();
  // the lazy adds into the slots; the peak
  u64 m = 0;
  for (u32 j = tid; j < K; j += WG) { const u64 x = E[j] + ladd[j >> shift_ch]; E[j] = x; m = x > m ? x : m; }
  m = wave_max64(m);
  if (lane == 0) atomicMax((unsigned long long*)&stats[2], (unsigned long long)m);
  if (tid == 0) { stats[0] = S->n_moved; stats[1] = S->slots; }
}

}  // namespace

int prefetch_run(g10_plan_s* h, g10_prefetch_result* out) {
  PlanWork* w = h->work;
  if (!w || !w->planned) return G10_EINVAL;
  hipStream_t s = h->stream;
  const u32 K = h->K, n = (u32)w->plan_n_mig;
  if (!w->h_pf_order) {
    const u64 C = w->C ? w->C : 1;
    w->h_pf_order = (u32*)malloc(C * 4); w->h_pf_gained = (u32*)malloc(C * 4); w->h_pf_last = (u32*)malloc(C * 4);
    w->h_pf_pressure = (u64*)malloc((u64)K * 8);
    if (!w->h_pf_order || !w->h_pf_gained || !w->h_pf_last || !w->h_pf_pressure) {
      // all four or none: the next call must find the same state as the first
      free(w->h_pf_order); free(w->h_pf_gained); free(w->h_pf_last); free(w->h_pf_pressure);
      w->h_pf_order = nullptr; w->h_pf_gained = nullptr; w->h_pf_last = nullptr; w->h_pf_pressure = nullptr;
      return G10_ENOMEM;
    }
  }
  G10_HIP(hipEventRecord(w->ev[0], s));
  G10_HIP(hipMemcpyAsync(w->pf_pressure, w->pressure_after, (u64)K * 8, hipMemcpyDeviceToDevice, s));
  G10_HIP(hipMemsetAsync(w->pf_stats, 0, 4 * 8, s));
  u64* keys = w->pf_keys; u64* alt = w->pf_keys_alt;
  u32* ord = w->pf_order; u32* oalt = w->pf_order_alt;
  if (n) {
    hipLaunchKernelGGL(k_pf_keys, dim3((n + G10_BLOCK - 1) / G10_BLOCK), dim3(G10_BLOCK), 0, s, (const g10_migration*)w->records, n,
                       w->start, K, w->T, keys, ord);
    G10_HIP(hipGetLastError());
    G10_TRY(radix_sort_u64_pairs(&keys, &alt, &ord, &oalt, n, bits_for(2 * w->T), w->hist, s));
  }
  const size_t lds = ((size_t)2 * w->nch * 8 + sizeof(PfShared) + 15) & ~(size_t)15;
  hipLaunchKernelGGL((w->spt == 1 ? k_eager<true> : k_eager<false>), dim3(1), dim3(WG), lds, s, (const g10_migration*)w->records, (const uint2*)w->rec_ab,
                     (const u32*)ord, n, w->pf_pressure, K, w->nch, w->spt, w->shift_ch, w->plan_cap, w->pf_gained, w->pf_last,
                     w->pf_stats);
  G10_HIP(hipGetLastError());
  u64 st[4] = {0, 0, 0, 0};
  G10_HIP(hipMemcpyAsync(st, w->pf_stats, sizeof st, hipMemcpyDeviceToHost, s));
  if (n) {
    G10_HIP(hipMemcpyAsync(w->h_pf_order, ord, (u64)n * 4, hipMemcpyDeviceToHost, s));
    G10_HIP(hipMemcpyAsync(w->h_pf_gained, w->pf_gained, (u64)n * 4, hipMemcpyDeviceToHost, s));
    G10_HIP(hipMemcpyAsync(w->h_pf_last, w->pf_last, (u64)n * 4, hipMemcpyDeviceToHost, s));
  }
  G10_HIP(hipMemcpyAsync(w->h_pf_pressure, w->pf_pressure, (u64)K * 8, hipMemcpyDeviceToHost, s));
  G10_HIP(hipEventRecord(w->ev[1], s));
  G10_HIP(hipStreamSynchronize(s));
  float ms = 0.f;
  G10_HIP(hipEventElapsedTime(&ms, w->ev[0], w->ev[1]));
  memset(out, 0, sizeof *out);
  out->n_migrations = n; out->n_moved = st[0]; out->slots_gained = st[1]; out->peak_bytes = st[2];
  out->order = w->h_pf_order; out->gained = w->h_pf_gained; out->absent_last = w->h_pf_last; out->pressure = w->h_pf_pressure;
  out->ms = ms;
  w->prefetched = true;
  return G10_OK;
}
