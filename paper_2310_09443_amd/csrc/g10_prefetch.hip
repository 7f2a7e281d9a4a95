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

struct PfShared {
  u64 n_moved, slots;
};

__global__ __launch_bounds__(WG) void k_eager(const g10_migration* __restrict__ rec, const uint2* __restrict__ rec_ab,
                                             const u32* __restrict__ order, u32 n, u64* __restrict__ E, u32 K, u32 nch,
                                             u32 spt, u32 shift_ch, u64 cap, u32* __restrict__ gained,
                                             u32* __restrict__ last, u64* __restrict__ stats) {
  extern __shared__ __align__(16) unsigned char smem[];
  u64* cmax = (u64*)smem;                          // [nch] largest pressure of the chunk (lazy add included)
  u64* ladd = cmax + nch;                          // [nch] added to every slot of the chunk, not yet in E
  PfShared* S = (PfShared*)(ladd + nch);
  const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, CH = 1u << shift_ch;

  for (u32 c = wave; c < nch; c += WG_WAVES) {           // chunk maxima
    u64 m = 0;
    for (u32 st = 0; st < spt; ++st) {
      const u32 j0 = c * CH + st * 256u + lane * 4u;
#pragma unroll
      for (u32 i = 0; i < 4; ++i) if (j0 + i < K) { const u64 x = E[j0 + i]; m = x > m ? x : m; }
    }
    m = wave_max(m);
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
  // A move is bound by its dependent trips to L2 (0.6 us each).  It takes one where the highest chunk that may refuse does:
  // that chunk and the one at the end of the window are loaded together, whole, and the chunks cut are written back from
  // those registers, without a wait - the accesses of one wavefront are served in order.  (Stress trace, 1226 moves: 3.4 ms;
  // 6.2 with a trip for the test, one or more for the search, one per cut chunk and one for the stores to arrive, and with a
  // look at every chunk of the timeline, seven a lane, in the search and in the update.)
  if (wave == 0) {
    u64 n_moved = 0, slots = 0;
    u32 nr = 0, na = 0, nb = 0;
    u64 nsz = 0;
    if (lane < n) { nr = order[lane]; nsz = rec[nr].size_bytes; const uint2 ab = rec_ab[nr]; na = ab.x; nb = ab.y; }
    u32 it = 0;                                    // first record of the 64
    u64 todo = 0;                                  // lanes whose record is not done yet
    u32 cr = 0, ca = 0, cb = 0, cbb = 0;           // this lane's record: its number, absent window, last absent slot
    u64 csz = 0, val = 0;                          // ... size; pressure of that slot
    struct Strip { u64 x[4]; };                    // a strip of 256 slots of a chunk, 64 apart in a lane
    auto load_strip = [&](u32 c, u32 st) -> Strip {
      Strip v;
#pragma unroll
      for (u32 i = 0; i < 4; ++i) { const u32 j = c * CH + st * 256u + i * 64u + lane; v.x[i] = E[j < K ? j : K - 1]; }
      return v;
    };
    while (true) {
      if (!todo) {                                 // the next 64
        if (it >= n) break;
        const u32 cnt = n - it < 64u ? n - it : 64u;
        todo = cnt == 64u ? ~0ull : (1ull << cnt) - 1ull;
        cr = nr; ca = na; cb = nb; csz = nsz;
        cbb = cb >= K ? cb - K : cb;
        it += cnt;
        if ((todo >> lane) & 1ull) val = E[cbb] + ladd[cbb >> shift_ch];
        if (it + lane < n) { nr = order[it + lane]; nsz = rec[nr].size_bytes; const uint2 ab = rec_ab[nr]; na = ab.x; nb = ab.y; }
      }
      const bool mine = (todo >> lane) & 1ull;
      const u64 pm = __ballot(mine && csz <= cap && val <= cap - csz);
      const u32 f = pm ? (u32)__builtin_ctzll(pm) : 64u;       // the records before it stay where they are
      if (mine && lane < f) { gained[cr] = 0u; last[cr] = cbb; }
      if (!pm) { todo = 0; continue; }
      todo &= f == 63u ? 0ull : ~0ull << (f + 1u);
      const u32 r = (u32)__builtin_amdgcn_readlane((int)cr, (int)f), a = (u32)__builtin_amdgcn_readlane((int)ca, (int)f),
                b = (u32)__builtin_amdgcn_readlane((int)cb, (int)f), bb = b >= K ? b - K : b;
      const u64 s = lane_value64(csz, f);

      // the earliest slot from which every slot up to b can hold the tensor: one past the last slot of [a, b]
      // that cannot.  The window in pieces of chunks, from its end back - the part in the second iteration, then the one in
      // the first -, a piece per lane: the chunk maxima say which piece may hold that slot, and that piece is scanned.
      const u64 lim = cap - s;                     // a slot holds the tensor iff its pressure <= lim
      const u32 c_end = bb >> shift_ch;            // the chunk at the end of the window
      const u32 n2 = b >= K ? c_end + 1u - ((a > K ? a - K : 0u) >> shift_ch) : 0u;     // pieces of the second iteration
      const u32 t1 = (b < K ? b : K - 1u) >> shift_ch, n1 = a < K ? t1 + 1u - (a >> shift_ch) : 0u;      // last chunk, pieces of the first
      auto chunk_of = [&](u32 t) -> u32 { return t < n2 ? c_end - t : t1 - (t - n2); };
      u32 p = a;
      u32 c_seen = NONE32;                         // the chunk scanned last; its first strip and the end chunk's
      Strip v_end = {}, v_seen = {};
      bool end_loaded = false;
      u32 t0 = 0, pieces = n1 + n2;                // (pieces from the end down to the one of p)
      while (t0 < n1 + n2) {
        const u32 t = t0 + lane;
        const u64 hits = __ballot(t < n1 + n2 && cmax[t < n1 + n2 ? chunk_of(t) : 0u] > lim);
        if (!hits) { t0 += 64u; continue; }
        const u32 th = uniform(t0 + (u32)__builtin_ctzll(hits)), c = chunk_of(th), second = th < n2 ? K : 0u;
        const u32 lo = c * CH + second > a ? c * CH + second : a, end_ = c * CH + CH < K ? c * CH + CH : K;
        const u32 hi = end_ - 1u + second < b ? end_ - 1u + second : b;
        u32 best = 0;                              // doubled coordinate + 1 of the last refusing slot of the piece
        const u64 lz = ladd[c];
        for (u32 st = 0; st < spt; ++st) {
          const Strip v = load_strip(c, st);
          if (!end_loaded) { v_end = c == c_end ? v : load_strip(c_end, 0); end_loaded = true; }
          if (spt == 1u) { c_seen = c; v_seen = v; }
#pragma unroll
          for (u32 i = 0; i < 4; ++i) {
            const u32 j = c * CH + st * 256u + i * 64u + lane + second;
            if (j >= lo && j <= hi && v.x[i] + lz > lim) best = j + 1;    // ascending: the last one stays
          }
        }
        best = wave_max(best);
        if (best) { p = best; pieces = best > hi ? th : th + 1u; break; }      // (one past the piece's end: the piece is not gained)
        t0 = th + 1u;
      }
      const u32 g = b + 1 - p;
      if (lane == 0) {
        gained[r] = g;
        const u32 nl = b - g;                      // last absent slot left (one before a if none)
        last[r] = nl >= K ? nl - K : nl;
      }
      if (g) {                                     // the slots gained take the tensor
        n_moved += 1; slots += g;
        if (mine && in_doubled(cbb, K, p, b) != NONE32) val += s;
        // whole chunks lazily; the window cuts the first and the last piece at most (of one chunk, where it goes around)
        u32 cut0 = NONE32, cut1 = NONE32;
        for (u32 q = 0; q < pieces; q += 64u) {
          const u32 t = q + lane;
          bool cut = false;
          u32 c = 0;
          if (t < pieces) {
            c = chunk_of(t);
            const u32 second = t < n2 ? K : 0u, lo = c * CH + second, end_ = (c * CH + CH < K ? c * CH + CH : K) + second;
            cut = lo < p || end_ > b + 1u;
            if (!cut) { ladd[c] += s; cmax[c] += s; }
          }
          u64 cm = __ballot(cut);
          if (cm && cut0 == NONE32) { cut0 = (u32)__builtin_amdgcn_readlane((int)c, (int)__builtin_ctzll(cm)); cm &= cm - 1; }
          if (cm) cut1 = (u32)__builtin_amdgcn_readlane((int)c, (int)__builtin_ctzll(cm));
        }
        if (cut1 == cut0) cut1 = NONE32;
        // (slots in [p, b]: both less K where it lies in the second iteration, or all but the (b - K, p) between)
        const bool both = p < K && b >= K;
        const u32 rlo = both ? b - K + 1u : p >= K ? p - K : p, rn = both ? p - rlo : b - p + 1u;
#pragma unroll 1
        for (u32 w = 0; w < 2; ++w) {
          const u32 cc = w ? cut1 : cut0;
          if (cc == NONE32) continue;
          const u64 lz = ladd[cc];
          u64 m = 0;
          for (u32 st = 0; st < spt; ++st) {
            const u32 j0 = cc * CH + st * 256u + lane;          // (64 neighbouring slots per load and store)
            Strip v;
            if (cc == c_seen) v = v_seen;                       // (strips of a chunk of one strip only)
            else if (spt == 1u && end_loaded && cc == c_end) v = v_end;
            else v = load_strip(cc, st);
#pragma unroll
            for (u32 i = 0; i < 4; ++i) {
              const u32 j = j0 + i * 64u;
              if ((j - rlo < rn) != both && j < K) { v.x[i] += s; E[j] = v.x[i]; }
              const u64 x = j < K ? v.x[i] + lz : 0ull;
              m = x > m ? x : m;
            }
          }
          m = wave_max(m);
          if (lane == 0) cmax[cc] = m;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the next loads find what was just written (in order)
      }
    }
    if (lane == 0) { S->n_moved = n_moved; S->slots = slots; }
  }
  __syncthreads();
  // the lazy adds into the slots; the peak
  u64 m = 0;
  for (u32 j = tid; j < K; j += WG) { const u64 x = E[j] + ladd[j >> shift_ch]; E[j] = x; m = x > m ? x : m; }
  m = wave_max(m);
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
  hipLaunchKernelGGL(k_eager, dim3(1), dim3(WG), lds, s, (const g10_migration*)w->records, (const uint2*)w->rec_ab,
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
