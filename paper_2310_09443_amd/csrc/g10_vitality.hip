// Tensor vitality analysis on the device (G10, Section 4.2).
//
//   pairs (kernel, tensor)  --pack-->  64-bit keys (tensor << kbits | kernel)
//     --LSD radix sort, 8-bit digits, only the significant digits-->
//     --adjacent compare + scan-->  distinct keys = per-tensor use lists
//     --adjacent difference-->      inactive periods (gap of >= 1 whole kernel),
//                                   plus the cross-iteration period of globals
//   lifetimes --interval add into a difference array + scan--> pressure[K]
//     --wavefront-shuffle max--> peak
//
// Everything is integer work bound by memory traffic; no matrix cores.

#include "g10_internal.h"

#include <atomic>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

namespace {

constexpr int ITEMS = 8;                        // elements per thread in tiled kernels
constexpr int TILE = G10_BLOCK * ITEMS;         // 2048

// ===========================================================================
// device-wide exclusive scan
// ===========================================================================
// What the tiles before this one sum up to, from the tiles' own sums; with `all`, the sum of all of them.
// Up to DIRECT tiles every workgroup adds them up itself (8 loads a thread at most), so that no launch
// is needed in between; above that the sums are scanned first (`scanned`).  The line: 2048 tiles are
// 8 KB of sums a workgroup, read from L2 in about the time of the launch they save (3.5 us).
constexpr u32 DIRECT = 2048;
template <class T>
__device__ __forceinline__ T tile_base(const T* __restrict__ sums, u32 nb, bool scanned, T* tmp, T* all) {
  if (scanned) {
    if (all) *all = sums[nb];
    return sums[blockIdx.x];
  }
  T before = 0, total = 0;
  for (u32 i = threadIdx.x; i < nb; i += G10_BLOCK) {
    const T x = sums[i];
    if (i < blockIdx.x) before += x;
    total += x;
  }
  if (all) *all = block_sum(total, tmp);
  return block_sum(before, tmp);
}

// (max: where given, it is raised to the largest value of out[0..n])
template <class T>
__global__ __launch_bounds__(G10_BLOCK) void k_scan_tiles(const T* __restrict__ in, T* out, u64 n, T* sums, T* max) {
  __shared__ T tmp[G10_WAVES + 1];
  const u64 base = (u64)blockIdx.x * TILE + (u64)threadIdx.x * ITEMS;
  T v[ITEMS];
  T acc = 0;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    v[i] = base + i < n ? in[base + i] : (T)0;
    acc += v[i];
  }
  T total;
  T run = block_scan_excl(acc, tmp, total), top = total;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    if (base + i < n) { out[base + i] = run; top = run > top ? run : top; }
    run += v[i];
  }
  if (sums) { if (threadIdx.x == 0) sums[blockIdx.x] = total; return; }
  if (threadIdx.x == 0) out[n] = total;         // single tile: finished
  if (max) {
    top = block_max(top, tmp);
    if (threadIdx.x == 0) *max = top;
  }
}

template <class T>
__global__ __launch_bounds__(G10_BLOCK) void k_scan_add(T* out, u64 n, const T* __restrict__ sums, u32 nb, u32 scanned, T* max) {
  __shared__ T tmp[G10_WAVES + 1];
  T all;
  const T add = tile_base<T>(sums, nb, scanned != 0, tmp, &all);
  const u64 base = (u64)blockIdx.x * TILE + (u64)threadIdx.x * ITEMS;
  T top = 0;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if (base + i < n) {
      const T x = out[base + i] + add;
      out[base + i] = x;
      top = x > top ? x : top;
    }
  if (blockIdx.x == 0 && threadIdx.x == 0) { out[n] = all; top = all > top ? all : top; }
  if (max) {
    top = block_max(top, tmp);
    if (threadIdx.x == 0) {
      if constexpr (sizeof(T) == 8) atomicMax((unsigned long long*)max, (unsigned long long)top);
      else atomicMax(max, top);
    }
  }
}

// max: device word (cleared) that takes the largest value of out[0..n], or null
template <class T>
int scan_excl(const T* in, T* out, u64 n, T* scratch, hipStream_t s, T* max = nullptr) {
  if (n == 0) {                                  // out[0] = 0
    hipLaunchKernelGGL(k_scan_tiles<T>, dim3(1), dim3(G10_BLOCK), 0, s, in, out, n, (T*)nullptr, (T*)nullptr);
    G10_HIP(hipGetLastError());
    return G10_OK;
  }
  const u64 nb = (n + TILE - 1) / TILE;
  hipLaunchKernelGGL(k_scan_tiles<T>, dim3((u32)nb), dim3(G10_BLOCK), 0, s, in, out, n, nb == 1 ? (T*)nullptr : scratch, nb == 1 ? max : (T*)nullptr);
  G10_HIP(hipGetLastError());
  if (nb == 1) return G10_OK;
  if (nb > DIRECT) G10_TRY(scan_excl<T>(scratch, scratch, nb, scratch + nb + 1, s));
  hipLaunchKernelGGL(k_scan_add<T>, dim3((u32)nb), dim3(G10_BLOCK), 0, s, out, n, scratch, (u32)nb, nb > DIRECT ? 1u : 0u, max);
  G10_HIP(hipGetLastError());
  return G10_OK;
}

// ===========================================================================
// validation of array contents (one pass each, flags + wide sums)
// ===========================================================================
struct VitStats {
  u32 bad_index, zero_dur, zero_size, size_overflow;
  u32 big_size, pad;         // a tensor of 2^43 bytes or more
  u64 max_size;              // the largest tensor
  u64 dur_lo, dur_hi;        // sum of low / high 32-bit halves of the durations
  u64 used_lo, used_hi;      // same for the sizes of used tensors
  u64 n_uses, n_periods, peak;
};

__global__ __launch_bounds__(G10_BLOCK) void k_check_dur(const u64* __restrict__ dur, u32 K, VitStats* st) {
  __shared__ u64 tmp[G10_WAVES + 1];
  u64 lo = 0, hi = 0;
  u32 zero = 0;
  for (u64 i = (u64)blockIdx.x * G10_BLOCK + threadIdx.x; i < K; i += (u64)gridDim.x * G10_BLOCK) {
    u64 d = dur[i];
    zero |= d == 0;
    lo += d & 0xffffffffull;
    hi += d >> 32;
  }
  lo = block_sum(lo, tmp);
  hi = block_sum(hi, tmp);
  if (__any(zero) && lane_id() == 0) atomicOr(&st->zero_dur, 1u);
  if (threadIdx.x == 0) {
    atomicAdd((unsigned long long*)&st->dur_lo, (unsigned long long)lo);
    atomicAdd((unsigned long long*)&st->dur_hi, (unsigned long long)hi);
  }
}

// One pass over everything the caller gave: checks, own copies where planning follows (else dur_out is
// null), and the sort keys (tensor, kernel) of the pairs.  A pair that names no kernel or no tensor of the
// trace is reported and stands in as (0, 0): every later kernel then indexes inside its arrays, and the
// host rejects the trace when it reads the report at the end of the analysis.  Bound by HBM on a large
// trace, by its launch on a small one: it stands for seven launches (three copies, two checks, the keys,
// a clear), which with the fewer launches below took the analysis of an 80-pair trace from 140 to 84 us.
__global__ __launch_bounds__(G10_BLOCK) void k_load(const u64* __restrict__ dur, const u64* __restrict__ size, const uint8_t* __restrict__ glob,
                                                   const u32* __restrict__ uk, const u32* __restrict__ ut, u32 K, u32 N, u64 P, u32 kbits,
                                                   u64* __restrict__ dur_out, u64* __restrict__ size_out, uint8_t* __restrict__ glob_out,
                                                   u64* __restrict__ keys, VitStats* st) {
  __shared__ u64 tmp[G10_WAVES + 1];
  const u64 first = (u64)blockIdx.x * G10_BLOCK, step = (u64)gridDim.x * G10_BLOCK;
  if (first < K) {
    u64 lo = 0, hi = 0;
    u32 zero = 0;
    for (u64 i = first + threadIdx.x; i < K; i += step) {
      const u64 d = dur[i];
      if (dur_out) dur_out[i] = d;
      zero |= d == 0;
      lo += d & 0xffffffffull;
      hi += d >> 32;
    }
    lo = block_sum(lo, tmp);
    hi = block_sum(hi, tmp);
    if (__any(zero) && lane_id() == 0) atomicOr(&st->zero_dur, 1u);
    if (threadIdx.x == 0) {
      atomicAdd((unsigned long long*)&st->dur_lo, (unsigned long long)lo);
      if (hi) atomicAdd((unsigned long long*)&st->dur_hi, (unsigned long long)hi);
    }
  }
  if (first < N) {
    u32 zero = 0, ovf = 0, big = 0;
    u64 mx = 0;
    for (u64 i = first + threadIdx.x; i < N; i += step) {
      const u64 x = size[i];
      if (size_out) { size_out[i] = x; glob_out[i] = glob[i]; }
      mx = x > mx ? x : mx;
      zero |= x == 0;
      ovf |= x > 0xffffffffffffffffull / 1000ull;
      big |= (x >> 43) != 0;
    }
    if (__any(zero) && lane_id() == 0) atomicOr(&st->zero_size, 1u);
    if (__any(ovf) && lane_id() == 0) atomicOr(&st->size_overflow, 1u);
    if (__any(big) && lane_id() == 0) atomicOr(&st->big_size, 1u);
    // (atomics on one address queue up behind each other: one per workgroup, and only where it can still raise the maximum)
    mx = block_max(mx, tmp);
    if (threadIdx.x == 0 && mx > *(volatile u64*)&st->max_size) atomicMax((unsigned long long*)&st->max_size, (unsigned long long)mx);
  }
  u32 bad = 0;
  for (u64 i = first + threadIdx.x; i < P; i += step) {
    u32 k = uk[i], t = ut[i];
    if (k >= K || t >= N) { bad = 1; k = 0; t = 0; }
    keys[i] = ((u64)t << kbits) | k;
  }
  if (__any(bad) && lane_id() == 0) atomicOr(&st->bad_index, 1u);
}

// ===========================================================================
// use lists: radix sort, distinct
// ===========================================================================
// Tile layout of the sort kernels: wavefront w of a workgroup owns the
// contiguous keys [tile + w*512, tile + (w+1)*512); in round r lane l holds key
// tile + w*512 + r*64 + l.  Key order = (wavefront, round, lane): that is what
// makes the per-digit ranks stable.
__device__ __forceinline__ u64 tile_index(u32 r) {
  return (u64)blockIdx.x * TILE + (u64)wave_id() * (G10_WAVE * ITEMS) + (u64)r * G10_WAVE + lane_id();
}

// The two kernels of a sort pass; blockIdx.x is the tile (the batched forms below put the job in blockIdx.y).
template <class KT>
__device__ __forceinline__ void radix_hist_tile(const KT* __restrict__ keys, u64 P, u32 shift, u32* __restrict__ hist, u32 nblocks,
                                                u32* cnt, bool by_tile = false) {
  cnt[threadIdx.x] = 0;
  __syncthreads();
#pragma unroll
  for (u32 r = 0; r < ITEMS; ++r) {
    u64 i = tile_index(r);
    if (i < P) atomicAdd(&cnt[(keys[i] >> shift) & 255u], 1u);
  }
  __syncthreads();
  hist[by_tile ? blockIdx.x * 256u + threadIdx.x : (u64)threadIdx.x * nblocks + blockIdx.x] = cnt[threadIdx.x];     // else by digit
}

template <class KT>
__global__ __launch_bounds__(G10_BLOCK) void k_radix_hist(const KT* __restrict__ keys, u64 P, u32 shift,
                                                         u32* __restrict__ hist, u32 nblocks, u32 by_tile) {
  __shared__ u32 cnt[256];
  radix_hist_tile<KT>(keys, P, shift, hist, nblocks, cnt, by_tile != 0);
}

// Exclusive scan of one digit's counts over the tiles, in place, by one workgroup; the digit's total goes
// behind the counts (256 totals).  A row each for 256 workgroups and the digits' own scan in every scatter
// workgroup take one launch where a scan over all 256 * nblocks counts took three; one workgroup
// scanning all counts of a sort took about 100 us for a million keys.
__device__ __forceinline__ void radix_row_scan(u32* __restrict__ hist, u32 nblocks, u32 d, u32* tmp) {
  u32* row = hist + (u64)d * nblocks;
  u32 carry = 0;
  for (u32 b0 = 0; b0 < nblocks; b0 += TILE) {
    const u32 i = b0 + threadIdx.x * ITEMS;
    u32 v[ITEMS], sum = 0;
#pragma unroll
    for (u32 q = 0; q < ITEMS; ++q) { v[q] = i + q < nblocks ? row[i + q] : 0u; sum += v[q]; }
    u32 total;
    u32 run = carry + block_scan_excl(sum, tmp, total);
#pragma unroll
    for (u32 q = 0; q < ITEMS; ++q) {
      if (i + q < nblocks) row[i + q] = run;
      run += v[q];
    }
    carry += total;
  }
  if (threadIdx.x == 0) hist[(u64)256 * nblocks + d] = carry;
}
__global__ __launch_bounds__(G10_BLOCK) void k_radix_rows(u32* __restrict__ hist, u32 nblocks) {
  __shared__ u32 tmp[G10_WAVES + 1];
  radix_row_scan(hist, nblocks, blockIdx.x, tmp);
}

template <class KT, bool PAIRS>
__device__ __forceinline__ void radix_scatter_tile(const KT* __restrict__ keys, KT* __restrict__ out,
                                                   const u32* __restrict__ vals, u32* __restrict__ vout,
                                                   u64 P, u32 shift, const u32* __restrict__ offs,
                                                   u32 nblocks, u32 (*cnt)[256], u32* gbase, u32* tmp, bool by_tile = false) {
  for (u32 i = threadIdx.x; i < G10_WAVES * 256; i += G10_BLOCK) (&cnt[0][0])[i] = 0;
  // counts by tile, not scanned yet (few tiles): a thread per digit adds them up
  u32 earlier = 0, every = 0;
  if (by_tile) {
#pragma unroll 8
    for (u32 b = 0; b < nblocks; ++b) {
      const u32 x = offs[b * 256u + threadIdx.x];
      earlier += b < blockIdx.x ? x : 0u;
      every += x;
    }
  }
  __syncthreads();
  const u32 w = wave_id(), l = lane_id();
  const u64 lt = (1ull << l) - 1ull;
  KT key[ITEMS];
  u32 rank[ITEMS], val[ITEMS];
#pragma unroll
  for (u32 r = 0; r < ITEMS; ++r) {
    const u64 i = tile_index(r);
    const bool ok = i < P;
    key[r] = ok ? keys[i] : (KT)0;
    val[r] = PAIRS && ok ? (vals ? vals[i] : (u32)i) : 0u;     // no values given: the positions themselves
    const u32 dig = (u32)(key[r] >> shift) & 255u;
    u64 peers = __ballot(ok);
#pragma unroll
    for (u32 b = 0; b < 8; ++b) {
      const u64 m = __ballot((dig >> b) & 1u);
      peers &= ((dig >> b) & 1u) ? m : ~m;
    }
    const u32 before = cnt[w][dig];          // all peers read, then the first one adds
    rank[r] = before + __popcll(peers & lt);
    __builtin_amdgcn_wave_barrier();
    if (ok && (peers & lt) == 0) cnt[w][dig] = before + __popcll(peers);
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  {                                           // one thread per digit: offsets of the wavefronts, and where the tile's keys of the digit go
    const u32 d = threadIdx.x;
    u32 all;
    const u32 before = block_scan_excl(by_tile ? every : offs[(u64)256 * nblocks + d], tmp, all);      // keys of lower digits
    u32 run = 0;
#pragma unroll
    for (u32 ww = 0; ww < G10_WAVES; ++ww) {
      u32 c = cnt[ww][d];
      cnt[ww][d] = run;
      run += c;
    }
    gbase[d] = before + (by_tile ? earlier : offs[(u64)d * nblocks + blockIdx.x]);
  }
  __syncthreads();
#pragma unroll
  for (u32 r = 0; r < ITEMS; ++r) {
    const u64 i = tile_index(r);
    if (i < P) {
      const u32 dig = (u32)(key[r] >> shift) & 255u;
      const u64 pos = (u64)gbase[dig] + cnt[w][dig] + rank[r];
      out[pos] = key[r];
      if (PAIRS) vout[pos] = val[r];
    }
  }
}

template <class KT, bool PAIRS>
__global__ __launch_bounds__(G10_BLOCK) void k_radix_scatter(const KT* __restrict__ keys, KT* __restrict__ out,
                                                            const u32* __restrict__ vals, u32* __restrict__ vout,
                                                            u64 P, u32 shift, const u32* __restrict__ offs,
                                                            u32 nblocks, u32 by_tile) {
  __shared__ u32 cnt[G10_WAVES][256];        // per wavefront: running count per digit
  __shared__ u32 gbase[256];
  __shared__ u32 tmp[G10_WAVES + 1];
  radix_scatter_tile<KT, PAIRS>(keys, out, vals, vout, P, shift, offs, nblocks, cnt, gbase, tmp, by_tile != 0);
}

// ---- a sort of at most SMALL keys in one launch ---------------------------------------------------------
// One workgroup of 16 wavefronts holds the keys in registers and orders them through LDS, all digits in
// turn: the passes of a small sort are bound by their launches (three each, 3 to 4 us apiece), not by
// their keys.  The limit is what LDS takes with 64-bit keys and values beside them.
constexpr u32 SMALL_WAVES = 16, SMALL = SMALL_WAVES * G10_WAVE * ITEMS;      // 8192
constexpr u32 RADIX_DIRECT = 64;
template <class KT, bool PAIRS>
struct SmallSort {
  KT key[SMALL];
  u32 val[PAIRS ? SMALL : 1];
  u32 cnt[SMALL_WAVES][256];
  u32 tmp[SMALL_WAVES];
};
template <class KT, bool PAIRS>
__global__ __launch_bounds__(SMALL_WAVES * G10_WAVE) void k_radix_small(const KT* __restrict__ keys, KT* __restrict__ out,
                                                                       const u32* __restrict__ vals, u32* __restrict__ vout, u32 n,
                                                                       u32 first_bit, u32 bits) {
  extern __shared__ __align__(16) unsigned char smem[];
  SmallSort<KT, PAIRS>& S = *(SmallSort<KT, PAIRS>*)smem;
  const u32 tid = threadIdx.x, w = tid >> 6, l = tid & 63u;
  const u64 lt = (1ull << l) - 1ull;
  const u32 rounds = (n + SMALL_WAVES * G10_WAVE - 1) / (SMALL_WAVES * G10_WAVE);   // keys per lane; a wavefront owns rounds * 64 neighbours
  const u32 first = w * rounds * G10_WAVE + l;
  KT key[ITEMS];
  u32 val[ITEMS], rank[ITEMS];
#pragma unroll
  for (u32 r = 0; r < ITEMS; ++r) {
    const u32 i = first + r * G10_WAVE;
    const bool ok = r < rounds && i < n;
    key[r] = ok ? keys[i] : (KT)0;
    val[r] = PAIRS && ok ? (vals ? vals[i] : i) : 0u;          // no values given: the positions themselves
  }
  for (u32 shift = first_bit; shift < bits; shift += 8) {
    for (u32 i = tid; i < SMALL_WAVES * 256; i += SMALL_WAVES * G10_WAVE) (&S.cnt[0][0])[i] = 0;
    __syncthreads();
#pragma unroll
    for (u32 r = 0; r < ITEMS; ++r) {
      if (r >= rounds) break;
      const bool ok = first + r * G10_WAVE < n;
      const u32 dig = (u32)(key[r] >> shift) & 255u;
      u64 peers = __ballot(ok);
#pragma unroll
      for (u32 b = 0; b < 8; ++b) {
        const u64 m = __ballot((dig >> b) & 1u);
        peers &= ((dig >> b) & 1u) ? m : ~m;
      }
      const u32 before = S.cnt[w][dig];
      rank[r] = before + (u32)__popcll(peers & lt);
      __builtin_amdgcn_wave_barrier();
      if (ok && (peers & lt) == 0) S.cnt[w][dig] = before + (u32)__popcll(peers);
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    u32 total = 0, inc = 0;
    if (tid < 256) {                          // a digit per thread: its count, then where its keys begin
      for (u32 x = 0; x < SMALL_WAVES; ++x) { const u32 c = S.cnt[x][tid]; S.cnt[x][tid] = total; total += c; }
      inc = wave_scan_incl(total);
      if (l == G10_WAVE - 1) S.tmp[w] = inc;
    }
    __syncthreads();
    if (tid < 256) {
      u32 base = inc - total;
      for (u32 x = 0; x < w; ++x) base += S.tmp[x];
      for (u32 x = 0; x < SMALL_WAVES; ++x) S.cnt[x][tid] += base;
    }
    __syncthreads();
#pragma unroll
    for (u32 r = 0; r < ITEMS; ++r) {
      if (r >= rounds) break;
      if (first + r * G10_WAVE < n) {
        const u32 pos = S.cnt[w][(u32)(key[r] >> shift) & 255u] + rank[r];
        S.key[pos] = key[r];
        if (PAIRS) S.val[pos] = val[r];
      }
    }
    __syncthreads();
#pragma unroll
    for (u32 r = 0; r < ITEMS; ++r) {
      if (r >= rounds) break;
      const u32 i = first + r * G10_WAVE;
      if (i < n) { key[r] = S.key[i]; if (PAIRS) val[r] = S.val[i]; }
    }
    // (the next pass writes the keys behind three more barriers)
  }
#pragma unroll
  for (u32 r = 0; r < ITEMS; ++r) {
    const u32 i = first + r * G10_WAVE;
    if (r < rounds && i < n) { out[i] = key[r]; if (PAIRS) vout[i] = val[r]; }
  }
}

// ---- many sorts of (32-bit key, 32-bit value) pairs at once: job = blockIdx.y -------------------------
__device__ __forceinline__ SortJob in_global(SortJob j) {
  j.keys = ::in_global(j.keys); j.alt = ::in_global(j.alt); j.vals = ::in_global(j.vals); j.valt = ::in_global(j.valt); j.hist = ::in_global(j.hist);
  return j;
}
__global__ __launch_bounds__(G10_BLOCK) void k_radix_hist_jobs(const SortJob* __restrict__ jobs, u32 shift, u32 flip) {
  __shared__ u32 cnt[256];
  const SortJob j = in_global(jobs[blockIdx.y]);
  if (blockIdx.x >= j.nb) return;
  radix_hist_tile<u32>(flip ? j.alt : j.keys, j.n, shift, j.hist, j.nb, cnt);
}

__global__ __launch_bounds__(G10_BLOCK) void k_radix_rows_jobs(const SortJob* __restrict__ jobs) {
  __shared__ u32 tmp[G10_WAVES + 1];
  const SortJob j = in_global(jobs[blockIdx.y]);
  radix_row_scan(j.hist, j.nb, blockIdx.x, tmp);
}

__global__ __launch_bounds__(G10_BLOCK) void k_radix_scatter_jobs(const SortJob* __restrict__ jobs, u32 shift, u32 flip, u32 iota) {
  __shared__ u32 cnt[G10_WAVES][256];
  __shared__ u32 gbase[256];
  __shared__ u32 tmp[G10_WAVES + 1];
  const SortJob j = in_global(jobs[blockIdx.y]);
  if (blockIdx.x >= j.nb) return;
  radix_scatter_tile<u32, true>(flip ? j.alt : j.keys, flip ? j.keys : j.alt, iota ? (const u32*)nullptr : (const u32*)(flip ? j.valt : j.vals),
                                flip ? j.vals : j.valt, j.n, shift, j.hist, j.nb, cnt, gbase, tmp);
}

// The sorted keys without duplicates, tile by tile: how many of a tile stay (one tile: not needed), then
// the keys and kernels that stay behind those of the tiles before.  The flags are made twice instead of
// written out, scanned and read back: two launches and two passes over the keys where five launches made
// four (243 000 pairs: analysis 242 -> 181 us with the same for the periods).
template <class F>
__device__ __forceinline__ void tile_count(u64 n, u32* __restrict__ sums, F&& of) {
  __shared__ u32 tmp[G10_WAVES + 1];
  const u64 base = (u64)blockIdx.x * TILE + threadIdx.x;
  u32 c = 0;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if (base + (u64)i * G10_BLOCK < n) c += of(base + (u64)i * G10_BLOCK);
  c = block_sum(c, tmp);
  if (threadIdx.x == 0) sums[blockIdx.x] = c;
}
__device__ __forceinline__ u32 is_distinct(const u64* __restrict__ keys, u64 i) { return i == 0 || keys[i] != keys[i - 1] ? 1u : 0u; }
__global__ __launch_bounds__(G10_BLOCK) void k_distinct_count(const u64* __restrict__ keys, u64 P, u32* __restrict__ sums) {
  tile_count(P, sums, [&](u64 i) { return is_distinct(keys, i); });
}
__global__ __launch_bounds__(G10_BLOCK) void k_distinct_write(const u64* __restrict__ keys, u64 P, const u32* __restrict__ sums, u32 nb,
                                                             u32 scanned, u64* __restrict__ ukeys, u32* __restrict__ use_k, u32 kbits,
                                                             VitStats* st) {
  __shared__ u32 tmp[G10_WAVES + 1];
  u32 all = 0, at = nb > 1 ? tile_base<u32>(sums, nb, scanned != 0, tmp, &all) : 0u;
  const u64 first = (u64)blockIdx.x * TILE;
  for (u32 r = 0; r < ITEMS; ++r) {            // 256 neighbouring keys at a time
    const u64 i = first + r * G10_BLOCK + threadIdx.x;
    const bool keep = i < P && is_distinct(keys, i);
    u32 total;
    const u32 pos = at + block_scan_excl(keep ? 1u : 0u, tmp, total);
    if (keep) {
      const u64 k = keys[i];
      ukeys[pos] = k;
      use_k[pos] = (u32)(k & ((1ull << kbits) - 1ull));
    }
    at += total;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) st->n_uses = nb > 1 ? all : at;
}

// use_off[t] = first position whose key has tensor >= t  (t in [0, N])
__global__ __launch_bounds__(G10_BLOCK) void k_use_off(const u64* __restrict__ ukeys, const u64* __restrict__ n_uses_p,
                                                      u32 N, u32 kbits, u64* __restrict__ use_off) {
  const u64 n = *n_uses_p;
  for (u64 t = (u64)blockIdx.x * G10_BLOCK + threadIdx.x; t <= N; t += (u64)gridDim.x * G10_BLOCK) {
    const u64 want = t << kbits;
    u64 lo = 0, hi = n;
    while (lo < hi) {
      u64 mid = (lo + hi) >> 1;
      if (ukeys[mid] >= want) hi = mid; else lo = mid + 1;
    }
    use_off[t] = lo;
  }
}

// ===========================================================================
// inactive periods: adjacent difference inside each tensor's use list
// ===========================================================================
// Position i of the distinct keys ends an in-iteration period when its
// predecessor is the same tensor at least two kernels earlier; the last use of
// a global tensor additionally starts the cross-iteration period.
__device__ __forceinline__ void period_at(const u64* ukeys, const u64* use_off, const uint8_t* glob, u64 i, u32 K,
                                          u32 kbits, u32 no_wrap, bool& inner, bool& wrap, u32& t, u32& k, u32& kprev,
                                          u32& kfirst) {
  const u64 key = ukeys[i];
  const u64 kmask = (1ull << kbits) - 1ull;
  t = (u32)(key >> kbits);
  k = (u32)(key & kmask);
  const u64 b = use_off[t], e = use_off[t + 1];
  inner = false;
  wrap = false;
  kprev = 0;
  kfirst = 0;
  if (i > b) {
    kprev = (u32)(ukeys[i - 1] & kmask);
    inner = k - kprev >= 2;
  }
  if (i + 1 == e && glob[t] && !no_wrap) {
    kfirst = (u32)(ukeys[b] & kmask);
    wrap = (u64)kfirst + K - k >= 2;
  }
}

__global__ __launch_bounds__(G10_BLOCK) void k_period_count(const u64* __restrict__ ukeys, const u64* __restrict__ use_off,
                                                           const uint8_t* __restrict__ glob, const u64* __restrict__ n_uses_p,
                                                           u32 K, u32 kbits, u32 no_wrap, u32* __restrict__ sums) {
  tile_count(*n_uses_p, sums, [&](u64 i) {
    bool inner, wrap;
    u32 t, k, kp, kf;
    period_at(ukeys, use_off, glob, i, K, kbits, no_wrap, inner, wrap, t, k, kp, kf);
    return (u32)inner + (u32)wrap;
  });
}

__global__ __launch_bounds__(G10_BLOCK) void k_period_write(const u64* __restrict__ ukeys, const u64* __restrict__ use_off,
                                                           const uint8_t* __restrict__ glob, u32 K, u32 kbits, u32 no_wrap,
                                                           const u32* __restrict__ sums, u32 nb, u32 scanned,
                                                           u32* __restrict__ per_t, u32* __restrict__ per_L,
                                                           u32* __restrict__ per_R, VitStats* st) {
  __shared__ u32 tmp[G10_WAVES + 1];
  const u64 n = st->n_uses, first = (u64)blockIdx.x * TILE;
  u32 all = 0, at = nb > 1 ? tile_base<u32>(sums, nb, scanned != 0, tmp, &all) : 0u;
  for (u32 r = 0; r < ITEMS; ++r) {            // 256 neighbouring uses at a time
    const u64 i = first + r * G10_BLOCK + threadIdx.x;
    bool inner = false, wrap = false;
    u32 t = 0, k = 0, kp = 0, kf = 0;
    if (i < n) period_at(ukeys, use_off, glob, i, K, kbits, no_wrap, inner, wrap, t, k, kp, kf);
    u32 total;
    u32 o = at + block_scan_excl((u32)inner + (u32)wrap, tmp, total);
    if (inner) { per_t[o] = t; per_L[o] = kp; per_R[o] = k; ++o; }
    if (wrap) { per_t[o] = t; per_L[o] = k; per_R[o] = kf + K; }
    at += total;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) st->n_periods = nb > 1 ? all : at;
}

// the periods gathered in the order of their start (order[i]: index of the i-th) as {L, R, tensor, index}
__global__ __launch_bounds__(G10_BLOCK) void k_gather_periods(const u32* __restrict__ order, u64 C,
                                                             const u32* __restrict__ per_t, const u32* __restrict__ per_L,
                                                             const u32* __restrict__ per_R, const u64* __restrict__ size,
                                                             uint4* __restrict__ out, u64* __restrict__ out_size) {
  for (u64 i = (u64)blockIdx.x * G10_BLOCK + threadIdx.x; i < C; i += (u64)gridDim.x * G10_BLOCK) {
    const u32 c = order[i];
    const u32 t = per_t[c];
    out[i] = make_uint4(per_L[c], per_R[c], t, c);
    out_size[i] = size[t];
  }
}

// ===========================================================================
// memory pressure: interval adds into a difference array, scan, max
// ===========================================================================
__global__ __launch_bounds__(G10_BLOCK) void k_begin(VitStats* st, u64* __restrict__ diff, u64 n) {   // both cleared
  if (blockIdx.x == 0 && threadIdx.x < sizeof(VitStats) / 8) ((u64*)st)[threadIdx.x] = 0;
  for (u64 i = (u64)blockIdx.x * G10_BLOCK + threadIdx.x; i < n; i += (u64)gridDim.x * G10_BLOCK) diff[i] = 0;
}

__device__ __forceinline__ void lifetime_adds(const u64* ukeys, const u64* use_off, const u64* __restrict__ size, const uint8_t* __restrict__ glob,
                                              u32 N, u32 K, u32 kbits, u64* diff, VitStats* st, u64* tmp) {
  const u64 kmask = (1ull << kbits) - 1ull;
  u64 gsum = 0, lo32 = 0, hi32 = 0;
  for (u64 t = (u64)blockIdx.x * G10_BLOCK + threadIdx.x; t < N; t += (u64)gridDim.x * G10_BLOCK) {
    const u64 b = use_off[t], e = use_off[t + 1];
    if (b == e) continue;                       // never used: ignored everywhere
    const u64 s = size[t];
    lo32 += s & 0xffffffffull;
    hi32 += s >> 32;
    if (glob[t]) {
      gsum += s;                                // resident in every slot
    } else {
      const u32 birth = (u32)(ukeys[b] & kmask), death = (u32)(ukeys[e - 1] & kmask);
      atomicAdd((unsigned long long*)&diff[birth], (unsigned long long)s);
      atomicAdd((unsigned long long*)&diff[death + 1], (unsigned long long)(0ull - s));
    }
  }
  gsum = block_sum(gsum, tmp);
  lo32 = block_sum(lo32, tmp);
  hi32 = block_sum(hi32, tmp);
  if (threadIdx.x == 0) {
    if (gsum) {
      atomicAdd((unsigned long long*)&diff[0], (unsigned long long)gsum);
      atomicAdd((unsigned long long*)&diff[K], (unsigned long long)(0ull - gsum));
    }
    atomicAdd((unsigned long long*)&st->used_lo, (unsigned long long)lo32);
    atomicAdd((unsigned long long*)&st->used_hi, (unsigned long long)hi32);
  }
}
__global__ __launch_bounds__(G10_BLOCK) void k_lifetime_adds(const u64* __restrict__ ukeys, const u64* __restrict__ use_off,
                                                            const u64* __restrict__ size, const uint8_t* __restrict__ glob,
                                                            u32 N, u32 K, u32 kbits, u64* diff, VitStats* st) {
  __shared__ u64 tmp[G10_WAVES + 1];
  lifetime_adds(ukeys, use_off, size, glob, N, K, kbits, diff, st, tmp);
}

// ===========================================================================
// distinct uses, use lists, periods and pressure of a trace of one tile of pairs, by one workgroup in one launch (six
// otherwise, 4 us each where they have nothing to do).  The limits: one tile of pairs; a few rounds of the workgroup
// over tensors and kernels.  Analysis of 189 pairs 96 -> 67 us, step of the 80-pair trace 399 -> 339.
// ===========================================================================
constexpr u32 TINY = 4096;
__global__ __launch_bounds__(G10_BLOCK) void k_tiny(const u64* __restrict__ keys, u32 P, u32 K, u32 N, u32 kbits, u32 no_wrap,
                                                   const u64* __restrict__ size, const uint8_t* __restrict__ glob, u64* ukeys, u32* use_k,
                                                   u64* use_off, u32* per_t, u32* per_L, u32* per_R, u64* diff, VitStats* st) {
  __shared__ u32 tmp[G10_WAVES + 1];
  __shared__ u64 tmp64[G10_WAVES + 1];
  const u64 kmask = (1ull << kbits) - 1ull;
  u32 n = 0;
  for (u32 r = 0; r < ITEMS; ++r) {               // distinct uses
    const u32 i = r * G10_BLOCK + threadIdx.x;
    const u64 k = i < P ? keys[i] : 0ull;
    const bool is_new = i < P && (i == 0 || keys[i - 1] != k);
    u32 total;
    const u32 o = n + block_scan_excl((u32)is_new, tmp, total);
    if (is_new) { ukeys[o] = k; use_k[o] = (u32)(k & kmask); }
    n += total;
  }
  __syncthreads();
  for (u32 t = threadIdx.x; t <= N; t += G10_BLOCK) {      // use lists
    const u64 key = (u64)t << kbits;
    u32 lo = 0, hi = n;
    while (lo < hi) { const u32 mid = (lo + hi) / 2; if (ukeys[mid] < key) lo = mid + 1; else hi = mid; }
    use_off[t] = lo;
  }
  __syncthreads();
  u32 at = 0;
  for (u32 r = 0; r < ITEMS; ++r) {               // periods
    const u32 i = r * G10_BLOCK + threadIdx.x;
    bool inner = false, wrap = false;
    u32 t = 0, k = 0, kp = 0, kf = 0;
    if (i < n) period_at(ukeys, use_off, glob, i, K, kbits, no_wrap, inner, wrap, t, k, kp, kf);
    u32 total;
    u32 o = at + block_scan_excl((u32)inner + (u32)wrap, tmp, total);
    if (inner) { per_t[o] = t; per_L[o] = kp; per_R[o] = k; ++o; }
    if (wrap) { per_t[o] = t; per_L[o] = k; per_R[o] = kf + K; }
    at += total;
  }
  if (threadIdx.x == 0) { st->n_uses = n; st->n_periods = at; }
  lifetime_adds(ukeys, use_off, size, glob, N, K, kbits, diff, st, tmp64);
  __syncthreads();
  u64 carry = 0, top = 0;                         // diff[0..K] into its exclusive sums, in place; their largest is the peak
  for (u32 b0 = 0; b0 <= K; b0 += TILE) {
    u64 v[ITEMS], acc = 0;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const u32 j = b0 + threadIdx.x * ITEMS + i;
      v[i] = j < K ? __hip_atomic_load(&diff[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
      acc += v[i];
    }
    u64 total, run = block_scan_excl(acc, tmp64, total);
    run += carry;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const u32 j = b0 + threadIdx.x * ITEMS + i;
      if (j <= K) { diff[j] = run; top = run > top ? run : top; }
      run += v[i];
    }
    carry += total;
  }
  top = block_max(top, tmp64);
  if (threadIdx.x == 0) st->peak = top;
}

// ===========================================================================
// the verdict and the results of g10_vitality_static
// ===========================================================================
__host__ __device__ inline int verdict_of(const VitStats& v) {
  if (v.bad_index || v.zero_dur || v.zero_size) return G10_EINVAL;
  if (v.size_overflow) return G10_EOVERFLOW;
  const unsigned __int128 T = ((unsigned __int128)v.dur_hi << 32) + v.dur_lo, used = ((unsigned __int128)v.used_hi << 32) + v.used_lo;
  return (T >> 62) || (used >> 64) ? G10_EOVERFLOW : G10_OK;
}

// The caller's buffers take the results only if the trace stands (the host learns that later): one launch
// and one synchronisation where seven copies followed the first synchronisation and a second one them.
__global__ __launch_bounds__(G10_BLOCK) void k_results_out(const VitStats* __restrict__ st, g10_vitality_buffers out, u32 K, u32 N,
                                                          const u64* __restrict__ use_off, const u32* __restrict__ use_k,
                                                          const u32* __restrict__ per_t, const u32* __restrict__ per_L,
                                                          const u32* __restrict__ per_R, const u64* __restrict__ start,
                                                          const u64* __restrict__ pressure) {
  const VitStats v = *st;
  if (verdict_of(v)) return;
  const u64 first = (u64)blockIdx.x * G10_BLOCK + threadIdx.x, step = (u64)gridDim.x * G10_BLOCK;
  for (u64 i = first; i <= N; i += step) out.use_off[i] = use_off[i];
  for (u64 i = first; i <= K; i += step) out.start[i] = start[i];
  for (u64 i = first; i < K; i += step) out.pressure[i] = pressure[i];
  for (u64 i = first; i < v.n_uses; i += step) out.use_k[i] = use_k[i];
  for (u64 i = first; i < v.n_periods; i += step) { out.per_tensor[i] = per_t[i]; out.per_L[i] = per_L[i]; out.per_R[i] = per_R[i]; }
}

inline u32 grid_for(u64 n, u32 cap = 4096) {
  u64 g = (n + G10_BLOCK - 1) / G10_BLOCK;
  return (u32)(g < 1 ? 1 : (g > cap ? cap : g));
}

inline u32 bits_for(u64 max_value) {            // bits needed to hold values 0..max_value, at least 1
  u32 b = 1;
  while (b < 64 && (max_value >> b)) ++b;
  return b;
}

// One device allocation carved into arrays (every hipMalloc / hipFree costs about 0.1 ms of host
// time, and the analysis needs twenty arrays).
struct Pool {
  char* base = nullptr;
  size_t off = 0, cap = 0;
  static size_t need(u64 elems, size_t size) { return (((elems ? elems : 1) * size) + 255) & ~(size_t)255; }
  int reserve(size_t bytes) {
    void* q = nullptr;
    G10_TRY(mem_dev_alloc(&q, bytes));
    base = (char*)q; cap = bytes; off = 0;
    return G10_OK;
  }
  template <class T>
  int take(T** out, u64 elems) {
    const size_t b = need(elems, sizeof(T));
    if (off + b > cap) return G10_ENOMEM;
    *out = (T*)(base + off);
    off += b;
    return G10_OK;
  }
};

}  // namespace

size_t scan_scratch_elems(u64 n) {
  size_t tot = 0;
  while (n > (u64)TILE) {
    n = (n + TILE - 1) / TILE;
    tot += n + 1;
  }
  return tot + 2;
}
int scan_excl_u32(const u32* in, u32* out, u64 n, u32* scratch, hipStream_t s) { return scan_excl<u32>(in, out, n, scratch, s); }
int scan_excl_u64(const u64* in, u64* out, u64 n, u64* scratch, hipStream_t s) { return scan_excl<u64>(in, out, n, scratch, s); }

int g10_hip_fail(hipError_t e, const char* file, int line) {
  if (getenv("G10_LOG")) fprintf(stderr, "g10: HIP error %d (%s) at %s:%d\n", (int)e, hipGetErrorString(e), file, line);
  (void)hipGetLastError();
  return e == hipErrorOutOfMemory ? G10_ENOMEM : G10_EDEVICE;
}


size_t radix_hist_elems(u64 n) { return (size_t)256 * ((n + TILE - 1) / TILE ? (n + TILE - 1) / TILE : 1) + 256; }

template <class KT, bool PAIRS>
static int radix_small(const KT* keys, KT* out, const u32* vals, u32* vout, u64 n, u32 first_bit, u32 bits, hipStream_t s) {
  constexpr size_t lds = sizeof(SmallSort<KT, PAIRS>);
  static_assert(lds <= 160 * 1024, "the LDS of one workgroup");
  static std::atomic<bool> allowed[64];           // (per device: the attribute belongs to the kernel)
  int dev = 0;
  G10_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64 || !allowed[dev].load(std::memory_order_acquire)) {
    G10_HIP(hipFuncSetAttribute((const void*)k_radix_small<KT, PAIRS>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    if (dev >= 0 && dev < 64) allowed[dev].store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL((k_radix_small<KT, PAIRS>), dim3(1), dim3(SMALL_WAVES * G10_WAVE), lds, s, keys, out, vals, vout, (u32)n, first_bit, bits);
  G10_HIP(hipGetLastError());
  return G10_OK;
}

// LSD radix sort of KT keys by their bits first_bit .. bits - 1, 8 bits per pass, stable; PAIRS: with a 32-bit value carried
// along with every key (iota: the values are the positions 0..n-1 and *vals need not be filled).
// On return *keys points at the sorted keys and *alt at the other buffer, *vals / *valt likewise.
// hist: radix_hist_elems(n) words.  src: where given, the keys are read from there and *keys need not be filled.
template <class KT, bool PAIRS>
static int radix_sort(KT** keys, KT** alt, u32** vals, u32** valt, u64 n, u32 bits, u32* hist, hipStream_t s, bool iota, const KT* src = nullptr,
                      u32 first_bit = 0) {
  if (n == 0) return G10_OK;
  auto swap = [&]() {
    KT* t = *keys; *keys = *alt; *alt = t;
    if (PAIRS) { u32* v = *vals; *vals = *valt; *valt = v; }
  };
  if (n <= SMALL) {
    const u32* v = PAIRS && !iota ? *vals : nullptr;
    G10_TRY((radix_small<KT, PAIRS>(src ? src : *keys, *alt, v, PAIRS ? *valt : nullptr, n, first_bit, bits, s)));
    swap();
    return G10_OK;
  }
  const u32 nb = (u32)((n + TILE - 1) / TILE);
  // Few tiles: every scatter workgroup adds the counts of the tiles up itself (nb rows of 1 KB from L2, all in flight at
  // once) and the launch in between falls away.  Analysis of 22 642 pairs 181 -> 160 us, 118 055 pairs (58 tiles) 214 -> 202;
  // of 243 340 (119 tiles) 234 -> 240, so from 64 tiles on the counts are scanned in a launch of their own.
  const u32 by_tile = nb <= RADIX_DIRECT ? 1u : 0u;
  for (u32 shift = first_bit; shift < bits; shift += 8) {
    const KT* from = src && shift == first_bit ? src : *keys;
    hipLaunchKernelGGL(k_radix_hist<KT>, dim3(nb), dim3(G10_BLOCK), 0, s, from, n, shift, hist, nb, by_tile);
    if (!by_tile) hipLaunchKernelGGL(k_radix_rows, dim3(256), dim3(G10_BLOCK), 0, s, hist, nb);
    const u32* v = PAIRS && !(iota && shift == first_bit) ? *vals : nullptr;
    hipLaunchKernelGGL((k_radix_scatter<KT, PAIRS>), dim3(nb), dim3(G10_BLOCK), 0, s, from, *alt, v, PAIRS ? *valt : nullptr, n,
                       shift, hist, nb, by_tile);
    swap();
  }
  G10_HIP(hipGetLastError());
  return G10_OK;
}
int radix_sort_u64(u64** keys, u64** alt, u64 n, u32 bits, u32* hist, hipStream_t s, u32 first_bit) {
  return radix_sort<u64, false>(keys, alt, nullptr, nullptr, n, bits, hist, s, false, nullptr, first_bit);
}
int radix_sort_u64_pairs(u64** keys, u64** alt, u32** vals, u32** valt, u64 n, u32 bits, u32* hist, hipStream_t s, bool iota) {
  return radix_sort<u64, true>(keys, alt, vals, valt, n, bits, hist, s, iota);
}
// (the score order of the planner's candidates)
int radix_sort_u32_pairs(u32** keys, u32** alt, u32** vals, u32** valt, u64 n, u32 bits, u32* hist, hipStream_t s, bool iota) {
  return radix_sort<u32, true>(keys, alt, vals, valt, n, bits, hist, s, iota);
}

// `njobs` sorts of pairs in the same launches (jobs: device array; max_nb: the largest nb among them).  The
// sorted pairs of a job end in (keys, vals) after an even number of passes, in (alt, valt) after an odd one;
// iota: the values are the positions 0..n-1 (vals need not be filled).  Every job has n > 0.
u32 radix_blocks(u64 n) { return (u32)((n + TILE - 1) / TILE); }
int radix_sort_u32_pairs_jobs(const SortJob* jobs, u32 njobs, u32 max_nb, u32 bits, bool iota, hipStream_t s) {
  if (njobs == 0 || max_nb == 0) return G10_OK;
  u32 flip = 0;
  for (u32 shift = 0; shift < bits; shift += 8, flip ^= 1u) {
    hipLaunchKernelGGL(k_radix_hist_jobs, dim3(max_nb, njobs), dim3(G10_BLOCK), 0, s, jobs, shift, flip);
    hipLaunchKernelGGL(k_radix_rows_jobs, dim3(256, njobs), dim3(G10_BLOCK), 0, s, jobs);
    hipLaunchKernelGGL(k_radix_scatter_jobs, dim3(max_nb, njobs), dim3(G10_BLOCK), 0, s, jobs, shift, flip, iota && shift == 0 ? 1u : 0u);
  }
  G10_HIP(hipGetLastError());
  return G10_OK;
}

// Durations given for one plan instead of the analysed trace's: own copy, the same checks as
// the analysis makes, slot start times.  `stats_dev` is 128 bytes of device memory, `check` 128
// bytes of host memory that slot_times_end reads once the stream has been synchronised.
static_assert(sizeof(VitStats) <= 128, "the callers keep 128 bytes for the checks");
int slot_times_begin(const u64* src, u32 K, u64* dur, u64* start, u64* scratch64, void* stats_dev, void* check,
                     hipStream_t s) {
  VitStats* st = (VitStats*)stats_dev;
  G10_HIP(hipMemsetAsync(st, 0, sizeof(VitStats), s));
  G10_HIP(hipMemcpyAsync(dur, src, (u64)K * 8, hipMemcpyDeviceToDevice, s));
  hipLaunchKernelGGL(k_check_dur, dim3(grid_for(K)), dim3(G10_BLOCK), 0, s, (const u64*)dur, K, st);
  G10_HIP(hipGetLastError());
  G10_HIP(hipMemcpyAsync(check, st, sizeof(VitStats), hipMemcpyDeviceToHost, s));
  return scan_excl_u64(dur, start, K, scratch64, s);
}

int slot_times_end(const void* check, u64* T_out) {
  VitStats hs;
  memcpy(&hs, check, sizeof hs);
  if (hs.zero_dur) return G10_EINVAL;
  const unsigned __int128 T = ((unsigned __int128)hs.dur_hi << 32) + hs.dur_lo;
  if (T >> 62) return G10_EOVERFLOW;
  *T_out = (u64)T;
  return G10_OK;
}

// Device memory an analysis of K kernels, N tensors and P pairs takes: the temporaries of the call,
// and what outlives it (`planning`: with own copies of the trace's arrays and the periods in the
// order of their start, which only planning needs).
// (a sum per tile, its total, and the scratch of a scan over them)
static u64 tile_sums_elems(u64 n) { const u64 nb = (n + TILE - 1) / TILE; return nb + 1 + scan_scratch_elems(nb); }
static size_t vit_tmp_bytes(u32 K, u32 N, u64 P) {
  const u64 ss_kn = scan_scratch_elems(K > N ? K : N), rh = radix_hist_elems(P), ss_p = tile_sums_elems(P);
  return Pool::need(1, sizeof(VitStats)) + Pool::need(ss_kn, 8) + 2 * Pool::need(P, 8) + Pool::need(rh, 4) + 2 * Pool::need(ss_p, 4);
}
static size_t vit_keep_bytes(u32 K, u32 N, u64 P, bool planning) {
  // (the arrays per period are sized for P entries: there are fewer periods than uses, fewer uses than pairs)
  size_t b = Pool::need((u64)K + 1, 8) + Pool::need(P, 8) + Pool::need(P, 4) + Pool::need((u64)N + 1, 8) + 3 * Pool::need(P, 4) +
             Pool::need((u64)K + 2, 8);
  if (planning) b += Pool::need(K, 8) + Pool::need(N, 8) + Pool::need(N, 1) + Pool::need(P, 16) + Pool::need(P, 8);
  return b;
}

// The analysis proper, in memory the caller of this function provides (two pools of at least
// vit_tmp_bytes / vit_keep_bytes).  out: where the results of an analysis without planning go.
static int vitality_core(g10_plan_s* h, const g10_trace* tr, Pool& tmp, Pool& keep, const bool planning, const g10_vitality_buffers* out) {
  hipStream_t s = h->stream;
  const u32 K = h->K, N = h->N;
  const u64 P = h->P;

  VitStats* st = nullptr;
  G10_TRY(tmp.take(&st, 1));
  static_assert(sizeof(VitStats) % 8 == 0 && sizeof(VitStats) / 8 <= G10_BLOCK, "cleared as 64-bit words, one per thread");
  G10_TRY(keep.take(&h->pressure_buf, (u64)K + 2));
  hipLaunchKernelGGL(k_begin, dim3(grid_for((u64)K + 2)), dim3(G10_BLOCK), 0, s, st, h->pressure_buf, (u64)K + 2);
  G10_HIP(hipGetLastError());

  // ---- the trace: checks, sort keys, and own copies of what planning needs later (the checks are read by
  // the host with the counts, at the one synchronisation below: nothing a kernel does with a zero
  // duration, a zero or huge size or a wrapped sum leaves its arrays) --------------------------------
  h->kbits = bits_for(K - 1);
  const u32 tbits = bits_for(N - 1);
  u64 *keys = nullptr, *alt = nullptr, *scratch64 = nullptr;
  u32 *sums = nullptr, *psums = nullptr, *hist = nullptr;
  G10_TRY(tmp.take(&keys, P));
  G10_TRY(tmp.take(&alt, P));
  if (planning) {
    G10_TRY(keep.take(&h->dur, K));
    G10_TRY(keep.take(&h->size, N));
    G10_TRY(keep.take(&h->glob, N));
  } else {                                        // the caller's arrays are read in place, during the call only
    h->dur = const_cast<u64*>(tr->dur_ns);
    h->size = const_cast<u64*>(tr->size_bytes);
    h->glob = const_cast<uint8_t*>(tr->is_global);
  }
  {
    u64 most = P > N ? P : N;
    if (K > most) most = K;
    hipLaunchKernelGGL(k_load, dim3(grid_for(most)), dim3(G10_BLOCK), 0, s, tr->dur_ns, tr->size_bytes, tr->is_global, tr->use_kernel,
                       tr->use_tensor, K, N, P, h->kbits, planning ? h->dur : (u64*)nullptr, planning ? h->size : (u64*)nullptr,
                       planning ? h->glob : (uint8_t*)nullptr, keys, st);
    G10_HIP(hipGetLastError());
  }

  // ---- slot start times ----------------------------------------------------
  G10_TRY(tmp.take(&scratch64, scan_scratch_elems(K > N ? K : N)));
  G10_TRY(keep.take(&h->start, (u64)K + 1));
  G10_TRY(scan_excl_u64(tr->dur_ns, h->start, K, scratch64, s));

  // ---- use lists -------------------------------------------------------------
  G10_TRY(tmp.take(&hist, radix_hist_elems(P)));
  G10_TRY(tmp.take(&sums, tile_sums_elems(P)));
  G10_TRY(tmp.take(&psums, tile_sums_elems(P)));
  G10_TRY(keep.take(&h->ukeys, P));                               // upper bounds: no host round trip here
  G10_TRY(keep.take(&h->use_k, P));
  G10_TRY(keep.take(&h->use_off, (u64)N + 1));
  G10_TRY(keep.take(&h->per_t, P));
  G10_TRY(keep.take(&h->per_L, P));
  G10_TRY(keep.take(&h->per_R, P));
  const u32 nb = (u32)((P + TILE - 1) / TILE);
  const u32 scanned = nb > DIRECT ? 1u : 0u;                      // (many tiles: their sums are scanned in a step of its own)
  const u32 no_wrap = (h->flags & G10_NO_WRAP) ? 1u : 0u;
  if (P) G10_TRY(radix_sort_u64(&keys, &alt, P, h->kbits + tbits, hist, s));
  if (nb == 1 && N <= TINY && K <= TINY) {                        // (uses, periods and pressure in one launch)
    hipLaunchKernelGGL(k_tiny, dim3(1), dim3(G10_BLOCK), 0, s, (const u64*)keys, (u32)P, K, N, h->kbits, no_wrap, (const u64*)h->size,
                       (const uint8_t*)h->glob, h->ukeys, h->use_k, h->use_off, h->per_t, h->per_L, h->per_R, h->pressure_buf, st);
    G10_HIP(hipGetLastError());
  } else {
  if (P) {
    if (nb > 1) hipLaunchKernelGGL(k_distinct_count, dim3(nb), dim3(G10_BLOCK), 0, s, (const u64*)keys, P, sums);
    if (scanned) G10_TRY(scan_excl_u32(sums, sums, nb, sums + nb + 1, s));
    hipLaunchKernelGGL(k_distinct_write, dim3(nb), dim3(G10_BLOCK), 0, s, (const u64*)keys, P, (const u32*)sums, nb, scanned, h->ukeys,
                       h->use_k, h->kbits, st);
    G10_HIP(hipGetLastError());
  }
  hipLaunchKernelGGL(k_use_off, dim3(grid_for((u64)N + 1)), dim3(G10_BLOCK), 0, s, (const u64*)h->ukeys, (const u64*)&st->n_uses, N, h->kbits, h->use_off);
  G10_HIP(hipGetLastError());

  // ---- inactive periods --------------------------------------------------------
  if (P) {
    if (nb > 1) hipLaunchKernelGGL(k_period_count, dim3(nb), dim3(G10_BLOCK), 0, s, (const u64*)h->ukeys, (const u64*)h->use_off, (const uint8_t*)h->glob,
                                   (const u64*)&st->n_uses, K, h->kbits, no_wrap, psums);
    if (scanned) G10_TRY(scan_excl_u32(psums, psums, nb, psums + nb + 1, s));
    hipLaunchKernelGGL(k_period_write, dim3(nb), dim3(G10_BLOCK), 0, s, (const u64*)h->ukeys, (const u64*)h->use_off, (const uint8_t*)h->glob, K,
                       h->kbits, no_wrap, (const u32*)psums, nb, scanned, h->per_t, h->per_L, h->per_R, st);
    G10_HIP(hipGetLastError());
  }

  // ---- memory pressure -----------------------------------------------------------
  hipLaunchKernelGGL(k_lifetime_adds, dim3(grid_for(N)), dim3(G10_BLOCK), 0, s, h->ukeys, h->use_off, h->size, h->glob, N, K, h->kbits, h->pressure_buf, st);
  G10_HIP(hipGetLastError());
  // exclusive scan of diff[0..K] in place: buf[k + 1] = sum diff[0..k] = pressure[k]; its largest value is the peak
  G10_TRY(scan_excl<u64>(h->pressure_buf, h->pressure_buf, (u64)K, scratch64, s, &st->peak));
  }
  if (out) {
    const u64 most = P > (u64)N + 1 ? P : (u64)N + 1;
    hipLaunchKernelGGL(k_results_out, dim3(grid_for(most > (u64)K + 1 ? most : (u64)K + 1, 1024)), dim3(G10_BLOCK), 0, s, (const VitStats*)st, *out, K, N,
                       (const u64*)h->use_off, (const u32*)h->use_k, (const u32*)h->per_t, (const u32*)h->per_L, (const u32*)h->per_R,
                       (const u64*)h->start, (const u64*)(h->pressure_buf + 1));
    G10_HIP(hipGetLastError());
  }
  VitStats hs;
  G10_HIP(hipMemcpyAsync(&hs, st, sizeof hs, hipMemcpyDeviceToHost, s));
  G10_HIP(hipStreamSynchronize(s));
  G10_TRY(verdict_of(hs));
  h->T = (u64)(((unsigned __int128)hs.dur_hi << 32) + hs.dur_lo);
  h->big_size = hs.big_size != 0;
  h->max_size = hs.max_size;
  h->n_uses = hs.n_uses;
  h->n_periods = hs.n_periods;
  h->peak = hs.peak;

  if (!planning) return G10_OK;

  // ---- the periods once more, ordered by their start --------------------------------------
  // Planning walks the periods with one thread each and looks up the timeline around their
  // start and end; in this order neighbouring threads look at neighbouring slots.
  const u64 C = h->n_periods;
  G10_TRY(keep.take(&h->per_by_start, C));      // (C <= P)
  G10_TRY(keep.take(&h->per_size, C));
  if (C) {
    // (a stable sort of the starts alone, the position carried along: equal starts keep the order of the periods)
    u32 *k32 = (u32*)keys, *k32_alt = k32 + C, *ord = (u32*)alt, *ord_alt = ord + C;      // (C <= P: two arrays of C words in one of P keys)
    G10_TRY((radix_sort<u32, true>(&k32, &k32_alt, &ord, &ord_alt, C, h->kbits, hist, s, true, (const u32*)h->per_L)));
    hipLaunchKernelGGL(k_gather_periods, dim3(grid_for(C)), dim3(G10_BLOCK), 0, s, (const u32*)ord, C, h->per_t, h->per_L, h->per_R,
                       h->size, h->per_by_start, h->per_size);
    G10_HIP(hipGetLastError());                     // (still running when this function returns: see vitality_run)
  }
  return G10_OK;
}

int vitality_run(g10_plan_s* h, const g10_trace* tr) {
  if (h->P >= (1ull << 32)) return G10_EINVAL;    // positions and counts are 32-bit on the device
  // The temporaries of the call and what the handle keeps.  The last kernels of the analysis
  // still read the temporaries when the call returns (planning follows on the same stream and
  // need not wait for them): they are released at the next point where the stream has been
  // waited for, at the latest with the handle.
  Pool tmp, keep;
  G10_TRY(tmp.reserve(vit_tmp_bytes(h->K, h->N, h->P)));
  h->tmp_arena = tmp.base;
  G10_TRY(keep.reserve(vit_keep_bytes(h->K, h->N, h->P, true)));
  h->arena = keep.base;
  return vitality_core(h, tr, tmp, keep, true, nullptr);
}

// ===========================================================================
// The analysis for callers that cannot allocate: all device memory beyond the caller's inputs
// and outputs is this array, one copy per GPU, held until the process ends.  Its address on the
// current device is asked for once per device (the array's name itself is only a host-side
// stand-in and is never passed to a kernel or a copy).
// ===========================================================================
static __device__ __align__(256) unsigned char scratch[G10_STATIC_SCRATCH_BYTES];

enum { G10_MAX_DEVICES = 64 };
static unsigned char* scratch_on_device[G10_MAX_DEVICES] = {};

extern "C" int g10_vitality_static(const g10_trace* tr, void* hip_stream, const g10_vitality_buffers* out,
                                   g10_vitality_stats* stats) {
  if (stats) memset(stats, 0, sizeof *stats);
  if (!tr || !out || !stats) return G10_EINVAL;
  if (!tr->K || !tr->N) return G10_EINVAL;
  if (!tr->dur_ns || !tr->size_bytes || !tr->is_global) return G10_EINVAL;
  if (tr->P && (!tr->use_kernel || !tr->use_tensor)) return G10_EINVAL;
  if (!out->use_off || !out->start || !out->pressure) return G10_EINVAL;
  if (tr->P && (!out->use_k || !out->per_tensor || !out->per_L || !out->per_R)) return G10_EINVAL;
  if (tr->K > G10_STATIC_MAX_K || tr->N > G10_STATIC_MAX_N || tr->P > G10_STATIC_MAX_P) return G10_ELIMIT;
  const size_t need_tmp = vit_tmp_bytes(tr->K, tr->N, tr->P), need_keep = vit_keep_bytes(tr->K, tr->N, tr->P, false);
  if (need_tmp + need_keep > (size_t)G10_STATIC_SCRATCH_BYTES) return G10_ELIMIT;
  int dev = 0;
  G10_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= G10_MAX_DEVICES) return G10_EDEVICE;
  if (!scratch_on_device[dev]) {
    void* q = nullptr;
    G10_HIP(hipGetSymbolAddress(&q, HIP_SYMBOL(scratch)));
    if (!q) return G10_EDEVICE;
    scratch_on_device[dev] = (unsigned char*)q;
  }
  unsigned char* const mem = scratch_on_device[dev];

  g10_plan_s h;                                   // (lives on the stack for the call; nothing of it is handed out)
  h.device = dev;
  h.stream = (hipStream_t)hip_stream;
  h.K = tr->K; h.N = tr->N; h.P = tr->P; h.flags = tr->flags;
  Pool tmp, keep;                                 // both inside the array
  tmp.base = (char*)mem; tmp.cap = need_tmp;
  keep.base = (char*)mem + need_tmp; keep.cap = need_keep;
  hipStream_t s = h.stream;
  const int rc = vitality_core(&h, tr, tmp, keep, false, out);   // (synchronises the stream where it succeeds)
  if (rc) { (void)hipStreamSynchronize(s); return rc; }
  stats->n_uses = h.n_uses; stats->n_periods = h.n_periods; stats->peak_bytes = h.peak; stats->iter_ns = h.T;
  return G10_OK;
}
