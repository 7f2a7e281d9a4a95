// The greedy loop of smart tensor eviction (G10, Section 4.3, Algorithm 1) as one persistent
// workgroup per plan: rank (tile bounds, score, arg-max), decide, commit (lazy chunk adds and
// chunk jobs), level-1 update.  See g10_plan.hip for the data structures and why the plan is
// the one Algorithm 1 makes.

#include "g10_plan_defs.h"

using namespace g10;

namespace {

// Threads of the loop workgroup: a chunk job takes a wavefront, and most rounds have more jobs than seven wavefronts
// take at once beside the one that picks, so twelve (loops with eight / twelve: ResNet 2.85 / 2.65 ms, ragged stress
// 4.7 / 4.25, stress 23.6 / 21.3, decoder 3.2 / 3.1, encoder 1.20 / 1.16).  Twelve leave 168 registers each, and the
// benefit key in the band reading spills four (with ROWS seven, with TIGHT six); sixteen leave 128.  The ratio key in the band reading commits one migration
// a pass, four jobs: eight (its passes with the scoring kernel take 5 % longer with twelve).
constexpr u32 LOOP_MIN = 512, LOOP_MAX = 768, LW_MAX = LOOP_MAX / G10_WAVE;   // ... least and most, and the most wavefronts
constexpr u32 loop_threads(bool ratio, bool clip) { return ratio && !clip ? LOOP_MIN : LOOP_MAX; }
static_assert(LOOP_MIN >= NCH_MAX && LOOP_MIN % UNIT == 0 && LOOP_MAX % UNIT == 0, "a thread per chunk; units are scored by four whole wavefronts");

struct alignas(16) Winner {   // what a commit needs of the winning candidate
  u64 hi, lo;                 // benefit
  u64 cost;                   // eviction + prefetch time (ranking by benefit / cost only)
  u64 s, fo_base, fi_end;     // size; free out-channel time before L1; free in-channel time before R
  u64 tau_o, tau_i;           // eviction and prefetch time to the destination
  u32 cand, tensor, pos, dest, L1, R, a, b;
  u32 exact;                  // clipped-area benefit only: the value was computed in this pass (else it is a bound)
  u32 slot;                   // its entry in the list of the pass (NONE32: it has none)
  u32 pad[2];
};

// Ranking by benefit / cost keeps a bound per candidate that holds whichever destination the
// policy ends up with: most of a long list then reaches the threshold of every pass and has to
// be scored again.  Such a round is left to all compute units: the loop kernel writes the list
// of tiles to score, ends in the middle of its pass, a scoring kernel takes the list (the tile
// bounds go into the array of tile bounds in device memory, every workgroup's best candidate
// into `win`), and the next launch of the loop kernel takes the pass up again with those.
constexpr u32 WIDE_WG = 2 * (loop_threads(true, false) - 1);   // workgroups of the scoring kernel that take part at most: two winners per thread of the
                                        // loop kernel, whose last thread takes the best of the pass's earlier rounds
struct WideCtx {
  u32 pending;                // the loop kernel has left a list and waits for it to be scored
  u32 nwg, scored;            // workgroups of the scoring kernel that take part; it has run
  u32 ntl, thr, rest;         // of the round left open: tiles on the list, its threshold, bound of the tiles not on it
  u32 rounds, pass_units;     // of the pass left open: rounds finished, units scored in them
  u32 seq, pad[3];            // launches of the loop kernel on this plan so far
};
struct WideKey {              // the ranking of a winner on its own, for the arg-max over them
  u64 hi, lo, cost;
  u32 cand, skipped;          // (the largest key its workgroup took from the memo instead of scoring)
};
constexpr u32 MEMO_SPAN = 2;   // migrations a memo of the scoring kernel may be older than the list (one per pass)
constexpr u32 MEMO_MARGIN = 2u << 24;   // kept keys lie this far under the round's threshold, in key steps (2^24 are a factor of two): a quarter of it
struct WideView {
  WideCtx* ctx;
  WideKey* key;               // [WIDE_WG + 1] of win[]
  Winner* win;                // [WIDE_WG], then the best of the earlier rounds
  u64* smark;                 // [NT_MAX / 64]  tiles scored in the pass left open
  unsigned short* alist;      // [NT_MAX]       the list
};
constexpr size_t WIDE_BYTES = sizeof(WideCtx) + (WIDE_WG + 1) * (sizeof(WideKey) + sizeof(Winner)) + (NT_MAX / 64) * 8 + (size_t)NT_MAX * 2;
__host__ __device__ __forceinline__ WideView wide_view(void* blob) {
  WideView v;
  char* q = (char*)blob;
  v.ctx = (WideCtx*)q; q += sizeof(WideCtx);
  v.key = (WideKey*)q; q += (WIDE_WG + 1) * sizeof(WideKey);
  v.win = (Winner*)q; q += (WIDE_WG + 1) * sizeof(Winner);
  v.smark = (u64*)q; q += (NT_MAX / 64) * 8;
  v.alist = (unsigned short*)q;
  return v;
}
static_assert(sizeof(WideCtx) % 16 == 0 && sizeof(WideKey) % 16 == 0 && sizeof(Winner) % 16 == 0, "the arrays of the scoring kernel's block stay aligned");

constexpr u32 MAXM = 16;      // migrations committed in one round at most (a multiple of 8, at most 16: the job words hold two sets of 16)
static_assert(MAXM % 8 == 0 && MAXM <= 16, "job words and chunk flags are laid out for 8 or 16");

constexpr u32 MC_GUESS_SHIFT_MIN = 2;   // the widest margin of a pass's first threshold under the last benefit: 2^-this
// The list of the pass: the candidates whose bound exceeds every bound not looked at one by one.  An entry is LIST_VECS
// arrays of 16 bytes - period and windows as in Cands (a committed one has no window left); {index, tensor, position};
// over-capacity times (NONE64: the destination cannot be used); free channel times at the ends of the transfer windows, out
// and in of either destination (Score), as doubles - and the keys of its benefits at either destination.  As many entries as
// fit the LDS beside chunks and tiles: 64 always do, 256 nearly always.  The picking wavefront holds 64, the best by bound.
// (Ranking passes of a plan with 64 in all / with 256 and the choice: ResNet 240 / 25, decoder 186 / 70, stress 500 / 160.)
constexpr u32 LIST_MIN = 64, LIST_MAX = 256, LIST_VECS = 8, LIST_ENTRY = LIST_VECS * 16 + 8;
// A plan by the clipped area goes on in the form with lists once LISTS_AFTER winners in a row had their band as their area, shown by
// the chunks alone; it leaves that form after LISTS_VAIN lists in a row that gave one migration at most, to come back after twice
// as many winners each time, but where LISTS_PAID lists had given several.  (Another launch is 25 us, a list in vain 8; a pass of
// the form with lists without one takes 2 us more than one of the other, and an area settled in it 0.4: registers.  With one form
// for both, lists tried less and less often, plans of 20 to 60 passes took 10 to 13 % more.  ResNet, 1622 migrations, after 8
// winners and 4 lists 3.4 ms, one migration a pass 17.8.)
// It stays where LISTS_LEFT periods - with a window or without one - are not left, which keeps the smallest traces out, and where its
// limit leaves it less than LISTS_PASSES passes.  (Twelve passes gain 120 us if the lists pay, and a change that does not costs 80.
// Plans of 20 passes that changed with less left / stay: ResNet at 0.6 of its peak 882 / 865 us, 90 slots 335 / 306, 2000 slots
// 510 / 492.)
constexpr u32 LISTS_AFTER = 8, LISTS_VAIN = 4, LISTS_PAID = 4, LISTS_MORE_MAX = 7, LISTS_LEFT = 128, LISTS_PASSES = 12;
// Where the chunks are no more than four per wavefront (but the last one) and the picks many, the chunk test takes a row of 16 lanes per chunk and a
// lane per migration, else a lane per chunk and the migrations one after the other.  (Steps of ResNet, 23 chunks and 12 picks a
// round 2875 -> 2743 us, encoder 1298 -> 1273, ResNet by the clipped area 3.89 -> 3.44 ms.  With rows wherever 80 chunks fit two turns
// of them decoder, 49 chunks and 4 picks, 3258 -> 3435, ragged stress, 79 and 12, 5663 -> 5824.)  Forms of their own (ROWS), taken where
// rows can be: in the one form for all, plans that never take them paid for it (plans of one migration a pass: 16.97 -> 16.65 ms on 20 011
// slots, 7.16 -> 7.03 on the decoder trace).
constexpr u32 ROW_CHUNKS = (LW_MAX - 1) * 4, ROW_PICKS = 8;
static_assert(MAXM == 16, "a row of lanes per chunk");
static_assert(LIST_MIN == G10_WAVE && LIST_MAX % G10_WAVE == 0, "an entry a lane; strips of whole wavefronts");
// LE_I's last word: host memory was found to have no room for the entry, at any later time neither, or to have room (as long
// as nothing else goes there: Shared::probed).
enum : u32 { E_NOROOM = 4, E_ROOM = 8 };
constexpr u32 PK_DROP = 1u << 17, PK_ROOM = 1u << 18;   // a pick that host memory has no room for: the candidate is refused; one it has room for
enum { LE_A = 0, LE_B = 1, LE_I = 2, LE_OT = 3, LE_O0 = 4, LE_I0 = 5, LE_O1 = 6, LE_I1 = 7 };
// How far under the round's threshold a scored candidate's bound may lie to go on the list, in key steps (2^24 are a
// factor of two); below zero: how far above it must lie.  Entries under the bound of the tiles left out cannot be picked,
// so that is the lowest; within that the margin follows the list towards a quarter to nine sixteenths of its length, in small steps near there.
// Which entries an overflowing list takes is left to chance, and the pass is then mostly ranked by an arg-max over all
// threads and begins with a round of one migration: with a list of 64, a margin that doubled into an overflow every few passes gave stress plans between 400 and
// 1100 ranking passes, and one that could not go above the threshold left six passes in ten overflowing on the model
// traces (many candidates of a repeated layer lie within the eighth under the last benefit).
constexpr int PUB_START = 1 << 22, PUB_MIN = -(1 << 23), PUB_MAX = 1 << 30;

// Beside the number of jobs, while an area is settled: some chunk has a slot over the capacity by less than the tensor's size.
constexpr u32 UNEVEN = 1u << 16;
static_assert(6 * NCH_MAX + 8 < UNEVEN, "the jobs of a round");

enum { NX_RESCORE = 0, NX_PICKED = 1 };   // how a further round of a pass begins: the list scored again; its migrations picked already

struct Floor {                // bound of the list's entries that the picking wavefront does not hold (see choose)
  u64 hi, lo;
  u32 key, cand, full, pad;
};

struct alignas(16) Shared {   // small per-pass state of the loop workgroup
  Winner mem[MAXM];           // migrations of the pass in commit order; [0] is the winner of the ranking (hi = lo = 0: none)
  Winner wave_win[LW_MAX];    // best of every wavefront (between two rankings: what the chunk test finds, ROW_CHUNKS)
  double bw[8];               // bandwidths out 0, 1, in 0, 1, and their reciprocals
  // What the picking wavefront leaves: the migrations of the round (entry of the list, destination << 16; free times
  // before the eviction window's start and the prefetch window's end as the picks before left them), and its state
  u32 pick[MAXM];             // entry | destination << 16 | PK_DROP, PK_ROOM (to host only)
  double pick_o[MAXM], pick_i[MAXM];
  u32 chain[2][4];            // per round (even, odd) and channel (out 0, 1, in 0, 1): some windows of the round's picks and entries meet
  double all[4];              // free time of each channel behind the picks
  Floor left;
  u32 sel[G10_WAVE], nsel;    // the entries of the list it holds
  u32 probed;                 // nothing has gone to host since the entries with E_ROOM were looked at
  u32 pick_max, next;         // migrations picked in a round at most; NX_*
  u32 dests[2];               // the round's migrations to flash, to host
  // (what the forms with lists added lies here, in place of words that were spare: before the counters below, where the
  // words that every round uses moved by 32 bytes, the benefit key spilled three registers more: decoder
  // 3.09 ms instead of 3.08, plans of one migration a pass 7.03 instead of 6.87)
  // clipped area: the plan's passes make lists, so often it has stopped doing so; this pass does not; lists in vain in a row, or winners
  // in a row whose area was their band by the chunks alone; migrations and refused candidates when the pass began
  u32 lists, lists_ended, no_list, in_row;
  u64 settled0;
  u32 paid, alone;            // lists that gave several; a change of form ends the launch (LoopArgs)
  u64 tight_at;               // refused candidates from which the plan goes on in the form for them (Ctl)
  u32 calm, pad2;             // rounds in a row of that form without one
  unsigned char spare[88];    // (free: with it 7899 tiles fill the LDS beside 512 chunks, see loop_tile_shift)
  u32 wave_f2[LW_MAX];        // per wavefront: largest bound among the candidates its threads scored but do not hold
  u32 F2, pad0;               // ... over the workgroup
  u32 nlist, m0, cut, need_exact;   // list length; migrations selected; how many of them may be committed; the winner's
                              // host-capacity test needs the exact per-slot maximum
  u32 by_floor, touched;      // the selection ended because the next candidate did not clear the floor; timelines (a bit
                              // per array of level 1) whose chunk totals change in this pass
  u32 fast, pad1;             // the pass's migrations were picked from the list without an arg-max over all threads
  u32 lim, pad3;              // the plan has made as many passes as it may
  u32 Fkeep, more;            // the floor of the pass; another round of commits follows from the same list
  u64 more_rounds, list_rescored;   // such rounds made; list entries scored again for them (statistics)
  u64 hq;                     // host-capacity query: maximum over the period
  u64 acc[3];                 // clipped area being summed: bits 0..31, 32..63 and 64.. of the terms, added apart
  u64 evals, refused;         // clipped areas found exactly, summed or shown to be bands; of those, how many came out below the bound
  u32 nl, restL;              // hot list: length; bound of the tiles outside it
  u32 ntl, filt;              // current round: tiles to score; bound of the hot tiles left out
  u32 njobs, jnext, ot_changed, stale_hot;   // jobs listed; the next one that a wavefront takes after its first
  u32 no_wide;                // this launch may not leave a round to the scoring kernel (none is queued behind it)
  // progress (mirrors Ctl)
  u64 n_iter, n_mig, n_drop, n_evals, units, second, jobs;
  u32 thr_key, status, done, stop;
  u32 gshift;                 // margins of the first threshold, and of the list under it
  int pub;
  u64 t_start;
};

// The lane of the wavefront holding the best (benefit, lowest index), or NONE32
// if every benefit is 0.  The 31-bit key decides unless several lanes share the
// largest key (equal or nearly equal benefits: common where a model repeats one
// layer); those are settled by three more reductions: high word, low word, index.
__device__ __forceinline__ u32 wave_best_lane(u64 hi, u64 lo, u32 cand) {
  const u32 k = upkey(hi, lo);
  const u32 kmax = wave_max(k);
  if (kmax == 0) return NONE32;
  u64 m = __ballot(k == kmax);
  if (m & (m - 1)) {
    const bool in1 = k == kmax;
    const u64 hmax = wave_max(in1 ? hi : 0ull);
    const bool in2 = in1 && hi == hmax;
    const u64 lmax = wave_max(in2 ? lo : 0ull);
    const bool in3 = in2 && lo == lmax;
    const u32 cmin = wave_min(in3 ? cand : NONE32);
    m = __ballot(in3 && cand == cmin);
  }
  return (u32)__builtin_ctzll(m);
}

__device__ __forceinline__ u64 read_lane64(u64 v, u32 l) {
  const u32 lo = (u32)__builtin_amdgcn_readlane((int)(u32)v, (int)l), hi = (u32)__builtin_amdgcn_readlane((int)(u32)(v >> 32), (int)l);
  return ((u64)hi << 32) | lo;
}

__device__ __forceinline__ u64 umin64(u64 a, u64 b) { return a < b ? a : b; }
__device__ __forceinline__ double read_lanef(double v, u32 l) { return __longlong_as_double((long long)read_lane64((u64)__double_as_longlong(v), l)); }

// The same for benefit / cost.  The approximate keys only narrow the field: a lane stays if
// its upper key reaches the largest lower key.  The lanes that stay are settled exactly: take
// the first, keep the lanes that beat it (fractions compared by cross multiplication, equal
// ones by index), repeat with the first of those.
__device__ __forceinline__ u32 wave_best_lane_ratio(u64 hi, u64 lo, u64 cost, u32 cand) {
  const bool has = (hi | lo) != 0;
  const double r = has ? ratio_approx(hi, lo, cost) : 0.0;
  const u32 kdn_max = wave_max(has ? rkey_dn(r) : 0u);
  u64 m = __ballot(has && rkey_up(r) >= kdn_max);
  if (!m) return NONE32;
  const u32 lane = lane_id();
  u32 p = (u32)__builtin_ctzll(m);
  while (m & (m - 1)) {
    const u64 ph = read_lane64(hi, p), pl = read_lane64(lo, p), pc = read_lane64(cost, p);
    const u32 pcand = (u32)__builtin_amdgcn_readlane((int)cand, (int)p);
    const bool beats = ((m >> lane) & 1ull) && lane != p && better_ratio(hi, lo, cost, cand, ph, pl, pc, pcand);
    m = __ballot(beats);
    if (!m) break;
    p = (u32)__builtin_ctzll(m);
  }
  return p;
}

// Exclusive sums of four strips of 64 values (v[i] of lane l stands at 64 i + l) from `carry` on, which moves past
// them.  T: the type that holds every sum.
template <class T>
__device__ __forceinline__ void scan_strips(const u64 (&v)[4], u64 (&run)[4], u64& carry) {
  T inc[4], at = (T)carry;
#pragma unroll
  for (u32 i = 0; i < 4; ++i) inc[i] = wave_scan_incl((T)v[i]);
#pragma unroll
  for (u32 i = 0; i < 4; ++i) {
    run[i] = (T)(at + inc[i] - (T)v[i]);
    at += wave_last(inc[i]);
  }
  carry = at;
}

// Times in doubles, which hold whole numbers up to 2^53 exactly: one instruction an addition, a minimum or a clamp
// where 64-bit integers take two to five.  Used where PICK_EXACT bounds every time and size.
// Channel time a migration takes between its window's start (eviction: the earliest free time is taken first) or end
// (prefetch: the latest first) and a point `away` of free time from there.  (Negative: the point lies on the other side.)
__device__ __forceinline__ double takenf(double away, double tau) { return fmin(fmax(away, 0.0), tau); }
// The free time f before a point of the doubled timeline once a migration took `tau` from its window: less by what it
// takes before that point, in the places that the window has around the doubled timeline, `all` of the channel's free
// time apart.  ref: the free time before the window's start (out), or before its end.  (Where neither the points nor the
// window lie in the second iteration the other places cancel.)
__device__ __forceinline__ double after_takingf(double f, double all, double ref, double tau, bool out, bool wrap) {
  double r = out ? f - takenf(f - ref, tau) : f + takenf(ref - f, tau) - tau;
  if (wrap) {
    if (out) r = r - takenf(f - all - ref, tau) - (takenf(f + all - ref, tau) - takenf(all - ref, tau));
    else r = r + (takenf(ref - f + all, tau) - tau) + (takenf(ref - f - all, tau) - takenf(ref - all, tau));
  }
  return r;
}
constexpr u64 PICK_EXACT = 1ull << 48;   // bound of the iteration's free time and of 1000 x the largest tensor (sums of a few stay exact)
__device__ __forceinline__ double exactf(u64 x) { return __fma_rn((double)(u32)(x >> 32), 4294967296.0, (double)(u32)x); }   // x < 2^53
// ceil(x / bw) for whole x < 2^50: the quotient by the reciprocal is off by one at most, the remainder exact
__device__ __forceinline__ double ceil_divf(double x, double bw, double inv) {
  double q = floor(x * inv), r = __fma_rn(-q, bw, x);
  if (r < 0.0) { q -= 1.0; r += bw; }
  if (r >= bw) { q += 1.0; r -= bw; }
  return r > 0.0 ? q + 1.0 : q;
}

// The thread's number, anew: what is made from it here cannot be moved out of the loops around.  (The compiler keeps the
// LDS addresses of every array and lane in registers across the whole kernel otherwise, and spills them: 30 registers.)
__device__ __forceinline__ u32 thread_here() {
  u32 t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// inclusive sums inside each row of 16 lanes
__device__ __forceinline__ u64 row_scan(u64 v) {
  v += dpp_move<0x111, 0xf, 0xf>((u64)0, v);
  v += dpp_move<0x112, 0xf, 0xf>((u64)0, v);
  v += dpp_move<0x114, 0xf, 0xf>((u64)0, v);
  v += dpp_move<0x118, 0xf, 0xf>((u64)0, v);
  return v;
}
__device__ __forceinline__ bool any(bool x) { return ballot(x) != 0; }

template <bool RATIO>
__device__ __forceinline__ u32 best_lane(u64 hi, u64 lo, u64 cost, u32 cand) {
  if (RATIO) return wave_best_lane_ratio(hi, lo, cost, cand);
  return wave_best_lane(hi, lo, cand);
}

// LDS of the loop workgroup up to the list of the pass, and the entries of that list
__host__ __device__ __forceinline__ size_t lds_before_list(u32 nch, u32 nt) {
  const size_t ns = (nt + 63) / 64;
  size_t b = sizeof(Shared);
  b += ((size_t)N_ARR * (nch + 1) + (size_t)N_ARR * nch + (size_t)4 * nch + ns + (size_t)6 * nch + 8) * 8;      // (six jobs a chunk at most)
  b += ((size_t)nt + ns + 2 * (size_t)nch) * 4 + (size_t)nt * 4;
  return (b + 15) & ~(size_t)15;
}
__host__ __device__ __forceinline__ u32 list_cap(u32 nch, u32 nt) {
  const size_t b = lds_before_list(nch, nt), room = b < LDS_MAX ? (LDS_MAX - b) / LIST_ENTRY : 0;
  return room >= LIST_MAX ? LIST_MAX : room < LIST_MIN ? LIST_MIN : (u32)room / G10_WAVE * G10_WAVE;
}

// TIGHT: the form for plans whose host memory refuses candidates, several of which go in one round (probe_host).  A form of its
// own because what it adds to the chunk test, the picks and the commit costs plans without any 1.4 to 2 % (20.93 ms instead of 20.65 on
// the stress trace), those that commit one migration a pass 3 to 4.  The clipped area and the ratio key refuse one candidate a pass.
// LISTS: the form of the clipped area that commits several migrations a pass, for plans whose winners' areas are their bands
// (LISTS_AFTER).
// ROWS: with the chunk test by rows of lanes (ROW_CHUNKS).
template <bool RATIO, bool CLIP, bool TIGHT, bool LISTS, bool ROWS>
__global__ __launch_bounds__(loop_threads(RATIO, CLIP)) void k_loop(const LoopArgs* __restrict__ plans) {
  constexpr u32 LB = loop_threads(RATIO, CLIP), LW = LB / G10_WAVE;    // threads and wavefronts of this form
  // Several migrations per ranking pass (ranking by the benefit itself): after the
  // winner, the next best candidates of the same pass are committed with it as long as it is
  // certain that each would have won the pass after the one before it - see "more migrations
  // of the same pass" below.  With the clipped area a pick stands for its band, which bounds every area, and is committed
  // only where the chunks show that its area is the band: every slot over the capacity in the chunks that its absent window
  // touches exceeds it by the tensor's size, behind what the picks before it take.  Where that fails for the first pick, the
  // pass goes on to the arg-max and the areas summed slot by slot (settle).
  constexpr bool MC = !RATIO && (!CLIP || LISTS);
  static_assert((MC && !CLIP) || !TIGHT, "several migrations a pass");
  static_assert((MC && CLIP) || !LISTS, "several migrations a pass");
  static_assert(MC || !ROWS, "rows of lanes take a list's migrations");
  static_assert(sizeof(Winner) * LW_MAX >= ROW_CHUNKS * sizeof(uint4), "the chunk test's results");
  constexpr bool WIDE = RATIO && !CLIP;        // long scoring rounds may be left to the scoring kernel (see WideCtx)
  extern __shared__ __align__(16) unsigned char smem[];
  const LoopArgs a = in_global(plans[blockIdx.x]);   // one workgroup per plan
  const Timelines tl = a.tl;
  const u32 nch = tl.nch, nb1 = nch + 1, K = tl.K, CH = 1u << tl.shift_ch, nt = a.nt, ns = (nt + 63) / 64;
  Shared* S = (Shared*)smem;
  u64* base = (u64*)(S + 1);                            // [5][nch + 1]
  u64* tot = base + (u64)N_ARR * nb1;                   // [5][nch]
  u64* lazyP = tot + (u64)N_ARR * nch;
  u64* minOver = lazyP + nch;
  u64* lazyH = minOver + nch;
  u64* hmax = lazyH + nch;
  u64* smark = hmax + nch;                              // [ns] tiles of a group of 64 scored in this pass
  u64* scr = (u64*)S->pick_o;                           // [3 * LW] (before the passes, over pick_o, pick_i and chain)
  static_assert(sizeof(S->pick_o) + sizeof(S->pick_i) + sizeof(S->chain) >= 3 * LW_MAX * 8, "the scan's scratch");
  u64* jobs = smark + ns;                               // [6 * nch + 8]  chunk | kind << 16 | a set of the pass's migrations << 24 | another << 40
  u32* keys = (u32*)(jobs + 6 * nch + 8);               // [nt]  bound of every tile
  u32* skeys = keys + nt;                               // [ns]  largest bound of every group of 64 tiles
  u32* hmat = skeys + ns;                               // [nch] host occupancy: migrations (by index) already added to the chunk's slots
  u32* hpend = hmat + nch;                              // [nch] ... and whether a later one that cuts the chunk is still missing (bit 0);
                                                        // a slot dropped under the capacity since the list was last scored (bit 1)
  unsigned short* tlist = (unsigned short*)(hpend + nch);  // [nt]  the hot list
  unsigned short* alist = tlist + nt;                            // [nt]  tiles scored in the current round
  const u32 lcap = MC ? list_cap(nch, nt) : 0u;         // entries of the list of the pass
  uint4* const list = (uint4*)(smem + lds_before_list(nch, nt));         // [LIST_VECS][lcap]
  u32* const lkey = (u32*)(list + (size_t)LIST_VECS * lcap);             // [2][lcap] keys: the larger one bounds the entry
  auto list_at = [&](u32 field, u32 i) -> uint4& { return list[field * lcap + i]; };
  auto list_ot = [&](u32 i, u32 d) -> u64& { return reinterpret_cast<u64*>(&list[LE_OT * lcap + i])[d]; };
  auto list_f = [&](u32 field, u32 i) -> double2& { return reinterpret_cast<double2&>(list[field * lcap + i]); };

  const u32 tid = threadIdx.x, lane = tid & 63u, wave = uniform(tid >> 6);
  Ctl* ctl = a.ctl;
  // A pass left open by the last launch: its list has been scored by the scoring kernel (1), or
  // has not (2: it is scored here).  Launches are queued ahead of what is known of the plan's
  // progress; one that finds nothing to do ends at once.
  WideView wv = {};
  u32 resume = 0;
  WideCtx wc = {};                                     // all that the launch reads of a pass left open, in one trip to memory:
  WideKey wk[2];                                       // the scoring kernel's winners, two per thread: their rankings only (the
                                                       // whole winners, 112 bytes each at 112-byte steps, kept this workgroup's
                                                       // texture unit busy for 18 us a pass); the last thread: the best of the rounds before
  u64 units0 = 0, second0 = 0, jobs0 = 0, launches0 = 0, wide0 = 0;   // the plan's counters
  constexpr u32 MPT = (NT_MAX / 64 + LB - 1) / LB;
  u64 wmark[MPT];
  if (tid == 0) S->no_wide = 0;
  if (WIDE && a.wide) {
    wv = wide_view(a.wide);
    wc = *wv.ctx;
    wk[0] = wv.key[tid < LB - 1 ? tid : WIDE_WG];
    wk[1] = wv.key[tid < LB - 1 ? tid + LB - 1 : WIDE_WG];
#pragma unroll
    for (u32 j = 0; j < MPT; ++j) wmark[j] = wv.smark[tid + j * LB < NT_MAX / 64 ? tid + j * LB : 0u];
    units0 = ctl->units_scored; second0 = ctl->second_rounds; jobs0 = ctl->jobs_run; wide0 = ctl->wide_rounds;
    if (wc.pending) resume = wc.scored ? 1u : 2u;   // (the launches of a stream follow one another: it ran to its end)
    if (tid == 0) {                                  // (read by everyone after the barrier that ends "state in")
      const u32 seq = wc.seq + 1;
      wv.ctx->seq = seq;
      S->no_wide = seq == a.wide_last_seq ? 1u : 0u;
    }
  }
  const u64 passes_before = ctl->passes;
  const u64 cap = ctl->gpu_cap, host_cap = ctl->host_cap, max_iter = ctl->max_iter, C = ctl->C;
  const u64 bwo0 = ctl->bw_out[0], bwo1 = ctl->bw_out[1], bwi0 = ctl->bw_in[0], bwi1 = ctl->bw_in[1];
  const u64 ivo0 = ctl->inv_out[0], ivo1 = ctl->inv_out[1], ivi0 = ctl->inv_in[0], ivi1 = ctl->inv_in[1];

  // ---- state in ----------------------------------------------------------------------
  // Every load is on its way before the first value is stored (a loop that copies word by word takes a trip to memory a
  // turn, and a trip right behind a launch is long): 22.5 -> 21.0 us a launch where every pass takes one, the loops of 500
  // passes by benefit / cost on the stress trace 18.3 -> 17.6 ms.
  {
    constexpr u32 TPT = (N_ARR * NCH_MAX + LB - 1) / LB, BPT = (N_ARR * (NCH_MAX + 1) + LB - 1) / LB, CPT = (NCH_MAX + LB - 1) / LB, KPT = 8;
    static_assert(CPT == 1, "a thread per chunk");
    const u32 nc0 = tid < nch ? tid : 0u;
    u64 vt[TPT], vb[BPT];
    u32 vk[KPT];
#pragma unroll
    for (u32 j = 0; j < TPT; ++j) { const u32 i = tid + j * LB; vt[j] = a.g_tot[i < N_ARR * nch ? i : 0u]; }
#pragma unroll
    for (u32 j = 0; j < BPT; ++j) { const u32 i = tid + j * LB; vb[j] = a.g_base[i < N_ARR * nb1 ? i : 0u]; }   // (level 1 as the plan's last launch left it, if there was one)
#pragma unroll
    for (u32 j = 0; j < KPT; ++j) { const u32 i = tid + j * LB; vk[j] = a.g_keys[i < nt ? i : 0u]; }
    const u64 c_lp = a.g_lazyP[nc0], c_mo = a.g_minOver[nc0], c_lh = a.g_lazyH[nc0], c_hm = a.g_hmax[nc0];
    const u32 c_ht = a.g_hmat[nc0], c_hp = a.g_hpend[nc0];
    launches0 = ctl->launches;
    const u32 ended = ctl->done;
    if (WIDE && a.wide && !resume && (ended || (a.pass_stop && passes_before >= a.pass_stop))) return;
#pragma unroll
    for (u32 j = 0; j < TPT; ++j) { const u32 i = tid + j * LB; if (i < N_ARR * nch) tot[i] = vt[j]; }
    if (launches0) {
#pragma unroll
      for (u32 j = 0; j < BPT; ++j) { const u32 i = tid + j * LB; if (i < N_ARR * nb1) base[i] = vb[j]; }
    }
#pragma unroll
    for (u32 j = 0; j < KPT; ++j) { const u32 i = tid + j * LB; if (i < nt) keys[i] = vk[j]; }
    for (u32 i = tid + KPT * LB; i < nt; i += LB) keys[i] = a.g_keys[i];
    if (tid < nch) { lazyP[tid] = c_lp; minOver[tid] = c_mo; lazyH[tid] = c_lh; hmax[tid] = c_hm; hmat[tid] = c_ht; hpend[tid] = c_hp; }
  }
  for (u32 i = tid; i < ns; i += LB) smark[i] = 0;
  if (tid == 0) {
    S->n_iter = ctl->n_iter; S->n_mig = ctl->n_mig; S->n_drop = ctl->n_drop; S->n_evals = ctl->n_evals;
    S->units = 0; S->second = 0; S->jobs = 0; S->evals = 0; S->refused = 0; S->more_rounds = 0; S->more = 0; S->list_rescored = 0;
    S->thr_key = ctl->thr_key; S->status = ctl->status; S->done = ctl->done;
    S->gshift = ctl->gshift ? ctl->gshift : GUESS_SHIFT;
    S->pub = ctl->pub ? ctl->pub : PUB_START;      // (0: not set yet; a margin of 0 starts over)
    S->nl = 0; S->restL = NONE32; S->stale_hot = 0; S->pick_max = MAXM;
    S->stop = 0; S->t_start = wall_clock64();
    S->lists = CLIP ? ctl->lists : 0u; S->lists_ended = ctl->lists_ended; S->no_list = LISTS && S->lists ? 0u : 1u; S->in_row = LISTS && S->lists ? NONE32 : 0u; S->paid = 0; S->alone = a.alone;   // (the launch opens a pass: no list in vain yet)
    S->settled0 = ctl->n_mig + ctl->n_drop;
    if (TIGHT) { S->tight_at = ctl->tight_at; S->calm = ctl->calm; }
    S->acc[0] = 0; S->acc[1] = 0; S->acc[2] = 0;
    S->mem[0].hi = 0; S->mem[0].lo = 0;
  }
  __syncthreads();
  for (u32 g = wave; g < ns; g += LW) {                 // group bounds
    const u32 t = g * 64 + lane;
    const u32 k = wave_max(t < nt ? keys[t] : 0u);
    if (lane == 0) skeys[g] = k;
  }

  // exclusive scan of the chunk totals of `na` arrays into base (three barriers)
  auto scan_bases = [&](u32 arr0, u32 arr1, u32 arr2, u32 na) {
    const u32 arrs[3] = {arr0, arr1, arr2};
    const bool act = tid < ((nch + 63u) & ~63u);
    u64 v[3] = {0, 0, 0}, inc[3] = {0, 0, 0};
    if (act) {
      for (u32 q = 0; q < na; ++q) {
        v[q] = tid < nch ? tot[(u64)arrs[q] * nch + tid] : 0ull;
        inc[q] = wave_scan_incl(v[q]);
        if (lane == G10_WAVE - 1) scr[q * LW + wave] = inc[q];
      }
    }
    __syncthreads();
    if (wave == 0) {                                    // the wavefront totals: one small scan
      const u32 nw = (nch + 63) / 64;
      for (u32 q = 0; q < na; ++q) {
        const u64 x = lane < nw ? scr[q * LW + lane] : 0ull;
        const u64 xi = wave_scan_incl(x);
        if (lane < nw) scr[q * LW + lane] = xi - x;
        if (lane == G10_WAVE - 1) base[(u64)arrs[q] * nb1 + nch] = xi;
      }
    }
    __syncthreads();
    if (act && tid < nch)
      for (u32 q = 0; q < na; ++q) base[(u64)arrs[q] * nb1 + tid] = scr[q * LW + wave] + inc[q] - v[q];
    __syncthreads();
  };
  if (!launches0) {                                     // the plan's first launch: level 1 from the chunk totals
    scan_bases(0, 1, 2, 3);
    scan_bases(3, 4, 0, 2);
  } else __syncthreads();


  // Are times and sizes small enough for doubles (PICK_EXACT)?  May the further migrations of a pass be picked (not on
  // timelines of 2^30 slots and more, which no test reaches)?
  // (The ratio key in the band reading keeps to whole numbers: its rounds have one migration, for which a scan of 32-bit
  // sums costs less than the clamped distances in doubles: a pass on 24 slots 9.1 us in doubles, 8.9 in whole numbers, on the
  // stress trace 30.6 and 30.1, most of it to flash 35.0 and 34.4.  With the clipped area 10.8 and 11.0 on the ResNet trace.)
  bool exact = !WIDE && ctl->smax < PICK_EXACT / 1000 && ((bwo0 | bwo1 | bwi0 | bwi1) < PICK_EXACT);
  for (u32 q = A_FO; q < N_ARR; ++q) exact = exact && base[(u64)q * nb1 + nch] < PICK_EXACT;
  exact = uniform((u32)exact) != 0u;
  const bool picks = MC && K < (1u << 30) && exact;
  if (MC && tid < 4) {
    const double bw = exactf(tid == 0 ? bwo0 : tid == 1 ? bwo1 : tid == 2 ? bwi0 : bwi1);
    S->bw[tid] = bw; S->bw[4 + tid] = 1.0 / bw;
  }

  // The hot list: every tile not scored in this pass whose bound reaches `thr`; restL bounds
  // the tiles left out.  Bounds only fall and only scored tiles change, so the list stays
  // complete for any later threshold above restL and is kept across passes.
  auto build_hot = [&](u32 thr) {
    if (tid == 0) { S->nl = 0; S->restL = 0; }
    __syncthreads();
    u32 rm = 0;
    for (u32 g0 = 0; g0 < ns; g0 += 64) {          // 64 groups at a time, one per lane, in every wavefront alike
      const u32 sk = g0 + lane < ns ? skeys[g0 + lane] : 0u;
      const bool q = sk != 0 && sk >= thr;
      if (!q && sk > rm) rm = sk;
      u64 qm = __ballot(q);
      for (u32 turn = 0; qm; ++turn) {             // the wavefronts share the groups that qualify
        const u32 g = g0 + (u32)__builtin_ctzll(qm);
        qm &= qm - 1;
        if (turn % LW != wave) continue;
        const u32 t = g * 64 + lane;
        const u32 k = t < nt ? keys[t] : 0u;
        const bool marked = (smark[g] >> lane) & 1ull;
        const bool sel = k != 0 && k >= thr && !marked;
        if (!sel && !marked && k > rm) rm = k;
        const u64 m = __ballot(sel);
        if (m) {
          u32 off = 0;
          if (lane == 0) off = atomicAdd(&S->nl, (u32)__popcll(m));
          off = (u32)__builtin_amdgcn_readfirstlane((int)off);
          if (sel) tlist[off + __popcll(m & ((1ull << lane) - 1ull))] = (unsigned short)t;
        }
      }
    }
    rm = wave_max(rm);
    if (lane == 0 && rm) atomicMax(&S->restL, rm);
    __syncthreads();
  };

  // The tiles of the hot list whose bound reaches `thr` and that were not scored in this pass
  // -> alist (marked, bound cleared: the scoring rebuilds it); filt bounds the others.
  // (`fresh`: the counters are cleared already)
  auto activate = [&](u32 thr, bool fresh) {
    const u32 tid = thread_here(), lane = tid & 63u;
    if (!fresh) {
      if (tid == 0) { S->ntl = 0; S->filt = 0; }
      __syncthreads();
    }
    const u32 nl = uniform(S->nl);
    u32 fm = 0;
    for (u32 i0 = 0; i0 < nl; i0 += LB) {
      const u32 i = i0 + tid;
      const u32 t = i < nl ? tlist[i] : 0u;
      const u32 k = i < nl ? keys[t] : 0u;
      const bool marked = i < nl && ((smark[t >> 6] >> (t & 63u)) & 1ull);
      const bool sel = k != 0 && k >= thr && !marked;
      if (!sel && !marked && k > fm) fm = k;
      const u64 m = __ballot(sel);
      if (m) {
        u32 off = 0;
        if (lane == 0) off = atomicAdd(&S->ntl, (u32)__popcll(m));
        off = (u32)__builtin_amdgcn_readfirstlane((int)off);
        if (sel) {
          alist[off + __popcll(m & ((1ull << lane) - 1ull))] = (unsigned short)t;
          keys[t] = 0;
          atomicOr((unsigned long long*)&smark[t >> 6], 1ull << (t & 63u));
        }
      }
      if (i0 + LB >= nl) break;
    }
    fm = wave_max(fm);
    if (lane == 0 && fm) atomicMax(&S->filt, fm);
    __syncthreads();
  };

  u32 pass_units = 0;           // units of 256 candidates scored in the current pass (the same in every thread)
  // this thread's best candidate of the pass
  Winner mine;
  mine.hi = 0; mine.lo = 0; mine.cost = 1; mine.cand = NONE32; mine.exact = 0; mine.tau_o = 0; mine.tau_i = 0; mine.slot = NONE32;
  u32 floor2 = 0;               // largest bound among the candidates this thread scored in the pass other than `mine`

  struct CandV { uint4 A, B; uint2 id; u32 p, t; };
  auto load_cand = [&](u32 u, u32 tid) -> CandV {
    CandV c;
    c.t = uniform((u32)alist[u >> a.tshift]);
    c.p = (((c.t << a.tshift) + (u & ((1u << a.tshift) - 1u))) << 8) + (tid & 255u);
    c.A = a.cd.A[c.p]; c.B = a.cd.B[c.p]; c.id = a.cd.id[c.p];
    return c;
  };

  // Scores the listed tiles: four wavefronts per 256 candidates, the next
  // candidate's record already in flight.  One workgroup has one texture
  // unit, about one cache line per clock: lanes whose candidate is dead load
  // nothing, and struck destinations are written back so later passes skip them.
  auto score_list = [&](const u32 thr_pub) {
    const u32 tid = thread_here(), lane = tid & 63u;
    const u32 nunits = uniform(S->ntl) << a.tshift;
    PrefixView pv; pv.px = tl.px; pv.base = base; pv.K = K; pv.nch = nch; pv.shift_ch = tl.shift_ch;
    Machine mc; mc.bwo0 = bwo0; mc.bwo1 = bwo1; mc.bwi0 = bwi0; mc.bwi1 = bwi1;
    mc.ivo0 = ivo0; mc.ivo1 = ivo1; mc.ivi0 = ivi0; mc.ivi1 = ivi1;
    u32 u = uniform(tid >> 8);
    CandV cur;
    if (u < nunits) cur = load_cand(u, tid);
    while (u < nunits) {
      const u32 un = u + LB / UNIT;
      CandV nxt;
      if (un < nunits) nxt = load_cand(un, tid);
      const uint4 A = cur.A, B = cur.B;
      const Score r = score_candidate(pv, mc, A, B);
      if (r.strike0) a.cd.A[cur.p] = make_uint4(A.x, A.y, 1u, 0u);
      if (r.strike1) a.cd.B[cur.p] = make_uint4(1u, 0u, B.z, B.w);
      u32 exact = 0;
      bool lowered = false;
      Score rr = r;
      if (CLIP && (rr.ok0 || rr.ok1)) {          // the band bounds the area; a value computed earlier bounds it closer
        const uint2 e = a.cd.ce[cur.p];
        if (e.y & 1u) {
          const uint4 v = a.cd.cv[cur.p];
          const u64 vlo = ((u64)v.y << 32) | v.x, vhi = ((u64)v.w << 32) | v.z;
          const u32 vd = (e.y >> 1) & 1u, pd = rr.ok0 ? 0u : 1u;
          if (vd == 0u && rr.ok0 && gt128(rr.h0, rr.l0, vhi, vlo)) { rr.h0 = vhi; rr.l0 = vlo; }
          if (vd == 1u && rr.ok1 && gt128(rr.h1, rr.l1, vhi, vlo)) { rr.h1 = vhi; rr.l1 = vlo; }
          lowered = true;
          exact = (vd == pd && e.x == (u32)S->n_iter) ? 1u : 0u;   // (the number of the pass stamps the values computed in it)
        }
      }
      u64 c0 = 1, c1 = 1;
      u32 kc;                                    // bound of the candidate: the larger of its destinations' keys
      if (RATIO) {
        if (rr.ok0 || rr.ok1) costs_of(mc, ((u64)B.w << 32) | B.z, c0, c1);
        const u32 k0 = key_up_of<true>(rr.h0, rr.l0, c0), k1 = key_up_of<true>(rr.h1, rr.l1, c1);
        kc = k0 > k1 ? k0 : k1;
      } else {
        const bool one = gt128(rr.h1, rr.l1, rr.h0, rr.l0);
        kc = upkey(one ? rr.h1 : rr.h0, one ? rr.l1 : rr.l0);
      }
      const u32 k = wave_max(kc);
      if (lane == 0 && k) atomicMax(&keys[cur.t], k);
      // flash first; host only if flash cannot take it
      const bool ok_any = rr.ok0 || rr.ok1;
      const u32 d = rr.ok0 ? 0u : 1u;
      const u64 hi = ok_any ? (d ? rr.h1 : rr.h0) : 0ull, lo = ok_any ? (d ? rr.l1 : rr.l0) : 0ull, cost = d ? c1 : c0;
      u32 listed = NONE32;                       // the candidate's entry in the list of the pass
      if (MC) {
        // every candidate whose bound reaches the list's threshold goes on the list of the pass
        // with all a commit needs; the others count with their bound only (floor2)
        // (a candidate whose area has been found below its band is not listed: picks stand for bands)
        const bool pub = kc >= thr_pub && kc != 0u && !lowered;
        const u64 pm = __ballot(pub);
        u32 slot = NONE32;
        if (pm) {
          const u32 leader = (u32)__builtin_ctzll(pm);
          u32 off = 0;
          if (lane == leader) off = atomicAdd(&S->nlist, (u32)__popcll(pm));
          off = (u32)__builtin_amdgcn_readlane((int)off, (int)leader);
          slot = off + (u32)__popcll(pm & ((1ull << lane) - 1ull));
        }
        if (pub && slot < lcap) {
          listed = slot;
          list_at(LE_A, slot) = A; list_at(LE_B, slot) = B;
          list_at(LE_I, slot) = make_uint4(cur.id.x, cur.id.y, cur.p, 0u);
          list_ot(slot, 0) = rr.ok0 ? rr.ot0 : NONE64; list_ot(slot, 1) = rr.ok1 ? rr.ot1 : NONE64;
          list_f(LE_O0, slot) = make_double2(exactf(rr.fL0), exactf(rr.fa0)); list_f(LE_I0, slot) = make_double2(exactf(rr.fb0), exactf(rr.fR0));
          list_f(LE_O1, slot) = make_double2(exactf(rr.fL1), exactf(rr.fa1)); list_f(LE_I1, slot) = make_double2(exactf(rr.fb1), exactf(rr.fR1));
          lkey[slot] = upkey(rr.h0, rr.l0); lkey[lcap + slot] = upkey(rr.h1, rr.l1);
        } else if (kc > floor2) floor2 = kc;
      }
      if ((hi | lo) != 0 && (RATIO ? better_ratio(hi, lo, cost, cur.id.x, mine.hi, mine.lo, mine.cost, mine.cand)
                                   : better(hi, lo, cur.id.x, mine.hi, mine.lo, mine.cand))) {
        mine.hi = hi; mine.lo = lo; mine.cost = cost; mine.cand = cur.id.x; mine.tensor = cur.id.y; mine.pos = cur.p; mine.dest = d;
        mine.L1 = A.x; mine.R = A.y; mine.a = d ? B.x : A.z; mine.b = d ? B.y : A.w; mine.s = ((u64)B.w << 32) | B.z;
        mine.fo_base = rr.fo_L; mine.fi_end = rr.fi_R; mine.exact = exact; mine.slot = listed;
      }
      u = un;
      cur = nxt;
    }
    if (tid == 0) S->units += nunits;
    pass_units += nunits;
  };

  // Bounds of the groups that hold tiles scored in the round, by LW - 1 wavefronts (this one is number w of
  // them): tile by tile where they are few, else the groups with any mark (a round of 840 tiles in 70 groups
  // spent 17 us here tile by tile).
  auto group_bounds = [&](const u32 w) {
    const u32 lane = thread_here() & 63u;
    const u32 ntl = uniform(S->ntl);
    const bool few = ntl <= 2 * (LW - 1);
    for (u32 i = w; i < (few ? ntl : ns); i += LW - 1) {
      const u32 g = few ? uniform((u32)alist[i]) >> 6 : i, t = g * 64 + lane;
      if (!few && uniform(smark[g]) == 0ull) continue;
      const u32 k = wave_max(t < nt ? keys[t] : 0u);
      if (lane == 0) skeys[g] = k;
    }
  };

  // block-wide arg-max of the threads' best (two barriers); refreshes the group bounds in between
  auto reduce_best = [&]() {
    const u32 bl = best_lane<RATIO>(mine.hi, mine.lo, mine.cost, mine.cand);
    if (bl == NONE32) { if (lane == 0) { S->wave_win[wave].hi = 0; S->wave_win[wave].lo = 0; S->wave_win[wave].cost = 1; S->wave_win[wave].cand = NONE32; } }
    else if (lane == bl) S->wave_win[wave] = mine;
    if (MC) {
      const u32 f2 = wave_max(floor2);
      if (lane == 0) S->wave_f2[wave] = f2;
    }
    __syncthreads();                               // all tile bounds and wavefront winners are in LDS
    if (wave) group_bounds(wave - 1);
    if (wave == 0) {
      u64 h = 0, l = 0, cs = 1;
      u32 c = NONE32;
      if (lane < LW) { h = S->wave_win[lane].hi; l = S->wave_win[lane].lo; cs = S->wave_win[lane].cost; c = S->wave_win[lane].cand; }
      const u32 w = best_lane<RATIO>(h, l, cs, c);
      if (MC) {
        const u32 f2 = wave_max(lane < LW ? S->wave_f2[lane] : 0u);
        if (lane == 0) S->F2 = f2;
      }
      if (lane == 0) {
        if (w == NONE32) { S->mem[0].hi = 0; S->mem[0].lo = 0; }
        else S->mem[0] = S->wave_win[w];
      }
    }
    __syncthreads();
  };

  // Host bytes of four slots of chunk c (strip st) a lane, brought up to date with the migrations `from` .. `to` - 1 of the plan
  // that cut the chunk (J_HQ says why they are not kept up to date).
  auto host_slots = [&](const u32 c, const u32 st, const bool bring, const u32 from, const u32 to, u64 (&h)[4]) {
    const u32 lane = thread_here() & 63u, j0 = c * CH + st * 256u + lane;
#pragma unroll
    for (u32 i = 0; i < 4; ++i) h[i] = j0 + i * 64u < K ? tl.H[j0 + i * 64u] : 0ull;
    if (!bring) return;
    for (u32 r0 = from; r0 < to; r0 += 64u) {
      const u32 r = r0 + lane;
      const uint4 q = r < to ? a.rec_h[r] : make_uint4(0u, 1u, 0u, 0u);
      const u64 qs = ((u64)q.w << 32) | q.z;
      u32 len = 0;
      const u32 cv = qs ? cover(c, CH, K, q.x, q.y - 1, len) : 0u;
      u64 rel = __ballot(qs != 0ull && cv != 0u && cv != len);
      while (rel) {
        const u32 l = (u32)__builtin_ctzll(rel);
        rel &= rel - 1;
        const u32 x = (u32)__builtin_amdgcn_readlane((int)q.x, (int)l), y = (u32)__builtin_amdgcn_readlane((int)q.y, (int)l);
        const u64 sz = read_lane64(qs, l);
#pragma unroll
        for (u32 i = 0; i < 4; ++i)
          if (j0 + i * 64u < K && in_doubled(j0 + i * 64u, K, x, y - 1) != NONE32) h[i] += sz;
      }
    }
#pragma unroll
    for (u32 i = 0; i < 4; ++i) if (j0 + i * 64u < K) tl.H[j0 + i * 64u] = h[i];
  };

  // ---- chunk jobs: one wavefront rewrites one chunk of one timeline, for all migrations of the
  // pass at once.  A job word: chunk | kind << 16 | set A << 24 | set B << 40, the sets being
  // bits over the pass's migrations: for a transfer-window job, A = the migrations of that
  // destination whose window meets the chunk; for a pressure job, A = those whose absent window
  // cuts the chunk, B = those that cover it whole.  (Host occupancy has no such job: see J_HQ.) --
  // Jobs begin .. end - 1 of the list, about the migrations in `keep`: a job for each wavefront but
  // the last, then whoever is done takes the next one (the last wavefront comes late to a round's
  // jobs, from the plan records and the next round's picks); jnext counts from LW - 1.
  // Slot s0 + 256 st + 64 i + lane belongs to lane `lane` (i = 0..3): every load and store of a job
  // covers 64 neighbouring slots.  A workgroup has one texture unit, about one cache line per clock,
  // and a job for every wavefront runs at once: with four neighbouring slots per lane and one 64-byte record
  // per slot a rewrite touched 64 lines per instruction, now 8 (see the tables of px).
  auto run_jobs = [&](const u32 begin, const u32 end, const u32 keep, const u32 odd) {
    const u32 tid = thread_here(), lane = tid & 63u;
    ulonglong2* const px = reinterpret_cast<ulonglong2*>(tl.px);
    auto take = [&]() -> u32 {
      u32 x = 0;
      if (lane == 0) x = atomicAdd(&S->jnext, 1u);
      return x;                                          // (in lane 0)
    };
    u32 jb = begin + (wave < LW - 1 ? wave : uniform(take()));
    while (jb < end) {
      const u64 jw = uniform(jobs[jb]);
      const u32 after = take();                            // (known by the time this job is done)
      const u32 type = (u32)(jw >> 16) & 0xffu, c = (u32)jw & 0xffffu, ma_ = (u32)(jw >> 24) & keep, mb_ = (u32)(jw >> 40) & keep;
      const u32 s0 = c * CH;
      if (type >= J_FO0 && type <= J_FI1) {
        if (ma_) {
        // channel time of the transfer windows of this destination that meet the chunk is taken
        // from its slots, one migration after the other (windows of one round may meet, see chain);
        // the slots, and the free-time prefixes before them, are stored where they changed
        const bool out = type < J_FI0;
        const u32 d = (type - J_FO0) & 1u;
        const u32 arr = (out ? A_FO : A_FI) + d;
        u64* fr = tl.fre + (u64)((out ? 0u : 2u) + d) * tl.Kp;
        ulonglong2* tab = px + (u64)((out ? T_FO : T_FI) + d) * tl.Kp;
        const u64 bc = base[(u64)arr * nb1 + c], ball = base[(u64)arr * nb1 + nch];
        const u32 mask = ma_;                            // the migrations of this destination whose window meets the chunk
        // (sums of free time inside the chunk stay under its old total: usually 32 bits hold them)
        const bool narrow = uniform((u32)(tot[(u64)arr * nch + c] >> 32)) == 0u;
        // Where windows of the round meet (chain), a migration's free time before its window (fo_base, fi_end) is the one
        // that the earlier ones of the channel left, and so is the free time before a slot here - before the chunk (cb),
        // inside it (loc) and all of the channel's (call).  Migrations behind the last one that meets the chunk change
        // nothing here.
        const bool linked = MC && uniform(S->chain[odd][type - J_FO0]) != 0u;
        const u32 dests = MC ? uniform(S->dests[d]) : 0u;
        const u32 all_of = linked ? dests & ((2u << (31u - (u32)__builtin_clz(mask))) - 1u) : mask;
        u64* const frc = fr + s0;
        ulonglong2* const tabc = tab + s0;
        u64 carry = 0;                                   // the chunk's new total
        for (u32 st = 0; st < tl.spt; ++st) {
          const u32 o = st * 256u + lane, jn = K - s0;   // (slots of the timeline from the chunk's first on)
          u64 fu[4], old[4], now[4], run[4];
#pragma unroll
          for (u32 i = 0; i < 4; ++i) {
            const u32 j = o + i * 64u;
            fu[i] = j < jn ? frc[j] : 0ull;
            old[i] = j < jn ? tabc[j].x : 0ull;          // free time of the chunk before the slot
          }
          if (exact) {
            // A migration takes what lies between its window's end point `ref` and tau of free time from there - ahead
            // of it for an eviction (the earliest free time first), behind it for a prefetch (the latest): so from
            // a slot the difference of the two clamped distances of its ends, 0 outside the window, and from the
            // free time before a slot what it takes between the chunk's start and the slot.  (So no sum over the
            // slots is made anew.)
            double f[4], loc[4], res[4], cb = exactf(bc), call = exactf(ball);
            const double sg = out ? 1.0 : -1.0;
            double end = exactf(tot[(u64)arr * nch + c]), end_res;     // the same for the chunk's end
            if (narrow) {
#pragma unroll
              for (u32 i = 0; i < 4; ++i) { f[i] = (double)(u32)fu[i]; loc[i] = (double)(u32)old[i]; res[i] = loc[i]; }
            } else {
#pragma unroll
              for (u32 i = 0; i < 4; ++i) { f[i] = exactf(fu[i]); loc[i] = exactf(old[i]); res[i] = loc[i]; }
            }
            end_res = end;
            for (u32 pb = all_of; pb; pb &= pb - 1) {
              const u32 mi = (u32)__builtin_ctz(pb);
              const Winner& W = S->mem[mi];
              const double ref = (double)(long long)(out ? W.fo_base : W.fi_end), tau = exactf(out ? W.tau_o : W.tau_i);
              const u32 x = uniform(out ? W.L1 : W.b + 1), y = uniform(out ? W.a - 1 : W.R - 1);
              if ((mask >> mi) & 1u) {
                auto place = [&](const double r) {       // the window's first or second place on the doubled timeline, seen from the chunk's start
                  const double p = -sg * r, gc = takenf(p, tau);
#pragma unroll
                  for (u32 i = 0; i < 4; ++i) {
                    const double p0 = __fma_rn(loc[i], sg, p), g0 = takenf(p0, tau), g1 = takenf(__fma_rn(f[i], sg, p0), tau);
                    f[i] = __fma_rn(-sg, g1 - g0, f[i]);
                    res[i] = __fma_rn(-sg, g0 - gc, res[i]);
                  }
                  end_res = __fma_rn(-sg, takenf(__fma_rn(end, sg, p), tau) - gc, end_res);
                };
                if (y < K) place(ref - cb);
                else if (x >= K) place(ref - call - cb);
                else { place(ref - cb); place(ref - call - cb); }     // (no slot lies in both places)
                if (linked) {
#pragma unroll
                  for (u32 i = 0; i < 4; ++i) loc[i] = res[i];
                  end = end_res;
                }
              }
              if (linked) { cb = after_takingf(cb, call, ref, tau, out, y >= K); call -= tau; }
            }
            if (narrow) {
#pragma unroll
              for (u32 i = 0; i < 4; ++i) { now[i] = (u32)f[i]; run[i] = (u32)res[i]; }
            } else {
#pragma unroll
              for (u32 i = 0; i < 4; ++i) { now[i] = (u64)f[i]; run[i] = (u64)res[i]; }
            }
            carry = (u64)end_res;
          } else {
            // the same in whole numbers, one migration a pass: the ratio key, and times over PICK_EXACT
#pragma unroll
            for (u32 i = 0; i < 4; ++i) now[i] = fu[i];
            for (u32 pb = mask; pb; pb &= pb - 1) {
              const Winner& W = S->mem[__builtin_ctz(pb)];
              const u32 x = uniform(out ? W.L1 : W.b + 1), y = uniform(out ? W.a - 1 : W.R - 1);
              const u64 tau = out ? W.tau_o : W.tau_i, ref = out ? W.fo_base : W.fi_end;
#pragma unroll
              for (u32 i = 0; i < 4; ++i) {
                const u32 j = s0 + o + i * 64u;
                const u32 jj = j < K ? in_doubled(j, K, x, y) : NONE32;
                if (jj != NONE32) {
                  const u64 before_slot = (jj >= K ? ball : 0ull) + bc + old[i];  // free time before slot jj
                  // eviction: earliest free time of the window first; prefetch: latest free time first
                  const u64 gone = out ? before_slot - ref : ref - (before_slot + now[i]);
                  const u64 used = gone < tau ? gone : tau;
                  now[i] -= now[i] < tau - used ? now[i] : tau - used;
                }
              }
            }
            if (narrow) scan_strips<u32>(now, run, carry);
            else scan_strips<u64>(now, run, carry);
          }
#pragma unroll
          for (u32 i = 0; i < 4; ++i) {
            const u32 j = o + i * 64u;
            if (now[i] != fu[i]) frc[j] = now[i];        // (slots beyond the timeline hold 0)
            if (j < jn && run[i] != old[i]) tabc[j].x = run[i];
          }
        }
        if (lane == 0) tot[(u64)arr * nch + c] = carry;
        }
      } else if (type == J_P) {
        // pressure of the chunk's slots: the migrations whose absent window cuts the chunk are
        // taken off slot by slot, the ones that cover it whole go into the chunk's lazy add
        // (here, not by the chunk's thread); where a slot drops under the capacity the
        // over-capacity prefix after it is rewritten
        const u64 lz0 = lazyP[c];                        // the lazy add before this pass
        u64 lz_full = 0;
        const u32 part = ma_;                            // migrations whose window cuts the chunk; mb_: those that cover it whole
        u64 mn = NONE64, carry = 0;
        u32 first = NONE32;                              // first slot that dropped under the capacity
        const bool narrow = uniform((u32)(tot[(u64)A_OT * nch + c] >> 32)) == 0u;   // (the over-capacity time only falls)
        u64* const Pc = tl.P + s0;
        const u64* const durc = tl.dur + s0;
        for (u32 st = 0; st < tl.spt; ++st) {
          const u32 j0 = s0 + st * 256u + lane, o = st * 256u + lane, jn = K - s0;
          u64 p[4], sub[4];
#pragma unroll
          for (u32 i = 0; i < 4; ++i) {
            const u32 j = o + i * 64u;
            p[i] = j < jn ? Pc[j] : 0ull;
            sub[i] = 0;
          }
          if (st == 0) for (u32 pb = mb_; pb; pb &= pb - 1) lz_full += S->mem[__builtin_ctz(pb)].s;
          const u64 lz = lz0 + lz_full;
          for (u32 pb = part; pb; pb &= pb - 1) {
            const Winner& W = S->mem[__builtin_ctz(pb)];
            const u32 x = uniform(W.a), y = uniform(W.b);
            const u64 s = W.s;
            // its slots: [x, y], both less K where it lies in the second iteration, or all but the (y - K, x) between
            const bool both = x < K && y >= K;
            const u32 lo = both ? y - K + 1 : x >= K ? x - K : x, n = both ? x - lo : y - x + 1;
#pragma unroll
            for (u32 i = 0; i < 4; ++i)
              if ((j0 + i * 64u - lo < n) != both) sub[i] += s;        // (beyond the timeline: not stored)
          }
          u32 myfirst = NONE32, overs = 0;               // (overs: a bit per slot over the capacity)
#pragma unroll
          for (u32 i = 0; i < 4; ++i) {
            const u64 before = p[i] - lz0, act = p[i] - sub[i] - lz;       // pressure before and after this pass
            const bool in = o + i * 64u < jn;
            if (in && sub[i]) Pc[o + i * 64u] = p[i] - sub[i];
            const bool over = in && act > cap;
            mn = over && act < mn ? act : mn;
            overs |= over ? 1u << i : 0u;
            if (in && !over && before > cap && myfirst == NONE32) myfirst = j0 + i * 64u;
          }
          if (first == NONE32) {
            first = wave_min(myfirst);
            if (first != NONE32 && st) carry = px[s0 + st * 256u].y;   // (nothing before this slot changes)
          }
          if (first != NONE32) {                         // rewrite the prefix of the slots after it (most jobs let no slot drop)
            u64 v[4], run[4];
#pragma unroll
            for (u32 i = 0; i < 4; ++i) v[i] = (overs >> i) & 1u ? durc[o + i * 64u] : 0ull;
            if (narrow) scan_strips<u32>(v, run, carry);
            else scan_strips<u64>(v, run, carry);
#pragma unroll
            for (u32 i = 0; i < 4; ++i) {
              const u32 j = j0 + i * 64u;
              if (j < K && j > first) {
#pragma unroll
                for (u32 t = 0; t < 4; ++t) px[(u64)t * tl.Kp + j].y = run[i];   // the four copies of OT
              }
            }
          }
        }
        {                                                // the minimum: its high word, then the low one among those
          const u32 hi = wave_min((u32)(mn >> 32)), lo = wave_min((u32)(mn >> 32) == hi ? (u32)mn : NONE32);
          mn = ((u64)hi << 32) | lo;
        }
        if (lane == 0) {
          minOver[c] = mn; lazyP[c] = lz0 + lz_full;
          if (first != NONE32) { tot[(u64)A_OT * nch + c] = carry; S->ot_changed = 1; if (MC) atomicOr(&hpend[c], 2u); }
        }
      } else if (type == J_CLIP) {
        // clipped area of the winner's absent window inside this chunk: per slot over the
        // capacity, duration x min(size, excess)
        const u32 wa = S->mem[0].a, wb = S->mem[0].b;
        const u64 s = S->mem[0].s;
        const u64 lz = lazyP[c];
        u64 alo = 0, ahi = 0;
        for (u32 st = 0; st < tl.spt; ++st) {
          const u32 j0 = s0 + st * 256u + lane;
#pragma unroll
          for (u32 i = 0; i < 4; ++i) {
            const u32 j = j0 + i * 64u;
            if (j < K && in_doubled(j, K, wa, wb) != NONE32) {
              const u64 act = tl.P[j] - lz;
              if (act > cap) {
                const u64 e = act - cap, m = e < s ? e : s, dj = tl.dur[j];
                const u64 plo = dj * m;
                ahi += __umul64hi(dj, m) + (alo + plo < alo ? 1ull : 0ull);
                alo += plo;
              }
            }
          }
        }
        const u64 p0 = wave_sum(alo & 0xffffffffull), p1 = wave_sum(alo >> 32), p2 = wave_sum(ahi);
        if (lane == 0) {
          atomicAdd((unsigned long long*)&S->acc[0], (unsigned long long)p0);
          atomicAdd((unsigned long long*)&S->acc[1], (unsigned long long)p1);
          atomicAdd((unsigned long long*)&S->acc[2], (unsigned long long)p2);
        }
      } else {
        // J_HQ: the largest host occupancy over the winner's period inside the chunk.  The slots'
        // host bytes are kept up to date on demand only: a migration to host that covers a chunk
        // whole goes into the chunk's lazy add when it is committed, one that cuts it is only
        // counted into the chunk's bound then (hmax, hpend); here the migrations committed since
        // the chunk was last brought up to date (hmat) are looked through, 64 at a time, and those
        // that cut the chunk are added to its slots, after which the bound is exact again.
        const u32 L1 = S->mem[0].L1, R = S->mem[0].R;
        const u64 lz = lazyH[c];
        const bool bring = (hpend[c] & 1u) != 0u;
        const u32 from = hmat[c], to = (u32)S->n_mig;
        u64 m_cov = 0, m_all = 0;
        for (u32 st = 0; st < tl.spt; ++st) {
          const u32 j0 = s0 + st * 256u + lane;
          u64 h[4];
          host_slots(c, st, bring, from, to, h);
#pragma unroll
          for (u32 i = 0; i < 4; ++i) {
            const u32 j = j0 + i * 64u;
            if (j < K) {
              const u64 act = h[i] + lz;
              m_all = act > m_all ? act : m_all;
              if (in_doubled(j, K, L1, R - 1) != NONE32) m_cov = act > m_cov ? act : m_cov;
            }
          }
        }
        m_cov = wave_max(m_cov);
        if (bring) {
          m_all = wave_max(m_all);
          if (lane == 0) { hmax[c] = m_all; hmat[c] = to; hpend[c] &= ~1u; }
        }
        if (lane == 0) atomicMax((unsigned long long*)&S->hq, (unsigned long long)m_cov);
      }
      jb = begin + uniform(after);
    }
    if (tid == 0) S->jobs += end - begin;
  };

  // Host memory's room for the entries the picking wavefront holds that can go there only, in the state as it is: a chunk a
  // wavefront; an entry whose period covers the chunk whole takes the chunk's maximum, one that cuts it the maximum over its
  // slots.  An entry without room is refused when its turn comes (PK_DROP), in a round with others: it changes nothing that the
  // entries behind it depend on.  (Loops, one candidate tested and refused per ranking pass / this: the encoder with 1031 refused
  // ones 15.8 / 3.15 ms, the decoder with 6275 89.8 / 24.7, ResNet with 1118 19.5 / 5.5, 105 000 tensors on 29 000 slots with 102 894
  // 2490 / 190.)
  auto probe_host = [&]() {
    const u32 tid = thread_here(), lane = tid & 63u;
    u64* const room = (u64*)S->wave_win;                 // [64] the largest occupancy over the entry's period
    static_assert(sizeof(S->wave_win) >= G10_WAVE * 8, "a word an entry");
    if (tid < G10_WAVE) room[tid] = 0;
    const u32 nl_ = uniform(S->nlist), n = nl_ < lcap ? nl_ : lcap;
    if (tid < n) list_at(LE_I, tid).w &= ~E_ROOM;        // (of an earlier state)
    __syncthreads();
    u32 x = 1, y = 0, slot = NONE32;                     // its period [x, y] (y < x: none)
    u64 s = 0;
    if (lane < uniform(S->nsel)) {
      const u32 i = S->sel[lane];
      if (list_ot(i, 0) == NONE64 && list_ot(i, 1) != NONE64) {
        const uint4 A = list_at(LE_A, i), B = list_at(LE_B, i);
        slot = i; x = A.x; y = A.y - 1; s = ((u64)B.w << 32) | B.z;
      }
    }
    const u32 to = (u32)uniform(S->n_mig);
    for (u32 c = wave; c < nch; c += LW) {
      u32 len = 0;
      const u32 cv = slot != NONE32 ? cover(c, CH, K, x, y, len) : 0u;
      const bool whole = cv != 0u && cv == len;
      const u64 cuts = __ballot(cv != 0u && !whole);
      if (!cuts && !__any(whole)) continue;
      const bool bring = (uniform(hpend[c]) & 1u) != 0u;
      u64 most = hmax[c];                                // (exact where nothing is missing)
      if (cuts || bring) {
        const u64 lz = lazyH[c];
        const u32 from = uniform(hmat[c]);
        u64 all = 0;
        for (u32 st = 0; st < tl.spt; ++st) {
          u64 h[4];
          host_slots(c, st, bring, from, to, h);
          const u32 j0 = c * CH + st * 256u + lane;
          for (u64 cb = cuts; cb; cb &= cb - 1) {
            const u32 l = (u32)__builtin_ctzll(cb);
            const u32 px_ = (u32)__builtin_amdgcn_readlane((int)x, (int)l), py_ = (u32)__builtin_amdgcn_readlane((int)y, (int)l);
            u64 mx = 0;
#pragma unroll
            for (u32 i = 0; i < 4; ++i) {
              const u32 j = j0 + i * 64u;
              if (j < K && in_doubled(j, K, px_, py_) != NONE32) mx = h[i] + lz > mx ? h[i] + lz : mx;
            }
            mx = wave_max(mx);
            if (lane == 0) atomicMax((unsigned long long*)&room[l], (unsigned long long)mx);
          }
#pragma unroll
          for (u32 i = 0; i < 4; ++i) if (j0 + i * 64u < K) all = h[i] + lz > all ? h[i] + lz : all;
        }
        if (bring) {
          most = wave_max(all);
          if (lane == 0) { hmax[c] = most; hmat[c] = to; hpend[c] &= ~1u; }
        }
      }
      if (whole) atomicMax((unsigned long long*)&room[lane], (unsigned long long)most);
    }
    __syncthreads();
    if (wave == LW - 1) {
      if (slot != NONE32) list_at(LE_I, slot).w |= s <= host_cap && room[lane] <= host_cap - s ? E_ROOM : E_NOROOM;
      if (lane == 0) S->probed = 1;
    }
  };

  // The next best entries of the list of the pass, a list entry per lane of one wavefront (entry: {period and windows},
  // identity, over-capacity times, free channel times): entry by entry in the order of their benefit, as far as it is
  // certain that each wins Algorithm 1's next pass (see "more migrations of the same pass" below).  F bounds every
  // candidate that is not on the list; at most `allowed` migrations are made.  Picked entries go to mem[]; the number of
  // migrations is returned.
  struct Entry { uint4 A, B, I; u64 ot0, ot1; double2 O0, I0, O1, I1; u32 k0, k1; };
  auto load_entry = [&](const u32 i) -> Entry {          // (NONE32: none)
    Entry e;
    const double2 z = make_double2(0.0, 0.0);
    e.A = make_uint4(1u, 1u, 1u, 0u); e.B = make_uint4(1u, 0u, 0u, 0u); e.I = make_uint4(NONE32, 0u, 0u, 0u);
    e.ot0 = NONE64; e.ot1 = NONE64; e.O0 = z; e.I0 = z; e.O1 = z; e.I1 = z; e.k0 = 0u; e.k1 = 0u;
    if (i != NONE32) {
      e.A = list_at(LE_A, i); e.B = list_at(LE_B, i); e.I = list_at(LE_I, i); e.ot0 = list_ot(i, 0); e.ot1 = list_ot(i, 1);
      e.O0 = list_f(LE_O0, i); e.I0 = list_f(LE_I0, i); e.O1 = list_f(LE_O1, i); e.I1 = list_f(LE_I1, i);
      e.k0 = lkey[i]; e.k1 = lkey[lcap + i];
    }
    return e;
  };
  // The entries of the list scored again, against the timelines as the rounds so far left them: a thread per entry and
  // destination, whole wavefronts per destination.
  static_assert(2 * LIST_MAX <= LOOP_MAX, "a thread per entry and destination");
  auto rescore_list = [&](const u32 n) {
    const u32 tid = thread_here();
    const u32 n64 = (n + 63u) & ~63u, d = uniform((u32)(tid >= n64 ? 1u : 0u)), i = tid - (d ? n64 : 0u);
    if (tid < 2 * n64 && i < n) {
      const uint4 A = list_at(LE_A, i), B = list_at(LE_B, i);
      const u32 wa = d ? B.x : A.z, wb = d ? B.y : A.w;
      u64 ot = NONE64;
      u32 key = 0;
      if (wa <= wb) {
        const bool sL = A.x >= K, sR = A.y >= K, sa = wa >= K, sb = wb + 1 >= K;
        const u32 jL = sL ? A.x - K : A.x, jR = sR ? A.y - K : A.y, ja = sa ? wa - K : wa, jb = sb ? wb + 1 - K : wb + 1;
        const ulonglong2* const to = reinterpret_cast<const ulonglong2*>(tl.px) + (u64)(T_FO + d) * tl.Kp;
        const ulonglong2* const ti = reinterpret_cast<const ulonglong2*>(tl.px) + (u64)(T_FI + d) * tl.Kp;
        const ulonglong2 gL = to[jL], ga = to[ja], gb = ti[jb], gR = ti[jR];
        const u64 *bO = base + (u64)(A_FO + d) * nb1, *bI = base + (u64)(A_FI + d) * nb1, *bT = base + (u64)A_OT * nb1;
        const u64 allO = bO[nch], allI = bI[nch], allT = bT[nch], s = ((u64)B.w << 32) | B.z, x1000 = s * 1000ull;
        const u32 cL = jL >> tl.shift_ch, cR = jR >> tl.shift_ch, ca = ja >> tl.shift_ch, cb = jb >> tl.shift_ch;
        const u64 fL = (sL ? allO : 0ull) + bO[cL] + gL.x, fa = (sa ? allO : 0ull) + bO[ca] + ga.x;
        const u64 fb = (sb ? allI : 0ull) + bI[cb] + gb.x, fR = (sR ? allI : 0ull) + bI[cR] + gR.x;
        list_f(d ? LE_O1 : LE_O0, i) = make_double2(exactf(fL), exactf(fa));
        list_f(d ? LE_I1 : LE_I0, i) = make_double2(exactf(fb), exactf(fR));
        if (carries(fa - fL, d ? bwo1 : bwo0, x1000) && carries(fR - fb, d ? bwi1 : bwi0, x1000)) {
          ot = ((sb ? allT : 0ull) + bT[cb] + gb.y) - ((sa ? allT : 0ull) + bT[ca] + ga.y);
          key = upkey(__umul64hi(s, ot), s * ot);
        }
      }
      list_ot(i, d) = ot;
      lkey[d * lcap + i] = key;
    }
    for (u32 c = tid; c < nch; c += LB) hpend[c] &= 1u;
    if (tid == 0) S->list_rescored += n;
  };
  // The entry this lane of the picking wavefront looks at (NONE32: none): all n entries, or the 64 with the best bounds,
  // equal keys by the lowest index.  What is left out counts with `fl`: its largest key and, where an entry looked at has
  // that key too, the best bound in full (value and index) among those left out with it.
  auto choose = [&](const u32 n, const u32 F, Floor& fl) -> u32 {
    fl.key = F; fl.full = 0u; fl.hi = 0; fl.lo = 0; fl.cand = 0; fl.pad = 0;
    if (n <= G10_WAVE) {
      if (lane == 0) S->nsel = n;
      S->sel[lane] = lane;
      return lane < n ? lane : NONE32;
    }
    constexpr u32 Q = LIST_MAX / G10_WAVE;
    u32 k[Q], top = 0;
#pragma unroll
    for (u32 q = 0; q < Q; ++q) {
      const u32 i = q * G10_WAVE + lane;
      const u32 k0 = i < n ? lkey[i] : 0u, k1 = i < n ? lkey[lcap + i] : 0u;
      k[q] = k0 > k1 ? k0 : k1;
      top = k[q] > top ? k[q] : top;
    }
    top = wave_max(top);
    if (top <= F) { if (lane == 0) S->nsel = 0; return NONE32; }
    auto above = [&](u32 t) -> u32 { u32 c = 0;
#pragma unroll
      for (u32 q = 0; q < Q; ++q) c += (u32)__popcll(__ballot(k[q] > t));
      return c; };
    u32 t = F, x = 0u;                             // chosen: keys above t; of those at t the ones with an index below x
    if (above(F) > G10_WAVE) {
      u32 lo = F, hi = top;                        // above(lo) > 64 >= above(hi)
      while (hi - lo > 1u) {
        const u32 mid = lo + (hi - lo) / 2u;
        const u32 c = above(mid);
        if (c > G10_WAVE) lo = mid;
        else { hi = mid; if (c >= G10_WAVE / 2) break; }             // (near enough)
      }
      t = hi;
      fl.key = t;
      const u32 room = hi - lo > 1u ? 0u : G10_WAVE - above(t);
      if (room) {                                  // (more than that have key t: above(t - 1) > 64)
        u32 id[Q];
#pragma unroll
        for (u32 q = 0; q < Q; ++q) id[q] = k[q] == t ? list_at(LE_I, q * G10_WAVE + lane).x : NONE32;
        auto under = [&](u32 y) -> u32 { u32 c = 0;
#pragma unroll
          for (u32 q = 0; q < Q; ++q) c += (u32)__popcll(__ballot(k[q] == t && id[q] < y));
          return c; };
        u32 ylo = 0, yhi = NONE32;                 // under(ylo) <= room < under(yhi): indices are distinct
        while (yhi - ylo > 1u) {
          const u32 mid = ylo + (yhi - ylo) / 2u;
          if (under(mid) > room) yhi = mid; else ylo = mid;
        }
        x = ylo;
        // the best of those left out with key t
        u64 bh = 0, bl = 0;
        u32 bc = NONE32;
#pragma unroll
        for (u32 q = 0; q < Q; ++q) {
          const bool out = k[q] == t && id[q] >= x;
          if (!__any(out)) continue;
          if (out) {
            const u32 i = q * G10_WAVE + lane;
            const uint4 B = list_at(LE_B, i);
            const u64 sz = ((u64)B.w << 32) | B.z;
            const u64 t0 = list_ot(i, 0), t1 = list_ot(i, 1), o0 = t0 == NONE64 ? 0ull : t0, o1 = t1 == NONE64 ? 0ull : t1;
            const u64 o = o0 > o1 ? o0 : o1, h = __umul64hi(sz, o), l = sz * o;
            if (better(h, l, id[q], bh, bl, bc)) { bh = h; bl = l; bc = id[q]; }
          }
        }
        fl.full = 1u;
        fl.hi = wave_max(bh);
        fl.lo = wave_max(bh == fl.hi ? bl : 0ull);
        fl.cand = wave_min(bh == fl.hi && bl == fl.lo ? bc : NONE32);
      }
    }
    u32 cnt = 0;
#pragma unroll
    for (u32 q = 0; q < Q; ++q) {
      const u32 i = q * G10_WAVE + lane;
      bool in = k[q] > t;
      if (x && k[q] == t) in = list_at(LE_I, i).x < x;
      const u64 mk = __ballot(in);
      if (in) S->sel[cnt + (u32)__popcll(mk & ((1ull << lane) - 1ull))] = i;
      cnt += (u32)__popcll(mk);
    }
    if (lane == 0) S->nsel = cnt;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    return lane < cnt ? S->sel[lane] : NONE32;
  };
  auto pick = [&](const Entry& e, const u32 slot, const Floor& fl, const u32 F, const u32 allowed, const bool fresh, const u32 odd) -> u32 {
    const u32 lane = thread_here() & 63u;
    const u64 s = ((u64)e.B.w << 32) | e.B.z;
    const u32 R = e.A.y;
    bool ok0 = e.ot0 != NONE64, ok1 = e.ot1 != NONE64, open = true;
    // free times before the ends of the windows, transfer times
    double f0L = e.O0.x, f0a = e.O0.y, f0b = e.I0.x, f0R = e.I0.y, f1L = e.O1.x, f1a = e.O1.y, f1b = e.I1.x, f1R = e.I1.y;
    const double x1000 = exactf(s) * 1000.0;
    const double to0 = ceil_divf(x1000, S->bw[0], S->bw[4]), to1 = ceil_divf(x1000, S->bw[1], S->bw[5]),
                 ti0 = ceil_divf(x1000, S->bw[2], S->bw[6]), ti1 = ceil_divf(x1000, S->bw[3], S->bw[7]);
    double all_o0 = fresh ? exactf(base[(u64)(A_FO + 0) * nb1 + nch]) : S->all[0], all_o1 = fresh ? exactf(base[(u64)(A_FO + 1) * nb1 + nch]) : S->all[1],
           all_i0 = fresh ? exactf(base[(u64)(A_FI + 0) * nb1 + nch]) : S->all[2], all_i1 = fresh ? exactf(base[(u64)(A_FI + 1) * nb1 + nch]) : S->all[3];
    u32 ch_o0 = 0, ch_o1 = 0, ch_i0 = 0, ch_i1 = 0;    // a window of a pick met one of an entry
    const bool wrap = __any(R > K);                    // (something lies in the second iteration)
    const u64 noroom = TIGHT ? __ballot((e.I.w & E_NOROOM) != 0u) : 0ull;
    const u32 word = TIGHT ? slot | (e.I.w & E_NOROOM ? PK_DROP : 0u) | (e.I.w & E_ROOM ? PK_ROOM : 0u) : slot;
    u32 m = 0, by_floor = 0;
    while (true) {
      // flash first; host only if flash cannot take it.  (0: cannot be picked)
      const u32 kB = open ? (ok0 ? e.k0 : ok1 ? e.k1 : 0u) : 0u;
      const u32 kmax = wave_max(kB);
      if (kmax <= F) { by_floor = fl.key <= F ? 1u : 0u; break; }     // (also when nothing is left)
      if (kmax < fl.key || (kmax == fl.key && !fl.full)) break;
      const bool in1 = kB == kmax;
      const u64 m1 = __ballot(in1);
      u32 bl = (u32)__builtin_ctzll(m1);
      const u64 ot = ok0 ? e.ot0 : e.ot1;
      if (m1 & (m1 - 1)) {                             // equal keys
        const u64 s_ = read_lane64(s, bl), ot_ = read_lane64(ot, bl);
        bool in3 = in1;
        if (__any(in1 && (s != s_ || ot != ot_))) {    // high word, low word (mostly the sizes and times are equal: a layer repeats)
          const u64 hi = __umul64hi(s, ot), lo = s * ot;
          const u64 hmx = wave_max(in1 ? hi : 0ull);
          const bool in2 = in1 && hi == hmx;
          const u64 lmx = wave_max(in2 ? lo : 0ull);
          in3 = in2 && lo == lmx;
        }
        const u32 cmin = wave_min(in3 ? e.I.x : NONE32);               // lowest index
        bl = (u32)__builtin_ctzll(__ballot(in3 && e.I.x == cmin));
      }
      if (kmax == fl.key) {                            // (as large a bound was left out: the whole values decide)
        const u64 s_ = read_lane64(s, bl), ot_ = read_lane64(ot, bl);
        if (!better(__umul64hi(s_, ot_), s_ * ot_, (u32)__builtin_amdgcn_readlane((int)e.I.x, (int)bl), fl.hi, fl.lo, fl.cand)) break;
      }
      const u64 flash = __ballot(ok0);
      const u32 d = (flash >> bl) & 1ull ? 0u : 1u;
      if (lane == bl) {
        S->pick[m] = word | d << 16;
        S->pick_o[m] = d ? f1L : f0L; S->pick_i[m] = d ? f1R : f0R;
        open = false;
      }
      ++m;
      // The free times of the entries become those that the picked migration leaves, and an entry that its destination
      // cannot carry any more gets the other destination, or none.
      // (Where no entry's window has less left, none of them meets what the pick took: `chain` stays.)
      auto commit = [&](bool& ok, double& fL, double& fa, double& fb, double& fR, const double to, const double ti,
                        double& all_o, double& all_i, u32& ch_o, u32& ch_i) {
        const double ro = read_lanef(fL, bl), po = read_lanef(to, bl), ri = read_lanef(fR, bl), pi = read_lanef(ti, bl);
        const double nL = after_takingf(fL, all_o, ro, po, true, wrap), nR = after_takingf(fR, all_i, ri, pi, false, wrap);
        const double na = after_takingf(fa, all_o, ro, po, true, wrap), nb = after_takingf(fb, all_i, ri, pi, false, wrap);
        const double wo = na - nL, wi = nR - nb;
        const bool may = open && ok;
        ch_o |= __any(may && wo != fa - fL) ? 1u : 0u; ch_i |= __any(may && wi != fR - fb) ? 1u : 0u;
        if (open) { fL = nL; fa = na; fb = nb; fR = nR; }      // (a picked one keeps its own)
        all_o -= po; all_i -= pi;
        ok = ok && wo >= to && wi >= ti;
      };
      if (d == 0u) commit(ok0, f0L, f0a, f0b, f0R, to0, ti0, all_o0, all_i0, ch_o0, ch_i0);
      else if (!TIGHT || !noroom || !((noroom >> bl) & 1ull)) commit(ok1, f1L, f1a, f1b, f1R, to1, ti1, all_o1, all_i1, ch_o1, ch_i1);   // (refused: nothing changes)
      if (m == allowed) break;
    }
    if (open && slot != NONE32) {                      // what a next round of picks goes on from
      list_f(LE_O0, slot) = make_double2(f0L, f0a); list_f(LE_I0, slot) = make_double2(f0b, f0R);
      list_f(LE_O1, slot) = make_double2(f1L, f1a); list_f(LE_I1, slot) = make_double2(f1b, f1R);
      if (!ok0) list_ot(slot, 0) = NONE64;
      if (!ok1) list_ot(slot, 1) = NONE64;
    }
    if (lane == 0) {
      S->chain[odd][0] = ch_o0; S->chain[odd][1] = ch_o1; S->chain[odd][2] = ch_i0; S->chain[odd][3] = ch_i1;
      S->all[0] = all_o0; S->all[1] = all_o1; S->all[2] = all_i0; S->all[3] = all_i1;
      S->m0 = m; S->by_floor = by_floor;
    }
    return m;
  };

  // Clipped-area benefit: the ranking went by bounds (the tensor's band, or a value computed
  // in an earlier pass: both can only be too large).  The best by bound stands only with a
  // value computed in this pass.  Otherwise its area is computed here - whole chunks of its
  // window in which every slot over the capacity exceeds it by the tensor's size count
  // size x over-capacity time, the others are summed slot by slot.  Returns true when the
  // winner stands (or nothing is left).  If the area comes out below the bound it is
  // remembered with the candidate and false is returned: the tiles scored in this pass are
  // then listed again (alist) and must be ranked once more.  (Four barriers; with three more, and words of their own for
  // what the number of jobs carries, an area cost 0.3 us more, 3 % of plans in which most come out below.)
  auto settle = [&]() -> bool {                        // (called behind the barrier that ends reduce_best, or a later one)
    if ((S->mem[0].hi | S->mem[0].lo) == 0 || S->mem[0].exact) return true;
    const u32 wa = S->mem[0].a, wb = S->mem[0].b;
    const u64 s = S->mem[0].s;
    if (tid < nch) {                                   // (no job is listed and the sums are zero: open_pass, and below)
      u32 len = 0;
      const u32 cv = cover(tid, CH, K, wa, wb, len);
      if (cv) {
        const u64 mo = minOver[tid];
        if (cv == len && mo == NONE64) {
          // no slot of the chunk is over the capacity
        } else if (cv == len && mo - cap >= s) {
          const u64 t = tot[(u64)A_OT * nch + tid], lo = s * t;
          atomicAdd((unsigned long long*)&S->acc[0], (unsigned long long)(lo & 0xffffffffull));
          atomicAdd((unsigned long long*)&S->acc[1], (unsigned long long)(lo >> 32));
          atomicAdd((unsigned long long*)&S->acc[2], (unsigned long long)__umul64hi(s, t));
        } else {
          const u32 one = mo != NONE64 && mo - cap < s ? 1u | UNEVEN : 1u;
          jobs[atomicAdd(&S->njobs, one) & (UNEVEN - 1u)] = ((u64)J_CLIP << 16) | tid;
        }
      }
    }
    __syncthreads();
    const u32 nj = uniform(S->njobs);
    const bool even = nj < UNEVEN;                     // (the area is the band: nothing is summed)
    if (!even) run_jobs(0u, nj & (UNEVEN - 1u), 0xffffu, 0u);
    __syncthreads();
    const u64 a0 = S->acc[0], a1 = S->acc[1], a2 = S->acc[2];
    const u64 vlo = a0 + (a1 << 32), vhi = a2 + (a1 >> 32) + (vlo < a0 ? 1ull : 0ull);
    const bool same = even || (vhi == S->mem[0].hi && vlo == S->mem[0].lo);
    if (tid == 0) {                                    // (words that nobody reads before the next barrier)
      S->evals += 1;
      S->njobs = 0; S->jnext = LW - 1;
      if (!RATIO && (!LISTS || !S->lists)) {
        if (!even) S->in_row = 0;
        else if (++S->in_row >= LISTS_AFTER << (S->lists_ended < LISTS_MORE_MAX ? S->lists_ended : LISTS_MORE_MAX) && C - S->n_mig - S->n_drop >= LISTS_LEFT && (!max_iter || max_iter - S->n_iter >= LISTS_PASSES)) { S->lists = 1; S->in_row = 0; if (!LISTS && S->alone) S->stop = 1; }
      }
      if (same) S->mem[0].exact = 1;
      else {
        S->refused += 1;
        if (LISTS) S->no_list = 1;                     // (the tiles scored again are not listed again)
        a.cd.cv[S->mem[0].pos] = make_uint4((u32)vlo, (u32)(vlo >> 32), (u32)vhi, (u32)(vhi >> 32));
        a.cd.ce[S->mem[0].pos] = make_uint2((u32)S->n_iter, 1u | (S->mem[0].dest << 1));
        S->ntl = 0;
      }
    }
    __syncthreads();                                   // everyone has read the sums
    if (tid == 0) { S->acc[0] = 0; S->acc[1] = 0; S->acc[2] = 0; }
    if (same) return true;
    for (u32 g = tid; g < ns; g += LB) {               // every tile scored in this pass, once more
      u64 m = smark[g];
      while (m) {
        const u32 t = g * 64 + (u32)__builtin_ctzll(m);
        m &= m - 1;
        alist[atomicAdd(&S->ntl, 1u)] = (unsigned short)t;
        keys[t] = 0;
      }
    }
    __syncthreads();
    return false;
  };

  // What the next ranking pass finds: made by the last wavefront at the end of the pass before,
  // beside the level-1 update, so that a pass begins without a barrier of its own.
  // (undo: the pass before settled no candidate: it is none of Algorithm 1's)
  auto open_pass = [&](const bool undo) {
    const u32 lane = thread_here() & 63u;
    for (u32 i = lane; i < ns; i += 64u) smark[i] = 0;   // no tile scored yet
    if (lane == 0) {
      if (TIGHT && undo) { S->n_iter -= 1; S->n_evals -= C - S->n_mig - S->n_drop; }
      S->hq = 0; S->njobs = 0; S->ntl = 0; S->filt = 0;
      if (CLIP) S->jnext = LW - 1;
      S->mem[0].hi = 0; S->mem[0].lo = 0;
      S->nlist = 0; S->F2 = 0; S->fast = 0; S->cut = MAXM; S->need_exact = 0; S->by_floor = 0;
      if (S->stale_hot) { S->restL = NONE32; S->stale_hot = 0; }
      if (LISTS) {
        const u64 settled = S->n_mig + S->n_drop;
        if (S->lists) {
          if (settled - S->settled0 > 1u) { S->in_row = 0; S->paid += 1; }
          else S->in_row += 1;
          if (S->in_row >= LISTS_VAIN) {                   // (the other form goes on)
            S->lists = 0; S->in_row = 0;
            if (S->alone) S->stop = 1;
            S->lists_ended = S->paid >= LISTS_PAID ? 0u : S->lists_ended + 1u; S->paid = 0;
          }
        }
        S->no_list = S->lists ? 0u : 1u; S->settled0 = settled;
      }
      S->lim = max_iter && S->n_iter >= max_iter ? 1u : 0u;
      if (a.tick_budget && wall_clock64() - S->t_start > a.tick_budget) S->stop = 1;
    }
  };
  __syncthreads();
  if (wave == LW - 1) open_pass(false);
  if (tid == 0) { S->m0 = 1; S->probed = 0; }
  __syncthreads();
  // ---- passes ------------------------------------------------------------------------
  u32 passes = 0, used = 0;                          // ranking passes of this launch; with the further rounds of commits: what the budget counts
  bool wide_exit = false;
  while (true) {
    u32 thr = uniform(S->thr_key);
    if (!resume) {                                   // (a pass taken up again has passed these tests)
      const u32 done = uniform(S->done), lim = uniform(S->lim), stop = uniform(S->stop);
      const u64 over = uniform(base[(u64)A_OT * nb1 + nch]);
      if (done) break;
      if (over == 0) { if (tid == 0) { S->done = 1; S->status = G10_FITS; } break; }
      if (lim) { if (tid == 0) { S->done = 1; S->status = G10_TRUNCATED; } break; }
      if (used >= a.pass_budget || stop || (a.pass_stop && passes_before + passes >= a.pass_stop)) break;
      if (WIDE && S->no_wide) break;               // (the last launch of a round only ends the pass left open)
      ++passes; ++used;
    }
    mine.hi = 0; mine.lo = 0; mine.cost = 1; mine.cand = NONE32; mine.exact = 0;
    floor2 = 0;
    pass_units = 0;
    if (!thr) thr = NONE32;
    bool fresh = true;
    if (WIDE && resume) {                          // the tiles the open pass has scored, and the list of its open round
      thr = wc.thr;
#pragma unroll
      for (u32 j = 0; j < MPT; ++j) if (tid + j * LB < ns) smark[tid + j * LB] = wmark[j];
#pragma unroll 4
      for (u32 i = tid; i < wc.ntl; i += LB) alist[i] = wv.alist[i];
      if (tid == 0) { S->ntl = wc.ntl; S->filt = 0; S->nl = 0; S->restL = NONE32; S->stale_hot = 0; S->F2 = 0; }
      fresh = false;
      __syncthreads();
    }
    if (tid == 0) {                                // (read again behind the next barrier only)
      if (!(WIDE && resume)) { S->n_iter += 1; S->n_evals += C - S->n_mig - S->n_drop; }
      S->touched = 0; S->ot_changed = 0;
    }
    if (MC) for (u32 c = tid; c < nch; c += LB) hpend[c] &= 1u;

    // rank: score the hot tiles whose bound reaches a threshold (first a guess a little under
    // the last benefit), lower the threshold to the best benefit found, repeat until no tile
    // left out could hold an equal or better candidate
    u32 rounds = 0, rest_final = 0;
    bool again = false;                          // CLIP: the listed tiles are the ones already scored in this pass
    while (true) {
      u32 rest;
      bool decided = false;                      // the best by bound is known
      if (WIDE && resume) {
        rest = wc.rest;
        rounds = wc.rounds;
        pass_units = wc.pass_units;
        if (tid == LB - 1 && rounds) {                         // the best of the rounds before
          if (resume == 1) { const WideKey k = wk[0]; mine.hi = k.hi; mine.lo = k.lo; mine.cost = k.cost; mine.cand = k.cand; mine.slot = WIDE_WG; }
          else mine = wv.win[WIDE_WG];
        }
      } else if (!again) {
        if (uniform(S->restL) >= thr) {                     // the hot list may miss a tile that reaches thr: build it anew,
          const u32 low = thr == NONE32 ? thr : (thr > (1u << 19) ? thr - (1u << 19) : 1u);   // a few percent lower to last a while
          __syncthreads();
          build_hot(low);
          if (rounds && tid == 0) S->stale_hot = 1;  // built without the tiles already scored: not kept for the next pass
        }
        activate(thr, fresh);
        fresh = false;
        const u32 ntl = uniform(S->ntl);
        rest = uniform(S->restL > S->filt ? S->restL : S->filt);
        if (ntl == 0) {
          if ((rounds && (S->mem[0].hi | S->mem[0].lo) != 0) || rest == 0) decided = true;   // nothing left that could win
          else {
            thr = rest;                                  // strictly lower than before: start from the largest bound left
            __syncthreads();
            continue;
          }
        }
      } else {
        again = false;
        rest = S->restL > S->filt ? S->restL : S->filt;
        mine.hi = 0; mine.lo = 0; mine.cost = 1; mine.cand = NONE32; mine.exact = 0;
      }
      if (!decided) {
        if (WIDE && a.wide_min && !resume && !S->no_wide && (S->ntl << a.tshift) >= a.wide_min) {
          // a long round: the list, the tiles marked and what the pass needs to go on (with the
          // best of its earlier rounds) are left for the scoring kernel and the next launch
          const u32 ntl = S->ntl, nu = ntl << a.tshift;
          for (u32 i = tid; i < ns; i += LB) wv.smark[i] = smark[i];
          for (u32 i = tid; i < ntl; i += LB) wv.alist[i] = alist[i];
          if (tid == 0) {
            wv.win[WIDE_WG] = S->mem[0];         // (hi = lo = 0: none yet)
            wv.key[WIDE_WG] = WideKey{S->mem[0].hi, S->mem[0].lo, S->mem[0].cost, S->mem[0].cand, 0u};
            wv.ctx->rounds = rounds; wv.ctx->pass_units = pass_units;
            wv.ctx->ntl = ntl; wv.ctx->thr = thr; wv.ctx->rest = rest;
            wv.ctx->nwg = nu < WIDE_WG ? nu : WIDE_WG; wv.ctx->scored = 0;
            wv.ctx->pending = 1;
            ctl->wide_rounds = wide0 + 1;          // (one a launch at most)
          }
          wide_exit = true;
          break;
        }
        bool from_wide = false;
        if (WIDE && resume == 1) {
          from_wide = true;
          const u32 nw = wc.nwg;
#pragma unroll
          for (u32 q = 0; q < 2; ++q) {
            const u32 i = tid + q * (LB - 1);
            if (tid < LB - 1 && i < nw) {
              const WideKey k = wk[q];
              floor2 = k.skipped > floor2 ? k.skipped : floor2;
              if ((k.hi | k.lo) != 0 && better_ratio(k.hi, k.lo, k.cost, k.cand, mine.hi, mine.lo, mine.cost, mine.cand)) {
                mine.hi = k.hi; mine.lo = k.lo; mine.cost = k.cost; mine.cand = k.cand; mine.slot = i;
              }
            }
          }
          const u32 f2 = wave_max(floor2);
          if (lane == 0 && f2) atomicMax(&S->F2, f2);
          const u32 nu = S->ntl << a.tshift;
          if (tid == 0) S->units += nu;
          pass_units += nu;
        } else {
          u32 low = thr;                           // the list's threshold
          if (LISTS && uniform(S->no_list)) low = NONE32;
          else if (MC) {
            const long long at = (long long)thr - (int)uniform((u32)S->pub);
            low = at > (long long)rest ? (u32)at : rest + 1u;
          }
          score_list(low);
        }
        if (WIDE && resume) {
          resume = 0;
          if (tid == 0) wv.ctx->pending = 0;
        }
        ++rounds;
        if (MC && picks && !(LISTS && uniform(S->no_list))) {
          // The winner is the best entry of the list if that clears every bound of what is not on the
          // list: then one wavefront takes it from there, and the next ones with it, while the others
          // bring the group bounds up to date, and no arg-max over the threads is needed (2.5 us a
          // pass: two stages of wavefront reductions over 128-bit values with a barrier between them).
          const u32 f2 = wave_max(floor2);
          if (lane == 0 && f2) atomicMax(&S->F2, f2);
          __syncthreads();
          if (wave == LW - 1) {
            const u32 nl_ = uniform(S->nlist), n = nl_ < lcap ? nl_ : lcap, f2_ = uniform(S->F2);
            const u32 F = rest > f2_ ? rest : f2_;
            Floor fl;
            const u32 slot = choose(n, F, fl);
            const Entry e = load_entry(slot);
            u32 allowed = uniform(S->pick_max);             // passes of Algorithm 1 this round may stand for
            if (max_iter && max_iter - uniform(S->n_iter) + 1 < allowed) allowed = (u32)(max_iter - uniform(S->n_iter) + 1);   // (n_iter counts this pass already)
            const u32 m = pick(e, slot, fl, F, allowed, true, 0u);
            if (lane == 0) { S->Fkeep = F; S->fast = m ? 1u : 0u; S->left = fl; }
          } else {
            group_bounds(wave);
          }
          __syncthreads();
          if (uniform(S->fast)) {
            if (LISTS && tid < nch) {                        // is the first one's area its band? (step 2 asks the same for the others)
              const u32 pk = S->pick[0], slot = pk & 0xffffu;
              const uint4 A = list_at(LE_A, slot), B = list_at(LE_B, slot);
              const bool host = (pk >> 16) & 1u;
              u32 len = 0;
              const u64 mo = minOver[tid];
              if (cover(tid, CH, K, host ? B.x : A.z, host ? B.y : A.w, len) && mo != NONE64 && mo - cap < (((u64)B.w << 32) | B.z)) S->no_list = 1;
            }
            if (LISTS) __syncthreads();
            if (!LISTS || !uniform(S->no_list)) { rest_final = rest; break; }
            if (tid == 0) S->fast = 0;                       // (the best by bound is settled slot by slot; read again behind two barriers)
          }
        }
        reduce_best();
        if (WIDE && from_wide) {                  // the rest of the best one
          const u32 i = S->mem[0].slot;
          const bool any = (S->mem[0].hi | S->mem[0].lo) != 0;
          if (wave == 0 && any && lane < sizeof(Winner) / 4) ((u32*)&S->mem[0])[lane] = ((const u32*)&wv.win[i])[lane];
          __syncthreads();
          // (the threads hold rankings without the rest: a further round of the pass goes on from the whole one, which
          // beats the others)
          mine.hi = 0; mine.lo = 0; mine.cost = 1; mine.cand = NONE32;
          if (any && tid == LB - 1) mine = S->mem[0];
        }
        const u32 kb = key_dn_of<RATIO>(S->mem[0].hi, S->mem[0].lo, S->mem[0].cost);
        const u32 need = kb ? kb : 1u;
        u32 out = rest;
        if (WIDE && from_wide) {
          // what the scoring kernel took from the memo lies under the threshold; where the best found does too, the
          // round's tiles are taken again with a lower one
          const u32 sk = uniform(S->F2);
          if (sk > out) out = sk;
          if (sk >= need) for (u32 i = tid; i < ns; i += LB) smark[i] = 0;
        }
        if (out < need) decided = true;                  // every tile left out is below the best found
        else {
          // a tile left out may hold an equal or better one; with nothing found yet, step down a few percent
          thr = kb ? kb : (out > (1u << 19) ? out - (1u << 19) : 1u);
          if (tid == 0) S->second += 1;
          __syncthreads();
          continue;
        }
      }
      rest_final = rest;
      if (!CLIP || settle()) break;
      again = true;
    }
    if (WIDE && wide_exit) break;

    const bool none = !(MC && uniform(S->fast)) && (S->mem[0].hi | S->mem[0].lo) == 0;
    if (none) { __syncthreads(); if (tid == 0) { S->done = 1; S->status = G10_RESIDUAL; } break; }

    // ---- decide and commit -------------------------------------------------------------------
    // More migrations of the same pass (MC): the ranking also tells which candidate comes second,
    // third, ...  Candidate w_j wins the pass after w_1 .. w_(j-1) were committed if its score is the
    // best of the list as those leave it, and clears the bound F of every candidate not on the list
    // (tiles left out, candidates under the list's threshold, its overflow: bounds only fall).  What a
    // commit changes in a score: the free time of transfer windows that meet its own on the same channel,
    // and with it whether the destination can carry the candidate - the picking wavefront follows that
    // exactly, in registers (pick); and the over-capacity time of absent windows in which a slot drops under
    // the capacity - a pick whose absent window touches a chunk where the picks before it may let one
    // drop waits for the list to be scored again (step 2).
    //
    // Step 1 (the last wavefront, a list entry per lane): the entries in the order of their benefit.  Where a
    // round of commits ends with entries that might clear the floor, the steps are taken again from here
    // (cround > 0) instead of from a new ranking: with picks made beside the round's jobs (NX_PICKED), or
    // from the list scored again.  (A further round's picking took 4 to 5 us for two or three migrations while it
    // stopped at the first window that met another; now 5 to 9 for eight to twelve, half of them beside the jobs.)
    bool opened = false;                                 // the next pass's state is made
    bool owed = true;                                    // no migration or refused candidate stands for the pass yet (kept by TIGHT; the other forms commit in a pass's first round)
    PrefixView pv; pv.px = tl.px; pv.base = base; pv.K = K; pv.nch = nch; pv.shift_ch = tl.shift_ch;
    for (u32 cround = 0;; ++cround) {
    const u32 tid = thread_here(), lane = tid & 63u;
    if (MC && cround && uniform(S->next) == NX_RESCORE) {
      // Another round from the same list: its entries are scored again against the timelines as
      // the earlier rounds left them (a committed candidate has no window any more and scores
      // nothing), and the best of them wins the next pass of Algorithm 1 if its key clears the
      // floor - every candidate not on the list is still bounded by it, since bounds only fall.
      const u32 nl_ = uniform(S->nlist), n = nl_ < lcap ? nl_ : lcap;
      rescore_list(n);
      __syncthreads();
      if (wave == LW - 1) {
        u32 allowed = uniform(S->pick_max);              // passes of Algorithm 1 this round may stand for
        const u32 F = uniform(S->Fkeep);
        if (max_iter) { const u32 left = (u32)umin64(max_iter - uniform(S->n_iter) + (TIGHT && owed ? 1u : 0u), NONE32); allowed = left < allowed ? left : allowed; }
        Floor fl;
        const u32 slot = choose(n, F, fl);
        const Entry e = load_entry(slot);
        const u32 m = pick(e, slot, fl, F, allowed, true, cround & 1u);
        if (lane == 0) S->left = fl;
        if (m == 0u) open_pass(TIGHT && owed);           // (nothing on the list clears the floor, or the bounds left out: the pass is over)
      }
      __syncthreads();
    } else if (MC && !cround && !uniform(S->fast)) {     // the winner of the arg-max alone; the list goes on in the next round
      if (tid == 0) {
        // (by_floor stays where nothing on the list cleared this very floor: scoring the list again would find nothing.
        // Where more candidates have one benefit than the list holds, that is every other pass.)
        const u32 f2_ = S->F2, F = rest_final > f2_ ? rest_final : f2_;
        S->m0 = 1; S->by_floor = S->by_floor && S->Fkeep == F ? 1u : 0u; S->Fkeep = F;
        S->chain[0][0] = 0; S->chain[0][1] = 0; S->chain[0][2] = 0; S->chain[0][3] = 0;
      }
      __syncthreads();
    }

    // Step 2, chunk by chunk: what every picked migration does to the chunk (sets of migrations, a
    // bit each), the jobs that follow - for a chunk that is cut, that holds a transfer window, or
    // in which a slot drops under the capacity - and how many migrations can go together: the first
    // whose absent window touches a chunk where the earlier ones may have let a slot drop, or that host
    // memory might not hold on top of the earlier ones, ends the set (the jobs leave it out).  (No branches in
    // the loop but the ones on the destination and the iteration: skipping what touches none of a wavefront's
    // chunks, or ending at the first that waits, cost up to 5 % of the loop.)  For the winner itself the two tests only decide how it is committed: alone, and with
    // the exact host-capacity test.
    const u32 m0 = uniform(S->m0);
    if (MC && m0 == 0u) { opened = true; break; }        // (a later round found nothing above the floor)
    u32 cutP = 0, allP = 0, cutH = 0, allH = 0, eF = 0, eH = 0, wF = 0, wH = 0;   // absent window / period cuts, covers the chunk whole;
                                                         // eviction and prefetch windows meet it, to flash and to host
    u64 runP = 0, runH = 0, lzH = 0;                     // sizes of allP and cutP, of allH and cutH, of allH
    bool jobP = false;
    const bool picked = MC && (cround || uniform(S->fast));     // the round's migrations are entries of the list
    if (MC && picked && wave == LW - 1) {                // ... and in full in mem[] for what follows
      u32 d = 0, to = NONE32;                            // where it goes: 0, 1, or 3, refused
      if (lane < m0) {
        const u32 pk = S->pick[lane], slot = pk & 0xffffu;
        d = (pk >> 16) & 1u; to = TIGHT && d ? (pk >> 16) & 3u : d;
        const uint4 A = list_at(LE_A, slot), B = list_at(LE_B, slot), I = list_at(LE_I, slot);
        const u64 s = ((u64)B.w << 32) | B.z, ot = list_ot(slot, d);
        // (free times behind the earlier picks only where the jobs follow those: run_jobs)
        const double fo = S->chain[cround & 1u][d] ? S->pick_o[lane] : list_f(d ? LE_O1 : LE_O0, slot).x;
        const double fi = S->chain[cround & 1u][2u + d] ? S->pick_i[lane] : list_f(d ? LE_I1 : LE_I0, slot).y;
        Winner& M = S->mem[lane];
        M.hi = __umul64hi(s, ot); M.lo = s * ot; M.s = s; M.fo_base = (u64)(long long)fo; M.fi_end = (u64)(long long)fi;
        M.cand = I.x; M.tensor = I.y; M.pos = I.z; M.dest = to; M.L1 = A.x; M.R = A.y; M.a = d ? B.x : A.z; M.b = d ? B.y : A.w; M.slot = slot;
      }
      const u64 hosts = __ballot(to == G10_HOST), flash = __ballot(to == G10_FLASH);
      if (lane == 0) { S->dests[G10_FLASH] = (u32)flash; S->dests[G10_HOST] = (u32)hosts; }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    if (wave == LW - 1 && (lane & 31u) < m0) {           // transfer times (needed by the jobs and the records): out in lane i, in in lane 32 + i
      Winner& M = S->mem[lane & 31u];
      const bool out = lane < 32u;
      const u64 tau = ceil_div_x1000(M.s, out ? (M.dest ? bwo1 : bwo0) : (M.dest ? bwi1 : bwi0), out ? (M.dest ? ivo1 : ivo0) : (M.dest ? ivi1 : ivi0));
      if (out) M.tau_o = tau;
      else M.tau_i = tau;
    }
    if (tid == 0) { S->jnext = LW - 1; S->touched = 0; S->ot_changed = 0; }
    const bool rows = ROWS && picked && m0 >= ROW_PICKS;
    uint4* const bits = (uint4*)S->wave_win;             // (free between two rankings) per chunk: allP | cutP << 16, eF | wF << 16, allH | cutH << 16, eH | wH << 16
    if (rows && wave < LW - 1) {
      // Few chunks: a row of 16 lanes per chunk, a migration per lane, over all wavefronts but the one that writes the picks out.
      // (A chunk per lane takes one wavefront 0.2 us a migration.)
      const u32 i = lane & 15u, r = lane >> 4;
      u32 gL = 0, gR = 0, ga = 1, gb = 0, gd = 0;
      u64 ms = 0;
      if (i < m0) {
        const u32 pk = S->pick[i], slot = pk & 0xffffu;
        const uint4 A = list_at(LE_A, slot), B = list_at(LE_B, slot);
        const u32 d = (pk >> 16) & 1u;
        gd = TIGHT && d ? (pk >> 16) & 3u : d;
        gL = A.x; gR = A.y; ga = d ? B.x : A.z; gb = d ? B.y : A.w; ms = ((u64)B.w << 32) | B.z;
      }
      const bool real = i < m0, host = real && gd == G10_HOST, flash = real && gd == G10_FLASH;     // (neither: refused, it changes nothing)
      const bool wrap = any(gR > K), hosts = any(host);
      u32 cut = MAXM;
      if (wave * 4u < nch) {
        const u32 c = wave * 4u + r;
        const bool in = c < nch;
        const u64 mo = in ? minOver[c] : NONE64, hm = in && hosts ? hmax[c] : 0ull;
        const bool stale = in && (hpend[c] & 2u) != 0u;
        const u32 c0 = in ? c * CH : 0u, c1 = in ? (c0 + CH < K ? c0 + CH : K) : 0u, len = c1 - c0;
        const u64 spare = stale ? 0ull : mo == NONE64 ? NONE64 : mo - cap;
        int nE = (int)((c1 < ga ? c1 : ga) - (c0 > gL ? c0 : gL)), nA = (int)((c1 < gb + 1 ? c1 : gb + 1) - (c0 > ga ? c0 : ga)),
            nW = (int)((c1 < gR ? c1 : gR) - (c0 > gb + 1 ? c0 : gb + 1));
        bool fP = gL <= c0 && c1 <= gR;
        if (wrap && gR > K) {                            // (ends in the second iteration)
          const u32 nP = covered(c0, c1, K, gL, gR);
          nE = (int)covered(c0, c1, K, gL, ga); nA = (int)covered(c0, c1, K, ga, gb + 1); nW = (int)nP - nE - nA;
          fP = nP != 0 && nP == len;
        }
        const bool tA = real && in && nA > 0, does = host || flash;
        const u64 sA = tA && does ? ms : 0ull, runP = row_scan(sA) - sA;
        bool wait = tA && (spare <= runP || (LISTS && spare - runP < ms));
        u64 mAllH = 0, mTH = 0, mEH = 0, mWH = 0;
        if (hosts) {
          const bool tH = host && in && (nE > 0 || nA > 0 || nW > 0);
          const u64 sH = tH ? ms : 0ull, runH = row_scan(sH) - sH, hroom = hm < host_cap ? host_cap - hm : 0ull;
          const bool full = tH && runH + ms > hroom;
          if (any(full && i == 0u) && lane == 0) S->need_exact = 1;
          wait = wait || (full && i != 0u);
          mTH = ballot(tH); mAllH = ballot(tH && fP); mEH = ballot(tH && nE > 0); mWH = ballot(tH && nW > 0);
        }
        const u64 wm = ballot(wait), mA = ballot(tA && does), mAll = ballot(tA && does && nA == (int)len), mE = ballot(flash && in && nE > 0), mW = ballot(flash && in && nW > 0);
        const u32 w16 = (u32)(wm | wm >> 16 | wm >> 32 | wm >> 48) & 0xffffu;
        if (w16 && (u32)__builtin_ctz(w16) < cut) cut = (u32)__builtin_ctz(w16);
        if (i == 0u && in) {
          const u32 sh = r * 16u;
          const u32 a_ = (u32)(mA >> sh) & 0xffffu, all_ = (u32)(mAll >> sh) & 0xffffu, th_ = (u32)(mTH >> sh) & 0xffffu, allh_ = (u32)(mAllH >> sh) & 0xffffu;
          bits[c] = make_uint4(all_ | (a_ & ~all_) << 16, ((u32)(mE >> sh) & 0xffffu) | (u32)(mW >> sh) << 16,
                               allh_ | (th_ & ~allh_) << 16, ((u32)(mEH >> sh) & 0xffffu) | (u32)(mWH >> sh) << 16);
        }
      }
      if (cut < MAXM && lane == 0) atomicMin(&S->cut, cut);
    }
    if (rows) __syncthreads();
    if (tid < ((nch + 63u) & ~63u)) {
      // migration i lies in lane i of every wavefront and is read from there into scalars: with a trip to
      // LDS for every migration this loop took 2.1 us a round on the stress trace
      u32 gL = 0, gR = 0, ga = 1, gb = 0, gd = 0;
      u64 gs = 0;
      if (MC && picked) {
        if (lane < m0) {
          const u32 pk = S->pick[lane], slot = pk & 0xffffu;
          const uint4 A = list_at(LE_A, slot), B = list_at(LE_B, slot);
          const u32 d = (pk >> 16) & 1u;
          gd = TIGHT && d ? (pk >> 16) & 3u : d;
          gL = A.x; gR = A.y; ga = d ? B.x : A.z; gb = d ? B.y : A.w; gs = ((u64)B.w << 32) | B.z;
        }
      } else if (lane < m0) { const Winner& M = S->mem[lane]; gL = M.L1; gR = M.R; ga = M.a; gb = M.b; gd = M.dest; gs = M.s; }
      const bool stale = MC && tid < nch && (hpend[tid] & 2u) != 0u;   // (picked by an over-capacity time that has fallen since)
      const bool in = tid < nch;
      const u64 mo = in ? minOver[tid] : NONE64, hm = in ? hmax[tid] : 0ull;
      const u32 c0 = in ? tid * CH : 0u, c1 = in ? (c0 + CH < K ? c0 + CH : K) : 0u, len = c1 - c0;
      // what the pressure over the capacity can still lose in this chunk (0: nothing may touch a stale one)
      const u64 spare = stale ? 0ull : mo == NONE64 ? NONE64 : mo - cap;
      const u64 hroom = hm < host_cap ? host_cap - hm : 0ull;
      u32 cut = MAXM;                                    // (of this wavefront's chunks: the migrations from there on wait)
      if (rows) {
        const uint4 b = in ? bits[tid] : make_uint4(0u, 0u, 0u, 0u);
        allP = b.x & 0xffffu; cutP = b.x >> 16; eF = b.y & 0xffffu; wF = b.y >> 16;
        allH = b.z & 0xffffu; cutH = b.z >> 16; eH = b.w & 0xffffu; wH = b.w >> 16;
        const u32 tP = allP | cutP, tH = allH | cutH;
        for (u32 i = 0; i < m0; ++i) {
          const u64 ms = read_lane64(gs, i);
          runP += (tP >> i) & 1u ? ms : 0ull;
        }
        if (any(tH != 0u))
          for (u32 i = 0; i < m0; ++i) {
            const u64 ms = read_lane64(gs, i);
            runH += (tH >> i) & 1u ? ms : 0ull;
            lzH += (allH >> i) & 1u ? ms : 0ull;
          }
      } else for (u32 i = 0; i < m0; ++i) {
        const u32 mL1 = (u32)__builtin_amdgcn_readlane((int)gL, (int)i), mR = (u32)__builtin_amdgcn_readlane((int)gR, (int)i);
        const u32 ma = (u32)__builtin_amdgcn_readlane((int)ga, (int)i), mb = (u32)__builtin_amdgcn_readlane((int)gb, (int)i);
        const u32 md = (u32)__builtin_amdgcn_readlane((int)gd, (int)i), bit = 1u << i;
        const u64 ms = read_lane64(gs, i);
        // slots that the chunk shares with the eviction window [L1, a), the absent window [a, b], the prefetch window
        // (b, R) (not above zero: none); does the whole period cover it?
        int nE, nA, nW;
        bool fP;
        if (mR <= K) {
          nE = (int)((c1 < ma ? c1 : ma) - (c0 > mL1 ? c0 : mL1));
          nA = (int)((c1 < mb + 1 ? c1 : mb + 1) - (c0 > ma ? c0 : ma));
          nW = (int)((c1 < mR ? c1 : mR) - (c0 > mb + 1 ? c0 : mb + 1));
          fP = mL1 <= c0 && c1 <= mR;
        } else {                                         // (ends in the second iteration)
          const u32 nP = covered(c0, c1, K, mL1, mR);
          nE = (int)covered(c0, c1, K, mL1, ma); nA = (int)covered(c0, c1, K, ma, mb + 1); nW = (int)nP - nE - nA;
          fP = nP != 0 && nP == len;
        }
        // the earlier ones may have let a slot of its absent window drop (its own pressure falls behind its win)
        bool wait = nA > 0 && spare <= runP;
        if (LISTS && picked) wait = wait || (nA > 0 && spare - runP < ms);
        const u64 sA = nA > 0 ? ms : 0ull;
        if (md == G10_HOST) {
          // host memory may not hold it on top of the earlier ones
          const bool tH = nE > 0 || nA > 0 || nW > 0;
          const bool full = tH && runH + ms > hroom;
          if (i == 0) { if (__any(full)) S->need_exact = 1; }
          else wait = wait || full;
          if (__any(wait) && cut == MAXM) cut = i;
          eH |= nE > 0 ? bit : 0u;
          wH |= nW > 0 ? bit : 0u;
          runH += tH ? ms : 0ull;
          lzH += tH && fP ? ms : 0ull;
          allH |= tH && fP ? bit : 0u;
          cutH |= tH && !fP ? bit : 0u;
        } else {
          if (__any(wait) && cut == MAXM) cut = i;
          if (TIGHT && md != G10_FLASH) continue;                   // (refused: it changes nothing)
          eF |= nE > 0 ? bit : 0u;
          wF |= nW > 0 ? bit : 0u;
        }
        runP += sA;
        cutP |= nA > 0 ? bit : 0u;
        allP |= nA == (int)len ? bit : 0u;               // (len > 0)
      }
      cutP &= ~allP;
      if (cut < MAXM && lane == 0) atomicMin(&S->cut, cut);
      // (a job adds the sizes of the migrations that cover its chunk whole itself)
      jobP = cutP != 0 || (runP != 0 && spare <= runP);
      const u64 b0 = __ballot(jobP), b1 = __ballot(eF != 0), b2 = __ballot(eH != 0), b3 = __ballot(wF != 0), b4 = __ballot(wH != 0);
      const u32 n0 = (u32)__popcll(b0), n1 = n0 + (u32)__popcll(b1), n2 = n1 + (u32)__popcll(b2), n3 = n2 + (u32)__popcll(b3), n4 = n3 + (u32)__popcll(b4);
      if (n4) {
        u32 off = 0;
        if (lane == 0) off = atomicAdd(&S->njobs, n4);
        off = (u32)__builtin_amdgcn_readfirstlane((int)off);
        const u64 lt = (1ull << lane) - 1ull;
        if (jobP) jobs[off + (u32)__popcll(b0 & lt)] = ((u64)allP << 40) | ((u64)cutP << 24) | ((u64)J_P << 16) | tid;
        if (eF) jobs[off + n0 + (u32)__popcll(b1 & lt)] = ((u64)eF << 24) | ((u64)J_FO0 << 16) | tid;
        if (eH) jobs[off + n1 + (u32)__popcll(b2 & lt)] = ((u64)eH << 24) | ((u64)J_FO1 << 16) | tid;
        if (wF) jobs[off + n2 + (u32)__popcll(b3 & lt)] = ((u64)wF << 24) | ((u64)J_FI0 << 16) | tid;
        if (wH) jobs[off + n3 + (u32)__popcll(b4 & lt)] = ((u64)wH << 24) | ((u64)J_FI1 << 16) | tid;
      }
    }
    __syncthreads();
    const u32 nj = uniform(S->njobs), cut_ = uniform(S->cut), need_exact = uniform(S->need_exact);   // (nj: the jobs of the round)
    u32 m = m0 < cut_ ? m0 : cut_;
    bool room = true;
    // (the first one host memory might not hold: looked up for all entries, which are then picked again)
    bool looked_up = false;
    if (TIGHT && picked && need_exact) {
      looked_up = (S->pick[0] & PK_ROOM) && S->probed;
      __syncthreads();                                   // (both may change from here on)
      if (!looked_up) { probe_host(); m = 0; }
    }
    if (LISTS && m == 0u && uniform(S->next) == NX_RESCORE) break;    // (its area may lie under its band: the next ranking pass settles it)
    if (MC && m == 0u) {                                 // (not even the first stands: the list is scored again)
      __syncthreads();
      if (tid == 0) { S->njobs = 0; S->cut = MAXM; S->need_exact = 0; S->next = NX_RESCORE; }
      __syncthreads();
      continue;
    }
    if (MC && !TIGHT && cround && need_exact) break;     // (the exact host-memory test is left to the next ranking pass)
    const bool first = TIGHT ? owed : cround == 0u;
    if (!first) ++used;                                  // (rounds that commit something: a launch's budget is bounded by the candidates)
    if (need_exact && !looked_up) {                   // the winner alone; host memory slot by slot where its period cuts a chunk
      m = 1;
      const u64 s = S->mem[0].s;
      if (tid == 0) S->hq = 0;
      __syncthreads();
      if ((cutH & 1u) || ((allH & 1u) && (hpend[tid] & 1u))) jobs[atomicAdd(&S->njobs, 1u)] = ((u64)J_HQ << 16) | tid;   // (behind the round's jobs)
      else if (allH & 1u) atomicMax((unsigned long long*)&S->hq, (unsigned long long)hmax[tid]);   // (exact: nothing is missing there)
      __syncthreads();
      run_jobs(nj, uniform(S->njobs), 0xffffu, cround & 1u);
      __syncthreads();
      room = s <= host_cap && S->hq <= host_cap - s;
      if (tid == 0) S->jnext = LW - 1;
      __syncthreads();
    }

    // Step 3: the commit.  A chunk a migration covers whole takes a lazy add, unless it has a job
    // that makes it; the jobs; and beside the first of them, in the last wavefront (lane i takes
    // migration i), the plan records, the counters and the next pass's first threshold.
    if (room && tid < nch) {
      const u32 c = tid;
      if (m != m0) {                                     // the migrations left out
        const u32 keep = (1u << m) - 1u;
        allP &= keep; allH &= keep; cutH &= keep;
        runP = 0; lzH = 0; runH = 0;
        for (u32 i = 0; i < m; ++i) {
          const u64 ms = S->mem[i].s;
          if ((allP >> i) & 1u) runP += ms;
          if ((allH >> i) & 1u) { lzH += ms; runH += ms; }
          if ((cutH >> i) & 1u) runH += ms;
        }
      }
      if (!jobP && runP) {                               // (no job: nothing cuts the chunk)
        lazyP[c] += runP;
        const u64 mo = minOver[c];
        if (mo != NONE64) minOver[c] = mo - runP;
      }
      // host occupancy: whole covers into the lazy add; cuts only into the chunk's bound, the slots follow on demand (J_HQ)
      if (runH) { lazyH[c] += lzH; hmax[c] += runH; }
      if (cutH) atomicOr(&hpend[c], 1u);
    }
    if (wave == LW - 1) {
      const u64 nm = S->n_mig, nd = S->n_drop;
      u32 drops = 0, hosts = 0;                            // of the round: candidates refused, migrations to host
      if (lane < m) {
        const Winner& M = S->mem[lane];
        const u32 to = M.dest;
        if (TIGHT) { drops = (u32)__ballot(to > G10_HOST); hosts = (u32)__ballot(to == G10_HOST); }
        u64 at = nm + lane, at_d = nd;
        bool refused = !room;
        if (TIGHT && drops) {
          const u32 before = (u32)__popc(drops & ((1u << lane) - 1u));
          refused = to > G10_HOST; at -= before; at_d += before;
        }
        const u32 mL1 = M.L1, mR = M.R, ma = M.a, mb = M.b;
        const u64 ms = M.s;
        a.cd.A[M.pos] = make_uint4(mL1, mR, 1u, 0u);       // the candidate leaves the live set
        a.cd.B[M.pos] = make_uint4(1u, 0u, (u32)ms, (u32)(ms >> 32));
        if (MC && M.slot != NONE32) {                      // (and has nothing left to win on the list of the pass)
          list_at(LE_A, M.slot) = make_uint4(mL1, mR, 1u, 0u);
          list_at(LE_B, M.slot) = make_uint4(1u, 0u, (u32)ms, (u32)(ms >> 32));
          lkey[M.slot] = 0u; list_ot(M.slot, 0) = NONE64; list_ot(M.slot, 1) = NONE64;
        }
        if (refused) {
          g10_dropped dr; dr.iteration = S->n_iter - (first ? 1u : 0u) + lane; dr.cand = M.cand; dr.reserved = 0;
          a.dropped[at_d] = dr;
        } else {
          g10_migration mg;
          mg.cand = M.cand; mg.tensor = M.tensor;
          mg.evict_after = mL1 - 1; mg.absent_first = ma >= K ? ma - K : ma; mg.absent_last = mb >= K ? mb - K : mb;
          mg.next_use = mR >= K ? mR - K : mR;
          mg.dest = to; mg.wraps = mR >= K ? 1u : 0u;
          mg.size_bytes = ms; mg.t_out_ns = M.tau_o; mg.t_in_ns = M.tau_i; mg.benefit_lo = M.lo; mg.benefit_hi = M.hi;
          a.records[at] = mg;
          a.rec_ab[at] = make_uint2(ma, mb);
          a.rec_h[at] = to == G10_HOST ? make_uint4(mL1, mR, (u32)ms, (u32)(ms >> 32)) : make_uint4(mL1, mR, 0u, 0u);
          atomicOr(&S->touched, (1u << (A_FO + to)) | (1u << (A_FI + to)));
        }
      }
      if (lane == 0) {
        // first threshold of the next pass: a little under the last benefit.  How little adapts:
        // where many candidates are nearly equal (a pass scored thousands) the margin halves; it
        // doubles when a pass ran out of candidates above the floor with little scored
        u32 gs = S->gshift;
        const bool listed = MC && !(LISTS && S->no_list);
        if (!first) {
          // (the margin adapts once per ranking pass)
        } else if (WIDE && a.wide_min) {
          // with the scoring kernel a longer list costs little and a second round a pair of launches:
          // the margin doubles whenever a pass needed one, and narrows only now and then
          if (rounds > 1u) { if (gs > 2u) --gs; }
          else if ((S->n_iter & 31u) == 0u && gs < GUESS_SHIFT) ++gs;
        } else if (pass_units > (listed ? 24u : 8u) && gs < GUESS_SHIFT_MAX) ++gs;
        // (Where a pass commits one migration, lists over 8 units do not pay: 600 passes by the ratio key with equal costs, 130 000
        // candidates, 15.0 ms with 24, 14.1 with 8.)
        else if (listed) { if ((S->by_floor || rounds > 1u) && pass_units <= 18u && gs > MC_GUESS_SHIFT_MIN) --gs; }
        else if (rounds > 1u && pass_units <= 2u && gs > GUESS_SHIFT) --gs;
        S->gshift = gs;
        if (listed && first) {
          const u32 nl_ = S->nlist;
          const int pub = S->pub, mag = pub < 0 ? -pub : pub;
          int x = pub;
          if (nl_ > lcap) x -= mag / 2 > (1 << 18) ? mag / 2 : 1 << 18;
          else if (nl_ > lcap / 16u * 9u) x -= mag / 8 > (1 << 15) ? mag / 8 : 1 << 15;
          else if (nl_ < lcap / 32u * 3u) x += mag / 2 > (1 << 18) ? mag / 2 : 1 << 18;
          else if (nl_ < lcap / 4u) x += mag / 4 > (1 << 16) ? mag / 4 : 1 << 16;
          S->pub = x < PUB_MIN ? PUB_MIN : x > PUB_MAX ? PUB_MAX : x;
        }
        const Winner& Z = S->mem[m - 1];
        u64 ghi = Z.hi, glo = Z.lo;
        const u64 dlo = (glo >> gs) | (ghi << (64 - gs)), dhi = ghi >> gs;
        const u64 nlo = glo - dlo;
        ghi = ghi - dhi - (glo < dlo ? 1ull : 0ull);
        S->thr_key = RATIO ? rkey_dn(ratio_approx(Z.hi, Z.lo, Z.cost) * (1.0 - 1.0 / (double)(1u << gs))) : upkey(ghi, nlo);
        if (!room) {
          S->n_drop = nd + 1; S->more = 0;
          if (TIGHT) S->calm = 0;
          else if (picks && !CLIP && nd + 1 >= TIGHT_FROM && S->alone) S->stop = 1;           // (the form for it goes on)
        }
        else {
          // the passes of Algorithm 1 this round stands for beyond the one the ranking pass counted
          // at its top (a later round: all of its own), each with one live candidate fewer to rank
          const u64 x = first ? m - 1 : m, live = C - nm - nd;
          S->n_mig = nm + m - (u32)__popc(drops); S->n_drop = nd + (u32)__popc(drops); S->n_iter += x;
          S->n_evals += first ? x * live - x * (x + 1) / 2 : x * live - x * (x - 1) / 2;
          if (TIGHT && hosts) S->probed = 0;
          if (TIGHT) {
            const u32 calm = drops ? 0u : S->calm + 1u;
            S->calm = calm;
            if (calm >= TIGHT_CALM && S->tight_at <= nd) {                          // (the other form goes on)
              S->tight_at = nd + 1; S->calm = 0;
              if (S->alone) S->stop = 1;
            }
          }
          // another round of commits from the same list: unless the picking ran out of entries above
          // the floor and every one it picked was committed
          const bool more = MC && S->nlist > 1u && picks && listed && (!S->by_floor || m < m0) && !(max_iter && S->n_iter >= max_iter);
          S->more = more ? 1u : 0u;
          // (where the chunks cut a round short the next one picks little more than went through)
          if (MC) { const u32 pm = S->pick_max; S->pick_max = m < m0 ? (m + 2u < MAXM ? m + 2u : MAXM) : m0 == pm ? (2u * pm < MAXM ? 2u * pm : MAXM) : pm; }
          if (!first) S->more_rounds += 1;
          if (LISTS && picked) S->evals += m;              // (areas shown to be their bands)
        }
      }
    }
    if (TIGHT) owed = false;
    if (!room) { __syncthreads(); break; }
    if (MC && wave == LW - 1) {
      // Beside the jobs the last wavefront picks the next round's migrations: it knows the channels as this round leaves
      // them, and over-capacity times that fall in this round are marked by the jobs (stale), which the next chunk test
      // heeds.  Not where the chunks cut this round short: the channels are then not as the picking left them.
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_s_setprio(3);                     // (the longest chain of the round; two job wavefronts share its SIMD)
      u32 next = NX_RESCORE;
      if (uniform(S->more) && picked && m == m0) {
        u32 allowed = uniform(S->pick_max);
        if (max_iter) { const u32 left = (u32)umin64(max_iter - uniform(S->n_iter), NONE32); allowed = left < allowed ? left : allowed; }
        const Floor fl = S->left;
        const u32 slot = lane < uniform(S->nsel) ? S->sel[lane] : NONE32;
        const Entry e = load_entry(slot);
        const u32 mn = pick(e, slot, fl, uniform(S->Fkeep), allowed, false, (cround + 1u) & 1u);
        if (mn) next = NX_PICKED;
        else if (uniform(S->by_floor)) { if (lane == 0) S->more = 0; }   // (what is left has only fallen: the pass is over)
      }
      if (lane == 0) S->next = next;
      __builtin_amdgcn_s_setprio(0);
    }
    run_jobs(0u, nj, (1u << m) - 1u, cround & 1u);
    __syncthreads();
    // level 1: the bases of the timelines whose chunk totals changed, one wavefront per timeline
    {
      const u32 touched = uniform(S->touched | (S->ot_changed ? 1u : 0u));
      if (wave < N_ARR && ((touched >> wave) & 1u)) {
        const u32 arr = wave;
        if (nch <= G10_WAVE) {                           // (a chunk per lane)
          const u64 v = lane < nch ? tot[(u64)arr * nch + lane] : 0ull;
          const u64 inc = wave_scan_incl(v);
          if (lane < nch) base[(u64)arr * nb1 + lane] = inc - v;
          if (lane == G10_WAVE - 1) base[(u64)arr * nb1 + nch] = inc;
        } else {
        constexpr u32 PER = (NCH_MAX + G10_WAVE - 1) / G10_WAVE;
        u64 v[PER], sum = 0;
#pragma unroll
        for (u32 k = 0; k < PER; ++k) {
          const u32 c = lane * PER + k;
          v[k] = c < nch ? tot[(u64)arr * nch + c] : 0ull;
          sum += v[k];
        }
        const u64 inc = wave_scan_incl(sum);
        u64 run = inc - sum;
#pragma unroll
        for (u32 k = 0; k < PER; ++k) {
          const u32 c = lane * PER + k;
          if (c < nch) base[(u64)arr * nb1 + c] = run;
          run += v[k];
        }
        if (lane == G10_WAVE - 1) base[(u64)arr * nb1 + nch] = inc;
        }
      }
      opened = !MC || !uniform(S->more);
      if (opened) { if (wave == LW - 1) open_pass(false); }
      else if (tid == LB - 1) { S->njobs = 0; S->cut = MAXM; S->need_exact = 0; S->hq = 0; }
      __syncthreads();
    }
    if (opened) break;
    }                                                    // (rounds of commits of one ranking pass)
    if (!opened) {                                       // (a refused candidate, or a test left to the next pass)
      __syncthreads();
      if (wave == LW - 1) open_pass(TIGHT && owed);
      __syncthreads();
    }
  }
  __syncthreads();

  // ---- state out ---------------------------------------------------------------------
  for (u32 i = tid; i < N_ARR * nch; i += LB) a.g_tot[i] = tot[i];
  for (u32 i = tid; i < nch; i += LB) { a.g_lazyP[i] = lazyP[i]; a.g_minOver[i] = minOver[i]; a.g_lazyH[i] = lazyH[i]; a.g_hmax[i] = hmax[i]; a.g_hmat[i] = hmat[i]; a.g_hpend[i] = hpend[i] & 1u; }
  for (u32 i = tid; i < nt; i += LB) a.g_keys[i] = keys[i];
  for (u32 i = tid; i < N_ARR * nb1; i += LB) a.g_base[i] = base[i];
  if (tid == 0) {
    ctl->n_iter = S->n_iter; ctl->n_mig = S->n_mig; ctl->n_drop = S->n_drop; ctl->n_evals = S->n_evals;
    ctl->thr_key = S->thr_key; ctl->status = S->status; ctl->done = S->done;
    ctl->gshift = S->gshift; ctl->pub = S->pub;
    if (CLIP) { ctl->lists = S->lists; ctl->lists_ended = S->lists_ended; }
    if (TIGHT) { ctl->tight_at = S->tight_at; ctl->calm = S->calm; }
    ctl->overtime_after = base[(u64)A_OT * nb1 + nch];
    if (WIDE && a.wide) {
      ctl->units_scored = units0 + S->units; ctl->second_rounds = second0 + S->second; ctl->jobs_run = jobs0 + S->jobs;
      ctl->launches = launches0 + 1; ctl->passes = passes_before + passes;
      return;                                            // (the other counters do not move in this form)
    }
    ctl->units_scored += S->units; ctl->second_rounds += S->second; ctl->jobs_run += S->jobs; ctl->launches += 1;
    ctl->passes += passes;
    ctl->area_evals += S->evals; ctl->area_refused += S->refused;
    ctl->more_rounds += S->more_rounds; ctl->list_rescored += S->list_rescored;
  }
}

// The scoring kernel of WideCtx: workgroup b goes through the units b, b + nwg, ... of the list the loop kernel left (256
// candidates each), scores the candidates whose key may have risen as the loop kernel's own rounds score theirs, raises the
// bounds of the tiles in device memory and leaves its best candidate in win[b], its ranking and the largest key that it did
// not make anew (skipped) in key[b].
// A list is 160 000 to 215 000 candidates on the stress trace, because their bounds hold for either destination while the
// policy keeps nearly all of them on flash; what bounded the kernel were the eight 16-byte gathers of each, from tables
// larger than an L2.  So every candidate's bound and the key of its policy's destination are kept (LoopArgs::memo, with the
// number of migrations there were, per wavefront of candidates).  A key kept can only have fallen since, unless a
// migration to flash took channel time from a flash window of the candidate and it moves to host: where the few migrations
// since meet none of its windows, and the key lies under the round's threshold, the candidate is not scored again and counts
// with the key kept: where the best that was scored does not clear the largest of those, the loop kernel has the round's
// tiles taken again with its key as the threshold, which scores every candidate whose kept key could reach it; each time
// the threshold falls, so the pass comes to its end.  12.6 -> 9.2 us a launch; what is left are the launch, three
// dependent trips and the records.
__device__ __forceinline__ bool may_meet(u64 K, u64 x, u64 y, u64 u, u64 v) {   // [x, y) and [u, v) of the doubled timeline, modulo K
  return (x < v && u < y) || (x + K < v && u < y + K) || (x < v + K && u + K < y);
}
// KEPT: keys are kept (the memo is there).
template <bool KEPT>
__global__ __launch_bounds__(UNIT) void k_wide_score(const LoopArgs* __restrict__ plans) {
  extern __shared__ __align__(16) unsigned char smem[];
  const LoopArgs a = in_global(plans[0]);
  if (!a.wide) return;
  const WideView wv = wide_view(a.wide);
  const u32 nwg = wv.ctx->nwg;
  if (!wv.ctx->pending || blockIdx.x >= nwg) return;
  const Timelines tl = a.tl;
  const u32 nch = tl.nch, K = tl.K;
  const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  Winner* wwin = (Winner*)smem;                         // [UNIT / 64]
  const Ctl* ctl = a.ctl;
  PrefixView pv; pv.px = tl.px; pv.K = K; pv.nch = nch; pv.shift_ch = tl.shift_ch;
  pv.base = a.g_base;                                   // (a few entries per candidate, read where they lie)
  Machine mc; mc.bwo0 = ctl->bw_out[0]; mc.bwo1 = ctl->bw_out[1]; mc.bwi0 = ctl->bw_in[0]; mc.bwi1 = ctl->bw_in[1];
  mc.ivo0 = ctl->inv_out[0]; mc.ivo1 = ctl->inv_out[1]; mc.ivi0 = ctl->inv_in[0]; mc.ivi1 = ctl->inv_in[1];
  Winner mine;
  mine.hi = 0; mine.lo = 0; mine.cost = 1; mine.cand = NONE32; mine.exact = 0; mine.tau_o = 0; mine.tau_i = 0; mine.slot = NONE32;
  mine.s = 0; mine.fo_base = 0; mine.fi_end = 0; mine.tensor = 0; mine.pos = 0; mine.dest = 0; mine.L1 = 0; mine.R = 0; mine.a = 1; mine.b = 0;
  const u32 nunits = wv.ctx->ntl << a.tshift, made = (u32)ctl->n_mig, top = wv.ctx->thr;
  // Keys from a quarter of the threshold on are made again: where the best lies under the threshold, the round is not
  // taken anew for a key that was kept.  (Loops of 500 passes, every key made anew / kept under a quarter of the threshold:
  // the stress trace on its own machine, where 498 migrations go to host and the keys on flash are a quarter of those to
  // host, 17.5 / 15.1 ms, the same with margins of 0.84, 0.7 and a half, and 18.0 with a sixteenth, where nothing is
  // kept.  Where it does not pay nothing is kept: see MEMO_MIN_CANDS.)
  const u32 thr = top > MEMO_MARGIN ? top - MEMO_MARGIN : 1u;
  u32* const stamp = (u32*)(a.memo + a.n_pad);          // 1 + the migrations made when the 64 candidates' memo held (0: it holds nothing)
  uint4 mh[MEMO_SPAN];                                  // the latest migrations: {L, R, size if to host} and {a, b}
  uint2 mw[MEMO_SPAN];
#pragma unroll
  for (u32 j = 0; j < MEMO_SPAN; ++j) {
    const u32 m = made > j ? made - 1u - j : 0u;
    mh[j] = made > j ? a.rec_h[m] : make_uint4(0, 0, 0, 0);
    mw[j] = made > j ? a.rec_ab[m] : make_uint2(0, 0);
  }
  u32 skipped = 0;
  for (u32 u = blockIdx.x; u < nunits; u += nwg) {
    const u32 t = wv.alist[u >> a.tshift];
    const u32 p = (((t << a.tshift) + (u & ((1u << a.tshift) - 1u))) << 8) + tid;
    const uint4 A = a.cd.A[p], B = a.cd.B[p];
    const uint2 id = a.cd.id[p], was = KEPT ? a.memo[p] : make_uint2(0u, 0u);
    const u32 st = KEPT ? uniform(stamp[p >> 6]) : 0u, since = made + 1u - st;
    bool anew = st == 0u || since > MEMO_SPAN || was.y >= thr;
    // (A key that is the bound itself cannot be passed, wherever the candidate goes.  Flash struck since: a round of the
    // loop kernel's own found it full.)
    if (!anew && was.x > was.y) {
      anew = A.z > A.w;
#pragma unroll
      for (u32 j = 0; j < MEMO_SPAN; ++j)
        if (j < since && (mh[j].z | mh[j].w) == 0u)                    // (to flash)
          anew |= may_meet(K, A.x, A.z, mh[j].x, mw[j].x) || may_meet(K, (u64)A.w + 1, A.y, (u64)mw[j].y + 1, mh[j].y);
    }
    if (KEPT && lane == 0 && st != made + 1u) stamp[p >> 6] = made + 1u;
    u32 kb = was.x;                                     // the candidate's bound
    Score r;
    r.ok0 = r.ok1 = false;
    u64 c0 = 1, c1 = 1;
    if (anew) {
      r = score_candidate(pv, mc, A, B);
      if (r.strike0) a.cd.A[p] = make_uint4(A.x, A.y, 1u, 0u);
      if (r.strike1) a.cd.B[p] = make_uint4(1u, 0u, B.z, B.w);
      if (r.ok0 || r.ok1) costs_of(mc, ((u64)B.w << 32) | B.z, c0, c1);
      const u32 k0 = key_up_of<true>(r.h0, r.l0, c0), k1 = key_up_of<true>(r.h1, r.l1, c1);
      kb = k0 > k1 ? k0 : k1;                           // it holds for either destination
      if (KEPT) a.memo[p] = make_uint2(kb, r.ok0 ? k0 : k1);
    } else if (was.y > skipped) skipped = was.y;
    const u32 k = wave_max(kb);
    if (lane == 0 && k) atomicMax(&a.g_keys[t], k);
    const bool ok_any = r.ok0 || r.ok1;                // flash first; host only if flash cannot take it
    const u32 d = r.ok0 ? 0u : 1u;
    const u64 hi = ok_any ? (d ? r.h1 : r.h0) : 0ull, lo = ok_any ? (d ? r.l1 : r.l0) : 0ull, cost = d ? c1 : c0;
    if ((hi | lo) != 0 && better_ratio(hi, lo, cost, id.x, mine.hi, mine.lo, mine.cost, mine.cand)) {
      mine.hi = hi; mine.lo = lo; mine.cost = cost; mine.cand = id.x; mine.tensor = id.y; mine.pos = p; mine.dest = d;
      mine.L1 = A.x; mine.R = A.y; mine.a = d ? B.x : A.z; mine.b = d ? B.y : A.w; mine.s = ((u64)B.w << 32) | B.z;
      mine.fo_base = r.fo_L; mine.fi_end = r.fi_R;
    }
  }
  skipped = wave_max(skipped);
  u32* const wskip = (u32*)(wwin + UNIT / 64);          // [UNIT / 64]
  if (lane == 0) wskip[wave] = skipped;
  const u32 bl = wave_best_lane_ratio(mine.hi, mine.lo, mine.cost, mine.cand);
  if (bl == NONE32) { if (lane == 0) { mine.hi = 0; mine.lo = 0; mine.cost = 1; mine.cand = NONE32; wwin[wave] = mine; } }
  else if (lane == bl) wwin[wave] = mine;
  __syncthreads();
  if (wave == 0) {
    u64 h = 0, l = 0, cs = 1;
    u32 c = NONE32;
    if (lane < UNIT / 64) { h = wwin[lane].hi; l = wwin[lane].lo; cs = wwin[lane].cost; c = wwin[lane].cand; }
    const u32 w = wave_best_lane_ratio(h, l, cs, c);
    const u32 sk = wave_max(lane < UNIT / 64 ? wskip[lane] : 0u);
    if (lane == 0) {
      const Winner& b = wwin[w == NONE32 ? 0u : w];     // (none: any of the four, all empty)
      wv.win[blockIdx.x] = b;
      wv.key[blockIdx.x] = WideKey{b.hi, b.lo, b.cost, b.cand, sk};
      // (No fence and no count of the workgroups that are done: the next launch on the stream sees what this one wrote.  A
      // device-wide fence in each of 840 workgroups writes an L2 back 840 times: 21.3 us a launch with it, 12.6 without.)
      if (blockIdx.x == 0) wv.ctx->scored = 1;
    }
  }
}

}  // namespace

size_t loop_wide_bytes() { return WIDE_BYTES; }

int loop_wide_launch(const LoopArgs* plans, bool kept, hipStream_t s) {
  const size_t lds = (UNIT / 64) * (sizeof(Winner) + sizeof(u32));
  hipLaunchKernelGGL((kept ? k_wide_score<true> : k_wide_score<false>), dim3(WIDE_WG), dim3(UNIT), lds, s, plans);
  G10_HIP(hipGetLastError());
  return G10_OK;
}

// (the least a plan needs: with the shortest list)
size_t loop_lds_bytes(u32 nch, u32 nt) { return lds_before_list(nch, nt) + (size_t)LIST_MIN * LIST_ENTRY; }
size_t loop_lds_taken(u32 nch, u32 nt) { return lds_before_list(nch, nt) + (size_t)list_cap(nch, nt) * LIST_ENTRY; }

// The smallest tile (256 << shift) with at most max_tiles tiles that fit the LDS beside the chunks: 8192 tiles
// and 512 chunks together are 2.4 KB more than a compute unit has (from 498 chunks on the tiles' limit is lower,
// 7899 at 512 chunks), half as many tiles always fit.
u32 loop_tile_shift(u64 n, u32 max_tiles, u32 nch) {
  const u64 units = (n + UNIT - 1) / UNIT;
  u32 sh = 0;
  while (true) {
    const u64 nt = (units + (1ull << sh) - 1) >> sh;
    if (nt <= max_tiles && loop_lds_bytes(nch, (u32)nt) <= LDS_MAX) return sh;
    ++sh;
  }
}

typedef void (*LoopKernel)(const LoopArgs*);
static LoopKernel loop_kernel(u32 rank, u32 area, bool second, bool rows) {
  if (rank == G10_RANK_RATIO) return area == G10_AREA_CLIPPED ? k_loop<true, true, false, false, false> : k_loop<true, false, false, false, false>;
  if (area == G10_AREA_CLIPPED) {
    if (!second) return k_loop<false, true, false, false, false>;
    return rows ? k_loop<false, true, false, true, true> : k_loop<false, true, false, true, false>;
  }
  if (second) return rows ? k_loop<false, false, true, false, true> : k_loop<false, false, true, false, false>;
  return rows ? k_loop<false, false, false, false, true> : k_loop<false, false, false, false, false>;
}

int loop_allow_large_lds() {                     // (once per device: the attribute belongs to the kernel, not to a handle)
  static bool done[64] = {};
  int dev = 0;
  G10_HIP(hipGetDevice(&dev));
  if (dev >= 0 && dev < 64 && done[dev]) return G10_OK;
  for (u32 rank = 0; rank < 2; ++rank)
    for (u32 area = 0; area < 2; ++area)
      for (u32 form = 0; form < (rank == G10_RANK_RATIO ? 1u : 4u); ++form)
        G10_HIP(hipFuncSetAttribute((const void*)loop_kernel(rank, area, (form & 1u) != 0, (form & 2u) != 0), hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_MAX));
  if (dev >= 0 && dev < 64) done[dev] = true;
  return G10_OK;
}

// A plan whose largest tensor is beyond PICK_EXACT commits one migration a pass: it never takes rows, nor refuses several candidates a round.
bool loop_picks(u64 smax) { return smax < PICK_EXACT / 1000; }
bool loop_rows(u32 nch, u64 smax) { return nch <= ROW_CHUNKS && loop_picks(smax); }

int loop_launch(const LoopArgs* plans, u32 n_plans, size_t lds, u32 rank, u32 area, bool second, bool rows, hipStream_t s) {
  hipLaunchKernelGGL(loop_kernel(rank, area, second, rows), dim3(n_plans), dim3(loop_threads(rank == G10_RANK_RATIO, area == G10_AREA_CLIPPED)), lds, s, plans);
  G10_HIP(hipGetLastError());
  return G10_OK;
}
