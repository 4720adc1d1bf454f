// The append, the correction test, the scan and the selection as launches of their own, and the host-side rules that size these
// launches, the step kernel's (fkv_step_dev.h) and the one-launch layer kernel's (fkv_layer_dev.h).
// The roles themselves are in fkv_step_dev.h, attention in fkv_attn_dev.h.
#include "fkv_step_dev.h"
#include "fkv_attn_dev.h"

#pragma clang fp contract(off)

namespace fkv {

// The append and the correction test as calls of their own (fkv_kv_append, fkv_corr_check).  Both are one trip to memory and
// little else, so what counts is what a launch brings along: no more waves than there is work for, and arguments that fit the
// registers the hardware preloads (8 heads, 2.7 us each as roles of the step kernel, whose arguments are fetched first; a kernel
// that does nothing takes 1.6).
template <int DT>
__global__ __launch_bounds__(D) void append_kernel(uint16_t* pool, uint16_t* summ, const uint16_t* k_new, const uint16_t* v_new, int L, int max_pages,
                                                   int units_per_head, int placement, int ring_base, int n_ring) {
  StepArgs a{};
  a.pd = PoolDesc{pool, units_per_head, placement, ring_base, n_ring, 0};
  a.summ = summ; a.k_new = k_new; a.v_new = v_new; a.max_pages = max_pages; a.g.L = L;
  append_role<DT>(a, blockIdx.x);
}
template <int DT, int G>
__global__ __launch_bounds__(G * 64) void corr_kernel(const uint16_t* q, const uint16_t* q_prev, uint16_t* q_stage, uint8_t* flags, uint8_t* flags_user,
                                                      double* cosine, float tau, int have_prev_and_pool) {
  StepArgs a{};
  a.q = q; a.q_prev = q_prev; a.q_stage = q_stage; a.flags = flags; a.flags_user = flags_user; a.cosine = cosine; a.tau = tau;
  a.have_prev = have_prev_and_pool & 1; a.corr_pool = have_prev_and_pool >> 1;
  corr_role<DT, G, G>(a, blockIdx.x);
}

// The two halves of the bandwidth-bound regime.  The scan: append, correction test and page weights, in 256-thread
// blocks of one 64-page chunk each; measured on the scan alone (256 heads x 992 pages, 130 MB; a plain read of the same
// bytes takes 22.1 us = 5.9 TB/s on this machine): 23.9 us in this shape against 25.7 us with 512-thread blocks of 128
// pages -- the smaller block leaves the unit's slots in finer pieces, so that more blocks are in different phases
// (loading, computing, draining) at any time; blocks that take several chunks, pipelined or not, are slower than either.
// A head's chunks are adjacent in block order (blocks that run together read one stretch of memory: 28.2 us with the KV
// cache between two scans of that size, 30.0 us with the heads next to each other): grid (chunks, rows), row by row first
// the other two roles, then a head each; beyond kGridRows rows (a grid dimension ends at 65535) folded into a third dimension.
constexpr int kGridRows = 1 << 15;
template <int DT, int G, bool PAST>
__global__ __launch_bounds__(SCAN_WAVES * 64) __attribute__((amdgpu_waves_per_eu(G <= 4 ? 7 : 5))) void scan_kernel(StepArgs a) {
  touch_args<sizeof(StepArgs)>();
  const int y = (int)(blockIdx.z * kGridRows + blockIdx.y);
  if (y >= a.other_rows + a.heads) return;
  if (y < a.other_rows) {
    int i = y * a.chunks + blockIdx.x;
    if (a.roles & ROLE_APPEND) {
      if (i < a.heads) { append_role<DT>(a, i); return; }
      i -= a.heads;
    }
    if ((a.roles & ROLE_CORR) && i < a.heads) corr_role<DT, G, SCAN_WAVES>(a, i);
    return;
  }
  score_role<DT, G, false, SCAN_WAVES, PAST>(a, y - a.other_rows, blockIdx.x);
}
// The selection after it: one block per slice of a head's candidates, dealt to the heads (deal_block).
template <int G, bool MEAN, bool HOME>
__global__ __launch_bounds__(SEL_THREADS) void select_kernel(StepArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint32_t dyn_lds[];
  touch_args<sizeof(StepArgs)>();
  a.home = HOME;
  if (MEAN) a.sel_pool = 0;
  int head, s;
  deal_block(blockIdx.x, a.slices, a.home, [&](uint32_t j) { return j >> a.slices_log2; }, head, s);
  if (head >= a.heads) return;
  int nw;
  Selected got;
  const auto again = [] {
    StepArgs b = args_from_memory<StepArgs>();
    b.home = HOME;
    if (MEAN) b.sel_pool = 0;
    return b;
  };
  if (select_begin<G, false, MEAN>(a, head, s, dyn_lds, nw, got, again)) select_finish<0, G, false>(a, head, s, dyn_lds, nw, got, again);
}

constexpr size_t kLdsPerUnit = 150 * 1024;   // of the 160 KiB of a compute unit
constexpr int kLayerResident = 2 * kComputeUnits;   // blocks of the layer kernel that the GPU holds at once (by its registers)

// experiment builds only (see knob())
static const int g_min_passes = knob("FKV_LAYER_PASSES", 0);      // passes a scoring block makes
static const int g_one_launch = knob("FKV_ONE_LAUNCH", -1);       // layer-step: 0 separate launches, 1 one launch whenever it can be

static const int g_fuse = knob("FKV_FUSE", -1);

// Selecting blocks of a head, a power of two.  One as long as it has the registers and not too much work: a shared list costs about
// 1.5 us for its exchanges (sums, then keys).  The work of a block that has the list alone is its rows of candidates per thread (one, two,
// four or eight, by the code that there is) times the query heads, and what sharing saves grows with it.  Layer-steps in us, alone and shared:
// - up to kFewShared heads, the method's pooling, KV in HBM: alone up to kLightWork rows times G.  At 12 and 16: 8 heads x 2000 candidates,
//   G = 3, 8.8 and 8.9; 8 x 992, G = 8, 9.5 and 9.9; 8 x 1515, G = 4, 8.6 and 8.6.  At 20, 24 and 32: 8 x 1200, G = 5, 9.5 and 9.0; 8 x 1200,
//   G = 6, 10.2 and 9.4; 6 x 1800, G = 5, 10.0 and 9.2; 8 x 1040, G = 8, 11.8 and 10.2; 1 x 1100, G = 8, 11.4 and 9.9.  The line is on the safe
//   side: 8 x 1700, G = 4, 9.2 and 8.7, and 8 x 2300, G = 2, 10.0 and 8.7, would gain, 1 x 1700, G = 4, 8.5 and 8.9, would not.
// - otherwise alone up to kMaxAloneWork weights.  With more heads it depends on what else the launch has to do: 16 x 2500, G = 3, 14.8
//   and 13.4, 24 x 1500, G = 5, 15.8 and 14.7, but 16 x 1100, G = 5, most corrected, 15.8 and 16.1, 32 x 2100, G = 3, 18.8 and 20.2, and in two
//   blocks a head 48 x 1300, G = 6, 20.1 and 20.2.  With the KV in a host pool the link decides (8 x 1100, G = 8, 23.7 and 23.4).  The other
//   poolings were not looked at again.
// A list that is shared is cut fine, since every phase but the exchanges gets shorter, as long as the blocks that wait for each other stay a
// small part of the launch: 8 heads, G = 4, in 4, 8, 16 blocks: 2300 candidates 10.6, 9.6, 10.1; 4000: 13.1, 12.0, 11.7; 8160: 17.8, 15.9,
// 15.2; 2016, G = 8, 12.5, 12.0, 13.3; but 16 heads x 1200, G = 6, 11.9, 12.0, 12.0, and 2 x 4000, G = 4, in 8 and 16, 10.6 and 11.4.
constexpr int kLightWork = 16, kFewShared = 8, kMaxAloneWork = 9400, kFineSlice = 320, kMaxFineBlocks = 128, kLongList = 1024, kFewHeads = 40, kFewSlices = 4;
static int selection_slices(const Dims& d, const Geom& g, bool host_pool) {
  const int n = g.n_cand, G = d.G, heads = d.batch * d.n_kv, regs = sel_regs_alone(G);
  int rows = 1;
  while (rows * SEL_THREADS < n) rows *= 2;
  const bool light = d.sel_pool == 0 && !host_pool && heads <= kFewShared ? rows * G <= kLightWork : (long)n * G <= kMaxAloneWork;
  if (g.k_eff == 0 || (rows <= regs && light)) return 1;
  int s = 2;
  while (s < MAX_SLICES && ((n + s - 1) / s > SEL_REGS * SEL_THREADS || ((n + s - 1) / s > kFineSlice && heads * s * 2 <= kMaxFineBlocks))) s *= 2;
  return s;
}

static const int g_home = knob("FKV_HOME", -1);                   // 0 never, 1 always

// A word that stays in the L2 it was written to is seen after 0.22 us, through memory after 0.3 to 0.5, and a block reads its
// head's 30 KB of weights from the L2 at several times the rate; an exchange of a layer-step takes 0.3 to 0.8 us less.  Where the heads do not
// go round evenly some XCDs have more to read than if everything were spread, at about 1 MB a us.  So what decides is that excess over an
// even share: kHomeExcess bytes, with fewer than 8 heads, where an XCD has one and others none, kFewHeadsRoom times that; for attention by
// itself, which has one exchange to gain by, kHomeExcessAttn.  Layer-steps in us (G = 4; few heads corrected; most), a head's blocks adjacent
// and on one XCD, with the excess in MB:
// - none: 8 heads x 992 candidates 9.1 and 8.3; 16 x 992 10.7 and 9.5; 64 x 992 25.6 and 23.8, 31.0 and 28.5; 8 x 2016, G = 8, 15.4 and 12.7;
// - up to 0.9: 28 x 992 x 33 pages, 0.5, 12.0 and 11.1, 17.1 and 15.4; 12 x 992 x 65, 0.8, 9.9 and 9.3, 15.1 and 13.7; 76 x 480 x 65, 0.7, 26.1
//   and 24.5, 30.7 and 28.9; but 12 x 100 x 129, 0.92, 9.5 and 10.8, 12.1 and 12.7; 9 x 992 x 129, 2.3, 10.2 and 12.2, 16.5 and 16.1;
// - few heads, up to 2.0: 1 x 992 x 65, 1.4, 8.3 and 7.9, 12.9 and 11.7; 4 x 992 x 129, 1.3, 8.9 and 9.0, 14.3 and 13.4; but 1 x 992 x 193, 3.2,
//   9.0 and 9.8, 15.4 and 14.9;
// - attention by itself, up to 0.45 (few heads 1.0): 12 x 33 pages, 0.3, 5.8 and 5.4; 1 x 65, 0.9, 5.9 and 5.6; but 12 x 65, 0.5, 7.2 and 7.3;
//   12 x 129, 1.1, 9.1 and 10.6; 4 x 129, 1.1, 8.2 and 8.5.
// With up to two heads to an XCD the launch also has to be there all at once (14 heads x 480 x 129, 0.6 MB, 11.3 and 12.3); with more it
// runs in rounds either way.
constexpr double kHomeExcess = 0.9e6, kHomeExcessAttn = 0.45e6, kFewHeadsRoom = 2.2;
constexpr int kSlotsOfXcd = 2 * kComputeUnits / kXcds;            // blocks of 512 threads that an XCD holds at once
static bool little_excess(const Dims& d, int heads, double bytes, bool attn_only) {
  const double excess = (by_xcd(heads) - heads) / (double)kXcds * bytes;
  return d.same_xcd && excess <= (attn_only ? kHomeExcessAttn : kHomeExcess) * (heads < kXcds ? kFewHeadsRoom : 1.0);
}
bool heads_at_home(const Dims& d, int heads, int rows, double bytes, bool attn_only) {
  if (g_home >= 0) return g_home == 1;
  const int most = by_xcd(heads) / kXcds;
  if (heads % kXcds != 0 && most <= 2 && most * rows > kSlotsOfXcd) return false;
  return little_excess(d, heads, bytes, attn_only);
}

// Which XCD a block runs on is the dispatcher's choice, not the programming model's, so it is looked at once for every context
// (here) and no result depends on it: where it is not so, words go through memory, and a word that a reader does not see is a
// wait that runs out.
__global__ void where_kernel(uint32_t* where) {
  uint32_t xcd;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcd));
  if (threadIdx.x == 0) where[blockIdx.x] = xcd;
}
bool blocks_by_xcd(uint32_t* where) {
  uint32_t at[kWhereBlocks];
  hipError_t e = hipMemset(where, 0xff, sizeof(at));               // (no XCD's number: what stays so was not written)
  void* args[] = {&where};
  // (the launch's own error: hipGetLastError would also say, and take away, what a call of the program's left behind)
  if (e == hipSuccess) e = hipLaunchKernel(reinterpret_cast<const void*>(&where_kernel), dim3(kWhereBlocks), dim3(64), args, 0, nullptr);
  if (e == hipSuccess) e = hipMemcpy(at, where, sizeof(at), hipMemcpyDeviceToHost);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  for (int i = 0; i < kWhereBlocks; ++i)
    if (at[i] == 0xffffffffu || at[i] != at[i % kXcds]) return false;
  return true;
}

// Passes of a scoring block: a launch runs in ceil(blocks / resident blocks) rounds, and blocks of a later round (the
// selection and attention come last) queue behind the scoring blocks.  The passes that give the fewest rounds -- one, the
// whole launch resident at once, where the shape allows -- and among those the fewest (most blocks).  Where four to seven heads are to be at
// home and share their lists, it is an XCD's slots that count: there the launch has to be resident all at once (heads_at_home), and with a
// shared list's exchanges that gains more than a pass more costs.  Layer-steps in us, one pass a block and away, two or four and at home: 4 heads
// x 2000 candidates, G = 7, 11.2 and 10.7; 6 x 1800, G = 5, 10.9 and 9.2; 6 x 3000, G = 4, 12.8 and 10.8; 4 x 4000 12.5 and 11.4; but 4 x 2000,
// G = 4, not shared, 9.2 and 9.3; 2 x 4000, which have too much to read for one XCD each, 11.3 and 12.5.
// home: the heads would be, and the link to a host pool does not decide.
static int scoring_passes(const Dims& d, const Geom& g, int slices, int other_rows, int resident, bool home) {
  if (g_min_passes > 0) return g_min_passes;
  const long heads = (long)d.batch * d.n_kv;
  auto blocks_of = [&](long wide, int passes) { return wide * (2 + (g.n_cand + PAGES_PER_PASS * passes - 1) / (PAGES_PER_PASS * passes) + slices + other_rows); };
  if (home && slices > 1 && heads >= kXcds / 2 && heads < kXcds) {
    for (int passes = 1; passes <= SCORE_PASSES; passes *= 2)
      if (blocks_of(by_xcd((int)heads), passes) <= resident) return passes;
  }
  int best = 1;
  long best_rounds = 0;
  for (int passes = 1; passes <= SCORE_PASSES; passes *= 2) {
    const long rounds = (blocks_of(heads, passes) + resident - 1) / resident;
    if (passes == 1 || rounds < best_rounds) { best = passes; best_rounds = rounds; }
  }
  return best;
}

static void fill_step_args(const Dims& d, int roles, const StepIO& io, Geom g, int pages_per_pass, int passes, int slices, StepArgs& a, int& rows, size_t& lds) {
  a = StepArgs{};
  a.roles = roles;
  a.heads = d.batch * d.n_kv; a.k = d.k; a.max_pages = d.max_pages;
  a.g = g;
  a.pd = io.pd; a.summ = io.summ; a.k_new = io.k_new; a.v_new = io.v_new;
  a.q = io.q; a.q_prev = io.q_prev; a.q_stage = io.q_stage; a.have_prev = io.have_prev; a.tau = io.tau;
  a.corr_pool = d.corr_pool; a.sel_pool = d.sel_pool;
  a.flags = io.flags; a.flags_user = io.flags_user; a.cosine = io.cosine;
  a.P = io.P; a.score = io.score; a.ids = io.ids; a.ids_user = io.ids_user; a.exch = io.exch; a.keyx = io.keyx; a.keyid = io.keyid; a.cmax = io.cmax;
  a.no = io.no; a.impatient = io.impatient; a.by_itself = &io.status->by_itself; a.tstamp = io.tstamp;
  a.passes = passes;
  a.slices = slices;
  rows = 0;
  lds = 0;
  if (roles & ROLE_APPEND) rows += 1;
  if (roles & ROLE_CORR) rows += 1;
  if (roles & ROLE_SELECT) {
    a.chunks = (g.n_cand + pages_per_pass * passes - 1) / (pages_per_pass * passes);
    while ((1 << a.slices_log2) < a.slices) a.slices_log2 += 1;
    a.slice = (g.n_cand + a.slices - 1) / a.slices;
    rows += a.chunks + a.slices;
    lds = (size_t)select_key_words(g.n_cand) * sizeof(uint32_t);
    if (io.plan_new_slots) {                       // the recall plan's LDS follows the keys
      a.plan_act_ids = io.plan_act_ids; a.plan_act_slots = io.plan_act_slots;
      a.plan_new_slots = io.plan_new_slots; a.plan_miss = io.plan_miss;
      a.plan_lds_off = (int)(lds / sizeof(uint32_t));
      lds += plan_lds_ints(d.k) * sizeof(int32_t);
    }
  }
}

// The roles of one launch run concurrently.  That is safe because the page being appended to
// is not a candidate -- except with an empty window, when the token that fills a page makes
// that very page a candidate in the same step.
static bool append_races_selection(int roles, const Geom& g) {
  return (roles & ROLE_APPEND) && (roles & ROLE_SELECT) && g.r == 0 && g.n_win == 0 && g.n_cand > 0;
}

// Scoring and selection in one launch up to this many pages to score, in units of 32: beyond, the scan is bandwidth-bound
// and its small blocks, which end the moment their weights are on the way, stream faster.  Whole step, one launch for both
// against two: 32 KV heads x 992 pages 25.9 us against 27.4, 248 x 320 117 against 119, 192 x 480 equal, 256 x 992 96 against 88.
constexpr long kFuseMaxChunks = 2560;

template <int DT, int G>
static int launch_step_g(const Dims& d, int roles, const StepIO& io, const Geom& g, hipStream_t st) {
  static constexpr void (*select_kernels[2][2])(StepArgs) = {{&select_kernel<G, true, false>, &select_kernel<G, true, true>},
                                                             {&select_kernel<G, false, false>, &select_kernel<G, false, true>}};
  static size_t granted[2][2] = {{48 * 1024, 48 * 1024}, {48 * 1024, 48 * 1024}};
  StepArgs a;
  int rows;
  size_t lds;
  const int heads = d.batch * d.n_kv;
  if (roles == ROLE_APPEND) {
    append_kernel<DT><<<heads, D, 0, st>>>(io.pd.pool, io.summ, io.k_new, io.v_new, g.L, d.max_pages, io.pd.units_per_head, io.pd.placement, io.pd.ring_base,
                                           io.pd.n_ring);
    return 1;
  }
  if (roles == ROLE_CORR) {
    corr_kernel<DT, G><<<heads, G * 64, 0, st>>>(io.q, io.q_prev, io.q_stage, io.flags, io.flags_user, io.cosine, io.tau,
                                                 (io.have_prev ? 1 : 0) | d.corr_pool << 1);
    return 1;
  }
  if (!(roles & ROLE_SELECT) || (g_fuse >= 0 ? g_fuse == 1 : (long)heads * ((g.n_cand + PAGES_PER_PASS - 1) / PAGES_PER_PASS) <= kFuseMaxChunks)) {
    const int slices = selection_slices(d, g, io.pd.placement != 0);
    fill_step_args(d, roles, io, g, PAGES_PER_PASS, scoring_passes(d, g, slices, 0, kLayerResident, io.pd.placement == 0 && little_excess(d, heads, g.n_cand * kSummaryBytes, false)), slices, a, rows, lds);
    const bool past = (stream_of(d, g) & STREAM_SUMMARIES) != 0;
    a.home = (roles & ROLE_SELECT) != 0 && heads_at_home(d, heads, rows, g.n_cand * kSummaryBytes);
    const bool other = d.sel_pool != 0;
    if (!(other ? (a.home ? launch_step_kernel_pool_home : launch_step_kernel_pool) : a.home ? launch_step_kernel_home : launch_step_kernel)(a, DT, G, past, rows, lds, st)) return -1;
    if (roles & ROLE_SELECT) *io.P_tagged = true;
    return 1;
  }
  fill_step_args(d, roles, io, g, SCAN_WAVES * 4, SCORE_PASSES, selection_slices(d, g, io.pd.placement != 0), a, rows, lds);
  a.P = reinterpret_cast<unsigned long long*>(io.P_plain);
  a.cmax = reinterpret_cast<unsigned long long*>(io.cmax_plain);
  a.home = a.slices > 1 && heads_at_home(d, heads, a.slices, (double)g.n_cand * d.G * sizeof(float));
  const int other = d.sel_pool != 0, home = a.home;
  if (!grant_lds(select_kernels[other][home], lds, granted[other][home])) return -1;
  a.other_rows = (((roles & ROLE_APPEND ? 1 : 0) + (roles & ROLE_CORR ? 1 : 0)) * heads + a.chunks - 1) / a.chunks;
  const int scan_rows = a.other_rows + heads;
  const dim3 scan_grid(a.chunks, scan_rows < kGridRows ? scan_rows : kGridRows, (scan_rows + kGridRows - 1) / kGridRows);
  if (stream_of(d, g) & STREAM_SUMMARIES) scan_kernel<DT, G, true><<<scan_grid, SCAN_WAVES * 64, 0, st>>>(a);
  else                                    scan_kernel<DT, G, false><<<scan_grid, SCAN_WAVES * 64, 0, st>>>(a);
  select_kernels[other][home]<<<(home ? by_xcd(heads) : heads) * a.slices, SEL_THREADS, lds, st>>>(a);
  *io.P_tagged = false;
  return 2;
}

int launch_step(const Dims& d, int roles, const StepIO& io, Geom g, hipStream_t st) {
  if (d.k == 0) roles &= ~ROLE_SELECT;
  if (roles == 0) return 0;
  if (append_races_selection(roles, g)) {      // then the append gets a launch of its own first
    const int n = launch_step(d, ROLE_APPEND, io, g, st);
    const int m = launch_step(d, roles & ~ROLE_APPEND, io, g, st);
    return n < 0 || m < 0 ? -1 : n + m;
  }
  switch (d.G) {
#define FKV_CASE(GG) case GG: return d.dtype == 0 ? launch_step_g<0, GG>(d, roles, io, g, st) : launch_step_g<1, GG>(d, roles, io, g, st);
    FKV_CASE(1) FKV_CASE(2) FKV_CASE(3) FKV_CASE(4) FKV_CASE(5) FKV_CASE(6) FKV_CASE(7) FKV_CASE(8)
#undef FKV_CASE
    default: return -1;
  }
}

// Which layer-steps take one launch: those that latency bounds.  Measured, one launch against separate ones: 32 KV heads of
// 8K / 32K / 128K tokens 11 / 16 / 28 us against 19 / 26 / 37, 128 of 2K / 16K / 32K 18 / 27 / 53 against 25 / 31 / 55, and
// 192 x 65 attended pages 62 against 65.  With 256 KV heads and more, attention by itself has a block for every compute
// unit and its bytes decide (256 heads of 32K tokens: 103 against 92), as they do beyond kLayerMaxAttended pages (128 x 129:
// 64 against 70; 248 x 129: 133 against 117).  With the KV in a host pool the link decides early: 64 heads of 16K tokens
// 241 against 243, 32 of 124K 183 against 183, so the bigger ones take the gather of its own.
constexpr int kLayerMaxHeads = kComputeUnits - 1;
constexpr int kShortStream = 96, kLooseBlocks = 192, kPagesEach = 16, kEnoughToCut = 40, kManyScored = 240, kFewAlone = 176;
constexpr long kLayerMaxAttended = 24576, kLayerMaxBlocks = 2560, kLayerMaxBlocksHost = 1024;

constexpr int kMaxLayersPacked = 1 << 13, kMaxCtxPacked = 1 << 19;
bool launch_layer(const Dims& d, const LayerIO& io, Geom g, hipStream_t st) {
  const int roles = ROLE_APPEND | ROLE_CORR | ROLE_SELECT;
  if (g_one_launch == 0 || d.k == 0 || append_races_selection(roles, g)) return false;
  if (io.layer >= kMaxLayersPacked || g.L > kMaxCtxPacked) return false;
  // KV in a host pool: the selecting blocks make the recall plan, the attention blocks of a corrected head fetch its
  // missing pages themselves; the tagged words have to hold a page id and a slot
  if (io.host_pool && (d.max_pages > TAGGED_MAX_PAGES || 2 * d.k > TAGGED_MAX_SLOTS)) return false;
  const int heads = d.batch * d.n_kv;
  const int n_att = g.n_sink + d.k + g.n_win + (g.r > 0 ? 1 : 0), n_there = n_att - d.k + g.k_eff;
  int slices = selection_slices(d, g, io.host_pool);
  // Attention's blocks, which come last, are fewer where a list is shared, since selecting blocks wait too.  Beside long lists of
  // many heads, a block each, a head is cut half as fine as it could be: with that many scoring blocks the launch runs in rounds, and
  // blocks of a later one queue.  A pass of 8 layer-steps, in full and half: 128 heads x 1234 candidates (2 splits and 1) 395 and
  // 347 us, and 434 and 375 where most heads are corrected; 64 x 1515 (4 and 2) 233 and 215, 288 and 255; 80 x 1234 (3 and 2) 254 and
  // 239, 293 and 271 (in one 256, 292); 48 x 1515 (5 and 3) 190 and 180, 241 and 229; but 40 x 1389 (5 and 3) 201 and 205, 24 x 1389
  // (9 and 5) 160 and 168.
  const bool half = g.n_cand > kLongList && heads > kFewHeads;
  auto most_waiting = [&]() { return slices > 1 ? kMaxWaiting - heads * slices : half ? (kMaxWaiting / heads + 1) / 2 * heads : kMaxWaiting; };
  const double bytes = (double)n_there * UNIT_BYTES + g.n_cand * kSummaryBytes;
  const bool home = !io.host_pool && little_excess(d, heads, bytes, false);
  int pps, n_splits, passes, rows;
  auto size = [&]() {
    passes = scoring_passes(d, g, slices, n_splits, kLayerResident, home);
    rows = 2 + (g.n_cand + PAGES_PER_PASS * passes - 1) / (PAGES_PER_PASS * passes) + slices + n_splits;
  };
  auto cut = [&](int max_blocks) {
    pps = attn_pages_per_block(n_att, heads, io.max_splits, STEP_WAVES, max_blocks);
    n_splits = (n_att + pps - 1) / pps;
    size();
  };
  cut(most_waiting());
  // One to three heads whose blocks just miss being on their XCD all at once share the list among half as many: 3 heads x 1500
  // candidates, G = 5, away in eight and at home in four, 10.6 and 9.3 us, 15.0 and 12.4 where most are corrected (one block a head,
  // at home, 10.4 and 13.9); 2 x 1500, G = 8, 11.3 and 10.8, 15.7 and 14.0.
  if (home && heads < kXcds / 2 && slices > kFewSlices && rows > kSlotsOfXcd && rows - slices / 2 <= kSlotsOfXcd) {
    slices /= 2;
    cut(most_waiting());
  }
  // As many blocks as fit, two to a compute unit, where the heads are many and the launch runs in rounds: with fewer, the dispatcher
  // puts two on some units and none on others, according to which scoring blocks have just ended, and those of a launch that is
  // bound by its bytes take that much longer.  G = 4, 65 pages, a block a unit and as many as fit (few corrected; most): 80 heads x 480 candidates
  // 27.1 and 25.0 us, 32.1 and 29.5; 96 x 100 31.0 and 23.7, 36.1 and 28.6; 112 x 480 37.1 and 31.0, 42.1 and 37.9; 128 x 992 47.6 and 42.2, 54.0
  // and 50.8; 240 x 480 (G = 7) 82.7 and 69.7, 82.4 and 69.2.  A launch that is there all at once has nothing to gain by it and gets a second round:
  // 36 heads x 480 candidates x 129 pages, 504 blocks, 18.4 and, in 936, 23.2, 25.3 and 28.0; 68 x 100 x 65, 476, 17.9 and 21.9; 60 x 100 x 129, 480, 23.5
  // and 26.4, 28.9 and 33.4.  (Which of it is faster is not a matter of rounds alone: 104 x 480 x 65 29.7 and 29.6, 33.2 and 35.8, between 96 heads, 32.0
  // and 28.8, and 112.)  Long streams of pages do better in few blocks as long as each has a unit of its own (129
  // pages: 96 heads, 192 blocks and 480, 42.3 and 47.5, most corrected), but not where that is just missed (112 heads, 224 and 448:
  // 59.7 and 48.0, 59.4 and 52.4; 80 heads, 240 and 480: 43.9 and 36.2, 46.2 and 41.9).  Over a host link nothing is gained.  And a
  // block is to have pages enough for what it costs by itself (168 heads x 33 pages, one block and two, 23.1 and 24.4 us, 200 29.3
  // and 31.3; a head of 65 pages keeps its four blocks where 256 fit, though six would be 10 % faster).  Heads of one block each that many scoring
  // blocks come before find units to themselves as long as they are few
  // (one block and three: 136 heads x 344 candidates 34.5 and 36.7, 168 42.0 and 43.7; but 160 x 218 47.5 and 39.8, 168 x 187 49.3
  // and 40.9, and 224 x 468, one and two, 71.8 and 61.4).
  const int blocks_now = heads * n_splits;
  const bool loose = n_splits == 1 && g.n_cand > kManyScored && blocks_now <= kFewAlone;
  const bool cut_finer = n_att <= kShortStream ? n_att >= kEnoughToCut && !loose : blocks_now > kLooseBlocks && blocks_now < kComputeUnits;
  if (slices == 1 && g.n_cand < kLongList && !io.host_pool && cut_finer && (long)heads * rows > kLayerResident) {
    cut(std::min(kLayerResident, heads * std::max(n_splits, n_att / kPagesEach)));
    if ((long)heads * rows > kLayerMaxBlocks) cut(most_waiting());
  }
  LayerLaunch l;
  l.home = heads_at_home(d, heads, rows, bytes);
  if (l.home && n_splits > kMaxWaitingHome) {
    n_splits = kMaxWaitingHome;
    pps = (n_att + n_splits - 1) / n_splits;
    if (io.host_pool) n_splits = (n_att + pps - 1) / pps;
    size();
  }
  if (n_splits > 63 || pps > 64 * STEP_WAVES) return false;
  const int passes_log2 = passes == 4 ? 2 : passes == 2 ? 1 : 0;
  int slices_log2 = 0;
  while ((1 << slices_log2) < slices) slices_log2 += 1;
  l.lds = (size_t)select_key_words(g.n_cand) * sizeof(uint32_t) + (io.host_pool ? plan_lds_ints(d.k) * sizeof(int32_t) : 0);
  const size_t lds_attn = (size_t)attn_lds_floats(STEP_WAVES, d.G) * sizeof(float);
  if (lds_attn > l.lds) l.lds = lds_attn;
  const long blocks = (long)heads * rows;
  if (g_one_launch < 0 && (heads > kLayerMaxHeads || (long)heads * n_att > kLayerMaxAttended ||
                           blocks > (io.host_pool ? kLayerMaxBlocksHost : kLayerMaxBlocks) || l.lds > kLdsPerUnit / 2)) return false;
  l.grid = dim3(l.home ? by_xcd(heads) : heads, rows);
  l.packed = (uint32_t)(g.L - 1) | (uint32_t)io.layer << 19;
  l.plan = (io.have_prev ? 1u : 0u) | (uint32_t)io.parity << 1 | (uint32_t)passes_log2 << 2 | (uint32_t)slices_log2 << 4 |
           (uint32_t)n_splits << 7 | (io.lose_selection ? 1u << 22 : 0u) | io.impatient << 23;
  l.split_magic = n_splits > 1 ? 0xffffffffu / (uint32_t)n_splits + 1u : 0u;      // exact for the block counts of a layer launch
  *io.launch_grid = (int)(l.grid.x * l.grid.y);
  *io.launch_lds = l.lds;
  *io.launch_home = l.home;
  const int stream = stream_of(d, g);
  const bool other = d.sel_pool != 0;
  const auto host = stream & STREAM_SUMMARIES ? (other ? launch_layer_host_stream_pool : launch_layer_host_stream) : other ? launch_layer_host_pool : launch_layer_host;
  const auto hbm = stream & STREAM_PAGES ? (other ? launch_layer_hbm_past_pool : launch_layer_hbm_past)
                   : stream & STREAM_SUMMARIES ? (other ? launch_layer_hbm_stream_pool : launch_layer_hbm_stream) : other ? launch_layer_hbm_pool : launch_layer_hbm;
  return (io.host_pool ? host : hbm)(io, l, d.dtype, d.G, st);
}

// ---------------------------------------------------------------------------------
// The cost of a launch as such: a kernel of the same shape whose blocks return at once.
// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(STEP_THREADS) void floor_kernel(uint32_t* sink) {
  extern __shared__ __attribute__((aligned(16))) uint32_t dyn_lds[];
  if (sink) *sink = dyn_lds[0];             // never taken: keeps the LDS allocation in the kernel
}

bool launch_floor(int grid, size_t lds, int reps, hipStream_t st) {
  static size_t granted = 48 * 1024;
  if (lds > granted) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&floor_kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
      (void)hipGetLastError();
      return false;
    }
    granted = lds;
  }
  for (int r = 0; r < reps; ++r) floor_kernel<<<grid, STEP_THREADS, lds, st>>>(nullptr);
  return true;
}

}  // namespace fkv
