// Internal declarations shared by the host API and the kernel files.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

namespace fkv {

// Dispatch overrides for experiments (sweeps of tile and launch shapes).  They are read from the
// environment only in a build with -DFKV_EXPERIMENT_KNOBS; the product library has none.
inline int knob(const char* name, int dflt) {
#ifdef FKV_EXPERIMENT_KNOBS
  const char* e = getenv(name);
  return e ? atoi(e) : dflt;
#else
  (void)name;
  return dflt;
#endif
}

constexpr int D = 128;            // head_dim
constexpr int PG = 32;            // page size p
constexpr int UNIT_ELEMS = 2 * PG * D;        // K page then V page of one (page, KV head)
constexpr int UNIT_BYTES = UNIT_ELEMS * 2;    // 16 KiB, the contiguous recall unit (Sec. 4.2)
constexpr int MAX_G = 8;

// Geometry of the budget at the current context length (Sec. 2.1: B, S, W).
struct Geom {
  int L;        // tokens cached, the appended one included
  int n_full;   // full pages
  int r;        // tokens in the open page
  int n_sink;   // sink pages [0, n_sink)
  int n_win;    // window pages [n_full - n_win, n_full)
  int cand_lo;  // candidate pages [cand_lo, cand_lo + n_cand)
  int n_cand;
  int k_eff;    // pages picked per KV head = min(k, n_cand)
};

__host__ __device__ inline Geom geom_of(int L, int n_sink, int n_win, int k) {   // sink, window and selectable pages of the budget
  Geom g;
  g.L = L;
  g.n_full = L / PG;
  g.r = L % PG;
  g.n_sink = n_sink < g.n_full ? n_sink : g.n_full;
  const int rest = g.n_full - g.n_sink;
  g.n_win = n_win < rest ? n_win : rest;
  g.cand_lo = g.n_sink;
  g.n_cand = g.n_full - g.n_sink - g.n_win;
  g.k_eff = k < g.n_cand ? k : g.n_cand;
  return g;
}

// The attend-list positions that a head's blocks have where they are dealt to them in turn: block `split` of n_splits the split-th,
// then every n_splits-th, in the order that nth_position counts; wave w of NW takes in lane 0 the one that nth_of_wave names, in lane 1
// another, and so on.  The last position comes first: it is the open page, whose wave also takes in the step's new token, and lane 0 deals
// from the last wave down, so that this wave is the one that gets a second page last.  (With the open page where its number puts
// it, it was a wave's second page wherever a block has nine to eleven: 20 heads of 129 pages x 992 candidates 14.5 us a layer-step, so
// 13.9; 32 of 65 13.3 and 12.6; 76 of 33 x 480 18.6 and 17.7; where most heads are corrected, 20.2 and 20.1, 18.5 and 18.5, 21.9 and
// 21.5, but 64 of 33 x 992 20.6 and 21.1.)
__host__ __device__ inline int nth_of_wave(int wave, int lane, int n_waves) { return lane == 0 ? n_waves - 1 - wave : wave + lane * n_waves; }
__host__ __device__ inline int nth_position(int nth, int n_att) { return nth == 0 ? n_att - 1 : nth < n_att ? nth - 1 : n_att; }      // (n_att: none)

// Where a KV head's pages live in HBM.  Unit u of head (b, m) starts at
// pool + ((b * n_kv + m) * units_per_head + u) * UNIT_ELEMS.
struct PoolDesc {
  uint16_t* pool;
  int units_per_head;
  int placement;     // 0: unit = page id.  1: sink page i -> unit i, window/open page j -> ring_base + j % n_ring,
  int ring_base;     //    picked page in slot s -> sel_base + s
  int n_ring;
  int sel_base;
};

// ---- element offsets inside a unit -------------------------------------
// K page: [s*2+mb (8)][kb (4)][m (16)][e (8)] with channel = (s*4+kb)*8 + e, token = mb*16 + m.
// Each group of 512 elements (1 KiB) is one operand load of the 16x16x32 MFMA
// computing S^T = K Q^T: lane (kb*16 + m) reads 8 consecutive channels of token m.
__host__ __device__ inline int k_elem_off(int t, int ch) {
  int s = ch >> 5, kb = (ch >> 3) & 3, e = ch & 7, mb = t >> 4, m = t & 15;
  return ((((s * 2 + mb) * 4 + kb) * 16 + m) * 8) + e;
}
// V page: [cb (8)][kb (4)][m (16)][e (8)] with channel = cb*16 + m and
// token = (e < 4) ? kb*4 + e : 16 + kb*4 + (e - 4): the token order in which the
// S^T accumulators of a lane come out, so P feeds the second MFMA from registers.
__host__ __device__ inline int v_elem_off(int t, int ch) {
  int cb = ch >> 4, m = ch & 15, hi = t >> 4, kb = (t & 15) >> 2, e = (t & 3) + 4 * hi;
  return PG * D + (((cb * 4 + kb) * 16 + m) * 8) + e;
}

// ---- launch wrappers (defined in the kernel files) ----------------------
// same_xcd: blocks whose numbers in a launch are equal modulo 8 run on the same XCD (blocks_by_xcd)
struct Dims { int batch, n_q, n_kv, G, k, max_pages, dtype, max_lds, sel_pool, corr_pool, n_layers; bool same_xcd; };
constexpr int kXcds = 8;
inline int by_xcd(int heads) { return (heads + kXcds - 1) / kXcds * kXcds; }
// Whether the blocks of launches on this device are dealt to its XCDs in turn: by what a launch of kWhereBlocks blocks, which
// each write where they are, leaves at `where` (device memory).
constexpr int kWhereBlocks = 1024;
bool blocks_by_xcd(uint32_t* where);
// Whether a head's blocks, `rows` of them (as blocks of 512 threads) that read `bytes`, are put on one XCD (deal_block).
bool heads_at_home(const Dims& d, int heads, int rows, double bytes, bool attn_only = false);
constexpr double kSummaryBytes = 2 * D * 2;        // of a page

// Launches are numbered (31 bits, from 1), and the values that a launch's blocks exchange carry its number as a tag.  The
// host counts.  A launch that is being captured runs again at every replay with the arguments it was captured with, so its
// number is counted on the device instead, by a small kernel ahead of it; the low bit keeps the two counts' tags apart.
struct LaunchNo {
  uint32_t tag;              // the tag, or
  const int* dev;            // if not null: where the number is
};
__host__ __device__ inline uint32_t host_tag(uint32_t launch) { return (launch << 1) | 1u; }
__host__ __device__ inline uint32_t device_tag(uint32_t launch) { return launch << 1; }

// What a decode step reads past the memory-side cache (256 MB), as bits.  All layers' summaries and attended pages are read again
// at the next token, so as long as they fit they are better left there.  If they do not, a cyclic order of reads keeps
// hardly any of them, and the summaries, of which more are read for every token served, go first: 8 layers of 32 heads x 992 candidates and 65
// pages, 400 MB in all, 75 us a layer-step -> 63; but 268 MB in all 1 % slower, and with the pages past the cache as well 71.
// Where the pages by themselves are too many, they go too.  A pass in the cache and past it, by the pages that there are to
// attend (a short context has fewer than its budget): 32 layers of 8 heads x 55 pages, 230 MB, 821 and 857 us; x 65, 272 MB, 843 and 854;
// x 82, 344 MB, 881 and 874; 3 layers of 320 heads x 17, 267 MB, 776 and 798; 2 x 33, 346 MB, 787 and 763; 2 layers of 384 heads
// x 33, 415 MB, 899 and 826.  In the launches of a scan as well: one layer of 256 heads x 942 candidates and 17 pages, 195 MB, 398 us past the
// cache and 381 in it.
constexpr int STREAM_SUMMARIES = 1, STREAM_PAGES = 2;      // (the second only with the first)
inline int stream_of(const Dims& d, const Geom& g) {
  const double heads = (double)d.n_layers * d.batch * d.n_kv;
  const double pages = heads * (g.n_sink + g.k_eff + g.n_win + 1) * UNIT_BYTES, summaries = heads * g.n_cand * 2 * D * 2;
  return (pages + summaries > 270e6 ? STREAM_SUMMARIES : 0) | (pages > 310e6 ? STREAM_PAGES : 0);
}

// Per layer, in device memory.  lost: ids that a block had written by then were not there (fkv_health).  by_itself: how often a selecting
// block or a wave of attention made alone what it else gets from other blocks of its launch (fkv_test_by_itself).
struct LayerStatus { int lost, by_itself; };

// what blocks of a launch wait for, as bits (a test makes waits of these kinds run out at once)
constexpr uint32_t WAIT_WEIGHTS = 1, WAIT_MAXIMA = 2, WAIT_SUMS = 4, WAIT_KEYS = 8, WAIT_SPLITS = 16, WAIT_IDS = 32;

// the fused step kernel: roles are OR-ed
constexpr int ROLE_APPEND = 1, ROLE_CORR = 2, ROLE_SELECT = 4;
struct StepIO {
  PoolDesc pd; uint16_t* summ; const uint16_t* k_new; const uint16_t* v_new;      // append
  const uint16_t* q; const uint16_t* q_prev; uint16_t* q_stage; int have_prev; float tau;
  uint8_t* flags; uint8_t* flags_user; double* cosine;                               // correction test
  unsigned long long* P; float* P_plain; float* score; int32_t* ids; int32_t* ids_user;              // selection
  unsigned long long* exch; unsigned long long* keyx; unsigned long long* keyid;     // its exchange between blocks
  unsigned long long* cmax; float* cmax_plain;                                       // largest weights of the scored chunks
  LaunchNo no; uint32_t impatient; LayerStatus* status;
  bool* P_tagged;                                                                    // out: whether the launch wrote P or P_plain
  long long* tstamp;                                                                 // debug timestamps or null
  // KV in a host pool (else all null): a launch with ROLE_SELECT also makes the recall plan of the new selection --
  // ACTIVE ids and slots in, PENDING slots and miss lists out
  const int32_t* plan_act_ids; const int32_t* plan_act_slots; int32_t* plan_new_slots; int32_t* plan_miss;
};
constexpr int EXCH_WORDS = 16 * 2 * MAX_G;   // per head: what the selecting blocks of a head tell each other
// Per head, the largest weight of every chunk of pages that was scored together, for each query head of the group (a power of
// two of them): by scoring blocks of the same launch, 32 pages or more each; by waves of the scan, 16 pages each
__host__ __device__ constexpr int group_pow2(int G) { return G <= 1 ? 1 : G <= 2 ? 2 : G <= 4 ? 4 : 8; }
__host__ __device__ constexpr size_t cmax_stride(int max_pages) { return (size_t)((max_pages + 31) / 32) * MAX_G; }
__host__ __device__ constexpr size_t cmax_plain_stride(int max_pages) { return (size_t)((max_pages + 63) / 64) * 4 * MAX_G; }
int launch_step(const Dims& d, int roles, const StepIO& io, Geom g, hipStream_t st);   // returns the launches made
// What the one-launch layer-step needs and no step changes: kept in device memory, one per context, so that a launch hands
// over 56 bytes -- which the hardware preloads into scalar registers -- and finds the rest in the L2 of every XCD.  (Fresh
// arguments are a miss of about 0.7 us for every 64 bytes that a block touches, one after the other along its chain.)
struct LayerConst {
  // per layer, as offsets from the layer's base in units of 256 bytes; ..._half: from the first to the second of a
  // ping-pong pair, in elements
  char* dev_base;
  unsigned long long layer_bytes;
  uint32_t o_summ, o_qprev, o_ids, o_slots, o_flags, o_miss, o_cosine, o_status, o_tagged;
  int32_t qprev_half, ids_half;
  // per context
  int32_t heads, n_kv, k, max_pages, max_splits, n_sink, n_win;      // heads: (request, KV head) pairs
  int32_t units_per_head, ring_base, n_ring, sel_base;
  int32_t corr_pool, sel_pool;
  float tau;
  unsigned long long *P, *part, *part_ml, *exch, *keyx, *keyid, *cmax;
  float* score;
  const int* launch_no;                      // number of the last captured launch
  const char* host_base;                     // KV in a host pool (else null)
  unsigned long long host_layer_bytes;
  long long* tstamp;                         // debug timestamps or null
};
// the whole layer-step (step roles + attention) in one launch; false if this shape or placement
// has to take the separate launches
struct LayerIO {
  const LayerConst* consts;                  // device memory
  int layer, parity, have_prev;
  const uint16_t *q, *k_new, *v_new;
  float* out;
  uint32_t tag;                              // of this launch; 0: number it by what is at consts->launch_no
  bool host_pool;
  int max_splits;
  uint32_t impatient;                        // WAIT_* bits
  bool lose_selection;                       // test of the bounded wait: attention waits for a tag that never comes
  hipEvent_t done;                           // if not null: recorded by the launch itself
  int* launch_grid; size_t* launch_lds; bool* launch_home;      // out: shape of the launch that was made, whether heads are at home
};
// `reps` launches of a kernel that does nothing, with the given grid, 512 threads and dynamic LDS
bool launch_floor(int grid, size_t lds, int reps, hipStream_t st);
bool launch_layer(const Dims& d, const LayerIO& lio, Geom g, hipStream_t st);
// how launch_layer has it launched, by the file that has the variant
struct LayerLaunch { dim3 grid; bool home; size_t lds; uint32_t packed, plan, split_magic; };
bool launch_layer_hbm(const LayerIO& io, const LayerLaunch& l, int dtype, int G, hipStream_t st);
bool launch_layer_hbm_stream(const LayerIO& io, const LayerLaunch& l, int dtype, int G, hipStream_t st);
bool launch_layer_hbm_past(const LayerIO& io, const LayerLaunch& l, int dtype, int G, hipStream_t st);
bool launch_layer_host(const LayerIO& io, const LayerLaunch& l, int dtype, int G, hipStream_t st);
bool launch_layer_host_stream(const LayerIO& io, const LayerLaunch& l, int dtype, int G, hipStream_t st);
// ... of the poolings beside the method's
bool launch_layer_hbm_pool(const LayerIO& io, const LayerLaunch& l, int dtype, int G, hipStream_t st);
bool launch_layer_hbm_stream_pool(const LayerIO& io, const LayerLaunch& l, int dtype, int G, hipStream_t st);
bool launch_layer_hbm_past_pool(const LayerIO& io, const LayerLaunch& l, int dtype, int G, hipStream_t st);
bool launch_layer_host_pool(const LayerIO& io, const LayerLaunch& l, int dtype, int G, hipStream_t st);
bool launch_layer_host_stream_pool(const LayerIO& io, const LayerLaunch& l, int dtype, int G, hipStream_t st);
// Dynamic LDS above the default 64 KiB per block has to be granted per kernel function; false if the device refuses.
template <typename F>
static bool grant_lds(F* fn, size_t lds, size_t& granted) {
  if (lds <= granted) return true;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  granted = lds;
  return true;
}

constexpr int kComputeUnits = 256;
// Most blocks of a launch that wait for each other (a head's attention blocks, and its selecting blocks where it has several):
// half of those that fit (two to a compute unit), and all of them where there is something to be had by that (launch_layer).  That
// keeps waits short: in block order at most one head's blocks are half there, so a launch by itself gets on, and two at once mostly
// do.  It is not what makes them end: with more launches on the machine, or another program's, a block may wait for one that cannot
// start, and goes on by itself (PATIENCE).
// At home one head per XCD and launch may be half there, in the XCD's 64 slots: no more blocks to a head than leave slots for others
// when all four launches that a process has on the machine at once (its hardware queues) are there with one block missing.
constexpr int kMaxWaiting = kComputeUnits, kMaxWaitingHome = 2 * kComputeUnits / kXcds / 4;
int attn_pages_per_block(int n_att, int heads, int max_splits, int nw, int max_blocks = kMaxWaiting);
void launch_load_prefix(const Dims& d, const PoolDesc& pd, uint16_t* summ, uint16_t* host_pool,
                        const uint16_t* K, const uint16_t* V, int n_tokens, int32_t* ids, hipStream_t st);   // ids: [2][heads][k], emptied
void launch_summary_recompute(const Dims& d, const PoolDesc& pd, uint16_t* summ, int first_page,
                              int n_pages, Geom g, hipStream_t st);
void launch_offload(const Dims& d, const PoolDesc& pd, uint16_t* host_pool, int page, hipStream_t st);
// new_ids is read and, where an id is not a full page (id < 0 or id >= n_full), rewritten to -1
void launch_plan(const Dims& d, int32_t* new_ids, const int32_t* act_ids, const int32_t* act_slots,
                 int32_t* new_slots, int32_t* miss, int n_full, hipStream_t st);
// recall of missing pages, host pool -> page-cache slots, for up to GATHER_MAX_LAYERS layers in one launch;
// heads: FKV_HEADS_* (all, flagged only, unflagged only -- by each layer's own flags)
constexpr int GATHER_MAX_LAYERS = 8;
struct GatherLayers {
  int n;
  PoolDesc pd[GATHER_MAX_LAYERS];
  const uint16_t* host_pool[GATHER_MAX_LAYERS];
  const int32_t* miss[GATHER_MAX_LAYERS];
  const uint8_t* flags[GATHER_MAX_LAYERS];
};
// done: if not null, an event that the (last) launch records
void launch_gather(const Dims& d, const GatherLayers& gl, int heads, hipStream_t st, hipEvent_t done = nullptr);
struct AttnIO {
  const uint16_t* q; const int32_t* act_ids; const int32_t* new_ids; const int32_t* act_slots; const int32_t* new_slots;
  const uint8_t* flags; int use;
  unsigned long long* part; unsigned long long* part_ml; int max_splits;
  LaunchNo no; uint32_t impatient;
  LayerStatus* status; float* out; long long* tstamp;
};
void launch_attn(const Dims& d, const PoolDesc& pd, const AttnIO& io, Geom g, hipStream_t st, hipEvent_t ev_begin, hipEvent_t ev_end);
void launch_next_number(int* p, hipStream_t st);            // *p to the next launch number, by a kernel
void launch_read_page(const uint16_t* unit, uint16_t* out_token_major, hipStream_t st);
void launch_export_nhd(const Dims& d, const PoolDesc& pd, const int32_t* act_ids, const int32_t* new_ids,
                       const int32_t* act_slots, const int32_t* new_slots, const uint8_t* flags, int use,
                       uint16_t* out, int32_t* slot_pages, int n_slots, Geom g, hipStream_t st,
                       const int32_t* skip_missing = nullptr);   // miss lists: leave the pages they name to the streamed recall
// recall of the missing pages into their page-cache slots AND, converted, into an NHD pool
void launch_gather_nhd(const Dims& d, const PoolDesc& pd, const uint16_t* host_pool, const int32_t* miss,
                       const uint8_t* flags, int heads, uint16_t* nhd, int n_slots, int n_sink, hipStream_t st);

}  // namespace fkv
