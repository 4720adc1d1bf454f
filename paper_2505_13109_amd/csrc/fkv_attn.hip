// Stand-alone launch of sparse decode attention (device code in fkv_attn_dev.h).
#include "fkv_attn_dev.h"

#include <algorithm>

namespace fkv {

// NW wavefronts per block.  grid: a head's n_splits blocks adjacent (n_splits, heads), beyond kHeadRows heads (a grid dimension ends at
// 65535) folded into a third dimension; at home (8, n_splits, heads / 8), so that a head's blocks are on one XCD (deal_block), up to
// kHomeHeads heads.  A block
// finds its head without a word of its arguments, and whether it is at home is known when this is compiled: with a division by
// n_splits and a test beside each store launches took 0.2 to 0.4 us longer (12 heads of 129 pages 9.2 and 9.0 us; at home, 8 of
// 65 6.2 and 5.9, 8 of 33 5.6 and 5.1).
constexpr int kHeadRows = 1 << 15, kHomeHeads = 65535 * kXcds;
template <int DT, int NW, bool PAST, bool HOME>
__device__ __forceinline__ void attn_of(AttnArgs a, int head, int split) {
  extern __shared__ __attribute__((aligned(16))) float attn_lds[];
  touch_args<sizeof(AttnArgs)>();
  if (head >= a.heads) return;
  a.home = HOME;
  const AttnLeft left = attn_block<DT, NW, false, false, PAST>(a, split, head, attn_lds);
  if (__builtin_expect(left.any(), 0))
    attn_finish<DT, NW, false, false>(args_from_memory<AttnArgs>(), split, head, left);
}
template <int DT, int NW, bool PAST>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(4))) void attn_kernel(AttnArgs a) {
  attn_of<DT, NW, PAST, false>(a, (int)(blockIdx.z * kHeadRows + blockIdx.y), (int)blockIdx.x);
}
template <int DT, int NW, bool PAST>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(4))) void home_attn_kernel(AttnArgs a) {
  attn_of<DT, NW, PAST, true>(a, (int)(blockIdx.z * kXcds + blockIdx.x), (int)blockIdx.y);
}

// experiment builds only (see knob()): pages per block (0 = choose from the shape)
static const int g_pps_override = knob("FKV_ATTN_PPS", 0);

// pages per block of nw waves for a head with n_att attended pages; max_blocks: most blocks of a launch in which a head has
// more than one
int attn_pages_per_block(int n_att, int heads, int max_splits, int nw, int max_blocks) {
  // a page per wave and pass; more pages per block (the page loop is pipelined, the merge gets
  // cheaper) as long as the launch keeps at least ~128 blocks, and never more than 32 splits
  // per KV head beyond that, so that the merge needs few round trips
  const int most = 64 * nw;                         // a wave looks up its positions with one load, one per lane
  int pps = nw;
  while (pps < 16 && (long)heads * ((n_att + pps * 2 - 1) / (pps * 2)) >= 128) pps *= 2;
  while ((n_att + pps - 1) / pps > 32 && (long)heads * ((n_att + pps * 2 - 1) / (pps * 2)) >= 128 && pps < most) pps *= 2;
  // With many heads the launch is bandwidth-bound and what counts is the fixed cost of a block
  // (its partial, the exchange, the merge): measured best at about one block per compute unit,
  // down to one block per head; in the one-launch layer-step at two, where launch_layer lets it.
  const int enough = std::max(kComputeUnits, max_blocks);
  while (pps < n_att && pps < most && (long)heads * ((n_att + pps * 2 - 1) / (pps * 2)) >= enough) pps *= 2;
  // (4-wave blocks fit four to a unit; of long lists, one block to a unit streams better: 248 heads of 129 pages 117.7 us in one
  // split, 120.6 in two)
  if (nw == 4 && n_att <= 96) max_blocks *= 2;
  const int most_splits = std::max(1, std::min(max_splits, max_blocks / heads));
  if ((n_att + pps - 1) / pps > most_splits) pps = std::min((n_att + most_splits - 1) / most_splits, std::max(pps, most));
  while ((n_att + pps - 1) / pps > max_splits) pps *= 2;
  const int n_splits = (n_att + pps - 1) / pps;     // the head split evenly (56 heads of 33 pages: 11 + 11 + 11 13.0 us, 16 + 16 + 1 13.7)
  pps = (n_att + n_splits - 1) / n_splits;
  if (g_pps_override > 0) pps = g_pps_override;
  return pps;
}

void launch_attn(const Dims& d, const PoolDesc& pd, const AttnIO& io, Geom g, hipStream_t st, hipEvent_t ev_begin, hipEvent_t ev_end) {
  const int n_att = g.n_sink + d.k + g.n_win + (g.r > 0 ? 1 : 0), heads = d.n_kv * d.batch;
  AttnArgs a{};
  a.pd = pd; a.q = io.q; a.act_ids = io.act_ids; a.new_ids = io.new_ids; a.act_slots = io.act_slots; a.new_slots = io.new_slots;
  a.flags = io.flags; a.use = io.use; a.part = io.part; a.part_ml = io.part_ml; a.max_splits = io.max_splits;
  a.no = io.no; a.impatient = io.impatient;
  const int pps = attn_pages_per_block(n_att, heads, io.max_splits, 4);
  a.n_splits = (n_att + pps - 1) / pps;
  a.share = (d.G * D + a.n_splits - 1) / a.n_splits;
  a.out = io.out; a.g = g; a.n_kv = d.n_kv; a.G = d.G; a.k = d.k; a.status = io.status; a.tstamp = io.tstamp;
  a.heads = heads;
  const int n_there = n_att - d.k + g.k_eff;
  a.home = a.n_splits > 1 && a.n_splits <= 2 * kMaxWaitingHome && heads <= kHomeHeads &&
           heads_at_home(d, heads, (a.n_splits + 1) / 2, (double)n_there * UNIT_BYTES, true);
  const dim3 grid = a.home ? dim3(kXcds, a.n_splits, by_xcd(heads) / kXcds) : dim3(a.n_splits, std::min(heads, kHeadRows), (heads + kHeadRows - 1) / kHeadRows);
  constexpr int NW = 4;
  const size_t lds = attn_lds_floats(NW, d.G) * sizeof(float);
  if (ev_begin) (void)hipEventRecord(ev_begin, st);
  const bool past = (stream_of(d, g) & STREAM_PAGES) != 0;
#define FKV_LAUNCH(DT, PAST) (a.home ? home_attn_kernel<DT, NW, PAST> : attn_kernel<DT, NW, PAST>)<<<grid, NW * 64, lds, st>>>(a)
  if (d.dtype == 0) { if (past) FKV_LAUNCH(0, true); else FKV_LAUNCH(0, false); }
  else              { if (past) FKV_LAUNCH(1, true); else FKV_LAUNCH(1, false); }
#undef FKV_LAUNCH
  if (ev_end) (void)hipEventRecord(ev_end, st);
}

__global__ void next_number_kernel(int* __restrict__ p) {
  const int n = (*p + 1) & 0x7fffffff;
  *p = n ? n : 1;
}
void launch_next_number(int* p, hipStream_t st) { next_number_kernel<<<1, 1, 0, st>>>(p); }

// ---------------------------------------------------------------------------------
// The pages a head attends, converted to the NHD layout of the paper's hybrid layouts
// (Sec. 4.2): out [batch][n_slots][2 (K, V)][page][n_kv][d], slot s of head m = position s of
// m's attend list; slot_pages [batch][n_kv][n_slots].  One block per (slot, head): the 16 KiB
// unit comes in with linear 16-byte loads, is turned in LDS, and goes out as 256-byte token rows.
// ---------------------------------------------------------------------------------
// `miss` (may be null): the recall plan's miss lists [heads][1 + 3k].  With it, a picked page that the
// plan marked missing is left alone -- its rows arrive through the streamed recall -- and only its
// page id is recorded.
__global__ __launch_bounds__(256) void export_nhd_kernel(AttnArgs a, uint16_t* __restrict__ out,
                                                         int32_t* __restrict__ slot_pages, int n_slots,
                                                         const int32_t* __restrict__ miss) {
  __shared__ __attribute__((aligned(16))) uint16_t unit_lds[UNIT_ELEMS];
  __shared__ int s_missing;
  const int slot = blockIdx.x, m = blockIdx.y, b = blockIdx.z;
  const int head = b * a.n_kv + m, k = a.k;
  const Geom& g = a.g;
  const bool pending = a.use == 1 || (a.use == 2 && a.flags[head] != 0);
  AttendList al;
  al.ids = (pending ? a.new_ids : a.act_ids) + (size_t)head * k;
  al.slots = a.pd.placement == 0 ? nullptr : (pending ? a.new_slots : a.act_slots) + (size_t)head * k;
  al.n_sink = g.n_sink; al.k = k; al.n_win = g.n_win; al.n_full = g.n_full; al.r = g.r;
  const int n_att = g.n_sink + k + g.n_win + (g.r > 0 ? 1 : 0);
  int n_valid = 0, page = -1, unit = -1;
  if (slot < n_att) unit = attend_unit(al, a.pd, slot, n_valid, page);
  if (unit < 0) { page = -1; n_valid = 0; }
  if (threadIdx.x == 0) slot_pages[(size_t)head * n_slots + slot] = page;
  if (miss && unit >= 0 && slot >= g.n_sink && slot < g.n_sink + k) {
    if (threadIdx.x == 0) s_missing = 0;
    __syncthreads();
    const int32_t* mh = miss + (size_t)head * (1 + 3 * k);
    for (int r = threadIdx.x; r < mh[0]; r += 256)
      if (mh[1 + 2 * k + r] == slot - g.n_sink) s_missing = 1;
    __syncthreads();
    if (s_missing) return;
  }
  if (unit >= 0) {
    const uint4* src = reinterpret_cast<const uint4*>(a.pd.pool + ((size_t)head * a.pd.units_per_head + unit) * UNIT_ELEMS);
    uint4* dst = reinterpret_cast<uint4*>(unit_lds);
#pragma unroll
    for (int i = 0; i < UNIT_ELEMS / 8 / 256; ++i) dst[threadIdx.x + i * 256] = src[threadIdx.x + i * 256];
  }
  __syncthreads();
  // 2 x 32 token rows of 16 chunks of 8 channels
  for (int i = threadIdx.x; i < 2 * PG * (D / 8); i += 256) {
    const int c8 = i % (D / 8), t = (i / (D / 8)) % PG, kv = i / (D / 8) / PG;
    uint4 w = make_uint4(0, 0, 0, 0);
    if (t < n_valid) {
      if (kv == 0) {
        w = *reinterpret_cast<const uint4*>(unit_lds + k_elem_off(t, c8 * 8));    // 8 channels lie together
      } else {
        uint16_t e[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) e[c] = unit_lds[v_elem_off(t, c8 * 8 + c)];
        w.x = e[0] | ((uint32_t)e[1] << 16); w.y = e[2] | ((uint32_t)e[3] << 16);
        w.z = e[4] | ((uint32_t)e[5] << 16); w.w = e[6] | ((uint32_t)e[7] << 16);
      }
    }
    uint16_t* row = out + ((((size_t)(b * n_slots + slot) * 2 + kv) * PG + t) * a.n_kv + m) * D;
    *reinterpret_cast<uint4*>(row + c8 * 8) = w;
  }
}

void launch_export_nhd(const Dims& d, const PoolDesc& pd, const int32_t* act_ids, const int32_t* new_ids,
                       const int32_t* act_slots, const int32_t* new_slots, const uint8_t* flags, int use,
                       uint16_t* out, int32_t* slot_pages, int n_slots, Geom g, hipStream_t st, const int32_t* skip_missing) {
  AttnArgs a{};
  a.pd = pd; a.act_ids = act_ids; a.new_ids = new_ids; a.act_slots = act_slots; a.new_slots = new_slots;
  a.flags = flags; a.use = use; a.g = g; a.n_kv = d.n_kv; a.G = d.G; a.k = d.k;
  dim3 grid(n_slots, d.n_kv, d.batch);
  export_nhd_kernel<<<grid, 256, 0, st>>>(a, out, slot_pages, n_slots, skip_missing);
}

}  // namespace fkv
