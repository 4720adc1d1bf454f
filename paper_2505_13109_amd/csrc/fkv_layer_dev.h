// The one-launch layer kernel (the step roles plus the attention blocks) and the launch of one of its variants.
#pragma once
#include "fkv_step_dev.h"
#include "fkv_attn_dev.h"

#include <hip/hip_ext.h>

#pragma clang fp contract(off)

namespace fkv {

// ---------------------------------------------------------------------------------
// The whole layer-step in ONE launch: the step roles followed by the attention blocks.  In a step without correction
// the two chains do not depend on each other -- attention reads the previous step's page ids, takes the new token from
// the step's inputs and redoes the (tiny) correction test itself -- so they overlap; the attention blocks
// of a corrected head wait for that head's selection, made by blocks with lower indices.
// grid (heads, step rows + splits)
// ---------------------------------------------------------------------------------
typedef const __attribute__((address_space(4))) LayerConst* LayerConstPtr;   // (scalar loads)

// packed: L - 1 (19 bits) | layer (13);   plan: have_prev, parity, passes log2 (2), slices log2 (3), splits (6), 9 unused
// bits, lose_selection, WAIT_* bits (6);   split_magic: 2^32 / splits rounded up, 0 for one split
struct LayerKernelArgs {                     // the kernel's arguments, in their order
  const LayerConst* consts;
  const uint16_t *q, *k_new, *v_new;
  float* out;
  uint32_t packed, host_numbered, plan, split_magic;
};

// what every block works out from the constants
template <bool HOSTPOOL, bool MEAN, bool HOME>
struct LayerSetup {
  LayerConstPtr c;
  char* base;
  uint16_t* qprev0;
  int32_t *ids0, *slots0;
  Geom g;
  uint32_t tag;
  PoolDesc pd;
  static constexpr bool home = HOME;
  int layer, now, before, chunks, passes_log2, slices_log2, slices, step_rows;      // now, before: halves (PENDING / staged, ACTIVE / previous)
  __device__ __forceinline__ explicit LayerSetup(const LayerKernelArgs& ka) {
    c = (LayerConstPtr)ka.consts;
    layer = (int)(ka.packed >> 19);
    now = (int)(ka.plan >> 1) & 1;
    before = now ^ 1;
    base = c->dev_base + c->layer_bytes * (unsigned long long)layer;
    g = geom_of((int)(ka.packed & 0x7ffffu) + 1, c->n_sink, c->n_win, c->k);
    tag = ka.host_numbered ? ka.host_numbered : device_tag((uint32_t)*(const __attribute__((address_space(4))) int*)c->launch_no);
    qprev0 = reinterpret_cast<uint16_t*>(at(c->o_qprev));
    ids0 = reinterpret_cast<int32_t*>(at(c->o_ids));
    slots0 = reinterpret_cast<int32_t*>(at(c->o_slots));
    pd.pool = reinterpret_cast<uint16_t*>(base);
    pd.units_per_head = c->units_per_head;
    pd.placement = HOSTPOOL ? 1 : 0;
    pd.ring_base = c->ring_base; pd.n_ring = c->n_ring; pd.sel_base = c->sel_base;
    passes_log2 = (int)(ka.plan >> 2) & 3;
    const int chunk_log2 = 5 + passes_log2;
    static_assert(PAGES_PER_PASS == 32, "chunks are a power of two of pages");
    chunks = (g.n_cand + (1 << chunk_log2) - 1) >> chunk_log2;
    slices_log2 = (int)(ka.plan >> 4) & 7;
    slices = 1 << slices_log2;
    step_rows = 2 + chunks + slices;
  }
  __device__ __forceinline__ char* at(uint32_t o) const { return base + (unsigned long long)o * 256; }
  __device__ __forceinline__ uint16_t* qprev(int half) const { return qprev0 + (size_t)half * c->qprev_half; }
  __device__ __forceinline__ int32_t* ids(int half) const { return ids0 + (size_t)half * c->ids_half; }
  __device__ __forceinline__ int32_t* slots(int half) const { return slots0 + (size_t)half * c->ids_half; }

  __device__ __forceinline__ StepArgs step_args(const LayerKernelArgs& ka) const {
    StepArgs a;
    a.roles = ROLE_APPEND | ROLE_CORR | ROLE_SELECT;
    a.heads = c->heads; a.k = c->k; a.max_pages = c->max_pages; a.g = g; a.pd = pd;
    a.summ = reinterpret_cast<uint16_t*>(at(c->o_summ));
    a.k_new = ka.k_new; a.v_new = ka.v_new; a.q = ka.q;
    a.q_prev = qprev(before); a.q_stage = qprev(now);
    a.have_prev = (int)(ka.plan & 1u); a.tau = c->tau; a.corr_pool = c->corr_pool;
    a.flags = reinterpret_cast<uint8_t*>(at(c->o_flags)); a.flags_user = nullptr;
    a.cosine = reinterpret_cast<double*>(at(c->o_cosine));
    a.sel_pool = MEAN ? 0 : c->sel_pool; a.P = c->P; a.score = c->score;
    a.ids = ids(now); a.ids_user = nullptr;
    a.chunks = chunks; a.passes = 1 << passes_log2; a.slices = slices; a.slices_log2 = slices_log2;
    a.slice = (g.n_cand + slices - 1) >> slices_log2;
    a.by_itself = &reinterpret_cast<LayerStatus*>(at(c->o_status))->by_itself;
    a.exch = c->exch; a.keyx = c->keyx; a.keyid = c->keyid; a.cmax = c->cmax; a.no = LaunchNo{tag, nullptr}; a.home = home; a.impatient = ka.plan >> 23; a.tstamp = c->tstamp;
    a.tagged = reinterpret_cast<unsigned long long*>(at(c->o_tagged));
    a.plan_act_ids = a.plan_act_slots = nullptr; a.plan_new_slots = a.plan_miss = nullptr; a.plan_lds_off = 0;
    if (HOSTPOOL) {
      a.plan_act_ids = ids(before);
      a.plan_act_slots = slots(before);
      a.plan_new_slots = slots(now);
      a.plan_miss = reinterpret_cast<int32_t*>(at(c->o_miss));
      a.plan_lds_off = select_key_words(g.n_cand);
    }
    return a;
  }
  __device__ __forceinline__ AttnArgs attn_args(const LayerKernelArgs& ka, int G) const {
    AttnArgs a;
    a.pd = pd; a.q = ka.q;
    a.act_ids = ids(before); a.new_ids = nullptr;
    a.act_slots = HOSTPOOL ? slots(before) : nullptr; a.new_slots = nullptr;
    a.flags = nullptr; a.use = 2; a.part = c->part; a.part_ml = c->part_ml; a.max_splits = c->max_splits;
    a.n_splits = (int)(ka.plan >> 7) & 63;
    a.share = ka.split_magic ? (int)__umulhi((uint32_t)(G * D + a.n_splits - 1), ka.split_magic) : G * D;
    const int n_att = g.n_sink + c->k + g.n_win + (g.r > 0 ? 1 : 0);
    a.pps = ka.split_magic ? (int)__umulhi((uint32_t)(n_att + a.n_splits - 1), ka.split_magic) : n_att;
    a.no = LaunchNo{}; a.out = ka.out; a.g = g; a.n_kv = c->n_kv; a.G = G; a.k = c->k;
    a.status = reinterpret_cast<LayerStatus*>(at(c->o_status)); a.tstamp = c->tstamp;
    a.q_prev = qprev(before); a.have_prev = (int)(ka.plan & 1u); a.tau = c->tau; a.corr_pool = c->corr_pool;
    a.k_new = ka.k_new; a.v_new = ka.v_new; a.tagged = reinterpret_cast<unsigned long long*>(at(c->o_tagged));
    a.tag = tag; a.pick_tag = tag + ((ka.plan >> 22) & 1u ? 2u : 0u);
    a.impatient = ka.plan >> 23; a.home = home; a.at_once = slices_log2 == 0;
    a.host_pool = HOSTPOOL ? reinterpret_cast<const uint16_t*>(c->host_base + c->host_layer_bytes * (unsigned long long)layer) : nullptr;
    a.max_pages = c->max_pages;
    return a;
  }
};

// what a kernel is compiled for, beside the STREAM_* bits: the method's pooling, or any other (select_rows)
constexpr int OTHER_POOLING = 4;
static_assert(OTHER_POOLING > (STREAM_SUMMARIES | STREAM_PAGES), "");

template <int DT, int G, bool HOSTPOOL, int KIND, bool HOME>
__device__ __forceinline__ void layer_step(const LayerConst* consts, const uint16_t* q, const uint16_t* k_new, const uint16_t* v_new, float* out,
                                           uint32_t packed, uint32_t host_numbered, uint32_t plan, uint32_t split_magic) {
  extern __shared__ __attribute__((aligned(16))) uint32_t dyn_lds[];
  constexpr int STREAM = KIND & ~OTHER_POOLING;
  constexpr bool MEAN = (KIND & OTHER_POOLING) == 0;
  touch<sizeof(LayerConst)>((LayerConstPtr)consts);
  const LayerKernelArgs ka{consts, q, k_new, v_new, out, packed, host_numbered, plan, split_magic};
  const LayerSetup<HOSTPOOL, MEAN, HOME> u(ka);
  StepArgs s;
  int head, nw = SEL_WAVES, own = 0;           // own: a selecting block's slice of the head's candidates, an attention block's split
  Selected got = Selected::NOTHING;
  AttnLeft left{};
  const bool step = (int)blockIdx.y < u.step_rows;
  const auto again = [] {
    const LayerKernelArgs ka = args_from_memory<LayerKernelArgs>();
    return LayerSetup<HOSTPOOL, MEAN, HOME>(ka).step_args(ka);
  };
  if (step) {
    s = u.step_args(ka);
    bool go_on = false;
    asm volatile(".p2align 6");       // (where the roles' code starts within 64 bytes is worth up to 2 %)
    step_roles<DT, G, (STREAM & STREAM_SUMMARIES) != 0>(s, blockIdx.x, blockIdx.y, [&](int m, int slice) {
      head = m;
      own = slice;
      go_on = select_begin<G, true, MEAN>(s, m, slice, dyn_lds, nw, got, again);
    });
    if (!go_on) return;
  } else {
    const AttnArgs a = u.attn_args(ka, G);
    // numbered through row by row and dealt to the heads, whose blocks wait for each other
    const uint32_t wide = (uint32_t)(HOME ? (u.c->heads + 7) & ~7 : u.c->heads);
    deal_block((blockIdx.y - (uint32_t)u.step_rows) * wide + blockIdx.x, a.n_splits, HOME,
               [&](uint32_t j) { return split_magic ? __umulhi(j, split_magic) : j; }, head, own);
    if (head >= u.c->heads) return;
    left = attn_block<DT, STEP_WAVES, true, HOSTPOOL, (STREAM & STREAM_PAGES) != 0>(a, own, head, reinterpret_cast<float*>(dyn_lds));
    if (__builtin_expect(!left.any(), 1)) return;
    // What follows is hardly ever run.  Its arguments come from memory once more: kept up to here they would cost the page
    // loop registers.
    s = again();
    if (left.ids) lds_barrier();                             // (the LDS is free)
  }
  if (step || left.ids) {
    select_finish<DT, G, true>(s, head, own, dyn_lds, nw, got, again);
  }
  if (step) return;
  const LayerKernelArgs args = args_from_memory<LayerKernelArgs>();
  attn_finish<DT, STEP_WAVES, true, HOSTPOOL>(LayerSetup<HOSTPOOL, MEAN, HOME>(args).attn_args(args, G), own, head, left);
}

// KIND: STREAM_* bits, OTHER_POOLING.  home_: a head's blocks on one XCD; two kernels, as in fkv_step_dev.h (8 heads x 992 candidates 8.5 us with a
// test beside each store, 8.2 without).  Four waves to a SIMD, no more and no fewer: with only the lower limit the compiler schedules for
// more and leaves a slot of scratch memory, that nobody reads or writes, to kernels of G = 7 and 8, which costs each launch 0.9 us.
template <int DT, int G, bool HOSTPOOL, int KIND>
__global__ __launch_bounds__(STEP_THREADS) __attribute__((amdgpu_waves_per_eu(4, 4)))
void layer_kernel(const LayerConst* consts, const uint16_t* q, const uint16_t* k_new, const uint16_t* v_new, float* out,
                  uint32_t packed, uint32_t host_numbered, uint32_t plan, uint32_t split_magic) {
  layer_step<DT, G, HOSTPOOL, KIND, false>(consts, q, k_new, v_new, out, packed, host_numbered, plan, split_magic);
}
template <int DT, int G, bool HOSTPOOL, int KIND>
__global__ __launch_bounds__(STEP_THREADS) __attribute__((amdgpu_waves_per_eu(4, 4)))
void home_layer_kernel(const LayerConst* consts, const uint16_t* q, const uint16_t* k_new, const uint16_t* v_new, float* out,
                       uint32_t packed, uint32_t host_numbered, uint32_t plan, uint32_t split_magic) {
  layer_step<DT, G, HOSTPOOL, KIND, true>(consts, q, k_new, v_new, out, packed, host_numbered, plan, split_magic);
}

template <int DT, int G, bool HOSTPOOL, int KIND, bool HOME>
static bool launch_layer_g(const LayerIO& io, const LayerLaunch& l, hipStream_t st) {
  static size_t granted = 48 * 1024;
  constexpr auto kernel = HOME ? &home_layer_kernel<DT, G, HOSTPOOL, KIND> : &layer_kernel<DT, G, HOSTPOOL, KIND>;
  if (!grant_lds(kernel, l.lds, granted)) return false;
  if (io.done)
    hipExtLaunchKernelGGL(kernel, l.grid, dim3(STEP_THREADS), l.lds, st, nullptr, io.done, 0,
                          io.consts, io.q, io.k_new, io.v_new, io.out, l.packed, io.tag, l.plan, l.split_magic);
  else
    kernel<<<l.grid, STEP_THREADS, l.lds, st>>>(io.consts, io.q, io.k_new, io.v_new, io.out, l.packed, io.tag, l.plan, l.split_magic);
  return true;
}

// one of these in each of the files that share the kernel's variants
template <bool HOSTPOOL, int KIND>
static bool launch_layer_variant(const LayerIO& io, const LayerLaunch& l, int dtype, int G, hipStream_t st) {
  switch (G) {
#define FKV_CASE(GG) case GG: return dtype == 0 ? (l.home ? launch_layer_g<0, GG, HOSTPOOL, KIND, true>(io, l, st) : launch_layer_g<0, GG, HOSTPOOL, KIND, false>(io, l, st)) \
                                                : (l.home ? launch_layer_g<1, GG, HOSTPOOL, KIND, true>(io, l, st) : launch_layer_g<1, GG, HOSTPOOL, KIND, false>(io, l, st));
    FKV_CASE(1) FKV_CASE(2) FKV_CASE(3) FKV_CASE(4) FKV_CASE(5) FKV_CASE(6) FKV_CASE(7) FKV_CASE(8)
#undef FKV_CASE
    default: return false;
  }
}

}  // namespace fkv
