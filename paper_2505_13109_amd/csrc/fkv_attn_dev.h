// Device code of sparse decode attention over sink + picked pages + window + open page
// (Sec. 2.1), split over pages with an online softmax; a head's blocks share the
// log-sum-exp merge of its splits.
//
// One wavefront owns one 32-token page at a time and keeps everything in registers:
//   S^T[32 tok x 16] = K[32 x 128] . Q^T[128 x 16]       8 x v_mfma_f32_16x16x32
//   O^T[128 x 16]   += V^T[128 x 32 tok] . P^T[32 x 16]   8 (x2: P split hi + lo) MFMAs
// The query group (G <= 8 heads, padded to the 16 columns of the tile) is the N
// dimension of both products, so lane (g = lane % 16, rb = lane / 16) ends the first
// product holding the logits of head g for tokens {rb*4+i, 16+rb*4+i}: exactly the 8
// tokens the same lane must supply as the B operand of the second product (the V page
// is stored in that token order).  Nothing goes through LDS inside the page loop.
//
// What bounds it.  A large launch: the bytes of the pages.  A small one (a request or a few): the chain of dependent
// steps -- page ids, pages, the block's combine, the exchange between the head's blocks, the merge -- each a round trip.
// So every step is entered as early as what it depends on allows: a wave looks up all its positions' ids with one load
// and requests its first page before the correction test is made; the block combines its waves behind one barrier; and
// the partial results are exchanged as tagged words (st_tag), one trip instead of store, counter and read.
//
// What a block waits for -- its head's picked ids, the sums of the head's other blocks -- comes from blocks that may not be
// running yet, and another launch may keep them from it; so a block whose patience ends makes it itself (attn_finish).
#pragma once
#include "fkv_device.h"

namespace fkv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

template <int DT> struct Mma;
template <> struct Mma<0> {
  typedef f16x8 vec;
  static __device__ __forceinline__ f32x4 mma(vec a, vec b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
  // p >= 0 split into two storage-type values whose sum carries ~22 bits of p; pairs, so that the conversions are the packed ones (round
  // to nearest even), which take fewer registers too
  typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
  static __device__ __forceinline__ f16x2 pack(float a, float b) { return __builtin_convertvector((f32x2{a, b}), f16x2); }
  static __device__ __forceinline__ void split(const float* p, vec& hi, vec& lo) {
    u32x4 h, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const f16x2 he = pack(p[2 * e], p[2 * e + 1]);
      h[e] = __builtin_bit_cast(uint32_t, he);
      l[e] = __builtin_bit_cast(uint32_t, pack(p[2 * e] - (float)he[0], p[2 * e + 1] - (float)he[1]));
    }
    hi = __builtin_bit_cast(vec, h);
    lo = __builtin_bit_cast(vec, l);
  }
  static __device__ __forceinline__ float add_pair(uint32_t w, float c) {
    return __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, w), f16x2{(_Float16)1.0f, (_Float16)1.0f}, c, false);
  }
};
template <> struct Mma<1> {
  typedef bf16x8 vec;
  static __device__ __forceinline__ f32x4 mma(vec a, vec b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
  // pairs, so that the conversions are the packed ones (round to nearest even)
  static __device__ __forceinline__ uint32_t pack(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
  }
  static __device__ __forceinline__ void split(const float* p, vec& hi, vec& lo) {
    u32x4 h, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      h[e] = pack(p[2 * e], p[2 * e + 1]);
      l[e] = pack(p[2 * e] - __uint_as_float(h[e] << 16), p[2 * e + 1] - __uint_as_float(h[e] & 0xffff0000u));
    }
    hi = __builtin_bit_cast(vec, h);
    lo = __builtin_bit_cast(vec, l);
  }
  static __device__ __forceinline__ float add_pair(uint32_t w, float c) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), bf16x2{(__bf16)1.0f, (__bf16)1.0f}, c, false);
  }
};

// over the four 16-lane rows of a wave: row pairs, then halves, by the row-swapping moves (no LDS traffic)
__device__ __forceinline__ float max_over_rows(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float sum_over_rows(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

struct AttnArgs {
  PoolDesc pd;
  const uint16_t* q;
  const int32_t* act_ids;    // ACTIVE selection (previous step) and its page-cache slots
  const int32_t* new_ids;    // PENDING selection (this step)
  const int32_t* act_slots;
  const int32_t* new_slots;
  const uint8_t* flags;
  int use;                   // FKV_USE_*: 0 active, 1 pending, 2 by flag
  unsigned long long* part;  // [heads][max_splits][G][D] tagged partial outputs, then [heads][max_splits][G][2] tagged (max, sum)
  unsigned long long* part_ml;
  int max_splits, n_splits;
  int pps;                   // fused, KV in a host pool: positions of a block
  int share;                 // outputs of a head that each of its blocks finishes
  bool home;                 // a head's blocks are on one XCD (deal_block)
  LaunchNo no;               // stand-alone attention: of this launch
  float* out;
  Geom g;
  int heads, n_kv, G, k;     // heads: stand-alone attention: (request, KV head) pairs
  LayerStatus* status;
  long long* tstamp;
  // --- when attention shares its launch with the step roles ("fused") ---
  // flags are recomputed here, the new token is taken from k_new/v_new, a corrected head waits for its selection
  const uint16_t* q_prev;
  int have_prev;
  float tau;
  int corr_pool;
  const uint16_t* k_new;
  const uint16_t* v_new;
  const unsigned long long* tagged;   // [heads][k]: this step's picked ids, tagged, written by the selection
  // the first loads need not wait for the ids: not where several blocks share a head's selection, which is what such a launch waits
  // for and whose scoring blocks' loads would come later (8 heads of 129 pages x 2016 candidates, G = 8: 13.0 us, at once 13.9)
  bool at_once;
  uint32_t tag;              // fused: tag of this launch
  uint32_t pick_tag;         // tag the picked ids are waited for with: the same (a test of the bounded wait asks for another)
  uint32_t impatient;        // WAIT_* bits: waits that run out at once (tests)
  // fused, KV in a host pool: the tagged words are tagged_pick() values; a corrected head's wave copies a missing page
  // from the host pool into its slot while it attends over it
  const uint16_t* host_pool; // [heads][max_pages] units
  int max_pages;
};

// position i of a head's attend list -> HBM unit, page id and number of valid tokens; -1 if empty
struct AttendList {
  const int32_t* ids;
  const int32_t* slots;
  int n_sink, k, n_win, n_full, r;
};
__device__ __forceinline__ int attend_unit(const AttendList& al, const PoolDesc& pd, int i, int& n_valid, int& page) {
  n_valid = PG;
  if (i < al.n_sink) { page = i; return i; }
  i -= al.n_sink;
  if (i < al.k) {
    const int id = al.ids[i];
    page = id;
    if (id < 0) return -1;
    return pd.placement == 0 ? id : pd.sel_base + al.slots[i];
  }
  i -= al.k;
  if (i < al.n_win) page = al.n_full - al.n_win + i;
  else { page = al.n_full; n_valid = al.r; }
  return resident_unit(pd, page);
}

// floats of LDS that a block of NW waves needs
__host__ __device__ constexpr int attn_lds_floats(int NW, int G) { return NW * G * (D + 4) + NW * 32 + G * (D / 2 + 4); }

// One output (query head gg, channel c) by one thread, over the whole attend list in fp32: for outputs whose block waited for
// the others in vain.  Slow (3 ms for 65 pages, 9 for 129), but it needs nobody.  corrected: the picked ids are this launch's;
// should they not be there (a test sees to that; a block makes them before it comes here), the output is NaN.
template <int DT, bool FUSED, bool HOSTFUSED>
__device__ __forceinline__ float output_alone(const AttnArgs& a, int head, bool corrected, int gg, int c) {
  const PoolDesc& pd = a.pd;
  const Geom& g = a.g;
  const float sl2 = 0.08838834764831845f * 1.4426950408889634f;
  const int k = a.k, n_att = g.n_sink + k + g.n_win + (g.r > 0 ? 1 : 0);
  const int new_page = FUSED ? (g.L - 1) / PG : -1, new_tok = (g.L - 1) % PG;
  const uint16_t* const q = a.q + ((size_t)head * a.G + gg) * D;
  const bool pending = !FUSED && (a.use == 1 || (a.use == 2 && a.flags[head] != 0));
  float M = -__builtin_inff(), den = 0.0f, o = 0.0f;
#pragma unroll 1
  for (int p = 0; p < n_att; ++p) {
    const int i = p - g.n_sink;                           // position in the picked list
    int page, unit;
    const uint16_t* up = pd.pool;
    bool from_host = false;
    if (i >= 0 && i < k) {
      int slot = 0;
      if (FUSED && corrected) {
        unsigned long long w;
        int it = 0;
        while ((uint32_t)((w = ld_tag(a.tagged + (size_t)head * k + i)) >> 32) != a.pick_tag) {
          if (++it > MAX_POLLS) { a.status->lost = 1; return __builtin_nanf(""); }
          __builtin_amdgcn_s_sleep(2);
        }
        if constexpr (HOSTFUSED) tagged_unpick((uint32_t)w, page, slot, from_host);
        else page = (int)(uint32_t)w;
      } else {
        page = (pending ? a.new_ids : a.act_ids)[(size_t)head * k + i];
        if (pd.placement != 0) slot = (pending ? a.new_slots : a.act_slots)[(size_t)head * k + i];
      }
      if (page < 0) continue;
      unit = pd.placement == 0 ? page : pd.sel_base + slot;
    } else {
      page = i < 0 ? p : g.n_full - g.n_win + (i - k);
      unit = resident_unit(pd, page);
    }
    if (HOSTFUSED && from_host) up = a.host_pool + ((size_t)head * a.max_pages + page) * UNIT_ELEMS;
    else up += ((size_t)head * pd.units_per_head + unit) * UNIT_ELEMS;
    const bool has_new = FUSED && page == new_page;      // (its last token comes from the step's inputs)
    const int n_tok = has_new ? new_tok + 1 : page == g.n_full ? g.r : PG;
#pragma unroll 1
    for (int t = 0; t < n_tok; ++t) {
      const bool is_new = has_new && t == new_tok;
      float dot = 0.0f;
#pragma unroll 1
      for (int c8 = 0; c8 < D; c8 += 8) {
        const uint16_t* kp = is_new ? a.k_new + (size_t)head * D + c8 : up + k_elem_off(t, c8);
        float kf[8], qf[8];
        unpack8<DT>(*reinterpret_cast<const uint4*>(kp), kf);
        unpack8<DT>(*reinterpret_cast<const uint4*>(q + c8), qf);
#pragma unroll
        for (int e = 0; e < 8; ++e) dot = __builtin_fmaf(kf[e], qf[e], dot);
      }
      const float s = dot * sl2, v = Unpack<DT>::one(is_new ? a.v_new[(size_t)head * D + c] : up[v_elem_off(t, c)]);
      const float m_new = fmaxf(M, s), alpha = m_new == M ? 1.0f : fast_exp2(M - m_new), w = fast_exp2(s - m_new);
      den = den * alpha + w;
      o = o * alpha + w * v;
      M = m_new;
    }
  }
  if (HOSTFUSED && __hip_atomic_load(&a.status->lost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return __builtin_nanf("");
  return o / den;
}

// One block of NW wavefronts: every n_splits-th attend-list position of `head` from `split` on (nth_position, nth_of_wave).  Dealt
// like that, and not a run of positions to each block, every block of a corrected head has its share of what can be attended at
// once and of what has to wait for the ids; with runs those of the picked pages alone had nothing to do until the ids came and
// all the work after that.  Layer-steps where most heads are corrected, runs against this: 8 heads of 65
// pages 10.9 and 10.1 us, 4 heads (G = 7) 10.7 and 10.2, 48 22.7 and 21.1, 112 40.7 and 36.8, 96 of 129 pages 47.1 and 43.3;
// where few are, the same to 1 % less.  With the KV in a host pool the link decides, and blocks have runs: the corrected heads' missing
// pages are then fetched by as few waves at once as it takes to fill it (8 heads x 32 missing pages, 1286 us and, in turn, 1292 with
// the load ahead of it).  `lds`: attn_lds_floats(NW, G) floats, 16-byte aligned.
// FUSED: in a launch with the step roles; HOSTFUSED: that, with the KV in a host pool (compile-time choices: what they
// add to the page loop would cost the other launches registers).  PAST: pages are read past the caches (STREAM_PAGES; as a branch
// around the loads it costs short launches 2 to 3 %).
// Returns what it waited for in vain and left to attn_finish.
struct AttnLeft {
  bool ids;                  // the head's picked ids (the same in every thread of the block); before that, the block makes them
  bool split;                // ... and so, of its own split, nothing is done
  bool corrected;            // the head's picked ids are this launch's
  uint32_t outputs;          // bit t: the thread's t-th output
  __device__ __forceinline__ bool any() const { return ids || __ballot(outputs != 0) != 0; }
};
template <int DT, int NW, bool FUSED, bool HOSTFUSED, bool PAST>
__device__ __forceinline__ AttnLeft attn_block(const AttnArgs& a, int split, int head, float* lds) {
  typedef typename Mma<DT>::vec vec;
  static_assert(!FUSED || NW >= MAX_G, "the correction test takes a wave per query head");
  const PoolDesc& pd = a.pd;
  const Geom& g = a.g;
  const int G = a.G, k = a.k;
#define FKV_ASTAMP(i) do { if (a.tstamp && head == 0 && thread_id(wave) == 0) a.tstamp[i] = wall_clock64(); } while (0)
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (split == 0) FKV_ASTAMP(16);
  const int gq = lane & 15, rb = lane >> 4;
  float* sm_o = lds;                                    // [NW][G][D + 4]
  float* sm_ml = lds + NW * G * (D + 4);                // [NW][16][2]
  uint32_t* sm_q = reinterpret_cast<uint32_t*>(sm_ml + NW * 32);        // [G][D / 2 + 4] pairs
  __shared__ double s_cos[MAX_G];
  __shared__ float s_near[MAX_G];
  __shared__ int s_no_ids;

  // the group's queries, for the correction test and (by way of LDS: registers are what this block is short of) as the
  // Q^T operand
  const uint16_t* qg = a.q + (size_t)head * G * D;
  uint32_t cq[MAX_G / NW + 1], cp = 0;
#pragma unroll
  for (int u = 0; u * NW < MAX_G; ++u)
    if (wave + u * NW < G) cq[u] = *reinterpret_cast<const uint32_t*>(qg + (wave + u * NW) * D + lane * 2);
  if (FUSED && a.have_prev && wave < G) cp = *reinterpret_cast<const uint32_t*>(a.q_prev + (size_t)head * G * D + wave * D + lane * 2);
  // ---- what the wave attends: lane l looks up its (l)-th position, one load for all of them ----
  const int n_att = g.n_sink + k + g.n_win + (g.r > 0 ? 1 : 0);
  const int pk_lo = g.n_sink, pk_hi = g.n_sink + k;
  auto position = [&](int ln) {                         // lane ln's (a wave has at most 64: attn_pages_per_block)
    if (HOSTFUSED) {
      const int nth = wave + ln * NW;
      return nth < a.pps ? split * a.pps + nth : n_att;
    }
    return nth_position(split + nth_of_wave(wave, ln, NW) * a.n_splits, n_att);
  };
  const int p = position(lane);
  const bool picked = p >= pk_lo && p < pk_hi;
  int page_l, unit_l;
  page_l = unit_l = -1;
  int id_l = -1, slot_l = 0;                            // FUSED: of the picked ones, waited for further down
  if (p < n_att) {
    if (picked) {
      const size_t at = (size_t)head * k + (p - pk_lo);
      if (FUSED) {
        id_l = a.act_ids[at];
        if (pd.placement != 0) slot_l = a.act_slots[at];
      } else {
        // by flag: both lists and the flag in one trip, not the list that the flag says after it
        const int32_t* const ids0 = a.use == 1 ? a.new_ids : a.act_ids;
        const int32_t* const ids1 = a.use == 0 ? a.act_ids : a.new_ids;
        const int id0 = ids0[at], id1 = ids1[at];
        int slot0 = 0, slot1 = 0;
        if (pd.placement != 0) {
          slot0 = (a.use == 1 ? a.new_slots : a.act_slots)[at];
          slot1 = (a.use == 0 ? a.act_slots : a.new_slots)[at];
        }
        const bool second = a.use == 2 && a.flags[head] != 0;
        page_l = second ? id1 : id0;
        if (page_l >= 0) unit_l = pd.placement == 0 ? page_l : pd.sel_base + (second ? slot1 : slot0);
      }
    } else {
      page_l = p < pk_lo ? p : g.n_full - g.n_win + (p - pk_hi);
      unit_l = resident_unit(pd, page_l);
    }
  }
  // The token appended at this step: in a fused launch its K/V may not be in the pool yet.  The wave that owns its page
  // takes it from the step's inputs -- it starts from that token instead of from nothing -- and attends the page without it.
  const int new_page = FUSED ? (g.L - 1) / PG : -1, new_tok = (g.L - 1) % PG;
  const bool owns_new = FUSED && __ballot(page_l == new_page && !picked) != 0;
  u32x4 kn[4];
  uint2 vn[8];
  auto k_part = [&](int s) { return *reinterpret_cast<const u32x4*>(a.k_new + (size_t)head * D + (s * 4 + rb) * 8); };
  auto v_part = [&](int cb) { return *reinterpret_cast<const uint2*>(a.v_new + (size_t)head * D + cb * 16 + rb * 4); };
  // requested as early as the queries: after the test, they were what the whole head waited for (8 heads of 65 pages, the open page's wave
  // done 4.7 us after its block began, the others 3.9; so, 3.9).  A host pool's kernels have no registers for that.
  if (FUSED && !HOSTFUSED && owns_new) {
#pragma unroll
    for (int s = 0; s < 4; ++s) kn[s] = k_part(s);
#pragma unroll
    for (int cb = 0; cb < 8; ++cb) vn[cb] = v_part(cb);
  }
  if (FUSED && new_tok == 0 && page_l == new_page) unit_l = -1;

  int number = 0;                                       // (waited for where the tag is needed)
  if (!FUSED && a.no.dev) number = *a.no.dev;

  const uint16_t* head_pool = pd.pool + (size_t)head * pd.units_per_head * UNIT_ELEMS;
  const float sl2 = 0.08838834764831845f * 1.4426950408889634f;   // 1/sqrt(d) * log2(e)
  float m_run = -__builtin_inff(), l_run = 0.0f;
  bool fresh = true;                                    // nothing is summed up yet
  f32x4 acc[8];
  u32x4 kw[8], vw[8];
  uint32_t miss_l = 0;                                  // HOSTFUSED: the lane's page has to come from the host pool

  const uint32_t lane16 = (uint32_t)lane * 16;
  auto source = [&](int i) -> const char* {             // where position i's bytes are
    const int u = __builtin_amdgcn_readlane(unit_l, i);
    const uint16_t* p = head_pool + (size_t)u * UNIT_ELEMS;
    if constexpr (HOSTFUSED) {
      if (__builtin_amdgcn_readlane((int)miss_l, i))
        p = a.host_pool + ((size_t)head * a.max_pages + __builtin_amdgcn_readlane(page_l, i)) * UNIT_ELEMS;
    }
    return reinterpret_cast<const char*>(p);
  };
  // 4 KiB of a page from a scalar base (the opaque copies keep one base register pair per group and the lanes' offset in one)
  typedef const __attribute__((address_space(1))) char* gptr;
  auto load4 = [&](u32x4* w, const char* from) {
    const unsigned long long u = (unsigned long long)from;
    gptr base = (gptr)(((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(u >> 32)) << 32) |
                       (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u));
    asm volatile("" : "+s"(base));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const auto p = (const __attribute__((address_space(1))) u32x4*)(base + j * 1024 + lane16);
      w[j] = PAST ? __builtin_nontemporal_load(p) : *p;
    }
  };
  auto load_k = [&](const char* up) { load4(kw, up); load4(kw + 4, up + 4096); };
  auto load_v = [&](const char* up) { load4(vw, up + 8192); load4(vw + 4, up + 12288); };
  // Q^T operand of k-step s: lane (g, kb) holds channels (s*4+kb)*8 .. +8 of head g (the idle columns repeat head 0)
  const uint32_t* const q_op = sm_q + (gq < G ? gq : 0) * (D / 2 + 4) + rb * 4;
  auto q_of = [&](int s) { return *reinterpret_cast<const vec*>(q_op + s * 16); };
  // One page: position i's, whose loads are under way.  Position `next` (-1: none) is requested on the way, its keys once
  // the products with this page's are made, its values once those are: the registers are free by then.
  auto attend_page = [&](int i, int next) {
    const char* const up_next = source(next >= 0 ? next : 0);
    const int page = __builtin_amdgcn_readlane(FUSED && !HOSTFUSED ? unit_l : page_l, i);   // (KV in HBM: the same)
    const int n_valid = FUSED ? (page == new_page ? new_tok : PG) : (page == g.n_full ? g.r : PG);
    if constexpr (HOSTFUSED) {
      if (__builtin_amdgcn_readlane((int)miss_l, i)) {
        // the page came from the host pool: it goes into its page-cache slot as it is (recall, Sec. 3.3: a corrected
        // head's pages are fetched before it attends; here the wave that attends over the page is the one that fetches it)
        u32x4* dp = reinterpret_cast<u32x4*>(pd.pool + ((size_t)head * pd.units_per_head + __builtin_amdgcn_readlane(unit_l, i)) * UNIT_ELEMS) + lane;
#pragma unroll
        for (int j = 0; j < 8; ++j) dp[j * 64] = kw[j];
#pragma unroll
        for (int j = 0; j < 8; ++j) dp[(8 + j) * 64] = vw[j];
      }
    }
    f32x4 st[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    auto products = [&](int s, vec qs) {
#pragma unroll
      for (int mb = 0; mb < 2; ++mb) st[mb] = Mma<DT>::mma(__builtin_bit_cast(vec, kw[s * 2 + mb]), qs, st[mb]);
      if (s < 3) __builtin_amdgcn_sched_barrier(0);     // (not all of the operand at once: registers)
    };
    if constexpr (HOSTFUSED) {
#pragma unroll
      for (int s = 0; s < 4; ++s) products(s, q_of(s));
    } else {                                            // (the operand a step ahead, for which a host pool's kernels have no registers)
      vec qs = q_of(0);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const vec q1 = s < 3 ? q_of(s + 1) : qs;
        products(s, qs);
        qs = q1;
      }
    }
    if (next >= 0) load_k(up_next);
    // logits (base 2) of head gq for tokens mb*16 + rb*4 + i
    float sc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) sc[e] = st[e >> 2][e & 3] * sl2;
    if (n_valid < PG) {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (rb * 4 >= n_valid - ((e >> 2) * 16 + (e & 3))) sc[e] = -__builtin_inff();
    }
    float mx = fmaxf(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])), fmaxf(fmaxf(sc[4], sc[5]), fmaxf(sc[6], sc[7])));
    mx = max_over_rows(mx);
    // The sums are kept relative to the running maximum itself: the tokens that set it, which weigh most, then have the
    // weight 1, which the split below represents exactly (a reference that lags behind, to save rescaling passes, costs
    // bf16 outputs a third of their precision).
    if (__ballot(mx > m_run)) {
      const float m_new = fmaxf(mx, m_run);
      const float alpha = m_new == m_run ? 1.0f : fast_exp2(m_run - m_new);
      l_run *= alpha;
      m_run = m_new;
      if (HOSTFUSED || !fresh) {                        // (the test takes a register that a host pool's kernels have not)
#pragma unroll
        for (int cb = 0; cb < 8; ++cb) acc[cb] *= alpha;
      }
    }
    fresh = false;
    float p[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) p[e] = fast_exp2(sc[e] - m_run);
    vec phi, plo;
    Mma<DT>::split(p, phi, plo);
    // the sum of the weights as they go into the products, so that what the split drops cancels in the quotient
    float l_lo = 0.0f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      l_run = Mma<DT>::add_pair(__builtin_bit_cast(u32x4, phi)[e], l_run);
      l_lo = Mma<DT>::add_pair(__builtin_bit_cast(u32x4, plo)[e], l_lo);
    }
    l_run += l_lo;
#pragma unroll
    for (int cb = 0; cb < 8; ++cb) {
      const vec va = __builtin_bit_cast(vec, vw[cb]);
      acc[cb] = Mma<DT>::mma(va, phi, acc[cb]);
      acc[cb] = Mma<DT>::mma(va, plo, acc[cb]);
    }
    if (next >= 0) load_v(up_next);
  };

  bool lost = false;
  bool two_phase = false;
  // The first page's loads.  In a layer-step a page that is not picked, if the wave has such: it is attended first whether the head
  // is corrected or not (no loads are made in vain), and need not wait for the ids.  Else a picked one, for the case that the head is
  // not corrected.  (us per layer-step, with the first page of the list after the ids and so: 56 heads of 33 pages, G = 5, 12.0 and
  // 11.4, most corrected 14.8 and 13.7; 8 heads of 65 8.8 and 8.6; 112 of 65, most corrected, 37.2 and 32.7.)
  const unsigned long long known = __ballot(unit_l >= 0);
  int i0 = known ? (int)__builtin_ctzll(known) : -1;
  const bool at_once = FUSED && a.at_once;
  if (at_once && i0 >= 0) load_k(source(i0));
  if (FUSED && picked) {
    page_l = id_l;
    if (page_l >= 0) unit_l = pd.placement == 0 ? page_l : pd.sel_base + slot_l;
  }
  const unsigned long long listed = FUSED ? __ballot(unit_l >= 0) : known;
  if (FUSED && i0 < 0 && listed) i0 = (int)__builtin_ctzll(listed);
  const char* const up0 = source(i0 >= 0 ? i0 : 0);
  if (!(at_once && known) && i0 >= 0) load_k(up0);
  if (FUSED && wave == 0) s_no_ids = 0;
#pragma unroll
  for (int u = 0; u * NW < MAX_G; ++u)
    if (wave + u * NW < G) sm_q[(wave + u * NW) * (D / 2 + 4) + lane] = cq[u];
  // the correction test again, so that this block does not have to wait for that role's result: in fp32 where that
  // decides it, else with the arithmetic of the step role
  if (FUSED && a.have_prev && wave < G) {
    const float c = near_cosine_of<DT>(cq[0], cp);
    if (lane == 63) s_near[wave] = c;
  }
#pragma unroll
  for (int cb = 0; cb < 8; ++cb) {
    acc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (!HOSTFUSED) asm volatile("" : "+v"(acc[cb]));      // (here, while loads are under way)
  }
  lds_barrier();
  if (FUSED) {
    int flag = a.have_prev ? __builtin_amdgcn_readfirstlane(near_flag(s_near, G, a.tau, a.corr_pool)) : 1;
    if (flag < 0) {
      if (wave < G) {
        const double c = cosine_of<DT>(cq[0], cp);
        if (lane == 63) s_cos[wave] = c;
      }
      lds_barrier();
      flag = __builtin_amdgcn_readfirstlane(pooled_flag(s_cos, G, a.tau, a.corr_pool));
    }
    two_phase = flag != 0;
  }
  if (HOSTFUSED && i0 >= 0) load_v(up0);
  if (FUSED && owns_new) {
    if (HOSTFUSED) {
#pragma unroll
      for (int cb = 0; cb < 8; ++cb) vn[cb] = v_part(cb);
    }
    f32x4 st = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4; ++s)                         // (the key in every row of the tile)
      st = Mma<DT>::mma(__builtin_bit_cast(vec, HOSTFUSED ? k_part(s) : kn[s]), q_of(s), st);
    m_run = st[0] * sl2;
    l_run = rb == 0 ? 1.0f : 0.0f;
    fresh = false;
#pragma unroll
    for (int cb = 0; cb < 8; ++cb)
      acc[cb] = f32x4{Unpack<DT>::lo(vn[cb].x), Unpack<DT>::hi(vn[cb].x), Unpack<DT>::lo(vn[cb].y), Unpack<DT>::hi(vn[cb].y)};
  }
  if (!HOSTFUSED && i0 >= 0) load_v(up0);
  // A corrected head of a fused launch attends with this step's selection, which other blocks of
  // the same launch are still making.  Only the k picked positions of the attend list depend on it:
  // the wave first attends its sink, window and open-page positions (phase 0), then waits for the selection and
  // attends its picked positions (phase 1).  Everything else runs as one phase.
  unsigned long long todo = two_phase ? __ballot(!picked && unit_l >= 0) : listed;
  bool loaded = !FUSED ? todo != 0 : i0 >= 0 && (todo >> i0 & 1ull) != 0;
  for (int phase = 0;; ++phase) {
    if (todo) {
      int i = FUSED && loaded ? i0 : (int)__builtin_ctzll(todo);
      if (!loaded) {
        const char* up = source(i);
        load_k(up);
        load_v(up);
      }
      do {
        todo &= FUSED ? ~(1ull << i) : todo - 1;
        const int next = todo ? (int)__builtin_ctzll(todo) : -1;
        attend_page(i, next);
        i = next;
      } while (i >= 0);
    }
    if (!two_phase || phase == 1) break;
    todo = __ballot(picked);
    loaded = false;
    if (todo == 0) break;
    // Wait for this step's ids of the positions: the selection writes every picked id as one tagged 64-bit word.
    // The blocks that make it have lower block indices than any attention block, so that as a rule they are running or
    // done.
    const int at = position(thread_id(wave) & 63) - pk_lo;
    const unsigned long long* word = a.tagged + (size_t)head * k + (picked ? at : 0);
    unsigned long long w = 0;
    for (int it = 0;; ++it) {
      w = ld_tag(word);
      if (__ballot(picked && (uint32_t)(w >> 32) != a.pick_tag) == 0) break;
      if (it > PATIENCE) { lost = true; break; }
      __builtin_amdgcn_s_sleep(2);
    }
    if (lost || a.impatient & WAIT_IDS) {
      if (lane == 0) s_no_ids = 1;
      break;
    }
    if (picked) {
      if constexpr (HOSTFUSED) {
        // the slot comes with the id (the slot table in memory is being written by another block of this launch);
        // a page the cache does not hold is read from the host pool
        int slot;
        bool miss;
        tagged_unpick((uint32_t)w, page_l, slot, miss);
        unit_l = slot >= 0 ? pd.sel_base + slot : -1;
        miss_l = miss ? 1u : 0u;
      } else {
        page_l = (int)(uint32_t)w;
        unit_l = page_l;
      }
    }
    todo = __ballot(picked && unit_l >= 0);
  }
  if constexpr (HOSTFUSED) {
    // With the KV in a host pool the wave that gives up also leaves the page-cache slot it was to fill unfilled, while
    // the recall plan lists the page as cached: the layer's state cannot be trusted from then on.  Every later step of
    // the layer therefore stays marked -- NaN outputs -- for as long as the flag is up (fkv_health takes it down).
    if (__hip_atomic_load(&a.status->lost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) l_run = __builtin_nanf("");
  }
  if (split == 0) FKV_ASTAMP(17);

  // ---- combine the waves: one barrier ----
  l_run = sum_over_rows(l_run);                         // per-wave totals of l over the 4 row blocks
  const int tid = thread_id(wave);
  if ((tid & 15) < G) {
    float* o = sm_o + ((size_t)wave * G + (tid & 15)) * (D + 4) + (tid >> 4 & 3) * 4;
#pragma unroll
    for (int cb = 0; cb < 8; ++cb) *reinterpret_cast<f32x4*>(o + cb * 16) = acc[cb];
    if ((tid & 63) < 16) *reinterpret_cast<float2*>(sm_ml + (wave * 16 + (tid & 15)) * 2) = make_float2(m_run, l_run);
  }
  const uint32_t tag = FUSED ? a.tag : a.no.dev ? device_tag((uint32_t)__builtin_amdgcn_readfirstlane(number)) : a.no.tag;
  lds_barrier();
  // ---- log-sum-exp merge of the head's splits, shared by its blocks ----
  // Block `split` finishes the split-th `share` of the head's G x D outputs: its threads keep their sums of that part, hand
  // the others to the blocks that finish them, and fold the other blocks' sums of their own part in as they arrive.  One
  // trip, and no block reads more than an n_splits-th of the partials (one block merging alone: 6 us of a 20 us launch at
  // 16 splits of G = 8).  A head's blocks, dealt as deal_block says, wait for each other only.
  const int n_splits = a.n_splits, items = G * D;
  const int own_lo = split * a.share, own_hi = min(items, own_lo + a.share);
  unsigned long long* const po = a.part + (size_t)head * a.max_splits * items;
  unsigned long long* const pml = a.part_ml + (size_t)head * a.max_splits * G * 2;
  constexpr int patience = HOSTFUSED ? PATIENCE_HOST : PATIENCE;
  const uint32_t want = tag + (a.impatient & WAIT_SPLITS ? 2u : 0u);      // (or a tag that no word has yet)
  constexpr int IT = (MAX_G * D + NW * 64 - 1) / (NW * 64);
  float o[IT], den[IT], M[IT];
  uint32_t left = 0;                                    // bit t: item t's output is left to be made alone
  const bool no_ids = FUSED && two_phase && __builtin_amdgcn_readfirstlane(s_no_ids) != 0;
  if (!no_ids) {
    // A wave's 64 outputs are of one query head, so what is the same for all of them -- the weights of the block's waves, and
    // then of the head's splits -- is worked out by a lane each and handed round as scalars.  (With every thread working them out
    // for itself, two thirds of its loads and nearly all of its exponentials were for that: layer-step of 4 KV heads, G = 7, all
    // of them corrected, 12.9 -> 11.8 us; 56 heads, G = 5, 13.3 -> 12.4.)
    const int ln = tid & 63;
#pragma unroll
    for (int t = 0; t < IT; ++t) {
      if (wave * 64 + t * NW * 64 >= items) break;
      const int idx = tid + t * NW * 64, gg = (wave * 64 + t * NW * 64) / D, c = idx % D;
      const float2 ml = *reinterpret_cast<const float2*>(sm_ml + ((ln & (NW - 1)) * 16 + gg) * 2);      // of wave lane % NW
      uint32_t top = __float_as_uint(ml.x);
      top = OpMaxF32()(top, dpp_u32<DPP_XOR1>(top));
      top = OpMaxF32()(top, dpp_u32<DPP_XOR2>(top));
      if (NW == 8) top = OpMaxF32()(top, dpp_u32<DPP_HALF_MIRROR>(top));
      const float Mt = __uint_as_float(top);
      // a wave that saw no page has m = -inf and zero sums (or a poisoned one)
      const bool saw = ml.x != -__builtin_inff();
      const float wgt = saw ? fast_exp2(ml.x - Mt) : 0.0f;
      uint32_t sum = __float_as_uint(saw ? ml.y * wgt : ml.y);
      sum = OpAddF32()(sum, dpp_u32<DPP_XOR1>(sum));
      sum = OpAddF32()(sum, dpp_u32<DPP_XOR2>(sum));
      if (NW == 8) sum = OpAddF32()(sum, dpp_u32<DPP_HALF_MIRROR>(sum));
      const float dt = __uint_as_float(sum);
      float ot = 0.0f;
#pragma unroll
      for (int w = 0; w < NW; ++w)
        ot += sm_o[((size_t)w * G + gg) * (D + 4) + c] * __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(wgt), w));
      o[t] = ot; den[t] = dt; M[t] = Mt;
      if (n_splits > 1) {
        if (idx < own_lo || idx >= own_hi) st_tag(po + (size_t)split * items + idx, __float_as_uint(ot), tag, a.home);
        if (c == 0) {
          st_tag(pml + (split * G + gg) * 2, __float_as_uint(Mt), tag, a.home);
          st_tag(pml + (split * G + gg) * 2 + 1, __float_as_uint(dt), tag, a.home);
        }
      }
    }
    if (split == 0) FKV_ASTAMP(18);
#pragma unroll
    for (int t = 0; t < IT; ++t) {
      const int first = wave * 64 + t * NW * 64;          // the wave's outputs
      if (first >= own_hi || first + 64 <= own_lo) continue;
      const int idx = tid + t * NW * 64, gg = first / D;
      const bool mine = idx >= own_lo && idx < own_hi;
      const unsigned long long* const po_i = po + min(max(idx, own_lo), own_hi - 1);
      // the others' splits, numbered from 0 (the block's own is left out), 16 at a time: lane s reads the maximum of the
      // s-th, lane 32 + s its sum of weights, in the same trip as the outputs
      for (int s0 = 0; s0 < n_splits - 1; s0 += 16) {
        const int n = min(16, n_splits - 1 - s0);
        auto nth = [&](int i) { const int sp = s0 + min(i, n - 1); return sp + (sp >= split ? 1 : 0); };
        const unsigned long long* const pml_i = pml + (nth(ln & 15) * G + gg) * 2 + (ln >> 5);
        unsigned long long wml, wo[16];
        int it = 0;
        for (;;) {
          wml = ld_tag(pml_i);
#pragma unroll
          for (int u = 0; u < 8; ++u) wo[u] = ld_tag(po_i + (size_t)nth(u) * items);
          if (n > 8) {
#pragma unroll
            for (int u = 8; u < 16; ++u) wo[u] = ld_tag(po_i + (size_t)nth(u) * items);
          }
          bool there = (uint32_t)(wml >> 32) == want;
#pragma unroll
          for (int u = 0; u < 8; ++u) there = there & ((uint32_t)(wo[u] >> 32) == want);
          if (n > 8) {
#pragma unroll
            for (int u = 8; u < 16; ++u) there = there & ((uint32_t)(wo[u] >> 32) == want);
          }
          if (__ballot(!there) == 0 || ++it > patience) break;
          __builtin_amdgcn_s_sleep(1);
        }
        if (it > patience) { left |= mine ? 1u << t : 0u; break; }
        const auto halves = __builtin_amdgcn_permlane32_swap((uint32_t)wml, (uint32_t)wml, false, false);
        const float m = (ln & 15) < n ? __uint_as_float(halves[0]) : -__builtin_inff(), l = __uint_as_float(halves[1]);
        const float Mc = fmaxf(M[t], __uint_as_float(class_reduce<1>(__float_as_uint(m), OpMaxF32())));
        const float wgt = m == -__builtin_inff() ? 0.0f : fast_exp2(m - Mc);
        const float part = ln < n ? (m == -__builtin_inff() ? l : wgt * l) : 0.0f;
        const float add = __uint_as_float(class_reduce<1>(__float_as_uint(part), OpAddF32()));
        const bool none = M[t] == -__builtin_inff();
        const float resc = none ? 0.0f : fast_exp2(M[t] - Mc);
        den[t] = (none ? den[t] : den[t] * resc) + add;
        o[t] *= resc;
        M[t] = Mc;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          if (u >= n) break;
          o[t] += __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(wgt), u)) * __uint_as_float((uint32_t)wo[u]);
        }
      }
      if (mine && !(left >> t & 1u)) a.out[(size_t)head * items + idx] = o[t] / den[t];
    }
  }
  if (split == 0) FKV_ASTAMP(21);
  bool need_ids = no_ids;
  if (FUSED && two_phase && n_splits > 1) {             // (outputs that were left need ids that may not be there)
    if (left) s_no_ids = 1;
    lds_barrier();
    need_ids = __builtin_amdgcn_readfirstlane(s_no_ids) != 0;
  }
  return AttnLeft{need_ids, no_ids, two_phase, no_ids ? ~0u : left};
#undef FKV_ASTAMP
}

// What a block left, without waiting for anyone.  If left.ids, the block has made the head's selection by now, into memory
// and into the tagged words.
template <int DT, int NW, bool FUSED, bool HOSTFUSED>
__device__ __forceinline__ void attn_finish(const AttnArgs& a, int split, int head, AttnLeft left) {
  if ((threadIdx.x & 63) == 0) atomicAdd(&a.status->by_itself, 1);
  if (FUSED && left.ids) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // (each wave's words are where the others read them)
    lds_barrier();
  }
  if (HOSTFUSED && left.split) {                        // the recall of the block's missing pages, as in attend_page
    const int lo = a.g.n_sink, hi = min(lo + a.k, (split + 1) * a.pps);
#pragma unroll 1
    for (int p = max(split * a.pps, lo); p < hi; ++p) {
      const unsigned long long w = ld_tag(a.tagged + (size_t)head * a.k + p - lo);
      int page, slot;
      bool miss;
      tagged_unpick((uint32_t)w, page, slot, miss);
      if ((uint32_t)(w >> 32) != a.pick_tag || page < 0 || !miss) continue;
      const u32x4* from = reinterpret_cast<const u32x4*>(a.host_pool + ((size_t)head * a.max_pages + page) * UNIT_ELEMS);
      u32x4* to = reinterpret_cast<u32x4*>(a.pd.pool + ((size_t)head * a.pd.units_per_head + a.pd.sel_base + slot) * UNIT_ELEMS);
      for (int i = threadIdx.x; i < UNIT_BYTES / 16; i += NW * 64) to[i] = from[i];
    }
  }
  constexpr int IT = (MAX_G * D + NW * 64 - 1) / (NW * 64);
#pragma unroll 1
  for (int t = 0; t < IT; ++t) {
    const int idx = threadIdx.x + t * NW * 64;
    if (idx < split * a.share || idx >= min(a.G * D, (split + 1) * a.share) || !(left.outputs >> t & 1u)) continue;
    a.out[(size_t)head * a.G * D + idx] = output_alone<DT, FUSED, HOSTFUSED>(a, head, left.corrected, idx / D, idx % D);
  }
}

}  // namespace fkv
