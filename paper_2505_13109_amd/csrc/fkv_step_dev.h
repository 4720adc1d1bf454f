// Device code of the "step" roles: token append + incremental summaries, correction test, page weights,
// and softmax -> group-mean pooling -> top-k.
// One launch; blocks take roles by index, because the three jobs do not depend on each
// other inside a step: the page being appended to is never a candidate, and a page that
// becomes a candidate had its summary completed at least a window ago.
//
// The selected page ids must be reproducible bit for bit, so the arithmetic that
// decides them is restricted to IEEE fp32/fp64 operations in a fixed order
// (this file is compiled with -ffp-contract=off; FMAs are written explicitly
// and only where the product is exact, so fusing cannot change the result):
//   weight:  128 exact products summed as 16 chunks of 8 consecutive channels,
//            left to right, then an adjacent-pair tree over the 16 chunk sums
//            (the xor-1,2,4,8 butterfly of a 16-lane group), times fl32(1/sqrt(128));
//   softmax: x = P - max; t = x * fl32(log2 e); n = rint(t); f = t - n;
//            degree-6 Horner in f with separate multiply and add; ldexp(., n);
//            0 below t < -64; E = rint(e * 2^31) as integer; Z = integer sum of E;
//   pooling: fl32( (sum_g fp64(E_g) / fp64(Z_g), g ascending) / fp64(G) ); the quotients are the
//            correctly rounded ones, computed from a reciprocal of Z_g with fused multiply-add
//            corrections (see div_rn);
//            (alternatives, App. B.2: fl32(max_g E_g / Z_g); the fp32 sum of the weights in head
//            order divided by G, or their maximum; the weight of the group's mean or maximum query)
//   top-k:   on the order-preserving image of the fp32 bit pattern, ties to the lower page id.
#pragma once
#include "fkv_device.h"
#include "fkv_plan_dev.h"
#include "fkv_attn_dev.h"

#pragma clang fp contract(off)

namespace fkv {

#define FKV_STAMP(a, head, i) do { if ((a).tstamp && (head) == 0 && threadIdx.x == 0) (a).tstamp[i] = wall_clock64(); } while (0)

#ifndef FKV_STEP_THREADS
#define FKV_STEP_THREADS 512
#endif
#ifndef FKV_SCORE_PASSES
#define FKV_SCORE_PASSES 4
#endif
constexpr int STEP_THREADS = FKV_STEP_THREADS;         // >= 256 (the radix histograms have 256 bins)
constexpr int STEP_WAVES = STEP_THREADS / 64;
constexpr int SCORE_PASSES = FKV_SCORE_PASSES;         // most passes a scoring block can make (StepArgs::passes <= this)
constexpr int PAGES_PER_PASS = STEP_WAVES * 4;         // a wave scores 4 pages per pass
constexpr int MAX_SLICES = 16;                         // most blocks that share one head's selection

template <int U> struct UnrollBy { static constexpr int value = U; };

struct StepArgs {
  int roles;                 // ROLE_* bits
  int heads, k, max_pages;
  Geom g;                    // geometry with the appended token counted
  // append
  PoolDesc pd;
  uint16_t* summ;
  const uint16_t* k_new;
  const uint16_t* v_new;
  // correction test
  const uint16_t* q;
  const uint16_t* q_prev;
  uint16_t* q_stage;
  int have_prev;
  float tau;
  int corr_pool;             // FKV_CORR_*
  uint8_t* flags;
  uint8_t* flags_user;
  double* cosine;
  // selection
  int sel_pool;              // FKV_POOL_*
  unsigned long long* P;     // page weights [query heads][max_pages], tagged; in a launch that only scores and one that
                             // only selects: plain fp32 in the same order (in memory of their own: the bits of a plain
                             // weight could be some launch's tag)
  float* score;
  int32_t* ids;
  int32_t* ids_user;
  int chunks;                // scoring blocks of a KV head
  int other_rows;            // scan: rows of its grid for the other roles
  int passes;                // passes a scoring block makes (1 .. SCORE_PASSES)
  int slices, slices_log2;   // selecting blocks of a KV head (1 .. MAX_SLICES, a power of two)
  int slice;                 // candidates of each (the last may have fewer)
  unsigned long long* exch;  // [heads][MAX_SLICES][3 * MAX_G] tagged: what a head's selecting blocks tell each other
  unsigned long long* keyx;  // [heads][max_pages] tagged: the candidates' keys, for the head's last selecting block
  LaunchNo no;               // of this launch
  uint32_t impatient;        // WAIT_* bits: waits that run out at once (tests)
  long long* tstamp;         // debug: 100 MHz timestamps of head 0's phases (may be null)
  unsigned long long* tagged; // if not null: [heads][k], every picked id once more as a tagged word: a block of
                              // this launch that waits for the selection polls the word it needs
  // KV in a host pool: the selecting block also makes the head's recall plan (fkv_plan_dev.h).  plan_new_slots null:
  // not here.  The tagged words then carry, instead of the bare id, what a waiting attention wave needs to fetch the
  // page: tagged_pick() of (page id, slot, miss).
  const int32_t* plan_act_ids;
  const int32_t* plan_act_slots;
  int32_t* plan_new_slots;
  int32_t* plan_miss;
  int plan_lds_off;           // where the plan's LDS starts, in 32-bit words of the block's dynamic LDS
};


// ---------------------------------------------------------------------------------
// role: append one token (Sec. 3.2 summaries; Sec. 4.2 paged layout).  128 active threads.
// ---------------------------------------------------------------------------------
template <int DT>
__device__ __forceinline__ void append_role(const StepArgs& a, int head) {
  const int c = threadIdx.x;
  if (c >= D) return;   // 128 of the block's threads
  const int pos = a.g.L - 1, page = pos / PG, t = pos % PG;
  const uint16_t kb = a.k_new[(size_t)head * D + c];
  const uint16_t vb = a.v_new[(size_t)head * D + c];
  uint16_t* pmax = a.summ + summ_idx(0, head, 0, 0, a.max_pages, page) + c;
  uint16_t* pmin = a.summ + summ_idx(0, head, 0, 1, a.max_pages, page) + c;
  uint16_t omax = kb, omin = kb;
  if (t != 0) { omax = *pmax; omin = *pmin; }
  uint16_t* unit = a.pd.pool + ((size_t)head * a.pd.units_per_head + resident_unit(a.pd, page)) * UNIT_ELEMS;
  unit[k_elem_off(t, c)] = kb;
  unit[v_elem_off(t, c)] = vb;
  const float kf = Unpack<DT>::one(kb);
  if (t == 0 || kf > Unpack<DT>::one(omax)) *pmax = kb;
  if (t == 0 || kf < Unpack<DT>::one(omin)) *pmin = kb;
}

// ---------------------------------------------------------------------------------
// role: correction test (Sec. 3.1, 3.3).  One wave per query head, fp64.
// ---------------------------------------------------------------------------------
template <int DT, int G, int WAVES = STEP_WAVES>
__device__ __forceinline__ void corr_role(const StepArgs& a, int head) {
  __shared__ double cg[MAX_G];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int gg = wave; gg < G; gg += WAVES) {
    const size_t off = ((size_t)head * G + gg) * D + lane * 2;
    const uint32_t qw = *reinterpret_cast<const uint32_t*>(a.q + off);
    double cosv = 0.0;
    if (a.have_prev) cosv = cosine_of<DT>(qw, *reinterpret_cast<const uint32_t*>(a.q_prev + off));
    *reinterpret_cast<uint32_t*>(a.q_stage + off) = qw;
    if (lane == 63) {
      cg[gg] = cosv;
      a.cosine[head * G + gg] = cosv;
    }
  }
  lds_barrier();
  if (threadIdx.x == 0) {
    uint8_t f = 1;
    if (a.have_prev) f = (uint8_t)pooled_flag(cg, G, a.tau, a.corr_pool);
    a.flags[head] = f;
    if (a.flags_user) a.flags_user[head] = f;
  }
}

// Scores can be negative in the variants that pool the weights themselves: map the fp32 bit
// pattern to an unsigned key with the same order (-0 counts as +0), and back.
__device__ __forceinline__ uint32_t score_key(float sc) {
  const uint32_t u = __float_as_uint(sc + 0.0f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_score(uint32_t key) {
  return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
}

// ---------------------------------------------------------------------------------
// role: page weights P^h_j from the min-max summaries (Sec. 3.2).
// A 16-lane group owns one page: lane c8 holds channels 8*c8 .. 8*c8+7 of kmax and
// kmin (one 16-byte load each, 1 KiB contiguous per wave and array), so a wave
// scores 4 pages per pass.  All loads of a block's passes are issued before the first use.
// Weights that blocks of the same launch wait for (TAGGED) are collected in LDS and go out as whole runs per query head;
// for a later launch each pass stores its own, which leaves the waves of a bandwidth-bound scan independent of each other
// (28.2 us against 30.3 us through LDS for 256 heads x 992 pages).
// ---------------------------------------------------------------------------------
template <int DT, int G, bool QMODE, bool TAGGED, int WAVES>
__device__ __forceinline__ void score_pages(const StepArgs& a, int head, int chunk) {
  constexpr int PASS = WAVES * 4;                         // pages per pass
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int grp = lane >> 4, c8 = lane & 15;
  const int passes = TAGGED ? a.passes : SCORE_PASSES;    // (the scan always makes as many as there are)
  const int n = a.g.n_cand, j0 = chunk * PASS * passes + wave * 4 + grp;
  uint4 wmax[SCORE_PASSES], wmin[SCORE_PASSES];
  const uint16_t* sm = a.summ + summ_idx(0, head, 0, 0, a.max_pages, a.g.cand_lo) + c8 * 8;
  const size_t to_min = (size_t)a.max_pages * D;
#pragma unroll
  for (int ps = 0; ps < SCORE_PASSES; ++ps) {
    if (ps < passes) {
      const int j = min(j0 + ps * PASS, n - 1);
      wmax[ps] = *reinterpret_cast<const uint4*>(sm + (size_t)j * D);
      wmin[ps] = *reinterpret_cast<const uint4*>(sm + (size_t)j * D + to_min);
    }
  }
  const uint32_t tag = TAGGED ? launch_tag(a.no) : 0u;
  uint4 wq[G];
#pragma unroll
  for (int gg = 0; gg < G; ++gg) wq[gg] = *reinterpret_cast<const uint4*>(a.q + ((size_t)head * G + gg) * D + c8 * 8);
  // Variants that pool the QUERY over the group (App. B.2, MeanQ / MaxQ): one pooled query per KV
  // head takes the place of head 0 of the group, and only its weight is written.
  constexpr int NG = QMODE ? 1 : G;                       // weights this launch writes per page
  float pooled[8];
  if (QMODE) {
#pragma unroll
    for (int gg = 0; gg < G; ++gg) {
      float f[8];
      unpack8<DT>(wq[gg], f);
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        pooled[c] = gg == 0 ? f[c] : a.sel_pool == 4 ? pooled[c] + f[c] : fmaxf(pooled[c], f[c]);
        asm volatile("" : "+v"(pooled[c]));               // (one head after the other: registers)
      }
    }
    // fp32 quotient by way of fp64: correctly rounded (53 >= 2 * 24 + 2 bits)
    if (a.sel_pool == 4) {
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        pooled[c] = (float)((double)pooled[c] / (double)G);
        asm volatile("" : "+v"(pooled[c]));
      }
    }
  }
  const float scale = 0x1.6a09e6p-4f;   // fl32(1/sqrt(128))
  __shared__ float s_w[NG][TAGGED ? PASS * SCORE_PASSES : 1];
  // The weights of N passes' pages.  A channel contributes q_c * (q_c >= 0 ? kmax_c : kmin_c): the choice is made on the
  // packed 16-bit values, by the signs of a query's channel pair as a bit mask (one instruction for two channels, and the
  // mask serves N passes; as comparisons, 8 G lane masks would have to live in scalar registers, which from G = 5 on there
  // are not enough of: a layer-step of 8 KV heads x 2016 candidates, G = 8, 21.7 us with those, 18.4 so).
  auto score = [&](auto nc) {
    constexpr int N = decltype(nc)::value;
    float mine[N];                                        // the total of query head c8, for lanes c8 < NG
#pragma unroll
    for (int gg = 0; gg < NG; ++gg) {
      uint32_t q2[4] = {wq[gg].x, wq[gg].y, wq[gg].z, wq[gg].w};
      // (opaque here: else every head's unpacked channels and masks are made ahead of the variants and kept: registers)
#pragma unroll
      for (int h = 0; h < 4; ++h) asm volatile("" : "+v"(q2[h]));
      // chunk sum, left to right.  The product of two 16-bit floats is exact in fp32, so the fma rounds once, exactly
      // like "s + product"; a mean query is a full fp32 number, so there the product is rounded on its own first.
      float s[N];
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        typedef __attribute__((ext_vector_type(2))) short s16x2;
        uint32_t neg;
        if (QMODE) neg = (pooled[2 * h] >= 0.0f ? 0u : 0xffffu) | (pooled[2 * h + 1] >= 0.0f ? 0u : 0xffff0000u);
        else neg = __builtin_bit_cast(uint32_t, __builtin_bit_cast(s16x2, q2[h]) >> 15);
#pragma unroll
        for (int i = 0; i < N; ++i) {
          const uint32_t kx = h == 0 ? wmax[i].x : h == 1 ? wmax[i].y : h == 2 ? wmax[i].z : wmax[i].w;
          const uint32_t kn = h == 0 ? wmin[i].x : h == 1 ? wmin[i].y : h == 2 ? wmin[i].z : wmin[i].w;
          uint32_t k2;                                    // (the compiler takes the expression apart)
          asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(k2) : "v"(neg), "v"(kn), "v"(kx));
          if (QMODE) {
            const float pr = pooled[2 * h] * Unpack<DT>::lo(k2);
            s[i] = h == 0 ? pr : s[i] + pr;
            s[i] = s[i] + pooled[2 * h + 1] * Unpack<DT>::hi(k2);
          } else {
            s[i] = __builtin_fmaf(Unpack<DT>::lo(q2[h]), Unpack<DT>::lo(k2), h == 0 ? 0.0f : s[i]);
            s[i] = __builtin_fmaf(Unpack<DT>::hi(q2[h]), Unpack<DT>::hi(k2), s[i]);
          }
        }
      }
      // adjacent-pair tree over the 16 chunk sums (xor 1, 2 in quads; the mirrors pair lanes
      // that hold equal partial sums' complements, which is the same tree); every lane ends up
      // with the total
#pragma unroll
      for (int i = 0; i < N; ++i) {
        s[i] = s[i] + __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(s[i]), 0xB1, 0xf, 0xf, false));
        s[i] = s[i] + __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(s[i]), 0x4E, 0xf, 0xf, false));
        s[i] = s[i] + __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(s[i]), 0x141, 0xf, 0xf, false));
        s[i] = s[i] + __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(s[i]), 0x140, 0xf, 0xf, false));
        mine[i] = gg == 0 || c8 == gg ? s[i] : mine[i];
        asm volatile("" : "+v"(mine[i]));                 // (chosen here, not all of them at the store)
      }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int j = j0 + i * PASS;
      if (TAGGED) {
        if (c8 < NG) s_w[c8][i * PASS + wave * 4 + grp] = mine[i] * scale;
      } else if (c8 < NG && j < n) {
        reinterpret_cast<float*>(a.P)[((size_t)head * G + c8) * a.max_pages + a.g.cand_lo + j] = mine[i] * scale;
      }
    }
  };
  static_assert(SCORE_PASSES == 4, "");
  if (passes == 1) score(UnrollBy<1>{});
  else if (passes == 2) score(UnrollBy<2>{});
  else score(UnrollBy<4>{});
  if (!TAGGED) return;
  lds_barrier();
  const int pages_log2 = __builtin_ctz(PASS * passes), pages = 1 << pages_log2, at0 = chunk * pages;     // (powers of two)
  for (int i = threadIdx.x; i < NG * pages; i += WAVES * 64) {
    const int gg = i >> pages_log2, jj = i & (pages - 1);
    if (at0 + jj < n) st_tag(a.P + ((size_t)head * G + gg) * a.max_pages + a.g.cand_lo + at0 + jj, __float_as_uint(s_w[gg][jj]), tag);
  }
}

template <int DT, int G, bool TAGGED, int WAVES>
__device__ __forceinline__ void score_role(const StepArgs& a, int head, int chunk) {
  if (a.sel_pool >= 4) score_pages<DT, G, true, TAGGED, WAVES>(a, head, chunk);
  else                 score_pages<DT, G, false, TAGGED, WAVES>(a, head, chunk);
}

// ---------------------------------------------------------------------------------
// softmax -> group mean -> top-k of one KV head: the arithmetic.
// ---------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t softmax_fixed(float p, float mx) {
  const float x = p - mx;
  const float t = x * 0x1.715476p+0f;          // fl32(log2 e)
  const float n = __builtin_rintf(t);
  const float f = t - n;
  float r = 0x1.430912p-13f;
  r = r * f; r = r + 0x1.5d87fep-10f;
  r = r * f; r = r + 0x1.3b2ab6p-7f;
  r = r * f; r = r + 0x1.c6b08ep-5f;
  r = r * f; r = r + 0x1.ebfbep-3f;
  r = r * f; r = r + 0x1.62e43p-1f;
  r = r * f; r = r + 1.0f;
  // e = ldexp(r, n) is exact here (n >= -64), and so is e * 2^31: one ldexp gives the same number
  float e31 = __builtin_ldexpf(r, (int)n + 31);
  if (t < -64.0f) e31 = 0.0f;
  return (uint32_t)__builtin_rintf(e31);
}

// A reciprocal of b good to an ulp or two: the hardware's approximation (a dozen bits would do)
// sharpened by three Newton steps.
__device__ __forceinline__ double reciprocal_near(double b) {
  double y = __builtin_amdgcn_rcp(b);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const double e = __builtin_fma(-b, y, 1.0);
    y = __builtin_fma(y, e, y);
  }
  return y;
}

// The correctly rounded fp64 quotient a / b of integers 0 <= a <= b < 2^48 from such a y (one
// reciprocal per head, not one division per candidate): q = a * y corrected twice with the exact
// remainder r = a - b * q.  After the first correction q is within an ulp; the second leaves an
// error of at most |r| * |y - 1/b| <= 2^-52 ulp, and a / b with b < 2^48 is either representable or at
// least 2^-49 ulp away from the nearest rounding boundary, so the rounding cannot go wrong.
__device__ __forceinline__ double div_rn(double a, double b, double y) {
  double q = a * y;
  double r = __builtin_fma(-b, q, a);
  q = __builtin_fma(r, y, q);
  r = __builtin_fma(-b, q, a);
  return __builtin_fma(r, y, q);
}

// pooled score of one candidate from the G per-head values e[] (softmax numerators, or the bits of
// the weights themselves), mode = FKV_POOL_*; zd = the heads' integer sums Z, zr = RN(1 / Z)
template <int G>
__device__ __forceinline__ float pooled_score(const uint32_t* e, const double* zd, const double* zr, int mode) {
  if (mode <= 1) {
    // mean (the method) or maximum over the group of the softmax values, in fp64
    double acc = div_rn((double)e[0], zd[0], zr[0]);
#pragma unroll
    for (int gg = 1; gg < G; ++gg) {
      const double sg = div_rn((double)e[gg], zd[gg], zr[gg]);
      if (mode == 0) acc = acc + sg;
      else acc = sg > acc ? sg : acc;
    }
    return mode == 0 ? (float)(acc / (double)G) : (float)acc;
  }
  // mean or maximum of the weights themselves in fp32, head order; or the pooled query's weight
  float acc = __uint_as_float(e[0]);
#pragma unroll
  for (int gg = 1; gg < G; ++gg) {
    if (mode == 2) acc = acc + __uint_as_float(e[gg]);
    else if (mode == 3) acc = fmaxf(acc, __uint_as_float(e[gg]));
  }
  return mode == 2 ? (float)((double)acc / (double)G) : acc;
}

// ---------------------------------------------------------------------------------
// role: selection of one KV head by a.slices groups of SEL_THREADS threads with a.slice candidates each.  Each group keeps
// its candidates' G values in registers from the weights to the key; what needs the whole head is exchanged as tagged
// words: the per-head maxima, the integer softmax sums (exact, so their order does not matter), and the keys, which the
// last group turns into the top-k.  A head's groups are adjacent in block order and wait for each other and for scoring
// blocks (lower indices) only, and for neither of them for long (PATIENCE).
//
// What bounds it: a chain of short phases, each of them instructions of the waves that share a SIMD one after the other
// (a wave-instruction takes the SIMD 4 cycles): about 26 per softmax numerator, 8 in fp64 per pooled term, and the
// reductions, which every wave makes.  A group is 8 waves, two to a SIMD, which fill each other's gaps (4 waves with twice
// the candidates each: 1 us more of a 10 us layer-step), and waves without a candidate end at once.  A long list is shared
// (selection_slices); each exchange costs a trip of about 1 us.
// TAGGED: the weights come from scoring blocks of this launch; else from a launch that has ended.
// ---------------------------------------------------------------------------------
constexpr int SEL_WAVES = 8, SEL_THREADS = SEL_WAVES * 64;
constexpr int SEL_REGS = 2, SEL_REGS_ALONE = 8;          // most candidates per thread, in the launches where scoring blocks
                                                         // share the unit and in the one that only selects
constexpr int TOPK_BINS = 512;

// 32-bit words of dynamic LDS that the keys of n candidates take (whole quads)
__host__ __device__ constexpr int select_key_words(int n) { return n > 0 ? (n + 3) & ~3 : 4; }

struct alignas(16) SelectLds {
  uint32_t hist[TOPK_BINS];
  uint32_t list[64];
  unsigned long long z[SEL_WAVES][MAX_G];
  float mx[SEL_WAVES][MAX_G];
  uint32_t scan[SEL_WAVES];
  uint32_t n_list;
  int alone;
  int failed[SEL_WAVES];
};

// The first histogram of the top-k decides nearly everything: for softmax scores its bins are a sixteenth of an octave
// wide below 1.0 (down to 2^-32), so the bin of the k-th score holds a handful of keys -- and few keys share a
// counter, where bins by the top byte put a whole selection on two or three of them.  Other scores: by the top 9 bits.
constexpr uint32_t kKeyOfOne = 0xBF800000u;               // score_key(1.0f)
__device__ __forceinline__ uint32_t topk_bin(uint32_t key, bool soft) {     // ascending bins: descending keys
  return soft ? min((uint32_t)TOPK_BINS - 1, (kKeyOfOne - min(key, kKeyOfOne)) >> 19) : (uint32_t)TOPK_BINS - 1 - (key >> 23);
}
// all keys of the bins up to `bin` are above this value, no other key is; bin < TOPK_BINS - 1
__device__ __forceinline__ uint32_t topk_floor(uint32_t bin, bool soft) {
  return soft ? kKeyOfOne - ((bin + 1) << 19) : (((uint32_t)TOPK_BINS - 1 - bin) << 23) - 1u;
}

// the bin of `hist` (ascending) that holds the `want`-th entry: bin, entries before it, entries in it.  Every wave
// scans by itself (lane l owns bins 8l .. 8l+7).
__device__ __forceinline__ void find_bin(const uint32_t* hist, uint32_t want, uint32_t& bin, uint32_t& before, uint32_t& in_bin) {
  const int lane = threadIdx.x & 63;
  const uint4 c0 = *reinterpret_cast<const uint4*>(hist + 8 * lane), c1 = *reinterpret_cast<const uint4*>(hist + 8 * lane + 4);
  const uint32_t c[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
  const uint32_t tot = ((c[0] + c[1]) + (c[2] + c[3])) + ((c[4] + c[5]) + (c[6] + c[7]));
  const uint32_t incl = wave_scan_u32(tot);
  uint32_t at = incl - tot, f = 0, cnt = c[0];
  const int src = __builtin_ctzll(__ballot(at < want && want <= incl));       // exactly one lane
#pragma unroll
  for (int i = 1; i < 8; ++i)
    if (f == i - 1 && at + cnt < want) { at += cnt; cnt = c[i]; f = i; }
  bin = (uint32_t)__builtin_amdgcn_readlane(8 * lane + (int)f, src);
  before = (uint32_t)__builtin_amdgcn_readlane((int)at, src);
  in_bin = (uint32_t)__builtin_amdgcn_readlane((int)cnt, src);
}

// Top-kk of n keys held in LDS, ties to the lower index, by nw waves: emit(pos, j) is called for the
// chosen j in ascending order of j with pos = 0 .. kk-1 (whichever thread owns j calls it).
// Before the call (and a barrier): sm.hist holds the counts of the keys' bins.  1 <= kk <= n.
// The keys of the one bin that is only partly wanted are collected and ranked against each other; only if there are
// more than 64 of them (ties, or scores that are not softmax values) the bytes are resolved one by one.
template <typename Emit>
__device__ __forceinline__ void block_topk(const uint32_t* key, int n, int kk, bool soft, int nw, SelectLds& sm, Emit emit) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nt = nw * 64;
  uint32_t T = 0, take_eq = 0;                       // take keys > T, and the first take_eq keys == T
  if (kk < n) {
    uint32_t bin, before, in_bin;
    find_bin(sm.hist, (uint32_t)kk, bin, before, in_bin);
    const uint32_t need = (uint32_t)kk - before;     // keys of the bin that are wanted
    if (need == in_bin && bin < TOPK_BINS - 1) {
      T = topk_floor(bin, soft);
    } else if (in_bin <= 64) {
      for (int j = tid; j < n; j += nt) {
        const uint32_t kj = key[j];
        if (topk_bin(kj, soft) == bin) sm.list[atomicAdd(&sm.n_list, 1u)] = kj;
      }
      lds_barrier();
      const uint32_t mine = lane < (int)in_bin ? sm.list[lane] : 0u;
      uint32_t above = 0, same = 0;
      for (uint32_t i = 0; i < in_bin; ++i) {
        const uint32_t ki = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)i);
        above += ki > mine ? 1u : 0u;
        same += ki == mine ? 1u : 0u;
      }
      const int src = __builtin_ctzll(__ballot(lane < (int)in_bin && above < need && need <= above + same));
      T = (uint32_t)__builtin_amdgcn_readlane((int)mine, src);
      take_eq = need - (uint32_t)__builtin_amdgcn_readlane((int)above, src);
    } else {
      // one byte at a time from the top; ends early once every key of the chosen bin is wanted (every wave sees the same
      // histogram, so the whole group leaves together)
      uint32_t prefix = 0, remaining = (uint32_t)kk;
      for (int shift = 24; shift >= 0; shift -= 8) {
        lds_barrier();                               // the last histogram has been read
        for (int i = tid; i < TOPK_BINS; i += nt) sm.hist[i] = 0;
        lds_barrier();
        for (int j = tid; j < n; j += nt) {
          const uint32_t kj = key[j];
          if (shift == 24 || (kj >> ((shift + 8) & 31)) == prefix) atomicAdd(&sm.hist[255u - ((kj >> shift) & 255u)], 1u);
        }
        lds_barrier();
        find_bin(sm.hist, remaining, bin, before, in_bin);
        remaining -= before;
        prefix = (prefix << 8) | (255u - bin);
        if (shift == 0) {
          T = prefix;                                // the kk-th largest key itself;
          take_eq = remaining;                       // of the keys equal to it, the lowest ids
        } else if (remaining == in_bin && (prefix << shift) != 0) {
          T = (prefix << shift) - 1;                 // everything from the bin's lowest key upwards
          break;
        }
      }
    }
  } else {
    take_eq = (uint32_t)n;
  }

  // ordered compaction: thread t owns the contiguous ids [4t, 4t + 4), and again nt * 4 further on
  uint32_t base = 0;                                 // chosen before this round: low 16 bits keys > T, high 16 bits keys == T
  for (int r0 = 0; r0 < n; r0 += nt * 4) {
    const int j = r0 + tid * 4;
    const uint4 k4 = *reinterpret_cast<const uint4*>(key + min(j, (n - 1) & ~3));      // (select_key_words)
    const uint32_t kj[4] = {k4.x, k4.y, k4.z, k4.w};
    uint32_t cnt = 0, is[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      is[i] = j + i < n ? (kj[i] > T ? 1u : kj[i] == T ? 0x10000u : 0u) : 0u;
      cnt += is[i];
    }
    const uint32_t incl = wave_scan_u32(cnt);
    if (r0) lds_barrier();                           // the last round's totals have been read
    if (lane == 63) sm.scan[wave] = incl;
    lds_barrier();
    uint32_t at = base + incl - cnt;
#pragma unroll
    for (int w = 0; w < SEL_WAVES; ++w) {
      const uint32_t v = w < nw ? sm.scan[w] : 0u;
      if (w < wave) at += v;
      base += v;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t eq_before = at >> 16;
      if (is[i] == 1u || (is[i] != 0u && eq_before < take_eq)) emit((int)((at & 0xffffu) + min(eq_before, take_eq)), j + i);
      at += is[i];
    }
  }
}

__device__ __forceinline__ SelectLds& select_lds() {
  __shared__ SelectLds sm;
  return sm;
}

// The keys of one head's candidates into `key`, and the counts of their bins into sm.hist, by the groups that share the head.
// A wave whose patience ends has nothing to say, and what it would have had to is never put into words under the tag: its
// group learns of it at the next barrier, from a value no maximum or sum has, and leaves.  Of the groups only the last one has to end with all the keys, and it
// can make them alone (alone_keys).  Returns whether this wave's keys (the last group: every key) are made.
template <int G, bool TAGGED, int REGS>
__device__ __forceinline__ bool shared_keys(const StepArgs& a, int head, int s, int nw, uint32_t* key, SelectLds& sm, uint32_t (&kreg)[REGS]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nt = nw * 64;
  const int n = a.g.n_cand, lo = a.g.cand_lo;
  const int S = a.slices, j0 = s * a.slice, j1 = min(n, j0 + a.slice);
  const bool last = s == S - 1;
  const uint32_t tag = launch_tag(a.no);
  const int mode = a.sel_pool;                         // FKV_POOL_*
  const bool soft = mode <= 1;                         // the variants that pool softmax values
  const int ng = mode >= 4 ? 1 : G;                    // weights in use per page (pooled query: the group's first)
  if (last) {
    for (int i = tid; i < TOPK_BINS; i += nt) sm.hist[i] = 0;
    if (tid == 0) { sm.n_list = 0; sm.alone = 0; }
  }
  // load_and_check() until every lane's words carry the tag; false: patience ended
  auto poll = [&](uint32_t kind, auto load_and_check) {
    int it = 0;
    while (__ballot(!load_and_check()) != 0) {
      if (++it > PATIENCE) return false;
      __builtin_amdgcn_s_sleep(1);
    }
    return (a.impatient & kind) == 0;
  };
  bool failed = false;                                 // this wave's patience ended
  auto any_failed = [&]() {                            // (by way of a barrier)
    if (lane == 0) sm.failed[wave] = failed ? 1 : 0;
    lds_barrier();
    return __ballot(sm.failed[min(lane, nw - 1)] != 0) != 0;
  };

  // ---- this group's weights: thread t has candidates j0 + t + u * nt ----
  const int U = (j1 - j0 + nt - 1) / nt;               // 1 .. REGS
  uint32_t e[REGS][G];                             // bits of the weights, then softmax numerators
  auto ours = [&](int u) { return j0 + tid + u * nt < j1; };
  // (All of a poll's loads are issued before the first is looked at, and none sits behind a branch of its own: one trip.)
  auto weights = [&](auto uc) {
    constexpr int UC = decltype(uc)::value;
    const size_t base = (size_t)head * G * a.max_pages + lo;
    size_t at[UC];
#pragma unroll
    for (int u = 0; u < UC; ++u) at[u] = base + min(j0 + tid + u * nt, j1 - 1);
    size_t row[G];
#pragma unroll
    for (int gg = 0; gg < G; ++gg) row[gg] = (size_t)min(gg, ng - 1) * a.max_pages;
    if (TAGGED) {
      failed = !poll(WAIT_WEIGHTS, [&]() {
        bool ok = true;
        unsigned long long w[UC][G];
#pragma unroll
        for (int u = 0; u < UC; ++u)
#pragma unroll
          for (int gg = 0; gg < G; ++gg) w[u][gg] = ld_tag(a.P + at[u] + row[gg]);
#pragma unroll
        for (int u = 0; u < UC; ++u)
#pragma unroll
          for (int gg = 0; gg < G; ++gg) {
            e[u][gg] = (uint32_t)w[u][gg];
            ok = ok & ((uint32_t)(w[u][gg] >> 32) == tag);
          }
        return ok;
      });
    } else {
#pragma unroll
      for (int u = 0; u < UC; ++u)
#pragma unroll
        for (int gg = 0; gg < G; ++gg) e[u][gg] = __float_as_uint(reinterpret_cast<const float*>(a.P)[at[u] + row[gg]]);
    }
  };
  if (U == 1) weights(UnrollBy<1>{});
  else if (REGS == 2 || U == 2) weights(UnrollBy<2>{});
  else weights(UnrollBy<REGS>{});
  FKV_STAMP(a, head, 2);

  // ---- fixed-point softmax: the head's maxima, numerators, integer denominators ----
  double zd[G], zr[G];
#pragma unroll
  for (int gg = 0; gg < G; ++gg) zd[gg] = zr[gg] = 1.0;
  if (soft) {
    unsigned long long* const mine = a.exch + ((size_t)head * MAX_SLICES + s) * 3 * MAX_G;
    const unsigned long long* const all = a.exch + (size_t)head * MAX_SLICES * 3 * MAX_G;
    const int gl = min(lane & 7, G - 1);               // lane 8r + g works on head g
    float mx[G];
#pragma unroll
    for (int gg = 0; gg < G; ++gg) {
      float v = __uint_as_float(e[0][gg]);             // (a thread without a candidate repeats the slice's last one)
#pragma unroll
      for (int u = 1; u < REGS; ++u)
        if (u < U) v = fmaxf(v, __uint_as_float(e[u][gg]));
      v = wave_max_f32(v);
      if (TAGGED && failed) v = __builtin_inff();
      if (lane == 0) sm.mx[wave][gg] = v;
    }
    lds_barrier();
    float v = -__builtin_inff();
#pragma unroll
    for (int w = 0; w < SEL_WAVES; ++w) v = fmaxf(v, sm.mx[min(w, nw - 1)][gl]);
    if (TAGGED && __ballot(v == __builtin_inff()) != 0 && any_failed()) return false;    // (a weight may be infinite)
    if (S > 1) {                                       // ... and over the slices: r is a slice
      if (wave == 0 && lane < G) st_tag(mine + lane, __float_as_uint(v), tag);
      const int r0 = min(lane >> 3, S - 1), r1 = min((lane >> 3) + 8, S - 1);
      unsigned long long w0 = 0, w1 = 0;
      failed = !poll(WAIT_MAXIMA, [&]() {
        w0 = ld_tag(all + (size_t)r0 * 3 * MAX_G + gl);
        w1 = ld_tag(all + (size_t)r1 * 3 * MAX_G + gl);
        return ((uint32_t)(w0 >> 32) == tag) & ((uint32_t)(w1 >> 32) == tag);
      });
      v = fmaxf(__uint_as_float((uint32_t)w0), __uint_as_float((uint32_t)w1));
      v = fmaxf(v, __shfl_xor(v, 8, 64));
      v = fmaxf(v, __shfl_xor(v, 16, 64));
      v = fmaxf(v, __shfl_xor(v, 32, 64));
    }
#pragma unroll
    for (int gg = 0; gg < G; ++gg) mx[gg] = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), gg));
    FKV_STAMP(a, head, 3);
#pragma unroll
    for (int gg = 0; gg < G; ++gg) {
      unsigned long long z = 0;
#pragma unroll
      for (int u = 0; u < REGS; ++u) {
        if (u < U) {
          e[u][gg] = softmax_fixed(__uint_as_float(e[u][gg]), mx[gg]);
          if (ours(u)) z += e[u][gg];
        }
      }
      z = wave_sum_u48(z);
      if (failed) z = 1ull << 56;                      // (sums are below 2^46)
      if (lane == 0) sm.z[wave][gg] = z;
    }
    lds_barrier();
    unsigned long long z = 0;
#pragma unroll
    for (int w = 0; w < SEL_WAVES; ++w) z += w < nw ? sm.z[w][gl] : 0ull;
    if (S > 1) {
      if (__ballot(z >> 56 != 0) != 0) return false;
      if (wave == 0 && lane < G) {
        st_tag(mine + MAX_G + lane, (uint32_t)z, tag);
        st_tag(mine + 2 * MAX_G + lane, (uint32_t)(z >> 32), tag);
      }
      const int r0 = min(lane >> 3, S - 1), r1 = min((lane >> 3) + 8, S - 1);
      unsigned long long w[4];
      failed = !poll(WAIT_SUMS, [&]() {
        const unsigned long long* p0 = all + (size_t)r0 * 3 * MAX_G + MAX_G + gl;
        const unsigned long long* p1 = all + (size_t)r1 * 3 * MAX_G + MAX_G + gl;
        w[0] = ld_tag(p0); w[1] = ld_tag(p0 + MAX_G); w[2] = ld_tag(p1); w[3] = ld_tag(p1 + MAX_G);
        return ((uint32_t)(w[0] >> 32) == tag) & ((uint32_t)(w[1] >> 32) == tag) & ((uint32_t)(w[2] >> 32) == tag) & ((uint32_t)(w[3] >> 32) == tag);
      });
      z = 0;
      if ((lane >> 3) < S) z += (w[0] & 0xffffffffull) | (w[1] << 32);
      if ((lane >> 3) + 8 < S) z += (w[2] & 0xffffffffull) | (w[3] << 32);
#pragma unroll
      for (int d = 8; d < 64; d <<= 1) {
        const uint32_t zl = (uint32_t)__shfl_xor((int)(uint32_t)z, d, 64), zh = (uint32_t)__shfl_xor((int)(uint32_t)(z >> 32), d, 64);
        z += ((unsigned long long)zh << 32) | zl;
      }
    }
    // one reciprocal per lane, handed to every lane as a scalar
    const double zv = (double)z, yv = reciprocal_near(zv);
    const unsigned long long zb = __builtin_bit_cast(unsigned long long, zv), yb = __builtin_bit_cast(unsigned long long, yv);
#pragma unroll
    for (int gg = 0; gg < G; ++gg) {
      zd[gg] = __builtin_bit_cast(double, ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(zb >> 32), gg) << 32) |
                                          (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)zb, gg));
      zr[gg] = __builtin_bit_cast(double, ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(yb >> 32), gg) << 32) |
                                          (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)yb, gg));
    }
  } else {
    if (any_failed()) return false;                    // (and behind its barrier the histogram is clear)
  }
  FKV_STAMP(a, head, 4);

  // ---- pooled scores -> keys ----
#pragma unroll
  for (int u = 0; u < REGS; ++u) {
    const int j = j0 + tid + u * nt;
    if (u < U) {
      kreg[u] = score_key(pooled_score<G>(e[u], zd, zr, mode));
      if (ours(u)) {
        if (last) {
          key[j] = kreg[u];
          atomicAdd(&sm.hist[topk_bin(kreg[u], soft)], 1u);
        } else if (!failed) {
          st_tag(a.keyx + (size_t)head * a.max_pages + j, kreg[u], tag);
        }
      }
    }
  }
  if (!last) return !failed;
  // the other slices' keys (lower block indices)
  for (int jj = tid; jj - lane < j0 && !failed; jj += 4 * nt) {
    unsigned long long w[4];
    failed = !poll(WAIT_KEYS, [&]() {
      bool ok = true;
#pragma unroll
      for (int u = 0; u < 4; ++u) w[u] = ld_tag(a.keyx + (size_t)head * a.max_pages + min(jj + u * nt, j0 - 1));
#pragma unroll
      for (int u = 0; u < 4; ++u) ok = ok & ((uint32_t)(w[u] >> 32) == tag);
      return ok;
    });
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (jj + u * nt < j0) {
        key[jj + u * nt] = (uint32_t)w[u];
        atomicAdd(&sm.hist[topk_bin((uint32_t)w[u], soft)], 1u);
      }
    }
  }
  if (failed) sm.alone = 1;
  lds_barrier();
  return S == 1 || sm.alone == 0;
}

// The weight of one page for one query head of the group by one thread, bit for bit score_pages'.
template <int DT, int G>
__device__ __forceinline__ float weight_alone(const StepArgs& a, int head, int gg, int j) {
  const uint16_t* const sm = a.summ + summ_idx(0, head, 0, 0, a.max_pages, a.g.cand_lo + j);
  const size_t to_min = (size_t)a.max_pages * D;
  const uint16_t* const q = a.q + (size_t)head * G * D;
  const bool pooled = a.sel_pool >= 4;                   // MeanQ, MaxQ
  float at1 = 0.0f, at2 = 0.0f, at4 = 0.0f, at8 = 0.0f, s = 0.0f;       // the tree over the 16 chunk sums: left halves in wait
#pragma unroll 1
  for (int c8 = 0; c8 < 16; ++c8) {
    float qc[8], mx[8], mn[8];
    unpack8<DT>(*reinterpret_cast<const uint4*>(q + (pooled ? 0 : gg) * D + c8 * 8), qc);
    if (pooled) {
#pragma unroll 1
      for (int g = 1; g < G; ++g) {
        float x[8];
        unpack8<DT>(*reinterpret_cast<const uint4*>(q + g * D + c8 * 8), x);
#pragma unroll
        for (int c = 0; c < 8; ++c) qc[c] = a.sel_pool == 4 ? qc[c] + x[c] : fmaxf(qc[c], x[c]);
      }
    }
    unpack8<DT>(*reinterpret_cast<const uint4*>(sm + c8 * 8), mx);
    unpack8<DT>(*reinterpret_cast<const uint4*>(sm + to_min + c8 * 8), mn);
    s = 0.0f;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      if (pooled) {
        if (a.sel_pool == 4) qc[c] = (float)((double)qc[c] / (double)G);
        const float pr = qc[c] * (qc[c] >= 0.0f ? mx[c] : mn[c]);
        s = c == 0 ? pr : s + pr;
      } else {
        s = __builtin_fmaf(qc[c], __float_as_uint(qc[c]) >> 31 ? mn[c] : mx[c], s);
      }
    }
    if (!(c8 & 1)) at1 = s;
    else if (!(c8 & 2)) at2 = at1 + s;
    else if (!(c8 & 4)) at4 = at2 + (at1 + s);
    else if (!(c8 & 8)) at8 = at4 + (at2 + (at1 + s));
    else s = at8 + (at4 + (at2 + (at1 + s)));
  }
  return s * 0x1.6a09e6p-4f;                             // fl32(1/sqrt(128))
}

// All keys of a head by one group alone, which waits for nobody: page weights (TAGGED: made here, whoever else makes them),
// maxima, sums, keys, in passes over the whole list.  The same numbers, bit for bit, by code that is short rather than fast:
// it is hardly ever run, and a compute unit's instruction cache (64 KB for two units) has to hold the rest of the kernel.
template <int DT, int G, bool TAGGED>
__device__ __forceinline__ void alone_keys(const StepArgs& a, int head, int nw, uint32_t* key, SelectLds& sm) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nt = nw * 64;
  const int n = a.g.n_cand;
  const int mode = a.sel_pool, ng = mode >= 4 ? 1 : G;
  const bool soft = mode <= 1;
  lds_barrier();                                         // (every wave is done with the LDS of what it did before)
  for (int i = tid; i < TOPK_BINS; i += nt) sm.hist[i] = 0;
  if (tid == 0) sm.n_list = 0;
  const size_t base = (size_t)head * G * a.max_pages + a.g.cand_lo;
  if (TAGGED) {
    const uint32_t tag = launch_tag(a.no);
#pragma unroll 1
    for (int i = tid; i < n * ng; i += nt) {
      const int gg = i / n, j = i - gg * n;
      st_tag(a.P + base + (size_t)gg * a.max_pages + j, __float_as_uint(weight_alone<DT, G>(a, head, gg, j)), tag);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // they are where the group's waves read them
    lds_barrier();
  }
  auto weight = [&](int j, int gg) {
    const size_t at = base + (size_t)(ng == 1 ? 0 : gg) * a.max_pages + j;
    return TAGGED ? (uint32_t)ld_tag(a.P + at) : reinterpret_cast<const uint32_t*>(a.P)[at];
  };
  if (soft) {
#pragma unroll 1
    for (int gg = 0; gg < G; ++gg) {
      float v = -__builtin_inff();
#pragma unroll 1
      for (int j = tid; j < n; j += nt) v = fmaxf(v, __uint_as_float(weight(j, gg)));
      v = wave_max_f32(v);
      if (lane == 0) sm.mx[wave][gg] = v;
      lds_barrier();
      v = sm.mx[0][gg];
#pragma unroll 1
      for (int w = 1; w < nw; ++w) v = fmaxf(v, sm.mx[w][gg]);
      unsigned long long z = 0;
#pragma unroll 1
      for (int j = tid; j < n; j += nt) z += softmax_fixed(__uint_as_float(weight(j, gg)), v);
      z = wave_sum_u48(z);
      if (lane == 0) sm.z[wave][gg] = z;
    }
    lds_barrier();
  }
#pragma unroll 1
  for (int j = tid; j < n; j += nt) {
    double acc = 0.0;
    float acc32 = 0.0f;
#pragma unroll 1
    for (int gg = 0; gg < ng; ++gg) {
      const uint32_t x = weight(j, gg);
      if (soft) {
        float v = sm.mx[0][gg];
        unsigned long long z = sm.z[0][gg];
#pragma unroll 1
        for (int w = 1; w < nw; ++w) {
          v = fmaxf(v, sm.mx[w][gg]);
          z += sm.z[w][gg];
        }
        const double zd = (double)z, sg = div_rn((double)softmax_fixed(__uint_as_float(x), v), zd, reciprocal_near(zd));
        acc = gg == 0 ? sg : mode == 0 ? acc + sg : sg > acc ? sg : acc;
      } else {
        const float w = __uint_as_float(x);
        acc32 = gg == 0 ? w : mode == 2 ? acc32 + w : fmaxf(acc32, w);
      }
    }
    const float sc = mode == 0 ? (float)(acc / (double)G) : mode == 1 ? (float)acc : mode == 2 ? (float)((double)acc32 / (double)G) : acc32;
    const uint32_t kj = score_key(sc);
    key[j] = kj;
    atomicAdd(&sm.hist[topk_bin(kj, soft)], 1u);
  }
  lds_barrier();
}

// Selecting block `s` of a head, up to the keys.  True for the waves that go on with select_finish -- the last block's, nw of
// them -- and `made`: whether the keys are there.
template <int G, bool TAGGED, int REGS = SEL_REGS>
__device__ __forceinline__ bool select_begin(const StepArgs& a, int head, int s, uint32_t* key, int& nw, bool& made) {
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = a.slices, j0 = s * a.slice, j1 = min(a.g.n_cand, j0 + a.slice);
  const bool last = s == S - 1;
  // The waves that take part: as many as there are candidates for; all of them where a plan has to be made or keys of
  // other slices have to be gathered.  The others of the block end here (a barrier counts the waves that are left).
  nw = (last && S > 1) || a.plan_new_slots || a.g.k_eff == 0 ? SEL_WAVES : min(SEL_WAVES, (j1 - j0 + 63) / 64);
  made = true;
  if (wave >= nw) return false;
  if (a.g.k_eff == 0) return true;
  // What select_finish needs of the arguments is read now, while the weights are waited for, and not at the end of the chain
  // (0.3 us of a layer-step of 8 to 20 us).
  asm volatile("" ::"s"(a.ids), "s"(a.ids_user), "s"(a.tagged), "s"(a.k), "s"(launch_tag(a.no)), "s"(a.plan_new_slots));
  uint32_t kreg[REGS];
  made = __builtin_amdgcn_readfirstlane(shared_keys<G, TAGGED, REGS>(a, head, s, nw, key, select_lds(), kreg));
  if (made) {                                            // the pooled scores, kept for inspection
#pragma unroll
    for (int u = 0; u < REGS; ++u) {
      const int j = j0 + tid + u * nw * 64;
      if (j < j1) a.score[(size_t)head * a.max_pages + a.g.cand_lo + j] = key_score(kreg[u]);
    }
  }
  return last;
}

// ... and from the keys on, by nw waves: the top-k, the ids out, the recall plan.
template <int DT, int G, bool TAGGED>
__device__ __forceinline__ void select_finish(const StepArgs& a, int head, uint32_t* key, int nw, bool made) {
  SelectLds& sm = select_lds();
  const int tid = threadIdx.x, nt = nw * 64;
  const int n = a.g.n_cand, lo = a.g.cand_lo, kk = a.g.k_eff, k = a.k;
  const uint32_t tag = launch_tag(a.no);
  int32_t* out = a.ids + (size_t)head * k;
  int32_t* outu = a.ids_user ? a.ids_user + (size_t)head * k : nullptr;
  // a picked id goes out three ways: the layer's id list, the caller's copy, and (one-launch layer-step) as a tagged
  // word, so that a waiting attention wave sees "this launch's id" in one read
  unsigned long long* tagw = a.tagged ? a.tagged + (size_t)head * k : nullptr;
  // With a recall plan to make, the ids are only collected in the plan's LDS here and everything goes out after it.
  int32_t* plan_sm = reinterpret_cast<int32_t*>(key) + a.plan_lds_off;
  int32_t* plan_nid = a.plan_new_slots ? plan_sm + 4 * k : nullptr;
  auto put_id = [&](int pos, int id) {
    if (plan_nid) { plan_nid[pos] = id; return; }
    if (tagw) st_tag(tagw + pos, (uint32_t)id, tag);
    out[pos] = id;
    if (outu) outu[pos] = id;
  };
  if (kk > 0) {
    if (__builtin_expect(!made, 0)) alone_keys<DT, G, TAGGED>(a, head, nw, key, sm);
    FKV_STAMP(a, head, 5);
    block_topk(key, n, kk, a.sel_pool <= 1, nw, sm, [&](int pos, int j) { put_id(pos, lo + j); });
  }
  for (int i = kk + tid; i < k; i += nt) put_id(i, -1);   // padding
  if (plan_nid) {
    lds_barrier();                                       // the ids are all in LDS
    plan_head<SEL_THREADS>(out, a.plan_act_ids + (size_t)head * k, a.plan_act_slots + (size_t)head * k,
                           a.plan_new_slots + (size_t)head * k, a.plan_miss + (size_t)head * (1 + 3 * k), k, a.g.n_full,
                           plan_sm, true);
    const int32_t* nslot = plan_sm + 5 * k;
    for (int i = tid; i < k; i += SEL_THREADS) {
      const int id = plan_nid[i], sl = nslot[i];
      if (tagw) st_tag(tagw + i, tagged_pick(id, sl & (TAGGED_MAX_SLOTS - 1), (sl & PLAN_MISS_BIT) != 0), tag);
      out[i] = id;
      if (outu) outu[i] = id;
    }
  }
  FKV_STAMP(a, head, 8);
  // the pooled scores, kept for inspection: the group's own, or all of them if it was alone
  if (!made) for (int j = tid; j < n; j += nt) a.score[(size_t)head * a.max_pages + lo + j] = key_score(key[j]);
}

// ---------------------------------------------------------------------------------
// role dispatch of one block: row y of the grid counts [append][correction test][scoring ...][selection ...], each
// present only if its role bit is set; x is the KV head, except that the selection's blocks are numbered through row by
// row so that a head's are adjacent (they wait for each other: in block order, at most one head's are ever half there).
// ---------------------------------------------------------------------------------
// select(head, slice): what a selecting block does.
template <int DT, int G, typename Select>
__device__ __forceinline__ void step_roles(const StepArgs& a, int x, int y, Select select) {
  if (a.roles & ROLE_APPEND) {
    if (y == 0) { append_role<DT>(a, x); return; }
    y -= 1;
  }
  if (a.roles & ROLE_CORR) {
    if (y == 0) { corr_role<DT, G>(a, x); return; }
    y -= 1;
  }
  if (y < a.chunks) {
    if (y == 0) FKV_STAMP(a, x, 0);
    score_role<DT, G, true, STEP_WAVES>(a, x, y);
    if (y == 0) FKV_STAMP(a, x, 1);
    return;
  }
  const int i = (y - a.chunks) * a.heads + x;
  select(i >> a.slices_log2, i & (a.slices - 1));
}

}  // namespace fkv
