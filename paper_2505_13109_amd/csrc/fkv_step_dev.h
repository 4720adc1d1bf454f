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

#define FKV_STAMP(a, head, i) do { if (__builtin_expect((a).tstamp != nullptr, 0) && (head) == 0 && threadIdx.x == 0) (a).tstamp[i] = wall_clock64(); } while (0)

#ifndef FKV_STEP_THREADS
#define FKV_STEP_THREADS 512
#endif
constexpr int STEP_THREADS = FKV_STEP_THREADS;         // >= 256 (the radix histograms have 256 bins)
constexpr int STEP_WAVES = STEP_THREADS / 64;
constexpr int SCORE_PASSES = 4;                        // most passes a scoring block can make (StepArgs::passes <= this)
constexpr int PAGES_PER_PASS = STEP_WAVES * 4;         // a wave scores 4 pages per pass
constexpr int MAX_SLICES = 16;                         // most blocks that share one head's selection
constexpr int SCAN_WAVES = 4;                          // of a block of the scan

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
  unsigned long long* exch;  // [heads][2 (halves)][MAX_G][MAX_SLICES] tagged: the softmax sums that a head's selecting blocks tell each other
  unsigned long long* keyx;  // [heads][max_pages] tagged: keys and page ids of each block's best candidates, for the head's
  unsigned long long* keyid; // last selecting block
  unsigned long long* cmax;  // the chunks' largest weights, [heads][cmax_stride] tagged, or (where P is plain) [heads][cmax_plain_stride]
  LaunchNo no;               // of this launch
  bool home;                 // a head's blocks are on one XCD (deal_block)
  uint32_t impatient;        // WAIT_* bits: waits that run out at once (tests)
  int* by_itself;            // one more for every head's list that a block chose from without the others (LayerStatus)
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
// PAST: the summaries are read past the caches (STREAM_SUMMARIES; as a branch around the loads it costs short launches 2 %).
template <int DT, int G, bool QMODE, bool TAGGED, int WAVES, bool PAST>
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
      const uint16_t* const p = sm + (size_t)min(j0 + ps * PASS, n - 1) * D;
      wmax[ps] = PAST ? load_past(p) : *reinterpret_cast<const uint4*>(p);
      wmin[ps] = PAST ? load_past(p + to_min) : *reinterpret_cast<const uint4*>(p + to_min);
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
  __shared__ float s_max[TAGGED ? WAVES : 1][MAX_G];
  float largest = -__builtin_inff();                      // of query head c8 among the pages of the row of lanes
  constexpr int GP = group_pow2(G);
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
      const float w = mine[i] * scale;
      largest = j < n ? fmaxf(largest, w) : largest;
      if (TAGGED) {
        if (c8 < NG) s_w[c8][i * PASS + wave * 4 + grp] = w;
      } else if (c8 < NG && j < n) {
        reinterpret_cast<float*>(a.P)[((size_t)head * G + c8) * a.max_pages + a.g.cand_lo + j] = w;
      }
    }
  };
  static_assert(SCORE_PASSES == 4, "");
  if (passes == 1) score(UnrollBy<1>{});
  else if (passes == 2) score(UnrollBy<2>{});
  else score(UnrollBy<4>{});
  // The chunk's largest weight of each query head: where several blocks share a head's selection, each of them knows the head's
  // maximum by these as soon as its own weights are there.
  const bool soft = !QMODE && a.sel_pool <= 1 && a.slices > 1;
  if (soft) largest = max_over_rows(largest);
  if (!TAGGED) {
    if (soft && lane < NG) reinterpret_cast<float*>(a.cmax)[head * cmax_plain_stride(a.max_pages) + (chunk * WAVES + wave) * GP + lane] = largest;
    return;
  }
  if (soft && lane < MAX_G) s_max[wave][lane] = largest;  // (what lanes from NG on have is nobody's)
  lds_barrier();
  static_assert(WAVES == 8 || !TAGGED, "");
  if (soft && wave == WAVES - 1) {                        // lane 8w + g has wave w's of head g
    const float v = __uint_as_float(class_reduce<8>(__float_as_uint(s_max[lane >> 3][lane & 7]), OpMaxF32()));
    if (lane < NG) st_tag(a.cmax + head * cmax_stride(a.max_pages) + chunk * GP + lane, __float_as_uint(v), tag, a.home);
  }
  const int pages_log2 = __builtin_ctz(PASS * passes), pages = 1 << pages_log2, at0 = chunk * pages;     // (powers of two)
  for (int i = threadIdx.x; i < NG * pages; i += WAVES * 64) {
    const int gg = i >> pages_log2, jj = i & (pages - 1);
    if (at0 + jj < n) st_tag(a.P + ((size_t)head * G + gg) * a.max_pages + a.g.cand_lo + at0 + jj, __float_as_uint(s_w[gg][jj]), tag, a.home);
  }
}

template <int DT, int G, bool TAGGED, int WAVES, bool PAST>
__device__ __forceinline__ void score_role(const StepArgs& a, int head, int chunk) {
  if (a.sel_pool >= 4) score_pages<DT, G, true, TAGGED, WAVES, PAST>(a, head, chunk);
  else                 score_pages<DT, G, false, TAGGED, WAVES, PAST>(a, head, chunk);
}

// ---------------------------------------------------------------------------------
// softmax -> group mean -> top-k of one KV head: the arithmetic.
// ---------------------------------------------------------------------------------
// (As written, up to exact scalings: the coefficients times 2^31 give e * 2^31; t + 3 * 2^22 is rint(t) + 3 * 2^22, with n in its
// last bits, from where it goes to the exponent by an integer addition; below t = -64 the result is below a half and so 0.)
__device__ __forceinline__ uint32_t softmax_fixed(float p, float mx) {
  const float x = p - mx;
  const float t = fmaxf(x * 0x1.715476p+0f, -64.0f);      // fl32(log2 e)
  const float shifted = t + 0x1.8p+23f;
  const float f = t - (shifted - 0x1.8p+23f);
  float r = 0x1.430912p+18f;
  r = r * f; r = r + 0x1.5d87fep+21f;
  r = r * f; r = r + 0x1.3b2ab6p+24f;
  r = r * f; r = r + 0x1.c6b08ep+26f;
  r = r * f; r = r + 0x1.ebfbep+28f;
  r = r * f; r = r + 0x1.62e43p+30f;
  r = r * f; r = r + 0x1p+31f;
  const float e31 = __uint_as_float(__float_as_uint(r) + (__float_as_uint(shifted) << 23));
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
// reciprocal per head, not one division per candidate): q = a * y is within 2^-51 of it, or four units in the last place; its
// remainder r = a - b * q, a multiple of q's last place and below 2^51 of them, is exact; and r * y corrects q up to
// |r| * |y - 1/b|, at most 4 * 2^-52 = 2^-50 of a unit in the last place.  a / b with b < 2^48 is either representable or at
// least 2^-49 of a unit away from the nearest rounding boundary, so the last rounding cannot go wrong.
__device__ __forceinline__ double div_rn(double a, double b, double y) {
  const double q = a * y;
  return __builtin_fma(__builtin_fma(-b, q, a), y, q);
}

// a / G, correctly rounded: one correction of a * RN(1 / G) by its exact remainder (Markstein); a power of two is exact anyway
template <int G>
__device__ __forceinline__ double div_by_group(double a) {
  constexpr double y = 1.0 / G;
  if constexpr ((G & (G - 1)) == 0) return a * y;
  const double q = a * y;
  return __builtin_fma(__builtin_fma(-(double)G, q, a), y, q);
}

// the method's score of a candidate: the mean of its G softmax values, from their numerators e, the heads' integer sums Z and RN(1 / Z)
template <int G>
__device__ __forceinline__ float mean_score(const uint32_t* e, const double* zd, const double* zr) {
  double acc = div_rn((double)e[0], zd[0], zr[0]);
#pragma unroll
  for (int gg = 1; gg < G; ++gg) acc = acc + div_rn((double)e[gg], zd[gg], zr[gg]);
  return (float)div_by_group<G>(acc);
}
// ... and by the other modes (FKV_POOL_*): the largest softmax value, in fp64; mean or maximum of the weights themselves (e: their bits) in
// fp32, head order; the pooled query's weight
template <int G>
__device__ __forceinline__ float pooled_score(const uint32_t* e, const double* zd, const double* zr, int mode) {
  if (mode == 1) {
    double most = div_rn((double)e[0], zd[0], zr[0]);
#pragma unroll
    for (int gg = 1; gg < G; ++gg) {
      const double sg = div_rn((double)e[gg], zd[gg], zr[gg]);
      most = sg > most ? sg : most;
    }
    return (float)most;
  }
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
// its candidates' G values in registers from the weights to the choice.  What needs the whole head comes as words of other
// blocks: the maxima from the blocks that scored (the largest of every chunk of pages), the integer softmax sums from the
// other groups (exact, so their order does not matter), and the keys and ids of each group's own best k, among which the
// last group finds the head's.  A head's groups, dealt as deal_block says, wait for each other and for scoring blocks (lower
// indices) only, and for neither of them for long (PATIENCE).
//
// What bounds it: a chain of short phases.  A wave issues an instruction every 4 cycles, a value takes 28 from the vector unit through
// a scalar and back, a branch 24 to 55, an LDS round trip 57, a trip between blocks 0.2 us and more (st_tag); so what counts is the
// number of dependent instructions, of branches and of barriers (see topk_items, and select_rows for what is told apart once instead of
// beside each row of candidates).  A group is 8 waves, two to a SIMD, which fill each other's gaps (4 waves with twice
// the candidates each: 1 us more of a 10 us layer-step), and waves without a candidate end at once.  A long list is shared
// (selection_slices); each exchange costs its trip and the barriers around it.
// TAGGED: the weights come from scoring blocks of this launch; else from a launch that has ended.
// ---------------------------------------------------------------------------------
constexpr int SEL_WAVES = 8, SEL_THREADS = SEL_WAVES * 64;
constexpr int SEL_REGS = 4;                              // most candidates per thread where a head's selection is shared
__host__ __device__ constexpr int sel_regs_alone(int G) { return G <= 3 ? 8 : 4; }      // ... and where one group has it (registers)
constexpr int SEL_OTHERS = 4;                            // most of the other groups' candidates per thread that are kept in registers
// candidates that each group but the last hands on, group after group: all of them where the last group's registers hold
// them, else its best k
__host__ __device__ constexpr int handed_on(int slices, int slice, int kk) {
  return (slices - 1) * slice <= SEL_OTHERS * SEL_THREADS || slice < kk ? slice : kk;
}
constexpr int TOPK_BINS = 512;
constexpr uint32_t kNoSum = 1u << 28;                    // in place of a sum: a wave has not seen its weights
// how far a group got: it has to make the keys alone; the keys of all that may be chosen are in LDS; the ids are out
enum class Selected : int { NOTHING, KEYS, IDS };

// 32-bit words of dynamic LDS that the keys of n candidates take (whole quads)
__host__ __device__ constexpr int select_key_words(int n) { return n > 0 ? (n + 3) & ~3 : 4; }

struct TopkBins { uint32_t top, shift; };
constexpr int SEL_ROWS = SEL_WAVES * 4;                 // rows of 16 lanes
struct alignas(16) SelectLds {
  uint32_t hist[TOPK_BINS + 64];                         // (and counters for threads without a candidate)
  uint32_t list[128];                                    // (and a place for lanes that have nothing to put on it)
  uint32_t count[64];
  union {
    float mx_row[MAX_G][SEL_ROWS];                       // by query head and row of 16 lanes
    unsigned long long whole[128];                       // the list with whole keys (the maxima are not read any more then)
  };
  uint2 z_row[MAX_G][SEL_ROWS];
  unsigned long long z[SEL_WAVES][MAX_G];
  float mx[SEL_WAVES][MAX_G];
  uint32_t scan[SEL_WAVES];
  uint32_t n_list;
  TopkBins bins;                                         // of scores that are not softmax values
  int alone;
  int failed[SEL_WAVES];
};

// The first histogram of the top-k decides nearly everything: its bins are so narrow that the bin of the k-th score holds a handful of
// keys -- and few keys share a counter, where bins by the top byte put a whole selection on two or three of them.  Below `top`,
// 2^(23 - shift) to an octave: for softmax scores 16 below 1.0 (down to 2^-32), for others 64 below the group's largest weight (8 heads
// x 992 candidates, MeanQK, a layer-step: 9.4 us; with bins by the top 9 bits, of which page weights have a few, 12.7, since
// hundreds of keys were left to block_topk).
constexpr TopkBins kSoftBins = {0xBF800000u, 19};         // (score_key(1.0f))
__device__ __forceinline__ TopkBins bins_below(uint32_t largest) { return TopkBins{min(largest, 0xff800000u) + (1u << 22), 17}; }
__device__ __forceinline__ uint32_t topk_bin(uint32_t key, TopkBins b) {     // ascending bins: descending keys
  return min((uint32_t)TOPK_BINS - 1, (b.top - min(key, b.top)) >> b.shift);
}
// all keys of the bins up to `bin` are above this value, no other key is; bin < TOPK_BINS - 1, and there are keys in later bins
__device__ __forceinline__ uint32_t topk_floor(uint32_t bin, TopkBins b) { return b.top - ((bin + 1) << b.shift); }

// the bin of `hist` (ascending) that holds the `want`-th entry: bin, entries before it, entries in it.  Every wave
// scans by itself: lane l sums bins 8l .. 8l+7, then the eight bins of the lane where the entry is are read again, one a lane
// (0.1 us less than picking it from a lane's eight registers).
__device__ __forceinline__ void find_bin(const uint32_t* hist, uint32_t want, uint32_t& bin, uint32_t& before, uint32_t& in_bin) {
  const int lane = threadIdx.x & 63;
  const uint4 c0 = *reinterpret_cast<const uint4*>(hist + 8 * lane), c1 = *reinterpret_cast<const uint4*>(hist + 8 * lane + 4);
  const uint32_t tot = ((c0.x + c0.y) + (c0.z + c0.w)) + ((c1.x + c1.y) + (c1.z + c1.w));
  const uint32_t incl = wave_scan_u32(tot);
  const int src = __builtin_ctzll(__ballot(incl >= want));                    // (there are as many entries)
  const uint32_t c = hist[8 * src + (lane & 7)];
  uint32_t at = c;                                                            // inclusive, over eight lanes
  at += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)at, 0x111, 0xf, 0xf, true);   // row_shr:1, 0 shifted in
  at += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)at, 0x112, 0xf, 0xf, true);
  at += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)at, 0x114, 0xf, 0xf, true);
  at += (uint32_t)__builtin_amdgcn_readlane((int)(incl - tot), src);
  const int f = __builtin_ctzll(__ballot(at >= want));                        // (one of the first eight lanes)
  bin = (uint32_t)(8 * src + f);
  in_bin = (uint32_t)__builtin_amdgcn_readlane((int)c, f);
  before = (uint32_t)__builtin_amdgcn_readlane((int)at, f) - in_bin;
}

// The best kk of a group's items, ties to the lower one in order.  A thread holds items key[u] (0: none), u < T; the order is by u,
// then by thread; T * nw <= 64.  emit(u, chosen, pos): the lanes of the mask `chosen` hold chosen items in slot u, in the order pos = 0 ..
// kk - 1.  n: items of the group.  Before the call (and a barrier): sm.hist holds the counts of the keys' bins, sm.n_list is 0.
// The keys of the one bin that is only partly wanted are collected with their places in the order and ranked against each other by every
// wave; the same barrier brings the counts per wave of what is chosen anyway, and which of the others are chosen is the same in every
// wave.  False, and nothing done, if there are more than 64 of them (ties, mostly).
// ANY: of any keys, in the slots below `first` and from A on, `second` of them.  Else of keys up to bins.top, in all slots: what is left
// of a key in a bin, and the place, fit 32 bits -- except in the last bin, which is as wide as it takes: false there too.
// The chain is what counts (a wave by itself: an instruction 4 cycles, a value that goes from the vector unit through a scalar and back 28,
// a branch that is not taken 24 and one that is 38, one by a lane's condition 55, an LDS trip 57): so everything is done for all T slots at
// once, by masks, and what a lane has no use for goes to a place that nobody reads -- a place of its own, since lanes queue up for one
// word (512 atomics on one counter take 1090 cycles, on 32 of them 120).  From the weights to the ids, with the slots in loops over those
// in use and the poolings told apart beside each, and so: 97 candidates, G = 4, 2.5 and 1.8 us; 992 3.8 and 3.0; 2015 in eight blocks, G = 8,
// 6.0 and 4.9; layer-steps of 96 candidates, G = 7, all heads corrected 11.0 and 10.1.
template <bool ANY, int A, int T, typename Emit>
__device__ __forceinline__ bool topk_items(const uint32_t (&key)[T], int first, int second, int n, int kk, TopkBins bins, int nw, SelectLds& sm, Emit emit) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto slots = [&](auto f) {
#pragma unroll
    for (int u = 0; u < A; ++u) {
      if (ANY && u >= first) break;
      f(u);
    }
#pragma unroll
    for (int u = A; u < T; ++u) {
      if (ANY && u - A >= second) break;
      f(u);
    }
  };
  uint32_t above = 0, from = 0, base = 0;            // keys > above are chosen; those > from, up to there, if their turn comes
  uint32_t take = 0, in_bin = 0;                     // how many of these are wanted
  bool ranked = false;
  if (kk < n) {
    uint32_t bin, before;
    find_bin(sm.hist, (uint32_t)kk, bin, before, in_bin);
    take = (uint32_t)kk - before;
    ranked = take != in_bin;
    const int tail = bin == TOPK_BINS - 1;
    if (__builtin_expect(((int)ranked & ((int)(in_bin > 64) | (ANY ? 0 : tail))) != 0, 0)) return false;
    base = bins.top - (bin << bins.shift);           // (the bin of a key: at most that, or the first)
    const uint32_t end = (bin + 1) << bins.shift;
    from = (tail | (int)(end > bins.top)) != 0 ? 0u : bins.top - end;
    above = !ranked ? from : bin == 0 ? ~0u : base;
  }
  static_assert(T * SEL_WAVES <= 64 && T * SEL_THREADS <= 4096 && 19 + 12 < 32, "");
  unsigned long long sure[T], maybe[T];              // (not ANY)
  uint32_t counts = 0;                               // lane u: slot u's
  uint32_t mine = 0;                                 // this lane's that go on the list
  slots([&](int u) {
    const unsigned long long b = __ballot(key[u] > above);
    if (ANY) mine += key[u] > from && !(key[u] > above) ? 1u : 0u;           // (one loop for both: a branch for each slot)
    else     sure[u] = b;
    const uint32_t c = (uint32_t)__popcll(b);
    counts = lane == u || (u == 0 && (!ANY || lane >= T)) ? c : counts;
  });
  auto place = [&](int u) { return (uint32_t)(u * nw * 64 + tid); };
  auto rank_of = [&](int u) { return ((base - min(key[u], base)) << 12) + place(u); };
  auto whole_rank_of = [&](int u) { return (unsigned long long)~key[u] << 32 | place(u); };
  if (ranked) {
    if (!ANY) {
      slots([&](int u) {
        maybe[u] = __ballot(key[u] > from) & ~sure[u];
        mine += key[u] > from && !(key[u] > above) ? 1u : 0u;
      });
    }
    if (mine != 0) {
      // (an atomic of each lane that has some: one for the wave would be a longer chain, and lanes queue up for one address)
      auto* n_list = (__attribute__((address_space(3))) uint32_t*)&sm.n_list;
      asm volatile("" : "+v"(n_list));
      uint32_t at = __hip_atomic_fetch_add(n_list, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      slots([&](int u) {
        const bool in = key[u] > from && !(key[u] > above);
        if (ANY) sm.whole[in ? at : 64u + (uint32_t)lane] = whole_rank_of(u);
        else     sm.list[in ? at : 64u + (uint32_t)lane] = rank_of(u);
        at += in ? 1u : 0u;
      });
    }
  }
  sm.count[lane < T ? lane * nw + wave : wave] = counts;                      // (lanes from T on repeat slot 0's)
  lds_barrier();
  uint32_t cnt = sm.count[lane];
  cnt = lane < T * nw ? cnt : 0u;
  unsigned long long picked = 0;                     // of the list
  uint32_t at = ~0u;                                 // the place of this lane's entry
  unsigned long long up_to = ((unsigned long long)~above << 32) - 1;         // (ANY: the last of the chosen, or what they are all before)
  if (ranked) {
    // an entry a lane
    if constexpr (ANY) {
      unsigned long long entry = sm.whole[lane];
      entry = lane < (int)in_bin ? entry : ~0ull;
      uint32_t before = 0;
#pragma unroll 1
      for (uint32_t i = 0; i < in_bin; i += 4) {
#pragma unroll
        for (uint32_t v = 0; v < 4; ++v) before += lane_u64(entry, (int)(i + v)) < entry ? 1u : 0u;
      }
      up_to = lane_u64(entry, __builtin_ctzll(__ballot(before == take - 1 && lane < (int)in_bin)));
      picked = __ballot(entry <= up_to);
      at = (uint32_t)entry;
    } else {
      uint32_t entry = sm.list[lane];
      entry = lane < (int)in_bin ? entry : ~0u;
      uint32_t before = 0;
#pragma unroll 1
      for (uint32_t i = 0; i < in_bin; i += 8) {
#pragma unroll
        for (uint32_t v = 0; v < 8; ++v) before += (uint32_t)__builtin_amdgcn_readlane((int)entry, (int)(i + v)) < entry ? 1u : 0u;
      }
      const uint32_t last = (uint32_t)__builtin_amdgcn_readlane((int)entry, __builtin_ctzll(__ballot(before == take - 1 && lane < (int)in_bin)));
      picked = __ballot(entry <= last);
      at = entry;
      slots([&](int u) { sure[u] |= maybe[u] & __ballot(rank_of(u) <= last); });
    }
  }
  const uint32_t excl = wave_scan_u32(cnt) - cnt, group = (at & 4095u) >> 6;
  slots([&](int u) {
    uint32_t before = (uint32_t)__builtin_amdgcn_readlane((int)excl, u * nw + wave);
    if (ranked) before += (uint32_t)__popcll(picked & __ballot(group < (uint32_t)(u * nw + wave)));
    const unsigned long long chosen = ANY ? __ballot(whole_rank_of(u) <= up_to) : sure[u];
    const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(chosen >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)chosen, before));
    emit(u, chosen, (int)pos);
  });
  return true;
}

// The same for n keys held in LDS: emit(pos, j) is called for the chosen j in ascending order of j with pos = 0 .. kk-1
// (whichever thread owns j calls it).  1 <= kk <= n.  Longer chains: for lists that do not fit the registers, and for a group
// that has made the keys alone.
template <typename Emit>
__device__ __forceinline__ void block_topk(const uint32_t* key, int n, int kk, TopkBins bins, int nw, SelectLds& sm, Emit emit) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nt = nw * 64;
  uint32_t T = 0, take_eq = 0;                       // take keys > T, and the first take_eq keys == T
  if (kk < n) {
    uint32_t bin, before, in_bin;
    find_bin(sm.hist, (uint32_t)kk, bin, before, in_bin);
    const uint32_t need = (uint32_t)kk - before;     // keys of the bin that are wanted
    if (need == in_bin && bin < TOPK_BINS - 1) {
      T = topk_floor(bin, bins);
    } else if (in_bin <= 64) {
      for (int j = tid; j < n; j += nt) {
        const uint32_t kj = key[j];
        if (topk_bin(kj, bins) == bin) sm.list[atomicAdd(&sm.n_list, 1u)] = kj;
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

// where a picked id goes: the layer's id list, the caller's copy, and (one-launch layer-step) as a tagged word, so that a
// waiting attention wave sees "this launch's id" in one read.  With a recall plan to make, the ids are only collected in the
// plan's LDS, and everything goes out after it.
struct PutId {
  int32_t *out, *outu, *plan_nid;
  unsigned long long* tagw;
  uint32_t tag;
  bool home;
  __device__ __forceinline__ PutId(const StepArgs& a, int head, uint32_t* key) {
    out = a.ids + (size_t)head * a.k;
    outu = a.ids_user ? a.ids_user + (size_t)head * a.k : nullptr;
    tagw = a.tagged ? a.tagged + (size_t)head * a.k : nullptr;
    plan_nid = a.plan_new_slots ? reinterpret_cast<int32_t*>(key) + a.plan_lds_off + 4 * a.k : nullptr;
    tag = launch_tag(a.no);
    home = a.home;
  }
  __device__ __forceinline__ void operator()(int pos, int id) const {
    if (plan_nid) { plan_nid[pos] = id; return; }
    if (tagw) st_tag(tagw + pos, (uint32_t)id, tag, home);
    out[pos] = id;
    if (outu) outu[pos] = id;
  }
};

// One group's part of a head's selection, up to the ids (the last group) or to its own best candidates in words (the others).
// A wave whose patience ends has nothing to say, and what it would have had to is never put into words under the tag: its
// group learns of it at the next barrier, from a value no sum has or a flag, and leaves.  Of the groups only the last one has to
// end with all the keys, and it can make them alone (alone_keys).  Returns how far the group got.
// MEAN: the method's own scores, straight through for U rows of candidates per thread; else any other pooling, by those of U rows that
// are in use.  SHARED: there may be several groups (MEAN: there are).
template <int G, bool TAGGED, bool MEAN, bool SHARED, int U>
__device__ __forceinline__ Selected select_group(const StepArgs& a, int head, int s, int nw, uint32_t* key_lds, SelectLds& sm) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nt = nw * 64;
  const int n = a.g.n_cand, lo = a.g.cand_lo, kk = a.g.k_eff;
  const int S = SHARED ? a.slices : 1, j0 = SHARED ? s * a.slice : 0, j1 = SHARED ? min(n, j0 + a.slice) : n;
  const bool shared = SHARED && (MEAN || S > 1), last = !SHARED || s == S - 1;
  const uint32_t tag = launch_tag(a.no);
  const int mode = MEAN ? 0 : a.sel_pool;              // FKV_POOL_*
  const bool soft = mode <= 1;                         // the variants that pool softmax values
  const int ng = mode >= 4 ? 1 : G;                    // weights in use per page (pooled query: the group's first)
  constexpr int GP = group_pow2(G);
  asm volatile(".p2align 6");                          // (here and at the polls: see select_rows)
  for (int i = tid * 4; i < TOPK_BINS; i += nt * 4) *reinterpret_cast<uint4*>(&sm.hist[i]) = make_uint4(0, 0, 0, 0);
  if (tid == 0) { sm.n_list = 0; sm.alone = 0; }
  // load_and_check() until every lane's words carry the tag; false: patience ended
  auto poll = [&](uint32_t kind, auto load_and_check) {
    int it = 0;
    asm volatile(".p2align 6");
    while (__ballot(!load_and_check()) != 0) {
      if (++it > PATIENCE) return false;
      __builtin_amdgcn_s_sleep(1);
    }
    return (a.impatient & kind) == 0;
  };
  bool failed = false;                                 // this wave's patience ended

  // ---- this group's weights: thread t has candidates j0 + t + u * nt; in a shared selection, wave w also reads its part of the
  // largest weights of the head's chunks: 64w + l, 512 + 64w + l, ... in lane l, which is for head l % GP ----
  uint32_t e[U][G];                                    // bits of the weights, then softmax numerators
  auto ours = [&](int u) { return tid + u * nt < j1 - j0; };
  const int rows = MEAN ? U : (j1 - j0 + SEL_THREADS - 1) / SEL_THREADS;       // (in a group that is not whole one)
  auto each = [&](auto f) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!MEAN && u >= rows) break;
      f(u);
    }
  };
  float largest = -__builtin_inff();
  const int n_max = shared && soft ? a.chunks * (TAGGED ? 1 : SCAN_WAVES) * GP : 0;
  const size_t max0 = head * (TAGGED ? cmax_stride(a.max_pages) : cmax_plain_stride(a.max_pages));
  const int past = max(0, (lane & (GP - 1)) - (G - 1));        // (lanes of no head read the last one's)
  auto max_at = [&](int i) { return max0 + (i + tid < n_max ? i + tid : lane & (GP - 1)) - past; };
  // UC rows of candidates from row u0 on.  (All of a poll's loads are issued before the first is looked at: one trip.  Not all
  // rows at a time, because a word takes two registers.)
  auto weights = [&](auto from, auto uc) {
    constexpr int u0 = decltype(from)::value, UC = decltype(uc)::value;
    uint32_t at[UC];                                   // (a head's weights are less than 1 MiB)
#pragma unroll
    for (int u = 0; u < UC; ++u) at[u] = (uint32_t)min(j0 + tid + (u0 + u) * nt, j1 - 1);
    const uint32_t row = ng == 1 ? 0u : (uint32_t)a.max_pages;
    const size_t base = (size_t)head * G * a.max_pages + lo;
    if (TAGGED) {
      const bool maxima = u0 == 0 && n_max > 0;
      failed = !poll(WAIT_WEIGHTS | (maxima ? WAIT_MAXIMA : 0u), [&]() {
        uint32_t off = 0;                              // (not 0: a tag is another)
        unsigned long long w[UC][G], m = 0;
#pragma unroll
        for (int u = 0; u < UC; ++u)
#pragma unroll
          for (int gg = 0; gg < G; ++gg) w[u][gg] = ld_tag(a.P + base + (at[u] + gg * row));
        if (maxima) m = ld_tag(a.cmax + max_at(0));
#pragma unroll
        for (int u = 0; u < UC; ++u)
#pragma unroll
          for (int gg = 0; gg < G; ++gg) {
            e[u0 + u][gg] = (uint32_t)w[u][gg];
            off |= (uint32_t)(w[u][gg] >> 32) ^ tag;
          }
        if (maxima) {
          off |= (uint32_t)(m >> 32) ^ tag;
          largest = __uint_as_float((uint32_t)m);
        }
        return off == 0;
      }) || failed;
    } else {
#pragma unroll
      for (int u = 0; u < UC; ++u)
#pragma unroll
        for (int gg = 0; gg < G; ++gg) e[u0 + u][gg] = __float_as_uint((reinterpret_cast<const float*>(a.P) + base)[at[u] + gg * row]);
    }
  };
  static_assert(U == 1 || U == 2 || U == 4 || U == 8, "");
  if constexpr (!MEAN) {
    if (rows == 1) {
      weights(UnrollBy<0>{}, UnrollBy<1>{});
    } else if (rows == 2) {
      weights(UnrollBy<0>{}, UnrollBy<2>{});
    } else if constexpr (U == 8) {
      weights(UnrollBy<0>{}, UnrollBy<4>{});
      if (rows > 4) weights(UnrollBy<4>{}, UnrollBy<4>{});
    } else {
      weights(UnrollBy<0>{}, UnrollBy<2>{});
      weights(UnrollBy<2>{}, UnrollBy<2>{});
    }
  } else if constexpr (U == 1) {
    weights(UnrollBy<0>{}, UnrollBy<1>{});
  } else if constexpr (U == 2) {
    weights(UnrollBy<0>{}, UnrollBy<2>{});
  } else if constexpr (U == 4) {
    weights(UnrollBy<0>{}, UnrollBy<2>{});
    weights(UnrollBy<2>{}, UnrollBy<2>{});
  } else {
    weights(UnrollBy<0>{}, UnrollBy<4>{});
    if (4 * nt < j1 - j0) weights(UnrollBy<4>{}, UnrollBy<4>{});
    else
#pragma unroll
      for (int u = 4; u < U; ++u)
#pragma unroll
        for (int gg = 0; gg < G; ++gg) e[u][gg] = e[0][gg];
  }
  if (TAGGED) {
    for (int i = nt; i < n_max && !failed; i += nt) {
      unsigned long long m = 0;
      failed = !poll(WAIT_MAXIMA, [&]() { m = ld_tag(a.cmax + max_at(i)); return (uint32_t)(m >> 32) == tag; });
      largest = fmaxf(largest, __uint_as_float((uint32_t)m));
    }
  } else {
    for (int i = 0; i < n_max; i += 2 * nt)
      largest = fmaxf(largest, fmaxf(reinterpret_cast<const float*>(a.cmax)[max_at(i)], reinterpret_cast<const float*>(a.cmax)[max_at(i + nt)]));
  }
  FKV_STAMP(a, head, 2);

  // ---- fixed-point softmax: the head's maxima, numerators, integer denominators.  What the group's rows of 16 lanes have found goes
  // through LDS; eight lanes then put a query head's together (the lanes of no head repeat the last one's). ----
  TopkBins bins = kSoftBins;
  double zd[G], zr[G];
#pragma unroll
  for (int gg = 0; gg < G; ++gg) zd[gg] = zr[gg] = 1.0;
  const int of_row = wave * 4 + (lane >> 4), gl = min(lane >> 3, G - 1), wl = lane & 7;
  if (__builtin_expect(soft, 1)) {
    if (shared) {
      largest = __uint_as_float(class_reduce_row<GP>(__float_as_uint(largest), OpMaxF32()));
    } else {                                           // (a thread without a candidate repeats the last one)
      uint32_t v[GP];
#pragma unroll
      for (int gg = 0; gg < GP; ++gg) v[gg] = gg < G ? e[0][gg < G ? gg : 0] : 0u;
      each([&](int u) {
        if (u == 0) return;
#pragma unroll
        for (int gg = 0; gg < G; ++gg) v[gg] = OpMaxF32()(v[gg], e[u][gg]);
      });
      largest = __uint_as_float(class_fold_row<GP>(v, OpMaxF32()));
    }
    sm.mx_row[lane & (GP - 1)][of_row] = largest;
    lds_barrier();
    const float4 m4 = *reinterpret_cast<const float4*>(&sm.mx_row[gl][min(wl, nw - 1) * 4]);
    largest = __uint_as_float(reduce8(__float_as_uint(fmaxf(fmaxf(m4.x, m4.y), fmaxf(m4.z, m4.w))), OpMaxF32()));
    uint32_t zl[GP], zh[GP];                           // a thread's sums, in 16-bit halves (sums of a head's halves are below 2^32)
    typedef __attribute__((ext_vector_type(2))) unsigned short u16x2;
    float mx[G];
#pragma unroll
    for (int gg = 0; gg < GP; ++gg) zl[gg] = zh[gg] = 0;
#pragma unroll
    for (int gg = 0; gg < G; ++gg) mx[gg] = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(largest), gg * 8));
    each([&](int u) {
#pragma unroll
      for (int gg = 0; gg < G; ++gg) {
        const uint32_t en = softmax_fixed(__uint_as_float(e[u][gg]), mx[gg]);
        e[u][gg] = ours(u) ? en : 0u;
        const u16x2 c = __builtin_bit_cast(u16x2, e[u][gg]);
        zl[gg] = __builtin_amdgcn_udot2(c, u16x2{1, 0}, zl[gg], false);
        zh[gg] = __builtin_amdgcn_udot2(c, u16x2{0, 1}, zh[gg], false);
      }
    });
    // (a group's upper halves come to 2^28 at most if one of its waves has not seen its weights, else to 2^27)
    uint2 z = make_uint2(class_fold_row<GP>(zl, OpAddU32()), class_fold_row<GP>(zh, OpAddU32()));
    if (failed && lane < 16) z.y = kNoSum;
    sm.z_row[lane & (GP - 1)][of_row] = z;
    lds_barrier();
    const uint4* const z8 = reinterpret_cast<const uint4*>(&sm.z_row[gl][min(wl, nw - 1) * 4]);
    const uint4 za = z8[0], zb = z8[1];
    z = make_uint2((za.x + za.z) + (zb.x + zb.z), (za.y + za.w) + (zb.y + zb.w));
    z = make_uint2(reduce8(wl < nw ? z.x : 0u, OpAddU32()), reduce8(wl < nw ? z.y : 0u, OpAddU32()));
    if (__builtin_expect(__ballot(z.y >= kNoSum) != 0, 0)) return Selected::NOTHING;
    if (shared) {                                      // ... and over the slices: lane 8g + r reads slice r's, r's and r + 8's
      // (a sum of all slices side by side, as they are read)
      unsigned long long* const every = a.exch + (size_t)head * EXCH_WORDS + gl * MAX_SLICES;
      constexpr int UPPER = MAX_G * MAX_SLICES;
      if (wave == 0 && wl == 0 && lane < 8 * G) {
        st_tag(every + s, z.x, tag, a.home);
        st_tag(every + UPPER + s, z.y, tag, a.home);
      }
      const unsigned long long* const p0 = every + min(wl, S - 1);
      const unsigned long long* const p1 = every + min(wl + 8, S - 1);
      unsigned long long w[4];
      failed = !poll(WAIT_SUMS, [&]() {
        w[0] = ld_tag(p0); w[1] = ld_tag(p0 + UPPER); w[2] = ld_tag(p1); w[3] = ld_tag(p1 + UPPER);
        return ((((uint32_t)(w[0] >> 32) ^ tag) | ((uint32_t)(w[1] >> 32) ^ tag)) | (((uint32_t)(w[2] >> 32) ^ tag) | ((uint32_t)(w[3] >> 32) ^ tag))) == 0;
      });
      const bool two = wl + 8 < S;
      z = make_uint2((uint32_t)w[0] + (two ? (uint32_t)w[2] : 0u), (uint32_t)w[1] + (two ? (uint32_t)w[3] : 0u));
      z = make_uint2(reduce8(wl < S ? z.x : 0u, OpAddU32()), reduce8(wl < S ? z.y : 0u, OpAddU32()));
    }
    // one reciprocal per query head
    const double zv = (double)(((unsigned long long)z.y << 16) + z.x), yv = reciprocal_near(zv);
#pragma unroll
    for (int gg = 0; gg < G; ++gg) {
      zd[gg] = lane_f64(zv, gg * 8);
      zr[gg] = lane_f64(yv, gg * 8);
    }
  } else {
    float most = -__builtin_inff();                    // weight: no score is above it (a thread without a candidate repeats the last one)
    each([&](int u) {
#pragma unroll
      for (int gg = 0; gg < G; ++gg) most = fmaxf(most, __uint_as_float(e[u][gg]));
    });
    sm.mx[wave][0] = wave_max_f32(most);
    if (lane == 0) sm.failed[wave] = failed ? 1 : 0;
    lds_barrier();
    if (__builtin_expect(__ballot(sm.failed[min(lane, nw - 1)] != 0) != 0, 0)) return Selected::NOTHING;        // (and the histogram is clear)
    bins = bins_below(score_key(wave_max_f32(sm.mx[min(lane, nw - 1)][0])));
    if (tid == 0) sm.bins = bins;
  }

  // what the other groups hand on to the last one, and the rows that takes
  unsigned long long* const keyx = a.keyx + (size_t)head * a.max_pages;
  unsigned long long* const keyid = a.keyid + (size_t)head * a.max_pages;
  const int m = handed_on(S, a.slice, kk);
  const bool all = m == a.slice;                       // (then a key's place says whose it is)
  const int others = shared && last ? (S - 1) * m : 0, X = (others + SEL_THREADS - 1) / SEL_THREADS;      // (a group that has others is whole)
  const bool fits = X <= SEL_OTHERS;

  // ---- pooled scores -> keys (0: no candidate) ----
  uint32_t key[U];
  if (!MEAN) {
#pragma unroll
    for (int u = 0; u < U; ++u) key[u] = 0;
  }
  each([&](int u) {
    const uint32_t ku = score_key(MEAN ? mean_score<G>(e[u], zd, zr) : pooled_score<G>(e[u], zd, zr, mode));
    key[u] = ours(u) ? ku : 0u;
  });
  auto id = [&](int u) { return lo + j0 + tid + u * nt; };
  auto store_scores = [&]() {                          // (kept for inspection: nobody waits for them)
    each([&](int u) {
      if (ours(u)) a.score[(size_t)head * a.max_pages + id(u)] = key_score(key[u]);
    });
  };
  if (shared && !last && all) {
    each([&](int u) {
      if (ours(u) && !failed) st_tag(keyx + id(u) - lo, key[u], tag, a.home);
    });
    store_scores();
    return failed ? Selected::NOTHING : Selected::IDS;
  }
  auto count = [&](uint32_t k, bool there) { atomicAdd(&sm.hist[there ? topk_bin(k, bins) : (uint32_t)(TOPK_BINS + lane)], 1u); };
  each([&](int u) {
    count(key[u], ours(u));
    if (shared && !fits && ours(u)) key_lds[others + tid + u * nt] = key[u];
  });
  uint32_t key_of[SEL_OTHERS];                         // the other groups'
  int id_of[SEL_OTHERS];
#pragma unroll
  for (int x = 0; x < SEL_OTHERS; ++x) { key_of[x] = 0; id_of[x] = 0; }
  if (shared) {
    if (fits) {
      if (X > 0) {
        unsigned long long w[SEL_OTHERS][2];
        const bool ok = poll(WAIT_KEYS, [&]() {
          uint32_t off = 0;
#pragma unroll
          for (int x = 0; x < SEL_OTHERS; ++x) w[x][0] = ld_tag(keyx + min(tid + min(x, X - 1) * SEL_THREADS, others - 1));
          if (!all) {
#pragma unroll
            for (int x = 0; x < SEL_OTHERS; ++x) w[x][1] = ld_tag(keyid + min(tid + min(x, X - 1) * SEL_THREADS, others - 1));
          }
#pragma unroll
          for (int x = 0; x < SEL_OTHERS; ++x) off |= (uint32_t)(w[x][0] >> 32) ^ tag;
          if (!all) {
#pragma unroll
            for (int x = 0; x < SEL_OTHERS; ++x) off |= (uint32_t)(w[x][1] >> 32) ^ tag;
          }
          return off == 0;
        });
        failed = failed || !ok;
#pragma unroll
        for (int x = 0; x < SEL_OTHERS; ++x) {
          const bool there = tid + x * SEL_THREADS < others;
          key_of[x] = there ? (uint32_t)w[x][0] : 0u;
          id_of[x] = all ? lo + tid + x * SEL_THREADS : (int)(uint32_t)w[x][1];
          if (x < X) count(key_of[x], there);
        }
      }
    } else {
      for (int i0 = tid; i0 - lane < others && !failed; i0 += 4 * nt) {
        unsigned long long w[4][2];
        failed = !poll(WAIT_KEYS, [&]() {
          bool there = true;
#pragma unroll
          for (int x = 0; x < 4; ++x) w[x][0] = ld_tag(keyx + min(i0 + x * nt, others - 1));
          if (!all) {
#pragma unroll
            for (int x = 0; x < 4; ++x) w[x][1] = ld_tag(keyid + min(i0 + x * nt, others - 1));
          }
#pragma unroll
          for (int x = 0; x < 4; ++x) there = there & ((uint32_t)(w[x][0] >> 32) == tag);
          if (!all) {
#pragma unroll
            for (int x = 0; x < 4; ++x) there = there & ((uint32_t)(w[x][1] >> 32) == tag);
          }
          return there;
        });
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          if (i0 + x * nt < others) {
            key_lds[i0 + x * nt] = (uint32_t)w[x][0];
            atomicAdd(&sm.hist[topk_bin((uint32_t)w[x][0], bins)], 1u);
          }
        }
      }
    }
    if (failed) sm.alone = 1;
  }
  lds_barrier();
  if (shared && __builtin_expect(__builtin_amdgcn_readfirstlane(sm.alone) != 0, 0)) return Selected::NOTHING;
  FKV_STAMP(a, head, 5);
  if (SHARED && __builtin_expect(!fits, 0)) {
    store_scores();
    return Selected::KEYS;
  }
  const PutId put(a, head, key_lds);
  bool done;
  if (!shared) {
    done = topk_items<!MEAN, U>(key, rows, 0, n, kk, bins, nw, sm, [&](int u, unsigned long long chosen, int pos) {
      if (__builtin_amdgcn_inverse_ballot_w64(chosen)) put(pos, id(u));
    });
    // (few keys of the last bin in a short list: still shorter than by way of block_topk -- 70 candidates, 48 wanted, most of them with
    // next to no weight, 8.6 and 7.1 us a layer-step)
    if (MEAN && U == 1 && __builtin_expect(!done, 0))
      done = topk_items<true, U>(key, 1, 0, n, kk, bins, nw, sm, [&](int u, unsigned long long chosen, int pos) {
        if (__builtin_amdgcn_inverse_ballot_w64(chosen)) put(pos, id(u));
      });
  } else if (!last) {
    done = topk_items<!MEAN, U>(key, rows, 0, j1 - j0, kk, bins, nw, sm, [&](int u, unsigned long long chosen, int pos) {
      if (__builtin_amdgcn_inverse_ballot_w64(chosen)) {
        st_tag(keyx + s * m + pos, key[u], tag, a.home);
        st_tag(keyid + s * m + pos, (uint32_t)id(u), tag, a.home);
      }
    });
  } else {                                             // the others' rows, then the group's own
    auto choose = [&](auto xc) {
      constexpr int XR = decltype(xc)::value, T = XR + (U < SEL_REGS ? U : SEL_REGS);     // (a slice's rows)
      uint32_t item[T];
#pragma unroll
      for (int u = 0; u < T; ++u) item[u] = u < XR ? key_of[u < XR ? u : 0] : key[u < XR ? 0 : u - XR];
      return topk_items<!MEAN, XR>(item, X, rows, others + j1 - j0, kk, bins, nw, sm, [&](int u, unsigned long long chosen, int pos) {
        if (__builtin_amdgcn_inverse_ballot_w64(chosen)) put(pos, u < XR ? id_of[u < XR ? u : 0] : id(u < XR ? 0 : u - XR));
      });
    };
    done = MEAN && X <= 1 ? choose(UnrollBy<1>{}) : choose(UnrollBy<SEL_OTHERS>{});
  }
  store_scores();
  if (__builtin_expect(done, 1)) return Selected::IDS;
  each([&](int u) {
    if (ours(u)) key_lds[others + tid + u * nt] = key[u];
  });
#pragma unroll
  for (int x = 0; x < SEL_OTHERS; ++x)
    if (tid + x * SEL_THREADS < others) key_lds[tid + x * SEL_THREADS] = key_of[x];
  lds_barrier();
  return Selected::KEYS;
}
// The method's own scores by the rows of candidates that a thread has: each is straight code then (a test of the pooling beside every row
// and of the rows in use beside every phase cost 0.6 to 1 us of what topk_items says).  The other poolings have kernels of their own.
// again(): the arguments once more, from memory: what several ways have in common would be worked out ahead of them all and kept in lanes of
// vector registers, of which a host pool's kernels have none to spare (with it for lists of one block too, 8 heads x 97 and 480 candidates
// 6.63 and 6.92 us a layer-step, so 6.51 and 6.82, and the step kernel has no scratch memory up to G = 6 but for fp16 G = 4).
// Where the ways and their polls start within 64 bytes is worth up to 10 % where few blocks have a list on units that are otherwise
// idle (page_select of one head x 5000 candidates 10.5 to 11.7 us with code ahead of it that is not run, 10.6 aligned; layer-steps of one to
// four heads x 1700 to 8160 candidates 1 % longer without, 1.5 % shorter so).
template <int G, bool TAGGED, bool MEAN, typename Again>
__device__ __forceinline__ Selected select_rows(const StepArgs& a, int head, int s, int nw, int mine, uint32_t* key, SelectLds& sm, Again again) {
  constexpr int REGS = sel_regs_alone(G);
  const int nt = nw * 64;
  if constexpr (!MEAN) return select_group<G, TAGGED, false, true, REGS>(a, head, s, nw, key, sm);
  if (a.slices > 1) {
    if (mine <= nt) return select_group<G, TAGGED, true, true, 1>(again(), head, s, nw, key, sm);
    if (mine <= 2 * nt) return select_group<G, TAGGED, true, true, 2>(again(), head, s, nw, key, sm);
    return select_group<G, TAGGED, true, true, SEL_REGS>(again(), head, s, nw, key, sm);
  }
  if (mine <= nt) return select_group<G, TAGGED, true, false, 1>(again(), head, s, nw, key, sm);
  if (mine <= 2 * nt) return select_group<G, TAGGED, true, false, 2>(again(), head, s, nw, key, sm);
  if (REGS == 4 || mine <= 4 * nt) return select_group<G, TAGGED, true, false, 4>(again(), head, s, nw, key, sm);
  return select_group<G, TAGGED, true, false, REGS>(again(), head, s, nw, key, sm);
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
      st_tag(a.P + base + (size_t)gg * a.max_pages + j, __float_as_uint(weight_alone<DT, G>(a, head, gg, j)), tag, a.home);
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
    atomicAdd(&sm.hist[topk_bin(kj, kSoftBins)], 1u);
  }
  lds_barrier();
}

// Selecting block `s` of a head.  True for the waves that go on with select_finish -- the last block's, nw of them, and another's
// that has its choice still to make -- and `got`: how far they are.
template <int G, bool TAGGED, bool MEAN, typename Again>
__device__ __forceinline__ bool select_begin(const StepArgs& a, int head, int s, uint32_t* key, int& nw, Selected& got, Again again) {
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = a.slices, j0 = s * a.slice, j1 = min(a.g.n_cand, j0 + a.slice);
  const bool last = s == S - 1;
  // The waves that take part: as many as there are candidates for; all of them where a plan has to be made or the best of
  // other slices have to be gathered.  The others of the block end here (a barrier counts the waves that are left).
  nw = (last && S > 1) || a.plan_new_slots || a.g.k_eff == 0 ? SEL_WAVES : min(SEL_WAVES, (j1 - j0 + 63) / 64);
  got = Selected::IDS;
  if (wave >= nw) return false;
  if (a.g.k_eff == 0) return true;
  // What the end of the chain needs of the arguments is read now, while the weights are waited for
  // (0.3 us of a layer-step of 8 to 20 us).
  got = (Selected)__builtin_amdgcn_readfirstlane((int)select_rows<G, TAGGED, MEAN>(a, head, s, nw, j1 - j0, key, select_lds(), again));
  return last || got == Selected::KEYS;
}

// ... and what is left after it, by nw waves: the ids where they are not out yet, the recall plan.  again(): the arguments once
// more, from memory, for what is hardly ever run (kept up to here they would cost the rest its scalar registers).
template <int DT, int G, bool TAGGED, typename Again>
__device__ __forceinline__ void select_finish(const StepArgs& hot, int head, int s, uint32_t* key, int nw, Selected got, Again again) {
  SelectLds& sm = select_lds();
  const int tid = threadIdx.x, nt = nw * 64;
  if (__builtin_expect(hot.g.k_eff > 0 && got != Selected::IDS, 0)) {
    const StepArgs a = again();
    const int n = a.g.n_cand, lo = a.g.cand_lo, kk = a.g.k_eff;
    const uint32_t tag = launch_tag(a.no);
    const PutId put(a, head, key);
    const bool alone = got == Selected::NOTHING;
    if (alone) {
      if (tid == 0) atomicAdd(a.by_itself, 1);
      alone_keys<DT, G, TAGGED>(a, head, nw, key, sm);
      for (int j = tid; j < n; j += nt) a.score[(size_t)head * a.max_pages + lo + j] = key_score(key[j]);
    }
    // the keys in LDS: every candidate's, or what the other groups handed on and then this one's
    const bool last = alone || s == a.slices - 1;
    const int j0 = alone ? 0 : s * a.slice, m = handed_on(a.slices, a.slice, kk), others = last && !alone ? (a.slices - 1) * m : 0;
    unsigned long long* const keyid = a.keyid + (size_t)head * a.max_pages;
    block_topk(key, last ? others + n - j0 : a.slice, kk, alone || a.sel_pool <= 1 ? kSoftBins : sm.bins, nw, sm, [&](int pos, int j) {
      const int id = j >= others ? lo + j0 + j - others : m == a.slice ? lo + j : (int)(uint32_t)ld_tag(keyid + j);
      if (last) { put(pos, id); return; }
      st_tag(a.keyx + (size_t)head * a.max_pages + s * m + pos, key[j], tag, a.home);
      st_tag(keyid + s * m + pos, (uint32_t)id, tag, a.home);
    });
    if (!last) return;
  }
  const StepArgs& a = hot;
  const int kk = a.g.k_eff, k = a.k;
  const uint32_t tag = launch_tag(a.no);
  const PutId put(a, head, key);
  for (int i = kk + tid; i < k; i += nt) put(i, -1);      // padding
  if (put.plan_nid) {
    int32_t* const plan_sm = reinterpret_cast<int32_t*>(key) + a.plan_lds_off;
    lds_barrier();                                       // the ids are all in LDS
    plan_head<SEL_THREADS>(put.out, a.plan_act_ids + (size_t)head * k, a.plan_act_slots + (size_t)head * k,
                           a.plan_new_slots + (size_t)head * k, a.plan_miss + (size_t)head * (1 + 3 * k), k, a.g.n_full,
                           plan_sm, true);
    const int32_t* nslot = plan_sm + 5 * k;
    for (int i = tid; i < k; i += SEL_THREADS) {
      const int id = put.plan_nid[i], sl = nslot[i];
      if (put.tagw) st_tag(put.tagw + i, tagged_pick(id, sl & (TAGGED_MAX_SLOTS - 1), (sl & PLAN_MISS_BIT) != 0), tag, a.home);
      put.out[i] = id;
      if (put.outu) put.outu[i] = id;
    }
  }
  FKV_STAMP(a, head, 8);
}

// ---------------------------------------------------------------------------------
// role dispatch of one block: row y of the grid counts [append][correction test][scoring ...][selection ...], each
// present only if its role bit is set; x is the KV head -- at home, the grid is a multiple of 8 wide -- except that the
// selection's blocks are numbered through row by row and dealt to the heads (deal_block; they wait for each other).
// ---------------------------------------------------------------------------------
// select(head, slice): what a selecting block does.  (Its code last: with it ahead of the scoring's a launch took 0.2 us longer.)
template <int DT, int G, bool PAST, typename Select>
__device__ __forceinline__ void step_roles(const StepArgs& a, int x, int y, Select select) {
  const bool there = x < a.heads;
  if (a.roles & ROLE_APPEND) {
    if (y == 0) { if (there) append_role<DT>(a, x); return; }
    y -= 1;
  }
  if (a.roles & ROLE_CORR) {
    if (y == 0) { if (there) corr_role<DT, G>(a, x); return; }
    y -= 1;
  }
  if (y < a.chunks) {
    if (!there) return;
    if (y == 0) FKV_STAMP(a, x, 0);
    score_role<DT, G, true, STEP_WAVES, PAST>(a, x, y);
    if (y == 0) FKV_STAMP(a, x, 1);
    return;
  }
  const int wide = a.home ? (a.heads + 7) & ~7 : a.heads;
  int head, s;
  deal_block((uint32_t)((y - a.chunks) * wide + x), a.slices, a.home, [&](uint32_t j) { return j >> a.slices_log2; }, head, s);
  if (head < a.heads) select(head, s);
}

// ---------------------------------------------------------------------------------
// grid (heads -- at home, the next multiple of 8 -- , rows): rows as in step_roles.  HOME is known when this is compiled because a
// launch is a chain of a few microseconds and the test beside every store that other blocks wait for costs it 0.1 to 0.3 of them
// (8 heads x 992 candidates 8.2 us with the test, 8.0 without; at home 7.6 and 7.5).  MEAN: the method's pooling, or any other (select_rows).
// ---------------------------------------------------------------------------------
template <int DT, int G, bool MEAN, bool PAST, bool HOME>
__global__ __launch_bounds__(STEP_THREADS) void step_kernel(StepArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint32_t dyn_lds[];              // selection: n_cand keys, then the recall plan
  touch_args<sizeof(StepArgs)>();
  a.home = HOME;
  if (MEAN) a.sel_pool = 0;
  step_roles<DT, G, PAST>(a, blockIdx.x, blockIdx.y, [&](int head, int s) {
    int nw;
    Selected got;
    const auto again = [] {
      StepArgs b = args_from_memory<StepArgs>();
      b.home = HOME;
      if (MEAN) b.sel_pool = 0;
      return b;
    };
    if (select_begin<G, true, MEAN>(a, head, s, dyn_lds, nw, got, again)) select_finish<DT, G, true>(a, head, s, dyn_lds, nw, got, again);
  });
}

template <int DT, int G, bool MEAN, bool PAST, bool HOME>
static bool launch_step_kernel_g(const StepArgs& a, int rows, size_t lds, hipStream_t st) {
  static size_t granted = 48 * 1024;
  if (!grant_lds(&step_kernel<DT, G, MEAN, PAST, HOME>, lds, granted)) return false;
  step_kernel<DT, G, MEAN, PAST, HOME><<<dim3(HOME ? by_xcd(a.heads) : a.heads, rows), STEP_THREADS, lds, st>>>(a);
  return true;
}

// one of these in each of the files that share the kernel's variants
template <bool MEAN, bool HOME>
static bool launch_step_kernel_variant(const StepArgs& a, int dtype, int G, bool past, int rows, size_t lds, hipStream_t st) {
  switch (G) {
#define FKV_CASE(GG) case GG: return dtype == 0 ? (past ? launch_step_kernel_g<0, GG, MEAN, true, HOME>(a, rows, lds, st) : launch_step_kernel_g<0, GG, MEAN, false, HOME>(a, rows, lds, st)) \
                                                : (past ? launch_step_kernel_g<1, GG, MEAN, true, HOME>(a, rows, lds, st) : launch_step_kernel_g<1, GG, MEAN, false, HOME>(a, rows, lds, st));
    FKV_CASE(1) FKV_CASE(2) FKV_CASE(3) FKV_CASE(4) FKV_CASE(5) FKV_CASE(6) FKV_CASE(7) FKV_CASE(8)
#undef FKV_CASE
    default: return false;
  }
}
bool launch_step_kernel(const StepArgs& a, int dtype, int G, bool past, int rows, size_t lds, hipStream_t st);        // a head's blocks adjacent
bool launch_step_kernel_home(const StepArgs& a, int dtype, int G, bool past, int rows, size_t lds, hipStream_t st);   // ... on one XCD
bool launch_step_kernel_pool(const StepArgs& a, int dtype, int G, bool past, int rows, size_t lds, hipStream_t st);   // the same for a.sel_pool != 0
bool launch_step_kernel_pool_home(const StepArgs& a, int dtype, int G, bool past, int rows, size_t lds, hipStream_t st);

}  // namespace fkv
