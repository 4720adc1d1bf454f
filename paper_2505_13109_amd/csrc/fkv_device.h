// Device-side helpers shared by the kernel files.
#pragma once
#include "fkv_internal.h"

namespace fkv {

// 16 bytes, or the same past the caches
typedef __attribute__((ext_vector_type(4))) uint32_t word4;
__device__ __forceinline__ uint4 load_past(const uint16_t* p) {
  return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const word4*>(p)));
}

// one storage element / a packed pair of them -> fp32 (exact)
template <int DT> struct Unpack;
template <> struct Unpack<0> {   // fp16
  static __device__ __forceinline__ float one(uint16_t b) { return (float)__builtin_bit_cast(_Float16, b); }
  static __device__ __forceinline__ float lo(uint32_t w) { return one((uint16_t)(w & 0xffffu)); }
  static __device__ __forceinline__ float hi(uint32_t w) { return one((uint16_t)(w >> 16)); }
};
template <> struct Unpack<1> {   // bf16
  static __device__ __forceinline__ float one(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
  static __device__ __forceinline__ float lo(uint32_t w) { return __uint_as_float(w << 16); }
  static __device__ __forceinline__ float hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
};
template <int DT>
__device__ __forceinline__ void unpack8(const uint4& w, float* f) {
  f[0] = Unpack<DT>::lo(w.x); f[1] = Unpack<DT>::hi(w.x);
  f[2] = Unpack<DT>::lo(w.y); f[3] = Unpack<DT>::hi(w.y);
  f[4] = Unpack<DT>::lo(w.z); f[5] = Unpack<DT>::hi(w.z);
  f[6] = Unpack<DT>::lo(w.w); f[7] = Unpack<DT>::hi(w.w);
}

__device__ __forceinline__ int resident_unit(const PoolDesc& pd, int page) {
  if (pd.placement == 0) return page;
  return page < pd.ring_base ? page : pd.ring_base + page % pd.n_ring;
}
__device__ __forceinline__ size_t head_base(const PoolDesc& pd, int b, int m, int n_kv) {
  return (size_t)(b * n_kv + m) * pd.units_per_head;
}
__device__ __forceinline__ size_t summ_idx(int b, int m, int n_kv, int which, int max_pages, int page) {
  return ((size_t)((b * n_kv + m) * 2 + which) * max_pages + page) * D;
}

// Brings BYTES at p into the scalar cache, which starts every launch empty, in one round trip: fetched where they are first
// needed they are a miss for every 64 bytes, one after the other along the chain.
template <int BYTES>
__device__ __forceinline__ void touch(const __attribute__((address_space(4))) void* p) {
  constexpr int LINES = (BYTES + 63) / 64;
  static_assert(LINES <= 8, "");
  auto line = [](int i) constexpr { return (i < LINES ? i : LINES - 1) * 64; };
  // one statement, with its wait: the register the loads go to is nobody else's while they are under way
  uint32_t t;
  asm volatile("s_load_dword %0, %1, %2\n\ts_load_dword %0, %1, %3\n\ts_load_dword %0, %1, %4\n\ts_load_dword %0, %1, %5\n\t"
               "s_load_dword %0, %1, %6\n\ts_load_dword %0, %1, %7\n\ts_load_dword %0, %1, %8\n\ts_load_dword %0, %1, %9\n\t"
               "s_waitcnt lgkmcnt(0)"
               : "=&s"(t)
               : "s"(p), "n"(line(0)), "n"(line(1)), "n"(line(2)), "n"(line(3)), "n"(line(4)), "n"(line(5)), "n"(line(6)), "n"(line(7))
               : "memory");
}

// the same for a kernel's own arguments, of which the first use of each line would wait for it alone
template <int BYTES>
__device__ __forceinline__ void touch_args() {
  touch<BYTES>((const __attribute__((address_space(4))) void*)__builtin_amdgcn_kernarg_segment_ptr());
}

// The same arguments (T: all of them, as one struct) once more from memory.  What this reads does not have to be kept in
// registers up to here, and the compiler, which knows nothing about the pointer, cannot decide to.
template <typename T>
__device__ __forceinline__ T args_from_memory() {
  typedef const __attribute__((address_space(4))) unsigned long long* WordPtr;
  WordPtr p = (WordPtr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  static_assert(sizeof(T) % 8 == 0, "");
  struct Words { unsigned long long w[sizeof(T) / 8]; } v;
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 8); ++i) v.w[i] = p[i];
  return __builtin_bit_cast(T, v);
}

// correction flag of a KV head from the similarities of its G query heads (Sec. 3.3): the
// group-pooled similarity strictly below tau.  pool: 0 mean (sum in head order / G), 1 maximum,
// 2 minimum (App. B.3).  fp64, one thread.
__device__ __forceinline__ int pooled_flag(const double* c, int G, float tau, int pool) {
  double acc = c[0];
  for (int gg = 1; gg < G; ++gg) {
    const double v = c[gg];
    if (pool == 0) acc = acc + v;
    else if (pool == 1) acc = v > acc ? v : acc;
    else acc = v < acc ? v : acc;
  }
  if (pool == 0) acc = acc / (double)G;
  return acc < (double)tau ? 1 : 0;
}

// ---- wavefront reductions on the DPP cross-lane path (no LDS traffic) ------------------
// xor-1, xor-2 inside quads, then half-row and row mirrors: every lane of a 16-lane row ends
// with the row's result; two row broadcasts carry it on, lane 63 holds the wave's result.
template <typename OP>
__device__ __forceinline__ uint32_t wave_reduce_u32(uint32_t v, OP op) {
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, false));   // quad_perm [1,0,3,2]
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, false));   // quad_perm [2,3,0,1]
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, false));  // row_half_mirror
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xf, 0xf, false));  // row_mirror
  // row_bcast:15 into rows 1 and 3, row_bcast:31 into rows 2 and 3; lanes not written keep v
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)OP::identity(), (int)v, 0x142, 0xa, 0xf, false));
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)OP::identity(), (int)v, 0x143, 0xc, 0xf, false));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
struct OpMaxF32 {   // on bit patterns of floats
  static __device__ __forceinline__ uint32_t identity() { return 0xff800000u; }   // -inf
  __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const {
    return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b)));
  }
};
struct OpAddF32 {   // on bit patterns of floats
  static __device__ __forceinline__ uint32_t identity() { return 0u; }
  __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return __float_as_uint(__uint_as_float(a) + __uint_as_float(b)); }
};
struct OpAddU32 {
  static __device__ __forceinline__ uint32_t identity() { return 0u; }
  __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return a + b; }
};
__device__ __forceinline__ float wave_max_f32(float v) {
  return __uint_as_float(wave_reduce_u32(__float_as_uint(v), OpMaxF32()));
}
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) { return wave_reduce_u32(v, OpAddU32()); }
// ---- reductions over the lanes that are equal modulo M (1, 2, 4, 8): every lane ends with its class's result ----------
// (in a quad by permutation, in a row of 16 lanes by rotation, over the rows by the row-swapping moves)
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false); }
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_ROR4 = 0x124, DPP_ROR8 = 0x128, DPP_HALF_MIRROR = 0x141;
// a lane's value, for all of them
__device__ __forceinline__ unsigned long long lane_u64(unsigned long long v, int lane) {
  return (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane) << 32 | (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
}
__device__ __forceinline__ double lane_f64(double v, int lane) {
  return __builtin_bit_cast(double, lane_u64(__builtin_bit_cast(unsigned long long, v), lane));
}
// ... of a row of 16 lanes, and of the wave
template <int M, typename OP>
__device__ __forceinline__ uint32_t class_reduce_row(uint32_t v, OP op) {
  static_assert(M == 1 || M == 2 || M == 4 || M == 8, "");
  if (M <= 1) v = op(v, dpp_u32<DPP_XOR1>(v));
  if (M <= 2) v = op(v, dpp_u32<DPP_XOR2>(v));
  if (M <= 4) v = op(v, dpp_u32<DPP_ROR4>(v));
  return op(v, dpp_u32<DPP_ROR8>(v));
}
template <int M, typename OP>
__device__ __forceinline__ uint32_t class_reduce(uint32_t v, OP op) {
  v = class_reduce_row<M>(v, op);
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = op(a[0], a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return op(b[0], b[1]);
}
// over eight adjacent lanes: every lane ends with their result
template <typename OP>
__device__ __forceinline__ uint32_t reduce8(uint32_t v, OP op) {
  v = op(v, dpp_u32<DPP_XOR1>(v));
  v = op(v, dpp_u32<DPP_XOR2>(v));
  return op(v, dpp_u32<DPP_HALF_MIRROR>(v));
}
// sum over the wave of values below 2^48, as two sums of 24-bit halves so that no 32-bit lane sum overflows
__device__ __forceinline__ unsigned long long wave_sum_u48(unsigned long long v) {
  return (unsigned long long)class_reduce<1>((uint32_t)(v & 0xffffffu), OpAddU32()) + ((unsigned long long)class_reduce<1>((uint32_t)(v >> 24), OpAddU32()) << 24);
}
// v[g]: a lane's value for class g.  Lane l ends with op over its row's lanes of v[l % M].  A step that joins two lanes also halves the
// classes that each of them goes on with.
template <int M, typename OP>
__device__ __forceinline__ uint32_t class_fold_row(const uint32_t (&v)[M], OP op) {
  const uint32_t lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  uint32_t x[M];
#pragma unroll
  for (int i = 0; i < M; ++i) x[i] = v[i];
  if constexpr (M >= 2) {
    const bool up = lane & 1u;
#pragma unroll
    for (int i = 0; i < M / 2; ++i) x[i] = op(up ? x[2 * i + 1] : x[2 * i], dpp_u32<DPP_XOR1>(up ? x[2 * i] : x[2 * i + 1]));
  }
  if constexpr (M >= 4) {
    const bool up = lane & 2u;
#pragma unroll
    for (int i = 0; i < M / 4; ++i) x[i] = op(up ? x[2 * i + 1] : x[2 * i], dpp_u32<DPP_XOR2>(up ? x[2 * i] : x[2 * i + 1]));
  }
  if constexpr (M >= 8) {
    const bool up = lane & 4u;                          // (a rotation by 4 flips this bit)
    x[0] = op(up ? x[1] : x[0], dpp_u32<DPP_ROR4>(up ? x[0] : x[1]));
  }
  return class_reduce_row<M>(x[0], op);
}

// sum of an fp64 value over the wave, valid in lane 63 (a DPP step moves the two halves)
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64(double v) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROWS, 0xf, false);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double wave_sum_f64(double v) {
  v += dpp_f64<0xB1, 0xf>(v);
  v += dpp_f64<0x4E, 0xf>(v);
  v += dpp_f64<0x141, 0xf>(v);
  v += dpp_f64<0x140, 0xf>(v);
  v += dpp_f64<0x142, 0xa>(v);     // (rows that receive nothing add +0)
  v += dpp_f64<0x143, 0xc>(v);
  return v;
}

// inclusive prefix sum across the 64 lanes (Hillis-Steele inside 16-lane rows, then two row broadcasts)
__device__ __forceinline__ uint32_t wave_scan_u32(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);   // row_shr:1, 0 shifted in
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);   // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);   // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);   // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // rows 1,3 += total of rows 0,2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // rows 2,3 += total of lanes 0..31
  return v;
}

// cosine of one query head against the previous step's query (Sec. 3.1), fp64: one wave, lane l holds channels 2l and
// 2l+1 of both; the result is lane 63's
template <int DT>
__device__ __forceinline__ double cosine_of(uint32_t qw, uint32_t pw) {
  const double a0 = (double)Unpack<DT>::lo(qw), a1 = (double)Unpack<DT>::hi(qw);
  const double p0 = (double)Unpack<DT>::lo(pw), p1 = (double)Unpack<DT>::hi(pw);
  const double dot = wave_sum_f64(a0 * p0 + a1 * p1), na = wave_sum_f64(a0 * a0 + a1 * a1), nb = wave_sum_f64(p0 * p0 + p1 * p1);
  const double den = sqrt(na * nb);
  return den > 0.0 ? dot / den : 0.0;
}

// The same in fp32, within 1e-5 of it (each sum of 128 products is off by less than 1e-6 of the product of the norms), or
// NaN where a norm is outside the range in which that holds: for a decision that only needs the exact value when it is
// close.  A tenth of the instructions: no fp64 move pairs, square root or division.
__device__ __forceinline__ float wave_sum_f32(float v) {     // valid in lane 63
  v += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0xB1, 0xf, 0xf, false));
  v += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0x4E, 0xf, 0xf, false));
  v += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0x141, 0xf, 0xf, false));
  v += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0x140, 0xf, 0xf, false));
  v += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0x142, 0xa, 0xf, false));
  v += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0x143, 0xc, 0xf, false));
  return v;
}
template <int DT>
__device__ __forceinline__ float near_cosine_of(uint32_t qw, uint32_t pw) {
  const float a0 = Unpack<DT>::lo(qw), a1 = Unpack<DT>::hi(qw), p0 = Unpack<DT>::lo(pw), p1 = Unpack<DT>::hi(pw);
  const float dot = wave_sum_f32(a0 * p0 + a1 * p1), na = wave_sum_f32(a0 * a0 + a1 * a1), nb = wave_sum_f32(p0 * p0 + p1 * p1);
  const bool ok = na > 1e-15f && na < 1e15f && nb > 1e-15f && nb < 1e15f;
  return ok ? dot * __builtin_amdgcn_rsqf(na * nb) : __builtin_nanf("");
}
// The correction flag from such values: 0 or 1 where they decide it, -1 where the pooled one is too close to tau.
__device__ __forceinline__ int near_flag(const float* c, int G, float tau, int pool) {
  float acc = c[0];
  if (pool == 0) {
#pragma unroll
    for (int gg = 1; gg < MAX_G; ++gg) acc = acc + (gg < G ? c[gg] : 0.0f);
    acc = acc * __builtin_amdgcn_rcpf((float)G);
  } else {
    for (int gg = 1; gg < G; ++gg) {
      const float v = c[gg];
      acc = v != v || (pool == 1 ? v > acc : v < acc) ? v : acc;
    }
  }
  const float d = acc - tau;
  return d < -1e-4f ? 1 : d > 1e-4f ? 0 : -1;
}

// ---- exchange between blocks of one launch ---------------------------------------
// Each XCD has its own L2, and one does not see what is in another's.  A device-scope fence per block would write back and
// invalidate the whole L2 each time; instead each value that is exchanged goes by itself, as a relaxed atomic: into the L2
// where its readers are on the writer's XCD, through to memory where they are not (st_tag).

// A picked page as one 32-bit value, for the exchange between the selecting block and waiting attention waves when the
// KV lives in a host pool: page id (< 2^16), page-cache slot (< 2^15), and whether the slot has yet to be filled from
// the host pool; all ones: no page at this position.
constexpr int TAGGED_MAX_PAGES = 1 << 16, TAGGED_MAX_SLOTS = 1 << 15;
__device__ __forceinline__ uint32_t tagged_pick(int id, int slot, bool miss) {
  return id < 0 ? 0xffffffffu : ((miss ? 0x80000000u : 0u) | ((uint32_t)slot << 16) | (uint32_t)id);
}
__device__ __forceinline__ void tagged_unpick(uint32_t w, int& id, int& slot, bool& miss) {
  if (w == 0xffffffffu) { id = -1; slot = -1; miss = false; return; }
  id = (int)(w & 0xffffu);
  slot = (int)((w >> 16) & 0x7fffu);
  miss = (w >> 31) != 0;
}

// Which head block i of a section of a launch's blocks works for, and which of the head's n it is.  Blocks go to the 8 XCDs in
// turn, by their number in the launch.  At home: heads by 8, each on an XCD of its own, so that what a head's blocks tell each
// other stays in that XCD's L2 (the section has to start at a multiple of 8; what is beyond the last head is nobody's).
// Else a head's blocks are adjacent, over all XCDs.  At home at most one head's blocks per XCD, else one's per launch, are ever half
// there.
// div: i -> i / n.
template <typename Div>
__device__ __forceinline__ void deal_block(uint32_t i, int n, bool home, Div div, int& head, int& own) {
  const uint32_t j = home ? i >> 3 : i, h = div(j);
  own = (int)(j - h * (uint32_t)n);
  head = (int)(home ? h * 8 + (i & 7u) : h);
}

// A value exchanged between blocks of one launch without a counter: one 64-bit word holding the value and a tag that no
// earlier writer of that word used (a launch number), written and read in one piece.  A reader that sees the tag has the value:
// no acknowledgement to wait for, no counter to bump, no second read.  Measured on this chip: one way 0.22 us in an L2 and
// 0.3 to 0.5 through memory, where store / counter / read takes 0.3 us (store acknowledged) + 0.4 (atomic) + 0.6 (read).
// home: a head's blocks are all on one XCD (deal_block), so the word only has to be in that XCD's L2, where it stays till the
// launch ends; else it is written through to memory.  Readers go past their L1 in either case, which is all there is between
// them and the L2, so they need not know.  (A store at work-group scope that other work-groups read is more than the memory model
// promises; it is what this machine does.  A word that could not be seen would be a wait that runs out, PATIENCE, and is counted,
// LayerStatus.)
__device__ __forceinline__ void st_tag(unsigned long long* p, uint32_t value, uint32_t tag, bool home) {
  const unsigned long long w = ((unsigned long long)tag << 32) | value;
  if (home) __hip_atomic_store(p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else      __hip_atomic_store(p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long ld_tag(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t launch_tag(const LaunchNo& n) { return n.dev ? device_tag((uint32_t)*n.dev) : n.tag; }
// A wait between blocks of a launch ends by itself only if the block waited for gets to run, and whether it does is not this
// launch's to decide: other launches may hold the compute units, with waits of their own.  So nothing depends on it: a block
// whose patience ends makes what it waits for itself, from what was in memory before the launch, bit for bit what the other
// block would have made, and goes on (and its compute unit is free again soon).
// Polls: 0.7 ms where a wave waits for ids, 2 ms where a thread waits for sums (0.17 and 0.5 us a turn; in a launch by
// itself a wait takes microseconds).  Blocks of a launch that fetches pages from a host pool wait for one another's transfers
// too, and to do without them is expensive there: eight times as long.
constexpr int PATIENCE = 1 << 12, PATIENCE_HOST = 8 * PATIENCE;
// Polls before a thread gives up on words that its block has written by then (10 ms): that many only if a test sees to it.
constexpr int MAX_POLLS = 1 << 16;

// threadIdx.x once more, from the wave's number in a scalar register: what is worked out from this after a stretch of code that
// needs every vector register does not have to be kept through it.
__device__ __forceinline__ int thread_id(int wave) {
  uint32_t t = (uint32_t)wave * 64 + __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  asm volatile("" : "+v"(t));
  __builtin_assume(t < 1024);
  return (int)t;
}

// A barrier that orders the block's LDS accesses and nothing else: global loads stay in flight across it, and no store's
// acknowledgement is waited for.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

}  // namespace fkv
