// route_impl.h — register-resident routing passes of bucket ORP
// (Algorithm 3.1 of Asharov et al., SOSA 2020) for gfx950.
//
// Same method and same results as orp_pass_kernel (orp_kernels.hip): one
// launch runs `klev` fused butterfly levels over blocks of 2^klev buckets, every
// MergeSplit a tight-compaction network over the 2Z slots of its two buckets
// (marks = reals whose next label bit is 0 plus the first Z - x dummies, the
// dummy tagging of Section 4.1; network = the offset-compaction recursion of
// Sasy, Johnson and Goldberg, CCS 2022).  This version is specialised on
// log2 Z so that every stage is unrolled with compile-time register pairs:
//
//   * A MergeSplit's 2Z slots live in the registers of 2Z/16 lanes, 16 slots
//     per lane.  In layout A lane l holds positions q = 16 l + e (e = 0..15):
//     stages over q bits 0..3 pair registers, stages over q bits 4 and 5 pair
//     lanes l and l^1 / l^2 through DPP quad permutes.  In layout B a lane holds
//     the 16 positions whose q bits LQ-4..LQ-1 vary (LQ = log2 2Z), so the
//     remaining stages pair registers again.  Each level therefore moves the
//     data through LDS twice: A -> B, and B -> next level's A (whose MergeSplits
//     pair other buckets).  At Z = 512 a MergeSplit is one wave: A -> B stays in
//     the wave's own LDS words (no barrier), and between levels a wave keeps one
//     of its buckets and hands the other to the wave it is paired with, half
//     the traffic.
//   * Blocks are persistent: a workgroup walks over several blocks of buckets,
//     and several workgroups share a CU, so one workgroup's HBM loads overlap
//     the others' networks.  Barriers wait for LDS traffic only.
//
// What bounds a pass (n = 2^28 records of 8 bytes, Z = 512): HBM at k = 3 (2.94
// ms for a middle pass, 4.4 TB/s of the 4.9 a copy reaches; 3.91 ms with the
// compare-and-select networks of v_cmp and v_cndmask); at k = 4 the networks and
// their LDS exchanges (3.46 ms, 3.8 before the wave-local exchanges), which
// still makes the fewer passes the faster sort.  The first pass of four levels
// takes 2.82 ms (the labels, and networks for three levels), the last 4.2 (and a
// compaction per bin).
//
// Obliviousness: every HBM and LDS address is a function of (n, Z, klev,
// level, block, lane, register) only; labels and records steer register
// selects, never an address.
#pragma once
#include "bos_common.h"

#include <type_traits>

namespace bos {

namespace route_detail {

constexpr uint32_t kDppXor1 = 0xB1;  // quad_perm [1,0,3,2]
constexpr uint32_t kDppXor2 = 0x4E;  // quad_perm [2,3,0,1]
constexpr uint32_t kDppB0022 = 0xA0; // quad_perm [0,0,2,2]
constexpr uint32_t kDppB1133 = 0xF5; // quad_perm [1,1,3,3]
constexpr uint32_t kDppB0000 = 0x00; // quad_perm [0,0,0,0]
constexpr uint32_t kDppB2222 = 0xAA; // quad_perm [2,2,2,2]

// Barrier that waits for this wave's LDS operations only (global loads issued
// earlier remain in flight).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
}

// Orders this wave's LDS writes before its later LDS reads.  Enough when the
// lanes that exchange data through LDS all belong to one wave: LDS executes a
// wave's instructions in order.
__device__ __forceinline__ void lds_wave_sync() {
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_wave_barrier();
}

// Keeps the compiler from moving this wave's LDS accesses across; the LDS
// unit runs a wave's accesses in order, so its lanes need no wait between a
// write and the read of another lane's word.
__device__ __forceinline__ void lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// LDS exchange among `LANES` consecutive lanes (a power of two): a wave-local
// wait when they fit in one wave, a workgroup barrier otherwise.
template <uint32_t LANES>
__device__ __forceinline__ void lds_group_sync() {
  if constexpr (LANES <= 64u) lds_wave_sync();
  else lds_barrier();
}

template <uint32_t CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
  return uint32_t(__builtin_amdgcn_mov_dpp(int(v), CTRL, 0xF, 0xF, false));
}
template <uint32_t CTRL>
__device__ __forceinline__ uint2 dpp(uint2 v) {
  return make_uint2(dpp<CTRL>(v.x), dpp<CTRL>(v.y));
}
template <uint32_t CTRL>
__device__ __forceinline__ uint4 dpp(uint4 v) {
  return make_uint4(dpp<CTRL>(v.x), dpp<CTRL>(v.y), dpp<CTRL>(v.z), dpp<CTRL>(v.w));
}

__device__ __forceinline__ uint2 rec_and(uint2 v, uint32_t m) { return make_uint2(v.x & m, v.y & m); }
__device__ __forceinline__ uint4 rec_and(uint4 v, uint32_t m) {
  return make_uint4(v.x & m, v.y & m, v.z & m, v.w & m);
}

__device__ __forceinline__ uint32_t brev_k(uint32_t x, uint32_t k) { return k ? (__brev(x) >> (32u - k)) : 0u; }

// Halves of a record for two-half LDS exchanges (8 bytes of a 16-byte
// record, 4 of an 8-byte one).
__device__ __forceinline__ uint2 rec_lo(uint4 v) { return make_uint2(v.x, v.y); }
__device__ __forceinline__ uint2 rec_hi(uint4 v) { return make_uint2(v.z, v.w); }
__device__ __forceinline__ void set_lo(uint4& v, uint2 l) {
  v.x = l.x;
  v.y = l.y;
}
__device__ __forceinline__ void set_hi(uint4& v, uint2 h) {
  v.z = h.x;
  v.w = h.y;
}
__device__ __forceinline__ uint32_t rec_lo(uint2 v) { return v.x; }
__device__ __forceinline__ uint32_t rec_hi(uint2 v) { return v.y; }
__device__ __forceinline__ void set_lo(uint2& v, uint32_t l) { v.x = l; }
__device__ __forceinline__ void set_hi(uint2& v, uint32_t h) { v.y = h; }
// 32-bit word w of a record.
__device__ __forceinline__ uint32_t rec_word(const uint2& v, uint32_t w) { return w == 0 ? v.x : v.y; }
__device__ __forceinline__ uint32_t rec_word(const uint4& v, uint32_t w) {
  return w == 0 ? v.x : w == 1 ? v.y : w == 2 ? v.z : v.w;
}
__device__ __forceinline__ void set_word(uint2& v, uint32_t w, uint32_t x) {
  if (w == 0) v.x = x;
  else v.y = x;
}
__device__ __forceinline__ void set_word(uint4& v, uint32_t w, uint32_t x) {
  if (w == 0) v.x = x;
  else if (w == 1) v.y = x;
  else if (w == 2) v.z = x;
  else v.w = x;
}
template <typename T> struct HalfOf;
template <> struct HalfOf<uint4> {
  using H = uint2;
  static __device__ __forceinline__ H zero() { return make_uint2(0u, 0u); }
};
template <> struct HalfOf<uint2> {
  using H = uint32_t;
  static __device__ __forceinline__ H zero() { return 0u; }
};

// Swap rule of the compaction network.  A node of 2*half slots starts at marks
// prefix P0 and has prefix Ph at its middle; the recursion of Sasy, Johnson
// and Goldberg swaps the pair at offset i when s != (i >= t), with z = P0 mod
// 2*half, mm = Ph - P0, t = (z + mm) mod half and s = (z mod half + mm >= half)
// != (z >= half).  Since z + mm = Ph (mod 2*half), t and s are the low and the
// high part of Ph mod 2*half, and the rule is one bit: the pair is swapped when
// bit log2(half) of Ph - 1 - i is set.  Prefixes are therefore kept as Ph - 1,
// shifted left so that this bit is the sign bit ("scaled"), and a decision is
// one subtraction and one arithmetic shift, a mask of all ones or zeros.
//
// The masks drive v_bitop3_b32 selects.  gfx950 issues the vector instructions
// of two waves of a SIMD together when at least one of them is a "light" one:
// measured with 4 waves per SIMD, v_bitop3, v_add/v_sub, v_and/v_or/v_xor and
// right shifts take 2.4 cycles each, while v_cmp, v_cndmask, v_min, v_bfe,
// left shifts and every DPP form take 4.5 on their own.  A conditional swap of
// three words is 8 light instructions (17.5 cycles) and was v_cmp, a scalar
// xor and 6 v_cndmask (28-30).
//
// The oldest wave wins arbitration, so a wave that runs light instructions
// alone keeps a wave that waits at a heavy one out, and nothing issues
// together until the first one stalls (8 heavy + 24 light instructions: 3.9
// cycles each).  Raising a wave's priority while it runs its heavy ones (2.3
// cycles each) lets it pass: kernels built on these networks run at priority
// 1 and drop to 0 inside runs of light instructions (light_begin, light_end).
__device__ __forceinline__ void light_begin() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_setprio(0);
}
__device__ __forceinline__ void light_end() {
  __builtin_amdgcn_s_setprio(1);
  __builtin_amdgcn_sched_barrier(0);
}
// The shift amounts and the bit come from registers the compiler cannot see
// through: with constants it folds these shifts into v_bfe_i32 or v_cmp and
// v_cndmask.
__device__ __forceinline__ uint32_t opaque31() {
  uint32_t s;
  asm("v_mov_b32 %0, 31" : "=v"(s));
  return s;
}
__device__ __forceinline__ uint32_t opaque1() {
  uint32_t s;
  asm("v_mov_b32 %0, 1" : "=v"(s));
  return s;
}
__device__ __forceinline__ uint32_t sign_mask(uint32_t d) { return uint32_t(int32_t(d) >> opaque31()); }
// Mask of bit 0 of x.
__device__ __forceinline__ uint32_t low_bit_mask(uint32_t x) { return 0u - (x & opaque1()); }
// Per bit: m ? a : b.
__device__ __forceinline__ uint32_t msel(uint32_t m, uint32_t a, uint32_t b) {
  return __builtin_amdgcn_bitop3_b32(m, a, b, 0xCA);
}
__device__ __forceinline__ uint2 msel(uint32_t m, uint2 a, uint2 b) {
  return make_uint2(msel(m, a.x, b.x), msel(m, a.y, b.y));
}
__device__ __forceinline__ uint4 msel(uint32_t m, uint4 a, uint4 b) {
  return make_uint4(msel(m, a.x, b.x), msel(m, a.y, b.y), msel(m, a.z, b.z), msel(m, a.w, b.w));
}
// Exchange (a, ta) and (b, tb) where m is set.
template <typename T>
__device__ __forceinline__ void mswap(uint32_t m, T& a, uint32_t& ta, T& b, uint32_t& tb) {
  const T na = msel(m, b, a), nb = msel(m, a, b);
  const uint32_t nta = msel(m, tb, ta), ntb = msel(m, ta, tb);
  a = na;
  b = nb;
  ta = nta;
  tb = ntb;
}

// Stages on slot bits 0..3 of a lane's 16 consecutive slots (register pairs);
// pm[e] = prefix - 1 at slot e of the lane.  Slot e is the middle of exactly
// one node, of half 2^ctz(e).
template <typename T>
__device__ __forceinline__ void lane_stages(T (&rv)[16], uint32_t (&tv)[16], const uint32_t (&pm)[16]) {
  uint32_t q[16];
#pragma unroll
  for (uint32_t e = 0; e < 16; ++e) q[e] = (e & 1u) ? pm[e] : pm[e] << (31u - __builtin_ctz(e | 16u));
  light_begin();
#pragma unroll
  for (uint32_t eb = 0; eb < 4; ++eb) {
    const uint32_t half = 1u << eb;
#pragma unroll
    for (uint32_t es = 0; es < 16; es += 2u * half) {
#pragma unroll
      for (uint32_t i = 0; i < half; ++i) {
        const uint32_t m = eb == 0 ? low_bit_mask(q[es | half]) : sign_mask(q[es | half] - (i << (31u - eb)));
        mswap(m, rv[es + i], tv[es + i], rv[es + i + half], tv[es + i + half]);
      }
    }
  }
  light_end();
}

// One stage between lanes: slot e of this lane and of its partner lane (DPP
// control CTRL) swap where bit 31 of q - e * step is set.  The partners' words
// of four slots are fetched (heavy), then selected (light).
template <uint32_t CTRL, typename T>
__device__ __forceinline__ void dpp_stage(T (&rv)[16], uint32_t (&tv)[16], uint32_t q, uint32_t step) {
#pragma unroll
  for (uint32_t e0 = 0; e0 < 16; e0 += 4) {
    T pr[4];
    uint32_t pt[4];
#pragma unroll
    for (uint32_t e = 0; e < 4; ++e) {
      pr[e] = dpp<CTRL>(rv[e0 + e]);
      pt[e] = dpp<CTRL>(tv[e0 + e]);
    }
    light_begin();
#pragma unroll
    for (uint32_t e = 0; e < 4; ++e) {
      const uint32_t m = sign_mask(q - (e0 + e) * step);
      rv[e0 + e] = msel(m, pr[e], rv[e0 + e]);
      tv[e0 + e] = msel(m, pt[e], tv[e0 + e]);
    }
    light_end();
  }
}

// Scaled prefix of lane lt's first slot (slot 16 lt of the node tree), the
// middle of the node of half 2^(4 + ctz(lt)); top = the tree's lane count.
__device__ __forceinline__ uint32_t lane_prefix(uint32_t pm0, uint32_t lt, uint32_t top) {
  return pm0 << (27u - uint32_t(__builtin_ctz(lt | top)));
}

// DPP source with lanes outside the pattern (or rows outside ROW_MASK)
// reading 0.
template <uint32_t CTRL, uint32_t ROW_MASK = 0xF>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v) {
  return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), CTRL, ROW_MASK, 0xF, true));
}

// Inclusive scan over aligned groups of W lanes (W a power of two <= 64):
// row_shr steps inside rows of 16 lanes, then row broadcasts across rows.
template <uint32_t W>
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x, uint32_t lane) {
  constexpr uint32_t kRowShr = 0x110, kRowBcast15 = 0x142, kRowBcast31 = 0x143;
  if constexpr (W >= 2) {
    const uint32_t y = dpp_or_zero<kRowShr + 1>(x);
    x += (W >= 16 || (lane & (W - 1u)) >= 1u) ? y : 0u;
  }
  if constexpr (W >= 4) {
    const uint32_t y = dpp_or_zero<kRowShr + 2>(x);
    x += (W >= 16 || (lane & (W - 1u)) >= 2u) ? y : 0u;
  }
  if constexpr (W >= 8) {
    const uint32_t y = dpp_or_zero<kRowShr + 4>(x);
    x += (W >= 16 || (lane & (W - 1u)) >= 4u) ? y : 0u;
  }
  if constexpr (W >= 16) x += dpp_or_zero<kRowShr + 8>(x);
  if constexpr (W >= 32) x += dpp_or_zero<kRowBcast15, 0xA>(x);  // row 0 -> row 1, row 2 -> row 3
  if constexpr (W >= 64) x += dpp_or_zero<kRowBcast31, 0xC>(x);  // lane 31 -> rows 2 and 3
  return x;
}

// Exclusive scan over aligned segments of SEG lanes (SEG a power of two).
template <uint32_t SEG>
__device__ __forceinline__ uint32_t seg_scan(uint32_t v, uint32_t* swave, uint32_t* total) {
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  constexpr uint32_t W = SEG < 64u ? SEG : 64u;
  const uint32_t x = wave_incl_scan<W>(v, lane);
  if constexpr (SEG <= 64u) {
    if constexpr (W == 64u)
      *total = uint32_t(__builtin_amdgcn_readlane(int(x), 63));
    else
      *total = __shfl(x, int(lane | (W - 1u)), 64);
    return x - v;
  } else {
    if (lane == 63u) {
      BOS_TR(0, 9, wave);
      swave[wave] = x;
    }
    lds_barrier();
    constexpr uint32_t WPS = SEG / 64u;
    const uint32_t w0 = wave & ~(WPS - 1u);
    uint32_t pre = 0, tot = 0;
#pragma unroll
    for (uint32_t q = 0; q < WPS; ++q) {
      BOS_TR(0, 9, w0 + q);
      const uint32_t t = swave[w0 + q];
      if (w0 + q < wave) pre += t;
      tot += t;
    }
    *total = tot;
    return pre + x - v;
  }
}

}  // namespace route_detail
using namespace route_detail;

// ---- per-bin finish of the last pass (Section 3.2) ---------------------------
//
// Each final bin (Z slots in LDS, padded by one slot per 16) is sorted by a
// bitonic network held in registers: lane lq of the bin's Z/16 lanes holds
// slots 16 lq + e (layout P; stages on slot bits 0..3 pair registers, bits 4
// and 5 pair lanes through DPP).  Stages on slot bits >= 6 run in layout Q,
// where a lane holds the 16 slots whose top four bits vary.  Sort keys:
// record order with dummies last (bos_sort, and the first half of the
// random permutation of bos_orp), then (r, p) with dummies last, r the 64-bit
// Philox key of the p-th real in record order (bos_orp).

// Sort elements.  Dummies are given the maximal record (record order) or the
// maximal key (random-key order), so that comparing keys alone puts them
// last; a real element can only tie with a dummy when both are byte-identical,
// where either order gives the same output bytes.
template <typename T>
struct ElemR {  // a record
  T r;
};
template <typename T>
struct ElemRK {  // a record with its 64-bit random key and rank p (0xFFFF for dummies)
  T r;
  uint32_t klo, khi, aux;
};

template <typename T>
__device__ __forceinline__ bool e_less(const ElemR<T>& a, const ElemR<T>& b) {
  return rec_less(a.r, b.r);
}
template <typename T>
__device__ __forceinline__ bool e_less(const ElemRK<T>& a, const ElemRK<T>& b) {
  const uint64_t ka = (uint64_t(a.khi) << 32) | a.klo, kb = (uint64_t(b.khi) << 32) | b.klo;
  return ka < kb || (ka == kb && a.aux < b.aux);
}
template <typename T>
__device__ __forceinline__ ElemR<T> e_sel(bool c, const ElemR<T>& a, const ElemR<T>& b) {
  return ElemR<T>{sel(c, a.r, b.r)};
}
template <uint32_t CTRL, typename T>
__device__ __forceinline__ ElemR<T> e_dpp(const ElemR<T>& a) {
  return ElemR<T>{dpp<CTRL>(a.r)};
}
template <uint32_t CTRL, typename T>
__device__ __forceinline__ ElemRK<T> e_dpp(const ElemRK<T>& a) {
  return ElemRK<T>{dpp<CTRL>(a.r), dpp<CTRL>(a.klo), dpp<CTRL>(a.khi), dpp<CTRL>(a.aux)};
}

// A record as the words that order it: one 64-bit word (key << 32 | payload)
// for 8-byte records, (key, payload) for 16-byte ones.
template <int R> struct FRec;
template <> struct FRec<8> {
  uint64_t k;
};
template <> struct FRec<16> {
  uint64_t k, p;
};
__device__ __forceinline__ bool f_less(const FRec<8>& a, const FRec<8>& b) { return a.k < b.k; }
__device__ __forceinline__ bool f_less(const FRec<16>& a, const FRec<16>& b) {
  return (a.k < b.k) | ((a.k == b.k) & (a.p < b.p));
}
__device__ __forceinline__ FRec<8> f_load(const uint2& r) { return {(uint64_t(r.x) << 32) | r.y}; }
__device__ __forceinline__ FRec<16> f_load(const uint4& r) {
  return {uint64_t(r.x) | (uint64_t(r.y) << 32), uint64_t(r.z) | (uint64_t(r.w) << 32)};
}
__device__ __forceinline__ uint2 f_store(const FRec<8>& f) { return make_uint2(uint32_t(f.k >> 32), uint32_t(f.k)); }
__device__ __forceinline__ uint4 f_store(const FRec<16>& f) {
  return make_uint4(uint32_t(f.k), uint32_t(f.k >> 32), uint32_t(f.p), uint32_t(f.p >> 32));
}
template <int R> __device__ __forceinline__ FRec<R> f_max();
template <> __device__ __forceinline__ FRec<8> f_max<8>() { return {~0ull}; }
template <> __device__ __forceinline__ FRec<16> f_max<16>() { return {~0ull, ~0ull}; }

template <int R>
struct FE1 {  // sort element: a record in record order
  FRec<R> r;
};
template <int R>
__device__ __forceinline__ bool e_less(const FE1<R>& a, const FE1<R>& b) { return f_less(a.r, b.r); }
__device__ __forceinline__ uint64_t msel64(uint32_t m, uint64_t a, uint64_t b) {
  return (uint64_t(msel(m, uint32_t(a >> 32), uint32_t(b >> 32))) << 32) | msel(m, uint32_t(a), uint32_t(b));
}
__device__ __forceinline__ FRec<8> f_msel(uint32_t m, const FRec<8>& a, const FRec<8>& b) {
  return {msel64(m, a.k, b.k)};
}
__device__ __forceinline__ FRec<16> f_msel(uint32_t m, const FRec<16>& a, const FRec<16>& b) {
  return {msel64(m, a.k, b.k), msel64(m, a.p, b.p)};
}
template <int R>
__device__ __forceinline__ FE1<R> e_msel(uint32_t m, const FE1<R>& a, const FE1<R>& b) {
  return {f_msel(m, a.r, b.r)};
}
template <uint32_t CTRL>
__device__ __forceinline__ uint64_t dpp64(uint64_t v) {
  return uint64_t(dpp<CTRL>(uint32_t(v))) | (uint64_t(dpp<CTRL>(uint32_t(v >> 32))) << 32);
}
template <uint32_t CTRL>
__device__ __forceinline__ FE1<8> e_dpp(const FE1<8>& a) { return {{dpp64<CTRL>(a.r.k)}}; }
template <uint32_t CTRL>
__device__ __forceinline__ FE1<16> e_dpp(const FE1<16>& a) { return {{dpp64<CTRL>(a.r.k), dpp64<CTRL>(a.r.p)}}; }

// LDS views of the bins (padded slot index)
// (tw: the trace buffer its accesses fold into in the digest build: 0 for
// the routing and the per-bin finish, 1 for the comparison sort)
template <typename T>
struct LdsR {
  T* rec;
  uint32_t tw = 0;
  __device__ ElemR<T> ld(uint32_t i) const {
    BOS_TR(tw, 4, i);
    return ElemR<T>{rec[i]};
  }
  __device__ void st(uint32_t i, const ElemR<T>& v) const {
    BOS_TR(tw, 4, i);
    rec[i] = v.r;
  }
};
template <int R>
struct LdsF {  // the ordering words themselves: no conversion between layouts
  FRec<R>* rec;
  uint32_t tw = 0;
  __device__ FE1<R> ld(uint32_t i) const {
    BOS_TR(tw, 4, i);
    return FE1<R>{rec[i]};
  }
  __device__ void st(uint32_t i, const FE1<R>& v) const {
    BOS_TR(tw, 4, i);
    rec[i] = v.r;
  }
};
template <typename T>
struct LdsRK {
  T* rec;
  uint32_t* klo;
  uint32_t* khi;
  uint16_t* aux;
  uint32_t tw = 0;
  __device__ ElemRK<T> ld(uint32_t i) const {
    BOS_TR(tw, 17, i);
    return ElemRK<T>{rec[i], klo[i], khi[i], aux[i]};
  }
  __device__ void st(uint32_t i, const ElemRK<T>& v) const {
    BOS_TR(tw, 17, i);
    rec[i] = v.r;
    klo[i] = v.klo;
    khi[i] = v.khi;
    aux[i] = uint16_t(v.aux);
  }
};

template <typename T>
__device__ __forceinline__ ElemR<T> e_msel(uint32_t m, const ElemR<T>& a, const ElemR<T>& b) {
  return ElemR<T>{msel(m, a.r, b.r)};
}
template <typename T>
__device__ __forceinline__ ElemRK<T> e_msel(uint32_t m, const ElemRK<T>& a, const ElemRK<T>& b) {
  return ElemRK<T>{msel(m, a.r, b.r), msel(m, a.klo, b.klo), msel(m, a.khi, b.khi), msel(m, a.aux, b.aux)};
}
// c ? a : b of whole elements, by a word mask
template <typename E>
__device__ __forceinline__ E e_pick(bool c, const E& a, const E& b) {
  if constexpr (std::is_same_v<E, ElemR<uint2>>) return e_sel(c, a, b);
  else return e_msel(c ? ~0u : 0u, a, b);
}

// One stage on register pairs (e, e | HB) of a lane; asc(e): the pair sorts
// ascending.  All comparisons first (heavy), then the selects on word masks
// (light, see above): 16.1 cycles per pair of 64-bit words measured against
// 20.5 with each comparison followed by its v_cndmask.  (Tiles of 8-byte
// records keep the v_cndmask form, ElemR<uint2>: with four waves a SIMD, three
// barriers a phase and LDS busy 58 % of the time the light form took 2.34 ms
// for 2^28 records and that one 2.18; 16-byte tiles 0.385 ms for 2^24 records
// and 0.426.)  Equal elements are byte-identical, so swapping them or not is
// the same.
template <uint32_t HB, typename E, typename ASC>
__device__ __forceinline__ void cx_stage(E (&v)[16], ASC asc) {
  if constexpr (std::is_same_v<E, ElemR<uint2>>) {
#pragma unroll
    for (uint32_t i = 0; i < 8; ++i) {
      const uint32_t e = ((i & ~(HB - 1u)) << 1) | (i & (HB - 1u));
      const bool sw = e_less(v[e | HB], v[e]) == asc(e);
      const E x = e_sel(sw, v[e | HB], v[e]), y = e_sel(sw, v[e], v[e | HB]);
      v[e] = x;
      v[e | HB] = y;
    }
    return;
  }
  bool sw[8];
#pragma unroll
  for (uint32_t i = 0; i < 8; ++i) {
    const uint32_t e = ((i & ~(HB - 1u)) << 1) | (i & (HB - 1u));
    sw[i] = e_less(v[e | HB], v[e]) == asc(e);
  }
  light_begin();
#pragma unroll
  for (uint32_t i = 0; i < 8; ++i) {
    const uint32_t e = ((i & ~(HB - 1u)) << 1) | (i & (HB - 1u));
    const uint32_t m = sw[i] ? ~0u : 0u;
    const E x = e_msel(m, v[e | HB], v[e]), y = e_msel(m, v[e], v[e | HB]);
    v[e] = x;
    v[e | HB] = y;
  }
  light_end();
}
template <uint32_t CTRL, typename E>
__device__ __forceinline__ void cx_lane(E& x, bool is_lo, bool asc) {
  const E p = e_dpp<CTRL>(x);
  const bool take = e_less(p, x) == (is_lo == asc);
  x = e_pick(take, p, x);
}

// Bitonic sort (ascending) of every bin; v holds layout P on entry and exit.
// bbase: padded LDS offset of this lane's bin; lq: lane within the bin.
// Phases KK = 1..LZ (merges of 2^KK slots), stages JJ = KK-1..0 (slot bit JJ);
// all indices are template parameters so every register index is static.
struct BinLane {
  uint32_t bbase, pbase, lq, lb0, lb1, lowQ;
  bool active;  // lanes past the block's bins hold no bin and touch no LDS
};

template <int LZ, int KK>
__device__ __forceinline__ bool asc_p(uint32_t e, const BinLane& bl) {
  if constexpr (KK == LZ) return true;
  else if constexpr (KK < 4) return ((e >> KK) & 1u) == 0u;
  else return ((bl.lq >> (KK - 4)) & 1u) == 0u;
}
template <int LZ, int KK>
__device__ __forceinline__ bool asc_q(uint32_t e, const BinLane& bl) {
  if constexpr (KK == LZ) return true;
  else if constexpr (KK >= LZ - 4) return ((e >> (KK - (LZ - 4))) & 1u) == 0u;
  else if constexpr (KK == LZ - 5) return bl.lb1 == 0u;  // lane bits of layout Q (Z >= 2048)
  else return bl.lb0 == 0u;
}

template <int LZ, int KK, int JJ, typename E>
__device__ __forceinline__ void p_stages(E (&v)[16], const BinLane& bl) {
  if constexpr (JJ >= 0) {
    if constexpr (JJ < 4) {
      cx_stage<(1u << JJ)>(v, [&](uint32_t e) { return asc_p<LZ, KK>(e, bl); });
    } else if constexpr (JJ == 4) {
      const bool asc = asc_p<LZ, KK>(0, bl);
#pragma unroll
      for (uint32_t e = 0; e < 16; ++e) cx_lane<kDppXor1>(v[e], bl.lb0 == 0u, asc);
    } else {
      const bool asc = asc_p<LZ, KK>(0, bl);
#pragma unroll
      for (uint32_t e = 0; e < 16; ++e) cx_lane<kDppXor2>(v[e], bl.lb1 == 0u, asc);
    }
    p_stages<LZ, KK, JJ - 1>(v, bl);
  }
}

template <int LZ, int KK, int JJ, typename E>
__device__ __forceinline__ void q_stages(E (&v)[16], const BinLane& bl) {
  if constexpr (JJ >= 6) {
    if constexpr (JJ >= LZ - 4) {
      cx_stage<(1u << (JJ - (LZ - 4)))>(v, [&](uint32_t e) { return asc_q<LZ, KK>(e, bl); });
    } else if constexpr (JJ == LZ - 5) {  // lane bit 1 of layout Q (2^LZ >= 2048)
#pragma unroll
      for (uint32_t e = 0; e < 16; ++e) cx_lane<kDppXor2>(v[e], bl.lb1 == 0u, asc_q<LZ, KK>(e, bl));
    } else {  // lane bit 0 of layout Q (2^LZ = 4096)
      static_assert(JJ == LZ - 6, "layout Q covers slot bits >= LZ-6");
#pragma unroll
      for (uint32_t e = 0; e < 16; ++e) cx_lane<kDppXor1>(v[e], bl.lb0 == 0u, asc_q<LZ, KK>(e, bl));
    }
    q_stages<LZ, KK, JJ - 1>(v, bl);
  }
}

template <int LZ, int KK, typename E, typename V>
__device__ __forceinline__ void bitonic_phase(E (&v)[16], const V& lds, const BinLane& bl) {
  if constexpr (KK <= LZ) {
    if constexpr (KK - 1 >= 6) {
      // layout Q for the stages on slot bits KK-1 .. 6
      if (bl.active) {
#pragma unroll
        for (uint32_t e = 0; e < 16; ++e) lds.st(bl.pbase + e, v[e]);
      }
      lds_group_sync<(1u << LZ) / 16u>();  // a bin's lanes
      if (bl.active) {
#pragma unroll
        for (uint32_t e = 0; e < 16; ++e) {
          const uint32_t sl = (e << (LZ - 4)) | bl.lowQ;
          v[e] = lds.ld(bl.bbase + sl + (sl >> 4));
        }
      }
      q_stages<LZ, KK, KK - 1>(v, bl);
      if (bl.active) {
#pragma unroll
        for (uint32_t e = 0; e < 16; ++e) {
          const uint32_t sl = (e << (LZ - 4)) | bl.lowQ;
          lds.st(bl.bbase + sl + (sl >> 4), v[e]);
        }
      }
      lds_group_sync<(1u << LZ) / 16u>();
      if (bl.active) {
#pragma unroll
        for (uint32_t e = 0; e < 16; ++e) v[e] = lds.ld(bl.pbase + e);
      }
    }
    p_stages<LZ, KK, (KK - 1 < 5 ? KK - 1 : 5)>(v, bl);
    bitonic_phase<LZ, KK + 1>(v, lds, bl);
  }
}

template <int LZ, typename E, typename V>
__device__ __forceinline__ void bin_bitonic(E (&v)[16], const V& lds, uint32_t bbase, uint32_t lq, bool active) {
  BinLane bl;
  bl.active = active;
  bl.bbase = bbase;
  bl.pbase = bbase + 17u * lq;  // layout P: slots 16 lq .. 16 lq + 15
  bl.lq = lq;
  bl.lb0 = lq & 1u;
  bl.lb1 = (lq >> 1) & 1u;
  const uint32_t rest = lq >> 2;
  // layout Q pairs lanes through DPP only for Z = 2048; otherwise lanes take
  // consecutive slots
  bl.lowQ = LZ >= 11 ? ((bl.lb1 << (LZ - 5)) | (bl.lb0 << (LZ - 6)) | rest) : (LZ >= 6 ? lq : 0u);
  bitonic_phase<LZ, 1>(v, lds, bl);
}

// Per-bin finish of the last pass (Section 3.2): every final bin (LDS bucket
// S, padded slots) is sorted in record order with its dummies (maximal
// record) last, and for fin == 0 then permuted uniformly: the p-th real of
// global bin gb gets the key r(gb*Z + p), word (g mod 4) of Philox block g/4
// with key (seed, 1), and the bin is sorted by (key, p).  On return outr holds
// this lane's 16 slots of its bin (slots 16 lq .. 16 lq + 15) and `load` the
// bin's real count; reals occupy the bin's first `load` slots.  FIN: 0 =
// choose by a.fin at run time, 1 = sort only, 2 = sort and permute.  FULL:
// every lane of the workgroup holds slots (no lane guards).
template <int R, int LZ, int FIN, bool FULL>
__device__ __forceinline__ void sort_bins(const PassArgs& a, uint64_t blk, uint32_t klev,
                                          typename RecOf<R>::T* srec, uint32_t* stag, uint32_t* srhi,
                                          uint16_t* saux, const uint32_t* sload, typename RecOf<R>::T (&outr)[16],
                                          uint32_t* load_out) {
  using T = typename RecOf<R>::T;
  constexpr uint32_t Z = 1u << LZ, ZP = Z + (Z >> 4), HL = Z >> 4;
  const uint32_t tid = threadIdx.x, NB = 1u << klev, m = Z << klev;
  const bool active = FULL || tid < (m >> 4);
  const uint32_t S = active ? tid / HL : 0u, lq = active ? tid % HL : 0u;
  const uint32_t bbase = S * ZP;
  // record order, dummies (maximal record) last
  const LdsR<T> lr{srec};
  ElemR<T> v[16];
#pragma unroll
  for (uint32_t e = 0; e < 16; ++e) {
    const uint32_t i = bbase + 17u * lq + e;
    if (active) {
      BOS_TR(0, 5, i);
      BOS_TR(0, 4, i);
    }
    v[e] = ElemR<T>{(active && stag[i] != kDummyTag) ? srec[i] : max_rec<T>()};
  }
  bin_bitonic<LZ>(v, lr, bbase, lq, active);
  if (active) BOS_TR(0, 7, S);
  const uint32_t load = active ? sload[S] : 0u;
  *load_out = load;
  const bool permute = FIN == 2 || (FIN == 0 && a.fin == 0);
  if (FIN != 1 && permute) {
    const uint64_t gb = blk * NB + brev_k(S, klev);
    ElemRK<T> w[16];
#pragma unroll
    for (uint32_t e4 = 0; e4 < 4; ++e4) {
      const uint32_t p0 = 16u * lq + 4u * e4;
      const Philox4 ph = philox4x64_10((gb * Z + p0) >> 2, a.attempt, a.seed, 1);
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q) {
        const uint32_t e = 4u * e4 + q;
        const bool real = p0 + q < load;  // reals occupy the first `load` slots
        w[e] = ElemRK<T>{v[e].r, real ? uint32_t(ph.v[q]) : ~0u, real ? uint32_t(ph.v[q] >> 32) : ~0u,
                         real ? p0 + q : 0xFFFFu};
      }
    }
    lds_barrier();  // the record sort's last LDS reads are done
    const LdsRK<T> lrk{srec, stag, srhi, saux};
    bin_bitonic<LZ>(w, lrk, bbase, lq, active);
#pragma unroll
    for (uint32_t e = 0; e < 16; ++e) outr[e] = w[e].r;
  } else {
#pragma unroll
    for (uint32_t e = 0; e < 16; ++e) outr[e] = v[e].r;
  }
}

// Value of lane (lane ^ X) within each group of 32 lanes (ds_swizzle in bit
// mode: and-mask 31, or-mask 0, xor-mask X; no LDS memory is touched).
template <uint32_t X>
__device__ __forceinline__ uint32_t swz_xor(uint32_t v) {
  static_assert(X >= 1 && X < 32, "xor-mask of 5 bits");
  return uint32_t(__builtin_amdgcn_ds_swizzle(int(v), int((X << 10) | 0x1F)));
}
template <uint32_t X>
__device__ __forceinline__ uint2 swz_xor(uint2 v) {
  return make_uint2(swz_xor<X>(v.x), swz_xor<X>(v.y));
}
template <uint32_t X>
__device__ __forceinline__ uint4 swz_xor(uint4 v) {
  return make_uint4(swz_xor<X>(v.x), swz_xor<X>(v.y), swz_xor<X>(v.z), swz_xor<X>(v.w));
}

// One compaction stage at distance 16 HLX (< 512 slots): the partner slot is
// held by lane lq ^ HLX, reached by a swizzle; bpfx holds the scaled prefixes
// of the bin's lanes, the node's middle is its lane HLX.
template <uint32_t HLX, typename T>
__device__ __forceinline__ void compact_xstage(T (&rv)[16], uint32_t (&tv)[16], const uint32_t* bpfx, uint32_t lq,
                                               bool active) {
  constexpr uint32_t LH = 4u + uint32_t(__builtin_ctz(HLX));  // log2 of the distance
  const uint32_t mid = (lq & ~(2u * HLX - 1u)) + HLX;
  if (active) BOS_TR(0, 6, mid);
  // index in the node's half: 16 (lq mod HLX) + e
  const uint32_t q = (active ? bpfx[mid] : 0u) - ((lq & (HLX - 1u)) << (35u - LH));
#pragma unroll
  for (uint32_t e = 0; e < 16; ++e) {
    const uint32_t m = sign_mask(q - (e << (31u - LH)));
    const T pr = swz_xor<HLX>(rv[e]);
    const uint32_t pt = swz_xor<HLX>(tv[e]);
    rv[e] = msel(m, pr, rv[e]);
    tv[e] = msel(m, pt, tv[e]);
  }
}

// Oblivious compaction of every final bin in LDS: the bin's reals move to
// its first slots.  The last level leaves each bin's reals interleaved with
// dummies; this is the tight compaction network a MergeSplit level runs
// (conditional swaps at distances 1, 2, .., Z/2, each decided by the swap rule
// above from the prefix counts of the reals), over one bin of Z slots with the reals as
// the marks.  Lane lq of the bin's Z/16 lanes holds slots 16 lq + e; stages at
// distances below 16 pair registers, those up to 256 pair lanes by swizzles,
// and longer ones exchange through the bin's own LDS slots.  On return rv
// holds this lane's 16 slots after the compaction.
// LOAD: read the bin's slots from LDS first; else rv and tv already hold
// them (layout P).
template <int R, int LZ, bool FULL, bool LOAD>
__device__ __forceinline__ void compact_bin(typename RecOf<R>::T* srec, uint32_t* stag, uint32_t* spfx,
                                            uint32_t* swave, uint32_t klev, typename RecOf<R>::T (&rv)[16],
                                            uint32_t (&tv)[16]) {
  using T = typename RecOf<R>::T;
  constexpr uint32_t Z = 1u << LZ, ZP = Z + (Z >> 4), HL = Z >> 4;
  const uint32_t tid = threadIdx.x, m = Z << klev;
  const bool active = FULL || tid < (m >> 4);
  const uint32_t S = active ? tid / HL : 0u, lq = active ? tid % HL : 0u;
  const uint32_t bbase = S * ZP;
  if constexpr (LOAD) {
#pragma unroll
    for (uint32_t e = 0; e < 16; ++e) {
      if (active) {
        BOS_TR(0, 4, bbase + 17u * lq + e);
        BOS_TR(0, 5, bbase + 17u * lq + e);
      }
      rv[e] = active ? srec[bbase + 17u * lq + e] : zero_rec<T>();
      tv[e] = active ? stag[bbase + 17u * lq + e] : kDummyTag;
    }
  }
  // prefix counts of the reals, minus one (a dummy's tag is all ones, a
  // label has its sign bit clear: 1 + the sign mask counts a real)
  uint32_t pm[16];
  uint32_t run = 0;
#pragma unroll
  for (uint32_t e = 0; e < 16; ++e) {
    pm[e] = run;
    run += 1u + sign_mask(tv[e]);
  }
  uint32_t tot;
  const uint32_t excl = seg_scan<HL>(active ? run : 0u, swave, &tot) - 1u;
#pragma unroll
  for (uint32_t e = 0; e < 16; ++e) pm[e] += excl;
  if (active) {
    BOS_TR(0, 6, S * HL + lq);
    spfx[S * HL + lq] = lane_prefix(pm[0], lq, HL);
  }
  // distances 1, 2, 4, 8: register pairs
  lane_stages(rv, tv, pm);
  // distances 16 .. 256: the partner lane is lq ^ (half / 16), within 32 lanes
  lds_group_sync<HL>();  // every lane's prefix is in spfx
  const uint32_t* bpfx = spfx + S * HL;
  if constexpr (HL >= 2) compact_xstage<1>(rv, tv, bpfx, lq, active);
  if constexpr (HL >= 4) compact_xstage<2>(rv, tv, bpfx, lq, active);
  if constexpr (HL >= 8) compact_xstage<4>(rv, tv, bpfx, lq, active);
  if constexpr (HL >= 16) compact_xstage<8>(rv, tv, bpfx, lq, active);
  if constexpr (HL >= 32) compact_xstage<16>(rv, tv, bpfx, lq, active);
  // distances 512 .. Z/2 (Z >= 1024): through the bin's LDS slots
#pragma unroll
  for (uint32_t lh = 9; lh + 1 <= LZ; ++lh) {
    lds_group_sync<HL>();  // spfx written; the previous stage's reads are done
    if (active) {
#pragma unroll
      for (uint32_t e = 0; e < 16; ++e) {
        BOS_TR(0, 4, bbase + 17u * lq + e);
        BOS_TR(0, 5, bbase + 17u * lq + e);
        srec[bbase + 17u * lq + e] = rv[e];
        stag[bbase + 17u * lq + e] = tv[e];
      }
    }
    lds_group_sync<HL>();
    const uint32_t hl = 1u << (lh - 4u);                  // lanes per half node
    const uint32_t mid = (lq & ~(2u * hl - 1u)) + hl;     // the node's middle lane
    const uint32_t plq = lq ^ hl;
    if (active) BOS_TR(0, 6, S * HL + mid);
    const uint32_t q = (active ? bpfx[mid] : 0u) - ((lq & (hl - 1u)) << (35u - lh));
#pragma unroll
    for (uint32_t e = 0; e < 16; ++e) {
      const uint32_t m = sign_mask(q - (e << (31u - lh)));
      const uint32_t pi = bbase + 17u * plq + e;
      if (active) {
        BOS_TR(0, 4, pi);
        BOS_TR(0, 5, pi);
      }
      const T pr = active ? srec[pi] : zero_rec<T>();
      const uint32_t pt = active ? stag[pi] : kDummyTag;
      rv[e] = msel(m, pr, rv[e]);
      tv[e] = msel(m, pt, tv[e]);
    }
  }
}

// Last pass, split form: after the per-bin finish, global bin gb keeps its
// reals in slots gb*Z .. gb*Z + load - 1 of rec_out, its real count in
// loads[gb] and the block's total in scan[blk]; a scan and a strip kernel then
// concatenate the bins (the addresses of both depend on the loads only, which
// the method reveals).  FIN = 3: the bins are compacted, not sorted (their
// reals keep the order the last level left).
// LOADED (FIN = 3): rv and tv already hold every bin's slots (layout P:
// lane lq of bin S holds slots 16 lq .. 16 lq + 15); else they are read from
// LDS.  rv and tv are scratch registers of the caller; S is the block's bin
// that this lane's slots belong to.
template <int R, int LZ, int FIN, bool FULL, bool LOADED>
__device__ __forceinline__ void finish_split(const PassArgs& a, uint32_t blk, uint32_t klev,
                                             typename RecOf<R>::T* srec, uint32_t* stag, uint32_t* srhi,
                                             uint16_t* saux, const uint32_t* sload, uint32_t* spfx,
                                             uint32_t* swave, typename RecOf<R>::T (&rv)[16],
                                             uint32_t (&tv)[16], uint32_t S) {
  using T = typename RecOf<R>::T;
  constexpr uint32_t Z = 1u << LZ, HL = Z >> 4;
  const uint32_t tid = threadIdx.x, NB = 1u << klev, m = Z << klev;
  const bool active = FULL || tid < (m >> 4);
  const uint32_t lq = active ? tid % HL : 0u;
  if (tid == 0) {
    uint64_t agg = 0;
    for (uint32_t b = 0; b < NB; ++b) {
      BOS_TR(0, 7, b);
      agg += sload[b] < Z ? sload[b] : Z;
    }
    BOS_TR(0, 14, blk);
    a.scan[blk] = agg;
  }
  T (&outr)[16] = rv;
  uint32_t load = 0;
  if constexpr (FIN == 3) {
    compact_bin<R, LZ, FULL, !LOADED>(srec, stag, spfx, swave, klev, outr, tv);
    if (active) BOS_TR(0, 7, S);
    load = active ? sload[S] : 0u;
  } else {
    static_assert(!LOADED, "the per-bin sorts read their bins from LDS");
    sort_bins<R, LZ, FIN, FULL>(a, blk, klev, srec, stag, srhi, saux, sload, outr, &load);
  }
  if (active) {
    // a bin holds at most Z reals (an overflowing attempt is discarded)
    const uint32_t kept = load < Z ? load : Z;
    const uint64_t gb = uint64_t(blk) * NB + brev_k(S, klev);
    T* BO = static_cast<T*>(a.rec_out);
    if (lq == 0) {
      BOS_TR(0, 13, gb);
      a.loads[gb] = kept;
    }
#pragma unroll
    for (uint32_t e = 0; e < 16; ++e) {
      const uint32_t p = 16u * lq + e;
      if (p < kept) {
        BOS_TR(0, 12, (gb << LZ) + p);
        BO[(gb << LZ) + p - a.out_slot0] = outr[e];
      }
    }
  }
}

// Last pass, fused form: sort (fin 1), compact (fin 2) or randomly permute (fin
// 0) every bin, then strip the dummies and write the bins' reals to their place in the output, found with
// a decoupled look-back over the blocks (block index = ticket order).
template <int R, int LZ, bool FULL>
__device__ __forceinline__ void finish_bins(const PassArgs& a, uint32_t blk, uint32_t klev,
                                            typename RecOf<R>::T* srec, uint32_t* stag, uint32_t* srhi,
                                            uint16_t* saux, uint32_t* sload, uint32_t* soff, uint32_t* spfx,
                                            uint32_t* swave) {
  using T = typename RecOf<R>::T;
  constexpr uint32_t Z = 1u << LZ, HL = Z >> 4;
  const uint32_t tid = threadIdx.x, NB = 1u << klev, m = Z << klev;
  const bool active = FULL || tid < (m >> 4);
  const uint32_t S = active ? tid / HL : 0u, lq = active ? tid % HL : 0u;
  // The bin loads (sload, written by the last level) are known before the
  // bins are sorted: publish the block's aggregate now so that later blocks'
  // look-back does not wait for this block's sort.
  uint64_t agg = 0;
  if (tid == 0) {
    for (uint32_t b = 0; b < NB; ++b) {
      BOS_TR(0, 7, b);
      agg += sload[b];
    }
    BOS_TR(0, 14, blk);
    __hip_atomic_store(&a.scan[blk], ((blk == 0 ? 2ull : 1ull) << 62) | agg, __ATOMIC_RELEASE,
                       __HIP_MEMORY_SCOPE_AGENT);
  }
  T outr[16];
  uint32_t load = 0;
  if (a.fin == 2u) {
    uint32_t tv[16];
    compact_bin<R, LZ, FULL, true>(srec, stag, spfx, swave, klev, outr, tv);
    if (active) BOS_TR(0, 7, S);
    load = active ? sload[S] : 0u;
  } else {
    sort_bins<R, LZ, 0, FULL>(a, blk, klev, srec, stag, srhi, saux, sload, outr, &load);
  }
  // look back for the block's output offset (reals occupy the first slots of
  // every sorted bin).  Wave 0 inspects 64 predecessors per step: it sums
  // their aggregates back to the nearest one whose inclusive prefix is known.
  if (tid < 64) {
    const uint32_t lane = tid;
    const uint64_t kVal = (1ull << 62) - 1ull;
    uint64_t excl = 0;
    int64_t p = int64_t(blk) - 1;
    while (p >= 0) {
      const int64_t idx = p - int64_t(lane);
      const unsigned long long w =
          idx >= 0 ? __hip_atomic_load(&a.scan[idx], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) : (2ull << 62);
      const uint32_t flag = uint32_t(w >> 62);
      const unsigned long long inc = __ballot(flag == 2u), none = __ballot(flag == 0u);
      const uint32_t first2 = inc ? uint32_t(__ffsll((long long)inc) - 1) : 64u;
      const unsigned long long need = first2 < 63u ? ((2ull << first2) - 1ull) : ~0ull;
      if (none & need) {
        __builtin_amdgcn_s_sleep(1);
        continue;
      }
      uint64_t v = lane <= first2 ? (w & kVal) : 0ull;
#pragma unroll
      for (uint32_t o = 32; o > 0; o >>= 1) v += __shfl_xor(v, int(o), 64);
      excl += v;
      if (first2 < 64u) break;
      p -= 64;
    }
    if (lane == 0) {
      if (blk != 0)
        __hip_atomic_store(&a.scan[blk], (2ull << 62) | (excl + agg), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
      uint64_t off = excl;
      for (uint32_t u = 0; u < NB; ++u) {
        const uint32_t b = brev_k(u, klev);
        BOS_TR(0, 8, b);
        BOS_TR(0, 7, b);
        soff[2 * b] = uint32_t(off);
        soff[2 * b + 1] = uint32_t(off >> 32);
        off += sload[b];
      }
    }
  }
  lds_barrier();
  if (active) {
    T* OUT = static_cast<T*>(a.out);
    BOS_TR(0, 8, S);
    const uint64_t off = (uint64_t(soff[2 * S + 1]) << 32) | soff[2 * S];
#pragma unroll
    for (uint32_t e = 0; e < 16; ++e) {
      const uint32_t p = 16u * lq + e;
      if (p < load && off + p < a.n) {
        BOS_TR(0, 16, off + p);
        OUT[off + p] = outr[e];
      }
    }
  }
}

// R: record bytes; LZ: log2 Z (4..11); MODE bit 0 = first pass, bit 1 = last,
// bit 2 = split form of the last pass (bins compacted and written to rec_out,
// then scan + strip; the sorts only), bit 4 = the launch has exactly Z 2^klev / 16 lanes
// (all of them hold slots, so no lane needs a guard).
// Body of one routing launch.  BATCH = false: a persistent workgroup walks
// over items blockIdx.x, + gridDim.x, ... (last pass: tickets).  BATCH = true:
// the workgroup runs the single item `item0` of one instance of a batch.
template <int R, int LZ, int MODE, bool BATCH>
__device__ __forceinline__ void route_run(const PassArgs& a, uint32_t nitems, uint32_t item0) {
  using T = typename RecOf<R>::T;
  constexpr bool FIRST = (MODE & 1) != 0, LAST = (MODE & 2) != 0, SPLIT = (MODE & 4) != 0;
  constexpr bool FULL = (MODE & 16) != 0;  // every lane holds slots: no lane guards
  static_assert(!SPLIT || (LAST && !FIRST), "the split form is a last pass that is not also the first");
  // the split form serves the sorts: it compacts its bins, and the strip puts
  // in order the bins that straddle a tile of the comparison sort's first
  // phase (the tile sort orders every other bin with its tile); bos_orp's
  // permuting finish keeps the fused form
  constexpr int SPLIT_FIN = 3;
  constexpr uint32_t Z = 1u << LZ, LQ = LZ + 1, TPM = 1u << (LQ - 4), ZP = Z + (Z >> 4);
  constexpr bool HAS_B = LQ > 6;
  constexpr uint32_t HALF_LANES = TPM / 2;  // lanes per bucket in layout A

  // Records exchange through LDS in two halves (the tags go with the
  // first): LDS holds half a record and a tag per slot, so more workgroups
  // share a CU.
  constexpr bool HALF = lds_rec_bytes(R, Z, LAST && !SPLIT) < uint32_t(R);
  static_assert(!HALF || HAS_B, "two-half exchanges use layout B (Z >= 64)");
  using H = typename HalfOf<T>::H;
  // Z = 512: a MergeSplit's lanes are one wave.  Only the change of buckets
  // between levels crosses waves, and a wave keeps one of its two buckets
  // there, so half of its slots move; layouts change word by word in the
  // wave's own kXWords words, with no barrier.
  constexpr bool WAVEX = HAS_B && TPM == 64 && (!LAST || SPLIT);
  static_assert(!WAVEX || FULL, "a wave without slots would index past the block's LDS words");
  extern __shared__ __align__(16) unsigned char smem[];
  const uint32_t klev = a.klev, NB = 1u << klev, m = Z << klev, mp = NB * ZP;
  T* srec = reinterpret_cast<T*>(smem);
  H* shalf = reinterpret_cast<H*>(smem);  // HALF: one half record per slot
  uint32_t* stag = reinterpret_cast<uint32_t*>(smem + size_t(mp) * lds_rec_bytes(R, Z, LAST && !SPLIT));
  // m/16 marks-prefix entries (16-slot granularity)
  uint32_t* spfx = WAVEX ? reinterpret_cast<uint32_t*>(smem) + (m >> 10) * kXWords : stag + mp;
  uint32_t* sload = spfx + (m >> 4);   // NB bin loads (last pass)
  uint32_t* soff = sload + NB;         // 2*NB words: output offsets (last pass)
  uint32_t* swave = soff + 2 * NB;     // 64 scan words
  uint32_t* smisc = swave + 64;        // 16 words
  uint32_t* srhi = smisc + 16;         // last pass, shuffle
  uint16_t* saux = reinterpret_cast<uint16_t*>(srhi + mp);

  __builtin_amdgcn_s_setprio(1);  // light_begin / light_end lower it inside the networks
  const uint32_t tid = threadIdx.x;
  const uint64_t n = a.n;
  const uint32_t L = a.levels, i0 = a.level0;
  const bool active = FULL || tid < (m >> 4);
  const uint32_t ms = active ? tid / TPM : 0u, lt = active ? tid % TPM : 0u;
  const T* RI = static_cast<const T*>(a.rec_in);
  const T* X = static_cast<const T*>(a.x_in);
  // ---- load one block into layout-A registers of level 0 -------------------
  // level 0 pairs LDS buckets 2ms and 2ms+1; lane lt holds slots 16*(lt mod
  // TPM/2) .. +15 of bucket 2ms + lt / (TPM/2).
  const uint32_t S_load = 2u * ms + (lt >= HALF_LANES ? 1u : 0u);
  const uint32_t sb_load = 16u * (lt % HALF_LANES);
  T rv[16];
  uint32_t tv[16];

  // bucket slot that register e of the bucket's lane lh loads (passes after
  // the first)
  auto in_slot = [&](uint32_t e, uint32_t lh) -> uint32_t {
    if constexpr (R == 8)
      return (e >> 1) * (2u * HALF_LANES) + 2u * lh + (e & 1u);
    else
      return e * HALF_LANES + lh;
  };
  // first pass: group [gs, ge), of at most Z/2 elements, in registers 0..7 of
  // its bucket's lanes.  Lane q takes the Philox block c = gs/8 + q, element i of
  // the block in register i; the elements of block gs/8 + Z/16 (of a group that
  // starts inside a block) take lane 0's registers that lie before gs.  Other
  // slots are dummies (tag 0 marks a real until finish_load puts its label there).
  auto load_group = [&](uint64_t c, uint64_t gs, uint64_t ge, T* dr, uint32_t* dt) {
#pragma unroll
    for (uint32_t i = 0; i < 8; i += 2) {
      uint64_t x0 = 8u * c + i, x1 = x0 + 1;
      x0 += x0 < gs ? 8u * HALF_LANES : 0u;
      x1 += x1 < gs ? 8u * HALF_LANES : 0u;
      const bool r0 = active && x0 < ge, r1 = active && x1 < ge;
      if (r0) BOS_TR(0, 3, x0);
      if (r1) BOS_TR(0, 3, x1);
      dr[i] = dr[i + 1] = zero_rec<T>();
      if constexpr (R == 8) {
        if (r0 && r1 && x1 == x0 + 1) {  // one 16-byte load (8-byte aligned: x_off may be odd)
          typedef v4u __attribute__((aligned(8))) v4u8;
          const v4u t = *reinterpret_cast<const v4u8*>(X + (x0 - a.x_off));
          dr[i] = make_uint2(t.x, t.y);
          dr[i + 1] = make_uint2(t.z, t.w);
        } else {
          if (r0) dr[i] = X[x0 - a.x_off];
          if (r1) dr[i + 1] = X[x1 - a.x_off];
        }
      } else {
        if (r0) dr[i] = X[x0 - a.x_off];
        if (r1) dr[i + 1] = X[x1 - a.x_off];
      }
      dt[i] = r0 ? 0u : kDummyTag;
      dt[i + 1] = r1 ? 0u : kDummyTag;
    }
#pragma unroll
    for (uint32_t i = 8; i < 16; ++i) {
      dr[i] = zero_rec<T>();
      dt[i] = kDummyTag;
    }
  };
  // label of element i of the Philox block ph
  auto label = [&](const Philox4& ph, uint32_t i) -> uint32_t {
    const uint32_t w = uint32_t(ph.v[i >> 1] >> (32u * (i & 1u)));
    return L ? (w >> (32u - L)) : 0u;
  };
  auto issue_load = [&](uint32_t item, T* dr, uint32_t* dt) {
    const uint64_t r = uint64_t(item) & ((1ull << i0) - 1ull), h = uint64_t(item) >> i0;
    if constexpr (!FIRST) {
      const uint64_t bucket = (h << (i0 + klev)) + (uint64_t(S_load) << i0) + r;
      const uint64_t gi = bucket << LZ;
      // staged chunk: input segment S_load holds buckets (S_load, r in0 ..)
      const uint64_t si = a.staged ? ((((h - a.in_h0) << (a.in_lseg + klev)) + (uint64_t(S_load) << a.in_lseg) +
                                       (r - a.in_r0)) << LZ)
                                   : gi;
      // A bucket is a set, so its slots take the network's positions in the
      // order that loads best: register pairs (e, e + 1) of a lane hold two
      // consecutive slots and consecutive lanes consecutive pairs (16-byte
      // records: consecutive lanes consecutive slots), so a wave's instruction
      // reads whole lines.  (With lane lt holding slots 16 lt .. 16 lt + 15
      // every instruction of a wave touched 64 lines.)
      const uint32_t lh = lt % HALF_LANES;
#pragma unroll
      for (uint32_t e = 0; e < 16; ++e) {
        const uint32_t s = in_slot(e, lh);
        if (active) {
          BOS_TR(0, 1, gi + s);
          BOS_TR(0, 2, gi + s);
        }
        dr[e] = active ? RI[si + s] : zero_rec<T>();
        dt[e] = active ? a.tag_in[si + s] : kDummyTag;
      }
    } else {
      // Group j = h*NB + S_load holds X[floor(jn/B), floor((j+1)n/B))
      const uint64_t j = h * NB + S_load;
      const uint64_t gs = (j * n) >> L, ge = ((j + 1) * n) >> L;
      load_group((gs >> 3) + lt % HALF_LANES, gs, ge, dr, dt);
    }
  };
  // first pass: labels of the loaded reals (word x mod 8 of Philox block x/8)
  auto finish_load = [&](uint32_t item, uint32_t* dt) {
    if constexpr (FIRST) {
      const uint64_t h = uint64_t(item) >> i0;
      const uint64_t j = h * NB + S_load;
      const uint64_t gs = (j * n) >> L, ge = ((j + 1) * n) >> L;
      const uint64_t c = (gs >> 3) + lt % HALF_LANES;
      const Philox4 ph = philox4x64_10(c, a.attempt, a.seed, 0);
#pragma unroll
      for (uint32_t i = 0; i < 8; ++i) dt[i] |= label(ph, i);  // (a dummy's tag is all ones)
      if (8u * (c + HALF_LANES) < ge) {  // lane 0, a group that starts inside a block
        const Philox4 p2 = philox4x64_10(c + HALF_LANES, a.attempt, a.seed, 0);
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i)
          if (8u * c + i < gs && 8u * (c + HALF_LANES) + i < ge) dt[i] = label(p2, i);
      }
    }
  };

  // ---- one block -----------------------------------------------------------
  // padded LDS index of this lane's slot e in layout B of the MergeSplit of
  // buckets at base0 / base1 (bB0, bB1: their layout-B lane bases; lB: the
  // lane's low slot bits)
  auto b_index = [&](uint32_t e, uint32_t b0, uint32_t b1, uint32_t bB0, uint32_t bB1, uint32_t lB) -> uint32_t {
    const uint32_t sl = (e & 7u) << (LQ - 4);
    // padded index of slot s = sl + lB: s + s/16 = sl + sl/16 + lB + lB/16
    // holds because sl is a multiple of 16 whenever LQ >= 8; for smaller Z
    // compute it directly
    if constexpr (LQ >= 8) {
      return ((e < 8) ? bB0 : bB1) + sl + (sl >> 4);
    } else {
      const uint32_t s2 = sl + lB;
      return (e < 8 ? b0 : b1) + s2 + (s2 >> 4);
    }
  };
  // HALF: second half of an exchange whose first halves (and tags) every
  // lane has stored at its indices src(e): read the first halves and tags at
  // dst(e), wait for the group, store this lane's second halves (still in rv)
  // at src(e), wait, read them at dst(e).
  // (the new first halves replace the stored ones in rv, which keeps the
  // second halves until they are stored: no extra registers)
  auto half_finish = [&](auto src, auto dst, auto sync) {
#pragma unroll
    for (uint32_t e = 0; e < 16; ++e) {
      if (active) {
        BOS_TR(0, 4, dst(e));
        BOS_TR(0, 5, dst(e));
      }
      set_lo(rv[e], active ? shalf[dst(e)] : HalfOf<T>::zero());
      tv[e] = active ? stag[dst(e)] : kDummyTag;
    }
    sync();
    if (active) {
#pragma unroll
      for (uint32_t e = 0; e < 16; ++e) {
        BOS_TR(0, 4, src(e));
        shalf[src(e)] = rec_hi(rv[e]);
      }
    }
    sync();
#pragma unroll
    for (uint32_t e = 0; e < 16; ++e) {
      if (active) BOS_TR(0, 4, dst(e));
      set_hi(rv[e], active ? shalf[dst(e)] : HalfOf<T>::zero());
    }
  };
  // WAVEX: this wave's words; slot q of the MergeSplit is at word q + q/32, so
  // that the 32 lanes of a half wave touch 32 different banks in layout A
  // (slots 16 l + e) and in layout B (64 e + l).  (With q + q/16 one lane of
  // layout B's half wave wrapped onto another's bank, which doubles the time of
  // the whole access: 4.1 instead of 2.1 cycles per b32 read.)
  uint32_t* xw = reinterpret_cast<uint32_t*>(smem) + (tid >> 6) * kXWords;
  const uint32_t slot_a = 16u * lt + (lt >> 1), slot_b = lt + (lt >> 5);
  auto wave_exchange = [&](auto src, auto dst) {
#pragma unroll
    for (uint32_t w = 0; w <= R / 4u; ++w) {
#pragma unroll
      for (uint32_t e = 0; e < 16; ++e) {
        BOS_TR(0, 4, (tid >> 6) * kXWords + src(e));
        xw[src(e)] = w < R / 4u ? rec_word(rv[e], w) : tv[e];
      }
      lds_order();
#pragma unroll
      for (uint32_t e = 0; e < 16; ++e) {
        BOS_TR(0, 4, (tid >> 6) * kXWords + dst(e));
        const uint32_t x = xw[dst(e)];
        if (w < R / 4u) set_word(rv[e], w, x);
        else tv[e] = x;
      }
      lds_order();
    }
  };
  // WAVEX, after level d: this wave holds buckets S0 (registers 0..7, layout
  // B) and S1 (8..15); level d + 1 pairs S0 with the S0, and S1 with the S1, of
  // wave w ^ 2^d.  The wave whose bit d is clear keeps S0 and takes the other
  // S0 for its S1, the other wave the reverse.  kXWords words hold three words
  // of eight slots; 16-byte records take two rounds.
  auto swap_buckets = [&](uint32_t d) {
    const uint32_t w = uint32_t(__builtin_amdgcn_readfirstlane(int(tid >> 6)));
    const bool keep1 = ((w >> d) & 1u) != 0u;
    const uint32_t pw = w ^ (1u << d);
    const uint32_t* px = reinterpret_cast<const uint32_t*>(smem) + pw * kXWords;
    auto put = [&](uint32_t e0, uint32_t w0, uint32_t w1) {
#pragma unroll
      for (uint32_t q = w0; q < w1; ++q)
#pragma unroll
        for (uint32_t e = 0; e < 8; ++e) {
          BOS_TR(0, 4, w * kXWords + ((q - w0) * 8u + e) * 64u + lt);
          xw[((q - w0) * 8u + e) * 64u + lt] = q < R / 4u ? rec_word(rv[e0 + e], q) : tv[e0 + e];
        }
    };
    auto get = [&](uint32_t e0, uint32_t w0, uint32_t w1) {
#pragma unroll
      for (uint32_t q = w0; q < w1; ++q)
#pragma unroll
        for (uint32_t e = 0; e < 8; ++e) {
          BOS_TR(0, 4, pw * kXWords + ((q - w0) * 8u + e) * 64u + lt);
          const uint32_t x = px[((q - w0) * 8u + e) * 64u + lt];
          if (q < R / 4u) set_word(rv[e0 + e], q, x);
          else tv[e0 + e] = x;
        }
    };
    constexpr uint32_t W = R / 4u + 1u;  // words per slot with the tag
#pragma unroll
    for (uint32_t w0 = 0; w0 < W; w0 += 3u) {
      const uint32_t w1 = w0 + 3u < W ? w0 + 3u : W;
      if (w0 > 0) {  // the first round is read
        lds_barrier();
        lds_order();
      }
      // (the empty asm statements keep the two sides of these wave-uniform
      // branches apart: merged, every word would go through a v_cndmask)
      if (keep1) {
        put(0, w0, w1);
        asm volatile("; keep S1" ::: "memory");
      } else {
        put(8, w0, w1);
        asm volatile("; keep S0" ::: "memory");
      }
      lds_order();
      lds_barrier();
      lds_order();
      if (keep1) {
        asm volatile("; keep S1" ::: "memory");
        get(0, w0, w1);
      } else {
        asm volatile("; keep S0" ::: "memory");
        get(8, w0, w1);
      }
    }
  };
  // where the previous level left this lane's slots (layout B), for HALF
  uint32_t pb0 = 0, pb1 = 0, pbB0 = 0, pbB1 = 0, plB = 0;

  // Level 0 of Algorithm 3.1 needs no network: a bucket starts with at most Z/2
  // reals, which lie in registers 0..7 of its lanes, so the MergeSplit's lanes
  // hold them all in Z slots.  Both outputs keep those slots, each with the other
  // one's reals turned into dummies: registers 0..7 the lower bucket, 8..15 the
  // upper one, as layout B has them.  It cannot overflow.  (First pass of four
  // levels at n = 2^28 x 8 B: 3.41 ms with a network, 2.82 so.)
  constexpr bool LEVEL0 = FIRST && !LAST && HAS_B;
  auto level0 = [&](uint32_t shift) {
#pragma unroll
    for (uint32_t e = 0; e < 8; ++e) {
      // all ones: upper bucket (or dummy, whose record is zero)
      const uint32_t up = 0u - (uint32_t(int32_t(tv[e]) >> shift) & 1u);
      rv[8 + e] = rec_and(rv[e], up);
      tv[8 + e] = tv[e] | ~up;
      rv[e] = rec_and(rv[e], ~up);
      tv[e] |= up;
    }
  };

  auto process = [&](uint32_t item) {
    const uint64_t r = uint64_t(item) & ((1ull << i0) - 1ull), h = uint64_t(item) >> i0;
    for (uint32_t d = 0; d < klev; ++d) {
      const uint32_t lev = i0 + d, shift = L - 1u - lev;
      const uint32_t S0 = ((ms >> d) << (d + 1)) | (ms & ((1u << d) - 1u)), S1 = S0 | (1u << d);
      const uint32_t base0 = S0 * ZP, base1 = S1 * ZP;
      // layout A: this lane's 16 slots are bucket (lt < TPM/2 ? S0 : S1),
      // slots 16*(lt mod TPM/2) + e
      const uint32_t baseA = (lt < HALF_LANES ? base0 : base1) + 17u * (lt % HALF_LANES);
      if (d > 0 && !WAVEX) {
        if constexpr (HALF) {
          half_finish([&](uint32_t e) { return b_index(e, pb0, pb1, pbB0, pbB1, plB); },
                      [&](uint32_t e) { return baseA + e; }, [] { lds_barrier(); });
        } else {
#pragma unroll
          for (uint32_t e = 0; e < 16; ++e) {
            if (active) {
              BOS_TR(0, 4, baseA + e);
              BOS_TR(0, 5, baseA + e);
            }
            rv[e] = active ? srec[baseA + e] : zero_rec<T>();
            tv[e] = active ? stag[baseA + e] : kDummyTag;
          }
        }
      }
      // lane lt in layout B: q = e << (LQ-4) | lb1 << (LQ-5) | lb0 << (LQ-6) | rest.
      // Layout B pairs lanes through DPP only for Z >= 1024; below that the
      // lanes simply take consecutive slots (conflict-free LDS access).
      const uint32_t lb0 = lt & 1u, lb1 = (lt >> 1) & 1u, rest = lt >> 2;
      const uint32_t lowB = (LQ >= 11) ? ((lb1 << (LQ - 5)) | (lb0 << (LQ - 6)) | rest) : lt;
      const uint32_t baseB0 = base0 + lowB + (lowB >> 4), baseB1 = base1 + lowB + (lowB >> 4);
      if (LEVEL0 && d == 0) {
        level0(shift);
      } else {
        // prefix counts of class-0 reals (bits 0 ..) and dummies (bits FB ..).
        // tag >> shift (arithmetic) is all ones for a dummy and a real's label
        // down to its routing bit, below 2^FB while L <= FB; longer labels
        // (L > FB) are cut to their routing bit first.
        constexpr uint32_t FB = 31u - LQ;
        uint32_t pk[16];
        uint32_t run = 0;
        uint32_t kf = (1u << FB) | 1u;
        asm("" : "+v"(kf));  // v_bitop3 takes no literal
        light_begin();
        if (L <= FB) {
#pragma unroll
          for (uint32_t e = 0; e < 16; ++e) {
            pk[e] = run;
            const uint32_t x = uint32_t(int32_t(tv[e]) >> shift);
            run += __builtin_amdgcn_bitop3_b32(x, kf, 1u, 0x6A);  // (x & kf) ^ 1
          }
        } else {
#pragma unroll
          for (uint32_t e = 0; e < 16; ++e) {
            pk[e] = run;
            const uint32_t x = uint32_t(int32_t(tv[e]) >> shift) & (sign_mask(tv[e]) | 1u);
            run += __builtin_amdgcn_bitop3_b32(x, kf, 1u, 0x6A);
          }
        }
        light_end();
        uint32_t tot;
        const uint32_t excl = seg_scan<TPM>(active ? run : 0u, swave, &tot);
        const uint32_t x = tot & ((1u << FB) - 1u), nd = tot >> FB, y = 2u * Z - x - nd;
        const uint32_t need = x <= Z ? Z - x : 0u;
        // marks before slot e: class-0 reals + min(dummies, need); pm[e] is one
        // less, modulo 2Z.  The count fields are biased (2Z - 1 + need below,
        // -need above), so that min(dummies, need) = need + min(upper field, 0).
        const uint32_t bias = excl + (2u * Z - 1u + need) - (need << FB);
        uint32_t pm[16];
        light_begin();
#pragma unroll
        for (uint32_t e = 0; e < 16; ++e) {
          const uint32_t pe = bias + pk[e];
          pm[e] = (pe & ((1u << FB) - 1u)) + (uint32_t(int32_t(pe) >> FB) & sign_mask(pe));
        }
        light_end();
        const uint32_t qm = lane_prefix(pm[0], lt, TPM);
        if (active) {
          BOS_TR(0, 6, ms * TPM + lt);
          spfx[ms * TPM + lt] = qm;
          if (LAST && lt == 0 && d + 1 == klev) {
            // bin loads of this block: S0 keeps min(x, Z) reals, S1 the rest of
            // the pair's reals (exact even when the MergeSplit overflowed)
            const uint32_t k0 = x < Z ? x : Z;
            BOS_TR(0, 7, S0);
            BOS_TR(0, 7, S1);
            sload[S0] = k0;
            sload[S1] = x + y - k0;
          }
          if (lt == 0 && (x > Z || y > Z)) {
            const uint64_t G = S0 >> (d + 1);
            const uint64_t v = brev_k(S0 & ((1u << d) - 1u), d);
            const uint64_t j = (((h << (klev - d - 1)) + G) << lev) + (r << d) + v;
            BOS_TR(0, 15, 0);
            atomicMin(a.status, (unsigned long long)((uint64_t(lev) << 32) | j));
          }
        }
        // -- layout A, q bits 0..3: register pairs
        lane_stages(rv, tv, pm);
        // -- layout A, q bit 4: lanes l and l^1 (node = 2 lanes, half = 16)
        if constexpr (LQ >= 5) {
          dpp_stage<kDppXor1>(rv, tv, dpp<kDppB1133>(qm), 1u << 27);
        }
        // -- layout A, q bit 5: lanes l and l^2 (node = 4 lanes, half = 32)
        if constexpr (LQ >= 6) {
          dpp_stage<kDppXor2>(rv, tv, dpp<kDppB2222>(qm) - ((lt & 1u) << 30), 1u << 26);
        }
        if constexpr (HAS_B) {
          // A -> LDS (HALF: the first halves)
          if constexpr (WAVEX) {
            // other waves have read what this one handed them after the last level
            if (d > 0) lds_barrier();
          } else if (active) {
#pragma unroll
            for (uint32_t e = 0; e < 16; ++e) {
              BOS_TR(0, 4, baseA + e);
              BOS_TR(0, 5, baseA + e);
              if constexpr (HALF)
                shalf[baseA + e] = rec_lo(rv[e]);
              else
                srec[baseA + e] = rv[e];
              stag[baseA + e] = tv[e];
            }
          }
          if constexpr (!WAVEX) lds_group_sync<TPM>();  // layouts A and B of one MergeSplit share its lanes
          // HALF: the exchange first (its registers are free before the prefixes load)
          if constexpr (WAVEX) {
            wave_exchange([&](uint32_t e) { return slot_a + e; }, [&](uint32_t e) { return slot_b + 66u * e; });
          } else if constexpr (HALF) {
            half_finish([&](uint32_t e) { return baseA + e; },
                        [&](uint32_t e) { return b_index(e, base0, base1, baseB0, baseB1, lowB); },
                        [] { lds_group_sync<TPM>(); });
          }
          // scaled marks prefixes at the node middles (multiples of 16 slots)
          uint32_t pv[16], pvh[16];
#pragma unroll
          for (uint32_t e = 0; e < 16; ++e) {
            const uint32_t q = e << (LQ - 4);
            pv[e] = 0;
            // slot q is the middle of a node of half 2^(LQ-4+ctz(e)), at least 64
            if (e != 0 && LQ - 4 + __builtin_ctz(e | 16u) >= 6) {
              if (active) BOS_TR(0, 6, ms * TPM + (q >> 4));
              pv[e] = active ? spfx[ms * TPM + (q >> 4)] : 0u;
            }
            if constexpr (LQ >= 11) {
              const uint32_t qh = q | (1u << (LQ - 5));
              if (active) BOS_TR(0, 6, ms * TPM + (qh >> 4));
              pvh[e] = active ? spfx[ms * TPM + (qh >> 4)] : 0u;
            } else {
              pvh[e] = 0;
            }
          }
          if constexpr (!HALF) {
#pragma unroll
            for (uint32_t e = 0; e < 16; ++e) {
              const uint32_t pi = b_index(e, base0, base1, baseB0, baseB1, lowB);
              if (active) {
                BOS_TR(0, 4, pi);
                BOS_TR(0, 5, pi);
              }
              rv[e] = active ? srec[pi] : zero_rec<T>();
              tv[e] = active ? stag[pi] : kDummyTag;
            }
          }
          // -- layout B, q bit LQ-6 (lane bit 0), only for Z = 2048
          if constexpr (LQ - 6 >= 6) {
            constexpr uint32_t LH = LQ - 6;
#pragma unroll
            for (uint32_t e = 0; e < 16; ++e) {
              // node: q bits 0..LQ-6 cleared; its middle is 16-aligned
              const uint32_t qn = (e << (LQ - 4)) | (lb1 << (LQ - 5)) | (1u << LH);
              BOS_TR(0, 6, ms * TPM + (qn >> 4));
              const uint32_t m = sign_mask(spfx[ms * TPM + (qn >> 4)] - (rest << (31u - LH)));
              const T pr = dpp<kDppXor1>(rv[e]);
              const uint32_t pt = dpp<kDppXor1>(tv[e]);
              rv[e] = msel(m, pr, rv[e]);
              tv[e] = msel(m, pt, tv[e]);
            }
          }
          // -- layout B, q bit LQ-5 (lane bit 1), for Z >= 1024
          if constexpr (LQ - 5 >= 6) {
            constexpr uint32_t LH = LQ - 5;
            const uint32_t il = ((lb0 << (LQ - 6)) | rest) << (31u - LH);
#pragma unroll
            for (uint32_t e = 0; e < 16; ++e) {
              const uint32_t m = sign_mask(pvh[e] - il);
              const T pr = dpp<kDppXor2>(rv[e]);
              const uint32_t pt = dpp<kDppXor2>(tv[e]);
              rv[e] = msel(m, pr, rv[e]);
              tv[e] = msel(m, pt, tv[e]);
            }
          }
          // -- layout B, q bits LQ-4 .. LQ-1: register pairs (those >= 6)
          // the lane's part of the pair index, scaled for each of the four bits
          const uint32_t ilB[4] = {lowB << (35u - LQ), lowB << (34u - LQ), lowB << (33u - LQ), lowB << (32u - LQ)};
          light_begin();
#pragma unroll
          for (uint32_t eb = 0; eb < 4; ++eb) {
            if (LQ - 4 + eb < 6) continue;
            const uint32_t hb = 1u << eb;
            const uint32_t il = ilB[eb];
#pragma unroll
            for (uint32_t es = 0; es < 16; es += 2u * hb) {
              const uint32_t q = pv[es | hb] - il;
#pragma unroll
              for (uint32_t i = 0; i < hb; ++i) {
                const uint32_t m = sign_mask(q - (i << (31u - eb)));
                mswap(m, rv[es + i], tv[es + i], rv[es + i + hb], tv[es + i + hb]);
              }
            }
          }
          light_end();
        }
      }
      // -- hand the level's output to LDS (next level or last-pass finish)
      if (WAVEX && (d + 1 < klev || LAST)) {
        if (d + 1 < klev) swap_buckets(d);
      } else if (d + 1 < klev || LAST) {
        if constexpr (HAS_B) {
          // every lane rewrites exactly the layout-B slots it read: no
          // barrier (HALF: the first halves; the next level's start, or the
          // last pass's finish, completes the exchange)
          if (active) {
#pragma unroll
            for (uint32_t e = 0; e < 16; ++e) {
              const uint32_t pi = b_index(e, base0, base1, baseB0, baseB1, lowB);
              BOS_TR(0, 4, pi);
              BOS_TR(0, 5, pi);
              if constexpr (HALF)
                shalf[pi] = rec_lo(rv[e]);
              else
                srec[pi] = rv[e];
              stag[pi] = tv[e];
            }
          }
          pb0 = base0;
          pb1 = base1;
          pbB0 = baseB0;
          pbB1 = baseB1;
          plB = lowB;
        } else {
          if (active) {
#pragma unroll
            for (uint32_t e = 0; e < 16; ++e) {
              BOS_TR(0, 4, baseA + e);
              BOS_TR(0, 5, baseA + e);
              srec[baseA + e] = rv[e];
              stag[baseA + e] = tv[e];
            }
          }
        }
        lds_barrier();
      } else {
        // last level of a non-last pass: write the 2^klev output buckets
        // (LDS bucket S is output digit bitrev(S)) straight from registers
        T* RO = static_cast<T*>(a.rec_out);
        const uint64_t og = (h << (i0 + klev)) + (r << klev);
        const uint64_t ob0 = og + brev_k(S0, klev), ob1 = og + brev_k(S1, klev);
        // staged chunk: its groups' buckets follow each other
        const uint64_t so =
            a.staged ? (og - ((h - a.in_h0) << (a.in_lseg + klev)) - ((r - a.in_r0) << klev)) << LZ : 0ull;
        if (active) {
#pragma unroll
          for (uint32_t e = 0; e < 16; ++e) {
            uint64_t gi;
            if constexpr (HAS_B) {
              const uint32_t s = ((e & 7u) << (LQ - 4)) | lowB;
              gi = (((e < 8) ? ob0 : ob1) << LZ) + s;
            } else {
              gi = (((lt < HALF_LANES) ? ob0 : ob1) << LZ) + sb_load + e;
            }
            BOS_TR(0, 10, gi);
            BOS_TR(0, 11, gi);
            RO[gi - so] = rv[e];
            a.tag_out[gi - so] = tv[e];
          }
        }
      }
    }
  };

  // split last pass: every bin's slots in layout P, then compaction and
  // the write of its reals
  auto finish_bins_split = [&](uint32_t blk) {
    if constexpr (WAVEX) {
      // layout A of the last level's MergeSplit is layout P of its two bins
      wave_exchange([&](uint32_t e) { return slot_b + 66u * e; }, [&](uint32_t e) { return slot_a + e; });
      lds_barrier();  // every bin's load is in sload, every prefix has been read
      const uint32_t S = (tid >> 6) + (lt < HALF_LANES ? 0u : NB / 2u);
      finish_split<R, LZ, SPLIT_FIN, FULL, true>(a, blk, klev, srec, stag, srhi, saux, sload, spfx, swave, rv, tv, S);
    } else if constexpr (HALF) {
      const uint32_t HLn = Z >> 4;
      const uint32_t S = active ? tid / HLn : 0u, lq = active ? tid % HLn : 0u;
      const uint32_t pbase = S * ZP + 17u * lq;
      half_finish([&](uint32_t e) { return b_index(e, pb0, pb1, pbB0, pbB1, plB); },
                  [&](uint32_t e) { return pbase + e; }, [] { lds_barrier(); });
      finish_split<R, LZ, SPLIT_FIN, FULL, true>(a, blk, klev, srec, stag, srhi, saux, sload, spfx, swave, rv, tv, S);
    } else {
      finish_split<R, LZ, SPLIT_FIN, FULL, false>(a, blk, klev, srec, stag, srhi, saux, sload, spfx, swave, rv, tv,
                                                  active ? tid / (Z >> 4) : 0u);
    }
  };

  if constexpr (BATCH && (!LAST || SPLIT)) {
    issue_load(item0, rv, tv);
    finish_load(item0, tv);
    process(item0);
    if constexpr (SPLIT) finish_bins_split(item0);
  } else if constexpr (!LAST || SPLIT) {
    // persistent walk over blocks: item = blockIdx.x, + gridDim.x, ...  The
    // next block's loads are issued after the current one is done: with no
    // prefetch registers a pass runs three workgroups per CU at 2^3 Z slots
    // per block, and their interleaving hides the loads better than a
    // register prefetch with fewer workgroups did.
    // global index of the launch's block t: in a staged launch, block t mod
    // 2^in_lseg of the chunk's group t >> in_lseg
    auto block_index = [&](uint32_t t) -> uint32_t {
      if (!a.staged) return t;
      return uint32_t(((a.in_h0 + (t >> a.in_lseg)) << i0) + a.in_r0 + (t & ((1u << a.in_lseg) - 1u)));
    };
    uint32_t t = item0;
    if (t >= nitems) return;
    uint32_t item = block_index(t);
    issue_load(item, rv, tv);
    finish_load(item, tv);
    for (;;) {
      const uint32_t next = t + gridDim.x;
      const bool has_next = next < nitems;
      process(item);
      if constexpr (SPLIT) finish_bins_split(item);
      if (!has_next) break;
      t = next;
      item = block_index(t);
      lds_barrier();  // LDS of the previous block is no longer read
      issue_load(item, rv, tv);
      finish_load(item, tv);
    }
  } else {
    // Last pass: one block per launch block; the block index is a ticket so
    // that the look-back of the strip only waits on blocks that started
    // earlier.
    if (tid == 0) smisc[0] = atomicAdd(a.ticket, 1u);
    lds_barrier();
    const uint32_t blk = smisc[0];
    issue_load(blk, rv, tv);
    finish_load(blk, tv);
    process(blk);
    // every final bin (LDS bucket S) now sits in LDS with padded slots
    finish_bins<R, LZ, FULL>(a, blk, klev, srec, stag, srhi, saux, sload, soff, spfx, swave);
  }
  (void)nitems;
}

template <int R, int LZ, int MODE>
__global__ __launch_bounds__(kMaxThreads) void route_kernel(PassArgs a, uint32_t nitems) {
  route_run<R, LZ, MODE, false>(a, nitems, blockIdx.x);
}

// The passes whose LDS exchanges go in two halves (64 <= Z < 512, passes after
// the first) or wave by wave (Z = 512) are compiled for a register budget that
// lets as many workgroups share a CU as their LDS allows: 8-byte records four
// waves per SIMD (at most 128 VGPRs), 16-byte ones two (at three, 168 VGPRs,
// the Z = 512 passes spill 36 registers and take 0.355 ms instead of 0.303 at
// n = 2^24, k = 3; two waves also pair up for light instructions).
template <int R, int LZ, int MODE>
constexpr bool kW3 = lds_rec_bytes(R, 1u << LZ, (MODE & 2) && !(MODE & 4)) < uint32_t(R) && LZ >= 6 &&
                     (LZ == 9 || !(MODE & 1));
template <int R, int LZ>
constexpr int kWavesPerSimd = R == 8 ? 4 : LZ == 9 ? 2 : 3;

template <int R, int LZ, int MODE>
__global__ __launch_bounds__(kMaxThreads) __attribute__((amdgpu_waves_per_eu(kWavesPerSimd<R, LZ>, 8))) void
route_kernel_w3(PassArgs a, uint32_t nitems) {
  route_run<R, LZ, MODE, false>(a, nitems, blockIdx.x);
}

// Batched routing: segment s of the launch is one instance's pass; its blocks
// are blockIdx.x in [blk_start[s], blk_start[s+1]).
template <int R, int LZ, int MODE>
__device__ __forceinline__ void route_b_body(const PassArgs* segs, const uint32_t* blk_start, uint32_t nsegs) {
  uint32_t lo = 0, hi = nsegs;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (blk_start[mid] <= blockIdx.x)
      lo = mid;
    else
      hi = mid;
  }
  const PassArgs a = segs[lo];
  route_run<R, LZ, MODE, true>(a, 0u, blockIdx.x - blk_start[lo]);
}
template <int R, int LZ, int MODE>
__global__ __launch_bounds__(kMaxThreads) void route_kernel_b(const PassArgs* segs, const uint32_t* blk_start,
                                                              uint32_t nsegs) {
  route_b_body<R, LZ, MODE>(segs, blk_start, nsegs);
}
template <int R, int LZ, int MODE>
__global__ __launch_bounds__(kMaxThreads) __attribute__((amdgpu_waves_per_eu(kWavesPerSimd<R, LZ>, 8))) void
route_kernel_b_w3(const PassArgs* segs, const uint32_t* blk_start, uint32_t nsegs) {
  route_b_body<R, LZ, MODE>(segs, blk_start, nsegs);
}

}  // namespace bos
