// strip_kernels.hip — strip of the dummies after the split form of the last
// routing pass (Section 3.2: the bins' reals, concatenated in bin order, are
// the permuted array).
//
// The last pass leaves bin gb's reals in slots gb*Z .. gb*Z + loads[gb] - 1 of
// the binned array and every routing block's real count in bsum[blk].  One
// workgroup scans the block counts into output offsets; the strip kernel then
// copies each block's bins to their offsets.  Every address is a function of
// the loads, which the method reveals (they are what a simulator of the
// access pattern gets, Lemma 3.3).
//
// The bins arrive compacted but unsorted (reals in the order the last level
// left them).  The comparison sort that follows (Section 3.3) starts with an
// oblivious sort of fixed tiles of `tile` records: a bin inside one tile is
// put in order with its tile, so its inner order never shows.  A bin that
// straddles a tile boundary would hand the tiles a split that depends on the
// input order, so the strip sorts such a bin (an oblivious network in LDS)
// before writing it: its lower records go to the first tile.  Which bins
// straddle depends on the loads only.
#include "bos_common.h"

namespace bos {

constexpr uint32_t kScanThreads = 1024;
constexpr uint32_t kStripThreads = 256, kStripItems = 8;

// In-place exclusive scan of v[0..count) by one workgroup: each thread sums a
// contiguous chunk, the chunk sums are scanned in LDS, then each thread
// rewrites its chunk.
__device__ __forceinline__ void scan_blocks(unsigned long long* v, uint32_t count) {
  __shared__ unsigned long long part[kScanThreads];
  const uint32_t t = threadIdx.x;
  const uint32_t per = (count + kScanThreads - 1) / kScanThreads;
  const uint32_t b = t * per < count ? t * per : count, e = b + per < count ? b + per : count;
  unsigned long long sum = 0;
  for (uint32_t i = b; i < e; ++i) {
    BOS_TR(0, 30, i);
    sum += v[i];
  }
  BOS_TR(0, 31, t);
  part[t] = sum;
  __syncthreads();
  for (uint32_t off = 1; off < kScanThreads; off <<= 1) {
    if (t >= off) BOS_TR(0, 31, t - off);
    const unsigned long long x = t >= off ? part[t - off] : 0ull;
    __syncthreads();
    BOS_TR(0, 31, t);
    part[t] += x;
    __syncthreads();
  }
  BOS_TR(0, 31, t);
  unsigned long long run = part[t] - sum;
  for (uint32_t i = b; i < e; ++i) {
    BOS_TR(0, 30, i);
    const unsigned long long x = v[i];
    v[i] = run;
    run += x;
  }
}

__global__ __launch_bounds__(kScanThreads) void scan_blocks_kernel(unsigned long long* v, uint32_t count) {
  scan_blocks(v, count);
}

// First level of the block-count scan: workgroup c turns v[c*1024 ..
// c*1024 + 1023] into its exclusive scan in place (coalesced, one count per
// thread) and writes the chunk's total to tot[c]; a second, one-workgroup
// scan of tot gives every chunk's offset.  One chunk (at most 1024 blocks) has
// offset 0 and writes it itself: no second launch (4.6 us of a small sort).
__global__ __launch_bounds__(kScanThreads) void scan_chunks_kernel(unsigned long long* v, uint32_t count,
                                                                   unsigned long long* tot) {
  __shared__ unsigned long long wsum[kScanThreads / 64];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wv = tid >> 6;
  const uint64_t idx = uint64_t(blockIdx.x) * kScanThreads + tid;
  if (idx < count) BOS_TR(0, 30, idx);
  const unsigned long long x = idx < count ? v[idx] : 0ull;
  unsigned long long incl = x;
#pragma unroll
  for (uint32_t o = 1; o < 64; o <<= 1) {
    const unsigned long long y = __shfl_up(incl, o, 64);
    if (lane >= o) incl += y;
  }
  if (lane == 63) {
    BOS_TR(0, 31, wv);
    wsum[wv] = incl;
  }
  __syncthreads();
  unsigned long long before = 0, total = 0;
#pragma unroll
  for (uint32_t w = 0; w < kScanThreads / 64; ++w) {
    BOS_TR(0, 31, w);
    const unsigned long long t = wsum[w];
    before += w < wv ? t : 0ull;
    total += t;
  }
  if (idx < count) {
    BOS_TR(0, 30, idx);
    v[idx] = before + incl - x;
  }
  if (tid == 0) {
    BOS_TR(0, 32, blockIdx.x);
    tot[blockIdx.x] = gridDim.x == 1 ? 0ull : total;
  }
}

// Bitonic sort of sb[0..P2) by (key, payload) (P2 a power of two), by the
// whole workgroup.  A wave's 64 pairs of a stage of stride <= 64 lie in 128
// slots that only this wave touches, whatever the stride, so such stages follow
// each other without a barrier (the LDS unit runs a wave's accesses in order);
// only strides above 64 need one on either side.
template <typename T>
__device__ __forceinline__ void lds_bitonic(T* sb, uint32_t P2) {
  for (uint32_t size = 2; size <= P2; size <<= 1) {
    for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
      for (uint32_t t = threadIdx.x; t < P2 / 2; t += kStripThreads) {
        const uint32_t i = ((t & ~(stride - 1u)) << 1) | (t & (stride - 1u)), k = i + stride;
        const bool asc = (i & size) == 0;
        BOS_TR(0, 33, i);
        BOS_TR(0, 33, k);
        const T x = sb[i], y = sb[k];
        const bool swap = asc ? rec_less(y, x) : rec_less(x, y);
        sb[i] = sel(swap, y, x);
        sb[k] = sel(swap, x, y);
      }
      // the next stage's stride: half of this one, or the next size's first
      const uint32_t next = stride > 1 ? stride >> 1 : size;
      if (stride > 64 || next > 64) {
        __syncthreads();
      } else {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
  __syncthreads();
}

// One routing block's bins (NB = 2^klev of them) to out[boff[blk] + coff[blk /
// 1024] ..) (coff null: boff alone); bins that straddle a multiple of `tile`
// are sorted first (tile = 0: none).
template <int R>
__device__ __forceinline__ void strip_block(const void* binned_, const uint32_t* loads,
                                            const unsigned long long* boff, const unsigned long long* coff,
                                            void* out_, uint64_t n, uint32_t klev, uint32_t lz, uint64_t blk,
                                            uint32_t tile) {
  using T = typename RecOf<R>::T;
  __shared__ uint32_t pre[513];  // NB <= 512: a block has at most 8192 slots, Z >= 16
  __shared__ uint16_t strad[512];
  __shared__ uint8_t sorted[512];  // bin straddles a tile: written sorted
  __shared__ uint32_t nstrad;
  __shared__ __align__(16) unsigned char sbin_raw[2048 * R];  // one bin of at most Z <= 2048 reals
  const T* binned = static_cast<const T*>(binned_);
  T* out = static_cast<T*>(out_);
  const uint32_t tid = threadIdx.x, NB = 1u << klev;
  const uint64_t bin0 = blk << klev;
  BOS_TR(0, 36, blk);
  const uint64_t base = boff[blk] + (coff ? coff[blk / kScanThreads] : 0ull);
  // wave 0, 64 bins at a time: prefix sums of the loads and the list, in bin
  // order, of the bins that straddle a tile (tile is a power of two)
  if (tid < 64) {
    const uint32_t tl = tile ? uint32_t(__builtin_ctz(tile)) : 0u;
    uint32_t run = 0, ns = 0;
    for (uint32_t j0 = 0; j0 < NB; j0 += 64) {
      const uint32_t j = j0 + tid;
      if (j < NB) BOS_TR(0, 34, bin0 + j);
      const uint32_t ld = j < NB ? loads[bin0 + j] : 0u;
      uint32_t incl = ld;
#pragma unroll
      for (uint32_t o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o, 64);
        if (tid >= o) incl += y;
      }
      const uint64_t b1 = base + run + incl, b0 = b1 - ld;
      const bool st = tile && ld >= 2 && (b0 >> tl) != ((b1 - 1) >> tl);
      const unsigned long long m = __ballot(st);
      if (j < NB) {
        BOS_TR(0, 35, j);
        pre[j] = run + incl - ld;
        sorted[j] = st;
        if (st) {
          const uint32_t c = ns + uint32_t(__popcll(m & ((1ull << tid) - 1ull)));
          BOS_TR(0, 37, c);
          strad[c] = uint16_t(j);
        }
      }
      run += uint32_t(__shfl(int(incl), 63, 64));
      ns += uint32_t(__popcll(m));
    }
    if (tid == 0) {
      BOS_TR(0, 35, NB);
      pre[NB] = run;
      nstrad = ns;
    }
  }
  __syncthreads();
  BOS_TR(0, 35, NB);
  const uint32_t total = pre[NB];
  if (tile) {
    T* sb = reinterpret_cast<T*>(sbin_raw);
    const uint32_t ns = nstrad;
    for (uint32_t k = 0; k < ns; ++k) {
      const uint32_t j = strad[k], ld = pre[j + 1] - pre[j];
      uint32_t P2 = 2;
      while (P2 < ld) P2 <<= 1;
      const T* src = binned + ((bin0 + j) << lz);
      for (uint32_t i = tid; i < P2; i += kStripThreads) {
        if (i < ld) BOS_TR(0, 38, ((bin0 + j) << lz) + i);
        BOS_TR(0, 33, i);
        sb[i] = i < ld ? src[i] : max_rec<T>();
      }
      __syncthreads();
      lds_bitonic(sb, P2);
      const uint64_t o = base + pre[j];
      for (uint32_t i = tid; i < ld; i += kStripThreads)
        if (o + i < n) {
          BOS_TR(0, 33, i);
          BOS_TR(0, 39, o + i);
          out[o + i] = sb[i];
        }
      __syncthreads();
    }
  }
  using V = typename NativeOf<T>::V;  // native vectors stay in registers
  const V* bv = reinterpret_cast<const V*>(binned);
  V* ov = reinterpret_cast<V*>(out);
  for (uint32_t q0 = 0; q0 < total; q0 += kStripThreads * kStripItems) {
    V v[kStripItems];
    uint64_t dst[kStripItems];
#pragma unroll
    for (uint32_t k = 0; k < kStripItems; ++k) {
      const uint32_t q = q0 + k * kStripThreads + tid;
      // bin j: the last with pre[j] <= q (lanes past the end read bin 0's
      // first slot and store nothing)
      const uint32_t qq = q < total ? q : 0u;
      uint32_t lo = 0, hi = NB;
      while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        BOS_TR(0, 35, mid);
        if (pre[mid] <= qq)
          lo = mid;
        else
          hi = mid;
      }
      // a straddling bin was written sorted above
      BOS_TR(0, 37, lo);
      const bool done = sorted[lo] != 0;
      BOS_TR(0, 35, lo);
      BOS_TR(0, 38, ((bin0 + lo) << lz) + (qq - pre[lo]));
      v[k] = bv[((bin0 + lo) << lz) + (qq - pre[lo])];
      dst[k] = q < total && !done ? base + q : ~0ull;
    }
#pragma unroll
    for (uint32_t k = 0; k < kStripItems; ++k)
      if (dst[k] < n) {
        BOS_TR(0, 39, dst[k]);
        ov[dst[k]] = v[k];
      }
  }
}

template <int R>
__global__ __launch_bounds__(kStripThreads) void strip_kernel(const void* binned, const uint32_t* loads,
                                                              const unsigned long long* boff,
                                                              const unsigned long long* coff, void* out, uint64_t n,
                                                              uint32_t klev, uint32_t lz, uint32_t tile) {
  strip_block<R>(binned, loads, boff, coff, out, n, klev, lz, blockIdx.x, tile);
}

// Batched forms: one scan workgroup per instance; the strip workgroups of
// instance s are blockIdx.x in [segs[s].first, segs[s].first + nblocks).
__global__ __launch_bounds__(kScanThreads) void scan_blocks_kernel_b(const StripSeg* segs) {
  const StripSeg sg = segs[blockIdx.x];
  scan_blocks(sg.bsum, sg.nblocks);
}

template <int R>
__global__ __launch_bounds__(kStripThreads) void strip_kernel_b(const StripSeg* segs, uint32_t nsegs) {
  uint32_t lo = 0, hi = nsegs;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (segs[mid].first <= blockIdx.x)
      lo = mid;
    else
      hi = mid;
  }
  const StripSeg sg = segs[lo];
  strip_block<R>(sg.binned, sg.loads, sg.bsum, nullptr, sg.out, sg.n, sg.klev, sg.lz, blockIdx.x - sg.first,
                 sg.tile);
}

// Batched scan + strip over nsegs instances (device table segs, `blocks` strip
// workgroups in all).
hipError_t launch_strip_batched(int rec, const StripSeg* segs, uint32_t nsegs, uint32_t blocks, hipStream_t s) {
  BOS_TRACE_BIND();
  if (nsegs == 0) return hipSuccess;
  hipLaunchKernelGGL(scan_blocks_kernel_b, dim3(nsegs), dim3(kScanThreads), 0, s, segs);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || blocks == 0) return e;
  if (rec == 8)
    hipLaunchKernelGGL(strip_kernel_b<8>, dim3(blocks), dim3(kStripThreads), 0, s, segs, nsegs);
  else
    hipLaunchKernelGGL(strip_kernel_b<16>, dim3(blocks), dim3(kStripThreads), 0, s, segs, nsegs);
  return hipGetLastError();
}

// The two-level scan of the block counts alone (bos_orp's finish reads the
// offsets): bsum scanned in place within chunks of 1024, coff the chunk offsets.
hipError_t launch_block_scan(unsigned long long* bsum, unsigned long long* coff, uint32_t nblocks, hipStream_t s) {
  BOS_TRACE_BIND();
  if (nblocks == 0 || !coff) return hipErrorInvalidValue;
  const uint32_t nchunks = (nblocks + kScanThreads - 1) / kScanThreads;
  hipLaunchKernelGGL(scan_chunks_kernel, dim3(nchunks), dim3(kScanThreads), 0, s, bsum, nblocks, coff);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || nchunks == 1) return e;
  hipLaunchKernelGGL(scan_blocks_kernel, dim3(1), dim3(kScanThreads), 0, s, coff, nchunks);
  return hipGetLastError();
}

// tile: records per tile of the comparison sort's first phase (bins that
// straddle a tile boundary are sorted); lz <= 11.  coff: device,
// nblocks / 1024 + 1 words (the chunk offsets of the two-level scan).
hipError_t launch_strip(int rec, const void* binned, const uint32_t* loads, unsigned long long* bsum,
                        unsigned long long* coff, void* out, uint64_t n, uint32_t nblocks, uint32_t klev, uint32_t lz,
                        uint32_t tile, hipStream_t s) {
  BOS_TRACE_BIND();
  if (klev > 9 || lz > 11 || nblocks == 0 || (tile & (tile - 1u)) || !coff) return hipErrorInvalidValue;
  const hipError_t e = launch_block_scan(bsum, coff, nblocks, s);
  if (e != hipSuccess) return e;
  if (rec == 8)
    hipLaunchKernelGGL(strip_kernel<8>, dim3(nblocks), dim3(kStripThreads), 0, s, binned, loads, bsum, coff, out, n,
                       klev, lz, tile);
  else
    hipLaunchKernelGGL(strip_kernel<16>, dim3(nblocks), dim3(kStripThreads), 0, s, binned, loads, bsum, coff, out, n,
                       klev, lz, tile);
  return hipGetLastError();
}

}  // namespace bos

namespace bos {

// words[0] = the overflow word, words[1] = the sum of the nb block counts: what
// the host reads of an out-of-core sort's chunk before it sorts it.
__global__ __launch_bounds__(256) void chunk_words_kernel(const unsigned long long* status,
                                                          const unsigned long long* counts, uint32_t nb,
                                                          unsigned long long* words) {
  __shared__ unsigned long long wsum[4];
  unsigned long long t = 0;
  for (uint32_t i = threadIdx.x; i < nb; i += 256) {
    BOS_TR(0, 14, i);
    t += counts[i];
  }
#pragma unroll
  for (uint32_t o = 32; o > 0; o >>= 1) t += __shfl_down(t, o, 64);
  if ((threadIdx.x & 63u) == 0) wsum[threadIdx.x >> 6] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
    words[0] = *status;
    words[1] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
  }
}
hipError_t launch_chunk_words(const unsigned long long* status, const unsigned long long* counts, uint32_t nb,
                              unsigned long long* words, hipStream_t s) {
  BOS_TRACE_BIND();
  hipLaunchKernelGGL(chunk_words_kernel, dim3(1), dim3(256), 0, s, status, counts, nb, words);
  return hipGetLastError();
}

// Loads of the buckets that the last K <= kCountLevels levels will form, from the
// slots that enter the first of them (out of core: the trip before the last), so
// that an overflow of those levels is known before they run.  cnt[d * B + b] counts
// the reals that level i0 + d puts into its output bucket b; of input bucket g = (m,
// r), those whose label's low K bits start with the d + 1 bits p go to bucket ((m >>
// (d + 1)) << (i0 + d + 1)) + (r << (d + 1)) + p.  A wave takes a bucket: lane v
// counts value v of the K bits by ballots, and the lanes fold in pairs from one level
// to the next, so that every address is a function of (bucket, K) only.  64 ballots
// a line of tags at most: under 2 % of the time that the chunk takes on the link.
__global__ __launch_bounds__(256) void count_buckets_kernel(const uint32_t* tags, uint32_t* cnt, uint64_t nbk,
                                                            uint64_t g0, uint32_t lz, uint32_t i0, uint32_t K,
                                                            uint64_t B) {
  const uint32_t lane = threadIdx.x & 63u, Z = 1u << lz, nv = 1u << K;
  const uint64_t u = uint64_t(blockIdx.x) * 4u + (threadIdx.x >> 6);
  if (u >= nbk) return;
  uint32_t c = 0;
  for (uint32_t s0 = 0; s0 < Z; s0 += 64) {
    uint32_t t = kDummyTag;
    if (s0 + lane < Z) {
      BOS_TR(0, 2, (u << lz) + s0 + lane);
      t = tags[(u << lz) + s0 + lane];
    }
    t = int32_t(t) < 0 ? kDummyTag : t & (nv - 1u);
    for (uint32_t v = 0; v < nv; ++v) {
      const uint32_t n = uint32_t(__popcll(__ballot(t == v)));
      c += lane == v ? n : 0u;
    }
  }
  const uint64_t g = g0 + u, m = g >> i0, r = g & ((1ull << i0) - 1ull);
  for (uint32_t d = K; d-- > 0;) {
    if (lane < (2u << d)) {
      const uint64_t at = d * B + (((m >> (d + 1)) << (i0 + d + 1)) | (r << (d + 1)) | lane);
      BOS_TR(0, 54, at);
      atomicAdd(&cnt[at], c);
    }
    c = uint32_t(__shfl(int(c), int((2u * lane) & 63u), 64)) + uint32_t(__shfl(int(c), int((2u * lane + 1u) & 63u), 64));
  }
}
__global__ __launch_bounds__(256) void count_check_kernel(const uint32_t* cnt, uint64_t total, uint64_t B, uint32_t i0,
                                                          uint32_t Z, unsigned long long* status) {
  const uint64_t step = uint64_t(gridDim.x) * 256u;
  for (uint64_t i = uint64_t(blockIdx.x) * 256u + threadIdx.x; i < total; i += step) {
    BOS_TR(0, 54, i);
    if (cnt[i] > Z) atomicMin(status, (unsigned long long)(((i0 + i / B) << 32) | ((i % B) >> 1)));
  }
}
// Adds nbk buckets from global bucket g0 (tags as the level before i0 left them).
hipError_t launch_count_buckets(const void* tags, uint32_t* cnt, uint64_t nbk, uint64_t g0, uint32_t lz, uint32_t i0,
                                uint32_t K, uint64_t B, hipStream_t s) {
  BOS_TRACE_BIND();
  if (K == 0 || K > kCountLevels || nbk == 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(count_buckets_kernel, dim3(uint32_t((nbk + 3) / 4)), dim3(256), 0, s,
                     static_cast<const uint32_t*>(tags), cnt, nbk, g0, lz, i0, K, B);
  return hipGetLastError();
}
// Folds the first overflow among the counted levels into the overflow word.
hipError_t launch_count_check(const uint32_t* cnt, uint32_t i0, uint32_t K, uint64_t B, uint32_t Z,
                              unsigned long long* status, hipStream_t s) {
  BOS_TRACE_BIND();
  hipLaunchKernelGGL(count_check_kernel, dim3(1024), dim3(256), 0, s, cnt, K * B, B, i0, Z, status);
  return hipGetLastError();
}

// Slots of an out-of-core trip as they cross the host link: units of 2^lu slots
// (a segment of the next trip), each its records followed by its tags, so that a
// segment is one copy.  A tag keeps the label bits that the next levels read, in
// TB = 1, 2 or 4 bytes, all ones for a dummy: 9 to 12 bytes a slot of 8-byte
// records over the link that bounds a trip (2^25 slots with 4 bits left: 302
// MB in place of 403).  A thread moves four slots; device copies of a chunk, far
// above the link's rate.
uint32_t packed_tag_bytes(uint32_t bits) { return bits < 8 ? 1u : bits < 16 ? 2u : 4u; }
template <typename TB>
__device__ __forceinline__ uint32_t widen_tag(TB v) {
  return v == TB(~TB(0)) ? kDummyTag : uint32_t(v);
}
template <int R, typename TB, bool PACK>
__global__ __launch_bounds__(256) void pack_slots_kernel(const char* rec_in, const char* tag_in, char* rec_out,
                                                         char* tag_out, uint64_t slots, uint32_t lu, uint32_t mask) {
  using T = typename RecOf<R>::T;
  typedef TB V __attribute__((ext_vector_type(4)));
  const uint64_t q = (uint64_t(blockIdx.x) * 256u + threadIdx.x) * 4u;
  if (q >= slots) return;
  const uint64_t unit = q >> lu, at = q & ((1ull << lu) - 1ull);
  const uint64_t r = (unit << lu) * (R + sizeof(TB)) + at * R;
  const uint64_t t = (unit << lu) * (R + sizeof(TB)) + (uint64_t(R) << lu) + at * sizeof(TB);
  BOS_TR(0, 55, q);  // four slots
  BOS_TR(0, 56, r);  // their packed records
  BOS_TR(0, 57, t);  // and tags
  if constexpr (PACK) {
    const uint4 w = *reinterpret_cast<const uint4*>(tag_in + q * 4);
    const T* ri = reinterpret_cast<const T*>(rec_in) + q;
    T* ro = reinterpret_cast<T*>(rec_out + r);
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) ro[i] = ri[i];
    // (a dummy's tag is all ones, a label is below 2^31)
    auto narrow = [&](uint32_t v) { return TB((v & mask) | uint32_t(int32_t(v) >> 31)); };
    *reinterpret_cast<V*>(rec_out + t) = V{narrow(w.x), narrow(w.y), narrow(w.z), narrow(w.w)};
  } else {
    const T* ri = reinterpret_cast<const T*>(rec_in + r);
    const V ti = *reinterpret_cast<const V*>(rec_in + t);
    T* ro = reinterpret_cast<T*>(rec_out) + q;
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) ro[i] = ri[i];
    *reinterpret_cast<uint4*>(tag_out + q * 4) =
        make_uint4(widen_tag(ti[0]), widen_tag(ti[1]), widen_tag(ti[2]), widen_tag(ti[3]));
  }
}

template <int R, bool PACK>
static hipError_t launch_slots(const void* rec_in, const void* tag_in, void* rec_out, void* tag_out, uint64_t slots,
                               uint32_t lu, uint32_t bits, hipStream_t s) {
  BOS_TRACE_BIND();
  const uint32_t tb = packed_tag_bytes(bits), mask = (1u << bits) - 1u;
  const dim3 grid(uint32_t((slots / 4 + 255) / 256)), block(256);
  const char *ri = static_cast<const char*>(rec_in), *ti = static_cast<const char*>(tag_in);
  char *ro = static_cast<char*>(rec_out), *to = static_cast<char*>(tag_out);
  if (tb == 1)
    hipLaunchKernelGGL((pack_slots_kernel<R, uint8_t, PACK>), grid, block, 0, s, ri, ti, ro, to, slots, lu,
                       mask);
  else if (tb == 2)
    hipLaunchKernelGGL((pack_slots_kernel<R, uint16_t, PACK>), grid, block, 0, s, ri, ti, ro, to, slots, lu,
                       mask);
  else
    hipLaunchKernelGGL((pack_slots_kernel<R, uint32_t, PACK>), grid, block, 0, s, ri, ti, ro, to, slots, lu,
                       mask);
  return hipGetLastError();
}

// slots and 2^lu: multiples of 16 (a bucket holds at least 16 slots), slots a
// multiple of 2^lu; bits < 32 label bits left.
hipError_t launch_pack_slots(int rec, const void* recs, const void* tags, void* out, uint64_t slots, uint32_t lu,
                             uint32_t bits, hipStream_t s) {
  return rec == 8 ? launch_slots<8, true>(recs, tags, out, nullptr, slots, lu, bits, s)
                  : launch_slots<16, true>(recs, tags, out, nullptr, slots, lu, bits, s);
}
hipError_t launch_unpack_slots(int rec, const void* in, void* recs, void* tags, uint64_t slots, uint32_t lu,
                               uint32_t bits, hipStream_t s) {
  return rec == 8 ? launch_slots<8, false>(in, nullptr, recs, tags, slots, lu, bits, s)
                  : launch_slots<16, false>(in, nullptr, recs, tags, slots, lu, bits, s);
}

}  // namespace bos
