// Zero-padding algorithm (Sec. III-D, Fig. 4): prefix sum of the mask matrix,
// position array, pack and unpack.  Integer / byte work: bit-exact.
#include <atomic>
#include <chrono>

#include "common.h"

namespace bt {
bt_status build_offsets(const int32_t* d_mask, const int32_t* d_lengths, int B, int S, int32_t* d_cu_seqlens,
                        int32_t* d_token_idx, int32_t* h_out, bool stats, bt_stream stream, void (*meanwhile)(void*),
                        void* context);

constexpr int kOffsetsThreads = 1024;  // 16 wavefronts
constexpr int kOffsetsWaves = kOffsetsThreads / kWave;

// Inclusive prefix sum over the wavefront on data-parallel-primitive moves: shifts by 1, 2, 4, 8 inside each row of
// 16 lanes, then the last lane of a row broadcast to the rows behind it.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
  return v;
}

// Exclusive prefix sum of v over the workgroup (1024 threads); *total receives the sum.  s_part: LDS, 16 words.
// The caller separates two uses of s_part by a barrier.
__device__ __forceinline__ int block_exclusive_scan(int v, int* s_part, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int x = wave_inclusive_scan(v);
  if (lane == kWave - 1) s_part[wave] = x;
  __syncthreads();
  // every row of 16 lanes scans the 16 wave sums
  int p = s_part[lane & 15];
  p += __builtin_amdgcn_update_dpp(0, p, 0x111, 0xf, 0xf, false);
  p += __builtin_amdgcn_update_dpp(0, p, 0x112, 0xf, 0xf, false);
  p += __builtin_amdgcn_update_dpp(0, p, 0x114, 0xf, 0xf, false);
  p += __builtin_amdgcn_update_dpp(0, p, 0x118, 0xf, 0xf, false);
  *total = __builtin_amdgcn_readlane(p, 15);
  const int w = __builtin_amdgcn_readfirstlane(wave);
  return (w ? __builtin_amdgcn_readlane(p, w - 1) : 0) + x - v;
}

__device__ __forceinline__ void publish_total(int total, int longest, bool bad, int32_t* host_total, int32_t* max_out) {
  if (max_out) *max_out = longest;
  if (host_total) {
    if (max_out) __hip_atomic_store(host_total + 1, longest, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(host_total, bad ? -1 : total, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// Both kernels: an invalid entry (a length outside [0,S], a mask entry outside {0,1}) sets cu[B] = -1.
// host_total (optional): device-visible host memory that receives the total (or -1) as soon as it is known, so
// that the host can go on without a stream sync.  max_out (optional): device word that receives the largest
// per-sentence valid count; with host_total it is also stored to host_total[1], before the total, so that a host
// that sees the total sees it too.

// Lengths.  Every workgroup scans all lengths (a few KB, 1024 at a time), workgroup 0 writes cu and the total,
// and each of the grid's wavefronts writes the positions of its own sentences: the T words of token_idx leave
// through as many compute units as there are groups of 16 sentences instead of through one.
__global__ __launch_bounds__(kOffsetsThreads) void offsets_lengths_kernel(const int32_t* __restrict__ lengths, int B,
                                                                         int S, int32_t* __restrict__ cu,
                                                                         int32_t* __restrict__ token_idx,
                                                                         int32_t* host_total, int32_t* max_out) {
  __shared__ int s_part[kOffsetsWaves], s_base[kOffsetsThreads], s_len[kOffsetsThreads], s_bad, s_max;
  const int tid = threadIdx.x, lane = tid & 63;
  const int gwave = (int)blockIdx.x * kOffsetsWaves + (tid >> 6), nwave = (int)gridDim.x * kOffsetsWaves;
  if (tid == 0) { s_bad = 0; s_max = 0; }
  int running = 0;
  for (int b0 = 0;; b0 += kOffsetsThreads) {  // left behind the last round: b0 + 1024 may not fit an int
    const int b = b0 + tid;
    int len = b < B ? lengths[b] : 0;
    const bool bad = len < 0 || len > S;
    if (bad) len = 0;
    __syncthreads();  // s_bad / s_max are set, the previous round's reads of the LDS arrays are done
    if (bad) s_bad = 1;
    if (max_out) {
      const int m = wave_max(len);
      if (lane == 0) atomicMax(&s_max, m);
    }
    int total;
    const int base = running + block_exclusive_scan(len, s_part, &total);
    s_base[tid] = base;
    s_len[tid] = len;
    running += total;
    __syncthreads();
    if (blockIdx.x == 0) {
      if (b < B) cu[b] = base;
      if (B - b0 <= kOffsetsThreads && tid == 0) {
        cu[B] = s_bad ? -1 : running;
        publish_total(running, s_max, s_bad != 0, host_total, max_out);
      }
    }
    const int here = min(B - b0, kOffsetsThreads);
    for (int i = (gwave - b0 % nwave + nwave) % nwave; i < here; i += nwave) {
      const int at = s_base[i], n = s_len[i], first = (b0 + i) * S;
      for (int t = lane; t < n; t += kWave) token_idx[at + t] = first + t;
    }
    if (B - b0 <= kOffsetsThreads) break;
  }
}

// Mask of 4 097 to 16 384 or more than 2^20 entries, or with the per-sentence maximum.  One workgroup; the mask is read once and kept as bits in
// LDS.  A token's entry in token_idx is its flat index b*S + t, and its position is the number of ones before it in flat
// order, so the mask is taken as
// one flat string of 64-bit words whatever S is: one prefix sum over the popcounts of the words gives the base of
// every word, and cu[b] is the prefix at flat index b*S.  A lane loads four entries at a time with kMaskLoads loads in
// flight (256 KB over the workgroup).  kMaskWords words per round (131 072 entries).
// Bound: one compute unit's read rate (~90 GB/s) for large masks, latency for small ones.  128 x 512: 54.7 us when
// each wavefront walked its sentences one dependent load at a time and read the mask twice.
constexpr int kMaskWords = 2 * kOffsetsThreads;
constexpr int kMaskLoads = 16;

__global__ __launch_bounds__(kOffsetsThreads) void offsets_mask_kernel(const int32_t* __restrict__ mask, int B, int S,
                                                                      int32_t* __restrict__ cu,
                                                                      int32_t* __restrict__ token_idx,
                                                                      int32_t* host_total, int32_t* max_out) {
  typedef int int4_t __attribute__((ext_vector_type(4)));
  __shared__ unsigned long long s_word[kMaskWords];
  __shared__ int s_pre[kMaskWords], s_part[kOffsetsWaves], s_bad, s_max;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = B * S;  // < 2^31
  const bool vec = (reinterpret_cast<uintptr_t>(mask) & 15u) == 0;
  const int sub = lane >> 4, shift = 4 * (lane & 15);  // this lane's word of a group of four, its nibble's place in it
  if (tid == 0) { s_bad = 0; s_max = 0; }
  __syncthreads();
  int running = 0;
  for (int f0 = 0; f0 < n; f0 += kMaskWords * kWave) {  // left by the break of the last round
    const int entries = min(n - f0, kMaskWords * kWave);
    const int groups = (entries + 4 * kWave - 1) / (4 * kWave);  // of four words
    const int run = (groups + kOffsetsWaves - 1) / kOffsetsWaves;
    const int g0 = wave * run, g1 = min(groups, g0 + run);
    bool bad = false;
    for (int g = g0; g < g1; g += kMaskLoads) {
      int4_t m[kMaskLoads];
#pragma unroll
      for (int k = 0; k < kMaskLoads; ++k) {
        m[k] = int4_t{0, 0, 0, 0};
        const int at = (g + k) * 4 * kWave + lane * 4;
        if (g + k < g1 && at < entries) {
          if (vec && at + 4 <= entries) {
            m[k] = *reinterpret_cast<const int4_t*>(mask + f0 + at);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (at + e < entries) m[k][e] = mask[f0 + at + e];
          }
        }
      }
#pragma unroll
      for (int k = 0; k < kMaskLoads; ++k) {
        if (g + k >= g1) break;  // wave-uniform
        bad |= ((m[k][0] | m[k][1] | m[k][2] | m[k][3]) & ~1) != 0;
        const unsigned long long nib = (unsigned)((m[k][0] & 1) | (m[k][1] & 1) << 1 | (m[k][2] & 1) << 2 | (m[k][3] & 1) << 3);
        const unsigned long long w = nib << shift;
        int lo = (int)(unsigned)w, hi = (int)(unsigned)(w >> 32);
        lo |= dpp_move<0xB1>(lo);
        hi |= dpp_move<0xB1>(hi);
        lo |= dpp_move<0x4E>(lo);
        hi |= dpp_move<0x4E>(hi);
        lo |= dpp_move<0x141>(lo);
        hi |= dpp_move<0x141>(hi);
        lo |= dpp_move<0x140>(lo);
        hi |= dpp_move<0x140>(hi);
        if ((lane & 15) == 0) s_word[(g + k) * 4 + sub] = (unsigned long long)(unsigned)hi << 32 | (unsigned)lo;
      }
    }
    if (__any(bad) && lane == 0) s_bad = 1;
    __syncthreads();
    const int words = groups * 4;
    const int c0 = 2 * tid < words ? __popcll(s_word[2 * tid]) : 0;
    const int c1 = 2 * tid < words ? __popcll(s_word[2 * tid + 1]) : 0;
    int total;
    const int base = running + block_exclusive_scan(c0 + c1, s_part, &total);
    s_pre[2 * tid] = base;
    s_pre[2 * tid + 1] = base + c0;
    running += total;
    __syncthreads();
    auto prefix = [&](int at) {  // ones before flat index f0 + at, at < entries
      return s_pre[at >> 6] + __popcll(s_word[at >> 6] & ((1ull << (at & 63)) - 1ull));
    };
    for (unsigned b = (f0 + S - 1) / S + tid; b < (unsigned)B && (long long)b * S < (long long)f0 + entries; b += kOffsetsThreads)
      cu[b] = prefix((int)b * S - f0);  // sentences that start in this round
    if (entries == n - f0) {  // last round: the total is known
      if (tid == 0) cu[B] = running;
      if (max_out) {
        __syncthreads();
        int m = 0;
        for (unsigned b = tid; b < (unsigned)B; b += kOffsetsThreads) m = max(m, cu[b + 1] - cu[b]);  // written by this workgroup
        m = wave_max(m);
        if (lane == 0) atomicMax(&s_max, m);
        __syncthreads();
      }
      if (tid == 0) {
        if (s_bad) cu[B] = -1;
        publish_total(running, s_max, s_bad != 0, host_total, max_out);
      }
    }
    for (int g = g0; g < g1; ++g) {
      const unsigned long long word = s_word[g * 4 + sub];
      int at = s_pre[g * 4 + sub] + __popcll(word & ((1ull << shift) - 1ull));
      const int nib = (int)(word >> shift) & 15, flat = f0 + g * 4 * kWave + lane * 4;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (nib >> e & 1) token_idx[at++] = flat + e;
    }
    if (entries == n - f0) break;
    __syncthreads();  // before the next round overwrites the LDS arrays
  }
  if (n == 0 && tid == 0) {
    cu[0] = 0;
    publish_total(0, 0, false, host_total, max_out);
  }
}

// One 16-byte chunk per thread; a row of H halves is H/8 consecutive threads, so every lane is busy whatever H is.
// Bound: memory.  262 144 rows of 768 halves 125.0 us (6.44 TB/s), 2 308 rows 2.81 us; four rows to a wavefront, with 96 chunks for
// 64 lanes in two passes, took 145.4 and 3.13 us (width 512: 85.1 against 91.8, width 1024: 164.9 against 192.3 at 262 144 rows).
__global__ __launch_bounds__(256) void pack_kernel(const uint4_t* __restrict__ padded,
                                                   const int32_t* __restrict__ token_idx, size_t total, int chunks,
                                                   uint4_t* __restrict__ packed) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const size_t tok = i / chunks;
  const int c = (int)(i - tok * chunks);
  packed[i] = padded[(size_t)token_idx[tok] * chunks + c];
}

// A wavefront writes ROWS consecutive padded rows.  One wave-wide search finds where they start in the
// strictly increasing token_idx (three rounds of 64 probes for 2^18 tokens), the next ROWS entries say
// which of the rows are valid and which packed row each one is.
// Bound: latency up to some thousand rows, then memory.  Two rows a wavefront are the best or within 2 % of the best of 1, 2, 4, 8 from 32 to
// 65 536 rows of 512 to 2048 halves (175 x 2048: 3.36 us, 4.93 with eight; 4 096 x 768: 3.98, 4.72; 65 536 x 768: 24.5, 24.9);
// many narrow rows want eight, which share a search (65 536 x 64: 8.1 us, 11.6 with two; 8 192 x 64: the same).
template <int ROWS>
__global__ __launch_bounds__(256) void unpack_kernel(const uint4_t* __restrict__ packed,
                                                     const int32_t* __restrict__ token_idx, int T, int rows,
                                                     int chunks, uint4_t* __restrict__ padded) {
  const int lane = threadIdx.x & 63;
  const int r0 = ((int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * ROWS;
  if (r0 >= rows) return;
  const int lo = wave_lower_bound(token_idx, T, r0, lane);
  const int e = lane < ROWS && lo + lane < T ? token_idx[lo + lane] - r0 : ROWS;
  int src[ROWS];  // packed row of each padded row, -1: padding; wave-uniform
#pragma unroll
  for (int k = 0; k < ROWS; ++k) {
    const unsigned long long hit = __ballot(e == k);
    src[k] = hit ? lo + __ffsll((long long)hit) - 1 : -1;
  }
  const uint4_t zero = {0u, 0u, 0u, 0u};
  for (int c = lane; c < chunks; c += kWave) {
    uint4_t v[ROWS];
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
      v[k] = zero;
      if (src[k] >= 0) v[k] = packed[(size_t)src[k] * chunks + c];
    }
#pragma unroll
    for (int k = 0; k < ROWS; ++k)
      if (r0 + k < rows) padded[(size_t)(r0 + k) * chunks + c] = v[k];
  }
}

// Mask, without the per-sentence maximum.  Workgroup w owns entries [w, w+1) * kMaskChunk, four a thread, and counts the ones
// ahead of them itself: nothing is handed from one workgroup to the next.  The last one has read every entry and knows the total,
// but the host may refill the mask once it has that, so the total goes out with whichever workgroup has read its entries last:
// each adds one to a counter, the last chunk's also the total, and the one that completes the count reports and clears it.
// Bound: the last workgroup's read rate (2^20 entries, 4 MiB: 33 us more than the smallest call, 125 GB/s).  The one-workgroup kernel
// above reads as much, then packs bits and writes every position: 65 536 entries 16.4 us there, 5.5 us here; the whole call at
// 4 096 entries 14.6 / 12.7 us, at 65 536 18.9 / 16.1, at 2^20 213 / 46.  The counter is 0.6 to 0.9 us of that, so two to four
// chunks stay with the kernel above (8 192 entries 15.0 / 15.2, 12 288 15.4 / 15.7, 16 384 15.7 / 15.7, 32 768 16.5 / 16.2).
constexpr int kMaskChunk = 4 * kOffsetsThreads;
// 2^20 entries: one workgroup per compute unit, all resident at once.  The entries read grow with the square of the chunks (0.5 GB
// in all at 2^20, from the caches) and the packed counts have 24 bits; larger masks stay with the kernel above.
constexpr int kMaskChunksMax = 256, kMaskChunksFew = 4;
// Counters of calls under way, zero in between; bits 0 to 15 workgroups, 16 to 47 the total, 48 an invalid entry.  A call holds one
// from its launch until the total has arrived (a call beyond as many at a time takes the kernel above).
constexpr int kMaskCounters = 64;
__device__ unsigned long long mask_counters[kMaskCounters];

// ONE: a single chunk, whose workgroup has nobody to wait for.
template <bool ONE>
__global__ __launch_bounds__(kOffsetsThreads) void offsets_mask_chunks_kernel(const int32_t* __restrict__ mask, int n, int B,
                                                                             int S, int32_t* __restrict__ cu,
                                                                             int32_t* __restrict__ token_idx,
                                                                             int32_t* host_total, int counter) {
  typedef int int4_t __attribute__((ext_vector_type(4)));
  constexpr int kAhead = 16, kBadBit = 24;  // loads in flight; the counts stay below 2^24
  __shared__ int s_part[kOffsetsWaves], s_before[kOffsetsWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int chunk = blockIdx.x, flat = chunk * kMaskChunk + 4 * tid;
  const bool vec = (reinterpret_cast<uintptr_t>(mask) & 15u) == 0;
  int4_t own = {0, 0, 0, 0};
  if (vec && flat + 4 <= n) {
    own = *reinterpret_cast<const int4_t*>(mask + flat);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (flat + e < n) own[e] = mask[flat + e];
  }
  int before = 0, seen = 0;
  for (int c = 0; c < chunk; c += kAhead) {  // the chunks ahead are whole; past the last of them: clamped, not counted
    int4_t m[kAhead];
    if (vec) {
#pragma unroll
      for (int k = 0; k < kAhead; ++k)
        m[k] = *reinterpret_cast<const int4_t*>(mask + min(c + k, chunk - 1) * kMaskChunk + 4 * tid);
    } else {
#pragma unroll
      for (int k = 0; k < kAhead; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) m[k][e] = mask[min(c + k, chunk - 1) * kMaskChunk + 4 * tid + e];
    }
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      seen |= m[k][0] | m[k][1] | m[k][2] | m[k][3];
      if (c + k < chunk) before += (m[k][0] & 1) + (m[k][1] & 1) + (m[k][2] & 1) + (m[k][3] & 1);
    }
  }
  seen |= own[0] | own[1] | own[2] | own[3];  // not used earlier: its round trip is that of the loads above
  const int nib = (own[0] & 1) | (own[1] & 1) << 1 | (own[2] & 1) << 2 | (own[3] & 1) << 3, ones = __popc(nib);
  const int x = wave_inclusive_scan(ones), y = wave_inclusive_scan(before);
  const int bad_here = __any((seen & ~1) != 0) ? 1 << kBadBit : 0;
  if (lane == kWave - 1) {
    s_part[wave] = x;
    s_before[wave] = y + bad_here;
  }
  __syncthreads();
  // every row of 16 lanes scans the 16 wave sums
  int p = s_part[lane & 15], q = s_before[lane & 15];
  p += __builtin_amdgcn_update_dpp(0, p, 0x111, 0xf, 0xf, false);
  q += __builtin_amdgcn_update_dpp(0, q, 0x111, 0xf, 0xf, false);
  p += __builtin_amdgcn_update_dpp(0, p, 0x112, 0xf, 0xf, false);
  q += __builtin_amdgcn_update_dpp(0, q, 0x112, 0xf, 0xf, false);
  p += __builtin_amdgcn_update_dpp(0, p, 0x114, 0xf, 0xf, false);
  q += __builtin_amdgcn_update_dpp(0, q, 0x114, 0xf, 0xf, false);
  p += __builtin_amdgcn_update_dpp(0, p, 0x118, 0xf, 0xf, false);
  q += __builtin_amdgcn_update_dpp(0, q, 0x118, 0xf, 0xf, false);
  const int ahead = __builtin_amdgcn_readlane(q, 15), first = ahead & ((1 << kBadBit) - 1);
  const int total = first + __builtin_amdgcn_readlane(p, 15);
  const bool bad = ahead >> kBadBit;
  if (tid == 0 && chunk == (int)gridDim.x - 1) {
    cu[B] = bad ? -1 : total;
    if (ONE) publish_total(total, 0, bad, host_total, nullptr);
  }
  if (!ONE && tid == 0 && host_total) {  // behind the barrier: every wavefront has its entries in registers
    unsigned long long* const slot = mask_counters + counter;
    unsigned long long count = 1;
    if (chunk == (int)gridDim.x - 1) count += ((unsigned long long)total << 16) + ((unsigned long long)bad << 48);
    count += __hip_atomic_fetch_add(slot, count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((count & 0xffff) == gridDim.x) {
      __hip_atomic_store(slot, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // ahead of the report, which releases it
      publish_total((int)(count >> 16), 0, count >> 48 != 0, host_total, nullptr);
    }
  }
  int at = first + (wave ? __builtin_amdgcn_readlane(p, wave - 1) : 0) + x - ones;
  int b = flat / S, r = flat - b * S;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (r == 0 && flat + e < n) cu[b] = at;  // a sentence starts here
    if (nib >> e & 1) token_idx[at++] = flat + e;
    if (++r == S) {
      r = 0;
      ++b;
    }
  }
}

}  // namespace bt

using namespace bt;

// One of the counters of offsets_mask_chunks_kernel, held by one call; index -1: all are held, or none was asked for.
class MaskCounter {
 public:
  explicit MaskCounter(bool wanted) {
    uint64_t b = wanted ? held.load(std::memory_order_relaxed) : ~0ull;
    while (~b && index < 0) {
      const int i = __builtin_ctzll(~b);
      if (held.compare_exchange_weak(b, b | 1ull << i, std::memory_order_acquire)) index = i;
    }
  }
  ~MaskCounter() {
    if (index >= 0 && !lost) held.fetch_and(~(1ull << index), std::memory_order_release);
  }
  MaskCounter(const MaskCounter&) = delete;
  MaskCounter& operator=(const MaskCounter&) = delete;
  int index = -1;
  bool lost = false;  // the kernel may not have ended: never handed out again

 private:
  static std::atomic<uint64_t> held;
};
std::atomic<uint64_t> MaskCounter::held{0};
static_assert(kMaskCounters == 64, "a bit each");

// Shared body of bt_build_offsets / bt_build_offsets_stats.  h_out[0] receives the total; with `stats`
// h_out[1] receives the largest per-sentence count and d_cu_seqlens has B+2 entries (the last one is
// the device copy of that maximum).
// meanwhile(context) runs between the launch and the wait, if the host polls for the total: work for the device that does not need
// the total on the host.
bt_status bt::build_offsets(const int32_t* d_mask, const int32_t* d_lengths, int B, int S, int32_t* d_cu_seqlens,
                            int32_t* d_token_idx, int32_t* h_out, bool stats, bt_stream stream, void (*meanwhile)(void*),
                            void* context) {
  if ((d_mask == nullptr) == (d_lengths == nullptr)) return BT_ERR_INVALID_ARG;
  if (!d_cu_seqlens || !d_token_idx || !h_out || B < 0 || S < 1) return BT_ERR_INVALID_ARG;
  if (S > BT_MAX_SEQ || (int64_t)B * S >= (int64_t)INT32_MAX) return BT_ERR_UNSUPPORTED;
  hipStream_t st = static_cast<hipStream_t>(stream);
  // The call waits for a result on the host: it cannot be recorded into a HIP graph.
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cap) != hipSuccess) {
    (void)hipGetLastError();
    return BT_ERR_HIP;
  }
  if (cap != hipStreamCaptureStatusNone) return BT_ERR_UNSUPPORTED;
  // Fast path: h_out lies in pinned host memory that the device can write (hipHostMalloc).  The
  // kernel stores the total there the moment it is known and the host polls for it: no copy, no
  // stream synchronisation, and later launches on the stream are ordered after the kernel anyway.
  hipPointerAttribute_t attr;
  int32_t* h_dev = nullptr;
  if (hipPointerGetAttributes(&attr, h_out) == hipSuccess && attr.type == hipMemoryTypeHost && attr.devicePointer)
    h_dev = static_cast<int32_t*>(attr.devicePointer);
  else
    (void)hipGetLastError();  // ordinary host memory: not an error
  constexpr int32_t kPending = INT32_MIN;
  volatile int32_t* slot = h_out;
  if (h_dev) *slot = kPending;
  // B == 0 runs the same kernel: it writes cu[0] = 0 and a total of 0 (no memset, no special case)
  int32_t* const d_max = stats ? d_cu_seqlens + B + 1 : nullptr;
  const int n = B * S, chunks = (int)(((int64_t)n + kMaskChunk - 1) / kMaskChunk);
  const bool by_chunks = d_mask && !stats && n > 0 && (chunks == 1 || chunks > kMaskChunksFew) && chunks <= kMaskChunksMax;
  MaskCounter counter(by_chunks && chunks > 1 && h_dev);
  if (by_chunks && (chunks == 1 || !h_dev || counter.index >= 0)) {
    auto* const kernel = chunks == 1 ? offsets_mask_chunks_kernel<true> : offsets_mask_chunks_kernel<false>;
    kernel<<<chunks, kOffsetsThreads, 0, st>>>(d_mask, n, B, S, d_cu_seqlens, d_token_idx, h_dev, counter.index);
  } else if (d_mask) {
    offsets_mask_kernel<<<1, kOffsetsThreads, 0, st>>>(d_mask, B, S, d_cu_seqlens, d_token_idx, h_dev, d_max);
  } else {  // one wavefront per sentence, up to one workgroup per compute unit
    const int wgs = (B + kOffsetsWaves - 1) / kOffsetsWaves;
    offsets_lengths_kernel<<<wgs < 1 ? 1 : (wgs > 256 ? 256 : wgs), kOffsetsThreads, 0, st>>>(
        d_lengths, B, S, d_cu_seqlens, d_token_idx, h_dev, d_max);
  }
  if (hipGetLastError() != hipSuccess) return counter.lost = true, BT_ERR_HIP;
  // Not with ordinary host memory: the copy of the total would queue up behind that work, the host would wait for both and the
  // device be idle afterwards all the same (masked call of one layer, 9 894 tokens: 251.1 us so, 247.7 without).
  if (meanwhile && h_dev) meanwhile(context);
  int32_t res[2] = {kPending, 0};
  if (h_dev) {
    const auto t0 = std::chrono::steady_clock::now();
    for (long spin = 0; (res[0] = slot[0]) == kPending; ++spin) {
      if ((spin & 1023) == 1023 && std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(200)) break;
      __builtin_ia32_pause();
    }
    if (res[0] != kPending && stats) {
      __atomic_thread_fence(__ATOMIC_ACQUIRE);  // the maximum was stored before the total
      res[1] = slot[1];
    }
  }
  if (res[0] == kPending) {  // pageable h_out, or the store has not shown up: copy and synchronise
    if (hipMemcpyAsync(res, d_cu_seqlens + B, (stats ? 2 : 1) * sizeof(int32_t), hipMemcpyDeviceToHost, st) !=
        hipSuccess)
      return counter.lost = true, BT_ERR_HIP;
    if (hipStreamSynchronize(st) != hipSuccess) return counter.lost = true, BT_ERR_HIP;
  }
  h_out[0] = res[0] < 0 ? 0 : res[0];
  if (stats) h_out[1] = res[0] < 0 ? 0 : res[1];
  return res[0] < 0 ? BT_ERR_INVALID_ARG : BT_OK;
}

extern "C" bt_status bt_build_offsets(const int32_t* d_mask, const int32_t* d_lengths, int B, int S,
                                      int32_t* d_cu_seqlens, int32_t* d_token_idx, int32_t* h_total,
                                      bt_stream stream) {
  return build_offsets(d_mask, d_lengths, B, S, d_cu_seqlens, d_token_idx, h_total, false, stream, nullptr, nullptr);
}

extern "C" bt_status bt_build_offsets_stats(const int32_t* d_mask, const int32_t* d_lengths, int B, int S,
                                            int32_t* d_cu_seqlens, int32_t* d_token_idx, int32_t* h_total_max,
                                            bt_stream stream) {
  return build_offsets(d_mask, d_lengths, B, S, d_cu_seqlens, d_token_idx, h_total_max, true, stream, nullptr, nullptr);
}

extern "C" bt_status bt_pack(const bt_half* d_padded, const int32_t* d_token_idx, int T, int H,
                             bt_half* d_packed, bt_stream stream) {
  if (T < 0 || H < 8 || (H % 8) != 0) return BT_ERR_INVALID_ARG;
  if (T == 0) return BT_OK;
  if (!d_padded || !d_token_idx || !d_packed || !aligned16(d_padded) || !aligned16(d_packed))
    return BT_ERR_INVALID_ARG;
  const int chunks = H / 8;
  const size_t total = (size_t)T * chunks;
  const size_t blocks = (total + 255) / 256;
  if (blocks > 0x7fffffffull) return BT_ERR_UNSUPPORTED;
  pack_kernel<<<(unsigned)blocks, 256, 0, static_cast<hipStream_t>(stream)>>>(
      reinterpret_cast<const uint4_t*>(d_padded), d_token_idx, total, chunks, reinterpret_cast<uint4_t*>(d_packed));
  return launch_status();
}

extern "C" bt_status bt_unpack(const bt_half* d_packed, const int32_t* d_token_idx, int T, int B, int S, int H,
                               bt_half* d_padded, bt_stream stream) {
  if (T < 0 || B < 0 || S < 1 || H < 8 || (H % 8) != 0) return BT_ERR_INVALID_ARG;
  if ((int64_t)B * S >= (int64_t)INT32_MAX) return BT_ERR_UNSUPPORTED;
  if ((int64_t)T > (int64_t)B * S) return BT_ERR_INVALID_ARG;
  if (B == 0) return BT_OK;
  if (!d_padded || !aligned16(d_padded)) return BT_ERR_INVALID_ARG;
  if (T > 0 && (!d_packed || !d_token_idx || !aligned16(d_packed))) return BT_ERR_INVALID_ARG;
  const int rows = B * S;
  const uint4_t* const packed = reinterpret_cast<const uint4_t*>(d_packed);
  uint4_t* const padded = reinterpret_cast<uint4_t*>(d_padded);
  hipStream_t st = static_cast<hipStream_t>(stream);
  auto grid = [&](int per_wave) { return (unsigned)(((size_t)rows + 4 * per_wave - 1) / (4 * per_wave)); };
  if (H < 512 && rows > 8192) unpack_kernel<8><<<grid(8), 256, 0, st>>>(packed, d_token_idx, T, rows, H / 8, padded);
  else unpack_kernel<2><<<grid(2), 256, 0, st>>>(packed, d_token_idx, T, rows, H / 8, padded);
  return launch_status();
}
