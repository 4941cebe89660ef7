// Stable LSD radix sort for gfx950, and the status and fill kernels.
#include "bgs_internal.h"

namespace bgs {

namespace {

__device__ inline uint32_t lane_id() { return __lane_id(); }

__device__ inline uint32_t wave_incl_scan(uint32_t v) {
    const uint32_t lane = lane_id();
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        uint32_t t = __shfl_up(v, off, 64);
        if (lane >= (uint32_t)off) v += t;
    }
    return v;
}

// Exclusive scan over the 256 threads of a block; lds needs 4 words.
__device__ inline uint32_t block_excl_scan(uint32_t v, uint32_t* lds, uint32_t* total) {
    const uint32_t lane = lane_id(), wave = threadIdx.x >> 6;
    uint32_t inc = wave_incl_scan(v);
    if (lane == 63) lds[wave] = inc;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        uint32_t x = lds[w];
        if ((uint32_t)w < wave) off += x;
        tot += x;
    }
    __syncthreads();
    if (total) *total = tot;
    return off + inc - v;
}

}  // namespace

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

__global__ void k_status_reset(DevStatus* st, int full) {
    constexpr int kWords = (int)(sizeof(DevStatus) / 4);
    constexpr int kSticky = (int)(offsetof(DevStatus, sticky) / 4);
    __shared__ uint32_t keep;
    if (threadIdx.x == 0) keep = full ? 0u : (st->sticky | st->overflow);
    __syncthreads();
    uint32_t* w = reinterpret_cast<uint32_t*>(st);
    for (int i = threadIdx.x; i < kWords; i += blockDim.x) w[i] = i == kSticky ? keep : 0u;
}

hipError_t launch_status_reset(DevStatus* st, int full, hipStream_t s) {
    static_assert(sizeof(DevStatus) % 4 == 0, "status block is made of 32-bit words");
    hipLaunchKernelGGL(k_status_reset, dim3(1), dim3(128), 0, s, st, full);
    return hipGetLastError();
}

__global__ void k_fill_u32(uint32_t* dst, int64_t n, uint32_t value) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = value;
}

hipError_t launch_fill_u32(uint32_t* dst, int64_t n, uint32_t value, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>(ceil_div(n, 256), 2048);
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, s, dst, n, value);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Radix sort.  Stable LSD with digits of up to 8 bits (a 32-bit key takes four
// passes, a 13-bit one two of 7 and 6 bits).  The grid is fixed by the
// capacity (at most kRsGrid blocks; always kRsSmallGrid for small sorts,
// which use 1024-key sub-chunks instead of 6144); block b owns the contiguous
// chunk [b C, b C + C) of the n keys, C = n / grid rounded up to 256.
// A pass is three launches:
//   1. k_rs_hist: per-block digit counts (LDS atomics), stored
//      digit-major: counts[d * grid + b].
//   2. k_rs_scan: one block per digit scans its row over the blocks and
//      writes the digit total.
//   3. k_rs_scatter: every block scans the digit totals, then walks its chunk
//      in sub-chunks of 6144 keys: each wave ranks its 1536 keys in 24 steps
//      of 64 (1024-key sub-chunks, 4 steps, for small sorts) with match-any
//      ballots and a per-wave LDS count per digit, the sub-chunk is
//      reordered by digit in LDS, and each digit's run (24 keys on average
//      at 8 bits) is written out contiguously.  Large sorts rank digits of
//      at most 7 bits with per-thread counters instead (k_rs_scatter_cnt).
// Blocks never wait on each other.
// ---------------------------------------------------------------------------
namespace {

constexpr int kRsMaxBits = 8;
constexpr int kRsBins = 1 << kRsMaxBits;
constexpr int kRsGrid = 1024;
// Small sorts use half the grid: a 300k-key depth sort then gives each
// block about 600 keys, and its count table and per-digit scans shrink by
// half (61.8 against 69.2 us).
constexpr int kRsSmallGrid = 512;
// Keys per thread per sub-chunk: 24 (6144-key sub-chunks, long digit runs;
// a 6M-key tile sort then gives each block one sub-chunk, not a full and a
// partial one in turn) for large sorts; 4 (1024-key sub-chunks) for small
// ones, where a block holds only a few hundred keys and its latency is the
// sort's.
constexpr int kRsItemsBig = 24, kRsItemsSmall = 4;
__device__ inline uint64_t match_digit(uint32_t d, uint64_t valid, int bits) {
    uint64_t peers = valid;
#pragma unroll
    for (int b = 0; b < kRsMaxBits; ++b) {
        if (b < bits) {
            const uint64_t bal = __ballot((d >> b) & 1u);
            peers &= ((d >> b) & 1u) ? bal : ~bal;
        }
    }
    return peers;
}

// Block b's chunk: n / grid keys rounded up to a multiple of 256.
__device__ inline void chunk_of(uint32_t n, uint32_t grid, uint32_t b, uint32_t* lo, uint32_t* hi) {
    const uint32_t per = (uint32_t)(((uint64_t)n + grid - 1) / grid);
    const uint64_t c = ((uint64_t)per + 255u) & ~255ull;
    const uint64_t l = min<uint64_t>((uint64_t)b * c, n);
    *lo = (uint32_t)l;
    *hi = (uint32_t)min<uint64_t>(l + c, n);
}

template <int kRsItems>
__global__ __launch_bounds__(256) void k_rs_hist(const uint32_t* __restrict__ keys, uint32_t n, int shift, int bits,
                                                 uint32_t* __restrict__ counts) {
    constexpr int kRsSub = 256 * kRsItems;
    __shared__ uint32_t h[kRsBins];
    const uint32_t bins = 1u << bits, mask = bins - 1u;
    h[threadIdx.x] = 0;
    __syncthreads();
    uint32_t lo, hi;
    chunk_of(n, gridDim.x, blockIdx.x, &lo, &hi);
    for (uint64_t sub = lo; sub < hi; sub += kRsSub) {
        uint32_t k[kRsItems];
#pragma unroll
        for (int it = 0; it < kRsItems; ++it) {
            const uint64_t i = sub + it * 256 + threadIdx.x;
            k[it] = i < hi ? keys[i] : 0u;
        }
        // Counts only (no ranks): one LDS add per key; lanes of a wave on
        // one digit are serialised by the LDS, which costs less than
        // matching the digits with ballots.
#pragma unroll
        for (int it = 0; it < kRsItems; ++it) {
            if (sub + it * 256 + threadIdx.x < hi) atomicAdd(&h[(k[it] >> shift) & mask], 1u);
        }
    }
    __syncthreads();
    if (threadIdx.x < bins) counts[(uint64_t)threadIdx.x * gridDim.x + blockIdx.x] = h[threadIdx.x];
}

// One block per digit: exclusive scan of counts[d * grid .. + grid) in place;
// totals[d] = the row's sum.
__global__ __launch_bounds__(256) void k_rs_scan(uint32_t* __restrict__ counts, uint32_t grid,
                                                 uint32_t* __restrict__ totals) {
    __shared__ uint32_t lds[4];
    uint32_t* row = counts + (uint64_t)blockIdx.x * grid;
    const uint32_t per = (grid + 255) / 256, b0 = threadIdx.x * per;
    uint32_t v[kRsGrid / 256];
    uint32_t sum = 0;
#pragma unroll
    for (int j = 0; j < kRsGrid / 256; ++j) {
        v[j] = ((uint32_t)j < per && b0 + j < grid) ? row[b0 + j] : 0u;
        sum += v[j];
    }
    uint32_t tot;
    uint32_t run = block_excl_scan(sum, lds, &tot);
#pragma unroll
    for (int j = 0; j < kRsGrid / 256; ++j) {
        if ((uint32_t)j < per && b0 + j < grid) row[b0 + j] = run;
        run += v[j];
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = tot;
}

template <int kRsItems>
__global__ __launch_bounds__(256) void k_rs_scatter(const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin,
                                                    uint32_t* __restrict__ kout, uint32_t* __restrict__ vout,
                                                    uint32_t n, int shift, int bits,
                                                    const uint32_t* __restrict__ counts,
                                                    const uint32_t* __restrict__ totals) {
    constexpr int kRsSub = 256 * kRsItems;
    __shared__ uint32_t s_keys[kRsSub], s_vals[kRsSub];
    __shared__ uint32_t cnt0[4 * kRsBins], dstart[kRsBins], gbase[kRsBins], run[kRsBins], lds[4];
    const uint32_t G = gridDim.x;
    const auto cnt = [&](uint32_t w) { return cnt0 + w * kRsBins; };
    const uint32_t bins = 1u << bits, mask = bins - 1u;
    uint32_t lo, hi;
    chunk_of(n, G, blockIdx.x, &lo, &hi);
    if (lo >= hi) return;
    const uint32_t lane = lane_id(), wave = threadIdx.x >> 6;
    const uint64_t lt = (1ull << lane) - 1ull;
    const uint32_t dt = threadIdx.x;  // the digit this thread looks after
    {
        // run[d] = (keys of smaller digits) + (keys of digit d in earlier blocks).
        const uint32_t t = dt < bins ? totals[dt] : 0u;
        const uint32_t acc = block_excl_scan(t, lds, nullptr);
        if (dt < bins) run[dt] = acc + counts[(uint64_t)dt * G + blockIdx.x];
#pragma unroll
        for (int w = 0; w < 4; ++w) cnt(w)[dt] = 0;
    }
    __syncthreads();
    for (uint64_t sub = lo; sub < hi; sub += kRsSub) {
        uint32_t k[kRsItems], v[kRsItems], r[kRsItems];
#pragma unroll
        for (int it = 0; it < kRsItems; ++it) {
            const uint64_t i = sub + wave * (64 * kRsItems) + it * 64 + lane;
            const bool ok = i < hi;
            k[it] = ok ? kin[i] : 0u;
            v[it] = ok ? (vin ? vin[i] : (uint32_t)i) : 0u;
        }
#pragma unroll
        for (int it = 0; it < kRsItems; ++it) {
            const uint64_t i = sub + wave * (64 * kRsItems) + it * 64 + lane;
            const bool ok = i < hi;
            const uint32_t d = (k[it] >> shift) & mask;
            const uint64_t peers = match_digit(d, __ballot(ok), bits);
            const uint32_t c = ok ? cnt(wave)[d] : 0u;
            r[it] = ok ? c + (uint32_t)__popcll(peers & lt) : 0xFFFFFFFFu;
            __builtin_amdgcn_wave_barrier();
            if (ok && (peers & lt) == 0) cnt(wave)[d] = c + (uint32_t)__popcll(peers);
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        {
            const uint32_t c0 = cnt(0)[dt], c1 = cnt(1)[dt], c2 = cnt(2)[dt], c3 = cnt(3)[dt];
            const uint32_t tot = c0 + c1 + c2 + c3;
            const uint32_t st = block_excl_scan(tot, lds, nullptr);
            cnt(0)[dt] = st;
            cnt(1)[dt] = st + c0;
            cnt(2)[dt] = st + c0 + c1;
            cnt(3)[dt] = st + c0 + c1 + c2;
            dstart[dt] = st;
            if (dt < bins) {
                gbase[dt] = run[dt];
                run[dt] += tot;
            }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kRsItems; ++it) {
            if (r[it] != 0xFFFFFFFFu) {
                const uint32_t lp = cnt(wave)[(k[it] >> shift) & mask] + r[it];
                s_keys[lp] = k[it];
                s_vals[lp] = v[it];
            }
        }
        __syncthreads();
        const uint32_t m = (uint32_t)min<uint64_t>((uint64_t)kRsSub, hi - sub);
        for (uint32_t p = threadIdx.x; p < m; p += 256) {
            const uint32_t kk = s_keys[p];
            const uint32_t d = (kk >> shift) & mask;
            const uint32_t o = gbase[d] + (p - dstart[d]);
            if (o < n) {  // always true for consistent counts; keeps every write in bounds
                kout[o] = kk;
                vout[o] = s_vals[p];
            }
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < 4; ++w) cnt(w)[dt] = 0;
        __syncthreads();
    }
}

// k_rs_scatter for digits of at most 7 bits and 6144-key sub-chunks, with
// the ranks taken from per-thread digit counters instead of ballots: thread
// t holds the sub-chunk's keys [24 t, 24 t + 24) (blocked, so input order is
// (thread, item) order), counts its digits in a 16-bit LDS counter per
// (digit, thread), a raking scan of the counters in (digit, thread) order
// gives every (digit, thread) its first rank, and the thread's own count
// before each key adds the rest.  Stable, like the ballot ranking, at a
// fraction of its vector work.  The counter words are padded by one word in
// 32 so the raking threads hit distinct banks; the same LDS holds the
// reordered keys and values once the ranks are known.  (At 24 keys per
// thread a counter reaches 24 and a rank 6143: 16 bits hold both.)
// Digits of 7 bits need 64 KiB of counters, which gfx950's 160 KiB of LDS
// per workgroup holds for two workgroups per CU: a 13-bit tile id then
// takes two counter-ranked passes (7 + 6 bits) instead of a ballot-ranked
// 7-bit pass and a counter-ranked one.  Digits of at most 6 bits keep the
// 32 KiB form.
constexpr int kRsCntMaxBits = 7;
__host__ __device__ constexpr int rs_cnt_words(int bits) { return (1 << bits) * 256 / 2; }  // two 16-bit counters a word
__host__ __device__ constexpr int rs_cnt_lds(int bits) { return rs_cnt_words(bits) + rs_cnt_words(bits) / 32; }  // padded
static_assert(kRsItemsBig % 4 == 0, "a thread's keys are loaded as 16-byte vectors");

__device__ __forceinline__ uint32_t cnt_slot(uint32_t w) { return w + (w >> 5); }

// The counters, then the sub-chunk's keys and values.
template <int kBits>
__host__ __device__ constexpr int rs_cnt_buf() {
    return rs_cnt_lds(kBits) > 2 * 256 * kRsItemsBig ? rs_cnt_lds(kBits) : 2 * 256 * kRsItemsBig;
}

template <int kBits>
__global__ __launch_bounds__(256, 2) void k_rs_scatter_cnt(const uint32_t* __restrict__ kin,
                                                           const uint32_t* __restrict__ vin,
                                                           uint32_t* __restrict__ kout, uint32_t* __restrict__ vout,
                                                           uint32_t n, int shift, int bits,
                                                           const uint32_t* __restrict__ counts,
                                                           const uint32_t* __restrict__ totals) {
    constexpr int kItems = kRsItemsBig;
    constexpr int kSub = 256 * kItems;
    constexpr int kBins = 1 << kBits;
    __shared__ uint32_t s_buf[rs_cnt_buf<kBits>()];
    __shared__ uint32_t dstart[kBins + 1], gbase[kBins], run[kBins], lds[4];
    uint32_t* s_keys = s_buf;
    uint32_t* s_vals = s_buf + kSub;
    const uint32_t G = gridDim.x;
    const uint32_t bins = 1u << bits, mask = bins - 1u;
    uint32_t lo, hi;
    chunk_of(n, G, blockIdx.x, &lo, &hi);
    if (lo >= hi) return;
    const uint32_t t = threadIdx.x;
    {
        // run[d] = (keys of smaller digits) + (keys of digit d in earlier blocks).
        const uint32_t tv = t < bins ? totals[t] : 0u;
        const uint32_t acc = block_excl_scan(tv, lds, nullptr);
        if (t < bins) run[t] = acc + counts[(uint64_t)t * G + blockIdx.x];
    }
    const uint32_t rake = bins / 2;         // counter words per thread (bins * 256 / 2 words over 256 threads)
    const uint32_t nclear = cnt_slot(bins * 128u);
    for (uint64_t sub = lo; sub < hi; sub += kSub) {
        const uint32_t m = (uint32_t)min<uint64_t>((uint64_t)kSub, hi - sub);
        const uint32_t i0 = t * kItems;
        uint32_t k[kItems], v[kItems];
        if (i0 + kItems <= m) {
            const uint4* kp = reinterpret_cast<const uint4*>(kin + sub + i0);
#pragma unroll
            for (int q = 0; q < kItems / 4; ++q) {
                const uint4 x = kp[q];
                k[4 * q] = x.x; k[4 * q + 1] = x.y; k[4 * q + 2] = x.z; k[4 * q + 3] = x.w;
            }
            if (vin) {
                const uint4* vp = reinterpret_cast<const uint4*>(vin + sub + i0);
#pragma unroll
                for (int q = 0; q < kItems / 4; ++q) {
                    const uint4 x = vp[q];
                    v[4 * q] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
                }
            } else {
#pragma unroll
                for (int it = 0; it < kItems; ++it) v[it] = (uint32_t)(sub + i0 + it);
            }
        } else {
#pragma unroll
            for (int it = 0; it < kItems; ++it) {
                const bool ok = i0 + it < m;
                k[it] = ok ? kin[sub + i0 + it] : 0u;
                v[it] = ok ? (vin ? vin[sub + i0 + it] : (uint32_t)(sub + i0 + it)) : 0u;
            }
        }
        for (uint32_t w = t; w < nclear; w += 256) s_buf[w] = 0u;
        __syncthreads();
        // This thread's count of each digit before each of its keys.  Ranks
        // stay below 2^16 (a sub-chunk holds 6144 keys), so two share a
        // register: fewer live registers, more waves per SIMD.
        uint32_t r2[kItems / 2];
#pragma unroll
        for (int q = 0; q < kItems / 2; ++q) r2[q] = 0u;
#pragma unroll
        for (int it = 0; it < kItems; ++it) {
            if (i0 + it < m) {
                const uint32_t d = (k[it] >> shift) & mask;
                const uint32_t e = d * 256u + t;
                const uint32_t h = 16u * (e & 1u);
                const uint32_t old = atomicAdd(&s_buf[cnt_slot(e >> 1)], 1u << h);
                r2[it >> 1] |= ((old >> h) & 0xFFFFu) << (16 * (it & 1));
            }
        }
        __syncthreads();
        // Raking exclusive scan of the counters in (digit, thread) order; the
        // words are read again for the second sweep rather than held.
        uint32_t sum = 0;
#pragma unroll
        for (int j = 0; j < kBins / 2; ++j) {
            if ((uint32_t)j < rake) {
                const uint32_t w = s_buf[cnt_slot(t * rake + j)];
                sum += (w & 0xFFFFu) + (w >> 16);
            }
        }
        uint32_t acc = block_excl_scan(sum, lds, nullptr);
#pragma unroll
        for (int j = 0; j < kBins / 2; ++j) {
            if ((uint32_t)j < rake) {
                const uint32_t w = s_buf[cnt_slot(t * rake + j)];
                const uint32_t e0 = acc;
                acc += w & 0xFFFFu;
                s_buf[cnt_slot(t * rake + j)] = e0 | (acc << 16);
                acc += w >> 16;
            }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kItems; ++it) {
            if (i0 + it < m) {
                const uint32_t e = ((k[it] >> shift) & mask) * 256u + t;
                const uint32_t first = (s_buf[cnt_slot(e >> 1)] >> (16u * (e & 1u))) & 0xFFFFu;
                r2[it >> 1] += first << (16 * (it & 1));  // no carry: every rank is below 2^16
            }
        }
        if (t < bins) dstart[t] = s_buf[cnt_slot(t * 128u)] & 0xFFFFu;
        if (t == 0) dstart[bins] = m;
        __syncthreads();  // every counter read is done before the keys overwrite them
        if (t < bins) {
            gbase[t] = run[t];
            run[t] += dstart[t + 1] - dstart[t];
        }
#pragma unroll
        for (int it = 0; it < kItems; ++it) {
            if (i0 + it < m) {
                const uint32_t rk = (r2[it >> 1] >> (16 * (it & 1))) & 0xFFFFu;
                s_keys[rk] = k[it];
                s_vals[rk] = v[it];
            }
        }
        __syncthreads();
        for (uint32_t p = t; p < m; p += 256) {
            const uint32_t kk = s_keys[p];
            const uint32_t d = (kk >> shift) & mask;
            const uint32_t o = gbase[d] + (p - dstart[d]);
            if (o < n) {  // always true for consistent counts; keeps every write in bounds
                kout[o] = kk;
                vout[o] = s_vals[p];
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Sorts of up to kBlockSort keys: one workgroup of 1024 threads does every
// pass in LDS, so a small frame's depth sort is one launch instead of
// twelve (each of which costs its start-up, whatever it moves).  Thread t of
// wave w holds the keys at w * 64 * kItems + it * 64 + lane; a pass ranks
// them as k_rs_scatter does (match-any ballots, a count per wave and digit),
// exchanges them through LDS and reads them back in order.  A digit that is
// the same in every key is passed over: depths within a factor of four or
// so share their upper bits.
// ---------------------------------------------------------------------------
constexpr int kBlockThreads = 1024, kBlockWaves = kBlockThreads / 64;
constexpr int64_t kBlockSort = 16 * kBlockThreads;

template <int kItems>
__global__ __launch_bounds__(kBlockThreads) void k_rs_block(uint32_t* keys, const uint32_t* vin, uint32_t* vout,
                                                            uint32_t n, int key_bits) {
    constexpr int kSub = kBlockThreads * kItems;
    __shared__ uint32_t s_keys[kSub], s_vals[kSub];
    __shared__ uint16_t cnt[kBlockWaves][kRsBins];
    __shared__ uint32_t wsum[4], wvary[kBlockWaves];
    const uint32_t t = threadIdx.x, lane = lane_id(), wave = t >> 6;
    const uint64_t lt = (1ull << lane) - 1ull;
    const uint32_t first = wave * (64 * kItems) + lane;
    uint32_t k[kItems], v[kItems], r[kItems];
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        const uint32_t i = first + it * 64;
        k[it] = i < n ? keys[i] : 0u;
        v[it] = i < n ? (vin ? vin[i] : i) : 0u;
    }
    // The bits in which any key differs from the first.
    uint32_t vary = 0;
    const uint32_t k0 = keys[0];
#pragma unroll
    for (int it = 0; it < kItems; ++it) vary |= first + it * 64 < n ? k[it] ^ k0 : 0u;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) vary |= (uint32_t)__shfl_xor((int)vary, off, 64);
    if (lane == 0) wvary[wave] = vary;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kBlockWaves; ++w) vary |= wvary[w];
    for (int shift = 0; shift < key_bits; shift += kRsMaxBits) {
        const int bits = min(kRsMaxBits, key_bits - shift);
        const uint32_t mask = (1u << bits) - 1u;
        if (((vary >> shift) & mask) == 0) continue;  // uniform over the block
        for (uint32_t i = t; i < kBlockWaves * kRsBins / 2; i += kBlockThreads) reinterpret_cast<uint32_t*>(cnt)[i] = 0u;
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kItems; ++it) {
            const bool ok = first + it * 64 < n;
            const uint32_t d = (k[it] >> shift) & mask;
            const uint64_t peers = match_digit(d, __ballot(ok), bits);
            const uint32_t c = ok ? cnt[wave][d] : 0u;
            r[it] = c + (uint32_t)__popcll(peers & lt);
            __builtin_amdgcn_wave_barrier();
            if (ok && (peers & lt) == 0) cnt[wave][d] = (uint16_t)(c + (uint32_t)__popcll(peers));
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        // First place of every (digit, wave): thread d < 256 for digit d.
        uint32_t c[kBlockWaves], tot = 0, inc = 0;
        if (t < kRsBins) {
#pragma unroll
            for (int w = 0; w < kBlockWaves; ++w) {
                c[w] = cnt[w][t];
                tot += c[w];
            }
            inc = wave_incl_scan(tot);
            if (lane == 63) wsum[wave] = inc;
        }
        __syncthreads();
        if (t < kRsBins) {
            uint32_t run = inc - tot;
            for (uint32_t w = 0; w < wave; ++w) run += wsum[w];
#pragma unroll
            for (int w = 0; w < kBlockWaves; ++w) {
                cnt[w][t] = (uint16_t)run;  // below n <= 16384
                run += c[w];
            }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kItems; ++it) {
            if (first + it * 64 < n) {
                const uint32_t p = cnt[wave][(k[it] >> shift) & mask] + r[it];
                s_keys[p] = k[it];
                s_vals[p] = v[it];
            }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kItems; ++it) {
            const uint32_t i = first + it * 64;
            if (i < n) {
                k[it] = s_keys[i];
                v[it] = s_vals[i];
            }
        }
    }
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        const uint32_t i = first + it * 64;
        if (i < n) {
            keys[i] = k[it];
            vout[i] = v[it];
        }
    }
}

uint32_t rs_grid(int64_t n_cap, int items) {
    const int64_t g = ceil_div(n_cap > 0 ? n_cap : 1, 256 * items);
    return (uint32_t)(g < kRsGrid ? g : kRsGrid);
}

}  // namespace

size_t radix_tmp_bytes(int64_t n_cap) {
    (void)n_cap;  // the grid, and so the count table, is at most kRsGrid blocks for any size
    return ((size_t)kRsBins * kRsGrid + kRsBins + 64) * sizeof(uint32_t) + 256;
}

hipError_t radix_sort(uint32_t* ka, uint32_t* va, uint32_t* kb, uint32_t* vb, int64_t n, int key_bits, bool iota,
                      void* tmp, hipStream_t s, bool* in_b) {
    *in_b = false;
    if (n <= 0 || key_bits <= 0) return hipSuccess;
    if (n > 0xFFFFFFFFll || key_bits > 32) return hipErrorInvalidValue;
    if (n <= kBlockSort) {  // one launch, in place
        const uint32_t* vin = iota ? nullptr : va;
        const dim3 one(1), wg(kBlockThreads);
        if (n <= 2 * kBlockThreads)
            hipLaunchKernelGGL(k_rs_block<2>, one, wg, 0, s, ka, vin, va, (uint32_t)n, key_bits);
        else if (n <= 6 * kBlockThreads)
            hipLaunchKernelGGL(k_rs_block<6>, one, wg, 0, s, ka, vin, va, (uint32_t)n, key_bits);
        else if (n <= 10 * kBlockThreads)
            hipLaunchKernelGGL(k_rs_block<10>, one, wg, 0, s, ka, vin, va, (uint32_t)n, key_bits);
        else
            hipLaunchKernelGGL(k_rs_block<16>, one, wg, 0, s, ka, vin, va, (uint32_t)n, key_bits);
        return hipGetLastError();
    }
    // Small sorts (keys per block of the full grid below 1024): 1024-key
    // sub-chunks.
    const bool small = n <= (int64_t)kRsGrid * 256 * kRsItemsSmall;
    const uint32_t grid = small ? kRsSmallGrid : rs_grid(n, kRsItemsBig);
    uint32_t* counts = (uint32_t*)tmp;
    uint32_t* totals = counts + (size_t)kRsBins * kRsGrid;  // past the largest count table
    const int passes = (key_bits + kRsMaxBits - 1) / kRsMaxBits;
    const int per = (key_bits + passes - 1) / passes;
    // The counter-ranked scatter loads 16-byte vectors.
    const auto a16 = [](const void* p) { return ((uintptr_t)p & 15u) == 0; };
    const bool aligned = a16(ka) && a16(kb) && a16(va) && a16(vb);
    uint32_t *ki = ka, *ko = kb, *vo = vb;
    const uint32_t* vi = iota ? nullptr : va;
    bool cur_b = false;
    for (int shift = 0; shift < key_bits; shift += per) {
        const int bits = key_bits - shift < per ? key_bits - shift : per;
        if (small)
            hipLaunchKernelGGL(k_rs_hist<kRsItemsSmall>, dim3(grid), dim3(256), 0, s, ki, (uint32_t)n, shift, bits, counts);
        else
            hipLaunchKernelGGL(k_rs_hist<kRsItemsBig>, dim3(grid), dim3(256), 0, s, ki, (uint32_t)n, shift, bits, counts);
        hipLaunchKernelGGL(k_rs_scan, dim3(1u << bits), dim3(256), 0, s, counts, grid, totals);
        if (small)
            hipLaunchKernelGGL(k_rs_scatter<kRsItemsSmall>, dim3(grid), dim3(256), 0, s, ki, vi, ko, vo, (uint32_t)n,
                               shift, bits, counts, totals);
        else if (bits <= 6 && aligned)
            hipLaunchKernelGGL(k_rs_scatter_cnt<6>, dim3(grid), dim3(256), 0, s, ki, vi, ko, vo, (uint32_t)n, shift,
                               bits, counts, totals);
        else if (bits <= kRsCntMaxBits && aligned)
            hipLaunchKernelGGL(k_rs_scatter_cnt<kRsCntMaxBits>, dim3(grid), dim3(256), 0, s, ki, vi, ko, vo,
                               (uint32_t)n, shift, bits, counts, totals);
        else
            hipLaunchKernelGGL(k_rs_scatter<kRsItemsBig>, dim3(grid), dim3(256), 0, s, ki, vi, ko, vo, (uint32_t)n,
                               shift, bits, counts, totals);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        cur_b = !cur_b;
        if (cur_b) {
            ki = kb; vi = vb; ko = ka; vo = va;
        } else {
            ki = ka; vi = va; ko = kb; vo = vb;
        }
    }
    *in_b = cur_b;
    return hipSuccess;
}

}  // namespace bgs
