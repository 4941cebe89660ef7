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
// passes, a 13-bit one two of 7 and 6 bits).  The grid is kRsGrid blocks;
// block b owns the contiguous chunk [b C, b C + C) of the n keys, C = n /
// kRsGrid rounded up to 256.  A pass is three launches:
//   1. k_rs_hist: per-block digit counts (LDS atomics), stored
//      digit-major: counts[d * grid + b].
//   2. k_rs_scan: one block per digit scans its row over the blocks and
//      writes the digit total.
//   3. k_rs_scatter: every block scans the digit totals, then walks its chunk
//      in sub-chunks of kThreads * kItems keys: each wave ranks its keys in
//      kItems steps of 64 with match-any ballots and a per-wave LDS count per
//      digit, the sub-chunk is reordered by digit in LDS, and each digit's
//      run is written out contiguously while the next sub-chunk's keys are
//      on their way.
// Blocks never wait on each other.
//
// Bound by memory on large sorts, by the latency of the launches and of a
// block's steps on small ones.  Two blocks a CU, all resident: every digit of
// every block has a line of keys and one of values open in its XCD's L2 (4
// MiB at 8 bits and 512 blocks), and more blocks only add to these.  What
// hides the steps' latency is waves: 512 threads with 8 keys each (16 waves
// a CU) took 19.6M 13-bit pairs from 288 to 214 us and 4M 32-bit pairs from
// 267 to 150, against 256 threads with 24 keys (8 waves); 12 or 16 keys a
// thread, whose registers halve the waves, took 305 and 281, and 768 or 1024
// blocks 255 and 223.
// ---------------------------------------------------------------------------
namespace {

constexpr int kRsMaxBits = 8;
constexpr int kRsBins = 1 << kRsMaxBits;
constexpr int kRsGrid = 512;
// Threads and keys per thread of a block, by the keys of its chunk: one
// sub-chunk where it can be, as small as it can be.  (300k pairs of 32 bits:
// 74 us with 256 threads of 4, 80 of 8, 85 with 512 of 8; 1M: 98, 92, 95;
// 1.2M: 110, 110, 99; it was 123.)
constexpr int64_t kRsSmall = kRsGrid * 256 * 4, kRsMedium = kRsGrid * 256 * 8;
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

template <int kThreads, int kItems>
__global__ __launch_bounds__(kThreads) void k_rs_hist(const uint32_t* __restrict__ keys, uint32_t n, int shift, int bits,
                                                      uint32_t* __restrict__ counts) {
    __shared__ uint32_t h[kRsBins];
    const uint32_t bins = 1u << bits, mask = bins - 1u;
    if (threadIdx.x < kRsBins) h[threadIdx.x] = 0u;
    __syncthreads();
    uint32_t lo, hi;
    chunk_of(n, gridDim.x, blockIdx.x, &lo, &hi);
    for (uint64_t sub = lo; sub < hi; sub += kThreads * kItems) {
        uint32_t k[kItems];
#pragma unroll
        for (int it = 0; it < kItems; ++it) {
            const uint64_t i = sub + it * kThreads + threadIdx.x;
            k[it] = i < hi ? keys[i] : 0u;
        }
        // Counts only (no ranks): one LDS add per key; lanes of a wave on
        // one digit are serialised by the LDS, which costs less than
        // matching the digits with ballots.
#pragma unroll
        for (int it = 0; it < kItems; ++it) {
            if (sub + it * kThreads + threadIdx.x < hi) atomicAdd(&h[(k[it] >> shift) & mask], 1u);
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

template <int kThreads, int kItems>
__global__ __launch_bounds__(kThreads) void k_rs_scatter(const uint32_t* __restrict__ kin,
                                                         const uint32_t* __restrict__ vin, uint32_t* __restrict__ kout,
                                                         uint32_t* __restrict__ vout, uint32_t n, int shift, int bits,
                                                         const uint32_t* __restrict__ counts,
                                                         const uint32_t* __restrict__ totals) {
    constexpr int kWaves = kThreads / 64;
    constexpr uint32_t kSub = kThreads * kItems;
    __shared__ uint32_t s_keys[kSub], s_vals[kSub];
    __shared__ uint32_t cnt[kWaves][kRsBins], to[kRsBins], lds[4];
    const uint32_t G = gridDim.x, bins = 1u << bits, mask = bins - 1u;
    uint32_t lo, hi;
    chunk_of(n, G, blockIdx.x, &lo, &hi);
    if (lo >= hi) return;
    const uint32_t t = threadIdx.x, lane = lane_id(), wave = t >> 6;
    const uint64_t lt = (1ull << lane) - 1ull;
    const uint32_t first = wave * (64 * kItems) + lane;  // the thread's first key of a sub-chunk
    uint32_t k[kItems], v[kItems];
    const auto load = [&](uint64_t sub) {
#pragma unroll
        for (int it = 0; it < kItems; ++it) {
            const uint64_t i = sub + first + it * 64;
            const bool ok = i < hi;
            k[it] = ok ? kin[i] : 0u;
            v[it] = ok ? (vin ? vin[i] : (uint32_t)i) : 0u;
        }
    };
    load(lo);
    // Of the digit that this thread looks after: where its next key goes,
    // i.e. (keys of smaller digits) + (keys of the digit in earlier blocks).
    uint32_t run = 0;
    const bool mine = t < bins;
    if (mine) run = counts[(uint64_t)t * G + blockIdx.x];
    {
        uint32_t x = 0;
        if (t < kRsBins) {
            x = wave_incl_scan(mine ? totals[t] : 0u);
            if (lane == 63) lds[wave] = x;
        }
        __syncthreads();
        if (mine) {
            run += x - totals[t];
            for (uint32_t w = 0; w < wave; ++w) run += lds[w];
        }
    }
    for (uint64_t sub = lo; sub < hi; sub += kSub) {
        const uint32_t m = (uint32_t)min<uint64_t>((uint64_t)kSub, hi - sub);
        for (uint32_t i = t; i < kWaves * kRsBins; i += kThreads) (&cnt[0][0])[i] = 0u;
        __syncthreads();
        uint32_t r[kItems];
#pragma unroll
        for (int it = 0; it < kItems; ++it) {
            const bool ok = first + it * 64 < m;
            const uint32_t d = (k[it] >> shift) & mask;
            const uint64_t peers = match_digit(d, __ballot(ok), bits);
            const uint32_t c = ok ? cnt[wave][d] : 0u;
            r[it] = c + (uint32_t)__popcll(peers & lt);
            __builtin_amdgcn_wave_barrier();
            if (ok && (peers & lt) == 0) cnt[wave][d] = c + (uint32_t)__popcll(peers);
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        // First place of every (digit, wave) in the sub-chunk.
        uint32_t tot = 0, x = 0;
        if (mine) {
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const uint32_t c = cnt[w][t];
                cnt[w][t] = tot;
                tot += c;
            }
        }
        if (t < kRsBins) {
            x = wave_incl_scan(tot);
            if (lane == 63) lds[wave] = x;
        }
        __syncthreads();
        if (mine) {
            uint32_t at = x - tot;
            for (uint32_t w = 0; w < wave; ++w) at += lds[w];
#pragma unroll
            for (int w = 0; w < kWaves; ++w) cnt[w][t] += at;
            to[t] = run - at;  // where the sub-chunk's places of this digit go
            run += tot;
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kItems; ++it) {
            if (first + it * 64 < m) {
                const uint32_t p = cnt[wave][(k[it] >> shift) & mask] + r[it];
                s_keys[p] = k[it];
                s_vals[p] = v[it];
            }
        }
        __syncthreads();
        if (sub + kSub < hi) load(sub + kSub);  // in flight while this one is written
#pragma unroll
        for (int it = 0; it < kItems; ++it) {
            const uint32_t p = t + it * kThreads;
            if (p < m) {
                const uint32_t kk = s_keys[p];
                const uint32_t o = to[(kk >> shift) & mask] + p;
                if (o < n) {  // always true for consistent counts; keeps every write in bounds
                    kout[o] = kk;
                    vout[o] = s_vals[p];
                }
            }
        }
        // The next sub-chunk's first barrier comes before any write to the
        // LDS that is read here.
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

template <int kThreads, int kItems>
void launch_rs_pass(const uint32_t* ki, const uint32_t* vi, uint32_t* ko, uint32_t* vo, uint32_t n, int shift, int bits,
                    uint32_t* counts, uint32_t* totals, hipStream_t s) {
    const dim3 grid(kRsGrid), wg(kThreads);
    hipLaunchKernelGGL((k_rs_hist<kThreads, kItems>), grid, wg, 0, s, ki, n, shift, bits, counts);
    hipLaunchKernelGGL(k_rs_scan, dim3(1u << bits), dim3(256), 0, s, counts, (uint32_t)kRsGrid, totals);
    hipLaunchKernelGGL((k_rs_scatter<kThreads, kItems>), grid, wg, 0, s, ki, vi, ko, vo, n, shift, bits, counts,
                       totals);
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
    // One launch, in place.  Pairs whose four digits all vary leave it at 10
    // keys a thread (16384 of them: 59 us here, 56 in twelve launches; with 22
    // bits, three digits, 45 here and 53); depth keys seldom do.
    if (n <= 10 * kBlockThreads || (n <= kBlockSort && (iota || key_bits <= 24))) {
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
    uint32_t* counts = (uint32_t*)tmp;
    uint32_t* totals = counts + (size_t)kRsBins * kRsGrid;
    const int passes = (key_bits + kRsMaxBits - 1) / kRsMaxBits;
    const int per = (key_bits + passes - 1) / passes;
    uint32_t *ki = ka, *ko = kb, *vo = vb;
    const uint32_t* vi = iota ? nullptr : va;
    bool cur_b = false;
    for (int shift = 0; shift < key_bits; shift += per) {
        const int bits = key_bits - shift < per ? key_bits - shift : per;
        const auto pass = n <= kRsSmall    ? launch_rs_pass<256, 4>
                          : n <= kRsMedium ? launch_rs_pass<256, 8>
                                           : launch_rs_pass<512, 8>;
        pass(ki, vi, ko, vo, (uint32_t)n, shift, bits, counts, totals, s);
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
