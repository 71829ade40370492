// Condensed query layout (Sec. 4.2, Sec. 5.1): after the build, the bucket
// table (one 8-byte slot per (feature, location) pair) is converted into a
// feature index (one 16-byte entry per feature) plus a value array holding,
// per feature with more than two locations, its locations in ascending order.
// A lookup then reads one index line and, for such features, one contiguous
// run, instead of every bucket line of the feature's chain.
//
// The conversion works on slices of 2^kCondSliceShift bucket-table buckets:
// all entries homed in a slice lie in its buckets or in the few buckets its
// chains run on into. The index has a whole number of buckets per slice
// (per_slice), and both home buckets are the high part of h2(feature) times
// the number of buckets, so the features homed in slice z of the table are
// those homed in index buckets [z, z + 1) * per_slice, and no other workgroup
// writes them. A workgroup gathers a slice's entries into LDS grouped by home
// bucket (a counting sort: about six entries a bucket), and every entry finds
// its feature's count and its own rank by comparing itself with the entries of
// its bucket. A count pass sizes the index and the value array; the write pass
// places the slice's features by a max-plus scan over its index buckets (as the
// slice insert of the build does) and writes every index line once.
//
// The write pass is bound by vector issue (72% of its peak) and the barriers
// between its phases; it moves 5.7 GB at 3.1 TB/s, two thirds of what a large
// copy reaches. The form this replaces sorted each slice's
// 64-bit entries in LDS twice, claimed every index entry with a global atomic
// and cleared the index first: a 1 Gbp table (2.3 GB, 141.6M pairs) took 9.8 ms
// to count, 11.3 to write and 1.7 for the clearing, the scan and the pair count;
// now 0.71 + 1.82 + 0.09 ms.
#include "mc_device.hpp"
#include "mc_internal.hpp"
#include "mc_slices.hpp"

namespace mc {

namespace {

constexpr int kCondThreads = kSliceThreads;
constexpr uint32_t kCondBuckets = kSliceBuckets;
constexpr uint32_t kCondMaxPer = kSliceSlots / 4;      // index buckets a slice at most
// Bins of a slice: an entry is compared with the others of its bin, and a wave
// takes as long as its largest bin, so buckets are split into finer bins by the
// next bits of the home bucket's product (four a table bucket in the count
// pass, up to four an index bucket in the write pass: conversion of a 1 Gbp
// table 3.1 -> 2.5 ms).
constexpr uint32_t kCondBinSplit = 2;                  // log2, most
constexpr uint32_t kCondCountBins = kCondBuckets << kCondBinSplit;
constexpr uint32_t kCondWriteBins = 2048;
// Entries of one slice in the write pass's usual form: a table at the default
// load holds about 2,048 (at most 4,096 slots); slices beyond it take the
// kCondCap form. 52,088 bytes of LDS against 115,064: three workgroups a CU, not
// one.
constexpr uint32_t kCondMid = 2944;
// A bin with more entries is sorted by the workgroup: the comparisons of every
// entry with all others of its bin grow with the square.
constexpr uint32_t kCondLong = 64;
constexpr uint32_t kCondMaxLong = kCondCap / (kCondLong + 1) + 1;

struct LongBins {
    uint32_t n;
    uint16_t bin[kCondMaxLong];
};

// Sort the bins of more than kCondLong keys: a bitonic network with every
// comparison ascending (keys past the end count as largest and never move).
// Called by the whole workgroup after a barrier; ends with one.
template <typename Lds>
__device__ __forceinline__ void sort_long_bins(Lds& L, LongBins& B, uint32_t nbins) {
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    if (tid == 0) B.n = 0u;
    __syncthreads();
    for (uint32_t r = tid; r < nbins; r += kCondThreads)
        if ((uint32_t)L.start[r + 1] - L.start[r] > kCondLong)
            B.bin[atomicAdd(&B.n, 1u)] = (uint16_t)r;
    __syncthreads();
    for (uint32_t x = 0; x < B.n; ++x) {
        const uint32_t r = B.bin[x];
        auto* const k = L.key + L.start[r];
        const uint32_t m = (uint32_t)L.start[r + 1] - L.start[r];
        uint32_t P = 1;
        while (P < m) P <<= 1;
        for (uint32_t size = 2; size <= P; size <<= 1) {
            for (uint32_t st = size >> 1; st > 0; st >>= 1) {
                for (uint32_t y = tid; y < P / 2; y += kCondThreads) {
                    const uint32_t o = y & (st - 1u), i = 2u * (y - o) + o;
                    // the first step of a size pairs mirrored places of a block
                    const uint32_t j = st == size >> 1 ? 2u * (y - o) + size - 1u - o : i + st;
                    if (j < m && k[j] < k[i]) {
                        const auto v = k[i];
                        k[i] = k[j];
                        k[j] = v;
                    }
                }
                __syncthreads();
            }
        }
    }
}

// First position in the sorted keys [lo, hi) whose feature is at least f (over:
// above f).
template <typename T>
__device__ __forceinline__ uint32_t feature_bound(const T* key, uint32_t lo, uint32_t hi,
                                                  uint32_t f, bool over) {
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        const uint32_t g = (uint32_t)(key[mid] >> (8 * sizeof(T) - 32));
        if (g < f || (over && g == f)) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Count pass: entries, distinct features and run values of every slice.
__global__ __launch_bounds__(kCondThreads) __attribute__((amdgpu_waves_per_eu(8))) void k_condense_count(CondArgs c) {
    __shared__ SliceLds<uint32_t, kCondCap, kCondCountBins, false> L;
    __shared__ LongBins B;
    __shared__ uint32_t sum[2];
    const uint32_t tid = threadIdx.x, nbins = kCondBuckets << c.split_t;
    const uint32_t nbs = (uint32_t)c.nb << c.split_t;
    for (uint32_t z = blockIdx.x; z < c.n_slices; z += gridDim.x) {
        __syncthreads();
        const uint32_t r0 = z * nbins;
        const uint32_t n = group_slice(c.table, (uint32_t)c.nb, z << kCondSliceShift, kCondBuckets,
                                       L, nbins, [=](uint32_t h) { return __umulhi(h, nbs) - r0; });
        if (tid < 2) sum[tid] = 0u;
        if (n <= kCondCap) sort_long_bins(L, B, nbins);
        __syncthreads();
        uint32_t feats = 0, vals = 0;
        for (uint32_t p = tid; p < (n <= kCondCap ? n : 0u); p += kCondThreads) {
            const uint32_t f = L.key[p];
            const uint32_t r = __umulhi(h2(f), nbs) - r0;
            const uint32_t s0 = L.start[r], s1 = L.start[r + 1];
            uint32_t same = 0, first = p;
            if (s1 - s0 <= kCondLong) {
                for (uint32_t q = s1; q-- > s0;)
                    if (L.key[q] == f) {
                        same += 1u;
                        first = q;
                    }
            } else {
                first = feature_bound(L.key, s0, s1, f, false);
                same = feature_bound(L.key, s0, s1, f, true) - first;
            }
            feats += first == p ? 1u : 0u;
            vals += same > kCondInline ? 1u : 0u;
        }
#pragma unroll
        for (int m = 1; m < kWave; m <<= 1) {
            feats += shfl_xor(feats, m);
            vals += shfl_xor(vals, m);
        }
        if (lane_id() == 0) {
            atomicAdd(&sum[0], feats);
            atomicAdd(&sum[1], vals);
        }
        __syncthreads();
        if (tid == 0) {
            c.slice_cnt[z] = ((unsigned long long)n << 32) | sum[0];
            c.slice_vals[z] = sum[1];
        }
    }
}

// Exclusive prefix of slice_vals in place (slice_vals[n_slices] = total) and
// the totals (CondResult), by one workgroup in tiles of four slices a thread.
constexpr int kCondScanThreads = 1024;
__global__ __launch_bounds__(kCondScanThreads) void k_condense_scan(CondArgs c) {
    constexpr uint32_t W = kCondScanThreads / kWave, U = 4;
    __shared__ unsigned long long ws[W], wf[W], wn[W];
    __shared__ uint32_t wm[W];
    const uint32_t t = threadIdx.x, lane = t & 63, w = t >> 6, n = c.n_slices;
    unsigned long long base = 0, feats = 0, pairs = 0;
    uint32_t most = 0;
    for (uint32_t i0 = 0; i0 < n; i0 += kCondScanThreads * U) {
        unsigned long long v[U], sum = 0;
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t i = i0 + t * U + u;
            v[u] = i < n ? c.slice_vals[i] : 0ull;
            const unsigned long long x = i < n ? c.slice_cnt[i] : 0ull;
            sum += v[u];
            feats += (uint32_t)x;
            pairs += x >> 32;
            most = max(most, (uint32_t)(x >> 32));
        }
        unsigned long long x = sum;   // inclusive wave scan
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int src = lane >= (uint32_t)d ? (int)lane - d : (int)lane;
            const uint32_t lo = shfl_idx((uint32_t)x, src), hi = shfl_idx((uint32_t)(x >> 32), src);
            if (lane >= (uint32_t)d) x += ((unsigned long long)hi << 32) | lo;
        }
        __syncthreads();
        if (lane == kWave - 1) ws[w] = x;
        __syncthreads();
        unsigned long long run = base + x - sum;
        for (uint32_t k = 0; k < W; ++k) {
            if (k < w) run += ws[k];
            base += ws[k];
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t i = i0 + t * U + u;
            if (i < n) c.slice_vals[i] = run;
            run += v[u];
        }
    }
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
        feats += ((unsigned long long)shfl_xor((uint32_t)(feats >> 32), m) << 32) +
                 shfl_xor((uint32_t)feats, m);
        pairs += ((unsigned long long)shfl_xor((uint32_t)(pairs >> 32), m) << 32) +
                 shfl_xor((uint32_t)pairs, m);
        most = max(most, shfl_xor(most, m));
    }
    if (lane == 0) {
        wf[w] = feats;
        wn[w] = pairs;
        wm[w] = most;
    }
    __syncthreads();
    if (t == 0) {
        CondResult r{};
        for (uint32_t k = 0; k < W; ++k) {
            r.feats += wf[k];
            r.pairs += wn[k];
            r.most = max(r.most, wm[k]);
        }
        r.vals = base;
        c.slice_vals[n] = base;
        *c.res = r;
    }
}

// Write pass: the slice's runs at its value prefix, its index lines whole.
// Slices of more than CAP entries, and in the kCondCap form those of at most
// kCondMid, are left to the other form.
template <uint32_t CAP>
__global__ __launch_bounds__(kCondThreads) __attribute__((amdgpu_waves_per_eu(CAP <= kCondMid ? 6 : 2))) void k_condense_write(CondArgs c) {
    constexpr uint32_t PER = (CAP + kCondThreads - 1) / kCondThreads;
    constexpr uint32_t BPER = kCondMaxPer / kCondThreads;
    __shared__ SliceLds<unsigned long long, CAP, kCondWriteBins, true> L;
    __shared__ LongBins B;
    __shared__ uint16_t voff[CAP];           // of a feature's first entry: offset of its run
    __shared__ uint16_t Te[kCondMaxPer];     // features homed below index bucket r
    __shared__ uint16_t Tp[kCondMaxPer];     // features placed in index buckets <= r
    __shared__ uint32_t vcur;
    const uint32_t R = c.per_slice;
    uint4* const idx = reinterpret_cast<uint4*>(c.idx);
    for (uint32_t z = blockIdx.x; z < c.n_slices; z += gridDim.x) {
        const uint32_t cnt = (uint32_t)(c.slice_cnt[z] >> 32);
        if (CAP == kCondMid ? cnt > kCondMid : cnt <= kCondMid) continue;
        __syncthreads();
        uint32_t tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const uint32_t sh = c.split_c, nbins = R << sh;
        const uint32_t nbs = (uint32_t)c.nbc << sh, r0 = z * nbins;
        const uint32_t n = group_slice(c.table, (uint32_t)c.nb, z << kCondSliceShift, kCondBuckets,
                                       L, nbins, [=](uint32_t h) { return __umulhi(h, nbs) - r0; });
        sort_long_bins(L, B, nbins);
        for (uint32_t r = tid; r < R; r += kCondThreads) L.cnt[r] = 0u;   // features per bucket
        if (tid == 0) vcur = 0u;
        __syncthreads();
        // each entry: its rank among its feature's locations, the feature's
        // first entry, the number of its locations, and for the first entry the
        // feature's number in its bucket and its second location
        uint32_t rank_first[PER], num_same[PER], second[PER];
#pragma unroll
        for (uint32_t k = 0; k < PER; ++k) {
            const uint32_t p = k * kCondThreads + tid;
            rank_first[k] = num_same[k] = second[k] = 0u;
            if (p >= n) continue;
            const unsigned long long e = L.key[p];
            const uint32_t f = (uint32_t)(e >> 32), loc = (uint32_t)e;
            const uint32_t r = L.bin[p], s0 = L.start[r], s1 = L.start[r + 1];
            uint32_t s = 0, rank = 0, first = p, least = loc, next = 0u;
            if (s1 - s0 <= kCondLong) {
                for (uint32_t q = s0; q < s1; ++q) {
                    const unsigned long long x = L.key[q];
                    if ((uint32_t)(x >> 32) != f) continue;
                    const uint32_t l = (uint32_t)x;
                    s += 1u;
                    if (l < loc || (l == loc && q < p)) rank += 1u;
                    if (l < least || (l == least && q < first)) {
                        least = l;
                        first = q;
                    }
                    if (q != p) next = l;    // the other location of two
                }
            } else {
                first = feature_bound(L.key, s0, s1, f, false);
                s = feature_bound(L.key, s0, s1, f, true) - first;
                rank = p - first;
                next = s > 1u ? (uint32_t)L.key[first + 1u] : 0u;
            }
            num_same[k] = s;
            rank_first[k] = (rank << 16) | first;
            if (rank == 0u) {
                num_same[k] |= atomicAdd(&L.cnt[r >> sh], 1u) << 16;
                second[k] = next;
                if (s > kCondInline) voff[p] = (uint16_t)atomicAdd(&vcur, s);
            }
        }
        __syncthreads();
        // placement of the features in the slice's index buckets
        place_scan<BPER>(
            L, tid, R, (int)kCondEntries, [&](uint32_t r) { return L.cnt[r]; },
            [&](uint32_t r, uint32_t homed_below, uint32_t placed_to) {
                Te[r] = (uint16_t)homed_below;
                Tp[r] = (uint16_t)placed_to;
            });
        const uint32_t placed = Tp[R - 1];
        const uint64_t v0 = c.slice_vals[z];
        uint4* const lines = idx + (uint64_t)z * R * kCondEntries;
#pragma unroll
        for (uint32_t k = 0; k < PER; ++k) {
            const uint32_t same = num_same[k] & 0xFFFFu;
            if (same == 0u) continue;
            const uint32_t p = k * kCondThreads + tid;
            const unsigned long long e = L.key[p];
            const uint32_t first = rank_first[k] & 0xFFFFu, rank = rank_first[k] >> 16;
            const bool run_of = same > kCondInline;
            const uint64_t off = v0 + voff[first];
            if (run_of) c.val[off + rank] = (uint32_t)e;
            if (rank != 0u) continue;
            const uint32_t f = (uint32_t)(e >> 32);
            uint4 x;
            x.x = f;
            x.y = same;
            x.z = run_of ? (uint32_t)off : (uint32_t)e;
            x.w = run_of ? (uint32_t)(off >> 32) : same == 2u ? second[k] : 0u;
            uint32_t b = L.bin[p] >> sh;
            const uint32_t j = Te[b] + (num_same[k] >> 16);
            if (j >= placed) {             // carried past the slice's index buckets
                const unsigned long long d = atomicAdd(&c.res->deferred, 1ull);
                if (d < c.defer_cap) c.defer[d] = x;
                continue;
            }
            while (j >= Tp[b]) b += 1u;
            lines[b * kCondEntries + (j - (b ? Tp[b - 1u] : 0u))] = x;
        }
        for (uint32_t i = tid; i < R * kCondEntries; i += kCondThreads) {   // free entries
            const uint32_t b = i / kCondEntries;
            if (i % kCondEntries >= (uint32_t)Tp[b] - (b ? Tp[b - 1u] : 0u))
                lines[i] = make_uint4(0u, 0u, 0u, 0u);
        }
    }
}

// Features carried past their slice's index buckets: each claims the first free
// entry from its home bucket on (feature and count by one 64-bit exchange).
__global__ __launch_bounds__(256) void k_condense_defer(CondArgs c) {
    const unsigned long long n = min(c.res->deferred, (unsigned long long)c.defer_cap);
    for (unsigned long long i = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (unsigned long long)gridDim.x * blockDim.x) {
        const uint4 x = c.defer[i];
        const unsigned long long tag = ((unsigned long long)x.y << 32) | x.x;
        uint64_t b = home_bucket(x.x, c.nbc);
        bool placed = false;
        for (uint64_t d = 0; d < c.nbc && !placed; ++d) {
            for (uint32_t p = 0; p < kCondEntries && !placed; ++p) {
                unsigned long long* const e =
                    reinterpret_cast<unsigned long long*>(c.idx) + (b * kCondEntries + p) * 2;
                if ((*e >> 32) == 0ull && atomicCAS(e, 0ull, tag) == 0ull) {
                    e[1] = ((unsigned long long)x.w << 32) | x.z;
                    placed = true;
                }
            }
            b = b + 1 == c.nbc ? 0 : b + 1;
        }
        if (!placed) c.res->failed = 1u;
    }
}

// Test export: every (feature, location) of the condensed layout whose feature
// lies in [lo, hi].
__global__ __launch_bounds__(256) void k_condense_dump(const unsigned int* idx, uint64_t nbc,
                                                       const uint32_t* val, uint32_t lo,
                                                       uint32_t hi, unsigned long long* out,
                                                       uint64_t cap, unsigned long long* count) {
    const uint64_t n = nbc * kCondEntries;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const uint4 e = reinterpret_cast<const uint4*>(idx)[i];
        if (e.y == 0 || e.x < lo || e.x > hi) continue;
        const unsigned long long pos = atomicAdd(count, (unsigned long long)e.y);
        const unsigned long long f = (unsigned long long)e.x << 32;
        for (uint32_t k = 0; k < e.y; ++k) {
            uint32_t loc;
            if (e.y > kCondInline) loc = val[((uint64_t)e.w << 32 | e.z) + k];
            else loc = k == 0 ? e.z : e.w;
            if (pos + k < cap) out[pos + k] = f | loc;
        }
    }
}

inline unsigned grid_cap(uint64_t items, unsigned max_blocks) {
    return (unsigned)(items < 1 ? 1 : items > max_blocks ? max_blocks : items);
}

// log2 of the bins per bucket: buckets << split stays below 2^32 and the bins
// of a slice (per buckets) within `most`.
uint32_t bin_split(uint64_t buckets, uint32_t per, uint32_t most) {
    uint32_t s = 0;
    while (s < kCondBinSplit && (buckets << (s + 1)) <= 0xFFFFFFFFull && (per << (s + 1)) <= most) ++s;
    return s;
}

}  // namespace

hipError_t launch_condense_count(CondArgs c, hipStream_t st) {
    c.split_t = bin_split(c.nb, kCondBuckets, kCondCountBins);
    hipLaunchKernelGGL(k_condense_count, dim3(grid_cap(c.n_slices, 1u << 20)), dim3(kCondThreads), 0,
                       st, c);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_condense_scan, dim3(1), dim3(kCondScanThreads), 0, st, c);
    return hipGetLastError();
}

hipError_t launch_condense_write(CondArgs c, uint32_t most, hipStream_t st) {
    c.split_c = bin_split(c.nbc, c.per_slice, kCondWriteBins);
    const dim3 grid(grid_cap(c.n_slices, 1u << 20)), blk(kCondThreads);
    hipLaunchKernelGGL(k_condense_write<kCondMid>, grid, blk, 0, st, c);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && most > kCondMid) {
        // few slices, if any: a small grid looks them up
        hipLaunchKernelGGL(k_condense_write<kCondCap>, dim3(grid_cap(c.n_slices, 1024)), blk, 0, st,
                           c);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    // the count of deferred features is known on the device only
    hipLaunchKernelGGL(k_condense_defer, dim3(64), dim3(256), 0, st, c);
    return hipGetLastError();
}

hipError_t launch_condense_dump(const unsigned int* idx, uint64_t nbc, const uint32_t* val,
                                uint32_t lo, uint32_t hi, unsigned long long* out, uint64_t cap,
                                unsigned long long* count, hipStream_t st) {
    if (nbc == 0) return hipSuccess;
    const uint64_t n = nbc * kCondEntries;
    hipLaunchKernelGGL(k_condense_dump, dim3(grid_cap((n + 255) / 256, 16384)), dim3(256), 0, st,
                       idx, nbc, val, lo, hi, out, cap, count);
    return hipGetLastError();
}

}  // namespace mc
