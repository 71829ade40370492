// Bucket-table slices gathered into LDS by a workgroup (conversion to the
// condensed layout, table growth): the entries homed in a range of buckets lie
// in these buckets or in the few buckets their chains run on into. They are
// grouped by home (or a finer or coarser division of the feature's hash) by a
// counting sort, and placed into fixed-size buckets by a max-plus scan.
#pragma once

#include "mc_device.hpp"

namespace mc {

constexpr int kSliceThreads = 512;
constexpr uint32_t kSliceWaves = kSliceThreads / kWave;
constexpr uint32_t kSliceBuckets = 1u << kCondSliceShift;      // most buckets of a range
constexpr uint32_t kSliceSlots = kSliceBuckets * kSlots;
constexpr int kSliceHeld = (int)(kSliceSlots / kSliceThreads);   // slots a thread holds

template <typename T, uint32_t CAP, uint32_t BINS, bool kKeepBins>
struct SliceLds {
    T key[CAP];                          // grouped by bin
    uint16_t bin[kKeepBins ? CAP : 1];   // of each key
    uint32_t cnt[BINS];                  // per bin: entries, then for the caller's use
    uint16_t start[BINS + 1];            // first key of each bin
    uint32_t wsum[kSliceWaves];
    int wA[kSliceWaves], wD[kSliceWaves];
    uint32_t tail;
};

// Exclusive prefix of one u32 per thread over the workgroup.
__device__ __forceinline__ uint32_t slice_scan(uint32_t v, uint32_t* wsum, uint32_t& total) {
    const uint32_t t = threadIdx.x, lane = t & 63, w = t >> 6;
    uint32_t x = v;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t y = shfl_idx(x, lane >= (uint32_t)d ? (int)lane - d : (int)lane);
        if (lane >= (uint32_t)d) x += y;
    }
    __syncthreads();
    if (lane == kWave - 1) wsum[w] = x;
    __syncthreads();
    uint32_t base = 0;
    total = 0;
    for (uint32_t i = 0; i < kSliceWaves; ++i) {
        const uint32_t y = wsum[i];
        if (i < w) base += y;
        total += y;
    }
    return base + x - v;
}

// Buckets past `last` that the chains of buckets up to it run on into: up to
// the first bucket that is not full at or after `last` (the table wraps
// around), at most `most`. One wave; kNone if no bucket has a free slot (not a
// valid table).
__device__ __forceinline__ uint32_t tail_buckets(const unsigned long long* table, uint32_t nb,
                                                 uint32_t last, uint32_t most) {
    const uint32_t lane = (uint32_t)lane_id();
    // chains are short: eight buckets first, then 64 at a time
    for (uint64_t base = 0, width = 8; base < nb; base += width, width = kWave) {
        const uint64_t o = base + lane, b = last + o;
        bool open = false;
        if (lane < width && o < nb)
            open = table[(b < nb ? b : b - nb) * kSlots + (kSlots - 1)] == kEmpty;
        const uint64_t m = ballot(open);
        if (m) return min((uint32_t)(base + __builtin_ctzll(m)), most);
    }
    return kNone;
}

// The entries of the buckets [b0, b0 + main) (main <= kSliceBuckets) and of
// their chains' tail for which bin_of(h2(feature)) is below nbins (<= BINS) into
// L.key, grouped by that bin: bin r holds key[start[r], start[r + 1]). Returns
// their number; more than CAP (then nothing is stored), or kNone for a table
// without a free slot. Called by the whole workgroup, which must be done with L.
template <typename T, uint32_t CAP, uint32_t BINS, bool kKeepBins, typename BinOf>
__device__ uint32_t group_slice(const unsigned long long* table, uint32_t nb, uint32_t b0,
                                uint32_t main, SliceLds<T, CAP, BINS, kKeepBins>& L,
                                uint32_t nbins, BinOf bin_of) {
    uint32_t tid = threadIdx.x;           // per-thread indices anew for each slice (not
    asm volatile("" : "+v"(tid));         // held in registers across the slices)
    const unsigned long long* const tab = table + (uint64_t)b0 * kSlots;
    for (uint32_t r = tid; r < nbins; r += kSliceThreads) L.cnt[r] = 0u;
    // the range's own slots, all loads in flight together
    unsigned long long e[kSliceHeld];
#pragma unroll
    for (int j = 0; j < kSliceHeld; ++j) {
        const uint32_t i = (uint32_t)j * kSliceThreads + tid;
        e[j] = i < main * kSlots ? tab[i] : kEmpty;
    }
    if (tid < kWave) {
        const uint32_t t = tail_buckets(table, nb, b0 + main - 1u, nb - main);
        if (tid == 0) L.tail = t;
    }
    __syncthreads();
    const uint32_t tail = L.tail;
    if (tail == kNone) return kNone;
    // bin << 16 | rank within the bin of an entry that counts, else kNone
    auto place = [&](unsigned long long x) -> uint32_t {
        const uint32_t r = bin_of(h2((uint32_t)(x >> 32)));
        if (!live_entry(x) || r >= nbins) return kNone;
        return (r << 16) | atomicAdd(&L.cnt[r], 1u);
    };
    auto tail_slot = [&](uint32_t i) -> unsigned long long {
        const uint64_t b = (uint64_t)b0 + main + i / kSlots;
        return table[(b < nb ? b : b - nb) * kSlots + i % kSlots];
    };
    uint32_t at[kSliceHeld], at_tail = kNone;
#pragma unroll
    for (int j = 0; j < kSliceHeld; ++j) at[j] = place(e[j]);
    // tails of up to kSliceThreads slots are held like the range's own; of
    // longer ones every entry is read again for its place
    const uint32_t n_tail = tail * kSlots;
    const bool again = n_tail > (uint32_t)kSliceThreads;
    unsigned long long et = kEmpty;
    if (tid < n_tail) {
        et = tail_slot(tid);
        at_tail = place(et);
    }
    for (uint32_t i = tid + kSliceThreads; i < n_tail; i += kSliceThreads) (void)place(tail_slot(i));
    __syncthreads();
    constexpr uint32_t PER = (BINS + kSliceThreads - 1) / kSliceThreads;
    uint32_t own[PER], sum = 0, n;
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
        const uint32_t r = tid * PER + k;
        own[k] = r < nbins ? L.cnt[r] : 0u;
        sum += own[k];
    }
    uint32_t run = slice_scan(sum, L.wsum, n);
    if (n > CAP) return n;
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
        const uint32_t r = tid * PER + k;
        if (r < nbins) {
            L.start[r] = (uint16_t)run;
            L.cnt[r] = run;            // cursors, where the entries are read again
            run += own[k];
        }
    }
    if (tid == 0) L.start[nbins] = (uint16_t)n;
    __syncthreads();
    auto put = [&](unsigned long long x, uint32_t r, uint32_t pos) {
        if constexpr (sizeof(T) == 8) L.key[pos] = x;
        else L.key[pos] = (uint32_t)(x >> 32);
        if constexpr (kKeepBins) L.bin[pos] = (uint16_t)r;
    };
    if (!again) {
#pragma unroll
        for (int j = 0; j < kSliceHeld; ++j)
            if (at[j] != kNone)
                put(e[j], at[j] >> 16, L.start[at[j] >> 16] + (at[j] & 0xFFFFu));
        if (at_tail != kNone)
            put(et, at_tail >> 16, L.start[at_tail >> 16] + (at_tail & 0xFFFFu));
    } else {
        auto put_again = [&](unsigned long long x) {
            const uint32_t r = bin_of(h2((uint32_t)(x >> 32)));
            if (live_entry(x) && r < nbins) put(x, r, atomicAdd(&L.cnt[r], 1u));
        };
#pragma unroll
        for (int j = 0; j < kSliceHeld; ++j) put_again(e[j]);
        for (uint32_t i = tid; i < n_tail; i += kSliceThreads) put_again(tail_slot(i));
    }
    __syncthreads();
    return n;
}

// Placement of items into n buckets of `room` places, bucket r being the home
// of homed(r) items: items carried past bucket r are carry(r) = max(0,
// carry(r - 1) + homed(r) - room), a max-plus scan (composition of x ->
// max(A, x + D)). Calls placed_to(r, items homed below r, items placed in
// buckets <= r), in home order: item j of the slice goes to the bucket r with
// placed(r - 1) <= j < placed(r). n <= PER * kSliceThreads; a barrier follows
// the last call.
template <uint32_t PER, typename Lds, typename Homed, typename Placed>
__device__ __forceinline__ void place_scan(Lds& L, uint32_t tid, uint32_t n, int room, Homed homed,
                                           Placed placed_to) {
    const uint32_t lane = tid & 63u, w = tid >> 6;
    const int kLow = -(1 << 30);
    uint32_t S = 0;
    int A = kLow, D = 0;
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
        const uint32_t r = tid * PER + k;
        if (r >= n) break;
        const uint32_t h = homed(r);
        S += h;
        A = max(0, A + (int)h - room);
        D += (int)h - room;
    }
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int src = lane >= (uint32_t)d ? (int)lane - d : (int)lane;
        const uint32_t pS = shfl_idx(S, src);
        const int pA = (int)shfl_idx((uint32_t)A, src), pD = (int)shfl_idx((uint32_t)D, src);
        if (lane >= (uint32_t)d) {
            S += pS;
            A = max(A, pA + D);
            D += pD;
        }
    }
    const int up = lane ? (int)lane - 1 : 0;
    uint32_t eS = shfl_idx(S, up);
    int eA = (int)shfl_idx((uint32_t)A, up), eD = (int)shfl_idx((uint32_t)D, up);
    if (lane == 0) {
        eS = 0;
        eA = kLow;
        eD = 0;
    }
    if (lane == kWave - 1) {
        L.wsum[w] = S;
        L.wA[w] = A;
        L.wD[w] = D;
    }
    __syncthreads();
    uint32_t PS = 0;
    int PA = kLow, PD = 0;
    for (uint32_t i = 0; i < w; ++i) {
        PS += L.wsum[i];
        PA = max(L.wA[i], PA + L.wD[i]);
        PD += L.wD[i];
    }
    uint32_t run = PS + eS;
    int carry = max(0, max(max(eA, PA + eD), PD + eD));
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
        const uint32_t r = tid * PER + k;
        if (r >= n) break;
        const uint32_t h = homed(r), first = run;
        run += h;
        carry = max(0, carry + (int)h - room);
        placed_to(r, first, run - (uint32_t)carry);
    }
    __syncthreads();
}

}  // namespace mc
