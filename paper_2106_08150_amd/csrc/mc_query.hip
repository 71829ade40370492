// Classification kernels (Sec. 4.2, Sec. 5.2-5.6). One wave classifies one
// record: it sketches every window of both mates (same code as the build),
// gathers the location lists of all sketch elements into LDS, sorts them,
// counts equal locations (window count statistic), scores the best range of
// `sws` consecutive windows per target, keeps the top m targets and labels the
// record, by LCA when the top scores are close. Records whose list does not
// fit the fast path's LDS are queued for a second pass with a larger list.
#include <algorithm>
#include <cstddef>

#include "mc_device.hpp"
#include "mc_internal.hpp"

namespace mc {

namespace {

// Kernel arguments used once per record or on rare paths are read where they
// are used (a scalar load from the argument segment at an offset the compiler
// treats as unknown), so they do not occupy scalar registers across the record
// loop; the hot loop needs every scalar register it can get.
template <typename T>
__device__ __forceinline__ T arg_at_use(uint32_t off) {
    asm volatile("" : "+s"(off));
    const __attribute__((address_space(4))) char* base =
        (const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr();
    return *(const __attribute__((address_space(4))) T*)(base + off);
}
// All of the arguments, read here.
template <typename T>
__device__ __forceinline__ T args_at_use() {
    constexpr uint32_t n = sizeof(T) / 4;
    static_assert(sizeof(T) % 4 == 0, "whole words");
    uint32_t w[n];
    uint32_t off = 0;
    asm volatile("" : "+s"(off));
    const __attribute__((address_space(4))) char* base =
        (const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr();
    const __attribute__((address_space(4))) uint32_t* p =
        (const __attribute__((address_space(4))) uint32_t*)(base + off);
#pragma unroll
    for (uint32_t i = 0; i < n; ++i) w[i] = p[i];
    T t;
    __builtin_memcpy(&t, w, sizeof t);
    return t;
}
#define MC_COLD(field) arg_at_use<decltype(QueryArgs::field)>((uint32_t)offsetof(QueryArgs, field))

constexpr int kStageWords = 20;    // one window of at most 271 bases (19 words)
constexpr uint32_t kMaxFeat = 128; // sketch elements buffered before lookups

constexpr uint32_t kRing = kMaxFeat;   // lookup work items: at most one per feature
// Entries [kRing, kRing + kRingMirror) repeat entries [0, kRingMirror), so that
// the 32 items of a batch are read without wrapping (immediate LDS offsets).
constexpr uint32_t kRingMirror = 32;

// LDS of one wave. The sketch area serves a record's sketches and lookups, the
// rank area its run-length and scoring after the last lookup; they overlap.
template <uint32_t LCAP>
struct QueryLds {
    uint2 ring[kRing + kRingMirror];  // (feature, bucket) lookup work items
    uint32_t list[LCAP + kWave];      // waves read up to 63 entries past its end
    union {
        struct {
            Word stage[2 * kStageWords];
            uint32_t scratch[kWave];
            uint32_t feats[kMaxFeat];
        } sk;
        struct {
            uint16_t uidx[LCAP + 2];
            uint16_t score[LCAP];
        } rk;
    };
    uint32_t sel_t[kMaxTopM], sel_s[kMaxTopM], sel_b[kMaxTopM];   // top-m list
};

// s_waitcnt immediate for vmcnt(0) with the other counters left alone (gfx9
// encoding: vmcnt bits 3..0 and 15..14, expcnt 6..4, lgkmcnt 11..8).
constexpr int kWaitVmem0 = 0x0F70;

// Lanes 7, 15, ..., 63: the lanes holding the last slot of the bucket each
// 8-lane group reads.
constexpr uint64_t kLastSlots = 0x8080808080808080ull;

// Inclusive prefix sum over the lanes.
__device__ __forceinline__ uint32_t wave_prefix(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);   // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);  // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);  // row_bcast:31
    return v;
}

// Queue the next bucket of the items whose lane is set in `full`: lane
// 8g + 4 + q stands for item 8q + g of the batch, which it reads again from the
// ring. One pass for the batch; a pass per step took as many instructions for
// each one's one or two items.
__device__ __forceinline__ void requeue(const QueryArgs& a, uint64_t full, const uint2* batch,
                                        uint32_t l3, uint2* ring, uint32_t& tail) {
    uint2 it = batch[8u * l3];                // batch: the lane's group's item of step 0
    // the bucket count is read here, not held across the loop
    it.y = it.y + 1u == (uint32_t)MC_COLD(nb) ? 0u : it.y + 1u;
    const uint32_t pos = rank_below(full, tail) & (kRing - 1u);
    wave_lds_sync();                          // a full ring's new items replace the batch's
    if (lane_in(full)) {
        ring[pos] = it;
        if (pos < kRingMirror) ring[pos + kRing] = it;
    }
    tail += popc64(full);
}

typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
constexpr uint32_t kGroups = 8;      // groups of 8 lanes, one bucket line each
constexpr int kBatchSteps = 4;       // lines in flight a group

// The work items of features F[0..nf) at their home buckets.
__device__ __forceinline__ void fill_ring(const QueryArgs& a, const uint32_t* F, uint32_t nf,
                                          uint2* ring) {
    for (uint32_t i = (uint32_t)lane_id(); i < nf; i += kWave) {
        const uint2 it = make_uint2(F[i], (uint32_t)home_bucket(F[i], a.nb));
        ring[i] = it;
        if (i < kRingMirror) ring[i + kRing] = it;
    }
    wave_lds_sync();
}

// One batch of lookup: c <= 8 NB items (kWhole: exactly that many), l3 the
// lane's place in its quad. Returns false if its hits do not fit the list.
template <uint32_t LCAP, int NB, bool kWhole>
__device__ __forceinline__ bool lookup_batch(const QueryArgs& a, const u64x2* slot2,
                                             const uint2* batch, uint32_t c, uint32_t l3,
                                             uint2* ring, uint32_t* list, uint32_t& nlist,
                                             uint32_t& tail) {
    const uint32_t lane = (uint32_t)lane_id();
    const uint32_t g = lane >> 3;
    uint32_t f[NB], b[NB];
    u64x2 sl[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) {
        const uint2 it = batch[kGroups * q];
        f[q] = it.x;
        b[q] = it.y;
    }
    // groups past the batch's last item load nothing and hold empty slots
#pragma unroll
    for (int q = 0; q < NB; ++q) {
        if (!kWhole) sl[q].x = sl[q].y = ~0ull;
        if (kWhole || (int)g < (int)(c - kGroups * q)) sl[q] = slot2[(uint64_t)b[q] * (kSlots / 2)];
    }
    // A slot is the item's if it holds the item's feature and a stored
    // location (not a tombstone): one 64-bit compare of the slot with the
    // feature taken off. The kernel is bound by instruction issue, scalar as
    // much as vector, so hits are counted a lane and placed by one prefix sum
    // a batch; a wave's hit masks in scalar registers took 15 scalar
    // instructions a slot and step more. With the requeue once a batch and the
    // shorter record header, 10M reads of 150 bases on 4 Gbp: 757 -> 619
    // scalar instructions a read, 14.84 -> 13.5 ms (12.5 with the sorting
    // networks of today; 385M random lines alone would take 10 ms).
    uint32_t nh = 0, fl = 0;
#pragma unroll
    for (int q = 0; q < NB; ++q) {
        const uint64_t fq = (uint64_t)f[q] << 32;
        sl[q].x ^= fq;
        sl[q].y ^= fq;
        nh += sl[q].x < kTombLoc ? 1u : 0u;
        nh += sl[q].y < kTombLoc ? 1u : 0u;
        // full: the location word of the last slot is not all ones (empty)
        fl |= (uint32_t)sl[q].y != 0xFFFFFFFFu ? 1u << q : 0u;
    }
    asm volatile("" : "+v"(fl));
    const uint32_t incl = wave_prefix(nh);
    const uint32_t total = nlist + (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    if (total > LCAP) return false;
    uint32_t* out = list + nlist + incl;
    nlist = total;
#pragma unroll
    for (int q = 0; q < NB; ++q) {
        // compared again: the masks would take 16 scalar registers
        asm volatile("" : "+v"(sl[q]));
        if (sl[q].x < kTombLoc) *--out = (uint32_t)sl[q].x;
        if (sl[q].y < kTombLoc) *--out = (uint32_t)sl[q].y;
    }
    // lane 8g + 4 + q: whether group g's bucket of step q is full
    // (quad broadcast of lane 3, to the odd quads)
    const uint32_t gf = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)fl, 0xFF, 0xF, 0xA, false);
    const uint64_t full = ballot(((gf >> l3) & 1u) != 0u);
    if (full) requeue(a, full, batch, l3, ring, tail);
    return true;
}

// Append the locations of features F[0..nf) to list (LDS). A work item is a
// (feature, bucket) pair; the wave takes up to 8 * NB items at a time, item
// 8q + g read by 8-lane group g as one 128-byte bucket line (16 bytes, two
// slots, a lane), so that NB lines per group are in flight. Slots of a bucket
// fill in order, so a bucket is full exactly when its last slot is occupied:
// a full bucket queues the feature's next bucket as a new item, and a
// feature's chain ends at its first bucket that is not full (inserts never
// pass such a bucket). Items wait in a ring in LDS, at most one per feature;
// every ring entry always holds some item of the launch (the ring is cleared
// to bucket 0 when a wave starts), so groups past a batch's last item may read
// any entry and their lines are simply ignored. Returns false once the list
// would outgrow LCAP (the record goes to the large-list pass).
template <uint32_t LCAP>
__device__ bool lookup(const QueryArgs& a, const uint32_t* F, uint32_t nf, uint2* ring,
                       uint32_t* list, uint32_t& nlist, uint32_t& probes) {
    const uint32_t lane = (uint32_t)lane_id();
    fill_ring(a, F, nf, ring);
    // slots 2 (lane & 7) and 2 (lane & 7) + 1 of a bucket, as one 16-byte load
    const u64x2* const slot2 = reinterpret_cast<const u64x2*>(a.table) + (lane & 7u);
    uint32_t l3 = lane & 3u;
    asm volatile("" : "+v"(l3));
    uint32_t head = 0, tail = nf;
    while (head < tail) {
        // every line issued so far has been used; saying so here lets this
        // batch's loads go out back to back (the compiler cannot tell which
        // of the previous batch's loads were issued)
        __builtin_amdgcn_s_waitcnt(kWaitVmem0);
        const uint32_t c = min(tail - head, kGroups * kBatchSteps);
        // item 8q + g at batch[8q]
        const uint2* const batch = ring + ((head & (kRing - 1u)) + (lane >> 3));
        head += c;
        probes += c;
        // a whole batch (two full windows of a read) needs no masks; a batch
        // of at most a line a group (mostly second buckets of chains) takes
        // one step: 14.0 -> 13.5 ms for 10M reads of 150 bases on 4 Gbp
        bool fits;
        if (c == kGroups * kBatchSteps)
            fits = lookup_batch<LCAP, kBatchSteps, true>(a, slot2, batch, c, l3, ring, list, nlist,
                                                         tail);
        else if (c > kGroups)
            fits = lookup_batch<LCAP, kBatchSteps, false>(a, slot2, batch, c, l3, ring, list,
                                                          nlist, tail);
        else
            fits = lookup_batch<LCAP, 1, false>(a, slot2, batch, c, l3, ring, list, nlist, tail);
        if (!fits) return false;
        wave_lds_sync();
    }
    return true;
}

// Condensed layout: a work item is a (feature, index bucket) pair; 8-lane
// group g reads item 8q + g's index line, one 16-byte entry a lane. A feature
// has exactly one entry: found, its locations are appended (inline ones at
// once; a run is noted in `runs` and copied after the batch, all runs of the
// batch by the whole wave with one flat index, so that their loads are in
// flight together); not found in a full bucket, the feature's next bucket is
// queued. runs: 96 words of LDS owned by the wave. Returns false once the
// list outgrew LCAP.
template <uint32_t LCAP>
__device__ bool lookup_cond(const QueryArgs& a, const uint32_t* F, uint32_t nf, uint2* ring,
                            uint32_t* list, uint32_t* runs, uint32_t& nlist, uint32_t& probes) {
    constexpr int NB = kBatchSteps;
    const uint32_t lane = (uint32_t)lane_id();
    const uint32_t g = lane >> 3;
    fill_ring(a, F, nf, ring);
    const uint4* ent = reinterpret_cast<const uint4*>(a.table) + (lane & 7u);
    uint32_t l3 = lane & 3u;
    asm volatile("" : "+v"(l3));
    uint32_t head = 0, tail = nf;
    while (head < tail) {
        __builtin_amdgcn_s_waitcnt(kWaitVmem0);
        const uint32_t c = min(tail - head, kGroups * NB);
        const uint2* const batch = ring + ((head & (kRing - 1u)) + g);
        uint32_t f[NB], b[NB];
        uint4 e[NB];
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            const uint2 it = batch[kGroups * q];
            f[q] = it.x;
            b[q] = it.y;
        }
#pragma unroll
        for (int q = 0; q < NB; ++q) {   // idle groups load nothing and hold empty entries
            e[q].y = 0u;
            if ((int)g < (int)(c - kGroups * q)) e[q] = ent[(uint64_t)b[q] * kCondEntries];
        }
        head += c;
        probes += c;
        // found and full, one bit a step, and inline locations, a lane at a
        // time (see lookup_batch); an entry that is not the item's counts 0
        uint32_t nh = 0, fl = 0, found = 0;
        uint64_t any_run = 0;
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            fl |= e[q].y != 0u ? 1u << q : 0u;
            if (e[q].x != f[q]) e[q].y = 0u;
            found |= e[q].y != 0u ? 1u << q : 0u;
            nh += e[q].y <= kCondInline ? e[q].y : 0u;
            any_run |= ballot(e[q].y > kCondInline);
        }
        asm volatile("" : "+v"(fl), "+v"(found));
        const uint32_t incl = wave_prefix(nh);
        const uint32_t total = nlist + (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        if (total > LCAP) return false;
        uint32_t* out = list + nlist + incl;
        nlist = total;
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            if (e[q].y - 1u < kCondInline) *--out = e[q].z;
            if (e[q].y == 2u) *--out = e[q].w;
        }
        uint32_t nrun = 0;   // runs of this batch (at most one a group and q: 32)
        if (any_run) {
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                const uint64_t hitR = ballot(e[q].y > kCondInline);
                if (lane_in(hitR)) {
                    const uint32_t r = nrun + rank_below(hitR);
                    runs[3 * r + 0] = e[q].y;
                    runs[3 * r + 1] = e[q].z;
                    runs[3 * r + 2] = e[q].w;
                }
                nrun += popc64(hitR);
            }
        }
        // a group that did not find its feature in a full line goes on:
        // found bits of the group's lanes together, the full bits from its
        // last lane, lane 8g + 4 + q for step q
        found |= xor_lanes<1>(found);
        found |= xor_lanes<2>(found);
        found |= (uint32_t)__builtin_amdgcn_mov_dpp((int)found, 0x141, 0xF, 0xF, false);  // half mirror
        const uint32_t gf =
            (uint32_t)__builtin_amdgcn_update_dpp(0, (int)fl, 0xFF, 0xF, 0xA, false) & ~found;
        const uint64_t full = ballot(((gf >> l3) & 1u) != 0u);
        if (full) requeue(a, full, batch, l3, ring, tail);
        if (nrun) {
            // lane r holds run r; an inclusive scan of the counts gives every
            // run's first list position
            wave_lds_sync();
            const uint32_t cnt = lane < nrun ? runs[3 * lane + 0] : 0u;
            uint32_t incl = cnt;
#pragma unroll
            for (int d = 1; d < 32; d <<= 1) {
                const uint32_t y = shfl_idx(incl, lane >= (uint32_t)d ? (int)lane - d : (int)lane);
                if (lane >= (uint32_t)d) incl += y;
            }
            const uint32_t total = uniform(shfl_idx(incl, (int)nrun - 1));
            if (nlist + total > LCAP) return false;
            wave_lds_sync();
            // runs[3r] = first position of run r (past the runs: above every
            // position), runs[3r + 1..2] = its offset in the value array
            if (lane < 32u) runs[3 * lane] = lane < nrun ? incl - cnt : 0xFFFFFFFFu;
            wave_lds_sync();
            for (uint32_t i = lane; i < total; i += kWave) {
                uint32_t r = 0;   // the last run whose first position is <= i
#pragma unroll
                for (uint32_t step = 16; step > 0; step >>= 1)
                    if (runs[3 * (r + step)] <= i) r += step;
                const uint64_t off = ((uint64_t)runs[3 * r + 2] << 32) | runs[3 * r + 1];
                list[nlist + i] = a.cval[off + (i - runs[3 * r])];
            }
            nlist += total;
        }
        wave_lds_sync();
    }
    return true;
}

template <int K>
__device__ __forceinline__ void sort_regs(uint32_t* list, uint32_t n) {
    const int lane = lane_id();
    uint32_t v[K];
#pragma unroll
    for (int r = 0; r < K; ++r) {
        uint32_t e = (uint32_t)(r * kWave + lane);
        v[r] = e < n ? list[e] : 0xFFFFFFFFu;
    }
    wave_sort<K>(v);
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < K; ++r) {
        uint32_t e = (uint32_t)(r * kWave + lane);
        if (e < n) list[e] = v[r];
    }
    wave_lds_sync();
}

// Lists of more than 128 locations, out of line: the hot loop stays small in
// the instruction cache. The pointer is an LDS pointer so that the out-of-line
// code keeps LDS instructions.
template <uint32_t LCAP>
__device__ __attribute__((noinline)) void sort_list_long(MC_LDS uint32_t* lds_list, uint32_t n) {
    uint32_t* const list = (uint32_t*)lds_list;
    if (n <= 256) sort_regs<4>(list, n);
    else if (n <= 512) sort_regs<8>(list, n);
    else if constexpr (LCAP >= 1024) sort_regs<16>(list, n);
}

// Ascending sort of list[0..n) in LDS (n <= LCAP <= 1024).
template <uint32_t LCAP>
__device__ __forceinline__ void sort_list(uint32_t* list, uint32_t n) {
    static_assert(LCAP <= 1024, "longer lists take the large-list pass");
    if (n <= 64) sort_regs<1>(list, n);
    else if (n <= 128) sort_regs<2>(list, n);
    else sort_list_long<LCAP>((MC_LDS uint32_t*)list, n);
}

// Label and top-m list of a record (lane x writes the x-th top hit).
template <typename Lds>
__device__ __forceinline__ void write_result(const QueryArgs& a, uint32_t rec, uint32_t label,
                                             const Lds& L, uint32_t nsel) {
    const uint32_t lane = (uint32_t)lane_id();
    if (lane == 0) a.out_labels[rec] = label;
    uint32_t* const out_top = MC_COLD(out_top);
    const uint32_t top_m = MC_COLD(top_m);
    if (out_top && lane < top_m) {
        // (opaque: the constants would be held in vector registers)
        uint32_t none = kNone, zero = 0u;
        asm volatile("" : "+v"(none), "+v"(zero));
        const bool h = lane < nsel;
        uint32_t* o = out_top + ((uint64_t)rec * top_m + lane) * 3;
        o[0] = h ? L.sel_t[lane] : none;
        o[1] = h ? L.sel_s[lane] : zero;
        o[2] = h ? L.sel_b[lane] : zero;
    }
}

// floor(n / S): a multiply-high for the counts of any real record, a 64-bit
// division only past 2^32.
__device__ __forceinline__ uint64_t div_by_S(const QueryArgs& a, uint64_t n) {
    if ((n >> 32) == 0) {
        const uint32_t x = (uint32_t)n, t = __umulhi(a.divS.m, x);
        return (t + ((x - t) >> a.divS.sh1)) >> a.divS.sh2;
    }
    uint32_t S = a.S;
    asm volatile("" : "+s"(S));   // its reciprocal is not prepared ahead
    return n / S;
}

// Windows of a mate of len bases, and the windows of reference a fragment of
// F bases can touch (sws; at most those of the longest target, so that the end
// of a range, its first window plus sws, does not wrap).
__device__ __forceinline__ uint64_t mate_windows(const QueryArgs& a, uint64_t len) {
    return len < a.k ? 0 : div_by_S(a, len - a.k + a.S);
}
// The same for a mate of a record shorter than 2^31 bytes: len - k + S then
// fits 32 bits, so the division needs no 64-bit fallback.
__device__ __forceinline__ uint32_t mate_windows32(const QueryArgs& a, uint32_t len) {
    if (len < a.k) return 0u;
    const uint32_t x = len - a.k + a.S, t = __umulhi(a.divS.m, x);
    return (t + ((x - t) >> a.divS.sh1)) >> a.divS.sh2;
}
__device__ __forceinline__ uint32_t fragment_sws(const QueryArgs& a, uint64_t F) {
    return F < a.k ? 1u
                   : (uint32_t)min(div_by_S(a, F - a.k + a.S - 1) + 1, (uint64_t)1 << kWindowBits);
}
// The same for a fragment below 2^32 bases: F - k + S - 1 fits 32 bits unless
// F lies within 512 of 2^32 (S is at most 256).
__device__ __forceinline__ uint32_t fragment_sws32(const QueryArgs& a, uint32_t F) {
    if (F < a.k) return 1u;
    if (F > 0xFFFFFE00u) return fragment_sws(a, F);
    const uint32_t x = F - a.k + a.S - 1u, t = __umulhi(a.divS.m, x);
    return min(((t + ((x - t) >> a.divS.sh1)) >> a.divS.sh2) + 1u, 1u << kWindowBits);
}

// One window of a record: its bytes [lo, hi) inside the mate [vlo, vhi), as
// 32-bit offsets from the record's first byte rounded down to 16 bytes (the
// staging base; records are shorter than 2^31 bytes), its number of k-mer
// starts and the offset of its first base in the staged words.
struct WinRef {
    uint32_t lo, hi, vlo, vhi, nk, x0;
};

// Window i of the record (mate 1's windows first; mate 2 follows mate 1);
// i >= nwt gives an empty one. r0: the record's first byte from the base.
__device__ __forceinline__ WinRef window_ref(const QueryArgs& a, uint32_t i, uint32_t nwt,
                                             uint32_t nw0, uint32_t r0, const uint32_t (&len)[2]) {
    WinRef r{0u, 0u, 0u, 0u, 0u, 0u};
    if (i >= nwt) return r;
    const int sg = i < nw0 ? 0 : 1;
    const uint32_t j = sg ? i - nw0 : i;
    r.vlo = r0 + (sg ? len[0] : 0u);
    r.vhi = r.vlo + len[sg];
    r.lo = r.vlo + j * a.S;
    r.hi = min(r.lo + a.w, r.vhi);
    r.nk = min(a.S, len[sg] - a.k + 1u - j * a.S);
    r.x0 = r.lo & 15u;
    return r;
}

// Words staged for a window: its bytes from the 16-byte boundary below it, plus
// one look-ahead word.
__device__ __forceinline__ uint32_t staged_words(const WinRef& r) {
    return r.nk ? (r.hi - (r.lo & ~15u) + 15u) / 16u + 1u : 0u;
}

// Stage two windows at once, A's words into W[0..) and B's into
// W[kStageWords..), one dword (4 bases) per lane: a 150-base read's two
// windows take a single pass of the wave. dirtyA / dirtyB (wave-uniform): a
// staged byte of that window's mate is not a base.
__device__ __forceinline__ void stage_pair(Word* W, uintptr_t base, const WinRef& A,
                                           const WinRef& B, int lane, uint32_t& dirtyA,
                                           uint32_t& dirtyB) {
    const uint32_t ndA = 4u * staged_words(A), nd = ndA + 4u * staged_words(B);
    // the flags are vector words, not lane masks: merging lane masks across
    // the loop took scalar instructions (scalar issue limits this kernel)
    uint32_t badA = 0u, badB = 0u;
    for (uint32_t q = (uint32_t)lane; q < nd; q += kWave) {
        const bool second = q >= ndA;
        const uint32_t bad = stage_dword(W + (second ? kStageWords : 0), base,
                                         (second ? B.lo : A.lo) & ~15u, second ? q - ndA : q,
                                         second ? B.vlo : A.vlo, second ? B.vhi : A.vhi);
        badA |= second ? 0u : bad;
        badB |= second ? bad : 0u;
    }
    dirtyA = ballot(badA != 0u) != 0 ? 1u : 0u;
    dirtyB = ballot(badB != 0u) != 0 ? 1u : 0u;
}

// A record's staging base and lengths, or false for a record of 2^31 bytes or
// more (beyond every pass: left unclassified and counted as too long).
struct RecordSpan {
    uintptr_t base;
    uint32_t r0;
    uint32_t len[2];
};
__device__ __forceinline__ bool record_span(const QueryArgs& a, uint64_t o0, uint64_t o1,
                                            uint64_t o2, RecordSpan& rs) {
    if (o2 - o0 >= (1ull << 31)) return false;
    const uintptr_t first = (uintptr_t)(a.reads + o0);
    rs.base = first & ~(uintptr_t)15;
    rs.r0 = (uint32_t)(first - rs.base);
    rs.len[0] = (uint32_t)(o1 - o0);
    rs.len[1] = (uint32_t)(o2 - o1);
    return true;
}

struct WaveStats {
    uint32_t features = 0, locations = 0, probes = 0, passed_on = 0;
};

// Label of a record from its top-m list (sel_* in LDS, nsel entries): the
// best target's taxon on a clear lead, else the LCA of the taxa of the listed
// targets within hit_diff of the best score.
// The taxonomy arrays are read by scalar loads (every index is wave-uniform;
// the arrays are small and do not change during a launch).
typedef const __attribute__((address_space(4))) uint32_t ConstU32;
__device__ __forceinline__ ConstU32* scalar_ptr(const uint32_t* p) {
    return (ConstU32*)(uintptr_t)p;
}

__device__ __forceinline__ uint32_t lca_uniform(uint32_t a, uint32_t b, ConstU32* parent,
                                                ConstU32* depth) {
    uint32_t da = depth[a], db = depth[b];
    while (da > db) { a = parent[a]; --da; }
    while (db > da) { b = parent[b]; --db; }
    while (a != b) { a = parent[a]; b = parent[b]; }
    return a;
}

template <typename Lds>
__device__ __forceinline__ uint32_t label_of(const QueryArgs& a, const Lds& L, uint32_t nsel) {
    const uint32_t min_hits = MC_COLD(min_hits), hit_diff = MC_COLD(hit_diff);
    uint32_t label = kNone;
    const uint32_t c1 = uniform(L.sel_s[0]);
    if (nsel > 0 && c1 >= min_hits) {
        const uint32_t c2 = nsel > 1 ? uniform(L.sel_s[1]) : 0u;
        ConstU32* const taxon = scalar_ptr(MC_COLD(target_taxon));
        label = taxon[uniform(L.sel_t[0])];
        if (c1 - c2 <= hit_diff) {
            ConstU32* const parents = scalar_ptr(MC_COLD(parents));
            ConstU32* const depth = scalar_ptr(MC_COLD(depth));
            for (uint32_t x = 1; x < nsel; ++x)
                if ((uint64_t)uniform(L.sel_s[x]) + hit_diff >= c1)
                    label = lca_uniform(label, taxon[uniform(L.sel_t[x])], parents, depth);
        }
    }
    return label;
}

// Whether the top-m rounds can stop after round m (score: its score): only
// when no top-hit list is written; then after the first round if the best
// score is below min_hits (unclassified), else at the first score more than
// hit_diff below the best (later, lower entries take no part in the label).
struct TopStop {
    bool whole_list;
    uint32_t min_hits, hit_diff, c_best = 0;
    __device__ __forceinline__ bool operator()(uint32_t m, uint32_t score) {
        if (whole_list) return false;
        if (m == 0) {
            c_best = score;
            return score < min_hits;
        }
        return (uint64_t)score + hit_diff < c_best;
    }
};

// Steps Q5-Q8 for a list of at most 64 locations (most records), held one a
// lane: sorted in registers; the runs of equal locations (window counts) are
// found with one ballot; distinct location u moves to lane u with its first
// list index P(u) (the number of smaller locations), so that a range's score
// is P(end) - P(u), end being the first distinct location past the range
// (at most sws windows of one target); top-m by wave maxima as below.
template <typename Lds>
__device__ __forceinline__ void label_short_list(const QueryArgs& a, uint32_t rec, Lds& L,
                                                 uint32_t n, uint32_t sws) {
    const uint32_t lane = (uint32_t)lane_id();
    uint32_t v[1] = {lane < n ? L.list[lane] : 0xFFFFFFFFu};
    wave_sort<1>(v);
    const uint32_t prev = (uint32_t)__builtin_amdgcn_mov_dpp((int)v[0], 0x138, 0xF, 0xF, false);
    const uint64_t firsts = lanes_below(n) & (ballot(v[0] != prev) | 1ull);
    const uint32_t U = popc64(firsts);
    uint32_t* const first_of = L.sk.scratch;          // lane of distinct location u
    if (lane_in(firsts)) first_of[rank_below(firsts)] = lane;
    wave_lds_sync();
    const uint32_t P = lane < U ? first_of[lane] : n;    // P(U) = n
    const uint32_t loc = shfl_idx(v[0], (int)(P & 63u));
    wave_lds_sync();
    // end of the range of sws windows starting at loc (not past its target)
    const uint32_t w = loc & kWindowMask, base = loc - w;
    const uint32_t lim = base + min(w + sws, 1u << kWindowBits);
    uint32_t end = lane + 1u;
    const uint32_t steps = min(sws, U);
    for (uint32_t j = 1; j < steps; ++j) {
        const uint32_t l2 = shfl_idx(loc, (int)min(lane + j, 63u));
        end += (lane + j < U && l2 < lim) ? 1u : 0u;
    }
    const uint32_t Pend = shfl_idx(P, (int)min(end, 63u));
    const uint32_t score = (end >= U ? n : Pend) - P;
    uint32_t key = lane < U ? (score << 16) | (0xFFFFu - lane) : 0u;
    const uint32_t t = loc >> kWindowBits;
    TopStop stop{MC_COLD(out_top) != nullptr, MC_COLD(min_hits), MC_COLD(hit_diff)};
    const uint32_t top_m = MC_COLD(top_m);
    uint32_t nsel = 0;
    for (uint32_t m = 0; m < top_m; ++m) {
        const uint32_t k = wave_max_u32(key);
        if (k == 0) break;
        const uint32_t sl = (uint32_t)__builtin_amdgcn_readlane((int)loc, (int)(0xFFFFu - (k & 0xFFFFu)));
        if (lane == 0) {
            L.sel_t[m] = sl >> kWindowBits;
            L.sel_s[m] = k >> 16;
            L.sel_b[m] = sl & kWindowMask;
        }
        nsel = m + 1;
        if (stop(m, k >> 16)) break;
        if (t == sl >> kWindowBits) key = 0;
    }
    wave_lds_sync();
    write_result(a, rec, label_of(a, L, nsel), L, nsel);
}

// A record with more sketch elements than the fast pass's list holds may
// outgrow it. From 2^kLongBits bases on it goes to the large-list pass at once,
// whose eight waves share its windows (a wave takes about 2 us a window, and the
// last records of a launch hold it up). A shorter one stays: each time its
// buffered features have been looked up, the locations it would have in all at
// the rate so far are compared with the list, and it goes on only when they
// exceed it by a sixteenth. What a record holds decides, not its length alone:
// a read of a stored genome has a location or more an element, one of an
// organism that the database does not hold has few. 60 MB of reads on 100 Mbp,
// list of 256 / 512, against handing on every record past the list's capacity:
// foreign reads of 2,200 bases 1.01 / .22 -> .21 / .21 ms, of 5,000 .60 / .60 ->
// .23 / .23, of 10,000 .49 either way (72 windows and more: eight waves each);
// stored reads of 5,000 .66 -> .67 / .69; 20,000 reads of 0.8 to 10 kbp, 5%
// foreign, on 1 Gbp 1.06 -> 1.09.
constexpr uint32_t kLongBits = 13;

template <uint32_t LCAP, int KPL, bool C>
__device__ void classify_record(const QueryArgs& a, uint32_t rec, QueryLds<LCAP>& L,
                                const Threshold& th, WaveStats& ws) {
    const int lane = lane_id();
    // the record's offsets by scalar loads (rec is wave-uniform; the array
    // does not change during the launch)
    typedef const __attribute__((address_space(4))) uint64_t ConstU64;
    ConstU64* const off = (ConstU64*)(uintptr_t)a.offsets;
    const uint32_t at0 = a.paired;
    const uint64_t o0 = off[(uint64_t)rec << at0], o1 = off[((uint64_t)rec << at0) + 1];
    const uint64_t o2 = at0 ? off[((uint64_t)rec << at0) + 2] : o1;
    // one test for every record that is not to be classified here: with both
    // lengths and their sum below 2^kLongBits and no wrap past 2^64 the offsets
    // ascend and the record is short
    const uint64_t d0 = o1 - o0, d1 = o2 - o1;
    RecordSpan rs;
    rs.len[0] = (uint32_t)d0;
    rs.len[1] = (uint32_t)d1;
    const uint32_t len = rs.len[0] + rs.len[1];
    if (__builtin_expect(((uint32_t)(d0 >> 32) | (uint32_t)(d1 >> 32) |
                          ((rs.len[0] | rs.len[1] | len) >> kLongBits)) != 0u ||
                          (uint32_t)(o2 >> 32) < (uint32_t)(o0 >> 32), 0)) {
        const bool malformed = o1 < o0 || o2 < o1;   // nothing to classify
        if (malformed || o2 - o0 >= (1ull << 31)) {  // or too long for every pass
            if (!malformed && lane == 0) atomicAdd(&MC_COLD(counters)[kQTooLong], 1u);
            write_result(a, rec, kNone, L, 0);
            return;
        }
        if ((mate_windows32(a, rs.len[0]) + mate_windows32(a, rs.len[1])) * a.s > LCAP) {
            if (lane == 0) MC_COLD(queue)[atomicAdd(&MC_COLD(counters)[kQOverflow], 1u)] = rec;
            ws.passed_on += 1;
            return;
        }
    }
    const uintptr_t first = (uintptr_t)(a.reads + o0);
    rs.base = first & ~(uintptr_t)15;
    rs.r0 = (uint32_t)first & 15u;

    // windows of the record, mate 1's then mate 2's, sketched two at a time,
    // and the reference windows its fragment can touch: the fragment is the
    // record's length, or the insert size when that is longer and both mates
    // are present
    uint32_t nws[2], sws;
    nws[0] = mate_windows32(a, rs.len[0]);
    nws[1] = 0u;
    if (rs.len[1] == 0u) {
        // ceil((len - k) / S) + 1 from floor((len - k) / S) + 1 windows
        sws = nws[0] + (rs.len[0] > a.k && (nws[0] - 1u) * a.S != rs.len[0] - a.k ? 1u : 0u);
        sws = max(sws, 1u);
    } else {
        nws[1] = mate_windows32(a, rs.len[1]);
        sws = fragment_sws32(a, rs.len[0] > 0u ? max(MC_COLD(insert_size), len) : len);
    }
    const uint32_t nwt = nws[0] + nws[1];
    uint32_t nlist = 0, nf = 0;
    bool fits = true;
    for (uint32_t p = 0; p < nwt && fits; p += 2) {
        WinRef wr[2];
        for (int h = 0; h < 2; ++h) wr[h] = window_ref(a, p + h, nwt, nws[0], rs.r0, rs.len);
        wave_lds_sync();
        uint32_t dirtyA, dirtyB;
        stage_pair(L.sk.stage, rs.base, wr[0], wr[1], lane, dirtyA, dirtyB);
        wave_lds_sync();
        const Word *const WA = L.sk.stage, *const WB = L.sk.stage + kStageWords;
        PairSketch ps = sketch_pair<KPL>(WA, wr[0].x0, wr[0].nk, WB, wr[1].x0, wr[1].nk, a.k, a.s,
                                         th, L.sk.scratch, dirtyA, dirtyB, lane_here());
        sketch_rest<KPL>(ps, WA, wr[0].x0, wr[0].nk, WB, wr[1].x0, wr[1].nk, a.k, a.s,
                         L.sk.feats + nf, L.sk.feats + nf + a.s, L.sk.scratch);
        const uint32_t nA = ps.nA, nB = ps.nB;
        wave_lds_sync();
        if (nA < a.s && nB) {      // close the gap after A's features
            const uint32_t f = (uint32_t)lane < nB ? L.sk.feats[nf + a.s + lane] : 0u;
            wave_lds_sync();
            if ((uint32_t)lane < nB) L.sk.feats[nf + nA + lane] = f;
            wave_lds_sync();
        }
        nf += nA + nB;
        // look up the buffered features after the last pair or before the
        // buffer could overflow (one call site keeps the loop compact)
        if (nf && (p + 2 >= nwt || nf + 2 * a.s > kMaxFeat)) {
            ws.features += nf;
            if constexpr (C)   // the stage and scratch areas hold the runs meanwhile
                fits = lookup_cond<LCAP>(a, L.sk.feats, nf, L.ring, L.list,
                                         reinterpret_cast<uint32_t*>(L.sk.stage), nlist,
                                         ws.probes);
            else
                fits = lookup<LCAP>(a, L.sk.feats, nf, L.ring, L.list, nlist, ws.probes);
            nf = 0;
            // (after the last lookup the list holds all of its locations)
            if (nlist * nwt > (LCAP + LCAP / 16) * (p + 2)) fits = false;
        }
    }
    if (!fits) {
        // queued for the large-list pass
        if (lane == 0) MC_COLD(queue)[atomicAdd(&MC_COLD(counters)[kQOverflow], 1u)] = rec;
        ws.passed_on += 1;
        return;
    }
    wave_lds_sync();
    const uint32_t n = nlist;
    ws.locations += n;
    if (n <= (uint32_t)kWave) {
        label_short_list(a, rec, L, n, sws);
        return;
    }
    sort_list<LCAP>(L.list, n);

    // run-length encoding: uidx[u] = first index of the u-th distinct location
    uint32_t U = 0;
    for (uint32_t c = 0; c < n; c += kWave) {
        // i < n + 63 < LCAP + 64: every lane reads inside the list
        const uint32_t i = c + (uint32_t)lane;
        const uint32_t cur = L.list[i], prev = L.list[i ? i - 1u : 0u];
        const uint64_t mb = lanes_below(n - c) & (ballot(cur != prev) | (c == 0 ? 1ull : 0ull));
        if (lane_in(mb)) L.rk.uidx[U + rank_below(mb)] = (uint16_t)i;
        U += popc64(mb);
    }
    if (lane == 0) L.rk.uidx[U] = (uint16_t)n;
    wave_lds_sync();

    // score of the range of sws windows starting at each distinct location
    for (uint32_t u = (uint32_t)lane; u < U; u += kWave) {
        const uint32_t loc = L.list[L.rk.uidx[u]];
        const uint32_t t = loc >> kWindowBits, w_end = (loc & kWindowMask) + sws;
        uint32_t score = 0;
        for (uint32_t v = u; v < U; ++v) {
            const uint32_t l2 = L.list[L.rk.uidx[v]];
            if ((l2 >> kWindowBits) != t || (l2 & kWindowMask) >= w_end) break;
            score += (uint32_t)L.rk.uidx[v + 1] - (uint32_t)L.rk.uidx[v];
        }
        L.rk.score[u] = (uint16_t)score;
    }
    wave_lds_sync();

    // top-m targets by (score desc, target asc); per target the range with the
    // highest score, ties to the smallest start window. The key of distinct
    // location u is score << 16 | (0xFFFF - u): distinct locations ascend with
    // u, so the wave maximum of the keys is the highest score and, among equal
    // scores, the smallest location (smallest target, then window). Each of
    // the m rounds takes one wave maximum and then drops the chosen target.
    //
    // Without a top-hit output only the label needs the list, and the rounds
    // stop once it is decided: after the first round if its score is below
    // min_hits (unclassified), else at the first score more than hit_diff
    // below the best (a clear lead after the second round; later entries
    // with lower scores take no part in the LCA).
    uint32_t nsel = 0;
    const uint32_t top_m = MC_COLD(top_m);
    TopStop decided{MC_COLD(out_top) != nullptr, MC_COLD(min_hits), MC_COLD(hit_diff)};
    if (U <= (uint32_t)kWave) {          // one distinct location per lane
        uint32_t key = 0, t = kNone;
        if ((uint32_t)lane < U) {
            t = L.list[L.rk.uidx[lane]] >> kWindowBits;
            key = ((uint32_t)L.rk.score[lane] << 16) | (0xFFFFu - (uint32_t)lane);
        }
        for (uint32_t m = 0; m < top_m; ++m) {
            const uint32_t k = wave_max_u32(key);
            if (k == 0) break;
            const uint32_t loc = L.list[L.rk.uidx[0xFFFFu - (k & 0xFFFFu)]];
            if (lane == 0) {
                L.sel_t[m] = loc >> kWindowBits;
                L.sel_s[m] = k >> 16;
                L.sel_b[m] = loc & kWindowMask;
            }
            nsel = m + 1;
            if (decided(m, k >> 16)) break;
            if (t == loc >> kWindowBits) key = 0;
        }
        wave_lds_sync();
    } else {
        for (uint32_t m = 0; m < top_m; ++m) {
            uint32_t key = 0;
            for (uint32_t u = (uint32_t)lane; u < U; u += kWave) {
                const uint32_t t = L.list[L.rk.uidx[u]] >> kWindowBits;
                bool excluded = false;
                for (uint32_t x = 0; x < m; ++x) excluded |= (L.sel_t[x] == t);
                const uint32_t ku = ((uint32_t)L.rk.score[u] << 16) | (0xFFFFu - u);
                if (!excluded && ku > key) key = ku;
            }
            const uint32_t k = wave_max_u32(key);
            if (k == 0) break;
            const uint32_t loc = L.list[L.rk.uidx[0xFFFFu - (k & 0xFFFFu)]];
            if (lane == 0) {
                L.sel_t[m] = loc >> kWindowBits;
                L.sel_s[m] = k >> 16;
                L.sel_b[m] = loc & kWindowMask;
            }
            wave_lds_sync();
            nsel = m + 1;
            if (decided(m, k >> 16)) break;
        }
    }

    write_result(a, rec, label_of(a, L, nsel), L, nsel);
}

// Occupancy: the lookups' memory latency is hidden by other waves' work, so
// occupancy pays for a few spilled scalar registers. A 512-entry list takes
// 5,736 bytes of LDS a wave, which holds a CU to 28 waves: seven a SIMD (at
// most 72 VGPRs). A 256-entry list takes 4,064, so eight waves a SIMD fit (64
// VGPRs), also with the condensed layout's lookups (63, more scalar spills than
// at seven, and 4% faster). A 1,024-entry list (9,832) allows four.
//
// The 256- and 512-entry variants take no scratch memory; the 1,024-entry ones
// take 40 bytes a lane (88 with the condensed layout), in which the out-of-line
// sort of 1,024 entries saves registers. A kernel with scratch makes the runtime
// set it up for the hardware queue it runs on: milliseconds on a queue's first
// such launch, so the first classification with that list is slower than the rest.
static_assert(sizeof(QueryLds<256>) == 4064 && sizeof(QueryLds<512>) == 5736 &&
              sizeof(QueryLds<1024>) == 9832, "LDS a wave");
template <uint32_t LCAP>
constexpr int classify_waves_per_simd() {
    return LCAP <= 256 ? 8 : LCAP <= 512 ? 7 : 4;
}

template <uint32_t LCAP, int WPB, int KPL, bool C>
__global__ __launch_bounds__(WPB * 64)
__attribute__((amdgpu_waves_per_eu(classify_waves_per_simd<LCAP>())))
void k_classify(QueryArgs a, int cls) {
    __shared__ QueryLds<LCAP> L[WPB];
    const int wave = (int)uniform(threadIdx.x >> 6);
    for (uint32_t i = (uint32_t)lane_id(); i < kRing + kRingMirror; i += kWave)
        L[wave].ring[i] = make_uint2(0u, 0u);   // any item must name a bucket of the table
    wave_lds_sync();
    // the records of this launch: all of them, or those of size class cls >= 0
    // (routed); the id arrays are read where they are used (no registers held
    // across the record loop)
    const uint32_t n_iter = cls >= 0 ? uniform(a.route_meta[cls]) : a.n_records;
    WaveStats ws;
    const Threshold th(a.S, a.s);
    for (uint32_t it = blockIdx.x * WPB + wave; it < n_iter; it += gridDim.x * WPB) {
        uint32_t rec = it;
        if (cls >= 0) {
            const uint32_t* const meta = MC_COLD(route_meta);
            rec = uniform(MC_COLD(route_queue)[meta[kMaxRoutes + cls] + it]);
        }
        classify_record<LCAP, KPL, C>(a, rec, L[wave], th, ws);
    }
    // work of records that go on to the large-list pass counts in both passes
    if (lane_id() == 0 && a.qstats) {
        unsigned long long* q = a.qstats + ((blockIdx.x * WPB + wave) % kQsCopies) * kQsStride;
        if (ws.features) atomicAdd(&q[kQsFeatures], (unsigned long long)ws.features);
        if (ws.locations) atomicAdd(&q[kQsLocations], (unsigned long long)ws.locations);
        if (ws.probes) atomicAdd(&q[kQsProbes], (unsigned long long)ws.probes);
        if (ws.passed_on) atomicAdd(&q[kQsLarge], (unsigned long long)ws.passed_on);
    }
}

// ---------------------------------------------------- large-list pass -----
// Records whose candidate list outgrew the fast path, up to kListLarge
// locations: one workgroup of eight waves a record. The waves share the
// record's windows (sketches into one feature buffer), its lookups (one list
// in LDS) and its sort; 79 KB of LDS, so two workgroups a CU overlap each
// other's phases. Bound by the latency of those phases at 16 waves a CU.
//
// One wave a record with a bitonic sort in LDS and a scan over each range (the
// form this replaces) left most of the chip idle and took O(range) steps per
// location: 20,000 reads of 0.8 to 10 kbp on 1 Gbp (11,530 records of about
// 1,450 locations) 296 -> 0.85 ms, 4,000 mixed records on 300 identical genomes
// (3,792 records of about 5,800) 336 -> 0.70 ms (0.97 and 0.75 before the sorting
// networks without directions; sorting and ranking were 0.27 and 0.34 of that).
// Vector issue is at 46% and 43% of its peak there.
constexpr int kLargeWaves = 8;
constexpr int kLargeThreads = kLargeWaves * kWave;
constexpr uint32_t kLargeFeats = 1024;   // sketch elements buffered before lookups

struct LargeWave {
    Word stage[2 * kStageWords];         // lookups of the condensed layout: runs
    uint32_t scratch[kWave];
    uint32_t sk[2 * 64];                 // sketches of a window pair
};
struct LargeLds {
    uint32_t list[kListLarge];
    uint32_t feats[kLargeFeats];
    LargeWave wv[kLargeWaves];
    uint32_t red[kLargeWaves];
    uint32_t nfeat, nlist;
    uint32_t sel_t[kMaxTopM], sel_s[kMaxTopM], sel_b[kMaxTopM];
};
static_assert(sizeof(LargeLds) + 16 <= 80 * 1024, "two workgroups a CU");

// Place of list entry i: the low five index bits are swapped around by the
// next five, so that neither the lanes' runs of consecutive entries (the
// register sort) nor entries a power of two apart fall into one LDS bank.
__device__ __forceinline__ uint32_t at(uint32_t i) { return i ^ ((i >> 5) & 31u); }

// All 8 lanes of the groups whose last lane is set in `last`.
__device__ __forceinline__ uint64_t groups_of(uint64_t last) {
    const uint64_t first = last >> 7;
    return (first << 8) - first;
}

// Append the locations of features F[0..nf) of the workgroup's buffer to the
// list; called by all waves (no barrier inside). An 8-lane group takes NB
// features and reads one bucket line of each at a time (kDeep: one feature,
// NB consecutive buckets of its chain at a time, for few features with long
// chains). L.nlist counts every location found, also past kListLarge (those
// are not stored).
template <bool kDeep>
__device__ __forceinline__ void large_lookup(const QueryArgs& a, LargeLds& L, uint32_t nf,
                                             uint32_t wave, uint32_t& probes) {
    constexpr int NB = 4;
    constexpr uint32_t kPerWave = kDeep ? 8u : 8u * NB;
    const uint32_t lane = (uint32_t)lane_id(), g = lane >> 3;
    const u64x2* slot2 = reinterpret_cast<const u64x2*>(a.table) + (lane & 7u);
    const uint32_t nb = (uint32_t)a.nb;
    for (uint32_t i0 = wave * kPerWave; i0 < nf; i0 += kLargeWaves * kPerWave) {
        uint32_t f[NB], b[NB];
        uint64_t alive[NB];     // groups whose chain goes on (deep: of the one feature)
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            const uint32_t i = i0 + (kDeep ? 0u : 8u * q) + g;
            f[q] = L.feats[min(i, nf - 1u)];
            alive[q] = ballot(i < nf);
            b[q] = (uint32_t)home_bucket(f[q], a.nb);
            if (kDeep) {
                b[q] += (uint32_t)q;
                if (b[q] >= nb) b[q] -= nb;
            }
        }
        for (;;) {
            u64x2 sl[NB];
#pragma unroll
            for (int q = 0; q < NB; ++q)
                if (lane_in(alive[q])) sl[q] = slot2[(uint64_t)b[q] * (kSlots / 2)];
            uint64_t hit0[NB], hit1[NB], any = 0;
            uint32_t c = 0;
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                if (kDeep && q) alive[q] = alive[q - 1];
                const unsigned long long s0 = sl[q].x, s1 = sl[q].y;
                hit0[q] = alive[q] & ballot((uint32_t)(s0 >> 32) == f[q]) &
                          ballot((uint32_t)s0 < kTombLoc);
                hit1[q] = alive[q] & ballot((uint32_t)(s1 >> 32) == f[q]) &
                          ballot((uint32_t)s1 < kTombLoc);
                c += popc64(hit0[q]) + popc64(hit1[q]);
                probes += popc64(alive[q] & kLastSlots);
                // a chain ends at its first bucket that is not full
                alive[q] = groups_of(alive[q] & kLastSlots & ballot((uint32_t)s1 != 0xFFFFFFFFu));
                any |= alive[q];
            }
            if (kDeep) any = alive[NB - 1];
            if (c) {
                uint32_t base = 0;
                if (lane == 0) base = atomicAdd(&L.nlist, c);
                base = uniform(base);
                if (base + c > kListLarge) return;
#pragma unroll
                for (int q = 0; q < NB; ++q) {
                    if (lane_in(hit0[q])) L.list[at(rank_below(hit0[q], base))] = (uint32_t)sl[q].x;
                    base += popc64(hit0[q]);
                    if (lane_in(hit1[q])) L.list[at(rank_below(hit1[q], base))] = (uint32_t)sl[q].y;
                    base += popc64(hit1[q]);
                }
            }
            if (!any) break;
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                if (kDeep) alive[q] = any;
                b[q] += kDeep ? (uint32_t)NB : 1u;
                if (b[q] >= nb) b[q] -= nb;
            }
        }
    }
}

// The same from the condensed layout: a feature's one entry is inline or a
// run of the value array; the runs of a step are copied by the whole wave with
// one flat index (see lookup_cond).
__device__ __forceinline__ void large_lookup_cond(const QueryArgs& a, LargeLds& L, uint32_t nf,
                                                  uint32_t wave, uint32_t& probes) {
    constexpr int NB = 4;
    const uint32_t lane = (uint32_t)lane_id(), g = lane >> 3;
    const uint4* ent = reinterpret_cast<const uint4*>(a.table) + (lane & 7u);
    const uint32_t nb = (uint32_t)a.nb;
    uint32_t* const runs = reinterpret_cast<uint32_t*>(L.wv[wave].stage);   // 96 words
    for (uint32_t i0 = wave * 8u * NB; i0 < nf; i0 += kLargeWaves * 8u * NB) {
        uint32_t f[NB], b[NB];
        uint64_t alive[NB];
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            const uint32_t i = i0 + 8u * q + g;
            f[q] = L.feats[min(i, nf - 1u)];
            alive[q] = ballot(i < nf);
            b[q] = (uint32_t)home_bucket(f[q], a.nb);
        }
        for (;;) {
            uint4 e[NB];
#pragma unroll
            for (int q = 0; q < NB; ++q)
                if (lane_in(alive[q])) e[q] = ent[(uint64_t)b[q] * kCondEntries];
            uint64_t hitA[NB], hitB[NB], any = 0;
            uint32_t nrun = 0, c = 0;
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                const uint64_t used = alive[q] & ballot(e[q].y != 0u);
                const uint64_t mine = used & ballot(e[q].x == f[q]);
                const uint64_t small = ballot(e[q].y <= kCondInline);
                const uint64_t hitR = mine & ~small;
                hitA[q] = mine & small;
                hitB[q] = hitA[q] & ballot(e[q].y == 2u);
                c += popc64(hitA[q]) + popc64(hitB[q]);
                if (lane_in(hitR)) {
                    const uint32_t r = nrun + rank_below(hitR);
                    runs[3 * r + 0] = e[q].y;
                    runs[3 * r + 1] = e[q].z;
                    runs[3 * r + 2] = e[q].w;
                }
                nrun += popc64(hitR);
                probes += popc64(alive[q] & kLastSlots);
                // groups that did not find their feature in a full line go on
                uint64_t gf = mine;
                gf |= gf >> 1;
                gf |= gf >> 2;
                gf |= gf >> 4;
                alive[q] = groups_of(used & kLastSlots & ~((gf & 0x0101010101010101ull) << 7));
                any |= alive[q];
            }
            uint32_t incl = 0, cnt = 0, total = 0;
            if (nrun) {   // lane r holds run r
                wave_lds_sync();
                cnt = lane < nrun ? runs[3 * lane + 0] : 0u;
                incl = cnt;
#pragma unroll
                for (int d = 1; d < 32; d <<= 1) {
                    const uint32_t y = shfl_idx(incl, lane >= (uint32_t)d ? (int)lane - d : (int)lane);
                    if (lane >= (uint32_t)d) incl += y;
                }
                total = uniform(shfl_idx(incl, (int)nrun - 1));
                wave_lds_sync();
                // first position of run r (past the runs: above every position)
                if (lane < 32u) runs[3 * lane] = lane < nrun ? incl - cnt : 0xFFFFFFFFu;
                wave_lds_sync();
            }
            if (c + total) {
                uint32_t base = 0;
                if (lane == 0) base = atomicAdd(&L.nlist, c + total);
                base = uniform(base);
                if (base + c + total > kListLarge) return;
#pragma unroll
                for (int q = 0; q < NB; ++q) {
                    if (lane_in(hitA[q])) L.list[at(rank_below(hitA[q], base))] = e[q].z;
                    base += popc64(hitA[q]);
                    if (lane_in(hitB[q])) L.list[at(rank_below(hitB[q], base))] = e[q].w;
                    base += popc64(hitB[q]);
                }
                for (uint32_t i = lane; i < total; i += kWave) {
                    uint32_t r = 0;   // the last run whose first position is <= i
#pragma unroll
                    for (uint32_t step = 16; step > 0; step >>= 1)
                        if (runs[3 * (r + step)] <= i) r += step;
                    const uint64_t off = ((uint64_t)runs[3 * r + 2] << 32) | runs[3 * r + 1];
                    L.list[at(base + i)] = a.cval[off + (i - runs[3 * r])];
                }
                wave_lds_sync();
            }
            if (!any) break;
#pragma unroll
            for (int q = 0; q < NB; ++q) b[q] = b[q] + 1u == nb ? 0u : b[q] + 1u;
        }
    }
}

// Compare-exchange steps of strides top/2, top/4, ..., 1 (all ascending) of a
// bitonic merge; element lane * K + r of the wave in v[r]. top <= 64 * K.
template <int K>
__device__ __forceinline__ void merge_steps(uint32_t (&v)[K], int top) {
#pragma unroll
    for (int stride = 32 * K; stride >= K; stride >>= 1) {
        if (stride >= top) continue;
        const uint32_t high = high_lanes((uint32_t)lane_id(), stride / K);
#pragma unroll
        for (int r = 0; r < K; ++r) v[r] = keep_of(v[r], xor_lanes_c(v[r], stride / K), high);
    }
#pragma unroll
    for (int stride = K / 2; stride >= 1; stride >>= 1) {
        if (stride >= top) continue;
#pragma unroll
        for (int r = 0; r < K; ++r) {
            if (r & stride) continue;
            const uint32_t x = v[r], y = v[r + stride];
            v[r] = x < y ? x : y;
            v[r + stride] = x < y ? y : x;
        }
    }
}

// Ascending sort of a wave's 64 * K keys (element lane * K + r in v[r]). Steps
// of strides below K stay inside a lane (one minimum and one maximum a pair),
// so most of the network needs no lane exchange. Descending blocks are sorted
// ascending with their keys complemented.
template <int K>
__device__ __forceinline__ void sort_blocked(uint32_t (&v)[K]) {
    const int lane = lane_id();
#pragma unroll
    for (int size = 2; size < K; size <<= 1) {
#pragma unroll
        for (int stride = size / 2; stride >= 1; stride >>= 1)
#pragma unroll
            for (int r = 0; r < K; ++r) {
                if (r & stride) continue;
                const uint32_t x = v[r], y = v[r + stride];
                const uint32_t lo = x < y ? x : y, hi = x < y ? y : x;
                v[r] = (r & size) ? hi : lo;
                v[r + stride] = (r & size) ? lo : hi;
            }
    }
#pragma unroll
    for (int size = K < 2 ? 2 : K; size <= 64 * K; size <<= 1) {
        const uint32_t flip = size < 64 * K && (lane & (size / K)) != 0 ? 0xFFFFFFFFu : 0u;
#pragma unroll
        for (int r = 0; r < K; ++r) v[r] ^= flip;
        merge_steps<K>(v, size);
#pragma unroll
        for (int r = 0; r < K; ++r) v[r] ^= flip;
    }
}

// The steps Q5-Q8 of a record whose n locations are in L.list, n <= 512 * K:
// bitonic sort by the workgroup (each wave sorts 64 * K entries in registers;
// the three merge levels across the eight waves start with one pass in which
// a thread holds the eight entries of a column, one per wave's run), then for
// each distinct location, at its first entry i of the sorted list, the score
// of its range as (first entry past the range) - i by binary search, and the
// top-m rounds on score << 16 | (0xFFFF - i), kept in registers.
template <int K>
__device__ __forceinline__ void large_rank(const QueryArgs& a, LargeLds& L, uint32_t rec,
                                           uint32_t n, uint32_t sws) {
    constexpr uint32_t kRun = 64 * K, P = kLargeThreads * K;
    // (entry places are computed for this record, not held across the records)
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const uint32_t lane = tid & 63u, wave = uniform(tid >> 6);
    // the first of the lane's entries, anew for every pass over them (the
    // entries' places are not kept in registers from one pass to the next)
    auto first_entry = [&]() -> uint32_t {
        uint32_t e = wave * kRun + lane * K;
        asm volatile("" : "+v"(e));
        return e;
    };
    auto store_run = [&](const uint32_t (&v)[K], uint32_t desc) {
        const uint32_t e0 = first_entry();
#pragma unroll
        for (int r = 0; r < K; ++r) L.list[at(e0 + r)] = v[r] ^ desc;
    };
    {
        uint32_t v[K];
        const uint32_t desc = (wave & 1u) ? 0xFFFFFFFFu : 0u, e0 = first_entry();
#pragma unroll
        for (int r = 0; r < K; ++r) v[r] = (e0 + r < n ? L.list[at(e0 + r)] : 0xFFFFFFFFu) ^ desc;
        sort_blocked<K>(v);
        store_run(v, desc);
    }
#pragma unroll
    for (uint32_t m = 2; m <= (uint32_t)kLargeWaves; m <<= 1) {   // runs of m * kRun entries
        __syncthreads();
        for (uint32_t j = tid; j < kRun; j += kLargeThreads) {
            uint32_t x[kLargeWaves];
#pragma unroll
            for (uint32_t c = 0; c < (uint32_t)kLargeWaves; ++c) x[c] = L.list[at(c * kRun + j)];
#pragma unroll
            for (uint32_t st = m / 2; st >= 1; st >>= 1)
#pragma unroll
                for (uint32_t c = 0; c < (uint32_t)kLargeWaves; ++c) {
                    if (c & st) continue;
                    const uint32_t p = x[c], q = x[c + st];
                    const uint32_t lo = p < q ? p : q, hi = p < q ? q : p;
                    x[c] = (c & m) ? hi : lo;
                    x[c + st] = (c & m) ? lo : hi;
                }
#pragma unroll
            for (uint32_t c = 0; c < (uint32_t)kLargeWaves; ++c) L.list[at(c * kRun + j)] = x[c];
        }
        __syncthreads();
        uint32_t v[K];
        const uint32_t desc = m < (uint32_t)kLargeWaves && (wave & m) ? 0xFFFFFFFFu : 0u;
        const uint32_t e0 = first_entry();
#pragma unroll
        for (int r = 0; r < K; ++r) v[r] = L.list[at(e0 + r)] ^ desc;
        merge_steps<K>(v, (int)kRun);
        store_run(v, desc);
    }
    __syncthreads();

    uint32_t key[K];
#pragma unroll
    for (int r = 0; r < K; ++r) {
        // (at most four searches in flight: more would not fit the registers)
        if (r % 4 == 0) asm volatile("" ::: "memory");
        const uint32_t i = (uint32_t)r * kLargeThreads + tid;
        key[r] = 0u;
        const uint32_t loc = L.list[at(i)];
        if (i < n && (i == 0u || L.list[at(i - 1u)] != loc)) {
            const uint32_t w = loc & kWindowMask;
            const uint32_t lim = loc - w + min(w + sws, 1u << kWindowBits);
            uint32_t end = 0;      // entries below lim (lim is at most the padding key)
#pragma unroll
            for (uint32_t step = P / 2; step > 0; step >>= 1)
                if (L.list[at(end + step - 1u)] < lim) end += step;
            if (L.list[at(end)] < lim) end += 1u;
            key[r] = ((end - i) << 16) | (0xFFFFu - i);
        }
    }
    uint32_t nsel = 0;
    const uint32_t top_m = MC_COLD(top_m);
    TopStop decided{MC_COLD(out_top) != nullptr, MC_COLD(min_hits), MC_COLD(hit_diff)};
    for (uint32_t m = 0; m < top_m; ++m) {
        uint32_t best = 0;
#pragma unroll
        for (int r = 0; r < K; ++r) best = key[r] > best ? key[r] : best;
        best = wave_max_u32(best);
        __syncthreads();
        if (lane == 0) L.red[wave] = best;
        __syncthreads();
        best = L.red[lane & (kLargeWaves - 1)];
        best = wave_max_u32(best);
        if (best == 0u) break;
        const uint32_t loc = uniform(L.list[at(0xFFFFu - (best & 0xFFFFu))]);
        if (tid == 0) {
            L.sel_t[m] = loc >> kWindowBits;
            L.sel_s[m] = best >> 16;
            L.sel_b[m] = loc & kWindowMask;
        }
        nsel = m + 1;
        if (decided(m, best >> 16)) break;
        uint32_t t = tid;               // the entries' places are not kept across the rounds
        asm volatile("" : "+v"(t));
#pragma unroll
        for (int r = 0; r < K; ++r)
            if (L.list[at((uint32_t)r * kLargeThreads + t)] >> kWindowBits == loc >> kWindowBits)
                key[r] = 0u;
    }
    if (wave == 0) {
        wave_lds_sync();
        write_result(a, rec, label_of(a, L, nsel), L, nsel);
    }
}

template <int KPL, bool C>
__device__ void classify_large_record(const QueryArgs& a, uint32_t rec, LargeLds& L,
                                      const Threshold& th, WaveStats& ws) {
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = uniform(tid >> 6);
    typedef const __attribute__((address_space(4))) uint64_t ConstU64;
    ConstU64* const off = (ConstU64*)(uintptr_t)a.offsets;
    uint64_t o0, o1, o2;
    if (a.paired) {
        o0 = off[2ull * rec]; o1 = off[2ull * rec + 1]; o2 = off[2ull * rec + 2];
    } else {
        o0 = off[rec]; o1 = off[rec + 1ull]; o2 = o1;
    }
    RecordSpan rs;
    (void)record_span(a, o0, o1, o2, rs);   // queued records are well formed and span < 2^31 bytes
    const uint32_t len = rs.len[0] + rs.len[1];
    const uint32_t F = rs.len[0] > 0 && rs.len[1] > 0 && a.insert_size > len ? a.insert_size : len;
    const uint32_t sws = fragment_sws32(a, F);
    const uint32_t nw0 = mate_windows32(a, rs.len[0]), nwt = nw0 + mate_windows32(a, rs.len[1]);
    const uint32_t per_round = (kLargeFeats / a.s) & ~1u;   // windows whose sketches fit the buffer
    __syncthreads();                       // the previous record is done with the LDS
    if (tid == 0) L.nlist = 0;
    for (uint32_t p0 = 0; p0 < nwt; p0 += per_round) {
        if (tid == 0) L.nfeat = 0;
        __syncthreads();
        const uint32_t p1 = min(nwt, p0 + per_round);
        LargeWave& W = L.wv[wave];
        for (uint32_t p = p0 + 2u * wave; p < p1; p += 2u * kLargeWaves) {
            WinRef wr[2];
            for (int h = 0; h < 2; ++h) wr[h] = window_ref(a, p + h, p1, nw0, rs.r0, rs.len);
            wave_lds_sync();
            uint32_t dirtyA, dirtyB;
            stage_pair(W.stage, rs.base, wr[0], wr[1], (int)lane, dirtyA, dirtyB);
            wave_lds_sync();
            const Word *const WA = W.stage, *const WB = W.stage + kStageWords;
            PairSketch ps = sketch_pair<KPL>(WA, wr[0].x0, wr[0].nk, WB, wr[1].x0, wr[1].nk, a.k,
                                             a.s, th, W.scratch, dirtyA, dirtyB, lane);
            sketch_rest<KPL>(ps, WA, wr[0].x0, wr[0].nk, WB, wr[1].x0, wr[1].nk, a.k, a.s, W.sk,
                             W.sk + 64, W.scratch);
            const uint32_t nA = ps.nA, nB = ps.nB;
            wave_lds_sync();
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(&L.nfeat, nA + nB);
            base = uniform(base);
            if (lane < nA) L.feats[base + lane] = W.sk[lane];
            if (lane < nB) L.feats[base + nA + lane] = W.sk[64 + lane];
        }
        __syncthreads();
        const uint32_t nf = uniform(L.nfeat);
        if (nf) {
            if (wave == 0) ws.features += nf;
            if constexpr (C) large_lookup_cond(a, L, nf, wave, ws.probes);
            else if (nf <= 8u * kLargeWaves) large_lookup<true>(a, L, nf, wave, ws.probes);
            else large_lookup<false>(a, L, nf, wave, ws.probes);
        }
        __syncthreads();
        if (uniform(L.nlist) > kListLarge) break;
    }
    __syncthreads();
    const uint32_t n = uniform(L.nlist);
    if (n > kListLarge) {                  // queued for the HBM-list path (ids from n_records on)
        if (tid == 0) {
            const uint32_t qi = atomicAdd(&MC_COLD(counters)[kQHuge], 1u);
            a.queue[a.n_records + qi] = rec;
            __threadfence();
            atomicAdd(&MC_COLD(counters)[kQHugeReady], 1u);
            __threadfence();
            ws.passed_on += 1;
        }
        return;
    }
    if (wave == 0) ws.locations += n;
    if (n <= 2 * kLargeThreads) large_rank<2>(a, L, rec, n, sws);
    else if (n <= 4 * kLargeThreads) large_rank<4>(a, L, rec, n, sws);
    else if (n <= 8 * kLargeThreads) large_rank<8>(a, L, rec, n, sws);
    else if (n <= 16 * kLargeThreads) large_rank<16>(a, L, rec, n, sws);
    else large_rank<32>(a, L, rec, n, sws);
}

// ------------------------------------------------------ HBM-list path -----
// Records whose candidate list outgrew the large-list pass: one workgroup a
// record, the lists in a region of the workspace's huge scratch. The steps
// are those of the other passes (Sec. 4.2, Sec. 5.3-5.6) without a sort: the
// window count of each distinct location is accumulated in a hash table in
// HBM (Q4-Q6), the score of the range of `sws` windows starting at each
// distinct location sums the counts of its windows looked up in that table,
// and each target keeps its best range with a 64-bit atomic maximum of
// score << 32 | ~location (highest score, then smallest start window, as the
// sorted passes' keys). Top-m and the label follow as in the other passes.
struct HugeRegion {
    uint32_t* feats;                 // kHugeFeats
    uint32_t* locs;                  // kHugeLocs
    uint32_t* keys;                  // kHugeSlots, kNone = empty
    uint32_t* cnt;                   // kHugeSlots
    unsigned long long* best;        // kHugeTargets, zero between records
    uint32_t* tlist;                 // kHugeTargets
};

__device__ __forceinline__ HugeRegion huge_region(unsigned char* base, uint32_t r) {
    unsigned char* p = base + (uint64_t)r * kHugeRegionBytes;
    HugeRegion h;
    h.best = reinterpret_cast<unsigned long long*>(p);
    p += 8ull * kHugeTargets;
    h.feats = reinterpret_cast<uint32_t*>(p);
    h.locs = h.feats + kHugeFeats;
    h.keys = h.locs + kHugeLocs;
    h.cnt = h.keys + kHugeSlots;
    h.tlist = h.cnt + kHugeSlots;
    return h;
}

// Values written by atomics of this workgroup are read at device scope (not
// from a possibly stale vector L1 line).
__device__ __forceinline__ uint32_t ld_dev(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long ld_dev64(const unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t loc_slot(uint32_t loc, uint32_t mask) {
    return (loc * 0x9E3779B1u >> 7) & mask;
}

// Window count of `loc` (0 if absent).
__device__ __forceinline__ uint32_t huge_count(const HugeRegion& h, uint32_t mask, uint32_t loc) {
    for (uint32_t i = loc_slot(loc, mask);; i = (i + 1) & mask) {
        const uint32_t k = ld_dev(&h.keys[i]);
        if (k == loc) return ld_dev(&h.cnt[i]);
        if (k == kNone) return 0u;
    }
}

constexpr int kHugeThreads = kLargeThreads, kHugeWaves = kLargeWaves;

struct HugeLds {
    Word stage[kHugeWaves][2 * kStageWords];
    uint32_t scratch[kHugeWaves][kWave];
    uint32_t sk[kHugeWaves][2 * 64];
    unsigned long long red[kHugeWaves];
    uint32_t nfeat, nloc, ntarget, overflow;
    uint32_t sel_t[kMaxTopM], sel_s[kMaxTopM], sel_b[kMaxTopM];
};

// Workgroup maximum of one u64 per thread.
__device__ __forceinline__ unsigned long long block_max_u64(unsigned long long v,
                                                            unsigned long long* red) {
    v = wave_max_u64(v);
    const uint32_t w = threadIdx.x >> 6;
    __syncthreads();
    if (lane_id() == 0) red[w] = v;
    __syncthreads();
    unsigned long long m = red[0];
    for (int i = 1; i < kHugeWaves; ++i) m = red[i] > m ? red[i] : m;
    return m;
}

template <int KPL, bool C>
__device__ void classify_huge_record(const QueryArgs& a, uint32_t rec, const HugeRegion& h,
                                     HugeLds& L, const Threshold& th) {
    const uint32_t tid = threadIdx.x, lane = (uint32_t)lane_id(), wave = tid >> 6;
    uint64_t o0, o1, o2;
    if (a.paired) {
        o0 = a.offsets[2ull * rec]; o1 = a.offsets[2ull * rec + 1]; o2 = a.offsets[2ull * rec + 2];
    } else {
        o0 = a.offsets[rec]; o1 = a.offsets[rec + 1ull]; o2 = o1;
    }
    // a record of 2^31 bytes or more never comes here (the fast pass counts
    // it as too long); were it to, it is counted the same way (overflow)
    RecordSpan rs;
    const bool spans = record_span(a, o0, o1, o2, rs);
    if (!spans) rs = RecordSpan{0, 0u, {0u, 0u}};
    uint64_t F = (uint64_t)rs.len[0] + rs.len[1];
    if (rs.len[0] > 0 && rs.len[1] > 0 && a.insert_size > F) F = a.insert_size;
    const uint32_t sws = fragment_sws(a, F);
    uint32_t nws[2];
    for (int sg = 0; sg < 2; ++sg)
        nws[sg] = mate_windows32(a, rs.len[sg]);
    const uint32_t nwt = nws[0] + nws[1];
    if (tid == 0) {
        L.nfeat = 0;
        L.nloc = 0;
        L.ntarget = 0;
        L.overflow = spans ? 0u : 1u;
    }
    __syncthreads();

    // sketches of all windows: each wave takes pairs of windows
    for (uint32_t p = 2u * wave; p < nwt; p += 2u * kHugeWaves) {
        WinRef wr[2];
        for (int x = 0; x < 2; ++x) wr[x] = window_ref(a, p + x, nwt, nws[0], rs.r0, rs.len);
        wave_lds_sync();
        uint32_t dirtyA, dirtyB;
        stage_pair(L.stage[wave], rs.base, wr[0], wr[1], (int)lane, dirtyA, dirtyB);
        wave_lds_sync();
        const Word *const WA = L.stage[wave], *const WB = L.stage[wave] + kStageWords;
        PairSketch ps = sketch_pair<KPL>(WA, wr[0].x0, wr[0].nk, WB, wr[1].x0, wr[1].nk, a.k, a.s,
                                         th, L.scratch[wave], dirtyA, dirtyB, lane);
        sketch_rest<KPL>(ps, WA, wr[0].x0, wr[0].nk, WB, wr[1].x0, wr[1].nk, a.k, a.s, L.sk[wave],
                         L.sk[wave] + 64, L.scratch[wave]);
        const uint32_t nA = ps.nA, nB = ps.nB;
        wave_lds_sync();
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(&L.nfeat, nA + nB);
        base = uniform(shfl_idx(base, 0));
        if (base + nA + nB > kHugeFeats) {
            if (lane == 0) L.overflow = 1;
        } else {
            if (lane < nA) h.feats[base + lane] = L.sk[wave][lane];
            if (lane < nB) h.feats[base + nA + lane] = L.sk[wave][64 + lane];
        }
        wave_lds_sync();
    }
    __syncthreads();
    const uint32_t nf = min(L.nfeat, kHugeFeats);

    // lookups: 8-lane groups walk one feature's chain each, appending its
    // locations with an LDS counter
    const u64x2* slot2 = reinterpret_cast<const u64x2*>(a.table) + (lane & 7u);
    const uint32_t nb = (uint32_t)a.nb;
    uint32_t probes = 0;
    if constexpr (C) {   // condensed layout: one entry a feature
        const uint4* ent = reinterpret_cast<const uint4*>(a.table) + (lane & 7u);
        for (uint32_t fi = tid >> 3; fi < nf && !L.overflow; fi += kHugeThreads / 8) {
            const uint32_t f = h.feats[fi];
            uint32_t b = (uint32_t)home_bucket(f, a.nb);
            for (;;) {
                const uint4 e = ent[(uint64_t)b * kCondEntries];
                probes += (lane & 7u) == 0 ? 1u : 0u;
                const bool mine = e.x == f && e.y != 0u;
                if (mine) {
                    const uint32_t pos = atomicAdd(&L.nloc, e.y);
                    if (pos + e.y > kHugeLocs) {
                        L.overflow = 1;
                    } else if (e.y <= kCondInline) {
                        h.locs[pos] = e.z;
                        if (e.y == 2u) h.locs[pos + 1] = e.w;
                    } else {
                        const uint64_t off = ((uint64_t)e.w << 32) | e.z;
                        for (uint32_t k = 0; k < e.y; ++k) h.locs[pos + k] = a.cval[off + k];
                    }
                }
                const uint64_t found = ballot(mine);
                const uint32_t last = (lane & ~7u) | 7u;
                const bool full = shfl_idx(e.y != 0u ? 1u : 0u, (int)last) != 0u;
                if (((found >> (lane & ~7u)) & 0xFFull) != 0 || !full) break;
                b = b + 1u == nb ? 0u : b + 1u;
            }
        }
    } else
    for (uint32_t fi = tid >> 3; fi < nf && !L.overflow; fi += kHugeThreads / 8) {
        const uint32_t f = h.feats[fi];
        uint32_t b = (uint32_t)home_bucket(f, a.nb);
        for (;;) {
            const u64x2 sl = slot2[(uint64_t)b * (kSlots / 2)];
            probes += (lane & 7u) == 0 ? 1u : 0u;
            const unsigned long long e[2] = {sl.x, sl.y};
            for (int x = 0; x < 2; ++x) {
                if ((uint32_t)(e[x] >> 32) == f && (uint32_t)e[x] < kTombLoc) {
                    const uint32_t pos = atomicAdd(&L.nloc, 1u);
                    if (pos < kHugeLocs) h.locs[pos] = (uint32_t)e[x];
                    else L.overflow = 1;
                }
            }
            // the group's last lane holds the bucket's last slot: full bucket
            // -> the chain goes on
            const uint32_t last = (lane & ~7u) | 7u;
            const bool full = shfl_idx(sl.y != kEmpty ? 1u : 0u, (int)last) != 0u;
            if (!full) break;
            b = b + 1u == nb ? 0u : b + 1u;
        }
    }
    __syncthreads();
    const uint32_t n = L.nloc;
    if (L.overflow) {
        if (tid == 0) {
            atomicAdd(&a.counters[kQTooLong], 1u);
            a.out_labels[rec] = kNone;
        }
        if (a.out_top && tid < a.top_m) {
            uint32_t* o = a.out_top + ((uint64_t)rec * a.top_m + tid) * 3;
            o[0] = kNone; o[1] = 0u; o[2] = 0u;
        }
        __syncthreads();
        return;
    }

    // window counts: hash table of 2^m >= 2n slots, cleared first
    uint32_t P = 64;
    while (P < 2 * n) P <<= 1;
    const uint32_t mask = P - 1;
    for (uint32_t i = tid; i < P; i += kHugeThreads) {
        h.keys[i] = kNone;
        h.cnt[i] = 0u;
    }
    __syncthreads();
    for (uint32_t i = tid; i < n; i += kHugeThreads) {
        const uint32_t loc = h.locs[i];
        for (uint32_t j = loc_slot(loc, mask);; j = (j + 1) & mask) {
            const uint32_t old = atomicCAS(&h.keys[j], kNone, loc);
            if (old == kNone || old == loc) {
                atomicAdd(&h.cnt[j], 1u);
                break;
            }
        }
    }
    __syncthreads();
    // score of the range starting at each distinct location; best per target
    for (uint32_t i = tid; i < P; i += kHugeThreads) {
        const uint32_t loc = ld_dev(&h.keys[i]);
        if (loc == kNone) continue;
        const uint32_t t = loc >> kWindowBits, w = loc & kWindowMask;
        uint32_t score = ld_dev(&h.cnt[i]);
        for (uint32_t d = 1; d < sws && w + d <= kWindowMask; ++d)
            score += huge_count(h, mask, (t << kWindowBits) | (w + d));
        const unsigned long long key = ((unsigned long long)score << 32) | (uint32_t)~loc;
        const unsigned long long old = atomicMax(&h.best[t], key);
        if (old == 0ull) h.tlist[atomicAdd(&L.ntarget, 1u)] = t;
    }
    __syncthreads();

    // top m targets by (score desc, target asc), one workgroup maximum a round
    const uint32_t nt = L.ntarget, top_m = a.top_m;
    uint32_t nsel = 0;
    for (uint32_t m = 0; m < top_m; ++m) {
        unsigned long long key = 0;
        for (uint32_t i = tid; i < nt; i += kHugeThreads) {
            const uint32_t t = h.tlist[i];
            bool excluded = false;
            for (uint32_t x = 0; x < m; ++x) excluded |= L.sel_t[x] == t;
            const unsigned long long ku = ((ld_dev64(&h.best[t]) >> 32) << 32) | (0xFFFFFFFFu - t);
            if (!excluded && ku > key) key = ku;
        }
        key = block_max_u64(key, L.red);
        if (key == 0ull) break;
        if (tid == 0) {
            const uint32_t t = 0xFFFFFFFFu - (uint32_t)key;
            const unsigned long long b = ld_dev64(&h.best[t]);
            L.sel_t[m] = t;
            L.sel_s[m] = (uint32_t)(key >> 32);
            L.sel_b[m] = (~(uint32_t)b) & kWindowMask;
        }
        __syncthreads();
        nsel = m + 1;
    }
    // the bests go back to zero for the next record
    for (uint32_t i = tid; i < nt; i += kHugeThreads) h.best[h.tlist[i]] = 0ull;

    if (tid == 0) {
        uint32_t label = kNone;
        if (nsel > 0 && L.sel_s[0] >= a.min_hits) {
            const uint32_t c1 = L.sel_s[0], c2 = nsel > 1 ? L.sel_s[1] : 0u;
            label = a.target_taxon[L.sel_t[0]];
            if (c1 - c2 <= a.hit_diff)
                for (uint32_t x = 1; x < nsel; ++x)
                    if ((uint64_t)L.sel_s[x] + a.hit_diff >= c1)
                        label = lca(label, a.target_taxon[L.sel_t[x]], a.parents, a.depth);
        }
        a.out_labels[rec] = label;
    }
    if (a.out_top && tid < top_m) {
        const bool hit = tid < nsel;
        uint32_t* o = a.out_top + ((uint64_t)rec * top_m + tid) * 3;
        o[0] = hit ? L.sel_t[tid] : kNone;
        o[1] = hit ? L.sel_s[tid] : 0u;
        o[2] = hit ? L.sel_b[tid] : 0u;
    }
    if (a.qstats) {
        unsigned long long* q = a.qstats + ((blockIdx.x * kHugeWaves + wave) % kQsCopies) * kQsStride;
        for (int m = 1; m < kWave; m <<= 1) probes += shfl_xor(probes, m);
        if (lane == 0 && probes) atomicAdd(&q[kQsProbes], (unsigned long long)probes);
        if (tid == 0) {
            atomicAdd(&q[kQsFeatures], (unsigned long long)nf);
            atomicAdd(&q[kQsLocations], (unsigned long long)n);
        }
    }
    __syncthreads();
}

// The next record of the HBM-list queue, or kNone (one thread). Records are
// taken only while every place given out in the queue has been written: a
// workgroup that is queuing one comes here itself once it is done.
__device__ __forceinline__ uint32_t take_huge(const QueryArgs& a) {
    uint32_t* const c = a.counters;
    for (;;) {
        const uint32_t ready =
            __hip_atomic_load(&c[kQHugeReady], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
        if (ready != ld_dev(&c[kQHuge])) return kNone;
        const uint32_t next = ld_dev(&c[kQHugeNext]);
        if (next >= ready) return kNone;
        if (atomicCAS(&c[kQHugeNext], next, next + 1u) == next) {
            __threadfence();
            return ld_dev(&a.queue[a.n_records + next]);
        }
    }
}

// A free region of the huge scratch while records are queued, or kNone (one
// thread; no waiting).
__device__ __forceinline__ uint32_t take_region(const QueryArgs& a) {
    if (ld_dev(&a.counters[kQHugeNext]) >= ld_dev(&a.counters[kQHugeReady])) return kNone;
    const uint32_t n = a.huge_groups ? a.huge_groups : kHugeGroups;
    for (uint32_t r = 0; r < n; ++r)
        if (!(atomicOr(&a.counters[kQHugeBusy], 1u << r) >> r & 1u)) return r;
    return kNone;
}

// Large-list pass and, in the same launch, the HBM-list path: a workgroup that
// is through with its records takes a free region and works on the HBM-list
// queue until it is empty. The last of the workgroups does so when all the
// others have finished, so that no record is left, and then sets the counts
// back for the next classification with this workspace. Nothing waits. As
// launches of their own, the HBM-list path and a clearing of the counts took
// about 3 us each: a call of 200 reads 20.4 -> 13.7 us, of 10,000 reads 25.4 ->
// 21.8 us, a graph of 3,001 records 29.6 -> 22.0 us.
template <int KPL, bool C>
__global__ __launch_bounds__(kLargeThreads) __attribute__((amdgpu_waves_per_eu(4)))
void k_classify_large(QueryArgs a) {
    __shared__ union {
        LargeLds large;
        HugeLds huge;
    } L;
    __shared__ uint32_t s_job;
    const uint32_t n_iter = uniform(a.counters[kQOverflow]);
    if (blockIdx.x >= n_iter) return;
    const Threshold th(a.S, a.s);
    {
        WaveStats ws;
        for (uint32_t it = blockIdx.x; it < n_iter; it += gridDim.x)
            classify_large_record<KPL, C>(a, uniform(a.queue[it]), L.large, th, ws);
        // work of records that go on to the HBM-list path counts in both
        if (lane_id() == 0 && a.qstats) {
            unsigned long long* q =
                a.qstats + ((blockIdx.x * kLargeWaves + (threadIdx.x >> 6)) % kQsCopies) * kQsStride;
            if (ws.features) atomicAdd(&q[kQsFeatures], (unsigned long long)ws.features);
            if (ws.locations) atomicAdd(&q[kQsLocations], (unsigned long long)ws.locations);
            if (ws.probes) atomicAdd(&q[kQsProbes], (unsigned long long)ws.probes);
            if (ws.passed_on) atomicAdd(&q[kQsHuge], (unsigned long long)ws.passed_on);
        }
    }
    const uint32_t groups = min(gridDim.x, n_iter);   // workgroups with records
    for (bool last = false;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_job = take_region(a);
        __syncthreads();
        const uint32_t region = uniform(s_job);
        if (region != kNone) {
            __threadfence();           // the region as its last user left it
            const QueryArgs b = args_at_use<QueryArgs>();   // (not kept from before)
            const HugeRegion h = huge_region(b.huge, region);
            const Threshold th2(b.S, b.s);
            for (;;) {
                __syncthreads();
                if (threadIdx.x == 0) s_job = take_huge(b);
                __syncthreads();
                const uint32_t rec = uniform(s_job);
                if (rec == kNone) break;
                classify_huge_record<KPL, C>(b, rec, h, L.huge, th2);
            }
            __threadfence();
            __syncthreads();
            if (threadIdx.x == 0) {
                atomicAnd(&a.counters[kQHugeBusy], ~(1u << region));
                __threadfence();
            }
        }
        if (last) break;
        __syncthreads();               // s_job has been read by all
        // (what this workgroup queued or gave back is ordered before this by
        // the fences there)
        if (threadIdx.x == 0) {
            s_job = atomicAdd(&a.counters[kQDone], 1u) + 1u == groups ? 1u : 0u;
            if (s_job) __threadfence();
        }
        __syncthreads();
        if (!uniform(s_job)) return;
        last = true;
    }
    if (threadIdx.x < kQTooLong) a.counters[threadIdx.x] = 0u;
}

__global__ __launch_bounds__(256) void k_clear_workspace(uint32_t* counters, unsigned char* huge,
                                                         uint32_t regions,
                                                         unsigned long long* qstats) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i < kNumQueryCounters) counters[i] = 0u;
    if (qstats && i < kQsWords) qstats[i] = 0ull;
    if (i < regions * kHugeTargets)
        reinterpret_cast<unsigned long long*>(huge + (i / kHugeTargets) *
                                              kHugeRegionBytes)[i % kHugeTargets] = 0ull;
}

template <uint32_t LCAP, int WPB, int KPL, bool C>
hipError_t launch_fast_t(const QueryArgs& a, uint32_t max_blocks, int cls, hipStream_t st) {
    uint64_t blocks = ((uint64_t)a.n_records + WPB - 1) / WPB;
    if (blocks > max_blocks) blocks = max_blocks;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL((k_classify<LCAP, WPB, KPL, C>), dim3((unsigned)blocks), dim3(WPB * 64), 0,
                       st, a, cls);
    return hipGetLastError();
}

// Tuned variants exist for windows of at most 128 k-mers (two per lane); other
// window sizes use the default list capacity and workgroup shape.
template <int KPL, bool C>
hipError_t launch_fast_k(const QueryArgs& a, const ClassifyConfig& c, int cls, hipStream_t st) {
    if constexpr (KPL == 2) {
        const uint32_t key = c.list_cap * 16 + c.waves_per_block;
        switch (key) {
            case 256 * 16 + 2: return launch_fast_t<256, 2, KPL, C>(a, c.max_blocks, cls, st);
            case 256 * 16 + 4: return launch_fast_t<256, 4, KPL, C>(a, c.max_blocks, cls, st);
            case 256 * 16 + 8: return launch_fast_t<256, 8, KPL, C>(a, c.max_blocks, cls, st);
            case 512 * 16 + 2: return launch_fast_t<512, 2, KPL, C>(a, c.max_blocks, cls, st);
            case 512 * 16 + 8: return launch_fast_t<512, 8, KPL, C>(a, c.max_blocks, cls, st);
            case 1024 * 16 + 2: return launch_fast_t<1024, 2, KPL, C>(a, c.max_blocks, cls, st);
            case 1024 * 16 + 4: return launch_fast_t<1024, 4, KPL, C>(a, c.max_blocks, cls, st);
            case 1024 * 16 + 8: return launch_fast_t<1024, 8, KPL, C>(a, c.max_blocks, cls, st);
            default: break;
        }
    }
    return launch_fast_t<kListSmall, 4, KPL, C>(a, c.max_blocks, cls, st);
}

template <int KPL>
hipError_t launch_fast_c(const QueryArgs& a, const ClassifyConfig& c, int cls, hipStream_t st) {
    return a.cval ? launch_fast_k<KPL, true>(a, c, cls, st)
                  : launch_fast_k<KPL, false>(a, c, cls, st);
}

hipError_t launch_fast_any(const QueryArgs& a, const ClassifyConfig& c, int cls, hipStream_t st) {
    if (a.n_records == 0) return hipSuccess;
    if (a.S <= 64) return launch_fast_c<1>(a, c, cls, st);
    if (a.S <= 128) return launch_fast_c<2>(a, c, cls, st);
    return launch_fast_c<4>(a, c, cls, st);
}

// Windows of record rec (both mates), as the classification counts them.
__device__ __forceinline__ uint64_t record_windows(const QueryArgs& a, uint32_t rec) {
    uint64_t o0, o1, o2;
    if (a.paired) {
        o0 = a.offsets[2ull * rec]; o1 = a.offsets[2ull * rec + 1]; o2 = a.offsets[2ull * rec + 2];
    } else {
        o0 = a.offsets[rec]; o1 = a.offsets[rec + 1ull]; o2 = o1;
    }
    if (o1 < o0 || o2 < o1) return 0;
    uint64_t nw = 0;
    const uint64_t len[2] = {o1 - o0, o2 - o1};
    for (int sg = 0; sg < 2; ++sg)
        nw += mate_windows(a, len[sg]);
    return nw;
}

__device__ __forceinline__ uint32_t size_class(uint64_t nw, const RouteConfig& r) {
    for (uint32_t c = 0; c + 1 < r.n; ++c)
        if (nw <= r.max_windows[c]) return c;
    return r.n - 1;
}

// Routing, pass 1: records per size class (wave-aggregated counters).
__global__ __launch_bounds__(256) void k_route_count(QueryArgs a, RouteConfig r) {
    uint32_t cnt[kMaxRoutes] = {0, 0, 0, 0};
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n_records;
         i += (uint64_t)gridDim.x * blockDim.x)
        cnt[size_class(record_windows(a, (uint32_t)i), r)] += 1;
    for (uint32_t c = 0; c < r.n; ++c) {
        uint32_t v = cnt[c];
#pragma unroll
        for (int m = 1; m < kWave; m <<= 1) v += shfl_xor(v, m);
        if (lane_id() == 0 && v) atomicAdd(&a.route_meta[c], v);
    }
}

// Routing, pass 2: first ids of the classes (their counts' prefix), cursors.
__global__ void k_route_scan(QueryArgs a, RouteConfig r) {
    if (threadIdx.x != 0) return;
    uint32_t run = 0;
    for (uint32_t c = 0; c < r.n; ++c) {
        a.route_meta[kMaxRoutes + c] = run;
        a.route_meta[2 * kMaxRoutes + c] = run;
        run += a.route_meta[c];
    }
}

// Routing, pass 3: every record's id at its class's cursor.
__global__ __launch_bounds__(256) void k_route_scatter(QueryArgs a, RouteConfig r) {
    const uint64_t step = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x; i0 < a.n_records; i0 += step) {
        const uint64_t i = i0 + threadIdx.x;
        const bool in = i < a.n_records;
        const uint32_t c = in ? size_class(record_windows(a, (uint32_t)i), r) : kMaxRoutes;
        for (uint32_t k = 0; k < r.n; ++k) {
            const uint64_t m = ballot(c == k);
            if (!m) continue;
            uint32_t base = 0;
            if (lane_id() == 0) base = atomicAdd(&a.route_meta[2 * kMaxRoutes + k], popc64(m));
            base = shfl_idx(base, 0);
            if (c == k) a.route_queue[base + rank_below(m)] = (uint32_t)i;
        }
    }
}

// Workgroups of the large-list pass when the number of queued records is not
// known on the host: as many as fit the chip at once (two a CU), at most one a
// record. Without queued records they end at once, alone (10,000 short reads:
// 25.6 us a call with 512 as with 8) and beside other streams, although each
// needs half a CU's LDS for its moment: against 8 workgroups that take a whole
// CU's (and launches of their own for the HBM-list records and the clearing of
// the counts), calls of 200 reads on four streams in turn 12.4 -> 7.0 us a call,
// of 20,000 reads 33 -> 27, of 200 reads beside a stream of 2M-read
// classifications 7.4 -> 5.8 ms at the median (their time there 2.44 -> 1.91 ms).
inline unsigned large_pass_groups(uint32_t n_records) {
    return (unsigned)std::min<uint32_t>(512u, n_records);
}

template <bool C>
void launch_large_c(const QueryArgs& a, uint32_t groups, hipStream_t st) {
    const dim3 grid(groups ? std::min<uint32_t>(groups, 512u) : large_pass_groups(a.n_records));
    if (a.S <= 128)
        hipLaunchKernelGGL((k_classify_large<2, C>), grid, dim3(kLargeThreads), 0, st, a);
    else
        hipLaunchKernelGGL((k_classify_large<4, C>), grid, dim3(kLargeThreads), 0, st, a);
}

}  // namespace

bool classify_config_valid(const ClassifyConfig& c) {
    return (c.list_cap == 256 || c.list_cap == 512 || c.list_cap == 1024) &&
           (c.waves_per_block == 2 || c.waves_per_block == 4 || c.waves_per_block == 8) &&
           c.max_blocks >= 1;
}

hipError_t launch_classify_fast(const QueryArgs& a, const ClassifyConfig& c, hipStream_t st) {
    return launch_fast_any(a, c, -1, st);
}

hipError_t launch_route(const QueryArgs& a, const RouteConfig& r, hipStream_t st) {
    if (a.n_records == 0) return hipSuccess;
    const unsigned grid = (unsigned)std::min<uint64_t>(4096, (a.n_records + 255) / 256);
    hipLaunchKernelGGL(k_route_count, dim3(grid), dim3(256), 0, st, a, r);
    hipLaunchKernelGGL(k_route_scan, dim3(1), dim3(64), 0, st, a, r);
    hipLaunchKernelGGL(k_route_scatter, dim3(grid), dim3(256), 0, st, a, r);
    return hipGetLastError();
}

hipError_t launch_classify_class(const QueryArgs& a, const ClassifyConfig& c, uint32_t cls,
                                 hipStream_t st) {
    return launch_fast_any(a, c, (int)cls, st);
}

hipError_t launch_clear_workspace(uint32_t* counters, unsigned char* huge, uint32_t regions,
                                  unsigned long long* qstats, hipStream_t st) {
    static_assert(kQsWords <= kHugeTargets && kNumQueryCounters <= 256, "covered by one region's threads");
    hipLaunchKernelGGL(k_clear_workspace, dim3(std::max(regions, 1u) * (kHugeTargets / 256)),
                       dim3(256), 0, st, counters, huge, regions, qstats);
    return hipGetLastError();
}

hipError_t launch_classify_large(const QueryArgs& a, hipStream_t st, uint32_t groups) {
    if (a.n_records == 0) return hipSuccess;
    if (a.cval) launch_large_c<true>(a, groups, st);
    else launch_large_c<false>(a, groups, st);
    return hipGetLastError();
}

}  // namespace mc
