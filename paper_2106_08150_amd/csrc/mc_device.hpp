// Device building blocks of the minhash classifier (gfx950, wave64).
//
// Everything here runs inside the library's kernels: 2-bit encoding of ASCII
// text staged in LDS, canonical k-mer extraction by funnel shifts, h1, a
// register bitonic sort across the 64 lanes of a wave, bottom-s selection with
// ballots, and the bucketed open-addressing table (16 x 64-bit slots = one
// 128-byte line per bucket).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mc_internal.hpp"

namespace mc {

constexpr uint32_t kWindowBits = 18;
constexpr uint32_t kWindowMask = (1u << kWindowBits) - 1;
constexpr uint32_t kNone = 0xFFFFFFFFu;        // unclassified label / unused hit
constexpr uint64_t kEmpty = ~0ull;             // empty table slot
// Location field of a capped-away entry (tombstone). Real locations stay below
// 0xFFFC0000 (targets < 16383), and a tombstone never equals an empty slot,
// not even for feature 0xFFFFFFFF.
constexpr uint32_t kTombLoc = 0xFFFFFFFEu;

// A slot holding a stored pair (neither empty nor a tombstone).
__device__ __forceinline__ bool live_entry(uint64_t e) { return (uint32_t)e < kTombLoc; }

constexpr int kWave = 64;

// ------------------------------------------------------------------ lanes --
__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

// Lanes whose predicate holds (the builtin takes the compare result directly;
// going through an int would materialise it in a VGPR first).
__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// Whether the calling lane's bit of a wave-uniform mask is set (the mask is
// used as the lane predicate as it is, without a per-lane shift and test).
// Combining the ballots of single compares with scalar ANDs, then taking
// lanes from the result, avoids the select-and-compare a ballot of a compound
// predicate compiles to.
__device__ __forceinline__ bool lane_in(uint64_t mask) {
    return __builtin_amdgcn_inverse_ballot_w64(mask);
}

// Number of set bits of `mask` in lanes below the calling lane, plus `base`.
__device__ __forceinline__ uint32_t rank_below(uint64_t mask, uint32_t base = 0u) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, base));
}

__device__ __forceinline__ uint32_t popc64(uint64_t m) { return (uint32_t)__popcll(m); }

__device__ __forceinline__ uint32_t shfl_idx(uint32_t v, int src) {
    return (uint32_t)__builtin_amdgcn_ds_bpermute(src << 2, (int)v);
}

__device__ __forceinline__ uint32_t shfl_xor(uint32_t v, int m) {
    return shfl_idx(v, lane_id() ^ m);
}

// Value of lane (lane ^ M), M a power of two < 64: DPP quad permutes for 1
// and 2, a row rotate for 8 (rotating a 16-lane row by 8 is xor 8),
// ds_swizzle's xor mode for 4 and 16 (within 32-lane halves), and a
// backwards permute for 32.
template <int M>
__device__ __forceinline__ uint32_t xor_lanes(uint32_t v) {
    if constexpr (M == 1) {
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);
    } else if constexpr (M == 2) {
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);
    } else if constexpr (M == 8) {
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, true);
    } else if constexpr (M == 4 || M == 16) {
        return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (M << 10) | 0x1F);
    } else {
        return shfl_idx(v, lane_id() ^ M);
    }
}

__device__ __forceinline__ uint32_t xor_lanes_c(uint32_t v, int m) {
    switch (m) {
        case 1: return xor_lanes<1>(v);
        case 2: return xor_lanes<2>(v);
        case 4: return xor_lanes<4>(v);
        case 8: return xor_lanes<8>(v);
        case 16: return xor_lanes<16>(v);
        default: return xor_lanes<32>(v);
    }
}

__device__ __forceinline__ uint32_t uniform(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
    uint32_t lo = uniform((uint32_t)v), hi = uniform((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
        uint32_t lo = shfl_xor((uint32_t)v, m), hi = shfl_xor((uint32_t)(v >> 32), m);
        uint64_t o = ((uint64_t)hi << 32) | lo;
        v = o > v ? o : v;
    }
    return v;
}

// Maximum over the wave: row rotations by 1, 2, 4 and 8 (DPP) reduce each
// 16-lane row, then the four row results are combined in scalar registers.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    uint32_t o;
    o = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x121, 0xF, 0xF, false); v = v > o ? v : o;
    o = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x122, 0xF, 0xF, false); v = v > o ? v : o;
    o = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x124, 0xF, 0xF, false); v = v > o ? v : o;
    o = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, false); v = v > o ? v : o;
    uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)v, 0);
    uint32_t r1 = (uint32_t)__builtin_amdgcn_readlane((int)v, 16);
    uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)v, 32);
    uint32_t r3 = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
    r0 = r0 > r1 ? r0 : r1;
    r2 = r2 > r3 ? r2 : r3;
    return r0 > r2 ? r0 : r2;
}

// Orders LDS accesses of different lanes of one wave (LDS executes a wave's
// operations in order; this keeps the compiler from moving them across).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------- mixers --
// h1: MurmurHash3's 32-bit finalizer, a bijection on 32-bit words.
__device__ __forceinline__ uint32_t h1(uint32_t x) {
    x ^= x >> 16;
    x *= 0x85ebca6bu;
    x ^= x >> 13;
    x *= 0xc2b2ae35u;
    x ^= x >> 16;
    return x;
}

// Slot hash h2 (Sec. 4.1 uses a second hash so that the skewed sketch values
// spread over the table): the two-round xorshift-multiply mixer published as
// "lowbias32" (C. Wellons, hash prospector), a bijection unrelated to h1.
__device__ __forceinline__ uint32_t h2(uint32_t f) {
    f ^= f >> 16;
    f *= 0x7feb352du;
    f ^= f >> 15;
    f *= 0x846ca68bu;
    f ^= f >> 16;
    return f;
}

// Home bucket: floor(h2 * nb / 2^32) (tables have fewer than 2^32 buckets).
__device__ __forceinline__ uint64_t home_bucket(uint32_t f, uint64_t nb) {
    return __umulhi(h2(f), (uint32_t)nb);
}

__device__ __forceinline__ uint64_t next_bucket(uint64_t b, uint64_t nb) {
    return b + 1 == nb ? 0 : b + 1;
}

// ------------------------------------------------------------- encoding --
// 16 bases packed as 2-bit codes (first base in bits 31..30) plus an invalid
// mask with the same layout (0b11 in the two bits of every invalid base), and
// the complements of the same bases in the opposite order (base j of the word
// in bits 2j+1..2j), from which reverse complements are read by a funnel
// shift. A=0 C=1 G=2 T=3, case-insensitive; every other byte is invalid.
struct Word {
    uint32_t code;
    uint32_t mask;
    uint32_t rc;
    uint32_t pad;
};

// The complement word of a code word: every 2-bit group complemented and the
// groups' order reversed (bit reversal, then the two bits of each group
// swapped back).
__device__ __forceinline__ uint32_t rc_word(uint32_t code) {
    const uint32_t r = __builtin_bitreverse32(~code);
    return ((r >> 1) & 0x55555555u) | ((r & 0x55555555u) << 1);
}

// Four 2-bit fields held in bits 8i..8i+1 (i = byte) packed below acc's bits,
// byte 0's field first (bits 7..6): a dot product with the fields' weights, one
// instruction for four (with the candidate lanes of a pair of windows as a scalar
// mask: 650 -> 635 vector instructions a 150-base read, 187 -> 171 a pair of
// windows of the build).
__device__ __forceinline__ uint32_t pack_fields(uint32_t v, uint32_t acc = 0u) {
    return __builtin_amdgcn_udot4(v, 0x01041040u, acc, false);
}
// The same in the opposite order (byte 0's field in bits 1..0).
__device__ __forceinline__ uint32_t pack_fields_back(uint32_t v) {
    return __builtin_amdgcn_udot4(v, 0x40100401u, 0u, false);
}
// 0b11 for each byte of v that is 1, in the order of pack_fields.
__device__ __forceinline__ uint32_t pack_flags(uint32_t v, uint32_t acc = 0u) {
    return __builtin_amdgcn_udot4(v, 0x030C30C0u, acc, false);
}

// Codes of 4 ASCII bytes x (byte 0 = first base). Bits 1..2 of a letter give
// its code, ((x >> 1) ^ (x >> 2)) & 3 maps A/a C/c G/g T/t to 0 1 2 3; a byte
// is a base iff it equals "acgt"[code] once lower-cased (v_perm looks the
// letter up). c: the 4 codes, one per byte (those of non-bases are
// arbitrary). Returns 0x80 in each byte that is not a base.
__device__ __forceinline__ uint32_t codes4(uint32_t x, uint32_t& c) {
    c = ((x >> 1) ^ (x >> 2)) & 0x03030303u;
    const uint32_t expect = __builtin_amdgcn_perm(0u, 0x74676361u, c);
    const uint32_t diff = (x | 0x20202020u) ^ expect;           // zero byte: a base
    const uint32_t t = (diff & 0x7F7F7F7Fu) + 0x7F7F7F7Fu;
    return (t | diff) & 0x80808080u;
}

// Encode 4 ASCII bytes x; ok: 0x80 in each byte that lies inside the
// sequence. c8: the 4 codes (those of invalid bases are arbitrary), first base
// in bits 7..6; m8: 0b11 in the positions of invalid bases; r8: their
// complements, first base in bits 1..0. Returns whether a byte inside the
// sequence is not a base.
__device__ __forceinline__ bool encode4(uint32_t x, uint32_t ok, uint32_t& c8, uint32_t& m8,
                                        uint32_t& r8) {
    uint32_t c;
    const uint32_t bad = codes4(x, c) & ok;                      // 0x80 per non-base inside
    r8 = pack_fields_back(c ^ 0x03030303u);
    const uint32_t inv = bad | (~ok & 0x80808080u);               // 0x80 per invalid base
    c8 = pack_fields(c);
    m8 = pack_flags(inv >> 7);
    return bad != 0u;
}

// 0x80 in the bytes [lo, hi) of a dword (0 <= lo < hi <= 4).
__device__ __forceinline__ uint32_t inside_bytes(uint32_t lo, uint32_t hi) {
    return (0x80808080u << (8 * lo)) & (0x80808080u >> (8 * (4 - hi)));
}

// Word covering absolute bytes [a, a+16), a 16-byte aligned. Bytes outside
// [vlo, vhi) count as invalid. A word that overlaps [vlo, vhi) is read with
// one 16-byte load: an aligned 16-byte block never crosses a page, so it lies
// in the same mapped page as the valid byte it contains. A word that does not
// overlap is not read at all. `bad` is set if a byte inside [vlo, vhi) is not
// a base. Words wholly inside [vlo, vhi) (nearly all) need no per-byte range
// test, and words without an invalid base no mask packing.
__device__ __forceinline__ Word load_word(uintptr_t a, uintptr_t vlo, uintptr_t vhi, bool& bad) {
    if (a + 16 <= vlo || a >= vhi) return Word{0u, 0xFFFFFFFFu, 0u, 0u};
    // the address is global memory; saying so gives a global (not flat) load
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = *reinterpret_cast<const __attribute__((address_space(1))) u32x4*>(a);
    uint32_t c[4], inv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) inv[i] = codes4(i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w, c[i]);
    if (a < vlo || a + 16 > vhi) {
        // bytes [lo, hi) of the word lie inside [vlo, vhi)
        const uint32_t lo = vlo > a ? (uint32_t)(vlo - a) : 0u;
        const uint32_t hi = vhi - a < 16 ? (uint32_t)(vhi - a) : 16u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t dlo = lo > 4u * i ? min(lo - 4u * i, 4u) : 0u;
            const uint32_t dhi = hi > 4u * i ? min(hi - 4u * i, 4u) : 0u;
            const uint32_t ok = dlo < dhi ? inside_bytes(dlo, dhi) : 0u;
            bad |= (inv[i] & ok) != 0u;
            inv[i] = (inv[i] & ok) | (~ok & 0x80808080u);
        }
    } else {
        bad |= (inv[0] | inv[1] | inv[2] | inv[3]) != 0u;
    }
    Word w;
    w.code = 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) w.code = pack_fields(c[i], w.code << 8);
    w.mask = 0u;
    if ((inv[0] | inv[1] | inv[2] | inv[3]) != 0u) {
        uint32_t m = 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) m = pack_flags(inv[i] >> 7, m << 8);
        w.mask = m;
    }
    w.rc = rc_word(w.code);
    w.pad = 0u;
    return w;
}

// Stage one dword (4 bases) of a word covering [A0, ...): dword d of word
// d >> 2 goes to byte 3 - (d & 3) of that word's code and mask (first base in
// the top byte) and to byte d & 3 of its complement word. Positions are
// 32-bit offsets from `base` (16-byte aligned), A0 a multiple of 16. Bytes
// outside [vlo, vhi) count as invalid; a dword that does not overlap them is
// not read. Aligned 4-byte loads never cross a page. Returns whether a byte
// inside [vlo, vhi) is not a base.
__device__ __forceinline__ uint32_t stage_dword(Word* W, uintptr_t base, uint32_t A0, uint32_t d,
                                                uint32_t vlo, uint32_t vhi) {
    const uint32_t a = A0 + 4u * d;
    // every lane loads (no branch): a dword outside [vlo, vhi) reads the
    // nearest dword that overlaps it (vlo < vhi) and marks all its bytes
    // invalid; its codes are then arbitrary
    const uint32_t ac = min(max(a, vlo & ~3u), (vhi - 1u) & ~3u);
    const uint32_t x = *reinterpret_cast<const __attribute__((address_space(1))) uint32_t*>(base + ac);
    const uint32_t lo = vlo > a ? min(vlo - a, 4u) : 0u;
    const uint32_t hi = vhi > a ? min(vhi - a, 4u) : 0u;
    uint32_t c8, m8, r8;
    const bool bad = encode4(x, lo < hi ? inside_bytes(lo, hi) : 0u, c8, m8, r8);
    uint8_t* w = reinterpret_cast<uint8_t*>(W + (d >> 2));
    w[3 - (d & 3u)] = (uint8_t)c8;
    w[7 - (d & 3u)] = (uint8_t)m8;
    w[8 + (d & 3u)] = (uint8_t)r8;
    return bad ? 1u : 0u;
}

// Canonical k-mer (k <= 16) starting o bases into word pair (a, b), both
// strands by a funnel shift: the forward k-mer is the top 2k bits of
// (a:b) << 2o, the reverse complement (its first base the complement of the
// k-mer's last) comes from the complement words, kmask = 4^k - 1. lo is b for
// o > 0 and a itself for o = 0: the forward funnel shift by 32 - 2o (taken mod
// 32) then needs no select between its two cases. Without kCheck the caller
// knows every base of the k-mer is valid; with it, returns false if one is
// not.
template <bool kCheck>
__device__ __forceinline__ bool kmer_of(const Word& a, const Word& lo, const Word& b, uint32_t o,
                                        uint32_t k, uint32_t kmask, uint32_t& canon) {
    const uint32_t top = __builtin_amdgcn_alignbit(a.code, lo.code, 32u - 2u * o);
    const uint32_t fwd = top >> (32 - 2 * k);
    bool bad = false;
    if constexpr (kCheck) {
        const uint32_t mtop = __builtin_amdgcn_alignbit(a.mask, lo.mask, 32u - 2u * o);
        bad = (mtop >> (32 - 2 * k)) != 0u;
    }
    const uint32_t r = __builtin_amdgcn_alignbit(b.rc, a.rc, 2u * o) & kmask;
    canon = fwd < r ? fwd : r;
    return !bad;
}

__device__ __forceinline__ uint32_t kmer_mask(uint32_t k) {
    return k >= 16 ? 0xFFFFFFFFu : (1u << (2 * k)) - 1u;
}

// Canonical k-mer starting x bases after the first staged word (k <= 16).
// Returns false if any of its bases is invalid.
__device__ __forceinline__ bool kmer_at(const Word* W, uint32_t x, uint32_t k, uint32_t& canon) {
    const uint32_t q = x >> 4, o = x & 15u;
    return kmer_of<true>(W[q], W[q + (o != 0u)], W[q + 1], o, k, kmer_mask(k), canon);
}

// ------------------------------------------------------- bitonic in regs --
// Ascending networks on keys held one a lane (element = lane) and K a lane
// (element = r * 64 + lane). A phase of `size` first exchanges each element with
// its mirror in the block (e ^ (size - 1)), then at strides size / 4 .. 1; the
// lower partner always keeps the smaller key, so no step has a direction. A
// phase over several registers has none to mirror across cheaply: there the
// odd blocks are sorted descending, as ascending blocks of complemented keys.
//
// A step is a lane exchange and one median of three: the median of two keys
// and 0 is the smaller, that of two keys and all ones the larger. Minimum,
// maximum and a select by a mask of constants took one vector and two scalar
// instructions more a step: 10M reads of 150 bases on 4 Gbp 13.5 -> 12.55 ms
// (692 -> 650 vector and 619 -> 526 scalar instructions a read), the sketches
// of 4 Gbp 7.1 -> 6.4 ms.

// The lane id as a value of this place: what is computed from it is not held
// in registers across the enclosing loops.
__device__ __forceinline__ uint32_t lane_here() {
    uint32_t lane = (uint32_t)lane_id();
    asm volatile("" : "+v"(lane));
    return lane;
}

// All ones in the lanes with bit m (a power of two) of the lane id set.
__device__ __forceinline__ uint32_t high_lanes(uint32_t lane, int m) {
    return 0u - (lane / (uint32_t)m & 1u);
}

// The smaller of two keys where high is 0, the larger where it is all ones.
__device__ __forceinline__ uint32_t keep_of(uint32_t v, uint32_t o, uint32_t high) {
    return max(min(v, o), min(max(v, o), high));
}

// Value of lane (lane ^ (size - 1)): DPP permutes up to the 16-lane row,
// ds_swizzle for 32 and a backwards permute for the wave.
__device__ __forceinline__ uint32_t mirror_lanes(uint32_t v, int size) {
    switch (size) {
        case 2: return xor_lanes<1>(v);
        case 4: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x1B, 0xF, 0xF, true);
        case 8: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);
        case 16: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true);
        case 32: return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (0x1F << 10) | 0x1F);
        default: return shfl_idx(v, 63 - lane_id());
    }
}

// Compile-time check of the scheme described above (mirror first steps,
// complemented odd blocks) on a model of its own over a few key patterns: every
// sequence ends ascending. The model shares no code with the device networks;
// those are tested on the device, for every number of keys a lane.
template <int KPL>
constexpr bool networks_sort(int top, uint32_t seed) {
    constexpr int N = 64 * KPL;
    uint32_t v[N] = {};
    for (int e = 0; e < N; ++e) v[e] = ((uint32_t)e * 2654435761u + seed) % 97u;   // duplicates too
    for (int size = 2; size <= top; size <<= 1) {
        const bool flips = size >= 64 && size < N;         // odd blocks descend
        for (int e = 0; e < N; ++e)
            if (flips && (e & size)) v[e] = ~v[e];
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            const bool mirror = stride == size >> 1 && size <= 64;
            uint32_t nv[N] = {};
            for (int e = 0; e < N; ++e) {
                const uint32_t o = v[mirror ? e ^ (size - 1) : e ^ stride];
                const bool low = (e & stride) == 0;
                nv[e] = low ? (v[e] < o ? v[e] : o) : (v[e] < o ? o : v[e]);
            }
            for (int e = 0; e < N; ++e) v[e] = nv[e];
        }
        for (int e = 0; e < N; ++e)
            if (flips && (e & size)) v[e] = ~v[e];
    }
    for (int e = 1; e < N; ++e)
        if (e % top != 0 && v[e - 1] > v[e]) return false;
    return true;
}
static_assert(networks_sort<1>(64, 0) && networks_sort<1>(64, 5), "64-key network");
static_assert(networks_sort<2>(128, 1) && networks_sort<4>(256, 3), "128- and 256-key networks");
static_assert(networks_sort<1>(32, 0) && networks_sort<1>(32, 7), "two 32-key networks");

// Ascending sort of 64*KPL keys held KPL per lane; element index r*64 + lane.
template <int KPL>
__device__ __forceinline__ void wave_sort(uint32_t (&v)[KPL]) {
    constexpr int N = kWave * KPL;
    const uint32_t lane = lane_here();
#pragma unroll
    for (int size = 2; size <= N; size <<= 1) {
#pragma unroll
        for (int r = 0; r < KPL; ++r)
            if (size >= kWave && size < N && (r * kWave & size)) v[r] = ~v[r];
#pragma unroll
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            if (stride >= kWave) {
                const int rs = stride / kWave;
#pragma unroll
                for (int r = 0; r < KPL; ++r) {
                    const int p = r ^ rs;
                    if (p > r) {
                        const uint32_t x = v[r], y = v[p];
                        v[r] = min(x, y);
                        v[p] = max(x, y);
                    }
                }
            } else {
#pragma unroll
                for (int r = 0; r < KPL; ++r) {
                    const uint32_t o = stride == size >> 1 && size <= kWave
                                           ? mirror_lanes(v[r], size)
                                           : xor_lanes_c(v[r], stride);
                    v[r] = keep_of(v[r], o, high_lanes(lane, stride));
                }
            }
        }
#pragma unroll
        for (int r = 0; r < KPL; ++r)
            if (size >= kWave && size < N && (r * kWave & size)) v[r] = ~v[r];
    }
}

// After wave_sort: write the s smallest distinct keys (0xFFFFFFFF excluded)
// to sk[0..] in ascending order and return their number; `distinct` receives
// the number of distinct keys below 0xFFFFFFFF. If a valid k-mer hashed to
// 0xFFFFFFFF (has_top) and fewer than s smaller distinct values exist, that
// value is appended as the last element.
template <int KPL>
__device__ __forceinline__ uint32_t select_distinct(const uint32_t (&v)[KPL], bool has_top,
                                                    uint32_t s, uint32_t* sk,
                                                    uint32_t& distinct) {
    const int lane = lane_id();
    uint32_t base = 0, prev_last = 0;
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        uint32_t up = shfl_idx(v[r], lane > 0 ? lane - 1 : 0);
        bool has_prev = lane > 0 || r > 0;
        uint32_t prev = lane > 0 ? up : prev_last;
        bool first = v[r] != 0xFFFFFFFFu && (!has_prev || v[r] != prev);
        uint64_t bal = ballot(first);
        uint32_t rank = base + rank_below(bal);
        if (first && rank < s) sk[rank] = v[r];
        base += popc64(bal);
        prev_last = (uint32_t)__builtin_amdgcn_readlane((int)v[r], kWave - 1);
    }
    distinct = base;
    uint32_t n = base < s ? base : s;
    if (has_top && base < s) {
        if (lane == 0) sk[base] = 0xFFFFFFFFu;
        n = base + 1;
    }
    return n;
}

// Hash threshold below which about `expect` of the nk hashes of a window are
// expected (uniform hashes). Any value is correct: callers verify that enough
// distinct candidates fell below it and otherwise take every hash.
__device__ __forceinline__ uint32_t hash_threshold(float expect, uint32_t nk) {
    const float t = expect * 4294967296.0f / (float)nk;
    return t >= 4294967040.0f ? 0xFFFFFFFFu : (uint32_t)t;
}

// Lanes below m (any m), computed in scalar registers.
__device__ __forceinline__ uint64_t lanes_below(uint32_t m) {
    return m >= 64u ? ~0ull : (1ull << m) - 1ull;
}

// Candidates of a window in sketch_pair: hashes below a threshold that about
// 1.5 s of its nk hashes pass (hash_threshold), computed once for the full window
// of S k-mers, divided out only for shorter windows; a window of at most 32
// k-mers takes them all. A number c of candidates decides the window if it is at
// least s and at most 32, as one comparison: c - lo <= span (never for s > 32).
struct Threshold {
    uint32_t S, tS, lo, span;
    __device__ __forceinline__ Threshold(uint32_t S_, uint32_t s)
        : S(S_),
          tS(uniform(S_ <= 32u ? 0xFFFFFFFFu : hash_threshold(1.5f * (float)s, S_))),
          lo(s <= 32u ? s : 1u << 16),
          span(s <= 32u ? 32u - s : 0u) {}
    // lanes of register r that hold a k-mer of a full window
    __device__ __forceinline__ uint64_t full_lanes(int r) const {
        return lanes_below(max(S, (uint32_t)(r * kWave)) - (uint32_t)(r * kWave));
    }
    __device__ __forceinline__ uint32_t of(uint32_t nk, uint32_t s) const {
        if (nk == S) return tS;
        if (nk <= 32u) return 0xFFFFFFFFu;
        return uniform(hash_threshold(1.5f * (float)s, nk));
    }
};

// h1 of the canonical k-mers of one window whose nk k-mer starts begin x0
// bases after the first staged word: key[r] belongs to k-mer r*64 + lane and is
// 0xFFFFFFFF for an invalid k-mer or past nk. Returns whether some valid k-mer
// hashed to 0xFFFFFFFF (that value then still counts as a distinct feature).
template <int KPL>
__device__ __forceinline__ bool window_keys(const Word* W, uint32_t x0, uint32_t nk, uint32_t k,
                                            uint32_t (&key)[KPL]) {
    const int lane = lane_id();
    bool top = false;
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        const uint32_t i = (uint32_t)(r * kWave + lane);
        key[r] = 0xFFFFFFFFu;
        uint32_t c;
        if (i < nk && kmer_at(W, x0 + i, k, c)) {
            key[r] = h1(c);
            top |= key[r] == 0xFFFFFFFFu;
        }
    }
    return ballot(top) != 0;
}

// The same hashes without a per-lane test: h[r] of the k-mer starting x0 +
// r*64 + lane, on every lane (lanes past nk read staged words beyond the window:
// W must hold 4 * KPL + 2 words from the window's first word on), and in valid[r]
// the lanes whose k-mer holds no invalid base. kCheck = false: the caller knows
// the window holds none. K-mer r*64 + lane starts 4r words after k-mer lane, at
// the same offset in its word. Registers whose k-mers all lie past nk are not
// hashed.
template <int KPL, bool kCheck>
__device__ __forceinline__ void window_hashes(const Word* W, uint32_t x0, uint32_t nk, uint32_t k,
                                              uint32_t (&h)[KPL], uint64_t (&valid)[KPL]) {
    const uint32_t x = x0 + (uint32_t)lane_id();
    const Word* Wq = W + (x >> 4);
    const uint32_t o = x & 15u;
    const Word* Wl = Wq + (o != 0u);
    const uint32_t kmask = kmer_mask(k);
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        h[r] = 0u;
        valid[r] = ~0ull;
        if (r > 0 && nk <= (uint32_t)(r * kWave)) continue;
        uint32_t c;
        const bool ok = kmer_of<kCheck>(Wq[4 * r], Wl[4 * r], Wq[4 * r + 1], o, k, kmask, c);
        h[r] = h1(c);
        if (kCheck) valid[r] = ballot(ok);
    }
}

// The s smallest distinct keys of one window (its nk keys as left by
// window_keys) into sk[0..), ascending; returns their number. scratch: 64
// words of LDS owned by the wave.
//
// For windows of more than 64 k-mers the wave first keeps only hashes below a
// threshold chosen so that about 1.75 s of them are expected; if at least s
// distinct values lie below it, the s smallest of the window are exactly the s
// smallest of those candidates, which fit one per lane. Otherwise (fewer than
// s distinct candidates, or more than 64) it sorts every hash of the window.
template <int KPL>
__device__ __forceinline__ uint32_t sketch_keys(uint32_t (&key)[KPL], uint32_t nk, bool has_top,
                                                uint32_t s, uint32_t* sk, uint32_t* scratch) {
    const int lane = lane_id();
    uint32_t distinct;
    if constexpr (KPL >= 2) {
        if (nk > (uint32_t)kWave) {
            const uint32_t T = hash_threshold(1.75f * (float)s, nk);
            uint64_t bal[KPL];
            uint32_t c = 0;
#pragma unroll
            for (int r = 0; r < KPL; ++r) {
                bal[r] = ballot(key[r] < T);
                c += popc64(bal[r]);
            }
            if (c >= s && c <= (uint32_t)kWave) {
                uint32_t base = 0;
#pragma unroll
                for (int r = 0; r < KPL; ++r) {
                    if (key[r] < T) scratch[base + rank_below(bal[r])] = key[r];
                    base += popc64(bal[r]);
                }
                wave_lds_sync();
                uint32_t v[1] = {(uint32_t)lane < c ? scratch[lane] : 0xFFFFFFFFu};
                wave_lds_sync();
                wave_sort<1>(v);
                uint32_t n = select_distinct<1>(v, false, s, sk, distinct);
                if (distinct >= s) return n;
            }
        }
        if (nk <= (uint32_t)kWave) {   // one key per lane: a 64-wide sort suffices
            uint32_t v[1] = {key[0]};
            wave_sort<1>(v);
            return select_distinct<1>(v, has_top, s, sk, distinct);
        }
    }
    wave_sort<KPL>(key);
    return select_distinct<KPL>(key, has_top, s, sk, distinct);
}

// Sketch of one window (B2-B4, Q2).
template <int KPL>
__device__ __forceinline__ uint32_t sketch_window(const Word* W, uint32_t x0, uint32_t nk,
                                                  uint32_t k, uint32_t s, uint32_t* sk,
                                                  uint32_t* scratch) {
    uint32_t key[KPL];
    const bool top = window_keys<KPL>(W, x0, nk, k, key);
    return sketch_keys<KPL>(key, nk, top, s, sk, scratch);
}

// Out-of-line copy for rare paths, so that the hot loops stay small in the
// instruction cache. Its pointers are LDS pointers (address space 3), so that
// the out-of-line code still uses LDS instructions rather than flat ones.
#define MC_LDS __attribute__((address_space(3)))
template <int KPL>
__device__ __attribute__((noinline)) uint32_t sketch_window_lds(const MC_LDS Word* W, uint32_t x0,
                                                                uint32_t nk, uint32_t k,
                                                                uint32_t s, MC_LDS uint32_t* sk,
                                                                MC_LDS uint32_t* scratch) {
    return sketch_window<KPL>((const Word*)W, x0, nk, k, s, (uint32_t*)sk, (uint32_t*)scratch);
}

template <int KPL>
__device__ __forceinline__ uint32_t sketch_window_rare(const Word* W, uint32_t x0, uint32_t nk,
                                                       uint32_t k, uint32_t s, uint32_t* sk,
                                                       uint32_t* scratch) {
    return sketch_window_lds<KPL>((const MC_LDS Word*)W, x0, nk, k, s, (MC_LDS uint32_t*)sk,
                                  (MC_LDS uint32_t*)scratch);
}

// Ascending sort of each 32-lane half of the wave (one key per lane).
__device__ __forceinline__ void wave_sort_halves(uint32_t& v, uint32_t lane) {
#pragma unroll
    for (int size = 2; size <= 32; size <<= 1) {
        v = keep_of(v, mirror_lanes(v, size), high_lanes(lane, size >> 1));
#pragma unroll
        for (int stride = size >> 2; stride > 0; stride >>= 1)
            v = keep_of(v, xor_lanes_c(v, stride), high_lanes(lane, stride));
    }
}

// Candidates of one window for a 32-entry half of scratch (see Threshold). If at
// least s distinct values lie below the threshold, the s smallest of the window
// are exactly the s smallest of the candidates. About one window in twenty has
// fewer than s or more than 32 candidates: its threshold is moved by a quarter
// and the hashes, still in registers, are compared again (a window that stays
// undecided is redone alone with every hash, which costs as much as two pairs).
// Returns the number of candidates written, plus kAllHashes if they are all of
// the window's hashes below 0xFFFFFFFF; kUndecided (none written) otherwise.
// most receives the lane's largest hash (of k-mers that may not count).
//
// A full window without an invalid base, the common case, has code of its own
// without the tests for either. The wave-uniform decisions are integers, not
// booleans: booleans that live across blocks become 64-bit lane masks, several
// scalar instructions each, and scalar issue bounds the kernels as much as
// vector issue does.
constexpr uint32_t kAllHashes = 64u, kUndecided = 128u;
template <int KPL>
__device__ __forceinline__ uint32_t below_threshold(const uint32_t (&h)[KPL],
                                                    const uint64_t (&valid)[KPL], uint32_t T,
                                                    uint64_t (&bal)[KPL]) {
    uint32_t c = 0;
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        bal[r] = valid[r] & ballot(h[r] < T);
        c += popc64(bal[r]);
    }
    return c;
}
template <int KPL>
__device__ __forceinline__ uint32_t half_candidates(const Word* W, uint32_t x0, uint32_t nk,
                                                    uint32_t k, uint32_t s, const Threshold& th,
                                                    uint32_t dirty, uint32_t* half,
                                                    uint32_t& most) {
    uint32_t h[KPL];
    uint64_t valid[KPL], bal[KPL];
    uint32_t c, T, state;
    if (__builtin_expect(nk == th.S && dirty == 0u, 1)) {
        window_hashes<KPL, false>(W, x0, KPL * kWave, k, h, valid);
#pragma unroll
        for (int r = 0; r < KPL; ++r) valid[r] = th.full_lanes(r);
        T = th.tS;
        c = below_threshold<KPL>(h, valid, T, bal);
    } else {
        if (dirty) window_hashes<KPL, true>(W, x0, nk, k, h, valid);
        else window_hashes<KPL, false>(W, x0, nk, k, h, valid);
#pragma unroll
        for (int r = 0; r < KPL; ++r)
            valid[r] &= nk > (uint32_t)(r * kWave) ? lanes_below(nk - (uint32_t)(r * kWave)) : 0ull;
        T = th.of(nk, s);
        c = below_threshold<KPL>(h, valid, T, bal);
    }
#pragma unroll
    for (int r = 0; r < KPL; ++r) most = max(most, h[r]);
    state = c;
    if (__builtin_expect(c - th.lo > th.span, 0)) {
        for (uint32_t tries = 0; T != 0xFFFFFFFFu && c - th.lo > th.span; ++tries) {
            if (tries == 3u || s > 32u) return kUndecided;
            T = c > 32u ? T - (T >> 2) : T + min(T >> 2, ~T);
            c = below_threshold<KPL>(h, valid, T, bal);
        }
        if (c > 32u) return kUndecided;
        state = T == 0xFFFFFFFFu ? c + kAllHashes : c;
    }
    uint32_t base = 0;
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        if (lane_in(bal[r])) half[rank_below(bal[r], base)] = h[r];
        base += popc64(bal[r]);
    }
    return state;
}

// Sketches of two windows A and B (either may be empty, nk = 0) at once: the
// candidates of A fill lanes 0..31 and those of B lanes 32..63, one 32-wide
// sort orders both halves, and one ballot ranks the distinct values of both.
// The lanes in `sel` hold the s smallest distinct candidates v of each window
// (A's below lane 32), each the rank-th of its window; dA and dB are the numbers
// of distinct candidates. When full(s), these are the two sketches; else
// sketch_rest completes them. scratch: 64 words of LDS owned by the wave. dirtyA
// / dirtyB (wave-uniform): the window may hold an invalid base. sort_lane: the
// lane id, from which the sort's lane constants are made.
struct PairSketch {
    uint32_t v, rank;
    uint64_t sel;
    uint32_t dA, dB;
    uint32_t stateA, stateB; // as half_candidates
    uint32_t nA, nB;         // set by sketch_rest
    __device__ __forceinline__ bool full(uint32_t s) const { return min(dA, dB) >= s; }
};
template <int KPL>
__device__ __forceinline__ PairSketch sketch_pair(const Word* WA, uint32_t xA, uint32_t nkA,
                                                  const Word* WB, uint32_t xB, uint32_t nkB,
                                                  uint32_t k, uint32_t s, const Threshold& th,
                                                  uint32_t* scratch, uint32_t dirtyA,
                                                  uint32_t dirtyB, uint32_t sort_lane) {
    const int lane = lane_id();
    PairSketch p;
    uint32_t most = 0;
    p.stateA = half_candidates<KPL>(WA, xA, nkA, k, s, th, dirtyA, scratch, most);
    p.stateB = half_candidates<KPL>(WB, xB, nkB, k, s, th, dirtyB, scratch + 32, most);
    // a k-mer that hashes to 0xFFFFFFFF (on a lane that may not even count)
    // leaves both windows undecided: no candidate stands for it
    if (__builtin_expect(ballot(most == 0xFFFFFFFFu) != 0ull, 0)) p.stateA = p.stateB = kUndecided;
    wave_lds_sync();
    const uint32_t word = scratch[lane];
    const uint32_t inA = (uint32_t)((1ull << (p.stateA & 63u)) - 1ull);   // at most 32 each
    const uint32_t inB = (uint32_t)((1ull << (p.stateB & 63u)) - 1ull);
    uint32_t v = lane_in((uint64_t)inB << 32 | inA) ? word : 0xFFFFFFFFu;
    wave_lds_sync();
    wave_sort_halves(v, sort_lane);
    // previous lane's key (whole-wave shift right by one lane)
    const uint32_t prev = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x138, 0xF, 0xF, false);
    // first of its value in its half: not the padding key, and lane 0 of the
    // half or unlike the lane before
    const uint64_t firsts =
        ballot(v != 0xFFFFFFFFu) & (ballot(v != prev) | 0x0000000100000001ull);
    p.dA = popc64(firsts & 0xFFFFFFFFull);
    p.dB = popc64(firsts >> 32);
    p.v = v;
    p.rank = rank_below(firsts) - (lane < 32 ? 0u : p.dA);
    p.sel = firsts & ballot(p.rank < s);
    return p;
}

// The pair's sketches into LDS: skA[0..nA) and skB[0..nB), ascending. A window
// that its candidates do not decide is done alone from its staged words (which
// must still be in place).
template <int KPL>
__device__ __forceinline__ void sketch_rest(PairSketch& p, const Word* WA, uint32_t xA,
                                            uint32_t nkA, const Word* WB, uint32_t xB,
                                            uint32_t nkB, uint32_t k, uint32_t s, uint32_t* skA,
                                            uint32_t* skB, uint32_t* scratch) {
    p.nA = min(p.dA, s);
    p.nB = min(p.dB, s);
    if (lane_in(p.sel)) (lane_id() < 32 ? skA : skB)[p.rank] = p.v;
    if (__builtin_expect(p.full(s), 1)) return;
    if (p.stateA == kUndecided || (p.dA < s && nkA > 32u && !(p.stateA & kAllHashes))) {
        wave_lds_sync();
        p.nA = uniform(sketch_window_rare<KPL>(WA, xA, nkA, k, s, skA, scratch));
    }
    if (p.stateB == kUndecided || (p.dB < s && nkB > 32u && !(p.stateB & kAllHashes))) {
        wave_lds_sync();
        p.nB = uniform(sketch_window_rare<KPL>(WB, xB, nkB, k, s, skB, scratch));
    }
    // the counts are wave-uniform; saying so keeps the callers' loops scalar
    p.nA = uniform(p.nA);
    p.nB = uniform(p.nB);
}

// Stage the bytes [lo, hi) into words relative to A0 = lo & ~15, one word per
// participating thread (tid in [0, nthreads)); bytes outside [vlo, vhi) are
// invalid. Returns whether a word of this thread holds a byte inside
// [vlo, vhi) that is not a base; callers synchronise before reading W.
__device__ __forceinline__ bool stage_words(Word* W, uintptr_t lo, uintptr_t hi, uintptr_t vlo,
                                            uintptr_t vhi, int tid, int nthreads) {
    uintptr_t A0 = lo & ~(uintptr_t)15;
    int nw = (int)((hi - A0 + 15) / 16) + 1;
    bool bad = false;
    for (int q = tid; q < nw; q += nthreads)
        W[q] = load_word(A0 + 16 * (uintptr_t)q, vlo, vhi, bad);
    return bad;
}

// ------------------------------------------------------------ LCA / taxa --
__device__ __forceinline__ uint32_t lca(uint32_t a, uint32_t b, const uint32_t* parent,
                                        const uint32_t* depth) {
    uint32_t da = depth[a], db = depth[b];
    while (da > db) { a = parent[a]; --da; }
    while (db > da) { b = parent[b]; --db; }
    while (a != b) { a = parent[a]; b = parent[b]; }
    return a;
}

}  // namespace mc
