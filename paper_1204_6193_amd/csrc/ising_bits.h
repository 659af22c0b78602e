// Strips of a lattice held as one bit per spin in registers: the update all
// sweeps of a call go through when a strip's rows divide over its threads.
//
// What bounds an on-chip sweep is VALU issue (small lattices: a pass's chain of
// barrier, LDS and tagged words).  With spins as bytes in LDS a site update
// cost 24 (LCG32) to 36 (Philox4x32-10) lane-instructions, of which the draw
// is only 3 to 13: the rest unpacked bytes, counted neighbours and chose a
// threshold per site.  Here a thread owns one column
// of units (4 sites wide, XS1024W 8) in every VB-th row of the strip, and
// keeps the colour-c sites of all its rows as the bits of one word W_c.  Per
// draw and threshold only a compare and an add-with-carry remain, which
// shifts the outcome into a word; neighbours, counts, decisions and energies
// are then bit operations on 32 sites at a time (about one instruction per
// site).
//
// Layout: thread t holds column t % (L/NB) of rows vb + i VB (vb = t / (L/NB),
// i = 0, 1, ...: its slots), i.e. slot i is unit t + i nt of the strip with
// nt = VB L/NB, so states load and store coalesced and an XS1024W instance
// (16 consecutive units) stays on one 16-lane row when nt is a multiple of
// 16.  Bit G i + j of W_c (G = NB/2) is the j-th colour-c site of slot i; a
// set bit is a down spin.  With p = (c + y) & 1 those sites are x0 + p + 2 j,
// so of a site's four neighbours (all of the other colour)
//   one is bit j of the same slot of the thread's own W_{1-c},
//   one is bit j - 1 (p = 0) or j + 1 (p = 1) of that slot, or the last bit
//       of the thread to the left or the first of the one to the right,
//   and those above and below are bit j of the rows y -+ 1: the same slot of
//       thread t -+ L/NB, or, across the ends of the VB rows, a word shifted
//       by one slot.
// Threads hand their words to each other through LDS (two words per
// thread), one barrier per pass.
//
// Strips exchange their top and bottom rows as tagged words (put_word), G + G
// bits per thread gathered from 16 / G neighbouring lanes into one word.
//
// Draws need no neighbour, so a pass's are made before the tagged words of
// the pass before are waited for, and hide that latency.  A word is read
// by every wave that needs it before the barrier of the pass that uses it, and
// its slot rewritten two passes later, by a strip that has read the words its
// readers stored after that barrier.
#pragma once

#include "ising_memory.h"

namespace rngx {

// Appends [v < t4] to a4 and [v < t8] to a8 (as their lowest bits) for
// v = y, then v = x.  A compare leaves its outcome as a lane mask in SGPRs
// and the add a + a + carry shifts it in: two instructions per bit, where a
// select, shift and or take three.  The four compares come first because a
// mask may be read as a carry no sooner than two instructions after it is
// written, and the block is opaque to the pass that would insert the waits.
__device__ __forceinline__ void push2(uint32_t &a4, uint32_t &a8, uint32_t y, uint32_t x, uint32_t t4, uint32_t t8) {
    uint64_t m0, m1, m2, m3;
    asm("v_cmp_gt_u32_e64 %2, %8, %6\n\t"
        "v_cmp_gt_u32_e64 %3, %9, %6\n\t"
        "v_cmp_gt_u32_e64 %4, %8, %7\n\t"
        "v_cmp_gt_u32_e64 %5, %9, %7\n\t"
        "v_addc_co_u32_e64 %0, %2, %0, %0, %2\n\t"
        "v_addc_co_u32_e64 %1, %3, %1, %1, %3\n\t"
        "v_addc_co_u32_e64 %0, %4, %0, %0, %4\n\t"
        "v_addc_co_u32_e64 %1, %5, %1, %1, %5"
        : "+v"(a4), "+v"(a8), "=&s"(m0), "=&s"(m1), "=&s"(m2), "=&s"(m3)
        : "v"(y), "v"(x), "s"(t4), "s"(t8));
}
// The same for one value.
__device__ __forceinline__ void push1(uint32_t &a4, uint32_t &a8, uint32_t x, uint32_t t4, uint32_t t8) {
    uint64_t m0, m1;
    asm("v_cmp_gt_u32_e64 %2, %5, %4\n\t"
        "v_cmp_gt_u32_e64 %3, %6, %4\n\t"
        "s_nop 0\n\t"
        "v_addc_co_u32_e64 %0, %2, %0, %0, %2\n\t"
        "v_addc_co_u32_e64 %1, %3, %1, %1, %3"
        : "+v"(a4), "+v"(a8), "=&s"(m0), "=&s"(m1)
        : "v"(x), "s"(t4), "s"(t8));
}

// Sum of v over the wave, in its last lane.
__device__ __forceinline__ int wave_sum_last(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31
    return v;
}

// Bits 0, 2, 4, ... of x as bits 0, 1, 2, ..., and back.
__device__ __forceinline__ uint32_t gather_even(uint32_t x) {
    x &= 0x55555555u;
    x = (x | (x >> 1)) & 0x33333333u;
    x = (x | (x >> 2)) & 0x0F0F0F0Fu;
    x = (x | (x >> 4)) & 0x00FF00FFu;
    return (x | (x >> 8)) & 0xFFFFu;
}
__device__ __forceinline__ uint32_t spread_even(uint32_t x) {
    x = (x | (x << 8)) & 0x00FF00FFu;
    x = (x | (x << 4)) & 0x0F0F0F0Fu;
    x = (x | (x << 2)) & 0x33333333u;
    return (x | (x << 1)) & 0x55555555u;
}

// (m & a) | (~m & b)
__device__ __forceinline__ uint32_t bfi(uint32_t m, uint32_t a, uint32_t b) { return (m & a) | (~m & b); }

// Tagged words per strip and slot: 16 / G threads share one.
template <int NB>
__host__ __device__ constexpr uint32_t bits_halo_words(uint32_t nt) { return (nt + 32 / NB - 1) / (32 / NB); }

template <class Unit> struct IsPhiloxKey : std::false_type {};
template <int ROUNDS> struct IsPhiloxKey<PhiloxKeyUnitR<ROUNDS>> : std::true_type {};

// All sweeps (one at least) of strip r (R rows at row r R0) by the calling workgroup.
// GANG: several strips (else the strip is the lattice).  TILE: a tile of a
// lattice in memory (k_ising_tiles), which wraps on itself instead of asking
// its neighbours and keeps only what lies farther from its edges than the
// passes it makes.
template <class Unit, int SPT, bool MH, bool GANG, bool TILE = false>
__device__ __forceinline__ void bits_body(const StripArgs &a, uint32_t r, uint32_t *lds) {
    constexpr int NB = Unit::kNB, G = NB / 2;
    constexpr uint32_t kGroup = 16 / G;  // lanes that share a halo word
    constexpr uint32_t GM = (1u << G) - 1;
    constexpr uint32_t kFirst = G == 2 ? 0x55555555u : 0x11111111u;  // first bit of every slot
    constexpr uint32_t kLast = kFirst << (G - 1);
    constexpr uint32_t kEvenSlots = G == 2 ? 0x33333333u : 0x0F0F0F0Fu;
    static_assert(SPT * G <= 32, "a colour's sites are one word");
    const uint32_t t = threadIdx.x;
    const uint32_t L = a.L, R = a.R, VB = a.VB, nwg = GANG ? a.nwg : 1, upr = (TILE ? a.tile_w : L) / NB, nt = VB * upr;
    const uint32_t nth = (nt + 63) / 64 * 64;  // threads of the waves that hold units
    if (t >= nth) {  // whole waves of a wider workgroup (a batch's): the barriers below, nothing else
        for (uint64_t n = 2 * a.n_sweeps; n; --n) __syncthreads();
        __syncthreads();
        if (a.trace && a.n_sweeps > 0) __syncthreads();
        return;
    }
    const uint64_t row0 = TILE ? a.y0 : static_cast<uint64_t>(r) * a.R0;
    const bool active = TILE || t < nt;
    const uint32_t vb = active ? t / upr : 0, col = active ? t - vb * upr : 0;
    // of this thread (a tile fills its workgroup, so all its loads can be in flight at once)
    const uint32_t rows = TILE ? SPT : active && vb < R ? (R - 1 - vb) / VB + 1 : 0;
    // the sites the energies count: the thread's own, of a tile those it keeps
    uint32_t own = rows * G >= 32 ? ~0u : (1u << (rows * G)) - 1;
    uint32_t counted = rows;
    if constexpr (TILE) {
        own = counted = 0;
        if (col - a.in_x < a.n_x)
            for (uint32_t i = 0; i < rows; ++i)
                if (vb + i * VB - a.in_y < a.n_y) {
                    own |= GM << (G * i);
                    ++counted;
                }
    }
    const uint32_t row_units = L / NB;
    // lattice row of slot i, and a thread's unit in that row
    auto row_of = [&](uint32_t vb_, int i) -> uint64_t {
        const uint64_t y = row0 + vb_ + static_cast<uint64_t>(i) * VB;
        return TILE && y >= L ? y - L : y;
    };
    auto unit_of = [&](uint32_t col_) -> uint32_t {
        if constexpr (!TILE) return col_;
        const uint32_t c = a.x0 / NB + col_;
        return c >= row_units ? c - row_units : c;
    };
    const uint32_t ucol = unit_of(col);
    // slots whose row is even
    const uint32_t flat = VB & 1 ? kEvenSlots : ~0u;
    const uint32_t even = (row0 + vb) & 1 ? ~flat : flat;
    // neighbours' words, and the shift of a word that crosses the VB rows
    const uint32_t at_l = !active ? t : col == 0 ? t + upr - 1 : t - 1;
    const uint32_t at_r = !active ? t : col == upr - 1 ? t - col : t + 1;
    const bool first_vb = vb == 0, last_vb = vb == VB - 1;
    const uint32_t at_u = !active ? t : first_vb ? t + (VB - 1) * upr : t - upr;
    const uint32_t at_d = !active ? t : last_vb ? col : t + upr;
    const uint32_t sh_u = first_vb ? G : 0, sh_d = last_vb ? G : 0;
    // the strip's top row is slot 0 of vb = 0, its bottom row slot sb / G of vb = (R - 1) mod VB
    const uint32_t sb = (R - 1) / VB * G;
    const bool top = active && first_vb, bottom = active && vb == (R - 1) % VB;
    const uint32_t top_m = top ? GM : 0, bot_m = bottom ? GM << sb : 0;

    uint32_t *X = lds;  // W_c of thread t at X[kMaxT c + t]
    constexpr uint32_t kMaxT = kBitsMaxThreads;
    uint32_t *zero_word = lds + 2 * kMaxT;
    int *e_ring = reinterpret_cast<int *>(lds + 2 * kMaxT + 4);
    constexpr bool kWeylLds = std::is_same<Unit, XorwowStripUnit>::value;
    uint32_t *weyl0 = lds + kBitsLds / 4 + t * (SPT + 1);  // XORWOW: Weyl words of the thread's slots at the start

    // spins and states
    uint32_t W[2] = {0, 0};
    auto colours = [&](uint32_t w, uint32_t (&b)[2]) {  // 4 sites as bytes -> bits (0, 2) and (1, 3)
        const uint32_t x = (w >> 1) & 0x01010101u, e = x & 0x00010001u, o = (x >> 8) & 0x00010001u;
        b[0] = (e | (e >> 15)) & 3;
        b[1] = (o | (o >> 15)) & 3;
    };
    auto row_bits = [&](uint64_t y, uint32_t (&b)[2]) {  // colour bits of the thread's unit in row y
        const uint32_t *p = reinterpret_cast<const uint32_t *>(a.spins + y * L + static_cast<uint64_t>(ucol) * NB);
        uint32_t q[2];
        colours(p[0], q);
        if constexpr (NB == 8) {
            uint32_t q2[2];
            colours(p[1], q2);
            q[0] |= q2[0] << 2;
            q[1] |= q2[1] << 2;
        }
        b[0] = y & 1 ? q[1] : q[0];  // colour 0: x + y even
        b[1] = y & 1 ? q[0] : q[1];
    };
    const uint64_t ubase = row0 * upr;
    constexpr bool kHasCst = std::is_same<Unit, PhiloxUnit>::value || std::is_same<Unit, PhiloxUnit7>::value ||
                             std::is_same<Unit, XsUnit>::value;  // image parts that no update changes
    constexpr bool kSub = !std::is_void<typename SubWord<Unit>::type>::value;
    LcgMap<std::conditional_t<kSub, typename SubWord<Unit>::type, uint32_t>> map{};
    if constexpr (kSub) map = Unit::map(TILE ? a.cst : a.st, a.S);
    Unit u[SPT];
#pragma unroll
    for (int i = 0; i < SPT; ++i) {
        u[i] = Unit{};
        if (static_cast<uint32_t>(i) < rows) {
            const uint64_t k = TILE ? row_of(vb, i) * row_units + ucol : ubase + t + static_cast<uint64_t>(i) * nt;
            if constexpr (kWeylLds) u[i].load(a.st, a.S, k, weyl0 + i);
            else if constexpr (TILE && kHasCst) u[i].load(a.st, a.cst, a.S, k);
            else if constexpr (TILE && IsPhiloxKey<Unit>::value) u[i].load(a.cst, a.S, k);
            else u[i].load(a.st, a.S, k);
            uint32_t b[2];
            row_bits(row_of(vb, i), b);
            W[0] |= b[0] << (G * i);
            W[1] |= b[1] << (G * i);
        }
    }
    // The byte offsets of the tagged words of slot 0: those that hold the
    // neighbours' boundary rows (bits from cut_u / cut_d on) and this thread's.
    uint32_t halo_u = 0, halo_d = 0, at_hu = 0, at_hd = 0, at_own = 0, cut_u = 0, cut_d = 0;
    bool publish = false;
    uint8_t *const halo = reinterpret_cast<uint8_t *>(a.halo);
    const uint32_t hw = bits_halo_words<NB>(nt), slot_bytes = 8 * nwg * hw;  // at most 8 nwg L / 2
    if constexpr (GANG) {
        const uint32_t up = (r + nwg - 1) % nwg, dn = (r + 1) % nwg;
        const uint32_t R_up = up == nwg - 1 ? L - (nwg - 1) * a.R0 : a.R0;
        const uint32_t k = (R_up - 1) % VB * upr + col;  // the thread above the top row
        at_hu = 8 * (up * hw + k / kGroup);
        cut_u = (k % kGroup) * 2 * G + G;
        at_hd = 8 * (dn * hw + col / kGroup);
        cut_d = (col % kGroup) * 2 * G;
        at_own = 8 * (r * hw + t / kGroup);
        // the first lane of a group stores it if the group holds boundary units
        const uint32_t last = min(t + kGroup - 1, nt - 1), vl = active ? last / upr : 0, bv = (R - 1) % VB;
        publish = active && t % kGroup == 0 && (vb == 0 || vb <= bv) && (vb == 0 || vl >= bv);
    }
    // The boundary rows of word w as the words of pass number n (the state
    // before pass 0 is number 0, pass q's outcome number q + 1).
    auto send = [&](uint32_t w, uint32_t n) {
        if constexpr (GANG) {
            uint32_t v = (w & GM) | ((w >> sb) & GM) << G;
            if constexpr (G == 2) v |= from_lane_plus<1>(v) << 4;
            v |= from_lane_plus<G == 2 ? 2 : 1>(v) << 8;
            v |= from_lane_plus<G == 2 ? 4 : 2>(v) << 16;
            if (publish) put_word(reinterpret_cast<uint64_t *>(halo + (n & 1) * slot_bytes + at_own), v, a.epoch0 + n + 1);
        }
    };
    X[t] = W[0];
    X[kMaxT + t] = W[1];
    if (t == 0) *zero_word = 0;
    for (uint32_t i = t; i < kBitsRing; i += nth) e_ring[i] = 0;

    send(W[1], 0);

    const Accept A = make_accept(a.T4, a.T8);
    const uint32_t all4 = A.lo <= 2 ? ~0u : 0u, all8 = A.lo == 0 ? ~0u : 0u;
    uint32_t q = 0;  // pass counter

    // The neighbours' words pass q uses (number q), by the top and bottom
    // rows' threads.  They are asked for in the middle of the pass's draws:
    // the neighbours stored them when this strip did, so a load right after
    // that would bring the word before and the next one its whole latency.
    uint64_t word_u = 0, word_d = 0;
    auto request = [&]() {
        if constexpr (GANG) {
            const uint8_t *slot = halo + (q & 1) * slot_bytes;
            if (top) word_u = __hip_atomic_load(reinterpret_cast<const uint64_t *>(slot + at_hu), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (bottom) word_d = __hip_atomic_load(reinterpret_cast<const uint64_t *>(slot + at_hd), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    };
    auto receive = [&]() {
        if constexpr (GANG) {
            const uint32_t tag = a.epoch0 + q + 1;
            uint32_t polls = 0;
            auto late = [&]() {
                return (top & (static_cast<uint32_t>(word_u >> 32) != tag)) | (bottom & (static_cast<uint32_t>(word_d >> 32) != tag));
            };
            while (__any(late())) {  // the wave together: bounded, and over soon in a lattice where a wait has given up
                ++polls;
                if (polls > kSpinLimit || ((polls & 63) == 0 && __hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
                    if ((t & 63) == 0) __hip_atomic_fetch_or(a.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
                request();
            }
            halo_u = (static_cast<uint32_t>(word_u) >> cut_u) & GM;
            halo_d = (static_cast<uint32_t>(word_d) >> cut_d) & GM;
        }
    };

    // The words of the neighbouring threads, other colour than c.
    struct Near {
        uint32_t l, r, u, d;
    };
    auto near = [&](int c) {
        const uint32_t *x = X + (1 - c) * kMaxT;
        return Near{x[at_l], x[at_r], x[at_u], x[at_d]};
    };
    // d[k]: where neighbour k differs from the colour-c sites.
    auto differ = [&](int c, const Near &x, uint32_t (&d)[4]) {
        const uint32_t O = W[1 - c], C = W[c];
        const uint32_t from_left = bfi(kFirst, x.l >> (G - 1), O << 1);
        const uint32_t from_right = bfi(kLast, x.r << (G - 1), O >> 1);
        const uint32_t p0 = c == 0 ? even : ~even;  // slots with p = 0
        if constexpr (!GANG) {  // periodic in y (VB divides R): the far rows of the strip itself
            halo_u = (x.u >> sb) & GM;
            halo_d = x.d & GM;
        }
        d[0] = O ^ C;
        d[1] = bfi(p0, from_left, from_right) ^ C;
        d[2] = bfi(top_m, halo_u, x.u << sh_u) ^ C;
        d[3] = bfi(bot_m, halo_d << sb, x.d >> sh_d) ^ C;
    };
    // Energy: a sweep's sum is made of the colour-1 pass's words during the
    // next pass, into a ring of kBitsRing sweeps that is written out when it is
    // full and at the end.  (One global atomic per sweep held its wave up in
    // every second pass: stores and loads complete in order.)
    uint32_t unlike = 0;  // differing neighbours of the thread's colour-1 sites
    auto reduce_energy = [&](uint64_t sweep) {
        const int v = wave_sum_last(static_cast<int>(4 * G * counted) - 2 * static_cast<int>(unlike));
        if ((t & 63) == 63) atomicAdd(&e_ring[sweep % kBitsRing], v);
    };
    auto flush_energy = [&](uint64_t first, uint32_t n) {
        for (uint32_t i = t; i < n; i += nth) {
            const int v = e_ring[i];
            e_ring[i] = 0;
            if constexpr (GANG || TILE) atomicAdd(a.trace + first + i, -v);
            else a.trace[first + i] = -v;  // the only contributor
        }
    };
    // What pass (sweep, c) does for the energies of the sweeps before.
    auto energies = [&](int c, uint64_t sweep) {
        if (!a.trace || sweep == 0) return;
        if (c == 0) reduce_energy(sweep - 1);
        else if (sweep % kBitsRing == 0) flush_energy(sweep - kBitsRing, kBitsRing);
    };
    auto finish = [&](int c, uint32_t flip, const uint32_t (&d)[4]) {
        W[c] ^= flip;
        X[c * kMaxT + t] = W[c];
        send(W[c], q + 1);
        if (c == 1) {
            unlike = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) unlike += __popc((d[k] ^ flip) & own);
        }
        ++q;
    };
    // A pass from the outcomes (a4, a8) of its draws, then the next pass's
    // draws.
    auto update = [&](int c, uint64_t sweep, uint32_t a4, uint32_t a8, auto &&more) {
        receive();
        __syncthreads();  // the other threads' words of the pass before
        const Near x = near(c);
        energies(c, sweep);
        uint32_t d[4];
        differ(c, x, d);
        a4 |= all4;
        a8 |= all8;
        const uint32_t s = d[0] ^ d[1] ^ d[2];
        const uint32_t two = (d[0] & d[1]) | (d[2] & (d[0] | d[1]));
        // at least two neighbours differ, or the draw is below the threshold
        // of one (odd: one or three) or of none
        finish(c, two | (s & d[3]) | a8 | ((s ^ d[3]) & a4), d);
        more();
    };

    if constexpr (MH) {
        // `hits` draws for the first colour-c site of every stream, then as
        // many for the second; a hit's outcomes (one bit per stream) decide
        // all streams' sites at once.  The first kAhead hits' draws are made
        // while the neighbours' words are on their way.
        constexpr uint32_t kAhead = 4;
        auto pass = [&](int c, uint64_t sweep) {
            request();
            uint32_t b4[kAhead], b8[kAhead];
            auto draws = [&](int j, uint32_t h, uint32_t &a4, uint32_t &a8) {  // hit h of site j
                a4 = a8 = 0;
#pragma unroll
                for (int i = SPT - 1; i >= 0; --i) {
                    if constexpr (NB == 8) {
                        uint32_t ra, rb;
                        u[i].pair(ra, rb);
                        push2(a4, a8, rb, ra, A.t4, A.t8);
                    } else if constexpr (kWeylLds) {
                        const uint32_t n = (2 * q + j) * a.hits + h + 1;  // draws of the call with this one
                        push1(a4, a8, u[i].next(weyl0[i], n * kWeylC), A.t4, A.t8);
                    } else if constexpr (kSub) {
                        push1(a4, a8, u[i].next(map), A.t4, A.t8);
                    } else if constexpr (!IsPhiloxKey<Unit>::value) {
                        push1(a4, a8, u[i].one(), A.t4, A.t8);
                    }
                    if constexpr (sizeof(Unit) >= 16) __builtin_amdgcn_sched_barrier(0);
                }
            };
            // Philox: every stream stands at position pos; the block of draw n
            const uint64_t pos = a.blk0 + q * 2ull * a.hits;
            auto block = [&](uint32_t n) {
                if constexpr (IsPhiloxKey<Unit>::value) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) b4[k] = b8[k] = 0;
#pragma unroll
                    for (int i = SPT - 1; i >= 0; --i) {
                        uint32_t w[4];
                        u[i].block((pos + n) >> 2, w);
#pragma unroll
                        for (int k = 0; k < 4; ++k) push1(b4[k], b8[k], w[k], A.t4, A.t8);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            };
            if constexpr (IsPhiloxKey<Unit>::value) {
                block(0);
            } else {
#pragma unroll
                for (uint32_t h = 0; h < kAhead; ++h)
                    if (h < a.hits) draws(0, h, b4[h], b8[h]);
            }
            receive();
            __syncthreads();
            const Near x = near(c);
            energies(c, sweep);
            uint32_t d[4];
            differ(c, x, d);
            const uint32_t s = d[0] ^ d[1] ^ d[2];
            const uint32_t two = (d[0] & d[1]) | (d[2] & (d[0] | d[1]));
            const uint32_t ge2 = two | (s & d[3]), le2 = ~(two & (s | d[3])), odd = s ^ d[3];
            uint32_t f[2] = {0, 0};
            // one hit: fl the flips so far; a flip turns m differing neighbours into 4 - m
            uint32_t hg = 0, hl = 0, ho = 0, fl = 0;
            auto begin = [&](int j) {
                hg = gather_even(ge2 >> j);
                hl = gather_even(le2 >> j);
                ho = gather_even(odd >> j);
                fl = 0;
            };
            auto hit = [&](uint32_t a4, uint32_t a8) {
                fl ^= bfi(fl, hl, hg) | a8 | all8 | (ho & (a4 | all4));
            };
            begin(0);
            if constexpr (IsPhiloxKey<Unit>::value) {
                const uint32_t n_draws = 2 * a.hits;
                uint32_t n = 0;
                while (true) {
                    const uint32_t k0 = static_cast<uint32_t>(pos + n) & 3;
#pragma unroll
                    for (uint32_t k = 0; k < 4; ++k) {
                        if (k >= k0 && n < n_draws) {
                            hit(b4[k], b8[k]);
                            if (++n == a.hits) {
                                f[0] = fl;
                                begin(1);
                            }
                        }
                    }
                    if (n == n_draws) break;
                    block(n);
                }
                f[1] = fl;
            } else {
#pragma unroll
                for (uint32_t h = 0; h < kAhead; ++h)
                    if (h < a.hits) hit(b4[h], b8[h]);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    for (uint32_t h = j == 0 ? kAhead : 0; h < a.hits; ++h) {
                        uint32_t a4, a8;
                        draws(j, h, a4, a8);
                        hit(a4, a8);
                    }
                    f[j] = fl;
                    if (j == 0) begin(1);
                }
            }
            finish(c, spread_even(f[0]) | spread_even(f[1]) << 1, d);
        };
        for (uint64_t sweep = 0; sweep < a.n_sweeps; ++sweep) {
            pass(0, sweep);
            pass(1, sweep);
        }
    } else if constexpr (IsPhiloxKey<Unit>::value) {
        // A block serves both passes of a sweep, so only its outcomes are
        // kept.  Half of the blocks of sweep s + 1 are made in each pass of
        // sweep s, so that both passes have work that hides their waits.
        uint32_t n4[2] = {0, 0}, n8[2] = {0, 0};
        auto blocks = [&](uint64_t sweep, auto upper) {
            constexpr int hi = decltype(upper)::value ? SPT : SPT / 2, lo = decltype(upper)::value ? SPT / 2 : 0;
#pragma unroll
            for (int i = hi - 1; i >= lo; --i) {
                uint32_t w[4];
                u[i].block(a.blk0 + sweep, w);
                push2(n4[0], n8[0], w[1], w[0], A.t4, A.t8);
                push2(n4[1], n8[1], w[3], w[2], A.t4, A.t8);
                if (i == (hi + lo) / 2) request();
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        blocks(0, std::true_type{});
        blocks(0, std::false_type{});
        for (uint64_t sweep = 0; sweep < a.n_sweeps; ++sweep) {
            const uint32_t c4[2] = {n4[0], n4[1]}, c8[2] = {n8[0], n8[1]};
            n4[0] = n4[1] = n8[0] = n8[1] = 0;
            const bool go_on = sweep + 1 < a.n_sweeps;
            update(0, sweep, c4[0], c8[0], [&]() { if (go_on) blocks(sweep + 1, std::true_type{}); else request(); });
            update(1, sweep, c4[1], c8[1], [&]() { if (go_on && SPT > 1) blocks(sweep + 1, std::false_type{}); else request(); });
        }
    } else {
        uint32_t n4 = 0, n8 = 0;
        auto draws = [&](int c, uint64_t sweep) {
            n4 = n8 = 0;
#pragma unroll
            for (int i = SPT - 1; i >= 0; --i) {
                uint32_t rr[G];
                if constexpr (kWeylLds) {
                    const uint32_t d0 = weyl0[i], w = static_cast<uint32_t>(4 * sweep + 2 * c) * kWeylC;
                    rr[0] = u[i].next(d0, w + kWeylC);
                    rr[1] = u[i].next(d0, w + 2 * kWeylC);
                } else if constexpr (kSub) {
                    rr[0] = u[i].next(map);
                    rr[1] = u[i].next(map);
                } else if constexpr (SweepCounter<Unit>::value) {
                    u[i].draw_at(rr, a, sweep, c);
                } else {
                    u[i].draw(rr);
                }
#pragma unroll
                for (int j = G - 2; j >= 0; j -= 2) push2(n4, n8, rr[j + 1], rr[j], A.t4, A.t8);
                if (i == SPT / 2) request();
                // wide units one at a time: only the held states stay live
                if constexpr (sizeof(Unit) >= 16) __builtin_amdgcn_sched_barrier(0);
            }
        };
        draws(0, 0);
        for (uint64_t sweep = 0; sweep < a.n_sweeps; ++sweep) {
            update(0, sweep, n4, n8, [&]() { draws(1, sweep); });
            update(1, sweep, n4, n8, [&]() { if (sweep + 1 < a.n_sweeps) draws(0, sweep + 1); else request(); });
        }
    }
    __syncthreads();
    if (a.trace && a.n_sweeps > 0) {
        reduce_energy(a.n_sweeps - 1);
        __syncthreads();
        const uint64_t first = (a.n_sweeps - 1) / kBitsRing * kBitsRing;
        flush_energy(first, static_cast<uint32_t>(a.n_sweeps - first));
    }

    // Spins back as bytes: +1 = 0x01, -1 = 0xFF.  The places are worked out
    // anew from a thread index that passes through LDS: else the addresses of
    // the loads above stay in registers through all sweeps (two per slot).
    const uint32_t t2 = t + *zero_word, vb2 = t2 < nt ? t2 / upr : 0, col2 = t2 - vb2 * upr;
    const uint32_t rows2 = t2 < nt && vb2 < R ? (R - 1 - vb2) / VB + 1 : 0;
    auto bytes = [&](uint32_t even_bits, uint32_t odd_bits) {  // 2 + 2 bits -> 4 sites
        const uint32_t e = (even_bits | even_bits << 15) & 0x00010001u, o = (odd_bits | odd_bits << 15) & 0x00010001u;
        return ((e | o << 8) * 0xFEu) ^ 0x01010101u;
    };
    const uint32_t ucol2 = unit_of(col2);
    int8_t *const spins_out = TILE ? a.spins_out : a.spins;
    uint8_t *const st_out = TILE ? a.st_out : a.st;
#pragma unroll
    for (int i = 0; i < SPT; ++i) {
        bool keep = static_cast<uint32_t>(i) < rows2;
        if constexpr (TILE) keep = keep && col2 - a.in_x < a.n_x && vb2 + i * VB - a.in_y < a.n_y;
        if (keep) {
            const uint64_t y = row_of(vb2, i);
            const uint32_t b0 = (W[0] >> (G * i)) & GM, b1 = (W[1] >> (G * i)) & GM;
            const uint32_t e = y & 1 ? b1 : b0, o = y & 1 ? b0 : b1;
            uint32_t *p = reinterpret_cast<uint32_t *>(spins_out + y * L + static_cast<uint64_t>(ucol2) * NB);
            p[0] = bytes(e & 3, o & 3);
            if constexpr (NB == 8) p[1] = bytes(e >> 2, o >> 2);
            const uint64_t k = TILE ? y * row_units + ucol2 : ubase + t2 + static_cast<uint64_t>(i) * nt;
            const uint64_t steps = 4 * a.n_sweeps * (MH ? a.hits : 1);
            if constexpr (IsPhiloxKey<Unit>::value)
                u[i].put_position(st_out, a.S, k, MH ? a.blk0 + steps : 4 * (a.blk0 + a.n_sweeps));
            else if constexpr (kWeylLds)
                u[i].store(st_out, a.S, k, weyl0[i] + static_cast<uint32_t>(steps) * kWeylC);
            else if constexpr (SweepCounter<Unit>::value) u[i].store_at(st_out, a.S, k, a);
            else if constexpr (TILE && std::is_same<Unit, XsUnit>::value) u[i].store(st_out, a.st, a.S, k, steps);
            else u[i].store(st_out, a.S, k, steps);
        }
    }
}

// Strip r in the form its streams allow: Philox streams that stand at one
// position (a multiple of 4 for single-hit sweeps) and XS1024W instances that
// have taken the same number of steps, the usual case as every call advances
// all alike, take what they share from the call's start.
template <class Unit, int SPT, bool MH, bool GANG>
__device__ __forceinline__ void bits_strip(const StripArgs &a, uint32_t r, uint32_t *lds) {
    StripArgs b = a;
    if constexpr (std::is_same<Unit, PhiloxUnit>::value || std::is_same<Unit, PhiloxUnit7>::value) {
        using Key = PhiloxKeyUnitR<std::is_same<Unit, PhiloxUnit>::value ? 10 : 7>;
        if (MH ? strip_positions_equal(a, r, &b.blk0) : strip_positions_aligned(a, r, &b.blk0)) {
            bits_body<Key, SPT, MH, GANG>(b, r, lds);
            return;
        }
    }
    if constexpr (std::is_same<Unit, XsUnit>::value && !MH) {
        if (strip_steps_uniform(a, r, &b.blk0, &b.y_start)) {
            bits_body<XsSweepUnit, SPT, false, GANG>(b, r, lds);
            return;
        }
    }
    // XORWOW multi-hit draws wait on the Weyl word's LDS read each time (L = 1024, 8 sweeps of 10 hits 103 us); up to 8
    // units of a thread keep it in a register (88)
    if constexpr (std::is_same<Unit, SmallUnit<Xorwow>>::value && MH && SPT <= 8) bits_body<Unit, SPT, MH, GANG>(a, r, lds);
    else if constexpr (std::is_same<Unit, SmallUnit<Xorwow>>::value) bits_body<XorwowStripUnit, SPT, MH, GANG>(a, r, lds);
    else if constexpr (std::is_same<Unit, SmallUnit<Lcg32Sub>>::value) bits_body<LcgSubStripUnit<uint32_t>, SPT, MH, GANG>(a, r, lds);
    else if constexpr (std::is_same<Unit, SmallUnit<Lcg64Sub>>::value) bits_body<LcgSubStripUnit<uint64_t>, SPT, MH, GANG>(a, r, lds);
    else bits_body<Unit, SPT, MH, GANG>(a, r, lds);
}

template <class Unit, int SPT, bool MH, bool GANG>
__global__ __launch_bounds__(kBitsMaxThreads) void k_ising_bits(StripArgs a) {
    extern __shared__ __align__(16) uint32_t bits_lds[];
    // Blocks b, b+8, b+16, ... share an XCD: give them consecutive strips so
    // that most neighbour exchanges stay inside one L2.
    const uint32_t b = blockIdx.x, nwg = a.nwg;
    const uint32_t r = (nwg % 8 == 0) ? (b % 8) * (nwg / 8) + b / 8 : b;
    bits_strip<Unit, SPT, MH, GANG>(a, r, bits_lds);
}

// The kernel for `slots` slots per thread, or null.
template <class Unit, bool MH, bool GANG>
const void *bits_kernel_of(int slots) {
    switch (slots) {
    case 1: return reinterpret_cast<const void *>(&k_ising_bits<Unit, 1, MH, GANG>);
    case 2: return reinterpret_cast<const void *>(&k_ising_bits<Unit, 2, MH, GANG>);
    case 4: return reinterpret_cast<const void *>(&k_ising_bits<Unit, 4, MH, GANG>);
    case 6: return reinterpret_cast<const void *>(&k_ising_bits<Unit, 6, MH, GANG>);
    case 8: return reinterpret_cast<const void *>(&k_ising_bits<Unit, 8, MH, GANG>);
    }
    if constexpr (Unit::kNB == 4) {
        if (slots == 12) return reinterpret_cast<const void *>(&k_ising_bits<Unit, 12, MH, GANG>);
        if (slots == 16) return reinterpret_cast<const void *>(&k_ising_bits<Unit, 16, MH, GANG>);
    }
    return nullptr;
}
template <class Unit>
const void *bits_kernel_of(int slots, bool hits, bool gang) {
    if (gang) return hits ? bits_kernel_of<Unit, true, true>(slots) : bits_kernel_of<Unit, false, true>(slots);
    return hits ? bits_kernel_of<Unit, true, false>(slots) : bits_kernel_of<Unit, false, false>(slots);
}

// A lattice that does not fit on chip, a few sweeps at a time: each workgroup
// takes a tile with `margin` rows and columns around the part it keeps, makes
// 2 n_sweeps <= margin passes on chip (the margin's sites are updated like all
// others, from their own streams, and turn wrong from the edge inwards one site
// a pass) and writes what it keeps, spins and states, to another image; the
// next block of sweeps goes back.  One launch per colour pass moves every
// state and spin twice per sweep and is bound by that; a block moves them once
// per n_sweeps and the margins once more, and its loads, all in flight at
// once, overlap the passes of the CU's other workgroups.  L = 8192, us per
// sweep of 8, per pass -> tiles: MWC 146 -> 31 (bytes 25, instructions 18),
// LCG32 123 -> 27, XORWOW 361 -> 87, Philox 4x32-10 226 -> 62, XS1024W
// 129 -> 78 (its margin of whole instances, 128 columns, costs 1.8 times the
// instructions).
// Tiles in the order of the lattice within each of the 8 dies.
__device__ __forceinline__ uint32_t xcd_order(uint32_t b, uint32_t n) {
    const uint32_t q = n / 8, rest = n % 8, x = b % 8;
    return x * q + min(x, rest) + b / 8;
}

template <class Unit, bool MH>
__global__ __launch_bounds__(kBitsMaxThreads) void k_ising_tiles(TileArgs ta) {
    constexpr int NB = Unit::kNB, SPT = 64 / NB;
    extern __shared__ __align__(16) uint32_t bits_lds[];
    StripArgs a = ta.s;
    const uint32_t tile = xcd_order(blockIdx.x, gridDim.x), tx = tile % ta.tiles_x, ty = tile / ta.tiles_x, L = a.L;
    const uint32_t kx = tx * ta.keep_w, ky = ty * ta.keep_h;  // the kept part's place in the lattice
    a.x0 = kx >= ta.margin_x ? kx - ta.margin_x : kx + L - ta.margin_x;
    a.y0 = ky >= ta.margin_y ? ky - ta.margin_y : ky + L - ta.margin_y;
    a.in_x = ta.margin_x / NB;
    a.in_y = ta.margin_y;
    a.n_x = min(ta.keep_w, L - kx) / NB;
    a.n_y = min(ta.keep_h, L - ky);
    // the tile's units, for the tests of what its streams share
    const uint32_t upr = a.tile_w / NB, row_units = L / NB, x0u = a.x0 / NB;
    auto all_equal = [&](auto &&value, uint64_t *first) {
        const uint32_t vb = threadIdx.x / upr;
        uint32_t x = x0u + threadIdx.x % upr;
        if (x >= row_units) x -= row_units;
        *first = value(static_cast<uint64_t>(a.y0) * row_units + x0u);
        uint64_t v[SPT];
#pragma unroll
        for (int i = 0; i < SPT; ++i) {
            uint32_t y = a.y0 + vb + i * a.VB;
            if (y >= L) y -= L;
            v[i] = value(static_cast<uint64_t>(y) * row_units + x);
        }
        int ok = 1;
#pragma unroll
        for (int i = 0; i < SPT; ++i) ok &= v[i] == *first;
        return __syncthreads_and(ok) != 0;
    };
    if constexpr (std::is_same<Unit, PhiloxUnit>::value || std::is_same<Unit, PhiloxUnit7>::value) {
        using Key = PhiloxKeyUnitR<std::is_same<Unit, PhiloxUnit>::value ? 10 : 7>;
        const uint64_t *pos = reinterpret_cast<const uint64_t *>(a.st + 8 * a.S);
        uint64_t p;
        if (all_equal([&](uint64_t u) { return pos[u]; }, &p) && (MH || (p & 3) == 0)) {
            a.blk0 = MH ? p : p >> 2;
            bits_body<Key, SPT, MH, false, true>(a, 0, bits_lds);
            return;
        }
    }
    if constexpr (std::is_same<Unit, XsUnit>::value && !MH) {
        const uint64_t *N = reinterpret_cast<const uint64_t *>(a.st + 4 * a.S);
        uint64_t n;
        if (all_equal([&](uint64_t u) { return N[u >> 4]; }, &n)) {
            a.blk0 = n;
            a.y_start = *reinterpret_cast<const uint32_t *>(a.cst + 4 * a.S + 8 * (a.S / 32)) + static_cast<uint32_t>(n) * kWeylC;
            bits_body<XsSweepUnit, SPT, false, false, true>(a, 0, bits_lds);
            return;
        }
    }
    if constexpr (std::is_same<Unit, SmallUnit<Xorwow>>::value) bits_body<XorwowStripUnit, SPT, MH, false, true>(a, 0, bits_lds);
    else if constexpr (std::is_same<Unit, SmallUnit<Lcg32Sub>>::value) bits_body<LcgSubStripUnit<uint32_t>, SPT, MH, false, true>(a, 0, bits_lds);
    else if constexpr (std::is_same<Unit, SmallUnit<Lcg64Sub>>::value) bits_body<LcgSubStripUnit<uint64_t>, SPT, MH, false, true>(a, 0, bits_lds);
    else bits_body<Unit, SPT, MH, false, true>(a, 0, bits_lds);
}

template <class Unit>
const void *tiles_kernel_of(bool hits) {
    if constexpr (!std::is_same<Unit, XsUnit>::value)
        if (hits) return reinterpret_cast<const void *>(&k_ising_tiles<Unit, true>);
    return hits ? nullptr : reinterpret_cast<const void *>(&k_ising_tiles<Unit, false>);
}

// Batches whose replicas all keep their spins as bits (or stream through
// memory): persistent workgroups take (replica, strip) items as k_ising_batch
// does.  The slots of a replica are one of three per kind, so that the kernel
// holds few copies of the strip's body.  60 replicas of L = 16 .. 1024, 50
// sweeps: XS1024W 1.34 -> 0.71 ms, LCG32 1.32 -> 0.48; 512 such, XS1024W,
// 1169 -> 2054 updates/ns; 2048 of L <= 128 990 (256-thread workgroups) -> 1767
// (512).
template <class Unit, int SPT>
__device__ __forceinline__ void bits_item(const StripArgs &a, uint32_t r, bool gang, uint32_t *lds) {
    if (gang) bits_strip<Unit, SPT, false, true>(a, r, lds);
    else bits_strip<Unit, SPT, false, false>(a, r, lds);
}

template <class Unit, int MAXT>
__global__ __launch_bounds__(MAXT) void k_ising_batch_bits(const ReplicaDesc *reps, const uint2 *items, uint32_t n_items,
                                                           uint32_t *next) {
    constexpr int kMost = 64 / Unit::kNB;  // slots: kMost, half or a quarter of it
    extern __shared__ __align__(16) uint32_t bits_lds[];
    __shared__ uint32_t idx_s;
    __shared__ int red_s[16];
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) idx_s = atomicAdd(next, 1u);
        __syncthreads();
        const uint32_t idx = idx_s;
        if (idx >= n_items) break;  // every workgroup leaves once the list is drained
        const uint2 item = items[idx];
        const ReplicaDesc d = reps[item.x];
        // No sweeps: nothing moves.  (A strip makes its first pass's draws before it enters the loop over the sweeps;
        // a test there, or where the strip's form is chosen, cost lone lattices 2%, XORWOW batches up to 18%.)
        if (d.n_sweeps == 0) continue;
        if (d.mode == kReplicaMemory) {
            replica_in_memory<Unit>(d, red_s);
            continue;
        }
        const bool gang = d.mode == kReplicaStrips;
        if (gang) gang_start(d);
        const uint32_t R = item.y + 1 == d.nwg ? d.R_last : d.R;
        const StripArgs a{d.spins, d.st, d.S, d.L, R, d.nwg, R * (d.L / Unit::kNB), d.T4, d.T8, d.n_sweeps, d.trace,
                          d.halo, 0, d.err, 1, d.R, 0, 0, d.VB};
        if (d.slots > kMost / 2) bits_item<Unit, kMost>(a, item.y, gang, bits_lds);
        else if (d.slots > kMost / 4) bits_item<Unit, kMost / 2>(a, item.y, gang, bits_lds);
        else bits_item<Unit, kMost / 4>(a, item.y, gang, bits_lds);
    }
}

template <class Unit>
const void *batch_bits_kernel_of(uint32_t threads) {
    if (threads > 512) return reinterpret_cast<const void *>(&k_ising_batch_bits<Unit, 1024>);
    return reinterpret_cast<const void *>(&k_ising_batch_bits<Unit, 512>);
}

}  // namespace rngx
