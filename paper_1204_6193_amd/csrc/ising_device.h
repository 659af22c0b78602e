// Device code shared by the Ising kernels: the update units, a strip's
// arguments, the tagged halo words, and the tests that pick a strip's form.
#pragma once

#include <type_traits>

#include "rngx_internal.h"

namespace rngx {

constexpr int kBlock = 256;

// ---------------------------------------------------------------- units
// A unit is what one thread updates with one set of draws: a stream (4
// sites) for the small-state kinds, a lane pair of an XS1024W instance (8
// sites) for the paper's generator.  Units are numbered like the stream
// (small kinds) or stream/2 (XS1024W).
template <class G>
struct SmallUnit {
    static constexpr int kNB = 4;
    G g;
    __device__ void load(const uint8_t *st, uint64_t S, uint64_t u) { g.load(st, S, u); }
    __device__ void store(uint8_t *st, uint64_t S, uint64_t u, uint64_t) const { g.store(st, S, u); }
    __device__ void draw(uint32_t (&r)[2]) { r[0] = g.next(); r[1] = g.next(); }
    __device__ uint32_t one() { return g.next(); }
    // multi-hit updates: n draws in order to f0, then n more to f1
    template <class F0, class F1>
    __device__ void draws2(uint32_t n, F0 &&f0, F1 &&f1) {
        for (uint32_t i = 0; i < n; ++i) f0(g.next());
        for (uint32_t i = 0; i < n; ++i) f1(g.next());
    }
};

// Philox with only key and position held: the two draws of a pass come from
// one block unless they straddle a block boundary.
template <int ROUNDS>
struct PhiloxUnitR {
    static constexpr int kNB = 4;
    uint32_t k0, k1;
    uint64_t pos;
    __device__ void load(const uint8_t *st, uint64_t S, uint64_t u) {
        const uint32_t *p = reinterpret_cast<const uint32_t *>(st);
        k0 = p[u]; k1 = p[S + u];
        pos = reinterpret_cast<const uint64_t *>(st + 8 * S)[u];
    }
    // keys from the image `cst`
    __device__ void load(const uint8_t *st, const uint8_t *cst, uint64_t S, uint64_t u) {
        const uint32_t *p = reinterpret_cast<const uint32_t *>(cst);
        k0 = p[u]; k1 = p[S + u];
        pos = reinterpret_cast<const uint64_t *>(st + 8 * S)[u];
    }
    __device__ void store(uint8_t *st, uint64_t S, uint64_t u, uint64_t) const {
        reinterpret_cast<uint64_t *>(st + 8 * S)[u] = pos;
    }
    __device__ void draw(uint32_t (&r)[2]) {
        uint32_t b0, b1, b2, b3;
        philox_block<ROUNDS>(k0, k1, pos >> 2, b0, b1, b2, b3);
        const uint32_t j = static_cast<uint32_t>(pos) & 3;
        r[0] = j == 0 ? b0 : j == 1 ? b1 : j == 2 ? b2 : b3;
        if (j == 3) philox_block<ROUNDS>(k0, k1, (pos >> 2) + 1, b0, b1, b2, b3);
        r[1] = j == 0 ? b1 : j == 1 ? b2 : j == 2 ? b3 : b0;
        pos += 2;
    }
    __device__ uint32_t one() {
        uint32_t b0, b1, b2, b3;
        philox_block<ROUNDS>(k0, k1, pos >> 2, b0, b1, b2, b3);
        const uint32_t j = static_cast<uint32_t>(pos++) & 3;
        return j == 0 ? b0 : j == 1 ? b1 : j == 2 ? b2 : b3;
    }
    // as SmallUnit::draws2, in one loop so that a block serves four draws in
    // a row also across the two runs
    template <class F0, class F1>
    __device__ void draws2(uint32_t n, F0 &&f0, F1 &&f1) {
        uint32_t b0 = 0, b1 = 0, b2 = 0, b3 = 0;
        for (uint32_t i = 0; i < 2 * n; ++i) {
            const uint32_t j = static_cast<uint32_t>(pos) & 3;
            if (i == 0 || j == 0) philox_block<ROUNDS>(k0, k1, pos >> 2, b0, b1, b2, b3);
            const uint32_t r = j == 0 ? b0 : j == 1 ? b1 : j == 2 ? b2 : b3;
            if (i < n) f0(r);
            else f1(r);
            ++pos;
        }
    }
};
using PhiloxUnit = PhiloxUnitR<10>;
using PhiloxUnit7 = PhiloxUnitR<7>;

// Philox in a strip whose streams all stand at the same block boundary at
// the start of a call (the usual case: seeded at 0, and every call advances
// every stream by the same multiple of 4).  A sweep takes the four words of
// one block: the colour-0 pass makes block blk0 + t, uses words 0 and 1 and
// keeps 2 and 3 for the colour-1 pass, so each block is made once rather
// than once per pass, and the position, the same for all units, is not held
// per unit.
template <int ROUNDS>
struct PhiloxSweepUnitR {
    static constexpr int kNB = 4;
    uint32_t k0, k1, c2, c3;
    __device__ void load(const uint8_t *st, uint64_t S, uint64_t u) {
        const uint32_t *p = reinterpret_cast<const uint32_t *>(st);
        k0 = p[u]; k1 = p[S + u];
        c2 = c3 = 0;
    }
    template <class Args>
    __device__ void store_at(uint8_t *st, uint64_t S, uint64_t u, const Args &g) const {
        reinterpret_cast<uint64_t *>(st + 8 * S)[u] = 4 * (g.blk0 + g.n_sweeps);
    }
    template <class Args>
    __device__ void draw_at(uint32_t (&r)[2], const Args &g, uint64_t sweep, int c) {
        if (c == 0) {
            philox_block<ROUNDS>(k0, k1, g.blk0 + sweep, r[0], r[1], c2, c3);
        } else {
            r[0] = c2;
            r[1] = c3;
        }
    }
};
// The same for spins held as bits, where only a block's outcomes are kept:
// the key alone.
template <int ROUNDS>
struct PhiloxKeyUnitR {
    static constexpr int kNB = 4;
    uint32_t k0, k1;
    __device__ void load(const uint8_t *st, uint64_t S, uint64_t u) {
        const uint32_t *p = reinterpret_cast<const uint32_t *>(st);
        k0 = p[u]; k1 = p[S + u];
    }
    __device__ void block(uint64_t blk, uint32_t (&w)[4]) const {
        philox_block<ROUNDS>(k0, k1, blk, w[0], w[1], w[2], w[3]);
    }
    __device__ void put_position(uint8_t *st, uint64_t S, uint64_t u, uint64_t pos) const {
        reinterpret_cast<uint64_t *>(st + 8 * S)[u] = pos;
    }
};
// XORWOW for spins held as bits.  Six words a unit do not fit beside 16 units
// per thread (96 of 128 VGPRs; the passes spilled 60 words), and the Weyl word
// moves alike for all streams of a call, so its start stays in LDS and a draw
// adds the steps since then.
struct XorwowStripUnit {
    static constexpr int kNB = 4;
    uint32_t x, y, z, w, v;
    __device__ void load(const uint8_t *st, uint64_t S, uint64_t u, uint32_t *d) {
        const uint32_t *p = reinterpret_cast<const uint32_t *>(st);
        x = p[u]; y = p[S + u]; z = p[2 * S + u]; w = p[3 * S + u]; v = p[4 * S + u];
        *d = p[5 * S + u];
    }
    __device__ void store(uint8_t *st, uint64_t S, uint64_t u, uint32_t d) const {
        uint32_t *p = reinterpret_cast<uint32_t *>(st);
        p[u] = x; p[S + u] = y; p[2 * S + u] = z; p[3 * S + u] = w; p[4 * S + u] = v; p[5 * S + u] = d;
    }
    // a draw: d0 the Weyl word at the start, weyl what the steps so far and this one add
    __device__ uint32_t next(uint32_t d0, uint32_t weyl) {
        const uint32_t t = x ^ (x >> 2);
        x = y; y = z; z = w; w = v;
        v = xor3(v, v << 4, t ^ (t << 1));
        return v + d0 + weyl;
    }
};
// Sub-stream LCGs for spins held as bits: the S-step map is one for all
// streams, so it is read once (to scalar registers) and not held per unit
// (6 words a unit spilled at 16 units per thread).
template <class T>
struct LcgMap {
    T A, C;
};
template <class T>
struct LcgSubStripUnit {
    static constexpr int kNB = 4;
    T x;
    __device__ static LcgMap<T> map(const uint8_t *st, uint64_t S) {
        const T *p = reinterpret_cast<const T *>(st) + S;
        return LcgMap<T>{p[0], p[1]};
    }
    __device__ void load(const uint8_t *st, uint64_t, uint64_t u) { x = reinterpret_cast<const T *>(st)[u]; }
    __device__ void store(uint8_t *st, uint64_t, uint64_t u, uint64_t) const { reinterpret_cast<T *>(st)[u] = x; }
    __device__ uint32_t next(const LcgMap<T> &m) {
        x = m.A * x + m.C;
        return sizeof(T) == 8 ? static_cast<uint32_t>(static_cast<uint64_t>(x) >> 32) : static_cast<uint32_t>(x);
    }
};
template <class Unit> struct SubWord { using type = void; };  // the word of a sub-stream LCG's unit
template <class T> struct SubWord<LcgSubStripUnit<T>> { using type = T; };
template <class Unit> struct SweepCounter : std::false_type {};  // units that derive their pass from the call's start
template <int ROUNDS> struct SweepCounter<PhiloxSweepUnitR<ROUNDS>> : std::true_type {};

// Lagged Fibonacci units in strips (single-hit).  A strip holds whole
// instances (1024 units each) and runs 1024 threads, so slot i of thread t is
// stream t of the strip's instance i.  Before each colour pass the workgroup
// makes that pass's two rows of every instance of the strip in LDS rings of B
// words (value v at v mod B; runs of at most kRun values, a barrier each,
// whose reads and writes never share a ring word) and each thread takes
// value t of both rows for every slot; the unit only hands them out, in the
// order of the per-pass path (row 1 to the first colour-c site, row 2 to the
// second).
template <int LR, int LS>
struct LfgStripUnit {
    static constexpr int kNB = 4;
    static constexpr uint32_t kR = LR, kS = LS;
    static constexpr uint32_t B = LR < 1024 ? 1024 : 2048;
    static constexpr uint32_t kRun = (B - LR) < static_cast<uint32_t>(LS) ? B - LR : LS;
    static_assert(B >= LR + 1 && kRun >= 1, "ring too small");
    uint32_t d0, d1;
    __device__ void load(const uint8_t *, uint64_t, uint64_t) {}
    __device__ void store(uint8_t *, uint64_t, uint64_t, uint64_t) const {}
    __device__ void draw(uint32_t (&r)[2]) { r[0] = d0; r[1] = d1; }
};
template <class Unit> struct IsLfgStrip : std::false_type {};
template <int LR, int LS> struct IsLfgStrip<LfgStripUnit<LR, LS>> : std::true_type {};
// LDS of the rings of a strip's instances (after the strip's own bytes).
template <class Unit>
__host__ __device__ constexpr uint64_t lfg_ring_bytes(uint32_t units) {
    if constexpr (IsLfgStrip<Unit>::value) return 4ull * Unit::B * (units / 1024) + 16;
    else return 0;
}

// XS1024W lane pair u: lane u%16 of instance u/16 of the handle (words 2u,
// 2u+1 = streams 2u and 2u+1).  Two instance steps per pass; the draws are
// ordered stream 2u first, stream 2u+1 second, each in step order.
struct XsUnit {
    static constexpr int kNB = 8;
    uint32_t a, b, y;
    __device__ void load(const uint8_t *st, uint64_t S, uint64_t u) {
        const uint2 w = reinterpret_cast<const uint2 *>(st)[u];
        a = w.x; b = w.y;
        const uint64_t n = reinterpret_cast<const uint64_t *>(st + 4 * S)[u >> 4];
        y = *reinterpret_cast<const uint32_t *>(st + 4 * S + 8 * (S / 32)) + static_cast<uint32_t>(n) * kWeylC;
    }
    // the Weyl seed from the image `cst`
    __device__ void load(const uint8_t *st, const uint8_t *cst, uint64_t S, uint64_t u) {
        const uint2 w = reinterpret_cast<const uint2 *>(st)[u];
        a = w.x; b = w.y;
        const uint64_t n = reinterpret_cast<const uint64_t *>(st + 4 * S)[u >> 4];
        y = *reinterpret_cast<const uint32_t *>(cst + 4 * S + 8 * (S / 32)) + static_cast<uint32_t>(n) * kWeylC;
    }
    __device__ void store(uint8_t *st, uint64_t S, uint64_t u, uint64_t steps) const {
        reinterpret_cast<uint2 *>(st)[u] = make_uint2(a, b);
        if ((u & 15) == 0) reinterpret_cast<uint64_t *>(st + 4 * S)[u >> 4] += steps;
    }
    // to another image than the one loaded from
    __device__ void store(uint8_t *st, const uint8_t *from, uint64_t S, uint64_t u, uint64_t steps) const {
        reinterpret_cast<uint2 *>(st)[u] = make_uint2(a, b);
        if ((u & 15) == 0)
            reinterpret_cast<uint64_t *>(st + 4 * S)[u >> 4] = reinterpret_cast<const uint64_t *>(from + 4 * S)[u >> 4] + steps;
    }
    __device__ void draw(uint32_t (&r)[4]) {
        xs1024_step(a, b);
        y += kWeylC;
        uint32_t m = weyl_mix(y);
        r[0] = a + m; r[2] = b + m;
        xs1024_step(a, b);
        y += kWeylC;
        m = weyl_mix(y);
        r[1] = a + m; r[3] = b + m;
    }
    // one instance step: the next draw of stream 2u (ra) and of 2u+1 (rb)
    __device__ void pair(uint32_t &ra, uint32_t &rb) {
        xs1024_step(a, b);
        y += kWeylC;
        const uint32_t m = weyl_mix(y);
        ra = a + m;
        rb = b + m;
    }
};

// XS1024W in a strip whose instances have all taken the same number of
// steps at the start of a call (the usual case: every call advances every
// instance alike).  The Weyl word of a pass is then the same for every unit:
// it follows from the call's start (step count blk0, Weyl word y_start) and
// the sweep, instead of being held and stepped per unit.
struct XsSweepUnit {
    static constexpr int kNB = 8;
    uint32_t a, b;
    __device__ void load(const uint8_t *st, uint64_t, uint64_t u) {
        const uint2 w = reinterpret_cast<const uint2 *>(st)[u];
        a = w.x; b = w.y;
    }
    template <class Args>
    __device__ void store_at(uint8_t *st, uint64_t S, uint64_t u, const Args &g) const {
        reinterpret_cast<uint2 *>(st)[u] = make_uint2(a, b);
        if ((u & 15) == 0) reinterpret_cast<uint64_t *>(st + 4 * S)[u >> 4] = g.blk0 + 4 * g.n_sweeps;
    }
    // as XsUnit::draw for the pass (sweep, c): 4 sweep + 2 c steps after the start
    template <class Args>
    __device__ void draw_at(uint32_t (&r)[4], const Args &g, uint64_t sweep, int c) {
        const uint32_t y = g.y_start + static_cast<uint32_t>(4 * sweep + 2 * c) * kWeylC;
        xs1024_step(a, b);
        uint32_t m = weyl_mix(y + kWeylC);
        r[0] = a + m; r[2] = b + m;
        xs1024_step(a, b);
        m = weyl_mix(y + 2 * kWeylC);
        r[1] = a + m; r[3] = b + m;
    }
};
template <> struct SweepCounter<XsSweepUnit> : std::true_type {};
template <class Unit> struct SweepOf { using type = void; };  // the sweep form of a unit, if it has one
template <int ROUNDS> struct SweepOf<PhiloxUnitR<ROUNDS>> { using type = PhiloxSweepUnitR<ROUNDS>; };
template <> struct SweepOf<XsUnit> { using type = XsSweepUnit; };

struct StripArgs {
    int8_t *spins;
    uint8_t *st;
    uint64_t S;
    uint32_t L, R, nwg, units;  // units per strip
    uint64_t T4, T8, n_sweeps;
    int32_t *trace;             // may be null
    uint64_t *halo;             // 2 slots x nwg x 2 rows x L/4 tagged words
    uint32_t epoch0;            // pass tags of this call are epoch0 + 1, epoch0 + 2, ...
    uint32_t *err;
    uint32_t hits;              // Metropolis updates per visited site (multi-hit kernels)
    uint32_t R0;                // rows of every strip but the last: strip r starts at row r*R0
    uint64_t blk0;              // sweep forms, at the start: Philox the common block index, XS1024W the step count
    uint32_t y_start;           // sweep-form XS1024W: the common Weyl word at the start
    uint32_t VB;                // spins as bits: rows side by side in a workgroup (slot i of a thread is row vb + i VB)
    // tiles (k_ising_tiles): the images the tile writes, and the one with what no update changes
    int8_t *spins_out;
    uint8_t *st_out;
    const uint8_t *cst;
    uint32_t tile_w, x0, y0;    // sites a tile's row holds; its first site (the tile wraps at the lattice's edge)
    uint32_t in_x, in_y;        // first column (in units) and row of the part the tile keeps
    uint32_t n_x, n_y;          // and its units per row and rows
};

// A tiled block of sweeps.
struct TileArgs {
    StripArgs s;
    uint32_t tiles_x, keep_w, keep_h, margin_x;  // of all tiles: kept sites per row and rows, columns before them
    uint32_t margin_y;
};

// LDS of a strip whose spins are bits: two words a thread, a zero, and the
// energy sums of a ring of sweeps.
constexpr uint32_t kBitsMaxThreads = 1024, kBitsRing = 512;
constexpr uint32_t kBitsLds = 8 * kBitsMaxThreads + 16 + 4 * kBitsRing;
// and XORWOW's Weyl words, one a unit (a thread's words an odd stride apart)
inline uint32_t bits_lds_bytes(rngx_kind kind, uint32_t threads, uint32_t slots) {
    return kBitsLds + (kind == RNGX_XORWOW ? 4 * threads * (slots + 1) : 0);
}

constexpr uint32_t kSpinLimit = 1u << 20;

// Halo words: 4 spins in the low half, the pass tag in the high half, both
// written by one 64-bit agent-scope atomic store, so a word read with the
// expected tag holds that pass's spins.  Polls one word until its tag is
// `tag`; gives up after kSpinLimit polls and records that in *err (once set,
// every later poll returns at once, so a failed exchange ends the kernel
// quickly with an invalid lattice instead of stalling it).
__device__ __forceinline__ uint32_t poll_word(const uint64_t *p, uint64_t v, uint32_t tag, uint32_t *err) {
    for (uint32_t it = 0; static_cast<uint32_t>(v >> 32) != tag; ++it) {
        if (it >= kSpinLimit || __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
            __hip_atomic_fetch_or(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            break;
        }
        __builtin_amdgcn_s_sleep(1);
        v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return static_cast<uint32_t>(v);
}

__device__ __forceinline__ void put_word(uint64_t *p, uint32_t spins, uint32_t tag) {
    __hip_atomic_store(p, (static_cast<uint64_t>(tag) << 32) | spins, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Acceptance in 32 bits.  With d = twice the number of a site's neighbours
// that differ from it (0, 2, .., 8), the flip is taken if d >= lo, else iff
// r < (d == 2 ? t4 : t8).  lo is 4 except when a threshold is 2^32 (every
// draw accepts), which 32 bits cannot hold: lo = 2 when that is T4, lo = 0
// when it is T8 (and then also T4, since T8 <= T4).
struct Accept {
    uint32_t t4, t8, lo;
};
__device__ __forceinline__ Accept make_accept(uint64_t T4, uint64_t T8) {
    constexpr uint64_t kAll = 1ull << 32;
    return Accept{T4 >= kAll ? 0xFFFFFFFFu : static_cast<uint32_t>(T4), T8 >= kAll ? 0xFFFFFFFFu : static_cast<uint32_t>(T8),
                  T8 >= kAll ? 0u : T4 >= kAll ? 2u : 4u};
}

// Whether every stream of strip r stands at the same position (Philox): then
// *p0 is that position.
__device__ inline bool strip_positions_equal(const StripArgs &a, uint32_t r, uint64_t *p0) {
    const uint64_t ubase = static_cast<uint64_t>(r) * a.R0 * (a.L / 4);
    const uint64_t *pos = reinterpret_cast<const uint64_t *>(a.st + 8 * a.S) + ubase;
    const uint64_t p = pos[0];
    int ok = 1;
    for (uint32_t k = threadIdx.x; k < a.units; k += blockDim.x) ok &= pos[k] == p;
    *p0 = p;
    return __syncthreads_and(ok) != 0;
}
// The same for a position that is a multiple of 4: *blk0 is its block.
__device__ inline bool strip_positions_aligned(const StripArgs &a, uint32_t r, uint64_t *blk0) {
    const bool same = strip_positions_equal(a, r, blk0);
    const bool aligned = (*blk0 & 3) == 0;
    *blk0 >>= 2;
    return same && aligned;
}

// Whether every XS1024W instance with a unit in strip r has taken the same
// number of steps: then *n0 is that count and *y_start the common Weyl word.
__device__ inline bool strip_steps_uniform(const StripArgs &a, uint32_t r, uint64_t *n0, uint32_t *y_start) {
    const uint64_t ubase = static_cast<uint64_t>(r) * a.R0 * (a.L / 8);
    const uint64_t *N = reinterpret_cast<const uint64_t *>(a.st + 4 * a.S);
    const uint64_t g0 = ubase >> 4, g1 = (ubase + a.units - 1) >> 4;
    const uint64_t n = N[g0];
    int ok = 1;
    for (uint64_t g = g0 + threadIdx.x; g <= g1; g += blockDim.x) ok &= N[g] == n;
    *n0 = n;
    *y_start = *reinterpret_cast<const uint32_t *>(a.st + 4 * a.S + 8 * (a.S / 32)) + static_cast<uint32_t>(n) * kWeylC;
    return __syncthreads_and(ok) != 0;
}

}  // namespace rngx
