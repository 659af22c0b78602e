// Seeding, bulk fill and consume kernels for all generator kinds.
//
// Fills are HBM-write-bound: each thread keeps its streams' state in VGPRs
// for the whole launch (loaded once, stored once) and writes output k of
// stream s to out[k*S + s], so a wavefront's stores cover one contiguous
// span per step.  Small-state kinds run V consecutive streams per thread
// (V = 4: one 16-byte store per step); XS1024W runs one instance per
// 16-lane DPP row with two words per lane (one 8-byte store per step).
#include <algorithm>

#include "rngx_internal.h"

namespace rngx {

namespace {

constexpr int kBlock = 256;
constexpr uint64_t kXsSync = 16;  // rows between its barriers when not paced (a power of two)
// --------------------------------------------------------------------------
// Seeding (definitions in rngx.h).
__global__ __launch_bounds__(kBlock) void k_seed_small(rngx_kind kind, uint8_t *st, uint64_t S, uint64_t seed) {
    const uint64_t s = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (s >= S) return;
    uint32_t *u32 = reinterpret_cast<uint32_t *>(st);
    uint64_t *u64 = reinterpret_cast<uint64_t *>(st);
    switch (kind) {
    case RNGX_LCG32: u32[s] = static_cast<uint32_t>(splitmix(seed, 1 + s)); break;
    case RNGX_LCG64: u64[s] = splitmix(seed, 1 + s); break;
    case RNGX_LCG32_SUB:
    case RNGX_LCG64_SUB: {
        // stream s at position s of the sequence from the plain stream-0 value;
        // the S-step map after the states
        const bool l32 = kind == RNGX_LCG32_SUB;
        const uint64_t a = l32 ? kLcg32A : kLcg64A, c = l32 ? kLcg32C : kLcg64C;
        const uint64_t g0 = l32 ? static_cast<uint32_t>(splitmix(seed, 1)) : splitmix(seed, 1);
        uint64_t A, C;
        affine_power(a, c, s, &A, &C);
        if (l32) u32[s] = static_cast<uint32_t>(A * g0 + C);
        else u64[s] = A * g0 + C;
        if (s == 0) {
            affine_power(a, c, S, &A, &C);
            if (l32) { u32[S] = static_cast<uint32_t>(A); u32[S + 1] = static_cast<uint32_t>(C); }
            else { u64[S] = A; u64[S + 1] = C; }
        }
        break;
    }
    case RNGX_MWC: {
        const uint64_t z = splitmix(seed, 1 + s);
        uint64_t x = z & 0xFFFFFFFFull, c = (z >> 32) % (kMwcA - 1);
        if (x == 0 && c == 0) x = 1;
        u64[s] = (c << 32) | x;
        break;
    }
    case RNGX_MWC_DIFF: {  // the multipliers are already in place after the states
        const uint64_t a = reinterpret_cast<const uint32_t *>(st + 8 * S)[s];
        const uint64_t z = splitmix(seed, 1 + s);
        uint64_t x = z & 0xFFFFFFFFull, c = (z >> 32) % (a - 1);
        if (x == 0 && c == 0) x = 1;
        u64[s] = (c << 32) | x;
        break;
    }
    case RNGX_XORWOW: {
        const uint64_t p = splitmix(seed, 1 + 3 * s), q = splitmix(seed, 2 + 3 * s), r = splitmix(seed, 3 + 3 * s);
        uint32_t w[6] = {static_cast<uint32_t>(p), static_cast<uint32_t>(p >> 32), static_cast<uint32_t>(q),
                         static_cast<uint32_t>(q >> 32), static_cast<uint32_t>(r), static_cast<uint32_t>(r >> 32)};
        if ((w[0] | w[1] | w[2] | w[3] | w[4]) == 0) w[0] = 1;
        for (int i = 0; i < 6; ++i) u32[i * S + s] = w[i];
        break;
    }
    case RNGX_PHILOX4X32_7:
    case RNGX_PHILOX4X32_10: {
        const uint64_t z = splitmix(seed, 1 + s);
        u32[s] = static_cast<uint32_t>(z);
        u32[S + s] = static_cast<uint32_t>(z >> 32);
        reinterpret_cast<uint64_t *>(st + 8 * S)[s] = 0;
        break;
    }
    default: break;
    }
}

// XS1024W: one thread per 64-bit seed word (two state words).  Among the 16
// words SM(1+16g .. 16+16g) of an instance at most one can be zero (mix64 is
// a bijection with mix64(0) = 0), so no instance is seeded all-zero.
__global__ __launch_bounds__(kBlock) void k_seed_xs(uint8_t *st, uint64_t S, uint64_t seed) {
    const uint64_t t = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;  // pair index
    const uint64_t G = S / 32;
    if (t >= 16 * G) return;
    const uint64_t z = splitmix(seed, 1 + t);  // t = 16 g + i/2
    reinterpret_cast<uint2 *>(st)[t] = make_uint2(static_cast<uint32_t>(z), static_cast<uint32_t>(z >> 32));
    if ((t & 15) == 0) reinterpret_cast<uint64_t *>(st + 4 * S)[t >> 4] = 0;
    if (t == 0) *reinterpret_cast<uint32_t *>(st + 4 * S + 8 * G) = static_cast<uint32_t>(splitmix(seed, 0) >> 32);
}

// --------------------------------------------------------------------------
// Output stores.
__device__ __forceinline__ float to_unit(uint32_t u) { return static_cast<float>(u >> 8) * 0x1.0p-24f; }

// Non-temporal stores: the outputs are streamed out and not read back by
// this kernel (XS1024W u32 fill at 2^20 x 4096: 6.30 -> 6.55 TB/s).  Plain ones
// (NT = false) where a thread's vectors are not whole lines, which the L2 puts
// together, and the output fits the memory-side cache: LCG32 99991 x 400 43 -> 39
// us on buffers taken in turn (38 -> 28 on one), but 300001 x 1000 (1.2 GB) 235 ->
// 258.  With one stream a thread, whose waves write whole lines, the two are
// alike at any size (LCG32, MWC, Philox and XORWOW, 300 sizes of 80 KB to 2.1 GB:
// 1.00 on average).
// A row of S words starts at any word when S is not a multiple of V; global
// stores of 2 and 4 words need no more than word alignment.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2), aligned(4)));

// The first n of V words (n = V: one store).
template <int MODE, int V, bool NT = true>
__device__ __forceinline__ void store_out(void *out, uint64_t idx, const uint32_t (&u)[V], uint32_t n = V) {
    uint32_t w[V];
    for (int v = 0; v < V; ++v) w[v] = MODE == kOutU32 ? u[v] : __float_as_uint(to_unit(u[v]));
    uint32_t *o = static_cast<uint32_t *>(out) + idx;
    if (n == V) {
        if constexpr (V == 4) {
            const u32x4 x = {w[0], w[1], w[2], w[3]};
            if constexpr (NT) __builtin_nontemporal_store(x, reinterpret_cast<u32x4 *>(o));
            else *reinterpret_cast<u32x4 *>(o) = x;
        } else if constexpr (V == 2) {
            const u32x2 x = {w[0], w[1]};
            __builtin_nontemporal_store(x, reinterpret_cast<u32x2 *>(o));
        } else {
            if constexpr (NT) __builtin_nontemporal_store(w[0], o);
            else *o = w[0];
        }
    } else {
        for (uint32_t v = 0; v < V; ++v)
            if (v < n) o[v] = w[v];
    }
}

// The state n outputs on, for the kinds that get there in a few dozen
// instructions.
template <class G> struct HasAdvance : std::false_type {};
template <> struct HasAdvance<Lcg32> : std::true_type {};
template <> struct HasAdvance<Lcg64> : std::true_type {};
template <> struct HasAdvance<Lcg32Sub> : std::true_type {};
template <> struct HasAdvance<Lcg64Sub> : std::true_type {};
template <> struct HasAdvance<Mwc> : std::true_type {};
template <> struct HasAdvance<MwcDiff> : std::true_type {};
template <int ROUNDS> struct HasAdvance<PhiloxR<ROUNDS>> : std::true_type {};

// The multiplier (MWC: a^n mod p) and increment of n steps, the same for all
// streams of a fill but MWC_DIFF's and the sub-stream LCGs', which the device
// works out.
struct RowMap {
    uint64_t a, c;
};
template <class G>
__device__ __forceinline__ RowMap row_map(const G &g, uint64_t n) {
    RowMap m{1, 0};
    if constexpr (std::is_same<G, Lcg32>::value) affine_power(kLcg32A, kLcg32C, n, &m.a, &m.c);
    else if constexpr (std::is_same<G, Lcg64>::value) affine_power(kLcg64A, kLcg64C, n, &m.a, &m.c);
    else if constexpr (std::is_same<G, Lcg32Sub>::value || std::is_same<G, Lcg64Sub>::value) affine_power(g.A, g.C, n, &m.a, &m.c);
    else if constexpr (std::is_same<G, Mwc>::value) {
        uint64_t b = kMwcA;
        for (; n; n >>= 1) {
            if (n & 1) m.a = mwc_mulmod(m.a, b);
            b = mwc_mulmod(b, b);
        }
    }
    return m;
}
template <class G>
__device__ __forceinline__ void advance(G &g, const RowMap &m, uint64_t n) {
    if constexpr (std::is_same<G, Mwc>::value) g.y = mwc_mulmod(g.y, m.a);
    else if constexpr (std::is_same<G, MwcDiff>::value) g.y = mwc_jump_mod(g.y, g.a, n);
    else g.x = static_cast<decltype(g.x)>(m.a * g.x + m.c);
}
template <int ROUNDS>
__device__ __forceinline__ void advance(PhiloxR<ROUNDS> &g, const RowMap &, uint64_t n) {
    g.pos += n;
    if (g.pos & 3) philox_block<ROUNDS>(g.k0, g.k1, g.pos >> 2, g.b0, g.b1, g.b2, g.b3);  // resume mid-block
}

// Small-state kinds: V consecutive streams per thread.  With SPLIT, row block
// blockIdx.y of `rows` rows: its threads start from their streams' states
// blockIdx.y * rows outputs on (a fill of few streams and many rows would
// otherwise run a few long chains).  The row blocks of a group of streams count
// themselves in arrived[blockIdx.x] once their states are loaded; the one that
// comes last writes the states after the fill, and a zero for the next fill.
template <class G, int MODE, int V, bool SPLIT, bool NT, bool WHOLE = false>
__global__ __launch_bounds__(kBlock) void k_fill_small(uint8_t *st, uint64_t S, uint64_t count, void *out,
                                                       uint64_t rows, uint32_t *arrived) {
    const uint64_t s0 = (static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x) * V;
    if (!SPLIT && s0 >= S) return;
    // WHOLE: V divides S (a tail tested for in every row: LCG32 2^20 x 8 9.1 us, without 7.6)
    const uint32_t live = WHOLE || (V == 1 && !SPLIT) ? V : s0 < S ? static_cast<uint32_t>(min(static_cast<uint64_t>(V), S - s0)) : 0;
    G g[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        if constexpr (!WHOLE && (V > 1 || SPLIT)) g[v] = G{};
        if (v < live) g[v].load(st, S, s0 + v);
    }
    uint64_t k = 0, end = count;
    if constexpr (SPLIT) {
        k = blockIdx.y * rows;
        end = min(count, k + rows);
        __shared__ uint32_t last;
        __builtin_amdgcn_s_waitcnt(0x0F70);  // the loads are complete
        __syncthreads();
        if (threadIdx.x == 0)
            last = __hip_atomic_fetch_add(arrived + blockIdx.x, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.y - 1;
        __syncthreads();
        if (last) {
            const RowMap m = row_map(g[0], count);
#pragma unroll
            for (int v = 0; v < V; ++v) {
                G f = g[v];
                if (v < live) {
                    advance(f, m, count);
                    f.store(st, S, s0 + v);
                }
            }
            if (threadIdx.x == 0) arrived[blockIdx.x] = 0;
        }
        if (!live) return;
        if (k) {
            const RowMap m = row_map(g[0], k);
#pragma unroll
            for (int v = 0; v < V; ++v)
                if (v < live) advance(g[v], m, k);
        }
    }
    uint32_t acc[V];
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] = 0;
    auto emit = [&](uint64_t row, const uint32_t (&u)[V]) {
        if constexpr (MODE == kOutXor) {
#pragma unroll
            for (int v = 0; v < V; ++v) acc[v] ^= u[v];
        } else {
            store_out<MODE, V, NT>(out, row * S + s0, u, live);
        }
    };
    if constexpr (HasNext8<G>::value) {  // 8 outputs of each stream at a time
        for (; k + 8 <= end; k += 8) {
            uint32_t d[V][8];
#pragma unroll
            for (int v = 0; v < V; ++v) g[v].next8(d[v]);
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {
                uint32_t u[V];
#pragma unroll
                for (int v = 0; v < V; ++v) u[v] = d[v][kk];
                emit(k + kk, u);
            }
        }
    }
    for (; k < end; ++k) {
        uint32_t u[V];
#pragma unroll
        for (int v = 0; v < V; ++v) u[v] = g[v].next();
        emit(k, u);
    }
    if constexpr (!SPLIT) {
#pragma unroll
        for (int v = 0; v < V; ++v)
            if (v < live) g[v].store(st, S, s0 + v);
    }
    if constexpr (MODE == kOutXor) {
        uint32_t *o = static_cast<uint32_t *>(out);
#pragma unroll
        for (int v = 0; v < V; ++v)
            if (v < live) o[s0 + v] = acc[v];
    }
}

// Small-state kinds, paced: V consecutive streams per thread, BLK threads
// per workgroup (threads past the last stream stay in the loop with their
// stores masked, since they take part in the barriers).
template <class G, int MODE, int V, int BLK, bool WHOLE>
__global__ __launch_bounds__(BLK) void k_fill_paced(uint8_t *st, uint64_t S, uint64_t count, void *out,
                                                    uint32_t *ring) {
    const uint64_t s0 = (static_cast<uint64_t>(blockIdx.x) * BLK + threadIdx.x) * V;
    // streams of the thread: V or none where V divides S (WHOLE)
    const uint32_t live = s0 >= S ? 0 : WHOLE ? V : static_cast<uint32_t>(min(static_cast<uint64_t>(V), S - s0));
    G g[V];
#pragma unroll
    for (int v = 0; v < V; ++v)
        if (WHOLE ? live != 0 : v < live) g[v].load(st, S, s0 + v);
    __shared__ uint32_t s_free;
    Pacer pc(ring);
    for (uint64_t k0 = 0, band = 0; k0 < count; k0 += kBand, ++band) {
        pc.before(band, &s_free);
        auto row = [&](uint64_t k) {
            uint32_t u[V];
#pragma unroll
            for (int v = 0; v < V; ++v) u[v] = g[v].next();
            if (live) store_out<MODE, V>(out, k * S + s0, u, WHOLE ? V : live);
        };
        const uint64_t k1 = k0 + kBand < count ? k0 + kBand : count;
        if (k1 - k0 == kBand) {
            if constexpr (HasNext8<G>::value) {  // a band is 8 outputs of each stream
                static_assert(kBand == 8, "next8 covers one band");
                uint32_t d[V][8];
#pragma unroll
                for (int v = 0; v < V; ++v) g[v].next8(d[v]);
#pragma unroll
                for (uint32_t kk = 0; kk < kBand; ++kk) {
                    uint32_t u[V];
#pragma unroll
                    for (int v = 0; v < V; ++v) u[v] = d[v][kk];
                    if (live) store_out<MODE, V>(out, (k0 + kk) * S + s0, u, WHOLE ? V : live);
                }
            } else {
#pragma unroll
                for (uint32_t kk = 0; kk < kBand; ++kk) row(k0 + kk);
            }
        } else {
            for (uint64_t k = k0; k < k1; ++k) row(k);
        }
        pc.after(band);
    }
#pragma unroll
    for (int v = 0; v < V; ++v)
        if (WHOLE ? live != 0 : v < live) g[v].store(st, S, s0 + v);
}

// XS1024W: thread t runs lane j = t % 16 of instance g = t / 16.  The output
// is written row by row across all streams.  How fast HBM takes these rows
// depends on how many distinct rows the chip writes at once, i.e. on how far
// the workgroups drift apart, so a paced launch (ring != null, whole grid
// resident) keeps them together: rows go in bands of kBand, and before band b
// a workgroup waits until every workgroup has finished band b - kSlack.
// Completion is counted in a ring of kRing band entries of kPaceSlots
// counters (workgroup w adds 1 to slot w % kPaceSlots), so that no counter is
// hit by more than a few workgroups; an entry's target after its u-th use is
// u times the workgroups of its slot (Pacer).  Waits are bounded: a workgroup
// that waited kPollLimit polls runs free for the rest of the launch.  Pacing
// only decides when a row is written, never what is written.  Unpaced launches
// meet at a block barrier every kXsSync rows instead.  Rows past the last
// instance stay in the loop with their loads and stores masked, since every
// wave of the block has to reach each barrier; they are whole 16-lane rows,
// so no active instance sees one of their words.
template <int MODE, int BLK>
__global__ __launch_bounds__(BLK) void k_fill_xs(uint8_t *st, uint64_t S, uint64_t count, void *out,
                                                 uint32_t *ring) {
    const uint64_t t = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const uint64_t G = S / 32, g = t >> 4;
    const bool live = g < G;
    if (MODE == kOutXor && !live) return;                 // no barriers in this mode
    uint2 *W = reinterpret_cast<uint2 *>(st);
    uint64_t *N = reinterpret_cast<uint64_t *>(st + 4 * S);
    const uint32_t y0 = *reinterpret_cast<const uint32_t *>(st + 4 * S + 8 * G);
    const uint2 w = live ? W[t] : make_uint2(0, 0);
    uint32_t a = w.x, b = w.y;
    const uint64_t n = live ? N[g] : 0;
    uint32_t y = y0 + static_cast<uint32_t>(n) * kWeylC;
    uint32_t acc0 = 0, acc1 = 0;
    __shared__ uint32_t s_free;
    Pacer pc(MODE != kOutXor ? ring : nullptr);
    for (uint64_t k0 = 0, band = 0; k0 < count; k0 += kBand, ++band) {
        if constexpr (MODE != kOutXor) pc.before(band, &s_free);
        auto row = [&](uint64_t k) {
            xs1024_step(a, b);
            y += kWeylC;
            const uint32_t m = weyl_mix(y);
            const uint32_t u[2] = {a + m, b + m};
            if constexpr (MODE == kOutXor) {
                acc0 ^= u[0];
                acc1 ^= u[1];
            } else {
                if (live) store_out<MODE, 2>(out, k * S + 2 * t, u);
            }
        };
        const uint64_t k1 = k0 + kBand < count ? k0 + kBand : count;
        if (k1 - k0 == kBand) {
#pragma unroll
            for (uint32_t kk = 0; kk < kBand; ++kk) row(k0 + kk);
        } else {
            for (uint64_t k = k0; k < k1; ++k) row(k);
        }
        if constexpr (MODE != kOutXor) {
            if (pc.ring) pc.after(band);
            else if ((k1 & (kXsSync - 1)) == 0) __syncthreads();
        }
    }
    if (!live) return;
    W[t] = make_uint2(a, b);
    if ((t & 15) == 0) N[g] = n + count;
    if constexpr (MODE == kOutXor) reinterpret_cast<uint2 *>(out)[t] = make_uint2(acc0, acc1);
}

__global__ __launch_bounds__(kBlock) void k_zero_ring(uint32_t *ring) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < kRing * kPaceSlots) ring[i] = 0;
}

// ---------------------------------------------------------------- configurations
// The fill configurations the autotuner chooses from; every one of them
// produces the same values.  Small-state kinds: paced or not, streams per
// thread, threads per workgroup (the unpaced one is k_fill_small).
// XS1024W: always one lane pair per thread; paced or not, threads per
// workgroup.  The first entry of each list is the default (XORWOW: the
// second), as measured at 2^20 streams x 4096.
constexpr rngx_fill_config kSmallConfigs[] = {{1, 4, 512}, {1, 4, 1024}, {1, 4, 256}, {1, 2, 1024},
                                              {1, 2, 512}, {1, 2, 256},  {0, 4, 256}};
constexpr rngx_fill_config kXsConfigs[] = {{1, 2, 1024}, {1, 2, 512}, {0, 2, 1024}, {0, 2, 256}};
// Lagged Fibonacci kinds: one wave per 1024-stream instance (16 streams per
// lane), four waves per workgroup, free-running.
constexpr rngx_fill_config kLfgConfigs[] = {{1, 16, 256}, {0, 16, 256}};
constexpr int kNumSmall = sizeof(kSmallConfigs) / sizeof(kSmallConfigs[0]);
constexpr int kNumXs = sizeof(kXsConfigs) / sizeof(kXsConfigs[0]);
static_assert(kNumSmall < kMaxFillConfigs && kNumXs <= kMaxFillConfigs, "Gen::resident too small");

int default_config(rngx_kind kind) { return kind == RNGX_XORWOW ? 1 : 0; }

// Kernel of a configuration (U32 or F32), for launches and occupancy.  Where V
// does not divide S only the default configurations have one.
template <class G, int MODE>
const void *paced_kernel(int v, int blk, bool whole) {
    constexpr int kDefaultBlk = std::is_same<G, Xorwow>::value ? 1024 : 512;
    if (!whole) return v == 4 && blk == kDefaultBlk ? reinterpret_cast<const void *>(&k_fill_paced<G, MODE, 4, kDefaultBlk, false>) : nullptr;
    if (v == 4 && blk == 256) return reinterpret_cast<const void *>(&k_fill_paced<G, MODE, 4, 256, true>);
    if (v == 4 && blk == 512) return reinterpret_cast<const void *>(&k_fill_paced<G, MODE, 4, 512, true>);
    if (v == 4 && blk == 1024) return reinterpret_cast<const void *>(&k_fill_paced<G, MODE, 4, 1024, true>);
    if (v == 2 && blk == 256) return reinterpret_cast<const void *>(&k_fill_paced<G, MODE, 2, 256, true>);
    if (v == 2 && blk == 512) return reinterpret_cast<const void *>(&k_fill_paced<G, MODE, 2, 512, true>);
    if (v == 2 && blk == 1024) return reinterpret_cast<const void *>(&k_fill_paced<G, MODE, 2, 1024, true>);
    return nullptr;
}
template <int MODE>
const void *xs_kernel(int blk) {
    if (blk == 256) return reinterpret_cast<const void *>(&k_fill_xs<MODE, 256>);
    if (blk == 512) return reinterpret_cast<const void *>(&k_fill_xs<MODE, 512>);
    if (blk == 1024) return reinterpret_cast<const void *>(&k_fill_xs<MODE, 1024>);
    return nullptr;
}
template <class G>
const void *config_kernel(int mode, const rngx_fill_config &c, bool whole) {
    return mode == kOutU32 ? paced_kernel<G, kOutU32>(c.streams_per_thread, c.block, whole)
                           : paced_kernel<G, kOutF32>(c.streams_per_thread, c.block, whole);
}
const void *config_kernel(rngx_kind kind, int mode, const rngx_fill_config &c, bool whole) {
    switch (kind) {
    case RNGX_LCG32: return config_kernel<Lcg32>(mode, c, whole);
    case RNGX_LCG64: return config_kernel<Lcg64>(mode, c, whole);
    case RNGX_MWC: return config_kernel<Mwc>(mode, c, whole);
    case RNGX_MWC_DIFF: return config_kernel<MwcDiff>(mode, c, whole);
    case RNGX_XORWOW: return config_kernel<Xorwow>(mode, c, whole);
    case RNGX_PHILOX4X32_10: return config_kernel<Philox>(mode, c, whole);
    case RNGX_PHILOX4X32_7: return config_kernel<Philox7>(mode, c, whole);
    case RNGX_LCG32_SUB: return config_kernel<Lcg32Sub>(mode, c, whole);
    case RNGX_LCG64_SUB: return config_kernel<Lcg64Sub>(mode, c, whole);
    case RNGX_XS1024W: return mode == kOutU32 ? xs_kernel<kOutU32>(c.block) : xs_kernel<kOutF32>(c.block);
    default: break;  // lagged Fibonacci kinds have their own kernel
    }
    return nullptr;
}

// Workgroups of configuration i that fit on the device at once (cached; the
// last entry is the default's kernel for an S that V does not divide).
uint32_t resident(Gen *g, int i, const rngx_fill_config &c, bool whole) {
    int &known = g->resident[whole ? i : kMaxFillConfigs - 1];
    if (known >= 0) return static_cast<uint32_t>(known);
    int u = 0, f = 0;
    const void *ku = config_kernel(g->kind, kOutU32, c, whole), *kf = config_kernel(g->kind, kOutF32, c, whole);
    if (!ku || !kf || hipOccupancyMaxActiveBlocksPerMultiprocessor(&u, ku, c.block, 0) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&f, kf, c.block, 0) != hipSuccess) {
        (void)hipGetLastError();
        u = f = 0;
    }
    known = std::min(u, f) * std::max(g->n_cu, 0);
    return static_cast<uint32_t>(known);
}

// Pace a launch of `blocks` workgroups of configuration i: large enough and
// every workgroup resident at once.
bool pace_ok(Gen *g, int i, const rngx_fill_config &c, uint64_t blocks, uint64_t count, bool whole = true) {
    return g->d_ring && count >= 4 * kBand && blocks >= 128 && blocks <= resident(g, i, c, whole);
}
// Where V does not divide S (rows unaligned, a test for the tail in every
// store), pacing pays later for the kinds with long chains or 8 rows at once: us
// with one stream a thread and paced, Philox4x32-10 300001 x 33 15 and 24, x 64 33
// and 25, x 200 112 and 64; XORWOW 524290 x 33 23 and 28, x 64 51 and 39.  LCG32
// 524290 x 33 22 and 17.
template <class G>
bool pace_ragged(uint64_t S, uint64_t count) {
    if (HasNext8<G>::value) return S * count >= 1ull << 24;
    return HasAdvance<G>::value || count >= 48;
}

void clear_ring(Gen *g, hipStream_t st) {
    hipLaunchKernelGGL(k_zero_ring, dim3((kRing * kPaceSlots + kBlock - 1) / kBlock), dim3(kBlock), 0, st, g->d_ring);
}

// Row blocks: as many as make kSplitWaves waves (two per SIMD), of at least
// split_rows rows each, about where a block's rows cost as much as the way to
// its first one: LCG32 1024 x 4096 285 -> 10 us, Philox4x32-10 4096 x 1000 220 ->
// 11.  (The arrival count is relaxed on purpose: its loads are waited for, and an
// ordered one writes back the L2 in every workgroup, 33 -> 43 us for Philox4x32-10
// FP32 99991 x 400.)
constexpr uint64_t kSplitWaves = 2048, kCached = 256ull << 20;
template <class G>
constexpr uint64_t split_rows() {
    if (HasNext8<G>::value) return 32;
    if (std::is_same<G, MwcDiff>::value) return 512;  // a power modulo each stream's own p
    return std::is_same<G, Mwc>::value ? 128 : 64;
}
template <class G>
uint64_t row_blocks(uint64_t waves, uint64_t count) {
    if (!HasAdvance<G>::value) return 1;
    return std::max<uint64_t>(1, std::min(kSplitWaves / waves, count / split_rows<G>()));
}

// An unpaced fill: V streams a thread, in `by` row blocks, with non-temporal
// stores or plain ones; or (bands) by the kernel of the kind's default
// configuration without its pacing.
struct FreeShape {
    int V;
    uint64_t by;
    bool nt, bands;
};
// Streams a thread: one where few streams or short fills leave the chip short
// of waves (a wave's row store is then 256 bytes, but four times as many waves
// hide the chain of a row), four otherwise.  Rows of whole vectors (S % 4 == 0)
// in bands of 8 unrolled rows where many streams are filled in few rows.  The
// lines below were drawn by timing each of these for 7 kinds, 27 stream counts of
// 20000 to 2^24 and 13 row counts of 1 to 4000 (outputs up to 4 GB, buffers
// taken in turn); us as (one stream, four, bands).
template <class G>
FreeShape free_shape(uint64_t S, uint64_t count) {
    constexpr bool kPhilox = HasNext8<G>::value, kXorwow = !HasAdvance<G>::value;
    const bool whole = S % 4 == 0, pages = S % 1024 == 0;
    const uint64_t n = S * count, waves = ((S + 3) / 4 + 63) / 64, by4 = row_blocks<G>(waves, count);
    const FreeShape one{1, row_blocks<G>((S + 63) / 64, count), false, false}, one_nt{1, 1, true, false};
    const FreeShape four{4, 1, whole || 4 * n > kCached, false}, bands{4, 1, true, true};
    if (kPhilox) {
        // Registers are what holds waves back, so whole lines in a row go one
        // stream a thread: 2^20 x 1024 (785, 945, 907); but 7 rounds 2^23 x 64
        // (453, 420, 425), 2^24 x 8 (161, -, 214).
        if (S < 1ull << 16 || S % 32 == 0)
            return std::is_same<G, Philox7>::value && S > 1ull << 21 && count >= 16 && n >= 1ull << 26 ? bands : one;
        if (n < 1ull << 23) return one;                     // 1032178 x 4 (8, 13, 13)
        if (whole) return n >= 1ull << 26 ? bands : four;   // 4194308 x 8 (43, 48, 50), x 128 (-, 762, 727)
        // 524290 x 31 (20, 30, -), 700001 x 31 (29, 36, -), 1032178 x 24 (34, 28, -), x 31 (50, 37, -); 3000001 x 16
        // (60, 71, -), x 24 (89, 75, -)
        if (S >= 1ull << 18) return n < 24'000'000 || (S > 1ull << 21 && count < 24) ? one_nt : four;
        // 131073 x 64 (13, 21, -), x 200 (36, 37, -), x 400 (74, 55, -)
        return count < 256 && n < 1ull << 25 ? one_nt : FreeShape{4, by4, four.nt, false};
    }
    if (kXorwow) {  // its rows cannot be split: 131073 x 500 (80, 110, -)
        if (S < 1ull << 19) return FreeShape{1, 1, false, false};
        if (n < 1ull << 24) return one_nt;  // states fill the L2 themselves: 1032178 x 4 10, plain stores 11, four 14
        if (whole)  // 2^22 x 16 (68, 81, 75), 2^24 x 31 (564, 658, 564), 2^20 x 24 (25, 28, 30), 3000000 x 24 (62, 66, 71)
            return S >= 1ull << 21 && count >= 16 && (pages || (S >= 1ull << 22 && count < 32)) ? bands : four;
        return count < 24 ? one_nt : four;  // 3000001 x 16 (62, 67, -), 1032178 x 24 (39, 32, -)
    }
    if (S < 1ull << 16) return one;  // LCG32 FP32 20001 x 300 (8, 16, -)
    // LCG32 100002 x 64 (7, 14, -); states of 8 bytes 2^22 x 1 (15, 13, 12)
    if (n < 1ull << 23) return whole && S >= 1ull << 22 ? bands : one;
    if (whole) {
        if (waves < 512) return FreeShape{4, by4, true, false};
        // LCG32 200000 x 400: row blocks 60, without 54, bands 59; 2^20 x 16 (-, 15, 13), 2^22 x 64 (-, 250, 237),
        // 2^24 x 64 (-, 780, 870), 3000000 x 24 (-, 47, 49), 4194308 x 24 (-, 130, 126)
        return S >= 1ull << 20 && ((pages && n < 1ull << 30) || (S >= 1ull << 22 && count < 32)) ? bands : four;
    }
    // Fewer than three waves a CU: MWC 65537 x 200 (15, 31, -), 99991 x 200 (22, 38, -); two are enough for long
    // columns: 131073 x 64 (11, 13, -), x 400 (66, 53, -)
    if (waves * by4 < 768 && (waves < 512 || count < 256)) return one_nt;
    return FreeShape{4, waves < 640 ? by4 : 1, four.nt, false};  // 200001 x 400: two row blocks 83, one 74
}

template <class G, int MODE, int V, bool NT, bool WHOLE = false>
hipError_t fill_free(Gen *g, void *out, uint64_t count, uint64_t by, hipStream_t st) {
    const uint64_t S = g->S;
    const uint64_t blocks = ((S + V - 1) / V + kBlock - 1) / kBlock;
    if constexpr (MODE != kOutXor && HasAdvance<G>::value && !(V == 1 && NT)) {
        if (by > 1 && g->d_ring && blocks <= kSplitGroups) {
            const uint64_t rows = ((count + by - 1) / by + 7) / 8 * 8;
            hipLaunchKernelGGL((k_fill_small<G, MODE, V, true, NT>),
                               dim3(static_cast<unsigned>(blocks), static_cast<unsigned>((count + rows - 1) / rows)),
                               dim3(kBlock), 0, st, g->d_state, S, count, out, rows, g->d_ring + kRing * kPaceSlots);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_fill_small<G, MODE, V, false, NT, WHOLE>), dim3(static_cast<unsigned>(blocks)), dim3(kBlock), 0, st,
                       g->d_state, S, count, out, count, static_cast<uint32_t *>(nullptr));
    return hipGetLastError();
}

template <class G, int MODE>
hipError_t fill_small(Gen *g, void *out, uint64_t count, hipStream_t st) {
    const uint64_t S = g->S;
    if constexpr (MODE != kOutXor) {
        const bool set = g->fill_cfg >= 0;
        const int i = set ? g->fill_cfg : default_config(g->kind);
        const rngx_fill_config c = kSmallConfigs[i];
        const int V = c.streams_per_thread;
        const bool whole = S % V == 0;
        const uint64_t blocks = ((S + V - 1) / V + c.block - 1) / c.block;
        const void *fn = c.paced ? config_kernel<G>(MODE, c, whole) : nullptr;
        const bool pace = fn && (whole || pace_ragged<G>(S, count)) && pace_ok(g, i, c, blocks, count, whole);
        // a configuration the caller chose is run as it is, paced or not, where its vectors divide a row
        const FreeShape f = set && whole ? FreeShape{4, 1, true, c.paced != 0} : free_shape<G>(S, count);
        if (pace || f.bands) {
            if (pace) clear_ring(g, st);
            uint32_t *ring = pace ? g->d_ring : nullptr;
            void *args[] = {&g->d_state, const_cast<uint64_t *>(&S), &count, &out, &ring};
            const hipError_t e = hipLaunchKernel(fn, dim3(static_cast<unsigned>(blocks)), dim3(c.block), args, 0, st);
            return e != hipSuccess ? e : hipGetLastError();
        }
        if (f.V == 1) return f.nt ? fill_free<G, MODE, 1, true>(g, out, count, 1, st) : fill_free<G, MODE, 1, false>(g, out, count, f.by, st);
        if (S % 4 == 0) return fill_free<G, MODE, 4, true, true>(g, out, count, f.by, st);
        return f.nt ? fill_free<G, MODE, 4, true>(g, out, count, f.by, st) : fill_free<G, MODE, 4, false>(g, out, count, f.by, st);
    } else {
        // Nothing to store: four times the waves hide a stream's chain of steps
        // (512 rows, four streams a thread and one: LCG32 2^12 streams 22 and 13
        // us, 2^18 36 and 18, 2^19 30 and 30, 2^20 45 and 51; MWC 2^18 29 and 21),
        // and of the sizes that fill no whole round of workgroups the smaller
        // ones lose less (Philox4x32-10 2^19 + 1 130 and 85).
        if (S < 1ull << 19 || (S % 4 && S < 1ull << 21)) return fill_free<G, MODE, 1, false>(g, out, count, 1, st);
        if (S % 4 == 0) return fill_free<G, MODE, 4, true, true>(g, out, count, 1, st);
        return fill_free<G, MODE, 4, true>(g, out, count, 1, st);
    }
}

template <int MODE>
hipError_t fill_xs(Gen *g, void *out, uint64_t count, hipStream_t st) {
    const int i = MODE == kOutXor ? 2 : (g->fill_cfg >= 0 ? g->fill_cfg : default_config(g->kind));
    const rngx_fill_config c = kXsConfigs[i];
    const uint64_t blocks = (g->S / 2 + c.block - 1) / c.block;
    const bool pace = MODE != kOutXor && c.paced && pace_ok(g, i, c, blocks, count);
    if (pace) clear_ring(g, st);
    uint32_t *ring = pace ? g->d_ring : nullptr;
    const void *fn = MODE == kOutXor ? reinterpret_cast<const void *>(&k_fill_xs<kOutXor, 1024>) : xs_kernel<MODE>(c.block);
    void *args[] = {&g->d_state, &g->S, &count, &out, &ring};
    const hipError_t e = hipLaunchKernel(fn, dim3(static_cast<unsigned>(blocks)), dim3(c.block), args, 0, st);
    return e != hipSuccess ? e : hipGetLastError();
}

template <int MODE>
hipError_t fill_mode(Gen *g, void *out, uint64_t count, hipStream_t st) {
    switch (g->kind) {
    case RNGX_LCG32: return fill_small<Lcg32, MODE>(g, out, count, st);
    case RNGX_LCG64: return fill_small<Lcg64, MODE>(g, out, count, st);
    case RNGX_MWC: return fill_small<Mwc, MODE>(g, out, count, st);
    case RNGX_MWC_DIFF: return fill_small<MwcDiff, MODE>(g, out, count, st);
    case RNGX_XORWOW: return fill_small<Xorwow, MODE>(g, out, count, st);
    case RNGX_PHILOX4X32_10: return fill_small<Philox, MODE>(g, out, count, st);
    case RNGX_PHILOX4X32_7: return fill_small<Philox7, MODE>(g, out, count, st);
    case RNGX_LCG32_SUB: return fill_small<Lcg32Sub, MODE>(g, out, count, st);
    case RNGX_LCG64_SUB: return fill_small<Lcg64Sub, MODE>(g, out, count, st);
    case RNGX_XS1024W: return fill_xs<MODE>(g, out, count, st);
    default: break;
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_seed(Gen *g, uint64_t seed, hipStream_t st) {
    if (is_lfg(g->kind)) return launch_seed_lfg(g, seed, st);
    if (g->kind == RNGX_XS1024W) {
        const uint64_t pairs = g->S / 2;
        const unsigned blocks = static_cast<unsigned>((pairs + kBlock - 1) / kBlock);
        hipLaunchKernelGGL(k_seed_xs, dim3(blocks), dim3(kBlock), 0, st, g->d_state, g->S, seed);
    } else {
        if (g->kind == RNGX_MWC_DIFF) {
            const hipError_t e = mwc_diff_multipliers(g->S, reinterpret_cast<uint32_t *>(g->d_state + 8 * g->S), st);
            if (e != hipSuccess) return e;
        }
        const unsigned blocks = static_cast<unsigned>((g->S + kBlock - 1) / kBlock);
        hipLaunchKernelGGL(k_seed_small, dim3(blocks), dim3(kBlock), 0, st, g->kind, g->d_state, g->S, seed);
    }
    return hipGetLastError();
}

hipError_t launch_clear_ring(Gen *g, hipStream_t st) {
    clear_ring(g, st);
    return hipGetLastError();
}

hipError_t fill_setup(Gen *g, int n_cu) {
    g->d_ring = nullptr;
    g->n_cu = n_cu;
    g->fill_cfg = -1;
    for (int i = 0; i < kMaxFillConfigs; ++i) g->resident[i] = -1;
    // pacing counters (each paced fill clears them), then k_fill_small's (zero between fills)
    const hipError_t e = hipMalloc(&g->d_ring, 4ull * (kRing * kPaceSlots + kSplitGroups));
    return e != hipSuccess ? e : launch_zero(g->d_ring + kRing * kPaceSlots, kSplitGroups, nullptr);
}

int fill_configs(rngx_kind kind, const rngx_fill_config **list) {
    if (is_lfg(kind)) { *list = kLfgConfigs; return 2; }
    *list = kind == RNGX_XS1024W ? kXsConfigs : kSmallConfigs;
    return kind == RNGX_XS1024W ? kNumXs : kNumSmall;
}

int fill_default(rngx_kind kind) { return default_config(kind); }

hipError_t launch_fill(Gen *g, void *d_out, uint64_t count, int mode, hipStream_t st) {
    if (is_lfg(g->kind)) return launch_fill_lfg(g, d_out, count, mode, st);
    if (mode == kOutU32) return fill_mode<kOutU32>(g, d_out, count, st);
    if (mode == kOutF32) return fill_mode<kOutF32>(g, d_out, count, st);
    return fill_mode<kOutXor>(g, d_out, count, st);
}

}  // namespace rngx
