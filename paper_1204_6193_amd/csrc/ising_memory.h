// Ising updates that keep spins and states in global memory, and what the
// batch kernels share: replica descriptors and the start of a gang.
#pragma once

#include "ising_device.h"

namespace rngx {

constexpr uint64_t kOnes8 = 0x0101010101010101ull;

// Bytewise count (0..4) of neighbours that differ from each site of an
// NB-site run w; up/dn are the runs above and below, lb/rb the spins left of
// byte 0 and right of byte NB-1.
template <int NB>
__device__ __forceinline__ uint64_t mismatches(uint64_t w, uint64_t up, uint64_t dn, uint32_t lb, uint32_t rb) {
    constexpr uint64_t M = NB == 8 ? kOnes8 : 0x01010101ull;
    const uint64_t nw = (w >> 1) & M, nu = (up >> 1) & M, nd = (dn >> 1) & M;
    const uint64_t nl = ((nw << 8) | ((lb >> 1) & 1u)) & M;
    const uint64_t nr = (nw >> 8) | (static_cast<uint64_t>((rb >> 1) & 1u) << (8 * (NB - 1)));
    return (nu ^ nw) + (nd ^ nw) + (nl ^ nw) + (nr ^ nw);
}

// Metropolis decision for byte i; returns s_i h_i after the update.  Written
// without branches: the flip is a masked xor and the result a select.
__device__ __forceinline__ int metropolis(uint64_t &w, uint64_t m, int i, uint32_t r, uint64_t T4, uint64_t T8) {
    const uint32_t mi = static_cast<uint32_t>(m >> (8 * i)) & 0xFFu;
    const uint64_t thr = mi == 1 ? T4 : T8;
    const uint32_t acc = static_cast<uint32_t>(mi >= 2) | static_cast<uint32_t>(static_cast<uint64_t>(r) < thr);
    w ^= static_cast<uint64_t>(acc * 0xFEu) << (8 * i);
    const int e = 2 * static_cast<int>(mi) - 4;
    return acc ? e : -e;
}

// One Metropolis update of a site with mi (0..4) differing neighbours and
// draw r (multi-hit updates: the site's neighbours stay fixed between its
// hits); a taken flip turns mi into 4 - mi and toggles `flip`.
__device__ __forceinline__ void hit_mem(uint32_t &mi, uint32_t &flip, uint32_t r, uint64_t T4, uint64_t T8) {
    const uint64_t thr = mi == 1 ? T4 : T8;
    const bool acc = (mi >= 2) | (static_cast<uint64_t>(r) < thr);
    mi = acc ? 4 - mi : mi;
    flip ^= acc ? 1u : 0u;
}

template <int NB>
__device__ __forceinline__ uint64_t lds_run(const uint8_t *p) {
    if constexpr (NB == 8) return *reinterpret_cast<const uint64_t *>(p);
    else return *reinterpret_cast<const uint32_t *>(p);
}
template <int NB>
__device__ __forceinline__ void lds_put(uint8_t *p, uint64_t w) {
    if constexpr (NB == 8) *reinterpret_cast<uint64_t *>(p) = w;
    else *reinterpret_cast<uint32_t *>(p) = static_cast<uint32_t>(w);
}

// Sum of v over the block (result valid in thread 0).
__device__ __forceinline__ int block_sum(int v, int *scratch) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    const uint32_t w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    if ((threadIdx.x & 63) == 0) scratch[w] = v;
    __syncthreads();
    int s = 0;
    if (threadIdx.x == 0)
        for (uint32_t i = 0; i < nw; ++i) s += scratch[i];
    __syncthreads();
    return s;
}

// Update unit k of colour c with spins and state in global memory; returns
// the sum of s*h over the updated sites.  A unit reads only other-colour
// bytes of its neighbour runs, which no thread writes during the pass.
template <class Unit, bool MH = false>
__device__ __forceinline__ int unit_in_memory_with(Unit &u, uint8_t *sp, uint8_t *st, uint64_t S, uint32_t L,
                                                   uint64_t k, int c, uint64_t T4, uint64_t T8, uint32_t hits);

template <class Unit, bool MH = false>
__device__ __forceinline__ int unit_in_memory(uint8_t *sp, uint8_t *st, uint64_t S, uint32_t L, uint64_t k, int c,
                                              uint64_t T4, uint64_t T8, uint32_t hits = 1) {
    Unit u;
    u.load(st, S, k);
    return unit_in_memory_with<Unit, MH>(u, sp, st, S, L, k, c, T4, T8, hits);
}

// The update with the unit's generator already loaded (it stores it back).
template <class Unit, bool MH>
__device__ __forceinline__ int unit_in_memory_with(Unit &u, uint8_t *sp, uint8_t *st, uint64_t S, uint32_t L,
                                                   uint64_t k, int c, uint64_t T4, uint64_t T8, uint32_t hits) {
    constexpr int NB = Unit::kNB;
    // L <= 16384: unit indices and site offsets fit 32 bits (no 64-bit division)
    const uint32_t upr = L / NB, k32 = static_cast<uint32_t>(k);
    const uint32_t y = k32 / upr;
    const uint32_t x0 = (k32 - y * upr) * NB;
    const uint32_t row = y * L, up_row = (y == 0 ? L - 1 : y - 1) * L;
    const uint32_t dn_row = (y == L - 1 ? 0 : y + 1) * L;
    uint64_t w = lds_run<NB>(sp + row + x0);
    const uint64_t upw = lds_run<NB>(sp + up_row + x0), dnw = lds_run<NB>(sp + dn_row + x0);
    const uint32_t lb = sp[row + (x0 == 0 ? L - 1 : x0 - 1)];
    const uint32_t rb = sp[row + (x0 + NB == L ? 0 : x0 + NB)];
    const uint64_t m = mismatches<NB>(w, upw, dnw, lb, rb);
    const int p = static_cast<int>((c + y) & 1);
    int sh = 0;
    if constexpr (MH) {
        // byte p + 2h is site h; the same draw order as the on-chip update
        uint32_t mi[NB / 2], fl[NB / 2];
#pragma unroll
        for (int h = 0; h < NB / 2; ++h) {
            mi[h] = static_cast<uint32_t>(m >> (8 * (p + 2 * h))) & 0xFFu;
            fl[h] = 0;
        }
        if constexpr (NB == 4) {
            u.draws2(hits, [&](uint32_t r) { hit_mem(mi[0], fl[0], r, T4, T8); },
                     [&](uint32_t r) { hit_mem(mi[1], fl[1], r, T4, T8); });
        } else {
            for (uint32_t i = 0; i < hits; ++i) {
                uint32_t ra, rb;
                u.pair(ra, rb);
                hit_mem(mi[0], fl[0], ra, T4, T8);
                hit_mem(mi[2], fl[2], rb, T4, T8);
            }
            for (uint32_t i = 0; i < hits; ++i) {
                uint32_t ra, rb;
                u.pair(ra, rb);
                hit_mem(mi[1], fl[1], ra, T4, T8);
                hit_mem(mi[3], fl[3], rb, T4, T8);
            }
        }
        u.store(st, S, k, 2 * hits);
#pragma unroll
        for (int h = 0; h < NB / 2; ++h) {
            w ^= static_cast<uint64_t>(fl[h] * 0xFEu) << (8 * (p + 2 * h));
            sh += 4 - 2 * static_cast<int>(mi[h]);
        }
    } else {
        uint32_t rr[NB / 2];
        u.draw(rr);
        u.store(st, S, k, 2);
#pragma unroll
        for (int h = 0; h < NB / 2; ++h) sh += metropolis(w, m, p + 2 * h, rr[h], T4, T8);
    }
    lds_put<NB>(sp + row + x0, w);
    return sh;
}

// A batch replica runs in one of three modes: in memory by one workgroup
// (kReplicaMemory), on chip by one workgroup (kReplicaOnChip, R = L), or as
// a gang of nwg strip workgroups of R rows each (kReplicaStrips) that
// exchange tagged halo words like the strips of one lattice.
constexpr uint32_t kReplicaMemory = 0, kReplicaOnChip = 1, kReplicaStrips = 2;
struct ReplicaDesc {
    int8_t *spins;
    uint8_t *st;
    uint64_t S;
    uint32_t L, mode;
    uint64_t T4, T8, n_sweeps;
    int32_t *trace;   // may be null
    uint32_t R, nwg, units;  // strips: rows and units per strip, strip count
    uint64_t *halo;   // strips: 2 slots x nwg x 2 rows x L/4 tagged words
    uint32_t *err;    // the lattice's error word (a strip gave up waiting)
    uint32_t R_last;  // strips: rows of the last strip (1..R; the others have R)
    uint32_t *gang;   // strips: arrival counter of the gang's workgroups (zeroed before each run)
    uint64_t start_ticks;  // strips: wall-clock ticks a gang member waits for the others to start
    uint32_t VB, slots;    // spins as bits: rows side by side, slots per thread
};

// Inlined: as a call it reads the descriptor back from the stack for every unit
// (XS1024W, a replica of L = 2816: 13.3 ms inlined, 17.7 called).
template <class Unit>
__device__ __forceinline__ void replica_in_memory(const ReplicaDesc &d, int *red) {
    constexpr int NB = Unit::kNB;
    const uint64_t n_units = static_cast<uint64_t>(d.L) * d.L / NB;
    uint8_t *sp = reinterpret_cast<uint8_t *>(d.spins);
    for (uint64_t sweep = 0; sweep < d.n_sweeps; ++sweep) {
        for (int c = 0; c < 2; ++c) {
            int sh = 0;
            // XS1024W: n_units and blockDim are multiples of 16, rows stay whole
            for (uint64_t k = threadIdx.x; k < n_units; k += blockDim.x)
                sh += unit_in_memory<Unit>(sp, d.st, d.S, d.L, k, c, d.T4, d.T8);
            __syncthreads();
            if (c == 1 && d.trace) {
                const int tot = block_sum(sh, red);
                if (threadIdx.x == 0) d.trace[sweep] = -tot;
            }
        }
    }
}

// A gang's strips wait on each other every pass, so none of them may start
// its sweeps before all of them run.  Items are claimed one at a time, so the
// first strips of a gang can be claimed long before the last ones (the other
// workgroups may be busy with long independent items): each member checks in
// and waits here, bounded by wall-clock time rather than a poll count, until
// all nwg have arrived.  They always do, as every other claimed item finishes
// on its own and frees its workgroup for the gang's next strip; if the bound
// is reached anyway (the device held by other work for that long), the
// lattice is marked invalid and its strips end quickly.
__device__ inline void gang_start(const ReplicaDesc &d) {
    if (threadIdx.x == 0) {
        __hip_atomic_fetch_add(d.gang, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t t0 = static_cast<uint64_t>(wall_clock64());
        while (__hip_atomic_load(d.gang, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < d.nwg) {
            if (static_cast<uint64_t>(wall_clock64()) - t0 > d.start_ticks || __hip_atomic_load(d.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                __hip_atomic_fetch_or(d.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            __builtin_amdgcn_s_sleep(127);
        }
    }
    __syncthreads();
}

}  // namespace rngx
