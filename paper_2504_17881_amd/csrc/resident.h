// Device routines of the kernels that hold a whole tile-set or state in LDS:
// state accesses, renormalisation and the run of a resident state (shared by
// kernels.hip and batch.hip).
#pragma once

#include "device.h"

namespace prx {

// State access of a tile pass, 16 bytes per lane and instruction: a lane
// moves G = 16 / sizeof(Cx<T>) consecutive amplitudes at once (two at
// complex64, one at complex128; measured 4.5 % faster than one complex64
// amplitude per access for the 14-qubit kernel).  Workgroups that own one
// tile-set take non-temporal or ordinary loads and stores by the state's size
// (streams_state); the persistent kernel, whose prefetched loads overlap the
// previous set's stores, is faster with ordinary ones (non-temporal: 7 %
// slower).
template <typename T>
struct Group {
    static constexpr int G = 16 / (int)sizeof(Cx<T>);  // amplitudes per access
    typedef T V __attribute__((ext_vector_type(2 * G)));
    static_assert(sizeof(V) == 16 && sizeof(V) == G * sizeof(Cx<T>), "16-byte groups");
};
template <bool NT, typename T>
__device__ __forceinline__ typename Group<T>::V group_load(const Cx<T> *p) {
    typedef typename Group<T>::V V;
    if constexpr (NT)
        return __builtin_nontemporal_load(reinterpret_cast<const V *>(p));
    else
        return *reinterpret_cast<const V *>(p);
}
template <bool NT, typename T>
__device__ __forceinline__ void group_store(Cx<T> *p, const typename Group<T>::V &v) {
    typedef typename Group<T>::V V;
    if constexpr (NT)
        __builtin_nontemporal_store(v, reinterpret_cast<V *>(p));
    else
        *reinterpret_cast<V *>(p) = v;
}

// One amplitude.
template <bool NT, typename T>
__device__ __forceinline__ Cx<T> amp_load(const Cx<T> *p) {
    typedef T W __attribute__((ext_vector_type(2)));
    if constexpr (NT) {
        const W w = __builtin_nontemporal_load(reinterpret_cast<const W *>(p));
        return Cx<T>{w.x, w.y};
    } else {
        return *p;
    }
}
template <bool NT, typename T>
__device__ __forceinline__ void amp_store(Cx<T> *p, const Cx<T> &v) {
    typedef T W __attribute__((ext_vector_type(2)));
    if constexpr (NT)
        __builtin_nontemporal_store(W{v.re, v.im}, reinterpret_cast<W *>(p));
    else
        *p = v;
}

// A 128 KiB tile-set (14 qubits at complex64, 13 at complex128) fills most
// of the CU's 160 KiB of LDS, so one workgroup runs per CU; it runs
// persistently, striding over the tile-sets and loading the next one into
// registers while it computes the current one.  Smaller tile-sets run one
// workgroup per tile-set (two to five per CU), which overlaps loads and
// compute across workgroups; with 13-qubit complex64 tile-sets that is 7 %
// faster than the persistent form.
template <typename T, int B>
struct TilePersist {
    static constexpr bool value = (sizeof(Cx<T>) << B) >= (128u << 10);
};

// Waves per SIMD that the LDS allows a tile shape (tile-sets per CU x waves
// per set / 4 SIMDs), the occupancy the register allocation is asked to
// keep: five 12-qubit complex64 workgroups per CU need at most 96 registers.
template <typename T, int B, int M>
struct TileWaves {
    static constexpr unsigned sets = (160u << 10) / (sizeof(Cx<T>) << B);
    static constexpr unsigned w = sets * ((1u << (B - M)) / 64u) / 4u;
    static constexpr unsigned value = w < 1 ? 1 : (w > 8 ? 8 : w);
};

// Only complex64 states are renormalised: complex128 passes hold no norm code
// (two FMAs per amplitude).
template <typename T>
static constexpr bool kRenorm = sizeof(T) == 4;

// 1 / sqrt(v): the hardware's estimate and two Newton steps (y <- y + y (1 -
// v y^2) / 2), which leave 0, infinity and NaN as the estimate has them.  A
// tenth of the code of a correctly rounded division and root, which a short
// pass fetches cold.
__device__ __forceinline__ double inv_sqrt(double v) {
    const double y0 = __builtin_amdgcn_rsq(v);
    double y = y0;
#pragma unroll
    for (int i = 0; i < 2; ++i) y = fma(0.5 * y, fma(-v * y, y, 1.0), y);
    return v > 0.0 && v < __builtin_huge_val() ? y : y0;
}

// -------------------------------------------------------------- resident

// A state that fits one workgroup's LDS (14 qubits at complex64, 13 at
// complex128) stays there for a whole plan: one launch instead of one per
// pass.  The frame is the global index, so every rotation fits it and a chunk
// ends only when its basis is full.  Bound by the latency of a chunk's chain
// (gather, rotations, scatter, barrier) up to 12 qubits, where a SIMD holds
// one wave, and by one CU's vector ALU and LDS at 14.  What only some chunks
// do stands in branches of its own (100 rotations of 10 qubits complex64 28.1
// us with selects in every chunk and 25.4 so, 300 of 14 qubits 132 and 124; a
// sample of 13 qubits complex128, 200 rotations, 104 and 89).
template <typename T, int B>
struct ResidentShape {
    static constexpr int M = 4;
    static constexpr int NT = B > 10 ? 1 << (B - M) : 64;
};

// Runs chunks [0, count) on the state at psi (n <= B qubits).  The workgroup
// has NT threads; states of fewer qubits leave whole waves idle (they only
// wait at the barriers), and below 10 qubits the lanes past the 2^(n-4)
// cosets repeat them (their complement vectors are zero): a wave's loads
// precede its stores, and the repeated stores carry equal values.
template <typename T, int B>
__device__ __forceinline__ void resident_run(Cx<T> *lds, double (*red)[16], Cx<T> *psi, int n,
                                             const ChunkRec<T> *__restrict__ chunks,
                                             uint32_t count, const RotRec<T> *__restrict__ rots,
                                             const double *rin, double *rout) {
    typedef ResidentShape<T, B> S;
    constexpr int M = S::M, NT = S::NT, PER = 1 << M;
    constexpr uint32_t SH = sizeof(Cx<T>) == 8 ? 3u : 4u;
    constexpr int G = Group<T>::G;
    constexpr int GPER = (1 << B) / (G * NT);
    typedef typename Group<T>::V V;
    // (global memory, whether the address came as an argument or from a table)
    typedef __attribute__((address_space(1))) V GlobalV;
    V *lds_v = reinterpret_cast<V *>(lds);
    unsigned char *lds_raw = reinterpret_cast<unsigned char *>(lds);
    const uint32_t tid = threadIdx.x;
    const uint32_t ncos = 1u << (n - M);       // cosets: threads with work
    const uint32_t ngroups = (1u << n) / G;
    const uint32_t waves = ncos > 64u ? ncos >> 6 : 1u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    {
        const GlobalV *src = (const GlobalV *)(uint64_t)psi;
        V r[GPER];
#pragma unroll
        for (int j = 0; j < GPER; ++j)
            if (tid + (uint32_t)j * NT < ngroups) r[j] = src[tid + (uint32_t)j * NT];
#pragma unroll
        for (int j = 0; j < GPER; ++j)
            if (tid + (uint32_t)j * NT < ngroups) lds_v[tid + (uint32_t)j * NT] = r[j];
    }
    double rn = rin ? *rin : 1.0;
    uint32_t tmask[B - M];
    tile_thread_masks<B - M>(tid, tmask);
    uint32_t par = 0;
    __syncthreads();
    for (uint32_t c = 0; c < count; ++c) {
        const ChunkRec<T> rec = chunks[c];
        const ChunkHead &ch = rec.h;
        if (wave < waves) {
            uint32_t k0 = 0;
#pragma unroll
            for (int i = 0; i < B - M; ++i) k0 = xor_and(k0, tmask[i], (uint32_t)ch.cvec[i]);
            const uint32_t k0b = k0 << SH;
            uint32_t Xb[PER];
            Xb[0] = 0;
#pragma unroll
            for (int v = 1; v < PER; ++v)
                Xb[v] = Xb[v & (v - 1)] ^ (ch.basis[__builtin_ctz(v)] << SH);
            Cx<T> amp[PER];
#pragma unroll
            for (int v = 0; v < PER; ++v)
                amp[v] = *reinterpret_cast<const Cx<T> *>(lds_raw + (k0b ^ Xb[v]));
            apply_chunk<T, kRotLean>(amp, k0, 0, rots + ch.rot_begin, ch.rot_count);
            // complex64 factors hold the chunk's cosines too, complex128 ones
            // leave label 0 as it is
#pragma unroll
            for (int v = kRenorm<T> ? 0 : 1; v < PER; ++v) {
                amp[v].re *= rec.fac[v];
                amp[v].im *= rec.fac[v];
            }
            double nrm = 0.0;
            if constexpr (kRenorm<T>) {
                if (ch.flags & kChunkRenormIn) {
                    // (rounded, a factor near 1 would be off by as much as the
                    // rotations of a chunk: the rest goes in too)
                    const double sc = rn * ch.scale;
                    const T s = (T)sc, s_lo = (T)(sc - (double)s);
#pragma unroll
                    for (int v = 0; v < PER; ++v) {
                        amp[v].re = fma(amp[v].re, s, amp[v].re * s_lo);
                        amp[v].im = fma(amp[v].im, s, amp[v].im * s_lo);
                    }
                }
                if (ch.flags & kChunkNormOut) {
#pragma unroll
                    for (int v = 0; v < PER; ++v) {
                        nrm = fma((double)amp[v].re, (double)amp[v].re, nrm);
                        nrm = fma((double)amp[v].im, (double)amp[v].im, nrm);
                    }
                }
            } else if (ch.flags & kChunkPassEnd) {
                const T s = (T)ch.scale;
#pragma unroll
                for (int v = 0; v < PER; ++v) {
                    amp[v].re *= s;
                    amp[v].im *= s;
                }
            }
#pragma unroll
            for (int v = 0; v < PER; ++v)
                *reinterpret_cast<Cx<T> *>(lds_raw + (k0b ^ Xb[v])) = amp[v];
            if (kRenorm<T> && (ch.flags & kChunkNormOut)) {
                if (tid >= ncos) nrm = 0.0;
                nrm = wave_sum(nrm);
                if ((tid & 63u) == 0) red[par][wave] = nrm;
            }
        }
        __syncthreads();
        if (kRenorm<T> && (ch.flags & kChunkNormOut)) {
            // the two places alternate: the next norm may be written before
            // every wave has read this one
            double sum = 0.0;
            for (uint32_t i = 0; i < waves; ++i) sum += red[par][i];
            rn = inv_sqrt(sum);
            par ^= 1u;
        }
    }
    {
        GlobalV *dst = (GlobalV *)(uint64_t)psi;
#pragma unroll
        for (int j = 0; j < GPER; ++j)
            if (tid + (uint32_t)j * NT < ngroups)
                dst[tid + (uint32_t)j * NT] = lds_v[tid + (uint32_t)j * NT];
    }
    if (kRenorm<T> && rout && tid == 0) *rout = rn;
}

}  // namespace prx
