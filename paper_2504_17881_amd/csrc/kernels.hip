// HIP kernels for gfx950 (CDNA4, wave64): Pauli-rotation sweeps over a
// 2^n complex state in HBM, and FP64 reductions.
//
// A rotation exp(i phi P) with P = (x, z) maps each index pair (k, k ^ x)
// through a 2x2 unitary (paper, "Software implementation": the rotation is a
// direct sum of 2x2 blocks, so (i) a permutation with phases by P and (ii) a
// linear combination):
//     new[k]  = cos(phi) psi[k]  + beta * sigma(k') psi[k']
//     new[k'] = cos(phi) psi[k'] + beta * sigma(k)  psi[k]
// with beta = i^{nY+1} sin(phi), nY = popcount(x & z) (the Y count, mod 4),
// sigma(j) = (-1)^{popcount(j & z)} taken from the source index, and
// sigma(k') = sigma(k) (-1)^{nY} (Supplementary Methods, "Pauli-string bit
// representation").  For x = 0 the rotation is diagonal:
// new[k] = (cos(phi) + i sin(phi) sigma(k)) psi[k].
//
// Kernels:
//   k_plain_pair / k_plain_diag : one rotation per HBM sweep.
//   k_span  : several consecutive rotations per sweep; every thread owns one
//             coset k0 XOR span(x_1..x_m) of the rotations' X masks and keeps
//             its 2^m amplitudes in registers.
//   k_tile  : one workgroup owns a tile-set of 2^B amplitudes (2^g tiles of
//             2^b contiguous amplitudes, g high-qubit XOR masks "virtual
//             qubits") held in LDS; the pass's rotations run in chunks, each
//             chunk gathered per thread as a coset of its X span.  The g = 1
//             case is the single-GPU form of the common-suffix grouping of
//             Eq. (core): all rotations sharing the high part of x are applied
//             while the two partner tiles are resident.
// Fused kernels use the factored update new = cos(phi) (psi + tau sigma
// psi'), tau = beta / cos(phi); a pass multiplies its cosines (and an FP64
// renormalisation factor) into one scale applied at the store.

#include <cmath>
#include <mutex>

#include "resident.h"

namespace prx {

// ----------------------------------------------------------------- plain

// Launch grids are capped at kMaxGridBlocks workgroups (2^30 work-items at
// 256 threads, inside the 32-bit work-item range of a dispatch); the sweep
// kernels stride over the rest of the state.
template <typename T, int U, bool STREAM>
__global__ void __launch_bounds__(256) k_plain_pair(Cx<T> *__restrict__ psi, PlainArgs a,
                                                    uint64_t npairs) {
    const T c = (T)a.c;
    const T be = (T)a.beta;
    const uint64_t stride = (uint64_t)gridDim.x * (256u * U);
    for (uint64_t base = (uint64_t)blockIdx.x * (256u * U) + threadIdx.x; base < npairs;
         base += stride) {
        uint64_t k[U], kp[U];
        Cx<T> u[U], w[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const uint64_t j = base + (uint64_t)i * 256u;
            k[i] = insert_zero64(j < npairs ? j : 0, a.pivot);
            kp[i] = k[i] ^ a.x;
            if (j < npairs) {
                u[i] = amp_load<STREAM>(psi + k[i]);
                w[i] = amp_load<STREAM>(psi + kp[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const uint64_t j = base + (uint64_t)i * 256u;
            if (j >= npairs) continue;
            const uint32_t sk = parity64(k[i] & a.z);
            const T bk = flip(be, sk ^ (uint32_t)a.nY_odd);  // beta sigma(k'), used for new[k]
            const T bkp = flip(be, sk);                      // beta sigma(k),  used for new[k']
            Cx<T> nu, nw;
            if (a.beta_imag) {
                nu.re = c * u[i].re - bk * w[i].im;
                nu.im = c * u[i].im + bk * w[i].re;
                nw.re = c * w[i].re - bkp * u[i].im;
                nw.im = c * w[i].im + bkp * u[i].re;
            } else {
                nu.re = c * u[i].re + bk * w[i].re;
                nu.im = c * u[i].im + bk * w[i].im;
                nw.re = c * w[i].re + bkp * u[i].re;
                nw.im = c * w[i].im + bkp * u[i].im;
            }
            amp_store<STREAM>(psi + k[i], nu);
            amp_store<STREAM>(psi + kp[i], nw);
        }
    }
}

template <typename T, int U, bool STREAM>
__global__ void __launch_bounds__(256) k_plain_diag(Cx<T> *__restrict__ psi, PlainArgs a,
                                                    uint64_t N) {
    const T c = (T)a.c;
    const T s = (T)a.beta;  // beta = i sin(phi) for x = 0
    const uint64_t stride = (uint64_t)gridDim.x * (256u * U);
    for (uint64_t base = (uint64_t)blockIdx.x * (256u * U) + threadIdx.x; base < N;
         base += stride) {
        Cx<T> u[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const uint64_t k = base + (uint64_t)i * 256u;
            if (k < N) u[i] = amp_load<STREAM>(psi + k);
        }
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const uint64_t k = base + (uint64_t)i * 256u;
            if (k >= N) continue;
            const T bs = flip(s, parity64(k & a.z));
            Cx<T> nu;
            nu.re = c * u[i].re - bs * u[i].im;
            nu.im = c * u[i].im + bs * u[i].re;
            amp_store<STREAM>(psi + k, nu);
        }
    }
}

// ------------------------------------------------- renormalisation hand-off

// Neumaier-compensated accumulator.
struct Neu {
    double s = 0.0, c = 0.0;
    __device__ __forceinline__ void add(double v) {
        const double t = s + v;
        if (fabs(s) >= fabs(v))
            c += (s - t) + v;
        else
            c += (v - t) + s;
        s = t;
    }
    __device__ __forceinline__ double value() const { return s + c; }
};

// The factor 1 / sqrt(norm) a pass takes over from the pass before it: read
// from one scalar, or, where the earlier pass left at most kRenormDirect
// partial sums, summed here by every wave (a fixed order, so all waves get
// the same bits).  The partials come from L2 while the pass's first state
// loads are in flight; the two reduction launches this replaces took 3.9 us
// of the 11.5 us of a 17-qubit complex64 pass and 7 of 20 us at 20 qubits.
// The sum stands in front of the pass's work, so its own chain counts: a lane
// takes one partial up to 64 (18 qubits), else four loads before the first
// addition, and the wave's sum goes over data-parallel moves instead of LDS
// permutes.  A 200-rotation qDRIFT plan, before and after (us): 17 qubits
// 125.3 / 119.0, 20 qubits 184.8 / 176.5, 24 qubits 746 / 735.
__device__ __forceinline__ double renorm_factor(const RenormIn &in) {
    if (!in.p) return 1.0;
    if (in.count == 0) return *in.p;
    const unsigned lane = threadIdx.x & 63u;
    double v;
    if (in.count <= 64u) {
        v = lane < in.count ? in.p[lane] : 0.0;
    } else {
        Neu acc;
        for (unsigned i = lane; i < in.count; i += 256u) {
            double d[4];
#pragma unroll
            for (unsigned k = 0; k < 4; ++k) d[k] = i + 64u * k < in.count ? in.p[i + 64u * k] : 0.0;
#pragma unroll
            for (unsigned k = 0; k < 4; ++k) acc.add(d[k]);
        }
        v = acc.value();
    }
    return inv_sqrt(wave_sum(v));
}

// ------------------------------------------------------------------ span

// The accesses are non-temporal where the tile passes' are (streams_state): an
// ordinary pass in between leaves its results dirty in the L2s, which are
// written back at its end, and the next pass starts cold.  Measured, ordinary /
// non-temporal (us): one span among the 12 tile passes of a 200-rotation qDRIFT
// plan of 22 qubits complex64 255 / 230, among the 9 of a 20-qubit Trotter step
// 134 / 127; three spans of 27 qubits 1254 / 1182, of 20 qubits complex128 24.8
// / 21.6.  (Three spans alone at 22 qubits complex64, the L2s' size, 39 / 43.)
template <typename T, int M, bool STREAM>
__global__ void __launch_bounds__(256) k_span(Cx<T> *__restrict__ psi, SpanArgs a,
                                              const RotRec<T> *__restrict__ rots,
                                              RenormIn renorm_in,
                                              double *__restrict__ norm_out) {
    __shared__ double red[4];
    const uint64_t ncos = 1ull << (a.n - M);
    uint64_t X[1 << M];
    X[0] = 0;
#pragma unroll
    for (int v = 1; v < (1 << M); ++v) X[v] = X[v & (v - 1)] ^ a.basis[__builtin_ctz(v)];
    double sc = a.scale;
    if constexpr (kRenorm<T>) sc *= renorm_factor(renorm_in);
    double F[1 << M];
    pending_factors<M>(F, a.fscale);
    double nrm = 0.0;
    // grid-stride over the cosets; every thread of a block runs the same
    // number of iterations (the rotation loop's control stays uniform)
    const uint64_t stride = (uint64_t)gridDim.x * 256u;
    for (uint64_t t0 = (uint64_t)blockIdx.x * 256u; t0 < ncos; t0 += stride) {
        const uint64_t t = t0 + threadIdx.x;
        const bool live = t < ncos;
        uint64_t k0 = live ? t : 0;
#pragma unroll
        for (int i = 0; i < M; ++i) k0 = insert_zero64(k0, a.pivot[i]);
        Cx<T> amp[1 << M];
        if (live) {
#pragma unroll
            for (int v = 0; v < (1 << M); ++v) amp[v] = amp_load<STREAM>(psi + (k0 ^ X[v]));
        }
        apply_rots<T, M>(amp, k0, 0, rots + a.rot_begin, a.rot_count);
        if (live) {
            // the thread's 2^M squares, each exact in FP64, summed in FP64
#pragma unroll
            for (int v = 0; v < (1 << M); ++v) {
                const T s = (T)(sc * F[v]);
                Cx<T> o;
                o.re = amp[v].re * s;
                o.im = amp[v].im * s;
                amp_store<STREAM>(psi + (k0 ^ X[v]), o);
                if constexpr (kRenorm<T>) {
                    nrm = fma((double)o.re, (double)o.re, nrm);
                    nrm = fma((double)o.im, (double)o.im, nrm);
                }
            }
        }
    }
    if (kRenorm<T> && norm_out) {
        nrm = block_sum<256>(nrm, red);
        if (threadIdx.x == 0) norm_out[blockIdx.x] = nrm;
    }
}

// ------------------------------------------------------------------ tile

// The rotation loop of a shape.  The lean one takes 300-rotation sequences at
// 15 qubits complex64 from 115 to 103 us (sorted) and 180 to 169 (qDRIFT), at
// 16 qubits complex128 from 130 to 122, a fifth of the 32-qubit step from 820
// to 810 ms.  The 10-qubit shape, which only callers who name it get, keeps
// rot_loop: the tests of the built code look for an instance of it here.  The
// lean loop would be 1 to 5 % faster in it (500-rotation sequences, sorted and
// qDRIFT, rot_loop / lean: 16 qubits complex64 202 / 191 and 273 / 266 us, 24
// qubits 2240 / 2211 and 3484 / 3460, 22 qubits complex128 1044 / 1023 and 1951 /
// 1940).
template <int B>
struct TileLoop {
    static constexpr RotLoop value = B == 10 ? kRotLoop : kRotLeanTile;
};

template <typename T, int B, int M, bool STREAM>
__global__ void __launch_bounds__(1 << (B - M))
    __attribute__((amdgpu_waves_per_eu(TileWaves<T, B, M>::value))) k_tile(Cx<T> *__restrict__ psi, TileArgs a,
                                                      const RotRec<T> *__restrict__ rots,
                                                      const ChunkRec<T> *__restrict__ chunks,
                                                      RenormIn renorm_in,
                                                      double *__restrict__ norm_out) {
    constexpr int NT = 1 << (B - M);  // threads
    constexpr int PER = 1 << M;       // amplitudes per thread (tile-set 2^B)
    constexpr bool PERSIST = TilePersist<T, B>::value;
    static_assert(PER <= 32 && B - M <= kMaxTileThreadBits, "tile shape");
    // The tile-set is the only LDS allocation (2^B amplitudes): 160 KB hold
    // five 12-qubit complex64 workgroups per CU.  Static, so that its address
    // is a link-time constant and LDS addresses are plain byte offsets.
    __shared__ __align__(16) Cx<T> lds[1 << B];
    unsigned char *lds_raw = reinterpret_cast<unsigned char *>(lds);
    const uint32_t tid = threadIdx.x;
    const uint32_t nsets = (uint32_t)(1ull << (a.n - B));

    // Tile v of set w has tile index t(w) ^ vc(v), vc(v) = XOR of the masks
    // selected by v's bits; t(w) inserts zeros at the masks' pivots.  Slot
    // s = G tid + u NT (u = G j) has disjoint thread and u bits, so its
    // global index splits into a per-thread part and the host's uniform
    // uoff[u] (the global offset of slot u NT).
    // HBM traffic moves groups of G slots: thread tid's group j holds slots
    // G (tid + j NT) .. + G - 1, contiguous in memory (b >= 4 low bits).
    constexpr int G = Group<T>::G;
    constexpr int GPER = PER / G;  // groups per thread
    typedef typename Group<T>::V V;
    V *lds_v = reinterpret_cast<V *>(lds);
    const uint32_t gtid = (uint32_t)G * tid;  // the thread's first slot
    const uint64_t vt = [&] {
        uint64_t c = 0;
        const uint32_t v = gtid >> a.b;
        for (int i = 0; i < a.g; ++i)
            if (v >> i & 1) c ^= a.vmask[i];
        return c;
    }();
    // (pivots unpacked with shifts: no indexed load from the argument block)
    auto tile_of = [&](uint32_t w) {
        uint64_t t = w;
        for (int i = 0; i < a.g; ++i) t = insert_zero64(t, (uint32_t)(a.tpivots >> (6 * i)) & 63u);
        return t;
    };
    auto base_of = [&](uint64_t t) { return ((t ^ vt) << a.b) | (gtid & ((1u << a.b) - 1u)); };

    uint32_t tmask[B - M];
    tile_thread_masks<B - M>(tid, tmask);

    double nrm = 0.0;

    // Set order: persistent workgroups stride over the sets; otherwise the
    // workgroups, dispatched round-robin over the 8 XCDs, give each XCD a
    // contiguous range of sets (and stride over the rest when the grid is
    // capped: the set count is then a multiple of the grid).
    uint32_t w = blockIdx.x;
    if (!PERSIST && (gridDim.x & 7u) == 0u)
        w = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    // Every thread issues all its loads before the first LDS store.  A
    // persistent workgroup enters each iteration with its set in LDS, loads
    // the next set into registers, computes and stores the current one, and
    // only then writes the loaded set to LDS: the loads' wait then sits
    // behind the stores in the same iteration, and the stores drain while
    // the next set is computed.
    // group j of the thread sits at offset uoff[G j] from its base
    V r[GPER];
    auto load_set = [&](uint64_t b0) {
#pragma unroll
        for (int j = 0; j < GPER; ++j) r[j] = group_load<STREAM>(psi + (b0 ^ a.uoff[G * j]));
    };
    auto stage_set = [&] {
#pragma unroll
        for (int j = 0; j < GPER; ++j) lds_v[tid + (uint32_t)j * NT] = r[j];
    };
    // The first set's loads are in flight while the previous pass's partials
    // are summed (the grid never exceeds the set count, so every workgroup
    // has a first set).
    T s = (T)a.scale;
    bool scaled = !kRenorm<T>;
    auto take_scale = [&] {
        if (!scaled) s = (T)(a.scale * renorm_factor(renorm_in));
        scaled = true;
    };
    if (PERSIST) {
        load_set(base_of(tile_of(w)));
        take_scale();
        stage_set();
        __syncthreads();
    }
    for (; w < nsets; w += gridDim.x) {
        const uint64_t tb = tile_of(w);
        const uint64_t base = base_of(tb);
        if (!PERSIST) {
            // one set per iteration (several when the grid is capped); a
            // thread writes only the slots it read in the previous store
            // epilogue, so no barrier is needed before the staging
            load_set(base);
            take_scale();
            stage_set();
            __syncthreads();
        }
        const uint32_t wn = w + gridDim.x;
        const bool next = PERSIST && wn < nsets;
        if (next) load_set(base_of(tile_of(wn)));

        tile_chunks<T, B, M, TileLoop<B>::value>(lds_raw, tmask, tb, chunks + a.chunk_begin, a.chunk_count, rots);

        {
            V q[GPER];
#pragma unroll
            for (int j = 0; j < GPER; ++j) q[j] = lds_v[tid + (uint32_t)j * NT];
            // the thread's squares, each exact in FP64, summed in FP64
#pragma unroll
            for (int j = 0; j < GPER; ++j) {
                const V o = q[j] * s;
                group_store<STREAM>(psi + (base ^ a.uoff[G * j]), o);
                if constexpr (kRenorm<T>) {
#pragma unroll
                    for (int c = 0; c < 2 * G; ++c) nrm = fma((double)o[c], (double)o[c], nrm);
                }
            }
        }
        if (next) {
            // the staging writes exactly the slots this thread read in the
            // store epilogue above (LDS operations of a wave stay in order),
            // so only the chunk gathers of the next set wait at a barrier
            stage_set();
            __syncthreads();
        }
    }
    if (kRenorm<T> && norm_out) {
        __syncthreads();  // the tile-set's LDS is reused for the partial sums
        nrm = block_sum<NT>(nrm, reinterpret_cast<double *>(lds_raw));
        if (tid == 0) norm_out[blockIdx.x] = nrm;
    }
}

// -------------------------------------------------------------- resident

template <typename T, int B>
__global__ void __launch_bounds__((ResidentShape<T, B>::NT))
    k_resident(Cx<T> *__restrict__ psi, int n, const ChunkRec<T> *__restrict__ chunks,
               uint32_t count, const RotRec<T> *__restrict__ rots, const double *rin,
               double *rout) {
    __shared__ __align__(16) Cx<T> lds[1 << B];
    __shared__ double red[2][16];
    resident_run<T, B>(lds, red, psi, n, chunks, count, rots, rin, rout);
}

// ------------------------------------------------------------ relabelling

// LDS slot of group coordinate s: the low four bits XORed with a fold of the
// higher ones, so that sixteen lanes reading coordinates that differ in any
// four high bits mostly hit distinct banks.
__device__ __forceinline__ uint32_t perm_slot(uint32_t s) {
    return s ^ (((s >> 4) ^ (s >> 8)) & 15u);
}

// One relabelling pass: every group of 2^12 elements (fixed bits outside
// pos[]) is read with sixteen contiguous amplitudes per access, permuted
// through LDS and written back in place, again sixteen contiguous
// amplitudes per access.
template <typename T>
__global__ void __launch_bounds__(256) k_permute(Cx<T> *__restrict__ psi, PermArgs a) {
    static_assert(kPermBits == 12, "256 threads x 16 slots per group");
    __shared__ __align__(16) Cx<T> lds[1 << kPermBits];
    const uint32_t t = threadIdx.x;
    const uint64_t ngroups = 1ull << (a.n - kPermBits);
    uint32_t it = 0;    // D^-1 of the thread's bits of the output coordinate
    uint64_t toff = 0;  // the thread's bits (coordinates 0..7) as index bits
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if ((t >> j) & 1u) {
            it ^= a.inv[j];
            toff |= 1ull << a.pos[j];
        }
    }
    for (uint64_t g = blockIdx.x; g < ngroups; g += gridDim.x) {
        uint64_t base = g;
#pragma unroll
        for (int j = 0; j < kPermBits; ++j) base = insert_zero64(base, a.pos[j]);
        base |= toff;
        Cx<T> r[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            uint64_t uo = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((u >> j) & 1) uo |= 1ull << a.pos[8 + j];
            r[u] = psi[base | uo];
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) lds[perm_slot(t + 256u * (uint32_t)u)] = r[u];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 16; ++u) r[u] = lds[perm_slot(it ^ a.ioff[u])];
        __syncthreads();  // the group's LDS is reused by the next iteration
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            uint64_t uo = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((u >> j) & 1) uo |= 1ull << a.pos[8 + j];
            psi[base | uo] = r[u];
        }
    }
}

// ------------------------------------------------------------ reductions

// Compensated accumulator: every addition's rounding error, exact in FP64
// (Knuth's two-sum, no comparison), is summed beside the sum.
struct Comp {
    double s = 0.0, c = 0.0;
    __device__ __forceinline__ void add(double v) {
        const double t = s + v, w = t - s;
        c += (s - (t - w)) + (v - w);
        s = t;
    }
    __device__ __forceinline__ void add(const Comp &o) {
        add(o.s);
        c += o.c;
    }
    __device__ __forceinline__ double value() const { return s + c; }
};

// Fixed-shape sum over a block of NT threads (deterministic for a fixed launch
// shape); the result is in thread 0.
template <int NT>
__device__ __forceinline__ Comp block_comp(Comp v, double *red) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        Comp o;
        o.s = __shfl_down(v.s, off, 64);
        o.c = __shfl_down(v.c, off, 64);
        v.add(o);
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __syncthreads();  // `red` may hold the sum before this one
    if (lane == 0) {
        red[2 * wave] = v.s;
        red[2 * wave + 1] = v.c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < NT / 64; ++i) {
            Comp o;
            o.s = red[2 * i];
            o.c = red[2 * i + 1];
            v.add(o);
        }
    }
    return v;
}

// The overlap's and the norm's first stage: 16 bytes per lane and load, U loads
// of every operand in flight, bound by the read bandwidth.  Block b leaves its
// sum at part[2b], or, when it is the only block, the result at out.
template <typename T, bool NORM>
__global__ void __launch_bounds__(kReduceThreads)
    k_reduce(const Cx<T> *__restrict__ a, const Cx<T> *__restrict__ b, uint64_t ngroups,
             double *__restrict__ part, double *__restrict__ out) {
    constexpr int G = Group<T>::G, U = 4;
    typedef typename Group<T>::V V;
    __shared__ double red[2 * kReduceThreads / 64];
    Comp re, im;
    auto take = [&](const V &u, const V &v) {
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const double ur = u[2 * i], ui = u[2 * i + 1];
            if constexpr (NORM) {
                re.add(ur * ur);
                re.add(ui * ui);
            } else {  // conj(u) * v
                const double vr = v[2 * i], vi = v[2 * i + 1];
                re.add(ur * vr);
                re.add(ui * vi);
                im.add(ur * vi);
                im.add(-ui * vr);
            }
        }
    };
    const V *pa = reinterpret_cast<const V *>(a), *pb = reinterpret_cast<const V *>(b);
    const uint64_t stride = (uint64_t)gridDim.x * kReduceThreads;
    uint64_t k = (uint64_t)blockIdx.x * kReduceThreads + threadIdx.x;
    for (; k + (U - 1) * stride < ngroups; k += U * stride) {
        V u[U], v[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            u[i] = __builtin_nontemporal_load(pa + k + i * stride);
            if constexpr (!NORM) v[i] = __builtin_nontemporal_load(pb + k + i * stride);
        }
#pragma unroll
        for (int i = 0; i < U; ++i) take(u[i], v[i]);
    }
    for (; k < ngroups; k += stride) {
        const V u = pa[k];
        if constexpr (NORM)
            take(u, u);
        else
            take(u, pb[k]);
    }
    re = block_comp<kReduceThreads>(re, red);
    if constexpr (!NORM) im = block_comp<kReduceThreads>(im, red);
    if (threadIdx.x == 0) {
        double *o = gridDim.x == 1 ? out : part + 2 * blockIdx.x;
        o[0] = re.value();
        o[1] = im.value();
    }
}

// Sums `count` <= 1024 (re, im) partials into out[0..1].
__global__ void __launch_bounds__(1024) k_finish_pairs(const double *__restrict__ part,
                                                       unsigned count, double *__restrict__ out) {
    static_assert(kReduceBlocks <= 1024, "one partial per thread");
    __shared__ double red[32];
    Comp re, im;
    if (threadIdx.x < count) {
        re.s = part[2 * threadIdx.x];
        im.s = part[2 * threadIdx.x + 1];
    }
    re = block_comp<1024>(re, red);
    im = block_comp<1024>(im, red);
    if (threadIdx.x == 0) {
        out[0] = re.value();
        out[1] = im.value();
    }
}

// Fixed-shape tree over the block (deterministic for a fixed launch shape).
__device__ __forceinline__ double tree256(double v, double *sh) {
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < (unsigned)w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    const double r = sh[0];
    __syncthreads();
    return r;
}

// Norm hand-off, stage 1: block b sums its contiguous share of the
// `count` partials into stage[b] (fixed shape, deterministic).
__global__ void __launch_bounds__(256) k_renorm_stage1(const double *__restrict__ part,
                                                       unsigned count, double *__restrict__ stage) {
    __shared__ double sh[256];
    const unsigned per = (count + gridDim.x - 1) / gridDim.x;
    const unsigned lo = blockIdx.x * per;
    const unsigned hi = min(count, lo + per);
    Neu acc;
    for (unsigned i = lo + threadIdx.x; i < hi; i += 256u) acc.add(part[i]);
    const double s = tree256(acc.value(), sh);
    if (threadIdx.x == 0) stage[blockIdx.x] = s;
}

// Last stage: sums `count` values and writes 1/sqrt(sum).
__global__ void __launch_bounds__(1024) k_renorm_finish(const double *__restrict__ v,
                                                        unsigned count,
                                                        double *__restrict__ scale_out) {
    __shared__ double red[16];
    Neu acc;
    for (unsigned i = threadIdx.x; i < count; i += 1024u) acc.add(v[i]);
    const double s = block_sum<1024>(acc.value(), red);
    if (threadIdx.x == 0) scale_out[0] = 1.0 / sqrt(s);
}

// Bound by the bandwidth of reading and writing the state, 16 bytes per lane;
// streaming, U groups in flight.  Measured after the norm's read, ordinary /
// streaming (us for both): 28 qubits complex128 2579 / 2387, 26 (1 GiB) 648 /
// 626; 25 qubits (512 MiB), half of which the last-level cache still holds,
// 293 / 331.  Four groups in flight slow the ordinary form (256 MiB: 147 / 152).
template <typename T, bool STREAM>
__global__ void __launch_bounds__(256) k_scale(Cx<T> *__restrict__ a, uint64_t ngroups, T s) {
    constexpr int G = Group<T>::G, U = STREAM ? 4 : 1;
    typedef typename Group<T>::V V;
    const uint64_t stride = (uint64_t)gridDim.x * 256u;
    uint64_t k = (uint64_t)blockIdx.x * 256u + threadIdx.x;
    for (; k + (U - 1) * stride < ngroups; k += U * stride) {
        V v[U];
#pragma unroll
        for (int i = 0; i < U; ++i) v[i] = group_load<STREAM>(a + G * (k + i * stride));
#pragma unroll
        for (int i = 0; i < U; ++i) group_store<STREAM>(a + G * (k + i * stride), v[i] * s);
    }
    for (; k < ngroups; k += stride)
        group_store<STREAM>(a + G * k, group_load<STREAM>(a + G * k) * s);
}

// ------------------------------------------------------------- launchers

static unsigned ceil_div_u(uint64_t a, uint64_t b) { return (unsigned)((a + b - 1) / b); }
static unsigned capped_blocks(uint64_t want, unsigned cap) {
    const uint64_t c = std::max<uint64_t>(1, std::min<uint64_t>(cap, kMaxGridBlocks));
    return (unsigned)std::min<uint64_t>(want ? want : 1, c);
}

template <typename T, bool STREAM>
static hipError_t plain_one(Cx<T> *p, const PlainArgs &a, hipStream_t s, unsigned cap) {
    constexpr int U = 4;
    const uint64_t items = a.x == 0 ? 1ull << a.n : 1ull << (a.n - 1);
    const dim3 grid(capped_blocks((items + 256u * U - 1) / (256u * U), cap)), nt(256);
    if (a.x == 0)
        hipLaunchKernelGGL((k_plain_diag<T, U, STREAM>), grid, nt, 0, s, p, a, items);
    else
        hipLaunchKernelGGL((k_plain_pair<T, U, STREAM>), grid, nt, 0, s, p, a, items);
    return hipGetLastError();
}

template <typename T>
static hipError_t plain_t(void *psi, const PlainArgs &a, hipStream_t s, unsigned cap) {
    return a.stream ? plain_one<T, true>((Cx<T> *)psi, a, s, cap)
                    : plain_one<T, false>((Cx<T> *)psi, a, s, cap);
}

hipError_t launch_plain(prx_dtype dt, void *psi, const PlainArgs &a, hipStream_t s, unsigned cap) {
    return dt == PRX_C64 ? plain_t<float>(psi, a, s, cap) : plain_t<double>(psi, a, s, cap);
}

unsigned permute_blocks(int n, unsigned cap) { return capped_blocks(1ull << (n - kPermBits), cap); }

hipError_t launch_permute(prx_dtype dt, void *psi, const PermArgs &a, hipStream_t s, unsigned cap) {
    const unsigned nb = permute_blocks(a.n, cap);
    if (dt == PRX_C64)
        hipLaunchKernelGGL(k_permute<float>, dim3(nb), dim3(256), 0, s, (Cx<float> *)psi, a);
    else
        hipLaunchKernelGGL(k_permute<double>, dim3(nb), dim3(256), 0, s, (Cx<double> *)psi, a);
    return hipGetLastError();
}

unsigned span_blocks(int n, int m, unsigned cap) {
    return capped_blocks(((1ull << (n - m)) + 255u) / 256u, cap);
}
unsigned tile_blocks(int n, int B, unsigned cap) { return capped_blocks(1ull << (n - B), cap); }
unsigned plain_blocks(int n, bool diag, unsigned cap) {
    const uint64_t items = diag ? (1ull << n) : (1ull << (n - 1));
    return capped_blocks((items + 1023u) / 1024u, cap);
}

// Persistent tile kernels stride over the 2^(n-B) tile-sets with the
// workgroups that fit on the device at once (cached per device and kernel).
static unsigned tile_grid(const void *kernel, int n, int B, int threads, unsigned cap) {
    struct Entry {
        const void *k;
        int dev;
        unsigned resident;
    };
    static Entry cache[64];
    static int used = 0;
    static std::mutex mu;
    std::lock_guard<std::mutex> lock(mu);
    int dev = 0;
    (void)hipGetDevice(&dev);
    unsigned resident = 0;
    for (int i = 0; i < used; ++i)
        if (cache[i].k == kernel && cache[i].dev == dev) resident = cache[i].resident;
    if (!resident) {
        int cus = 0, per = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, threads, 0) != hipSuccess ||
            cus <= 0 || per <= 0)
            return tile_blocks(n, B, cap);  // one workgroup per tile-set
        resident = (unsigned)(cus * per);
        if (used < 64) cache[used++] = Entry{kernel, dev, resident};
    }
    const unsigned sets = tile_blocks(n, B, cap);
    return sets < resident ? sets : resident;
}

bool span_supported(prx_dtype, int m) { return m >= 1 && m <= 5; }

template <typename T, int M>
static void span_one(Cx<T> *p, const SpanArgs &a, const RotRec<T> *r, const RenormIn &rin,
                     double *nout, hipStream_t s, unsigned nb) {
    if (streams_state(std::ldexp((double)sizeof(Cx<T>), a.n)))
        hipLaunchKernelGGL((k_span<T, M, true>), dim3(nb), dim3(256), 0, s, p, a, r, rin, nout);
    else
        hipLaunchKernelGGL((k_span<T, M, false>), dim3(nb), dim3(256), 0, s, p, a, r, rin, nout);
}

template <typename T>
static hipError_t span_t(int m, void *psi, const SpanArgs &a, const void *rots,
                         const RenormIn &rin, double *nout, hipStream_t s, unsigned nb) {
    const RotRec<T> *r = (const RotRec<T> *)rots;
    Cx<T> *p = (Cx<T> *)psi;
    switch (m) {
    case 1: span_one<T, 1>(p, a, r, rin, nout, s, nb); break;
    case 2: span_one<T, 2>(p, a, r, rin, nout, s, nb); break;
    case 3: span_one<T, 3>(p, a, r, rin, nout, s, nb); break;
    case 4: span_one<T, 4>(p, a, r, rin, nout, s, nb); break;
    case 5: span_one<T, 5>(p, a, r, rin, nout, s, nb); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_span(prx_dtype dt, int m, void *psi, const SpanArgs &a, const void *rots,
                       const RenormIn &renorm_in, double *norm_out, hipStream_t s,
                       unsigned blocks) {
    return dt == PRX_C64 ? span_t<float>(m, psi, a, rots, renorm_in, norm_out, s, blocks)
                         : span_t<double>(m, psi, a, rots, renorm_in, norm_out, s, blocks);
}

// (B, M) pairs instantiated for the tile kernel.
#define PRX_TILE_SHAPES(X) X(10, 3) X(10, 4) X(11, 4) X(12, 4) X(12, 5) X(13, 4) X(13, 5) X(14, 4)

bool tile_supported(prx_dtype dt, int B, int m) {
// complex128 tile-sets up to 12 qubits, and 13 qubits (128 KiB) with rank-4
// chunks (rank 5 would need 256 registers per lane for the set and its
// prefetch)
#define PRX_TS(BB, MM) \
    if (B == BB && m == MM) return dt == PRX_C64 || BB <= 12 || (BB == 13 && MM == 4);
    PRX_TILE_SHAPES(PRX_TS)
#undef PRX_TS
    return false;
}

template <typename T, int B, int M>
static unsigned tile_blocks_one(int n, unsigned cap) {
    return TilePersist<T, B>::value
               ? tile_grid((const void *)k_tile<T, B, M, false>, n, B, 1 << (B - M), cap)
               : tile_blocks(n, B, cap);
}

template <typename T, int B, int M>
static hipError_t tile_launch_one(void *psi, const TileArgs &a, const void *rots,
                                  const void *chunks, const RenormIn &rin, double *nout,
                                  hipStream_t s, unsigned nb) {
    if (!TilePersist<T, B>::value && a.stream)
        hipLaunchKernelGGL((k_tile<T, B, M, !TilePersist<T, B>::value>), dim3(nb),
                           dim3(1 << (B - M)), 0, s, (Cx<T> *)psi, a, (const RotRec<T> *)rots,
                           (const ChunkRec<T> *)chunks, rin, nout);
    else
        hipLaunchKernelGGL((k_tile<T, B, M, false>), dim3(nb), dim3(1 << (B - M)), 0, s,
                           (Cx<T> *)psi, a, (const RotRec<T> *)rots,
                           (const ChunkRec<T> *)chunks, rin, nout);
    return hipGetLastError();
}

// Expands X(T, B, M) for the built shape (T, B, m).
#define PRX_TILE_CASE(BB, MM)                                                  \
    if (B == BB && m == MM) {                                                  \
        if constexpr (sizeof(T) == 4 || BB <= 12 || (BB == 13 && MM == 4)) {   \
            PRX_TILE_BODY(BB, MM)                                              \
        }                                                                      \
    }

template <typename T>
static hipError_t tile_t(int B, int m, void *psi, const TileArgs &a, const void *rots,
                         const void *chunks, const RenormIn &rin, double *nout, hipStream_t s,
                         unsigned nb) {
#define PRX_TILE_BODY(BB, MM) return tile_launch_one<T, BB, MM>(psi, a, rots, chunks, rin, nout, s, nb);
    PRX_TILE_SHAPES(PRX_TILE_CASE)
#undef PRX_TILE_BODY
    return hipErrorInvalidValue;
}

template <typename T>
static unsigned tile_launch_blocks_t(int B, int m, int n, unsigned cap) {
#define PRX_TILE_BODY(BB, MM) return tile_blocks_one<T, BB, MM>(n, cap);
    PRX_TILE_SHAPES(PRX_TILE_CASE)
#undef PRX_TILE_BODY
    return tile_blocks(n, B, cap);
}

unsigned tile_launch_blocks(prx_dtype dt, int B, int m, int n, unsigned cap) {
    return dt == PRX_C64 ? tile_launch_blocks_t<float>(B, m, n, cap)
                         : tile_launch_blocks_t<double>(B, m, n, cap);
}

hipError_t launch_tile(prx_dtype dt, int B, int m, void *psi, const TileArgs &a,
                       const void *rots, const void *chunks, const RenormIn &renorm_in,
                       double *norm_out, hipStream_t s, unsigned blocks) {
    return dt == PRX_C64
               ? tile_t<float>(B, m, psi, a, rots, chunks, renorm_in, norm_out, s, blocks)
               : tile_t<double>(B, m, psi, a, rots, chunks, renorm_in, norm_out, s, blocks);
}

// A hand-off too long for the next pass to sum itself: one workgroup up to
// kRenormOneBlock partials (a 24-qubit pass of 4096), two launches beyond.
hipError_t launch_renorm_finish(const double *partials, unsigned count, double *scale_out,
                                hipStream_t s) {
    // scale_out[1 .. kRenormStage] holds the stage-1 sums
    double *stage = scale_out + 1;
    if (count > kRenormOneBlock) {
        hipLaunchKernelGGL(k_renorm_stage1, dim3(kRenormStage), dim3(256), 0, s, partials, count,
                           stage);
        partials = stage;
        count = kRenormStage;
    }
    hipLaunchKernelGGL(k_renorm_finish, dim3(1), dim3(1024), 0, s, partials, count, scale_out);
    return hipGetLastError();
}

unsigned resident_threads(int n) { return n > 10 ? 1u << (n - 4) : 64u; }

template <typename T>
static hipError_t resident_t(void *psi, int n, const void *rots, const void *chunks,
                             uint32_t begin, uint32_t count, const double *rin, double *rout,
                             hipStream_t s) {
    Cx<T> *p = (Cx<T> *)psi;
    const ChunkRec<T> *c = (const ChunkRec<T> *)chunks + begin;
    const RotRec<T> *r = (const RotRec<T> *)rots;
    if (n < kResidentMinQubits || n > resident_max_qubits(sizeof(T) == 4 ? PRX_C64 : PRX_C128))
        return hipErrorInvalidValue;
    const dim3 one(1), nt(resident_threads(n));
    switch (n) {
    case 11: hipLaunchKernelGGL((k_resident<T, 11>), one, nt, 0, s, p, n, c, count, r, rin, rout); break;
    case 12: hipLaunchKernelGGL((k_resident<T, 12>), one, nt, 0, s, p, n, c, count, r, rin, rout); break;
    case 13: hipLaunchKernelGGL((k_resident<T, 13>), one, nt, 0, s, p, n, c, count, r, rin, rout); break;
    case 14:
        if constexpr (sizeof(T) == 4)
            hipLaunchKernelGGL((k_resident<T, 14>), one, nt, 0, s, p, n, c, count, r, rin, rout);
        break;
    default: hipLaunchKernelGGL((k_resident<T, 10>), one, nt, 0, s, p, n, c, count, r, rin, rout); break;
    }
    return hipGetLastError();
}

hipError_t launch_resident(prx_dtype dt, void *psi, int n, const void *rots, const void *chunks,
                           uint32_t chunk_begin, uint32_t chunk_count, const double *rin,
                           double *rout, hipStream_t s) {
    return dt == PRX_C64
               ? resident_t<float>(psi, n, rots, chunks, chunk_begin, chunk_count, rin, rout, s)
               : resident_t<double>(psi, n, rots, chunks, chunk_begin, chunk_count, rin, rout, s);
}

template <typename T, bool NORM>
static hipError_t reduce_t(const void *a, const void *b, int n, double *part, double *out,
                           hipStream_t s) {
    const uint64_t ngroups = (1ull << n) / Group<T>::G;
    // one block up to 2^13 amplitudes (no second launch), else blocks of eight
    // groups per thread up to kReduceBlocks
    const unsigned g =
        n <= 13 ? 1u
                : (unsigned)std::min<uint64_t>(kReduceBlocks, (ngroups + kReduceThreads * 8u - 1) /
                                                                  (kReduceThreads * 8u));
    hipLaunchKernelGGL((k_reduce<T, NORM>), dim3(g), dim3(kReduceThreads), 0, s, (const Cx<T> *)a,
                       (const Cx<T> *)b, ngroups, part, out);
    if (g > 1)
        hipLaunchKernelGGL(k_finish_pairs, dim3(1), dim3(1024), 0, s, part, g, out);
    return hipGetLastError();
}

hipError_t launch_overlap(prx_dtype dt, const void *psi0, const void *psi, int n, double *part,
                          double *out, hipStream_t s) {
    return dt == PRX_C64 ? reduce_t<float, false>(psi0, psi, n, part, out, s)
                         : reduce_t<double, false>(psi0, psi, n, part, out, s);
}

hipError_t launch_norm2(prx_dtype dt, const void *psi, int n, double *part, double *out,
                        hipStream_t s) {
    return dt == PRX_C64 ? reduce_t<float, true>(psi, psi, n, part, out, s)
                         : reduce_t<double, true>(psi, psi, n, part, out, s);
}

template <typename T>
static hipError_t scale_t(void *psi, int n, double scale, hipStream_t s) {
    const uint64_t ngroups = (1ull << n) / Group<T>::G;
    const unsigned g = (unsigned)std::min<uint64_t>((ngroups + 255) / 256, 256u * 64u);
    if (std::ldexp((double)sizeof(Cx<T>), n) >= 0x1p30)
        hipLaunchKernelGGL((k_scale<T, true>), dim3(g), dim3(256), 0, s, (Cx<T> *)psi, ngroups,
                           (T)scale);
    else
        hipLaunchKernelGGL((k_scale<T, false>), dim3(g), dim3(256), 0, s, (Cx<T> *)psi, ngroups,
                           (T)scale);
    return hipGetLastError();
}

hipError_t launch_scale(prx_dtype dt, void *psi, int n, double scale, hipStream_t s) {
    return dt == PRX_C64 ? scale_t<float>(psi, n, scale, s) : scale_t<double>(psi, n, scale, s);
}

}  // namespace prx
