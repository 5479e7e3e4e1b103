// Batched execution of many independent samples (qDRIFT or partially
// randomised draws, circuits of uneven qubit counts).
//
// A sample whose state fits one workgroup's LDS (up to 14 qubits at
// complex64, 13 at complex128) runs its whole sequence there: one launch for
// all such samples, one workgroup each.  Larger samples are planned into tile
// passes with as many virtual qubits as 16 contiguous amplitudes allow: a
// random-order qDRIFT sequence then fuses 2-2.5 times more rotations per pass
// than with spans.  Round p applies pass p of every sample that has one, as
// one grid-stride kernel over the round's (sample, tile-set) items.  Kernel
// boundaries order the rounds, so no workgroup ever waits on another; the
// whole sequence of kernels is enqueued back to back (and can be captured as
// one graph).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "objects.h"
#include "resident.h"

namespace prx {

static constexpr int kBatchTileM = 4;
// Tile rounds launch one workgroup per (sample, tile-set) item up to this
// many (the hardware keeps as many resident as fit and starts the next as
// soon as one ends), striding beyond it.
static constexpr uint64_t kTileGridCap = 1u << 20;
// Resident samples that take one launch whatever their sizes: one per CU.
// More are launched by size, so that small ones share a CU.
static constexpr size_t kResidentOneLaunch = 256;
static int batch_tile_qubits(prx_dtype dt) { return dt == PRX_C64 ? 12 : 11; }
// Tile qubits of a batch's rounds, by the amplitudes of its tile samples and
// the fewest qubits among them.  Larger frames make fewer sweeps (32 samples
// of 16 to 22 qubits: 2485, 2121, 1805 passes with 12, 13, 14 qubits), smaller
// ones leave more workgroups on a CU to overlap and shorter ends of rounds.
// Measured (us per batch, 12 / 13 / 14 qubits): 20 samples of 17 qubits 472 /
// 491 / 636, 20 of 19 1280 / 1182 / 1248, 24 of 23 21456 / 19488 / 20786, 6 of
// 24 6448 / 5845 / 5479, 4 of 25 8212 / 7609 / 7289; 24 samples of 22 qubits,
// one 14-qubit set of each per CU, take 12311 with 14 and 8847 with 13.  Mixed
// sizes gain nothing from 14 either: 32 samples of 16 to 22 qubits move 40.0 GB
// in 8541 us with 13 and 34.3 GB in 8667 with 14.
// complex128, 32 of 15 to 21: 10773 with 11 qubits, 9539 with 12, 10444 with
// 13; 64 of 14 to 17 3096 with 11 and 2736 with 12.
static int batch_frame_qubits(prx_dtype dt, double amps, int fewest) {
    if (dt == PRX_C64) return fewest >= 24 ? 14 : amps >= 0x1p23 ? 13 : 12;
    return amps >= 0x1p19 ? 12 : 11;
}

// The overlap read-out of a sample.
struct BSample {
    uint64_t psi;        // device address of the state
    uint64_t basis_idx;
};

// A sample that stays in one workgroup's LDS.
struct BResident {
    uint64_t psi;
    uint32_t n, chunk_begin, chunk_count, pad;
};

// One pass of a sample in tile passes of fixed (B, M).  A round's passes lie
// together, with their first items in a table of their own beside them.
struct BTilePass {
    TileArgs a;
    uint64_t psi;
};

// State amplitudes addressed as global memory: the states' addresses come
// from the sample tables, and without the address space the compiler would
// use flat accesses, which also count against the LDS/scalar wait counter.
// 16 bytes per lane: G = 16 / sizeof(Cx<T>) consecutive amplitudes from
// amplitude index i (a multiple of G).  Non-temporal: every amplitude is read
// and written once per pass, and between two passes of a sample lie those of
// all others (32 samples of 16 to 22 qubits: 11.7 ms against 15.0 ms with
// ordinary accesses; the same when groups of samples that the last-level
// cache holds run all their rounds before the next).
template <bool NT, typename T>
__device__ __forceinline__ typename Group<T>::V gload(uint64_t psi, uint64_t i) {
    typedef const __attribute__((address_space(1))) typename Group<T>::V *P;
    const P p = (P)(psi + i * sizeof(Cx<T>));
    if constexpr (NT)
        return __builtin_nontemporal_load(p);
    else
        return *p;
}
template <bool NT, typename T>
__device__ __forceinline__ void gstore(uint64_t psi, uint64_t i, const typename Group<T>::V &v) {
    typedef __attribute__((address_space(1))) typename Group<T>::V *P;
    const P p = (P)(psi + i * sizeof(Cx<T>));
    if constexpr (NT)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

// Item j of a round: the last pass k with first[k] <= j, found from the
// passes' first items read all at once, one per lane.
__device__ __forceinline__ uint32_t pass_of(uint32_t j, const uint32_t *__restrict__ first,
                                            uint32_t count) {
    uint32_t k = 0;
    for (uint32_t i = 0; i < count; i += 64u) {
        const uint32_t at = i + (threadIdx.x & 63u);
        k += (uint32_t)__popcll(__ballot(at < count && first[at] <= j));
    }
    return __builtin_amdgcn_readfirstlane(k - 1u);
}

// The base tile of set w of a pass and this thread's first amplitude in it.
struct SetBase {
    uint64_t tb, base;
};
__device__ __forceinline__ SetBase set_base(const TileArgs *ta, uint32_t w, uint32_t gtid) {
    SetBase s;
    uint64_t t = w;
    for (int i = 0; i < ta->g; ++i)
        t = insert_zero64(t, (uint32_t)(ta->tpivots >> (6 * i)) & 63u);
    s.tb = t;
    uint64_t c = t;
    const uint32_t v = gtid >> ta->b;
    for (int i = 0; i < ta->g; ++i)
        if (v >> i & 1) c ^= ta->vmask[i];
    s.base = (c << ta->b) | (gtid & ((1u << ta->b) - 1u));
    return s;
}

// The tables arrive as separate __restrict__ arguments: the compiler then
// knows the state stores cannot change them and reads them with scalar
// loads, so the rotation loop's control values stay uniform.  A tile-set
// works as in k_tile: small ones one per workgroup and item; the 128 KiB ones
// (TilePersist) in workgroups that stride over the items and hold the next
// item's set in registers while they compute the current one.
// The small sets' accesses are non-temporal at every size: ordinary ones where
// a round's states fit the last-level cache took 678 against 584 us (24 samples
// of 16 to 22 qubits complex64), 6630 against 5408 (48 of 17 to 21 complex128).
template <typename T, int B, int M>
__global__ void __launch_bounds__(1 << (B - M))
    __attribute__((amdgpu_waves_per_eu(TileWaves<T, B, M>::value)))
    k_batch_tile_round(const BTilePass *__restrict__ passes, const uint32_t *__restrict__ first,
                       uint32_t count, uint32_t items, const ChunkRec<T> *__restrict__ chunks,
                       const void *__restrict__ rot_table) {
    constexpr int NT = 1 << (B - M);
    constexpr int PER = 1 << M;
    constexpr bool PERSIST = TilePersist<T, B>::value;
    constexpr int G = Group<T>::G;
    constexpr int GPER = PER / G;
    typedef typename Group<T>::V V;
    __shared__ __align__(16) Cx<T> lds[1 << B];
    unsigned char *lds_raw = reinterpret_cast<unsigned char *>(lds);
    V *lds_v = reinterpret_cast<V *>(lds);
    const uint32_t tid = threadIdx.x;
    const uint32_t gtid = (uint32_t)G * tid;  // the thread's first slot (see k_tile)
    uint32_t tmask[B - M];
    tile_thread_masks<B - M>(tid, tmask);
    V r[GPER];
    auto load_set = [&](const BTilePass *bp, const SetBase &s) {
#pragma unroll
        for (int i = 0; i < GPER; ++i)
            r[i] = gload<!PERSIST, T>(bp->psi, s.base ^ bp->a.uoff[G * i]);
    };
    auto stage_set = [&] {
#pragma unroll
        for (int i = 0; i < GPER; ++i) lds_v[tid + (uint32_t)i * NT] = r[i];
    };
    uint32_t j = blockIdx.x;  // (the grid never exceeds the items)
    uint32_t k = pass_of(j, first, count);
    SetBase set = set_base(&passes[k].a, j - first[k], gtid);
    load_set(passes + k, set);
    stage_set();
    __syncthreads();
    while (true) {
        const BTilePass *bp = passes + k;
        const uint32_t jn = j + gridDim.x;
        const bool next = jn < items;
        SetBase nset;
        if (next) {
            k = pass_of(jn, first, count);
            nset = set_base(&passes[k].a, jn - first[k], gtid);
            if (PERSIST) load_set(passes + k, nset);
        }
        // (the base tile is uniform, but the compiler carries it in vector
        // registers from one iteration to the next)
        const uint64_t tb =
            ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(set.tb >> 32)) << 32) |
            __builtin_amdgcn_readfirstlane((uint32_t)set.tb);
        // (rot_loop where the round is bound by its sweeps and the loops are within
        // 2 %; the tests of the built code look for instances of it here.  rot_loop /
        // lean: 6 samples of 24 qubits 10.31 / 10.15 ms, complex128 8 of 23 16.15 /
        // 16.12, 32 of 15 to 21 4.57 / 4.50)
        constexpr bool swept = PERSIST || (sizeof(T) == 8 && B == 12);
        tile_chunks<T, B, M, swept ? kRotLoop : kRotLeanTile>(lds_raw, tmask, tb, chunks + bp->a.chunk_begin, bp->a.chunk_count,
                             reinterpret_cast<const RotRec<T> *>(rot_table));
        const T s = (T)bp->a.scale;
        {
            V q[GPER];
#pragma unroll
            for (int i = 0; i < GPER; ++i) q[i] = lds_v[tid + (uint32_t)i * NT];
#pragma unroll
            for (int i = 0; i < GPER; ++i)
                gstore<!PERSIST, T>(bp->psi, set.base ^ bp->a.uoff[G * i], q[i] * s);
        }
        if (!next) break;
        // (the staging writes the slots this thread has just read)
        if (!PERSIST) load_set(passes + k, nset);
        stage_set();
        __syncthreads();
        j = __builtin_amdgcn_readfirstlane(jn);
        set = nset;
    }
}

// One workgroup per resident sample (striding beyond the grid); B covers the
// launch's largest sample.
template <typename T, int B>
__global__ void __launch_bounds__((ResidentShape<T, B>::NT))
    k_batch_resident(const BResident *__restrict__ samples, uint32_t count,
                     const ChunkRec<T> *__restrict__ chunks, const void *__restrict__ rot_table) {
    __shared__ __align__(16) Cx<T> lds[1 << B];
    __shared__ double red[2][16];
    for (uint32_t i = blockIdx.x; i < count; i += gridDim.x) {
        const BResident s = samples[i];
        resident_run<T, B>(lds, red, (Cx<T> *)s.psi, (int)s.n, chunks + s.chunk_begin,
                           s.chunk_count, reinterpret_cast<const RotRec<T> *>(rot_table), nullptr,
                           nullptr);
        __syncthreads();  // the next sample overwrites the LDS
    }
}

template <typename T>
__global__ void k_batch_overlaps(const BSample *samples, uint32_t S, double *out) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= S) return;
    const Cx<T> *psi = reinterpret_cast<const Cx<T> *>(samples[i].psi);
    const Cx<T> v = psi[samples[i].basis_idx];
    out[2 * i] = (double)v.re;
    out[2 * i + 1] = (double)v.im;
}

}  // namespace prx

// ------------------------------------------------------------------- host

struct prx_batch {
    size_t S = 0;
    prx_dtype dtype = PRX_C64;
    std::vector<prx::BSample> samples;
    std::vector<prx::BResident> residents;  // largest first
    std::vector<uint32_t> rsrc;             // resident -> sample
    std::vector<prx::BTilePass> tpasses;    // round by round, most rotations first
    std::vector<uint32_t> tfirst;           // beside them: first item within the round
    std::vector<uint32_t> tsrc;             // and sample
    std::vector<unsigned char> chunks;      // ChunkRec<float> or ChunkRec<double> image
    std::vector<unsigned char> rots;        // RotRec<float> or RotRec<double> image
    struct Launch {                         // resident samples [first, first + count)
        int B;
        uint32_t first, count;
    };
    std::vector<Launch> launches;
    struct Round {                          // passes [begin, begin + count)
        uint32_t begin, count, items;
    };
    std::vector<Round> rounds;
    int B = 12;                             // their tile qubits
    prx_batch_info info = {};               // without the samples of `counted`
    std::vector<prx_sched> counted;         // those whose passes prx_batch_get_info counts
    unsigned max_grid = 0;  // 0: the default grid caps
    // workspace layout
    size_t off_samples = 0, off_residents = 0, off_tpasses = 0, off_tfirst = 0, off_chunks = 0,
           off_rots = 0, total = 0;
};

struct prx_graph {
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};

using namespace prx;

static size_t al256(size_t v) { return (v + 255) & ~(size_t)255; }

namespace prx {

// Appends a plan's chunk and rotation tables; returns the plan's first chunk.
static uint32_t append_tables(prx_batch *b, const prx_plan *P, size_t csz, size_t rsz) {
    const uint32_t rot_base = (uint32_t)(b->rots.size() / rsz);
    const size_t at = b->chunks.size();
    b->chunks.insert(b->chunks.end(), P->chunk_table.begin(), P->chunk_table.end());
    for (size_t c = at; c < b->chunks.size(); c += csz)
        reinterpret_cast<ChunkHead *>(b->chunks.data() + c)->rot_begin += rot_base;
    b->rots.insert(b->rots.end(), P->rot_table.begin(), P->rot_table.end());
    return (uint32_t)(at / csz);
}

// Plans of tile passes only; the caller sets the frames.
static PlanCfg tile_settings() {
    PlanCfg c;
    c.tile_only = true;
    c.narrow = false;
    c.m = kBatchTileM;
    c.renorm_every = -1;
    c.max_fuse = 128;
    // exact reorders: a later rotation that fits the pass's frame and
    // commutes with every rotation it passes joins the pass (10-20 %
    // fewer passes on random-order qDRIFT sequences)
    c.commuting = true;
    return c;
}

static void count_passes(prx_batch_info &info, size_t passes, int n) {
    info.passes += passes;
    info.rounds = std::max(info.rounds, passes);
    info.amp_sweeps += (double)passes * std::ldexp(1.0, n);
}

// A sample's tile passes before they are laid out by rounds.
struct TileSample {
    uint32_t sample, nsets;
    std::vector<TileArgs> passes;
    std::vector<uint32_t> rots;  // rotations per pass
};

// Lays the passes out round by round.  Within a round the passes with most
// rotations come first: their workgroups take longest, and the last ones to
// start decide when the round ends.
static void make_rounds(prx_batch *b, const std::vector<TileSample> &ts) {
    for (uint32_t p = 0;; ++p) {
        std::vector<uint32_t> act;
        for (uint32_t k = 0; k < ts.size(); ++k)
            if (p < ts[k].passes.size()) act.push_back(k);
        if (act.empty()) break;
        std::stable_sort(act.begin(), act.end(), [&](uint32_t x, uint32_t y) {
            return ts[x].rots[p] > ts[y].rots[p];
        });
        prx_batch::Round r{(uint32_t)b->tpasses.size(), (uint32_t)act.size(), 0};
        for (uint32_t k : act) {
            b->tpasses.push_back(BTilePass{ts[k].passes[p], 0});
            b->tfirst.push_back(r.items);
            b->tsrc.push_back(ts[k].sample);
            r.items += ts[k].nsets;
        }
        b->rounds.push_back(r);
    }
}

// One launch for all resident samples, or one per size when there are more of
// them than CUs.
static void make_launches(prx_batch *b) {
    const size_t Sr = b->residents.size();
    std::vector<uint32_t> order(Sr);
    for (size_t s = 0; s < Sr; ++s) order[s] = (uint32_t)s;
    std::stable_sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) {
        const BResident &a = b->residents[x], &c = b->residents[y];
        return a.n != c.n ? a.n > c.n : a.chunk_count > c.chunk_count;
    });
    std::vector<BResident> rs(Sr);
    std::vector<uint32_t> src(Sr);
    for (size_t k = 0; k < Sr; ++k) {
        rs[k] = b->residents[order[k]];
        src[k] = b->rsrc[order[k]];
    }
    b->residents.swap(rs);
    b->rsrc.swap(src);
    auto size_of = [&](size_t k) { return std::max(10, (int)b->residents[k].n); };
    for (size_t i = 0; i < Sr;) {
        size_t e = i + 1;
        while (e < Sr && (Sr <= kResidentOneLaunch || size_of(e) == size_of(i))) ++e;
        b->launches.push_back(prx_batch::Launch{size_of(i), (uint32_t)i, (uint32_t)(e - i)});
        i = e;
    }
}

template <typename T>
static hipError_t launch_residents(int B, unsigned grid, const BResident *r, uint32_t count,
                                   const void *chunks, const void *rots, hipStream_t st) {
    const dim3 g(grid), nt(resident_threads(B));
    const ChunkRec<T> *c = (const ChunkRec<T> *)chunks;
    switch (B) {
    case 10: hipLaunchKernelGGL((k_batch_resident<T, 10>), g, nt, 0, st, r, count, c, rots); break;
    case 11: hipLaunchKernelGGL((k_batch_resident<T, 11>), g, nt, 0, st, r, count, c, rots); break;
    case 12: hipLaunchKernelGGL((k_batch_resident<T, 12>), g, nt, 0, st, r, count, c, rots); break;
    case 13: hipLaunchKernelGGL((k_batch_resident<T, 13>), g, nt, 0, st, r, count, c, rots); break;
    case 14:
        if constexpr (sizeof(T) == 4) {
            hipLaunchKernelGGL((k_batch_resident<T, 14>), g, nt, 0, st, r, count, c, rots);
            break;
        }
        return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename T, int B>
static hipError_t launch_round_b(unsigned grid, const BTilePass *passes, const uint32_t *first,
                                 uint32_t count, uint32_t items, const void *chunks,
                                 const void *rots, hipStream_t st) {
    hipLaunchKernelGGL((k_batch_tile_round<T, B, kBatchTileM>), dim3(grid),
                       dim3(1u << (B - kBatchTileM)), 0, st, passes, first, count, items,
                       (const ChunkRec<T> *)chunks, rots);
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_round(int B, unsigned grid, const BTilePass *ps, const uint32_t *first,
                               uint32_t count, uint32_t items, const void *chunks,
                               const void *rots, hipStream_t st) {
    if constexpr (sizeof(T) == 4) {
        if (B == 14) return launch_round_b<T, 14>(grid, ps, first, count, items, chunks, rots, st);
        if (B == 13) return launch_round_b<T, 13>(grid, ps, first, count, items, chunks, rots, st);
    } else {
        if (B == 11) return launch_round_b<T, 11>(grid, ps, first, count, items, chunks, rots, st);
    }
    if (B == 12) return launch_round_b<T, 12>(grid, ps, first, count, items, chunks, rots, st);
    return hipErrorInvalidValue;
}

}  // namespace prx

extern "C" {

prx_status prx_batch_create(size_t S, const int *n, const prx_sched *const *sched,
                            prx_dtype dtype, const uint64_t *basis_idx, prx_batch **out) {
    if (!out || !n || !sched || !basis_idx) return fail(PRX_ERR_INVALID, "null pointer");
    if (S == 0) return fail(PRX_ERR_INVALID, "S must be positive");
    if (dtype != PRX_C64 && dtype != PRX_C128) return fail(PRX_ERR_INVALID, "bad dtype");
    for (size_t s = 0; s < S; ++s) {
        if (!sched[s]) return fail(PRX_ERR_INVALID, "null schedule");
        if (n[s] < 6 || n[s] > 34) return fail(PRX_ERR_INVALID, "n must be in [6, 34]");
        if (sched[s]->n != n[s]) return fail(PRX_ERR_INVALID, "schedule n differs from n[s]");
        if (basis_idx[s] >> n[s]) return fail(PRX_ERR_INVALID, "basis index out of range");
    }
    prx_batch *b = new (std::nothrow) prx_batch;
    if (!b) return fail(PRX_ERR_OOM, "out of host memory");
    try {
        b->S = S;
        b->dtype = dtype;
        const size_t rsz = dtype == PRX_C64 ? sizeof(RotRec<float>) : sizeof(RotRec<double>);
        const size_t csz = dtype == PRX_C64 ? sizeof(ChunkRec<float>) : sizeof(ChunkRec<double>);
        const int TB = batch_tile_qubits(dtype);
        const int nres = resident_max_qubits(dtype);
        PlanCfg res_cfg;
        res_cfg.resident = true;
        res_cfg.m = kBatchTileM;
        res_cfg.renorm_every = -1;
        res_cfg.max_fuse = 128;
        res_cfg.commuting = true;
        PlanCfg tile_cfg = tile_settings();
        double amps = 0.0;
        int fewest = 64;
        for (size_t s = 0; s < S; ++s)
            if (n[s] > nres) {
                amps += std::ldexp(1.0, n[s]);
                fewest = std::min(fewest, n[s]);
            }
        b->B = batch_frame_qubits(dtype, amps, fewest);
        b->info.samples = S;
        std::vector<TileSample> tiles;
        for (size_t s = 0; s < S; ++s) {
            const bool resident = n[s] <= nres;
            b->samples.push_back(BSample{0, basis_idx[s]});
            size_t passes = 0;
            prx_plan *P = nullptr;
            if (n[s] >= TB) ++b->info.tile_samples;
            if (n[s] >= TB && n[s] <= 14) b->counted.push_back(*sched[s]);
            if (!resident) {
                tile_cfg.B = b->B;
                tile_cfg.max_virtual = b->B - kMinTileLow;
                prx_status st = plan_create_cfg(sched[s], n[s], dtype, tile_cfg, &P);
                if (st != PRX_OK) {
                    delete b;
                    return st;
                }
                if (n[s] > 14) passes = P->passes.size();
                TileSample ts;
                ts.sample = (uint32_t)s;
                ts.nsets = (uint32_t)(1ull << (n[s] - b->B));
                const uint32_t chunk_base = append_tables(b, P, csz, rsz);
                for (const Pass &ps : P->passes) {
                    if (ps.kind != kTile || ps.B != b->B || ps.m != kBatchTileM) {
                        prx_plan_destroy(P);
                        delete b;
                        return fail(PRX_ERR_UNSUPPORTED, "tile-only plan with another pass kind");
                    }
                    TileArgs ta;
                    tile_args(n[s], dtype, ps, ta);
                    ta.chunk_begin += chunk_base;
                    ts.passes.push_back(ta);
                    ts.rots.push_back((uint32_t)(ps.r1 - ps.r0));
                }
                tiles.push_back(std::move(ts));
                prx_plan_destroy(P);
            }
            if (resident) {
                res_cfg.B = n[s];
                prx_status st = plan_create_cfg(sched[s], n[s], dtype, res_cfg, &P);
                if (st != PRX_OK) {
                    delete b;
                    return st;
                }
                if (n[s] < TB) passes = P->passes.size();
                if (!P->chunks.empty()) {
                    BResident r;
                    std::memset(&r, 0, sizeof(r));
                    r.n = (uint32_t)n[s];
                    r.chunk_count = (uint32_t)P->chunks.size();
                    r.chunk_begin = append_tables(b, P, csz, rsz);
                    b->residents.push_back(r);
                    b->rsrc.push_back((uint32_t)s);
                }
                prx_plan_destroy(P);
            }
            count_passes(b->info, passes, n[s]);
        }
        make_launches(b);
        make_rounds(b, tiles);
        size_t o = 0;
        b->off_samples = o;   o = al256(o + S * sizeof(BSample));
        b->off_residents = o; o = al256(o + b->residents.size() * sizeof(BResident));
        b->off_tpasses = o;   o = al256(o + b->tpasses.size() * sizeof(BTilePass));
        b->off_tfirst = o;    o = al256(o + b->tfirst.size() * sizeof(uint32_t));
        b->off_chunks = o;    o = al256(o + b->chunks.size());
        b->off_rots = o;      o = al256(o + b->rots.size() + kRecordReadAhead);
        b->total = o;
    } catch (const std::bad_alloc &) {
        delete b;
        return fail(PRX_ERR_OOM, "out of host memory");
    }
    *out = b;
    return PRX_OK;
}

size_t prx_batch_workspace_bytes(const prx_batch *b) { return b ? b->total : 0; }

prx_status prx_batch_get_info(const prx_batch *b, prx_batch_info *out) {
    if (!b || !out) return fail(PRX_ERR_INVALID, "null pointer");
    prx_batch_info info = b->info;
    // samples up to two qubits above the tile size report the passes of narrow
    // frames, whatever they run: planned here, where they are asked for
    PlanCfg c = tile_settings();
    c.narrow = true;
    c.B = batch_tile_qubits(b->dtype);
    c.max_virtual = c.B - kMinTileLow;
    for (const prx_sched &s : b->counted) {
        prx_plan *P = nullptr;
        const prx_status st = plan_create_cfg(&s, s.n, b->dtype, c, &P);
        if (st != PRX_OK) return st;
        count_passes(info, P->passes.size(), s.n);
        prx_plan_destroy(P);
    }
    *out = info;
    return PRX_OK;
}

prx_status prx_batch_upload(prx_batch *b, void *const *psi, void *ws, size_t ws_bytes,
                            void *stream) {
    if (!b || !psi || !ws) return fail(PRX_ERR_INVALID, "null pointer");
    if (ws_bytes < b->total) return fail(PRX_ERR_INVALID, "workspace too small");
    if ((uintptr_t)ws & 255) return fail(PRX_ERR_INVALID, "workspace not 256-byte aligned");
    for (size_t s = 0; s < b->S; ++s) {
        if (!psi[s] || ((uintptr_t)psi[s] & 15))
            return fail(PRX_ERR_INVALID, "null or misaligned state pointer");
        b->samples[s].psi = (uint64_t)(uintptr_t)psi[s];
    }
    for (size_t t = 0; t < b->tpasses.size(); ++t) b->tpasses[t].psi = b->samples[b->tsrc[t]].psi;
    for (size_t r = 0; r < b->residents.size(); ++r)
        b->residents[r].psi = b->samples[b->rsrc[r]].psi;
    hipStream_t st = (hipStream_t)stream;
    char *w = (char *)ws;
    const struct {
        size_t off;
        const void *src;
        size_t bytes;
    } tables[] = {
        {b->off_samples, b->samples.data(), b->S * sizeof(BSample)},
        {b->off_residents, b->residents.data(), b->residents.size() * sizeof(BResident)},
        {b->off_tpasses, b->tpasses.data(), b->tpasses.size() * sizeof(BTilePass)},
        {b->off_tfirst, b->tfirst.data(), b->tfirst.size() * sizeof(uint32_t)},
        {b->off_chunks, b->chunks.data(), b->chunks.size()},
        {b->off_rots, b->rots.data(), b->rots.size()},
    };
    for (const auto &t : tables)
        if (t.bytes)
            PRX_HIP(hipMemcpyAsync(w + t.off, t.src, t.bytes, hipMemcpyHostToDevice, st));
    PRX_HIP(hipStreamSynchronize(st));
    return PRX_OK;
}

// The resident samples' launches.
static prx_status execute_residents(const prx_batch *b, char *w, hipStream_t st) {
    const void *chunks = w + b->off_chunks, *rots = w + b->off_rots;
    const uint64_t cap = b->max_grid ? b->max_grid : kTileGridCap;
    for (const prx_batch::Launch &l : b->launches) {
        const BResident *r = (const BResident *)(w + b->off_residents) + l.first;
        const unsigned grid = (unsigned)std::min<uint64_t>(l.count, cap);
        PRX_HIP(b->dtype == PRX_C64
                    ? launch_residents<float>(l.B, grid, r, l.count, chunks, rots, st)
                    : launch_residents<double>(l.B, grid, r, l.count, chunks, rots, st));
    }
    return PRX_OK;
}

// The tile samples' rounds.
static prx_status execute_rounds(const prx_batch *b, char *w, hipStream_t st) {
    const void *chunks = w + b->off_chunks, *rots = w + b->off_rots;
    const uint64_t cap = b->max_grid ? b->max_grid : kTileGridCap;
    const uint64_t tcap = std::min(cap, kTileGridCap);
    int dev = 0, cus = 256;
    PRX_HIP(hipGetDevice(&dev));
    PRX_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    // (128 KiB sets: one resident workgroup per CU)
    const uint64_t rcap = b->B == 14 ? std::min<uint64_t>(tcap, std::max(1, cus)) : tcap;
    for (const prx_batch::Round &r : b->rounds) {
        const BTilePass *ps = (const BTilePass *)(w + b->off_tpasses) + r.begin;
        const uint32_t *first = (const uint32_t *)(w + b->off_tfirst) + r.begin;
        const unsigned grid = (unsigned)std::min<uint64_t>(r.items, rcap);
        PRX_HIP(b->dtype == PRX_C64
                    ? launch_round<float>(b->B, grid, ps, first, r.count, r.items, chunks, rots, st)
                    : launch_round<double>(b->B, grid, ps, first, r.count, r.items, chunks, rots, st));
    }
    return PRX_OK;
}

static prx_status execute_overlaps(const prx_batch *b, char *w, double *overlaps_dev,
                                   hipStream_t st) {
    const unsigned rb = (unsigned)((b->S + 255) / 256);
    const BSample *samples = (const BSample *)(w + b->off_samples);
    if (b->dtype == PRX_C64)
        hipLaunchKernelGGL(k_batch_overlaps<float>, dim3(rb), dim3(256), 0, st, samples,
                           (uint32_t)b->S, overlaps_dev);
    else
        hipLaunchKernelGGL(k_batch_overlaps<double>, dim3(rb), dim3(256), 0, st, samples,
                           (uint32_t)b->S, overlaps_dev);
    PRX_HIP(hipGetLastError());
    return PRX_OK;
}

prx_status prx_batch_execute(const prx_batch *b, void *ws, size_t ws_bytes,
                             double *overlaps_dev, void *stream) {
    if (!b || !ws || !overlaps_dev) return fail(PRX_ERR_INVALID, "null pointer");
    if (ws_bytes < b->total) return fail(PRX_ERR_INVALID, "workspace too small");
    hipStream_t st = (hipStream_t)stream;
    char *w = (char *)ws;
    prx_status rc = execute_residents(b, w, st);
    if (rc == PRX_OK) rc = execute_rounds(b, w, st);
    if (rc == PRX_OK) rc = execute_overlaps(b, w, overlaps_dev, st);
    return rc;
}

prx_status prx_batch_set_max_grid(prx_batch *b, unsigned max_grid) {
    if (!b) return fail(PRX_ERR_INVALID, "null batch");
    b->max_grid = max_grid;
    return PRX_OK;
}

prx_status prx_batch_check(const prx_batch *b, const void *ws, void *stream) {
    if (!b || !ws) return fail(PRX_ERR_INVALID, "null pointer");
    PRX_HIP(hipStreamSynchronize((hipStream_t)stream));
    PRX_HIP(hipGetLastError());
    return PRX_OK;
}

void prx_batch_destroy(prx_batch *b) { delete b; }

prx_status prx_batch_run(size_t S, void *const *psi, const int *n, const prx_sched *const *sched,
                         prx_dtype dtype, const uint64_t *basis_idx, double *overlaps, void *ws,
                         size_t ws_bytes, void *stream) {
    if (!overlaps) return fail(PRX_ERR_INVALID, "null pointer");
    prx_batch *b = nullptr;
    prx_status st = prx_batch_create(S, n, sched, dtype, basis_idx, &b);
    if (st != PRX_OK) return st;
    // overlaps land after the batch tables in the workspace
    const size_t need = b->total + al256(2 * S * sizeof(double));
    if (ws_bytes < need) {
        prx_batch_destroy(b);
        return fail(PRX_ERR_INVALID, "workspace too small (need prx_batch_workspace_bytes + 16 S)");
    }
    double *ov_dev = (double *)((char *)ws + b->total);
    st = prx_batch_upload(b, psi, ws, ws_bytes, stream);
    if (st == PRX_OK) st = prx_batch_execute(b, ws, ws_bytes, ov_dev, stream);
    if (st == PRX_OK) st = prx_batch_check(b, ws, stream);
    if (st == PRX_OK) {
        hipError_t e = hipMemcpyAsync(overlaps, ov_dev, 2 * S * sizeof(double),
                                      hipMemcpyDeviceToHost, (hipStream_t)stream);
        if (e == hipSuccess) e = hipStreamSynchronize((hipStream_t)stream);
        if (e != hipSuccess) st = hip_fail(e, "overlap copy");
    }
    prx_batch_destroy(b);
    return st;
}

// ----------------------------------------------------------------- graphs

static prx_status capture_end(hipStream_t st, prx_status body, prx_graph **out) {
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamEndCapture(st, &g);
    if (body != PRX_OK) {
        if (g) (void)hipGraphDestroy(g);
        return body;
    }
    if (e != hipSuccess) return hip_fail(e, "hipStreamEndCapture");
    prx_graph *G = new (std::nothrow) prx_graph;
    if (!G) {
        (void)hipGraphDestroy(g);
        return fail(PRX_ERR_OOM, "out of host memory");
    }
    G->graph = g;
    e = hipGraphInstantiate(&G->exec, g, nullptr, nullptr, 0);
    if (e != hipSuccess) {
        (void)hipGraphDestroy(g);
        delete G;
        return hip_fail(e, "hipGraphInstantiate");
    }
    *out = G;
    return PRX_OK;
}

// A stream and two events beside the caller's stream while a batch's graph is
// captured; they end with the capture.
struct Side {
    hipStream_t st = nullptr;
    hipEvent_t begin = nullptr, end = nullptr;
    bool open() {
        const bool ok = hipStreamCreateWithFlags(&st, hipStreamNonBlocking) == hipSuccess &&
                        hipEventCreateWithFlags(&begin, hipEventDisableTiming) == hipSuccess &&
                        hipEventCreateWithFlags(&end, hipEventDisableTiming) == hipSuccess;
        if (!ok) (void)hipGetLastError();
        return ok;
    }
    ~Side() {
        if (end) (void)hipEventDestroy(end);
        if (begin) (void)hipEventDestroy(begin);
        if (st) (void)hipStreamDestroy(st);
    }
};

// The resident samples in a branch of their own beside the rounds (the
// samples' states are disjoint).  One workgroup takes all passes of a resident
// sample, 60 to 200 us on one CU each; the rounds of a few larger samples
// leave most of the chip idle meanwhile.  Measured, one branch / two (us per
// graph launch): 12 samples of 11 to 16 qubits complex128 187 / 132, 38 of 10
// to 15 complex64 161 / 102, 9 of 12 to 20 complex128 1785 / 1513, 95 of 13 to
// 19 complex64 2702 / 2396, 167 of 13 to 15 814 / 591; with residents or
// rounds alone nothing changes.
static prx_status execute_forked(const prx_batch *b, char *w, double *overlaps_dev,
                                 hipStream_t st, const Side &side) {
    PRX_HIP(hipEventRecord(side.begin, st));
    PRX_HIP(hipStreamWaitEvent(side.st, side.begin, 0));
    prx_status rc = execute_residents(b, w, side.st);
    if (rc == PRX_OK) rc = execute_rounds(b, w, st);
    PRX_HIP(hipEventRecord(side.end, side.st));
    PRX_HIP(hipStreamWaitEvent(st, side.end, 0));
    if (rc == PRX_OK) rc = execute_overlaps(b, w, overlaps_dev, st);
    return rc;
}

prx_status prx_batch_graph(const prx_batch *b, void *ws, size_t ws_bytes, double *overlaps_dev,
                           void *stream, prx_graph **out) {
    if (!out) return fail(PRX_ERR_INVALID, "null pointer");
    if (!stream) return fail(PRX_ERR_INVALID, "capture needs a non-default stream");
    hipStream_t st = (hipStream_t)stream;
    Side side;
    const bool fork = b && ws && overlaps_dev && ws_bytes >= b->total && !b->launches.empty() &&
                      !b->rounds.empty() && side.open();
    PRX_HIP(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
    prx_status body = fork ? execute_forked(b, (char *)ws, overlaps_dev, st, side)
                           : prx_batch_execute(b, ws, ws_bytes, overlaps_dev, stream);
    return capture_end(st, body, out);
}

prx_status prx_plan_graph(const prx_plan *p, void *psi, void *ws, size_t ws_bytes, void *stream,
                          prx_graph **out) {
    if (!out) return fail(PRX_ERR_INVALID, "null pointer");
    if (!stream) return fail(PRX_ERR_INVALID, "capture needs a non-default stream");
    hipStream_t st = (hipStream_t)stream;
    PRX_HIP(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
    prx_status body = prx_plan_execute(p, psi, ws, ws_bytes, stream);
    return capture_end(st, body, out);
}

prx_status prx_graph_launch(const prx_graph *g, void *stream) {
    if (!g) return fail(PRX_ERR_INVALID, "null graph");
    PRX_HIP(hipGraphLaunch(g->exec, (hipStream_t)stream));
    return PRX_OK;
}

void prx_graph_destroy(prx_graph *g) {
    if (!g) return;
    if (g->exec) (void)hipGraphExecDestroy(g->exec);
    if (g->graph) (void)hipGraphDestroy(g->graph);
    delete g;
}

}  // extern "C"
