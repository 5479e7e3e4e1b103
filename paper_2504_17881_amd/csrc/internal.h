// Internal declarations shared by the host code (sched.cpp, plan.cpp, tune.cpp) and the HIP
// kernels (kernels.hip, batch.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <string>

#include "prx.h"

namespace prx {

// ---------------------------------------------------------------- errors
void set_error(const std::string &msg);
prx_status fail(prx_status st, const std::string &msg);
prx_status hip_fail(hipError_t e, const char *what);

#define PRX_HIP(call)                                                  \
    do {                                                               \
        hipError_t e_ = (call);                                        \
        if (e_ != hipSuccess) return ::prx::hip_fail(e_, #call);       \
    } while (0)

// ------------------------------------------------------- device tables
//
// One record per rotation of a fused (span or tile) pass.  The rotation
// exp(i phi P) is applied in the factored form
//     new[k] = cos(phi) * ( psi[k] + tau * sigma(k') * psi[k'] ),
// k' = k XOR x, sigma(j) = (-1)^{popcount(j & z)}, tau = i^{nY+1} tan(phi)
// (nY = popcount(x & z)); the cos(phi) factors of a pass are multiplied
// into one scale applied when the pass stores the state.  For x = 0 the
// partner is k itself.
//
// Pair updates run in place: with a = psi[k] (the pair's element whose
// basis bit is clear) and b = psi[k'],
//     a <- a + tau_a s_b b,   then   b <- b + tau_b s_a a   (new a),
// s_a, s_b the signs sigma; for imaginary tau both terms carry a factor i.
// This equals the 2x2 update when b is stored divided by kappa = 1 -/+
// tau^2 and a per-slot factor K is carried: tau_a = tau K, tau_b =
// tau / (K kappa), K <- K kappa.  An element's stored value times the
// product of K over the basis slots set in its coset label is its true
// value; chunks (and span passes) record those K as `fscale`.
//
//   z      : z mask in the frame the kernel indexes (span: global index;
//            tile: workgroup-local index)
//   zhigh  : tile only: z restricted to the tile-index bits, for the sign
//            contributed by the workgroup's base tile
//   info   : bits 0-3  basis slot of x in the chunk (15 = diagonal, x = 0)
//            bit  4    tau is imaginary (nY + 1 odd)
//            bit  5    static-sign variant (chunk rank <= kStaticSignRank)
//            bits 8-15 zeta: bit i = parity(basis_i & z)
//            bits 16-23 variant index (static-sign chunks)
//   jump   : variant index times the stride of the lean loop of the plan's
//            kind (resident or tile chunks)
//   tau_a, tau_b : signed magnitudes (real or imaginary parts); for x = 0
//            only tau_a is used (tan(phi))
template <typename T>
struct RotRec {
    uint64_t z;
    uint64_t zhigh;
    uint32_t info;
    uint32_t jump;  // rank-4 records: the variant's byte offset in the lean loops' tables
    T tau_a;
    T tau_b;
};

// Bytes of one variant of the lean rotation loop of resident states, and what
// those of tile chunks have more (checked against the built code).
template <typename T>
static constexpr uint32_t kLeanStride = sizeof(T) == 4 ? 324u : 340u;
static constexpr uint32_t kLeanTileMore = 8u;

static constexpr uint32_t kSlotDiag = 15;
// Chunks of rank up to kStaticSignRank run one compiled variant per
// (slot, imag, sign pattern); their records carry the variant index in
// info bits 16..23 and tau_a multiplied by (-1)^zeta_slot.
static constexpr int kStaticSignRank = 4;
static constexpr int kMaxChunkRank = 6;
// Virtual qubits of a tile pass: at most 10 XOR masks of tile-index bits,
// and at least 16 contiguous amplitudes per tile (128 B at complex64).
static constexpr int kMaxVirtual = 10;
static constexpr int kMinTileLow = 4;
// Readable bytes after a rotation table: the threaded rotation loops load
// the record after the current one (32 bytes at complex64, 40 at
// complex128) before they know whether one follows.
static constexpr size_t kRecordReadAhead = 64;

// Most threads of a tile workgroup (2^(B - m) <= 2^10).
static constexpr int kMaxTileThreadBits = 10;

// A chunk of a tile pass: up to kMaxChunkRank basis directions in the
// workgroup-local frame and a run of rotations whose x masks are basis
// directions (or zero).  Thread t holds the coset k0(t) XOR span(basis),
// k0(t) = XOR of cvec[i] over the bits i set in t; the cvec span a
// complement of the basis span, and the first ones have independent low
// bits so that the lanes of one LDS access cycle use distinct banks.
struct ChunkHead {
    uint32_t rot_begin;
    uint32_t rot_count;
    uint32_t flags;  // resident plans: kChunk* bits
    uint32_t basis[kMaxChunkRank];
    uint16_t cvec[kMaxTileThreadBits];
    double scale;    // resident plans, complex128: at a pass's last chunk its scale;
                     // complex64: what the factors' roundings leave on average
};
// The device record, in cache lines: the head, then the factors of the coset
// labels in the state's precision (label v's pending factor, the product of
// the chunk's per-slot factors K over the bits set in v; v < 2^m, m <= 5; in
// resident complex64 plans times the cosines of the chunk's rotations).  A
// rank-4 complex64 chunk reads two lines.
template <typename T>
struct ChunkRec {
    ChunkHead h;
    T fac[32];
};
static_assert(sizeof(ChunkHead) == 64 && sizeof(ChunkRec<float>) == 192 &&
              sizeof(ChunkRec<double>) == 320, "whole cache lines");
static constexpr uint32_t kChunkPassEnd = 1;   // last chunk of a pass: takes its scale (complex128)
static constexpr uint32_t kChunkRenormIn = 2;  // takes the renormalisation factor in force
static constexpr uint32_t kChunkNormOut = 4;   // the norm after it makes the next factor

// Longest run of rotations in one chunk (bounds the pending factors: with
// tau^2 <= 1/2 each kappa lies in [1/2, 3/2]).
static constexpr int kMaxChunkRots = 64;

// Kernel arguments of a span pass (one chunk in the global frame).
struct SpanArgs {
    uint64_t basis[kMaxChunkRank];
    uint32_t pivot[kMaxChunkRank];
    uint32_t rot_begin, rot_count;
    int n;
    double scale;                  // product of the pass's cosines
    double fscale[kMaxChunkRank];  // pending per-slot factors K
};

// State accesses of the tile workgroups that own one tile-set, by the bytes of
// state a sequence of passes comes back to.  Between the L2s' 32 MiB and the
// 256 MiB of the last-level cache, ordinary accesses keep it there (12-qubit
// passes of a qDRIFT sequence: 24 qubits complex64 53 us against 59 us
// non-temporal, 25 qubits 95 / 112; 24 qubits complex128 96 / 114).  Larger
// states stream through (28 qubits complex64 854 / 811 us), and what the L2s
// hold is written back during a pass rather than at its end (21 qubits
// complex64 17.8 / 16.0 us, 20 qubits complex128 17.2 / 15.5).
static inline bool streams_state(double bytes) {
    return bytes <= 32.0 * 1048576.0 || bytes > 256.0 * 1048576.0;
}

// State accesses of a plain sweep, which has nothing else to wait for.  States
// above 256 MiB stream (us per sweep, ordinary / non-temporal: 28 qubits
// complex64 pair 781 / 727, diagonal 764 / 686; 26 qubits complex128 378 / 346
// and 384 / 336).  A sequence of sweeps over a smaller state is best served by
// the L2s and the last-level cache (18 qubits complex64 3.2 / 3.4, 22 qubits
// 10.8 / 12.0, 24 qubits alike), except that a sweep beside the streaming
// passes of a fused plan goes with them.
static inline bool plain_streams(double bytes, bool beside_fused) {
    return beside_fused ? streams_state(bytes) : bytes > 256.0 * 1048576.0;
}

// Kernel arguments of a tile pass.
struct TileArgs {
    // Slot s = tid + u NT of the tile-set holds amplitude
    // ((t ^ vc(tid >> b)) << b | (tid & (2^b - 1))) ^ uoff[u], with vc(v) the
    // XOR of the virtual masks selected by v's bits.
    uint64_t uoff[32];  // 2^m entries (tile chunk rank m <= 5)
    uint64_t vmask[kMaxVirtual];  // virtual masks (tile-index space): tile v of a workgroup's
                                  // set is t XOR (the masks selected by the bits of v)
    uint64_t tpivots;             // pivot bits of the masks' echelon form, ascending,
                                  // 6 bits each (pivot i in bits 6i .. 6i+5)
    int n, b, g;
    int stream;      // non-temporal state accesses (see streams_state)
    uint32_t chunk_begin, chunk_count;
    double scale;
};

// Renormalisation hand-off from the pass before: p null, none; count 0, *p is
// the factor; else the factor is 1 / sqrt of the sum of p[0 .. count).
struct RenormIn {
    const double *p;
    unsigned count;
};
// Partials a pass sums itself (every wave reads them all, 4 KB at most: 8 per
// lane at 512).  A 200-rotation qDRIFT plan of 22 qubits, whose passes leave
// 512: 271 us through a launch of its own, 253 summed by the next pass.  With
// 1024 the gain is used up (12-qubit frames at 22 qubits: 605 / 607 us), with
// 2048 the sums cost more than the launch (23 qubits: 1081 / 1231).
static constexpr unsigned kRenormDirect = 512;
static constexpr unsigned kRenormOneBlock = 16384;

// Arguments of a single-rotation sweep.
struct PlainArgs {
    uint64_t x, z;
    int n;
    int pivot;       // highest set bit of x (pair kernels)
    int nY_odd;      // popcount(x & z) odd
    int beta_imag;   // beta = i^{nY+1} sin(phi) is imaginary
    int stream;      // non-temporal state accesses (see plain_streams)
    double c;        // cos(phi)
    double beta;     // signed magnitude of beta
};

// Arguments of a qubit-relabelling pass: a permutation of the index bits
// at the kPermBits positions pos[0..11] (ascending; pos[j] = j for j < 4,
// the 16 contiguous amplitudes that coalesce one access), all other bits
// fixed.  Group coordinate s in [0, 2^12) has bit j at index bit pos[j];
// the element at input coordinate s moves to output coordinate D(s), which
// has bit dst[j] set for every bit j of s.  The kernel needs, for output
// coordinate s' = t + 256 u (thread t, slot u), the input coordinate
// D^-1(s') = D^-1(t) XOR D^-1(256 u); inv[j] is D^-1 of bit j, and ioff[u]
// = D^-1(256 u) is precomputed on the host.
static constexpr int kPermBits = 12;
struct PermArgs {
    uint32_t pos[kPermBits];
    uint16_t inv[kPermBits];
    uint16_t ioff[16];
    int n;
};

// Autotune cache (tune.cpp), keyed by (arch, n, dtype).
bool tune_lookup(int n, prx_dtype dt, prx_plan_opts *out);
void tune_store(int n, prx_dtype dt, const prx_plan_opts &o);

struct PlanCfg;
// Plan with explicit internal settings (batched plans).
prx_status plan_create_cfg(const prx_sched *sched, int n, prx_dtype dtype, const PlanCfg &cfg,
                           prx_plan **out);
// Plan of a range whose default plan's tables are too large: span passes, which
// have no chunk records, wherever a frame of n - B masks covers no more.
prx_status plan_create_small(const prx_sched *sched, int n, prx_dtype dtype, size_t begin,
                             size_t end, prx_kernel kernel, prx_plan **out);

// ------------------------------------------------------------ launchers
// All enqueue on `stream` and return hipGetLastError() of the launch.
// `cap` limits the workgroups of a launch (at most kMaxGridBlocks), `blocks`
// is their number (span_blocks, tile_launch_blocks); the kernels stride over
// the rest.
hipError_t launch_plain(prx_dtype dt, void *psi, const PlainArgs &a, hipStream_t s,
                        unsigned cap);
hipError_t launch_span(prx_dtype dt, int m, void *psi, const SpanArgs &a, const void *rots,
                       const RenormIn &renorm_in, double *norm_out, hipStream_t s,
                       unsigned blocks);
hipError_t launch_tile(prx_dtype dt, int B, int m, void *psi, const TileArgs &a,
                       const void *rots, const void *chunks, const RenormIn &renorm_in,
                       double *norm_out, hipStream_t s, unsigned blocks);
// Resident plans: a state of up to resident_max_qubits(dt) qubits stays in one
// workgroup's LDS for chunks [chunk_begin, +chunk_count), whatever passes they
// belong to.  rin (nullable): the renormalisation factor on entry; rout
// (nullable) receives the one on exit.
static constexpr int kResidentMinQubits = 4;
static constexpr int resident_max_qubits(prx_dtype dt) { return dt == PRX_C64 ? 14 : 13; }
hipError_t launch_resident(prx_dtype dt, void *psi, int n, const void *rots, const void *chunks,
                           uint32_t chunk_begin, uint32_t chunk_count, const double *rin,
                           double *rout, hipStream_t s);
unsigned resident_threads(int n);
// Qubit relabelling: one pass over the state, in place (every 2^12-element
// group is closed under the permutation).
hipError_t launch_permute(prx_dtype dt, void *psi, const PermArgs &a, hipStream_t s,
                          unsigned cap);
unsigned permute_blocks(int n, unsigned cap);
// partial sums -> 1/sqrt(sum) into scale_out[0]; scale_out[1 .. kRenormStage]
// is stage-1 scratch (two fixed-shape kernels, deterministic)
static constexpr unsigned kRenormStage = 128;
hipError_t launch_renorm_finish(const double *partials, unsigned count, double *scale_out,
                                hipStream_t s);
// Workgroups of one launch: at most kMaxGridBlocks (at 256 threads, 2^30
// work-items, inside a dispatch's 32-bit work-item range); the kernels
// stride over the rest.
static constexpr uint64_t kMaxGridBlocks = 1ull << 22;
unsigned span_blocks(int n, int m, unsigned cap);
unsigned tile_blocks(int n, int B, unsigned cap);
// the workgroups of a tile pass's launch: tile_blocks, or for the persistent
// shapes those resident on the device, if fewer
unsigned tile_launch_blocks(prx_dtype dt, int B, int m, int n, unsigned cap);
unsigned plain_blocks(int n, bool diag, unsigned cap);
bool span_supported(prx_dtype dt, int m);
bool tile_supported(prx_dtype dt, int B, int m);

// Reductions.  `part` holds kReduceBlocks * 2 doubles of partials; `out` (2
// doubles) is memory that the device writes: a workspace or a host slot.
static constexpr unsigned kReduceBlocks = 1024;
static constexpr unsigned kReduceThreads = 512;
hipError_t launch_overlap(prx_dtype dt, const void *psi0, const void *psi, int n, double *part,
                          double *out, hipStream_t s);
hipError_t launch_norm2(prx_dtype dt, const void *psi, int n, double *part, double *out,
                        hipStream_t s);
hipError_t launch_scale(prx_dtype dt, void *psi, int n, double scale, hipStream_t s);

}  // namespace prx
