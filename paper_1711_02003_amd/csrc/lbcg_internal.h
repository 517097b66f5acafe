// Internal interface between the C-ABI runtime and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbcg_device.h"

namespace lbcg {

// Model parameters in double; launchers convert to the compute type.
struct ModelD {
    double ivR, ivB, Abar, beta, aR, aB, eps_F;  // ivR, ivB: 1/nu_k
    double w0;  // rest weight of the lattice
    double omR, omB;  // 1/tau_k
    int bgk;    // 0 regularized, 1 BGK at the node's rate, 2 BGK per colour
};

template <typename T>
inline Model<T> to_model(const ModelD &m) {
    Model<T> r;
    r.ivR = T(m.ivR);
    r.ivB = T(m.ivB);
    r.Abar = T(m.Abar);
    r.beta = T(m.beta);
    r.aR = T(m.aR);
    r.aB = T(m.aB);
    r.dR0 = T(m.aR - m.w0);
    r.dB0 = T(m.aB - m.w0);
    r.kR = T((m.w0 - m.aR) / (1.0 - m.w0));
    r.kB = T((m.w0 - m.aB) / (1.0 - m.w0));
    r.eps_F = T(m.eps_F);
    r.omR = T(m.omR);
    r.omB = T(m.omB);
    r.bgk = m.bgk;
    return r;
}

// Number of doubles per block in the diagnostics partials.
constexpr int kDiagVals = 13;
// Blocks of the diagnostics reduction (partials = kDiagBlocks * kDiagVals).
constexpr int kDiagBlocks = 1024;

// lattice: 0 = D2Q9, 1 = D3Q19; prec: 0 = F64, 1 = F32, 2 = F16.
// Equilibrium state (Eq. (6)) of nodes [n0, n0 + cnt) from chunk-local fields
// rhoR, rhoB (cnt each) and u (3 * cnt, component-major, nullable).
hipError_t launch_init(int lattice, int prec, const Geo &g, const ModelD &md, int64_t n0, int64_t cnt,
                       const double *rhoR, const double *rhoB, const double *u, void *st, hipStream_t s);
hipError_t launch_psi(int lattice, int prec, const Geo &g, const ModelD &md, const void *st,
                      bool pulled, void *psi, hipStream_t s);
// ctr_in / ctr_out: the time-step counter read by this step and the slot
// that receives its successor (device memory, one uint32 each).
hipError_t launch_step_generic(int lattice, int prec, const Geo &g, const ModelD &md,
                               const void *in, bool pulled, const void *psi, void *out,
                               const uint32_t *ctr_in, uint32_t *ctr_out, hipStream_t s);
// Fields of nodes [n0, n0 + cnt): out = rhoR | rhoB | ux | uy | uz | psi (cnt each).
hipError_t launch_fields(int lattice, int prec, const Geo &g, const ModelD &md, const void *st,
                         bool pulled, int64_t n0, int64_t cnt, double *out, hipStream_t s);
// Populations of nodes [n0, n0 + cnt): out[(k * Q + i) * cnt + (n - n0)].
hipError_t launch_pops(int lattice, int prec, const Geo &g, const ModelD &md, const void *st,
                       bool pulled, int64_t n0, int64_t cnt, double *out, hipStream_t s);
// Populations of cnt listed nodes: out[(j * 2 + k) * Q + i].
hipError_t launch_pops_at(int lattice, int prec, const Geo &g, const ModelD &md, const void *st,
                          bool pulled, const int64_t *nodes, int64_t cnt, double *out, hipStream_t s);
// Deterministic two-stage FP64 reduction into res[kDiagVals].
hipError_t launch_diag(int lattice, int prec, const Geo &g, const ModelD &md, const void *st,
                       bool pulled, double *partials, double *res, hipStream_t s);

// Fused single-pass D3Q19 step; F32 or F16 storage, with or without geometry;
// the regularized collision, or plain BGK (md.bgk: 8-row tiles only).
struct FusedShape {
    int rows;     // rows of the x-y tile (one wave of 64 nodes per row)
    int zchunks;  // z range split per column of tiles
    int tx = 64;  // tile width (the compact D3Q19 sweep: 64 or 32)
    // periodic D3Q19 lattices: the split step of lbcg_split.hip instead of
    // the sweep (rows, zchunks and tx then only say which sweep it replaces)
    bool split = false;
};

// Kernel view of one lattice for the fused sweep.
template <typename S>
struct FusedArgs {
    const S *in;
    S *out;
    int nx, ny, nz;
    int64_t pitch;
    const uint8_t *mask;  // nullptr = every node fluid
    const DevInlet *inlets;
    const DevOutlet *outlets;
    const DevWall *walls;
    const uint32_t *links;   // link words (with a mask)
    const uint32_t *ctr_in;  // time-step counter of this step
    uint32_t *ctr_out;       // receives ctr_in + 1
    int ntx, nty, zchunks;
};
template <typename S>
FusedArgs<S> fused_args(const Geo &g, const void *in, void *out, const uint32_t *ctr_in, uint32_t *ctr_out,
                        FusedShape sh);

hipError_t launch_step_fused(int prec, const Geo &g, const ModelD &md, const void *in, void *out,
                             const uint32_t *ctr_in, uint32_t *ctr_out, FusedShape shape, hipStream_t s);
bool fused_supported(int lattice, int prec, const Geo &g);
// Blocks of the fused kernel that fit on the device at once (pops: its plain
// BGK form).
int fused_resident_blocks(int prec, int rows, bool masked, bool pops = false);

// Split D3Q19 steps (F32 or F16 storage, regularized): a moments kernel writes
// psi and the kSplitMoments collision moments of every fluid node, a collision
// kernel takes the gradient, collides and stores, with geometry the boundary
// values too.  Bitwise the column sweeps' results.
constexpr int kSplitMoments = 12;
constexpr int kBatchLatMax = 256;           // lattices of a batched split launch

// Unsigned division by a constant of the launch: n / d = mulhi(n, mul) >> sh
// for n < 2^31 (d > 1).  With s = floor(log2 d) and mul = ceil(2^(32 + s) / d)
// the error mul d - 2^(32 + s) is below d < 2^(s + 1), so n < 2^31 divides
// exactly; a power of two takes s - 1, whose mul is 2^31 exactly.
struct FastDiv {
    uint32_t d, mul, sh;
};
inline FastDiv fast_div(uint32_t d) {
    FastDiv f{d, 0, 0};
    if (d <= 1) return f;
    uint32_t s = 31u - uint32_t(__builtin_clz(d));
    if ((d & (d - 1)) == 0) --s;
    f.sh = s;
    f.mul = uint32_t(((uint64_t(1) << (32 + s)) + d - 1) / d);
    return f;
}
__device__ __forceinline__ uint32_t div_by(uint32_t n, const FastDiv &f) {
    return f.d <= 1 ? n : __umulhi(n, f.mul) >> f.sh;
}

// Kernel view of one lattice for the split steps.  Periodic: blocks of 256
// consecutive nodes of a plane (div0: blocks per plane, div1: nx); with
// geometry: blocks of 256 entries of the list of fluid nodes (div0: nx, div1:
// ny).
struct SplitDesc {
    const void *in;  // state read (pairs or compact)
    void *out;       // state written
    float *psi;      // psi of every node; with geometry what a non-fluid node shows the gradient
    void *mom;       // moments, kSplitMoments floats per node
    int nx, ny, nz;
    uint32_t pitch;
    uint32_t nblocks;  // of the moments and collision kernels
    FastDiv div0, div1;
    const uint32_t *ctr_in;
    uint32_t *ctr_out;
    // geometry
    const uint32_t *list;  // fluid nodes {node, link word}
    uint32_t count;
    const uint8_t *mask;
    const DevInlet *inlets;
    const DevOutlet *outlets;
    Model<float> mo;
};

// List of the fluid nodes of a lattice with geometry, built on the device once
// per lattice in `scratch` (split_scratch_bytes).
size_t split_scratch_bytes(int64_t pitch);
struct SplitPlan {
    int64_t fluid = 0;  // its length
    int64_t io = 0;     // nodes with inlet or outlet links
};
// Builds the list and writes what the non-fluid nodes show the gradient into
// the scratch's psi; returns the length (waits for the stream).
hipError_t split_prepare(const Geo &g, void *scratch, SplitPlan &sp, hipStream_t s);

// A step of one lattice.  Periodic: compact_in / compact_out: the state read /
// written is compact (else pairs); mom (compact_out only; a pair step keeps
// its moments in `out`): kSplitMoments * pitch floats.
hipError_t launch_step_psplit(int prec, const Geo &g, const ModelD &md, const void *in, bool compact_in, void *out,
                              bool compact_out, void *psi, void *mom, const uint32_t *ctr_in, uint32_t *ctr_out,
                              hipStream_t s);
hipError_t launch_step_split(int prec, const Geo &g, const ModelD &md, const void *in, void *out, void *scratch,
                             const SplitPlan &sp, const uint32_t *ctr_in, uint32_t *ctr_out, hipStream_t s);
// The split step on the compact state (D3Q19 F32 or F16 with geometry): reads the
// compact state `in` (or, with pair_in, the pair state `in`, on the first
// step after an initialisation or a restore), the inlet and outlet values in
// the pair buffer gin, writes the compact state `cout` and the new inlet and
// outlet values into the pair buffer gout.
hipError_t launch_step_cgeo(int prec, const Geo &g, const ModelD &md, bool pair_in, const void *in, const void *gin,
                            void *cout, void *gout, void *scratch, const SplitPlan &sp, const uint32_t *ctr_in,
                            uint32_t *ctr_out, hipStream_t s);
// Its compact state as pairs (fluid nodes and wall values) into pout, which
// already holds the inlet and outlet values.
hipError_t launch_expand_cgeo(int prec, const Geo &g, const void *cin, void *pout, void *scratch, const SplitPlan &sp,
                              hipStream_t s);

bool psplit_supported(int prec, const Geo &g);

// The same steps of many lattices, a launch per kernel: descriptors and block
// maps in device memory.  A block map says which lattice a block belongs to:
// block b is block b - start[q] of lattice lat[q] for the last q with start[q]
// <= b.  A launch of start[k] blocks steps the first k lattices of the map.
struct LatMap {
    int n;
    uint32_t start[kBatchLatMax + 1];
    uint8_t lat[kBatchLatMax];
};
hipError_t launch_step_psplit_batch(int prec, bool compact, const SplitDesc *desc, const LatMap *map, uint32_t blocks,
                                    hipStream_t s);
hipError_t launch_step_split_batch(int prec, const SplitDesc *desc, const LatMap *map, uint32_t blocks, hipStream_t s);
// Descriptors of one lattice's step (compact: periodic lattices on the compact
// state; else the pair state).
SplitDesc psplit_desc(const Geo &g, const ModelD &md, const void *in, void *out, bool compact, void *psi, void *mom,
                      const uint32_t *ctr_in, uint32_t *ctr_out);
SplitDesc split_desc(const Geo &g, const ModelD &md, const void *in, void *out, void *scratch, const SplitPlan &sp,
                     const uint32_t *ctr_in, uint32_t *ctr_out);

// Fused single-pass D2Q9 step over tiles (lbcg_tile2d.hip): F64, F32 or F16
// storage, with or without geometry, any collision form.
hipError_t launch_step_tile2d(int prec, const Geo &g, const ModelD &md, const void *in, void *out,
                              const uint32_t *ctr_in, uint32_t *ctr_out, hipStream_t s);
bool tile2d_supported(int prec, const Geo &g);

// Fused D3Q19 step on the compact state (periodic, regularized, tiles of 8
// rows, FP32 or FP16 storage): 19 arrays of pitch totals and 5 colour
// scalars per node in two record arrays, kCompactBytes (FP32) or
// kCompactBytes16 (FP16) per pitch node.  pair_in: `in` is a pair state of
// the same precision (the first step after an initialisation or a restore);
// `out` is always compact.
constexpr int kCompactBytes = 19 * 4 + 20;    // D3Q19, FP32: 19 totals, 5 scalars
constexpr int kCompactBytes16 = 19 * 2 + 12;  // D3Q19, FP16 (M kept FP32)
constexpr int kCompactBytes2d = 9 * 4 + 16;   // D2Q9: 9 totals, 4 scalars
hipError_t launch_step_compact(int prec, const Geo &g, const ModelD &md, const void *in, bool pair_in, void *out,
                               const uint32_t *ctr_in, uint32_t *ctr_out, FusedShape shape, hipStream_t s);
bool compact_supported(int lattice, int prec, const Geo &g);
int compact_resident_blocks(int tile_width, int prec);
// Pair state (post-collision, as the pair kernels store it) of a compact state.
hipError_t launch_expand(int prec, const Geo &g, const void *cin, void *pout, hipStream_t s);
// The D2Q9 step on the compact state (periodic, FP32, regularized): 9 arrays
// of pitch floats and 4 colour scalars per node in one record array,
// kCompactBytes2d per pitch node.
hipError_t launch_step_compact2d(const Geo &g, const ModelD &md, const void *in, bool pair_in, void *out,
                                 const uint32_t *ctr_in, uint32_t *ctr_out, hipStream_t s);
hipError_t launch_expand2d(const Geo &g, const void *cin, void *pout, hipStream_t s);

// Batched fused step: one launch steps many lattices by one time level.
// Block b sweeps work item bitem[b] (tile-major (tile, z chunk) index) of
// lattice blat[b], described by desc[blat[b]].
template <typename S>
struct BatchDesc {
    FusedArgs<S> a;
    Model<float> mo;
};
hipError_t launch_step_fused_batch(int prec, const void *desc, const int *blat, const int *bitem, int nblocks,
                                   int rows, bool masked, hipStream_t s);
// Batched compact step: desc are BatchDesc<float> of compact lattices (in,
// out: compact buffers of storage prec, 1 = F32 or 2 = F16; shapes of 8
// rows).
hipError_t launch_step_compact_batch(int prec, const void *desc, const int *blat, const int *bitem, int nblocks,
                                     hipStream_t s);

}  // namespace lbcg
