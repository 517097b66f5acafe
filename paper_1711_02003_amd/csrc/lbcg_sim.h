// Internal layout of a simulation handle, shared by the single-lattice and
// batched runtimes.
#pragma once

#include "../../include/lbcg.h"
#include "lbcg_internal.h"

struct lbcg_sim {
    int lattice, prec, collision, kernel;
    bool auto_kernel;       // kernel was the library's choice
    int device;             // HIP device current at creation
    int Q, D;
    lbcg::Geo g;
    lbcg::ModelD md;
    lbcg::FusedShape shape;
    lbcg::FusedShape own_shape;  // chosen by lbcg_create or lbcg_tune (shape: also by lbcg_set_step_form)
    int form;               // LBCG_FORM_SWEEP or _SPLIT if lbcg_set_step_form chose it, else LBCG_FORM_AUTO
    size_t elem;            // bytes per stored value
    size_t state_bytes;     // one state buffer
    void *buf[2];
    int cur;                // buffer holding the current state
    bool pulled;            // true: buffer holds post-collision values (pull to read S_t)
    bool initialised;
    int64_t step;
    void *psi;              // generic phase-field scratch (N values of the compute type)
    void *moms;             // split geometry step: its scratch (split_scratch_bytes), or null
    int64_t fluid;          // fluid nodes
    lbcg::SplitPlan split;  // its node list's length
    double *partials, *diag;
    uint32_t *ctr;          // time-step counter pair: ctr[cur] = steps taken since initialisation
    double *staging;        // field / population staging
    int64_t staging_nodes;
    uint8_t *mask_dev;
    lbcg::DevInlet *in_dev;
    lbcg::DevOutlet *out_dev;
    hipStream_t stream;         // where the handle's work is queued
    hipStream_t owned_stream;   // the stream the library created for it, or null
    void *arena;
    bool own_arena;
    size_t arena_bytes;
    // Compact state (LBCG_KERNEL_COMPACT): cbuf[cur] holds the state while
    // compact is true; before a read of the state it is expanded into buf[cur]
    // (expanded marks that buf[cur] is current).
    void *cbuf[2];
    bool compact, expanded;
    hipGraphExec_t graph[2];  // graph_steps steps starting from buffer 0 / 1
    int graph_steps;
    bool graph_failed;
};

namespace lbcg {

// Reads `rows` values per node to the host (lbcg_readback.hip): `launch` queues
// the values of nodes [n0, n0 + cnt) into device memory as rows of cnt
// doubles; row r of all nodes goes to dst[r] (null: not read).  Synchronizes.
typedef hipError_t (*RowsLaunch)(lbcg_sim *s, int64_t n0, int64_t cnt, double *out);
hipError_t read_rows(lbcg_sim *s, RowsLaunch launch, int rows, double *const *dst);
// A handle comes and goes: the read slots are freed with the last one.
void slots_use();
void slots_release();

// Descriptor of a batched handle's step from buffer cur ^ par (0: its state)
// into the other on the split step.
inline SplitDesc batch_split_desc(const lbcg_sim *s, int par) {
    const int a = s->cur ^ par, b = a ^ 1;
    if (s->g.mask)
        return split_desc(s->g, s->md, s->buf[a], s->buf[b], s->moms, s->split, s->ctr + a, s->ctr + b);
    const bool cmp = s->kernel == LBCG_KERNEL_COMPACT;
    // (a compact step's moments go to the pair buffer that holds no state)
    return psplit_desc(s->g, s->md, cmp ? s->cbuf[a] : s->buf[a], cmp ? s->cbuf[b] : s->buf[b], cmp, s->psi,
                       s->buf[b], s->ctr + a, s->ctr + b);
}

// Whether the batched split step applies to the handle.
inline bool batch_split_ok(const lbcg_sim *s) {
    return s->collision == LBCG_REGULARIZED && (s->g.mask ? s->moms != nullptr : psplit_supported(s->prec, s->g));
}

// Expected us per time level of the handle's share of a batched launch, on the
// sweep (tiles of 64 x 8, z chunks of 32 planes, each with about three planes
// of halo and start; with geometry the tiles in proportion to the fluid) and
// on the split step, with the device full: the plane and node times of the
// single-lattice steps, and with geometry 10.3 us per plane and 90 ps per
// fluid node (FP16 8 us, 65 ps).
inline void batch_cost(const lbcg_sim *s, double &sweep, double &split) {
    const bool cmp = s->kernel == LBCG_KERNEL_COMPACT, half = s->prec == LBCG_F16, geo = s->g.mask != nullptr;
    const double plane = geo ? (half ? 8.0 : 10.3) : (half ? (cmp ? 4.7 : 6.5) : (cmp ? 4.9 : 8.6));
    const double node = geo ? (half ? 65e-6 : 90e-6) : (half ? (cmp ? 53e-6 : 54e-6) : (cmp ? 66e-6 : 80e-6));
    const double tiles = double((s->g.nx + 63) / 64) * double((s->g.ny + 7) / 8);
    const double planes = s->g.nz + 3.0 * ((s->g.nz + 31) / 32);
    sweep = tiles * planes * plane / 256.0 * (double(s->fluid) / double(s->g.N));
    split = double(s->fluid) * node;
}

}  // namespace lbcg
