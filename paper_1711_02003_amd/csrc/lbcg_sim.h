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
    int resident[2];        // blocks of the batched D3Q19 sweep that the device holds: tiles of 4, of 8 rows
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

// Relaxed capture mode for the calling thread: its allocations, frees and waits
// for streams that do not capture neither end a capture that another thread has
// begun in global mode nor fail for it (a wait for a stream does both otherwise).
class RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;

public:
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    RelaxedCapture(const RelaxedCapture &) = delete;
    RelaxedCapture &operator=(const RelaxedCapture &) = delete;
};

// Reads `rows` values per node to the host (lbcg_readback.hip): `launch` queues
// the values of nodes [n0, n0 + cnt) into device memory as rows of cnt
// doubles; row r of all nodes goes to dst[r] (null: not read).  Synchronizes.
typedef hipError_t (*RowsLaunch)(lbcg_sim *s, int64_t n0, int64_t cnt, double *out);
hipError_t read_rows(lbcg_sim *s, RowsLaunch launch, int rows, double *const *dst);
// A handle comes and goes: the read slots are freed with the last one (call it
// in relaxed capture mode).
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

// Times that the choices between a D3Q19 sweep and the split step are made by:
// us per plane iteration of a 64 x 8 sweep block with every CU busy, ps per
// fluid node of a single lattice's split step, and of a batched split launch,
// whose rate falls from `small` to `large` as its nodes grow from `from` to `to`
// million (the states no longer stay in the cache).  Batched split step, us
// measured: one 96^3 pairs FP32 58 (FP16 48), compact 65 (48); 128^3 143 (101),
// 151 (107); 256 x 128 x 128 336 (208), 316 (221); 64 boxes of 17.6 M nodes 1569
// (1025), 1541 (1180); four channels of 1.95 M fluid nodes 209 (159).
struct StepCost {
    double plane, node, small, large, from, to;
};
inline StepCost step_cost(const lbcg_sim *s) {
    const bool half = s->prec == LBCG_F16;
    if (s->g.mask) return half ? StepCost{12.9, 76, 76, 76, 1, 2} : StepCost{11.7, 98, 98, 98, 1, 2};
    if (s->kernel == LBCG_KERNEL_COMPACT)
        return half ? StepCost{4.7, 53, 46, 68, 2, 8} : StepCost{4.9, 66, 66, 88, 2, 8};
    return half ? StepCost{6.5, 54, 47, 58, 2, 8} : StepCost{8.6, 80, 65, 90, 2, 4};
}

// Expected us of one level of a group of lattices (all periodic or all with
// geometry) on the batched sweep in a given launch shape and on the batched split
// step.  The sweep's blocks run on `resident` places; each takes its planes and
// about three more.  Blocks of one length run in rounds; of mixed lengths, the
// places share the work, and the last of them wait for half a block on average.
// With geometry a tile counts in proportion to the fluid.  Sweep against split,
// measured (allocation-free step): 128^3 compact FP32 in chunks of 16 planes
// 112 / 151, of 64 320 / 151; 16 boxes of 3.7 M nodes FP32 pairs in chunks of 8
// planes 384 / 316; two junctions of 0.17 M fluid nodes 94 to 381 / 28.
struct GroupCost {
    const lbcg_sim *first = nullptr;
    double work = 0, items = 0, longest = 0, nodes = 0, resident = 1;
    void add(const lbcg_sim *s, int rows, int64_t zchunks) {
        const double part = double(s->fluid) / double(s->g.N);
        const double tiles = double((s->g.nx + 63) / 64) * double((s->g.ny + rows - 1) / rows) * part;
        const double planes = double((s->g.nz + zchunks - 1) / zchunks + 3);
        work += tiles * double(s->g.nz + 3 * zchunks);
        items += tiles * double(zchunks);
        if (planes > longest) longest = planes;
        nodes += double(s->fluid);
        if (!first) {
            first = s;
            resident = s->resident[rows == 8];
        }
    }
    double sweep_us() const {
        const double rounds = double(int64_t((items + resident - 1) / resident)) * longest;
        const double shared = work / resident + 0.5 * longest;
        return (rounds < shared ? rounds : shared) * step_cost(first).plane;
    }
    double split_us() const {
        const StepCost c = step_cost(first);
        double a = (nodes * 1e-6 - c.from) / (c.to - c.from);
        a = a < 0 ? 0 : (a > 1 ? 1 : a);
        return 6.0 + nodes * 1e-6 * (c.small + (c.large - c.small) * a);
    }
};

}  // namespace lbcg
