// Split D3Q19 step of periodic lattices (arXiv:1711.02003, Sec. II, Eqs.
// (1)-(11)), pair or compact state, FP32 or FP16 storage: the fused step as
// two kernels, one thread per node.
//
// The column sweeps (lbcg_fused.hip, lbcg_compact_sweep.h) step a 64 x 8 tile
// through a chunk of planes, 4 to 9 us per plane with a barrier in each.  A
// lattice of a few hundred thousand nodes has too few tiles for 256 CUs: it
// needs chunks of two or three planes, which then pull twice as many, and a
// 45-wide tile leaves a third of the lanes idle.  Here:
//   moments: every node pulls its 19 populations, takes the 12 collision
//     moments and psi and writes them (52 bytes);
//   collide: every node forms the gradient from its neighbours' psi, collides
//     and stores its new state.
// Threads are numbered along a plane (x fastest, rows run together), so every
// lane works whatever the width, and the grid has a thread per node.  The
// price is the moments written and read back, 104 bytes per node, and a
// second launch, so large lattices stay on the sweeps (split_faster).
// Every value is formed by the sweeps' expressions in their order: the
// results are bitwise the sweeps'.
//
// The moments take no memory of their own.  On the pair state they go to the
// buffer that the step writes, into slots of the node's own pairs (FP32: 6
// pairs of 8 bytes, FP16: 12 of 4), which only that node's collision reads
// and then overwrites; on the compact state to the pair buffer that holds no
// state.
//
// What bounds it: memory (FP32: 412 bytes per node on the pair state at
// 4.8 TB/s on 210 x 150 x 131) and, with FP16 storage, arithmetic as much;
// below ~100 000 nodes the two launches.  Measured per step, us, the sweep in
// its default / its best timed shape -> this: pair FP32 45 x 38 x 53
// 62 / 20 -> 10.8, 96^3 135 / 92 -> 62, 210 x 150 x 131 548 / 398 -> 355;
// pair FP16 96^3 126 / 92 -> 46; compact FP32 70 x 50 x 90 53 / 38 -> 25,
// 96^3 98 / 68 -> 61; compact FP16 96^3 101 / 67 -> 44.
#include "lbcg_split.h"

namespace lbcg {

namespace {

constexpr int kSB = 256;  // threads per block

// FP32 pair slots are 8 bytes wide, and a compact step's moments lie in a
// buffer of their own; the FP16 pair state's slots hold one float each.
template <typename S, bool COMPACT_OUT>
constexpr bool kPaired = COMPACT_OUT || sizeof(S) == 4;

// The node of this thread in block `item`: (x, y) of plane z, element p of
// the plane.
struct PNode {
    uint32_t p, x, y, z;
};
__device__ __forceinline__ bool p_node(const SplitDesc &a, uint32_t item, PNode &h) {
    h.z = uint32_t(uniform(int(div_by(item, a.div0))));
    h.p = (item - h.z * a.div0.d) * kSB + threadIdx.x;
    h.y = div_by(h.p, a.div1);
    h.x = h.p - h.y * uint32_t(a.nx);
    return h.p < uint32_t(a.nx) * uint32_t(a.ny);
}

template <typename S, bool COMPACT_IN, bool PAIRED>
__device__ __forceinline__ void p_moments(const SplitDesc &a, uint32_t item) {
    PNode h;
    if (!p_node(a, item, h)) return;
    const Around<true> ar(h.x, h.y, h.z, uint32_t(a.nx), uint32_t(a.ny), uint32_t(a.nz));
    Mom<float> m;
    if constexpr (COMPACT_IN) {
        CPops<D3Q19, float> q;
        pull_compact<S>(a.in, a.pitch, ar, q);
        moments<D3Q19, float>(q, m);
    } else {
        Pops<D3Q19, float> q;
        pull_pairs<S>(a.in, a.pitch, ar, q);
        moments<D3Q19, float>(q, m);
    }
    put_psi(a.psi, a.pitch, h.p, ar.zp[1], float(psi_of<float>(m.drho, m.r36R, m.r36B)));
    MomStore<PAIRED>::put(a.mom, a.pitch, h.p, ar.zp[1], m);
}

// Gradient, collision and store (COMPACT: totals and record, else pairs).
template <typename S, bool COMPACT>
__device__ __forceinline__ void p_collide(const SplitDesc &a, uint32_t item) {
    using L = D3Q19;
    if (item == 0 && threadIdx.x == 0) *a.ctr_out = *a.ctr_in + 1u;
    PNode h;
    if (!p_node(a, item, h)) return;
    const Around<true> ar(h.x, h.y, h.z, uint32_t(a.nx), uint32_t(a.ny), uint32_t(a.nz));
    uint32_t step = 0;  // seeds the stochastic rounding of FP16 storage
    if constexpr (sizeof(S) == 2) step = *a.ctr_in;
    float F[3], mv[kSplitMoments];
    MomStore<kPaired<S, COMPACT>>::get(a.mom, a.pitch, h.p, ar.zp[1], mv);
    split_gradient<false>(a.psi, a.pitch, ar, F);
    if constexpr (COMPACT) {
        typedef CStore<S> St;
        CompactOut<L, float> o;
        split_collide(a.mo, mv, F, o);
        const __amdgpu_buffer_rsrc_t rout =
            state_rsrc(static_cast<uint8_t *>(a.out), a.pitch * (uint32_t(L::Q) * St::E + St::kRecA + St::kRecB));
        St::store(rout, h.p * St::E, ar.zp[1], a.pitch, o, step);
    } else {
        typedef typename PairOf<S>::type P2;
        constexpr uint32_t E = sizeof(P2);
        PostOut<L, float> o;
        split_collide(a.mo, mv, F, o);
        Dither dz(step, h.p + ar.zp[1]);
        const __amdgpu_buffer_rsrc_t rout = state_rsrc(static_cast<S *>(a.out), uint32_t(L::Q) * a.pitch * E);
#pragma unroll
        for (int i = 0; i < L::Q; ++i)
            store_pair<P2>(rout, h.p * E, uint32_t(su((uint32_t(i) * a.pitch + ar.zp[1]) * E)),
                           encode_step<L, S, float>(o.df[i], o.mm[i], o.red(i), i, dz));
    }
}

template <typename S, bool COMPACT_IN, bool PAIRED>
__global__ void __launch_bounds__(kSB) k_split_moments(SplitDesc a) {
    p_moments<S, COMPACT_IN, PAIRED>(a, banded(a.nblocks));
}
template <typename S, bool COMPACT>
__global__ void __launch_bounds__(kSB) k_split_collide(SplitDesc a) {
    p_collide<S, COMPACT>(a, banded(a.nblocks));
}
// Many lattices in one launch.
template <typename S, bool COMPACT>
__global__ void __launch_bounds__(kSB) k_split_moments_batch(const SplitDesc *__restrict__ desc,
                                                             const LatMap *__restrict__ map) {
    uint32_t item;
    const int lat = find_lat(*map, banded(gridDim.x), item);
    const SplitDesc a = desc[lat];
    p_moments<S, COMPACT, kPaired<S, COMPACT>>(a, item);
}
template <typename S, bool COMPACT>
__global__ void __launch_bounds__(kSB) k_split_collide_batch(const SplitDesc *__restrict__ desc,
                                                             const LatMap *__restrict__ map) {
    uint32_t item;
    const int lat = find_lat(*map, banded(gridDim.x), item);
    const SplitDesc a = desc[lat];
    p_collide<S, COMPACT>(a, item);
}

template <typename S>
hipError_t run(const SplitDesc &a, bool compact_in, bool compact_out, hipStream_t s) {
    const dim3 grid{a.nblocks}, block{unsigned(kSB)};
    if (compact_in)
        hipLaunchKernelGGL((k_split_moments<S, true, true>), grid, block, 0, s, a);
    else if (compact_out)
        hipLaunchKernelGGL((k_split_moments<S, false, true>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL((k_split_moments<S, false, kPaired<S, false>>), grid, block, 0, s, a);
    if (compact_out)
        hipLaunchKernelGGL((k_split_collide<S, true>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL((k_split_collide<S, false>), grid, block, 0, s, a);
    return hipGetLastError();
}

template <typename S, bool COMPACT>
hipError_t run_batch(const SplitDesc *desc, const LatMap *map, uint32_t blocks, hipStream_t s) {
    const dim3 grid{blocks}, block{unsigned(kSB)};
    hipLaunchKernelGGL((k_split_moments_batch<S, COMPACT>), grid, block, 0, s, desc, map);
    hipLaunchKernelGGL((k_split_collide_batch<S, COMPACT>), grid, block, 0, s, desc, map);
    return hipGetLastError();
}

}  // namespace

// 32-bit byte offsets must cover a pair state (the moments, 48 bytes per
// node, are smaller), and blocks a 31-bit count.
bool psplit_supported(int prec, const Geo &g) {
    const int64_t bpp = (int64_t(g.nx) * g.ny + kSB - 1) / kSB;
    return !g.mask && (prec == 1 || prec == 2) &&
           uint64_t(2 * D3Q19::Q) * uint64_t(g.pitch) * (prec == 1 ? 4u : 2u) < (uint64_t(1) << 32) &&
           bpp * g.nz <= 0x7fffffff;
}

SplitDesc psplit_desc(const Geo &g, const ModelD &md, const void *in, void *out, bool compact, void *psi, void *mom,
                      const uint32_t *ctr_in, uint32_t *ctr_out) {
    SplitDesc a{};
    a.in = in;
    a.out = out;
    a.psi = static_cast<float *>(psi);
    a.mom = compact ? mom : out;
    a.nx = g.nx;
    a.ny = g.ny;
    a.nz = g.nz;
    a.pitch = uint32_t(g.pitch);
    const uint32_t bpp = uint32_t((int64_t(g.nx) * g.ny + kSB - 1) / kSB);
    a.nblocks = bpp * uint32_t(g.nz);
    a.div0 = fast_div(bpp);
    a.div1 = fast_div(uint32_t(g.nx));
    a.ctr_in = ctr_in;
    a.ctr_out = ctr_out;
    a.mo = to_model<float>(md);
    return a;
}

hipError_t launch_step_psplit(int prec, const Geo &g, const ModelD &md, const void *in, bool compact_in, void *out,
                              bool compact_out, void *psi, void *mom, const uint32_t *ctr_in, uint32_t *ctr_out,
                              hipStream_t s) {
    if (md.bgk || !psi || (compact_in && !compact_out) || (compact_out && !mom) || !psplit_supported(prec, g))
        return hipErrorInvalidValue;
    const SplitDesc a = psplit_desc(g, md, in, out, compact_out, psi, mom, ctr_in, ctr_out);
    return prec == 1 ? run<float>(a, compact_in, compact_out, s) : run<_Float16>(a, compact_in, compact_out, s);
}

hipError_t launch_step_psplit_batch(int prec, bool compact, const SplitDesc *desc, const LatMap *map, uint32_t blocks,
                                    hipStream_t s) {
    if (blocks == 0) return hipSuccess;
    if (prec == 1)
        return compact ? run_batch<float, true>(desc, map, blocks, s) : run_batch<float, false>(desc, map, blocks, s);
    return compact ? run_batch<_Float16, true>(desc, map, blocks, s) : run_batch<_Float16, false>(desc, map, blocks, s);
}

}  // namespace lbcg
