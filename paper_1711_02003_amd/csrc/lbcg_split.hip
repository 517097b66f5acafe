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
// second launch, so large lattices stay on the sweeps (split_preferred).
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
#include "lbcg_buffer.h"
#include "lbcg_compact_sweep.h"  // CStore: the compact state's storage
#include "lbcg_internal.h"

namespace lbcg {

namespace {

constexpr int kSB = 256;   // threads per block
constexpr int kSXCD = 8;

// Unsigned division by a constant of the launch: n / d = mulhi(n, mul) >> sh
// for n < 2^31 (d > 1).  With s = floor(log2 d) and mul = ceil(2^(32 + s) / d)
// the error mul d - 2^(32 + s) is below d < 2^(s + 1), so n < 2^31 divides
// exactly; a power of two takes s - 1, whose mul is 2^31 exactly.
struct FastDiv {
    uint32_t d, mul, sh;
};
FastDiv fast_div(uint32_t d) {
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

struct PArgs {
    const void *in;  // state read
    void *out;       // state written
    float *psi;      // pitch floats
    void *mom;       // kSplitMoments * pitch floats (MomStore)
    int nx, ny, nz;
    uint32_t pitch;
    uint32_t bpp;    // blocks per plane
    FastDiv bydiv, nxdiv;
    const uint32_t *ctr_in;
    uint32_t *ctr_out;
};

// The node of this thread: (x, y) of plane z, element p of the plane; blocks
// are dealt to the 8 XCDs in contiguous bands of planes, so that a node's
// neighbours' psi mostly come from its own XCD's L2.
struct PNode {
    uint32_t p, x, y, z;
};
__device__ __forceinline__ bool p_node(const PArgs &a, PNode &h) {
    const uint32_t total = a.bpp * uint32_t(a.nz);
    const uint32_t xcd = blockIdx.x % kSXCD, l = blockIdx.x / kSXCD;
    const uint32_t item = xcd * (total / kSXCD) + min(xcd, total % kSXCD) + l;
    h.z = uint32_t(uniform(int(div_by(item, a.bydiv))));
    h.p = (item - h.z * a.bpp) * kSB + threadIdx.x;
    h.y = div_by(h.p, a.nxdiv);
    h.x = h.p - h.y * uint32_t(a.nx);
    return h.p < uint32_t(a.nx) * uint32_t(a.ny);
}

// Elements x' + nx y' of the 9 columns x' = x + dx, y' = y + dy, entry
// (dx + 1) + 3 (dy + 1), and the first elements of planes z - 1, z, z + 1,
// periodic.
__device__ __forceinline__ void p_columns(const PArgs &a, const PNode &h, uint32_t t[9], uint32_t zp[3]) {
    const uint32_t nx = uint32_t(a.nx), ny = uint32_t(a.ny), nz = uint32_t(a.nz);
    const uint32_t xs[3] = {h.x == 0 ? nx - 1 : h.x - 1, h.x, h.x == nx - 1 ? 0 : h.x + 1};
    const uint32_t rows[3] = {(h.y == 0 ? ny - 1 : h.y - 1) * nx, h.p - h.x, (h.y == ny - 1 ? 0 : h.y + 1) * nx};
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int c = 0; c < 3; ++c) t[c + 3 * b] = xs[c] + rows[b];
    const uint32_t plane = nx * ny;
    zp[0] = (h.z == 0 ? nz - 1 : h.z - 1) * plane;
    zp[1] = h.z * plane;
    zp[2] = (h.z == nz - 1 ? 0 : h.z + 1) * plane;
}

// Storage of the moments: float pairs (6 arrays of pitch pairs, one 8-byte
// access each), or single floats (12 arrays of pitch floats) where they share
// the FP16 pair state's 4-byte slots.
template <bool PAIRED>
struct MomStore {
    static constexpr int n = PAIRED ? kSplitMoments / 2 : kSplitMoments;
    static constexpr uint32_t E = PAIRED ? 8 : 4;
    __device__ static __forceinline__ void put(const PArgs &a, const PNode &h, uint32_t zcol,
                                               const float v[kSplitMoments]) {
        const __amdgpu_buffer_rsrc_t r = state_rsrc(static_cast<float *>(a.mom), a.pitch * E * uint32_t(n));
#pragma unroll
        for (int k = 0; k < n; ++k) {
            const int so = su((uint32_t(k) * a.pitch + zcol) * E);
            if constexpr (PAIRED) {
                const f2 w = {v[2 * k], v[2 * k + 1]};
                __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, w), r, int(h.p * E), so, 0);
            } else {
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[k]), r, int(h.p * E), so, 0);
            }
        }
    }
    __device__ static __forceinline__ void get(const PArgs &a, const PNode &h, uint32_t zcol, float v[kSplitMoments]) {
        const __amdgpu_buffer_rsrc_t r = state_rsrc(static_cast<float *>(a.mom), a.pitch * E * uint32_t(n));
#pragma unroll
        for (int k = 0; k < n; ++k) {
            const int so = su((uint32_t(k) * a.pitch + zcol) * E);
            if constexpr (PAIRED) {
                const f2 w = __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b64(r, int(h.p * E), so, 0));
                v[2 * k] = w.x;
                v[2 * k + 1] = w.y;
            } else {
                v[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, int(h.p * E), so, 0));
            }
        }
    }
};

template <bool PAIRED>
__device__ __forceinline__ void put_moments(const PArgs &a, const PNode &h, uint32_t zcol, const Mom<float> &m) {
    const __amdgpu_buffer_rsrc_t rp = state_rsrc(a.psi, a.pitch * 4u);
    const float v[kSplitMoments] = {m.drho, m.r36R, m.r36B, m.j[0], m.j[1], m.j[2],
                                    m.S[0], m.S[1], m.S[2], m.S[3], m.S[4], m.S[5]};
    const float psi = float(psi_of<float>(m.drho, m.r36R, m.r36B));
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(psi), rp, int(h.p * 4u), su(zcol * 4u), 0);
    MomStore<PAIRED>::put(a, h, zcol, v);
}

// Moments and psi from the pair state.
template <typename S, bool PAIRED>
__device__ __forceinline__ void moments_pairs(const PArgs &a) {
    using L = D3Q19;
    typedef typename PairOf<S>::type P2;
    constexpr uint32_t E = sizeof(P2);
    PNode h;
    if (!p_node(a, h)) return;
    uint32_t t[9], zp[3];
    p_columns(a, h, t, zp);
    const __amdgpu_buffer_rsrc_t rin = state_rsrc(a.in, uint32_t(L::Q) * a.pitch * E);
    P2 v[L::Q];
#pragma unroll
    for (int i = 0; i < L::Q; ++i)
        v[i] = load_pair<P2>(rin, t[(1 - L::cx[i]) + 3 * (1 - L::cy[i])] * E,
                             uint32_t(su((uint32_t(i) * a.pitch + zp[1 - L::cz[i]]) * E)));
    Pops<L, float> q;
    q.red = 0;
#pragma unroll
    for (int i = 0; i < L::Q; ++i) decode_pair<L, S, float>(v[i], i, q);
    Mom<float> m;
    moments<L, float>(q, m);
    put_moments<PAIRED>(a, h, zp[1], m);
}

// Moments and psi from the compact state: each pulled total split with its
// sender's record (from the cache: a record serves 19 receivers).
template <typename S, bool PAIRED>
__device__ __forceinline__ void moments_compact(const PArgs &a) {
    using L = D3Q19;
    typedef CStore<S> St;
    PNode h;
    if (!p_node(a, h)) return;
    uint32_t t[9], zp[3];
    p_columns(a, h, t, zp);
    const uint32_t base = uint32_t(L::Q) * a.pitch * St::E;
    const __amdgpu_buffer_rsrc_t rin = state_rsrc(a.in, base + a.pitch * (St::kRecA + St::kRecB));
    CPops<L, float> q;
    q.red = 0;
#pragma unroll
    for (int i = 0; i < L::Q; ++i) {
        const uint32_t c = t[(1 - L::cx[i]) + 3 * (1 - L::cy[i])], z = zp[1 - L::cz[i]];
        const typename St::Raw d = St::load(rin, c * St::E, (uint32_t(i) * a.pitch + z) * St::E);
        const typename St::RawA ra = St::load_a(rin, c * St::kRecA, base + z * St::kRecA);
        const typename St::RawB rb = St::load_b(rin, c * St::kRecB, base + a.pitch * St::kRecA + z * St::kRecB);
        const f4 e = St::entry(ra, rb);
        bool fl;
        q.df[i] = St::df(d, i);
        q.mm[i] = Codec<float>::col<float>(e[0], fl);
        const int cv[3] = {L::cx[i], L::cy[i], L::cz[i]};
        const int n2 = csq<L>(i);
        if (n2 == 0) {
            q.vd[i] = 0.0f;
        } else if (n2 == 1) {
            const int ax = cv[0] ? 0 : (cv[1] ? 1 : 2);
            q.vd[i] = cv[ax] > 0 ? e[1 + ax] : -e[1 + ax];
        } else {
            const int a0 = cv[0] ? 0 : 1, a1 = cv[2] ? 2 : 1;
            const float s0 = cv[a0] > 0 ? e[1 + a0] : -e[1 + a0];
            q.vd[i] = St::ratio(rb) * (cv[a1] > 0 ? s0 + e[1 + a1] : s0 - e[1 + a1]);
        }
        q.red |= fl ? (1u << i) : 0u;
    }
    Mom<float> m;
    moments<L, float>(q, m);
    put_moments<PAIRED>(a, h, zp[1], m);
}

// FP32 pair slots are 8 bytes wide, and a compact step's moments lie in a
// buffer of their own; the FP16 pair state's slots hold one float each.
template <typename S, bool COMPACT_OUT>
constexpr bool kPaired = COMPACT_OUT || sizeof(S) == 4;

// Gradient, collision and store (COMPACT: totals and record, else pairs).
template <typename S, bool COMPACT>
__device__ __forceinline__ void collide_node(const PArgs &a, const Model<float> &mo) {
    using L = D3Q19;
    typedef float T;
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.ctr_out = *a.ctr_in + 1u;
    PNode h;
    if (!p_node(a, h)) return;
    uint32_t t[9], zp[3];
    p_columns(a, h, t, zp);
    uint32_t step = 0;  // seeds the stochastic rounding of FP16 storage
    if constexpr (sizeof(S) == 2) step = *a.ctr_in;
    const __amdgpu_buffer_rsrc_t rp = state_rsrc(a.psi, a.pitch * 4u);
    float pv[L::Q];
#pragma unroll
    for (int i = 1; i < L::Q; ++i)
        pv[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
            rp, int(t[(1 + L::cx[i]) + 3 * (1 + L::cy[i])] * 4u), su(zp[1 + L::cz[i]] * 4u), 0));
    float mv[kSplitMoments];
    MomStore<kPaired<S, COMPACT>>::get(a, h, zp[1], mv);
    T fx = 0, fy = 0, fz = 0;
#pragma unroll
    for (int i = 1; i < L::Q; ++i) {
        const T wp = T(3.0 * wgt<L>(i)) * T(pv[i]);
        if (L::cx[i]) fx += L::cx[i] > 0 ? wp : -wp;
        if (L::cy[i]) fy += L::cy[i] > 0 ? wp : -wp;
        if (L::cz[i]) fz += L::cz[i] > 0 ? wp : -wp;
    }
    const T F[3] = {fx, fy, fz};
    const T cj[3] = {mv[3], mv[4], mv[5]}, cS[6] = {mv[6], mv[7], mv[8], mv[9], mv[10], mv[11]};
    if constexpr (COMPACT) {
        typedef CStore<S> St;
        CompactOut<L, T> o;
        collide<L, T>(mo, mv[0], mv[1], mv[2], cj, cS, F, nullptr, o);
        const __amdgpu_buffer_rsrc_t rout =
            state_rsrc(a.out, a.pitch * (uint32_t(L::Q) * St::E + St::kRecA + St::kRecB));
        St::store(rout, h.p * St::E, zp[1], a.pitch, o, step);
    } else {
        typedef typename PairOf<S>::type P2;
        constexpr uint32_t E = sizeof(P2);
        PostOut<L, T> o;
        collide<L, T>(mo, mv[0], mv[1], mv[2], cj, cS, F, nullptr, o);
        Dither dz(step, h.p + zp[1]);
        const __amdgpu_buffer_rsrc_t rout = state_rsrc(a.out, uint32_t(L::Q) * a.pitch * E);
#pragma unroll
        for (int i = 0; i < L::Q; ++i)
            store_pair<P2>(rout, h.p * E, uint32_t(su((uint32_t(i) * a.pitch + zp[1]) * E)),
                           encode_step<L, S, T>(o.df[i], o.mm[i], (o.red >> i) & 1u, i, dz));
    }
}

template <typename S, bool COMPACT_IN, bool PAIRED>
__global__ void __launch_bounds__(kSB) k_split_moments(PArgs a) {
    if constexpr (COMPACT_IN)
        moments_compact<S, PAIRED>(a);
    else
        moments_pairs<S, PAIRED>(a);
}
template <typename S, bool COMPACT>
__global__ void __launch_bounds__(kSB) k_split_collide(PArgs a, Model<float> mo) {
    collide_node<S, COMPACT>(a, mo);
}

template <typename S>
hipError_t run(const PArgs &a, const Model<float> &mo, bool compact_in, bool compact_out, hipStream_t s) {
    const dim3 grid{a.bpp * unsigned(a.nz)}, block{unsigned(kSB)};
    if (compact_in)
        hipLaunchKernelGGL((k_split_moments<S, true, true>), grid, block, 0, s, a);
    else if (compact_out)
        hipLaunchKernelGGL((k_split_moments<S, false, true>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL((k_split_moments<S, false, kPaired<S, false>>), grid, block, 0, s, a);
    if (compact_out)
        hipLaunchKernelGGL((k_split_collide<S, true>), grid, block, 0, s, a, mo);
    else
        hipLaunchKernelGGL((k_split_collide<S, false>), grid, block, 0, s, a, mo);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_step_psplit(int prec, const Geo &g, const ModelD &md, const void *in, bool compact_in, void *out,
                              bool compact_out, void *psi, void *mom, const uint32_t *ctr_in, uint32_t *ctr_out,
                              hipStream_t s) {
    if (g.mask || md.bgk || !psi || (compact_in && !compact_out) || (compact_out && !mom) ||
        (prec != 1 && prec != 2))
        return hipErrorInvalidValue;
    // 32-bit byte offsets must cover a pair state (the moments, 48 bytes per
    // node, are smaller)
    if (uint64_t(2 * D3Q19::Q) * uint64_t(g.pitch) * (prec == 1 ? 4u : 2u) >= (uint64_t(1) << 32))
        return hipErrorInvalidValue;
    PArgs a;
    a.in = in;
    a.out = out;
    a.psi = static_cast<float *>(psi);
    a.mom = compact_out ? mom : out;
    a.nx = g.nx;
    a.ny = g.ny;
    a.nz = g.nz;
    a.pitch = uint32_t(g.pitch);
    const int64_t plane = int64_t(g.nx) * g.ny;
    const int64_t bpp = (plane + kSB - 1) / kSB;
    if (bpp * g.nz > 0x7fffffff) return hipErrorInvalidValue;
    a.bpp = uint32_t(bpp);
    a.bydiv = fast_div(a.bpp);
    a.nxdiv = fast_div(uint32_t(g.nx));
    a.ctr_in = ctr_in;
    a.ctr_out = ctr_out;
    const Model<float> mo = to_model<float>(md);
    return prec == 1 ? run<float>(a, mo, compact_in, compact_out, s)
                     : run<_Float16>(a, mo, compact_in, compact_out, s);
}

}  // namespace lbcg
