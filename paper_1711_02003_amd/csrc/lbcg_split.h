#pragma once
// Device code shared by the split D3Q19 steps (a moments kernel and a
// collision kernel, one thread per node): lbcg_split.hip (periodic) and
// lbcg_geo.hip (with geometry).
#include "lbcg_buffer.h"
#include "lbcg_compact_sweep.h"  // CStore: the compact state's storage
#include "lbcg_internal.h"

namespace lbcg {

namespace {

// psi that a neutral wall or an outlet shows the gradient: replaced by the
// fluid node's own
constexpr float kPsiOwn = 1e30f;

constexpr int kSXCD = 8;
// Contiguous bands of blocks per XCD (blocks go to the 8 XCDs round-robin),
// so that a node's neighbours' psi mostly come from its own XCD's L2.
__device__ __forceinline__ uint32_t banded(uint32_t total) {
    const uint32_t xcd = blockIdx.x % kSXCD, l = blockIdx.x / kSXCD;
    return xcd * (total / kSXCD) + min(xcd, total % kSXCD) + l;
}

// Storage of the moments: float pairs (6 arrays of pitch pairs, one 8-byte
// access each), or single floats (12 arrays of pitch floats) where they share
// the FP16 pair state's 4-byte slots.  p: element of the plane, zcol: first
// element of the plane.
template <bool PAIRED>
struct MomStore {
    static constexpr int n = PAIRED ? kSplitMoments / 2 : kSplitMoments;
    static constexpr uint32_t E = PAIRED ? 8 : 4;
    __device__ static __forceinline__ void put(void *mom, uint32_t pitch, uint32_t p, uint32_t zcol,
                                               const Mom<float> &m) {
        const float v[kSplitMoments] = {m.drho, m.r36R, m.r36B, m.j[0], m.j[1], m.j[2],
                                        m.S[0], m.S[1], m.S[2], m.S[3], m.S[4], m.S[5]};
        const __amdgpu_buffer_rsrc_t r = state_rsrc(static_cast<float *>(mom), pitch * E * uint32_t(n));
#pragma unroll
        for (int k = 0; k < n; ++k) {
            const int so = su((uint32_t(k) * pitch + zcol) * E);
            if constexpr (PAIRED) {
                const f2 w = {v[2 * k], v[2 * k + 1]};
                __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, w), r, int(p * E), so, 0);
            } else {
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[k]), r, int(p * E), so, 0);
            }
        }
    }
    __device__ static __forceinline__ void get(const void *mom, uint32_t pitch, uint32_t p, uint32_t zcol,
                                               float v[kSplitMoments]) {
        const __amdgpu_buffer_rsrc_t r = state_rsrc(static_cast<const float *>(mom), pitch * E * uint32_t(n));
#pragma unroll
        for (int k = 0; k < n; ++k) {
            const int so = su((uint32_t(k) * pitch + zcol) * E);
            if constexpr (PAIRED) {
                const f2 w = __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b64(r, int(p * E), so, 0));
                v[2 * k] = w.x;
                v[2 * k + 1] = w.y;
            } else {
                v[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, int(p * E), so, 0));
            }
        }
    }
};

// The moments in the node's slots of an FP16 compact state: nine floats as
// halves in the totals' 2-byte slots, three in the records' 12 bytes.
struct MomHalves {
    typedef CStore<_Float16> St;
    // per node: of a total, before each record, in all
    static constexpr uint32_t E = St::E, A = D3Q19::Q * E, B = A + St::kRecA, bytes = B + St::kRecB;
    __device__ static __forceinline__ void put(void *mom, uint32_t pitch, uint32_t p, uint32_t zcol,
                                               const Mom<float> &m) {
        const float v[kSplitMoments] = {m.drho, m.r36R, m.r36B, m.j[0], m.j[1], m.j[2],
                                        m.S[0], m.S[1], m.S[2], m.S[3], m.S[4], m.S[5]};
        const __amdgpu_buffer_rsrc_t r = state_rsrc(static_cast<uint8_t *>(mom), bytes * pitch);
#pragma unroll
        for (int k = 0; k < 18; ++k) {
            const uint32_t b = __float_as_uint(v[k / 2]);
            __builtin_amdgcn_raw_buffer_store_b16(uint16_t(k & 1 ? b >> 16 : b), r, int(p * E),
                                                  su((uint32_t(k) * pitch + zcol) * E), 0);
        }
        const f2 w = {v[9], v[10]};
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, w), r, int(p * St::kRecA),
                                              su(A * pitch + zcol * St::kRecA), 0);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[11]), r, int(p * St::kRecB),
                                              su(B * pitch + zcol * St::kRecB), 0);
    }
    __device__ static __forceinline__ void get(const void *mom, uint32_t pitch, uint32_t p, uint32_t zcol,
                                               float v[kSplitMoments]) {
        const __amdgpu_buffer_rsrc_t r = state_rsrc(static_cast<const uint8_t *>(mom), bytes * pitch);
        uint32_t h[18];
#pragma unroll
        for (int k = 0; k < 18; ++k)
            h[k] = __builtin_amdgcn_raw_buffer_load_b16(r, int(p * E), su((uint32_t(k) * pitch + zcol) * E), 0);
        const f2 w = __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b64(
                                                r, int(p * St::kRecA), su(A * pitch + zcol * St::kRecA), 0));
        v[11] = __uint_as_float(
            __builtin_amdgcn_raw_buffer_load_b32(r, int(p * St::kRecB), su(B * pitch + zcol * St::kRecB), 0));
#pragma unroll
        for (int k = 0; k < 9; ++k) v[k] = __uint_as_float(h[2 * k] | (h[2 * k + 1] << 16));
        v[9] = w.x;
        v[10] = w.y;
    }
};

__device__ __forceinline__ void put_psi(float *psi, uint32_t pitch, uint32_t p, uint32_t zcol, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), state_rsrc(psi, pitch * 4u), int(p * 4u), su(zcol * 4u), 0);
}

// The nodes around node (x, y, z), periodic.  With the plane uniform over the
// wave (UZ) a neighbour's address is a per-lane column of its plane and a
// plane offset in a scalar register; else the lane adds the two.
template <bool UZ>
struct Around {
    uint32_t t[9], zp[3];
    __device__ __forceinline__ Around(uint32_t x, uint32_t y, uint32_t z, uint32_t nx, uint32_t ny, uint32_t nz) {
        const uint32_t xs[3] = {x == 0 ? nx - 1 : x - 1, x, x == nx - 1 ? 0 : x + 1};
        const uint32_t rows[3] = {(y == 0 ? ny - 1 : y - 1) * nx, y * nx, (y == ny - 1 ? 0 : y + 1) * nx};
#pragma unroll
        for (int b = 0; b < 3; ++b)
#pragma unroll
            for (int c = 0; c < 3; ++c) t[c + 3 * b] = xs[c] + rows[b];
        const uint32_t plane = nx * ny;
        zp[0] = (z == 0 ? nz - 1 : z - 1) * plane;
        zp[1] = z * plane;
        zp[2] = (z == nz - 1 ? 0 : z + 1) * plane;
    }
    // lane and scalar part of node x + (dx, dy, dz)
    __device__ __forceinline__ uint32_t lane(int dx, int dy, int dz) const {
        const uint32_t c = t[(dx + 1) + 3 * (dy + 1)];
        return UZ ? c : c + zp[1 + dz];
    }
    __device__ __forceinline__ uint32_t base(int dz) const { return UZ ? zp[1 + dz] : 0u; }
    // of the upstream node x - c_i
    __device__ __forceinline__ uint32_t vo(int i) const { return lane(-D3Q19::cx[i], -D3Q19::cy[i], -D3Q19::cz[i]); }
    __device__ __forceinline__ uint32_t so(int i) const { return base(-D3Q19::cz[i]); }
};

// The 19 pairs that a node pulls, plain loads all (boundary values lie in the
// upstream nodes' slots).
template <typename S, bool UZ>
__device__ __forceinline__ void pull_pairs(const void *in, uint32_t pitch, const Around<UZ> &ar, Pops<D3Q19, float> &q) {
    using L = D3Q19;
    typedef typename PairOf<S>::type P2;
    constexpr uint32_t E = sizeof(P2);
    const __amdgpu_buffer_rsrc_t r = state_rsrc(static_cast<const S *>(in), uint32_t(L::Q) * pitch * E);
    P2 v[L::Q];
#pragma unroll
    for (int i = 0; i < L::Q; ++i)
        v[i] = load_pair<P2>(r, ar.vo(i) * E, uint32_t(su((uint32_t(i) * pitch + ar.so(i)) * E)));
#pragma unroll
    for (int i = 0; i < L::Q; ++i) decode_pair<L, S, float>(v[i], i, q);
}

// 36 x the recolouring term of a population that the sender of record entry e
// = {M, V_axis} and R_d sends along c_i.
__device__ __forceinline__ float rec_term(int i, const f4 e, float Rd) {
    using L = D3Q19;
    const int cv[3] = {L::cx[i], L::cy[i], L::cz[i]};
    const int n2 = csq<L>(i);
    if (n2 == 0) return 0.0f;
    if (n2 == 1) {
        const int ax = cv[0] ? 0 : (cv[1] ? 1 : 2);
        return cv[ax] > 0 ? e[1 + ax] : -e[1 + ax];
    }
    const int a0 = cv[0] ? 0 : 1, a1 = cv[2] ? 2 : 1;
    const float s0 = cv[a0] > 0 ? e[1 + a0] : -e[1 + a0];
    return Rd * (cv[a1] > 0 ? s0 + e[1 + a1] : s0 - e[1 + a1]);
}

// The 19 totals that a node pulls, each split with its sender's record (from
// the cache: a record serves 19 receivers).
template <typename S, bool UZ, class F>
__device__ __forceinline__ void pull_compact(const void *in, uint32_t pitch, const Around<UZ> &ar,
                                             CPops<D3Q19, float, F> &q) {
    using L = D3Q19;
    typedef CStore<S> St;
    const uint32_t base = uint32_t(L::Q) * pitch * St::E;
    const __amdgpu_buffer_rsrc_t r = state_rsrc(static_cast<const uint8_t *>(in), base + pitch * (St::kRecA + St::kRecB));
#pragma unroll
    for (int i = 0; i < L::Q; ++i) {
        const uint32_t c = ar.vo(i), z = ar.so(i);
        const typename St::Raw d = St::load(r, c * St::E, (uint32_t(i) * pitch + z) * St::E);
        const typename St::RawA ra = St::load_a(r, c * St::kRecA, base + z * St::kRecA);
        const typename St::RawB rb = St::load_b(r, c * St::kRecB, base + pitch * St::kRecA + z * St::kRecB);
        const f4 e = St::entry(ra, rb);
        q.df[i] = St::df(d, i);
        uint32_t word;
        q.mm[i] = Codec<float>::colw<float>(e[0], word);
        q.red.put(i, word);
        q.vd[i] = rec_term(i, e, St::ratio(rb));
    }
}

// Colour gradient from the neighbours' psi, in the sweeps' order (SOLID: the
// array holds kPsiOwn where the node's own psi stands in).
template <bool SOLID, bool UZ>
__device__ __forceinline__ void split_gradient(const float *psi, uint32_t pitch, const Around<UZ> &ar, float F[3]) {
    using L = D3Q19;
    typedef float T;
    const __amdgpu_buffer_rsrc_t r = state_rsrc(psi, pitch * 4u);
    auto at = [&](int i) {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
            r, int(ar.lane(L::cx[i], L::cy[i], L::cz[i]) * 4u), su(ar.base(L::cz[i]) * 4u), 0));
    };
    float pv[L::Q];
#pragma unroll
    for (int i = SOLID ? 0 : 1; i < L::Q; ++i) pv[i] = at(i);
    T fx = 0, fy = 0, fz = 0;
#pragma unroll
    for (int i = 1; i < L::Q; ++i) {
        const float v = SOLID ? (pv[i] == kPsiOwn ? pv[0] : pv[i]) : pv[i];
        const T wp = T(3.0 * wgt<L>(i)) * T(v);
        if (L::cx[i]) fx += L::cx[i] > 0 ? wp : -wp;
        if (L::cy[i]) fy += L::cy[i] > 0 ? wp : -wp;
        if (L::cz[i]) fz += L::cz[i] > 0 ? wp : -wp;
    }
    F[0] = fx;
    F[1] = fy;
    F[2] = fz;
}

template <class O>
__device__ __forceinline__ void split_collide(const Model<float> &mo, const float mv[kSplitMoments], const float F[3], O &o) {
    const float cj[3] = {mv[3], mv[4], mv[5]}, cS[6] = {mv[6], mv[7], mv[8], mv[9], mv[10], mv[11]};
    collide<D3Q19, float>(mo, mv[0], mv[1], mv[2], cj, cS, F, nullptr, o);
}

// Lattice and block of a batched launch's block b (a few scalar loads).
__device__ __forceinline__ int find_lat(const LatMap &m, uint32_t b, uint32_t &item) {
    int lo = 0, hi = m.n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (m.start[mid] <= b)
            lo = mid;
        else
            hi = mid - 1;
    }
    item = b - m.start[lo];
    return m.lat[lo];
}

}  // namespace

}  // namespace lbcg
