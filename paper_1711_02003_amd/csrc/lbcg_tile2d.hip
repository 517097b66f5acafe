// Fused single-pass D2Q9 step over tiles (arXiv:1711.02003, Sec. II, Eqs.
// (1)-(11)): pair state in FP64, FP32 or FP16 storage, with or without
// geometry, any collision form; compact state in FP32 (periodic); and the
// conversion of a compact state to a pair state.
//
// A block owns a tile of TX x TY nodes.  It pulls its nodes and a ring of one
// node around them (Eq. (1)), keeps the moments of its own nodes in registers
// and puts psi of all of them into LDS; after one barrier it forms the
// gradient, collides and stores.  In two dimensions the ring is small (a 64 x
// 16 tile: 16 % more pulls, from cache), so one pass with no loop over rows
// beats a strip that sweeps its rows one after another: every load of a tile
// is requested before the first is used, and a lattice gives thousands of
// independent blocks.  The strips this replaced (a wave per 64 columns and
// row chunk) took 24 us per step however small the lattice, 4-5 us a row.
//
// Compact state (LBCG_KERNEL_COMPACT): a node stores its 9 new total
// deviations and 4 colour scalars (minority share M with the majority flag in
// its lowest bit, V_axis (x, y) and R_d, with V_diag = R_d V_axis), from which
// the receiver of a population splits it into colours (Eq. (10): the minority
// colour part of f_i is M f_i + (c_i . V_c) / 36 with the sender's M and the V
// of the speed class of c_i): 2 x (9 x 4 + 16) = 104 bytes per node and step
// instead of 2 x 18 x 4 = 144.  Layout: 9 arrays of `pitch` floats (total
// deviation f_i - w_i of direction i at i * pitch + node), then `pitch`
// 16-byte records {M, V_axis x, y, R_d} (at float 9 * pitch + 4 n), read with
// 16-byte loads and written with two 8-byte stores per lane (a wider store may
// read its data registers after the compiler has already reused them).  The
// records of the tile and two nodes around it are staged in LDS first.  The
// first step after an initialisation or a restore reads the pair state
// instead (COUT).
//
// POPS (plain BGK, Eq. (5), at the node's rate or per colour): every
// population relaxes from its own pulled value, pulled again at the collision
// (from the cache).
//
// What bounds it: memory on large lattices, a block's chain of load, barrier
// and store on small ones.  us per step, strips (FP64: the two-pass generic
// kernel) -> tiles: 64 x 64 FP64 9.2 -> 5.0, FP32 24 -> 4.1; 512 x 512 FP32
// 33 -> 10, compact 27 -> 7.9; 3000 x 2100 FP32 244 -> 187 (4.9 TB/s),
// compact 219 -> 164 (4.0 TB/s); 4096 x 4096 FP32 521 -> 461, compact 429 ->
// 351 (5.0 TB/s), FP16 433 -> 318; junction 2048 x 512 FP32 92 -> 26, 8192 x
// 2048 480 -> 197.
#include "lbcg_buffer.h"
#include "lbcg_internal.h"

namespace lbcg {

namespace {

constexpr int kTileXCD = 8;
constexpr int kRec2 = 16;  // bytes of a compact record {M, V_axis x, y, R_d}

typedef float tf2 __attribute__((ext_vector_type(2)));
typedef float tf4 __attribute__((ext_vector_type(4)));
typedef unsigned int tu2 __attribute__((ext_vector_type(2)));

struct Tile2dArgs {
    const void *in;
    void *out;
    int nx, ny;
    uint32_t pitch;
    const uint8_t *mask;  // nullptr = every node fluid
    const DevInlet *inlets;
    const DevOutlet *outlets;
    const DevWall *walls;
    const uint32_t *links;
    const uint32_t *ctr_in;
    uint32_t *ctr_out;
    int ntx, nty;
};

__device__ __forceinline__ int tsu(uint32_t v) { return __builtin_amdgcn_readfirstlane(int(v)); }

// A pair of any width: 16-byte (FP64) pairs are loaded whole and stored in
// two halves (see put_pair).
template <typename P2>
__device__ __forceinline__ P2 tload(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    if constexpr (sizeof(P2) == 16)
        return __builtin_bit_cast(P2, __builtin_amdgcn_raw_buffer_load_b128(r, int(voff), tsu(soff), 0));
    else
        return load_pair<P2>(r, voff, uint32_t(tsu(soff)));
}
template <typename P2>
__device__ __forceinline__ void tstore(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, P2 v) {
    if constexpr (sizeof(P2) == 16) {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(tu2, double(v.x)), r, int(voff), tsu(soff), kNonTemporal);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(tu2, double(v.y)), r, int(voff + 8u), tsu(soff), kNonTemporal);
    } else {
        store_pair<P2>(r, voff, uint32_t(tsu(soff)), v);
    }
}

// Moments that a D2Q9 collision reads.
template <typename T>
struct Mom2 {
    T d, R, B, jx, jy, Sxx, Syy, Sxy;
};
template <typename T, class P>
__device__ __forceinline__ T moments2(const P &q, Mom2<T> &o) {
    Mom<T> m;
    moments<D2Q9, T>(q, m);
    o = {m.drho, m.r36R, m.r36B, m.j[0], m.j[1], m.S[0], m.S[1], m.S[3]};
    return psi_of<T>(m.drho, m.r36R, m.r36B);
}

template <typename T, int TX, int TY>
__device__ __forceinline__ void gradient2(const T *psi, int c, bool masked, T F[3]) {
    using L = D2Q9;
    constexpr int W = TX + 2;
    const T pc = psi[c];
    T fx = 0, fy = 0;
#pragma unroll
    for (int i = 1; i < L::Q; ++i) {
        T pv = psi[c + L::cy[i] * W + L::cx[i]];
        if (masked) pv = pv == T(1e30f) ? pc : pv;
        const T wp = T(3.0 * wgt<L>(i)) * pv;
        if (L::cx[i]) fx += L::cx[i] > 0 ? wp : -wp;
        if (L::cy[i]) fy += L::cy[i] > 0 ? wp : -wp;
    }
    F[0] = fx;
    F[1] = fy;
    F[2] = T(0);
}

// Tile geometry shared by the kernels: NT threads, K nodes per thread (rows
// ly + k NT / TX), the ring node r of the tile.
template <int TX, int TY, int NT>
struct Tile2d {
    static constexpr int W = TX + 2, H = TY + 2, PN = W * H;
    static constexpr int K = TX * TY / NT, RS = NT / TX;
    static constexpr int NR = (2 * (TX + 2) + 2 * TY + NT - 1) / NT;  // ring nodes per thread
    int x0, y0, tw, th, lx, ly;
    __device__ __forceinline__ Tile2d(const Tile2dArgs &a, int tile) {
        const int ty = tile / a.ntx, tx = tile - ty * a.ntx;
        x0 = tx * TX;
        y0 = ty * TY;
        tw = min(TX, a.nx - x0);
        th = min(TY, a.ny - y0);
        lx = int(threadIdx.x) % TX;
        ly = int(threadIdx.x) / TX;
    }
    __device__ __forceinline__ bool in(int k) const { return lx < tw && ly + k * RS < th; }
    __device__ __forceinline__ bool ring(int q, int &rx, int &ry) const {
        const int r = int(threadIdx.x) + q * NT;
        const int nr = 2 * (tw + 2) + 2 * th;
        rx = ry = 0;
        if (r >= nr) return false;
        if (r < tw + 2) {
            rx = r - 1;
            ry = -1;
        } else if (r < 2 * (tw + 2)) {
            rx = r - (tw + 2) - 1;
            ry = th;
        } else {
            const int s = r - 2 * (tw + 2);
            rx = s < th ? -1 : tw;
            ry = s < th ? s : s - th;
        }
        return true;
    }
};

// Node indices of the three columns x - 1, x, x + 1 and row starts y - 1, y,
// y + 1 of node (x, y), periodic.
struct Cols2d {
    uint32_t x[3], r[3];
    __device__ __forceinline__ Cols2d(int xx, int yy, int nx, int ny) {
        x[0] = uint32_t(xx == 0 ? nx - 1 : xx - 1);
        x[1] = uint32_t(xx);
        x[2] = uint32_t(xx == nx - 1 ? 0 : xx + 1);
        r[0] = uint32_t(yy == 0 ? ny - 1 : yy - 1) * uint32_t(nx);
        r[1] = uint32_t(yy) * uint32_t(nx);
        r[2] = uint32_t(yy == ny - 1 ? 0 : yy + 1) * uint32_t(nx);
    }
    // node x - cx, y - cy
    __device__ __forceinline__ uint32_t from(int cx, int cy) const { return x[1 - cx] + r[1 - cy]; }
};

template <typename S, typename T>
struct Raw2d {
    typename PairOf<S>::type v[D2Q9::Q];
    __device__ __forceinline__ void pull(__amdgpu_buffer_rsrc_t r, const Cols2d &c, uint32_t pitch) {
        typedef typename PairOf<S>::type P2;
        constexpr uint32_t E = sizeof(P2);
#pragma unroll
        for (int i = 0; i < D2Q9::Q; ++i)
            v[i] = tload<P2>(r, c.from(D2Q9::cx[i], D2Q9::cy[i]) * E, uint32_t(i) * pitch * E);
    }
    __device__ __forceinline__ void take(Pops<D2Q9, T> &q) const {
#pragma unroll
        for (int i = 0; i < D2Q9::Q; ++i) decode_pair<D2Q9, S, T>(v[i], i, q);
    }
};

// Tile of this block: periodic lattices deal contiguous bands of tiles to
// the 8 XCDs (neighbouring tiles share ring pulls in an L2), lattices with
// geometry consecutive tiles to consecutive XCDs (their fluid sits in a few
// bands).
template <bool MASKED>
__device__ __forceinline__ int tile_index(int total) {
    if (MASKED) return int(blockIdx.x);
    const int xcd = int(blockIdx.x) % kTileXCD, l = int(blockIdx.x) / kTileXCD;
    return xcd * (total / kTileXCD) + min(xcd, total % kTileXCD) + l;
}

// Compact output of node n.
__device__ __forceinline__ void store_compact2(__amdgpu_buffer_rsrc_t rout, uint32_t n, uint32_t pitch,
                                               const CompactOut<D2Q9, float> &o) {
    const uint32_t base = uint32_t(D2Q9::Q) * pitch * 4u;
#pragma unroll
    for (int i = 0; i < D2Q9::Q; ++i) store_pair<float>(rout, n * 4u, uint32_t(tsu(uint32_t(i) * pitch * 4u)), o.df[i]);
    const tf2 qa = {Codec<float>::enc_col<float>(o.M, o.redmaj), o.Va[0]};
    const tf2 qb = {o.Va[1], o.Rd};
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(tu2, qa), rout, int(n * kRec2), tsu(base), kNonTemporal);
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(tu2, qb), rout, int(n * kRec2), tsu(base + 8u), kNonTemporal);
}

// COUT: the new state is stored compact (periodic, FP32, regularized).
template <typename S, typename T, bool MASKED, bool POPS, bool COUT, int TX, int TY, int NT>
__global__ void __launch_bounds__(NT) k_tile2d(Tile2dArgs a, Model<T> mo) {
    using L = D2Q9;
    typedef typename PairOf<S>::type P2;
    typedef Tile2d<TX, TY, NT> G;
    constexpr uint32_t E = sizeof(P2);
    __shared__ T psi[G::PN];
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.ctr_out = *a.ctr_in + 1u;
    const G t(a, tile_index<MASKED>(a.ntx * a.nty));
    const uint32_t step = *a.ctr_in;  // seeds the stochastic rounding of 16-bit shares
    const __amdgpu_buffer_rsrc_t rin = state_rsrc(static_cast<const S *>(a.in), uint32_t(L::Q) * a.pitch * E);
    const __amdgpu_buffer_rsrc_t rout =
        state_rsrc(static_cast<S *>(a.out), COUT ? a.pitch * (uint32_t(L::Q) * 4u + kRec2) : uint32_t(L::Q) * a.pitch * E);
    // LDS psi of a non-fluid node: the inlet's or the wetting wall's phase
    // value, or a sentinel that the gradient replaces by the centre node's own
    auto solid_psi = [&](uint8_t c) -> T {
        if (is_inlet(c)) {
            const DevInlet in = a.inlets[c - kInlet0];
            return T((in.rhoR - in.rhoB) / (in.rhoR + in.rhoB));
        }
        if (c >= kWall0 && c < kOutlet0) return T(a.walls[c - kWall0].psi);
        return T(1e30f);
    };
    // link words of the thread's own nodes and of its ring nodes
    uint32_t lk[G::K], rl[G::NR];
    int rx[G::NR], ry[G::NR], gx[G::NR], gy[G::NR];
    bool has_ring[G::NR];
#pragma unroll
    for (int q = 0; q < G::NR; ++q) {
        has_ring[q] = t.ring(q, rx[q], ry[q]);
        gx[q] = wrap_m1(t.x0 + rx[q], a.nx);
        gy[q] = wrap_m1(t.y0 + ry[q], a.ny);
        rl[q] = kLinkFluid;
        if (MASKED && has_ring[q]) rl[q] = a.links[uint32_t(gx[q]) + uint32_t(a.nx) * uint32_t(gy[q])];
    }
#pragma unroll
    for (int k = 0; k < G::K; ++k) {
        lk[k] = MASKED ? 0u : kLinkFluid;
        if (MASKED && t.in(k))
            lk[k] = a.links[uint32_t(t.x0 + t.lx) + uint32_t(a.nx) * uint32_t(t.y0 + t.ly + k * G::RS)];
    }
    if (MASKED) {
        // a tile with no fluid node of its own has nothing to do
        bool any = false;
#pragma unroll
        for (int k = 0; k < G::K; ++k) any = any || (lk[k] & kLinkFluid) != 0u;
        if (!__syncthreads_or(any)) return;  // uniform over the block
    }
    auto cols = [&](int k) { return Cols2d(t.x0 + t.lx, t.y0 + t.ly + k * G::RS, a.nx, a.ny); };
    // every load of the tile is requested before the first is used
    Raw2d<S, T> own[G::K], side[G::NR];
#pragma unroll
    for (int k = 0; k < G::K; ++k)
        if (t.in(k) && (lk[k] & kLinkFluid)) own[k].pull(rin, cols(k), a.pitch);
#pragma unroll
    for (int q = 0; q < G::NR; ++q)
        if (has_ring[q] && (rl[q] & kLinkFluid)) side[q].pull(rin, Cols2d(gx[q], gy[q], a.nx, a.ny), a.pitch);
    Mom2<T> m[G::K];
#pragma unroll
    for (int k = 0; k < G::K; ++k) {
        m[k] = Mom2<T>{};
        if (!t.in(k)) continue;
        T v;
        if (lk[k] & kLinkFluid) {
            Pops<L, T> p;
            own[k].take(p);
            v = moments2<T>(p, m[k]);
        } else {
            v = solid_psi(link_code(lk[k]));
        }
        psi[(t.ly + k * G::RS + 1) * G::W + t.lx + 1] = v;
    }
#pragma unroll
    for (int q = 0; q < G::NR; ++q) {
        if (!has_ring[q]) continue;
        T v;
        if (rl[q] & kLinkFluid) {
            Pops<L, T> p;
            side[q].take(p);
            T dr, rR, rB;
            densities<L, T>(p, dr, rR, rB);
            v = psi_of<T>(dr, rR, rB);
        } else {
            v = solid_psi(link_code(rl[q]));
        }
        psi[(ry[q] + 1) * G::W + rx[q] + 1] = v;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < G::K; ++k) {
        if (!t.in(k) || !(lk[k] & kLinkFluid)) continue;
        T F[3];
        gradient2<T, TX, TY>(psi, (t.ly + k * G::RS + 1) * G::W + t.lx + 1, MASKED, F);
        const T j[3] = {m[k].jx, m[k].jy, T(0)};
        const T flux[6] = {m[k].Sxx, m[k].Syy, T(0), m[k].Sxy, T(0), T(0)};
        const Cols2d c = cols(k);
        if constexpr (COUT) {
            CompactOut<L, T> o;
            collide<L, T>(mo, m[k].d, m[k].R, m[k].B, j, flux, F, nullptr, o);
            store_compact2(rout, c.from(0, 0), a.pitch, o);
            continue;
        }
        PostOut<L, T> o;
        if constexpr (POPS) {
            // plain BGK relaxes every population from its own pulled value:
            // pulled again, from the cache
            Raw2d<S, T> raw;
            raw.pull(rin, c, a.pitch);
            Pops<L, T> p;
            raw.take(p);
            collide<L, T>(mo, m[k].d, m[k].R, m[k].B, j, flux, F, &p, o);
        } else {
            collide<L, T>(mo, m[k].d, m[k].R, m[k].B, j, flux, F, nullptr, o);
        }
        const uint32_t n = c.from(0, 0);
        // each pair is stored as it is encoded (an array filled first and
        // stored afterwards went through LDS: 13 us against 5 on 200 x 130)
        P2 enc[L::Q];
        Dither dz(step, n);
#pragma unroll
        for (int i = 0; i < L::Q; ++i) {
            const P2 v = encode_step<L, S, T>(o.df[i], o.mm[i], o.red(i), i, dz);
            tstore<P2>(rout, n * E, uint32_t(i) * a.pitch * E, v);
            if (MASKED) enc[i] = v;
        }
        // boundary values of the node's non-fluid links, stored in the
        // upstream nodes' slots (the addresses it pulls them from)
        if (MASKED && (lk[k] & kLinkBits)) {
            Geo g{};
            g.inlets = a.inlets;
            g.outlets = a.outlets;
            OwnMom<T> om{};
            if (lk[k] & kLinkOutlet) om = own_moments<L, S, T>(enc);
#pragma unroll
            for (int i = 1; i < L::Q; ++i) {
                if (!((lk[k] >> i) & 1u)) continue;
                const uint32_t up = c.from(L::cx[i], L::cy[i]);
                const uint8_t code = (lk[k] & kLinkMixed) ? a.mask[up] : link_code(lk[k]);
                tstore<P2>(rout, up * E, uint32_t(i) * a.pitch * E,
                           boundary_pair<L, S, T>(g, mo, i, code, enc[L::opp[i]], om));
            }
        }
    }
}

// ------------------------------------------------------------ compact state
// Split of the 9 pulled totals d with their senders' records (LDS entries
// {M, V_axis x, y, R_d}, W per row) at entry c of the node.
template <int W>
__device__ __forceinline__ void split_tile(const float d[D2Q9::Q], const tf4 *rec, int c, CPops<D2Q9, float> &p) {
    using L = D2Q9;
#pragma unroll
    for (int i = 0; i < L::Q; ++i) {
        const int cx = L::cx[i], cy = L::cy[i];
        const tf4 s = rec[c - cy * W - cx];
        p.df[i] = d[i];
        uint32_t word;
        p.mm[i] = Codec<float>::colw<float>(s[0], word);
        p.red.put(i, word);
        const int n2 = cx * cx + cy * cy;
        if (n2 == 0) {
            p.vd[i] = 0.0f;
        } else if (n2 == 1) {
            const float v = cx ? s[1] : s[2];
            p.vd[i] = (cx + cy) > 0 ? v : -v;
        } else {
            const float sx = cx > 0 ? s[1] : -s[1];
            p.vd[i] = s[3] * (cy > 0 ? sx + s[2] : sx - s[2]);
        }
    }
}

template <int TX, int TY, int NT>
__global__ void __launch_bounds__(NT) k_tile2d_compact(Tile2dArgs a, Model<float> mo) {
    using L = D2Q9;
    typedef float T;
    typedef Tile2d<TX, TY, NT> G;
    constexpr int RW = TX + 4, RN = RW * (TY + 4), RL = (RN + NT - 1) / NT;
    __shared__ tf4 rec[RN];
    __shared__ float psi[G::PN];
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.ctr_out = *a.ctr_in + 1u;
    const G t(a, tile_index<false>(a.ntx * a.nty));
    const uint32_t base = uint32_t(L::Q) * a.pitch * 4u, bytes = base + a.pitch * kRec2;
    const __amdgpu_buffer_rsrc_t rin = state_rsrc(static_cast<const float *>(a.in), bytes);
    const __amdgpu_buffer_rsrc_t rout = state_rsrc(static_cast<float *>(a.out), bytes);
    // records of the tile and two nodes around it
    tf4 rr[RL];
#pragma unroll
    for (int q = 0; q < RL; ++q) {
        const int r = int(threadIdx.x) + q * NT;
        const int sy = r / RW, sx = r - sy * RW;
        if (r < RN && sx < t.tw + 4 && sy < t.th + 4) {
            int xx = t.x0 + sx - 2, yy = t.y0 + sy - 2;
            // (at most two beyond a side; lattices narrower than two wrap again)
            xx = wrap_m1(wrap_m1(xx, a.nx), a.nx);
            yy = wrap_m1(wrap_m1(yy, a.ny), a.ny);
            const uint32_t n = uint32_t(xx) + uint32_t(a.nx) * uint32_t(yy);
            rr[q] = __builtin_bit_cast(tf4, __builtin_amdgcn_raw_buffer_load_b128(rin, int(n * kRec2), tsu(base), 0));
        }
    }
    auto pull = [&](const Cols2d &c, float d[L::Q]) {
#pragma unroll
        for (int i = 0; i < L::Q; ++i)
            d[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                 rin, int(c.from(L::cx[i], L::cy[i]) * 4u), tsu(uint32_t(i) * a.pitch * 4u), 0));
    };
    auto cols = [&](int k) { return Cols2d(t.x0 + t.lx, t.y0 + t.ly + k * G::RS, a.nx, a.ny); };
    float di[G::K][L::Q], dr[G::NR][L::Q];
#pragma unroll
    for (int k = 0; k < G::K; ++k)
        if (t.in(k)) pull(cols(k), di[k]);
#pragma unroll
    for (int q = 0; q < G::NR; ++q) {
        int rx, ry;
        if (t.ring(q, rx, ry)) pull(Cols2d(wrap_m1(t.x0 + rx, a.nx), wrap_m1(t.y0 + ry, a.ny), a.nx, a.ny), dr[q]);
    }
#pragma unroll
    for (int q = 0; q < RL; ++q) {
        const int r = int(threadIdx.x) + q * NT;
        if (r < RN) rec[r] = rr[q];
    }
    __syncthreads();
    Mom2<T> m[G::K];
#pragma unroll
    for (int k = 0; k < G::K; ++k) {
        m[k] = Mom2<T>{};
        if (!t.in(k)) continue;
        const int ry = t.ly + k * G::RS;
        CPops<L, T> p;
        split_tile<RW>(di[k], rec, (ry + 2) * RW + t.lx + 2, p);
        psi[(ry + 1) * G::W + t.lx + 1] = moments2<T>(p, m[k]);
    }
#pragma unroll
    for (int q = 0; q < G::NR; ++q) {
        int rx, ry;
        if (!t.ring(q, rx, ry)) continue;
        CPops<L, T> p;
        split_tile<RW>(dr[q], rec, (ry + 2) * RW + rx + 2, p);
        T d, rR, rB;
        densities<L, T>(p, d, rR, rB);
        psi[(ry + 1) * G::W + rx + 1] = psi_of<T>(d, rR, rB);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < G::K; ++k) {
        if (!t.in(k)) continue;
        T F[3];
        gradient2<T, TX, TY>(psi, (t.ly + k * G::RS + 1) * G::W + t.lx + 1, false, F);
        const T j[3] = {m[k].jx, m[k].jy, T(0)};
        const T flux[6] = {m[k].Sxx, m[k].Syy, T(0), m[k].Sxy, T(0), T(0)};
        CompactOut<L, T> o;
        collide<L, T>(mo, m[k].d, m[k].R, m[k].B, j, flux, F, nullptr, o);
        store_compact2(rout, cols(k).from(0, 0), a.pitch, o);
    }
}

// Pair state of nodes [0, N) from a compact D2Q9 state (see k_expand).
__global__ void k_expand2d(const float *__restrict__ cin, typename PairOf<float>::type *__restrict__ pout,
                           int64_t N, int64_t pitch) {
    using L = D2Q9;
    const int64_t n = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (n >= N) return;
    const float *ra = cin + int64_t(L::Q) * pitch + 4 * n;
    bool fl;
    const float M = Codec<float>::col<float>(ra[0], fl);
    const float Va[2] = {ra[1], ra[2]}, Rd = ra[3];
#pragma unroll
    for (int i = 0; i < L::Q; ++i) {
        const float d = cin[int64_t(i) * pitch + n];
        const int n2 = csq<L>(i);
        // the receiver's expression: c_i . V_axis, times R_d for a diagonal
        const float cva = float(L::cx[i]) * Va[0] + float(L::cy[i]) * Va[1];
        const float vd = n2 == 0 ? 0.0f : (n2 == 1 ? cva : Rd * cva);
        const float f = float(wgt<L>(i)) + d;
        const float mu36 = M * (float(w36<L>(i)) + 36.0f * d) + vd;
        const float q = f != 0.0f ? mu36 / (36.0f * f) : 0.0f;
        const bool keep = q <= 0.5f;
        pout[int64_t(i) * pitch + n] = encode_pair<L, float, float>(d, keep ? q : 1.0f - q, keep ? fl : !fl, i);
    }
}

Tile2dArgs tile_args(const Geo &g, const void *in, void *out, const uint32_t *ctr_in, uint32_t *ctr_out, int tx, int ty) {
    Tile2dArgs a;
    a.in = in;
    a.out = out;
    a.nx = g.nx;
    a.ny = g.ny;
    a.pitch = uint32_t(g.pitch);
    a.mask = g.mask;
    a.inlets = g.inlets;
    a.outlets = g.outlets;
    a.walls = g.walls;
    a.links = g.links;
    a.ctr_in = ctr_in;
    a.ctr_out = ctr_out;
    a.ntx = (g.nx + tx - 1) / tx;
    a.nty = (g.ny + ty - 1) / ty;
    return a;
}

// Shapes.  32 x 8 tiles, one node per thread, while there are too few large
// ones to fill the device; above, 64 x 16 tiles of two nodes per thread (half
// the ring): they cross at about a million nodes (1100 x 900: FP32 37.4
// against 36.8 us, compact 33 against 30; 512 x 512: 10.9 against 9.9,
// compact 7.9 against 8.3; 4096 x 4096: 507 against 461, 405 against 351).
// With geometry the large tiles are 32 x 16 (a channel's edges leave fewer
// idle lanes) from four million nodes on (2048 x 512 26.4 against 28.3 us,
// 8192 x 2048 203 against 197).  FP64 keeps the small ones.
constexpr int64_t kBigTiles = 800000, kBigTilesGeo = 4000000;

template <typename S, typename T, bool COUT, int TX, int TY, int NT>
hipError_t launch_tile(const Geo &g, const ModelD &md, const void *in, void *out, const uint32_t *ctr_in,
                       uint32_t *ctr_out, hipStream_t s) {
    const Tile2dArgs a = tile_args(g, in, out, ctr_in, ctr_out, TX, TY);
    if (int64_t(a.ntx) * a.nty > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid{unsigned(a.ntx * a.nty)}, block{unsigned(NT)};
    const Model<T> mo = to_model<T>(md);
    if constexpr (COUT) {
        hipLaunchKernelGGL((k_tile2d<S, T, false, false, true, TX, TY, NT>), grid, block, 0, s, a, mo);
    } else if (g.mask) {
        if (md.bgk)
            hipLaunchKernelGGL((k_tile2d<S, T, true, true, false, TX, TY, NT>), grid, block, 0, s, a, mo);
        else
            hipLaunchKernelGGL((k_tile2d<S, T, true, false, false, TX, TY, NT>), grid, block, 0, s, a, mo);
    } else {
        if (md.bgk)
            hipLaunchKernelGGL((k_tile2d<S, T, false, true, false, TX, TY, NT>), grid, block, 0, s, a, mo);
        else
            hipLaunchKernelGGL((k_tile2d<S, T, false, false, false, TX, TY, NT>), grid, block, 0, s, a, mo);
    }
    return hipGetLastError();
}

template <typename S, typename T>
hipError_t run_tile(const Geo &g, const ModelD &md, const void *in, void *out, const uint32_t *ctr_in,
                    uint32_t *ctr_out, hipStream_t s) {
    if constexpr (sizeof(T) == 4) {
        if (g.mask && g.N >= kBigTilesGeo) return launch_tile<S, T, false, 32, 16, 256>(g, md, in, out, ctr_in, ctr_out, s);
        if (!g.mask && g.N >= kBigTiles) return launch_tile<S, T, false, 64, 16, 512>(g, md, in, out, ctr_in, ctr_out, s);
    }
    return launch_tile<S, T, false, 32, 8, 256>(g, md, in, out, ctr_in, ctr_out, s);
}

template <int TX, int TY, int NT>
hipError_t launch_ctile(const Geo &g, const ModelD &md, const void *in, void *out, const uint32_t *ctr_in,
                        uint32_t *ctr_out, hipStream_t s) {
    const Tile2dArgs a = tile_args(g, in, out, ctr_in, ctr_out, TX, TY);
    if (int64_t(a.ntx) * a.nty > 0x7fffffff) return hipErrorInvalidValue;
    const Model<float> mo = to_model<float>(md);
    hipLaunchKernelGGL((k_tile2d_compact<TX, TY, NT>), dim3(unsigned(a.ntx * a.nty)), dim3(NT), 0, s, a, mo);
    return hipGetLastError();
}

}  // namespace

bool tile2d_supported(int prec, const Geo &g) {
    // 32-bit byte offsets must cover a state buffer
    const uint64_t elem = prec == 0 ? 8 : (prec == 1 ? 4 : 2);
    return g.nz == 1 && (g.mask == nullptr || g.links != nullptr) &&
           uint64_t(2 * D2Q9::Q) * uint64_t(g.pitch) * elem < (uint64_t(1) << 32);
}

hipError_t launch_step_tile2d(int prec, const Geo &g, const ModelD &md, const void *in, void *out,
                              const uint32_t *ctr_in, uint32_t *ctr_out, hipStream_t s) {
    if (!tile2d_supported(prec, g)) return hipErrorInvalidValue;
    if (prec == 0) return run_tile<double, double>(g, md, in, out, ctr_in, ctr_out, s);
    if (prec == 1) return run_tile<float, float>(g, md, in, out, ctr_in, ctr_out, s);
    return run_tile<_Float16, float>(g, md, in, out, ctr_in, ctr_out, s);
}

hipError_t launch_step_compact2d(const Geo &g, const ModelD &md, const void *in, bool pair_in, void *out,
                                 const uint32_t *ctr_in, uint32_t *ctr_out, hipStream_t s) {
    if (g.mask || md.bgk || !tile2d_supported(1, g)) return hipErrorInvalidValue;
    if (pair_in) return launch_tile<float, float, true, 32, 8, 256>(g, md, in, out, ctr_in, ctr_out, s);
    if (g.N >= kBigTiles) return launch_ctile<64, 16, 512>(g, md, in, out, ctr_in, ctr_out, s);
    return launch_ctile<32, 8, 256>(g, md, in, out, ctr_in, ctr_out, s);
}

hipError_t launch_expand2d(const Geo &g, const void *cin, void *pout, hipStream_t s) {
    if (g.N <= 0) return hipSuccess;
    const int64_t blocks = (g.N + 255) / 256;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_expand2d, dim3(unsigned(blocks)), dim3(256), 0, s, static_cast<const float *>(cin),
                       static_cast<typename PairOf<float>::type *>(pout), g.N, g.pitch);
    return hipGetLastError();
}

}  // namespace lbcg
