// Split D3Q19 step for lattices with geometry (arXiv:1711.02003, Sec. II,
// Eqs. (1)-(11)): the fused step in two kernels, one thread per node.
//
// The column sweep (lbcg_fused.hip) keeps a tile's phase field in LDS and
// recomputes a one-node ring of neighbour psi from their pulled populations;
// a z chunk re-pulls the two planes around it.  On a channel geometry the
// fluid fills few tiles, so filling the device takes short chunks, and the
// ring and the chunk halo then cost as much as the nodes themselves.  Here:
//   k_geo_moments: each fluid node pulls its 19 pairs (Eq. (1)), takes the
//     moments the collision needs (drho, 36 rho^R, 36 rho^B, j, trace-adjusted
//     flux S: 12 values) and psi (Eq. (4) input), and writes them;
//   k_geo_collide: each fluid node forms the colour gradient from its
//     neighbours' psi, collides (Eqs. (9)-(11)) and stores its 19 new pairs
//     and, for links from non-fluid nodes, their boundary values.
// Every value is computed by the expressions and in the order of the column
// sweep, so the results are bitwise those of the sweep.  Traffic per fluid
// node: pairs read and written once (2 x 38 x E bytes), plus 12 moments and
// psi written and read once (2 x 52 bytes) and the neighbours' psi from cache.
// The same kernels also run on the compact state (below): 2 x 96 (FP32) or 2 x
// 50 (FP16) bytes of state per fluid node instead of 2 x 152 or 2 x 76.
//
// Work: thread k takes entry k of the list of fluid nodes {node, link word},
// built once per lattice.  Blocks of 64 x 4 nodes (with a list
// of those that hold fluid) left a third of the lanes idle on step-emulsifier
// channels and read the link words of solid nodes: 412 us a level for eight
// of them (FP32) against 370.  With the nodes that have inlet or outlet links
// first in the list, in waves of their own, the collision of the 512 x 128 x
// 64 junction took 54 us instead of 64, but such a wave on a face across x
// touches 64 lines per access: its moments took 47 instead of 43, and a 256 x
// 64 x 32 junction 52 us a step instead of 33 (16-bit, compact).
//
// psi: non-fluid nodes hold what they show the gradient, written once when
// the lattice is made (the inlet's or wetting wall's phase value, or kPsiOwn
// where the fluid node's own psi stands in), so the gradient is 19 plain
// loads; looking each non-fluid neighbour up in the mask took the collision
// kernel 110 registers and 1560 vector instructions.
//
// The moments lie in the fluid node's own slots of the buffer that the step
// writes (see lbcg_split.hip): the lines come from the caches when the new
// state is stored, and an area of their own is neither written nor read.  On
// the 512 x 128 x 64 junction (FP32) 50 + 58 us against 62 + 70; on the
// compact state, collision kernel only, 37 us (FP16: 30) against 40 (34).
//
// Inlet and outlet values.  On pairs the collision kernel forms them from each
// new pair as it is stored, at 112 registers: 62 us on that junction against
// 57 without them and 6 and a launch in a kernel of their own, and on eight
// step-emulsifier channels 190 against 174 + 45.  On the compact state, where
// the values go to another buffer, a kernel of one thread per link follows:
// 37 + 6 us against 48 (FP16: 30 + 6 against 54).
#include "lbcg_split.h"

namespace lbcg {

namespace {

constexpr int kGeoBlock = 256;
constexpr int kIoBlock = 64;
constexpr int kChunk = 1024;  // nodes per count of the list builder

// Scratch: psi of every node, the list of fluid nodes {node, link word}, that
// of the ones with inlet or outlet links, the counts of the list builder (two
// per chunk of nodes) and the totals.  (The lists have the room that the
// moments' 48 bytes per node once took.)
struct ScratchMap {
    float *psi;
    uint32_t *list, *io;
    uint32_t *counts, *totals;
};
inline size_t align256(size_t v) { return (v + 255) / 256 * 256; }
inline ScratchMap scratch_map(void *scratch, int64_t pitch) {
    char *p = static_cast<char *>(scratch);
    const size_t chunks = size_t((pitch + kChunk - 1) / kChunk);
    ScratchMap m;
    m.psi = reinterpret_cast<float *>(p);
    p += align256(sizeof(float) * size_t(pitch));
    m.list = reinterpret_cast<uint32_t *>(p);
    p += align256(2 * sizeof(uint32_t) * size_t(pitch));
    m.io = reinterpret_cast<uint32_t *>(p);
    p += align256(2 * sizeof(uint32_t) * size_t(pitch));
    m.counts = reinterpret_cast<uint32_t *>(p);
    p += align256(2 * sizeof(uint32_t) * chunks);
    m.totals = reinterpret_cast<uint32_t *>(p);
    return m;
}

// A fluid node with a link from a non-fluid node that is not a wall (mixed
// codes count: each link is checked where it is used).
__device__ __forceinline__ bool has_io_link(uint32_t lk) {
    return (lk & kLinkBits) && ((lk & kLinkMixed) || !is_wall(link_code(lk)));
}

// Order of the lists: number t of a lattice's N nodes.  Rows one after another,
// except where every row starts on a 64-node boundary: there by 64 x 8 nodes, so
// that a block reads its neighbours' lines (and on the compact state the records,
// which serve 19 receivers) for eight rows at once.  Junction 512 x 128 x 64 FP32
// compact 112 -> 107 us a step (110 with blocks of 64 x 4 nodes before there was a
// list), 256 x 64 x 32 FP16 compact 28 -> 26; on rows that start anywhere a wave
// then reaches over two rows that share no line (channel of 386 x 130 x 66 nodes
// 125 -> 153 us, duct of 300 x 40 x 30 40 -> 42).
constexpr uint32_t kListX = 64, kListY = 8;
__device__ __forceinline__ uint32_t listed_node(uint32_t t, uint32_t nx, uint32_t ny) {
    if (nx % kListX != 0) return t;
    const uint32_t plane = nx * ny, z = t / plane, p = t - z * plane;
    const uint32_t band = p / (kListY * nx), h = min(kListY, ny - kListY * band);  // rows of the band
    const uint32_t q = p - band * kListY * nx, b = q / (kListX * h), r = q - b * kListX * h;
    return z * plane + (kListY * band + r / kListX) * nx + kListX * b + r % kListX;
}

// List builder.  Block b goes through numbers [b kChunk, (b + 1) kChunk):
// without lists it counts its fluid nodes and those with inlet or outlet
// links; with them it writes their entries from the offsets that k_geo_scan
// put in place of the counts.
__global__ void __launch_bounds__(kGeoBlock) k_geo_list(const uint32_t *__restrict__ links, uint32_t N, uint32_t nx,
                                                       uint32_t ny, uint32_t *__restrict__ counts,
                                                       uint32_t *__restrict__ list, uint32_t *__restrict__ io) {
    __shared__ uint32_t wc[2][kGeoBlock / 64];
    const int w = int(threadIdx.x / 64);
    uint32_t at[2] = {0, 0};
    if (list)
        for (int c = 0; c < 2; ++c) at[c] = counts[2 * blockIdx.x + c];
    for (uint32_t k = 0; k < kChunk; k += kGeoBlock) {
        const uint32_t t = blockIdx.x * kChunk + k + threadIdx.x;
        const uint32_t n = t < N ? listed_node(t, nx, ny) : 0u;
        const uint32_t lk = t < N ? links[n] : 0u;
        const bool mine[2] = {(lk & kLinkFluid) != 0u, (lk & kLinkFluid) && has_io_link(lk)};
        uint32_t e[2];
        __syncthreads();  // the counts of the pass before have been read
        for (int c = 0; c < 2; ++c) {
            const uint64_t bal = __builtin_amdgcn_ballot_w64(mine[c]);
            e[c] = at[c] + __builtin_amdgcn_mbcnt_hi(uint32_t(bal >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(bal), 0u));
            if (threadIdx.x % 64 == 0) wc[c][w] = uint32_t(__builtin_popcountll(bal));
        }
        __syncthreads();
        for (int c = 0; c < 2; ++c) {
            for (int v = 0; v < kGeoBlock / 64; ++v) {
                e[c] += v < w ? wc[c][v] : 0u;
                at[c] += wc[c][v];
            }
            uint32_t *to = c == 0 ? list : io;
            if (list && mine[c]) {
                to[2 * size_t(e[c])] = n;
                to[2 * size_t(e[c]) + 1] = lk;
            }
        }
    }
    if (!list && threadIdx.x == 0)
        for (int c = 0; c < 2; ++c) counts[2 * blockIdx.x + c] = at[c];
}

// Counts to offsets in the two lists, by one block: thread t takes a
// contiguous range of chunks.
constexpr int kScanThreads = 1024;
__global__ void __launch_bounds__(kScanThreads) k_geo_scan(uint32_t *__restrict__ counts, uint32_t chunks,
                                                          uint32_t *__restrict__ totals) {
    __shared__ uint32_t s[2][kScanThreads];
    const uint32_t per = (chunks + kScanThreads - 1) / kScanThreads;
    const uint32_t b0 = min(chunks, threadIdx.x * per), b1 = min(chunks, b0 + per);
    for (int c = 0; c < 2; ++c) {
        uint32_t sum = 0;
        for (uint32_t b = b0; b < b1; ++b) sum += counts[2 * b + c];
        s[c][threadIdx.x] = sum;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        uint32_t t = 0;
        for (int k = 0; k < kScanThreads; ++k) {
            const uint32_t v = s[threadIdx.x][k];
            s[threadIdx.x][k] = t;
            t += v;
        }
        totals[threadIdx.x] = t;
    }
    __syncthreads();
    for (int c = 0; c < 2; ++c) {
        uint32_t at = s[c][threadIdx.x];
        for (uint32_t b = b0; b < b1; ++b) {
            const uint32_t v = counts[2 * b + c];
            counts[2 * b + c] = at;
            at += v;
        }
    }
}

// What the non-fluid nodes show the gradient of a fluid neighbour.
__global__ void __launch_bounds__(kGeoBlock) k_geo_solid_psi(Geo g, float *__restrict__ psi) {
    const int64_t n = int64_t(blockIdx.x) * kGeoBlock + threadIdx.x;
    if (n >= g.N) return;
    const uint8_t c = g.mask[n];
    if (c == kFluid) return;
    float v = kPsiOwn;
    if (is_inlet(c)) {
        const DevInlet in = g.inlets[c - kInlet0];
        v = float((in.rhoR - in.rhoB) / (in.rhoR + in.rhoB));
    } else if (c >= kWall0 && c < kOutlet0) {
        v = float(g.walls[c - kWall0].psi);
    }
    psi[n] = v;
}

// The fluid node of this thread in block `item` (false past the end), its
// link word and its surroundings.
typedef Around<false> Near;
struct Here {
    uint32_t n, lk, x, y, z;
};
__device__ __forceinline__ Here node_at(const SplitDesc &a, uint32_t n, uint32_t lk) {
    Here h;
    h.n = n;
    h.lk = lk;
    const uint32_t row = div_by(n, a.div0);
    h.z = div_by(row, a.div1);
    h.y = row - h.z * a.div1.d;
    h.x = n - row * a.div0.d;
    return h;
}
__device__ __forceinline__ bool here(const SplitDesc &a, uint32_t item, Here &h) {
    const uint32_t k = item * kGeoBlock + threadIdx.x;
    if (k >= a.count) return false;
    const uint2 e = reinterpret_cast<const uint2 *>(a.list)[k];
    h = node_at(a, e.x, e.y);
    return true;
}
__device__ __forceinline__ Near near(const SplitDesc &a, const Here &h) {
    return Near(h.x, h.y, h.z, uint32_t(a.nx), uint32_t(a.ny), uint32_t(a.nz));
}

// The moments' slots: those of FP32 pairs are 8 bytes wide, those of FP16
// pairs and of the FP32 compact state's totals 4, of the FP16 totals 2.
template <typename S, bool COMPACT>
using GeoMom = std::conditional_t<COMPACT && sizeof(S) == 2, MomHalves, MomStore<sizeof(S) == 4 && !COMPACT>>;

template <typename S, bool COMPACT>
__device__ __forceinline__ void geo_put(const SplitDesc &a, const Here &h, const Mom<float> &m) {
    put_psi(a.psi, a.pitch, h.n, 0u, float(psi_of<float>(m.drho, m.r36R, m.r36B)));
    GeoMom<S, COMPACT>::put(a.mom, a.pitch, h.n, 0u, m);
}

template <typename S, bool COMPACT>
__device__ __forceinline__ void geo_moments(const SplitDesc &a, uint32_t item) {
    Here h;
    if (!here(a, item, h)) return;
    Pops<D3Q19, float> q;
    pull_pairs<S>(a.in, a.pitch, near(a, h), q);
    Mom<float> m;
    moments<D3Q19, float>(q, m);
    geo_put<S, COMPACT>(a, h, m);
}

// The wall links among a fluid node's non-fluid links.
__device__ __forceinline__ uint32_t wall_links(const SplitDesc &a, uint32_t lk, const Near &ar) {
    using L = D3Q19;
    if (!(lk & kLinkMixed)) return is_wall(link_code(lk)) ? lk & kLinkBits : 0u;
    uint32_t wall = 0;
#pragma unroll
    for (int i = 1; i < L::Q; ++i)
        if ((lk >> i) & 1u) wall |= is_wall(a.mask[ar.vo(i)]) ? (1u << i) : 0u;
    return wall;
}

// Inlet and outlet links of a wave's nodes: the value that a node will pull
// through such a link at the next step, from its new pair of the opposite
// direction as stored and, for outlets, the moments of its stored pairs.
// Waves without such nodes skip it, the others run the directions that their
// nodes have (a face: five).
template <typename S>
struct IoLinks {
    typedef typename PairOf<S>::type P2;
    uint32_t io, any;  // the lane's links, the wave's
    IoVals<float> iv;
    OwnMom<float> om;
    __device__ __forceinline__ IoLinks(const SplitDesc &a, const Here &h, uint32_t wall) : io(0), any(0), iv{}, om{} {
        io = h.lk & kLinkBits & ~wall;
        if (__builtin_amdgcn_ballot_w64(io != 0u) == 0) return;
#pragma unroll
        for (int i = 1; i < D3Q19::Q; ++i)
            if (__builtin_amdgcn_ballot_w64((io >> i) & 1u) != 0) any |= 1u << i;
        if (io && !(h.lk & kLinkMixed)) iv = vals(a, link_code(h.lk));
    }
    __device__ __forceinline__ bool outlets(const Here &h) const {
        return any && __builtin_amdgcn_ballot_w64((h.lk & kLinkOutlet) != 0u) != 0;
    }
    __device__ __forceinline__ static IoVals<float> vals(const SplitDesc &a, uint8_t c) {
        Geo g{};
        g.inlets = a.inlets;
        g.outlets = a.outlets;
        return io_vals<float>(g, c);
    }
    // link i, from the node's new pair `own` of direction opp(i)
    __device__ __forceinline__ void put(const SplitDesc &a, const Here &h, const Near &ar, __amdgpu_buffer_rsrc_t rg,
                                        int i, P2 own) {
        constexpr uint32_t E = sizeof(P2);
        if (!((any >> i) & 1u)) return;  // uniform over the wave
        if (!((io >> i) & 1u)) return;
        uint8_t c = link_code(h.lk);
        if (h.lk & kLinkMixed) {
            c = a.mask[ar.vo(i)];
            iv = vals(a, c);
        }
        store_pair<P2>(rg, ar.vo(i) * E, uint32_t(su(uint32_t(i) * a.pitch * E)),
                       boundary_pair_v<D3Q19, S, float>(a.mo, i, c, iv, own, om));
    }
};

template <typename S>
__device__ __forceinline__ void geo_collide(const SplitDesc &a, uint32_t item) {
    using L = D3Q19;
    typedef typename PairOf<S>::type P2;
    constexpr uint32_t E = sizeof(P2);
    if (item == 0 && threadIdx.x == 0) *a.ctr_out = *a.ctr_in + 1u;
    Here h;
    if (!here(a, item, h)) return;
    uint32_t step = 0;  // seeds the stochastic rounding of 16-bit shares
    if constexpr (sizeof(S) == 2) step = *a.ctr_in;
    const Near ar = near(a, h);
    float F[3], mv[kSplitMoments];
    GeoMom<S, false>::get(a.mom, a.pitch, h.n, 0u, mv);
    split_gradient<true>(a.psi, a.pitch, ar, F);
    PostOut<L, float> o;
    split_collide(a.mo, mv, F, o);
    const __amdgpu_buffer_rsrc_t rout = state_rsrc(static_cast<S *>(a.out), uint32_t(L::Q) * a.pitch * E);
    // Half-way bounce-back: where link i comes from a wall, the new pair of
    // the opposite direction is also stored in the wall node's slot.  Waves
    // with no wall link skip it.
    const uint32_t wall = (h.lk & kLinkBits) ? wall_links(a, h.lk, ar) : 0u;
    const bool walls = __builtin_amdgcn_ballot_w64(wall != 0u) != 0;
    IoLinks<S> io(a, h, wall);
    if (io.outlets(h)) {
        // the moments of the pairs before they are stored below (16-bit
        // storage: with the same random bits)
        Dither dz(step, h.n);
        OwnSum<L, S, float> sum;
#pragma unroll
        for (int j = 0; j < L::Q; ++j)
            sum.add(j, encode_step<L, S, float>(o.df[j], o.mm[j], o.red(j), j, dz));
        io.om = sum.moments();
    }
    Dither dz(step, h.n);
#pragma unroll
    for (int j = 0; j < L::Q; ++j) {
        const P2 v = encode_step<L, S, float>(o.df[j], o.mm[j], o.red(j), j, dz);
        store_pair<P2>(rout, h.n * E, uint32_t(su(uint32_t(j) * a.pitch * E)), v);
        if (j == 0) continue;
        const int i = L::opp[j];
        if (walls && ((wall >> i) & 1u))
            store_pair<P2>(rout, ar.vo(i) * E, uint32_t(su(uint32_t(i) * a.pitch * E)), v);
        io.put(a, h, ar, rout, i, v);
    }
}

template <typename S, bool COMPACT>
__global__ void __launch_bounds__(kGeoBlock) k_geo_moments(SplitDesc a) {
    geo_moments<S, COMPACT>(a, blockIdx.x);
}
template <typename S>
__global__ void __launch_bounds__(kGeoBlock) k_geo_collide(SplitDesc a) {
    geo_collide<S>(a, blockIdx.x);
}
// Many lattices in one launch.
template <typename S>
__global__ void __launch_bounds__(kGeoBlock) k_geo_moments_batch(const SplitDesc *__restrict__ desc,
                                                                const LatMap *__restrict__ map) {
    uint32_t item;
    const SplitDesc a = desc[find_lat(*map, blockIdx.x, item)];
    geo_moments<S, false>(a, item);
}
template <typename S>
__global__ void __launch_bounds__(kGeoBlock) k_geo_collide_batch(const SplitDesc *__restrict__ desc,
                                                                const LatMap *__restrict__ map) {
    uint32_t item;
    const SplitDesc a = desc[find_lat(*map, blockIdx.x, item)];
    geo_collide<S>(a, item);
}

// ------------------------------------------------------------ compact state
// The same split step on the compact state, FP32 or FP16 storage (the
// layout and rounding of the periodic compact sweep, CStore: 19 arrays of
// totals, then records {M with the majority flag, V_axis} and R_d; 96 or 50
// B per node).  A receiver splits each pulled total with its sender's record
// (the recolouring of Eq. (10) done at the receiver).  A link from a wall
// brings back the node's own new total of the opposite direction, split with
// its own record for that direction, so walls need no stored values.  A link
// from an inlet or an outlet reads the pair (total deviation, minority share)
// that the boundary kernel stored in that node's slot of a pair buffer (the
// values of the pair-state step, formed from the node's own new
// populations).
struct CGeoArgs {
    SplitDesc s;      // s.in, s.out: compact state read and written
    const void *gin;  // pair buffer read (inlet and outlet values)
    void *gout;       // pair buffer written
};
template <typename S>
constexpr uint32_t c_bytes() {  // bytes per node of the compact state
    return uint32_t(D3Q19::Q) * CStore<S>::E + CStore<S>::kRecA + CStore<S>::kRecB;
}

// Record of node u: minority share M and majority flag, V_axis, R_d.
struct CRec {
    float M, Va[3], Rd;
    bool fl;
};
template <typename S>
__device__ __forceinline__ CRec c_record_of(typename CStore<S>::RawA ra, typename CStore<S>::RawB rb) {
    const f4 e = CStore<S>::entry(ra, rb);
    CRec c;
    c.M = Codec<float>::col<float>(e[0], c.fl);
    c.Va[0] = e[1];
    c.Va[1] = e[2];
    c.Va[2] = e[3];
    c.Rd = CStore<S>::ratio(rb);
    return c;
}
template <typename S>
__device__ __forceinline__ CRec c_record(__amdgpu_buffer_rsrc_t rc, uint32_t u, uint32_t pitch) {
    typedef CStore<S> St;
    const uint32_t base = uint32_t(D3Q19::Q) * pitch * St::E;
    const typename St::RawB rb = St::load_b(rc, u * St::kRecB, base + pitch * St::kRecA);
    return c_record_of<S>(St::load_a(rc, u * St::kRecA, base), rb);
}
// Total deviation f_i - w_i stored at element `at` of the totals (i * pitch
// + node; a direction of the speed class of i).
template <typename S>
__device__ __forceinline__ float c_total(__amdgpu_buffer_rsrc_t rc, uint32_t at, int i) {
    return CStore<S>::df(CStore<S>::load(rc, at * CStore<S>::E, 0u), i);
}
// 36 x the recolouring term of a population the record's node sends along
// c_i: c_i . V_axis, times R_d on a diagonal (the periodic sweep's split)
__device__ __forceinline__ float c_vd(int i, const CRec &r) {
    using L = D3Q19;
    const float cva = float(L::cx[i]) * r.Va[0] + float(L::cy[i]) * r.Va[1] + float(L::cz[i]) * r.Va[2];
    const int n2 = csq<L>(i);
    return n2 == 0 ? 0.0f : (n2 == 1 ? cva : r.Rd * cva);
}
// Pair (total deviation, minority share with flag) of the population the
// record's node sends along c_i with total deviation d: the conversion the
// periodic compact state's export uses.
template <typename S>
__device__ __forceinline__ typename PairOf<S>::type c_pair(float d, int i, const CRec &r) {
    using L = D3Q19;
    const float f = float(wgt<L>(i)) + d;
    const float mu36 = r.M * (float(w36<L>(i)) + 36.0f * d) + c_vd(i, r);
    const float q = f != 0.0f ? mu36 / (36.0f * f) : 0.0f;
    const bool keep = q <= 0.5f;
    return encode_pair<L, S, float>(d, keep ? q : 1.0f - q, keep ? r.fl : !r.fl, i);
}

// The node's own moments (density, red density, velocity) from its new totals
// and record: own_moments of its populations, each split as a receiver splits
// it (no division per population).
template <class Tot>
__device__ __forceinline__ OwnMom<float> c_own_moments(const CRec &r, Tot total) {
    using L = D3Q19;
    float drho = 0, Ra = 0, jx = 0, jy = 0, jz = 0;
    int K = 0;
#pragma unroll
    for (int k = 0; k < L::Q; ++k) {
        const float d = total(k);
        const float mu = r.M * (float(w36<L>(k)) + 36.0f * d) + c_vd(k, r);
        const float t = 36.0f * d - mu;
        drho += d;
        Ra += r.fl ? t : mu;
        K += r.fl ? w36<L>(k) : 0;
        jx += float(L::cx[k]) * d;
        jy += float(L::cy[k]) * d;
        jz += float(L::cz[k]) * d;
    }
    OwnMom<float> om;
    om.rho = 1.0f + drho;
    om.rR = (float(K) + Ra) / 36.0f;
    om.u[0] = jx / om.rho;
    om.u[1] = jy / om.rho;
    om.u[2] = jz / om.rho;
    return om;
}

// Each link is one load of a total and one of a record (from the cache: a
// record serves up to 19 receivers).  Staging the block's records with a
// one-node halo in LDS first measured slower (0.129 against 0.119 ms on the
// 512 x 128 x 64 junction).  A wave whose nodes have no non-fluid link takes
// the periodic step's loads.
template <typename S>
__global__ void __launch_bounds__(kGeoBlock) k_cgeo_moments(CGeoArgs ca) {
    using L = D3Q19;
    typedef float T;
    typedef typename PairOf<S>::type P2;
    constexpr uint32_t E = sizeof(P2);
    const SplitDesc &a = ca.s;
    Here h;
    if (!here(a, banded(gridDim.x), h)) return;
    const uint32_t pitch = a.pitch;
    const Near ar = near(a, h);
    // (flags as bits: with masks fewer loads were in flight, 92 us against 68 on
    // the 512 x 128 x 64 junction)
    CPops<L, T, FlagBits<L::Q>> q;
    if (__builtin_amdgcn_ballot_w64((h.lk & kLinkBits) != 0u) == 0) {
        pull_compact<S>(a.in, pitch, ar, q);
    } else {
        const __amdgpu_buffer_rsrc_t rc = state_rsrc(static_cast<const uint8_t *>(a.in), c_bytes<S>() * pitch);
        // links from walls and from inlets or outlets
        const uint32_t wall = (h.lk & kLinkBits) ? wall_links(a, h.lk, ar) : 0u;
        const uint32_t io = h.lk & kLinkBits & ~wall;
        // Every link as a plain load with a per-lane address: from a fluid
        // node its total of direction i and its record; from a wall the node's
        // own total of the opposite direction and its own record, the
        // recolouring term with the opposite sign.  Links from inlets and
        // outlets are replaced below.
#pragma unroll
        for (int i = 0; i < L::Q; ++i) {
            const bool wl = (wall >> i) & 1u;
            const uint32_t u = ar.vo(i);
            const uint32_t src = wl ? uint32_t(L::opp[i]) * pitch + h.n : uint32_t(i) * pitch + u;
            const float d = c_total<S>(rc, src, i);
            const CRec r = c_record<S>(rc, wl ? h.n : u, pitch);
            const float vd = c_vd(i, r);
            q.df[i] = d;
            q.mm[i] = r.M;
            q.vd[i] = wl ? -vd : vd;
            q.red.put(i, r.fl ? 1u : 0u);
        }
        if (io) {
            const __amdgpu_buffer_rsrc_t rg = state_rsrc(static_cast<const S *>(ca.gin), uint32_t(L::Q) * pitch * E);
#pragma unroll
            for (int i = 1; i < L::Q; ++i) {
                if (!((io >> i) & 1u)) continue;
                const P2 v = load_pair<P2>(rg, ar.vo(i) * E, uint32_t(su(uint32_t(i) * pitch * E)));
                q.df[i] = Codec<S>::template df<L, T>(v.x, i);
                uint32_t word;
                q.mm[i] = Codec<S>::template colw<T>(v.y, word);
                q.red.put(i, word);
                q.vd[i] = 0.0f;
            }
        }
    }
    Mom<T> mm;
    moments<L, T>(q, mm);
    geo_put<S, true>(a, h, mm);
}

template <typename S>
__global__ void __launch_bounds__(kGeoBlock) k_cgeo_collide(CGeoArgs ca) {
    using L = D3Q19;
    typedef CStore<S> St;
    const SplitDesc &a = ca.s;
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.ctr_out = *a.ctr_in + 1u;
    Here h;
    if (!here(a, banded(gridDim.x), h)) return;
    uint32_t step = 0;  // seeds the stochastic rounding of FP16 storage
    if constexpr (sizeof(S) == 2) step = *a.ctr_in;
    const Near ar = near(a, h);
    float F[3], mv[kSplitMoments];
    GeoMom<S, true>::get(a.mom, a.pitch, h.n, 0u, mv);
    split_gradient<true>(a.psi, a.pitch, ar, F);
    CompactOut<L, float> o;
    split_collide(a.mo, mv, F, o);
    const __amdgpu_buffer_rsrc_t rout = state_rsrc(static_cast<uint8_t *>(a.out), c_bytes<S>() * a.pitch);
    St::store(rout, h.n * St::E, 0u, a.pitch, o, step);
}

// Inlet and outlet values from the stored totals and record of the node that
// pulls them: thread k takes one link direction I of entry k of the list of
// nodes with such links.
template <typename S, int I>
__device__ __forceinline__ void io_link(const CGeoArgs &ca, uint32_t dir, uint32_t n, uint32_t lk) {
    using L = D3Q19;
    if constexpr (I < L::Q) {
        if (dir != I) return io_link<S, I + 1>(ca, dir, n, lk);  // uniform over the block
        typedef typename PairOf<S>::type P2;
        constexpr uint32_t E = sizeof(P2);
        if (!((lk >> I) & 1u)) return;
        const SplitDesc &a = ca.s;
        const uint32_t u = near(a, node_at(a, n, lk)).vo(I);
        const uint8_t c = (lk & kLinkMixed) ? a.mask[u] : link_code(lk);
        if (is_wall(c)) return;
        const uint32_t pitch = a.pitch;
        const __amdgpu_buffer_rsrc_t rc = state_rsrc(static_cast<const uint8_t *>(a.out), c_bytes<S>() * pitch);
        const CRec own = c_record<S>(rc, n, pitch);
        OwnMom<float> om{};
        if (c >= kOutlet0) om = c_own_moments(own, [&](int k) { return c_total<S>(rc, uint32_t(k) * pitch + n, k); });
        const P2 v = c_pair<S>(c_total<S>(rc, uint32_t(L::opp[I]) * pitch + n, L::opp[I]), L::opp[I], own);
        Geo g{};
        g.inlets = a.inlets;
        g.outlets = a.outlets;
        store_pair<P2>(state_rsrc(static_cast<S *>(ca.gout), uint32_t(L::Q) * pitch * E), u * E,
                       uint32_t(su(uint32_t(I) * pitch * E)),
                       boundary_pair_v<L, S, float>(a.mo, I, c, io_vals<float>(g, c), v, om));
    }
}
template <typename S>
__global__ void __launch_bounds__(kIoBlock) k_cgeo_boundary(CGeoArgs ca) {
    const uint32_t k = blockIdx.x * kIoBlock + threadIdx.x;
    if (k >= ca.s.count) return;
    const uint2 e = reinterpret_cast<const uint2 *>(ca.s.list)[k];
    io_link<S, 1>(ca, blockIdx.y + 1u, e.x, e.y);
}

// The compact state of the fluid nodes as pairs, for reads of the state:
// each fluid node's 19 pairs in its own slots and, for links from walls, its
// bounce-back values in the wall nodes' slots; the inlet and outlet values
// are already in the pair buffer.
template <typename S>
__global__ void __launch_bounds__(kGeoBlock) k_cgeo_expand(CGeoArgs ca) {
    using L = D3Q19;
    typedef typename PairOf<S>::type P2;
    constexpr uint32_t E = sizeof(P2);
    const SplitDesc &a = ca.s;
    Here h;
    if (!here(a, banded(gridDim.x), h)) return;
    const uint32_t pitch = a.pitch;
    const Near ar = near(a, h);
    const __amdgpu_buffer_rsrc_t rc = state_rsrc(static_cast<const uint8_t *>(a.in), c_bytes<S>() * pitch);
    const __amdgpu_buffer_rsrc_t rg = state_rsrc(static_cast<S *>(ca.gout), uint32_t(L::Q) * pitch * E);
    const CRec own = c_record<S>(rc, h.n, pitch);
    const uint32_t wall = (h.lk & kLinkBits) ? wall_links(a, h.lk, ar) : 0u;
#pragma unroll
    for (int j = 0; j < L::Q; ++j) {
        const P2 v = c_pair<S>(c_total<S>(rc, uint32_t(j) * pitch + h.n, j), j, own);
        store_pair<P2>(rg, h.n * E, uint32_t(su(uint32_t(j) * pitch * E)), v);
        const int i = L::opp[j];
        if (j != 0 && ((wall >> i) & 1u))
            store_pair<P2>(rg, ar.vo(i) * E, uint32_t(su(uint32_t(i) * pitch * E)), v);
    }
}

// Whether a lattice and its plan fit the kernels (32-bit byte offsets must
// cover a pair state).
bool geo_ok(int prec, const Geo &g, const ModelD &md, const SplitPlan &sp) {
    if (md.bgk || !g.mask || !g.links || (prec != 1 && prec != 2)) return false;
    if (uint64_t(2 * D3Q19::Q) * uint64_t(g.pitch) * (prec == 1 ? 4u : 2u) >= (uint64_t(1) << 32)) return false;
    return sp.fluid >= 0 && sp.fluid <= g.N && sp.io >= 0 && sp.io <= sp.fluid;
}

template <typename S>
hipError_t run_split(const SplitDesc &a, hipStream_t s) {
    hipLaunchKernelGGL((k_geo_moments<S, false>), dim3(a.nblocks), dim3(kGeoBlock), 0, s, a);
    hipLaunchKernelGGL(k_geo_collide<S>, dim3(a.nblocks), dim3(kGeoBlock), 0, s, a);
    return hipGetLastError();
}

template <typename S>
hipError_t run_cgeo(CGeoArgs ca, bool pair_in, const uint32_t *io, uint32_t nio, hipStream_t s) {
    const SplitDesc &a = ca.s;
    if (pair_in)
        hipLaunchKernelGGL((k_geo_moments<S, true>), dim3(a.nblocks), dim3(kGeoBlock), 0, s, a);
    else
        hipLaunchKernelGGL(k_cgeo_moments<S>, dim3(a.nblocks), dim3(kGeoBlock), 0, s, ca);
    hipLaunchKernelGGL(k_cgeo_collide<S>, dim3(a.nblocks), dim3(kGeoBlock), 0, s, ca);
    if (nio > 0) {
        ca.s.list = io;
        ca.s.count = nio;
        hipLaunchKernelGGL(k_cgeo_boundary<S>, dim3((nio + kIoBlock - 1) / kIoBlock, D3Q19::Q - 1), dim3(kIoBlock), 0,
                           s, ca);
    }
    return hipGetLastError();
}

template <typename S>
hipError_t run_batch(const SplitDesc *desc, const LatMap *map, uint32_t blocks, hipStream_t s) {
    hipLaunchKernelGGL(k_geo_moments_batch<S>, dim3(blocks), dim3(kGeoBlock), 0, s, desc, map);
    hipLaunchKernelGGL(k_geo_collide_batch<S>, dim3(blocks), dim3(kGeoBlock), 0, s, desc, map);
    return hipGetLastError();
}

}  // namespace

// (The size is that of the moments, a node list and the counts, which callers
// plan their memory by; the lists and psi take 20 bytes of it.)
size_t split_scratch_bytes(int64_t pitch) {
    const size_t chunks = size_t((pitch + kChunk - 1) / kChunk);
    return align256(sizeof(float) * kSplitMoments * size_t(pitch)) + align256(sizeof(uint32_t) * size_t(pitch)) +
           align256(2 * sizeof(uint32_t) * chunks) + align256(sizeof(uint32_t));
}

hipError_t split_prepare(const Geo &g, void *scratch, SplitPlan &sp, hipStream_t s) {
    sp = SplitPlan{};
    if (!g.links || !g.mask || !scratch) return hipErrorInvalidValue;
    const ScratchMap m = scratch_map(scratch, g.pitch);
    const uint32_t N = uint32_t(g.N), nx = uint32_t(g.nx), ny = uint32_t(g.ny), chunks = uint32_t((g.N + kChunk - 1) / kChunk);
    uint32_t *none = nullptr;
    hipLaunchKernelGGL(k_geo_solid_psi, dim3(unsigned((g.N + kGeoBlock - 1) / kGeoBlock)), dim3(kGeoBlock), 0, s, g,
                       m.psi);
    hipLaunchKernelGGL(k_geo_list, dim3(chunks), dim3(kGeoBlock), 0, s, g.links, N, nx, ny, m.counts, none, none);
    hipLaunchKernelGGL(k_geo_scan, dim3(1), dim3(kScanThreads), 0, s, m.counts, chunks, m.totals);
    hipLaunchKernelGGL(k_geo_list, dim3(chunks), dim3(kGeoBlock), 0, s, g.links, N, nx, ny, m.counts, m.list, m.io);
    hipError_t e = hipGetLastError();
    uint32_t c[2] = {0, 0};
    if (e == hipSuccess) e = hipMemcpyAsync(c, m.totals, sizeof(c), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    if (int64_t(c[0]) > g.N || c[1] > c[0]) return hipErrorUnknown;
    sp.fluid = c[0];
    sp.io = c[1];
    return hipSuccess;
}

SplitDesc split_desc(const Geo &g, const ModelD &md, const void *in, void *out, void *scratch, const SplitPlan &sp,
                     const uint32_t *ctr_in, uint32_t *ctr_out) {
    const ScratchMap m = scratch_map(scratch, g.pitch);
    SplitDesc a{};
    a.in = in;
    a.out = out;
    a.psi = m.psi;
    a.mom = out;
    a.nx = g.nx;
    a.ny = g.ny;
    a.nz = g.nz;
    a.pitch = uint32_t(g.pitch);
    a.list = m.list;
    a.count = uint32_t(sp.fluid);
    // one block at least: it advances the step counter
    a.nblocks = uint32_t(sp.fluid > 0 ? (sp.fluid + kGeoBlock - 1) / kGeoBlock : 1);
    a.div0 = fast_div(uint32_t(g.nx));
    a.div1 = fast_div(uint32_t(g.ny));
    a.ctr_in = ctr_in;
    a.ctr_out = ctr_out;
    a.mask = g.mask;
    a.inlets = g.inlets;
    a.outlets = g.outlets;
    a.mo = to_model<float>(md);
    return a;
}

hipError_t launch_step_split(int prec, const Geo &g, const ModelD &md, const void *in, void *out, void *scratch,
                             const SplitPlan &sp, const uint32_t *ctr_in, uint32_t *ctr_out, hipStream_t s) {
    if (!scratch || !geo_ok(prec, g, md, sp)) return hipErrorInvalidValue;
    const SplitDesc a = split_desc(g, md, in, out, scratch, sp, ctr_in, ctr_out);
    return prec == 1 ? run_split<float>(a, s) : run_split<_Float16>(a, s);
}

hipError_t launch_step_split_batch(int prec, const SplitDesc *desc, const LatMap *map, uint32_t blocks,
                                   hipStream_t s) {
    if (blocks == 0) return hipSuccess;
    return prec == 1 ? run_batch<float>(desc, map, blocks, s) : run_batch<_Float16>(desc, map, blocks, s);
}

hipError_t launch_step_cgeo(int prec, const Geo &g, const ModelD &md, bool pair_in, const void *in, const void *gin,
                            void *cout, void *gout, void *scratch, const SplitPlan &sp, const uint32_t *ctr_in,
                            uint32_t *ctr_out, hipStream_t s) {
    if (!scratch || !geo_ok(prec, g, md, sp)) return hipErrorInvalidValue;
    CGeoArgs ca;
    ca.s = split_desc(g, md, in, cout, scratch, sp, ctr_in, ctr_out);
    ca.gin = gin;
    ca.gout = gout;
    const uint32_t *io = scratch_map(scratch, g.pitch).io;
    const uint32_t nio = uint32_t(sp.io);
    return prec == 1 ? run_cgeo<float>(ca, pair_in, io, nio, s) : run_cgeo<_Float16>(ca, pair_in, io, nio, s);
}

hipError_t launch_expand_cgeo(int prec, const Geo &g, const void *cin, void *pout, void *scratch, const SplitPlan &sp,
                              hipStream_t s) {
    if (!scratch || !geo_ok(prec, g, ModelD{}, sp)) return hipErrorInvalidValue;
    if (sp.fluid == 0) return hipSuccess;
    CGeoArgs ca;
    ca.s = split_desc(g, ModelD{}, cin, nullptr, scratch, sp, nullptr, nullptr);
    ca.gin = nullptr;
    ca.gout = pout;
    if (prec == 1)
        hipLaunchKernelGGL(k_cgeo_expand<float>, dim3(ca.s.nblocks), dim3(kGeoBlock), 0, s, ca);
    else
        hipLaunchKernelGGL(k_cgeo_expand<_Float16>, dim3(ca.s.nblocks), dim3(kGeoBlock), 0, s, ca);
    return hipGetLastError();
}

}  // namespace lbcg
