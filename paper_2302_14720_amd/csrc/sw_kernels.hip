// sw_kernels.hip -- gfx950 kernels of one Swendsen-Wang sweep (see
// sw_internal.h for the pipeline).  Written for 64-wide wavefronts: a tile
// row of 64 sites is one 64-bit mask, so row runs of horizontal bonds come
// from bit arithmetic on ballot-sized masks, and only vertical bonds go
// through the LDS union-find.
#include <math.h>

#include <algorithm>

#include "sw_device.h"
#include "sw_internal.h"
#include "sw_philox.h"
#include "sw_uf.h"

namespace swmi {
namespace {

constexpr uint32_t kEmpty = 0xFFFFFFFFu;

// Accesses at agent scope: seen by every XCD without cache fences.
template <class T> __device__ __forceinline__ T ag_load(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T> __device__ __forceinline__ void ag_store(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int TW> struct RowOf;
template <> struct RowOf<64> { using T = uint64_t; };
template <> struct RowOf<32> { using T = uint32_t; };

// Highest set bit of B at a position <= x (bit 0 of B is always set).
__device__ __forceinline__ uint32_t hsb_le(uint64_t B, uint32_t x) {
    const uint64_t m = B & (~0ull >> (63u - x));
    return 63u - (uint32_t)__clzll((long long)m);
}
__device__ __forceinline__ uint32_t hsb_le(uint32_t B, uint32_t x) {
    const uint32_t m = B & (~0u >> (31u - x));
    return 31u - (uint32_t)__clz((int)m);
}

// A lane's segment of SPT consecutive sites (bytes).
template <int SPT> struct Seg {
    uint32_t w[SPT / 4];
};
template <int SPT> __device__ __forceinline__ Seg<SPT> load_seg(const int8_t *p) {
    Seg<SPT> v;
    if constexpr (SPT == 16) {
        const uint4 x = *reinterpret_cast<const uint4 *>(p);
        v.w[0] = x.x;
        v.w[1] = x.y;
        v.w[2] = x.z;
        v.w[3] = x.w;
    } else {
        v.w[0] = *reinterpret_cast<const uint32_t *>(p);
    }
    return v;
}
template <int SPT> __device__ __forceinline__ void store_seg(void *p, const uint32_t *w) {
    if constexpr (SPT == 16)
        *reinterpret_cast<uint4 *>(p) = make_uint4(w[0], w[1], w[2], w[3]);
    else
        *reinterpret_cast<uint32_t *>(p) = w[0];
}
template <int SPT> __device__ __forceinline__ uint32_t byte_at(const Seg<SPT> &v, int q) {
    return (v.w[q >> 2] >> (8 * (q & 3))) & 0xFFu;
}

// The TW-bit row mask whose SPT-bit pieces are held by the TW / SPT
// consecutive lanes of a tile row: data-parallel moves within rows of 16
// lanes, no LDS.  Four lanes (a quad) or two exchange their 16-bit pieces;
// sixteen or eight or together their 4-bit pieces, each at its place.
template <int CTRL> __device__ __forceinline__ uint32_t dpp(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, false);
}
template <int K, int RPT>
__device__ __forceinline__ uint32_t row_piece(uint32_t v) {
    return dpp<RPT == 4 ? K * 0x55 : (K | (K << 2) | ((2 + K) << 4) | ((2 + K) << 6))>(v);
}
template <int RPT> __device__ __forceinline__ uint32_t row_or(uint32_t v) {
    v |= dpp<0xB1>(v);   // lane ^ 1
    v |= dpp<0x4E>(v);   // lane ^ 2
    v |= dpp<0x141>(v);  // the other quad of 8 lanes
    if constexpr (RPT == 16) v |= dpp<0x140>(v);  // the other half of 16
    return v;
}
template <int TW, int SPT>
__device__ __forceinline__ typename RowOf<TW>::T row_gather(uint32_t piece, uint32_t seg) {
    if constexpr (SPT == 4 && TW == 64) {
        const uint32_t v = piece << (4u * (seg & 7u));
        const uint32_t lo = row_or<16>(seg < 8u ? v : 0u), hi = row_or<16>(seg < 8u ? 0u : v);
        return lo | ((uint64_t)hi << 32);
    } else if constexpr (SPT == 4) {
        return row_or<8>(piece << (4u * seg));
    } else if constexpr (TW == 64) {
        const uint64_t lo = row_piece<0, 4>(piece) | (row_piece<1, 4>(piece) << 16);
        const uint64_t hi = row_piece<2, 4>(piece) | (row_piece<3, 4>(piece) << 16);
        return lo | (hi << 32);
    } else {
        return row_piece<0, 2>(piece) | (row_piece<1, 2>(piece) << 16);
    }
}

// New value of a node's cluster in the previous sweep: the Potts value, or 1
// for spin +1 and 0 for -1 (Ising).  Lattices merged by k_merge keep a
// reference per node: the value itself, or kRef + j for cluster j of the
// tile's group, whose table starts at gb (ref_slots per group); the others
// keep the spin.  Both steps are loads without a compare behind them, so that
// the loads of several nodes overlap (a compare between them makes the tile
// kernel wait for each: 0.93 -> 0.97 ms at 16384^2).
// TWO: 1 merged by k_merge, 0 not, 2 as d.two says (batches of both): the
// test alone cost the tile kernel 2 % at 1600^2.
template <int TWO> __device__ __forceinline__ bool has_refs(const Dev &d) { return TWO == 1 || (TWO == 2 && d.two); }
template <int TWO> __device__ __forceinline__ uint32_t node_ref(const Dev &d, uint32_t node) {
    return has_refs<TWO>(d) ? d.nref[node] : (uint32_t)(int32_t)d.rspin[node];
}
template <int TWO> __device__ __forceinline__ uint32_t follow_ref(const Dev &d, uint32_t ref, uint32_t gb) {
    if (has_refs<TWO>(d) && ref >= kRef) return d.gspin[gb + ref - kRef];
    return ref;
}
template <bool POTTS, int TWO> __device__ __forceinline__ uint32_t value_of(const Dev &d, uint32_t v) {
    if (POTTS || has_refs<TWO>(d)) return v;
    return (uint32_t)((int32_t)v > 0);
}
// Start of the cluster table of the group that holds tile (tx, ty).
__device__ __forceinline__ uint32_t ref_base(const Dev &d, uint32_t tx, uint32_t ty) {
    return ((ty / kUG) * ((d.ntx + kUG - 1u) / kUG) + tx / kUG) * ref_slots(d.tw);
}

// Output bytes of the Potts model on the tile path: a byte below
// potts_code<TW>() is a final value, potts_code<TW>() + k refers to node k of
// its tile.  A 32-wide tile has at most 124 nodes, so all values 0..7 fit
// below 8; a 64-wide tile has up to 252 nodes, which leaves bytes 0..3 for
// the values of q <= 4.
template <int TW> constexpr uint32_t potts_code() { return TW == 64 ? 4u : 8u; }

// Shared front end of k_tile and k_resolve: the table that maps every byte
// of this tile's previous output to its value (Ising: an up bit, 1 for +1):
// final spins map to themselves, node code 2 + k (Potts: potts_code<TW>() + k)
// to the new value of node k's cluster.
// The node spins are loaded whether or not the node exists (every slot is
// in bounds), so that this load does not wait for the node count.
template <int TW, bool POTTS, int TWO, int NT>
__device__ __forceinline__ void load_table(const Dev &d, uint32_t tile, uint32_t gb, uint32_t pp, uint8_t *s_tab,
                                           uint32_t tid) {
    const uint32_t kprev = min(d.nk[pp][tile], 252u);
    for (uint32_t b = tid; b < 256u; b += NT) {
        uint8_t val;
        uint32_t k;
        if constexpr (POTTS) {
            val = (uint8_t)(b & 7u);
            k = b - potts_code<TW>();
        } else {
            val = b == 0xFFu ? 0u : 1u;
            k = b - 2u;
        }
        const uint32_t ref = k < 252u ? node_ref<TWO>(d, tile * kNodeSlots + k) : 0u;
        const uint32_t ns = value_of<POTTS, TWO>(d, follow_ref<TWO>(d, k < kprev ? ref : 0u, gb));
        if (k < kprev) val = (uint8_t)ns;
        s_tab[b] = val;
    }
}

template <int SPT>
__device__ __forceinline__ uint32_t decode(const Seg<SPT> &v, const uint8_t *s_tab) {
    uint32_t up = 0;
#pragma unroll
    for (int q = 0; q < SPT; ++q) up |= (uint32_t)s_tab[byte_at(v, q)] << q;
    return up;
}

// Values (Ising: up bits) of N bytes of tile `tile`'s previous output, which
// is not this workgroup's: final bytes as they are, a code refers to a node.
template <int TW, bool POTTS, int TWO, int N>
__device__ __forceinline__ void remote_values(const Dev &d, const uint32_t *b, uint32_t tile, uint32_t gb, uint32_t *val) {
    constexpr uint32_t CB = POTTS ? potts_code<TW>() : 2u;
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const uint32_t k = b[q] - CB;
        val[q] = POTTS ? b[q] : has_refs<TWO>(d) ? (uint32_t)(b[q] == 1u) : (uint32_t)(int32_t)(int8_t)b[q];
        if (k < 252u) val[q] = node_ref<TWO>(d, tile * kNodeSlots + k);
    }
    if (has_refs<TWO>(d)) {
#pragma unroll
        for (int q = 0; q < N; ++q)
            if (b[q] - CB < 252u) val[q] = follow_ref<TWO>(d, val[q], gb);
    }
#pragma unroll
    for (int q = 0; q < N; ++q) val[q] = value_of<POTTS, TWO>(d, val[q]);
}

template <int TWO, int SPT>
__device__ __forceinline__ uint32_t decode_remote(const Dev &d, const Seg<SPT> &v, uint32_t tile, uint32_t gb) {
    uint32_t b[SPT], x[SPT], up = 0;
#pragma unroll
    for (int q = 0; q < SPT; ++q) b[q] = byte_at(v, q);
    remote_values<64, false, TWO, SPT>(d, b, tile, gb, x);
#pragma unroll
    for (int q = 0; q < SPT; ++q) up |= x[q] << q;
    return up;
}

// Values of a segment's sites as three bit planes (bit q of pl[i] = bit i of
// site q).
template <int SPT>
__device__ __forceinline__ void decode_potts(const Seg<SPT> &v, const uint8_t *s_tab, uint32_t pl[3]) {
    pl[0] = pl[1] = pl[2] = 0u;
#pragma unroll
    for (int q = 0; q < SPT; ++q) {
        const uint32_t x = s_tab[byte_at(v, q)];
        pl[0] |= (x & 1u) << q;
        pl[1] |= ((x >> 1) & 1u) << q;
        pl[2] |= (x >> 2) << q;
    }
}

template <int TW, int TWO, int SPT>
__device__ __forceinline__ void decode_potts_remote(const Dev &d, const Seg<SPT> &v, uint32_t tile, uint32_t gb,
                                                    uint32_t pl[3]) {
    uint32_t b[SPT], x[SPT];
#pragma unroll
    for (int q = 0; q < SPT; ++q) b[q] = byte_at(v, q);
    remote_values<TW, true, TWO, SPT>(d, b, tile, gb, x);
    pl[0] = pl[1] = pl[2] = 0u;
#pragma unroll
    for (int q = 0; q < SPT; ++q) {
        pl[0] |= (x[q] & 1u) << q;
        pl[1] |= ((x[q] >> 1) & 1u) << q;
        pl[2] |= ((x[q] >> 2) & 1u) << q;
    }
}

// Bits 0-7 of v at the even positions of a 16-bit mask.
__device__ __forceinline__ uint32_t spread8(uint32_t v) {
    v &= 0xFFu;
    v = (v | (v << 4)) & 0x0F0Fu;
    v = (v | (v << 2)) & 0x3333u;
    return (v | (v << 1)) & 0x5555u;
}

// =====================================================================
// k_tile: bonds (Sec. 2.1), tile-local clusters (Sec. 2.3), new spins of
// tile-interior clusters (Sec. 2.4), measurement of the incoming
// configuration (Sec. 2.5).  One workgroup per TW x TW tile, SPT = 16 or 4
// sites of a row per thread, so per-row bond and run data are bit masks and
// most per-site work is one bit operation per SPT sites.
// Cluster formation: every site's LDS word first points at the start of its
// row run; vertical bonds (one per group that joins the same two runs) are
// unions of run starts; each run start is then pointed at its root, which
// collects the cluster size and, after numbering, the output byte.
// =====================================================================
// POTTS: the q-state Potts model (64-wide tiles for q <= 4, else 32-wide):
// spins are values held as three bit planes, bonds join equal values, an
// interior cluster takes the Potts value of its root site, node codes start
// at potts_code<TW>(), and the tile measures equal pairs and the population
// of every value.
// DENSE: interior clusters also go to the exact size histogram -- those
// below kDenseBins sites through LDS counts that leave with the tile
// (tdense) and are added up per group in k_roots.
// LDS of a tile workgroup.
template <int TW, bool POTTS, bool DENSE, int SPT> struct TileShared {
    using Row = typename RowOf<TW>::T;
    static constexpr int NPL = POTTS ? 3 : 1, NWAVE = (TW * TW / SPT + 63) / 64;
    // One word per site, rows padded to TW + 1 words so that the sites the
    // lanes gather at equal offsets fall in distinct banks.  Low 16 bits:
    // parent, as the byte offset of its word.  High 16 bits: the union work
    // list while the unions run, then the cluster size (roots), then the
    // root's output byte.
    alignas(16) uint32_t par[TW * (TW + 1)];
    Row up[POTTS && TW != 64 ? NPL * (TW + 1) : 1];  // bit planes (Potts)
    Row ebnb[2 * TW];  // bond masks to E of every row (rows 0..TW-1)
    Row fb[TW];        // new spins of every site as a root (Ising)
    Row xn;            // bonds out to N
    Row pw;            // permitted incoming bonds by row (from the W tile's last column)
    uint32_t ps[2];    // and by column, even and odd (from the S tile's last row)
    uint32_t eup[NPL * ((TW + 31) / 32)];
    uint32_t xe[(TW + 31) / 32];
    uint32_t bf[TW * TW / 32];
    uint32_t hist[kTileBins];
    uint32_t dense[DENSE ? kDenseBins : 1];
    uint32_t node[TW == 64 ? 1 : 4 * TW];
    int32_t red[NWAVE][POTTS ? 8 : 4];
    uint8_t tab[256];
};

// SPT: sites per thread, 16 or 4.  With 16 the row masks cost least per site
// and the tiles of a large lattice fill the GPU; a lattice of few tiles leaves
// a wavefront or less per SIMD, which waits through every chain of its 16
// sites alone, so there four times as many threads take 4 each (512^2,
// beta_c: 22 -> 14 us).
template <int TW, bool POTTS, bool DENSE, int TWO, int SPT>
__device__ __forceinline__ void tile_body(const Dev &d, const uint32_t tile, TileShared<TW, POTTS, DENSE, SPT> &sh) {
    using Row = typename RowOf<TW>::T;
    constexpr int NT = TW * TW / SPT;
    constexpr uint32_t RPT = TW / SPT;  // lanes per row
    constexpr uint32_t M = (1u << SPT) - 1u, TOP = 1u << (SPT - 1);  // a lane's sites, its last
    constexpr int NS = TW * TW;
    constexpr int NW = NS / 32;
    constexpr int NWAVE = (NT + 63) / 64;
    constexpr int NPL = POTTS ? 3 : 1;  // bit planes of a spin
    constexpr uint32_t EW = (TW + 31) / 32;
    constexpr uint32_t CB = POTTS ? potts_code<TW>() : 2u;  // output byte of node 0
    // Which clusters become nodes: those with a bond out of the tile, for which
    // the bonds that come in are drawn again, or all that touch the tile's edge.
    // A 32-wide tile of one wavefront pays a ninth Philox call beside its eight
    // and gains less than that: us per sweep all / bonded, 4064^2 at beta_c
    // 165.7 / 170.0, beta = 0.6 170.3 / 175.3, 8160^2 at beta_c 464 / 473 (only
    // in the disordered phase of few tiles it loses: 2080^2, beta = 0.3, 70.9 /
    // 67.6).
    constexpr bool INCOMING = TW == 64 || SPT == 4;

    constexpr uint32_t PS = TW + 1;
    auto &s_par = sh.par;
    // the 64-wide Potts tile keeps its three planes in par, which is not in use
    // yet while they live
    constexpr bool UP_IN_PAR = POTTS && TW == 64;
    static_assert(!UP_IN_PAR || 3 * (TW + 1) * sizeof(Row) <= TW * PS * 4, "planes must fit in par");
    Row *const s_up = UP_IN_PAR ? reinterpret_cast<Row *>(sh.par) : sh.up;
    Row *const s_eb = sh.ebnb;
    auto &s_fb = sh.fb;
    auto &s_xn = sh.xn;
    auto &s_pw = sh.pw;
    auto &s_ps = sh.ps;
    auto &s_eup = sh.eup;
    auto &s_xe = sh.xe;
    auto &s_bf = sh.bf;
    auto &s_tab = sh.tab;
    auto &s_hist = sh.hist;
    auto &s_dense = sh.dense;
    // root | size << 16 of each node; for 64-wide tiles it reuses the bond
    // masks, which are dead once the unions are done
    uint32_t *const s_node = TW == 64 ? reinterpret_cast<uint32_t *>(sh.ebnb) : sh.node;
    auto &s_red = sh.red;

    const uint32_t tid = threadIdx.x;
    const uint32_t L = d.L, ntx = d.ntx;
    const uint32_t tx = tile % ntx, ty = tile / ntx;
    const uint64_t tsw = *d.tdev;
    const uint32_t t = (uint32_t)tsw;
    const uint32_t pc = (uint32_t)(tsw & 1u), pp = pc ^ 1u;
    const int8_t *__restrict__ sin = d.spins[pc];
    int8_t *__restrict__ sout = d.spins[pp];
    uint32_t *__restrict__ par_cur = d.parent;

    const uint32_t ly = tid / RPT, seg = tid % RPT, x0 = seg * (uint32_t)SPT;
    const uint32_t gy = ty * TW + ly, gx0 = tx * TW + x0;
    const uint32_t east = ty * ntx + (tx + 1u == ntx ? 0u : tx + 1u);
    const uint32_t north = (ty + 1u == ntx ? 0u : ty + 1u) * ntx + tx;
    const uint32_t txw = tx == 0u ? ntx - 1u : tx - 1u, tys = ty == 0u ? ntx - 1u : ty - 1u;
    const uint32_t gbe = ref_base(d, tx + 1u == ntx ? 0u : tx + 1u, ty);
    const uint32_t gbn = ref_base(d, tx, ty + 1u == ntx ? 0u : ty + 1u);
    const uint32_t rowbase = ly * PS;  // padded index of the row's first site
    const uint32_t rowoff = 4u * rowbase;  // its byte offset
    const uint32_t srow = ly * TW;     // site index of the row's first site

    // rows of the tile a wavefront holds; lanes of a wavefront's last row
    // (Ising) decode the next row's spins themselves, the others take them
    // from the lanes RPT above
    constexpr uint32_t RPW = 64u / RPT;
    const bool wlast = (ly % RPW) == RPW - 1u;

    // ---- issue the spin loads first, then build the node table
    const Seg<SPT> v = load_seg<SPT>(sin + (size_t)gy * L + gx0);
    Seg<SPT> vn{};
    if (POTTS ? ly == TW - 1 : wlast) {
        const uint32_t gyn = (gy + 1u == L) ? 0u : gy + 1u;
        vn = load_seg<SPT>(sin + (size_t)gyn * L + gx0);
    }
    uint32_t ve = 0;
    if (seg == RPT - 1) {
        const uint32_t gxe = (gx0 + SPT == L) ? 0u : gx0 + SPT;
        ve = (uint8_t)sin[(size_t)gy * L + gxe];
    }
    // and the neighbours whose bonds come in through the W and S edges
    Seg<SPT> vs{};
    const uint32_t xw = txw * TW + TW - 1u, ys = tys * TW + TW - 1u;
    uint32_t vw = 0u;
    if (INCOMING && ly == 0u) vs = load_seg<SPT>(sin + (size_t)ys * L + gx0);
    if (INCOMING && seg == 0u) vw = (uint8_t)sin[(size_t)gy * L + xw];
    // the bond words of this lane's sites (Sec. 2.1), drawn while the
    // loads are in flight: bit 2j (2j+1) of rE / rN is the E / N edge of
    // site 2j (2j+1) past the lane's first site, set iff its word is below T
    uint32_t rE = 0u, rN = 0u;
    {
        const uint32_t c0 = (gy * L + gx0) >> 1;
        const uint32_t T = d.T;
#pragma unroll
        for (int j = SPT / 2 - 1; j >= 0; --j) {
            uint32_t w0 = c0 + (uint32_t)j, w1 = t, w2 = 0u, w3 = 0u;
            philox10(w0, w1, w2, w3, d.seed_lo, d.seed_hi);
            rE = shift_in_below(shift_in_below(rE, w2, T), w0, T);
            rN = shift_in_below(shift_in_below(rN, w3, T), w1, T);
        }
    }
    load_table<TW, POTTS, TWO, NT>(d, tile, ref_base(d, tx, ty), pp, s_tab, tid);

    // Potts: the value each of this lane's sites would give its cluster
    // as its root (4 bits per site): word i of the output for counter
    // {s >> 2, t, 3, 0} for site s = 4j + i past the lane's first site
    uint64_t pv = 0;
    if constexpr (POTTS) {
        const uint32_t r0 = gy * L + gx0, q = d.q;
#pragma unroll
        for (uint32_t j = 0; j < SPT / 4u; ++j) {
            uint32_t w0 = (r0 >> 2) + j, w1 = t, w2 = 3u, w3 = 0u;
            philox10(w0, w1, w2, w3, d.seed_lo, d.seed_hi);
            const uint64_t v4 = (uint64_t)(((uint64_t)w0 * q) >> 32) | ((((uint64_t)w1 * q) >> 32) << 4) |
                                ((((uint64_t)w2 * q) >> 32) << 8) | ((((uint64_t)w3 * q) >> 32) << 12);
            pv |= v4 << (16u * j);
        }
    }
    // Ising: flip bits of every tile row, one Philox call per row of TW sites
    if (!POTTS && tid < (uint32_t)TW) {
        const uint32_t r0 = (ty * TW + tid) * L + tx * TW;
        uint32_t w0 = r0 >> 7, w1 = t, w2 = 1u, w3 = 0u;
        philox10(w0, w1, w2, w3, d.seed_lo, d.seed_hi);
        const uint32_t off = r0 & 127u;
        if constexpr (TW == 64) {
            s_fb[tid] = off == 0u ? (((uint64_t)w1 << 32) | w0) : (((uint64_t)w3 << 32) | w2);
        } else {
            const uint32_t q = off >> 5;
            s_fb[tid] = q == 0 ? w0 : q == 1 ? w1 : q == 2 ? w2 : w3;
        }
    }
    // The neighbours' words of the bonds that come in (they own those edges):
    // one lane per row (site (xw, y), whose E word is word 2: xw is odd) and
    // one per two columns, 1.5 calls per 64 of a tile side beside its 8 per 16
    // sites.  With them only clusters that do go on outside become nodes: 48
    // of the 80 that touch the edge of a 64-wide tile at beta_c.
    if constexpr (INCOMING) {
        constexpr uint32_t W0 = NT > 64 ? 64u : 0u;  // a wavefront other than the one above, if there is one
        const uint32_t r = tid - W0, c = TW == 64 ? tid - 128u : tid - W0 - 32u;
        const bool isw = r < (uint32_t)TW, iss = c < (uint32_t)TW / 2u;
        if (tid >= W0 && tid < W0 + (TW == 64 ? 128u : 64u)) {
            uint32_t w0 = (isw ? (ty * TW + r) * L + xw : iss ? ys * L + tx * TW + 2u * c : 0u) >> 1;
            uint32_t w1 = t, w2 = 0u, w3 = 0u;
            philox10(w0, w1, w2, w3, d.seed_lo, d.seed_hi);
            const uint64_t bw = __ballot(isw && w2 < d.T);
            const uint64_t b0 = __ballot(iss && w1 < d.T), b1 = __ballot(iss && w3 < d.T);
            if (r == 0u) s_pw = (Row)bw;
            if (c == 0u) {
                s_ps[0] = (uint32_t)(TW == 64 ? b0 : b0 >> 32);
                s_ps[1] = (uint32_t)(TW == 64 ? b1 : b1 >> 32);
            }
        }
    }
    for (uint32_t i = tid; i < (uint32_t)NW; i += NT) s_bf[i] = 0u;
    if (tid < EW) s_xe[tid] = 0u;
    if (tid < NPL * EW) s_eup[tid] = 0u;
    if (tid < kTileBins) s_hist[tid] = 0u;
    if constexpr (DENSE)
        for (uint32_t i = tid; i < kDenseBins; i += NT) s_dense[i] = 0u;
    if (tid == 0) s_xn = 0;
    __syncthreads();

    // ---- decode the incoming configuration (Sec. 2.5 measures it; Sec. 2.1
    // bonds it).  Ising: the up-spin mask of the lane's sites, of the
    // sites above (lanes RPT further on, or decoded here by a wavefront's
    // last row) and the east neighbour of its last site (the next lane, or
    // the east tile).  Potts: three bit planes per row, through LDS.
    // a lane's piece of a row mask in LDS
    auto put_piece = [&](Row *row, uint32_t piece) {
        if constexpr (SPT == 16) {
            reinterpret_cast<uint16_t *>(row)[seg] = (uint16_t)piece;
        } else {
            const Row m = row_gather<TW, SPT>(piece, seg);
            if (seg == 0u) *row = m;
        }
    };
    uint32_t up = 0u, pl[3] = {0u, 0u, 0u};
    uint32_t upN = 0u, ebit = 0u;
    uint32_t inS = 0u, inW = 0u;  // equal neighbours across the S edge (first row) and W edge (first column)
    if constexpr (POTTS) {
        decode_potts(v, s_tab, pl);
#pragma unroll
        for (int b = 0; b < 3; ++b) put_piece(s_up + b * (TW + 1) + ly, pl[b]);
        if (ly == TW - 1) {
            uint32_t pn[3];
            decode_potts_remote<TW, TWO>(d, vn, north, gbn, pn);
#pragma unroll
            for (int b = 0; b < 3; ++b) put_piece(s_up + b * (TW + 1) + TW, pn[b]);
        }
        if (seg == RPT - 1) {
            uint32_t ev;
            remote_values<TW, true, TWO, 1>(d, &ve, east, gbe, &ev);
#pragma unroll
            for (uint32_t b = 0; b < 3u; ++b)
                if ((ev >> b) & 1u) atomicOr(&s_eup[b * EW + (ly >> 5)], 1u << (ly & 31u));
        }
        // bit 0: the W neighbour's value equals this row's first site's
        if (INCOMING && ly == 0u) {
            uint32_t pn[3];
            decode_potts_remote<TW, TWO>(d, vs, tys * ntx + tx, ref_base(d, tx, tys), pn);
            inS = ~((pl[0] ^ pn[0]) | (pl[1] ^ pn[1]) | (pl[2] ^ pn[2])) & M;
        }
        if (INCOMING && seg == 0u) {
            uint32_t wv;
            remote_values<TW, true, TWO, 1>(d, &vw, ty * ntx + txw, ref_base(d, txw, ty), &wv);
            inW = wv == ((pl[0] & 1u) | ((pl[1] & 1u) << 1) | ((pl[2] & 1u) << 2)) ? 1u : 0u;
        }
        __syncthreads();
    } else {
        up = decode(v, s_tab);
        if (INCOMING && ly == 0u) inS = ~(up ^ decode_remote<TWO>(d, vs, tys * ntx + tx, ref_base(d, tx, tys))) & M;
        if (INCOMING && seg == 0u) {
            uint32_t wv;
            remote_values<TW, false, TWO, 1>(d, &vw, ty * ntx + txw, ref_base(d, txw, ty), &wv);
            inW = ~(up ^ wv) & 1u;
        }
        const uint32_t upA = (uint32_t)__shfl_down((int)up, (int)RPT, 64);
        const uint32_t upR = (uint32_t)__shfl_down((int)up, 1, 64);
        if (wlast)
            upN = ly == TW - 1 ? decode_remote<TWO>(d, vn, north, gbn) : decode(vn, s_tab);
        else
            upN = upA;
        ebit = upR & 1u;
        if (seg == RPT - 1) remote_values<TW, false, TWO, 1>(d, &ve, east, gbe, &ebit);
    }

    // ---- bonds (Sec. 2.1) and energy / magnetisation of the incoming spins
    // (Potts: equal pairs and value populations); then every site points at
    // the start of its row run (the row's E bonds are gathered from its RPT
    // lanes), and the bond masks go to LDS for the vertical unions
    int32_t e_part, m_part;
    uint32_t cpk[4] = {0u, 0u, 0u, 0u};
    uint32_t bE, bN;
    uint32_t linked = 0u;  // this lane's sites whose clusters become nodes
    {
        uint32_t eqE, eqN;
        if constexpr (POTTS) {
            uint32_t dE = 0u, dN = 0u;
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const Row rowv = s_up[b * (TW + 1) + ly];
                const uint32_t pN = (uint32_t)(s_up[b * (TW + 1) + ly + 1] >> x0) & M;
                const uint32_t eb = (s_eup[b * EW + (ly >> 5)] >> (ly & 31u)) & 1u;
                const uint32_t nxt = (x0 + SPT < (uint32_t)TW) ? ((uint32_t)(rowv >> (x0 + SPT)) & 1u) : eb;
                const uint32_t pE = (pl[b] >> 1) | (nxt << (SPT - 1));
                dE |= pl[b] ^ pE;
                dN |= pl[b] ^ pN;
            }
            eqE = ~dE & M;
            eqN = ~dN & M;
            e_part = __popc(eqE) + __popc(eqN);
            m_part = 0;
            potts_counts<M>(pl, cpk);
        } else {
            const uint32_t upE = (up >> 1) | (ebit << (SPT - 1));
            eqE = ~(up ^ upE) & M;
            eqN = ~(up ^ upN) & M;
            e_part = 2 * (__popc(eqE) + __popc(eqN)) - 2 * SPT;
            m_part = 2 * __popc(up) - SPT;
        }
        bE = eqE & rE;
        bN = eqN & rN;
        if (seg == RPT - 1) {
            if (bE & TOP) atomicOr(&s_xe[ly >> 5], 1u << (ly & 31u));
            if (INCOMING) linked = bE & TOP;
            bE &= TOP - 1u;
        }
        if (ly == TW - 1) {
            put_piece(&s_xn, bN);
            if (INCOMING) linked |= bN;
            bN = 0u;
        }
        if constexpr (INCOMING) {
            if (ly == 0u) linked |= M & inS & (spread8(s_ps[0] >> (x0 / 2u)) | (spread8(s_ps[1] >> (x0 / 2u)) << 1));
            if (seg == 0u) linked |= inW & (uint32_t)(s_pw >> ly);
        } else {
            linked = ly == 0u || ly == (uint32_t)TW - 1u ? M : (seg == 0u ? 1u : 0u) | (seg == RPT - 1u ? TOP : 0u);
        }
        if constexpr (SPT == 16) put_piece(&s_eb[ly], bE);
    }
    const Row E0 = row_gather<TW, SPT>(bE, seg);  // this row's E bonds inside the tile
    const Row V = row_gather<TW, SPT>(bN, seg);   // this row's N bonds inside the tile
    if constexpr (SPT != 16)
        if (seg == 0u) s_eb[ly] = E0;
    const Row B0 = (Row)~(Row)(E0 << 1);
    const uint32_t st = (uint32_t)(B0 >> x0) & M;
    const uint32_t rs0 = rowoff + 4u * hsb_le(B0, x0);  // byte offset of the run start at x0
    // the 64-wide Potts tile keeps its planes in s_par: wait until every
    // lane has read them
    if constexpr (UP_IN_PAR) __syncthreads();
    {
        uint32_t cur = rs0;
#pragma unroll
        for (int q = 0; q < SPT; ++q) {
            if ((st >> q) & 1u) cur = rowoff + 4u * (x0 + (uint32_t)q);
            s_par[rowbase + x0 + q] = cur;
        }
        if (seg == RPT - 1u) s_par[rowbase + TW] = 0u;  // pad word: list slot only
    }
    __syncthreads();

    // ---- vertical bonds join runs of adjacent rows.  One union per group of
    // vertical bonds that connect the same pair of runs; each wavefront lists
    // its unions in the high halves of its own rows' words and then works
    // through the list 64 at a time, so that lanes with many bonds do not
    // hold up the rest.  The list is private to the wavefront; the compare-
    // and-swap of a union keeps a word's high half and retries if it
    // changed, so other wavefronts may build or clear their lists meanwhile.
    uint32_t r = 0u;  // representative vertical bonds of this segment
    if (ly + 1u < (uint32_t)TW) {
        const Row E1 = s_eb[ly + 1];
        const Row R = V & (Row)~(Row)((V << 1) & (E0 << 1) & (E1 << 1));
        r = (uint32_t)(R >> x0) & M;
    }
    const uint32_t lane = tid & 63u;
    const uint32_t wbase = (tid >> 6) * (64u / RPT) * PS;
    uint32_t nlist;
    {
        const uint32_t c = __popc(r);
        uint32_t pre = 0u;
        nlist = 0u;
#pragma unroll
        for (int j = 0; j < (SPT == 16 ? 5 : 3); ++j) {  // the bits of a count up to SPT
            const uint64_t bal = __ballot((c >> j) & 1u);
            pre += (uint32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                      __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u))
                   << j;
            nlist += (uint32_t)__popcll(bal) << j;
        }
        uint32_t w = wbase + pre, rr = r;
        while (rr) {
            const uint32_t i = (uint32_t)__ffs((int)rr) - 1u;
            rr &= rr - 1u;
            __hip_atomic_fetch_or(&s_par[w], (rowoff + 4u * (x0 + i)) << 16, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_WORKGROUP);
            ++w;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (uint32_t k = lane; k < nlist; k += 64u) {
        const uint32_t n = lds_load(&s_par[wbase + k]) >> 16;
        __hip_atomic_fetch_and(&s_par[wbase + k], 0xFFFFu, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        lds_union_lo(s_par, n, n + 4u * PS);
    }
    __syncthreads();

    // ---- cluster sizes.  Every run start in this lane's sites is pointed
    // at its root and adds the whole run's length (read off the row's
    // run-start mask; the run may go on into the next lanes' sites).  Runs
    // with linked sites mark their root.
    uint32_t rootmask = 0u;
    {
        // where the run holding the lane's last site ends: the first run
        // start past the lane's sites, or the row's end
        uint32_t end_out = (uint32_t)TW;
        if (x0 + SPT < (uint32_t)TW) {
            const Row past = (Row)(B0 >> (x0 + SPT));
            if (past) end_out = x0 + SPT + (uint32_t)__builtin_ctzll((unsigned long long)past);
        }
        // lengths of consecutive runs with the same root are summed in a
        // register (at most TW per lane) and added with one atomic
        uint32_t acc_root = 0u, acc_len = 0u;
        uint32_t m = st;
        while (m) {
            const uint32_t i = (uint32_t)__ffs((int)m) - 1u;
            m &= m - 1u;
            const uint32_t n = rowoff + 4u * (x0 + i);
            const uint32_t root = lds_root_b(s_par, n);
            if (root != n)
                __hip_atomic_store(word_at(s_par, n), root, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            else
                rootmask |= 1u << i;
            // the run's sites in this lane: up to the next start or the lane's last
            const uint32_t upto = m ? (m & (0u - m)) - 1u : M;
            if ((linked & upto) >> i) {
                const uint32_t rsite = root / 4u - root / (4u * PS);
                atomicOr(&s_bf[rsite >> 5], 1u << (rsite & 31u));
            }
            // the run goes on to the lane's next run start, or past the lane
            const uint32_t len = (m ? (uint32_t)__ffs((int)m) - 1u + x0 : end_out) - (x0 + i);
            if (root != acc_root && acc_len != 0u)
                __hip_atomic_fetch_add(word_at(s_par, acc_root), acc_len << 16, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            acc_len = root != acc_root ? len : acc_len + len;
            acc_root = root;
        }
        if (acc_len != 0u)
            __hip_atomic_fetch_add(word_at(s_par, acc_root), acc_len << 16, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        // a segment that starts inside a run: its sites before the first start
        if (linked & (st ? (st & (0u - st)) - 1u : M)) {
            const uint32_t root = lds_root_b(s_par, rs0);
            const uint32_t rsite = root / 4u - root / (4u * PS);
            atomicOr(&s_bf[rsite >> 5], 1u << (rsite & 31u));
        }
    }
    __syncthreads();

    // ---- number the marked clusters (nodes) in site order: every
    // wavefront scans the marks itself, lane l holding the prefix of mark
    // words (NW / 64) l .. (NW / 64) (l + 1) - 1
    uint32_t pf_a, pf_b, n_nodes;
    {
        uint32_t wa = 0u, wb = 0u, c;
        if constexpr (NW == 128) {
            wa = s_bf[2 * lane];
            wb = s_bf[2 * lane + 1];
            c = __popc(wa) + __popc(wb);
        } else {
            wa = lane < (uint32_t)NW ? s_bf[lane] : 0u;
            c = __popc(wa);
        }
        uint32_t incl = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t n = __shfl_up(incl, o, 64);
            if (lane >= (uint32_t)o) incl += n;
        }
        pf_a = incl - c;
        pf_b = pf_a + __popc(wa);
        // at most 4 (TW - 1) of them; the bound keeps the node
        // tables in their slots whatever the marks
        n_nodes = min((uint32_t)__shfl((int)incl, 63, 64), 4u * ((uint32_t)TW - 1u));
    }

    // ---- roots: output byte into the root's word; node entries staged in
    // LDS; statistics of the clusters complete in the tile (size classes 0-2
    // packed in one register, 11, 10 and 11 bits: a wavefront's 1024 sites may
    // all be single)
    uint32_t max_int = 0u, sq_int = 0u, hpk = 0u;
    {
        const uint32_t sbase = srow + x0;  // site index of this lane's first site
        const uint32_t bfw = s_bf[sbase >> 5];
        const uint32_t bsh = sbase & 31u;
        const uint32_t bmask = (bfw >> bsh) & M;
        // prefix of mark word sbase >> 5, held by lane (sbase >> 5) / (NW / 64)
        uint32_t pf;
        if constexpr (NW == 128) {
            const uint32_t qa = (uint32_t)__shfl((int)pf_a, (int)((sbase >> 5) >> 1), 64);
            const uint32_t qb = (uint32_t)__shfl((int)pf_b, (int)((sbase >> 5) >> 1), 64);
            pf = ((sbase >> 5) & 1u) ? qb : qa;
        } else {
            pf = (uint32_t)__shfl((int)pf_a, (int)(sbase >> 5), 64);
        }
        const uint32_t kbase = pf + __popc(bfw & ((1u << bsh) - 1u));
        const uint32_t fl = POTTS ? 0u : (uint32_t)(s_fb[ly] >> x0) & M;
        while (rootmask) {
            const uint32_t q = (uint32_t)__ffs((int)rootmask) - 1u;
            rootmask &= rootmask - 1u;
            const uint32_t root = rowbase + x0 + q;
            const uint32_t S = hi16_at(s_par, 4u * root);
            uint32_t code;
            if ((bmask >> q) & 1u) {
                const uint32_t k = kbase + __popc(bmask & ((1u << q) - 1u));
                s_node[k] = (sbase + q) | (S << 16);
                code = CB + k;
            } else {
                if constexpr (POTTS)
                    code = (uint32_t)(pv >> (4u * q)) & 0xFu;
                else
                    code = ((fl >> q) & 1u) ? 0xFFu : 0x01u;
                max_int = max(max_int, S);
                sq_int += S * S;
                const uint32_t bin = 31u - (uint32_t)__clz((int)S);
                if (bin < 3u)
                    hpk += 1u << (11u * bin - (bin >> 1));
                else
                    atomicAdd(&s_hist[bin], 1u);
                if constexpr (DENSE) {
                    if (S < kDenseBins)
                        atomicAdd(&s_dense[S], 1u);
                    else
                        atomicAdd(reinterpret_cast<unsigned long long *>(&d.dense[S]), 1ull);
                }
            }
            s_par[root] = (4u * root) | (code << 16);
        }
    }
    __syncthreads();
    if constexpr (DENSE)
        for (uint32_t i = tid; i < kDenseBins; i += NT)
            d.tdense[(size_t)tile * kDenseBins + i] = (uint16_t)s_dense[i];
    // node tables of this tile, written in node order
    for (uint32_t k = tid; k < n_nodes; k += NT) {
        const uint32_t e = s_node[k], site = e & 0xFFFFu, node = tile * kNodeSlots + k;
        d.key[node] = (ty * TW + site / TW) * L + tx * TW + site % TW;
        d.nsize[node] = e >> 16;
        par_cur[node] = node;
    }

    // ---- outputs: one byte per site (final spin or node code)
    uint32_t out[SPT / 4] = {};
    {
        uint32_t cur = rs0;
#pragma unroll
        for (int q = 0; q < SPT; ++q) {
            if ((st >> q) & 1u) cur = rowoff + 4u * (x0 + (uint32_t)q);
            const uint32_t root = lo16_at(s_par, cur);
            const uint32_t code = hi16_at(s_par, root);
            out[q >> 2] |= code << (8 * (q & 3));
        }
    }
    store_seg<SPT>(sout + (size_t)gy * L + gx0, out);
    if (d.labels) {
        uint32_t lab[SPT];
        uint32_t cur = rs0;
#pragma unroll
        for (int q = 0; q < SPT; ++q) {
            if ((st >> q) & 1u) cur = rowoff + 4u * (x0 + (uint32_t)q);
            const uint32_t root = lo16_at(s_par, cur);
            const uint32_t rsite = root / 4u - root / (4u * PS);
            const uint32_t code = (out[q >> 2] >> (8 * (q & 3))) & 0xFFu;
            lab[q] = (code >= CB && code < CB + 252u) ? (0x80000000u | (tile * kNodeSlots + code - CB))
                                                      : (ty * TW + rsite / TW) * L + tx * TW + rsite % TW;
        }
        uint4 *lp = reinterpret_cast<uint4 *>(d.labels + (size_t)gy * L + gx0);
#pragma unroll
        for (int q = 0; q < SPT / 4; ++q) lp[q] = make_uint4(lab[4 * q], lab[4 * q + 1], lab[4 * q + 2], lab[4 * q + 3]);
    }
    {
        // node index of every edge site that belongs to a node (read only
        // where the bond through the edge is set): bytes less CB
        uint8_t *eg = d.edge + (size_t)tile * 4u * TW;
        auto less = [](uint32_t w) {  // bytewise, without borrows between the bytes
            constexpr uint32_t CB4 = CB * 0x01010101u, H = 0x80808080u;
            return ((w | H) - CB4) ^ (~w & H);
        };
        if (seg == 0u) eg[0 * TW + ly] = (uint8_t)((out[0] & 0xFFu) - CB);
        if (seg == RPT - 1u) eg[1 * TW + ly] = (uint8_t)((out[SPT / 4 - 1] >> 24) - CB);
        if (ly == 0u || ly == (uint32_t)TW - 1u) {
            uint32_t e[SPT / 4];
#pragma unroll
            for (int q = 0; q < SPT / 4; ++q) e[q] = less(out[q]);
            store_seg<SPT>(eg + (ly == 0u ? 2 : 3) * TW + x0, e);
        }
    }
    // energy and magnetisation packed as (e + 2 SPT) | (m + SPT) << 16 per
    // lane: the wavefront sums stay below 2^13 and 2^12
    // (Potts: the equal pairs alone, at most 2 SPT per lane)
    uint32_t em = POTTS ? (uint32_t)e_part : (uint32_t)(e_part + 2 * SPT) | ((uint32_t)(m_part + SPT) << 16);

    // ---- workgroup reductions -> tile partial
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        em += __shfl_xor(em, o, 64);
        hpk += __shfl_xor(hpk, o, 64);
        max_int = max(max_int, (uint32_t)__shfl_xor((int)max_int, o, 64));
        sq_int += __shfl_xor(sq_int, o, 64);
        if constexpr (POTTS) {
#pragma unroll
            for (int i = 0; i < 4; ++i) cpk[i] += __shfl_xor(cpk[i], o, 64);
        }
    }
    if ((tid & 63u) == 0u) {
        s_red[tid >> 6][0] = (int32_t)em;
        s_red[tid >> 6][1] = (int32_t)hpk;
        s_red[tid >> 6][2] = (int32_t)max_int;
        s_red[tid >> 6][3] = (int32_t)sq_int;
        if constexpr (POTTS) {
#pragma unroll
            for (int i = 0; i < 4; ++i) s_red[tid >> 6][4 + i] = (int32_t)cpk[i];
        }
    }
    __syncthreads();
    if (tid == 0u) {
        int32_t e = 0, m = 0, mx = 0, sq = 0, b0 = 0, b1 = 0, b2 = 0;
        for (int w = 0; w < NWAVE; ++w) {
            const uint32_t ew = (uint32_t)s_red[w][0], hw = (uint32_t)s_red[w][1];
            if constexpr (POTTS) {
                e += (int32_t)ew;
            } else {
                e += (int32_t)(ew & 0xFFFFu) - 2 * SPT * 64;
                m += (int32_t)(ew >> 16) - SPT * 64;
            }
            b0 += (int32_t)(hw & 0x7FFu);
            b1 += (int32_t)((hw >> 11) & 0x3FFu);
            b2 += (int32_t)(hw >> 21);
            mx = max(mx, s_red[w][2]);
            sq += s_red[w][3];
        }
        int32_t n = b0 + b1 + b2;
        for (uint32_t b = 3; b < kTileBins; ++b) n += (int32_t)s_hist[b];
        int32_t *tp = d.tpart + (size_t)tile * kTilePart;
        tp[TP_E] = e;
        tp[TP_M] = m;
        tp[TP_N] = n;
        tp[TP_MAX] = mx;
        tp[TP_SQ] = sq;
        tp[TP_HIST + 0] = b0;
        tp[TP_HIST + 1] = b1;
        tp[TP_HIST + 2] = b2;
        for (uint32_t b = 3; b < kTileBins; ++b) tp[TP_HIST + b] = (int32_t)s_hist[b];
        if constexpr (POTTS) {
            for (int k = 0; k < 8; ++k) {
                int32_t c = 0;
                for (int w = 0; w < NWAVE; ++w) c += (int32_t)(((uint32_t)s_red[w][4 + k / 2] >> (16 * (k & 1))) & 0xFFFFu);
                tp[TP_CNT + k] = c;
            }
        }
        d.nk[pc][tile] = n_nodes;
        uint64_t xe = s_xe[0];
        if constexpr (TW == 64) xe |= (uint64_t)s_xe[1] << 32;
        d.xb[2u * tile] = xe;
        d.xb[2u * tile + 1u] = (uint64_t)s_xn;
    }
}

// 64-wide tiles: at most 64 VGPRs, so that the 8 workgroups per CU that the
// LDS allows (8 wavefronts per SIMD) all fit.
constexpr int kTileWavesPerEU = 8;

template <int TW, bool POTTS, bool DENSE, int TWO, int SPT>
__global__ __launch_bounds__(TW *TW / SPT, TW == 64 && SPT == 16 && !DENSE ? kTileWavesPerEU : 1) void k_tile(Dev d) {
    __shared__ TileShared<TW, POTTS, DENSE, SPT> sh;
    tile_body<TW, POTTS, DENSE, TWO, SPT>(d, tile_of_block(blockIdx.x, d.ntiles), sh);
}

// Batched launches run the same bodies over a table of replicas (map
// entries replica << kMapShift | unit index), so every replica's bits are
// those of its own plain sweep.
template <int TW, bool POTTS, int TWO, int SPT>
__global__ __launch_bounds__(TW *TW / SPT, TW == 64 && SPT == 16 ? kTileWavesPerEU : 1) void k_tile_b(const Dev *devs, const uint32_t *map) {
    __shared__ TileShared<TW, POTTS, false, SPT> sh;
    const uint32_t e = map[tile_of_block(blockIdx.x, gridDim.x)];
    tile_body<TW, POTTS, false, TWO, SPT>(devs[e >> kMapShift], e & kMapMask, sh);
}

// Tiles of every kind in one launch, for batches of several launch groups whose
// tiles do not fill the GPU group by group (kMixTiles).  256 threads suit a
// 64-wide tile with 16 sites per thread and a 32-wide one with 4.  The bodies
// take turns in one block of LDS; 80 VGPRs (at the 64 of the kernels of one
// kind the four bodies together spill 54 words, here 24).  map: the groups'
// tile maps one after another, blocks in map order, so that the slower tiles
// spread over the XCDs.
union MixShared {
    TileShared<64, false, false, 16> i64;
    TileShared<64, true, false, 16> p64;
    TileShared<32, false, false, 4> i32;
    TileShared<32, true, false, 4> p32;
    __device__ MixShared() {}
};

__global__ __launch_bounds__(256, 6) void k_tile_mix(const Dev *devs, const uint32_t *map) {
    __shared__ __align__(16) unsigned char mem[sizeof(MixShared)];
    MixShared &sh = *reinterpret_cast<MixShared *>(mem);
    const uint32_t e = map[blockIdx.x], tile = e & kMapMask;
    const Dev &d = devs[e >> kMapShift];
    if (d.tw == 64u) {
        if (d.q)
            tile_body<64, true, false, 2, 16>(d, tile, sh.p64);
        else
            tile_body<64, false, false, 2, 16>(d, tile, sh.i64);
    } else {
        if (d.q)
            tile_body<32, true, false, 2, 4>(d, tile, sh.p32);
        else
            tile_body<32, false, false, 2, 4>(d, tile, sh.i32);
    }
}

// =====================================================================
// k_union: bonds that leave a tile through its E or N edge join the nodes
// on both sides (Sec. 2.3, global part).  One wavefront per tile.
// =====================================================================
// The global union-find links nodes by index (sw_uf.h); the cluster's
// smallest site is gathered separately (k_flatten takes the minimum of the
// nodes' keys into the root's key), so finds never read keys.
template <int TW, class Order>
__device__ __forceinline__ void union_body(const Dev &d, const uint32_t tile, const uint32_t dir) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t ntx = d.ntx, tx = tile % ntx, ty = tile / ntx;
    // edges to a tile of the same kUG x kUG group were joined by k_ulocal
    const bool glob = dir == 0u ? ((tx % kUG) == kUG - 1u || tx + 1u == ntx)
                                : ((ty % kUG) == kUG - 1u || ty + 1u == ntx);
    if (!glob) return;
    static_assert(TW <= 64, "one lane per edge position");
    const uint32_t nb = dir == 0u ? ty * ntx + (tx + 1u == ntx ? 0u : tx + 1u)
                                  : (ty + 1u == ntx ? 0u : ty + 1u) * ntx + tx;
    const uint8_t *eg = d.edge + (size_t)tile * 4u * TW;
    const uint8_t *egb = d.edge + (size_t)nb * 4u * TW;
    // one lane per edge position; the bond bits and both sides' node bytes are
    // all loaded before any of them is waited on
    const bool in = lane < (uint32_t)TW;
    const uint32_t i = in ? lane : 0u;
    const uint32_t an = dir == 0u ? eg[1 * TW + i] : eg[3 * TW + i];
    const uint32_t bn = dir == 0u ? egb[0 * TW + i] : egb[2 * TW + i];
    const uint64_t bits = d.xb[2u * tile + dir];
    uint32_t *par = d.parent;
    const bool has = in && ((bits >> i) & 1u);
    const uint32_t a = tile * kNodeSlots + an, b = nb * kNodeSlots + bn;
    // every union starts from the two nodes' parents (their group roots, or
    // nearer the root); a bond whose parents equal those of the previous
    // bond along the edge adds nothing, so only the first of such a run
    // links (fewer lanes compete for the same roots' compare-and-swap)
    uint32_t ra = 0u, rb = 0u;
    if (has) {
        ra = g_load(&par[a]);
        rb = g_load(&par[b]);
    }
    const uint64_t below = __ballot(has) & ((1ull << lane) - 1ull);
    const int prev = below ? 63 - __clzll((long long)below) : (int)lane;
    const uint32_t pra = (uint32_t)__shfl((int)ra, prev, 64), prb = (uint32_t)__shfl((int)rb, prev, 64);
    const bool dup = below != 0ull && pra == ra && prb == rb;
    if (has && !dup) g_union<Order>(par, ra, rb);
}

// =====================================================================
// k_ulocal: the bonds between tiles of one kUG x kUG group join their nodes
// in LDS (local index = tile-in-group * kNodeSlots + node, which orders
// nodes as their global indices do, so the smaller index is the root in
// both); every node then points at its group-local root in global memory,
// and k_union only has the edges between groups left.
// =====================================================================
template <int TW>
__device__ __forceinline__ void ulocal_body(const Dev &d, const uint32_t ugroup, uint32_t *s_p) {
    constexpr uint32_t NG = kUG * kUG;
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t pc = (uint32_t)(*d.tdev & 1u);
    const uint32_t ntx = d.ntx, ngx = (ntx + kUG - 1u) / kUG;
    const uint32_t gx = ugroup % ngx, gy = ugroup / ngx;
    auto tile_of = [&](uint32_t t) { return (gy * kUG + t / kUG) * ntx + gx * kUG + t % kUG; };
    auto valid = [&](uint32_t t) { return gx * kUG + t % kUG < ntx && gy * kUG + t / kUG < ntx; };
    // tile-edges inside the group: E edges (lx < kUG-1), then N edges (ly <
    // kUG-1), one position per thread and iteration; all of a thread's loads
    // are issued first (they do not depend on the sweep parity), then the
    // node counts, then the unions
    constexpr uint32_t NE = (kUG - 1u) * kUG;
    constexpr uint32_t NIT = 2u * NE * TW / 256u;
    static_assert(2u * NE * TW % 256u == 0u, "edge positions must fill the workgroup");
    uint32_t ua[NIT], ub[NIT];
    bool uh[NIT];
#pragma unroll
    for (uint32_t it = 0; it < NIT; ++it) {
        const uint32_t f = tid + 256u * it, e = f / TW, i = f % TW;
        const bool isn = e >= NE;
        const uint32_t e2 = isn ? e - NE : e;
        const uint32_t lx = isn ? e2 % kUG : e2 % (kUG - 1u), ly = isn ? e2 / kUG : e2 / (kUG - 1u);
        const uint32_t ta = ly * kUG + lx, tb = isn ? ta + kUG : ta + 1u;
        const bool ok = valid(ta) && valid(tb);
        const uint32_t A = ok ? tile_of(ta) : 0u, B = ok ? tile_of(tb) : 0u;  // tile 0: read and ignored
        const uint8_t *ea = d.edge + (size_t)A * 4u * TW, *eb = d.edge + (size_t)B * 4u * TW;
        uh[it] = ok && ((d.xb[2u * A + (isn ? 1u : 0u)] >> i) & 1u);
        ua[it] = ta * kNodeSlots + (isn ? ea[3 * TW + i] : ea[1 * TW + i]);
        ub[it] = tb * kNodeSlots + (isn ? eb[2 * TW + i] : eb[0 * TW + i]);
    }
    // 16 threads per tile of the group (thread tid: tile tid / 16, node
    // slots tid % 16 + 16 m), so that the slots of every tile's nodes, and
    // only those, are set up and later resolved in about nk / 16 steps
    static_assert(NG * 16u == 256u, "16 threads per tile");
    const uint32_t mt = tid >> 4, mk = tid & 15u;
    const uint32_t nkt = valid(mt) ? min(d.nk[pc][tile_of(mt)], 252u) : 0u;
    for (uint32_t k = mk; k < nkt; k += 16u) s_p[mt * kNodeSlots + k] = mt * kNodeSlots + k;
    __syncthreads();
#pragma unroll
    for (uint32_t it = 0; it < NIT; ++it) {
        const uint32_t i = (tid + 256u * it) % TW, a = ua[it], b = ub[it];
        const bool has = uh[it];
        // a run of bonds along the edge between the same two nodes needs one union
        const uint32_t pa = __shfl_up(a, 1, 64), pb = __shfl_up(b, 1, 64);
        const int ph = __shfl_up((int)has, 1, 64);
        const bool dup = i > 0u && lane > 0u && ph && pa == a && pb == b;
        if (has && !dup) lds_union(s_p, a, b);
    }
    __syncthreads();

    uint32_t *par = d.parent;
    const uint32_t gt = tile_of(mt);
    for (uint32_t k = mk; k < nkt; k += 16u) {
        const uint32_t li = mt * kNodeSlots + k;
        const uint32_t r = lds_find(s_p, li);
        if (r != li) par[gt * kNodeSlots + k] = tile_of(r / kNodeSlots) * kNodeSlots + r % kNodeSlots;
    }
}

template <int TW>
__global__ __launch_bounds__(256) void k_ulocal(Dev d) {
    __shared__ uint32_t s_p[kUG * kUG * kNodeSlots];
    ulocal_body<TW>(d, blockIdx.x, s_p);
}

__global__ __launch_bounds__(256) void k_ulocal_b(const Dev *devs, const uint32_t *map) {
    __shared__ uint32_t s_p[kUG * kUG * kNodeSlots];
    const uint32_t e = map[blockIdx.x];
    const Dev &d = devs[e >> kMapShift];
    if (d.tw == 64u)
        ulocal_body<64>(d, e & kMapMask, s_p);
    else
        ulocal_body<32>(d, e & kMapMask, s_p);
}

// One wavefront per (tile, direction): wave w of the launch takes tile w / 2
// and its E (w even) or N (w odd) edge.
// Plain lattices launch only the edges between kUG x kUG groups: wave w <
// ngx * ntx takes the E edge of the last tile column of a group in tile row
// w / ngx; the next ngx * ntx waves the N edges of the groups' last tile rows.
template <int TW, class Order>
__global__ __launch_bounds__(256) void k_union(Dev d) {
    const uint32_t ntx = d.ntx, ngx = (ntx + kUG - 1u) / kUG, nE = ngx * ntx;
    uint32_t w = blockIdx.x * 4u + (threadIdx.x >> 6);
    if (w < nE) {
        const uint32_t ty = w / ngx, tx = min((w % ngx) * kUG + kUG - 1u, ntx - 1u);
        union_body<TW, Order>(d, ty * ntx + tx, 0u);
    } else if ((w -= nE) < nE) {
        const uint32_t tx = w % ntx, ty = min((w / ntx) * kUG + kUG - 1u, ntx - 1u);
        union_body<TW, Order>(d, ty * ntx + tx, 1u);
    }
}

// One wavefront per map entry: the first nE of the n entries are tiles whose E
// edge is a group edge, the rest tiles whose N edge is.
__device__ __forceinline__ void union_b_body(const Dev *devs, const uint32_t *map, uint32_t n, uint32_t nE, uint32_t w) {
    if (w >= n) return;
    const uint32_t e = map[w], dir = w < nE ? 0u : 1u;
    const Dev &d = devs[e >> kMapShift];
    if (d.tw == 64u)
        union_body<64, ByIndex>(d, e & kMapMask, dir);
    else
        union_body<32, ByIndex>(d, e & kMapMask, dir);
}

__global__ __launch_bounds__(256) void k_union_b(const Dev *devs, const uint32_t *map, uint32_t n, uint32_t nE) {
    union_b_body(devs, map, n, nE, blockIdx.x * 4u + (threadIdx.x >> 6));
}

// =====================================================================
// k_flatten: every node points at its root; node sizes are summed into the
// root's size and node keys (smallest sites) reduced to their minimum in the
// root's key, first per workgroup in an LDS hash, then with one global
// atomic of each kind per (workgroup, root).  The structure is final here,
// so finds only read and the only stores are roots.
// =====================================================================
constexpr int kHashSlots = 2048;

// Node count of tile i in the sweep of parity pc: both parities are loaded,
// so that the loads need not wait for the sweep index.
__device__ __forceinline__ uint32_t nk_either(const Dev &d, uint32_t pc, uint32_t i) {
    const uint32_t a = d.nk[0][i], b = d.nk[1][i];
    return pc ? b : a;
}

__device__ __forceinline__ void hash_add(uint32_t *hk, uint32_t *hv, uint32_t *hm, uint32_t root, uint32_t size,
                                         uint32_t key, const Dev &d) {
    uint32_t h = (root * 2654435761u) >> 21;  // 11 bits
    for (int probe = 0; probe < 64; ++probe) {
        const uint32_t cur = lds_load(&hk[h]);
        bool mine = cur == root;
        if (cur == kEmpty) {
            const uint32_t old = atomicCAS(&hk[h], kEmpty, root);
            mine = old == kEmpty || old == root;
        }
        if (mine) {
            atomicAdd(&hv[h], size);
            atomicMin(&hm[h], key);
            return;
        }
        h = (h + 1u) & (kHashSlots - 1);
    }
    atomicAdd(&d.nsize[root], size);
    if (key < g_load(&d.key[root])) atomicMin(&d.key[root], key);
}

// FT tiles per workgroup (16: the tile groups): a root gets one atomic of
// each kind per workgroup that holds some of its nodes, so a cluster that
// spans the lattice receives ntiles / FT of them, one after the other.  A key
// minimum is skipped when a plain read already shows a key no larger (keys
// only decrease).
template <uint32_t FT>
__device__ __forceinline__ void flatten_body(const Dev &d, const uint32_t group) {
    __shared__ uint32_t hk[kHashSlots];
    __shared__ uint32_t hv[kHashSlots];
    __shared__ uint32_t hm[kHashSlots];
    for (uint32_t i = threadIdx.x; i < (uint32_t)kHashSlots; i += 256u) {
        hk[i] = kEmpty;
        hv[i] = 0u;
        hm[i] = kEmpty;
    }
    __syncthreads();
    const uint32_t pc = (uint32_t)(*d.tdev & 1u);
    uint32_t *par = d.parent;
    const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6;
    const uint32_t g0 = group * FT;
    static_assert(FT % 16u == 0u, "four tiles per wavefront and quad");
    // wavefront wv owns tiles g0 + wv + 4q, taken four at a time (a quad);
    // the nodes of a quad are numbered one after the other (about 80 per
    // tile at beta_c, so mostly one batch), and each lane chases the roots
    // of up to 8 nodes at once, one level per round, so their loads overlap
    for (uint32_t quad = 0; quad < FT / 16u; ++quad) {
    uint32_t nkq[4];
#pragma unroll
    for (uint32_t q = 0; q < 4u; ++q) {
        const uint32_t tile = g0 + wv + 4u * (4u * quad + q);
        const uint32_t v = nk_either(d, pc, min(tile, d.ntiles - 1u));  // issued unconditionally
        nkq[q] = tile < d.ntiles ? min(v, 252u) : 0u;
    }
    const uint32_t pre1 = nkq[0], pre2 = pre1 + nkq[1], pre3 = pre2 + nkq[2], tot = pre3 + nkq[3];
    constexpr uint32_t kChase = 8;
#pragma unroll
    for (uint32_t m0 = 0; m0 < 4u * 252u / 64u + 1u; m0 += kChase) {
        if (64u * m0 >= tot) break;
        uint32_t nd[kChase], r[kChase];
#pragma unroll
        for (uint32_t j = 0; j < kChase; ++j) {
            const uint32_t i = lane + 64u * (m0 + j);
            const uint32_t q = (uint32_t)(i >= pre1) + (uint32_t)(i >= pre2) + (uint32_t)(i >= pre3);
            const uint32_t base = q == 0u ? 0u : q == 1u ? pre1 : q == 2u ? pre2 : pre3;
            nd[j] = i < tot ? (g0 + wv + 4u * (4u * quad + q)) * kNodeSlots + (i - base) : kEmpty;
            r[j] = nd[j];
        }
        bool more = true;
        while (more) {
            // all loads first (an empty slot reads node 0 and ignores it)
            uint32_t p[kChase];
#pragma unroll
            for (uint32_t j = 0; j < kChase; ++j)
                p[j] = __hip_atomic_load(&par[r[j] == kEmpty ? 0u : r[j]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            more = false;
#pragma unroll
            for (uint32_t j = 0; j < kChase; ++j) {
                const uint32_t q = r[j] == kEmpty ? kEmpty : p[j];
                more |= q != r[j];
                r[j] = q;
            }
        }
#pragma unroll
        for (uint32_t j = 0; j < kChase; ++j) {
            if (nd[j] == kEmpty || r[j] == nd[j]) continue;
            g_store(&par[nd[j]], r[j]);
            hash_add(hk, hv, hm, r[j], d.nsize[nd[j]], d.key[nd[j]], d);
        }
    }
    }
    __syncthreads();
    // each thread flushes kHashSlots / 256 slots; the current keys of all its
    // roots are read before any atomic so that those loads overlap
    constexpr uint32_t kPer = (uint32_t)kHashSlots / 256u;
    uint32_t fk[kPer], fm[kPer];
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) fk[j] = hk[threadIdx.x + 256u * j];
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) fm[j] = fk[j] != kEmpty ? g_load(&d.key[fk[j]]) : 0u;
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
        if (fk[j] == kEmpty) continue;
        const uint32_t i = threadIdx.x + 256u * j;
        atomicAdd(&d.nsize[fk[j]], hv[i]);
        if (hm[i] < fm[j]) atomicMin(&d.key[fk[j]], hm[i]);
    }
}

template <uint32_t FT>
__global__ __launch_bounds__(256) void k_flatten(Dev d) { flatten_body<FT>(d, blockIdx.x); }

__global__ __launch_bounds__(256) void k_flatten_b(const Dev *devs, const uint32_t *map) {
    const uint32_t e = map[blockIdx.x];
    flatten_body<kGroupTiles>(devs[e >> kMapShift], e & kMapMask);
}

// Canonical labels of sites of cross-tile clusters (only with SW_FLAG_LABELS).
__global__ __launch_bounds__(256) void k_relabel(Dev d) {
    const size_t n = (size_t)d.L * d.L;
    const uint32_t *par = d.parent;
    const uint32_t nnodes = d.ntiles * kNodeSlots;
    for (size_t i = blockIdx.x * (size_t)256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const uint32_t l = d.labels[i];
        if (l & 0x80000000u) {
            uint32_t node = l & 0x7FFFFFFFu;
            node = node < nnodes ? node : 0u;
            uint32_t r = par[node];
            r = r < nnodes ? r : 0u;
            d.labels[i] = d.key[r];
        }
    }
}

// =====================================================================
// k_roots: new spin of every cross-tile cluster (Sec. 2.4) and the cluster
// statistics of the workgroup's tiles -> group partial.
// =====================================================================
// RB: nodes a lane takes at once (see below).  AG: the group partial is
// written with agent-scope stores, for a fold in the same launch.
// DENSE: the exact size histogram.  Sizes below kDenseBins -- nearly all --
// are counted in LDS together with the tiles' own counts, so a histogram
// word takes one device-scope atomic per group of tiles: one atomic per
// cluster instead serialised on the few words of the small sizes (about 22 ns
// each: k_tile 1196 us and k_roots 90 us at 1024^2, beta_c, against 21 and 14
// without the histogram).  Five sweeps of 1024^2 with labels and histogram
// read back: 6.85 -> 1.44 ms.
template <uint32_t RB, bool AG = false, bool DENSE = false>
__device__ __forceinline__ void roots_body(const Dev &d, const uint32_t group) {
    __shared__ uint32_t s_hist[33];
    __shared__ uint32_t s_cnt[kMaxQ];  // Potts value populations of the group's tiles
    __shared__ uint64_t s_red[4][5];
    __shared__ uint32_t s_dense[DENSE ? kDenseBins : 1];
    static_assert(kDenseBins == 256u, "one size per thread");
    if constexpr (DENSE) s_dense[threadIdx.x] = 0u;
    if (threadIdx.x < 33u) s_hist[threadIdx.x] = 0u;
    if (threadIdx.x < (uint32_t)kMaxQ) s_cnt[threadIdx.x] = 0u;
    const uint64_t tsw = *d.tdev;
    const uint32_t t = (uint32_t)tsw, pc = (uint32_t)(tsw & 1u);
    const uint32_t *par = d.parent;
    const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6;
    const uint32_t g0 = group * (uint32_t)kGroupTiles;
    uint64_t n = 0, mx = 0, sq = 0;
    int64_t e = 0, m = 0;
    // the nodes of the wavefront's four tiles g0 + wv + 4q, one after the other
    uint32_t nkq[4];
#pragma unroll
    for (uint32_t q = 0; q < 4u; ++q) {
        const uint32_t tile = g0 + wv + 4u * q;
        const uint32_t v = nk_either(d, pc, min(tile, d.ntiles - 1u));
        nkq[q] = tile < d.ntiles ? min(v, 252u) : 0u;
    }
    const uint32_t pre1 = nkq[0], pre2 = pre1 + nkq[1], pre3 = pre2 + nkq[2], tot = pre3 + nkq[3];
    int32_t tw[4];  // word `lane` of their partials, used at the end
#pragma unroll
    for (uint32_t q = 0; q < 4u; ++q) {
        const uint32_t tile = g0 + wv + 4u * q;
        tw[q] = tile < d.ntiles && lane < (uint32_t)kTilePart ? d.tpart[(size_t)tile * kTilePart + lane] : 0;
    }
    __syncthreads();  // s_hist and s_cnt cleared
    // every node (flattened: its parent is its root) stores its cluster's
    // new spin, drawn from the cluster's smallest site (the root's key).  A
    // lane takes up to RB nodes at once and issues all their parent loads,
    // then all their key and size loads, so that the wavefront waits on two
    // rounds of loads per batch rather than on two for every node: launches
    // of a few workgroups per CU wait on those rounds; full ones hide them
    // behind other wavefronts and run faster with RB = 1 (fewer registers).
    constexpr uint32_t kRootBatch = RB;
    for (uint32_t m0 = 0; 64u * m0 < tot; m0 += kRootBatch) {
        uint32_t nd[kRootBatch], rt[kRootBatch], rk[kRootBatch], sz[kRootBatch];
#pragma unroll
        for (uint32_t j = 0; j < kRootBatch; ++j) {
            const uint32_t i = lane + 64u * (m0 + j);
            const uint32_t q = (uint32_t)(i >= pre1) + (uint32_t)(i >= pre2) + (uint32_t)(i >= pre3);
            const uint32_t base = q == 0u ? 0u : q == 1u ? pre1 : q == 2u ? pre2 : pre3;
            nd[j] = i < tot ? (g0 + wv + 4u * q) * kNodeSlots + (i - base) : kEmpty;
        }
#pragma unroll
        for (uint32_t j = 0; j < kRootBatch; ++j) rt[j] = nd[j] != kEmpty ? par[nd[j]] : 0u;
#pragma unroll
        for (uint32_t j = 0; j < kRootBatch; ++j) {
            rk[j] = nd[j] != kEmpty ? d.key[rt[j]] : 0u;
            sz[j] = nd[j] != kEmpty && rt[j] == nd[j] ? d.nsize[nd[j]] : 0u;
        }
#pragma unroll
        for (uint32_t j = 0; j < kRootBatch; ++j) {
            if (64u * (m0 + j) >= tot) break;  // wavefront-uniform
            if (nd[j] == kEmpty) continue;
            d.rspin[nd[j]] = d.q ? potts_spin(rk[j], t, d.q, d.seed_lo, d.seed_hi)
                                 : cluster_spin(rk[j], t, d.seed_lo, d.seed_hi);
            if (rt[j] == nd[j]) {
                const uint32_t S = sz[j];
                ++n;
                mx = max(mx, (uint64_t)S);
                sq += (uint64_t)S * S;
                atomicAdd(&s_hist[31 - __clz((int)max(S, 1u))], 1u);
                if constexpr (DENSE) {
                    if (S < kDenseBins)
                        atomicAdd(&s_dense[S], 1u);
                    else
                        atomicAdd(reinterpret_cast<unsigned long long *>(&d.dense[S]), 1ull);
                }
            }
        }
    }
    uint32_t dn = 0u;  // interior clusters of threadIdx.x sites in the group's tiles
    if constexpr (DENSE) {
#pragma unroll
        for (uint32_t i = 0; i < (uint32_t)kGroupTiles; ++i)
            if (g0 + i < d.ntiles) dn += d.tdense[(size_t)(g0 + i) * kDenseBins + threadIdx.x];
    }
    // the tile partials, one word per lane
    if (lane < (uint32_t)TP_CNT + (uint32_t)kMaxQ) {
        int64_t v = 0;
#pragma unroll
        for (uint32_t q = 0; q < 4u; ++q) v = lane == (uint32_t)TP_MAX ? max(v, (int64_t)tw[q]) : v + tw[q];
        if (lane == (uint32_t)TP_E)
            e += v;
        else if (lane == (uint32_t)TP_M)
            m += v;
        else if (lane == (uint32_t)TP_N)
            n += (uint64_t)v;
        else if (lane == (uint32_t)TP_MAX)
            mx = max(mx, (uint64_t)v);
        else if (lane == (uint32_t)TP_SQ)
            sq += (uint64_t)v;
        else if (lane < (uint32_t)TP_CNT)
            atomicAdd(&s_hist[lane - (uint32_t)TP_HIST], (uint32_t)v);
        else if (d.q)
            atomicAdd(&s_cnt[lane - (uint32_t)TP_CNT], (uint32_t)v);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        n += __shfl_xor(n, o, 64);
        mx = max(mx, (uint64_t)__shfl_xor((unsigned long long)mx, o, 64));
        sq += __shfl_xor(sq, o, 64);
        e += __shfl_xor(e, o, 64);
        m += __shfl_xor(m, o, 64);
    }
    if (lane == 0u) {
        s_red[wv][0] = n;
        s_red[wv][1] = mx;
        s_red[wv][2] = sq;
        s_red[wv][3] = (uint64_t)e;
        s_red[wv][4] = (uint64_t)m;
    }
    __syncthreads();
    if constexpr (DENSE) {
        dn += s_dense[threadIdx.x];
        if (dn) atomicAdd(reinterpret_cast<unsigned long long *>(&d.dense[threadIdx.x]), (unsigned long long)dn);
    }
    uint64_t *gp = d.gpart + (size_t)group * kGroupPart;
    auto put = [&](int f, uint64_t v) {
        if constexpr (AG)
            __hip_atomic_store(&gp[f], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else
            gp[f] = v;
    };
    if (threadIdx.x == 0u) {
        uint64_t a0 = 0, a1 = 0, a2 = 0, a3 = 0, a4 = 0;
        for (int w = 0; w < 4; ++w) {
            a0 += s_red[w][0];
            a1 = max(a1, s_red[w][1]);
            a2 += s_red[w][2];
            a3 += s_red[w][3];
            a4 += s_red[w][4];
        }
        put(GP_N, a0);
        put(GP_MAX, a1);
        put(GP_SQ, a2);
        put(GP_E, a3);
        put(GP_M, a4);
    }
    if (threadIdx.x < 33u) put(GP_HIST + (int)threadIdx.x, s_hist[threadIdx.x]);
    if (threadIdx.x < (uint32_t)kMaxQ) put(GP_CNT + (int)threadIdx.x, s_cnt[threadIdx.x]);
}


// =====================================================================
// k_record: fold group partials (mode 0, end of a sweep) or tile partials
// (mode 1, end of k_resolve) into the record ring; the last workgroup to
// finish writes the record and clears the accumulator.
// =====================================================================
// Folds partials [begin, end) into the workgroup's LDS accumulator.  Group
// partials (mode 0): thread t sums field t % 64 over every fourth partial,
// so each accumulator word takes four LDS atomics.  Tile partials (mode 1,
// energy and magnetisation only): per-thread sums, reduced per wavefront.
constexpr uint32_t kRecordGroups = 64;   // group partials per k_record workgroup
constexpr uint32_t kRecordTiles = 2048;  // tile partials per k_record workgroup

// AG: the group partials were written in the same launch (agent-scope
// stores), so they are read with agent-scope loads.
template <bool AG = false>
__device__ __forceinline__ void record_fold(const Dev &d, uint32_t begin, uint32_t end, int mode, uint64_t *s_acc) {
    const uint32_t tid = threadIdx.x;
    unsigned long long *a = reinterpret_cast<unsigned long long *>(s_acc);
    if (mode != 1) {
        const uint32_t f = tid & 63u, sub = tid >> 6;
        if (f < (uint32_t)GP_END) {
            // four partials per round, their loads issued together (0 is
            // the identity of both the sums and the maximum)
            uint64_t v = 0;
            for (uint32_t item = begin + sub; item < end; item += 16u) {
                uint64_t x[4];
#pragma unroll
                for (uint32_t u = 0; u < 4u; ++u) {
                    const uint32_t it = item + 4u * u;
                    const uint64_t *src = &d.gpart[(size_t)min(it, end - 1u) * kGroupPart + f];
                    const uint64_t y = AG ? __hip_atomic_load(src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *src;
                    x[u] = it < end ? y : 0u;
                }
#pragma unroll
                for (uint32_t u = 0; u < 4u; ++u) v = f == (uint32_t)GP_MAX ? max(v, x[u]) : v + x[u];
            }
            if (f == (uint32_t)GP_MAX)
                atomicMax(&a[f], (unsigned long long)v);
            else if (v)
                atomicAdd(&a[f], (unsigned long long)v);
        }
    } else {
        int64_t e = 0, m = 0;
        uint32_t c[kMaxQ] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
        for (uint32_t item = begin + tid; item < end; item += 256u) {
            const int32_t *tp = d.tpart + (size_t)item * kTilePart;
            e += tp[TP_E];
            m += tp[TP_M];
            if (d.q)
                for (int k = 0; k < kMaxQ; ++k) c[k] += (uint32_t)tp[TP_CNT + k];
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            e += __shfl_xor(e, o, 64);
            m += __shfl_xor(m, o, 64);
        }
        if ((tid & 63u) == 0u) {
            atomicAdd(&a[GP_E], (unsigned long long)e);
            atomicAdd(&a[GP_M], (unsigned long long)m);
        }
        if (d.q)
            for (int k = 0; k < kMaxQ; ++k)
                if (c[k]) atomicAdd(&a[GP_CNT + k], (unsigned long long)c[k]);
    }
}

// Writes the totals in s_acc.  Mode 0 (end of a tile-pipeline sweep): the
// record of sweep t = *tdev gets the cluster statistics and t advances; the
// energy and magnetisation are those of the configuration sweep t-1 left
// (measured by this sweep's tile kernel), written into record t-1.  Mode 1
// (end of k_resolve): only that energy and magnetisation.  Mode 2 (end of a
// label-equivalence sweep): every field of record t, and t advances.
__device__ __forceinline__ void record_write(const Dev &d, const uint64_t *s_acc, int mode) {
    const uint32_t tid = threadIdx.x;
    const uint64_t tsw = *d.tdev;
    if (mode != 1) {
        sw_obs *rec = &d.ring[tsw % d.ring_cap];
        if (tid == 0u) {
            rec->sweep = tsw;
            rec->n_clusters = s_acc[GP_N];
            rec->max_cluster = s_acc[GP_MAX];
            rec->sum_sq_sizes = s_acc[GP_SQ];
        }
        if (tid < 33u) rec->hist_log2[tid] = s_acc[GP_HIST + tid];
    }
    const bool own = mode == 2;
    if (tid == 0u && (own || tsw >= 1u)) {
        sw_obs *rec = &d.ring[(own ? tsw : tsw - 1u) % d.ring_cap];
        const int64_t e = (int64_t)s_acc[GP_E];
        rec->e_sum = e;
        rec->energy = -d.J * (double)e;
        int64_t m = (int64_t)s_acc[GP_M];
        if (d.q) {  // Potts: population of the most populated value
            m = 0;
            for (uint32_t k = 0; k < d.q; ++k) m = max(m, (int64_t)s_acc[GP_CNT + k]);
        }
        rec->m_sum = m;
    }
    __syncthreads();  // every thread has read the sweep index
    if (tid == 0u && mode != 1) *d.tdev = tsw + 1u;  // (the kernel's end publishes it)
}

__global__ __launch_bounds__(256) void k_record(Dev d, uint32_t nitems, int mode) {
    __shared__ uint64_t s_acc[GP_END];
    __shared__ int s_last;
    const uint32_t tid = threadIdx.x;
    if (tid < (uint32_t)GP_END) s_acc[tid] = 0u;
    __syncthreads();
    const uint32_t per = mode != 1 ? kRecordGroups : kRecordTiles;
    const uint32_t begin = blockIdx.x * per;
    record_fold(d, begin, min(begin + per, nitems), mode, s_acc);
    __syncthreads();
    unsigned long long *acc = reinterpret_cast<unsigned long long *>(d.acc);
    if (tid < (uint32_t)GP_END && s_acc[tid] != 0u) {
        if (tid == (uint32_t)GP_MAX)
            atomicMax(&acc[tid], (unsigned long long)s_acc[tid]);
        else
            atomicAdd(&acc[tid], (unsigned long long)s_acc[tid]);
    }
    // device-scope atomics are performed where every XCD sees them: once each
    // wavefront has seen its own complete, the count may go up, and the last
    // workgroup reads the totals with device-scope loads (no cache fences)
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0u) {
        const unsigned long long old = atomicAdd(&acc[ACC_COUNT], 1ull);
        s_last = (old == (unsigned long long)gridDim.x - 1ull) ? 1 : 0;
    }
    __syncthreads();
    if (!s_last) return;
    // the last workgroup: take the totals (one field per thread) and clear
    // the accumulator for the next fold
    if (tid < (uint32_t)GP_END) {
        s_acc[tid] = __hip_atomic_load(&acc[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&acc[tid], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (tid == (uint32_t)GP_END)
        __hip_atomic_store(&acc[ACC_COUNT], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    record_write(d, s_acc, mode);
}

// Batched record of the tile partials at the end of a resolve (mode 1): one
// workgroup per replica folds all of that replica's partials itself, so no
// cross-workgroup accumulator is needed (the group partials of a sweep are
// folded by k_roots_b).
__global__ __launch_bounds__(256) void k_record_b(const Dev *devs, const uint32_t *rmap, int mode) {
    __shared__ uint64_t s_acc[GP_END];
    const Dev &d = devs[rmap[blockIdx.x]];
    const uint32_t tid = threadIdx.x;
    if (tid < (uint32_t)GP_END) s_acc[tid] = 0u;
    __syncthreads();
    record_fold(d, 0u, mode != 1 ? d.ngroups : d.ntiles, mode, s_acc);
    __syncthreads();
    record_write(d, s_acc, mode);
}

// k_roots, and the record folded into the same launch: the last workgroup of
// a lattice to write its group partial folds them all and writes the record
// (one launch less per sweep).  The partials go out as agent-scope stores
// and every wavefront waits for its own to complete before its workgroup
// counts itself in, so the last one reads them all with agent-scope loads
// (no cache fences).  Used where a lattice has few groups (the fold is one
// workgroup's work) and for every replica of a batch.
template <uint32_t RB, bool DENSE = false>
__device__ __forceinline__ void roots_fold_body(const Dev &d, const uint32_t group) {
    __shared__ uint64_t s_acc[GP_END];
    __shared__ int s_last;
    roots_body<RB, true, DENSE>(d, group);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    unsigned long long *acc = reinterpret_cast<unsigned long long *>(d.acc);
    if (threadIdx.x == 0u) {
        const unsigned long long old = atomicAdd(&acc[ACC_COUNT], 1ull);
        s_last = old == (unsigned long long)d.ngroups - 1ull ? 1 : 0;
    }
    if (threadIdx.x < (uint32_t)GP_END) s_acc[threadIdx.x] = 0u;
    __syncthreads();
    if (!s_last) return;
    if (threadIdx.x == 0u) __hip_atomic_store(&acc[ACC_COUNT], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    record_fold<true>(d, 0u, d.ngroups, 0, s_acc);
    __syncthreads();
    record_write(d, s_acc, 0);
}

// Plain lattices: up to kRootsFold groups the record is folded by k_roots;
// from kRootsWide groups (32768 tiles) on, a lane takes one node at a time.
constexpr uint32_t kRootsFold = 64;
constexpr uint32_t kRootsWide = 2048;

template <uint32_t RB, bool DENSE = false>
__global__ __launch_bounds__(256) void k_roots(Dev d) { roots_body<RB, false, DENSE>(d, blockIdx.x); }

template <bool DENSE>
__global__ __launch_bounds__(256) void k_roots_fold(Dev d) { roots_fold_body<4, DENSE>(d, blockIdx.x); }

__global__ __launch_bounds__(256) void k_roots_b(const Dev *devs, const uint32_t *map) {
    const uint32_t e = map[blockIdx.x];
    roots_fold_body<4>(devs[e >> kMapShift], e & kMapMask);
}

// =====================================================================
// k_merge: the whole cross-tile part of a sweep (Sec. 2.3-2.5) of a lattice
// of few tiles in one launch: the work of k_ulocal, k_union, k_flatten,
// k_roots and k_record, same results.  On such lattices each of those is a few
// chains of dependent loads on an idle GPU (42 of 63 us a sweep at 512^2), so
// one workgroup of 1024 threads per kUG x kUG group of tiles takes them
// together, in LDS:
//   level 1  unions across the tile edges inside the group; sizes and smallest
//            sites at the roots; a cluster with no bond out of the group is
//            complete and draws its spin
//   level 2  the other clusters, numbered per group (ref_slots slots; each
//            holds a bond on the group's perimeter, of at most 1024 sites): the
//            last workgroup of the lattice to count itself in unites them
//            across the group edges, draws their spins and writes the record
// A lattice of one group (at most 16 tiles) has its periodic wrap inside
// level 1 and no level 2.  Nodes keep a reference (nref) that the next
// k_tile or k_resolve follows, so no workgroup has to visit them again.
// What goes from the groups to the last workgroup is written and read with
// agent-scope accesses, completed before the count (no cache fences).
// =====================================================================
constexpr uint32_t kMergeThreads = 1024;
constexpr uint32_t kMergeWaves = kMergeThreads / 64;
constexpr uint32_t kNoRef = 0xFFFFu;
static_assert(kUG * kUG == kMergeWaves, "one wavefront per tile of a group");

__device__ __forceinline__ uint32_t new_value(const Dev &d, uint32_t key, uint32_t t) {
    return d.q ? (uint32_t)potts_spin(key, t, d.q, d.seed_lo, d.seed_hi)
               : (uint32_t)(cluster_spin(key, t, d.seed_lo, d.seed_hi) > 0);
}


// Cluster statistics of a workgroup: per-thread sums, then LDS totals.
struct Stats {
    uint32_t n = 0, mx = 0;
    uint64_t sq = 0;
    __device__ __forceinline__ void add(uint32_t S, unsigned long long *acc) {
        ++n;
        mx = max(mx, S);
        sq += (uint64_t)S * S;
        atomicAdd(&acc[GP_HIST + 31 - __clz((int)max(S, 1u))], 1ull);
    }
    __device__ __forceinline__ void flush(unsigned long long *acc) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            n += __shfl_xor(n, o, 64);
            mx = max(mx, (uint32_t)__shfl_xor((int)mx, o, 64));
            sq += __shfl_xor(sq, o, 64);
        }
        if ((threadIdx.x & 63u) == 0u && n != 0u) {
            atomicAdd(&acc[GP_N], (unsigned long long)n);
            atomicMax(&acc[GP_MAX], (unsigned long long)mx);
            atomicAdd(&acc[GP_SQ], (unsigned long long)sq);
        }
        n = mx = 0u;
        sq = 0u;
    }
};

// Unions of the pairs (a[u], b[u]) of this wavefront's lanes, a[u] kEmpty
// where there is none; a pair equal to that of the lane below is dropped, the
// others are packed in the wavefront's own part of an LDS list (R * 64 words,
// indices below 2^16) and taken 64 at a time: a quarter of the edge positions
// have a union, and a round costs what its slowest lane does.  (Joining all
// pairs in rounds -- hook every larger root under the smallest it meets,
// compress, until no pair is left -- was measured and dropped: three barriers
// of 1024 threads a round made level 2 of 512^2 7.3 us instead of 5.2.)
template <uint32_t R>
__device__ __forceinline__ void join_pairs(uint32_t *par, uint32_t *list, const uint32_t *a, const uint32_t *b) {
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t n = 0u;
#pragma unroll
    for (uint32_t u = 0; u < R; ++u) {
        const uint32_t pa = __shfl_up(a[u], 1, 64), pb = __shfl_up(b[u], 1, 64);
        const bool has = a[u] != kEmpty && !(lane > 0u && pa == a[u] && pb == b[u]);
        const uint64_t bal = __ballot(has);
        if (has)
            list[n + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u))] =
                a[u] | (b[u] << 16);
        n += (uint32_t)__popcll(bal);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (uint32_t k = lane; k < n; k += 64u) lds_union(par, list[k] & 0xFFFFu, list[k] >> 16);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// A first step for join_pairs, while every entry of par is a root (an entry that
// is not would lose its link): every pair hooks its larger index under the
// smallest it meets, compress() points all entries at their roots, and pairs
// that share a root are done.  Level 2 of 1024^2 (beta = 0.44, 3264 clusters):
// unions 9.6 -> 6.8 us; of 512^2 (758) 4.4 -> 4.7.
template <uint32_t R, class Compress>
__device__ __forceinline__ void hook_pairs(uint32_t *par, uint32_t *a, uint32_t *b, Compress &&compress) {
#pragma unroll
    for (uint32_t u = 0; u < R; ++u)
        if (a[u] != kEmpty) atomicMin(&par[max(a[u], b[u])], min(a[u], b[u]));
    __syncthreads();
    compress();
    __syncthreads();
#pragma unroll
    for (uint32_t u = 0; u < R; ++u) {
        const uint32_t ra = a[u] != kEmpty ? lds_load(&par[a[u]]) : kEmpty, rb = a[u] != kEmpty ? lds_load(&par[b[u]]) : kEmpty;
        a[u] = ra == rb ? kEmpty : ra;
        b[u] = rb;
    }
}

// What level 2 loads of the groups' results, in batches whose loads overlap;
// the first batch is loaded while the clusters are being counted.  Clusters:
// a wavefront takes a group at a time, kEnt rounds of 64 (about 200 are
// open).  Bonds: position f of the groups' E and N sides, one per thread and
// round, all in the one batch.
struct TopLoads {
    static constexpr uint32_t kEnt = 5, kPos = 8;
    uint64_t e[kEnt];
    uint32_t a[kPos], b[kPos];  // clusters on both sides (kNoRef: no bond)
    const uint64_t *gnode;      // key | size << 32 of a group's clusters
    const uint16_t *gedge;      // numbers of the clusters at the bonds on its E, N, W, S sides (kNoRef: none)
    uint32_t slots;             // of each, per group

    __device__ __forceinline__ void clusters(uint32_t g, uint32_t ng, uint32_t j0) {
#pragma unroll
        for (uint32_t u = 0; u < kEnt; ++u) {
            const uint32_t j = j0 + 64u * u + (threadIdx.x & 63u);
            e[u] = g < ng && j < slots ? ag_load(&gnode[(size_t)g * slots + j]) : 0u;
        }
    }
    // Group g, its neighbour nb, the direction and the place p of position f,
    // the f0-th and following 64 of a wavefront: all but the place (and, with
    // 32-wide tiles, the tile it lies in) are the same for its lanes and
    // computed once, on the scalar unit.
    static __device__ __forceinline__ bool place(const Dev &d, uint32_t f0, uint32_t ngx, uint32_t &g, uint32_t &nb,
                                                 uint32_t &dir, uint32_t &p) {
        const uint32_t lw = d.tw == 64u ? 6u : 5u, per = 8u << lw;
        const uint32_t fw = (uint32_t)__builtin_amdgcn_readfirstlane((int)f0);
        const bool in = fw < ngx * ngx * per;
        g = in ? fw >> (lw + 3u) : 0u;
        dir = (fw >> (lw + 2u)) & 1u;
        p = (fw & ((4u << lw) - 1u)) + (threadIdx.x & 63u);
        const uint32_t gy = g / ngx, gx = g - gy * ngx;
        nb = dir == 0u ? gy * ngx + (gx + 1u == ngx ? 0u : gx + 1u) : (gy + 1u == ngx ? 0u : gy + 1u) * ngx + gx;
        return in && (dir == 0u ? gy : gx) * kUG + (p >> lw) < d.ntx;
    }
    __device__ __forceinline__ void bonds(const Dev &d, uint32_t ngx) {
#pragma unroll
        for (uint32_t u = 0; u < kPos; ++u) {
            uint32_t g, nb, dir, p;
            const bool ok = place(d, kMergeThreads * u + (threadIdx.x & ~63u), ngx, g, nb, dir, p);
            a[u] = ok ? ag_load(&gedge[(size_t)g * slots + dir * (slots / 4u) + p]) : kNoRef;
            b[u] = ok ? ag_load(&gedge[(size_t)nb * slots + (2u + dir) * (slots / 4u) + p]) : kNoRef;
        }
    }
};

// Level 2 over the m = s_off[ng] open clusters of all groups; the union-find
// arrays are in LDS, or (more clusters than fit) in the lattice's node tables,
// which level 1 has finished with.
template <bool LDS>
__device__ __forceinline__ void merge_top(const Dev &d, uint32_t ng, uint32_t ngx, uint32_t t, const uint32_t *s_off,
                                          TopLoads &ld1, uint32_t *par, uint32_t *sz, uint32_t *key,
                                          unsigned long long *s_acc) {
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    auto ld = [](uint32_t *p) { return LDS ? lds_load(p) : g_load(p); };
    auto st = [](uint32_t *p, uint32_t v) {
        if (LDS)
            *p = v;
        else
            g_store(p, v);
    };
    // global accesses of this workgroup complete before it goes on
    auto barrier = [] {
        if (!LDS) __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    };
    const uint32_t m = s_off[ng];
    for (uint32_t i = tid; i < m; i += kMergeThreads) st(&par[i], i);
    barrier();
    // bonds across the E and N edges of every group: all of them at once, since
    // hook_pairs is right only while every entry is a root
    static_assert(kMergeGroups * 8u * 64u <= kMergeThreads * TopLoads::kPos, "one position per thread and round");
#pragma unroll
    for (uint32_t u = 0; u < TopLoads::kPos; ++u) {
        uint32_t g, nb, dir, p;
        TopLoads::place(d, kMergeThreads * u + (tid & ~63u), ngx, g, nb, dir, p);
        const bool has = ld1.a[u] != kNoRef && ld1.b[u] != kNoRef;
        ld1.a[u] = has ? s_off[g] + ld1.a[u] : kEmpty;
        ld1.b[u] = has ? s_off[nb] + ld1.b[u] : kEmpty;
    }
    if (LDS) {  // the lists lie where sizes and keys go afterwards
        hook_pairs<TopLoads::kPos>(par, ld1.a, ld1.b, [&] {
            for (uint32_t i = tid; i < m; i += kMergeThreads) lds_store(&par[i], lds_find(par, i));
        });
        join_pairs<TopLoads::kPos>(par, sz + wv * 64u * TopLoads::kPos, ld1.a, ld1.b);
    } else {
#pragma unroll
        for (uint32_t u = 0; u < TopLoads::kPos; ++u)
            if (ld1.a[u] != kEmpty) g_union(par, ld1.a[u], ld1.b[u]);
    }
    if (LDS) __syncthreads();
    for (uint32_t g = wv; g < ng; g += kMergeWaves) {
        const uint32_t off = s_off[g], n = s_off[g + 1u] - off;
        for (uint32_t j0 = 0; j0 < n; j0 += 64u * TopLoads::kEnt) {
            if (g != wv || j0 != 0u) ld1.clusters(g, ng, j0);
#pragma unroll
            for (uint32_t u = 0; u < TopLoads::kEnt; ++u) {
                const uint32_t j = j0 + 64u * u + lane, i = off + j;
                if (j >= n) continue;
                st(&sz[i], (uint32_t)(ld1.e[u] >> 32));
                st(&key[i], (uint32_t)ld1.e[u]);
            }
        }
    }
    barrier();
    for (uint32_t i = tid; i < m; i += kMergeThreads) {
        uint32_t r = i, q = ld(&par[r]);
        while (q != r) {
            r = q;
            q = ld(&par[r]);
        }
        if (r == i) continue;
        st(&par[i], r);  // (an ancestor of i and of every other chain through i)
        atomicAdd(&sz[r], ld(&sz[i]));
        atomicMin(&key[r], ld(&key[i]));
    }
    barrier();
    Stats cs;
    for (uint32_t g = wv; g < ng; g += kMergeWaves)
        for (uint32_t j = lane; j < s_off[g + 1u] - s_off[g]; j += 64u) {
            const uint32_t i = s_off[g] + j, r = ld(&par[i]);
            d.gspin[(size_t)g * ld1.slots + j] = (uint8_t)new_value(d, ld(&key[r]), t);
            if (r == i) cs.add(ld(&sz[i]), s_acc);
        }
    cs.flush(s_acc);
}

// Open clusters that level 2 holds in LDS (75 KB with the rest; a workgroup's
// registers leave no room for a second one on its CU); a group
// of 64-wide tiles has at most about 270 (beta = 0.4), so that 16 groups fit;
// more goes through the node tables.
constexpr uint32_t kTopLds = 6144;

__device__ __forceinline__ void merge_body(const Dev &d, const uint32_t ug) {
    constexpr uint32_t NL = kUG * kUG * kNodeSlots;  // local node = tile-in-group * kNodeSlots + node
    static_assert(kTopLds >= NL + 128u * kMergeWaves, "level 1 uses the same arrays, with its lists behind the parents");
    static_assert(2u * kTopLds >= 64u * TopLoads::kPos * kMergeWaves, "level 2's lists lie in the sizes and keys");
    __shared__ uint32_t s_buf[3u * kTopLds];
    __shared__ uint32_t s_link[NL / 32], s_pre[NL / 32];  // roots of clusters that go on outside, and their numbers
    __shared__ uint32_t s_off[kMergeGroups + 1u];
    __shared__ unsigned long long s_acc[GP_END];
    __shared__ int s_last;
    // (index arithmetic that is the same for a wavefront's lanes goes to the
    // scalar unit: a workgroup of 16 wavefronts on one CU is bound by the
    // instructions it issues)
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const uint64_t tsw = *d.tdev;
    const uint32_t t = (uint32_t)tsw, pc = (uint32_t)(tsw & 1u);
    const uint32_t ntx = d.ntx, tw = d.tw, lw = tw == 64u ? 6u : 5u;
    const uint32_t ngx = (ntx + kUG - 1u) / kUG, ng = ngx * ngx, gy = ug / ngx, gx = ug - gy * ngx;
    const bool whole = ng == 1u;
    // the groups' results for the last workgroup lie in the spins that k_tile has
    // read and replaced by then, of no more use until the next sweep writes them
    const uint32_t slots = 16u << lw, side = 4u << lw;  // (ref_slots; positions of a side)
    uint64_t *const gnode = reinterpret_cast<uint64_t *>(d.spins[pc]);
    uint16_t *const gedge = reinterpret_cast<uint16_t *>(gnode + ng * slots);
    uint32_t *const s_par = s_buf, *const s_sz = s_buf + kTopLds, *const s_key = s_buf + 2u * kTopLds;

    // edge positions: E and N of every tile (two per thread, one with 32-wide
    // tiles), and W and S of the tiles on the group's low sides (bonds that
    // come in); all loads before any is waited on
    uint32_t ua[2], ub[2];     // nodes joined; ub kEmpty: the bond leaves the group
    uint32_t uo[2];            // its place on the group's perimeter
#pragma unroll
    for (uint32_t u = 0; u < 2u; ++u) {
        const uint32_t fw = 64u * wv + kMergeThreads * u, T = (fw >> (lw + 1u)) & 15u;  // (the tile is the wavefront's)
        const uint32_t f = fw + lane, dir = (f >> lw) & 1u, i = f & (tw - 1u);
        const uint32_t lx = T % kUG, ly = T / kUG, tx = gx * kUG + lx, ty = gy * kUG + ly;
        const bool ok = fw < (32u << lw) && tx < ntx && ty < ntx;
        const uint32_t A = ok ? ty * ntx + tx : 0u;
        const uint32_t nx = dir == 0u ? (tx + 1u == ntx ? 0u : tx + 1u) : tx;
        const uint32_t ny = dir == 0u ? ty : (ty + 1u == ntx ? 0u : ty + 1u);
        const bool inside = whole || (dir == 0u ? lx + 1u < kUG && tx + 1u < ntx : ly + 1u < kUG && ty + 1u < ntx);
        const uint32_t B = ok ? ny * ntx + nx : 0u, TB = whole ? ny * kUG + nx : T + (dir == 0u ? 1u : kUG);
        const uint64_t bits = d.xb[2u * A + dir];
        const uint32_t an = d.edge[((size_t)A * 4u + (dir == 0u ? 1u : 3u)) * tw + i];
        const uint32_t bn = d.edge[((size_t)B * 4u + (dir == 0u ? 0u : 2u)) * tw + i];
        const bool has = ok && ((bits >> i) & 1u);
        ua[u] = has ? T * kNodeSlots + an : kEmpty;
        ub[u] = inside ? TB * kNodeSlots + bn : kEmpty;
        uo[u] = ok && !inside ? dir * side + (dir == 0u ? ly : lx) * tw + i : kEmpty;
    }
    uint32_t va = kEmpty, vo = kEmpty;  // incoming: node, place
    if (!whole) {
        const uint32_t dir = (tid >> (lw + 2u)) & 1u, l = (tid >> lw) & 3u, i = tid & (tw - 1u);
        const uint32_t tx = gx * kUG + (dir == 0u ? 0u : l), ty = gy * kUG + (dir == 0u ? l : 0u);
        const bool ok = tid < (8u << lw) && tx < ntx && ty < ntx;
        const uint32_t A = ok ? ty * ntx + tx : 0u;
        const uint32_t px = dir == 0u ? (tx == 0u ? ntx - 1u : tx - 1u) : tx, py = dir == 0u ? ty : (ty == 0u ? ntx - 1u : ty - 1u);
        const uint32_t P = ok ? py * ntx + px : 0u;
        const uint64_t bits = d.xb[2u * P + dir];
        const uint32_t an = d.edge[((size_t)A * 4u + (dir == 0u ? 0u : 2u)) * tw + i];
        if (ok && ((bits >> i) & 1u)) va = (dir == 0u ? l * kUG : l) * kNodeSlots + an;
        if (ok) vo = (2u + dir) * side + l * tw + i;
    }
    // nodes: wavefront wv has tile wv of the group, its node slots lane + 64 j
    const uint32_t mx = gx * kUG + wv % kUG, my = gy * kUG + wv / kUG;
    const bool mok = mx < ntx && my < ntx;
    const uint32_t mtile = mok ? my * ntx + mx : 0u;
    const uint32_t nk = mok ? min(nk_either(d, pc, mtile), 252u) : 0u;
    constexpr uint32_t NJ = kNodeSlots / 64u;
    uint32_t kk[NJ], kz[NJ];
#pragma unroll
    for (uint32_t j = 0; j < NJ; ++j) {
        const uint32_t node = mtile * kNodeSlots + 64u * j + lane;
        const bool in = j == 0u || 64u * j < nk;  // the first round is loaded without waiting for nk
        kk[j] = in ? d.key[node] : 0u;
        kz[j] = in ? d.nsize[node] : 0u;
    }
    if (tid < NL / 32u) s_link[tid] = 0u;
    if (tid < (uint32_t)GP_END) s_acc[tid] = 0ull;
#pragma unroll
    for (uint32_t j = 0; j < NJ; ++j) {
        const uint32_t k = 64u * j + lane, li = wv * kNodeSlots + k;
        if (k >= nk) continue;
        s_par[li] = li;
        s_sz[li] = kz[j];
        s_key[li] = kk[j];
    }
    __syncthreads();
    {
        uint32_t ja[2];
#pragma unroll
        for (uint32_t u = 0; u < 2u; ++u) ja[u] = ub[u] == kEmpty ? kEmpty : ua[u];
        join_pairs<2>(s_par, s_buf + NL + 128u * wv, ja, ub);
    }
    __syncthreads();
    uint32_t rt[NJ];
#pragma unroll
    for (uint32_t j = 0; j < NJ; ++j) {
        const uint32_t k = 64u * j + lane, li = wv * kNodeSlots + k;
        rt[j] = li;
        if (k >= nk) continue;
        rt[j] = lds_find(s_par, li);
        if (rt[j] != li) {
            atomicAdd(&s_sz[rt[j]], kz[j]);
            atomicMin(&s_key[rt[j]], kk[j]);
        }
    }
    uint32_t ur[2] = {kEmpty, kEmpty}, vr = kEmpty;  // roots at the perimeter's bonds
    if (!whole) {
#pragma unroll
        for (uint32_t u = 0; u < 2u; ++u)
            if (ua[u] != kEmpty && uo[u] != kEmpty) ur[u] = lds_find(s_par, ua[u]);
        if (va != kEmpty) vr = lds_find(s_par, va);
#pragma unroll
        for (uint32_t u = 0; u < 2u; ++u)
            if (ur[u] != kEmpty) atomicOr(&s_link[ur[u] >> 5], 1u << (ur[u] & 31u));
        if (vr != kEmpty) atomicOr(&s_link[vr >> 5], 1u << (vr & 31u));
    }
    __syncthreads();
    uint32_t open = 0u;  // clusters that go on outside (in wavefront 0)
    if (!whole) {
        if (wv == 0u) {
            const uint32_t ca = __popc(s_link[2u * lane]), c = ca + __popc(s_link[2u * lane + 1u]);
            uint32_t incl = c;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t n = __shfl_up(incl, o, 64);
                if (lane >= (uint32_t)o) incl += n;
            }
            s_pre[2u * lane] = incl - c;
            s_pre[2u * lane + 1u] = incl - c + ca;
            open = min((uint32_t)__shfl((int)incl, 63, 64), slots);
        }
        __syncthreads();
    }
    auto number = [&](uint32_t r) {
        return min(s_pre[r >> 5] + __popc(s_link[r >> 5] & ((1u << (r & 31u)) - 1u)), slots - 1u);
    };
    Stats cs;
#pragma unroll
    for (uint32_t j = 0; j < NJ; ++j) {
        const uint32_t k = 64u * j + lane, li = wv * kNodeSlots + k, r = rt[j];
        if (k >= nk) continue;
        uint32_t ref;
        if ((s_link[r >> 5] >> (r & 31u)) & 1u) {
            const uint32_t n = number(r);
            ref = kRef + n;
            if (r == li) ag_store(&gnode[(size_t)ug * slots + n], (uint64_t)s_key[r] | ((uint64_t)s_sz[r] << 32));
        } else {
            ref = new_value(d, s_key[r], t);
            if (r == li) cs.add(s_sz[r], s_acc);
        }
        d.nref[mtile * kNodeSlots + k] = (uint16_t)ref;
    }
    if (!whole) {
        uint16_t *ge = gedge + (size_t)ug * slots;
#pragma unroll
        for (uint32_t u = 0; u < 2u; ++u)
            if (uo[u] != kEmpty) ag_store(&ge[uo[u]], (uint16_t)(ur[u] == kEmpty ? kNoRef : number(ur[u])));
        if (vo != kEmpty) ag_store(&ge[vo], (uint16_t)(vr == kEmpty ? kNoRef : number(vr)));
    }
    cs.flush(s_acc);
    // the tiles' partials (interior clusters, energy and magnetisation of the
    // incoming configuration, Potts populations): wavefront wv its tile's,
    // one word per lane
    if (mok && lane < (uint32_t)TP_CNT + (uint32_t)kMaxQ) {
        const int32_t v = d.tpart[(size_t)mtile * kTilePart + lane];
        uint32_t f = 0u;
        if (lane == (uint32_t)TP_E)
            f = GP_E;
        else if (lane == (uint32_t)TP_M)
            f = GP_M;
        else if (lane == (uint32_t)TP_N)
            f = GP_N;
        else if (lane == (uint32_t)TP_MAX)
            f = GP_MAX;
        else if (lane == (uint32_t)TP_SQ)
            f = GP_SQ;
        else if (lane < (uint32_t)TP_CNT)
            f = (uint32_t)GP_HIST + lane - (uint32_t)TP_HIST;
        else
            f = (uint32_t)GP_CNT + lane - (uint32_t)TP_CNT;
        if (f == (uint32_t)GP_MAX)
            atomicMax(&s_acc[f], (unsigned long long)v);
        else if (v != 0 && (f < (uint32_t)GP_CNT || d.q))
            atomicAdd(&s_acc[f], (unsigned long long)(int64_t)v);
    }
    if (!whole) {
        __syncthreads();
        if (tid < (uint32_t)GP_END) ag_store(&d.mpart[(size_t)ug * kGroupPart + tid], (uint64_t)s_acc[tid]);
        if (tid == 0u) ag_store(&d.gcount[ug], open);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        unsigned long long *acc = reinterpret_cast<unsigned long long *>(d.acc);
        if (tid == 0u) s_last = atomicAdd(&acc[ACC_COUNT], 1ull) == (unsigned long long)ng - 1ull;
        if (tid < (uint32_t)GP_END) s_acc[tid] = 0ull;
        __syncthreads();
        if (!s_last) return;
        if (tid == 0u) ag_store(&d.acc[ACC_COUNT], (uint64_t)0);
        TopLoads top;
        top.gnode = gnode;
        top.gedge = gedge;
        top.slots = slots;
        top.clusters(wv, ng, 0u);
        top.bonds(d, ngx);
        // the groups' partials, and in wavefront 0 the first cluster of every group
        uint64_t v = 0u;
        for (uint32_t g = wv; g < ng; g += kMergeWaves) {
            const uint64_t x = lane < (uint32_t)GP_END ? ag_load(&d.mpart[(size_t)g * kGroupPart + lane]) : 0u;
            v = lane == (uint32_t)GP_MAX ? max(v, x) : v + x;
        }
        if (wv == 0u) {
            uint32_t c[2];
#pragma unroll
            for (uint32_t h = 0; h < 2u; ++h) c[h] = 2u * lane + h < ng ? min(ag_load(&d.gcount[2u * lane + h]), slots) : 0u;
            uint32_t incl = c[0] + c[1];
            const uint32_t own = incl;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t n = __shfl_up(incl, o, 64);
                if (lane >= (uint32_t)o) incl += n;
            }
            const uint32_t pre = incl - own;
            if (2u * lane <= ng) s_off[2u * lane] = pre;
            if (2u * lane + 1u <= ng) s_off[2u * lane + 1u] = pre + c[0];
        }
        if (lane == (uint32_t)GP_MAX)
            atomicMax(&s_acc[lane], (unsigned long long)v);
        else if (v && lane < (uint32_t)GP_END)
            atomicAdd(&s_acc[lane], (unsigned long long)v);
        __syncthreads();
        if (s_off[ng] <= kTopLds)
            merge_top<true>(d, ng, ngx, t, s_off, top, s_par, s_sz, s_key, s_acc);
        else
            merge_top<false>(d, ng, ngx, t, s_off, top, d.parent, d.nsize, d.key, s_acc);
    }
    __syncthreads();
    record_write(d, reinterpret_cast<const uint64_t *>(s_acc), 0);
}

__global__ __launch_bounds__(kMergeThreads) void k_merge(Dev d) { merge_body(d, blockIdx.x); }

__global__ __launch_bounds__(kMergeThreads) void k_merge_b(const Dev *devs, const uint32_t *map) {
    const uint32_t e = map[blockIdx.x];
    merge_body(devs[e >> kMapShift], e & kMapMask);
}

// k_merge of the small replicas (the first ns workgroups) beside the unions of
// the large ones (16 wavefronts, of k_union_b, per workgroup): both are chains
// of dependent accesses that leave the GPU nearly idle.  us per sweep, two
// launches / one: a 64^2 and k 1088^2 lattices, k = 1 81.5 / 76.9, 16 162.0 /
// 154.7, 96 563 / 567; 100 of 256^2 and k of 1088^2, k = 1 111.9 / 103.1, 16
// 190.6 / 185.1.  (A second stream for k_merge was 10 % better on a server where
// it had a hardware queue of its own and 10 % worse where it had none.)
__global__ __launch_bounds__(kMergeThreads) void k_join_b(const Dev *devs, const uint32_t *smap, uint32_t ns,
                                                          const uint32_t *wmap, uint32_t nw, uint32_t nE) {
    if (blockIdx.x < ns) {
        const uint32_t e = smap[blockIdx.x];
        merge_body(devs[e >> kMapShift], e & kMapMask);
    } else {
        union_b_body(devs, wmap, nw, nE, (blockIdx.x - ns) * kMergeWaves + (threadIdx.x >> 6));
    }
}

// =====================================================================
// k_resolve: replace node codes by final spins in place and measure the
// configuration (runs once at the end of every sw_sweep call).  No byte refers
// to a node then, and the tiles have none left for the next sweep's tables (a
// server may give the lattice another merge with other tables).
// =====================================================================
template <int TW, bool POTTS, int TWO>
__device__ __forceinline__ void resolve_body(const Dev &d, const uint32_t tile) {
    constexpr int NT = TW * TW / 16;
    constexpr uint32_t RPT = TW / 16;
    constexpr int NWAVE = (NT + 63) / 64;
    constexpr int NPL = POTTS ? 3 : 1;
    constexpr uint32_t EW = (TW + 31) / 32;
    using Row = typename RowOf<TW>::T;
    __shared__ uint8_t s_tab[256];
    __shared__ Row s_up[NPL * (TW + 1)];
    __shared__ uint32_t s_eup[NPL * EW];
    __shared__ int32_t s_red[NWAVE][POTTS ? 6 : 2];

    const uint32_t tid = threadIdx.x;
    const uint32_t L = d.L, ntx = d.ntx;
    const uint32_t tx = tile % ntx, ty = tile / ntx;
    const uint64_t tsw = *d.tdev;
    const uint32_t pc = (uint32_t)(tsw & 1u), pp = pc ^ 1u;
    int8_t *sp = d.spins[pc];
    const uint32_t ly = tid / RPT, seg = tid % RPT, x0 = seg * 16u;
    const uint32_t gy = ty * TW + ly, gx0 = tx * TW + x0;
    const uint32_t east = ty * ntx + (tx + 1u == ntx ? 0u : tx + 1u);
    const uint32_t north = (ty + 1u == ntx ? 0u : ty + 1u) * ntx + tx;
    const uint32_t gbe = ref_base(d, tx + 1u == ntx ? 0u : tx + 1u, ty);
    const uint32_t gbn = ref_base(d, tx, ty + 1u == ntx ? 0u : ty + 1u);

    const Seg<16> v = load_seg<16>(sp + (size_t)gy * L + gx0);
    Seg<16> vn{};
    if (ly == TW - 1) {
        const uint32_t gyn = (gy + 1u == L) ? 0u : gy + 1u;
        vn = load_seg<16>(sp + (size_t)gyn * L + gx0);
    }
    uint32_t ve = 0;
    if (seg == RPT - 1) {
        const uint32_t gxe = (gx0 + 16u == L) ? 0u : gx0 + 16u;
        ve = (uint8_t)sp[(size_t)gy * L + gxe];
    }
    load_table<TW, POTTS, TWO, NT>(d, tile, ref_base(d, tx, ty), pp, s_tab, tid);
    if (tid < NPL * EW) s_eup[tid] = 0u;
    __syncthreads();
    uint32_t up = 0u, pl[3] = {0u, 0u, 0u};
    if constexpr (POTTS) {
        decode_potts(v, s_tab, pl);
#pragma unroll
        for (int b = 0; b < 3; ++b) reinterpret_cast<uint16_t *>(s_up + b * (TW + 1))[ly * RPT + seg] = (uint16_t)pl[b];
        if (ly == TW - 1) {
            uint32_t pn[3];
            decode_potts_remote<TW, TWO>(d, vn, north, gbn, pn);
#pragma unroll
            for (int b = 0; b < 3; ++b)
                reinterpret_cast<uint16_t *>(s_up + b * (TW + 1))[TW * RPT + seg] = (uint16_t)pn[b];
        }
        if (seg == RPT - 1) {
            uint32_t ev;
            remote_values<TW, true, TWO, 1>(d, &ve, east, gbe, &ev);
#pragma unroll
            for (uint32_t b = 0; b < 3u; ++b)
                if ((ev >> b) & 1u) atomicOr(&s_eup[b * EW + (ly >> 5)], 1u << (ly & 31u));
        }
    } else {
        up = decode(v, s_tab);
        reinterpret_cast<uint16_t *>(s_up)[ly * RPT + seg] = (uint16_t)up;
        if (ly == TW - 1) {
            const uint32_t upn = decode_remote<TWO>(d, vn, north, gbn);
            reinterpret_cast<uint16_t *>(s_up)[TW * RPT + seg] = (uint16_t)upn;
        }
        if (seg == RPT - 1) {
            uint32_t ev;
            remote_values<TW, false, TWO, 1>(d, &ve, east, gbe, &ev);
            if (ev) atomicOr(&s_eup[ly >> 5], 1u << (ly & 31u));
        }
    }
    __syncthreads();
    int32_t e_part, m_part = 0;
    uint32_t cpk[4] = {0u, 0u, 0u, 0u};
    uint32_t out[4] = {0u, 0u, 0u, 0u};
    if constexpr (POTTS) {
        uint32_t dE = 0u, dN = 0u;
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const Row rowv = s_up[b * (TW + 1) + ly];
            const uint32_t pN = (uint32_t)(s_up[b * (TW + 1) + ly + 1] >> x0) & 0xFFFFu;
            const uint32_t ebit = (s_eup[b * EW + (ly >> 5)] >> (ly & 31u)) & 1u;
            const uint32_t nxt = (x0 + 16u < (uint32_t)TW) ? ((uint32_t)(rowv >> (x0 + 16u)) & 1u) : ebit;
            dE |= pl[b] ^ ((pl[b] >> 1) | (nxt << 15));
            dN |= pl[b] ^ pN;
        }
        e_part = __popc(~dE & 0xFFFFu) + __popc(~dN & 0xFFFFu);
        potts_counts<0xFFFFu>(pl, cpk);
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const uint32_t x = ((pl[0] >> q) & 1u) | (((pl[1] >> q) & 1u) << 1) | (((pl[2] >> q) & 1u) << 2);
            out[q >> 2] |= x << (8 * (q & 3));
        }
    } else {
        const Row rowv = s_up[ly];
        const uint32_t upN = (uint32_t)(s_up[ly + 1] >> x0) & 0xFFFFu;
        const uint32_t ebit = (s_eup[ly >> 5] >> (ly & 31u)) & 1u;
        const uint32_t nxt = (x0 + 16u < (uint32_t)TW) ? ((uint32_t)(rowv >> (x0 + 16u)) & 1u) : ebit;
        const uint32_t upE = (up >> 1) | (nxt << 15);
        e_part = 2 * (__popc(~(up ^ upE) & 0xFFFFu) + __popc(~(up ^ upN) & 0xFFFFu)) - 32;
        m_part = 2 * __popc(up) - 16;
#pragma unroll
        for (int q = 0; q < 16; ++q) out[q >> 2] |= (((up >> q) & 1u) ? 0x01u : 0xFFu) << (8 * (q & 3));
    }
    *reinterpret_cast<uint4 *>(sp + (size_t)gy * L + gx0) = make_uint4(out[0], out[1], out[2], out[3]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        e_part += __shfl_xor(e_part, o, 64);
        m_part += __shfl_xor(m_part, o, 64);
        if constexpr (POTTS) {
#pragma unroll
            for (int i = 0; i < 4; ++i) cpk[i] += __shfl_xor(cpk[i], o, 64);
        }
    }
    if ((tid & 63u) == 0u) {
        s_red[tid >> 6][0] = e_part;
        s_red[tid >> 6][1] = m_part;
        if constexpr (POTTS) {
#pragma unroll
            for (int i = 0; i < 4; ++i) s_red[tid >> 6][2 + i] = (int32_t)cpk[i];
        }
    }
    __syncthreads();
    if (tid == 0u) {
        d.nk[pp][tile] = 0u;  // (its readers are this workgroup's, before the barriers)
        int32_t e = 0, m = 0;
        for (int w = 0; w < NWAVE; ++w) {
            e += s_red[w][0];
            m += s_red[w][1];
        }
        int32_t *tp = d.tpart + (size_t)tile * kTilePart;
        tp[TP_E] = e;
        tp[TP_M] = m;
        if constexpr (POTTS) {
            for (int k = 0; k < 8; ++k) {
                int32_t c = 0;
                for (int w = 0; w < NWAVE; ++w) c += (int32_t)(((uint32_t)s_red[w][2 + k / 2] >> (16 * (k & 1))) & 0xFFFFu);
                tp[TP_CNT + k] = c;
            }
        }
    }
}

template <int TW, bool POTTS, int TWO>
__global__ __launch_bounds__(TW *TW / 16) void k_resolve(Dev d) {
    resolve_body<TW, POTTS, TWO>(d, tile_of_block(blockIdx.x, d.ntiles));
}

template <int TW, bool POTTS, int TWO>
__global__ __launch_bounds__(TW *TW / 16) void k_resolve_b(const Dev *devs, const uint32_t *map) {
    const uint32_t e = map[tile_of_block(blockIdx.x, gridDim.x)];
    resolve_body<TW, POTTS, TWO>(devs[e >> kMapShift], e & kMapMask);
}

// Initial spins (Fig. 1): hot = bit 0 of word 0 of Philox({s, 0, 2, 0}),
// cold = all +1; for the Potts model hot = floor(w q / 2^32) of that word,
// cold = all 0.  16 sites per thread.
__global__ __launch_bounds__(256) void k_init(Dev d, int cold) {
    const size_t n16 = d.nsite / 16u;
    const uint32_t pc = (uint32_t)(*d.tdev & 1u);
    int8_t *sp = d.spins[pc];
    const uint32_t fill = d.q ? 0u : 0x01010101u;
    for (size_t i = blockIdx.x * (size_t)256 + threadIdx.x; i < n16; i += (size_t)gridDim.x * 256) {
        uint32_t out[4] = {fill, fill, fill, fill};
        if (!cold) {
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                uint32_t w0 = (uint32_t)(i * 16u + q), w1 = 0u, w2 = 2u, w3 = 0u;
                philox10(w0, w1, w2, w3, d.seed_lo, d.seed_hi);
                if (d.q)
                    out[q >> 2] |= (uint32_t)(((uint64_t)w0 * d.q) >> 32) << (8 * (q & 3));
                else if (w0 & 1u)
                    out[q >> 2] |= 0xFFu << (8 * (q & 3));
            }
        }
        *reinterpret_cast<uint4 *>(sp + i * 16u) = make_uint4(out[0], out[1], out[2], out[3]);
    }
}

__global__ __launch_bounds__(256) void k_zero_u64(uint64_t *p, size_t n) {
    for (size_t i = blockIdx.x * (size_t)256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) p[i] = 0u;
}

inline uint32_t grid_for(size_t n, uint32_t per_block, uint32_t cap) {
    size_t g = (n + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (uint32_t)g;
}

template <bool DENSE, int TWO, int SPT>
void launch_tile(const Dev &d, hipStream_t s) {
    if (d.q && d.tw == 64)
        k_tile<64, true, DENSE, TWO, SPT><<<d.ntiles, 4096 / SPT, 0, s>>>(d);
    else if (d.q)
        k_tile<32, true, DENSE, TWO, SPT><<<d.ntiles, 1024 / SPT, 0, s>>>(d);
    else if (d.tw == 64)
        k_tile<64, false, DENSE, TWO, SPT><<<d.ntiles, 4096 / SPT, 0, s>>>(d);
    else
        k_tile<32, false, DENSE, TWO, SPT><<<d.ntiles, 1024 / SPT, 0, s>>>(d);
}

// The order in which k_union links.  Above the critical coupling (bond
// probability above sqrt(q) / (1 + sqrt(q))) one cluster spans the lattice, and
// index order links its part in every group under the next group's: chains as
// long as the lattice is wide, which bit-reversed order breaks up.  Elsewhere
// index order is better: it makes the node with the smallest site the root
// nearly always, and spares k_flatten an atomic per workgroup and root.  Sweeps
// index / bits: beta = 0.5, 4064^2 202 / 186, 8192^2 386 / 370, 16384^2 1300 /
// 1238 us; beta_c, 161 / 164, 341 / 344, 1168 / 1184; on fewer than 16 groups
// a side there is nothing between them (1344^2, beta = 0.5, 65.8 / 65.9).
constexpr uint32_t kBitsGroups = 16;
bool ordered(const Dev &d) {
    const double q = sqrt((double)(d.q ? d.q : 2u));
    return (double)d.T > q / (1.0 + q) * 4294967296.0;
}

// Whether the tile kernels of a launch take 4 sites per thread (else 16): while
// the GPU would not be filled with 16.  Sweeps with 4 / 16 sites at beta_c:
// 64-wide tiles, 1024^2 53 / 64, 1280^2 (400 tiles) 72 / 76, 1536^2 82 / 79,
// 2048^2 91 / 84 us; 32-wide, 512^2 42 / 53, 1056^2 59 / 69, 1536^2 (2304
// tiles) 70 / 74, 1824^2 77 / 79, 2080^2 88 / 86 us.  64-wide Potts tiles take more registers:
// q = 3, 1024^2 (256 tiles) 55 / 68, 1280^2 86 / 78 us.
bool few_tiles(uint32_t ntiles, uint32_t tw, bool potts) {
    return ntiles <= (tw == 32u ? 2304u : potts ? 256u : 400u);
}

template <bool DENSE, int TWO>
void launch_tile(const Dev &d, hipStream_t s) {
    if (few_tiles(d.ntiles, d.tw, d.q != 0u))
        launch_tile<DENSE, TWO, 4>(d, s);
    else
        launch_tile<DENSE, TWO, 16>(d, s);
}

template <int TWO>
void resolve_tiles(const Dev &d, hipStream_t s) {
    if (d.q && d.tw == 64)
        k_resolve<64, true, TWO><<<d.ntiles, 256, 0, s>>>(d);
    else if (d.q)
        k_resolve<32, true, TWO><<<d.ntiles, 64, 0, s>>>(d);
    else if (d.tw == 64)
        k_resolve<64, false, TWO><<<d.ntiles, 256, 0, s>>>(d);
    else
        k_resolve<32, false, TWO><<<d.ntiles, 64, 0, s>>>(d);
}

template <int TWO, int SPT>
void launch_tile_b(const BatchDev &b, hipStream_t s) {
    if (b.potts && b.tw == 64)
        k_tile_b<64, true, TWO, SPT><<<b.ntiles, 4096 / SPT, 0, s>>>(b.devs, b.tmap);
    else if (b.potts)
        k_tile_b<32, true, TWO, SPT><<<b.ntiles, 1024 / SPT, 0, s>>>(b.devs, b.tmap);
    else if (b.tw == 64)
        k_tile_b<64, false, TWO, SPT><<<b.ntiles, 4096 / SPT, 0, s>>>(b.devs, b.tmap);
    else
        k_tile_b<32, false, TWO, SPT><<<b.ntiles, 1024 / SPT, 0, s>>>(b.devs, b.tmap);
}

template <int TWO>
void launch_tile_b(const BatchDev &b, hipStream_t s) {
    if (few_tiles(b.ntiles, b.tw, b.potts != 0u))
        launch_tile_b<TWO == 1 ? 1 : 2, 4>(b, s);
    else
        launch_tile_b<TWO, 16>(b, s);
}

template <int TWO>
void resolve_tiles_b(const BatchDev &b, hipStream_t s) {
    if (b.potts && b.tw == 64)
        k_resolve_b<64, true, TWO><<<b.ntiles, 256, 0, s>>>(b.devs, b.tmap);
    else if (b.potts)
        k_resolve_b<32, true, TWO><<<b.ntiles, 64, 0, s>>>(b.devs, b.tmap);
    else if (b.tw == 64)
        k_resolve_b<64, false, TWO><<<b.ntiles, 256, 0, s>>>(b.devs, b.tmap);
    else
        k_resolve_b<32, false, TWO><<<b.ntiles, 64, 0, s>>>(b.devs, b.tmap);
}

}  // namespace

hipError_t launch_init(const Dev &d, int cold, hipStream_t s) {
    const size_t n16 = d.nsite / 16u;
    k_init<<<grid_for(n16, 256, 65536), 256, 0, s>>>(d, cold);
    return hipGetLastError();
}

hipError_t launch_stage(const Dev &d, int stage, hipStream_t s) {
    const size_t n = d.nsite;
    if (d.le_grid || d.brick) {  // label equivalence, cubic bricks
        if (stage == 0 && d.dense) k_zero_u64<<<grid_for(n + 1, 256, 65536), 256, 0, s>>>(d.dense, n + 1);
        if (stage != 4) {
            const hipError_t e = hipGetLastError();
            return e != hipSuccess ? e : d.brick ? launch_brick_stage(d, stage, s) : launch_le_stage(d, stage, s);
        }
        k_record<<<(d.ngroups + kRecordGroups - 1) / kRecordGroups, 256, 0, s>>>(d, d.ngroups, d.brick ? 0 : 2);
        return hipGetLastError();
    }
    if (d.two && stage > 1) return hipSuccess;  // k_merge does it all
    switch (stage) {
    case 0:  // bonds + tile-local clusters
        if (d.dense) {
            k_zero_u64<<<grid_for(n + 1, 256, 65536), 256, 0, s>>>(d.dense, n + 1);
            launch_tile<true, 0>(d, s);
        } else if (d.two) {
            launch_tile<false, 1>(d, s);
        } else {
            launch_tile<false, 0>(d, s);
        }
        break;
    case 1: {  // the whole merge, or cross-tile unions: inside groups of tiles, then between groups
        const uint32_t ngx = (d.ntx + kUG - 1u) / kUG, nwaves = 2u * ngx * d.ntx;
        if (d.two) {
            k_merge<<<ngx * ngx, kMergeThreads, 0, s>>>(d);
        } else if (d.tw == 64) {
            k_ulocal<64><<<ngx * ngx, 256, 0, s>>>(d);
            if (ngx >= kBitsGroups && ordered(d))
                k_union<64, ByBits><<<(nwaves + 3u) / 4u, 256, 0, s>>>(d);
            else
                k_union<64, ByIndex><<<(nwaves + 3u) / 4u, 256, 0, s>>>(d);
        } else {
            k_ulocal<32><<<ngx * ngx, 256, 0, s>>>(d);
            if (ngx >= kBitsGroups && ordered(d))
                k_union<32, ByBits><<<(nwaves + 3u) / 4u, 256, 0, s>>>(d);
            else
                k_union<32, ByIndex><<<(nwaves + 3u) / 4u, 256, 0, s>>>(d);
        }
        break;
    }
    case 2:  // flatten + cluster sizes
        k_flatten<kGroupTiles><<<d.ngroups, 256, 0, s>>>(d);
        if (d.labels) k_relabel<<<grid_for(n, 256, 65536), 256, 0, s>>>(d);
        break;
    case 3:  // spins of cross-tile clusters, statistics (and the record, on few groups)
        if (d.dense && d.ngroups > kRootsFold)
            k_roots<1, true><<<d.ngroups, 256, 0, s>>>(d);
        else if (d.dense)
            k_roots_fold<true><<<d.ngroups, 256, 0, s>>>(d);
        else if (d.ngroups >= kRootsWide)
            k_roots<1><<<d.ngroups, 256, 0, s>>>(d);
        else if (d.ngroups > kRootsFold)
            k_roots<4><<<d.ngroups, 256, 0, s>>>(d);
        else
            k_roots_fold<false><<<d.ngroups, 256, 0, s>>>(d);
        break;
    case 4:  // record (folded by k_roots on few groups)
        if (d.ngroups > kRootsFold)
            k_record<<<(d.ngroups + kRecordGroups - 1) / kRecordGroups, 256, 0, s>>>(d, d.ngroups, 0);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_sweep(const Dev &d, hipStream_t s) {
    for (int stage = 0; stage < kStages; ++stage) {
        const hipError_t e = launch_stage(d, stage, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_resolve(const Dev &d, hipStream_t s) {
    if (d.le_grid) return hipSuccess;  // label equivalence writes final spins and full records
    if (d.brick) {  // spins are final; their energy and magnetisation go into the last record
        const hipError_t e = launch_brick_measure(d, s);
        if (e != hipSuccess) return e;
        k_record<<<(d.ntiles + kRecordTiles - 1) / kRecordTiles, 256, 0, s>>>(d, d.ntiles, 1);
        return hipGetLastError();
    }
    if (d.two)
        resolve_tiles<1>(d, s);
    else
        resolve_tiles<0>(d, s);
    k_record<<<(d.ntiles + kRecordTiles - 1) / kRecordTiles, 256, 0, s>>>(d, d.ntiles, 1);
    return hipGetLastError();
}

// Batches and servers whose replicas are of several launch groups take
// k_tile_mix up to kMixTiles tiles per group: below, each group's own launch
// leaves most of the GPU idle for the length of one tile; above, the groups'
// own kernels gain from their occupancy and from 16 sites per thread in 32-wide
// tiles.  us per sweep of a batch of k 512^2 and k 544^2 lattices, one launch
// per group / k_tile_mix: k = 1 (353 tiles) 79.0 / 76.5, 8 (2824) 108.1 /
// 101.8, 16 (5648) 125.0 / 138.5; 3-state 82.3 / 76.4, 111.4 / 102.9, 132.2 /
// 141.9; 1024^2 and 1056^2, k = 2 (2690) 106.6 / 102.2, 4 (5380) 126.3 / 138.0.
// A server of 24 Ising and Potts jobs of 128^2 to 2048^2 (three groups), whole
// run: never 73.5 ms, up to this limit 62.5, always 62.5.
constexpr uint32_t kMixTiles = 2048;

hipError_t launch_batch_sweep(const BatchDev *b, int ngroups, hipStream_t s) {
    uint32_t kinds = 0, ntiles = 0;
    for (int g = 0; g < ngroups; ++g) {
        kinds += b[g].nall != 0;
        ntiles += b[g].ntiles;
    }
    const BatchDev &a = b[0];  // the units of every launch group but for the tiles
    if (kinds > 1 && ntiles <= kMixTiles * kinds) {
        k_tile_mix<<<ntiles, 256, 0, s>>>(a.devs, a.tmap);
    } else {
        for (int g = 0; g < ngroups; ++g) {
            if (b[g].nall == 0) continue;
            // n replicas of the global merge, the others of k_merge
            if (b[g].n == 0)
                launch_tile_b<1>(b[g], s);
            else if (b[g].n == b[g].nall)
                launch_tile_b<0>(b[g], s);
            else
                launch_tile_b<2>(b[g], s);
        }
    }
    if (a.nugroups != 0) k_ulocal_b<<<a.nugroups, 256, 0, s>>>(a.devs, a.umap);
    if (a.nsmall != 0 && a.nwmap != 0) {
        k_join_b<<<a.nsmall + (a.nwmap + kMergeWaves - 1u) / kMergeWaves, kMergeThreads, 0, s>>>(
            a.devs, a.smap, a.nsmall, a.wmap, a.nwmap, a.nwE);
    } else {
        if (a.nsmall != 0) k_merge_b<<<a.nsmall, kMergeThreads, 0, s>>>(a.devs, a.smap);
        if (a.nwmap != 0) k_union_b<<<(a.nwmap + 3u) / 4u, 256, 0, s>>>(a.devs, a.wmap, a.nwmap, a.nwE);
    }
    if (a.ngroups != 0) {
        k_flatten_b<<<a.ngroups, 256, 0, s>>>(a.devs, a.gmap);
        k_roots_b<<<a.ngroups, 256, 0, s>>>(a.devs, a.gmap);  // and the records
    }
    return hipGetLastError();
}

hipError_t launch_batch_resolve(const BatchDev &b, hipStream_t s) {
    if (b.nall == 0) return hipSuccess;
    if (b.n == 0)
        resolve_tiles_b<1>(b, s);
    else if (b.n == b.nall)
        resolve_tiles_b<0>(b, s);
    else
        resolve_tiles_b<2>(b, s);
    k_record_b<<<b.nall, 256, 0, s>>>(b.devs, b.amap, 1);
    return hipGetLastError();
}

}  // namespace swmi
