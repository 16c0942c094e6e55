// sw_brick.hip -- the simple cubic lattice on 16^3 bricks (the default for
// dims = 3).  One sweep:
//   k_brick3   bonds (Sec. 2.1) and the connected components of the bonds
//              inside each brick, in LDS; energy and magnetisation of the
//              incoming configuration (Sec. 2.5).  A component with a bond
//              through the brick's surface becomes a node of a global graph.
//   k_blocal3  node unions across the faces inside each 2x2x2 group of
//              bricks, in LDS (not on lattices of few bricks)
//   k_bunion3  node unions across the faces between groups, or all (lock-free
//              union-find in global memory, the smaller node index is root)
//   k_bflat3   every node to its root; sizes and smallest sites into the roots
//   k_bspin3   new spins (Sec. 2.4): a brick's interior components and its
//              nodes' clusters; cluster statistics
// and k_record.  Between k_brick3 and k_bspin3 a site is a 16-bit code, the
// brick-local index of its component's smallest site, so the label of a site
// (2 bytes, not 4) is written once and read once; 32-bit labels are made
// from the codes only when they are asked for (k_blabels3).
//
// At 512^3, q = 3 at 0.5505 (times per sweep): k_brick3 0.58 ms, bound by VALU
// issue (399 M wavefront instructions, 83 % of what independent integer chains
// reach, a quarter of them Philox); k_bflat3 0.17, k_bunion3 0.17, k_blocal3
// 0.10 and k_bspin3 0.13 ms, bound by their dependent loads and device-scope
// atomics over 228 nodes a brick.  32-bit labels in global memory took 2.9 ms.
#include <math.h>

#include "sw_device.h"
#include "sw_internal.h"
#include "sw_philox.h"
#include "sw_uf.h"

namespace swmi {
namespace {

constexpr uint32_t kEmpty = 0xFFFFFFFFu;
constexpr uint32_t kNoNode = 0xFFFFu;
constexpr uint32_t kRows = kBrick * kBrick;   // x-rows of a brick: one thread each
constexpr uint32_t kVol = kRows * kBrick;     // sites of a brick
constexpr uint32_t kPS = kBrick + 1u;         // words of a row in LDS: lanes reading equal x fall in distinct banks
// 64 VGPRs (the Philox calls unrolled by 4, not 16) and 19.9 KB of LDS: eight
// workgroups per CU
constexpr int kBrickWavesPerEU = 8;
static_assert(kBrickNodes == kVol - 14u * 14u * 14u, "a node holds a site of the brick's surface");

// Brick coordinates.
struct Brick {
    uint32_t b, x, y, z;
};
__device__ __forceinline__ Brick brick_of(uint32_t b, uint32_t nb) {
    const uint32_t q = b / nb, z = q / nb;
    return {b, b - q * nb, q - z * nb, z};
}
// Lattice site of brick-local site s.
__device__ __forceinline__ uint32_t site_at(const Brick &B, uint32_t L, uint32_t s) {
    return ((B.z * kBrick + (s >> 8)) * L + B.y * kBrick + ((s >> 4) & 15u)) * L + B.x * kBrick + (s & 15u);
}

// Bit `bit` of each of 16 bytes, as a 16-bit mask.
__device__ __forceinline__ uint32_t plane4(uint32_t w, uint32_t bit) {
    return (((w >> bit) & 0x01010101u) * 0x01020408u) >> 24;
}
__device__ __forceinline__ uint32_t plane16(const uint4 &v, uint32_t bit) {
    return plane4(v.x, bit) | (plane4(v.y, bit) << 4) | (plane4(v.z, bit) << 8) | (plane4(v.w, bit) << 12);
}
// Bit plane b of a spin: Ising, the sign bit; Potts, bit b of the value.
template <bool POTTS> __device__ __forceinline__ uint32_t spin_bit(uint32_t b) { return POTTS ? b : 7u; }

// Site index of the word at byte offset off of a padded brick.
__device__ __forceinline__ uint32_t site_of(uint32_t off) {
    const uint32_t o = off >> 2;
    return o - ((o * 61681u) >> 20);  // o - o / 17 (o < 4352)
}

// Equal-pair masks of a row of 16 sites against its +x, +y, +z neighbours.
struct Equal {
    uint32_t x, y, z;
};

// The spins of this thread's row and its neighbours': bit planes through LDS
// for the rows of this brick, loaded for the rows past its faces.
template <bool POTTS>
__device__ __forceinline__ Equal row_equal(const Dev &d, const Brick &B, uint16_t (*s_pl)[kRows], uint32_t pl[3]) {
    constexpr uint32_t NPL = POTTS ? 3u : 1u;
    const uint32_t tid = threadIdx.x, y = tid & 15u, z = tid >> 4, L = d.L;
    const uint32_t gx0 = B.x * kBrick, gy = B.y * kBrick + y, gz = B.z * kBrick + z;
    const uint32_t gyn = gy + 1u == L ? 0u : gy + 1u, gzn = gz + 1u == L ? 0u : gz + 1u;
    const int8_t *sp = d.spins[0];
    const uint4 v = *reinterpret_cast<const uint4 *>(sp + (gz * L + gy) * L + gx0);  // N < 2^32
    uint4 vy = make_uint4(0u, 0u, 0u, 0u), vz = vy;
    if (y == 15u) vy = *reinterpret_cast<const uint4 *>(sp + (gz * L + gyn) * L + gx0);
    if (z == 15u) vz = *reinterpret_cast<const uint4 *>(sp + (gzn * L + gy) * L + gx0);
    const uint32_t vx = (uint8_t)sp[(gz * L + gy) * L + (gx0 + kBrick == L ? 0u : gx0 + kBrick)];
#pragma unroll
    for (uint32_t b = 0; b < NPL; ++b) {
        pl[b] = plane16(v, spin_bit<POTTS>(b));
        s_pl[b][tid] = (uint16_t)pl[b];
    }
    __syncthreads();
    Equal e = {0u, 0u, 0u};
#pragma unroll
    for (uint32_t b = 0; b < NPL; ++b) {
        const uint32_t bit = spin_bit<POTTS>(b);
        const uint32_t ny = y == 15u ? plane16(vy, bit) : s_pl[b][tid + 1u];
        const uint32_t nz = z == 15u ? plane16(vz, bit) : s_pl[b][(tid + 16u) & (kRows - 1u)];
        e.x |= pl[b] ^ ((pl[b] >> 1) | (((vx >> bit) & 1u) << 15));
        e.y |= pl[b] ^ ny;
        e.z |= pl[b] ^ nz;
    }
    return {~e.x & 0xFFFFu, ~e.y & 0xFFFFu, ~e.z & 0xFFFFu};
}

// Energy (Ising: sum of the products over the row's 48 edges; Potts: equal
// pairs), magnetisation and value populations of the configuration, summed
// over the brick into its partial.
template <bool POTTS>
__device__ __forceinline__ void brick_measure(const Dev &d, uint32_t b, const Equal &q, const uint32_t pl[3]) {
    __shared__ int32_t s_em[kRows / 64][6];
    const uint32_t tid = threadIdx.x;
    const int32_t eq = __popc(q.x) + __popc(q.y) + __popc(q.z);
    // Ising: both sums offset to be non-negative, 16 bits each per wavefront
    uint32_t em = POTTS ? (uint32_t)eq : (uint32_t)eq | ((uint32_t)__popc(pl[0]) << 16);
    uint32_t cpk[4] = {0u, 0u, 0u, 0u};
    if constexpr (POTTS) potts_counts<0xFFFFu>(pl, cpk);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        em += __shfl_xor(em, o, 64);
        if constexpr (POTTS) {
#pragma unroll
            for (int i = 0; i < 4; ++i) cpk[i] += __shfl_xor(cpk[i], o, 64);
        }
    }
    if ((tid & 63u) == 0u) {
        s_em[tid >> 6][0] = (int32_t)em;
        if constexpr (POTTS)
            for (int i = 0; i < 4; ++i) s_em[tid >> 6][1 + i] = (int32_t)cpk[i];
    }
    __syncthreads();
    if (tid == 0u) {
        int32_t e = 0, dn = 0;
        for (uint32_t w = 0; w < kRows / 64u; ++w) {
            e += s_em[w][0] & 0xFFFF;
            dn += (int32_t)((uint32_t)s_em[w][0] >> 16);
        }
        int32_t *tp = d.tpart + (size_t)b * kTilePart;
        tp[TP_E] = POTTS ? e : 2 * e - 3 * (int32_t)kVol;
        tp[TP_M] = POTTS ? 0 : (int32_t)kVol - 2 * dn;
    }
    if (POTTS && tid < (uint32_t)kMaxQ) {
        uint32_t c = 0u;
        for (uint32_t w = 0; w < kRows / 64u; ++w) c += ((uint32_t)s_em[w][1 + tid / 2u] >> (16u * (tid & 1u))) & 0xFFFFu;
        d.tpart[(size_t)b * kTilePart + TP_CNT + tid] = (int32_t)c;
    }
}

// Appends the set bits of R (sites of this lane's row) to the wavefront's
// union list, held in the high halves of the wavefront's own rows' words, and
// works through the list 64 unions at a time: lanes with many bonds do not
// hold up the rest.  Each bond joins its site with the one `step` bytes on.
__device__ __forceinline__ void join_listed(uint32_t *s_par, uint32_t R, uint32_t step) {
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wbase = (tid >> 6) * 64u * kPS;
    const uint32_t c = __popc(R);
    uint32_t pre = 0u, nlist = 0u;
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        const uint64_t bal = __ballot((c >> j) & 1u);
        pre += (uint32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u)) << j;
        nlist += (uint32_t)__popcll(bal) << j;
    }
    uint32_t w = wbase + pre;
    while (R) {
        const uint32_t i = (uint32_t)__ffs((int)R) - 1u;
        R &= R - 1u;
        __hip_atomic_fetch_or(&s_par[w], (4u * (tid * kPS + i)) << 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        ++w;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (uint32_t k = lane; k < nlist; k += 64u) {
        const uint32_t n = lds_load(&s_par[wbase + k]) >> 16;
        __hip_atomic_fetch_and(&s_par[wbase + k], 0xFFFFu, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        lds_union_lo(s_par, n, n + step);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// =====================================================================
// k_brick3: one workgroup per brick; thread (y, z) = (tid & 15, tid >> 4)
// owns the x-row of 16 sites at (y, z), so a row's bonds and runs are 16-bit
// masks of one lane.  A site's word holds the byte offset of its run's first
// site; the +y and +z bonds (one per group that joins the same two runs)
// are unions of runs; then each run start points at its root, which collects
// the component's size and, after numbering, its node.  Brick-local indices
// order the sites of a brick as their global indices do, so a root is its
// component's smallest site.
// =====================================================================
// LOCAL: k_blocal3 comes next and sets up the nodes; else they are set up here.
template <bool POTTS, bool DENSE, bool LOCAL>
__global__ __launch_bounds__(256, kBrickWavesPerEU) void k_brick3(Dev d) {
    constexpr uint32_t NPL = POTTS ? 3u : 1u;
    __shared__ uint32_t s_par[kRows * kPS];
    __shared__ uint16_t s_pl[NPL][kRows];
    __shared__ uint16_t s_ex[kRows];
    __shared__ uint16_t s_hi[2][kBrick];  // bonds that leave through +y (by z) and +z (by y)
    __shared__ uint16_t s_in[2][kBrick];  // bonds that come in through y = 0 (by z) and z = 0 (by y)
    __shared__ uint32_t s_bf[kVol / 32];
    __shared__ uint32_t s_hist[kTileBins];
    __shared__ uint32_t s_dense[DENSE ? kDenseBins : 1];
    __shared__ int32_t s_red[kRows / 64][3];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, y = tid & 15u, z = tid >> 4;
    const Brick B = brick_of(tile_of_block(blockIdx.x, gridDim.x), d.L / kBrick);
    const uint32_t L = d.L;
    const uint32_t s0 = site_at(B, L, tid * kBrick);
    const uint32_t t = (uint32_t)*d.tdev, T = d.T;
    if (tid < kVol / 32u) s_bf[tid] = 0u;
    if (tid < kTileBins) s_hist[tid] = 0u;
    if constexpr (DENSE) s_dense[tid] = 0u;
    uint32_t pl[3];
    const Equal eq = row_equal<POTTS>(d, B, s_pl, pl);
    brick_measure<POTTS>(d, B.b, eq, pl);

    // bonds that come in through the x = 0, y = 0 and z = 0 faces, one site of
    // each face per thread: the neighbours own them, so their words are drawn
    // here a second time (3 calls beside a thread's 16), which leaves only
    // components that do go on outside as nodes -- a third of those that touch
    // the surface (228 of 640-700 per brick at the critical points)
    uint32_t in_x;
    {
        const uint32_t a = tid & 15u, c = tid >> 4;
        const uint32_t gx0 = B.x * kBrick, gy0 = B.y * kBrick, gz0 = B.z * kBrick;
        const uint32_t nx = s0 - gx0 + (gx0 == 0u ? L - 1u : gx0 - 1u);
        const uint32_t ny = ((gz0 + c) * L + (gy0 == 0u ? L - 1u : gy0 - 1u)) * L + gx0 + a;
        const uint32_t nz = ((gz0 == 0u ? L - 1u : gz0 - 1u) * L + gy0 + c) * L + gx0 + a;
        const int8_t *sp = d.spins[0];
        const uint32_t vx = (uint8_t)sp[nx], vy = (uint8_t)sp[ny], vz = (uint8_t)sp[nz];
        uint32_t dx = 0u, dy = 0u, dz = 0u;
#pragma unroll
        for (uint32_t b = 0; b < NPL; ++b) {
            const uint32_t bit = spin_bit<POTTS>(b);
            dx |= (vx >> bit) ^ pl[b];
            dy |= (vy >> bit) ^ ((uint32_t)s_pl[b][c * 16u] >> a);
            dz |= (vz >> bit) ^ ((uint32_t)s_pl[b][c] >> a);
        }
        uint32_t n[3] = {nx, ny, nz};
        bool in[3];
#pragma unroll
        for (uint32_t f = 0; f < 3u; ++f) {
            uint32_t w[4] = {n[f], t, 4u, 0u};
            philox10(w[0], w[1], w[2], w[3], d.seed_lo, d.seed_hi);
            in[f] = w[f] < T && !((f == 0u ? dx : f == 1u ? dy : dz) & 1u);
        }
        in_x = in[0] ? 1u : 0u;
        const uint64_t by = __ballot(in[1]), bz = __ballot(in[2]);
        if (a == 0u) {
            s_in[0][c] = (uint16_t)(by >> (tid & 48u));
            s_in[1][c] = (uint16_t)(bz >> (tid & 48u));
        }
    }

    // bonds (Sec. 2.1): one Philox call per site, words 0, 1, 2 of counter
    // {s, t, 4, 0} for +x, +y, +z
    uint32_t EX = 0u, EY = 0u, EZ = 0u;
#pragma unroll 4
    for (uint32_t j = 15u; j < 16u; --j) {
        uint32_t w0 = s0 + j, w1 = t, w2 = 4u, w3 = 0u;
        philox10(w0, w1, w2, w3, d.seed_lo, d.seed_hi);
        EX = shift_in_below(EX, w0, T);
        EY = shift_in_below(EY, w1, T);
        EZ = shift_in_below(EZ, w2, T);
    }
    EX &= eq.x;
    EY &= eq.y;
    EZ &= eq.z;
    const uint32_t EXi = EX & 0x7FFFu;
    const uint32_t st = ~(EXi << 1) & 0xFFFFu;  // run starts
    const uint32_t row = tid * kPS, rowoff = 4u * row;
    s_ex[tid] = (uint16_t)EXi;
    if (y == 15u) s_hi[0][z] = (uint16_t)EY;
    if (z == 15u) s_hi[1][y] = (uint16_t)EZ;
    {
        uint32_t cur = rowoff;
#pragma unroll
        for (uint32_t j = 0; j < 16u; ++j) {
            if ((st >> j) & 1u) cur = rowoff + 4u * j;
            s_par[row + j] = cur;
        }
        s_par[row + 16u] = 0u;  // pad word: list slot only
    }
    __syncthreads();
    {
        uint32_t Ry = 0u, Rz = 0u;
        if (y < 15u) {
            const uint32_t E1 = s_ex[tid + 1u];
            Ry = EY & ~((EY << 1) & (EXi << 1) & (E1 << 1));
        }
        if (z < 15u) {
            const uint32_t E1 = s_ex[tid + 16u];
            Rz = EZ & ~((EZ << 1) & (EXi << 1) & (E1 << 1));
        }
        join_listed(s_par, Ry, 4u * kPS);
        join_listed(s_par, Rz, 4u * kPS * kBrick);
    }
    __syncthreads();

    // sizes at the roots; components with a bond through the surface marked
    uint32_t rootmask = 0u;
    {
        const uint32_t linked = (EX & 0x8000u) | in_x | (y == 15u ? EY : 0u) | (z == 15u ? EZ : 0u) |
                                (y == 0u ? s_in[0][z] : 0u) | (z == 0u ? s_in[1][y] : 0u);
        uint32_t acc_root = 0u, acc_len = 0u, m = st;
        while (m) {
            const uint32_t i = (uint32_t)__ffs((int)m) - 1u;
            m &= m - 1u;
            const uint32_t n = rowoff + 4u * i;
            const uint32_t root = lds_root_b(s_par, n);
            if (root != n)
                __hip_atomic_store(word_at(s_par, n), root, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            else
                rootmask |= 1u << i;
            const uint32_t len = (m ? (uint32_t)__ffs((int)m) - 1u : kBrick) - i;
            if ((linked >> i) & ((1u << len) - 1u)) {
                const uint32_t rs = site_of(root);
                atomicOr(&s_bf[rs >> 5], 1u << (rs & 31u));
            }
            if (root != acc_root && acc_len != 0u)
                __hip_atomic_fetch_add(word_at(s_par, acc_root), acc_len << 16, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            acc_len = root != acc_root ? len : acc_len + len;
            acc_root = root;
        }
        __hip_atomic_fetch_add(word_at(s_par, acc_root), acc_len << 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __syncthreads();

    // number the marked components in site order: lane l holds the prefix of
    // mark words 2 l and 2 l + 1
    uint32_t pf_a, pf_b, n_nodes;
    {
        const uint32_t wa = s_bf[2u * lane], c = __popc(wa) + __popc(s_bf[2u * lane + 1u]);
        uint32_t incl = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t n = __shfl_up(incl, o, 64);
            if (lane >= (uint32_t)o) incl += n;
        }
        pf_a = incl - c;
        pf_b = pf_a + __popc(wa);
        n_nodes = min((uint32_t)__shfl((int)incl, 63, 64), kBrickNodes);
    }

    // roots: node into the root's word, node entries, interior-component
    // statistics (size classes 0-2 packed in 11, 10 and 11 bits: a wavefront's
    // 1024 sites may all be single)
    uint32_t max_int = 0u, sq_int = 0u, hpk = 0u;
    {
        const uint32_t sbase = tid * kBrick, word = sbase >> 5, bsh = sbase & 31u;
        const uint32_t bfw = s_bf[word], bmask = (bfw >> bsh) & 0xFFFFu;
        const uint32_t qa = (uint32_t)__shfl((int)pf_a, (int)(word >> 1), 64);
        const uint32_t qb = (uint32_t)__shfl((int)pf_b, (int)(word >> 1), 64);
        const uint32_t kbase = ((word & 1u) ? qb : qa) + __popc(bfw & ((1u << bsh) - 1u));
        while (rootmask) {
            const uint32_t i = (uint32_t)__ffs((int)rootmask) - 1u;
            rootmask &= rootmask - 1u;
            const uint32_t off = rowoff + 4u * i, S = hi16_at(s_par, off);
            uint32_t k = kNoNode;
            if ((bmask >> i) & 1u) {
                k = min(kbase + __popc(bmask & ((1u << i) - 1u)), kBrickNodes - 1u);
                const uint32_t node = B.b * kBrickNodes + k;
                d.node[node] = (sbase + i) | (S << 16);
                if constexpr (!LOCAL) {
                    d.parent[node] = node;
                    d.nsize[node] = S;
                    d.key[node] = s0 + i;
                }
            } else {
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
            s_par[off >> 2] = off | (k << 16);
        }
    }
    __syncthreads();
    if constexpr (DENSE)
        if (s_dense[tid]) atomicAdd(reinterpret_cast<unsigned long long *>(&d.dense[tid]), (unsigned long long)s_dense[tid]);
    // codes
    {
        uint32_t out[8], cur = rowoff;
#pragma unroll
        for (uint32_t j = 0; j < 16u; ++j) {
            if ((st >> j) & 1u) cur = rowoff + 4u * j;
            const uint32_t code = site_of(lo16_at(s_par, cur));
            out[j >> 1] = (j & 1u) ? out[j >> 1] | (code << 16) : code;
        }
        uint4 *cp = reinterpret_cast<uint4 *>(d.codes + (size_t)B.b * kVol + tid * kBrick);
        cp[0] = make_uint4(out[0], out[1], out[2], out[3]);
        cp[1] = make_uint4(out[4], out[5], out[6], out[7]);
    }
    // nodes of the face sites, one site of each face per thread (kNoNode on
    // the +x, +y, +z faces unless the site's bond through the face is set; on
    // the others the entry matters only where the neighbour's is set)
    {
        const uint32_t a = tid & 15u, c = tid >> 4;
        auto node_at = [&](uint32_t r, uint32_t x) {
            const uint32_t r1 = lo16_at(s_par, 4u * (r * kPS + x));
            return hi16_at(s_par, lo16_at(s_par, r1));
        };
        const uint32_t hx = node_at(tid, 15u), lx = node_at(tid, 0u);
        const uint32_t hy = node_at(c * 16u + 15u, a), ly = node_at(c * 16u, a);
        const uint32_t hz = node_at(240u + c, a), lz = node_at(c, a);
        uint16_t *fp = d.faces + (size_t)B.b * 6u * kRows + tid;
        fp[0u * kRows] = (uint16_t)((EX >> 15) & 1u ? hx : kNoNode);
        fp[1u * kRows] = (uint16_t)((s_hi[0][c] >> a) & 1u ? hy : kNoNode);
        fp[2u * kRows] = (uint16_t)((s_hi[1][c] >> a) & 1u ? hz : kNoNode);
        fp[3u * kRows] = (uint16_t)lx;
        fp[4u * kRows] = (uint16_t)ly;
        fp[5u * kRows] = (uint16_t)lz;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        hpk += __shfl_xor(hpk, o, 64);
        max_int = max(max_int, (uint32_t)__shfl_xor((int)max_int, o, 64));
        sq_int += __shfl_xor(sq_int, o, 64);
    }
    if (lane == 0u) {
        s_red[tid >> 6][0] = (int32_t)hpk;
        s_red[tid >> 6][1] = (int32_t)max_int;
        s_red[tid >> 6][2] = (int32_t)sq_int;
    }
    __syncthreads();
    if (tid == 0u) {
        int32_t mx = 0, sq = 0, h[3] = {0, 0, 0};
        for (uint32_t w = 0; w < kRows / 64u; ++w) {
            const uint32_t hw = (uint32_t)s_red[w][0];
            h[0] += (int32_t)(hw & 0x7FFu);
            h[1] += (int32_t)((hw >> 11) & 0x3FFu);
            h[2] += (int32_t)(hw >> 21);
            mx = max(mx, s_red[w][1]);
            sq += s_red[w][2];
        }
        int32_t n = h[0] + h[1] + h[2];
        int32_t *tp = d.tpart + (size_t)B.b * kTilePart;
        for (int k = 0; k < 3; ++k) tp[TP_HIST + k] = h[k];
        for (uint32_t k = 3; k < kTileBins; ++k) {
            n += (int32_t)s_hist[k];
            tp[TP_HIST + k] = (int32_t)s_hist[k];
        }
        tp[TP_N] = n;
        tp[TP_MAX] = mx;
        tp[TP_SQ] = sq;
        d.nk[0][B.b] = n_nodes;
    }
}

// Bricks of 2x2x2 group g: brick t = (lz * 2 + ly) * 2 + lx, false past the
// lattice's end (odd numbers of bricks).  Their order is that of the global
// brick indices.
__device__ __forceinline__ bool group_brick(uint32_t g, uint32_t t, uint32_t nb, uint32_t &b) {
    const uint32_t ng = (nb + 1u) / 2u, q = g / ng, gz = q / ng;
    const uint32_t x = 2u * (g - q * ng) + (t & 1u), y = 2u * (q - gz * ng) + ((t >> 1) & 1u), z = 2u * gz + (t >> 2);
    b = (z * nb + y) * nb + x;
    return x < nb && y < nb && z < nb;
}

// =====================================================================
// k_blocal3: the twelve faces inside a group of 2x2x2 bricks (half of all
// faces) join their nodes in LDS (local index = brick-in-group * kBrickNodes +
// node); every node then points at its group root, so that k_bunion3 has the
// other half of the faces left and starts it from the group roots.
// =====================================================================
constexpr uint32_t kGroupThreads = 512;

__global__ __launch_bounds__(kGroupThreads) void k_blocal3(Dev d) {
    __shared__ uint32_t s_p[8u * kBrickNodes];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wv = tid >> 6, nb = d.L / kBrick;
    const uint32_t g = tile_of_block(blockIdx.x, gridDim.x);
    // face e = 4 f + j of direction f: the j-th brick of the four on its low side
    constexpr uint32_t NIT = 12u * kRows / kGroupThreads;
    uint32_t ua[NIT], ub[NIT];
#pragma unroll
    for (uint32_t it = 0; it < NIT; ++it) {
        const uint32_t p = tid + kGroupThreads * it, e = p / kRows, i = p % kRows, f = e >> 2, j = e & 3u;
        const uint32_t ta = f == 0u ? 2u * j : f == 1u ? (j & 1u) | ((j & 2u) << 1) : j, tb = ta + (1u << f);
        uint32_t a, b;
        const bool ok = group_brick(g, ta, nb, a) & group_brick(g, tb, nb, b);
        const uint32_t na = ok ? d.faces[((size_t)a * 6u + f) * kRows + i] : kNoNode;
        const uint32_t nn = ok ? d.faces[((size_t)b * 6u + 3u + f) * kRows + i] : 0u;
        ua[it] = na == kNoNode ? kEmpty : ta * kBrickNodes + na;
        ub[it] = tb * kBrickNodes + nn;
    }
    uint32_t bw;
    const bool okw = group_brick(g, wv, nb, bw);
    const uint32_t nk = okw ? min(d.nk[0][bw], kBrickNodes) : 0u;
    for (uint32_t k = lane; k < nk; k += 64u) s_p[wv * kBrickNodes + k] = wv * kBrickNodes + k;
    constexpr uint32_t kAhead = 5;  // node entries loaded before the unions (320 per brick)
    uint32_t ahead[kAhead];
#pragma unroll
    for (uint32_t j = 0; j < kAhead; ++j) ahead[j] = lane + 64u * j < nk ? d.node[bw * kBrickNodes + lane + 64u * j] : 0u;
    __syncthreads();
#pragma unroll
    for (uint32_t it = 0; it < NIT; ++it) {
        const uint32_t a = ua[it], b = ub[it];
        const uint32_t pa = __shfl_up(a, 1, 64), pb = __shfl_up(b, 1, 64);
        const bool dup = lane > 0u && pa == a && pb == b;
        if (a != kEmpty && !dup) lds_union(s_p, a, b);
    }
    __syncthreads();
    const Brick B = brick_of(bw, nb);
    auto settle = [&](uint32_t k, uint32_t e) {
        const uint32_t li = wv * kBrickNodes + k, node = bw * kBrickNodes + k;
        const uint32_t r = lds_find(s_p, li), tr = r / kBrickNodes;
        uint32_t br;
        group_brick(g, tr, nb, br);
        d.parent[node] = br * kBrickNodes + (r - tr * kBrickNodes);
        if (r == li) {  // only a group root can be a cluster's root
            d.nsize[node] = e >> 16;
            d.key[node] = site_at(B, d.L, e & 0xFFFFu);
        }
    };
#pragma unroll
    for (uint32_t j = 0; j < kAhead; ++j)
        if (lane + 64u * j < nk) settle(lane + 64u * j, ahead[j]);
    for (uint32_t k = lane + 64u * kAhead; k < nk; k += 64u) settle(k, d.node[bw * kBrickNodes + k]);
}

// =====================================================================
// k_bunion3: the faces between groups, one workgroup per face: direction
// blockIdx.y, the low side in brick layer min(2 j + 1, nb - 1); with layers = nb
// all faces, the low side in layer j.  Unions start
// from the nodes' parents; a bond that joins the same two as the bond of the
// lane below is skipped.
// =====================================================================
__global__ __launch_bounds__(256) void k_bunion3(Dev d, uint32_t layers) {
    const uint32_t nb = d.L / kBrick, f = blockIdx.y, i = threadIdx.x;
    uint32_t p = tile_of_block(blockIdx.x, gridDim.x);
    // the layer is the slowest coordinate but one, so that consecutive
    // workgroups take neighbouring bricks
    const uint32_t u = p % nb, q = p / nb, v = q % nb, j = q / nb;
    const uint32_t c = layers == nb ? j : min(2u * j + 1u, nb - 1u), c1 = c + 1u == nb ? 0u : c + 1u;
    uint32_t A, Bn;
    if (f == 0u) {
        A = (v * nb + u) * nb + c;
        Bn = (v * nb + u) * nb + c1;
    } else if (f == 1u) {
        A = (v * nb + c) * nb + u;
        Bn = (v * nb + c1) * nb + u;
    } else {
        A = (c * nb + v) * nb + u;
        Bn = (c1 * nb + v) * nb + u;
    }
    const uint32_t na = d.faces[((size_t)A * 6u + f) * kRows + i], nn = d.faces[((size_t)Bn * 6u + 3u + f) * kRows + i];
    const bool has = na != kNoNode;
    uint32_t *par = d.parent;
    const uint32_t ra = has ? g_load(&par[A * kBrickNodes + na]) : kEmpty;
    const uint32_t rb = has ? g_load(&par[Bn * kBrickNodes + nn]) : 0u;
    const uint32_t pa = __shfl_up(ra, 1, 64), pb = __shfl_up(rb, 1, 64);
    const bool dup = (i & 63u) != 0u && pa == ra && pb == rb;
    if (has && !dup) g_union(par, ra, rb);
}

// =====================================================================
// k_bflat3: every node points at its root; sizes and keys into the roots,
// gathered per workgroup (a group of eight bricks, one per wavefront, or one
// brick) in an LDS hash, then one global atomic of each kind per (workgroup,
// root).
// =====================================================================
constexpr uint32_t kHash = 2048;

template <bool GROUP>
__global__ __launch_bounds__(kGroupThreads) void k_bflat3(Dev d) {
    __shared__ uint32_t hk[kHash], hv[kHash], hm[kHash];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wv = tid >> 6;
    for (uint32_t i = tid; i < kHash; i += kGroupThreads) {
        hk[i] = kEmpty;
        hv[i] = 0u;
        hm[i] = kEmpty;
    }
    __syncthreads();
    uint32_t *par = d.parent;
    uint32_t b = blockIdx.x;
    const bool ok = !GROUP || group_brick(tile_of_block(blockIdx.x, gridDim.x), wv, d.L / kBrick, b);
    const uint32_t nk = ok ? min(d.nk[0][b], kBrickNodes) : 0u;
    const uint32_t node0 = b * kBrickNodes;
    const Brick B = brick_of(b, d.L / kBrick);
    constexpr uint32_t kChase = 4, STEP = GROUP ? 64u : kGroupThreads;
    for (uint32_t k0 = GROUP ? 0u : 64u * wv; k0 < nk; k0 += STEP * kChase) {
        // up to four nodes per lane, their chains followed together
        uint32_t p0[kChase], r[kChase], en[kChase];
#pragma unroll
        for (uint32_t j = 0; j < kChase; ++j) {
            const uint32_t k = k0 + STEP * j + lane;
            p0[j] = k < nk ? g_load(&par[node0 + k]) : kEmpty;
            en[j] = k < nk ? d.node[node0 + k] : 0u;
        }
#pragma unroll
        for (uint32_t j = 0; j < kChase; ++j) r[j] = p0[j];
        bool more = true;
        while (more) {
            uint32_t p[kChase];
#pragma unroll
            for (uint32_t j = 0; j < kChase; ++j) p[j] = r[j] != kEmpty ? g_load(&par[r[j]]) : kEmpty;
            more = false;
#pragma unroll
            for (uint32_t j = 0; j < kChase; ++j) {
                more |= p[j] != r[j];
                r[j] = p[j];
            }
        }
#pragma unroll
        for (uint32_t j = 0; j < kChase; ++j) {
            const uint32_t node = node0 + k0 + STEP * j + lane, root = r[j];
            if (root == kEmpty || root == node) continue;
            if (root != p0[j]) g_store(&par[node], root);
            const uint32_t e = en[j], size = e >> 16, key = site_at(B, d.L, e & 0xFFFFu);
            uint32_t h = (root * 2654435761u) >> 21;  // 11 bits
            bool placed = false;
            for (int probe = 0; probe < 64 && !placed; ++probe) {
                uint32_t cur = lds_load(&hk[h]);
                if (cur == kEmpty) {
                    const uint32_t old = atomicCAS(&hk[h], kEmpty, root);
                    cur = old == kEmpty ? root : old;
                }
                if (cur == root) {
                    atomicAdd(&hv[h], size);
                    atomicMin(&hm[h], key);
                    placed = true;
                }
                h = (h + 1u) & (kHash - 1u);
            }
            if (!placed) {
                atomicAdd(&d.nsize[root], size);
                if (key < g_load(&d.key[root])) atomicMin(&d.key[root], key);
            }
        }
    }
    __syncthreads();
    // the current keys of a thread's roots are read before any atomic
    constexpr uint32_t kPer = kHash / kGroupThreads;
    uint32_t fk[kPer], fm[kPer];
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) fk[j] = hk[tid + kGroupThreads * j];
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) fm[j] = fk[j] != kEmpty ? g_load(&d.key[fk[j]]) : 0u;
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
        if (fk[j] == kEmpty) continue;
        const uint32_t i = tid + kGroupThreads * j;
        atomicAdd(&d.nsize[fk[j]], hv[i]);
        if (hm[i] < fm[j]) atomicMin(&d.key[fk[j]], hm[i]);
    }
}

// =====================================================================
// k_bspin3: one workgroup per brick.  A table by code holds every
// component's new spin: each thread draws what the 16 sites of its row would
// give their components as roots (a Philox call per row, Ising, or four,
// Potts), the nodes' entries are then replaced by their clusters' draws; the
// codes are looked up and the spins written in place.  Statistics of the
// clusters rooted in the brick and of its interior components -> the brick's
// group partial.
// =====================================================================
template <bool POTTS, bool DENSE>
__global__ __launch_bounds__(256) void k_bspin3(Dev d) {
    __shared__ __align__(16) uint8_t s_tab[kVol];
    __shared__ uint32_t s_hist[33];
    __shared__ uint64_t s_red[kRows / 64][3];
    __shared__ uint32_t s_dense[DENSE ? kDenseBins : 1];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, L = d.L;
    const Brick B = brick_of(tile_of_block(blockIdx.x, gridDim.x), L / kBrick);
    const uint32_t s0 = site_at(B, L, tid * kBrick);
    const uint32_t t = (uint32_t)*d.tdev;
    const uint4 *cp = reinterpret_cast<const uint4 *>(d.codes + (size_t)B.b * kVol + tid * kBrick);
    const uint4 c0 = cp[0], c1 = cp[1];
    const uint32_t nk = min(d.nk[0][B.b], kBrickNodes);
    // the first round's node entries (a brick rarely has more than 256 nodes)
    const uint32_t *par = d.parent;
    const uint32_t mine = B.b * kBrickNodes + tid;
    const uint32_t root0 = tid < nk ? par[mine] : 0u, site0 = tid < nk ? d.node[mine] : 0u;
    const uint32_t key0 = tid < nk ? d.key[root0] : 0u;
    if (tid < 33u) s_hist[tid] = 0u;
    if constexpr (DENSE) s_dense[tid] = 0u;
    {
        uint32_t out[4];
        if constexpr (POTTS) {
#pragma unroll
            for (uint32_t j = 0; j < 4u; ++j) {  // value i of word i for site 4 j + i (s0 is a multiple of 16)
                uint32_t w0 = (s0 >> 2) + j, w1 = t, w2 = 3u, w3 = 0u;
                philox10(w0, w1, w2, w3, d.seed_lo, d.seed_hi);
                const uint32_t q = d.q;
                out[j] = (uint32_t)(((uint64_t)w0 * q) >> 32) | ((uint32_t)(((uint64_t)w1 * q) >> 32) << 8) |
                         ((uint32_t)(((uint64_t)w2 * q) >> 32) << 16) | ((uint32_t)(((uint64_t)w3 * q) >> 32) << 24);
            }
        } else {  // the row's 16 bits lie in one word of one 128-site block
            uint32_t w0 = s0 >> 7, w1 = t, w2 = 1u, w3 = 0u;
            philox10(w0, w1, w2, w3, d.seed_lo, d.seed_hi);
            const uint32_t q = (s0 >> 5) & 3u;
            const uint32_t w = (q == 0 ? w0 : q == 1 ? w1 : q == 2 ? w2 : w3) >> (s0 & 31u);
#pragma unroll
            for (uint32_t j = 0; j < 4u; ++j) {
                out[j] = 0u;
#pragma unroll
                for (uint32_t i = 0; i < 4u; ++i) out[j] |= ((w >> (4u * j + i)) & 1u ? 0xFFu : 0x01u) << (8u * i);
            }
        }
        *reinterpret_cast<uint4 *>(s_tab + tid * kBrick) = make_uint4(out[0], out[1], out[2], out[3]);
    }
    __syncthreads();
    uint64_t n = 0, mx = 0, sq = 0;
    for (uint32_t k = tid; k < nk; k += kRows) {
        const uint32_t node = B.b * kBrickNodes + k;
        const uint32_t root = k == tid ? root0 : par[node], rkey = k == tid ? key0 : d.key[root];
        const uint32_t site = k == tid ? site0 : d.node[node];
        s_tab[site & (kVol - 1u)] = (uint8_t)(POTTS ? potts_spin(rkey, t, d.q, d.seed_lo, d.seed_hi)
                                               : cluster_spin(rkey, t, d.seed_lo, d.seed_hi));
        if (root == node) {
            const uint32_t S = d.nsize[node];
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
    __syncthreads();
    {
        const uint32_t c[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
        uint32_t out[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (uint32_t j = 0; j < 16u; ++j)
            out[j >> 2] |= (uint32_t)s_tab[(c[j >> 1] >> (16u * (j & 1u))) & (kVol - 1u)] << (8u * (j & 3u));
        *reinterpret_cast<uint4 *>(d.spins[0] + s0) = make_uint4(out[0], out[1], out[2], out[3]);
    }
    if constexpr (DENSE)
        if (s_dense[tid]) atomicAdd(reinterpret_cast<unsigned long long *>(&d.dense[tid]), (unsigned long long)s_dense[tid]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        n += __shfl_xor(n, o, 64);
        mx = max(mx, (uint64_t)__shfl_xor((unsigned long long)mx, o, 64));
        sq += __shfl_xor(sq, o, 64);
    }
    if (lane == 0u) {
        s_red[tid >> 6][0] = n;
        s_red[tid >> 6][1] = mx;
        s_red[tid >> 6][2] = sq;
    }
    __syncthreads();
    const int32_t *tp = d.tpart + (size_t)B.b * kTilePart;
    uint64_t *gp = d.gpart + (size_t)B.b * kGroupPart;
    if (tid == 0u) {
        uint64_t a = (uint32_t)tp[TP_N], b = (uint32_t)tp[TP_MAX], c = (uint32_t)tp[TP_SQ];
        for (uint32_t w = 0; w < kRows / 64u; ++w) {
            a += s_red[w][0];
            b = max(b, s_red[w][1]);
            c += s_red[w][2];
        }
        gp[GP_N] = a;
        gp[GP_MAX] = b;
        gp[GP_SQ] = c;
        gp[GP_E] = (uint64_t)(int64_t)tp[TP_E];
        gp[GP_M] = (uint64_t)(int64_t)tp[TP_M];
    }
    if (tid < 33u) gp[GP_HIST + tid] = s_hist[tid] + (tid < kTileBins ? (uint32_t)tp[TP_HIST + tid] : 0u);
    if (tid < (uint32_t)kMaxQ) gp[GP_CNT + tid] = POTTS ? (uint32_t)tp[TP_CNT + tid] : 0u;
}

// Energy and magnetisation of the configuration a call's last sweep left.
template <bool POTTS>
__global__ __launch_bounds__(256) void k_bmeasure3(Dev d) {
    __shared__ uint16_t s_pl[POTTS ? 3 : 1][kRows];
    const Brick B = brick_of(tile_of_block(blockIdx.x, gridDim.x), d.L / kBrick);
    uint32_t pl[3];
    const Equal eq = row_equal<POTTS>(d, B, s_pl, pl);
    brick_measure<POTTS>(d, B.b, eq, pl);
}

// Canonical labels of the last sweep, from its codes and nodes.
__global__ __launch_bounds__(256) void k_blabels3(Dev d) {
    __shared__ uint32_t s_lab[kVol];
    const uint32_t tid = threadIdx.x, L = d.L;
    const Brick B = brick_of(tile_of_block(blockIdx.x, gridDim.x), L / kBrick);
    const uint32_t s0 = site_at(B, L, tid * kBrick);
    for (uint32_t j = 0; j < 16u; ++j) s_lab[tid * kBrick + j] = s0 + j;
    __syncthreads();
    const uint32_t nk = min(d.nk[0][B.b], kBrickNodes);
    for (uint32_t k = tid; k < nk; k += kRows) {
        const uint32_t node = B.b * kBrickNodes + k;
        s_lab[d.node[node] & (kVol - 1u)] = d.key[d.parent[node]];
    }
    __syncthreads();
    const uint16_t *cp = d.codes + (size_t)B.b * kVol + tid * kBrick;
    for (uint32_t j = 0; j < 16u; ++j) d.labels[s0 + j] = s_lab[cp[j] & (kVol - 1u)];
}

// Whether a lattice of nb bricks a side leaves out k_blocal3 and flattens with a
// workgroup per brick: all faces' unions go to k_bunion3, where so few nodes
// are in nobody's way, and a launch of one workgroup per eight bricks is a chain
// of loads on an idle GPU (k_blocal3 9 us and k_bflat3 10 of the 53 us of 64^3 at
// beta = 0.1).  us per sweep with k_blocal3 / without: 32^3, beta = 0.1, 47.3 /
// 37.7, 64^3 53.1 / 40.1, 80^3 51.7 / 41.2; 64^3, 3-state at 0.5505, 72.0 / 53.5.
// In the ordered phase (bond probabilities from about the one below, which is
// 0.366 for Ising, 0.430, 0.473, 0.533 and 0.572 for q = 3, 4, 6 and 8) the
// group-local unions keep a giant cluster's links and atomics apart, and the line
// lies lower: beta = 0.3, 80^3 81.8 / 75.6, 96^3 86.1 / 93.8, 144^3 130 / 158;
// beta = 0.2, 96^3 72.0 / 53.6; 96^3 with q = 6 at 0.75, 68.1 / 51.7.
bool few_bricks(const Dev &d, uint32_t nb) {
    const double q = d.q ? d.q : 2u, p = sqrt(q) / (sqrt(q) + 2.0 + 0.9 / q);
    return nb <= ((double)d.T > p * 4294967296.0 ? 5u : 6u);
}

template <bool LOCAL> void launch_brick3(const Dev &d, uint32_t n, hipStream_t s) {
    if (d.dense) {
        if (d.q)
            k_brick3<true, true, LOCAL><<<n, 256, 0, s>>>(d);
        else
            k_brick3<false, true, LOCAL><<<n, 256, 0, s>>>(d);
    } else if (d.q) {
        k_brick3<true, false, LOCAL><<<n, 256, 0, s>>>(d);
    } else {
        k_brick3<false, false, LOCAL><<<n, 256, 0, s>>>(d);
    }
}

}  // namespace

hipError_t launch_brick_stage(const Dev &d, int stage, hipStream_t s) {
    const uint32_t nb = d.L / kBrick, n = nb * nb * nb, ng = (nb + 1u) / 2u;
    const bool few = few_bricks(d, nb);
    switch (stage) {
    case 0:
        if (few)
            launch_brick3<false>(d, n, s);
        else
            launch_brick3<true>(d, n, s);
        break;
    case 1:
        if (!few) k_blocal3<<<ng * ng * ng, kGroupThreads, 0, s>>>(d);
        k_bunion3<<<dim3((few ? nb : ng) * nb * nb, 3), 256, 0, s>>>(d, few ? nb : ng);
        break;
    case 2:
        if (few)
            k_bflat3<false><<<n, kGroupThreads, 0, s>>>(d);
        else
            k_bflat3<true><<<ng * ng * ng, kGroupThreads, 0, s>>>(d);
        break;
    case 3:
        if (d.dense) {
            if (d.q)
                k_bspin3<true, true><<<n, 256, 0, s>>>(d);
            else
                k_bspin3<false, true><<<n, 256, 0, s>>>(d);
        } else if (d.q) {
            k_bspin3<true, false><<<n, 256, 0, s>>>(d);
        } else {
            k_bspin3<false, false><<<n, 256, 0, s>>>(d);
        }
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_brick_measure(const Dev &d, hipStream_t s) {
    if (d.q)
        k_bmeasure3<true><<<d.ngroups, 256, 0, s>>>(d);
    else
        k_bmeasure3<false><<<d.ngroups, 256, 0, s>>>(d);
    return hipGetLastError();
}

hipError_t launch_brick_labels(const Dev &d, hipStream_t s) {
    k_blabels3<<<d.ngroups, 256, 0, s>>>(d);
    return hipGetLastError();
}

}  // namespace swmi
