// sw_phi4.hip -- the O(4) phi^4 theory on the L^4 periodic lattice (paper
// Sec. 3): one multicluster update of the Wolff embedding per sweep.
//
// Fields are unit 4-vectors (the self-coupling lambda and the radial update
// are not given in the paper; with |phi| = 1, the lambda -> infinity limit,
// the cluster update alone samples exp(2 kappa sum_<xy> phi_x . phi_y)).
// A sweep t:
//   k_phi_bond    the sweep's random direction r (unnormalised, drawn by
//                 4-ball rejection from Philox({k, t, 5, 0})); link (x, mu) is
//                 bonded (eq. 2) iff a = ((p_x p_y) 4 kappa) / (r . r) > 0,
//                 p the projections on r, and its word (word mu of
//                 Philox({x, t, 7, 0})) times 2^-32 is below 1 - E(a); bonded
//                 sites of one chunk of kPhiChunk consecutive sites are
//                 joined in LDS
//   k_phi_union   bonds between chunks join the chunks' local roots by the
//                 lock-free union-find of sw_uf.h (smaller index is root)
//   k_phi_flat    every site points at its root (the cluster's smallest
//                 site); the local components' sizes are added at the roots;
//                 a cluster whose root's Philox bit ({root >> 7, t, 6, 0},
//                 bit root mod 128) is set is reflected (eq. 3):
//                 phi -= ((2 p_x) / (r . r)) r
//   k_phi_record  exact int64 sums of rint(2^32 phi_x . phi_y) over links and
//                 of rint(2^32 phi_x^a), cluster statistics at the roots;
//                 the last workgroup writes the sweep's record
// Every floating-point value is an IEEE double produced by one correctly
// rounded operation at a time in the order written (no multiply-add is
// contracted in this file), so the results are a function of the inputs
// alone, and equal to any other evaluation in the same order.
#pragma clang fp contract(off)

#include <math.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <new>
#include <string>

#include "sw_host.h"
#include "sw_philox.h"
#include "sw_uf.h"

namespace swmi {
namespace {

constexpr int kPhiBlock = 256;
// Sites per workgroup (one per thread) whose bonds are joined in LDS.  A sweep
// is bound by its chains of dependent loads and atomics, not by its 400 B per
// site: joining every bond in global memory, counting sizes with an atomic
// per wavefront and root, and summing the record with 42 atomics and two
// cache fences per 256 sites took 28 + 20 + 42 us at 20^4, kappa = 0.304;
// local components first leave about a third of the bonds and one size per
// component to the global steps: bond 10, union 15, flat with reflection 7,
// record 13 us; 117 -> 57 us an update with its launches.
constexpr uint32_t kPhiChunk = 1024;
constexpr uint32_t kPhiRecGroups = 512;  // most workgroups of k_phi_record (2 per CU)
constexpr int kPhiMaxL = 64;
constexpr double kPhiMaxKappa = 4.0;
// accumulator words: e, m[4], n, max, sum_sq, hist[33], completion counter
enum { PA_E = 0, PA_M = 1, PA_N = 5, PA_MAX = 6, PA_SQ = 7, PA_HIST = 8, PA_END = 41 };
constexpr int kPhiPart = 48;  // words of a workgroup's partial

struct PhiDev {
    double *phi;      // [N][4] fields
    uint32_t *parent; // [N] union-find parents, then roots (labels)
    uint32_t *csize;  // [N] size of the chunk's component at local roots, 0 elsewhere; then cluster sizes at roots
    uint8_t *cross;   // [N] bit mu: the link to x + mu-hat is bonded and leaves the chunk
    double *dir;      // [8] r[4], r . r of the current sweep
    uint64_t *part;   // [kPhiRecGroups][kPhiPart] partial records
    uint64_t *acc;    // [0] workgroups of k_phi_record done
    uint64_t *tdev;   // [0] index of the next sweep
    sw_phi4_obs *ring;
    uint32_t L, N, ring_cap, seed_lo, seed_hi;
    double kappa;
};

__device__ __forceinline__ double phi_uniform(uint32_t w) { return ((double)w + 0.5) * 0x1p-31 - 1.0; }

__device__ __forceinline__ double dot4(double a0, double a1, double a2, double a3, double b0, double b1, double b2,
                                       double b3) {
    return ((a0 * b0 + a1 * b1) + a2 * b2) + a3 * b3;
}

// The sweep's random direction: the first of 64 candidates
// (Philox({k, t, 5, 0}) as four uniforms in (-1, 1)) inside the unit ball;
// (1, 0, 0, 0) if none is.  Lane k of the wavefront draws candidate k.
__device__ __forceinline__ void phi_direction(uint32_t t, uint32_t k0, uint32_t k1, double r[4], double &rr) {
    uint32_t w0 = threadIdx.x & 63u, w1 = t, w2 = 5u, w3 = 0u;
    philox10(w0, w1, w2, w3, k0, k1);
    const double v[4] = {phi_uniform(w0), phi_uniform(w1), phi_uniform(w2), phi_uniform(w3)};
    const double vv = dot4(v[0], v[1], v[2], v[3], v[0], v[1], v[2], v[3]);
    const uint64_t in = __ballot(vv < 1.0);
    const int first = in ? __ffsll((unsigned long long)in) - 1 : 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = in ? __shfl(v[i], first, 64) : i == 0 ? 1.0 : 0.0;
    rr = in ? __shfl(vv, first, 64) : 1.0;
}

// exp(-a) for the bond test: halve a to at most 1/8 (k times), Taylor
// polynomial of degree 13 in Horner form with rounded 1/j, square k times.
__device__ __forceinline__ double phi_expm(double a) {
    double b = a;
    int k = 0;
    while (b > 0.125) {
        b = b * 0.5;
        ++k;
    }
    double q = 1.0;
#pragma unroll
    for (int j = 13; j >= 1; --j) q = 1.0 - (q * b) * (1.0 / (double)j);
    for (int i = 0; i < k; ++i) q = q * q;
    return q;
}

// x + mu-hat, mu = 0..3, on the periodic L^4 lattice (x_0 fastest)
__device__ __forceinline__ void phi_neighbours(uint32_t x, uint32_t L, uint32_t nb[4]) {
    uint32_t rest = x, stride = 1u;
#pragma unroll
    for (uint32_t mu = 0; mu < 4u; ++mu) {
        const uint32_t q = rest / L, c = rest - q * L;
        nb[mu] = c + 1u == L ? x - c * stride : x + stride;
        rest = q;
        stride *= L;
    }
}

__global__ __launch_bounds__(kPhiBlock) void k_phi_init(PhiDev d, int cold) {
    const uint32_t x = blockIdx.x * kPhiBlock + threadIdx.x;
    if (x >= d.N) return;
    double f0 = 1.0, f1 = 0.0, f2 = 0.0, f3 = 0.0;
    if (!cold) {
        for (uint32_t k = 0; k < 64u; ++k) {
            uint32_t w0 = x, w1 = k, w2 = 8u, w3 = 0u;
            philox10(w0, w1, w2, w3, d.seed_lo, d.seed_hi);
            const double v0 = phi_uniform(w0), v1 = phi_uniform(w1), v2 = phi_uniform(w2), v3 = phi_uniform(w3);
            const double vv = dot4(v0, v1, v2, v3, v0, v1, v2, v3);
            if (vv < 1.0) {
                const double len = sqrt(vv);
                f0 = v0 / len;
                f1 = v1 / len;
                f2 = v2 / len;
                f3 = v3 / len;
                break;
            }
        }
    }
    double4 *p = reinterpret_cast<double4 *>(d.phi);
    p[x] = make_double4(f0, f1, f2, f3);
}

__global__ __launch_bounds__(kPhiChunk) void k_phi_bond(PhiDev d) {
    __shared__ uint32_t s_par[kPhiChunk];
    __shared__ uint32_t s_cnt[kPhiChunk];
    const uint32_t tid = threadIdx.x, base = blockIdx.x * kPhiChunk, x = base + tid;
    const bool valid = x < d.N;
    const uint32_t t = (uint32_t)*d.tdev;
    const uint32_t xs = valid ? x : 0u;  // past the lattice: site 0, bonds ignored
    const double4 *p = reinterpret_cast<const double4 *>(d.phi);
    uint32_t nb[4];
    phi_neighbours(xs, d.L, nb);
    const double4 f = p[xs];
    double4 g[4];
#pragma unroll
    for (uint32_t mu = 0; mu < 4u; ++mu) g[mu] = p[nb[mu]];
    s_par[tid] = tid;
    s_cnt[tid] = 0u;
    double r[4], rr;
    phi_direction(t, d.seed_lo, d.seed_hi, r, rr);
    if (x == 0u) {
        d.dir[0] = r[0];
        d.dir[1] = r[1];
        d.dir[2] = r[2];
        d.dir[3] = r[3];
        d.dir[4] = rr;
    }
    uint32_t w[4] = {x, t, 7u, 0u};
    philox10(w[0], w[1], w[2], w[3], d.seed_lo, d.seed_hi);
    const double k4 = 4.0 * d.kappa;
    const double px = dot4(f.x, f.y, f.z, f.w, r[0], r[1], r[2], r[3]);
    uint32_t bonds = 0u;
#pragma unroll
    for (uint32_t mu = 0; mu < 4u; ++mu) {
        const double py = dot4(g[mu].x, g[mu].y, g[mu].z, g[mu].w, r[0], r[1], r[2], r[3]);
        const double a = ((px * py) * k4) / rr;
        if (a > 0.0) {
            const double u = (double)w[mu] * 0x1p-32;
            if (u < 1.0 - phi_expm(a)) bonds |= 1u << mu;
        }
    }
    if (!valid) bonds = 0u;
    __syncthreads();
    uint32_t cross = 0u;
#pragma unroll
    for (uint32_t mu = 0; mu < 4u; ++mu) {
        if (!((bonds >> mu) & 1u)) continue;
        const uint32_t y = nb[mu] - base;
        if (y < kPhiChunk)
            lds_union(s_par, tid, y);
        else
            cross |= 1u << mu;
    }
    __syncthreads();
    const uint32_t root = lds_find(s_par, tid);
    // sizes: one add per run of lanes with the same root
    const uint32_t lane = tid & 63u;
    const uint32_t prev = __shfl_up(root, 1, 64);
    const uint64_t starts = __ballot(lane == 0u || prev != root);
    if ((starts >> lane) & 1u) {
        const uint64_t later = lane == 63u ? 0ull : starts >> (lane + 1u);
        const uint32_t len = later ? (uint32_t)__ffsll((unsigned long long)later) : 64u - lane;
        atomicAdd(&s_cnt[root], len);
    }
    __syncthreads();
    if (!valid) return;
    d.parent[x] = base + root;
    d.csize[x] = s_cnt[tid];
    d.cross[x] = (uint8_t)cross;
}

// One thread per site and direction (blockIdx.y) with a bond that leaves its
// chunk, so that a site's unions run beside each other instead of one after
// the other (17.0 -> 14.6 us at 20^4, kappa = 0.304).  Every union starts
// from the two sites' local roots; a bond that joins the same two as the bond
// of the lane below is skipped.
__global__ __launch_bounds__(kPhiBlock) void k_phi_union(PhiDev d) {
    const uint32_t x = blockIdx.x * kPhiBlock + threadIdx.x, mu = blockIdx.y;
    const bool has = x < d.N && ((d.cross[x] >> mu) & 1u);
    if (__ballot(has) == 0ull) return;
    uint32_t nb[4];
    phi_neighbours(has ? x : 0u, d.L, nb);
    const uint32_t y = mu == 0u ? nb[0] : mu == 1u ? nb[1] : mu == 2u ? nb[2] : nb[3];
    const uint32_t ra = has ? g_load(&d.parent[x]) : 0u, rb = has ? g_load(&d.parent[y]) : 0u;
    const uint32_t pa = __shfl_up(ra, 1, 64), pb = __shfl_up(rb, 1, 64);
    const int ph = __shfl_up((int)has, 1, 64);
    const bool dup = (threadIdx.x & 63u) != 0u && ph && pa == ra && pb == rb;
    if (has && !dup) g_union(d.parent, ra, rb);
}

// The local components' sizes are gathered per workgroup in an LDS hash (at
// most one entry per thread, so a free slot is always found) and added with
// one atomic per workgroup and root.
__global__ __launch_bounds__(kPhiChunk) void k_phi_flat(PhiDev d) {
    constexpr uint32_t kNone = 0xFFFFFFFFu;
    __shared__ uint32_t s_key[kPhiChunk];
    __shared__ uint32_t s_val[kPhiChunk];
    const uint32_t tid = threadIdx.x, x = blockIdx.x * kPhiChunk + tid;
    const bool valid = x < d.N;
    const uint32_t t = (uint32_t)*d.tdev;
    s_key[tid] = kNone;
    s_val[tid] = 0u;
    const uint32_t p0 = valid ? g_load(&d.parent[x]) : 0u;
    double4 *p = reinterpret_cast<double4 *>(d.phi);
    const double4 f = p[valid ? x : 0u];
    const double r0 = d.dir[0], r1 = d.dir[1], r2 = d.dir[2], r3 = d.dir[3], rr = d.dir[4];
    uint32_t root = p0;
    if (valid) {
        while (true) {
            const uint32_t q = g_load(&d.parent[root]);
            if (q == root) break;
            root = q;
        }
        if (root != p0) g_store(&d.parent[x], root);
    }
    __syncthreads();  // the hash is clear
    // a component that is not its cluster's root holds its own size alone
    const uint32_t size = valid && root != x ? d.csize[x] : 0u;
    if (size) {
        uint32_t h = (root * 2654435761u) >> 22;
        static_assert(kPhiChunk == 1024u, "ten hash bits");
        while (true) {
            const uint32_t old = atomicCAS(&s_key[h], kNone, root);
            if (old == kNone || old == root) break;
            h = (h + 1u) & (kPhiChunk - 1u);
        }
        atomicAdd(&s_val[h], size);
    }
    if (valid) {
        uint32_t w0 = root >> 7, w1 = t, w2 = 6u, w3 = 0u;
        philox10(w0, w1, w2, w3, d.seed_lo, d.seed_hi);
        const uint32_t q = (root >> 5) & 3u;
        const uint32_t w = q == 0 ? w0 : q == 1 ? w1 : q == 2 ? w2 : w3;
        if ((w >> (root & 31u)) & 1u) {
            const double c = (2.0 * dot4(f.x, f.y, f.z, f.w, r0, r1, r2, r3)) / rr;
            p[x] = make_double4(f.x - c * r0, f.y - c * r1, f.z - c * r2, f.w - c * r3);
        }
    }
    __syncthreads();
    if (s_key[tid] != kNone) atomicAdd(&d.csize[s_key[tid]], s_val[tid]);
}

__device__ __forceinline__ int64_t fix32(double v) { return (int64_t)rint(v * 0x1p32); }

// Workgroup partials go out as agent-scope stores, every wavefront waits for
// its own to complete before its workgroup counts itself in, and the last
// workgroup folds them with agent-scope loads (no cache fences).
__global__ __launch_bounds__(kPhiChunk) void k_phi_record(PhiDev d) {
    constexpr uint32_t NW = kPhiChunk / 64u;
    __shared__ uint32_t s_hist[33];
    __shared__ int64_t s_red[NW][8];
    __shared__ unsigned long long s_tot[PA_END];
    __shared__ int s_last;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wv = tid >> 6;
    if (tid < 33u) s_hist[tid] = 0u;
    if (tid < (uint32_t)PA_END) s_tot[tid] = 0ull;
    __syncthreads();
    int64_t e = 0, m0 = 0, m1 = 0, m2 = 0, m3 = 0;
    uint64_t n = 0, mx = 0, sq = 0;
    for (uint32_t x = blockIdx.x * kPhiChunk + tid; x < d.N; x += gridDim.x * kPhiChunk) {
        const double4 *p = reinterpret_cast<const double4 *>(d.phi);
        uint32_t nb[4];
        phi_neighbours(x, d.L, nb);
        const double4 f = p[x];
        double4 g[4];
#pragma unroll
        for (uint32_t mu = 0; mu < 4u; ++mu) g[mu] = p[nb[mu]];
        const uint32_t par = d.parent[x];
        const uint64_t S = d.csize[x];
#pragma unroll
        for (uint32_t mu = 0; mu < 4u; ++mu)
            e += fix32(dot4(f.x, f.y, f.z, f.w, g[mu].x, g[mu].y, g[mu].z, g[mu].w));
        m0 += fix32(f.x);
        m1 += fix32(f.y);
        m2 += fix32(f.z);
        m3 += fix32(f.w);
        if (par == x) {
            n += 1u;
            mx = max(mx, S);
            sq += S * S;
            atomicAdd(&s_hist[63 - __clzll((long long)S)], 1u);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        e += __shfl_xor(e, o, 64);
        m0 += __shfl_xor(m0, o, 64);
        m1 += __shfl_xor(m1, o, 64);
        m2 += __shfl_xor(m2, o, 64);
        m3 += __shfl_xor(m3, o, 64);
        n += __shfl_xor(n, o, 64);
        mx = max(mx, (uint64_t)__shfl_xor((unsigned long long)mx, o, 64));
        sq += __shfl_xor(sq, o, 64);
    }
    if (lane == 0u) {
        s_red[wv][0] = e;
        s_red[wv][1] = m0;
        s_red[wv][2] = m1;
        s_red[wv][3] = m2;
        s_red[wv][4] = m3;
        s_red[wv][5] = (int64_t)n;
        s_red[wv][6] = (int64_t)mx;
        s_red[wv][7] = (int64_t)sq;
    }
    __syncthreads();
    if (tid < (uint32_t)PA_END) {
        int64_t v = 0;
        if (tid < 8u) {
            for (uint32_t w = 0; w < NW; ++w) v = tid == (uint32_t)PA_MAX ? max(v, s_red[w][tid]) : v + s_red[w][tid];
        } else {
            v = s_hist[tid - (uint32_t)PA_HIST];
        }
        __hip_atomic_store(&d.part[(size_t)blockIdx.x * kPhiPart + tid], (uint64_t)v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    unsigned long long *count = reinterpret_cast<unsigned long long *>(d.acc);
    if (tid == 0u) s_last = atomicAdd(count, 1ull) == (unsigned long long)gridDim.x - 1ull;
    __syncthreads();
    if (!s_last) return;
    // the last workgroup: fold the partials (thread t: field t % 64 of every
    // NW-th one), then the record of sweep t
    if (tid == 0u) __hip_atomic_store(count, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (lane < (uint32_t)PA_END) {
        uint64_t v = 0;
        for (uint32_t i = wv; i < gridDim.x; i += 4u * NW) {
            uint64_t y[4];
#pragma unroll
            for (uint32_t u = 0; u < 4u; ++u) {
                const uint32_t it = i + u * NW;
                y[u] = it < gridDim.x ? __hip_atomic_load(&d.part[(size_t)it * kPhiPart + lane], __ATOMIC_RELAXED,
                                                          __HIP_MEMORY_SCOPE_AGENT)
                                      : 0u;
            }
#pragma unroll
            for (uint32_t u = 0; u < 4u; ++u) v = lane == (uint32_t)PA_MAX ? max(v, y[u]) : v + y[u];
        }
        if (lane == (uint32_t)PA_MAX)
            atomicMax(&s_tot[lane], (unsigned long long)v);
        else if (v)
            atomicAdd(&s_tot[lane], (unsigned long long)v);
    }
    __syncthreads();
    const uint64_t tsw = *d.tdev;
    sw_phi4_obs *rec = &d.ring[tsw % d.ring_cap];
    if (tid < 33u) rec->hist_log2[tid] = s_tot[PA_HIST + tid];
    if (tid == 0u) {
        rec->sweep = tsw;
        const int64_t ef = (int64_t)s_tot[PA_E];
        rec->e_fix = ef;
        rec->action = -(2.0 * d.kappa) * ((double)ef * 0x1p-32);
        double ms = 0.0;
        for (int a = 0; a < 4; ++a) {
            const int64_t ma = (int64_t)s_tot[PA_M + a];
            rec->m_fix[a] = ma;
            const double v = (double)ma * 0x1p-32;
            ms = ms + v * v;
        }
        rec->m_abs = sqrt(ms);
        rec->n_clusters = s_tot[PA_N];
        rec->max_cluster = s_tot[PA_MAX];
        rec->sum_sq_sizes = s_tot[PA_SQ];
    }
    __syncthreads();
    if (tid == 0u) *d.tdev = tsw + 1u;
}

constexpr int kPhiStages = 5;

hipError_t phi_launch_stage(const PhiDev &d, int stage, hipStream_t s) {
    const uint32_t g = (d.N + kPhiChunk - 1) / kPhiChunk;
    switch (stage) {
    case 0: break;  // projections: taken in k_phi_bond and k_phi_flat
    case 1:
        k_phi_bond<<<g, kPhiChunk, 0, s>>>(d);
        if (g > 1u) k_phi_union<<<dim3((d.N + kPhiBlock - 1) / kPhiBlock, 4), kPhiBlock, 0, s>>>(d);
        break;
    case 2: k_phi_flat<<<g, kPhiChunk, 0, s>>>(d); break;
    case 3: break;  // reflections: done by k_phi_flat
    case 4: k_phi_record<<<std::min(g, kPhiRecGroups), kPhiChunk, 0, s>>>(d); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t phi_launch_sweep(const PhiDev &d, hipStream_t s) {
    for (int i = 0; i < kPhiStages; ++i) {
        const hipError_t e = phi_launch_stage(d, i, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

struct PhiLayout {
    size_t phi, parent, csize, cross, dir, part, acc, tdev, ring, total;
};

PhiLayout phi_layout(int32_t L, int64_t ring) {
    const size_t N = (size_t)L * L * L * L;
    PhiLayout lo;
    size_t off = 0;
    auto take = [&](size_t b) {
        const size_t o = off;
        off += align_up(b);
        return o;
    };
    lo.phi = take(N * 4 * sizeof(double));
    lo.parent = take(N * sizeof(uint32_t));
    lo.csize = take(N * sizeof(uint32_t));
    lo.cross = take(N);
    lo.dir = take(8 * sizeof(double));
    lo.part = take(std::min<size_t>((N + kPhiChunk - 1) / kPhiChunk, kPhiRecGroups) * kPhiPart * sizeof(uint64_t));
    lo.acc = take(2 * sizeof(uint64_t));
    lo.tdev = lo.acc + sizeof(uint64_t);
    lo.ring = take((size_t)ring * sizeof(sw_phi4_obs));
    lo.total = off;
    return lo;
}

int phi_validate(int32_t L, double kappa, int32_t init, int64_t ring) {
    if (L < 2 || L > kPhiMaxL) return fail(SW_EINVAL, "L must be in [2, 64] for the phi^4 lattice (N = L^4)");
    if (!(kappa >= 0.0 && kappa <= kPhiMaxKappa)) return fail(SW_EINVAL, "kappa must be finite and in [0, 4]");
    if (init != SW_INIT_HOT && init != SW_INIT_COLD) return fail(SW_EINVAL, "init must be SW_INIT_HOT or SW_INIT_COLD");
    if (ring < 0 || ring > (int64_t)1 << 24) return fail(SW_EINVAL, "ring must be in [0, 2^24]");
    return SW_OK;
}

}  // namespace
}  // namespace swmi

using swmi::fail;
using swmi::hip_fail;

struct sw_phi4 {
    swmi::PhiDev dev;
    hipStream_t stream;
    bool own_stream;
    void *ws;
    bool own_ws;
    hipGraph_t graph;
    hipGraphExec_t gexec;
    bool graph_tried;
    uint64_t next_sweep;
    uint64_t first_valid;
    int device;
    swmi::StageUser stage_user;
};

namespace {

int phi_ensure_device(const sw_phi4 *p) {
    int cur = -1;
    HIP_TRY(hipGetDevice(&cur));
    if (cur != p->device) HIP_TRY(hipSetDevice(p->device));
    return SW_OK;
}

int phi_set_tdev(sw_phi4 *p, uint64_t t) {
    HIP_TRY(hipMemcpyAsync(p->dev.tdev, &t, sizeof(t), hipMemcpyHostToDevice, p->stream));
    HIP_TRY(hipStreamSynchronize(p->stream));
    p->next_sweep = t;
    p->first_valid = t;
    return SW_OK;
}

// One sweep captured into a graph; on any capture failure the kernels are
// launched directly.
void phi_ensure_graph(sw_phi4 *p) {
    if (p->graph_tried) return;
    p->graph_tried = true;
    if (p->stream == nullptr) return;
    if (hipStreamBeginCapture(p->stream, hipStreamCaptureModeThreadLocal) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    const hipError_t le = swmi::phi_launch_sweep(p->dev, p->stream);
    hipGraph_t g = nullptr;
    const hipError_t ce = hipStreamEndCapture(p->stream, &g);
    if (le != hipSuccess || ce != hipSuccess || g == nullptr) {
        if (g) (void)hipGraphDestroy(g);
        (void)hipGetLastError();
        return;
    }
    hipGraphExec_t ge = nullptr;
    if (hipGraphInstantiate(&ge, g, nullptr, nullptr, 0) != hipSuccess) {
        (void)hipGraphDestroy(g);
        (void)hipGetLastError();
        return;
    }
    p->graph = g;
    p->gexec = ge;
}

}  // namespace

extern "C" {

size_t sw_phi4_workspace_bytes(int32_t L, int64_t ring) {
    if (swmi::phi_validate(L, 0.0, SW_INIT_HOT, ring) != SW_OK) return 0;
    return swmi::phi_layout(L, ring ? ring : swmi::kDefaultRing).total;
}

int sw_phi4_create(int32_t L, double kappa, uint64_t seed, int32_t init, int64_t ring, void *dev_workspace,
                   size_t ws_bytes, void *hip_stream, sw_phi4 **out) {
    using namespace swmi;
    if (!out) return fail(SW_EINVAL, "out is NULL");
    *out = nullptr;
    int rc = phi_validate(L, kappa, init, ring);
    if (rc != SW_OK) return rc;
    if (ring == 0) ring = kDefaultRing;
    const PhiLayout lo = phi_layout(L, ring);
    if (dev_workspace && ws_bytes < lo.total)
        return fail(SW_ENOMEM, "workspace too small: need " + std::to_string(lo.total) + " bytes");
    if (dev_workspace && ((uintptr_t)dev_workspace % kAlign) != 0)
        return fail(SW_EINVAL, "workspace must be 256-byte aligned");
    sw_phi4 *p = new (std::nothrow) sw_phi4();
    if (!p) return fail(SW_ENOMEM, "host allocation failed");
    hipError_t e = hipGetDevice(&p->device);
    if (e != hipSuccess) {
        delete p;
        return hip_fail(e, "hipGetDevice");
    }
    if (dev_workspace) {
        p->ws = dev_workspace;
        p->own_ws = false;
    } else {
        e = hipMalloc(&p->ws, lo.total);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            delete p;
            return fail(SW_ENOMEM, "hipMalloc of " + std::to_string(lo.total) + " bytes failed");
        }
        p->own_ws = true;
    }
    if (hip_stream || dev_workspace) {
        p->stream = (hipStream_t)hip_stream;
        p->own_stream = false;
    } else {
        e = hipStreamCreateWithFlags(&p->stream, hipStreamNonBlocking);
        if (e != hipSuccess) {
            if (p->own_ws) (void)hipFree(p->ws);
            delete p;
            return hip_fail(e, "hipStreamCreateWithFlags");
        }
        p->own_stream = true;
    }
    char *base = (char *)p->ws;
    PhiDev &d = p->dev;
    d.phi = (double *)(base + lo.phi);
    d.parent = (uint32_t *)(base + lo.parent);
    d.csize = (uint32_t *)(base + lo.csize);
    d.dir = (double *)(base + lo.dir);
    d.cross = (uint8_t *)(base + lo.cross);
    d.part = (uint64_t *)(base + lo.part);
    d.acc = (uint64_t *)(base + lo.acc);
    d.tdev = (uint64_t *)(base + lo.tdev);
    d.ring = (sw_phi4_obs *)(base + lo.ring);
    d.L = (uint32_t)L;
    d.N = (uint32_t)((size_t)L * L * L * L);
    d.ring_cap = (uint32_t)ring;
    d.seed_lo = (uint32_t)(seed & 0xFFFFFFFFu);
    d.seed_hi = (uint32_t)(seed >> 32);
    d.kappa = kappa;
    e = hipMemsetAsync(p->ws, 0, lo.total, p->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(p->stream);
    if (e != hipSuccess) {
        rc = hip_fail(e, "clearing the workspace");
        sw_phi4_destroy(p);
        return rc;
    }
    rc = sw_phi4_reset(p, init);
    if (rc != SW_OK) {
        const std::string msg = last_error();
        sw_phi4_destroy(p);
        return fail(rc, msg);
    }
    *out = p;
    return SW_OK;
}

int sw_phi4_reset(sw_phi4 *p, int32_t init) {
    if (!p) return fail(SW_EINVAL, "phi4 sim is NULL");
    if (init != SW_INIT_HOT && init != SW_INIT_COLD) return fail(SW_EINVAL, "init must be SW_INIT_HOT or SW_INIT_COLD");
    int rc = phi_ensure_device(p);
    if (rc != SW_OK) return rc;
    rc = phi_set_tdev(p, 0);
    if (rc != SW_OK) return rc;
    const uint32_t g = (p->dev.N + swmi::kPhiBlock - 1) / swmi::kPhiBlock;
    swmi::k_phi_init<<<g, swmi::kPhiBlock, 0, p->stream>>>(p->dev, init == SW_INIT_COLD ? 1 : 0);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(p->stream));
    return SW_OK;
}

int sw_phi4_sweep(sw_phi4 *p, int64_t n) {
    if (!p) return fail(SW_EINVAL, "phi4 sim is NULL");
    if (n < 0) return fail(SW_EINVAL, "n must be >= 0");
    if (n == 0) return SW_OK;
    int rc = phi_ensure_device(p);
    if (rc != SW_OK) return rc;
    phi_ensure_graph(p);
    for (int64_t i = 0; i < n; ++i) {
        if (p->gexec)
            HIP_TRY(hipGraphLaunch(p->gexec, p->stream));
        else
            HIP_TRY(swmi::phi_launch_sweep(p->dev, p->stream));
    }
    p->next_sweep += (uint64_t)n;
    return SW_OK;
}

int sw_phi4_sync(sw_phi4 *p) {
    if (!p) return fail(SW_EINVAL, "phi4 sim is NULL");
    int rc = phi_ensure_device(p);
    if (rc != SW_OK) return rc;
    HIP_TRY(hipStreamSynchronize(p->stream));
    return SW_OK;
}

int sw_phi4_profile(sw_phi4 *p, int64_t n, double *ms, int32_t nk) {
    if (!p || !ms) return fail(SW_EINVAL, "phi4 sim or ms is NULL");
    if (n < 1) return fail(SW_EINVAL, "n must be >= 1");
    if (nk < swmi::kPhiStages) return fail(SW_ERANGE, "nk must be >= 5");
    int rc = phi_ensure_device(p);
    if (rc != SW_OK) return rc;
    constexpr int kEv = swmi::kPhiStages + 1;
    hipEvent_t ev[kEv];
    for (int i = 0; i < kEv; ++i) {
        const hipError_t e = hipEventCreate(&ev[i]);
        if (e != hipSuccess) {
            for (int j = 0; j < i; ++j) (void)hipEventDestroy(ev[j]);
            return hip_fail(e, "hipEventCreate");
        }
    }
    double acc[swmi::kPhiStages] = {0};
    hipError_t e = hipSuccess;
    for (int64_t i = 0; i < n && e == hipSuccess; ++i) {
        e = hipEventRecord(ev[0], p->stream);
        for (int st = 0; st < swmi::kPhiStages && e == hipSuccess; ++st) {
            e = swmi::phi_launch_stage(p->dev, st, p->stream);
            if (e == hipSuccess) e = hipEventRecord(ev[st + 1], p->stream);
        }
        if (e == hipSuccess) e = hipEventSynchronize(ev[kEv - 1]);
        for (int st = 0; st < swmi::kPhiStages && e == hipSuccess; ++st) {
            float f = 0.f;
            e = hipEventElapsedTime(&f, ev[st], ev[st + 1]);
            acc[st] += f;
        }
        if (e == hipSuccess) p->next_sweep += 1u;
    }
    for (int i = 0; i < kEv; ++i) (void)hipEventDestroy(ev[i]);
    if (e != hipSuccess) return hip_fail(e, "sw_phi4_profile");
    for (int i = 0; i < nk; ++i) ms[i] = i < swmi::kPhiStages ? acc[i] / (double)n : 0.0;
    return SW_OK;
}

int sw_phi4_series(sw_phi4 *p, int64_t first, int64_t count, sw_phi4_obs *out) {
    if (!p) return fail(SW_EINVAL, "phi4 sim is NULL");
    if (count < 0 || (count > 0 && !out)) return fail(SW_EINVAL, "bad count or NULL out");
    const int64_t lo = std::max<int64_t>((int64_t)p->first_valid, (int64_t)p->next_sweep - (int64_t)p->dev.ring_cap);
    if (first < lo || first + count > (int64_t)p->next_sweep)
        return fail(SW_ERANGE, "records requested outside the sweeps run and held in the ring");
    if (count == 0) return SW_OK;
    int rc = phi_ensure_device(p);
    if (rc != SW_OK) return rc;
    const int64_t cap = p->dev.ring_cap;
    int64_t done = 0;
    while (done < count) {
        const int64_t slot = (first + done) % cap;
        const int64_t run = std::min(count - done, cap - slot);
        HIP_TRY(swmi::copy_to_host(out + done, p->dev.ring + slot, (size_t)run * sizeof(sw_phi4_obs), p->stream));
        done += run;
    }
    return SW_OK;
}

int sw_phi4_get_field(sw_phi4 *p, double *host, int64_t n) {
    if (!p || !host) return fail(SW_EINVAL, "phi4 sim or host is NULL");
    if (n != 4 * (int64_t)p->dev.N) return fail(SW_ERANGE, "n must equal 4 L^4");
    int rc = phi_ensure_device(p);
    if (rc != SW_OK) return rc;
    HIP_TRY(swmi::copy_to_host(host, p->dev.phi, (size_t)n * sizeof(double), p->stream));
    return SW_OK;
}

int sw_phi4_set_field(sw_phi4 *p, const double *host, int64_t n, uint64_t next_sweep) {
    if (!p || !host) return fail(SW_EINVAL, "phi4 sim or host is NULL");
    if (n != 4 * (int64_t)p->dev.N) return fail(SW_ERANGE, "n must equal 4 L^4");
    for (int64_t i = 0; i < n; ++i)
        if (!std::isfinite(host[i])) return fail(SW_EINVAL, "field component " + std::to_string(i) + " is not finite");
    int rc = phi_ensure_device(p);
    if (rc != SW_OK) return rc;
    HIP_TRY(hipStreamSynchronize(p->stream));
    HIP_TRY(hipMemcpy(p->dev.phi, host, (size_t)n * sizeof(double), hipMemcpyHostToDevice));
    return phi_set_tdev(p, next_sweep);
}

int sw_phi4_get_labels(sw_phi4 *p, uint32_t *host, int64_t n) {
    if (!p || !host) return fail(SW_EINVAL, "phi4 sim or host is NULL");
    if (n != (int64_t)p->dev.N) return fail(SW_ERANGE, "n must equal L^4");
    if (p->next_sweep == p->first_valid) return fail(SW_ESTATE, "no sweep has run since create / reset / set_field");
    int rc = phi_ensure_device(p);
    if (rc != SW_OK) return rc;
    HIP_TRY(swmi::copy_to_host(host, p->dev.parent, (size_t)n * sizeof(uint32_t), p->stream));
    return SW_OK;
}

int64_t sw_phi4_sites(const sw_phi4 *p) { return p ? (int64_t)p->dev.N : -1; }

int64_t sw_phi4_next_sweep(const sw_phi4 *p) { return p ? (int64_t)p->next_sweep : -1; }

void sw_phi4_destroy(sw_phi4 *p) {
    if (!p) return;
    if (phi_ensure_device(p) == SW_OK && p->stream) (void)hipStreamSynchronize(p->stream);
    if (p->gexec) (void)hipGraphExecDestroy(p->gexec);
    if (p->graph) (void)hipGraphDestroy(p->graph);
    if (p->own_ws && p->ws) (void)hipFree(p->ws);
    if (p->own_stream && p->stream) (void)hipStreamDestroy(p->stream);
    delete p;
}

}  // extern "C"
