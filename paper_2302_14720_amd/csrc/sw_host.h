// sw_host.h -- host-side helpers shared by the C ABI (sw_api.hip) and the
// serving runtime (sw_server.hip): error reporting, validation, and the
// carving of one lattice's device buffers out of a workspace.
#pragma once

#include <string>
#include <vector>

#include "sw_internal.h"

namespace swmi {

constexpr size_t kAlign = 256;
constexpr int64_t kDefaultRing = 4096;

inline size_t align_up(size_t v) { return (v + kAlign - 1) & ~(kAlign - 1); }

// Sets the thread's last-error message and returns code.
int fail(int code, const std::string &msg);
int hip_fail(hipError_t e, const char *what);
// The thread's last-error message.
const std::string &last_error();

// Copies n device bytes to host memory after everything enqueued on s, and
// waits (into pageable memory through pinned staging; without any to be had, a
// pageable copy).
hipError_t copy_to_host(void *dst, const void *src, size_t n, hipStream_t s);
// Held by every object that copies; the last one gives the staging back, but
// for one buffer.
struct StageUser {
    StageUser();
    ~StageUser();
    StageUser(const StageUser &) = delete;
    StageUser &operator=(const StageUser &) = delete;
};

// Bond probability p = 1 - exp(-2 beta J) as a 32-bit threshold.
uint32_t bond_threshold(double beta, double J);

struct Layout {
    size_t spins[2], parent, nk[2], key, nsize, rspin, edge, xb, gspin, gcount, mpart, tpart, gpart, acc, tdev, ring, labels,
        dense, tdense, le_mask, le_cnt, le_rsp, le_ctl, codes, faces, node, total;
};

int resolve_tile(const sw_config &c);
int validate(const sw_config *c);
Layout layout_of(const sw_config &c);
Dev make_dev(const sw_config &c, char *base, const Layout &lo);

// Whether k_merge takes a lattice that it can (at most 16 groups).
bool merge_in_one(const sw_config &c);
// Its workgroups for such a lattice of more than 16 tiles (0 for any other).
uint32_t wide_groups(const sw_config &c);

// Whether k_merge takes those larger lattices of a batch or server too: while
// they make at most kWideGroups of its workgroups, and nothing is merged globally
// in any case.  One of those workgroups fills a CU (16 wavefronts of 76 to 86
// VGPRs), so from two rounds of them on the global merge's small workgroups are
// faster.  us per sweep, global / k_merge: 512^2, 32 replicas (128 groups) 99.8 /
// 77.3, 128 (512) 201.8 / 199.5, 256 (1024) 334.3 / 376.3; 1024^2, 16 (256)
// 139.1 / 121.2, 32 (512) 204.8 / 207.4, 64 (1024) 337.4 / 385.8; sides 64 to
// 1024, 128 replicas (500) 221.6 / 215.6, 160 (640) 258.9 / 267.0, 256 (1020)
// 369.6 / 407.4.  Servers: 64 jobs of 1024^2 333.0 / 371.4, 256 of 512^2 331.2 /
// 371.9, 400 of 320^2 (1600) 240.2 / 343.0.  Beside a lattice of the global merge,
// whose launches are there anyway, k_merge only adds its own time: 512^2 and
// 1088^2 75.5 / 91.7, 16 of 512^2 and four of 2048^2 156.2 / 175.2, 128 of 320^2
// and one of 1088^2 130.8 / 175.9, 32 of 1024^2 and 20 of 2048^2 551 / 598.
constexpr uint32_t kWideGroups = 512;
inline bool take_wide(uint32_t groups, bool global) { return groups <= kWideGroups && !global; }

// Launch groups of a batch: Ising and Potts replicas, each with 64-wide or
// 32-wide tiles, run different instantiations of the tile kernels.
constexpr int kBatchGroups = 4;
inline int batch_group(const Dev &d) { return (d.q ? 2 : 0) + (d.tw == 64 ? 0 : 1); }
inline void set_groups(BatchDev *bd) {
    for (int g = 0; g < kBatchGroups; ++g) {
        bd[g].tw = (g & 1) ? 32u : 64u;
        bd[g].potts = g >= 2 ? 1u : 0u;
    }
}

// Host-side work maps of one launch group: add() files the replica in slot
// `slot` of the Dev table, whose launch group is one of the kBatchGroups `all`,
// under k_merge (d.two) or under the global merge; emit() appends the maps to
// `host` (which will be copied to dev_base) and points the BatchDev at them.
// Only the tile kernels differ by group: those of the merges take replicas of
// every kind and have all their units in the first group's maps -- kernels of a
// few us each, once a sweep instead of once per group.
struct BatchMaps {
    std::vector<uint32_t> t, w, wn, g, u, s, a;  // w / wn: tiles with an E / N group edge
    uint32_t n = 0;                              // replicas of the global merge
    static void add(uint32_t slot, const Dev &d, BatchMaps *all) { all[batch_group(d)].add_to(slot, d, all[0]); }
    void add_to(uint32_t slot, const Dev &d, BatchMaps &merge) {
        const uint32_t tag = slot << kMapShift;
        a.push_back(slot);
        for (uint32_t i = 0; i < d.ntiles; ++i) t.push_back(tag | i);
        const uint32_t ngx = (d.ntx + kUG - 1u) / kUG;
        if (d.two) {
            for (uint32_t i = 0; i < ngx * ngx; ++i) merge.s.push_back(tag | i);
            return;
        }
        ++n;
        // edges between kUG x kUG groups of tiles (those inside a group are
        // joined by k_ulocal): the last tile column / row of every group
        for (uint32_t i = 0; i < d.ntiles; ++i) {
            const uint32_t tx = i % d.ntx, ty = i / d.ntx;
            if (tx % kUG == kUG - 1u || tx + 1u == d.ntx) merge.w.push_back(tag | i);
            if (ty % kUG == kUG - 1u || ty + 1u == d.ntx) merge.wn.push_back(tag | i);
        }
        for (uint32_t i = 0; i < d.ngroups; ++i) merge.g.push_back(tag | i);
        for (uint32_t i = 0; i < ngx * ngx; ++i) merge.u.push_back(tag | i);
    }
    size_t words() const {
        return t.size() + w.size() + wn.size() + g.size() + u.size() + s.size() + a.size();
    }
    // the tile maps of all launch groups first, so that they are one map
    static void emit(const BatchMaps *all, std::vector<uint32_t> &host, const uint32_t *dev_base, BatchDev *b) {
        for (int g = 0; g < kBatchGroups; ++g) {
            b[g].ntiles = (uint32_t)all[g].t.size();
            b[g].tmap = dev_base + host.size();
            host.insert(host.end(), all[g].t.begin(), all[g].t.end());
        }
        for (int g = 0; g < kBatchGroups; ++g) all[g].emit(host, dev_base, b[g]);
    }
    void emit(std::vector<uint32_t> &host, const uint32_t *dev_base, BatchDev &b) const {
        const uint32_t *p = dev_base + host.size();
        b.nwmap = (uint32_t)(w.size() + wn.size());
        b.nwE = (uint32_t)w.size();
        b.ngroups = (uint32_t)g.size();
        b.nugroups = (uint32_t)u.size();
        b.n = n;
        b.nsmall = (uint32_t)s.size();
        b.nall = (uint32_t)a.size();
        host.insert(host.end(), w.begin(), w.end());
        host.insert(host.end(), wn.begin(), wn.end());
        host.insert(host.end(), g.begin(), g.end());
        host.insert(host.end(), u.begin(), u.end());
        host.insert(host.end(), s.begin(), s.end());
        host.insert(host.end(), a.begin(), a.end());
        b.wmap = p;
        b.gmap = b.wmap + b.nwmap;
        b.umap = b.gmap + b.ngroups;
        b.smap = b.umap + b.nugroups;
        b.amap = b.smap + b.nsmall;
    }
};

}  // namespace swmi

#define HIP_TRY(expr)                                             \
    do {                                                          \
        hipError_t e_ = (expr);                                   \
        if (e_ != hipSuccess) return swmi::hip_fail(e_, #expr);   \
    } while (0)
