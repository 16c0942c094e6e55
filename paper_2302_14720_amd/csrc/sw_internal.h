// sw_internal.h -- device-state layout and kernel entry points of libswmi.
//
// One sweep (paper Sec. 2) runs as these kernels on the sim's stream:
//   k_tile    bond formation (Sec. 2.1) and cluster formation (Sec. 2.3)
//             inside one 64x64 (or 32x32) tile per workgroup, in LDS; new
//             spins (Sec. 2.4) of clusters that stay inside the tile; the
//             tile's clusters with a bond out of the tile (of 32-wide tiles
//             with 16 sites per thread, all that touch its edge) become
//             "nodes" of a global graph;
//             the spins of the previous sweep are resolved on the fly and
//             measured (Sec. 2.5).
//   k_union   union of nodes joined by bonds that cross tile edges: first
//             (k_ulocal) inside each 4x4 group of tiles in LDS, then, for
//             the edges between groups, by lock-free union-find in global
//             memory (the root is the node with the smaller index, or,
//             in the ordered phase of a large lattice, with the smaller
//             bit-reversed index).
//   k_flatten point every node at its root; add node sizes into the roots
//             and reduce node keys to the cluster's smallest site.
//   k_roots   new spin of each cross-tile cluster, cluster statistics.
//   k_record  fold partial statistics into the per-sweep record ring (on
//             lattices of at most 64 groups the last k_roots workgroup
//             folds them, and the sweep is four launches).
// On lattices of at most 16 groups of 4x4 tiles, k_merge does all after k_tile
// in one launch.  Batches and servers run the same bodies over work maps (k_*_b).
// Spins are double-buffered by sweep parity (the buffer that a sweep has read
// then holds k_merge's results of the groups).  A written spin byte is either
// the final spin (0x01 = +1, 0xFF = -1) or 2 + k, a reference to node k of
// the tile, resolved through the node tables of that sweep when the byte is
// read next (by the next sweep's k_tile, or by k_resolve at the end of
// every sw_sweep call).  The q-state Potts model runs the same kernels with
// values 0..q-1 as final bytes and node codes from 4 (64-wide tiles, q <= 4)
// or 8 (32-wide tiles).
//
// The simple cubic lattice has the same pipeline on 16^3 bricks
// (sw_brick.hip).  The paper's label equivalence, on either lattice, keeps
// 32-bit labels per site in global memory instead (sw_le.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "swmi.h"

namespace swmi {

constexpr uint32_t kNodeSlots = 256;  // node slots per tile (64x64 tile: <= 252 nodes)
constexpr int kTilePart = 32;         // int32 words of a per-tile partial
constexpr int kGroupPart = 48;        // uint64 words of a per-group partial
constexpr int kMaxQ = 8;              // largest q of the Potts model
constexpr int kAccWords = 64;         // record accumulator + completion counter
constexpr int kGroupTiles = 16;       // tiles per workgroup in k_flatten / k_roots
constexpr uint32_t kDenseBins = 256;  // sizes below this are counted per tile and group (dense histogram)
constexpr uint32_t kUG = 4;           // side, in tiles, of a k_ulocal or k_merge group
constexpr uint32_t kRef = 8;          // nref: below, a final value
constexpr uint32_t kMergeGroups = 16; // most groups of a lattice merged by k_merge
// Slots of a k_merge group for its clusters that go on outside it: the sites of its perimeter.
__host__ __device__ constexpr uint32_t ref_slots(uint32_t tw) { return 4u * kUG * tw; }
// What the groups hand to the lattice's last workgroup (10 bytes a slot) lies in
// the spin buffer that the sweep has read by then; 5, 9 and 13 tiles a side are
// the smallest lattices of 4, 9 and 16 groups.
static_assert(4u * ref_slots(32) * 10u <= 25u * 32u * 32u && 9u * ref_slots(32) * 10u <= 81u * 32u * 32u &&
                  16u * ref_slots(32) * 10u <= 169u * 32u * 32u,
              "the group tables must fit in a lattice's spins (64-wide tiles: half of this share)");

// tile partial (int32 words)
// hist: kTileBins bins (sizes up to 64 * 64 or 16^3); TP_CNT..: population of each Potts value
constexpr uint32_t kTileBins = 13;
enum { TP_E = 0, TP_M = 1, TP_N = 2, TP_MAX = 3, TP_SQ = 4, TP_HIST = 5, TP_CNT = 18 };
// group partial / accumulator (uint64 words)
// GP_CNT..: population of each Potts value
enum { GP_N = 0, GP_MAX = 1, GP_SQ = 2, GP_E = 3, GP_M = 4, GP_HIST = 5, GP_CNT = 38, GP_END = 46 };
enum { ACC_COUNT = 48 };

struct Dev {
    int8_t *spins[2];     // [N] by sweep parity
    uint32_t *parent;     // [ntiles * kNodeSlots] of the sweep that runs
    uint32_t *nk[2];      // [ntiles] number of nodes per tile, by parity
    uint32_t *key;        // [ntiles * kNodeSlots] smallest site of the node
    uint32_t *nsize;      // [ntiles * kNodeSlots] node size; cluster size at roots
    int8_t *rspin;        // [ntiles * kNodeSlots] new spin of each node's cluster (in the place of nref)
    uint8_t *edge;        // [ntiles][4][tw] node index of W, E, S, N edge sites
    uint64_t *xb;         // [ntiles][2] bonds leaving the tile: E (bit y), N (bit x)
    int32_t *tpart;       // [ntiles][kTilePart]
    uint64_t *gpart;      // [ngroups][kGroupPart]
    uint64_t *acc;        // [kAccWords]
    uint64_t *tdev;       // [0] = index of the next sweep
    // lattices merged by k_merge (two = 1); the last three with several groups
    uint16_t *nref;       // [ntiles * kNodeSlots] value of the node's cluster, or kRef + its number in the group
    uint8_t *gspin;       // [groups][ref_slots] new values of the clusters that go on outside the group
    uint32_t *gcount;     // [groups] how many
    uint64_t *mpart;      // [groups][kGroupPart] partial statistics
    sw_obs *ring;         // [ring_cap]
    uint32_t *labels;     // [N] or nullptr (bricks: in the place of faces, nsize and on)
    uint64_t *dense;      // [N + 1] or nullptr
    uint16_t *tdense;     // [ntiles][kDenseBins] interior clusters by size (with dense, tile path)
    // label-equivalence path (SW_FLAG_LABEL_EQUIV); nullptr otherwise
    uint8_t *le_mask;     // [N] bonds of each site: bit 0 to E, bit 1 to N
    uint32_t *le_cnt;     // [N] cluster size at each root
    int8_t *le_rsp;       // [N] new spin, valid at roots
    uint32_t *le_ctl;     // [8] pass flags (3), passes of the last sweep, status
    // simple cubic lattice on bricks (sw_brick.hip); parent, nk[0], key, nsize
    // and tpart by brick, kBrickNodes node slots each; gpart one per brick
    uint16_t *codes;      // [nbricks][4096] brick-local index of the site's component's smallest site
    uint16_t *faces;      // [nbricks][6][256] nodes of the sites of the +x, +y, +z faces (0xFFFF unless
                          // bonded through the face) and of the x = 0, y = 0, z = 0 faces
    uint32_t *node;       // [nbricks][kBrickNodes] smallest brick-local site | size << 16 of every node
    uint32_t L, tw, ntx, ntiles, ngroups;
    uint32_t T, seed_lo, seed_hi;
    uint32_t ring_cap;
    uint32_t le_grid;     // workgroups of the cooperative labelling kernel (0: tile path)
    uint32_t q;           // 0: Ising; 2..kMaxQ: q-state Potts (label-equivalence path)
    uint32_t dims;        // 2: L x L; 3: L x L x L (labels in global memory)
    uint32_t two;         // 1: merged by k_merge (one launch)
    uint32_t brick;       // 1: simple cubic lattice on kBrick^3 bricks (else label equivalence)
    uint64_t nsite;       // N = L^dims
    double J;
};

// Four Ising spin bytes: 0xFF stays -1, every other byte becomes +1.
__host__ __device__ inline uint32_t spin_bytes(uint32_t w) {
    const uint32_t m = (((w & 0x7F7F7F7Fu) + 0x01010101u) & w & 0x80808080u) >> 7;  // 1 in every byte that is 0xFF
    return 0x01010101u | m * 0xFFu;
}

constexpr int kStages = 5;  // kernels of one sweep, in stream order

hipError_t launch_init(const Dev &d, int cold, hipStream_t s);
hipError_t launch_stage(const Dev &d, int stage, hipStream_t s);
hipError_t launch_sweep(const Dev &d, hipStream_t s);
hipError_t launch_resolve(const Dev &d, hipStream_t s);

// Batched sweeps: each kernel of a sweep runs once over a table of
// independent lattices (replicas), each with its own Dev, so the launches
// per sweep do not grow with the batch (five per launch group under the
// global merge, the record folded by k_roots_b).  The maps list the work units
// of every replica: entry = replica << kMapShift | unit.
constexpr uint32_t kMapShift = 20;
constexpr uint32_t kMapMask = (1u << kMapShift) - 1u;
constexpr int32_t kMaxReplicas = 4095;
static_assert(kMaxReplicas <= 1 << (32 - kMapShift), "a replica's index must fit its map entries");

// The LDS merge a caller can ask for in a batch takes at most kSmallTiles tiles.
constexpr uint32_t kSmallTiles = 16;

struct BatchDev {
    const Dev *devs;       // the replicas' Dev, in device memory
    const uint32_t *tmap;  // [ntiles] one entry per tile of every replica (k_tile, k_resolve)
    const uint32_t *wmap;  // [nwmap] tiles with an E (first nwE) or N group edge (k_union)
    const uint32_t *gmap;  // [ngroups] one per group of kGroupTiles tiles (k_flatten, k_roots)
    const uint32_t *umap;  // [nugroups] one per kUG x kUG group of tiles (k_ulocal)
    const uint32_t *smap;  // [nsmall] one per kUG x kUG group of tiles of the replicas merged by k_merge
    const uint32_t *amap;  // [nall] every replica of the launch (records after k_resolve)
    uint32_t n;            // replicas of the global merge
    uint32_t ntiles, nwmap, ngroups, nugroups, tw;
    uint32_t nwE, nsmall, nall;
    uint32_t potts;        // 1: every replica is a Potts model (q in its Dev)
};


// Label equivalence: stages 0..3 of a sweep (bonds; labelling; new spins and
// sizes; statistics) and the cooperative grid size.
hipError_t launch_le_stage(const Dev &d, int stage, hipStream_t s);
uint32_t le_grid_size(uint32_t dims);
constexpr uint32_t kLeChunk = 4096;  // sites per workgroup in the per-site passes
constexpr uint32_t kBrick = 16;      // side of a brick of the simple cubic lattice
constexpr uint32_t kBrickNodes = 1352;  // node slots per brick: its surface sites
enum { LE_PASSES = 3, LE_STATUS = 4 };

// Cubic bricks: stages 0..3 of a sweep, the closing measurement (brick
// partials), and the labels of the last sweep.
hipError_t launch_brick_stage(const Dev &d, int stage, hipStream_t s);
hipError_t launch_brick_measure(const Dev &d, hipStream_t s);
hipError_t launch_brick_labels(const Dev &d, hipStream_t s);

// One sweep of all launch groups: the tiles (of every group in one launch where
// they are few), then k_merge and the global merge of the replicas of each.
hipError_t launch_batch_sweep(const BatchDev *b, int ngroups, hipStream_t s);
hipError_t launch_batch_resolve(const BatchDev &b, hipStream_t s);

}  // namespace swmi
