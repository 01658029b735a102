// HIP kernels for gfx950 (MI355X): box-histogram queries over the Mixture
// Graph, the naive level-0 range scan, transfer-function propagation, and the
// device side of upload / workspaces / timing.
//
// Box decomposition (Sec. "Fast Sub-Volume Queries" and the appendix
// algorithm "Footprint assembly in 3D"). The footprint of a box is the set of
// maximal aligned mipmap cubes inside it. Per axis and level l, the level-l
// cells fully inside [x0, x1) are [a_l, b_l) with a_l = ceil(x0 / 2^l) and
// b_l = floor(x1 / 2^l); the cells of that range not covered by a level-(l+1)
// cell inside the box are the (at most two) 1D footprint steps of level l.
// The tensor product of the 1D step lists, tessellated by cubes of the
// smallest level, groups by level into a hollow shell: the outer block
// [a_l, b_l)^3 minus the inner block [2 a_{l+1}, 2 b_{l+1})^3, i.e. at most
// six slabs one cell thick. The kernels enumerate those <= 6 slabs per level
// instead of the up to (2 log2 D)^3 rectangles; the cube set is the same.
// Slabs that are one cell thick along x are read from a transposed copy of
// the level's node map (y fastest) so that every slab streams contiguous rows.
//
// Each cube contributes its 8^l voxels to the node its mip voxel holds
// ("denormalized" samples). Cubes whose node is a source add straight to the
// segment's integer count, those on nodes of rank 1 and 2 through the node's
// record of its two to four sources; nodes of rank >= 3 collect integer counts in
// a per-query hash table, then each adds its count times its mixture row. Graphs
// too large for rows, and calls that report the nodes a box reaches, push mass
// down the DAG instead, rank by rank in reverse order (node n = (1 - w_n) a_n +
// w_n b_n gives a the share 1 - w_n and b the share w_n). Mass is fp32 with a
// two-sum compensation term per entry; the final per-segment count is summed in
// fp64 and divided by the box volume. A box is answered by one workgroup, or in
// parts by several whose sums meet in the workspace.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "mg_internal.hpp"

namespace mg {
namespace {

constexpr int kBlock = 256;                    // plain / fallback / naive workgroup size
constexpr int kBlockBig = 512;                 // big-box tier workgroup size
constexpr uint32_t kEmpty = 0xFFFFFFFFu;
constexpr uint32_t kMaxLevelsDev = 16;          // dims up to 32768 per axis
constexpr int kMaxSlabs = 6 * kMaxLevelsDev;
constexpr uint32_t kHashPlain = 2048;         // per-box hash slots in LDS, plain kernel
constexpr uint32_t kHashSmall = 256;          // small-box tier (per-source arrays in LDS)
constexpr uint32_t kHashBig = 2048;           // big-box tier (per-source arrays in LDS)
// Uncertainty queries: nodes of every rank are entries. 10,000 boxes of 256^3 (353 segments, 7.9
// thousand nodes): 638 us with tables of 256 and 2,048 slots (a tenth of the boxes done twice),
// 603 with 512 and 2,048, 472 with 512 and 4,096, 516 with 1,024 and 4,096, 490 with 512 and 8,192.
constexpr uint32_t kHashSmallErr = 512;
constexpr uint32_t kHashBigErr = 4096;
constexpr uint32_t kHashSmallSparse = 2048;   // small-box tier, sources as table entries
constexpr uint32_t kHashBigSparse = 4096;     // big-box tier, sources as table entries
constexpr uint32_t kHashRetry = 8192;         // boxes that overflowed a tier table
constexpr uint32_t kBigLog2 = 14;             // boxes of >= 2^14 cubes go to the big tier
// The same where small boxes keep sources in the table: 20,000 boxes of a 307x480x300 volume of
// 3,980 fibres with 2^8 / 2^10 / 2^12 / 2^14: 4.70 / 4.76 / 4.88 / 5.41 ms.
constexpr uint32_t kBigLog2Sparse = 10;
constexpr uint32_t kStaticLds = 10240;        // LDS set aside for the query kernels' fixed arrays (9,952 at most)
// A table size set by the caller that fits the LDS beside this much is always taken; where only the
// kernels' larger fixed arrays leave no room for it, half the size is.
constexpr uint32_t kStaticLdsSet = 6448;
constexpr uint32_t kHashGlobal = 1u << 16;    // fewest per-worker hash slots in the fallback tables
constexpr uint32_t kSegLdsMax = 2048;         // sources kept in LDS
constexpr uint32_t kFallbackWorkers = 128;    // workers of the final global-table launch (budget)
constexpr uint32_t kLeastTiles = 16;            // tiles and row segments (64 are described at once) worth a
constexpr uint32_t kLeastRunItems = 32;         // piece of their own where waves share them
constexpr uint32_t kLeastItems = 8;            // row segments worth a wave's while
constexpr uint32_t kRunSeg = 256;             // cells of a row one thread sums from the runs
// Rows shorter than this stream cube by cube (default). 100,000 boxes of 512^3 with 8 / 16 / 32 / 128:
// 1.126 / 1.112 / 1.146 / 1.728 ms; 5,000 of 199x181x163: 101 / 100 / 112 / 157 us.
constexpr uint32_t kRunMinRow = 16;
constexpr uint32_t kTfPlanes = 4;             // transfer functions per thread of a propagation step
constexpr uint32_t kTfTailPairs = 4096;        // steps of at most this many node x TF pairs may share a launch
constexpr uint32_t kTfTailSteps = 16;          // at most this many of them
constexpr uint32_t kTfTailBlock = 1024;        // threads of that launch (one workgroup)
constexpr uint32_t kMidWorkers = 256;         // workers of the mid-size global-table launch
constexpr uint32_t kMaxSlots = 1024;           // boxes of one call that several workgroups may share
constexpr uint64_t kSlotBytes = 32ull << 20;  // their accumulators take at most this much of a workspace
constexpr uint32_t kMinSlots = 16;            // (but hold at least this many boxes)
constexpr uint32_t kNoallocWorkers = 16;      // workers of the static scratch that come before shared boxes
// Fewest cubes worth a workgroup of their own: when others idle (one box of 205,000 cubes of a
// 400x375x263 volume in parts of 2,048 / 4,096 / 8,192 / 16,384 / 32,768: 36 / 36 / 40 / 46 / 55 us,
// whole: 105), and in a large batch (5,000 boxes of 199x181x163, parts of 16,384 / 32,768 /
// 65,536: 105 / 102 / 106 us, whole: 111).
constexpr uint32_t kMinPart = 4096;
constexpr uint32_t kMinPartBatch = 1u << 15;
constexpr uint32_t kMinPartRedo = 1u << 14;   // the same for boxes that overflowed: the others are done
// Uncertainty queries: classes of the nodes of a large box that overflowed its table, each taken
// by a workgroup that reads all its cubes (10,000 boxes of 256^3: 0.47 ms; with such boxes redone
// whole, mostly in tables in global memory in the end: 1.03). Boxes of the small tier fit the
// larger LDS table whole.
constexpr uint32_t kClassesRedo = 4;
constexpr uint32_t kDirectMax = 1024;         // boxes of a call answered without a planning launch
constexpr uint32_t kNoallocSlots = 256;        // the same on the library's static scratch
constexpr int kBlockDirect = 256;             // workgroup size of that path
constexpr uint32_t kHashDirect = 1024;        // its fewest and most LDS hash slots (per-source arrays in LDS)
constexpr uint32_t kHashDirectMax = 4096;
constexpr uint32_t kQueues = 8;                // work queues per tier
constexpr uint32_t kQueueStride = 64;          // u32 between queue counters (256 bytes)
constexpr int kGroup = 4;                      // tiles per load group (plain, fallback)
constexpr uint32_t kMaxSteps = 64;              // graph depth the step table holds
constexpr uint32_t kDeferSlots = 128;           // per-wave ring of deferred internal-node runs (dense state)

#define HIP_TRY(expr)                                                                  \
    do {                                                                               \
        hipError_t e_ = (expr);                                                        \
        if (e_ != hipSuccess) {                                                        \
            *err = std::string(#expr) + ": " + hipGetErrorString(e_);                  \
            return MG_EDEVICE;                                                         \
        }                                                                              \
    } while (0)

// ---------------------------------------------------------------- constants

struct LevelTable {
    uint32_t n_levels;
    uint32_t vol[3];
    uint32_t dims[MG_MAX_LEVELS][3];
    uint64_t off[MG_MAX_LEVELS];     // element offset of each level in maps
    uint64_t total;                  // elements of one full copy (maps_t starts here)
    // 16-bit copy of level 0 (both orientations), rows padded to an even length:
    // x-fastest index x + pitch_x (y + Y z), then at total16 the y-fastest index
    // y + pitch_y (z + Z x); used when `use16` (dense mode, sources < 65535)
    uint32_t use16;
    uint32_t pitch_x, pitch_y;
    uint64_t total16;
    // row runs (kind-2 slabs): bit 2 l + o set where level l has runs along x (o = 0)
    // or y (o = 1) and the launch reads them; slabs whose rows are at least run_min
    // cubes long are summed from runs
    uint32_t runs_mask;
    uint32_t run_min;
};

// Row runs of one level and orientation as the kernels read them (the device copy
// of the host's LevelRuns): runs[j] = exclusive end << 32 | node; skip[r][c] =
// index of the run holding cell kRunSkipCells c of row r.
struct RunLevel {
    const uint32_t *skip;      // [rows][chunks]
    const uint64_t *runs;      // [n_runs]
    uint32_t rows, chunks, n_runs;
    uint32_t first;            // index of runs[0] from the graph's first run (GraphView::runs)
};

// A slab of cubes at one level, as the query kernels read it: e2 slices (slow
// axis, the thinnest) of e1 rows (mid axis) of e0 cubes (fast axis, the
// contiguous axis of the chosen copy: x in maps, y in maps_t), read as `units`
// 4-byte units per row: one 32-bit node ID per cube (kind 0), or, from the
// 16-bit level-0 copy, aligned pairs of source IDs (kind 1; a row whose first
// cube is at an odd position starts one element early, `odd`); or, kind 2, each
// row segment summed from the row runs of its level and orientation (base, s1b,
// s2b, units unused).
// (kind 2, in the same words: base: the first row's index in the level's runs, above it the
// reciprocal of e1 (run_item); s1b, s2b: row indices between rows / slices; units: the first
// cube's cell along its row; odd: log2 of the segments per row)
struct Slab {
    uint64_t base;         // byte offset of the first unit in its buffer (maps or maps16)
    uint32_t e0, e1, e2;   // cubes along the fast, mid and slow axes
    uint32_t s1b, s2b;     // bytes between rows / slices (0 where the extent is 1)
    uint32_t units;        // 4-byte units per row
    uint32_t bx, by, bz;   // first cube, level coordinates
    uint8_t level;
    uint8_t kind;          // 0: 32-bit node IDs, 1: pairs of 16-bit level-0 source IDs, 2: row runs
    uint8_t axes;          // fast | mid << 2 | slow << 4 (0 = x, 1 = y, 2 = z)
    uint8_t odd;           // kind 1: the row's first unit starts one element before the slab
};
static_assert(sizeof(Slab) == 48, "Slab layout");

__host__ __device__ inline uint32_t slab_count(const Slab &sl) { return sl.e0 * sl.e1 * sl.e2; }

// Level coordinates of the cube at (fast, mid, slow) offsets (i0, i1, i2).
__host__ __device__ inline void slab_coords(const Slab &sl, uint32_t i0, uint32_t i1, uint32_t i2, uint32_t *x,
                                            uint32_t *y, uint32_t *z)
{
    // selects, not an indexed local array (which the device code would keep in scratch)
    const uint32_t f = sl.axes & 3, m = (sl.axes >> 2) & 3, w = (sl.axes >> 4) & 3;
    *x = sl.bx + (f == 0 ? i0 : 0u) + (m == 0 ? i1 : 0u) + (w == 0 ? i2 : 0u);
    *y = sl.by + (f == 1 ? i0 : 0u) + (m == 1 ? i1 : 0u) + (w == 1 ? i2 : 0u);
    *z = sl.bz + (f == 2 ? i0 : 0u) + (m == 2 ? i1 : 0u) + (w == 2 ? i2 : 0u);
}

// Clipped box: half-open ranges; returns false for an empty box.
__host__ __device__ inline bool clip_box(const uint32_t *b, const LevelTable &lt, uint32_t lo[3], uint32_t hi[3])
{
    bool ok = true;
    for (int a = 0; a < 3; ++a) {
        const uint64_t l = b[a], h = uint64_t(b[a]) + b[3 + a];
        lo[a] = uint32_t(l < lt.vol[a] ? l : lt.vol[a]);
        hi[a] = uint32_t(h < lt.vol[a] ? h : lt.vol[a]);
        ok = ok && lo[a] < hi[a];
    }
    return ok;
}

// One level's extents and its first element in maps: what the slab builder reads of the
// level table (a copy in LDS for the kernels, whose lanes each work on another level).
struct LevelRow {
    uint32_t X, Y, Z, pad;
    uint64_t off;
};

__host__ __device__ inline LevelRow level_row(const LevelTable &lt, uint32_t lev)
{
    return LevelRow{lt.dims[lev][0], lt.dims[lev][1], lt.dims[lev][2], 0u, lt.off[lev]};
}

// Least k with 2^k >= v (v >= 1, at most 2^31).
__host__ __device__ inline uint32_t ceil_log2(uint32_t v) { return v > 1 ? 32u - uint32_t(__builtin_clz(v - 1)) : 0u; }

// Segments per row of a kind-2 slab, as log2 of the power of two >= ceil(e0 / kRunSeg).
__host__ __device__ inline uint32_t run_lseg(uint32_t e0)
{
    return ceil_log2((e0 + kRunSeg - 1) / kRunSeg);
}

// The slab of level `lev` covering cells [x0, x1) x [y0, y1) x [z0, z1) (not empty): the
// fast axis is x (rows from maps) unless the block is thinner in x than in y
// (rows along y from maps_t); of the other two, the thinner is the slow axis.
// Level 0 uses the 16-bit copy when lt.use16.
__host__ __device__ inline Slab make_slab(const LevelTable &lt, const LevelRow &lr, uint32_t lev, uint32_t x0,
                                          uint32_t x1, uint32_t y0, uint32_t y1, uint32_t z0, uint32_t z1)
{
    const uint32_t ex = x1 - x0, ey = y1 - y0, ez = z1 - z0;
    Slab s;
    s.level = uint8_t(lev);
    s.bx = x0, s.by = y0, s.bz = z0;
    // fast axis f (x unless the block is thinner in x than in y), then mid m and slow w
    const uint32_t f = ex < ey ? 1u : 0u, ef = f ? ey : ex;
    uint32_t m, w, em, ew;
    if (f) {
        if (ez >= ex) m = 2, em = ez, w = 0, ew = ex;
        else m = 0, em = ex, w = 2, ew = ez;
    } else {
        if (ey >= ez) m = 1, em = ey, w = 2, ew = ez;
        else m = 2, em = ez, w = 1, ew = ey;
    }
    s.axes = uint8_t(f | (m << 2) | (w << 4));
    s.e0 = ef, s.e1 = em, s.e2 = ew;
    // rows from the runs (while the slab's (row, segment) items fit 32 bits)
    if (ef >= lt.run_min && ((lt.runs_mask >> (2 * lev + f)) & 1u) &&
        uint64_t(em) * ew * ((ef + kRunSeg - 1) / kRunSeg) < (1ull << 30)) {
        const uint32_t pitch = f ? lr.Z : lr.Y;  // rows of a slice: z (f: y fast) or y
        const bool in_slice = f ? m == 2 : m == 1;
        s.kind = 2, s.odd = uint8_t(run_lseg(ef)), s.units = f ? y0 : x0;
        s.s1b = in_slice ? 1u : pitch, s.s2b = in_slice ? pitch : 1u;
        s.base = (f ? z0 + pitch * x0 : y0 + pitch * z0) | uint64_t(0xFFFFFFFFu / em + 1) << 32;
        return s;
    }
    // element strides of the mid and slow axes in the chosen copy, and the first element
    const uint32_t X = lr.X, Y = lr.Y, Z = lr.Z;
    const bool pairs = lev == 0 && lt.use16;
    const uint32_t px = pairs ? lt.pitch_x : X, py = pairs ? lt.pitch_y : Y;
    s.kind = pairs ? 1 : 0;
    uint64_t sm, sw, first;
    if (f) {  // y fastest: element y + py (z + Z x)
        const uint64_t sz = py, sx = uint64_t(py) * Z;
        sm = m == 2 ? sz : sx, sw = m == 2 ? sx : sz;
        first = (pairs ? lt.total16 : lt.total + lr.off) + y0 + uint64_t(py) * (z0 + uint64_t(Z) * x0);
    } else {  // x fastest: element x + px (y + Y z)
        const uint64_t sy = px, sz = uint64_t(px) * Y;
        sm = m == 1 ? sy : sz, sw = m == 1 ? sz : sy;
        first = (pairs ? 0 : lr.off) + x0 + uint64_t(px) * (y0 + uint64_t(Y) * z0);
    }
    const uint32_t odd = pairs ? ((f == 1 ? y0 : x0) & 1u) : 0u;
    const uint32_t esz = pairs ? 2u : 4u;
    s.odd = uint8_t(odd);
    s.base = esz * (first - odd);
    s.s1b = em > 1 ? uint32_t(esz * sm) : 0u;  // < 2^32 whenever the extent is above 1
    s.s2b = ew > 1 ? uint32_t(esz * sw) : 0u;
    s.units = pairs ? (ef + odd + 1) >> 1 : ef;
    return s;
}

// Slab `face` (0 .. 5) of level `lev` of the box's footprint, if it holds any cube: the faces
// of the hollow shell (x low, x high, y low, y high, z low, z high, each cut short by the ones
// before it), or the whole block as face 0 where no coarser cube lies inside the box.
__host__ __device__ inline bool face_slab(const LevelTable &lt, const LevelRow &lr, const uint32_t lo[3],
                                          const uint32_t hi[3], uint32_t lev, uint32_t face, Slab *out)
{
    uint32_t a[3], b[3], ia[3], ib[3];
    bool outer = true, inner = true;
    for (int d = 0; d < 3; ++d) {
        const uint64_t one = uint64_t(1) << lev;
        a[d] = uint32_t((uint64_t(lo[d]) + one - 1) >> lev);
        b[d] = hi[d] >> lev;
        outer = outer && a[d] < b[d];
        const uint32_t pa = uint32_t((uint64_t(lo[d]) + 2 * one - 1) >> (lev + 1));
        const uint32_t pb = hi[d] >> (lev + 1);
        inner = inner && pa < pb;
        ia[d] = 2 * pa;
        ib[d] = 2 * pb;
    }
    if (!outer || (!inner && face > 0)) return false;
    uint32_t x0 = a[0], x1 = b[0], y0 = a[1], y1 = b[1], z0 = a[2], z1 = b[2];
    if (inner) {
        if (face == 0) x1 = ia[0];
        if (face == 1) x0 = ib[0];
        if (face >= 2) x0 = ia[0], x1 = ib[0];
        if (face == 2) y1 = ia[1];
        if (face == 3) y0 = ib[1];
        if (face >= 4) y0 = ia[1], y1 = ib[1];
        if (face == 4) z1 = ia[2];
        if (face == 5) z0 = ib[2];
    }
    if (x1 <= x0 || y1 <= y0 || z1 <= z0) return false;
    *out = make_slab(lt, lr, lev, x0, x1, y0, y1, z0, z1);
    return true;
}

// Tiles of a streamed slab (kind 0 or 1). A tile is what a wave loads at once, one 4-byte
// unit per lane: 2^ltx units of 2^(6 - ltx) rows, lane (lx, ly) = (lane mod 2^ltx,
// lane / 2^ltx). ltx is the smallest power of two that holds a row, at most 64 units; rows
// at least 2^24 bytes apart take one row per tile, so that a lane's byte offset is a 24-bit
// product below 2^32.
__host__ __device__ inline uint32_t tile_ltx(const Slab &sl)
{
    const uint32_t ltx = sl.units > 32 ? 6u : ceil_log2(sl.units);
    return sl.s1b >= (1u << 24) ? 6u : ltx;
}

__host__ __device__ inline uint32_t slab_tiles(const Slab &sl)
{
    if (sl.kind == 2) return 0;
    const uint32_t ltx = tile_ltx(sl), lty = 6u - ltx;
    return ((sl.units + (1u << ltx) - 1) >> ltx) * ((sl.e1 + (1u << lty) - 1) >> lty) * sl.e2;
}

// (row, segment) items of a slab summed from row runs.
__host__ __device__ inline uint32_t slab_items(const Slab &sl)
{
    return sl.kind == 2 ? (sl.e1 * sl.e2) << sl.odd : 0u;
}

// Lane src's value of v (all lanes active).
__device__ inline uint32_t lane_value(uint32_t v, uint32_t src)
{
    return uint32_t(__builtin_amdgcn_ds_bpermute(int(4 * src), int(v)));
}

// Inclusive sums over the lanes of a wave (all active), by DPP shifts inside rows of 16 lanes and
// two broadcasts across them.
__device__ inline uint32_t wave_sums(uint32_t v)
{
    v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x111, 0xF, 0xF, true));
    v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x112, 0xF, 0xF, true));
    v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x114, 0xF, 0xF, true));
    v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x118, 0xF, 0xF, true));
    v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x142, 0xA, 0xF, false));
    v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x143, 0xC, 0xF, false));
    return v;
}

// Wave 0 fills the slab table of one box in LDS, lane (level, face) one slab (two rounds
// where there are more than 64 such pairs), with the prefix sums of the slabs' tiles and run
// items (tile0 / item0, entry *n_slabs the totals; null: not wanted). `rows` holds the levels'
// extents in LDS. All threads may call; contains no barrier.
__device__ inline void build_slabs(const LevelTable &lt, const LevelRow *rows, const uint32_t lo[3],
                                   const uint32_t hi[3], Slab *slabs, int *n_slabs, uint32_t *tile0,
                                   uint32_t *item0)
{
    if (threadIdx.x >= 64) return;
    const uint32_t lane = threadIdx.x;
    uint32_t n = 0, tiles = 0, items = 0;
    for (uint32_t r = 0; r < 6 * lt.n_levels; r += 64) {
        const uint32_t id = r + lane, lev = (id * 43) >> 8;  // id / 6 (exact below 128)
        Slab sl;
        const bool have = lev < lt.n_levels && face_slab(lt, rows[lev], lo, hi, lev, id - 6 * lev, &sl);
        const uint64_t mask = __builtin_amdgcn_ballot_w64(have);
        const uint32_t at = n + __builtin_amdgcn_mbcnt_hi(uint32_t(mask >> 32),
                                                          __builtin_amdgcn_mbcnt_lo(uint32_t(mask), 0u));
        const uint32_t t1 = have ? slab_tiles(sl) : 0u, k1 = have ? slab_items(sl) : 0u;
        const uint32_t t = wave_sums(t1), k = wave_sums(k1);
        if (have) {
            slabs[at] = sl;
            if (tile0) tile0[at] = tiles + t - t1, item0[at] = items + k - k1;
        }
        n += uint32_t(__builtin_popcountll(mask));
        tiles += uint32_t(__builtin_amdgcn_readlane(int(t), 63));
        items += uint32_t(__builtin_amdgcn_readlane(int(k), 63));
    }
    if (lane == 0) {
        *n_slabs = int(n);
        if (tile0) tile0[n] = tiles, item0[n] = items;
    }
}

// ---------------------------------------------------------------- per-query state

// Per-query accumulators. Internal nodes of rank >= 3 live in an
// open-addressing table (key and voxel count, or, where they are pushed, mass and
// compensation); nodes of rank 1 (both predecessors are sources) and rank 2
// (predecessors of rank <= 1) never enter it: their voxels go straight to the
// sources by the node's record (Leaf). Sources keep an exact integer count (cubes
// whose node is a source, whole voxels of nodes of rank 1 and 2) plus fp32 mass with
// its compensation term: in dense mode in per-source arrays [S], in sparse mode
// (many sources) as entries of the same table. Pointers are into LDS or into a global per-worker region; the same
// code serves both (the compiler resolves the address space after inlining).
struct QueryState {
    uint32_t *keys;     // [cap] node ID or kEmpty
    uint32_t *cnt;      // [cap] exact integer counts: of source entries (sparse mode) and, with
                        // `counts`, of nodes
    float *hi, *lo;     // [cap] mass and its compensation (sources in sparse mode, nodes to be pushed)
    bool counts;        // nodes collect voxel counts, to be expanded by rows; else mass, to be pushed
    uint32_t *used;     // [cap] slots in insertion order
    uint32_t *n_used;   // scalar
    uint32_t *flags;    // scalar: bit 0 = overflow
    uint32_t *max_key;  // scalar: largest node ID inserted
    uint32_t cap;       // power of two
    uint32_t limit;     // load-factor cap on n_used
    uint32_t *seg_cnt;  // [S] exact integer counts (dense mode)
    float *seg_hi, *seg_lo;  // [S] pushed mass and its compensation (dense mode)
    Slab *slabs;        // [6 * levels] the box's slabs (LDS)
    uint32_t *tile0, *item0;  // [6 * levels + 1] tiles and run items before each slab (LDS)
    float *seg_var;     // [S] accumulated variance per source (uncertainty queries), or null
    uint32_t cls, n_cls;  // only nodes of class cls of n_cls (a power of two) count; 1: every node
};

// A node of rank 1 or 2 by its sources: (1 - w) of it goes to the a side, w to the b side;
// the a side is (1 - wa) s[0] + wa s[1], the b side (1 - wb) s[2] + wb s[3]. A side that is a
// source itself has weight 0 (and names it twice); every other weight is above 0. One 32-byte
// record instead of the node's triple and then its predecessors': a node met on a cube costs one
// load latency and one cache line, where rank 2 took two in a row and three lines.
struct Leaf {
    uint32_t s[4];
    float w, wa, wb;
    uint32_t pad;
};
static_assert(sizeof(Leaf) == 32, "Leaf must stay 32 bytes");

struct DeepEntry {
    uint32_t seg;
    float val;
};

struct GraphView {
    const NodeTriple *__restrict__ nodes;
    const Leaf *__restrict__ leaf;   // [node - nseg] for the nodes of rank 1 and 2
    const uint64_t *__restrict__ runs;   // the graph's first run: RunLevel::first counts from here
    // mixtures of the nodes of rank >= 3 by their sources (node n: entries deep_ptr[n - r2_end] ..
    // deep_ptr[n - r2_end + 1]), or null
    const uint32_t *__restrict__ deep_ptr;
    const DeepEntry *__restrict__ deep;
    uint32_t nseg;     // sources are IDs [0, nseg)
    uint32_t r1_end;   // rank-1 nodes are IDs [nseg, r1_end)
    uint32_t r2_end;   // rank-2 nodes are IDs [r1_end, r2_end)
};

// Loads of per-query state written by other threads of the block: relaxed
// agent-scope atomics, so that the global-memory variant reads L2 rather than
// a possibly stale L1 line (in LDS these are plain ds_read).
template <class T>
__device__ inline T ld(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The stores that go with them.
template <class T>
__device__ inline void st_atomic(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline uint32_t hash_node(uint32_t k)
{
    k ^= k >> 16;
    k *= 0x7feb352dU;
    k ^= k >> 15;
    k *= 0x846ca68bU;
    k ^= k >> 16;
    return k;
}

// Class of a node where a box's nodes are dealt to several workgroups (by bits of the hash
// that the table's slots do not use).
__device__ inline uint32_t node_class(uint32_t key, uint32_t n_cls) { return (hash_node(key) >> 24) & (n_cls - 1); }

// Slot of node `key`, inserting it if absent. Returns kEmpty on overflow.
__device__ inline uint32_t table_slot(const QueryState &st, uint32_t key)
{
    const uint32_t mask = st.cap - 1;
    uint32_t slot = hash_node(key) & mask;
    for (uint32_t probe = 0; probe < st.cap; ++probe) {
        const uint32_t k = ld(&st.keys[slot]);
        if (k == key) return slot;
        if (k == kEmpty) {
            const uint32_t old = atomicCAS(&st.keys[slot], kEmpty, key);
            if (old == kEmpty) {
                const uint32_t idx = atomicAdd(st.n_used, 1u);
                st.used[idx] = slot;
                if (!st.counts) atomicMax(st.max_key, key);  // (only the push needs it)
                if (idx >= st.limit) atomicOr(st.flags, 1u);
                return slot;
            }
            if (old == key) return slot;
        }
        slot = (slot + 1) & mask;
    }
    atomicOr(st.flags, 1u);
    return kEmpty;
}

// Compensated accumulation: the atomic returns the value it added to, so the
// exact rounding error of that addition is recovered with two-sum and
// accumulated, with the incoming compensation, in the second word.
__device__ inline void add_mass_at(float *hi, float *lo, float h, float l)
{
    const float old = atomicAdd(hi, h);
    const float s = old + h;
    const float bp = s - old;
    const float e = (old - (s - bp)) + (h - bp);
    atomicAdd(lo, e + l);
}

// w * (h + l) as an unevaluated pair: exact product error via fma, plus w * l.
__device__ inline void scale_pair(float w, float h, float l, float *oh, float *ol)
{
    const float p = w * h;
    *oh = p;
    *ol = fmaf(w, h, -p) + w * l;
}

template <bool SPARSE>
__device__ inline void add_source_count(const QueryState &st, uint32_t s, uint32_t c)
{
    if (SPARSE) {
        const uint32_t slot = table_slot(st, s);
        if (slot != kEmpty) atomicAdd(&st.cnt[slot], c);
    } else {
        atomicAdd(&st.seg_cnt[s], c);
    }
}

template <bool SPARSE>
__device__ inline void add_source_mass(const QueryState &st, uint32_t s, float h, float l)
{
    if (SPARSE) {
        const uint32_t slot = table_slot(st, s);
        if (slot != kEmpty) add_mass_at(&st.hi[slot], &st.lo[slot], h, l);
    } else {
        add_mass_at(&st.seg_hi[s], &st.seg_lo[s], h, l);
    }
}

// Mass (h, l) on one side of a node of rank 1 or 2.
template <bool SPARSE>
__device__ inline void push_side(const QueryState &st, uint32_t s0, uint32_t s1, float w, float h, float l)
{
    if (w == 0.0f) {
        add_source_mass<SPARSE>(st, s0, h, l);
        return;
    }
    float ah, al, bh, bl;
    scale_pair(1.0f - w, h, l, &ah, &al);
    scale_pair(w, h, l, &bh, &bl);
    add_source_mass<SPARSE>(st, s0, ah, al);
    add_source_mass<SPARSE>(st, s1, bh, bl);
}

// Mass (h, l) on a node of rank 1 or 2, straight to its sources.
template <bool SPARSE>
__device__ inline void push_leaf(const QueryState &st, const Leaf &t, float h, float l)
{
    float ah, al, bh, bl;
    scale_pair(1.0f - t.w, h, l, &ah, &al);
    scale_pair(t.w, h, l, &bh, &bl);
    push_side<SPARSE>(st, t.s[0], t.s[1], t.wa, ah, al);
    push_side<SPARSE>(st, t.s[2], t.s[3], t.wb, bh, bl);
}

// Mass pushed into `node` during the reverse push. Nodes of rank <= 2 go straight
// to the sources; only nodes of rank >= 3 accumulate in the table.
template <bool SPARSE>
__device__ inline void route_mass(const QueryState &st, const GraphView &gv, uint32_t node, float h, float l)
{
    if (node < gv.nseg) {
        add_source_mass<SPARSE>(st, node, h, l);
    } else if (node < gv.r2_end) {
        push_leaf<SPARSE>(st, gv.leaf[node - gv.nseg], h, l);
    } else {
        const uint32_t slot = table_slot(st, node);
        if (slot != kEmpty) add_mass_at(&st.hi[slot], &st.lo[slot], h, l);
    }
}

// Integer voxel count c (< 2^32) scattered onto `node` by cubes.
template <bool SPARSE>
__device__ inline void scatter_count(const QueryState &st, const GraphView &gv, uint32_t node, uint32_t c)
{
    if (node < gv.nseg) {
        add_source_count<SPARSE>(st, node, c);
        return;
    }
    if (st.n_cls > 1 && node_class(node, st.n_cls) != st.cls) return;
    const float h = float(c & 0xFFFFFF00u), l = float(c & 0xFFu);  // both exact in fp32
    if (node < gv.r2_end) {
        push_leaf<SPARSE>(st, gv.leaf[node - gv.nseg], h, l);
    } else {
        const uint32_t slot = table_slot(st, node);
        if (slot == kEmpty) return;
        if (st.counts) atomicAdd(&st.cnt[slot], c);
        else add_mass_at(&st.hi[slot], &st.lo[slot], h, l);
    }
}

__device__ inline uint64_t lane_above_mask()
{
    const uint32_t lane = threadIdx.x & 63;
    return lane == 63 ? 0 : (~uint64_t(0) << (lane + 1));
}

// Run starts of a wave: lane 0, and every lane whose value differs from lane
// i-1's (DPP wave shift right by one lane; the shift fills lane 0 with 0, and
// lane 0 is a start regardless). Returned as the wave mask of start lanes,
// taken straight from the vector compare.
__device__ inline uint64_t run_starts(uint32_t v, uint32_t *prev_out)
{
    const uint32_t prev = uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x138, 0xF, 0xF, true));
    *prev_out = prev;
    return __builtin_amdgcn_uicmp(v, prev, 33 /* ne */) | 1u;
}

// Distance from this lane to the next run start above it (64 if none):
// the length of the run this lane starts. `above` = lane_above_mask().
__device__ inline uint32_t run_len(uint64_t starts, uint64_t above, uint32_t lane)
{
    const uint64_t m = starts & above;
    return (m ? uint32_t(__builtin_ctzll(m)) : 64u) - lane;
}

// Run-length merge of equal neighbours in a wave: true at the start lane of a
// run of a real value (not kEmpty), with the run's length in *len.
__device__ inline bool run_head(uint32_t v, uint64_t above, uint32_t *len)
{
    const uint32_t lane = threadIdx.x & 63;
    uint32_t prev;
    const uint64_t starts = run_starts(v, &prev);
    *len = run_len(starts, above, lane);
    return (v != prev || lane == 0) && v != kEmpty;
}

__device__ inline uint32_t uni(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// ---------------------------------------------------------------- tiled slab walk (naive scan)
//
// The naive scan's box is read as e2 slices of e1 rows of `units` 4-byte units (32-bit node
// IDs, or aligned pairs of 16-bit level-0 IDs). A wave covers a tile of 2^ltx
// units x 2^(6 - ltx) rows (lane (lx, ly) = (lane mod 2^ltx, lane / 2^ltx)),
// and a block is UNROLL tiles stacked along the rows, so a lane's UNROLL loads
// are independent and all in flight together. Blocks (t0, rb, k2) are dealt
// to the waves round-robin. The row of tile u is a wave-uniform pointer (scalar
// registers): the block's first row plus u row steps; a lane adds its 32-bit
// byte offset. Row tiles that start past the slab's last row are not consumed
// (the wave-uniform bound n_u) and load from the last tile that starts inside
// it; lanes outside the slab read their tile's first unit (inside the slab) and
// see kEmpty, so every load stays inside the slab. The same helpers give the
// addresses to the kernel and to the host-side replay (mg_check_load_addresses).

struct TileWalk {
    uint32_t units, e1, e2;   // units per row, rows per slice, slices
    uint32_t s1b;             // bytes between rows
    uint64_t s2b;             // bytes between slices
    uint32_t ltx, lty, ty;    // tile: 2^ltx units x ty = 2^lty rows
    uint32_t rows;            // rows per block (ty * UNROLL)
    uint32_t n_t0, n_rb, n_blk;
    uint64_t row_step;        // bytes between the rows of tiles u and u + 1
};

__host__ __device__ inline TileWalk tile_walk(uint32_t units, uint32_t e1, uint32_t e2, uint32_t s1b, uint64_t s2b,
                                              uint32_t unroll)
{
    TileWalk w;
    w.units = units, w.e1 = e1, w.e2 = e2, w.s1b = s1b, w.s2b = s2b;
    uint32_t ltx = 0;
    while (ltx < 6 && (1u << ltx) < units) ++ltx;   // smallest power of two >= units, at most 64
    if (s1b >= (1u << 26)) ltx = 6;                 // one row per tile: lane offsets stay below 2^32
    w.ltx = ltx;
    w.lty = 6u - ltx;
    w.ty = 1u << w.lty;
    w.rows = w.ty * unroll;
    w.n_t0 = (units + (1u << ltx) - 1) >> ltx;
    w.n_rb = (e1 + w.rows - 1) / w.rows;
    w.n_blk = w.n_t0 * w.n_rb * e2;
    w.row_step = uint64_t(w.ty) * s1b;
    return w;
}

// Byte offset, from the slab's first unit, of block (t0, rb, k2)'s first row.
__host__ __device__ inline uint64_t tile_block_offset(const TileWalk &w, uint32_t t0, uint32_t rb, uint32_t k2)
{
    return uint64_t(rb) * w.rows * w.s1b + uint64_t(k2) * w.s2b + (uint64_t(t0) << w.ltx) * 4u;
}

// Row tiles of block row rb that start inside the slab (>= 1 for rb < n_rb).
__host__ __device__ inline uint32_t tile_n_u(const TileWalk &w, uint32_t rb, uint32_t unroll)
{
    const uint32_t n = (w.e1 - rb * w.rows + w.ty - 1) >> w.lty;
    return n < unroll ? n : unroll;
}

// A lane's byte offset inside its tile (< 2^32: ly < 64 and s1b < 2^26 unless ly == 0).
__host__ __device__ inline uint32_t tile_lane_bytes(const TileWalk &w, uint32_t lane)
{
    return (lane >> w.ltx) * w.s1b + (lane & ((1u << w.ltx) - 1)) * 4u;
}

// Its unit index along the row in tile column t0.
__host__ __device__ inline uint32_t tile_unit(const TileWalk &w, uint32_t t0, uint32_t lane)
{
    return (t0 << w.ltx) + (lane & ((1u << w.ltx) - 1));
}

// Row tiles of block (t0, rb) in which the lane's unit lies inside the slab (<= n_u).
__host__ __device__ inline uint32_t tile_n_ok(const TileWalk &w, uint32_t t0, uint32_t rb, uint32_t lane)
{
    const uint32_t row0 = rb * w.rows + (lane >> w.ltx);
    return (tile_unit(w, t0, lane) < w.units && row0 < w.e1) ? ((w.e1 - row0 + w.ty - 1) >> w.lty) : 0u;
}

// The byte offset of load u of a lane in block (t0, rb, k2): the tile row stays on
// tile n_u - 1 past it, and lanes outside the slab read the tile's first unit.
__host__ __device__ inline uint64_t tile_load_offset(const TileWalk &w, uint64_t blk, uint32_t u, uint32_t n_u,
                                                     uint32_t n_ok, uint32_t lane_bytes)
{
    return blk + uint64_t(u < n_u ? u : n_u - 1) * w.row_step + (u < n_ok ? lane_bytes : 0u);
}

// Which elements of a 16-bit pair unit lie in the slab (bit 0: low, bit 1: high); the
// row's first unit starts one element early when `odd`.
__host__ __device__ inline uint32_t pair_bits(uint32_t unit, uint32_t e0, uint32_t odd)
{
    return ((unit > 0 || odd == 0) ? 1u : 0u) | ((2 * unit + 1 < e0 + odd) ? 2u : 0u);
}

// The naive scan's walk of a clipped box: level 0 as one slab of ez slices of ey rows,
// from the 16-bit x-fastest copy (pairs; *odd = parity of the first x) or the 32-bit
// map; *base = byte offset of the first unit.
__host__ __device__ inline TileWalk naive_walk(const LevelTable &lt, const uint32_t lo[3], const uint32_t hi[3],
                                               bool use16, uint32_t unroll, uint64_t *base, uint32_t *odd)
{
    const uint32_t ex = hi[0] - lo[0], ey = hi[1] - lo[1], ez = hi[2] - lo[2];
    if (use16) {
        const uint64_t px = lt.pitch_x, pxy = px * lt.vol[1];
        *odd = lo[0] & 1u;
        *base = 2 * (lo[0] - *odd + px * lo[1] + pxy * lo[2]);
        return tile_walk((ex + *odd + 1) >> 1, ey, ez, ey > 1 ? uint32_t(2 * px) : 0u, ez > 1 ? 2 * pxy : 0u, unroll);
    }
    const uint64_t X = lt.vol[0], XY = X * lt.vol[1];
    *odd = 0;
    *base = 4 * (lo[0] + X * lo[1] + XY * lo[2]);
    return tile_walk(ex, ey, ez, ey > 1 ? uint32_t(4 * X) : 0u, ez > 1 ? 4 * XY : 0u, unroll);
}

// Streams a slab of 32-bit node IDs; `use(v)` consumes each of a block's n_u
// values (every lane calls it, kEmpty outside the slab). The next block's loads
// are in flight while a block is consumed. Blocks are dealt round-robin to the
// waves.
template <int UNROLL, int WAVES, class Use>
__device__ inline void stream_slab(const char *__restrict__ p, const TileWalk &tw, Use use)
{
    const uint32_t lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6);  // the wave index is uniform
    const uint32_t lane_bytes = tile_lane_bytes(tw, lane);
    uint32_t fb = wave;
    if (fb >= tw.n_blk) return;
    // block fb < WAVES as (t0, rb, k2), by subtraction (no division)
    uint32_t t0 = fb, rb = 0, k2 = 0;
    while (t0 >= tw.n_t0) {
        t0 -= tw.n_t0;
        if (++rb == tw.n_rb) rb = 0, ++k2;
    }
    auto load = [&](uint32_t (&v)[UNROLL], uint32_t &n_u, uint32_t &n_ok, uint32_t bt0, uint32_t brb,
                    uint32_t bk2) {
        n_u = tile_n_u(tw, brb, UNROLL);
        __builtin_assume(n_u >= 1);  // brb < n_rb: the block's first tile starts inside the slab
        n_ok = tile_n_ok(tw, bt0, brb, lane);
        const char *blk = p + tile_block_offset(tw, bt0, brb, bk2);
        const char *row = blk;
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            if (u > 0 && uint32_t(u) < n_u) row += tw.row_step;  // stays on tile n_u - 1 after it
            v[u] = *reinterpret_cast<const uint32_t *>(row + (uint32_t(u) < n_ok ? lane_bytes : 0u));
        }
    };
    uint32_t v[UNROLL], n_u, n_ok;
    load(v, n_u, n_ok, t0, rb, k2);
    for (; fb < tw.n_blk; fb += WAVES) {
        // this wave's next block; after its last one, the current block again (loaded, unused)
        uint32_t nt0 = t0 + WAVES, nrb = rb, nk2 = k2;
        while (nt0 >= tw.n_t0) {
            nt0 -= tw.n_t0;
            if (++nrb == tw.n_rb) nrb = 0, ++nk2;
        }
        const bool more = fb + WAVES < tw.n_blk;
        if (!more) nt0 = t0, nrb = rb, nk2 = k2;
        uint32_t w[UNROLL], w_n_u, w_n_ok;
        load(w, w_n_u, w_n_ok, nt0, nrb, nk2);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
            if (uint32_t(u) < n_u) use(uint32_t(u) < n_ok ? v[u] : kEmpty);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) v[u] = w[u];
        n_u = w_n_u, n_ok = w_n_ok;
        t0 = nt0, rb = nrb, k2 = nk2;
    }
}

// Streams a slab of the 16-bit level-0 copy, two elements per unit; `use(lo, hi)`
// gets 0xFFFF (no source: there are fewer than 65,535) for elements outside the slab (e0 elements per row, the row's first
// unit one element early when `odd`). Three blocks in flight (level 0 is most of
// the cubes, and its 32-bit words leave registers to spare): a block past the
// wave's last one is replaced by the block before it (valid addresses, never consumed).
template <int UNROLL, int WAVES, class Use>
__device__ inline void stream_pairs(const char *__restrict__ p, const TileWalk &tw, uint32_t e0, uint32_t odd,
                                    Use use)
{
    const uint32_t lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6);
    const uint32_t lane_bytes = tile_lane_bytes(tw, lane);
    uint32_t fb = wave;
    if (fb >= tw.n_blk) return;
    uint32_t t0 = fb, rb = 0, k2 = 0;
    while (t0 >= tw.n_t0) {
        t0 -= tw.n_t0;
        if (++rb == tw.n_rb) rb = 0, ++k2;
    }
    // n_lo / n_hi: row tiles in which this lane's low / high element is inside the slab
    auto load = [&](uint32_t (&v)[UNROLL], uint32_t &n_u, uint32_t &n_lo, uint32_t &n_hi, uint32_t bt0,
                    uint32_t brb, uint32_t bk2) {
        n_u = tile_n_u(tw, brb, UNROLL);
        __builtin_assume(n_u >= 1);
        const uint32_t n_ok = tile_n_ok(tw, bt0, brb, lane);
        const uint32_t pb = pair_bits(tile_unit(tw, bt0, lane), e0, odd);
        n_lo = (pb & 1u) ? n_ok : 0u;
        n_hi = (pb & 2u) ? n_ok : 0u;
        const char *blk = p + tile_block_offset(tw, bt0, brb, bk2);
        const char *row = blk;
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            if (u > 0 && uint32_t(u) < n_u) row += tw.row_step;
            v[u] = *reinterpret_cast<const uint32_t *>(row + (uint32_t(u) < n_ok ? lane_bytes : 0u));
        }
    };
    auto advance = [&](uint32_t &bt0, uint32_t &brb, uint32_t &bk2) {
        bt0 += WAVES;
        while (bt0 >= tw.n_t0) {
            bt0 -= tw.n_t0;
            if (++brb == tw.n_rb) brb = 0, ++bk2;
        }
    };
    uint32_t v[UNROLL], n_u, n_lo, n_hi;
    load(v, n_u, n_lo, n_hi, t0, rb, k2);
    uint32_t t1 = t0, rb1 = rb, k21 = k2;
    if (fb + WAVES < tw.n_blk) advance(t1, rb1, k21);
    uint32_t w[UNROLL], w_n_u, w_n_lo, w_n_hi;
    load(w, w_n_u, w_n_lo, w_n_hi, t1, rb1, k21);
    for (; fb < tw.n_blk; fb += WAVES) {
        uint32_t t2 = t1, rb2 = rb1, k22 = k21;
        if (fb + 2 * WAVES < tw.n_blk) advance(t2, rb2, k22);
        uint32_t x[UNROLL], x_n_u, x_n_lo, x_n_hi;
        load(x, x_n_u, x_n_lo, x_n_hi, t2, rb2, k22);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
            if (uint32_t(u) < n_u)
                use(uint32_t(u) < n_lo ? (v[u] & 0xFFFFu) : 0xFFFFu, uint32_t(u) < n_hi ? (v[u] >> 16) : 0xFFFFu);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) v[u] = w[u], w[u] = x[u];
        n_u = w_n_u, n_lo = w_n_lo, n_hi = w_n_hi;
        w_n_u = x_n_u, w_n_lo = x_n_lo, w_n_hi = x_n_hi;
        t1 = t2, rb1 = rb2, k21 = k22;
    }
}

// Counts a wave's 128 level-0 elements (lane l holds elements 2l and 2l+1) into
// integer per-source counters: a run of equal sources over elements a..b adds
// -a at its start element and b+1 at its end element (uint32 wrap-around); 0xFFFF marks
// an element outside.
__device__ inline void count_pairs(uint32_t *cnt, uint32_t lo, uint32_t hi, uint32_t lane)
{
    const uint32_t prev_hi = uint32_t(__builtin_amdgcn_update_dpp(0, int(hi), 0x138, 0xF, 0xF, true));
    const uint32_t next_lo = uint32_t(__builtin_amdgcn_update_dpp(0, int(lo), 0x130, 0xF, 0xF, true));
    const bool s_lo = lo != prev_hi || lane == 0;   // element 2l starts a run
    const bool e_lo = lo != hi;                     // element 2l ends one, 2l+1 starts one
    const bool e_hi = hi != next_lo || lane == 63;  // element 2l+1 ends one
    if (lo != 0xFFFFu && (s_lo || e_lo)) atomicAdd(&cnt[lo], (s_lo ? 0u - 2 * lane : 0u) + (e_lo ? 2 * lane + 1 : 0u));
    if (hi != 0xFFFFu && (e_lo || e_hi))
        atomicAdd(&cnt[hi], (e_lo ? 0u - (2 * lane + 1) : 0u) + (e_hi ? 2 * lane + 2 : 0u));
}

// A load through a pointer that was itself read from memory (the run table): the
// cast tells the compiler it is global memory, so it issues a global load rather
// than a flat one.
template <class T>
__device__ inline T load_global(const T *p)
{
    return *(const __attribute__((address_space(1))) T *)(p);
}

// The skip entries that bound the runs of cells [p0, p1) of row r: c0, that of p0's chunk, and the
// one after p1's chunk, *n entries on, which past the row's last chunk (*row_end) is the next
// row's first. True if that lies past the last row (the level's runs end there: no entry).
__host__ __device__ inline bool run_skips(uint32_t rows, uint32_t chunks, uint32_t r, uint32_t p0, uint32_t p1,
                                          uint64_t *c0, uint32_t *n, bool *row_end)
{
    const uint32_t k0 = p0 / kRunSkipCells, k1 = (p1 - 1) / kRunSkipCells + 1;
    *c0 = uint64_t(r) * chunks + k0;
    *n = k1 - k0;
    *row_end = k1 == chunks;
    return *row_end && r + 1 == rows;
}

// Item `it` of a kind-2 slab: its row index r in the level's runs and its cells [p0, p1) along
// the row; false for a padding item past the row. (row / e1 by the slab's reciprocal, rounded up:
// for the fewer than 2^30 rows of a slab the product is at most one too large.)
__host__ __device__ inline bool run_item(const Slab &sp, uint32_t it, uint32_t *r, uint32_t *p0, uint32_t *p1)
{
    const uint32_t lseg = sp.odd, c = it & ((1u << lseg) - 1), row = it >> lseg;
    uint32_t i2 = uint32_t((uint64_t(row) * uint32_t(sp.base >> 32)) >> 32);
    if (i2 * sp.e1 > row) --i2;
    *r = uint32_t(sp.base) + (row - i2 * sp.e1) * sp.s1b + i2 * sp.s2b;
    *p0 = sp.units + c * kRunSeg;
    *p1 = min(*p0 + kRunSeg, sp.units + sp.e0);
    return *p0 < *p1;
}

// Runs of cubes on internal nodes (dense state), deferred per wave: entries (node,
// run length | level << 9) in a ring in LDS, resolved 64 at a time, one per lane.
// Resolving one loads the node's record, so the loads of 64 runs are in flight
// together instead of one in nearly every step of a slab walk. At most 63 entries wait
// after an append; the ring holds those plus the 64 one append can add.
struct DeferRing {
    uint32_t *node;  // [waves][kDeferSlots]
    uint16_t *code;  // [waves][kDeferSlots]
    uint32_t wbase;  // this wave's ring (wave-uniform, as head and tail)
    uint32_t head;   // entries resolved
    uint32_t tail;   // entries appended
};

// A run of `len` cubes of level `lev` on internal node `node` (dense state). The
// node on a cube stands for the cube's own mixture, so the weight of a rank-1 or
// rank-2 node there is (voxels on the b side) / 8^lev: when w 8^lev is an integer
// k (levels <= 7, where the product is exact in fp32), the run's voxels split
// exactly into len (8^lev - k) on the a side and len k on the b side. A side that
// is a source takes its voxels as an integer count; a side that is a rank-1 node
// (rank 2 only) splits its n voxels per cube by its own weight w': n w' is a
// whole number of voxels (w' is a ratio of voxel counts of the mixtures the node
// serves) up to the fp32 rounding of w', which a distance to the nearest integer
// of at most n 2^-22 bounds, and that integer is the split. Any other weight (as
// in a quantized graph) pushes the mass instead. Both ranks read the node's one
// record (Leaf).
template <bool SPARSE>
__device__ inline void resolve_count(const QueryState &st, const GraphView &gv, uint32_t node, uint32_t len,
                                     uint32_t lev)
{
    if (!SPARSE && node < gv.r2_end) {
        const Leaf t = gv.leaf[node - gv.nseg];
        const uint32_t cube = 1u << (3u * lev);
        const float kf = t.w * float(cube);  // exact: a power-of-two scale
        const uint32_t k = uint32_t(kf);
        // voxels of one cube on the a side and the b side, and of those the ones on s[1] and s[3]
        const uint32_t na = cube - k, nb = k;
        const float fa = t.wa * float(na), fb = t.wb * float(nb), ra = rintf(fa), rb = rintf(fb);
        if (lev <= 7u && float(k) == kf && k <= cube && fabsf(fa - ra) <= float(na) * 0x1p-22f && ra >= 0.0f &&
            ra <= float(na) && fabsf(fb - rb) <= float(nb) * 0x1p-22f && rb >= 0.0f && rb <= float(nb)) {
            const uint32_t ma = uint32_t(ra), mb = uint32_t(rb);
            if (na != ma) atomicAdd(&st.seg_cnt[t.s[0]], len * (na - ma));
            if (ma) atomicAdd(&st.seg_cnt[t.s[1]], len * ma);
            if (nb != mb) atomicAdd(&st.seg_cnt[t.s[2]], len * (nb - mb));
            if (mb) atomicAdd(&st.seg_cnt[t.s[3]], len * mb);
            return;
        }
        const uint32_t c = len << (3u * lev);
        push_leaf<SPARSE>(st, t, float(c & 0xFFFFFF00u), float(c & 0xFFu));
        return;
    }
    scatter_count<SPARSE>(st, gv, node, len << (3u * lev));
}

// Resolves the n <= 64 oldest entries. Every lane of the wave must call.
template <bool SPARSE>
__device__ inline void ring_resolve(DeferRing &q, const QueryState &st, const GraphView &gv, uint32_t n)
{
    const uint32_t lane = threadIdx.x & 63;
    __builtin_amdgcn_wave_barrier();
    // nothing more into a table that has overflowed (a full one is probed end to end)
    if (lane < n && (ld(st.flags) & 1u) == 0) {
        const uint32_t k = q.wbase + ((q.head + lane) & (kDeferSlots - 1));
        const uint32_t code = q.code[k];
        resolve_count<SPARSE>(st, gv, q.node[k], code & 511u, code >> 9);
    }
    q.head += n;
    // vmcnt(0): no load of a resolve is left pending on any path out of it. Without it the
    // compiler waits for all loads, the walk's prefetched tiles among them, wherever a register
    // is used again that some path of a resolve loaded, which is in every step of the walk.
    __builtin_amdgcn_s_waitcnt(0x0f70);
    __builtin_amdgcn_wave_barrier();
}

// Appends a run of `len` (<= 256) cubes of level `lev` on `node` from each lane
// with `want`; resolves 64 entries once 64 wait. Every lane of the wave must call.
template <bool SPARSE>
__device__ inline void ring_put(DeferRing &q, const QueryState &st, const GraphView &gv, bool want, uint32_t node,
                                uint32_t len, uint32_t lev)
{
    const uint64_t put = __builtin_amdgcn_ballot_w64(want);
    if (put == 0) return;
    if (want) {
        const uint32_t below =
            __builtin_amdgcn_mbcnt_hi(uint32_t(put >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(put), 0u));
        const uint32_t k = q.wbase + ((q.tail + below) & (kDeferSlots - 1));
        q.node[k] = node;
        q.code[k] = uint16_t(len | (lev << 9));
    }
    q.tail += uint32_t(__builtin_popcountll(put));
    if (q.tail - q.head >= 64u) ring_resolve<SPARSE>(q, st, gv, 64u);
}

// ---------------------------------------------------------------- scatter
//
// Every cube of every slab adds 8^level to its node. The work of a box is one
// sequence of tiles (the streamed slabs, slab after slab) and one of (row, segment)
// items (the slabs summed from row runs); each wave that answers the box (of one
// workgroup, or of several that share it) takes contiguous pieces of both. A
// wave so meets few slabs instead of a share of every one: a box of 25,000 cubes has
// ~30 slabs, most of them a tile or two, and walking all of them with every wave
// cost one exposed load latency per slab and wave. What bounds it is the issue of
// vector instructions (about 75 per tile, 45 per 64 runs), so rows go to runs from
// kRunMinRow cubes on. 100,000 boxes of a 512^3 volume, default launch: 2.82 ms with
// the waves of a box dealt the blocks of every slab in turn and one lane per row
// segment, 1.54 ms so.

// One tile of a streamed slab: the byte offset of its first unit in its buffer, the bytes
// between its rows, and, packed: ltx (3 bits), units and rows of it inside the slab (7 bits
// each), level (5), kind (1), and whether its first unit's low element (23: kind 1, the row
// starts one element before the slab) or its last unit's high element (24) lies outside.
struct TileDesc {
    uint64_t off;
    uint32_t s1b, pack;
};

__host__ __device__ inline uint32_t tile_ltx_of(uint32_t pack) { return pack & 7u; }
__host__ __device__ inline uint32_t tile_units(uint32_t pack) { return (pack >> 3) & 127u; }
__host__ __device__ inline uint32_t tile_rows(uint32_t pack) { return (pack >> 10) & 127u; }
__host__ __device__ inline uint32_t tile_level(uint32_t pack) { return (pack >> 17) & 31u; }
__host__ __device__ inline bool tile_pairs(uint32_t pack) { return (pack >> 22) & 1u; }
constexpr uint32_t kTileSpan = (127u << 3) | (127u << 10);  // no unit inside: nothing to consume

// Tile `o` of a slab: along the row first, then down the rows, then the slices.
__host__ __device__ inline TileDesc tile_desc(const Slab &sl, uint32_t o)
{
    const uint32_t ltx = tile_ltx(sl), lty = 6u - ltx, ty = 1u << lty;
    const uint32_t n_t0 = (sl.units + (1u << ltx) - 1) >> ltx, n_rt = (sl.e1 + ty - 1) >> lty;
    uint32_t t0 = 0, r = o;
    if (n_t0 > 1) r = o / n_t0, t0 = o - r * n_t0;
    uint32_t rt = r, k2 = 0;
    if (sl.e2 > 1) k2 = r / n_rt, rt = r - k2 * n_rt;
    const uint32_t left = sl.units - (t0 << ltx), ucap = left < (1u << ltx) ? left : 1u << ltx;
    const uint32_t below = sl.e1 - (rt << lty), rcap = below < ty ? below : ty;
    const bool pairs = sl.kind == 1;
    TileDesc d;
    d.off = sl.base + uint64_t(k2) * sl.s2b + uint64_t(rt << lty) * sl.s1b + (uint64_t(t0) << ltx) * 4u;
    d.s1b = sl.s1b;
    d.pack = ltx | (ucap << 3) | (rcap << 10) | (uint32_t(sl.level) << 17) | (pairs ? 1u << 22 : 0u) |
             (pairs && sl.odd && t0 == 0 ? 1u << 23 : 0u) |
             (pairs && ((sl.e0 + sl.odd) & 1u) && t0 == n_t0 - 1 ? 1u << 24 : 0u);
    return d;
}

// A lane's byte offset in its tile (0, the tile's first unit, where its own unit is outside
// the slab: every load stays inside) and the bits its loaded word is OR-ed with: all ones in
// every part outside the slab, so that kEmpty (kind 0) or 0xFFFF (kind 1) marks it.
__host__ __device__ inline uint32_t tile_lane(uint32_t pack, uint32_t s1b, uint32_t lane, uint32_t *mask)
{
    const uint32_t ltx = tile_ltx_of(pack), lx = lane & ((1u << ltx) - 1), ly = lane >> ltx;
    const uint32_t ucap = tile_units(pack);
    const bool ok = lx < ucap && ly < tile_rows(pack);
    const uint32_t part = (((pack >> 23) & 1u) && lx == 0 ? 0xFFFFu : 0u) |
                          (((pack >> 24) & 1u) && lx + 1 == ucap ? 0xFFFF0000u : 0u);
    *mask = ok ? part : kEmpty;
#if defined(__HIP_DEVICE_COMPILE__)
    const uint32_t off = __umul24(ly, s1b) + lx * 4u;  // s1b < 2^24 unless ly == 0
#else
    const uint32_t off = ly * s1b + lx * 4u;
#endif
    return ok ? off : 0u;
}

// The slab that holds tile (or item) `t`, below the total in first[n_slabs]: the last one with
// first[i] <= t. (No branch in a step: one cost as much again in execution masks.)
__device__ inline uint32_t find_slab(const uint32_t *first, uint32_t n_slabs, uint32_t t)
{
    uint32_t i = n_slabs > 64 && first[64] <= t ? 64u : 0u;
#pragma unroll
    for (uint32_t step = 32; step > 0; step >>= 1)
        if (first[min(i + step, n_slabs)] <= t) i += step;
    return i;
}

// One wave's tiles [a, b), b > a. The descriptors of 64 tiles are computed at once, one per
// lane; a tile's load then takes its scalars from the lane that holds it. GROUP tiles are
// loaded while the GROUP before them are consumed (2 GROUP loads in flight per lane), across
// slabs and levels alike; past the range the last tile's first unit is loaded and not
// consumed.
template <int GROUP, bool SPARSE>
__device__ __attribute__((always_inline)) inline void stream_tiles(const char *maps, const char *maps16,
                                                                   const QueryState &st, const GraphView &gv,
                                                                   uint32_t n_slabs, uint32_t a, uint32_t b,
                                                                   DeferRing &dq, const uint32_t *flags_lds)
{
    typedef uint32_t Words __attribute__((ext_vector_type(GROUP)));
    const uint32_t lane = threadIdx.x & 63, nseg = gv.nseg;
    const uint64_t above = lane_above_mask();
    uint64_t d_at = 0;
    uint32_t d_s1b = 0, d_pack = 0;
    auto describe = [&](uint32_t first) {  // lane i: tile first + i
        const uint32_t t = min(first + lane, b - 1);
        const uint32_t i = find_slab(st.tile0, n_slabs, t);
        const TileDesc d = tile_desc(st.slabs[i], t - st.tile0[i]);
        d_at = reinterpret_cast<uint64_t>(tile_pairs(d.pack) ? maps16 : maps) + d.off;
        d_s1b = d.s1b;
        d_pack = first + lane < b ? d.pack : d.pack & ~kTileSpan;
    };
    auto load = [&](Words &v, Words &m, uint32_t i0) {  // tiles i0 .. i0 + GROUP - 1 of the described 64
#pragma unroll
        for (int u = 0; u < GROUP; ++u) {
            const int i = int(i0) + u;
            const uint64_t at = uint64_t(uint32_t(__builtin_amdgcn_readlane(int(uint32_t(d_at)), i))) |
                                (uint64_t(uint32_t(__builtin_amdgcn_readlane(int(uint32_t(d_at >> 32)), i))) << 32);
            const uint32_t s1b = uint32_t(__builtin_amdgcn_readlane(int(d_s1b), i));
            const uint32_t pack = uint32_t(__builtin_amdgcn_readlane(int(d_pack), i));
            uint32_t mask;
            const uint32_t off = tile_lane(pack, s1b, lane, &mask);
            typedef const __attribute__((address_space(1))) char *Global;
            v[u] = *(const __attribute__((address_space(1))) uint32_t *)(Global(at) + off);
            m[u] = mask;
        }
    };
    Words v, m;
    describe(a);
    load(v, m, 0);
    uint32_t packs = d_pack, i0 = 0;  // the descriptors and position of the group in v
    uint32_t iter = 0;
    for (uint32_t t = a; t < b; t += GROUP) {
        if ((++iter & 7u) == 0 && (uni(*flags_lds) & 1u)) return;  // overflowed: the box is redone elsewhere
        uint32_t n0 = i0 + GROUP;
        if (n0 == 64) {
            n0 = 0;
            describe(t + GROUP < b ? t + GROUP : b - 1);
            if (t + GROUP >= b) d_pack &= ~kTileSpan;
        }
        Words w, wm;
        load(w, wm, n0);
        const uint32_t n_u = min(uint32_t(GROUP), b - t);
#pragma unroll 1
        for (uint32_t u = 0; u < n_u; ++u) {
            const uint32_t pack = uint32_t(__builtin_amdgcn_readlane(int(packs), int(i0 + u)));
            const uint32_t x = v[u] | m[u];
            if (!SPARSE && tile_pairs(pack)) {  // level 0: every node is a source; two cubes per unit
                count_pairs(st.seg_cnt, x & 0xFFFFu, x >> 16, lane);
                continue;
            }
            const uint32_t lev = tile_level(pack), lw8 = 3 * lev;
            if (SPARSE) {
                // every insertion into a full table probes all of it (250,000 boxes of 15,917 fibres:
                // 1.5 s without this test in every step, 0.19 s with it)
                if (uni(ld(flags_lds)) & 1u) return;
                uint32_t len;
                if (run_head(x, above, &len)) scatter_count<SPARSE>(st, gv, x, len << lw8);
                continue;
            }
            // a run of lanes [a, b] on one source adds (b + 1 - a) 8^l as -a 8^l at its start
            // lane and (b + 1) 8^l at its end lane (uint32 wrap-around; the counts stay below
            // 2^32); neighbours by DPP wave shifts (lane 0 / lane 63 read 0 and are a start / an end)
            const uint32_t prev = uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x138, 0xF, 0xF, true));
            const uint32_t next = uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x130, 0xF, 0xF, true));
            const bool start = x != prev || lane == 0;
            const bool end = x != next || lane == 63;
            if (x < nseg) {  // a source (kEmpty is not)
                if (start) atomicAdd(&st.seg_cnt[x], 0u - (lane << lw8));
                if (end) atomicAdd(&st.seg_cnt[x], (lane + 1) << lw8);
            }
            // runs on internal nodes: a branch the wave skips unless a lane needs it
            // (wave masks straight from the vector compares: every lane is active here)
            const bool isint = x - nseg < kEmpty - nseg;
            const uint64_t internal = __builtin_amdgcn_uicmp(x - nseg, kEmpty - nseg, 36 /* ult */);
            if (internal != 0) {
                const uint64_t put = internal & (__builtin_amdgcn_uicmp(x, prev, 33 /* ne */) | 1u);
                const uint64_t ends = __builtin_amdgcn_uicmp(x, next, 33 /* ne */) | (1ull << 63);
                if (start && isint) {
                    // the run ends at the first end lane at or above this one
                    const uint32_t len = uint32_t(__builtin_ctzll(ends >> lane)) + 1u;
                    const uint32_t below = __builtin_amdgcn_mbcnt_hi(
                        uint32_t(put >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(put), 0u));
                    const uint32_t k = dq.wbase + ((dq.tail + below) & (kDeferSlots - 1));
                    dq.node[k] = x;
                    dq.code[k] = uint16_t(len | (lev << 9));
                }
                dq.tail += uint32_t(__builtin_popcountll(put));
                if (dq.tail - dq.head >= 64u) ring_resolve<SPARSE>(dq, st, gv, 64u);
            }
        }
        v = w, m = wm;
        packs = d_pack, i0 = n0;
    }
}

// One wave's run items [a, b). 64 items (one row segment each, at most kRunSeg cells) are
// described at once, one per lane: its cells [p0, p1), and from two skip entries the runs that
// may cross it (from the one holding the first cell of p0's chunk to the one holding the first
// cell past p1's chunk, or the row's last). The wave then takes the 64 items' runs as one
// sequence, a run per lane and step: every load is coalesced and issued one step ahead, and no
// lane waits for another's longer segment. (One lane per segment, four runs at a time, spent
// a load latency on every four runs of the longest of 64 segments.) A run starts where the one
// before it ends: the lane below's, the step before's for lane 0; of an item's first run every
// cell from p0 on counts.
// Which item a run of the step at s belongs to: the items that start in the 64 positions from s
// mark theirs in LDS (with a number of the step's own, so that no mark is ever cleared), and a lane
// counts the marks up to its own. (Six steps of a binary search through the lanes before: 40 of the
// 75 vector instructions of a step; 100,000 boxes of 512^3: 1.22 ms, 1.14 so,
// with find_slab, run_item and the prefix sums shortened as well.)
template <bool SPARSE>
__device__ __attribute__((always_inline)) inline void sum_runs(const RunLevel *runs, const QueryState &st,
                                                               const GraphView &gv, uint32_t n_slabs, uint32_t a,
                                                               uint32_t b, DeferRing &dq, uint32_t *marks,
                                                               uint32_t *tags, const uint32_t *flags_lds)
{
    const uint32_t lane = threadIdx.x & 63;
    uint32_t &tag = *tags;
    for (uint32_t b0 = a; b0 < b; b0 += 64) {
        if (uni(*flags_lds) & 1u) return;
        const uint32_t it = b0 + lane;
        // span: p0 (rows hold at most 2^15 cells), p1 - p0 << 16 (<= kRunSeg), level << 25
        uint32_t span = 0, j0 = 0, cnt = 0;
        if (it < b) {
            const uint32_t i = find_slab(st.item0, n_slabs, it);
            const Slab &sp = st.slabs[i];
            const uint32_t lev = sp.level;
            const RunLevel &rl = runs[2 * lev + (sp.axes & 3u)];
            uint32_t r, p0, p1;
            cnt = 1;  // a padding item: one place in the sequence, no cells
            if (run_item(sp, it - st.item0[i], &r, &p0, &p1)) {
                span = p0 | (p1 - p0) << 16 | lev << 25;
                uint64_t c0;
                uint32_t n;
                bool row_end;
                const bool last = run_skips(rl.rows, rl.chunks, r, p0, p1, &c0, &n, &row_end);
                const uint32_t *const skip = rl.skip + c0;
                const uint32_t lo = load_global(skip);
                uint32_t hi = last ? rl.n_runs : load_global(skip + n);  // a row's first run or one inside it
                if (row_end) --hi;                                       // the run before the next row's first
                hi = min(hi, rl.n_runs - 1);
                j0 = rl.first + lo;
                cnt = hi >= lo ? hi - lo + 1 : 1u;
            }
        }
        // position of each item's first run in the sequence
        uint32_t pos = wave_sums(cnt);
        const uint32_t total = uint32_t(__builtin_amdgcn_readlane(int(pos), 63));
        pos -= cnt;
        j0 -= pos;  // run index less position
        if (cnt == 0) pos = kEmpty;  // past the wave's items: starts nowhere
        uint32_t begun = 0;          // items that start before the step's positions
        auto fetch = [&](uint32_t s, uint64_t *v, uint32_t *sp, bool *first) {
            ++tag;
            const uint32_t d = pos - s;
            if (d < 64) marks[d] = tag;
            __builtin_amdgcn_wave_barrier();
            *first = marks[lane] == tag;
            __builtin_amdgcn_wave_barrier();
            const uint64_t m = __builtin_amdgcn_ballot_w64(*first);
            // marks at the positions up to this lane's own, as those below it of m shifted by one
            const uint32_t i = __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 33),
                                                         __builtin_amdgcn_mbcnt_lo(uint32_t(m >> 1),
                                                                                   begun - 1 + (uint32_t(m) & 1u)));
            begun += uint32_t(__builtin_popcountll(m));
            *v = load_global(gv.runs + (lane_value(j0, i) + min(s + lane, total - 1)));
            const uint32_t sc = lane_value(span, i);
            *sp = s + lane < total ? sc : 0u;  // no cells past the end
        };
        uint64_t v, w;
        uint32_t sp, sp1, carry = 0;
        bool first, first1;
        fetch(0, &v, &sp, &first);
        for (uint32_t s = 0; s < total; s += 64) {
            // (at or past the end: nothing starts, the last run again, not counted)
            fetch(s + 64, &w, &sp1, &first1);
            const uint32_t end = uint32_t(v >> 32), node = uint32_t(v), lv = sp >> 25;
            uint32_t begin = uint32_t(__builtin_amdgcn_update_dpp(int(carry), int(end), 0x138, 0xF, 0xF, false));
            carry = uint32_t(__builtin_amdgcn_readlane(int(end), 63));
            begin = max(first ? 0u : begin, sp & 0xFFFFu);
            const uint32_t to = min(end, (sp & 0xFFFFu) + ((sp >> 16) & 0x1FFu));
            const bool act = to > begin;
            const uint32_t len = to - begin;
            if (SPARSE) {
                if (uni(ld(flags_lds)) & 1u) return;
                if (act) scatter_count<SPARSE>(st, gv, node, len << (3 * lv));
            } else {
                if (act && node < gv.nseg) atomicAdd(&st.seg_cnt[node], len << (3 * lv));
                ring_put<SPARSE>(dq, st, gv, act && node >= gv.nseg, node, len, lv);
            }
            v = w, sp = sp1, first = first1;
        }
    }
}

// The waves of a workgroup share [0, n) of a box's tiles or items: each has one piece to begin with
// and takes the next from a counter in LDS when it is done with its last. WAVES pieces of half of what is left between
// them, then WAVES of half of the rest, and so on, and equal shares once those are below twice
// `least`: an item of a long row holds
// forty runs, one of a coarse level's three, and with one equal range per wave the waves of a box
// waited 27,000 of its 92,000 cycles for the last one (boxes of 2^14 cubes and more of a 512^3
// volume, 353 segments; anisotropic, 591 segments: 43,000 of 98,000).
template <uint32_t WAVES>
struct Pieces {
    uint32_t n, least, mult;            // pieces above `mult` are multiples of it
    uint32_t at = 0, first = 0, per;    // of the current round: first unit, first piece, units per piece
    uint32_t k;                         // the wave's first piece; then the last it took
    bool began = false;
    __device__ Pieces(uint32_t n_, uint32_t least_, uint32_t mult_, uint32_t k_) : n(n_), least(least_), mult(mult_), k(k_)
    {
        size();
    }
    __device__ void size()
    {
        const uint32_t left = n - at;
        per = left > 2 * WAVES * least ? left / (2 * WAVES) : (left + WAVES - 1) / WAVES;
        if (per > mult && left > 2 * WAVES * least) per -= per % mult;
    }
    // The wave's next piece [*a, *b); false when there is none.
    __device__ bool next(uint32_t *taken, uint32_t *a, uint32_t *b)
    {
        if (began) {
            if (n <= 2 * WAVES * least) return false;  // one share each
            uint32_t v = 0;
            if ((threadIdx.x & 63) == 0) v = atomicAdd(taken, 1u);
            k = WAVES + uni(v);
        }
        began = true;
        while (k - first >= WAVES) {
            at += WAVES * per, first += WAVES;
            if (at >= n) return false;
            size();
        }
        *a = at + (k - first) * per;
        if (*a >= n) return false;
        *b = min(n, *a + per);
        return true;
    }
};

// Part `part` of `parts` of a box's scatter, by one workgroup. Runs on sources add to an
// integer counter; runs on internal nodes go through the wave's deferral ring (dense state)
// or are scattered at once (sparse state).
template <int BLOCK, int GROUP, bool SPARSE>
__device__ __attribute__((always_inline)) inline void scatter_box(const char *maps, const char *maps16,
                                                                  const RunLevel *runs, const QueryState &st,
                                                                  const GraphView &gv, uint32_t n_slabs, uint32_t part, uint32_t parts,
                                                                  uint32_t *taken, const uint32_t *flags_lds)
{
    constexpr uint32_t kWaves = BLOCK / 64;
    __shared__ uint32_t dq_node[kWaves * (SPARSE ? 1u : kDeferSlots)];
    __shared__ uint16_t dq_code[kWaves * (SPARSE ? 1u : kDeferSlots)];
    __shared__ uint32_t marks[kWaves * 64];
    const uint32_t wave = uni(threadIdx.x >> 6);
    DeferRing dq{dq_node, dq_code, wave * kDeferSlots, 0u, 0u};
    // The part's range first, then the wave's range of it: a part is the same work whatever
    // the size of the workgroup that answers it.
    auto range = [&](uint32_t n, uint32_t least, uint32_t p, uint32_t of, uint32_t *a, uint32_t *b) {
        const uint32_t per = max(least, (n + of - 1) / of);
        *a = min(n, p * per), *b = min(n, *a + per);
    };
    const uint32_t tiles = uni(st.tile0[n_slabs]), items = uni(st.item0[n_slabs]);
    uint32_t t0 = 0, t1 = tiles, i0 = 0, i1 = items, a, b;
    if (parts > 1) {
        range(tiles, 1, part, parts, &t0, &t1);
        range(items, kLeastItems, parts - 1 - part, parts, &i0, &i1);  // from the end that got the fewer tiles
    }
    uint32_t tag = 0;
    marks[threadIdx.x] = 0;
    if constexpr (kWaves > 2) {
        Pieces<kWaves> tp(t1 - t0, kLeastTiles, GROUP, wave), ip(i1 - i0, kLeastRunItems, 64, kWaves - 1 - wave);
        while (tp.next(&taken[0], &a, &b))
            stream_tiles<GROUP, SPARSE>(maps, maps16, st, gv, n_slabs, t0 + a, t0 + b, dq, flags_lds);
        while (ip.next(&taken[1], &a, &b))
            sum_runs<SPARSE>(runs, st, gv, n_slabs, i0 + a, i0 + b, dq, marks + 64 * wave, &tag, flags_lds);
    } else {  // two waves, small boxes: one range each, from opposite ends
        range(t1 - t0, 1, wave, kWaves, &a, &b);
        if (a < b) stream_tiles<GROUP, SPARSE>(maps, maps16, st, gv, n_slabs, t0 + a, t0 + b, dq, flags_lds);
        range(i1 - i0, kLeastItems, kWaves - 1 - wave, kWaves, &a, &b);
        if (a < b)
            sum_runs<SPARSE>(runs, st, gv, n_slabs, i0 + a, i0 + b, dq, marks + 64 * wave, &tag, flags_lds);
    }
    if (!SPARSE && dq.tail != dq.head) ring_resolve<SPARSE>(dq, st, gv, dq.tail - dq.head);
}

// Reverse push through the nodes of rank >= 3 in the table, rank by rank from
// the highest present. All threads of the block must call.
template <int BLOCK, bool SPARSE>
__device__ inline void push_mass(const QueryState &st, const GraphView &gv, const uint32_t *rank_ptr_lds,
                                 uint32_t depth)
{
    const uint32_t nu = ld(st.n_used);
    if (nu == 0 || (ld(st.flags) & 1u)) return;  // uniform
    const uint32_t top_key = ld(st.max_key);
    if (top_key < gv.r2_end) return;  // only sources in the table: nothing to push
    uint32_t r = depth;
    while (r > 3 && rank_ptr_lds[r] > top_key) --r;
    for (; r >= 3; --r) {  // ranks <= 2 never enter the table
        const uint32_t lo_id = rank_ptr_lds[r], hi_id = rank_ptr_lds[r + 1];
        const uint32_t n_now = ld(st.n_used), over = ld(st.flags) & 1u;
        __syncthreads();  // every thread has read both before any insert of this rank
        if (over) return;
        for (uint32_t i = threadIdx.x; i < n_now; i += BLOCK) {
            // An overflowed table is full before long, and every insertion into a full one probes it
            // end to end (one box of 3.2 million voxels of noise, 2,000 sources, a graph of 6.3 million
            // nodes: 4.0 s pushing on into a full table of 65,536 slots, 15 ms so; a box of 52,000
            // voxels 9.5 and 0.85 ms).
            if (ld(st.flags) & 1u) break;
            const uint32_t slot = ld(&st.used[i]);
            const uint32_t key = ld(&st.keys[slot]);
            if (key < lo_id || key >= hi_id) continue;
            const float mh = ld(&st.hi[slot]), ml = ld(&st.lo[slot]);
            const NodeTriple t = gv.nodes[key];
            float ah, al, bh, bl;
            scale_pair(1.0f - t.w, mh, ml, &ah, &al);
            scale_pair(t.w, mh, ml, &bh, &bl);
            route_mass<SPARSE>(st, gv, t.a, ah, al);
            route_mass<SPARSE>(st, gv, t.b, bh, bl);
        }
        __syncthreads();
    }
}

// Mixture rows of the table's nodes: the graph's own of its nodes of rank >= 3 ...
struct DeepRows {
    typedef uint32_t Pos;
    typedef DeepEntry Entry;
    const uint32_t *__restrict__ ptr;
    const DeepEntry *__restrict__ row;
    uint32_t first;  // the first node that has one
    __device__ DeepRows(const GraphView &gv) : ptr(gv.deep_ptr), row(gv.deep), first(gv.r2_end) {}
    __device__ Pos begin(uint32_t node) const { return ptr[node - first]; }
    __device__ Entry entry(Pos j) const { return row[j]; }
};
// ... or the mixture lookup table's, of every node, with the uncertainties of a quantized graph.
template <bool ERR>
struct LutRows {
    typedef uint64_t Pos;
    struct Entry {
        uint32_t seg;
        float val, err;
    };
    const uint64_t *__restrict__ ptr;
    const uint32_t *__restrict__ seg;
    const float *__restrict__ val, *__restrict__ dev;
    uint32_t first;  // (with ERR r1_end is nseg: nodes of every rank enter the table)
    __device__ LutRows(const uint64_t *p, const uint32_t *s, const float *v, const float *e, const GraphView &gv)
        : ptr(p), seg(s), val(v), dev(e), first(gv.r1_end)
    {
    }
    __device__ Pos begin(uint32_t node) const { return ptr[node]; }
    __device__ Entry entry(Pos j) const { return Entry{seg[j], val[j], ERR ? dev[j] : 0.f}; }
};
__device__ inline uint64_t lane_value(uint64_t v, uint32_t src)
{
    return lane_value(uint32_t(v), src) | uint64_t(lane_value(uint32_t(v >> 32), src)) << 32;
}

// Expansion of the table's nodes: every node adds its voxel count times its
// mixture row to the sources. The nodes are dealt to the waves; a wave takes the entries of up
// to 64 nodes' rows as one sequence, one per lane and step (as sum_runs does with runs). One
// pass of independent additions instead of a pass per rank of the push, each with a table
// insertion or two per node: the part of a 205,000-cube box that held 147 such nodes pushed for
// 20,000 cycles. All threads of the block must call.
template <int BLOCK, bool SPARSE, bool ERR, class ROWS>
__device__ inline void expand_rows(const QueryState &st, const ROWS &rows)
{
    constexpr uint32_t kWaves = BLOCK / 64;
    const uint32_t nu = uni(ld(st.n_used)), over = uni(ld(st.flags)) & 1u;
    // (sparse state: the additions below insert sources, so n_used grows) every wave has read the
    // count that its range follows from, and of entries all of which are written, before any of them
    if (SPARSE) __syncthreads();
    if (nu == 0 || over) return;
    const uint32_t lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6);
    const uint32_t per = max(8u, (nu + kWaves - 1) / kWaves), n0 = min(nu, wave * per), n1 = min(nu, n0 + per);
    for (uint32_t b0 = n0; b0 < n1; b0 += 64) {
        uint32_t c = 0, len = 0;
        typename ROWS::Pos j0 = 0;
        if (b0 + lane < n1) {
            const uint32_t slot = ld(&st.used[b0 + lane]), key = ld(&st.keys[slot]);
            if (key >= rows.first) {  // (sparse mode: sources are entries too)
                j0 = rows.begin(key);
                len = uint32_t(rows.begin(key + 1) - j0);
                c = ld(&st.cnt[slot]);
            }
        }
        uint32_t pos = wave_sums(len);
        const uint32_t total = uint32_t(__builtin_amdgcn_readlane(int(pos), 63));
        if (total == 0) continue;
        pos -= len;
        j0 -= pos;
        auto fetch = [&](uint32_t s, typename ROWS::Entry *e, uint32_t *cc) {
            const uint32_t x = min(s + lane, total - 1);
            uint32_t i = 0;
#pragma unroll
            for (uint32_t step = 32; step > 0; step >>= 1)
                if (lane_value(pos, i + step) <= x) i += step;
            *e = rows.entry(lane_value(j0, i) + x);
            const uint32_t v = lane_value(c, i);
            *cc = s + lane < total ? v : 0u;
        };
        typename ROWS::Entry e, e1;
        uint32_t cc, cc1;
        fetch(0, &e, &cc);
        for (uint32_t s = 0; s < total; s += 64) {
            fetch(s + 64, &e1, &cc1);  // past the end: the last entry again, not added
            if (cc) {
                const float mh = float(cc & 0xFFFFFF00u), ml = float(cc & 0xFFu);  // both exact in fp32
                float ph, pl;
                scale_pair(e.val, mh, ml, &ph, &pl);
                add_source_mass<SPARSE>(st, e.seg, ph, pl);
                if constexpr (ERR) {
                    const float d = (mh + ml) * e.err;
                    atomicAdd(&st.seg_var[e.seg], d * d);
                }
            }
            e = e1, cc = cc1;
        }
    }
}

// Per-worker tables in global memory: node table and per-source arrays.
struct GlobalPool {
    uint32_t workers, slots;
    uint32_t *keys, *cnt, *used;
    float *hi, *lo;
    uint32_t *seg_cnt;
    float *seg_hi, *seg_lo, *seg_var;
};

struct QueryArgs {
    LevelTable lt;
    const uint32_t *boxes;
    float *out;                   // dense output [n][S], or nullptr for sparse output
    uint32_t *sp_index;           // sparse output: [n][2] (first entry, entries) per box
    uint32_t *sp_seg;             // sparse output: source of each entry
    float *sp_val;                // sparse output: fraction of each entry
    uint32_t sp_cap;              // entries sp_seg / sp_val hold
    uint32_t *sp_total;           // entries produced (may exceed sp_cap: then the rest are dropped)
    const uint32_t *maps;         // maps then maps_t
    const uint16_t *maps16;       // level 0 as 16-bit IDs (both orientations), if lt.use16
    const RunLevel *runs;         // [2 l + o] row runs of level l along x / y, where lt.runs_mask says
    GraphView gv;
    const uint32_t *rank_ptr;     // [depth + 2]
    uint32_t depth;
    uint32_t n;
    const uint32_t *order;        // query order (batched; kEmpty: a box whose parts are in `split`)
    uint32_t *counters;           // kCount* below
    uint32_t table_cap;           // LDS hash slots of this launch
    uint32_t chunk;               // small tier: boxes per dequeue (0: automatic)
    uint32_t *queues;             // tier work queues: counter of queue j at [j * kQueueStride]
    uint32_t *buckets;            // box counts by size, for the order
    uint32_t *overflow;           // list 1: boxes (and parts) whose LDS table overflowed
    uint32_t *overflow2;          // list 2: those no LDS table holds
    uint32_t *overflow3;          // list 3: those the mid-size global tables do not hold either
    // boxes that several workgroups share: their parts, and per box the sources' sums so far
    uint32_t n_slots;             // boxes there is room for (0: every box is one workgroup's)
    uint4 *split;                 // [2 n_slots] parts (box, part, parts, slot) of a planned call
    uint4 *split_over;            // [4 n_slots] parts in list 1 (entry: kPartFlag | index here)
    uint32_t *slot_done;          // [n_slots] parts finished
    uint32_t *slot_cnt;           // [n_slots][S] exact integer counts
    float *slot_hi, *slot_lo;     // [n_slots][S] mass and its compensation
    float *slot_var;              // [n_slots][S] variance (uncertainty queries)
    uint32_t *stats;              // optional [n][2]: cubes, table entries (graph nodes) touched
    uint32_t counts;              // nodes collect counts, expanded by rows; 0: mass, pushed rank by rank
    const uint64_t *lut_ptr;      // mixture lookup table rows, where the call names it (else nullptr)
    const uint32_t *lut_seg;
    const float *lut_val;
    const float *lut_err;         // propagated uncertainty of each row entry (uncertainty queries)
    float *out_err;               // [n][S] uncertainty of each fraction, or null (dense output only)
};

// Counters of a workspace. Every call leaves all of them (and the queues, buckets and slots)
// zero, so no call needs a launch to clear them.
enum : uint32_t {
    kCountOver = 1,     // entries of list 1
    kCountOver2 = 2,    // entries of list 2
    kCountOver3 = 3,    // entries of list 3
    kCountRetry = 4,    // next entry of list 1
    kCountNext2 = 5,    // next entry of list 2
    kCountNext3 = 6,    // next entry of list 3
    kCountBig = 8,      // boxes of the big tier
    kCountExit = 9,     // workgroups of the last launch that are done
    kCountSplit = 10,   // parts in `split`
    kCountSlot = 11,    // slots taken
    kCountSplitOver = 12,  // parts in the first half of `split_over`
    kCountRedo = 13,    // parts in its second half: boxes cut up after they overflowed
    kCountTotal = 14,   // cubes of all boxes (64 bits)
    kCountLayout = 32,  // the library's scratch: the layout it was last cleared for (ScratchLayout)
};
constexpr uint32_t kPartFlag = 0x80000000u;

// Dynamic LDS of the query kernels: per-source arrays (dense mode) and the table,
// then the slab list (6 per level) at a 16-byte aligned offset.
__host__ __device__ inline uint32_t lds_state_bytes(uint32_t nseg, uint32_t cap, bool sparse, bool counts)
{
    return ((sparse ? cap * 20u : nseg * 12u + cap * (counts ? 12u : 16u)) + 15u) & ~15u;
}
// The slab list and its two prefix arrays.
__host__ __device__ inline uint32_t lds_slab_bytes(uint32_t n_levels)
{
    return 6u * n_levels * uint32_t(sizeof(Slab)) + 2u * (6u * n_levels + 1u) * 4u;
}
__host__ __device__ inline uint32_t lds_bytes(uint32_t nseg, uint32_t cap, bool sparse, bool counts,
                                              uint32_t n_levels, bool err)
{
    return lds_state_bytes(nseg, cap, sparse, counts) + lds_slab_bytes(n_levels) + (err ? 4u * nseg : 0u);
}

struct QueryShared {
    uint32_t rank_ptr[kMaxSteps + 2];
    LevelRow rows[kMaxLevelsDev];          // extents of every level
    RunLevel runs[2 * kMaxLevelsDev];      // row runs of every level and orientation
    int n_slabs;
    uint32_t n_used;
    uint32_t flags;
    uint32_t max_key;
    uint32_t taken[2];  // pieces of the box's tiles and run items taken beyond the waves' first
    uint32_t q;
    uint32_t last;   // this workgroup finished its box's last part
    uint32_t nnz;    // sparse output: entries of this box
    uint32_t base;   // sparse output: first entry of this box
};

// Fraction of voxels of each source of one box, written to the dense row or
// appended to the sparse output. All threads of the block must call.
template <int BLOCK, bool SPARSE, bool ERR>
__device__ inline void write_result(const QueryArgs &A, QueryShared &sh, const QueryState &st, uint32_t q,
                                    bool nonempty, double vol)
{
    const uint32_t nseg = A.gv.nseg;
    if (!SPARSE && !A.out) {
        // per-source arrays, sparse output (the global-table launches): count the box's
        // non-zero sources, reserve their entries with one global atomic, write them
        if (threadIdx.x == 0) sh.nnz = 0;
        __syncthreads();
        // a source got voxels iff any of its three words is non-zero (mass below 256 voxels
        // can sit in the compensation word alone; an untouched source is exactly zero)
        uint32_t mine = 0;
        for (uint32_t s = threadIdx.x; s < nseg; s += BLOCK)
            mine += (ld(&st.seg_cnt[s]) | __float_as_uint(ld(&st.seg_hi[s])) | __float_as_uint(ld(&st.seg_lo[s]))) !=
                    0u;
        if (mine) atomicAdd(&sh.nnz, mine);
        __syncthreads();
        if (threadIdx.x == 0) {
            sh.base = sh.nnz ? atomicAdd(A.sp_total, sh.nnz) : 0u;
            A.sp_index[2 * uint64_t(q)] = sh.base;
            A.sp_index[2 * uint64_t(q) + 1] = sh.nnz;
            sh.nnz = 0;
        }
        __syncthreads();
        for (uint32_t s = threadIdx.x; s < nseg; s += BLOCK) {
            const uint32_t c_int = ld(&st.seg_cnt[s]);
            const float h = ld(&st.seg_hi[s]), l = ld(&st.seg_lo[s]);
            if ((c_int | __float_as_uint(h) | __float_as_uint(l)) == 0u) continue;
            const double c = double(c_int) + double(h) + double(l);
            const uint32_t pos = sh.base + atomicAdd(&sh.nnz, 1u);
            if (pos < A.sp_cap) {
                A.sp_seg[pos] = s;
                A.sp_val[pos] = float(c / vol);
            }
        }
        return;
    }
    if (!SPARSE) {
        float *o = A.out + uint64_t(q) * nseg;
        for (uint32_t s = threadIdx.x; s < nseg; s += BLOCK) {
            const double c = double(ld(&st.seg_cnt[s])) + double(ld(&st.seg_hi[s])) + double(ld(&st.seg_lo[s]));
            o[s] = nonempty ? float(c / vol) : 0.0f;
        }
        if (ERR) {
            float *e = A.out_err + uint64_t(q) * nseg;
            for (uint32_t s = threadIdx.x; s < nseg; s += BLOCK)
                e[s] = nonempty ? float(sqrt(double(ld(&st.seg_var[s]))) / vol) : 0.0f;
        }
        return;
    }
    const uint32_t nu = min(sh.n_used, st.cap);
    if (A.out) {
        float *o = A.out + uint64_t(q) * nseg;
        for (uint32_t s = threadIdx.x; s < nseg; s += BLOCK) o[s] = 0.0f;
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < nu; i += BLOCK) {
            const uint32_t slot = ld(&st.used[i]);
            const uint32_t key = ld(&st.keys[slot]);
            if (key >= nseg) continue;
            const double c = double(ld(&st.cnt[slot])) + double(ld(&st.hi[slot])) + double(ld(&st.lo[slot]));
            o[key] = float(c / vol);
        }
        return;
    }
    if (threadIdx.x == 0) sh.nnz = 0;
    __syncthreads();
    uint32_t mine = 0;
    for (uint32_t i = threadIdx.x; i < nu; i += BLOCK) mine += ld(&st.keys[ld(&st.used[i])]) < nseg;
    if (mine) atomicAdd(&sh.nnz, mine);
    __syncthreads();
    if (threadIdx.x == 0) {
        sh.base = sh.nnz ? atomicAdd(A.sp_total, sh.nnz) : 0u;
        A.sp_index[2 * uint64_t(q)] = sh.base;
        A.sp_index[2 * uint64_t(q) + 1] = sh.nnz;
        sh.nnz = 0;
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < nu; i += BLOCK) {
        const uint32_t slot = ld(&st.used[i]);
        const uint32_t key = ld(&st.keys[slot]);
        if (key >= nseg) continue;
        const double c = double(ld(&st.cnt[slot])) + double(ld(&st.hi[slot])) + double(ld(&st.lo[slot]));
        const uint32_t pos = sh.base + atomicAdd(&sh.nnz, 1u);
        if (pos < A.sp_cap) {
            A.sp_seg[pos] = key;
            A.sp_val[pos] = float(c / vol);
        }
    }
}

// Marks a box that no table could hold: NaN row (dense) or a NaN entry count.
template <int BLOCK>
__device__ inline void write_failure(const QueryArgs &A, uint32_t q)
{
    if (A.out) {
        float *o = A.out + uint64_t(q) * A.gv.nseg;
        for (uint32_t s = threadIdx.x; s < A.gv.nseg; s += BLOCK) o[s] = __builtin_nanf("");
    } else if (threadIdx.x == 0) {
        A.sp_index[2 * uint64_t(q)] = 0xFFFFFFFFu;
        A.sp_index[2 * uint64_t(q) + 1] = 0xFFFFFFFFu;
    }
}

// Cubes of a box's footprint, level by level in closed form (below 2^31, the volume's voxels).
__device__ inline uint32_t box_cubes(const LevelTable &lt, const uint32_t *box)
{
    uint32_t lo[3], hi[3], cubes = 0;
    if (!clip_box(box, lt, lo, hi)) return 0;
    for (uint32_t l = 0; l < lt.n_levels; ++l) {
        uint32_t outer = 1, inner = 1;
        for (int d = 0; d < 3; ++d) {
            const uint32_t one = 1u << l;  // extents are at most 2^15: no sum leaves 32 bits
            const uint32_t a = (lo[d] + one - 1) >> l, b = hi[d] >> l;
            const uint32_t pa = (lo[d] + 2 * one - 1) >> (l + 1), pb = hi[d] >> (l + 1);
            outer *= b > a ? b - a : 0u;
            inner *= pb > pa ? 2 * (pb - pa) : 0u;
        }
        if (outer == 0) break;  // nothing at coarser levels either
        cubes += outer - inner;
    }
    return cubes;
}

// Cubes above which a box is split, and the parts it is split into (about that many cubes
// each): the share of one of `ways` workgroups in all boxes' cubes, so that no workgroup
// works much longer than the others, but at least `least`. At most `ways` boxes exceed their
// share, in at most 2 `ways` parts.
__device__ inline uint32_t part_cubes(uint64_t total, uint32_t ways, uint32_t least)
{
    if (ways == 0) return 0xFFFFFFFFu;
    return uint32_t(max(uint64_t(least), min(total / ways + 1, uint64_t(0xFFFFFFFFu))));
}
__device__ inline uint32_t parts_of(uint32_t cubes, uint32_t target)
{
    return cubes > target ? (cubes + target - 1) / target : 1u;
}

// Zeroes what an entry of the table collects.
template <bool SPARSE>
__device__ inline void clear_entry(const QueryState &st, uint32_t slot)
{
    if (SPARSE || st.counts) st.cnt[slot] = 0;
    if (SPARSE || !st.counts) st.hi[slot] = 0.f, st.lo[slot] = 0.f;
}

// One box (parts == 1) or one part of a box that several workgroups share.
struct Item {
    uint32_t q, part, parts, slot;
};

__device__ inline Item whole_box(uint32_t q) { return Item{q, 0u, 1u, 0u}; }
__device__ inline Item part_of(const uint4 &p) { return Item{p.x, p.y, p.z, p.w}; }

// The item of a list-1 (or list-2) entry.
__device__ inline Item listed_item(const QueryArgs &A, uint32_t e)
{
    if (A.n_slots && (e & kPartFlag)) return part_of(A.split_over[e & ~kPartFlag]);
    return whole_box(e);
}

// Adds the sources of this workgroup's part to its box's sums. Returns true in the workgroup
// that finished the box's last part: its sums are then complete, in its own per-source arrays
// (dense state; the slot is left zero) or in the slot. Every thread must call.
//
// Nothing but atomics touches a slot, and the dense state takes the sums out of it with atomics
// too, so it needs no fence between workgroups, only that a part's additions are done when it is
// counted: every wave waits for its own, then the barrier. (A device-scope fence writes back and
// invalidates caches: 32,000 of 140,000 cycles of a part were spent here with two of them;
// 256 boxes of a 589x563x395 volume: 57 us with them, 40 without; 20,000 anisotropic boxes, 591
// segments: 441 and 351.)
template <int BLOCK, bool SPARSE, bool ERR>
__device__ inline bool merge_part(const QueryArgs &A, QueryShared &sh, const QueryState &st, const Item &it)
{
    const uint64_t at = uint64_t(it.slot) * A.gv.nseg;
    auto add = [&](uint32_t s, uint32_t c, float h, float l) {
        if (c) atomicAdd(&A.slot_cnt[at + s], c);
        if ((__float_as_uint(h) | __float_as_uint(l)) != 0u) add_mass_at(&A.slot_hi[at + s], &A.slot_lo[at + s], h, l);
    };
    if (SPARSE) {
        const uint32_t nu = min(sh.n_used, st.cap);
        for (uint32_t i = threadIdx.x; i < nu; i += BLOCK) {
            const uint32_t slot = ld(&st.used[i]), key = ld(&st.keys[slot]);
            if (key < A.gv.nseg) add(key, ld(&st.cnt[slot]), ld(&st.hi[slot]), ld(&st.lo[slot]));
        }
    } else {
        for (uint32_t s = threadIdx.x; s < A.gv.nseg; s += BLOCK) {
            // (with ERR every part counted the cubes on sources)
            add(s, ERR && it.part ? 0u : ld(&st.seg_cnt[s]), ld(&st.seg_hi[s]), ld(&st.seg_lo[s]));
            if (ERR) {
                const float v = ld(&st.seg_var[s]);
                if (v != 0.0f) atomicAdd(&A.slot_var[at + s], v);
            }
        }
    }
    if (SPARSE) __threadfence();
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    __syncthreads();
    if (threadIdx.x == 0) sh.last = atomicAdd(&A.slot_done[it.slot], 1u) + 1u == it.parts;
    __syncthreads();
    if (!uni(sh.last)) return false;
    if (SPARSE) {
        __threadfence();
        return true;
    }
    for (uint32_t s = threadIdx.x; s < A.gv.nseg; s += BLOCK) {
        st_atomic(&st.seg_cnt[s], atomicExch(&A.slot_cnt[at + s], 0u));
        st_atomic(&st.seg_hi[s], atomicExch(&A.slot_hi[at + s], 0.f));
        st_atomic(&st.seg_lo[s], atomicExch(&A.slot_lo[at + s], 0.f));
        if (ERR) st_atomic(&st.seg_var[s], atomicExch(&A.slot_var[at + s], 0.f));
    }
    if (threadIdx.x == 0) A.slot_done[it.slot] = 0;
    __syncthreads();
    return true;
}

// One query, by the whole block. `st` must be clean (keys empty, values 0).
// ERR: lookup-table expansion that also accumulates uncertainties (dense output).
// tag: OR-ed into the box's stats (which launch answered it). Returns true where the table
// overflowed: nothing was written then, or, with `fail`, the box is marked as failed.
// (always inlined: each query kernel is one function, whatever the inliner's size limit)
// Parts of a box: ranges of its cubes; with ERR, where every node's count has to meet its row
// whole (uncertainties add in quadrature), classes of its nodes, each part reading all cubes.
template <int BLOCK, int GROUP, bool SPARSE, bool ERR>
__device__ __attribute__((always_inline)) inline bool run_query(const QueryArgs &A, QueryShared &sh,
                                                                const QueryState &state, const Item it, bool fail,
                                                                uint32_t tag)
{
    QueryState st = state;
    if (ERR) st.cls = uni(it.part), st.n_cls = uni(it.parts);
    const uint32_t q = uni(it.q);
    uint32_t lo[3], hi[3];
    const bool nonempty = clip_box(A.boxes + 6 * uint64_t(q), A.lt, lo, hi);
    if (threadIdx.x == 0) {
        sh.n_used = 0;
        sh.flags = 0;
        sh.max_key = 0;
        sh.taken[0] = sh.taken[1] = 0;
        sh.n_slabs = 0;
    }
    __syncthreads();
    if (nonempty) build_slabs(A.lt, sh.rows, lo, hi, st.slabs, &sh.n_slabs, st.tile0, st.item0);
    __syncthreads();
    const uint32_t n_slabs = uni(uint32_t(sh.n_slabs));
    if (n_slabs)
        scatter_box<BLOCK, GROUP, SPARSE>(reinterpret_cast<const char *>(A.maps),
                                          reinterpret_cast<const char *>(A.maps16), sh.runs, st, A.gv,
                                          n_slabs, ERR ? 0u : uni(it.part), ERR ? 1u : uni(it.parts), sh.taken, &sh.flags);
    __syncthreads();
    if (ERR || A.lut_ptr)
        expand_rows<BLOCK, SPARSE, ERR>(st, LutRows<ERR>(A.lut_ptr, A.lut_seg, A.lut_val, A.lut_err, A.gv));
    else if (A.counts)
        expand_rows<BLOCK, SPARSE, false>(st, DeepRows(A.gv));
    else
        push_mass<BLOCK, SPARSE>(st, A.gv, sh.rank_ptr, A.depth);
    __syncthreads();
    const bool overflow = (uni(sh.flags) & 1u) != 0;
    if (A.stats && threadIdx.x == 0 && (!overflow || fail)) {
        uint32_t cubes = 0;
        for (int i = 0; i < sh.n_slabs; ++i) cubes += slab_count(st.slabs[i]);
        A.stats[2 * uint64_t(q)] = cubes;
        // bit 30: answered by the retry launch, bit 31: by a global-memory one
        A.stats[2 * uint64_t(q) + 1] = sh.n_used | tag;
    }
    const uint32_t nseg = A.gv.nseg;
    const double vol = nonempty ? double(hi[0] - lo[0]) * double(hi[1] - lo[1]) * double(hi[2] - lo[2]) : 0.0;
    if (overflow) {
        if (fail) write_failure<BLOCK>(A, q);  // even a table for the whole graph overflowed
    } else if (uni(it.parts) == 1) {
        write_result<BLOCK, SPARSE, ERR>(A, sh, st, q, nonempty, vol);
    } else if (merge_part<BLOCK, SPARSE, ERR>(A, sh, st, it)) {
        if (SPARSE) {
            QueryState all = st;  // the box's sums, and zeros for the next call
            const uint64_t at = uint64_t(it.slot) * nseg;
            all.seg_cnt = A.slot_cnt + at, all.seg_hi = A.slot_hi + at, all.seg_lo = A.slot_lo + at;
            write_result<BLOCK, false, false>(A, sh, all, q, nonempty, vol);
            __syncthreads();
            for (uint32_t s = threadIdx.x; s < nseg; s += BLOCK)
                all.seg_cnt[s] = 0, all.seg_hi[s] = 0.f, all.seg_lo[s] = 0.f;
            if (threadIdx.x == 0) A.slot_done[it.slot] = 0;
        } else {
            write_result<BLOCK, false, ERR>(A, sh, st, q, nonempty, vol);
        }
    }
    __syncthreads();
    // restore a clean state for the next query
    const uint32_t nu = min(sh.n_used, st.cap);
    for (uint32_t i = threadIdx.x; i < nu; i += BLOCK) {
        const uint32_t slot = ld(&st.used[i]);
        st.keys[slot] = kEmpty;
        clear_entry<SPARSE>(st, slot);
    }
    if (!SPARSE)
        for (uint32_t s = threadIdx.x; s < nseg; s += BLOCK) {
            st.seg_cnt[s] = 0;
            st.seg_hi[s] = 0.f;
            st.seg_lo[s] = 0.f;
            if (ERR) st.seg_var[s] = 0.f;
        }
    __syncthreads();
    return overflow;
}

// Hands an item whose table overflowed to the retry launch (list 1). Any thread, once. A whole
// box of a planned call is cut into parts there and then (`cubes` of it, while slots last), so
// that the retry launch does not end with one workgroup redoing a large box on its own.
template <bool ERR>
__device__ inline void report_overflow(const QueryArgs &A, const Item &it, uint32_t cubes)
{
    if (it.parts > 1) {
        const uint32_t k = atomicAdd(&A.counters[kCountSplitOver], 1u);
        A.split_over[k] = make_uint4(it.q, it.part, it.parts, it.slot);
        A.overflow[atomicAdd(&A.counters[kCountOver], 1u)] = kPartFlag | k;
        return;
    }
    const uint32_t parts = ERR ? (cubes >> kBigLog2 ? kClassesRedo : 1u) : cubes ? parts_of(cubes, kMinPartRedo) : 1u;
    if (parts > 1 && A.n_slots) {
        // (both counters may pass their limits: then the box stays whole)
        const uint32_t k = atomicAdd(&A.counters[kCountRedo], parts);
        if (k < 2 * A.n_slots && parts <= 2 * A.n_slots - k) {
            const uint32_t slot = atomicAdd(&A.counters[kCountSlot], 1u);
            if (slot < A.n_slots) {
                const uint32_t at = atomicAdd(&A.counters[kCountOver], parts), first = 2 * A.n_slots + k;
                for (uint32_t p = 0; p < parts; ++p) {
                    A.split_over[first + p] = make_uint4(it.q, p, parts, slot);
                    A.overflow[at + p] = kPartFlag | (first + p);
                }
                return;
            }
        }
    }
    A.overflow[atomicAdd(&A.counters[kCountOver], 1u)] = it.q;
}

template <int BLOCK, int GROUP, bool SPARSE, bool ERR>
__device__ __attribute__((always_inline)) inline void answer(const QueryArgs &A, QueryShared &sh,
                                                             const QueryState &st, const Item it, bool planned)
{
    if (run_query<BLOCK, GROUP, SPARSE, ERR>(A, sh, st, it, false, 0u) && threadIdx.x == 0)
        report_overflow<ERR>(A, it, planned || ERR ? box_cubes(A.lt, A.boxes + 6 * uint64_t(it.q)) : 0u);
}

// The graph's tables every query reads, copied to LDS. The loads are issued together and ahead
// of other set-up work; put() stores them.
struct GraphTables {
    static_assert(kMaxSteps + 2 <= 128 && 2 * kMaxLevelsDev <= 128, "one entry per thread of any workgroup");
    uint32_t rank_ptr = 0;
    LevelRow row;
    RunLevel run;

    __device__ explicit GraphTables(const QueryArgs &A)
    {
        const uint32_t i = threadIdx.x;
        if (i < A.depth + 2) rank_ptr = A.rank_ptr[i];
        if (i < 2 * A.lt.n_levels) run = A.runs[i];
        if (i < A.lt.n_levels) row = level_row(A.lt, i);
    }
    __device__ void put(const QueryArgs &A, QueryShared &sh) const
    {
        const uint32_t i = threadIdx.x;
        if (i < A.depth + 2) sh.rank_ptr[i] = rank_ptr;
        if (i < 2 * A.lt.n_levels) sh.runs[i] = run;
        if (i < A.lt.n_levels) sh.rows[i] = row;
    }
};

// The slab list and its prefix arrays at `p` (LDS, lds_slab_bytes).
__device__ inline void place_slabs(QueryState &st, char *p, uint32_t n_levels)
{
    st.slabs = reinterpret_cast<Slab *>(p);
    st.tile0 = reinterpret_cast<uint32_t *>(p + 6u * n_levels * uint32_t(sizeof(Slab)));
    st.item0 = st.tile0 + 6u * n_levels + 1u;
}

template <bool SPARSE>
__device__ inline QueryState lds_state(char *dyn, QueryShared &sh, uint32_t nseg, uint32_t cap, uint32_t n_levels,
                                      bool counts, bool err)
{
    QueryState st;
    char *const slabs = dyn + lds_state_bytes(nseg, cap, SPARSE, counts);
    place_slabs(st, slabs, n_levels);
    st.seg_var = err ? reinterpret_cast<float *>(slabs + lds_slab_bytes(n_levels)) : nullptr;
    st.counts = counts;
    st.cls = 0, st.n_cls = 1;
    uint32_t *t = reinterpret_cast<uint32_t *>(dyn);
    if (SPARSE) {
        st.seg_cnt = nullptr;
        st.seg_hi = st.seg_lo = nullptr;
        st.hi = reinterpret_cast<float *>(t + cap);
        st.lo = reinterpret_cast<float *>(t + 2 * cap);
        st.used = t + 3 * cap;
        st.cnt = t + 4 * cap;
    } else {
        st.seg_cnt = t;
        st.seg_hi = reinterpret_cast<float *>(t + nseg);
        st.seg_lo = reinterpret_cast<float *>(t + 2 * nseg);
        t += 3 * nseg;
        st.used = t + cap;
        st.cnt = t + 2 * cap;                       // with `counts`, else
        st.hi = reinterpret_cast<float *>(t + 2 * cap);
        st.lo = reinterpret_cast<float *>(t + 3 * cap);
    }
    st.keys = t;
    st.cap = cap;
    st.limit = cap / 4 * 3;
    st.n_used = &sh.n_used;
    st.flags = &sh.flags;
    st.max_key = &sh.max_key;
    return st;
}

template <int BLOCK, bool SPARSE, bool ERR>
__device__ inline void clear_lds_state(const QueryState &st, uint32_t nseg)
{
    for (uint32_t i = threadIdx.x; i < st.cap; i += BLOCK) {
        st.keys[i] = kEmpty;
        clear_entry<SPARSE>(st, i);
    }
    if (!SPARSE)
        for (uint32_t s = threadIdx.x; s < nseg; s += BLOCK) {
            st.seg_cnt[s] = 0;
            st.seg_hi[s] = 0.f;
            st.seg_lo[s] = 0.f;
            if (ERR) st.seg_var[s] = 0.f;
        }
}

// Plain: one block per query in input order, state in LDS.
template <bool SPARSE>
__global__ __launch_bounds__(kBlock) void query_plain_kernel(QueryArgs A)
{
    extern __shared__ __align__(16) char dyn[];
    __shared__ QueryShared sh;
    const QueryState st = lds_state<SPARSE>(dyn, sh, A.gv.nseg, A.table_cap, A.lt.n_levels, A.counts != 0, false);
    GraphTables(A).put(A, sh);
    clear_lds_state<kBlock, SPARSE, false>(st, A.gv.nseg);
    __syncthreads();
    answer<kBlock, kGroup, SPARSE, false>(A, sh, st, whole_box(blockIdx.x), false);
}

// Calls of at most kDirectMax boxes, in one launch: every workgroup counts the cubes of all
// boxes (a few per thread, closed form), so each knows the parts of every box without a
// planning launch, and takes items blockIdx, blockIdx + gridDim, ... of the boxes' parts in
// order. A box's part count does not depend on the workgroup, so all agree. The slot of a
// shared box is its rank among the shared ones.
template <int BLOCK, int GROUP, bool SPARSE, bool ERR>
__global__ __launch_bounds__(BLOCK, 6) void query_direct_kernel(QueryArgs A, uint32_t ways, uint32_t least)
{
    extern __shared__ __align__(16) char dyn[];
    __shared__ QueryShared sh;
    __shared__ uint32_t first[kDirectMax + 1];  // items before box q | shared boxes before it << 16
    __shared__ uint64_t wave_sum[BLOCK / 64];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const GraphTables tables(A);
    uint64_t mine = 0;
    for (uint32_t q = threadIdx.x; q < A.n; q += BLOCK) {
        const uint32_t c = box_cubes(A.lt, A.boxes + 6 * q);
        first[q] = c;
        mine += c;
    }
    for (int off = 32; off > 0; off >>= 1) mine += __shfl_down(mine, off, 64);
    if (lane == 0) wave_sum[wave] = mine;
    __syncthreads();
    uint64_t total = 0;
    for (int w = 0; w < BLOCK / 64; ++w) total += wave_sum[w];
    const uint32_t target = part_cubes(total, ways, least);
    __syncthreads();
    // exclusive sums over the boxes, a contiguous stretch per thread
    const uint32_t per = (A.n + BLOCK - 1) / BLOCK, b0 = min(A.n, threadIdx.x * per), b1 = min(A.n, b0 + per);
    uint32_t sum = 0;
    for (uint32_t q = b0; q < b1; ++q) {
        const uint32_t p = parts_of(first[q], target);
        sum += p + (p > 1 ? 1u << 16 : 0u);
    }
    uint32_t incl = sum;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t v = uint32_t(__shfl_up(int(incl), off, 64));
        if (lane >= uint32_t(off)) incl += v;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    uint32_t before = incl - sum;
    for (uint32_t w = 0; w < wave; ++w) before += uint32_t(wave_sum[w]);
    for (uint32_t q = b0; q < b1; ++q) {
        const uint32_t p = parts_of(first[q], target);
        first[q] = before;
        before += p + (p > 1 ? 1u << 16 : 0u);
    }
    if (b1 == A.n && b0 < b1) first[A.n] = before;
    __syncthreads();
    const uint32_t items = uni(first[A.n]) & 0xFFFFu;
    if (blockIdx.x >= items) return;
    const QueryState st = lds_state<SPARSE>(dyn, sh, A.gv.nseg, A.table_cap, A.lt.n_levels, A.counts != 0, ERR);
    tables.put(A, sh);
    clear_lds_state<BLOCK, SPARSE, ERR>(st, A.gv.nseg);
    for (uint32_t i = blockIdx.x; i < items; i += gridDim.x) {
        uint32_t q = 0;  // the last box whose items start at or before i
        for (uint32_t step = kDirectMax / 2; step > 0; step >>= 1)
            if (q + step < A.n && (first[q + step] & 0xFFFFu) <= i) q += step;
        q = uni(q);
        const uint32_t f = uni(first[q]), e = uni(first[q + 1]);
        answer<BLOCK, GROUP, SPARSE, ERR>(A, sh, st,
                                          Item{q, i - (f & 0xFFFFu), (e & 0xFFFFu) - (f & 0xFFFFu), f >> 16}, false);
    }
}

// Batched tiers: persistent blocks take queries from the largest-first order.
// BIG: the parts of shared boxes, then positions [0, counters[kCountBig]); otherwise the
// positions from there to n.
// Six waves per SIMD (the second argument counts them): at most 80 VGPRs, so that
// the memory latency of the streamed node IDs stays hidden.
template <int BLOCK, bool BIG, int GROUP, bool SPARSE, bool ERR>
__global__ __launch_bounds__(BLOCK, 6) void query_tier_kernel(QueryArgs A)
{
    extern __shared__ __align__(16) char dyn[];
    __shared__ QueryShared sh;
    const QueryState st = lds_state<SPARSE>(dyn, sh, A.gv.nseg, A.table_cap, A.lt.n_levels, A.counts != 0, ERR);
    GraphTables(A).put(A, sh);
    clear_lds_state<BLOCK, SPARSE, ERR>(st, A.gv.nseg);
    const uint32_t big = uni(A.counters[kCountBig]), n_split = BIG ? uni(A.counters[kCountSplit]) : 0u;
    const uint32_t begin = BIG ? 0u : big, end = BIG ? n_split + big : A.n;
    // Work queues: a single counter that every workgroup increments serialises
    // at one L2 atomic unit (about 12 ns per box), so the tier's positions of
    // the largest-first order are dealt to kQueues interleaved queues (queue j:
    // positions begin + j, begin + j + kQueues, ...), each with its own counter
    // on its own 256-byte line; workgroup b serves queue b mod kQueues. Each
    // queue is still largest-first. A dequeue takes `chunk` positions (small
    // tier only; 1 by default).
    // (fewer queues when the grid is smaller, so that every queue has a workgroup)
    const uint32_t nq = min(kQueues, gridDim.x);
    const uint32_t qn = blockIdx.x % nq;
    uint32_t *const qc = A.queues + qn * kQueueStride + (BIG ? 0u : 16u);
    const uint32_t chunk = BIG ? 1u : (A.chunk ? A.chunk : 1u);
    for (;;) {
        if (threadIdx.x == 0) sh.q = atomicAdd(qc, chunk);
        __syncthreads();
        const uint32_t i0 = uni(sh.q);
        if (i0 >= end) break;  // uniform; keeps begin + qn + i0 * nq below 2^32
        const uint32_t k0 = begin + qn + i0 * nq;
        if (k0 >= end) break;  // uniform
        // run_query ends with a barrier, so thread 0 rewrites sh.q only after every thread read it
        for (uint32_t i = 0; i < chunk; ++i) {
            const uint32_t k = k0 + i * nq;
            if (k >= end) break;
            Item it;
            if (BIG && k < n_split) {
                it = part_of(A.split[k]);
            } else {
                const uint32_t q = uni(A.order[k - n_split]);
                if (q == kEmpty) {  // its parts are in `split` (uniform)
                    __syncthreads();
                    continue;
                }
                it = whole_box(q);
            }
            answer<BLOCK, GROUP, SPARSE, ERR>(A, sh, st, it, true);
        }
    }
}

// State in worker w's tables of a global pool (slab list in LDS at `slabs`).
__device__ inline QueryState pool_state(const GlobalPool &p, uint32_t w, char *slabs, QueryShared &sh, uint32_t nseg,
                                        uint32_t n_levels, bool counts, bool err)
{
    QueryState st;
    st.counts = counts;
    st.cls = 0, st.n_cls = 1;
    const uint64_t at = uint64_t(w) * p.slots, sat = uint64_t(w) * nseg;
    st.keys = p.keys + at;
    st.cnt = p.cnt + at;
    st.hi = p.hi + at;
    st.lo = p.lo + at;
    st.used = p.used + at;
    st.cap = p.slots;
    st.limit = st.cap / 4 * 3;
    place_slabs(st, slabs, n_levels);
    st.n_used = &sh.n_used;
    st.flags = &sh.flags;
    st.max_key = &sh.max_key;
    st.seg_cnt = p.seg_cnt + sat;
    st.seg_hi = p.seg_hi + sat;
    st.seg_lo = p.seg_lo + sat;
    st.seg_var = err ? p.seg_var + sat : nullptr;
    return st;
}

// The last workgroup of a call's last launch leaves the lists empty for the next call. Every
// workgroup of that launch must call, past its last use of the counters.
__device__ inline void clear_lists(const QueryArgs &A)
{
    if (threadIdx.x != 0) return;
    __threadfence();
    if (atomicAdd(&A.counters[kCountExit], 1u) + 1u != gridDim.x) return;
    A.counters[kCountOver] = A.counters[kCountOver2] = A.counters[kCountOver3] = 0;
    A.counters[kCountRetry] = A.counters[kCountNext2] = A.counters[kCountNext3] = 0;
    A.counters[kCountExit] = A.counters[kCountSplitOver] = A.counters[kCountRedo] = 0;
}

// What overflowed its LDS table (list 1; usually nothing, and then every workgroup leaves at
// once) with the largest LDS table of a workgroup; what overflows again goes to list 2. The
// first workgroup also clears what the launches before this one counted with.
// last: no launch follows (the table holds any box of this graph), so it clears the lists too.
template <int BLOCK, int GROUP, bool SPARSE, bool ERR>
__global__ __launch_bounds__(BLOCK) void query_retry_kernel(QueryArgs A, uint32_t last)
{
    extern __shared__ __align__(16) char dyn[];
    __shared__ QueryShared sh;
    if (blockIdx.x == 0) {
        for (uint32_t i = threadIdx.x; i < kQueues * kQueueStride; i += BLOCK) A.queues[i] = 0;
        if (threadIdx.x < 64) A.buckets[threadIdx.x] = 0;
        if (threadIdx.x == 0) {
            A.counters[kCountBig] = A.counters[kCountSplit] = A.counters[kCountSlot] = 0;
            A.counters[kCountTotal] = A.counters[kCountTotal + 1] = 0;
        }
    }
    const uint32_t n_list = uni(A.counters[kCountOver]);  // final: the launches before this one counted it
    if (n_list == 0) return;
    const QueryState st = lds_state<SPARSE>(dyn, sh, A.gv.nseg, A.table_cap, A.lt.n_levels, A.counts != 0, ERR);
    GraphTables(A).put(A, sh);
    clear_lds_state<BLOCK, SPARSE, ERR>(st, A.gv.nseg);
    for (;;) {
        if (threadIdx.x == 0) sh.q = atomicAdd(&A.counters[kCountRetry], 1u);
        __syncthreads();
        const uint32_t k = uni(sh.q);
        if (k >= n_list) break;
        const uint32_t e = uni(A.overflow[k]);
        if (run_query<BLOCK, GROUP, SPARSE, ERR>(A, sh, st, listed_item(A, e), false, 0x40000000u) &&
            threadIdx.x == 0)
            A.overflow2[atomicAdd(&A.counters[kCountOver2], 1u)] = e;
    }
    if (last) clear_lists(A);
}

// What overflowed every LDS table (list 2), with per-worker tables and source arrays in global
// memory: first by many workers with mid-size tables (what overflows those goes to list 3),
// then by a few workers whose tables hold every node of the graph (list 3, or list 2 where the
// graph is small enough for those tables alone). Sources always have per-worker arrays here
// (dense state, whatever the output): a cube run on a source is one global atomic add without
// a returned value, where a table entry would take a probe round trip. The last workgroup of
// the last of these launches clears the counters of the lists for the next call.
template <bool ERR>
__global__ __launch_bounds__(kBlock) void query_fallback_kernel(QueryArgs A, GlobalPool pool, uint32_t list,
                                                                uint32_t last)
{
    extern __shared__ __align__(16) char dyn[];
    __shared__ QueryShared sh;
    if (uni(A.counters[kCountOver]) == 0) return;  // nothing overflowed at all: the same in every workgroup
    const uint32_t *const entries = list == 2 ? A.overflow2 : A.overflow3;
    const uint32_t n_list = uni(A.counters[list == 2 ? kCountOver2 : kCountOver3]);
    const uint32_t next = list == 2 ? kCountNext2 : kCountNext3;
    if (n_list) {
        const QueryState st = pool_state(pool, blockIdx.x, dyn, sh, A.gv.nseg, A.lt.n_levels, A.counts != 0, ERR);
        GraphTables(A).put(A, sh);
        __syncthreads();
        for (;;) {
            if (threadIdx.x == 0) sh.q = atomicAdd(&A.counters[next], 1u);
            __syncthreads();
            const uint32_t k = uni(sh.q);
            if (k >= n_list) break;
            const uint32_t e = uni(entries[k]);
            if (run_query<kBlock, kGroup, false, ERR>(A, sh, st, listed_item(A, e), last != 0, 0x80000000u) &&
                !last && threadIdx.x == 0)
                A.overflow3[atomicAdd(&A.counters[kCountOver3], 1u)] = e;
        }
    }
    if (last) clear_lists(A);
}

// Per-block histogram of 32 buckets, merged with one global atomic per
// non-empty bucket (instead of one contended atomic per box). Every thread of
// the block must call it.
__device__ inline void block_histogram_add(uint32_t bkt, uint32_t *bucket_count)
{
    __shared__ uint32_t h[32];
    if (threadIdx.x < 32) h[threadIdx.x] = 0;
    __syncthreads();
    if (bkt < 32) atomicAdd(&h[bkt], 1u);
    __syncthreads();
    if (threadIdx.x < 32 && h[threadIdx.x]) atomicAdd(&bucket_count[threadIdx.x], h[threadIdx.x]);
}

// Size bucket of a box, largest first: bucket 0 holds >= 2^31 cubes.
__device__ inline uint32_t size_bucket(uint32_t cubes) { return 31u - (cubes ? 31u - uint32_t(__clz(int(cubes))) : 0u); }

// Planning, first launch: cubes of every box, how many boxes fall into each of 32 log2 size
// buckets, and all boxes' cubes together. `zero` (the sparse output's total, or null) is reset.
__global__ void query_size_kernel(LevelTable lt, const uint32_t *boxes, uint32_t n, uint32_t *work,
                                  uint32_t *bucket_count, uint32_t *counters, uint32_t *zero)
{
    const uint32_t q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q == 0 && zero) *zero = 0;
    const uint32_t cubes = q < n ? box_cubes(lt, boxes + 6 * uint64_t(q)) : 0u;
    if (q < n) work[q] = cubes;
    uint64_t sum = cubes;
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_down(sum, off, 64);
    __shared__ unsigned long long block_sum;
    if (threadIdx.x == 0) block_sum = 0;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) atomicAdd(&block_sum, (unsigned long long)sum);
    block_histogram_add(q < n ? size_bucket(cubes) : 32u, bucket_count);  // every thread, one call site
    if (threadIdx.x == 0) atomicAdd(reinterpret_cast<unsigned long long *>(counters + kCountTotal), block_sum);
}

// Planning, second launch: the largest-first order. bucket_count[b] holds the boxes of bucket
// b and bucket_count[32 + b] counts those placed; each block reserves one range per bucket and
// ranks its boxes inside it. Boxes above their share of the work (part_cubes) are split into
// parts instead, and leave a hole.
__global__ void query_order_kernel(const uint32_t *work, uint32_t n, uint32_t *bucket_count, uint32_t *order,
                                   uint32_t *counters, uint4 *split, uint32_t ways, uint32_t least,
                                   uint32_t big_log2)
{
    __shared__ uint32_t h[32], base[32];
    const uint32_t q = blockIdx.x * blockDim.x + threadIdx.x;
    if (threadIdx.x < 32) h[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t cubes = q < n ? work[q] : 0u, bkt = q < n ? size_bucket(cubes) : 32u;
    const uint32_t local = bkt < 32 ? atomicAdd(&h[bkt], 1u) : 0u;
    __syncthreads();
    if (threadIdx.x < 64) {
        const uint32_t c = threadIdx.x < 32 ? bucket_count[threadIdx.x] : 0u;
        uint32_t incl = c;
        for (int off = 1; off < 32; off <<= 1) {
            const uint32_t v = uint32_t(__shfl_up(int(incl), off, 64));
            if (threadIdx.x >= uint32_t(off)) incl += v;
        }
        if (threadIdx.x < 32 && h[threadIdx.x])
            base[threadIdx.x] = incl - c + atomicAdd(&bucket_count[32 + threadIdx.x], h[threadIdx.x]);
        // boxes of >= 2^big_log2 cubes come first
        if (blockIdx.x == 0 && threadIdx.x == 31 - big_log2) counters[kCountBig] = incl;
    }
    __syncthreads();
    if (bkt >= 32) return;
    const uint32_t target = part_cubes(*reinterpret_cast<const uint64_t *>(counters + kCountTotal), ways, least);
    const uint32_t parts = parts_of(cubes, target);
    order[base[bkt] + local] = parts > 1 ? kEmpty : q;
    if (parts > 1) {
        const uint32_t slot = atomicAdd(&counters[kCountSlot], 1u), k = atomicAdd(&counters[kCountSplit], parts);
        for (uint32_t p = 0; p < parts; ++p) split[k + p] = make_uint4(q, p, parts, slot);
    }
}

// ---------------------------------------------------------------- naive scan

struct NaiveArgs {
    LevelTable lt;
    const uint32_t *boxes;
    float *out;
    const uint32_t *map0;
    const uint16_t *map16;        // 16-bit level 0 (x-fastest, row pitch lt.pitch_x), if lt.use16
    uint32_t nseg;
    uint32_t n;
};

// Naive range query: every level-0 voxel of the box is read and counted
// (same wave-level run merging and unconditional loads as the graph path).
template <int UNROLL>
__global__ __launch_bounds__(kBlock) void naive_kernel(NaiveArgs A)
{
    extern __shared__ __align__(16) char dyn[];
    uint32_t *cnt = reinterpret_cast<uint32_t *>(dyn);
    const uint32_t q = blockIdx.x;
    for (uint32_t s = threadIdx.x; s < A.nseg; s += kBlock) cnt[s] = 0;
    uint32_t lo[3], hi[3];
    const bool nonempty = clip_box(A.boxes + 6 * uint64_t(q), A.lt, lo, hi);
    __syncthreads();
    if (nonempty) {
        uint64_t base;
        uint32_t odd;
        const TileWalk tw = naive_walk(A.lt, lo, hi, A.lt.use16 != 0, UNROLL, &base, &odd);
        const uint32_t lane = threadIdx.x & 63;
        if (A.lt.use16) {
            stream_pairs<UNROLL, kBlock / 64>(reinterpret_cast<const char *>(A.map16) + base, tw, hi[0] - lo[0], odd,
                                              [&](uint32_t a, uint32_t b) { count_pairs(cnt, a, b, lane); });
        } else {
            // runs of equal IDs: -start lane at the start, end lane + 1 at the end (as in stream_tiles)
            const uint32_t w_start = 0u - lane, w_end = lane + 1;
            stream_slab<UNROLL, kBlock / 64>(
                reinterpret_cast<const char *>(A.map0) + base, tw, [&](uint32_t v) {
                    const uint32_t prev = uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x138, 0xF, 0xF, true));
                    const uint32_t next = uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x130, 0xF, 0xF, true));
                    if (v != kEmpty) {
                        if (v != prev || lane == 0) atomicAdd(&cnt[v], w_start);
                        if (v != next || lane == 63) atomicAdd(&cnt[v], w_end);
                    }
                });
        }
    }
    __syncthreads();
    const double vol = nonempty ? double(hi[0] - lo[0]) * double(hi[1] - lo[1]) * double(hi[2] - lo[2]) : 0.0;
    float *o = A.out + uint64_t(q) * A.nseg;
    for (uint32_t s = threadIdx.x; s < A.nseg; s += kBlock) o[s] = nonempty ? float(double(cnt[s]) / vol) : 0.0f;
}

// ---------------------------------------------------------------- footprint (test view)

__global__ __launch_bounds__(kBlock) void footprint_kernel(LevelTable lt, const uint32_t *boxes, uint32_t n,
                                                           const uint32_t *maps, uint32_t *level_counts,
                                                           uint32_t *cubes, uint32_t cap, uint32_t *count)
{
    __shared__ Slab slabs[kMaxSlabs];
    __shared__ int n_slabs;
    __shared__ uint32_t per_level[MG_MAX_LEVELS];
    __shared__ LevelRow rows[kMaxLevelsDev];
    const uint32_t q = blockIdx.x;
    if (threadIdx.x == 0) n_slabs = 0;
    if (threadIdx.x < lt.n_levels) rows[threadIdx.x] = level_row(lt, threadIdx.x);
    if (threadIdx.x < MG_MAX_LEVELS) per_level[threadIdx.x] = 0;
    uint32_t lo[3], hi[3];
    const bool nonempty = clip_box(boxes + 6 * uint64_t(q), lt, lo, hi);
    __syncthreads();
    if (nonempty) build_slabs(lt, rows, lo, hi, slabs, &n_slabs, nullptr, nullptr);
    __syncthreads();
    for (int si = 0; si < n_slabs; ++si) {
        const Slab sl = slabs[si];
        if (threadIdx.x == 0) atomicAdd(&per_level[sl.level], slab_count(sl));
        if (!cubes) continue;
        for (uint32_t r = threadIdx.x; r < slab_count(sl); r += kBlock) {
            const uint32_t i0 = r % sl.e0, i1 = (r / sl.e0) % sl.e1, i2 = r / (sl.e0 * sl.e1);
            uint32_t x, y, z;
            slab_coords(sl, i0, i1, i2, &x, &y, &z);
            // kind-0 slab (the table is built without the 16-bit copy): 4-byte units
            const uint32_t node = maps[sl.base / 4 + i0 + uint64_t(i1) * (sl.s1b / 4) + uint64_t(i2) * (sl.s2b / 4)];
            const uint32_t k = atomicAdd(count, 1u);
            if (k < cap) {
                uint32_t *c = cubes + 6 * uint64_t(k);
                c[0] = q, c[1] = sl.level, c[2] = x, c[3] = y, c[4] = z, c[5] = node;
            }
        }
    }
    __syncthreads();
    for (uint32_t l = threadIdx.x; l < lt.n_levels; l += kBlock) level_counts[uint64_t(q) * lt.n_levels + l] = per_level[l];
}

// ---------------------------------------------------------------- sparse-output sizing

// Upper bound on the non-zero segments of each box (sizes the sparse output).
// The clipped box lies inside the cells it touches at any level; at the finest
// level where it touches at most 64 cells, one lane per cell reads the cell's
// node, and the bound is the sum of mixlen over the distinct nodes, capped by
// the source count and the box volume. That needs every finer cube's mixture
// to lie inside its enclosing cell's, which holds for exact weights; graphs
// with quantized (merged) weights get the source count and volume cap only.
// One wave per box.
__global__ __launch_bounds__(kBlock) void nnz_bound_kernel(LevelTable lt, const uint32_t *boxes, uint32_t n,
                                                           const uint32_t *__restrict__ maps,
                                                           const uint32_t *__restrict__ mixlen, uint32_t nseg,
                                                           uint32_t exact, uint32_t *bound)
{
    const uint32_t q = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63;
    if (q >= n) return;  // whole waves leave together
    uint32_t lo[3], hi[3];
    if (!clip_box(boxes + 6 * uint64_t(q), lt, lo, hi)) {
        if (lane == 0) bound[q] = 0;
        return;
    }
    // cells touched at level `lane` (levels past the last count as too many)
    uint64_t cells = ~uint64_t(0);
    if (lane < lt.n_levels) {
        cells = 1;
        for (int d = 0; d < 3; ++d) cells *= uint64_t(((hi[d] - 1) >> lane) - (lo[d] >> lane) + 1);
    }
    const uint64_t fits = __ballot(cells <= 64);  // the top level (one cell) always fits
    const uint32_t l = uint32_t(__builtin_ctzll(fits));
    uint32_t c0[3], ext[3];
    for (int d = 0; d < 3; ++d) {
        c0[d] = lo[d] >> l;
        ext[d] = ((hi[d] - 1) >> l) - c0[d] + 1;
    }
    const uint32_t ncell = ext[0] * ext[1] * ext[2];
    uint32_t node = kEmpty, m = 0;
    if (lane < ncell) {
        const uint32_t x = c0[0] + lane % ext[0], y = c0[1] + (lane / ext[0]) % ext[1],
                       z = c0[2] + lane / (ext[0] * ext[1]);
        node = maps[lt.off[l] + x + uint64_t(lt.dims[l][0]) * (y + uint64_t(lt.dims[l][1]) * z)];
        m = mixlen[node];
    }
    // count each distinct node once: drop a lane whose node a lower lane holds
    bool dup = false;
    for (uint32_t j = 0; j < ncell; ++j) {
        const uint32_t v = uint32_t(__shfl(int(node), int(j), 64));
        dup = dup || (j < lane && v == node);
    }
    uint32_t sum = dup ? 0u : m;
    for (int off = 32; off > 0; off >>= 1) sum += uint32_t(__shfl_down(int(sum), off, 64));
    if (lane == 0) {
        const uint64_t vol = uint64_t(hi[0] - lo[0]) * (hi[1] - lo[1]) * (hi[2] - lo[2]);
        bound[q] = uint32_t(std::min<uint64_t>(std::min<uint64_t>(exact ? sum : nseg, nseg), vol));
    }
}

// ---------------------------------------------------------------- TF propagation

// A source's colour under transfer function t: its RGBA8 entry scaled to [0, 1],
// each channel one rounded product (never contracted into a later subtraction, so
// a step that reads it here computes exactly what it computes from the stored value).
__device__ inline float4 tf_source_colour(const uchar4 *tf, uint32_t nseg, uint32_t t, uint32_t src)
{
#pragma clang fp contract(off)
    const uchar4 c = tf[uint64_t(t) * nseg + src];
    const float k = 1.0f / 255.0f;
    return make_float4(float(c.x) * k, float(c.y) * k, float(c.z) * k, float(c.w) * k);
}

// A node's colour from its predecessors' colours va, vb and its weight w: one
// fma per channel, v_a + w (v_b - v_a) (every thread that computes a node's
// colour evaluates exactly this, so a value rebuilt elsewhere is bit-identical).
__device__ inline float4 tf_lerp(float w, float4 va, float4 vb)
{
#pragma clang fp contract(off)
    float4 r;
    r.x = fmaf(w, vb.x - va.x, va.x);
    r.y = fmaf(w, vb.y - va.y, va.y);
    r.z = fmaf(w, vb.z - va.z, va.z);
    r.w = fmaf(w, vb.w - va.w, va.w);
    return r;
}

// The entry of position i of a propagation order: with RANKS the nodes in ID
// order (IDs are sorted by rank, so a rank is a contiguous ID range and node i's
// triple is nodes[i]); else the deferred step schedule's entry sched[i].
template <bool RANKS>
__device__ inline SchedNode tf_entry(const NodeTriple *__restrict__ nodes, const SchedNode *__restrict__ sched,
                                     uint32_t i)
{
    if (RANKS) {
        const NodeTriple t = nodes[i];
        return SchedNode{t.a, t.b, t.w, i};
    }
    return sched[i];
}

// One step of the order (a rank, or a step of the deferred schedule): thread
// (x, y) computes the node at position lo_i + x for the transfer functions
// P y .. P y + P - 1 (grid.y = ceil(T / P)): it loads the node's entry and both
// predecessors' colours in all P planes before it stores any, so 2 P gathers
// per thread are in flight together. Lanes of a wave take consecutive entries
// (coalesced entry reads and, nodes being numbered by rank, contiguous stores).
// FIRST: the first launch: the nodes of the first step (every predecessor a
// source) and, in rank order, those of rank 2 too (every predecessor a source or
// a rank-1 node). It reads source colours from the transfer functions
// themselves and rebuilds a rank-1 predecessor's colour from that node's own two
// sources by the same expression the rank-1 node's thread evaluates (so bit for
// bit the value that thread stores), instead of waiting for it in a launch of
// its own; threads x >= hi_i - lo_i write the sources' own colours (the same
// values), so the frame needs no separate source pass.
template <int P, bool FIRST, bool RANKS>
__global__ void tf_step_kernel(const NodeTriple *__restrict__ nodes, const SchedNode *__restrict__ sched,
                               uint32_t lo_i, uint32_t hi_i, uint32_t n_nodes, uint32_t T,
                               const uchar4 *__restrict__ tf, uint32_t nseg, float4 *out)
{
#pragma clang fp contract(off)
    const uint32_t x = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t p0 = blockIdx.y * P;
    const uint32_t n_step = hi_i - lo_i;
    if (x >= n_step) {
        if (!FIRST || x - n_step >= nseg) return;
        const uint32_t src = x - n_step;
#pragma unroll
        for (int p = 0; p < P; ++p)
            if (P == 1 || p0 + p < T) out[uint64_t(p0 + p) * n_nodes + src] = tf_source_colour(tf, nseg, p0 + p, src);
        return;
    }
    const SchedNode t = tf_entry<RANKS>(nodes, sched, lo_i + x);
    NodeTriple ta{0u, 0u, 0.0f}, tb{0u, 0u, 0.0f};  // a rank-1 predecessor's own triple
    if (FIRST) {
        if (t.a >= nseg) ta = nodes[t.a];
        if (t.b >= nseg) tb = nodes[t.b];
    }
    float4 va[P], vb[P];
#pragma unroll
    for (int p = 0; p < P; ++p)
        if (P == 1 || p0 + p < T) {
            if (FIRST) {
                va[p] = t.a < nseg ? tf_source_colour(tf, nseg, p0 + p, t.a)
                                   : tf_lerp(ta.w, tf_source_colour(tf, nseg, p0 + p, ta.a),
                                             tf_source_colour(tf, nseg, p0 + p, ta.b));
                vb[p] = t.b < nseg ? tf_source_colour(tf, nseg, p0 + p, t.b)
                                   : tf_lerp(tb.w, tf_source_colour(tf, nseg, p0 + p, tb.a),
                                             tf_source_colour(tf, nseg, p0 + p, tb.b));
            } else {
                const float4 *o = out + uint64_t(p0 + p) * n_nodes;
                va[p] = o[t.a];
                vb[p] = o[t.b];
            }
        }
#pragma unroll
    for (int p = 0; p < P; ++p)
        if (P == 1 || p0 + p < T) out[uint64_t(p0 + p) * n_nodes + t.id] = tf_lerp(t.w, va[p], vb[p]);
}

// The last steps of the schedule when each is small (at most kTfTailPairs node x
// transfer-function pairs): one workgroup runs them in order, a block barrier
// between steps (all its waves share one CU and its L1, so the stores of a step
// are visible to the loads of the next), instead of one launch per step.
struct TfTail {
    uint32_t n_steps;
    uint32_t lo[kTfTailSteps + 1];  // step k: schedule entries lo[k] .. lo[k + 1]
};

template <bool RANKS>
__global__ __launch_bounds__(kTfTailBlock) void tf_tail_kernel(const NodeTriple *__restrict__ nodes,
                                                               const SchedNode *__restrict__ sched, TfTail tail,
                                                               uint32_t n_nodes, uint32_t T, float4 *out)
{
    for (uint32_t k = 0; k < tail.n_steps; ++k) {
        const uint32_t lo = tail.lo[k], n = tail.lo[k + 1] - lo;
        for (uint32_t j = threadIdx.x; j < n * T; j += kTfTailBlock) {  // plane-major: lanes take consecutive nodes
            const uint32_t t = j / n;
            const SchedNode e = tf_entry<RANKS>(nodes, sched, lo + j % n);
            float4 *o = out + uint64_t(t) * n_nodes;
            o[e.id] = tf_lerp(e.w, o[e.a], o[e.b]);
        }
        __syncthreads();
    }
}

// Mean colour of a box under one propagated palette: every footprint cube adds
// its 8^l voxels times the palette entry of its node, divided by the box
// volume. One workgroup of kColourBlock threads per box; sums in fp64. Boxes
// whose palette index is kEmpty get zeros. The level table carries no 16-bit
// copy and no row runs, so every slab is read as 32-bit node IDs. A thread
// walks its cubes of a slab kColourBlock apart, its (fast, mid, slow) offsets
// advanced by carries rather than divided out, kColourUnroll node IDs and then
// their palette entries in flight at a time.
constexpr int kColourBlock = 1024;
constexpr int kColourUnroll = 8;
__global__ __launch_bounds__(kColourBlock) void box_colour_kernel(LevelTable lt, const uint32_t *boxes, uint32_t n,
                                                                  const uint32_t *__restrict__ maps,
                                                                  const float4 *__restrict__ palette, uint32_t T,
                                                                  uint32_t n_nodes, const uint32_t *pal_of_box,
                                                                  float4 *out)
{
    __shared__ Slab slabs[kMaxSlabs];
    __shared__ int n_slabs;
    __shared__ double part[kColourBlock / 64][4];
    __shared__ LevelRow rows[kMaxLevelsDev];
    if (threadIdx.x < lt.n_levels) rows[threadIdx.x] = level_row(lt, threadIdx.x);
    const uint32_t q = blockIdx.x;
    const uint32_t t = pal_of_box[q];
    uint32_t lo[3], hi[3];
    const bool nonempty = clip_box(boxes + 6 * uint64_t(q), lt, lo, hi) && t < T;
    if (threadIdx.x == 0) n_slabs = 0;
    __syncthreads();
    if (nonempty) build_slabs(lt, rows, lo, hi, slabs, &n_slabs, nullptr, nullptr);
    __syncthreads();
    const float4 *pal = palette + uint64_t(t < T ? t : 0) * n_nodes;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int si = 0; si < n_slabs; ++si) {
        const Slab sl = slabs[si];
        const double w = double(uint64_t(1) << (3 * sl.level));
        const uint32_t c = slab_count(sl);
        if (threadIdx.x >= c) continue;
        // this thread's first cube, and the step of kColourBlock cubes, as (fast, mid, slow) offsets
        const uint32_t e01 = sl.e0 * sl.e1;
        uint32_t i0 = threadIdx.x % sl.e0, i1 = (threadIdx.x / sl.e0) % sl.e1, i2 = threadIdx.x / e01;
        const uint32_t d0 = uint32_t(kColourBlock) % sl.e0, d1 = (uint32_t(kColourBlock) / sl.e0) % sl.e1,
                       d2 = uint32_t(kColourBlock) / e01;
        const uint32_t *slab = maps + sl.base / 4;
        const uint64_t s1 = sl.s1b / 4, s2 = sl.s2b / 4;
        for (uint32_t r = threadIdx.x; r < c; r += kColourBlock * kColourUnroll) {
            uint32_t node[kColourUnroll];
#pragma unroll
            for (int u = 0; u < kColourUnroll; ++u) {
                // cube r + u kColourBlock, if inside the slab
                node[u] = r + uint32_t(u) * kColourBlock < c ? slab[i0 + i1 * s1 + i2 * s2] : kEmpty;
                i0 += d0;
                const uint32_t c0 = i0 >= sl.e0 ? 1u : 0u;
                i0 -= c0 ? sl.e0 : 0u;
                i1 += d1 + c0;
                const uint32_t c1 = i1 >= sl.e1 ? 1u : 0u;
                i1 -= c1 ? sl.e1 : 0u;
                i2 += d2 + c1;
            }
            float4 v[kColourUnroll];
#pragma unroll
            for (int u = 0; u < kColourUnroll; ++u)
                v[u] = node[u] != kEmpty ? pal[node[u]] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int u = 0; u < kColourUnroll; ++u)
                acc[0] += w * v[u].x, acc[1] += w * v[u].y, acc[2] += w * v[u].z, acc[3] += w * v[u].w;
        }
    }
    for (int k = 0; k < 4; ++k)
        for (int off = 32; off > 0; off >>= 1) acc[k] += __shfl_down(acc[k], off, 64);
    if ((threadIdx.x & 63) == 0)
        for (int k = 0; k < 4; ++k) part[threadIdx.x >> 6][k] = acc[k];
    __syncthreads();
    if (threadIdx.x == 0) {
        double s[4] = {0.0, 0.0, 0.0, 0.0};
        for (int wv = 0; wv < kColourBlock / 64; ++wv)
            for (int k = 0; k < 4; ++k) s[k] += part[wv][k];
        const double vol = nonempty ? double(hi[0] - lo[0]) * double(hi[1] - lo[1]) * double(hi[2] - lo[2]) : 1.0;
        out[q] = nonempty ? make_float4(float(s[0] / vol), float(s[1] / vol), float(s[2] / vol), float(s[3] / vol))
                          : make_float4(0.f, 0.f, 0.f, 0.f);
    }
}

// ---------------------------------------------------------------- upload helpers

// Palette fetch: the node of each voxel at one level indexes the palette.
__global__ void palette_fetch_kernel(const float4 *__restrict__ palette, uint32_t T, uint32_t n_nodes,
                                     const uint32_t *__restrict__ map, uint32_t X, uint32_t Y, uint32_t Z,
                                     const uint32_t *__restrict__ xyz, uint32_t n, float4 *__restrict__ out)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t x = xyz[3 * uint64_t(i)], y = xyz[3 * uint64_t(i) + 1], z = xyz[3 * uint64_t(i) + 2];
    const bool in = x < X && y < Y && z < Z;
    const uint32_t node = in ? map[x + uint64_t(X) * (y + uint64_t(Y) * z)] : 0u;
    for (uint32_t t = 0; t < T; ++t)
        out[uint64_t(t) * n + i] = in ? palette[uint64_t(t) * n_nodes + node] : make_float4(0.f, 0.f, 0.f, 0.f);
}

// The voxel data (A) of a graph stream (Table "bitstream"): per level, voxel by
// voxel (x fastest), the node ID minus i_min(l) in r(l) bits, least significant
// bit first. One thread per voxel: the field is read from the two 32-bit words
// that hold it; level-0 IDs are sources, the others are renumbered by `perm`.
// An ID out of range sets *bad and writes node 0.
struct StreamLevels {
    uint32_t n_levels;
    uint32_t nseg, n_nodes;
    uint64_t off[MG_MAX_LEVELS + 1];     // first voxel of each level
    uint64_t bit[MG_MAX_LEVELS];         // bit of its first field, from the first word
    uint32_t r[MG_MAX_LEVELS], lo[MG_MAX_LEVELS];
};

__global__ void unpack_maps_kernel(StreamLevels sl, const uint32_t *__restrict__ words,
                                   const uint32_t *__restrict__ perm, uint32_t *__restrict__ maps, uint32_t *bad)
{
    const uint64_t total = sl.off[sl.n_levels];
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < total; i += stride) {
        uint32_t l = 0;
        while (i >= sl.off[l + 1]) ++l;
        const uint32_t r = sl.r[l];
        const uint64_t b = sl.bit[l] + (i - sl.off[l]) * r;
        const uint64_t w = b >> 5;
        const uint64_t two = (uint64_t(words[w + 1]) << 32) | words[w];
        const uint64_t field = r ? (two >> (b & 31)) & ((uint64_t(1) << r) - 1) : 0;
        const uint64_t id = sl.lo[l] + field;
        const uint64_t limit = l == 0 ? sl.nseg : sl.n_nodes;
        uint32_t node = 0;
        if (id < limit) node = l == 0 ? uint32_t(id) : perm[id];
        else atomicOr(bad, 1u);
        maps[i] = node;
    }
}

// 16-bit copies of level 0: x-fastest with row pitch px, and y-fastest (y + py (z + Z x))
// with row pitch py; padding elements hold 0xFFFF.
__global__ void pack16_kernel(const uint32_t *__restrict__ map0, uint16_t *__restrict__ out, uint32_t X, uint32_t Y,
                              uint32_t Z, uint32_t px, uint32_t py, uint64_t total16, uint64_t total16t)
{
    const uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < total16) {  // x-fastest copy: element i = x + px (y + Y z)
        const uint32_t x = uint32_t(i % px);
        const uint64_t yz = i / px;
        out[i] = x < X ? uint16_t(map0[x + uint64_t(X) * yz]) : uint16_t(0xFFFF);
    }
    if (i < total16t) {  // y-fastest copy: element i = y + py (z + Z x)
        const uint32_t y = uint32_t(i % py);
        const uint64_t zx = i / py;
        const uint32_t z = uint32_t(zx % Z), x = uint32_t(zx / Z);
        out[total16 + i] = y < Y ? uint16_t(map0[x + uint64_t(X) * (y + uint64_t(Y) * z)]) : uint16_t(0xFFFF);
    }
}

__global__ void transpose_level_kernel(const uint32_t *src, uint32_t *dst, uint32_t X, uint32_t Y, uint32_t Z)
{
    // dst[y + Y (z + Z x)] = src[x + X (y + Y z)]
    const uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const uint64_t total = uint64_t(X) * Y * Z;
    if (i >= total) return;
    const uint32_t x = uint32_t(i % X);
    const uint64_t yz = i / X;
    const uint32_t y = uint32_t(yz % Y), z = uint32_t(yz / Y);
    dst[y + uint64_t(Y) * (z + uint64_t(Z) * x)] = src[i];
}

// The records of the nodes of rank 1 and 2 from their triples.
__global__ void leaf_kernel(const NodeTriple *__restrict__ nodes, uint32_t nseg, uint32_t n, Leaf *__restrict__ out)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const NodeTriple t = nodes[nseg + i];
    Leaf r;
    r.s[0] = r.s[1] = t.a;
    r.s[2] = r.s[3] = t.b;
    r.w = t.w, r.wa = r.wb = 0.0f, r.pad = 0;
    if (t.a >= nseg) {
        const NodeTriple u = nodes[t.a];
        r.s[0] = u.a, r.s[1] = u.b, r.wa = u.w;
    }
    if (t.b >= nseg) {
        const NodeTriple u = nodes[t.b];
        r.s[2] = u.a, r.s[3] = u.b, r.wb = u.w;
    }
    out[i] = r;
}

__global__ void fill_u32_kernel(uint32_t *p, uint64_t n, uint32_t v)
{
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

// Arrays of a workspace with the word each holds when clean.
constexpr uint32_t kMaxRanges = 24;
struct ClearRanges {
    uint32_t n;
    struct {
        uint32_t *p;
        uint64_t words;
        uint32_t value;
    } r[kMaxRanges];
};

// (sources, table slots, workers, shared boxes + 1) that the library's scratch is carved for
struct ScratchLayout {
    uint64_t v[4];
};

// Clears a workspace; with `have`, only where the layout it was last cleared for is not `want`
// (the same words for every workgroup: they are written by a launch of their own).
__global__ void clear_kernel(ClearRanges c, const uint64_t *have, ScratchLayout want)
{
    if (have) {
        bool same = true;
        for (int k = 0; k < 4; ++k) same = same && have[k] == want.v[k];
        if (same) return;
    }
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x, first = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    for (uint32_t k = 0; k < c.n; ++k)
        for (uint64_t i = first; i < c.r[k].words; i += stride) c.r[k].p[i] = c.r[k].value;
}

__global__ void stamp_kernel(uint64_t *have, ScratchLayout want)
{
    if (threadIdx.x < 4) have[threadIdx.x] = want.v[threadIdx.x];
}

// Levels, offsets and the 16-bit copy's pitches of a volume (the graph's own
// level table for its dims; the host-side address check builds one from dims).
LevelTable level_table_dims(const uint32_t dims[3])
{
    LevelTable lt;
    std::memset(&lt, 0, sizeof(lt));
    std::vector<uint32_t> ld;
    level_dims(dims, &ld);
    lt.n_levels = uint32_t(ld.size() / 3);
    for (int a = 0; a < 3; ++a) lt.vol[a] = dims[a];
    uint64_t off = 0;
    for (uint32_t l = 0; l < lt.n_levels && l < MG_MAX_LEVELS; ++l) {
        for (int a = 0; a < 3; ++a) lt.dims[l][a] = ld[3 * l + a];
        lt.off[l] = off;
        off += uint64_t(ld[3 * l]) * ld[3 * l + 1] * ld[3 * l + 2];
    }
    lt.total = off;
    lt.pitch_x = dims[0] + (dims[0] & 1u);
    lt.pitch_y = dims[1] + (dims[1] & 1u);
    lt.total16 = uint64_t(lt.pitch_x) * dims[1] * dims[2];
    lt.use16 = 0;  // set per launch where the 16-bit copy is used
    lt.runs_mask = 0, lt.run_min = 0xFFFFFFFFu;  // and where row runs are read
    return lt;
}

LevelTable level_table(const Graph &g) { return level_table_dims(g.dims); }

// ---------------------------------------------------------------- workspace layout

struct Workspace {
    uint32_t *counters;   // 64 u32
    uint32_t *queues;     // kQueues * kQueueStride u32: per-queue counters of the two tiers
    uint32_t *buckets;    // 64 u32
    uint32_t *work;       // [max_boxes] cubes of each box
    uint32_t *order;      // [max_boxes]
    uint32_t *overflow;   // [max_boxes + 4 n_slots] list 1: boxes and parts whose LDS table overflowed
    uint32_t *overflow2;  // [max_boxes + 4 n_slots] list 2: overflowed the retry table too
    uint32_t *overflow3;  // [max_boxes + 4 n_slots] list 3: overflowed a mid-size global table too
    uint32_t n_slots;     // boxes that several workgroups may share
    uint4 *split, *split_over;      // [2 n_slots], [4 n_slots]
    uint32_t *slot_done, *slot_cnt; // [n_slots], [n_slots][S]
    float *slot_hi, *slot_lo;       // [n_slots][S]
    float *slot_var;                // [n_slots][S]
    GlobalPool fin;       // tables that hold every node of the graph
    GlobalPool mid;       // many workers with mid-size tables (workers 0: none)
    uint64_t bytes;
    uint32_t max_boxes;
};

inline uint64_t align256(uint64_t v) { return (v + 255) & ~uint64_t(255); }

// Global fallback tables: each worker's table holds every node of the graph below
// its 3/4 load limit (a box touches a node at most once), so no box can overflow
// it, with at least 2^16 and at most 2^26 slots; the workers share a budget of
// 128 x 2^16 slots (fewer workers for larger graphs, at least 16).
inline uint32_t fallback_slots(const Graph &g)
{
    const uint64_t need = uint64_t(g.n_nodes) * 4 / 3 + 2;
    uint64_t cap = kHashGlobal;
    while (cap < need && cap < (uint64_t(1) << 26)) cap <<= 1;
    return uint32_t(cap);
}
inline uint32_t fallback_workers(const Graph &g)
{
    return std::max<uint32_t>(16u, uint32_t(uint64_t(kFallbackWorkers) * kHashGlobal / fallback_slots(g)));
}
// Mid-size global tables: kMidWorkers workers of kHashGlobal slots each, for
// boxes that overflow every LDS table but touch fewer than 3/4 x kHashGlobal
// nodes (the largest boxes of the 15,917-capsule volume touch ~30,000). Only
// where the final tables are larger than that.
inline uint32_t mid_workers(const Graph &g) { return fallback_slots(g) > kHashGlobal ? kMidWorkers : 0u; }

// Boxes that several workgroups may share in one call (each takes 16 bytes per source). None on
// graphs whose boxes can overflow even the final tables.
inline uint32_t split_slots(const Graph &g)
{
    if (uint64_t(g.n_nodes) * 4 / 3 + 2 > (uint64_t(1) << 26)) return 0;
    return uint32_t(std::min<uint64_t>(kMaxSlots, std::max<uint64_t>(kMinSlots, kSlotBytes / (16ull * g.nseg))));
}

// Carves the workspace for `fin_workers` workers of the final tables (0:
// fallback_workers(g)), `mid_workers` of the mid-size ones (~0u: mid_workers(g)) and n_slots
// shared boxes (~0u: split_slots(g)); with base == nullptr only computes the size.
Workspace carve(const Graph &g, char *base, uint32_t max_boxes, uint32_t fin_workers = 0,
                uint32_t n_mid = ~0u, uint32_t n_slots = ~0u)
{
    Workspace w;
    uint64_t off = 0;
    auto take = [&](uint64_t bytes) {
        char *p = base ? base + off : nullptr;
        off += align256(bytes);
        return p;
    };
    auto pool = [&](GlobalPool &p, uint32_t workers, uint32_t slots) {
        p.workers = workers, p.slots = slots;
        const uint64_t hs = uint64_t(workers) * slots;
        p.keys = reinterpret_cast<uint32_t *>(take(hs * 4));
        p.cnt = reinterpret_cast<uint32_t *>(take(hs * 4));
        p.used = reinterpret_cast<uint32_t *>(take(hs * 4));
        p.hi = reinterpret_cast<float *>(take(hs * 4));
        p.lo = reinterpret_cast<float *>(take(hs * 4));
        const uint64_t ss = uint64_t(workers) * g.nseg;
        p.seg_cnt = reinterpret_cast<uint32_t *>(take(ss * 4));
        p.seg_hi = reinterpret_cast<float *>(take(ss * 4));
        p.seg_lo = reinterpret_cast<float *>(take(ss * 4));
        p.seg_var = reinterpret_cast<float *>(take(ss * 4));
    };
    // fixed-size part first, so that its layout does not depend on max_boxes
    w.counters = reinterpret_cast<uint32_t *>(take(64 * 4));
    w.buckets = reinterpret_cast<uint32_t *>(take(64 * 4));
    w.queues = reinterpret_cast<uint32_t *>(take(uint64_t(kQueues) * kQueueStride * 4));
    pool(w.fin, fin_workers ? fin_workers : fallback_workers(g), fallback_slots(g));
    pool(w.mid, n_mid == ~0u ? mid_workers(g) : n_mid, kHashGlobal);
    w.n_slots = n_slots == ~0u ? split_slots(g) : n_slots;
    const uint64_t ns = w.n_slots;
    w.slot_done = reinterpret_cast<uint32_t *>(take(ns * 4));
    w.slot_cnt = reinterpret_cast<uint32_t *>(take(ns * g.nseg * 4));
    w.slot_hi = reinterpret_cast<float *>(take(ns * g.nseg * 4));
    w.slot_lo = reinterpret_cast<float *>(take(ns * g.nseg * 4));
    w.slot_var = reinterpret_cast<float *>(take(ns * g.nseg * 4));
    w.split = reinterpret_cast<uint4 *>(take(2 * ns * sizeof(uint4)));
    w.split_over = reinterpret_cast<uint4 *>(take(4 * ns * sizeof(uint4)));
    w.work = reinterpret_cast<uint32_t *>(take(uint64_t(max_boxes) * 4));
    w.order = reinterpret_cast<uint32_t *>(take(uint64_t(max_boxes) * 4));
    w.overflow = reinterpret_cast<uint32_t *>(take((uint64_t(max_boxes) + 4 * ns) * 4));
    w.overflow2 = reinterpret_cast<uint32_t *>(take((uint64_t(max_boxes) + 4 * ns) * 4));
    w.overflow3 = reinterpret_cast<uint32_t *>(take((uint64_t(max_boxes) + 4 * ns) * 4));
    w.bytes = off;
    w.max_boxes = max_boxes;
    return w;
}

int check_device(Graph *g, std::string *err)
{
    if (g->dev.device < 0) {
        *err = "graph is not on a device: call mg_upload first";
        return MG_ESTATE;
    }
    int cur = -1;
    HIP_TRY(hipGetDevice(&cur));
    if (cur != g->dev.device) HIP_TRY(hipSetDevice(g->dev.device));
    return MG_OK;
}

struct DeviceGuard {
    int prev = -1;
    DeviceGuard() { (void)hipGetDevice(&prev); }
    ~DeviceGuard()
    {
        if (prev >= 0) (void)hipSetDevice(prev);
    }
};

int timing_begin(Graph *g, hipStream_t s, std::string *err)
{
    DeviceState &d = g->dev;
    if (!d.timing) return MG_OK;
    if (d.ev_used >= d.ev_start.size()) {
        hipEvent_t a, b;
        HIP_TRY(hipEventCreate(&a));
        HIP_TRY(hipEventCreate(&b));
        d.ev_start.push_back(a);
        d.ev_stop.push_back(b);
    }
    HIP_TRY(hipEventRecord(static_cast<hipEvent_t>(d.ev_start[d.ev_used]), s));
    return MG_OK;
}

int timing_end(Graph *g, hipStream_t s, std::string *err)
{
    DeviceState &d = g->dev;
    if (!d.timing) return MG_OK;
    HIP_TRY(hipEventRecord(static_cast<hipEvent_t>(d.ev_stop[d.ev_used]), s));
    d.ev_used++;
    return MG_OK;
}

using QueryKernel = void (*)(QueryArgs);
using NaiveKernel = void (*)(NaiveArgs);

template <int BLOCK, bool BIG, bool SPARSE, bool ERR>
QueryKernel tier_kernel(uint32_t unroll)
{
    if constexpr (ERR) {
        return query_tier_kernel<BLOCK, BIG, 4, SPARSE, true>;  // one group size for uncertainty queries
    } else {  // loads in flight per lane: two groups
        switch (unroll) {
        case 4: return query_tier_kernel<BLOCK, BIG, 2, SPARSE, false>;
        case 8: return query_tier_kernel<BLOCK, BIG, 4, SPARSE, false>;
        default: return query_tier_kernel<BLOCK, BIG, 8, SPARSE, false>;
        }
    }
}

NaiveKernel naive_variant(uint32_t unroll)
{
    switch (unroll) {
    case 4: return naive_kernel<4>;
    case 8: return naive_kernel<8>;
    default: return naive_kernel<16>;
    }
}

bool valid_unroll(uint32_t u) { return u == 4 || u == 8 || u == 16; }

// Blocks per CU of a kernel variant (queried once, cached per device); also
// raises the kernel's dynamic LDS limit.
// Static LDS of a kernel (its __shared__ variables), as the code object states it.
int static_lds(const void *k, uint32_t *out, std::string *err)
{
    hipFuncAttributes fa{};
    HIP_TRY(hipFuncGetAttributes(&fa, k));
    *out = uint32_t(fa.sharedSizeBytes);
    return MG_OK;
}

int occupancy(DeviceState &d, const void *k, int block, uint32_t dyn, int *out, std::string *err)
{
    for (const auto &e : d.occupancy)
        if (e.kernel == k && e.dyn == dyn) {
            *out = e.blocks;
            return MG_OK;
        }
    uint32_t stat = 0;
    if (int rc = static_lds(k, &stat, err)) return rc;
    if (uint64_t(dyn) + stat > uint64_t(d.lds_max)) {
        *err = "kernel state of " + std::to_string(uint64_t(dyn) + stat) + " bytes exceeds the " +
               std::to_string(d.lds_max) + " bytes of LDS per workgroup";
        return MG_ELIMIT;
    }
    // the attribute is the largest dynamic LDS any launch of this kernel uses
    uint32_t dmax = dyn;
    for (const auto &e : d.occupancy)
        if (e.kernel == k) dmax = std::max(dmax, e.dyn);
    HIP_TRY(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, int(dmax)));
    int occ = 1;
    HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k, block, dyn));
    d.occupancy.push_back(DeviceState::Occ{k, dyn, std::max(occ, 1)});
    *out = std::max(occ, 1);
    return MG_OK;
}

// ---------------------------------------------------------------- no-allocation scratch

// The workspace of mg_query_boxes_noalloc: one array per device, held from the
// module's load until the process ends. Host code never passes `scratch`
// itself to a kernel (in host code the name is a stand-in, not a device
// address); it uses the address hipGetSymbolAddress returns for each device.
constexpr uint64_t kScratchBytes = uint64_t(MG_NOALLOC_SCRATCH_BYTES);
static __device__ __align__(256) char scratch[kScratchBytes];

struct ScratchSlot {
    char *ptr = nullptr;         // device address of `scratch` on this device
    ScratchLayout layout = {};   // last cleared (zeros: never), while no call was captured
    bool captured = false;       // a call was captured: its replays change the layout unseen
};
std::mutex g_scratch_mu;
std::vector<ScratchSlot> g_scratch;      // per device ordinal

// The device address of the scratch array on the current device (looked up once per device).
int scratch_slot(int device, ScratchSlot **out, std::string *err)
{
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (device < 0) {
        *err = "no device";
        return MG_ESTATE;
    }
    if (g_scratch.size() <= size_t(device)) g_scratch.resize(size_t(device) + 1);
    ScratchSlot &sl = g_scratch[size_t(device)];
    if (!sl.ptr) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            *err = std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e);
            return MG_EDEVICE;
        }
        sl.ptr = static_cast<char *>(p);
    }
    *out = &sl;
    return MG_OK;
}

}  // namespace

// ---------------------------------------------------------------- host-side address check

// Every load the query kernels (and, if naive, the naive scan) issue for these
// boxes, replayed on the host with the kernels' own slab builder and tile-walk
// helpers, UNROLL loads per block. counts: [0] boxes, [1] slabs, [2] lane
// loads checked, [3] cubes read.
int check_load_addresses(const uint32_t dims[3], bool use16, bool naive, bool runs, uint32_t run_min,
                         const uint32_t *boxes, uint32_t n, uint32_t unroll, uint64_t counts[4], std::string *err)
{
    LevelTable lt = level_table_dims(dims);
    if (lt.n_levels > kMaxLevelsDev) {
        *err = "more than " + std::to_string(kMaxLevelsDev) + " mip levels";
        return MG_ELIMIT;
    }
    lt.use16 = use16 ? 1u : 0u;
    if (runs) {  // row runs at every level and orientation whose rows the run builder accepts
        lt.run_min = run_min ? run_min : kRunMinRow;
        for (uint32_t l = 0; l < lt.n_levels && 2 * l + 1 < 32; ++l) {
            const uint64_t X = lt.dims[l][0], Y = lt.dims[l][1], Z = lt.dims[l][2];
            if (Y * Z < 0xFFFFFFFFull) lt.runs_mask |= 1u << (2 * l);
            if (Z * X < 0xFFFFFFFFull) lt.runs_mask |= 1u << (2 * l + 1);
        }
    }
    const uint64_t bytes32 = 2 * lt.total * 4;  // maps then maps_t
    const uint64_t n16t = uint64_t(lt.pitch_y) * dims[2] * dims[0];
    const uint64_t bytes16 = (lt.total16 + n16t) * 2;
    for (int k = 0; k < 4; ++k) counts[k] = 0;
    std::vector<Slab> slabs(kMaxSlabs);
    std::string where;
    // Replays every load of a streamed slab's tiles, one per lane, and hands each in-slab
    // unit to unit(t, row, slice, pair bits).
    auto replay_slab = [&](const Slab &sl, uint64_t buf, auto unit) -> bool {
        const uint64_t extent = uint64_t(sl.e2 - 1) * sl.s2b + uint64_t(sl.e1 - 1) * sl.s1b + 4ull * sl.units;
        if (sl.base % 4 != 0) {
            where = "unaligned slab base";
            return false;
        }
        const uint32_t ltx = tile_ltx(sl), ty = 64u >> ltx, n_t0 = (sl.units + (1u << ltx) - 1) >> ltx,
                       n_rt = (sl.e1 + ty - 1) / ty, tiles = slab_tiles(sl);
        if (tiles != uint64_t(n_t0) * n_rt * sl.e2) {
            where = "tile count";
            return false;
        }
        uint64_t seen = 0;
        for (uint32_t o = 0; o < tiles; ++o) {
            const TileDesc d = tile_desc(sl, o);
            const uint32_t t0 = o % n_t0, rt = o / n_t0 % n_rt, k2 = o / n_t0 / n_rt;
            for (uint32_t lane = 0; lane < 64; ++lane) {
                uint32_t mask;
                const uint64_t off = d.off + tile_lane(d.pack, d.s1b, lane, &mask);
                const uint32_t ly = lane >> ltx;
                if (ly && ly < tile_rows(d.pack) &&
                    (d.s1b >= (1u << 24) || uint64_t(ly) * d.s1b + 256u >= (1ull << 32))) {
                    where = "lane offset is no 24-bit product";
                    return false;
                }
                ++counts[2];
                if (off < sl.base || off + 4 > sl.base + extent) {
                    where = "load past the slab";
                    return false;
                }
                if (off + 4 > buf) {
                    where = "load past the buffer";
                    return false;
                }
                if (mask == kEmpty) continue;  // no part of the unit is inside
                const uint32_t x = (t0 << ltx) + (lane & ((1u << ltx) - 1)), row = rt * ty + ly;
                const uint32_t pb = sl.kind ? (mask & 0xFFFFu ? 0u : 1u) | (mask >> 16 ? 0u : 2u) : 1u;
                if (pb != (sl.kind ? pair_bits(x, sl.e0, sl.odd) : 1u) || (sl.kind == 0 && mask)) {
                    where = "elements inside the slab";
                    return false;
                }
                if (x >= sl.units || row >= sl.e1 || tile_level(d.pack) != sl.level ||
                    tile_pairs(d.pack) != (sl.kind == 1) ||
                    off != sl.base + uint64_t(k2) * sl.s2b + uint64_t(row) * sl.s1b + 4ull * x) {
                    where = "load is not its unit";
                    return false;
                }
                ++seen;
                if (!unit(x, row, k2, pb)) return false;
            }
        }
        if (seen != uint64_t(sl.units) * sl.e1 * sl.e2) {
            where = "units read " + std::to_string(seen) + " of " + std::to_string(uint64_t(sl.units) * sl.e1 * sl.e2);
            return false;
        }
        return true;
    };
    // Replays every load of the naive scan's tile walk (all UNROLL loads of every block, consumed
    // or not) and hands each consumed in-slab unit to unit(t, row, slice, pair bits).
    auto replay = [&](const TileWalk &tw, uint64_t base, uint64_t buf, uint32_t e0, uint32_t odd, bool pairs,
                      auto unit) -> bool {
        const uint64_t extent = uint64_t(tw.e2 - 1) * tw.s2b + uint64_t(tw.e1 - 1) * tw.s1b + 4ull * tw.units;
        if (base % 4 != 0) {
            where = "unaligned slab base";
            return false;
        }
        uint64_t seen = 0;
        for (uint32_t b = 0; b < tw.n_blk; ++b) {
            const uint32_t t0 = b % tw.n_t0, rb = (b / tw.n_t0) % tw.n_rb, k2 = b / (tw.n_t0 * tw.n_rb);
            const uint64_t blk = tile_block_offset(tw, t0, rb, k2);
            const uint32_t n_u = tile_n_u(tw, rb, unroll);
            if (n_u < 1) {
                where = "a block without a row tile";
                return false;
            }
            for (uint32_t lane = 0; lane < 64; ++lane) {
                const uint32_t lane_bytes = tile_lane_bytes(tw, lane);
                const uint32_t n_ok = tile_n_ok(tw, t0, rb, lane);
                if (uint64_t((lane >> tw.ltx)) * tw.s1b + (lane & ((1u << tw.ltx) - 1)) * 4ull >= (1ull << 32)) {
                    where = "lane offset does not fit 32 bits";
                    return false;
                }
                const uint32_t x = tile_unit(tw, t0, lane);
                const uint32_t pb = pairs ? pair_bits(x, e0, odd) : 1u;
                for (uint32_t u = 0; u < unroll; ++u) {
                    const uint64_t off = tile_load_offset(tw, blk, u, n_u, n_ok, lane_bytes);
                    ++counts[2];
                    if (off + 4 > extent) {
                        where = "load past the slab";
                        return false;
                    }
                    if (base + off + 4 > buf) {
                        where = "load past the buffer";
                        return false;
                    }
                    if (u < n_u && u < n_ok) {  // consumed, inside the slab
                        const uint32_t row = rb * tw.rows + u * tw.ty + (lane >> tw.ltx);
                        if (off != uint64_t(k2) * tw.s2b + uint64_t(row) * tw.s1b + 4ull * x) {
                            where = "load is not its unit";
                            return false;
                        }
                        ++seen;
                        if (!unit(x, row, k2, pb)) return false;
                    }
                }
            }
        }
        if (seen != uint64_t(tw.units) * tw.e1 * tw.e2) {
            where = "units read " + std::to_string(seen) + " of " + std::to_string(uint64_t(tw.units) * tw.e1 * tw.e2);
            return false;
        }
        return true;
    };
    for (uint32_t q = 0; q < n; ++q) {
        uint32_t lo[3], hi[3];
        if (!clip_box(boxes + 6 * uint64_t(q), lt, lo, hi)) continue;
        ++counts[0];
        int ns = 0;
        uint64_t cubes_closed = 0;
        for (uint32_t l = 0; l < lt.n_levels; ++l) {
            const LevelRow row = level_row(lt, l);
            for (uint32_t face = 0; face < 6; ++face)
                if (face_slab(lt, row, lo, hi, l, face, &slabs[ns])) ++ns;
            uint64_t outer = 1, inner = 1;
            for (int d = 0; d < 3; ++d) {
                const uint64_t one = uint64_t(1) << l;
                const uint64_t a = (uint64_t(lo[d]) + one - 1) >> l, b = hi[d] >> l;
                const uint64_t pa = (uint64_t(lo[d]) + 2 * one - 1) >> (l + 1), pb = hi[d] >> (l + 1);
                outer *= b > a ? b - a : 0;
                inner *= pb > pa ? 2 * (pb - pa) : 0;
            }
            cubes_closed += outer - inner;
        }
        uint64_t cubes = 0;
        for (int i = 0; i < ns; ++i) {
            const Slab &sl = slabs[i];
            ++counts[1];
            const uint32_t L = sl.level;
            if (sl.kind == 2) {  // row runs: every item's row and skip entry, its cells inside the box
                const uint32_t f = sl.axes & 3u, lseg = run_lseg(sl.e0);
                const uint64_t len = lt.dims[L][f], rows = f == 0 ? uint64_t(lt.dims[L][1]) * lt.dims[L][2]
                                                                 : uint64_t(lt.dims[L][2]) * lt.dims[L][0];
                const uint64_t chunks = (len + kRunSkipCells - 1) / kRunSkipCells;
                const uint64_t items = slab_items(sl);
                if (f > 1 || items != (uint64_t(sl.e1) * sl.e2) << lseg) where = "run slab orientation or size";
                for (uint64_t it = 0; where.empty() && it < items; ++it) {
                    uint32_t r, p0, p1;
                    if (!run_item(sl, uint32_t(it), &r, &p0, &p1)) continue;
                    ++counts[2];
                    uint64_t c0;
                    uint32_t n;
                    bool row_end;
                    const bool last = run_skips(uint32_t(rows), uint32_t(chunks), r, p0, p1, &c0, &n, &row_end);
                    const uint64_t c1 = c0 + n;
                    if (r >= rows || c0 >= rows * chunks || last != (c1 == rows * chunks) ||
                        row_end != (c1 == (uint64_t(r) + 1) * chunks) || (!last && c1 >= rows * chunks) || p1 > len || p1 >= 65536) {
                        where = "run row or skip entry out of range";
                        break;
                    }
                    // the segment's first and last cube, and the row they lie on
                    const uint32_t row = uint32_t(it >> lseg);
                    const uint32_t i2 = sl.e2 == 1 ? 0u : row / sl.e1, i1 = row - i2 * sl.e1;
                    const uint32_t fa = f == 0 ? sl.bx : sl.by;
                    for (const uint32_t i0 : {p0 - fa, p1 - 1 - fa}) {
                        uint32_t cx, cy, cz;
                        slab_coords(sl, i0, i1, i2, &cx, &cy, &cz);
                        const uint32_t cc[3] = {cx, cy, cz};
                        for (int d = 0; d < 3; ++d)
                            if ((uint64_t(cc[d]) + 1) << L > hi[d] || uint64_t(cc[d]) << L < lo[d])
                                where = "run segment outside the box";
                        if ((f == 0 ? cy + uint64_t(lt.dims[L][1]) * cz : cz + uint64_t(lt.dims[L][2]) * cx) != r)
                            where = "run segment is not on its row";
                    }
                    cubes += p1 - p0;
                }
                if (!where.empty()) {
                    *err = "box " + std::to_string(q) + " level " + std::to_string(L) + " run slab " +
                           std::to_string(sl.e0) + "x" + std::to_string(sl.e1) + "x" + std::to_string(sl.e2) + ": " +
                           where;
                    return MG_ELIMIT;
                }
                continue;
            }
            const bool tr = (sl.axes & 3) == 1;
            const uint32_t X = lt.dims[L][0], Y = lt.dims[L][1], Z = lt.dims[L][2];
            auto unit = [&](uint32_t x, uint32_t row, uint32_t k2, uint32_t pb) -> bool {
                for (uint32_t h = 0; h < (sl.kind ? 2u : 1u); ++h) {
                    if (!((pb >> h) & 1u)) continue;
                    const uint32_t i0 = sl.kind ? 2 * x + h - sl.odd : x;
                    uint32_t cx, cy, cz;
                    slab_coords(sl, i0, row, k2, &cx, &cy, &cz);
                    const uint32_t cc[3] = {cx, cy, cz};
                    for (int d = 0; d < 3; ++d)
                        if ((uint64_t(cc[d]) + 1) << L > hi[d] || uint64_t(cc[d]) << L < lo[d]) {
                            where = "cube outside the box";
                            return false;
                        }
                    uint64_t el;
                    if (sl.kind) el = tr ? lt.total16 + cy + uint64_t(lt.pitch_y) * (cz + uint64_t(Z) * cx)
                                         : cx + uint64_t(lt.pitch_x) * (cy + uint64_t(Y) * cz);
                    else el = tr ? lt.total + lt.off[L] + cy + uint64_t(Y) * (cz + uint64_t(Z) * cx)
                                 : lt.off[L] + cx + uint64_t(X) * (cy + uint64_t(Y) * cz);
                    const uint64_t byte = sl.base + uint64_t(k2) * sl.s2b + uint64_t(row) * sl.s1b + 4ull * x;
                    const uint64_t at = sl.kind ? byte / 2 + h : byte / 4;
                    if (el != at) {
                        where = "address is not the cube's element";
                        return false;
                    }
                    ++cubes;
                }
                return true;
            };
            if (!replay_slab(sl, sl.kind ? bytes16 : bytes32, unit)) {
                *err = "box " + std::to_string(q) + " level " + std::to_string(L) + " slab " + std::to_string(sl.e0) +
                       "x" + std::to_string(sl.e1) + " kind " + std::to_string(sl.kind) + ": " + where;
                return MG_ELIMIT;
            }
        }
        if (cubes != cubes_closed) {
            *err = "box " + std::to_string(q) + ": " + std::to_string(cubes) + " cubes read, the footprint has " +
                   std::to_string(cubes_closed);
            return MG_ELIMIT;
        }
        counts[3] += cubes;
        if (naive) {  // the naive scan reads level 0 of the box from the x-fastest copy
            uint64_t base;
            uint32_t odd;
            const TileWalk tw = naive_walk(lt, lo, hi, use16, unroll, &base, &odd);
            uint64_t vox = 0;
            auto unit = [&](uint32_t x, uint32_t row, uint32_t k2, uint32_t pb) -> bool {
                for (uint32_t h = 0; h < (use16 ? 2u : 1u); ++h) {
                    if (!((pb >> h) & 1u)) continue;
                    const uint32_t cx = lo[0] + (use16 ? 2 * x + h - odd : x), cy = lo[1] + row, cz = lo[2] + k2;
                    if (cx >= hi[0] || cy >= hi[1] || cz >= hi[2]) {
                        where = "voxel outside the box";
                        return false;
                    }
                    const uint64_t el = use16 ? cx + uint64_t(lt.pitch_x) * (cy + uint64_t(dims[1]) * cz)
                                              : cx + uint64_t(dims[0]) * (cy + uint64_t(dims[1]) * cz);
                    const uint64_t off = base + uint64_t(k2) * tw.s2b + uint64_t(row) * tw.s1b + 4ull * x;
                    if (el != (use16 ? off / 2 + h : off / 4)) {
                        where = "address is not the voxel's element";
                        return false;
                    }
                    ++vox;
                }
                return true;
            };
            const uint64_t vox0 = uint64_t(dims[0]) * dims[1] * dims[2];  // level 0 of the 32-bit maps
            if (!replay(tw, base, use16 ? lt.total16 * 2 : vox0 * 4, hi[0] - lo[0], odd, use16, unit)) {
                *err = "box " + std::to_string(q) + " naive scan: " + where;
                return MG_ELIMIT;
            }
            if (vox != uint64_t(hi[0] - lo[0]) * (hi[1] - lo[1]) * (hi[2] - lo[2])) {
                *err = "box " + std::to_string(q) + " naive scan: voxels read " + std::to_string(vox);
                return MG_ELIMIT;
            }
        }
    }
    return MG_OK;
}

// ---------------------------------------------------------------- entry points

// Byte offsets of the graph's device arrays inside one buffer (each 256-byte
// aligned): what mg_device_bytes sizes and mg_bind_device fills.
struct DeviceLayout {
    uint64_t nodes, leaf, deep_ptr, deep, sched, rank_ptr, mixlen, maps, maps16;
    uint64_t n16, n16t;   // elements of the two 16-bit level-0 copies (0 if none)
    uint64_t run_table;   // RunLevel [2 n_levels]
    std::vector<uint64_t> run_sk, run_rn;  // per level and orientation: skip, runs
    uint64_t bytes;
};

// The nodes of rank 1 and 2 are IDs [nseg, rank1_end) and [rank1_end, rank2_end).
uint32_t rank1_end(const Graph &g) { return g.depth >= 1 ? g.rank_ptr[2] : g.nseg; }
uint32_t rank2_end(const Graph &g) { return g.depth >= 2 ? g.rank_ptr[3] : rank1_end(g); }

DeviceLayout device_layout(const Graph &g)
{
    DeviceLayout L;
    uint64_t off = 0;
    auto take = [&](uint64_t bytes) {
        const uint64_t at = off;
        off += align256(bytes);
        return at;
    };
    const uint64_t nmap = g.lev_off[g.n_levels];
    L.nodes = take(uint64_t(g.n_nodes) * sizeof(NodeTriple));
    L.leaf = take(uint64_t(rank2_end(g) - g.nseg) * sizeof(Leaf));
    ensure_deep(g);
    L.deep_ptr = take(g.deep_ptr.size() * 4);
    L.deep = take(g.deep.size() * sizeof(DeepEntry));
    L.sched = take(uint64_t(g.n_nodes) * sizeof(SchedNode));
    L.rank_ptr = take(g.rank_ptr.size() * 4);
    L.mixlen = take(uint64_t(g.n_nodes) * 4);
    L.maps = take(2 * nmap * 4);  // x-fastest copy, then the y-fastest one
    L.n16 = L.n16t = 0;
    if (g.nseg < 0xFFFFu) {       // 16-bit level 0 for the hot path when every source ID fits
        const LevelTable lt = level_table(g);
        L.n16 = lt.total16;
        L.n16t = uint64_t(lt.pitch_y) * g.dims[2] * g.dims[0];
    }
    L.maps16 = take((L.n16 + L.n16t) * sizeof(uint16_t));
    // row runs of every level and orientation that has them (built from the host maps)
    ensure_runs(g);
    L.run_table = take(2 * uint64_t(g.n_levels) * sizeof(RunLevel));
    for (const LevelRuns &r : g.runs) {
        L.run_sk.push_back(r.rows ? take(r.skip.size() * 4) : 0);
        L.run_rn.push_back(r.rows ? take(r.runs.size() * 8) : 0);
    }
    L.bytes = off;
    return L;
}

// Fills `base` (device memory of layout.bytes bytes on `device`) with the
// graph's arrays and derived copies, enqueued on `stream`, then waits for
// them; the graph then reads only this memory. owned: mg_free releases it.
// Where a graph's maps come from when they are not on the host: its stream.
struct StreamSrc {
    const uint8_t *buf;
    uint64_t size;
    const StreamMaps *sm;
};

// Decodes the stream's voxel data into d.maps (x fastest, every level) on `s`;
// waits for it and checks every node ID.
int decode_stream_maps(Graph *g, const StreamSrc &src, hipStream_t s, std::string *err)
{
    const StreamMaps &sm = *src.sm;
    DeviceState &d = g->dev;
    StreamLevels lv;
    std::memset(&lv, 0, sizeof(lv));
    lv.n_levels = g->n_levels;
    lv.nseg = g->nseg;
    lv.n_nodes = g->n_nodes;
    // the staged words start at the 32-bit word holding (A)'s first bit
    const uint64_t first_byte = (sm.a_bit >> 5) * 4;
    const uint64_t lead = sm.a_bit - first_byte * 8;
    uint64_t bits = 0;
    for (uint32_t l = 0; l < g->n_levels; ++l) {
        lv.off[l] = g->lev_off[l];
        lv.bit[l] = lead + sm.bit_off[l];
        lv.r[l] = sm.r[l];
        lv.lo[l] = sm.lo[l];
        bits = sm.bit_off[l] + uint64_t(sm.r[l]) * (g->lev_off[l + 1] - g->lev_off[l]);
    }
    lv.off[g->n_levels] = g->lev_off[g->n_levels];
    // every field lies in the staged words; one zero word past the last field
    const uint64_t words = (lead + bits + 31) / 32 + 1;
    const uint64_t avail = src.size > first_byte ? std::min<uint64_t>(src.size - first_byte, words * 4) : 0;
    // one allocation for the staged words, the renumbering and the error flag
    void *block = nullptr;
    const uint64_t perm_at = align256(words * 4), bad_at = perm_at + align256(sm.perm.size() * 4);
    if (hipMalloc(&block, bad_at + 4) != hipSuccess) {
        (void)hipGetLastError();
        *err = "device allocation for decoding the graph stream failed";
        return MG_ENOMEM;
    }
    void *const stage = block, *const perm = static_cast<char *>(block) + perm_at,
                *const bad = static_cast<char *>(block) + bad_at;
    int rc = MG_OK;
    uint32_t flag = 0;
    auto run = [&]() -> int {
        HIP_TRY(hipMemcpyAsync(stage, src.buf + first_byte, avail, hipMemcpyHostToDevice, s));
        if (avail < words * 4)  // the stream ends inside the last words: zero the rest
            hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(64), 0, s,
                               static_cast<uint32_t *>(stage) + avail / 4, words - avail / 4, 0u);
        if (avail % 4) {       // a partial last word: its bytes past the stream read as zero
            uint32_t tail = 0;
            std::memcpy(&tail, src.buf + first_byte + (avail / 4) * 4, avail % 4);
            HIP_TRY(hipMemcpyAsync(static_cast<uint32_t *>(stage) + avail / 4, &tail, 4, hipMemcpyHostToDevice, s));
            HIP_TRY(hipStreamSynchronize(s));  // `tail` lives on this stack frame
        }
        if (!sm.perm.empty())
            HIP_TRY(hipMemcpyAsync(perm, sm.perm.data(), sm.perm.size() * 4, hipMemcpyHostToDevice, s));
        hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(64), 0, s, static_cast<uint32_t *>(bad), uint64_t(1), 0u);
        const uint64_t total = g->lev_off[g->n_levels];
        const uint32_t blocks = uint32_t(std::min<uint64_t>((total + 255) / 256, 65536));
        hipLaunchKernelGGL(unpack_maps_kernel, dim3(blocks), dim3(256), 0, s, lv,
                           static_cast<const uint32_t *>(stage), static_cast<const uint32_t *>(perm), d.maps,
                           static_cast<uint32_t *>(bad));
        HIP_TRY(hipGetLastError());
        HIP_TRY(hipMemcpyAsync(&flag, bad, 4, hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
        return MG_OK;
    };
    rc = run();
    (void)hipFree(block);
    if (rc) return rc;
    if (flag) {
        *err = "graph stream: voxel node ID out of range";
        return MG_EFORMAT;
    }
    return MG_OK;
}

int dev_bind(Graph *g, int device, void *base, uint64_t bytes, hipStream_t s, bool owned, std::string *err,
             const StreamSrc *src = nullptr)
{
    DeviceState &d = g->dev;
    const DeviceLayout L = device_layout(*g);
    if (bytes < L.bytes) {
        *err = "device buffer of " + std::to_string(bytes) + " bytes; the graph needs " + std::to_string(L.bytes);
        return MG_EINVAL;
    }
    if (reinterpret_cast<uintptr_t>(base) % 256 != 0) {
        *err = "device buffer must be 256-byte aligned";
        return MG_EINVAL;
    }
    char *b = static_cast<char *>(base);
    const uint64_t nmap = g->lev_off[g->n_levels];
    std::vector<NodeTriple> nodes(g->n_nodes);
    for (uint32_t n = 0; n < g->n_nodes; ++n) nodes[n] = NodeTriple{g->child_a[n], g->child_b[n], g->alpha[n]};
    std::vector<SchedNode> sched(g->n_nodes);
    for (uint32_t i = 0; i < g->n_nodes; ++i) {
        const uint32_t n = g->sched[i];
        sched[i] = SchedNode{g->child_a[n], g->child_b[n], g->alpha[n], n};
    }
    // sources in a node's mixture, bounded by the sum over its two predecessors (IDs are
    // sorted by rank, so predecessors come first); exact when the two are disjoint
    std::vector<uint32_t> mixlen(g->n_nodes, 1u);
    for (uint32_t n = g->nseg; n < g->n_nodes; ++n)
        mixlen[n] = uint32_t(std::min<uint64_t>(g->nseg, uint64_t(mixlen[g->child_a[n]]) + mixlen[g->child_b[n]]));
    d.base = base;
    d.owned = owned;
    d.device = device;
    d.bytes = L.bytes;
    d.nodes = reinterpret_cast<NodeTriple *>(b + L.nodes);
    d.leaf = b + L.leaf;
    d.sched = reinterpret_cast<SchedNode *>(b + L.sched);
    d.rank_ptr = reinterpret_cast<uint32_t *>(b + L.rank_ptr);
    d.mixlen = reinterpret_cast<uint32_t *>(b + L.mixlen);
    d.maps = reinterpret_cast<uint32_t *>(b + L.maps);
    d.maps_t = d.maps + nmap;
    d.maps16 = L.n16 ? reinterpret_cast<uint16_t *>(b + L.maps16) : nullptr;
    HIP_TRY(hipMemcpyAsync(d.nodes, nodes.data(), nodes.size() * sizeof(NodeTriple), hipMemcpyHostToDevice, s));
    static_assert(sizeof(DeepEntry) == sizeof(uint64_t), "entries are staged as 64-bit words");
    if (!g->deep_ptr.empty()) {
        d.deep_ptr = reinterpret_cast<uint32_t *>(b + L.deep_ptr);
        d.deep = b + L.deep;
        HIP_TRY(hipMemcpyAsync(d.deep_ptr, g->deep_ptr.data(), g->deep_ptr.size() * 4, hipMemcpyHostToDevice, s));
        if (!g->deep.empty())
            HIP_TRY(hipMemcpyAsync(d.deep, g->deep.data(), g->deep.size() * 8, hipMemcpyHostToDevice, s));
    }
    if (const uint32_t n_leaf = rank2_end(*g) - g->nseg) {
        hipLaunchKernelGGL(leaf_kernel, dim3((n_leaf + 255) / 256), dim3(256), 0, s, d.nodes, g->nseg, n_leaf,
                           static_cast<Leaf *>(d.leaf));
        HIP_TRY(hipGetLastError());
    }
    HIP_TRY(hipMemcpyAsync(d.sched, sched.data(), sched.size() * sizeof(SchedNode), hipMemcpyHostToDevice, s));
    HIP_TRY(hipMemcpyAsync(d.rank_ptr, g->rank_ptr.data(), g->rank_ptr.size() * 4, hipMemcpyHostToDevice, s));
    HIP_TRY(hipMemcpyAsync(d.mixlen, mixlen.data(), mixlen.size() * 4, hipMemcpyHostToDevice, s));
    if (src) {
        if (int rc = decode_stream_maps(g, *src, s, err)) return rc;
    } else {
        HIP_TRY(hipMemcpyAsync(d.maps, g->maps.data(), nmap * 4, hipMemcpyHostToDevice, s));
    }
    for (uint32_t l = 0; l < g->n_levels; ++l) {
        const uint32_t X = g->lev_dims[3 * l], Y = g->lev_dims[3 * l + 1], Z = g->lev_dims[3 * l + 2];
        const uint64_t cnt = uint64_t(X) * Y * Z;
        const uint32_t blocks = uint32_t((cnt + 255) / 256);
        hipLaunchKernelGGL(transpose_level_kernel, dim3(blocks), dim3(256), 0, s, d.maps + g->lev_off[l],
                           d.maps_t + g->lev_off[l], X, Y, Z);
        HIP_TRY(hipGetLastError());
    }
    if (L.n16) {
        const LevelTable lt = level_table(*g);
        const uint64_t n = std::max(L.n16, L.n16t);
        hipLaunchKernelGGL(pack16_kernel, dim3(uint32_t((n + 255) / 256)), dim3(256), 0, s, d.maps, d.maps16,
                           g->dims[0], g->dims[1], g->dims[2], lt.pitch_x, lt.pitch_y, L.n16, L.n16t);
        HIP_TRY(hipGetLastError());
    }
    // row runs and their table
    std::vector<RunLevel> table(2 * size_t(g->n_levels));
    d.runs_mask = 0;
    d.runs = nullptr;
    for (size_t k = 0; k < g->runs.size() && k < table.size(); ++k) {
        const LevelRuns &r = g->runs[k];
        RunLevel &t = table[k];
        t = RunLevel{nullptr, nullptr, 0, 0, 0, 0};
        if (!r.rows || r.runs.empty()) continue;
        t.skip = reinterpret_cast<const uint32_t *>(b + L.run_sk[k]);
        t.runs = reinterpret_cast<const uint64_t *>(b + L.run_rn[k]);
        t.rows = r.rows, t.chunks = r.chunks, t.n_runs = uint32_t(r.runs.size());
        // runs are read by their 32-bit index from the first array (levels past that keep none)
        if (!d.runs) d.runs = t.runs;
        if (uint64_t(t.runs - d.runs) + t.n_runs > 0xFFFFFFFFull) {
            t = RunLevel{nullptr, nullptr, 0, 0, 0, 0};
            continue;
        }
        t.first = uint32_t(t.runs - d.runs);
        HIP_TRY(hipMemcpyAsync(b + L.run_sk[k], r.skip.data(), r.skip.size() * 4, hipMemcpyHostToDevice, s));
        HIP_TRY(hipMemcpyAsync(b + L.run_rn[k], r.runs.data(), r.runs.size() * 8, hipMemcpyHostToDevice, s));
        if (k < 32) d.runs_mask |= 1u << k;
    }
    d.run_table = b + L.run_table;
    if (!table.empty())
        HIP_TRY(hipMemcpyAsync(d.run_table, table.data(), table.size() * sizeof(RunLevel), hipMemcpyHostToDevice, s));
    // the host staging vectors above die with this call
    HIP_TRY(hipStreamSynchronize(s));
    // set-up of the no-allocation path on this device (the scratch array's address)
    ScratchSlot *sl = nullptr;
    if (int rc = scratch_slot(device, &sl, err)) return rc;
    if (!g->lut_ptr.empty()) return dev_upload_lut(g, err);
    return MG_OK;
}

uint64_t dev_device_bytes(const Graph &g) { return device_layout(g).bytes; }

int dev_bind_device(Graph *g, int device, void *base, uint64_t bytes, void *stream, std::string *err)
{
    if (g->maps_on_device) {
        *err = "the graph's node maps exist only on its device (decoded from a stream there)";
        return MG_ESTATE;
    }
    DeviceGuard guard;
    if (g->dev.device >= 0) dev_free(g);
    int ndev = 0;
    HIP_TRY(hipGetDeviceCount(&ndev));
    if (device < 0 || device >= ndev) {
        *err = "device " + std::to_string(device) + " does not exist";
        return MG_EINVAL;
    }
    HIP_TRY(hipSetDevice(device));
    int rc = MG_ENOMEM;
    try {
        rc = dev_bind(g, device, base, bytes, static_cast<hipStream_t>(stream), false, err);
    } catch (const std::bad_alloc &) {
        *err = "out of host memory";
    }
    if (rc) dev_free(g);
    return rc;
}

int upload_with(Graph *g, int device, const StreamSrc *src, std::string *err)
{
    DeviceGuard guard;
    if (g->dev.device >= 0) dev_free(g);
    int ndev = 0;
    HIP_TRY(hipGetDeviceCount(&ndev));
    if (device >= ndev) {
        *err = "mg_upload: device " + std::to_string(device) + " does not exist";
        return MG_EINVAL;
    }
    HIP_TRY(hipSetDevice(device));
    const uint64_t bytes = device_layout(*g).bytes;
    void *base = nullptr;
    if (hipMalloc(&base, bytes) != hipSuccess) {
        (void)hipGetLastError();
        *err = "mg_upload: device allocation of " + std::to_string(bytes) + " bytes failed";
        return MG_ENOMEM;
    }
    int rc = MG_ENOMEM;
    try {
        rc = dev_bind(g, device, base, bytes, nullptr, true, err, src);
    } catch (const std::bad_alloc &) {
        *err = "out of host memory";
    }
    if (rc) {
        if (g->dev.base != base) (void)hipFree(base);  // not recorded yet: release it here
        dev_free(g);
    }
    return rc;
}

int dev_upload(Graph *g, int device, std::string *err)
{
    if (g->maps_on_device) {
        *err = "the graph's node maps exist only on its device (decoded from a stream there)";
        return MG_ESTATE;
    }
    return upload_with(g, device, nullptr, err);
}

int dev_upload_stream(Graph *g, const uint8_t *buf, uint64_t size, const StreamMaps &sm, int device,
                      std::string *err)
{
    const StreamSrc src{buf, size, &sm};
    return upload_with(g, device, &src, err);
}

int dev_export_map(const Graph &g, uint32_t level, uint32_t *out, std::string *err)
{
    if (g.dev.device < 0 || !g.dev.maps) {
        *err = "the graph is not on a device";
        return MG_ESTATE;
    }
    DeviceGuard guard;
    HIP_TRY(hipSetDevice(g.dev.device));
    const uint64_t n = g.lev_off[level + 1] - g.lev_off[level];
    HIP_TRY(hipMemcpy(out, g.dev.maps + g.lev_off[level], n * 4, hipMemcpyDeviceToHost));
    return MG_OK;
}

int dev_upload_lut(Graph *g, std::string *err)
{
    DeviceGuard guard;
    DeviceState &d = g->dev;
    if (d.device < 0) {
        *err = "graph not on a device";
        return MG_ESTATE;
    }
    HIP_TRY(hipSetDevice(d.device));
    if (d.lut_ptr) (void)hipFree(d.lut_ptr);
    if (d.lut_seg) (void)hipFree(d.lut_seg);
    if (d.lut_val) (void)hipFree(d.lut_val);
    if (d.lut_err) (void)hipFree(d.lut_err);
    d.lut_ptr = nullptr, d.lut_seg = nullptr, d.lut_val = nullptr, d.lut_err = nullptr;
    const uint64_t bp = g->lut_ptr.size() * sizeof(uint64_t), nnz = g->lut_seg.size();
    if (hipMalloc(&d.lut_ptr, bp) != hipSuccess || hipMalloc(&d.lut_seg, nnz * 4) != hipSuccess ||
        hipMalloc(&d.lut_val, nnz * 4) != hipSuccess) {
        (void)hipGetLastError();
        if (d.lut_ptr) (void)hipFree(d.lut_ptr);
        if (d.lut_seg) (void)hipFree(d.lut_seg);
        d.lut_ptr = nullptr, d.lut_seg = nullptr, d.lut_val = nullptr;
        *err = "mixture lookup table: device allocation failed";
        return MG_ENOMEM;
    }
    HIP_TRY(hipMemcpy(d.lut_ptr, g->lut_ptr.data(), bp, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(d.lut_seg, g->lut_seg.data(), nnz * 4, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(d.lut_val, g->lut_val.data(), nnz * 4, hipMemcpyHostToDevice));
    d.bytes += bp + 8 * nnz;
    if (g->lut_err.size() == nnz && nnz) {
        if (hipMalloc(&d.lut_err, nnz * 4) != hipSuccess) {
            (void)hipGetLastError();
            d.lut_err = nullptr;
            *err = "mixture lookup table: device allocation failed (uncertainties)";
            return MG_ENOMEM;
        }
        HIP_TRY(hipMemcpy(d.lut_err, g->lut_err.data(), nnz * 4, hipMemcpyHostToDevice));
        d.bytes += 4 * nnz;
    }
    return MG_OK;
}

int dev_palette_fetch(Graph *g, const float *palette, uint32_t T, uint32_t level, const uint32_t *xyz, uint32_t n,
                      float *out, void *stream, std::string *err)
{
    DeviceGuard guard;
    int rc = check_device(g, err);
    if (rc) return rc;
    const uint32_t X = g->lev_dims[3 * level], Y = g->lev_dims[3 * level + 1], Z = g->lev_dims[3 * level + 2];
    hipLaunchKernelGGL(palette_fetch_kernel, dim3((n + 255) / 256), dim3(256), 0, static_cast<hipStream_t>(stream),
                       reinterpret_cast<const float4 *>(palette), T, g->n_nodes, g->dev.maps + g->lev_off[level], X,
                       Y, Z, xyz, n, reinterpret_cast<float4 *>(out));
    HIP_TRY(hipGetLastError());
    return MG_OK;
}

int dev_box_colour(Graph *g, const float *palette, uint32_t T, const uint32_t *boxes, uint32_t n,
                   const uint32_t *pal_of_box, float *out, void *stream, std::string *err)
{
    DeviceGuard guard;
    int rc = check_device(g, err);
    if (rc) return rc;
    if (g->n_levels > kMaxLevelsDev) {
        *err = "more than " + std::to_string(kMaxLevelsDev) + " mip levels";
        return MG_ELIMIT;
    }
    const LevelTable lt = level_table(*g);
    hipLaunchKernelGGL(box_colour_kernel, dim3(n), dim3(kColourBlock), 0, static_cast<hipStream_t>(stream), lt, boxes, n,
                       g->dev.maps, reinterpret_cast<const float4 *>(palette), T, g->n_nodes, pal_of_box,
                       reinterpret_cast<float4 *>(out));
    HIP_TRY(hipGetLastError());
    return MG_OK;
}

void dev_free(Graph *g)
{
    DeviceState &d = g->dev;
    if (d.device < 0 && !d.base) return;
    DeviceGuard guard;
    if (d.device >= 0) (void)hipSetDevice(d.device);
    if (d.base && d.owned) (void)hipFree(d.base);
    if (d.lut_ptr) (void)hipFree(d.lut_ptr);
    if (d.lut_seg) (void)hipFree(d.lut_seg);
    if (d.lut_val) (void)hipFree(d.lut_val);
    if (d.lut_err) (void)hipFree(d.lut_err);
    for (void *e : d.ev_start) (void)hipEventDestroy(static_cast<hipEvent_t>(e));
    for (void *e : d.ev_stop) (void)hipEventDestroy(static_cast<hipEvent_t>(e));
    d = DeviceState();
}

uint64_t dev_workspace_bytes(const Graph &g, uint32_t max_boxes)
{
    return carve(g, nullptr, std::max<uint32_t>(max_boxes, 1)).bytes;
}

// Everything a query expects clean and leaves clean: the fixed part of a workspace.
ClearRanges clean_state(const Graph &g, const Workspace &w)
{
    ClearRanges c;
    c.n = 0;
    auto add = [&](void *p, uint64_t words, uint32_t value) {
        if (!words) return;
        c.r[c.n].p = static_cast<uint32_t *>(p), c.r[c.n].words = words, c.r[c.n].value = value;
        ++c.n;
    };
    for (const GlobalPool *p : {&w.fin, &w.mid}) {
        const uint64_t hs = uint64_t(p->workers) * p->slots, ss = uint64_t(p->workers) * g.nseg;
        add(p->keys, hs, kEmpty);
        for (void *a : {static_cast<void *>(p->cnt), static_cast<void *>(p->hi), static_cast<void *>(p->lo)})
            add(a, hs, 0);
        for (void *a : {static_cast<void *>(p->seg_cnt), static_cast<void *>(p->seg_hi), static_cast<void *>(p->seg_lo),
                        static_cast<void *>(p->seg_var)})
            add(a, ss, 0);
    }
    const uint64_t ns = w.n_slots;
    add(w.counters, 64, 0);
    add(w.buckets, 64, 0);
    add(w.queues, uint64_t(kQueues) * kQueueStride, 0);
    add(w.slot_done, ns, 0);
    for (void *a : {static_cast<void *>(w.slot_cnt), static_cast<void *>(w.slot_hi), static_cast<void *>(w.slot_lo),
                    static_cast<void *>(w.slot_var)})
        add(a, ns * g.nseg, 0);
    static_assert(2 * 8 + 3 + 5 <= kMaxRanges, "one entry per array");
    return c;
}

// By a kernel on `s` (no memset: callers may capture the stream into a graph).
void clear_workspace(const Graph &g, const Workspace &w, hipStream_t s)
{
    hipLaunchKernelGGL(clear_kernel, dim3(1024), dim3(256), 0, s, clean_state(g, w),
                       static_cast<const uint64_t *>(nullptr), ScratchLayout{});
}

int dev_workspace_init(Graph *g, void *work, uint64_t bytes, void *stream, std::string *err)
{
    int rc = check_device(g, err);
    if (rc) return rc;
    // the fixed-size part (counters, queues, fallback tables) comes first, so its
    // layout does not depend on the box capacity
    Workspace w = carve(*g, static_cast<char *>(work), 1);
    if (bytes < w.bytes) {
        *err = "workspace smaller than mg_workspace_bytes(g, 1)";
        return MG_EINVAL;
    }
    clear_workspace(*g, w, static_cast<hipStream_t>(stream));
    HIP_TRY(hipGetLastError());
    return MG_OK;
}

// Every kernel, table size and launch size of a call is settled before its first launch, so that a
// call refused for its limits has enqueued nothing; *began tells a caller whose call failed that
// launches before the failure may have left the workspace's counters and slots in use.
template <bool SPARSE, bool ERR>
int launch_query(Graph *g, QueryArgs &A, const LevelTable &lt, const Workspace &w, uint32_t n, hipStream_t s,
                 int variant, bool *began, std::string *err)
{
    int rc = MG_OK;
    DeviceState &d = g->dev;
    const uint32_t L = g->n_levels;
    auto bytes = [&](uint32_t cap, bool table) -> uint32_t {
        if (!table && g->nseg > (1u << 20)) return 1u << 30;  // no LDS holds them (nor 32 bits their bytes)
        return lds_bytes(g->nseg, cap, table, A.counts != 0, L, ERR);
    };
    // nodes that can become entries of a box's table: with counts only those its cubes are on
    const uint32_t n_entries = g->n_nodes - A.gv.r2_end;
    auto holds_all = [&](uint32_t cap, bool table) { return !table && A.counts && n_entries <= cap / 4 * 3; };
    // SPARSE (sparse output, or many sources): small boxes keep their few sources as table entries.
    // Large ones would fill any table with them, mostly after much of their work (20,000 boxes of
    // a 307x480x300 volume of 3,980 fibres: 90 ms, nearly all of it boxes done once in a table of
    // 4,096 slots that overflowed and once more in one of 8,192), so they get per-source arrays
    // wherever those fit the LDS of a workgroup beside a node table of this size.
    auto by_table = [&](uint32_t cap) {
        return SPARSE && uint64_t(bytes(cap, false)) + kStaticLds > uint64_t(d.lds_max);
    };
    auto set_size = [&](uint32_t cap) {
        const uint64_t state = lds_state_bytes(g->nseg, cap, false, A.counts != 0) + 6u * L * sizeof(Slab) + (ERR ? 4u * g->nseg : 0u);
        return !SPARSE && uint64_t(bytes(cap, false)) + kStaticLds > uint64_t(d.lds_max) &&
                       state + kStaticLdsSet <= uint64_t(d.lds_max) ? cap / 2 : cap;
    };
    auto level0 = [&](bool table) { A.lt.use16 = (!table && d.maps16) ? 1u : 0u; };  // sources only: 16 bits
    // workgroups of a kernel that are resident together
    auto resident = [&](const void *k, int block, uint32_t dyn, uint32_t *out) -> int {
        int occ = 1;
        if (int r = occupancy(d, k, block, dyn, &occ, err)) return r;
        *out = uint32_t(d.ncu) * uint32_t(occ);
        return MG_OK;
    };
    // what overflows its table: once more with a larger LDS table, then in global memory
    uint32_t cap_retry = d.cfg.table_retry ? set_size(d.cfg.table_retry) : kHashRetry;
    if (!d.cfg.table_retry)  // the largest table up to kHashRetry that fits the LDS of a workgroup
        while (cap_retry > kHashBig && uint64_t(bytes(cap_retry, false)) + kStaticLds > uint64_t(d.lds_max)) cap_retry /= 2;
    const bool retry_table = by_table(cap_retry);
    if (retry_table && !d.cfg.table_retry) cap_retry = kHashBigSparse;
    const auto kretry = retry_table ? query_retry_kernel<kBlockBig, 4, SPARSE, ERR>
                                    : query_retry_kernel<kBlockBig, 4, false, ERR>;
    const uint32_t dyn_retry = bytes(cap_retry, retry_table);
    uint32_t wretry = 0;
    auto resident_retry = [&]() { return resident(reinterpret_cast<const void *>(kretry), kBlockBig, dyn_retry, &wretry); };
    const bool batched = variant == kQueryBatched || variant == kQueryLut;
    if (batched && n <= kDirectMax) {
        // few boxes: no planning launches
        // the default table holds every node that can enter it where a small one does: then no
        // box can overflow, and no launch has to follow
        A.table_cap = kHashDirect;
        while (A.table_cap < kHashDirectMax && !holds_all(A.table_cap, false)) A.table_cap *= 2;
        if (!holds_all(A.table_cap, false)) A.table_cap = ERR ? kHashBigErr : kHashBig;
        if (d.cfg.table_big) A.table_cap = set_size(d.cfg.table_big);
        const bool table = by_table(A.table_cap);
        if (table && !d.cfg.table_big) A.table_cap = kHashBigSparse;
        const auto kdirect = table ? query_direct_kernel<kBlockDirect, 4, SPARSE, ERR>
                                   : query_direct_kernel<kBlockDirect, 4, false, ERR>;
        const uint32_t dyn = bytes(A.table_cap, table);
        level0(table);
        uint32_t grid = 0;
        const bool alone = holds_all(A.table_cap, table);
        if ((rc = resident(reinterpret_cast<const void *>(kdirect), kBlockDirect, dyn, &grid))) return rc;
        if (!alone && (rc = resident_retry())) return rc;
        *began = true;
        if (A.sp_total) hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(64), 0, s, A.sp_total, uint64_t(1), 0u);
        // about two parts per CU: 256 boxes of a 589x563x395 volume take 34 us so, 40 with one
        const uint32_t ways = ERR ? 0u : std::min({grid, 2u * uint32_t(d.ncu), A.n_slots});
        if ((rc = timing_begin(g, s, err))) return rc;
        hipLaunchKernelGGL(kdirect, dim3(std::min(grid, n + 2 * ways)), dim3(kBlockDirect), dyn, s, A, ways, kMinPart);
        HIP_TRY(hipGetLastError());
        if (alone) return timing_end(g, s, err);
    } else if (batched) {
        // Default table: half the size where the graph has few nodes that can enter it (the largest
        // boxes hold up to about an eighth of them). 353 segments, 2,624 such nodes, 100,000 boxes:
        // 1.11 ms with 1,024 slots, 1.20 with 2,048; 591 segments, 9,958 nodes, 20,000 boxes: 444 us
        // with 1,024 (some boxes overflow), 352 with 2,048.
        const bool few = A.counts && !ERR && n_entries / 8 <= kHashDirect / 4 * 3;
        uint32_t cap_big = d.cfg.table_big ? set_size(d.cfg.table_big) : ERR ? kHashBigErr : few ? kHashDirect : kHashBig;
        const bool table = by_table(cap_big);
        if (table && !d.cfg.table_big) cap_big = kHashBigSparse;
        const uint32_t dyn_big = bytes(cap_big, table);
        auto big = [&](int block) {
            return table ? (block == 256 ? tier_kernel<256, true, SPARSE, ERR>(d.cfg.unroll_big)
                                         : tier_kernel<kBlockBig, true, SPARSE, ERR>(d.cfg.unroll_big))
                         : (block == 256 ? tier_kernel<256, true, false, ERR>(d.cfg.unroll_big)
                                         : tier_kernel<kBlockBig, true, false, ERR>(d.cfg.unroll_big));
        };
        // Threads per big-tier box: the choice that keeps more waves resident beside the per-box
        // LDS, and of two equal ones the smaller workgroup (100,000 boxes of 512^3, 353 segments, 24
        // waves per CU both: 1.11 ms with 256 threads, 1.20 with 512; 20,000 boxes of 591 segments,
        // 16 and 24 waves: 410 and 351 us). Batches of few boxes per workgroup take the larger one,
        // whose boxes end sooner (5,000 boxes of 199x181x163: 113 us with 256, 100 with 512).
        uint32_t wbig = 0, w512 = 0;
        int bbig = d.cfg.block_big ? int(d.cfg.block_big) : 256;
        if ((rc = resident(reinterpret_cast<const void *>(big(bbig)), bbig, dyn_big, &wbig))) return rc;
        if (!d.cfg.block_big && uint64_t(dyn_big) + kStaticLds <= uint64_t(d.lds_max)) {
            if ((rc = resident(reinterpret_cast<const void *>(big(kBlockBig)), kBlockBig, dyn_big, &w512))) return rc;
            if (2 * w512 > wbig || n < 8 * wbig) bbig = kBlockBig, wbig = w512;
        }
        const QueryKernel kbig = big(bbig);
        const int bsmall = d.cfg.block_small == 256 ? kBlock : 128;  // threads per small-tier box
        const QueryKernel ksmall = bsmall == 128 ? tier_kernel<128, false, SPARSE, ERR>(d.cfg.unroll_small)
                                                 : tier_kernel<kBlock, false, SPARSE, ERR>(d.cfg.unroll_small);
        const uint32_t cap_small = d.cfg.table_small ? d.cfg.table_small : (SPARSE ? kHashSmallSparse : ERR ? kHashSmallErr : kHashSmall);
        const uint32_t dyn_small = bytes(cap_small, SPARSE);
        uint32_t wsmall = 0;
        if ((rc = resident(reinterpret_cast<const void *>(ksmall), bsmall, dyn_small, &wsmall))) return rc;
        if ((rc = resident_retry())) return rc;
        *began = true;
        const uint32_t blocks = (n + 255) / 256;
        hipLaunchKernelGGL(query_size_kernel, dim3(blocks), dim3(256), 0, s, lt, A.boxes, n, w.work, w.buckets,
                           w.counters, A.sp_total);
        hipLaunchKernelGGL(query_order_kernel, dim3(blocks), dim3(256), 0, s, w.work, n, w.buckets, w.order,
                           w.counters, w.split, ERR ? 0u : A.n_slots, kMinPartBatch, SPARSE ? kBigLog2Sparse : kBigLog2);
        A.order = w.order;
        if ((rc = timing_begin(g, s, err))) return rc;
        A.table_cap = cap_big;
        level0(table);
        hipLaunchKernelGGL(kbig, dim3(std::min(n + 2 * A.n_slots, wbig)), dim3(bbig), dyn_big, s, A);
        HIP_TRY(hipGetLastError());
        A.table_cap = cap_small;
        level0(SPARSE);
        A.chunk = d.cfg.chunk_small;
        hipLaunchKernelGGL(ksmall, dim3(std::min(n, wsmall)), dim3(bsmall), dyn_small, s, A);
        HIP_TRY(hipGetLastError());
    } else {
        const QueryKernel kplain = query_plain_kernel<SPARSE>;
        A.table_cap = kHashPlain;
        uint32_t all = 0;
        if ((rc = resident(reinterpret_cast<const void *>(kplain), kBlock, bytes(kHashPlain, SPARSE), &all))) return rc;
        if ((rc = resident_retry())) return rc;
        *began = true;
        if (A.sp_total) hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(64), 0, s, A.sp_total, uint64_t(1), 0u);
        if ((rc = timing_begin(g, s, err))) return rc;
        level0(SPARSE);
        hipLaunchKernelGGL(kplain, dim3(n), dim3(kBlock), bytes(kHashPlain, SPARSE), s, A);
        HIP_TRY(hipGetLastError());
    }
    A.table_cap = cap_retry;
    level0(retry_table);
    // no more workgroups than there can be entries for (a box, or its parts)
    const bool last = holds_all(cap_retry, retry_table);
    hipLaunchKernelGGL(kretry, dim3(std::min(wretry, n + 4 * A.n_slots)), dim3(kBlockBig), dyn_retry, s, A,
                       last ? 1u : 0u);
    HIP_TRY(hipGetLastError());
    if (last) return timing_end(g, s, err);
    const auto kfallback = query_fallback_kernel<ERR>;
    const uint32_t dyn_fb = lds_slab_bytes(L);
    level0(false);  // per-source arrays
    if (w.mid.workers) {
        hipLaunchKernelGGL(kfallback, dim3(w.mid.workers), dim3(kBlock), dyn_fb, s, A, w.mid, 2u, 0u);
        HIP_TRY(hipGetLastError());
    }
    hipLaunchKernelGGL(kfallback, dim3(w.fin.workers), dim3(kBlock), dyn_fb, s, A, w.fin, w.mid.workers ? 3u : 2u, 1u);
    HIP_TRY(hipGetLastError());
    // the timed region: every kernel that answers boxes
    return timing_end(g, s, err);
}

namespace {

// The query path on a carved workspace (the caller's or the library's scratch).
int query_in(Graph *g, const uint32_t *boxes, uint32_t n, float *out, const SparseOut *sp, const Workspace &w,
             hipStream_t s, int variant, uint32_t *stats, std::string *err, float *out_err)
{
    int rc = MG_OK;
    if (g->depth > kMaxSteps) {
        *err = "graph depth " + std::to_string(g->depth) + " beyond the kernels' step table (" +
               std::to_string(kMaxSteps) + ")";
        return MG_ELIMIT;
    }
    if (g->n_levels > kMaxLevelsDev) {
        *err = "more than " + std::to_string(kMaxLevelsDev) + " mip levels";
        return MG_ELIMIT;
    }
    const LevelTable lt = level_table(*g);
    if (!g->dev.launch_ready) {
        HIP_TRY(hipDeviceGetAttribute(&g->dev.lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, g->dev.device));
        HIP_TRY(hipDeviceGetAttribute(&g->dev.ncu, hipDeviceAttributeMultiprocessorCount, g->dev.device));
        g->dev.launch_ready = true;
    }

    if (variant == kQueryNaive) {
        if (g->nseg > 16384) {
            *err = "naive scan keeps per-source counts in LDS: at most 16384 sources";
            return MG_ELIMIT;
        }
        if (sp) {
            *err = "the naive scan writes dense output only";
            return MG_EINVAL;
        }
        NaiveArgs A;
        A.lt = lt;
        A.boxes = boxes;
        A.out = out;
        A.map0 = g->dev.maps;
        A.map16 = g->dev.maps16;
        A.lt.use16 = g->dev.maps16 ? 1u : 0u;
        A.nseg = g->nseg;
        A.n = n;
        rc = timing_begin(g, s, err);
        if (rc) return rc;
        hipLaunchKernelGGL(naive_variant(g->dev.cfg.unroll_naive), dim3(n), dim3(kBlock), g->nseg * 4, s, A);
        HIP_TRY(hipGetLastError());
        return timing_end(g, s, err);
    }

    QueryArgs A;
    std::memset(&A, 0, sizeof(A));
    A.lt = lt;
    A.boxes = boxes;
    A.out = sp ? nullptr : out;
    if (sp) {
        A.sp_index = sp->index;
        A.sp_seg = sp->seg;
        A.sp_val = sp->val;
        A.sp_cap = sp->cap;
        A.sp_total = sp->total;
    }
    A.maps = g->dev.maps;
    A.maps16 = g->dev.maps16;
    A.gv.nodes = g->dev.nodes;
    A.gv.nseg = g->nseg;
    A.gv.leaf = reinterpret_cast<const Leaf *>(g->dev.leaf);
    A.gv.runs = g->dev.runs;
    A.gv.deep_ptr = g->dev.deep_ptr;
    A.gv.deep = static_cast<const DeepEntry *>(g->dev.deep);
    A.gv.r1_end = rank1_end(*g);
    A.gv.r2_end = rank2_end(*g);
    A.rank_ptr = g->dev.rank_ptr;
    A.depth = g->depth;
    A.n = n;
    A.counters = w.counters;
    A.queues = w.queues;
    A.buckets = w.buckets;
    A.overflow = w.overflow;
    A.overflow2 = w.overflow2;
    A.overflow3 = w.overflow3;
    A.stats = stats;
    // Shared boxes: not where a box's table entries are reported; list entries hold box numbers
    // below kPartFlag.
    A.n_slots = stats || variant == kQueryPlain || n >= kPartFlag ? 0u : w.n_slots;
    A.split = w.split;
    A.split_over = w.split_over;
    A.slot_done = w.slot_done;
    A.slot_cnt = w.slot_cnt;
    A.slot_hi = w.slot_hi;
    A.slot_lo = w.slot_lo;
    A.slot_var = w.slot_var;
    if (variant == kQueryLut || variant == kQueryLutErr) {
        if (!g->dev.lut_ptr) {
            *err = "the mixture lookup table is not on the device (mg_lut_build)";
            return MG_ESTATE;
        }
        A.lut_ptr = g->dev.lut_ptr;
        A.lut_seg = g->dev.lut_seg;
        A.lut_val = g->dev.lut_val;
    }
    if (variant == kQueryLutErr) {
        if (!g->dev.lut_err) {
            *err = "uncertainties need a graph with quantized weights (mg_quantize) and its lookup table";
            return MG_ESTATE;
        }
        if (sp || g->nseg > kSegLdsMax) {
            *err = "uncertainty queries keep per-source arrays in LDS: at most " + std::to_string(kSegLdsMax) +
                   " sources, dense output";
            return MG_ELIMIT;
        }
        A.lut_err = g->dev.lut_err;
        A.out_err = out_err;
        // every internal node is a table entry, so each node's count meets its row's uncertainty once
        A.gv.r1_end = A.gv.r2_end = g->nseg;
        variant = kQueryLut;
    }
    // Nodes of rank >= 3 are expanded by the lookup table where the call names it, else by the graph's
    // own rows; without rows, and where the nodes a box reaches are reported, mass is pushed instead.
    // (100,000 boxes of a 512^3 volume by the table / by the rows: 1.114 / 1.112 ms, 5,000 boxes of
    // 199x181x163: 106.6 / 106.1 us.)
    A.counts = A.lut_ptr || (A.gv.deep_ptr && !stats) ? 1u : 0u;
    // sources in LDS arrays while they fit, else as table entries (sparse mode)
    const bool sparse = sp != nullptr || g->nseg > kSegLdsMax;
    // row runs where the graph has them, for slabs whose rows are long enough
    const uint32_t run_min = g->dev.cfg.run_min_row ? g->dev.cfg.run_min_row : kRunMinRow;
    A.lt.runs_mask = run_min == 0xFFFFFFFFu ? 0u : g->dev.runs_mask;
    A.lt.run_min = run_min;
    A.runs = static_cast<const RunLevel *>(g->dev.run_table);
    bool began = false;
    if (A.out_err) rc = launch_query<false, true>(g, A, lt, w, n, s, variant, &began, err);
    else rc = sparse ? launch_query<true, false>(g, A, lt, w, n, s, variant, &began, err)
                     : launch_query<false, false>(g, A, lt, w, n, s, variant, &began, err);
    // a call that ends early does not reach the launches that leave the workspace clean
    if (rc && began) {
        clear_workspace(*g, w, s);
        (void)hipGetLastError();  // *err already says what failed; nothing is left for the next call to find
    }
    return rc;
}

}  // namespace

int dev_query(Graph *g, const uint32_t *boxes, uint32_t n, float *out, const SparseOut *sp, void *work,
              uint64_t bytes, void *stream, int variant, uint32_t *stats, std::string *err, float *out_err)
{
    DeviceGuard guard;
    int rc = check_device(g, err);
    if (rc) return rc;
    const uint64_t need = dev_workspace_bytes(*g, n);
    if (bytes < need) {
        *err = "workspace of " + std::to_string(bytes) + " bytes is smaller than the " + std::to_string(need) +
               " bytes that " + std::to_string(n) + " boxes need";
        return MG_EINVAL;
    }
    const Workspace w = carve(*g, static_cast<char *>(work), n);
    return query_in(g, boxes, n, out, sp, w, static_cast<hipStream_t>(stream), variant, stats, err, out_err);
}

int dev_query_noalloc(Graph *g, const uint32_t *boxes, uint32_t n, float *out, void *stream, std::string *err)
{
    DeviceGuard guard;
    int rc = check_device(g, err);
    if (rc) return rc;
    ScratchSlot *sl = nullptr;
    if ((rc = scratch_slot(g->dev.device, &sl, err))) return rc;
    // as many workers of the final global tables as fit beside the per-box arrays (at least
    // one), none with mid-size tables (a speed-up only: every box fits the final tables)
    uint32_t workers = fallback_workers(*g), slots = std::min(split_slots(*g), kNoallocSlots);
    auto size = [&](uint32_t f, uint32_t ns) { return carve(*g, nullptr, n, f, 0, ns).bytes; };
    if (size(std::min(workers, kNoallocWorkers), slots) > kScratchBytes) slots = 0;  // room for the workers first
    while (workers > 1 && size(workers, slots) > kScratchBytes) --workers;
    if (size(workers, slots) > kScratchBytes) {
        const uint64_t fixed = carve(*g, nullptr, 1, 1, 0, 0).bytes;
        *err = fixed > kScratchBytes
                   ? "mg_query_boxes_noalloc: the graph's global fallback table (" + std::to_string(fixed) +
                         " bytes for " + std::to_string(g->n_nodes) + " nodes) exceeds the " +
                         std::to_string(kScratchBytes) + "-byte scratch"
                   : "mg_query_boxes_noalloc: " + std::to_string(n) + " boxes exceed the " +
                         std::to_string(kScratchBytes) + "-byte scratch (at most " +
                         std::to_string((kScratchBytes - fixed) / 20) + " boxes on this graph)";
        return MG_ELIMIT;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    const Workspace w = carve(*g, sl->ptr, n, workers, 0, slots);
    // The scratch keeps the last call's contents, and every query leaves its part of it clean, so
    // it is cleared only where its layout changes. The layout it has is noted on the device as well:
    // once a call was captured, a graph's replay may be the last to have used it, which only the
    // device knows, and every call, replayed or not, looks there.
    const ScratchLayout layout = {{g->nseg, fallback_slots(*g), workers, slots + 1ull}};
    uint64_t *const have = reinterpret_cast<uint64_t *>(w.counters + kCountLayout);
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &status) != hipSuccess) (void)hipGetLastError();
    sl->captured = sl->captured || status != hipStreamCaptureStatusNone;
    if (sl->captured || std::memcmp(&layout, &sl->layout, sizeof(layout)) != 0) {
        hipLaunchKernelGGL(clear_kernel, dim3(1024), dim3(256), 0, s, clean_state(*g, w), have, layout);
        HIP_TRY(hipGetLastError());
        hipLaunchKernelGGL(stamp_kernel, dim3(1), dim3(64), 0, s, have, layout);
        HIP_TRY(hipGetLastError());
        sl->layout = layout;
    }
    const bool timing = g->dev.timing;
    g->dev.timing = false;  // no events are created on this path
    rc = query_in(g, boxes, n, out, nullptr, w, s, kQueryBatched, nullptr, err, nullptr);
    g->dev.timing = timing;
    if (rc) sl->layout = ScratchLayout{};  // looked at again by the next call
    return rc;
}

int dev_footprint(Graph *g, const uint32_t *boxes, uint32_t n, uint32_t *level_counts, uint32_t *cubes, uint32_t cap,
                  uint32_t *count, void *stream, std::string *err)
{
    DeviceGuard guard;
    int rc = check_device(g, err);
    if (rc) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const LevelTable lt = level_table(*g);
    hipLaunchKernelGGL(footprint_kernel, dim3(n), dim3(kBlock), 0, s, lt, boxes, n, g->dev.maps, level_counts, cubes,
                       cap, count);
    HIP_TRY(hipGetLastError());
    return MG_OK;
}

int dev_nnz_bound(Graph *g, const uint32_t *boxes, uint32_t n, uint32_t *bound, void *stream, std::string *err)
{
    DeviceGuard guard;
    int rc = check_device(g, err);
    if (rc) return rc;
    const LevelTable lt = level_table(*g);
    const uint32_t per = kBlock / 64;
    hipLaunchKernelGGL(nnz_bound_kernel, dim3((n + per - 1) / per), dim3(kBlock), 0, static_cast<hipStream_t>(stream),
                       lt, boxes, n, g->dev.maps, g->dev.mixlen, g->nseg, g->quant_bits == 0 ? 1u : 0u, bound);
    HIP_TRY(hipGetLastError());
    return MG_OK;
}

int dev_propagate_tf(Graph *g, const uint8_t *tf, uint32_t T, float *out, void *stream, std::string *err)
{
    DeviceGuard guard;
    int rc = check_device(g, err);
    if (rc) return rc;
    if (T > 65535) {
        *err = "at most 65535 transfer functions per call";
        return MG_ELIMIT;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    float4 *o = reinterpret_cast<float4 *>(out);
    // the timed region is the whole frame: sources, then every step
    rc = timing_begin(g, s, err);
    if (rc) return rc;
    const uint32_t tb = g->dev.cfg.tf_block;
    const uint32_t P = std::min<uint32_t>(g->dev.cfg.tf_planes ? g->dev.cfg.tf_planes : kTfPlanes, T);
    const uint32_t P2 = P >= 8 ? 8u : P >= 4 ? 4u : P >= 2 ? 2u : 1u;  // planes per thread
    using StepKernel = void (*)(const NodeTriple *, const SchedNode *, uint32_t, uint32_t, uint32_t, uint32_t,
                                const uchar4 *, uint32_t, float4 *);
    // the order: ranks (default) or the graph's deferred step schedule
    const bool ranks = g->dev.cfg.tf_schedule == 0;
    const std::vector<uint32_t> &ptr = ranks ? g->rank_ptr : g->step_ptr;
    auto pick = [&](bool first) -> StepKernel {
#define MG_TF_STEP(F, R)                                                                                       \
    (P2 == 8 ? tf_step_kernel<8, F, R> : P2 == 4 ? tf_step_kernel<4, F, R> : P2 == 2 ? tf_step_kernel<2, F, R> \
                                                                           : tf_step_kernel<1, F, R>)
        if (ranks) return first ? MG_TF_STEP(true, true) : MG_TF_STEP(false, true);
        return first ? MG_TF_STEP(true, false) : MG_TF_STEP(false, false);
#undef MG_TF_STEP
    };
    const uchar4 *tf4 = reinterpret_cast<const uchar4 *>(tf);
    const uint32_t D = g->depth;
    auto step_size = [&](uint32_t st) { return ptr[st + 1] - ptr[st]; };
    // the first launch takes steps 1 .. first_end - 1: in rank order ranks 1 and 2
    const uint32_t first_end = (ranks && D >= 2) ? 3u : 2u;
    // trailing small steps (two or more) go to the one-workgroup kernel
    uint32_t tail0 = D + 1;
    while (tail0 > first_end && D + 2 - tail0 <= kTfTailSteps && uint64_t(step_size(tail0 - 1)) * T <= kTfTailPairs)
        --tail0;
    if (D + 1 - tail0 < 2) tail0 = D + 1;
    // the first launch (possibly empty) with the sources' colours, then the other steps
    const uint32_t n1 = D >= 1 ? ptr[first_end] - ptr[1] : 0u;
    hipLaunchKernelGGL(pick(true), dim3((n1 + g->nseg + tb - 1) / tb, (T + P2 - 1) / P2), dim3(tb), 0, s,
                       g->dev.nodes, g->dev.sched, g->nseg, g->nseg + n1, g->n_nodes, T, tf4, g->nseg, o);
    HIP_TRY(hipGetLastError());
    for (uint32_t st = first_end; st < tail0; ++st) {
        const uint32_t lo = ptr[st], hi = ptr[st + 1];
        if (hi <= lo) continue;
        hipLaunchKernelGGL(pick(false), dim3((hi - lo + tb - 1) / tb, (T + P2 - 1) / P2), dim3(tb), 0, s,
                           g->dev.nodes, g->dev.sched, lo, hi, g->n_nodes, T, tf4, g->nseg, o);
        HIP_TRY(hipGetLastError());
    }
    if (tail0 <= D) {
        TfTail tail;
        tail.n_steps = D + 1 - tail0;
        for (uint32_t k = 0; k <= tail.n_steps; ++k) tail.lo[k] = ptr[tail0 + k];
        hipLaunchKernelGGL(ranks ? tf_tail_kernel<true> : tf_tail_kernel<false>, dim3(1), dim3(kTfTailBlock), 0, s,
                           g->dev.nodes, g->dev.sched, tail, g->n_nodes, T, o);
        HIP_TRY(hipGetLastError());
    }
    return timing_end(g, s, err);
}

int dev_set_launch(Graph *g, const mg_launch_cfg *cfg, std::string *err)
{
    if (cfg->chunk_small > 64) {
        *err = "mg_set_launch: chunk_small must be in [0, 64]";
        return MG_EINVAL;
    }
    if (!(cfg->block_small == 0 || cfg->block_small == 128 || cfg->block_small == 256) ||
        !(cfg->block_big == 0 || cfg->block_big == 256 || cfg->block_big == 512)) {
        *err = "mg_set_launch: block_small must be 0, 128 or 256 and block_big 0, 256 or 512";
        return MG_EINVAL;
    }
    for (uint32_t t : {cfg->table_big, cfg->table_small, cfg->table_retry})
        if (t != 0 && (t < 64 || t > 8192 || (t & (t - 1)) != 0)) {
            *err = "mg_set_launch: table sizes must be 0 or a power of two in [64, 8192]";
            return MG_EINVAL;
        }
    if (!(cfg->tf_planes == 0 || cfg->tf_planes == 1 || cfg->tf_planes == 2 || cfg->tf_planes == 4 ||
          cfg->tf_planes == 8) || cfg->tf_schedule > 1) {
        *err = "mg_set_launch: tf_planes must be 0, 1, 2, 4 or 8 and tf_schedule 0 or 1";
        return MG_EINVAL;
    }
    const uint32_t tb = cfg->tf_block;
    if (!valid_unroll(cfg->unroll_big) || !valid_unroll(cfg->unroll_small) || !valid_unroll(cfg->unroll_naive) ||
        !(tb == 64 || tb == 128 || tb == 256 || tb == 512 || tb == 1024)) {
        *err = "mg_set_launch: unroll must be 4, 8 or 16 and tf_block a power of two in [64, 1024]";
        return MG_EINVAL;
    }
    g->dev.cfg = *cfg;
    return MG_OK;
}

int dev_autotune(Graph *g, const uint32_t *boxes, uint32_t n, float *out, void *work, uint64_t bytes, uint32_t reps,
                 void *stream, mg_launch_cfg *chosen, std::string *err)
{
    DeviceGuard guard;
    int rc = check_device(g, err);
    if (rc) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipEvent_t e0, e1;
    HIP_TRY(hipEventCreate(&e0));
    HIP_TRY(hipEventCreate(&e1));
    const mg_launch_cfg saved = g->dev.cfg;
    const bool timing = g->dev.timing;
    g->dev.timing = false;
    auto time_variant = [&](int variant, float *best_ms) -> int {
        float best = 1e30f;
        for (uint32_t r = 0; r <= reps; ++r) {  // the first run warms up
            HIP_TRY(hipEventRecord(e0, s));
            int rc2 = dev_query(g, boxes, n, out, nullptr, work, bytes, stream, variant, nullptr, err);
            if (rc2) return rc2;
            HIP_TRY(hipEventRecord(e1, s));
            HIP_TRY(hipEventSynchronize(e1));
            float ms = 0;
            HIP_TRY(hipEventElapsedTime(&ms, e0, e1));
            if (r > 0) best = std::min(best, ms);
        }
        *best_ms = best;
        return MG_OK;
    };
    const uint32_t us[3] = {4, 8, 16};
    mg_launch_cfg best_cfg = saved;
    float best = 1e30f;
    // calls of few boxes read none of the tiers' settings: what was set for larger ones stays
    const bool tiers = n > kDirectMax;
    if (!tiers) rc = time_variant(kQueryBatched, &best);
    for (uint32_t ub : us)
        for (uint32_t usm : us) {
            if (rc || !tiers) break;
            g->dev.cfg.unroll_big = ub;
            g->dev.cfg.unroll_small = usm;
            float ms = 0;
            if ((rc = time_variant(kQueryBatched, &ms))) break;
            if (ms < best) best = ms, best_cfg.unroll_big = ub, best_cfg.unroll_small = usm;
        }
    // table sizes (LDS per workgroup, hence occupancy), one tier at a time
    const uint32_t tb[3] = {1024, 2048, 4096}, ts[3] = {256, 512, 1024};
    for (uint32_t bbg : {512u, 256u})
        for (uint32_t t : tb) {
            if (rc || (!tiers && bbg != 512u)) break;
            g->dev.cfg = best_cfg;
            g->dev.cfg.table_big = t;
            g->dev.cfg.block_big = tiers ? bbg : saved.block_big;
            float ms = 0;
            if ((rc = time_variant(kQueryBatched, &ms))) break;
            if (ms < best) best = ms, best_cfg.table_big = t, best_cfg.block_big = g->dev.cfg.block_big;
        }
    for (uint32_t bsm : {128u, 256u})
        for (uint32_t t : ts) {
            if (rc || !tiers) break;
            g->dev.cfg = best_cfg;
            g->dev.cfg.table_small = t;
            g->dev.cfg.block_small = bsm;
            float ms = 0;
            if ((rc = time_variant(kQueryBatched, &ms))) break;
            if (ms < best) best = ms, best_cfg.table_small = t, best_cfg.block_small = bsm;
        }
    for (uint32_t c : {0u, 2u, 4u}) {
        if (rc || !tiers) break;
        g->dev.cfg = best_cfg;
        g->dev.cfg.chunk_small = c;
        float ms = 0;
        if ((rc = time_variant(kQueryBatched, &ms))) break;
        if (ms < best) best = ms, best_cfg.chunk_small = c;
    }
    // shortest row summed from runs (where the graph keeps runs): both sides of the default
    for (uint32_t m : {8u, 32u, 64u}) {
        if (rc || !g->dev.runs_mask) break;
        g->dev.cfg = best_cfg;
        g->dev.cfg.run_min_row = m;
        float ms = 0;
        if ((rc = time_variant(kQueryBatched, &ms))) break;
        if (ms < best) best = ms, best_cfg.run_min_row = m;
    }
    float best_naive = 1e30f;
    for (uint32_t u : us) {
        if (rc) break;
        g->dev.cfg = best_cfg;
        g->dev.cfg.unroll_naive = u;
        float ms = 0;
        if ((rc = time_variant(kQueryNaive, &ms))) break;
        if (ms < best_naive) best_naive = ms, best_cfg.unroll_naive = u;
    }
    g->dev.timing = timing;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    g->dev.cfg = rc ? saved : best_cfg;
    if (!rc && chosen) *chosen = best_cfg;
    return rc;
}

int dev_timing_enable(Graph *g, int enable, std::string *err)
{
    (void)err;
    g->dev.timing = enable != 0;
    return MG_OK;
}

int dev_timing_read(Graph *g, double *ms, uint32_t *launches, std::string *err)
{
    DeviceGuard guard;
    int rc = check_device(g, err);
    if (rc) return rc;
    double tot = 0;
    DeviceState &d = g->dev;
    for (uint32_t i = 0; i < d.ev_used; ++i) {
        HIP_TRY(hipEventSynchronize(static_cast<hipEvent_t>(d.ev_stop[i])));
        float t = 0;
        HIP_TRY(hipEventElapsedTime(&t, static_cast<hipEvent_t>(d.ev_start[i]), static_cast<hipEvent_t>(d.ev_stop[i])));
        tot += t;
    }
    *ms = tot;
    *launches = d.ev_used;
    d.ev_used = 0;
    return MG_OK;
}

int dev_check_load_addresses(const uint32_t dims[3], uint32_t flags, const uint32_t *boxes, uint32_t n,
                              uint32_t unroll, uint64_t counts[4], std::string *err)
{
    return check_load_addresses(dims, (flags & 1u) != 0, (flags & 2u) != 0, (flags & 4u) != 0, flags >> 8, boxes, n,
                                unroll, counts, err);
}

}  // namespace mg
