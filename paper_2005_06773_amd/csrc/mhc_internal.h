// Internal device-side layouts shared by the host runtime and the kernels.
//
// A packed "scene image" (built on the host during ingest, copied to HBM in
// one transfer) holds these tables; the kernels read nothing else besides the
// pose buffer they produce and the result buffers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mhc {

enum Kind : int32_t { KIND_VEHICLE = 0, KIND_PEDESTRIAN = 1 };
enum Model : int32_t { MODEL_KINEMATIC = 0, MODEL_PED_ACCEL = 1, MODEL_ONE_TRACK = 2 };

// Shape class of an object pair: which overlap test applies and which side
// holds the rectangle or polygon.
// CLS_VV_PIP: two rectangles under the point-in-polygon test.
// CLS_GG, CLS_GG_PIP: two convex polygons (at least one a vehicle outline, a
//   rectangle otherwise by its corners), separating axes / point-in-polygon.
// CLS_GC, CLS_CG: polygon and circle (polygon first / second).
enum PairClass : int32_t {
    CLS_VV = 0, CLS_VP = 1, CLS_PV = 2, CLS_PP = 3, CLS_VV_PIP = 4,
    CLS_GG = 5, CLS_GG_PIP = 6, CLS_GC = 7, CLS_CG = 8, N_CLS = 9
};
// Families of test classes, each carried by its own collision-kernel
// instances (a family includes the ones before it).
enum ClassFamily : int32_t { FAM_PLAIN = 0, FAM_PIP = 1, FAM_POLY = 2 };
constexpr int class_family(int cls) { return cls >= CLS_GG ? FAM_POLY : (cls == CLS_VV_PIP ? FAM_PIP : FAM_PLAIN); }

constexpr int MAX_VERTICES = 8;

// Convex polygon of a vehicle in a polygon pair, body frame, CCW, as FP32
// test constants: vertices, unit outward edge normals and offsets (a point
// is inside iff nx*x + ny*y <= h on every edge), and for the circle test the
// edge vectors (vertex e to e+1) with 1 / |edge|^2. k is 4 or 8: a polygon
// of fewer vertices is padded with copies of vertex 0 and of edge 0, which
// change none of the tests.
struct alignas(16) DEdge {        // read as two 16-byte words
    float nx, ny, h, il;          // normal and offset, 1 / |edge|^2
    float vx, vy, ex, ey;         // first vertex, edge vector
};
struct DPoly {
    int32_t k, pad0, pad1, pad2;
    DEdge edge[MAX_VERTICES];
};

// Reading of the conditional-probability approximation (mhc.h MHC_RISK_*).
enum RiskModel : int32_t { RISK_EXCLUSIVE = 0, RISK_INDEPENDENT = 1 };

// One object of one scene. Offsets are global across all scenes of a launch.
struct DObj {
    int32_t kind, n_u, n_w, T;
    int32_t strip, H;             // traj_at's strip height
    int32_t local, n_scene_obj;   // index within its scene, object count of the scene
    int32_t risk, timeline;       // RiskModel of its scene; 1: time-resolved risk
    int32_t tl_w;                 // time-resolved: lanes per trajectory, the power of two >= n_scene_obj
    int32_t model;                // motion model (mhc.h MHC_MODEL_*)
    int64_t traj_off;             // index of trajectory 0 in the p / traj_crit arrays
    int64_t q_row;                // q index of (this object, i = 0, b = 0)
    int64_t pose_off;             // byte offset of the pose block [H][T], by position (traj_at)
    int64_t box_off;              // byte offset of the leaves' boxes [leaf][H] (x_min, x_max, y_min, y_max);
                                  // -1: none (the collision kernel tests every step)
    int64_t u_off, w_off, score_off;  // offsets (doubles) into the value array; score_off -1: uniform
    int64_t obj_out;              // index in the object_crit array
    // time-resolved risk (timeline scenes only)
    int64_t hist_off;             // slot sums [s][i][b < tl_w]: index of (s = 0, i = 0, b = 0)
    int64_t tl_traj;              // [s][i] criticality over time, and traj_crit_t (i, s): index of i = 0, s = 0
    int64_t tl_obj;               // crit_t index of (this object, s = 0)
    int64_t tl_att;               // attrib index of (this object, b = 0)
    float hl, hw;                 // half length and half width the shape's bounds are taken from, rounded up
    double x, y, heading, speed;  // position relative to the scene origin (scene_origin)
    double tau;
    double params[6];             // motion-model parameters
};

// One object pair (a < b within its scene). The collision kernel covers the
// T_a x T_b trajectory pairs as a grid of n_ig x n_jg "items": item (ig, jg) is
// the micro-tile of the positions ig*RI + r (r < RI) of a and jg*RJ + s
// (s < RJ) of b.
struct DPair {
    int32_t a, b;                 // global object indices
    int32_t cls, H;
    int32_t Ta, Tb;
    int32_t n_ig, n_jg;
    int64_t hit_off;              // first-hit entry of (i = 0, j = 0)
    int64_t pose_a, pose_b;       // byte offsets of the two pose blocks
    int64_t box_a, box_b;         // byte offsets of the two objects' leaf boxes, -1: none
    float la, wa, lb, wb;         // half length / half width of vehicles
    float rr;                     // squared test radius: r_Q^2 (rect-circle), (r_P + r_Q)^2 (circle-circle)
    int32_t tshift;               // time split S = 2^tshift (S <= H): a unit's steps go round S parts of the wave
    int32_t nui, nuj;             // grid of the pair's units
    int32_t unit_rs, unit_cs;     // log2 of a unit's positions of a and of b
    int32_t block_ur, block_ucs;  // units of a block: block_ur rows by 2^block_ucs columns
    int32_t nbi, nbj;             // grid of its blocks
    int32_t nsj;                  // strips of a block row
    int32_t step_i, step_j;       // strip_at's order of them
    int32_t poly_a, poly_b;       // DPoly of a and of b (polygon classes), else -1
    int32_t bshift;               // unit shape: (E >> bshift) item rows x 2^bshift item columns, E = 64 >> tshift
};

// A pair's items (ig, jg) form an n_ig x n_jg grid, cut into nui x nuj units of
// E / 2^bshift item rows and 2^bshift item columns, E = 64 / S with time split
// S. In a unit lane l takes item l % E and every S-th of the steps the unit has
// to test, those of part l / E, so S steps of an item run side by side in one
// wave. Items past the grid are idle lanes. Units are looked at a block at a
// time (block_ur x 2^block_ucs units, a square of positions), blocks in
// strips of a block row: strip of the pair's sequence number u, each strip
// once. Consecutive strips are step_i block rows (coprime to nbi) and step_j
// strips apart.
__host__ __device__ inline void strip_at(const DPair &pr, uint32_t u, int *bi, int *sj)
{
    const uint32_t q = u / (uint32_t)pr.nbi, ru = u - q * (uint32_t)pr.nbi;
    *bi = (int)(ru * (uint32_t)pr.step_i % (uint32_t)pr.nbi);
    *sj = (int)((q + ru * (uint32_t)pr.step_j) % (uint32_t)pr.nsj);
}

// A plan of n strips cut into `parts`: the strips before part `part`. No part is
// empty while there are as many strips.
inline int64_t strips_before_part(int64_t n, int part, int parts) { return n / parts * part + n % parts * part / parts; }

// The strip of its row of `grid` strips that workgroup x looks at: the
// workgroups are turned from row to row, so that none meets the same part of
// every pair.
__host__ __device__ inline int strip_in_row(int row, int x, int grid)
{
    const uint32_t c = ((uint32_t)(row & 0xFFFF) * 40503u) % (uint32_t)grid + (uint32_t)x;
    return (int)(c < (uint32_t)grid ? c : c - (uint32_t)grid);
}

// The trajectory (index k * n_w + l of the n_u x n_w control grid) at a
// position of its object. Positions run through strips of `strip` rows of the
// grid (accelerations or speeds), column by column, the next strip backwards:
// neighbouring positions are neighbours in both controls, so a leaf of them,
// and a group of leaves, keeps close together over the horizon.
__host__ __device__ inline void controls_at(int pos, int n_u, int n_w, int strip, int *k, int *l)
{
    const int b = pos / (strip * n_w);
    const int k0 = b * strip, left = n_u - k0, rows = left < strip ? left : strip;
    const int r = pos - k0 * n_w;
    const int c = r / rows;
    *k = k0 + (r - c * rows);
    *l = (b & 1) ? n_w - 1 - c : c;
}

__host__ __device__ inline int traj_at(int pos, int n_u, int n_w, int strip)
{
    int k, l;
    controls_at(pos, n_u, n_w, strip, &k, &l);
    return k * n_w + l;
}

constexpr int WG = 256;           // threads per workgroup, other kernels
constexpr int WAVE = 64;          // wavefront size
constexpr int MAX_TSHIFT = 3;     // time split of a collision unit: S <= 8
constexpr int K1_WG = 512;         // threads per workgroup of the trajectory kernel
constexpr int K2_WG = 512;         // and of the collision kernel
constexpr int K1_TPB = K1_WG / 64; // trajectories per trajectory workgroup (one wave each)
constexpr int LEAF = K1_TPB;      // trajectories of consecutive positions that share a box per step
// A pose with a coordinate beyond kBoxMax (or not finite) makes its leaf's box
// infinite; a step is left out of the tests where the boxes lie apart by more
// than kBoxSlack times their largest coordinate, and by more than kBoxLeast.
constexpr float kBoxMax = 1e15f, kBoxSlack = 0x1p-16f, kBoxLeast = 0x1p-50f;
// q sums are accumulated exactly as integers. EXCLUSIVE reading: p scaled by
// 2^62 and rounded (sum <= 1). INDEPENDENT reading: -log(1 - p), capped at 64,
// scaled by 2^56 and rounded; over one object's trajectories (sum p = 1) the
// sum stays below 66 * 2^56 < 2^63.
constexpr double kQScale = 4611686018427387904.0;        // 2^62
constexpr double kQInvScale = 2.168404344971009e-19;     // 2^-62
constexpr double kLScale = 72057594037927936.0;          // 2^56
constexpr double kLInvScale = 1.3877787807814457e-17;    // 2^-56
constexpr double kLCap = 64.0;                           // exp(-64) rounds 1 - q to 0

// A collision block holds at most BLOCK_LEAVES leaves, BLOCK_SIDE positions, of
// either object; a strip at most MAX_STRIP blocks of a block row. A collision
// workgroup takes K2_SLOTS blocks together, up to K2_UNITS listed units (a unit
// holds at least MIN_UNIT_PAIRS pairs, for two windows of 64 steps).
constexpr int BLOCK_LEAVES = 4, BLOCK_SIDE = BLOCK_LEAVES * LEAF, BLOCK_PAIRS = BLOCK_SIDE * BLOCK_SIDE;
constexpr int MAX_STRIP = 8, MIN_UNIT_PAIRS = 32, K2_SLOTS = K2_WG / WAVE;
constexpr int K2_UNITS = 2 * K2_SLOTS * BLOCK_PAIRS / MIN_UNIT_PAIRS;

// Micro-tile shape per class, selected by a kernel variant id.
struct TileShape {
    int ri, rj;
};
constexpr int N_VARIANTS = 4;
// variant -> shape per class {VV, VP, PV, PP, VV_PIP, GG, GG_PIP, GC, CG}.
// The shapes keep the loads per test low (25, 12, 6 and 58 VALU per rect-rect,
// rect-circle, circle-circle and point-in-polygon test, 100-500 for polygon
// pairs): a rectangle-circle tile pairs each rectangle pose (taken to its own
// frame) with 2 or 4 circles, and with a time split of 8 the tiles of variants 0
// and 1 make units of one pair of leaves. Variants 2 and 3 cut the work into
// smaller units.
// Polygon-polygon pairs always take one test per thread (their tests are
// long, and the kernel has one code path per padded vertex-count pair).
constexpr TileShape kTiles[N_VARIANTS][N_CLS] = {
    {{4, 2}, {2, 4}, {4, 2}, {4, 2}, {4, 2}, {1, 1}, {1, 1}, {4, 1}, {1, 4}},
    {{2, 4}, {4, 2}, {2, 4}, {2, 4}, {2, 4}, {1, 1}, {1, 1}, {2, 2}, {2, 2}},
    {{2, 2}, {2, 2}, {2, 2}, {2, 2}, {2, 2}, {1, 1}, {1, 1}, {4, 1}, {1, 4}},
    {{4, 1}, {1, 4}, {4, 1}, {2, 2}, {4, 1}, {1, 1}, {1, 1}, {1, 1}, {1, 1}},
};
static_assert(kTiles[0][CLS_GG].ri == 1 && kTiles[1][CLS_GG].ri == 1 && kTiles[2][CLS_GG].ri == 1 &&
                  kTiles[3][CLS_GG].ri == 1 && kTiles[0][CLS_GG].rj == 1 && kTiles[1][CLS_GG].rj == 1 &&
                  kTiles[2][CLS_GG].rj == 1 && kTiles[3][CLS_GG].rj == 1,
              "polygon-polygon tiles are 1 x 1");
static_assert(kTiles[0][CLS_GG_PIP].ri == 1 && kTiles[1][CLS_GG_PIP].ri == 1 && kTiles[2][CLS_GG_PIP].ri == 1 &&
                  kTiles[3][CLS_GG_PIP].ri == 1 && kTiles[0][CLS_GG_PIP].rj == 1 && kTiles[1][CLS_GG_PIP].rj == 1 &&
                  kTiles[2][CLS_GG_PIP].rj == 1 && kTiles[3][CLS_GG_PIP].rj == 1,
              "polygon-polygon tiles are 1 x 1");
constexpr bool tiles_fit()
{
    for (const auto &v : kTiles)
        for (const TileShape &t : v)
            if ((t.ri & (t.ri - 1)) || (t.rj & (t.rj - 1)) || t.ri > 8 || t.rj > 8)
                return false;
    return true;
}
static_assert(tiles_fit(), "tile sides are powers of two, at most 8");

// Launch entry points (kernels.hip).
struct Launch {
    const DObj *objs;
    const double *vals;
    const DPair *pairs;
    char *poses;
    unsigned long long *pfix;     // p * 2^62, per trajectory
    unsigned long long *qacc;     // integer q sums [n_q]
    const int64_t *strip0;        // [n_pairs+1] first strip of collision blocks of each pair
    const DPoly *polys;           // polygons of the polygon pairs
    double *p;
    int16_t *hits;
    double *q;
    double *traj_crit;
    double *obj_crit;
    int n_obj, n_pairs;
    int64_t n_strips, n_hits;     // strips of collision blocks, first-hit entries
    int strip_len;                // blocks of a strip
    int item_shift;               // log2 of the rounds of steps that a wave tests at a time
    int side_shift;               // log2 of the positions to a side of a block
    int k2_grid;                  // workgroups of the collision kernel
    int k1_x;                     // trajectory kernel grid x: blocks of a row
    int k1_nrows;                 // trajectory kernel grid y: rows (objects, or k1_rows entries)
    const int2 *k1_rows;          // per row: object and its first block; null when row = object
    int k3_x;                     // risk kernel grid x: 256-trajectory chunks of the largest object
    unsigned long long *done;     // per object: risk chunks finished (bits 56..63) and their
                                  // criticality sum in units of 2^-55 (bits 0..55)
    // time-resolved risk (null / 0 when no scene of the launch asks for it)
    int timeline;
    int k3t_x, k4t_y;             // time-resolved kernel grids: a wave of lanes of the largest object per workgroup; rows
    unsigned long long *hist;     // per-slot integer q sums
    double *att_w;                // attribution [b][i] per object
    double *ct_w;                 // criticality over time [s][i] per object
    double *crit_t, *traj_crit_t, *attrib, *traj_attrib;
    int collide_parts;            // parts of the collision plan (0: launch all of it)
    int part_lo, part_hi;         // of them, those that one launch takes together
    int clear_hits;               // collide writes -1 over the first hits first (no trajgen in this call does)
    int one_track;                // some object follows the one-track model (heavier trajectory kernel)
    int variant;
    int family;                   // ClassFamily covering every pair of the launch
};

// trajgen also writes -1 (no collision) over the first hits, of which collide
// stores the colliding pairs' only
hipError_t launch_trajgen(const Launch &L, hipStream_t s);
hipError_t launch_collide(const Launch &L, hipStream_t s);
// risk: the time-resolved kernels (timeline launches) and the risk kernel
hipError_t launch_risk(const Launch &L, hipStream_t s);
// Bytes of the allocation-free entry point's device array (mhc.h
// MHC_NOALLOC_MAX_BYTES) and the most GPUs whose copy of it is looked up.
constexpr size_t kNoallocBytes = size_t(64) << 20;
constexpr int kMaxDevices = 64;
// This GPU's address of that array (the device must be current on the
// calling thread); looked up once per device, then cached.
hipError_t noalloc_scratch_address(int device, char **out);
// resident workgroups (or their waves) per CU of the collision kernel for a
// variant, class family, with or without the per-slot sums
int collide_blocks_per_cu(int variant, int family, bool timeline, bool waves);

}  // namespace mhc
