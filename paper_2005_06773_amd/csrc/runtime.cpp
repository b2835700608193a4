// Host runtime behind the C ABI: scene ingest (validation, pair list, work
// list), packing of the scene image, device memory, launches, and the plain,
// asynchronous, plan and batched entry points.
#include "runtime.h"

#include <algorithm>
#include <functional>
#include <queue>
#include <cmath>
#include <numeric>
#include <cstdio>
#include <cstdint>
#include <climits>
#include <cstring>
#include <string>
#include <vector>

namespace mhc {

static size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

int pair_class(int ka, int kb, int overlap, bool outline_a, bool outline_b)
{
    if (outline_a || outline_b) {
        // a polygon on either side: vehicles are polygons (rectangles by their corners)
        if (ka == KIND_VEHICLE && kb == KIND_VEHICLE) return overlap == MHC_OVERLAP_PIP ? CLS_GG_PIP : CLS_GG;
        if (ka == KIND_VEHICLE) return CLS_GC;
        return CLS_CG;
    }
    if (overlap == MHC_OVERLAP_PIP) return CLS_VV_PIP;  // validated: vehicles only
    if (ka == KIND_VEHICLE && kb == KIND_VEHICLE) return CLS_VV;
    if (ka == KIND_VEHICLE) return CLS_VP;
    if (kb == KIND_VEHICLE) return CLS_PV;
    return CLS_PP;
}

bool scene_has_outline(const mhc_scene *s)
{
    for (int a = 0; a < s->n_objects; ++a)
        if (s->objects[a].n_vertices > 0) return true;
    return false;
}

int scene_family(const mhc_scene *s)
{
    if (scene_has_outline(s)) return FAM_POLY;
    return s->overlap == MHC_OVERLAP_PIP ? FAM_PIP : FAM_PLAIN;
}

// Padded vertex count of an object's polygon in a polygon pair (4 for a
// rectangle, 4 or 8 for an outline).
static int padded_vertices(int n) { return n <= 4 ? 4 : MAX_VERTICES; }
// Below this many collision units per resident wave, units are split in time
// (up to S = 8 steps of an item side by side in a wave): units of 8 x 8 pairs,
// one pair of leaves, whose boxes separate more steps than those of the 32 x 16
// pairs of an unsplit unit. Split or not (collision kernel): 383 or 467 us on
// the 64-scene batch (85 unsplit units a wave), 319 or 329 us on the stress
// scene (260). A GPU partition of few waves was not measured and keeps the
// split to plans of few units.
static double split_below_units_per_wave(int max_waves) { return max_waves < 1024 ? 16.0 : 1000.0; }

// How many blocks a plan should have per resident wave: the largest side of a
// block (8, 16 or 32 positions) that still gives as many is taken. Larger
// blocks take fewer looks, smaller ones spread the pairs that meet over more
// workgroups. Collision kernel on the 11-object scene: 13 us with half a block
// a wave (sides of 32), 17 with one (16: a second round of looks); octagons,
// whose tests take 15 times as long, 39 us (mean of four scenes) with two blocks
// a wave (sides of 16), 54 with eight (sides of 8). Sides of 8, whose blocks
// hold one pair of leaves, pay only while no wave looks twice, except for
// outlines: plans of sides of 8 and of 16, step of 16 objects of 49 trajectories
// (0.96 blocks of side 8 a wave) 21 and 25 us, of 12 of 81 (1.2) 21 and 17, of 9
// of 121 (1.5) 24 and 19; nine vehicles with octagons 45 and 95.
static double blocks_per_wave(int family) { return family == FAM_POLY ? 2.0 : 0.5; }

// The strip height of traj_at for an n_u x n_w grid: a leaf's positions cover
// about as large a share of either control's range.
static int strip_height(int n_u, int n_w)
{
    const int h = (int)std::lround(std::sqrt((double)LEAF * n_u / n_w));
    return std::min(std::max(h, 1), n_u);
}

// Collision units of a pair with time split 2^tshift (E = 64 >> tshift items a
// unit) in blocks of E >> bs item rows by 2^bs item columns.
static int64_t pair_units(const DPair &pr, int tshift, int bs, int *nui = nullptr, int *nuj = nullptr)
{
    const int rows = (WAVE >> tshift) >> bs, cols = 1 << bs;
    const int bi = (pr.n_ig + rows - 1) / rows, bj = (pr.n_jg + cols - 1) / cols;
    if (nui) *nui = bi;
    if (nuj) *nuj = bj;
    return (int64_t)bi * bj;
}

// Unit shape of a pair: bs of the block whose positions (ri and rj to an item
// row and column) have the smallest perimeter, so that few leaves meet it,
// among those that need at most a quarter more units than the fewest.
static int unit_shape(const DPair &pr, int tshift, const TileShape &ts)
{
    int64_t fewest = INT64_MAX;
    const int top = 6 - tshift;
    auto fits = [&](int bs) {
        return ((WAVE >> tshift) >> bs) * ts.ri <= BLOCK_SIDE && (1 << bs) * ts.rj <= BLOCK_SIDE;
    };
    for (int bs = 0; bs <= top; ++bs)
        if (fits(bs)) fewest = std::min(fewest, pair_units(pr, tshift, bs));
    int best = -1, best_side = 0;
    for (int bs = 0; bs <= top; ++bs) {
        if (!fits(bs) || pair_units(pr, tshift, bs) * 4 > fewest * 5) continue;
        const int side = ((WAVE >> tshift) >> bs) * ts.ri + (1 << bs) * ts.rj;
        if (best < 0 || side < best_side) {
            best = bs;
            best_side = side;
        }
    }
    return best;
}

// A step through n block rows (or columns) that is coprime to n, about 0.38 n.
static int coprime_step(int n)
{
    if (n <= 1) return 0;
    int s = std::max(1, (int)std::lround(0.382 * n));
    while (std::gcd(s, n) != 1) ++s;
    return s % n;
}

// Steps per part of a unit with time split 2^tshift: ceil(H / S).
static int split_chunk(int H, int tshift) { return (H + (1 << tshift) - 1) >> tshift; }

// A split fits a horizon when every part has a step and a walk through all
// steps leaves at most an eighth of H idle (S * ceil(H / S) - H).
static bool split_fits(int H, int tshift)
{
    const int S = 1 << tshift;
    return S <= H && 8 * (S * split_chunk(H, tshift) - H) <= H;
}

static bool finite(double v) { return std::isfinite(v); }

// ---------------------------------------------------------------------------
// Ingest: validation. Every rule here is checked before anything is launched.
// ---------------------------------------------------------------------------

// A vehicle outline: finite, strictly convex and counter-clockwise (every
// turn to the left), each interior angle at least 45 degrees (so that a
// vertex outside another polygon by more than the test tolerance is outside
// one of its edge lines by a comparable distance).
bool outline_ok(int k, const double *v)
{
    for (int e = 0; e < 2 * k; ++e)
        if (!finite(v[e])) return false;
    const double cos45 = std::sqrt(0.5);
    for (int e = 0; e < k; ++e) {
        const int p = (e + k - 1) % k, q = (e + 1) % k;
        const double ax = v[2 * e] - v[2 * p], ay = v[2 * e + 1] - v[2 * p + 1];   // incoming edge
        const double bx = v[2 * q] - v[2 * e], by = v[2 * q + 1] - v[2 * e + 1];   // outgoing edge
        if (!(ax * by - ay * bx > 0.0)) return false;                              // left turn
        // interior angle between -a and b
        const double la = std::hypot(ax, ay), lb = std::hypot(bx, by);
        if (!(la > 0.0) || !(lb > 0.0)) return false;
        const double cosint = (-ax * bx - ay * by) / (la * lb);
        if (cosint > cos45) return false;
    }
    return true;
}
bool validate_scene(const mhc_scene *s, std::string &err, int scene_index)
{
    char buf[256];
    auto fail = [&](const char *fmt, int a) {
        if (scene_index >= 0) {
            char b2[200];
            snprintf(b2, sizeof b2, fmt, a);
            snprintf(buf, sizeof buf, "scene %d: %s", scene_index, b2);
        } else {
            snprintf(buf, sizeof buf, fmt, a);
        }
        err = buf;
        return false;
    };
    if (!s) return fail("scene is NULL%.0d", 0);
    if (s->n_objects < 2) return fail("n_objects must be >= 2 (got %d)", s->n_objects);
    if (s->n_objects > kMaxObjects) return fail("n_objects must be <= %d", kMaxObjects);
    if (!s->objects) return fail("objects is NULL%.0d", 0);
    if (s->horizon < 1 || s->horizon > 32767) return fail("horizon must be in [1, 32767] (got %d)", s->horizon);
    if (!finite(s->dt) || !(s->dt > 0.0)) return fail("dt must be finite and > 0%.0d", 0);
    if (s->pairs != MHC_PAIRS_ALL && s->pairs != MHC_PAIRS_EGO) return fail("pairs must be 0 or 1 (got %d)", s->pairs);
    if (s->overlap != MHC_OVERLAP_EXACT && s->overlap != MHC_OVERLAP_PIP)
        return fail("overlap must be 0 or 1 (got %d)", s->overlap);
    if (s->risk != MHC_RISK_EXCLUSIVE && s->risk != MHC_RISK_INDEPENDENT)
        return fail("risk must be 0 or 1 (got %d)", s->risk);
    if (s->timeline != 0 && s->timeline != 1) return fail("timeline must be 0 or 1 (got %d)", s->timeline);
    if (s->timeline && s->n_objects > kMaxTimelineObjects)
        return fail("a time-resolved scene has at most %d objects", kMaxTimelineObjects);
    for (int a = 0; a < s->n_objects; ++a) {
        const mhc_object &o = s->objects[a];
        if (o.kind != MHC_VEHICLE && o.kind != MHC_PEDESTRIAN) return fail("object %d: kind must be 0 or 1", a);
        if (!finite(o.x) || !finite(o.y) || !finite(o.heading) || !finite(o.speed))
            return fail("object %d: state must be finite", a);
        if (!(o.speed >= 0.0)) return fail("object %d: speed must be >= 0", a);
        if (o.model != MHC_MODEL_KINEMATIC && o.model != MHC_MODEL_PED_ACCEL && o.model != MHC_MODEL_ONE_TRACK)
            return fail("object %d: model must be 0, 1 or 2", a);
        if (o.model == MHC_MODEL_PED_ACCEL) {
            if (o.kind != MHC_PEDESTRIAN) return fail("object %d: the acceleration model is for pedestrians", a);
            if (!finite(o.params[0]) || !(o.params[0] > 0.0)) return fail("object %d: v_max must be finite and > 0", a);
        }
        if (o.model == MHC_MODEL_ONE_TRACK) {
            if (o.kind != MHC_VEHICLE) return fail("object %d: the one-track model is for vehicles", a);
            for (int k = 0; k < 6; ++k)
                if (!finite(o.params[k]) || !(o.params[k] > 0.0))
                    return fail("object %d: one-track parameters must be finite and > 0", a);
            if (o.params[3] * o.params[1] < o.params[2] * o.params[0])
                return fail("object %d: the one-track parameters must understeer (l_r c_r >= l_f c_f)", a);
        }
        if (o.n_vertices != 0) {
            if (o.kind != MHC_VEHICLE) return fail("object %d: only vehicles take an outline", a);
            if (o.n_vertices < 3 || o.n_vertices > MHC_MAX_VERTICES)
                return fail("object %d: an outline has 3 to 8 vertices", a);
            if (!o.vertices) return fail("object %d: outline vertices must not be NULL", a);
            if (!outline_ok(o.n_vertices, o.vertices))
                return fail("object %d: the outline must be finite, strictly convex, counter-clockwise, "
                            "with interior angles >= 45 degrees", a);
        } else if (o.kind == MHC_VEHICLE) {
            if (!finite(o.length) || !(o.length > 0.0) || !finite(o.width) || !(o.width > 0.0))
                return fail("object %d: vehicle length and width must be finite and > 0", a);
        } else {
            if (!finite(o.radius) || !(o.radius > 0.0)) return fail("object %d: pedestrian radius must be finite and > 0", a);
        }
        if (o.n_u < 1 || o.n_w < 1) return fail("object %d: n_u and n_w must be >= 1", a);
        if ((int64_t)o.n_u * o.n_w > kMaxTraj) return fail("object %d: n_u*n_w exceeds the trajectory limit", a);
        if ((int64_t)o.n_u * o.n_w * s->horizon > kMaxPosesPerObject)
            return fail("object %d: horizon * n_u * n_w exceeds the per-object pose limit (2^27)", a);
        if (!o.u || !o.w) return fail("object %d: control grids u and w must not be NULL", a);
        for (int k = 0; k < o.n_u; ++k)
            if (!finite(o.u[k])) return fail("object %d: control grid u must be finite", a);
        for (int k = 0; k < o.n_w; ++k)
            if (!finite(o.w[k])) return fail("object %d: control grid w must be finite", a);
        if (o.score) {
            double l1 = 0.0;
            const int T = o.n_u * o.n_w;
            for (int k = 0; k < T; ++k) {
                if (!finite(o.score[k]) || !(o.score[k] >= 0.0)) return fail("object %d: scores must be finite and >= 0", a);
                l1 += o.score[k];
            }
            if (!(l1 > 0.0) || !finite(l1)) return fail("object %d: scores must have a positive finite sum", a);
        }
    }
    if (s->objects[0].kind != MHC_VEHICLE && s->pairs == MHC_PAIRS_EGO)
        return fail("EGO pair mode needs object 0 to be a vehicle%.0d", 0);
    if (s->overlap == MHC_OVERLAP_PIP)
        for (int a = 0; a < s->n_objects; ++a)
            if (s->objects[a].kind != MHC_VEHICLE)
                return fail("object %d: the point-in-polygon overlap test needs every object to be a vehicle", a);
    return true;
}

bool validate_outputs(const mhc_scene *s, const mhc_result *r, std::string &err, int scene_index)
{
    if (!r || s->timeline) return true;
    if (r->crit_t || r->traj_crit_t || r->attrib || r->traj_attrib) {
        err = (scene_index >= 0 ? "scene " + std::to_string(scene_index) + ": " : std::string()) +
              "crit_t, traj_crit_t, attrib and traj_attrib need a scene with timeline = 1";
        return false;
    }
    return true;
}

// ---------------------------------------------------------------------------
// Ingest: pair list, work list and the packed scene image.
// ---------------------------------------------------------------------------
static void pair_list(const mhc_scene *s, std::vector<std::pair<int, int>> &out)
{
    out.clear();
    for (int a = 0; a < s->n_objects; ++a)
        for (int b = a + 1; b < s->n_objects; ++b)
            if (s->pairs == MHC_PAIRS_ALL || a == 0) out.emplace_back(a, b);
}

// Empties a layout for the next build. Its tables keep their storage: a
// batch's tables span megabytes, and freshly allocated ones would be paged in
// again on every launch (about half of the host time of a 64-scene launch).
static void reset_layout(Layout &L)
{
    Layout fresh;
    auto keep = [](auto &to, auto &from) {
        to = std::move(from);
        to.clear();
    };
    keep(fresh.objs, L.objs);
    keep(fresh.vals, L.vals);
    keep(fresh.pairs, L.pairs);
    keep(fresh.strip0, L.strip0);
    keep(fresh.polys, L.polys);
    keep(fresh.sc, L.sc);
    keep(fresh.k1_rows, L.k1_rows);
    L = std::move(fresh);
}

static void build_layout_once(const mhc_scene *scenes, int n_scenes, int variant, int max_waves, Layout &L,
                              bool with_hits, bool boxes);

void build_layout(const mhc_scene *scenes, int n_scenes, int variant, int max_waves, Layout &L, bool with_hits,
                  size_t max_bytes)
{
    build_layout_once(scenes, n_scenes, variant, max_waves, L, with_hits, true);
    if (L.total_bytes > max_bytes) build_layout_once(scenes, n_scenes, variant, max_waves, L, with_hits, false);
}

static void build_layout_once(const mhc_scene *scenes, int n_scenes, int variant, int max_waves, Layout &L,
                              bool with_hits, bool boxes)
{
    reset_layout(L);
    L.variant = variant;
    L.with_hits = with_hits;
    L.boxes = boxes;
    std::vector<std::pair<int, int>> plist;
    for (int k = 0; k < n_scenes; ++k) {
        const mhc_scene &s = scenes[k];
        const int n = s.n_objects;
        SceneExt ext{};
        ext.n_obj = n;
        ext.H = s.horizon;
        ext.obj0 = L.n_obj;
        ext.traj0 = L.n_traj;
        ext.hit0 = L.n_hits;
        ext.q0 = L.n_q;
        ext.timeline = s.timeline != 0;
        ext.tl_obj0 = L.n_tl_obj;
        ext.tl_traj0 = L.n_tl_traj;
        ext.tl_att0 = L.n_tl_att;
        L.timeline |= ext.timeline;
        const int obj_base = (int)L.objs.size();
        int64_t toff = 0;
        for (int a = 0; a < n; ++a) {
            const mhc_object &o = s.objects[a];
            DObj d{};
            d.kind = o.kind;
            d.n_u = o.n_u;
            d.n_w = o.n_w;
            d.T = o.n_u * o.n_w;
            d.H = s.horizon;
            d.local = a;
            d.n_scene_obj = n;
            d.risk = s.risk;
            d.timeline = s.timeline;
            d.model = o.model;
            L.one_track |= o.model == MHC_MODEL_ONE_TRACK;
            if (s.timeline) {
                int W = 1;
                while (W < n) W <<= 1;
                d.tl_w = W;
                d.hist_off = L.n_hist;
                d.tl_traj = L.n_tl_traj;
                d.tl_obj = L.n_tl_obj;
                d.tl_att = L.n_tl_att;
                L.n_hist += (int64_t)W * s.horizon * d.T;
                L.k3t_x = std::max<int64_t>(L.k3t_x, ((int64_t)d.T * W + WAVE - 1) / WAVE);
                L.k4t_y = std::max(L.k4t_y, s.horizon + n);
                L.n_tl_traj += (int64_t)s.horizon * d.T;
                L.n_tl_obj += s.horizon;
                L.n_tl_att += n;
            }
            d.traj_off = L.n_traj + toff;
            d.q_row = L.n_q + toff * n;
            d.pose_off = (int64_t)L.pose_bytes;
            L.pose_bytes += align256((size_t)s.horizon * d.T * (o.kind == MHC_VEHICLE ? 16 : 8));
            d.strip = strip_height(o.n_u, o.n_w);
            d.box_off = -1;
            if (boxes) {
                d.box_off = (int64_t)L.pose_bytes;
                L.pose_bytes += align256((size_t)s.horizon * ((d.T + LEAF - 1) / LEAF) * sizeof(float4));
            }
            d.u_off = (int64_t)L.vals.size();
            d.w_off = d.u_off + o.n_u;
            d.score_off = o.score ? d.w_off + o.n_w : -1;
            L.vals.resize(L.vals.size() + o.n_u + o.n_w + (o.score ? d.T : 0));
            d.obj_out = L.n_obj + a;
            L.k3_x = std::max(L.k3_x, (d.T + WG - 1) / WG);
            L.objs.push_back(d);
            toff += d.T;
        }
        // polygons: with an outline anywhere in the scene, every vehicle of the
        // scene gets one (its rectangle's corners if it has no outline)
        std::vector<int32_t> poly_of(n, -1);
        if (scene_has_outline(&s))
            for (int a = 0; a < n; ++a)
                if (s.objects[a].kind == MHC_VEHICLE) {
                    poly_of[a] = (int32_t)L.polys.size();
                    L.polys.push_back(DPoly{});
                }
        pair_list(&s, plist);
        int64_t hoff = 0;
        for (auto &ab : plist) {
            const int a = ab.first, b = ab.second;
            const mhc_object &oa = s.objects[a], &ob = s.objects[b];
            DPair pr{};
            pr.a = obj_base + a;
            pr.b = obj_base + b;
            pr.cls = pair_class(oa.kind, ob.kind, s.overlap, oa.n_vertices > 0, ob.n_vertices > 0);
            pr.poly_a = poly_of[a];
            pr.poly_b = poly_of[b];
            L.family = std::max(L.family, class_family(pr.cls));
            pr.H = s.horizon;
            pr.Ta = oa.n_u * oa.n_w;
            pr.Tb = ob.n_u * ob.n_w;
            const TileShape ts = kTiles[variant][pr.cls];
            pr.n_ig = (pr.Ta + ts.ri - 1) / ts.ri;
            pr.n_jg = (pr.Tb + ts.rj - 1) / ts.rj;
            pr.hit_off = L.n_hits + hoff;
            const DObj &da = L.objs[obj_base + a], &db = L.objs[obj_base + b];
            pr.pose_a = da.pose_off;
            pr.pose_b = db.pose_off;
            pr.box_a = da.box_off;
            pr.box_b = db.box_off;
            L.pairs.push_back(pr);
            hoff += (int64_t)pr.Ta * pr.Tb;
            ext.checks += (int64_t)pr.Ta * pr.Tb * s.horizon;
        }
        ext.n_traj = toff;
        ext.n_hits = hoff;
        ext.n_pairs = (int64_t)plist.size();
        L.sc.push_back(ext);
        L.n_traj += toff;
        L.n_hits += hoff;
        L.n_q += toff * n;
        L.n_obj += n;
        L.n_checks += ext.checks;
    }
    // Trajectory kernel grid. An object takes a normalisation block and a
    // block per K1_TPB trajectories. With objects of one size the grid is
    // (blocks, objects); otherwise rows of as many blocks as the smallest
    // object has, each row a stretch of one object's blocks (the row table),
    // so that no workgroup of a large object's extent is launched for a small
    // one (empty workgroups cost dispatch time).
    {
        int bmin = INT_MAX, bmax = 0;
        for (const DObj &d : L.objs) {
            const int b = (d.T + K1_TPB - 1) / K1_TPB + 1;
            bmin = std::min(bmin, b);
            bmax = std::max(bmax, b);
        }
        L.k1_x = bmax;
        L.k1_nrows = (int)L.objs.size();
        if (bmin < bmax) {
            int B = bmin;
            auto rows_of = [&](int w) {
                int64_t r = 0;
                for (const DObj &d : L.objs) r += ((d.T + K1_TPB - 1) / K1_TPB + 1 + w - 1) / w;
                return r;
            };
            while (rows_of(B) > 65535) B *= 2;  // the grid's y extent
            for (int a = 0; a < (int)L.objs.size(); ++a) {
                const int b = (L.objs[a].T + K1_TPB - 1) / K1_TPB + 1;
                for (int s0 = 0; s0 < b; s0 += B) {
                    L.k1_rows.push_back(a);
                    L.k1_rows.push_back(s0);
                }
            }
            L.k1_x = B;
            L.k1_nrows = (int)(L.k1_rows.size() / 2);
        }
    }
    // Time split. With few units for the resident waves, S steps of an item
    // run side by side in a wave (64/S items per unit). S is the smallest of
    // 1, 2, 4, 8 that gives enough units (the largest for the size bound,
    // max_waves = 0), lowered per pair until it fits the horizon (split_fits).
    int want = MAX_TSHIFT;
    if (max_waves > 0) {
        for (want = 0; want < MAX_TSHIFT; ++want) {
            int64_t u = 0;
            for (const DPair &pr : L.pairs) {
                const TileShape ts = kTiles[variant][pr.cls];
                u += pair_units(pr, want, unit_shape(pr, want, ts));
            }
            if ((double)u >= split_below_units_per_wave(max_waves) * max_waves) break;
        }
    }
    L.n_units = 0;
    for (DPair &pr : L.pairs) {
        int sh = want;
        const TileShape ts = kTiles[variant][pr.cls];
        while (sh > 0 && (!split_fits(pr.H, sh) || (WAVE >> sh) * ts.ri * ts.rj < MIN_UNIT_PAIRS)) --sh;
        pr.tshift = sh;
        pr.bshift = unit_shape(pr, sh, kTiles[variant][pr.cls]);
        L.n_units += pair_units(pr, sh, pr.bshift, &pr.nui, &pr.nuj);
    }
    // Collision plan: the pairs' strips of blocks one after another, looked at
    // in rounds by as many waves as the GPU holds (k2_collide).
    int64_t n_blocks = 0;
    auto unit_rows = [&](const DPair &pr) { return ((WAVE >> pr.tshift) >> pr.bshift) * kTiles[variant][pr.cls].ri; };
    auto unit_cols = [&](const DPair &pr) { return (1 << pr.bshift) * kTiles[variant][pr.cls].rj; };
    int least = LEAF;   // no unit is larger than a block
    for (const DPair &pr : L.pairs) least = std::max({least, unit_rows(pr), unit_cols(pr)});
    auto cut = [&](int side) {
        n_blocks = 0;
        L.side_shift = 0;
        while ((1 << L.side_shift) < side) ++L.side_shift;
        for (DPair &pr : L.pairs) {
            const int rows = unit_rows(pr), cols = unit_cols(pr);
            for (pr.unit_rs = 0; (1 << pr.unit_rs) < rows;) ++pr.unit_rs;
            for (pr.unit_cs = 0; (1 << pr.unit_cs) < cols;) ++pr.unit_cs;
            pr.block_ur = side / rows;
            pr.block_ucs = L.side_shift - pr.unit_cs;
            pr.nbi = (pr.nui + pr.block_ur - 1) / pr.block_ur;
            pr.nbj = (pr.nuj + (1 << pr.block_ucs) - 1) >> pr.block_ucs;
            n_blocks += (int64_t)pr.nbi * pr.nbj;
        }
    };
    int side = BLOCK_SIDE;
    cut(side);
    while (side > least && (double)n_blocks < blocks_per_wave(L.family) * max_waves) cut(side /= 2);
    if (side == LEAF && least < 2 * LEAF && max_waves > 0 && n_blocks > max_waves && L.family != FAM_POLY)
        cut(side = 2 * LEAF);
    // Large plans: several blocks to a look, whose row's boxes are read once.
    // Neighbouring blocks meet together, so a strip is long only where a wave
    // still gets eight of them. Collision kernel with strips of three blocks
    // and of one: octagons 43 and 32 us (mean of four scenes); with two and
    // with four to eight a wave on the 64-scene batch: 380 and 338 us.
    L.strip_len = max_waves > 0 ? (int)std::max<int64_t>(1, std::min<int64_t>(MAX_STRIP, n_blocks / (8 * (int64_t)max_waves)))
                                : 1;
    int64_t n_strips = 0;
    L.strip0.clear();
    for (DPair &pr : L.pairs) {
        pr.nsj = (pr.nbj + L.strip_len - 1) / L.strip_len;
        pr.step_i = coprime_step(pr.nbi);
        pr.step_j = coprime_step(pr.nsj);
        L.strip0.push_back(n_strips);
        n_strips += (int64_t)pr.nbi * pr.nsj;
    }
    L.strip0.push_back(n_strips);
    // Rounds of S steps that a wave tests at a time: few where the waves of a
    // workgroup hardly fill (octagons 34 us with 2, 38 with 4), more where
    // there is work for all of them and an item's set-up counts (stress scene
    // 332 us with 4, 357 with 2; 64-scene batch 470 and 510). Without boxes
    // every step of every unit is tested: collision kernel on the stress scene
    // 21.2 ms with 4, 16.8 with 16; 30 pedestrians in a crowd 293 and 219 us.
    L.item_shift = !boxes ? 4 : L.strip_len > 1 ? 2 : 1;
    constexpr int kWaves = K2_WG / WAVE;
    // a strip a wave, but few strips on more workgroups, half of those that the
    // GPU holds (1.5 a CU) and all of them for outlines, whose tests are long:
    // what meets in a strip is tested by its workgroup's eight waves together.
    // Whole call on four octagon vehicles of up to 48 trajectories: 88 us with a
    // strip a wave, 66 on 170 workgroups. Step on one workgroup a CU and so: a
    // queue of 12 vehicles of 81 trajectories (2376 strips) 26 and 22 us, of six
    // 19 and 17, of six octagons of 49 (735 strips) 31 and 24; six octagons of
    // 81 crossing 22.6 and 21.8, twelve of 49 29 and 30. Without boxes everything
    // is tested, by all of them (11-object scene, 3520 strips: 67 us on 440, 55
    // on 768).
    const int held = max_waves / kWaves;
    const int64_t want_wg = std::max<int64_t>((n_strips + kWaves - 1) / kWaves,
                                              std::min<int64_t>(n_strips, !boxes || L.family == FAM_POLY ? held : held / 2));
    L.k2_grid = (int)std::min<int64_t>(want_wg, max_waves > 0 ? std::max(1, max_waves / kWaves) : INT_MAX);

    size_t off = 0;
    auto put = [&](size_t bytes) {
        size_t o = off;
        off = align256(off + bytes);
        return o;
    };
    // the tables fill_values rewrites come first, the collision plan (which
    // depends on the shapes only) last
    L.o_objs = put(L.objs.size() * sizeof(DObj));
    L.o_vals = put(L.vals.size() * sizeof(double));
    L.o_pairs = put(L.pairs.size() * sizeof(DPair));
    L.o_polys = put(L.polys.size() * sizeof(DPoly));
    L.value_bytes = off;
    L.o_strip0 = put(L.strip0.size() * sizeof(int64_t));
    L.o_k1rows = put(L.k1_rows.size() * sizeof(int32_t));
    L.image_bytes = off;
    L.o_poses = put(L.pose_bytes);
    L.o_pfix = put((size_t)L.n_traj * sizeof(unsigned long long));
    L.o_qacc = put((size_t)L.n_q * sizeof(unsigned long long));
    L.o_done = put((size_t)L.n_obj * sizeof(unsigned long long));
    // the outputs most calls ask for are neighbours, so they come down together
    L.o_p = put((size_t)L.n_traj * sizeof(double));
    L.o_tc = put((size_t)L.n_traj * sizeof(double));
    L.o_oc = put((size_t)L.n_obj * sizeof(double));
    L.o_q = put((size_t)L.n_q * sizeof(double));
    L.o_hits = put(with_hits ? (size_t)L.n_hits * sizeof(int16_t) : 0);
    const size_t tq = L.timeline ? (size_t)L.n_q : 0;
    L.o_hist = put((size_t)L.n_hist * sizeof(unsigned long long));
    L.o_attw = put(tq * sizeof(double));
    L.o_ctw = put((size_t)L.n_tl_traj * sizeof(double));
    L.o_ct = put((size_t)L.n_tl_obj * sizeof(double));
    L.o_tct = put((size_t)L.n_tl_traj * sizeof(double));
    L.o_at = put((size_t)L.n_tl_att * sizeof(double));
    L.o_tat = put(tq * sizeof(double));
    L.total_bytes = off;
    fill_values(scenes, n_scenes, L);
}

// The value part of a layout: states, control grids, scores and extents.
// Everything else in a layout depends only on the scene shapes.
// The test constants of a vehicle's polygon: its outline, or the corners of
// its rectangle, counter-clockwise in the body frame (FP64, then FP32).
static void fill_poly(const mhc_object &o, DPoly &g)
{
    double vx[MAX_VERTICES], vy[MAX_VERTICES];
    int k;
    if (o.n_vertices > 0) {
        k = o.n_vertices;
        for (int e = 0; e < k; ++e) {
            vx[e] = o.vertices[2 * e];
            vy[e] = o.vertices[2 * e + 1];
        }
    } else {
        const double l = o.length / 2.0, w = o.width / 2.0;
        k = 4;
        const double cx[4] = {l, l, -l, -l}, cy[4] = {-w, w, w, -w};
        for (int e = 0; e < 4; ++e) {
            vx[e] = cx[e];
            vy[e] = cy[e];
        }
    }
    g = DPoly{};
    g.k = padded_vertices(k);
    for (int e = 0; e < g.k; ++e) {
        DEdge &d = g.edge[e];
        if (e >= k) {  // padding: copies of vertex 0 and of edge 0
            d = g.edge[0];
            continue;
        }
        const int f = (e + 1) % k;
        const double ex = vx[f] - vx[e], ey = vy[f] - vy[e];
        const double len = std::hypot(ex, ey);
        const double nx = ey / len, ny = -ex / len;   // outward for a CCW polygon
        d.vx = (float)vx[e];
        d.vy = (float)vy[e];
        d.nx = (float)nx;
        d.ny = (float)ny;
        d.h = (float)(nx * vx[e] + ny * vy[e]);
        d.ex = (float)ex;
        d.ey = (float)ey;
        d.il = (float)(1.0 / (ex * ex + ey * ey));
    }
}

// The origin a scene's positions are taken relative to before the GPU sees
// them: the middle of the box of the initial positions, rounded to a multiple
// of kOriginGrid metres. The overlap tests are invariant under a shift of the
// whole scene, but their FP32 rounding grows with the coordinates; relative
// to this origin a scene far from (0, 0) is tested with the precision of one
// near it. The subtraction costs at most one FP64 rounding (1e-12 m at
// 10 km), and a scene whose box is centred within 128 m of (0, 0) keeps its
// coordinates unchanged.
static const double kOriginGrid = 256.0;

void scene_origin(const mhc_scene &s, double *ox, double *oy)
{
    double x0 = s.objects[0].x, x1 = x0, y0 = s.objects[0].y, y1 = y0;
    for (int a = 1; a < s.n_objects; ++a) {
        x0 = std::min(x0, s.objects[a].x);
        x1 = std::max(x1, s.objects[a].x);
        y0 = std::min(y0, s.objects[a].y);
        y1 = std::max(y1, s.objects[a].y);
    }
    *ox = kOriginGrid * std::nearbyint((x0 / 2.0 + x1 / 2.0) / kOriginGrid);
    *oy = kOriginGrid * std::nearbyint((y0 / 2.0 + y1 / 2.0) / kOriginGrid);
}

// Half length and half width (about the tracked position) of a rectangle
// around the object's shape, rounded up well above the FP32 rounding of the
// extents that the tests use.
static void half_extents(const mhc_object &o, float *hl, float *hw)
{
    double l = o.length / 2.0, w = o.width / 2.0;
    if (o.kind != MHC_VEHICLE) l = w = o.radius;
    if (o.n_vertices > 0) l = w = 0.0;
    for (int e = 0; e < o.n_vertices; ++e) {
        l = std::max(l, std::fabs(o.vertices[2 * e]));
        w = std::max(w, std::fabs(o.vertices[2 * e + 1]));
    }
    *hl = (float)(l * (1.0 + 1e-6));
    *hw = (float)(w * (1.0 + 1e-6));
}

void fill_values(const mhc_scene *scenes, int n_scenes, Layout &L)
{
    size_t oi = 0, pi = 0, gi = 0;
    std::vector<std::pair<int, int>> plist;
    for (int k = 0; k < n_scenes; ++k) {
        const mhc_scene &s = scenes[k];
        double ox, oy;
        scene_origin(s, &ox, &oy);
        for (int a = 0; a < s.n_objects; ++a, ++oi) {
            const mhc_object &o = s.objects[a];
            DObj &d = L.objs[oi];
            d.x = o.x - ox;
            d.y = o.y - oy;
            d.heading = o.heading;
            d.speed = o.speed;
            d.tau = s.dt;
            half_extents(o, &d.hl, &d.hw);
            for (int k = 0; k < 6; ++k) d.params[k] = o.params[k];
            std::copy(o.u, o.u + o.n_u, L.vals.begin() + d.u_off);
            std::copy(o.w, o.w + o.n_w, L.vals.begin() + d.w_off);
            if (o.score) std::copy(o.score, o.score + d.T, L.vals.begin() + d.score_off);
        }
        if (scene_has_outline(&s))
            for (int a = 0; a < s.n_objects; ++a)
                if (s.objects[a].kind == MHC_VEHICLE) fill_poly(s.objects[a], L.polys[gi++]);
        pair_list(&s, plist);
        for (auto &ab : plist) {
            const mhc_object &oa = s.objects[ab.first], &ob = s.objects[ab.second];
            DPair &pr = L.pairs[pi++];
            pr.la = (float)(oa.length / 2.0);
            pr.wa = (float)(oa.width / 2.0);
            pr.lb = (float)(ob.length / 2.0);
            pr.wb = (float)(ob.width / 2.0);
            pr.rr = 0.0f;
            if (pr.cls == CLS_VP || pr.cls == CLS_GC) pr.rr = (float)(ob.radius * ob.radius);
            else if (pr.cls == CLS_PV || pr.cls == CLS_CG) pr.rr = (float)(oa.radius * oa.radius);
            else if (pr.cls == CLS_PP) pr.rr = (float)((oa.radius + ob.radius) * (oa.radius + ob.radius));
        }
    }
}

void pack_image(const Layout &L, char *dst, bool values_only)
{
    // each table, then zeros up to the next one (the image is written once)
    auto cp = [&](size_t o, const void *src, size_t bytes, size_t next) {
        if (bytes) std::memcpy(dst + o, src, bytes);
        std::memset(dst + o + bytes, 0, next - o - bytes);
    };
    cp(L.o_objs, L.objs.data(), L.objs.size() * sizeof(DObj), L.o_vals);
    cp(L.o_vals, L.vals.data(), L.vals.size() * sizeof(double), L.o_pairs);
    cp(L.o_pairs, L.pairs.data(), L.pairs.size() * sizeof(DPair), L.o_polys);
    cp(L.o_polys, L.polys.data(), L.polys.size() * sizeof(DPoly), L.value_bytes);
    if (values_only) return;
    cp(L.o_strip0, L.strip0.data(), L.strip0.size() * sizeof(int64_t), L.o_k1rows);
    cp(L.o_k1rows, L.k1_rows.data(), L.k1_rows.size() * sizeof(int32_t), L.image_bytes);
}

Launch make_launch(const Layout &L, char *base, const mhc_result *dev_out, bool keep_hits, int n_cu)
{
    Launch X{};
    X.objs = reinterpret_cast<const DObj *>(base + L.o_objs);
    X.vals = reinterpret_cast<const double *>(base + L.o_vals);
    X.pairs = reinterpret_cast<const DPair *>(base + L.o_pairs);
    X.poses = base + L.o_poses;
    X.pfix = reinterpret_cast<unsigned long long *>(base + L.o_pfix);
    X.qacc = reinterpret_cast<unsigned long long *>(base + L.o_qacc);
    X.done = reinterpret_cast<unsigned long long *>(base + L.o_done);
    X.strip0 = reinterpret_cast<const int64_t *>(base + L.o_strip0);
    X.k1_rows = L.k1_rows.empty() ? nullptr : reinterpret_cast<const int2 *>(base + L.o_k1rows);
    X.k1_nrows = L.k1_nrows;
    X.polys = reinterpret_cast<const DPoly *>(base + L.o_polys);
    X.p = reinterpret_cast<double *>(base + L.o_p);
    X.hits = reinterpret_cast<int16_t *>(base + L.o_hits);
    X.q = reinterpret_cast<double *>(base + L.o_q);
    X.traj_crit = reinterpret_cast<double *>(base + L.o_tc);
    X.obj_crit = reinterpret_cast<double *>(base + L.o_oc);
    if (!keep_hits || !L.with_hits) X.hits = nullptr;
    X.timeline = L.timeline ? 1 : 0;
    X.one_track = L.one_track ? 1 : 0;
    if (L.timeline) {
        X.hist = reinterpret_cast<unsigned long long *>(base + L.o_hist);
        X.att_w = reinterpret_cast<double *>(base + L.o_attw);
        X.ct_w = reinterpret_cast<double *>(base + L.o_ctw);
        X.crit_t = reinterpret_cast<double *>(base + L.o_ct);
        X.traj_crit_t = reinterpret_cast<double *>(base + L.o_tct);
        X.attrib = reinterpret_cast<double *>(base + L.o_at);
        X.traj_attrib = reinterpret_cast<double *>(base + L.o_tat);
    }
    if (dev_out) {
        if (dev_out->traj_prob) X.p = dev_out->traj_prob;
        if (dev_out->first_hit) X.hits = dev_out->first_hit;
        if (dev_out->q) X.q = dev_out->q;
        if (dev_out->traj_crit) X.traj_crit = dev_out->traj_crit;
        if (dev_out->object_crit) X.obj_crit = dev_out->object_crit;
        if (L.timeline) {
            if (dev_out->crit_t) X.crit_t = dev_out->crit_t;
            if (dev_out->traj_crit_t) X.traj_crit_t = dev_out->traj_crit_t;
            if (dev_out->attrib) X.attrib = dev_out->attrib;
            if (dev_out->traj_attrib) X.traj_attrib = dev_out->traj_attrib;
        }
    }
    X.n_obj = (int)L.objs.size();
    X.n_pairs = (int)L.pairs.size();
    X.n_strips = L.strip0.back();
    X.strip_len = L.strip_len;
    X.item_shift = L.item_shift;
    X.side_shift = L.side_shift;
    X.n_hits = L.n_hits;
    X.k2_grid = L.k2_grid;
    X.k1_x = L.k1_x;
    X.k3_x = L.k3_x;
    X.k3t_x = (int)L.k3t_x;
    X.k4t_y = L.k4t_y;
    X.variant = L.variant;
    X.family = L.family;
    (void)n_cu;
    return X;
}

int collide_parts(const Layout &L, int64_t checks_per_part)
{
    const int64_t want = (L.n_checks + checks_per_part - 1) / checks_per_part;
    return (int)std::max<int64_t>(2, std::min<int64_t>({want, L.strip0.back(), 64}));
}

hipError_t launch_all(const Launch &X, hipStream_t s)
{
    hipError_t e = launch_trajgen(X, s);
    if (e == hipSuccess) e = launch_collide(X, s);
    if (e == hipSuccess) e = launch_risk(X, s);
    return e;
}

}  // namespace mhc

using namespace mhc;

// ===========================================================================
// Context
// ===========================================================================

static mhc_status dev_err(mhc_ctx *ctx, hipError_t e, const char *what)
{
    if (ctx) ctx->err = std::string(what) + ": " + hipGetErrorString(e);
    return MHC_E_DEVICE;
}

#define HIPC(call)                                          \
    do {                                                    \
        hipError_t e_ = (call);                             \
        if (e_ != hipSuccess) return dev_err(ctx, e_, #call); \
    } while (0)

extern "C" mhc_status mhc_create(int device, size_t hbm_budget_bytes, mhc_ctx **out)
{
    if (!out) return MHC_E_INVAL;
    *out = nullptr;
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess || n <= 0) return MHC_E_DEVICE;
    if (device < 0 || device >= n) return MHC_E_INVAL;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) != hipSuccess) return MHC_E_DEVICE;
    if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0) return MHC_E_DEVICE;
    if (hipSetDevice(device) != hipSuccess) return MHC_E_DEVICE;
    mhc_ctx *ctx = new mhc_ctx();
    ctx->device = device;
    ctx->budget = hbm_budget_bytes;
    ctx->n_cu = prop.multiProcessorCount;
    if (hipStreamCreateWithFlags(&ctx->stream, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&ctx->staging_ev, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&ctx->noalloc_ev, hipEventDisableTiming) != hipSuccess ||
        noalloc_scratch_address(device, &ctx->scratch) != hipSuccess) {
        if (ctx->noalloc_ev) (void)hipEventDestroy(ctx->noalloc_ev);
        if (ctx->staging_ev) (void)hipEventDestroy(ctx->staging_ev);
        if (ctx->stream) (void)hipStreamDestroy(ctx->stream);
        delete ctx;
        return MHC_E_DEVICE;
    }
    *out = ctx;
    return MHC_OK;
}

extern "C" void mhc_destroy(mhc_ctx *ctx)
{
    if (!ctx) return;
    hipSetDevice(ctx->device);
    hipStreamSynchronize(ctx->stream);
    ctx->batch_graphs.clear();
    hipEventSynchronize(ctx->staging_ev);
    if (ctx->dbuf) hipFree(ctx->dbuf);
    if (ctx->staging) hipHostFree(ctx->staging);
    if (ctx->res_pin) hipHostFree(ctx->res_pin);
    hipEventSynchronize(ctx->noalloc_ev);
    hipEventDestroy(ctx->staging_ev);
    hipEventDestroy(ctx->noalloc_ev);
    hipStreamDestroy(ctx->stream);
    delete ctx;
}

int mhc_ctx::max_waves(int v, const mhc_scene *scenes, int n)
{
    int fam = 0, tl = 0;
    for (int k = 0; k < n; ++k) {
        fam = std::max(fam, scene_family(&scenes[k]));
        tl |= scenes[k].timeline != 0;
    }
    return max_waves_of(v, fam, tl != 0);
}

int mhc_ctx::max_waves_of(int v, int fam, bool tl)
{
    if (v < 0 || v >= N_VARIANTS) v = 0;
    int &w = waves_cache[v][fam][tl ? 1 : 0];
    if (!w) w = n_cu * collide_blocks_per_cu(v, fam, tl, true);
    return w;
}

extern "C" const char *mhc_last_error(const mhc_ctx *ctx) { return ctx ? ctx->err.c_str() : "no context"; }

extern "C" mhc_status mhc_query_sizes(const mhc_scene *scene, mhc_sizes *out)
{
    if (!out) return MHC_E_INVAL;
    std::string err;
    if (!validate_scene(scene, err)) return MHC_E_INVAL;
    // The workspace size depends on the micro-tile variant and on how many
    // waves the GPU holds; report the largest over all variants with one
    // wave per work unit, which bounds every actual layout.
    size_t bytes = 0;
    Layout L;
    for (int v = 0; v < N_VARIANTS; ++v) {
        build_layout(scene, 1, v, 0, L, true);
        bytes = std::max(bytes, L.total_bytes);
    }
    out->n_traj = L.n_traj;
    out->n_pairs = (int64_t)L.pairs.size();
    out->n_traj_pairs = L.n_hits;
    out->n_checks = L.n_checks;
    out->device_bytes = bytes;
    return MHC_OK;
}

// Walks a collision plan the way k2_collide decodes it: launches -> workgroups ->
// waves -> strips -> blocks -> units -> lanes -> items -> trajectory pairs, counting how
// often each item is tested and every index that leaves its pair.
static void walk_plan(const Layout &L, mhc_plan_info &info)
{
    std::vector<int64_t> item_base(L.pairs.size() + 1, 0);
    for (size_t p = 0; p < L.pairs.size(); ++p)
        item_base[p + 1] = item_base[p] + (int64_t)L.pairs[p].n_ig * L.pairs[p].n_jg;
    std::vector<uint8_t> seen((size_t)item_base.back(), 0);
    int64_t bad = 0, units = 0;
    int32_t time_split = 1;
    if (L.strip0.size() != L.pairs.size() + 1 || L.strip0[0] != 0 || L.k2_grid < 1) ++bad;
    for (size_t p = 0; p < L.pairs.size() && !bad; ++p) {
        const DPair &pr = L.pairs[p];
        const TileShape ts = kTiles[L.variant][pr.cls];
        // every position of an object holds another of its trajectories
        for (const DObj *o : {&L.objs[pr.a], &L.objs[pr.b]}) {
            std::vector<uint8_t> held((size_t)o->T, 0);
            for (int k = 0; k < o->T; ++k) {
                const int i = traj_at(k, o->n_u, o->n_w, o->strip);
                if (i < 0 || i >= o->T || held[(size_t)i]++) ++bad;
            }
        }
        // the units tile the items, the blocks the units, and a block's leaves
        // hold its units' positions
        if (pr.tshift < 0 || pr.tshift > MAX_TSHIFT || pr.bshift < 0 || pr.bshift > 6 - pr.tshift ||
            (1 << pr.tshift) > pr.H || L.strip0[p + 1] - L.strip0[p] != (int64_t)pr.nbi * pr.nsj) {
            ++bad;
            continue;
        }
        const int rows = (WAVE >> pr.tshift) >> pr.bshift, cols = 1 << pr.bshift;
        if ((int64_t)pr.nui * rows < pr.n_ig || (int64_t)pr.nuj * cols < pr.n_jg || pr.nbi * pr.block_ur < pr.nui ||
            (pr.nbj << pr.block_ucs) < pr.nuj || pr.block_ur * rows * ts.ri != (1 << L.side_shift) ||
            (cols * ts.rj) << pr.block_ucs != (1 << L.side_shift) || 1 << pr.unit_rs != rows * ts.ri ||
            1 << pr.unit_cs != cols * ts.rj || rows * ts.ri > BLOCK_SIDE || cols * ts.rj > BLOCK_SIDE || (pr.nbi - 1) * (1 << L.side_shift) >= pr.Ta ||
            (pr.nbj - 1) * (1 << L.side_shift) >= pr.Tb || pr.nsj * L.strip_len < pr.nbj ||
            (pr.nsj - 1) * L.strip_len >= pr.nbj || 1 << L.side_shift > BLOCK_SIDE ||
            (pr.block_ur << pr.block_ucs) * MIN_UNIT_PAIRS > BLOCK_PAIRS)
            ++bad;
        time_split = std::max(time_split, 1 << pr.tshift);
    }
    const int64_t n_strips = bad ? 0 : L.strip0.back();
    const int64_t per_round = (int64_t)L.k2_grid * (K2_WG / WAVE);
    const int64_t rounds = (n_strips + per_round - 1) / std::max<int64_t>(1, per_round);
    // cut as a large server tick cuts it: every strip in one of the parts
    const int parts = collide_parts(L, kPartChecks);
    for (int part = 0; part < parts && !bad; ++part) {
        const int64_t lo = strips_before_part(n_strips, part, parts), hi = strips_before_part(n_strips, part + 1, parts);
        if (lo < 0 || hi > n_strips || (lo >= hi && n_strips >= 2)) ++bad;
        for (int64_t rw = 0; rw * L.k2_grid < hi - lo; ++rw)
            for (int wg = 0; wg < L.k2_grid; ++wg) {
                const int64_t g = lo + rw * L.k2_grid + strip_in_row((int)rw, wg, L.k2_grid);
                if (g >= hi) continue;
                const size_t p = (size_t)(std::upper_bound(L.strip0.begin(), L.strip0.end(), g) - L.strip0.begin()) - 1;
                const DPair &pr = L.pairs[p];
                const TileShape ts = kTiles[L.variant][pr.cls];
                const DObj &oa = L.objs[pr.a], &ob = L.objs[pr.b];
                const int ri = ts.ri, rj = ts.rj, per = WAVE >> pr.tshift;
                int bi, sj;
                strip_at(pr, (uint32_t)(g - L.strip0[p]), &bi, &sj);
                if (bi < 0 || bi >= pr.nbi || sj < 0 || sj >= pr.nsj) ++bad;
                const int units_of = pr.block_ur << pr.block_ucs;
                for (int x = 0; x < units_of * L.strip_len; ++x) {
                    const int bj = sj * L.strip_len + x / units_of, u = x % units_of;
                    if (bj >= pr.nbj) break;
                    const int ui = bi * pr.block_ur + (u >> pr.block_ucs);
                    const int uj = (bj << pr.block_ucs) + (u & ((1 << pr.block_ucs) - 1));
                    if (ui >= pr.nui || uj >= pr.nuj) continue;
                    ++units;
                    for (int lane = 0; lane < per; ++lane) {   // the lanes of part 0
                        const int ig = ui * (per >> pr.bshift) + (lane >> pr.bshift);
                        const int jg = (uj << pr.bshift) + (lane & ((1 << pr.bshift) - 1));
                        if (ig >= pr.n_ig || jg >= pr.n_jg) continue;
                        if (ig < 0 || jg < 0) {
                            ++bad;
                            continue;
                        }
                        for (int r = 0; r < ri; ++r)
                            for (int sidx = 0; sidx < rj; ++sidx) {
                                const int64_t pi = (int64_t)ig * ri + r, pj = (int64_t)jg * rj + sidx;
                                if (pi >= pr.Ta || pj >= pr.Tb) continue;  // idle tile slot
                                const int64_t i = traj_at((int)pi, oa.n_u, oa.n_w, oa.strip);
                                const int64_t j = traj_at((int)pj, ob.n_u, ob.n_w, ob.strip);
                                const int64_t h = pr.hit_off + i * pr.Tb + j;
                                if (h < 0 || h >= L.n_hits) ++bad;
                                if (oa.q_row + i * oa.n_scene_obj + ob.local >= L.n_q ||
                                    ob.q_row + j * ob.n_scene_obj + oa.local >= L.n_q)
                                    ++bad;
                            }
                        uint8_t &s = seen[(size_t)(item_base[p] + (int64_t)ig * pr.n_jg + jg)];
                        if (s < 255) ++s;
                    }
                }
            }
    }
    int64_t uncovered = 0, repeated = 0;
    for (uint8_t c : seen) {
        uncovered += c == 0;
        repeated += c > 1;
    }
    // the trajectory kernel's grid: every block of every object (its
    // normalisation block and one per K1_TPB trajectories) taken by exactly
    // one workgroup, as the kernel maps (row, x) to (object, block)
    {
        const int n_obj = (int)L.objs.size();
        std::vector<int64_t> first(n_obj + 1, 0);
        for (int a = 0; a < n_obj; ++a) first[a + 1] = first[a] + (L.objs[a].T + K1_TPB - 1) / K1_TPB + 1;
        std::vector<uint8_t> took((size_t)first[n_obj], 0);
        const bool table = !L.k1_rows.empty();
        if (table ? (int64_t)L.k1_rows.size() != 2LL * L.k1_nrows : L.k1_nrows != n_obj) ++bad;
        for (int r = 0; r < L.k1_nrows && !bad; ++r) {
            const int obj = table ? L.k1_rows[2 * r] : r, b0 = table ? L.k1_rows[2 * r + 1] : 0;
            if (obj < 0 || obj >= n_obj || b0 < 0) {
                ++bad;
                break;
            }
            for (int x = 0; x < L.k1_x; ++x)
                if (first[obj] + b0 + x < first[obj + 1]) {
                    uint8_t &c = took[(size_t)(first[obj] + b0 + x)];
                    if (c < 255) ++c;
                }
        }
        for (uint8_t c : took) bad += c != 1;
    }
    int64_t blocked = 0;
    for (const DPair &pr : L.pairs) blocked += pr.bshift != 0;
    info.n_units = units;
    info.n_waves = per_round;
    info.blocked_pairs = blocked;
    info.uncovered = uncovered;
    info.repeated = repeated;
    info.out_of_range = bad;
    info.contiguous = rounds > 1 ? 1 : 0;
    info.time_split = time_split;
}

extern "C" mhc_status mhc_plan_check(int32_t n_scenes, const mhc_scene *scenes, int32_t variant, int32_t max_waves,
                                     mhc_plan_info *info)
{
    if (n_scenes < 1 || !scenes || !info || variant < 0 || variant >= N_VARIANTS || max_waves < 0)
        return MHC_E_INVAL;
    std::string err;
    int64_t total_objects = 0;
    for (int k = 0; k < n_scenes; ++k) {
        if (!validate_scene(&scenes[k], err, k)) return MHC_E_INVAL;
        total_objects += scenes[k].n_objects;
    }
    if (total_objects > kMaxObjectsPerLaunch) return MHC_E_INVAL;
    Layout L;
    build_layout(scenes, n_scenes, variant, max_waves, L, true);
    walk_plan(L, *info);
    return info->uncovered == 0 && info->repeated == 0 && info->out_of_range == 0 ? MHC_OK : MHC_E_INVAL;
}

extern "C" mhc_status mhc_anticipation_time(int32_t n_frames, const double *crit, double frame_dt, double threshold,
                                            int32_t event_frame, double *out_seconds)
{
    if (!crit || !out_seconds || n_frames < 1 || event_frame < 1 || event_frame > n_frames) return MHC_E_INVAL;
    if (!std::isfinite(frame_dt) || !(frame_dt > 0.0) || !std::isfinite(threshold)) return MHC_E_INVAL;
    for (int32_t f = 0; f < event_frame; ++f)
        if (!std::isfinite(crit[f])) return MHC_E_INVAL;
    // walk back from the last frame before the event while the criticality
    // stays at or above the threshold
    int32_t first = event_frame;
    while (first > 0 && crit[first - 1] >= threshold) --first;
    *out_seconds = (double)(event_frame - first) * frame_dt;
    return MHC_OK;
}

std::vector<int32_t> mhc::shape_of(const mhc_scene *s)
{
    std::vector<int32_t> v{s->n_objects, s->horizon, s->pairs, s->overlap, s->risk, s->timeline};
    for (int a = 0; a < s->n_objects; ++a) {
        v.push_back(s->objects[a].kind);
        v.push_back(s->objects[a].n_u);
        v.push_back(s->objects[a].n_w);
        v.push_back(s->objects[a].score != nullptr);
        v.push_back(s->objects[a].n_vertices);
        v.push_back(s->objects[a].model);
    }
    return v;
}

// Layout of `scene` for this context: the shape-dependent tables of the
// previous call are reused when the shape (and the tile variant) repeats.
static bool layout_for(mhc_ctx *ctx, const mhc_scene *scene, Layout &L, bool with_hits)
{
    const int v = ctx->variant_for(scene, 1);
    std::vector<int32_t> shape = shape_of(scene);
    shape.push_back(v);
    shape.push_back(ctx->max_waves(v, scene, 1));
    shape.push_back(with_hits);
    if (!L.objs.empty() && shape == ctx->layout_shape) {
        fill_values(scene, 1, L);
        return true;
    }
    build_layout(scene, 1, v, ctx->max_waves(v, scene, 1), L, with_hits, ctx->budget ? ctx->budget : SIZE_MAX);
    ctx->layout_shape = std::move(shape);
    return false;
}

// Pinned staging for the scene image. The previous upload from it must have
// left the host buffer before it is rewritten.
static mhc_status stage_image(mhc_ctx *ctx, const Layout &L, char **host, bool values_only = false)
{
    HIPC(hipEventSynchronize(ctx->staging_ev));
    if (ctx->staging_bytes < L.image_bytes) {
        if (ctx->staging) HIPC(hipHostFree(ctx->staging));
        ctx->staging = nullptr;
        ctx->staging_bytes = 0;
        size_t want = std::max<size_t>(L.image_bytes, 1 << 20);
        HIPC(hipHostMalloc(reinterpret_cast<void **>(&ctx->staging), want, hipHostMallocDefault));
        ctx->staging_bytes = want;
    }
    pack_image(L, ctx->staging, values_only);
    *host = ctx->staging;
    return MHC_OK;
}

mhc_status ensure_device(mhc_ctx *ctx, size_t bytes)
{
    if (ctx->budget && bytes > ctx->budget) {
        ctx->err = "scene needs " + std::to_string(bytes) + " device bytes, above the context budget";
        return MHC_E_NOMEM;
    }
    if (ctx->dbuf_bytes >= bytes) return MHC_OK;
    HIPC(hipStreamSynchronize(ctx->stream));
    ctx->batch_graphs.clear();  // their launches point into the old workspace
    ctx->resident_image.clear();
    if (ctx->dbuf) HIPC(hipFree(ctx->dbuf));
    ctx->dbuf = nullptr;
    ctx->dbuf_bytes = 0;
    size_t want = align256(bytes + bytes / 4);
    if (ctx->budget) want = std::min(want, ctx->budget);
    hipError_t e = hipMalloc(&ctx->dbuf, want);
    if (e != hipSuccess) {
        ctx->err = std::string("hipMalloc of the context workspace failed: ") + hipGetErrorString(e);
        return MHC_E_NOMEM;
    }
    ctx->dbuf_bytes = want;
    return MHC_OK;
}

static mhc_status upload_and_launch(mhc_ctx *ctx, const Layout &L, char *dbase, const mhc_result *dev_out,
                                    bool keep_hits, hipStream_t s)
{
    char *host = nullptr;
    mhc_status st = stage_image(ctx, L, &host);
    if (st != MHC_OK) return st;
    HIPC(hipMemcpyAsync(dbase, host, L.image_bytes, hipMemcpyHostToDevice, s));
    HIPC(hipEventRecord(ctx->staging_ev, s));
    Launch X = make_launch(L, dbase, dev_out, keep_hits, ctx->n_cu);
    HIPC(launch_all(X, s));
    return MHC_OK;
}

// Upload + trajectory/collision/risk launches of a context-owned layout,
// replayed as one graph per shape key (the scene image's values change from
// call to call, its layout and every launch argument do not). A key's first
// launch is direct (GraphCache::repeated): capturing costs more than it saves
// for a shape that does not come back soon.
static mhc_status graph_upload_and_launch(mhc_ctx *ctx, const Layout &L, char *dbase, bool keep_hits,
                                          std::vector<int64_t> key, hipStream_t s, bool values_only = false)
{
    char *host = nullptr;
    mhc_status st = stage_image(ctx, L, &host, values_only);
    if (st != MHC_OK) return st;
    const size_t up = values_only ? L.value_bytes : L.image_bytes;
    key.push_back((int64_t)(uintptr_t)dbase);
    key.push_back((int64_t)(uintptr_t)host);
    key.push_back(keep_hits);
    key.push_back((int64_t)L.image_bytes);
    key.push_back((int64_t)up);
    Launch X = make_launch(L, dbase, nullptr, keep_hits, ctx->n_cu);
    if (ctx->batch_graphs.repeated(key)) {
        hipGraphExec_t exec = nullptr;
        HIPC(ctx->batch_graphs.get(key, [&](hipStream_t cs) {
            hipError_t e = hipMemcpyAsync(dbase, host, up, hipMemcpyHostToDevice, cs);
            return e == hipSuccess ? launch_all(X, cs) : e;
        }, &exec));
        HIPC(hipGraphLaunch(exec, s));
    } else {
        HIPC(hipMemcpyAsync(dbase, host, up, hipMemcpyHostToDevice, s));
        HIPC(launch_all(X, s));
    }
    HIPC(hipEventRecord(ctx->staging_ev, s));
    return MHC_OK;
}

// Every output is one region of the workspace in which scene k's part starts
// at a known offset, so each requested output of all scenes comes down in one
// transfer into pinned host memory (one DMA instead of one staged copy into
// pageable memory per scene and output), and the host then copies each
// scene's part to its buffer. Unless every output is to be staged, regions
// above kResultStageMax (the first hits of large scenes), and the largest
// ones while the staged total exceeds kResultStageTotal, are copied per scene
// straight to the callers' buffers.
static const size_t kResultStageMax = size_t(64) << 20;
static const size_t kResultStageTotal = size_t(256) << 20;
// Staged outputs at most this far apart in the workspace share one transfer
// (the bytes between them come along).
static const size_t kResultMergeGap = size_t(64) << 10;

namespace mhc {

// Output f (RESULT order, then the time-resolved ones) of scene k: its host
// buffer (NULL when not asked for) and its bytes in the workspace.
static void result_part(const Layout &L, const mhc_result *res, int f, int k, void **dst, size_t *off,
                        size_t *bytes)
{
    const SceneExt &e = L.sc[k];
    const mhc_result &r = res[k];
    const size_t H = (size_t)e.H, nq = (size_t)e.n_traj * e.n_obj;
    switch (f) {
    case 0: *dst = r.object_crit; *off = L.o_oc + e.obj0 * 8; *bytes = (size_t)e.n_obj * 8; break;
    case 1: *dst = r.traj_crit; *off = L.o_tc + e.traj0 * 8; *bytes = (size_t)e.n_traj * 8; break;
    case 2: *dst = r.traj_prob; *off = L.o_p + e.traj0 * 8; *bytes = (size_t)e.n_traj * 8; break;
    case 3: *dst = r.q; *off = L.o_q + e.q0 * 8; *bytes = nq * 8; break;
    case 4: *dst = r.first_hit; *off = L.o_hits + e.hit0 * 2; *bytes = (size_t)e.n_hits * 2; break;
    case 5: *dst = e.timeline ? r.crit_t : nullptr; *off = L.o_ct + e.tl_obj0 * 8; *bytes = (size_t)e.n_obj * H * 8; break;
    case 6: *dst = e.timeline ? r.traj_crit_t : nullptr; *off = L.o_tct + e.tl_traj0 * 8; *bytes = (size_t)e.n_traj * H * 8; break;
    case 7: *dst = e.timeline ? r.attrib : nullptr; *off = L.o_at + e.tl_att0 * 8; *bytes = (size_t)e.n_obj * e.n_obj * 8; break;
    default: *dst = e.timeline ? r.traj_attrib : nullptr; *off = L.o_tat + e.q0 * 8; *bytes = nq * 8; break;
    }
    if (!*bytes) *dst = nullptr;
}

ResultPlan plan_results(const Layout &L, int n, const mhc_result *res, bool stage_all)
{
    ResultPlan R;
    size_t total = 0;
    for (int f = 0; f < ResultPlan::kOutputs; ++f) {
        R.lo[f] = SIZE_MAX;
        R.hi[f] = 0;
        for (int k = 0; k < n; ++k) {
            void *dst;
            size_t off, bytes;
            result_part(L, res, f, k, &dst, &off, &bytes);
            if (!dst) continue;
            R.lo[f] = std::min(R.lo[f], off);
            R.hi[f] = std::max(R.hi[f], off + bytes);
        }
        R.stage[f] = R.hi[f] > R.lo[f] && (stage_all || R.hi[f] - R.lo[f] <= kResultStageMax);
        if (R.stage[f]) total += R.hi[f] - R.lo[f];
    }
    while (!stage_all && total > kResultStageTotal) {
        int big = -1;
        for (int f = 0; f < ResultPlan::kOutputs; ++f)
            if (R.stage[f] && (big < 0 || R.hi[f] - R.lo[f] > R.hi[big] - R.lo[big])) big = f;
        R.stage[big] = false;
        total -= R.hi[big] - R.lo[big];
    }
    // staged outputs in workspace order; one transfer for each run of them
    // separated by at most kResultMergeGap bytes
    int ord[ResultPlan::kOutputs], m = 0;
    for (int f = 0; f < ResultPlan::kOutputs; ++f)
        if (R.stage[f]) ord[m++] = f;
    std::sort(ord, ord + m, [&](int x, int y) { return R.lo[x] < R.lo[y]; });
    R.staged = 0;
    R.n_copies = 0;
    for (int i = 0; i < m; ++i) {
        const int f = ord[i];
        if (R.n_copies > 0 && R.lo[f] <= R.copy_hi[R.n_copies - 1] + kResultMergeGap) {
            R.copy_hi[R.n_copies - 1] = std::max(R.copy_hi[R.n_copies - 1], R.hi[f]);
        } else {
            R.copy_lo[R.n_copies] = R.lo[f];
            R.copy_hi[R.n_copies] = R.hi[f];
            ++R.n_copies;
        }
    }
    for (int c = 0; c < R.n_copies; ++c) {
        R.copy_at[c] = R.staged;
        R.staged += (R.copy_hi[c] - R.copy_lo[c] + 255) & ~size_t(255);
    }
    for (int i = 0; i < m; ++i) {
        const int f = ord[i];
        int c = 0;
        while (!(R.copy_lo[c] <= R.lo[f] && R.hi[f] <= R.copy_hi[c])) ++c;
        R.at[f] = R.copy_at[c] + (R.lo[f] - R.copy_lo[c]);
    }
    return R;
}

hipError_t enqueue_results(const ResultPlan &R, const Layout &L, int n, const char *dbase, char *pinned,
                           const mhc_result *res, hipStream_t s)
{
    for (int c = 0; c < R.n_copies; ++c) {
        const hipError_t e = hipMemcpyAsync(pinned + R.copy_at[c], dbase + R.copy_lo[c],
                                            R.copy_hi[c] - R.copy_lo[c], hipMemcpyDeviceToHost, s);
        if (e != hipSuccess) return e;
    }
    for (int f = 0; f < ResultPlan::kOutputs; ++f) {
        if (R.hi[f] <= R.lo[f] || R.stage[f]) continue;
        for (int k = 0; k < n; ++k) {
            void *dst;
            size_t off, bytes;
            result_part(L, res, f, k, &dst, &off, &bytes);
            if (!dst) continue;
            const hipError_t e = hipMemcpyAsync(dst, dbase + off, bytes, hipMemcpyDeviceToHost, s);
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

void scatter_results(const ResultPlan &R, const Layout &L, int n, const char *pinned, const mhc_result *res)
{
    for (int f = 0; f < ResultPlan::kOutputs; ++f) {
        if (!R.stage[f]) continue;
        for (int k = 0; k < n; ++k) {
            void *dst;
            size_t off, bytes;
            result_part(L, res, f, k, &dst, &off, &bytes);
            if (dst) std::memcpy(dst, pinned + R.at[f] + (off - R.lo[f]), bytes);
        }
    }
}

}  // namespace mhc

mhc_status download_results(mhc_ctx *ctx, const Layout &L, int n, const char *dbase, const mhc_result *res,
                            hipStream_t s)
{
    const ResultPlan R = plan_results(L, n, res, false);
    if (R.staged > ctx->res_pin_bytes) {
        if (ctx->res_pin) HIPC(hipHostFree(ctx->res_pin));
        ctx->res_pin = nullptr;
        ctx->res_pin_bytes = 0;
        const size_t want = std::max(R.staged, size_t(1) << 20);
        HIPC(hipHostMalloc(reinterpret_cast<void **>(&ctx->res_pin), want, hipHostMallocDefault));
        ctx->res_pin_bytes = want;
    }
    HIPC(enqueue_results(R, L, n, dbase, ctx->res_pin, res, s));
    HIPC(hipStreamSynchronize(s));
    scatter_results(R, L, n, ctx->res_pin, res);
    return MHC_OK;
}

extern "C" mhc_status mhc_evaluate(mhc_ctx *ctx, const mhc_scene *scene, mhc_result *res)
{
    if (!ctx) return MHC_E_INVAL;
    if (!res || !res->object_crit) {
        ctx->err = "result and result->object_crit must not be NULL";
        return MHC_E_INVAL;
    }
    if (!validate_scene(scene, ctx->err) || !validate_outputs(scene, res, ctx->err)) return MHC_E_INVAL;
    HIPC(hipSetDevice(ctx->device));
    Layout &L = ctx->layout;
    const bool reused = layout_for(ctx, scene, L, res->first_hit != nullptr);
    mhc_status st = ensure_device(ctx, L.total_bytes);
    if (st != MHC_OK) return st;
    char *dbase = static_cast<char *>(ctx->dbuf);
    std::vector<int64_t> key(ctx->layout_shape.begin(), ctx->layout_shape.end());
    key.push_back(-1);  // single scene
    // When the previous launch in this workspace was this shape's, its
    // collision plan is still there and only the image's value part goes up.
    std::vector<int64_t> resident = key;
    resident.push_back((int64_t)(uintptr_t)dbase);
    const bool values_only = reused && ctx->resident_image == resident;
    ctx->resident_image.clear();
    st = graph_upload_and_launch(ctx, L, dbase, res->first_hit != nullptr, key, ctx->stream, values_only);
    if (st != MHC_OK) return st;
    ctx->resident_image = std::move(resident);
    return download_results(ctx, L, 1, dbase, res, ctx->stream);
}

extern "C" mhc_status mhc_evaluate_async(mhc_ctx *ctx, const mhc_scene *scene, void *dev_workspace,
                                         size_t workspace_bytes, const mhc_result *dev_out, void *hip_stream)
{
    if (!ctx) return MHC_E_INVAL;
    if (!dev_out || !dev_out->object_crit || !dev_workspace) {
        ctx->err = "dev_workspace, dev_out and dev_out->object_crit must not be NULL";
        return MHC_E_INVAL;
    }
    if (reinterpret_cast<uintptr_t>(dev_workspace) % 256 != 0) {
        ctx->err = "dev_workspace must be 256-byte aligned";
        return MHC_E_INVAL;
    }
    if (!validate_scene(scene, ctx->err) || !validate_outputs(scene, dev_out, ctx->err)) return MHC_E_INVAL;
    Layout L;
    const int v = ctx->variant_for(scene, 1);
    build_layout(scene, 1, v, ctx->max_waves(v, scene, 1), L, true, workspace_bytes);
    if (workspace_bytes < L.total_bytes) {
        ctx->err = "workspace too small: need " + std::to_string(L.total_bytes) + " bytes";
        return MHC_E_INVAL;
    }
    HIPC(hipSetDevice(ctx->device));
    return upload_and_launch(ctx, L, static_cast<char *>(dev_workspace), dev_out, false,
                             static_cast<hipStream_t>(hip_stream));
}

extern "C" mhc_status mhc_evaluate_noalloc(mhc_ctx *ctx, const mhc_scene *scene, const mhc_result *dev_out,
                                           void *hip_stream)
{
    if (!ctx) return MHC_E_INVAL;
    if (!dev_out || !dev_out->object_crit) {
        ctx->err = "dev_out and dev_out->object_crit must not be NULL";
        return MHC_E_INVAL;
    }
    if (!validate_scene(scene, ctx->err) || !validate_outputs(scene, dev_out, ctx->err)) return MHC_E_INVAL;
    HIPC(hipSetDevice(ctx->device));
    if (!ctx->scratch) {
        ctx->err = "the allocation-free workspace of this device was not found";
        return MHC_E_DEVICE;
    }
    // the first hits go to dev_out->first_hit only, so the array holds none
    Layout &L = ctx->noalloc_layout;
    const int v = ctx->variant_for(scene, 1);
    build_layout(scene, 1, v, ctx->max_waves(v, scene, 1), L, false, kNoallocBytes);
    if (L.total_bytes > kNoallocBytes) {
        ctx->err = "scene needs " + std::to_string(L.total_bytes) + " workspace bytes, above MHC_NOALLOC_MAX_BYTES (" +
                   std::to_string(kNoallocBytes) + ")";
        return MHC_E_NOMEM;
    }
    const hipStream_t s = static_cast<hipStream_t>(hip_stream);
    // the previous call's upload must have left the host image before it is
    // rewritten
    HIPC(hipEventSynchronize(ctx->noalloc_ev));
    if (ctx->noalloc_image.size() < L.image_bytes) ctx->noalloc_image.resize(L.image_bytes);
    pack_image(L, ctx->noalloc_image.data());
    HIPC(hipMemcpyAsync(ctx->scratch, ctx->noalloc_image.data(), L.image_bytes, hipMemcpyHostToDevice, s));
    HIPC(hipEventRecord(ctx->noalloc_ev, s));
    Launch X = make_launch(L, ctx->scratch, dev_out, false, ctx->n_cu);
    HIPC(launch_all(X, s));
    return MHC_OK;
}

// ===========================================================================
// Graph cache: one instantiated HIP graph per key, captured from a launch
// sequence on a private stream (capture does not execute anything).
// ===========================================================================

GraphCache::~GraphCache() { clear(); }

void GraphCache::clear()
{
    for (auto &kv : graphs) hipGraphExecDestroy(kv.second);
    graphs.clear();
    order.clear();
    seen.clear();
    if (capture) hipStreamDestroy(capture);
    capture = nullptr;
}

bool GraphCache::repeated(const std::vector<int64_t> &key)
{
    ++uses;
    if (graphs.count(key)) return true;
    for (auto it = seen.begin(); it != seen.end(); ++it)
        if (it->first == key) {
            if (uses - it->second <= (int64_t)kMaxGraphs) {
                seen.erase(it);
                return true;
            }
            it->second = uses;
            return false;
        }
    if (seen.size() >= kMaxSeen) seen.pop_front();
    seen.emplace_back(key, uses);
    return false;
}

hipError_t GraphCache::get(const std::vector<int64_t> &key, const std::function<hipError_t(hipStream_t)> &enqueue,
                           hipGraphExec_t *out)
{
    auto it = graphs.find(key);
    if (it != graphs.end()) {
        *out = it->second;
        return hipSuccess;
    }
    hipError_t e = hipSuccess;
    if (!capture) e = hipStreamCreateWithFlags(&capture, hipStreamNonBlocking);
    if (e != hipSuccess) return e;
    e = hipStreamBeginCapture(capture, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) return e;
    const hipError_t le = enqueue(capture);
    hipGraph_t g = nullptr;
    e = hipStreamEndCapture(capture, &g);
    if (le != hipSuccess) {
        if (g) hipGraphDestroy(g);
        return le;
    }
    if (e != hipSuccess) return e;
    hipGraphExec_t ex = nullptr;
    e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
    hipGraphDestroy(g);
    if (e != hipSuccess) return e;
    if (graphs.size() >= kMaxGraphs) {  // drop the oldest
        auto old = graphs.find(order.front());
        if (old != graphs.end()) {
            hipGraphExecDestroy(old->second);
            graphs.erase(old);
        }
        order.erase(order.begin());
    }
    graphs[key] = ex;
    order.push_back(key);
    *out = ex;
    return hipSuccess;
}

// ===========================================================================
// Plans: inputs resident in device memory, launched repeatedly.
// ===========================================================================

struct mhc_plan {
    mhc_ctx *ctx = nullptr;
    Layout L;
    mhc_scene flags{};            // pair mode, overlap, risk and timeline of the planned scene
    char *dbuf = nullptr;
    std::vector<int32_t> shape;   // kinds, grid sizes, horizon, pair mode
    GraphCache graphs;            // K1 -> K2 -> K3 per set of output pointers
    bool use_graphs = false;
};


extern "C" mhc_status mhc_plan_create(mhc_ctx *ctx, const mhc_scene *scene, mhc_plan **out)
{
    if (!ctx || !out) return MHC_E_INVAL;
    *out = nullptr;
    if (!validate_scene(scene, ctx->err)) return MHC_E_INVAL;
    HIPC(hipSetDevice(ctx->device));
    mhc_plan *pl = new mhc_plan();
    pl->ctx = ctx;
    const int v = ctx->variant_for(scene, 1);
    build_layout(scene, 1, v, ctx->max_waves(v, scene, 1), pl->L, true, ctx->budget ? ctx->budget : SIZE_MAX);
    pl->shape = shape_of(scene);
    pl->flags = *scene;
    pl->flags.objects = nullptr;
    if (ctx->budget && pl->L.total_bytes > ctx->budget) {
        ctx->err = "plan needs more device memory than the context budget";
        delete pl;
        return MHC_E_NOMEM;
    }
    if (hipMalloc(reinterpret_cast<void **>(&pl->dbuf), pl->L.total_bytes) != hipSuccess) {
        ctx->err = "hipMalloc for the plan failed";
        delete pl;
        return MHC_E_NOMEM;
    }
    std::vector<char> img(pl->L.image_bytes);
    pack_image(pl->L, img.data());
    hipError_t e = hipMemcpy(pl->dbuf, img.data(), pl->L.image_bytes, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        hipFree(pl->dbuf);
        delete pl;
        return dev_err(ctx, e, "plan upload");
    }
    *out = pl;
    return MHC_OK;
}

extern "C" mhc_status mhc_plan_update(mhc_plan *pl, const mhc_scene *scene)
{
    if (!pl) return MHC_E_INVAL;
    mhc_ctx *ctx = pl->ctx;
    if (!validate_scene(scene, ctx->err)) return MHC_E_INVAL;
    if (shape_of(scene) != pl->shape) {
        ctx->err = "mhc_plan_update: scene shape differs from the plan";
        return MHC_E_INVAL;
    }
    HIPC(hipSetDevice(ctx->device));
    Layout L;
    build_layout(scene, 1, pl->L.variant, ctx->max_waves(pl->L.variant, scene, 1), L, true, pl->L.total_bytes);
    std::vector<char> img(L.image_bytes);
    pack_image(L, img.data());
    HIPC(hipDeviceSynchronize());
    HIPC(hipMemcpy(pl->dbuf, img.data(), L.image_bytes, hipMemcpyHostToDevice));
    pl->L = std::move(L);
    pl->flags = *scene;
    pl->flags.objects = nullptr;
    return MHC_OK;
}

extern "C" mhc_status mhc_plan_execute(mhc_plan *pl, const mhc_result *dev_out, void *hip_stream)
{
    if (!pl) return MHC_E_INVAL;
    mhc_ctx *ctx = pl->ctx;
    if (!validate_outputs(&pl->flags, dev_out, ctx->err)) return MHC_E_INVAL;
    HIPC(hipSetDevice(ctx->device));
    Launch X = make_launch(pl->L, pl->dbuf, dev_out, true, ctx->n_cu);
    const hipStream_t s = static_cast<hipStream_t>(hip_stream);
    if (!pl->use_graphs) {
        HIPC(launch_all(X, s));
        return MHC_OK;
    }
    // The launch sequence depends only on the plan and the output pointers:
    // it is captured once per pointer set and replayed as one graph.
    std::vector<int64_t> key{(int64_t)(uintptr_t)pl->dbuf};
    if (dev_out)
        for (const void *ptr : {(const void *)dev_out->object_crit, (const void *)dev_out->traj_crit,
                                (const void *)dev_out->traj_prob, (const void *)dev_out->q,
                                (const void *)dev_out->first_hit, (const void *)dev_out->crit_t,
                                (const void *)dev_out->traj_crit_t, (const void *)dev_out->attrib,
                                (const void *)dev_out->traj_attrib})
            key.push_back((int64_t)(uintptr_t)ptr);
    hipGraphExec_t exec = nullptr;
    HIPC(pl->graphs.get(key, [&](hipStream_t cs) { return launch_all(X, cs); }, &exec));
    HIPC(hipGraphLaunch(exec, s));
    return MHC_OK;
}

extern "C" mhc_status mhc_plan_execute_stages(mhc_plan *pl, const mhc_result *dev_out, void *hip_stream,
                                              uint32_t stages)
{
    if (!pl) return MHC_E_INVAL;
    mhc_ctx *ctx = pl->ctx;
    if (stages == 0 || stages > MHC_STAGE_ALL) {
        ctx->err = "stages must be a non-empty combination of MHC_STAGE_* bits";
        return MHC_E_INVAL;
    }
    if (!validate_outputs(&pl->flags, dev_out, ctx->err)) return MHC_E_INVAL;
    HIPC(hipSetDevice(ctx->device));
    const hipStream_t s = static_cast<hipStream_t>(hip_stream);
    Launch X = make_launch(pl->L, pl->dbuf, dev_out, true, ctx->n_cu);
    // The first hits are the collision stage's: the trajectory kernel clears
    // them only where that stage follows in this call, else it does so itself.
    Launch traj = X;
    if (!(stages & MHC_STAGE_COLLIDE)) traj.hits = nullptr;
    if (stages & MHC_STAGE_TRAJ) HIPC(launch_trajgen(traj, s));
    X.clear_hits = !(stages & MHC_STAGE_TRAJ);
    if (stages & MHC_STAGE_COLLIDE) HIPC(launch_collide(X, s));
    if (stages & MHC_STAGE_RISK) HIPC(launch_risk(X, s));
    return MHC_OK;
}

extern "C" mhc_status mhc_plan_set_graph(mhc_plan *pl, int32_t enable)
{
    if (!pl || (enable != 0 && enable != 1)) return MHC_E_INVAL;
    pl->use_graphs = enable == 1;
    return MHC_OK;
}

extern "C" mhc_status mhc_plan_download(mhc_plan *pl, mhc_result *host_out)
{
    if (!pl || !host_out) return MHC_E_INVAL;
    mhc_ctx *ctx = pl->ctx;
    if (!validate_outputs(&pl->flags, host_out, ctx->err)) return MHC_E_INVAL;
    HIPC(hipSetDevice(ctx->device));
    HIPC(hipDeviceSynchronize());
    return download_results(ctx, pl->L, 1, static_cast<const char *>(pl->dbuf), host_out, ctx->stream);
}

extern "C" void mhc_plan_destroy(mhc_plan *pl)
{
    if (!pl) return;
    hipSetDevice(pl->ctx->device);
    hipDeviceSynchronize();
    pl->graphs.clear();
    if (pl->dbuf) hipFree(pl->dbuf);
    delete pl;
}

// ===========================================================================
// Batched
// ===========================================================================

extern "C" mhc_status mhc_evaluate_batch(mhc_ctx *ctx, int32_t n, const mhc_scene *scenes, mhc_result *res)
{
    if (!ctx) return MHC_E_INVAL;
    if (n < 1 || !scenes || !res) {
        ctx->err = "batch needs n >= 1, scenes and results";
        return MHC_E_INVAL;
    }
    int64_t total_objects = 0;
    for (int k = 0; k < n; ++k) {
        if (!validate_scene(&scenes[k], ctx->err, k)) return MHC_E_INVAL;
        total_objects += scenes[k].n_objects;
        if (total_objects > kMaxObjectsPerLaunch) {
            ctx->err = "batch holds more than 65535 objects";
            return MHC_E_INVAL;
        }
        if (!res[k].object_crit) {
            ctx->err = "result " + std::to_string(k) + ": object_crit must not be NULL";
            return MHC_E_INVAL;
        }
        if (!validate_outputs(&scenes[k], &res[k], ctx->err, k)) return MHC_E_INVAL;
    }
    HIPC(hipSetDevice(ctx->device));
    return batch_run(ctx, n, scenes, res);
}

// Batched form: all scenes share one scene image, one trajectory launch, one
// collision launch over all their pairs' units and one risk launch.
mhc_status batch_run(mhc_ctx *ctx, int n, const mhc_scene *scenes, mhc_result *res)
{
    Layout &L = ctx->layout;
    bool keep = false;
    for (int k = 0; k < n; ++k) keep |= res[k].first_hit != nullptr;
    const int v = ctx->variant_for(scenes, n);
    const int waves = ctx->max_waves(v, scenes, n);
    std::vector<int64_t> key{v, waves, n};
    // the layout's shape: a batch marker (a single scene's shape starts with
    // its object count), the key and whether first hits are kept
    std::vector<int32_t> shape{-2, v, waves, n, keep};
    for (int k = 0; k < n; ++k) {
        const std::vector<int32_t> sh = shape_of(&scenes[k]);
        key.insert(key.end(), sh.begin(), sh.end());
        shape.insert(shape.end(), sh.begin(), sh.end());
    }
    // A batch of the previous call's shapes keeps its layout (pairs, plan,
    // offsets) and only takes the new values, and when the workspace still
    // holds that layout's image only the value part goes up.
    const bool reused = !L.objs.empty() && shape == ctx->layout_shape;
    if (reused) {
        fill_values(scenes, n, L);
    } else {
        build_layout(scenes, n, v, waves, L, keep, ctx->budget ? ctx->budget : SIZE_MAX);
        ctx->layout_shape = std::move(shape);
    }
    mhc_status st = ensure_device(ctx, L.total_bytes);
    if (st != MHC_OK) return st;
    char *dbase = static_cast<char *>(ctx->dbuf);
    std::vector<int64_t> resident = key;
    resident.push_back(keep);
    resident.push_back((int64_t)(uintptr_t)dbase);
    const bool values_only = reused && ctx->resident_image == resident;
    ctx->resident_image.clear();
    st = graph_upload_and_launch(ctx, L, dbase, keep, key, ctx->stream, values_only);
    if (st != MHC_OK) return st;
    ctx->resident_image = std::move(resident);
    return download_results(ctx, L, n, dbase, res, ctx->stream);
}
