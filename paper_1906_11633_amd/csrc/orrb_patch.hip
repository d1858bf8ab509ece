// Patch path (k_patch): rectangles of frames, for batches with too few frames to occupy the
// chip with one workgroup per frame, for frames larger than the frame kernel takes and for
// scenes that do not fit in LDS.
//
// One 1024-thread workgroup renders one patch.  Scenes that fit in LDS (the frame kernel's
// limits) need no intermediate data in global memory; for larger ones (G) k_vertex has put
// the snapped vertices and the objects' pixel ranges in the workspace, steps 1 and 2 fall
// away, and the patch may be larger:
//   1. eight lanes per object project its mesh's bounding box; objects that miss the patch
//      are left out;
//   2. the kept objects' vertices are transformed and snapped (FP64) into LDS, 64 vertices
//      of one object per wave and step, so that everything about the object is
//      wave-uniform;
//   3. their triangles are tested the same way; each wave collects the visible ones and, 64
//      at a time, rasterizes them into the patch's 64-bit visibility keys in LDS
//      (ds_min_u64), one lane to a triangle; larger triangles are queued and then shared out
//      over all waves, sixteen lanes to a triangle;
//   4. each wave stores its background pixels, collects its covered ones and, 64 at a time,
//      shades and stores them.
// The arithmetic is the other paths' (orrb_primitives.h), so the outputs have the same bits.
//
// What bounds it: with few patches, the chain of phases in one workgroup (about 4 k cycles
// for the objects, 4 to 10 k for vertices, as much for shading, more for the triangles of
// crowded patches); with many, VALU issue, a third of it in testing triangles that turn out
// to face away or miss the patch, which every patch of a frame repeats.  A patch holds as
// many pixels as fit in LDS beside the largest scene's vertices.  Per-object work lists
// leave nothing to look up per vertex or triangle; collecting visible triangles fills the
// lanes (a quarter of the tested ones are visible, half of those cover no more than three
// pixel centres); one lane steps through at most kPOwn pixels because a longer loop keeps
// the other 63 waiting (8 to 12 measured alike, 32 up to 15 % slower).
// One MI355X, us a call, one workgroup per frame before / patches: 4 plain 64 x 64 frames
// 27 / 9.5, 6 hand frames of 128 x 128 68 / 16, 48 of 200 x 200 118 / 45; 2 of 1024 x 768
// (tiled path before) 113 / 30.  Larger scenes (G), 24 / 192 / 384 uneven frames: tiled path
// 132 / 387 / 683, frame kernel with global scratch 175 / 365 / 382, patches 47 / 146 / 256.
#include <cstddef>

#include "orrb_post.h"

namespace orrb {

constexpr int kPT = 1024;            // threads of a patch workgroup
constexpr int kPW = kPT / kWave;     // waves
constexpr int kPVMax = 6976;         // scene vertices held in LDS (the frame kernel's limit)
constexpr int kPOMax = 48;           // scene objects (likewise; one lane each)
constexpr int kPPixels = 6784;       // pixels of a patch
constexpr int kPGOMax = 127;         // objects of a larger scene
constexpr int kPGPixels = 16384;     // pixels of its patches
constexpr int kPOwn = 10;            // most pixels (of its range) of a triangle that one lane rasterizes
constexpr int kPBig = 1024;          // larger triangles queued (beyond: one lane's work as well)

template <bool G>
struct PatchLds {
    static constexpr int kObj = G ? kPGOMax : kPOMax;
    // G = false: the kept objects' snapped vertices, all objects' matrices
    int2 XY[G ? 1 : kPVMax];
    float iw[G ? 1 : kPVMax];
    double M[G ? 1 : kPOMax][12];
    unsigned char keep[G ? 1 : kPOMax];
    alignas(16) unsigned long long vis[G ? kPGPixels : kPPixels];  // (depth bits << 32) | object << 16 | scene triangle
    float R[kObj][9];
    Material mat[kObj];
    int tbase[kObj], mtb[kObj], mvb[kObj], vbase[kObj], seg[kObj];
    float4 light[kMaxLights];
    int ltype[kMaxLights];
    SpotLight spot[kMaxSpots];
    // per wave: visible small triangles (object << 16 | triangle), then covered pixels
    unsigned small[kPW][2 * kWave];
    unsigned big[kPBig];             // queued larger ones
    int n_big, next_big;
    unsigned account[2];  // bin entries and survivors the frame kernel would count
};
static_assert(sizeof(PatchLds<false>) <= 160 * 1024 && sizeof(PatchLds<true>) <= 160 * 1024, "patch LDS exceeds 160 KB");
static_assert(offsetof(PatchLds<false>, vis) % 16 == 0 && offsetof(PatchLds<true>, vis) % 16 == 0,
              "the keys are cleared with 16-byte stores");

int patch_max_pixels(bool global) { return global ? kPGPixels : kPPixels; }
bool patch_fits_global(int n_obj, int64_t n_tris) { return n_obj <= kPGOMax && n_tris < 65536; }

// The snapped vertices of the frame: in LDS, or k_vertex's records (X, Y, bits of 1 / w,
// valid) in the workspace.
template <bool G>
struct PatchVerts {
    const PatchLds<G> &S;
    const int4 *records;
    ORRB_INLINE int4 get(int v) const {
        if constexpr (G) {
            return records[v];
        } else {
            const int2 p = S.XY[v];
            return make_int4(p.x, p.y, __float_as_int(S.iw[v]), p.x != kInvalidX);
        }
    }
};

// Objects of the patch: keep[k] = 1 where scene object k may touch its pixels.  Eight lanes
// per object project the corners of its mesh's bounding box (FP64, any affine pose).  When
// every corner is in front of the near plane and well inside the guard band, so is every
// vertex, and the triangles lie inside the corners' range (perspective maps the box's
// convex hull into the hull of its corners); the object is then left out if that range,
// widened by a pixel for rounding, misses the patch.  Otherwise it is kept: objects left out
// have no vertex that the call's counters would count.  Also leaves the objects' matrices
// in M and R.
ORRB_INLINE void patch_cull(const RenderArgs &a, PatchLds<false> &S, const PatchItem &it, const FrameInfo &fi, int tid) {
    const int k = tid >> 3, c = tid & 7;
    if (tid - lane_id() >= 8 * fi.n_obj) return;  // wave-uniform
    const float *V = a.view + 12 * (int64_t)it.frame, *K = a.intr + 4 * (int64_t)it.frame;
    bool safe = false, shown = false;
    int x0 = 0, x1 = 0, y0 = 0, y1 = 0;
    if (k < fi.n_obj) {
        const int o = fi.obj_begin + k;
        const float *lo = a.mesh_box + 6 * (int64_t)a.objs[o].mesh, *hi = lo + 3;
        const float *P = a.pose + 12 * (int64_t)o;
        shown = a.visible[o] != 0;
        const double px = c & 1 ? hi[0] : lo[0], py = c & 2 ? hi[1] : lo[1], pz = c & 4 ? hi[2] : lo[2];
        double q[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const double m0 = compose_entry(V, P, 4 * r), m1 = compose_entry(V, P, 4 * r + 1),
                         m2 = compose_entry(V, P, 4 * r + 2), m3 = compose_entry(V, P, 4 * r + 3);
            q[r] = m0 * px + m1 * py + m2 * pz + m3;
            if (c == r) {  // one row each for lanes 0, 1, 2 of the object
                S.M[k][4 * r] = m0;
                S.M[k][4 * r + 1] = m1;
                S.M[k][4 * r + 2] = m2;
                S.M[k][4 * r + 3] = m3;
                S.R[k][3 * r] = (float)m0;
                S.R[k][3 * r + 1] = (float)m1;
                S.R[k][3 * r + 2] = (float)m2;
            }
        }
        const double w = -q[2];
        const double X = (double)K[0] * (q[0] / w) + (double)K[2], Y = (double)K[3] - (double)K[1] * (q[1] / w);
        safe = w >= 1.0001 * (double)a.near_plane[it.frame] && fabs(X) <= 60000.0 && fabs(Y) <= 60000.0;  // not NaN
        if (safe) {
            x0 = (int)floor(X) - 1;
            x1 = (int)ceil(X) + 1;
            y0 = (int)floor(Y) - 1;
            y1 = (int)ceil(Y) + 1;
        }
    }
    auto lo8 = [](int v) {  // over the object's eight lanes: neighbours, pairs, quads
        v = min(v, __builtin_amdgcn_update_dpp(v, v, 0xB1, 0xf, 0xf, false));
        v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x4E, 0xf, 0xf, false));
        return min(v, __builtin_amdgcn_update_dpp(v, v, 0x141, 0xf, 0xf, false));
    };
    x0 = lo8(x0);
    y0 = lo8(y0);
    x1 = -lo8(-x1);
    y1 = -lo8(-y1);
    const unsigned long long m = __ballot(safe);
    const bool all = ((m >> (lane_id() & ~7)) & 0xff) == 0xff;
    if (c == 0 && k < fi.n_obj)
        S.keep[k] = shown && !(all && (x1 < (int)it.x0 || x0 >= (int)it.x1 || y1 < (int)it.y0 || y0 >= (int)it.y1));
}

// Unit u of the wave's per-object work list: lane k holds [first, first + n) of object k.
// Returns the object (uniform) and u's position in it.
ORRB_INLINE int patch_unit(int u, int first, int n, int &chunk) {
    const int k = __builtin_ctzll(__ballot(u >= first && u < first + n));
    chunk = u - __builtin_amdgcn_readlane(first, k);
    return k;
}

struct PatchTri {
    int xa, ya, xb, yb, xc, yc;  // positive-area order
    float iwa, iwb, iwc, area;
    int i0, j0, i1, j1;          // pixel-centre range inside the patch
    int flags, id;               // edge flags (tri_flags); object << 16 | scene triangle
};

ORRB_INLINE void patch_pixel(unsigned long long *vis, const PatchTri &t, const Edges &e, int cell) {
    atomicMin(&vis[cell], vis_key(fragment_depth(e, t.iwa, t.iwb, t.iwc, t.area), t.id));
}

// Rasterize the pixels (i0 + sc + m step, j0 + sr + n step) of the triangle's range, step =
// 1 << shift.  Integer edge functions are stepped (the same integers as evaluated ones).
ORRB_INLINE void patch_raster(unsigned long long *vis, const PatchTri &t, int x0, int y0, int pw, int sc, int sr, int shift) {
    const int step = 1 << shift;
    if (!(t.flags & 8)) {
        const int b0 = (t.flags & 1) ? 0 : 1, b1 = (t.flags & 2) ? 0 : 1, b2 = (t.flags & 4) ? 0 : 1;
        EdgeStep es = edge_start(t.xa, t.ya, t.xb, t.yb, t.xc, t.yc, ((t.i0 + sc) << 8) + 128, ((t.j0 + sr) << 8) + 128);
        es.dx0 <<= shift, es.dx1 <<= shift, es.dx2 <<= shift;
        es.dy0 <<= shift, es.dy1 <<= shift, es.dy2 <<= shift;
        int row = (t.j0 + sr - y0) * pw - x0;
        for (int jj = t.j0 + sr; jj <= t.j1; jj += step, row += pw << shift) {
            int e0 = es.e0, e1 = es.e1, e2 = es.e2;
            for (int ii = t.i0 + sc; ii <= t.i1; ii += step) {
                if (((e0 - b0) | (e1 - b1) | (e2 - b2)) >= 0) {
                    Edges ed;
                    ed.e0 = (float)e0;
                    ed.e1 = (float)e1;
                    ed.e2 = (float)e2;
                    patch_pixel(vis, t, ed, row + ii);
                }
                e0 += es.dx0;
                e1 += es.dx1;
                e2 += es.dx2;
            }
            es.e0 += es.dy0;
            es.e1 += es.dy1;
            es.e2 += es.dy2;
        }
    } else {
        for (int jj = t.j0 + sr; jj <= t.j1; jj += step)
            for (int ii = t.i0 + sc; ii <= t.i1; ii += step) {
                const Edges e = edge_eval(t.xa, t.ya, t.xb, t.yb, t.xc, t.yc, (ii << 8) + 128, (jj << 8) + 128, t.flags);
                if (e.covered) patch_pixel(vis, t, e, (jj - y0) * pw + (ii - x0));
            }
    }
}

// Set-up of the triangle with snapped vertices A, B, C (PatchVerts; positive-area order of a
// front face), clipped to the patch: its pixels' number, 0 if it is invalid, a back face or
// misses the patch.
ORRB_INLINE int patch_setup(int4 A, int4 B, int4 C, int px0, int py0, int pw, int ph, PatchTri &T) {
    if (!(A.w & B.w & C.w)) return 0;
    const int xmin = min(A.x, min(B.x, C.x)), xmax = max(A.x, max(B.x, C.x));
    const int ymin = min(A.y, min(B.y, C.y)), ymax = max(A.y, max(B.y, C.y));
    T.i0 = max(ceil256(xmin - 128), px0);
    T.i1 = min(floor256(xmax - 128), px0 + pw - 1);
    T.j0 = max(ceil256(ymin - 128), py0);
    T.j1 = min(floor256(ymax - 128), py0 + ph - 1);
    if (T.i0 > T.i1 || T.j0 > T.j1) return 0;
    const bool large = max(xmax - xmin, ymax - ymin) > kSmallExtent;
    const long long area = large ? (long long)(B.x - A.x) * (C.y - A.y) - (long long)(B.y - A.y) * (C.x - A.x)
                                 : (long long)(__mul24(B.x - A.x, C.y - A.y) - __mul24(B.y - A.y, C.x - A.x));
    if (area <= 0) return 0;
    T.xa = A.x, T.ya = A.y, T.xb = B.x, T.yb = B.y, T.xc = C.x, T.yc = C.y;
    T.area = (float)area;
    T.flags = top_left(C.x - B.x, C.y - B.y) | (top_left(A.x - C.x, A.y - C.y) << 1) |
              (top_left(B.x - A.x, B.y - A.y) << 2) | (large ? 8 : 0);
    T.iwa = __int_as_float(A.z);
    T.iwb = __int_as_float(B.z);
    T.iwc = __int_as_float(C.z);
    return (T.i1 - T.i0 + 1) * (T.j1 - T.j0 + 1);
}

// The bin-overflow and survivor counters describe frames as the frame kernel renders them
// whole.  A patch adds the triangles whose first pixel it holds (so each counts once) and
// their 64 x 4 tiles to its frame's sums; the frame's last patch (or only one, which needs no
// sums) compares them with the frame kernel's limits.
ORRB_INLINE void patch_account(const RenderArgs &a, const PatchItem &it, int slot, unsigned entries, unsigned survivors,
                               const PatchLimits &limits) {
    unsigned long long sum = ((unsigned long long)survivors << 32) | entries;
    if (slot >= 0) {
        sum += 1ull << 52;
        sum += atomicAdd(a.p_account + slot, sum);
        if ((int)(sum >> 52) != it.parts) return;
    }
    const bool overflow = (unsigned)sum > (unsigned)limits.bin_max;
    stat_add(a, ORRB_STAT_BIN_OVERFLOW, overflow ? 1u : 0u);
    stat_add(a, ORRB_STAT_SURVIVOR_RESETUP, !overflow && ((sum >> 32) & 0xfffff) > (unsigned)limits.surv_max ? 1u : 0u);
}

template <bool AUX, bool G, int SHADE>
ORRB_INLINE void patch_render(const RenderArgs &a, PatchLds<G> &S, const PatchItem it) {
    const PatchLimits limits = a.p_limits[G];
    const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid) / kWave;
    const int f = it.frame;
    const FrameInfo fi = a.frames[f];
    const int n_obj = fi.n_obj;
    const bool account = a.p_account && limits.bin_max > 0 && fi.account != kUncounted;
    const int px0 = it.x0, py0 = it.y0, pw = it.x1 - it.x0, ph = it.y1 - it.y0, n_pix = pw * ph;

    // ---- 1: objects, lights, tables ----
    const PatchVerts<G> verts{S, G ? a.vtx_pos + fi.vbase : nullptr};
    if constexpr (!G) patch_cull(a, S, it, fi, tid);
    if (wave == kPW - 1) {
        if (lane < fi.n_lights) {
            if constexpr (SHADE == 1 || SHADE == 3) {
                frame_light(a, f, fi.light_begin, lane, S.light, S.ltype, S.spot);
            } else if constexpr (SHADE != 4) {
                const int l = fi.light_begin + lane;
                S.light[lane] = view_light(a.view + 12 * (int64_t)f, a.light_vec + 3 * (int64_t)l, a.light_type[l],
                                           a.light_intensity[l]);
                S.ltype[lane] = a.light_type[l];
            }
        }
        if (lane < 2) S.account[lane] = 0u;
        if (lane == 2) S.n_big = S.next_big = 0;
    }
    // lane k of every wave: scene object k (G: of the current 64 objects)
    int nv = 0, nt = 0, mvb = 0, mtb = 0, tbase = 0;
    if (!G && lane < n_obj) {
        const ObjInfo &ob = a.objs[fi.obj_begin + lane];
        nv = ob.n_verts;
        nt = ob.n_tris;
        mvb = ob.mesh_vbegin;
        mtb = ob.mesh_tbegin;
        tbase = ob.scene_tbase;
    }
    if constexpr (G) {
        if (tid < n_obj) {
            const int o = fi.obj_begin + tid;
            const ObjInfo &ob = a.objs[o];
            S.tbase[tid] = ob.scene_tbase;
            S.mtb[tid] = ob.mesh_tbegin;
            S.mvb[tid] = ob.mesh_vbegin;
            S.vbase[tid] = ob.scene_vbase;
            S.seg[tid] = a.seg[o];
            S.mat[tid] = object_material(a, o);
        }
        for (int e = tid; e < 3 * n_obj; e += kPT) {
            const float4 r = a.obj_rot[3 * (int64_t)fi.oi_base + e];
            float *R = S.R[e / 3] + 3 * (e % 3);
            R[0] = r.x;
            R[1] = r.y;
            R[2] = r.z;
        }
    } else if (wave == kPW - 2 && lane < n_obj) {
        const int o = fi.obj_begin + lane;
        S.tbase[lane] = tbase;
        S.mtb[lane] = mtb;
        S.mvb[lane] = mvb;
        S.seg[lane] = a.seg[o];
        S.mat[lane] = object_material(a, o);
    }
    for (int p = 2 * tid; p < n_pix; p += 2 * kPT)  // (one key past an odd count is still in the array)
        *reinterpret_cast<uint4 *>(&S.vis[p]) = make_uint4(~0u, ~0u, ~0u, ~0u);
    __syncthreads();

    // the kept objects' work lists: 64 vertices, or 64 triangles, of one object per unit
    int tu = 0, tfirst = 0, t_units = 0, vb = 0;
    if constexpr (!G) {
        const bool keep = lane < n_obj && S.keep[lane] != 0;
        tu = keep ? (nt + kWave - 1) / kWave : 0;
        const int ti = wave_scan_add(tu);
        tfirst = ti - tu;
        t_units = __builtin_amdgcn_readlane(ti, kWave - 1);
        vb = wave_scan_add(keep ? nv : 0) - nv;
        if (wave == 0 && keep) S.vbase[lane] = vb;
    }

    // ---- 2: vertices (the next unit's positions are loaded before this one's are used) ----
    if constexpr (!G) {
        const bool keep = tu > 0;
        const int vu = keep ? (nv + kWave - 1) / kWave : 0, vi = wave_scan_add(vu), vfirst = vi - vu;
        const int v_units = __builtin_amdgcn_readlane(vi, kWave - 1);
        const float *K = a.intr + 4 * (int64_t)f;
        const double fx = K[0], fy = K[1], cx = K[2], cy = K[3], nearp = a.near_plane[f];
        unsigned n_near = 0, n_guard = 0;
        int kn = 0, vn = 0;
        float4 pn = make_float4(0.f, 0.f, 0.f, 0.f);
        auto fetch = [&](int u) {
            int chunk;
            kn = patch_unit(u, vfirst, vu, chunk);
            vn = chunk * kWave + lane;
            const int n = __builtin_amdgcn_readlane(nv, kn);
            if (vn >= n) vn = -1;
            else pn = a.mesh_pos[__builtin_amdgcn_readlane(mvb, kn) + vn];
        };
        if (wave < v_units) fetch(wave);
        for (int u = wave; u < v_units; u += kPW) {
            const int k = kn, v = vn;
            const float4 p = pn;
            if (u + kPW < v_units) fetch(u + kPW);
            double M[12];
#pragma unroll
            for (int q = 0; q < 12; ++q) M[q] = S.M[k][q];
            if (v >= 0) {
                const Snapped s = snap_vertex(M, p, fx, fy, cx, cy, nearp);
                const int at = __builtin_amdgcn_readlane(vb, k) + v;
                S.XY[at] = make_int2(s.valid ? s.X : kInvalidX, s.Y);
                S.iw[at] = s.iw;
                n_near += s.cull == 1;
                n_guard += s.cull == 2;
            }
        }
        if ((it.x0 | it.y0) == 0) {  // the frame's first patch counts for the frame
            stat_add(a, ORRB_STAT_NEAR_VERTICES, n_near);
            stat_add(a, ORRB_STAT_GUARD_VERTICES, n_guard);
        }
    }
    // first triangles on their way before the barrier
    int kn = 0, tn = -1;
    int4 trn = make_int4(0, 0, 0, 0);
    auto tfetch = [&](int u) {
        int chunk;
        kn = patch_unit(u, tfirst, tu, chunk);
        tn = chunk * kWave + lane;
        if (tn >= __builtin_amdgcn_readlane(nt, kn)) tn = -1;
        else trn = a.mesh_tri[__builtin_amdgcn_readlane(mtb, kn) + tn];
    };
    if constexpr (!G) {
        if (wave < t_units) tfetch(wave);
        __syncthreads();
    }

    // ---- 3: triangles ----
    // entry q of a list of n: set up (again) and rasterize, by (sc, sr, shift) of patch_raster
    auto raster = [&](int q, int n, const unsigned *list, int sc, int sr, int shift) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (q < n) {
            const unsigned e = list[q];
            const int k = (int)(e >> 16), t = (int)(e & 0xffffu), base = S.vbase[k];
            const int4 tri = a.mesh_tri[S.mtb[k] + t];
            PatchTri T;
            if (patch_setup(verts.get(base + tri.x), verts.get(base + tri.z), verts.get(base + tri.y), px0, py0, pw, ph,
                            T) > 0) {
                T.id = (k << 16) | (S.tbase[k] + t);
                patch_raster(S.vis, T, px0, py0, pw, sc, sr, shift);
            }
        }
        __builtin_amdgcn_wave_barrier();
    };
    unsigned *buf = S.small[wave];
    int n_buf = 0;
    unsigned entries = 0, survivors = 0;
    int group = 0;  // first of the lanes' objects
    do {
        if constexpr (G) {
            const bool in = group + lane < n_obj;
            const ObjInfo &ob = a.objs[fi.obj_begin + (in ? group + lane : 0)];
            const int4 bb = in ? a.obj_bbox[fi.oi_base + group + lane] : make_int4(1, 1, 0, 0);
            const bool keep = bb.x <= bb.z && bb.y <= bb.w && bb.z >= px0 && bb.x < px0 + pw && bb.w >= py0 && bb.y < py0 + ph;
            nt = ob.n_tris;
            mtb = ob.mesh_tbegin;
            vb = ob.scene_vbase;
            tu = keep ? (nt + kWave - 1) / kWave : 0;
            const int ti = wave_scan_add(tu);
            tfirst = ti - tu;
            t_units = __builtin_amdgcn_readlane(ti, kWave - 1);
            if (wave < t_units) tfetch(wave);
        }
        for (int u = wave; u < t_units; u += kPW) {
            const int k = kn, t = tn;
            const int4 tri = trn;
            if (u + kPW < t_units) tfetch(u + kPW);
            const int base = __builtin_amdgcn_readlane(vb, k);
            PatchTri T;
            const int n = t >= 0 ? patch_setup(verts.get(base + tri.x), verts.get(base + tri.z), verts.get(base + tri.y),
                                               px0, py0, pw, ph, T)
                                 : 0;
            if (account && n > 0) {
                const int xmin = min(T.xa, min(T.xb, T.xc)), xmax = max(T.xa, max(T.xb, T.xc));
                const int ymin = min(T.ya, min(T.yb, T.yc)), ymax = max(T.ya, max(T.yb, T.yc));
                const int i0 = max(ceil256(xmin - 128), 0), j0 = max(ceil256(ymin - 128), 0);
                if (i0 >= px0 && j0 >= py0) {  // its first pixel lies here
                    const int i1 = min(floor256(xmax - 128), fi.width - 1), j1 = min(floor256(ymax - 128), fi.height - 1);
                    entries += (unsigned)((i1 / 64 - i0 / 64 + 1) * (j1 / 4 - j0 / 4 + 1));
                    ++survivors;
                }
            }
            const unsigned entry = ((unsigned)(group + k) << 16) | (unsigned)t;
            bool small = n > 0;
            const unsigned long long mb = __ballot(n > kPOwn);
            if (mb) {
                int at = 0;
                if (lane == 0) at = atomicAdd(&S.n_big, __popcll(mb));
                at = __builtin_amdgcn_readlane(at, 0) + lanes_below(mb);
                if (n > kPOwn && at < kPBig) {
                    S.big[at] = entry;
                    small = false;
                }
            }
            const unsigned long long ms = __ballot(small);
            if (small) buf[n_buf + lanes_below(ms)] = entry;
            n_buf += __popcll(ms);
            if (n_buf >= kWave) {
                n_buf -= kWave;
                raster(n_buf + lane, n_buf + kWave, buf, 0, 0, 0);
            }
        }
        group += kWave;
    } while (G && group < n_obj);
    if (n_buf > 0) raster(lane, n_buf, buf, 0, 0, 0);
    __syncthreads();
    // queued triangles, four per wave and step
    const int n_big = min(S.n_big, kPBig);
    while (true) {
        int first = 0;
        if (lane == 0) first = atomicAdd(&S.next_big, 4);
        first = __builtin_amdgcn_readlane(first, 0);
        if (first >= n_big) break;
        raster(first + (lane >> 4), n_big, S.big, lane & 3, (lane >> 2) & 3, 2);
    }
    if (account) {
        if (entries) atomicAdd(&S.account[0], entries);
        if (survivors) atomicAdd(&S.account[1], survivors);
    }
    __syncthreads();
    if (account && tid == 0) patch_account(a, it, fi.account, S.account[0], S.account[1], limits);

    // ---- 4: shade and store ----
    const CamF cam = frame_camera(a, f);
    const int64_t HW = (int64_t)fi.width * fi.height, po = fi.pixel_offset;
    const float rpw = 1.0f / (float)pw;
    const bool fused = AUX && a.out_rgb8;
    PostFrame pq;
    float3 graded_bg = f3(0.f, 0.f, 0.f);
    if (fused) {
        pq = post_frame(a, f);
        graded_bg = post_grade(pq, 0.f, 0.f, 0.f);
    }
    // Pixel (li, lj) of the patch with its key: shaded if covered, stored, and the lane's
    // Tracker record (-1: none).
    auto finish = [&](int li, int lj, unsigned long long key) __attribute__((always_inline)) {
        const int i = px0 + li, j = py0 + lj;
        const bool cov = key != kEmptyKey;
        PixelOut o = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        float z = 0.f;
        int rec = -1, segv = -1, tri = -1;
        if (cov) {
            tri = (int)(unsigned)(key & 0xffffu);
            const int k = (int)(unsigned)((key >> 16) & 0xffu);
            z = __uint_as_float((unsigned)(key >> 32));
            key &= ~0xffff0000ull;
            segv = S.seg[k];
            rec = fi.track_base + k;
            if constexpr (SHADE != 4) {
                constexpr bool kSpot = (SHADE & 1) != 0, kMat = (SHADE & 2) != 0;
                const int4 tv = a.mesh_tri[S.mtb[k] + (tri - S.tbase[k])];
                const int m = S.mvb[k], b = S.vbase[k];
                MatTex mt;
                if constexpr (kMat) mt = mat_inputs(a, fi.obj_begin + k, m, tv);
                const int4 A = verts.get(b + tv.x), B = verts.get(b + tv.z), C = verts.get(b + tv.y);
                o = shade_pixel<kSpot, kMat>(A.x, A.y, B.x, B.y, C.x, C.y, __int_as_float(A.z), __int_as_float(B.z),
                                             __int_as_float(C.z), a.mesh_nrm[m + tv.x], a.mesh_nrm[m + tv.z],
                                             a.mesh_nrm[m + tv.y], S.R[k], i, j, z, cam, S.light, S.ltype, fi.n_lights,
                                             S.mat[k], S.spot, a.shadow_maps, a.shadow_res, &mt, a.tex_texels,
                                             a.tex_info);
            }
        }
        const int64_t pix = (int64_t)j * fi.width + i;
        store_pixel(a, po, HW, pix, o, z, segv, tri, key);
        if (fused)
            store_rgb8(a, pq, po, HW, pix, i, j, __ballot(cov) ? post_grade(pq, o.r0, o.r1, o.r2) : graded_bg);
        return rec;
    };
    auto track = [&](int rec, int li, int lj) {  // every lane of the wave takes part
        if (fi.width <= 1024 && fi.height <= 1024)
            track_wave<true>(a.out_track, rec, px0 + li, py0 + lj);
        else
            track_wave<false>(a.out_track, rec, px0 + li, py0 + lj);
    };
    // Spot lights and textures cost enough per pixel to collect the wave's covered pixels
    // (patch column | row << 16) and shade them by full waves, the background being stored at
    // once: 144 spot-lit, textured frames of 128 x 128 139 us without, 124 us with; plain
    // shading is faster without (120 frames of 177 x 131 81 us, 84 us with).
    constexpr bool kCollect = SHADE >= 1 && SHADE <= 3;
    int n_cov = 0;
    auto collected = [&](int q, int n) __attribute__((always_inline)) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        int rec = -1, li = 0, lj = 0;
        if (q < n) {
            li = (int)(buf[q] & 0xffffu);
            lj = (int)(buf[q] >> 16);
            rec = finish(li, lj, S.vis[lj * pw + li]);
        }
        if (AUX && a.out_track) track(rec, li, lj);
        __builtin_amdgcn_wave_barrier();
    };
    // (with kCollect, until the collected pixels are done too: one copy of the shading code)
    for (int p0 = wave * kWave; p0 < n_pix || n_cov > 0; p0 += kPT) {
        const int p = p0 + lane;
        int rec = -1, li = 0, lj = 0;
        bool cov = false;
        if (p < n_pix) {
            lj = div_small(p, pw, rpw);
            li = p - lj * pw;
            const unsigned long long key = S.vis[p];
            if constexpr (!kCollect) {
                rec = finish(li, lj, key);
            } else {
                cov = key != kEmptyKey;
                if (!cov) {
                    const int64_t pix = (int64_t)(py0 + lj) * fi.width + px0 + li;
                    store_pixel(a, po, HW, pix, PixelOut{0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, 0.f, -1, -1, kEmptyKey);
                    if (fused) store_rgb8(a, pq, po, HW, pix, px0 + li, py0 + lj, graded_bg);
                }
            }
        }
        if constexpr (kCollect) {
            const unsigned long long m = __ballot(cov);
            if (cov) buf[n_cov + lanes_below(m)] = (unsigned)li | ((unsigned)lj << 16);
            n_cov += __popcll(m);
            if (n_cov >= kWave || (n_cov > 0 && p0 + kPT >= n_pix)) {
                const int n = min(n_cov, kWave);
                n_cov -= n;
                collected(n_cov + lane, n_cov + n);
            }
        } else if (AUX && a.out_track) {
            track(rec, li, lj);
        }
    }
}

// KIND: every patch's scene is held in LDS (0) or larger (1), or either (2, FrameInfo::mode 2):
// one launch for both halves of a mixed batch, whose patches share out the CUs between them
// (60 mixed frames: 88 us
// in two launches, 73 in one; 231: 197 and 178).
template <bool AUX, int KIND, int SHADE>
__global__ __launch_bounds__(kPT) void k_patch(RenderArgs a) {
    __shared__ union {
        PatchLds<KIND == 1> one;
        PatchLds<KIND != 0> larger;
    } S;
    const PatchItem it = a.pitems[blockIdx.x];
    if constexpr (KIND != 2) {
        patch_render<AUX, KIND == 1, SHADE>(a, S.one, it);
    } else {
        if (a.frames[it.frame].mode == 2)
            patch_render<AUX, true, SHADE>(a, S.larger, it);
        else
            patch_render<AUX, false, SHADE>(a, S.one, it);
    }
}

// What must hold before the patches start: their frames' counter sums at 0 and Tracker
// records empty (patches add to them in any order).  One workgroup per patch; each frame's
// first patch does the frame's.
__global__ __launch_bounds__(kWave) void k_patch_prepare(RenderArgs a) {
    const PatchItem it = a.pitems[blockIdx.x];
    if ((it.x0 | it.y0) != 0) return;
    const FrameInfo fi = a.frames[it.frame];
    if (a.p_account && fi.account >= 0 && threadIdx.x == 0) a.p_account[fi.account] = 0ull;
    const int k = threadIdx.x;
    if (!a.out_track || k >= fi.n_obj || fi.n_obj > kPOMax) return;  // (larger scenes: k_vertex)
    const float *V = a.view + 12 * (int64_t)it.frame, *P = a.pose + 12 * (int64_t)(fi.obj_begin + k);
    const float *K = a.intr + 4 * (int64_t)it.frame;
    track_init(a.out_track + fi.track_base + k, compose_entry(V, P, 3), compose_entry(V, P, 7), compose_entry(V, P, 11),
               K[0], K[1], K[2], K[3]);
}

// A launch holds fewer than 2^32 threads (beyond, the grid is cut short without an error).
constexpr int kPLaunch = 1 << 21;  // most patches of one launch
int patch_launches(int64_t n_patches) { return (int)((n_patches + kPLaunch - 1) / kPLaunch); }

static hipError_t launch_patches(const RenderArgs &a, int kind, hipStream_t stream) {
    const bool aux = a.out_alpha || a.out_track || a.out_rgb8;
    const dim3 g(a.n_pitems), b(kPT);
#define ORRB_PATCH_KIND(KIND_, SHADE_)                                                               \
    do {                                                                                             \
        if (aux) hipLaunchKernelGGL((k_patch<true, KIND_, SHADE_>), g, b, 0, stream, a);             \
        else hipLaunchKernelGGL((k_patch<false, KIND_, SHADE_>), g, b, 0, stream, a);                \
    } while (0)
#define ORRB_PATCH(SHADE_)                                                                           \
    do {                                                                                             \
        if (kind == 2) ORRB_PATCH_KIND(2, SHADE_);                                                   \
        else if (kind == 1) ORRB_PATCH_KIND(1, SHADE_);                                              \
        else ORRB_PATCH_KIND(0, SHADE_);                                                             \
    } while (0)
    switch (a.shade_mode) {
        case 4: ORRB_PATCH(4); break;
        case 1: ORRB_PATCH(1); break;
        case 2: ORRB_PATCH(2); break;
        case 3: ORRB_PATCH(3); break;
        default: ORRB_PATCH(0);
    }
#undef ORRB_PATCH
#undef ORRB_PATCH_KIND
    return hipGetLastError();
}

// a.pitems: the patches of scenes held in LDS (kind 0), of larger ones, whose vertices
// k_vertex has written (1; it also starts their Tracker records), or of both (2).
hipError_t launch_patch(const RenderArgs &a, int kind, hipStream_t stream) {
    const bool prepare = (a.p_account && a.n_account > 0) || (a.out_track && kind != 1);
    RenderArgs part = a;
    for (int patches = prepare ? 0 : 1; patches < 2; ++patches)  // every frame is prepared before its first patch
        for (int64_t k = 0; k < a.n_pitems; k += kPLaunch) {
            part.pitems = a.pitems + k;
            part.n_pitems = (int32_t)(a.n_pitems - k < kPLaunch ? a.n_pitems - k : kPLaunch);
            if (!patches) hipLaunchKernelGGL(k_patch_prepare, dim3(part.n_pitems), dim3(kWave), 0, stream, part);
            const hipError_t e = patches ? launch_patches(part, kind, stream) : hipGetLastError();
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

}  // namespace orrb
