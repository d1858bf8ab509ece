// Adjoint of the shading over a fixed visibility buffer (HIP, gfx950).
//
// Given the visibility keys of a forward render and dL/d(rgb), computes dL/d of the
// per-object albedo (3), roughness and specular, the per-light world vector (3: the
// position of a point light, the direction vector of a directional light) and
// intensity, and the per-frame exposure.  Visibility is fixed: none of these
// parameters moves geometry.
//
//   k_grad_tile    one workgroup per (frame, 32x32 tile): list the covered pixels, then,
//                  64 of them per wave and pass, rebuild each fragment from its key
//                  (exact edge functions of the snapped vertices, perspective-correct
//                  normal, view-space position: the forward's own fp32 arithmetic),
//                  evaluate the analytic adjoint of the shading in fp32 and sum in FP64:
//                  per light and per distinct object of the pass over the wave, then the
//                  four waves in order.  The tile's sums go to a per-tile FP64 partial
//                  vector; a tile without a fragment writes none and is marked empty.
//   k_grad_reduce  per (scene, 64 parameters): the sixteen waves sum interleaved parts of
//                  the scene's non-empty tiles' partials, then combine in order, and
//                  write the gradient.
// No floating-point atomics: repeated calls are bit-identical.
#include "orrb_primitives.h"

namespace orrb {

constexpr int kGTile = 32;
constexpr int kGPix = kGTile * kGTile;      // pixels per tile
constexpr int kGPer = kGPix / kBlock;       // pixels per thread
constexpr int kGWaves = kBlock / kWave;
constexpr int kGMaxObj = 1024;              // objects per scene supported by the adjoint
constexpr int kGPresent = 64;               // distinct objects per tile summed in one round
constexpr int kGChunk = 64;                 // parameters per reduce workgroup
constexpr int kRBlock = 1024;               // threads of a reduce workgroup
constexpr int kRWaves = kRBlock / kWave;

struct GradLds {
    float4 light[kMaxLights];     // view space: point position / unit direction to the light; w = intensity
    float light_qn[kMaxLights];   // directional: |R_V u| before normalization
    int light_type[kMaxLights];
    int o_tbase[kGMaxObj];        // scene triangle base of each object (object lookup)
    unsigned list[kGPix];         // covered pixels: pixel in the tile | local object << 10
    unsigned char present[kGMaxObj];
    unsigned short slot_of[kGMaxObj];  // present objects: their compact slot
    double oacc[kGWaves][kGPresent][5];               // per-wave object sums
    double wacc[kGWaves][4 * kMaxLights + 1];         // per-wave light / exposure sums
    int count[kGWaves];
    int n_present;
};

// Shift of a double across lanes by a DPP control (both halves moved alike; lanes
// without a source get 0.0).
template <int CTRL, int ROW_MASK>
ORRB_INLINE double dpp_d(double x) {
    const unsigned long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, ROW_MASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, ROW_MASK, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// Sum over the 16 lanes of a row, in every lane (rotations by 8, 4, 2 and 1).
ORRB_INLINE double row_sum(double x) {
    x += dpp_d<0x128, 0xf>(x);
    x += dpp_d<0x124, 0xf>(x);
    x += dpp_d<0x122, 0xf>(x);
    x += dpp_d<0x121, 0xf>(x);
    return x;
}

// a in lanes 0-31 plus a in lanes 32-63 in the low half, the same of b in the high half:
// the half-wave swap exchanges a's upper lanes with b's lower ones.
ORRB_INLINE double fold32(double a, double b) {
    const unsigned long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    return __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0])) +
           __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}

// The same for neighbouring 16-lane rows: a's row sums in rows 0 and 2, b's in 1 and 3.
ORRB_INLINE double fold16(double a, double b) {
    const unsigned long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    return __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0])) +
           __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}

// Sums over the wave of four values at once, in a fixed order: row r of the result (16
// lanes, all alike) holds the sum of value r.  Folding different values into the halves
// and rows takes 7 FP64 additions where four separate sums take 24.
ORRB_INLINE double wave_sum4(double v0, double v1, double v2, double v3) {
    return row_sum(fold16(fold32(v0, v2), fold32(v1, v3)));
}

// Sum over the wave of one value, in every lane.
ORRB_INLINE double wave_sum(double x) {
    x = fold32(x, x);
    return row_sum(fold16(x, x));
}

// Work item of workgroup b.  Consecutive workgroups go to the eight XCDs in turn: each XCD gets
// runs of as many consecutive items as a frame has on average, so that a frame's tiles find
// its snapped vertices in one L2 and no XCD gets the middle tile of every frame (192 hand
// frames of 100 x 100 or 128 x 128, 16 tiles each: 96 and 80 us a call in plain order, 68 and 67
// so; others level or 1-4 % faster).  Items past the last full set of runs keep their place.
ORRB_INLINE int grad_item(const GradArgs &g, int b) {
    const int run = g.n_gitems / g.n_frames, set = 8 * run;
    if (run < 2 || b >= g.n_gitems / set * set) return b;
    const int s = b / set, r = b - s * set;
    return s * set + (r & 7) * run + (r >> 3);
}

// What bounds it: VALU issue of the adjoint itself (about 250 instructions per covered
// pixel and light) and the FP64 sums over the wave.  Working through the list of covered
// pixels (hand scenes cover about a quarter of a busy frame's pixels) keeps the lanes
// full, and sums of four values fold together; 192 frames of 200 x 200: 241 us with one
// pass per 64 tile pixels and a separate sum per value, 66 us so.
__global__ __launch_bounds__(kBlock) void k_grad_tile(GradArgs g) {
    __shared__ GradLds S;
    const RenderArgs &a = g.r;
    const int item = grad_item(g, blockIdx.x);
    const int2 it = g.gitems[item];
    const int f = it.x;
    const FrameInfo fi = a.frames[f];
    const int W = fi.width, H = fi.height;
    const int ntx = (W + kGTile - 1) / kGTile;
    const int x0 = (it.y % ntx) * kGTile, y0 = (it.y / ntx) * kGTile;
    const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    const int nl = fi.n_lights, n_obj = fi.n_obj;
    const int64_t HW = (int64_t)W * H, po = fi.pixel_offset;

    // the thread's pixels: each wave reads 16 x 4 blocks, so that the 64 pixels of a pass
    // lie close together and show few objects
    int tri[kGPer];
#pragma unroll
    for (int q = 0; q < kGPer; ++q) {
        const int blk = kGPer * wave + q;  // 2 x 8 blocks
        const int i = x0 + (blk & 1) * 16 + (lane & 15), j = y0 + (blk >> 1) * 4 + (lane >> 4);
        unsigned long long key = kEmptyKey;
        if (i < W && j < H) key = g.vis[po + (int64_t)j * W + i];
        tri[q] = key == kEmptyKey ? -1 : (int)(unsigned)(key & 0xffffffffu);
    }
    int n = 0;
#pragma unroll
    for (int q = 0; q < kGPer; ++q) n += __popcll(__ballot(tri[q] >= 0));
    if (lane == 0) S.count[wave] = n;
    for (int k = tid; k < n_obj; k += kBlock) {
        S.o_tbase[k] = a.objs[fi.obj_begin + k].scene_tbase;
        S.present[k] = 0;
    }
    __syncthreads();
    int n_list = 0, base = 0;
#pragma unroll
    for (int w = 0; w < kGWaves; ++w) {
        if (w < wave) base += S.count[w];
        n_list += S.count[w];
    }
    if (tid == 0) g.live[item] = n_list > 0;
    if (n_list == 0) return;  // the reduction skips the tile

    const float *V = a.view + 12 * (int64_t)f;
    if (tid < nl) {
        const int l = fi.light_begin + tid;
        const float *u = a.light_vec + 3 * (int64_t)l;
        const int type = a.light_type[l];
        double q[3];
        for (int r = 0; r < 3; ++r) {
            const double d = (double)V[r * 4 + 0] * u[0] + (double)V[r * 4 + 1] * u[1] + (double)V[r * 4 + 2] * u[2];
            q[r] = type == 0 ? d + (double)V[r * 4 + 3] : -d;
        }
        double qn = 1.0;
        if (type != 0) {
            qn = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2]);
            for (int r = 0; r < 3; ++r) q[r] /= qn;
        }
        // the forward's view-space light (view_light), so the fragment terms agree
        S.light[tid] = view_light(V, u, type, a.light_intensity[l]);
        S.light_qn[tid] = (float)qn;
        S.light_type[tid] = type;
    }
    for (int k = tid; k < kGWaves * (4 * kMaxLights + 1); k += kBlock) (&S.wacc[0][0])[k] = 0.0;
#pragma unroll
    for (int q = 0; q < kGPer; ++q) {
        const bool c = tri[q] >= 0;
        const unsigned long long m = __ballot(c);
        if (c) {
            const int blk = kGPer * wave + q;
            const int li = (blk & 1) * 16 + (lane & 15), lj = (blk >> 1) * 4 + (lane >> 4);
            const int k = find_slot(S.o_tbase, n_obj, tri[q]);
            S.list[base + lanes_below(m)] = (unsigned)(lj * kGTile + li) | ((unsigned)k << 10);
            S.present[k] = 1;
        }
        base += __popcll(m);
    }
    __syncthreads();

    // compact slots of the objects present in the tile (wave 0: a scan over the flags)
    if (wave == 0) {
        int nb = 0;
        for (int k0 = 0; k0 < n_obj; k0 += kWave) {
            const int k = k0 + lane;
            const bool pr = k < n_obj && S.present[k];
            const unsigned long long mk = __ballot(pr);
            if (pr) S.slot_of[k] = (unsigned short)(nb + lanes_below(mk));
            nb += __popcll(mk);
        }
        if (lane == 0) S.n_present = nb;
    }
    __syncthreads();
    const int n_present = S.n_present;
    double *part = g.partial + g.gitem_pbase[item];
    const CamF cam = frame_camera(a, f);
    const float e = cam.expo;

    // kGPresent object slots per round (one round unless a tile shows more objects; the
    // light and exposure sums are taken in the first)
    for (int s0 = 0; s0 < n_present; s0 += kGPresent) {
        const int ns = min(n_present - s0, kGPresent);
        for (int k = tid; k < kGWaves * kGPresent * 5; k += kBlock)
            if (k % (kGPresent * 5) < 5 * ns) (&S.oacc[0][0][0])[k] = 0.0;
        __syncthreads();
        for (int c0 = wave * kWave; c0 < n_list; c0 += kBlock) {  // wave-uniform
            const int c = c0 + lane;
            float gc0 = 0.f, gc1 = 0.f, gc2 = 0.f;
            float3 n3 = f3(0.f, 0.f, 1.f), pp = f3(0.f, 0.f, -1.f), v = f3(0.f, 0.f, 1.f);
            float al0 = 0.f, al1 = 0.f, al2 = 0.f, r = 1.f, ks = 0.f, m = 0.f, G = 0.f;
            int obj_local = -1;
            if (c < n_list) {
                const unsigned entry = S.list[c];
                const int p = entry & (kGPix - 1);
                const int i = x0 + (p & (kGTile - 1)), j = y0 + p / kGTile;
                const int64_t pix = (int64_t)j * W + i;
                gc0 = g.grad_rgb[3 * po + pix];
                gc1 = g.grad_rgb[3 * po + HW + pix];
                gc2 = g.grad_rgb[3 * po + 2 * HW + pix];
                if (gc0 != 0.f || gc1 != 0.f || gc2 != 0.f) {
                    obj_local = (int)(entry >> 10);
                    const unsigned long long key = g.vis[po + pix];
                    const int tr = (int)(unsigned)(key & 0xffffffffu);
                    const float z = __uint_as_float((unsigned)(key >> 32));
                    const int o = fi.obj_begin + obj_local;
                    const ObjInfo ob = a.objs[o];
                    const int4 tv = a.mesh_tri[ob.mesh_tbegin + (tr - ob.scene_tbase)];
                    const int64_t vb = fi.vbase + ob.scene_vbase;
                    const int4 pa = a.vtx_pos[vb + tv.x], pb = a.vtx_pos[vb + tv.z], pc = a.vtx_pos[vb + tv.y];
                    const Edges ed = edge_eval(pa.x, pa.y, pb.x, pb.y, pc.x, pc.y, (i << 8) + 128, (j << 8) + 128,
                                               extent_flag(pa.x, pa.y, pb.x, pb.y, pc.x, pc.y));
                    const float t0 = ed.e0 * __int_as_float(pa.z), t1 = ed.e1 * __int_as_float(pb.z),
                                t2 = ed.e2 * __int_as_float(pc.z);
                    const float4 na = a.mesh_nrm[ob.mesh_vbegin + tv.x], nb = a.mesh_nrm[ob.mesh_vbegin + tv.z],
                                 nc = a.mesh_nrm[ob.mesh_vbegin + tv.y];
                    const float4 *rot = a.obj_rot + 3 * (int64_t)(fi.oi_base + obj_local);
                    const float4 R0 = rot[0], R1 = rot[1], R2 = rot[2];
                    const float R[9] = {R0.x, R0.y, R0.z, R1.x, R1.y, R1.z, R2.x, R2.y, R2.z};
                    {
#pragma clang fp contract(off)
                        const float4 no = make_float4(fmaf(t0, na.x, fmaf(t1, nb.x, t2 * nc.x)),
                                                      fmaf(t0, na.y, fmaf(t1, nb.y, t2 * nc.y)),
                                                      fmaf(t0, na.z, fmaf(t1, nb.z, t2 * nc.z)), 0.f);
                        n3 = rotate_normal(R, no);
                        pp = f3(z * (((float)i + 0.5f - cam.cx) * cam.ifx), -z * (((float)j + 0.5f - cam.cy) * cam.ify), -z);
                        const float pinv = rsqrtf(dot3(pp, pp));
                        v = f3(-pp.x * pinv, -pp.y * pinv, -pp.z * pinv);
                    }
                    r = a.roughness[o];
                    ks = a.specular[o];
                    m = 2.0f * __builtin_amdgcn_rcpf(r * r) - 2.0f;
                    al0 = a.albedo[3 * o + 0];
                    al1 = a.albedo[3 * o + 1];
                    al2 = a.albedo[3 * o + 2];
                    G = gc0 + gc1 + gc2;
                }
            }
            const bool frag = obj_local >= 0;
            float U0 = 0.f, U1 = 0.f, U2 = 0.f, sAnd = 0.f, sAnds = 0.f, sAndsln = 0.f;
            for (int l = 0; l < nl; ++l) {  // wave-uniform trip count
#pragma clang fp contract(off)
                float gq0 = 0.f, gq1 = 0.f, gq2 = 0.f, gI = 0.f;
                const bool point = S.light_type[l] == 0;
                if (frag) {
                    const float4 Lq = S.light[l];
                    float3 ld;
                    float D = 1.f, dist = 1.f, A;
                    if (point) {
                        const float3 d = f3(Lq.x - pp.x, Lq.y - pp.y, Lq.z - pp.z);
                        D = dot3(d, d);
                        const float dinv = rsqrtf(D);
                        dist = D * dinv;
                        ld = f3(d.x * dinv, d.y * dinv, d.z * dinv);
                        A = Lq.w * __builtin_amdgcn_rcpf(fmaxf(D, 1e-4f));
                    } else {
                        ld = f3(Lq.x, Lq.y, Lq.z);
                        A = Lq.w;
                    }
                    const float ndl = dot3(n3, ld);
                    if (ndl > 0.f) {  // max(0, n.l) inactive: no contribution, sub-gradient 0
                        const float3 hh = f3(ld.x + v.x, ld.y + v.y, ld.z + v.z);
                        const float H2 = dot3(hh, hh);
                        float s = 0.f, ndh = 0.f, lnh = 0.f, hinv = 0.f;
                        float3 h = f3(0.f, 0.f, 0.f), w = f3(0.f, 0.f, 0.f);
                        if (H2 >= 1e-12f) {
                            hinv = rsqrtf(H2);
                            h = f3(hh.x * hinv, hh.y * hinv, hh.z * hinv);
                            const float3 dd = f3(n3.x - h.x, n3.y - h.y, n3.z - h.z);
                            const float u = 0.5f * dot3(dd, dd);  // 1 - n.h, without cancellation
                            if (u < 1.0f) {
                                ndh = 1.0f - u;
                                const float l2 = log2_one_minus(u);
                                s = m == 0.f ? 1.0f : __builtin_amdgcn_exp2f(m * l2);
                                lnh = l2 * 0.69314718055994531f;
                                // n - (n.h) h = (n - h) + u h
                                w = f3(dd.x + u * h.x, dd.y + u * h.y, dd.z + u * h.z);
                            }
                        }
                        const float c0 = fmaf(ks, s, al0), c1 = fmaf(ks, s, al1), c2 = fmaf(ks, s, al2);
                        const float An = A * ndl;
                        U0 = fmaf(An, c0, U0);
                        U1 = fmaf(An, c1, U1);
                        U2 = fmaf(An, c2, U2);
                        const float Gh = gc0 * c0 + gc1 * c1 + gc2 * c2;
                        sAnd += An;
                        sAnds += An * s;
                        if (ndh > 0.f) sAndsln += An * s * lnh;
                        // n.h^(m - 1) = s / n.h; hl = |l + v| = 1 / hinv
                        const float spec = (ndh > 0.f && m != 0.f) ? e * G * An * ks * m * (s / ndh) * hinv : 0.f;
                        if (point) {
                            const float Ainv = __builtin_amdgcn_rcpf(fmaxf(D, 1e-4f));
                            gI = e * Gh * ndl * Ainv;
                            if (D > 1e-4f) {  // d A / d q through 1 / D
                                const float kk = e * Gh * ndl * (-2.0f * Lq.w) * Ainv * Ainv;
                                gq0 = kk * (ld.x * dist);
                                gq1 = kk * (ld.y * dist);
                                gq2 = kk * (ld.z * dist);
                            }
                            const float dinv = 1.0f / dist;
                            const float kn = e * Gh * A * dinv;
                            gq0 += kn * (n3.x - ndl * ld.x);
                            gq1 += kn * (n3.y - ndl * ld.y);
                            gq2 += kn * (n3.z - ndl * ld.z);
                            if (spec != 0.f) {
                                const float lw = dot3(ld, w), ks2 = spec * dinv;
                                gq0 += ks2 * (w.x - lw * ld.x);
                                gq1 += ks2 * (w.y - lw * ld.y);
                                gq2 += ks2 * (w.z - lw * ld.z);
                            }
                        } else {
                            // directional: l = a / |a| with a = -R_V u reaches the shade through
                            // n.l and h = (l + v) / |l + v|; dL/da = (I - l l^T) dL/dl / |a|;
                            // gq holds dL/d(R_V u) = -dL/da (rotated to world below)
                            gI = e * Gh * ndl;
                            const float kn = e * Gh * A;
                            float3 gl = f3(kn * n3.x, kn * n3.y, kn * n3.z);
                            if (spec != 0.f) gl = f3(gl.x + spec * w.x, gl.y + spec * w.y, gl.z + spec * w.z);
                            const float lg = dot3(ld, gl), qi = 1.0f / S.light_qn[l];
                            gq0 = -(gl.x - lg * ld.x) * qi;
                            gq1 = -(gl.y - lg * ld.y) * qi;
                            gq2 = -(gl.z - lg * ld.z) * qi;
                        }
                    }
                }
                if (s0 == 0) {  // row k of the sums holds value k
                    const double s = wave_sum4((double)gq0, (double)gq1, (double)gq2, (double)gI);
                    if ((lane & 15) == 0) S.wacc[wave][4 * l + (lane >> 4)] += s;
                }
            }
            if (s0 == 0) {
                const double se = wave_sum((double)gc0 * U0 + (double)gc1 * U1 + (double)gc2 * U2);
                if (lane == 0) S.wacc[wave][4 * kMaxLights] += se;
            }
            // the pass's distinct objects, each summed over the lanes that show it
            const float o0 = e * gc0 * sAnd, o1 = e * gc1 * sAnd, o2 = e * gc2 * sAnd;
            const float o3 = e * G * ks * sAndsln * (-4.0f / (r * r * r)), o4 = e * G * sAnds;
            unsigned long long pend = __ballot(frag);
            while (pend) {
                const int k0 = __builtin_amdgcn_readlane(obj_local, __builtin_ctzll(pend));
                const bool mine = obj_local == k0;
                pend &= ~__ballot(mine);
                const int sl = (int)S.slot_of[k0] - s0;
                if (sl < 0 || sl >= ns) continue;  // another round's slot
                const double s = wave_sum4(mine ? (double)o0 : 0.0, mine ? (double)o1 : 0.0, mine ? (double)o2 : 0.0,
                                           mine ? (double)o3 : 0.0);
                const double s4 = wave_sum(mine ? (double)o4 : 0.0);
                if ((lane & 15) == 0) S.oacc[wave][sl][lane >> 4] += s;
                if (lane == 1) S.oacc[wave][sl][4] += s4;
            }
        }
        __syncthreads();
        for (int k = tid; k < 5 * n_obj; k += kBlock) {
            const int o = k / 5, c = k - 5 * o;
            const int sl = S.present[o] ? (int)S.slot_of[o] - s0 : -1;
            if (sl >= 0 && sl < ns) {
                double x = 0.0;
                for (int w = 0; w < kGWaves; ++w) x += S.oacc[w][sl][c];
                part[k] = x;
            } else if (s0 == 0 && sl < 0) {
                part[k] = 0.0;
            }
        }
        __syncthreads();
    }
    // lights (view -> world: dL/dq_world = R_V^T dL/dq_view) and exposure: waves summed in order
    double *lp = part + 5 * n_obj;
    if (tid < nl) {
        const int l = tid;
        double gv[4] = {0, 0, 0, 0};
        for (int w = 0; w < kGWaves; ++w)
            for (int c = 0; c < 4; ++c) gv[c] += S.wacc[w][4 * l + c];
        for (int c = 0; c < 3; ++c)
            lp[4 * l + c] = (double)V[0 * 4 + c] * gv[0] + (double)V[1 * 4 + c] * gv[1] + (double)V[2 * 4 + c] * gv[2];
        lp[4 * l + 3] = gv[3];
    }
    if (tid == kBlock - 1) {
        double se = 0.0;
        for (int w = 0; w < kGWaves; ++w) se += S.wacc[w][4 * kMaxLights];
        lp[4 * nl] = se;
    }
}

// Grid: x over 64-parameter chunks, y over scenes.  A scene's parameters: 5 per object,
// 4 per light, then 1 per frame (its exposure).  The scene's non-empty tiles are numbered
// in order; wave w sums tiles w, w + 16, ..., and the sixteen results are added in order.
// Bound by memory latency (a scene's partials are a few hundred KB): sixteen waves, each
// reading 64 tiles' marks and partial offsets in two loads and then only the non-empty
// tiles' partials, independent of one another; 64 scenes: 23 us with four waves walking
// every tile through its offset, 7 us so.
__global__ __launch_bounds__(kRBlock) void k_grad_reduce(GradArgs g, int s_base) {
    __shared__ double red[kRWaves][kGChunk];
    const int sc = s_base + (int)blockIdx.y;
    const int ob = g.scene_obj_begin[sc], no = g.scene_obj_begin[sc + 1] - ob;
    const int lb = g.scene_light_begin[sc], nl = g.scene_light_begin[sc + 1] - lb;
    const int fb = g.scene_frame_begin[sc], nf = g.scene_frame_begin[sc + 1] - fb;
    const int n_par = 5 * no + 4 * nl + nf;
    const int lane = lane_id(), wave = threadIdx.x / kWave;
    const int p = blockIdx.x * kGChunk + lane;
    if (blockIdx.x * kGChunk >= n_par) return;  // whole block past the scene's parameters
    double acc = 0.0;
    // lights follow the objects in every tile's vector, then the frame's exposure
    const bool expo = p >= 5 * no + 4 * nl && p < n_par;
    const int off = expo ? 5 * no + 4 * nl : p;
    const int f_only = expo ? g.scene_frames[fb + (p - 5 * no - 4 * nl)] : -1;
    int t = 0;  // non-empty tiles so far
    for (int fk = 0; fk < nf; ++fk) {
        const int f = g.scene_frames[fb + fk];
        const int i0 = g.frame_item_begin[f], i1 = g.frame_item_begin[f + 1];
        const bool take = p < n_par && (!expo || f_only == f);
        for (int ib = i0; ib < i1; ib += kWave) {
            const int it = ib + lane;
            const bool live = it < i1 && g.live[it] != 0;
            const int64_t pb = live ? g.gitem_pbase[it] : 0;
            const unsigned long long m = __ballot(live);
            unsigned long long mine = m;
            // this wave's tiles: those whose number is wave modulo kRWaves
            const int nth = t + lanes_below(m);
            mine = __ballot(live && (nth & (kRWaves - 1)) == wave);
            t += __popcll(m);
            while (mine) {
                const int src = __builtin_ctzll(mine);
                mine &= mine - 1;
                const int64_t base = (int64_t)(((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(pb >> 32), src) << 32) |
                                               (unsigned)__builtin_amdgcn_readlane((int)(unsigned)pb, src));
                if (take) acc += g.partial[base + off];
            }
        }
    }
    red[wave][lane] = acc;
    __syncthreads();
    if (wave != 0 || p >= n_par) return;
    double x = 0.0;
    for (int w = 0; w < kRWaves; ++w) x += red[w][lane];
    if (p < 5 * no) {
        const int o = ob + p / 5, k = p % 5;
        if (k < 3) g.g_albedo[3 * o + k] = (float)x;
        else if (k == 3) g.g_rough[o] = (float)x;
        else g.g_spec[o] = (float)x;
    } else if (p < 5 * no + 4 * nl) {
        const int l = lb + (p - 5 * no) / 4, k = (p - 5 * no) % 4;
        if (k < 3) g.g_lpos[3 * l + k] = (float)x;
        else g.g_lint[l] = (float)x;
    } else {
        g.g_expo[g.scene_frames[fb + (p - 5 * no - 4 * nl)]] = (float)x;
    }
}

hipError_t launch_grad(const GradArgs &g, hipStream_t stream) {
    hipError_t e = launch_vertex(g.r, stream);
    if (e != hipSuccess) return e;
    if (g.n_gitems > 0) {
        hipLaunchKernelGGL(k_grad_tile, dim3(g.n_gitems), dim3(kBlock), 0, stream, g);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const int chunks = (g.max_scene_params + kGChunk - 1) / kGChunk;
    constexpr int kMaxY = 32768;  // scenes per launch (grid y)
    for (int s0 = 0; s0 < g.n_scenes && e == hipSuccess; s0 += kMaxY) {
        const int ns = g.n_scenes - s0 < kMaxY ? g.n_scenes - s0 : kMaxY;
        hipLaunchKernelGGL(k_grad_reduce, dim3(chunks > 0 ? chunks : 1, ns), dim3(kRBlock), 0, stream, g, s0);
        e = hipGetLastError();
    }
    return e;
}

int grad_tile_size() { return kGTile; }
int grad_max_objects() { return kGMaxObj; }

}  // namespace orrb
