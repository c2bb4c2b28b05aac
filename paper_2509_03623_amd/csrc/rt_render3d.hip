// rt_render3d.hip -- line emission of fields on a 3-D spherical grid (gfx950).
//
// The fields of a non-axisymmetric disk (a hydrodynamic snapshot: density,
// temperature, all three velocity components, CO abundance) live on nodes
// r_i (log-spaced), theta_j (uniform polar angle), phi_k (uniform, periodic).
// The march keeps them as one interleaved record of eight floats per node,
// {ln n_H2, T, x_CO, v_r, v_theta, v_phi, 0, 0}: a sample's eight corners are
// sixteen 16-byte loads, and the two phi neighbours of a corner sit in one
// 64-byte run, where six separate planes would cost 48 scalar loads touching
// six times as many cache lines.  rt_pack_fields3d writes that layout from
// six planes once per snapshot; renders of the same snapshot (other channel
// sets, inclinations, position angles) reuse it.
//
// Per sample: spherical coordinates of the point, trilinear weights of its
// cell (computed once, applied to all six fields), the density fading to
// zero one cell beyond the radial and polar node ranges, LTE populations and
// source function as in the axisymmetric march, and the line-of-sight
// velocity v . w from the three components and the local unit vectors.  The
// channel loop, the lanes-per-ray split and its front-to-back composition
// are those of the axisymmetric march.  A sample beyond the fade (density
// and depth exactly 0) stops after its indices.  The march goes over line
// windows (march3_win); march3_fwd, all channels of a block at every sample
// with opacity, is what a chosen channel block or ray split runs.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <type_traits>
#include <vector>

#include "../../include/rtcube.h"
#include "rt_host.h"
#include "rt_kernels.h"

namespace rt {

// Per-launch camera geometry (float, the per-ray set-up included).
struct Geometry3 {
    float d_pix, cpa, spa, si, ci;
    float rc2;               // squared radius of the bounding sphere r_max e^dln [au^2]
    float xc, yc;
    int32_t nx, ny, nsamp, pad_;
};

// The ray through pixel (p, q) in the sky frame (x', y'), and h^2 = rc^2 -
// x'^2 - y'^2: the chord through the bounding sphere is s in [-h, h], its
// midpoint at s = 0 on the sky plane.
struct Chord3 {
    float xp, yp, h2;
};

__device__ __forceinline__ Chord3 chord3(const Geometry3 &g, int p, int q) {
    const float X = ((float)p + 0.5f - g.xc) * g.d_pix;
    const float Y = ((float)q + 0.5f - g.yc) * g.d_pix;
    Chord3 c;
    c.xp = fmaf(g.cpa, X, -g.spa * Y);
    c.yp = fmaf(g.spa, X, g.cpa * Y);
    c.h2 = fmaf(-c.xp, c.xp, fmaf(-c.yp, c.yp, g.rc2));
    return c;
}

// Fields and channel-independent constants.
struct Shade3 {
    const float4 *node;      // [nr][nt][np] records, two float4 each
    const float4 *ztab;
    const float *inv_r2n;    // [nr] 1 / r_i^2 of the radial nodes [au^-2]
    int32_t nr, nt, np, pad_;
    float u_scale, log2_rmin;   // coarse radial index (log2 r - log2 r_min) u_scale
    float h_r;                  // u_scale / 2: cells per unit of log2 (r^2 / r_i^2)
    float cth_c, sth_c;         // cos, sin of the middle polar angle theta_c of the nodes
    float inv_dth, half_nt1;    // w = (theta - theta_c) inv_dth + (nt - 1) / 2
    float inv_dph, fnp;         // s = phi inv_dph, phi in [0, 2 pi)
    float fnr, fnt;
    float zt_l2t0, zt_scale;    // partition-function table index
    float el_log2e, theta, c_s;
    float c_k;                  // as the axisymmetric c_k, without x_CO (a field here)
    float c_alpha, sqrt_log2e;
    float si, ci, vsys;
    float zeta;                 // |z| / rho beyond which every sample is past the fade (0: not a wedge)
};

// Z(T): the table lookup of the axisymmetric march reads only the table's
// index constants of its shading block.
__device__ __forceinline__ float partition3(const Shade3 &s, const float4 *tab, float log2t) {
    Shade z{};
    z.zt_l2t0 = s.zt_l2t0;
    z.zt_scale = s.zt_scale;
    return partition_fn(z, tab, log2t);
}

// Where a sample falls on the grid: its cell and the fractions in it, valid
// indices for a sample beyond the fade too (taper 0).
struct Cell3 {
    float rho2, r2, rho, taper;
    float fu, fw, fs;           // radial, polar and azimuthal fraction
    uint32_t n0, n1;            // nodes (i, j, k) and (i, j, k + 1)
};

__device__ __forceinline__ void locate3(const Shade3 &s, float px, float py, float pz, Cell3 &c, int &i0, float &fr,
                                        float &w) {
    c.rho2 = fmaf(px, px, py * py);
    c.r2 = fmaf(pz, pz, c.rho2);
    c.rho = fsqrt(c.rho2);
    // Radial index.  A float index near 500 carries ~3e-5 of a cell of
    // rounding and log2 of r^2 ~ 1e5 an absolute error that the cell scale
    // multiplies; so the cell comes from the coarse index and the fraction
    // from log2 of r^2 / r_i^2, a ratio near 1.  The coarse index is within
    // 1e-4 of a cell: one re-centring step suffices.  r = 0 gives a fraction
    // of -inf: clamped fetch, zero taper, zero depth.
    const float uco = fmaf(0.5f, flog2(c.r2), -s.log2_rmin) * s.u_scale;
    i0 = (int)clampf(uco, 0.0f, s.fnr - 2.0f);
    fr = flog2(1.0f + fmaf(c.r2, s.inv_r2n[i0], -1.0f)) * s.h_r;
    if (fr < 0.0f && i0 > 0) { --i0; fr += 1.0f; }
    else if (fr >= 1.0f && i0 < s.nr - 2) { ++i0; fr -= 1.0f; }
    // Polar index from the angle to the middle node direction theta_c, which
    // is small over a wedge about the midplane (finer float spacing than theta).
    const float a1 = fmaf(c.rho, s.cth_c, -pz * s.sth_c);   // r sin(theta - theta_c)
    const float a2 = fmaf(pz, s.cth_c, c.rho * s.sth_c);    // r cos(theta - theta_c)
    w = fmaf(atan2f(a1, a2), s.inv_dth, s.half_nt1);
    // fade one cell beyond the node ranges (radially from the cell and its
    // fraction, exact near both ends); beyond the fade the density and the
    // depth are exactly 0: no azimuth, no fetch, no physics
    c.taper = clampf((float)i0 + fr + 1.0f, 0.0f, 1.0f) * clampf((s.fnr - (float)i0) - fr, 0.0f, 1.0f) *
                        clampf(w + 1.0f, 0.0f, 1.0f) * clampf(s.fnt - w, 0.0f, 1.0f);
}

// the rest of the cell, which only a sample with taper > 0 needs
__device__ __forceinline__ void locate3_nodes(const Shade3 &s, float px, float py, Cell3 &c, int i0, float fr,
                                              float w) {
    float sp = atan2f(py, px) * s.inv_dph;
    sp = sp < 0.0f ? sp + s.fnp : sp;
    c.fu = clampf(fr, 0.0f, 1.0f);
    const float wc = clampf(w, 0.0f, s.fnt - 1.0f);
    const int j0 = min((int)wc, s.nt - 2);
    c.fw = wc - (float)j0;
    int k0 = (int)sp;
    c.fs = sp - (float)k0;
    k0 = k0 >= s.np ? k0 - s.np : k0;       // sp may round up to np
    const int k1 = k0 + 1 >= s.np ? 0 : k0 + 1;
    const uint32_t b00 = ((uint32_t)i0 * (uint32_t)s.nt + (uint32_t)j0) * (uint32_t)s.np;
    c.n0 = b00 + (uint32_t)k0;
    c.n1 = b00 + (uint32_t)k1;
}

// The line physics of the fields of a sample, A = (ln n, T, x_CO, v_r), vt and vp
// (cf. physics() of the axisymmetric march): S, line-centre depth K (log2 units),
// and d = a - v b.
__device__ __forceinline__ SampleQ physics3(const Shade3 &s, const float4 *tab, const Cell3 &c, float4 A, float vt,
                                            float vp, float px, float py, float pz, float ds) {
    const float ln_n = A.x, T = A.y, xco = A.z, vr = A.w;
    const float rho2 = c.rho2, r2 = c.r2, rho = c.rho;
    const float nco = xco * fexp2(ln_n * kLog2E) * c.taper;
    // LTE populations and source function
    const float rT = frcp(T);
    const float Z = partition3(s, tab, flog2(T));
    const float el = fexp2(-s.el_log2e * rT);
    const float x = fminf(s.theta * rT, 80.0f);
    const float em1 = expm1_pos(x);
    SampleQ q;
    q.S = s.c_s * frcp(em1);
    const float inv_alpha = frsq(T * s.c_alpha);
    q.K = s.c_k * nco * el * em1 * frcp(Z * (1.0f + em1)) * ds * inv_alpha;
    q.b = s.sqrt_log2e * inv_alpha;
    // v . w with w = (0, sin i, -cos i): radial, polar and azimuthal unit
    // vectors at the sample (the polar and azimuthal terms vanish on the axis)
    const float inv_r = r2 > 0.0f ? frsq(r2) : 0.0f;
    const float inv_rho = rho2 > 0.0f ? frsq(rho2) : 0.0f;
    const float er = fmaf(py, s.si, -pz * s.ci) * inv_r;
    const float et = fmaf((pz * inv_r) * (py * inv_rho), s.si, rho * inv_r * s.ci);
    const float ep = px * inv_rho * s.si;
    const float vlos = fmaf(vp, ep, fmaf(vt, et, fmaf(vr, er, s.vsys)));
    q.a = vlos * q.b;
    return q;
}

__device__ __forceinline__ SampleQ shade3(const Shade3 &s, const float4 *tab, float px, float py, float pz,
                                          float ds) {
    Cell3 cell;
    int i0;
    float fr, w;
    locate3(s, px, py, pz, cell, i0, fr, w);
    if (cell.taper <= 0.0f) {
        SampleQ z;
        z.S = 0.0f; z.K = 0.0f; z.a = 0.0f; z.b = 0.0f;
        return z;
    }
    locate3_nodes(s, px, py, cell, i0, fr, w);
    const uint32_t np = (uint32_t)s.np, plane = (uint32_t)s.nt * np;
    const uint32_t off[4] = {0u, np, plane, plane + np};   // (i,j), (i,j+1), (i+1,j), (i+1,j+1)
    float4 A[8], B[8];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const size_t n0 = 2 * (size_t)(off[c] + cell.n0), n1 = 2 * (size_t)(off[c] + cell.n1);
        A[2 * c] = s.node[n0];
        B[2 * c] = s.node[n0 + 1];
        A[2 * c + 1] = s.node[n1];
        B[2 * c + 1] = s.node[n1 + 1];
    }
    // trilinear weights, in the corner order of the loads
    const float fu = cell.fu, fw = cell.fw, fs = cell.fs;
    const float gu = 1.0f - fu, gw = 1.0f - fw, gs = 1.0f - fs;
    const float cuw[4] = {gu * gw, gu * fw, fu * gw, fu * fw};
    float wt[8];
#pragma unroll
    for (int c = 0; c < 4; ++c) { wt[2 * c] = cuw[c] * gs; wt[2 * c + 1] = cuw[c] * fs; }
    float4 f = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    float vt = 0.0f, vp = 0.0f;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        f.x = fmaf(wt[c], A[c].x, f.x);
        f.y = fmaf(wt[c], A[c].y, f.y);
        f.z = fmaf(wt[c], A[c].z, f.z);
        f.w = fmaf(wt[c], A[c].w, f.w);
        vt = fmaf(wt[c], B[c].x, vt);
        vp = fmaf(wt[c], B[c].y, vp);
    }
    return physics3(s, tab, cell, f, vt, vp, px, py, pz, ds);
}

// The fields of the four samples of a quad, one a lane (every lane active).
// Each sample's eight records are four runs of 64 bytes (nodes k and k + 1);
// the four lanes read a run together, a float4 each, and the weighted sums of
// the four samples are then handed to their lanes: a load touches 16 lines of
// memory instead of the 64 that lanes reading their own records would.
__device__ __forceinline__ void gather3(const Shade3 &s, const Cell3 &cell, int h, float4 &A, float &vt, float &vp) {
    const size_t np = (size_t)s.np, plane = (size_t)s.nt * np;
    const float fu = cell.fu, fw = cell.fw, gu = 1.0f - fu, gw = 1.0f - fw;
    const float cuw[4] = {gu * gw, gu * fw, fu * gw, fu * fw};
    const bool hi = (h & 2) != 0, odd = (h & 1) != 0;   // this lane's piece: node k + 1, second half of the record
    const float4 *base = s.node + (odd ? 1 : 0);
    float4 sum[4];
    auto one = [&](auto jc) {
        constexpr int J = decltype(jc)::value;
        const int n0 = group_lane_i<J>((int)cell.n0), n1 = group_lane_i<J>((int)cell.n1);
        const float fs = group_lane<4, J>(cell.fs), ws = hi ? fs : 1.0f - fs;
        const float4 *p = base + 2 * (size_t)(uint32_t)(hi ? n1 : n0);
        const float4 v0 = p[0], v1 = p[2 * np], v2 = p[2 * plane], v3 = p[2 * (plane + np)];
        const float w0 = group_lane<4, J>(cuw[0]) * ws, w1 = group_lane<4, J>(cuw[1]) * ws;
        const float w2 = group_lane<4, J>(cuw[2]) * ws, w3 = group_lane<4, J>(cuw[3]) * ws;
        sum[J].x = fmaf(w3, v3.x, fmaf(w2, v2.x, fmaf(w1, v1.x, w0 * v0.x)));
        sum[J].y = fmaf(w3, v3.y, fmaf(w2, v2.y, fmaf(w1, v1.y, w0 * v0.y)));
        sum[J].z = fmaf(w3, v3.z, fmaf(w2, v2.z, fmaf(w1, v1.z, w0 * v0.z)));
        sum[J].w = fmaf(w3, v3.w, fmaf(w2, v2.w, fmaf(w1, v1.w, w0 * v0.w)));
    };
    one(std::integral_constant<int, 0>{});
    one(std::integral_constant<int, 1>{});
    one(std::integral_constant<int, 2>{});
    one(std::integral_constant<int, 3>{});
    // node k + node k + 1 (lanes two apart), then first and second halves (lanes one apart)
    auto keep = [&](float a, float b) { return (hi ? b : a) + quad_xor<2>(hi ? a : b); };
    const float4 e = make_float4(keep(sum[0].x, sum[2].x), keep(sum[0].y, sum[2].y), keep(sum[0].z, sum[2].z),
                                 keep(sum[0].w, sum[2].w));      // sample 0 or 2
    const float4 o = make_float4(keep(sum[1].x, sum[3].x), keep(sum[1].y, sum[3].y), keep(sum[1].z, sum[3].z),
                                 keep(sum[1].w, sum[3].w));      // sample 1 or 3
    const float rx = quad_xor<1>(odd ? e.x : o.x), ry = quad_xor<1>(odd ? e.y : o.y);
    const float rz = quad_xor<1>(odd ? e.z : o.z), rw = quad_xor<1>(odd ? e.w : o.w);
    A = make_float4(odd ? rx : e.x, odd ? ry : e.y, odd ? rz : e.z, odd ? rw : e.w);
    vt = odd ? o.x : rx;
    vp = odd ? o.y : ry;
}

// One lane = one pixel (or a sub-chord of it, NSPLIT lanes per ray) x CB
// channels.  Blocks are numbered XCD-aware: the dispatcher deals consecutive
// workgroup ids to the eight XCDs in turn, so id L runs on XCD L % 8; logical
// work item (L % 8) * per_xcd + L / 8 gives each XCD one contiguous run of
// tiles with all their channel blocks, which read the same grid cells from
// that XCD's L2.  Blocks of up to 24 channels are held to 128 VGPRs (4 waves
// per SIMD, no spills): at 24 channels the unconstrained kernel takes ~137
// and runs 3, and the extra resident waves are worth 14% at 512^2 pixels.
template <int CB, int NSPLIT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CB <= 16 ? 4 : 1))) void march3_fwd(Geometry3 g, Shade3 s, Channels ch, float *__restrict__ cube,
                                                   int ch_stride, int nchb, int nwork, int per_xcd) {
    const int L = blockIdx.x;
    const int work = (L % 8) * per_xcd + L / 8;
    if (work >= nwork) return;                       // whole workgroup: padding of the grid to 8 x per_xcd
    __shared__ float4 ztab[kZTableNodes - 1];
    for (int i = threadIdx.x; i < kZTableNodes - 1; i += blockDim.x) ztab[i] = s.ztab[i];
    __syncthreads();
    constexpr int TW = NSPLIT <= 2 ? 16 : 8;
    constexpr int TH = 256 / NSPLIT / TW;
    const int tiles_x = (g.nx + TW - 1) / TW;
    const int tile = work / nchb, c0 = (work % nchb) * CB;
    const int split = threadIdx.x % NSPLIT;
    const int slot = threadIdx.x / NSPLIT;
    const int p = (tile % tiles_x) * TW + slot % TW;
    const int q = (tile / tiles_x) * TH + slot / TW;
    const bool inside = p < g.nx && q < g.ny;
    float I[CB], Tr[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) { I[c] = 0.0f; Tr[c] = 1.0f; }
    // ray set-up: chord through the bounding sphere, midpoint at s = 0
    const Chord3 cr = chord3(g, inside ? p : 0, inside ? q : 0);
    if (inside && cr.h2 > 0.0f) {
        const float ds = 2.0f * sqrtf(cr.h2) / (float)g.nsamp;
        const float pxr = cr.xp, pmy = cr.yp * g.ci, pmz = cr.yp * g.si;
        const float wy = g.si, wz = -g.ci;
        const float half = 0.5f * (float)g.nsamp;
        const int len = (g.nsamp + NSPLIT - 1) / NSPLIT;
        const int k0 = split * len;
        const int k1 = min(g.nsamp, k0 + len);
        for (int k = k0; k < k1; ++k) {
            const float t = ((float)k + 0.5f - half) * ds;
            const SampleQ sq = shade3(s, ztab, pxr, fmaf(t, wy, pmy), fmaf(t, wz, pmz), ds);
            // no ray of the wave with opacity at this sample: no channel changes
            if (__ballot(sq.K > 0.0f) == 0) continue;
            march_sample<CB, true>(I, Tr, sq, [&](int c) { return ch.v[c0 + c]; });
        }
    }
#pragma unroll
    for (int d = 1; d < NSPLIT; d <<= 1) {
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            const float Ib = __shfl_down(I[c], d, NSPLIT);
            const float Tb = __shfl_down(Tr[c], d, NSPLIT);
            if ((split & (2 * d - 1)) == 0) {
                I[c] = fmaf(Tr[c], Ib, I[c]);
                Tr[c] *= Tb;
            }
        }
    }
    if (!inside || split != 0) return;
    const size_t pix = (size_t)q * g.nx + p;
#pragma unroll
    for (int c = 0; c < CB; ++c)
        if (c0 + c < ch.n) cube[(size_t)(c0 + c) * ch_stride + pix] = I[c];
}

// Windowed march (rt_forward.hip, march_win): four lanes per pixel with the
// channels interleaved over them, 4 x 4 pixels a wave, the rays in parts over
// the waves of a workgroup, over the samples that can lie in the polar wedge;
// a wave passes over steps beyond the fade and steps without CO.  Bound: 62 %
// of the time issue of vector instructions (cells and physics of the samples
// inside the fade), the rest the latency of the gathers (58 % of a wave's time is
// spent waiting for loads) and waves of unequal work.
// 512 x 96 x 256 grid, 256^2 x 512 samples, 64 channels: 1.30 ms as
// march3_fwd, 0.43 ms with windows, 0.39 ms with the quad's gather (gather3),
// 0.29 ms with the work order below, 0.25 ms with up to four ray parts.
//
// Block b runs on XCD b % 8, so consecutive work goes to an XCD in chunks of
// 16 tiles: their neighbours share its L2's lines.  One run of tiles per XCD,
// an eighth of the image, leaves the XCDs of the image's edge idle: 0.39 ms
// against 0.29 (chunks of 16) and 0.36 (of 1); 512^2 x 20 channels 0.90, 0.65
// and 0.81 ms.  A launch under 1024 blocks takes smaller chunks, 8 per XCD.
// 128 VGPRs (four waves a SIMD) hold the 16-channel form without spills: 0.39
// against 0.43 ms at its natural 132; 24 and 32 channels would spill.
template <int CB, bool UNIFORM>
__global__ __launch_bounds__(512, CB <= 16 ? 4 : 2) void march3_win(Geometry3 g, Shade3 s, Channels ch, Windows win, int lsplit,
                                                  float *__restrict__ cube, int ch_stride, int nchb, int nwork,
                                                  int chunk) {
    const int L = blockIdx.x;
    const int work = ((L / 8) / chunk * 8 + L % 8) * chunk + (L / 8) % chunk;
    if (work >= nwork) return;                       // whole workgroup: padding of the grid to 8 x chunk
    __shared__ float4 ztab[kZTableNodes - 1];
    extern __shared__ float parts[];
    for (int i = threadIdx.x; i < kZTableNodes - 1; i += blockDim.x) ztab[i] = s.ztab[i];
    __syncthreads();
    constexpr int G = kLanesPerPixel, U = unit_slots(CB), NU = CB / U;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nsplit = 1 << lsplit, nsub = (int)(blockDim.x >> 6) >> lsplit;   // 4 x 4 tiles of this workgroup
    const int split = wave & (nsplit - 1), sub = wave >> lsplit;
    const int lane = threadIdx.x & 63, h = lane & 3, slot = lane >> 2;
    const int tw = nsub >= 2 ? 8 : 4, th = nsub >= 4 ? 8 : 4;
    const int tiles_x = (g.nx + tw - 1) / tw;
    const int tile = work / nchb, blk = work % nchb;
    const int p = (tile % tiles_x) * tw + (sub & 1) * 4 + (slot & 3);
    const int q = (tile / tiles_x) * th + (sub >> 1) * 4 + (slot >> 2);
    const int c0 = blk * CB * G, u0 = blk * NU;
    const bool inside = p < g.nx && q < g.ny;
    const Chord3 cr = chord3(g, inside ? p : 0, inside ? q : 0);
    const bool live = inside && cr.h2 > 0.0f;
    float I[CB], Tr[CB], vc[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        I[c] = 0.0f;
        Tr[c] = 1.0f;
        vc[c] = ch.v[c0 + c * G + h];
    }
    if (__ballot(live) != 0) {
        const float ds = live ? 2.0f * sqrtf(cr.h2) / (float)g.nsamp : 0.0f;
        const float pmy = cr.yp * g.ci, pmz = cr.yp * g.si, wy = g.si, wz = -g.ci;
        const float half = 0.5f * (float)g.nsamp;
        const int2 own = !live ? make_int2(g.nsamp, -1)
                       : s.zeta > 0.0f ? cone_range(s.zeta, cr.xp, pmy, pmz, wy, wz, ds, g.nsamp)
                                       : make_int2(0, g.nsamp - 1);
        const int kf = wave_min(own.x), kn = max(wave_max(own.y) + 1 - kf, 0);
        const int len = (((kn + nsplit - 1) >> lsplit) + G - 1) / G * G;
        const int k1 = kf + min(kn, (split + 1) * len);
        const float v0 = ch.v[c0];
        for (int k = kf + split * len; k < k1; k += G) {
            const float t = ((float)min(k + h, k1 - 1) + 0.5f - half) * ds;
            const float py = fmaf(t, wy, pmy), pz = fmaf(t, wz, pmz);
            Cell3 cell;
            int i0;
            float fr, w;
            locate3(s, cr.xp, py, pz, cell, i0, fr, w);
            const bool in = live && k + h < k1 && cell.taper > 0.0f;
            if (__builtin_amdgcn_ballot_w64(in) == 0) continue;
            locate3_nodes(s, cr.xp, py, cell, i0, fr, w);
            if (!in) cell.n0 = cell.n1 = 0;
            float4 A;
            float vt, vp;
            gather3(s, cell, h, A, vt, vp);
            // no CO at any of the wave's samples
            if (__builtin_amdgcn_ballot_w64(in && A.z != 0.0f) == 0) continue;
            SampleQ own = physics3(s, ztab, cell, A, vt, vp, cr.xp, py, pz, ds);
            if (!in) own.S = own.K = own.a = own.b = 0.0f;
            const float own_lk = flog2(own.K);
            const unsigned mask = or_over_pixels(unit_mask<NU, G * U, UNIFORM>(own, own_lk, in, v0, win, u0));
            const unsigned long long bright = __builtin_amdgcn_ballot_w64(!(own_lk < kFaintLog2K));
            const unsigned long long thick = __builtin_amdgcn_ballot_w64(!(own_lk < kThinLog2K));
            auto step = [&](auto jc) {
                constexpr int J = decltype(jc)::value;
                constexpr unsigned long long mine = 0x1111111111111111ull << J;
                const unsigned m = (unsigned)__builtin_amdgcn_readlane((int)mask, J);
                if (m == 0) return;
                const float S = group_lane<G, J>(own.S), lK = group_lane<G, J>(own_lk);
                const float a = group_lane<G, J>(own.a), b = group_lane<G, J>(own.b);
                march_units<CB>(I, Tr, S, lK, m, (bright & mine) != 0, (thick & mine) != 0,
                                [&](int c) { return fmaf(-vc[c], b, a); });
            };
            step(std::integral_constant<int, 0>{});
            step(std::integral_constant<int, 1>{});
            step(std::integral_constant<int, 2>{});
            step(std::integral_constant<int, 3>{});
        }
    }
    if (nsplit > 1) {
        float *mine = parts + (size_t)(sub * (nsplit - 1)) * (2 * CB * 64) + lane;
        if (split > 0) {
            float *o = mine + (size_t)(split - 1) * (2 * CB * 64);
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                o[c * 64] = I[c];
                o[(CB + c) * 64] = Tr[c];
            }
        }
        __syncthreads();
        if (split > 0) return;
        for (int j = 0; j < nsplit - 1; ++j) {
            const float *o = mine + (size_t)j * (2 * CB * 64);
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                I[c] = fmaf(Tr[c], o[c * 64], I[c]);
                Tr[c] *= o[(CB + c) * 64];
            }
        }
    }
    if (!inside) return;
    const size_t pix = (size_t)q * g.nx + p;
#pragma unroll
    for (int c = 0; c < CB; ++c)
        if (c0 + c * G + h < ch.n) cube[(size_t)(c0 + c * G + h) * ch_stride + pix] = I[c];
}

// Waves asked for before rays stop being parted: twice the axisymmetric march's,
// since tiles at the sphere's edge and rays that miss the CO layer end early.
// 8192 against 16384 (us): 256^2 x 64 293, 254; 256^2 x 20 237, 210; 360^2 x 64 434,
// 395; 360^2 x 30 376, 337; the same at 128^2 to 200^2 (parts already at most) and
// at 512^2.  32768: 360^2 x 30 357, the rest within 3 %.
constexpr long kWinWaves3 = 16384;

template <int CB>
static hipError_t launch3_win(const Geometry3 &g, const Shade3 &s, const Channels &ch, const Windows &win, float *cube,
                              bool uniform, int lsplit, hipStream_t st) {
    const int waves = std::max(4, 1 << lsplit), nsub = waves >> lsplit;
    const int tw = nsub >= 2 ? 8 : 4, th = nsub >= 4 ? 8 : 4;
    const long tiles = (long)((g.nx + tw - 1) / tw) * ((g.ny + th - 1) / th);
    const int nchb = (ch.n + CB * kLanesPerPixel - 1) / (CB * kLanesPerPixel);
    const long nwork = tiles * nchb;
    if (nwork > (1L << 30)) return hipErrorInvalidValue;
    const int chunk = (int)std::min(16L, std::max(1L, nwork / 64));
    const int nblocks = (int)((nwork + 8 * chunk - 1) / (8 * chunk)) * (8 * chunk);
    const size_t lds = (size_t)nsub * ((1 << lsplit) - 1) * 2 * CB * 64 * sizeof(float);
    const int cs = g.nx * g.ny;
    if (uniform) hipLaunchKernelGGL((march3_win<CB, true>), dim3(nblocks), dim3(64 * waves), lds, st, g, s, ch, win, lsplit, cube, cs, nchb, (int)nwork, chunk);
    else hipLaunchKernelGGL((march3_win<CB, false>), dim3(nblocks), dim3(64 * waves), lds, st, g, s, ch, win, lsplit, cube, cs, nchb, (int)nwork, chunk);
    return hipGetLastError();
}

static hipError_t launch_forward3_win(const Geometry3 &g, const Shade3 &s, const Channels &ch, const Windows &win,
                                      float *cube, int cb, bool uniform, int lsplit, hipStream_t st) {
    switch (cb) {
    case 4: return launch3_win<4>(g, s, ch, win, cube, uniform, lsplit, st);
    case 8: return launch3_win<8>(g, s, ch, win, cube, uniform, lsplit, st);
    case 12: return launch3_win<12>(g, s, ch, win, cube, uniform, lsplit, st);
    case 16: return launch3_win<16>(g, s, ch, win, cube, uniform, lsplit, st);
    case 24: return launch3_win<24>(g, s, ch, win, cube, uniform, lsplit, st);
    case 32: return launch3_win<32>(g, s, ch, win, cube, uniform, lsplit, st);
    default: return hipErrorInvalidValue;
    }
}

template <int CB, int NSPLIT>
static hipError_t launch3_t(const Geometry3 &g, const Shade3 &s, const Channels &ch, float *cube, hipStream_t st) {
    constexpr int TW = NSPLIT <= 2 ? 16 : 8;
    constexpr int TH = 256 / NSPLIT / TW;
    const int tiles = ((g.nx + TW - 1) / TW) * ((g.ny + TH - 1) / TH);
    const int nchb = (ch.n + CB - 1) / CB;
    const long nwork = (long)tiles * nchb;
    if (nwork > (1L << 30)) return hipErrorInvalidValue;
    const int per_xcd = (int)((nwork + 7) / 8);
    hipLaunchKernelGGL((march3_fwd<CB, NSPLIT>), dim3(8 * per_xcd), dim3(256), 0, st, g, s, ch, cube, g.nx * g.ny,
                       nchb, (int)nwork, per_xcd);
    return hipGetLastError();
}

template <int CB>
static hipError_t launch3_cb(const Geometry3 &g, const Shade3 &s, const Channels &ch, float *cube, int nsplit,
                             hipStream_t st) {
    switch (nsplit) {
    case 1: return launch3_t<CB, 1>(g, s, ch, cube, st);
    case 2: return launch3_t<CB, 2>(g, s, ch, cube, st);
    case 4: return launch3_t<CB, 4>(g, s, ch, cube, st);
    case 8: return launch3_t<CB, 8>(g, s, ch, cube, st);
    default: return hipErrorInvalidValue;
    }
}

static hipError_t launch_forward3(const Geometry3 &g, const Shade3 &s, const Channels &ch, float *cube, int cb,
                                  int nsplit, hipStream_t st) {
    switch (cb) {
    case 8: return launch3_cb<8>(g, s, ch, cube, nsplit, st);
    case 16: return launch3_cb<16>(g, s, ch, cube, nsplit, st);
    case 24: return launch3_cb<24>(g, s, ch, cube, nsplit, st);
    case 32: return launch3_cb<32>(g, s, ch, cube, nsplit, st);
    case 48: return launch3_cb<48>(g, s, ch, cube, nsplit, st);
    case 64: return launch3_cb<64>(g, s, ch, cube, nsplit, st);
    default: return hipErrorInvalidValue;
    }
}

// Six planes [nr][nt][np] -> interleaved records; NULL velocity planes are zero.
__global__ __launch_bounds__(256) void pack3(const float *__restrict__ ln_n, const float *__restrict__ temp,
                                             const float *__restrict__ xco, const float *__restrict__ vr,
                                             const float *__restrict__ vt, const float *__restrict__ vp,
                                             float4 *__restrict__ node, uint32_t n) {
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        node[2 * (size_t)i] = make_float4(ln_n[i], temp[i], xco[i], vr ? vr[i] : 0.0f);
        node[2 * (size_t)i + 1] = make_float4(vt ? vt[i] : 0.0f, vp ? vp[i] : 0.0f, 0.0f, 0.0f);
    }
}

constexpr double kPI3 = 3.14159265358979323846;
constexpr int64_t kMaxNodes3 = (int64_t)1 << 28;

// 1 / r_i^2 of the radial nodes, in double then rounded once, kept per
// (device, grid) for the life of the process like the partition table.
static rt_status radius_table(const rt_grid3d &g, const float **out) {
    static std::mutex mu;
    static std::map<std::tuple<int, int, double, double>, float *> cache;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
    const auto key = std::make_tuple(dev, (int)g.nr, g.r_min_au, g.r_max_au);
    std::lock_guard<std::mutex> lk(mu);
    auto it = cache.find(key);
    if (it != cache.end()) { *out = it->second; return RT_OK; }
    std::vector<float> tab(g.nr);
    const double dln = std::log(g.r_max_au / g.r_min_au) / (g.nr - 1);
    for (int i = 0; i < g.nr; ++i) {
        const double r = g.r_min_au * std::exp(i * dln);
        tab[i] = (float)(1.0 / (r * r));
    }
    float *d = nullptr;
    e = hipMalloc(&d, sizeof(float) * g.nr);
    if (e != hipSuccess) return fail_hip(e, "hipMalloc(radius table)");
    e = hipMemcpy(d, tab.data(), sizeof(float) * g.nr, hipMemcpyHostToDevice);
    if (e != hipSuccess) { (void)hipFree(d); return fail_hip(e, "hipMemcpy(radius table)"); }
    cache[key] = d;
    *out = d;
    return RT_OK;
}

// Launch shape of march3_fwd, where one of its two options is chosen.  Its shading (two atan2, sixteen scattered
// loads, the physics) costs ~25 channels' worth of issue slots per sample, so
// a pixel's channels stay in one block (the smallest of 8..64 holding them,
// never split into two 32-channel blocks as the axisymmetric march does).
// Two lanes per ray (two half-chords in flight per pixel) were best at every
// image size measured; rays split further only while the launch stays at or
// under 1024 waves.  Measured on the 512 x 96 x 256 grid (ms): 256^2 x 20 ch
// (24, 2) 0.75 against (24, 4) 0.85; 256^2 x 64 (64, 2) 1.00 against (32, 2)
// 1.52; 256^2 x 128 (64, 2) 1.89 against (32, 1) 2.96; 512^2 x 20 (24, 2)
// 2.17 against (24, 1) 2.38; 128^2 x 20 (24, 4) 0.33 against (24, 8) 0.37.
static void forward_shape3(int nch, long npix, int nsamp, int *cb_out, int *split_out) {
    static const int cands[] = {8, 16, 24, 32, 48, 64};
    int cb = 64;
    for (int c : cands)
        if (c >= nch) { cb = c; break; }
    auto waves = [&](int ns) { return ((npix * ns + 63) / 64) * (long)((nch + cb - 1) / cb); };
    int ns = nsamp >= 128 ? 2 : 1;
    while (ns < 8 && waves(2 * ns) <= 1024 && nsamp >= 128 * ns) ns <<= 1;
    *cb_out = cb;
    *split_out = ns;
}

// camera and bounding sphere of a 3-D problem
static Geometry3 geometry3(const rt_problem3d *p) {
    const rt_grid3d &gr = p->grid;
    const double dln = std::log(gr.r_max_au / gr.r_min_au) / (gr.nr - 1);
    const double ang = p->cam.incl_deg * kPI3 / 180.0, pa = p->cam.pa_deg * kPI3 / 180.0;
    Geometry3 g;
    std::memset(&g, 0, sizeof g);
    g.d_pix = p->cam.fov_au / p->cam.nx;
    g.cpa = std::cos(pa);
    g.spa = std::sin(pa);
    g.si = std::sin(ang);
    g.ci = std::cos(ang);
    if (p->cam.incl_deg == 0.0) { g.si = 0.0; g.ci = 1.0; }
    if (p->cam.incl_deg == 90.0) { g.si = 1.0; g.ci = 0.0; }
    if (p->cam.incl_deg == 180.0) { g.si = 0.0; g.ci = -1.0; }
    const double rc = gr.r_max_au * std::exp(dln);
    g.rc2 = rc * rc;
    g.xc = 0.5 * p->cam.nx;
    g.yc = 0.5 * p->cam.ny;
    g.nx = p->cam.nx;
    g.ny = p->cam.ny;
    g.nsamp = p->nsamp;
    return g;
}

// Rays of a 3-D render that cross the bounding sphere (the march's own
// test) and, with shade, their pixel-samples that are thin in the march's
// sense, that have any opacity, and that lie inside the grid's fade (the
// march's own shading).  blockIdx.y: a chunk of the samples of each ray.
__global__ __launch_bounds__(256) void census3(Geometry3 g, Shade3 s, uint8_t *__restrict__ mask,
                                               unsigned long long *__restrict__ counts, int shade) {
    __shared__ float4 ztab[kZTableNodes - 1];
    __shared__ unsigned long long part[4];
    if (shade)
        for (int i = threadIdx.x; i < kZTableNodes - 1; i += blockDim.x) ztab[i] = s.ztab[i];
    if (threadIdx.x < 4) part[threadIdx.x] = 0ull;
    __syncthreads();
    const int pix = blockIdx.x * 256 + threadIdx.x;
    if (pix < g.nx * g.ny) {
        const int p = pix % g.nx, q = pix / g.nx;
        const Chord3 cr = chord3(g, p, q);
        const bool live = cr.h2 > 0.0f;
        if (blockIdx.y == 0) {
            if (mask) mask[pix] = live ? 1 : 0;
            if (live) atomicAdd(&part[0], 1ull);
        }
        if (live && shade) {
            const float ds = 2.0f * sqrtf(cr.h2) / (float)g.nsamp;
            const float pmy = cr.yp * g.ci, pmz = cr.yp * g.si, wy = g.si, wz = -g.ci;
            const float half = 0.5f * (float)g.nsamp;
            const int len = (g.nsamp + gridDim.y - 1) / gridDim.y;
            const int k0 = blockIdx.y * len, k1 = min(g.nsamp, k0 + len);
            unsigned thin = 0, emit = 0, inside = 0;
            for (int k = k0; k < k1; ++k) {
                const float t = ((float)k + 0.5f - half) * ds;
                const SampleQ sq = shade3(s, ztab, cr.xp, fmaf(t, wy, pmy), fmaf(t, wz, pmz), ds);
                thin += sq.K < kThinK ? 1u : 0u;
                emit += sq.K > 0.0f ? 1u : 0u;
                inside += sq.b > 0.0f ? 1u : 0u;   // b = 0 only for a sample beyond the fade
            }
            if (thin) atomicAdd(&part[1], (unsigned long long)thin);
            if (emit) atomicAdd(&part[2], (unsigned long long)emit);
            if (inside) atomicAdd(&part[3], (unsigned long long)inside);
        }
    }
    __syncthreads();
    if (threadIdx.x < 4 && part[threadIdx.x]) atomicAdd(counts + threadIdx.x, part[threadIdx.x]);
}

__global__ void census3_zero(unsigned long long *c) {
    if (threadIdx.x < 4) c[threadIdx.x] = 0ull;
}

static rt_status validate_grid3(const rt_grid3d *g) {
    if (!g) return fail(RT_EINVAL, "grid is NULL");
    if (g->nr < 2 || g->nt < 2 || g->np < 1)
        return fail(RT_EINVAL, "grid needs nr >= 2, nt >= 2, np >= 1 (got %d, %d, %d)", g->nr, g->nt, g->np);
    if ((int64_t)g->nr * g->nt * g->np > kMaxNodes3) return fail(RT_EINVAL, "grid has more than 2^28 nodes");
    if (!(std::isfinite(g->r_min_au) && std::isfinite(g->r_max_au) && g->r_min_au > 0 && g->r_max_au > g->r_min_au))
        return fail(RT_EINVAL, "need 0 < r_min_au < r_max_au");
    if (!(std::isfinite(g->th_min) && std::isfinite(g->th_max) && g->th_min >= 0 && g->th_max > g->th_min &&
          g->th_max <= kPI3))
        return fail(RT_EINVAL, "need 0 <= th_min < th_max <= pi");
    return RT_OK;
}

// Shading constants of a 3-D problem (grid, line, camera): shared by the
// render and its census.  Needs the validated problem.
static rt_status build_shade3(const rt_problem3d *p, Shade3 *s) {
    rt_status st = RT_OK;
    const rt_grid3d &gr = p->grid;
    const rt_line &l = p->line;
    const float4 *tab = nullptr;
    st = partition_table(l, &tab);
    if (st != RT_OK) return st;
    constexpr double kH = 6.62607015e-27, kKB = 1.380649e-16, kC = 2.99792458e10, kAMU = 1.66053906660e-24,
                     kAU = 1.495978707e13, kZT0 = 0.1, kZT1 = 1.0e4;
    const double dln = std::log(gr.r_max_au / gr.r_min_au) / (gr.nr - 1);
    const double dth = (gr.th_max - gr.th_min) / (gr.nt - 1);
    const Geometry3 g = geometry3(p);
    std::memset(s, 0, sizeof *s);
    s->node = (const float4 *)p->nodes;
    s->ztab = tab;
    s->nr = gr.nr;
    s->nt = gr.nt;
    s->np = gr.np;
    const float *inv_r2n = nullptr;
    st = radius_table(gr, &inv_r2n);
    if (st != RT_OK) return st;
    s->inv_r2n = inv_r2n;
    s->u_scale = (float)(std::log(2.0) / dln);
    s->h_r = (float)(0.5 * std::log(2.0) / dln);
    s->log2_rmin = (float)std::log2(gr.r_min_au);
    const double thc = 0.5 * (gr.th_min + gr.th_max);
    s->cth_c = (float)std::cos(thc);
    s->sth_c = (float)std::sin(thc);
    s->inv_dth = (float)(1.0 / dth);
    s->half_nt1 = 0.5f * (float)(gr.nt - 1);
    s->inv_dph = (float)(gr.np / (2.0 * kPI3));
    s->fnp = (float)gr.np;
    s->fnr = (float)gr.nr;
    s->fnt = (float)gr.nt;
    const double l0 = std::log2(kZT0), l1 = std::log2(kZT1), log2e = 1.0 / std::log(2.0);
    s->zt_l2t0 = (float)l0;
    s->zt_scale = (float)((kZTableNodes - 1) / (l1 - l0));
    s->el_log2e = (float)(l.e_l_k * log2e);
    const double nu = l.nu0_hz;
    s->theta = (float)(kH * nu / kKB);
    s->c_s = (float)(p->intensity_scale * 2.0 * kH * nu * nu * nu / (kC * kC));
    const double bul = l.a_ul * kC * kC / (2.0 * kH * nu * nu * nu);
    const double blu = l.g_u / l.g_l * bul;
    s->c_k = (float)((kH * nu / (4.0 * kPI3)) * blu * l.g_l * (kC / nu) * kAU / (std::sqrt(kPI3) * 1e5) * log2e);
    s->c_alpha = (float)((2.0 * kKB / (l.m_co_amu * kAMU) + p->v_turb * p->v_turb * 2.0 * kKB / (l.m_mol_amu * kAMU)) /
                        1e10);
    s->sqrt_log2e = (float)std::sqrt(log2e);
    s->si = (float)g.si;
    s->ci = (float)g.ci;
    s->vsys = (float)p->spec.v_sys_kms;
    const double edge = std::max(0.5 * kPI3 - gr.th_min, gr.th_max - 0.5 * kPI3) + dth;
    s->zeta = edge < 1.5 ? (float)std::tan(edge) : 0.0f;
    return RT_OK;
}

} // namespace rt

using namespace rt;

extern "C" {

rt_status rt_pack_fields3d(const rt_grid3d *grid, const float *ln_nh2, const float *temp_k, const float *x_co,
                           const float *v_r, const float *v_theta, const float *v_phi, float *nodes, void *stream) {
    rt_status st = validate_grid3(grid);
    if (st != RT_OK) return st;
    if (!ln_nh2 || !temp_k || !x_co) return fail(RT_EINVAL, "ln_nh2, temp_k and x_co are required");
    if (!nodes) return fail(RT_EINVAL, "nodes is NULL");
    if (((uintptr_t)nodes & 15) != 0) return fail(RT_EINVAL, "nodes must be 16-byte aligned");
    const uint32_t n = (uint32_t)((int64_t)grid->nr * grid->nt * grid->np);
    const unsigned blocks = (unsigned)std::min<uint32_t>((n + 255) / 256, 16384u);
    hipLaunchKernelGGL(pack3, dim3(blocks), dim3(256), 0, (hipStream_t)stream, ln_nh2, temp_k, x_co, v_r, v_theta,
                       v_phi, (float4 *)nodes, n);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? RT_OK : fail_hip(e, "pack launch");
}

rt_status rt_render_census_3d(const rt_problem3d *p, uint8_t *mask, int64_t *counts, void *stream) {
    if (!p) return fail(RT_EINVAL, "problem is NULL");
    rt_status st = validate_grid3(&p->grid);
    if (st != RT_OK) return st;
    st = validate_view(p->line, p->cam, p->spec, p->nsamp, p->intensity_scale, 180.0);
    if (st != RT_OK) return st;
    if (!counts) return fail(RT_EINVAL, "counts is NULL");
    const Geometry3 g = geometry3(p);
    // the shading counts need the node records
    const int shade = p->nodes && ((uintptr_t)p->nodes & 15) == 0 ? 1 : 0;
    Shade3 s;
    std::memset(&s, 0, sizeof s);
    if (shade && (st = build_shade3(p, &s)) != RT_OK) return st;
    hipStream_t hs = (hipStream_t)stream;
    hipError_t e;
    unsigned long long *d = (unsigned long long *)stream_workspace(hs, kWsCensus, 4 * sizeof(unsigned long long), &e);
    if (!d) return fail_hip(e, "census counters");
    const int npix = p->cam.nx * p->cam.ny;
    int chunks = 1;
    while (shade && chunks < 64 && (long)((npix + 255) / 256) * chunks < 4096 && p->nsamp >= 16 * chunks) chunks *= 2;
    hipLaunchKernelGGL(census3_zero, dim3(1), dim3(64), 0, hs, d);
    hipLaunchKernelGGL(census3, dim3((npix + 255) / 256, chunks), dim3(256), 0, hs, g, s, mask, d, shade);
    unsigned long long h[4] = {0, 0, 0, 0};
    if ((e = hipGetLastError()) == hipSuccess) e = hipMemcpyAsync(h, d, sizeof h, hipMemcpyDeviceToHost, hs);
    if (e == hipSuccess) e = hipStreamSynchronize(hs);
    if (e != hipSuccess) return fail_hip(e, "3-D census");
    counts[0] = (int64_t)h[0];
    counts[1] = (int64_t)h[0] * p->nsamp;
    counts[2] = shade ? (int64_t)h[1] : -1;
    counts[3] = shade ? (int64_t)h[2] : -1;
    counts[4] = shade ? (int64_t)h[3] : -1;
    return RT_OK;
}

rt_status rt_render_cube_3d(const rt_problem3d *p, float *cube, void *stream) {
    if (!p) return fail(RT_EINVAL, "problem is NULL");
    rt_status st = validate_grid3(&p->grid);
    if (st != RT_OK) return st;
    if (!p->nodes) return fail(RT_EINVAL, "nodes is NULL");
    if (((uintptr_t)p->nodes & 15) != 0) return fail(RT_EINVAL, "nodes must be 16-byte aligned");
    if (!(std::isfinite(p->v_turb) && p->v_turb >= 0)) return fail(RT_EINVAL, "need v_turb >= 0");
    st = validate_view(p->line, p->cam, p->spec, p->nsamp, p->intensity_scale, 180.0);
    if (st != RT_OK) return st;
    if (!cube) return fail(RT_EINVAL, "cube is NULL");
    Shade3 s;
    st = build_shade3(p, &s);
    if (st != RT_OK) return st;
    const Geometry3 g = geometry3(p);
    const long npix = (long)p->cam.nx * p->cam.ny;
    const bool windows = !channel_block_option() && !ray_split_option();
    int cb, nsplit;
    forward_shape3(std::min(p->spec.nch, kLaunchChannels), npix, p->nsamp, &cb, &nsplit);
    if (channel_block_option()) cb = channel_block_option();
    if (ray_split_option()) nsplit = ray_split_option();
    const size_t plane = (size_t)p->cam.nx * p->cam.ny;
    for (int c0 = 0; c0 < p->spec.nch; c0 += kLaunchChannels) {
        Channels ch;
        std::memset(&ch, 0, sizeof ch);
        ch.n = std::min(kLaunchChannels, p->spec.nch - c0);
        for (int c = 0; c < ch.n; ++c) ch.v[c] = (float)p->spec.v_kms[c0 + c];
        if (windows) {
            int wcb, lsplit;
            double dv = 0.0;
            window_shape(ch.n, npix, p->nsamp, &wcb, &lsplit, kWinWaves3);
            const bool uniform = uniform_spacing(p->spec.v_kms + c0, ch.n, &dv) && dv != 0.0;
            Windows win;
            unit_windows(ch, wcb, uniform ? dv : 0.0, &win);
            const hipError_t e = launch_forward3_win(g, s, ch, win, cube + (size_t)c0 * plane, wcb, uniform, lsplit,
                                                     (hipStream_t)stream);
            if (e != hipSuccess) return fail_hip(e, "3-D forward launch");
            continue;
        }
        const hipError_t e = launch_forward3(g, s, ch, cube + (size_t)c0 * plane, cb, nsplit, (hipStream_t)stream);
        if (e != hipSuccess) return fail_hip(e, "3-D forward launch");
    }
    return RT_OK;
}

} // extern "C"
