// rt_beam.hip -- restoring-beam convolution of a model cube (gfx950).
//
// A model cube is compared with an interferometric image only after both are
// at the same resolution: every channel map is convolved with the image's
// elliptical Gaussian beam (FWHM bmaj >= bmin in pixels, major axis at bpa
// from +y towards -x), sampled at integer offsets within |dx|, |dy| <= R =
// ceil(3 sigma_maj), normalised to unit sum, zero outside the image.  The
// kernel is point-symmetric and the padding is zeros, so the operator is its
// own adjoint: the backward of the convolution is the same call.
//
// beam_weights (one workgroup) evaluates the (2R+1)^2 weights in float,
// normalises them by their workgroup-reduced sum and stores them.  beam_conv: one
// workgroup per 64 x 64 output tile of one channel (64 x 32 in small launches),
// compiled for each R; the
// tile plus its halo is staged in LDS (zeros outside the image), all of a
// lane's float4 loads in flight together, with the weights; each lane forms 8
// consecutive outputs of two rows (or one) from the float4 of a tile row it reads
// once, the taps and their window all in registers by constant index.
//
// Bound: FMA issue, (2R+1)^2 FMAs per output; with three registers read of
// which two are often of one bank an FMA takes 3 cycles of the 2 it could.
// 512^2 x 64 channels, R = 8: 109 us a call; 153 with 4-byte reads and stores
// and the taps in a loop.  Same loop of calls, back to back: R = 3 55 (90), R = 4
// 48 (88), R = 8 134 (175), R = 12 221 (280), R = 23 804 (1036); 150 x 133 x 40,
// R = 8, 20 (22).
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "../../include/rtcube.h"
#include "rt_host.h"

namespace rt {

constexpr int kBeamOut = 8;                                // outputs of a lane: columns, and 1 or 2 rows
constexpr int kBeamTX = 64;
constexpr int beam_ty(int rows) { return 256 / (kBeamTX / kBeamOut) * rows; }
// halo left and right in whole float4; values of a tile row that a lane reads
// (from its first column of the halo); half of the float4 of a tile row, stored
// even ones first (a lane's outputs are two float4 wide, so that neighbouring
// lanes then read neighbouring float4), and the row pitch in float4
constexpr int beam_halo(int R) { return (R + 3) / 4 * 4; }
constexpr int beam_values(int R) { return (beam_halo(R) + R + kBeamOut + 3) / 4 * 4; }
constexpr int beam_half(int R) { return (kBeamTX / 4 + beam_halo(R) / 2 + 1) / 2; }
constexpr int beam_pitch(int R) { return 2 * beam_half(R); }

__global__ __launch_bounds__(256) void beam_weights(float *__restrict__ w, int R, float inv_smaj, float inv_smin,
                                                    float spa, float cpa) {
    __shared__ float part[256];
    const int n = 2 * R + 1, nn = n * n;
    auto weight = [&](int idx) {
        const float dy = (float)(idx / n - R), dx = (float)(idx % n - R);
        const float u = fmaf(-dx, spa, dy * cpa) * inv_smaj, v = fmaf(dx, cpa, dy * spa) * inv_smin;
        return expf(-0.5f * fmaf(u, u, v * v));
    };
    float s = 0.0f;
    for (int i = threadIdx.x; i < nn; i += blockDim.x) s += weight(i);
    part[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) part[threadIdx.x] += part[threadIdx.x + h];
        __syncthreads();
    }
    const float inv = 1.0f / part[0];
    for (int i = threadIdx.x; i < nn; i += blockDim.x) w[i] = weight(i) * inv;
}

template <int R, bool VEC, int ROWS>
__global__ __launch_bounds__(256) void beam_conv(const float *__restrict__ in, float *__restrict__ out,
                                                 const float *__restrict__ w, int nx, int ny) {
    constexpr int n = 2 * R + 1, NW = (n + 3) / 4 * 4;       // taps of a row, padded to whole float4
    constexpr int TY = beam_ty(ROWS);
    constexpr int RX = beam_halo(R), W4 = kBeamTX / 4 + RX / 2;   // a tile row in float4
    constexpr int H = TY + 2 * R, P = beam_pitch(R), E = beam_half(R), NV = beam_values(R);
    __shared__ float4 tile[H * P];
    __shared__ __attribute__((aligned(16))) float wk[n * NW];
    const int x0 = blockIdx.x * kBeamTX, y0 = blockIdx.y * TY;
    const size_t plane = (size_t)nx * ny;
    const float *src = in + blockIdx.z * plane;
    constexpr int NL = (H * W4 + 255) / 256;                 // all loads of a lane in flight at once
    float4 f[NL];
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        const int i = (int)threadIdx.x + 256 * k;
        const int ly = i / W4, gy = y0 - R + ly, gx = x0 - RX + 4 * (i - ly * W4);
        f[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (gy < 0 || gy >= ny || ly >= H) continue;
        const float *p = src + (size_t)gy * nx;
        if (VEC) {
            if (gx >= 0 && gx < nx) f[k] = *(const float4 *)(p + gx);
        } else {
            if (gx >= 0 && gx < nx) f[k].x = p[gx];
            if (gx >= -1 && gx < nx - 1) f[k].y = p[gx + 1];
            if (gx >= -2 && gx < nx - 2) f[k].z = p[gx + 2];
            if (gx >= -3 && gx < nx - 3) f[k].w = p[gx + 3];
        }
    }
    for (int i = threadIdx.x; i < n * NW; i += 256) {
        const int j = i / NW, k = i - j * NW;
        wk[i] = k < n ? w[j * n + k] : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        const int i = (int)threadIdx.x + 256 * k, ly = i / W4, c = i - ly * W4;
        if (ly < H) tile[ly * P + (c & 1) * E + (c >> 1)] = f[k];
    }
    __syncthreads();
    constexpr int LX = kBeamTX / kBeamOut;
    const int ty = (int)threadIdx.x / LX * ROWS;         // first of the lane's output rows
    const int tx = (int)threadIdx.x % LX * kBeamOut;          // and columns
    float acc[ROWS][kBeamOut];
#pragma unroll
    for (int y = 0; y < ROWS; ++y)
#pragma unroll
        for (int q = 0; q < kBeamOut; ++q) acc[y][q] = 0.0f;
    // out(y, x) = sum_{j, i} K[j][i] in(y + R - j, x + R - i); K is point-symmetric
    // (K[j][i] = K[2R-j][2R-i]), so equally sum K[j][i] in(y - R + j, x - R + i).
    // Row r of the tile is row j = r - y of the kernel for output row y.
    auto row = [&](int r, auto first, auto last) {
        float v[NV];
        const float4 *src4 = tile + (ty + r) * P + tx / kBeamOut;
#pragma unroll
        for (int i = 0; i < NV / 4; ++i) {
            const float4 f = src4[(i & 1) * E + (i >> 1)];
            v[4 * i] = f.x; v[4 * i + 1] = f.y; v[4 * i + 2] = f.z; v[4 * i + 3] = f.w;
        }
#pragma unroll
        for (int y = decltype(first)::value; y <= decltype(last)::value; ++y) {
            const float4 *k4 = (const float4 *)(wk + (r - y) * NW);
#pragma unroll
            for (int i4 = 0; i4 < NW / 4; ++i4) {
                const float4 f = k4[i4];
                const float k[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (4 * i4 + t < n)
#pragma unroll
                        for (int q = 0; q < kBeamOut; ++q) acc[y][q] = fmaf(k[t], v[RX - R + 4 * i4 + t + q], acc[y][q]);
            }
        }
    };
    constexpr std::integral_constant<int, 0> top{};
    constexpr std::integral_constant<int, ROWS - 1> bottom{};
    if constexpr (ROWS == 2) row(0, top, top);
    for (int r = ROWS - 1; r < n; ++r) row(r, top, bottom);
    if constexpr (ROWS == 2) row(n, bottom, bottom);
#pragma unroll
    for (int yy = 0; yy < ROWS; ++yy) {
        const int y = y0 + ty + yy;
        if (y >= ny) return;
        float *dst = out + blockIdx.z * plane + (size_t)y * nx + x0 + tx;
        if (VEC) {
#pragma unroll
            for (int q = 0; q < kBeamOut; q += 4)
                if (x0 + tx + q < nx)
                    *(float4 *)(dst + q) = make_float4(acc[yy][q], acc[yy][q + 1], acc[yy][q + 2], acc[yy][q + 3]);
        } else {
#pragma unroll
            for (int q = 0; q < kBeamOut; ++q)
                if (x0 + tx + q < nx) dst[q] = acc[yy][q];
        }
    }
}

// Launches of at most one two-row tile a CU (256) have a wave on each SIMD, which
// issues no more than an FMA in 5 cycles: from R = 8 on one row a lane, twice the
// waves, is faster there.  Two rows and one, us: 65 x 65 x 8 R = 8 16.8, 11.8, R =
// 23 97, 56; 256 tiles R = 8 16.4, 15.1, R = 23 93, 79; but 256 tiles R = 5 10.6,
// 12.8, and 384 tiles R = 8 17.7, 18.6, 512 R = 23 113, 140.
constexpr long kBeamFew = 256;
constexpr int kBeamFewR = 8;

template <int R>
static hipError_t launch_conv(const float *in, float *out, const float *w, int R_, int nch, int ny, int nx,
                              hipStream_t st) {
    if constexpr (R > RT_BEAM_MAX_RADIUS) {
        return hipErrorInvalidValue;
    } else {
        if (R_ != R) return launch_conv<R + 1>(in, out, w, R_, nch, ny, nx, st);
        const unsigned tx = (nx + kBeamTX - 1) / kBeamTX;
        const dim3 one(tx, (ny + beam_ty(1) - 1) / beam_ty(1), nch), two(tx, (ny + beam_ty(2) - 1) / beam_ty(2), nch);
        // rows of whole, aligned float4: every float4 of the tile is inside or outside as a whole
        const bool vec = nx % 4 == 0 && (((uintptr_t)in | (uintptr_t)out) & 15) == 0;
        if constexpr (R >= kBeamFewR) {
            if ((long)two.x * two.y * two.z <= kBeamFew) {
                hipLaunchKernelGGL((beam_conv<R, false, 1>), one, dim3(256), 0, st, in, out, w, nx, ny);
                return hipGetLastError();
            }
        }
        if (vec) hipLaunchKernelGGL((beam_conv<R, true, 2>), two, dim3(256), 0, st, in, out, w, nx, ny);
        else hipLaunchKernelGGL((beam_conv<R, false, 2>), two, dim3(256), 0, st, in, out, w, nx, ny);
        return hipGetLastError();
    }
}

} // namespace rt

using namespace rt;

namespace rt {

rt_status validate_beam(const rt_beam &b) {
    if (!(std::isfinite(b.bmaj_px) && std::isfinite(b.bmin_px) && std::isfinite(b.bpa_deg) && b.bmin_px > 0.0 &&
          b.bmaj_px >= b.bmin_px))
        return fail(RT_EINVAL, "need 0 < bmin_px <= bmaj_px and a finite bpa_deg");
    const int R = (int)std::ceil(3.0 * b.bmaj_px / (2.0 * std::sqrt(2.0 * std::log(2.0))));
    if (R > RT_BEAM_MAX_RADIUS) return fail(RT_EINVAL, "beam support radius %d exceeds %d pixels", R, RT_BEAM_MAX_RADIUS);
    return RT_OK;
}

rt_status beam_in_place(float *cube, int nch, int ny, int nx, const rt_beam &b, hipStream_t st) {
    const size_t bytes = (size_t)nch * nx * ny * sizeof(float);
    hipError_t e;
    float *tmp = (float *)stream_workspace(st, kWsBeamCube, bytes, &e);
    if (!tmp) return fail_hip(e, "beam cube workspace");
    rt_status rs = rt_beam_convolve(cube, tmp, nch, ny, nx, &b, st);
    if (rs != RT_OK) return rs;
    e = hipMemcpyAsync(cube, tmp, bytes, hipMemcpyDeviceToDevice, st);
    return e == hipSuccess ? RT_OK : fail_hip(e, "beam copy");
}

} // namespace rt

extern "C" rt_status rt_beam_convolve(const float *in, float *out, int32_t nch, int32_t ny, int32_t nx,
                                      const rt_beam *beam, void *stream) {
    if (!in || !out) return fail(RT_EINVAL, "in and out are required");
    if (!beam) return fail(RT_EINVAL, "beam is NULL");
    if (nch < 1 || ny < 1 || nx < 1) return fail(RT_EINVAL, "need nch, ny, nx >= 1");
    if (nch > 65535 || (int64_t)nx * ny > (int64_t)1 << 30) return fail(RT_EINVAL, "cube too large");
    rt_status vs = validate_beam(*beam);
    if (vs != RT_OK) return vs;
    const double bmaj = beam->bmaj_px, bmin = beam->bmin_px, bpa = beam->bpa_deg;
    const double fw = 2.0 * std::sqrt(2.0 * std::log(2.0));
    const double smaj = bmaj / fw, smin = bmin / fw;
    const int R = (int)std::ceil(3.0 * smaj);
    const size_t bytes = (size_t)nch * nx * ny * sizeof(float);
    const char *a = (const char *)in, *b = (const char *)out;
    if (a < b + bytes && b < a + bytes) return fail(RT_EINVAL, "in and out overlap");
    hipStream_t st = (hipStream_t)stream;
    const int n = 2 * R + 1;
    hipError_t e;
    float *w = (float *)stream_workspace(st, kWsBeam, sizeof(float) * n * n, &e);
    if (!w) return fail_hip(e, "beam workspace");
    const double pa = bpa * 3.14159265358979323846 / 180.0;
    hipLaunchKernelGGL(beam_weights, dim3(1), dim3(256), 0, st, w, R, (float)(1.0 / smaj), (float)(1.0 / smin),
                       (float)std::sin(pa), (float)std::cos(pa));
    if ((e = hipGetLastError()) != hipSuccess) return fail_hip(e, "beam weights launch");
    if ((e = launch_conv<1>(in, out, w, R, nch, ny, nx, st)) != hipSuccess) return fail_hip(e, "beam convolution launch");
    return RT_OK;
}
