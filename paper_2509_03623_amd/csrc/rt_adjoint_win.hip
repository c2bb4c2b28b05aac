// rt_adjoint_win.hip -- the checkpoint-free reverse march over line windows.
//
// The arithmetic is that of march_tau_pixel (rt_adjoint_dev.h): sweep 1, back
// to front, adds up each channel's depth (compensated) and runs J to the
// observer; sweep 2 re-adds the depths from -tau_tot and writes each sample's
// cotangents.  The layout is that of the windowed forward march: four lanes
// share a pixel with the channels interleaved over them (lane h: c0 + 4 i + h),
// a wave holds a 4 x 4 tile, lane h reads every fourth tape entry and forms the
// unit mask of its line, and the quad marches the units that some pixel of the
// wave needs (rt_kernels.h, "line windows").  A channel outside the window has
// x = 0 to float, so J, both depth sums and every cotangent stay as they are.
//
// Faint samples have loops of their own: 1 - 2^-x is x ln2 to the bit there.
// Sweep 1, K < min(2^-26, nsamp^-2): the depth goes to the low word of the sum
// alone.  That word stays under nsamp K, so a ray's additions to it are off by
// less than 2^-25 in all, half the last bit of the transmission.  Sweep 2, K <
// min(2^-40, 2^-26 / nsamp): besides, the transmission is kept from the last
// sample that was not faint; a ray's faint samples together change it by less than
// half its last bit.  Up to 8192 samples the bounds are 2^-26 and 2^-40, and a
// kernel of its own has them as literals (146 x 88 x 16 x 457: 272 us, and 280 with
// the bounds in registers; 2^-26 / nsamp for both sweeps: 288).
//
// Bound: VALU issue (512^2 x 64 x 512: an instruction every 5.5 cycles of a SIMD,
// 4 being an FMA's) and, at 16 channels a lane, the registers of sweep 2 (sums,
// w, J, u and the velocity of each channel: 137, three waves per SIMD; held to
// four waves it gains 2 % on large images and loses 6 % on small ones).
// Measured against adj_march_tau: 512^2 x 64 x 512 4.86 -> 1.74 ms, 256^2 x 48
// x 256 0.587 -> 0.249 ms.
#include <type_traits>

#include "rt_adjoint.h"
#include "rt_adjoint_dev.h"

namespace rt {

// log2 of the faint samples' bounds: nsamp rounded up to a power of two, or for up to
// 2^kLongLog2 samples (LONG false) literals
constexpr int kLongLog2 = 13;
template <bool LONG>
__device__ __forceinline__ float faint_sum(int nsamp) {
    return LONG ? -2.0f * (float)(32 - __clz(nsamp - 1)) : -2.0f * kLongLog2;
}
template <bool LONG>
__device__ __forceinline__ float faint_still(int nsamp) {
    return LONG ? -fmaxf(40.0f, (float)(26 + 32 - __clz(nsamp - 1))) : -40.0f;
}

template <int CB, bool CUBE, bool UNIFORM, bool LONG>
__global__ __launch_bounds__(256) void adj_march_win(int nsamp, int nx, int ny, int plane, int nblk, Channels ch,
                                                     Windows win, const float4 *__restrict__ tape,
                                                     const int2 *__restrict__ span,
                                                     const float *__restrict__ dl_dcube,
                                                     const float *__restrict__ target, float4 *__restrict__ cot,
                                                     float *__restrict__ cube_out) {
    constexpr int G = kLanesPerPixel, U = unit_slots(CB), NU = CB / U;
    static_assert(U == 1, "one channel per lane in a unit");
    // the channel blocks of one tile take workgroup ids 8 apart: one XCD's L2
    // holds the tile's tape for all of them
    const int id = blockIdx.x, r8 = id >> 3;
    const int blk = r8 % nblk, tile = (r8 / nblk) * 8 + (id & 7);
    const int tiles_x = (nx + 7) / 8;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, h = lane & 3, slot = lane >> 2;
    const int p = (tile % tiles_x) * 8 + (wave & 1) * 4 + (slot & 3);
    const int q = (tile / tiles_x) * 8 + (wave >> 1) * 4 + (slot >> 2);
    const bool inside = p < nx && q < ny;
    const int pix = inside ? q * nx + p : 0;
    const size_t npix = (size_t)nx * ny;
    const int c0 = blk * CB * G, u0 = blk * NU;
    // this lane's own run of samples with opacity (empty: first > last)
    int2 ks = inside ? span_of(span[pix], nsamp) : make_int2(nsamp, -1);
    const int kf = wave_min(ks.x), kl = wave_max(ks.y);
    const float faint1 = faint_sum<LONG>(nsamp), faint2 = faint_still<LONG>(nsamp);
    float vc[CB], th[CB], tl[CB], J[CB], w[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        vc[c] = ch.v[c0 + c * G + h];
        th[c] = 0.0f;
        tl[c] = 0.0f;
        J[c] = 0.0f;
    }
    const float v0 = ch.v[c0];
    // this lane's tape entry of the step that starts at sample k; the tape may
    // hold nothing valid outside the ray's own run, which counts as no opacity
    auto entry = [&](int k) { return tape[(size_t)max(k - h, 0) * npix + pix]; };
    auto in_run = [&](int k) { return k - h >= ks.x && k - h <= ks.y; };
    auto clean = [&](const float4 &e, bool on) {
        return make_float4(on ? e.x : 0.0f, on ? e.y : 0.0f, on ? e.z : 0.0f, on ? e.w : 0.0f);
    };
    auto own_mask = [&](const float4 &e, float lK, bool on) {
        SampleQ s;
        s.S = e.x; s.K = e.y; s.a = e.z; s.b = e.w;
        return or_over_pixels(unit_mask<NU, G, UNIFORM>(s, lK, on, v0, win, u0));
    };
    auto sweep1 = [&](int k, const float4 &e) {
        const float own_lk = flog2(e.y);
        const unsigned mask = own_mask(e, own_lk, in_run(k));
        const unsigned long long bright = __builtin_amdgcn_ballot_w64(!(own_lk < faint1));
        const unsigned long long thick = __builtin_amdgcn_ballot_w64(!(own_lk < kThinLog2K));
        auto step = [&](auto jc) {
            constexpr int N = decltype(jc)::value;
            constexpr unsigned long long mine = 0x1111111111111111ull << N;
            const unsigned m = (unsigned)__builtin_amdgcn_readlane((int)mask, N);
            if (m == 0) return;
            const float S = group_lane<G, N>(e.x), lK = group_lane<G, N>(own_lk);
            const float a = group_lane<G, N>(e.z), b = group_lane<G, N>(e.w);
            if ((bright & mine) == 0) {
#pragma unroll
                for (int c = 0; c < CB; ++c) {
                    if (!(m & (1u << c))) continue;
                    const float d = fmaf(-vc[c], b, a);
                    const float x = fexp2(fmaf(-d, d, lK));
                    tl[c] += x;
                    if (CUBE) J[c] = fmaf(x * kLn2, S - J[c], J[c]);
                }
                return;
            }
            // the error of th + x, exact with the larger operand first (both
            // are >= 0, so their bit patterns order like the values)
            auto depth = [&](int c, float x) {
                const float sum = th[c] + x;
                const unsigned ut = __float_as_uint(th[c]), ux = __float_as_uint(x);
                tl[c] += __uint_as_float(min(ut, ux)) - (sum - __uint_as_float(max(ut, ux)));
                th[c] = sum;
            };
            if ((thick & mine) == 0) {
#pragma unroll
                for (int c = 0; c < CB; ++c) {
                    if (!(m & (1u << c))) continue;
                    const float d = fmaf(-vc[c], b, a);
                    const float x = fexp2(fmaf(-d, d, lK));
                    depth(c, x);
                    if (CUBE) J[c] = fmaf(om_series3(x), S - J[c], J[c]);
                }
                return;
            }
            // a depth of kThinK or less takes the series, also in a thick
            // sample's wings: x = 0 keeps J to the bit
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                if (!(m & (1u << c))) continue;
                const float d = fmaf(-vc[c], b, a);
                const float x = fexp2(fmaf(-d, d, lK));
                depth(c, x);
                if (CUBE) {
                    const bool thin = x < kThinK;
                    const float smj = S - J[c];
                    J[c] = fmaf(thin ? om_series3(x) : -fexp2(-x), smj, thin ? J[c] : S);
                }
            }
        };
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
        step(std::integral_constant<int, 2>{});
        step(std::integral_constant<int, 3>{});
    };
    if (kf <= kl) {
        float4 next = entry(kl);
        for (int k = kl; k >= kf; k -= G) {
            const float4 e = clean(next, in_run(k));
            next = entry(k - G);
            sweep1(k, e);
        }
    }
    // padding channels read a valid channel's plane and get w = 0
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        const int cc = c0 + c * G + h;
        const size_t i = (size_t)min(cc, ch.n - 1) * plane + pix;
        const bool valid = inside && cc < ch.n;
        if (CUBE && cube_out && valid) cube_out[i] = J[c];
        const float wc = CUBE && target ? 2.0f * (J[c] - target[i]) : dl_dcube[i];
        w[c] = valid ? wc : 0.0f;
    }
    if (kf > kl) return;
    // (th, tl): minus the prefix depth in front of the current sample; u = w Tr
    float u[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        th[c] = -th[c];
        tl[c] = -tl[c];
        J[c] = 0.0f;
        u[c] = w[c] * fexp2(th[c] + tl[c]);
    }
    float4 next = entry(kl);
    for (int k = kl; k >= kf; k -= G) {
        const int kk = k - h;
        const bool on = in_run(k);
        const float4 e = clean(next, on);
        next = entry(k - G);
        const float own_lk = flog2(e.y);
        const unsigned mask = own_mask(e, own_lk, on);
        const unsigned long long bright = __builtin_amdgcn_ballot_w64(!(own_lk < faint2));
        const unsigned long long thick = __builtin_amdgcn_ballot_w64(!(own_lk < kThinLog2K));
        float4 res = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        auto step = [&](auto jc) {
            constexpr int N = decltype(jc)::value;
            constexpr unsigned long long mine = 0x1111111111111111ull << N;
            const unsigned m = (unsigned)__builtin_amdgcn_readlane((int)mask, N);
            if (m == 0) return;
            const float S = group_lane<G, N>(e.x), lK = group_lane<G, N>(own_lk);
            const float a = group_lane<G, N>(e.z), b = group_lane<G, N>(e.w);
            float cS = 0.0f, cX = 0.0f, ca = 0.0f, cb = 0.0f;
            // the products of one channel: gg = u (S - J) x into the sums
            auto sums = [&](int c, float d, float gg) {
                cX += gg;
                const float gd = gg * d;
                ca += gd;
                cb = fmaf(-vc[c], gd, cb);
            };
            // adds x to the running sum and renews u.  The sum is minus the depth
            // of this sample and of those in front of it, so not the smaller
            // operand, but for rounding and for the samples that sweep 1 put in
            // the low word: there the correction may be off by an ulp of x (2^-49,
            // under 2^-29 for a ray)
            auto renew = [&](int c, float x) {
                const float sum = th[c] + x;
                tl[c] += x - (sum - th[c]);
                th[c] = sum;
                u[c] = w[c] * fexp2(sum + tl[c]);
            };
            if ((bright & mine) == 0) {
#pragma unroll
                for (int c = 0; c < CB; ++c) {
                    if (!(m & (1u << c))) continue;
                    const float d = fmaf(-vc[c], b, a);
                    const float x = fexp2(fmaf(-d, d, lK));
                    const float smj = S - J[c], ux = u[c] * x;
                    tl[c] += x;
                    J[c] = fmaf(x * kLn2, smj, J[c]);
                    cS += ux;
                    sums(c, d, ux * smj);
                }
                cS *= kLn2;
            } else if ((thick & mine) == 0) {
#pragma unroll
                for (int c = 0; c < CB; ++c) {
                    if (!(m & (1u << c))) continue;
                    const float d = fmaf(-vc[c], b, a);
                    const float x = fexp2(fmaf(-d, d, lK));
                    const float smj = S - J[c], gg = u[c] * smj * x, om = om_series3(x);
                    J[c] = fmaf(om, smj, J[c]);
                    renew(c, x);
                    cS = fmaf(u[c], om, cS);
                    sums(c, d, gg);
                }
            } else {
#pragma unroll
                for (int c = 0; c < CB; ++c) {
                    if (!(m & (1u << c))) continue;
                    const float d = fmaf(-vc[c], b, a);
                    const float x = fexp2(fmaf(-d, d, lK));
                    const float smj = S - J[c], gg = u[c] * smj * x;
                    const bool thin = x < kThinK;
                    const float att = fexp2(-x), om = thin ? om_series3(x) : 1.0f - att;
                    J[c] = fmaf(thin ? om : -att, smj, thin ? J[c] : S);
                    renew(c, x);
                    cS = fmaf(u[c], om, cS);
                    sums(c, d, gg);
                }
            }
            const float md = -2.0f * kLn2 * kLn2;
            float4 o = make_float4(cS, cX * kLn2, ca * md, cb * md);
            o.x += swap_pair(o.x); o.y += swap_pair(o.y); o.z += swap_pair(o.z); o.w += swap_pair(o.w);
            o.x += swap_half_quad(o.x); o.y += swap_half_quad(o.y);
            o.z += swap_half_quad(o.z); o.w += swap_half_quad(o.w);
            // every lane keeps the sums of its own sample
            res.x = h == N ? o.x : res.x;
            res.y = h == N ? o.y : res.y;
            res.z = h == N ? o.z : res.z;
            res.w = h == N ? o.w : res.w;
        };
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
        step(std::integral_constant<int, 2>{});
        step(std::integral_constant<int, 3>{});
        if (on) cot[((size_t)blk * nsamp + kk) * npix + pix] = res;
    }
}

template <int CB>
static hipError_t launch_win_t(int nsamp, int nx, int ny, int plane, const Channels &ch, const Windows &win,
                               bool uniform, const float4 *tape, const int2 *span, const float *dl,
                               const float *target, float4 *cot, float *cube_out, hipStream_t st) {
    const int nblk = (ch.n + kLanesPerPixel * CB - 1) / (kLanesPerPixel * CB);
    const long tiles = (long)((nx + 7) / 8) * ((ny + 7) / 8);
    const dim3 grid((unsigned)((tiles + 7) / 8 * 8 * nblk));
    const bool cube = target || cube_out;
    const bool lng = nsamp > 1 << kLongLog2;
#define RT_WIN_CASE(C, U, L)                                                                                     \
    if (cube == C && uniform == U && lng == L) {                                                                 \
        hipLaunchKernelGGL((adj_march_win<CB, C, U, L>), grid, dim3(256), 0, st, nsamp, nx, ny, plane, nblk, ch, \
                           win, tape, span, dl, target, cot, cube_out);                                          \
        return hipGetLastError();                                                                                \
    }
    RT_WIN_CASE(true, true, false) RT_WIN_CASE(true, false, false)
    RT_WIN_CASE(false, true, false) RT_WIN_CASE(false, false, false)
    RT_WIN_CASE(true, true, true) RT_WIN_CASE(true, false, true)
    RT_WIN_CASE(false, true, true) RT_WIN_CASE(false, false, true)
#undef RT_WIN_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_adj_march_win(int cb, int nsamp, int nx, int ny, int plane, const Channels &ch, const Windows &win,
                                bool uniform, const float4 *tape, const int2 *span, const float *dl,
                                const float *target, float4 *cot, float *cube_out, hipStream_t st) {
    switch (cb) {
    case 4: return launch_win_t<4>(nsamp, nx, ny, plane, ch, win, uniform, tape, span, dl, target, cot, cube_out, st);
    case 8: return launch_win_t<8>(nsamp, nx, ny, plane, ch, win, uniform, tape, span, dl, target, cot, cube_out, st);
    case 10: return launch_win_t<10>(nsamp, nx, ny, plane, ch, win, uniform, tape, span, dl, target, cot, cube_out, st);
    case 12: return launch_win_t<12>(nsamp, nx, ny, plane, ch, win, uniform, tape, span, dl, target, cot, cube_out, st);
    case 14: return launch_win_t<14>(nsamp, nx, ny, plane, ch, win, uniform, tape, span, dl, target, cot, cube_out, st);
    case 16: return launch_win_t<16>(nsamp, nx, ny, plane, ch, win, uniform, tape, span, dl, target, cot, cube_out, st);
    default: return hipErrorInvalidValue;
    }
}

} // namespace rt
