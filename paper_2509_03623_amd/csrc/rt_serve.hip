// rt_serve.hip -- device side of the render server: a persistent forward
// launch over the work items of every request in a batch, and the fused L2
// loss / cotangent of forward+adjoint requests.
//
// A batch holds up to max_slots requests; its work items are (request, 4 x 4
// pixel tile, 32-channel block) in request order.  An item is the windowed
// march of rt_forward.hip on one tile: the workgroup's four waves take
// consecutive quarters of the samples that can lie below the top taper, and
// the first composes the quarters front to back through LDS (the composition
// is associative), so an item's latency is a quarter of its rays'.  The launch
// has a fixed number of workgroups; each pulls the next item index from a
// device counter until the batch is exhausted, so items of small and large
// requests of the batch share the GPU.  Every wave exits once the counter
// passes the item count.
//
// Bound: VALU issue, as the forward march.  60 walkers at 128^2 x 32 x 256:
// 875 -> 295 us a launch (of about ten that overlap).  With blocks of 64
// channels (152 VGPRs, three waves per SIMD) an iteration took 4.9 ms against
// 4.2, and 64-channel requests no less.
#include <type_traits>

#include "rt_host.h"
#include "rt_serve.h"

namespace rt {

static_assert(kServeTile * kServeTile * kLanesPerPixel == 64, "one tile per wave");

// the unit ranges of a block in LDS (unevenly spaced channels)
struct ServeWindows {
    float lo[kServeCB], hi[kServeCB];
    float inv_unit;
};

template <bool UNIFORM>
__device__ __forceinline__ void serve_item(const ServeDesc &D, const float4 *ztab, const ServeWindows &win, int blk,
                                           int tile, float *parts) {
    constexpr int CB = kServeCB, G = kLanesPerPixel;
    const Geometry &g = D.g;
    const int split = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, h = lane & 3, slot = lane >> 2;
    const int p = (tile % D.tiles_x) * kServeTile + (slot & 3), q = (tile / D.tiles_x) * kServeTile + (slot >> 2);
    const int c0 = blk * kServeBlock;
    const bool inside = p < g.nx && q < g.ny;
    const RaySetup r = ray_setup(g, inside ? p : 0, inside ? q : 0);
    const bool live = inside && r.live;
    float I[CB], Tr[CB], vc[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        I[c] = 0.0f;
        Tr[c] = 1.0f;
        vc[c] = D.vch[c0 + c * G + h];
    }
    // (a ray that misses the grid goes beside it, as in rt_forward.hip: no
    // opacity, and no read of nodes that no ray of the image samples)
    const float px = live ? r.px : 4.0f * g.rc;
    if (__ballot(live) != 0) {
        const float half = 0.5f * (float)g.nsamp;
        const float v0 = D.vch[c0];
        const int2 own_range = live ? taper_range(g, D.s, r) : make_int2(g.nsamp, -1);
        const int kf = wave_min(own_range.x), kn = max(wave_max(own_range.y) + 1 - kf, 0);
        const int len = ((kn + 3) / 4 + G - 1) / G * G;
        const int k1 = kf + min(kn, (split + 1) * len);
        for (int k = kf + split * len; k < k1; k += G) {
            const int kk = min(k + h, k1 - 1);
            const float t = ((float)kk + 0.5f - half) * r.ds;
            const SampleQ own = shade_sample<false>(D.s, ztab, px, fmaf(t, r.wy, r.pmy), fmaf(t, r.wz, r.pmz), r.ds, 0);
            const float own_lk = flog2(own.K);
            const unsigned mask =
                or_over_pixels(unit_mask<CB, G, UNIFORM>(own, own_lk, live && k + h < k1, v0, win, 0));
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
    if (split > 0) {
        float *o = parts + (size_t)(split - 1) * (2 * CB * 64) + lane;
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            o[c * 64] = I[c];
            o[(CB + c) * 64] = Tr[c];
        }
    }
    __syncthreads();
    if (split == 0) {
        for (int j = 0; j < 3; ++j) {
            const float *o = parts + (size_t)j * (2 * CB * 64) + lane;
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                I[c] = fmaf(Tr[c], o[c * 64], I[c]);
                Tr[c] *= o[(CB + c) * 64];
            }
        }
        if (inside) {
            const size_t plane = (size_t)g.nx * g.ny, pix = (size_t)q * g.nx + p;
#pragma unroll
            for (int c = 0; c < CB; ++c)
                if (c0 + c * G + h < D.nch) D.cube[(size_t)(c0 + c * G + h) * plane + pix] = I[c];
        }
    }
}

__global__ __launch_bounds__(256) void serve_fwd(const ServeDesc *__restrict__ descs, int nreq, uint32_t nitems,
                                                 uint32_t *__restrict__ counter) {
    __shared__ float4 ztab[kZTableNodes - 1];
    __shared__ float parts[3 * 2 * kServeCB * 64];
    __shared__ ServeWindows win;
    __shared__ uint32_t s_item;
    __shared__ const float4 *s_tab;
    if (threadIdx.x == 0) s_tab = nullptr;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_item = atomicAdd(counter, 1u);
        __syncthreads();
        const uint32_t item = __builtin_amdgcn_readfirstlane(s_item);   // uniform: scalar from here on
        if (item >= nitems) break;
        // request of this item: last descriptor whose first item <= item
        int lo = 0, hi = nreq - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (descs[mid].item0 <= item) lo = mid; else hi = mid - 1;
        }
        // the request index is the same for every lane: keep its descriptor in
        // scalar registers for the whole item
        const ServeDesc D = descs[__builtin_amdgcn_readfirstlane(lo)];
        const uint32_t local = item - D.item0;
        const int blk = (int)(local % (uint32_t)D.nblk);
        const int tile = (int)(local / (uint32_t)D.nblk);
        const bool new_tab = s_tab != D.s.ztab;     // uniform: every lane reads the same s_tab
        const bool uniform = D.inv_unit != 0.0f;
        if (new_tab || !uniform) {
            __syncthreads();
            if (new_tab)
                for (int i = threadIdx.x; i < kZTableNodes - 1; i += 256) ztab[i] = D.s.ztab[i];
            if (threadIdx.x < kServeCB) {
                const int c = blk * kServeBlock + threadIdx.x * kLanesPerPixel;
                float a = __builtin_huge_valf(), b = -a;
                for (int j = c; j < min(c + kLanesPerPixel, D.nch); ++j) {
                    a = fminf(a, D.vch[j]);
                    b = fmaxf(b, D.vch[j]);
                }
                win.lo[threadIdx.x] = a;
                win.hi[threadIdx.x] = b;
            }
            __syncthreads();
            if (threadIdx.x == 0) s_tab = D.s.ztab;
        }
        if (uniform) {
            ServeWindows w;
            w.inv_unit = D.inv_unit;
            serve_item<true>(D, ztab, w, blk, tile, parts);
        } else {
            serve_item<false>(D, ztab, win, blk, tile, parts);
        }
    }
}

hipError_t launch_serve_fwd(const ServeDesc *descs, int nreq, uint32_t nitems, uint32_t *counter, int nwg,
                            hipStream_t st) {
    hipLaunchKernelGGL(serve_fwd, dim3(nwg), dim3(256), 0, st, descs, nreq, nitems, counter);
    return hipGetLastError();
}

// dl = 2 (cube - target); L += sum (cube - target)^2 (double atomics)
__global__ __launch_bounds__(256) void l2_loss(const float *__restrict__ cube, const float *__restrict__ target,
                                               float *__restrict__ dl, size_t n, double *__restrict__ loss) {
    __shared__ double part[256];
    double acc = 0.0;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const float r = cube[i] - target[i];
        dl[i] = 2.0f * r;
        acc += (double)r * (double)r;
    }
    part[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) part[threadIdx.x] += part[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) atomicAdd(loss, part[0]);
}

__global__ void zero_double(double *p) { *p = 0.0; }

// sum (cube - target)^2 over the elements of a grid of blocks in x, added to
// *loss by one double atomic a block; four loads of each array in flight a lane
__device__ __forceinline__ void l2_sum(const float *__restrict__ cube, const float *__restrict__ target, size_t n,
                                       double *__restrict__ loss) {
    __shared__ double part[256];
    const size_t step = (size_t)gridDim.x * 256;
    double acc = 0.0;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += 4 * step) {
        float c[4], t[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bool on = i + k * step < n;
            c[k] = on ? cube[i + k * step] : 0.0f;
            t[k] = on ? target[i + k * step] : 0.0f;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double r = (double)c[k] - (double)t[k];
            acc += r * r;
        }
    }
    part[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) part[threadIdx.x] += part[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) atomicAdd(loss, part[0]);
}

__global__ __launch_bounds__(256) void l2_value(const float *__restrict__ cube, const float *__restrict__ target,
                                                size_t n, double *__restrict__ loss) {
    l2_sum(cube, target, n, loss);
}

hipError_t launch_l2_value(const float *cube, const float *target, size_t n, double *loss, hipStream_t st) {
    hipLaunchKernelGGL(zero_double, dim3(1), dim3(1), 0, st, loss);
    // the blocks' additions to one address queue up (about 10 ns each): a block
    // for every 24 elements a lane, at most 1024.  256^2 x 48 (us): 2048 blocks
    // 29, 1024 18, 512 14.5, 256 17; 512^2 x 64: 46, 41, 54, 93.
    const int blocks = (int)std::min<size_t>((n + 255) / 256, std::clamp<size_t>(n / (256 * 24), 256, 1024));
    hipLaunchKernelGGL(l2_value, dim3(blocks), dim3(256), 0, st, cube, target, n, loss);
    return hipGetLastError();
}

__global__ void zero_doubles(double *p, int n) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0.0;
}

// blockIdx.y = request of the batch; each request's elements grid-strided
// over blockIdx.x, block partial sums added with FP64 atomics
__global__ __launch_bounds__(256) void l2_batch(const ServeDesc *__restrict__ descs) {
    const ServeDesc &D = descs[blockIdx.y];
    if (!D.target) return;
    l2_sum(D.cube, D.target, (size_t)D.nch * D.g.nx * D.g.ny, D.loss);
}

hipError_t launch_l2_batch(const ServeDesc *descs, int nreq, double *losses, size_t max_n, hipStream_t st) {
    hipLaunchKernelGGL(zero_doubles, dim3(1), dim3(256), 0, st, losses, nreq);
    // (64 blocks a request: 50 us a launch of 60 walkers' requests of 128^2 x 32
    // on average, 128 blocks 56, 256 blocks 79: their additions queue up)
    const int blocks = (int)std::min<size_t>((max_n + 255) / 256, 64);
    hipLaunchKernelGGL(l2_batch, dim3(blocks, nreq), dim3(256), 0, st, descs);
    return hipGetLastError();
}

hipError_t launch_l2_loss(const float *cube, const float *target, float *dl, size_t n, double *loss, hipStream_t st) {
    hipLaunchKernelGGL(zero_double, dim3(1), dim3(1), 0, st, loss);
    const int blocks = (int)std::min<size_t>((n + 255) / 256, 2048);
    hipLaunchKernelGGL(l2_loss, dim3(blocks), dim3(256), 0, st, cube, target, dl, n, loss);
    return hipGetLastError();
}

} // namespace rt
