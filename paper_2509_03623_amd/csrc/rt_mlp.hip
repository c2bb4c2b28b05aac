// rt_mlp.hip -- neural CO layer on the matrix cores.
//
// Network: 16 Fourier frequencies on the two normalised grid coordinates of a
// sample (64 features) -> 4 SiLU layers of width 128 -> 3 outputs.  Its points
// are the (pixel, sample) points of the render, index m = k * npix + pix; the
// forward evaluates those that the march reads, the backward those with a
// gradient.
//
// The BF16 path runs mlp_fwd_rr and mlp_bwd_rr; the FP32 path runs mlp_fwd_fr
// and mlp_bwd_fr, the same designs on v_mfma_f32_16x16x4_f32.
//
// mlp_fwd_rr (BF16): persistent workgroups holding all hidden weights in LDS;
//   each wave evaluates 64 points at a time with the transposed product
//   Z^T = W H^T, output neurons as MFMA rows and points as columns.  The
//   accumulator of a 16-neuron output tile leaves every lane with 4
//   consecutive neurons of one point; two such tiles are exactly the 8
//   operand values a lane supplies for one 32-deep K chunk of the next layer,
//   once that layer's input order is permuted to match (done when the
//   weights are prepared).  Activations therefore never leave registers; the
//   output layer is evaluated in FP32 on the VALU and reduced across the
//   four lane groups by shuffles.  A wave evaluates only the points where the
//   march reads the network, gathered 64 at a time in a queue of its own:
//   256^2 x 256 samples 3.20 -> 1.65 ms (less than half of the points; the rest
//   miss the grid or lie beyond its taper, in no pattern that would leave
//   whole waves of consecutive points out).
// mlp_bwd_rr (BF16): see its definition below.
// mlp_fwd_fr, mlp_bwd_fr (FP32): see "register-resident FP32" below.
#include <algorithm>
#include <cmath>

#include "rt_adjoint.h"
#include "rt_mlp.h"

namespace rt {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kW = 128;     // hidden width
constexpr int kF = 64;      // features
constexpr int kLayerIn[4] = {kF, kW, kW, kW};

__device__ __forceinline__ floatx4 mfma_bf16(bf16x8 a, bf16x8 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ floatx4 mfma_f32(float a, float b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Normalised grid coordinates of point m (same positions as the march); true if
// the march reads the network there: on a ray that meets the grid, inside the
// edge taper.  Elsewhere the density is 0 whatever the network says.
__device__ __forceinline__ bool point_coords(const Geometry &g, const Shade &s, size_t m, float *rh, float *zh) {
    const int npix = g.nx * g.ny;
    const int k = (int)(m / npix);
    const int pix = (int)(m - (size_t)k * npix);
    const RaySetup r = ray_setup(g, pix % g.nx, pix / g.nx);
    const float t = ((float)k + 0.5f - 0.5f * (float)g.nsamp) * r.ds;
    const Locus L = locate(s, r.px, fmaf(t, r.wy, r.pmy), fmaf(t, r.wz, r.pmz));
    *rh = clampf(L.u, -1.0f, s.fnr) / (s.fnr - 1.0f);
    *zh = clampf(L.v, 0.0f, s.fnz) / (s.fnz - 1.0f);
    return r.live && L.taper > 0.0f;
}

// Entry of a queue of points to evaluate: the index and the coordinates.
struct PointEntry {
    uint32_t lo, hi;
    float rh, zh;
};
__device__ __forceinline__ PointEntry point_entry(size_t m, float rh, float zh) {
    return PointEntry{(uint32_t)m, (uint32_t)(m >> 32), rh, zh};
}
__device__ __forceinline__ size_t point_index(const PointEntry &e) { return (size_t)e.hi << 32 | e.lo; }

// Group of 64 consecutive points that taker w of n takes in round r: each round
// deals n groups, turned by 37 from the last, so that no taker keeps the same
// part of the image (the disk's middle or its empty corners).
__device__ __forceinline__ size_t dealt_group(size_t r, unsigned w, unsigned n) {
    return r * n + (w + (unsigned)(r % n) * 37u) % n;
}

// Phase f c reduced to (-2, 2) in float: the product is split exactly into
// hi + lo with an FMA (Ogita, Rump and Oishi's TwoProduct), hi loses its even
// integer part exactly (|hi| < 2^23), and lo is added back with one rounding,
// so the reduced phase is the exact one rounded once.
__device__ __forceinline__ float phase2(float f, float c) {
    const float hi = f * c;
    const float lo = fmaf(f, c, -hi);
    return (hi - 2.0f * floorf(0.5f * hi)) + lo;
}

// ---------------------------------------------------------------- register-resident BF16 forward
// Rows in LDS are padded by 32 bytes: a wave's 16-byte operand reads (16 rows,
// four 16-byte columns) then take 4.9 cycles (the same as 64 consecutive
// pieces); any other padding measured, 16 bytes among them, takes 8.4, none 16
// to 32.
constexpr int kRrRow0 = kF + 16;       // padded row of layer 0 (bf16 elements)
constexpr int kRrRow = kW + 16;        // padded row of layers 1..3
// 16-point column tiles per wave and lanes per workgroup (one workgroup per
// CU, the weights filling most of its LDS); 4 x 512 measured fastest of
// 2 x 1024, 2 x 768 and 4 x 512, and the same as 3 x 512 (which spills no
// registers where 4 x 512 spills 31: the spills cost nothing measurable)
constexpr int kRrTiles = 4;
constexpr int kRrThreads = 512;
constexpr size_t kRrWeightElems = (size_t)kW * kRrRow0 + 3 * (size_t)kW * kRrRow;
constexpr size_t kRrHead = kRrWeightElems * 2 + 4 * (4 * kW) + 4 * (3 * kW) + 16;
constexpr size_t kRrLds = kRrHead + sizeof(PointEntry) * 128 * (kRrThreads / 64);
static_assert(kRrHead % 16 == 0, "the queues are 16-byte aligned");

// input slot s of a 32-deep K chunk -> neuron of the previous layer: lane
// group g holds slots 8g..8g+7 = neurons 4g..4g+3 of the chunk's first
// 16-neuron output tile and 4g..4g+3 of its second
__host__ __device__ constexpr int rr_perm(int s) {
    return (s & ~31) + 16 * ((s & 7) >> 2) + 4 * ((s >> 3) & 3) + (s & 3);
}

// Layer 0 is scaled by log2(e) so that its pre-activation comes out as
// log2(e) z; layers 1..3 take log2(e) SiLU(z) as input and need no scale.
__global__ void mlp_prep_rr(const float *__restrict__ flat, MlpDev w) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    __bf16 *Wr = (__bf16 *)w.Wr;
    if (i < kW * kRrRow0) {
        const int o = i / kRrRow0, k = i - o * kRrRow0;
        Wr[i] = (__bf16)(k < kF ? kLog2E * flat[w.off[0] + o * kF + k] : 0.0f);
    }
    __bf16 *WrT = (__bf16 *)w.WrT;
    for (int l = 1; l < 4; ++l) {
        if (i < kW * kRrRow) {
            const int o = i / kRrRow, k = i - o * kRrRow;
            Wr[(size_t)kW * kRrRow0 + (size_t)(l - 1) * kW * kRrRow + i] =
                (__bf16)(k < kW ? flat[w.off[l] + o * kW + rr_perm(k)] : 0.0f);
            // transposed: row = input neuron o, column = output slot k
            WrT[(size_t)(l - 1) * kW * kRrRow + i] = (__bf16)(k < kW ? flat[w.off[l] + rr_perm(k) * kW + o] : 0.0f);
        }
    }
}

// One hidden layer of the register-resident forward for the NP column tiles
// of a wave: z' = W h' + b' (the weights and biases carry the log2(e) scale
// of the prepared layout, so z' = log2(e) z), h' = z' sigma(z) -- i.e.
// log2(e) SiLU(z), the scale being absorbed by the next layer's prepared
// weights.  The accumulators start from the biases.  The last layer feeds
// the FP32 output layer instead of the next operands.
template <int NP>
__device__ __forceinline__ void rr_layer(const bf16x8 (&hin)[4][NP], bf16x8 (&hout)[4][NP], float (&o)[3][NP],
                                         const __bf16 *sW, const float *sB, const float *sW5, int l, int lg, int lc,
                                         bool last) {
    const int nk = l == 0 ? kF / 32 : kW / 32;
    const int row = l == 0 ? kRrRow0 : kRrRow;
    const __bf16 *Wl = sW + (l == 0 ? 0 : (size_t)kW * kRrRow0 + (size_t)(l - 1) * kW * kRrRow);
    const float *bl = sB + l * kW;
#pragma unroll
    for (int cp = 0; cp < 4; ++cp) {           // output tiles 2cp, 2cp+1
        floatx4 acc[2][NP];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const floatx4 b4 = *(const floatx4 *)(bl + 32 * cp + 16 * h + 4 * lg);
#pragma unroll
            for (int tp = 0; tp < NP; ++tp) acc[h][tp] = b4;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (c >= nk) break;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const bf16x8 a = *(const bf16x8 *)(Wl + (size_t)(32 * cp + 16 * h + lc) * row + 32 * c + 8 * lg);
#pragma unroll
                for (int tp = 0; tp < NP; ++tp) acc[h][tp] = mfma_bf16(a, hin[c][tp], acc[h][tp]);
            }
        }
        if (!last) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int tp = 0; tp < NP; ++tp)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float z = acc[h][tp][i];
                        hout[cp][tp][4 * h + i] = (__bf16)(z * frcp(1.0f + fexp2(-z)));
                    }
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int n = 32 * cp + 16 * h + 4 * lg;
                const floatx4 w0 = *(const floatx4 *)(sW5 + n), w1 = *(const floatx4 *)(sW5 + kW + n),
                              w2 = *(const floatx4 *)(sW5 + 2 * kW + n);
#pragma unroll
                for (int tp = 0; tp < NP; ++tp)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float z = acc[h][tp][i];
                        const float hv = z * frcp(1.0f + fexp2(-z));
                        o[0][tp] = fmaf(hv, w0[i], o[0][tp]);
                        o[1][tp] = fmaf(hv, w1[i], o[1][tp]);
                        o[2][tp] = fmaf(hv, w2[i], o[2][tp]);
                    }
            }
        }
    }
}

template <int NP, int NT>
__global__ __launch_bounds__(NT) void mlp_fwd_rr(Geometry g, Shade s, MlpDev w, size_t M, float4 *__restrict__ out) {
    extern __shared__ __attribute__((aligned(16))) unsigned char rr_lds[];
    __bf16 *sW = (__bf16 *)rr_lds;                                  // layer 0, then layers 1..3
    float *sB = (float *)(rr_lds + kRrWeightElems * 2);             // [4][128]
    float *sW5 = sB + 4 * kW;                                       // [3][128]
    float *sB5 = sW5 + 3 * kW;                                      // [3]
    static_assert(NP == 4, "64 points a wave");
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int lg = lane >> 4, lc = lane & 15;
    {
        const uint4 *src = (const uint4 *)w.Wr;
        uint4 *dst = (uint4 *)sW;
        for (size_t i = tid; i < kRrWeightElems / 8; i += NT) dst[i] = src[i];
        for (int i = tid; i < 4 * kW; i += NT) sB[i] = kLog2E * w.b[i / kW][i % kW];
        for (int i = tid; i < 3 * kW; i += NT) sW5[i] = kLn2 * w.W5[i];
        if (tid < 3) sB5[tid] = w.b5[tid];
    }
    __syncthreads();
    // The wave's queue: it takes groups of 64 points, keeps those where the
    // network is read (less than half of them: the rest miss the grid or lie
    // beyond its taper), and evaluates 64 as soon as it has them.
    PointEntry *queue = (PointEntry *)(rr_lds + kRrHead) + 128 * wv;
    const unsigned takers = gridDim.x * (NT / 64), taker = blockIdx.x * (NT / 64) + wv;
    const size_t rounds = ((M + 63) / 64 + takers - 1) / takers;
    size_t round = 0;
    int fill = 0;
    for (;;) {
        while (fill < 64 && round < rounds) {
            const size_t m = dealt_group(round++, taker, takers) * 64 + lane;
            float rh = 0.0f, zh = 0.0f;
            const bool read = m < M && point_coords(g, s, m, &rh, &zh);
            const unsigned long long mk = __ballot(read);
            if (read) queue[fill + __popcll(mk & ((1ull << lane) - 1ull))] = point_entry(m, rh, zh);
            fill += __popcll(mk);
        }
        if (fill == 0) break;
        const int n = min(fill, 64);
        float rh = 0.0f, zh = 0.0f;
        if (lane < n) {
            rh = queue[lane].rh;
            zh = queue[lane].zh;
        }
        // layer-0 operands: features of chunk c (0: r, 1: z); lane group g
        // supplies slots 8g..8g+7 = sin (g < 2) or cos (g >= 2) of
        // frequencies 8 (g & 1) .. 8 (g & 1) + 7.  Lanes g and g ^ 2 share
        // the work: each evaluates four frequencies (hardware sine and cosine
        // of the phase reduced to one period) and passes the partner the half
        // it needs.
        bf16x8 hin[4][NP];
        const int fb = 8 * (lg & 1) + (lg < 2 ? 0 : 4);
#pragma unroll
        for (int tp = 0; tp < NP; ++tp) {
            const float cr = __shfl(rh, tp * 16 + lc), cz = __shfl(zh, tp * 16 + lc);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                float own[4], sent[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    // sin(pi f x) = sin(2 pi t) with t = (f x mod 2) / 2 in [0, 1)
                    const float x = w.freq[fb + q] * (c == 0 ? cr : cz);
                    const float t = 0.5f * (x - 2.0f * floorf(0.5f * x));
                    const float sv = __builtin_amdgcn_sinf(t), cv = __builtin_amdgcn_cosf(t);
                    own[q] = lg < 2 ? sv : cv;
                    sent[q] = lg < 2 ? cv : sv;
                }
                bf16x8 f;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float r = __shfl_xor(sent[q], 32);
                    f[q] = (__bf16)(lg < 2 ? own[q] : r);
                    f[4 + q] = (__bf16)(lg < 2 ? r : own[q]);
                }
                hin[c][tp] = f;
            }
        }
        float o[3][NP];
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int tp = 0; tp < NP; ++tp) o[j][tp] = 0.0f;
        bf16x8 hb[4][NP];
        // layers in pairs, activations ping-ponging between hin and hb
#pragma unroll 1
        for (int lp = 0; lp < 2; ++lp) {
            rr_layer<NP>(hin, hb, o, sW, sB, sW5, 2 * lp, lg, lc, false);
            rr_layer<NP>(hb, hin, o, sW, sB, sW5, 2 * lp + 1, lg, lc, lp == 1);
        }
        // sum the four lane groups' partial outputs; group 0 writes
#pragma unroll
        for (int tp = 0; tp < NP; ++tp) {
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                o[j][tp] += __shfl_xor(o[j][tp], 16);
                o[j][tp] += __shfl_xor(o[j][tp], 32);
            }
            if (lg == 0 && tp * 16 + lc < n)
                out[point_index(queue[tp * 16 + lc])] =
                    make_float4(o[0][tp] + sB5[0], o[1][tp] + sB5[1], o[2][tp] + sB5[2], 0.0f);
        }
        // what is left moves to the front
        fill -= n;
        if (lane < fill) {
            const PointEntry e = queue[64 + lane];
            queue[lane] = e;
        }
    }
}

// ---------------------------------------------------------------- register-resident BF16 backward
// mlp_bwd_rr: one workgroup of eight waves per CU, 64 points a pass.  Two waves
// share 16 points, each with half of every layer's neurons: they recompute the
// forward with the transposed product (weights read as A operands from LDS,
// where the workgroup stages each layer's weights from L2: one copy per pass
// for all waves, written by loads that go to LDS directly and are issued one
// stage ahead into a free buffer -- the forward's layers alternate between the
// weight buffer and the point-major rows, which the forward does not use; the
// backward's transposed weights are issued before the weight-gradient products
// that precede them -- so their latency overlaps the matrix work), pass each
// other their halves of h' through LDS, and keep z' of every layer as BF16;
// walk back through the layers (dL/dh' of the layer below by the product with
// the transposed weights, the SiLU derivative recomputed from z'); and for the
// weight gradient, which sums over points, write dL/dz' and h' of the pass
// into LDS as point-major rows, so that after a barrier each wave accumulates
// its own block of every layer's gradient (32 output rows by half the input
// columns of the hidden layers, a 16-column tile of the output layer) in MFMA
// accumulators over all 64 points.  Bias gradients are row sums of the same
// LDS rows.  Everything is flushed with atomics once, at the end.
//
// Bound: issue of the vector instructions beside the matrix ones (SiLU and its
// derivative, conversions, the row writes) and the staging of the weights (240
// KB a pass; without it 3.5 ms where it takes 4.4).  A single wave issues no
// more than one vector instruction in 5 cycles, two of them twice that.  256^2
// x 256 samples (over two thirds of its points): four waves with all neurons of
// 16 points each 6.0 ms, eight waves 5.1, rows written two points at once 4.85,
// LDS rows without conflicts 4.7, weights fetched from scalar addresses 4.4; over
// all points 6.4, with 44 % of the vector units' cycles and 16 % of the matrix
// units' taken.
constexpr int kBrPts = 64;                 // points per workgroup pass
constexpr int kBrThreads = 512;
// global-memory views (the pass loop launders the weight pointers, which
// would otherwise turn their loads into flat loads)
typedef const __attribute__((address_space(1))) __bf16 gbf16;
typedef const __attribute__((address_space(1))) bf16x8 gbf16x8;
constexpr int kBrStride = kBrPts + 16;     // LDS row of the point-major buffers (bf16)

// features of one coordinate
__device__ __forceinline__ bf16x8 br_features(const MlpDev &w, float x0, int lg) {
    const int fb = 8 * (lg & 1) + (lg < 2 ? 0 : 4);
    float own[4], sent[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float x = w.freq[fb + q] * x0;
        const float t = 0.5f * (x - 2.0f * floorf(0.5f * x));
        const float sv = __builtin_amdgcn_sinf(t), cv = __builtin_amdgcn_cosf(t);
        own[q] = lg < 2 ? sv : cv;
        sent[q] = lg < 2 ? cv : sv;
    }
    bf16x8 f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float r = __shfl_xor(sent[q], 32);
        f[q] = (__bf16)(lg < 2 ? own[q] : r);
        f[4 + q] = (__bf16)(lg < 2 ? r : own[q]);
    }
    return f;
}

// h' = z' sigma(z) and dL/dz' = dL/dh' SiLU'(z) of one neuron, z = ln2 z'
__device__ __forceinline__ void br_act_grad(__bf16 zq16, float dh, bf16x8 &hp, bf16x8 &dz, int e) {
    const float zq = (float)zq16;
    const float sg = frcp(1.0f + fexp2(-zq));
    const float z = kLn2 * zq;
    hp[e] = (__bf16)(zq * sg);
    dz[e] = (__bf16)(dh * (sg * (1.0f + z * (1.0f - sg))));
}

// (a, b) of this lane's point and its neighbour's -> this lane's neuron of the
// pair at both points: a of (even, odd lane) in even lanes, b in odd ones
__device__ __forceinline__ uint32_t br_swap(uint32_t ab, uint32_t sel) {
    const uint32_t other = (uint32_t)__builtin_amdgcn_mov_dpp((int)ab, 0xB1, 0xF, 0xF, false);
    return __builtin_amdgcn_perm(other, ab, sel);
}
// v_perm_b32 selector of br_swap: even lanes (own low, other low), odd ones (other high, own high)
__device__ __forceinline__ uint32_t br_swap_sel(int lane) { return lane & 1 ? 0x03020706u : 0x05040100u; }

// point-major write of 8 consecutive-pair values of the lane's point, value j
// in row row0(j), j even, and the next row: neighbouring lanes swap values so
// that each writes two points of one row at once.  (One 2-byte write a value
// took the LDS twice the instructions and 4 cycles of conflicts each.)
template <class Row>
__device__ __forceinline__ void br_write8(__bf16 *X, bf16x8 v, int lane, int col, Row row0) {
    const uint32_t sel = br_swap_sel(lane);
    union { bf16x8 h; uint32_t u[4]; } p;
    p.h = v;
    __bf16 *o = X + (lane & 1) * kBrStride + (col & ~1);
#pragma unroll
    for (int q = 0; q < 4; ++q) *(uint32_t *)(o + row0(2 * q) * kBrStride) = br_swap(p.u[q], sel);
}

// 16 accumulator-layout values (neurons 16t + 4lg + i, t = 2cp + h, element
// 4h + i of pair cp = cp0, cp0 + 1) of the lane's point
__device__ __forceinline__ void br_write_rows(__bf16 *X, const bf16x8 (&v)[2], int cp0, int lane, int col) {
    __bf16 *o = X + (32 * cp0 + 4 * (lane >> 4)) * kBrStride;
#pragma unroll
    for (int cq = 0; cq < 2; ++cq)
        br_write8(o, v[cq], lane, col, [=](int j) { return 32 * cq + 16 * (j >> 2) + (j & 3); });
}

// dW block of one hidden layer: rows [32 rq, 32 rq + 32) of XD against the NI
// 16-row tiles of XH from tile it0, over the 64 points
template <int NI>
__device__ __forceinline__ void br_dw(floatx4 (&acc)[2][NI], const __bf16 *XD, const __bf16 *XH, int rq, int it0,
                                      int lg, int lc) {
#pragma unroll
    for (int kc = 0; kc < kBrPts / 32; ++kc) {
        const bf16x8 a0 = *(const bf16x8 *)(XD + (32 * rq + lc) * kBrStride + 32 * kc + 8 * lg);
        const bf16x8 a1 = *(const bf16x8 *)(XD + (32 * rq + 16 + lc) * kBrStride + 32 * kc + 8 * lg);
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            const bf16x8 b = *(const bf16x8 *)(XH + (16 * (it0 + it) + lc) * kBrStride + 32 * kc + 8 * lg);
            acc[0][it] = mfma_bf16(a0, b, acc[0][it]);
            acc[1][it] = mfma_bf16(a1, b, acc[1][it]);
        }
    }
}

// sum over the 64 points of LDS row r (four lanes per row, 16 points each);
// two values per instruction, as a dot product with (1, 1)
__device__ __forceinline__ float br_rowsum(const __bf16 *X, int r, int part) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 one = {(__bf16)1.0f, (__bf16)1.0f};
    float sum = 0.0f;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const bf16x8 v = *(const bf16x8 *)(X + r * kBrStride + 16 * part + 8 * q);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bf16x2 p = {v[2 * j], v[2 * j + 1]};
            sum = __builtin_amdgcn_fdot2_f32_bf16(p, one, sum, false);
        }
    }
    sum += __shfl_xor(sum, 1);
    return sum + __shfl_xor(sum, 2);
}

// copy n bf16 elements (a multiple of 8) of one layer's prepared weights
// from global memory into the workgroup's staging buffer (512 lanes): global
// loads that write LDS directly (16 B per lane, lane i of a wave to the
// wave's base + 16 i), so the copy holds no registers; every load is waited
// for (br_wait) before the barrier that precedes the first read
// (scalar base and 32-bit lane offset: per-lane 64-bit addresses of every
// stage would be kept, and spilled, across the pass)
template <int N>
__device__ __forceinline__ void br_issue(__bf16 *dst, const gbf16 *src, int wv, int lane) {
    typedef __attribute__((address_space(3))) void lds_void;
    typedef const __attribute__((address_space(1))) void g_void;
    typedef const __attribute__((address_space(1))) char g_char;
    constexpr int kChunks = N / 8;
    static_assert(N % 8 == 0 && kChunks % 64 == 0, "whole waves of 16 bytes a lane");
    // (kept apart from the surrounding matrix code: interleaved with it, the
    // address arithmetic lengthens live ranges into spills)
    __builtin_amdgcn_sched_barrier(0);
    const uint32_t off = 16u * (uint32_t)lane;
#pragma unroll
    for (int i = 0; i < (kChunks + kBrThreads - 1) / kBrThreads; ++i) {
        const int c0 = 64 * wv + i * kBrThreads;
        if ((i + 1) * kBrThreads <= kChunks || c0 < kChunks)
            __builtin_amdgcn_global_load_lds((g_void *)((g_char *)(src + 8 * c0) + off), (lds_void *)(dst + 8 * c0), 16,
                                             0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ void br_wait() { __builtin_amdgcn_s_waitcnt(0); }

// The points with any dL/do != 0, in order, for the backward kernels.  dL/do = 0
// at a point (no opacity there) makes every layer's dL/dz zero: the point adds
// nothing to any gradient, so the backward takes the others only, packed 64 to
// a pass.  A point with however small a dL/do stays: it may be all that some
// weight's gradient has (a neuron that is silent wherever dL/do is large).
// Three launches over kLiveChunks chunks of the points: the
// count of each chunk, a scan of the counts, then each
// chunk writing its points' indices (1024 consecutive points at a time, each
// lane's place from a ballot within its wave and the waves' counts in LDS).
// list: [0] the number of points, [1 ...] their indices; then the chunks'
// counts and offsets.
constexpr int kLiveChunks = 4096;

__device__ __forceinline__ bool live_point(const float4 *dO, size_t m) {
    const float4 d = dO[m];
    return d.x != 0.0f || d.y != 0.0f || d.z != 0.0f;
}

__global__ __launch_bounds__(1024) void mlp_live_count(const float4 *__restrict__ dO, size_t M, size_t chunk,
                                                       uint32_t *__restrict__ counts) {
    __shared__ uint32_t tot;
    if (threadIdx.x == 0) tot = 0u;
    __syncthreads();
    const size_t b0 = (size_t)blockIdx.x * chunk, b1 = min(M, b0 + chunk);
    uint32_t n = 0;
    for (size_t i = b0 + threadIdx.x; i < b1; i += 1024) n += live_point(dO, i) ? 1u : 0u;
    if (n) atomicAdd(&tot, n);
    __syncthreads();
    if (threadIdx.x == 0) counts[blockIdx.x] = tot;
}

// exclusive offsets of nb <= 4 * 1024 counts (one workgroup) and their total into list[0]
__global__ __launch_bounds__(1024) void mlp_live_scan(const uint32_t *__restrict__ counts, int nb,
                                                      uint32_t *__restrict__ offsets, uint32_t *__restrict__ list) {
    __shared__ uint32_t part[1024];
    const int t = threadIdx.x;
    uint32_t c[4], n = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        c[j] = 4 * t + j < nb ? counts[4 * t + j] : 0u;
        n += c[j];
    }
    part[t] = n;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const uint32_t v = t >= off ? part[t - off] : 0u;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    uint32_t o = part[t] - n;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (4 * t + j < nb) offsets[4 * t + j] = o;
        o += c[j];
    }
    if (t == 1023) list[0] = part[1023];
}

__global__ __launch_bounds__(1024) void mlp_live_write(const float4 *__restrict__ dO, size_t M, size_t chunk,
                                                       const uint32_t *__restrict__ offsets,
                                                       uint32_t *__restrict__ list) {
    __shared__ uint32_t wsum[16];
    const uint32_t t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const size_t b0 = (size_t)blockIdx.x * chunk, b1 = min(M, b0 + chunk);
    uint32_t done = offsets[blockIdx.x];   // the same in every lane
    for (size_t c0 = b0; c0 < b1; c0 += 1024) {
        const size_t i = c0 + t;
        const bool f = i < b1 && live_point(dO, i);
        const uint64_t mk = __ballot(f);
        if (lane == 0) wsum[wv] = (uint32_t)__popcll(mk);
        __syncthreads();
        uint32_t off = done, tot = 0;
        for (uint32_t j = 0; j < 16; ++j) {
            const uint32_t n = wsum[j];
            off += j < wv ? n : 0u;
            tot += n;
        }
        if (f) list[1 + off + (uint32_t)__popcll(mk & ((1ull << lane) - 1ull))] = (uint32_t)i;
        done += tot;
        __syncthreads();
    }
}

__global__ __launch_bounds__(kBrThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void mlp_bwd_rr(
    Geometry g, Shade s, MlpDev w, size_t M, const float4 *__restrict__ dO, const uint32_t *__restrict__ list,
    float *__restrict__ dW) {
    // point-major rows of the backward: dL/dz' (or dL/do) rows x points, then
    // h' (or features) rows x points; in the forward, layers 1 and 3's weights
    __shared__ __attribute__((aligned(16))) __bf16 XU[2 * kW * kBrStride];
    static_assert(2 * kW * kBrStride >= kW * kRrRow, "a hidden layer's weights fit the row buffers");
    __bf16 *const XD = XU;
    __bf16 *const XH = XU + kW * kBrStride;
    __shared__ __attribute__((aligned(16))) float sB[4 * kW];
    __shared__ __attribute__((aligned(16))) float sW5[3 * kW];
    // parking of z' (layers 0 to 2, packs 4 l + cp) and the two feature packs
    // (16, 17) between the forward and the backward of a pass, and where the
    // two waves of a point pass packs to each other: h' of layers 0 and 2 in
    // packs 12.., of layer 1 in 8.. (z' of layer 2 is parked there a barrier
    // later), dL/dz' of layer l in 4 l.. once its z' is read
    __shared__ bf16x8 ZP[18][256];
    // one layer's weights (forward) or transposed weights (backward)
    __shared__ __attribute__((aligned(16))) __bf16 SW[kW * kRrRow];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lg = lane >> 4, lc = lane & 15;
    const int pt = wv >> 1, hf = wv & 1;       // 16-point tile, half of the neurons
    const int cp0 = 2 * hf, pl = 64 * pt + lane;
    for (int i = tid; i < 4 * kW; i += kBrThreads) sB[i] = kLog2E * w.b[i / kW][i % kW];
    for (int i = tid; i < 3 * kW; i += kBrThreads) sW5[i] = kLn2 * w.W5[i];
    // this wave's blocks of the weight gradients: rows from 32 pt, half hf of
    // the columns; columns from 16 wv of the output layer
    floatx4 g0[2][2], g1[2][4], g2[2][4], g3[2][4], g4 = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int a = 0; a < 2; ++a) {
#pragma unroll
        for (int b = 0; b < 2; ++b) g0[a][b] = g4;
#pragma unroll
        for (int b = 0; b < 4; ++b) g1[a][b] = g2[a][b] = g3[a][b] = g4;
    }
    float db0 = 0.0f, db1 = 0.0f, db2 = 0.0f, db3 = 0.0f, db5 = 0.0f;
    const int brow = 16 * wv + (lane >> 2), bpart = lane & 3;     // bias row of this lane
    const int col = 16 * pt + lc;                                 // this lane's point within the pass
    // layer 0's weights for the first pass (each pass stages the next's)
    br_issue<kW * kRrRow0>(SW, (const gbf16 *)(uint64_t)w.Wr, wv, lane);
    // the points with any dL/do != 0, listed in order (list[0] of them), 64 to
    // a pass
    const uint32_t npts = list[0];
    const uint32_t npass = (npts + kBrPts - 1) / kBrPts;
    for (uint32_t ip = blockIdx.x; ip < npass; ip += gridDim.x) {
        const uint32_t base = ip * kBrPts;
        // the weight operands are the same every pass: hide that from the
        // compiler, or it keeps all their fragments in registers across passes
        uint64_t wr_u = (uint64_t)w.Wr, wrt_u = (uint64_t)w.WrT;
        asm volatile("" : "+s"(wr_u), "+s"(wrt_u));
        const gbf16 *Wr = (const gbf16 *)wr_u;
        const gbf16 *WrT = (const gbf16 *)wrt_u;
        const size_t m = base + col < npts ? (size_t)list[1 + base + col] : M;   // M: no point
        float rh = 0.0f, zh = 0.0f;
        if (lane < 16 && m < M) point_coords(g, s, m, &rh, &zh);
        // each wave the features of one coordinate
        ZP[16 + hf][pl] = br_features(w, __shfl(hf ? zh : rh, lc), lg);
        br_wait();
        __syncthreads();
        // ---- forward, parking z' of every layer
        bf16x8 z2[2], z3[2];
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            const int nk = l == 0 ? kF / 32 : kW / 32;
            const int row = l == 0 ? kRrRow0 : kRrRow;
            // layer l's weights are in place; the next stage goes into the
            // other buffer, free since the barrier that ended layer l - 1:
            // layer l + 1's weights, or after layer 3 the transposed weights
            // of the backward's first product
            if (l < 3) br_issue<kW * kRrRow>(l & 1 ? SW : XU, Wr + (size_t)kW * kRrRow0 + (size_t)l * kW * kRrRow, wv, lane);
            else br_issue<kW * kRrRow>(SW, WrT + (size_t)2 * kW * kRrRow, wv, lane);
            const __bf16 *Wl = l & 1 ? XU : SW;
            const int in = l == 0 ? 16 : l == 2 ? 8 : 12;      // the packs of this layer's input
            bf16x8 hin[4];
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (c < nk) hin[c] = ZP[in + c][pl];
            if (l == 3) {
                ZP[8 + cp0][pl] = z2[0];
                ZP[9 + cp0][pl] = z2[1];
            }
#pragma unroll
            for (int cq = 0; cq < 2; ++cq) {
                const int cp = cp0 + cq;
                floatx4 acc[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) acc[h] = *(const floatx4 *)(sB + l * kW + 32 * cp + 16 * h + 4 * lg);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (c >= nk) break;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const bf16x8 a = *(const bf16x8 *)(Wl + (32 * cp + 16 * h + lc) * row + 32 * c + 8 * lg);
                        acc[h] = mfma_bf16(a, hin[c], acc[h]);
                    }
                }
                bf16x8 zq, hout;
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float z = acc[h][i];
                        zq[4 * h + i] = (__bf16)z;
                        if (l < 3) hout[4 * h + i] = (__bf16)(z * frcp(1.0f + fexp2(-z)));
                    }
                if (l == 2) z2[cq] = zq;
                else if (l == 3) z3[cq] = zq;
                else ZP[4 * l + cp][pl] = zq;
                if (l < 3) ZP[(l == 1 ? 8 : 12) + cp][pl] = hout;
            }
            br_wait();
            __syncthreads();
        }
        // ---- output layer: dL/dh'_3 = W5'^T dL/do, then h'_3 and dL/dz'_3
        const float4 d = m < M ? dO[m] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        bf16x8 hp[2], dz[2], dzu[2];   // h' and dL/dz' of the current layer, dL/dz' of the layer above
#pragma unroll
        for (int cq = 0; cq < 2; ++cq)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int n = 32 * (cp0 + cq) + 16 * (e >> 2) + 4 * lg + (e & 3);
                const float dh = fmaf(sW5[n], d.x, fmaf(sW5[kW + n], d.y, sW5[2 * kW + n] * d.z));
                br_act_grad(z3[cq][e], dh, hp[cq], dz[cq], e);
            }
#pragma unroll
        for (int l = 3; l >= 0; --l) {
            // gradient of the layer above (the output layer when l == 3):
            // its dL/dz' and this layer's h', point-major, into LDS
            br_write_rows(XH, hp, cp0, lane, col);
            if (l == 3) {
                if (hf == 0) {
                    if (lg == 0) {
                        XD[0 * kBrStride + col] = (__bf16)d.x;
                        XD[1 * kBrStride + col] = (__bf16)d.y;
                        XD[2 * kBrStride + col] = (__bf16)d.z;
                    } else {
                        // rows 3..15 are zero padding of the 16-row tile
#pragma unroll
                        for (int r = 0; r < 5; ++r) {
                            const int rr = 3 + 5 * (lg - 1) + r;
                            if (rr < 16) XD[rr * kBrStride + col] = (__bf16)0.0f;
                        }
                    }
                }
            } else {
                br_write_rows(XD, dzu, cp0, lane, col);
            }
            if (l >= 1) {
                ZP[4 * l + cp0][pl] = dz[0];
                ZP[4 * l + cp0 + 1][pl] = dz[1];
            }
            __syncthreads();
            // SW is free (every wave's product with it came before its rows):
            // issue the transposed weights of the next product down, or after
            // the last one the next pass's layer-0 weights
            if (l == 2 || l == 1) br_issue<kW * kRrRow>(SW, WrT + (size_t)(l - 1) * kW * kRrRow, wv, lane);
            else if (l == 0) br_issue<kW * kRrRow0>(SW, Wr, wv, lane);
            if (l == 3) {
#pragma unroll
                for (int kc = 0; kc < kBrPts / 32; ++kc) {
                    const bf16x8 a = *(const bf16x8 *)(XD + lc * kBrStride + 32 * kc + 8 * lg);
                    const bf16x8 b = *(const bf16x8 *)(XH + (16 * wv + lc) * kBrStride + 32 * kc + 8 * lg);
                    g4 = mfma_bf16(a, b, g4);
                }
                if (wv == 0) db5 += br_rowsum(XD, lane >> 2, bpart);   // rows 0..2 are dL/do
            } else if (l == 2) {
                br_dw<4>(g3, XD, XH, pt, 4 * hf, lg, lc);
                db3 += br_rowsum(XD, brow, bpart);
            } else if (l == 1) {
                br_dw<4>(g2, XD, XH, pt, 4 * hf, lg, lc);
                db2 += br_rowsum(XD, brow, bpart);
            } else {
                br_dw<4>(g1, XD, XH, pt, 4 * hf, lg, lc);
                db1 += br_rowsum(XD, brow, bpart);
            }
            if (l != 0) br_wait();
            __syncthreads();
            // dL/dh' of the layer below through the transposed weights, and
            // at once its h' and dL/dz'
            dzu[0] = dz[0];
            dzu[1] = dz[1];
            if (l >= 1) {
                // (the transposed weights are in SW, waited for before the
                // barrier above)
                const __bf16 *WT = SW;
                bf16x8 up[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) up[c] = ZP[4 * l + c][pl];
#pragma unroll
                for (int cq = 0; cq < 2; ++cq) {
                    const int cp = cp0 + cq;
                    floatx4 acc[2] = {floatx4{0.0f, 0.0f, 0.0f, 0.0f}, floatx4{0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
                    for (int c = 0; c < 4; ++c)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const bf16x8 a = *(const bf16x8 *)(WT + (32 * cp + 16 * h + lc) * kRrRow + 32 * c + 8 * lg);
                            acc[h] = mfma_bf16(a, up[c], acc[h]);
                        }
                    const bf16x8 zq = ZP[4 * (l - 1) + cp][pl];
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int i = 0; i < 4; ++i) br_act_grad(zq[4 * h + i], acc[h][i], hp[cq], dz[cq], 4 * h + i);
                }
            }
        }
        // ---- layer 0: features and dz'_0
        const bf16x8 f = ZP[16 + hf][pl];
        br_write8(XH + (32 * hf + 8 * lg) * kBrStride, f, lane, col, [](int j) { return j; });
        br_write_rows(XD, dz, cp0, lane, col);
        __syncthreads();
        br_dw<2>(g0, XD, XH, pt, 2 * hf, lg, lc);
        db0 += br_rowsum(XD, brow, bpart);
        // (the barrier after the next pass's features comes before anything
        // writes the rows again)
    }
    br_wait();   // layer 0's weights for a pass that does not come
    // ---- flush: flat layout per layer W [out][in] then b [out]
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int o = 32 * pt + 16 * a + 4 * lg + i;
#pragma unroll
            for (int it = 0; it < 2; ++it)
                atomicAdd(dW + w.off[0] + o * kF + 16 * (2 * hf + it) + lc, kLog2E * g0[a][it][i]);
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int j = 16 * (4 * hf + it) + lc;
                atomicAdd(dW + w.off[1] + o * kW + j, g1[a][it][i]);
                atomicAdd(dW + w.off[2] + o * kW + j, g2[a][it][i]);
                atomicAdd(dW + w.off[3] + o * kW + j, g3[a][it][i]);
            }
        }
    if (bpart == 0) {
        atomicAdd(dW + w.off[0] + kW * kF + brow, kLog2E * db0);
        atomicAdd(dW + w.off[1] + kW * kW + brow, kLog2E * db1);
        atomicAdd(dW + w.off[2] + kW * kW + brow, kLog2E * db2);
        atomicAdd(dW + w.off[3] + kW * kW + brow, kLog2E * db3);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int j = 4 * lg + i;
        if (j < 3) atomicAdd(dW + w.off[4] + j * kW + 16 * wv + lc, kLn2 * g4[i]);
    }
    if (wv == 0 && lane < 12 && bpart == 0) atomicAdd(dW + w.off[4] + 3 * kW + (lane >> 2), db5);
}

// ---------------------------------------------------------------- register-resident FP32
// mlp_fwd_fr, mlp_bwd_fr: the transposed product Z^T = W H^T on
// v_mfma_f32_16x16x4_f32.  The accumulator of output tile t leaves lane group
// lg (16 lanes) with neurons 16 t + 4 lg + i, i < 4, of its lane's point, and a
// 4-deep step of the next product takes one value per lane group: step (t, i)
// takes neurons 16 t + 4 lg + i, which is the accumulator register itself.  The
// weights of four steps are then four consecutive values of a row, one 16-byte
// read; rows are padded by 32 bytes as kRrRow is.  A layer's weights
// (66 KB) go from L2 to LDS once per pass for all waves of a workgroup, issued
// one stage ahead with loads that write LDS directly.
//
// Bound: the FP32 matrix rate (157 TFLOP/s; 32 cycles an instruction).  The
// tiled kernels before these read every operand from LDS or L2 at its use, one
// tile after another through LDS, over every point: 90 x 83 px x 128 samples
// 5.76 -> 0.82 ms forward (the matrix units busy 68 % of the time), 12.8 ->
// 2.38 ms backward (43 %) (one wave per SIMD: its activations, LDS rows and barriers
// run beside nothing).
constexpr int kFrRow0 = kF + 8, kFrRow = kW + 8;      // padded rows (floats)
constexpr size_t kFrWeightElems = (size_t)kW * kFrRow0 + 3 * (size_t)kW * kFrRow;
constexpr int kFrTiles = 2;                           // 16-point column tiles per wave
constexpr int kFrThreads = 512;
constexpr int kFrQueue = 16 * kFrTiles + 64;          // points a wave holds at most
constexpr int kFrStride = kBrPts + 8;                 // LDS row of the point-major buffers
constexpr int kFrSlab = 36 * 256;                     // floatx4 a workgroup parks: z of 4 layers, features

__global__ void mlp_prep_fr(const float *__restrict__ flat, MlpDev w) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    float *Wr = (float *)w.Wr, *WrT = (float *)w.WrT;
    if (i < kW * kFrRow0) {
        const int o = i / kFrRow0, k = i - o * kFrRow0;
        Wr[i] = k < kF ? flat[w.off[0] + o * kF + k] : 0.0f;
    }
    if (i < kW * kFrRow) {
        const int o = i / kFrRow, k = i - o * kFrRow;
        for (int l = 1; l < 4; ++l) {
            Wr[(size_t)kW * kFrRow0 + (size_t)(l - 1) * kW * kFrRow + i] = k < kW ? flat[w.off[l] + o * kW + k] : 0.0f;
            WrT[(size_t)(l - 1) * kW * kFrRow + i] = k < kW ? flat[w.off[l] + k * kW + o] : 0.0f;
        }
    }
}

// copy n floats (a multiple of 256) to LDS, 16 B per lane and load
typedef const __attribute__((address_space(1))) float gfloat;
template <int NT>
__device__ __forceinline__ void fr_issue(float *dst, const gfloat *src, int n, int tid) {
    typedef __attribute__((address_space(3))) void lds_void;
    typedef const __attribute__((address_space(1))) void g_void;
    const int wv = tid >> 6, lane = tid & 63;
    __builtin_amdgcn_sched_barrier(0);
    for (int c0 = 64 * wv; c0 < n / 4; c0 += NT)
        __builtin_amdgcn_global_load_lds((g_void *)(src + 4 * (c0 + lane)), (lds_void *)(dst + 4 * c0), 16, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
}
static_assert(kW * kFrRow0 % 256 == 0 && kW * kFrRow % 256 == 0, "whole waves of 16-byte lanes");

// features 16 t + 4 lg + i of the lane's point: sin r, cos r, sin z, cos z of
// frequencies 4 lg + i
__device__ __forceinline__ void fr_features(floatx4 (&f)[4], const MlpDev &w, float cr, float cz, int lg) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float s, c;
        sincospif(phase2(w.freq[4 * lg + i], cr), &s, &c);
        f[0][i] = s;
        f[1][i] = c;
        sincospif(phase2(w.freq[4 * lg + i], cz), &s, &c);
        f[2][i] = s;
        f[3][i] = c;
    }
}

// U output tiles from tile u0 on, over the 16 NK inputs: acc += W h
template <int NK, int U, int NP>
__device__ __forceinline__ void fr_product(floatx4 (&acc)[U][NP], const floatx4 (&h)[8][NP], const float *W, int row,
                                           int u0, int lg, int lc) {
#pragma unroll
    for (int t = 0; t < NK; ++t) {
        floatx4 a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = *(const floatx4 *)(W + (16 * (u0 + u) + lc) * row + 16 * t + 4 * lg);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int p = 0; p < NP; ++p) acc[u][p] = mfma_f32(a[u][i], h[t][p][i], acc[u][p]);
    }
}

template <int NK, bool LAST>
__device__ __forceinline__ void fr_layer(const floatx4 (&hin)[8][kFrTiles], floatx4 (&hout)[8][kFrTiles],
                                         float (&o)[3][kFrTiles], const float *W, int row, const float *b,
                                         const float *sW5, int lg, int lc) {
#pragma unroll
    for (int u0 = 0; u0 < 8; u0 += 2) {
        floatx4 acc[2][kFrTiles];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int p = 0; p < kFrTiles; ++p) acc[u][p] = *(const floatx4 *)(b + 16 * (u0 + u) + 4 * lg);
        fr_product<NK, 2, kFrTiles>(acc, hin, W, row, u0, lg, lc);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int n = 16 * (u0 + u) + 4 * lg;
#pragma unroll
            for (int p = 0; p < kFrTiles; ++p)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float z = acc[u][p][i], hv = z * sigmoidf_(z);
                    if (LAST) {
#pragma unroll
                        for (int j = 0; j < 3; ++j) o[j][p] = fmaf(hv, sW5[j * kW + n + i], o[j][p]);
                    } else {
                        hout[u0 + u][p][i] = hv;
                    }
                }
        }
    }
}

__global__ __launch_bounds__(kFrThreads) void mlp_fwd_fr(Geometry g, Shade s, MlpDev w, size_t M,
                                                         float4 *__restrict__ out) {
    // the weights of layers 0 and 2, and of 1 and 3
    __shared__ __attribute__((aligned(16))) float SW[2][kW * kFrRow];
    __shared__ __attribute__((aligned(16))) float sB[4 * kW];
    __shared__ float sW5[3 * kW];
    __shared__ PointEntry queues[kFrThreads / 64][kFrQueue];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int lg = lane >> 4, lc = lane & 15;
    for (int i = tid; i < 4 * kW; i += kFrThreads) sB[i] = w.b[i / kW][i % kW];
    for (int i = tid; i < 3 * kW; i += kFrThreads) sW5[i] = w.W5[i];
    const gfloat *Wr = (const gfloat *)(uint64_t)w.Wr;
    fr_issue<kFrThreads>(SW[0], Wr, kW * kFrRow0, tid);
    br_wait();
    __syncthreads();
    PointEntry *queue = queues[wv];
    // (a wave's groups go to it wave by wave over the workgroups: a launch with few
    // points then has one wave busy in each of many.  Where groups of 32 reach all
    // points in one round the waves take 32, one pass instead of two: 8 x 8 x 16
    // samples 146 -> 85 us a render, 24 x 24 x 64 148 -> 87)
    const unsigned takers = gridDim.x * (kFrThreads / 64), taker = wv * gridDim.x + blockIdx.x;
    const int deal = M <= (size_t)takers * 32 ? 32 : 64;
    const size_t rounds = ((M + deal - 1) / deal + takers - 1) / takers;
    size_t round = 0;
    int fill = 0;
    for (;;) {
        // the points the march reads, gathered as in mlp_fwd_rr; the waves of a
        // workgroup pass through the layers together, the idle ones with no points
        while (fill < 16 * kFrTiles && round < rounds) {
            const size_t m = dealt_group(round++, taker, takers) * deal + lane;
            float rh = 0.0f, zh = 0.0f;
            const bool read = lane < deal && m < M && point_coords(g, s, m, &rh, &zh);
            const unsigned long long mk = __ballot(read);
            if (read) queue[fill + __popcll(mk & ((1ull << lane) - 1ull))] = point_entry(m, rh, zh);
            fill += __popcll(mk);
        }
        if (!__syncthreads_or(fill > 0)) break;
        const int n = min(fill, 16 * kFrTiles);
        floatx4 ha[8][kFrTiles], hb[8][kFrTiles];
#pragma unroll
        for (int p = 0; p < kFrTiles; ++p) {
            const int e = 16 * p + lc;
            const float cr = e < n ? queue[e].rh : 0.0f, cz = e < n ? queue[e].zh : 0.0f;
            floatx4 f[4];
            fr_features(f, w, cr, cz, lg);
#pragma unroll
            for (int t = 0; t < 4; ++t) ha[t][p] = f[t];
        }
        float o[3][kFrTiles];
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int p = 0; p < kFrTiles; ++p) o[j][p] = 0.0f;
        auto next = [&](int buf, size_t off, int count) { fr_issue<kFrThreads>(SW[buf], Wr + off, count, tid); };
        auto done = [&] { br_wait(); __syncthreads(); };
        constexpr size_t L1 = (size_t)kW * kFrRow0, LN = (size_t)kW * kFrRow;
        next(1, L1, kW * kFrRow);
        fr_layer<4, false>(ha, hb, o, SW[0], kFrRow0, sB, sW5, lg, lc);
        done();
        next(0, L1 + LN, kW * kFrRow);
        fr_layer<8, false>(hb, ha, o, SW[1], kFrRow, sB + kW, sW5, lg, lc);
        done();
        next(1, L1 + 2 * LN, kW * kFrRow);
        fr_layer<8, false>(ha, hb, o, SW[0], kFrRow, sB + 2 * kW, sW5, lg, lc);
        done();
        next(0, 0, kW * kFrRow0);
        fr_layer<8, true>(hb, ha, o, SW[1], kFrRow, sB + 3 * kW, sW5, lg, lc);
        done();
#pragma unroll
        for (int p = 0; p < kFrTiles; ++p) {
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                o[j][p] += __shfl_xor(o[j][p], 16);
                o[j][p] += __shfl_xor(o[j][p], 32);
            }
            if (lg == 0 && 16 * p + lc < n)
                out[point_index(queue[16 * p + lc])] =
                    make_float4(o[0][p] + w.b5[0], o[1][p] + w.b5[1], o[2][p] + w.b5[2], 0.0f);
        }
        fill -= n;
        if (lane < fill) {
            const PointEntry e = queue[16 * kFrTiles + lane];
            queue[lane] = e;
        }
    }
}

// h and dL/dz = dL/dh SiLU'(z) of one neuron
__device__ __forceinline__ void fr_act_grad(float z, float dh, float *h, float *dz) {
    const float sg = sigmoidf_(z);
    *h = z * sg;
    *dz = dh * (sg * (1.0f + z * (1.0f - sg)));
}

// point-major write of a lane's neurons 16 t + 4 lg + i of its point
template <int N>
__device__ __forceinline__ void fr_write_rows(float *X, const floatx4 (&v)[N], int lg, int col) {
#pragma unroll
    for (int t = 0; t < N; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) X[(16 * t + 4 * lg + i) * kFrStride + col] = v[t][i];
}

// dW slice of one hidden layer over the 64 points, as br_dw
template <int NI>
__device__ __forceinline__ void fr_dw(floatx4 (&acc)[2][NI], const float *XD, const float *XH, int wv, int lg, int lc) {
#pragma unroll
    for (int kc = 0; kc < kBrPts / 16; ++kc) {
        const floatx4 a0 = *(const floatx4 *)(XD + (32 * wv + lc) * kFrStride + 16 * kc + 4 * lg);
        const floatx4 a1 = *(const floatx4 *)(XD + (32 * wv + 16 + lc) * kFrStride + 16 * kc + 4 * lg);
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            const floatx4 b = *(const floatx4 *)(XH + (16 * it + lc) * kFrStride + 16 * kc + 4 * lg);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc[0][it] = mfma_f32(a0[i], b[i], acc[0][it]);
                acc[1][it] = mfma_f32(a1[i], b[i], acc[1][it]);
            }
        }
    }
}

__device__ __forceinline__ float fr_rowsum(const float *X, int r, int half) {
    float sum = 0.0f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const floatx4 v = *(const floatx4 *)(X + r * kFrStride + 32 * half + 4 * q);
        sum += (v[0] + v[1]) + (v[2] + v[3]);
    }
    return sum + __shfl_xor(sum, 1);
}

// The passes of mlp_bwd_rr in FP32: one workgroup of four waves per CU, 64
// listed points a pass, 16 per wave; the recomputed forward parks z of every
// layer and the features lane-privately in the workgroup's slab of global
// memory (147 KB, 38 MB for the chip: past the L2s, in the memory-side cache; LDS holds the
// weights and the point-major rows), and the weight gradient accumulates in 232
// registers of each wave over all passes.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void mlp_bwd_fr(
    Geometry g, Shade s, MlpDev w, size_t M, const float4 *dO, const uint32_t *list, float *dW, floatx4 *slabs) {
    // point-major rows of the backward: dL/dz (or dL/do), then h (or features);
    // in the forward, layers 1 and 3's weights
    __shared__ __attribute__((aligned(16))) float XU[2 * kW * kFrStride];
    static_assert(2 * kW * kFrStride >= kW * kFrRow, "a hidden layer's weights fit the row buffers");
    float *const XD = XU;
    float *const XH = XU + kW * kFrStride;
    __shared__ __attribute__((aligned(16))) float SW[kW * kFrRow];
    __shared__ __attribute__((aligned(16))) float sB[4 * kW];
    __shared__ __attribute__((aligned(16))) float sW5[3 * kW];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int lg = lane >> 4, lc = lane & 15;
    floatx4 *const slab = slabs + (size_t)blockIdx.x * kFrSlab + tid;
    for (int i = tid; i < 4 * kW; i += 256) sB[i] = w.b[i / kW][i % kW];
    for (int i = tid; i < 3 * kW; i += 256) sW5[i] = w.W5[i];
    const floatx4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    floatx4 g0[2][4], g1[2][8], g2[2][8], g3[2][8], g4[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
#pragma unroll
        for (int b = 0; b < 4; ++b) g0[a][b] = zero;
#pragma unroll
        for (int b = 0; b < 8; ++b) { g1[a][b] = zero; g2[a][b] = zero; g3[a][b] = zero; }
        g4[a] = zero;
    }
    float db0 = 0.0f, db1 = 0.0f, db2 = 0.0f, db3 = 0.0f, db5 = 0.0f;
    const int brow = 32 * wv + (lane >> 1), bhalf = lane & 1;     // bias row of this lane
    const int col = 16 * wv + lc;                                 // this lane's point within the pass
    constexpr size_t L1 = (size_t)kW * kFrRow0, LN = (size_t)kW * kFrRow;
    fr_issue<256>(SW, (const gfloat *)(uint64_t)w.Wr, kW * kFrRow0, tid);
    br_wait();
    __syncthreads();
    const uint32_t npts = list[0];
    const uint32_t npass = (npts + kBrPts - 1) / kBrPts;
    for (uint32_t ip = blockIdx.x; ip < npass; ip += gridDim.x) {
        const uint32_t base = ip * kBrPts;
        const gfloat *Wr = (const gfloat *)(uint64_t)w.Wr, *WrT = (const gfloat *)(uint64_t)w.WrT;
        const size_t m = base + col < npts ? (size_t)list[1 + base + col] : M;   // M: no point
        float rh = 0.0f, zh = 0.0f;
        if (lane < 16 && m < M) point_coords(g, s, m, &rh, &zh);
        floatx4 h[8][1];
        {
            floatx4 f[4];
            fr_features(f, w, __shfl(rh, lc), __shfl(zh, lc), lg);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                slab[(32 + t) * 256] = f[t];
                h[t][0] = f[t];
            }
        }
        // ---- forward, parking z of every layer
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            // the next stage goes into the buffer that layer l does not read
            if (l < 3) fr_issue<256>(l & 1 ? SW : XU, Wr + L1 + l * LN, kW * kFrRow, tid);
            else fr_issue<256>(SW, WrT + 2 * LN, kW * kFrRow, tid);
            const float *W = l & 1 ? XU : SW;
            floatx4 hout[8];
#pragma unroll
            for (int u0 = 0; u0 < 8; u0 += 4) {
                floatx4 acc[4][1];
#pragma unroll
                for (int u = 0; u < 4; ++u) acc[u][0] = *(const floatx4 *)(sB + l * kW + 16 * (u0 + u) + 4 * lg);
                if (l == 0) fr_product<4, 4, 1>(acc, h, W, kFrRow0, u0, lg, lc);
                else fr_product<8, 4, 1>(acc, h, W, kFrRow, u0, lg, lc);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    slab[(8 * l + u0 + u) * 256] = acc[u][0];
                    if (l < 3) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) hout[u0 + u][i] = acc[u][0][i] * sigmoidf_(acc[u][0][i]);
                    }
                }
            }
            if (l < 3) {
#pragma unroll
                for (int t = 0; t < 8; ++t) h[t][0] = hout[t];
            }
            br_wait();
            __syncthreads();
        }
        // ---- output layer: dL/dh_3 = W5^T dL/do, then h_3 and dL/dz_3
        const float4 d = m < M ? dO[m] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        floatx4 hp[8], dz[8][1], dzu[8][1];   // h and dL/dz of the current layer, dL/dz of the layer above
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const floatx4 z = slab[(24 + u) * 256];
            const int n = 16 * u + 4 * lg;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float dh = fmaf(sW5[n + i], d.x, fmaf(sW5[kW + n + i], d.y, sW5[2 * kW + n + i] * d.z));
                float hv, dv;
                fr_act_grad(z[i], dh, &hv, &dv);
                hp[u][i] = hv;
                dz[u][0][i] = dv;
            }
        }
#pragma unroll
        for (int l = 3; l >= 0; --l) {
            // gradient of the layer above (the output layer when l == 3): its
            // dL/dz and this layer's h, point-major
            fr_write_rows<8>(XH, hp, lg, col);
            if (l == 3) {
                if (lg == 0) {
                    XD[0 * kFrStride + col] = d.x;
                    XD[1 * kFrStride + col] = d.y;
                    XD[2 * kFrStride + col] = d.z;
                } else {
                    // rows 3..15 are zero padding of the 16-row tile
#pragma unroll
                    for (int r = 0; r < 5; ++r) {
                        const int rr = 3 + 5 * (lg - 1) + r;
                        if (rr < 16) XD[rr * kFrStride + col] = 0.0f;
                    }
                }
            } else {
                floatx4 v[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) v[t] = dzu[t][0];
                fr_write_rows<8>(XD, v, lg, col);
            }
            __syncthreads();
            // SW is free: the transposed weights of the next product down, or
            // after the last one the next pass's layer 0
            if (l == 2 || l == 1) fr_issue<256>(SW, WrT + (l - 1) * LN, kW * kFrRow, tid);
            else if (l == 0) fr_issue<256>(SW, Wr, kW * kFrRow0, tid);
            if (l == 3) {
#pragma unroll
                for (int kc = 0; kc < kBrPts / 16; ++kc) {
                    const floatx4 a = *(const floatx4 *)(XD + lc * kFrStride + 16 * kc + 4 * lg);
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const floatx4 b = *(const floatx4 *)(XH + (16 * (wv + 4 * q) + lc) * kFrStride + 16 * kc + 4 * lg);
#pragma unroll
                        for (int i = 0; i < 4; ++i) g4[q] = mfma_f32(a[i], b[i], g4[q]);
                    }
                }
                if (wv == 0) {
                    const float v = fr_rowsum(XD, (lane >> 1) & 15, bhalf);   // rows 0..2 are dL/do
                    if (lane < 6) db5 += v;
                }
            } else if (l == 2) {
                fr_dw<8>(g3, XD, XH, wv, lg, lc);
                db3 += fr_rowsum(XD, brow, bhalf);
            } else if (l == 1) {
                fr_dw<8>(g2, XD, XH, wv, lg, lc);
                db2 += fr_rowsum(XD, brow, bhalf);
            } else {
                fr_dw<8>(g1, XD, XH, wv, lg, lc);
                db1 += fr_rowsum(XD, brow, bhalf);
            }
            if (l != 0) br_wait();
            __syncthreads();
#pragma unroll
            for (int t = 0; t < 8; ++t) dzu[t][0] = dz[t][0];
            // dL/dh of the layer below through the transposed weights, and at
            // once its h and dL/dz
            if (l >= 1) {
#pragma unroll
                for (int u0 = 0; u0 < 8; u0 += 4) {
                    floatx4 acc[4][1] = {{zero}, {zero}, {zero}, {zero}};
                    fr_product<8, 4, 1>(acc, dzu, SW, kFrRow, u0, lg, lc);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const floatx4 z = slab[(8 * (l - 1) + u0 + u) * 256];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            float hv, dv;
                            fr_act_grad(z[i], acc[u][0][i], &hv, &dv);
                            hp[u0 + u][i] = hv;
                            dz[u0 + u][0][i] = dv;
                        }
                    }
                }
            }
        }
        // ---- layer 0: features and dz_0
        {
            floatx4 f[4], v[8];
#pragma unroll
            for (int t = 0; t < 4; ++t) f[t] = slab[(32 + t) * 256];
#pragma unroll
            for (int t = 0; t < 8; ++t) v[t] = dz[t][0];
            fr_write_rows<4>(XH, f, lg, col);
            fr_write_rows<8>(XD, v, lg, col);
        }
        __syncthreads();
        fr_dw<4>(g0, XD, XH, wv, lg, lc);
        db0 += fr_rowsum(XD, brow, bhalf);
        br_wait();   // the next pass's layer-0 weights
        __syncthreads();
    }
    // ---- flush: flat layout per layer W [out][in] then b [out]
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int o = 32 * wv + 16 * a + 4 * lg + i;
#pragma unroll
            for (int it = 0; it < 4; ++it) atomicAdd(dW + w.off[0] + o * kF + 16 * it + lc, g0[a][it][i]);
#pragma unroll
            for (int it = 0; it < 8; ++it) {
                atomicAdd(dW + w.off[1] + o * kW + 16 * it + lc, g1[a][it][i]);
                atomicAdd(dW + w.off[2] + o * kW + 16 * it + lc, g2[a][it][i]);
                atomicAdd(dW + w.off[3] + o * kW + 16 * it + lc, g3[a][it][i]);
            }
        }
    if (bhalf == 0) {
        atomicAdd(dW + w.off[0] + kW * kF + brow, db0);
        atomicAdd(dW + w.off[1] + kW * kW + brow, db1);
        atomicAdd(dW + w.off[2] + kW * kW + brow, db2);
        atomicAdd(dW + w.off[3] + kW * kW + brow, db3);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int j = 4 * lg + i;
            if (j < 3) atomicAdd(dW + w.off[4] + j * kW + 16 * (wv + 4 * q) + lc, g4[q][i]);
        }
    if (wv == 0 && lane < 6 && bhalf == 0) atomicAdd(dW + w.off[4] + 3 * kW + (lane >> 1), db5);
}

// biases and output layer in float, both paths
__global__ void mlp_prep(const float *__restrict__ flat, MlpDev w) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    for (int l = 0; l < 4; ++l)
        if (i < kW) ((float *)w.b[l])[i] = flat[w.off[l] + kW * kLayerIn[l] + i];
    if (i < 3 * kW) ((float *)w.W5)[i] = flat[w.off[4] + i];
    if (i < 3) ((float *)w.b5)[i] = flat[w.off[4] + 3 * kW + i];
}

size_t mlp_prep_bytes(int precision) {
    const size_t hid = precision == RT_MLP_BF16 ? 2 * (kRrWeightElems + 3 * (size_t)kW * kRrRow)
                                                : 4 * (kFrWeightElems + 3 * (size_t)kW * kFrRow);
    return hid + 4 * (4 * kW + 3 * kW + 3) + 256 * 8;
}

hipError_t mlp_prepare(const float *flat, int precision, void *buf, MlpDev *w, hipStream_t st) {
    char *p = (char *)buf;
    auto take = [&](size_t b) { char *q = p; p += (b + 255) / 256 * 256; return q; };
    int off = 0;
    for (int l = 0; l < 4; ++l) {
        w->off[l] = off;
        off += kW * kLayerIn[l] + kW;
        w->b[l] = (const float *)take(4 * kW);
    }
    w->off[4] = off;
    w->W5 = (const float *)take(4 * 3 * kW);
    w->b5 = (const float *)take(4 * 3);
    const bool bf16 = precision == RT_MLP_BF16;
    w->Wr = take(bf16 ? 2 * kRrWeightElems : 4 * kFrWeightElems);
    w->WrT = take(bf16 ? 2 * 3 * (size_t)kW * kRrRow : 4 * 3 * (size_t)kW * kFrRow);
    for (int q = 0; q < 16; ++q) w->freq[q] = (float)std::exp2(3.0 * q / 15.0);
    hipLaunchKernelGGL(mlp_prep, dim3(2), dim3(256), 0, st, flat, *w);
    const int n = kW * (bf16 ? kRrRow : kFrRow);
    if (bf16) hipLaunchKernelGGL(mlp_prep_rr, dim3((n + 255) / 256), dim3(256), 0, st, flat, *w);
    else hipLaunchKernelGGL(mlp_prep_fr, dim3((n + 255) / 256), dim3(256), 0, st, flat, *w);
    return hipGetLastError();
}

hipError_t mlp_forward(const Geometry &g, const Shade &s, const MlpDev &w, int precision, size_t M, float4 *out,
                       hipStream_t st) {
    int dev = 0, ncu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    if (precision == RT_MLP_BF16) {
        constexpr int NP = kRrTiles, NT = kRrThreads;
        e = hipFuncSetAttribute((const void *)mlp_fwd_rr<NP, NT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)kRrLds);
        if (e != hipSuccess) return e;
        constexpr size_t pts = NT / 64 * NP * 16;
        const unsigned grid = (unsigned)std::min<size_t>((M + pts - 1) / pts, (size_t)ncu);
        hipLaunchKernelGGL((mlp_fwd_rr<NP, NT>), dim3(grid), dim3(NT), kRrLds, st, g, s, w, M, out);
    } else {
        constexpr size_t pts = kFrTiles * 16;     // a wave's pass
        const unsigned grid = (unsigned)std::min<size_t>((M + pts - 1) / pts, (size_t)ncu);
        hipLaunchKernelGGL(mlp_fwd_fr, dim3(grid), dim3(kFrThreads), 0, st, g, s, w, M, out);
    }
    return hipGetLastError();
}

// workgroups of the FP32 backward, each with a slab to park its pre-activations
static size_t fr_bwd_groups(size_t M) { return std::min<size_t>((M + kBrPts - 1) / kBrPts, 256); }

size_t mlp_backward_list_bytes(size_t M, int precision) {
    const size_t list = (sizeof(uint32_t) * (1 + M + 2 * (size_t)kLiveChunks) + 255) / 256 * 256;
    return list + (precision == RT_MLP_BF16 ? 0 : sizeof(floatx4) * kFrSlab * fr_bwd_groups(M));
}

hipError_t mlp_backward(const Geometry &g, const Shade &s, const MlpDev &w, int precision, size_t M,
                        const float4 *dO, uint32_t *list, float *dW, hipStream_t st) {
    int dev = 0, ncu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    const size_t passes = (M + kBrPts - 1) / kBrPts;
    // chunks of at least 1024 points, at most kLiveChunks of them
    const size_t chunk = std::max<size_t>(1024, (M + kLiveChunks - 1) / kLiveChunks);
    const int nb = (int)((M + chunk - 1) / chunk);
    uint32_t *counts = list + 1 + M, *offsets = counts + kLiveChunks;
    hipLaunchKernelGGL(mlp_live_count, dim3(nb), dim3(1024), 0, st, dO, M, chunk, counts);
    hipLaunchKernelGGL(mlp_live_scan, dim3(1), dim3(1024), 0, st, counts, nb, offsets, list);
    hipLaunchKernelGGL(mlp_live_write, dim3(nb), dim3(1024), 0, st, dO, M, chunk, offsets, list);
    if (precision == RT_MLP_BF16) {
        const unsigned grid = (unsigned)std::min<size_t>(passes, (size_t)ncu);
        hipLaunchKernelGGL(mlp_bwd_rr, dim3(grid), dim3(kBrThreads), 0, st, g, s, w, M, dO, list, dW);
    } else {
        const size_t list_b = (sizeof(uint32_t) * (1 + M + 2 * (size_t)kLiveChunks) + 255) / 256 * 256;
        hipLaunchKernelGGL(mlp_bwd_fr, dim3((unsigned)fr_bwd_groups(M)), dim3(256), 0, st, g, s, w, M, dO, list, dW,
                           (floatx4 *)((char *)list + list_b));
    }
    return hipGetLastError();
}

} // namespace rt
