// Learned preconditioner: a 3-level 3-D U-Net residual -> correction map used
// inside flexible GMRES, with block ILU(0) as the fallback (the paper's
// user-defined preconditioner hook, PC_USER with assemble / solve / destroy).
//
// Network (channels c0/c1/c2, default 16/32/64, 3x3x3 kernels, zero padding):
//   x0 = [r/s (3 channels), standardised ln k]           s = rms(r)
//   a1 = relu(conv0(x0)),  s1 = relu(conv1(a1))           full resolution
//   a2 = relu(conv2(pool(s1))), s2 = relu(conv3(a2))     1/2
//   a3 = relu(conv4(pool(s2))), b3 = relu(conv5(a3))     1/4
//   d2a = relu(conv6(up(b3)) + s2), d2 = relu(conv7(d2a))
//   d1a = relu(conv8(up(d2)) + s1), d1 = relu(conv9(d1a))
//   y = conv10(d1)  (1x1x1 linear to 3 channels),  z = s * y
// pool = 2x2x2 average, up = nearest-neighbour x2.  Activations and weights
// are BF16; every convolution is an implicit GEMM on the CDNA matrix cores
// (v_mfma_f32_16x16x32_bf16, FP32 accumulation).  Training: the backward
// data pass is the same kernel on transposed, tap-flipped weights; the weight
// gradient is a split-K MFMA GEMM over voxels with a fixed-order reduction;
// Adam keeps FP32 master weights.
#include "rsv_internal.h"

#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <type_traits>

typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
// a caller's BF16 input is at least 8-byte aligned
typedef short v8su __attribute__((ext_vector_type(8), aligned(8)));
typedef uint32_t v4wu __attribute__((ext_vector_type(4), aligned(8)));
typedef float v4fu __attribute__((ext_vector_type(4), aligned(4)));
typedef uint16_t v4hu __attribute__((ext_vector_type(4), aligned(4)));

namespace {

__device__ __host__ inline uint16_t f2bf(float f)
{
#ifdef __HIP_DEVICE_COMPILE__
    uint32_t u = __float_as_uint(f);
#else
    uint32_t u;
    std::memcpy(&u, &f, 4);
#endif
    if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ inline float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

constexpr int NL = 11;   // layers (10 convolutions 3x3x3 + final 1x1x1)

struct Arch {
    int c[3];
    int cin[NL], cout[NL];
    int64_t woff[NL], boff[NL], np;
    void init(int c0, int c1, int c2)
    {
        c[0] = c0; c[1] = c1; c[2] = c2;
        const int ci[NL] = {4, c0, c0, c1, c1, c2, c2, c1, c1, c0, c0};
        const int co[NL] = {c0, c0, c1, c1, c2, c2, c1, c1, c0, c0, 3};
        int64_t off = 0;
        for (int l = 0; l < NL; ++l) {
            cin[l] = ci[l];
            cout[l] = co[l];
            woff[l] = off;
            off += (int64_t)(l < 10 ? 27 : 1) * ci[l] * co[l];
            boff[l] = off;
            off += co[l];
        }
        np = off;
    }
    // K blocks (of 32 for inputs with a multiple of 8 channels, else 16): forward, backward data
    int kb(int l) const { return (27 * cin[l] + (cin[l] % 8 ? 15 : 31)) / (cin[l] % 8 ? 16 : 32); }
    int kbt(int l) const { return (27 * cout[l] + (cout[l] % 8 ? 15 : 31)) / (cout[l] % 8 ? 16 : 32); }
};

// A level of a batch: the samples' voxels follow one another, so the batch is
// one grid of nz = samples x nzs layers in which no stencil crosses a multiple
// of nzs.
struct ConvGeo {
    int nx, ny, nz;   // output resolution, all samples
    int nzs;          // layers of one sample
    int up;           // input is the half-resolution tensor, read nearest-up-sampled
    int cin, cout;
    int64_t V;        // voxels of all samples
};

// Bricks of 16 (x) x 4 (y) x TZ (z) output voxels; none spans two samples.
struct Brick {
    int x0, y0, z0;   // first voxel
    int zlo, zhi;     // layers of its sample
};
__host__ __device__ inline int brick_count(const ConvGeo &g, int tz)
{
    return ((g.nx + 15) / 16) * ((g.ny + 3) / 4) * ((g.nzs + tz - 1) / tz) * (g.nz / g.nzs);
}
__device__ inline Brick brick_of(const ConvGeo &g, int b, int tz)
{
    const int ntx = (g.nx + 15) / 16, nty = (g.ny + 3) / 4, ntz = (g.nzs + tz - 1) / tz;
    const int bz = b / (ntx * nty), smp = bz / ntz;
    Brick k;
    k.x0 = (b % ntx) * 16;
    k.y0 = ((b / ntx) % nty) * 4;
    k.zlo = smp * g.nzs;
    k.zhi = k.zlo + g.nzs;
    k.z0 = k.zlo + (bz - smp * ntz) * tz;
    return k;
}

// input voxel of (x, y, z) + (dx, dy, dz), or -1 outside the sample zlo .. zhi - 1
__device__ inline int64_t src_voxel(const ConvGeo &g, int x, int y, int z, int dx, int dy, int dz, int zlo, int zhi)
{
    const int a = x + dx, b = y + dy, c = z + dz;
    if (a < 0 || a >= g.nx || b < 0 || b >= g.ny || c < zlo || c >= zhi) return -1;
    if (g.up) {
        const int hx = g.nx >> 1, hy = g.ny >> 1;
        return (a >> 1) + (int64_t)hx * ((b >> 1) + (int64_t)hy * (c >> 1));
    }
    return a + (int64_t)g.nx * (b + (int64_t)g.ny * c);
}

// What a convolution does with its FP32 sums: + bias (+ skip), ReLU; or, for a
// data gradient, the ReLU mask of the activations the gradient belongs to
// (zero where mask <= 0), with an optional FP32 copy of the masked gradient.
struct Epilogue {
    const float *bias;
    const uint16_t *skip;
    int relu;
    const uint16_t *mask;
    float *copy;
    void *out;
};

// ---------------------------------------------------------------- convolution as implicit GEMM
// K per MFMA: 32 (v_mfma_f32_16x16x32_bf16, 8 k per lane) when the input has a
// multiple of 8 channels, so that a lane's 8 consecutive k are 8 channels of
// one tap; else 16 (v_mfma_f32_16x16x16_bf16, 4 k per lane).
__host__ __device__ constexpr int conv_kw(int cin) { return cin % 8 == 0 ? 32 : 16; }
__host__ __device__ constexpr int conv_kblocks(int cin) { return (27 * cin + conv_kw(cin) - 1) / conv_kw(cin); }
// bytes of one lane's packed weight fragment
__host__ __device__ constexpr int conv_frag_bytes(int cin) { return conv_kw(cin) / 2; }
template <bool K32> struct Frag { using T = v4s; static constexpr int KW = 16; };
template <> struct Frag<true> { using T = v8s; static constexpr int KW = 32; };
__device__ inline v4f mfma_k(v4s a, v4s b, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0); }
__device__ inline v4f mfma_k(v8s a, v8s b, v4f c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}

// Any multiple of 4 input channels, operands from global memory (the single
// layers of rsv_conv3d whose channel count has no staged kernel below).
// One wavefront: 16*MB output voxels x (16*NB) output channels.  GEMM row m =
// voxel, column n = output channel, k = tap*cin + ci.  Operand fragments
// (KW = 16 or 32, w = KW / 4 k per lane): lane l holds A[m = l%16][k = w*(l/16)
// .. + w-1] and B[k = w*(l/16) .. + w-1][n = l%16]; the result holds
// D[m = 4*(l/16) + i][n = l%16].  Weights are pre-packed so that B fragments
// are one load per lane; an A fragment's lane reads w consecutive channels of
// one voxel.  Each B fragment feeds MB products and each A fragment NB.
template <int MB, int NB, bool K32>
__global__ __launch_bounds__(256) void k_conv(ConvGeo g, const uint16_t *__restrict__ X, const void *__restrict__ Wfv,
                                              int KB, const float *__restrict__ bias, float *__restrict__ out)
{
    using FT = typename Frag<K32>::T;
    constexpr int KW = Frag<K32>::KW;
    const FT *Wf = (const FT *)Wfv;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t v0 = ((int64_t)blockIdx.x * 4 + wave) * (16 * MB);
    if (v0 >= g.V) return;
    const int m = lane & 15, kq = (KW / 4) * (lane >> 4);
    int px[MB], py[MB], pz[MB];
    bool live[MB];   // the last tile of a level may be partial
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        const int64_t v = v0 + mb * 16 + m;
        live[mb] = v < g.V;
        px[mb] = (int)(v % g.nx);
        py[mb] = (int)((v / g.nx) % g.ny);
        pz[mb] = (int)(v / ((int64_t)g.nx * g.ny));
    }
    v4f acc[MB][NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = v4f{0.f, 0.f, 0.f, 0.f};
    const int K = 27 * g.cin;
    for (int kb = 0; kb < KB; ++kb) {
        const int k = kb * KW + kq;
        const bool kin = k < K;
        const int tap = kin ? k / g.cin : 0, ci = k - tap * g.cin;
        const int dz = tap / 9 - 1, dy = (tap / 3) % 3 - 1, dx = tap % 3 - 1;
        FT a[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            a[mb] = FT{};
            if (kin && live[mb]) {
                const int64_t u = src_voxel(g, px[mb], py[mb], pz[mb], dx, dy, dz, 0, g.nz);
                if (u >= 0) a[mb] = *(const FT *)(X + u * g.cin + ci);
            }
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const FT b = Wf[((int64_t)kb * NB + nb) * 64 + lane];
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) acc[mb][nb] = mfma_k(a[mb], b, acc[mb][nb]);
        }
    }
    const int n = lane & 15, mr = 4 * (lane >> 4);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int co = nb * 16 + n;
        const float bb = bias ? bias[co] : 0.f;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t vo = v0 + mb * 16 + mr + i;
                if (vo < g.V) out[vo * g.cout + co] = acc[mb][nb][i] + bb;
            }
    }
}

// The convolution of the network's channel counts (4, 16, 32 or 64 inputs).  A
// workgroup takes bricks of 16 (x) x 4 (y) x TZ (z) output voxels (brick b,
// b + gridDim.x, ...): a brick's input halo (zero outside the sample, nearest
// up-sampled when `up`) goes to LDS from registers that were loaded during the
// previous brick's MFMAs.  Wave w owns the brick's plane w % TZ and the output
// channels of its split w / TZ: four x-rows of 16 voxels x 16 NBW channels.
// blockIdx.y and the splits divide the output channels.
//
// The weights are the MFMA's rows (m = output channel) and the voxels its
// columns (n = voxel), so a lane ends with 4 consecutive channels of one voxel
// and stores them, and reads bias, skip and mask, in one access; a wave's
// store covers 16 whole neighbouring voxels.  The K order (tap, channel) is the
// packed weights'.
//
// The K loop is unrolled: with 32 and 64 channels every operand address is one
// per-lane base and an immediate, and the x-rows that two taps of one (z, x)
// offset share are read once; with 4 and 16, where a K block spans taps, the
// per-lane offsets of the blocks are kept in registers.  (Decoding the tap of
// every K block cost about as many cycles as its MFMAs, and an epilogue through
// LDS as many again.  Measured at 128x128x64, before and after: 4->16 33 -> 22
// us, 16->16 67 -> 37, up-sampled 32->16 118 -> 58 (500 TFLOP/s); at 64x64x32:
// 16->32 18 -> 13, up-sampled 64->32 75 -> 28.  With 16 output channels an MFMA
// takes one 16-byte operand per lane from LDS, which is active in 60 % of the
// cycles with 16 inputs and 40 % with 32, the MFMAs in 23 %.)  The weights are
// staged in LDS once per workgroup; those of 64 channels do not fit beside a
// halo and come through the L1 from the L2 (460 registers, one workgroup per CU:
// LDS 20 %, MFMAs 18 %).  VS, the LDS stride of a voxel, is an odd number of
// 16-byte units, so that the 16 voxels of a quad's read fall on distinct banks;
// the quads', which are other taps or channels, still meet: bank conflicts are 45 %
// of the LDS cycles.
template <int CIN, int NBW, int NSPLIT, int TZ> struct ConvCfg {
    static constexpr int NT = 64 * TZ * NSPLIT;
    static constexpr int KB = conv_kblocks(CIN);
    static constexpr int FB = conv_frag_bytes(CIN);
    static constexpr bool WLDS = CIN <= 32;
    static constexpr int HN = 18 * 6 * (TZ + 2);
    static constexpr int VS = CIN == 4 ? 4 : CIN + 8;   // shorts
    static constexpr size_t WBYTES = WLDS ? (size_t)KB * NSPLIT * NBW * 64 * FB : 0;
    static constexpr size_t LDS = WBYTES + (size_t)HN * VS * 2;
};

template <int CIN, int NBW, int NSPLIT, int TZ, bool OUT_BF16>
__global__ __launch_bounds__(64 * TZ * NSPLIT) void k_conv_lds(ConvGeo g, const uint16_t *__restrict__ X,
                                                               const void *__restrict__ Wfv, Epilogue ep)
{
    using C = ConvCfg<CIN, NBW, NSPLIT, TZ>;
    using FT = typename Frag<CIN % 8 == 0>::T;
    constexpr int NT = C::NT, KB = C::KB, VS = C::VS, NBG = NSPLIT * NBW;
    constexpr int WPT = CIN == 4 ? 4 : 8, CW = CIN / WPT;       // channels per halo word, words per voxel
    constexpr int NI = (C::HN * CW + NT - 1) / NT;
    extern __shared__ __align__(16) unsigned char cl[];
    FT *wl = (FT *)cl;                                          // [KB][NBG][64]
    uint16_t *xl = (uint16_t *)(cl + C::WBYTES);                // [HN][VS]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int plane = wave % TZ, split = wave / TZ;
    const int NB = g.cout / 16;
    const int nbw0 = blockIdx.y * NBG + split * NBW;            // this wave's first channel block
    const FT *Wf = (const FT *)Wfv;
    if constexpr (C::WLDS)
        for (int e = tid; e < KB * NBG * 64; e += NT)
            wl[e] = Wf[((int64_t)(e / (NBG * 64)) * NB + blockIdx.y * NBG + (e / 64) % NBG) * 64 + (e & 63)];
    // halo words of this thread: voxel (hx, hy, hz) packed, and its input voxel from the brick's
    int hpos[NI], hrel[NI];
    const int sx = g.up ? g.nx >> 1 : g.nx, sy = g.up ? g.ny >> 1 : g.ny;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int h = (tid + NT * i) / CW;
        const int hx = h % 18, hy = (h / 18) % 6, hz = h / 108;
        hpos[i] = hx | hy << 8 | hz << 16;
        hrel[i] = g.up ? ((hx - 1) >> 1) + sx * (((hy - 1) >> 1) + sy * ((hz - 1) >> 1))
                       : (hx - 1) + sx * ((hy - 1) + sy * (hz - 1));
    }
    using WT = std::conditional_t<CIN == 4, v4s, v8s>;
    WT hv[NI];
    auto load = [&](const Brick &k) {
        const int64_t base = g.up ? (k.x0 >> 1) + (int64_t)sx * ((k.y0 >> 1) + (int64_t)sy * (k.z0 >> 1))
                                  : k.x0 + (int64_t)sx * (k.y0 + (int64_t)sy * k.z0);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int e = tid + NT * i, ha = hpos[i];
            const int a = k.x0 + (ha & 255) - 1, b = k.y0 + ((ha >> 8) & 255) - 1, c = k.z0 + (ha >> 16) - 1;
            hv[i] = WT{};
            if (e < C::HN * CW && (unsigned)a < (unsigned)g.nx && (unsigned)b < (unsigned)g.ny && c >= k.zlo && c < k.zhi) {
                const uint16_t *src = X + (base + hrel[i]) * CIN + WPT * (e % CW);
                if constexpr (CIN == 4) hv[i] = *(const v4s *)src;
                else hv[i] = *(const v8su *)src;
            }
        }
    };
    const int n = lane & 15, quad = lane >> 4;
    // LDS offset (shorts) of K block kb for this lane, row 0 of its plane
    auto tap_off = [](int t) { return ((t / 9) * 108 + ((t / 3) % 3) * 18 + t % 3) * VS; };
    const int lane_base = (plane * 108 + n) * VS + (CIN >= 32 ? 8 * quad : CIN == 16 ? 8 * (quad & 1) : 0);
    int koff[CIN <= 16 ? KB : 1];
    if constexpr (CIN <= 16)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const int t = CIN == 16 ? 2 * kb + (quad >> 1) : 4 * kb + quad;
            koff[kb] = lane_base + tap_off(t < 27 ? t : 26);
        }
    const bool last_in = CIN == 16 ? quad < 2 : CIN == 4 ? quad < 3 : true;   // the last K block ends at tap 27
    v4f bias[NBW];
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
        for (int i = 0; i < 4; ++i) bias[nb][i] = ep.bias ? ep.bias[(nbw0 + nb) * 16 + 4 * quad + i] : 0.f;
    const int nbricks = brick_count(g, TZ);
    Brick cur = brick_of(g, blockIdx.x, TZ);
    if ((int)blockIdx.x < nbricks) load(cur);
    for (int b = blockIdx.x; b < nbricks; b += gridDim.x) {
        const Brick k = cur;
        __syncthreads();   // the previous brick's operands have been read (and the weights written)
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int e = tid + NT * i;
            if (e < C::HN * CW) *(WT *)(xl + (e / CW) * VS + WPT * (e % CW)) = hv[i];
        }
        __syncthreads();
        if (b + (int)gridDim.x < nbricks) {
            cur = brick_of(g, b + gridDim.x, TZ);
            load(cur);
        }
        v4f acc[4][NBW];
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) acc[r][nb] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            FT x[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int at = CIN <= 16 ? koff[CIN <= 16 ? kb : 0]
                                         : lane_base + tap_off(CIN == 64 ? kb >> 1 : kb) + (CIN == 64 ? 32 * (kb & 1) : 0);
                x[r] = *(const FT *)(xl + at + r * 18 * VS);
                if (kb == KB - 1 && !last_in) x[r] = FT{};
            }
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) {
                const FT w = C::WLDS ? wl[(kb * NBG + split * NBW + nb) * 64 + lane]
                                     : Wf[((int64_t)kb * NB + nbw0 + nb) * 64 + lane];
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[r][nb] = mfma_k(w, x[r], acc[r][nb]);
            }
        }
        const int vx = k.x0 + n, vz = k.z0 + plane;
        if (vx < g.nx && vz < k.zhi) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (k.y0 + r >= g.ny) break;
                const int64_t vo = (vx + (int64_t)g.nx * (k.y0 + r + (int64_t)g.ny * vz)) * g.cout + nbw0 * 16 + 4 * quad;
#pragma unroll
                for (int nb = 0; nb < NBW; ++nb) {
                    v4f v = acc[r][nb] + bias[nb];
                    const int64_t o = vo + 16 * nb;
                    if (ep.skip) {
                        const v4hu q = *(const v4hu *)(ep.skip + o);
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] += bf2f(q[i]);
                    }
                    if (ep.relu)
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] = v[i] > 0.f ? v[i] : 0.f;
                    if (ep.mask) {
                        const v4hu q = *(const v4hu *)(ep.mask + o);
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] = bf2f(q[i]) > 0.f ? v[i] : 0.f;
                    }
                    if (ep.copy) *(v4fu *)(ep.copy + o) = v;
                    if (OUT_BF16) {
                        v4hu h;
#pragma unroll
                        for (int i = 0; i < 4; ++i) h[i] = f2bf(v[i]);
                        *(v4hu *)((uint16_t *)ep.out + o) = h;
                    } else {
                        *(v4fu *)((float *)ep.out + o) = v;
                    }
                }
            }
        }
    }
}

template <int CIN, int NBW, int NSPLIT, int TZ, bool OUT_BF16>
hipError_t launch_conv_lds(const rsv_ctx *c, const ConvGeo &g, const uint16_t *X, const void *Wf, const Epilogue &ep)
{
    using C = ConvCfg<CIN, NBW, NSPLIT, TZ>;
    auto *fn = &k_conv_lds<CIN, NBW, NSPLIT, TZ, OUT_BF16>;
    if (C::LDS > 65536) {
        const hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS);
        if (e != hipSuccess) return e;
    }
    // As many workgroups as the CUs hold at once (1 to 5 each, by registers and
    // LDS), walking the bricks with their weights staged once: more would run as a
    // second, part-empty round.  1024 in all cases, then resident: 4 -> 16 channels
    // 22.1 -> 21.2 us at 128x128x64, 16 -> 16 37.6 -> 33.2, 32 -> 16 58.4 -> 55.9,
    // 32 -> 32 (64x64x32) 20.2 -> 18.1, 64 -> 32 28.2 -> 22.9.
    static const int resident = [&] {
        int nb = 0;
        const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void *)fn, C::NT, C::LDS);
        return e == hipSuccess && nb > 0 ? nb : 2;
    }();
    const unsigned groups = (unsigned)(g.cout / (16 * NSPLIT * NBW));
    const unsigned nwg = std::min<unsigned>((unsigned)brick_count(g, TZ), std::max(1u, (unsigned)c->num_cu * resident / groups));
    hipLaunchKernelGGL(fn, dim3(nwg, groups), dim3(C::NT), C::LDS, c->stream, g, X, Wf, ep);
    return hipGetLastError();
}

// Convolution launch: the staged kernels for the network's channel counts, else
// the general one (rsv_conv3d alone: FP32 out, bias).
template <bool OUT_BF16>
hipError_t launch_conv(const rsv_ctx *c, const ConvGeo &g, const uint16_t *X, const void *Wf, int KB, const Epilogue &ep)
{
    const int NB = g.cout / 16;
    if (g.cout % 16 || (NB != 1 && NB != 2 && NB != 4)) return hipErrorInvalidValue;
    const bool staged = (int64_t)g.nx * g.ny < (1 << 28);   // the staged kernel's halo offsets are 32-bit
    if (!staged) {
    } else if (g.cin == 4) {
        if (NB == 1) return launch_conv_lds<4, 1, 1, 4, OUT_BF16>(c, g, X, Wf, ep);
        if (NB == 2) return launch_conv_lds<4, 2, 1, 4, OUT_BF16>(c, g, X, Wf, ep);
        return launch_conv_lds<4, 4, 1, 4, OUT_BF16>(c, g, X, Wf, ep);
    } else if (g.cin == 16) {
        if (NB == 1) return launch_conv_lds<16, 1, 1, 4, OUT_BF16>(c, g, X, Wf, ep);
        if (NB == 2) return launch_conv_lds<16, 2, 1, 4, OUT_BF16>(c, g, X, Wf, ep);
        return launch_conv_lds<16, 4, 1, 4, OUT_BF16>(c, g, X, Wf, ep);
    } else if (g.cin == 32) {
        if (NB == 1) return launch_conv_lds<32, 1, 1, 4, OUT_BF16>(c, g, X, Wf, ep);
        return launch_conv_lds<32, 2, 1, 4, OUT_BF16>(c, g, X, Wf, ep);
    } else if (g.cin == 64) {
        if (NB == 1) return launch_conv_lds<64, 1, 1, 4, OUT_BF16>(c, g, X, Wf, ep);
        return launch_conv_lds<64, 1, 2, 2, OUT_BF16>(c, g, X, Wf, ep);
    }
    if (OUT_BF16 || ep.skip || ep.relu || ep.mask || ep.copy || g.up || g.nz != g.nzs) return hipErrorInvalidValue;
    const int MB = g.V >= 131072 ? 4 : 1;   // four voxel blocks per wave reuse the weights; small levels need the waves
    const int64_t waves = (g.V + 16 * MB - 1) / (16 * MB);
    const dim3 grid((unsigned)((waves + 3) / 4)), blk(256);
#define RSV_CONV(mb, nb)                                                                                             \
    do {                                                                                                             \
        if (g.cin % 8 == 0)                                                                                          \
            hipLaunchKernelGGL((k_conv<mb, nb, true>), grid, blk, 0, c->stream, g, X, Wf, KB, ep.bias, (float *)ep.out);    \
        else                                                                                                         \
            hipLaunchKernelGGL((k_conv<mb, nb, false>), grid, blk, 0, c->stream, g, X, Wf, KB, ep.bias, (float *)ep.out);   \
    } while (0)
    if (MB == 4) {
        if (NB == 1) RSV_CONV(4, 1);
        else if (NB == 2) RSV_CONV(4, 2);
        else RSV_CONV(4, 4);
    } else {
        if (NB == 1) RSV_CONV(1, 1);
        else if (NB == 2) RSV_CONV(1, 2);
        else RSV_CONV(1, 4);
    }
#undef RSV_CONV
    return hipGetLastError();
}

// Weight and bias gradients, dW[tap][ci][co] = sum_v X[v + off(tap)][ci] G[v][co]
// and db[co] = sum_v G[v][co], as an MFMA GEMM over voxels on
// v_mfma_f32_16x16x32_bf16 (rows m = ci, columns n = co, k = voxel; lane l
// holds A[m = l%16][k = 8*(l/16) .. +7], B[k = 8*(l/16) .. +7][n = l%16], and
// D[m = 4*(l/16) + i][n = l%16]).  A workgroup owns one 16 x 16 channel pair
// (ci block, co block) and a chunk of bricks of 16 (x) x 4 (y) x 4 (z)
// voxels.  Per brick it stages in LDS, as they lie in memory (a voxel's 16
// channels in a row), the input halo and the gradient tile; the fragments, one
// channel of eight voxels per lane, come from transposing LDS reads: the 16 lanes
// of a group read four voxels' rows (lane i: voxel i / 4, channels 4 (i % 4) ..
// + 3), and lane i receives channel i of the four.  k runs over x of two rows, so
// that a read takes 512 bytes in a line, and a tap's shift is an offset.  Wave w
// computes the taps t = w, w + 4, ... for all 256 voxels (the B fragment of a
// k-step serves all its taps).  The next brick's global loads are issued before
// the MFMAs of the current one.
//
// Bound by latency, at two workgroups per CU: of 32 us for 16 x 16 channels on
// 2^20 voxels (4096 bricks, 67 MB: 14 us), 27 remain without the global loads, the
// 1 KiB fragments of LDS take 15 at 128 bytes per cycle and the MFMAs 6.  Steps:
// channel-major staging, one copy per dx, 24 transposing stores and 20 loads of 8
// bytes per thread and brick, 63 KB: 110 us (32 x 16 channels 199); transposing
// reads 44 (74); places of the halo's pieces computed once 41; bias sums by
// shuffles instead of one thread per channel 37; a step's fragments read before
// the last one's MFMAs 32 (54).  All ten layers of the network, 8 samples of
// 64 x 64 x 32: 820 -> 236 us.  256 workgroups: 322 us; 1024: 273, and the
// reduction 77 instead of 59.
//
// Split over voxels: each chunk writes one partial (taps, then the bias sums
// for ci block 0); k_dw_reduce adds them in a fixed order into the gradients.
// (Summing them inside this kernel, by the last workgroup to finish, needs a
// device-scope release per workgroup, which writes back the XCD's L2: 5x the
// time of this kernel and the reduction together at 64x64x32.)
constexpr int CT_Y = 4, CT_Z = 4, CH_X = 18, CH_Y = CT_Y + 2, CH_Z = CT_Z + 2;
constexpr int DW_PART = 27 * 256 + 16;        // floats per partial: 27 taps x 16 x 16, then 16 bias sums
constexpr int DW_WGS = 512;                   // workgroups aimed at, so chunks per pair at most
constexpr int DW_XU = CH_Z * CH_Y * CH_X * 2; // 16-byte pieces of the input halo: (voxel, channel octet)
constexpr int DW_GU = CT_Z * CT_Y * 16 * 2;   // of the gradient tile
constexpr int DW_NX = (DW_XU + 255) / 256, DW_NG = DW_GU / 256;

// channel l%16 of the voxels 4 (l/16) .. + 3 of the row of 32-byte voxels at p; p: the lane's own 8 bytes
__device__ __forceinline__ v4s lds_tr(const unsigned char *p)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)p);
}

__global__ __launch_bounds__(256) void k_conv_dw(ConvGeo g, const uint16_t *__restrict__ X,
                                                 const uint16_t *__restrict__ G, int npairs,
                                                 int bricks_per_chunk, float *__restrict__ partials)
{
    __shared__ __align__(16) uint4 xs[DW_XU], gs[DW_GU];   // [z][y][x][16 channels]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int blk = (int)xcd_block(blockIdx.x, gridDim.x);   // a chunk's pairs, and its neighbours, on one die
    const int pair = blk % npairs, chunk = blk / npairs;
    const int cob_n = g.cout / 16, cib = pair / cob_n, cob = pair % cob_n;
    const int nbricks = brick_count(g, CT_Z);
    const int b_begin = chunk * bricks_per_chunk;
    const int b_end = b_begin + bricks_per_chunk < nbricks ? b_begin + bricks_per_chunk : nbricks;
    const bool wide = g.cin % 8 == 0;
    const int c0 = cib * 16 + 8 * (tid & 1);      // first channel of this thread's pieces
    v4f acc[7];
#pragma unroll
    for (int j = 0; j < 7; ++j) acc[j] = v4f{0.f, 0.f, 0.f, 0.f};
    float bq[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};   // bias sums of channels 8 (tid & 1) .. + 7
    v4wu rx[DW_NX], rg[DW_NG];
    // Places of this thread's pieces from the brick's first voxel; bricks begin at
    // even coordinates, so halving them (up) is exact.
    const int sx = g.up ? g.nx >> 1 : g.nx, sy = g.up ? g.ny >> 1 : g.ny;
    int64_t xo[DW_NX], go[DW_NG];
    int hc[DW_NX];               // halo coordinates, a byte each; 31 in each byte: no piece
#pragma unroll
    for (int k = 0; k < DW_NX; ++k) {
        const int u = tid + 256 * k, v = u >> 1;
        const int hx = v % CH_X, hy = (v / CH_X) % CH_Y, hz = v / (CH_X * CH_Y);
        const bool on = u < DW_XU && c0 < g.cin;
        hc[k] = on ? hx | hy << 8 | hz << 16 : 31 | 31 << 8 | 31 << 16;
        xo[k] = ((hx - 1) >> g.up) + (int64_t)sx * (((hy - 1) >> g.up) + (int64_t)sy * ((hz - 1) >> g.up));
        xo[k] = xo[k] * g.cin + c0;
    }
#pragma unroll
    for (int k = 0; k < DW_NG; ++k) {
        const int v = (tid + 256 * k) >> 1;
        go[k] = ((v & 15) + (int64_t)g.nx * (((v >> 4) & 3) + (int64_t)g.ny * (v >> 6))) * g.cout + cob * 16 + 8 * (tid & 1);
    }
    auto load = [&](int b) {
        const Brick bk = brick_of(g, b, CT_Z);
        // halo coordinates inside the sample: lo .. lo + n - 1
        const int xl = bk.x0 == 0, xn = min(CH_X, g.nx - bk.x0 + 1) - xl, yl = bk.y0 == 0, yn = min(CH_Y, g.ny - bk.y0 + 1) - yl;
        const int zl = bk.z0 == bk.zlo, zn = min(CH_Z, bk.zhi - bk.z0 + 1) - zl;
        const uint16_t *xb =
            X + ((bk.x0 >> g.up) + (int64_t)sx * ((bk.y0 >> g.up) + (int64_t)sy * (bk.z0 >> g.up))) * g.cin;
#pragma unroll
        for (int k = 0; k < DW_NX; ++k) {
            rx[k] = v4wu{0, 0, 0, 0};
            const bool in = ((unsigned)((hc[k] & 255) - xl) < (unsigned)xn) & ((unsigned)((hc[k] >> 8 & 255) - yl) < (unsigned)yn) &
                            ((unsigned)((hc[k] >> 16) - zl) < (unsigned)zn);
            if (!in) continue;
            const uint16_t *p = xb + xo[k];
            if (wide) {
                rx[k] = *(const v4wu *)p;
            } else {
                const uint2 lo = *(const uint2 *)p;
                rx[k].x = lo.x;
                rx[k].y = lo.y;
                if (c0 + 4 < g.cin) {
                    const uint2 hi = *(const uint2 *)(p + 4);
                    rx[k].z = hi.x;
                    rx[k].w = hi.y;
                }
            }
        }
        const uint16_t *gb = G + (bk.x0 + (int64_t)g.nx * (bk.y0 + (int64_t)g.ny * bk.z0)) * g.cout;
#pragma unroll
        for (int k = 0; k < DW_NG; ++k) {
            const int v = (tid + 256 * k) >> 1;
            rg[k] = v4wu{0, 0, 0, 0};
            if ((v & 15) < g.nx - bk.x0 && ((v >> 4) & 3) < g.ny - bk.y0 && (v >> 6) < bk.zhi - bk.z0)
                rg[k] = *(const v4wu *)(gb + go[k]);
        }
    };
    auto store = [&]() {
#pragma unroll
        for (int k = 0; k < DW_NX; ++k)
            if (tid + 256 * k < DW_XU) xs[tid + 256 * k] = uint4{rx[k].x, rx[k].y, rx[k].z, rx[k].w};
#pragma unroll
        for (int k = 0; k < DW_NG; ++k) {
            gs[tid + 256 * k] = uint4{rg[k].x, rg[k].y, rg[k].z, rg[k].w};
            if (cib == 0) {
                const uint32_t w[4] = {rg[k].x, rg[k].y, rg[k].z, rg[k].w};
#pragma unroll
                for (int i = 0; i < 8; ++i) bq[i] += bf2f((uint16_t)(w[i >> 1] >> (16 * (i & 1))));
            }
        }
    };
    // this lane's place in a row of voxels, and with its taps' shifts
    const int at = (4 * (lane >> 4) + ((lane & 15) >> 2)) * 32 + (lane & 3) * 8;
    const unsigned char *gp = (const unsigned char *)gs + at, *xp[7];
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        const int t = wave + 4 * j < 27 ? wave + 4 * j : 26;
        xp[j] = (const unsigned char *)xs + ((t / 9 * CH_Y + (t / 3) % 3) * CH_X + t % 3) * 32 + at;
    }
    auto frag = [](const unsigned char *p, int row) {   // two rows, row bytes apart
        const v4s lo = lds_tr(p), hi = lds_tr(p + row);
        return __builtin_bit_cast(v8bf, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    if (b_begin < b_end) load(b_begin);
    for (int b = b_begin; b < b_end; ++b) {
        __syncthreads();   // the previous brick's fragments have been read
        store();
        __syncthreads();
        if (b + 1 < b_end) load(b + 1);
        // k-step s: plane s / 2, rows 2 (s % 2) and the next; the next step's
        // fragments are read before this one's MFMAs
        struct Frags {
            v8bf a[7], b;
        } f[2];
        auto read = [&](Frags &o, int s) {
            const int z = s >> 1, row = 2 * (s & 1);
            o.b = frag(gp + (z * CT_Y + row) * 16 * 32, 16 * 32);
#pragma unroll
            for (int j = 0; j < 7; ++j) o.a[j] = frag(xp[j] + (z * CH_Y + row) * CH_X * 32, CH_X * 32);
        };
        read(f[0], 0);
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            if (s < 7) read(f[(s + 1) & 1], s + 1);
            asm volatile("" ::: "memory");   // not sunk to their uses
#pragma unroll
            for (int j = 0; j < 7; ++j)   // wave 3 repeats tap 26: a branch would cost copies of the sums
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[s & 1].a[j], f[s & 1].b, acc[j], 0, 0, 0);
        }
    }
    // this chunk's partial: taps of this wave, then (ci block 0) the bias sums
    float *part = partials + ((int64_t)chunk * npairs + pair) * DW_PART;
    const int m = lane & 15;
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        const int t = wave + 4 * j;
        if (t < 27)
#pragma unroll
            for (int i = 0; i < 4; ++i) part[t * 256 + (4 * (lane >> 4) + i) * 16 + m] = acc[j][i];
    }
    if (cib == 0) {
        __syncthreads();
        float *red = (float *)xs;   // [wave][16 channels]
#pragma unroll
        for (int c = 0; c < 8; ++c) {   // the lanes of this octet
#pragma unroll
            for (int d = 2; d < 64; d *= 2) bq[c] += __shfl_xor(bq[c], d);
            if (lane < 2) red[wave * 16 + 8 * lane + c] = bq[c];
        }
        __syncthreads();
        if (tid < 16) part[27 * 256 + tid] = (red[tid] + red[16 + tid]) + (red[32 + tid] + red[48 + tid]);
    }
}

// grad_w += scale * (sum of the chunks' weight partials), grad_b likewise for
// the bias sums, in a fixed order: a workgroup owns 16 float4 of one pair's
// partial; thread t sums chunk group t / 16 (chunks t / 16, + 16, ...: up to
// 16 loads in flight), then 16 threads add the 16 group sums in group order.
__global__ __launch_bounds__(256) void k_dw_reduce(const float *__restrict__ partials, int npairs, int nchunks,
                                                   int cin, int cout, float scale, float *__restrict__ grad_w,
                                                   float *__restrict__ grad_b)
{
    __shared__ float4 gsum[16][16];
    constexpr int NE4 = DW_PART / 4, SLICES = (NE4 + 15) / 16;
    const int pair = blockIdx.x / SLICES, slice = blockIdx.x % SLICES;
    const int cob_n = cout / 16, cib = pair / cob_n, cob = pair % cob_n;
    const int gr = threadIdx.x >> 4, e4 = slice * 16 + (threadIdx.x & 15);
    const int64_t stride = (int64_t)npairs * DW_PART;
    float4 s4 = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int c0 = 0; c0 < nchunks; c0 += 256) {
        float4 v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int ch = c0 + gr + 16 * i;
            v[i] = (e4 < NE4 && ch < nchunks) ? *(const float4 *)(partials + ch * stride + (int64_t)pair * DW_PART + 4 * e4)
                                              : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) { s4.x += v[i].x; s4.y += v[i].y; s4.z += v[i].z; s4.w += v[i].w; }
    }
    gsum[gr][threadIdx.x & 15] = s4;
    __syncthreads();
    if (threadIdx.x >= 16 || e4 >= NE4) return;
    float4 t4 = gsum[0][threadIdx.x];
    for (int q = 1; q < 16; ++q) {
        const float4 u = gsum[q][threadIdx.x];
        t4.x += u.x; t4.y += u.y; t4.z += u.z; t4.w += u.w;
    }
    const float sv[4] = {t4.x, t4.y, t4.z, t4.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int e = 4 * e4 + i;
        if (e < 27 * 256) {
            const int t = e >> 8, ci = cib * 16 + ((e >> 4) & 15), co = cob * 16 + (e & 15);
            if (ci < cin) grad_w[((int64_t)t * cin + ci) * cout + co] += scale * sv[i];
        } else if (cib == 0) {
            grad_b[cob * 16 + (e - 27 * 256)] += scale * sv[i];
        }
    }
}


// ---------------------------------------------------------------- elementwise pieces

// The level changes and the final layer work on 8 channels (16 bytes of BF16)
// per access; channel counts are multiples of 16.  (One channel per thread was
// bound by its 2-byte loads and index arithmetic: final layer 35 us, pools 21,
// their adjoints 79 and the up-sampling's 39 per 2^20 voxels.)
struct H8 { uint32_t w[4]; };   // 8 BF16 values
__device__ inline H8 h8_load(const uint16_t *p) { const uint4 v = *(const uint4 *)p; return H8{{v.x, v.y, v.z, v.w}}; }
__device__ inline float h8_get(const H8 &h, int i) { return bf2f((uint16_t)(h.w[i >> 1] >> (16 * (i & 1)))); }
__device__ inline void h8_store(uint16_t *p, const float *v)
{
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = (uint32_t)f2bf(v[2 * i]) | ((uint32_t)f2bf(v[2 * i + 1]) << 16);
    *(uint4 *)p = uint4{w[0], w[1], w[2], w[3]};
}
// 8 FP32 values
__device__ inline void f8_load(const float *p, float *v)
{
    const float4 a = ((const float4 *)p)[0], b = ((const float4 *)p)[1];
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
// thread -> 8 channels from c of voxel (i, j, k) of an nx x ny x .. level
struct Oct {
    int64_t v;
    int c, i, j, k;
    __device__ inline Oct(int64_t e, int nx, int ny, int C)
    {
        v = e / (C / 8);
        c = 8 * (int)(e - v * (C / 8));
        const int64_t row = v / nx;
        i = (int)(v - row * nx);
        k = (int)(row / ny);
        j = (int)(row - (int64_t)k * ny);
    }
};

__global__ void k_pool(int nx, int ny, int nz, int C, const uint16_t *__restrict__ x, uint16_t *__restrict__ y)
{
    const int mx = nx / 2, my = ny / 2;
    const int64_t n = (int64_t)mx * my * (nz / 2) * (C / 8);
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) {
        const Oct o(e, mx, my, C);
        H8 h[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int ii = 2 * o.i + (q & 1), jj = 2 * o.j + ((q >> 1) & 1), kk = 2 * o.k + (q >> 2);
            h[q] = h8_load(x + (ii + (int64_t)nx * (jj + (int64_t)ny * kk)) * C + o.c);
        }
        float s[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            float t = 0.f;
#pragma unroll
            for (int q = 0; q < 8; ++q) t += h8_get(h[q], c);
            s[c] = 0.125f * t;
        }
        h8_store(y + o.v * C + o.c, s);
    }
}

// The backward pass's gradients are masked by the ReLU of the layer they reach
// and rounded to BF16 by the kernel that forms them: G = bf16(g * [act > 0]).

// skip path + adjoint of the average pool (fine grid nx,ny,nz): g = gs + dy(parent) / 8
__global__ void k_pool_bwd(int nx, int ny, int nz, int C, const float *__restrict__ dy, const float *__restrict__ gs,
                           const uint16_t *__restrict__ act, uint16_t *__restrict__ G)
{
    const int mx = nx / 2, my = ny / 2;
    const int64_t n = (int64_t)nx * ny * nz * (C / 8);
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) {
        const Oct o(e, nx, ny, C);
        float g[8], d[8];
        f8_load(gs + o.v * C + o.c, g);
        f8_load(dy + ((o.i / 2) + (int64_t)mx * ((o.j / 2) + (int64_t)my * (o.k / 2))) * C + o.c, d);
        const H8 a = h8_load(act + o.v * C + o.c);
#pragma unroll
        for (int c = 0; c < 8; ++c) g[c] = h8_get(a, c) > 0.f ? g[c] + 0.125f * d[c] : 0.f;
        h8_store(G + o.v * C + o.c, g);
    }
}

// adjoint of nearest up-sampling (fine grid nx,ny,nz): g(parent) = sum of 8 children
__global__ void k_up_bwd(int nx, int ny, int nz, int C, const float *__restrict__ dyf, const uint16_t *__restrict__ act,
                         uint16_t *__restrict__ G)
{
    const int mx = nx / 2, my = ny / 2;
    const int64_t n = (int64_t)mx * my * (nz / 2) * (C / 8);
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) {
        const Oct o(e, mx, my, C);
        float d[8][8], s[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int ii = 2 * o.i + (q & 1), jj = 2 * o.j + ((q >> 1) & 1), kk = 2 * o.k + (q >> 2);
            f8_load(dyf + (ii + (int64_t)nx * (jj + (int64_t)ny * kk)) * C + o.c, d[q]);
        }
        const H8 a = h8_load(act + o.v * C + o.c);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            float t = 0.f;
#pragma unroll
            for (int q = 0; q < 8; ++q) t += d[q][c];
            s[c] = h8_get(a, c) > 0.f ? t : 0.f;
        }
        h8_store(G + o.v * C + o.c, s);
    }
}

// final 1x1x1 layer: y[v][co] = b[co] + sum_ci W[ci][co] d1[v][ci]
__global__ void k_final(int64_t V, int C, const uint16_t *__restrict__ d1, const float *__restrict__ W,
                        const float *__restrict__ b, float *__restrict__ y)
{
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < V; v += (int64_t)gridDim.x * 256) {
        float o[3] = {b[0], b[1], b[2]};
        for (int c8 = 0; c8 < C; c8 += 8) {
            const H8 h = h8_load(d1 + v * C + c8);
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int co = 0; co < 3; ++co) o[co] += W[(c8 + i) * 3 + co] * h8_get(h, i);
        }
        for (int co = 0; co < 3; ++co) y[v * 3 + co] = o[co];
    }
}

// Backward of the final layer: G[v][ci] = bf16((sum_co W[ci][co] gy[v][co]) *
// [d1 > 0]) and the partial weight and bias sums of the block's voxels,
// partials[block][ci * 3 + co] = sum_v d1[v][ci] gy[v][co], [3 C + co] =
// sum_v gy[v][co].  A thread keeps one channel (C divides the block), so d1 is
// read once, whole voxels at a time.
__global__ __launch_bounds__(256) void k_final_bwd(int64_t V, int C, const float *__restrict__ W,
                                                   const uint16_t *__restrict__ d1, const float *__restrict__ gy,
                                                   uint16_t *__restrict__ G, float *__restrict__ partials)
{
    __shared__ float red[6][256];
    const int ci = threadIdx.x % C, vg = threadIdx.x / C, nv = 256 / C;
    const float w0 = W[ci * 3], w1 = W[ci * 3 + 1], w2 = W[ci * 3 + 2];
    float s[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int64_t v = (int64_t)blockIdx.x * nv + vg; v < V; v += (int64_t)gridDim.x * nv) {
        const float a = bf2f(d1[v * C + ci]);
        const float g0 = gy[v * 3], g1 = gy[v * 3 + 1], g2 = gy[v * 3 + 2];
        const float g = w0 * g0 + w1 * g1 + w2 * g2;
        G[v * C + ci] = f2bf(a > 0.f ? g : 0.f);
        s[0] += a * g0; s[1] += a * g1; s[2] += a * g2;
        s[3] += g0; s[4] += g1; s[5] += g2;
    }
#pragma unroll
    for (int q = 0; q < 6; ++q) red[q][threadIdx.x] = s[q];
    __syncthreads();
    float *out = partials + (int64_t)blockIdx.x * (3 * C + 3);
    for (int q = threadIdx.x; q < 3 * C + 3; q += 256) {
        const int c = q < 3 * C ? q / 3 : 0, k = q < 3 * C ? q % 3 : 3 + q - 3 * C;
        float t = 0.f;
        for (int h = 0; h < nv; ++h) t += red[k][h * C + c];
        out[q] = t;
    }
}

// grad[q] += scale * (sum of partials[b][q] over the blocks), one workgroup per
// q: thread t adds blocks t, t + 256, ..., then a fixed tree over the threads
__global__ __launch_bounds__(256) void k_sum_blocks(const float *__restrict__ partials, int nb, int n, float scale,
                                                    float *__restrict__ grad)
{
    __shared__ float red[256];
    float s = 0.f;
    for (int b = threadIdx.x; b < nb; b += 256) s += partials[(int64_t)b * n + blockIdx.x];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) grad[blockIdx.x] += scale * red[0];
}

// Batched kernels: nb samples, sample b's residual at r + b 3V, its scalars
// s2[b] and so on.

// partials[block][b] = the block's part of sum r^2 of sample b = blockIdx.y
__global__ __launch_bounds__(256) void k_sumsq(int64_t n, const double *__restrict__ r, double *__restrict__ partials)
{
    __shared__ double lds[4];
    const double *x = r + (int64_t)blockIdx.y * n;
    double s = 0.0;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) s += x[e] * x[e];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) partials[(int64_t)blockIdx.x * gridDim.y + blockIdx.y] = lds[0] + lds[1] + lds[2] + lds[3];
}

// partials[block][b] = the block's part of sum ln k (sum == nullptr), or of
// sum (ln k - mean)^2 with mean = sum[b] / V, for sample b = blockIdx.y
__global__ __launch_bounds__(256) void k_lnk_sums(int64_t V, const float *__restrict__ lnk,
                                                  const double *__restrict__ sum, double *__restrict__ partials)
{
    __shared__ double lds[4];
    const float *x = lnk + (int64_t)blockIdx.y * V;
    const double m = sum ? sum[blockIdx.y] / (double)V : 0.0;
    double s = 0.0;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < V; e += (int64_t)gridDim.x * 256) {
        const double d = (double)x[e] - m;
        s += sum ? d * d : d;
    }
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) partials[(int64_t)blockIdx.x * gridDim.y + blockIdx.y] = lds[0] + lds[1] + lds[2] + lds[3];
}

// network input from a residual.  rtl: tile-lane FP64 vector (or NULL, one
// sample), rnat: natural block-row FP64 vectors (or NULL); s2[b] = sum r^2 over
// all entries.  x0[v][0..2] = r/s (s = rms), x0[v][3] = standardised ln k
// (precomputed).
__global__ void k_prep(Geo geo, int nb, const double *__restrict__ rtl, const double *__restrict__ rnat,
                       const double *__restrict__ s2, const uint16_t *__restrict__ lnk_std,
                       uint16_t *__restrict__ x0)
{
    const int64_t V = (int64_t)geo.nx * geo.ny * geo.nz;
    for (int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x; g < V * nb; g += (int64_t)gridDim.x * 256) {
        const int64_t b = g / V, v = g - b * V;
        const double s = sqrt(s2[b] / (double)(3 * V));
        const double inv = s > 0.0 ? 1.0 / s : 0.0;
        const int i = (int)(v % geo.nx), j = (int)((v / geo.nx) % geo.ny), k = (int)(v / ((int64_t)geo.nx * geo.ny));
        double r[3];
        if (rtl) {
            const int64_t sl = slot_of(geo, i, j, k);
            for (int p = 0; p < 3; ++p) r[p] = rtl[vidx(sl, p)];
        } else {
            const int64_t row = b * V + row_of(geo, i, j, k);
            for (int p = 0; p < 3; ++p) r[p] = rnat[3 * row + p];
        }
        for (int p = 0; p < 3; ++p) x0[g * 4 + p] = f2bf((float)(r[p] * inv));
        x0[g * 4 + 3] = lnk_std[g];
    }
}

// z = s * y (+ add, tile-lane, when given) back to a tile-lane (ztl) or natural (znat) FP64 vector
__global__ void k_post(Geo geo, const float *__restrict__ y, const double *__restrict__ s2, double *__restrict__ ztl,
                       double *__restrict__ znat, const double *__restrict__ add = nullptr)
{
    const int64_t V = (int64_t)geo.nx * geo.ny * geo.nz;
    const double s = sqrt(s2[0] / (double)(3 * V));
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < V; v += (int64_t)gridDim.x * 256) {
        const int i = (int)(v % geo.nx), j = (int)((v / geo.nx) % geo.ny), k = (int)(v / ((int64_t)geo.nx * geo.ny));
        if (ztl) {
            const int64_t sl = slot_of(geo, i, j, k);
            for (int p = 0; p < 3; ++p)
                ztl[vidx(sl, p)] = (add ? add[vidx(sl, p)] : 0.0) + s * (double)y[v * 3 + p];
        } else {
            const int64_t row = row_of(geo, i, j, k);
            for (int p = 0; p < 3; ++p) znat[3 * row + p] = s * (double)y[v * 3 + p];
        }
    }
}

// standardised ln k in voxel order, BF16; lnk given per block row, its sum and
// sum of squared deviations per sample
__global__ void k_lnk_std(Geo geo, int nb, const float *__restrict__ lnk, const double *__restrict__ sum,
                          const double *__restrict__ dev2, uint16_t *__restrict__ out)
{
    const int64_t V = (int64_t)geo.nx * geo.ny * geo.nz;
    for (int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x; g < V * nb; g += (int64_t)gridDim.x * 256) {
        const int64_t b = g / V, v = g - b * V;
        const double mean = sum[b] / (double)V, sd = sqrt(dev2[b] / (double)V);
        const double inv_sd = sd > 0.0 ? 1.0 / sd : 0.0;
        const int i = (int)(v % geo.nx), j = (int)((v / geo.nx) % geo.ny), k = (int)(v / ((int64_t)geo.nx * geo.ny));
        out[g] = f2bf((float)(((double)lnk[b * V + row_of(geo, i, j, k)] - mean) * inv_sd));
    }
}

// loss partials of sample b = blockIdx.y, partials[block][2 b ..]: sum (y - e/s)^2
// and sum (e/s)^2; e natural FP64
__global__ __launch_bounds__(256) void k_loss(Geo geo, const float *__restrict__ y, const double *__restrict__ e,
                                              const double *__restrict__ s2, double *__restrict__ partials)
{
    __shared__ double r0[256], r1[256];
    const int64_t V = (int64_t)geo.nx * geo.ny * geo.nz, vb = (int64_t)blockIdx.y * V;
    const double s = sqrt(s2[blockIdx.y] / (double)(3 * V));
    const double inv = s > 0.0 ? 1.0 / s : 0.0;
    double a = 0.0, b = 0.0;
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < V; v += (int64_t)gridDim.x * 256) {
        const int i = (int)(v % geo.nx), j = (int)((v / geo.nx) % geo.ny), k = (int)(v / ((int64_t)geo.nx * geo.ny));
        const int64_t row = vb + row_of(geo, i, j, k);
        for (int p = 0; p < 3; ++p) {
            const double t = e[3 * row + p] * inv;
            const double d = (double)y[(vb + v) * 3 + p] - t;
            a += d * d;
            b += t * t;
        }
    }
    r0[threadIdx.x] = a;
    r1[threadIdx.x] = b;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) { r0[threadIdx.x] += r0[threadIdx.x + w]; r1[threadIdx.x] += r1[threadIdx.x + w]; }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        double *out = partials + 2 * ((int64_t)blockIdx.x * gridDim.y + blockIdx.y);
        out[0] = r0[0];
        out[1] = r1[0];
    }
}

// gy = scale * 2 (y - e/s) / ||e/s||^2   (loss[2 b + 1] = ||e/s||^2 of sample b)
__global__ void k_gy(Geo geo, int nb, const float *__restrict__ y, const double *__restrict__ e,
                     const double *__restrict__ s2, const double *__restrict__ loss, float scale,
                     float *__restrict__ gy)
{
    const int64_t V = (int64_t)geo.nx * geo.ny * geo.nz;
    for (int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x; g < V * nb; g += (int64_t)gridDim.x * 256) {
        const int64_t b = g / V, v = g - b * V;
        const double s = sqrt(s2[b] / (double)(3 * V));
        const double inv = s > 0.0 ? 1.0 / s : 0.0;
        const double f = 2.0 * (double)scale / loss[2 * b + 1];
        const int i = (int)(v % geo.nx), j = (int)((v / geo.nx) % geo.ny), k = (int)(v / ((int64_t)geo.nx * geo.ny));
        const int64_t row = b * V + row_of(geo, i, j, k);
        for (int p = 0; p < 3; ++p) gy[g * 3 + p] = (float)(f * ((double)y[g * 3 + p] - e[3 * row + p] * inv));
    }
}

__global__ void k_adam(int64_t n, float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, float lr, float c1, float c2)
{
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) {
        const float mm = 0.9f * m[e] + 0.1f * g[e];
        const float vv = 0.999f * v[e] + 0.001f * g[e] * g[e];
        m[e] = mm;
        v[e] = vv;
        p[e] -= lr * (mm / c1) / (sqrtf(vv / c2) + 1e-8f);
    }
}

// pack W[tap][ci][co] (FP32) into B fragments of kw k per block (kw / 4 per
// lane): forward (k = tap*cin + ci, n = co) or transposed for the data
// gradient (k = tap'*cout + co with tap' = 26 - tap, n = ci)
__global__ void k_pack(const float *__restrict__ W, int cin, int cout, int transposed, int KB, int NB, int kw,
                       short *__restrict__ Wf)
{
    const int64_t n = (int64_t)KB * NB * 64;
    const int w = kw / 4;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) {
        const int lane = (int)(e % 64);
        const int nb = (int)((e / 64) % NB);
        const int kb = (int)(e / (64 * NB));
        const int col = nb * 16 + (lane & 15);
        for (int i = 0; i < w; ++i) {
            const int k = kb * kw + w * (lane >> 4) + i;
            float wv = 0.f;
            if (!transposed) {
                if (k < 27 * cin && col < cout) wv = W[(int64_t)k * cout + col];   // k = tap*cin + ci
            } else {
                if (k < 27 * cout && col < cin) {
                    const int tp = k / cout, co = k - tp * cout;
                    wv = W[((int64_t)(26 - tp) * cin + col) * cout + co];
                }
            }
            Wf[e * w + i] = (short)f2bf(wv);
        }
    }
}

// seeded He-uniform initialisation (SplitMix64 counter hash), biases zero
__global__ void k_init(int64_t n, float *__restrict__ p, const int64_t *__restrict__ seg, int nseg, uint64_t seed)
{
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) {
        // seg: [woff, boff, fan_in, scale*1e6] per layer
        float val = 0.f;
        for (int l = 0; l < nseg; ++l) {
            const int64_t wo = seg[4 * l], bo = seg[4 * l + 1];
            if (e >= wo && e < bo) {
                uint64_t z = seed + (uint64_t)(e + 1) * 0x9E3779B97F4A7C15ull;
                z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
                z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
                z ^= z >> 31;
                const double u = (double)(z >> 11) * 0x1.0p-53;
                const double a = sqrt(6.0 / (double)seg[4 * l + 2]) * (double)seg[4 * l + 3] * 1e-6;
                val = (float)((2.0 * u - 1.0) * a);
            }
        }
        p[e] = val;
    }
}

inline int nblk(int64_t n) { return (int)std::min<int64_t>(std::max<int64_t>((n + 255) / 256, 1), 4096); }

}  // namespace

// ---------------------------------------------------------------- the network object

struct rsv_net {
    rsv_ctx *c = nullptr;
    Arch a;
    int64_t step = 0;
    float *P = nullptr, *G = nullptr, *M = nullptr, *Vv = nullptr;   // FP32 master, gradient, Adam moments
    v4s *wf[10] = {nullptr}, *wt[10] = {nullptr};                    // packed BF16 weights
    bool packed = false;
    // workspace for up to `wb` samples of one grid
    int wx = 0, wy = 0, wz = 0, wb = 0;
    uint16_t *x0 = nullptr, *a1 = nullptr, *s1 = nullptr, *p1 = nullptr, *a2 = nullptr, *s2 = nullptr, *p2 = nullptr,
             *a3 = nullptr, *b3 = nullptr, *d2a = nullptr, *d2 = nullptr, *d1a = nullptr, *d1 = nullptr;
    uint16_t *lnk_std = nullptr;
    float *y = nullptr;
    // backward pass: BF16 gradients of the layer at hand and the next, FP32 ones that a pool
    // or an up-sampling sums, and the skip paths'
    bool wback = false;
    uint16_t *Ga = nullptr, *Gb = nullptr;
    float *gy = nullptr, *g1 = nullptr, *gs1 = nullptr, *gs2 = nullptr, *part = nullptr;
    // per sample: sum r^2 [wb]; sum ln k [wb]; sum (ln k - mean)^2 [wb]; loss sums [wb][2]
    double *d_sc = nullptr;
    int64_t part_cap = 0;
    double *sum_r2() const { return d_sc; }
    double *sum_lnk() const { return d_sc + wb; }
    double *dev_lnk() const { return d_sc + 2 * wb; }
    double *loss() const { return d_sc + 3 * wb; }

    ~rsv_net() { release(); }
    void free_ws()
    {
        void *ps[] = {x0, a1, s1, p1, a2, s2, p2, a3, b3, d2a, d2, d1a, d1, Ga, Gb, lnk_std, y, gy, g1, gs1, gs2, part, d_sc};
        for (void *p : ps) dev_free(p);
        x0 = a1 = s1 = p1 = a2 = s2 = p2 = a3 = b3 = d2a = d2 = d1a = d1 = Ga = Gb = lnk_std = nullptr;
        y = gy = g1 = gs1 = gs2 = part = nullptr;
        d_sc = nullptr;
        part_cap = 0;
        wx = wy = wz = wb = 0;
        wback = false;
    }
    void release()
    {
        free_ws();
        dev_free(P); dev_free(G); dev_free(M); dev_free(Vv);
        for (int l = 0; l < 10; ++l) { dev_free(wf[l]); dev_free(wt[l]); }
    }
};

static rsv_status net_pack(rsv_net *n)
{
    rsv_ctx *c = n->c;
    for (int l = 0; l < 10; ++l) {
        const int NB = n->a.cout[l] / 16, NBt = (n->a.cin[l] + 15) / 16;
        hipLaunchKernelGGL(k_pack, dim3(nblk((int64_t)n->a.kb(l) * NB * 64)), dim3(256), 0, c->stream, n->P + n->a.woff[l],
                           n->a.cin[l], n->a.cout[l], 0, n->a.kb(l), NB, conv_kw(n->a.cin[l]), (short *)n->wf[l]);
        if (l > 0)
            hipLaunchKernelGGL(k_pack, dim3(nblk((int64_t)n->a.kbt(l) * NBt * 64)), dim3(256), 0, c->stream,
                               n->P + n->a.woff[l], n->a.cin[l], n->a.cout[l], 1, n->a.kbt(l), NBt, conv_kw(n->a.cout[l]),
                               (short *)n->wt[l]);
    }
    RSV_LAUNCH(c);
    n->packed = true;
    return RSV_OK;
}

// Workspace for nb samples of a grid, with the backward pass's when `back`;
// kept while it is large enough.
static rsv_status net_ws(rsv_net *n, int nx, int ny, int nz, int nb, bool back)
{
    const bool same = n->wx == nx && n->wy == ny && n->wz == nz;
    if (same && n->wb >= nb && (n->wback || !back)) return RSV_OK;
    rsv_ctx *c = n->c;
    RSV_HIP(c, hipStreamSynchronize(c->stream));
    if (same) {
        nb = std::max(nb, n->wb);
        back = back || n->wback;
    }
    n->free_ws();
    const int64_t V1 = (int64_t)nx * ny * nz * nb, V2 = V1 / 8, V3 = V2 / 8;
    const int c0 = n->a.c[0], c1 = n->a.c[1], c2 = n->a.c[2];
    // masked gradients: each level's own channels
    const int64_t gmask = std::max(V1 * c0, std::max(V2 * c1, V3 * c2));
    // unmasked ones: the up-sampled inputs of the decoder levels (full resolution with c1
    // channels, half with c2) and the pooled ones (half with c0, quarter with c1)
    const int64_t gfull = std::max(std::max(V1 * c1, V2 * c2), std::max(V2 * c0, V3 * c1));
    struct { void **p; size_t b; bool back; } L[] = {
        {(void **)&n->x0, (size_t)V1 * 4 * 2, false}, {(void **)&n->a1, (size_t)V1 * c0 * 2, false},
        {(void **)&n->s1, (size_t)V1 * c0 * 2, false}, {(void **)&n->p1, (size_t)V2 * c0 * 2, false},
        {(void **)&n->a2, (size_t)V2 * c1 * 2, false}, {(void **)&n->s2, (size_t)V2 * c1 * 2, false},
        {(void **)&n->p2, (size_t)V3 * c1 * 2, false}, {(void **)&n->a3, (size_t)V3 * c2 * 2, false},
        {(void **)&n->b3, (size_t)V3 * c2 * 2, false}, {(void **)&n->d2a, (size_t)V2 * c1 * 2, false},
        {(void **)&n->d2, (size_t)V2 * c1 * 2, false}, {(void **)&n->d1a, (size_t)V1 * c0 * 2, false},
        {(void **)&n->d1, (size_t)V1 * c0 * 2, false}, {(void **)&n->lnk_std, (size_t)V1 * 2, false},
        {(void **)&n->y, (size_t)V1 * 3 * 4, false}, {(void **)&n->d_sc, (size_t)nb * 5 * sizeof(double), false},
        {(void **)&n->Ga, (size_t)gmask * 2, true}, {(void **)&n->Gb, (size_t)gmask * 2, true},
        {(void **)&n->gy, (size_t)V1 * 3 * 4, true}, {(void **)&n->g1, (size_t)gfull * 4, true},
        {(void **)&n->gs1, (size_t)V1 * c0 * 4, true}, {(void **)&n->gs2, (size_t)V2 * c1 * 4, true},
    };
    for (auto &e : L) {
        if (e.back && !back) continue;
        rsv_status s = dev_alloc(c, e.p, e.b);
        if (s != RSV_OK) { n->free_ws(); return s; }
    }
    n->wx = nx; n->wy = ny; n->wz = nz; n->wb = nb;
    n->wback = back;
    return RSV_OK;
}

static rsv_status part_reserve(rsv_net *n, int64_t nfloat)
{
    if (nfloat <= n->part_cap) return RSV_OK;
    RSV_HIP(n->c, hipStreamSynchronize(n->c->stream));
    dev_free(n->part);
    n->part = nullptr;
    rsv_status s = dev_alloc(n->c, (void **)&n->part, (size_t)nfloat * sizeof(float));
    if (s == RSV_OK) n->part_cap = nfloat;
    return s;
}

// relu(conv(X) + b [+ skip]), BF16; nz layers in all, nzs per sample
static rsv_status conv_fwd(rsv_net *n, int l, int nx, int ny, int nz, int nzs, int up, const uint16_t *X,
                           const uint16_t *skip, uint16_t *out)
{
    rsv_ctx *c = n->c;
    ConvGeo g{nx, ny, nz, nzs, up, n->a.cin[l], n->a.cout[l], (int64_t)nx * ny * nz};
    const Epilogue ep{n->P + n->a.boff[l], skip, 1, nullptr, nullptr, out};
    const hipError_t e = launch_conv<true>(c, g, X, n->wf[l], n->a.kb(l), ep);
    if (e != hipSuccess) return set_err(c, RSV_ERR_HIP, std::string("conv launch: ") + hipGetErrorString(e));
    return RSV_OK;
}

// dX (resolution of G) = transposed conv of the BF16 gradient G: FP32 into dX32,
// or masked by the activations `mask` and BF16 into dX16 (FP32 copy of that in `copy`)
static rsv_status conv_bwd_data(rsv_net *n, int l, int nx, int ny, int nz, int nzs, const uint16_t *G, float *dX32,
                                const uint16_t *mask, uint16_t *dX16, float *copy)
{
    rsv_ctx *c = n->c;
    ConvGeo g{nx, ny, nz, nzs, 0, n->a.cout[l], n->a.cin[l], (int64_t)nx * ny * nz};
    if (g.cout % 16) return set_err(c, RSV_ERR_ARG, "channel count must be 16, 32 or 64");
    const Epilogue ep{nullptr, nullptr, 0, mask, copy, mask ? (void *)dX16 : (void *)dX32};
    const hipError_t e = mask ? launch_conv<true>(c, g, G, n->wt[l], n->a.kbt(l), ep)
                              : launch_conv<false>(c, g, G, n->wt[l], n->a.kbt(l), ep);
    if (e != hipSuccess) return set_err(c, RSV_ERR_HIP, std::string("conv launch: ") + hipGetErrorString(e));
    return RSV_OK;
}

// grad(W_l) += scale * X^T G, grad(b_l) += scale * colsum(G)
static rsv_status conv_bwd_weight(rsv_net *n, int l, int nx, int ny, int nz, int nzs, int up, const uint16_t *X,
                                  const uint16_t *G, float scale, float *grad_w, float *grad_b)
{
    rsv_ctx *c = n->c;
    ConvGeo g{nx, ny, nz, nzs, up, n->a.cin[l], n->a.cout[l], (int64_t)nx * ny * nz};
    if (g.cout % 16 || g.cin > 64) return set_err(c, RSV_ERR_ARG, "channel count must be 16, 32 or 64");
    const int npairs = ((g.cin + 15) / 16) * (g.cout / 16);
    const int64_t nbricks = brick_count(g, CT_Z);
    // about DW_WGS workgroups (two per CU) of at least two bricks
    const int64_t want = std::max<int64_t>(1, std::min<int64_t>((nbricks + 1) / 2, std::max(1, DW_WGS / npairs)));
    const int per = (int)((nbricks + want - 1) / want);
    const int nchunks = (int)((nbricks + per - 1) / per);
    rsv_status s = part_reserve(n, (int64_t)nchunks * npairs * DW_PART);
    if (s != RSV_OK) return s;
    hipLaunchKernelGGL(k_conv_dw, dim3(nchunks * npairs), dim3(256), 0, c->stream, g, X, G, npairs, per, n->part);
    constexpr int slices = (DW_PART / 4 + 15) / 16;
    hipLaunchKernelGGL(k_dw_reduce, dim3(npairs * slices), dim3(256), 0, c->stream, (const float *)n->part, npairs, nchunks,
                       g.cin, g.cout, scale, grad_w, grad_b);
    RSV_LAUNCH(c);
    return RSV_OK;
}

// forward pass of nb samples; x0 must be filled; result y (FP32 [nb][V][3])
static rsv_status net_forward(rsv_net *n, int nx, int ny, int nzs, int nb)
{
    if (!n->packed) {
        rsv_status s = net_pack(n);
        if (s != RSV_OK) return s;
    }
    const int nz = nzs * nb;
    const int mx = nx / 2, my = ny / 2, mz = nz / 2, ms = nzs / 2, lx = nx / 4, ly = ny / 4, lz = nz / 4, ls = nzs / 4;
    const int c0 = n->a.c[0], c1 = n->a.c[1];
    rsv_ctx *c = n->c;
    ProfScope ps(c, RSV_K_NET);
    rsv_status s;
    if ((s = conv_fwd(n, 0, nx, ny, nz, nzs, 0, n->x0, nullptr, n->a1)) != RSV_OK) return s;
    if ((s = conv_fwd(n, 1, nx, ny, nz, nzs, 0, n->a1, nullptr, n->s1)) != RSV_OK) return s;
    hipLaunchKernelGGL(k_pool, dim3(nblk((int64_t)mx * my * mz * c0 / 8)), dim3(256), 0, c->stream, nx, ny, nz, c0, n->s1, n->p1);
    if ((s = conv_fwd(n, 2, mx, my, mz, ms, 0, n->p1, nullptr, n->a2)) != RSV_OK) return s;
    if ((s = conv_fwd(n, 3, mx, my, mz, ms, 0, n->a2, nullptr, n->s2)) != RSV_OK) return s;
    hipLaunchKernelGGL(k_pool, dim3(nblk((int64_t)lx * ly * lz * c1 / 8)), dim3(256), 0, c->stream, mx, my, mz, c1, n->s2, n->p2);
    if ((s = conv_fwd(n, 4, lx, ly, lz, ls, 0, n->p2, nullptr, n->a3)) != RSV_OK) return s;
    if ((s = conv_fwd(n, 5, lx, ly, lz, ls, 0, n->a3, nullptr, n->b3)) != RSV_OK) return s;
    if ((s = conv_fwd(n, 6, mx, my, mz, ms, 1, n->b3, n->s2, n->d2a)) != RSV_OK) return s;
    if ((s = conv_fwd(n, 7, mx, my, mz, ms, 0, n->d2a, nullptr, n->d2)) != RSV_OK) return s;
    if ((s = conv_fwd(n, 8, nx, ny, nz, nzs, 1, n->d2, n->s1, n->d1a)) != RSV_OK) return s;
    if ((s = conv_fwd(n, 9, nx, ny, nz, nzs, 0, n->d1a, nullptr, n->d1)) != RSV_OK) return s;
    const int64_t V1 = (int64_t)nx * ny * nz;
    hipLaunchKernelGGL(k_final, dim3(nblk(V1)), dim3(256), 0, c->stream, V1, c0, n->d1, n->P + n->a.woff[10],
                       n->P + n->a.boff[10], n->y);
    RSV_LAUNCH(c);
    return RSV_OK;
}

// backward pass of nb samples for n->gy, adding to the gradient n->G
static rsv_status net_backward(rsv_net *n, int nx, int ny, int nzs, int nb)
{
    rsv_ctx *c = n->c;
    ProfScope ps(c, RSV_K_NET);
    const int nz = nzs * nb;
    const int mx = nx / 2, my = ny / 2, mz = nz / 2, ms = nzs / 2, lx = nx / 4, ly = ny / 4, lz = nz / 4, ls = nzs / 4;
    const int c0 = n->a.c[0], c1 = n->a.c[1], c2 = n->a.c[2];
    const int64_t V1 = (int64_t)nx * ny * nz, V2 = V1 / 8, V3 = V2 / 8;
    float *gw = n->G;
    rsv_status s;
    {
        const int nwf = c0 * 3 + 3;
        const int nbl = (int)std::max<int64_t>(1, std::min<int64_t>(V1 * c0 / 4096, 1024));
        if ((s = part_reserve(n, (int64_t)nbl * nwf)) != RSV_OK) return s;
        hipLaunchKernelGGL(k_final_bwd, dim3(nbl), dim3(256), 0, c->stream, V1, c0, (const float *)(n->P + n->a.woff[10]),
                           (const uint16_t *)n->d1, (const float *)n->gy, n->Ga, n->part);
        hipLaunchKernelGGL(k_sum_blocks, dim3(nwf), dim3(256), 0, c->stream, (const float *)n->part, nbl, nwf, 1.0f,
                           gw + n->a.woff[10]);
        RSV_LAUNCH(c);
    }
    // layer l at lx x ly x lz (ls layers per sample) with input X and masked output gradient G:
    // weight gradients, then the data gradient, masked by `act` into `next` or FP32 into n->g1
    auto layer = [&](int l, int x, int y, int z, int zs, int up, const uint16_t *X, const uint16_t *G,
                     const uint16_t *act, uint16_t *next, float *gskip) -> rsv_status {
        rsv_status st = conv_bwd_weight(n, l, x, y, z, zs, up, X, G, 1.0f, gw + n->a.woff[l], gw + n->a.boff[l]);
        if (st == RSV_OK && l > 0) st = conv_bwd_data(n, l, x, y, z, zs, G, n->g1, act, next, gskip);
        return st;
    };
    // dec1b, then dec1a: out d1a = relu(conv8(up(d2)) + s1), skip gradient -> gs1
    if ((s = layer(9, nx, ny, nz, nzs, 0, n->d1a, n->Ga, n->d1a, n->Gb, n->gs1)) != RSV_OK) return s;
    if ((s = layer(8, nx, ny, nz, nzs, 1, n->d2, n->Gb, nullptr, nullptr, nullptr)) != RSV_OK) return s;
    hipLaunchKernelGGL(k_up_bwd, dim3(nblk(V2 * c1 / 8)), dim3(256), 0, c->stream, nx, ny, nz, c1, (const float *)n->g1,
                       (const uint16_t *)n->d2, n->Ga);
    // dec2b, dec2a: skip gradient -> gs2
    if ((s = layer(7, mx, my, mz, ms, 0, n->d2a, n->Ga, n->d2a, n->Gb, n->gs2)) != RSV_OK) return s;
    if ((s = layer(6, mx, my, mz, ms, 1, n->b3, n->Gb, nullptr, nullptr, nullptr)) != RSV_OK) return s;
    hipLaunchKernelGGL(k_up_bwd, dim3(nblk(V3 * c2 / 8)), dim3(256), 0, c->stream, mx, my, mz, c2, (const float *)n->g1,
                       (const uint16_t *)n->b3, n->Ga);
    // enc3b, enc3a
    if ((s = layer(5, lx, ly, lz, ls, 0, n->a3, n->Ga, n->a3, n->Gb, nullptr)) != RSV_OK) return s;
    if ((s = layer(4, lx, ly, lz, ls, 0, n->p2, n->Gb, nullptr, nullptr, nullptr)) != RSV_OK) return s;
    hipLaunchKernelGGL(k_pool_bwd, dim3(nblk(V2 * c1 / 8)), dim3(256), 0, c->stream, mx, my, mz, c1, (const float *)n->g1,
                       (const float *)n->gs2, (const uint16_t *)n->s2, n->Ga);
    // enc2b, enc2a
    if ((s = layer(3, mx, my, mz, ms, 0, n->a2, n->Ga, n->a2, n->Gb, nullptr)) != RSV_OK) return s;
    if ((s = layer(2, mx, my, mz, ms, 0, n->p1, n->Gb, nullptr, nullptr, nullptr)) != RSV_OK) return s;
    hipLaunchKernelGGL(k_pool_bwd, dim3(nblk(V1 * c0 / 8)), dim3(256), 0, c->stream, nx, ny, nz, c0, (const float *)n->g1,
                       (const float *)n->gs1, (const uint16_t *)n->s1, n->Ga);
    // enc1b, enc1a
    if ((s = layer(1, nx, ny, nz, nzs, 0, n->a1, n->Ga, n->a1, n->Gb, nullptr)) != RSV_OK) return s;
    if ((s = layer(0, nx, ny, nz, nzs, 0, n->x0, n->Gb, nullptr, nullptr, nullptr)) != RSV_OK) return s;
    RSV_LAUNCH(c);
    return RSV_OK;
}

static rsv_status dims_check(rsv_ctx *c, const rsv_grid *g)
{
    if (g->geo.nx % 4 || g->geo.ny % 4 || g->geo.nz % 4)
        return set_err(c, RSV_ERR_ARG, "learned preconditioner needs grid dimensions that are multiples of 4");
    return RSV_OK;
}

// blocks of a batched reduction: as many as launch_dot takes for one sample
static int red_blocks(int64_t len) { return vec_blocks(len); }

// standardised ln k channel (mean and standard deviation over each sample's
// grid, FP64) of nb samples into out[nb][V]; sums: 2 nb doubles of scratch
static rsv_status set_lnk(rsv_net *n, const rsv_grid *g, int nb, const float *lnk_dev, double *sum, double *dev2,
                          uint16_t *out)
{
    rsv_ctx *c = n->c;
    const int64_t V = g->ncell;
    const int nbl = red_blocks(V);
    rsv_status s = partials_reserve(c, (int64_t)nbl * nb);
    if (s != RSV_OK) return s;
    hipLaunchKernelGGL(k_lnk_sums, dim3(nbl, nb), dim3(256), 0, c->stream, V, lnk_dev, (const double *)nullptr, c->d_partials);
    if ((s = launch_reduce_to(c, nbl, nb, sum)) != RSV_OK) return s;
    hipLaunchKernelGGL(k_lnk_sums, dim3(nbl, nb), dim3(256), 0, c->stream, V, lnk_dev, (const double *)sum, c->d_partials);
    if ((s = launch_reduce_to(c, nbl, nb, dev2)) != RSV_OK) return s;
    hipLaunchKernelGGL(k_lnk_std, dim3(nblk(V * nb)), dim3(256), 0, c->stream, g->geo, nb, lnk_dev, (const double *)sum,
                       (const double *)dev2, out);
    RSV_LAUNCH(c);
    return RSV_OK;
}

// Fills x0 of nb samples from r (tile-lane rtl, one sample, or natural rnat)
// and leaves their sums of r^2 in n->sum_r2()
static rsv_status prep(rsv_net *n, const rsv_grid *g, int nb, const double *rtl, const double *rnat,
                       const uint16_t *lnk_std)
{
    rsv_ctx *c = n->c;
    const int64_t len = rtl ? g->nv : 3 * g->ncell;
    const int nbl = red_blocks(len);
    rsv_status s = partials_reserve(c, (int64_t)nbl * nb);
    if (s != RSV_OK) return s;
    hipLaunchKernelGGL(k_sumsq, dim3(nbl, nb), dim3(256), 0, c->stream, len, rtl ? rtl : rnat, c->d_partials);
    if ((s = launch_reduce_to(c, nbl, nb, n->sum_r2())) != RSV_OK) return s;
    hipLaunchKernelGGL(k_prep, dim3(nblk(g->ncell * nb)), dim3(256), 0, c->stream, g->geo, nb, rtl, rnat,
                       (const double *)n->sum_r2(), lnk_std, n->x0);
    RSV_LAUNCH(c);
    return RSV_OK;
}

struct Learned : PcImpl {
    rsv_matrix *M = nullptr;
    rsv_net *net = nullptr;
    uint16_t *lnk_std = nullptr;   // this preconditioner's standardised ln k channel
    PcImpl *base = nullptr;        // mode 1: the BILU0 step the network corrects
    double *t1 = nullptr, *r1 = nullptr;   // mode 1: BILU0^-1 r and r - A t1 (tile-lane)
    ~Learned() override
    {
        dev_free(lnk_std);
        dev_free(t1);
        dev_free(r1);
    }
    int64_t bytes() const override { return M->g->ncell * 2 + (base ? 2 * M->g->nv * (int64_t)sizeof(double) : 0); }
    rsv_status apply(const double *r, double *z) override
    {
        rsv_grid *g = M->g;
        rsv_ctx *c = net->c;
        rsv_status s = net_ws(net, g->geo.nx, g->geo.ny, g->geo.nz, 1, false);
        const double *in = r;
        if (s == RSV_OK && base) {
            s = base->apply(r, t1);
            if (s == RSV_OK) s = launch_spmv(c, g->geo, M->d_A, SPMV_RESID, t1, r1, r, 0.0, 0.0, SC_MISC);
            in = r1;
        }
        if (s == RSV_OK) s = prep(net, g, 1, in, nullptr, lnk_std);
        if (s == RSV_OK) s = net_forward(net, g->geo.nx, g->geo.ny, g->geo.nz, 1);
        if (s != RSV_OK) return s;
        hipLaunchKernelGGL(k_post, dim3(nblk(g->ncell)), dim3(256), 0, c->stream, g->geo, (const float *)net->y,
                           (const double *)net->sum_r2(), z, (double *)nullptr, (const double *)(base ? t1 : nullptr));
        RSV_LAUNCH(c);
        return RSV_OK;
    }
};

rsv_status learned_create(rsv_matrix *A, const rsv_pc_params *p, PcImpl **out, PcImpl *base)
{
    rsv_ctx *c = A->g->ctx;
    if (!p->net || !p->lnk) return set_err(c, RSV_ERR_ARG, "learned preconditioner needs net and lnk");
    rsv_status s = dims_check(c, A->g);
    if (s != RSV_OK) return s;
    rsv_net *n = p->net;
    if (n->c != c) return set_err(c, RSV_ERR_ARG, "network belongs to another context");
    Learned *L = new (std::nothrow) Learned();
    if (!L) return set_err(c, RSV_ERR_OOM, "learned");
    L->M = A;
    L->net = n;
    s = dev_alloc(c, (void **)&L->lnk_std, (size_t)A->g->ncell * 2);
    if (s == RSV_OK) s = net_ws(n, A->g->geo.nx, A->g->geo.ny, A->g->geo.nz, 1, false);
    if (s == RSV_OK) s = set_lnk(n, A->g, 1, p->lnk, n->sum_lnk(), n->dev_lnk(), L->lnk_std);
    if (s == RSV_OK && p->learned_mode == 1) {
        if (!base) s = set_err(c, RSV_ERR_ARG, "learned mode 1 needs the BILU0 base");
        L->base = base;
        if (s == RSV_OK) s = dev_alloc(c, (void **)&L->t1, (size_t)A->g->nv * sizeof(double));
        if (s == RSV_OK) s = dev_alloc(c, (void **)&L->r1, (size_t)A->g->nv * sizeof(double));
        // phantom slots of the tile-lane vectors stay zero
        if (s == RSV_OK && (hipMemsetAsync(L->t1, 0, (size_t)A->g->nv * sizeof(double), c->stream) != hipSuccess ||
                            hipMemsetAsync(L->r1, 0, (size_t)A->g->nv * sizeof(double), c->stream) != hipSuccess))
            s = set_err(c, RSV_ERR_HIP, "hipMemsetAsync");
    } else if (s == RSV_OK && p->learned_mode != 0) {
        s = set_err(c, RSV_ERR_ARG, "learned_mode must be 0 or 1");
    }
    if (s != RSV_OK) { delete L; return s; }
    *out = L;
    return RSV_OK;
}

extern "C" {

rsv_status rsv_net_create(rsv_ctx *c, const rsv_net_arch *arch, uint64_t seed, rsv_net **out)
{
    if (!c || !arch || !out) return set_err(c, RSV_ERR_ARG, "NULL argument");
    *out = nullptr;
    if (arch->levels != 3) return set_err(c, RSV_ERR_ARG, "only 3-level networks are supported");
    for (int q : {arch->c0, arch->c1, arch->c2})
        if (q != 16 && q != 32 && q != 64) return set_err(c, RSV_ERR_ARG, "channel counts must be 16, 32 or 64");
    rsv_net *n = new (std::nothrow) rsv_net();
    if (!n) return set_err(c, RSV_ERR_OOM, "net");
    n->c = c;
    n->a.init(arch->c0, arch->c1, arch->c2);
    const size_t pb = (size_t)n->a.np * sizeof(float);
    rsv_status s = dev_alloc(c, (void **)&n->P, pb);
    if (s == RSV_OK) s = dev_alloc(c, (void **)&n->G, pb);
    if (s == RSV_OK) s = dev_alloc(c, (void **)&n->M, pb);
    if (s == RSV_OK) s = dev_alloc(c, (void **)&n->Vv, pb);
    for (int l = 0; l < 10 && s == RSV_OK; ++l) {
        s = dev_alloc(c, (void **)&n->wf[l], (size_t)n->a.kb(l) * (n->a.cout[l] / 16) * 64 * conv_frag_bytes(n->a.cin[l]));
        if (s == RSV_OK)
            s = dev_alloc(c, (void **)&n->wt[l],
                          (size_t)n->a.kbt(l) * ((n->a.cin[l] + 15) / 16) * 64 * conv_frag_bytes(n->a.cout[l]));
    }
    if (s != RSV_OK) { delete n; return s; }
    // He-uniform init; the final layer is scaled by 0.1 so an untrained net starts small
    std::vector<int64_t> seg(4 * NL);
    for (int l = 0; l < NL; ++l) {
        seg[4 * l] = n->a.woff[l];
        seg[4 * l + 1] = n->a.boff[l];
        seg[4 * l + 2] = (int64_t)(l < 10 ? 27 : 1) * n->a.cin[l];
        seg[4 * l + 3] = l < 10 ? 1000000 : 100000;
    }
    int64_t *dseg = nullptr;
    s = dev_alloc(c, (void **)&dseg, seg.size() * sizeof(int64_t));
    if (s == RSV_OK && hipMemcpy(dseg, seg.data(), seg.size() * sizeof(int64_t), hipMemcpyHostToDevice) != hipSuccess)
        s = set_err(c, RSV_ERR_HIP, "hipMemcpy");
    if (s == RSV_OK) {
        hipLaunchKernelGGL(k_init, dim3(nblk(n->a.np)), dim3(256), 0, c->stream, n->a.np, n->P, (const int64_t *)dseg, NL,
                           seed * 0xD1B54A32D192ED03ull + 0x632BE59BD9B4E019ull);
        if (hipMemsetAsync(n->M, 0, pb, c->stream) != hipSuccess || hipMemsetAsync(n->Vv, 0, pb, c->stream) != hipSuccess)
            s = set_err(c, RSV_ERR_HIP, "hipMemsetAsync");
        if (hipStreamSynchronize(c->stream) != hipSuccess) s = set_err(c, RSV_ERR_HIP, "sync");
    }
    dev_free(dseg);
    if (s == RSV_OK) s = net_pack(n);
    if (s != RSV_OK) { delete n; return s; }
    *out = n;
    return RSV_OK;
}

void rsv_net_destroy(rsv_net *n)
{
    if (!n) return;
    (void)hipStreamSynchronize(n->c->stream);
    delete n;
}

int64_t rsv_net_num_params(const rsv_net *n) { return n ? n->a.np : 0; }

rsv_status rsv_net_get_params(rsv_net *n, float *h, int64_t cnt)
{
    if (!n || !h || cnt != n->a.np) return set_err(n ? n->c : nullptr, RSV_ERR_ARG, "bad parameter buffer");
    RSV_HIP(n->c, hipMemcpyAsync(h, n->P, cnt * sizeof(float), hipMemcpyDeviceToHost, n->c->stream));
    RSV_HIP(n->c, hipStreamSynchronize(n->c->stream));
    return RSV_OK;
}

rsv_status rsv_net_set_params(rsv_net *n, const float *h, int64_t cnt)
{
    if (!n || !h || cnt != n->a.np) return set_err(n ? n->c : nullptr, RSV_ERR_ARG, "bad parameter buffer");
    RSV_HIP(n->c, hipMemcpyAsync(n->P, h, cnt * sizeof(float), hipMemcpyHostToDevice, n->c->stream));
    RSV_HIP(n->c, hipMemsetAsync(n->M, 0, cnt * sizeof(float), n->c->stream));
    RSV_HIP(n->c, hipMemsetAsync(n->Vv, 0, cnt * sizeof(float), n->c->stream));
    n->step = 0;
    rsv_status s = net_pack(n);
    if (s != RSV_OK) return s;
    RSV_HIP(n->c, hipStreamSynchronize(n->c->stream));
    return RSV_OK;
}

rsv_status rsv_net_save(rsv_net *n, const char *path)
{
    if (!n || !path) return set_err(n ? n->c : nullptr, RSV_ERR_ARG, "NULL argument");
    std::vector<float> h(n->a.np);
    rsv_status s = rsv_net_get_params(n, h.data(), n->a.np);
    if (s != RSV_OK) return s;
    FILE *f = fopen(path, "wb");
    if (!f) return set_err(n->c, RSV_ERR_ARG, std::string("cannot open ") + path);
    const char magic[8] = {'R', 'S', 'V', 'N', 'E', 'T', '1', 0};
    const int32_t hdr[4] = {3, n->a.c[0], n->a.c[1], n->a.c[2]};
    const int64_t meta[2] = {n->a.np, n->step};
    bool ok = fwrite(magic, 1, 8, f) == 8 && fwrite(hdr, 4, 4, f) == 4 && fwrite(meta, 8, 2, f) == 2 &&
              fwrite(h.data(), 4, h.size(), f) == h.size();
    fclose(f);
    return ok ? RSV_OK : set_err(n->c, RSV_ERR_ARG, "write failed");
}

rsv_status rsv_net_load(rsv_net *n, const char *path)
{
    if (!n || !path) return set_err(n ? n->c : nullptr, RSV_ERR_ARG, "NULL argument");
    FILE *f = fopen(path, "rb");
    if (!f) return set_err(n->c, RSV_ERR_ARG, std::string("cannot open ") + path);
    char magic[8];
    int32_t hdr[4];
    int64_t meta[2];
    bool ok = fread(magic, 1, 8, f) == 8 && std::memcmp(magic, "RSVNET1", 7) == 0 && fread(hdr, 4, 4, f) == 4 &&
              fread(meta, 8, 2, f) == 2 && hdr[1] == n->a.c[0] && hdr[2] == n->a.c[1] && hdr[3] == n->a.c[2] &&
              meta[0] == n->a.np;
    std::vector<float> h(ok ? n->a.np : 0);
    if (ok) ok = fread(h.data(), 4, h.size(), f) == h.size();
    fclose(f);
    if (!ok) return set_err(n->c, RSV_ERR_ARG, "not a network file of this architecture");
    rsv_status s = rsv_net_set_params(n, h.data(), n->a.np);
    n->step = meta[1];
    return s;
}

rsv_status rsv_net_forward(rsv_net *n, rsv_grid *g, const double *r, const float *lnk, double *z)
{
    if (!n || !g || !r || !lnk || !z) return set_err(n ? n->c : nullptr, RSV_ERR_ARG, "NULL argument");
    rsv_ctx *c = n->c;
    rsv_status s = dims_check(c, g);
    if (s == RSV_OK) s = net_ws(n, g->geo.nx, g->geo.ny, g->geo.nz, 1, false);
    if (s == RSV_OK) s = set_lnk(n, g, 1, lnk, n->sum_lnk(), n->dev_lnk(), n->lnk_std);
    if (s == RSV_OK) s = prep(n, g, 1, nullptr, r, n->lnk_std);
    if (s == RSV_OK) s = net_forward(n, g->geo.nx, g->geo.ny, g->geo.nz, 1);
    if (s != RSV_OK) return s;
    hipLaunchKernelGGL(k_post, dim3(nblk(g->ncell)), dim3(256), 0, c->stream, g->geo, (const float *)n->y,
                       (const double *)n->sum_r2(), (double *)nullptr, z);
    RSV_LAUNCH(c);
    RSV_HIP(c, hipStreamSynchronize(c->stream));
    return RSV_OK;
}

// Loss and gradient of a batch.  Samples go through the network together, as
// many as keep a pass within 2^21 voxels (at 64x64x32 all of a batch of 8 or
// 16): one sample's quarter-resolution layers are 16 workgroups, and each of
// the backward pass's launches costs about what such a layer computes.  Larger
// passes gain nothing and cost about 600 bytes of workspace per voxel.
static rsv_status loss_grad_batch(rsv_net *n, rsv_grid *g, int32_t nb, const double *r, const double *e,
                                  const float *lnk, float *loss_out)
{
    rsv_ctx *c = n->c;
    if (nb < 1) return set_err(c, RSV_ERR_ARG, "batch must be >= 1");
    rsv_status s = dims_check(c, g);
    if (s != RSV_OK) return s;
    const int64_t V = g->ncell, N = 3 * V;
    const int nx = g->geo.nx, ny = g->geo.ny, nz = g->geo.nz;
    int per = (int)std::max<int64_t>(1, std::min<int64_t>(nb, ((int64_t)1 << 21) / V));
    s = net_ws(n, nx, ny, nz, per, true);
    if (s == RSV_ERR_OOM && per > 1) s = net_ws(n, nx, ny, nz, per = 1, true);   // one sample's may still fit
    if (s != RSV_OK) return s;
    if (!n->packed && (s = net_pack(n)) != RSV_OK) return s;
    RSV_HIP(c, hipMemsetAsync(n->G, 0, (size_t)n->a.np * sizeof(float), c->stream));
    double total = 0.0;
    std::vector<double> sums(2 * (size_t)per);
    const int nbk = nblk(V) < 1024 ? nblk(V) : 1024;
    for (int b0 = 0; b0 < nb; b0 += per) {
        const int q = std::min<int>(per, nb - b0);
        const double *rb = r + (int64_t)b0 * N, *eb = e + (int64_t)b0 * N;
        if ((s = set_lnk(n, g, q, lnk + (int64_t)b0 * V, n->sum_lnk(), n->dev_lnk(), n->lnk_std)) != RSV_OK) return s;
        if ((s = prep(n, g, q, nullptr, rb, n->lnk_std)) != RSV_OK) return s;
        if ((s = net_forward(n, nx, ny, nz, q)) != RSV_OK) return s;
        if ((s = partials_reserve(c, 2 * (int64_t)nbk * q)) != RSV_OK) return s;
        hipLaunchKernelGGL(k_loss, dim3(nbk, q), dim3(256), 0, c->stream, g->geo, (const float *)n->y, eb,
                           (const double *)n->sum_r2(), c->d_partials);
        RSV_LAUNCH(c);
        if ((s = launch_reduce_to(c, nbk, 2 * q, n->loss())) != RSV_OK) return s;
        // gy = (2 / nb) (y - e/s) / ||e/s||^2
        hipLaunchKernelGGL(k_gy, dim3(nblk(V * q)), dim3(256), 0, c->stream, g->geo, q, (const float *)n->y, eb,
                           (const double *)n->sum_r2(), (const double *)n->loss(), 1.0f / (float)nb, n->gy);
        RSV_LAUNCH(c);
        if ((s = net_backward(n, nx, ny, nz, q)) != RSV_OK) return s;
        RSV_HIP(c, hipMemcpyAsync(sums.data(), n->loss(), 2 * (size_t)q * sizeof(double), hipMemcpyDeviceToHost, c->stream));
        RSV_HIP(c, hipStreamSynchronize(c->stream));
        for (int b = 0; b < q; ++b) total += sums[2 * b] / sums[2 * b + 1];
    }
    if (loss_out) *loss_out = (float)(total / nb);
    return RSV_OK;
}

rsv_status rsv_net_loss_grad(rsv_net *n, rsv_grid *g, int32_t nb, const double *r, const double *e, const float *lnk,
                             float *loss_out, float *grad_out)
{
    if (!n || !g || !r || !e || !lnk) return set_err(n ? n->c : nullptr, RSV_ERR_ARG, "NULL argument");
    rsv_status s = loss_grad_batch(n, g, nb, r, e, lnk, loss_out);
    if (s != RSV_OK) return s;
    if (grad_out) {
        RSV_HIP(n->c, hipMemcpyAsync(grad_out, n->G, (size_t)n->a.np * sizeof(float), hipMemcpyDeviceToHost, n->c->stream));
    }
    RSV_HIP(n->c, hipStreamSynchronize(n->c->stream));
    return RSV_OK;
}

rsv_status rsv_net_train_step(rsv_net *n, rsv_grid *g, int32_t nb, const double *r, const double *e, const float *lnk,
                              float lr, float *loss_out)
{
    if (!n || !g || !r || !e || !lnk) return set_err(n ? n->c : nullptr, RSV_ERR_ARG, "NULL argument");
    rsv_status s = loss_grad_batch(n, g, nb, r, e, lnk, loss_out);
    if (s != RSV_OK) return s;
    n->step += 1;
    const float c1 = 1.0f - powf(0.9f, (float)n->step), c2 = 1.0f - powf(0.999f, (float)n->step);
    hipLaunchKernelGGL(k_adam, dim3(nblk(n->a.np)), dim3(256), 0, n->c->stream, n->a.np, n->P, (const float *)n->G, n->M,
                       n->Vv, lr, c1, c2);
    RSV_LAUNCH(n->c);
    s = net_pack(n);
    if (s != RSV_OK) return s;
    RSV_HIP(n->c, hipStreamSynchronize(n->c->stream));
    return RSV_OK;
}

// ---------------------------------------------------------------- single-layer entry points

rsv_status rsv_conv3d(rsv_ctx *c, int32_t nx, int32_t ny, int32_t nz, int32_t cin, int32_t cout, const uint16_t *x,
                      const float *w, const float *b, float *y)
{
    if (!c || !x || !w || !y) return set_err(c, RSV_ERR_ARG, "NULL argument");
    if (cin % 4 || cin < 4 || cin > 64 || (cout != 16 && cout != 32 && cout != 64) || nx < 1 || ny < 1 || nz < 1)
        return set_err(c, RSV_ERR_ARG, "conv3d needs cin a multiple of 4 up to 64, cout 16/32/64, positive dims");
    const int KB = conv_kblocks(cin), NB = cout / 16;
    short *wf = nullptr;
    rsv_status s = dev_alloc(c, (void **)&wf, (size_t)KB * NB * 64 * conv_frag_bytes(cin));
    if (s != RSV_OK) return s;
    hipLaunchKernelGGL(k_pack, dim3(nblk((int64_t)KB * NB * 64)), dim3(256), 0, c->stream, w, cin, cout, 0, KB, NB,
                       conv_kw(cin), wf);
    ConvGeo g{nx, ny, nz, nz, 0, cin, cout, (int64_t)nx * ny * nz};
    hipError_t e = launch_conv<false>(c, g, x, wf, KB, Epilogue{b, nullptr, 0, nullptr, nullptr, y});
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    dev_free(wf);
    if (e != hipSuccess) return set_err(c, RSV_ERR_HIP, std::string("conv3d: ") + hipGetErrorString(e));
    return RSV_OK;
}

rsv_status rsv_conv3d_bwd(rsv_ctx *c, int32_t nx, int32_t ny, int32_t nz, int32_t cin, int32_t cout, const uint16_t *x,
                          const float *w, const uint16_t *dy, float *dx, float *dw, float *db)
{
    if (!c || !x || !w || !dy) return set_err(c, RSV_ERR_ARG, "NULL argument");
    if (cin % 4 || cin < 4 || cin > 64 || (cout != 16 && cout != 32 && cout != 64) || nx < 1 || ny < 1 || nz < 1)
        return set_err(c, RSV_ERR_ARG, "conv3d needs cin a multiple of 4 up to 64, cout 16/32/64, positive dims");
    if (dx && cin % 16) return set_err(c, RSV_ERR_ARG, "the data gradient needs cin in {16, 32, 64}");
    // a one-layer network-like view to reuse the layer kernels
    rsv_net tmp;
    tmp.c = c;
    tmp.a.init(16, 16, 16);
    tmp.a.cin[1] = cin;
    tmp.a.cout[1] = cout;
    const int KBt = conv_kblocks(cout), NBt = (cin + 15) / 16;
    rsv_status s = RSV_OK;
    if (dx) {
        s = dev_alloc(c, (void **)&tmp.wt[1], (size_t)KBt * NBt * 64 * conv_frag_bytes(cout));
        if (s == RSV_OK) {
            hipLaunchKernelGGL(k_pack, dim3(nblk((int64_t)KBt * NBt * 64)), dim3(256), 0, c->stream, w, cin, cout, 1, KBt,
                               NBt, conv_kw(cout), (short *)tmp.wt[1]);
            s = conv_bwd_data(&tmp, 1, nx, ny, nz, nz, dy, dx, nullptr, nullptr, nullptr);
        }
    }
    if (s == RSV_OK && (dw || db)) {
        float *gw = nullptr;
        const int64_t nwb = 27LL * cin * cout + cout;
        s = dev_alloc(c, (void **)&gw, (size_t)nwb * sizeof(float));
        if (s == RSV_OK && hipMemsetAsync(gw, 0, (size_t)nwb * sizeof(float), c->stream) != hipSuccess)
            s = set_err(c, RSV_ERR_HIP, "hipMemsetAsync");
        if (s == RSV_OK) s = conv_bwd_weight(&tmp, 1, nx, ny, nz, nz, 0, x, dy, 1.0f, gw, gw + 27LL * cin * cout);
        if (s == RSV_OK && dw)
            if (hipMemcpyAsync(dw, gw, 27LL * cin * cout * sizeof(float), hipMemcpyDeviceToDevice, c->stream) != hipSuccess)
                s = set_err(c, RSV_ERR_HIP, "hipMemcpyAsync");
        if (s == RSV_OK && db)
            if (hipMemcpyAsync(db, gw + 27LL * cin * cout, cout * sizeof(float), hipMemcpyDeviceToDevice, c->stream) != hipSuccess)
                s = set_err(c, RSV_ERR_HIP, "hipMemcpyAsync");
        if (hipStreamSynchronize(c->stream) != hipSuccess && s == RSV_OK) s = set_err(c, RSV_ERR_HIP, "sync");
        dev_free(gw);
    }
    if (hipStreamSynchronize(c->stream) != hipSuccess && s == RSV_OK) s = set_err(c, RSV_ERR_HIP, "sync");
    return s;
}

}  // extern "C"
