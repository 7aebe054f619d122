// Block ILU(0) of the 7-point, 3x3-block matrix in natural (bottom-up) order:
// factorisation and the two triangular sweeps (Preconditioners section: LU x
// = b <=> L y = b, U x = y, solved row by row; ILU(0) is the default local
// solver of the RAS default-parameter figure).
//
// On the bipartite 7-point graph, ILU(0) reduces to pivots
//   D_c = A_cc - sum_{k in {-z,-y,-x}} A_ck D_k^{-1} A_kc,
// with L_ck = A_ck D_k^{-1} (unit lower factor) and U = D + strict upper of A.
// Cell c depends only on its -x,-y,-z neighbours, all on hyperplane
// i+j+k-1, so processing hyperplanes in order reproduces natural-order ILU(0)
// exactly (same operations per cell; only the FP order inside a cell may
// differ from a row-by-row code).
//
// Two executions of the sweeps:
//  * one launch per hyperplane (reference; also the factorisation);
//  * pipelined tiles: a workgroup of nine waves sweeps an 8x8 column of cells, cell
//    (i,j) walking up the column skewed by i+j steps, so that a step's 64 cells
//    lie on one hyperplane; updating, loading and handing on are different waves'
//    work, exchanged through LDS with one barrier per step.  Neighbouring tiles
//    hand over their boundary faces through epoch-tagged 64-bit words (value
//    and tag in one single-copy-atomic word, so no fences are needed).  Tiles
//    are taken from an atomic ticket in topological order, so a tile only
//    ever waits on tiles already held by running workgroups (no deadlock);
//    every wait is bounded by a wall-clock limit that raises an error flag.
#include "rsv_internal.h"

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <new>

namespace {

constexpr int BS = 256;

__device__ inline int64_t fidx(int64_t slot, int e, int ne) { return ((slot >> 6) * ne + e) * 64 + (slot & 63); }

// Arithmetic of a cell in the sweeps by hyperplanes.  The pipelined sweeps form the
// same chains, a component per lane, so that FP64 gives the same bits either way:
// explicit fused multiply-adds, the same operation sequence whatever the
// contraction choices around them.
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
// forward: out = r - (L_-z vz + L_-y vy + L_-x vx), one FMA chain per
// component (terms in the order -z, -y, -x), the three chains advanced in
// lockstep; negated products are free operand modifiers
template <typename T>
__device__ __forceinline__ void fwd_cell(const T *l, const T *vz, const T *vy, const T *vx, const T *rr, T *out)
{
    T acc[3] = {rr[0], rr[1], rr[2]};
    const T *v[3] = {vz, vy, vx};
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int p = 0; p < 3; ++p) acc[p] = fma_t(-l[9 * s + 3 * p + q], v[s][q], acc[p]);
#pragma unroll
    for (int p = 0; p < 3; ++p) out[p] = acc[p];
}
// backward: out = Dinv (y - (U_+x vx + U_+y vy + U_+z vz)), same chain order (+x, +y, +z)
template <typename T>
__device__ __forceinline__ void bwd_cell(const T *u, const T *dd, const T *vx, const T *vy, const T *vz, const T *yy,
                                         T *out)
{
    T tv[3] = {yy[0], yy[1], yy[2]};
    const T *v[3] = {vx, vy, vz};
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int p = 0; p < 3; ++p) tv[p] = fma_t(-u[9 * s + 3 * p + q], v[s][q], tv[p]);
#pragma unroll
    for (int p = 0; p < 3; ++p) out[p] = fma_t(dd[3 * p + 2], tv[2], fma_t(dd[3 * p + 1], tv[1], dd[3 * p] * tv[0]));
}

// ---------------------------------------------------------------- hyperplanes
// Hyperplane p of a grid of boxes: the cells with (i mod mx) + (j mod my) +
// (k mod mz) = p.  A wave of a launch takes one tile of one box (plane_tiles), whose
// cells of p share a row.  (Lists of each plane's slots, built on the host with every
// grid and auxiliary grid, were 12 of the 14.7 ms of a RAS setup at 128x128x64,
// which takes 2.4 ms without.)
struct Planes {
    Geo g;
    PlaneTiles t;
    int mz, p, d;            // d: first row of the launch
    int nbx, nbox, nunit;    // boxes in x, in a layer of boxes, in all
};
__device__ inline bool plane_cell(const Planes &P, int &gx, int &gy, int &k, int64_t &slot)
{
    int w = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)));
    int unit = 0, zb = 0, tx, ty;
    if (P.nunit > 1) {
        unit = w / P.t.row;
        w -= unit * P.t.row;
        if (unit >= P.nunit) return false;
    }
    if (!plane_tile(P.t, w, P.d + (int)blockIdx.y, tx, ty)) return false;
    const int q = P.p - 8 * (tx + ty);   // k mod mz of the tile's lane (0, 0)
    if (q < 0 || q >= P.mz + 14) return false;
    if (P.nunit > 1) {
        zb = unit / P.nbox;
        const int box = unit - zb * P.nbox, by = box / P.nbx;
        tx += (box - by * P.nbx) * P.t.btx;
        ty += by * P.t.bty;
    }
    int i, j;
    lane_ij((int)(threadIdx.x & 63), i, j);
    gx = tx * 8 + i;
    gy = ty * 8 + j;
    const int kk = q - i - j;
    k = zb * P.mz + kk;
    if (kk < 0 || kk >= P.mz || gx >= P.g.nx || gy >= P.g.ny || k >= P.g.nz) return false;
    // slot_of, whose row k + i + j is the wave's
    slot = ((int64_t)(ty * P.g.ntx + tx) * P.g.nz + wrap_nz(zb * P.mz + q, P.g.nz)) * 64 + (threadIdx.x & 63);
    return true;
}

// ---------------------------------------------------------------- factorisation (one launch per hyperplane)
__global__ __launch_bounds__(BS) void k_factor_plane(Planes P, const double *__restrict__ A, double *__restrict__ Lf,
                                                     double *__restrict__ Dinv, int32_t *flags)
{
    const Geo &g = P.g;
    int gx, gy, k;
    int64_t slot;
    if (!plane_cell(P, gx, gy, k, slot)) return;
    double D[9];
    for (int e = 0; e < 9; ++e) D[e] = A[aidx(slot, 27 + e)];
    for (int s = 0; s < 3; ++s) {   // -z, -y, -x: ascending column order
        int di, dj, dk;
        dir_off(s, di, dj, dk);
        double L[9];
        if (gx + di >= 0 && gy + dj >= 0 && k + dk >= 0) {
            const int64_t ns = slot_of(g, gx + di, gy + dj, k + dk);
            double Ack[9], Dk[9], Akc[9];
            for (int e = 0; e < 9; ++e) {
                Ack[e] = A[aidx(slot, s * 9 + e)];
                Dk[e] = Dinv[fidx(ns, e, 9)];
                Akc[e] = A[aidx(ns, (6 - s) * 9 + e)];
            }
            for (int p = 0; p < 3; ++p)
                for (int q = 0; q < 3; ++q)
                    L[3 * p + q] = Ack[3 * p] * Dk[q] + Ack[3 * p + 1] * Dk[3 + q] + Ack[3 * p + 2] * Dk[6 + q];
            for (int p = 0; p < 3; ++p)
                for (int q = 0; q < 3; ++q)
                    D[3 * p + q] -= L[3 * p] * Akc[q] + L[3 * p + 1] * Akc[3 + q] + L[3 * p + 2] * Akc[6 + q];
        } else {
            for (int e = 0; e < 9; ++e) L[e] = 0.0;
        }
        for (int e = 0; e < 9; ++e) Lf[fidx(slot, s * 9 + e, 27)] = L[e];
    }
    double Di[9];
    if (!inv3(D, Di)) {
        atomicOr(&flags[0], FLAG_PIVOT);
        atomicMin(&flags[1], (int32_t)row_of(g, gx, gy, k));
        for (int e = 0; e < 9; ++e) Di[e] = 0.0;
    }
    for (int e = 0; e < 9; ++e) Dinv[fidx(slot, e, 9)] = Di[e];
}

template <typename T>
__global__ __launch_bounds__(BS) void k_to_f32(int64_t n, const double *__restrict__ a, T *__restrict__ b)
{
    for (int64_t e = (int64_t)blockIdx.x * BS + threadIdx.x; e < n; e += (int64_t)gridDim.x * BS) b[e] = (T)a[e];
}

// strict upper blocks of A (+x,+y,+z) as FP32 in [row][27][64]
__global__ __launch_bounds__(BS) void k_upper_f32(int64_t nslot, const double *__restrict__ A, float *__restrict__ U)
{
    const int64_t slot = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (slot >= nslot) return;
    for (int e = 0; e < 27; ++e) U[fidx(slot, e, 27)] = (float)A[aidx(slot, 36 + e)];
}

// ---------------------------------------------------------------- sweeps, one launch per hyperplane
// T: arithmetic / factor type.  Upper blocks: U (T, [row][27][64]) when
// non-null, else the FP64 matrix A directly.
template <typename T>
__global__ __launch_bounds__(BS) void k_fwd_plane(Planes P, const T *__restrict__ Lf, const double *__restrict__ r,
                                                  T *__restrict__ y)
{
    const Geo &g = P.g;
    int gx, gy, k;
    int64_t slot;
    if (!plane_cell(P, gx, gy, k, slot)) return;
    T v[3][3];   // -z, -y, -x neighbour values
    for (int s = 0; s < 3; ++s) {
        int di, dj, dk;
        dir_off(s, di, dj, dk);
        v[s][0] = v[s][1] = v[s][2] = 0;
        if (gx + di >= 0 && gy + dj >= 0 && k + dk >= 0) {
            const int64_t ns = slot_of(g, gx + di, gy + dj, k + dk);
            for (int p = 0; p < 3; ++p) v[s][p] = y[vidx(ns, p)];
        }
    }
    T l[27], rr[3], out[3];
    for (int e = 0; e < 27; ++e) l[e] = Lf[fidx(slot, e, 27)];
    for (int p = 0; p < 3; ++p) rr[p] = (T)r[vidx(slot, p)];
    fwd_cell(l, v[0], v[1], v[2], rr, out);
    for (int p = 0; p < 3; ++p) y[vidx(slot, p)] = out[p];
}

template <typename T>
__global__ __launch_bounds__(BS) void k_bwd_plane(Planes P, const T *__restrict__ Dinv, const T *__restrict__ U,
                                                  const double *__restrict__ A, const T *__restrict__ y,
                                                  T *__restrict__ zt, double *__restrict__ z)
{
    const Geo &g = P.g;
    int gx, gy, k;
    int64_t slot;
    if (!plane_cell(P, gx, gy, k, slot)) return;
    T v[3][3];   // +x, +y, +z neighbour values
    for (int s = 4; s < 7; ++s) {
        int di, dj, dk;
        dir_off(s, di, dj, dk);
        v[s - 4][0] = v[s - 4][1] = v[s - 4][2] = 0;
        if (gx + di < g.nx && gy + dj < g.ny && k + dk < g.nz) {
            const int64_t ns = slot_of(g, gx + di, gy + dj, k + dk);
            for (int p = 0; p < 3; ++p) v[s - 4][p] = zt[vidx(ns, p)];
        }
    }
    T u[27], dd[9], yy[3], out[3];
    for (int e = 0; e < 27; ++e) u[e] = U ? U[fidx(slot, e, 27)] : (T)A[aidx(slot, 36 + e)];
    for (int e = 0; e < 9; ++e) dd[e] = Dinv[fidx(slot, e, 9)];
    for (int p = 0; p < 3; ++p) yy[p] = y[vidx(slot, p)];
    bwd_cell(u, dd, v[0], v[1], v[2], yy, out);
    for (int p = 0; p < 3; ++p) {
        zt[vidx(slot, p)] = out[p];
        z[vidx(slot, p)] = (double)out[p];
    }
}

// factors of the real slots into block-row order: L[row][27], Dinv[row][9]
__global__ __launch_bounds__(BS) void k_factors_to_rows(Geo g, const double *__restrict__ Lf,
                                                        const double *__restrict__ Dinv, double *__restrict__ Lr,
                                                        double *__restrict__ Dr)
{
    const int64_t slot = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (slot >= g.nslot) return;
    int gx, gy, k;
    if (!cell_of(g, slot, gx, gy, k)) return;
    const int64_t row = row_of(g, gx, gy, k);
    for (int e = 0; e < 27; ++e) Lr[row * 27 + e] = Lf[fidx(slot, e, 27)];
    for (int e = 0; e < 9; ++e) Dr[row * 9 + e] = Dinv[fidx(slot, e, 9)];
}

// ---------------------------------------------------------------- pipelined tile-lane sweeps
//
// One workgroup of nine waves per tile at a time.  Step t of a tile: lane (i, j)
// handles cell k = t - (i+j) (forward) or k = nz-1-(t-(14-i-j)) (backward), so
// the 64 cells of a step lie on one hyperplane; the cell's data sit in row (t
// mod nz) (forward) or ((nz+13-t) mod nz) (backward) of the tile.
//
// What bounds a sweep of a small or medium grid is the length of a step, since
// the steps of a tile, and of the tiles behind it, follow one another.  A step
// done by one wave is that wave's instruction issue (27 multiply-adds, 30 or 39
// operand reads, addresses, tags, faces: 1070 cycles forward, 1450 backward), so
// it is cut up: waves 0 to 3 update 16 cells each, one component of a cell per
// lane in groups of four lanes (9 multiply-adds; the backward sweep exchanges the
// three inside the group before the product with D^-1), waves 4 to 6 bring in
// operands, wave 7 the next step's faces, and wave 8 hands on the previous step's
// and stores its results.  One workgroup barrier per step orders them; there are
// no tags inside the workgroup.
//
// Operands and faces go from memory to LDS without passing through registers:
// the loading waves copy a step's rows with 16-byte LDS loads (1 KiB per
// instruction) into a ring of D slots, D steps ahead, and wait for a step's
// copies by the count of loads issued since.  The updating waves read a step's
// operands during the step before and keep their own last values in registers:
// between two barriers lie two reads, of one component of the x and y neighbours
// (the lanes of a group exchange them), and six multiply-adds.  The components of
// a cell are three rows apart, in the same banks; so the copies turn row r by
// (r mod 4) times eight cells.  Tiles follow one another in the ring without a
// gap.  A tile has one empty step at its end, in which the last results leave
// before wave 7 waits for the next tile's first faces.
//
// Against one updating wave fed by 7 (3) register-loading waves, forward/backward
// in us: 8 x 8 x 2048 cells FP64 912/1241 -> 607/694 (0.29/0.33 per step, bound by
// the reads and copies of LDS and the barrier), 64 x 64 x 256 231/301 -> 173/204,
// 128 x 128 x 64 236/283 -> 183/209, 20 x 20 x 10 40/48 -> 34/38; FP32 785/861 ->
// 530/580, 177/192 -> 150/159, 177/192 -> 167/175, 33/35 -> 32/34.  Between tiles a
// hop costs eight steps and about 2 us, from the store of a face to its arrival;
// loading faces 4 or 8 steps ahead instead of 2 makes that longer (128 x 128 x 64
// forward 199 and 237).
//
// Face exchange between neighbouring tiles: face row s of a tile holds the
// eight boundary values (three components each) that the neighbouring tile
// needs at its local step s; the producing lane computes them at its own step
// s + 7.  FP64 values are split into 32-bit halves, each stored with the
// 32-bit call epoch in the upper half of a 64-bit word (FP32 values: one
// word), so a word is valid exactly when its tag equals the current epoch --
// no fences between tiles, no clearing between calls (the buffers are cleared
// once, when allocated: memory another object wrote, possibly under another
// context's epochs, could otherwise hold a word with a matching tag).  Word (p*W + h)*8 + e
// of a row holds half h of component p of entry e.  A row is loaded SW_FACE
// steps before it is needed and, if it was not there yet, loaded again with those
// behind it until it is.  Tiles are
// handed out by an atomic ticket in topological order, so a tile only waits on
// tiles held by running workgroups; every wait is bounded by a wall-clock limit
// that raises an error flag and makes all other waits give up.

template <typename T> struct FaceW;
template <> struct FaceW<double> { static constexpr int W = 2; };
template <> struct FaceW<float> { static constexpr int W = 1; };

struct SweepArgs {
    Geo g;
    const int32_t *tile_order;   // tiles in topological (anti-diagonal) order
    uint64_t *ticket;
    uint64_t ticket_base;
    uint64_t *faceX;             // [NT][nz+7][24*W] words
    uint64_t *faceY;
    uint32_t epoch;
    int32_t *flags;
    uint64_t wait_limit;         // wall-clock ticks a wait may last
    int btx, bty;                // tiles per box in x and y: faces are exchanged only between
                                 // tiles of one box (the whole grid is one box for BILU0)
    uint64_t *trace;             // optional: per tile [start, step 8 reached, end, steps that waited for data]
};

// per-step operands streamed by the loaders; all rows are [entries][64 lanes]
template <typename T>
struct SweepSrc {
    const T *p0; int64_t s0, o0;                  // factor blocks (27): L (fwd) or U (bwd)
    const T *p1; int64_t s1, o1;                  // D^{-1} (bwd only, 9)
    const double *v64; const T *vT;               // 3-vector input: r (FP64, fwd) or y (T, bwd)
    const int32_t *zmap;                          // bwd, optional: slot of the output vector that takes
                                                  // each cell's result ([slot], -1: no store); null:
                                                  // the output has this grid's layout
};

constexpr int SW_FACE = 2;       // steps a face row is loaded ahead
constexpr int SW_MAXD = 10;      // ring slots at most: the next tile is claimed D + 5 steps before a tile's end
constexpr int SW_LDS = 160 * 1024;
constexpr int SW_THREADS = 64 * 9;
constexpr int64_t SW_NT_SLOTS = (int64_t)2 << 20;   // FP64 sweeps of this many slots load without keeping

// One step's operands in LDS: factor blocks (27 rows of 64), D^-1 (backward, 9),
// the right-hand side (3; FP64 forward), each as it lies in memory.
template <int DIR, typename T> struct SweepCfg {
    static constexpr int W = FaceW<T>::W, RW = 24 * W;
    static constexpr int ROWB = 64 * (int)sizeof(T);
    static constexpr int FB = 27 * ROWB, DB = DIR == 0 ? 0 : 9 * ROWB;
    static constexpr int VB = DIR == 0 ? 192 * 8 : 3 * ROWB;
    static constexpr int NF = (FB + 1023) / 1024, ND = (DB + 1023) / 1024, NV = (VB + 1023) / 1024;
    static constexpr int SLOT = FB + DB + VB;
    static constexpr int NCH = NF + ND + NV;                 // 1 KiB copies per step
    static constexpr int per(int w) { return (NCH - w + 2) / 3; }   // of loading wave w: w, w + 3, ...
    static constexpr int BUF = 3 * 80 * (int)sizeof(T);      // results [3][64] and faces [3][8 + 8] of one step
    static constexpr int ZB = DIR == 0 ? 0 : 2 * SW_FACE * 256;   // backward: output map entries of 2 SW_FACE steps
    static constexpr int FIXED = 2 * BUF + ZB + SW_FACE * 1024 + 16;
    // slots: what fits one workgroup, and no more loads in flight per wave than its counter holds
    static constexpr int dmin(int x, int y) { return x < y ? x : y; }
    static constexpr int D = dmin(SW_MAXD, dmin((SW_LDS - FIXED) / SLOT, 63 / per(0)));
    static constexpr int BYTES = D * SLOT + FIXED;
    static_assert(D >= 3 && D <= SW_MAXD && SW_FACE >= 2, "a tile has at least 16 steps: it is claimed D + 5 before the end");
};

// 16 (or 4) bytes per lane from src + voff to LDS address dst + 16 (4) lane (both
// + AT, below 4096); src uniform.  The compiler does not count these loads: the
// waits are explicit.  NT: nontemporal, the lines are not kept.  m0 is named as written,
// so that no use of it by the compiler is moved across; it warns that it reserves m0 for
// itself, as it does for LDS addresses like these.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int AT, bool NT> __device__ __forceinline__ void lds_copy(uint32_t voff, const void *src, uint32_t dst)
{
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%3 nt"
                     :
                     : "v"(voff), "s"(src), "s"(dst), "n"(AT)
                     : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%3"
                     :
                     : "v"(voff), "s"(src), "s"(dst), "n"(AT)
                     : "memory", "m0");
}
// the same past the caches that other dies do not see, as the face words need it
__device__ __forceinline__ void lds_copy_face(const void *p, uint32_t dst)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off sc1" ::"v"(p), "s"(dst) : "memory", "m0");
}
__device__ __forceinline__ void lds_copy4(const void *p, uint32_t dst)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(p), "s"(dst) : "memory", "m0");
}
#pragma clang diagnostic pop
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
template <int N> __device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// A loading wave's share of one step's copies: chunks c, c + 3, ... of the slot at
// LDS address dst.  f, d, v: the step's rows; vt, v8: the lanes' offsets within
// even and odd KiB of T and of FP64 rows.
template <int DIR, typename T, bool NT, int c>
__device__ __forceinline__ void sweep_copy(const char *f, const char *d, const char *v, const uint32_t (&vt)[2],
                                           const uint32_t (&v8)[2], uint32_t dst, int L)
{
    using C = SweepCfg<DIR, T>;
    if constexpr (c < C::NCH) {
        constexpr bool isf = c < C::NF, isd = !isf && c < C::NF + C::ND;
        constexpr int q = isf ? c : isd ? c - C::NF : c - C::NF - C::ND;          // KiB within its rows
        constexpr int len = (isf ? C::FB : isd ? C::DB : C::VB) - 1024 * q;
        constexpr int at = isf ? 0 : isd ? C::FB : C::FB + C::DB;
        constexpr int big = q / 4 * 4096, imm = q % 4 * 1024;
        const char *src = (isf ? f : isd ? d : v) + big;
        const uint32_t vo = (DIR == 0 && !isf) ? v8[q & 1] : vt[q & 1];
        if (len >= 1024 || L < len / 16) lds_copy<imm, NT>(vo, src, dst + at + big);
        sweep_copy<DIR, T, NT, c + 3>(f, d, v, vt, v8, dst, L);
    }
}

// lane Q's value in every group of four lanes
template <int Q> __device__ __forceinline__ float quad_get(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), Q * 0x55, 0xf, 0xf, true));
}
template <int Q> __device__ __forceinline__ double quad_get(double v)
{
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), Q * 0x55, 0xf, 0xf, true),
                            __builtin_amdgcn_mov_dpp(__double2loint(v), Q * 0x55, 0xf, 0xf, true));
}

template <int DIR, typename T, bool NT>
__global__ __launch_bounds__(SW_THREADS) void k_sweep(SweepArgs a, SweepSrc<T> src, T *__restrict__ yout,
                                               double *__restrict__ zout)
{
    using C = SweepCfg<DIR, T>;
    constexpr int W = C::W, RW = C::RW;
    extern __shared__ __align__(16) unsigned char smem[];
    const Geo &g = a.g;
    const int nz = g.nz, ntile = g.ntx * g.nty, nsteps = nz + 14, nst = nsteps + 1;
    constexpr int D = C::D;
    unsigned char *buf = smem + (size_t)D * C::SLOT;        // [parity][3][80]: 64 results, x face, y face
    int32_t *zb = (int32_t *)(buf + 2 * C::BUF);            // backward: [step % (2 SW_FACE)][64]
    unsigned char *fcb = (unsigned char *)zb + C::ZB;       // [step % SW_FACE]: x row, y row (512 bytes apart)
    int32_t *next = (int32_t *)(fcb + SW_FACE * 1024);
    auto lds_of = [](const void *p) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p; };
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), L = threadIdx.x & 63;
    const int64_t frow = (int64_t)(nz + 7) * RW;
    auto take = [&]() -> uint64_t { return atomicAdd((unsigned long long *)a.ticket, 1ull) - a.ticket_base; };
    auto tile_of = [&](uint64_t tk) -> int32_t {
        return tk >= (uint64_t)ntile ? -1 : a.tile_order[DIR == 0 ? (int)tk : ntile - 1 - (int)tk];
    };
    for (int e = threadIdx.x; e < 2 * C::BUF / 4; e += SW_THREADS) ((uint32_t *)buf)[e] = 0;
    if (threadIdx.x == 448) *next = tile_of(take());
    __syncthreads();
    int T_ = __builtin_amdgcn_readfirstlane(*next);
    if (T_ < 0) return;
    int gs = 0;      // steps so far, of all tiles
    if (wave < 4) {
        // ------------------------------------------------ updating waves
        const int cell = 16 * wave + (L >> 2), cp = min(L & 3, 2);   // the fourth lane repeats the third
        int li, lj;
        lane_ij(cell, li, lj);
        const int dd = DIR == 0 ? li + lj : 14 - li - lj;   // step at which the lane's column starts
        const int ax = DIR == 0 ? (li > 0 ? ij_lane(li - 1, lj) : 64 + lj) : (li < 7 ? ij_lane(li + 1, lj) : 64 + lj);
        const int ay = DIR == 0 ? (lj > 0 ? ij_lane(li, lj - 1) : 72 + li) : (lj < 7 ? ij_lane(li, lj + 1) : 72 + li);
        // row 3 cp + k of a slot's factors lies at r4[k & 3] + k ROWB, turned by eight cells times its number mod 4
        constexpr int E = sizeof(T), EV = DIR == 0 ? 8 : E;
        int r4[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) r4[k] = 3 * cp * C::ROWB + ((cell + 8 * ((3 * cp + k) & 3)) & 63) * E;
        const int rv = C::FB + C::DB + (cp * 64 + ((cell + 8 * cp) & 63)) * EV;
        struct Ops {
            T f[9], d[3], r;
        } A, B;
        int slot = 0, t = 0;
        T own = 0;      // this lane's value of the step before
        auto operands = [&](Ops &o) {
            const unsigned char *sl = smem + (size_t)slot * C::SLOT;
            auto row = [&](int at, int k) { return *(const T *)(sl + r4[k & 3] + at + k * C::ROWB); };
#pragma unroll
            for (int s = 0; s < 3; ++s)
#pragma unroll
                for (int q = 0; q < 3; ++q) o.f[3 * s + q] = row(0, 9 * s + q);
            if constexpr (DIR == 0) {
                o.r = (T)*(const double *)(sl + rv);
            } else {
                o.r = *(const T *)(sl + rv);
#pragma unroll
                for (int q = 0; q < 3; ++q) o.d[q] = row(C::FB, q);
            }
            slot = slot + 1 == D ? 0 : slot + 1;
        };
        // one step with operands o, reading the next one's; false after the last tile
        auto step = [&](const Ops &o, Ops &n, int par) {
            const T *rp = (const T *)(buf + (par ^ 1) * C::BUF);   // last step's results, this step's faces
            const T vx = rp[cp * 80 + ax], vy = rp[cp * 80 + ay];
            asm volatile("" ::: "memory");   // these first: reads return in order
            operands(n);
            asm volatile("" ::: "memory");
            const bool act = (unsigned)(t - dd) < (unsigned)nz;
            bool more = true;
            if (++t == nst) {
                t = 0;
                more = __builtin_amdgcn_readfirstlane(*next) >= 0;
            }
            auto block = [&](T acc, int s, T v) {
                acc = fma_t(-o.f[3 * s], quad_get<0>(v), acc);
                acc = fma_t(-o.f[3 * s + 1], quad_get<1>(v), acc);
                return fma_t(-o.f[3 * s + 2], quad_get<2>(v), acc);
            };
            if constexpr (DIR == 0) {
                own = block(block(block(o.r, 0, own), 1, vy), 2, vx);
            } else {
                own = block(block(block(o.r, 0, vx), 1, vy), 2, own);
                own = fma_t(o.d[2], quad_get<2>(own), fma_t(o.d[1], quad_get<1>(own), o.d[0] * quad_get<0>(own)));
            }
            own = act ? own : (T)0;
            if ((L & 3) < 3) ((T *)(buf + par * C::BUF))[cp * 80 + cell] = own;
            lds_barrier();
            return more;
        };
        lds_barrier();
        operands(A);
        lds_barrier();
        while (step(A, B, 0) && step(B, A, 1)) {}
        return;
    }
    if (wave < 7) {
        // ------------------------------------------------ loading waves
        // the next copies: step of the tile, its row's pointers, ring slot
        int tl = 0, row = DIR == 0 ? 0 : 13 % nz, slot = 0;
        const char *f, *d, *v;
        constexpr int sv = DIR == 0 ? 192 * 8 : 3 * C::ROWB;
        const int64_t sf = src.s0 * (int64_t)sizeof(T), sd = DIR == 0 ? 0 : src.s1 * (int64_t)sizeof(T);
        // rows go up (down) and around
        const int up = DIR == 0 ? 1 : -1, back = up * (1 - nz);
        const int64_t uf = up * sf, ud = up * sd, bf = back * sf, bd = back * sd;
        auto start = [&](int id) {
            tl = 0;
            row = DIR == 0 ? 0 : 13 % nz;
            const int64_t rb = (int64_t)id * nz + row;
            f = (const char *)(src.p0 + src.o0) + rb * sf;
            d = DIR == 0 ? nullptr : (const char *)(src.p1 + src.o1) + rb * sd;
            v = (DIR == 0 ? (const char *)src.v64 : (const char *)src.vT) + rb * sv;
        };
        auto next_row = [&]() {
            const bool wrap = row == (DIR == 0 ? nz - 1 : 0);
            row += wrap ? back : up;
            f += wrap ? bf : uf;
            if constexpr (DIR == 1) d += wrap ? bd : ud;
            v += wrap ? back * sv : up * sv;
        };
        start(T_);
        // a lane's offset in even (o = 0) or odd KiB of rows of E-byte entries, the cells held to [lo, hi]
        auto lane_at = [&](auto e, int o, int lo, int hi) -> uint32_t {
            constexpr int E = decltype(e)::value, CPR = 4 * E, LPC = 16 / E;   // 16-byte pieces per row, cells per piece
            const int r = L / CPR, turn = (r + (E == 8 ? 2 * o : 0)) * (8 / LPC);
            return (r * CPR + min(max((L - turn) & (CPR - 1), lo / LPC), hi / LPC)) * 16;
        };
        uint32_t vt0[2], v80[2];
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            vt0[o] = lane_at(std::integral_constant<int, sizeof(T)>{}, o, 0, 63);
            v80[o] = lane_at(std::integral_constant<int, 8>{}, o, 0, 63);
        }
        const uint32_t base = lds_of(smem);
        // Out-of-range lanes of the first and last steps copy the nearest in-range
        // lane's 16 bytes, so a step touches only the lines it needs (the wrapped
        // layout would re-read the rows at both ends of a column).
        auto copy = [&](auto w) {
            const int tc = tl < nsteps ? tl : nsteps - 1;
            uint32_t vt[2] = {vt0[0], vt0[1]}, v8[2] = {v80[0], v80[1]};
            if (tc < 14 || tc >= nz) {
                const int dlo = DIR == 0 ? max(tc - nz + 1, 0) : max(14 - tc, 0);
                const int dhi = DIR == 0 ? min(tc, 14) : min(13 - tc + nz, 14);
                const int lo = lane_first(dlo), hi = lane_first(dhi + 1) - 1;
#pragma unroll
                for (int o = 0; o < 2; ++o) {
                    vt[o] = lane_at(std::integral_constant<int, sizeof(T)>{}, o, lo, hi);
                    v8[o] = lane_at(std::integral_constant<int, 8>{}, o, lo, hi);
                }
            }
            const uint32_t dst = base + (uint32_t)slot * C::SLOT;
            sweep_copy<DIR, T, NT, decltype(w)::value>(f, d, v, vt, v8, dst, L);
            slot = slot + 1 == D ? 0 : slot + 1;
            if (tl + 1 < nsteps) next_row();   // the empty step copies the last row again
            ++tl;
        };
        auto run = [&](auto w) {
            constexpr int left = C::per(decltype(w)::value) * (D - 2);   // loads of the last D - 2 steps
            for (int q = 0; q < D; ++q) copy(w);       // D < nst: all of the first tile
            wait_loads<left>();
            lds_barrier();
            lds_barrier();
            for (;;) {
                for (int t = 0; t < nst; ++t) {
                    if (tl == nst) {
                        // the next tile was published two steps ago
                        const int nx = __builtin_amdgcn_readfirstlane(*next);
                        if (nx >= 0) start(nx);
                        else tl = nsteps;   // nothing follows: copy the last row again, to keep the count
                    }
                    copy(w);   // D steps ahead, into the slot whose operands the step before read
                    wait_loads<left>();
                    lds_barrier();
                }
                if (__builtin_amdgcn_readfirstlane(*next) < 0) break;
            }
            wait_loads<0>();   // no copy outlives the workgroup
        };
        if (wave == 4) run(std::integral_constant<int, 0>{});
        else if (wave == 5) run(std::integral_constant<int, 1>{});
        else run(std::integral_constant<int, 2>{});
        return;
    }
    // ---------------------------------------------------- face and result waves
    // lane q < RW holds word q of a face row: half (q >> 3) % W of component
    // (q >> 3) / W of entry e = q & 7; outgoing words come from the boundary
    // lane of entry e (x face: i = 7 forward, 0 backward, j = e; y face: i = e)
    const int fe = L & 7, fp = (L >> 3) / W, fh = (L >> 3) % W;
    struct Tile {
        int id;
        bool ix, iy, ox, oy;             // faces come in from, go out to the x and y neighbour
        int xs, ys;                      // tiles whose rows are read (its own where there is no neighbour: a dummy)
    };
    auto tile = [&](int id) {
        Tile k;
        k.id = id;
        const int bx = (id % g.ntx) % a.btx, by = (id / g.ntx) % a.bty;
        k.ix = DIR == 0 ? bx > 0 : bx < a.btx - 1;
        k.iy = DIR == 0 ? by > 0 : by < a.bty - 1;
        k.ox = DIR == 0 ? bx < a.btx - 1 : bx > 0;
        k.oy = DIR == 0 ? by < a.bty - 1 : by > 0;
        const int s = DIR == 0 ? -1 : 1;
        k.xs = k.ix ? id + s : id;
        k.ys = k.iy ? id + s * g.ntx : id;
        return k;
    };
    Tile cur = tile(T_);
    if (wave == 7) {
        const int fk_in = DIR == 0 ? fe : 7 - fe;
        const int xin = (fp * 80 + 64 + fe) * W + fh, yin = xin + 8 * W;        // 32-bit places in a buffer
        // lanes 0 to RW/2 - 1 copy an x row, those from 32 on a y row, 16 bytes each
        const bool copies = (L & 31) < RW / 2;
        const uint64_t *fsrc = (L < 32 ? a.faceX : a.faceY) + 2 * (L & 31), *fptr = nullptr;
        const int32_t *zp = nullptr;
        const uint32_t fdst = lds_of(fcb), zdst = lds_of(zb);
        Tile nxt = cur;                  // the tile after this step's
        int ta = 0, ga = 0;              // step of the next prefetch, in its tile and in all
        uint64_t tk = 0;
        bool over = false;               // a wait gave up: the flag is set, no wait lasts any more
        uint32_t waited = 0;
        const bool mapped = DIR == 1 && src.zmap != nullptr, tracing = a.trace != nullptr;
        int zrow = 0;
        auto face_row = [&](const Tile &k) { return fsrc + (int64_t)(L < 32 ? k.xs : k.ys) * frow; };
        auto start = [&](const Tile &k) {   // the prefetch goes to tile k
            ta = 0;
            fptr = face_row(k);
            zrow = 13 % nz;
            if (mapped) zp = src.zmap + ((int64_t)k.id * nz + zrow) * 64 + L;
        };
        auto fetch = [&]() {
            if (copies) lds_copy_face(fptr, fdst + ga % SW_FACE * 1024);
            if (ta < nz + 6) fptr += RW;      // rows end there; the steps behind need none
            if (mapped) {
                lds_copy4(zp, zdst + ga % (2 * SW_FACE) * 256);
                if (ta + 1 < nsteps) {
                    zp += zrow == 0 ? (nz - 1) * 64 : -64;
                    zrow = zrow == 0 ? nz - 1 : zrow - 1;
                }
            }
            ++ta;
            ++ga;
        };
        // the faces of a tile's step t (gt in all) into buffer b: zero where no neighbour or no cell
        auto bring = [&](const Tile &k, int t, int gt, unsigned char *b) {
            if (mapped) wait_loads<2 * (SW_FACE - 1)>();
            else wait_loads<SW_FACE - 1>();
            const bool need = L < RW && (unsigned)(t - fk_in) < (unsigned)nz;
            const bool nx = need & k.ix, ny = need & k.iy;
            const int Lc = L < RW ? L : RW - 1;
            const uint64_t *xr = (const uint64_t *)(fcb + gt % SW_FACE * 1024) + Lc, *yr = xr + 64;
            uint64_t x = *xr, y = *yr;
            auto missing = [&]() {
                return __ballot((nx & ((uint32_t)(x >> 32) != a.epoch)) | (ny & ((uint32_t)(y >> 32) != a.epoch))) != 0ull;
            };
            if (missing() && !over) {
                ++waited;
                const uint64_t t0 = wall_clock64();
                uint32_t n = 0;
                do {
                    if (spin_guard(a.flags, t0, n, a.wait_limit)) { over = true; break; }
                    wait_loads<0>();
                    for (int q = 0; q < SW_FACE && t + q < nz + 7; ++q)
                        if (copies) lds_copy_face(face_row(k) + (t + q) * RW, fdst + (gt + q) % SW_FACE * 1024);
                    wait_loads<0>();
                    x = *xr;
                    y = *yr;
                } while (missing());
            }
            if (L < RW) {
                ((uint32_t *)b)[xin] = nx ? (uint32_t)x : 0u;
                ((uint32_t *)b)[yin] = ny ? (uint32_t)y : 0u;
            }
        };
        start(cur);
        for (int q = 0; q < SW_FACE; ++q) fetch();
        bring(cur, 0, 0, buf + C::BUF);           // step 0 reads the odd buffer
        lds_barrier();
        lds_barrier();
        if (a.trace && L == 0) a.trace[4 * cur.id + 0] = wall_clock64();
        // the next tile is published this long before a tile's end: two steps before the first copies
        // and a step before the first prefetch that need it
        constexpr int early = D + 2 > SW_FACE + 1 ? D + 2 : SW_FACE + 1;
        int t = 0;
        bool done = false;
        while (!done) {
            fetch();      // step gs + SW_FACE, into the slot of step gs
            if (t >= nst - early - 3) {   // near the tile's end: the next one
                if (t == nst - early - 3 && L == 0) tk = take();
                if (t == nst - early) {
                    const int32_t id = __builtin_amdgcn_readfirstlane(L == 0 ? tile_of(tk) : 0);
                    if (L == 0) *next = id;
                    nxt.id = id;
                    if (id >= 0) nxt = tile(id);
                }
                if (ta == nst && nxt.id >= 0) start(nxt);
                if (t + 1 == nst) {
                    if (tracing && L == 0) {
                        a.trace[4 * cur.id + 2] = wall_clock64();
                        a.trace[4 * cur.id + 3] = waited;
                    }
                    waited = 0;
                    done = nxt.id < 0;
                    cur = nxt;
                    t = -1;
                    if (tracing && L == 0 && !done) a.trace[4 * cur.id + 0] = wall_clock64();
                }
            }
            // the next step's faces
            if (!done) bring(cur, t + 1, gs + 1, buf + (gs & 1) * C::BUF);
            if (t == 8 && tracing && L == 0) a.trace[4 * cur.id + 1] = wall_clock64();
            lds_barrier();
            ++gs;
            ++t;
        }
        wait_loads<0>();
    } else {
        int li, lj;
        lane_ij(L, li, lj);
        const int fb = DIR == 0 ? 7 : 0, fk_out = DIR == 0 ? 7 + fe : 14 - fe;
        const int fpc = L < RW ? fp : 0;
        const int xw = (fpc * 80 + ij_lane(fb, fe)) * W + fh, yw = (fpc * 80 + ij_lane(fe, fb)) * W + fh;
        const int dd = DIR == 0 ? li + lj : 14 - li - lj;
        const uint64_t ep = (uint64_t)a.epoch << 32;
        lds_barrier();
        lds_barrier();
        for (;;) {
            // where step t - 1's results and faces go
            int row = DIR == 0 ? 0 : 13 % nz;
            int64_t at = ((int64_t)cur.id * nz + row) * 192 + L;
            uint64_t *fx = a.faceX + (int64_t)cur.id * frow - 7 * RW + L, *fy = a.faceY + (int64_t)cur.id * frow - 7 * RW + L;
            lds_barrier();      // step 0 has nothing to hand on
            ++gs;
            for (int ts = 0; ts < nsteps; ++ts, ++gs) {
                const unsigned char *b = buf + ((gs + 1) & 1) * C::BUF;
                const T *res = (const T *)b + L;
                const T o[3] = {res[0], res[80], res[160]};
                const uint32_t wx = ((const uint32_t *)b)[xw], wy = ((const uint32_t *)b)[yw];
                if (L < RW && (unsigned)(ts - fk_out) < (unsigned)nz) {
                    if (cur.ox) face_st(fx, ep | wx);
                    if (cur.oy) face_st(fy, ep | wy);
                }
                fx += RW;
                fy += RW;
                if ((unsigned)(ts - dd) < (unsigned)nz) {
                    if constexpr (DIR == 0) {
#pragma unroll
                        for (int p = 0; p < 3; ++p) __builtin_nontemporal_store(o[p], yout + at + p * 64);
                    } else {
                        int64_t to = at;
                        bool st = true;
                        if (src.zmap) {
                            const int32_t zm = zb[(gs - 1) % (2 * SW_FACE) * 64 + L];
                            to = ((int64_t)(zm >> 6)) * 192 + (zm & 63);
                            st = zm >= 0;
                        }
                        if (st)
#pragma unroll
                            for (int p = 0; p < 3; ++p) __builtin_nontemporal_store((double)o[p], zout + to + p * 64);
                    }
                }
                const bool wrap = DIR == 0 ? row + 1 == nz : row == 0;
                const int m = DIR == 0 ? (wrap ? 1 - nz : 1) : (wrap ? nz - 1 : -1);
                row += m;
                at += (int64_t)m * 192;
                lds_barrier();
            }
            const int id = __builtin_amdgcn_readfirstlane(*next);
            if (id < 0) break;
            cur = tile(id);
        }
    }
}

// zero n 64-bit words
__global__ __launch_bounds__(256) void k_zero_words(int64_t n, uint64_t *__restrict__ p)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = 0ull;
}

// ---------------------------------------------------------------- the preconditioner object

struct Bilu0 : PcImpl {
    rsv_matrix *M = nullptr;
    rsv_ctx *c = nullptr;
    bool fp32 = false;
    bool pipelined = true;
    double *Lf = nullptr, *Dinv = nullptr;      // FP64 factors [row][27|9][64]
    float *Lf32 = nullptr, *Dinv32 = nullptr, *U32 = nullptr;
    void *ybuf = nullptr;                        // T-typed intermediate vector
    float *zt32 = nullptr;                       // FP32 z for the per-plane path
    double *zt64 = nullptr;
    uint64_t *faceX = nullptr, *faceY = nullptr;
    int64_t face_words = 0;                      // words per face buffer
    int32_t *tile_order = nullptr;
    int64_t nbytes = 0;
    int btx = 0, bty = 0;                        // tiles per box (0: the whole grid)
    const int32_t *zmap = nullptr;               // optional output map of the pipelined apply (not owned)

    ~Bilu0() override
    {
        dev_free(Lf); dev_free(Dinv); dev_free(Lf32); dev_free(Dinv32); dev_free(U32);
        dev_free(ybuf); dev_free(zt32); dev_free(zt64); dev_free(faceX); dev_free(faceY); dev_free(tile_order);
        dev_free(trace);
    }
    int64_t bytes() const override { return nbytes; }

    rsv_status bilu0_factors(double *L, double *D) override
    {
        if (fp32 || !Lf || !Dinv) return set_err(c, RSV_ERR_ARG, "factors are kept for the FP64 BILU0 form only");
        const Geo &g = M->g->geo;
        const int64_t nc = M->g->ncell;
        double *buf = nullptr;
        rsv_status s = dev_alloc(c, (void **)&buf, (size_t)nc * 36 * sizeof(double));
        if (s != RSV_OK) return s;
        hipLaunchKernelGGL(k_factors_to_rows, dim3((unsigned)((g.nslot + BS - 1) / BS)), dim3(BS), 0, c->stream, g, Lf,
                           Dinv, buf, buf + nc * 27);
        hipError_t e = hipGetLastError();
        if (e == hipSuccess) e = hipMemcpyAsync(L, buf, (size_t)nc * 27 * sizeof(double), hipMemcpyDeviceToHost, c->stream);
        if (e == hipSuccess)
            e = hipMemcpyAsync(D, buf + nc * 27, (size_t)nc * 9 * sizeof(double), hipMemcpyDeviceToHost, c->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
        dev_free(buf);
        if (e != hipSuccess) return set_err(c, RSV_ERR_HIP, std::string("factor export: ") + hipGetErrorString(e));
        return RSV_OK;
    }

    rsv_status alloc(void **p, size_t b)
    {
        rsv_status s = dev_alloc(c, p, b);
        if (s == RSV_OK) {
            nbytes += (int64_t)b;
            hipError_t e = hipMemsetAsync(*p, 0, b, c->stream);
            if (e != hipSuccess) return set_err(c, RSV_ERR_HIP, "hipMemsetAsync");
        }
        return s;
    }

    rsv_status setup(int64_t *bad_cell)
    {
        const Geo &g = M->g->geo;
        const int64_t rows = g.nslot / 64;
        if (btx <= 0) btx = g.ntx;
        if (bty <= 0) bty = g.nty;
        if (g.ntx % btx != 0 || g.nty % bty != 0) return set_err(c, RSV_ERR_ARG, "boxes must tile the grid");
        rsv_status s = alloc((void **)&Lf, (size_t)rows * 27 * 64 * sizeof(double));
        if (s == RSV_OK) s = alloc((void **)&Dinv, (size_t)rows * 9 * 64 * sizeof(double));
        if (s != RSV_OK) return s;
        s = flags_reset(c);
        if (s != RSV_OK) return s;
        ProfScope ps(c, RSV_K_FACTOR);
        for (int p = 0; p < M->g->nplanes; ++p) {
            on_plane(p, [&](const Planes &P, dim3 grid, dim3 blk) {
                hipLaunchKernelGGL(k_factor_plane, grid, blk, 0, c->stream, P, M->d_A, Lf, Dinv, c->d_flags);
            });
            RSV_LAUNCH(c);
        }
        s = flags_check(c, bad_cell);
        if (s != RSV_OK) return s;
        const int NT = g.ntx * g.nty;
        if (fp32) {
            s = alloc((void **)&Lf32, (size_t)rows * 27 * 64 * sizeof(float));
            if (s == RSV_OK) s = alloc((void **)&Dinv32, (size_t)rows * 9 * 64 * sizeof(float));
            if (s == RSV_OK) s = alloc((void **)&U32, (size_t)rows * 27 * 64 * sizeof(float));
            if (s == RSV_OK) s = alloc(&ybuf, (size_t)M->g->nv * sizeof(float));
            if (s == RSV_OK) s = alloc((void **)&zt32, (size_t)M->g->nv * sizeof(float));
            if (s != RSV_OK) return s;
            hipLaunchKernelGGL(k_to_f32<float>, dim3(2048), dim3(BS), 0, c->stream, rows * 27 * 64, Lf, Lf32);
            hipLaunchKernelGGL(k_to_f32<float>, dim3(2048), dim3(BS), 0, c->stream, rows * 9 * 64, Dinv, Dinv32);
            hipLaunchKernelGGL(k_upper_f32, dim3((unsigned)((g.nslot + BS - 1) / BS)), dim3(BS), 0, c->stream,
                               g.nslot, M->d_A, U32);
            RSV_LAUNCH(c);
            // FP64 factors are not needed by the FP32 sweeps
            RSV_HIP(c, hipStreamSynchronize(c->stream));
            dev_free(Lf); Lf = nullptr;
            dev_free(Dinv); Dinv = nullptr;
            nbytes -= (int64_t)rows * 36 * 64 * sizeof(double);
        } else {
            s = alloc(&ybuf, (size_t)M->g->nv * sizeof(double));
            if (s == RSV_OK) s = alloc((void **)&zt64, (size_t)M->g->nv * sizeof(double));
            if (s != RSV_OK) return s;
        }
        if (pipelined) {
            const int W = fp32 ? 1 : 2;
            face_words = (int64_t)NT * (g.nz + 7) * 24 * W;
            const size_t fb = (size_t)face_words * sizeof(uint64_t);
            // the sweeps keep a multi-slot ring in LDS: allow the full LDS per workgroup
            const void *fn[6] = {(const void *)k_sweep<0, double, false>, (const void *)k_sweep<1, double, false>,
                                 (const void *)k_sweep<0, double, true>,  (const void *)k_sweep<1, double, true>,
                                 (const void *)k_sweep<0, float, false>,  (const void *)k_sweep<1, float, false>};
            for (const void *f : fn) RSV_HIP(c, hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, c->lds_max));
            s = alloc((void **)&faceX, fb);
            if (s == RSV_OK) s = alloc((void **)&faceY, fb);
            if (s == RSV_OK) s = alloc((void **)&tile_order, (size_t)NT * sizeof(int32_t));
            if (s != RSV_OK) return s;
            // no word may carry a tag before its first write (epochs are never 0)
            const int nzb = (int)std::min<int64_t>((face_words + 255) / 256, 4096);
            hipLaunchKernelGGL(k_zero_words, dim3(nzb), dim3(256), 0, c->stream, face_words, faceX);
            hipLaunchKernelGGL(k_zero_words, dim3(nzb), dim3(256), 0, c->stream, face_words, faceY);
            RSV_LAUNCH(c);
            std::vector<int32_t> ord(NT);
            for (int t = 0; t < NT; ++t) ord[t] = t;
            // topological order: by anti-diagonal of the tile inside its box
            std::stable_sort(ord.begin(), ord.end(), [&](int a, int b) {
                const int da = (a % g.ntx) % btx + (a / g.ntx) % bty, db = (b % g.ntx) % btx + (b / g.ntx) % bty;
                return da < db;
            });
            // on the stream: behind the clearing of the same memory, whatever kind of stream it is
            RSV_HIP(c, hipMemcpyAsync(tile_order, ord.data(), NT * sizeof(int32_t), hipMemcpyHostToDevice, c->stream));
            RSV_HIP(c, hipStreamSynchronize(c->stream));   // ord is read
        }
        RSV_HIP(c, hipStreamSynchronize(c->stream));
        return RSV_OK;
    }

    template <class F> void on_plane(int p, const F &launch) const
    {
        const rsv_grid *G = M->g;
        // tiles per plane box: the grid's own, whatever boxes the sweeps have
        const int tx = std::min((G->mx + 7) / 8, G->geo.ntx), ty = std::min((G->my + 7) / 8, G->geo.nty);
        const int nbx = (G->geo.ntx + tx - 1) / tx, nby = (G->geo.nty + ty - 1) / ty, nbz = (G->geo.nz + G->mz - 1) / G->mz;
        Planes P{G->geo, plane_tiles(p, std::min(G->mz, G->geo.nz), tx, ty), G->mz, p, 0, nbx, nbx * nby, nbx * nby * nbz};
        plane_launch(c, P.t, P.nunit, [&](int d, dim3 grid, dim3 blk) {
            P.d = d;
            launch(P, grid, blk);
        });
    }

    template <typename T>
    rsv_status apply_plane(const double *r, double *z, const T *L_, const T *D_, const T *U_, T *zt)
    {
        T *y = (T *)ybuf;
        for (int p = 0; p < M->g->nplanes; ++p)
            on_plane(p, [&](const Planes &P, dim3 grid, dim3 blk) {
                hipLaunchKernelGGL(k_fwd_plane<T>, grid, blk, 0, c->stream, P, L_, r, y);
            });
        RSV_LAUNCH(c);
        for (int p = M->g->nplanes - 1; p >= 0; --p)
            on_plane(p, [&](const Planes &P, dim3 grid, dim3 blk) {
                hipLaunchKernelGGL(k_bwd_plane<T>, grid, blk, 0, c->stream, P, D_, U_, M->d_A, (const T *)y, zt, z);
            });
        RSV_LAUNCH(c);
        return RSV_OK;
    }

    uint64_t *trace = nullptr;   // RSV_SWEEP_TRACE=<file>: per-tile timestamps of every pipelined sweep

    SweepArgs sweep_args(uint64_t nwaves)
    {
        const Geo &g = M->g->geo;
        SweepArgs a;
        a.g = g;
        a.tile_order = tile_order;
        a.ticket = c->d_tickets;
        a.ticket_base = c->ticket_base[0];
        a.faceX = faceX;
        a.faceY = faceY;
        a.epoch = c->epoch++;
        if (c->epoch == 0) c->epoch = 1;
        a.flags = c->d_flags;
        a.wait_limit = c->wait_ticks;
        a.btx = btx;
        a.bty = bty;
        a.trace = trace;
        c->ticket_base[0] += (uint64_t)(g.ntx * g.nty) + nwaves;
        return a;
    }

    // workgroups of the pipelined sweeps: one per CU (each holds a large LDS ring)
    int nwaves() const
    {
        const int NT = M->g->geo.ntx * M->g->geo.nty;
        return std::max(1, std::min(NT, c->num_cu));
    }

    void dump_trace(int dir)
    {
        const char *path = getenv("RSV_SWEEP_TRACE");
        if (!path || !trace) return;
        const int NT = M->g->geo.ntx * M->g->geo.nty;
        std::vector<uint64_t> h((size_t)NT * 4);
        if (hipStreamSynchronize(c->stream) != hipSuccess) return;
        if (hipMemcpy(h.data(), trace, h.size() * sizeof(uint64_t), hipMemcpyDeviceToHost) != hipSuccess) return;
        FILE *fp = fopen(path, "a");
        if (!fp) return;
        fprintf(fp, "sweep dir=%d ntx=%d nty=%d nz=%d\n", dir, M->g->geo.ntx, M->g->geo.nty, M->g->geo.nz);
        for (int t = 0; t < NT; ++t)
            fprintf(fp, "%d %llu %llu %llu %llu\n", t, (unsigned long long)h[4 * t], (unsigned long long)h[4 * t + 1],
                    (unsigned long long)h[4 * t + 2], (unsigned long long)h[4 * t + 3]);
        fclose(fp);
    }

    rsv_status apply(const double *r, double *z) override
    {
        if (pipelined && getenv("RSV_SWEEP_TRACE") && !trace) {
            const int NT = M->g->geo.ntx * M->g->geo.nty;
            rsv_status s = alloc((void **)&trace, (size_t)NT * 4 * sizeof(uint64_t));
            if (s != RSV_OK) return s;
        }
        if (!pipelined) {
            ProfScope ps(c, RSV_K_ILU_FWD);
            if (fp32) return apply_plane<float>(r, z, Lf32, Dinv32, U32, zt32);
            return apply_plane<double>(r, z, Lf, Dinv, nullptr, zt64);
        }
        const int nw = nwaves();
        if (fp32) {
            SweepArgs a = sweep_args(nw);
            SweepSrc<float> s0{Lf32, (int64_t)27 * 64, 0, nullptr, 0, 0, r, nullptr, nullptr};
            size_t sh = SweepCfg<0, float>::BYTES;
            int t1 = prof_begin(c, RSV_K_ILU_FWD);
            hipLaunchKernelGGL((k_sweep<0, float, false>), dim3(nw), dim3(SW_THREADS), sh, c->stream, a, s0,
                               (float *)ybuf, (double *)nullptr);
            prof_end(c, t1);
            RSV_LAUNCH(c);
            SweepArgs b = sweep_args(nw);
            SweepSrc<float> s1{U32, (int64_t)27 * 64, 0, Dinv32, (int64_t)9 * 64, 0, nullptr, (const float *)ybuf, zmap};
            sh = SweepCfg<1, float>::BYTES;
            int t2 = prof_begin(c, RSV_K_ILU_BWD);
            hipLaunchKernelGGL((k_sweep<1, float, false>), dim3(nw), dim3(SW_THREADS), sh, c->stream, b, s1,
                               (float *)nullptr, z);
            prof_end(c, t2);
            RSV_LAUNCH(c);
        } else {
            // From 2 M slots the factors are loaded without keeping: up to there some of
            // them are still found in the 256 MB cache.  Forward/backward us, kept and not, one box:
            // 2.1 M slots 233/279 and 223/275, 2.5 M 254/308 and 254/306, 4.1 M 337/421 and 321/411,
            // 8.4 M 590/731 and 548/704.  RAS in 4 x 4 x 4 boxes (apply): 1.7 M slots 292 and 295, 1.8 M 320
            // and 334, 3.8 M 681 and 652, 11 M 1781 and 1692, 512 x 512 x 128 5620 and 5422.
            // FP32 sweeps gain nothing (8.4 M 397/440 to 419/450, not kept 407/445).
            const bool nt = M->g->geo.nslot >= SW_NT_SLOTS;
            SweepArgs a = sweep_args(nw);
            SweepSrc<double> s0{Lf, (int64_t)27 * 64, 0, nullptr, 0, 0, r, nullptr, nullptr};
            size_t sh = SweepCfg<0, double>::BYTES;
            int t1 = prof_begin(c, RSV_K_ILU_FWD);
            const auto fwd = nt ? k_sweep<0, double, true> : k_sweep<0, double, false>;
            hipLaunchKernelGGL(fwd, dim3(nw), dim3(SW_THREADS), sh, c->stream, a, s0, (double *)ybuf, (double *)nullptr);
            prof_end(c, t1);
            RSV_LAUNCH(c);
            dump_trace(0);
            SweepArgs b = sweep_args(nw);
            SweepSrc<double> s1{M->d_A, (int64_t)63 * 64, (int64_t)36 * 64, Dinv, (int64_t)9 * 64, 0, nullptr,
                                (const double *)ybuf, zmap};
            sh = SweepCfg<1, double>::BYTES;
            int t2 = prof_begin(c, RSV_K_ILU_BWD);
            const auto bwd = nt ? k_sweep<1, double, true> : k_sweep<1, double, false>;
            hipLaunchKernelGGL(bwd, dim3(nw), dim3(SW_THREADS), sh, c->stream, b, s1, (double *)nullptr, z);
            prof_end(c, t2);
            RSV_LAUNCH(c);
            dump_trace(1);
        }
        return RSV_OK;
    }
};

}  // namespace

int64_t sweep_ring_depth(const rsv_ctx *, int dir, int fp32)
{
    if (fp32) return dir == 0 ? SweepCfg<0, float>::D : SweepCfg<1, float>::D;
    return dir == 0 ? SweepCfg<0, double>::D : SweepCfg<1, double>::D;
}

rsv_status bilu0_create(rsv_matrix *A, const rsv_pc_params *p, PcImpl **out, int64_t *bad_cell)
{
    return bilu0_create_boxed(A, p, 0, 0, nullptr, out, bad_cell);
}

rsv_status bilu0_create_boxed(rsv_matrix *A, const rsv_pc_params *p, int btx, int bty, const int32_t *zmap,
                              PcImpl **out, int64_t *bad_cell)
{
    rsv_ctx *c = A->g->ctx;
    Bilu0 *B = new (std::nothrow) Bilu0();
    if (!B) return set_err(c, RSV_ERR_OOM, "bilu0");
    B->M = A;
    B->c = c;
    B->fp32 = (p->precision == RSV_FP32);
    B->pipelined = (p->pipelined != 0);
    B->btx = btx;
    B->bty = bty;
    B->zmap = zmap;
    if (zmap && !B->pipelined) {
        delete B;
        return set_err(c, RSV_ERR_ARG, "an output map needs the pipelined sweeps");
    }
    rsv_status s = B->setup(bad_cell);
    if (s != RSV_OK) {
        delete B;
        return s;
    }
    *out = B;
    return RSV_OK;
}
