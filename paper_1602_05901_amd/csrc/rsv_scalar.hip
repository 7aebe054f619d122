// Scalar (one unknown per cell) 7-point systems, for the paper's Poisson
// Equation example: GMRES(30) with restricted additive Schwarz, overlap one,
// ILU(0) on every subdomain (Restricted Additive Schwarz Method subsection,
// RAS default parameters; Poisson Equation example).
//
// Storage: the seven coefficients of every row as seven row-ordered arrays
// coef[s][row] (slots -z,-y,-x,D,+x,+y,+z by cell direction), vectors in row
// order; the product is one thread per row with the residual, norm and dot
// epilogues of the block product.
//
// RAS: px x py x pz boxes (the first n mod p boxes one cell longer), each
// extended to Omega_s = the cells within graph distance `overlap` of the box
// (L1 distance on the lattice: faces, no edges or corners for overlap 1).
// The local ILU(0) in ascending global order has no fill on the 7-point graph
// (two neighbours of a cell are never neighbours), so D_c = a_cc -
// sum_{k lower} a_ck a_kc / D_k.  Two forms: tile columns, swept by waves that
// exchange faces (the default but for thin boxes that are long in x), and one
// workgroup per subdomain, which walks planes of x-chunks (each depending only on
// the plane before) with a barrier between them, for the factorisation and for
// both sweeps of an apply.  Only the owner of a cell writes its result.
#include "rsv_internal.h"

#include <algorithm>
#include <cmath>
#include <new>
#include <thread>
#include <vector>

namespace {

constexpr int SB = 256;          // product / assembly threads per block
constexpr int RAS_T = 1024;      // threads of a subdomain's workgroup (factorisation)
constexpr int APPLY_T = 512;     // threads of a subdomain's workgroup (apply: 8 slots of values per thread)

// row -> cell (inverse of row_of)
__host__ __device__ inline void cell_of_row(const Geo &g, int64_t r, int &i, int &j, int &k)
{
    i = (int)(r % g.nx);
    j = (int)((r / g.nx) % g.ny);
    const int kk = (int)(r / ((int64_t)g.nx * g.ny));
    k = (g.ordering == RSV_TOP_DOWN) ? g.nz - 1 - kk : kk;
}

__device__ inline double sblock_sum(double v, double *lds)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[w] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int q = 0; q < nw; ++q) s += lds[q];
    return s;
}

__global__ __launch_bounds__(SB) void k_sassemble(Geo g, const double *__restrict__ src, double *__restrict__ coef,
                                                  int32_t *flags)
{
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    const int64_t r = (int64_t)blockIdx.x * SB + threadIdx.x;
    if (r >= n) return;
    int i, j, k;
    cell_of_row(g, r, i, j, k);
    for (int s = 0; s < 7; ++s) {
        int di, dj, dk;
        dir_off(s, di, dj, dk);
        const bool inside = i + di >= 0 && i + di < g.nx && j + dj >= 0 && j + dj < g.ny && k + dk >= 0 && k + dk < g.nz;
        const double v = src[7 * r + s];
        if (!isfinite(v)) {
            atomicOr(&flags[0], (int32_t)FLAG_NAN);
            atomicMin(&flags[1], (int32_t)r);
        } else if (!inside && v != 0.0) {
            atomicOr(&flags[0], (int32_t)FLAG_PATTERN);
            atomicMin(&flags[1], (int32_t)r);
        }
        coef[s * n + r] = inside ? v : 0.0;
    }
}

template <int MODE, bool NT>
__global__ __launch_bounds__(SB) void k_sspmv(Geo g, const double *__restrict__ coef, const double *__restrict__ x,
                                              double *__restrict__ y, const double *__restrict__ aux,
                                              double alpha, double beta, double *__restrict__ partials)
{
    __shared__ double lds[SB / 64];
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    const int64_t r = (int64_t)blockIdx.x * SB + threadIdx.x;
    double r0 = 0.0, r1 = 0.0;
    if (r < n) {
        int i, j, k;
        cell_of_row(g, r, i, j, k);
        double acc = 0.0;
#pragma unroll
        for (int s = 0; s < 7; ++s) {
            int di, dj, dk;
            dir_off(s, di, dj, dk);
            const int a = i + di, b = j + dj, c = k + dk;
            if (a >= 0 && a < g.nx && b >= 0 && b < g.ny && c >= 0 && c < g.nz)
                acc += (NT ? __builtin_nontemporal_load(coef + s * n + r) : coef[s * n + r]) * x[(s == 3) ? r : row_of(g, a, b, c)];
        }
        double o = acc;
        if (MODE == SPMV_AXPBY) {
            o *= alpha;
            if (beta != 0.0) o += beta * y[r];
        } else if (MODE == SPMV_RESID) {
            o = aux[r] - acc;
        }
        y[r] = o;
        if (MODE == SPMV_RESID || MODE == SPMV_NORM) r0 = o * o;
        if (MODE == SPMV_DOT1 || MODE == SPMV_DOT2) r0 = aux[r] * o;
        if (MODE == SPMV_DOT2) r1 = o * o;
    }
    if (MODE >= SPMV_RESID) {
        const int K = (MODE == SPMV_DOT2) ? 2 : 1;
        const double s0 = sblock_sum(r0, lds);
        if (threadIdx.x == 0) partials[(int64_t)blockIdx.x * K] = s0;
        if (MODE == SPMV_DOT2) {
            const double s1 = sblock_sum(r1, lds);
            if (threadIdx.x == 0) partials[(int64_t)blockIdx.x * K + 1] = s1;
        }
    }
}

// ---------------------------------------------------------------- RAS
// A subdomain is walked in chunks of SW consecutive x-cells: chunk (c, j, k)
// of the extended box [ex0, ex1) x [ey0, ey1) x [ez0, ez1) holds the cells
// x = ex0 + SW c + t (t < SW) of grid row (ey0 + j, ez0 + k).  The lower
// neighbours of its cells (x - 1 of slot 0, y - 1, z - 1) lie in chunks
// (c-1, j, k), (c, j-1, k) and (c, j, k-1), so chunk plane P = c + j + k
// depends only on plane P - 1, and one thread solves the slots of a chunk in
// x order: a topological order of the same triangular dependencies as the
// cell hyperplanes, with the same arithmetic per cell.  Only chunks holding
// an Omega_s cell are stored; a slot outside Omega_s (x beyond the extended
// box, or an edge or corner of it) has zero couplings, a zero pivot inverse
// and the value zero.
//
// Chunk arrays (grouped by subdomain, then by plane, inside a plane by
// (k, j, c)): row0 = row of slot 0; mask = bit t: slot t in Omega_s, bit
// OWN_SHIFT + t: slot t owned by the subdomain; nlo[q] = position inside
// plane P - 1 of the (c, j, k-1), (c, j-1, k), (c-1, j, k) chunk and nhi[q] =
// position inside plane P + 1 of the (c+1, j, k), (c, j+1, k), (c, j, k+1)
// chunk, or -1.  Slot arrays: l[q] = a_ck / D_k (q = -z, -y, -x), u[q] = a_cm
// (q = +x, +y, +z), dinv = 1 / D_c, y = the sweeps' values; slot t of the
// chunk at position p of plane P is element SW pl[P] + t n_P + p (n_P chunks
// in the plane), so one slot of a plane's chunks is one contiguous row.
constexpr int SW = 8;
constexpr int OWN_SHIFT = 16;

struct SRasDev {
    int64_t nitem;                     // chunks over all subdomains
    const int32_t *row0, *mask, *nlo, *nhi;
    double *l, *u, *dinv, *y;          // SW * nitem elements each (l and u: three arrays)
    const int64_t *pl;                 // pl[pl_off[s] + P]: first chunk of plane P of subdomain s
    const int32_t *pl_off, *pl_cnt;
};

__device__ constexpr int LO_SLOT[3] = {0, 1, 2};   // -z, -y, -x
__device__ constexpr int HI_SLOT[3] = {4, 5, 6};   // +x, +y, +z

// D_c = a_cc - sum over lower neighbours k in Omega_s of (a_ck / D_k) a_kc,
// plane by plane (the planes before P are final when P starts)
__global__ __launch_bounds__(RAS_T) void k_sras_factor(Geo g, const double *__restrict__ coef, SRasDev d,
                                                       int32_t *flags)
{
    const int64_t n = (int64_t)g.nx * g.ny * g.nz, ns = SW * d.nitem;
    const int s = blockIdx.x, np = d.pl_cnt[s];
    const int64_t *pl = d.pl + d.pl_off[s];
    for (int P = 0; P < np; ++P) {
        const int64_t f = pl[P], cnt = pl[P + 1] - f;
        const int64_t fm = P > 0 ? pl[P - 1] : f, cm = f - fm;                  // plane P - 1
        const int64_t fp = pl[P + 1];                                          // plane P + 1
        for (int64_t p = threadIdx.x; p < cnt; p += RAS_T) {
            const int64_t q = f + p;
            const int64_t r0 = d.row0[q];
            const int m = d.mask[q];
            int32_t lo[3], hi[3];
            int lm[3], hm[3];
            int64_t lr[2];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                lo[a] = d.nlo[a * d.nitem + q];
                hi[a] = d.nhi[a * d.nitem + q];
                lm[a] = lo[a] >= 0 ? d.mask[fm + lo[a]] : 0;
                hm[a] = hi[a] >= 0 ? d.mask[fp + hi[a]] : 0;
            }
            lr[0] = lo[0] >= 0 ? d.row0[fm + lo[0]] : 0;
            lr[1] = lo[1] >= 0 ? d.row0[fm + lo[1]] : 0;
            // x - 1 of slot 0: slot SW - 1 of chunk lo[2]
            bool xl = lo[2] >= 0 && ((lm[2] >> (SW - 1)) & 1);
            double dxl = xl ? d.dinv[SW * fm + (SW - 1) * cm + lo[2]] : 0.0;
            for (int t = 0; t < SW; ++t) {
                const int64_t e = SW * f + t * cnt + p;
                if (!((m >> t) & 1)) {
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        d.l[a * ns + e] = 0.0;
                        d.u[a * ns + e] = 0.0;
                    }
                    d.dinv[e] = 0.0;
                    xl = false;
                    continue;
                }
                const int64_t r = r0 + t;
                double dd = coef[3 * n + r];
#pragma unroll
                for (int a = 0; a < 2; ++a) {            // -z, -y: slot t of chunks lo[0], lo[1]
                    double lv = 0.0;
                    if (lo[a] >= 0 && ((lm[a] >> t) & 1)) {
                        const double a_ck = coef[LO_SLOT[a] * n + r];
                        const double a_kc = coef[(6 - LO_SLOT[a]) * n + lr[a] + t];
                        lv = a_ck * d.dinv[SW * fm + t * cm + lo[a]];
                        dd -= lv * a_kc;
                    }
                    d.l[a * ns + e] = lv;
                }
                {                                        // -x: slot t - 1, or chunk lo[2]
                    double lv = 0.0;
                    if (xl) {
                        lv = coef[LO_SLOT[2] * n + r] * dxl;
                        dd -= lv * coef[(6 - LO_SLOT[2]) * n + r - 1];
                    }
                    d.l[2 * ns + e] = lv;
                }
                const bool up[3] = {t < SW - 1 ? (((m >> (t + 1)) & 1) != 0) : (hi[0] >= 0 && (hm[0] & 1)),
                                    hi[1] >= 0 && ((hm[1] >> t) & 1), hi[2] >= 0 && ((hm[2] >> t) & 1)};
#pragma unroll
                for (int a = 0; a < 3; ++a) d.u[a * ns + e] = up[a] ? coef[HI_SLOT[a] * n + r] : 0.0;
                double di;
                if (!(fabs(dd) > 1e-300) || !isfinite(dd)) {
                    atomicOr(&flags[0], (int32_t)FLAG_PIVOT);
                    atomicMin(&flags[1], (int32_t)r);
                    di = 0.0;
                } else {
                    di = 1.0 / dd;
                }
                d.dinv[e] = di;
                dxl = di;
                xl = true;
            }
        }
        __syncthreads();
    }
}

// ids of the chunk at position p of a plane (first chunk f, cnt chunks): row
// of slot 0, mask and three neighbour positions from nb; a position past the
// plane gets mask 0 and no neighbours
struct ChunkIds {
    int32_t r0, m, a, b, c;
};

__device__ inline ChunkIds chunk_ids(const SRasDev &d, const int32_t *nb, int64_t f, int64_t cnt, int64_t p)
{
    ChunkIds k{0, 0, -1, -1, -1};
    if (p < cnt) {
        const int64_t q = f + p;
        k.r0 = d.row0[q];
        k.m = d.mask[q];
        k.a = nb[q];
        k.b = nb[d.nitem + q];
        k.c = nb[2 * d.nitem + q];
    }
    return k;
}

// operands of one chunk's forward step: r, the z-1 and y-1 neighbours' values
// (plane P - 1: first chunk fm, cm chunks), the x-1 value of slot 0, l
struct FwdOps {
    double rv[SW], yz[SW], yy[SW], l[3][SW], yx;
};

__device__ inline void fwd_load(const SRasDev &d, const double *rin, const ChunkIds &k, int64_t f, int64_t cnt,
                                int64_t p, int64_t fm, int64_t cm, FwdOps &o)
{
    const int64_t ns = SW * d.nitem;
    const bool live = p < cnt;
#pragma unroll
    for (int t = 0; t < SW; ++t) {
        const int64_t e = SW * f + t * cnt + p;
        o.rv[t] = ((k.m >> t) & 1) ? rin[k.r0 + t] : 0.0;
        o.yz[t] = k.a >= 0 ? d.y[SW * fm + t * cm + k.a] : 0.0;
        o.yy[t] = k.b >= 0 ? d.y[SW * fm + t * cm + k.b] : 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) o.l[a][t] = live ? __builtin_nontemporal_load(d.l + a * ns + e) : 0.0;
    }
    o.yx = k.c >= 0 ? d.y[SW * fm + (SW - 1) * cm + k.c] : 0.0;
}

__device__ inline void fwd_solve(const SRasDev &d, int64_t f, int64_t cnt, int64_t p, const FwdOps &o)
{
    if (p >= cnt) return;
    double v = o.yx;
#pragma unroll
    for (int t = 0; t < SW; ++t) {
        double w = o.rv[t];
        w -= o.l[0][t] * o.yz[t];
        w -= o.l[1][t] * o.yy[t];
        w -= o.l[2][t] * v;
        d.y[SW * f + t * cnt + p] = w;
        v = w;
    }
}

// operands of one chunk's backward step: its forward values, the y+1 and z+1
// neighbours' results (plane P + 1: first chunk fp, cp chunks), the x+1
// result of slot SW - 1, u and the pivot inverses
struct BwdOps {
    double yv[SW], zy[SW], zz[SW], u[3][SW], di[SW], zx;
};

__device__ inline void bwd_load(const SRasDev &d, const ChunkIds &k, int64_t f, int64_t cnt, int64_t p, int64_t fp,
                                int64_t cp, BwdOps &o)
{
    const int64_t ns = SW * d.nitem;
    const bool live = p < cnt;
#pragma unroll
    for (int t = 0; t < SW; ++t) {
        const int64_t e = SW * f + t * cnt + p;
        o.yv[t] = live ? d.y[e] : 0.0;
        o.zy[t] = k.b >= 0 ? d.y[SW * fp + t * cp + k.b] : 0.0;
        o.zz[t] = k.c >= 0 ? d.y[SW * fp + t * cp + k.c] : 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) o.u[a][t] = live ? __builtin_nontemporal_load(d.u + a * ns + e) : 0.0;
        o.di[t] = live ? __builtin_nontemporal_load(d.dinv + e) : 0.0;
    }
    o.zx = k.a >= 0 ? d.y[SW * fp + k.a] : 0.0;
}

__device__ inline void bwd_solve(const SRasDev &d, double *zout, const ChunkIds &k, int64_t f, int64_t cnt,
                                 int64_t p, const BwdOps &o)
{
    if (p >= cnt) return;
    double v = o.zx;
#pragma unroll
    for (int t = SW - 1; t >= 0; --t) {
        double w = o.yv[t];
        w -= o.u[0][t] * v;
        w -= o.u[1][t] * o.zy[t];
        w -= o.u[2][t] * o.zz[t];
        w *= o.di[t];
        d.y[SW * f + t * cnt + p] = w;
        if ((k.m >> (OWN_SHIFT + t)) & 1) zout[k.r0 + t] = w;
        v = w;
    }
}

// forward y_c = r_c - sum_k l_ck y_k over the planes, then backward
// z_c = (y_c - sum_m u_cm z_m) / D_c in reverse; the owner of a cell writes z.
// A thread takes positions tid and tid + APPLY_T of every plane (and more on
// planes of over 2 APPLY_T chunks); their ids are read one plane ahead, and
// in the forward sweep the operands of both are loaded before either is
// solved, so a plane costs one round trip to memory.  The factors are
// streamed past the caches' retention (one slot of a plane's chunks is one
// contiguous row); r and z, which a thread reads and writes 8 bytes at a time
// along its chunk, and the sweeps' values, which the next plane reads, go
// through the caches (streaming r and z as well doubled the traffic).
__global__ __launch_bounds__(APPLY_T) void k_sras_apply(SRasDev d, const double *__restrict__ rin,
                                                        double *__restrict__ zout)
{
    const int s = blockIdx.x, np = d.pl_cnt[s], tid = threadIdx.x;
    const int64_t *pl = d.pl + d.pl_off[s];
    if (np <= 0) return;
    ChunkIds n0 = chunk_ids(d, d.nlo, pl[0], pl[1] - pl[0], tid);
    ChunkIds n1 = chunk_ids(d, d.nlo, pl[0], pl[1] - pl[0], tid + APPLY_T);
    for (int P = 0; P < np; ++P) {
        const int64_t f = pl[P], cnt = pl[P + 1] - f;
        const int64_t fm = P > 0 ? pl[P - 1] : f, cm = f - fm;
        const ChunkIds k0 = n0, k1 = n1;
        if (P + 1 < np) {
            const int64_t fn = pl[P + 1], cn = pl[P + 2] - fn;
            n0 = chunk_ids(d, d.nlo, fn, cn, tid);
            n1 = chunk_ids(d, d.nlo, fn, cn, tid + APPLY_T);
        }
        FwdOps o0, o1;
        fwd_load(d, rin, k0, f, cnt, tid, fm, cm, o0);
        fwd_load(d, rin, k1, f, cnt, tid + APPLY_T, fm, cm, o1);
        fwd_solve(d, f, cnt, tid, o0);
        fwd_solve(d, f, cnt, tid + APPLY_T, o1);
        for (int64_t p = tid + 2 * APPLY_T; p < cnt; p += APPLY_T) {
            const ChunkIds k = chunk_ids(d, d.nlo, f, cnt, p);
            fwd_load(d, rin, k, f, cnt, p, fm, cm, o0);
            fwd_solve(d, f, cnt, p, o0);
        }
        __syncthreads();
    }
    n0 = chunk_ids(d, d.nhi, pl[np - 1], pl[np] - pl[np - 1], tid);
    n1 = chunk_ids(d, d.nhi, pl[np - 1], pl[np] - pl[np - 1], tid + APPLY_T);
    for (int P = np - 1; P >= 0; --P) {
        const int64_t f = pl[P], cnt = pl[P + 1] - f;
        const int64_t fp = pl[P + 1], cp = P + 1 < np ? pl[P + 2] - fp : 0;
        const ChunkIds k0 = n0, k1 = n1;
        if (P > 0) {
            const int64_t fn = pl[P - 1], cn = f - fn;
            n0 = chunk_ids(d, d.nhi, fn, cn, tid);
            n1 = chunk_ids(d, d.nhi, fn, cn, tid + APPLY_T);
        }
        BwdOps o;                      // one chunk at a time: two would not fit the registers
        bwd_load(d, k0, f, cnt, tid, fp, cp, o);
        bwd_solve(d, zout, k0, f, cnt, tid, o);
        if (tid + APPLY_T < cnt) {
            bwd_load(d, k1, f, cnt, tid + APPLY_T, fp, cp, o);
            bwd_solve(d, zout, k1, f, cnt, tid + APPLY_T, o);
        }
        for (int64_t p = tid + 2 * APPLY_T; p < cnt; p += APPLY_T) {
            const ChunkIds k = chunk_ids(d, d.nhi, f, cnt, p);
            bwd_load(d, k, f, cnt, p, fp, cp, o);
            bwd_solve(d, zout, k, f, cnt, p, o);
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------- RAS by pipelined tile columns
// Every subdomain's extended box, padded to whole 8 x 8 tiles, has a place of
// its own in an auxiliary tile-lane grid (SX x SY boxes of GX x GY cells, EZ
// layers), as the block systems' boxes do, and one wave sweeps one tile column
// at a time: lane (i, j) walks up its column skewed by i + j steps, so a step's
// 64 cells lie on one hyperplane.  A step reads its neighbours' previous results
// from LDS and costs one LDS round trip and three dependent multiply-adds, so
// the wave needs no helper waves: its factors, its right-hand side and its face
// words are loaded ST_AHEAD steps early into registers.  Tiles exchange faces
// through epoch-tagged words and are handed out by a ticket in topological order
// inside their boxes, so a tile waits only on tiles that run already, and every
// wait is bounded.
//
// Against one workgroup per subdomain (above) this fills the chip from a few
// subdomains: 27 boxes of 88^3 are 3267 tile columns.  One apply at 256^3 in 27
// boxes 3.48 -> 0.57 ms (2.8 TB/s of its 80 + 8 bytes a cell); what bounds it
// is the pipeline's fill, 21 anti-diagonals of tiles per box.
//
// The local matrices are zero outside Omega_s, where values are zero too.  r is
// read from and z written to the caller's order a layer of the tile at a time,
// eight runs of 64 bytes, and an LDS ring of 16 layers delays a lane's value by
// its i + j steps (the 64 cells of a step are 64 separate lines there: 130 us
// more to read r and 180 to write z at 256^3).
// Steps loaded ahead, and waves (tile columns at a time) per CU.  A tile falls
// behind its upstream neighbours until their face words are there when it loads
// them, so a longer lead is a longer pipeline (loads return in order: faces
// loaded later than the factors would only wait for them), and more columns in
// flight queue behind one another: at 256^3 in 27 boxes, forward / backward us,
// 4 waves with a lead of 4, 6, 8 steps 264/301, 280/317, 307/343; 2 waves
// 360/362; 6 waves 273/321; 8 waves with a lead of 8 335/377.
constexpr int ST_AHEAD = 4;
constexpr int ST_WAVES = 4;

struct STBox {
    int32_t x0, x1, y0, y1, z0, z1, ex, ey, ez;   // core and the extended box's origin
};

struct STDev {
    Geo a, g;                    // auxiliary grid, the matrix's grid
    int32_t btx, bty, SX, nsub, ov;
    const STBox *box;
    double *l;                   // [row][3][64]: a_ck / D_k toward -z, -y, -x
    double *u;                   // [row][4][64]: a_cm toward +x, +y, +z; 1 / D_c
    double *y;                   // [row][64]
};

// the column of a box's cell (x, y): its grid column, the range [klo, khi) of its layers
// in Omega_s and [olo, ohi) of those the box owns (all empty outside Omega_s)
struct STColumn {
    int gx, gy, ez, klo, khi, olo, ohi;
};
__device__ inline STColumn st_column(const STDev &d, const STBox &q, int x, int y)
{
    STColumn c{0, 0, q.ez, 0, 0, 0, 0};
    const int gx = q.ex + x, gy = q.ey + y;
    const int dx = gx < q.x0 ? q.x0 - gx : (gx >= q.x1 ? gx - q.x1 + 1 : 0);
    const int dy = gy < q.y0 ? q.y0 - gy : (gy >= q.y1 ? gy - q.y1 + 1 : 0);
    const int64_t rest = (int64_t)d.ov - dx - dy;
    if (x < 0 || y < 0 || gx >= d.g.nx || gy >= d.g.ny || rest < 0) return c;
    c.gx = gx;
    c.gy = gy;
    c.klo = (int)max((int64_t)0, q.z0 - rest) - q.ez;
    c.khi = (int)min((int64_t)d.g.nz, q.z1 + rest) - q.ez;
    if (dx == 0 && dy == 0) {
        c.olo = q.z0 - q.ez;
        c.ohi = q.z1 - q.ez;
    }
    return c;
}

// The layers [klo, khi) of the columns toward -y, -x, +x, +y of a box's cell (x, y).
struct STNear {
    int klo[4], khi[4];
};
__device__ inline STNear st_near(const STDev &d, const STBox &q, int x, int y)
{
    const int dx[4] = {0, -1, 1, 0}, dy[4] = {-1, 0, 0, 1};
    STNear m;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const STColumn c = st_column(d, q, x + dx[e], y + dy[e]);
        const bool in = x + dx[e] < 8 * d.btx && y + dy[e] < 8 * d.bty;
        m.klo[e] = in ? c.klo : 0;
        m.khi[e] = in ? c.khi : 0;
    }
    return m;
}

// factors of layer k of column c, cell (X, Y) (those it depends on are final)
__device__ inline void st_factor_cell(const STDev &d, const STColumn &c, const STNear &m, int X, int Y, int k,
                                      const double *__restrict__ coef, int32_t *flags)
{
    const int64_t n = (int64_t)d.g.nx * d.g.ny * d.g.nz;
    const int64_t r = row_of(d.g, c.gx, c.gy, c.ez + k);
    const int64_t slot = slot_of(d.a, X, Y, k), e = (slot >> 6), la = slot & 63;
    double dd = coef[3 * n + r];
#pragma unroll
    for (int a = 0; a < 3; ++a) {        // -z, -y, -x
        const int dX = a == 2 ? -1 : 0, dY = a == 1 ? -1 : 0, dk = a == 0 ? -1 : 0;
        const bool in = a == 0 ? k > c.klo : k >= m.klo[a - 1] && k < m.khi[a - 1];
        double lv = 0.0;
        if (in) {
            const int64_t ns = slot_of(d.a, X + dX, Y + dY, k + dk);
            const double a_ck = coef[LO_SLOT[a] * n + r];
            const double a_kc = coef[(6 - LO_SLOT[a]) * n + row_of(d.g, c.gx + dX, c.gy + dY, c.ez + k + dk)];
            lv = a_ck * d.u[(ns >> 6) * 256 + 192 + (ns & 63)];
            dd -= lv * a_kc;
        }
        d.l[e * 192 + a * 64 + la] = lv;
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {        // +x, +y, +z
        const bool in = a == 2 ? k + 1 < c.khi : k >= m.klo[a + 2] && k < m.khi[a + 2];
        d.u[e * 256 + a * 64 + la] = in ? coef[HI_SLOT[a] * n + r] : 0.0;
    }
    double di = 0.0;
    if (!(fabs(dd) > 1e-300) || !isfinite(dd)) {
        atomicOr(&flags[0], (int32_t)FLAG_PIVOT);
        atomicMin(&flags[1], (int32_t)r);
    } else {
        di = 1.0 / dd;
    }
    d.u[e * 256 + 192 + la] = di;
}

// One hyperplane p of every box's factorisation (the planes before p are final): a wave
// per tile that it meets.  d0: first row of the launch.
__global__ __launch_bounds__(SB) void k_st_factor(STDev d, PlaneTiles t, int p, int d0, const double *__restrict__ coef,
                                                  int32_t *flags)
{
    const int w = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)));
    const int box = w / t.row;
    int bx, by, i, j;
    if (box >= d.nsub || !plane_tile(t, w - box * t.row, d0 + (int)blockIdx.y, bx, by)) return;
    const int q = p - 8 * (bx + by);
    if (q < 0 || q >= d.a.nz + 14) return;
    lane_ij((int)(threadIdx.x & 63), i, j);
    const STBox b = d.box[box];
    const int x = 8 * bx + i, y = 8 * by + j, k = q - i - j;
    const STColumn c = st_column(d, b, x, y);
    if (k < c.klo || k >= c.khi) return;
    st_factor_cell(d, c, st_near(d, b, x, y), 8 * (box % d.SX * d.btx) + x, 8 * (box / d.SX * d.bty) + y, k, coef, flags);
}

// All hyperplanes of one box of at most 16 tiles: a workgroup per box, a wave per tile,
// a barrier between planes.  A plane costs 1 to 3 us, a launch per plane 4 and more: set-up
// of one column of 50000 cells 204 -> 49 ms, 64 x 64 x 64 in 8 x 8 x 8 boxes 1.02 -> 0.48.
__global__ __launch_bounds__(1024) void k_st_factor_box(STDev d, int nplane, const double *__restrict__ coef, int32_t *flags)
{
    const int T = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), box = blockIdx.x;
    int i, j;
    lane_ij((int)(threadIdx.x & 63), i, j);
    const int bx = T % d.btx, by = T / d.btx;
    const STBox b = d.box[box];
    const int x = 8 * bx + i, y = 8 * by + j, k0 = x + y;
    const int X = 8 * (box % d.SX * d.btx) + x, Y = 8 * (box / d.SX * d.bty) + y;
    const STColumn c = st_column(d, b, x, y);
    const STNear m = st_near(d, b, x, y);
    for (int p = 0; p < nplane; ++p) {
        const int k = p - k0;
        if (k >= c.klo && k < c.khi) st_factor_cell(d, c, m, X, Y, k, coef, flags);
        __syncthreads();
    }
}

struct STSweep {
    const int32_t *tile_order;
    uint64_t *ticket;
    uint64_t ticket_base;
    uint64_t *face;              // [tile][nz + 7][x: 16 words, y: 16 words]
    uint32_t epoch;
    int32_t *flags;
    uint64_t wait_limit;
};

// DIR 0: y = L^-1 r, v the caller's r.  DIR 1: z = U^-1 y, v the caller's z.
// Step t of a tile: lane (i, j) is at k = t - (i + j) (DIR 0) or nz - 1 - (t -
// (14 - i - j)) (DIR 1), on row t mod nz or (nz + 13 - t) mod nz.  Lanes whose k
// is out of range load the nearest in-range lane's entry, so a step touches only
// the lines it needs and every load is unconditional.
template <int DIR>
__global__ __launch_bounds__(64) void k_st_sweep(STDev d, STSweep a, double *__restrict__ v)
{
    __shared__ double lds[80];   // 64 results, then the x and the y face's 8 values
    __shared__ double ring[16 * 64];   // layer k of r (DIR 0) or z (DIR 1) in entry k mod 16
    uint32_t *ldw = (uint32_t *)lds;
    constexpr int NF = DIR == 0 ? 3 : 4;
    const int nz = d.a.nz, NT = d.a.ntx * d.a.nty, nsteps = nz + 14, L = threadIdx.x;
    const int64_t frow = (int64_t)(nz + 7) * 32, plane = (int64_t)d.g.nx * d.g.ny;
    int li, lj;
    lane_ij(L, li, lj);
    const int dd = DIR == 0 ? li + lj : 14 - li - lj;       // step at which the lane's column starts
    // where the lane's x and y neighbour values are (indices into lds)
    const int ax = DIR == 0 ? (li > 0 ? ij_lane(li - 1, lj) : 64 + lj) : (li < 7 ? ij_lane(li + 1, lj) : 64 + lj);
    const int ay = DIR == 0 ? (lj > 0 ? ij_lane(li, lj - 1) : 72 + li) : (lj < 7 ? ij_lane(li, lj + 1) : 72 + li);
    // face words: lane q < 32 holds half (q >> 3) & 1 of entry q & 7 of the x (q < 16) or y face
    const int fe = L & 7, fh = (L >> 3) & 1, fy = (L >> 4) & 1;
    const bool flane = L < 32;
    const int fdst = 128 + 16 * fy + 2 * fe + fh;                                          // incoming, 32-bit index
    const int fsrc = 2 * (fy ? ij_lane(fe, DIR == 0 ? 7 : 0) : ij_lane(DIR == 0 ? 7 : 0, fe)) + fh;   // outgoing
    const int fk_in = DIR == 0 ? fe : 7 - fe, fk_out = DIR == 0 ? 7 + fe : 14 - fe;
    const int lq = L & 31;
    struct Pre {
        double f[NF], v;
        uint64_t w;
    };
    bool over = false;   // a wait gave up: the flag is set, no wait lasts any more
    for (;;) {
        uint64_t tk = 0;
        if (L == 0) tk = atomicAdd((unsigned long long *)a.ticket, 1ull) - a.ticket_base;
        tk = __shfl(tk, 0, 64);
        if (tk >= (uint64_t)NT) break;
        const int T = a.tile_order[DIR == 0 ? (int)tk : NT - 1 - (int)tk];
        const int tx = T % d.a.ntx, ty = T / d.a.ntx, bx = tx % d.btx, by = ty % d.bty;
        const bool has_x = DIR == 0 ? bx > 0 : bx < d.btx - 1, has_y = DIR == 0 ? by > 0 : by < d.bty - 1;
        const bool out_x = DIR == 0 ? bx < d.btx - 1 : bx > 0, out_y = DIR == 0 ? by < d.bty - 1 : by > 0;
        const bool fin = flane && (fy ? has_y : has_x), fout = flane && (fy ? out_y : out_x);
        // a tile without that neighbour reads its own row, an in-range dummy
        const int Tn = !fin ? T : (DIR == 0 ? (fy ? T - d.a.ntx : T - 1) : (fy ? T + d.a.ntx : T + 1));
        const uint64_t *fsp = a.face + Tn * frow + lq;
        uint64_t *fdp = a.face + T * frow + lq;
        const int box = ty / d.bty * d.SX + tx / d.btx;   // the last places of the square of boxes may be empty
        const STColumn c = box < d.nsub ? st_column(d, d.box[box], 8 * bx + li, 8 * by + lj) : STColumn{0, 0, 0, 0, 0, 0, 0};
        // the caller's entry of layer k is cv[k * ck]
        const bool td = d.g.ordering == RSV_TOP_DOWN;
        const int64_t ck = td ? -plane : plane;
        double *cv = v + row_of(d.g, c.gx, c.gy, c.ez);
        const int64_t rowbase = (int64_t)T * nz;
        auto issue = [&](Pre &R, int t) {
            const int tc = t < nsteps ? t : nsteps - 1;
            const int dmin = DIR == 0 ? max(tc - nz + 1, 0) : max(14 - tc, 0);
            const int dmax = DIR == 0 ? min(tc, 14) : min(13 - tc + nz, 14);
            const int Ls = min(max(L, lane_first(dmin)), lane_first(dmax + 1) - 1);
            const int64_t row = rowbase + (DIR == 0 ? wrap_nz(tc, nz) : wrap_nz(nz + 13 - tc, nz));
            const double *f = (DIR == 0 ? d.l : d.u) + row * (NF * 64) + Ls;
#pragma unroll
            for (int q = 0; q < NF; ++q) R.f[q] = __builtin_nontemporal_load(f + q * 64);
            if constexpr (DIR == 0) {
                R.v = cv[min(max(tc, c.klo), max(c.khi - 1, c.klo)) * ck];   // layer t; taken up dd steps later
            } else {
                R.v = d.y[row * 64 + Ls];
            }
            const int tr = t < nz + 7 ? t : nz + 6;
            R.w = face_ld(fsp + (int64_t)tr * 32);
        };
        double last = 0.0;
        auto step = [&](Pre &R, int t) {
            // the faces this step's boundary lanes need
            const bool need = fin && (unsigned)(t - fk_in) < (unsigned)nz;
            uint64_t w = R.w;
            if (!over && __ballot(need && (uint32_t)(w >> 32) != a.epoch) != 0ull) {
                const uint64_t t0 = wall_clock64();
                uint32_t n = 0;
                for (;;) {
                    if (need) w = face_ld(fsp + (int64_t)t * 32);
                    if (__ballot(need && (uint32_t)(w >> 32) != a.epoch) == 0ull) break;
                    if (spin_guard(a.flags, t0, n, a.wait_limit)) {
                        over = true;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
            }
            if (flane) ldw[fdst] = need ? (uint32_t)w : 0u;
            if constexpr (DIR == 0) ring[(t & 15) * 64 + L] = R.v;
            __atomic_signal_fence(__ATOMIC_SEQ_CST);   // one wave: its LDS accesses complete in program order
            const double vx = lds[ax], vy = lds[ay];
            const int k = DIR == 0 ? t - dd : nz - 1 - (t - dd);
            const bool in = k >= c.klo && k < c.khi;
            double o = DIR == 0 ? ring[((t - dd) & 15) * 64 + L] : R.v;
            if constexpr (DIR == 0) {
                o -= R.f[0] * last;
                o -= R.f[1] * vy;
                o -= R.f[2] * vx;
            } else {
                o -= R.f[0] * vx;
                o -= R.f[1] * vy;
                o -= R.f[2] * last;
                o *= R.f[3];
            }
            o = in ? o : 0.0;
            last = o;
            lds[L] = o;
            if constexpr (DIR == 1) ring[(k & 15) * 64 + L] = o;
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            const uint32_t fo = ldw[fsrc];
            if (fout && (unsigned)(t - fk_out) < (unsigned)nz)
                face_st(fdp + (int64_t)(t - 7) * 32, ((uint64_t)a.epoch << 32) | fo);
            if constexpr (DIR == 0) {
                if (k >= 0 && k < nz) d.y[(rowbase + wrap_nz(t, nz)) * 64 + L] = o;
            } else {
                // every lane has passed layer kz
                const int kz = nz - 1 - (t - 14);
                const double z = ring[(kz & 15) * 64 + L];
                if (kz >= c.olo && kz < c.ohi) cv[kz * ck] = z;
            }
        };
        Pre R[ST_AHEAD];
#pragma unroll
        for (int q = 0; q < ST_AHEAD; ++q) issue(R[q], q);
        // steps past the last have no lane in range
        for (int t = 0; t < nsteps; t += ST_AHEAD)
#pragma unroll
            for (int q = 0; q < ST_AHEAD; ++q) {
                step(R[q], t + q);
                issue(R[q], t + q + ST_AHEAD);
            }
    }
}

int64_t box_start(int64_t b, int64_t len, int64_t p)
{
    const int64_t base = len / p, rem = len % p;
    return b * base + std::min(b, rem);
}

struct SRas final : PcImpl {
    rsv_matrix *M = nullptr;
    rsv_ctx *c = nullptr;
    int nsub = 0;
    int64_t nitem = 0, ncell = 0, tplanes = 0;   // chunks, Omega_s cells, plane table entries
    std::vector<void *> mem;
    SRasDev d{};

    ~SRas() override
    {
        if (c) (void)hipStreamSynchronize(c->stream);
        for (void *p : mem) dev_free(p);
    }
    // per chunk: row, mask, 3 + 3 neighbour positions (32 B); per slot: 3 + 3
    // coefficients, the pivot inverse and the working value (64 B)
    int64_t bytes() const override { return nitem * (32 + SW * 64) + tplanes * 8 + nsub * 8; }
    // per Omega_s cell: 3 + 3 coefficients and the pivot inverse (56 B), r in,
    // y out, y in (24 B); z out once per grid cell; per chunk its 32 B
    int64_t apply_bytes() const override
    {
        const Geo &G = M->g->geo;
        return ncell * 80 + (int64_t)G.nx * G.ny * G.nz * 8 + nitem * 32;
    }

    template <class T> rsv_status alloc(T **p, size_t n)
    {
        rsv_status s = dev_alloc(c, (void **)p, n * sizeof(T));
        if (s == RSV_OK) mem.push_back(*p);
        return s;
    }

    rsv_status apply(const double *r, double *z) override
    {
        ProfScope ps(c, RSV_K_RAS);
        hipLaunchKernelGGL(k_sras_apply, dim3(nsub), dim3(APPLY_T), 0, c->stream, d, r, z);
        RSV_LAUNCH(c);
        return RSV_OK;
    }

    rsv_status setup(int px, int py, int pz, int ov, int64_t *bad_cell)
    {
        const Geo &G = M->g->geo;
        const int64_t nx = G.nx, ny = G.ny, nz = G.nz;
        if (nx * ny * nz >= ((int64_t)1 << 31)) return set_err(c, RSV_ERR_ARG, "scalar RAS: more than 2^31 cells");
        nsub = px * py * pz;
        // per subdomain: its box, extended box, chunk count and first chunk
        struct Box { int64_t x0, x1, y0, y1, z0, z1, ex0, ex1, ey0, ey1, ez0, ez1, nc, count, first; int nplane; };
        std::vector<Box> B(nsub);
        for (int s = 0; s < nsub; ++s) {
            Box &b = B[s];
            const int sx = s % px, sy = (s / px) % py, sz = s / (px * py);
            b.x0 = box_start(sx, nx, px); b.x1 = box_start(sx + 1, nx, px);
            b.y0 = box_start(sy, ny, py); b.y1 = box_start(sy + 1, ny, py);
            b.z0 = box_start(sz, nz, pz); b.z1 = box_start(sz + 1, nz, pz);
            b.ex0 = std::max<int64_t>(0, b.x0 - ov); b.ex1 = std::min<int64_t>(nx, b.x1 + ov);
            b.ey0 = std::max<int64_t>(0, b.y0 - ov); b.ey1 = std::min<int64_t>(ny, b.y1 + ov);
            b.ez0 = std::max<int64_t>(0, b.z0 - ov); b.ez1 = std::min<int64_t>(nz, b.z1 + ov);
            b.nc = (b.ex1 - b.ex0 + SW - 1) / SW;
            b.nplane = (int)(b.nc + (b.ey1 - b.ey0) + (b.ez1 - b.ez0) - 2);
        }
        auto dist = [](int64_t v, int64_t lo, int64_t hi) { return v < lo ? lo - v : (v >= hi ? v - hi + 1 : 0); };
        // the cells of grid row (j, k) inside Omega_s: one x-interval [lo, hi)
        auto row_range = [&](const Box &b, int64_t j, int64_t k, int64_t &lo, int64_t &hi) {
            const int64_t rest = dist(j, b.y0, b.y1) + dist(k, b.z0, b.z1);
            if (rest > ov) return false;
            lo = std::max(b.ex0, b.x0 - (ov - rest));
            hi = std::min(b.ex1, b.x1 + (ov - rest));
            return hi > lo;
        };
        int64_t total = 0, cells = 0;
        tplanes = 0;
        for (int s = 0; s < nsub; ++s) {
            Box &b = B[s];
            int64_t cnt = 0, lo, hi;
            for (int64_t k = b.ez0; k < b.ez1; ++k)
                for (int64_t j = b.ey0; j < b.ey1; ++j)
                    if (row_range(b, j, k, lo, hi)) {
                        cnt += (hi - 1 - b.ex0) / SW - (lo - b.ex0) / SW + 1;
                        cells += hi - lo;
                    }
            b.count = cnt;
            b.first = total;
            total += cnt;
            tplanes += b.nplane + 1;
        }
        nitem = total;
        ncell = cells;
        std::vector<int32_t> row0(total), mask(total), nlo(3 * total), nhi(3 * total);
        std::vector<int64_t> pl(tplanes);
        std::vector<int32_t> pl_off(nsub), pl_cnt(nsub);
        {
            int64_t off = 0;
            for (int s = 0; s < nsub; ++s) {
                pl_off[s] = (int32_t)off;
                pl_cnt[s] = B[s].nplane;
                off += B[s].nplane + 1;
            }
        }
        auto build = [&](int s) {
            const Box &b = B[s];
            const int64_t NC = b.nc, EY = b.ey1 - b.ey0, EZ = b.ez1 - b.ez0;
            const int NP = b.nplane;
            std::vector<int64_t> start(NP + 1, 0);
            int64_t lo, hi;
            for (int64_t k = 0; k < EZ; ++k)
                for (int64_t j = 0; j < EY; ++j)
                    if (row_range(b, b.ey0 + j, b.ez0 + k, lo, hi))
                        for (int64_t cc = (lo - b.ex0) / SW; cc <= (hi - 1 - b.ex0) / SW; ++cc) start[cc + j + k + 1]++;
            for (int P = 0; P < NP; ++P) start[P + 1] += start[P];
            int64_t *plp = pl.data() + pl_off[s];
            for (int P = 0; P <= NP; ++P) plp[P] = b.first + start[P];
            std::vector<int32_t> pos((size_t)(NC * EY * EZ), -1);
            std::vector<int64_t> fill(NP, 0);
            for (int64_t k = 0; k < EZ; ++k)                  // (k, j, c) order inside every plane
                for (int64_t j = 0; j < EY; ++j) {
                    if (!row_range(b, b.ey0 + j, b.ez0 + k, lo, hi)) continue;
                    const int64_t gj = b.ey0 + j, gk = b.ez0 + k;
                    const bool own_row = gj >= b.y0 && gj < b.y1 && gk >= b.z0 && gk < b.z1;
                    for (int64_t cc = (lo - b.ex0) / SW; cc <= (hi - 1 - b.ex0) / SW; ++cc) {
                        const int64_t P = cc + j + k, p = fill[P]++;
                        pos[(k * EY + j) * NC + cc] = (int32_t)p;
                        const int64_t q = b.first + start[P] + p;
                        const int64_t x = b.ex0 + cc * SW;
                        row0[q] = (int32_t)row_of(G, (int)x, (int)gj, (int)gk);
                        int mk = 0;
                        for (int t = 0; t < SW; ++t) {
                            const int64_t i = x + t;
                            if (i < lo || i >= hi) continue;
                            mk |= 1 << t;
                            if (own_row && i >= b.x0 && i < b.x1) mk |= 1 << (OWN_SHIFT + t);
                        }
                        mask[q] = mk;
                    }
                }
            auto at = [&](int64_t cc, int64_t j, int64_t k) -> int32_t {
                if (cc < 0 || cc >= NC || j < 0 || j >= EY || k < 0 || k >= EZ) return -1;
                return pos[(k * EY + j) * NC + cc];
            };
            for (int64_t k = 0; k < EZ; ++k)
                for (int64_t j = 0; j < EY; ++j)
                    for (int64_t cc = 0; cc < NC; ++cc) {
                        const int32_t p = at(cc, j, k);
                        if (p < 0) continue;
                        const int64_t q = b.first + start[cc + j + k] + p;
                        nlo[0 * total + q] = at(cc, j, k - 1);
                        nlo[1 * total + q] = at(cc, j - 1, k);
                        nlo[2 * total + q] = at(cc - 1, j, k);
                        nhi[0 * total + q] = at(cc + 1, j, k);
                        nhi[1 * total + q] = at(cc, j + 1, k);
                        nhi[2 * total + q] = at(cc, j, k + 1);
                    }
        };
        {
            const int nth = (int)std::max(1u, std::min(16u, std::thread::hardware_concurrency()));
            std::vector<std::thread> th;
            for (int t = 0; t < nth; ++t)
                th.emplace_back([&, t] { for (int s = t; s < nsub; s += nth) build(s); });
            for (auto &x : th) x.join();
        }
        int32_t *drow0, *dmask, *dlo, *dhi, *dploff, *dplcnt;
        int64_t *dpl;
        double *dl, *du, *ddinv, *dy;
        const size_t nslot = (size_t)SW * total;
        rsv_status st = alloc(&drow0, (size_t)total);
        if (st == RSV_OK) st = alloc(&dmask, (size_t)total);
        if (st == RSV_OK) st = alloc(&dlo, (size_t)3 * total);
        if (st == RSV_OK) st = alloc(&dhi, (size_t)3 * total);
        if (st == RSV_OK) st = alloc(&dl, 3 * nslot);
        if (st == RSV_OK) st = alloc(&du, 3 * nslot);
        if (st == RSV_OK) st = alloc(&ddinv, nslot);
        if (st == RSV_OK) st = alloc(&dy, nslot);
        if (st == RSV_OK) st = alloc(&dpl, (size_t)tplanes);
        if (st == RSV_OK) st = alloc(&dploff, (size_t)nsub);
        if (st == RSV_OK) st = alloc(&dplcnt, (size_t)nsub);
        if (st != RSV_OK) return st;
        RSV_HIP(c, hipMemcpyAsync(drow0, row0.data(), total * 4, hipMemcpyHostToDevice, c->stream));
        RSV_HIP(c, hipMemcpyAsync(dmask, mask.data(), total * 4, hipMemcpyHostToDevice, c->stream));
        RSV_HIP(c, hipMemcpyAsync(dlo, nlo.data(), 3 * total * 4, hipMemcpyHostToDevice, c->stream));
        RSV_HIP(c, hipMemcpyAsync(dhi, nhi.data(), 3 * total * 4, hipMemcpyHostToDevice, c->stream));
        RSV_HIP(c, hipMemcpyAsync(dpl, pl.data(), tplanes * 8, hipMemcpyHostToDevice, c->stream));
        RSV_HIP(c, hipMemcpyAsync(dploff, pl_off.data(), nsub * 4, hipMemcpyHostToDevice, c->stream));
        RSV_HIP(c, hipMemcpyAsync(dplcnt, pl_cnt.data(), nsub * 4, hipMemcpyHostToDevice, c->stream));
        d = SRasDev{total, drow0, dmask, dlo, dhi, dl, du, ddinv, dy, dpl, dploff, dplcnt};
        rsv_status fs = flags_reset(c);   // synchronises: the host arrays may be released after it
        if (fs != RSV_OK) return fs;
        {
            ProfScope ps(c, RSV_K_FACTOR);
            hipLaunchKernelGGL(k_sras_factor, dim3(nsub), dim3(RAS_T), 0, c->stream, G, M->d_coef, d, c->d_flags);
        }
        RSV_LAUNCH(c);
        return flags_check(c, bad_cell);
    }
};

// The tile-column form of the scalar RAS (and of BILU0: one subdomain).
struct STile final : PcImpl {
    rsv_matrix *M = nullptr;
    rsv_ctx *c = nullptr;
    STDev d{};
    int64_t ncell = 0, nbytes = 0;          // cells over all Omega_s
    int nplane = 0;
    std::vector<void *> mem;
    int32_t *tile_order = nullptr;
    uint64_t *face = nullptr;
    bool unfit = false;                     // the chunk form is the better one, or the boxes exceed the index range

    ~STile() override
    {
        if (c) (void)hipStreamSynchronize(c->stream);
        for (void *p : mem) dev_free(p);
    }
    int64_t bytes() const override { return nbytes; }
    // per Omega_s cell: 3 + 3 coefficients and the pivot inverse (56 B), r in,
    // y out, y in (24 B); z out once per grid cell
    int64_t apply_bytes() const override
    {
        const Geo &G = M->g->geo;
        return ncell * 80 + (int64_t)G.nx * G.ny * G.nz * 8;
    }
    template <class T> rsv_status alloc(T **p, int64_t n, bool zero)
    {
        rsv_status s = dev_alloc(c, (void **)p, (size_t)n * sizeof(T));
        if (s != RSV_OK) return s;
        mem.push_back(*p);
        nbytes += n * (int64_t)sizeof(T);
        if (zero) RSV_HIP(c, hipMemsetAsync(*p, 0, (size_t)n * sizeof(T), c->stream));
        return RSV_OK;
    }

    rsv_status setup(int px, int py, int pz, int ov, int64_t *bad_cell)
    {
        const Geo &G = M->g->geo;
        const int64_t nsub = (int64_t)px * py * pz;
        auto lo = [](int64_t v, int64_t o) { return (int32_t)std::max<int64_t>(0, v - o); };
        int EX = 1, EY = 1, EZ = 1;
        // extended box sizes, and the cells of Omega_s (at most the extended boxes')
        std::vector<STBox> B((size_t)nsub);
        for (int64_t s = 0; s < nsub; ++s) {
            const int64_t sx = s % px, sy = (s / px) % py, sz = s / ((int64_t)px * py);
            STBox &b = B[s];
            b.x0 = (int32_t)box_start(sx, G.nx, px); b.x1 = (int32_t)box_start(sx + 1, G.nx, px);
            b.y0 = (int32_t)box_start(sy, G.ny, py); b.y1 = (int32_t)box_start(sy + 1, G.ny, py);
            b.z0 = (int32_t)box_start(sz, G.nz, pz); b.z1 = (int32_t)box_start(sz + 1, G.nz, pz);
            b.ex = lo(b.x0, ov); b.ey = lo(b.y0, ov); b.ez = lo(b.z0, ov);
            const int ex = (int)std::min<int64_t>(G.nx, (int64_t)b.x1 + ov) - b.ex;
            const int ey = (int)std::min<int64_t>(G.ny, (int64_t)b.y1 + ov) - b.ey;
            const int ez = (int)std::min<int64_t>(G.nz, (int64_t)b.z1 + ov) - b.ez;
            EX = std::max(EX, ex); EY = std::max(EY, ey); EZ = std::max(EZ, ez);
            // columns at distance a + b from the box (a in x, b in y) are as high as its z range
            // widened by what is left of the overlap
            auto columns = [](int64_t lo_, int64_t hi_, int64_t nn, int64_t at) {
                return at == 0 ? hi_ - lo_ : (int64_t)(lo_ - at >= 0) + (hi_ - 1 + at < nn);
            };
            for (int64_t a = 0; a <= ov; ++a) {
                const int64_t nc = columns(b.x0, b.x1, G.nx, a);
                if (nc == 0) break;
                for (int64_t e = 0; a + e <= ov; ++e) {
                    const int64_t nr = columns(b.y0, b.y1, G.ny, e), rest = ov - a - e;
                    if (nr == 0) break;
                    ncell += nc * nr * (std::min<int64_t>(G.nz, b.z1 + rest) - std::max<int64_t>(0, b.z0 - rest));
                }
            }
        }
        d.btx = (EX + 7) / 8;
        d.bty = (EY + 7) / 8;
        int64_t SX = 1;
        while (SX * SX < nsub) ++SX;
        const int64_t SY = (nsub + SX - 1) / SX, slots = SX * d.btx * SY * d.bty * (int64_t)EZ * 64;
        // Small boxes pad much (64 slots per layer however few of its columns a
        // box has), but the tile columns stay ahead of the chunk form down to
        // single-cell boxes (64^3 in 64^3 boxes: 6.5 against 21 ms an apply; 96^3
        // in 31^3: 0.85 against 4.5).  They fall behind where a box is a few layers
        // thin and long in x, so that its diagonals of tiles are the chain (6.1 us a
        // diagonal, 0.375 a step; a tile occupies a wave for 7.2 us and its steps), while
        // the other form has a plane per eight cells of x (2.1 us a plane and 0.0135 a
        // chunk, a box per CU at a time).  These figures give each form's time within
        // about 25 % and the choice (apply, chunk form against tile columns, ms): 100000
        // x 1 x 1 52 and 153, in 64 boxes 0.87 and 2.5, 20000 x 8 x 1 11.2 and 30.4, 4096 x
        // 4096 x 1 in 64 x 64 boxes 5.4 and 8.3; in 4 x 4 boxes 6.8 and 7.1, one box 77 and
        // 14, 1024 x 1024 x 1 5.9 and 3.4.  The chunk form, with up to a fifth of the
        // memory, also takes what exceeds the slots' index range or the memory.
        const double planes = (EX + SW - 1) / SW + EY + EZ - 2, chunks = (double)((EX + SW - 1) / SW) * EY * EZ;
        const double t_chunk = (double)((nsub + c->num_cu - 1) / c->num_cu) * (2.1 * planes + 0.0135 * chunks);
        const double steps = 0.375 * (EZ + 14), rounds = std::ceil((double)slots / 64 / EZ / (ST_WAVES * c->num_cu));
        const double t_tile = std::max(6.1 * (d.btx + d.bty - 2) + steps, rounds > 1 ? rounds * (7.2 + steps) : 0.0);
        if (t_chunk < t_tile) {
            unfit = true;
            return RSV_OK;
        }
        if (3 * slots >= ((int64_t)1 << 31)) {
            unfit = true;
            return RSV_OK;
        }
        d.SX = (int32_t)SX;
        d.nsub = (int32_t)nsub;
        d.ov = ov;
        d.g = G;
        const int ntx = (int)(SX * d.btx), nty = (int)(SY * d.bty), NT = ntx * nty;
        d.a = Geo{8 * ntx, 8 * nty, EZ, ntx, nty, RSV_BOTTOM_UP, slots};
        nplane = 8 * d.btx + 8 * d.bty + EZ - 2;
        const int64_t rows = slots / 64;
        STBox *dbox = nullptr;
        rsv_status st = alloc(&dbox, nsub, false);
        if (st == RSV_OK) st = alloc(&d.l, rows * 192, true);
        if (st == RSV_OK) st = alloc(&d.u, rows * 256, true);
        if (st == RSV_OK) st = alloc(&d.y, rows * 64, true);
        if (st == RSV_OK) st = alloc(&tile_order, (int64_t)NT, false);
        if (st == RSV_OK) st = alloc(&face, (int64_t)NT * (EZ + 7) * 32, true);   // no word may carry a tag (epochs are never 0)
        if (st != RSV_OK) return st;
        d.box = dbox;
        // tiles by their diagonal inside the box
        std::vector<int32_t> ord(NT), at(d.btx + d.bty);
        for (int y = 0; y < d.bty; ++y)
            for (int x = 0; x < d.btx; ++x) at[x + y + 1] += (int32_t)(SX * SY);
        for (int q = 1; q < d.btx + d.bty; ++q) at[q] += at[q - 1];
        for (int y = 0, t = 0; y < nty; ++y)
            for (int x = 0, by = y % d.bty, bx = 0; x < ntx; ++x, ++t, bx = bx + 1 == d.btx ? 0 : bx + 1) ord[at[bx + by]++] = t;
        RSV_HIP(c, hipMemcpyAsync(dbox, B.data(), (size_t)nsub * sizeof(STBox), hipMemcpyHostToDevice, c->stream));
        RSV_HIP(c, hipMemcpyAsync(tile_order, ord.data(), (size_t)NT * sizeof(int32_t), hipMemcpyHostToDevice, c->stream));
        st = flags_reset(c);   // synchronises: the host arrays may be released after it
        if (st != RSV_OK) return st;
        {
            ProfScope ps(c, RSV_K_FACTOR);
            if (d.btx * d.bty <= 16)
                hipLaunchKernelGGL(k_st_factor_box, dim3((unsigned)nsub), dim3((unsigned)(64 * d.btx * d.bty)), 0, c->stream, d,
                                   nplane, M->d_coef, c->d_flags);
            else
                for (int p = 0; p < nplane; ++p) {
                    const PlaneTiles t = plane_tiles(p, EZ, d.btx, d.bty);
                    plane_launch(c, t, (int)nsub, [&](int d0, dim3 grid, dim3 blk) {
                        hipLaunchKernelGGL(k_st_factor, grid, blk, 0, c->stream, d, t, p, d0, M->d_coef, c->d_flags);
                    });
                }
        }
        RSV_LAUNCH(c);
        return flags_check(c, bad_cell);
    }

    rsv_status apply(const double *r, double *z) override
    {
        ProfScope ps(c, RSV_K_RAS);
        const int NT = d.a.ntx * d.a.nty;
        const int nw = std::min(NT, c->num_cu * ST_WAVES);
        auto args = [&]() {
            STSweep a{tile_order, c->d_tickets, c->ticket_base[0], face, c->epoch++, c->d_flags, c->wait_ticks};
            if (c->epoch == 0) c->epoch = 1;
            c->ticket_base[0] += (uint64_t)NT + nw;
            return a;
        };
        hipLaunchKernelGGL(k_st_sweep<0>, dim3(nw), dim3(64), 0, c->stream, d, args(), const_cast<double *>(r));
        RSV_LAUNCH(c);
        hipLaunchKernelGGL(k_st_sweep<1>, dim3(nw), dim3(64), 0, c->stream, d, args(), z);
        RSV_LAUNCH(c);
        return RSV_OK;
    }
};

}  // namespace

rsv_status launch_sspmv(rsv_ctx *c, const Geo &g, const double *coef, int mode, const double *x, double *y,
                        const double *aux, double alpha, double beta, int k0)
{
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    const int nb = (int)((n + SB - 1) / SB);
    if (mode >= SPMV_RESID) {
        rsv_status s = partials_reserve(c, (int64_t)nb * 2);
        if (s != RSV_OK) return s;
    }
    double *P = c->d_partials;
    const int tok = prof_begin(c, RSV_K_SPMV);
    const dim3 grid(nb), blk(SB);
    const bool nt = once_through(n, n * 56, STAYS_SCALAR);
#define L_SSPMV(M)                                                                                              \
    case M:                                                                                                     \
        if (nt)                                                                                                 \
            hipLaunchKernelGGL((k_sspmv<M, true>), grid, blk, 0, c->stream, g, coef, x, y, aux, alpha, beta, P);  \
        else                                                                                                    \
            hipLaunchKernelGGL((k_sspmv<M, false>), grid, blk, 0, c->stream, g, coef, x, y, aux, alpha, beta, P); \
        break;
    switch (mode) {
    L_SSPMV(SPMV_Y)
    L_SSPMV(SPMV_AXPBY)
    L_SSPMV(SPMV_RESID)
    L_SSPMV(SPMV_NORM)
    L_SSPMV(SPMV_DOT1)
    L_SSPMV(SPMV_DOT2)
    default: return set_err(c, RSV_ERR_ARG, "bad spmv mode");
    }
#undef L_SSPMV
    prof_end(c, tok);
    RSV_LAUNCH(c);
    if (mode >= SPMV_RESID && k0 >= 0) return launch_reduce(c, nb, mode == SPMV_DOT2 ? 2 : 1, k0);
    return RSV_OK;
}

rsv_status mat_spmv(rsv_matrix *M, int mode, const double *x, double *y, const double *aux, double alpha,
                    double beta, int k0)
{
    if (M->bs == 1) return launch_sspmv(M->g->ctx, M->g->geo, M->d_coef, mode, x, y, aux, alpha, beta, k0);
    return launch_spmv(M->g->ctx, M->g->geo, M->d_A, mode, x, y, aux, alpha, beta, k0);
}

int mat_spmv_blocks(rsv_matrix *M)
{
    const Geo &g = M->g->geo;
    return M->bs == 1 ? (int)(((int64_t)g.nx * g.ny * g.nz + SB - 1) / SB) : spmv_blocks(g);
}

rsv_status mat_in(rsv_matrix *M, const double *nat, double *v)
{
    if (M->bs == 1) return launch_copy(M->g->ctx, M->nv, nat, v);
    return launch_nat_to_tl(M->g->ctx, M->g->geo, nat, v);
}

rsv_status mat_out(rsv_matrix *M, const double *v, double *nat, double alpha, double beta)
{
    if (M->bs == 1) return launch_axpby(M->g->ctx, M->nv, alpha, v, beta, nat);
    return launch_tl_to_nat(M->g->ctx, M->g->geo, v, nat, alpha, beta);
}

rsv_status sras_create(rsv_matrix *A, const rsv_pc_params *p, PcImpl **out, int64_t *bad_cell)
{
    rsv_ctx *c = A->g->ctx;
    const Geo &G = A->g->geo;
    int px = 1, py = 1, pz = 1, ov = 0;      // BILU0 of a scalar matrix: one subdomain, no overlap
    if (p->type == RSV_PC_RAS) {
        px = p->ras_px; py = p->ras_py; pz = p->ras_pz; ov = p->ras_overlap;
        if (px < 1 || py < 1 || pz < 1 || px > G.nx || py > G.ny || pz > G.nz || ov < 0)
            return set_err(c, RSV_ERR_ARG, "bad RAS subdomain counts or overlap");
    }
    if (p->precision != RSV_FP64) return set_err(c, RSV_ERR_ARG, "scalar systems have FP64 preconditioners only");
    if (p->pipelined) {
        STile *T = new (std::nothrow) STile();
        if (!T) return set_err(c, RSV_ERR_OOM, "scalar RAS");
        T->M = A;
        T->c = c;
        rsv_status st = T->setup(px, py, pz, ov, bad_cell);
        if (st == RSV_OK && !T->unfit) {
            *out = T;
            return RSV_OK;
        }
        const bool unfit = T->unfit || st == RSV_ERR_OOM;
        delete T;
        if (!unfit) return st;
    }
    SRas *R = new (std::nothrow) SRas();
    if (!R) return set_err(c, RSV_ERR_OOM, "scalar RAS");
    R->M = A;
    R->c = c;
    rsv_status s = R->setup(px, py, pz, ov, bad_cell);
    if (s != RSV_OK) {
        delete R;
        return s;
    }
    *out = R;
    return RSV_OK;
}

extern "C" {

rsv_status rsv_matrix_assemble_scalar(rsv_grid *g, const double *coef, int32_t where, rsv_matrix **out)
{
    if (!g || !coef || !out) return set_err(g ? g->ctx : nullptr, RSV_ERR_ARG, "NULL argument");
    *out = nullptr;
    rsv_ctx *c = g->ctx;
    rsv_matrix *M = new (std::nothrow) rsv_matrix();
    if (!M) return set_err(c, RSV_ERR_OOM, "matrix");
    M->g = g;
    M->bs = 1;
    M->nv = g->ncell;
    rsv_status s = dev_alloc(c, (void **)&M->d_coef, (size_t)g->ncell * 7 * sizeof(double));
    if (s == RSV_OK) {
        M->bytes = g->ncell * 7 * (int64_t)sizeof(double);
        s = scalar_assemble_values(M, coef, where);
    }
    if (s != RSV_OK) {
        rsv_matrix_destroy(M);
        return s;
    }
    *out = M;
    return RSV_OK;
}

}  // extern "C"

rsv_status scalar_assemble_values(rsv_matrix *M, const double *coef, int32_t where)
{
    rsv_grid *g = M->g;
    rsv_ctx *c = g->ctx;
    const size_t bytes = (size_t)g->ncell * 7 * sizeof(double);
    const double *src = coef;
    double *stage = nullptr;
    if (where == RSV_MEM_HOST) {
        rsv_status s = dev_alloc(c, (void **)&stage, bytes);
        if (s != RSV_OK) return s;
        hipError_t e = hipMemcpyAsync(stage, coef, bytes, hipMemcpyHostToDevice, c->stream);
        if (e != hipSuccess) {
            dev_free(stage);
            return set_err(c, RSV_ERR_HIP, std::string("hipMemcpyAsync: ") + hipGetErrorString(e));
        }
        src = stage;
    } else if (where != RSV_MEM_DEVICE) {
        return set_err(c, RSV_ERR_ARG, "bad memory kind");
    }
    rsv_status s = flags_reset(c);
    if (s == RSV_OK) {
        hipLaunchKernelGGL(k_sassemble, dim3((unsigned)((g->ncell + SB - 1) / SB)), dim3(SB), 0, c->stream, g->geo, src,
                           M->d_coef, c->d_flags);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) s = set_err(c, RSV_ERR_HIP, std::string("kernel launch: ") + hipGetErrorString(e));
    }
    if (s == RSV_OK) s = flags_check(c, nullptr);
    if (stage) dev_free(stage);
    return s;
}
