// Hilbert space-filling-curve keys of points and grid cells, the equal-count
// cut of the curve into parts, and the partition-quality measures
// (Space-filling Partitioning Method section: Hilbert orders, the table-driven
// algorithm, Algorithm "Space-filling curve method", Partition Quality).
//
// Keys: each point of [0,1]^3 is scaled by 2^32 - 1 and truncated to three
// 32-bit coordinates; level l (l = 0 first) reads bit 31 - l of each (x
// weight 4, y 2, z 1 in the octant index) and walks the 24-state machine of
// the paper's ordering and orientation tables, emitting one base-8 digit per
// level, most significant first (a 3*levels-bit integer key).
//
// Partition: the cells in (key, index) order are cut into nparts runs of
// sizes differing by at most one (the cell of rank r goes to part
// floor(r nparts / n)).  Up to 4096 parts the cut is found without ordering the
// cells: a digit trie over (key, index) counts the cells under each prefix,
// most significant digit first, and follows only the prefixes that a cut goes
// through.  More parts take the order itself, from a stable least-significant-
// digit radix sort over the 3*levels key bits, 8 bits per pass: per-tile
// digit histograms, one exclusive scan, and a scatter in which each tile
// ranks its elements by digit with wave ballots (eight ballots match the
// lanes holding the same digit) so equal digits keep their input order.
#include "rsv_internal.h"

#include <algorithm>
#include <vector>

namespace {

// The paper's ordering table: per state, the digit of octant t in bits 3t..3t+2.
__constant__ uint32_t c_digits[24] = {
    0xab18f8u, 0xb374c8u, 0xb919d8u, 0xf8195au,
    0x2374ecu, 0x2b50fcu, 0x68197eu, 0xb13dc8u,
    0xf03d4au, 0x70754eu, 0xaa3c78u, 0xf350cau,
    0x283d7cu, 0x213decu, 0x7151ceu, 0xba7458u,
    0xfa505au, 0x6a507eu, 0xe23c6au, 0x3951dcu,
    0x38755cu, 0x62746eu, 0xe318eau, 0x6119eeu,
};
// The paper's orientation table: per state, the next state of octant t in bits 5t..5t+4.
__constant__ uint64_t c_next[24] = {
    0x000a220cc1ull, 0x094890a0e0ull, 0x14c40a5ecfull, 0xb428678ee3ull,
    0x6d8342308bull, 0x994055d196ull, 0x11923a9811ull, 0x3b0eb6b82aull,
    0x5a98e92128ull, 0x3c4c14a515ull, 0x529b063e27ull, 0x402cb2a5cbull,
    0xa3113530b2ull, 0x249a53cda8ull, 0x099ce89d77ull, 0x7d2757aa42ull,
    0x90c509c6b0ull, 0x7c6f174146ull, 0x834f145652ull, 0x28a7383483ull,
    0x63c64a51b0ull, 0x55dcfacaa9ull, 0x1917709ad6ull, 0x056f648aeeull,
};

enum { FLAG_RANGE = 16 };

__device__ inline uint32_t unit_to_u32(double c) { return (uint32_t)(c * 4294967295.0); }

__device__ inline uint64_t hilbert_key(const uint32_t *dig, const uint64_t *nxt, uint32_t u0, uint32_t u1,
                                       uint32_t u2, int levels)
{
    uint32_t st = 0;
    uint64_t k = 0;
    for (int l = 0; l < levels; ++l) {
        const int b = 31 - l;
        const uint32_t t = (((u0 >> b) & 1u) << 2) | (((u1 >> b) & 1u) << 1) | ((u2 >> b) & 1u);
        k = (k << 3) | ((dig[st] >> (3 * t)) & 7u);
        st = (uint32_t)((nxt[st] >> (5 * t)) & 31u);
    }
    return k;
}

// the two tables staged in LDS (per-lane state indices differ)
#define RSV_HSFC_TABLES                                   \
    __shared__ uint32_t s_dig[24];                        \
    __shared__ uint64_t s_nxt[24];                        \
    if (threadIdx.x < 24) {                               \
        s_dig[threadIdx.x] = c_digits[threadIdx.x];       \
        s_nxt[threadIdx.x] = c_next[threadIdx.x];         \
    }                                                     \
    __syncthreads();

__global__ __launch_bounds__(256) void k_hsfc_points(int64_t n, const double *__restrict__ xyz, int levels,
                                                     uint64_t *__restrict__ keys, int32_t *flags)
{
    RSV_HSFC_TABLES
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) {
        const double x = xyz[3 * e], y = xyz[3 * e + 1], z = xyz[3 * e + 2];
        if (!(x >= 0.0 && x <= 1.0 && y >= 0.0 && y <= 1.0 && z >= 0.0 && z <= 1.0)) {
            atomicOr(&flags[0], (int32_t)FLAG_RANGE);
            keys[e] = 0;
            continue;
        }
        keys[e] = hilbert_key(s_dig, s_nxt, unit_to_u32(x), unit_to_u32(y), unit_to_u32(z), levels);
    }
}

// keys of the grid's cells by block row: centroid ((i, j, k) + 1/2) / L with
// L the largest extent, so the cells stay cubes in [0,1)^3
__global__ __launch_bounds__(256) void k_hsfc_grid(Geo g, int levels, uint64_t *__restrict__ keys)
{
    RSV_HSFC_TABLES
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    const double L = (double)max(g.nx, max(g.ny, g.nz));
    for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < n; r += (int64_t)gridDim.x * 256) {
        const int i = (int)(r % g.nx), j = (int)((r / g.nx) % g.ny);
        const int kk = (int)(r / ((int64_t)g.nx * g.ny));
        const int k = (g.ordering == RSV_TOP_DOWN) ? g.nz - 1 - kk : kk;
        keys[r] = hilbert_key(s_dig, s_nxt, unit_to_u32(((double)i + 0.5) / L), unit_to_u32(((double)j + 0.5) / L),
                              unit_to_u32(((double)k + 0.5) / L), levels);
    }
}

// ---------------------------------------------------------------- radix sort
constexpr int RS_ITEMS = 16, RS_TILE = 256 * RS_ITEMS;

// per-tile histogram of the digit at `shift`, stored digit-major: hist[d * ntile + tile]
__global__ __launch_bounds__(256) void k_rs_hist(const uint64_t *__restrict__ keys, int64_t n, int shift,
                                                 uint32_t *__restrict__ hist, int ntile)
{
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * RS_TILE;
    for (int it = 0; it < RS_ITEMS; ++it) {
        const int64_t e = base + it * 256 + threadIdx.x;
        if (e < n) atomicAdd(&h[(uint32_t)(keys[e] >> shift) & 255u], 1u);
    }
    __syncthreads();
    hist[(int64_t)threadIdx.x * ntile + blockIdx.x] = h[threadIdx.x];
}

// exclusive scan of a tile of 4096 counts (16 consecutive per thread); the
// tile total goes to sums[tile]
__global__ __launch_bounds__(256) void k_scan_tile(const uint32_t *__restrict__ in, uint32_t *__restrict__ out,
                                                   int64_t m, uint32_t *__restrict__ sums)
{
    __shared__ uint32_t t[256];
    const int64_t base = (int64_t)blockIdx.x * RS_TILE + (int64_t)threadIdx.x * RS_ITEMS;
    uint32_t v[RS_ITEMS], s = 0;
#pragma unroll
    for (int q = 0; q < RS_ITEMS; ++q) {
        v[q] = (base + q < m) ? in[base + q] : 0u;
        s += v[q];
    }
    t[threadIdx.x] = s;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {   // inclusive scan of the thread totals
        const uint32_t a = ((int)threadIdx.x >= off) ? t[threadIdx.x - off] : 0u;
        __syncthreads();
        t[threadIdx.x] += a;
        __syncthreads();
    }
    uint32_t run = t[threadIdx.x] - s;
#pragma unroll
    for (int q = 0; q < RS_ITEMS; ++q) {
        if (base + q < m) out[base + q] = run;
        run += v[q];
    }
    if (threadIdx.x == 255) sums[blockIdx.x] = t[255];
}

__global__ __launch_bounds__(256) void k_scan_add(uint32_t *__restrict__ out, int64_t m,
                                                  const uint32_t *__restrict__ add)
{
    const int64_t base = (int64_t)blockIdx.x * RS_TILE;
    const uint32_t a = add[blockIdx.x];
    for (int q = threadIdx.x; q < RS_TILE; q += 256)
        if (base + q < m) out[base + q] += a;
}

// stable scatter of one digit pass; iin == nullptr: the indices are the positions
__global__ __launch_bounds__(256) void k_rs_scatter(const uint64_t *__restrict__ kin, const uint32_t *__restrict__ iin,
                                                    uint64_t *__restrict__ kout, uint32_t *__restrict__ iout,
                                                    int64_t n, int shift, const uint32_t *__restrict__ offs, int ntile)
{
    __shared__ uint32_t base_off[256];
    __shared__ uint32_t wcnt[4][256];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    base_off[tid] = offs[(int64_t)tid * ntile + blockIdx.x];
    for (int q = 0; q < 4; ++q) wcnt[q][tid] = 0;
    __syncthreads();
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    for (int it = 0; it < RS_ITEMS; ++it) {
        const int64_t e = (int64_t)blockIdx.x * RS_TILE + it * 256 + tid;
        const bool valid = e < n;
        const uint64_t key = valid ? kin[e] : 0ull;
        const uint32_t idx = valid ? (iin ? iin[e] : (uint32_t)e) : 0u;
        const uint32_t d = (uint32_t)(key >> shift) & 255u;
        uint64_t same = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint64_t ones = __ballot(valid && ((d >> b) & 1u));
            same &= ((d >> b) & 1u) ? ones : ~ones;
        }
        const uint64_t earlier = same & below;
        if (valid && earlier == 0ull) wcnt[w][d] = (uint32_t)__popcll(same);
        __syncthreads();
        if (valid) {
            uint32_t pos = base_off[d] + (uint32_t)__popcll(earlier);
            for (int q = 0; q < w; ++q) pos += wcnt[q][d];
            kout[pos] = key;
            iout[pos] = idx;
        }
        __syncthreads();
        base_off[tid] += wcnt[0][tid] + wcnt[1][tid] + wcnt[2][tid] + wcnt[3][tid];
        for (int q = 0; q < 4; ++q) wcnt[q][tid] = 0;
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_assign_parts(const uint32_t *__restrict__ idx, int64_t n, int32_t nparts,
                                                      int32_t *__restrict__ part)
{
    for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < n; r += (int64_t)gridDim.x * 256)
        part[idx[r]] = (int32_t)((r * (int64_t)nparts) / n);
}

// ---------------------------------------------------------------- the cut by a digit trie
// A node stands for the cells that share a prefix of the word (key, index); its
// entries, one per value of the next digit, hold how many cells follow that
// digit.  Ranks are prefix sums of the counts, so an entry whose cells all lie
// in one part is a leaf with that part, and one that a cut goes through has a
// child node: at most nparts - 1 nodes per level, since a cut goes through one
// node of a level only.  Index digits follow the key's, so equal keys are cut
// in index order and every path ends.  A level without nodes costs two empty
// launches; nothing is read back.
//
// Each level that has nodes reads the keys once (8 bytes a cell) and the last
// pass writes the parts, against 4 x 32 bytes a cell and scattered writes for
// the sort of a 30-bit key, whose 0.8 GB of buffers were allocated and freed in
// every call: keys and cut of 33.5 M cells in grid order into 64 parts 4.23 ->
// 0.44 ms, of which the keys are 0.22 (there every cut falls on an octant and
// the root decides it; each further level that is reached adds about 0.06).
// Keys in no order, 30 M at 10 levels, 64 / 4096 parts, sort / trie in ms: spread
// over the cube 4.5 / 0.36, 4.5 / 2.3; 200 values in five crowds 3.3 / 1.0,
// 3.2 / 2.9; two values 2.3 / 0.67, 2.3 / 1.1.
constexpr int TRIE_PARTS = 4096;      // most parts the trie takes
constexpr int TRIE_TOP = 12;          // digit bits of the root
constexpr int TRIE_ROWS_BITS = 20;    // log2 of the most entries a level may have
constexpr int TRIE_MAXLEV = 12;       // 12 bits, then 51 of the key and 31 of the index by 8

struct Trie {
    int nlev;                         // levels, the root first
    int width[TRIE_MAXLEV];           // digit bits
    int shift[TRIE_MAXLEV];           // lowest bit of the digit in its word
    int of_index[TRIE_MAXLEV];        // the digit is the index's, not the key's
    int32_t *entry[TRIE_MAXLEV];      // [node][2^width]: part, or ~child node
    uint32_t *first;                  // [2][nparts]: rank of a node's first cell, by level parity
    uint32_t *nodes;                  // [nlev + 1]: nodes per level
    uint32_t *stray;                  // set when a key has bits above the ones its levels give it
    int kbits;
    uint32_t *count;                  // [node][2^width] of the level at hand; all zero between levels
};

__device__ __forceinline__ uint32_t trie_digit(const Trie &t, int l, uint64_t key, uint32_t idx)
{
    const uint64_t w = t.of_index[l] ? (uint64_t)idx : key;
    return (uint32_t)(w >> t.shift[l]) & ((1u << t.width[l]) - 1u);
}

// entry of (key, idx) at level `to`, or the leaf met before it
__device__ __forceinline__ int32_t trie_walk(const Trie &t, int to, uint64_t key, uint32_t idx)
{
    int32_t e = t.entry[0][trie_digit(t, 0, key, idx)];
    for (int l = 1; l <= to && e < 0; ++l)
        e = t.entry[l][((int64_t)~e << t.width[l]) + trie_digit(t, l, key, idx)];
    return e;
}

__global__ __launch_bounds__(256) void k_trie_reset(Trie t, int64_t words)
{
    const int64_t e0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
    for (int64_t e = e0; e < words; e += (int64_t)gridDim.x * 256) t.count[e] = 0;
    if (e0 <= t.nlev) t.nodes[e0] = e0 == 0 ? 1u : 0u;
    if (e0 == 0) t.first[0] = *t.stray = 0;
}

// The cells' counts at level l.  Cells in grid order change their leading
// digits rarely, so neighbouring lanes mostly count the same entry: the first
// lane of each run of equal entries adds the run's length.  Counts are gathered
// in LDS first: the root's 4096 entries one to one, a lower level's through a
// direct-mapped table of as many (entry, count) pairs, past which an entry goes
// whose place another one holds.  Keys in no order that crowd under a few cut
// prefixes would otherwise all meet at a few addresses in memory, about 5 ns an
// addition (30 M keys of two values at 10 levels, 64 parts: 176 ms, 0.67 with the
// table).
template <bool ROOT>
__global__ __launch_bounds__(512) void k_trie_count(Trie t, int l, int64_t n, const uint64_t *__restrict__ keys)
{
    __shared__ uint32_t h[1 << TRIE_TOP];
    __shared__ int32_t tag[ROOT ? 1 : 1 << TRIE_TOP];   // entry counted at a place, -1: none
    if (!ROOT && t.nodes[l] == 0) return;
    for (int e = threadIdx.x; e < 1 << TRIE_TOP; e += 512) {
        h[e] = 0;
        if (!ROOT) tag[e] = -1;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const uint64_t after = lane == 63 ? 0ull : ~0ull << (lane + 1);
    constexpr int U = 4;
    uint64_t above = 0;
    const int64_t stride = (int64_t)gridDim.x * 512;
    for (int64_t e0 = (int64_t)blockIdx.x * 512; e0 < n; e0 += U * stride) {   // whole waves stay together
        uint64_t key[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t e = e0 + u * stride + threadIdx.x;
            key[u] = e < n ? keys[e] : 0ull;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t e = e0 + u * stride + threadIdx.x;
            int32_t at = -1;   // entry counted (at most 2^20 of them)
            if (e < n) {
                if (ROOT) {
                    above |= key[u] >> t.kbits;
                    at = (int32_t)trie_digit(t, 0, key[u], (uint32_t)e);
                } else {
                    const int32_t w = trie_walk(t, l - 1, key[u], (uint32_t)e);
                    if (w < 0) at = (int32_t)(((uint32_t)~w << t.width[l]) + trie_digit(t, l, key[u], (uint32_t)e));
                }
            }
            const int32_t prev = __shfl_up(at, 1, 64);
            const bool head = lane == 0 || prev != at;
            const uint64_t heads = __ballot(head) & after;
            const uint32_t len = (uint32_t)((heads ? __ffsll((unsigned long long)heads) - 1 : 64) - lane);
            if (head && at >= 0) {
                if (ROOT) {
                    atomicAdd(&h[at], len);
                } else {
                    const uint32_t q = ((uint32_t)at * 2654435761u) >> (32 - TRIE_TOP);
                    int32_t who = tag[q];
                    if (who < 0) who = atomicCAS(&tag[q], -1, at);
                    if (who < 0 || who == at) atomicAdd(&h[q], len);
                    else atomicAdd(&t.count[at], len);
                }
            }
        }
    }
    if (ROOT && above) *t.stray = 1;
    __syncthreads();
    for (int e = threadIdx.x; e < 1 << TRIE_TOP; e += 512)
        if (h[e]) atomicAdd(&t.count[ROOT ? e : tag[e]], h[e]);
}

// Entries of a level from its counts, one workgroup per node: ranks by an
// exclusive scan, leaves and children; the counts are left zero.
__global__ __launch_bounds__(256) void k_trie_split(Trie t, int l, int64_t n, int64_t nparts)
{
    if (blockIdx.x >= t.nodes[l]) return;
    __shared__ uint32_t sums[256];
    const int bins = 1 << t.width[l], per = (bins + 255) / 256;
    uint32_t *c = t.count + ((int64_t)blockIdx.x << t.width[l]);
    int32_t *out = t.entry[l] + ((int64_t)blockIdx.x << t.width[l]);
    uint32_t s = 0;
    for (int q = 0; q < per; ++q) {
        const int b = (int)threadIdx.x * per + q;
        s += b < bins ? c[b] : 0u;
    }
    sums[threadIdx.x] = s;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const uint32_t a = (int)threadIdx.x >= off ? sums[threadIdx.x - off] : 0u;
        __syncthreads();
        sums[threadIdx.x] += a;
        __syncthreads();
    }
    int64_t r = (int64_t)t.first[(l & 1) * nparts + blockIdx.x] + (sums[threadIdx.x] - s);
    for (int q = 0; q < per; ++q) {
        const int b = (int)threadIdx.x * per + q;
        if (b >= bins) break;
        const int64_t k = c[b];
        c[b] = 0;
        const int64_t p0 = k ? (r * nparts) / n : 0, p1 = k ? ((r + k - 1) * nparts) / n : 0;
        int32_t v = (int32_t)p0;
        if (p0 != p1) {
            const uint32_t child = atomicAdd(&t.nodes[l + 1], 1u);
            t.first[((l + 1) & 1) * nparts + child] = (uint32_t)r;
            v = ~(int32_t)child;
        }
        out[b] = v;
        r += k;
    }
}

__global__ __launch_bounds__(256) void k_trie_assign(Trie t, int64_t n, const uint64_t *__restrict__ keys,
                                                     int32_t *__restrict__ part)
{
    constexpr int U = 4;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t e0 = (int64_t)blockIdx.x * 256 + threadIdx.x; e0 < n; e0 += U * stride) {
        uint64_t key[U];
#pragma unroll
        for (int u = 0; u < U; ++u) key[u] = e0 + u * stride < n ? keys[e0 + u * stride] : 0ull;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t e = e0 + u * stride;
            if (e < n) part[e] = trie_walk(t, t.nlev - 1, key[u], (uint32_t)e);
        }
    }
}

// ---------------------------------------------------------------- partition quality
// per part: cnt[p] = {|G_p|, f_p, b_p}; adjacency bit (p, q) set when a face
// joins parts p and q.  A face inside a part is counted by its lower cell.
__global__ __launch_bounds__(256) void k_quality(Geo g, const int32_t *__restrict__ part, int32_t nparts,
                                                 unsigned long long *__restrict__ cnt, uint32_t *__restrict__ adj,
                                                 int words, int32_t *flags)
{
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    const int lane = threadIdx.x & 63;
    for (int64_t r0 = (int64_t)blockIdx.x * 256; r0 < n; r0 += (int64_t)gridDim.x * 256) {
        const int64_t r = r0 + threadIdx.x;
        const bool valid = r < n;
        int p = valid ? part[r] : -1;
        if (valid && (p < 0 || p >= nparts)) {
            atomicOr(&flags[0], (int32_t)FLAG_RANGE);
            p = -1;
        }
        unsigned long long f = 0, b = 0;
        if (p >= 0) {
            const int i = (int)(r % g.nx), j = (int)((r / g.nx) % g.ny), kk = (int)(r / ((int64_t)g.nx * g.ny));
            const int k = (g.ordering == RSV_TOP_DOWN) ? g.nz - 1 - kk : kk;
            for (int s = 0; s < 7; ++s) {
                if (s == 3) continue;
                int di, dj, dk;
                dir_off(s, di, dj, dk);
                const int ii = i + di, jj = j + dj, k2 = k + dk;
                if (ii < 0 || ii >= g.nx || jj < 0 || jj >= g.ny || k2 < 0 || k2 >= g.nz) { ++f; continue; }
                const int64_t m = row_of(g, ii, jj, k2);
                const int q = part[m];
                if (q != p) {
                    ++f;
                    ++b;
                    if (q >= 0 && q < nparts) atomicOr(&adj[(int64_t)p * words + (q >> 5)], 1u << (q & 31));
                } else if (s > 3) {
                    ++f;   // +x, +y, +z neighbour in the same part: the shared face once
                }
            }
        }
        // one atomic per wave when the wave's cells share a part
        const int p0 = __shfl(p, 0);
        const bool uniform = __ballot(valid && p == p0) == __ballot(valid);
        if (uniform && p0 >= 0) {
            unsigned long long sf = f, sb = b, sc = valid ? 1ull : 0ull;
            for (int off = 32; off > 0; off >>= 1) {
                sf += __shfl_xor(sf, off);
                sb += __shfl_xor(sb, off);
                sc += __shfl_xor(sc, off);
            }
            if (lane == 0) {
                atomicAdd(&cnt[3 * (int64_t)p0], sc);
                atomicAdd(&cnt[3 * (int64_t)p0 + 1], sf);
                atomicAdd(&cnt[3 * (int64_t)p0 + 2], sb);
            }
        } else if (p >= 0) {
            atomicAdd(&cnt[3 * (int64_t)p], 1ull);
            atomicAdd(&cnt[3 * (int64_t)p + 1], f);
            atomicAdd(&cnt[3 * (int64_t)p + 2], b);
        }
    }
}

// per part: connectivity (set bits of its adjacency row) into cnt4[p] = {|G|, f, b, c}
__global__ __launch_bounds__(256) void k_quality_rows(const unsigned long long *__restrict__ cnt,
                                                      const uint32_t *__restrict__ adj, int words, int32_t nparts,
                                                      long long *__restrict__ per)
{
    for (int p = blockIdx.x * 256 + threadIdx.x; p < nparts; p += gridDim.x * 256) {
        long long c = 0;
        for (int q = 0; q < words; ++q) c += __popc(adj[(int64_t)p * words + q]);
        per[4 * (int64_t)p] = (long long)cnt[3 * (int64_t)p];
        per[4 * (int64_t)p + 1] = (long long)cnt[3 * (int64_t)p + 1];
        per[4 * (int64_t)p + 2] = (long long)cnt[3 * (int64_t)p + 2];
        per[4 * (int64_t)p + 3] = c;
    }
}

// the five measures from the per-part counts (one workgroup, fixed order)
__global__ __launch_bounds__(256) void k_quality_final(const long long *__restrict__ per, int32_t nparts, int64_t n,
                                                       double *__restrict__ q)
{
    __shared__ long long s_max[256], s_f[256], s_b[256], s_c[256];
    __shared__ double s_r[256], s_rsum[256];
    long long mx = 0, sf = 0, sb = 0, cm = 0;
    double rm = 0.0, rs = 0.0;
    for (int p = threadIdx.x; p < nparts; p += 256) {
        const long long sz = per[4 * (int64_t)p], f = per[4 * (int64_t)p + 1], b = per[4 * (int64_t)p + 2];
        const long long c = per[4 * (int64_t)p + 3];
        mx = max(mx, sz);
        sf += f;
        sb += b;
        cm = max(cm, c);
        const double r = f > 0 ? (double)b / (double)f : 0.0;
        rm = fmax(rm, r);
        rs += r;
    }
    const int t = threadIdx.x;
    s_max[t] = mx; s_f[t] = sf; s_b[t] = sb; s_c[t] = cm; s_r[t] = rm; s_rsum[t] = rs;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (t < off) {
            s_max[t] = max(s_max[t], s_max[t + off]);
            s_f[t] += s_f[t + off];
            s_b[t] += s_b[t + off];
            s_c[t] = max(s_c[t], s_c[t + off]);
            s_r[t] = fmax(s_r[t], s_r[t + off]);
            s_rsum[t] += s_rsum[t + off];
        }
        __syncthreads();
    }
    if (t == 0) {
        q[0] = (double)nparts * (double)s_max[0] / (double)n;
        q[1] = s_r[0];
        q[2] = (s_f[0] - s_b[0]) > 0 ? (double)s_b[0] / (double)(s_f[0] - s_b[0]) : 0.0;
        q[3] = s_rsum[0] / (double)nparts;
        q[4] = (double)s_c[0];
    }
}

int grid_for(int64_t n) { return (int)std::min<int64_t>(std::max<int64_t>((n + 255) / 256, 1), 16384); }

rsv_status flags_range_check(rsv_ctx *c, const char *what)
{
    int32_t f[2];
    RSV_HIP(c, hipMemcpyAsync(f, c->d_flags, sizeof(f), hipMemcpyDeviceToHost, c->stream));
    RSV_HIP(c, hipStreamSynchronize(c->stream));
    if (f[0] & FLAG_RANGE) return set_err(c, RSV_ERR_ARG, what);
    return RSV_OK;
}

// exclusive scan of m counts in place of out (out may equal in), recursing on tile sums
rsv_status scan_counts(rsv_ctx *c, const uint32_t *in, uint32_t *out, int64_t m, std::vector<void *> &tmp)
{
    const int64_t ntile = (m + RS_TILE - 1) / RS_TILE;
    uint32_t *sums = nullptr;
    rsv_status s = dev_alloc(c, (void **)&sums, (size_t)ntile * sizeof(uint32_t));
    if (s != RSV_OK) return s;
    tmp.push_back(sums);
    hipLaunchKernelGGL(k_scan_tile, dim3((unsigned)ntile), dim3(256), 0, c->stream, in, out, m, sums);
    RSV_LAUNCH(c);
    if (ntile > 1) {
        s = scan_counts(c, sums, sums, ntile, tmp);
        if (s != RSV_OK) return s;
        hipLaunchKernelGGL(k_scan_add, dim3((unsigned)ntile), dim3(256), 0, c->stream, out, m, sums);
        RSV_LAUNCH(c);
    }
    return RSV_OK;
}

// The cut by the trie.  The context keeps the workspace: at most 2^20 entries a level
// below the root and as many counts, 48 MB for the longest word, 63 + 31 bits in
// 12 levels.  Every call waits for its last kernel, so the next one, on whatever
// stream, finds it idle.
// *stray: some key has bits above its 3*levels, which the sort's whole bytes
// count in part; those keys are left to it.
rsv_status trie_partition(rsv_ctx *c, int64_t n, const uint64_t *keys, int levels, int32_t nparts, int32_t *part,
                          uint32_t *stray)
{
    Trie t{};
    t.kbits = 3 * levels;
    int pbits = 0, ibits = 0;
    while (((int64_t)1 << pbits) < nparts) ++pbits;
    while (((int64_t)1 << ibits) < n) ++ibits;
    const int w = std::min(TRIE_TOP, TRIE_ROWS_BITS - pbits);   // 8 to 12 bits below the root
    int kbits = 3 * levels, top = std::min(kbits, TRIE_TOP);
    auto level = [&](int width, int shift, int of_index) {
        t.width[t.nlev] = width;
        t.shift[t.nlev] = shift;
        t.of_index[t.nlev] = of_index;
        ++t.nlev;
    };
    level(top, kbits - top, 0);
    for (int left = kbits - top; left > 0;) {
        const int q = std::min(w, left);
        left -= q;
        level(q, left, 0);
    }
    for (int left = ibits; left > 0;) {
        const int q = std::min(w, left);
        left -= q;
        level(q, left, 1);
    }
    const int64_t rows = std::max<int64_t>(1, nparts - 1);
    int64_t words = 0, cnt = 0, at[TRIE_MAXLEV];
    for (int l = 0; l < t.nlev; ++l) {
        const int64_t e = (l ? rows : 1) << t.width[l];
        at[l] = words;
        words += e;
        cnt = std::max(cnt, e);
    }
    const int64_t total = words + cnt + 2 * (int64_t)nparts + TRIE_MAXLEV + 2;
    if (total > c->trie_cap) {
        dev_free(c->d_trie);
        c->d_trie = nullptr;
        c->trie_cap = 0;
        rsv_status s = dev_alloc(c, (void **)&c->d_trie, (size_t)total * 4);
        if (s != RSV_OK) return s;
        c->trie_cap = total;
    }
    for (int l = 0; l < t.nlev; ++l) t.entry[l] = c->d_trie + at[l];
    t.count = (uint32_t *)(c->d_trie + words);
    t.first = t.count + cnt;
    t.nodes = t.first + 2 * nparts;
    t.stray = t.nodes + TRIE_MAXLEV + 1;
    hipLaunchKernelGGL(k_trie_reset, dim3((unsigned)std::min<int64_t>((cnt + 255) / 256, 1024)), dim3(256), 0, c->stream,
                       t, cnt);
    const unsigned nb = (unsigned)std::min<int64_t>((n + 2047) / 2048, 1024);
    for (int l = 0; l < t.nlev; ++l) {
        if (l == 0) hipLaunchKernelGGL(k_trie_count<true>, dim3(nb), dim3(512), 0, c->stream, t, l, n, keys);
        else hipLaunchKernelGGL(k_trie_count<false>, dim3(nb), dim3(512), 0, c->stream, t, l, n, keys);
        hipLaunchKernelGGL(k_trie_split, dim3((unsigned)(l ? rows : 1)), dim3(256), 0, c->stream, t, l, n,
                           (int64_t)nparts);
        RSV_LAUNCH(c);
    }
    hipLaunchKernelGGL(k_trie_assign, dim3((unsigned)std::min<int64_t>((n + 1023) / 1024, 8192)), dim3(256), 0, c->stream,
                       t, n, keys, part);
    RSV_LAUNCH(c);
    RSV_HIP(c, hipMemcpyAsync(stray, t.stray, sizeof(uint32_t), hipMemcpyDeviceToHost, c->stream));
    RSV_HIP(c, hipStreamSynchronize(c->stream));
    return RSV_OK;
}

struct Tmp {
    std::vector<void *> p;
    ~Tmp() { for (void *q : p) dev_free(q); }
};

}  // namespace

extern "C" {

rsv_status rsv_hsfc_keys(rsv_ctx *c, int64_t n, const double *coords, int32_t levels, uint64_t *keys)
{
    if (!c || n < 0 || (n > 0 && (!coords || !keys))) return set_err(c, RSV_ERR_ARG, "bad argument");
    if (levels < 1 || levels > 21) return set_err(c, RSV_ERR_ARG, "levels must be in [1, 21]");
    if (n == 0) return RSV_OK;
    rsv_status s = flags_reset(c);
    if (s != RSV_OK) return s;
    hipLaunchKernelGGL(k_hsfc_points, dim3(grid_for(n)), dim3(256), 0, c->stream, n, coords, levels, keys, c->d_flags);
    RSV_LAUNCH(c);
    return flags_range_check(c, "a coordinate is outside [0, 1] or not a number");
}

rsv_status rsv_grid_hsfc_keys(rsv_grid *g, int32_t levels, uint64_t *keys)
{
    if (!g || !keys) return set_err(g ? g->ctx : nullptr, RSV_ERR_ARG, "NULL argument");
    rsv_ctx *c = g->ctx;
    if (levels < 1 || levels > 21) return set_err(c, RSV_ERR_ARG, "levels must be in [1, 21]");
    hipLaunchKernelGGL(k_hsfc_grid, dim3(grid_for(g->ncell)), dim3(256), 0, c->stream, g->geo, levels, keys);
    RSV_LAUNCH(c);
    RSV_HIP(c, hipStreamSynchronize(c->stream));
    return RSV_OK;
}

rsv_status rsv_hsfc_partition(rsv_ctx *c, int64_t n, const uint64_t *keys, int32_t levels, int32_t nparts,
                              int32_t *part)
{
    if (!c || n < 0 || (n > 0 && (!keys || !part))) return set_err(c, RSV_ERR_ARG, "bad argument");
    if (levels < 1 || levels > 21) return set_err(c, RSV_ERR_ARG, "levels must be in [1, 21]");
    if (nparts < 1) return set_err(c, RSV_ERR_ARG, "nparts must be >= 1");
    if (n > ((int64_t)1 << 31)) return set_err(c, RSV_ERR_ARG, "at most 2^31 keys");
    if (n == 0) return RSV_OK;
    // Up to 4096 parts a node of the trie keeps at least 8 digit bits within
    // 2^20 entries a level.  Each level reads all keys once, and more parts mean
    // fewer bits and more levels: for 30 M keys in five crowds at 10 levels the sort
    // and the trie take 3.25 and 2.9 ms at 4096 parts, 3.23 and 3.2 at 8192, 3.24
    // and 4.3 at 16384 (sorted keys: 3.95 and 0.75, 0.80, 0.94).
    // The sort reads its own copies after its first pass, so part may lie on keys;
    // the trie reads keys while it writes part.
    const uintptr_t k0 = (uintptr_t)keys, p0 = (uintptr_t)part;
    const bool apart = p0 + (uintptr_t)n * 4 <= k0 || k0 + (uintptr_t)n * 8 <= p0;
    if (nparts <= TRIE_PARTS && apart) {
        uint32_t stray = 0;
        const rsv_status st = trie_partition(c, n, keys, levels, nparts, part, &stray);
        // few cells in many parts: the sort's 24 bytes a cell may still fit
        if (st != RSV_ERR_OOM && (st != RSV_OK || !stray)) return st;
    }
    const int64_t ntile = (n + RS_TILE - 1) / RS_TILE;
    Tmp t;
    uint64_t *k2[2] = {nullptr, nullptr};
    uint32_t *i2[2] = {nullptr, nullptr}, *hist = nullptr;
    rsv_status s = RSV_OK;
    for (int q = 0; q < 2 && s == RSV_OK; ++q) {
        s = dev_alloc(c, (void **)&k2[q], (size_t)n * sizeof(uint64_t));
        if (s == RSV_OK) { t.p.push_back(k2[q]); s = dev_alloc(c, (void **)&i2[q], (size_t)n * sizeof(uint32_t)); }
        if (s == RSV_OK) t.p.push_back(i2[q]);
    }
    if (s == RSV_OK) s = dev_alloc(c, (void **)&hist, (size_t)ntile * 256 * sizeof(uint32_t));
    if (s != RSV_OK) return s;
    t.p.push_back(hist);
    const int bits = 3 * levels, passes = (bits + 7) / 8;
    const uint64_t *kin = keys;
    const uint32_t *iin = nullptr;
    for (int ps = 0; ps < passes; ++ps) {
        const int shift = 8 * ps;
        hipLaunchKernelGGL(k_rs_hist, dim3((unsigned)ntile), dim3(256), 0, c->stream, kin, n, shift, hist, (int)ntile);
        RSV_LAUNCH(c);
        s = scan_counts(c, hist, hist, ntile * 256, t.p);
        if (s != RSV_OK) return s;
        hipLaunchKernelGGL(k_rs_scatter, dim3((unsigned)ntile), dim3(256), 0, c->stream, kin, iin, k2[ps & 1],
                           i2[ps & 1], n, shift, hist, (int)ntile);
        RSV_LAUNCH(c);
        kin = k2[ps & 1];
        iin = i2[ps & 1];
    }
    hipLaunchKernelGGL(k_assign_parts, dim3(grid_for(n)), dim3(256), 0, c->stream, iin, n, nparts, part);
    RSV_LAUNCH(c);
    RSV_HIP(c, hipStreamSynchronize(c->stream));
    return RSV_OK;
}

rsv_status rsv_partition_quality(rsv_grid *g, const int32_t *part, int32_t nparts, double *q, int64_t *per_part)
{
    if (!g || !part || !q) return set_err(g ? g->ctx : nullptr, RSV_ERR_ARG, "NULL argument");
    rsv_ctx *c = g->ctx;
    if (nparts < 1 || nparts > 16384) return set_err(c, RSV_ERR_ARG, "nparts must be in [1, 16384]");
    const int words = (nparts + 31) / 32;
    Tmp t;
    unsigned long long *cnt = nullptr;
    uint32_t *adj = nullptr;
    long long *per = nullptr;
    double *dq = nullptr;
    rsv_status s = dev_alloc(c, (void **)&cnt, (size_t)nparts * 3 * sizeof(unsigned long long));
    if (s == RSV_OK) { t.p.push_back(cnt); s = dev_alloc(c, (void **)&adj, (size_t)nparts * words * sizeof(uint32_t)); }
    if (s == RSV_OK) { t.p.push_back(adj); s = dev_alloc(c, (void **)&per, (size_t)nparts * 4 * sizeof(long long)); }
    if (s == RSV_OK) { t.p.push_back(per); s = dev_alloc(c, (void **)&dq, 5 * sizeof(double)); }
    if (s != RSV_OK) return s;
    t.p.push_back(dq);
    RSV_HIP(c, hipMemsetAsync(cnt, 0, (size_t)nparts * 3 * sizeof(unsigned long long), c->stream));
    RSV_HIP(c, hipMemsetAsync(adj, 0, (size_t)nparts * words * sizeof(uint32_t), c->stream));
    s = flags_reset(c);
    if (s != RSV_OK) return s;
    hipLaunchKernelGGL(k_quality, dim3(grid_for(g->ncell)), dim3(256), 0, c->stream, g->geo, part, nparts, cnt, adj,
                       words, c->d_flags);
    RSV_LAUNCH(c);
    hipLaunchKernelGGL(k_quality_rows, dim3(grid_for(nparts)), dim3(256), 0, c->stream, cnt, adj, words, nparts, per);
    RSV_LAUNCH(c);
    hipLaunchKernelGGL(k_quality_final, dim3(1), dim3(256), 0, c->stream, per, nparts, g->ncell, dq);
    RSV_LAUNCH(c);
    s = flags_range_check(c, "a part number is outside [0, nparts)");
    if (s != RSV_OK) return s;
    RSV_HIP(c, hipMemcpyAsync(q, dq, 5 * sizeof(double), hipMemcpyDeviceToHost, c->stream));
    if (per_part)
        RSV_HIP(c, hipMemcpyAsync(per_part, per, (size_t)nparts * 4 * sizeof(long long), hipMemcpyDeviceToHost,
                                  c->stream));
    RSV_HIP(c, hipStreamSynchronize(c->stream));
    return RSV_OK;
}

}  // extern "C"
