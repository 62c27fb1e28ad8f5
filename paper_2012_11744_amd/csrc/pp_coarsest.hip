// pp_coarsest.hip -- the FP64 pseudo-inverse of the coarsest level's operator
// (gfx950), rebuilt on the device at every coefficient load.
//
// With K = -A + (s/n) 1 1^T positive definite (A is singular, constants in its
// null space; s is its largest diagonal entry), A^+ = (1/(s n)) 1 1^T - K^-1,
// everything over the active cells; with a diagonal term A - diag(sigma) is
// definite there and A^+ = -K^-1 with K = -A + diag(sigma).  Cells without an
// open face or diagonal term get zero rows and columns.
//
// K^-1 comes from block Gauss-Jordan elimination without pivoting (K is
// symmetric positive definite: its pivots are those of a Cholesky
// factorisation), 64 columns a step, one launch a step.  The chain of
// dependent pivots bounds it, not its 2 n^3 operations: a workgroup inverts
// the 64 x 64 pivot block with the matrix held in registers, one barrier per
// four pivots, and every workgroup does so redundantly, which spares each step
// a second launch and a round trip through memory.  Steps are out of place
// (two work matrices), so no workgroup reads what another writes.  The chain
// is halved where the cells have two colours (k_pinv_reduce).
//
// Measured: 26 us for up to 64 cells (17 of them the pivots, 1.03 us per four;
// pivot by pivot, with divisions and vector arithmetic, 32); 27 us a step above
// (41), 14 us to form the half-size matrix and 11 to expand it.  720 cells
// (144 x 80 x 32) take 185 us, against 510 without the two changes; the
// projection step there 1.16 ms, against 1.47, and 32 with a Cholesky
// factorisation on the host (29 ms of it).
#include <hip/hip_runtime.h>

#include "pp_internal.h"

namespace pp {

constexpr int PB = 64;                   // columns per elimination step
constexpr int PTHREADS = 256;            // 16 x 16 threads, 4 x 4 entries each
constexpr int PLD = PB + 2;              // LDS row
constexpr int CELLS_MAX = 1024;          // cells of a coarsest level

struct PinvArgs {
    Dims d;
    Bc bc;
    double ih2;
    const double *b[3];                  // FP64 face coefficients of the coarsest level
    const double *sg;                    // its sigma, or null
    int singular;                        // the constants on the active cells are the null space
    int n;                               // cells
    int m, np;                           // order of the eliminated matrix, rounded up to whole blocks
    int step;                            // elimination step (block column)
    int direct;                          // last step of an unreduced matrix: writes pinv
    const double *in;                    // np x np work matrix
    double *out;                         // np x np work matrix
    double *meta;                        // per cell: -A_cc if active, else 0; then M_COUNT scalars
    double *pinv;                        // n x n
    double *bad;                         // PINV_GOOD, PINV_BAD or PINV_ZERO
};

// scalars behind the cells' entries of meta
enum { M_SHIFT, M_GAMMA, M_INVN, M_SUMQ, M_COUNT };

// the links of one cell: their coefficients / h^2 and neighbours (-1: none)
struct Row {
    double w[6];
    int nb[6];
    double dg;                           // -A_cc; the cell is active if positive
};

__device__ __forceinline__ Row row_of(const PinvArgs &a, int c)
{
    Row r;
    const int nx = a.d.nx, ny = a.d.ny, nz = a.d.nz;
    const int k = c / (nx * ny), rem = c - k * nx * ny, j = rem / nx, i = rem - j * nx;
    const int q[3] = {i, j, k}, nn[3] = {nx, ny, nz}, st[3] = {1, nx, nx * ny};
    const int wall[3] = {a.bc.x, a.bc.y, a.bc.z};
    r.dg = 0.0;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        const int lo = q[m] > 0 ? c - st[m] : (wall[m] ? -1 : c + (nn[m] - 1) * st[m]);
        const int hi = q[m] < nn[m] - 1 ? c + st[m] : (wall[m] ? -1 : c - (nn[m] - 1) * st[m]);
        r.nb[2 * m] = lo;
        r.nb[2 * m + 1] = hi;
        r.w[2 * m] = lo < 0 ? 0.0 : a.b[m][c] * a.ih2;
        r.w[2 * m + 1] = hi < 0 ? 0.0 : a.b[m][hi] * a.ih2;
        r.dg += r.w[2 * m] + r.w[2 * m + 1];
    }
    if (a.sg)
        r.dg += a.sg[c];
    return r;
}

// sums (or the larger, for MAX0's first) of two values over the workgroup
template <bool MAX0, int NT>
__device__ __forceinline__ void reduce2(double &u, double &v, double (*red)[NT / 64])
{
    const int t = threadIdx.x;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double w = __shfl_xor(u, o, 64);
        u = MAX0 ? fmax(u, w) : u + w;
        v += __shfl_xor(v, o, 64);
    }
    if ((t & 63) == 0) {
        red[0][t >> 6] = u;
        red[1][t >> 6] = v;
    }
    __syncthreads();
    u = red[0][0];
    v = red[1][0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) {
        u = MAX0 ? fmax(u, red[0][w]) : u + red[0][w];
        v += red[1][w];
    }
}

// s / n, 1 / (s n) and 1 / n over the active cells (0 for a definite operator),
// whether there are any, by the whole workgroup, and every cell's -A_cc (0 if
// inactive) to dg
struct Shift {
    double base, shift, invn;
    bool any;
};

template <int NT>
__device__ __forceinline__ Shift shift_of(const PinvArgs &a, double *dg, double (*red)[NT / 64])
{
    double s = 0.0, na = 0.0;
    for (int c = threadIdx.x; c < a.n; c += NT) {
        const double g = row_of(a, c).dg;
        dg[c] = g > 0.0 ? g : 0.0;
        na += g > 0.0 ? 1.0 : 0.0;
        s = g > s ? g : s;
    }
    reduce2<true, NT>(s, na, red);
    const bool on = a.singular && na > 0.0;
    return Shift{on ? s / na : 0.0, on ? 1.0 / (s * na) : 0.0, on ? 1.0 / na : 0.0, na > 0.0};
}

// A row of K = -A + base 1 1^T over the active cells, after the workgroup has
// filled it with base: an inactive cell's row is the identity's, an active
// one's gets its diagonal and links (a link of weight 0 may lead to an
// inactive cell, whose column is 0).
__device__ __forceinline__ void finish_row(const Row &q, int c, double base, double *row)
{
#pragma unroll
    for (int m = 0; m < 6; ++m)
        if (q.nb[m] >= 0 && q.w[m] != 0.0)
            row[q.nb[m]] -= q.w[m];
    row[c] = q.dg > 0.0 ? row[c] + q.dg : 1.0;
}

constexpr int PROWS = 8;                 // rows per workgroup of the fill
constexpr int FTHREADS = 1024;           // a thread per cell: the loads' latency once

// K into the work matrix: PROWS rows per workgroup
__global__ __launch_bounds__(FTHREADS) void k_pinv_fill(PinvArgs a)
{
    __shared__ double red[2][FTHREADS / 64];
    __shared__ double dg[CELLS_MAX];
    const int t = threadIdx.x;
    const Shift sh = shift_of<FTHREADS>(a, dg, red);   // its barrier also completes dg
    const int r0 = blockIdx.x * PROWS;
    for (int q = t; q < PROWS * a.np; q += FTHREADS) {
        const int r = r0 + q / a.np, c = q % a.np;
        a.out[(size_t)r * a.np + c] = r < a.n && c < a.n
                                          ? (dg[r] > 0.0 && dg[c] > 0.0 ? sh.base : 0.0)
                                          : (r == c ? 1.0 : 0.0);
    }
    __syncthreads();
    if (t < PROWS && r0 + t < a.n) {
        finish_row(row_of(a, r0 + t), r0 + t, sh.base, a.out + (size_t)(r0 + t) * a.np);
        a.meta[r0 + t] = dg[r0 + t];
        if (r0 + t == 0) {
            a.meta[a.n + M_SHIFT] = sh.shift;
            *a.bad = sh.any ? PINV_GOOD : PINV_ZERO;
        }
    }
}

// Where no link joins two cells of one colour (periodic extents are even), the
// cells of colour 0 are eliminated in closed form and the pivots halve.  With
// D = -A_cc, B the links between the colours, w = 1 / D on colour 0,
// q_b = sum_r B_rb w_r, and gamma = base / (1 + base sum w), the block of
// colour 0 is D + base 1 1^T with inverse D^-1 - gamma w w^T, and its Schur
// complement on colour 1 is
//   S = D_b - B^T D^-1 B + gamma (1 + q) (1 + q)^T.
// From Z = S^-1, x_r = Z's row for a cell of colour 1 and
//   x_r = w_r (B Z)_r - w_r / n
// for one of colour 0 are the columns of colour 1 of K^-1: the gamma term of
// the latter is gamma w (1 + q)^T Z, and K 1 = s 1 makes gamma (1 + q)^T Z
// equal 1 / n.  The columns of colour 0 come from x_r the same way, plus the
// diagonal block's own inverse.  Without the null space base, gamma and 1 / n
// are 0.  Two neighbours of the cells' numbering have different colours, so
// c >> 1 numbers the cells of either.
__device__ __forceinline__ int colour_of(const PinvArgs &a, int c)
{
    const int nx = a.d.nx, ny = a.d.ny;
    const int k = c / (nx * ny), rem = c - k * nx * ny, j = rem / nx;
    return (rem - j * nx + j + k) & 1;
}

__device__ __forceinline__ int cell_of(const PinvArgs &a, int idx, int colour)
{
    return 2 * idx + (colour_of(a, 2 * idx) != colour);
}

// S into the work matrix: PROWS rows per workgroup
__global__ __launch_bounds__(FTHREADS) void k_pinv_reduce(PinvArgs a)
{
    __shared__ double red[2][2][FTHREADS / 64];
    __shared__ double dg[CELLS_MAX];
    __shared__ double q1[CELLS_MAX / 2];           // 1 + q_b, 0 at inactive cells
    __shared__ double rows[PROWS][CELLS_MAX / 2];
    __shared__ double lw[PROWS * 6][6];            // the two-link paths of a row
    __shared__ int ln[PROWS * 6][6];
    const int t = threadIdx.x;
    const Shift sh = shift_of<FTHREADS>(a, dg, red[0]);
    double sw = 0.0, sq = 0.0;
    for (int c = t; c < a.n; c += FTHREADS) {
        if (colour_of(a, c) == 0) {
            sw += dg[c] > 0.0 ? 1.0 / dg[c] : 0.0;
            continue;
        }
        const Row r = row_of(a, c);
        double q = 1.0;
#pragma unroll
        for (int m = 0; m < 6; ++m)
            if (r.nb[m] >= 0 && r.w[m] != 0.0)
                q += r.w[m] / (dg[r.nb[m]] > 0.0 ? dg[r.nb[m]] : 1.0);
        q1[c >> 1] = r.dg > 0.0 ? q : 0.0;
        sq += q1[c >> 1];
    }
    const int r0 = blockIdx.x * PROWS;
    if (t < PROWS * 6 && r0 + t / 6 < a.m) {
        const Row r = row_of(a, cell_of(a, r0 + t / 6, 1));
        double w = 0.0;
        int nb = -1;
#pragma unroll
        for (int m = 0; m < 6; ++m)
            if (m == t % 6) {
                w = r.w[m];
                nb = r.nb[m];
            }
        if (nb >= 0 && w != 0.0) {
            const double f = w / (dg[nb] > 0.0 ? dg[nb] : 1.0);
            const Row s = row_of(a, nb);
#pragma unroll
            for (int m = 0; m < 6; ++m) {
                lw[t][m] = f * s.w[m];
                ln[t][m] = s.w[m] != 0.0 ? s.nb[m] >> 1 : -1;
            }
        } else {
#pragma unroll
            for (int m = 0; m < 6; ++m)
                ln[t][m] = -1;
        }
    }
    reduce2<false, FTHREADS>(sw, sq, red[1]);                // its barrier also completes q1, lw and ln
    const double gamma = sh.base / (1.0 + sh.base * sw);
    for (int q = t; q < PROWS * a.np; q += FTHREADS) {
        const int r = q / a.np, c = q % a.np;
        rows[r][c] = r0 + r < a.m && c < a.m ? gamma * q1[r0 + r] * q1[c]
                                             : (r0 + r == c ? 1.0 : 0.0);
    }
    __syncthreads();
    if (t < PROWS && r0 + t < a.m) {
        const double g = dg[cell_of(a, r0 + t, 1)];
        double *row = rows[t];
        for (int e = 0; e < 36; ++e)
            if (ln[6 * t + e / 6][e % 6] >= 0)
                row[ln[6 * t + e / 6][e % 6]] -= lw[6 * t + e / 6][e % 6];
        row[r0 + t] = g > 0.0 ? row[r0 + t] + g : 1.0;
    }
    __syncthreads();
    for (int q = t; q < PROWS * a.np; q += FTHREADS)
        a.out[(size_t)r0 * a.np + q] = rows[q / a.np][q % a.np];
    if (blockIdx.x == 0) {
        for (int c = t; c < a.n; c += FTHREADS)
            a.meta[c] = dg[c];
        if (t == 0) {
            a.meta[a.n + M_SHIFT] = sh.shift;
            a.meta[a.n + M_GAMMA] = gamma;
            a.meta[a.n + M_INVN] = sh.invn;
            a.meta[a.n + M_SUMQ] = sq;
            *a.bad = sh.any ? PINV_GOOD : PINV_ZERO;
        }
    }
}

constexpr int EROWS = 4;                 // rows of the pseudo-inverse per workgroup
constexpr int ETHREADS = 512;            // a thread per cell of one colour

// A^+ of all cells from Z, the inverse of S
__global__ __launch_bounds__(ETHREADS) void k_pinv_expand(PinvArgs a)
{
    __shared__ double x[EROWS][CELLS_MAX / 2];
    __shared__ double fw[EROWS][6];
    __shared__ int fn[EROWS][6];
    const int t = threadIdx.x, c0 = blockIdx.x * EROWS;
    const double *meta = a.meta + a.n;
    const double shift = meta[M_SHIFT], invn = meta[M_INVN];
    const double gg = meta[M_GAMMA] * (1.0 - meta[M_SUMQ] * invn);
    if (t < EROWS && c0 + t < a.n) {
        const int c = c0 + t;
        const Row r = row_of(a, c);
        const bool one = colour_of(a, c) != 0;     // its own row of Z
#pragma unroll
        for (int m = 0; m < 6; ++m) {
            const bool on = !one && r.nb[m] >= 0 && r.w[m] != 0.0;
            fn[t][m] = one ? c >> 1 : on ? r.nb[m] >> 1 : 0;
            fw[t][m] = one ? (m == 0 ? 1.0 : 0.0) : on ? r.w[m] / r.dg : 0.0;
        }
    }
    double wr[EROWS];                    // 1 / D of a row of colour 0, else 0
    bool act[EROWS];
#pragma unroll
    for (int r = 0; r < EROWS; ++r) {
        const double g = c0 + r < a.n ? a.meta[c0 + r] : 0.0;
        act[r] = g > 0.0;
        wr[r] = act[r] && colour_of(a, c0 + r) == 0 ? 1.0 / g : 0.0;
    }
    __syncthreads();
    for (int b = t; b < a.m; b += ETHREADS) {
        const int c = cell_of(a, b, 1);
        const bool on = a.meta[c] > 0.0;
#pragma unroll
        for (int r = 0; r < EROWS; ++r) {
            if (c0 + r >= a.n)
                break;
            double v = -wr[r] * invn;
#pragma unroll
            for (int m = 0; m < 6; ++m)
                v = fma(fw[r][m], a.in[(size_t)fn[r][m] * a.np + b], v);
            x[r][b] = v;
            a.pinv[(size_t)(c0 + r) * a.n + c] = act[r] && on ? shift - v : 0.0;
        }
    }
    __syncthreads();
    for (int q = t; q < a.n - a.m; q += ETHREADS) {
        const int c = cell_of(a, q, 0);
        const Row s = row_of(a, c);
        const bool on = s.dg > 0.0;
        const double w = on ? 1.0 / s.dg : 0.0;
#pragma unroll
        for (int r = 0; r < EROWS; ++r) {
            if (c0 + r >= a.n)
                break;
            double v = (c == c0 + r ? w : 0.0) - w * (invn + gg * wr[r]);
#pragma unroll
            for (int m = 0; m < 6; ++m)
                if (s.nb[m] >= 0 && s.w[m] != 0.0)
                    v = fma(s.w[m] * w, x[r][s.nb[m] >> 1], v);
            a.pinv[(size_t)(c0 + r) * a.n + c] = act[r] && on ? shift - v : 0.0;
        }
    }
}

// 1 / p for a pivot: the hardware's estimate and two Newton steps, zero and
// infinity as a division gives them
__device__ __forceinline__ double reciprocal(double p)
{
    double r = __builtin_amdgcn_rcp(p);
    r = fma(r, fma(-p, r, 1.0), r);
    r = fma(r, fma(-p, r, 1.0), r);
    return __builtin_amdgcn_div_fixup(r, p, 1.0);
}

// A 64 x 64 tile is held as 4 x 4 entries a thread in the layout of the FP64
// matrix instruction's result: thread (ti, tj) of 16 x 16 has rows
// tile_row(ti, p) and columns tj + 16 q, wave ti / 4 has 16 rows.
using Acc = __attribute__((__vector_size__(4 * sizeof(double)))) double;

__device__ __forceinline__ int tile_row(int ti, int p) { return (ti >> 2) * 16 + (ti & 3) + 4 * p; }

// Gauss-Jordan inversion of such a tile in place, four pivots at a time: rows
// and columns tile_row(g, 0..3), whose rows belong to one ti and whose columns
// to four tj.  They go through LDS once (one barrier, the buffers alternate),
// every thread solves for the row of the pivot block's inverse that its lanes
// need, and the update is one matrix instruction per 16 x 16 entries,
//   v <- v - C P^-1 R.
// What the pivot rows and columns become fits the same update: columns are
// cleared and take the identity for R, rows are cleared and take minus the
// identity for C.  Returns whether a pivot was not positive.
constexpr int PBS = PB + 8;
struct PivotBuf {
    double row[4][PBS], col[4][PBS], piv[4][4];
};

__device__ __forceinline__ bool invert_tile(Acc (&v)[4], int ti, int tj, PivotBuf *buf)
{
    const int kk = ti & 3;               // the lane's k of the matrix operands
    bool bad = false;
    // the columns of v turn with the pivots, so that theirs are v[0]'s
#pragma unroll 1
    for (int g = 0; g < 16; ++g) {
        PivotBuf &b = buf[g & 1];
        const int a0 = tj >> 2;
        const bool prow = ti == g, pcol = (tj & 3) == (g & 3);
        if (prow)
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    double w = v[q][p];
                    if (q == 0 && pcol) {
                        b.piv[p][a0] = w;
                        w = p == a0 ? 1.0 : 0.0;
                    }
                    b.row[p][tj + 16 * q] = w;
                }
        if (pcol)
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                b.col[a0][tile_row(ti, p)] = prow ? (p == a0 ? 1.0 : 0.0) : -v[0][p];
                v[0][p] = 0.0;
            }
        if (prow)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                v[q] = Acc{0.0, 0.0, 0.0, 0.0};
        __syncthreads();
        // z: row kk of the (symmetric) pivot block's inverse, by L D L^T
        double l[4][4], z[4], id[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            z[p] = p == kk ? 1.0 : 0.0;
#pragma unroll
            for (int q = 0; q <= p; ++q)
                l[p][q] = b.piv[p][q];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            bad |= !(l[k][k] > 0.0);
            id[k] = reciprocal(l[k][k]);
            double f[4];
#pragma unroll
            for (int p = k + 1; p < 4; ++p) {
                f[p] = l[p][k] * id[k];
                z[p] = fma(-f[p], z[k], z[p]);
#pragma unroll
                for (int q = k + 1; q <= p; ++q)
                    l[p][q] = fma(-f[p], l[q][k], l[p][q]);
            }
#pragma unroll
            for (int p = k + 1; p < 4; ++p)
                l[p][k] = f[p];
        }
#pragma unroll
        for (int k = 3; k >= 0; --k) {
            z[k] *= id[k];
#pragma unroll
            for (int p = k + 1; p < 4; ++p)
                z[k] = fma(-l[p][k], z[p], z[k]);
        }
        const double c = b.col[kk][(ti >> 2) * 16 + tj];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            double m = z[0] * b.row[0][tj + 16 * q];
#pragma unroll
            for (int a = 1; a < 4; ++a)
                m = fma(z[a], b.row[a][tj + 16 * q], m);
            v[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(c, m, v[q], 0, 0, 0);
        }
        if ((g & 3) == 3) {
            const Acc w = v[0];
            v[0] = v[1];
            v[1] = v[2];
            v[2] = v[3];
            v[3] = w;
        }
    }
    return bad;
}

// Coarsest levels of one tile (n <= 64, every power-of-two grid): the whole
// rebuild in one workgroup, little enough LDS and registers to sit beside a
// smoother pass that holds every CU.
__global__ __launch_bounds__(PTHREADS) void k_pinv_small(PinvArgs a)
{
    __shared__ double Km[PB * PLD];
    __shared__ PivotBuf piv[2];
    __shared__ double red[2][PTHREADS / 64];
    __shared__ double dg[PB];
    const int t = threadIdx.x, ti = t >> 4, tj = t & 15;
    Row row;
    if (t < a.n)
        row = row_of(a, t);
    const Shift sh = shift_of<PTHREADS>(a, dg, red);
    for (int q = t; q < PB * PB; q += PTHREADS) {
        const int r = q / PB, c = q % PB;
        Km[r * PLD + c] = r < a.n && c < a.n ? (dg[r] > 0.0 && dg[c] > 0.0 ? sh.base : 0.0)
                                             : (r == c ? 1.0 : 0.0);
    }
    __syncthreads();
    if (t < a.n)
        finish_row(row, t, sh.base, Km + t * PLD);
    __syncthreads();
    Acc v[4];
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            v[q][p] = Km[tile_row(ti, p) * PLD + tj + 16 * q];
    const bool bad = invert_tile(v, ti, tj, piv);
    if (t == 0)
        *a.bad = bad ? PINV_BAD : (sh.any ? PINV_GOOD : PINV_ZERO);
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = tile_row(ti, p), c = tj + 16 * q;
            if (r < a.n && c < a.n)
                a.pinv[(size_t)r * a.n + c] =
                    dg[r] > 0.0 && dg[c] > 0.0 ? sh.shift - v[q][p] : 0.0;
        }
}

// X Y, by the matrix instruction
__device__ __forceinline__ void tile_product(const double *X, const double *Y, int ti, int tj,
                                             Acc (&v)[4])
{
    const double *x = X + ((ti >> 2) * 16 + tj) * PLD + (ti & 3), *y = Y + (ti & 3) * PLD + tj;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        v[q] = Acc{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int k = 0; k < PB; k += 4)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            v[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[k], y[k * PLD + 16 * q], v[q], 0, 0, 0);
}

// One elimination step.  Block (I, J) of the grid writes tile (I, J):
// with P the inverse of the pivot tile (k, k),
//   (k, k) <- P, (k, J) <- P M_kJ, (I, k) <- -M_Ik P, (I, J) <- M_IJ - M_Ik P M_kJ.
__global__ __launch_bounds__(PTHREADS) void k_pinv_step(PinvArgs a)
{
    __shared__ double Pm[PB * PLD];      // the pivot tile's inverse
    __shared__ double Xm[PB * PLD];      // M_Ik, then M_Ik P
    __shared__ double Ym[PB * PLD];      // M_kJ
    __shared__ PivotBuf piv[2];
    const int t = threadIdx.x, ti = t >> 4, tj = t & 15;
    const int I = blockIdx.x, J = blockIdx.y, K = a.step;
    // every load first: the pivot tile into registers, the panels into LDS
    Acc v[4], x[4];
    const double *row = a.in + (size_t)tile_row(ti, 0) * a.np + tj;
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const size_t o = (size_t)(4 * p) * a.np + 16 * q;
            v[q][p] = row[o + (size_t)K * PB * a.np + K * PB];
            const int l = tile_row(ti, p) * PLD + tj + 16 * q;
            Xm[l] = row[o + (size_t)I * PB * a.np + K * PB];
            Ym[l] = row[o + (size_t)K * PB * a.np + J * PB];
        }
    const bool bad = invert_tile(v, ti, tj, piv);
    if (I == 0 && J == 0 && t == 0 && bad)
        *a.bad = PINV_BAD;               // (the fill wrote the verdict before)
    if (I != K || J != K) {
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                Pm[tile_row(ti, p) * PLD + tj + 16 * q] = v[q][p];
        __syncthreads();
        if (I == K) {
            tile_product(Pm, Ym, ti, tj, v);
        } else {
            tile_product(Xm, Pm, ti, tj, x);
            if (J != K) {
                __syncthreads();
#pragma unroll
                for (int p = 0; p < 4; ++p)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        Xm[tile_row(ti, p) * PLD + tj + 16 * q] = x[q][p];
                __syncthreads();
                tile_product(Xm, Ym, ti, tj, x);
            }
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const size_t o = (size_t)(I * PB + 4 * p) * a.np + J * PB + 16 * q;
                    v[q][p] = (J == K ? 0.0 : row[o]) - x[q][p];
                }
        }
    }
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = I * PB + tile_row(ti, p), c = J * PB + tj + 16 * q;
            if (!a.direct)
                a.out[(size_t)r * a.np + c] = v[q][p];
            else if (r < a.n && c < a.n)
                a.pinv[(size_t)r * a.n + c] =
                    a.meta[r] > 0.0 && a.meta[c] > 0.0 ? a.meta[a.n + M_SHIFT] - v[q][p] : 0.0;
        }
}

size_t pinv_work_doubles(int n)
{
    const size_t np = (size_t)(n + PB - 1) / PB * PB;
    return np > PB ? 2 * np * np + n + M_COUNT : 0;
}

void launch_pinv(Dims d, Bc bc, double h, const double *const b[3], const double *sg,
                 bool singular, double *work, double *pinv, double *bad, hipStream_t s)
{
    PinvArgs a{};
    a.d = d;
    a.bc = bc;
    a.ih2 = 1.0 / (h * h);
    for (int m = 0; m < 3; ++m)
        a.b[m] = b[m];
    a.sg = sg;
    a.singular = singular ? 1 : 0;
    a.n = (int)cells(d);
    a.pinv = pinv;
    a.bad = bad;
    if (a.n <= PB) {
        hipLaunchKernelGGL(k_pinv_small, dim3(1), dim3(PTHREADS), 0, s, a);
        return;
    }
    // two colours (a half-size matrix) unless a periodic odd extent joins cells of one
    const bool two = (bc.x || d.nx % 2 == 0) && (bc.y || d.ny % 2 == 0) && (bc.z || d.nz % 2 == 0);
    a.m = two ? a.n / 2 : a.n;
    a.np = (a.m + PB - 1) / PB * PB;
    const int nb = a.np / PB;
    double *buf[2] = {work, work + (size_t)a.np * a.np};
    a.meta = buf[1] + (size_t)a.np * a.np;
    a.out = buf[1];
    if (two)
        hipLaunchKernelGGL(k_pinv_reduce, dim3(a.np / PROWS), dim3(FTHREADS), 0, s, a);
    else
        hipLaunchKernelGGL(k_pinv_fill, dim3(a.np / PROWS), dim3(FTHREADS), 0, s, a);
    for (int k = 0; k < nb; ++k) {
        a.step = k;
        a.in = buf[(k + 1) & 1];
        a.out = buf[k & 1];
        a.direct = !two && k + 1 == nb;
        hipLaunchKernelGGL(k_pinv_step, dim3(nb, nb), dim3(PTHREADS), 0, s, a);
    }
    if (two) {
        a.in = a.out;
        hipLaunchKernelGGL(k_pinv_expand, dim3((a.n + EROWS - 1) / EROWS), dim3(ETHREADS), 0, s, a);
    }
}

}  // namespace pp
