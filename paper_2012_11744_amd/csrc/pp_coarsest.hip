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
// factorisation), 64 columns a step, one launch a step.  The chain of n
// dependent pivots bounds it, not its 2 n^3 operations: a workgroup inverts
// the 64 x 64 pivot block with the matrix held in registers, one barrier a
// pivot, and every workgroup does so redundantly, which spares each step a
// second launch and a round trip through memory.  Steps are out of place
// (two work matrices), so no workgroup reads what another writes.  Measured:
// 33 us for up to 64 cells, 41 us a step above; a projection step at
// 144 x 80 x 32 (720 coarsest cells) takes 3.0 ms, against 31.7 ms with a
// Cholesky factorisation on the host (29 ms of it).
#include <hip/hip_runtime.h>

#include "pp_internal.h"

namespace pp {

constexpr int PB = 64;                   // columns per elimination step
constexpr int PTHREADS = 256;            // 16 x 16 threads, 4 x 4 entries each
constexpr int PLD = PB + 1;              // LDS row

struct PinvArgs {
    Dims d;
    Bc bc;
    double ih2;
    const double *b[3];                  // FP64 face coefficients of the coarsest level
    const double *sg;                    // its sigma, or null
    int singular;                        // the constants on the active cells are the null space
    int n, np;                           // cells, and rounded up to whole blocks
    int step;                            // elimination step (block column)
    const double *in;                    // np x np work matrix
    double *out;                         // np x np work matrix (not written by the last step)
    double *meta;                        // per cell: 1 if active, else 0; [n]: 1 / (s n) or 0
    double *pinv;                        // n x n, written by the last step
    double *bad;                         // 1 where a pivot is not a positive number, else 0
};

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

// s / n and 1 / (s n) over the active cells (0 for a definite operator), by
// the whole workgroup
struct Shift {
    double base, shift;
};

__device__ __forceinline__ Shift shift_of(const PinvArgs &a, double (*red)[PTHREADS / 64])
{
    const int t = threadIdx.x;
    double s = 0.0, na = 0.0;
    for (int c = t; c < a.n; c += PTHREADS) {
        const double dg = row_of(a, c).dg;
        na += dg > 0.0 ? 1.0 : 0.0;
        s = dg > s ? dg : s;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        na += __shfl_xor(na, o, 64);
        s = fmax(s, __shfl_xor(s, o, 64));
    }
    if ((t & 63) == 0) {
        red[0][t >> 6] = s;
        red[1][t >> 6] = na;
    }
    __syncthreads();
    s = fmax(fmax(red[0][0], red[0][1]), fmax(red[0][2], red[0][3]));
    na = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
    const bool on = a.singular && na > 0.0;
    return Shift{on ? s / na : 0.0, on ? 1.0 / (s * na) : 0.0};
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

constexpr int PROWS = 8;                 // rows of K per workgroup of the fill

// K into the work matrix: PROWS rows per workgroup
__global__ __launch_bounds__(PTHREADS) void k_pinv_fill(PinvArgs a)
{
    __shared__ double red[2][PTHREADS / 64];
    __shared__ unsigned char actv[1024];
    const int t = threadIdx.x;
    for (int c = t; c < a.n; c += PTHREADS)
        actv[c] = row_of(a, c).dg > 0.0;
    const Shift sh = shift_of(a, red);   // its barrier also completes actv
    const int r0 = blockIdx.x * PROWS;
    for (int q = t; q < PROWS * a.np; q += PTHREADS) {
        const int r = r0 + q / a.np, c = q % a.np;
        a.out[(size_t)r * a.np + c] =
            r < a.n && c < a.n ? (actv[r] && actv[c] ? sh.base : 0.0) : (r == c ? 1.0 : 0.0);
    }
    __syncthreads();
    if (t < PROWS && r0 + t < a.n) {
        finish_row(row_of(a, r0 + t), r0 + t, sh.base, a.out + (size_t)(r0 + t) * a.np);
        a.meta[r0 + t] = actv[r0 + t];
        if (r0 + t == 0)
            a.meta[a.n] = sh.shift;
    }
}

// Gauss-Jordan inversion in place of a 64 x 64 tile held as 4 x 4 entries a
// thread (rows ti + 16 p, columns tj + 16 q); one barrier a pivot, the row and
// column buffers alternate.  Returns whether a pivot was not positive.
__device__ __forceinline__ bool invert_tile(double (&v)[4][4], int ti, int tj, double (*rowb)[PB],
                                            double (*colb)[PB])
{
    bool bad = false;
#pragma unroll
    for (int kp = 0; kp < 4; ++kp)
#pragma unroll 1                         // unrolled, its 64 steps spill
        for (int kr = 0; kr < 16; ++kr) {
            const int buf = kr & 1;
            if (ti == kr)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    rowb[buf][tj + 16 * q] = v[kp][q];
            if (tj == kr)
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    colb[buf][ti + 16 * p] = v[p][kp];
            __syncthreads();
            const double piv = rowb[buf][kr + 16 * kp];
            bad |= !(piv > 0.0);
            const double ip = 1.0 / piv;
            double f[4], r[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                f[p] = colb[buf][ti + 16 * p] * ip;
                r[p] = rowb[buf][tj + 16 * p];
            }
            // the pivot's row and column take the update's form with the old
            // value 0 and the factor -1/pivot, or the row entry 1
            if (ti == kr) {
                f[kp] = -ip;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    v[kp][q] = 0.0;
            }
            if (tj == kr) {
                r[kp] = 1.0;
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    v[p][kp] = 0.0;
            }
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    v[p][q] = fma(-f[p], r[q], v[p][q]);
        }
    return bad;
}

// Coarsest levels of one tile (n <= 64, every power-of-two grid): the whole
// rebuild in one workgroup, little enough LDS and registers to sit beside a
// smoother pass that holds every CU.
__global__ __launch_bounds__(PTHREADS) void k_pinv_small(PinvArgs a)
{
    __shared__ double Km[PB * PLD];
    __shared__ double rowb[2][PB], colb[2][PB];
    __shared__ double red[2][PTHREADS / 64];
    __shared__ unsigned char actv[PB];
    const int t = threadIdx.x, ti = t >> 4, tj = t & 15;
    Row row;
    if (t < a.n) {
        row = row_of(a, t);
        actv[t] = row.dg > 0.0;
    }
    const Shift sh = shift_of(a, red);
    for (int q = t; q < PB * PB; q += PTHREADS) {
        const int r = q / PB, c = q % PB;
        Km[r * PLD + c] =
            r < a.n && c < a.n ? (actv[r] && actv[c] ? sh.base : 0.0) : (r == c ? 1.0 : 0.0);
    }
    __syncthreads();
    if (t < a.n)
        finish_row(row, t, sh.base, Km + t * PLD);
    __syncthreads();
    double v[4][4];
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            v[p][q] = Km[(ti + 16 * p) * PLD + tj + 16 * q];
    const bool bad = invert_tile(v, ti, tj, rowb, colb);
    if (t == 0)
        *a.bad = bad ? 1.0 : 0.0;
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = ti + 16 * p, c = tj + 16 * q;
            if (r < a.n && c < a.n)
                a.pinv[(size_t)r * a.n + c] = actv[r] && actv[c] ? sh.shift - v[p][q] : 0.0;
        }
}

// X Y for the thread's 4 x 4 entries (rows ti + 16 a, columns tj + 16 b)
__device__ __forceinline__ void tile_product(const double *X, const double *Y, int ti, int tj,
                                             double (&v)[4][4])
{
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            v[p][q] = 0.0;
#pragma unroll 4
    for (int k = 0; k < PB; ++k) {
        double x[4], y[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            x[p] = X[(ti + 16 * p) * PLD + k];
            y[p] = Y[k * PLD + tj + 16 * p];
        }
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                v[p][q] = fma(x[p], y[q], v[p][q]);
    }
}

// One elimination step.  Block (I, J) of the grid writes tile (I, J):
// with P the inverse of the pivot tile (k, k),
//   (k, k) <- P, (k, J) <- P M_kJ, (I, k) <- -M_Ik P, (I, J) <- M_IJ - M_Ik P M_kJ.
__global__ __launch_bounds__(PTHREADS) void k_pinv_step(PinvArgs a)
{
    __shared__ double Pm[PB * PLD];      // the pivot tile's inverse
    __shared__ double Xm[PB * PLD];      // M_Ik, then M_Ik P
    __shared__ double Ym[PB * PLD];      // M_kJ
    __shared__ double rowb[2][PB], colb[2][PB];
    const int t = threadIdx.x, ti = t >> 4, tj = t & 15;
    const int I = blockIdx.x, J = blockIdx.y, K = a.step;
    const bool last = (K + 1) * PB >= a.np;
    // every load first: the pivot tile into registers, the panels into LDS
    double v[4][4], x[4][4];
    const double *row = a.in + (size_t)ti * a.np + tj;
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const size_t o = (size_t)(16 * p) * a.np + 16 * q;
            v[p][q] = row[o + (size_t)K * PB * a.np + K * PB];
            const int l = (ti + 16 * p) * PLD + tj + 16 * q;
            Xm[l] = row[o + (size_t)I * PB * a.np + K * PB];
            Ym[l] = row[o + (size_t)K * PB * a.np + J * PB];
        }
    const bool bad = invert_tile(v, ti, tj, rowb, colb);
    if (I == 0 && J == 0 && t == 0 && (K == 0 || bad))
        *a.bad = bad ? 1.0 : 0.0;
    if (I != K || J != K) {
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                Pm[(ti + 16 * p) * PLD + tj + 16 * q] = v[p][q];
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
                        Xm[(ti + 16 * p) * PLD + tj + 16 * q] = x[p][q];
                __syncthreads();
                tile_product(Xm, Ym, ti, tj, x);
            }
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const size_t o = (size_t)(I * PB + 16 * p) * a.np + J * PB + 16 * q;
                    v[p][q] = (J == K ? 0.0 : row[o]) - x[p][q];
                }
        }
    }
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = I * PB + ti + 16 * p, c = J * PB + tj + 16 * q;
            if (!last)
                a.out[(size_t)r * a.np + c] = v[p][q];
            else if (r < a.n && c < a.n)
                a.pinv[(size_t)r * a.n + c] =
                    a.meta[r] != 0.0 && a.meta[c] != 0.0 ? a.meta[a.n] - v[p][q] : 0.0;
        }
}

size_t pinv_work_doubles(int n)
{
    const size_t np = (size_t)(n + PB - 1) / PB * PB;
    return np > PB ? 2 * np * np + n + 1 : 0;
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
    a.np = (a.n + PB - 1) / PB * PB;
    a.pinv = pinv;
    a.bad = bad;
    const int nb = a.np / PB;
    if (nb == 1) {
        hipLaunchKernelGGL(k_pinv_small, dim3(1), dim3(PTHREADS), 0, s, a);
        return;
    }
    double *buf[2] = {work, work + (size_t)a.np * a.np};
    a.meta = buf[1] + (size_t)a.np * a.np;
    a.out = buf[1];
    hipLaunchKernelGGL(k_pinv_fill, dim3(a.np / PROWS), dim3(PTHREADS), 0, s, a);
    for (int k = 0; k < nb; ++k) {
        a.step = k;
        a.in = buf[(k + 1) & 1];
        a.out = buf[k & 1];
        hipLaunchKernelGGL(k_pinv_step, dim3(nb, nb), dim3(PTHREADS), 0, s, a);
    }
}

}  // namespace pp
