// pp_tail.hip -- the bottom of the V-cycle (gfx950): every level of at most
// TAIL_CELLS cells and the coarsest solve in one workgroup.
//
// These levels cost a kernel launch per step and little else, so they run in
// a single 1024-thread workgroup that walks them with barriers between steps.
// The latency of a half sweep bounds it (38 barriers at two smoothed levels
// and nu = 4), so a half sweep does as little as it can between two barriers:
//  - a thread owns one quad (an x-pair of cells in two planes 2K, 2K+1) of
//    each level and keeps its face coefficients, reciprocal diagonals,
//    right-hand side and corrections in registers (levels of 4096 cells have
//    1024 quads); a smoothed level has even sides of at least 8 cells, so at
//    most two levels of the tail are smoothed;
//  - of a cell's six neighbours two are the quad's own; the other four are
//    read from LDS;
//  - LDS holds each colour in an array of its own, one entry per x-pair: the
//    neighbours of a cell are the other colour's entries of the same pair in
//    the rows beside it and of the pair next to it, so the lanes of a wave
//    read consecutive words;
//  - the restriction's four x-z sums go through LDS once and become the next
//    level's right-hand side in registers.
// Measured with 16^3, 8^3 and 4^3 cells, per V-cycle: 18 us in FP32 arithmetic
// and 29 to 31 us in FP64; 33 and 70 us when every value of a pair came from LDS
// (FP64 coefficients from L2), two pairs of one plane a thread, a division a cell.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "pp_device.h"
#include "pp_internal.h"

namespace pp {

constexpr int TAIL_THREADS = 1024;
constexpr int TAIL_PINV = 4096;           // coarsest pseudo-inverses of up to 64 cells are staged in LDS
constexpr int TAIL_COARSE = 512;          // cells below a level of TAIL_CELLS
// Coarsest levels above this many cells are solved by a kernel of their own
// between the tail's way down and its way up: one workgroup reads their
// pseudo-inverse at some 10 B a cycle, many workgroups in 4 us whatever its
// size.  Measured per V-cycle, in one launch / split: 480 cells 92 / 21 us
// (the former in the tail before it held its levels in registers), 216 cells
// 35 / 21 us; below about 160 cells the two further launches (10 us) cost more.
constexpr int TAIL_SPLIT = 160;

template <typename T>
struct TailArgs {
    int n;                     // levels in the tail (the last is the coarsest): 2 or 3
    Dims d[TAIL_MAX];
    typename Acc<T>::type h2[TAIL_MAX];
    const T *b[TAIL_MAX][3];
    const T *s[TAIL_MAX];      // diagonal term of the general operator (h^2 sigma), or null
    const unsigned *w[TAIL_MAX];   // prolongation weights of each level but the last
    const T *r;                // right-hand side of the first level
    T *e;                      // its correction
    Bc bc;
    int nu_pre, nu_post;
    typename Acc<T>::type omega;   // the smoother's over-relaxation
    const double *pinv;        // pseudo-inverse of the coarsest operator
    int ncoarse;
    int warm;                  // e holds a correction to start the first level from
    double *state;             // split solve: what the way up takes from the way down
};

// split-solve state (one smoothed level: two need 16^3, 8^3 and 4^3 cells):
// its corrections, the coarsest right-hand side and the coarsest correction
constexpr int TAIL_STATE_RS = 4 * TAIL_THREADS;
constexpr int TAIL_STATE_EC = TAIL_STATE_RS + TAIL_COARSE;
static_assert(TAIL_STATE_EC + TAIL_COARSE == TAIL_STATE, "size of the split-solve state");
static_assert(TAIL_CELLS == 4 * TAIL_THREADS, "one quad per thread");

// One quad of a smoothed level.  Cells are indexed [colour][plane of the
// quad]: the red ((i+j+k) even) cell of plane z sits at x offset (j+z) & 1 of
// the pair, the black one at the other.
template <typename C>
struct Quad {
    bool on;
    int t, j, K;               // pair along x, row, plane pair
    int own[2];                // LDS entries of the pair in its two planes
    int adj[2][2];             // ... of the x-neighbouring pair of each cell
    int ym, yp;                // offsets of the rows below and above
    int zl, zh;                // LDS entries of the pair in the planes below and above the quad
    C xin[2];                  // the face inside the pair, per plane
    C xout[2][2];              // the cell's outer x face
    C yl[2][2], yh[2][2];
    C zin[2];                  // the face between the planes at red's x offset of plane 0, of plane 1
    C zout[2][2];              // the cell's outer z face
    C r[2][2];
    C inv[2][2];               // omega / diagonal, 0 for an excluded cell (EXACT: the diagonal)
    C e[2][2];
};

// FP16 storage rounds every level's correction to 11 bits, and where a value
// falls between two of them an FP32 rounding decides, so its iterates repeat
// only if every FP32 operation does: EXACT keeps faces in the order x, y, z,
// low before high, a division per update, and the choice of which products
// are rounded and which are fused, per phase (TailSweep).  FP32 and FP64
// storage multiply by the reciprocal.
enum TailSweep { SWEEP_FIRST, SWEEP_DOWN, SWEEP_UP };

template <typename T>
constexpr bool exact_order()
{
    return std::is_same<T, _Float16>::value;
}

template <typename C>
__device__ __forceinline__ C pick2(bool hi, C lo_v, C hi_v)
{
    return hi ? hi_v : lo_v;
}

// coordinates and LDS entries of quad q of a level
template <typename C>
__device__ __forceinline__ void quad_place(Quad<C> &Q, Dims d, int q)
{
    const int hx = d.nx / 2;
    Q.on = q < hx * d.ny * (d.nz / 2);
    if (!Q.on)
        q = 0;
    Q.K = q / (hx * d.ny);
    const int rem = q - Q.K * hx * d.ny;
    Q.j = rem / hx;
    Q.t = rem - Q.j * hx;
    const int plane = hx * d.ny, row = Q.j * hx;
    const int k = 2 * Q.K;
    Q.own[0] = k * plane + row + Q.t;
    Q.own[1] = Q.own[0] + plane;
    const int left = Q.t == 0 ? hx - 1 : -1, right = Q.t == hx - 1 ? 1 - hx : 1;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int z = 0; z < 2; ++z)
            Q.adj[c][z] = Q.own[z] + (((Q.j + z + c) & 1) ? right : left);
    Q.ym = Q.j == 0 ? (d.ny - 1) * hx : -hx;
    Q.yp = Q.j == d.ny - 1 ? -(d.ny - 1) * hx : hx;
    Q.zl = k == 0 ? Q.own[0] + (d.nz - 1) * plane : Q.own[0] - plane;
    Q.zh = k + 2 == d.nz ? Q.own[1] - (d.nz - 1) * plane : Q.own[1] + plane;
}

// the quad's face coefficients (walls 0) and reciprocal diagonals
template <typename C, typename T>
__device__ __forceinline__ void quad_coeffs(Quad<C> &Q, Dims d, Bc bc, const T *const b[3],
                                            const T *sg, C om)
{
    using T2 = typename Vec2<T>::type;
    auto ld2 = [](const T *p, int i) -> T2 { return *reinterpret_cast<const T2 *>(p + i); };
    const int nxy = d.nx * d.ny;
    const int x = 2 * Q.t, k = 2 * Q.K;
    const int xr = x + 2 == d.nx ? -x : 2;                     // right neighbour of the pair
    const int up = Q.j == d.ny - 1 ? -(d.ny - 1) * d.nx : d.nx;
    const bool wxl = bc.x && x == 0, wxh = bc.x && x + 2 == d.nx;
    const bool wyl = bc.y && Q.j == 0, wyh = bc.y && Q.j == d.ny - 1;
    const bool wzl = bc.z && k == 0, wzh = bc.z && k + 2 == d.nz;
    const int c0 = (k * d.ny + Q.j) * d.nx + x;
    const int c2 = k + 2 == d.nz ? c0 - k * nxy : c0 + 2 * nxy;   // the plane above the quad
    T2 fx[2], fl[2], fh[2], sv[2];
    T xh[2];
#pragma unroll
    for (int z = 0; z < 2; ++z) {
        const int c = c0 + z * nxy;
        fx[z] = ld2(b[0], c);
        xh[z] = b[0][c + xr];
        fl[z] = ld2(b[1], c);
        fh[z] = ld2(b[1], c + up);
        if (sg)
            sv[z] = ld2(sg, c);
    }
    const T2 z0 = ld2(b[2], c0), z1 = ld2(b[2], c0 + nxy), z2 = ld2(b[2], c2);
    const C zero = C(0);
#pragma unroll
    for (int z = 0; z < 2; ++z)
        Q.xin[z] = C(fx[z].y);
    const bool o0 = (Q.j & 1) != 0;                            // red's x offset in plane 0
    Q.zin[0] = pick2<C>(o0, C(z1.x), C(z1.y));
    Q.zin[1] = pick2<C>(o0, C(z1.y), C(z1.x));
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int z = 0; z < 2; ++z) {
            const bool o = ((Q.j + z + c) & 1) != 0;
            Q.xout[c][z] = o ? (wxh ? zero : C(xh[z])) : (wxl ? zero : C(fx[z].x));
            Q.yl[c][z] = wyl ? zero : pick2<C>(o, C(fl[z].x), C(fl[z].y));
            Q.yh[c][z] = wyh ? zero : pick2<C>(o, C(fh[z].x), C(fh[z].y));
            Q.zout[c][z] = z == 0 ? (wzl ? zero : pick2<C>(o, C(z0.x), C(z0.y)))
                                  : (wzh ? zero : pick2<C>(o, C(z2.x), C(z2.y)));
            // red's offset in plane 1 is black's in plane 0
            C dg = (Q.xin[z] + Q.xout[c][z]) + (Q.yl[c][z] + Q.yh[c][z]) +
                   (Q.zin[c ^ z] + Q.zout[c][z]);
            if (sg)
                dg += pick2<C>(o, C(sv[z].x), C(sv[z].y));
            Q.inv[c][z] = exact_order<T>() ? dg : (dg > zero ? om / dg : zero);
        }
}

// four values of a level's array as [colour][plane]
template <typename C, typename T>
__device__ __forceinline__ void quad_values(const Quad<C> &Q, Dims d, const T *p, C (&v)[2][2])
{
    using T2 = typename Vec2<T>::type;
    const int c0 = (2 * Q.K * d.ny + Q.j) * d.nx + 2 * Q.t;
#pragma unroll
    for (int z = 0; z < 2; ++z) {
        const T2 q = *reinterpret_cast<const T2 *>(p + c0 + z * d.nx * d.ny);
        const bool o = ((Q.j + z) & 1) != 0;
        v[0][z] = pick2<C>(o, C(q.x), C(q.y));
        v[1][z] = pick2<C>(o, C(q.y), C(q.x));
    }
}

// Over-relaxed Gauss-Seidel update of the quad's cells of one colour (eq.
// beta_pressure), and their publication.  O: the other colour's LDS array.
// zero: every correction is 0 on entry; own_zero: the cells' own old values
// are (the second colour of the first sweep).
template <int COL, bool EXACT, typename C>
__device__ __forceinline__ void quad_gs(Quad<C> &Q, C *own, const C *O, C h2, C om, C om1,
                                        TailSweep kind, bool zero, bool own_zero)
{
    if (!Q.on)
        return;
    C s[2] = {C(0), C(0)};
    if (!zero) {
#pragma unroll
        for (int z = 0; z < 2; ++z) {
            const int o = Q.own[z];
            const C ein = Q.e[1 - COL][z], eout = O[Q.adj[COL][z]];
            const C eyl = O[o + Q.ym], eyh = O[o + Q.yp];
            const C ezin = Q.e[1 - COL][1 - z], ezout = O[z == 0 ? Q.zl : Q.zh];
            const C zin = Q.zin[COL ^ z], zout = Q.zout[COL][z];
            if (EXACT) {
                const bool hi = ((Q.j + z + COL) & 1) != 0;    // the high cell of the pair
                const C xl = hi ? Q.xin[z] : Q.xout[COL][z], xh = hi ? Q.xout[COL][z] : Q.xin[z];
                const C el = hi ? ein : eout, eh = hi ? eout : ein;
                const C zl = z ? zin : zout, zh = z ? zout : zin;
                const C fl = z ? ezin : ezout, fh = z ? ezout : ezin;
                C t = fma(xl, el, xh * eh);
                t = fma(Q.yl[COL][z], eyl, t);
                t = fma(Q.yh[COL][z], eyh, t);
                t = fma(zl, fl, t);
                s[z] = fma(zh, fh, t);
            } else {
                s[z] = Q.xin[z] * ein + Q.xout[COL][z] * eout + Q.yl[COL][z] * eyl +
                       Q.yh[COL][z] * eyh + zin * ezin + zout * ezout;
            }
        }
    }
#pragma unroll
    for (int z = 0; z < 2; ++z) {
        C v;
        if (EXACT) {
            C num, up;
            {
#pragma clang fp contract(off)
                num = s[z] - h2 * Q.r[COL][z];
                up = om1 * Q.e[COL][z];
            }
            if (kind == SWEEP_FIRST)
                num = fma(-h2, Q.r[COL][z], s[z]);
            const C g = num / Q.inv[COL][z], og = om * g;
            v = (zero || own_zero) ? og
                                   : (kind == SWEEP_UP ? fma(om1, Q.e[COL][z], og) : fma(om, g, up));
            v = Q.inv[COL][z] > C(0) ? v : C(0);
        } else {
            const C g = fma(-h2, Q.r[COL][z], s[z]) * Q.inv[COL][z];
            v = (zero || own_zero) ? g : fma(om1, Q.e[COL][z], g);
            v = Q.inv[COL][z] != C(0) ? v : C(0);
        }
        // a cell with no open face and no diagonal term is excluded: it stays 0
        Q.e[COL][z] = v;
        own[Q.own[z]] = v;
    }
}

// r - A e summed over the pair of each of the quad's planes (sg: h^2 sigma of
// the level)
template <typename C, typename T>
__device__ __forceinline__ void quad_residual(const Quad<C> &Q, Dims d, const C *R, const C *B,
                                              C h2, const T *sg, C (&sum)[2])
{
    C sv[2][2] = {{C(0), C(0)}, {C(0), C(0)}};
    if (sg)
        quad_values<C, T>(Q, d, sg, sv);
    const C ih2 = C(1) / h2;
#pragma unroll
    for (int z = 0; z < 2; ++z) {
        C v[2];                            // by colour
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const C *O = c == 0 ? B : R;
            const C ec = Q.e[c][z];
            const int o = Q.own[z];
            const C ein = Q.e[1 - c][z], eout = O[Q.adj[c][z]];
            const C eyl = O[o + Q.ym], eyh = O[o + Q.yp];
            const C ezin = Q.e[1 - c][1 - z], ezout = O[z == 0 ? Q.zl : Q.zh];
            const C zin = Q.zin[c ^ z], zout = Q.zout[c][z];
            // the product of the pair's own face is rounded, as the one both its
            // cells share; the others are fused: y high, low, z high, low
            C fl = fma(Q.xout[c][z], eout - ec, Q.xin[z] * (ein - ec));
            fl = fma(Q.yh[c][z], eyh - ec, fl);
            fl = fma(Q.yl[c][z], eyl - ec, fl);
            fl = fma(z ? zout : zin, (z ? ezout : ezin) - ec, fl);
            fl = fma(z ? zin : zout, (z ? ezin : ezout) - ec, fl);
            v[c] = fma(ih2, sv[c][z] * ec, fma(-ih2, fl, Q.r[c][z]));
        }
        sum[z] = v[0] + v[1];
    }
}

// Restriction: the mean of r - A e over the 8 children of coarse cell
// (I, J, K) from the quads' pair sums (two quads per coarse cell: rows 2J,
// 2J+1; Sp[z]: their plane 2K + z)
template <typename C>
__device__ __forceinline__ C restricted(const C (*Sp)[TAIL_THREADS], Dims fd, int I, int J, int K)
{
    const int hx = fd.nx / 2;
    const int q = (K * fd.ny + 2 * J) * hx + I;
    return C(0.125) * ((Sp[0][q] + Sp[0][q + hx]) + (Sp[1][q] + Sp[1][q + hx]));
}

// e += P eH on the quad (the interpolation of k_prolong with the level's
// weights); EH(I, J, K) reads the coarse correction
template <typename C, typename F>
__device__ __forceinline__ void quad_prolong(Quad<C> &Q, Dims fd, Bc bc, const unsigned (&w)[2][2],
                                             F EH)
{
    const Dims cd{fd.nx / 2, fd.ny / 2, fd.nz / 2};
    const int I = Q.t, J = Q.j >> 1, K = Q.K;
    const int J1 = other_parent(Q.j, cd.ny, bc.y);
    const int In[2] = {other_parent(2 * I, cd.nx, bc.x), other_parent(2 * I + 1, cd.nx, bc.x)};
#pragma unroll
    for (int z = 0; z < 2; ++z) {
        const int K1 = other_parent(2 * K + z, cd.nz, bc.z);
        const C p00 = EH(I, J, K), p01 = EH(I, J1, K), p10 = EH(I, J, K1), p11 = EH(I, J1, K1);
        C v[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const C ax = C(w[z][x] & 255u) * C(1.0 / 256.0);
            const C ay = C((w[z][x] >> 8) & 255u) * C(1.0 / 256.0);
            const C az = C((w[z][x] >> 16) & 255u) * C(1.0 / 256.0);
            const C a = p00 + ax * (EH(In[x], J, K) - p00), b = p01 + ax * (EH(In[x], J1, K) - p01);
            const C c = p10 + ax * (EH(In[x], J, K1) - p10), f = p11 + ax * (EH(In[x], J1, K1) - p11);
            const C y0 = a + ay * (b - a), y1 = c + ay * (f - c);
            v[x] = y0 + az * (y1 - y0);
        }
        const bool o = ((Q.j + z) & 1) != 0;
        Q.e[0][z] += pick2<C>(o, v[0], v[1]);
        Q.e[1][z] += pick2<C>(o, v[1], v[0]);
    }
}

__device__ __forceinline__ void quad_weights(int t, int j, int K, Dims d, const unsigned *w,
                                             unsigned (&q)[2][2])
{
    using U2 = unsigned __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int z = 0; z < 2; ++z) {
        const U2 v = *reinterpret_cast<const U2 *>(w + ((size_t)(2 * K + z) * d.ny + j) * d.nx + 2 * t);
        q[z][0] = v.x;
        q[z][1] = v.y;
    }
}

enum TailPhase { TAIL_ALL = 0, TAIL_DOWN = 1, TAIL_UP = 2 };

template <typename T, int PHASE>
__global__ __launch_bounds__(TAIL_THREADS) void k_tail_cycle(TailArgs<T> a)
{
    using C = typename Acc<T>::type;
    // corrections of the two smoothed levels by colour, and the coarsest
    __shared__ C EA[2][TAIL_CELLS / 2];
    __shared__ C EB[2][TAIL_CELLS / 16];
    __shared__ C EC[TAIL_COARSE];
    __shared__ C Sp[2][TAIL_THREADS];      // pair sums of a restriction, by plane
    __shared__ double rs[TAIL_COARSE];     // the coarsest right-hand side
    __shared__ double Pv[PHASE == TAIL_ALL ? TAIL_PINV : 1];
    const int tid = threadIdx.x;
    const bool two = PHASE == TAIL_ALL && a.n == 3;   // a second smoothed level
    const C om = a.omega, om1 = C(1) - om;
    const Dims dA = a.d[0], dB = a.d[1], dC = a.d[a.n - 1];
    const int nc = a.ncoarse;
    Quad<C> A, B;
    quad_place(A, dA, tid);
    quad_place(B, dB, two ? tid : TAIL_CELLS);
    // FP32 arithmetic holds both levels' coefficients throughout, loaded here
    // at once.  FP64's are loaded (from L2) when each level's turn comes; with two
    // levels in one launch 51 of its values are spilled all the same (188 bytes a
    // lane), with one (the split phases) none.
    constexpr bool KEEP = sizeof(C) == 4;
    constexpr bool EXACT = exact_order<T>();
    quad_coeffs<C, T>(A, dA, a.bc, a.b[0], a.s[0], om);
    quad_values<C, T>(A, dA, a.r, A.r);
    unsigned wA[2][2], wB[2][2] = {{0, 0}, {0, 0}};
    if (PHASE != TAIL_DOWN)
        quad_weights(A.t, A.j, A.K, dA, a.w[0], wA);
    if (KEEP && two && B.on) {
        quad_coeffs<C, T>(B, dB, a.bc, a.b[1], a.s[1], om);
        if (PHASE != TAIL_DOWN)
            quad_weights(B.t, B.j, B.K, dB, a.w[1], wB);
    }
    const bool pvl = PHASE == TAIL_ALL && nc * nc <= TAIL_PINV;
    if (PHASE == TAIL_ALL && pvl) {
        constexpr int UP = TAIL_PINV / TAIL_THREADS;
        double pv[UP];
#pragma unroll
        for (int u = 0; u < UP; ++u)
            pv[u] = a.pinv[min(tid + u * TAIL_THREADS, nc * nc - 1)];
#pragma unroll
        for (int u = 0; u < UP; ++u)
            if (tid + u * TAIL_THREADS < nc * nc)
                Pv[tid + u * TAIL_THREADS] = pv[u];
    }
    auto publish = [](const Quad<C> &Q, C *own, int c) {
        if (Q.on) {
            own[Q.own[0]] = Q.e[c][0];
            own[Q.own[1]] = Q.e[c][1];
        }
    };
    // nu red-black sweeps, red first
    auto sweeps_down = [&](Quad<C> &Q, C *E0, C *E1, C h2, bool warm) {
        for (int sw = 0; sw < a.nu_pre; ++sw) {
            const bool z = sw == 0 && !warm;
            const TailSweep kind = sw == 0 ? SWEEP_FIRST : SWEEP_DOWN;
            quad_gs<0, EXACT>(Q, E0, E1, h2, om, om1, kind, z, z);
            __syncthreads();
            quad_gs<1, EXACT>(Q, E1, E0, h2, om, om1, kind, false, z);
            __syncthreads();
        }
    };
    // nu sweeps, black first
    auto sweeps_up = [&](Quad<C> &Q, C *E0, C *E1, C h2) {
        for (int sw = 0; sw < a.nu_post; ++sw) {
            quad_gs<1, EXACT>(Q, E1, E0, h2, om, om1, SWEEP_UP, false, false);
            __syncthreads();
            quad_gs<0, EXACT>(Q, E0, E1, h2, om, om1, SWEEP_UP, false, false);
            __syncthreads();
        }
    };
    if (PHASE != TAIL_UP) {
        if (a.warm) {
            quad_values<C, T>(A, dA, a.e, A.e);
            publish(A, EA[1], 1);
            __syncthreads();
        }
        sweeps_down(A, EA[0], EA[1], a.h2[0], a.warm != 0);
        auto residual = [&](const Quad<C> &Q, Dims d, const C *E0, const C *E1, C h2, const T *sg) {
            C sum[2];
            if (!Q.on)
                return;
            quad_residual<C, T>(Q, d, E0, E1, h2, sg, sum);
            Sp[0][tid] = sum[0];
            Sp[1][tid] = sum[1];
        };
        residual(A, dA, EA[0], EA[1], a.h2[0], a.s[0]);
        __syncthreads();
        if (two) {
            if (!KEEP && B.on) {
                quad_coeffs<C, T>(B, dB, a.bc, a.b[1], a.s[1], om);
                quad_weights(B.t, B.j, B.K, dB, a.w[1], wB);
            }
#pragma unroll
            for (int z = 0; z < 2; ++z)
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    B.r[c][z] = B.on ? restricted<C>(Sp, dA, 2 * B.t + ((B.j + z + c) & 1), B.j,
                                                     2 * B.K + z)
                                     : C(0);
            __syncthreads();               // Sp is written again below
            sweeps_down(B, EB[0], EB[1], a.h2[1], false);
            residual(B, dB, EB[0], EB[1], a.h2[1], a.s[1]);
            __syncthreads();
        }
        for (int c = tid; c < nc; c += TAIL_THREADS) {
            const int K = c / (dC.nx * dC.ny), rem = c - K * dC.nx * dC.ny;
            const int J = rem / dC.nx, I = rem - J * dC.nx;
            const double v = static_cast<double>(restricted<C>(Sp, two ? dB : dA, I, J, K));
            if (PHASE == TAIL_DOWN)
                a.state[TAIL_STATE_RS + c] = v;
            else
                rs[c] = v;
        }
    }
    if (PHASE == TAIL_DOWN) {
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int z = 0; z < 2; ++z)
                a.state[(2 * c + z) * TAIL_THREADS + tid] = A.e[c][z];
        return;
    }
    if (PHASE == TAIL_ALL) {
        // coarsest level: e = A^+ r in FP64, gs threads per output reduced by shuffles
        __syncthreads();
        int gs = 1;
        while (gs < 64 && 2 * gs * nc <= TAIL_THREADS)
            gs *= 2;
        const int outp = tid / gs, lane = tid % gs;
        double s = 0.0;
        if (outp < nc) {
            if (pvl) {
                for (int jj = lane; jj < nc; jj += gs)
                    s += Pv[jj * nc + outp] * rs[jj];
            } else {
                const double *pc = a.pinv + outp;
#pragma unroll 8
                for (int jj = lane; jj < nc; jj += gs)
                    s += pc[(size_t)jj * nc] * rs[jj];
            }
        }
        for (int o = gs >> 1; o > 0; o >>= 1)
            s += __shfl_xor(s, o, 64);
        if (lane == 0 && outp < nc)
            EC[outp] = static_cast<C>(s);
    } else {
        for (int c = tid; c < nc; c += TAIL_THREADS)
            EC[c] = static_cast<C>(a.state[TAIL_STATE_EC + c]);
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int z = 0; z < 2; ++z)
                A.e[c][z] = static_cast<C>(a.state[(2 * c + z) * TAIL_THREADS + tid]);
    }
    __syncthreads();
    auto coarsest = [&](int I, int J, int K) { return EC[(K * dC.ny + J) * dC.nx + I]; };
    if (two) {
        if (B.on)
            quad_prolong<C>(B, dB, a.bc, wB, coarsest);
        publish(B, EB[0], 0);
        __syncthreads();
        sweeps_up(B, EB[0], EB[1], a.h2[1]);
        const int hx = dB.nx / 2;
        quad_prolong<C>(A, dA, a.bc, wA, [&](int I, int J, int K) {
            return EB[(I + J + K) & 1][(K * dB.ny + J) * hx + (I >> 1)];
        });
    } else {
        quad_prolong<C>(A, dA, a.bc, wA, coarsest);
    }
    publish(A, EA[0], 0);
    if (!KEEP && PHASE == TAIL_ALL)
        quad_coeffs<C, T>(A, dA, a.bc, a.b[0], a.s[0], om);
    __syncthreads();
    sweeps_up(A, EA[0], EA[1], a.h2[0]);
    // the correction of the tail's first level goes back to global memory
    if (A.on) {
        using T2 = typename Vec2<T>::type;
        const int c0 = (2 * A.K * dA.ny + A.j) * dA.nx + 2 * A.t;
#pragma unroll
        for (int z = 0; z < 2; ++z) {
            const bool o = ((A.j + z) & 1) != 0;
            T2 v;
            v.x = static_cast<T>(pick2<C>(o, A.e[0][z], A.e[1][z]));
            v.y = static_cast<T>(pick2<C>(o, A.e[1][z], A.e[0][z]));
            *reinterpret_cast<T2 *>(a.e + c0 + z * dA.nx * dA.ny) = v;
        }
    }
}

// The coarsest correction in storage, by way of the arithmetic's type as every
// level's: FP16 is rounded twice, to FP32 and from there (the compiler would make
// one conversion of the two, and now and then another value).
template <typename TE>
__device__ __forceinline__ TE stored(double s)
{
    if constexpr (exact_order<TE>()) {
        float f = static_cast<float>(s);
        asm("" : "+v"(f));
        return static_cast<TE>(f);
    }
    return static_cast<TE>(s);
}

// Coarsest level by itself: e = A^+ r in FP64, a wave per row of the
// (symmetric) pseudo-inverse, four rows per workgroup, so that all of it is
// in flight at once.  720 cells: 4 us, where one workgroup takes 210.
template <typename TR, typename TE>
__global__ __launch_bounds__(256) void k_coarsest(int n, const double *__restrict__ pinv,
                                                  const TR *__restrict__ r, TE *__restrict__ e)
{
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= n)
        return;
    const double *p = pinv + (size_t)row * n;
    double s = 0.0;
#pragma unroll 4
    for (int c = lane; c < n; c += 64)
        s += p[c] * static_cast<double>(r[c]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        s += __shfl_xor(s, o, 64);
    if (lane == 0)
        e[row] = stored<TE>(s);
}

template <typename T>
void launch_tail(int nlev, const Dims *d, const double *h2, const void *const (*b)[3], void *const *e,
                 void *const *r, const void *const *sg, const unsigned *const *w, Bc bc,
                 int nu_pre, int nu_post, double omega, const double *pinv, int ncoarse,
                 bool warm, double *state, hipStream_t s)
{
    using C = typename Acc<T>::type;
    const dim3 cgrid((ncoarse + 3) / 4);
    if (nlev == 1) {
        hipLaunchKernelGGL((k_coarsest<T, T>), cgrid, dim3(256), 0, s, ncoarse, pinv,
                           (const T *)r[0], (T *)e[0]);
        return;
    }
    TailArgs<T> a{};
    a.n = nlev;
    for (int l = 0; l < nlev; ++l) {
        a.d[l] = d[l];
        a.h2[l] = (C)h2[l];
        for (int m = 0; m < 3; ++m)
            a.b[l][m] = (const T *)b[l][m];
        a.w[l] = w[l];
        a.s[l] = (const T *)sg[l];
    }
    a.r = (const T *)r[0];
    a.e = (T *)e[0];
    a.bc = bc;
    a.nu_pre = nu_pre;
    a.nu_post = nu_post;
    a.omega = (C)omega;
    a.warm = warm ? 1 : 0;
    a.pinv = pinv;
    a.ncoarse = ncoarse;
    a.state = state;
    if (ncoarse <= TAIL_SPLIT) {
        hipLaunchKernelGGL((k_tail_cycle<T, TAIL_ALL>), dim3(1), dim3(TAIL_THREADS), 0, s, a);
        return;
    }
    hipLaunchKernelGGL((k_tail_cycle<T, TAIL_DOWN>), dim3(1), dim3(TAIL_THREADS), 0, s, a);
    hipLaunchKernelGGL((k_coarsest<double, double>), cgrid, dim3(256), 0, s, ncoarse, pinv,
                       state + TAIL_STATE_RS, state + TAIL_STATE_EC);
    hipLaunchKernelGGL((k_tail_cycle<T, TAIL_UP>), dim3(1), dim3(TAIL_THREADS), 0, s, a);
}

#define PP_INSTANTIATE_TAIL(T)                                                                  \
    template void launch_tail<T>(int, const Dims *, const double *, const void *const (*)[3],   \
                                 void *const *, void *const *, const void *const *,             \
                                 const unsigned *const *, Bc, int, int, double, const double *, \
                                 int, bool, double *, hipStream_t);

PP_INSTANTIATE_TAIL(double)
PP_INSTANTIATE_TAIL(float)
PP_INSTANTIATE_TAIL(_Float16)

}  // namespace pp
