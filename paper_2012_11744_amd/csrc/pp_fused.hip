// pp_fused.hip -- the fused red-black Gauss-Seidel sweep (gfx950), the
// dominant kernel of the V-cycle: both colours of one sweep in one pass over
// the level, out of place.
//
// The update is the seven-point Gauss-Seidel step of Sec. 3.7.1 with
// relaxation 1 (the SOR iteration of that section with omega = 1), cells
// coloured red ((i+j+k) even) and black; walls (Sec. 3.8) zero the link
// coefficient of the wall face.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "pp_device.h"
#include "pp_internal.h"

namespace pp {

// ---------------------------------------------------------------------------
// Fused red-black Gauss-Seidel sweep (both colours in one pass, out of place).
//
// A block owns an FTX x FTY tile of an x-y plane and marches along z through a
// chunk of planes [k0, k1).  Each thread owns one x-pair of cells (2p, 2p+1)
// of one row: at every plane exactly one cell of a pair has each colour.  At
// step k a thread updates the first-colour cell of its pair in plane k and
// publishes it in an LDS plane slot; after one barrier the tile threads
// update the second-colour cell of plane k-1 from the slots (in-plane
// neighbours) and from their own registers (the z neighbours, which are the
// first-colour cells of the same pair in planes k-2 and k), and store the
// finished pair of plane k-1.
//
// The threads of a one-pair / one-row ring around the tile, and the planes
// k0-1 and k1, recompute first-colour values that belong to neighbouring
// tiles and chunks from the same inputs, so blocks never read each other's
// output (e_in is read only, e_out written only) and every cell gets the
// update of a red-black sweep.  Every input cell is fetched from memory once
// per sweep apart from the ring.
//
// The step has no data-dependent branches: every thread of the layout
// computes the first-colour cell of its pair, reading in-plane neighbours
// from LDS at a column chosen by the pair's colour parity; ring rows also
// publish the row beyond them (two extra LDS rows), padding columns hold
// zeros, and x-wall faces are zeroed as they are published.  Each plane is
// read through buffer resources: a missing plane has an empty range, and an
// inactive thread or a y-wall face uses an offset past the range, so those
// values arrive as zero from the hardware range check and nothing is masked
// after the load.  The loads of plane k+1+FPD therefore stay in flight across
// FPD steps; the loop is unrolled by the buffer rotation period so no buffer
// with loads in flight is copied.
// ---------------------------------------------------------------------------
constexpr int FTX = 128;                // tile width in cells (64 pairs)
constexpr int FTY = 8;                  // tile height in rows
constexpr int FPX = FTX / 2 + 2;        // pairs per row including the ring pairs
constexpr int FRY = FTY + 2;            // thread rows including the ring rows
constexpr int FTHREADS = (FPX * FRY + 63) / 64 * 64;   // whole waves
constexpr int FLW = FTX + 8;            // LDS row: cells i0-4 .. i0+FTX+3
constexpr int FLR = FTY + 4;            // LDS rows: j0-2 .. j0+FTY+1

// Planes of loads in flight beyond plane k+1, per storage type: two for FP32
// (its loads are small, so it needs more of them in flight); one for FP64,
// whose registers would otherwise spill, and for FP16 (measured best at one).
template <typename T>
struct FusedDepth {
    static constexpr int value = sizeof(T) == 4 ? 2 : 1;
};

// Inputs of one thread's pair at one plane, as loaded (storage precision).
// eo / byo: e_in and beta_y of the row beyond an outermost ring row (zero
// for the other threads, which read no such row).  Values a thread must
// treat as zero (inactive thread, missing plane, wall faces of y and z)
// arrive as zero from the buffer range check.
template <typename T>
struct PairIn {
    using T2 = typename Vec2<T>::type;
    T2 e, r, bx, by, bz, eo, byo;
    T2 sg;                     // diagonal term (general operator only)
};

// Buffer resource over one plane: loads at byte offsets >= `bytes` return
// zero and stores there are dropped.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const void *base, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes,
                                             0x00020000);
}

template <typename T>
__device__ __forceinline__ typename Vec2<T>::type ld_pair(__amdgpu_buffer_rsrc_t rs, unsigned off)
{
    using T2 = typename Vec2<T>::type;
    if constexpr (sizeof(T) == 8)
        return __builtin_bit_cast(T2, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
    else if constexpr (sizeof(T) == 4)
        return __builtin_bit_cast(T2, __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0));
    else
        return __builtin_bit_cast(T2, __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
}

template <typename T>
__device__ __forceinline__ void st_pair(__amdgpu_buffer_rsrc_t rs, unsigned off,
                                        typename Vec2<T>::type v)
{
    if constexpr (sizeof(T) == 8)
        __builtin_amdgcn_raw_buffer_store_b128(
            __builtin_bit_cast(unsigned __attribute__((ext_vector_type(4))), v), rs, off, 0, 0);
    else if constexpr (sizeof(T) == 4)
        __builtin_amdgcn_raw_buffer_store_b64(
            __builtin_bit_cast(unsigned __attribute__((ext_vector_type(2))), v), rs, off, 0, 0);
    else
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rs, off, 0, 0);
}

// an offset past every plane (planes of a fused sweep stay below 2^31 bytes)
constexpr unsigned OFF_NONE = 0x80000000u;

__device__ __forceinline__ int slot3(int k) { return ((k % 3) + 3) % 3; }

// The Gauss-Seidel quotient.  FP32 arithmetic (FP32 and FP16 storage) takes
// the hardware reciprocal (within 1 ulp) times the numerator: the smoother
// only has to reduce the error, and its result is a preconditioner that the
// FP64 outer iteration corrects; FP64 keeps the exact quotient.
__device__ __forceinline__ float gs_quot(float a, float b) { return a * __builtin_amdgcn_rcpf(b); }
__device__ __forceinline__ double gs_quot(double a, double b) { return a / b; }

// Block id -> (tile x, tile y, chunk), spreading contiguous ranges of tiles over
// the 8 XCDs: consecutive workgroups are dispatched round-robin to the XCDs,
// so workgroup b is given logical tile (b % 8) * (n / 8) + b / 8, which keeps
// neighbouring tiles (which share halo lines) in one XCD's L2.  The grid is
// (tiles of a plane) x (z chunks); b is the linear workgroup index.
__device__ __forceinline__ void xcd_tile(unsigned tx_tiles, unsigned ty_tiles, int &bxi, int &byi,
                                         int &bzi)
{
    const unsigned nb = gridDim.x * gridDim.y;
    unsigned b = blockIdx.x + gridDim.x * blockIdx.y;
    const unsigned full = nb & ~7u;
    if (b < full)
        b = (b & 7u) * (full >> 3) + (b >> 3);
    bxi = (int)(b % tx_tiles);
    byi = (int)((b / tx_tiles) % ty_tiles);
    bzi = (int)(b / (tx_tiles * ty_tiles));
}

// SIG: the general operator's diagonal term, stored as h^2 sigma, is read
// with the other inputs and added to the diagonal.  In every variant a cell with a
// zero diagonal (no open face, no diagonal term) is excluded and gets 0.
// WHOLE: the march runs whole blocks of its unroll length (see the loop).
// om: the over-relaxation of eq. beta_pressure, e <- (1 - om) e + om e_GS
// (ZERO: the old value is 0).
template <typename T, bool ZERO, bool SIG, bool WHOLE>
__global__ __launch_bounds__(FTHREADS) void k_rbgs_fused(Dims d, Bc bc, const T *__restrict__ bx,
                                                         const T *__restrict__ by,
                                                         const T *__restrict__ bz,
                                                         const T *__restrict__ r,
                                                         const T *__restrict__ ein,
                                                         T *__restrict__ eout,
                                                         const T *__restrict__ sg,
                                                         typename Acc<T>::type h2,
                                                         typename Acc<T>::type om, int c0, int kz,
                                                         unsigned tx_tiles, unsigned ty_tiles)
{
    using C = typename Acc<T>::type;
    using T2 = typename Vec2<T>::type;
    const C om1 = C(1) - om;
    constexpr int FPD = FusedDepth<T>::value;   // planes of loads in flight beyond k+1
    constexpr int FNB = FPD + 3;                // input buffers: k-1, k, k+1 and those in flight
    // LDS: e_in, beta_x and beta_y of planes k and k+1 (two slots) for the
    // in-plane neighbours, and the first-colour values of planes k-2..k
    __shared__ C SE[2][FLR][FLW];
    __shared__ C SX[2][FLR][FLW];
    __shared__ C SY[2][FLR][FLW];
    __shared__ C RED[3][FLR][FLW];
    int bxi, byi, bzi;
    xcd_tile(tx_tiles, ty_tiles, bxi, byi, bzi);
    const int i0 = bxi * FTX, j0 = byi * FTY;
    const int k0 = bzi * kz;
    const int k1 = min(k0 + kz, d.nz);

    const int tid = threadIdx.x;
    const bool in_layout = tid < FPX * FRY;
    // threads past the layout shadow thread 0 (inactive: they publish and
    // store nothing, and their LDS reads stay inside the arrays)
    const int tl = in_layout ? tid : 0;
    const int pl = tl % FPX - 1;      // pair within the tile; -1 and FTX/2 are ring pairs
    const int rl = tl / FPX - 1;      // row within the tile; -1 and FTY are ring rows
    int x = i0 + 2 * pl;
    int j = j0 + rl;
    // the pair / row just past the grid's end is the periodic wrap: ring only
    const bool ringx = pl < 0 || pl >= FTX / 2 || x == d.nx;
    const bool ringy = rl < 0 || rl >= FTY || j == d.ny;
    bool act = in_layout;             // holds a pair of the grid
    if (x < 0) {
        if (bc.x) act = false; else x += d.nx;
    } else if (x >= d.nx) {
        if (bc.x || x > d.nx) act = false; else x = 0;
    }
    if (j < 0) {
        if (bc.y) act = false; else j += d.ny;
    } else if (j >= d.ny) {
        if (bc.y || j > d.ny) act = false; else j = 0;
    }
    if (!act) {
        x = 0;
        j = 0;
    }
    const bool owned = act && !ringx && !ringy;
    const bool dn_row = act && rl < 0;                 // publishes the row below it
    const bool up_row = act && ringy && rl >= 0;       // publishes the row above it
    const int jm = (j == 0) ? d.ny - 1 : j - 1;
    const int jp = (j == d.ny - 1) ? 0 : j + 1;
    const bool wyl = bc.y && j == 0, wyh = bc.y && j == d.ny - 1;
    const bool wxl = bc.x && x == 0;
    const int jo = dn_row ? jm : (up_row ? jp : j);
    const bool zo = up_row ? wyh : wyl;   // the y faces published in row lyo are walls
    const bool beyond = dn_row || up_row;   // only these threads read the row beyond
    // byte offsets of the pair within a plane; OFF_NONE reads zero (and, for
    // the row beyond, spares the other threads a load of their own row)
    const unsigned oc0 = (unsigned)(((size_t)j * d.nx + x) * sizeof(T));
    const unsigned oo0 = (unsigned)(((size_t)jo * d.nx + x) * sizeof(T));
    const unsigned oc = act ? oc0 : OFF_NONE;
    const unsigned oo = (act && beyond) ? oo0 : OFF_NONE;
    const unsigned ocy = (act && !wyl) ? oc0 : OFF_NONE;
    const unsigned ooy = (act && beyond && !zo) ? oo0 : OFF_NONE;
    const unsigned ost = owned ? oc0 : OFF_NONE;
    const unsigned pbytes = (unsigned)((size_t)d.nx * d.ny * sizeof(T));
    const int lx = 2 * pl + 4;        // LDS column of the pair's first cell
    const int ly = rl + 2;            // LDS row of the pair
    const int lyo = dn_row ? ly - 1 : (up_row ? ly + 1 : ly);

    // plane q: its wrapped index, and whether it exists (walls end the grid)
    auto plane = [&](int q, int &qw) -> bool {
        qw = q;
        if (q < 0) {
            if (bc.z) { qw = 0; return false; }
            qw = q + d.nz;
        } else if (q >= d.nz) {
            if (bc.z) { qw = 0; return false; }
            qw = q - d.nz;
        }
        return true;
    };
    auto load_in = [&](int q, PairIn<T> &v) __attribute__((always_inline)) {
        int qw;
        const unsigned nb = plane(q, qw) ? pbytes : 0u;
        const size_t pb = (size_t)qw * pbytes;
        auto rs = [&](const T *base, unsigned n) {
            return plane_rsrc(reinterpret_cast<const char *>(base) + pb, n);
        };
        if (!ZERO) {
            const auto re = rs(ein, nb);
            v.e = ld_pair<T>(re, oc);
            v.eo = ld_pair<T>(re, oo);
        }
        v.r = ld_pair<T>(rs(r, nb), oc);
        v.bx = ld_pair<T>(rs(bx, nb), oc);
        const auto ry = rs(by, nb);
        v.by = ld_pair<T>(ry, ocy);
        v.byo = ld_pair<T>(ry, ooy);
        v.bz = ld_pair<T>(rs(bz, (bc.z && qw == 0) ? 0u : nb), oc);   // the wall below plane 0
        if (SIG)
            v.sg = ld_pair<T>(rs(sg, nb), oc);
    };
    auto pick = [](int o, T2 v) -> C { return C(o ? v.y : v.x); };
    // Only active threads write LDS: the positions of inactive ones (past a
    // wall, past a ragged grid end) keep the zeros of the initial fill, and
    // the row a wrapping ring row publishes beyond itself may be the own row
    // of an inactive thread.
    auto publish = [&](int slot, const PairIn<T> &v) __attribute__((always_inline)) {
        if (!act)
            return;
        if (!ZERO) {
            SE[slot][ly][lx] = C(v.e.x);
            SE[slot][ly][lx + 1] = C(v.e.y);
        }
        SX[slot][ly][lx] = wxl ? C(0) : C(v.bx.x);
        SX[slot][ly][lx + 1] = C(v.bx.y);
        SY[slot][ly][lx] = C(v.by.x);
        SY[slot][ly][lx + 1] = C(v.by.y);
        if (beyond) {
            if (!ZERO) {
                SE[slot][lyo][lx] = C(v.eo.x);
                SE[slot][lyo][lx + 1] = C(v.eo.y);
            }
            SY[slot][lyo][lx] = C(v.byo.x);
            SY[slot][lyo][lx + 1] = C(v.byo.y);
        }
    };

    // padding columns and rows read as zero
    for (int i = tid; i < 2 * FLR * FLW; i += FTHREADS) {
        (&SE[0][0][0])[i] = C(0);
        (&SX[0][0][0])[i] = C(0);
        (&SY[0][0][0])[i] = C(0);
    }
    for (int i = tid; i < 3 * FLR * FLW; i += FTHREADS)
        (&RED[0][0][0])[i] = C(0);

    C red_km2 = C(0), red_km1 = C(0);
    // in-plane faces of the second-colour cell of plane k-1 (read at step k-1)
    C sxl = C(0), sxh = C(0), syl = C(0), syh = C(0);

    // One plane step: inputs of planes k-1 (pm), k (pc), k+1 (pn) resident,
    // plane k+1+FPD (pf) loaded here and left in flight for FPD steps.
    auto step = [&](int k, PairIn<T> &pm, PairIn<T> &pc, PairIn<T> &pn, PairIn<T> &pf)
                    __attribute__((always_inline)) {
        load_in(k + 1 + FPD, pf);
        const int si = k & 1;
        int kw;
        const bool kin = act && plane(k, kw);
        const int o = (c0 + j + k) & 1;   // first-colour cell of the pair in plane k
        // phase A: first colour of plane k
        const int ca = lx + o;
        const C xl = SX[si][ly][ca], xh = SX[si][ly][ca + 1];
        const C yl = SY[si][ly][ca], yh = SY[si][ly + 1][ca];
        const C zl = pick(o, pc.bz), zh = pick(o, pn.bz);
        C diag = (xl + xh) + (yl + yh) + (zl + zh);
        if (SIG)
            diag += pick(o, pc.sg);          // h^2 sigma
        C s = C(0);
        if (!ZERO)
            s = xl * SE[si][ly][ca - 1] + xh * SE[si][ly][ca + 1] + yl * SE[si][ly - 1][ca] +
                yh * SE[si][ly + 1][ca] + zl * pick(o, pm.e) + zh * pick(o, pn.e);
        const C val = gs_quot(s - h2 * pick(o, pc.r), diag);
        // a missing plane (0/0) and an excluded cell (zero diagonal) get 0
        const C rel = ZERO ? om * val : om1 * pick(o, pc.e) + om * val;
        const C red = (kin && diag > C(0)) ? rel : C(0);
        // in-plane faces of this plane's second-colour cell, for phase B at
        // the next step (the slot is overwritten before then)
        const int cb = lx + 1 - o;
        const C nxl = SX[si][ly][cb], nxh = SX[si][ly][cb + 1];
        const C nyl = SY[si][ly][cb], nyh = SY[si][ly + 1][cb];
        if (act)
            RED[slot3(k)][ly][ca] = red;
        publish(si ^ 1, pn);          // plane k+1 for the next step's phase A
        __syncthreads();
        // phase B: second colour of plane k-1 (at the column of this plane's
        // first colour); the store of a thread outside the tile is dropped
        const int kb = k - 1;
        if (kb >= k0 && kb < k1) {
            const int sb = slot3(kb);
            const C bzl = pick(o, pm.bz), bzh = pick(o, pc.bz);
            const C sbv = sxl * RED[sb][ly][ca - 1] + sxh * RED[sb][ly][ca + 1] +
                          syl * RED[sb][ly - 1][ca] + syh * RED[sb][ly + 1][ca] + bzl * red_km2 +
                          bzh * red;
            C dg = (sxl + sxh) + (syl + syh) + (bzl + bzh);
            if (SIG)
                dg += pick(o, pm.sg);
            const C q = gs_quot(sbv - h2 * pick(o, pm.r), dg);
            const C blk = dg > C(0) ? (ZERO ? om * q : om1 * pick(o, pm.e) + om * q) : C(0);
            T2 outv;
            outv.x = static_cast<T>(o ? red_km1 : blk);
            outv.y = static_cast<T>(o ? blk : red_km1);
            st_pair<T>(plane_rsrc(reinterpret_cast<const char *>(eout) + (size_t)kb * pbytes, pbytes),
                       ost, outv);
        }
        red_km2 = red_km1;
        red_km1 = red;
        sxl = nxl;
        sxh = nxh;
        syl = nyl;
        syh = nyh;
    };

    // FNB input buffers rotate through the roles (k-1, k, k+1, and the planes
    // in flight); the loop is unrolled by FNB so no buffer with loads in
    // flight is ever copied.  WHOLE: it runs whole blocks of FNB steps, the
    // last up to FNB - 1 steps past k1 (they store nothing), with one exit
    // test per block, which keeps the loop-carried registers in place across
    // the back edge; an exit after every step makes the compiler copy
    // registers with loads in flight there (waiting for them), which costs
    // less than the extra steps only on short chunks.
    PairIn<T> buf[FNB];
#pragma unroll
    for (int u = 0; u < FNB - 1; ++u)
        load_in(k0 - 2 + u, buf[u]);
    __syncthreads();                  // the zero fill is complete
    publish((k0 - 1) & 1, buf[1]);
    __syncthreads();
    if constexpr (WHOLE) {
        for (int k = k0 - 1; k <= k1; k += FNB) {
#pragma unroll
            for (int u = 0; u < FNB; ++u)
                step(k + u, buf[u % FNB], buf[(u + 1) % FNB], buf[(u + 2) % FNB],
                     buf[(u + FNB - 1) % FNB]);
        }
    } else {
        for (int k = k0 - 1;;) {
#pragma unroll
            for (int u = 0; u < FNB; ++u) {
                step(k, buf[u % FNB], buf[(u + 1) % FNB], buf[(u + 2) % FNB],
                     buf[(u + FNB - 1) % FNB]);
                if (++k > k1)
                    return;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// launcher
// ---------------------------------------------------------------------------

// Workgroups of a fused-sweep kernel that the whole GPU holds at once
// (occupancy x CUs), queried once per kernel instantiation and device.  The
// cache lives in the (T, ZERO) instantiation: the two variants of one storage
// type have the same function type but different register counts.
template <typename T, bool ZERO, bool SIG>
static long long fused_slots()
{
    static long long cached[64] = {0};
    int dev = 0;
    (void)hipGetDevice(&dev);
    if (dev < 0 || dev >= 64)
        dev = 0;
    if (cached[dev] == 0) {
        int per_cu = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_rbgs_fused<T, ZERO, SIG, false>,
                                                         FTHREADS, 0) != hipSuccess ||
            per_cu < 1)
            per_cu = 1;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            cus < 1)
            cus = 256;
        cached[dev] = (long long)per_cu * cus;
    }
    return cached[dev];
}

// Marches of at least this many plane steps run whole blocks of the unroll
// length (the WHOLE variants): the few steps a block runs past the chunk cost
// less there than the register copies at the back edge of the other form.
constexpr int WHOLE_MIN_STEPS = 48;

// Chunk length along z.  A chunk of kz planes marches kz + halo plane steps
// (halo: the planes beyond its ends, recomputed) and takes the time of about
// two more to start; `slots` workgroups are resident at once, so the pass takes
// rounds x (kz + halo + 2) steps, and the chunk that makes this least is used
// (the longest of equals: less recomputed).  It is at least kmin planes, in at
// most max_chunks chunks.  Where the tiles do not divide the slots,
// the chunk that fills them exactly leaves a few workgroups to a second round:
// 96 x 80 x 112 (20 tiles): 13 chunks of 9 planes, 260 workgroups on 256 CUs,
// 22.4 us zero start; 12 chunks of 10 planes, one round, 15.1 us.
static int chunk_planes(int nz, long long tiles, long long slots, int halo, int kmin,
                        long long max_chunks)
{
    int best = nz;
    long long cost = -1;
    if (kmin > nz)
        kmin = nz;
    // the most chunks that R rounds hold, R = 1, 2, ...
    for (long long R = (tiles + slots - 1) / slots, R1 = R + 16; R < R1; ++R) {
        long long m = R * slots / tiles;
        if (m > max_chunks)
            m = max_chunks;
        int kz = (int)((nz + m - 1) / m);
        if (kz < kmin)
            kz = kmin;
        const long long c = (tiles * ((nz + kz - 1) / kz) + slots - 1) / slots * (kz + halo + 2);
        if (cost < 0 || c < cost) {
            cost = c;
            best = kz;
        }
        if (kz == kmin || m == max_chunks)
            break;
    }
    return best;
}

template <typename T>
void prepare_fused()
{
    (void)fused_slots<T, true, false>();
    (void)fused_slots<T, false, false>();
    (void)fused_slots<T, true, true>();
    (void)fused_slots<T, false, true>();
}

template <typename T>
void launch_rbgs_fused(Dims d, Bc bc, const T *bx, const T *by, const T *bz, const T *r,
                       const T *ein, T *eout, const T *sg, double h2, double omega,
                       int first_colour, bool zero, hipStream_t s)
{
    using C = typename Acc<T>::type;
    const unsigned tx = (d.nx + FTX - 1) / FTX, ty = (d.ny + FTY - 1) / FTY;
    const long long slots = sg ? (zero ? fused_slots<T, true, true>() : fused_slots<T, false, true>())
                               : (zero ? fused_slots<T, true, false>() : fused_slots<T, false, false>());
    const int kz = chunk_planes(d.nz, (long long)tx * ty, slots, 2, 4, d.nz);
    const unsigned tz = (d.nz + kz - 1) / kz;
    const dim3 grid(tx * ty, tz);   // distinct shapes per level in profiles
    const bool whole = kz + 2 >= WHOLE_MIN_STEPS;   // a chunk marches kz + 2 steps
#define PP_FUSED_LAUNCH(Z, S)                                                                  \
    do {                                                                                       \
        if (whole)                                                                             \
            PP_LAUNCH((k_rbgs_fused<T, Z, S, true>), grid, dim3(FTHREADS), 0, s, d, bc, bx,    \
                      by, bz, r, ein, eout, sg, (C)h2, (C)omega, first_colour, kz, tx, ty);    \
        else                                                                                   \
            PP_LAUNCH((k_rbgs_fused<T, Z, S, false>), grid, dim3(FTHREADS), 0, s, d, bc, bx,   \
                      by, bz, r, ein, eout, sg, (C)h2, (C)omega, first_colour, kz, tx, ty);    \
    } while (0)
    if (sg) {
        if (zero)
            PP_FUSED_LAUNCH(true, true);
        else
            PP_FUSED_LAUNCH(false, true);
    } else {
        if (zero)
            PP_FUSED_LAUNCH(true, false);
        else
            PP_FUSED_LAUNCH(false, false);
    }
#undef PP_FUSED_LAUNCH
}

// ---------------------------------------------------------------------------
// Two sweeps in one pass.
//
// The plane step above, extended by two phases that lag behind it.  At step k
//   A: first colour of plane k, sweep 1 (from e_in, as above);
//   B: second colour of plane k-1, sweep 1;
//   C: first colour of plane k-2, sweep 2, from the finished sweep-1 values;
//   D: second colour of plane k-3, sweep 2, which completes that plane.
// Of a cell's six neighbours three are the thread's own: the other cell of its
// pair and the same cell in the planes above and below, all in registers.  The
// other three, the next pair's cell in x and the rows beside it, are read from
// an LDS plane written one step earlier (A from the published inputs, B from
// A's values, C from B's, D from C's).  Every such plane holds one value per
// pair, since a phase reads the other colour only, so a wave reads consecutive
// words.  C and D update the same cells as A and B two steps before, so they
// reuse the coefficients, reciprocal diagonal and right-hand side of A and B,
// carried in registers.  One barrier per step separates A (and the publication
// of the next plane's inputs) from B, C and D.  Each phase consumes one ring
// cell, so the ring around the tile is two pairs wide and three rows deep, and
// a chunk of output planes [k0, k1) is marched from k0-3 to k1+2.  Per cell the
// pass moves the bytes of one sweep.
//
// What bounds it (256^3 FP32, one workgroup of 512 threads per CU): mostly its
// loads.  With the arithmetic taken out a march took 121 of then 130 us, whatever
// the number of planes in flight (1 to 9), with the loads taken out 80.  An L1 has
// 73 reads on their way on average (75 in the zero-start pass; the copy kernel, at
// the rate of HBM, 91, the residual update 80), and waits for them in 44% (53%) of
// its cycles; the rest is the latency of the plane step.  A row of 72 cells that
// starts 16 bytes before a cache line touches four lines for 2.25, so rows start
// on a line (three).  Measured, regular / zero start: 256^3 FP32 133 / 105 ->
// 120 / 101 us, 112 / 96 since the outer kernels stream past the caches (512^3
// 1006 / 784 -> 877 / 730), FP16 storage 95 / 93 -> 80 / 85; FP64 in this form,
// with r.z, 191 / 175, where two single sweeps take 335 / 323 and the dot product
// 47; at 64^3 FP64 10.6 / 10.1, where a launch per colour takes 8 x 5 for two
// sweeps on each side.
// ---------------------------------------------------------------------------
constexpr int GTX = 64;                   // tile width in cells (32 pairs)
constexpr int GTY = 8;                    // tile height in rows
constexpr int GPX = GTX / 2 + 4;          // pairs per row: two ring pairs on each side
constexpr int GRY = GTY + 6;              // rows: three ring rows on each side
constexpr int GTHREADS = (GPX * GRY + 63) / 64 * 64;
constexpr int GLW = GPX + 2;              // LDS row: the pairs and one beyond on each side
constexpr int GLR = GRY + 2;              // LDS rows: one beyond on each side

// Whole-array buffer resources (FLAT) take a plane's byte offset in the 32-bit
// address of each load: a missing plane is at an offset past every array, and
// that offset plus OFF_NONE still does not wrap.  Arrays up to this size.
constexpr unsigned FLAT_NONE = 0x7ffffff0u;
inline bool fused2_flat(Dims d, size_t word) { return cells(d) * word <= FLAT_NONE; }

// what phase A (B) computed for a cell, for phase C (D) two steps later
template <typename C>
struct GsLag {
    C xi, xo, yl, yh, zl, zh;       // link coefficients (xi: inside the pair, xo: beyond it)
    C inv;                          // om / diagonal, or 0 for an excluded cell or missing plane
    C r;                            // right-hand side (EXACT: h^2 r, rounded)
};

__device__ __forceinline__ float om_over(float om, float d) { return om * __builtin_amdgcn_rcpf(d); }
__device__ __forceinline__ double om_over(double om, double d) { return om / d; }

// a b, kept a product of its own (no contraction with the sum that takes it)
template <typename C>
__device__ __forceinline__ C rounded_product(C a, C b)
{
#pragma clang fp contract(off)
    return a * b;
}

// om: the over-relaxation of eq. beta_pressure, folded into the reciprocal
// diagonal that the lag registers carry (inv = om / diag), so every phase
// forms e <- (1 - om) e + inv (sum - h^2 r); the old value of phases A and B
// is e_in (0 in the ZERO pass), that of C and D the sweep-1 value.
// DOT (FP32 and FP64 storage, regular pass): also the partial sums of r . e_out over each
// workgroup's output cells, r the pass's own right-hand side, products summed
// in FP64 (the outer iteration's residual against the preconditioned one,
// both in units of the V-cycle's scale); part[workgroup].  The values of r that
// phases C and D already carry supply it (as h^2 r), so nothing more is loaded.
// CLOSED: the operator may have closed links, so a cell may be excluded (the
// pressure operator has none).  Such a cell holds what the prolongation left
// there and gets 0, as from the other smoothers.
// FP16 storage sums x, y, z faces low before high (EXACT): its iterates
// repeat only with every FP32 rounding, so which products are fused is spelt
// out below.
template <typename T, bool ZERO, bool SIG, bool CLOSED, bool DOT, bool WHOLE, bool FLAT>
__global__ __launch_bounds__(GTHREADS, sizeof(T) == 2 ? 4 : 2) void k_rbgs_fused2(
    Dims d, Bc bc, const T *__restrict__ bx, const T *__restrict__ by, const T *__restrict__ bz,
    const T *__restrict__ r, const T *__restrict__ ein, T *__restrict__ eout,
    const T *__restrict__ sg, typename Acc<T>::type h2, typename Acc<T>::type om, int c0, int kz,
    unsigned tx_tiles, unsigned ty_tiles, double *__restrict__ part)
{
    using C = typename Acc<T>::type;
    using T2 = typename Vec2<T>::type;
    constexpr bool EXACT = std::is_same<T, _Float16>::value;
    // The loop is unrolled by the buffer count FNB, a multiple of both slot
    // periods (2 and NRED), so every LDS slot index is a compile-time constant.
    constexpr int FPD = two_sweep_depth(sizeof(T));
    constexpr int FNB = two_sweep_unroll(sizeof(T));
    constexpr int NRED = FNB % 3 == 0 ? 3 : (FNB % 4 == 0 ? 4 : 5);
    static_assert(FNB % 2 == 0 && FNB % NRED == 0, "slot periods");
    static_assert(!DOT || (!ZERO && !SIG), "the dot product rides on regular passes");
    const C om1 = C(1) - om;
    __shared__ C SE[2][GLR * GLW];        // e_in of planes k, k+1: second colour
    __shared__ C SX[2][GLR * GLW];        // beta_x of planes k, k+1: a pair's low face
    __shared__ T2 SY[2][GLR * GLW];       // beta_y of planes k, k+1: both cells
    __shared__ C RED1[NRED][GLR * GLW];   // phase A values (sweep 1, first colour)
    __shared__ C BLK1[2][GLR * GLW];      // phase B values (sweep 1, second colour)
    __shared__ C RED2[2][GLR * GLW];      // phase C values (sweep 2, first colour)
    int bxi, byi, bzi;
    xcd_tile(tx_tiles, ty_tiles, bxi, byi, bzi);
    const int i0 = bxi * GTX, j0 = byi * GTY;
    const int k0 = bzi * kz;
    const int k1 = min(k0 + kz, d.nz);
    const int yend = min(j0 + GTY, d.ny);

    const int tid = threadIdx.x;
    const bool in_layout = tid < GPX * GRY;
    const int tl = in_layout ? tid : 0;
    const int pl = tl % GPX;          // pair of the tile; the first two and the last two are ring
    const int rl = tl / GPX - 3;      // row within the tile; -3..-1 and those past yend are ring
    const int xu = i0 + 2 * pl, ju = j0 + rl;
    int x = xu, j = ju;
    // A tile is read from i0 on, so that its rows start on a cache line, and
    // owns the cells from i0 + 4 (with a wall at x = 0 the first tile owns from 0)
    // to i0 + GTX + 3; along a periodic x the tiles own [4, nx + 4).  Pairs and
    // rows past the grid's end wrap when periodic (ring: at most two pairs,
    // three rows); with walls they hold no cell.
    const int xlim = bc.x ? d.nx : d.nx + 4;          // end of the cells owned along x
    const int xown = bc.x && i0 == 0 ? 0 : i0 + 4, xend = min(i0 + GTX + 4, xlim);
    bool act = in_layout;
    if (xu >= d.nx) {
        if (bc.x || xu >= d.nx + 8) act = false; else x = xu - d.nx;
    }
    if (ju < 0) {
        if (bc.y) act = false; else j = ju + d.ny;
    } else if (ju >= d.ny) {
        if (bc.y || ju >= d.ny + 3) act = false; else j = ju - d.ny;
    }
    if (!act) {
        x = 0;
        j = 0;
    }
    const bool owned = act && xu >= xown && xu < xend && rl >= 0 && ju < yend;
    const bool dn_row = act && rl == -3;              // publishes the row below it
    const bool up_row = act && ju == yend + 2;        // publishes the row above it
    const int jm = (j == 0) ? d.ny - 1 : j - 1;
    const int jp = (j == d.ny - 1) ? 0 : j + 1;
    const bool wyl = bc.y && j == 0, wyh = bc.y && j == d.ny - 1;
    const bool wxl = bc.x && x == 0;
    const int jo = dn_row ? jm : jp;
    const bool beyond = dn_row || up_row;   // only these threads read the row beyond
    const unsigned oc0 = (unsigned)(((size_t)j * d.nx + x) * sizeof(T));
    const unsigned oo0 = (unsigned)(((size_t)jo * d.nx + x) * sizeof(T));
    const unsigned oc = act ? oc0 : OFF_NONE;
    const unsigned oo = beyond ? oo0 : OFF_NONE;
    const unsigned ocy = (act && !wyl) ? oc0 : OFF_NONE;
    const unsigned ooy = (up_row && !wyh) ? oo0 : OFF_NONE;   // the row below has no face to lend
    const unsigned ost = owned ? oc0 : OFF_NONE;
    const unsigned pbytes = (unsigned)((size_t)d.nx * d.ny * sizeof(T));
    const int li = (rl + 4) * GLW + pl + 1;          // LDS entry of the pair
    const int lio = li + (dn_row ? -GLW : GLW);      // ... of the row beyond

    // plane q: its wrapped index, and whether it is read.  Planes past the last
    // one needed lie outside the array where the grid does not have them: the
    // range check of a whole-array resource answers those with zeros, resources
    // of single planes must not be made for them.  (Bounding both forms costs the
    // FP32 cases 2%: 161 -> 177 registers.)
    auto plane = [&](int q, int &qw) {
        return march_plane<!FLAT>(q, d.nz, bc.z, two_sweep_last_plane(k1), qw);
    };
    const unsigned abytes = FLAT ? pbytes * (unsigned)d.nz : 0u;
    const auto fe = plane_rsrc(ein, abytes), fr = plane_rsrc(r, abytes),
               fbx = plane_rsrc(bx, abytes), fby = plane_rsrc(by, abytes),
               fbz = plane_rsrc(bz, abytes), fsg = plane_rsrc(sg, abytes),
               fo = plane_rsrc(eout, abytes);
    auto load_in = [&](int q, PairIn<T> &v) __attribute__((always_inline)) {
        int qw;
        const bool ok = plane(q, qw);
        const bool okz = ok && !(bc.z && qw == 0);   // the wall below plane 0
        if constexpr (FLAT) {
            const unsigned po = ok ? (unsigned)qw * pbytes : FLAT_NONE;
            const unsigned poz = okz ? po : FLAT_NONE;
            if (!ZERO) {
                v.e = ld_pair<T>(fe, oc + po);
                v.eo = ld_pair<T>(fe, oo + po);
            }
            v.r = ld_pair<T>(fr, oc + po);
            v.bx = ld_pair<T>(fbx, oc + po);
            v.by = ld_pair<T>(fby, ocy + po);
            v.byo = ld_pair<T>(fby, ooy + po);
            v.bz = ld_pair<T>(fbz, oc + poz);
            if (SIG)
                v.sg = ld_pair<T>(fsg, oc + po);
        } else {
            const unsigned nb = ok ? pbytes : 0u;
            const size_t pb = (size_t)qw * pbytes;
            auto rs = [&](const T *base, unsigned n) {
                return plane_rsrc(reinterpret_cast<const char *>(base) + pb, n);
            };
            if (!ZERO) {
                const auto re = rs(ein, nb);
                v.e = ld_pair<T>(re, oc);
                v.eo = ld_pair<T>(re, oo);
            }
            v.r = ld_pair<T>(rs(r, nb), oc);
            v.bx = ld_pair<T>(rs(bx, nb), oc);
            const auto ry = rs(by, nb);
            v.by = ld_pair<T>(ry, ocy);
            v.byo = ld_pair<T>(ry, ooy);
            v.bz = ld_pair<T>(rs(bz, okz ? nb : 0u), oc);
            if (SIG)
                v.sg = ld_pair<T>(rs(sg, nb), oc);
        }
    };
    auto store_out = [&](int q, T2 v) __attribute__((always_inline)) {
        if constexpr (FLAT)
            st_pair<T>(fo, ost + (unsigned)q * pbytes, v);
        else
            st_pair<T>(plane_rsrc(reinterpret_cast<const char *>(eout) + (size_t)q * pbytes, pbytes),
                       ost, v);
    };
    auto pick = [](int o, T2 v) -> C { return C(o ? v.y : v.x); };
    // inputs of a plane whose first-colour cells are at offset o1 of this row
    auto publish = [&](int slot, int o1, const PairIn<T> &v) __attribute__((always_inline)) {
        if (!act)
            return;
        if (!ZERO)
            SE[slot][li] = pick(1 - o1, v.e);
        SX[slot][li] = C(v.bx.x);
        SY[slot][li] = v.by;
        if (beyond) {
            if (!ZERO)
                SE[slot][lio] = pick(o1, v.eo);
            if (up_row)
                SY[slot][lio] = v.byo;
        }
    };

    for (int i = tid; i < GLR * GLW; i += GTHREADS) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            SE[q][i] = C(0);
            SX[q][i] = C(0);
            SY[q][i] = T2{T(0), T(0)};
            BLK1[q][i] = C(0);
            RED2[q][i] = C(0);
        }
#pragma unroll
        for (int q = 0; q < NRED; ++q)
            RED1[q][i] = C(0);
    }

    // own-pair values of earlier planes: A's of k-1, k-2; B's of k-2, k-3;
    // C's of k-3, k-4
    C red_km1 = C(0), red_km2 = C(0);
    C blk_km1 = C(0), blk_km2 = C(0);
    C r2_km1 = C(0), r2_km2 = C(0);
    // faces of the second-colour cell of plane k-1
    C sxi = C(0), sxo = C(0), syl = C(0), syh = C(0);
    GsLag<C> a1{}, a2{}, b1{}, b2{};
    // DOT: r of C's cell of the previous step (the first-colour cell of the
    // plane phase D completes), and the sum of h^2 r e_out
    C rc = C(0);
    double dacc = 0.0;

    // LDS slots are counted from the first plane of the march, kb = k0 - 3:
    // plane k's inputs sit in slot (k - kb) mod 2, its phase-A values in slot
    // (k - kb) mod NRED; u is the unrolled step index, (k - kb) mod FNB
    const int kb = two_sweep_first(k0);
    const int p0 = (c0 + j + kb) & 1;
    // the next pair in x of a cell at offset p0 of its pair, and at the other
    const int ladj[2] = {li + (p0 ? 1 : -1), li + (p0 ? -1 : 1)};
    // waves that hold only outer ring rows, whose phase C and D values no
    // thread reads, skip those phases
    const bool cdw = __any(in_layout && rl >= -1 && rl <= GTY);
    // sum of the six links of a cell at offset o: own values ei (x) and zl, zh
    // (z), the rest from LDS
    auto links6 = [&](bool second, int o, C xi, C xo, C yl, C yh, C zl, C zh, C ei, C eo, C el,
                      C eh, C fl, C fh) __attribute__((always_inline)) -> C {
        C t;
        if (EXACT) {
            const C x0 = o ? xi : xo, x1 = o ? xo : xi;
            const C e0 = o ? ei : eo, e1 = o ? eo : ei;
            t = second ? fma(x1, e1, x0 * e0) : fma(x0, e0, x1 * e1);
        } else {
            t = fma(xo, eo, xi * ei);
        }
        t = fma(yl, el, t);
        t = fma(yh, eh, t);
        t = fma(zl, fl, t);
        return fma(zh, fh, t);
    };
    auto minus_h2r = [&](C t, C rl) -> C { return EXACT ? t - rl : fma(-h2, rl, t); };
    auto step = [&](int k, int u, PairIn<T> &pm, PairIn<T> &pc, PairIn<T> &pn, PairIn<T> &pf)
                    __attribute__((always_inline)) {
        const int si = u & 1, s3 = u % NRED, sb = (u + NRED - 1) % NRED;
        int kw;
        const bool kin = act && plane(k, kw);
        const int o = p0 ^ si;            // first-colour cell of the pair in plane k
        const int la = ladj[si];          // every phase of this step updates offset o
        // phase A: first colour of plane k, sweep 1
        const C xr = SX[si][li + 1];
        const T2 yu = SY[si][li + GLW];
        const C xl = wxl ? C(0) : C(pc.bx.x);
        const C xi = C(pc.bx.y), xo = o ? xr : xl, nxo = o ? xl : xr;
        const C yl = pick(o, pc.by), nyl = pick(1 - o, pc.by);
        const C yh = pick(o, yu), nyh = pick(1 - o, yu);
        const C zl = pick(o, pc.bz), zh = pick(o, pn.bz);
        C diag = (xi + xo) + (yl + yh) + (zl + zh);
        if (SIG)
            diag += pick(o, pc.sg);
        C s = C(0);
        if (!ZERO)
            s = links6(false, o, xi, xo, yl, yh, zl, zh, pick(1 - o, pc.e), SE[si][la],
                       SE[si][li - GLW], SE[si][li + GLW], pick(o, pm.e), pick(o, pn.e));
        const C inva = (kin && diag > C(0)) ? om_over(om, diag) : C(0);
        const C ra = pick(o, pc.r);
        C red = fma(-h2, ra, s) * inva;
        if (!ZERO) {
            red = fma(om1, pick(o, pc.e), red);
            if (SIG || CLOSED)
                red = inva == C(0) ? C(0) : red;   // an excluded cell stays 0
        }
        if (act)
            RED1[s3][li] = red;
        publish(si ^ 1, 1 - o, pn);
        load_in(k + 1 + FPD, pf);   // here the registers of phase A are free again
        __syncthreads();
        // The in-plane neighbours of phases B, C and D were all written before
        // this barrier (A's of plane k-1 in this step, B's of plane k-2 and C's
        // of plane k-3 in the previous one), and none is overwritten below, so
        // all nine LDS reads are issued at once.
        const C bo = RED1[sb][la], bs = RED1[sb][li - GLW], bn = RED1[sb][li + GLW];
        C co = C(0), cs = C(0), cn = C(0), dq = C(0), ds = C(0), dn = C(0);
        if (cdw) {
            co = BLK1[si][la];
            cs = BLK1[si][li - GLW];
            cn = BLK1[si][li + GLW];
            dq = RED2[si ^ 1][la];
            ds = RED2[si ^ 1][li - GLW];
            dn = RED2[si ^ 1][li + GLW];
        }
        // phase B: second colour of plane k-1, sweep 1
        const C bzl = pick(o, pm.bz), bzh = pick(o, pc.bz);
        C dg = (sxi + sxo) + (syl + syh) + (bzl + bzh);
        if (SIG)
            dg += pick(o, pm.sg);
        const C invb = dg > C(0) ? om_over(om, dg) : C(0);
        const C rb = pick(o, pm.r);
        C blk = fma(-h2, rb,
                    links6(false, o, sxi, sxo, syl, syh, bzl, bzh, red_km1, bo, bs, bn, red_km2, red)) *
                invb;
        if (!ZERO) {
            blk = fma(om1, pick(o, pm.e), blk);
            if (SIG || CLOSED)
                blk = invb == C(0) ? C(0) : blk;
        }
        if (act)
            BLK1[si ^ 1][li] = blk;
        C red2 = C(0);
        if (cdw) {
            // phase C: first colour of plane k-2, sweep 2 (A's cell of step k-2)
            red2 = links6(true, o, a2.xi, a2.xo, a2.yl, a2.yh, a2.zl, a2.zh, blk_km1, co, cs, cn, blk_km2,
                          blk);
            red2 = fma(om1, red_km2, minus_h2r(red2, a2.r) * a2.inv);
            if (act)
                RED2[si][li] = red2;
            // phase D: second colour of plane k-3, sweep 2 (B's cell of step k-2)
            C blk2 = links6(true, o, b2.xi, b2.xo, b2.yl, b2.yh, b2.zl, b2.zh, r2_km1, dq, ds, dn, r2_km2,
                            red2);
            blk2 = fma(om1, blk_km2, minus_h2r(blk2, b2.r) * b2.inv);
            const int kd = k - 3;
            if (kd >= k0 && kd < k1) {
                T2 outv;
                outv.x = static_cast<T>(o ? r2_km1 : blk2);
                outv.y = static_cast<T>(o ? blk2 : r2_km1);
                store_out(kd, outv);
                if (DOT && owned)
                    dacc += static_cast<double>(h2 * rc) * static_cast<double>(r2_km1) +
                            static_cast<double>(h2 * b2.r) * static_cast<double>(blk2);
            }
        }
        red_km2 = red_km1;
        red_km1 = red;
        blk_km2 = blk_km1;
        blk_km1 = blk;
        r2_km2 = r2_km1;
        r2_km1 = red2;
        if (DOT)
            rc = a2.r;
        a2 = a1;
        a1 = GsLag<C>{xi, xo, yl, yh, zl, zh, inva, EXACT ? rounded_product(h2, ra) : ra};
        b2 = b1;
        b1 = GsLag<C>{sxi, sxo, syl, syh, bzl, bzh, invb, EXACT ? rounded_product(h2, rb) : rb};
        sxi = xi;
        sxo = nxo;
        syl = nyl;
        syh = nyh;
    };

    PairIn<T> buf[FNB];
#pragma unroll
    for (int u = 0; u < FNB - 1; ++u)
        load_in(k0 - 4 + u, buf[u]);
    __syncthreads();                  // the zero fill is complete
    publish(0, p0, buf[1]);
    __syncthreads();
    if constexpr (WHOLE) {
        // whole blocks of FNB steps, the last up to FNB - 1 steps past k1 + 2
        // (they store nothing), as in the single sweep
        for (int k = kb; k <= two_sweep_end(k1); k += FNB) {
#pragma unroll
            for (int u = 0; u < FNB; ++u)
                step(k + u, u, buf[u % FNB], buf[(u + 1) % FNB], buf[(u + 2) % FNB],
                     buf[(u + FNB - 1) % FNB]);
        }
    } else {
        for (int k = kb, more = 1; more;) {
#pragma unroll
            for (int u = 0; u < FNB; ++u) {
                step(k, u, buf[u % FNB], buf[(u + 1) % FNB], buf[(u + 2) % FNB],
                     buf[(u + FNB - 1) % FNB]);
                if (++k > two_sweep_end(k1)) {
                    more = 0;
                    break;
                }
            }
        }
    }
    if (DOT) {
        __shared__ double wsum[GTHREADS / 64];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
            dacc += __shfl_xor(dacc, o, 64);
        if ((tid & 63) == 0)
            wsum[tid >> 6] = dacc;
        __syncthreads();
        if (tid == 0) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < GTHREADS / 64; ++w)
                t += wsum[w];
            part[blockIdx.x + gridDim.x * blockIdx.y] = t / static_cast<double>(h2);
        }
    }
}

template <typename T, bool ZERO, bool SIG, bool CLOSED, bool DOT>
static long long fused2_slots()
{
    static long long cached[64] = {0};
    int dev = 0;
    (void)hipGetDevice(&dev);
    if (dev < 0 || dev >= 64)
        dev = 0;
    if (cached[dev] == 0) {
        int per_cu = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &per_cu, k_rbgs_fused2<T, ZERO, SIG, CLOSED, DOT, !std::is_same<T, float>::value, true>,
                GTHREADS, 0) != hipSuccess ||
            per_cu < 1)
            per_cu = 1;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            cus < 1)
            cus = 256;
        cached[dev] = (long long)per_cu * cus;
    }
    return cached[dev];
}

// FP16 storage keeps the excluded cells of an operator without a diagonal term as
// they were prolonged: its iterates repeat only with them.
template <typename T>
constexpr bool zeroes_excluded = !std::is_same<T, _Float16>::value;

template <typename T>
void prepare_fused2()
{
    constexpr bool ZX = zeroes_excluded<T>, MAY = !std::is_same<T, _Float16>::value;
    (void)fused2_slots<T, true, false, false, false>();
    (void)fused2_slots<T, false, false, false, false>();
    (void)fused2_slots<T, false, false, ZX, false>();
    (void)fused2_slots<T, true, true, false, false>();
    (void)fused2_slots<T, false, true, false, false>();
    if constexpr (MAY) {
        (void)fused2_slots<T, false, false, false, true>();
        (void)fused2_slots<T, false, false, ZX, true>();
    }
}

template <typename T>
int launch_rbgs_fused2(Dims d, Bc bc, const T *bx, const T *by, const T *bz, const T *r,
                       const T *ein, T *eout, const T *sg, bool closed, double h2, double omega,
                       int first_colour, bool zero, hipStream_t s, double *part, long long max_parts)
{
    using C = typename Acc<T>::type;
    // the first tile of a row with walls owns four cells more (see the kernel)
    const unsigned tx = bc.x ? (d.nx > GTX + 4 ? (d.nx - 4 + GTX - 1) / GTX : 1) : (d.nx + GTX - 1) / GTX;
    const unsigned ty = (d.ny + GTY - 1) / GTY;
    const long long tiles = (long long)tx * ty;
    // A chunk marches kz + 6 steps.  FP32 runs short ones with an exit after
    // every step (whole blocks of six would march 12 steps for 8); FP16 and FP64
    // always run whole blocks, of four: the other form's registers spill (of the
    // whole blocks' only the regular pass with a diagonal term, 6 values in FP64
    // and 1 in FP16).
    constexpr bool SHORT = std::is_same<T, float>::value;
    auto form = [&](auto z, auto g, auto x, auto dt) -> int {
        constexpr bool Z = decltype(z)::value, G = decltype(g)::value, X = decltype(x)::value,
                       DT = decltype(dt)::value;
        // chunks of at least two planes; a pass that forms the dot product writes a
        // partial sum per workgroup, at most max_parts of them
        const int kz = chunk_planes(d.nz, tiles, fused2_slots<T, Z, G, X, DT>(), 6, 2,
                                    DT ? max_parts / tiles : d.nz);
        const dim3 grid(tx * ty, (d.nz + kz - 1) / kz);
        const bool whole = !SHORT || kz + 6 >= WHOLE_MIN_STEPS;
        auto go = [&](auto kern) {
            PP_LAUNCH(kern, grid, dim3(GTHREADS), 0, s, d, bc, bx, by, bz, r, ein, eout, sg, (C)h2,
                      (C)omega, first_colour, kz, tx, ty, part);
        };
        if (!fused2_flat(d, sizeof(T)))
            go(k_rbgs_fused2<T, Z, G, X, DT, true, false>);
        else if (whole)
            go(k_rbgs_fused2<T, Z, G, X, DT, true, true>);
        else
            go(k_rbgs_fused2<T, Z, G, X, DT, !SHORT, true>);
        return DT ? (int)(grid.x * grid.y) : 0;
    };
    constexpr std::true_type Y{};
    constexpr std::false_type N{};
    if (sg)
        return zero ? form(Y, Y, N, N) : form(N, Y, N, N);
    if (zero)
        return form(Y, N, N, N);
    constexpr std::bool_constant<zeroes_excluded<T>> ZX{};
    // the fused dot product: regular passes without a diagonal term (FP16
    // storage keeps the sum of its own kernel)
    if constexpr (!std::is_same<T, _Float16>::value)
        if (part)
            return closed ? form(N, N, ZX, Y) : form(N, N, N, Y);
    return closed ? form(N, N, ZX, N) : form(N, N, N, N);
}

#define PP_INSTANTIATE_FUSED2(T)                                                                 \
    template void prepare_fused2<T>();                                                          \
    template int launch_rbgs_fused2<T>(Dims, Bc, const T *, const T *, const T *, const T *,    \
                                       const T *, T *, const T *, bool, double, double, int,     \
                                       bool, hipStream_t, double *, long long);

PP_INSTANTIATE_FUSED2(double)
PP_INSTANTIATE_FUSED2(float)
PP_INSTANTIATE_FUSED2(_Float16)

#define PP_INSTANTIATE_FUSED(T)                                                                  \
    template void prepare_fused<T>();                                                           \
    template void launch_rbgs_fused<T>(Dims, Bc, const T *, const T *, const T *, const T *,    \
                                       const T *, T *, const T *, double, double, int, bool,     \
                                       hipStream_t);

PP_INSTANTIATE_FUSED(double)
PP_INSTANTIATE_FUSED(float)
PP_INSTANTIATE_FUSED(_Float16)

}  // namespace pp
