// pp_planes.h -- which planes along z the kernels read (plain C++: the host can
// go through every case).
#ifndef PP_PLANES_H
#define PP_PLANES_H

#include <cstddef>

namespace pp {

// Kernels that reduce, and the density load, walk several planes per block
// (fewer partial sums, neighbours from cache), but no more than leave 2048
// blocks, eight per CU: on a small grid a walk is a chain of memory round
// trips on a few CUs (32^3 in blocks of 8 planes: 16 blocks, 33 us for the
// density load, 12 us in blocks of one coarse plane).
constexpr int walk_planes(int nz, std::size_t xy_blocks, int most)
{
    while (most > 1 && xy_blocks * ((nz + most - 1) / most) < 2048)
        most /= 2;
    return most;
}

// Planes of a block where the order of the sums must not depend on the grid's size
constexpr int FIXED_PLANES = 8;

// Planes per block from the grid's z extent ceil(nz / planes): as many in every
// block but the last, or (fixed) FIXED_PLANES and what is left in the last.
constexpr int planes_of(int nz, int grid_z, bool fixed)
{
    return fixed ? FIXED_PLANES : (nz + grid_z - 1) / grid_z;
}


// Plane q of a march along z: its wrapped index in qw, and whether it is read
// (walls end the grid; BOUNDED: planes past `last` are not needed).  Selects
// rather than branches.
template <bool BOUNDED>
constexpr bool march_plane(int q, int nz, int wall, int last, int &qw)
{
    const bool lo = q < 0, hi = q >= nz;
    qw = lo ? q + nz : (hi ? q - nz : q);
    bool there = !(wall && (lo || hi));
    if constexpr (BOUNDED)
        there = there && q <= last;
    qw = there ? qw : 0;
    return there;
}

// The two-sweep pass: a chunk of output planes [k0, k1) needs planes k0 - 4 to
// k1 + 3.  It is marched from step k0 - 3 to step k1 + 2, whole blocks of
// two_sweep_unroll steps at a time or exactly; step k loads plane
// k + 1 + two_sweep_depth, so the last steps, above all those of a whole block
// past k1 + 2, reach beyond the planes needed: to k1 + 11 in FP32, which a grid of
// eight planes does not have even wrapped once.
constexpr int two_sweep_first(int k0) { return k0 - 3; }
constexpr int two_sweep_end(int k1) { return k1 + 2; }
constexpr int two_sweep_last_plane(int k1) { return k1 + 3; }

// Planes of loads in flight beyond k+1, by bytes of a stored value: three for
// FP32; one for FP16 (whose registers then allow two workgroups per CU) and for
// FP64 (two spill).
constexpr int two_sweep_depth(int word) { return word == 4 ? 3 : 1; }
constexpr int two_sweep_unroll(int word) { return two_sweep_depth(word) + 3; }

}  // namespace pp
#endif
