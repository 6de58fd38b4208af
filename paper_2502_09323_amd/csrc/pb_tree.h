// pb_tree.h -- the energy read-back's sums over cut points by box expansions (pb_tree.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "pb_internal.h"

namespace pbk {

// what the kernels take of a plan
struct TreeGeom {
    int64_t S;         // z-row stride and rows per plane of the grid
    int ny;
    int B;             // lattice cells along a box
    int nb[3];         // boxes along each axis
    int c0[3];         // first lattice cell of box 0
    int bits;          // 2^bits bins per axis order the atoms along a Hilbert curve
    int nfar, nnear;   // chunks that a group's boxes are shared among, for the expansions and the points
    double side;       // edge of a box
    double ctr[3];     // centre of box 0 relative to the atoms' centre
    double rinv;       // 1 / (half-diagonal of a box)
    double alo[3], ainv;   // low corner, and 1 / edge of the curve's cells
};

struct TreePlan {
    int n = 0;             // atoms
    int64_t ncut = 0;      // cut points
    TreeGeom geom{};
};

// Fewest atoms (16 groups), and atoms x cut points, for which the expansions take over from the
// direct sum.  Read-back by the direct sum against the expansions: 1.20 and 1.25 ms for 5000 atoms
// and 3.5e5 points (1.7e9 pairs), 1.26 and 1.23 for 8000 and 2.2e5 (1.8e9), 1.65 and 1.40 for 6000
// and 4.2e5 (2.5e9), 12.5 and 4.1 for 18000 and 1.2e6 (2.2e10), 133 and 19.9 for 60000 and 3.9e6
// (2.3e11); below, the expansions of the few boxes leave the device idle (0.87 and 1.07 ms at 1.1e9).
constexpr int kTreeMinAtoms = 1024;
constexpr double kTreeMinPairs = 2e9;

// Plans the sums of at.n atoms (centres within lo .. hi, radii up to rmax) over ncut cut points in
// `bytes` of work space; false: the direct sum is the better one, or the space does not do.
bool tree_plan(const Grid& g, const Atoms& at, const double* lo, const double* hi, double rmax, int64_t ncut,
               size_t bytes, TreePlan* out);

// Sorts the cut points into the plan's boxes and the atoms into groups; *pos (in the work space)
// is where each cut point goes in the list that launch_tree_sums takes.
hipError_t launch_tree_order(hipStream_t s, const TreePlan& t, const Atoms& at, const int64_t* cutkey, void* work,
                             const int** pos);

// The sums, from the sorted cut points: partial sums per atom in tree_chunks(t) chunks at the start
// of the work space, as k_nbody leaves them.
hipError_t launch_tree_sums(hipStream_t s, const TreePlan& t, const double* pts, void* work);
inline int tree_chunks(const TreePlan& t) { return t.geom.nfar + t.geom.nnear; }

}  // namespace pbk
