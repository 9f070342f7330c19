// Eigenvalues and eigenvectors of one axis of uneven cells, for the direct
// solve (spectral.hip).  Host code without device types.
#pragma once

#include <vector>

namespace cgd {

// A symmetric tridiagonal matrix's eigenvectors as the plane rotations that
// make it diagonal: sweep i turns the vectors lo, lo + 1, ..., lo + count by
// the next `count` rotations (c, s), each taking (z[k], z[k + 1]) to
// (c z[k] + s z[k + 1], c z[k + 1] - s z[k]), starting from the unit vectors.
// O(n^2) numbers stand for the O(n^3) work of forming the vectors, which is
// left to the device.
struct Rotations {
    struct Sweep {
        int lo, count;
    };
    std::vector<Sweep> sweeps;
    std::vector<double> cs;  // c, s of every rotation
};

// The same rotations, kLanes sweeps at a time: a group's step t (t = 0 .. count
// - 1, a multiple of kGroupSteps) takes row lo + t + 1 in at its first sweep,
// turns it with the row that sweep holds, hands the finished one on to the
// next sweep and so on; what leaves the last sweep is row lo + t + 1 - kLanes
// as all of them left it.  Sweep j's rotation of rows k and k + 1 is cs[step k
// - lo + j][j]; where it has none, c = 1 and s = 0 pass the rows through.
// The rows are lo .. lo + rows - 1.
struct RotationGroups {
    static constexpr int kLanes = 4, kGroupSteps = 16;
    struct Group {
        int lo, rows, count;
    };
    std::vector<Group> groups;
    std::vector<double> cs;  // [steps of all groups][kLanes] (c, s)
};
void group_rotations(const Rotations& rot, RotationGroups& out);

// Replaces the diagonal d by the eigenvalues (e: the off-diagonal, d.size()
// - 1 entries).  False where an off-diagonal does not vanish within 60 n
// sweeps or something is not finite; d and rot are of no use then.
bool tridiagonal_modes(std::vector<double>& d, std::vector<double> e, Rotations& rot);

// The modes of an axis of cell widths h: the eigenvectors v of its symmetric
// matrix M^-1/2 K M^-1/2, zero-flux ends or periodic (sym only).  sym: h is
// its own mirror image, and the modes are even ones in [0] (of the first (n +
// 1) / 2 cells) and odd ones in [1] (of the first n / 2), each cell m < n / 2
// standing for itself and its mirror image with 1 / sqrt 2; else all in [0].
// lam: the eigenvalues, [0]'s then [1]'s.  False as tridiagonal_modes.
bool axis_modes(const std::vector<double>& h, bool sym, bool periodic, RotationGroups rot[2], std::vector<double>& lam);

}  // namespace cgd
