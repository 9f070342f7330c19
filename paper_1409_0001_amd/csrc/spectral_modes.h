// Eigenvalues and eigenvectors of one axis of uneven cells, for the direct
// solve (spectral.hip).  Host code without device types.
#pragma once

#include <vector>

namespace cgd {

// Eigenvalues in stored order, and the packed matrices (forward even, odd,
// inverse even, odd).
struct AxisModes {
    std::vector<double> lam, mats;
};

// Eigenvalues d and eigenvectors (z[k], one array per eigenvalue) of the
// symmetric tridiagonal matrix with diagonal d and off-diagonal e.  False
// where an off-diagonal does not vanish within 60 n steps or something is not
// finite; d and z are of no use then.
bool tridiagonal_modes(std::vector<double>& d, std::vector<double> e, std::vector<std::vector<double>>& z);

// The modes of an axis of cell widths h, zero-flux ends or periodic (sym
// only).  sym: h is its own mirror image.  False as tridiagonal_modes.
bool axis_modes(const std::vector<double>& h, bool sym, bool periodic, AxisModes* out);

}  // namespace cgd
