// Direct solve of the implicit steps on uniform hex grids (spectral.hip).
#pragma once

#include <vector>

#include "cgd_internal.h"
#include "spectral_modes.h"

namespace cgd {

// Tables of one axis (device pointers; see k_spec_tables).
struct SpecAxis {
    int n = 0;
    double* lam = nullptr;   // eigenvalues at the stored positions [n] (closed forms: see k_spec_tables)
    double2* tw = nullptr;   // FFT lengths: e^{-2 pi i q / n} [n]
    double2* pw = nullptr;   //    and e^{-i pi k / 2n} [n / 2]
    double* fe = nullptr;    // dense lengths: packed matrices, forward even and odd modes,
    double* fo = nullptr;
    double* ie = nullptr;    //    inverse even and odd modes
    double* io = nullptr;
};

struct AxisModes {
    RotationGroups rot[2];
    std::vector<double> lam;
};

// The cells that diffuse, lo .. lo + len of a grid of nn per axis.
struct SpecBox {
    int nn[3], lo[3], len[3];
};

// What the transforms need to know of a mesh: the box of cells that diffuse
// (a uniform grid: all of them; a rectilinear one: those with a diffusivity),
// its axes of more than one cell, the contiguous one first.  Owned by the
// mesh, made on its first call.
struct SpecTables {
    bool ok = false;          // the transforms apply to this mesh
    int rank = 0;
    int n[3] = {1, 1, 1};
    bool eigen[3] = {};       // modes by eigenvectors (else cosines, and sines on a periodic axis)
    bool sym[3] = {};         // even and odd modes about the axis's middle
    bool per[3] = {};
    double scale[3] = {};     // eigenvalue of A - I over dtau = scale * lam
    double diag = 0.0;        // bound of the diagonal of (A - I) / dtau
    std::vector<double> h[3]; // eigen axes: cell widths
    AxisModes modes[3];       //    and their modes, until they are on the device
    int64_t off = 0;          // the box's first cell in a field
    int rows_y = 0;           // rows per plane where rows are not one after the other, else 0
    int64_t sy = 0, sz = 0;   //    and the strides between rows and planes in a field
    int64_t pitch = 0;        // else the stride between rows
    int64_t cells = 0;        // of the box
    SpecBox box = {};
    double* dev = nullptr;
    SpecAxis axis[3];
    uint32_t* neg = nullptr;  // device, [kSpecFields] (SpecPass)
    uint32_t calls = 0;       // calls so far
};
constexpr int kSpecFields = 4096;  // fields of a call at most
constexpr int kTopSlots = 8, kTopStride = 32;  // SpecPass::top: words per field, each in a cache line of its own

// One pass of transforms along one axis of all fields.
struct SpecPass {
    const float* in;      // the caller's fields: the first pass's input
    float* out;           //    and the last one's output
    double* W;            // the modes between the passes, worked on in place
    int64_t cells;        // per field of W
    int64_t fcells;       // per field of the caller's array (the first pass's input, the last one's output)
    int64_t off, sy, sz, pitch;  // ... where its row r begins: off + r pitch, or (rows_y) off + (r % rows_y) sy + (r / rows_y) sz
    int32_t rows_y;
    int32_t n;            // length of a line
    int32_t hm, ho;       // dense: even and odd modes (n and 0: one full matrix)
    int64_t lines;        // lines per field
    int64_t pairs;        // FFT: pairs of lines per field
    int64_t inner;        // strided lines: neighbouring lines (at unit stride),
    int64_t inner_pairs;  //    their pairs, the stride between points of a line
    int64_t estride;      //    and between groups of neighbouring lines
    int64_t ostride;
    int32_t vec2;         // both lines of a pair in one aligned 16-byte access (contiguous lines: two points in 8 bytes)
    const double2* tw;
    const double2* pw;
    const double* fe;
    const double* fo;
    const double* ie;
    const double* io;
    double sf, sf0, si, si0;  // FFT: scale of a mode (mode 0) forward and inverse
    // the gain pass: mu = c0 lam0[line % n0] + c1 lam1[line / n0] + cm lamm[mode]
    double cm, c0, c1;
    const double* lamm;
    const double* lam0;
    const double* lam1;
    int64_t n0;
    int32_t n_steps, cn;
    int* bad;       // device, per field: set by the gain pass where a value of W is beyond float32 or not finite
    int* bad_host;  // nullable: the same in pinned host memory
    uint32_t* top;  // device, kTopSlots per field: the largest |value| in W after the gain pass (upper 32 bits)
    uint32_t* neg;  // device, per field: `call` where the input holds a negative value
    uint32_t call;
    double cut;     // results below cut * (the largest of top) of a field without negative values are 0
};

// Whether a call is answered by the direct solve (stats: its statistics are
// asked for); the same for any number of fields.
bool spectral_applies(cgd_mesh m, const DiffuseArgs& da, bool stats);
// Bytes of scratch (W) for F fields, where spectral_applies.
size_t spectral_bytes(const cgd_mesh m, int32_t F);
// Enqueues all steps of `da` on n_fields fields at da.field [n_fields][cells]
// (da.F is not used), with W as scratch; at most kSpecFields.  Where a field
// has a mode beyond float32 or not finite, its entries of bad and bad_host
// (nullable, cleared by the caller) are set and the field is left as it was.
// timing: nullable.
cgd_status spectral_enqueue(cgd_mesh m, const DiffuseArgs& da, int n_fields, double* W, int* bad, int* bad_host,
                            Timing* timing, hipStream_t s);
// The diffusion of cgd_diffuse by the direct solve; waits for the stream.
cgd_status diffuse_spectral(cgd_mesh m, const DiffuseArgs& da, hipStream_t s);
void destroy_spectral(cgd_mesh m);

}  // namespace cgd
