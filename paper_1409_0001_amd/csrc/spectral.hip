// Direct solve of the implicit steps on uniform hex grids, and on rectilinear
// ones whose diffusivity is one value on a box of cells and 0 elsewhere.
//
// The zero-flux finite-volume Laplacian of a uniform box is diagonal in the
// products of the axes' cosine modes (DCT-II): with c_a = dtau / h_a^2 the
// step matrix A = I + sum_a c_a L_a has the eigenvalues
// 1 + sum_a 4 c_a sin^2(pi k_a / 2 N_a).  All n steps of a call are then one
// multiplication of the modes by gain(k) = 1 / A(k)^n (backward Euler) or
// (2 / A(k) - 1)^n with half dtau in c_a (Crank-Nicolson), between a forward
// and an inverse transform.
//
// Passes over memory (three axes): x forward, y forward, z forward + gain +
// z inverse in one kernel, y inverse, x inverse; 12 bytes per cell along x,
// 16 for the inner ones, in place on one float64 workspace vector.  All is
// float64 (gfx950 issues float64 and unpacked float32 multiply-adds at the
// same rate) but the field itself, rounded once.  The vectors between the
// passes have to be float64 as well: a mode's rounding error reaches every
// cell of its line, and in float32 it put noise of 1e-8 of a line's largest
// values, of either sign, into cells that no particle is near (a bed in half
// of 64 x 64 x 128 cells: 29,994 negative cells, and velocities from momentum
// 20 % off where eps is 1e-7 of its maximum).  It costs 38 % of the dense
// bed's transforms (256 x 256 x 512: 340 -> 500 us).
//
// Rectilinear grids: with one diffusivity d on the cells that diffuse at all
// (the product of per-axis factors that are constant on one range of the axis
// and 0 elsewhere; faces to cells of diffusivity 0 carry nothing), the
// operator of that box is I + dtau d sum_a M_a^-1 K_a, and the modes of an
// axis are the eigenvectors of its tridiagonal M_a^-1/2 K_a M_a^-1/2 (of the
// cyclic one on a periodic axis), scaled by sqrt(h) on the way in and
// 1 / sqrt(h) on the way out: where the widths are equal, cosines between
// zero-flux ends, cosines and sines on a periodic axis.  Cells outside the
// box keep their values.
//
// A transform of length 128, 256, 512 or 1024 runs as a complex FFT of two
// lines at once (k_fft); any other length up to 512 (and other modes) as
// two half-size matrix products on the float64 matrix cores, the even modes
// from x[m] + x[N-1-m] and the odd ones from x[m] - x[N-1-m] (k_dense): every
// axis that is its own mirror image has only such modes; one that is not
// takes one full-size product.
#include <math.h>

#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <new>
#include <string>
#include <type_traits>

#include "cg_common.h"
#include "spectral.h"

namespace cgd {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

struct Cd {
    double x, y;
};
__device__ __forceinline__ Cd cadd(Cd a, Cd b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ Cd csub(Cd a, Cd b) { return {a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ Cd cmul(Cd a, Cd b) { return {a.x * b.x - a.y * b.y, fma(a.x, b.y, a.y * b.x)}; }
__device__ __forceinline__ Cd cmulj(Cd a) { return {a.y, -a.x}; }  // -i a

// Forward DFTs (kernel e^{-2 pi i n k / R}) in registers.
__device__ __forceinline__ void dft4(Cd& a, Cd& b, Cd& c, Cd& d) {
    const Cd s0 = cadd(a, c), s1 = csub(a, c), s2 = cadd(b, d), s3 = cmulj(csub(b, d));
    a = cadd(s0, s2);
    c = csub(s0, s2);
    b = cadd(s1, s3);
    d = csub(s1, s3);
}

template <int R>
__device__ __forceinline__ void dft(Cd* v);

template <>
__device__ __forceinline__ void dft<8>(Cd* v) {
    constexpr double kH = 0.70710678118654752440;
    dft4(v[0], v[2], v[4], v[6]);
    dft4(v[1], v[3], v[5], v[7]);
    // odd branch times e^{-2 pi i k / 8}; slots hold k = 0..3 at 1, 3, 5, 7
    const Cd o0 = v[1], o1 = {(v[3].x + v[3].y) * kH, (v[3].y - v[3].x) * kH}, o2 = cmulj(v[5]),
             o3 = {(v[7].y - v[7].x) * kH, -(v[7].x + v[7].y) * kH};
    const Cd e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
    v[0] = cadd(e0, o0);
    v[4] = csub(e0, o0);
    v[1] = cadd(e1, o1);
    v[5] = csub(e1, o1);
    v[2] = cadd(e2, o2);
    v[6] = csub(e2, o2);
    v[3] = cadd(e3, o3);
    v[7] = csub(e3, o3);
}

template <>
__device__ __forceinline__ void dft<16>(Cd* v) {
    // 4 x 4: X[k1 + 4 k2] = sum_n2 e^{-2 pi i n2 k1 / 16} (sum_n1 x[4 n1 + n2] (-i)^{n1 k1}) (-i)^{n2 k2}
    constexpr double c1 = 0.92387953251128675613, s1 = 0.38268343236508977173, kH = 0.70710678118654752440;
#pragma unroll
    for (int n2 = 0; n2 < 4; ++n2) dft4(v[n2], v[4 + n2], v[8 + n2], v[12 + n2]);
    // v[4 k1 + n2] *= w16^{n2 k1}
    const Cd w1 = {c1, -s1}, w3 = {s1, -c1}, w9 = {-c1, s1};
    v[5] = cmul(v[5], w1);
    v[6] = {(v[6].x + v[6].y) * kH, (v[6].y - v[6].x) * kH};
    v[7] = cmul(v[7], w3);
    v[9] = {(v[9].x + v[9].y) * kH, (v[9].y - v[9].x) * kH};
    v[10] = cmulj(v[10]);
    v[11] = {(v[11].y - v[11].x) * kH, -(v[11].x + v[11].y) * kH};
    v[13] = cmul(v[13], w3);
    v[14] = {(v[14].y - v[14].x) * kH, -(v[14].x + v[14].y) * kH};
    v[15] = cmul(v[15], w9);
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) dft4(v[4 * k1], v[4 * k1 + 1], v[4 * k1 + 2], v[4 * k1 + 3]);
    // slot 4 k1 + k2 holds X[k1 + 4 k2]
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = a + 1; b < 4; ++b) {
            const Cd t = v[4 * a + b];
            v[4 * a + b] = v[4 * b + a];
            v[4 * b + a] = t;
        }
}

// The gain of a mode whose eigenvalue of A is 1 + mu.  (Two or four modes
// side by side overlap these chains but spill: 129 us -> 157 for the gain
// pass of the dense bed.)
__device__ __forceinline__ double mode_gain(double mu, int n, int cn) {
    const double d = 1.0 + mu;
    double r = __builtin_amdgcn_rcp(d);  // 4.6e-8 off at most (measured over 1 .. 1e6)
    r = fma(r, fma(-d, r, 1.0), r);      // 2.1e-15
    if (cn) r = fma(2.0, r, -1.0);
    double g = 1.0;
    for (int e = n;; r *= r) {
        if (e & 1) g *= r;
        e >>= 1;
        if (!e) break;
    }
    return g;
}

// A field with a value beyond float32 in W: the last pass leaves it alone,
// and the host solves it by CG.
__device__ __forceinline__ void mark_bad(const SpecPass& a) {
    __hip_atomic_store(a.bad + blockIdx.y, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (a.bad_host) a.bad_host[blockIdx.y] = 1;
}
// |x|'s upper 32 bits, which order as |x| does (infinities and NaN above all
// numbers): 2^128 and more is beyond float32.
__device__ __forceinline__ uint32_t upper(double x) {
    return (uint32_t)((unsigned long long)__double_as_longlong(x) >> 32) & 0x7fffffffu;
}
constexpr uint32_t kBeyond = 0x47f00000u;
// The first pass (x forward) clears what the gain pass notes per field.
__device__ __forceinline__ void clear_notes(const SpecPass& a) {
    if (blockIdx.x) return;
    if (threadIdx.x == 0) __hip_atomic_store(a.bad + blockIdx.y, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (threadIdx.x < kTopSlots) a.top[(size_t)(blockIdx.y * kTopSlots + threadIdx.x) * kTopStride] = 0u;
}
__device__ __forceinline__ bool is_bad(const SpecPass& a) {
    return __hip_atomic_load(a.bad + blockIdx.y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}

// A negative value anywhere in a field: noted as this call's number, which
// no earlier call has left there, so nothing has to be cleared first.  A
// plain store (every wave stores the same, and only later kernels read it):
// one that goes past the XCD's L2 took x forward of 4 x 128^3 from 17 to 53
// us.  least: the least value the thread has seen.  (All threads of a wave.)
__device__ __forceinline__ void mark_negative(const SpecPass& a, float least) {
    if (__ballot(least < 0.f) && (threadIdx.x & 63) == 0) a.neg[blockIdx.y] = a.call;
}
// The largest |value| the gain pass leaves in W (its upper 32 bits), in one of
// a field's kTopSlots cache lines: one word per field took the gain pass of 4
// x 128^3 from 29 to 60 us, and a look at the word before the atomic, which
// nothing waits for, that of 2 x 96 x 64 x 80 from 16 to 19.  (All threads of
// a wave.)
__device__ __forceinline__ void note_top(const SpecPass& a, uint32_t top) {
    for (int o = 32; o > 0; o >>= 1) top = max(top, __shfl_xor(top, o));
    const unsigned wave = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if ((threadIdx.x & 63) == 0) atomicMax(a.top + (size_t)(blockIdx.y * kTopSlots + wave % kTopSlots) * kTopStride, top);
}
// Results of a field without negative values are right to about 2^-53 of the
// largest plane mean times the square root of a plane's cells, whatever
// their own size.  Below a.cut times the largest value between the gain pass
// and the inverse ones, which is 2^-32 of something between that mean (the
// plane's mode 0) and the largest result (the transforms keep the norm), they
// are returned as 0: no backward Euler result is negative, and the quotient
// of two fields is right wherever the divisor is not 0 (in a float64 model to
// 2e-5 for beds in half or a corner of 512 x 512 x 8 cells and smaller
// boxes, 3e-3 for a single particle in the first).
__device__ __forceinline__ float cut_of(const SpecPass& a) {
    uint32_t top = 0u;
#pragma unroll
    for (int i = 0; i < kTopSlots; ++i) top = max(top, a.top[(size_t)(blockIdx.y * kTopSlots + i) * kTopStride]);
    const double t = __longlong_as_double((long long)((unsigned long long)top << 32));
    const float c = a.neg[blockIdx.y] == a.call ? 0.f : (float)(a.cut * t);
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(c)));  // (the same in all lanes: a scalar register)
}
__device__ __forceinline__ float result(double x, float cut) {
    const float r = (float)x;
    return fabsf(r) < cut ? 0.f : r;
}

// Where row r of the caller's array begins.
__device__ __forceinline__ int64_t field_row(const SpecPass& a, int64_t r) {
    if (!a.rows_y) return a.off + r * a.pitch;
    const int64_t z = r / a.rows_y;
    return a.off + (r - z * a.rows_y) * a.sy + z * a.sz;
}

// ------------------------------------------------------------------- FFT

template <int N>
struct FftCfg;
template <>
struct FftCfg<128> {
    static constexpr int R1 = 16, R2 = 8, R3 = 1;
};
template <>
struct FftCfg<256> {
    static constexpr int R1 = 16, R2 = 16, R3 = 1;
};
template <>
struct FftCfg<512> {
    static constexpr int R1 = 8, R2 = 8, R3 = 8;
};
template <>
struct FftCfg<1024> {
    static constexpr int R1 = 16, R2 = 8, R3 = 8;
};

constexpr int kE = 16;  // points of a line held by a thread

// Pairs of lines per block: small blocks, whose barriers wait for few waves
// (with float32 vectors, the gain pass at 512: 131 us with 16 pairs on the
// dense bed, 120 with 8; contiguous lines at 128: 60 us with 32 pairs on 16
// fields of 128^3, 53 with 16), but longer rows where a block is small anyway
// (strided lines at 128: 14 us with 32 pairs against 17 on 128 x 115 x 256).
template <int N, bool XK>
constexpr int fft_pairs() { return N >= 512 ? 8 : (N == 256 || XK ? 16 : 32); }

// LDS slot of point m of pair p.  Strided lines: the P pairs of a point side
// by side (a wave's 16 consecutive pairs read 128 bytes).  Contiguous lines:
// a pair's points side by side, one slot of padding in 16, so that lanes at a
// stride of 8 or 16 points fall in distinct banks.
template <int N, int P, bool XK>
__device__ __forceinline__ int slot(int m, int p) {
    return XK ? p * (N + N / 16) + m + (m >> 4) : m * P + p;
}
template <int N, bool XK>
constexpr int fft_lds_doubles() {
    return fft_pairs<N, XK>() * (XK ? N + N / 16 : N);
}

// One Stockham stage of radix R over what the threads hold (slot j of a
// thread: point t + T j), L the product of the earlier radices: twiddles and
// butterflies; the outputs' places are out_place below.
template <int N, int R, int L>
__device__ __forceinline__ void stage(Cd* v, int t, const double2* __restrict__ tw) {
    constexpr int T = N / kE, B = kE / R;
#pragma unroll
    for (int i = 0; i < B; ++i) {
        Cd u[R];
#pragma unroll
        for (int r = 0; r < R; ++r) u[r] = v[i + r * B];
        if (L > 1) {
            const double2 q = tw[((t + T * i) % L) * (N / (L * R))];
            const Cd w = {q.x, q.y};
            Cd c = w;
#pragma unroll
            for (int r = 1; r < R; ++r) {
                u[r] = cmul(u[r], c);
                if (r + 1 < R) c = cmul(c, w);
            }
        }
        dft<R>(u);
#pragma unroll
        for (int r = 0; r < R; ++r) v[i + r * B] = u[r];
    }
}

template <int N, int R, int L>
__device__ __forceinline__ int out_place(int t, int j) {
    constexpr int T = N / kE, B = kE / R;
    const int b = t + T * (j % B), r = j / B;
    return (b / L) * (L * R) + (b % L) + r * L;
}

// Moves the outputs of a stage to the next one's inputs through LDS, real
// and imaginary parts one after the other (half the LDS, so twice the blocks
// per compute unit).
template <int N, int P, bool XK, int R, int L>
__device__ __forceinline__ void exchange(Cd* v, double* sh, int t, int p) {
    constexpr int T = N / kE;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kE; ++j) sh[slot<N, P, XK>(out_place<N, R, L>(t, j), p)] = v[j].x;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kE; ++j) v[j].x = sh[slot<N, P, XK>(t + T * j, p)];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kE; ++j) sh[slot<N, P, XK>(out_place<N, R, L>(t, j), p)] = v[j].y;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kE; ++j) v[j].y = sh[slot<N, P, XK>(t + T * j, p)];
}

// The complex DFT of a line pair; in and out: slot j holds point t + T j.
// The value again, as one the compiler does not know: index arithmetic on it
// is done anew instead of being kept in registers over a whole transform (16
// offsets of 64 bits cost the 32 registers that the points then spill).
__device__ __forceinline__ int again(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

template <int N, int P, bool XK>
__device__ __forceinline__ void fft_line(Cd* v, double* sh, int t, int p, const double2* __restrict__ tw) {
    constexpr int R1 = FftCfg<N>::R1, R2 = FftCfg<N>::R2, R3 = FftCfg<N>::R3;
    stage<N, R1, 1>(v, t, tw);
    exchange<N, P, XK, R1, 1>(v, sh, t, p);
    stage<N, R2, R1>(v, t, tw);
    if constexpr (R3 > 1) {
        exchange<N, P, XK, R2, R1>(v, sh, t, p);
        stage<N, R3, R1 * R2>(v, t, tw);
    }
}

// Between the natural order (slot j: point t + T j) and the pairs (k, N - k)
// of k = t + T i, i < 8 (slot i: point k, slot 8 + i: point N - k; k = 0 pairs
// with N / 2): only the upper half of the points changes hands, its real and
// imaginary parts side by side in LDS.
template <int N, int P, bool XK>
__device__ __forceinline__ void to_pairs(Cd* v, double* sh, int t, int p) {
    constexpr int T = N / kE, H = kE / 2;
    __syncthreads();
#pragma unroll
    for (int j = H; j < kE; ++j) {
        sh[slot<N, P, XK>(t + T * (j - H), p)] = v[j].x;
        sh[slot<N, P, XK>(t + T * j, p)] = v[j].y;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const int n = i == 0 && t == 0 ? N / 2 : N - (t + T * i);
        v[H + i] = {sh[slot<N, P, XK>(n - N / 2, p)], sh[slot<N, P, XK>(n, p)]};
    }
}

template <int N, int P, bool XK>
__device__ __forceinline__ void from_pairs(Cd* v, double* sh, int t, int p) {
    constexpr int T = N / kE, H = kE / 2;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const int n = i == 0 && t == 0 ? N / 2 : N - (t + T * i);
        sh[slot<N, P, XK>(n - N / 2, p)] = v[H + i].x;
        sh[slot<N, P, XK>(n, p)] = v[H + i].y;
    }
    __syncthreads();
#pragma unroll
    for (int j = H; j < kE; ++j)
        v[j] = {sh[slot<N, P, XK>(t + T * (j - H), p)], sh[slot<N, P, XK>(t + T * j, p)]};
}

// Modes of both lines from the pair (k, N - k) of the packed transform:
// m = {Xa[k], Xa[N-k], Xb[k], Xb[N-k]} (k = 0: modes 0 and N / 2), times s
// (mode 0: s0); w = e^{-i pi k / 2N}.
__device__ __forceinline__ v4d modes_of(Cd zk, Cd zn, Cd w, bool k0, double s, double s0) {
    if (k0) {
        constexpr double kH = 0.70710678118654752440;
        return v4d{zk.x * s0, zn.x * (kH * s), zk.y * s0, zn.y * (kH * s)};
    }
    const double hs = 0.5 * s;
    const Cd a = {hs * (zk.x + zn.x), hs * (zk.y - zn.y)}, b = {hs * (zk.y + zn.y), hs * (zn.x - zk.x)};
    const Cd ua = cmul(w, a), ub = cmul(w, b);
    return v4d{ua.x, -ua.y, ub.x, -ub.y};
}
// The reverse (s, s0: the inverse's factors).
__device__ __forceinline__ void pair_of(v4d m, Cd w, bool k0, double s, double s0, Cd* zk, Cd* zn) {
    if (k0) {
        constexpr double kR = 1.41421356237309504880;
        *zk = {m.x * s0, m.z * s0};
        *zn = {m.y * (kR * s), m.w * (kR * s)};
        return;
    }
    const Cd cw = {w.x * s, -w.y * s};
    const Cd a = cmul(cw, Cd{m.x, -m.y}), b = cmul(cw, Cd{m.z, -m.w});
    *zk = {a.x - b.y, a.y + b.x};
    *zn = {a.x + b.y, b.x - a.y};
}

// MODE 0 forward, 1 inverse, 2 forward + gain + inverse.  XK: lines
// contiguous in memory (two rows per pair), else strided (two neighbouring
// lines per pair, P pairs per block).  Bound by float64 instructions and the
// LDS exchanges' barriers together; loads and stores walk one pointer per
// stream and the special modes (0 and N / 2) are a test on thread 0's first
// point, where offsets and tests per point took registers and issue slots.
// Large fields are bound by memory: 256 x 256 x 512, one field, whose W of
// 268 MB the memory-side cache does not hold: forward and back along x 70 and
// 82 us (403 MB in and out; 61 and 57 with float32 W), y 98 and 87 (537 MB,
// 5.5 to 6.2 TB/s; 53 and 50), the gain pass along z 159 (118).  4 fields of
// 128^3 (67 MB): 19, 22, 21, 21 and 37 us (17, 18, 15, 16, 29).
template <int N, int MODE, bool XK>
__global__ __launch_bounds__((fft_pairs<N, XK>() * N / kE), 4) void k_fft(SpecPass a) {
    constexpr int T = N / kE, P = fft_pairs<N, XK>(), H = kE / 2;
    __shared__ double sh[fft_lds_doubles<N, XK>()];
    if (MODE == 1 && XK && is_bad(a)) return;
    if (MODE == 0 && XK) clear_notes(a);
    int t = XK ? threadIdx.x % T : threadIdx.x / P;
    const int p = XK ? threadIdx.x / T : threadIdx.x % P;
    // P = 8: the two blocks whose rows share cache lines (rows not a multiple
    // of 16 long) on one XCD (blocks go to the XCDs in turn)
    unsigned qb = blockIdx.x;
    if (P == 8 && !XK && qb < gridDim.x / 16 * 16) qb = qb / 16 * 16 + qb % 8 * 2 + qb / 8 % 2;
    const int64_t q = (int64_t)qb * P + p;
    const bool live = q < a.pairs;
    const float* __restrict__ in = a.in + (size_t)blockIdx.y * a.fcells;
    float* __restrict__ out = a.out + (size_t)blockIdx.y * a.fcells;
    double* __restrict__ W = a.W + (size_t)blockIdx.y * a.cells;
    const double2* __restrict__ tw = a.tw;
    const double2* __restrict__ pw = a.pw;
    const double sf = a.sf, sf0 = a.sf0, si = a.si, si0 = a.si0;
    Cd v[kE];
    bool two;
    int64_t base, base2, line;
    int64_t fbase = 0, fbase2 = 0;  // XK: the same rows in the caller's array
    if (XK) {
        line = 2 * q;
        two = live && line + 1 < a.lines;
        base = (live ? line : 0) * N;
        base2 = two ? base + N : base;
        fbase = field_row(a, live ? line : 0);
        fbase2 = two ? field_row(a, line + 1) : fbase;
    } else {
        const int64_t qq = live ? q : 0;
        const int64_t o = qq / a.inner_pairs;
        const int64_t i = (qq - o * a.inner_pairs) * 2;
        line = o * a.inner + i;
        two = live && i + 1 < a.inner;
        base = o * a.ostride + i;
        base2 = two ? base + 1 : base;
    }
    const int64_t es = a.estride;
    if (MODE == 0 || MODE == 2) {
        if (XK) {
            // element 2m goes to point m, 2m + 1 to point N - 1 - m, which the
            // mirror thread of the line holds
            float2 xa[H], xb[H];
            if (a.vec2) {
#pragma unroll
                for (int j = 0; j < H; ++j) {
                    xa[j] = *reinterpret_cast<const float2*>(in + fbase + 2 * (t + T * j));
                    xb[j] = *reinterpret_cast<const float2*>(in + fbase2 + 2 * (t + T * j));
                }
            } else {
#pragma unroll
                for (int j = 0; j < H; ++j) {
                    const int e = 2 * (t + T * j);
                    xa[j] = make_float2(in[fbase + e], in[fbase + e + 1]);
                    xb[j] = make_float2(in[fbase2 + e], in[fbase2 + e + 1]);
                }
            }
            float least = 0.f;
#pragma unroll
            for (int j = 0; j < H; ++j)
                least = fminf(fminf(least, fminf(xa[j].x, xa[j].y)), fminf(xb[j].x, xb[j].y));
            mark_negative(a, least);
#pragma unroll
            for (int j = 0; j < H; ++j) {
                v[j] = {xa[j].x, two ? xb[j].x : 0.f};
                const float ya = __shfl_xor(xa[j].y, T - 1), yb = __shfl_xor(xb[j].y, T - 1);
                v[kE - 1 - j] = {ya, two ? yb : 0.f};
            }
        } else if (a.vec2) {
            // points t + T j, j < 8: rows 2 t, 2 t + 2 T, ...; the others: N - 1 - 2 t downwards
            const double* p0 = W + base + es * (2 * t);
            const double* p1 = W + base + es * (N - 1 - 2 * t);
#pragma unroll
            for (int j = 0; j < H; ++j) {
                const double2 x0 = *reinterpret_cast<const double2*>(p0);
                const double2 x1 = *reinterpret_cast<const double2*>(p1);
                v[j] = {x0.x, x0.y};
                v[H + j] = {x1.x, x1.y};
                p0 += es * (2 * T);
                p1 -= es * (2 * T);
            }
        } else {
#pragma unroll
            for (int j = 0; j < kE; ++j) {
                const int m = t + T * j;
                const int64_t o = es * (j < H ? 2 * m : 2 * N - 1 - 2 * m);
                v[j] = {W[base + o], W[base2 + o]};
            }
#pragma unroll
            for (int j = 0; j < kE; ++j) v[j].y = two ? v[j].y : 0.0;
        }
        if (MODE == 2) {
            uint32_t most = 0u;
#pragma unroll
            for (int j = 0; j < kE; ++j) most = max(most, max(upper(v[j].x), upper(v[j].y)));
            if (live && most >= kBeyond) mark_bad(a);
        }
        fft_line<N, P, XK>(v, sh, t, p, tw);
        t = again(t);
        to_pairs<N, P, XK>(v, sh, t, p);
    }
    t = again(t);
    if (MODE == 0) {
        if (!live) return;  // (no barrier follows)
        double* p0 = W + base + es * (2 * t);
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const int k = t + T * i;
            const double2 c = pw[k];
            const v4d m = modes_of(v[i], v[H + i], Cd{c.x, c.y}, i == 0 && t == 0, sf, sf0);
            if (XK) {
                *reinterpret_cast<double2*>(W + base + 2 * k) = make_double2(m.x, m.y);
                if (two) *reinterpret_cast<double2*>(W + base2 + 2 * k) = make_double2(m.z, m.w);
            } else if (a.vec2) {
                *reinterpret_cast<double2*>(p0) = make_double2(m.x, m.z);
                *reinterpret_cast<double2*>(p0 + es) = make_double2(m.y, m.w);
                p0 += es * (2 * T);
            } else {
                const int64_t o = es * (2 * k);
                W[base + o] = m.x;
                W[base + o + es] = m.y;
                if (two) {
                    W[base2 + o] = m.z;
                    W[base2 + o + es] = m.w;
                }
            }
        }
        return;
    }
    if (MODE == 2) {
        // the two lines' share of mu, from the modes they stand at on the
        // other axes
        const int64_t l1 = two ? line + 1 : line;
        const int64_t y0 = line / a.n0, y1 = l1 / a.n0;
        const double mua = a.c0 * a.lam0[line - y0 * a.n0] + (a.lam1 ? a.c1 * a.lam1[y0] : 0.0);
        const double mub = a.c0 * a.lam0[l1 - y1 * a.n0] + (a.lam1 ? a.c1 * a.lam1[y1] : 0.0);
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const int k = t + T * i;
            const double2 c = pw[k];
            const Cd w = {c.x, c.y};
            const bool k0 = k == 0;
            v4d m = modes_of(v[i], v[H + i], w, k0, 1.0, 1.0);
            // 4 sin^2(pi k / 2N) and 4 cos^2 of the same for N - k (k = 0: modes 0 and N / 2)
            const double lk = 4.0 * a.cm * c.y * c.y, ln = k0 ? 2.0 * a.cm : 4.0 * a.cm * c.x * c.x;
            m.x *= mode_gain(mua + lk, a.n_steps, a.cn);
            m.y *= mode_gain(mua + ln, a.n_steps, a.cn);
            m.z *= mode_gain(mub + lk, a.n_steps, a.cn);
            m.w *= mode_gain(mub + ln, a.n_steps, a.cn);
            pair_of(m, w, k0, 1.0 / N, 1.0 / N, &v[i], &v[H + i]);
        }
    } else {
        v4d x[H];  // modes of line a (k, N - k), then of line b
        if (XK) {
#pragma unroll
            for (int i = 0; i < H; ++i) {
                const double2 xa = *reinterpret_cast<const double2*>(W + base + 2 * (t + T * i));
                const double2 xb = *reinterpret_cast<const double2*>(W + base2 + 2 * (t + T * i));
                x[i] = v4d{xa.x, xa.y, xb.x, xb.y};
            }
        } else if (a.vec2) {
            const double* p0 = W + base + es * (2 * t);
#pragma unroll
            for (int i = 0; i < H; ++i) {
                const double2 x0 = *reinterpret_cast<const double2*>(p0);
                const double2 x1 = *reinterpret_cast<const double2*>(p0 + es);
                x[i] = v4d{x0.x, x1.x, x0.y, x1.y};
                p0 += es * (2 * T);
            }
        } else {
#pragma unroll
            for (int i = 0; i < H; ++i) {
                const int64_t o = es * (2 * (t + T * i));
                x[i] = v4d{W[base + o], W[base + o + es], W[base2 + o], W[base2 + o + es]};
            }
        }
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const int k = t + T * i;
            const double2 c = pw[k];
            const v4d m = {x[i].x, x[i].y, two ? x[i].z : 0.0, two ? x[i].w : 0.0};
            pair_of(m, Cd{c.x, c.y}, i == 0 && t == 0, si, si0, &v[i], &v[H + i]);
        }
    }
    t = again(t);
    from_pairs<N, P, XK>(v, sh, t, p);
    t = again(t);
    // the inverse DFT by the forward one with real and imaginary parts swapped
#pragma unroll
    for (int j = 0; j < kE; ++j) v[j] = {v[j].y, v[j].x};
    fft_line<N, P, XK>(v, sh, t, p, tw);
    t = again(t);
    if (MODE == 2) {
        uint32_t top = 0u;
#pragma unroll
        for (int j = 0; j < kE; ++j) top = max(top, max(upper(v[j].x), upper(v[j].y)));
        note_top(a, live ? top : 0u);
    }
    if (XK) {
        const float cut = cut_of(a);
#pragma unroll
        for (int j = 0; j < H; ++j) {
            const int e = 2 * (t + T * j);
            const float2 xa = make_float2(result(v[j].y, cut), __shfl_xor(result(v[kE - 1 - j].y, cut), T - 1));
            const float2 xb = make_float2(result(v[j].x, cut), __shfl_xor(result(v[kE - 1 - j].x, cut), T - 1));
            if (a.vec2) {
                if (live) *reinterpret_cast<float2*>(out + fbase + e) = xa;
                if (two) *reinterpret_cast<float2*>(out + fbase2 + e) = xb;
            } else {
                if (live) {
                    out[fbase + e] = xa.x;
                    out[fbase + e + 1] = xa.y;
                }
                if (two) {
                    out[fbase2 + e] = xb.x;
                    out[fbase2 + e + 1] = xb.y;
                }
            }
        }
    } else {
        if (!live) return;  // (no barrier follows)
        if (a.vec2) {
            double* p0 = W + base + es * (2 * t);
            double* p1 = W + base + es * (N - 1 - 2 * t);
#pragma unroll
            for (int j = 0; j < H; ++j) {
                *reinterpret_cast<double2*>(p0) = make_double2(v[j].y, v[j].x);
                *reinterpret_cast<double2*>(p1) = make_double2(v[H + j].y, v[H + j].x);
                p0 += es * (2 * T);
                p1 -= es * (2 * T);
            }
            return;
        }
#pragma unroll
        for (int j = 0; j < kE; ++j) {
            const int m = t + T * j;
            const int64_t o = es * (j < H ? 2 * m : 2 * N - 1 - 2 * m);
            W[base + o] = v[j].y;
            if (two) W[base2 + o] = v[j].x;
        }
    }
}

// The cells outside the box keep their values, but one that is not finite
// makes its field the CG's, which says what it makes of it.  A wave per row;
// after the first pass, which clears the mark (128 x 128 x 256 cells, 12
// outside in each row: 5.3 us).
__global__ __launch_bounds__(256) void k_outside(SpecPass a, SpecBox b) {
    const float* __restrict__ in = a.in + (size_t)blockIdx.y * a.fcells;
    const int lane = threadIdx.x & 63;
    const int64_t rows = (int64_t)b.nn[1] * b.nn[2], step = (int64_t)gridDim.x * 4;
    bool ok = true;
    for (int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); r < rows; r += step) {
        const int z = (int)(r / b.nn[1]), y = (int)(r - (int64_t)z * b.nn[1]);
        const bool inside = y >= b.lo[1] && y < b.lo[1] + b.len[1] && z >= b.lo[2] && z < b.lo[2] + b.len[2];
        const int skip = inside ? b.len[0] : 0;
        for (int i = lane; i < b.nn[0] - skip; i += 64) ok = ok && isfinite(in[r * b.nn[0] + (i < b.lo[0] ? i : i + skip)]);
    }
    if (!ok) mark_bad(a);
}

// ----------------------------------------------------------- dense lengths

// Row of D element r of v_mfma_f64_16x16x4f64 in a lane (column: lane % 16).
__device__ __forceinline__ int d_row(int r, int lane) { return 4 * r + (lane >> 4); }

// Even and odd halves in LDS, [m][line].  A wave forms one 16-row tile of
// the half-size products for the block's 16 lines: its even and odd products
// are two independent accumulator chains.  SPLIT, for one or two tiles: 32
// lines, a wave per tile and half.  A block has as many waves as tiles, so
// none idles in the products, and at least four, for the latency of its loads.
// 16 lines rather than 32 with both halves in one wave: twice the blocks, of
// half the LDS (37 KB at n = 275), so a block's load, product and store
// phases overlap another's.  Measured, 32 -> 16 lines: 66 us -> 61 forward or
// back along contiguous n = 275 for 7.5M cells (30 us at the 78.6 TFLOP/s of
// the float64 matrix cores, which bound it together with the phases), 51 ->
// 50 along strided 147, gain pass along 93 66 -> 65 (with float32 vectors
// between the passes; with float64 ones 62 and 65, 54 and 48, 70); 96 x 64 x
// 80 cells, 2 fields: 19.4 -> 15.1 us for the gain pass (now 17.4), 13.6 ->
// 10.5 and 11.7 -> 8.9 along x (now 12.0 and 9.8).
template <int MODE, bool XK, bool SPLIT, int kTL>
__global__ __launch_bounds__(1024) void k_dense(SpecPass a) {
    extern __shared__ double shd[];
    constexpr int TLP = XK ? kTL + 1 : kTL;
    constexpr int CT = SPLIT ? 1 : kTL / 16;
    const int n = a.n, hm = a.hm, ho = a.ho, mt = (hm + 15) / 16, rows = 16 * mt;
    double* E = shd;
    double* O = shd + (size_t)rows * TLP;
    if (MODE == 1 && XK && is_bad(a)) return;
    if (MODE == 0 && XK) clear_notes(a);
    const float* __restrict__ in = a.in + (size_t)blockIdx.y * a.fcells;
    float* __restrict__ out = a.out + (size_t)blockIdx.y * a.fcells;
    double* __restrict__ W = a.W + (size_t)blockIdx.y * a.cells;
    // 16 strided lines share cache lines with the next block's (unless rows
    // are a multiple of 16 long): the two blocks go to one XCD (y at 275 x 147
    // x 93, 2 fields: 54 us against 59)
    unsigned lb = blockIdx.x;
    if (!SPLIT && !XK && lb < gridDim.x / 16 * 16) lb = lb / 16 * 16 + lb % 8 * 2 + lb / 8 % 2;
    const int64_t l0 = (int64_t)lb * kTL;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int tile = SPLIT ? wave >> 1 : wave, c0 = SPLIT ? (wave & 1) * 16 : 0;
    const bool work = tile < mt;  // (a block of few tiles has waves that only move data)
    const int64_t es = a.estride;
    auto base_of = [&](int64_t l, bool field) -> int64_t {
        if (XK) return field ? field_row(a, l) : l * n;
        const int64_t o = l / a.inner;
        return o * a.ostride + (l - o * a.inner);
    };
    // E and O: x[m] +- x[N-1-m], or (inverse) the even and odd modes.  Loads
    // at clamped places, four pairs in flight per thread.
    float least = 0.f;
    uint32_t most = 0u;
    auto fill = [&](const auto* __restrict__ src, int64_t step, int m0, int dm, int line, bool ok) {
        for (int m = m0; m < rows; m += 4 * dm) {
            std::remove_cv_t<std::remove_reference_t<decltype(*src)>> u[4], w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int mc = std::min(m + i * dm, hm - 1);
                u[i] = src[step * mc];
                w[i] = src[step * (MODE == 1 ? std::min(hm + mc, n - 1) : n - 1 - mc)];
            }
            if (MODE == 0 && XK) {
#pragma unroll
                for (int i = 0; i < 4; ++i) least = fminf(least, fminf(u[i], w[i]));  // (!ok: some of the box)
            }
            if (MODE == 2) {
#pragma unroll
                for (int i = 0; i < 4; ++i) most = max(most, ok ? max(upper(u[i]), upper(w[i])) : 0u);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int mi = m + i * dm;
                if (mi >= rows) break;
                const double e = MODE == 1 || mi >= ho ? (double)u[i] : (double)u[i] + (double)w[i];
                const double o = MODE == 1 ? (double)w[i] : (double)u[i] - (double)w[i];
                E[mi * TLP + line] = ok && mi < hm ? e : 0.0;
                O[mi * TLP + line] = ok && mi < ho ? o : 0.0;
            }
        }
    };
    if (XK) {
        for (int line = wave; line < kTL; line += nw) {
            const bool ok = l0 + line < a.lines;
            if constexpr (MODE == 0) fill(in + (ok ? base_of(l0 + line, true) : a.off), 1, lane, 64, line, ok);
            else fill(W + (ok ? base_of(l0 + line, false) : 0), 1, lane, 64, line, ok);
        }
        if (MODE == 0) mark_negative(a, least);
    } else {
        const int line = threadIdx.x % kTL;
        const bool ok = l0 + line < a.lines;
        fill(W + (ok ? base_of(l0 + line, false) : 0), es, threadIdx.x / kTL, nw * 64 / kTL, line, ok);
        if (MODE == 2 && most >= kBeyond) mark_bad(a);
    }
    __syncthreads();
    v4d ae[CT], ao[CT];
    auto multiply = [&](const double* __restrict__ me, const double* __restrict__ mo) {
#pragma unroll
        for (int c = 0; c < CT; ++c) ae[c] = ao[c] = v4d{0, 0, 0, 0};
        if (!work) return;
        const double* fe = me + (size_t)tile * mt * 256 + lane;
        const double* fo = mo + (size_t)tile * mt * 256 + lane;
        const int at = (lane >> 4) * TLP + c0 + (lane & 15);
        // 16 reduction rows at a time, the matrices' next fragments in flight
        double ce[4], co[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ce[i] = fe[i * 64];
            co[i] = fo[i * 64];
        }
        for (int k = 0; k < mt; ++k) {
            double ne[4], no[4];
            const bool odd = ho > 0;
            const size_t nk = (size_t)std::min(k + 1, mt - 1) * 256;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                ne[i] = fe[nk + i * 64];
                no[i] = fo[nk + i * 64];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    const int o = (16 * k + 4 * i) * TLP + at + 16 * c;
                    const double de = E[o], dd = O[o];
                    if (XK) {
                        ae[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(de, ce[i], ae[c], 0, 0, 0);
                        if (odd) ao[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(dd, co[i], ao[c], 0, 0, 0);
                    } else {
                        ae[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(ce[i], de, ae[c], 0, 0, 0);
                        if (odd) ao[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(co[i], dd, ao[c], 0, 0, 0);
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                ce[i] = ne[i];
                co[i] = no[i];
            }
        }
    };
    if (MODE != 1) multiply(a.fe, a.fo);
    if (MODE == 0) {
#pragma unroll
        for (int c = 0; c < CT; ++c) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int k = tile * 16 + (XK ? (lane & 15) : d_row(r, lane));
                const int line = c0 + c * 16 + (XK ? d_row(r, lane) : (lane & 15));
                if (l0 + line >= a.lines || k >= hm) continue;
                double* dst = W + base_of(l0 + line, false);
                dst[es * k] = ae[c][r];
                if (k < ho) dst[es * (hm + k)] = ao[c][r];
            }
        }
        return;
    }
    if (MODE == 2) {
        __syncthreads();
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const int line = c0 + c * 16 + (lane & 15);
            const int64_t l = std::min(l0 + line, a.lines - 1);
            const int64_t y = l / a.n0;
            const double mu = a.c0 * a.lam0[l - y * a.n0] + (a.lam1 ? a.c1 * a.lam1[y] : 0.0);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int k = tile * 16 + d_row(r, lane);
                const bool ie = k < hm, io = k < ho;
                const double e = ie ? ae[c][r] * mode_gain(fma(a.cm, a.lamm[k], mu), a.n_steps, a.cn) : 0.0;
                const double o = io ? ao[c][r] * mode_gain(fma(a.cm, a.lamm[hm + k], mu), a.n_steps, a.cn) : 0.0;
                if (work) {
                    E[k * TLP + line] = e;
                    O[k * TLP + line] = o;
                }
            }
        }
        __syncthreads();
    }
    multiply(a.ie, a.io);
    const float cut = XK ? cut_of(a) : 0.f;
    uint32_t top = 0u;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = tile * 16 + (XK ? (lane & 15) : d_row(r, lane));
            const int line = c0 + c * 16 + (XK ? d_row(r, lane) : (lane & 15));
            if (l0 + line >= a.lines || m >= hm) continue;
            const double p = ae[c][r] + ao[c][r], q = ae[c][r] - ao[c][r];
            if (XK) {
                float* dst = out + base_of(l0 + line, true);
                dst[m] = result(p, cut);
                if (m < ho) dst[n - 1 - m] = result(q, cut);
            } else {
                double* dst = W + base_of(l0 + line, false);
                dst[es * m] = p;
                if (m < ho) dst[es * (n - 1 - m)] = q;
                top = max(top, max(upper(p), m < ho ? upper(q) : 0u));
            }
        }
    }
    if (MODE == 2) note_top(a, top);
}

// ------------------------------------------------------------------ tables

// Per axis: the eigenvalues 4 sin^2(pi k / 2n) at the stored positions, then
// for an FFT length e^{-2 pi i q / n} [n] and e^{-i pi k / 2n} [n / 2], for a
// dense length the four packed half-size matrices (orthonormal scaling).
// per: a periodic axis, 4 sin^2(pi k / n) and the matrices of the cosines
// (even) and sines (odd) of 2 pi k (m + 1/2) / n.
__global__ __launch_bounds__(256) void k_spec_tables(int n, int fft, int per, double* lam, double2* tw, double2* pw, double* fe,
                                                    double* fo, double* ie, double* io) {
    const int hm = (n + 1) / 2, ho = n / 2, mt = (hm + 15) / 16, ks = 4 * mt;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t p = t0; p < n; p += stride) {
        int k;
        if (fft) k = p == 0 ? 0 : (p == 1 ? n / 2 : ((p & 1) ? n - (int)p / 2 : (int)p / 2));
        else if (per) k = 2 * (p < hm ? (int)p : (int)p - hm + 1);
        else k = p < hm ? 2 * (int)p : 2 * ((int)p - hm) + 1;
        const double s = sinpi(0.5 * k / n);
        lam[p] = 4.0 * s * s;
    }
    if (fft) {
        for (int64_t q = t0; q < n; q += stride) {
            double s, c;
            sincospi(2.0 * (double)q / n, &s, &c);
            tw[q] = make_double2(c, -s);
            if (q < n / 2) {
                sincospi(0.5 * (double)q / n, &s, &c);
                pw[q] = make_double2(c, -s);
            }
        }
        return;
    }
    const int64_t frag = (int64_t)mt * ks * 64;
    for (int64_t i = t0; i < frag; i += stride) {
        const int lane = (int)(i & 63);
        const int64_t f = i >> 6;
        const int row = (int)(f / ks) * 16 + (lane & 15), col = (int)(f % ks) * 4 + (lane >> 4);
        // orthonormal DCT-II entry of mode k at point m
        auto entry = [&](int k, int m) {
            const int64_t ph = ((int64_t)k * (2 * m + 1)) % (4 * (int64_t)n);
            return sqrt((k ? 2.0 : 1.0) / n) * cospi((double)ph / (2.0 * n));
        };
        // ... and of the sine of (even) k at point m
        auto sine = [&](int k, int m) {
            const int64_t ph = ((int64_t)k * (2 * m + 1)) % (4 * (int64_t)n);
            return sqrt((k == n ? 1.0 : 2.0) / n) * sinpi((double)ph / (2.0 * n));
        };
        fe[i] = row < hm && col < hm ? entry(2 * row, col) : 0.0;
        fo[i] = row < ho && col < ho ? (per ? sine(2 * row + 2, col) : entry(2 * row + 1, col)) : 0.0;
        ie[i] = row < hm && col < hm ? entry(2 * col, row) : 0.0;
        io[i] = row < ho && col < ho ? (per ? sine(2 * col + 2, row) : entry(2 * col + 1, row)) : 0.0;
    }
}

__global__ void k_spec_clear(uint32_t* p, int n) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0u;
}

bool fft_length(int n) { return n == 128 || n == 256 || n == 512 || n == 1024; }

// Doubles of one packed half-size matrix: tiles of 16 rows, 4 fragments of 64
// per 16 reduction rows.
size_t dense_fragment(int n, bool sym = true) {
    const size_t mt = ((sym ? (n + 1) / 2 : n) + 15) / 16;
    return mt * 4 * mt * 64;
}

bool uses_fft(const SpecTables& t, int a) { return !t.eigen[a] && !t.per[a] && fft_length(t.n[a]); }

size_t table_doubles(int n, bool fft) {
    if (fft) return (size_t)n + 2 * (size_t)n + (size_t)n;
    return (((size_t)n + 1) & ~(size_t)1) + 4 * dense_fragment(n);
}

template <int N, int MODE, bool XK>
void launch_fft(const SpecPass& a, int F, hipStream_t s) {
    constexpr int P = fft_pairs<N, XK>();
    const dim3 grid((unsigned)((a.pairs + P - 1) / P), F);
    hipLaunchKernelGGL((k_fft<N, MODE, XK>), grid, dim3(P * N / kE), 0, s, a);
}

template <int MODE, bool XK>
cgd_status launch_pass(const SpecPass& a, int F, hipStream_t s) {
    switch (a.tw ? a.n : 0) {
        case 128: launch_fft<128, MODE, XK>(a, F, s); return CGD_OK;
        case 256: launch_fft<256, MODE, XK>(a, F, s); return CGD_OK;
        case 512: launch_fft<512, MODE, XK>(a, F, s); return CGD_OK;
        case 1024: launch_fft<1024, MODE, XK>(a, F, s); return CGD_OK;
        default: break;
    }
    const int mt = (a.hm + 15) / 16;
    auto go = [&](auto kern, int nw, int tl) -> cgd_status {
        const dim3 grid((unsigned)((a.lines + tl - 1) / tl), F);
        const size_t lds = (size_t)2 * mt * 16 * (XK ? tl + 1 : tl) * sizeof(double);
        if (lds > 64 * 1024)
            CGD_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        hipLaunchKernelGGL(kern, grid, dim3(nw * 64), lds, s, a);
        return CGD_OK;
    };
    // one or two tiles: a wave per tile and column tile, for the latency
    if (mt <= 2) return go(k_dense<MODE, XK, true, 32>, 4, 32);
    return go(k_dense<MODE, XK, false, 16>, std::max(4, mt), 16);
}

// Forms an axis's packed matrices from its modes' rotations: a thread per
// cell (column of the eigenvector matrix z, in LDS as [vector][thread], with
// one row more for what is not stored), the rotations in groups of four
// sweeps (RotationGroups), whose chains overlap.  One wave per block, bound by
// the rotations' latency: 65,000 (a half of 512 mirror-symmetric cells) in
// 1,600 us; one sweep at a time 4,200 us.  Together with finding the
// rotations, a first call on 512 x 32 x 16 cells takes 3.9 ms, where the host
// formed z in 10.8 (the CG 5.9, making the mesh 11).
// blockIdx.y: half (even, odd modes).
struct ModeArgs {
    const double2* cs[2];
    const RotationGroups::Group* groups[2];
    int n_groups[2];
    int nn[2];          // vectors and cells of the half
    int mt, ho;         // tiles of the packed matrices; cells that stand for two
    const double* h;    // cell widths
    double* f[2];
    double* inv[2];
};
// x of lane k (the same k in all lanes).
__device__ __forceinline__ double lane_value(double x, int k) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, k), hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), k);
    return __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
}
__global__ __launch_bounds__(64) void k_spec_modes(ModeArgs a) {
    constexpr int L = RotationGroups::kLanes, S = RotationGroups::kGroupSteps, B = 8;
    static_assert(L * S == 64 && S % B == 0);
    extern __shared__ double z[];
    const int lane = threadIdx.x, half = blockIdx.y, nn = a.nn[half], m = blockIdx.x * 64 + lane;
    if ((int)blockIdx.x * 64 >= nn) return;
    for (int k = 0; k < nn; ++k) z[k * 64 + lane] = k == m ? 1.0 : 0.0;
    // (a thread only touches its own column: no barrier)
    const double2* cs = a.cs[half] + lane;
    double2 next = a.n_groups[half] ? cs[0] : make_double2(1.0, 0.0);
    for (int i = 0; i < a.n_groups[half]; ++i) {
        const RotationGroups::Group g = a.groups[half][i];
        const double* in = z + g.lo * 64 + lane;
        double u[L] = {in[0]};
        for (int t0 = 0; t0 < g.count; t0 += S) {
            // a lane holds one of the 64 rotations of S steps; the next ones are in flight
            const double2 mine = next;
            cs += 64;
            if (t0 + S < g.count || i + 1 < a.n_groups[half]) next = cs[0];
#pragma unroll
            for (int b = 0; b < S; b += B) {
                double v[B];
#pragma unroll
                for (int t = 0; t < B; ++t) v[t] = in[64 * min(t0 + b + t + 1, g.rows - 1)];
#pragma unroll
                for (int t = 0; t < B; ++t) {
#pragma unroll
                    for (int j = 0; j < L; ++j) {
                        const double c = lane_value(mine.x, (b + t) * L + j), s = lane_value(mine.y, (b + t) * L + j);
                        const double o = c * u[j] + s * v[t];
                        u[j] = c * v[t] - s * u[j];
                        v[t] = o;
                    }
                }
#pragma unroll
                for (int t = 0; t < B; ++t) {
                    const int r = t0 + b + t + 1 - L;
                    z[(r >= 0 && r < g.rows ? g.lo + r : nn) * 64 + lane] = v[t];
                }
            }
        }
    }
    if (m >= nn) return;
    const double g = m < a.ho ? 0.70710678118654752440 : 1.0, r = sqrt(a.h[m]);
    for (int k = 0; k < nn; ++k) {
        // entry (row, col) of a packed matrix
        auto at = [&](int row, int col) {
            return (((size_t)(row / 16) * 4 * a.mt + col / 4) * 64) + (size_t)(col % 4) * 16 + row % 16;
        };
        const double v = z[k * 64 + lane] * g;
        a.f[half][at(k, m)] = v * r;
        a.inv[half][at(m, k)] = v / r;
    }
}

}  // namespace

// The cells that diffuse, as a box of axes the transforms take.
static void analyse_grid(const cgd_mesh m, SpecTables* t) {
    const HexGeom& g = m->hex;
    const int nn[3] = {g.nx, g.ny, g.nz};
    int i0[3] = {0, 0, 0}, len[3] = {nn[0], nn[1], nn[2]};
    double d = 1.0;
    if (m->kind == 2) {
        const RectOp* ro = m->rop;
        for (int a = 0; a < 3; ++a) {
            const std::vector<double>& f = ro->fac[a];
            int lo = 0, hi = nn[a];
            while (lo < hi && !(f[lo] > 0.0)) ++lo;
            while (hi > lo && !(f[hi - 1] > 0.0)) --hi;
            if (lo == hi) return;  // nothing diffuses
            for (int i = lo; i < hi; ++i)
                if (std::fabs(f[i] - f[lo]) > 1e-12 * f[lo]) return;
            d *= f[lo];
            i0[a] = lo;
            len[a] = hi - lo;
        }
    }
    for (int a = 0; a < 3; ++a) {
        t->box.nn[a] = nn[a];
        t->box.lo[a] = i0[a];
        t->box.len[a] = len[a];
    }
    int64_t st = 1;
    for (int a = 0; a < 3; ++a) {
        if (m->kind == 0 || a > 0) {
            if (len[a] == 1) continue;
        } else if (len[0] < 2) {
            return;
        }
        const int r = t->rank++, n = len[a];
        t->n[r] = n;
        bool even = true, sym = true;
        double diag = 0.0, mean = g.h[a];
        if (m->kind == 2) {
            const RectOp* ro = m->rop;
            const std::vector<double> h(ro->h[a].begin() + i0[a], ro->h[a].begin() + i0[a] + n);
            mean = 0.0;
            for (double w : h) mean += w / n;
            for (int i = 0; i < n; ++i) {
                even = even && std::fabs(h[i] - mean) <= 1e-9 * mean;
                sym = sym && std::fabs(h[i] - h[n - 1 - i]) <= 1e-9 * h[i];
                const double w0 = h[i > 0 ? i - 1 : n - 1], w1 = h[i + 1 < n ? i + 1 : 0];
                diag = std::max(diag, (2.0 / (w0 + h[i]) + 2.0 / (h[i] + w1)) / h[i]);
            }
            t->per[r] = (ro->per >> a & 1) && n == nn[a];
            t->eigen[r] = !even;
            if (t->eigen[r]) t->h[r] = h;
        } else {
            diag = 2.0 / (mean * mean);
        }
        t->sym[r] = sym;
        t->scale[r] = t->eigen[r] ? d : d / (mean * mean);
        t->diag += d * diag;
        if (!sym && (t->per[r] || n > 256)) return;
        if (n > 512 && !uses_fft(*t, r)) return;
        st *= n;
    }
    if (t->rank < 2) return;
    t->cells = st;
    t->off = i0[0] + (int64_t)nn[0] * (i0[1] + (int64_t)nn[1] * i0[2]);
    t->pitch = m->kind == 0 ? t->n[0] : nn[0];
    if (m->kind == 2 && len[1] != nn[1] && len[2] > 1) {
        t->rows_y = len[1];
        t->sy = nn[0];
        t->sz = (int64_t)nn[0] * nn[1];
    }
    t->ok = true;
}

static const SpecTables* grid_of(cgd_mesh m) {
    if (!m->spec) {
        SpecTables* t = new (std::nothrow) SpecTables();
        if (!t) return nullptr;
        try {
            analyse_grid(m, t);
        } catch (const std::bad_alloc&) {
            delete t;
            return nullptr;
        }
        m->spec = t;
    }
    return m->spec;
}

// Fields per group: their vector W (with the field itself about 192 MB) stays
// in the memory-side cache between the passes.
static int fields_per_group(const cgd_mesh m, int F) {
    const int64_t most = (int64_t)128 * 1024 * 1024 / (m->spec->cells * (int64_t)sizeof(double));
    return (int)std::max<int64_t>(1, std::min<int64_t>(F, most));
}

size_t spectral_bytes(const cgd_mesh m, int32_t F) {
    return (size_t)fields_per_group(m, F) * (m->spec->cells * sizeof(double) + kTopSlots * kTopStride * sizeof(uint32_t));
}

// The modes of the axes of uneven cells, on the first call that needs them; a
// mesh for which they are not found stays with the CG.
static bool modes_found(SpecTables* t) {
    if (t->dev) return true;
    try {
        for (int a = 0; a < t->rank && t->ok; ++a)
            if (t->eigen[a] && t->modes[a].lam.empty())
                t->ok = axis_modes(t->h[a], t->sym[a], t->per[a], t->modes[a].rot, t->modes[a].lam);
    } catch (const std::bad_alloc&) {
        for (AxisModes& mo : t->modes) mo = AxisModes();  // (half an axis is no axis: the next call starts again)
        return false;
    }
    return t->ok;
}

// The environment switches that choose how the CG runs: set, they mean it.
static bool switched_to_cg() {
    for (const char* e : {"CGD_NO_DIRECT", "CGD_HEX_PRECOND_DEG", "CGD_HEX_LDS_ZC", "CGD_HEX_DIR", "CGD_HEX_DIR_NW",
                          "CGD_HEX_DIR_ZC", "CGD_HEX_NO_SWAP", "CGD_HEX_TILE", "CGD_HEX_TILE1", "CGD_HEX_TILE2",
                          "CGD_HEX_TILEZ", "CGD_NO_BUDGET"})
        if (getenv(e)) return true;
    return false;
}

// The direct solve stands in for the CG where nothing asks for the CG itself:
// its iterations and residuals (statistics), a start from a guess, plain CG,
// or a switch of its own; where the float32 result can meet the
// stopping rule's meaning (rounding the result alone leaves a relative
// residual of up to lmax 2^-25, 4e-7 at dtau / h^2 = 1, so tolerances below
// the default stay with the CG's recursive residual); where the CG would
// have converged within max_iter by its bound for the unpreconditioned
// operator, so that a call that came back not converged still does; and
// where it is the faster one: a transform takes about 2.45 ps per cell for an
// FFT length and 3.3 + 0.021 n for a dense one (7.5M cells: 62 and 65 us at n
// = 275, 54 and 48 at 147, 35 at 93), the CG 25 ps per cell and step at its
// best (256 x 256 x 512, dtau / h^2 = 1) and 50 us and more per step in
// launches on the smallest grids, so only one or two steps on lengths of
// hundreds that are no FFT lengths are left to the CG (1 step at b = 2h and 4h,
// 275 x 147 x 93: direct 189 us, CG 160 and 360; 400 x 300 x 64: 381, 214 and
// 538; 120^3: 109, 201 and 203).  Rectilinear grids: the CG takes 136 ps per
// cell and step (128 x 128 x 256, diffusivity 0 in the outer layers).  The
// times are one field's, whatever their number, so that a field comes out as
// the same bits alone, among others and in a batch.
bool spectral_applies(cgd_mesh m, const DiffuseArgs& da, bool stats) {
    if (stats || da.x0_mode != 0 || da.precond != 0 || da.rtol < 5e-7) return false;
    if (m->kind == 2 ? !m->rop || getenv("CGD_RECT_SLOTS") : m->kind != 0) return false;
    if (switched_to_cg()) return false;
    const SpecTables* t = grid_of(m);
    if (!t || !t->ok) return false;
    const double dtau = da.bandwidth * da.bandwidth / 4.0 / da.n_steps * (da.scheme == 1 ? 0.5 : 1.0);
    double ps = 0.0;
    for (int a = 0; a < t->rank; ++a)
        ps += 2.0 * (uses_fft(*t, a) ? 2.45 : 3.3 + (t->sym[a] ? 0.021 : 0.042) * t->n[a]);
    const double mcells = 1e-6 * (double)m->cells;
    if (25.0 + mcells * ps > da.n_steps * (50.0 + mcells * (m->kind == 0 ? 25.0 : 100.0))) return false;
    const double r = sqrt(1.0 + 2.0 * dtau * t->diag);
    return 0.5 * r * log(2.0 * r / std::min(da.rtol, 1.0)) + 1.0 <= (double)da.max_iter && modes_found(m->spec);
}

void destroy_spectral(cgd_mesh m) {
    if (!m->spec) return;
    if (m->spec->dev) (void)hipFree(m->spec->dev);
    delete m->spec;
    m->spec = nullptr;
}

// Doubles of an eigenvector axis's data on the device: eigenvalues, widths
// (both padded to an even number), and per half the rotations and groups.
static size_t group_doubles(const RotationGroups& r) {
    return (r.groups.size() * sizeof(RotationGroups::Group) + 15) / 16 * 2;
}
static size_t modes_doubles(const AxisModes& mo, int n) {
    size_t d = 2 * ((size_t)n + (n & 1));
    for (const RotationGroups& r : mo.rot) d += r.cs.size() + group_doubles(r);
    return d;
}

// An eigenvector axis's data and packed matrices; dst: modes_doubles, 16-byte
// aligned.  Waits for the stream.
static hipError_t upload_modes(const SpecTables& t, int a, double* dst, SpecAxis& x, hipStream_t s) {
    const AxisModes& mo = t.modes[a];
    const int n = t.n[a];
    ModeArgs ma = {};
    std::vector<double> up;
    try {
        up = mo.lam;
        up.resize(modes_doubles(mo, n));
    } catch (const std::bad_alloc&) {
        return hipErrorOutOfMemory;
    }
    size_t at = (size_t)n + (n & 1);
    ma.h = dst + at;
    std::copy(t.h[a].begin(), t.h[a].end(), up.begin() + at);
    at += (size_t)n + (n & 1);
    for (int odd = 0; odd < 2; ++odd) {
        const RotationGroups& r = mo.rot[odd];
        ma.cs[odd] = reinterpret_cast<const double2*>(dst + at);
        std::copy(r.cs.begin(), r.cs.end(), up.begin() + at);
        at += r.cs.size();
        ma.groups[odd] = reinterpret_cast<const RotationGroups::Group*>(dst + at);
        if (!r.groups.empty()) memcpy(up.data() + at, r.groups.data(), r.groups.size() * sizeof(RotationGroups::Group));
        at += group_doubles(r);
        ma.n_groups[odd] = (int)r.groups.size();
    }
    x.lam = dst;
    const size_t frag = dense_fragment(n, t.sym[a]);
    ma.nn[0] = t.sym[a] ? (n + 1) / 2 : n;
    ma.ho = ma.nn[1] = t.sym[a] ? n / 2 : 0;
    ma.mt = (ma.nn[0] + 15) / 16;
    ma.f[0] = x.fe;
    ma.f[1] = x.fo;
    ma.inv[0] = x.ie;
    ma.inv[1] = x.io;
    hipError_t e = hipMemcpyAsync(dst, up.data(), up.size() * sizeof(double), hipMemcpyHostToDevice, s);
    const size_t lds = ((size_t)ma.nn[0] + 1) * 64 * sizeof(double);  // <= 128.5 KB (256 vectors)
    if (e == hipSuccess && lds > 64 * 1024)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_spec_modes), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_spec_clear, dim3(64), dim3(256), 0, s, reinterpret_cast<uint32_t*>(x.fe), (int)(8 * frag));
        hipLaunchKernelGGL(k_spec_modes, dim3((ma.nn[0] + 63) / 64, ma.ho ? 2 : 1), dim3(64), lds, s, ma);
        e = hipGetLastError();
    }
    const hipError_t w = hipStreamSynchronize(s);  // (`up` goes)
    return e == hipSuccess ? w : e;
}

static cgd_status spectral_tables(cgd_mesh m, hipStream_t s) {
    SpecTables* t = m->spec;
    if (t->dev) return CGD_OK;
    size_t off[3], total = 0;
    for (int a = 0; a < t->rank; ++a) {
        off[a] = total;
        total += t->eigen[a] ? (((size_t)t->n[a] + 1) & ~(size_t)1) + 4 * dense_fragment(t->n[a], t->sym[a])
                             : table_doubles(t->n[a], uses_fft(*t, a));
    }
    size_t off_modes[3] = {};
    for (int a = 0; a < t->rank; ++a) {
        if (!t->eigen[a]) continue;
        total += total & 1;  // (16-byte rotations)
        off_modes[a] = total;
        total += modes_doubles(t->modes[a], t->n[a]);
    }
    const size_t neg = total;  // after the tables: a 32-bit word per field
    total += kSpecFields / 2;
    void* dev = nullptr;
    if (hipMalloc(&dev, total * sizeof(double)) != hipSuccess) {
        (void)hipGetLastError();
        set_error("allocation of the transform tables failed");
        return CGD_E_NOMEM;
    }
    t->neg = reinterpret_cast<uint32_t*>(static_cast<double*>(dev) + neg);
    hipLaunchKernelGGL(k_spec_clear, dim3(8), dim3(256), 0, s, t->neg, kSpecFields);
    hipError_t e = hipGetLastError();
    for (int a = 0; a < t->rank && e == hipSuccess; ++a) {
        SpecAxis& x = t->axis[a];
        double* p = static_cast<double*>(dev) + off[a];
        const int n = t->n[a];
        x = SpecAxis{};
        x.n = n;
        x.lam = p;
        const bool fft = uses_fft(*t, a);
        if (fft) {
            x.tw = reinterpret_cast<double2*>(p + n);
            x.pw = x.tw + n;
        } else {
            const size_t frag = dense_fragment(n, t->sym[a]);
            x.fe = p + ((n + 1) & ~1);
            x.fo = x.fe + frag;
            x.ie = x.fo + frag;
            x.io = x.ie + frag;
        }
        if (t->eigen[a]) {
            e = upload_modes(*t, a, static_cast<double*>(dev) + off_modes[a], x, s);
        } else {
            hipLaunchKernelGGL(k_spec_tables, dim3(64), dim3(256), 0, s, n, (int)fft, (int)t->per[a], x.lam, x.tw, x.pw,
                               x.fe, x.fo, x.ie, x.io);
            e = hipGetLastError();
        }
    }
    if (e != hipSuccess) {
        (void)hipFree(dev);
        set_error(std::string("transform tables: ") + hipGetErrorString(e));
        return e == hipErrorOutOfMemory ? CGD_E_NOMEM : CGD_E_HIP;
    }
    t->dev = static_cast<double*>(dev);
    for (AxisModes& mo : t->modes) mo = AxisModes();
    return CGD_OK;
}

cgd_status spectral_enqueue(cgd_mesh m, const DiffuseArgs& da, int n_fields, double* W, int* bad, int* bad_host,
                            Timing* timing, hipStream_t s) {
    cgd_status rc = spectral_tables(m, s);
    if (rc != CGD_OK) return rc;
    if (++m->spec->calls == 0) ++m->spec->calls;  // (0 is what the notes start from)
    const SpecTables& tb = *m->spec;
    const int rank = tb.rank;
    const int* n = tb.n;
    double c[3];
    const double dtau = da.bandwidth * da.bandwidth / 4.0 / da.n_steps * (da.scheme == 1 ? 0.5 : 1.0);
    for (int a = 0; a < rank; ++a) c[a] = dtau * tb.scale[a];
    // the mode that holds a plane's sum, over its mean (a weighted one on an eigenvector axis)
    double plane = 1.0;
    for (int a = 0; a + 1 < rank; ++a) {
        double len = n[a];
        if (tb.eigen[a]) {
            len = 0.0;
            for (double w : tb.h[a]) len += w;
        }
        plane *= len;
    }
    SpecPass pass[3];
    for (int ax = 0; ax < rank; ++ax) {
        SpecPass& p = pass[ax];
        p = SpecPass{};
        const SpecAxis& t = tb.axis[ax];
        const double nn = n[ax];
        p.cells = tb.cells;
        p.fcells = m->cells;
        p.off = tb.off;
        p.sy = tb.sy;
        p.sz = tb.sz;
        p.pitch = tb.pitch;
        p.rows_y = tb.rows_y;
        p.hm = tb.sym[ax] ? (n[ax] + 1) / 2 : n[ax];
        p.ho = tb.sym[ax] ? n[ax] / 2 : 0;
        p.n_steps = da.n_steps;
        p.cn = da.scheme == 1;
        p.n = n[ax];
        p.tw = t.tw;
        p.pw = t.pw;
        p.fe = t.fe;
        p.fo = t.fo;
        p.ie = t.ie;
        p.io = t.io;
        p.sf = sqrt(2.0 / nn);
        p.sf0 = sqrt(1.0 / nn);
        p.si = sqrt(0.5 / nn);
        p.si0 = sqrt(1.0 / nn);
        p.lines = tb.cells / n[ax];
        int64_t st = 1;
        for (int b = 0; b < ax; ++b) st *= n[b];
        p.estride = st;
        p.inner = st;
        p.inner_pairs = (st + 1) / 2;
        p.ostride = st * n[ax];
        p.pairs = ax == 0 ? (p.lines + 1) / 2 : p.inner_pairs * (p.lines / st);
        p.vec2 = ax > 0 && st % 2 == 0;
        p.W = W;
        p.call = tb.calls;
        p.cut = 0x1p-32 / sqrt(plane);
    }
    SpecPass& z = pass[rank - 1];
    z.cm = c[rank - 1];
    z.lamm = m->spec->axis[rank - 1].lam;
    z.n0 = n[0];
    z.c0 = c[0];
    z.lam0 = m->spec->axis[0].lam;
    if (rank == 3) {
        z.c1 = c[1];
        z.lam1 = m->spec->axis[1].lam;
    }
    const int group = fields_per_group(m, n_fields);
    uint32_t* top = reinterpret_cast<uint32_t*>(W + (size_t)group * tb.cells);
    for (int f0 = 0; f0 < n_fields; f0 += group) {
        const int nf = std::min(group, n_fields - f0);
        float* field = da.field + (size_t)f0 * m->cells;
        for (int ax = 0; ax < rank; ++ax) {
            pass[ax].bad = bad + f0;
            pass[ax].bad_host = bad_host ? bad_host + f0 : nullptr;
            pass[ax].top = top;
            pass[ax].neg = tb.neg + f0;
        }
        SpecPass x = pass[0];
        x.in = field;
        x.out = field;
        x.vec2 = reinterpret_cast<uintptr_t>(field) % 8 == 0 && tb.off % 2 == 0 &&
                 (tb.rows_y ? (tb.sy | tb.sz) % 2 == 0 : tb.pitch % 2 == 0) && (nf == 1 || m->cells % 2 == 0);
        // a timed pass: 12 bytes per cell along x (kind 0), 16 along the other axes (kind 1)
        auto timed = [&](int kind, cgd_status (*launch)(const SpecPass&, int, hipStream_t), const SpecPass& p) {
            const int t = timing ? timing_begin(timing, s) : -1;
            const cgd_status r = launch(p, nf, s);
            if (timing) timing_end(timing, t, kind, (kind ? 16.0 : 12.0) * (double)tb.cells * nf, s);
            return r;
        };
        rc = timed(0, launch_pass<0, true>, x);
        if (rc == CGD_OK && tb.cells < m->cells) {
            const int64_t rows = (int64_t)tb.box.nn[1] * tb.box.nn[2];
            hipLaunchKernelGGL(k_outside, dim3((unsigned)std::min<int64_t>(2048, (rows + 3) / 4), nf), dim3(256), 0, s, x,
                               tb.box);
        }
        if (rc == CGD_OK && rank == 3) rc = timed(1, launch_pass<0, false>, pass[1]);
        if (rc == CGD_OK) rc = timed(1, launch_pass<2, false>, z);
        if (rc == CGD_OK && rank == 3) rc = timed(1, launch_pass<1, false>, pass[1]);
        if (rc == CGD_OK) rc = timed(0, launch_pass<1, true>, x);
        if (rc != CGD_OK) return rc;
    }
    CGD_HIP_TRY(hipGetLastError());
    return CGD_OK;
}

cgd_status diffuse_spectral(cgd_mesh m, const DiffuseArgs& da, hipStream_t s) {
    cgd_status rc = ensure_workspace(m, kSmallFixed + spectral_bytes(m, da.F));
    if (rc != CGD_OK) return rc;
    rc = ensure_pinned(m, kPinBytes);
    if (rc != CGD_OK) return rc;
    char* base = static_cast<char*>(m->ws.ptr);
    int* bad_host = reinterpret_cast<int*>(static_cast<char*>(m->pinned) + kPinStatus);
    for (int f = 0; f < da.F; ++f) bad_host[f] = 0;
    rc = spectral_enqueue(m, da, da.F, reinterpret_cast<double*>(base + kSmallFixed),
                          reinterpret_cast<int*>(base + kOffStatus), bad_host, &m->timing, s);
    if (rc != CGD_OK) return rc;
    CGD_HIP_TRY(hipStreamSynchronize(s));
    timing_collect(&m->timing);
    // fields the transforms cannot carry (their sums overflow float32, or a
    // value is not finite) are as they were: each is solved by CG
    int todo[CGD_MAX_FIELDS], n_todo = 0;
    for (int f = 0; f < da.F; ++f)
        if (bad_host[f]) todo[n_todo++] = f;
    cgd_status worst = CGD_OK;
    for (int i = 0; i < n_todo; ++i) {
        DiffuseArgs d1 = da;
        d1.F = 1;
        d1.field = da.field + (size_t)todo[i] * m->cells;
        rc = m->kind == 0 ? diffuse_hex(m, d1, nullptr, s) : diffuse_tet(m, d1, nullptr, s);
        if (rc < 0 && rc != CGD_E_BREAKDOWN) return rc;
        if (rc == CGD_E_BREAKDOWN) {  // (solved as the only field of its call: give its own number)
            std::string e = cgd_last_error();
            const size_t at = e.rfind(", field ");
            if (at != std::string::npos) set_error(e.substr(0, at) + ", field " + std::to_string(todo[i]));
        }
        if (rc == CGD_E_BREAKDOWN || worst == CGD_OK) worst = rc;
    }
    return worst;
}

}  // namespace cgd
