// spx_dipolar.hip -- open-boundary dipolar field by zero-padded FFT
// convolution (Methods, reciprocal-space convolution for long-range dipolar
// fields) on gfx950.
//
// The dipole tensor T(r) = (mu0/4pi) mu_B^2 (3 rhat rhat - 1)/r^3 is sampled
// on a grid of P_a >= 2 L_a - 1 points per axis (P_a a power of two) holding
// every displacement in [-(L_a-1), L_a-1]; its six-component real spectrum is
// built once in FP64 (scaled by mu^2 and by the 1/(Px Py Pz) of the
// unnormalised inverse).  Per evaluation the three spin components go through
// a pruned FP32 transform pipeline that never touches the zero padding:
//   x: R2C of rows of length Px on the Ly x Lz occupied rows only;
//   y: column FFT of length Py reading the Ly occupied rows (the rest are
//      zero by construction), on the Lz occupied planes only;
//   z: column FFT of length Pz reading the Lz occupied planes;
// then the 3x3 spectral product, and the inverse transforms in reverse order
// keeping only the outputs inside the lattice (z < Lz, then y < Ly, then the
// C2R rows and x < Lx).  Linear (aperiodic) convolution = open boundaries.
// Padded extents of 64 to 1024 points: register kernels of radix 8 (two to
// four passes, LDS exchanges between), x rows in pairs as one complex
// transform, and z transform, product and inverse in one pass.  Others: hipFFT
// for the x rows and an LDS radix-2 kernel for the columns (a block stages P
// rows x W adjacent columns, bit-reverses on load, runs log2 P in-place
// butterfly stages), z, product and inverse z as three passes.  Both write
// only the rows that are kept.  The register kernels are bound by HBM; at 256
// points (sc 100^3) the radix-2 ones took 84 - 100 us a column pass, 100 us
// for the product and 71 us for the x rows with hipFFT.
#include <hipfft/hipfft.h>

#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "spx_ext.hpp"

namespace spx {

struct DipolarPlan {
    int L[3];              // x, y, z cells
    int P[3];              // padded extents (powers of two >= 2L - 1)
    int H;                 // Px / 2 + 1 complex points per x row
    int64_t N;             // sites
    int64_t n_cplx;        // Pz * Py * H spectrum points per component
    float *R = nullptr;    // [3][Lz][Ly][Px] real rows (padded spins in, field rows out)
    float2 *X = nullptr;   // [3][Lz][Ly][H] after the x transform
    float2 *Y = nullptr;   // [3][Lz][Py][H] after the y transform
    float2 *Z = nullptr;   // [3][Pz][Py][H] full spectrum (not with the fused z pass)
    float *kern = nullptr; // [6][Pz][Py][H] real dipole spectrum xx, xy, xz, yy, yz, zz
    // own z transform: the spectrum in the fused z pass's order instead,
    // [column group][kz < nkz][6][columns] (nkz = Pz / 2 + 1 with z parity, else Pz)
    float *kernb = nullptr;
    int nkz = 0;
    // the third cell vector is along z and the first two have no z part: the
    // sampled tensor is even (xx, xy, yy, zz) or odd (xz, yz) under dz -> -dz,
    // so is its spectrum under kz -> Pz - kz, and the fused z pass reads only
    // kz <= Pz / 2 (half the spectrum traffic)
    bool zsym = false;
    float2 *tw_y = nullptr, *tw_z = nullptr;  // exp(-2 pi i k / P), k < P
    float2 *tw_x = nullptr;                    // own x transform (k_xfft_fwd, k_xfft_inv)
    hipfftHandle fwd = 0, inv = 0;
    bool fwd_ok = false, inv_ok = false;
};

namespace {

constexpr int kB = 256;
constexpr int kColThreads = 256;
constexpr int kMaxLds = 65536;

// (mu0/4pi) mu_B^2 in meV nm^3 from SI values (CODATA 2018).
double dipole_prefactor() {
    const double mu0_over_4pi = 1.0e-7;      // T m / A
    const double muB_SI = 9.2740100783e-24;  // J / T
    const double meV_in_J = 1.602176634e-22;
    return mu0_over_4pi * muB_SI * muB_SI / meV_in_J * 1.0e27;
}

int next_pow2(int v) {
    int p = 1;
    while (p < v) p <<= 1;
    return p;
}

int log2i(int p) {
    int l = 0;
    while ((1 << l) < p) ++l;
    return l;
}

// columns per block of the column FFT: a power of two <= 16 whose staged tile
// (P x W complex) plus the twiddle table fits the LDS budget
int col_width(int P) {
    int w = 16;
    while (w > 1 && (size_t)P * w * sizeof(float2) + (size_t)(P / 2) * sizeof(float2) > (size_t)kMaxLds) w >>= 1;
    return w;
}

// displacement of padded index k on an axis of L cells and P points, or
// INT_MIN inside the gap between +(L-1) and -(L-1)
__device__ __forceinline__ int pad_disp(int k, int L, int P) {
    if (k < L) return k;
    if (k > P - L) return k - P;
    return -0x7fffffff;
}

// One component (a,b) of the real-space dipole tensor on the padded grid, FP64.
__global__ void k_dipole_component(int Lx, int Ly, int Lz, int Px, int Py, int Pz, double c00, double c01,
                                   double c02, double c10, double c11, double c12, double c20, double c21,
                                   double c22, int ca, int cb, double pref, double *__restrict__ out) {
    const int64_t idx = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (idx >= (int64_t)Px * Py * Pz) return;
    const int kx = (int)(idx % Px), ky = (int)((idx / Px) % Py), kz = (int)(idx / ((int64_t)Px * Py));
    const int ix = pad_disp(kx, Lx, Px), iy = pad_disp(ky, Ly, Py), iz = pad_disp(kz, Lz, Pz);
    double v = 0.0;
    if (ix != -0x7fffffff && iy != -0x7fffffff && iz != -0x7fffffff) {
        const double dx = ix, dy = iy, dz = iz;
        const double r[3] = {dx * c00 + dy * c10 + dz * c20, dx * c01 + dy * c11 + dz * c21,
                             dx * c02 + dy * c12 + dz * c22};
        const double r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
        if (r2 > 0.0) {
            const double rn = sqrt(r2);
            const double inv3 = 1.0 / (r2 * rn);
            v = pref * (3.0 * r[ca] * r[cb] / r2 - (ca == cb ? 1.0 : 0.0)) * inv3;
        }
    }
    out[idx] = v;
}

__global__ void k_take_real(const double2 *__restrict__ in, int64_t n, float *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (i < n) out[i] = (float)in[i].x;
}

// FP32 x rows of the occupied (y, z) lines, zero beyond x = Lx.
// One block per padded x row (c, line = y + Ly z): the occupied Lx values
// converted to FP32, zero up to Px.
__global__ __launch_bounds__(kB) void k_pad_rows(const double *__restrict__ S, int Lx, int Px, int64_t rows,
                                                 int64_t N, float *__restrict__ R) {
    const int64_t row = blockIdx.x;
    const int64_t c = row / rows, line = row - c * rows;
    const double *src = S + c * N + line * Lx;
    float *dst = R + row * Px;
    for (int x = threadIdx.x; x < Px; x += kB) dst[x] = x < Lx ? (float)src[x] : 0.0f;
}

// One block per row: the occupied Lx values of padded row (c, line) into b.
__global__ __launch_bounds__(kB) void k_crop_rows(const float *__restrict__ R, int Lx, int Px, int64_t rows,
                                                  int64_t N, float *__restrict__ b) {
    const int64_t row = blockIdx.x;
    const int64_t c = row / rows, line = row - c * rows;
    const float *src = R + row * Px;
    float *dst = b + c * N + line * Lx;
    for (int x = threadIdx.x; x < Lx; x += kB) dst[x] = src[x];
}

// b^_a = sum_b T^_ab S^_b at every frequency (T^ real symmetric).
__global__ void k_spectral_mult(float2 *__restrict__ spec, const float *__restrict__ kern, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
    if (i >= n) return;
    const float2 sx = spec[i], sy = spec[n + i], sz = spec[2 * n + i];
    const float txx = kern[i], txy = kern[n + i], txz = kern[2 * n + i];
    const float tyy = kern[3 * n + i], tyz = kern[4 * n + i], tzz = kern[5 * n + i];
    spec[i] = make_float2(txx * sx.x + txy * sy.x + txz * sz.x, txx * sx.y + txy * sy.y + txz * sz.y);
    spec[n + i] = make_float2(txy * sx.x + tyy * sy.x + tyz * sz.x, txy * sx.y + tyy * sy.y + tyz * sz.y);
    spec[2 * n + i] = make_float2(txz * sx.x + tyz * sy.x + tzz * sz.x, txz * sx.y + tyz * sy.y + tzz * sz.y);
}

// Column FFT of length P = 2^logP over W adjacent columns of batch
// blockIdx.y.  Element (row r, column j) of a batch sits at
// base + r * J + j; rows r >= nin are zero; only rows r < nout are written.
// INV: exp(+2 pi i ...) (unnormalised).
template <bool INV>
__global__ __launch_bounds__(kColThreads) void k_colfft(const float2 *__restrict__ in, float2 *__restrict__ out,
                                                        int logP, int wl, int nin, int nout, int64_t J,
                                                        int64_t in_bs, int64_t out_bs,
                                                        const float2 *__restrict__ tw) {
    extern __shared__ float2 sm[];
    const int P = 1 << logP, W = 1 << wl;
    float2 *a = sm;
    float2 *twl = sm + (size_t)P * W;
    const int tid = threadIdx.x;
    const int64_t j0 = (int64_t)blockIdx.x * W;
    const int w = (int)((J - j0) < W ? (J - j0) : W);
    const int64_t b = blockIdx.y;
    const float2 *src = in + b * in_bs + j0;
    float2 *dst = out + b * out_bs + j0;
    for (int k = tid; k < P / 2; k += kColThreads) {
        const float2 t = tw[k];
        twl[k] = INV ? make_float2(t.x, -t.y) : t;
    }
    for (int idx = tid; idx < P * W; idx += kColThreads) {
        const int r = idx >> wl, c = idx & (W - 1);
        float2 v = make_float2(0.0f, 0.0f);
        if (r < nin && c < w) v = src[(int64_t)r * J + c];
        const int rr = (int)(__brev((unsigned)r) >> (32 - logP));
        a[(rr << wl) + c] = v;
    }
    __syncthreads();
    const int nbf = (P / 2) * W;
    for (int s = 0; s < logP; ++s) {
        const int half = 1 << s;
        for (int k = tid; k < nbf; k += kColThreads) {
            const int c = k & (W - 1);
            const int bf = k >> wl;
            const int pos = bf & (half - 1);
            const int i = ((bf >> s) << (s + 1)) + pos;
            const float2 t = twl[pos << (logP - s - 1)];
            const float2 u = a[(i << wl) + c];
            const float2 x = a[((i + half) << wl) + c];
            const float2 v = make_float2(x.x * t.x - x.y * t.y, x.x * t.y + x.y * t.x);
            a[(i << wl) + c] = make_float2(u.x + v.x, u.y + v.y);
            a[((i + half) << wl) + c] = make_float2(u.x - v.x, u.y - v.y);
        }
        __syncthreads();
    }
    for (int idx = tid; idx < nout * W; idx += kColThreads) {
        const int r = idx >> wl, c = idx & (W - 1);
        if (c < w) dst[(int64_t)r * J + c] = a[idx];
    }
}

// ---- N-point FFTs in registers, N = 64 .. 1024 ----------------------------
// Stockham's autosort form (T. G. Stockham, 1966): N / 8 threads per column
// with 8 values each, passes of radix 8 and a last one of radix N / 8^k, the
// values exchanged through LDS in between.  With Ns the product of the radices
// done, butterfly j of a pass of radix R takes x[j + r N / R] W^(r (j mod Ns)),
// W = exp(-2 pi i / (Ns R)), and puts its results at (j div Ns) Ns R + j mod
// Ns + r Ns.  Thread t has butterflies t + k N / 8, k < 8 / R, so it always
// reads rows t + m N / 8 (m = k + r 8 / R) and, after the last pass, holds
// rows t + m N / 8 in natural order: what the inverse starts from.
constexpr bool fft_own(int P) { return P >= 64 && P <= 1024; }
// Columns (y, z): a block takes W adjacent columns, consecutive lanes on
// consecutive columns, and exchanges through LDS rows of W values with block
// barriers.  W is 16 (128-byte row segments), 8 for 1024 points (threads) and
// in the fused z pass from 256 points on, so that two blocks share a CU.
// Rows (x): consecutive lanes on consecutive points, so up to 512 points a
// pair of rows is part of one wavefront and needs no barrier (1024 points: two
// wavefronts, barriers).  The same for the columns, staged through LDS to and
// from their wavefronts, was slower (sc 256^3: y 390 against 335 us then, the z
// pass 1116 against 835), as were persistent z blocks that load ahead (971).  At sc
// 100^3 (256 points) the passes take 15 + 25 + 89 + 24 + 13 us.
constexpr int fft_w(int N) { return N <= 512 ? 16 : 8; }
constexpr int fft_zw(int N) { return N <= 128 ? 16 : 8; }
constexpr int fft_xw(int N) { return N <= 256 ? 16 : 8; }  // row pairs per block
// ... where blocks of as many would leave CUs without one: a wavefront's (1024
// points: two wavefronts).  500 x 200 x 1: 96 us a field evaluation, 107 with 38
// full blocks for the rows; 300 x 100 x 1 63 against 74.
constexpr int fft_xfew(int N) { return N <= 512 ? 512 / N : 1; }
// position p of an exchange: one row (value) skipped after every eight, so
// that the steps of 1 and of 8 between the rows that half a wavefront touches
// both fall on different banks
__device__ __forceinline__ int fft_pos(int p) { return p + (p >> 3); }
constexpr int fft_lds(int N, int W) { return N / 8 * 9 * W; }

template <bool INV>
__device__ __forceinline__ float2 cmulw(float2 x, float2 w) {
    // x * w (forward) or x * conj(w) (inverse)
    if (INV) return make_float2(x.x * w.x + x.y * w.y, x.y * w.x - x.x * w.y);
    return make_float2(x.x * w.x - x.y * w.y, x.x * w.y + x.y * w.x);
}

// In-place 8-point DFT, natural order in and out.  HIN: v[4..7] are zero on
// entry (and not read); HOUT: only v[0..3] are wanted.
template <bool INV, bool HIN = false, bool HOUT = false>
__device__ __forceinline__ void dft8(float2 v[8]) {
    const float h = 0.70710678118654752f;
    // two 4-point DFTs of the even and odd samples
    float2 E[4], O[4];
#pragma unroll
    for (int part = 0; part < 2; ++part) {
        const float2 a0 = v[part], a1 = v[part + 2];
        float2 s02 = a0, d02 = a0, s13 = a1, d13 = a1;
        if constexpr (!HIN) {
            const float2 a2 = v[part + 4], a3 = v[part + 6];
            s02 = make_float2(a0.x + a2.x, a0.y + a2.y);
            d02 = make_float2(a0.x - a2.x, a0.y - a2.y);
            s13 = make_float2(a1.x + a3.x, a1.y + a3.y);
            d13 = make_float2(a1.x - a3.x, a1.y - a3.y);
        }
        // W4 d13: -i d13 forward, +i d13 inverse
        const float2 wd = INV ? make_float2(-d13.y, d13.x) : make_float2(d13.y, -d13.x);
        float2 *T = part ? O : E;
        T[0] = make_float2(s02.x + s13.x, s02.y + s13.y);
        T[1] = make_float2(d02.x + wd.x, d02.y + wd.y);
        T[2] = make_float2(s02.x - s13.x, s02.y - s13.y);
        T[3] = make_float2(d02.x - wd.x, d02.y - wd.y);
    }
    // W8^k O[k], k = 0..3
    const float2 o1 = INV ? make_float2(h * (O[1].x - O[1].y), h * (O[1].x + O[1].y))
                          : make_float2(h * (O[1].x + O[1].y), h * (O[1].y - O[1].x));
    const float2 o2 = INV ? make_float2(-O[2].y, O[2].x) : make_float2(O[2].y, -O[2].x);
    const float2 o3 = INV ? make_float2(-h * (O[3].x + O[3].y), h * (O[3].x - O[3].y))
                          : make_float2(h * (O[3].y - O[3].x), -h * (O[3].x + O[3].y));
    const float2 t[4] = {O[0], o1, o2, o3};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k] = make_float2(E[k].x + t[k].x, E[k].y + t[k].y);
        if constexpr (!HOUT) v[k + 4] = make_float2(E[k].x - t[k].x, E[k].y - t[k].y);
    }
}

// radix-R DFTs of the sets {v[k + (8 / R) r], r < R}, k < 8 / R
// (HOUT: v[4..7] are not wanted; the compiler drops what only they need)
template <int R, bool INV, bool HOUT>
__device__ __forceinline__ void dft_sets(float2 v[8]) {
    if constexpr (R == 8) {
        dft8<INV, false, HOUT>(v);
    } else if constexpr (R == 4) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const float2 a0 = v[k], a1 = v[k + 2], a2 = v[k + 4], a3 = v[k + 6];
            const float2 s02 = make_float2(a0.x + a2.x, a0.y + a2.y), d02 = make_float2(a0.x - a2.x, a0.y - a2.y);
            const float2 s13 = make_float2(a1.x + a3.x, a1.y + a3.y), d13 = make_float2(a1.x - a3.x, a1.y - a3.y);
            const float2 wd = INV ? make_float2(-d13.y, d13.x) : make_float2(d13.y, -d13.x);
            v[k] = make_float2(s02.x + s13.x, s02.y + s13.y);
            v[k + 2] = make_float2(d02.x + wd.x, d02.y + wd.y);
            v[k + 4] = make_float2(s02.x - s13.x, s02.y - s13.y);
            v[k + 6] = make_float2(d02.x - wd.x, d02.y - wd.y);
        }
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float2 a = v[k], b = v[k + 4];
            v[k] = make_float2(a.x + b.x, a.y + b.y);
            v[k + 4] = make_float2(a.x - b.x, a.y - b.y);
        }
    }
}

// How an FFT's threads wait for each other's LDS accesses.
enum { SYNC_WAVE = 0, SYNC_BLOCK = 1 };
template <int SYNC>
__device__ __forceinline__ void fft_sync() {
    if constexpr (SYNC == SYNC_WAVE) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    } else {
        __syncthreads();
    }
}

// Twiddles of a pass (product Ns of the radices before it) for thread t's rows.
template <int N, int Ns>
__device__ __forceinline__ void fft_twiddles(float2 w[8], int t, const float2 *__restrict__ tw) {
    constexpr int R = N / Ns < 8 ? N / Ns : 8;
#pragma unroll
    for (int k = 0; k < 8 / R; ++k) {
        const int a = (t + k * (N / 8)) % Ns * (N / (Ns * R));
#pragma unroll
        for (int r = 1; r < R; ++r) w[k + (8 / R) * r] = tw[a * r];
    }
}

// One exchange and the pass after it: the results of the pass of radix RP
// (product NSP before it) are put in order in LDS (buf[fft_pos(p) W], buf at
// the column's slot) and thread t's rows of the next pass read back,
// multiplied by their twiddles and transformed.  TWO: consecutive exchanges
// take two buffers in turn, and one barrier each suffices, since a buffer is
// written again only after the barrier that followed its last read; with one
// buffer a second barrier precedes the write.  AHEAD: the twiddles are loaded
// before the barriers instead of after them.
template <int N, int NSP, int RP, bool INV, int SYNC, bool TWO, int W, bool AHEAD>
__device__ __forceinline__ void fft_pass(float2 v[8], float2 *buf, int t, const float2 *__restrict__ tw) {
    constexpr int Ns = NSP * RP, R = N / Ns < 8 ? N / Ns : 8;
    static_assert(RP == 8, "only the last pass has a smaller radix");
    float2 w[8];
    if constexpr (AHEAD) fft_twiddles<N, Ns>(w, t, tw);
    if (!TWO) fft_sync<SYNC>();
    const int o = fft_pos((t / NSP) * Ns + t % NSP);
#pragma unroll
    for (int r = 0; r < RP; ++r) buf[(o + r * NSP / 8 * 9 + (NSP < 8 ? r : 0)) * W] = v[r];  // fft_pos of + r NSP
    fft_sync<SYNC>();
#pragma unroll
    for (int m = 0; m < 8; ++m) v[m] = buf[(fft_pos(t) + m * (N / 64 * 9)) * W];
    if constexpr (!AHEAD) fft_twiddles<N, Ns>(w, t, tw);
#pragma unroll
    for (int k = 0; k < 8 / R; ++k)
#pragma unroll
        for (int r = 1; r < R; ++r) v[k + (8 / R) * r] = cmulw<INV>(v[k + (8 / R) * r], w[k + (8 / R) * r]);
    dft_sets<R, INV, INV && Ns * R == N>(v);
}

// N-point FFT of a column: v[m] = row t + (N / 8) m on entry and exit.  A
// padded extent is at least twice the lattice's, so the forward transform's
// rows from N / 2 on (v[4..7]) are zero, and with HIN not read; the inverse
// leaves v[4..7] undefined: those rows are cropped.  X: exchanges done so far
// in the two buffers A and B (which one comes next).
template <int N, bool INV, int SYNC, bool TWO, int W, int X = 0, bool HIN = !INV, bool AHEAD = false>
__device__ __forceinline__ void fft_col(float2 v[8], float2 *A, float2 *B, int t, const float2 *__restrict__ tw) {
    float2 *const b0 = (X & 1) ? B : A, *const b1 = (X & 1) ? A : B;
    dft8<INV, HIN>(v);
    fft_pass<N, 1, 8, INV, SYNC, TWO, W, AHEAD>(v, b0, t, tw);
    if constexpr (N > 64) fft_pass<N, 8, 8, INV, SYNC, TWO, W, AHEAD>(v, b1, t, tw);
    if constexpr (N > 512) fft_pass<N, 64, 8, INV, SYNC, TWO, W, AHEAD>(v, b0, t, tw);
}
constexpr int fft_exchanges(int N) { return N > 512 ? 3 : N > 64 ? 2 : 1; }

// Blocks renumbered so that each XCD takes one contiguous range of them
// (workgroups are dealt to the 8 XCDs in turn): lines that straddle
// neighbouring column groups then meet in one L2.
__device__ __forceinline__ int64_t xcd_range(int64_t id, int64_t T) {
    const int64_t q = T / 8, r = T % 8, k = id % 8;
    return k * q + (k < r ? k : r) + id / 8;
}

template <int N, bool INV>
__global__ __launch_bounds__(N / 8 * fft_w(N)) void k_colfft_reg(const float2 *__restrict__ in,
                                                                 float2 *__restrict__ out, int nin, int nout,
                                                                 int64_t J, int64_t in_bs, int64_t out_bs,
                                                                 const float2 *__restrict__ tw) {
    constexpr int W = fft_w(N), T = N / 8;
    // 512 points: twiddles ahead of the barriers (inverse, sc 256^3: 325 -> 297
    // us; the fused z pass 809 -> 858) and the forward transform's first
    // butterflies over all eight rows, zeros included (334 -> 311).  Other
    // extents are the same or slower with either.
    constexpr bool HIN = !INV && N != 512, AHEAD = N == 512;
    __shared__ float2 lds[fft_lds(N, W)];
    const int w = threadIdx.x % W, t = threadIdx.x / W;  // column in the tile, thread of the column
    const int64_t vb = xcd_range(blockIdx.x + (int64_t)gridDim.x * blockIdx.y, (int64_t)gridDim.x * gridDim.y);
    const int64_t bx = vb % gridDim.x, b = vb / gridDim.x;
    const int64_t j = bx * W + w;
    const bool col = j < J;
    const float2 *src = in + b * in_bs + j;
    float2 *dst = out + b * out_bs + j;
    float2 v[8];
#pragma unroll
    for (int m = 0; m < (HIN ? 4 : 8); ++m) {
        const int r = t + m * T;
        v[m] = (col && r < nin) ? src[(int64_t)r * J] : make_float2(0.0f, 0.0f);
    }
    fft_col<N, INV, SYNC_BLOCK, false, W, 0, HIN, AHEAD>(v, lds + w, lds + w, t, tw);
    if (col) {
#pragma unroll
        for (int m = 0; m < (INV ? 4 : 8); ++m) {
            const int r = t + m * T;
            if (r < nout) dst[(int64_t)r * J] = v[m];
        }
    }
}

// x rows: two real rows (A, B) of one pair transformed as one complex N-point
// FFT z = a + i b, whose spectrum Z gives both halves, A[k] = (Z[k] + conj
// Z[N - k]) / 2 and B[k] = (Z[k] - conj Z[N - k]) / 2i for k <= N / 2.  A pair's
// threads are consecutive lanes and its rows contiguous, so they load and
// store directly.  Row r = (c, line) of the pair index holds spins S[r Lx + x]
// (x < Lx, zero to N) and spectrum X[r H + k] (H = N / 2 + 1).
template <int N, int W>
__global__ __launch_bounds__(N / 8 * W) void k_xfft_fwd(const double *__restrict__ S, float2 *__restrict__ X, int Lx,
                                                        int64_t nrows, const float2 *__restrict__ tw) {
    constexpr int T = N / 8, H = N / 2 + 1, RUN = fft_lds(N, 1) + 4;
    constexpr int SYNC = N <= 512 ? SYNC_WAVE : SYNC_BLOCK;
    __shared__ float2 lds[W * RUN];
    const int t = threadIdx.x % T;
    float2 *const run = lds + threadIdx.x / T * RUN;
    const int64_t ra = 2 * ((int64_t)blockIdx.x * W + threadIdx.x / T), rb = ra + 1;
    float2 v[8];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const int n = t + m * T;
        v[m] = make_float2((n < Lx && ra < nrows) ? (float)S[ra * Lx + n] : 0.0f,
                           (n < Lx && rb < nrows) ? (float)S[rb * Lx + n] : 0.0f);
    }
    fft_col<N, false, SYNC, false, 1>(v, run, run, t, tw);
    fft_sync<SYNC>();
#pragma unroll
    for (int m = 0; m < 8; ++m) run[t + m * T] = v[m];
    fft_sync<SYNC>();
#pragma unroll
    for (int m = 0; m < 5; ++m) {
        const int k = t + T * m;
        if (k > N / 2) break;
        const float2 zk = m < 4 ? v[m] : run[k], zm = run[(N - k) & (N - 1)];
        if (ra < nrows) X[ra * H + k] = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y - zm.y));
        if (rb < nrows) X[rb * H + k] = make_float2(0.5f * (zk.y + zm.y), 0.5f * (zm.x - zk.x));
    }
}

// The inverse: Z[n] = A[n] + i B[n] over all N bins from the stored half
// (A[N - k] = conj A[k]; the imaginary parts of bins 0 and N / 2 dropped, as
// for a real inverse transform), one unnormalised inverse FFT, and rows
// x < Lx of z = a + i b written to the field.
template <int N, int W>
__global__ __launch_bounds__(N / 8 * W) void k_xfft_inv(const float2 *__restrict__ X, float *__restrict__ b, int Lx,
                                                        int64_t nrows, const float2 *__restrict__ tw) {
    constexpr int T = N / 8, H = N / 2 + 1, RUN = fft_lds(N, 1) + 4;
    constexpr int SYNC = N <= 512 ? SYNC_WAVE : SYNC_BLOCK;
    __shared__ float2 lds[W * RUN];
    const int t = threadIdx.x % T;
    const int64_t ra = 2 * ((int64_t)blockIdx.x * W + threadIdx.x / T), rb = ra + 1;
    float2 v[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        const int n = t + m * T;
        const int k = n <= N / 2 ? n : N - n;
        float2 A = ra < nrows ? X[ra * H + k] : make_float2(0.0f, 0.0f);
        float2 B = rb < nrows ? X[rb * H + k] : make_float2(0.0f, 0.0f);
        if (k == 0 || k == N / 2) {
            A.y = 0.0f;
            B.y = 0.0f;
        } else if (n > N / 2) {
            A.y = -A.y;
            B.y = -B.y;
        }
        v[m] = make_float2(A.x - B.y, A.y + B.x);
    }
    float2 *const run = lds + threadIdx.x / T * RUN;
    fft_col<N, true, SYNC, false, 1>(v, run, run, t, tw);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const int n = t + m * T;
        if (n >= Lx) break;
        if (ra < nrows) b[ra * Lx + n] = v[m].x;
        if (rb < nrows) b[rb * Lx + n] = v[m].y;
    }
}

// The dipole spectrum reordered for the fused z pass: block g of W columns
// reads kernb[g][kz][c][0..W-1] for its kz, one contiguous run per kz.
__global__ void k_kern_block(const float *__restrict__ kern, float *__restrict__ kernb, int64_t J, int64_t n_cplx,
                             int nkz, int W, int64_t total) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= total) return;
    const int w = (int)(q % W);
    int64_t r = q / W;
    const int c = (int)(r % 6);
    r /= 6;
    const int kz = (int)(r % nkz);
    const int64_t g = r / nkz;
    const int64_t j = g * W + w;
    kernb[q] = j < J ? kern[c * n_cplx + (int64_t)kz * J + j] : 0.0f;
}

// z transform, spectral product and inverse z transform fused: each block
// takes W (y, kx) columns of the three components (rows z < Lz of Y, zero
// above), transforms them forward, multiplies by the dipole spectrum at its N
// kz and transforms back, writing rows z < Lz in place.  HBM (2.42 GB at sc
// 256^3, 510 us at the rate of a copy), the vector ALU (390 us) and LDS (200
// us) are of a size and overlap in part.
template <int N>
__global__ __launch_bounds__(N / 8 * fft_zw(N)) void k_zconv(float2 *__restrict__ Y, const float *__restrict__ kernb,
                                                             int Lz, int64_t J, int nkz,
                                                             const float2 *__restrict__ tw, int zsym) {
    constexpr int W = fft_zw(N), T = N / 8, E = fft_exchanges(N);
    constexpr bool TWO = N <= 512;  // two buffers fit the CU's LDS
    __shared__ float2 lds[(TWO ? 2 : 1) * fft_lds(N, W)];
    const int w = threadIdx.x % W, t = threadIdx.x / W;
    float2 *const A = lds + w, *const B = A + (TWO ? fft_lds(N, W) : 0);
    const int64_t blk = xcd_range(blockIdx.x, gridDim.x);
    const int64_t j = blk * W + w;
    const bool col = j < J;
    const int64_t cs = (int64_t)Lz * J;
    // all three components' loads in flight before the first transform
    float2 v[3][8];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int r = t + m * T;
            v[c][m] = (col && r < Lz) ? Y[c * cs + (int64_t)r * J + j] : make_float2(0.0f, 0.0f);
        }
    // the thread's index hidden from each transform: their twiddles and
    // addresses are equal, and held over all six they spill
    auto hid = [](int x) __attribute__((always_inline)) {
        asm volatile("" : "+v"(x));
        return x;
    };
    fft_col<N, false, SYNC_BLOCK, TWO, W, 0>(v[0], A, B, hid(t), tw);
    fft_col<N, false, SYNC_BLOCK, TWO, W, E>(v[1], A, B, hid(t), tw);
    fft_col<N, false, SYNC_BLOCK, TWO, W, 2 * E>(v[2], A, B, hid(t), tw);
    if (col) {
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            // kz and N - kz read the same stored entries (sign flip for xz, yz)
            const int kz = t + m * T;
            const bool mirror = zsym && kz > N / 2;
            const float sgn = mirror ? -1.0f : 1.0f;
            const float *kb = kernb + ((blk * nkz + (mirror ? N - kz : kz)) * 6) * W + w;
            const float txx = kb[0], txy = kb[W], txz = sgn * kb[2 * W];
            const float tyy = kb[3 * W], tyz = sgn * kb[4 * W], tzz = kb[5 * W];
            const float2 sx = v[0][m], sy = v[1][m], sz = v[2][m];
            v[0][m] = make_float2(txx * sx.x + txy * sy.x + txz * sz.x, txx * sx.y + txy * sy.y + txz * sz.y);
            v[1][m] = make_float2(txy * sx.x + tyy * sy.x + tyz * sz.x, txy * sx.y + tyy * sy.y + tyz * sz.y);
            v[2][m] = make_float2(txz * sx.x + tyz * sy.x + tzz * sz.x, txz * sx.y + tyz * sy.y + tzz * sz.y);
        }
    }
    auto store = [&](int c) __attribute__((always_inline)) {
        if (!col) return;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int r = t + m * T;
            if (r < Lz) Y[c * cs + (int64_t)r * J + j] = v[c][m];
        }
    };
    fft_col<N, true, SYNC_BLOCK, TWO, W, 3 * E>(v[0], A, B, hid(t), tw);
    store(0);
    fft_col<N, true, SYNC_BLOCK, TWO, W, 4 * E>(v[1], A, B, hid(t), tw);
    store(1);
    fft_col<N, true, SYNC_BLOCK, TWO, W, 5 * E>(v[2], A, B, hid(t), tw);
    store(2);
}

// f(std::integral_constant<int, P>) for a padded extent with own transforms
template <typename F>
hipError_t with_points(int P, F &&f) {
    switch (P) {
    case 64: f(std::integral_constant<int, 64>{}); break;
    case 128: f(std::integral_constant<int, 128>{}); break;
    case 256: f(std::integral_constant<int, 256>{}); break;
    case 512: f(std::integral_constant<int, 512>{}); break;
    case 1024: f(std::integral_constant<int, 1024>{}); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

unsigned nblocks(int64_t n) { return (unsigned)((n + kB - 1) / kB); }

spx_status fft_fail(hipfftResult r, const char *where) {
    return set_error(SPX_ERR_FFT, std::string(where) + ": hipFFT error " + std::to_string((int)r));
}

template <bool INV>
hipError_t colfft(const float2 *in, float2 *out, int P, int nin, int nout, int64_t J, int64_t nbatch, int64_t in_bs,
                  int64_t out_bs, const float2 *tw, hipStream_t st) {
    if (fft_own(P))
        return with_points(P, [&](auto n) {
            constexpr int N = decltype(n)::value;
            dim3 grid((unsigned)((J + fft_w(N) - 1) / fft_w(N)), (unsigned)nbatch);
            k_colfft_reg<N, INV><<<grid, N / 8 * fft_w(N), 0, st>>>(in, out, nin, nout, J, in_bs, out_bs, tw);
        });
    const int W = col_width(P);  // P >= 2 (padded extents are at least 2)
    const size_t smem = ((size_t)P * W + P / 2) * sizeof(float2);
    dim3 grid((unsigned)((J + W - 1) / W), (unsigned)nbatch);
    k_colfft<INV><<<grid, kColThreads, smem, st>>>(in, out, log2i(P), log2i(W), nin, nout, J, in_bs, out_bs, tw);
    return hipGetLastError();
}

}  // namespace

void destroy_dipolar(DipolarPlan *p) {
    if (!p) return;
    if (p->fwd_ok) hipfftDestroy(p->fwd);
    if (p->inv_ok) hipfftDestroy(p->inv);
    for (void *q : {(void *)p->R, (void *)p->X, (void *)p->Y, (void *)p->Z, (void *)p->kern, (void *)p->kernb, (void *)p->tw_y,
                    (void *)p->tw_z, (void *)p->tw_x})
        if (q) (void)hipFree(q);
    delete p;
}

spx_status create_dipolar(const int32_t dims[3], const double cell[9], double mu, hipStream_t st,
                          DipolarPlan **out, int64_t *ws_bytes) {
    for (int k = 0; k < 3; ++k)
        if (dims[k] < 1 || dims[k] > 2048)
            return set_error(SPX_ERR_UNSUPPORTED, "dipolar FFT path: extents must be 1 .. 2048 per axis");
    DipolarPlan *p = new DipolarPlan();
    for (int k = 0; k < 3; ++k) {
        p->L[k] = dims[k];
        p->P[k] = next_pow2(2 * dims[k] - 1 < 2 ? 2 : 2 * dims[k] - 1);
    }
    const int Lx = p->L[0], Ly = p->L[1], Lz = p->L[2], Px = p->P[0], Py = p->P[1], Pz = p->P[2];
    p->H = Px / 2 + 1;
    p->N = (int64_t)Lx * Ly * Lz;
    p->n_cplx = (int64_t)Pz * Py * p->H;
    const int64_t rows = (int64_t)Ly * Lz;
    auto alloc = [&](void **ptr, size_t bytes, const char *what) -> spx_status {
        if (hipMalloc(ptr, bytes) != hipSuccess) {
            (void)hipGetLastError();
            *ptr = nullptr;
            return set_error(SPX_ERR_OUT_OF_MEMORY, std::string("hipMalloc failed for ") + what);
        }
        *ws_bytes += (int64_t)bytes;
        return SPX_OK;
    };
    spx_status s;
    if ((!fft_own(Px) && (s = alloc((void **)&p->R, sizeof(float) * 3 * rows * Px, "dipolar rows")) != SPX_OK) ||
        (fft_own(Px) && (s = alloc((void **)&p->tw_x, sizeof(float2) * Px, "dipolar twiddles")) != SPX_OK) ||
        (s = alloc((void **)&p->X, sizeof(float2) * 3 * rows * p->H, "dipolar x spectra")) != SPX_OK ||
        (s = alloc((void **)&p->Y, sizeof(float2) * 3 * (int64_t)Lz * Py * p->H, "dipolar xy spectra")) != SPX_OK ||
        (!fft_own(Pz) && (s = alloc((void **)&p->Z, sizeof(float2) * 3 * p->n_cplx, "dipolar spectra")) != SPX_OK) ||
        (s = alloc((void **)&p->kern, sizeof(float) * 6 * p->n_cplx, "dipole spectrum")) != SPX_OK ||
        (s = alloc((void **)&p->tw_y, sizeof(float2) * Py, "dipolar twiddles")) != SPX_OK ||
        (s = alloc((void **)&p->tw_z, sizeof(float2) * Pz, "dipolar twiddles")) != SPX_OK) {
        destroy_dipolar(p);
        return s;
    }
    // twiddle tables exp(-2 pi i k / P), k < P, from FP64
    std::vector<float2> ty(Py), tz(Pz);
    for (int k = 0; k < Py; ++k)
        ty[k] = make_float2((float)std::cos(2.0 * M_PI * k / Py), (float)(-std::sin(2.0 * M_PI * k / Py)));
    for (int k = 0; k < Pz; ++k)
        tz[k] = make_float2((float)std::cos(2.0 * M_PI * k / Pz), (float)(-std::sin(2.0 * M_PI * k / Pz)));
    hipError_t e = hipMemcpyAsync(p->tw_y, ty.data(), sizeof(float2) * ty.size(), hipMemcpyHostToDevice, st);
    if (e == hipSuccess)
        e = hipMemcpyAsync(p->tw_z, tz.data(), sizeof(float2) * tz.size(), hipMemcpyHostToDevice, st);
    std::vector<float2> tx(fft_own(Px) ? Px : 0);
    for (size_t k = 0; k < tx.size(); ++k)
        tx[k] = make_float2((float)std::cos(2.0 * M_PI * k / Px), (float)(-std::sin(2.0 * M_PI * k / Px)));
    if (e == hipSuccess && !tx.empty())
        e = hipMemcpyAsync(p->tw_x, tx.data(), sizeof(float2) * tx.size(), hipMemcpyHostToDevice, st);
    // kernel spectrum, one tensor component at a time in FP64
    const int64_t n_real = (int64_t)Px * Py * Pz;
    double *treal = nullptr;
    double2 *tcplx = nullptr;
    if ((s = alloc((void **)&treal, sizeof(double) * n_real, "dipole tensor (setup)")) != SPX_OK) {
        destroy_dipolar(p);
        return s;
    }
    if ((s = alloc((void **)&tcplx, sizeof(double2) * p->n_cplx, "dipole tensor spectrum (setup)")) != SPX_OK) {
        (void)hipFree(treal);
        destroy_dipolar(p);
        return s;
    }
    *ws_bytes -= (int64_t)(sizeof(double) * n_real + sizeof(double2) * p->n_cplx);
    hipfftHandle dplan;
    hipfftResult fr = hipfftPlan3d(&dplan, Pz, Py, Px, HIPFFT_D2Z);
    if (fr != HIPFFT_SUCCESS) {
        (void)hipFree(treal);
        (void)hipFree(tcplx);
        destroy_dipolar(p);
        return fft_fail(fr, "dipolar setup plan");
    }
    hipfftSetStream(dplan, st);
    const double pref = dipole_prefactor() * mu * mu / (double)n_real;
    const int comps[6][2] = {{0, 0}, {0, 1}, {0, 2}, {1, 1}, {1, 2}, {2, 2}};
    // z parity of the sampled tensor: no coupling of the z axis with x, y in the
    // cell matrix (either storage order)
    p->zsym = cell[2] == 0.0 && cell[5] == 0.0 && cell[6] == 0.0 && cell[7] == 0.0;
    for (int c = 0; c < 6 && s == SPX_OK && e == hipSuccess; ++c) {
        k_dipole_component<<<nblocks(n_real), kB, 0, st>>>(Lx, Ly, Lz, Px, Py, Pz, cell[0], cell[1], cell[2], cell[3],
                                                            cell[4], cell[5], cell[6], cell[7], cell[8], comps[c][0],
                                                            comps[c][1], pref, treal);
        fr = hipfftExecD2Z(dplan, treal, (hipfftDoubleComplex *)tcplx);
        if (fr != HIPFFT_SUCCESS) { s = fft_fail(fr, "dipolar setup transform"); break; }
        k_take_real<<<nblocks(p->n_cplx), kB, 0, st>>>(tcplx, p->n_cplx, p->kern + c * p->n_cplx);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    hipfftDestroy(dplan);
    (void)hipFree(treal);
    (void)hipFree(tcplx);
    if (s == SPX_OK && e != hipSuccess) s = set_hip_error(e, "dipolar setup");
    if (s != SPX_OK) {
        destroy_dipolar(p);
        return s;
    }
    if (fft_own(Pz)) {
        // the fused z pass's order; the [6][Pz][Py][H] spectrum is then no
        // longer needed
        const int W = fft_zw(Pz);
        const int64_t plane = (int64_t)Py * p->H, ngroup = (plane + W - 1) / W;
        p->nkz = p->zsym ? Pz / 2 + 1 : Pz;
        const int64_t total = ngroup * p->nkz * 6 * W;
        if ((s = alloc((void **)&p->kernb, sizeof(float) * total, "dipole spectrum (z pass order)")) != SPX_OK) {
            destroy_dipolar(p);
            return s;
        }
        k_kern_block<<<nblocks(total), kB, 0, st>>>(p->kern, p->kernb, plane, p->n_cplx, p->nkz, W, total);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) {
            destroy_dipolar(p);
            return set_hip_error(e, "dipolar spectrum reorder");
        }
        (void)hipFree(p->kern);
        p->kern = nullptr;
        *ws_bytes -= (int64_t)(sizeof(float) * 6 * p->n_cplx);
    }
    if (fft_own(Px)) {  // the x rows run in k_xfft_fwd / k_xfft_inv
        *out = p;
        return SPX_OK;
    }
    // batched FP32 x-row transforms of the occupied lines of the three components
    int n[1] = {Px};
    int rembed[1] = {Px}, cembed[1] = {p->H};
    const int batch = (int)(3 * rows);
    fr = hipfftPlanMany(&p->fwd, 1, n, rembed, 1, Px, cembed, 1, p->H, HIPFFT_R2C, batch);
    if (fr != HIPFFT_SUCCESS) {
        destroy_dipolar(p);
        return fft_fail(fr, "dipolar R2C plan");
    }
    p->fwd_ok = true;
    fr = hipfftPlanMany(&p->inv, 1, n, cembed, 1, p->H, rembed, 1, Px, HIPFFT_C2R, batch);
    if (fr != HIPFFT_SUCCESS) {
        destroy_dipolar(p);
        return fft_fail(fr, "dipolar C2R plan");
    }
    p->inv_ok = true;
    *out = p;
    return SPX_OK;
}

spx_status eval_dipolar(DipolarPlan *p, const double *S, float *bdip, hipStream_t st) {
    if (!p) return set_error(SPX_ERR_INVALID_ARG, "dipolar path not set up");
    const int Lx = p->L[0], Ly = p->L[1], Lz = p->L[2], Px = p->P[0], Py = p->P[1], Pz = p->P[2], H = p->H;
    const int64_t rows = (int64_t)Ly * Lz;
    hipError_t e;
    // x rows in pairs, one pair per column slot
    auto few_rows = [&](int W) { return (3 * rows + 1) / 2 < (int64_t)W * device_cus(); };
    auto xgrid = [&](int W) { return (unsigned)(((3 * rows + 1) / 2 + W - 1) / W); };
    if (fft_own(Px)) {
        e = with_points(Px, [&](auto n) {
            constexpr int N = decltype(n)::value;
            constexpr int W = fft_xw(N), F = fft_xfew(N);
            if (few_rows(W)) k_xfft_fwd<N, F><<<xgrid(F), N / 8 * F, 0, st>>>(S, p->X, Lx, 3 * rows, p->tw_x);
            else k_xfft_fwd<N, W><<<xgrid(W), N / 8 * W, 0, st>>>(S, p->X, Lx, 3 * rows, p->tw_x);
        });
        if (e != hipSuccess) return set_hip_error(e, "dipolar x rows");
    } else {
        k_pad_rows<<<(unsigned)(3 * rows), kB, 0, st>>>(S, Lx, Px, rows, p->N, p->R);
        e = hipGetLastError();
        if (e != hipSuccess) return set_hip_error(e, "dipolar pad");
        hipfftSetStream(p->fwd, st);
        hipfftResult fr = hipfftExecR2C(p->fwd, p->R, (hipfftComplex *)p->X);
        if (fr != HIPFFT_SUCCESS) return fft_fail(fr, "dipolar R2C");
    }
    const int64_t plane = (int64_t)Py * H;
    // y: X [3 Lz][Ly rows][H] -> Y [3 Lz][Py][H]
    e = colfft<false>(p->X, p->Y, Py, Ly, Py, H, 3 * (int64_t)Lz, (int64_t)Ly * H, plane, p->tw_y, st);
    if (fft_own(Pz)) {
        // z transform, product and inverse z transform in one pass over Y
        if (e == hipSuccess)
            e = with_points(Pz, [&](auto n) {
                constexpr int N = decltype(n)::value;
                k_zconv<N><<<(unsigned)((plane + fft_zw(N) - 1) / fft_zw(N)), N / 8 * fft_zw(N), 0, st>>>(
                    p->Y, p->kernb, Lz, plane, p->nkz, p->tw_z, p->zsym ? 1 : 0);
            });
    } else {
        // z: Y [3][Lz planes][Py H] -> Z [3][Pz][Py H]
        if (e == hipSuccess)
            e = colfft<false>(p->Y, p->Z, Pz, Lz, Pz, plane, 3, (int64_t)Lz * plane, p->n_cplx, p->tw_z, st);
        if (e == hipSuccess) {
            k_spectral_mult<<<nblocks(p->n_cplx), kB, 0, st>>>(p->Z, p->kern, p->n_cplx);
            e = hipGetLastError();
        }
        // inverse z keeps planes z < Lz
        if (e == hipSuccess)
            e = colfft<true>(p->Z, p->Y, Pz, Pz, Lz, plane, 3, p->n_cplx, (int64_t)Lz * plane, p->tw_z, st);
    }
    // inverse y keeps rows y < Ly
    if (e == hipSuccess)
        e = colfft<true>(p->Y, p->X, Py, Py, Ly, H, 3 * (int64_t)Lz, plane, (int64_t)Ly * H, p->tw_y, st);
    if (e != hipSuccess) return set_hip_error(e, "dipolar column transforms");
    if (fft_own(Px)) {
        e = with_points(Px, [&](auto n) {
            constexpr int N = decltype(n)::value;
            constexpr int W = fft_xw(N), F = fft_xfew(N);
            if (few_rows(W)) k_xfft_inv<N, F><<<xgrid(F), N / 8 * F, 0, st>>>(p->X, bdip, Lx, 3 * rows, p->tw_x);
            else k_xfft_inv<N, W><<<xgrid(W), N / 8 * W, 0, st>>>(p->X, bdip, Lx, 3 * rows, p->tw_x);
        });
        if (e != hipSuccess) return set_hip_error(e, "dipolar x rows");
        return SPX_OK;
    }
    hipfftSetStream(p->inv, st);
    hipfftResult fr = hipfftExecC2R(p->inv, (hipfftComplex *)p->X, p->R);
    if (fr != HIPFFT_SUCCESS) return fft_fail(fr, "dipolar C2R");
    k_crop_rows<<<(unsigned)(3 * rows), kB, 0, st>>>(p->R, Lx, Px, rows, p->N, bdip);
    e = hipGetLastError();
    if (e != hipSuccess) return set_hip_error(e, "dipolar crop");
    return SPX_OK;
}

}  // namespace spx
