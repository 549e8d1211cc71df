// Spectral post-processing of a detector (Sec. 4: the detector data Fourier
// transformed with respect to time, compared there with Eq. 7 and Eq. 8).
//
// A slot holds the field averaged over the slot, so the transform of the
// piecewise-constant signal at omega is
//     F(omega) = sum_j E_j e^{-i omega j dt} (e^{-i omega dt} - 1) / (-i omega)
// and, with R the cell's distance from the origin,
//     d2I/domega dOmega = c R^2 / (4 pi^2) |F(omega)|^2
//     dI/domega         = sum over cells of weight_c d2I/domega dOmega
//     dI/dOmega         = c R^2 / (4 pi) sum_j |E_j|^2 dt          (Parseval)
// at omega_m = 2 pi m / (N dt), m = 0 .. N/2, the signal zero beyond its
// n_t slots (N a power of two >= n_t).
//
// Each cell gives two complex signals of length N (zero padded): Z1 = Ex + i Ey
// and Z2 = Ez + 0i.  The power of the three real components at omega_m is
// (Q(m) + Q(N - m)) / 2 with Q(m) = |Z1(m)|^2 + |Z2(m)|^2.  Kernels, per group
// of cells that fits the workspace:
//   spec_cols_kernel   (N = N1 * N2, N1 and N2 <= kFftTile) the first of the
//                      two steps of the four-step FFT: with n = N2 n1 + n2,
//                      tiles of columns (fixed n2, n1 = 0 .. N1 - 1) are read
//                      from the detector, transformed in LDS, multiplied by
//                      exp(-2 pi i n2 k1 / N) and stored at N2 k1 + n2;
//                      spec_cols2_kernel does the same for both signals of a
//                      cell in one tile, so that each slot is read once;
//   spec_rows_kernel   the second step: tiles of rows (fixed k1, contiguous)
//                      transformed in LDS and stored at k1 + N1 k2, the
//                      spectrum in natural order; spec_rows_q32_kernel
//                      transforms the rows of both signals of a cell together
//                      and stores only Q, row-major (8 bytes a frequency
//                      instead of 32);
//   spec_small_kernel  for N <= 2 kFftTile: all of it in one pass, cell by cell;
//   spec_load_kernel + spec_fft_pass   for N > kFftTile^2: packing, then
//                      log2(N) radix-2 Stockham passes between two buffers;
//   spec_power_kernel  a thread per frequency and block of cells: the power
//                      from Z1 and Z2 at m and N - m, scaled to d2I, and the
//                      weighted sum over its cells added to dI/domega
//                      (atomically); spec_power_t_kernel does the same from
//                      the row-major Q, transposing tiles through LDS;
// and spec_parseval_kernel, one workgroup per cell, for dI/dOmega.
#include <algorithm>

#include "radio_internal.h"

namespace radio {

namespace {

constexpr double kPi = 3.14159265358979323846;
constexpr int kFftTileLg = 11;
constexpr int kFftTile = 1 << kFftTileLg;  // complex values transformed per workgroup in LDS
constexpr int kFftThreads = 256;

// value n (< N) of signal s (2 g: Ex + i Ey of cell r0 + g; 2 g + 1: Ez) of the
// detector's accumulator; zero past its n_t slots
template <bool PAIRS>
__device__ __forceinline__ double2 signal_at(const double* __restrict__ acc, int64_t n_t,
                                             int64_t r0, int64_t s, int64_t n)
{
    if (n >= n_t)
        return make_double2(0.0, 0.0);
    const int64_t i = (r0 + (s >> 1)) * n_t + n;
    double e[3];
    if (PAIRS) {
        const float* q = reinterpret_cast<const float*>(acc) + i * 12;
#pragma unroll
        for (int k = 0; k < 3; ++k)
            e[k] = (double)q[k] + (double)q[6 + k];
    } else {
#pragma unroll
        for (int k = 0; k < 3; ++k)
            e[k] = acc[i * 6 + k];
    }
    return (s & 1) ? make_double2(e[2], 0.0) : make_double2(e[0], e[1]);
}

__device__ __forceinline__ double2 cmul(double2 a, double2 b)
{
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// Twiddle tables of a transform of N = 2^lg (lg <= 2 kFftTileLg), written by
// spec_tables_kernel into kSpecTableValues complex values:
//   tab[k]          = exp(-2 pi i k / kFftTile), k < kFftTile / 2: an LDS
//                     transform of length len <= kFftTile takes every
//                     (kFftTile / len)-th entry;
//   tab[kTabLo + b] = exp(-2 pi i b / N), b < S = 2^ceil(lg / 2);
//   tab[kTabHi + a] = exp(-2 pi i a S / N), a < N / S;
// so that exp(-2 pi i r / N) = tab[kTabHi + r / S] tab[kTabLo + r mod S].
constexpr int kTabLo = kFftTile / 2;
constexpr int kTabHi = kTabLo + kFftTile;
static_assert(kTabHi + kFftTile <= kSpecTableValues, "twiddle table layout");
static_assert(kSpecOneLaunch == 2 * kFftTile, "spec_small_kernel's lengths");

__global__ __launch_bounds__(256) void spec_tables_kernel(double2* __restrict__ tab, int lg)
{
    const int lgS = (lg + 1) / 2;
    const int64_t N = (int64_t)1 << lg;
    const int S = 1 << lgS;
    const int A = (int)(N >> lgS);
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < (int)kSpecTableValues;
         i += gridDim.x * blockDim.x) {
        double x;  // the angle in units of -2 pi
        if (i < kTabLo)
            x = (double)i / (double)kFftTile;
        else if (i < kTabLo + S)
            x = (double)(i - kTabLo) / (double)N;
        else if (i >= kTabHi && i < kTabHi + A)
            x = (double)((int64_t)(i - kTabHi) << lgS) / (double)N;
        else
            continue;
        double sn, cs;
        sincospi(-2.0 * x, &sn, &cs);
        tab[i] = make_double2(cs, sn);
    }
}

// exp(-2 pi i r / N) for 0 <= r < N, lgS = ceil(log2(N) / 2)
__device__ __forceinline__ double2 twiddle(const double2* __restrict__ tab, int64_t r, int lgS)
{
    return cmul(tab[kTabHi + (r >> lgS)], tab[kTabLo + (r & (((int64_t)1 << lgS) - 1))]);
}

// exp(-2 pi i k / len) for k = 0 .. len/2 - 1 (len = 2^lg <= kFftTile), into tw
__device__ __forceinline__ void fill_twiddles(double2* tw, const double2* __restrict__ tab, int lg)
{
    for (int k = threadIdx.x; k < (1 << lg) / 2; k += blockDim.x)
        tw[k] = tab[k << (kFftTileLg - lg)];
}

// In-place radix-2 transform (decimation in time) of T sequences of length
// len = 2^lg in LDS, sequence t at buf[t * len], loaded in bit-reversed order;
// leaves them in natural order.  Two consecutive stages (spans h and 2h) are
// done per pass on the four values k, k + h, k + 2h, k + 3h of each block of
// 4h -- the same butterflies as two radix-2 stages, with half the passes,
// barriers and LDS traffic; an odd lg starts with one stage of span 1.  tw holds
// exp(-2 pi i j / len), j < len / 2; a pass reads one twiddle per butterfly
// and derives the other two.  Ends with a barrier.
__device__ __forceinline__ void lds_fft(double2* buf, const double2* tw, int lg, int T)
{
    const int len = 1 << lg;
    const int halfn = len >> 1;
    int lgh = 0;
    if (lg & 1) {
        __syncthreads();
        for (int b = threadIdx.x; b < T * halfn; b += blockDim.x) {
            double2* x = buf + 2 * b;
            const double2 a = x[0], c = x[1];
            x[0] = make_double2(a.x + c.x, a.y + c.y);
            x[1] = make_double2(a.x - c.x, a.y - c.y);
        }
        lgh = 1;
    }
    for (; lgh + 2 <= lg; lgh += 2) {
        __syncthreads();
        const int h = 1 << lgh;
        const int tws = halfn >> lgh;  // W_2h^k = tw[k tws], W_4h^k = tw[k tws / 2]
        for (int b = threadIdx.x; b < T * (len >> 2); b += blockDim.x) {
            const int k = b & (h - 1);
            double2* x = buf + ((b >> lgh) << (lgh + 2)) + k;
            const double2 a0 = x[0], a1 = x[h], a2 = x[2 * h], a3 = x[3 * h];
            // W_4h^k from the table; W_2h^k = (W_4h^k)^2 and W_4h^(k+h) = -i W_4h^k
            const double2 w2 = tw[k * (tws >> 1)];
            const double2 w1 = cmul(w2, w2);
            const double2 w3 = make_double2(w2.y, -w2.x);
            const double2 t1 = cmul(a1, w1), t3 = cmul(a3, w1);
            const double2 b0 = make_double2(a0.x + t1.x, a0.y + t1.y);
            const double2 b1 = make_double2(a0.x - t1.x, a0.y - t1.y);
            const double2 b2 = make_double2(a2.x + t3.x, a2.y + t3.y);
            const double2 b3 = make_double2(a2.x - t3.x, a2.y - t3.y);
            const double2 t2 = cmul(b2, w2), t4 = cmul(b3, w3);
            x[0] = make_double2(b0.x + t2.x, b0.y + t2.y);
            x[2 * h] = make_double2(b0.x - t2.x, b0.y - t2.y);
            x[h] = make_double2(b1.x + t4.x, b1.y + t4.y);
            x[3 * h] = make_double2(b1.x - t4.x, b1.y - t4.y);
        }
    }
    __syncthreads();
}

__device__ __forceinline__ int bitrev(int v, int lg)
{
    return lg == 0 ? 0 : (int)(__builtin_bitreverse32((unsigned)v) >> (32 - lg));
}

// First step: tile = T columns c (c = s * N2 + n2 over the group's 2 G signals)
// of N1 = 2^lg1 values each.  Output Y[s][N2 k1 + n2] = twiddled column FFTs.
template <bool PAIRS>
__global__ __launch_bounds__(kFftThreads) void spec_cols_kernel(const double* __restrict__ acc,
                                                                 int64_t n_t, int64_t r0,
                                                                 int64_t n_sig, int lg1, int lg2,
                                                                 const double2* __restrict__ tab,
                                                                 double2* __restrict__ Y)
{
    extern __shared__ double2 lds[];
    const int N1 = 1 << lg1;
    const int64_t N2 = (int64_t)1 << lg2;
    const int64_t N = (int64_t)N1 * N2;
    const int lgT = kFftTileLg - lg1;  // lg1 <= kFftTileLg
    const int T = 1 << lgT;             // columns per tile
    double2* buf = lds;
    double2* tw = lds + T * N1;
    const int64_t c0 = (int64_t)blockIdx.x * T;
    const int64_t n_cols = n_sig * N2;
    const int lgS = (lg1 + lg2 + 1) / 2;
    fill_twiddles(tw, tab, lg1);
    // load: consecutive threads take consecutive columns of one row n1
    for (int e = threadIdx.x; e < T * N1; e += blockDim.x) {
        const int n1 = e >> lgT;
        const int t = e & (T - 1);
        const int64_t c = c0 + t;
        double2 v = make_double2(0.0, 0.0);
        if (c < n_cols) {
            const int64_t sg = c >> lg2;
            const int64_t n2 = c & (N2 - 1);
            v = signal_at<PAIRS>(acc, n_t, r0, sg, N2 * n1 + n2);
        }
        buf[t * N1 + bitrev(n1, lg1)] = v;
    }
    lds_fft(buf, tw, lg1, T);
    for (int e = threadIdx.x; e < T * N1; e += blockDim.x) {
        const int k1 = e >> lgT;
        const int t = e & (T - 1);
        const int64_t c = c0 + t;
        if (c >= n_cols)
            continue;
        const int64_t sg = c >> lg2;
        const int64_t n2 = c & (N2 - 1);
        // exp(-2 pi i n2 k1 / N), argument reduced exactly
        const double2 v =
            cmul(buf[t * N1 + k1], twiddle(tab, (n2 * (int64_t)k1) & (N - 1), lgS));
        Y[sg * N + N2 * k1 + n2] = v;
    }
}

// Second step: tile = R rows (k1) of N2 = 2^lg2 contiguous values of one
// signal; X[s][k1 + N1 k2] = FFT over n2 of Y[s][N2 k1 + n2].
__global__ __launch_bounds__(kFftThreads) void spec_rows_kernel(const double2* __restrict__ Y,
                                                                 int64_t n_sig, int lg1, int lg2,
                                                                 const double2* __restrict__ tab,
                                                                 double2* __restrict__ X)
{
    extern __shared__ double2 lds[];
    const int64_t N1 = (int64_t)1 << lg1;
    const int N2 = 1 << lg2;
    const int64_t N = N1 * N2;
    const int lgR = kFftTileLg - lg2;  // lg2 <= kFftTileLg <= lg1 + lg2
    const int R = 1 << lgR;             // rows per tile (N1 is a multiple of R)
    double2* buf = lds;
    double2* tw = lds + R * N2;
    const int64_t tiles_per_sig = N1 / R;
    const int64_t sg = blockIdx.x / tiles_per_sig;
    const int64_t k10 = (blockIdx.x - sg * tiles_per_sig) * R;
    if (sg >= n_sig)
        return;
    fill_twiddles(tw, tab, lg2);
    const double2* y = Y + sg * N + N2 * k10;  // R contiguous rows
    for (int e = threadIdx.x; e < R * N2; e += blockDim.x) {
        const int r = e >> lg2;
        const int n2 = e & (N2 - 1);
        buf[r * N2 + bitrev(n2, lg2)] = y[e];
    }
    lds_fft(buf, tw, lg2, R);
    // store: consecutive threads take consecutive rows of one k2
    double2* x = X + sg * N + k10;
    for (int e = threadIdx.x; e < R * N2; e += blockDim.x) {
        const int k2 = e >> lgR;
        const int r = e & (R - 1);
        x[N1 * k2 + r] = buf[r * N2 + k2];
    }
}

// First step for both signals of cell g at once: tile = Tc consecutive columns
// n2 (Tc = kFftTile / (2 N1), so lg1 < kFftTileLg; N2 is a multiple of Tc),
// buf[s][tc][N1] for signal s = 0 (Ex + i Ey) and 1 (Ez).  Each slot of the
// detector is read once; the twiddle is shared by the two signals.  With part
// set, the tile also leaves the sum of |E|^2 over its slots in
// part[g][tile] (Parseval, reduced per cell by spec_parseval_parts_kernel).
template <bool PAIRS>
__global__ __launch_bounds__(kFftThreads) void spec_cols2_kernel(const double* __restrict__ acc,
                                                                  int64_t n_t, int64_t r0,
                                                                  int64_t G, int lg1, int lg2,
                                                                  const double2* __restrict__ tab,
                                                                  double2* __restrict__ Y,
                                                                  double* __restrict__ part)
{
    __shared__ double red[kFftThreads];
    extern __shared__ double2 lds[];
    const int N1 = 1 << lg1;
    const int64_t N2 = (int64_t)1 << lg2;
    const int64_t N = (int64_t)N1 * N2;
    const int lgTc = kFftTileLg - 1 - lg1;
    const int Tc = 1 << lgTc;
    double2* buf = lds;
    double2* tw = lds + 2 * Tc * N1;
    const int64_t tiles_per_cell = N2 >> lgTc;
    const int64_t g = blockIdx.x / tiles_per_cell;
    const int64_t n20 = (blockIdx.x - g * tiles_per_cell) << lgTc;
    if (g >= G)
        return;
    const int lgS = (lg1 + lg2 + 1) / 2;
    fill_twiddles(tw, tab, lg1);
    // load: consecutive threads take consecutive columns (slots) of one row n1
    double e2 = 0.0;
    for (int e = threadIdx.x; e < Tc * N1; e += blockDim.x) {
        const int n1 = e >> lgTc;
        const int tc = e & (Tc - 1);
        const int j = bitrev(n1, lg1);
        const double2 v0 = signal_at<PAIRS>(acc, n_t, r0, 2 * g, N2 * n1 + n20 + tc);
        const double2 v1 = signal_at<PAIRS>(acc, n_t, r0, 2 * g + 1, N2 * n1 + n20 + tc);
        buf[tc * N1 + j] = v0;
        buf[(Tc + tc) * N1 + j] = v1;
        e2 += (v0.x * v0.x + v0.y * v0.y) + v1.x * v1.x;
    }
    if (part) {
        red[threadIdx.x] = e2;
        for (int w = kFftThreads / 2; w > 0; w >>= 1) {
            __syncthreads();
            if ((int)threadIdx.x < w)
                red[threadIdx.x] += red[threadIdx.x + w];
        }
        if (threadIdx.x == 0)
            part[blockIdx.x] = red[0];
    }
    lds_fft(buf, tw, lg1, 2 * Tc);
    double2* y1 = Y + (2 * g) * N;
    double2* y2 = y1 + N;
    for (int e = threadIdx.x; e < Tc * N1; e += blockDim.x) {
        const int k1 = e >> lgTc;
        const int tc = e & (Tc - 1);
        const int64_t n2 = n20 + tc;
        // exp(-2 pi i n2 k1 / N), argument reduced exactly
        const double2 w = twiddle(tab, (n2 * (int64_t)k1) & (N - 1), lgS);
        y1[N2 * k1 + n2] = cmul(buf[tc * N1 + k1], w);
        y2[N2 * k1 + n2] = cmul(buf[(Tc + tc) * N1 + k1], w);
    }
}

// In-register radix-2 transform (decimation in time) of 2^LG values loaded in
// bit-reversed order, leaving them in natural order.  W[j] = exp(-2 pi i j /
// 2^LG), j < 2^(LG-1), read with uniform addresses (scalar loads: the same
// twiddles for every lane); the j = 0 butterflies take no product.
template <int LG>
__device__ __forceinline__ void reg_fft(double2 (&v)[1 << LG], const double2* __restrict__ W)
{
#pragma unroll
    for (int s = 0; s < LG; ++s) {
        const int h = 1 << s;
#pragma unroll
        for (int j = 0; j < h; ++j) {
            const double2 w = j == 0 ? make_double2(1.0, 0.0) : W[j << (LG - 1 - s)];
#pragma unroll
            for (int blk = 0; blk < (1 << LG); blk += 2 * h) {
                const double2 a = v[blk + j];
                const double2 t = j == 0 ? v[blk + j + h] : cmul(v[blk + j + h], w);
                v[blk + j] = make_double2(a.x + t.x, a.y + t.y);
                v[blk + j + h] = make_double2(a.x - t.x, a.y - t.y);
            }
        }
    }
}

constexpr int kRow32 = 32;  // N2 = 1024 = 32 x 32

// The second step for rows of N2 = 1024, held in registers instead of LDS
// passes: a row is a 32 x 32 four-step transform (n = 32 a + b, k = c + 32 d),
//     X[c + 32 d] = sum_b W_32^(b d) W_1024^(b c) sum_a x[32 a + b] W_32^(a c).
// One wavefront per row k1 of a cell: lanes 0-31 take signal Z1, lanes 32-63
// signal Z2.  Lane b loads x[32 a + b] (a = 0 .. 31, coalesced over the lanes),
// transforms over a in registers, multiplies by W_1024^(b c) and writes the 32
// values to LDS; lane c then reads A[b][c] (b = 0 .. 31) and transforms over b.
// Q = |Z1|^2 + |Z2|^2 is folded through LDS and stored row-major at
// Qt[g][1024 k1 + c + 32 d] at frequency k1 + N1 (c + 32 d), so that the stores are
// contiguous; spec_power_t_kernel transposes it.
__global__ __launch_bounds__(64) void spec_rows_q32_kernel(const double2* __restrict__ Y,
                                                           int64_t G, int lg1,
                                                           const double2* __restrict__ tab,
                                                           double* __restrict__ Q)
{
    __shared__ double2 T[2][kRow32][kRow32 + 1];  // A[b][c] per signal, rows padded
    const int lane = threadIdx.x;
    const int sig = lane >> 5;
    const int b = lane & (kRow32 - 1);
    const int64_t N1 = (int64_t)1 << lg1;
    const int64_t N = N1 * (kRow32 * kRow32);
    const int64_t g = blockIdx.x >> lg1;
    const int64_t k1 = blockIdx.x & (N1 - 1);
    if (g >= G)
        return;
    // exp(-2 pi i j / 32) = tab[64 j] (tab[k] = exp(-2 pi i k / kFftTile))
    static_assert(kFftTile == 64 * kRow32, "32-point twiddles from the LDS-transform table");
    double2 w32[kRow32 / 2];
#pragma unroll
    for (int j = 0; j < kRow32 / 2; ++j)
        w32[j] = tab[64 * j];
    const double2* y = Y + (2 * g + sig) * N + (kRow32 * kRow32) * k1;
    double2 v[kRow32];
#pragma unroll
    for (int a = 0; a < kRow32; ++a)
        v[bitrev(a, 5)] = y[kRow32 * a + b];
    reg_fft<5>(v, w32);
#pragma unroll
    for (int c = 0; c < kRow32; ++c) {
        // W_1024^m = tab[2 m] for m < 512, -tab[2 m - 1024] above
        const int m = (b * c) & 1023;
        const double2 t = tab[(2 * m) & 1023];
        const double2 w = m < 512 ? t : make_double2(-t.x, -t.y);
        T[sig][c][b] = c == 0 ? v[0] : cmul(v[c], w);
    }
    __syncthreads();
#pragma unroll
    for (int bb = 0; bb < kRow32; ++bb)
        v[bitrev(bb, 5)] = T[sig][b][bb];
    reg_fft<5>(v, w32);
    __syncthreads();  // T is reused for |Z2|^2
    double* P = reinterpret_cast<double*>(&T[0][0][0]);  // [32][33] doubles
    if (sig == 1) {
#pragma unroll
        for (int d = 0; d < kRow32; ++d)
            P[d * (kRow32 + 1) + b] = v[d].x * v[d].x + v[d].y * v[d].y;
    }
    __syncthreads();
    if (sig == 0) {
        double* q = Q + g * N + (kRow32 * kRow32) * k1;
#pragma unroll
        for (int d = 0; d < kRow32; ++d)
            q[b + kRow32 * d] = (v[d].x * v[d].x + v[d].y * v[d].y) + P[d * (kRow32 + 1) + b];
    }
}

// ---------------------------------------------------------------------------
// transforms of up to 2 kFftTile slots
// ---------------------------------------------------------------------------

// The whole spectrum of C = min(2^LGT / N, 64) cells at a time in one kernel:
// a slot is read once (from the detector's E beside B: 48 bytes for 24), its
// |E|^2 summed for dI/dOmega, both signals transformed in LDS, and the power
// stored and added up over the workgroup's cells.  Persistent workgroups, two a CU:
// a thread keeps its output frequencies, their slot weights and their part of
// dI/domega in registers over all cells, and has the next cells' slots in flight
// while it transforms.  Bound by the LDS passes and by HBM reading the detector
// (2.9 TB/s).  Measured against columns, power and a separate Parseval pass, which
// wrote and read both signals' spectra between them: 16384 cells x 2048 slots with
// weights 1.35 -> 0.56 ms a call, 4000 cells x 300 slots 94 -> 74 us, 37 x 37 41 -> 40.
// LGT: log2 of the slots at a time; 2048 for transforms up to that, in 512 threads
// (two workgroups a CU), and 4096 in 1024 threads (one): four wavefronts a SIMD.
constexpr int kSmallCells = 64;                           // cells at a time, at most
constexpr int kSmallPer = 4;                              // slots, and outputs, of a thread
constexpr int small_threads(int lgt) { return (1 << lgt) / kSmallPer; }

// Position of value i of a transform of 2^lg in LDS.  Sixteen values span the
// banks, and sixteen consecutive threads reach a pass's values at strides of 4 or 16
// (bits 4 and 5 of the index) or store them in bit-reversed order (the four highest
// bits): these bits are folded into the lowest four, so that each of these meets
// every bank once.
__device__ __forceinline__ int lds_at(int i, int lg)
{
    const int s = (i >> 4) & 3;
    return i ^ s ^ (s << 2) ^ ((i >> max(5, lg - 4)) & 15);
}

// lds_fft on values kept at lds_at(); tw holds the first quarter of the circle, all
// that two stages per pass read.
template <int THREADS>
__device__ __forceinline__ void lds_fft_at(double2* buf, const double2* tw, int lg, int T)
{
    const int len = 1 << lg;
    int lgh = 0;
    if (lg & 1) {
        __syncthreads();
        for (int b = threadIdx.x; b < T * (len >> 1); b += THREADS) {
            double2* x = buf + lds_at(2 * b, lg);
            double2* y = buf + lds_at(2 * b + 1, lg);
            const double2 a = *x, c = *y;
            *x = make_double2(a.x + c.x, a.y + c.y);
            *y = make_double2(a.x - c.x, a.y - c.y);
        }
        lgh = 1;
    }
    for (; lgh + 2 <= lg; lgh += 2) {
        __syncthreads();
        const int h = 1 << lgh;
        const int step = len >> (lgh + 2);  // W_4h^k = tw[k step]
#pragma unroll 1
        for (int b = threadIdx.x; b < T * (len >> 2); b += THREADS) {
            const int k = b & (h - 1);
            const int i = ((b >> lgh) << (lgh + 2)) + k;
            double2* x0 = buf + lds_at(i, lg);
            double2* x1 = buf + lds_at(i + h, lg);
            double2* x2 = buf + lds_at(i + 2 * h, lg);
            double2* x3 = buf + lds_at(i + 3 * h, lg);
            const double2 a0 = *x0, a1 = *x1, a2 = *x2, a3 = *x3;
            const double2 w2 = tw[k * step];
            const double2 w1 = cmul(w2, w2);
            const double2 w3 = make_double2(w2.y, -w2.x);
            const double2 t1 = cmul(a1, w1), t3 = cmul(a3, w1);
            const double2 b0 = make_double2(a0.x + t1.x, a0.y + t1.y);
            const double2 b1 = make_double2(a0.x - t1.x, a0.y - t1.y);
            const double2 b2 = make_double2(a2.x + t3.x, a2.y + t3.y);
            const double2 b3 = make_double2(a2.x - t3.x, a2.y - t3.y);
            const double2 t2 = cmul(b2, w2), t4 = cmul(b3, w3);
            *x0 = make_double2(b0.x + t2.x, b0.y + t2.y);
            *x2 = make_double2(b0.x - t2.x, b0.y - t2.y);
            *x1 = make_double2(b1.x + t4.x, b1.y + t4.y);
            *x3 = make_double2(b1.x - t4.x, b1.y - t4.y);
        }
    }
    __syncthreads();
}

template <bool PAIRS, int LGT>
__global__ __launch_bounds__(small_threads(LGT), 4) void spec_small_kernel(
    const double* __restrict__ acc, int64_t n_t, int64_t n_c, int lg,
    const double2* __restrict__ tab, const double* __restrict__ cells,
    const int64_t* __restrict__ user_index, const double* __restrict__ weights, double dt, double c,
    double* __restrict__ d2I, double* __restrict__ sums, double* __restrict__ dIdO)
{
    constexpr int kSmallThreads = small_threads(LGT);
    constexpr int kTile = 1 << LGT;
    __shared__ double2 buf[2 * kTile];  // [signal][cell][slot], at lds_at()
    __shared__ double2 tw[kTile / 4];
    __shared__ double part[kSmallCells];   // sums of |E|^2
    const int tid = threadIdx.x;
    const int N = 1 << lg;
    const int lgC = min(LGT - lg, 6);
    const int C = 1 << lgC;
    const int total = C << lg;             // slots at a time (at most kTile)
    const int n_f = N / 2 + 1;
    for (int k = tid; k < N / 4; k += kSmallThreads)
        tw[k] = lg <= kFftTileLg ? tab[k << (kFftTileLg - lg)] : twiddle(tab, k, (lg + 1) / 2);
    if (tid < kSmallCells)
        part[tid] = 0.0;
    // the thread's outputs: cell of the tile, frequency, |(e^{-i w dt} - 1)/(-i w)|^2
    int oc[kSmallPer], om[kSmallPer];
    double W2[kSmallPer], sum[kSmallPer];
#pragma unroll
    for (int i = 0; i < kSmallPer; ++i) {
        const int o = tid + kSmallThreads * i;
        oc[i] = o < C * n_f ? o / n_f : -1;
        om[i] = o - (o / n_f) * n_f;
        const double omega = 2.0 * kPi * (double)om[i] / ((double)N * dt);
        const double sw = om[i] == 0 ? dt : 2.0 * sin(0.5 * omega * dt) / omega;
        W2[i] = sw * sw;
        sum[i] = 0.0;
    }
    const int64_t n_tiles = (n_c + C - 1) >> lgC;
    double2 v0[kSmallPer];
    double v1[kSmallPer];
    auto load = [&](int64_t tile) {
#pragma unroll
        for (int i = 0; i < kSmallPer; ++i) {
            const int e = tid + kSmallThreads * i;
            const int64_t r = (tile << lgC) + (e >> lg);
            v0[i] = make_double2(0.0, 0.0);
            v1[i] = 0.0;
            if (e < total && tile < n_tiles && r < n_c) {
                v0[i] = signal_at<PAIRS>(acc, n_t, r, 0, e & (N - 1));
                v1[i] = signal_at<PAIRS>(acc, n_t, r, 1, e & (N - 1)).x;
            }
        }
    };
    load(blockIdx.x);
    __syncthreads();
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        double e2 = 0.0;
#pragma unroll
        for (int i = 0; i < kSmallPer; ++i) {
            const int e = tid + kSmallThreads * i;
            if (e < total) {
                const int at = (e & ~(N - 1)) + bitrev(e & (N - 1), lg);
                buf[lds_at(at, lg)] = v0[i];
                buf[lds_at(total + at, lg)] = make_double2(v1[i], 0.0);
            }
            if (dIdO) {  // |E|^2 of the lanes that share the cell, cell by cell
                e2 += (v0[i].x * v0[i].x + v0[i].y * v0[i].y) + v1[i] * v1[i];
                if (N <= kSmallThreads || ((kSmallThreads * (i + 1)) & (N - 1)) == 0) {
                    const int width = min(N, 64);
                    for (int m = width >> 1; m > 0; m >>= 1)
                        e2 += __shfl_xor(e2, m);
                    if ((tid & (width - 1)) == 0 && e < total)
                        __hip_atomic_fetch_add(&part[e >> lg], e2, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
                    e2 = 0.0;
                }
            }
        }
        load(tile + gridDim.x);
        lds_fft_at<kSmallThreads>(buf, tw, lg, 2 * C);
        const int64_t r0 = tile << lgC;
#pragma unroll
        for (int i = 0; i < kSmallPer; ++i) {
            const int64_t r = r0 + oc[i];
            if (oc[i] < 0 || r >= n_c)
                continue;
            const int b1 = oc[i] << lg, b2 = total + b1, m = om[i], mm = (N - m) & (N - 1);
            const double2 p1 = buf[lds_at(b1 + m, lg)], q1 = buf[lds_at(b1 + mm, lg)];
            const double2 p2 = buf[lds_at(b2 + m, lg)], q2 = buf[lds_at(b2 + mm, lg)];
            const double p = 0.5 * ((p1.x * p1.x + p1.y * p1.y) + (q1.x * q1.x + q1.y * q1.y) +
                                    (p2.x * p2.x + p2.y * p2.y) + (q2.x * q2.x + q2.y * q2.y));
            const double* x = cells + 3 * r;
            const double R2 = x[0] * x[0] + x[1] * x[1] + x[2] * x[2];
            const double S = c * R2 / (4.0 * kPi * kPi) * W2[i] * p;
            const int64_t cell = user_index[r];
            if (d2I)
                d2I[cell * n_f + m] = S;
            sum[i] += (weights ? weights[cell] : 1.0) * S;
        }
        if (dIdO && tid < C) {
            if (r0 + tid < n_c) {
                const double* x = cells + 3 * (r0 + tid);
                const double R2 = x[0] * x[0] + x[1] * x[1] + x[2] * x[2];
                dIdO[user_index[r0 + tid]] = c * R2 / (4.0 * kPi) * part[tid] * dt;
            }
            part[tid] = 0.0;
        }
        __syncthreads();  // buf and part are filled again
    }
    if (!sums)
        return;
    // the workgroup's part of dI/domega: its cells' sums added up in LDS
    double* s = reinterpret_cast<double*>(buf);
    for (int m = tid; m < n_f; m += kSmallThreads)
        s[m] = 0.0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSmallPer; ++i)
        if (oc[i] >= 0)
            __hip_atomic_fetch_add(s + om[i], sum[i], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
    __syncthreads();
    for (int m = tid; m < n_f; m += kSmallThreads)
        sums[(int64_t)blockIdx.x * n_f + m] = s[m];
}

// dI/domega from the workgroups' parts [n][n_f] (adding all of them to it atomically,
// hundreds to an address, took longer than the transforms of a small detector):
// 32 frequencies a workgroup, 32 threads to each
__global__ __launch_bounds__(1024) void spec_sums_kernel(const double* __restrict__ sums, int n,
                                                         int n_f, double* __restrict__ dIdw)
{
    __shared__ double red[32][33];
    const int m = blockIdx.x * 32 + threadIdx.x % 32;
    const int k = threadIdx.x / 32;
    double v = 0.0;
    if (m < n_f)
        for (int i = k; i < n; i += 32)
            v += sums[(int64_t)i * n_f + m];
    red[k][threadIdx.x % 32] = v;
    __syncthreads();
    if (k == 0 && m < n_f) {
        for (int i = 1; i < 32; ++i)
            v += red[i][threadIdx.x];
        dIdw[m] = v;
    }
}

template <bool PAIRS>
__global__ __launch_bounds__(256) void spec_load_kernel(const double* __restrict__ acc,
                                                        int64_t n_t, int64_t r0, int64_t G,
                                                        int64_t N, double2* __restrict__ Z)
{
    const int64_t total = G * N;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t g = i / N;
        const int64_t j = i - g * N;
        double e[3] = {0.0, 0.0, 0.0};
        if (j < n_t) {
            const int64_t s = (r0 + g) * n_t + j;
            if (PAIRS) {
                const float* q = reinterpret_cast<const float*>(acc) + s * 12;
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    e[k] = (double)q[k] + (double)q[6 + k];
            } else {
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    e[k] = acc[s * 6 + k];
            }
        }
        Z[(2 * g) * N + j] = make_double2(e[0], e[1]);
        Z[(2 * g + 1) * N + j] = make_double2(e[2], 0.0);
    }
}

// y = one radix-2 Stockham pass of x for butterflies of span Ns, over n_sig
// signals of length N: with k = j mod Ns, x[j] and x[j + N/2] e^{-i pi k/Ns}
// combine into y[2j - k] and y[2j - k + Ns].
__global__ __launch_bounds__(256) void spec_fft_pass(const double2* __restrict__ x,
                                                     double2* __restrict__ y, int64_t N,
                                                     int64_t Ns, int64_t n_sig)
{
    const int64_t half = N / 2;
    const int64_t total = n_sig * half;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t sig = i / half;
        const int64_t j = i - sig * half;
        const double2* xs = x + sig * N;
        double2* ys = y + sig * N;
        const int64_t k = j & (Ns - 1);
        const double2 a = xs[j];
        const double2 b = xs[j + half];
        double sn, cs;
        sincospi(-(double)k / (double)Ns, &sn, &cs);
        const double2 bw = make_double2(b.x * cs - b.y * sn, b.x * sn + b.y * cs);
        const int64_t idx = 2 * j - k;  // (j / Ns) * 2 Ns + k
        ys[idx] = make_double2(a.x + bw.x, a.y + bw.y);
        ys[idx + Ns] = make_double2(a.x - bw.x, a.y - bw.y);
    }
}

// d2I of kPowerCells cells of the group per thread, one thread per frequency
// m of a block, from Z1, Z2 of cell g (at Z[2g], Z[2g+1], natural order);
// their weighted sum is added to dIdw[m] (zeroed beforehand)
constexpr int kPowerCells = 16;

__global__ __launch_bounds__(256) void spec_power_kernel(
    const double2* __restrict__ Z, int64_t N, int64_t G, int64_t r0,
    const double* __restrict__ cells, const int64_t* __restrict__ user_index,
    const double* __restrict__ weights, double dt, double c, double* __restrict__ d2I,
    double* __restrict__ dIdw)
{
    const int64_t n_f = N / 2 + 1;
    const int64_t m = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (m >= n_f)
        return;
    const double omega = 2.0 * kPi * (double)m / ((double)N * dt);
    double W2;  // |(e^{-i w dt} - 1) / (-i w)|^2
    if (m == 0) {
        W2 = dt * dt;
    } else {
        const double s = 2.0 * sin(0.5 * omega * dt) / omega;
        W2 = s * s;
    }
    const int64_t mm = (N - m) & (N - 1);
    double sum = 0.0;
    const int64_t g0 = (int64_t)blockIdx.y * kPowerCells;
    const int64_t g1 = g0 + kPowerCells < G ? g0 + kPowerCells : G;
    for (int64_t g = g0; g < g1; ++g) {
        const double2* z1 = Z + (2 * g) * N;
        const double2* z2 = z1 + N;
        const double p = 0.5 * ((z1[m].x * z1[m].x + z1[m].y * z1[m].y) +
                                (z1[mm].x * z1[mm].x + z1[mm].y * z1[mm].y) +
                                (z2[m].x * z2[m].x + z2[m].y * z2[m].y) +
                                (z2[mm].x * z2[mm].x + z2[mm].y * z2[mm].y));
        const int64_t r = r0 + g;
        const double* x = cells + 3 * r;
        const double R2 = x[0] * x[0] + x[1] * x[1] + x[2] * x[2];
        const double S = c * R2 / (4.0 * kPi * kPi) * W2 * p;
        const int64_t cell = user_index[r];
        if (d2I)
            d2I[cell * n_f + m] = S;
        sum += (weights ? weights[cell] : 1.0) * S;
    }
    if (dIdw)
        unsafeAtomicAdd(dIdw + m, sum);
}

// Power spectra from Qt (row-major Q of spec_rows_q32_kernel, N1 = 2^lg1 rows of
// N2 = 2^lg2 with lg1 + lg2 = log2 N, lg2 >= 5): a workgroup takes a tile of
// B1 = min(N1, 32) consecutive k1 by B2 = kPowerTile / B1 consecutive k2 and
// transposes it through LDS, so that its reads (along k2, both Q(m) and
// Q(N - m)) and its d2I stores (along m = k1 + N1 k2) are contiguous.  Tiles
// cover k2 <= N2 / 2, i.e. m <= N / 2; kPowerCells cells per workgroup, whose
// weighted sum is added to dIdw[m] (zeroed beforehand).
constexpr int kPowerTileLg = 10;
constexpr int kPowerTile = 1 << kPowerTileLg;

__global__ __launch_bounds__(256) void spec_power_t_kernel(
    const double* __restrict__ Qt, int lg1, int lg2, int64_t G, int64_t r0,
    const double* __restrict__ cells, const int64_t* __restrict__ user_index,
    const double* __restrict__ weights, double dt, double c, double* __restrict__ d2I,
    double* __restrict__ dIdw)
{
    constexpr int kPer = kPowerTile / 256;  // tile values per thread
    const int lgB1 = lg1 < 5 ? lg1 : 5;
    const int B1 = 1 << lgB1;
    const int lgB2 = kPowerTileLg - lgB1;
    const int B2 = 1 << lgB2;
    const int stride = B2 + 1;  // LDS row of one k1, padded
    __shared__ double tile[kPowerTile + 32];
    const int64_t N1 = (int64_t)1 << lg1, N2 = (int64_t)1 << lg2;
    const int64_t N = N1 * N2;
    const int64_t n_f = N / 2 + 1;
    const int64_t tiles1 = N1 >> lgB1;
    const int64_t k1_0 = (int64_t)(blockIdx.x % tiles1) << lgB1;
    const int64_t k2_0 = (int64_t)(blockIdx.x / tiles1) << lgB2;
    // the thread's store slots: m and the slot weight |(e^{-i w dt} - 1)/(-i w)|^2
    int64_t mo[kPer];
    double W2[kPer], sum[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int e = threadIdx.x + 256 * i;
        const int64_t m = (k1_0 + (e & (B1 - 1))) + N1 * (k2_0 + (e >> lgB1));
        mo[i] = m < n_f ? m : -1;
        const double omega = 2.0 * kPi * (double)m / ((double)N * dt);
        const double sw = m == 0 ? dt : 2.0 * sin(0.5 * omega * dt) / omega;
        W2[i] = sw * sw;
        sum[i] = 0.0;
    }
    const int64_t g0 = (int64_t)blockIdx.y * kPowerCells;
    const int64_t g1 = g0 + kPowerCells < G ? g0 + kPowerCells : G;
    for (int64_t g = g0; g < g1; ++g) {
        const double* q = Qt + g * N;
        // load along k2: Q(m) and Q(N - m), m = k1 + N1 k2 (k2 < N2 / 2 + B2 <= N2)
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int e = threadIdx.x + 256 * i;
            const int k1l = e >> lgB2, k2l = e & (B2 - 1);
            const int64_t k1 = k1_0 + k1l, k2 = k2_0 + k2l;
            const int64_t k1m = (N1 - k1) & (N1 - 1);
            const int64_t k2m = k1 == 0 ? (N2 - k2) & (N2 - 1) : N2 - 1 - k2;
            tile[k1l * stride + k2l] = 0.5 * (q[k1 * N2 + k2] + q[k1m * N2 + k2m]);
        }
        __syncthreads();
        const int64_t r = r0 + g;
        const double* x = cells + 3 * r;
        const double R2 = x[0] * x[0] + x[1] * x[1] + x[2] * x[2];
        const double scale = c * R2 / (4.0 * kPi * kPi);
        const int64_t cell = user_index[r];
        const double wc = weights ? weights[cell] : 1.0;
        // store along m
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            if (mo[i] < 0)
                continue;
            const int e = threadIdx.x + 256 * i;
            const double S = scale * W2[i] * tile[(e & (B1 - 1)) * stride + (e >> lgB1)];
            if (d2I)
                d2I[cell * n_f + mo[i]] = S;
            sum[i] += wc * S;
        }
        __syncthreads();  // the tile is refilled for the next cell
    }
    if (dIdw) {
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            if (mo[i] >= 0)
                unsafeAtomicAdd(dIdw + mo[i], sum[i]);
    }
}

__global__ __launch_bounds__(256) void spec_zero_kernel(double* __restrict__ p, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.0;
}

template <bool PAIRS>
__global__ __launch_bounds__(256) void spec_parseval_kernel(const double* __restrict__ acc,
                                                            int64_t n_t,
                                                            const double* __restrict__ cells,
                                                            const int64_t* __restrict__ user_index,
                                                            double dt, double c,
                                                            double* __restrict__ dIdO)
{
    __shared__ double part[256];
    const int64_t r = blockIdx.x;
    double s = 0.0;
    for (int64_t j = threadIdx.x; j < n_t; j += 256) {
        const int64_t i = r * n_t + j;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            double e;
            if (PAIRS) {
                const float* q = reinterpret_cast<const float*>(acc) + i * 12;
                e = (double)q[k] + (double)q[6 + k];
            } else {
                e = acc[i * 6 + k];
            }
            s += e * e;
        }
    }
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double* x = cells + 3 * r;
        const double R2 = x[0] * x[0] + x[1] * x[1] + x[2] * x[2];
        dIdO[user_index[r]] = c * R2 / (4.0 * kPi) * part[0] * dt;
    }
}

// dI/dOmega of the cells of a group from the per-tile sums of |E|^2 left by
// spec_cols2_kernel (part[g][0 .. tiles_per_cell), added in order)
__global__ __launch_bounds__(256) void spec_parseval_parts_kernel(
    const double* __restrict__ part, int64_t tiles_per_cell, int64_t G, int64_t r0,
    const double* __restrict__ cells, const int64_t* __restrict__ user_index, double dt, double c,
    double* __restrict__ dIdO)
{
    const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (g >= G)
        return;
    double sum = 0.0;
    for (int64_t i = 0; i < tiles_per_cell; ++i)
        sum += part[g * tiles_per_cell + i];
    const int64_t r = r0 + g;
    const double* x = cells + 3 * r;
    const double R2 = x[0] * x[0] + x[1] * x[1] + x[2] * x[2];
    dIdO[user_index[r]] = c * R2 / (4.0 * kPi) * sum * dt;
}

unsigned grid_for(int64_t n);

// power spectra of a group from its transforms Z in natural order, or from
// the row-major Qt of the rows step (lg_q1 = log2 N1 > 0); dIdw is zeroed
// before the first group adds to it
hipError_t launch_power(const double2* Z, int lg_q1, int64_t N, int64_t G, int64_t r0,
                        const double* cells, const int64_t* user_index, const double* weights,
                        double dt, double c, double* d2I, double* dIdw, bool first_group,
                        hipStream_t s)
{
    const int64_t n_f = N / 2 + 1;
    if (dIdw && first_group)
        hipLaunchKernelGGL(spec_zero_kernel, dim3(grid_for(n_f)), dim3(256), 0, s, dIdw, n_f);
    const unsigned grid_y = (unsigned)((G + kPowerCells - 1) / kPowerCells);
    if (lg_q1 > 0) {
        int lg = 0;
        while (((int64_t)1 << lg) < N)
            ++lg;
        const int lg2 = lg - lg_q1;
        const int lgB1 = lg_q1 < 5 ? lg_q1 : 5;
        const int64_t B2 = (int64_t)1 << (kPowerTileLg - lgB1);
        const int64_t tiles2 = (((int64_t)1 << lg2) / 2 + 1 + B2 - 1) / B2;
        const int64_t tiles1 = ((int64_t)1 << lg_q1) >> lgB1;
        hipLaunchKernelGGL(spec_power_t_kernel, dim3((unsigned)(tiles1 * tiles2), grid_y),
                           dim3(256), 0, s, reinterpret_cast<const double*>(Z), lg_q1, lg2, G, r0,
                           cells, user_index, weights, dt, c, d2I, dIdw);
    } else {
        hipLaunchKernelGGL(spec_power_kernel, dim3((unsigned)((n_f + 255) / 256), grid_y),
                           dim3(256), 0, s, Z, N, G, r0, cells, user_index, weights, dt, c, d2I,
                           dIdw);
    }
    return hipGetLastError();
}

unsigned grid_for(int64_t n)
{
    int64_t b = (n + 255) / 256;
    return (unsigned)(b > 65536 ? 65536 : (b < 1 ? 1 : b));
}

}  // namespace

hipError_t launch_spectrum_group(const double* acc, bool pairs, int64_t n_t, int64_t r0,
                                 int64_t G, int64_t N, const double* cells,
                                 const int64_t* user_index, const double* weights, double dt,
                                 double c, double2* work0, double2* work1, double2* tables,
                                 double* d2I, double* dIdw, double* dIdO, bool* parseval_done,
                                 bool first_group, int64_t n_cus, hipStream_t s)
{
    *parseval_done = false;
    int lg = 0;
    while (((int64_t)1 << lg) < N)
        ++lg;
    if (N <= kSpecOneLaunch) {  // all cells at once (the caller's group is the detector)
        hipLaunchKernelGGL(spec_tables_kernel, dim3(20), dim3(256), 0, s, tables, lg);
        const bool wide = N > kFftTile;
        const int lgC = wide ? 0 : std::min(kFftTileLg - lg, 6);
        const int64_t tiles = (G + ((int64_t)1 << lgC) - 1) >> lgC;
        const int n_f = (int)(N / 2 + 1);
        // the workgroups their LDS allows
        const int64_t blocks =
            std::min<int64_t>(std::min<int64_t>(tiles, (wide ? 1 : 2) * n_cus), kSpecParts);
        double* sums = dIdw ? reinterpret_cast<double*>(work0) : nullptr;
        auto kernel = wide ? (pairs ? spec_small_kernel<true, kFftTileLg + 1>
                                    : spec_small_kernel<false, kFftTileLg + 1>)
                           : (pairs ? spec_small_kernel<true, kFftTileLg>
                                    : spec_small_kernel<false, kFftTileLg>);
        const unsigned threads = small_threads(wide ? kFftTileLg + 1 : kFftTileLg);
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(threads), 0, s, acc, n_t, G, lg,
                           tables, cells, user_index, weights, dt, c, d2I, sums, dIdO);
        if (dIdw)
            hipLaunchKernelGGL(spec_sums_kernel, dim3((unsigned)((n_f + 31) / 32)), dim3(1024), 0,
                               s, sums, (int)blocks, n_f, dIdw);
        *parseval_done = true;
        return hipGetLastError();
    }
    if (N <= (int64_t)kFftTile * kFftTile) {
        // four-step: N1 = 2^lg1 in the columns step, N2 = 2^lg2 in the rows
        // step, both <= kFftTile; each workgroup holds kFftTile values (32 KiB
        // of LDS) plus its twiddles.  Rows of kFftTile / 2 let the rows step
        // take both signals of a cell and store Q; the columns step does the
        // same while N1 <= kFftTile / 2.
        const int lg2 = std::max(kFftTileLg - 1, lg - kFftTileLg);
        const int lg1 = lg - lg2;
        const int64_t n_sig = 2 * G;
        hipLaunchKernelGGL(spec_tables_kernel, dim3(20), dim3(256), 0, s, tables, lg);
        // kFftTile values and len/2 twiddles (40 KiB for len 1024: four workgroups per CU)
        const size_t lds_a = ((size_t)kFftTile + ((size_t)1 << lg1) / 2) * sizeof(double2);
        if (lg1 < kFftTileLg) {
            const int64_t tiles_per_cell = (int64_t)1 << (lg2 - (kFftTileLg - 1 - lg1));
            const int64_t tiles = G * tiles_per_cell;
            // Parseval's per-tile sums after the row step's output in work1 (G N
            // doubles of its 4 G N)
            double* part = dIdO ? reinterpret_cast<double*>(work1) + G * N : nullptr;
            if (pairs)
                hipLaunchKernelGGL(spec_cols2_kernel<true>, dim3((unsigned)tiles),
                                   dim3(kFftThreads), lds_a, s, acc, n_t, r0, G, lg1, lg2, tables,
                                   work0, part);
            else
                hipLaunchKernelGGL(spec_cols2_kernel<false>, dim3((unsigned)tiles),
                                   dim3(kFftThreads), lds_a, s, acc, n_t, r0, G, lg1, lg2, tables,
                                   work0, part);
            if (part) {
                hipLaunchKernelGGL(spec_parseval_parts_kernel, dim3((unsigned)((G + 255) / 256)),
                                   dim3(256), 0, s, part, tiles_per_cell, G, r0, cells, user_index,
                                   dt, c, dIdO);
                *parseval_done = true;
            }
        } else {
            const int T = kFftTile >> lg1;
            const int64_t n_cols = n_sig << lg2;
            const unsigned blocks_a = (unsigned)((n_cols + T - 1) / T);
            if (pairs)
                hipLaunchKernelGGL(spec_cols_kernel<true>, dim3(blocks_a), dim3(kFftThreads), lds_a,
                                   s, acc, n_t, r0, n_sig, lg1, lg2, tables, work0);
            else
                hipLaunchKernelGGL(spec_cols_kernel<false>, dim3(blocks_a), dim3(kFftThreads),
                                   lds_a, s, acc, n_t, r0, n_sig, lg1, lg2, tables, work0);
        }
        int lg_q1 = 0;
        const size_t lds_b = ((size_t)kFftTile + ((size_t)1 << lg2) / 2) * sizeof(double2);
        if (lg2 == 10) {
            // rows of 1024 in registers, one wavefront per row of a cell
            hipLaunchKernelGGL(spec_rows_q32_kernel, dim3((unsigned)(G << lg1)), dim3(64), 0,
                               s, work0, G, lg1, tables, reinterpret_cast<double*>(work1));
            lg_q1 = lg1;
        } else {
            const int R = kFftTile >> lg2;
            const unsigned blocks_b = (unsigned)(n_sig * (((int64_t)1 << lg1) / R));
            hipLaunchKernelGGL(spec_rows_kernel, dim3(blocks_b), dim3(kFftThreads), lds_b, s,
                               work0, n_sig, lg1, lg2, tables, work1);
        }
        return launch_power(work1, lg_q1, N, G, r0, cells, user_index, weights, dt, c, d2I, dIdw,
                            first_group, s);
    }
    if (pairs)
        hipLaunchKernelGGL(spec_load_kernel<true>, dim3(grid_for(G * N)), dim3(256), 0, s, acc,
                           n_t, r0, G, N, work0);
    else
        hipLaunchKernelGGL(spec_load_kernel<false>, dim3(grid_for(G * N)), dim3(256), 0, s, acc,
                           n_t, r0, G, N, work0);
    double2* x = work0;
    double2* y = work1;
    for (int64_t Ns = 1; Ns < N; Ns *= 2) {
        hipLaunchKernelGGL(spec_fft_pass, dim3(grid_for(2 * G * (N / 2))), dim3(256), 0, s, x, y,
                           N, Ns, 2 * G);
        double2* t = x;
        x = y;
        y = t;
    }
    return launch_power(x, 0, N, G, r0, cells, user_index, weights, dt, c, d2I, dIdw,
                        first_group, s);
}

hipError_t launch_spectrum_parseval(const double* acc, bool pairs, int64_t n_c, int64_t n_t,
                                    const double* cells, const int64_t* user_index, double dt,
                                    double c, double* dIdO, hipStream_t s)
{
    if (n_c <= 0)
        return hipSuccess;
    if (pairs)
        hipLaunchKernelGGL(spec_parseval_kernel<true>, dim3((unsigned)n_c), dim3(256), 0, s, acc,
                           n_t, cells, user_index, dt, c, dIdO);
    else
        hipLaunchKernelGGL(spec_parseval_kernel<false>, dim3((unsigned)n_c), dim3(256), 0, s,
                           acc, n_t, cells, user_index, dt, c, dIdO);
    return hipGetLastError();
}

}  // namespace radio
