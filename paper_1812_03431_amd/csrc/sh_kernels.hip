// Spherical-harmonic transforms on gfx950 (Section 3).
//
// Analysis:  xi_n^m = sum_j w_j P_n^m(mu_j) F_j^m,  F_j^m = (1/nlon) sum_k xi(mu_j, lam_k) e^{-i m lam_k}
// Synthesis: xi(mu_j, lam_k) = sum_m c_m Re( sum_n xi_n^m P_n^m(mu_j) e^{i m lam_k} ), c_0 = 1, c_m = 2
// (the m = 0 term uses Re(xi_n^0)).
//
// Longitude: one complex FFT of length nlon in registers per field and pair of
// grid rows j, j' = nlat-1-j, a workgroup taking the pair's FFTs of several
// fields.  Latitude: per zonal order m the Legendre sum is a small dense
// contraction (T+1-m degrees x nlat/2 latitudes x 2B real columns) and runs on
// FP64 MFMA (v_mfma_f64_4x4x4f64, four blocks).  Gauss latitudes are symmetric about the equator
// and P_n^m(-mu) = (-1)^{n-m} P_n^m(mu), so only northern latitudes are used
// and each sum splits into an even part (F_j + F_{j'}) and an odd part
// (F_j - F_{j'}).
//
// Fourier workspace (c = 2b + {0: re, 1: im}): the analysis writes the
// weighted even/odd parts EO[m][0|1][j][c], j < nlat/2; the synthesis writes
// the coefficients Fw[m][j][c].  Each (m, parity) plane and each order's plane is
// padded by kFourPad doubles.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "internal.hpp"

namespace rexi {
namespace {

// Plane strides of the Fourier workspace, in doubles: an EO plane [j][c] of one
// (order, parity) and an order's plane [row][c] are padded by kFourPad so that
// the lines of consecutive planes are not a power of two apart.
constexpr int kFourPad = 32;
__host__ __device__ __forceinline__ long long eo_plane(int H, int C) { return (long long)H * C + kFourPad; }
__host__ __device__ __forceinline__ long long fw_plane(int nlat, int C) { return (long long)nlat * C + kFourPad; }

__device__ __forceinline__ double2 cmul(double2 w, double2 v) {
    return make_double2(fma(w.x, v.x, -w.y * v.y), fma(w.x, v.y, w.y * v.x));
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

// FFT of 2^BITS points, kE of them per thread in registers: radix-8, -4 and -2
// passes in self-sorting (Stockham) order.  Before pass p, of radix r, after passes
// of product L, thread t holds x[t + kT i], i < kE; its butterfly b takes j = t + kT b,
// u = j mod L, the inputs x[j + k n / r] with twiddles exp(-2 pi i u k / (L r)),
// k < r, and its outputs go to y[(j - u) r + u + k L].  So the first pass's inputs and
// the last pass's outputs are in natural order, a wave's part contiguous, and the
// data cross the LDS once between two passes (n = 512: two times, n = 2048: three),
// one FFT per wave or less up to n = 512, where no barrier is needed.
template <int BITS>
struct Fft {
    static constexpr int kN = 1 << BITS;
    static constexpr int kE = kN < 8 ? kN : 8;             // points per thread
    static constexpr int kT = kN / kE;                     // threads per FFT
    // threads per workgroup: at least two fields, whose orders are then 32 bytes, up to
    // n = 2048 (there 512 / 256 threads: 510 / 532 us an analysis of 16 fields at
    // T1023), and not more than that needs (n = 512, 12 fields at T256: 256 / 512 /
    // 1024 threads 24.9 / 25.1 / 28.1 us)
    static constexpr int kBlock = kT > 128 ? 512 : 256;
    static constexpr int kF = kBlock / kT;                 // FFTs per workgroup
    static constexpr int kPasses = (BITS + 2) / 3;
    // one point of padding every eight: neither the strided writes nor the reads meet in a bank
    static constexpr int kPitch = kN + (kN + 7) / 8;
    static __device__ __forceinline__ int at(int i) { return i + (i >> 3); }
    static constexpr int radix_bits(int pass) { return BITS / kPasses + (pass < BITS % kPasses); }
    static constexpr int before_bits(int pass) {
        int b = 0;
        for (int p = 0; p < pass; ++p) b += radix_bits(p);
        return b;
    }

    // orders the LDS accesses of an FFT's threads
    static __device__ __forceinline__ void sync() {
        if constexpr (kT > 64) {
            __syncthreads();
        } else {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    }

    // -i v (forward) or i v
    template <bool INV>
    static __device__ __forceinline__ double2 quarter(double2 v) {
        return INV ? make_double2(-v.y, v.x) : make_double2(v.y, -v.x);
    }

    template <bool INV, int R, int S>
    static __device__ __forceinline__ void dft(double2 (&x)[kE], int b) {  // of x[b + S k], k < R
        if constexpr (R == 2) {
            const double2 a = x[b], c = x[b + S];
            x[b] = cadd(a, c);
            x[b + S] = csub(a, c);
        } else if constexpr (R == 4) {
            const double2 a = cadd(x[b], x[b + 2 * S]), c = csub(x[b], x[b + 2 * S]);
            const double2 d = cadd(x[b + S], x[b + 3 * S]), e = quarter<INV>(csub(x[b + S], x[b + 3 * S]));
            x[b] = cadd(a, d);
            x[b + S] = cadd(c, e);
            x[b + 2 * S] = csub(a, d);
            x[b + 3 * S] = csub(c, e);
        } else {
            // two radix-4 butterflies of the even and odd inputs, then radix 2
            dft<INV, 4, 2 * S>(x, b);
            dft<INV, 4, 2 * S>(x, b + S);
            const double h = 0.70710678118654752440;
            const double2 o1 = x[b + 3 * S], o3 = x[b + 7 * S];
            const double2 q1 = quarter<INV>(o1), q3 = quarter<INV>(o3);
            const double2 w0 = x[b + S], w1 = make_double2(h * (o1.x + q1.x), h * (o1.y + q1.y));
            const double2 w2 = quarter<INV>(x[b + 5 * S]), w3 = make_double2(h * (q3.x - o3.x), h * (q3.y - o3.y));
            const double2 e0 = x[b], e1 = x[b + 2 * S], e2 = x[b + 4 * S], e3 = x[b + 6 * S];
            x[b] = cadd(e0, w0);
            x[b + S] = cadd(e1, w1);
            x[b + 2 * S] = cadd(e2, w2);
            x[b + 3 * S] = cadd(e3, w3);
            x[b + 4 * S] = csub(e0, w0);
            x[b + 5 * S] = csub(e1, w1);
            x[b + 6 * S] = csub(e2, w2);
            x[b + 7 * S] = csub(e3, w3);
        }
    }

    static __device__ __forceinline__ void read(double2 (&x)[kE], const double2* X, int t) {
#pragma unroll
        for (int i = 0; i < kE; ++i) x[i] = X[at(t + kT * i)];
    }
    static __device__ __forceinline__ void write(const double2 (&x)[kE], double2* X, int t) {
#pragma unroll
        for (int i = 0; i < kE; ++i) X[at(t + kT * i)] = x[i];
    }

    // pass PASS and those after it, from and to registers; X: the FFT's kPitch points of LDS
    template <bool INV, int PASS>
    static __device__ __forceinline__ void passes(double2 (&x)[kE], double2* X, const double2* __restrict__ tw, int t) {
        constexpr int rb = radix_bits(PASS), R = 1 << rb, lb = before_bits(PASS), L = 1 << lb, NB = kE / R;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if constexpr (PASS > 0) {
                const int u = ((t + kT * b) & (L - 1)) << (BITS - lb - rb);
                double2 w[R];
#pragma unroll
                for (int k = 1; k < R; k *= 2) {
                    w[k] = tw[k * u];
                    if (INV) w[k].y = -w[k].y;
                }
                if constexpr (R >= 4) w[3] = cmul(w[1], w[2]);
                if constexpr (R >= 8) {
                    w[5] = cmul(w[1], w[4]);
                    w[6] = cmul(w[2], w[4]);
                    w[7] = cmul(w[3], w[4]);
                }
#pragma unroll
                for (int k = 1; k < R; ++k) x[b + NB * k] = cmul(w[k], x[b + NB * k]);
            }
            dft<INV, R, NB>(x, b);
        }
        if constexpr (PASS + 1 < kPasses) {
            if constexpr (PASS > 0) sync();  // the points read before this pass
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int j = t + kT * b, u = j & (L - 1), base = ((j - u) << rb) + u;
#pragma unroll
                for (int k = 0; k < R; ++k) X[at(base + k * L)] = x[b + NB * k];
            }
            sync();
            read(x, X, t);
            passes<INV, PASS + 1>(x, X, tw, t);
        }
    }
};

// Two real rows share one complex FFT: with z = x + i y,
//   X_m = (Z_m + conj(Z_{N-m})) / 2,  Y_m = (Z_m - conj(Z_{N-m})) / (2 i),
// and for the inverse, Z = X + i Y of two Hermitian spectra transforms back to
// x + i y.  Rows j and j' = nlat-1-j of a field are the pair in both
// directions, which is also what the Legendre kernels' equatorial symmetry
// needs.  A workgroup takes the pair for kF consecutive fields (four at n = 512), so
// that the per-order outputs (forward) and inputs (inverse) of the group are
// contiguous.

// Rows j and j' (j < nlat/2) of fields b0 .. -> the Gauss-weighted
// even and odd parts of their Fourier coefficients, for m <= T (T < nlon):
//   EO[m][0][j][c] = w_j s_j (F_j + F_j')_m,  EO[m][1][j][c] = w_j s_j (F_j - F_j')_m,
// F = (1/nlon) DFT, c = 2b + {0: re, 1: im}, s_j = rs[j] (rs may be NULL; it
// is symmetric about the equator).  These are the B operands of the forward
// Legendre contraction.  Workgroup g H + j takes field group g.
// Block b of a launch over G field groups x H row pairs -> (g, j). Blocks are
// dispatched to the eight XCDs in turn (b mod 8), so when H is a multiple of 8
// all G groups of row pair j get consecutive blocks of XCD j mod 8: the groups
// read (inverse) or write (forward) disjoint pieces of the same
// spectral-side lines, which then meet in that XCD's L2 instead of being
// fetched or written back once per group. Otherwise the plain g-major split.
__device__ inline void fft_block(int b, int G, int H, int& g, int& j) {
    if ((H & 7) == 0) {
        const int i = b >> 3, q = i / G;
        g = i - q * G;
        j = q * 8 + (b & 7);
    } else {
        g = b / H;
        j = b - g * H;
    }
}

// Both kernels are bound by the memory traffic of rows and orders, the orders in
// pieces of 16 kF bytes; where the launch is one round of workgroups, by the latency
// of loads, passes and stores.  Against radix-2 stage pairs in the LDS with a barrier
// each: whole analysis / synthesis at T1023 on 2048 x 1024, 16 fields 569 -> 510 / 576
// -> 510 us (536 MB in the FFT, 120 us at 4.5 TB/s), T256 on 512 x 256, 12 fields 29.4
// -> 24.9 / 28.6 -> 22.9.
template <int BITS>
__global__ void __launch_bounds__(Fft<BITS>::kBlock) k_fft_forward(const double* __restrict__ grid,
                                                                   double* __restrict__ EO,
                                                                   const double2* __restrict__ tw,
                                                                   const double* __restrict__ wts,
                                                                   const double* __restrict__ rs, int nlat, int T,
                                                                   int C) {
    using F = Fft<BITS>;
    extern __shared__ double2 X[];  // [kF][kPitch]
    const int H = nlat >> 1, nf = C >> 1, tid = threadIdx.x;
    int g, j;
    fft_block(blockIdx.x, (nf + F::kF - 1) / F::kF, H, g, j);
    const int b0 = g * F::kF, f = tid / F::kT, t = tid - f * F::kT;
    double2 x[F::kE];
    {
        const long long fi = min(b0 + f, nf - 1);  // fields past the last one repeat it and store nothing
        const double *north = grid + (fi * nlat + j) * F::kN + t, *south = grid + (fi * nlat + (nlat - 1 - j)) * F::kN + t;
#pragma unroll
        for (int i = 0; i < F::kE; ++i) x[i] = make_double2(north[F::kT * i], south[F::kT * i]);
    }
    double2* Xf = X + f * F::kPitch;
    F::template passes<false, 0>(x, Xf, tw, t);
    F::sync();
    F::write(x, Xf, t);
    __syncthreads();
    const double sc = 0.5 * wts[j] * (rs ? rs[j] : 1.0) / F::kN;
    for (int e = tid; e < (T + 1) * F::kF; e += F::kBlock) {
        const int m = e / F::kF, h = e - m * F::kF;
        if (b0 + h >= nf) continue;
        const double2 z = X[h * F::kPitch + F::at(m)], w = X[h * F::kPitch + F::at((F::kN - m) & (F::kN - 1))];
        // 2 X_m = z + conj(w), 2 Y_m = -i (z - conj(w))
        const double xr2 = z.x + w.x, xi2 = z.y - w.y;
        const double yr2 = z.y + w.y, yi2 = w.x - z.x;
        double* to = EO + (long long)(m * 2) * eo_plane(H, C) + (long long)j * C + 2 * (b0 + h);
        *reinterpret_cast<double2*>(to) = make_double2(sc * (xr2 + yr2), sc * (xi2 + yi2));
        *reinterpret_cast<double2*>(to + eo_plane(H, C)) = make_double2(sc * (xr2 - yr2), sc * (xi2 - yi2));
    }
}

// Fw -> rows j and j' = nlat-1-j (j < nlat/2) of fields b0 .. of the
// grid [B][nlat][nlon], scaled by rs[j] (rs may be NULL); orders m <= T < nlon.
// Bin k of the FFT is A_k + B_{N-k} with A_m = F_m + i G_m, B_m = conj(F_m) + i
// conj(G_m) (m >= 1) of the rows' coefficients F and G (orders past N/2 alias).
template <int BITS>
__global__ void __launch_bounds__(Fft<BITS>::kBlock) k_fft_inverse(const double* __restrict__ Fw,
                                                                   double* __restrict__ grid,
                                                                   const double2* __restrict__ tw,
                                                                   const double* __restrict__ rs, int nlat, int T,
                                                                   int C) {
    using F = Fft<BITS>;
    extern __shared__ double2 X[];  // [kF][kPitch]
    const int H = nlat >> 1, nf = C >> 1, tid = threadIdx.x;
    int g, j;
    fft_block(blockIdx.x, (nf + F::kF - 1) / F::kF, H, g, j);
    const int j2 = nlat - 1 - j, b0 = g * F::kF;
    // bins k and N - k of field h, k <= N/2: kE/2 (and one for N/2) per thread
    constexpr int kI = F::kE / 2 + 1;
    double2 fv[kI], gv[kI];
#pragma unroll
    for (int q = 0; q < kI; ++q) {
        const int e = tid + q * F::kBlock, k = e / F::kF, h = e - k * F::kF;
        const bool ok = k <= F::kN / 2 && k <= T && b0 + h < nf;
        const double* p = Fw + k * fw_plane(nlat, C) + 2 * (b0 + h);
        fv[q] = ok ? *reinterpret_cast<const double2*>(p + (long long)j * C) : make_double2(0.0, 0.0);
        gv[q] = ok ? *reinterpret_cast<const double2*>(p + (long long)j2 * C) : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int q = 0; q < kI; ++q) {
        const int e = tid + q * F::kBlock, k = e / F::kF, h = e - k * F::kF;
        if (k > F::kN / 2) continue;
        double2 v = fv[q], w = gv[q];
        if (k == 0) v.y = w.y = 0.0;  // real fields: Re F_0
        double2 lo = make_double2(v.x - w.y, v.y + w.x), hi = make_double2(v.x + w.y, w.x - v.y);  // A_k, B_k
        if (k == 0) hi = make_double2(0.0, 0.0);
        const int k2 = F::kN - k;
        if (k2 != k && k2 <= T && b0 + h < nf) {  // k >= 1: T < nlon
            const double* p = Fw + k2 * fw_plane(nlat, C) + 2 * (b0 + h);
            v = *reinterpret_cast<const double2*>(p + (long long)j * C);
            w = *reinterpret_cast<const double2*>(p + (long long)j2 * C);
            lo = cadd(lo, make_double2(v.x + w.y, w.x - v.y));
            hi = cadd(hi, make_double2(v.x - w.y, v.y + w.x));
        }
        double2* Xh = X + h * F::kPitch;
        if (k == 0 || k2 == k) Xh[F::at(k)] = cadd(lo, hi);
        else {
            Xh[F::at(k)] = lo;
            Xh[F::at(k2)] = hi;
        }
    }
    __syncthreads();
    const int f = tid / F::kT, t = tid - f * F::kT;
    double2 x[F::kE];
    double2* Xf = X + f * F::kPitch;
    F::read(x, Xf, t);
    if constexpr (F::kPasses > 1) F::sync();
    F::template passes<true, 0>(x, Xf, tw, t);
    if (b0 + f >= nf) return;
    const double sc = rs ? rs[j] : 1.0;
    // streaming stores for the contiguous output rows (measured 22.3 -> 20.5 us
    // at T256, 12 fields; scattered outputs elsewhere measured slower with them)
    double *north = grid + ((long long)(b0 + f) * nlat + j) * F::kN + t,
           *south = grid + ((long long)(b0 + f) * nlat + j2) * F::kN + t;
#pragma unroll
    for (int i = 0; i < F::kE; ++i) {
        __builtin_nontemporal_store(x[i].x * sc, north + F::kT * i);
        __builtin_nontemporal_store(x[i].y * sc, south + F::kT * i);
    }
}

// Legendre contractions with P_n^m generated on the device.  The table
// itself (34 MB at T256) is never stored: P follows from the three-term
// recurrence P_n = s_n Q_n, Q_n = c_n mu Q_{n-1} - Q_{n-2} (the factors s_n are
// applied to the spectral coefficients), restarted from exact host
// values every kRun degrees (and, for the inverse, at the quarters of an order's
// last, shorter segment), which keeps the FP64 recurrence error at a few ulp.
constexpr int kRun = 32;         // degrees per restart row of the table
constexpr int kInvSeg = 4 * kRun;  // degrees per inverse segment (at most; four parts)
constexpr int kInvPad = 8;       // doubles between the parts of a staged segment
constexpr int kFwdDeg = 32;      // degrees per forward run: two 16-row parity tiles
constexpr int kFwdLat = 64;      // latitudes per generated forward block

// Forward work: nrun consecutive 32-degree runs of order m from degree n0,
// first restart row `row` (m = -1: an empty slot).  Inverse work: the latitude
// tiles from t0 on of order m, R per wave; row0 is the order's first restart row.
struct LegRun {
    int m, n0, row, nrun;
};
struct LegWork {
    int m, t0, row0;
};

// FP64 MFMA of four independent 4x4x4 blocks (v_mfma_f64_4x4x4f64): with
// lane = 16 q + 4 b + p, block b takes A[i = p][k = q], B[k = q][j = p] and
// returns D[i = q][j = p] (layout checked on the GPU).  On this part it keeps
// the matrix pipe near its FP64 rate with one or two waves per SIMD, where the
// 16x16x4 shape needs about eight; and four-column groups fit any even column
// count with at most two idle columns.
__device__ __forceinline__ double mfma4(double a, double b, double c) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// Forward: out[b][idx(m, n)] = sum_{j<H} P_n^m(mu_j) EO[m][r][j][c], r the
// parity of n - m (EO holds the Gauss-weighted even / odd Fourier parts),
// over the up to G runs of one work item.  Per block of kFwdLat latitudes, wave g
// generates the 32 degrees of run g, a lane per latitude, into Pt[g][d][lat], one
// barrier, then every wave contracts all runs.
// Wave w = 2 h + r owns degree parity r (16 degrees per run, four groups of 4) and
// the column groups [h NH, h NH + NH) of 4 columns.  Its MFMA blocks split the
// latitude sum: block b of k-step s takes latitudes 16 s + 4 b + q, so a lane's B
// operands are EO[16 s + 4 b + q][column], 4 x NH values per 64 latitudes, held in
// registers for all runs; columns 8 k + 2 p and 8 k + 2 p + 1 of a wave's group pair
// (one 16-byte load), 8 (NH / 2) + p of its last single group.  The four blocks'
// partial sums are added across the row at the end.  The recurrence coefficients
// of a wave's run are uniform and stay in scalar registers.
//
// Bound by the FP64 rate, with the generation (two instructions per value, each
// for up to 32 columns) and the loads of B beside it.  Legendre kernel / whole
// analysis, against one run after the other over blocks of 128 latitudes, with two
// waves generating three-operation recurrences behind readlanes, B reloaded for
// each run by eight-byte loads, and bank conflicts in the operand reads: T1023 on
// 2048 x 1024, 16 fields 579 -> 385 / 761 -> 569 us; T511 on 1024 x 512, 6 fields 46
// -> 39 / 66 -> 59; T256 on 512 x 256, 12 fields 16.9 -> 16.0 / 30.8 -> 29.4.
// Block row y takes columns [y cw, y cw + cw) of the Cs columns, cw <= 32.
template <int NH, int G>
__global__ void __launch_bounds__(256) k_legendre_forward(const LegRun* __restrict__ runs,
                                                          const double* __restrict__ restart,
                                                          const double* __restrict__ coef,
                                                          const double* __restrict__ scale,
                                                          const double* __restrict__ mu,
                                                          const double* __restrict__ EO, double* __restrict__ spec,
                                                          int T, int H, int Cs, int cw) {
    constexpr int kTile = kFwdDeg * kFwdLat, kSteps = kFwdLat / 16;
    __shared__ double Pt[G * kTile];
    const LegRun rn = runs[blockIdx.x];
    if (rn.m < 0) return;  // padding slot of the XCD-ordered list
    const int c_off = blockIdx.y * cw, C = min(cw, Cs - c_off);
    const int m = rn.m, nrun = rn.nrun;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int p = lane & 3, bq = (lane >> 2) & 3, q = lane >> 4;
    const int r = wave & 1, h = wave >> 1;  // degree parity and column half of this wave
    const bool busy = h * NH * 4 < C;        // the wave has columns
    const long long so = spec_offset(T, m);
    const long long ns = nspec_of(T);
    const double* Bsrc = EO + (long long)(m * 2 + r) * eo_plane(H, Cs) + c_off;
    // column of operand g: pairs of groups interleaved, then a single one
    auto column = [&](int g) { return 4 * h * NH + (g < (NH & ~1) ? 8 * (g / 2) + 2 * p + (g & 1) : 4 * g + p); };
    int bcol[(NH + 1) / 2];
#pragma unroll
    for (int k = 0; k < (NH + 1) / 2; ++k) bcol[k] = min(column(2 * k), 2 * k + 1 < NH ? C - 2 : C - 1);
    // generation: run and latitude of this thread
    const int gg = tid / kFwdLat, gl = tid - gg * kFwdLat;
    const bool gen = gg < nrun;  // uniform over a wave
    // recurrence coefficients of the run's degrees, kept in scalar registers (the table
    // is padded: past degree T they are another order's, for rows that nothing stores)
    const int gu = __builtin_amdgcn_readfirstlane(min(gg, nrun - 1));
    const auto cs = (const __attribute__((address_space(4))) double*)(coef + so + (rn.n0 + kFwdDeg * gu + 1 - m));
    double cn[kFwdDeg];
#pragma unroll
    for (int d = 0; d < kFwdDeg; ++d) cn[d] = cs[d];
    const double* rs = restart + (long long)(rn.row + min(gg, nrun - 1)) * 2 * H;
    double pm = 0.0, pc = 0.0, x = 0.0;
    auto fetch = [&](int lb) {
        const int j = min(lb + gl, H - 1);
        const bool ok = gen && lb + gl < H;
        const double a = rs[j], c = rs[H + j];
        pm = ok ? a : 0.0;
        pc = ok ? c : 0.0;
        x = mu[j];
    };
    fetch(0);
    double acc[G][4][NH];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int c = 0; c < NH; ++c) acc[g][d][c] = 0.0;
    // Degree d = 2 (4 k + p) + r keeps latitude l at Pt[g][d][l ^ swz(p)], so that the
    // 32 values which half a wave reads at once (p, two q, bq) lie in different banks.
    // A operand of run g, degree group d, k-step s: row 2 (4 d + p) + r, latitude 16 s + 4 bq + q
    auto swz = [](int pp) { return 2 * (pp & 1) + 16 * (pp >> 1); };
    const double* Ap = Pt + (2 * p + r) * kFwdLat + ((4 * bq + q) ^ (2 * (p & 1)));
    const double *A0 = Ap + 16 * (p >> 1), *A1 = Ap - 16 * (p >> 1);  // even and odd s
    for (int lb = 0; lb < H; lb += kFwdLat) {
        // latitudes past the last one: any value, the generated ones are zero there
        double bf[kSteps][NH];
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            const int row = min(lb + 16 * s + 4 * bq + q, H - 1) * Cs;
#pragma unroll
            for (int k = 0; k < (NH + 1) / 2; ++k) {
                if (2 * k + 1 < NH) {
                    const double2 v = *reinterpret_cast<const double2*>(Bsrc + (row + bcol[k]));
                    bf[s][2 * k] = v.x;
                    bf[s][2 * k + 1] = v.y;
                } else {
                    bf[s][2 * k] = Bsrc[row + bcol[k]];
                }
            }
        }
        __syncthreads();  // the previous tiles are consumed
        if (gen) {
            double* to = Pt + gg * kTile;
#pragma unroll
            for (int d = 0; d < kFwdDeg; ++d) {
                to[d * kFwdLat + (gl ^ swz((d >> 1) & 3))] = pc;  // zero beyond H
                const double nx = fma(cn[d] * x, pc, -pm);
                pm = pc;
                pc = nx;
            }
        }
        fetch(lb + kFwdLat);
        __syncthreads();
        if (!busy) continue;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (g >= nrun) continue;
#pragma unroll
            for (int s = 0; s < kSteps; ++s) {
                double av[4];
#pragma unroll
                for (int d = 0; d < 4; ++d) av[d] = (s & 1 ? A1 : A0)[g * kTile + 8 * d * kFwdLat + 16 * s];
#pragma unroll
                for (int d = 0; d < 4; ++d)
#pragma unroll
                    for (int c = 0; c < NH; ++c) acc[g][d][c] = mfma4(av[d], bf[s][c], acc[g][d][c]);
            }
        }
    }
    // lane 16 q + 4 bq + p holds block bq's partial D[degree q][column p] of each
    // degree group; the row's four blocks are added by two exchanges, and lane bq
    // keeps degree group bq
#pragma unroll
    for (int g = 0; g < G; ++g) {
        double v[NH];
#pragma unroll
        for (int c = 0; c < NH; ++c)
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                double w = acc[g][d][c];
                w += __shfl_xor(w, 4);
                w += __shfl_xor(w, 8);
                v[c] = d == 0 || bq == d ? w : v[c];
            }
        const int n = rn.n0 + kFwdDeg * g + 2 * (4 * bq + q) + r;
        if (!busy || n > T || g >= nrun) continue;
        const double sn = scale[so + (n - m)];
#pragma unroll
        for (int c = 0; c < NH; c += 2) {
            const int col = column(c);
            if (col >= C) continue;
            double* to = spec + (((c_off + col) >> 1) * ns + so + (n - m)) * 2;
            if (c + 1 < NH) *reinterpret_cast<double2*>(to) = make_double2(sn * v[c], sn * v[c + 1]);  // a field's re, im
            else to[col & 1] = sn * v[c];
        }
    }
}

// Inverse: Fw[m][j] = Fe + Fo, Fw[m][j'] = Fe - Fo with Fe / Fo the sums of
// P_n^m(mu_j) S_n over the order's n with n - m even / odd.  A workgroup takes 4 R
// 16-latitude tiles of one order, R per wave, and all its degrees, in segments of
// kInvSeg staged in LDS.  A segment is four parts (kRun degrees each, in an order's
// last segment the shortest multiple of 8 that covers it in four), and the parts
// are the k index of the four-block MFMA: lane 16 kq + i (i < 16) runs the
// recurrence of latitude i over part kq from exact restart values, so no two lanes
// repeat a recurrence and no lane selects values, and per step s it holds
// A_even = P at part degree 2 s and A_odd = P at 2 s + 1 (parts start an even
// number of degrees from m, so the parity of n - m is that of the part degree).
// In the MFMA that lane is A[i & 3][kq] of block i >> 2: latitude i of the
// tile.  The blocks share B, the coefficients of part kq, degree 2 s (+1) and one
// column per p = lane & 3: columns 8 h + 2 p and 8 h + 2 p + 1 of a group pair
// (one 16-byte LDS read), 8 (NG / 2) + p of a last single group.  Result D[q][p] of
// lane 16 q + 4 b + p is latitude 4 b + q and that column.
// The parts are staged kInvPad doubles (and two coefficients) apart, so that the
// four a wave reads at once lie in different banks (the stores that stage a segment
// do meet: with eight groups all degrees of a wave's store lie in one bank, with two
// in four; 3.0e7 conflict cycles a launch at T1023, 16 fields).  Degrees past the segment need
// no checks: their staged columns are zero.
//
// Bound by the FP64 rate, which matrix and vector instructions share (the 4x4x4
// shape reaches 70 of the card's 71.5 TFLOP/s, the 16x16x4 shape 48), plus two
// recurrence instructions per one to eight MFMAs.  Legendre kernel / whole
// synthesis, against one workgroup per segment with the partial sums added
// by the FFT (and the 16x16x4 shape above 128 northern latitudes): T1023 on 2048 x
// 1024, 16 fields 597 -> 369 / 1090 -> 576 us; T511 on 1024 x 512, 6 fields 51 -> 26
// / 88 -> 48; T256 on 512 x 256, 12 fields 19.1 -> 15.2 / 36.3 -> 28.4.
template <int NG, int R>
__global__ void __launch_bounds__(256) k_legendre_inverse(const LegWork* __restrict__ work,
                                                          const double* __restrict__ restart,
                                                          const double* __restrict__ tail,
                                                          const double* __restrict__ coef,
                                                          const double* __restrict__ scale,
                                                          const double* __restrict__ mu,
                                                          const double* __restrict__ spec,
                                                          double* __restrict__ Fw, int T, int nlat, int H, int Cs,
                                                          int cw) {
    constexpr int kCp = 4 * NG, kPart = kRun * kCp + kInvPad;  // pitches of a degree and of a part
    extern __shared__ double Sm[];                             // [4][kPart]
    double* cf = Sm + 4 * kPart;                               // [4][kRun + 2]: degrees 1 .. kRun of a part
    const LegWork wk = work[blockIdx.x];
    if (wk.m < 0) return;  // padding slot of the XCD-ordered list
    const int c_off = blockIdx.y * cw, C = min(cw, Cs - c_off);
    const int m = wk.m, L = T + 1 - m, tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int i = lane & 15, kq = lane >> 4, p = lane & 3;
    const int t = wk.t0 + wave * R;  // first latitude tile of the wave (past the last one: nothing is stored)
    const long long so = spec_offset(T, m), ns = nspec_of(T);
    const int nb = C >> 1;  // fields of this column chunk (C even, c_off even)
    const double* sp = spec + 2 * ((c_off >> 1) * ns + so) + tid;

    // one segment's inputs: double `tid` of every field's run of coefficients (all
    // coalesced), a recurrence coefficient, the lane's restart values
    double v[2 * NG], pv[R], cu[R], x[R];
    double cv, sv;
    const int cpart = tid / kRun, cdeg = tid - cpart * kRun + 1;
    auto fetch = [&](int n0) {
        const int Ls = min(kInvSeg, L - n0), Lp = 8 * ((Ls + 31) / 32);
#pragma unroll
        for (int f = 0; f < 2 * NG; ++f) v[f] = (tid < 2 * Ls && f < nb) ? sp[2 * (f * ns + n0)] : 0.0;
        const int d = cpart * Lp + cdeg;
        cv = (cpart < 4 && d < Ls) ? coef[so + n0 + d] : 0.0;
        sv = tid < 2 * Ls ? scale[so + n0 + (tid >> 1)] : 0.0;
        const double* rs = Ls == kInvSeg ? restart + (long long)(wk.row0 + n0 / kRun + kq) * 2 * H
                                         : tail + (long long)(m * 4 + kq) * 2 * H;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int j = min((t + r) * 16 + i, H - 1);
            pv[r] = rs[j];
            cu[r] = rs[H + j];
        }
    };
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = mu[min((t + r) * 16 + i, H - 1)];
    double ae[R][NG], ao[R][NG];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int g = 0; g < NG; ++g) ae[r][g] = ao[r][g] = 0.0;
    fetch(0);
    for (int n0 = 0; n0 < L; n0 += kInvSeg) {
        const int Ls = min(kInvSeg, L - n0), Lp = 8 * ((Ls + 31) / 32);
        if (n0 > 0) __syncthreads();  // the previous segment is consumed
        {
            const int d = tid >> 1, part = d / Lp;  // degree d of the segment, re / im
            double* to = Sm + part * kPart + (d - part * Lp) * kCp + (tid & 1);
            if (part < 4) {
#pragma unroll
                for (int f = 0; f < 2 * NG; ++f) to[2 * f] = sv * v[f];
            }
            if (cpart < 4) cf[cpart * (kRun + 2) + cdeg - 1] = cv;
        }
        double pa[R], ca[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            pa[r] = pv[r];
            ca[r] = cu[r];
        }
        if (n0 + kInvSeg < L) fetch(n0 + kInvSeg);
        __syncthreads();
        const double* B = Sm + kq * kPart;
        const double* c = cf + kq * (kRun + 2);
        for (int s0 = 0; s0 < Lp; s0 += 8) {
#pragma unroll
            for (int u = 0; u < 8; u += 2) {
                const int s = s0 + u;
                const double2 cc = *reinterpret_cast<const double2*>(c + s);  // degrees s + 1, s + 2
                double a_e[R], a_o[R];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    a_e[r] = ca[r];
                    a_o[r] = fma(cc.x * x[r], ca[r], -pa[r]);
                    ca[r] = fma(cc.y * x[r], a_o[r], -a_e[r]);
                    pa[r] = a_o[r];
                }
                const double* be = B + s * kCp;
                const double* bo = be + kCp;
#pragma unroll
                for (int h = 0; h < NG / 2; ++h) {
                    const double2 e = *reinterpret_cast<const double2*>(be + 8 * h + 2 * p);
                    const double2 o = *reinterpret_cast<const double2*>(bo + 8 * h + 2 * p);
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        ae[r][2 * h] = mfma4(a_e[r], e.x, ae[r][2 * h]);
                        ae[r][2 * h + 1] = mfma4(a_e[r], e.y, ae[r][2 * h + 1]);
                        ao[r][2 * h] = mfma4(a_o[r], o.x, ao[r][2 * h]);
                        ao[r][2 * h + 1] = mfma4(a_o[r], o.y, ao[r][2 * h + 1]);
                    }
                }
                if constexpr (NG & 1) {
                    const double e = be[8 * (NG / 2) + p], o = bo[8 * (NG / 2) + p];
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        ae[r][NG - 1] = mfma4(a_e[r], e, ae[r][NG - 1]);
                        ao[r][NG - 1] = mfma4(a_o[r], o, ao[r][NG - 1]);
                    }
                }
            }
        }
    }
    // streaming stores: they go out while the kernel runs instead of as dirty L2
    // lines written back at its end
    typedef double v2d __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int jj = (t + r) * 16 + 4 * ((lane >> 2) & 3) + kq;
        if (jj >= H) continue;
        double* fn = Fw + m * fw_plane(nlat, Cs) + (long long)jj * Cs + c_off;
        double* fs = Fw + m * fw_plane(nlat, Cs) + (long long)(nlat - 1 - jj) * Cs + c_off;
#pragma unroll
        for (int h = 0; h < NG / 2; ++h) {
            const int col = 8 * h + 2 * p;
            if (col < C) {
                const double *e = &ae[r][2 * h], *o = &ao[r][2 * h];
                __builtin_nontemporal_store(v2d{e[0] + o[0], e[1] + o[1]}, reinterpret_cast<v2d*>(fn + col));
                __builtin_nontemporal_store(v2d{e[0] - o[0], e[1] - o[1]}, reinterpret_cast<v2d*>(fs + col));
            }
        }
        if constexpr (NG & 1) {
            const int col = 8 * (NG / 2) + p;
            if (col < C) {
                __builtin_nontemporal_store(ae[r][NG - 1] + ao[r][NG - 1], fn + col);
                __builtin_nontemporal_store(ae[r][NG - 1] - ao[r][NG - 1], fs + col);
            }
        }
    }
}

// Vector transforms (Eq. (1): V = k x grad(psi) + grad(chi), lap psi = zeta,
// lap chi = delta; Section 3's scaled winds U = u cos(lat), V = v cos(lat)).
// On degree n, lap = -n(n+1)/a^2, and with eps_n = sqrt((n^2 - m^2)/(4n^2 - 1))
// the latitude derivative of the orthonormal P_n^m obeys
//   (1 - mu^2) dP_n^m/dmu = (n + 1) eps_n P_{n-1}^m - n eps_{n+1} P_{n+1}^m,
// so the derivative moves a coefficient one degree up or down and U, V are
// fields of degree T + 1.  Written through zeta and delta directly:
//   U_n = -a [ eps_n zeta_{n-1} / n - eps_{n+1} zeta_{n+1} / (n+1) + i m delta_n / (n(n+1)) ]
//   V_n = -a [ i m zeta_n / (n(n+1)) - eps_n delta_{n-1} / n + eps_{n+1} delta_{n+1} / (n+1) ]
// over m <= n <= T + 1, terms outside m <= degree <= T dropped (the n = 0
// coefficient carries no wind).  Back: with A, B the analyses (degree T + 1)
// of u / cos(lat), v / cos(lat), integration by parts in mu gives
//   zeta_n  = (1/a) [ i m B_n - n eps_{n+1} A_{n+1} + (n+1) eps_n A_{n-1} ]
//   delta_n = (1/a) [ i m A_n + n eps_{n+1} B_{n+1} - (n+1) eps_n B_{n-1} ].
// Layouts: vd pair b at vd + b * stride (zeta, then delta at + nspec(T));
// uvs / ab fields 2b (U or A) and 2b + 1 (V or B) of nspec(T + 1) each.
__device__ __forceinline__ double eps_nm(int n, int m) {
    return sqrt((double)(n * n - m * m) / (4.0 * n * n - 1.0));
}

__global__ void __launch_bounds__(256) k_vd_to_uv_spec(const double2* __restrict__ vd, long long stride,
                                                      double2* __restrict__ uvs, int T, double a) {
    const int m = blockIdx.y, b = blockIdx.z;
    const int n = m + blockIdx.x * blockDim.x + threadIdx.x;
    if (n > T + 1) return;
    const double2* z = vd + b * stride + spec_offset(T, m) - m;  // z[k] = zeta_k^m, m <= k <= T
    const double2* d = z + nspec_of(T);
    double ur = 0.0, ui = 0.0, vr = 0.0, vi = 0.0;
    if (n - 1 >= max(m, 1)) {
        const double e = eps_nm(n, m) / n;
        const double2 zl = z[n - 1], dl = d[n - 1];
        ur += e * zl.x, ui += e * zl.y;
        vr -= e * dl.x, vi -= e * dl.y;
    }
    if (n + 1 <= T) {
        const double e = eps_nm(n + 1, m) / (n + 1);
        const double2 zh = z[n + 1], dh = d[n + 1];
        ur -= e * zh.x, ui -= e * zh.y;
        vr += e * dh.x, vi += e * dh.y;
    }
    if (m > 0 && n <= T) {
        const double f = (double)m / ((double)n * (n + 1));
        const double2 zc = z[n], dc = d[n];
        ur -= f * dc.y, ui += f * dc.x;
        vr -= f * zc.y, vi += f * zc.x;
    }
    const long long ns1 = nspec_of(T + 1), o = spec_offset(T + 1, m) + (n - m);
    uvs[(2LL * b) * ns1 + o] = make_double2(-a * ur, -a * ui);
    uvs[(2LL * b + 1) * ns1 + o] = make_double2(-a * vr, -a * vi);
}

__global__ void __launch_bounds__(256) k_uv_spec_to_vd(const double2* __restrict__ ab, double2* __restrict__ vd,
                                                      long long stride, int T, double a) {
    const int m = blockIdx.y, b = blockIdx.z;
    const int n = m + blockIdx.x * blockDim.x + threadIdx.x;
    if (n > T) return;
    const long long ns1 = nspec_of(T + 1);
    const double2* A = ab + (2LL * b) * ns1 + spec_offset(T + 1, m) - m;  // A[k], m <= k <= T + 1
    const double2* Bv = A + ns1;
    const double2 ac = A[n], bc = Bv[n], ah = A[n + 1], bh = Bv[n + 1];
    const double eh = n * eps_nm(n + 1, m);
    double zr = -m * bc.y - eh * ah.x, zi = m * bc.x - eh * ah.y;
    double dr = -m * ac.y + eh * bh.x, di = m * ac.x + eh * bh.y;
    if (n - 1 >= m) {
        const double el = (n + 1) * eps_nm(n, m);
        const double2 al = A[n - 1], bl = Bv[n - 1];
        zr += el * al.x, zi += el * al.y;
        dr -= el * bl.x, di -= el * bl.y;
    }
    const double ia = 1.0 / a;
    double2* z = vd + b * stride + spec_offset(T, m) + (n - m);
    z[0] = make_double2(zr * ia, zi * ia);
    z[nspec_of(T)] = make_double2(dr * ia, di * ia);
}


size_t inverse_lds(int ng) {
    return sizeof(double) * (4 * (size_t)(kRun * 4 * ng + kInvPad) + 4 * (size_t)(kRun + 2));
}

}  // namespace

namespace {

int device_alloc(void** p, size_t bytes) {
    hipError_t e = hipMalloc(p, bytes ? bytes : 1);
    if (e != hipSuccess) {
        (void)hipGetLastError();  // reported here; a later launch's check would find it again
        return fail(REXI_ENOMEM, std::string("hipMalloc failed: ") + hipGetErrorString(e));
    }
    return REXI_OK;
}

// Restart rows, coefficients and work lists of the Legendre kernels for
// degrees 0..Tt over orders m <= the plan's T.
int leg_build(rexi_plan* pl, LegTables& t, int Tt, const std::vector<double>& north) {
    const int T = pl->T, H = pl->nhalf;
    std::vector<int> run_base;
    std::vector<double> tail;
    std::vector<double> restart = legendre_restarts(Tt, kRun, kInvSeg, north, run_base, tail);
    std::vector<double> lcoef, lscale;
    legendre_coefs(Tt, lcoef, lscale);
    lcoef.resize(lcoef.size() + kFwdDeg + 1, 0.0);  // a forward run reads past the last order
    // forward: one workgroup per G consecutive 32-degree runs of an order: four,
    // which load the order's Fourier block half as often, where that leaves 16
    // workgroups per CU (T1023: 388 us against 398 for two; T511 41.6 against 39.2,
    // T300 18.9 against 16.5, so two there).  Workgroups go to the eight
    // XCDs round-robin by index, so slot s is filled from the queue of XCD
    // s % 8, which holds the runs of the orders m = s (mod 8), longest orders
    // first: all runs of an order share one XCD and its L2, where the order's
    // Fourier block is read from HBM once.  Queues that run out early are
    // padded with empty slots (m = -1).
    constexpr int kXcd = 8;
    int fours = 0;
    for (int m = 0; m <= T; ++m) fours += (Tt - m) / (4 * kFwdDeg) + 1;
    t.fwd_g = fours >= 4096 ? 4 : 2;
    std::vector<std::vector<LegRun>> q(kXcd);
    for (int m = 0; m <= T; ++m) {
        const int nr = (Tt - m) / kFwdDeg + 1;
        for (int r = 0; r < nr; r += t.fwd_g)
            q[m % kXcd].push_back(LegRun{m, m + kFwdDeg * r, run_base[m] + r * (kFwdDeg / kRun),
                                         std::min(t.fwd_g, nr - r)});
    }
    // within a queue, items of more runs before those of fewer (the longest
    // orders still first among equals): the short items fill in at the end
    for (auto& v : q)
        std::stable_sort(v.begin(), v.end(), [](const LegRun& a, const LegRun& b) { return a.nrun > b.nrun; });
    size_t qmax = 0;
    for (auto& v : q) qmax = std::max(qmax, v.size());
    std::vector<LegRun> tf;
    for (size_t k = 0; k < qmax; ++k)
        for (int x = 0; x < kXcd; ++x) tf.push_back(k < q[x].size() ? q[x][k] : LegRun{-1, 0, 0, 0});
    // inverse: 4 R latitude tiles of one order per workgroup; the groups of an order
    // read the same spectral coefficients and go to one XCD, longest orders first.
    // R = 2 reads each staged value for two tiles (the LDS then serves the matrix
    // cores' operands in half their time) where that leaves four workgroups per CU
    std::vector<LegWork> ti;
    const int nl = (H + 15) / 16;
    t.inv_r = (long long)(T + 1) * ((nl + 7) / 8) >= 1024 ? 2 : 1;
    for (int m8 = 0; m8 <= T; m8 += kXcd)
        for (int t0 = 0; t0 < nl; t0 += 4 * t.inv_r)
            for (int m = m8; m < m8 + kXcd; ++m) ti.push_back(m <= T ? LegWork{m, t0, run_base[m]} : LegWork{-1, 0, 0});
    t.T = Tt;
    int rc = device_alloc((void**)&t.d_restart, restart.size() * sizeof(double));
    if (!rc) rc = device_alloc((void**)&t.d_tail, tail.size() * sizeof(double));
    if (!rc) rc = device_alloc((void**)&t.d_lcoef, lcoef.size() * sizeof(double));
    if (!rc) rc = device_alloc((void**)&t.d_lscale, lscale.size() * sizeof(double));
    if (!rc) rc = device_alloc((void**)&t.d_tiles_f, tf.size() * sizeof(LegRun));
    if (!rc) rc = device_alloc((void**)&t.d_tiles_i, ti.size() * sizeof(LegWork));
    if (rc) return rc;
    REXI_HIP(hipMemcpy(t.d_restart, restart.data(), restart.size() * sizeof(double), hipMemcpyHostToDevice));
    REXI_HIP(hipMemcpy(t.d_tail, tail.data(), tail.size() * sizeof(double), hipMemcpyHostToDevice));
    REXI_HIP(hipMemcpy(t.d_lcoef, lcoef.data(), lcoef.size() * sizeof(double), hipMemcpyHostToDevice));
    REXI_HIP(hipMemcpy(t.d_lscale, lscale.data(), lscale.size() * sizeof(double), hipMemcpyHostToDevice));
    REXI_HIP(hipMemcpy(t.d_tiles_f, tf.data(), tf.size() * sizeof(LegRun), hipMemcpyHostToDevice));
    REXI_HIP(hipMemcpy(t.d_tiles_i, ti.data(), ti.size() * sizeof(LegWork), hipMemcpyHostToDevice));
    t.ntiles_f = (int)tf.size();
    t.ntiles_i = (int)ti.size();
    return REXI_OK;
}

void leg_release(LegTables& t) {
    void* ptrs[] = {t.d_restart, t.d_tail, t.d_lcoef, t.d_lscale, t.d_tiles_f, t.d_tiles_i};
    for (void* p : ptrs)
        if (p) (void)hipFree(p);
    t = LegTables{};
}

// One instantiation per length; f(Fft<bits>) for the plan's.
template <class Fn, int BITS = 2>
int with_fft(int nlon, Fn f) {
    if constexpr (BITS > 12) {
        return fail(REXI_EINVAL, "nlon must be a power of two in [4, 4096]");
    } else {
        return nlon == 1 << BITS ? f(std::integral_constant<int, BITS>()) : with_fft<Fn, BITS + 1>(nlon, f);
    }
}

template <int BITS>
constexpr size_t fft_lds() {
    return (size_t)Fft<BITS>::kF * Fft<BITS>::kPitch * sizeof(double2);
}

// grid rows [nf][nlat][nlon] -> EO (C = 2 nf columns), row scale rs or NULL
int fft_forward(rexi_plan* pl, const double* grid, int nf, const double* rs, hipStream_t s) {
    return with_fft(pl->nlon, [&](auto bits) -> int {
        constexpr int kBits = decltype(bits)::value;
        using F = Fft<kBits>;
        hipLaunchKernelGGL(k_fft_forward<kBits>, dim3((nf + F::kF - 1) / F::kF * pl->nhalf), dim3(F::kBlock),
                           fft_lds<kBits>(), s, grid, pl->d_four, pl->d_twiddle, pl->d_wts, rs, pl->nlat, pl->T,
                           2 * nf);
        REXI_HIP(hipGetLastError());
        return REXI_OK;
    });
}

// Fw (C = 2 nf columns) -> grid rows, row scale rs or NULL
int fft_inverse(rexi_plan* pl, double* grid, int nf, const double* rs, hipStream_t s) {
    return with_fft(pl->nlon, [&](auto bits) -> int {
        constexpr int kBits = decltype(bits)::value;
        using F = Fft<kBits>;
        hipLaunchKernelGGL(k_fft_inverse<kBits>, dim3((nf + F::kF - 1) / F::kF * pl->nhalf), dim3(F::kBlock),
                           fft_lds<kBits>(), s, pl->d_four, grid, pl->d_twiddle, rs, pl->nlat, pl->T, 2 * nf);
        REXI_HIP(hipGetLastError());
        return REXI_OK;
    });
}

template <int NH>
void launch_forward(rexi_plan* pl, const LegTables& t, double* spec, int C, int cw, hipStream_t s) {
    const auto k = t.fwd_g == 4 ? k_legendre_forward<NH, 4> : k_legendre_forward<NH, 2>;
    hipLaunchKernelGGL(k, dim3(t.ntiles_f, (C + cw - 1) / cw), dim3(256), 0, s, (const LegRun*)t.d_tiles_f,
                       t.d_restart, t.d_lcoef, t.d_lscale, pl->d_mu, pl->d_four, spec, t.T, pl->nhalf, C, cw);
}

// EO (C columns) -> spec [C/2][nspec(t.T)]; each wave takes half of a workgroup's
// four-column groups
int leg_forward(rexi_plan* pl, const LegTables& t, double* spec, int C, hipStream_t s) {
    using Launcher = void (*)(rexi_plan*, const LegTables&, double*, int, int, hipStream_t);
    static constexpr Launcher of[4] = {launch_forward<1>, launch_forward<2>, launch_forward<3>, launch_forward<4>};
    const int cw = column_chunk(C, 1);
    of[(cw / 4 + 1) / 2 - 1](pl, t, spec, C, cw, s);
    REXI_HIP(hipGetLastError());
    return REXI_OK;
}

template <int NG>
void launch_inverse(rexi_plan* pl, const LegTables& t, const double* spec, int C, int cw, hipStream_t s) {
    const auto k = t.inv_r == 2 ? k_legendre_inverse<NG, 2> : k_legendre_inverse<NG, 1>;
    hipLaunchKernelGGL(k, dim3(t.ntiles_i, (C + cw - 1) / cw), dim3(256), inverse_lds(NG), s,
                       (const LegWork*)t.d_tiles_i, t.d_restart, t.d_tail, t.d_lcoef, t.d_lscale, pl->d_mu, spec,
                       pl->d_four, t.T, pl->nlat, pl->nhalf, C, cw);
}

// spec [C/2][nspec(t.T)] -> Fw (C columns)
int leg_inverse(rexi_plan* pl, const LegTables& t, const double* spec, int C, hipStream_t s) {
    using Launcher = void (*)(rexi_plan*, const LegTables&, const double*, int, int, hipStream_t);
    static constexpr Launcher of[8] = {launch_inverse<1>, launch_inverse<2>, launch_inverse<3>, launch_inverse<4>,
                                       launch_inverse<5>, launch_inverse<6>, launch_inverse<7>, launch_inverse<8>};
    const int cw = inverse_columns(C, t.inv_r, t.ntiles_i);
    of[cw / 4 - 1](pl, t, spec, C, cw, s);
    REXI_HIP(hipGetLastError());
    return REXI_OK;
}

}  // namespace

int sh_setup(rexi_plan* pl) {
    const int T = pl->T, nlat = pl->prm.nlat, nlon = pl->prm.nlon;
    // the plan's parameter check has already refused these (before allocating)
    if (nlat % 2 || nlat > 2048 || nlon > 4096) return fail(REXI_EINVAL, "grid outside the supported range");
    pl->nlat = nlat;
    pl->nlon = nlon;
    pl->nhalf = nlat / 2;
    const int H = pl->nhalf;
    gauss_legendre(nlat, pl->mu, pl->w);
    std::vector<double> north(pl->mu.begin(), pl->mu.begin() + H);
    std::vector<double> wn(pl->w.begin(), pl->w.begin() + H);
    std::vector<double> rcos(nlat);
    for (int j = 0; j < nlat; ++j) {
        const long double x = pl->mu[j];
        rcos[j] = (double)(1.0L / sqrtl((1.0L - x) * (1.0L + x)));
    }
    std::vector<double2> tw(nlon / 2);
    const long double pi = 3.141592653589793238462643383279502884L;
    for (int k = 0; k < nlon / 2; ++k) {
        const long double a = -2 * pi * k / nlon;
        tw[k] = make_double2((double)cosl(a), (double)sinl(a));
    }
    int rc = leg_build(pl, pl->leg, T, north);
    if (!rc) rc = leg_build(pl, pl->legv, T + 1, north);
    if (!rc) rc = device_alloc((void**)&pl->d_mu, north.size() * sizeof(double));
    if (!rc) rc = device_alloc((void**)&pl->d_wts, wn.size() * sizeof(double));
    if (!rc) rc = device_alloc((void**)&pl->d_rcos, rcos.size() * sizeof(double));
    if (!rc) rc = device_alloc((void**)&pl->d_twiddle, tw.size() * sizeof(double2));
    // Fourier workspace: (T + 1) x 2 EO planes or T + 1 order planes, each padded by kFourPad
    if (!rc)
        rc = device_alloc((void**)&pl->d_four,
                          (size_t)(T + 1) * (nlat * 2 * pl->prm.max_fields + 2 * kFourPad) * sizeof(double));
    if (!rc && pl->prm.max_fields >= 2)
        rc = device_alloc((void**)&pl->d_vspec, (size_t)pl->prm.max_fields * nspec_of(T + 1) * sizeof(double2));
    if (rc) return rc;
    REXI_HIP(hipMemcpy(pl->d_mu, north.data(), north.size() * sizeof(double), hipMemcpyHostToDevice));
    REXI_HIP(hipMemcpy(pl->d_wts, wn.data(), wn.size() * sizeof(double), hipMemcpyHostToDevice));
    REXI_HIP(hipMemcpy(pl->d_rcos, rcos.data(), rcos.size() * sizeof(double), hipMemcpyHostToDevice));
    REXI_HIP(hipMemcpy(pl->d_twiddle, tw.data(), tw.size() * sizeof(double2), hipMemcpyHostToDevice));
    // dynamic LDS above 64 KB per workgroup
    static_assert(fft_lds<11>() == fft_lds<12>());
    for (const void* f : {(const void*)k_fft_forward<11>, (const void*)k_fft_inverse<11>,
                          (const void*)k_fft_forward<12>, (const void*)k_fft_inverse<12>})
        REXI_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)fft_lds<12>()));
    return REXI_OK;
}

void sh_release(rexi_plan* pl) {
    leg_release(pl->leg);
    leg_release(pl->legv);
    void* ptrs[] = {pl->d_mu, pl->d_wts, pl->d_rcos, pl->d_twiddle, pl->d_four, pl->d_vspec};
    for (void* p : ptrs)
        if (p) (void)hipFree(p);
    pl->d_mu = nullptr;
    pl->d_wts = nullptr;
    pl->d_rcos = nullptr;
    pl->d_twiddle = nullptr;
    pl->d_four = nullptr;
    pl->d_vspec = nullptr;
}

static bool overlaps(const void* a, size_t na, const void* b, size_t nb) {
    const char* x = (const char*)a;
    const char* y = (const char*)b;
    return x < y + nb && y < x + na;
}

int sh_run(rexi_plan* pl, const void* in, void* out, int B, bool forward, hipStream_t s) {
    if (pl->nlat == 0) return fail(REXI_EUNSUPPORTED, "plan was created without a grid (nlat = nlon = 0)");
    if (!in || !out) return fail(REXI_EINVAL, "NULL pointer");
    if (B < 1) return fail(REXI_EINVAL, "B must be >= 1");
    if (B > pl->prm.max_fields) return fail(REXI_EUNSUPPORTED, "B exceeds the plan's max_fields");
    const size_t gbytes = (size_t)B * pl->nlat * pl->nlon * sizeof(double);
    const size_t sbytes = (size_t)B * pl->nspec * 16;
    if (overlaps(in, forward ? gbytes : sbytes, out, forward ? sbytes : gbytes))
        return fail(REXI_EALIAS, "output overlaps input");
    const int C = 2 * B;
    int rc;
    if (forward) {
        if ((rc = fft_forward(pl, (const double*)in, B, nullptr, s))) return rc;
        REXI_HIP(timed_begin(pl, REXI_KERNEL_LEGENDRE_FWD, s));
        if ((rc = leg_forward(pl, pl->leg, (double*)out, C, s))) return rc;
        REXI_HIP(timed_end(pl, REXI_KERNEL_LEGENDRE_FWD, s));
    } else {
        REXI_HIP(timed_begin(pl, REXI_KERNEL_LEGENDRE_INV, s));
        if ((rc = leg_inverse(pl, pl->leg, (const double*)in, C, s))) return rc;
        REXI_HIP(timed_end(pl, REXI_KERNEL_LEGENDRE_INV, s));
        if ((rc = fft_inverse(pl, (double*)out, B, nullptr, s))) return rc;
    }
    return REXI_OK;
}

// Vector transforms: vd pairs (zeta, delta) at stride `stride` complex entries
// <-> winds uv [B][2][nlat][nlon].  Through the degree-(T+1) fields of
// u / cos(lat), v / cos(lat) (forward) or u cos(lat), v cos(lat) (inverse) in
// d_vspec; the 1 / cos(lat) row scale is applied inside the FFT kernels.
int sh_vec_run(rexi_plan* pl, const void* in, void* out, long long stride, int B, bool to_uv, hipStream_t s) {
    if (pl->nlat == 0) return fail(REXI_EUNSUPPORTED, "plan was created without a grid (nlat = nlon = 0)");
    if (!in || !out) return fail(REXI_EINVAL, "NULL pointer");
    if (B < 1) return fail(REXI_EINVAL, "B must be >= 1");
    if (stride < 2 * pl->nspec) return fail(REXI_EINVAL, "stride must be at least 2 nspec");
    if (2LL * B > pl->prm.max_fields) return fail(REXI_EUNSUPPORTED, "2 B exceeds the plan's max_fields");
    const size_t gbytes = (size_t)2 * B * pl->nlat * pl->nlon * sizeof(double);
    const size_t sbytes = ((size_t)(B - 1) * stride + 2 * (size_t)pl->nspec) * 16;
    if (overlaps(in, to_uv ? sbytes : gbytes, out, to_uv ? gbytes : sbytes))
        return fail(REXI_EALIAS, "output overlaps input");
    const int T = pl->T;
    const int C = 4 * B;
    const dim3 grid((T + 2 + 255) / 256, T + 1, B);
    int rc;
    if (to_uv) {
        hipLaunchKernelGGL(k_vd_to_uv_spec, grid, dim3(256), 0, s, (const double2*)in, stride, pl->d_vspec, T,
                           pl->prm.radius);
        REXI_HIP(hipGetLastError());
        if ((rc = leg_inverse(pl, pl->legv, (const double*)pl->d_vspec, C, s))) return rc;
        if ((rc = fft_inverse(pl, (double*)out, 2 * B, pl->d_rcos, s))) return rc;
    } else {
        if ((rc = fft_forward(pl, (const double*)in, 2 * B, pl->d_rcos, s))) return rc;
        if ((rc = leg_forward(pl, pl->legv, (double*)pl->d_vspec, C, s))) return rc;
        hipLaunchKernelGGL(k_uv_spec_to_vd, grid, dim3(256), 0, s, (const double2*)pl->d_vspec, (double2*)out,
                           stride, T, pl->prm.radius);
        REXI_HIP(hipGetLastError());
    }
    return REXI_OK;
}

}  // namespace rexi
