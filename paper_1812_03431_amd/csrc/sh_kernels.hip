// Spherical-harmonic transforms on gfx950 (Section 3).
//
// Analysis:  xi_n^m = sum_j w_j P_n^m(mu_j) F_j^m,  F_j^m = (1/nlon) sum_k xi(mu_j, lam_k) e^{-i m lam_k}
// Synthesis: xi(mu_j, lam_k) = sum_m c_m Re( sum_n xi_n^m P_n^m(mu_j) e^{i m lam_k} ), c_0 = 1, c_m = 2
// (the m = 0 term uses Re(xi_n^0)).
//
// Longitude: one workgroup per pair of grid rows j, j' = nlat-1-j runs one
// complex FFT of length nlon (radix-2 stages taken in pairs) in LDS for both
// rows.  Latitude: per
// zonal order m the Legendre sum is a small dense contraction (T+1-m degrees
// x nlat/2 latitudes x 2B real columns) and runs on FP64 MFMA
// (v_mfma_f64_16x16x4f64).  Gauss latitudes are symmetric about the equator
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

#include "internal.hpp"

namespace rexi {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));


__device__ __forceinline__ int bitrev(int x, int bits) { return (int)(__brev((unsigned)x) >> (32 - bits)); }

// Plane strides of the Fourier workspace, in doubles: an EO plane [j][c] of one
// (order, parity) and an order's plane [row][c] are padded by kFourPad so that
// the lines of consecutive planes are not a power of two apart.
constexpr int kFourPad = 32;
__host__ __device__ __forceinline__ long long eo_plane(int H, int C) { return (long long)H * C + kFourPad; }
__host__ __device__ __forceinline__ long long fw_plane(int nlat, int C) { return (long long)nlat * C + kFourPad; }

__device__ __forceinline__ double2 cmul(double2 w, double2 v) {
    return make_double2(fma(w.x, v.x, -w.y * v.y), fma(w.x, v.y, w.y * v.x));
}

__device__ __forceinline__ double2 twiddle(const double2* tw, int k, bool inverse) {
    double2 w = tw[k];
    if (inverse) w.y = -w.y;
    return w;
}

// In-place decimation-in-time FFTs of nb arrays X + f n, f < nb, in LDS (input
// already in bit-reversed order); n = 2^bits.  tw[k] = exp(-2 pi i k / n),
// k < n/2; conj for the inverse direction.  Two radix-2 stages at a time: the
// butterflies of half-lengths h and 2h over the four elements pos + {0, h, 2h,
// 3h} of a block of 4h are one radix-4 step with the same arithmetic and
// twiddles, so a stage pair needs one barrier instead of two.  An odd number of
// stages starts with one radix-2 stage.  The FFTs are bound by the latency of
// their barrier-separated stages (11 -> 6 barriers at n = 2048).
__device__ void fft_lds(double2* X, const double2* tw, int bits, int nb, bool inverse) {
    const int n = 1 << bits, hb = bits - 1;
    int lh = 0;  // half-length 2^lh of the next radix-2 stage
    if (bits & 1) {
        const double2 w = twiddle(tw, 0, inverse);
        for (int t = threadIdx.x; t < (nb << hb); t += blockDim.x) {
            const int i = 2 * t, j = i + 1;
            const double2 u = X[i], v = cmul(w, X[j]);
            X[i] = make_double2(u.x + v.x, u.y + v.y);
            X[j] = make_double2(u.x - v.x, u.y - v.y);
        }
        __syncthreads();
        lh = 1;
    }
    for (; lh + 2 <= bits; lh += 2) {
        const int h = 1 << lh, q = hb - 1;  // n/4 = 2^q radix-4 steps per array
        for (int t = threadIdx.x; t < (nb << q); t += blockDim.x) {
            const int f = t >> q, tt = t & ((1 << q) - 1);
            const int grp = tt >> lh, pos = tt & (h - 1);
            const int i0 = f * n + (grp << (lh + 2)) + pos, i1 = i0 + h, i2 = i1 + h, i3 = i2 + h;
            const double2 w1 = twiddle(tw, pos << (hb - lh), inverse);
            const double2 w2 = twiddle(tw, pos << (q - lh), inverse);
            const double2 w3 = twiddle(tw, (pos + h) << (q - lh), inverse);
            const double2 a0 = X[i0], a2 = X[i2];
            const double2 t1 = cmul(w1, X[i1]), t3 = cmul(w1, X[i3]);
            const double2 c0 = make_double2(a0.x + t1.x, a0.y + t1.y), c1 = make_double2(a0.x - t1.x, a0.y - t1.y);
            const double2 c2 = make_double2(a2.x + t3.x, a2.y + t3.y), c3 = make_double2(a2.x - t3.x, a2.y - t3.y);
            const double2 u = cmul(w2, c2), v = cmul(w3, c3);
            X[i0] = make_double2(c0.x + u.x, c0.y + u.y);
            X[i2] = make_double2(c0.x - u.x, c0.y - u.y);
            X[i1] = make_double2(c1.x + v.x, c1.y + v.y);
            X[i3] = make_double2(c1.x - v.x, c1.y - v.y);
        }
        __syncthreads();
    }
}

// Two real rows share one complex FFT: with z = x + i y,
//   X_m = (Z_m + conj(Z_{N-m})) / 2,  Y_m = (Z_m - conj(Z_{N-m})) / (2 i),
// and for the inverse, Z = X + i Y of two Hermitian spectra transforms back to
// x + i y.  Rows j and j' = nlat-1-j of a field are the pair in both
// directions, which is also what the Legendre kernels' equatorial symmetry
// needs.  A workgroup takes the pair for a group of up to nb fields, so that
// the per-order outputs (forward) and inputs (inverse) of the group are
// contiguous.

// Rows j and j' (j < nlat/2) of fields b0 .. b0+nbr-1 -> the Gauss-weighted
// even and odd parts of their Fourier coefficients, for m <= T (T < nlon):
//   EO[m][0][j][c] = w_j s_j (F_j + F_j')_m,  EO[m][1][j][c] = w_j s_j (F_j - F_j')_m,
// F = (1/nlon) DFT, c = 2b + {0: re, 1: im}, s_j = rs[j] (rs may be NULL; it
// is symmetric about the equator).  These are the B operands of the forward
// Legendre contraction.  Workgroup g H + j takes field group g.
// Block b of a launch over G field groups x H row pairs -> (g, j). Blocks are
// dispatched to the eight XCDs in turn (b mod 8), so when H is a multiple of 8
// all G groups of row pair j get consecutive blocks of XCD j mod 8: the groups
// read (inverse) or write (forward) disjoint 16-byte pieces of the same
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

__global__ void __launch_bounds__(256) k_fft_forward(const double* __restrict__ grid, double* __restrict__ EO,
                                                     const double2* __restrict__ tw, const double* __restrict__ wts,
                                                     const double* __restrict__ rs, int nlat, int nlon, int bits,
                                                     int T, int C, int nb) {
    extern __shared__ double2 X[];  // [nb][nlon] data, then [nlon/2] twiddles
    const int H = nlat >> 1, nf = C >> 1;
    int g, j;
    fft_block(blockIdx.x, (nf + nb - 1) / nb, H, g, j);
    const int b0 = g * nb, nbr = min(nb, nf - b0);
    double2* tws = X + nb * nlon;
    for (int k = threadIdx.x; k < nlon / 2; k += blockDim.x) tws[k] = tw[k];
    constexpr int kU = 8;  // all loads of a thread issued before its stores
    const int tot = nbr * nlon;
    for (int k0 = 0; k0 < tot; k0 += kU * 256) {
        double vx[kU], vy[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int e = min(k0 + u * 256 + threadIdx.x, tot - 1);
            const int f = e >> bits, k = e & (nlon - 1);
            vx[u] = grid[((long long)(b0 + f) * nlat + j) * nlon + k];
            vy[u] = grid[((long long)(b0 + f) * nlat + (nlat - 1 - j)) * nlon + k];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int e = k0 + u * 256 + threadIdx.x;
            if (e < tot) {
                const int f = e >> bits, k = e & (nlon - 1);
                X[f * nlon + bitrev(k, bits)] = make_double2(vx[u], vy[u]);
            }
        }
    }
    __syncthreads();
    fft_lds(X, tws, bits, nbr, false);
    const double sc = 0.5 * wts[j] * (rs ? rs[j] : 1.0) / nlon;
    for (int m = threadIdx.x; m <= T; m += blockDim.x) {
        double* e = EO + (long long)(m * 2) * eo_plane(H, C) + (long long)j * C + 2 * b0;
        double* o = e + eo_plane(H, C);
        for (int f = 0; f < nbr; ++f) {
            const double2 z = X[f * nlon + m], w = X[f * nlon + (nlon - m) % nlon];
            // 2 X_m = z + conj(w), 2 Y_m = -i (z - conj(w))
            const double xr2 = z.x + w.x, xi2 = z.y - w.y;
            const double yr2 = z.y + w.y, yi2 = w.x - z.x;
            e[2 * f] = sc * (xr2 + yr2);
            e[2 * f + 1] = sc * (xi2 + yi2);
            o[2 * f] = sc * (xr2 - yr2);
            o[2 * f + 1] = sc * (xi2 - yi2);
        }
    }
}

// Fw -> rows j and j' = nlat-1-j (j < nlat/2) of fields b0 .. b0+nbr-1 of the
// grid [B][nlat][nlon], scaled by rs[j] (rs may be NULL); orders m <= T < 1024.
__global__ void __launch_bounds__(256) k_fft_inverse(const double* __restrict__ Fw, double* __restrict__ grid, const double2* __restrict__ tw,
                                                     const double* __restrict__ rs, int nlat, int nlon, int bits,
                                                     int T, int C, int nb) {
    extern __shared__ double2 X[];  // [nb][nlon] data, then [nlon/2] twiddles
    const int H = nlat >> 1, nf = C >> 1;
    int g, j;
    fft_block(blockIdx.x, (nf + nb - 1) / nb, H, g, j);
    const int j2 = nlat - 1 - j;
    const int b0 = g * nb, nbr = min(nb, nf - b0);
    double2* tws = X + nb * nlon;
    for (int k = threadIdx.x; k < nb * nlon; k += blockDim.x) X[k] = make_double2(0.0, 0.0);
    for (int k = threadIdx.x; k < nlon / 2; k += blockDim.x) tws[k] = tw[k];
    __syncthreads();
    for (int f = 0; f < nbr; ++f) {
        double2* Xf = X + f * nlon;
        const int cb = 2 * (b0 + f);
        constexpr int kM = 4;  // orders per thread: m = tid + 256 k
        double2 fv[kM], gv[kM];  // coefficients of rows j and j'
#pragma unroll
        for (int k = 0; k < kM; ++k) {
            const int m = threadIdx.x + 256 * k;
            double2 v = make_double2(0.0, 0.0), w = v;
            if (m <= T) {
                const double* p = Fw + m * fw_plane(nlat, C) + cb;
                v = make_double2(p[(long long)j * C], p[(long long)j * C + 1]);
                w = make_double2(p[(long long)j2 * C], p[(long long)j2 * C + 1]);
                if (m == 0) v.y = w.y = 0.0;  // real fields: Re F_0
            }
            fv[k] = v;
            gv[k] = w;
        }
        // Z = X + i Y with X[m] = F_m, X[N-m] = conj(F_m) (and Y alike from G):
        // Z[m] += F_m + i G_m, Z[N-m] += conj(F_m) + i conj(G_m); two passes, as
        // orders past N/2 alias onto the same bins
#pragma unroll
        for (int k = 0; k < kM; ++k) {
            const int m = threadIdx.x + 256 * k;
            if (m <= T) Xf[m % nlon] = make_double2(fv[k].x - gv[k].y, fv[k].y + gv[k].x);
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kM; ++k) {
            const int m = threadIdx.x + 256 * k;
            if (m >= 1 && m <= T) {
                const int q = (nlon - m % nlon) % nlon;
                Xf[q] = make_double2(Xf[q].x + fv[k].x + gv[k].y, Xf[q].y - fv[k].y + gv[k].x);
            }
        }
        __syncthreads();
    }
    // bit-reverse permutation in place
    for (int e = threadIdx.x; e < nbr * nlon; e += blockDim.x) {
        const int f = e >> bits, k = e & (nlon - 1);
        const int r = bitrev(k, bits);
        if (r > k) {
            const double2 t = X[f * nlon + k];
            X[f * nlon + k] = X[f * nlon + r];
            X[f * nlon + r] = t;
        }
    }
    __syncthreads();
    fft_lds(X, tws, bits, nbr, true);
    const double sc = rs ? rs[j] : 1.0;
    // streaming stores for the contiguous output rows (measured 22.3 -> 20.5 us
    // at T256, 12 fields; scattered outputs elsewhere measured slower with them)
    for (int e = threadIdx.x; e < nbr * nlon; e += blockDim.x) {
        const int f = e >> bits, k = e & (nlon - 1);
        const double2 z = X[e];
        __builtin_nontemporal_store(z.x * sc, grid + ((long long)(b0 + f) * nlat + j) * nlon + k);
        __builtin_nontemporal_store(z.y * sc, grid + ((long long)(b0 + f) * nlat + j2) * nlon + k);
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
// Columns [c_off, c_off + C) of EO (row stride Cs), C <= 32.
template <int NH, int G>
__global__ void __launch_bounds__(256) k_legendre_forward(const LegRun* __restrict__ runs,
                                                          const double* __restrict__ restart,
                                                          const double* __restrict__ coef,
                                                          const double* __restrict__ scale,
                                                          const double* __restrict__ mu,
                                                          const double* __restrict__ EO, double* __restrict__ spec,
                                                          int T, int H, int Cs, int c_off, int C) {
    constexpr int kTile = kFwdDeg * kFwdLat, kSteps = kFwdLat / 16;
    __shared__ double Pt[G * kTile];
    const LegRun rn = runs[blockIdx.x];
    if (rn.m < 0) return;  // padding slot of the XCD-ordered list
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
// four a wave reads at once lie in different banks.  Degrees past the segment need
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
                                                          int c_off, int C) {
    constexpr int kCp = 4 * NG, kPart = kRun * kCp + kInvPad;  // pitches of a degree and of a part
    extern __shared__ double Sm[];                             // [4][kPart]
    double* cf = Sm + 4 * kPart;                               // [4][kRun + 2]: degrees 1 .. kRun of a part
    const LegWork wk = work[blockIdx.x];
    if (wk.m < 0) return;  // padding slot of the XCD-ordered list
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
    if (e != hipSuccess) return fail(REXI_ENOMEM, std::string("hipMalloc failed: ") + hipGetErrorString(e));
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
    while (!tf.empty() && tf.back().m < 0) tf.pop_back();
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

constexpr size_t kFftLds = 96 * 1024;  // LDS allowance of the FFT kernels (nlon = 4096 needs 96 KB)

int fft_bits(int nlon) {
    int bits = 0;
    while ((1 << bits) < nlon) ++bits;
    return bits;
}

// grid rows [nf][nlat][nlon] -> Fw (C = 2 nf columns), row scale rs or NULL
// Fields per FFT workgroup.  One: the FFTs are latency-bound per workgroup,
// and four fields per workgroup (contiguous per-order writes, a quarter of the
// workgroups) measured slower at T256, 12 fields (22.4 / 30.7 us against
// 16.5 / 20.9 us forward / inverse).
int fft_group(const rexi_plan*, int) { return 1; }

int fft_forward(rexi_plan* pl, const double* grid, int nf, const double* rs, hipStream_t s) {
    const int nb = fft_group(pl, nf);
    const size_t lds = (size_t)(nb * pl->nlon + pl->nlon / 2) * sizeof(double2);
    hipLaunchKernelGGL(k_fft_forward, dim3(((nf + nb - 1) / nb) * pl->nhalf), dim3(256), lds, s, grid, pl->d_four,
                       pl->d_twiddle, pl->d_wts, rs, pl->nlat, pl->nlon, fft_bits(pl->nlon), pl->T, 2 * nf, nb);
    REXI_HIP(hipGetLastError());
    return REXI_OK;
}

int fft_inverse(rexi_plan* pl, double* grid, int nf, const double* rs, hipStream_t s) {
    const int nb = fft_group(pl, nf);
    const size_t lds = (size_t)(nb * pl->nlon + pl->nlon / 2) * sizeof(double2);
    hipLaunchKernelGGL(k_fft_inverse, dim3(((nf + nb - 1) / nb) * pl->nhalf), dim3(256), lds, s, pl->d_four,
                       grid, pl->d_twiddle, rs, pl->nlat, pl->nlon, fft_bits(pl->nlon), pl->T, 2 * nf, nb);
    REXI_HIP(hipGetLastError());
    return REXI_OK;
}

template <int NH>
void launch_forward(rexi_plan* pl, const LegTables& t, double* spec, int C, int c0, int w, hipStream_t s) {
    const auto k = t.fwd_g == 4 ? k_legendre_forward<NH, 4> : k_legendre_forward<NH, 2>;
    hipLaunchKernelGGL(k, dim3(t.ntiles_f), dim3(256), 0, s, (const LegRun*)t.d_tiles_f, t.d_restart, t.d_lcoef,
                       t.d_lscale, pl->d_mu, pl->d_four, spec, t.T, pl->nhalf, C, c0, w);
}

// EO (C columns) -> spec [C/2][nspec(t.T)], in launches of at most 32 columns;
// each wave takes half of a launch's four-column groups
int leg_forward(rexi_plan* pl, const LegTables& t, double* spec, int C, hipStream_t s) {
    using Launcher = void (*)(rexi_plan*, const LegTables&, double*, int, int, int, hipStream_t);
    static constexpr Launcher of[4] = {launch_forward<1>, launch_forward<2>, launch_forward<3>, launch_forward<4>};
    for (int c0 = 0; c0 < C; c0 += 32) {
        const int w = std::min(32, C - c0);
        of[((w + 3) / 4 + 1) / 2 - 1](pl, t, spec, C, c0, w, s);
        REXI_HIP(hipGetLastError());
    }
    return REXI_OK;
}

template <int NG>
void launch_inverse(rexi_plan* pl, const LegTables& t, const double* spec, int C, int c0, int w, hipStream_t s) {
    const auto k = t.inv_r == 2 ? k_legendre_inverse<NG, 2> : k_legendre_inverse<NG, 1>;
    hipLaunchKernelGGL(k, dim3(t.ntiles_i), dim3(256), inverse_lds(NG), s, (const LegWork*)t.d_tiles_i, t.d_restart,
                       t.d_tail, t.d_lcoef, t.d_lscale, pl->d_mu, spec, pl->d_four, t.T,
                       pl->nlat, pl->nhalf, C, c0, w);
}

// spec [C/2][nspec(t.T)] -> Fw (C columns), in launches of at most 32 columns
// (up to eight four-column groups)
int leg_inverse(rexi_plan* pl, const LegTables& t, const double* spec, int C, hipStream_t s) {
    using Launcher = void (*)(rexi_plan*, const LegTables&, const double*, int, int, int, hipStream_t);
    static constexpr Launcher of[8] = {launch_inverse<1>, launch_inverse<2>, launch_inverse<3>, launch_inverse<4>,
                                       launch_inverse<5>, launch_inverse<6>, launch_inverse<7>, launch_inverse<8>};
    for (int c0 = 0; c0 < C; c0 += 32) {
        const int w = std::min(32, C - c0);
        of[(w + 3) / 4 - 1](pl, t, spec, C, c0, w, s);
        REXI_HIP(hipGetLastError());
    }
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
    REXI_HIP(hipFuncSetAttribute((const void*)k_fft_forward, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kFftLds));
    REXI_HIP(hipFuncSetAttribute((const void*)k_fft_inverse, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kFftLds));

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
