// The fused T-REXI step with one pole per lane (gfx950).
//
// Same sum over poles as rexi_kernels.hip: a lane solves a whole tridiagonal
// chain for its pole by plain elimination (no partitioning, no cross-lane
// reduction of interface unknowns), 64 poles per wave.  A step is k_sweep (or
// k_sweep_short) and k_sweep_reduce.
//
// Real form.  With zeta = i zeta', Phi = i Phi' the shifted operator of a chain
// is alpha + i dt H with H real symmetric: off-diagonals i c_t, diagonal
// alpha + i th (vorticity) and alpha + i th + om^2/alpha (divergence, Phi'
// eliminated: Phi' = (r_Phi' - i om delta)/alpha).  A complex right-hand side
// splits into two real ones (a, b), and the minus-sign solves are conjugates of
// the plus-sign solves of real data at the conjugate pole, which is again in
// the list.  With X_a, X_b the solutions at pole k and wx, wy the weight pair
// of the pole (see rexi_kernels.hip), W1 = wx + wy, W2 = wx - wy:
//   Re y = sum_k Re(W1 X_a) - Im(W2 X_b),  Im y = sum_k Im(W2 X_a) + Re(W1 X_b),
// and the same with V = -i W / alpha for the Phi' sums.
//
// Scaling.  x = D x~ with D_t D_{t+1} = 1/c_{t+1} makes every off-diagonal i:
//   pivots   b_t = D2 alpha + i th' (+ om2' / alpha) + q_{t-1},  q_t = 1/b_t
//   forward  F_t = g_t - i q_{t-1} F_{t-1}
//   backward x_t = q_t (F_t - i x_{t+1})
// Chains alternate vorticity and divergence; a chain that would start with a
// divergence gets a dummy vorticity in front, and its end is padded to whole
// groups of two pairs, with D2 = kDummy: a pivot so large that the dummy's
// contribution to its neighbour rounds away.
//
// Uniform data.  All lanes of a wave are at the same chain position, so the
// operator constants and the right-hand sides are scalar loads and every FMA
// takes them from scalar registers.
//
// Memory.  Elimination needs every forward value again in the backward sweep,
// 16 bytes per right-hand side, element and pole: too much for registers, and
// tens of GB for HBM.  So the chain is cut into blocks of kBlk pairs: pass 1 runs
// forward and keeps only the pivot and the forward values at the block
// boundaries (global scratch, 16 (1 + 2 states) bytes per lane and block), pass 2
// takes the blocks in reverse, repeats the forward sweep of one block into
// registers and substitutes back.  Pass 1 needs the block-end values alone, a sum
// of products of the (real, uniform) right-hand sides with per-pole coefficients
// that all states share.
//
// What bounds it.  FP64 issue: a pair of elements takes 140 FP64 instructions and
// four reciprocals with one state, some 720 cycles of a SIMD.  At T127 with 8215
// poles that is 75% of the time (482 us; 478 without the scalar loads' misses, 446
// without the LDS).  With four states at T256 and 2071 poles the instructions alone
// take 0.98 of 1.53 ms; the rest is waits that two waves per SIMD do not cover: the
// block-boundary loads (0.1 ms), LDS reads (0.1), scalar loads (0.06).  256 registers
// are needed for a block of six pairs (four or eight pairs, or one wave per SIMD, took
// 1.9 to 2.4 ms).  Few poles or short chains leave latency: one item alone takes
// 0.6 us a pair, and 5 us to start and end.
//
// A step, with the tiled schedules and the partial sums' reduction before / with one
// pole per lane: T256, 2071 poles, four states 2468 / 1537 us; T301, 1245 poles, three
// states 2457 / 969; T128, 535 poles, eight states 341 / 228; T128, 407 poles, one
// state 80 / 47; T63, 151 poles, one state 37 / 13 in a run of 24.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.hpp"

namespace rexi {
namespace {

struct cd {
    double r, i;
};

__device__ __forceinline__ cd mk(double r, double i) { return cd{r, i}; }
__device__ __forceinline__ cd cmul(cd a, cd b) {
    return cd{fma(a.r, b.r, -a.i * b.i), fma(a.r, b.i, a.i * b.r)};
}
// 1 / a: v_rcp_f64 of |a|^2 refined by one third-order step
__device__ __forceinline__ cd crcp(cd a) {
    const double d = fma(a.r, a.r, a.i * a.i);
    const double r0 = __builtin_amdgcn_rcp(d);
    const double e = fma(-d, r0, 1.0);
    const double r = fma(r0, fma(e, e, e), r0);
    return cd{a.r * r, -a.i * r};
}
// -i q v
__device__ __forceinline__ cd miqv(cd q, cd v) { return cd{fma(q.i, v.r, q.r * v.i), fma(q.i, v.i, -q.r * v.r)}; }

// wave-uniform read-only data: scalar loads
typedef const double __attribute__((address_space(4)))* sptr;
__device__ __forceinline__ sptr uniform(const double* p) { return (sptr)(unsigned long long)p; }

// A scalar value of its own: without this the compiler keeps whole groups of
// kernel arguments together in scalar registers and spills them together.
template <class T>
__device__ __forceinline__ T detach(T x) {
    asm volatile("" : "+s"(x));
    return x;
}
// a b + s, s scalar: the compiler would copy s to vector registers first (to use
// the two-address form)
__device__ __forceinline__ double fma_s(double a, double b, double s) {
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(s));
    return r;
}

struct SweepPole {
    double2 al, ai, w1, w2, v1, v2;
};

struct SweepArgs {
    const SweepItem* items;
    const double* cst;       // [pair][kSweepCst]: D2, th' of the vorticity; D2, th', om2' of the divergence
    const double* rec;       // [S][npairs + 1][kSweepRec]: a, b of the vorticity; a, b, psi_a, psi_b of the divergence
    const SweepPole* poles;
    unsigned state_stride;  // doubles between two states' data
    double* part;            // [item][state][pair][kSweepRec]
    double2* scratch;        // per wave: [blocks][1 + 2 states][64]
    long long scratch_stride;
    int nitems, nst;         // nst: most states of an item
};

constexpr int kGroup = 2;                      // pairs per reduction group
constexpr int kBlk = kSweepBlock;              // pairs per block
constexpr int kVals = kGroup * kSweepRec;      // sums per reduction group

// Pivots of one pair after the pivot qp of the element before it.
__device__ __forceinline__ void pivots(const double* c, cd al, cd ai, cd qp, cd& qz, cd& qd) {
    qz = crcp(mk(fma(c[0], al.r, qp.r), fma(c[0], al.i, qp.i + c[1])));
    qd = crcp(mk(fma(c[2], al.r, fma(c[4], ai.r, qz.r)), fma(c[2], al.i, fma(c[4], ai.i, qz.i + c[3]))));
}

__device__ __forceinline__ double dpp_quad_xor(double x, const int ctrl_is_2) {
    const long long v = __double_as_longlong(x);
    int lo, hi;
    if (ctrl_is_2) {
        lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)v, 0x4E, 0xF, 0xF, true);  // quad_perm [2,3,0,1]
        hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), 0x4E, 0xF, 0xF, true);
    } else {
        lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)v, 0xB1, 0xF, 0xF, true);  // quad_perm [1,0,3,2]
        hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), 0xB1, 0xF, 0xF, true);
    }
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// weighted sums of one element (see the top): 2 values
__device__ __forceinline__ void weigh(cd w1, cd w2, cd xa, cd xb, double& re, double& im) {
    re = fma(w1.r, xa.r, fma(-w1.i, xa.i, fma(-w2.r, xb.i, -w2.i * xb.r)));
    im = fma(w2.r, xa.i, fma(w2.i, xa.r, fma(w1.r, xb.r, -w1.i * xb.i)));
}

// orders LDS accesses of the wave's lanes (the hardware keeps a wave's LDS
// operations in order; this keeps the compiler from moving them)
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Wave-uniform loads of N doubles into scalar registers, kept where the source
// has them (the compiler would sink them to their first use and wait there).
template <int N>
__device__ __forceinline__ void fetch(double (&h)[N], sptr p) {
#pragma unroll
    for (int k = 0; k < N; ++k) h[k] = p[k];
    __builtin_amdgcn_sched_barrier(0);
}

// Brings the data of a block's states and the constants of the block after it
// into the scalar cache: one load per 64-byte line, waited for only at warm_wait,
// after work that needs no LDS or scalar data.
constexpr int kLines = (kBlk * kSweepRec * 8 + 63) / 64 + 1, kCstLines = (kBlk * kSweepCst * 8 + 63) / 64 + 1;
struct Warm {
    int x[kSweepStates][kLines], c[kCstLines];
};
__device__ __forceinline__ void warm(Warm& w, sptr p, unsigned sstep, int nst, sptr cst) {
    typedef const int __attribute__((address_space(4)))* iptr;
#pragma unroll
    for (int s = 0; s < kSweepStates; ++s) {
        const iptr q = (iptr)(p + (s < nst ? s : 0) * sstep);
#pragma unroll
        for (int k = 0; k < kLines; ++k) w.x[s][k] = q[k + 1 < kLines ? 16 * k : 2 * kBlk * kSweepRec - 1];
    }
#pragma unroll
    for (int k = 0; k < kCstLines; ++k) w.c[k] = ((iptr)cst)[k + 1 < kCstLines ? 16 * k : 2 * kBlk * kSweepCst - 1];
    __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ void warm_wait(const Warm& w) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < kSweepStates; ++s)
#pragma unroll
        for (int k = 0; k < kLines; ++k) asm volatile("" ::"s"(w.x[s][k]));
#pragma unroll
    for (int k = 0; k < kCstLines; ++k) asm volatile("" ::"s"(w.c[k]));
}

constexpr int kPitch = 68;                  // row pitch of the reduction buffer: 4 mod 32 banks of 8 bytes
constexpr int kRedDoubles = kVals * kPitch;
static_assert(kBlk % kGroup == 0 && kBlk / kGroup <= 4, "a block's groups are stored by the four lanes of a row");
constexpr int kPart = kGroup * kSweepRec;   // data of a group of pairs and one state

// Sums over the wave's lanes.  A reduction group leaves kVals values per lane
// in LDS rows; lane 4 v + r then reads every fourth term of row v from r (lanes
// past the rows do what lanes 0..3 do).  The reads are issued at once and added
// only after the next group's work, so that their latency is not waited for.
struct Pending {
    double term[16];
};
__device__ __forceinline__ void pend_read(Pending& P, const double* src) {
    wave_sync();
#pragma unroll
    for (int i = 0; i < 16; ++i) P.term[i] = src[4 * i];
    __builtin_amdgcn_sched_barrier(0);
}
// the sum of row rv, in all four lanes of the row
__device__ __forceinline__ double pend_add(const Pending& P) {
    double s[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        s[i] = (P.term[4 * i] + P.term[4 * i + 1]) + (P.term[4 * i + 2] + P.term[4 * i + 3]);
    double sum = (s[0] + s[1]) + (s[2] + s[3]);
    sum += dpp_quad_xor(sum, 0);
    sum += dpp_quad_xor(sum, 1);
    return sum;
}

// What the backward pass of one batch keeps.
struct Back {
    cd al, ai, w1, w2, v1, v2;
    const double* rsrc;   // this lane's terms in the reduction buffer
    double* red;          // this lane's column there
    double2* car;         // [state][2][64]: x of the element above the block, this lane
    int rp;               // this lane stores the sums of group rp (of group 0 past the last)
    bool add;             // the sums are added to those of earlier batches
    int nst;
    unsigned sstep, pstep;  // between states: data, partial sums
};

// What a block needs first of the boundary values before it (this lane's),
// loaded one block ahead.
struct Boundary {
    double2 q, fa, fb;
};
__device__ __forceinline__ Boundary load_boundary(const double2* ckpt) { return Boundary{ckpt[0], ckpt[64], ckpt[128]}; }

// One block of the backward pass (pass 2) for all states of an item: the block's
// pivots from the one before it (qin), then per state the forward values into
// registers, the back substitution, and the weighted sums over the wave's poles.
// FULL: the block has all kBlk pairs, else ng groups of kGroup pairs.  head: the
// chain's first block (no boundary values before it).  h0 holds the first state's
// data of the block's first group on entry and those of rec_next on return (a
// whole block's do not fit in the scalar registers beside the rest).
//
// All global loads and stores are unconditional and issued at the start of a
// state (the store of a state's sums: after the next state's forward sweep), so
// that every wait for one finds it, and what was issued before it, a state's work
// old; where there is nothing to load, the address is any valid one and the value
// is dropped.
// ADD: there may be earlier batches' sums to add to (B.add).
template <bool FULL, bool ADD>
__device__ __forceinline__ void back_block(const Back& B, int ng, bool head, sptr cst, sptr cst_next, sptr rec,
                                           sptr rec_next, const double2* ckpt, const double2* ckpt_next, Boundary& bd,
                                           double* out, double (&h0)[kPart]) {
    constexpr int kGroups = kBlk / kGroup;
    const cd ai = B.ai;
    cd qin = cd{bd.q.x, bd.q.y};
    if (head) qin = mk(0, 0);
    double2 fan = bd.fa, fbn = bd.fb;
    bd = load_boundary(ckpt_next);
    cd q[2 * kBlk];
    Warm wm;
    {
        double c[kBlk * kSweepCst];
        fetch(c, cst);
        warm(wm, rec, B.sstep, B.nst, cst_next);
        cd qq = qin;
#pragma unroll
        for (int g = 0; g < kGroups; ++g)
            if (FULL || g < ng) {
#pragma unroll
                for (int t = g * kGroup; t < (g + 1) * kGroup; ++t) {
                    pivots(c + t * kSweepCst, B.al, ai, qq, q[2 * t], q[2 * t + 1]);
                    qq = q[2 * t + 1];
                }
            }
    }
    warm_wait(wm);
    Pending P;
    double2* cr = B.car;
    double sum0 = 0.0, sum1 = 0.0, old = 0.0;   // this lane's group's sum (groups 0 and others), what it is added to
    double* prev = out;                         // the previous state's place
#pragma unroll 1
    for (int s = 0; s < B.nst; ++s, cr += 128) {
        cd fa = cd{fan.x, fan.y}, fb = cd{fbn.x, fbn.y};
        if (head) fa = fb = mk(0, 0);
        const double before = old;
        if (ADD) old = *out;
        {
            const double2* n = ckpt + (s + 1 < B.nst ? 3 + 2 * s : 1) * 64;
            fan = n[0];
            fbn = n[64];
        }
        cd xa = cd{cr[0].x, cr[0].y}, xb = cd{cr[64].x, cr[64].y};
        cd Fa[2 * kBlk], Fb[2 * kBlk];
        const sptr rs = rec + s * B.sstep;
        double hg[kGroups][kPart];
#pragma unroll
        for (int k = 0; k < kPart; ++k) hg[0][k] = h0[k];
        fetch(hg[1], rs + kPart);
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            if (FULL || g < ng) {
#pragma unroll
                for (int t = g * kGroup; t < (g + 1) * kGroup; ++t) {
                    const double* rt = hg[g] + (t - g * kGroup) * kSweepRec;
                    const cd qz = t > 0 ? q[2 * t - 1] : qin, qd = q[2 * t];
                    fa = mk(fma(qz.i, fa.r, fma_s(qz.r, fa.i, rt[0])), fma(qz.i, fa.i, -qz.r * fa.r));
                    fb = mk(fma(qz.i, fb.r, fma_s(qz.r, fb.i, rt[1])), fma(qz.i, fb.i, -qz.r * fb.r));
                    Fa[2 * t] = fa;
                    Fb[2 * t] = fb;
                    fa = mk(fma(qd.i, fa.r, fma(ai.i, rt[4], fma_s(qd.r, fa.i, rt[2]))),
                            fma(qd.i, fa.i, fma(-qd.r, fa.r, -ai.r * rt[4])));
                    fb = mk(fma(qd.i, fb.r, fma(ai.i, rt[5], fma_s(qd.r, fb.i, rt[3]))),
                            fma(qd.i, fb.i, fma(-qd.r, fb.r, -ai.r * rt[5])));
                    Fa[2 * t + 1] = fa;
                    Fb[2 * t + 1] = fb;
                }
            }
            if (g + 2 < kGroups) fetch(hg[g + 2], rs + (g + 2) * kPart);
        }
        // The previous state's last group before the scalar loads: while scalar
        // loads are in flight, any wait for LDS waits for them too.
        if (FULL && s > 0) {
            const double v = pend_add(P);
            *prev = (B.rp == 0 || B.rp >= kGroups ? v : sum1) + (ADD && B.add ? before : 0.0);
        }
        fetch(h0, s + 1 < B.nst ? rec + (s + 1) * B.sstep : rec_next);
#pragma unroll
        for (int g = kGroups - 1; g >= 0; --g)
            if (FULL || g < ng) {
#pragma unroll
                for (int t = (g + 1) * kGroup - 1; t >= g * kGroup; --t) {
                    double* v = B.red + (t - g * kGroup) * kSweepRec * kPitch;
                    double re, im;
                    cd qq = q[2 * t + 1];
                    xa = cmul(qq, mk(Fa[2 * t + 1].r + xa.i, Fa[2 * t + 1].i - xa.r));
                    xb = cmul(qq, mk(Fb[2 * t + 1].r + xb.i, Fb[2 * t + 1].i - xb.r));
                    weigh(B.w1, B.w2, xa, xb, re, im);
                    v[2 * kPitch] = re;
                    v[3 * kPitch] = im;
                    weigh(B.v1, B.v2, xa, xb, re, im);
                    v[4 * kPitch] = re;
                    v[5 * kPitch] = im;
                    qq = q[2 * t];
                    xa = cmul(qq, mk(Fa[2 * t].r + xa.i, Fa[2 * t].i - xa.r));
                    xb = cmul(qq, mk(Fb[2 * t].r + xb.i, Fb[2 * t].i - xb.r));
                    weigh(B.w1, B.w2, xa, xb, re, im);
                    v[0] = re;
                    v[kPitch] = im;
                }
                if (FULL && g < kGroups - 1) {
                    const double v = pend_add(P);
                    sum1 = (g == kGroups - 2 || B.rp == g + 1) ? v : sum1;
                }
                pend_read(P, B.rsrc);
                if (!FULL) {
                    const double v = pend_add(P);
                    if (g == 0) sum0 = v;
                    else sum1 = B.rp == g ? v : sum1;
                }
            }
        if (!FULL) {
            // groups past the block's end have no place: their lanes repeat group 0
            *out = (B.rp == 0 || B.rp >= ng ? sum0 : sum1) + (ADD && B.add ? old : 0.0);
        }
        cr[0] = make_double2(xa.r, xa.i);
        cr[64] = make_double2(xb.r, xb.i);
        prev = out;
        out += B.pstep;
    }
    if (FULL) {
        const double v = pend_add(P);
        *prev = (B.rp == 0 || B.rp >= kGroups ? v : sum1) + (ADD && B.add ? old : 0.0);
    }
}

// One group of a block in pass 1: adds the products of one state's data and the
// coefficients of the block-end values.
__device__ __forceinline__ void forward_group(const cd* c, const cd* cpsi, const double (&h)[kPart], cd& fa, cd& fb) {
#pragma unroll
    for (int t = 0; t < kGroup; ++t) {
        const double* rt = h + t * kSweepRec;
        fa = mk(fma(c[2 * t].r, rt[0], fa.r), fma(c[2 * t].i, rt[0], fa.i));
        fb = mk(fma(c[2 * t].r, rt[1], fb.r), fma(c[2 * t].i, rt[1], fb.i));
        fa = mk(fma(c[2 * t + 1].r, rt[2], fa.r), fma(c[2 * t + 1].i, rt[2], fa.i));
        fb = mk(fma(c[2 * t + 1].r, rt[3], fb.r), fma(c[2 * t + 1].i, rt[3], fb.i));
        fa = mk(fma(cpsi[t].r, rt[4], fa.r), fma(cpsi[t].i, rt[4], fa.i));
        fb = mk(fma(cpsi[t].r, rt[5], fb.r), fma(cpsi[t].i, rt[5], fb.i));
    }
}

// One block of pass 1: pivots, then for every state the forward value at the
// block's end (car) from the one at its start, stored with the last pivot at o.
// FULL as in back_block.
template <bool FULL>
__device__ __forceinline__ void forward_block(cd al, cd ai, int ng, sptr cst, sptr cst_next, sptr rec, unsigned sstep,
                                              int nst, cd& qp, double2* car, double2* o) {
    constexpr int kGroups = kBlk / kGroup;
    cd q[2 * kBlk];
    const cd qin = qp;
    Warm wm;
    {
        double c[kBlk * kSweepCst];
        fetch(c, cst);
        warm(wm, rec, sstep, nst, cst_next);
#pragma unroll
        for (int g = 0; g < kGroups; ++g)
            if (FULL || g < ng) {
#pragma unroll
                for (int t = g * kGroup; t < (g + 1) * kGroup; ++t) {
                    pivots(c + t * kSweepCst, al, ai, qp, q[2 * t], q[2 * t + 1]);
                    qp = q[2 * t + 1];
                }
            }
    }
    warm_wait(wm);
    double h0[kPart];
    fetch(h0, rec);
    // q[t] -> coefficient of g_t in F at the block's end; the last is 1
    cd cpsi[kBlk];
    cd cc = mk(1, 0);
#pragma unroll
    for (int t = 2 * kBlk - 1; t >= 0; --t)
        if (FULL || t < 2 * kGroup * ng) {
            const cd below = t > 0 ? q[t - 1] : qin;
            q[t] = cc;
            const bool unit = FULL && t == 2 * kBlk - 1;
            if (t & 1) cpsi[t >> 1] = unit ? mk(ai.i, -ai.r) : miqv(ai, cc);
            cc = unit ? mk(below.i, -below.r) : miqv(below, cc);
        }
    o[0] = make_double2(qp.r, qp.i);
    double2 f0 = car[0], f1 = car[64];
#pragma unroll 1
    for (int s = 0; s < nst; ++s) {
        const cd ga = cmul(cc, cd{f0.x, f0.y}), gb = cmul(cc, cd{f1.x, f1.y});
        const sptr rs = rec + s * sstep;
        cd fa = mk(0, 0), fb = mk(0, 0);
        double hg[kGroups][kPart];
#pragma unroll
        for (int k = 0; k < kPart; ++k) hg[0][k] = h0[k];
        fetch(hg[1], rs + kPart);
        const int sn = s + 1 < nst ? s + 1 : s;
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            if (FULL || g < ng) forward_group(q + g * 2 * kGroup, cpsi + g * kGroup, hg[g], fa, fb);
            if (g + 2 < kGroups) fetch(hg[g + 2], rs + (g + 2) * kPart);
            if (g + 2 == kGroups) {
                f0 = car[(2 * sn) * 64];
                f1 = car[(2 * sn + 1) * 64];
                fetch(h0, rec + sn * sstep);
            }
        }
        const double2 g0 = make_double2(fa.r + ga.r, fa.i + ga.i);
        const double2 g1 = make_double2(fb.r + gb.r, fb.i + gb.i);
        car[(2 * s) * 64] = g0;
        car[(2 * s + 1) * 64] = g1;
        o[(1 + 2 * s) * 64] = g0;
        o[(2 + 2 * s) * 64] = g1;
    }
}

// ---- items of one state: the forward sweep of a block runs beside its pivots
//
// The pivots are a serial chain (some 90 cycles an element, of which their
// instructions fill two thirds).  With one state there is little other work to
// hide it behind, so both passes advance the forward values in the same loop, and
// pass 1 needs no block-end coefficients.
constexpr int kGc = kGroup * kSweepCst, kGr = kGroup * kSweepRec;
struct Scalars {
    double c[kGc], h[kGr];  // a group's constants and data
};
__device__ __forceinline__ void fetch(Scalars& x, sptr cst, sptr rec) {
#pragma unroll
    for (int k = 0; k < kGc; ++k) x.c[k] = cst[k];
#pragma unroll
    for (int k = 0; k < kGr; ++k) x.h[k] = rec[k];
    __builtin_amdgcn_sched_barrier(0);
}

// One element: F = g - i q F with g = a (vorticity) or a - i psi / alpha
// (divergence).
__device__ __forceinline__ void advance_z(cd q, double a, double b, cd& fa, cd& fb) {
    fa = mk(fma(q.i, fa.r, fma_s(q.r, fa.i, a)), fma(q.i, fa.i, -q.r * fa.r));
    fb = mk(fma(q.i, fb.r, fma_s(q.r, fb.i, b)), fma(q.i, fb.i, -q.r * fb.r));
}
__device__ __forceinline__ void advance_d(cd q, cd ai, const double* r, cd& fa, cd& fb) {
    fa = mk(fma(q.i, fa.r, fma(ai.i, r[2], fma_s(q.r, fa.i, r[0]))),
            fma(q.i, fa.i, fma(-q.r, fa.r, -ai.r * r[2])));
    fb = mk(fma(q.i, fb.r, fma(ai.i, r[3], fma_s(q.r, fb.i, r[1]))),
            fma(q.i, fb.i, fma(-q.r, fb.r, -ai.r * r[3])));
}

// Pivots and forward values over a block; keep(t, q, fa, fb) takes those of
// element t.  x holds the first group's scalars; the group after the block's last
// (next_c, next_h) is in it on return.
template <bool FULL, class Keep>
__device__ __forceinline__ void advance_block(cd al, cd ai, int ng, sptr cst, sptr rec, sptr next_c, sptr next_h,
                                              Scalars& x, cd& q, cd& fa, cd& fb, Keep keep) {
    constexpr int kGroups = kBlk / kGroup;
#pragma unroll
    for (int g = 0; g < kGroups; ++g)
        if (FULL || g < ng) {
            const bool last = FULL ? g + 1 == kGroups : g + 1 >= ng;
            Scalars n;
            fetch(n, last ? next_c : cst + (g + 1) * kGc, last ? next_h : rec + (g + 1) * kGr);
#pragma unroll
            for (int t = 0; t < kGroup; ++t) {
                cd qz, qd;
                pivots(x.c + t * kSweepCst, al, ai, q, qz, qd);
                const double* r = x.h + t * kSweepRec;
                advance_z(q, r[0], r[1], fa, fb);
                keep(2 * (g * kGroup + t), qz, fa, fb);
                advance_d(qz, ai, r + 2, fa, fb);
                keep(2 * (g * kGroup + t) + 1, qd, fa, fb);
                q = qd;
            }
            x = n;
        }
}

template <bool FULL, bool ADD>
__device__ __forceinline__ void back_block1(const Back& B, int ng, bool head, sptr cst, sptr rec, sptr next_c,
                                            sptr next_h, const double2* ckpt_next, Boundary& bd, double* out,
                                            Scalars& x, cd& xa, cd& xb) {
    constexpr int kGroups = kBlk / kGroup;
    cd q[2 * kBlk], Fa[2 * kBlk], Fb[2 * kBlk];
    {
        cd qq = cd{bd.q.x, bd.q.y}, fa = cd{bd.fa.x, bd.fa.y}, fb = cd{bd.fb.x, bd.fb.y};
        if (head) qq = fa = fb = mk(0, 0);
        bd = load_boundary(ckpt_next);
        advance_block<FULL>(B.al, B.ai, ng, cst, rec, next_c, next_h, x, qq, fa, fb, [&](int t, cd p, cd u, cd v) {
            q[t] = p;
            Fa[t] = u;
            Fb[t] = v;
        });
    }
    double old = 0.0;
    if (ADD) old = *out;
    Pending P;
    double sum0 = 0.0, sum1 = 0.0;
#pragma unroll
    for (int g = kGroups - 1; g >= 0; --g)
        if (FULL || g < ng) {
#pragma unroll
            for (int t = (g + 1) * kGroup - 1; t >= g * kGroup; --t) {
                double* v = B.red + (t - g * kGroup) * kSweepRec * kPitch;
                double re, im;
                cd qq = q[2 * t + 1];
                xa = cmul(qq, mk(Fa[2 * t + 1].r + xa.i, Fa[2 * t + 1].i - xa.r));
                xb = cmul(qq, mk(Fb[2 * t + 1].r + xb.i, Fb[2 * t + 1].i - xb.r));
                weigh(B.w1, B.w2, xa, xb, re, im);
                v[2 * kPitch] = re;
                v[3 * kPitch] = im;
                weigh(B.v1, B.v2, xa, xb, re, im);
                v[4 * kPitch] = re;
                v[5 * kPitch] = im;
                qq = q[2 * t];
                xa = cmul(qq, mk(Fa[2 * t].r + xa.i, Fa[2 * t].i - xa.r));
                xb = cmul(qq, mk(Fb[2 * t].r + xb.i, Fb[2 * t].i - xb.r));
                weigh(B.w1, B.w2, xa, xb, re, im);
                v[0] = re;
                v[kPitch] = im;
            }
            if (FULL && g < kGroups - 1) {
                const double v = pend_add(P);
                sum1 = (g == kGroups - 2 || B.rp == g + 1) ? v : sum1;
            }
            pend_read(P, B.rsrc);
            if (!FULL || g == 0) {
                const double v = pend_add(P);
                if (g == 0) sum0 = v;
                else sum1 = B.rp == g ? v : sum1;
            }
        }
    *out = (B.rp == 0 || B.rp >= (FULL ? kGroups : ng) ? sum0 : sum1) + (ADD && B.add ? old : 0.0);
}

// The two waves of a split chain (partners w and w ^ 1 of a workgroup) meet at
// its middle vorticity element h: with the pivots and forward values at both
// ends next to it,
//   (b_h + q + q') x_h = g_h - i q F - i q' F',
// which both compute (from the same operands, so to the same bits) and take as
// the element above their last block.  half 0 stores the element's sums.
// Every wave of the workgroup comes here once per item.
__device__ __forceinline__ void meet(const SweepArgs& A, const SweepItem& it, bool split, const Back& B, cd q,
                                     double2* lds_q, int wave, int lane, int car_stride) {
    lds_q += lane;
    if (split) lds_q[wave * 64] = make_double2(q.r, q.i);
    __syncthreads();
    cd xa[kSweepStates], xb[kSweepStates];
    if (split) {
        const double2 qo = lds_q[(wave ^ 1) * 64];
        const cd qp = cd{qo.x, qo.y};
        const double2* other = B.car + ((wave & 1) ? -car_stride : car_stride);
        const sptr c = uniform(A.cst + (long long)it.mid * kSweepCst);
        const cd z = crcp(mk(fma(c[0], B.al.r, q.r + qp.r), fma(c[0], B.al.i, (q.i + qp.i) + c[1])));
#pragma unroll
        for (int s = 0; s < kSweepStates; ++s)
            if (s < it.nst) {
                const sptr r = uniform(A.rec + (long long)(it.s0 + s) * A.state_stride + (long long)it.mid * kSweepRec);
                const double2 f0 = B.car[128 * s], f1 = B.car[128 * s + 64], e0 = other[128 * s], e1 = other[128 * s + 64];
                const cd ua = miqv(q, cd{f0.x, f0.y}), va = miqv(qp, cd{e0.x, e0.y});
                const cd ub = miqv(q, cd{f1.x, f1.y}), vb = miqv(qp, cd{e1.x, e1.y});
                xa[s] = cmul(z, mk((ua.r + va.r) + r[0], ua.i + va.i));
                xb[s] = cmul(z, mk((ub.r + vb.r) + r[1], ub.i + vb.i));
            }
    }
    __syncthreads();
    if (!split) return;
#pragma unroll
    for (int s = 0; s < kSweepStates; ++s)
        if (s < it.nst) {
            B.car[128 * s] = make_double2(xa[s].r, xa[s].i);
            B.car[128 * s + 64] = make_double2(xb[s].r, xb[s].i);
            if (it.half == 0) {
                double re, im;
                weigh(B.w1, B.w2, xa[s], xb[s], re, im);
                wave_sync();
                B.red[0] = re;
                B.red[kPitch] = im;
                Pending P;
                pend_read(P, B.rsrc);
                const double v = pend_add(P);
                if ((lane & 3) == 0 && lane < 8)  // rows 0 and 1
                    A.part[it.mid_off + (long long)s * B.pstep + (lane >> 2)] = v;
            }
        }
}

// One wave's work item.  SPLIT: items of one batch of poles; where it.mid >= 0 the
// item is one half of a chain (see meet).  ONE: items of one state.
template <bool SPLIT, bool ONE>
__device__ __forceinline__ void sweep_wave(const SweepArgs& A, const SweepItem& it, double2* scr, double* red,
                                           double2* car, double2* lds_q, int wave, int lane, int car_stride) {
    const int nst = detach(it.nst), npair = detach(it.npair), k0 = detach(it.k0), k1 = detach(it.k1);
    const int ckpt = (1 + 2 * nst) * 64;  // scratch entries per block
    const sptr cst = detach(uniform(A.cst + (long long)it.pair0 * kSweepCst));
    const unsigned sstep = detach(A.state_stride);
    const sptr rec = detach(uniform(A.rec + (long long)it.s0 * sstep + (long long)it.pair0 * kSweepRec));
    // this lane sums row rv from term rp, and stores that row of group rp
    const int rv = (lane >> 2) < kVals ? lane >> 2 : 0, rp = lane & 3;
    double* part = A.part + it.part_off + rv;
    const int nblk = (npair + kBlk - 1) / kBlk;
    const SweepPole* poles = detach(A.poles);
    const bool split = SPLIT && it.mid >= 0;
    scr += lane;
    car += lane;

    for (int kb = k0; kb < k1; kb += 64) {
        const bool act = kb + lane < k1;
        const SweepPole& pd = poles[act ? kb + lane : k1 - 1];
        const cd al = cd{pd.al.x, pd.al.y}, ai = cd{pd.ai.x, pd.ai.y};

        // ---- pass 1: pivots and forward values at the block boundaries
        cd qp = mk(0, 0), fa = mk(0, 0), fb = mk(0, 0);
        Scalars x;
        if (ONE) {
            fetch(x, cst, rec);
            auto none = [](int, cd, cd, cd) {};
            for (int b = 0; b + 1 < nblk; ++b) {
                const sptr c = cst + b * kBlk * kSweepCst, rb = rec + b * kBlk * kSweepRec;
                advance_block<true>(al, ai, 0, c, rb, c + kBlk * kSweepCst, rb + kBlk * kSweepRec, x, qp, fa, fb, none);
                double2* o = scr + (long long)b * ckpt;
                o[0] = make_double2(qp.r, qp.i);
                o[64] = make_double2(fa.r, fa.i);
                o[128] = make_double2(fb.r, fb.i);
            }
            // the group that pass 2 starts with, after the last block's forward values if they are needed
            const int b = nblk - 1;
            const sptr c = cst + b * kBlk * kSweepCst, rb = rec + b * kBlk * kSweepRec;
            if (split) {
                advance_block<false>(al, ai, (npair - b * kBlk) / kGroup, c, rb, c, rb, x, qp, fa, fb, none);
                car[0] = make_double2(fa.r, fa.i);
                car[64] = make_double2(fb.r, fb.i);
            }
        } else {
            for (int s = 0; s < 2 * nst; ++s) car[s * 64] = make_double2(0.0, 0.0);
        }
        for (int b = 0; !ONE && b + 1 < nblk; ++b) {
            const sptr c = cst + b * kBlk * kSweepCst;
            forward_block<true>(al, ai, 0, c, c + kBlk * kSweepCst, rec + b * kBlk * kSweepRec, sstep, nst, qp, car,
                                scr + (long long)b * ckpt);
        }
        if (!ONE && split) {
            const int b = nblk - 1;
            const sptr c = cst + b * kBlk * kSweepCst;
            forward_block<false>(al, ai, (npair - b * kBlk) / kGroup, c, c, rec + b * kBlk * kSweepRec, sstep, nst, qp,
                                 car, scr + (long long)b * ckpt);
        }

        // ---- pass 2: blocks in reverse
        const double keep = act ? 1.0 : 0.0;
        Back B;
        B.al = al;
        B.ai = ai;
        B.w1 = cd{keep * pd.w1.x, keep * pd.w1.y};
        B.w2 = cd{keep * pd.w2.x, keep * pd.w2.y};
        B.v1 = cd{keep * pd.v1.x, keep * pd.v1.y};
        B.v2 = cd{keep * pd.v2.x, keep * pd.v2.y};
        B.rsrc = red + rv * kPitch + rp;
        B.red = red + lane;
        B.car = car;
        B.rp = rp;
        B.add = kb != k0;
        B.nst = nst;
        B.sstep = sstep;
        B.pstep = detach((unsigned)it.pstride * kSweepRec);
        if constexpr (SPLIT) meet(A, it, split, B, qp, lds_q, wave, lane, car_stride);
        if (!split && !ONE)
            for (int s = 0; s < 2 * nst; ++s) car[s * 64] = make_double2(0.0, 0.0);
        double h0[kPart];
        if (!ONE) fetch(h0, rec + (nblk - 1) * kBlk * kSweepRec);
        cd xa = mk(0, 0), xb = mk(0, 0);
        if (ONE && split) {
            xa = cd{car[0].x, car[0].y};
            xb = cd{car[64].x, car[64].y};
        }
        // boundary values before block b >= 1 are at scr + (b - 1) ckpt
        Boundary bd = load_boundary(scr + (long long)max(nblk - 2, 0) * ckpt);
        for (int b = nblk - 1; b >= 0; --b) {
            const int ng = min(kBlk, npair - b * kBlk) / kGroup;  // groups of this block
            const int bn = max(b - 1, 0);
            const sptr c = cst + b * kBlk * kSweepCst, cn = cst + bn * kBlk * kSweepCst;
            const sptr rb = rec + b * kBlk * kSweepRec, rn = rec + bn * kBlk * kSweepRec;
            const double2* ck = scr + (long long)bn * ckpt;
            const double2* cx = scr + (long long)max(b - 2, 0) * ckpt;
            double* out = part + b * kBlk * kSweepRec + (rp < ng ? rp : 0) * kVals;
            if (ONE) {
                if (ng == kBlk / kGroup) back_block1<true, !SPLIT>(B, ng, b == 0, c, rb, cn, rn, cx, bd, out, x, xa, xb);
                else back_block1<false, !SPLIT>(B, ng, b == 0, c, rb, cn, rn, cx, bd, out, x, xa, xb);
                continue;
            }
            if (ng == kBlk / kGroup) back_block<true, !SPLIT>(B, ng, b == 0, c, cn, rb, rn, ck, cx, bd, out, h0);
            else back_block<false, !SPLIT>(B, ng, b == 0, c, cn, rb, rn, ck, cx, bd, out, h0);
        }
    }
}

// Workgroups of kSweepWaves waves, one work item each: the schedule gives the
// waves of a workgroup items of one chain where it can, so that they read its
// scalar data at about the same time from the scalar cache that they share.
// counter == null: workgroup w takes groups w, w + grid, ... of kSweepWaves
// items; else the groups come from the atomic counter (starting at zero).
template <bool SPLIT, bool ONE>
__global__ void __launch_bounds__(64 * kSweepWaves) __attribute__((amdgpu_waves_per_eu(2)))
k_sweep(const SweepArgs A, int* counter) {
    extern __shared__ double2 lds[];  // per wave: [2 states][64], then the reduction buffer
    __shared__ int next;
    __shared__ double2 lds_q[SPLIT ? kSweepWaves * 64 : 1];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    double2* scr = A.scratch + ((long long)blockIdx.x * kSweepWaves + wave) * A.scratch_stride;
    const int car_stride = A.nst * 128 + kRedDoubles / 2;
    double2* car = lds + wave * car_stride;
    double* red = reinterpret_cast<double*>(car + A.nst * 128);
    int i = blockIdx.x;
    for (;;) {
        if (counter) {
            if (threadIdx.x == 0) next = atomicAdd(counter, 1);
            __syncthreads();
            i = __builtin_amdgcn_readfirstlane(next);
            __syncthreads();
        }
        if (i < 0 || i * kSweepWaves >= A.nitems) break;
        if (i * kSweepWaves + wave < A.nitems) {
            typedef const SweepItem __attribute__((address_space(4)))* iptr;
            const iptr p = (iptr)(unsigned long long)(A.items + (i * kSweepWaves + wave));
            const SweepItem it{p->pair0, p->npair, p->pstride, p->s0, p->nst, p->k0, p->k1, p->mid, p->half, p->part_off,
                               p->mid_off};
            sweep_wave<SPLIT, ONE>(A, it, scr, red, car, lds_q, wave, lane, car_stride);
        } else if (SPLIT) {  // the barriers of meet
            __syncthreads();
            __syncthreads();
        }
        i += gridDim.x;
    }
}

// ---- short chains: a wave's part of a chain in registers
//
// Where every part has at most kShort pairs (whole chains, or halves of split
// ones) and one wave per SIMD is enough, nothing has to be repeated or stored:
// pivots and forward values of the whole part stay in registers (512 per lane).
// One batch of poles per item.  The time is the latency of one wave, about 10 us
// with up to 16 pairs and one state, half of it before the first pivot and after the
// last sum: its scalar lines are requested at once, beside the poles.  T63, 151 poles,
// one state: 15.5 us a step against 21 with split chains in blocks and 27 with whole
// ones.
constexpr int kShort = kSweepShort;

// scalar lines of [p, p + 8 n): requested here, waited for at warm_done
template <int LINES>
struct Lines {
    int x[LINES];
};
template <int LINES>
__device__ __forceinline__ void request(Lines<LINES>& l, sptr p, int n) {
    typedef const int __attribute__((address_space(4)))* iptr;
#pragma unroll
    for (int k = 0; k < LINES; ++k) l.x[k] = ((iptr)p)[min(16 * k, 2 * n - 1)];
}
template <int LINES>
__device__ __forceinline__ void arrived(const Lines<LINES>& l) {
#pragma unroll
    for (int k = 0; k < LINES; ++k) asm volatile("" ::"s"(l.x[k]));
}

__device__ __forceinline__ void short_item(const SweepArgs& A, const SweepItem& it, double* red, double2* ex, int wave,
                                           int lane) {
    constexpr int kGroups = kShort / kGroup;
    constexpr int kC = kGroup * kSweepCst, kR = kGroup * kSweepRec;
    const int nst = it.nst, ng = it.npair / kGroup;
    const bool split = it.mid >= 0;
    const bool act = it.k0 + lane < it.k1;
    const SweepPole& pd = A.poles[act ? it.k0 + lane : it.k1 - 1];
    const cd al = cd{pd.al.x, pd.al.y}, ai = cd{pd.ai.x, pd.ai.y};
    const double keep = act ? 1.0 : 0.0;
    const cd w1 = cd{keep * pd.w1.x, keep * pd.w1.y}, w2 = cd{keep * pd.w2.x, keep * pd.w2.y};
    const cd v1 = cd{keep * pd.v1.x, keep * pd.v1.y}, v2 = cd{keep * pd.v2.x, keep * pd.v2.y};
    const sptr cst = uniform(A.cst + (long long)it.pair0 * kSweepCst);
    const sptr rec = uniform(A.rec + (long long)it.s0 * A.state_stride + (long long)it.pair0 * kSweepRec);
    const sptr mcst = uniform(A.cst + (long long)max(it.mid, 0) * kSweepCst);
    const sptr mrec = uniform(A.rec + (long long)it.s0 * A.state_stride + (long long)max(it.mid, 0) * kSweepRec);
    constexpr int kCl = (kShort * kSweepCst * 8 + 63) / 64 + 1, kRl = (kShort * kSweepRec * 8 + 63) / 64 + 1;
    {
        Lines<kCl> lc;
        Lines<kRl> lr;
        Lines<1> lm, ln;
        request(lc, cst, it.npair * kSweepCst);
        request(lr, rec, it.npair * kSweepRec);
        request(lm, mcst, 1);
        request(ln, mrec, 1);
        __builtin_amdgcn_sched_barrier(0);
        arrived(lc);
        arrived(lr);
        arrived(lm);
        arrived(ln);
    }
    cd q[2 * kShort];
    cd qend = mk(0, 0);
    {
        double c[2][kC];
        fetch(c[0], cst);
#pragma unroll
        for (int g = 0; g < kGroups; ++g)
            if (g < ng) {
                fetch(c[(g + 1) & 1], cst + (g + 1 < ng ? g + 1 : g) * kC);
#pragma unroll
                for (int t = g * kGroup; t < (g + 1) * kGroup; ++t) {
                    pivots(c[g & 1] + (t - g * kGroup) * kSweepCst, al, ai, qend, q[2 * t], q[2 * t + 1]);
                    qend = q[2 * t + 1];
                }
            }
    }
    // exchange area: [wave][1 + 2 states][64]
    const int exs = (1 + 2 * A.nst) * 64;
    double2* own = ex + wave * exs + lane;
    const double2* other = ex + (wave ^ 1) * exs + lane;
    if (split) own[0] = make_double2(qend.r, qend.i);
    const int rv = (lane >> 2) < kVals ? lane >> 2 : 0, rp = lane & 3;
    const double* rsrc = red + rv * kPitch + rp;
    double* rcol = red + lane;
    const unsigned pstep = (unsigned)it.pstride * kSweepRec;
#pragma unroll 1
    for (int s = 0; s < A.nst; ++s) {
        cd Fa[2 * kShort], Fb[2 * kShort];
        cd fa = mk(0, 0), fb = mk(0, 0);
        const sptr rs = rec + (s < nst ? s : 0) * A.state_stride;
        if (s < nst) {
            double h[2][kR];
            fetch(h[0], rs);
#pragma unroll
            for (int g = 0; g < kGroups; ++g)
                if (g < ng) {
                    fetch(h[(g + 1) & 1], rs + (g + 1 < ng ? g + 1 : g) * kR);
#pragma unroll
                    for (int t = g * kGroup; t < (g + 1) * kGroup; ++t) {
                        const double* rt = h[g & 1] + (t - g * kGroup) * kSweepRec;
                        const cd qz = t > 0 ? q[2 * t - 1] : mk(0, 0), qd = q[2 * t];
                        fa = mk(fma(qz.i, fa.r, fma_s(qz.r, fa.i, rt[0])), fma(qz.i, fa.i, -qz.r * fa.r));
                        fb = mk(fma(qz.i, fb.r, fma_s(qz.r, fb.i, rt[1])), fma(qz.i, fb.i, -qz.r * fb.r));
                        Fa[2 * t] = fa;
                        Fb[2 * t] = fb;
                        fa = mk(fma(qd.i, fa.r, fma(ai.i, rt[4], fma_s(qd.r, fa.i, rt[2]))),
                                fma(qd.i, fa.i, fma(-qd.r, fa.r, -ai.r * rt[4])));
                        fb = mk(fma(qd.i, fb.r, fma(ai.i, rt[5], fma_s(qd.r, fb.i, rt[3]))),
                                fma(qd.i, fb.i, fma(-qd.r, fb.r, -ai.r * rt[5])));
                        Fa[2 * t + 1] = fa;
                        Fb[2 * t + 1] = fb;
                    }
                }
            if (split) {
                own[(1 + 2 * s) * 64] = make_double2(fa.r, fa.i);
                own[(2 + 2 * s) * 64] = make_double2(fb.r, fb.i);
            }
        }
        __syncthreads();  // every wave of the workgroup, once per state
        if (s >= nst) continue;
        double* out = A.part + it.part_off + (long long)s * pstep + rv;
        cd xa = mk(0, 0), xb = mk(0, 0);
        if (split) {  // the middle element, as in meet
            const double2 qo = other[0], e0 = other[(1 + 2 * s) * 64], e1 = other[(2 + 2 * s) * 64];
            const cd qp = cd{qo.x, qo.y};
            const cd z = crcp(mk(fma(mcst[0], al.r, qend.r + qp.r), fma(mcst[0], al.i, (qend.i + qp.i) + mcst[1])));
            const cd ua = miqv(qend, fa), va = miqv(qp, cd{e0.x, e0.y}), ub = miqv(qend, fb), vb = miqv(qp, cd{e1.x, e1.y});
            const sptr r = mrec + s * A.state_stride;
            xa = cmul(z, mk((ua.r + va.r) + r[0], ua.i + va.i));
            xb = cmul(z, mk((ub.r + vb.r) + r[1], ub.i + vb.i));
            if (it.half == 0) {
                double re, im;
                weigh(w1, w2, xa, xb, re, im);
                wave_sync();
                rcol[0] = re;
                rcol[kPitch] = im;
                Pending P;
                pend_read(P, rsrc);
                const double v = pend_add(P);
                if (rp == 0 && lane < 8) A.part[it.mid_off + (long long)s * pstep + rv] = v;
            }
        }
        Pending P;
#pragma unroll
        for (int g = kGroups - 1; g >= 0; --g)
            if (g < ng) {
                wave_sync();
#pragma unroll
                for (int t = (g + 1) * kGroup - 1; t >= g * kGroup; --t) {
                    double* v = rcol + (t - g * kGroup) * kSweepRec * kPitch;
                    double re, im;
                    cd qq = q[2 * t + 1];
                    xa = cmul(qq, mk(Fa[2 * t + 1].r + xa.i, Fa[2 * t + 1].i - xa.r));
                    xb = cmul(qq, mk(Fb[2 * t + 1].r + xb.i, Fb[2 * t + 1].i - xb.r));
                    weigh(w1, w2, xa, xb, re, im);
                    v[2 * kPitch] = re;
                    v[3 * kPitch] = im;
                    weigh(v1, v2, xa, xb, re, im);
                    v[4 * kPitch] = re;
                    v[5 * kPitch] = im;
                    qq = q[2 * t];
                    xa = cmul(qq, mk(Fa[2 * t].r + xa.i, Fa[2 * t].i - xa.r));
                    xb = cmul(qq, mk(Fb[2 * t].r + xb.i, Fb[2 * t].i - xb.r));
                    weigh(w1, w2, xa, xb, re, im);
                    v[0] = re;
                    v[kPitch] = im;
                }
                if (g + 1 < ng) out[(g + 1) * kVals] = pend_add(P);  // lanes of a row store the same value
                pend_read(P, rsrc);
            }
        out[0] = pend_add(P);
    }
}

__global__ void __launch_bounds__(64 * kSweepWaves) __attribute__((amdgpu_waves_per_eu(1, 1)))
k_sweep_short(const SweepArgs A, int* counter) {
    extern __shared__ double2 lds[];  // exchange area, then the waves' reduction buffers
    __shared__ int next;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    double* red = reinterpret_cast<double*>(lds + kSweepWaves * (1 + 2 * A.nst) * 64) + wave * kRedDoubles;
    int i = blockIdx.x;
    for (;;) {
        if (counter && threadIdx.x == 0) next = atomicAdd(counter, 1);
        __syncthreads();  // also: the exchange area's last readers are done
        if (counter) i = __builtin_amdgcn_readfirstlane(next);
        if (i < 0 || i * kSweepWaves >= A.nitems) break;
        if (i * kSweepWaves + wave < A.nitems) {
            typedef const SweepItem __attribute__((address_space(4)))* iptr;
            const iptr p = (iptr)(unsigned long long)(A.items + (i * kSweepWaves + wave));
            const SweepItem it{p->pair0, p->npair, p->pstride, p->s0, p->nst, p->k0, p->k1, p->mid, p->half, p->part_off,
                               p->mid_off};
            short_item(A, it, red, lds, wave, lane);
        } else {
            for (int s = 0; s < A.nst; ++s) __syncthreads();
        }
        if (!counter) break;
    }
}

// Physical state [S][3][nspec] -> records; fin[pair][3]: factors into scaled
// energy variables of vorticity, divergence and Phi.  One thread per (pair, variable),
// block row y per state.
__global__ void k_sweep_prep(const double2* __restrict__ u, double2* __restrict__ rec, const int2* __restrict__ idx,
                             const double* __restrict__ fin, int npairs, long long nspec) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x, q = e / 3, v = e - 3 * q;
    if (q > npairs) return;
    const long long s = blockIdx.y;
    const double2* us = u + (s * 3 + (v < 2 ? v + 1 : 0)) * nspec;  // zeta, delta, Phi
    double2* r = rec + (s * (npairs + 1) + q) * 3 + v;
    if (q == npairs) {  // (n, m) = (0, 0), in the order Phi, zeta, delta
        *r = u[(s * 3 + v) * nspec];
        return;
    }
    const int2 ix = idx[q];
    const int i = v == 0 ? ix.x : ix.y;
    double2 x = us[max(i, 0)];
    const double f = i >= 0 ? fin[e] : 0.0;
    // zeta' = -i zeta; delta; psi = om Phi', Phi' = -i Phi
    if (v != 1) x = make_double2(x.y, -x.x);
    *r = i >= 0 ? make_double2(x.x * f, x.y * f) : make_double2(0.0, 0.0);
}

struct SweepReduceArgs {
    const SweepTile* tiles;      // per state
    const SweepGroup* groups;    // [pair][tiles]
    const int2* idx;
    const double* cst;
    const double* fout;          // [pair][3]: factors back to physical variables
    const double2* part;
    const double2* rec_in;
    double2* rec_out;            // next records, or null
    double2* u_out;              // physical state, or null
    int npairs, ntiles;
    long long nspec;
    cd g00, gphi;
};

// Sum a pair's partials in order and finish Phi; write the next records or the
// physical state.  One thread per (pair, variable), block row y per state, so that
// a wave reads consecutive 16-byte values; kReduce partials are in flight at once.
// Bound by the partials' bytes where there are many (T256, four states: 113 MB,
// 35 us), by the latency of three dependent loads where there are few.  One thread
// per pair, with all six values of one partial after the other, took 38 us there,
// 26 at T127 with 8215 poles and one state, and 5 to 6 for the smallest steps.
constexpr int kReduce = 8;
__global__ void __launch_bounds__(256) k_sweep_reduce(const SweepReduceArgs R) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x, q = e / 3, v = e - 3 * q;
    if (q > R.npairs) return;
    const long long s = blockIdx.y;
    const long long at = (s * (R.npairs + 1) + q) * 3 + v;
    if (q == R.npairs) {  // the operator is zero at (0, 0)
        const double2 x = R.rec_in[at];
        const cd y = cmul(R.g00, cd{x.x, x.y});
        (R.u_out ? R.u_out[(s * 3 + v) * R.nspec] : R.rec_out[at]) = make_double2(y.r, y.i);
        return;
    }
    const SweepTile tl = R.tiles[s];
    const SweepGroup gr = R.groups[(long long)q * R.ntiles + tl.tile];
    const int2 ix = R.idx[q];
    const int i = v == 0 ? ix.x : ix.y;
    double2 psi = make_double2(0.0, 0.0);
    if (v == 2) psi = R.rec_in[at];
    const double c = R.cst[(long long)q * kSweepCst + 2 * v];  // D2, D2, om2'
    const double f = R.u_out ? R.fout[e] : c;
    const long long step = 3LL * tl.nst * gr.npair;
    const double2* p = R.part + gr.part_off + 3LL * tl.pos * gr.npair + v;
    double sr = 0.0, si = 0.0;
    for (int r = 0; r < gr.nr; r += kReduce) {
        double2 t[kReduce];
#pragma unroll
        for (int k = 0; k < kReduce; ++k) t[k] = p[min(r + k, gr.nr - 1) * step];
#pragma unroll
        for (int k = 0; k < kReduce; ++k) {
            sr += r + k < gr.nr ? t[k].x : 0.0;
            si += r + k < gr.nr ? t[k].y : 0.0;
        }
    }
    if (v == 2) {
        const cd y = cmul(R.gphi, cd{psi.x, psi.y});
        sr = fma(c, sr, y.r);
        si = fma(c, si, y.i);
    }
    if (R.u_out) {
        if (i < 0) return;
        double2* us = R.u_out + (s * 3 + (v < 2 ? v + 1 : 0)) * R.nspec + i;
        *us = v == 1 ? make_double2(sr * f, si * f) : make_double2(-si * f, sr * f);
    } else {
        const double g = v == 2 ? 1.0 : f;
        R.rec_out[at] = i >= 0 ? make_double2(sr * g, si * g) : make_double2(0.0, 0.0);
    }
}

}  // namespace

hipError_t enqueue_sweep_prep(rexi_plan* pl, const Workspace& ws, const Schedule& sc, const void* u, int buf, int S,
                              int adjoint, hipStream_t s) {
    const SweepTables& t = pl->sweep[sc.split];
    hipLaunchKernelGGL(k_sweep_prep, dim3((3 * (t.npairs + 1) + 255) / 256, S), dim3(256), 0, s, (const double2*)u,
                       (double2*)ws.rec[buf], t.d_idx, t.d_fin[adjoint], t.npairs, pl->nspec);
    return hipGetLastError();
}

hipError_t enqueue_sweep_solve(rexi_plan* pl, const Workspace& ws, const Schedule& sc, int buf, int S, int adjoint,
                               hipStream_t s) {
    const SweepTables& t = pl->sweep[sc.split];
    SweepArgs a;
    a.items = sc.d_sweep_items;
    a.cst = t.d_cst;
    a.rec = ws.rec[buf];
    a.poles = reinterpret_cast<const SweepPole*>(t.d_poles[adjoint]);
    a.part = reinterpret_cast<double*>(ws.part);
    a.scratch = ws.sweep_scratch;
    a.scratch_stride = sc.sweep_stride;
    a.state_stride = (unsigned)(t.npairs + 1) * kSweepRec;
    a.nitems = (int)sc.sweep_items.size();
    int grid = std::min((a.nitems + kSweepWaves - 1) / kSweepWaves, ws.sweep_groups);
    if (grid < 1) return hipErrorInvalidValue;
    a.nst = sc.sweep_nst;
    const bool one = sc.sweep_nst == 1;
    typedef void (*Kernel)(SweepArgs, int*);
    const Kernel kernel = sc.short_chains ? (Kernel)k_sweep_short
                          : sc.split      ? (one ? (Kernel)k_sweep<true, true> : (Kernel)k_sweep<true, false>)
                                          : (one ? (Kernel)k_sweep<false, true> : (Kernel)k_sweep<false, false>);
    const size_t lds = sizeof(double2) * kSweepWaves *
                       ((sc.short_chains ? 64 : 0) + 128 * (size_t)sc.sweep_nst + kRedDoubles / 2);
    int* counter = nullptr;
    if (!sc.persistent && ws.counters && sweep_resident(sc)) {
        grid = std::min(grid, kSweepGroups);
        counter = ws.counters;
        const hipError_t e = enqueue_reset_counters(counter, 1, s);
        if (e != hipSuccess) return e;
    }
    if (sc.persistent) {
        int dev = 0, ncu = 0, per_cu = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
        if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)kernel, 64 * kSweepWaves, lds);
        if (e != hipSuccess) return e;
        grid = std::max(1, std::min(grid, std::max(1, per_cu) * ncu));
        counter = ws.counters;
        e = enqueue_reset_counters(counter, 1, s);
        if (e != hipSuccess) return e;
    }
    kernel<<<dim3(grid), dim3(64 * kSweepWaves), lds, s>>>(a, counter);
    return hipGetLastError();
}

hipError_t enqueue_sweep_reduce(rexi_plan* pl, const Workspace& ws, const Schedule& sc, int buf_in, int buf_out,
                                void* u_out, int S, int adjoint, hipStream_t s) {
    const SweepTables& t = pl->sweep[sc.split];
    SweepReduceArgs r;
    r.tiles = sc.d_sweep_tiles;
    r.groups = sc.d_sweep_groups;
    r.idx = t.d_idx;
    r.cst = t.d_cst;
    r.fout = t.d_fout[adjoint];
    r.part = ws.part;
    r.rec_in = (const double2*)ws.rec[buf_in];
    r.rec_out = u_out ? nullptr : (double2*)ws.rec[buf_out];
    r.u_out = (double2*)u_out;
    r.npairs = t.npairs;
    r.ntiles = sc.sweep_ntiles;
    r.nspec = pl->nspec;
    const std::complex<double> g00 = adjoint ? pl->g00_adj : pl->g00_fwd;
    const std::complex<double> gp = adjoint ? pl->gphi_adj : pl->gphi_fwd;
    r.g00 = cd{g00.real(), g00.imag()};
    r.gphi = cd{gp.real(), gp.imag()};
    hipLaunchKernelGGL(k_sweep_reduce, dim3((3 * (t.npairs + 1) + 255) / 256, S), dim3(256), 0, s, r);
    return hipGetLastError();
}

}  // namespace rexi
