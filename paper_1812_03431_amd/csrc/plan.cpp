// C ABI of the T-REXI library: argument checking, plans, schedules, step
// drivers and the schedule autotuner.  The arithmetic runs in the HIP kernels
// (rexi_kernels.hip, sh_kernels.hip); this file only prepares tables and
// enqueues work.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <memory>
#include <string>

#include "internal.hpp"

namespace rexi {


namespace {
thread_local std::string g_err;
}

int fail(int code, const std::string& msg) {
    g_err = msg;
    return code;
}

int caught() noexcept {
    try {
        return fail(REXI_ENOMEM, "host allocation failed");
    } catch (...) {
        g_err.clear();
        return REXI_ENOMEM;
    }
}

int hip_fail(hipError_t e, const char* what) {
    return fail(REXI_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

hipError_t timed_begin(rexi_plan* pl, int kind, hipStream_t s) {
    if (!pl->timing) return hipSuccess;
    auto& v = pl->events[kind];
    if (v.size() == v.capacity()) v.reserve(2 * v.size() + 16);  // before the events, which a throw would leak
    hipEvent_t a = nullptr, b = nullptr;
    hipError_t e = hipEventCreate(&a);
    if (e != hipSuccess) return e;
    e = hipEventCreate(&b);
    if (e != hipSuccess) { (void)hipEventDestroy(a); return e; }
    v.push_back({a, b});
    return hipEventRecord(a, s);
}

hipError_t timed_end(rexi_plan* pl, int kind, hipStream_t s) {
    if (!pl->timing || pl->events[kind].empty()) return hipSuccess;
    return hipEventRecord(pl->events[kind].back().second, s);
}

namespace {

template <class T>
int dev_alloc(T** p, size_t count) {
    if (count == 0) count = 1;
    hipError_t e = hipMalloc((void**)p, count * sizeof(T));
    if (e != hipSuccess) {
        *p = nullptr;
        (void)hipGetLastError();  // reported here; a later launch's check would find it again
        return fail(REXI_ENOMEM, std::string("hipMalloc of ") + std::to_string(count * sizeof(T)) +
                                     " bytes failed: " + hipGetErrorString(e));
    }
    return REXI_OK;
}

template <class T>
int upload(T** p, const std::vector<T>& v) {
    int rc = dev_alloc(p, v.size());
    if (rc) return rc;
    REXI_HIP(hipMemcpy(*p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice));
    return REXI_OK;
}

template <class T>
void dev_free(T*& p) {
    if (p) (void)hipFree(p);
    p = nullptr;
}

int check_params(const rexi_params* p) {
    if (!p) return fail(REXI_EINVAL, "params is NULL");
    if (p->T < 1 || p->T > 1023) return fail(REXI_EINVAL, "T must be in [1, 1023]");
    if (!(p->dt > 0) || !std::isfinite(p->dt)) return fail(REXI_EINVAL, "dt must be positive and finite");
    if (!(p->radius > 0) || !(p->gravity > 0) || !(p->mean_depth > 0) || !std::isfinite(p->omega))
        return fail(REXI_EINVAL, "radius, gravity and mean_depth must be positive, omega finite");
    if (p->M < 1 || p->M > 1 << 20) return fail(REXI_EINVAL, "M must be in [1, 2^20]");
    if (!(p->h > 0) || !std::isfinite(p->h)) return fail(REXI_EINVAL, "h must be positive");
    if (p->L < 1 || p->L > 32) return fail(REXI_EINVAL, "L must be in [1, 32]");
    if (p->max_states < 1 || p->max_states > 64) return fail(REXI_EINVAL, "max_states must be in [1, 64]");
    if (p->fsphere != 0 && p->fsphere != 1) return fail(REXI_EINVAL, "fsphere must be 0 or 1");
    if (p->fsphere && !std::isfinite(p->f0)) return fail(REXI_EINVAL, "f0 must be finite");
    if (p->nlat != 0 || p->nlon != 0) {
        if (p->nlat < 2 || p->nlat > 2048 || (p->nlat & 1))
            return fail(REXI_EINVAL, "nlat must be even and in [2, 2048]");
        if (p->nlon < 4 || p->nlon > 4096 || (p->nlon & (p->nlon - 1)))
            return fail(REXI_EINVAL, "nlon must be a power of two in [4, 4096]");
        if (p->T >= p->nlon) return fail(REXI_EINVAL, "T must be below nlon");
        if (p->max_fields < 1 || p->max_fields > 1024) return fail(REXI_EINVAL, "max_fields must be in [1, 1024]");
    }
    return REXI_OK;
}

long double eps_nm(int n, int m) {
    if (n <= 0 || n < m) return 0.0L;
    return sqrtl((long double)((long long)n * n - (long long)m * m) / (4.0L * n * n - 1.0L));
}

// Layout of the chain slots (independent of the lane tiling).
std::vector<MInfo> chain_layout(int T) {
    std::vector<MInfo> mi(T + 1);
    long long slot = 0;
    for (int m = 0; m <= T; ++m) {
        MInfo x{};
        x.n0 = std::max(m, 1);
        x.L = T + 1 - x.n0;
        x.spec_off = (int)spec_offset(T, m);
        x.slot_base = (int)slot;
        slot += 2LL * x.L;
        mi[m] = x;
    }
    return mi;
}

// Elements-per-lane class SE and cross-lane move kind of a chain of L
// elements under a policy.  Kinds: 0 ds_bpermute (groups up to 64 lanes),
// 1 DPP row shifts (groups inside one 16-lane row), 2 DPP over a pair of rows
// (groups of exactly 32 lanes).
//   0 "8":       8 (L <= 128, rows), 8 (L <= 256, row pairs)
//   1 "8/16":    8 (L <= 128), 16 (<= 256), rows
//   2 "16":      16 (L <= 256), rows
//   3 "8/12/16": 8 (L <= 128), 12 (<= 192), 16 (<= 256), rows
//   4 "4/8":     4 (L <= 64, rows), 4 (L <= 128, row pairs), 8 (L <= 256, row pairs)
//   5 "fine":    8 (L <= 64), 6 (<= 96), 8 (<= 128), 10 (<= 160), 12 (<= 192),
//                14 (<= 224), 16 (<= 256), rows: padding at most 2 elements per lane
// Beyond 256 elements every policy uses 16 with ds_bpermute (L <= 1024).
void tile_class(int policy, int L, int& SE, int& kind) {
    kind = 1;
    switch (policy) {
        case 0:
            if (L <= 128) { SE = 8; return; }
            if (L <= 256) { SE = 8; kind = 2; return; }
            break;
        case 1:
            if (L <= 128) { SE = 8; return; }
            if (L <= 256) { SE = 16; return; }
            break;
        case 2:
            if (L <= 256) { SE = 16; return; }
            break;
        case 3:
            if (L <= 128) { SE = 8; return; }
            if (L <= 192) { SE = 12; return; }
            if (L <= 256) { SE = 16; return; }
            break;
        case 4:
            if (L <= 64) { SE = 4; return; }
            if (L <= 128) { SE = 4; kind = 2; return; }
            if (L <= 256) { SE = 8; kind = 2; return; }
            break;
        default:
            if (L <= 64) { SE = 8; return; }
            if (L <= 256) { SE = 2 * ((L + 31) / 32); return; }  // 16 lanes x SE >= L
            break;
    }
    kind = 0;
    SE = 16;
}

const char* kPolicyName[] = {"8", "8/16", "16", "8/12/16", "4/8", "fine"};
constexpr int kPolicies = 6;

// Work split of one candidate schedule.  Items are (m, chain, state tile,
// pole range).  Per order the tile holds R states, the largest of 4, 2, 1
// that is at most the mode's limit, divides S, fits the chain groups of a wave
// (P R <= 64) and is compiled; the item's waves then factorise each pole
// once for its R states.  Modes: 0 one state per item; 1 the most states per
// item in every class; 2 the same only for tiles of at most 6 or at least 14
// elements per lane (measured at T256: sharing gains 14-20% there, while
// the 8-element tile loses its second wave per SIMD to the factorisation's
// LDS and the 10- and 12-element tiles gain nothing).  The number of items per (m, chain, tile) follows a
// cost model per wave iteration (elements x sweep work + log2(P) reduction
// levels, the factorising pass and R - 1 passes that reuse it, scaled by the
// waves a SIMD can hold for the class).  One launch per (SE, kind, R) class;
// items in a launch run longest first.
int build_schedule(rexi_plan* pl, int S, int policy, long long target_items, bool per_term, int rot_mode,
                   Schedule& out) {
    const int rot_max = rot_mode == 0 ? 1 : 4;
    const int T = pl->T, N = per_term ? 1 : pl->N;
    out = Schedule();
    out.rot_max = rot_max;
    out.S = S;
    out.minfo = chain_layout(T);
    struct Unit { int m, p, tile, rot; double cost; int iters; int G; int cls; };
    std::vector<Unit> units;
    struct Cls { int SE, kind, rot; };
    std::vector<Cls> classes;
    double total = 0;
    for (int m = 0; m <= T; ++m) {
        MInfo& mi = out.minfo[m];
        int SE, kind;
        tile_class(policy, mi.L, SE, kind);
        int P = 1;
        while (P * SE < mi.L) P *= 2;
        if (kind == 1 ? P > 16 : kind == 2 ? P != 32 : P > 64)
            return fail(REXI_EUNSUPPORTED, "chain length does not fit this tiling");
        int rot = 1;
        const bool share = rot_mode == 1 || (rot_mode == 2 && (SE <= 6 || SE >= 14));
        for (int r : {4, 2})
            if (share && r <= rot_max && S % r == 0 && P * r <= 64 && solve_variant_supported(SE, kind, r, per_term)) {
                rot = r;
                break;
            }
        if (!solve_variant_supported(SE, kind, rot, per_term)) return fail(REXI_EUNSUPPORTED, "tile class not compiled");
        mi.P = P;
        mi.s = SE;
        out.SM = std::max(out.SM, SE);
        int cls = -1;
        for (int c = 0; c < (int)classes.size(); ++c)
            if (classes[c].SE == SE && classes[c].kind == kind && classes[c].rot == rot) cls = c;
        if (cls < 0) { cls = (int)classes.size(); classes.push_back({SE, kind, rot}); }
        const int G = 64 / P * (per_term ? 1 : solve_waves_per_item());  // poles per workgroup iteration
        int lg = 0;
        while ((1 << lg) < P) ++lg;
        const double occ = (SE <= 8 && rot == 1) ? 2.0 : 1.0;
        const double lvl = kind == 0 ? 160.0 : kind == 2 ? 100.0 : 90.0;
        const double fused = SE * 100.0 + lg * lvl + 60.0;
        const double reuse = SE * 65.0 + lg * 0.5 * lvl + 40.0;
        const double it_cost = (fused + (rot - 1) * reuse) / occ;
        const int iters = (N + G - 1) / G;
        for (int p = 0; p < 2; ++p)
            for (int t = 0; t < S / rot; ++t) {
                units.push_back({m, p, t, rot, it_cost * iters, iters, G, cls});
                total += it_cost * iters;
            }
    }
    const double target = per_term ? 1e300 : total / (double)std::max<long long>(1, target_items);
    out.groups.assign((size_t)(T + 1) * 2 * S, Group{0, 0, 0});
    long long off = 0;
    std::vector<std::vector<std::pair<double, Item>>> by_class(classes.size());
    for (const Unit& u : units) {
        int nr = (int)std::lround(u.cost / target);
        nr = std::max(1, std::min(nr, u.iters));
        const long long L2 = 2LL * out.minfo[u.m].L;
        for (int q = 0; q < u.rot; ++q) {
            Group& gr = out.groups[((size_t)u.m * 2 + u.p) * S + u.tile * u.rot + q];
            gr.part_off = off + q * L2;
            gr.nr = nr;
            gr.st = u.rot;
        }
        for (int r = 0; r < nr; ++r) {
            const int i0 = (int)((long long)u.iters * r / nr), i1 = (int)((long long)u.iters * (r + 1) / nr);
            Item it;
            it.m = u.m;
            it.p = u.p;
            it.tile = u.tile;
            it.k0 = i0 * u.G;
            it.k1 = std::min(N, i1 * u.G);
            it.part_off = off;
            off += u.rot * L2;
            by_class[u.cls].push_back({u.cost * (i1 - i0) / u.iters, it});
        }
    }
    for (int c = 0; c < (int)classes.size(); ++c) {
        auto& v = by_class[c];
        std::stable_sort(v.begin(), v.end(), [](const std::pair<double, Item>& a, const std::pair<double, Item>& b) {
            return a.first > b.first;
        });
        int pmax = 1;
        for (auto& x : v) pmax = std::max(pmax, out.minfo[x.second.m].P);
        Launch L{classes[c].SE, classes[c].kind, (int)out.items.size(), (int)v.size(), pmax, classes[c].rot};
        for (auto& x : v) out.items.push_back(x.second);
        out.launches.push_back(L);
    }
    out.part_size = off;
    // "_shared": every class shares factorisations among states, "_mixed": some do
    int nshare = 0;
    for (const Cls& c : classes) nshare += c.rot > 1;
    const char* share_tag = nshare == 0 ? "" : nshare == (int)classes.size() ? "_shared" : "_mixed";
    char buf[96];
    std::snprintf(buf, sizeof buf, "%s_items%lld%s%s", kPolicyName[policy], (long long)out.items.size(), share_tag,
                  per_term ? "_perterm" : "");
    out.name = buf;
    return REXI_OK;
}

// Slots of chain (m, p) in pairs (an element or -1): even ones vorticity, odd ones
// divergence; element j (degree max(m, 1) + j) is a vorticity iff pre + j is even.
// half: pairs of the two halves of a chain split around its middle pair, or 0.
std::vector<int> sweep_slots(int T, int m, int p, bool split, int2* half) {
    const int n0 = std::max(m, 1), L = T + 1 - n0, pre = (n0 + p) & 1;
    std::vector<int> slot;
    *half = make_int2(0, 0);
    auto whole_groups = [](int n) { return 4 * ((n + 3) / 4); };
    if (split && L >= kSweepSplit) {
        const int h = L / 2 + ((pre + L / 2) & 1);  // the middle vorticity element
        const int na = whole_groups(h), nb = whole_groups(L - 1 - h);
        slot.assign(na + 2 + nb, -1);
        for (int j = 0; j < h; ++j) slot[na - h + j] = j;
        slot[na] = h;
        for (int j = L - 1; j > h; --j) slot[na + 2 + nb - (j - h)] = j;
        *half = make_int2(na / 2, nb / 2);
    } else {
        slot.assign(whole_groups(pre + L), -1);
        for (int j = 0; j < L; ++j) slot[pre + j] = j;
    }
    return slot;
}

// The chains' places in the tables (host only).
void sweep_layout(rexi_plan* pl, bool split) {
    SweepTables& t = pl->sweep[split];
    if (!t.chains.empty()) return;
    std::vector<SweepChain> chains;
    std::vector<int2> halves;
    int npairs = 0;
    for (int m = 0; m <= pl->T; ++m)
        for (int p = 0; p < 2; ++p) {
            int2 half;
            const int np = (int)sweep_slots(pl->T, m, p, split, &half).size() / 2;
            chains.push_back({npairs, np});
            halves.push_back(half);
            npairs += np;
        }
    t.chains = std::move(chains);
    t.halves = std::move(halves);
    t.npairs = npairs;
}

void free_sweep_tables(SweepTables& t) {
    dev_free(t.d_cst);
    dev_free(t.d_idx);
    for (int d = 0; d < 2; ++d) {
        dev_free(t.d_fin[d]);
        dev_free(t.d_fout[d]);
        dev_free(t.d_poles[d]);
    }
}

// Tables of the pole-per-lane solve (see sweep_kernels.hip), built with the
// first schedule that reads them.  Not usable without a Coriolis force (the scaling
// divides by the couplings) or where the scaled constants leave a comfortable FP64
// range.  The couplings are c_n^m = g_n sqrt(n^2 - m^2), so that an element costs
// one square root and one division in long double (x87: about 20 ns each, and
// T301 has 45 thousand elements); the rest depends on n alone.
int build_sweep_tables(rexi_plan* pl, bool split) {
    SweepTables& t = pl->sweep[split];
    if (t.built) return REXI_OK;
    sweep_layout(pl, split);
    const int T = pl->T, N = pl->N;
    const long double a = pl->prm.radius, Om = pl->prm.omega, pb = pl->phibar, dt = pl->prm.dt;
    const double kDummy = 1e100;
    const size_t np = t.npairs;
    std::vector<double> cst(np * kSweepCst, 0.0), fin[2], fout[2];
    std::vector<int2> idx(np, make_int2(-1, -1));
    for (int d = 0; d < 2; ++d) {
        fin[d].assign(np * 3, 0.0);
        fout[d].assign(np * 3, 0.0);
    }
    bool ok = true;
    auto in_range = [](long double x) { return fabsl(x) > 1e-40L && fabsl(x) < 1e40L; };
    struct PerDegree { long double g, th, om, iom, s, is; };
    std::vector<PerDegree> deg(T + 1);
    for (int n = 1; n <= T; ++n) {
        const long double nn = (long double)n * (n + 1), n2 = (long double)n * n;
        PerDegree& d = deg[n];
        d.g = 2 * Om * dt * sqrtl((n2 - 1) / (4 * n2 - 1)) / n;
        d.th = 2 * Om / nn * dt;
        d.om = sqrtl(pb * nn) / a * dt;
        d.iom = 1 / d.om;
        d.s = a * sqrtl(pb / nn);
        d.is = 1 / d.s;
        ok = ok && in_range(d.om) && in_range(d.s);
    }
    std::vector<long double> D(T + 1), iD(T + 1);
    for (int m = 0; m <= T && ok; ++m) {
        const int n0 = std::max(m, 1), L = T + 1 - n0;
        // D_j D_{j+1} = 1 / c_{j+1}, the couplings of consecutive elements
        auto couple = [&](int n) { return deg[n].g * sqrtl((long double)((long long)n * n - (long long)m * m)); };
        iD[0] = L > 1 ? sqrtl(fabsl(couple(n0 + 1))) : 1.0L;
        D[0] = 1 / iD[0];
        for (int j = 1; j < L; ++j) {
            iD[j] = couple(n0 + j) * D[j - 1];
            D[j] = 1 / iD[j];
        }
        for (int j = 0; j < L; ++j) ok = ok && in_range(D[j]);
        for (int p = 0; p < 2; ++p) {
            int2 half;
            const std::vector<int> slot = sweep_slots(T, m, p, split, &half);
            const size_t q0 = t.chains[2 * m + p].pair0;
            for (size_t k = 0; k < slot.size(); ++k) {
                const size_t q = q0 + k / 2;
                const bool div = (k & 1) != 0;
                double* c = &cst[q * kSweepCst];
                if (slot[k] < 0) {
                    c[div ? 2 : 0] = kDummy;
                    continue;
                }
                const int j = slot[k], n = n0 + j;
                const PerDegree& e = deg[n];
                const long double Dj = D[j], D2 = Dj * Dj;
                const int i = (int)(spec_offset(T, m) + (n - m));
                c[div ? 2 : 0] = (double)D2;
                c[div ? 3 : 1] = (double)(D2 * e.th * m);
                if (div) c[4] = (double)(D2 * e.om * e.om);
                (div ? idx[q].y : idx[q].x) = i;
                for (int d = 0; d < 2; ++d) {
                    fin[d][3 * q + div] = (double)(Dj * (d ? e.is : e.s));
                    fout[d][3 * q + div] = (double)(Dj * (d ? e.s : e.is));
                    if (div) {
                        fin[d][3 * q + 2] = (double)(Dj * e.om);
                        fout[d][3 * q + 2] = (double)(iD[j] * e.iom);
                    }
                }
            }
        }
    }
    cst.resize(cst.size() + kSweepPad, 0.0);
    if (!ok) {
        t.built = true;
        return REXI_OK;
    }
    free_sweep_tables(t);  // of a build that did not end
    int rc = upload(&t.d_cst, cst);
    if (!rc) rc = upload(&t.d_idx, idx);
    for (int d = 0; d < 2 && !rc; ++d) {
        rc = upload(&t.d_fin[d], fin[d]);
        if (!rc) rc = upload(&t.d_fout[d], fout[d]);
        std::vector<double2> pd;
        pd.reserve(6 * (size_t)N);
        auto put = [&](const cld& z) { pd.push_back(make_double2((double)z.real(), (double)z.imag())); };
        for (int k = 0; k < N; ++k) {
            const std::complex<double> bp = pl->poles.beta_plus[k], bm = std::conj(pl->poles.beta_minus[N - 1 - k]);
            const cld al(pl->poles.alpha[k]), wx(d ? bm : bp), wy(d ? bp : bm);
            const cld ai = cld(1) / al, mi = cld(0, -1) * ai;
            for (const cld& z : {al, ai, wx + wy, wx - wy, mi * (wx + wy), mi * (wx - wy)}) put(z);
        }
        if (!rc) rc = upload(&t.d_poles[d], pd);
    }
    if (rc) {
        free_sweep_tables(t);
        return rc;
    }
    t.usable = t.built = true;
    return REXI_OK;
}

// Where the chip is not filled, a long chain's time is what counts: with at most
// kSplitWaves waves of one batch and a whole chain each, chains are split between
// two waves (measured, whole / split: 258 chains x 7 batches, four states 130 / 116
// us, T110 x 5 batches 108 / 79, T200 x 3 batches 192 / 128; but 1992 waves 74 / 81,
// 2548 waves 44 / 50).  The register-resident form runs one wave per SIMD, so it is
// taken while its waves are few enough for that (1050 waves, four states 48 -> 36 us,
// one state 24 -> 17 us; 3360 waves, four states 81 -> 87), for one state up to two
// rounds (2100 waves 28 -> 26 us).
constexpr long long kSplitWaves = 1900, kShortWaves = 1100;

// A pole-per-lane schedule: the states in tiles of up to `most`, split
// evenly; items are (chain, tile, range of 64-pole batches), as many per
// (chain, tile) as its share of target_items, longest first.  split: one batch per
// item, and the two halves of a split chain are consecutive items from an even
// index on (waves of one workgroup).
int build_sweep_schedule(rexi_plan* pl, int S, int most, long long target_items, bool split, bool short_chains,
                         Schedule& out) {
    sweep_layout(pl, split);
    const SweepTables& t = pl->sweep[split];
    const int nt = (S + most - 1) / most, nb = (pl->N + 63) / 64;
    if (short_chains) {
        long long waves = 0;
        int npmax = 0;
        for (size_t ch = 0; ch < t.chains.size(); ++ch) {
            const int2 half = t.halves[ch];
            waves += (half.x > 0 ? 2LL : 1LL) * nt * nb;
            npmax = std::max(npmax, half.x > 0 ? std::max(half.x, half.y) : t.chains[ch].npair);
        }
        if (npmax > kSweepShort || waves > kShortWaves * (S == nt ? 2 : 1))
            return fail(REXI_EUNSUPPORTED, "chains too long or too many for registers");
    }
    out = Schedule();
    out.sweep = true;
    out.split = split;
    out.short_chains = short_chains;
    out.S = S;
    out.sweep_ntiles = nt;
    std::vector<SweepTile>& tiles = out.sweep_tiles;
    tiles.resize(S);
    std::vector<int> s0(nt + 1);
    for (int k = 0; k <= nt; ++k) s0[k] = S * k / nt;
    for (int k = 0; k < nt; ++k)
        for (int s = s0[k]; s < s0[k + 1]; ++s) tiles[s] = {k, s - s0[k], s0[k + 1] - s0[k]};
    // relative cost of a pair's batch: pivots of both passes, then each state
    auto cost = [&](int npair, int nst) { return (npair + 1) * (30.0 + 50.0 * nst); };
    double total = 0;
    for (const SweepChain& c : t.chains)
        for (int k = 0; k < nt; ++k) total += cost(c.npair, s0[k + 1] - s0[k]) * nb;
    const double target = total / (double)std::max<long long>(1, target_items);
    std::vector<SweepGroup>& groups = out.sweep_groups;
    groups.resize((size_t)t.npairs * nt);
    struct Unit { double cost; SweepItem a, b; bool two; };
    std::vector<Unit> units;
    long long off = 0;
    int npmax = 0;
    for (size_t ch = 0; ch < t.chains.size(); ++ch) {
        const SweepChain& c = t.chains[ch];
        const int2 half = t.halves[ch];
        const bool two = half.x > 0;
        npmax = std::max(npmax, two ? std::max(half.x, half.y) : c.npair);
        for (int k = 0; k < nt; ++k) {
            const int nst = s0[k + 1] - s0[k];
            out.sweep_nst = std::max(out.sweep_nst, nst);
            const double u = cost(two ? half.x : c.npair, nst);
            const int per = split ? 1 : std::max(1, std::min((int)std::lround(target / u), nb));  // batches per item
            const long long first = off;
            int nr = 0;
            for (int b = 0; b < nb; b += per) {
                const int b1 = std::min(nb, b + per), k0 = 64 * b, k1 = std::min(pl->N, 64 * b1);
                Unit x{u * (b1 - b), {c.pair0, c.npair, c.npair, s0[k], nst, k0, k1, -1, 0, off, 0}, {}, two};
                if (two) {
                    x.a.npair = half.x;
                    x.a.mid = c.pair0 + half.x;
                    x.a.mid_off = off + (long long)half.x * kSweepRec;
                    x.b = x.a;
                    x.b.pair0 = x.a.mid + 1;
                    x.b.npair = half.y;
                    x.b.half = 1;
                    x.b.part_off = x.a.mid_off + kSweepRec;
                }
                units.push_back(x);
                off += (long long)nst * c.npair * kSweepRec;
                ++nr;
            }
            for (int q = 0; q < c.npair; ++q)
                groups[(size_t)(c.pair0 + q) * nt + k] = {first / 2 + 3LL * q, nr, c.npair};
        }
    }
    // pairs of halves first (they start at even indices), each kind longest first
    std::stable_sort(units.begin(), units.end(), [](const Unit& x, const Unit& y) {
        return x.two != y.two ? x.two : x.cost > y.cost;
    });
    for (const Unit& x : units) {
        out.sweep_items.push_back(x.a);
        if (x.two) out.sweep_items.push_back(x.b);
    }
    out.part_size = (off + 1) / 2;
    out.sweep_stride = (long long)((npmax + kSweepBlock - 1) / kSweepBlock) * (1 + 2 * out.sweep_nst) * 64;
    out.rot_max = out.sweep_nst;
    if (short_chains) out.sweep_stride = 0;
    out.launches.push_back({2 * kSweepBlock, kSweepKind, 0, (int)out.sweep_items.size(), 1, out.sweep_nst});
    char buf[96];
    std::snprintf(buf, sizeof buf, "%s_items%lld%s", short_chains ? "sweep_short" : split ? "sweep2" : "sweep", (long long)out.sweep_items.size(),
                  out.sweep_nst > 1 ? "_shared" : "");
    out.name = buf;
    return REXI_OK;
}

void free_schedule(Schedule& s) {
    s.on_device = false;
    dev_free(s.d_sweep_items);
    dev_free(s.d_sweep_tiles);
    dev_free(s.d_sweep_groups);
    dev_free(s.d_minfo);
    dev_free(s.d_items);
    dev_free(s.d_groups);
}

// Each graph is destroyed only after its last launch has completed (its
// buffers may be freed or reused right after: grow, schedule and
// stream changes).
void drop_graphs(rexi_plan* pl) {
    for (auto& g : pl->graphs) {
        if (g.done) {
            (void)hipEventSynchronize(g.done);
            (void)hipEventDestroy(g.done);
        }
        (void)hipGraphExecDestroy(g.exec);
    }
    pl->graphs.clear();
    ++pl->graph_gen;
}

// A step enqueued on a capturing stream: the caller's graph holds the workspace.
void note_capture(rexi_plan* pl, hipStream_t s) {
    if (pl->captured) return;
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) != hipSuccess) (void)hipGetLastError();
    else pl->captured = st != hipStreamCaptureStatusNone;
}

// A buffer of at least n entries.  The buffers are shared by all state counts: once
// a caller has captured a step, smaller ones are kept until the plan is destroyed;
// else they are freed, before the new one is there only where both do not fit.
template <class T>
int grow(rexi_plan* pl, T** p, long long* capacity, long long n) {
    if (n <= *capacity) return REXI_OK;
    pl->retired.reserve(pl->retired.size() + 1);
    drop_graphs(pl);
    T* q = nullptr;
    int rc = dev_alloc(&q, (size_t)n);
    if (rc && !pl->captured && *p) {
        dev_free(*p);
        *capacity = 0;
        rc = dev_alloc(&q, (size_t)n);
    }
    if (rc) return rc;
    if (pl->captured && *p) pl->retired.push_back(*p);  // (room reserved)
    else dev_free(*p);
    *p = q;
    *capacity = n;
    return REXI_OK;
}

// Workspace of a schedule: partial sums; for a pole-per-lane schedule the
// records of S states and its scratch, one slot per workgroup, at most
// kSweepScratch bytes of them (workgroups beyond take several items in turn).
constexpr long long kSweepScratch = 1LL << 30;
struct Sizes {
    long long part = 0, rec = 0, scratch = 0, slot = 0;
    bool chains = false;  // the tiled solve's states
};

void add_sizes(const rexi_plan* pl, const Schedule& sc, Sizes& z) {
    z.part = std::max(z.part, sc.part_size);
    if (!sc.sweep) {
        z.chains = true;
        return;
    }
    z.rec = std::max(z.rec, (long long)(pl->sweep[sc.split].npairs + 1) * sc.S * kSweepRec + kSweepPad);
    if (sc.sweep_stride == 0) return;
    const long long most = std::max(1LL, kSweepScratch / 16 / kSweepWaves / sc.sweep_stride);
    const long long wgs = sweep_resident(sc) ? kSweepGroups : ((long long)sc.sweep_items.size() + kSweepWaves - 1) / kSweepWaves;
    z.slot = std::max(z.slot, kSweepWaves * sc.sweep_stride);
    z.scratch = std::max(z.scratch, std::min(wgs, most) * kSweepWaves * sc.sweep_stride);
}

// The states in chain layout, with the first tiled schedule or per-term step: the
// pole-per-lane schedules do not read them (64 states at T1023: 3.2 GB).
int ensure_chains(rexi_plan* pl) {
    int rc = REXI_OK;
    for (int d = 0; d < 2 && !rc; ++d) {
        if (!pl->d_ch_var[d]) rc = dev_alloc(&pl->d_ch_var[d], (size_t)pl->prm.max_states * (pl->nslots + 2));
        if (!rc && !pl->d_ch_phi[d]) rc = dev_alloc(&pl->d_ch_phi[d], (size_t)pl->prm.max_states * pl->nspec);
    }
    return rc;
}

// Every step checks its schedule's sizes here: the buffers are shared by all
// schedules, and a growth that failed may have left smaller ones.  Where memory is
// short, fewer slots of scratch do (their workgroups take more items in turn); what
// failed once is then tried again only by a call that selects a schedule (`retry`).
int ensure_sizes(rexi_plan* pl, const Sizes& z, bool retry) {
    int rc = z.chains ? ensure_chains(pl) : REXI_OK;
    if (!rc) rc = grow(pl, &pl->d_part, &pl->part_capacity, z.part);
    for (int d = 0; d < 2 && !rc; ++d) rc = grow(pl, &pl->d_rec[d], &pl->rec_capacity[d], z.rec);
    if (rc) return rc;
    if (!retry && pl->sweep_scratch_capacity >= z.slot && z.scratch >= pl->scratch_refused) return REXI_OK;
    rc = grow(pl, &pl->d_sweep_scratch, &pl->sweep_scratch_capacity, z.scratch);
    if (rc == REXI_ENOMEM) pl->scratch_refused = z.scratch;
    for (long long n = z.scratch; rc == REXI_ENOMEM && n > z.slot;) {
        n = std::max(z.slot, n / 2);
        rc = grow(pl, &pl->d_sweep_scratch, &pl->sweep_scratch_capacity, n);
    }
    return rc;
}

// The device side of a schedule, once: its lists and the tables that it reads.
int upload_schedule(rexi_plan* pl, Schedule& sc) {
    if (sc.on_device) return REXI_OK;
    int rc = REXI_OK;
    if (sc.sweep) {
        rc = build_sweep_tables(pl, sc.split);
        if (!rc) rc = upload(&sc.d_sweep_items, sc.sweep_items);
        if (!rc) rc = upload(&sc.d_sweep_tiles, sc.sweep_tiles);
        if (!rc) rc = upload(&sc.d_sweep_groups, sc.sweep_groups);
    } else {
        rc = upload(&sc.d_minfo, sc.minfo);
        if (!rc) rc = upload(&sc.d_items, sc.items);
        if (!rc) rc = upload(&sc.d_groups, sc.groups);
    }
    if (rc) {
        free_schedule(sc);
        return rc;
    }
    sc.on_device = true;
    return REXI_OK;
}

// The tiled schedules' default for S states: "fine", ~2816 items, one launch per
// item, states sharing factorisations where that measured faster.  (Item targets:
// ~2816 measured fastest at T256, four states per item and concurrent classes, by
// 3% over ~4096, with ~2048 and ~3072 on either side slower.)
constexpr int kTiledPolicy = 5;
constexpr long long kTiledTarget = 2816;
int tiled_rot(int S) { return S % 2 == 0 ? 2 : 0; }

// The pole-per-lane solve's default: one pole per lane wherever the operator
// allows it, which with the states of an item chosen as below beats the tiled
// schedules at every size, state count and number of poles measured (T15 to T1023, 1
// to 64 states, 25 to 8215 poles; the least gains are 8 to 11%, at T127 with four
// states and 129 poles and at T256 with 16 states and 39 poles).  ~8192 items (four per
// wave slot of the chip) against ~4096 at T256 with four states: 1527 / 1570 us per
// step; within 1% of each other elsewhere.
long long sweep_waves(const rexi_plan* pl, int S, int most) {
    return 2LL * (pl->T + 1) * ((S + most - 1) / most) * ((pl->N + 63) / 64);
}
constexpr long long kSweepTarget = 8192;

// States of an item: up to kSweepStates share a pole's pivots, but one after the
// other.  Where few poles or short chains leave the chip idle, an item's time is what
// counts (T127, 25 poles, by states of an item 1 / 2 / 4: 30 / 42 / 70 us a step, the
// tiled schedule 51), so an item takes one state, or else two, where the waves are at
// most kTileWaves, or where registers hold the chains so that kShortWaves is the
// limit.  Four states, 1 / 2 / 4 of them an item: T127, 25 poles 33 / 44 / 70; T256, 25
// poles 92 (2056 waves) / 90 (1028) / 141; six states, T100, 151 poles 53 (3636) / 58
// (1818) / 54 (1212, three an item).
constexpr long long kTileWaves = 1500;

int default_sweep_schedule(rexi_plan* pl, int S, Schedule& out) {
    const bool split = sweep_waves(pl, S, kSweepStates) <= kSplitWaves;
    if (split) {
        for (int most : {1, 2, kSweepStates})
            if (sweep_waves(pl, S, most) <= kSplitWaves) {
                const int rc = build_sweep_schedule(pl, S, most, 0, true, true, out);
                if (rc != REXI_EUNSUPPORTED) return rc;
            }
        for (int most : {1, 2})
            if (sweep_waves(pl, S, most) <= kTileWaves) return build_sweep_schedule(pl, S, most, 0, true, false, out);
    }
    return build_sweep_schedule(pl, S, kSweepStates, split ? 0 : kSweepTarget, split, false, out);
}

// Uploads schedule `sc` and, where the no-allocation step's array does not hold
// it, before it the tiled schedule that takes that step in its place.
int upload_with_tiled(rexi_plan* pl, Schedule& sc, Schedule* tiled) {
    int rc = tiled && !noalloc_takes(pl, sc) ? upload_schedule(pl, *tiled) : REXI_OK;
    if (!rc) rc = upload_schedule(pl, sc);
    return rc;
}

// Entries of S states in the plan's lists; sched, by whose size the entries are
// looked up, last.
void room_for(rexi_plan* pl, int S) {
    const size_t n = (size_t)S + 1;
    if (pl->sched.size() >= n) return;
    pl->first.resize(n);
    pl->first_tiled.resize(n);
    pl->chosen.resize(n, -1);
    pl->own.resize(n, -1);
    pl->tiled.resize(n, -1);
    pl->sched.resize(n);
}

// The default schedule of S states alone, for the first step; the candidate list,
// of which it is a part, is built by the first call that asks for it.  A new
// plan's first step, with all of the list built and uploaded in it / the default
// alone: T301, three states, 21 / 4 ms; T256, four states, 39 / 5 ms; T15, two
// states, 7.9 / 0.4 ms.  REXI_EUNSUPPORTED: the default is a tiled schedule.
int first_schedule(rexi_plan* pl, int S) {
    room_for(pl, S);
    Schedule &sc = pl->first[S], &t = pl->first_tiled[S];
    Sizes z;
    if (sc.on_device) {
        add_sizes(pl, sc, z);
        return ensure_sizes(pl, z, false);
    }
    const bool split = sweep_waves(pl, S, kSweepStates) <= kSplitWaves;
    int rc = build_sweep_tables(pl, split);
    if (rc) return rc;
    if (!pl->sweep[split].usable) return REXI_EUNSUPPORTED;
    rc = default_sweep_schedule(pl, S, sc);
    if (rc) return rc;
    bool tiled = !t.on_device && !noalloc_takes(pl, sc);
    if (tiled && (build_schedule(pl, S, kTiledPolicy, kTiledTarget, false, tiled_rot(S), t) != REXI_OK ||
                  (int)t.launches.size() > kMaxLaunches)) {
        t = Schedule();  // the no-allocation step refuses then
        tiled = false;
    }
    rc = upload_with_tiled(pl, sc, tiled ? &t : nullptr);
    if (rc) return rc;
    add_sizes(pl, sc, z);  // last: the scratch takes what memory there is
    return ensure_sizes(pl, z, false);
}

// Candidate schedules for S states (built on first use, on the host only; those
// that run are uploaded).  all: the workspace holds any of them afterwards.
int schedules_for(rexi_plan* pl, int S, bool all, std::vector<Schedule>** out) {
    room_for(pl, S);
    std::vector<Schedule>& c = pl->sched[S];
    if (c.empty()) {
        const long long tg[] = {2048, kTiledTarget, 4096, 8192};
        // states per item (see build_schedule): one (each state factorises
        // its own poles), and for an even number of states up to four sharing
        // each factorisation, in every tile class or in some
        std::vector<int> rots = {0};
        if (S % 2 == 0) {
            rots.push_back(1);
            rots.push_back(2);
        }
        const bool few = sweep_waves(pl, S, kSweepStates) <= kSplitWaves;
        int rc = build_sweep_tables(pl, few);
        if (rc) return rc;
        Schedule own;  // the pole-per-lane default, for its name
        if (pl->sweep[few].usable && (rc = default_sweep_schedule(pl, S, own))) return rc;
        std::vector<Schedule> list;
        int tiled = -1, dflt = -1, from_first = -1, from_tiled = -1;
        for (int rot : rots)
        for (int persistent = 0; persistent < 2; ++persistent)
            for (int policy = 0; policy < kPolicies; ++policy)
                for (long long t : tg) {
                    Schedule sc;
                    rc = build_schedule(pl, S, policy, t, false, rot, sc);
                    if (rc == REXI_EUNSUPPORTED) continue;
                    if (rc) return rc;
                    if ((int)sc.launches.size() > kMaxLaunches) continue;
                    sc.persistent = persistent != 0;
                    if (sc.persistent) sc.name = "persistent_" + sc.name;
                    if (!persistent && policy == kTiledPolicy && t == kTiledTarget && rot == tiled_rot(S)) {
                        tiled = (int)list.size();
                        if (pl->first_tiled[S].on_device) from_tiled = tiled;
                    }
                    list.push_back(std::move(sc));
                }
        dflt = tiled;
        for (int persistent = 0; pl->sweep[few].usable && persistent < 2; ++persistent)
            for (int most : {kSweepStates, 2, 1}) {
                if (most < kSweepStates && (S <= most || sweep_waves(pl, S, most) > kSplitWaves)) continue;
                for (long long t : {4096LL, kSweepTarget, 0LL, -1LL}) {  // 0: split chains, -1: split and in registers
                    Schedule sc;
                    if (t <= 0 ? !few : most < kSweepStates) continue;
                    rc = build_sweep_schedule(pl, S, most, t, t <= 0, t < 0, sc);
                    if (rc == REXI_EUNSUPPORTED) continue;
                    if (rc) return rc;
                    sc.persistent = persistent != 0;
                    if (sc.persistent) sc.name = "persistent_" + sc.name;
                    if (t != 4096 && sc.name == own.name) {
                        dflt = (int)list.size();
                        if (pl->first[S].on_device) from_first = dflt;
                    }
                    list.push_back(std::move(sc));
                }
            }
        if (list.empty()) return fail(REXI_EUNSUPPORTED, "no schedule fits this truncation");
        // the device copies of the first step's schedules move with them
        if (from_first >= 0) list[from_first] = std::exchange(pl->first[S], Schedule());
        if (from_tiled >= 0) list[from_tiled] = std::exchange(pl->first_tiled[S], Schedule());
        c = std::move(list);
        pl->tiled[S] = tiled;
        pl->chosen[S] = pl->own[S] = dflt >= 0 ? dflt : 0;
    }
    *out = &c;
    const int rc = upload_with_tiled(pl, c[pl->chosen[S]], pl->tiled[S] >= 0 ? &c[pl->tiled[S]] : nullptr);
    if (rc) return rc;
    Sizes z;
    for (int i = 0; i < (int)c.size(); ++i)
        if (all || i == pl->chosen[S]) add_sizes(pl, c[i], z);
    return ensure_sizes(pl, z, all);
}

bool overlaps(const void* a, size_t na, const void* b, size_t nb) {
    const char* x = (const char*)a;
    const char* y = (const char*)b;
    return x < y + nb && y < x + na;
}


// The graph of one step for (S, direction, input buffer): solve launches and
// the reduction into the other chain buffer, captured on the plan's stream.
int step_graph(rexi_plan* pl, const Schedule& sc, int S, int adjoint, int buf, hipGraphExec_t* out,
               hipEvent_t* done) {
    for (auto& g : pl->graphs)
        if (g.sched == &sc && g.S == S && g.adjoint == adjoint && g.buf == buf && g.gen == pl->graph_gen) {
            *out = g.exec;
            *done = g.done;
            return REXI_OK;
        }
    pl->graphs.reserve(pl->graphs.size() + 1);
    hipGraph_t graph = nullptr;
    REXI_HIP(hipStreamBeginCapture(pl->cap_stream, hipStreamCaptureModeThreadLocal));
    const Workspace ws = plan_workspace(pl, sc);
    hipError_t e1 = enqueue_solve(pl, ws, sc, buf, S, adjoint, pl->cap_stream);
    hipError_t e2 = hipSuccess;
    if (e1 == hipSuccess)
        e2 = enqueue_reduce(pl, ws, sc, ws.part, buf, buf ^ 1, nullptr, S, adjoint, pl->d_slot_m, pl->cap_stream);
    hipError_t e3 = hipStreamEndCapture(pl->cap_stream, &graph);
    if (e1 != hipSuccess) { if (graph) (void)hipGraphDestroy(graph); return hip_fail(e1, "capture solve"); }
    if (e2 != hipSuccess) { if (graph) (void)hipGraphDestroy(graph); return hip_fail(e2, "capture reduce"); }
    if (e3 != hipSuccess) return hip_fail(e3, "hipStreamEndCapture");
    hipGraphExec_t exec = nullptr;
    hipError_t e4 = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e4 != hipSuccess) return hip_fail(e4, "hipGraphInstantiate");
    hipEvent_t ev = nullptr;
    hipError_t e5 = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
    if (e5 != hipSuccess) {
        (void)hipGraphExecDestroy(exec);
        return hip_fail(e5, "hipEventCreateWithFlags");
    }
    pl->graphs.push_back({&sc, S, adjoint, buf, pl->graph_gen, exec, ev});
    *out = exec;
    *done = ev;
    return REXI_OK;
}

}  // namespace

int run_sweep_steps(rexi_plan* pl, const Workspace& ws, const Schedule& sc, const void* u0, void* u1, int S,
                    int nsteps, int adjoint, bool timed, hipStream_t s) {
    REXI_HIP(enqueue_sweep_prep(pl, ws, sc, u0, 0, S, adjoint, s));
    int cur = 0;
    for (int k = 0; k < nsteps; ++k) {
        const bool last = (k == nsteps - 1);
        if (timed) REXI_HIP(timed_begin(pl, REXI_KERNEL_SOLVE, s));
        REXI_HIP(enqueue_sweep_solve(pl, ws, sc, cur, S, adjoint, s));
        if (timed && !pl->use_graphs) REXI_HIP(timed_end(pl, REXI_KERNEL_SOLVE, s));
        REXI_HIP(enqueue_sweep_reduce(pl, ws, sc, cur, cur ^ 1, last ? u1 : nullptr, S, adjoint, s));
        if (timed && pl->use_graphs) REXI_HIP(timed_end(pl, REXI_KERNEL_SOLVE, s));
        cur ^= 1;
    }
    return REXI_OK;
}

namespace {

int run_steps(rexi_plan* pl, const Schedule& sc, const void* u0, void* u1, int S, int nsteps, int adjoint,
              hipStream_t s) {
    const size_t bytes = (size_t)S * 3 * pl->nspec * 16;
    if (nsteps == 0) {
        REXI_HIP(hipMemcpyAsync(u1, u0, bytes, hipMemcpyDeviceToDevice, s));
        return REXI_OK;
    }
    const Workspace ws = plan_workspace(pl, sc);
    if (sc.sweep) return run_sweep_steps(pl, ws, sc, u0, u1, S, nsteps, adjoint, true, s);
    REXI_HIP(enqueue_prep(pl, ws, u0, 0, S, adjoint, pl->sched_layout, s));
    int cur = 0;
    if (pl->use_graphs) {
        // captured step graphs (solve + reduction), then the final layout
        // change; with timing on, each replay is bracketed by an event pair
        for (int k = 0; k < nsteps; ++k) {
            hipGraphExec_t exec = nullptr;
            hipEvent_t done = nullptr;
            int rc = step_graph(pl, sc, S, adjoint, cur, &exec, &done);
            if (rc) return rc;
            REXI_HIP(timed_begin(pl, REXI_KERNEL_SOLVE, s));
            REXI_HIP(hipGraphLaunch(exec, s));
            REXI_HIP(timed_end(pl, REXI_KERNEL_SOLVE, s));
            REXI_HIP(hipEventRecord(done, s));
            cur ^= 1;
        }
        REXI_HIP(enqueue_finish(pl, ws, cur, u1, S, adjoint, pl->sched_layout, s));
        return REXI_OK;
    }
    for (int k = 0; k < nsteps; ++k) {
        const bool last = (k == nsteps - 1);
        REXI_HIP(timed_begin(pl, REXI_KERNEL_SOLVE, s));
        REXI_HIP(enqueue_solve(pl, ws, sc, cur, S, adjoint, s));
        REXI_HIP(timed_end(pl, REXI_KERNEL_SOLVE, s));
        REXI_HIP(enqueue_reduce(pl, ws, sc, ws.part, cur, cur ^ 1, last ? u1 : nullptr, S, adjoint, pl->d_slot_m, s));
        cur ^= 1;
    }
    return REXI_OK;
}

}  // namespace

int check_state_call(rexi_plan* pl, const void* in, const void* out, int S, int nsteps) {
    if (!pl) return fail(REXI_EINVAL, "plan is NULL");
    if (!in || !out) return fail(REXI_EINVAL, "state pointer is NULL");
    if (S < 1) return fail(REXI_EINVAL, "S must be >= 1");
    if (S > pl->prm.max_states) return fail(REXI_EUNSUPPORTED, "S exceeds the plan's max_states");
    if (nsteps < 0) return fail(REXI_EINVAL, "nsteps must be >= 0");
    const size_t bytes = (size_t)S * 3 * pl->nspec * 16;
    if (overlaps(in, bytes, out, bytes)) return fail(REXI_EALIAS, "output overlaps input");
    return REXI_OK;
}

}  // namespace rexi

using namespace rexi;

namespace {

// f-sphere steps: the closed-form kernel takes all of them at once.
int run_fsphere(rexi_plan* pl, const void* u0, void* u1, int S, int nsteps, int adjoint, hipStream_t s) {
    if (nsteps == 0) {
        REXI_HIP(hipMemcpyAsync(u1, u0, (size_t)S * 3 * pl->nspec * 16, hipMemcpyDeviceToDevice, s));
        return REXI_OK;
    }
    REXI_HIP(enqueue_fsphere_steps(pl, u0, u1, S, nsteps, adjoint, s));
    return REXI_OK;
}

int do_step(rexi_plan* pl, const void* u0, void* u1, int S, int nsteps, int adjoint, void* stream) {
    int rc = check_state_call(pl, u0, u1, S, nsteps);
    if (rc) return rc;
    if (pl->prm.fsphere) return run_fsphere(pl, u0, u1, S, nsteps, adjoint, (hipStream_t)stream);
    note_capture(pl, (hipStream_t)stream);
    const Schedule* sc = nullptr;
    if ((int)pl->sched.size() <= S || pl->sched[S].empty()) {
        rc = first_schedule(pl, S);
        if (rc && rc != REXI_EUNSUPPORTED) return rc;
        if (!rc) sc = &pl->first[S];
    }
    if (!sc) {
        std::vector<Schedule>* c = nullptr;
        rc = schedules_for(pl, S, false, &c);
        if (rc) return rc;
        sc = &(*c)[pl->chosen[S]];
    }
    return run_steps(pl, *sc, u0, u1, S, nsteps, adjoint, (hipStream_t)stream);
}

void drop_events(rexi_plan* pl) {
    for (auto& v : pl->events) {
        for (auto& ab : v) {
            (void)hipEventDestroy(ab.first);
            (void)hipEventDestroy(ab.second);
        }
        v.clear();
    }
}

void release(rexi_plan* pl) {
    drop_events(pl);
    drop_graphs(pl);
    dev_free(pl->d_counters);
    if (pl->cap_stream) (void)hipStreamDestroy(pl->cap_stream);
    pl->cap_stream = nullptr;
    for (int c = 0; c < kMaxLaunches; ++c) {
        if (pl->side[c]) (void)hipStreamDestroy(pl->side[c]);
        if (pl->join_ev[c]) (void)hipEventDestroy(pl->join_ev[c]);
        pl->side[c] = nullptr;
        pl->join_ev[c] = nullptr;
    }
    if (pl->fork_ev) (void)hipEventDestroy(pl->fork_ev);
    pl->fork_ev = nullptr;
    for (auto& c : pl->sched)
        for (auto& s : c) free_schedule(s);
    for (auto& s : pl->per_term) free_schedule(s);
    for (auto& s : pl->first) free_schedule(s);
    for (auto& s : pl->first_tiled) free_schedule(s);
    for (void* p : pl->retired) (void)hipFree(p);
    pl->retired.clear();
    dev_free(pl->d_th);
    dev_free(pl->d_om);
    dev_free(pl->d_cc);
    dev_free(pl->d_sc);
    dev_free(pl->d_idx_n);
    dev_free(pl->d_idx_m);
    for (int d = 0; d < 2; ++d) {
        dev_free(pl->d_poles[d]);
        dev_free(pl->d_ch_var[d]);
        dev_free(pl->d_ch_phi[d]);
    }
    dev_free(pl->d_part);
    dev_free(pl->d_acc);
    dev_free(pl->d_fs_poles);
    dev_free(pl->sched_layout);
    dev_free(pl->d_slot_m);
    for (auto& t : pl->sweep) free_sweep_tables(t);
    dev_free(pl->d_rec[0]);
    dev_free(pl->d_rec[1]);
    dev_free(pl->d_sweep_scratch);
    sh_release(pl);
}

std::vector<double2> to_d2(const std::vector<std::complex<double>>& v) {
    std::vector<double2> o(v.size());
    for (size_t i = 0; i < v.size(); ++i) o[i] = make_double2(v[i].real(), v[i].imag());
    return o;
}

struct Destroy {
    void operator()(rexi_plan* pl) const {
        release(pl);
        delete pl;
    }
};

int create(const rexi_params* p, rexi_plan** out) {
    int rc = check_params(p);
    if (rc) return rc;
    std::unique_ptr<rexi_plan, Destroy> own(new rexi_plan());
    rexi_plan* const pl = own.get();
    pl->prm = *p;
    const int T = p->T;
    pl->T = T;
    pl->N = 2 * (p->M + p->L) + 1;
    pl->nspec = nspec_of(T);
    pl->nslots = 2 * (pl->nspec - 1);
    pl->phibar = p->gravity * p->mean_depth;
    pl->poles = make_poles(p->M, p->h, p->L, p->normalize);
    const int N = pl->N;
    typedef std::complex<double> C;
    std::vector<C> ainv(N), wx[2], wy[2], wxa[2], wya[2];
    for (int d = 0; d < 2; ++d) {
        wx[d].resize(N);
        wy[d].resize(N);
        wxa[d].resize(N);
        wya[d].resize(N);
    }
    C g00(0, 0), gx[2] = {C(0, 0), C(0, 0)}, gy[2] = {C(0, 0), C(0, 0)};
    for (int k = 0; k < N; ++k) {
        const C a = pl->poles.alpha[k];
        ainv[k] = 1.0 / a;
        const C bp = pl->poles.beta_plus[k];
        const C bm_mirror = std::conj(pl->poles.beta_minus[N - 1 - k]);  // conj(beta-_{-k})
        wx[0][k] = bp;
        wy[0][k] = bm_mirror;
        wx[1][k] = bm_mirror;
        wy[1][k] = bp;
        for (int d = 0; d < 2; ++d) {
            wxa[d][k] = wx[d][k] / a;
            wya[d][k] = wy[d][k] / a;
            gx[d] += wxa[d][k];
            gy[d] += wya[d][k];
        }
        g00 += (pl->poles.beta_plus[k] + pl->poles.beta_minus[k]) / a;
    }
    pl->g00_fwd = g00;
    pl->g00_adj = std::conj(g00);
    pl->gphi_fwd = gx[0] + std::conj(gy[0]);
    pl->gphi_adj = gx[1] + std::conj(gy[1]);

    // per-(n, m) constants of the energy-scaled operator (times dt)
    const long long ns = pl->nspec;
    std::vector<double> th(ns), om(ns), cc(ns), sc(ns);
    std::vector<int> in(ns), im(ns);
    const long double a = p->radius, Om = p->omega, pb = pl->phibar, dt = p->dt;
    for (int m = 0; m <= T; ++m)
        for (int n = m; n <= T; ++n) {
            const long long i = spec_offset(T, m) + (n - m);
            in[i] = n;
            im[i] = m;
            if (n == 0) {
                th[i] = om[i] = cc[i] = 0.0;
                sc[i] = 1.0;
                continue;
            }
            const long double nn = (long double)n * (n + 1);
            th[i] = (double)(2 * Om * m / nn * dt);
            om[i] = (double)(sqrtl(pb * nn) / a * dt);
            const long double kap = eps_nm(n, m) * sqrtl((long double)n * n - 1) / n;
            cc[i] = (double)(2 * Om * dt * kap);
            sc[i] = (double)(a * sqrtl(pb / nn));
        }
    std::vector<MInfo> lay = chain_layout(T);
    std::vector<int> slot_m(pl->nslots);
    for (int m = 0; m <= T; ++m)
        for (int q = 0; q < 2 * lay[m].L; ++q) slot_m[lay[m].slot_base + q] = m;

    rc = upload(&pl->d_th, th);
    if (!rc) rc = upload(&pl->d_om, om);
    if (!rc) rc = upload(&pl->d_cc, cc);
    if (!rc) rc = upload(&pl->d_sc, sc);
    if (!rc) rc = upload(&pl->d_idx_n, in);
    if (!rc) rc = upload(&pl->d_idx_m, im);
    for (int d = 0; d < 2 && !rc; ++d) {
        std::vector<std::complex<double>> pd;
        pd.reserve(6 * (size_t)N);
        for (int k = 0; k < N; ++k) {
            pd.push_back(pl->poles.alpha[k]);
            pd.push_back(ainv[k]);
            pd.push_back(wx[d][k]);
            pd.push_back(wy[d][k]);
            pd.push_back(wxa[d][k]);
            pd.push_back(wya[d][k]);
        }
        rc = upload(&pl->d_poles[d], to_d2(pd));
    }
    if (!rc) rc = upload(&pl->sched_layout, lay);
    if (!rc) rc = upload(&pl->d_slot_m, slot_m);
    if (!rc && p->fsphere) {
        pl->f0dt = p->f0 * p->dt;
        std::vector<std::complex<double>> fp;
        fp.reserve(3 * (size_t)N);
        for (int k = 0; k < N; ++k) {
            fp.push_back(pl->poles.alpha[k]);
            fp.push_back(pl->poles.beta_plus[k]);
            fp.push_back(pl->poles.beta_minus[k]);
        }
        rc = upload(&pl->d_fs_poles, to_d2(fp));
    }
    if (!rc) rc = dev_alloc(&pl->d_counters, kMaxLaunches);
    if (!rc) {
        hipError_t e = hipMemset(pl->d_counters, 0, kMaxLaunches * sizeof(int));
        if (e != hipSuccess) rc = hip_fail(e, "hipMemset");
    }
    if (!rc) {
        hipError_t e = hipStreamCreateWithFlags(&pl->cap_stream, hipStreamNonBlocking);
        if (e != hipSuccess) rc = hip_fail(e, "hipStreamCreateWithFlags");
    }
    for (int c = 0; c < kMaxLaunches && !rc; ++c) {
        hipError_t e = hipStreamCreateWithFlags(&pl->side[c], hipStreamNonBlocking);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&pl->join_ev[c], hipEventDisableTiming);
        if (e != hipSuccess) rc = hip_fail(e, "side stream / event");
    }
    if (!rc) {
        hipError_t e = hipEventCreateWithFlags(&pl->fork_ev, hipEventDisableTiming);
        if (e != hipSuccess) rc = hip_fail(e, "hipEventCreateWithFlags");
    }
    if (!rc) {
        hipError_t e = hipGetDevice(&pl->device);
        if (e != hipSuccess) rc = hip_fail(e, "hipGetDevice");
    }
    // the no-allocation step's workspace on this device (looked up once per device)
    if (!rc) rc = scratch_setup(&pl->scratch, &pl->scratch_bytes);
    if (!rc && p->nlat > 0) rc = sh_setup(pl);
    if (rc) return rc;
    *out = own.release();
    return REXI_OK;
}

}  // namespace

extern "C" {

const char* rexi_last_error(void) { return g_err.c_str(); }

int rexi_coeffs(int M, double h, int L, int normalize, int capacity, double* alpha, double* beta_plus,
                double* beta_minus, int* n_poles) try {
    g_err.clear();
    if (M < 1 || M > 1 << 20) return fail(REXI_EINVAL, "M must be in [1, 2^20]");
    if (!(h > 0) || !std::isfinite(h)) return fail(REXI_EINVAL, "h must be positive");
    if (L < 1 || L > 32) return fail(REXI_EINVAL, "L must be in [1, 32]");
    if (capacity < 0) return fail(REXI_EINVAL, "capacity must be >= 0");
    const int N = 2 * (M + L) + 1;
    if (n_poles) *n_poles = N;
    if (capacity == 0) return REXI_OK;
    if (capacity < N) return fail(REXI_EINVAL, "capacity below the number of poles");
    if (!alpha || !beta_plus || !beta_minus) return fail(REXI_EINVAL, "output array is NULL");
    const Poles P = make_poles(M, h, L, normalize);
    for (int k = 0; k < N; ++k) {
        alpha[2 * k] = P.alpha[k].real();
        alpha[2 * k + 1] = P.alpha[k].imag();
        beta_plus[2 * k] = P.beta_plus[k].real();
        beta_plus[2 * k + 1] = P.beta_plus[k].imag();
        beta_minus[2 * k] = P.beta_minus[k].real();
        beta_minus[2 * k + 1] = P.beta_minus[k].imag();
    }
    return REXI_OK;
} catch (...) {
    return caught();
}

int rexi_plan_create(const rexi_params* p, rexi_plan** out) try {
    if (!out) return fail(REXI_EINVAL, "out is NULL");
    *out = nullptr;
    return create(p, out);
} catch (...) {
    return caught();
}

int rexi_plan_destroy(rexi_plan* plan) try {
    if (!plan) return fail(REXI_EINVAL, "plan is NULL");
    release(plan);
    delete plan;
    return REXI_OK;
} catch (...) {
    return caught();
}

int rexi_plan_info(const rexi_plan* plan, int* n_poles, int* nspec, long long* blocks) try {
    if (!plan) return fail(REXI_EINVAL, "plan is NULL");
    if (n_poles) *n_poles = plan->N;
    if (nspec) *nspec = (int)plan->nspec;
    if (blocks) *blocks = (long long)plan->N * (plan->T + 1);
    return REXI_OK;
} catch (...) {
    return caught();
}

int rexi_plan_coeffs(const rexi_plan* plan, double* alpha, double* beta_plus, double* beta_minus) try {
    if (!plan || !alpha || !beta_plus || !beta_minus) return fail(REXI_EINVAL, "NULL argument");
    for (int k = 0; k < plan->N; ++k) {
        alpha[2 * k] = plan->poles.alpha[k].real();
        alpha[2 * k + 1] = plan->poles.alpha[k].imag();
        beta_plus[2 * k] = plan->poles.beta_plus[k].real();
        beta_plus[2 * k + 1] = plan->poles.beta_plus[k].imag();
        beta_minus[2 * k] = plan->poles.beta_minus[k].real();
        beta_minus[2 * k + 1] = plan->poles.beta_minus[k].imag();
    }
    return REXI_OK;
} catch (...) {
    return caught();
}

int rexi_step(rexi_plan* plan, const void* u0, void* u1, int S, int nsteps, void* stream) try {
    return do_step(plan, u0, u1, S, nsteps, 0, stream);
} catch (...) {
    return caught();
}

int rexi_step_adjoint(rexi_plan* plan, const void* g1, void* g0, int S, int nsteps, void* stream) try {
    return do_step(plan, g1, g0, S, nsteps, 1, stream);
} catch (...) {
    return caught();
}

int rexi_step_per_term(rexi_plan* plan, const void* u0, void* u1, int S, void* stream) try {
    int rc = check_state_call(plan, u0, u1, S, 1);
    if (rc) return rc;
    if (plan->prm.fsphere) return fail(REXI_EUNSUPPORTED, "the per-term form is not built for f-sphere plans");
    if ((int)plan->per_term.size() <= S) plan->per_term.resize(S + 1);
    Schedule& sc = plan->per_term[S];
    if (!sc.on_device) {
        rc = build_schedule(plan, S, 0, 0, true, 0, sc);  // 8 elements per lane, one wave per chain
        if (!rc) rc = upload_schedule(plan, sc);
        if (rc) return rc;
    }
    hipStream_t s = (hipStream_t)stream;
    note_capture(plan, s);
    rc = grow(plan, &plan->d_acc, &plan->acc_capacity, sc.part_size);
    if (!rc) rc = ensure_chains(plan);
    if (rc) return rc;
    const Workspace ws = plan_workspace(plan, sc);
    REXI_HIP(enqueue_prep(plan, ws, u0, 0, S, 0, plan->sched_layout, s));
    REXI_HIP(enqueue_zero(plan->d_acc, sc.part_size, s));
    for (int k = 0; k < plan->N; ++k) REXI_HIP(enqueue_per_term_pole(plan, ws, sc, k, 0, S, s));
    REXI_HIP(enqueue_reduce(plan, ws, sc, plan->d_acc, 0, 1, u1, S, 0, plan->d_slot_m, s));
    return REXI_OK;
} catch (...) {
    return caught();
}

int rexi_plan_set_schedule(rexi_plan* plan, int S, int index, int* count) try {
    if (!plan) return fail(REXI_EINVAL, "plan is NULL");
    if (plan->prm.fsphere) return fail(REXI_EUNSUPPORTED, "f-sphere plans have no schedules");
    if (S < 1 || S > plan->prm.max_states) return fail(REXI_EINVAL, "S out of range");
    std::vector<Schedule>* c = nullptr;
    int rc = schedules_for(plan, S, index >= 0, &c);
    if (rc) return rc;
    if (count) *count = (int)c->size();
    if (index < 0) return REXI_OK;
    if (index >= (int)c->size()) return fail(REXI_EINVAL, "schedule index out of range");
    const int was = plan->chosen[S];
    if (was != index) drop_graphs(plan);
    plan->chosen[S] = index;
    rc = schedules_for(plan, S, true, &c);
    if (rc) plan->chosen[S] = was;
    return rc;
} catch (...) {
    return caught();
}

int rexi_plan_get_schedule(rexi_plan* plan, int S, int* index) try {
    if (!plan || !index) return fail(REXI_EINVAL, "NULL argument");
    if (plan->prm.fsphere) return fail(REXI_EUNSUPPORTED, "f-sphere plans have no schedules");
    if (S < 1 || S > plan->prm.max_states) return fail(REXI_EINVAL, "S out of range");
    std::vector<Schedule>* c = nullptr;
    int rc = schedules_for(plan, S, false, &c);
    if (rc) return rc;
    *index = plan->chosen[S];
    return REXI_OK;
} catch (...) {
    return caught();
}

int rexi_plan_autotune(rexi_plan* plan, int S, void* stream, int* chosen) try {
    if (!plan) return fail(REXI_EINVAL, "plan is NULL");
    if (plan->prm.fsphere) return fail(REXI_EUNSUPPORTED, "f-sphere plans have no schedules");
    if (S < 1 || S > plan->prm.max_states) return fail(REXI_EINVAL, "S out of range");
    std::vector<Schedule>* c = nullptr;
    int rc = schedules_for(plan, S, true, &c);
    if (rc) return rc;
    struct Held {
        hipStream_t s;
        void *u0 = nullptr, *u1 = nullptr;
        hipEvent_t a = nullptr, b = nullptr;
        ~Held() {
            if (a) (void)hipEventDestroy(a);
            if (b) (void)hipEventDestroy(b);
            (void)hipStreamSynchronize(s);
            (void)hipFree(u0);
            (void)hipFree(u1);
        }
    } held{(hipStream_t)stream};
    hipStream_t& s = held.s;
    void *&u0 = held.u0, *&u1 = held.u1;
    hipEvent_t &a = held.a, &b = held.b;
    const size_t bytes = (size_t)S * 3 * plan->nspec * 16;
    hipError_t e = hipMalloc(&u0, bytes);
    if (e == hipSuccess) e = hipMalloc(&u1, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return hip_fail(e, "hipMalloc");
    }
    int fastest[2] = {-1, -1};  // of the ordinary and of the persistent schedules
    float fastest_ms[2] = {0, 0};
    rc = REXI_OK;
    do {
        if ((e = hipMemsetAsync(u0, 0, bytes, s)) != hipSuccess) { rc = hip_fail(e, "hipMemsetAsync"); break; }
        if ((e = hipEventCreate(&a)) != hipSuccess || (e = hipEventCreate(&b)) != hipSuccess) {
            rc = hip_fail(e, "hipEventCreate");
            break;
        }
        for (int i = 0; i < (int)c->size() && !rc; ++i) {
            Schedule& sc = (*c)[i];
            rc = upload_schedule(plan, sc);
            if (!rc) rc = run_steps(plan, sc, u0, u1, S, 1, 0, s);
            if (rc) break;
            if ((e = hipEventRecord(a, s)) != hipSuccess) { rc = hip_fail(e, "hipEventRecord"); break; }
            rc = run_steps(plan, sc, u0, u1, S, 3, 0, s);
            if (rc) break;
            if ((e = hipEventRecord(b, s)) != hipSuccess) { rc = hip_fail(e, "hipEventRecord"); break; }
            if ((e = hipEventSynchronize(b)) != hipSuccess) { rc = hip_fail(e, "hipEventSynchronize"); break; }
            float ms = 0;
            if ((e = hipEventElapsedTime(&ms, a, b)) != hipSuccess) { rc = hip_fail(e, "hipEventElapsedTime"); break; }
            const int k = sc.persistent;
            if (fastest[k] < 0 || ms < fastest_ms[k]) {
                fastest[k] = i;
                fastest_ms[k] = ms;
            }
        }
    } while (0);
    if (rc) return rc;
    // a persistent schedule, which the no-allocation step refuses, only where it is
    // clearly faster: timings one after another drift by 1 to 2% with the clock, and
    // the pole-per-lane twins run the same code where they are large
    const int best = fastest[0] < 0 || (fastest[1] >= 0 && fastest_ms[1] < 0.97f * fastest_ms[0]) ? fastest[1] : fastest[0];
    if (plan->chosen[S] != best) drop_graphs(plan);
    plan->chosen[S] = plan->own[S] = best;
    if (chosen) *chosen = best;
    return schedules_for(plan, S, true, &c);  // what the no-allocation step needs with it
} catch (...) {
    return caught();
}

int rexi_solve_variants(int per_term, int capacity, int* se, int* kind, int* states_per_item, int* count) try {
    if (capacity < 0) return fail(REXI_EINVAL, "capacity must be >= 0");
    const int n = solve_variant_list(per_term != 0, se, kind, states_per_item, capacity);
    if (count) *count = n;
    return REXI_OK;
} catch (...) {
    return caught();
}

int rexi_plan_schedule_classes(rexi_plan* plan, int S, int index, int capacity, int* se, int* kind,
                               int* states_per_item, int* count) try {
    if (!plan) return fail(REXI_EINVAL, "plan is NULL");
    if (plan->prm.fsphere) return fail(REXI_EUNSUPPORTED, "f-sphere plans have no schedules");
    if (S < 1 || S > plan->prm.max_states) return fail(REXI_EINVAL, "S out of range");
    if (capacity < 0) return fail(REXI_EINVAL, "capacity must be >= 0");
    const Schedule* sc = nullptr;
    if (index == -1) {
        if ((int)plan->per_term.size() <= S || !plan->per_term[S].on_device)
            return fail(REXI_EINVAL, "the per-term schedule for S is built by the first rexi_step_per_term call");
        sc = &plan->per_term[S];
    } else {
        std::vector<Schedule>* c = nullptr;
        int rc = schedules_for(plan, S, false, &c);
        if (rc) return rc;
        if (index < -1 || index >= (int)c->size()) return fail(REXI_EINVAL, "schedule index out of range");
        sc = &(*c)[index];
    }
    const int n = (int)sc->launches.size();
    for (int i = 0; i < n && i < capacity; ++i) {
        if (se) se[i] = sc->launches[i].SE;
        if (kind) kind[i] = sc->launches[i].kind;
        if (states_per_item) states_per_item[i] = sc->launches[i].rot;
    }
    if (count) *count = n;
    return REXI_OK;
} catch (...) {
    return caught();
}

int rexi_plan_schedule_name(rexi_plan* plan, int S, int index, char* buf, int capacity) try {
    if (!plan) return fail(REXI_EINVAL, "plan is NULL");
    if (!buf || capacity < 1) return fail(REXI_EINVAL, "buf is NULL or capacity < 1");
    buf[0] = 0;
    if (plan->prm.fsphere) return fail(REXI_EUNSUPPORTED, "f-sphere plans have no schedules");
    if (S < 1 || S > plan->prm.max_states) return fail(REXI_EINVAL, "S out of range");
    const Schedule* sc = nullptr;
    if (index == -1) {
        if ((int)plan->per_term.size() <= S || !plan->per_term[S].on_device)
            return fail(REXI_EINVAL, "the per-term schedule for S is built by the first rexi_step_per_term call");
        sc = &plan->per_term[S];
    } else {
        std::vector<Schedule>* c = nullptr;
        int rc = schedules_for(plan, S, false, &c);
        if (rc) return rc;
        if (index < -1 || index >= (int)c->size()) return fail(REXI_EINVAL, "schedule index out of range");
        sc = &(*c)[index];
    }
    std::snprintf(buf, (size_t)capacity, "%s", sc->name.c_str());
    return REXI_OK;
} catch (...) {
    return caught();
}

int rexi_plan_set_streams(rexi_plan* plan, int enable) try {
    if (!plan) return fail(REXI_EINVAL, "plan is NULL");
    const bool on = enable != 0;
    if (on != plan->concurrent) drop_graphs(plan);
    plan->concurrent = on;
    return REXI_OK;
} catch (...) {
    return caught();
}

int rexi_plan_set_graphs(rexi_plan* plan, int enable) try {
    if (!plan) return fail(REXI_EINVAL, "plan is NULL");
    plan->use_graphs = enable != 0;
    return REXI_OK;
} catch (...) {
    return caught();
}

int rexi_plan_set_timing(rexi_plan* plan, int enable) try {
    if (!plan) return fail(REXI_EINVAL, "plan is NULL");
    plan->timing = enable != 0;
    return REXI_OK;
} catch (...) {
    return caught();
}

int rexi_plan_kernel_time(rexi_plan* plan, int kernel, double* total_ms, long long* launches) try {
    if (!plan) return fail(REXI_EINVAL, "plan is NULL");
    if (kernel < 0 || kernel > 2) return fail(REXI_EINVAL, "unknown kernel");
    double tot = 0;
    long long n = 0;
    for (auto& ab : plan->events[kernel]) {
        REXI_HIP(hipEventSynchronize(ab.second));
        float ms = 0;
        REXI_HIP(hipEventElapsedTime(&ms, ab.first, ab.second));
        tot += ms;
        ++n;
        (void)hipEventDestroy(ab.first);
        (void)hipEventDestroy(ab.second);
    }
    plan->events[kernel].clear();
    if (total_ms) *total_ms = tot;
    if (launches) *launches = n;
    return REXI_OK;
} catch (...) {
    return caught();
}

int sh_forward(rexi_plan* plan, const double* grid, void* spec, int B, void* stream) try {
    if (!plan) return fail(REXI_EINVAL, "plan is NULL");
    return sh_run(plan, grid, spec, B, true, (hipStream_t)stream);
} catch (...) {
    return caught();
}

int sh_inverse(rexi_plan* plan, const void* spec, double* grid, int B, void* stream) try {
    if (!plan) return fail(REXI_EINVAL, "plan is NULL");
    return sh_run(plan, spec, grid, B, false, (hipStream_t)stream);
} catch (...) {
    return caught();
}

int sh_vortdiv_to_uv(rexi_plan* plan, const void* vd, long long stride, double* uv, int B, void* stream) try {
    if (!plan) return fail(REXI_EINVAL, "plan is NULL");
    return sh_vec_run(plan, vd, uv, stride, B, true, (hipStream_t)stream);
} catch (...) {
    return caught();
}

int sh_uv_to_vortdiv(rexi_plan* plan, const double* uv, void* vd, long long stride, int B, void* stream) try {
    if (!plan) return fail(REXI_EINVAL, "plan is NULL");
    return sh_vec_run(plan, uv, vd, stride, B, false, (hipStream_t)stream);
} catch (...) {
    return caught();
}

}  // extern "C"
