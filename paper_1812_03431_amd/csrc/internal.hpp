// Internal declarations shared by the library's host and device sources.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <complex>
#include <string>
#include <vector>

#include "../../include/rexi.h"

namespace rexi {

using cld = std::complex<long double>;

// ---------------------------------------------------------------- errors
int fail(int code, const std::string& msg);
int hip_fail(hipError_t e, const char* what);
int caught() noexcept;  // of a C entry whose body threw: the host's memory ran out
#define REXI_HIP(call)                                            \
    do {                                                          \
        hipError_t e_ = (call);                                   \
        if (e_ != hipSuccess) return ::rexi::hip_fail(e_, #call); \
    } while (0)

// ---------------------------------------------------------------- host math
// Gaussian rational fit (Section 4.1): mu and a_l, l = -L..L.
struct GaussFit {
    long double mu;
    std::vector<cld> a;  // size 2L+1, index l + L
    double max_err;
};
GaussFit fit_gaussian(int L);

// Two-sided REXI list (see rexi.h).  Index k + M + L for k = -(M+L)..(M+L).
struct Poles {
    std::vector<std::complex<double>> alpha, beta_plus, beta_minus;
};
Poles make_poles(int M, double h, int L, int normalize);

// Gauss-Legendre nodes (descending, north to south) and weights.
void gauss_legendre(int nlat, std::vector<double>& mu, std::vector<double>& w);

// Orthonormal P_n^m = s_n Q_n with Q_n = c_n mu Q_{n-1} - Q_{n-2}: c_n and s_n in
// spectral order, [nspec] each, and exact restart rows (Q_{n0-1}, Q_{n0}) at n0 = m +
// run r, [row][2][nmu] with row = run_base[m] + r (run_base has T + 2 entries); tail:
// the same at the parts of an order's last segment (see tables.cpp).
void legendre_coefs(int T, std::vector<double>& coef, std::vector<double>& scale);
std::vector<double> legendre_restarts(int T, int run, int seg, const std::vector<double>& mu,
                                      std::vector<int>& run_base, std::vector<double>& tail);

// Device tables of the Legendre kernels for degrees 0..T (orders m <= the
// plan's truncation): restart rows, recurrence coefficients and work lists.
struct LegTables {
    int T = 0;
    double* d_restart = nullptr;  // [row][2][nhalf], rows every 32 degrees
    double* d_tail = nullptr;     // [m][4][2][nhalf], the four parts of an order's last inverse segment
    double* d_lcoef = nullptr;    // [nspec(T)] and padding
    double* d_lscale = nullptr;   // [nspec(T)]
    void* d_tiles_f = nullptr;    // forward runs
    void* d_tiles_i = nullptr;    // inverse work
    int ntiles_f = 0, ntiles_i = 0;
    int fwd_g = 2;                // runs per workgroup of the forward
    int inv_r = 1;                // latitude tiles per wave of the inverse
};

// Columns per workgroup: C split evenly into `parts` of whole groups of four, at most 32.
inline int column_chunk(int C, int parts) {
    const int groups = (C + 3) / 4;
    parts = std::max(parts, (groups + 7) / 8);
    return 4 * ((groups + parts - 1) / parts);
}

// Columns per workgroup of the inverse of C columns, `tiles` workgroups to a chunk of
// them.  With one latitude tile per wave and at most 850 workgroups of as many columns
// as fit, each takes two column groups instead, if they pair up evenly: whole
// syntheses, all / two groups, T256 on 512 x 256, 12 fields (528 workgroups) 21.6 /
// 19.8 us, 16 fields 25.9 / 23.6; T127, 24 fields (256) 12.8 / 12.0, 96 fields (768)
// 25.7 / 24.9; T279 on 1024 x 280, 8 fields (840) 25.3 / 24.6.  Beyond that the
// recurrences, repeated for every eight columns, cost more than the waiting that the
// further workgroups cover: T300, 12 fields (912) 35.3 / 37.7; T256, 24 fields (1056)
// 31.1 / 32.5, 512 fields 518 / 563; T127, 1024 fields 220 / 249.  Three groups at
// T300 took 16.3 us of kernel against 13.0, and two tiles per wave at T511 36 against
// 32.
inline int inverse_columns(int C, int tiles_per_wave, int tiles) {
    const int groups = (C + 3) / 4, all = column_chunk(C, 1);
    if (tiles_per_wave > 1 || groups % 2 || tiles * ((C + all - 1) / all) > 850) return all;
    return column_chunk(C, groups / 2);
}

__host__ __device__ inline long long spec_offset(int T, int m) {
    return (long long)m * (T + 1) - (long long)m * (m - 1) / 2;
}
__host__ __device__ inline long long nspec_of(int T) { return (long long)(T + 1) * (T + 2) / 2; }

// ---------------------------------------------------------------- device-side structs
// Per zonal order m: the two parity chains of the Phi-eliminated block.
//   chain p holds vorticity at degrees n == p (mod 2) and divergence at the
//   others; Phi_n is carried with the divergence element of degree n.
//   n0 = max(m, 1) (the (0,0) mode is handled on its own), L = T + 1 - n0.
//   P lanes per chain problem (a power of two), s elements per lane.
struct MInfo {
    int n0, L, P, s;
    int spec_off;   // idx(m, m)
    int slot_base;  // first chain slot of this m (chain p at slot_base + p L)
};

// One work item of the fused solve: chain p of order m, the R states
// [tile*R, tile*R + R) (R = the launch's states per item), poles [k0, k1).
// Its partial sums go to part + part_off (complex units), layout [R][2][L].
struct Item {
    int m, p, tile, k0, k1;
    long long part_off;
};

// Per (m, p, state): where the partial sums of that state start in the
// first of its nr consecutive items, and the states per item st of those
// items (successive items are st * 2L complex entries apart).
struct Group {
    long long part_off;
    int nr;
    int st;
};

// One launch of the solve kernel: items [item0, item0 + nitems) share the
// elements-per-lane class SE, the cross-lane move kind and the number of
// states per item (rot), whose solves share each pole's factorisation.
struct Launch {
    int SE;
    int kind;  // cross-lane moves: 0 ds_bpermute, 1 DPP within 16-lane rows, 2 DPP over row pairs
    int item0, nitems;
    int pmax;  // largest lane group of the launch (sizes its LDS)
    int rot;   // states per work item
};

// The pole-per-lane solve (sweep_kernels.hip).  Chains are stored as pairs of a
// vorticity and a divergence element, every chain padded to whole groups of two
// pairs; kSweepBlock pairs form a block of its backward pass.
constexpr int kSweepBlock = 6;
constexpr int kSweepCst = 5;      // doubles of operator constants per pair
constexpr int kSweepRec = 6;      // doubles of data per pair and state
constexpr int kSweepPad = 2 * kSweepBlock * kSweepRec;  // doubles past the end of constants and data that a block may read
constexpr int kSweepStates = 4;   // most states per work item
constexpr int kSweepWaves = 4;    // waves of a workgroup
constexpr int kSweepGroups = 512; // workgroups that the chip holds, two per CU
constexpr int kSweepSplit = 24;   // shortest chain that is split between two waves
constexpr int kSweepShort = 16;   // most pairs of a chain (or half) that a wave holds in registers
constexpr int kSweepKind = 3;     // its kind in a schedule's classes (no moves between lanes)
struct SweepItem {                // a wave's work: pairs of one chain, states [s0, s0 + nst), poles [k0, k1)
    int pair0, npair;
    int pstride;                  // pairs of the whole chain (a split chain: both halves and the middle)
    int s0, nst, k0, k1;
    int mid, half;                // a half of a split chain: its middle pair and which half, else mid = -1
    long long part_off;           // doubles; layout [nst][pstride][kSweepRec], from this item's first pair
    long long mid_off;            // the same from the middle pair
};
struct SweepChain { int pair0, npair; };
struct SweepTile { int tile, pos, nst; };               // of a state: its tile, place there, states of the tile
struct SweepGroup { long long part_off; int nr, npair; };  // of a (pair, tile): its first partial (double2), of nr items, pairs of the chain
struct SweepTables {
    bool built = false, usable = false;
    int npairs = 0;
    std::vector<SweepChain> chains;  // index 2 m + p
    // split tables: chains of at least kSweepSplit elements are laid out as the
    // part before their middle vorticity element, that element, and the part after
    // it in reverse; pairs of the two parts (0, 0: not split)
    std::vector<int2> halves;
    double* d_cst = nullptr;         // [pair][kSweepCst]
    int2* d_idx = nullptr;           // [pair] spectral index of its vorticity and divergence (-1: a dummy)
    double *d_fin[2] = {nullptr, nullptr}, *d_fout[2] = {nullptr, nullptr};  // [pair][3]
    double2* d_poles[2] = {nullptr, nullptr};                                // [N][6]
};

constexpr int kMaxLaunches = 8;  // solve launches per step (tile classes)

// Device workspace of a step: the states in chain layout (double buffered
// between steps), the solve's partial sums and the work counters of
// persistent launches.  A plan owns one; the no-allocation step carves one
// out of a fixed device array.
struct Workspace {
    double2* ch_var[2];  // [S][nslots + 2]
    double2* ch_phi[2];  // [S][nspec]
    double2* part;       // partial sums, the schedule's part_size entries
    int* counters;       // kMaxLaunches
    double* rec[2];          // pole-per-lane solve: [S][pairs + 1][kSweepRec] and kSweepPad
    double2* sweep_scratch;  // its block-boundary values, one slot per workgroup
    int sweep_groups;        // slots there
};

struct Schedule {
    bool persistent = false;  // resident grid + atomic work counter per launch
    int SM = 4;       // largest elements-per-lane class used
    int rot_max = 1;  // largest states-per-item the schedule may use
    int S = 0;        // states this schedule serves
    std::vector<Launch> launches;
    std::vector<MInfo> minfo;
    std::vector<Item> items;
    std::vector<Group> groups;  // index ((m * 2 + p) * S + state)
    long long part_size = 0;    // complex entries
    // device copies
    MInfo* d_minfo = nullptr;
    Item* d_items = nullptr;
    Group* d_groups = nullptr;
    // pole-per-lane schedules (then the members above hold one launch for the
    // queries and nothing else)
    bool sweep = false;
    bool split = false;                   // long chains split between two waves
    bool short_chains = false;            // every part of a chain in registers
    int sweep_nst = 0, sweep_ntiles = 0;  // most states of an item, state tiles
    long long sweep_stride = 0;           // scratch of one wave (double2)
    std::vector<SweepItem> sweep_items;
    std::vector<SweepTile> sweep_tiles;
    std::vector<SweepGroup> sweep_groups;
    SweepItem* d_sweep_items = nullptr;
    SweepTile* d_sweep_tiles = nullptr;
    SweepGroup* d_sweep_groups = nullptr;
    bool on_device = false;  // the device copies are there
    std::string name;
};

}  // namespace rexi

// ---------------------------------------------------------------- the plan
struct rexi_plan {
    rexi_params prm;
    int T = 0, N = 0;
    long long nspec = 0, nslots = 0;
    double phibar = 0;
    rexi::Poles poles;
    std::complex<double> g00_fwd, g00_adj, gphi_fwd, gphi_adj;

    // per-(n, m) constants in spectral order (device)
    double *d_th = nullptr, *d_om = nullptr, *d_cc = nullptr, *d_sc = nullptr;
    int *d_idx_n = nullptr, *d_idx_m = nullptr;
    // per pole, forward [0] and adjoint [1]: alpha, 1/alpha, wx, wy, wx/alpha,
    // wy/alpha (6 complex, see rexi_kernels.hip)
    double2* d_poles[2] = {nullptr, nullptr};
    // states of the tiled solve, for max_states, where it runs
    double2 *d_ch_var[2] = {nullptr, nullptr};  // [S][nslots + 2]
    double2 *d_ch_phi[2] = {nullptr, nullptr};  // [S][nspec]
    double2 *d_part = nullptr;
    long long part_capacity = 0;
    double2 *d_acc = nullptr;                    // per-term form accumulator [S][2][nslots]
    // chain-slot layout (device) and slot -> m table
    rexi::MInfo* sched_layout = nullptr;
    int* d_slot_m = nullptr;
    // schedules: candidates per S, chosen index per S; per-term form per S
    std::vector<std::vector<rexi::Schedule>> sched;  // [S] -> candidates
    std::vector<int> chosen;
    std::vector<int> own;    // what the plan chose itself, the default or autotune's, [S]
    std::vector<int> tiled;  // the default among the tiled schedules, [S]
    // until the candidates of S are asked for: the default alone, and the tiled one
    // that takes its no-allocation steps (see schedules_for)
    std::vector<rexi::Schedule> first, first_tiled;
    bool captured = false;       // a caller has captured a step
    std::vector<void*> retired;  // smaller workspace that its graph may hold
    std::vector<rexi::Schedule> per_term;             // [S]
    long long acc_capacity = 0;

    // transforms
    int nlat = 0, nlon = 0, nhalf = 0;
    std::vector<double> mu, w;
    rexi::LegTables leg;          // degrees 0..T (scalar transforms)
    rexi::LegTables legv;         // degrees 0..T+1 (vector transforms)
    double* d_mu = nullptr;       // northern Gauss nodes [nhalf]
    double* d_wts = nullptr;      // Gauss weights
    double* d_rcos = nullptr;     // 1 / cos(lat_j) [nlat]
    double* d_four = nullptr;     // Fourier workspace [T+1][nlat][2B] + padding per plane
    double2* d_twiddle = nullptr; // FFT twiddles
    double2* d_vspec = nullptr;   // vector transforms: [max_fields][nspec(T+1)]

    // f-sphere variant: constant Coriolis parameter times dt, poles
    // [N][3] (alpha, beta+, beta-)
    double f0dt = 0.0;
    double2* d_fs_poles = nullptr;

    // persistent launches: one work counter per solve launch
    int* d_counters = nullptr;
    // pole-per-lane solve: tables, records of two buffers, scratch
    rexi::SweepTables sweep[2];  // whole chains, split chains
    double* d_rec[2] = {nullptr, nullptr};
    double2* d_sweep_scratch = nullptr;
    long long rec_capacity[2] = {0, 0}, sweep_scratch_capacity = 0;
    long long scratch_refused = 1LL << 62;  // scratch that could not be had (double2)
    // captured step graphs: key (S, adjoint, input buffer), valid for `graph_gen`
    struct StepGraph {
        const rexi::Schedule* sched;
        int S, adjoint, buf;
        long long gen;
        hipGraphExec_t exec;
        hipEvent_t done;  // recorded after each launch of exec
    };
    std::vector<StepGraph> graphs;
    long long graph_gen = 0;
    bool use_graphs = true;
    hipStream_t cap_stream = nullptr;
    // concurrent tile-class launches: side streams, fork and join events
    bool concurrent = true;
    hipStream_t side[rexi::kMaxLaunches] = {};
    hipEvent_t fork_ev = nullptr;
    hipEvent_t join_ev[rexi::kMaxLaunches] = {};

    // the device the plan was created on, and the no-allocation step's fixed
    // workspace there (see rexi_step_noalloc)
    int device = 0;
    void* scratch = nullptr;
    size_t scratch_bytes = 0;

    // measurement: event pairs around timed launches, per kernel kind
    bool timing = false;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> events[3];
};

namespace rexi {
// Launchers (rexi_kernels.hip, sh_kernels.hip) and library internals used
// across the sources.
bool solve_variant_supported(int SE, int kind, int rot, bool per_term);
int solve_waves_per_item();
int solve_variant_list(bool per_term, int* se, int* kind, int* st, int cap);
hipError_t enqueue_prep(rexi_plan* pl, const Workspace& ws, const void* u, int buf, int S, int adjoint,
                        const MInfo* d_layout, hipStream_t s);
hipError_t enqueue_solve(rexi_plan* pl, const Workspace& ws, const Schedule& sc, int buf, int S, int adjoint,
                         hipStream_t s);
hipError_t enqueue_reduce(rexi_plan* pl, const Workspace& ws, const Schedule& sc, const double2* part, int buf_in,
                          int buf_out, void* u_out, int S, int adjoint, const int* d_slot_m, hipStream_t s);
hipError_t enqueue_zero(double2* p, long long n, hipStream_t s);
hipError_t enqueue_fsphere_steps(rexi_plan* pl, const void* in, void* out, int S, int nsteps, int adjoint,
                                 hipStream_t s);
hipError_t enqueue_finish(rexi_plan* pl, const Workspace& ws, int buf, void* u, int S, int adjoint,
                          const MInfo* d_layout, hipStream_t s);
hipError_t enqueue_per_term_pole(rexi_plan* pl, const Workspace& ws, const Schedule& sc, int k, int buf, int S,
                                 hipStream_t s);
hipError_t enqueue_reset_counters(int* c, int n, hipStream_t s);
hipError_t enqueue_sweep_prep(rexi_plan* pl, const Workspace& ws, const Schedule& sc, const void* u, int buf, int S,
                              int adjoint, hipStream_t s);
hipError_t enqueue_sweep_solve(rexi_plan* pl, const Workspace& ws, const Schedule& sc, int buf, int S, int adjoint,
                               hipStream_t s);
hipError_t enqueue_sweep_reduce(rexi_plan* pl, const Workspace& ws, const Schedule& sc, int buf_in, int buf_out,
                                void* u_out, int S, int adjoint, hipStream_t s);
// nsteps steps of a pole-per-lane schedule, launched one by one (plan.cpp); timed:
// between events where the plan's timing is on.
int run_sweep_steps(rexi_plan* pl, const Workspace& ws, const Schedule& sc, const void* u0, void* u1, int S,
                    int nsteps, int adjoint, bool timed, hipStream_t s);
int sh_setup(rexi_plan* pl);
void sh_release(rexi_plan* pl);
int sh_run(rexi_plan* pl, const void* in, void* out, int B, bool forward, hipStream_t s);
int sh_vec_run(rexi_plan* pl, const void* in, void* out, long long stride, int B, bool to_uv, hipStream_t s);
// Whether the no-allocation step's array holds the workspace of a pole-per-lane
// schedule (noalloc.hip; true for the others, which it carves or refuses).
bool noalloc_takes(const rexi_plan* pl, const Schedule& sc);
int check_state_call(rexi_plan* pl, const void* in, const void* out, int S, int nsteps);
// The no-allocation step's fixed device array: its address on the current
// device, looked up once per device (noalloc.hip).
int scratch_setup(void** ptr, size_t* bytes);

// Whole-chain schedules whose workgroups' block-boundary values, one slot each,
// exceed the 256 MB memory-side cache run as a resident grid that takes the items
// from a counter, so that kSweepGroups slots (0.4 GB) are written and read again and
// again.  T301, three states (1.5 GB otherwise) 993 -> 969 us a step; T256, four
// states (1.8 GB) 1542 -> 1534; within 0.5% at T128, eight states (0.42 GB) and T127,
// one state (0.29 GB).  Split and register-resident schedules are smaller.
inline bool sweep_resident(const Schedule& sc) {
    const long long wgs = ((long long)sc.sweep_items.size() + kSweepWaves - 1) / kSweepWaves;
    return !sc.split && wgs > kSweepGroups && wgs * kSweepWaves * sc.sweep_stride * 16 > (256LL << 20);
}

// The plan's own workspace.
inline Workspace plan_workspace(const rexi_plan* pl, const Schedule& sc) {
    const int groups = sc.sweep_stride > 0 ? (int)std::min<long long>(pl->sweep_scratch_capacity / (kSweepWaves * sc.sweep_stride), 1 << 20)
                                           : 1 << 20;
    return Workspace{{pl->d_ch_var[0], pl->d_ch_var[1]}, {pl->d_ch_phi[0], pl->d_ch_phi[1]}, pl->d_part,
                     pl->d_counters, {pl->d_rec[0], pl->d_rec[1]}, pl->d_sweep_scratch, groups};
}
// Record an event before / after a timed launch when timing is on.
hipError_t timed_begin(rexi_plan* pl, int kind, hipStream_t s);
hipError_t timed_end(rexi_plan* pl, int kind, hipStream_t s);
}  // namespace rexi
