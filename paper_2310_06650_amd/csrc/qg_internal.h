// Internal types shared by the host builder, the kernels and the C ABI.
#pragma once

#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

#include "qg.h"

namespace qg {

constexpr int kAlign = 256;
constexpr int kMaxT = 64;          // periods per problem (4 MFMA row tiles of 16)
constexpr int kBlock = 256;        // threads per block of the streaming kernels
constexpr int kCtgLanes = 64;      // contingencies per wavefront in the map-reduce
constexpr int kParams = 16;        // doubles in the per-step parameter block
constexpr int kCtgMaxTc = 8;            // periods per block of the contingency kernel
constexpr int kCtgSlices = 16;          // most branch slices (wavefronts) of a k_ctg_rows block
constexpr int kCtgLdsBytes = 64 * 1024; // LDS budget of one contingency block
constexpr int kAdjStepsPerBlock = 32;   // MFMA k-steps per block of the adjoint product
constexpr int kUpdateBlock = 1024;      // threads per block of k_update
constexpr int kUpdateMaxL = 768;        // most branches of a grid that takes it
constexpr int kSchedCap = 2048;         // solve steps per uploaded schedule table
constexpr int kSchedStride = 16;        // doubles per step in the schedule table
constexpr int kStepGraphs = 6;          // cached step graphs of 1, 2, 4, ..., 32 steps

inline int64_t round_up(int64_t a, int64_t b) { return (a + b - 1) / b * b; }

// Parameter block layout (DevWork::params): the homotopy and step sizes of
// the step being evaluated.
enum ParamSlot { PB_EPS = 0, PB_BETA = 1, PB_RHO = 2, PB_ALPHA = 4, PB_BC1 = 10, PB_BC2 = 11 };

// Storage kind of the outage factors, from the build flags.
enum LodfKind { kLodfF64 = 0, kLodfF32 = 1, kLodfBF16 = 2 };
inline int lodf_kind_of(uint32_t flags) {
  return (flags & QG_FLAG_CTG_BF16) ? kLodfBF16 : (flags & QG_FLAG_CTG_FP32) ? kLodfF32 : kLodfF64;
}
inline size_t lodf_elem_bytes(int kind) { return kind == kLodfF64 ? 8 : kind == kLodfF32 ? 4 : 2; }

// Pointer to device memory in a kernel's arguments.  Kernels of a batch read
// their arguments from memory, where the compiler cannot see that the pointers
// are to global memory: it would use flat accesses, which also count and wait
// as LDS accesses.
#ifdef __HIPCC__
#define QG_BOTH __host__ __device__
#else
#define QG_BOTH
#endif
template <class T>
struct DevPtr {
  T* p;
  DevPtr() = default;
  QG_BOTH DevPtr(T* q) : p(q) {}
  QG_BOTH operator T*() const {
#if defined(__HIP_DEVICE_COMPILE__) && __HIP_DEVICE_COMPILE__
    return (T*)(__attribute__((address_space(1))) T*)reinterpret_cast<uintptr_t>(p);
#else
    return p;
#endif
  }
};

// Device view of the constant arena (all pointers into caller memory).
struct DevProblem {
  int N, L, G, T, M, K;
  int Lp;    // L padded to 64 (row count of the outage-factor tile space)
  int Kp;    // K padded to 64 (one wavefront of contingencies)
  int G16;   // G padded to 16 (MFMA output columns of the adjoint product)
  int G4;    // G padded to 4  (MFMA reduction depth of the flow product)
  int Tp;    // T padded to 16 (MFMA rows)
  int twoL;  // endpoint slots per period
  // branches
  DevPtr<const int> br_from, br_to, slot_fr, slot_to;
  DevPtr<const double> br_g, br_b, br_bh, br_smax;
  DevPtr<const double> ctg_smax;  // [Lp] contingency rating (1 on padding)
  DevPtr<const double> ctg_smax2;  // [Lp] its square
  DevPtr<const int> kof;  // [Lp] contingency index of a branch, -1 if none
  DevPtr<const int> brk;  // [Kp] outaged branch of a contingency (0 on padding)
  // buses
  DevPtr<const int> bptr;  // [N+1] endpoint-slot ranges (bus-sorted)
  DevPtr<const int> gptr;  // [N+1] generator ranges
  DevPtr<const int> glist;  // [G]   generators sorted by bus
  DevPtr<const double> vmin, vmax;
  // generators
  DevPtr<const int> gen_bus;
  DevPtr<const double> pmin, pmax, qmin, qmax, rmax, ru, rd, rusu, rdsd, p0, u0;
  DevPtr<const double> con, csu, csd, cr;
  DevPtr<const double> seg_cost, seg_size, pcum;  // [G*M]
  // periods
  DevPtr<const double> load_p, load_q;  // [T*N]
  DevPtr<const double> dt, rsv_req, sum_load;  // [T]
  // sensitivities, restricted to generator buses
  // [G4][Lp] ISF[l][bus(j)] - rsum[l]/N, zero padded (B of the flow product)
  DevPtr<const double> isf_gT;
  DevPtr<const double> isf_ga;  // [Lp][G16] ISF[l][bus(j)] - rsum[l]/N (B of the adjoint product)
  DevPtr<const double> cload;  // [T][Lp]   sum_i ISF[l][i] load_p[t][i] - rsum[l] sum_load[t] / N
  DevPtr<const double> rsum;  // [Lp]      sum_i ISF[l][i]
  DevPtr<const double> lodf;  // [Lp][Kp]  outage factors; NaN marks (k,k) and padding
  DevPtr<const float> lodf32;  //           the same in FP32 (QG_FLAG_CTG_FP32)
  DevPtr<const uint16_t> lodf16;  //         the same in BF16 (QG_FLAG_CTG_BF16)
  int lodf_kind;         // 0 FP64, 1 FP32, 2 BF16 (one of the three pointers is set)
  DevPtr<const double> lmax;  // [Kp/64][Lp] max |lodf| (as stored) of each branch over
                         // 64 contingencies, NaN left out (null with QG_FLAG_CTG_NO_SKIP)
  int ctg_sum;           // 1: per-period sum over contingencies instead of max + mean
  // prices
  double c_p, c_q, c_s, c_ang, ang_max, c_rsv, rho, vload;
};

// Two doubles moved together.
struct alignas(16) Pair {
  double x, y;
};

// Device view of the caller's workspace.
struct DevWork {
  DevPtr<double> params;  // [kParams] parameters of the step being evaluated
  DevPtr<int64_t> step;  // [1] index of the current step in the schedule table
  DevPtr<double> sched;  // [kSchedCap][kSchedStride] per-step eps, beta, rho_s, alpha[6], bc1, bc2
  DevPtr<double> snext;  // [kSchedStride] the schedule row of the next scheduled evaluation
  DevPtr<Pair> ep;  // [T][2L] branch flows (p, q) at bus-sorted endpoint slots
  // [3][T][L] per-branch reverse coefficients: cosine and sine, thermal derivative
  // by p and q, angle derivative and 2 q, the latter two pairs of the sides in bside
  DevPtr<Pair> bco;
  DevPtr<uint8_t> bside;  // [T][L] kThermalTo, kReactiveTo
  DevPtr<double> q2;  // [T][Lp]  max(q_fr^2, q_to^2)
  DevPtr<double> F;  // [T][Lp]  base-case DC flows
  DevPtr<double> Fk;  // [T][Kp]  flows of the outaged branches
  DevPtr<double> lamp, lamq;  // [T][N] balance multipliers
  DevPtr<double> gdev;  // [4][T][G] device-only partials of p, q, r, u
  DevPtr<double> zpart, spart;  // [nLb][T][Kp]
  DevPtr<double> rpart, qpart;  // [nKb][T][Lp] (branch-stacked tile)
  DevPtr<double> rq;  // [T][Lp][nKb_max][2] R and Q per contingency block (period-split
                       // tile; the memory of rpart and qpart), stored where flagged:
  DevPtr<uint64_t> hot;  // [T][Lp/64][nKb_max] flags of 64 branches per contingency block
  DevPtr<double> smean;  // [T][Kp]
  DevPtr<double> zval;  // [T][Kp]
  DevPtr<double> gfT;  // [Lp][Tp] dL/dF, transposed
  DevPtr<double> qtot;  // [T][Lp]  dL/d qmax2
  DevPtr<double> gpdc;  // [nsplit][T][G16] DC part of dL/dp (split-K partials)
  DevPtr<Pair> epG;  // [T][2L] endpoint adjoints (V, theta)
  DevPtr<double> tpart;  // term partial sums
  DevPtr<double> terms;  // [QG_NTERMS] last evaluated terms
  DevPtr<double> drs;  // [T]       reserve-shortfall derivative, subtracted from dL/dr
  DevPtr<double> zmaxp;  // [T][nKc]  per-chunk worst penalty
  DevPtr<double> zargp;  // [T][nKc]  its contingency index
  DevPtr<double> zsump;  // [T][nKc]  per-chunk penalty sum
  DevPtr<double> kstar;  // [T]       worst contingency of the period
  DevPtr<double> smaxp;  // [T][nLc]  per-chunk dL/dF of the worst contingency's own branch
  DevPtr<double> lamg, lamqg;  // [T][G] balance multipliers at each generator's bus
  DevPtr<double> isfk;  // [T][G16]  ISF[br(k*_t)][bus(j)] - rowsum/N of the period's worst outage
  DevPtr<double> thr;  // [T][Lp]  test radius of the outage flows
};

// Sides of a branch in DevWork::bside: set where the larger apparent power, the
// larger reactive flow is the to side's.
constexpr uint8_t kThermalTo = 1, kReactiveTo = 2;

// Offsets of the term partial sums inside DevWork::tpart.
struct TermOffsets {
  int br, ang, dev, pen, rsv, bal, cmax, cmean, total;
};

// Tile shape of the contingency map-reduce.
struct CtgTile {
  int bl;   // branches per wavefront (8, 16 or 32)
  int wl;   // wavefronts per block, stacked along branches
  int tc;   // periods per block (the period range is split over grid.z)
  int lt;   // consecutive tiles of wl * bl branches per block (split: of 8
            // branches per wavefront, see ctg_slices)
  int split = 0;  // 1: period-split blocks, one period each (k_ctg_rows)
  int lt_auto = 0;  // 1: lt is the default, not the caller's
};

// Homotopy source of one evaluation.
struct EvalMode {
  int schedule;          // 0: homotopy from args, 1: from the solve schedule
  double eps, beta, rho_s;
  // schedule (mode 1)
  int64_t n_total;
  double alpha0[QG_NCLASS], alphaf[QG_NCLASS];
  double eps0, epsf, beta0, betaf, rho0, rhof;
  double adam_b1, adam_b2, adam_eps;
  int eps_in_num;
  int screened;          // 1: score only the problem's chosen contingency set
};

struct Problem;

// Contingency screening (Alg. 2): the set of contingencies scored by the
// screened steps, and its outage factors gathered into contiguous columns.
// All device arrays live in the caller's screening buffer.
struct Screen {
  bool on = false;
  bool chosen = false;       // a set has been selected or given
  int n_top = 0;             // worst-set slots
  int n_act = 0;             // contingencies scored (slots in use)
  int cap = 0;               // most slots the buffer holds
  int Ka = 0;                // n_act padded to 64: row stride of lodf_act
  double zeta = 0.0;         // severity threshold of the worst set
  int refresh = 0;           // steps between exact refresh steps in qg_solve
  uint64_t seed = 0;         // seed of the random draw
  int* act_k = nullptr;      // [Kp] slot -> contingency (0 past n_act)
  int* act_slot = nullptr;   // [Kp] contingency -> slot, -1 if not scored
  int* top = nullptr;        // [Kp] worst-set flags of the last selection
  int* sel = nullptr;        // [Kp] chosen flags of the last selection
  double* sev = nullptr;     // [Kp] severities of the last refresh
  uint64_t* key = nullptr;   // [Kp] draw keys of the last refresh
  void* lodf_act = nullptr;  // [Lp][Ka] outage factors of the slots, NaN past n_act
  double* lmax_act = nullptr;  // [Ka/64][Lp] largest |factor| of a branch over 64 slots
  size_t bytes = 0;          // bytes of the buffer in use
};
// Bytes of a screening buffer for up to cap scored contingencies, and the
// carve of one (sets the pointers of sc).
size_t screen_bytes(const Problem& p, int cap);
void carve_screen(const Problem& p, void* buf, int cap, Screen* sc);

struct Problem {
  int device = -1;  // HIP device current at build (the arena's device)
  // sizes
  int N, L, G, T, M, K;
  int Lp, Kp, G16, G4, Tp;
  int64_t n_x;
  uint32_t flags;
  std::vector<int32_t> ctg;
  // launch geometry
  int nb_br;      // blocks of the per-(t, branch) kernels
  int nb_bus;     // blocks of the per-(t, bus chunk) kernels
  int bus_chunks; // bus chunks per period
  int nb_gen;     // blocks of one variable of every (t, generator) in the final stage
  int nsplit;     // reduction splits of the adjoint product
  int nKc, nLc;   // chunks of Kp (64 wide) and Lp (256 wide)
  CtgTile tile;
  int nLb, nKb;   // partial counts of the contingency map-reduce
  int nLb_max, nKb_max;
  TermOffsets toff;
  size_t const_bytes, work_bytes;
  DevProblem dp;
  void* arena = nullptr;
  // graph cache of qg_solve: graph_exec holds one screening refresh cycle;
  // step_graph[i] holds 2^i plain steps (i < kStepGraphs), so that a solve of
  // any length replays cached graphs (n = sum of powers of two)
  void* graph_exec = nullptr;
  void* step_graph[kStepGraphs] = {};
  const void* graph_key[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};
  int graph_steps = 0;
  EvalMode graph_mode{};
  CtgTile graph_tile{};   // contingency tile the cached graph was captured with
  // host data kept for load updates (same grid, new loads)
  std::vector<double> isf_host;  // [L][isf_np] injection shift factors (reference column 0)
  int isf_np = 0;
  std::vector<double> rsum_host; // [Lp] ISF row sums
  std::vector<double> dt_host;   // [T]
  double load_value = 0.0;
  Screen scr;
  // pinned host staging of the schedule table (two halves, each reused only
  // after the event recorded behind its last upload), and the events that
  // time a solve's steps; created at the first qg_solve
  double* sched_host = nullptr;
  void* sched_ev[2] = {nullptr, nullptr};
  // what the device schedule table holds: rows of iterations
  // [sched_base, sched_base + sched_rows) for the schedule sched_key (bytes
  // of the solve options and Adam constants the rows depend on, and the
  // workspace they live in); sched_base < 1 when unknown
  unsigned char sched_key[192] = {};
  int64_t sched_base = -1;
  int sched_rows = 0;
  // iteration the device step counter and the copied-ahead row point at
  // after the last scheduled step (-1: unknown); a call continuing there
  // needs no counter reset
  int64_t sched_next = -1;
  void* step_ev[2] = {nullptr, nullptr};
};

// Host build products (before upload).
struct HostBuild {
  std::vector<unsigned char> image;  // arena image
  size_t const_bytes = 0;
};

// Set the thread-local error text; returns s.
qg_status fail(qg_status s, const std::string& msg);

// Validate the description and find the contingency set.  Fills p's sizes.
qg_status plan_problem(const qg_grid_desc* d, const qg_build_opts* o, Problem* p);
// Factor, sensitivities and the arena image.
qg_status build_arena(const qg_grid_desc* d, const qg_build_opts* o, Problem* p,
                      HostBuild* hb);
void rebase_pointers(Problem* p, void* arena);
// Load-dependent parts of the arena for new loads: byte offsets and host
// values of load_p, load_q, rsv_req, sum_load and the flow constant, and the
// consumer value.  Uses the ISF kept at build.
struct LoadBlock {
  size_t off_lp, off_lq, off_rsv, off_sum, off_cload;
  std::vector<double> sum_load, cload;
  double vload;
};
void load_block(const Problem* p, const double* load_p, LoadBlock* out);
DevWork carve_workspace(const Problem* p, void* ws);
int default_ctg_tc(const Problem& p, int wl);
int default_ctg_lt(const Problem& p, const CtgTile& t);  // tiles per block for tile t
void apply_ctg_tile(Problem* p, const CtgTile& t);        // set the tile and the l-block count
CtgTile default_ctg_tile(const Problem& p);               // the tile a new problem starts with
// branch slices of a period-split block over nkb contingency blocks (0: branch-stacked)
int ctg_slices(const Problem& p, int nkb);
int ctg_tc_cap(int wl);  // most periods per block the LDS budget allows

// Kernel launchers (qg_kernels.hip).  A step is kStages kernels.
constexpr int kStages = 6;
int launch_eval(const Problem* p, const DevWork& w, const double* x, double* grad,
                double* terms_out, const EvalMode& mode, int fuse_adam, double* m,
                double* v, void* stream, void** events /* nullable [QG_NKERNELS] */);
// Mean duration of one kernel of the step (0..kStages-1), launched reps times
// back to back after a full evaluation at x has produced its inputs.
int time_stage(const Problem* p, const DevWork& w, const double* x, const EvalMode& mode,
               int stage, int reps, void* stream, double* mean_ms);
int launch_adam(const Problem* p, double* x, double* m, double* v, const double* g,
                const double lr[QG_NCLASS], double bc1, double bc2, double b1,
                double b2, double eps, int eps_in_num, void* stream);
int launch_set_step(const Problem* p, const DevWork& w, int64_t value, void* stream);

// Batched step of independent problems: kStages launches for all of them.
// The caller's batch buffer holds every problem's kernel arguments and, per
// stage, a table of the launch's blocks (problem index << 22 | block of that
// problem).
struct BatchPlan {
  int n = 0;
  int nblk[kStages] = {};      // blocks of each batched launch
  size_t off_args = 0;         // byte offsets into the batch buffer
  size_t off_tab[kStages] = {};
  size_t bytes = 0;            // size of the batch buffer
  int lodf_kind = 0;
  int nsl = 0;                 // most branch slices of a problem (map-reduce LDS)
  bool test_wide = false;      // form of k_ctg_test
  int row_waves = 0;           // wavefronts per block of the map-reduce
};
constexpr int kBatchLocBits = 22;                  // block index bits of a table entry
constexpr int kBatchWl = 4;        // the tile a batch asks of its problems: wavefronts
constexpr int kBatchTcw = 4;       // and periods per wavefront
// Sizes, validation and (image != nullptr) the host image of a batch buffer
// for problems whose steps take x[i], m[i], v[i] and workspaces ws[i]; 0 or
// a message in *err.
int plan_batch(const Problem* const* prs, const DevWork* ws, int n, const double* const* x,
               double* const* m, double* const* v, const EvalMode& mode, BatchPlan* plan,
               std::vector<unsigned char>* image, std::string* err);
int launch_eval_batch(const BatchPlan& plan, void* d_buf, void* stream);
int launch_check_finite(const Problem* p, const double* x, int* flag, void* stream);
// Screening (qg_screen.hip): choose the set from the severities of the last
// exact evaluation (its z_tk and homotopy in the workspace), then gather its
// outage factors; or gather only, for a set uploaded by the host.  round < 0:
// the refresh index follows from the schedule row of the step just taken.
int launch_screen_select(const Problem* p, const DevWork& w, int64_t round, void* stream);
int launch_screen_gather(const Problem* p, void* stream);

}  // namespace qg
