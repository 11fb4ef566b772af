// Internal declarations shared by the host API and the HIP kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <array>
#include <functional>
#include <string>
#include <vector>

#include "fr_sg.h"

namespace frsg {

constexpr int kMaxNp1 = 8;      // p <= 7
constexpr int kMaxModes = 128;  // gPC modes
constexpr int kMaxNodes = 256;  // random quadrature nodes
constexpr int kProjBlock = 3;   // modes per projection task of the whole-step 1D kernel

// device status bits (latched, cleared by fr_sg_sync)
constexpr unsigned kStatusNonFinite = 1u;
constexpr unsigned kStatusNotRealizable = 2u;

// ---------------------------------------------------------------------------
// host tables (FP64), built once per context
// ---------------------------------------------------------------------------
struct HostTables {
  int np1 = 0;                     // p + 1 solution points per direction
  std::vector<double> r, w;        // Legendre-Gauss points / weights (sum 2)
  std::vector<double> D;           // D[i*np1 + j] = l_j'(r_i)
  std::vector<double> lL, lR;      // l_j(-1), l_j(+1)
  std::vector<double> dhL, dhR;    // Radau correction derivatives at r_j
  std::vector<double> V, Vinv;     // V[j*np1 + k] = sqrt(2k+1) P_k(r_j)
  int M = 0, Nq = 0, rdim = 1;
  std::vector<std::array<int, 2>> kidx;  // gPC multi-indices
  std::vector<int> kdeg;                 // |k|
  std::vector<double> z;                 // [Nq * rdim]
  std::vector<double> wq;                // [Nq], sum 1
  std::vector<double> Phi, PW;           // [M * Nq]
  std::vector<double> filt;              // [M * nsp]: exp filter exponent sum or L2 factor
  std::vector<double> shell;             // [M * nsp]: 1 on the outer modal shell
  std::vector<double> swts;              // [nsp]: element-mean weights
  std::vector<double> Dt;                // D - h_L' l(-1)^T - h_R' l(+1)^T (np1 x np1)
  std::vector<double> cmax;              // [M]: max_q |Phi_k(z_q)|
  std::vector<double> PhiT, PWT;         // [Nq * M] node-major copies of Phi, PW
  std::vector<double> op1;               // 1D point operators in one block (DevTab)
  std::vector<double> PWB;               // PW by blocks of kProjBlock modes (DevTab)
  std::vector<double> qfrag;             // matrix-core operand tables (quadrilateral 2D path)
};

// offsets (in doubles) of the matrix-core operand tables of the quadrilateral
// 2D stage kernel (tables_quad.cpp), for nb = ceil(N_q / 16) node blocks:
//   aexp_f [nb][4][64]  chaos basis, FP64 instruction, mode 4 t + lane/16
//   aexp_b [nb][4][64]  chaos basis, FP64 instruction, mode 4 lane/16 + t
//   aprj   [nb][4][64]  weighted basis for the FP64 projection
//   bexp   [nb][2][64]  chaos basis as bfloat16 high / low parts (4 per lane)
//   bprj   [nb][2][64]  weighted basis as bfloat16 high / low parts
//   wslot  [nb][16]     quadrature weight of the node in register r, lane group g
struct QuadFragLayout {
  int nb = 0;
  int aexp_f = 0, aexp_b = 0, aprj = 0, bexp = 0, bprj = 0, wslot = 0, total = 0;
};
__host__ __device__ inline QuadFragLayout quad_frag_layout(int Nq) {
  QuadFragLayout L;
  L.nb = (Nq + 15) / 16;
  L.aexp_f = 0;
  L.aexp_b = L.aexp_f + L.nb * 4 * 64;
  L.aprj = L.aexp_b + L.nb * 4 * 64;
  L.bexp = L.aprj + L.nb * 4 * 64;
  L.bprj = L.bexp + L.nb * 2 * 64;
  L.wslot = L.bprj + L.nb * 2 * 64;
  L.total = L.wslot + L.nb * 16;
  return L;
}
void build_quad_fragments(HostTables& T);

bool build_host_tables(const fr_sg_problem& P, HostTables& T, std::string& err);
// exponent of the exponential filter along one dimension (Sec. 4.1.1): 0 below the
// cutoff eta* (modes untouched), ((eta - eta*) / (1 - eta*))^s from it on
double exp_filter_term(double eta, double eta_star, double s);
// n-point Gauss-Legendre rule (weights sum 2); Gauss-Jordan inverse of an n x n matrix
void gauss_rule(int n, std::vector<double>& x, std::vector<double>& w);
bool invert_matrix(int n, const std::vector<double>& A, std::vector<double>& Ainv);

// ---------------------------------------------------------------------------
// triangles (element = FRSG_ELEM_TRI): reference operators and per-element geometry
// ---------------------------------------------------------------------------
constexpr int kTriMaxDeg = 4;                                   // p <= 4
constexpr int kTriMaxNp = (kTriMaxDeg + 1) * (kTriMaxDeg + 2) / 2;  // 15 solution points
constexpr int kTriGeo = 16;                                     // doubles of geometry per triangle
// geometry record of a triangle: dr/dx, dr/dy, ds/dx, ds/dy, det (= area / 2),
// unit outward normals (nx, ny) of faces 0..2, the factors (face length /
// reference face length / det) of faces 0..2, inscribed-circle diameter
enum : int { kGeoRx = 0, kGeoRy, kGeoSx, kGeoSy, kGeoDet, kGeoN0 = 5, kGeoSc0 = 11, kGeoDin = 14 };
// fused triangle stage: elements per block, and the split of an element operator's rows over
// the block's waves (4 elements x 4 nodes x 4 variables are the 64 columns of a wave)
constexpr int kTriEPB = 4;
constexpr int tri_row_groups(int p) { return (kTriEPB * 4 * 3 * (p + 1) + 63) / 64; }
constexpr int tri_trace_rows(int p) { return (3 * (p + 1) + tri_row_groups(p) - 1) / tri_row_groups(p); }
constexpr int tri_point_rows(int p) { return ((p + 1) * (p + 2) / 2 + tri_row_groups(p) - 1) / tri_row_groups(p); }

struct TriTables {
  int p = 0, np = 0, nfp = 0;
  std::vector<double> r, s;        // solution points on the reference triangle
  std::vector<double> Dr, Ds;      // [np][np]: d l_i/dr, d l_i/ds at point j (row j)
  std::vector<double> Lf;          // [3 nfp][np]: l_i at the flux points, face-major
  std::vector<double> lift;        // [np][3 nfp]: divergence of the correction fields
  std::vector<double> rows;        // the element operators by row groups (KParams::tri_rows)
  std::vector<double> mean_w;      // [np]: element mean = sum_j mean_w[j] u_j
  std::vector<double> geo;         // [E][kTriGeo]
  std::vector<int> nbr;            // [E][6]: neighbour element (or -1 - side), then neighbour face
  std::vector<double> xy_pts;      // [E][np][2]: physical solution-point coordinates
  std::vector<double> V, Vinv;     // [np][np]: V[j][m] = psi_m(r_j) and its inverse
};
// reference tables for degree p, mesh checks and geometry from the problem's arrays
bool build_tri_tables(const fr_sg_problem& P, TriTables& T, std::string& err);
// sensor shell, filter factors and element-mean weights of the host tables, by total degree
void tri_filter_tables(const fr_sg_problem& P, const TriTables& R, HostTables& T);

// ---------------------------------------------------------------------------
// device-side view of the tables (one allocation, sub-arrays by offset)
// ---------------------------------------------------------------------------
struct DevTab {
  const double* r;
  const double* w;
  const double* D;
  const double* lL;
  const double* lR;
  const double* dhL;
  const double* dhR;
  const double* V;
  const double* Vinv;
  const double* Phi;
  const double* PW;
  const double* filt;
  const double* shell;
  const double* swts;
  const double* cmax;  // [M] max over the random nodes of |Phi_k|
  const double* PhiT;  // [Nq][M] node-major copies of Phi and PW (one node's modes contiguous)
  const double* PWT;
  const double* op1;   // 1D point operators in one block: lL, lR, dhL, dhR, mean weights, D, Vinv, V
  const double* PWB;   // [ceil(M / kProjBlock)][Nq][kProjBlock] PW by blocks of modes, zeros past the last mode
};

// Everything a kernel needs about the problem, passed by value.
struct KParams {
  int eq, dim;
  int E, nx, ny, nsp, M, Nq, S, np1;
  double dx, dy, Jx, Jy;
  double adv, gamma;
  int bc[4];
  double bc_state[4][4];
  double cfl;
  int filter, sensor, limiter;
  int flux;  // FRSG_FLUX_*
  double alpha, sensor_thr;
  int fp32;  // 1: FP32-mixed node loops (1D stage and adjoint kernels)
  int bf16;  // 1: BF16-split matrix-core transforms (1D stage kernel)
  DevTab tab;
  // triangles (element = FRSG_ELEM_TRI; tri = 0 on quadrilateral meshes)
  int tri, nfp;
  const double* tri_Dr;    // [N_p][N_p]
  const double* tri_Ds;
  const double* tri_Lf;    // [3 nfp][N_p]
  const double* tri_lift;  // [N_p][3 nfp]
  // per row group (tri_row_groups): for each point j the group's rows of L, Dr~ and Ds~ at
  // column j, then for each flux point the group's rows of the lifting; rows past the last are 0
  const double* tri_rows;
  const double* tri_geo;   // [E][kTriGeo]
  const double* tri_V;     // [N_p][N_p] orthonormal modes at the solution points, and inverse
  const double* tri_Vinv;
  const int* tri_nbr;      // [E][6]
  unsigned* status;
  unsigned long long* lam_bits;  // CFL accumulator (bit pattern of a positive double)
  double* dt;                    // device time step of the current step
};

constexpr int kRkMaxTerms = 8;  // stages of the largest tableau integrator, and more

struct Workspace {
  double* w1 = nullptr;
  double* w2 = nullptr;
  double* Un = nullptr;    // [S][Nq][E][nsp] nodal solution, then nodal residual
  double* Fn = nullptr;    // [S][Nq][E][nsp] nodal x-flux
  double* Gn = nullptr;    // [S][Nq][E][nsp] nodal y-flux (2D)
  double* Corr = nullptr;  // [S][Nq][E][nface] interface-flux minus interpolated flux
  // fused triangles: modal traces [S][M][E][3 nfp] of a stage input, two buffers used in turn
  double* Tm[2] = {nullptr, nullptr};
  double* scal = nullptr;  // scalars: dt, lam bits, status
  double* lam1d[2] = {nullptr, nullptr};  // whole 1D steps: per-workgroup CFL maxima, two arrays in turn
  // adjoint (scalar 1D problems): stage adjoints, trace adjoints, partial sums
  double* avb = nullptr;   // adjoint of the unfiltered end-of-step state
  double* ab2 = nullptr;   // adjoint of w2
  double* ab1 = nullptr;   // adjoint of w1
  double* agT = nullptr;   // [Nq][E][2] adjoints of the traces at r = -1, +1
  double* apart = nullptr; // per-block partial sums of the parameter derivative
  // fused 2D: modal face traces on tile boundaries, written by one stage launch
  // for the next (two buffers, used in turn)
  double* tr[2] = {nullptr, nullptr};
  // tableau integrators: one right-hand-side buffer per stage
  double* rk[kRkMaxTerms] = {nullptr};
  size_t bytes = 0;
};

// byte offsets of the workspace sub-arrays (each 256-byte aligned) and its size
struct Layout {
  size_t sc = 0, tab = 0, f32 = 0, tri = 0, nbr = 0;
  size_t w1 = 0, w2 = 0, un = 0, fn = 0, gn = 0, co = 0;
  size_t avb = 0, ab2 = 0, ab1 = 0, agt = 0, apt = 0;
  size_t tr0 = 0, tr1 = 0, tm0 = 0, tm1 = 0;
  size_t more = 0, lam0 = 0, lam1 = 0;
  size_t rk[kRkMaxTerms] = {0};
  int nrk = 0;
  bool adj = false, has_tr = false, has_tm = false;
  size_t total = 0;
  size_t opt = 0;    // from here on what steps are faster with (and a triangle operator table)
  size_t need = 0;   // enough to run
  size_t least = 0;  // what counts against the size of the static workspace
};

}  // namespace frsg

struct PassRecord {
  std::string name;
  double alg_bytes;
  int ev0, ev1;  // indices into the event pool
};

struct PassTotal {
  std::string name;
  long launches = 0;
  double ms = 0.0;
  double alg_bytes = 0.0;
};

struct fr_sg_ctx {
  fr_sg_problem prob;
  bool timing = false;
  std::vector<hipEvent_t> events;
  int events_used = 0;
  std::vector<PassRecord> pending;
  frsg::HostTables T;
  frsg::TriTables tri;           // triangle operators and geometry (element = FRSG_ELEM_TRI)
  bool is_tri = false;
  bool fused_tri = false;        // fused triangle stage kernel
  hipStream_t stream = nullptr;
  int dim = 1;
  int S = 1;
  int E = 0;
  int nsp = 0;
  const double* dDt = nullptr;
  const double* dcmax = nullptr;
  const double* dPhiT = nullptr;
  const double* dPWT = nullptr;
  const float* dPhiT32 = nullptr;  // FP32 copies of the node-major tables
  const float* dPWT32 = nullptr;
  bool fused = false;            // fused 2D Euler stage kernel (FP32-mixed, and the element-wise passes)
  bool quad = false;             // matrix-core 2D Euler stage kernel (FP64, BF16-split)
  bool quad_rhs = false;         // ... for fr_sg_rhs too (or for it alone)
  const double* dfrag = nullptr; // its operand tables
  bool fused1d = false;          // fused 1D stage kernel
  bool step1d = false;           // a whole 1D step in one launch
  bool resident1d = false;       // SSP-RK3 steps of a small 1D problem in one one-workgroup launch
  int lam_cur = 0;              // which CFL accumulator holds the maximum of the current state
  const double* lam_for = nullptr;  // state whose maximum the previous step recorded (fr_sg_steps)
  int tr_cur = 0;               // fused 2D: which face-trace buffer holds the traces of the current state
  int tm_cur = 0;               // fused triangles: which trace buffer holds the traces of the current state
  frsg::KParams kp;
  frsg::Workspace ws;
  frsg::Layout lay;                  // sub-arrays of the caller's workspace
  std::vector<double> host_tab;      // tables waiting for the upload in fr_sg_init
  std::vector<size_t> tab_off;       // offsets of the tables in host_tab (and on the device)
  std::vector<double> host_tri;      // triangle operators and geometry
  std::vector<double> host_more;     // tables of the whole-step 1D kernel or of the fused triangle stage
  std::vector<float> host_f32;       // FP32 chaos tables of the fused 2D path
  std::string err;
};

namespace frsg {
// fr_sg_init's work on a given device workspace (frsg_api.cpp), and the text that
// fr_sg_last_error(NULL) reports after a failed init
// (check_device: confirm that the caller's pointer is device memory)
// sizes for fr_sg_workspace_size and for the static workspace (Layout::total, Layout::least)
fr_sg_status workspace_sizes(const fr_sg_problem* problem, int64_t* bytes, int64_t* least);
fr_sg_status init_with_workspace(const fr_sg_problem* problem, void* hip_stream, void* workspace,
                                 int64_t workspace_bytes, fr_sg_ctx** out, bool check_device);
void set_init_error(const std::string& msg);

// one fused stage of the 2D Euler path (kernels_euler2d.hip)
struct RkTerms {
  const double* K[kRkMaxTerms];
  double a[kRkMaxTerms];
  int n;
};
// Where a stage of the wave kernel has its time step from: P.dt, or (first stage of a CFL step) the
// CFL maximum in lam; the kernel then publishes it in P.dt and dt_used (may be null) and clears lam_reset, the
// accumulator of the step's last stage.  Launches of their own for that cost up to 10 us of a step
// (100 x 50 elements, Bogacki-Shampine, flags cleared by the first stage too: 279 -> 270 us).
struct StageDt {
  const unsigned long long* lam = nullptr;
  unsigned long long* lam_reset = nullptr;
  double* dt_used = nullptr;
};
struct FusedStage {
  const double* in;
  const double* u;
  double* out;
  double cu, cw;
  int stage;  // 0: rhs; 1, 2: limited stage output; 3: end of step
  unsigned char* flag_lim;
  unsigned char* flag_filt;
  unsigned long long* lam_next;
  const double* Dt;
  const double* cmax;
  const double* PhiT;  // [Nq][M] chaos basis at the nodes, node-major
  const double* PWT;   // [Nq][M] quadrature-weighted basis, node-major
  int fp32;            // 1: node loop in FP32 (FP32-mixed precision)
  const float* PhiT32;
  const float* PWT32;
  const double* tr_in = nullptr;  // modal face traces of `in` on tile boundaries (null: from the state)
  double* tr_out = nullptr;       // where to write those of `out` (may be null)
  // tab: out = u + dt (sum_j terms.a[j] terms.K[j] + ka_cur R(in)) instead of cu u + cw (in + dt R),
  // R(in) stored in k_out (may be null)
  int tab = 0;
  RkTerms terms{};
  double ka_cur = 0.0;
  double* k_out = nullptr;
  int flag_or = 0;                     // limiter flags OR-ed into flag_lim (set only where it acts)
  unsigned char* flag_zero = nullptr;  // flags that no stage sets, cleared by the wave kernel (may be null)
  StageDt sdt{};
};
bool fused2d_supported(const KParams& P);
bool fused2d_whole(const KParams& P);  // p = 3 elements in whole tiles: every precision's instances exist

// one stage of the matrix-core 2D Euler path on quadrilaterals (kernels_quad_mfma.hip)
struct QuadStage {
  const double* in;
  const double* u;
  double* out;
  double cu, cw;
  int stage;  // 0: rhs; 1, 2: limited stage output; 3: end of step
  unsigned char* flag_lim;
  unsigned char* flag_filt;
  unsigned long long* lam_next;
  const double* Dt;
  const double* cmax;
  const double* frag;   // operand tables (QuadFragLayout)
  int bf16;             // 1: bfloat16-split transforms (FRSG_BF16_SPLIT)
  const double* tr_in;  // modal face traces of `in` on tile boundaries (required)
  double* tr_out;       // where to write those of `out` (may be null)
};
// modes with which the FP64 steps, and the right-hand side on its own, may take it
constexpr bool quad_fp64_modes(int M) { return M > 10; }
constexpr bool quad_fp64_rhs_modes(int M) { return M >= 10; }
bool quad_mfma_supported(const KParams& P);
// doubles of one modal face-trace buffer of the matrix-core path
size_t quad_trace_count(int nx, int ny, int M);
hipError_t launch_quad_stage(const KParams& P, const QuadStage& S, hipStream_t s);
// modal face traces of a state on every tile boundary face
hipError_t launch_quad_traces(const KParams& P, const double* u, double* tr, hipStream_t s);
// doubles of one modal face-trace buffer of the fused 2D kernel
size_t fused2d_trace_count(const KParams& P, bool fp64);
hipError_t launch_fused_stage(const KParams& P, const FusedStage& S, hipStream_t s);
// ... in FP64 with one element per wave (kernels_wave2d.hip), nodes in groups of four, or with two
// variables per lane and nodes in pairs (the pair kernel, k_stage2d).  The pair kernel has two
// workgroups of 8 elements per compute unit: with half of that or less (256 workgroups) a SIMD has
// one wave of it, and the wave kernel wins at every mode count and integrator (0.6 to 0.87 of its
// time up to 64 x 32 elements).  From there to a full round of workgroups (512) the pair kernel's
// round ends sooner; beyond it the wave kernel's smaller workgroups leave less of the last round
// empty and overlap one another's loads and node loops, at the price of a tenth more instructions
// per element, which pays with 15 modes while the rounds are few.  Four SSP-RK3 steps, p = 3, wave
// against pair kernel in us: 15 modes 722 / 661 at 80 x 40, 937 / 1032 at 100 x 50, 2014 / 2140 at
// 160 x 80, 2744 / 2737 at 192 x 96, 3622 / 3722 at 224 x 112, 4732 / 4638 at 256 x 128; 10 modes 420 /
// 413, 567 / 638, 1314 / 1257 and 3127 / 2766 at the first three and the last of these; 3 modes 310 /
// 273 at 100 x 50.  The line is the SSP-RK3 steps': Butcher rows of 15 modes at p = 3, in which
// the pair kernel spills, would gain on the meshes it keeps too (746 / 977 at 80 x 40, 5425 /
// 7286 at 256 x 128), at p = 2 they lose from 192 x 96 on (3593 / 3446).
// A group of four pads 9 nodes by a third: they go to the wave kernel only where its one wave per
// element fills no SIMD twice (four steps, 154 against 216 us at 18 x 10, 169 against 220 at 30 x 34;
// 0.58 against 0.52 ms per five at 100 x 50), and 5 nodes (padded to 8) never.
constexpr int wave2d_padding(int nq) { return ((nq + 3) & ~3) - nq; }
constexpr bool wave2d_nodes(int nq) { return 3 * wave2d_padding(nq) <= nq; }
constexpr int kWaveTile = 2;  // workgroup of the wave kernel: 2 x 2 elements
inline int wave2d_tiles(int nx, int ny) { return ((nx + kWaveTile - 1) / kWaveTile) * ((ny + kWaveTile - 1) / kWaveTile); }
inline long pair2d_blocks(const KParams& P) { return (long)((P.nx + 3) / 4) * ((P.ny + 1) / 2); }
constexpr long kWaveSmall = 144;  // workgroups of the pair kernel
inline bool wave2d_chosen(const KParams& P) {
  const long blocks = pair2d_blocks(P);
  if (!wave2d_nodes(P.Nq)) return false;
  if (8 * wave2d_padding(P.Nq) > P.Nq) return blocks <= kWaveSmall;
  return blocks <= 256 || (blocks > 512 && blocks <= 2560 && P.M > 10);
}
// A right-hand side on its own has no traces of its input and takes them from the neighbours'
// states, twice as many per element with the wave kernel's tiles: with up to 10 modes the pair
// kernel is ahead from fewer workgroups on (64 x 32 elements: 10 modes 27.9 against 29.2 us, 3
// modes 11.0 against 11.8; 32 x 16 9.7 against 9.0).  Small even p = 3 meshes of 10 modes take the
// matrix-core kernel with a trace pass before it (18 x 10: 15.1 us against the wave kernel's 18.4).
inline bool wave2d_rhs(const KParams& P) { return wave2d_chosen(P) && (P.M > 10 || pair2d_blocks(P) <= kWaveSmall); }
hipError_t launch_wave_stage(const KParams& P, const FusedStage& S, hipStream_t s);
hipError_t launch_fused_cfl(const KParams& P, const double* u, unsigned long long* lam, hipStream_t s);
// sensor-gated filter and/or limiter in place, with the fused kernel's tile layout
hipError_t launch_fused_post(const KParams& P, const double* PhiTd, const double* cmax, double* u, int do_filter,
                             int do_limit, unsigned char* flag_filt, unsigned char* flag_lim, hipStream_t s);
hipError_t launch_dt_from(const KParams& P, const unsigned long long* lam, unsigned long long* lam_reset,
                          double* dt_used, hipStream_t s);
hipError_t launch_set_dt(const KParams& P, double dt, double* dt_used, unsigned long long* lam_reset, hipStream_t s);

// launchers (kernels_generic.hip)
hipError_t launch_set_scalars(const KParams& P, double dt_fixed, hipStream_t s);
hipError_t launch_nodal(const KParams& P, const double* u, double* Un, double* Fn, double* Gn, int do_cfl,
                        hipStream_t s);
hipError_t launch_dt(const KParams& P, int dim, double* dt_used, hipStream_t s);
hipError_t launch_faces(const KParams& P, const double* Un, const double* Fn, const double* Gn, double* Corr,
                        hipStream_t s);
hipError_t launch_resid(const KParams& P, const double* Fn, const double* Gn, const double* Corr, double* Rn,
                        hipStream_t s);
hipError_t launch_project_stage(const KParams& P, const double* Rn, const double* u, const double* w,
                                double* out, double cu, double cw, int rhs_only, hipStream_t s);
hipError_t launch_project_ic(const KParams& P, const double* U0, double* u, hipStream_t s);
hipError_t launch_limiter(const KParams& P, double* u, unsigned char* flags, hipStream_t s);
hipError_t launch_sensor_filter(const KParams& P, double* u, unsigned char* flags, hipStream_t s);
hipError_t launch_fill_flags(unsigned char* flags, long n, hipStream_t s);
// triangle passes (kernels_tri.hip): interactive-flux jumps [S][Nq][E][3 nfp],
// nodal residual into Rn, CFL maximum of the nodal values into P.lam_bits
hipError_t launch_faces_tri(const KParams& P, const double* Un, const double* Fn, const double* Gn, double* Jump,
                            hipStream_t s);
hipError_t launch_resid_tri(const KParams& P, const double* Fn, const double* Gn, const double* Jump, double* Rn,
                            hipStream_t s);
hipError_t launch_cfl_tri(const KParams& P, const double* Un, hipStream_t s);
// end-of-stage work of the fused triangle kernels: the sensor-gated filter (flags of the
// filtered elements into flag_filt) and/or the limiter (flags of the limited ones into
// flag_lim); the flag pointers may be null
struct TriPost {
  int filter = 0, limit = 0;
  unsigned char *flag_filt = nullptr, *flag_lim = nullptr;
};
// where a stage's time step comes from: the CFL maximum in P.lam_bits (the kernel then stores
// it in P.dt), or P.dt; dt_used receives it (may be null)
struct TriDt {
  int from_lam = 0;
  double* dt_used = nullptr;
};
// fused triangle stage (p = 1..4 and the (M, Nq) pairs of the fused 2D kernel): a trace pass
// over `in` into Tm ([E][3][M][S][nfp]) unless traces_ready, then out = cu u + cw (in + dt R(in)),
// or R(in) with rhs_only; `post` on the output (not with rhs_only); with Tm_out the traces
// of the final `out` go there
bool tri_fused_supported(const KParams& P);
hipError_t launch_stage_tri(const KParams& P, const double* in, const double* u, double* out, double cu, double cw,
                            int rhs_only, double* Tm, int traces_ready, double* Tm_out, hipStream_t s,
                            const TriPost& post = TriPost(), const TriDt& tdt = TriDt());
// positivity limiter on triangles with the fused lane layout (fused (p, M, N_q) set)
hipError_t launch_limit_tri(const KParams& P, double* u, unsigned char* flags, hipStream_t s);
// the sensor-gated filter and/or the limiter of `post` as a pass of its own (same set)
hipError_t launch_post_tri(const KParams& P, double* u, const TriPost& post, hipStream_t s);
// CFL maximum of a modal state on triangles into P.lam_bits
hipError_t launch_cfl_tri_modal(const KParams& P, const double* u, hipStream_t s);
// explicit Runge-Kutta stage combination: out = u + dt sum_j a[j] K[j] (flat state of n doubles)
hipError_t launch_rk_combine(const double* u, const RkTerms& T, const double* dt, double* out, long n,
                             hipStream_t s);
hipError_t launch_or_flags(unsigned char* dst, const unsigned char* src, long n, hipStream_t s);
hipError_t launch_copy_dt(const KParams& P, double* dt_used, hipStream_t s);

// fused 1D stage kernel (kernels_fr1d.hip)
bool fr1d_supported(const KParams& P);
// limit: positivity limiter on the output (flag_lim); end_of_step: detector-
// switched filter before the limiter (flag_filt) and the CFL maximum of the
// output into lam_next (may be null).  dt_source: 0 reads the device dt; 1 uses
// dt_fixed; 2 derives it from lam_in; with 1 or 2 the kernel also publishes dt
// (device dt, dt_used) and zeroes lam_reset.
hipError_t launch_stage1d(const KParams& P, const double* in, const double* u, const double* w, double* out, double cu,
                          double cw, int rhs_only, unsigned char* clear_flags, hipStream_t s, int limit = 0,
                          int end_of_step = 0, unsigned char* flag_lim = nullptr, unsigned char* flag_filt = nullptr,
                          unsigned long long* lam_next = nullptr, int dt_source = 0, double dt_fixed = 0.0,
                          const unsigned long long* lam_in = nullptr, unsigned long long* lam_reset = nullptr,
                          double* dt_used = nullptr);
// one stage of a Butcher-tableau step: out = u + dt (sum_j T.a[j] T.K[j] + ka_cur R(in)),
// R(in) also stored in k_out (may be null); the limiter acts on out (flags OR-ed into
// flag_lim), and with end_of_step the detector-switched filter, the limiter and the CFL
// maximum follow as in the SSP-RK3 stage; dt as in launch_stage1d
hipError_t launch_stage1d_tab(const KParams& P, const double* in, const double* u, double* out, double* k_out,
                              const RkTerms& T, double ka_cur, hipStream_t s, int limit, int end_of_step,
                              unsigned char* flag_lim, unsigned char* flag_filt, unsigned long long* lam_next,
                              int dt_source, double dt_fixed, const unsigned long long* lam_in,
                              unsigned long long* lam_reset, double* dt_used);
hipError_t launch_cfl1d(const KParams& P, const double* u, unsigned long long* lam, hipStream_t s);
// whole 1D steps per launch (kernels_step1d.hip).  CFL maxima: n values at `at`, whose
// maximum is that of a state
struct Lam1d {
  const double* at = nullptr;
  int n = 0;
};
struct Step1D {
  const double* in = nullptr;
  double* out = nullptr;             // equal to in only where one workgroup covers the mesh
  double *w1 = nullptr, *w2 = nullptr;  // SSP-RK3: stage states handed out (or null)
  int stages = 3;
  bool tab = false;                  // Butcher rows instead of SSP-RK3
  double rows[4][4] = {};            // row i forms the state after right-hand side i, the last the result
  int limit = 0;
  unsigned char* flags = nullptr;    // [4][E] or null
  double dt = 0.0;                   // > 0: fixed; else from lam
  Lam1d lam;
  double* lam_part = nullptr;        // where the result's maxima go (step1d_partials doubles), or null
  double* dt_used = nullptr;
};
bool step1d_supported(const KParams& P, int stages, bool tab);
bool step1d_one_workgroup(const KParams& P, int stages, bool tab);
long step1d_partials(const KParams& P);  // doubles of one array of CFL maxima
hipError_t launch_step1d(const KParams& P, const Step1D& T, Lam1d* lam_out, hipStream_t s);
// CFL maxima of u into part; with copy the state goes there too
hipError_t launch_cfl1d_part(const KParams& P, const double* u, double* part, double* copy, Lam1d* lam, hipStream_t s);
hipError_t launch_copy_state(const double* a, double* b, long n, hipStream_t s);
// nsteps SSP-RK3 steps (CFL time steps, limiter on every stage output when limit,
// end-of-step filter and CFL maximum) of an FP64 1D problem whose elements fit one
// workgroup, in one launch; lam_in holds the CFL maxima of u, lam_out receives
// that of the result.  flags [nsteps][4][E] and dt_used [nsteps] may be null.
bool fr1d_resident_fits(const KParams& P);
bool fr1d_resident_small(const KParams& P);  // the smaller of them, which the pass record names apart
hipError_t launch_steps1d_resident(const KParams& P, double* u, int nsteps, int limit, unsigned char* flags,
                                   double* dt_used, const Lam1d& lam_in, double* lam_out, hipStream_t s);

// adjoint launchers (kernels_adjoint.hip)
long adjoint_partials(const KParams& P);
hipError_t launch_rhs_adjoint(const KParams& P, const double* Un, const double* g, double* GU, double* Gside,
                              double* gT, const double* x0, const double* x1, const double* x2, double* out,
                              double c0, double c1, double c2, double cg, double* part, double param_scale,
                              double* dparam, hipStream_t s);
bool adj1d_fused_supported(const KParams& P);
long adj1d_partials(const KParams& P);
hipError_t launch_adj_stage1d(const KParams& P, const double* w, const double* g, const double* x0, const double* x1,
                              const double* x2, double* out, double c0, double c1, double c2, double cg, double* part,
                              double param_scale, double* dparam, hipStream_t s);
hipError_t launch_filter_adjoint(const KParams& P, const double* g, const unsigned char* flags, double* out,
                                 hipStream_t s);
}  // namespace frsg
