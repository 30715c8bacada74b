// Kernel entry points and launch helpers of the NNP engine.
#pragma once

#include "common.h"

namespace nnp {

enum { EPI_CELU = 0, EPI_HEAD = 1, EPI_BWD = 2, EPI_OUT = 3 };

struct GemmArgs {
  const void* A;
  int lda;
  const void* B;   // element s uses B + s * sB: [N][K] row-major, stride ldb
  const void* Bq;  // the same in MFMA fragment order (BF16; nullptr if absent)
  long sB;
  int ldb;
  const float* bias;
  int sBias;
  int N, K;
  const GroupTable* gt;
  void* C;
  int ldc;
  const void* H;   // EPI_BWD: activation whose CELU derivative scales acc
  int ldh;
  const float* w_out;  // EPI_HEAD: output-layer weights [S][N]
  int sWout;
  const float* b_out;  // [S]
  float* erow;         // [atoms] atomic energies in input atom order (EPI_HEAD)
  void* H3;            // optional store of the last hidden activation
  int ldh3;
  const int* perm;     // sorted row -> atom
  const int* mol;      // atom -> molecule
  const double* dLdE;  // per-molecule upstream gradient, or null for ones
  float* uprow;        // optional store of the per-row upstream gradient (EPI_HEAD)
  float alpha;
  float inv_alpha_l2e; // log2(e) / alpha
  float escale = 1.f;  // EPI_HEAD: factor on the upstream gradient (1 / ensemble size)
  // optional per-row k-step masks of the feature rows (launch_aev_fwd's
  // kmask; FP32 LDS-staged kernel): kmask_k skips the K stages (32 columns)
  // that every row of the tile has zero (layer 1, K = the feature columns);
  // kmask_n skips the column blocks no row of the tile needs (dE/dG: the
  // adjoint reads only a row's own k-steps)
  const unsigned long long* kmask_k = nullptr;
  const unsigned long long* kmask_n = nullptr;
};

// The fused network (mlp_net.h).  Weights in fragment order, weight slot
// member * S + element; T is the operand type of the launch.
// A feature row as the fused network takes it: its k-steps, row and atom.
struct alignas(16) NetRow {
  unsigned long long mask;
  int row, atom;
};
constexpr int kNetWindow = 1024;
// order[p] for p over each species group: its rows, in windows of kNetWindow
// by their k-step masks; tiles: the tiles of tile_rows rows in the order the
// workgroups take them.
void launch_net_order(const GroupTable* gt, const unsigned long long* kmask, const int* perm,
                      int ldx, int rows_cap, int tile_rows, NetRow* order, int* tiles,
                      hipStream_t st);
// Rows per tile of the fused network.
template <typename T>
int net_tile(int n_rows, int members, bool ordered);
struct NetArgs {
  const GroupTable* gt;
  int S;
  const void* X;                  // [rows][ldx] feature rows (T)
  int ldx;                        // row stride of X and G, layer 1's K (a multiple of 32)
  const unsigned long long* kmask;  // [rows]: the k-steps (32 columns of X) that may be
                                    // nonzero; X is read, and G written, only there
  const void* W0;                 // [slots][W1][ldx]
  const void* W1;                 // [slots][W2][W1]
  const void* W2;                 // [slots][W3][W2]
  const void* W2T;                // [slots][W2][W3]
  const void* W1T;                // [slots][W1][W2]
  const void* W0T;                // [slots][ldx][W1]
  const float* b0;                // [slots][W1]
  const float* b1;                // [slots][W2]
  const float* b2;                // [slots][W3]
  const float* wout;              // [slots][W3]
  const float* bout;              // [slots]
  float alpha;
  float inv_alpha_l2e;            // log2(e) / alpha
  float escale;                   // factor on the upstream gradient (1 / ensemble size)
  const int* perm;                // sorted row -> atom
  const NetRow* order;            // the rows in the order the tiles take them, or null
  const int* tiles;               // with order: the tiles as the workgroups take them
  const int* mol;                 // atom -> molecule
  const double* dLdE;             // per-molecule upstream gradient, or null for ones
  float* erow;                    // [members][erow_stride] atomic energies, input atom order
  long erow_stride;
  bool bwd;                       // gradients wanted (D1, and G when set)
  void* G;                        // [rows][ldx] dE/dG, or null
  void* D1;                       // optional [rows][ld_d1], member k at columns k * W1
  int ld_d1;
  // the weight gradients' operands, all or none ([rows][width]; D1 too)
  void* H1;
  void* H2;
  void* H3;
  void* D3;
  void* D2;
  float* uprow;                   // [rows] upstream gradient of each row
};

// dE/dG of an ensemble: G = D1 Wc over the members' delta1 side by side
// (lda = K = members * W1), Wc the member-concatenated W_0^T in fragment order
// [S][ldx][K].  Each row is written on its own k-steps.
struct NetGradArgs {
  const GroupTable* gt;
  const void* D1;
  int K;
  const void* Wc;
  const unsigned long long* kmask;
  void* G;
  int ldx;
  const NetRow* order;  // as the network took them (D1's rows lie in that order)
};

// Weight slots: member k of an ensemble, element s -> slot k * S + s.
struct PackArgs {
  const float* flat;
  long off[kMaxModels * kMaxS * kLayers];  // flat offset of W for (slot, layer)
  int S;                  // elements (slot = member * S + element)
  int n_models;
  // ensembles: [S][F_pad][M * width1] member-concatenated W_0^T, row-major
  // (FP32) or in MFMA fragment order (N = F_pad, K = M * width1)
  float* WT0cf;
  bf16_t* WT0cq;
  float* WT0cqf;
  int width[kLayers + 1];
  int Fp;
  int r0, a0;             // layer 1: inputs from r0 on sit at columns from a0 on
  // null: not wanted
  float* Wf[kLayers];     // W [slots][out][in_pad], row-major
  bf16_t* Wb[kLayers];
  float* WTf[kLayers];    // W^T [slots][in_pad][out], row-major
  bf16_t* Wqb[kLayers];   // W in MFMA fragment order (N = out, K = in_pad)
  bf16_t* WTqb[kLayers];  // W^T in MFMA fragment order (N = in_pad, K = out)
  float* Wqf[kLayers];
  float* WTqf[kLayers];
  float* bias[kLayers];
  float* wout;
  float* bout;
};

struct EnergyArgs;  // energy_sum.h

// stage.hip
inline int stage_blocks(int n_cap) { return n_cap > 0 ? (n_cap + 255) / 256 : 1; }
// molecule offsets sampled into LDS by each staging block
constexpr int kOffSamples = 1024;
__global__ void k_fill_i32(int* p, int v, int n);
__global__ void k_fill_f32(float* p, float v, long n);
__global__ void k_fill_f64(double* p, double v, int n);
void launch_stage(int n_arg, int nmol_arg, int n_cap, int* dims, const float* pos,
                  const double* pos64, const int* gidx, int n_total, const int* species,
                  const int* off, int S, float4* xyzs, int* mol, int2* mrange, float* Fzero,
                  int* hist, uint32_t* status, bool clear_status,
                  int* zero, int nzero, hipStream_t st);
void launch_groups(const int* dims, int n_cap, int S, int* hist, GroupTable* gt, int* perm,
                   int rows_cap, const int* off, int wchunk_rows, uint32_t* status,
                   hipStream_t st);
// k_groups + k_scatter in one launch; for n_cap <= 256 * kFusedSortBlocks
// (each block adds up all blocks' counts: beside the pair scan of 77,163 atoms
// that hides, while the two launches took 12 us)
constexpr int kFusedSortBlocks = 512;
void launch_sort_scatter(const int* dims, int n_cap, int S, const float4* xyzs, const int* hist,
                         GroupTable* gt, int* row, int* perm, int rows_cap, const int* off,
                         int wchunk_rows, uint32_t* status, hipStream_t st);
void launch_scatter(const int* dims, int n_cap, int S, const float4* xyzs, const int* hist,
                    int* row, int* perm, hipStream_t st);
void launch_energy(const int* dims, int nmol_cap, const int* off, const float4* xyzs,
                   const float* eatom, int n_models, long mstride, const double* eself,
                   double* E, uint32_t* status, hipStream_t st);
void launch_fill_i32(int* p, int v, int n, hipStream_t st);
void launch_fill_f32(float* p, float v, long n, hipStream_t st);
void launch_fill_f64(double* p, double v, int n, hipStream_t st);

// neighbors.hip
// Neighbor rows (ELL, row i at i * cap): nbr holds atom indices, rec the
// matching records (dx, dy, dz, species bits) with d = x_j - x_i (minimum
// image when periodic), computed by the cutoff predicate's own arithmetic.
void launch_pairs_mol(const int* dims, int n_cap, int nmol_cap, const AevConst& C,
                      const float4* xyzs, const int2* mrange, int cap, int* nbr, float4* rec,
                      int2* counts, uint32_t* status, hipStream_t st);
// launch_sort_scatter and launch_pairs_mol in one launch (n_cap <= 256 * kFusedSortBlocks)
void launch_sort_pairs_mol(const int* dims, int n_cap, int nmol_cap, int S, const int* hist,
                           GroupTable* gt, int* row, int* perm, int rows_cap, const int* off,
                           int wchunk_rows, const AevConst& C, const float4* xyzs, const int2* mrange, int cap,
                           int* nbr, float4* rec, int2* counts, uint32_t* status,
                           hipStream_t st);
// Periodic boxes: cell_cnt holds cell_zero_ints(ncell) ints that staging
// zeroed: the per-cell counts, then (more than kCellScanLds cells) the counting
// launch's done counter.  With gt, the species sort as well
// (n_cap <= 256 * kFusedSortBlocks).
constexpr int kCellScanLds = 8192;
inline size_t cell_zero_ints(int ncell) {
  return (size_t)ncell + (ncell > kCellScanLds ? 1 : 0);
}
void launch_pairs_cell(const int* dims, int n_cap, const AevConst& C, const BoxConst& B,
                       const float4* xyzs, int* cell_of, int* cell_cnt, int* cell_start,
                       int* cursor, int* cell_atoms, float4* cell_xyzs, int cap, int* nbr,
                       float4* rec, int2* counts, uint32_t* status, int S, const int* hist,
                       GroupTable* gt, int* row, int* perm, int rows_cap, const int* off,
                       int wchunk_rows, hipStream_t st);
// Deterministic forces from the adjoint's per-entry rows pgrad ([n][cap],
// dE_i/d(displacement of entry e)): atom a's row out[gidx ? gidx[a] : a] +=
// sign * sum over a's entries e, in list order, of pgrad[a][e] -
// pgrad[j_e][slot of a in j_e's list] (the lists are symmetric; the slot is
// found by binary search on the sort key).  One wave per atom; each row is
// added to once (no atomics).
void launch_force_gather(const int* dims, int n_cap, const float4* xyzs, const float4* rec,
                         const int* nbr, const int2* counts, int cap, const float4* pgrad,
                         float* out, float sign, const int* gidx, int n_total, hipStream_t st);

// aev.hip
// det: one atom per wave.  nmol_cap: molecules (1 or 2 for a box).  kmask (optional, [rows]):
// per row, bit q set when k-step q (feature columns 32 q .. 32 q + 31) holds
// a block the atom touches; sparse (needs kmask and ld <= 2048): only those
// k-steps of the row are stored (the rest of the row is left as it was).
template <typename OutT>
void launch_aev_fwd(const int* dims, int n_cap, int nmol_cap, const AevConst& C,
                    const float4* rec, const int2* counts, int cap, const int* row_of, OutT* out,
                    int ld, bool det, unsigned long long* kmask, bool sparse, hipStream_t st);
// status: whether the lists are whole (the launches before have set its bits).
// pgrad: the deterministic adjoint, writing per-entry rows to pgrad (the
// caller then runs launch_force_gather) instead of scattering into out
template <typename GT>
void launch_aev_bwd(const int* dims, int n_cap, const AevConst& C, const float4* xyzs,
                    const float4* rec, const int* nbr, const int2* counts, int cap, const int* row_of, const GT* g,
                    int ldg, float* out, float sign, const int* gidx, int n_total,
                    const int2* mrange, const uint32_t* status, const EnergyArgs* energy,
                    int nmol_cap, float4* pgrad, hipStream_t st);

// mlp.hip
template <typename T>
bool launch_gemm(int epi, const GemmArgs& a, int rows_cap, hipStream_t st);
// Weight gradients of all layers (input layer first): per-chunk partials in
// one launch (plus one per layer whose widths the MFMA tiles do not take),
// then the chunk-ordered sum into dparams[param_off_dev[s] + e], e over the
// element's whole flat parameter vector.  partial holds n_chunks_cap times
// wgrad_part_pitch of that vector's length in floats.  kmask (null unless
// wgrad_sparse_fits and chunk <= 1,024): the feature rows' k-steps; layer 1
// reads only those (act: n_chunks_cap * 64 bytes).
struct WgradLayer {
  const void* D;  // [rows][ldd] adjoint of the layer's output
  const void* H;  // [rows][ldh] the layer's input
  int ldd, ldh, Nout, Nin;
  bool d_fp32;    // D is FP32 (the output layer's), else the operand type
  // input i (of Nin, in the parameters' order) is column i of H, or
  // i + hgap from hgap0 on (the feature rows' gap before the angular blocks)
  int hgap0 = 1 << 30, hgap = 0;
};
// Floats from one chunk's partial to the next (16-byte aligned).
inline long wgrad_part_pitch(long len) { return (len + 3) / 4 * 4; }
bool wgrad_sparse_fits(int Nout, int ldx, int Nin, int gap0);
template <typename T>
void launch_wgrad_net(const GroupTable* gt, int S, int n_chunks_cap, int chunk,
                      const WgradLayer* layers, int n_layers, const unsigned long long* kmask,
                      unsigned char* act, float* partial, float* dparams,
                      const long* param_off_dev, hipStream_t st);
void launch_pack(const PackArgs& p, int slots, hipStream_t st);

// mlp_net_*.hip: the whole network of a row tile in one workgroup, every
// member of an ensemble in one launch (then launch_net_grad for dE/dG).
// Hidden widths 256-192-160 and 160-128-96, feature rows of at most 2,048
// columns; n_rows: atoms (the tile size follows from it).
inline bool net_widths(const int* width, int ldx) {
  return ldx % 32 == 0 && ldx <= 2048 &&
         ((width[1] == 256 && width[2] == 192 && width[3] == 160) ||
          (width[1] == 160 && width[2] == 128 && width[3] == 96));
}
template <typename T>
bool launch_mlp_net(const int* width, const NetArgs& a, int n_rows, int rows_cap, int members,
                    hipStream_t st);
template <typename T>
void launch_net_grad(const NetGradArgs& a, int n_rows, int rows_cap, hipStream_t st);

// md.hip
void launch_vv_kick_drift(const int* dims, int n_cap, double* x, double* v, const float* F,
                          const double* mass, double dt, float* pos32, hipStream_t st);
void launch_vv_kick(const int* dims, int n_cap, double* v, const float* F, const double* mass,
                    double dt, hipStream_t st);
void launch_lfm_step(const int* dims, int n_cap, double* x, double* v, const float* F,
                     const double* mass, double dt, double c, double kT_acc, uint64_t seed,
                     uint64_t step, float* pos32, hipStream_t st);
void launch_serve_lfm(const int* dims, int n_cap, const int* mol, const int* off,
                      const int* kdone, const int* nsteps, const uint64_t* seed, double* x,
                      double* v, const float* F, const double* mass, double dt, double c,
                      double kT_acc, hipStream_t st);
void launch_kinetic(const int* dims, int nmol_cap, const int* off, const double* v,
                    const double* mass, double* ke, int* kdone, hipStream_t st);
void launch_gather_rows(const int* src, int n, const double* x_old, const double* v_old,
                        const int* sp_old, const double* m_old, const float* f_old,
                        const double* x_new_in, const double* v_new_in, const int* sp_new_in,
                        const double* m_new_in, double* x, double* v, int* sp, double* m, float* f,
                        hipStream_t st);
void launch_serve_integrate(const int* dims, int n_cap, const int* mol, const int* kdone,
                            const int* nsteps, double* x, double* v, const float* F,
                            const double* mass, double dt, hipStream_t st);


}  // namespace nnp
