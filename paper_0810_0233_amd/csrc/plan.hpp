// plan.hpp -- the plan object: tree, lists, derivative tensors and M2L tiles
// of one geometry, plus the expansion buffers of its evaluations.
#pragma once
#include <array>
#include <memory>

#include "internal.hpp"

namespace ccfmm {

// Geometry passed by value to kernels that need the level table.
struct TreeGeom {
  LevelGeom lev[kLMax + 1];
  double lo[3];
  double W[3];
  int L;
  int pad;
};

struct LevelData {
  int32_t ncells = 0;   // occupied cells
  int64_t heap0 = 0;    // first heap id of the level (2^l - 1)
  DevBuf key;           // compact -> key (int32)
  DevBuf coord;         // compact -> integer cell coordinates (3 int32)
  DevBuf parent;        // compact -> parent compact (int32), level >= 1
  DevBuf child;         // compact -> 2 child compact (int32, -1 empty), level < L
  DevBuf near_ptr;      // CSR (ncells+1) of near cells (compact), self included
  DevBuf near_idx;
  int64_t nnear = 0;
  DevBuf far_ptr;       // CSR (ncells+1) of far cells (M2L sources)
  DevBuf far_idx;
  DevBuf far_did;       // dense offset id of each far entry (box wfar)
  int64_t nfar = 0;
  // offset bounds (host): near offsets lie in [-wnear, wnear], every candidate
  // (near or far) in [-wfar, wfar]; cnear = most near cells any cell can have
  int wnear[3] = {0, 0, 0};
  int wfar[3] = {0, 0, 0};
  int64_t cnear = 1;
  int64_t nbox = 1;     // dense offset ids of the level: prod(2 wfar + 1)
  int64_t drow0 = 0;    // derivative-tensor row of dense id 0
  int64_t qoff = 0;     // element offset of the level in Q/V
};

struct Plan {
  MemBudget mem;  // first member: destroyed after every buffer charged to it
  int device = 0;
  int64_t n = 0;
  ccfmm_params prm{};
  int p = 0, L = 0;
  int precision = 0;
  int nbmax = 1;
  int class_bits = 3;
  double s_used = 0.0;
  TreeGeom geo{};
  hipStream_t own_stream = nullptr;
  // the near field runs on a second stream beside the expansion passes
  // (forked after the moment permutation, joined before L2P)
  bool overlap = true;
  double tune_eval_ms[2] = {0.0, 0.0};  // the last autotune's evaluation times: [0] overlapped, [1] one stream
  DevBuf heap_flag_prev;       // occupancy of every heap cell at the previous build
  DevBuf pos_check;            // [0] a position is not finite, [1] one lies outside the caller's box
  bool pairs_stale = false;    // info's direct-pair count not yet taken for the current cells
  bool ever_built = false;     // a build succeeded once (buffers and parameters in place)
  int64_t n_rebuilds_kept = 0;  // rebuilds that kept lists and tiles (same geometry and occupied cells)
  hipStream_t side = nullptr;
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;

  // sorted dipoles
  DevBuf pos;        // [n][3] FP64 input order (device copy)
  DevBuf key, val, key_tmp, val_tmp;
  DevBuf perm;       // sorted -> input index (int32)
  DevBuf yd;         // SoA [3][n] FP64 leaf-relative scaled offsets
  DevBuf yf;         // SoA [3][n] FP32, then [3][n] FP32 residuals (yd - yf)
  DevBuf leaf_start; // 2^L + 1 (int32), by leaf key
  DevBuf lstart, lcount;  // per occupied leaf (compact)
  DevBuf heap_flag, heap_scan;  // occupancy and compact ids over all heap cells
  DevBuf cmap;       // heap id -> compact id within its level, -1 if empty
  std::vector<std::unique_ptr<LevelData>> lev;

  // derivative tensors: one dense table per distinct (g, wfar) of the levels,
  // kept across rebuilds while the keys do not change
  int64_t nrows = 0;
  DevBuf Dd, Df;
  DevBuf Dx;  // rows expanded into the wide M2L kernels' LDS order (three bf16 numbers an entry if ops_bf16)
  bool ops_bf16 = false;
  int64_t pos_later = 0;  // bytes of positions a plan made from host memory takes in at the end
  DevBuf Qr;  // folded (traceless-form) moments, nred_stride(p) per row, for the wide M2L kernels
  int dtab_p = 0;
  std::vector<std::array<double, 6>> dtab_keys;
  // M2L tiles
  int TB = 64, TC = 1, ncg = 1;  // configs per tile, targets per tile, config groups
  int m2l_variant = kM2LBlock;    // kernel used by run_m2l
  // the last M2L left the local rows folded (their n_z <= 1 components only)
  // from level 2 (staged L2L) or level 1 (tree form) on; L2L completes them
  bool v_folded = false;
  // lowest level whose folded moments the last M2M wrote with all deeper ones
  // (the M2L pass folds the levels above; -1: none, it folds every level)
  int q_folded = -1;
  int tiles_variant = -1, tiles_class_bits = -1;  // what the current tiles were built for
  DevBuf tiles, tile_tgt, step_delta, step_src, bitmap, gcount;
  DevBuf tile_order;  // launch order of the M2L tiles: longest step list first (+ sort temporaries)
  DevBuf tile_sort;   // target ordering of all levels (keys, order, temporaries, inverse)
  DevBuf near_tmp;    // reordering buffer of the smallest level's near lists
  bool tile_signature = true;  // M2L targets also grouped by their set of far offsets
  int64_t ntiles = 0, nsteps = 0;
  // M2L of a small system: a tile's step list is cut into parts, each a block
  // of its own that leaves its sums in m2l_part (nlaunch blocks in all)
  int64_t nlaunch = 0;
  bool m2l_split = false;
  bool m2l_whole = false;  // never again: the parts' sums were given back
  DevBuf part_off, m2l_part;
  // P2P chunks (built on the device; their count stays in device memory)
  DevBuf chunks, chunk_cnt;
  int64_t nchunks_cap = 0;
  int64_t nchunks = 0;  // filled at info time
  // expansions (compact cells of all levels)
  DevBuf Q, V;
  int64_t qv_elems = 0;
  int qv_batch = 0;  // nbatch the Q/V buffers are laid out for
  DevBuf m_sorted;   // moments in sorted order [b][3][n] (FP64 or FP32)
  DevBuf chunks_b, dleaf;     // pieces of the several-configuration near field; smallest cell of each dipole
  int64_t nchunks_b_cap = 0;  // capacity of that list (the launches cover it)
  // FP16 near field of a mixed plan: granules of 8 sources (first of each cell,
  // first dipole and count of each), their positions and residuals, and the
  // split moments of an evaluation with each configuration's largest and smallest
  DevBuf gran_start, gran_src, gran_pos, gran_m, gran_top;
  int64_t ngran_cap = 0;
  bool has_gran = false;   // granules are laid out for the current positions
  bool gran_off = false;   // they were given back once: not laid out again for later positions
  bool near_f16 = false;  // the current batch runs that near field
  DevBuf scratch;    // scan/sort temporaries
  DevBuf scratch2;
  DevBuf flags;      // device error flags
  // per-smallest-cell order and opening angle (compact leaf order); the levels
  // above keep (p, theta).  theta is stored squared, as the list test uses it.
  bool has_leaf = false;
  DevBuf leaf_p, leaf_th2;
  std::vector<int32_t> h_leaf_p;    // host copies of the per-cell parameters
  std::vector<double> h_leaf_theta;
  double leaf_theta_min = 1.0;
  int tiles_nb = 1;                 // nbatch the M2L tiles were built for
  DevBuf judge_a, judge_b;          // field buffers of the selector's judge
  // learned mode (selector = 1): network weights, and whether the per-cell
  // choice must be made at the next evaluation (new plan, new weights, or an
  // update that changed the occupied cells)
  DevBuf sel_w;
  bool has_sel_w = false;
  bool sel_stale = true;
  // captured evaluation graph, valid for (g_nb, g_m, g_H) until the next rebuild
  bool use_graph = true;
  hipGraphExec_t gexec = nullptr;
  int g_nb = 0;
  const void* g_m = nullptr;
  void* g_H = nullptr;
  DevBuf host_m, host_H;  // staging of the host-pointer evaluation (stable addresses)
  DevBuf energy_part;     // per-block partial sums of the energy (nbatch x kEnergyBlocks)
  ccfmm_info info{};
  bool built = false;
  void drop_graph() {
    if (gexec) (void)hipGraphExecDestroy(gexec);
    gexec = nullptr;
  }
  // the FP16 near field's buffers given back, the next evaluation on the vector
  // units (false: there were none)
  bool drop_granules() {
    if (!has_gran) return false;
    drop_graph();
    for (DevBuf* b : {&gran_start, &gran_src, &gran_pos, &gran_m, &gran_top, &chunks_b}) b->release();
    has_gran = near_f16 = false;
    gran_off = true;
    qv_batch = 0;
    return true;
  }
  // (MemBudget::spare)  A cap is kept with what the chosen forms need, except for
  // the FP16 near field; where the device itself has no more memory, the plan goes
  // on with the forms that need the least.
  bool give_back(bool no_memory) {
    if (m2l_part.p && !m2l_split) {  // of an earlier batch's tiles
      m2l_part.release();
      return true;
    }
    if (drop_granules()) return true;
    if (!no_memory) return false;
    if (m2l_part.p) {
      drop_graph();
      m2l_part.release();
      m2l_whole = true;
      tiles_variant = -1;
      return true;
    }
    if (ops_bf16 && Dx.p) {
      drop_graph();
      Dx.release();
      ops_bf16 = false;
      dtab_p = 0;
      return true;
    }
    return false;
  }
  ~Plan() {
    drop_graph();
    if (ev_fork) (void)hipEventDestroy(ev_fork);
    if (ev_join) (void)hipEventDestroy(ev_join);
    if (side) (void)hipStreamDestroy(side);
  }
};

// build steps (tree.hip, lists.hip, expansions.hip)
// occupied smallest cells for every depth 0..24 (G24: the geometry at depth 24)
void count_occupied_by_depth(Plan& P, const double* d_pos, const TreeGeom& G24, hipStream_t st, int64_t* occupied);
void build_tree(Plan& P, const double* d_pos, hipStream_t st, bool* same_cells = nullptr,
                const int32_t* d_check = nullptr, int32_t* h_check = nullptr);
void build_lists(Plan& P, hipStream_t st);
void build_dtensors(Plan& P, hipStream_t st);
void build_m2l_tiles(Plan& P, int nbatch, hipStream_t st);
void build_p2p_chunks(Plan& P, hipStream_t st);
// whether a mixed plan's near field of nb configurations runs on the FP16 matrix
// cores, which take the same time for 1 to 8
bool near_f16_wanted(const Plan& P, int nb);
// alloc(), buffers the plan can do without: nothing is given back for them, nor do
// they take the room of the positions that are still to come in (a plan with bf16
// operators gives those up for the positions).  False where the cap has no room;
// what was allocated until then is kept.
template <typename F>
bool optional_room(Plan& P, F&& alloc) {
  struct Scope {
    Plan& P;
    decltype(P.mem.spare) spare;
    int64_t later;
    explicit Scope(Plan& q) : P(q), spare(q.mem.spare), later(q.ops_bf16 ? 0 : q.pos_later) {
      P.mem.spare = nullptr;
      P.mem.used += later;
    }
    ~Scope() {
      P.mem.spare = spare;
      P.mem.used -= later;
    }
  } scope(P);
  try {
    alloc();
  } catch (const StatusError& e) {
    if (e.status != CCFMM_ENOMEM) throw;
    return false;
  }
  return true;
}
// the same for the FP16 near field's buffers, all of them given back if one has no room
template <typename F>
bool spare_room(Plan& P, F&& alloc) {
  if (optional_room(P, alloc)) return true;
  P.has_gran = true;
  P.drop_granules();
  return false;
}
void build_granules(Plan& P, hipStream_t st);
size_t near_f16_moment_bytes(const Plan& P, int nb);
void run_gran_moments(Plan& P, int nb, hipStream_t st);

// evaluation passes
void run_p2m(Plan& P, int nb, const double* d_m, hipStream_t st);
void run_m2m(Plan& P, int nb, hipStream_t st);
// M2M and L2L with one level per launch (the fastest for a batch alone on its
// stream) or several levels per launch (a single configuration, or beside the
// near field, where every launch waits for room on the compute units)
inline bool shifts_staged(const Plan& P, int nb) { return !P.overlap && nb >= 2; }
void run_m2m_tree(Plan& P, int nb, bool fold, hipStream_t st);
void run_l2l_tree(Plan& P, int nb, bool folded, hipStream_t st);
void run_m2l(Plan& P, int nb, hipStream_t st);
void run_l2l(Plan& P, int nb, hipStream_t st);
void run_p2p_l2p(Plan& P, int nb, double* d_H, hipStream_t st);  // near + smooth field, one stream
void run_near(Plan& P, int nb, double* d_H, hipStream_t st);     // near field written to H
void run_l2p(Plan& P, int nb, double* d_H, hipStream_t st);      // smooth field added to H
void run_permute(Plan& P, int nb, const double* d_m, hipStream_t st);
void build_wide_ops(Plan& P, hipStream_t st);  // expanded operator rows (Dx) from Df
double m2l_row_share(const Plan& P, int q);  // smallest-level M2L tile work at order q (0..1]
void run_energy(Plan& P, int nb, const double* d_m, const double* d_H, double* d_E, hipStream_t st);
void run_energy_noalloc(int64_t n, int nb, const double* d_m, const double* d_H, double* d_E, hipStream_t st);
void run_direct_targets(int64_t n, const double* d_pos, const double* d_m, int64_t nt,
                        const int64_t* d_idx, double* d_H, hipStream_t st);

// learned selector and per-cell data (selector.hip)
void run_leaf_ids(Plan& P, int32_t* d_out, hipStream_t st);
void run_leaf_errors(Plan& P, int nb, const double* d_H, const double* d_Href, double* d_num, double* d_den,
                     hipStream_t st);
void run_leaf_features(Plan& P, int nb, const double* d_m, float* d_feat, hipStream_t st);
void run_mlp_forward(const float* d_params, int64_t rows, const float* d_x, float* d_y, hipStream_t st);
size_t mlp_grad_bytes(int64_t rows);  // of tmp
void run_mlp_loss_grad(const float* d_params, int64_t rows, const float* d_x, const float* d_t, const float* d_mask,
                       float* d_grad, float* d_loss, DevBuf& tmp, hipStream_t st);
void run_mlp_adam(float* d_params, const float* d_grad, float* d_m1, float* d_m2, int step, float lr,
                  hipStream_t st);
void run_select(Plan& P, const float* d_params, double log_bound, double cost_far, int nb, const double* d_m,
                const double* d_F, int32_t* d_p, double* d_theta, std::vector<int32_t>& hist, double* pred_err,
                hipStream_t st);
double run_rel_rms(const double* d_A, const double* d_B, int64_t count, DevBuf& tmp, hipStream_t st);
void run_scatter_rows(int64_t nt, const int64_t* d_idx, const double* d_src, double* d_dst, hipStream_t st);

// plan-level steps shared by the C ABI and the selector trainer (api.hip)
void apply_leaf_params(Plan& P, const int32_t* hp, const double* hth, hipStream_t st);
void eval_once(Plan& P, int nb, const double* d_m, double* d_H, hipStream_t st);
int select_impl(Plan& P, const float* d_params, double err_bound, double margin, double cost_far, int nbatch,
                const double* d_m, bool judge, hipStream_t st, ccfmm_select_info* out);
// selector weights files (train.hip): write, and read (false if the file
// does not exist; any other problem throws CCFMM_EINVAL)
void selector_file_write(const char* path, const float* h_params);
bool selector_file_read(const char* path, float* h_params);
void train_selector(const ccfmm_train_spec* spec, const char* out_path, float* h_out, ccfmm_train_info* info);

inline int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// Dense offset id of (dx, dy, dz) in the box [-w, w]^3: the eight parities of
// dx + w[0], dy + w[1], dz + w[2] one after another.  M2L steps run in id order
// and the cells of a tile have one parity, so consecutive steps read source cells
// of one parity, an eighth of the surroundings, which stays in an XCD's L2 until
// the tiles beside it ask for it (M2L of a 16.8-million-dipole film x 8, with
// runs of tiles per XCD: 54.1 -> 48.3 ms).
__host__ __device__ inline int64_t box_index(const int w[3], int dx, int dy, int dz) {
  const int a[3] = {dx + w[0], dy + w[1], dz + w[2]};
  int n[3];  // offsets of this parity along each axis
  int64_t base = 0;
  for (int q = 2; q >= 0; q--) {
    // the even half of axis q comes before the odd one, within the halves of the
    // axes before it and with the whole ranges of those after it
    n[q] = w[q] + 1 - (a[q] & 1);
    int64_t size = 1;
    for (int r = 0; r < q; r++) size *= w[r] + 1 - (a[r] & 1);
    for (int r = q + 1; r < 3; r++) size *= 2 * w[r] + 1;
    if (a[q] & 1) base += size * (w[q] + 1);
  }
  return base + ((int64_t)(a[0] >> 1) * n[1] + (a[1] >> 1)) * n[2] + (a[2] >> 1);
}
// the offset of an id
__host__ __device__ inline void box_offset(const int w[3], int64_t id, int& dx, int& dy, int& dz) {
  int n[3], odd[3];
  for (int q = 0; q < 3; q++) {
    int64_t even = w[q] + 1;
    for (int r = 0; r < q; r++) even *= n[r];
    for (int r = q + 1; r < 3; r++) even *= 2 * w[r] + 1;
    odd[q] = id >= even;
    if (odd[q]) id -= even;
    n[q] = w[q] + 1 - odd[q];
  }
  dz = 2 * (int)(id % n[2]) + odd[2] - w[2];
  id /= n[2];
  dy = 2 * (int)(id % n[1]) + odd[1] - w[1];
  dx = 2 * (int)(id / n[1]) + odd[0] - w[0];
}

}  // namespace ccfmm

// the opaque plan handle of the C ABI
struct ccfmm_plan_s {
  ccfmm::Plan P;
};
