// Internal interface between the C-ABI host code and the HIP kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gcdf {

constexpr int kInDim = 9;         // configuration coordinates per knot (x, y, yaw, a1..a6)
constexpr int kInDimSphere = 10;  // network inputs for sphere obstacles: [p', r, a]
constexpr int kTileQ = 64;   // queries per tile (two 32-wide MFMA column blocks)
constexpr int kWaves = 4;    // row groups of the packed weights; a workgroup has as many waves or twice (see waves_for)
constexpr int kThreads = 64 * kWaves;

// kBF16X2F16: forward layers as kBF16X2, reverse sweep as single-pass FP16
// products (transposed weights packed in FP16).
enum Mode : int { kFP32 = 0, kBF16 = 1, kBF16X2 = 2, kBF16X2F16 = 3 };

// Device-resident network in kernel layout.
// Row-indexed arrays are in the kernel's lane-major row order (pack_input_layer,
// pack_row_vectors).
struct DevNet {
  int width;
  int mode;
  int in_dim;         // 9: point obstacles [Np][3]; 10: spheres [Np][4], input [p', r, a]
  const float* w1p;   // [width][12]: W1[r][p'x, p'y, p'z], b1[r], W1[r][a1..a6], W1[r][radius] (0 when in_dim 9), 0
  const float* bh;    // [depth-1][width]: b2, b3, b4
  const float* w5;    // [width]
  const float* b5p;   // device pointer to the output bias
  const void* fwd[3]; // W2, W3, W4 as matrix-core A fragments (see pack_matrix)
  const void* bwd[3]; // W2^T, W3^T, W4^T, same layout
  // kBF16X2F16: set to 1 (host-visible memory) by any query whose d is finite but
  // whose J is not, i.e. the FP16 reverse sweep overflowed (nullable)
  uint32_t* overflow;
};

// What one fused launch computes.
struct Job {
  const float* knots;        // [K][9]
  const float* points;       // [Np][3]
  int64_t K, Np;
  // pair list (pairs mode): pair i = (knots[i], points[i]), or (knots[i],
  // points[pidx32[i]]) when set (a per-knot argmin array); a point index outside
  // [0, Np) yields NaN outputs for that pair
  const int32_t* pidx32;
  int64_t npairs;
  // Gathered knot tiles (dense mode, when tile_off is set): knot i owns rows
  // row_off[i] .. row_off[i+1]-1, row r pairing it with point pgather[r]; its rows
  // form tile_off[i+1] - tile_off[i] tiles of up to tile_q (tile_off[0] = 0), so no tile
  // mixes knots; d and J are indexed by row; ntiles_bound >= tile_off[K] sizes the grid,
  // ntiles_likely estimates tile_off[K] for the choice of the kernel.
  const int64_t* tile_off;
  const int64_t* row_off;
  const int32_t* pgather;
  int64_t ntiles_bound, ntiles_likely;
  int tile_q;                // rows per gathered tile: kTileQ or kTileQ / 2
  float* d;                  // dense: [K][Np]; pairs: [npairs]      (nullable)
  float* J;                  // dense: [K][Np][9]; pairs: [npairs][9] (nullable)
  unsigned long long* minkey;// dense only: [K] inverted (distance, index) keys, zero on entry (nullable)
  // pairs mode, when set: pair i is knot i and the point of key dec_keys[i], which is
  // decoded to dec_dmin[i] and dec_argmin[i] and set back to zero
  unsigned long long* dec_keys;
  float* dec_dmin;
  int32_t* dec_argmin;
  // training (pairs mode): the reverse sweep is seeded with seed[i] = dL/dd_i instead
  // of 1, and the tile's layer inputs h_{l+1} (dumpH[l]) and back-propagated
  // gradients dL/dz_{l+2} (dumpG[l]), l = 0..2, are written as [W x ldb] arrays in
  // the blocked feature-major layout (element (f, i) at ((i / S) W + f) S + i % S,
  // S = 16 bytes of samples), ldb a multiple of 64 (h_4 and dL/dz_1 are only summed).
  const float* seed;
  void* dumpH;
  void* dumpG;
  int64_t ldb;
  // fused MSE loss (training, seed NULL, target set): each tile finishes d before its
  // reverse sweep and seeds it with dL/dd_i = mse_scale (d_i - target_i); the loss
  // adds inv_b (d_i - target_i)^2.
  const float* target;
  float mse_scale, inv_b;
  // training: per-workgroup sums, BF16 [kTrainSumRows][W][grid], FP32
  // [grid][kTrainSumRows][W] (rows: sum_i g_l for l = 1..4; sum_i seed_i h4_i;
  // sum_i g1_i v_c(i) for the nine inputs c; sum_i seed_i; the fused loss), for the
  // train_grid workgroups of the launch; bias_parts: workgroups it has room for
  float* bias_part;
  int bias_parts;
};
constexpr int kTrainSumRows = 16;

// Packed fragment bytes for one width x width matrix.
size_t packed_matrix_bytes(int width, int mode);

// Convert a row-major float32 width x width matrix (device) into the kernel's
// A-fragment layout (device), transposing first if `transpose`.
hipError_t pack_matrix(const float* src, void* dst, int width, int mode, bool transpose, hipStream_t s);

// Build w1p (device) from W1 [width][in_dim] and b1 [width] (device).
hipError_t pack_input_layer(const float* W1, const float* b1, float* w1p, int width, int in_dim, hipStream_t s);

// Reorder nvec consecutive row vectors of length width into lane-major row order.
hipError_t pack_row_vectors(const float* src, float* dst, int width, int nvec, hipStream_t s);

// Every packed array of a network (pack_matrix of W2..W4 and their transposes,
// pack_row_vectors of b2, b3, b4 and w_out, pack_input_layer) in one launch.
struct PackJob {
  int width, mode, in_dim;
  const float* W1;     // [width][in_dim]
  const float* b1;     // [width]
  const float* Wl[3];  // W2, W3, W4 (row-major, width x width)
  const float* bl[3];  // b2, b3, b4
  const float* w5;     // w_out [width]
  void* fwd[3];        // packed W2..W4
  void* bwd[3];        // packed W2^T..W4^T
  float* bh;           // [3][width] lane-major
  float* w5p;          // [width] lane-major
  float* w1p;          // [width][12]
};
hipError_t pack_network(const PackJob& pj, hipStream_t s);

// Obstacle partitions: offsets[i+1] - offsets[i] = number of points within `radius`
// (planar distance) of reference base position i (ref + i * ref_stride), offsets[0] = 0.
// spheres: points hold (x, y, z, s) and the limit is radius + s.
hipError_t launch_partition_count(const float* ref, int64_t N, int64_t ref_stride, const float* points, int64_t M,
                                  bool spheres, float radius, int64_t* offsets, hipStream_t s);
// idx[offsets[i] + k] = k-th point (ascending) of partition i; entries at positions >=
// capacity are not written.
hipError_t launch_partition_fill(const float* ref, int64_t N, int64_t ref_stride, const float* points, int64_t M,
                                 bool spheres, float radius, const int64_t* offsets, int32_t* idx, int64_t capacity,
                                 int num_cu, hipStream_t s);
// tile_off[0] = 0, tile_off[i+1] = tile_off[i] + ceil((offsets[i+1] - offsets[i]) / tile_q).
hipError_t launch_csr_tile_offsets(const int64_t* offsets, int64_t N, int tile_q, int64_t* tile_off, hipStream_t s);
// Sparsity pattern of the stacked constraint Jacobian: row_ptr[r] = n_conf * r (r <= total),
// cols[n_conf * r + c] = col0 + state_dim * knot(r) + c.
hipError_t launch_jacobian_pattern(const int64_t* offsets, int64_t N, int64_t total, int32_t state_dim, int64_t col0,
                                   int64_t* row_ptr, int32_t* cols, hipStream_t s);

// Single-step projection (Theorem 1) over stacked rows r < rows: the knot of row r
// is r / Np (offsets == NULL, dense knot-major rows) or the CSR row's knot;
// qz[r] = knot - f[r] * minv .* J[r] and eik[r] = sqrt(sum_c minv_c J[r][c]^2)
// (either output may be NULL).
struct Minv9 {
  float v[kInDim];
};
hipError_t launch_project(const float* knots, int64_t N, int64_t Np, const int64_t* offsets, int64_t rows,
                          const float* f, const float* J, const Minv9& minv, float* qz, float* eik, hipStream_t s);

// Tiles of tq queries that a job runs (an upper bound for gathered tiles, whose
// offsets are made for one tile size).
inline int64_t query_tiles(const Job& job, bool pairs, int tq) {
  if (pairs) return (job.npairs + tq - 1) / tq;
  return job.tile_off ? job.ntiles_bound : job.K * ((job.Np + tq - 1) / tq);
}
// Whether a query job runs in 32-query tiles (gathered tiles: as its offsets were
// made): when every such tile has a compute unit to itself.  A tile's time is then the
// call's, and 32 queries take little more than half of what 64 take (us a call, 64 /
// 32 queries: W=256 BF16X2_F16 16 x 64 26.3 / 14.8, 100 x 64 26.4 / 15.7; FP32 16 x 64
// 104 / 58; W=512 128 x 64 57 / 46).  Past that, two of them follow each other on a
// compute unit, and 64-query tiles are as fast or faster (200 x 64: W=256 27.5 / 28.6,
// W=512 63 / 79), since each weight fragment then serves twice the queries.
inline bool narrow_tiles(int64_t tiles32, int num_cu) { return tiles32 <= num_cu; }
inline bool narrow_tiles(const Job& job, bool pairs, int num_cu) {
  if (job.dumpH) return false;  // training dumps 64-sample tiles
  if (!pairs && job.tile_off) return job.tile_q == kTileQ / 2;
  return narrow_tiles(query_tiles(job, pairs, kTileQ / 2), num_cu);
}

// Whether a query job in 64-query tiles of width 256 in a split mode runs as one 8-wave
// workgroup per compute unit instead of two 4-wave ones: when each tile has a compute
// unit to itself, so that the second workgroup would have nothing to do and 8 waves
// share the tile's layers (us a call, two 4-wave / one 8-wave, BF16X2_F16: 200 x 64 with
// J 27.7 / 24.5, values 17.0 / 15.2; 250 x 64 with J 30.2 / 27.3; one tile past a round,
// 257 x 64, 35.6 / 44.1, values 23.0 / 26.5).  Gathered tiles: by their likely number
// (128 partitions, 11,763 rows, 247 tiles, at most 312: 35.2 / 31.4).
inline bool one_round(const DevNet& net, const Job& job, bool pairs, int num_cu) {
  return net.width == 256 && (net.mode == kBF16X2 || net.mode == kBF16X2F16) && !job.dumpH &&
         (!pairs && job.tile_off ? job.ntiles_likely : query_tiles(job, pairs, kTileQ)) <= num_cu;
}

// Launch the fused query kernel (dense all-pairs if !pairs, else the pair list).
hipError_t launch_fused(const DevNet& net, const Job& job, bool pairs, bool want_grad, int num_cu, hipStream_t s);
// The same for a sphere network (net.in_dim == 10; points hold (x, y, z, r)); no training.
hipError_t launch_fused_sphere(const DevNet& net, const Job& job, bool pairs, bool want_grad, int num_cu,
                               hipStream_t s);
// Their 32-query tiles (narrow_tiles).
hipError_t launch_fused_narrow(const DevNet& net, const Job& job, bool pairs, bool want_grad, int num_cu, hipStream_t s);
hipError_t launch_fused_sphere_narrow(const DevNet& net, const Job& job, bool pairs, bool want_grad, int num_cu,
                                      hipStream_t s);

// The 8-wave workgroups of one_round.
hipError_t launch_fused_one_round(const DevNet& net, const Job& job, bool pairs, bool want_grad, int num_cu, hipStream_t s);
hipError_t launch_fused_sphere_one_round(const DevNet& net, const Job& job, bool pairs, bool want_grad, int num_cu,
                                         hipStream_t s);

// Decode keys into dmin / argmin and set them back to zero.
hipError_t launch_minkey_decode(unsigned long long* minkey, int64_t K, float* dmin, int32_t* argmin, hipStream_t s);

// ----------------------------------------------------------------------------
// Serving: a persistent kernel claims tiles of published requests.
// ----------------------------------------------------------------------------
constexpr int kMaxSlots = 256;

// One request as the device sees it (written by the host before publication).
// The host rewrites a slot's descriptor only after its previous request has
// completed, seqlock-style: seq = kDescWriting, the fields, then seq = the new
// request's number.  A reader that finds seq != the request it wants (before or
// after reading a field) knows that request has completed.
constexpr uint64_t kDescWriting = ~0ull;
struct ServeDesc {
  uint64_t seq;         // request sequence number; slot = seq % slots
  const float* knots;
  const float* points;
  int64_t K, Np, nblk, ntiles;
  uint64_t done_target; // value of the slot's cumulative done counter when this request is complete
  float* d;
  float* J;
  unsigned long long* minkey;  // [K], zero on entry; set back to zero on completion
  float* dmin;
  int32_t* argmin;
  float* Jmin;                 // [K][9] J at the argmin pairs (NULL: not wanted; needs dmin)
  int32_t want_grad;
  int32_t pad;
};

// Control block in pinned, coherent host memory (host <-> device).
struct ServeCtl {
  uint64_t published;              // number of requests published (host writes, release)
  uint32_t stop;                   // host: exit when no work is claimable
  uint32_t slots;                  // number of request slots in use (<= kMaxSlots)
  uint32_t fault;                  // device: a protocol invariant failed (the host stops serving)
  uint32_t pad;
  uint64_t complete[kMaxSlots];    // seq + 1 of the last request completed in each slot (device writes)
  ServeDesc desc[kMaxSlots];
};

// Claim / completion counters in device memory.
struct ServeDev {
  unsigned long long claim[kMaxSlots];  // (seq << 32) | tiles claimed of request seq
  unsigned long long done[kMaxSlots];   // tiles finished in the slot, cumulative over its requests
  uint32_t drain;                       // epoch of the launch that is draining (0: none yet)
  unsigned long long pub;               // the largest ServeCtl::published any workgroup has seen
  // device copies of the descriptors: ready[slot] = seq + 1 of the request in
  // desc[slot], 0 while it is being written (see store_copy)
  unsigned long long ready[kMaxSlots];
  ServeDesc desc[kMaxSlots];
};

// Launch the persistent serving kernel; it processes published requests from
// sequence number first_seq on and returns once `stop` is set or a workgroup has
// found no work for idle_ticks of the 100 MHz real-time counter.  Exit is
// collective: that workgroup writes `epoch` (non-zero, distinct per launch) into
// dev->drain, and every workgroup stops claiming at its next claim, reports the
// tiles it ran and returns, so a launch never lingers with part of its grid.
// Tiles left unclaimed stay in the claim words for the next launch.
hipError_t launch_serve(const DevNet& net, ServeCtl* ctl, ServeDev* dev, uint64_t first_seq, uint64_t idle_ticks,
                        uint32_t epoch, int num_cu, hipStream_t s);

// p[i] = 0 for i < n (fill kernel; graph-capture safe).
hipError_t launch_fill_zero(unsigned long long* p, int64_t n, hipStream_t s);

// ----------------------------------------------------------------------------
// Training: weight gradients from the dumped H / G (element type = bf16 for the
// BF16 modes, float for FP32).
// ----------------------------------------------------------------------------
// Up to kWgMaxJobs products in one launch: out_j[f][g] = sum_{i < B} G_j[f][i] H_j[g][i]
// for f, g < width (a multiple of 128), via split-K partial sums in `partial`
// (wgrad_partial_floats(B, width, num_cu) floats) reduced in a fixed order.  Rows
// of G and H have stride ldb and hold zeros from B up to the next multiple of 64.
// The batch is cut into as few chunks as keep one workgroup per (product, chunk,
// 128 x 128 output tile) within num_cu, so every workgroup runs in one round.  (Two
// FP32 workgroups per compute unit: batch 65,536 step 732 -> 907 us.)
constexpr int kWgMaxJobs = 3;
struct WgradJobs {
  const void* G[kWgMaxJobs];
  const void* H[kWgMaxJobs];
  float* out[kWgMaxJobs];
  int n;
};
// The training kernel's per-workgroup sums (Job::bias_part, nparts workgroups)
// added in a fixed order: entry f < n[r] of row r goes to base[r][f * stride[r]]
// (rows with a NULL base are dropped).
struct PartOut {
  float* base[kTrainSumRows];
  int stride[kTrainSumRows];
  int n[kTrainSumRows];
};
struct PartSum {
  const float* part;
  int nparts, width;
  bool by_wg;  // part is [nparts][kTrainSumRows][width] (FP32), else [kTrainSumRows][width][nparts]
  PartOut out;
};
// ps (optional): those sums too, in the launch that adds the chunks.
// hipErrorInvalidValue if the launch needs more than partial_floats.
hipError_t launch_wgrad_gemm(const WgradJobs& jobs, int width, int mode, int64_t ldb, int64_t B, float* partial,
                             int64_t partial_floats, int num_cu, hipStream_t s, bool accumulate = false,
                             const PartSum* ps = nullptr);
// samples per chunk (a multiple of 64) for n products, and the floats of `partial`
// any launch of up to kWgMaxJobs products over at most B samples needs
int64_t wgrad_chunk_len(int64_t B, int n, int width, int num_cu);
int64_t wgrad_partial_floats(int64_t B, int width, int num_cu);
// Workgroups of a one-shot launch over ntiles tiles: as many as the device holds at
// once (`resident`), fewer for small launches.
inline int fused_grid(int64_t ntiles, int resident) { return (int)(ntiles < resident ? ntiles : resident); }
// Workgroups of a training launch (and of table1_tiles), by which the per-workgroup
// sums are indexed.  Per compute unit: Geo::WGS of width 256, checked at each launch.
constexpr int train_wgs(int mode) { return mode == kFP32 ? 2 : 1; }
inline int train_grid(int64_t ntiles, int mode, int num_cu) { return fused_grid(ntiles, num_cu * train_wgs(mode)); }


// Table I training loss (width 256, FP32): per 64-sample tile, the forward, the
// reverse sweep for e = dF/dv, the tangent pass along u and the reverse mode through
// both programs (see table1_tiles).  Dumps (blocked feature-major, [W x ldb] each):
//   H[l] = h_{l+1}, G[l] = g_{l+2} (reverse sweep, = d/dz of the tangent output),
//   Hd[l] = hdot_{l+1} (tangent), Zb[l] = zbar_{l+2} (adjoint of the primal), l = 0..2
// (h_4, g_1, hdot_4 and zbar_1 are only summed).  scratch: per workgroup of the grid,
// 11 arrays of kThreads * 64 floats (pre-activations, tangent pre-activations, reverse
// products).
struct T1Job {
  const float* knots;
  const float* points;
  int64_t B, ldb;
  const float* fbar;  // [B] dL/dF per sample
  const float* u;     // [9][ldb] A^T dL/dJ per sample (input-space tangent direction)
  float* H;
  float* G;
  float* Hd;
  float* Zb;
  float* part;  // [grid][kTrainSumRows][W]: sum_i zbar_l (l = 1..4); sum_i fbar_i h4_i + hdot4_i;
                // sum_i zbar1_i v_c(i) + g1_i u_c(i); sum_i fbar_i
  float* scratch;
  int parts;  // workgroups that part and scratch have room for
};
constexpr int kT1ScratchArrays = 11;
hipError_t launch_table1_tiles(const DevNet& net, const T1Job& job, int num_cu, hipStream_t s);
// Per-sample loss terms and their derivatives: from d[i], J[i][9] (the query), targets
// fstar, Jstar, m_diag (9) and lambda (4): fbar[i] = dL/dd_i, u[c][i] (row stride ldb,
// zero from B to ldb), and losses[0..3] = the four averaged terms, losses[4] = total,
// summed in a fixed order (part: 4 * ceil(ldb / 256) floats of scratch).
hipError_t launch_table1_loss(const float* knots, const float* points, const float* d, const float* J,
                              const float* fstar, const float* Jstar, const float* m_diag, const float* lambda,
                              int64_t B, int64_t ldb, float* fbar, float* u, float* part, float* losses,
                              hipStream_t s);

// Adam step over n floats (see gcdf_adam_step).
hipError_t launch_adam(float* p, const float* g, float* m, float* v, int64_t n, float lr, float b1, float b2,
                       float eps, int64_t step, hipStream_t s);

// One Adam update of element i in torch.optim.Adam's operation order (no weight
// decay, no amsgrad); lr_corr = lr / (1 - b1^t), inv_sqrt_bc2 = 1 / sqrt(1 - b2^t).
struct AdamConsts {
  float lr_corr, b1, b2, inv_sqrt_bc2, eps;
  static AdamConsts make(float lr, float b1, float b2, float eps, int64_t step);
};
__device__ __forceinline__ float adam_update(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                                             float* __restrict__ v, int64_t i, const AdamConsts& a) {
  const float gi = g[i];
  const float mi = a.b1 * m[i] + (1.0f - a.b1) * gi;
  const float vi = a.b2 * v[i] + (1.0f - a.b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float denom = sqrtf(vi) * a.inv_sqrt_bc2 + a.eps;
  const float pi = p[i] - a.lr_corr * (mi / denom);
  p[i] = pi;
  return pi;
}
// Adam over the flat parameters of a point network (pj's source pointers point into
// params; grad, m, v share its layout; b_out at params[b5_off]) with every updated
// value also written to pj's packed arrays, in one launch, so the packing of the
// next forward is done.  FP32 and pure-BF16 packings (the training precisions).
hipError_t launch_adam_pack(const PackJob& pj, float* params, const float* grad, float* m, float* v,
                            const AdamConsts& a, int64_t b5_off, hipStream_t s);

}  // namespace gcdf
