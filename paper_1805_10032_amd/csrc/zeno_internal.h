// Internal declarations shared by the translation units of the Zeno HIP library.
// Nothing here is part of the C ABI (that is include/zeno.h).
#ifndef ZENO_INTERNAL_H_
#define ZENO_INTERNAL_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "zeno.h"

// Host-side model object behind zeno_model_t: a chain of linear layers (kind 0) or a
// convolutional network (kind 1: 3 x 3 convolutions, then one fully connected layer).
struct zeno_model {
  int kind;
  zeno_model_desc_t desc;          // kind 0; for kind 1 it describes the fully connected layer alone
  int64_t w_off[ZENO_MAX_LAYERS];  // offset of W_l (l = 0..L-1) inside a parameter vector
  int64_t b_off[ZENO_MAX_LAYERS];  // offset of b_l, or -1
  int64_t d;
  // kind 1
  zeno_cnn_desc_t cnn;
  int map_h[ZENO_MAX_CONV + 1], map_w[ZENO_MAX_CONV + 1], map_c[ZENO_MAX_CONV + 1];  // input and every map
  int64_t conv_w_off[ZENO_MAX_CONV], conv_b_off[ZENO_MAX_CONV];
};

namespace zeno {

// Four floats with 4-byte alignment: rows of G and the per-layer blocks inside a
// row start at arbitrary 4-byte offsets, and gfx950 global loads/stores of 128
// bits only need dword alignment.
struct __attribute__((packed, aligned(4))) f4u {
  float x, y, z, w;
};

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_a4 __attribute__((aligned(4)));  // same, for 4-byte aligned addresses

// Streaming (non-temporal) 128-bit load from a 4-byte aligned address: rows of G
// are read exactly once, so they should not displace reusable lines in the caches.
__device__ inline f32x4 load_stream4(const float* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const f32x4_a4*>(p));
}
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

inline int ceil_div(long long a, long long b) { return (int)((a + b - 1) / b); }
inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// One linear layer as a launch of the streaming layer kernel sees it.
struct LayerJob {
  long long w_off;     // offset of W_l inside a parameter vector
  long long b_off;     // offset of b_l, or -1
  int N, K;            // layer width out / in
  int Kp;              // K rounded up to a multiple of 64 (tiled operand width)
  int Np;              // N rounded up to a multiple of 64 (tiled width of the next layer's operand)
  int last;            // 1: output layer (raw fp32 results instead of tiled activations)
  const void* A_base;  // tiled activations of the pass at x that feed this layer
  void* Wt;            // W_l in matrix-operand order (written by the pass at x, read by the candidates); may be NULL
  float* Z0;           // [n_r x N] pre-activations at x (written by the pass at x, read by the candidates)
  void* H_base;        // tiled output activations of the pass at x (hidden layers)
};

// One launch of the streaming layer kernel (zeno_layer.hip): the candidates'
// pass through layer `cj` (n_cand workgroup columns, may be 0) and, in the same
// launch, the pass at x through layer `bj` (has_base; normally the NEXT layer,
// whose input the previous launch finished), so that the short pass at x hides
// behind the long candidate stream.
struct LayerArgs {
  const float* G;       // [m x d]
  const float* x;       // [d]
  long long ldg;        // floats between consecutive rows of G
  int n_cand;           // candidates in this launch (0 or m)
  int has_base;         // 1: the launch also runs the pass at x through bj
  int base_blocks;      // leading block indices reserved for the pass at x (multiple of 8)
  int n_r;              // valid samples (rows) in this pass
  int passes;           // groups of 128 samples that the launch runs side by side (0 or 1: one group, of at most 128)
  int row_groups;       // groups of 32 MB rows, a workgroup each (filled in by the launcher: passes, twice that for split operands)
  int float_products;   // wide workgroups with float32 matrix instructions (filled in by the launcher)
  LayerJob cj, bj;
  const void* D_cand;   // tiled scaled activation differences of candidate 0 (delta launches only)
  long long A_stride;   // bytes between consecutive candidates in D_cand
  float* dZ;            // [m x n_r x N] change of the output layer's pre-activations (last layer)
  void* Dl_cand;        // tiled scaled output differences of candidate 0 (hidden layers)
  long long H_stride;   // bytes between consecutive candidates in Dl_cand
  float gamma;
  float neg_inv_gamma;  // -1/gamma, or 0 when gamma == 0 (D is that times the difference, float32: times kScaleD)
  double* norm_partials;  // [m x P] partial sums of squares, or NULL in passes after the first
  // K split of a launch of one-wave tiles (the launcher fills these in from layer_k_plan): k_waves waves of a
  // workgroup share a feature tile and split K (1, or the widest split the LDS layout allows), and K is also
  // split over k_slices workgroups per tile.  Each of those writes its partial accumulators to slice_partials,
  // and the last one to arrive (slice_counters, zero on entry, zero again on exit) adds them in slice order and
  // finishes the tile.  Tiles are numbered [pass at x: its feature tiles] [candidates: slice_group0 +
  // candidate x tiles + tile].
  int k_waves;
  int k_slices;
  long long slice_group0;
  float* slice_partials;
  unsigned int* slice_counters;
  int P;                // partial slots per candidate
  int p_off;            // first slot of this layer
  int wide_nw;          // waves per workgroup a plan chose (4 or 8; 0: from the launch's size)
  // Sliced tail of a launch of eight-wave workgroups (see layer_tail_slices): the tiles of the last tail_cand
  // candidates, and of the pass at x if the launch carries it, run as tail_slices K slices each, in the blocks
  // from main_blocks on.  tail_cand = n_cand: all tiles of a launch of four-wave workgroups (see layer_wide_plan).  Their partial accumulators go through slice_partials / slice_counters as well; their
  // partial norms to the slots tail_p_off + tile * tail_slices + slice.
  int tail_cand;
  int tail_slices;
  int tail_p_off;
  int main_blocks;      // filled in by the launcher
  int src_chunk;        // sources per scheduling unit, filled in by the launcher
};

// Float32 operands of a linear layer that stand in operand order are stored scaled by powers of two: the activations of the pass at x,
// the candidates' D and the copy of W.  The split of an operand into bf16 pieces rounds the leading one to nearest, to infinity from
// 0x1.ffp127 (3.396e38) on: scaled, no finite operand gets there, and sums have two binary digits of room at the end of the range.  Both
// products of a candidate, (H0 / 4) U and (D / 2) ((W - gamma U) / 2), come out at a quarter; the epilogue's addition of the bias takes
// the factor back.  A candidate's own values are not scaled: where one is that large its squared norm, summed in float32, is infinite and
// the score minus infinity or a NaN, which ranks as minus infinity, whatever the products are.
// (Without scaling: a test of every operand, one instruction in ten of the split, or a leading piece cut toward
// zero, which makes the dropped piece products four times as large.  U scaled as well: score and update of 14 models 2 % longer on
// average, up to 14 %; its largest values taken down in LDS where squares overflow: 0.88 to 1.05 times as long on 54 models, by
// what the compiler made of the branch.)
constexpr float kScaleH = 0.25f, kScaleD = 0.5f, kScaleW = 0.5f;

inline int launch_passes(const LayerArgs& a) { return a.passes > 1 ? a.passes : 1; }

// Launchers.  Each returns the hipError_t of its launches.
// also clears the n_counters workgroup-arrival counters of the pass (may be 0)
// ... and n_zero doubles at `zero` (the candidates' partial-norm slots; may be 0)
hipError_t launch_pack_features(const float* features, int n_r, int K, int Kp, int n_pad, bool bf16,
                                void* tiled, unsigned int* counters, int n_counters, double* zero, long long n_zero,
                                hipStream_t stream);
// Limits of a launch whose K is split over workgroups: bytes of partial accumulators (tiles x slices x row
// blocks x 4 KB) and tiles (= arrival counters).  One buffer of each serves all launches of a pass, which run
// one after the other and leave the counters at zero.
constexpr size_t kSlicePartialBytes = size_t(8) << 20;
constexpr int kMaxSliceGroups = 2048;
// Sliced tails: at most this many eight-wave workgroups (tiles x slices), each handing over 8 x row blocks x 4 KB
constexpr int kMaxTailWorkgroups = 256;
inline size_t tail_partial_bytes(int MB) { return (size_t)kMaxTailWorkgroups * 8 * MB * 16 * 64 * sizeof(float); }
// Launches of four-wave workgroups cut into K slices: bytes one workgroup hands over, and the most a launch may
constexpr size_t kWidePartialBytes = size_t(32) << 20;
inline size_t wide_slice_bytes(int MB) { return (size_t)4 * MB * 16 * 64 * sizeof(float); }
struct KPlan {
  int k_waves;    // waves of a workgroup that share a feature tile and split K
  int k_slices;   // workgroups per feature tile
};
// The K split a launch with NW waves per workgroup takes (NW > 1: none).  device = false: no device is asked
// for occupancies and the result is the widest split any device could be given (for sizing and checking).
KPlan layer_k_plan(const LayerArgs& a, bool bf16, bool delta, int MB, int NW, bool device);
// Which instantiation of the layer kernel a launch took (reported in the per-launch timing records).
struct LaunchShape {
  int waves;       // waves per workgroup that own different feature tiles (1, 4 or 8)
  int k_split;     // waves that share one feature tile and split K (1, 2 or 4; 4, 8 or 16 in launch_first_layer)
  int k_slices;    // workgroups that share one feature tile and split K (1 to 8)
  int streaming;   // 1: rows read with non-temporal loads (line-aligned layout), 2: the same on the shifted column grid
  int row_blocks;  // 32-sample accumulator blocks of a group of 128 samples (1, 2 or 4), whatever number of workgroups shares them
};
hipError_t launch_layer(const LayerArgs& a, bool bf16, bool delta, int MB, hipStream_t stream,
                        LaunchShape* shape = nullptr);
// ---- the packing of the batch and the pass at x through layer 0 in one launch (zeno_first.hip)
struct FirstArgs {
  const float* x;
  const float* features;   // [n_r x job.K]
  int n_r;
  LayerJob job;            // layer 0 (a hidden layer); Z0 and H_base are written
  void* tiled;             // the batch in operand order, written
  unsigned int* counters;  // cleared, with n_zero doubles at zero, as launch_pack_features does
  int n_counters;
  double* zero;
  long long n_zero;
};
bool first_layer_fits(int K, int n_r);
hipError_t launch_first_layer(const FirstArgs& a, bool bf16, hipStream_t stream, LaunchShape* shape);
bool layer_merge_pays(const LayerArgs& a, bool bf16, bool delta, int MB);  // run a.bj inside the candidates' launch?
// K slices of all tiles of a launch of four-wave workgroups (1: whole tiles), 0: the launch keeps its shape
int layer_wide_plan(const LayerArgs& a, bool bf16, bool delta, int MB, size_t budget);
// ... and the most it may be whatever the device (0: never such a launch)
int layer_wide_most(const LayerArgs& a, bool bf16, bool delta, int MB, size_t budget);
// K slices for the tiles of the last (n_cand - *n_main) candidates of an eight-wave launch, or 0: no sliced tail
int layer_tail_slices(const LayerArgs& a, bool bf16, bool delta, int MB, int* n_main);
int layer_tiles(const LayerArgs& a, bool bf16, bool delta, int MB);   // partial-norm slots per candidate the launch fills
int layer_nw(const LayerArgs& a, bool bf16, bool delta, int MB);     // waves per workgroup the launch will use
// Extents a launch with NW waves per workgroup writes (bytes / floats / slots, counted from the start of each buffer).
struct LayerExtents {
  long long wt_bytes;          // operand-order copy of W (pass at x)
  long long hbase_bytes;       // tiled activations of the pass at x
  long long z0_floats;         // pre-activations at x
  long long d_bytes_per_cand;  // tiled scaled activation differences of one candidate
  long long dz_floats;         // output layer's change of pre-activations, all candidates
  int norm_slots;              // partial-norm slots per candidate
  long long slice_bytes;       // partial accumulators of a launch with K split over workgroups
  int slice_counters;          // arrival counters it uses
};
bool layer_passes_merge(const int* dims, int L, int m);   // may groups of 128 samples share their launches?
LayerExtents layer_extents(const LayerArgs& a, bool bf16, bool delta, int MB, int NW, bool device);
hipError_t launch_loss(const float* Z0, const float* dZ, const int32_t* labels, const float* targets,
                       int loss, int m, int n_r_total, int chunk_begin, int chunk_rows, int C,
                       double* sample_diff, hipStream_t stream);
hipError_t launch_score_combine(const double* sample_diff, const double* norm_partials, int P, int m,
                                int n_r_total, float rho, float* scores, hipStream_t stream);
// the same with the candidates' partial norms P_stride slots apart, the first P of them in use
hipError_t launch_score_combine_strided(const double* sample_diff, const double* norm_partials, int P_stride, int P,
                                        int m, int n_r_total, float rho, float* scores, hipStream_t stream);
// both in one launch, for samples that are all there at once and where loss_score_fits
bool loss_score_fits(int n_r, int C);
hipError_t launch_loss_score(const float* Z0, const float* dZ, const int32_t* labels, const float* targets, int loss, int m, int n_r,
                             int C, const double* norm_partials, int P_stride, int P, float rho, float* scores, hipStream_t stream);
// ---- small models in one launch (zeno_small.hip)
struct SmallArgs {
  const float* G;
  const float* x;
  long long ldg;
  int L, dims[ZENO_MAX_LAYERS + 1];
  long long w_off[ZENO_MAX_LAYERS], b_off[ZENO_MAX_LAYERS];
  int loss, n_r;
  const float* features;
  const int32_t* labels;
  const float* targets;
  float gamma, neg_inv_gamma, rho;
  float* scores;
  int pitch;   // filled in by the launcher
};
bool small_model_fits(const int* dims, int L, int m, int n_r, bool bf16);
hipError_t launch_score_small(SmallArgs a, bool bf16, int m, hipStream_t stream);
// x_next != nullptr: also write x_next = x - gamma * average (out may then be nullptr)
hipError_t launch_masked_average(const float* G, long long ldg, const float* scores, int m, long long d, int b,
                                 float* out, int32_t* selected, hipStream_t stream, float gamma = 0.f,
                                 const float* x = nullptr, float* x_next = nullptr);
size_t krum_workspace_bytes(int m);
hipError_t launch_krum(const float* G, long long ldg, int m, long long d, int b, float* out, int32_t* chosen,
                       float* scores_out, void* workspace, hipStream_t stream);
hipError_t launch_median(const float* G, long long ldg, int m, long long d, float* out, hipStream_t stream);          // m <= 128
hipError_t launch_median_select(const float* G, long long ldg, int m, long long d, float* out, hipStream_t stream);   // m <= 1024

// ---- convolutional models (zeno_conv.hip)
// One 3 x 3 convolution (zero padding 1) as the kernel sees it.
struct ConvLayer {
  long long w_off, b_off;  // offsets inside a parameter vector; b_off = -1: no bias
  int Hin, Win, Cin, Hout, Wout, Cout, stride;
};
// One convolution of one pass: of the pass at x or of the candidates.
struct ConvJob {
  ConvLayer L;
  const float* H0_in;     // input map of the pass at x, NHWC [n_r * Hin * Win x Cin] (the images for the first convolution)
  const float* D_in;      // candidate 0's scaled change of the input map, or nullptr (first convolution, pass at x)
  long long D_in_stride;  // floats between candidates
  float* Z0;              // [rows x Cout] pre-activations at x: written by the pass at x, read by the candidates
  float* out;             // pass at x: relu map; candidates: candidate 0's scaled change of the output map
  long long out_stride;   // floats between candidates (candidates' pass)
  int split_out;          // 1: out is a split map (below)
  float out_scale;        // what results are multiplied by: kScaleH or kScaleD with tiled_out, else 1
  int tiled_out;          // 1: out is the operand of the fully connected layer: rows = samples, k = (position, channel),
  int Kp_fc;              //    in matrix-operand order of padded width Kp_fc
  long long pack_off;     // byte offset of the layer's kernel fragments inside a source's
  int pack_sets;          // 2, or 1 for the first convolution
  // filled in by the launcher: (map, channel chunk) units staged at once, groups of eight channels a unit has, multipliers
  // of the quick divisions
  int stage_units, flat, offs_at;
  unsigned magic_wout, magic_hout, magic_wv, magic_hv, magic_ctiles;
};
// Kernels of one convolution as the matrix instructions take them: fragments of 32 output channels x 16 k (a step), split into
// three bf16 pieces of 64 lanes x 16 bytes.  A source's fragments of a layer: [channel tile][U, then W - gamma U][step][piece][lane].
struct ConvPack {
  long long w_off, off;   // of the kernels inside a parameter vector; byte offset inside a source's fragments
  int Cin, Cout, groups;  // groups of eight channels per unit: 2 (a step is a tap of 16 channels) or 1 (two taps of eight)
  int steps, sets;        // steps of one set; 2 sets, or 1 for the first convolution (and W alone for the pass at x)
  int first;              // jobs (channel tile, step) of the layers before
};
constexpr int kConvFragBytes = 3 * 64 * 16;
inline int conv_steps(int Cin) { return Cin > 8 ? (Cin + 15) / 16 * 9 : 5; }
// One launch: the candidates through cj (n_cand > 0) and the pass at x through bj (has_base), which do not
// depend on each other, and two small jobs: the squared norms of the leading aux_count coordinates of aux_m candidates in
// aux_pieces fixed pieces (-> aux_norm[s * aux_P + aux_p_off + piece]) and clearing 16 * aux_zero16 bytes at aux_zero.
struct ConvArgs {
  const float* G;         // [m x d]
  const float* x;         // [d]
  long long ldg;
  int n_cand;             // m, or 0
  int has_base;
  int n_r;
  float gamma, neg_inv_gamma;
  ConvJob cj, bj;
  int aux_m, aux_pieces, aux_P, aux_p_off;
  long long aux_count;
  double* aux_norm;
  void* aux_zero;
  int aux_zero16;
  // the pass at x through a narrow fully connected layer (fc_N > 0): Z0 = H0 W^T + b, [n_r x fc_N], and W in matrix-operand order
  int fc_N, fc_K, fc_Kp;
  long long fc_w_off, fc_b_off;
  const float* fc_h0;     // in matrix-operand order of width fc_Kp
  float *fc_wt, *fc_z0;
  // kernel fragments of candidates 0 .. n_sources - 2 and of x, written by the launch that has pack_jobs, read by the later ones; or nullptr
  unsigned char* pack;
  long long pack_stride;  // bytes between sources
  int pack_jobs, pack_layers, pack_x;   // jobs per source; number of layers; the source that is x
  ConvPack pack_layer[ZENO_MAX_CONV];
  // filled in by the launcher
  int base_blocks, cand_blocks;
  unsigned magic_cand;
};
hipError_t launch_conv(const ConvArgs& a, hipStream_t stream);
// Whether launch_conv takes the pass at x through a fully connected layer of N outputs and K columns as a small job.  With few samples
// and more than eight outputs a million columns keep its few workgroups busy for longer than a launch of its own (step with that / with
// the small job on random models beyond 2^20 columns: up to 8 samples, more than 8 outputs 0.98 on 19, the lowest 0.90; up to 8 outputs
// 1.08 on 15; more samples 1.03 on 10.  2^19 to 2^20 columns, up to 8 samples, more than 8 outputs: 1.08 on 12).
inline bool conv_fc_rides(int N, int K, int n_r) { return N <= 32 && (N <= 8 || K <= (1 << 20) || n_r > 8); }
// Whether convolution `index` of a model may take its kernels as fragments (a model does if all of its convolutions do).  The
// input maps of all but the first are then split maps: three bf16 pieces per value, [sixteen channels][piece][eight
// channels][position][8], one more position of zeros behind the last, channels up to a multiple of 16 (zeros).
bool conv_takes_fragments(const ConvLayer& L, int n_r, int index);
// Estimate by how many microseconds a call with m candidates is longer that way (negative: shorter).
double conv_fragments_cost(const ConvLayer* layers, int n, int n_r, int m);
inline size_t split_map_bytes(int positions, int C) { return (size_t)3 * ((C + 15) / 16 * 2) * (positions + 1) * 16; }
hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t stream);

}  // namespace zeno
#endif
