// Dispatcher of the streaming layer kernel: launch shapes, the choice between merged
// and separate launches of the pass at x, and the packing of the batch.  The kernel
// itself lives in zeno_layer_impl.h and is compiled in ten objects (the four files
// zeno_layer_{bf16,f32}_{first,delta}.hip, each once per number of row blocks).
#include <cstring>

#include "zeno_layer_impl.h"

namespace zeno {

// the entry points of the ten kernel objects: (operand type, second product) x row blocks (four of them in bf16 only)
#define ZENO_DECLARE_LAYER_MB(NAME, MB)                                                                              \
  hipError_t launch_layer_##NAME##_mb##MB(const LayerArgs& a, int NW, hipStream_t stream, LaunchShape* shape);       \
  int wgs_per_cu_##NAME##_mb##MB(int NW, int k_waves);
#define ZENO_DECLARE_LAYER(NAME, MOST)                                                                              \
  ZENO_DECLARE_LAYER_MB(NAME, 1)                                                                                    \
  ZENO_DECLARE_LAYER_MB(NAME, 2)                                                                                    \
  ZENO_DECLARE_LAYER_MB(NAME, MOST)                                                                                 \
  static hipError_t launch_layer_##NAME(const LayerArgs& a, int MB, int NW, hipStream_t stream, LaunchShape* shape) { \
    return MB == 1 ? launch_layer_##NAME##_mb1(a, NW, stream, shape)                                              \
         : MB == 2 ? launch_layer_##NAME##_mb2(a, NW, stream, shape)                                              \
                   : launch_layer_##NAME##_mb##MOST(a, NW, stream, shape);                                          \
  }                                                                                                               \
  static int wgs_per_cu_##NAME(int MB, int NW, int k_waves) {                                                     \
    return MB == 1 ? wgs_per_cu_##NAME##_mb1(NW, k_waves) : MB == 2 ? wgs_per_cu_##NAME##_mb2(NW, k_waves)        \
                                                                     : wgs_per_cu_##NAME##_mb##MOST(NW, k_waves);   \
  }
ZENO_DECLARE_LAYER(bf16_delta, 4)
ZENO_DECLARE_LAYER(bf16_first, 4)
ZENO_DECLARE_LAYER(f32_delta, 2)
ZENO_DECLARE_LAYER(f32_first, 2)
#undef ZENO_DECLARE_LAYER
#undef ZENO_DECLARE_LAYER_MB

template <bool BF16, bool DELTA>
static int ks_waves_for(int MB) {   // (float32: a workgroup has at most two row blocks)
  return MB == 1 ? split_k_waves<BF16, DELTA, 1>() : MB == 2 ? split_k_waves<BF16, DELTA, 2>() : split_k_waves<BF16, DELTA, BF16 ? 4 : 2>();
}

static int compute_units() {
  static const int n_cu = [] {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 1)
      v = 256;
    return v;
  }();
  return n_cu;
}

// Float32 operands: four row blocks run as two groups of two, a workgroup each (G is read twice, the second time mostly from the L2 of
// the XCD both run on).  Split operands have two accumulators per block, and with four blocks neither the LDS nor the registers held
// the buffers that keep loads in flight.  As one group, on float32 matrix instructions (us): 2048 -> 2048, 20 candidates, 573 (now 317);
// one-wave tiles with the second product, whose K no two waves could share, 777 -> 333, 33 candidates, 155.
static int row_groups(bool bf16, int MB) { return !bf16 && MB == 4 ? 2 : 1; }

static int wgs_per_cu(bool bf16, bool delta, int MB, int NW, int k_waves = 1) {
  MB /= row_groups(bf16, MB);
  return bf16 ? (delta ? wgs_per_cu_bf16_delta(MB, NW, k_waves) : wgs_per_cu_bf16_first(MB, NW, k_waves))
              : (delta ? wgs_per_cu_f32_delta(MB, NW, k_waves) : wgs_per_cu_f32_first(MB, NW, k_waves));
}

static int ks_waves(bool bf16, bool delta, int MB) {
  return bf16 ? (delta ? ks_waves_for<true, true>(MB) : ks_waves_for<true, false>(MB))
              : (delta ? ks_waves_for<false, true>(MB) : ks_waves_for<false, false>(MB));
}

// Waves per workgroup of a launch.  Where eight would be picked, four are taken instead if two
// such workgroups fit on a compute unit and the eight-wave workgroups do not fill their rounds of
// (compute units x resident workgroups) almost exactly: the eight waves of a workgroup that has a
// compute unit to itself all wait at the same barrier once per chunk, while two four-wave
// workgroups run out of step and fill each other's waits (workload 4: 800 eight-wave workgroups
// are 3.1 rounds, four waves gain 2-4 % per layer; workload 5: 1024 are exactly four rounds and
// eight waves, which copy the activations once per 256 features instead of once per 128, win).
static int nw_for(const LayerArgs& a, bool bf16, bool delta, int MB) {
  if (a.wide_nw > 0) return a.wide_nw;   // planned (layer_wide_plan, layer_tail_slices)
  const int groups = row_groups(bf16, MB);
  const int nw = launch_nw_for(a);
  if (nw != 8 || a.n_cand <= 0) return nw;
  if (wgs_per_cu(bf16, delta, MB, 4) < 2) return 8;
  const long long slots = (long long)compute_units() * wgs_per_cu(bf16, delta, MB, 8);
  const long long wgs = (long long)job_tiles(a.cj, 256) * a.n_cand * groups;
  const long long rounds = (wgs + slots - 1) / slots;
  return 10 * wgs >= 9 * rounds * slots ? 8 : 4;
}

int layer_nw(const LayerArgs& a, bool bf16, bool delta, int MB) { return nw_for(a, bf16, delta, MB); }

static long long one_wave_tiles(const LayerArgs& a) {
  return (a.has_base ? job_tiles(a.bj, 32) : 0) + (long long)(a.n_cand > 0 ? job_tiles(a.cj, 32) : 0) * a.n_cand;
}

// K split of a launch of one-wave tiles.  Such a launch has few feature tiles (the pass at x: N/32; a narrow
// layer: one or a few per candidate), so a tile's K is divided among the k_waves waves of its workgroup (which
// add their accumulators through LDS) and among k_slices workgroups (which add theirs through memory, the
// last one to arrive finishing the tile).
//  * The waves of a workgroup split K as widely as the LDS layout allows (four or two private copies), wherever each gets a chunk of
//    the candidates' K (a pass at x with fewer chunks leaves some of them without any).
//  * Workgroups per tile: as many as bring the launch to about one workgroup per compute unit, at most 8; every wave keeps two chunks.
//    Measured: on an otherwise idle chip every doubling helps down to two chunks per wave (a ten-class
//    layer behind 4096 inputs, 20 candidates: 8 slices 35 us, 4 slices 42 us), while a launch that already
//    has a workgroup per compute unit only gets slower (its workgroups queue, and the round trips of the
//    hand-over, cheap on an idle chip, take several microseconds each once the memory system is loaded).
//  * One exception: a launch with somewhat more tiles than compute units whose wide workgroups fit only one
//    per compute unit (four LDS layouts) would run a full round and a nearly empty one.  One-wave
//    workgroups, two per tile, several per compute unit, run it in one round.  Most launches of more than 64
//    features take four-wave workgroups instead (layer_wide_plan).  Score and update, without / with it: fp32, n_r = 32,
//    2048 -> 64, m = 140 and 185: 81.1 / 77.1, 92.3 / 88.2 us; 3072 -> 50, m = 150: 102.5 / 99.3; 4096 -> 64, m = 130:
//    102.0 / 98.4; with n_r = 64 103.3 / 98.0, 115.2 / 131.6 (the one shape that loses), 133.3 / 129.3, 140.4 / 136.1.
KPlan layer_k_plan(const LayerArgs& a, bool bf16, bool delta, int MB, int NW, bool device) {
  KPlan plan = {1, 1};
  if (NW != 1 || (!a.has_base && a.n_cand <= 0)) return plan;
  const int base_chunks = a.has_base ? a.bj.Kp >> 6 : 1 << 30, cand_chunks = a.n_cand > 0 ? a.cj.Kp >> 6 : 1 << 30;
  const int min_chunks = base_chunks < cand_chunks ? base_chunks : cand_chunks;
  const int row_blocks = MB / row_groups(bf16, MB);
  const long long groups = row_groups(bf16, MB) * one_wave_tiles(a);
  const int ks_max = ks_waves(bf16, delta, row_blocks);
  const bool wide_ok = ks_max > 1 && (a.n_cand > 0 ? cand_chunks : base_chunks) >= ks_max;
  const bool can_slice = a.slice_partials != nullptr && a.slice_counters != nullptr && groups <= kMaxSliceGroups;
  // most workgroups per tile that the buffers and the two-chunk rule allow
  auto max_slices = [&](int kw) {
    if (!can_slice) return 1;
    long long s = min_chunks / (2 * kw);
    const long long by_bytes = (long long)(kSlicePartialBytes / ((size_t)row_blocks * 16 * 64 * sizeof(float))) / groups;
    if (s > by_bytes) s = by_bytes;
    if (s > 8) s = 8;
    return s < 1 ? 1 : (int)s;
  };
  plan.k_waves = wide_ok ? ks_max : 1;
  if (!device) {
    // sizing: the split over workgroups is widest for one-wave workgroups
    plan.k_slices = max_slices(1);
    return plan;
  }
  const int n_cu = compute_units();
  long long s = n_cu / groups;
  const int cap = max_slices(plan.k_waves);
  if (s > cap) s = cap;
  plan.k_slices = s < 1 ? 1 : (int)s;
  if (wide_ok && plan.k_slices == 1 && max_slices(1) >= 2 && (a.n_cand > 0 ? cand_chunks : base_chunks) >= 32 &&
      groups > (long long)n_cu * wgs_per_cu(bf16, delta, MB, 1, ks_max) && 2 * groups <= 3LL * n_cu &&
      2 * groups <= (long long)n_cu * wgs_per_cu(bf16, delta, MB, 1, 1)) {
    plan.k_waves = 1;
    plan.k_slices = 2;
  }
  return plan;
}

// Does any candidate launch of these layers take eight-wave workgroups?  Those run one group of 128 samples at a time.  Host
// arithmetic only: the workspace's size depends on it.
bool layer_passes_merge(const int* dims, int L, int m) {
  for (int l = 0; l < L; ++l)
    if (pick_nw(cover_rows(dims[l + 1], l + 1 == L), m) == 8) return false;
  return true;
}

// What a launch of workgroup width NW writes, from the kernel's own index formulas: the
// host checks these against the workspace slots before anything is enqueued.
LayerExtents layer_extents(const LayerArgs& a, bool bf16, bool delta, int MB, int NW, bool device) {
  LayerExtents e;
  std::memset(&e, 0, sizeof(e));
  const int esize = bf16 ? 2 : 4, wregs = bf16 ? 4 : 8, passes = launch_passes(a), n_pad = 32 * MB * passes;
  auto tiled_bytes = [&](int Np) {
    const long long last = bf16 ? tiled_index<true>(n_pad - 1, Np - 1, Np) : tiled_index<false>(n_pad - 1, Np - 1, Np);
    return (last + 1) * esize;
  };
  if (a.has_base) {
    const LayerJob& j = a.bj;
    // every wave of every workgroup of the pass at x stores its 32-row tile of W, chunk by chunk
    if (j.Wt != nullptr) e.wt_bytes = (long long)job_tiles(j, 32 * NW) * NW * (j.Kp >> 6) * wregs * 1024;
    e.z0_floats = (long long)a.n_r * j.N;
    if (!j.last) e.hbase_bytes = tiled_bytes(j.Np);
  }
  if (a.n_cand > 0) {
    const LayerJob& j = a.cj;
    if (j.last) e.dz_floats = (long long)a.n_cand * a.n_r * j.N;
    else e.d_bytes_per_cand = tiled_bytes(j.Np);
    e.norm_slots = job_tiles(j, 32 * NW);
  }
  // K split over workgroups as well (one-wave tiles)
  const KPlan kp = layer_k_plan(a, bf16, delta, MB, NW, device);
  if (kp.k_slices > 1) {
    e.slice_bytes = one_wave_tiles(a) * passes * kp.k_slices * MB * 16 * 64 * (long long)sizeof(float);
    e.slice_counters = (int)one_wave_tiles(a) * passes * row_groups(bf16, MB);
    if (a.n_cand > 0) e.norm_slots *= kp.k_slices;
  }
  if (a.tail_slices >= 2 && NW == a.wide_nw) {
    const long long tiles = (a.has_base ? job_tiles(a.bj, 32 * NW) : 0) + (long long)job_tiles(a.cj, 32 * NW) * a.tail_cand;
    e.slice_bytes = tiles * passes * a.tail_slices * NW * MB * 16 * 64 * (long long)sizeof(float);
    e.slice_counters = (int)tiles * passes * row_groups(bf16, MB);
    e.norm_slots = a.tail_p_off - a.p_off + job_tiles(a.cj, 32 * NW) * a.tail_slices;   // both ranges, counted from p_off
  }
  return e;
}

// One-wave workgroups (k_waves of them sharing a tile) that fit on a compute unit by their LDS.
static int one_wave_residents(bool bf16, bool delta, int MB, int k_waves) {
  auto pick = [&](auto mb) {
    constexpr int M = decltype(mb)::value;
    return bf16 ? (delta ? Lds<true, true, M, 1>::TOTAL : Lds<true, false, M, 1>::TOTAL)
                : (delta ? Lds<false, true, M < 4 ? M : 2, 1>::TOTAL : Lds<false, false, M < 4 ? M : 2, 1>::TOTAL);
  };
  const int lds = MB == 1 ? pick(std::integral_constant<int, 1>{}) : MB == 2 ? pick(std::integral_constant<int, 2>{})
                                                                              : pick(std::integral_constant<int, 4>{});
  const int n = 160 * 1024 / (lds * k_waves);
  return n < 1 ? 1 : n;
}

// 128-feature tiles of a launch.
static long long wide_tiles(const LayerArgs& a) {
  return (a.has_base ? job_tiles(a.bj, 128) : 0) + (long long)job_tiles(a.cj, 128) * a.n_cand;
}

// Most K slices a launch of four-wave workgroups may be cut into: every slice keeps two chunks of every job, and the hand-over
// buffers hold all tiles.  0: the launch never takes such workgroups by layer_wide_plan.  No device is asked.
int layer_wide_most(const LayerArgs& a, bool bf16, bool delta, int MB, size_t budget) {
  if (a.n_cand <= 0 || a.cj.N <= 64 || launch_nw_for(a) == 8) return 0;
  const long long tiles = wide_tiles(a);
  if (a.slice_partials == nullptr || a.slice_counters == nullptr || tiles * row_groups(bf16, MB) > kMaxSliceGroups) return 1;
  const int chunks = a.cj.Kp >> 6, min_chunks = a.has_base && (a.bj.Kp >> 6) < chunks ? a.bj.Kp >> 6 : chunks;
  const long long by_bytes = (long long)(budget / wide_slice_bytes(MB)) / tiles;
  const long long most = min_chunks / 2 < 8 ? min_chunks / 2 : 8;
  return most > by_bytes ? (by_bytes < 1 ? 1 : (int)by_bytes) : most < 1 ? 1 : (int)most;
}

// Would a candidate launch that is too small for wide workgroups be slower as one-wave tiles than as four-wave workgroups in
// `slices` K slices, which take `cost` chunk times (see layer_wide_plan)?
// One wave per tile with K split over the waves of a workgroup copies the activations once per 32 features and holds so much
// LDS for it that a compute unit runs one to four such workgroups; but it hands nothing over through memory, and as long as
// its workgroups are resident all at once it is the faster of the two.  Measured on 3692 random launches (K 64 to 4096, 66 to
// 2048 features, 3 to 100 candidates; time as one-wave tiles / as four-wave workgroups, geometric mean, and how many of the latter
// are more than 3 % slower; by the rule as a whole 1.43, 27 of 832).  The float32 ones among them ran wide workgroups on float32
// matrix instructions.  With split operands, score and update of 350 models of one to three layers over buffers in turn, the launch
// the one way and the other: what the rule takes to four waves 1.22 (6 of 101 slower), what it leaves to one 0.94 (four waves
// more than 3 % faster on 67 of 249):
//  * K split over waves, all resident at once: 0.93, 999 of 1473; more than one round of them: 1.44, 33 of 642.
//    Two waves are few for a compute unit: where no more fit and the tile is not cut into K slices either, more than half a round is
//    enough from 16 chunks on (1.41, 5 of 70).
//  * No split (a K of the launch is short): a quarter of a round or less, or at most 20 MB of activations copied in all: 1.03, 393
//    of 1313; beyond both: 1.22, 13 of 264.  And, where only the pass at x has a short K, if the slices take less than 0.8 of the
//    chunks that a one-wave tile walks: 1.52, none of 21.
//  * Not where K is split over waves and the pass at x has more than twice the candidates' chunks: it sets the pace, and four waves
//    of one-wave tiles walk its K in parallel (27 launches: 1.03, 10 of them slower, by up to 44 %: 512 -> 1630, 8 candidates,
//    fp32: 30 -> 54 us; 37 without the split: 1.20, 3 slower).
//  * Layers without the second product in bf16, which wait for memory either way, only for four row blocks, or two beyond 1.25
//    rounds (the others: 1.10, 8 of 49).
static bool one_wave_tiles_slower(const LayerArgs& a, bool bf16, bool delta, int MB, int slices, double cost) {
  const int chunks = a.cj.Kp >> 6, base_chunks = a.has_base ? a.bj.Kp >> 6 : 0;
  const long long base_tiles = a.has_base ? job_tiles(a.bj, 32) : 0, cand_tiles = (long long)job_tiles(a.cj, 32) * a.n_cand;
  if (!bf16 && MB == 4) {
    // Two groups of two row blocks (row_groups): with the second product always (1.41, 2 of 24); without it from 16 chunks on or where
    // the one-wave tiles of one group outnumber the compute units (1.24, none of 17; the others 0.97, 14 of 44 more than 3 % faster).
    return delta || (base_chunks <= 2 * chunks && (chunks >= 16 || base_tiles + cand_tiles > compute_units()));
  }
  KPlan one = layer_k_plan(a, bf16, delta, MB, 1, true);
  // the lines below were measured with K split over waves where every job of the launch gives each wave two chunks
  if (chunks < 2 * one.k_waves || (a.has_base && base_chunks < 2 * one.k_waves)) one.k_waves = 1;
  if (one.k_waves > 1 && base_chunks > 2 * chunks) return false;
  const long long workgroups = (base_tiles + cand_tiles) * one.k_slices;
  const long long round = (long long)compute_units() * one_wave_residents(bf16, delta, MB, one.k_waves);
  if (bf16 && !delta && MB < 4) return MB == 2 && one.k_waves > 1 && 4 * workgroups > 5 * round;
  if (one.k_waves == 2 && one.k_slices == 1 && chunks >= 16) return true;
  if (one.k_waves > 1) return workgroups > round;
  if (slices >= 2 && cost < 0.8 * chunks / one.k_slices) return true;
  const long long chunk_bytes = MB * 32LL * 64 * (bf16 ? 2 : 4) * (delta ? 2 : 1);
  return 4 * workgroups > round && (cand_tiles * chunks + base_tiles * base_chunks) * chunk_bytes > 20000000;
}

// Does a launch of four-wave workgroups stream its rows on the shifted column grid, which its slices do not have?
static bool on_shifted_grid(const LayerArgs& a, bool bf16) { return bf16 && !launch_lines_aligned(a) && launch_ring_kind(a) != 0; }

// Candidate launches with too few 256-feature tiles for eight-wave workgroups.
// Fewer 128-feature tiles than compute units (one-wave tiles otherwise): four-wave workgroups, all tiles (and those of
// the pass at x, if it rides along) cut into as many K slices as cost least by the count
//     rounds x (chunks of a slice + hand-over if sliced),   rounds = workgroups per compute unit, rounded up,
// in chunk times, the hand-over of the partial accumulators being 4 of them, 6 in bf16 without the second product, whose chunks
// are the shortest (113 launches with four row blocks: 1.35 and 1.37 times as fast as one-wave tiles with 4 and 6).
// Measured (us; slices 1 / 2 / 3 / 4, before): bf16, n_r = 128, m = 33: 1001 -> 777 (234 tiles) 41 / 63 / 72 / 80, 88; 777 -> 333
// with the second product (100 tiles) 41 / 37 / 49 / 49, 57.  fp32, n_r = 32, m = 20: 3072 -> 512 (81 tiles) 35 in three slices.
// With split operands, score and update of 60 models each whose launch it changes: 6 chunk times instead of 4 take 1.15 times as long, 2
// 0.95 times.
// More of them (whole four-wave tiles otherwise): three slices where the candidates fill more than one round of compute units and
// all tiles at most 4/3, which the slices make four full rounds of a third, for K from 28 chunks on.  Random launches, whole /
// sliced: in bf16 without the second product, which waits for memory either way, 1.02 (20 of 64 more than 3 % slower); on the
// shifted grid, which slices do not have, 0.93 (5 of 10).  Split operands, score and update: with one product 1.07 (none of 14; from 12
// chunks on 0.99, 2 of 11), with the second 1.12 (none of 31; from 12 chunks on 1.04, 2 of 21); beyond 4/3 rounds 1.03 (none of 10).
// Layers of at most 64 features keep the one-wave tiles (half a workgroup or more would be idle), and so do launches that
// are faster on them (one_wave_tiles_slower) or make no half round of workgroups this way.
// Returns the slices (1: none) or 0 where the launch keeps its shape; budget: bytes for the partial accumulators.
int layer_wide_plan(const LayerArgs& a, bool bf16, bool delta, int MB, size_t budget) {
  const int most = layer_wide_most(a, bf16, delta, MB, budget);
  if (most == 0) return 0;
  const bool whole_tiles = launch_nw_for(a) == 4;
  const long long tiles = wide_tiles(a);
  const int n_cu = compute_units(), chunks = a.cj.Kp >> 6;
  const double hand_over = bf16 && !delta ? 6.0 : 4.0;
  if (whole_tiles) {
    const bool last_round_empty = (long long)job_tiles(a.cj, 128) * a.n_cand > n_cu && 3 * tiles <= 4 * n_cu;
    return last_round_empty && chunks >= 28 && most >= 3 && (delta || !bf16) && !on_shifted_grid(a, bf16) ? 3 : 0;
  }
  int best = 1;
  double best_cost = 0.0;
  for (int S = 1; S <= most; ++S) {
    const double cost = (double)((tiles * S + n_cu - 1) / n_cu) * ((double)chunks / S + (S > 1 ? hand_over : 0.0));
    if (S == 1 || cost < best_cost) {
      best = S;
      best_cost = cost;
    }
  }
  return 2 * tiles * best < n_cu || !one_wave_tiles_slower(a, bf16, delta, MB, best, best_cost) ? 0 : best;
}

// Sliced tail of a candidate launch of eight-wave workgroups.  When the workgroups of the launch do not fill their
// last round of resident slots, the candidates of that round (and the pass at x, if the launch carries it) are cut
// into K slices, as many as bring their workgroups to about one round: the round then lasts a fraction of a whole
// tile's time, and the slices start as soon as slots free up behind the whole tiles.  Workload 4's 2048-wide layers
// (100 candidates x 8 tiles = 3.125 rounds of 256): candidates 96..99 and the pass at x are 40 tiles, cut six ways.
int layer_tail_slices(const LayerArgs& a, bool bf16, bool delta, int MB, int* n_main_out) {
  *n_main_out = a.n_cand;
  if (a.n_cand <= 0 || launch_nw_for(a) != 8 || a.slice_partials == nullptr || a.slice_counters == nullptr) return 0;
  // Float32 layers with the second product and four row blocks keep whole tiles of four waves: eight-wave workgroups with the tail
  // are faster for a long K only (score and update of 20 models, whole / tail: 32 chunks 1.05 to 1.11, 16 1.03 to 1.06, 8 0.94 to 1.02).
  if (!bf16 && delta && MB == 4) return 0;
  const long long slots = (long long)compute_units() * wgs_per_cu(bf16, delta, MB, 8);
  const int groups = row_groups(bf16, MB);
  const int tiles8 = job_tiles(a.cj, 256) * groups;
  const long long full = (long long)tiles8 * a.n_cand / slots * slots;
  const int n_main = (int)(full / tiles8), rest = a.n_cand - n_main;
  // (candidates that fill their rounds exactly leave the pass at x to a launch of its own: as a sliced tail of 16
  // tiles x 8 slices behind workload 5's 4096-wide layers it took 60 us, twice what the launch of one-wave tiles
  // with K split over waves and workgroups takes; with four row blocks the hand-over alone is seven round trips)
  if (n_main <= 0 || rest <= 0 || full % tiles8 != 0) return 0;
  const long long tail_tiles = (long long)rest * tiles8 + (a.has_base ? job_tiles(a.bj, 256) * groups : 0);
  int min_chunks = a.cj.Kp >> 6;
  if (a.has_base && (a.bj.Kp >> 6) < min_chunks) min_chunks = a.bj.Kp >> 6;
  long long S = slots / tail_tiles;
  if (S > kMaxTailWorkgroups / tail_tiles) S = kMaxTailWorkgroups / tail_tiles;
  if (S > min_chunks / 4) S = min_chunks / 4;
  if (S > 8) S = 8;
  if (S < 2) return 0;
  *n_main_out = n_main;
  return (int)S;
}

int layer_tiles(const LayerArgs& a, bool bf16, bool delta, int MB) {
  const int NW = nw_for(a, bf16, delta, MB);
  const int tail = a.tail_slices >= 2 ? job_tiles(a.cj, 32 * NW) * a.tail_slices : 0;
  if (tail > 0 && a.tail_cand == a.n_cand) return tail;
  return job_tiles(a.cj, 32 * NW) * layer_k_plan(a, bf16, delta, MB, NW, true).k_slices + tail;
}

// Should the pass at x (a.bj) ride in the candidates' launch?  Workgroups run in
// rounds of (compute units x resident workgroups); the extra workgroups are free
// when they fit into the last round and cost a whole extra round when the
// candidates fill their rounds exactly, unless there are many rounds anyway.
bool layer_merge_pays(const LayerArgs& a, bool bf16, bool delta, int MB) {
  if (a.n_cand <= 0) return true;
  const int n_cu = compute_units();
  const int NW = nw_for(a, bf16, delta, MB);
  const int per_cu = wgs_per_cu(bf16, delta, MB, NW);
  const long long slots = (long long)n_cu * per_cu;
  const int groups = row_groups(bf16, MB);
  const long long cand = (long long)job_tiles(a.cj, 32 * NW) * a.n_cand * groups;
  const long long base = job_tiles(a.bj, 32 * NW) * groups;
  const long long rounds_without = (cand + slots - 1) / slots, rounds_with = (cand + base + slots - 1) / slots;
  return rounds_with == rounds_without || rounds_without >= 8;
}

hipError_t launch_pack_features(const float* features, int n_r, int K, int Kp, int n_pad, bool bf16, void* tiled,
                                unsigned int* counters, int n_counters, double* zero, long long n_zero,
                                hipStream_t stream) {
  const long long total = (long long)n_pad * Kp;
  const int grid = (int)((total + 255) / 256 > 4096 ? 4096 : (total + 255) / 256);
  if (bf16) {
    hipLaunchKernelGGL(pack_features_kernel<true>, dim3(grid), dim3(256), 0, stream, features, n_r, K, Kp, n_pad, tiled,
                       counters, n_counters, zero, n_zero);
  } else {
    hipLaunchKernelGGL(pack_features_kernel<false>, dim3(grid), dim3(256), 0, stream, features, n_r, K, Kp, n_pad, tiled,
                       counters, n_counters, zero, n_zero);
  }
  return hipGetLastError();
}

hipError_t launch_layer(const LayerArgs& a, bool bf16, bool delta, int MB, hipStream_t stream, LaunchShape* shape) {
  const int NW = nw_for(a, bf16, delta, MB);
  LayerArgs b = a;
  const int groups = row_groups(bf16, MB);
  b.row_groups = groups * launch_passes(a);
  // Packed rows, one row block, one product and four-wave workgroups for at least four fifths of the compute units but at most one each
  // keep the float32 matrix instructions: a wave has its SIMD to itself, without a second one whose products hide the split of its
  // operand.  Score and update of models of one and two layers over buffers in turn, split / float32 products: there 1.00 (30 of them,
  // 0.97 to 1.03; 3072 -> 512 -> 10, 20 candidates 88.7 / 86.9 us), with fewer workgroups 0.99 (20), with line-aligned rows, whose
  // loads arrive sooner, 0.98 (30).
  if (!bf16 && !delta && MB == 1 && NW == 4 && a.n_cand > 0 && !launch_lines_aligned(a)) {
    const long long wgs = wide_tiles(a) * (a.tail_slices >= 2 && a.tail_cand == a.n_cand ? a.tail_slices : 1);
    b.float_products = wgs <= compute_units() && 5 * wgs >= 4LL * compute_units();
  }
  const KPlan kp = layer_k_plan(a, bf16, delta, MB, NW, true);
  b.k_waves = kp.k_waves;
  b.k_slices = kp.k_slices;
  b.slice_group0 = (a.has_base && a.n_cand > 0) ? job_tiles(a.bj, 32) * b.row_groups : 0;
  MB /= groups;
  if (bf16) {
    return delta ? launch_layer_bf16_delta(b, MB, NW, stream, shape) : launch_layer_bf16_first(b, MB, NW, stream, shape);
  }
  return delta ? launch_layer_f32_delta(b, MB, NW, stream, shape) : launch_layer_f32_first(b, MB, NW, stream, shape);
}

}  // namespace zeno
