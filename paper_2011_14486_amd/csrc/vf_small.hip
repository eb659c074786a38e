// Small MLPs (hidden layers of up to 128 units) in one launch (gfx950).
//
// The whole network fits the LDS, so a workgroup stages the weights once and then walks over its
// candidates; every wave takes candidates of its own through all layers and never waits for another
// one.  Between two layers nothing moves: the accumulator of a product holds, for a lane's own column,
// rows that the B operand of the next product wants from exactly this lane, only in another order
// inside a k-step, and that order is free as long as the weights are packed to match
// (pack_k_bf16, and the rows as they come for fp32).  bf16 runs on 32x32x16 products, fp32 on
// 16x16x4 products, whose sums stay in fp32.
//
// 64-128-128-1 through vf_score, one launch and the scan (before: a workgroup per 128 candidates with
// two barriers per layer and the weights out of L2 for bf16; layer after layer through memory, on the
// vector ALU, for fp32): bf16 200,003 vectors 102 -> 32 us, a million 447 -> 83 us (3.2 TB/s of inputs);
// fp32 192,000 vectors 286 -> 90 us, a million 1889 -> 454 us (109 TFLOP/s of the 154 that a large fp32
// matrix product reaches).  Where the network does not fit (a hidden layer of more than 128 units:
// the activations' registers; more than 150 KB of weights) the kernels of vf_score.hip run.
#include "vf_internal.h"

namespace {

#include "vf_sched_dev.h"

#include "vf_score_dev.h"

#include "vf_chain_dev.h"

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef int32_t intx2 __attribute__((ext_vector_type(2), aligned(4)));  // 8-byte loads and stores of 4-byte aligned pairs
typedef float floatx2 __attribute__((ext_vector_type(2), aligned(4)));

constexpr int SMALL_MAX = 128;        // widest hidden layer
constexpr int SMALL_LDS = 150 * 1024; // weights and biases
constexpr int GEN_LDS = 124 * 1024;   // the same where every wave has a decision's context next to them

// Input row (within a k-step of 16) of element e of lane half h: as they come for the first layer,
// in the order of the accumulator's rows for the others.
__device__ __forceinline__ int pack_k_bf16(bool first, int h, int e) { return first ? 8 * h + e : (e < 4 ? 4 * h + e : 4 + 4 * h + e); }

// out[tile][kstep][lane][e] = W[tile * 32 + lane % 32][kstep * 16 + pack_k_bf16(lane / 32, e)], zeros in the padding
__global__ __launch_bounds__(256) void k_pack_small_bf16(const float *W, int N, int K, int ntiles, int ksteps, int first,
                                                         uint16_t *out) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= ntiles * ksteps * 512) return;
  const int e = i & 7, lane = (i >> 3) & 63, s = (i >> 9) % ksteps, tile = (i >> 9) / ksteps;
  const int row = tile * 32 + (lane & 31), k = s * 16 + pack_k_bf16(first != 0, lane >> 5, e);
  out[i] = row < N && k < K ? (uint16_t)bf16_bits(W[(size_t)row * K + k]) : (uint16_t)0;
}

// out[tile][kgroup][lane][e] = W[tile * 16 + lane % 16][kgroup * 16 + 4 (lane / 16) + e], zeros in the padding
__global__ __launch_bounds__(256) void k_pack_small_f32(const float *W, int N, int K, int ntiles, int groups, float *out) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= ntiles * groups * 256) return;
  const int e = i & 3, lane = (i >> 2) & 63, g = (i >> 8) % groups, tile = (i >> 8) / groups;
  const int row = tile * 16 + (lane & 15), k = g * 16 + 4 * (lane >> 4) + e;
  out[i] = row < N && k < K ? W[(size_t)row * K + k] : 0.0f;
}

__global__ __launch_bounds__(256) void k_pad_f32(const float *src, int n, int npad, float *dst) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < npad) dst[i] = i < n ? src[i] : 0.0f;
}

// A unit is one partial minimum: `spp` sub-tiles of candidates in a row, taken by one wave.
struct SmallArgs {
  vf_small_dev md;
  const int32_t *x;
  int64_t prob_stride, M, ld;
  int use_valid_row;
  float *scores;      // nullable
  int64_t ld_scores;
  float *pval;
  int32_t *pidx;
  int nparts, units, spp;
  int xcd_bits, run;  // see first_unit
  NoiseArgs na;
  // GEN: the decisions' contexts; the ids of a decision in blocks of `block`, dealt out to `nparts` shares
  // (share c has the blocks c, c + nparts, ...: valid ids come in runs), one share at a time per wave
  const uint32_t *decpack;
  int block, nblocks;
};

// What a kernel scores: given features, the valid ids that its waves collect, ids as they come, or ids as they
// come through a whole schedule (vf_chain_dev.h).  GIVEN_ONE: given features and one minimum over all of them.
enum { GIVEN = 0, COLLECTED = 1, IDS = 2, CHAINED = 3, GIVEN_ONE = 4 };

// What two of them need besides.  (In arguments of their own: in those of every form, 816 bytes instead of 584,
// they cost scoring with a minimum per group 0.7 %, 192,000 vectors 64-128-128-1 fp32 89.8 / 89.2 us.)
struct SmallOneArgs : SmallArgs {
  unsigned long long *words;  // of one_minimum, and the bound of its wait
  unsigned int wait_rounds;
  int32_t *one_idx;           // the results, nullable
  float *one_val;
};
struct SmallChainArgs : SmallArgs {
  ChainArgs ca;
  int spw;                    // a tile is `spw` sub-tiles in a row, one each for the first waves of a workgroup
};
template <int MODE> struct small_args { typedef SmallArgs type; };
template <> struct small_args<GIVEN_ONE> { typedef SmallOneArgs type; };
template <> struct small_args<CHAINED> { typedef SmallChainArgs type; };
__device__ __forceinline__ ChainArgs chain_of(const SmallArgs &) { return ChainArgs(); }
__device__ __forceinline__ const ChainArgs &chain_of(const SmallChainArgs &a) { return a.ca; }

// GEN: the candidates are enumerated and featurized where they are scored (x is not used); scores of
// ids that are not valid candidates read +inf.  Every wave keeps the context of its problem, looks its ids
// over a block at a time - their digits and the validity rules, a lane each - and collects the valid
// ones until a sub-tile is full, so that the network runs on valid candidates only (a third of the ids, as a
// rule).  64-128-128-1 fp32, 6000 ids, per schedule of two decisions: 64 problems 413 -> 285 us, 16: 160 -> 102;
// 256-96-64-1 bf16, one decision of 4096 ids: 200 problems 91 -> 69 us, 37: 31 -> 25.
// A share of one block of a sub-tile's ids has nothing to collect: the ids go on as they come (IDS), and the
// evaluation itself tells the valid ones (6000 ids, one problem: 57.2 us by way of the queue, 55.6 without; two
// problems 59.1 / 57.7; one problem in bf16 42.9 / 41.9).
struct WaveDec {
  DecPack pk;
  EvalTabs tabs;
  uint32_t queue[128];  // valid ids, ascending: fewer than a sub-tile, and one block more
};
__device__ __forceinline__ void load_wave_dec(WaveDec &wd, const uint32_t *decpack, int p, int lane) {
  uint32_t *const dst = reinterpret_cast<uint32_t *>(&wd.pk);
#pragma unroll
  for (int i = 0; i < (VF_DECPACK_DWORDS + 63) / 64; ++i)
    if (i * 64 + lane < VF_DECPACK_DWORDS) dst[i * 64 + lane] = decpack[(size_t)p * VF_DECPACK_DWORDS + i * 64 + lane];
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  fill_evaltabs_at(wd.tabs, wd.pk.d, wd.pk.sp, lane, 64);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}
// Goes on through the share's blocks (blk: the next one) until `want` valid ids are queued or there are
// no more blocks; masked ids' scores are written.  All lanes call it.
__device__ __forceinline__ void fill_queue(WaveDec &wd, const SmallArgs &a, int p, int &blk, int &queued, int want, int lane) {
  while (queued < want && blk < a.nblocks) {
    const int64_t n0 = (int64_t)blk * a.block, to = n0 + a.block < a.M ? n0 + a.block : a.M;
    const bool in = n0 + lane < to;
    bool valid = in && !range_closed(wd.pk.d, wd.pk.sp, (uint32_t)n0, (uint32_t)to);
    if (valid)
      valid = eval_digits<false>(wd.pk.d, wd.pk.sp, digits_small(wd.pk.sp, (uint32_t)(n0 + lane)), nullptr, nullptr);
    if (a.scores && in && !valid) a.scores[(size_t)p * a.ld_scores + n0 + lane] = __builtin_inff();
    const unsigned long long m = __ballot(valid);
    if (valid) wd.queue[queued + __popcll(m & ((1ull << lane) - 1ull))] = (uint32_t)(n0 + lane);
    queued += __popcll(m);
    blk += a.nparts;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}
// Takes the first `n` ids off the queue.
__device__ __forceinline__ void drop_queue(WaveDec &wd, int &queued, int n, int lane) {
  queued -= n;
  const uint32_t id = lane < queued ? wd.queue[n + lane] : 0u;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  if (lane < queued) wd.queue[lane] = id;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}
// value `lane group` of four (or two) registers, without indexing them
__device__ __forceinline__ int32_t pick(int g, int32_t a, int32_t b) { return g ? b : a; }
__device__ __forceinline__ int32_t pick(int g, int32_t a, int32_t b, int32_t c, int32_t d) {
  return g & 2 ? (g & 1 ? d : c) : (g & 1 ? b : a);
}

__device__ __forceinline__ NoiseArgs noise_of(const SmallArgs &a, bool chain, int stage) {
  NoiseArgs na = a.na;
  if (chain) na.stage = stage;
  return na;
}
// (CHAINED) The first minimum of a workgroup's tile from its waves' (v, c), to the other workgroups.
__device__ __forceinline__ void post_tile(const ChainArgs &ca, unsigned long long *slots, float *tile_v, int32_t *tile_c, int stage,
                                          int tile, float v, int32_t c, int lane, int w) {
  wave_min(v, c);
  if (lane == 0) {
    tile_v[w] = v;
    tile_c[w] = c;
  }
  __syncthreads();
  if (w == 0) {
    v = tile_v[lane & 7];
    c = tile_c[lane & 7];
    wave_min(v, c);
    if (lane == 0)
      __hip_atomic_store(&slots[(size_t)stage * ca.ntiles + tile], word_of(v, c), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// The first minimum over all candidates from the waves' (v, c), in the launch that scores them: every workgroup
// leaves its own in a word past the caches (value and id; a word that is not zero is complete), and the last
// workgroup waits for all of them, reduces them and leaves zeros for the next launch.  (The others wait for
// nothing, so every word comes.  Counting the arrivals, so that nobody waits, costs 4 us with 256 workgroups: atomics on
// one word.)  A launch of its own for it / this: 64-128-128-1 bf16, 200,003 vectors 27.0 / 24.0 us, 20,000: 13.4 / 10.4,
// fp32, 192,000: 90.7 / 87.4; 64-32-1 bf16, 1,000,000: 48.1 / 44.0.
// The wait is bounded all the same: behind `wait_rounds` the last workgroup marks the words that are missing as
// taken, leaves what it has in a word of its own and goes; those that find their word taken put theirs there all the
// same, and the last of them (words[0] counts) does the reduction.  Words of workgroup b: words[1 + b].
constexpr unsigned long long WORD_TAKEN = 0xfffffffeull;  // (ids are below 2^30)
__device__ __forceinline__ void take_word(unsigned long long *words, int q, unsigned long long word, float &v, int32_t &c) {
  const uint32_t id = (uint32_t)word;
  if (id == 0u) return;
  __hip_atomic_store(&words[1 + q], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  take_min(v, c, __uint_as_float((uint32_t)(word >> 32)), id == 0xffffffffu ? -1 : (int32_t)id - 1);
}
__device__ __forceinline__ void one_minimum(unsigned long long *words, unsigned int wait_rounds, int32_t *one_idx, float *one_val, float v,
                                            int32_t c) {
  __shared__ float wave_v[8];
  __shared__ int32_t wave_c[8];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, last = (int)gridDim.x - 1;
  wave_min(v, c);
  if (lane == 0) { wave_v[w] = v; wave_c[w] = c; }
  __syncthreads();
  if (w != 0) return;
  v = wave_v[lane & 7];
  c = wave_c[lane & 7];
  wave_min(v, c);
  int late = -1;       // lane 0: words still to come behind this workgroup's own; 0: the reduction is its
  bool handed = true;  // and all that there is to reduce is in the words
  if ((int)blockIdx.x != last) {
    if (lane == 0) {
      unsigned long long was = 0ull;
      const unsigned long long mine = word_of(v, c);
      if (!__hip_atomic_compare_exchange_strong(&words[1 + blockIdx.x], &was, mine, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT) &&
          was == WORD_TAKEN) {
        __hip_atomic_store(&words[1 + blockIdx.x], mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        late = (int)__hip_atomic_fetch_add(&words[0], ~0ull, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) - 1;
      }
    }
  } else {
    unsigned int rounds = 0;
    int q0 = 0;
    for (bool all = true; q0 < last; q0 += 256) {
      unsigned long long word[4] = {0ull, 0ull, 0ull, 0ull};
      for (;;) {
        bool lack = false;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int q = q0 + 64 * k + lane;
          if (q < last && word[k] == 0ull) word[k] = __hip_atomic_load(&words[1 + q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) lack = lack || (q0 + 64 * k + lane < last && word[k] == 0ull);
        all = __ballot(lack) == 0ull;
        if (all || rounds++ >= wait_rounds) break;
        __builtin_amdgcn_s_sleep(1);
      }
      if (!all) break;
#pragma unroll
      for (int k = 0; k < 4; ++k) take_word(words, q0 + 64 * k + lane, word[k], v, c);
    }
    handed = q0 < last;
    if (!handed) late = 0;
    else {
      // (what has been taken so far is in v and c, and those words are zero again)
      wave_min(v, c);
      int n = 0;
      for (int q = q0 + lane; q < last; q += 64) {
        unsigned long long was = 0ull;
        n += __hip_atomic_compare_exchange_strong(&words[1 + q], &was, WORD_TAKEN, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT) ? 1 : 0;
      }
      for (int off = 32; off > 0; off >>= 1) n += __shfl_xor(n, off);
      if (lane == 0) {
        __hip_atomic_store(&words[1 + last], word_of(v, c), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        late = (int)__hip_atomic_fetch_add(&words[0], (unsigned long long)n, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) + n;
      }
    }
  }
  if (__builtin_amdgcn_readfirstlane(late) != 0) return;
  if (handed) {
    v = __builtin_inff();
    c = -1;
    for (int q = lane; q <= last; q += 64)
      take_word(words, q, __hip_atomic_load(&words[1 + q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), v, c);
  }
  wave_min(v, c);
  if (lane == 0) {
    if (one_idx) one_idx[0] = c;
    if (one_val) one_val[0] = v;
  }
}

__device__ __forceinline__ void stage_small(const SmallArgs &a, uint4 *wl, float *bl) {
#pragma unroll 4
  for (int i = threadIdx.x; i < a.md.nw; i += 512) wl[i] = a.md.w[i];
  for (int i = threadIdx.x; i < a.md.nbias; i += 512) bl[i] = a.md.bias[i];
  __syncthreads();
}

// The units of a wave: the returned one, then every gridDim.x * 8 >> xcd_bits -th up to `end`.  Workgroups are
// dealt out to the eight XCDs in turn; xcd_bits = 3 gives each XCD a run of units.
// Given features: the columns of neighbouring units share cache lines wherever the rows do not begin
// on one, and with neighbours on different XCDs those lines are fetched twice.  Neighbours dealt out / in
// runs, odd numbers of vectors: 64-128-128-1 bf16, 200,003: 32.8 / 29.0 us; 64-32-1 bf16, 500,003: 44.1 / 34.4;
// 256-128-128-128-1 bf16, 200,003: 76.2 / 61.5; rows that begin on a line, and fp32 networks: the same to 1 %.
// (One set of vectors over and over, part of which the last cache keeps.  Out of memory, 16, 8 and 6 sets in
// turn, a gigabyte together: 32.2 / 29.5, 40.3 / 36.3, 78.4 / 69.7.)
__device__ __forceinline__ int first_unit(const SmallArgs &a, int w, int &end) {
  const int q = (int)blockIdx.x >> a.xcd_bits, x = (int)blockIdx.x - (q << a.xcd_bits), from = x * a.run;
  end = from + a.run < a.units ? from + a.run : a.units;
  return from + q + ((int)gridDim.x >> a.xcd_bits) * w;
}

// ROWS rows of raw values of a lane: N consecutive ones of every row, the rows `ld` apart, and
// `skip` more between row SPLIT - 1 and row SPLIT.  Whole sub-tiles take a row in one load; otherwise
// only the `left` values that there are get loaded.  (One address at a time: the scheduler would
// work them all out first and fill the registers with them.)
template <int ROWS, int SPLIT, int N>
__device__ __forceinline__ void load_raw(int32_t (&r)[ROWS][N], const int32_t *p, int64_t ld, int64_t skip, int left, bool whole) {
  if (whole) {
#pragma unroll
    for (int e = 0; e < ROWS; ++e) {
      if (N == 2) {
        const intx2 v = *reinterpret_cast<const intx2 *>(p);
        r[e][0] = v[0];
        r[e][N - 1] = v[1];
      } else {
        r[e][0] = p[0];
      }
      p += e + 1 == SPLIT ? ld + skip : ld;
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
#pragma unroll
    for (int e = 0; e < ROWS; ++e) {
#pragma unroll
      for (int c = 0; c < N; ++c) r[e][c] = c < left ? p[c] : 0;
      p += e + 1 == SPLIT ? ld + skip : ld;
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// 32 * CT candidates per sub-tile, lane l has columns CT (l % 32) + 0 .. CT - 1.  The matrix products
// of a sub-tile of 64 (64-128-128-1: 100 of them, 3200 cycles) and the conversion of its inputs cost
// about the same; two waves per SIMD overlap one's with the other's, and the next 32 input rows are
// always under way.
template <int CT, int NT, int MODE>
__global__ __launch_bounds__(512) void k_small_bf16(typename small_args<MODE>::type a) {
  constexpr bool ONE = MODE == GIVEN_ONE, GEN = MODE != GIVEN && !ONE, DIRECT = MODE == IDS, CHAIN = MODE == CHAINED;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  uint4 *const wl = reinterpret_cast<uint4 *>(smem);
  float *const bl = reinterpret_cast<float *>(wl + a.md.nw);
  WaveDec &wd = reinterpret_cast<WaveDec *>(bl + (a.md.nbias + 3) / 4 * 4)[threadIdx.x >> 6];  // (GEN only)
  const ChainArgs &ca = chain_of(a);
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  stage_small(a, wl, bl);
  const int L = a.md.L, K0 = a.md.dims[0], chunks = K0 / 32;
  floatx16 zero;
#pragma unroll
  for (int j = 0; j < 16; ++j) zero[j] = 0.0f;
  auto mfma = [](uint4 x, uint4 y, floatx16 z) __attribute__((always_inline)) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), z, 0, 0, 0);
  };
  // (Rows that fill the row tiles up have zero weights.  On an infinite activation their products are
  // NaN with the sign bit set, 0xffc00000, of which the ReLU on the bits makes 0 again.)
  // plus bias, rounded to bf16, ReLU on the pairs: half a row tile of the accumulator as the B operand
  // of a k-step.  (The bias as the products' first addend would be less work, but the sums would be
  // less exact: 4.1e-5 instead of 3.3e-5 off a 64-bit sum in the scores of 64-128-128-1.)
  auto frag = [&](const floatx16 &v, int l, int t, int s2, int at) __attribute__((always_inline)) {
    const float *bb = bl + a.md.boff[l] + t * 32 + 16 * s2 + 4 * (at >> 5);
    const float4 p = *reinterpret_cast<const float4 *>(bb), q = *reinterpret_cast<const float4 *>(bb + 8);
    uint4 b;
    b.x = relu_bf16x2(pack_bf16(v[8 * s2 + 0] + p.x, v[8 * s2 + 1] + p.y));
    b.y = relu_bf16x2(pack_bf16(v[8 * s2 + 2] + p.z, v[8 * s2 + 3] + p.w));
    b.z = relu_bf16x2(pack_bf16(v[8 * s2 + 4] + q.x, v[8 * s2 + 5] + q.y));
    b.w = relu_bf16x2(pack_bf16(v[8 * s2 + 6] + q.z, v[8 * s2 + 7] + q.w));
    return b;
  };
  int32_t raw[16][CT];  // 32 input rows: per k-step eight rows of the lane half; column
  auto fetch = [&](int p, int64_t n0, int ch) __attribute__((always_inline)) {
    const int32_t *row = a.x + (size_t)p * a.prob_stride + n0 + (size_t)(ch * 32 + 8 * h) * a.ld;
    const int left = (int)(a.M - n0 < 32 * CT ? a.M - n0 : 32 * CT) - CT * (lane & 31);
    load_raw<16, 8, CT>(raw, row + CT * (lane & 31), a.ld, 8 * a.ld, left, n0 + 32 * CT <= a.M);
  };
  // (GEN: a unit is a share of a problem's ids)
  const int stride = ((int)gridDim.x >> a.xcd_bits) * 8;
  int u_end = 0, u = CHAIN ? 0 : first_unit(a, w, u_end), sub = 0;
  const bool idle = ONE && u >= u_end;
  if (!CHAIN && !ONE && u >= u_end) return;
  int p = CHAIN ? (int)blockIdx.x % ca.nprob : u / a.nparts, part = CHAIN ? 0 : u - p * a.nparts;
  int64_t n0 = GEN ? 0 : (int64_t)part * a.spp * 32 * CT;
  int blk = part, queued = 0;  // (GEN)
  // (CHAINED)
  __shared__ ChainShared sh;
  __shared__ float tile_v[8];
  __shared__ int32_t tile_c[8];
  const int member = CHAIN ? (int)blockIdx.x / ca.nprob : 0;
  const size_t row = (size_t)p * ca.t.S;
  unsigned long long *const slots = CHAIN ? ca.slots + row * ca.ntiles : nullptr;
  unsigned int *const claims = CHAIN ? ca.claims + (size_t)p * (ca.t.S + 1) : nullptr;
  int cur = 1, stage = ca.first - 1, tile = ca.ntiles;
  unsigned int c_next = NO_CLAIM;
  int32_t pre = 0;
  if constexpr (CHAIN) chain_begin(sh, ca, row, member, threadIdx.x);
  else if constexpr (GEN) load_wave_dec(wd, a.decpack, p, lane);
  else if (!idle) fetch(p, n0, 0);
  float v = __builtin_inff();
  int32_t vc = -1;
  for (; !idle;) {
    // the sub-tile after this one
    int nu = u, nsub = sub + 1, np = p, npart = part;
    int64_t nn0 = n0 + 32 * CT;
    bool ends = nsub >= a.spp || nn0 >= a.M;
    if (!GEN && ends) {
      nu = u + stride;
      nsub = 0;
      np = nu / a.nparts;
      npart = nu - np * a.nparts;
      nn0 = (int64_t)npart * a.spp * 32 * CT;
    }
    int have = 0;  // (GEN) candidates of this sub-tile
    if constexpr (CHAIN) {
      while (tile >= ca.ntiles)
        if (!chain_between(sh, ca, slots, claims, p, row, member, cur, stage, tile, c_next, pre, threadIdx.x)) {
          chain_leave(sh, ca, slots, claims, p, ca.ntiles, threadIdx.x);
          return;
        }
      n0 = ((int64_t)tile * a.spw + w) * (32 * CT);
      have = w < a.spw && n0 < a.M ? (int)(a.M - n0 < 32 * CT ? a.M - n0 : 32 * CT) : 0;
      nu = u;
    } else if constexpr (GEN) {
      if constexpr (DIRECT) {
        n0 = (int64_t)blk * (32 * CT);
        have = (int)(a.M - n0 < 32 * CT ? a.M - n0 : 32 * CT);
        blk += a.nparts;
        ends = blk >= a.nblocks;
      } else {
        fill_queue(wd, a, p, blk, queued, 32 * CT, lane);
        have = queued < 32 * CT ? queued : 32 * CT;
        ends = blk >= a.nblocks && queued == have;
      }
      nu = ends ? u + stride : u;
    }
    const bool more = CHAIN || nu < u_end;
    if (!more) { np = p; nn0 = n0; }
    // (the weights and biases that a sub-tile starts with are read afresh from LDS for every one: kept
    // across the sub-tiles they would fill the registers)
    int at = lane;
    asm volatile("" : "+v"(at));
    bool ok[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) ok[c] = GEN ? CT * (lane & 31) + c < have : n0 + CT * (lane & 31) + c < a.M;
    uint32_t id[CT];  // (GEN)
    if constexpr (GEN) {
#pragma unroll
      for (int c = 0; c < CT; ++c)
        id[c] = !ok[c] ? 0u : DIRECT || CHAIN ? (uint32_t)n0 + CT * (lane & 31) + c : wd.queue[CT * (lane & 31) + c];
    }
    uint4 own[GEN ? 4 : 1][CT];  // (GEN) the candidates' rows 0..63, as the k-steps 0..3 want them
    // (GEN) no candidate in the share, or in the block
    const DecPack &kc = CHAIN ? sh.pks[cur] : wd.pk;
    const EvalTabs &tc = CHAIN ? sh.tabs : wd.tabs;
    const bool closed = GEN && (DIRECT || CHAIN ? have == 0 || range_closed(kc.d, kc.sp, (uint32_t)n0, (uint32_t)(n0 + have)) : have == 0);
    uint32_t dig[CT];  // (CHAINED) the digits of the ids
    if constexpr (GEN) {
      if (!closed) {
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          int32_t core[64];
          const Digits dg = digits_small(kc.sp, id[c]);
          const bool valid = eval_digits<true>(kc.d, kc.sp, dg, &tc, core);  // (behind the last one too: core must be defined)
          dig[c] = pack_digits(dg);
          ok[c] = ok[c] && valid;
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            float f[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) f[e] = plog2_dev(pick(h, core[16 * s + e], core[16 * s + 8 + e]));
            own[s][c] = make_uint4(pack_bf16(f[0], f[1]), pack_bf16(f[2], f[3]), pack_bf16(f[4], f[5]), pack_bf16(f[6], f[7]));
          }
        }
      }
    }
    floatx16 acc[NT][CT];
    if (!closed) {
    // ---- first layer (a network without a hidden layer has one row tile there: its output vector)
    const int ks0 = a.md.kst[0];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int c = 0; c < CT; ++c) acc[t][c] = zero;
    // (a weight fragment is refilled in place behind its last product; the refill behind the last
    // k-step reads into what follows the layer's weights and is not used)
    const uint4 *wp = wl + at;
    uint4 x[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) x[t] = wp[t * ks0 * 64];
    auto products = [&](const uint4 (&in)[2][CT]) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        wp += 64;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
          for (int c = 0; c < CT; ++c) acc[t][c] = mfma(x[t], in[s][c], acc[t][c]);
          x[t] = wp[t * ks0 * 64];
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    if constexpr (GEN) {
#pragma unroll
      for (int ch = 0; ch < 2; ++ch) {
        uint4 in[2][CT];
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int c = 0; c < CT; ++c) in[s][c] = own[2 * ch + s][c];
        products(in);
      }
    }
    for (int ch = GEN ? 2 : 0; ch < chunks; ++ch) {
      uint4 in[2][CT];
      if constexpr (GEN) {
        // rows 64..255, the same for all candidates of the decision (DecPack::stat holds them as pairs)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const uint32_t *nb = kc.stat + 16 + (ch * 32 - 64 + 16 * s + 8 * h) / 2;
          const uint4 q = make_uint4(nb[0], nb[1], nb[2], nb[3]);
#pragma unroll
          for (int c = 0; c < CT; ++c) in[s][c] = q;
        }
        products(in);
        continue;
      }
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          uint4 q;
          q.x = pack_bf16(plog2_dev(raw[8 * s + 0][c]), plog2_dev(raw[8 * s + 1][c]));
          q.y = pack_bf16(plog2_dev(raw[8 * s + 2][c]), plog2_dev(raw[8 * s + 3][c]));
          q.z = pack_bf16(plog2_dev(raw[8 * s + 4][c]), plog2_dev(raw[8 * s + 5][c]));
          q.w = pack_bf16(plog2_dev(raw[8 * s + 6][c]), plog2_dev(raw[8 * s + 7][c]));
          in[s][c] = q;
          // row 16 is the validity flag (lane half 0; only its columns are scanned)
          if (s == 1 && ch == 0 && a.use_valid_row) ok[c] = ok[c] && raw[8][c] != 0;
        }
      const bool onward = ch + 1 == chunks;  // (behind the last sub-tile of all: the same one once more)
      fetch(onward ? np : p, onward ? nn0 : n0, onward ? 0 : ch + 1);
      products(in);
    }
    // ---- the other hidden layers, two row tiles at a time (all of them at once would not leave
    // registers for the input rows under way), then the output vector as a row tile with one row
    if (L > 1) {
      uint4 act[2 * NT][CT];
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          act[2 * t][c] = frag(acc[t][c], 0, t, 0, at);
          act[2 * t + 1][c] = frag(acc[t][c], 0, t, 1, at);
        }
      for (int l = 1; l < L - 1; ++l) {
        constexpr int TH = NT < 2 ? NT : 2;
        uint4 out[2 * NT][CT];
#pragma unroll
        for (int t0 = 0; t0 < NT; t0 += TH) {
          floatx16 part[TH][CT];
          wp = wl + a.md.woff[l] + at;
#pragma unroll
          for (int t = 0; t < TH; ++t)
            if (t0 + t < NT) {
#pragma unroll
              for (int c = 0; c < CT; ++c) part[t][c] = zero;
              x[t] = wp[(t0 + t) * 2 * NT * 64];
            }
#pragma unroll
          for (int s = 0; s < 2 * NT; ++s)
#pragma unroll
            for (int t = 0; t < TH; ++t)
              if (t0 + t < NT) {
#pragma unroll
                for (int c = 0; c < CT; ++c) part[t][c] = mfma(x[t], act[s][c], part[t][c]);
                if (s + 1 < 2 * NT) x[t] = wp[((t0 + t) * 2 * NT + s + 1) * 64];
                __builtin_amdgcn_sched_barrier(0);
              }
#pragma unroll
          for (int t = 0; t < TH; ++t)
            if (t0 + t < NT) {
#pragma unroll
              for (int c = 0; c < CT; ++c) {
                out[2 * (t0 + t)][c] = frag(part[t][c], l, t0 + t, 0, at);
                out[2 * (t0 + t) + 1][c] = frag(part[t][c], l, t0 + t, 1, at);
              }
            }
        }
#pragma unroll
        for (int s = 0; s < 2 * NT; ++s)
#pragma unroll
          for (int c = 0; c < CT; ++c) act[s][c] = out[s][c];
      }
      wp = wl + a.md.woff[L - 1] + at;
#pragma unroll
      for (int c = 0; c < CT; ++c) acc[0][c] = zero;
#pragma unroll
      for (int s = 0; s < 2 * NT; ++s) {
        const uint4 y = wp[s * 64];
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[0][c] = mfma(y, act[s][c], acc[0][c]);
      }
    }
    }  // (not closed)
    // ---- row 0 of the last product (element 0 of lanes 0..31) is the score
    {
      float s[CT];
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        s[c] = closed ? __builtin_inff() : acc[0][c][0] + bl[a.md.boff[L - 1]];
        if (GEN && (closed || !ok[c])) { s[c] = __builtin_inff(); ok[c] = false; }
      }
      const int64_t n = n0 + CT * (lane & 31);
      if (lane < 32) {
        if (GEN) {
#pragma unroll
          for (int c = 0; c < CT; ++c)
            if (a.scores && CT * (lane & 31) + c < have) a.scores[(size_t)p * a.ld_scores + id[c]] = s[c];
        } else if (a.scores) {
          float *dst = a.scores + (size_t)p * a.ld_scores + n;
          if (CT == 2 && n + 1 < a.M) {
            *reinterpret_cast<floatx2 *>(dst) = floatx2{s[0], s[CT - 1]};
          } else {
#pragma unroll
            for (int c = 0; c < CT; ++c)
              if (n + c < a.M) dst[c] = s[c];
          }
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          float sc = s[c];
          const int32_t at_id = GEN ? (int32_t)id[c] : (int32_t)(n + c);
          if (a.na.eps != 0.0f) sc = add_noise(noise_of(a, CHAIN, stage), sc, p, at_id);
          if (ok[c] && sc < v) { v = sc; vc = CHAIN ? (int32_t)dig[c] : at_id; }
        }
      }
      if constexpr (CHAIN) {
        post_tile(ca, slots, tile_v, tile_c, stage, tile, v, vc, lane, w);
        tile = ca.ntiles;
        v = __builtin_inff();
        vc = -1;
        continue;
      }
      if (!ONE && ends) {
        wave_min(v, vc);
        if (lane == 0) {
          a.pval[u] = v;
          a.pidx[u] = vc;
        }
        v = __builtin_inff();
        vc = -1;
      }
    }
    if (!more) break;
    if constexpr (GEN) {
      if constexpr (!DIRECT) drop_queue(wd, queued, have, lane);
      if (ends) {
        np = nu / a.nparts;
        blk = nu - np * a.nparts;
        if (np != p) load_wave_dec(wd, a.decpack, np, lane);
      }
      u = nu; p = np;
      continue;
    }
    u = nu; sub = nsub; p = np; part = npart; n0 = nn0;
  }
  if constexpr (ONE) one_minimum(a.words, a.wait_rounds, a.one_idx, a.one_val, v, vc);
}

// 16 * CT candidates per sub-tile, lane l has columns CT (l % 16) + 0 .. CT - 1 and rows 4 (l / 16) + 0..3
// of every 16.  The output vector is a dot product on the vector ALU (a sixteenth of a row tile
// would be used), the four lane groups' parts added at the end.
// Every 32 rows of a product are summed by themselves and the sums added up, in both forms: sums of
// few terms are the more exact ones (scores of 64-128-128-1 off a 64-bit sum, relative: 1.5e-7; 2.0e-7
// when two columns per lane had one sum each and 192,000 vectors took 88 instead of 90 us), and a
// candidate's score does not depend on how many candidates the call has.
template <int CT, int NT, int MODE>
__global__ __launch_bounds__(512) void k_small_f32(typename small_args<MODE>::type a) {
  constexpr bool ONE = MODE == GIVEN_ONE, GEN = MODE != GIVEN && !ONE, DIRECT = MODE == IDS, CHAIN = MODE == CHAINED;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  uint4 *const wl = reinterpret_cast<uint4 *>(smem);
  const floatx4 *const wf = reinterpret_cast<const floatx4 *>(smem);
  float *const bl = reinterpret_cast<float *>(wl + a.md.nw);
  WaveDec &wd = reinterpret_cast<WaveDec *>(bl + (a.md.nbias + 3) / 4 * 4)[threadIdx.x >> 6];  // (GEN only)
  const ChainArgs &ca = chain_of(a);
  const int lane = threadIdx.x & 63, q = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  stage_small(a, wl, bl);
  const int L = a.md.L, K0 = a.md.dims[0], groups0 = a.md.kst[0], chunks = groups0 / 2;
  int32_t raw[8][CT];  // 32 input rows: per group of 16 four rows of the lane group; column
  auto fetch = [&](int p, int64_t n0, int ch) __attribute__((always_inline)) {
    const int32_t *col = a.x + (size_t)p * a.prob_stride + n0 + CT * (lane & 15);
    const int left = (int)(a.M - n0 < 16 * CT ? a.M - n0 : 16 * CT) - CT * (lane & 15);
    if (ch * 32 + 32 <= K0) {
      load_raw<8, 4, CT>(raw, col + (size_t)(ch * 32 + 4 * q) * a.ld, a.ld, 12 * a.ld, left, n0 + 16 * CT <= a.M);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int r = ch * 32 + (e >> 2) * 16 + 4 * q + (e & 3);
        // (a row past the last one has zero weights: any row will do, its values are finite)
#pragma unroll
        for (int c = 0; c < CT; ++c) raw[e][c] = c < left ? col[(r < K0 ? r : 0) * a.ld + c] : 0;
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // (GEN: a unit is a share of a problem's ids)
  const int stride = ((int)gridDim.x >> a.xcd_bits) * 8;
  int u_end = 0, u = CHAIN ? 0 : first_unit(a, w, u_end), sub = 0;
  const bool idle = ONE && u >= u_end;
  if (!CHAIN && !ONE && u >= u_end) return;
  int p = CHAIN ? (int)blockIdx.x % ca.nprob : u / a.nparts, part = CHAIN ? 0 : u - p * a.nparts;
  int64_t n0 = GEN ? 0 : (int64_t)part * a.spp * 16 * CT;
  int blk = part, queued = 0;  // (GEN)
  // (CHAINED)
  __shared__ ChainShared sh;
  __shared__ float tile_v[8];
  __shared__ int32_t tile_c[8];
  const int member = CHAIN ? (int)blockIdx.x / ca.nprob : 0;
  const size_t row = (size_t)p * ca.t.S;
  unsigned long long *const slots = CHAIN ? ca.slots + row * ca.ntiles : nullptr;
  unsigned int *const claims = CHAIN ? ca.claims + (size_t)p * (ca.t.S + 1) : nullptr;
  int cur = 1, stage = ca.first - 1, tile = ca.ntiles;
  unsigned int c_next = NO_CLAIM;
  int32_t pre = 0;
  if constexpr (CHAIN) chain_begin(sh, ca, row, member, threadIdx.x);
  else if constexpr (GEN) load_wave_dec(wd, a.decpack, p, lane);
  else if (!idle) fetch(p, n0, 0);
  float v = __builtin_inff();
  int32_t vc = -1;
  for (; !idle;) {
    int nu = u, nsub = sub + 1, np = p, npart = part;
    int64_t nn0 = n0 + 16 * CT;
    bool ends = nsub >= a.spp || nn0 >= a.M;
    if (!GEN && ends) {
      nu = u + stride;
      nsub = 0;
      np = nu / a.nparts;
      npart = nu - np * a.nparts;
      nn0 = (int64_t)npart * a.spp * 16 * CT;
    }
    int have = 0;  // (GEN) candidates of this sub-tile
    if constexpr (CHAIN) {
      while (tile >= ca.ntiles)
        if (!chain_between(sh, ca, slots, claims, p, row, member, cur, stage, tile, c_next, pre, threadIdx.x)) {
          chain_leave(sh, ca, slots, claims, p, ca.ntiles, threadIdx.x);
          return;
        }
      n0 = ((int64_t)tile * a.spw + w) * (16 * CT);
      have = w < a.spw && n0 < a.M ? (int)(a.M - n0 < 16 * CT ? a.M - n0 : 16 * CT) : 0;
      nu = u;
    } else if constexpr (GEN) {
      if constexpr (DIRECT) {
        n0 = (int64_t)blk * (16 * CT);
        have = (int)(a.M - n0 < 16 * CT ? a.M - n0 : 16 * CT);
        blk += a.nparts;
        ends = blk >= a.nblocks;
      } else {
        fill_queue(wd, a, p, blk, queued, 16 * CT, lane);
        have = queued < 16 * CT ? queued : 16 * CT;
        ends = blk >= a.nblocks && queued == have;
      }
      nu = ends ? u + stride : u;
    }
    const bool more = CHAIN || nu < u_end;
    if (!more) { np = p; nn0 = n0; }
    // (the weights and biases that a sub-tile starts with are read afresh from LDS for every one: kept
    // across the sub-tiles they would fill the registers)
    int at = lane;
    asm volatile("" : "+v"(at));
    bool ok[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) ok[c] = GEN ? CT * (lane & 15) + c < have : n0 + CT * (lane & 15) + c < a.M;
    uint32_t id[CT];  // (GEN)
    if constexpr (GEN) {
#pragma unroll
      for (int c = 0; c < CT; ++c)
        id[c] = !ok[c] ? 0u : DIRECT || CHAIN ? (uint32_t)n0 + CT * (lane & 15) + c : wd.queue[CT * (lane & 15) + c];
    }
    float own[GEN ? 4 : 1][4][CT];  // (GEN) the candidates' rows 0..63: group of 16, row of the lane group, column
    // (GEN) no candidate in the share, or in the block
    const DecPack &kc = CHAIN ? sh.pks[cur] : wd.pk;
    const EvalTabs &tc = CHAIN ? sh.tabs : wd.tabs;
    const bool closed = GEN && (DIRECT || CHAIN ? have == 0 || range_closed(kc.d, kc.sp, (uint32_t)n0, (uint32_t)(n0 + have)) : have == 0);
    uint32_t dig[CT];  // (CHAINED) the digits of the ids
    if constexpr (GEN) {
      if (!closed) {
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          int32_t core[64];
          const Digits dg = digits_small(kc.sp, id[c]);
          const bool valid = eval_digits<true>(kc.d, kc.sp, dg, &tc, core);  // (behind the last one too: core must be defined)
          dig[c] = pack_digits(dg);
          ok[c] = ok[c] && valid;
#pragma unroll
          for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              own[g][e][c] = plog2_dev(pick(q, core[16 * g + e], core[16 * g + 4 + e], core[16 * g + 8 + e], core[16 * g + 12 + e]));
        }
      }
    }
    floatx4 acc[NT][CT];
    float s[CT];
    const bool only = L == 1;  // no hidden layer: the inputs go straight into the output dot
#pragma unroll
    for (int c = 0; c < CT; ++c) s[c] = 0.0f;
    if (!closed) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int c = 0; c < CT; ++c) acc[t][c] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    // (a weight fragment is refilled in place behind its last product; the refills behind the last
    // 32 rows read the next tiles' weights and are not used)
    constexpr int TH = NT / 2;  // fragments in flight: row tile by row tile, both groups of 16 rows
    floatx4 x[TH];
#pragma unroll
    for (int i = 0; i < TH; ++i) x[i] = only ? floatx4{0.0f, 0.0f, 0.0f, 0.0f} : wf[(i / 2 * groups0 + i % 2) * 64 + at];
    auto products = [&](const float (&in)[2][4][CT], int ch) __attribute__((always_inline)) {
      if (only) {
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          const floatx4 y = *reinterpret_cast<const floatx4 *>(bl + a.md.wl_off + (ch * 2 + g) * 16 + 4 * (at >> 4));
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int c = 0; c < CT; ++c) s[c] = fmaf(y[e], in[g][e][c], s[c]);
        }
        return;
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        floatx4 part[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) part[c] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          const int i = 2 * t + g, n = (i + TH) % (2 * NT), nch = i + TH < 2 * NT ? ch : ch + 1;
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int c = 0; c < CT; ++c) part[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i % TH][e], in[g][e][c], part[c], 0, 0, 0);
          x[i % TH] = wf[(n / 2 * groups0 + 2 * nch + n % 2) * 64 + at];
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[t][c] += part[c];
      }
    };
    if constexpr (GEN) {
#pragma unroll
      for (int ch = 0; ch < 2; ++ch) {
        float in[2][4][CT];
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int c = 0; c < CT; ++c) in[g][e][c] = own[2 * ch + g][e][c];
        products(in, ch);
      }
    }
    for (int ch = GEN ? 2 : 0; ch < chunks; ++ch) {
      float in[2][4][CT];
      if constexpr (GEN) {
        // rows 64..255, the same for all candidates of the decision
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float f = plog2_dev(kc.d.nb[ch * 32 - 64 + 16 * g + 4 * q + e]);
#pragma unroll
            for (int c = 0; c < CT; ++c) in[g][e][c] = f;
          }
        products(in, ch);
        continue;
      }
#pragma unroll
      for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int c = 0; c < CT; ++c) in[g][e][c] = plog2_dev(raw[4 * g + e][c]);
      if (ch == 0 && a.use_valid_row) {
#pragma unroll
        for (int c = 0; c < CT; ++c) ok[c] = ok[c] && raw[4][c] != 0;
      }
      const bool onward = ch + 1 == chunks;  // (behind the last sub-tile of all: the same one once more)
      fetch(onward ? np : p, onward ? nn0 : n0, onward ? 0 : ch + 1);
      products(in, ch);
    }
    if (!only) {
      // a finished layer: bias, ReLU, and its rows are the next one's inputs as they lie
      auto finish = [&](const floatx4 &v, int l, int t) __attribute__((always_inline)) {
        const floatx4 b = *reinterpret_cast<const floatx4 *>(bl + a.md.boff[l] + t * 16 + 4 * (at >> 4));
        floatx4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = relu_keep_nan(v[e] + b[e]);
        return o;
      };
      floatx4 act[NT][CT];
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c) act[t][c] = finish(acc[t][c], 0, t);
      for (int l = 1; l < L - 1; ++l) {
        // a row tile at a time, its weights one behind the other
        floatx4 out[NT][CT];
        const floatx4 *wp = wf + a.md.woff[l] + at;
#pragma unroll
        for (int i = 0; i < TH; ++i) x[i] = wp[i * 64];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          floatx4 part[CT], tot[CT];
#pragma unroll
          for (int kg = 0; kg < NT; ++kg) {
            const int i = t * NT + kg;
            if (kg % 2 == 0) {
#pragma unroll
              for (int c = 0; c < CT; ++c) part[c] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
              for (int c = 0; c < CT; ++c) part[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i % TH][e], act[kg][c][e], part[c], 0, 0, 0);
            if (i + TH < NT * NT) x[i % TH] = wp[(i + TH) * 64];
            if (kg % 2 == 1) {
#pragma unroll
              for (int c = 0; c < CT; ++c) tot[c] = kg == 1 ? part[c] : tot[c] + part[c];
            }
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int c = 0; c < CT; ++c) out[t][c] = finish(tot[c], l, t);
          // (the rows that fill the tiles up behind the layer's own stay 0: zero weights on an infinite
          // activation have made them NaN)
          const int rows = a.md.dims[l + 1] - 16 * t;
          if (rows < 16) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (4 * (at >> 4) + e >= rows) {
#pragma unroll
                for (int c = 0; c < CT; ++c) out[t][c][e] = 0.0f;
              }
          }
        }
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int c = 0; c < CT; ++c) act[t][c] = out[t][c];
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const floatx4 y = *reinterpret_cast<const floatx4 *>(bl + a.md.wl_off + t * 16 + 4 * (at >> 4));
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int c = 0; c < CT; ++c) s[c] = fmaf(y[e], act[t][c][e], s[c]);
      }
    }
    }  // (not closed)
    const float bout = bl[a.md.boff[L - 1]];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      s[c] += __shfl_xor(s[c], 16);
      s[c] += __shfl_xor(s[c], 32);
      s[c] += bout;
      if (GEN && (closed || !ok[c])) { s[c] = __builtin_inff(); ok[c] = false; }
    }
    const int64_t n = n0 + CT * (lane & 15);
    if (lane < 16) {
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        const int32_t at_id = GEN ? (int32_t)id[c] : (int32_t)(n + c);
        if (a.scores && (GEN ? CT * (lane & 15) + c < have : n + c < a.M)) a.scores[(size_t)p * a.ld_scores + at_id] = s[c];
        float sc = s[c];
        if (a.na.eps != 0.0f) sc = add_noise(noise_of(a, CHAIN, stage), sc, p, at_id);
        if (ok[c] && sc < v) { v = sc; vc = CHAIN ? (int32_t)dig[c] : at_id; }
      }
    }
    if constexpr (CHAIN) {
      post_tile(ca, slots, tile_v, tile_c, stage, tile, v, vc, lane, w);
      tile = ca.ntiles;
      v = __builtin_inff();
      vc = -1;
      continue;
    }
    if (!ONE && ends) {
      wave_min(v, vc);
      if (lane == 0) {
        a.pval[u] = v;
        a.pidx[u] = vc;
      }
      v = __builtin_inff();
      vc = -1;
    }
    if (!more) break;
    if constexpr (GEN) {
      if constexpr (!DIRECT) drop_queue(wd, queued, have, lane);
      if (ends) {
        np = nu / a.nparts;
        blk = nu - np * a.nparts;
        if (np != p) load_wave_dec(wd, a.decpack, np, lane);
      }
      u = nu; p = np;
      continue;
    }
    u = nu; sub = nsub; p = np; part = npart; n0 = nn0;
  }
  if constexpr (ONE) one_minimum(a.words, a.wait_rounds, a.one_idx, a.one_val, v, vc);
}

}  // namespace

// Packs the model for the kernels above if it is small enough for them (pm.small.w stays null
// otherwise).
int vfk_pack_small(vf_ctx *c, const float *wdev) {
  const vf_model &m = c->model;
  vf_small_dev &d = c->pm.small;
  d = vf_small_dev();
  const int L = m.n_layers;
  const bool bf16 = m.dtype == VF_BF16;
  for (int l = 1; l < L; ++l)
    if (m.dims[l] > SMALL_MAX) return VF_OK;
  size_t nw = 0, nbias = 0;  // 16-byte units, floats
  // every hidden layer gets as many row tiles as the widest one needs (fp32: an even number), the
  // others' filled up with zeros: the kernels' loops then have no conditions
  const int unit = bf16 ? 32 : 16;
  int wide = 1;
  for (int l = 1; l < L; ++l) wide = m.dims[l] > wide ? m.dims[l] : wide;
  d.NT = (wide + 31) / 32 * (32 / unit);
  for (int l = 0; l < L; ++l) {
    const int K = m.dims[l], N = m.dims[l + 1];
    d.dims[l] = K;
    d.nt[l] = l < L - 1 ? d.NT : 1;
    // (fp32: whole chunks of 32 rows)
    d.kst[l] = l > 0 ? d.NT * unit / 16 : bf16 ? (K + 15) / 16 : (K + 31) / 32 * 2;
    d.woff[l] = (int)nw;
    d.boff[l] = (int)nbias;
    if (bf16 || l < L - 1) nw += (size_t)d.nt[l] * d.kst[l] * 64;
    nbias += (size_t)d.nt[l] * unit;
    if ((nw + nbias) * 16 > (size_t)SMALL_LDS * 4) return VF_OK;  // (no overflow of the offsets)
  }
  d.wl_off = (int)nbias;
  if (!bf16) nbias += (size_t)d.kst[L - 1] * 16;
  if (nw * 16 + nbias * 4 > SMALL_LDS) return VF_OK;
  d.L = L;
  d.nw = (int)nw;
  d.nbias = (int)nbias;
  void *buf = nullptr;
  // (and one_minimum's words: with the model, so that they stay where they are until there is another)
  int ncu = 256;
  (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, c->device);
  const size_t words_at = nw * 16 + (nbias * 4 + 15) / 16 * 16;
  const int nwords = 1 + ncu;
  VF_HIP(c, hipMalloc(&buf, words_at + (size_t)nwords * 8));
  c->pm.small_buf = buf;
  float *bias = reinterpret_cast<float *>(reinterpret_cast<uint4 *>(buf) + nw);
  c->pm.small_words = reinterpret_cast<unsigned long long *>(reinterpret_cast<char *>(buf) + words_at);
  c->pm.small_nwords = nwords;
  // (cleared as the padding of what lies in front of them)
  const int tail = (int)(words_at / 4 + 2 * nwords - nw * 4 - nbias);
  size_t off = 0;
  for (int l = 0; l < L; ++l) {
    const int K = m.dims[l], N = m.dims[l + 1];
    const float *W = wdev + off, *b = W + (size_t)K * N;
    const int n = d.nt[l] * d.kst[l] * (bf16 ? 512 : 256);
    if (bf16)
      hipLaunchKernelGGL(k_pack_small_bf16, dim3((n + 255) / 256), dim3(256), 0, c->stream, W, N, K, d.nt[l], d.kst[l],
                         (int)(l == 0),
                         reinterpret_cast<uint16_t *>(reinterpret_cast<uint4 *>(buf) + d.woff[l]));
    else if (l < L - 1)
      hipLaunchKernelGGL(k_pack_small_f32, dim3((n + 255) / 256), dim3(256), 0, c->stream, W, N, K, d.nt[l], d.kst[l],
                         reinterpret_cast<float *>(reinterpret_cast<uint4 *>(buf) + d.woff[l]));
    else
      hipLaunchKernelGGL(k_pad_f32, dim3((d.kst[l] * 16 + tail + 255) / 256), dim3(256), 0, c->stream, W, K, d.kst[l] * 16 + tail,
                         bias + d.wl_off);
    VF_HIP(c, hipGetLastError());
    const int nb = d.nt[l] * unit + (bf16 && l == L - 1 ? tail : 0);
    hipLaunchKernelGGL(k_pad_f32, dim3((nb + 255) / 256), dim3(256), 0, c->stream, b, N, nb, bias + d.boff[l]);
    VF_HIP(c, hipGetLastError());
    off += (size_t)K * N + N;
  }
  d.w = reinterpret_cast<const uint4 *>(buf);
  d.bias = bias;
  return VF_OK;
}

// Whether the search's candidates can be generated in the kernels above.
bool vfk_small_generates(const vf_ctx *c) {
  const vf_small_dev &d = c->pm.small;
  return c->has_model && d.w && c->model.kind == VF_MLP && c->model.dims[0] == c->space.F &&
         (size_t)d.nw * 16 + (size_t)d.nbias * 4 <= GEN_LDS;
}

// Scores on the kernels above.  part_out: candidates per partial minimum, a divisor of 128.  x null: the
// candidates of the decisions whose contexts d_decpack holds are generated (masked scores).
int vfk_score_small(vf_ctx *c, const int32_t *x, int64_t prob_stride, int nprob, int64_t M, int64_t ld, int use_valid_row,
                    float *scores, int64_t ld_scores, int noise_stage, const vf_partbuf *parts, int *nparts_out, int *part_out) {
  const bool bf16 = c->model.dtype == VF_BF16;
  int ncu = 256;
  (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, c->device);
  // sub-tiles of one column per lane while that leaves waves idle otherwise (two waves per SIMD; of ids to be
  // looked over two in five become candidates, as a rule, or more where the space is mostly root-level: all of
  // 2048 ids, 64 problems, 64-96-64-1 bf16, six decisions with one column per lane 178 us, with two 155)
  const int base = bf16 ? 32 : 16;
  const double sure = x ? 1.0 : c->root_share[c->dec_stage], share = sure > 0.4 ? sure : 0.4;
  const int ct = (double)((M + base - 1) / base * nprob) * share <= ncu * 8.0 ? 1 : 2;
  SmallArgs a;
  // a partial minimum per sub-tile, but 128 candidates each for very many (the buffer of
  // vf_score_static holds 65536)
  a.spp = (M + base * ct - 1) / (base * ct) * nprob <= 32768 ? 1 : 128 / (base * ct);
  const int part = base * ct * a.spp;
  a.nparts = (int)((M + part - 1) / part);
  *nparts_out = a.nparts;
  *part_out = part;
  a.block = a.nblocks = 0;
  bool ids = false;
  if (!x) {
    // blocks of 64 ids, of fewer down to a sub-tile's where there would not be two of them per wave; as many
    // shares per problem as there are waves for it, or four where a wave has several problems
    const int64_t waves = (int64_t)ncu * 8;
    // Where nearly all ids are valid looking them over is work for nothing: collected / as they come, six
    // decisions of 2048 ids, 200 problems, all valid 64-128-128-1 fp32 1494 / 1359 us, 64-96-64-1 bf16 389 / 360,
    // 64-32-1 bf16 (seven in eight) 338 / 309; three in four: 1198 / 1357, 340 / 359, 303 / 310.
    ids = sure > 0.8;
    int block = ids ? base * ct : 64;
    while (block > base * ct && (M + block - 1) / block * nprob < 2 * waves) block /= 2;
    a.block = block;
    a.nblocks = (int)((M + block - 1) / block);
    const int64_t each = nprob * 2 > waves ? 4 : waves / nprob;
    a.nparts = each < a.nblocks ? (int)each : a.nblocks;
    ids = ids || (a.nparts == a.nblocks && block == base * ct);
    *nparts_out = a.nparts;
  }
  const int64_t units = (int64_t)a.nparts * nprob;
  if (parts) {
    if ((size_t)units > parts->cap) return VF_EINVAL;
    a.pval = parts->val; a.pidx = parts->idx;
  } else {
    const int rc = vfk_ensure_parts(c, (size_t)(units > 0 ? units : 1));
    if (rc != VF_OK) return rc;
    a.pval = c->d_pval; a.pidx = c->d_pidx;
  }
  if (units == 0) return VF_OK;
  const int grid = units < ncu ? (int)units : ncu;
  const bool one = c->one_wanted && grid < c->pm.small_nwords;
  a.md = c->pm.small;
  a.x = x; a.prob_stride = prob_stride; a.M = M; a.ld = ld; a.use_valid_row = use_valid_row;
  a.scores = scores; a.ld_scores = ld_scores;
  a.units = (int)units;
  a.na.eps = noise_stage >= 0 ? c->noise_eps : 0.0f;
  a.na.k0 = (uint32_t)c->noise_seed; a.na.k1 = (uint32_t)(c->noise_seed >> 32);
  a.na.stage = noise_stage; a.na.first_rollout = c->noise_first;
  a.decpack = c->d_decpack;
  // (a kilobyte more: the last refill of a weight fragment reads behind the weights)
  size_t smem = (size_t)a.md.nw * 16 + (size_t)a.md.nbias * 4 + 1024;
  if (!x) smem = (smem + 15) / 16 * 16 + 8 * sizeof(WaveDec);
#define VF_SMALL(k, ct, mode, n1, n2, n3, n4) {k<ct, n1, mode>, k<ct, n2, mode>, k<ct, n3, mode>, k<ct, n4, mode>}
#define VF_SMALL_ALL(mode)                                                                                  \
  {{VF_SMALL(k_small_bf16, 1, mode, 1, 2, 3, 4), VF_SMALL(k_small_bf16, 2, mode, 1, 2, 3, 4)},              \
   {VF_SMALL(k_small_f32, 1, mode, 2, 4, 6, 8), VF_SMALL(k_small_f32, 2, mode, 2, 4, 6, 8)}}
  static constexpr void (*kerns[3][2][2][4])(SmallArgs) = {VF_SMALL_ALL(GIVEN), VF_SMALL_ALL(COLLECTED), VF_SMALL_ALL(IDS)};
  static constexpr void (*one_kerns[2][2][4])(SmallOneArgs) = VF_SMALL_ALL(GIVEN_ONE);
#undef VF_SMALL_ALL
#undef VF_SMALL
  const int dt = bf16 ? 0 : 1, rt = a.md.NT * base / 32 - 1;
  a.xcd_bits = x && grid % 8 == 0 ? 3 : 0;
  a.run = (int)((units + (1 << a.xcd_bits) - 1) >> a.xcd_bits);
  vf_prof_scope prof(c, VF_PROF_SCORE);
  if (one) {
    SmallOneArgs oa;
    static_cast<SmallArgs &>(oa) = a;
    oa.words = c->pm.small_words;
    oa.wait_rounds = c->wait_rounds;
    oa.one_idx = c->one_idx; oa.one_val = c->one_val;
    const auto kern = one_kerns[dt][ct - 1][rt];
    VF_HIP(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(512), smem, c->stream, oa);
  } else {
    const auto kern = kerns[x ? GIVEN : ids ? IDS : COLLECTED][dt][ct - 1][rt];
    VF_HIP(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(512), smem, c->stream, a);
  }
  VF_HIP(c, hipGetLastError());
  c->one_done = one;
  return VF_OK;
}

// Whole schedules in one launch (CHAINED) while a decision's tiles are one round: a launch per step of a decision
// costs more than the decision.  Launches per layer / one launch, 6000 ids, two layers: 64-128-128-1 fp32, one
// problem 55.9 / 46.6 us, five 69.5 / 60.8, bf16 41.8 / 34.3, 64-96-32-1 bf16, ten problems 46.5 / 35.9; 20 layers of
// 4096 ids, 256-96-64-1 bf16, one problem 393 / 264, 256-64-1, four 371 / 239.  What is left of a decision is a
// chain of small steps (vf_chain.hip) and the products of one sub-tile per SIMD.
// Sub-tiles per workgroup with which all tiles of a decision are on the compute units at once (one wave per SIMD
// if that does), 0: there are too many.
static int small_chain_spw(const vf_ctx *c) {
  if (!vfk_small_generates(c) || c->M < 1) return 0;
  int ncu = 256;
  (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, c->device);
  const int64_t subs = (c->M + (c->model.dtype == VF_BF16 ? 31 : 15)) / (c->model.dtype == VF_BF16 ? 32 : 16);
  for (int spw = 4; spw <= 8; spw += 4)
    if ((subs + spw - 1) / spw * c->B <= ncu) return spw;
  return 0;
}

bool vfk_small_can_chain(const vf_ctx *c) { return small_chain_spw(c) != 0; }

int vfk_small_chain(vf_ctx *c, int first, int last, int32_t *out_states, int32_t *out_cids, float *out_vals) {
  const int spw = small_chain_spw(c);
  if (spw == 0 || first > last) return VF_ESTATE;
  const bool bf16 = c->model.dtype == VF_BF16;
  const int base = bf16 ? 32 : 16;
  SmallChainArgs a = {};
  const int rc = chain_args(c, first, last, (int)((c->M + base * spw - 1) / (base * spw)), out_states, out_cids, out_vals, &a.ca);
  if (rc != VF_OK) return rc;
  a.md = c->pm.small;
  a.M = c->M;
  a.spp = 1;
  a.spw = spw;
  a.na.eps = c->noise_eps;
  a.na.k0 = (uint32_t)c->noise_seed; a.na.k1 = (uint32_t)(c->noise_seed >> 32);
  a.na.stage = first; a.na.first_rollout = c->noise_first;
  const size_t smem = (size_t)a.md.nw * 16 + (size_t)a.md.nbias * 4 + 1024;
  static constexpr void (*kerns[2][4])(SmallChainArgs) = {
      {k_small_bf16<1, 1, CHAINED>, k_small_bf16<1, 2, CHAINED>, k_small_bf16<1, 3, CHAINED>, k_small_bf16<1, 4, CHAINED>},
      {k_small_f32<1, 2, CHAINED>, k_small_f32<1, 4, CHAINED>, k_small_f32<1, 6, CHAINED>, k_small_f32<1, 8, CHAINED>}};
  const auto kern = kerns[bf16 ? 0 : 1][a.md.NT * base / 32 - 1];
  vf_prof_scope prof(c, VF_PROF_SCORE);
  VF_HIP(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
  hipLaunchKernelGGL(kern, dim3((unsigned)(c->B * a.ca.ntiles)), dim3(512), smem, c->stream, a);
  VF_HIP(c, hipGetLastError());
  c->dec_stage = last + 1 < c->S ? last + 1 : -1;
  return VF_OK;
}
