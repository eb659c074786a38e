// The recurrent value network of Sec. 3.2 wired to the search (gfx950).
//
// V reads a state as a sequence with one timestep per stage of the pipeline, in
// scheduling order: a stage that is scheduled in the state gives its 64 core features,
// a stage that is not gives its intrinsic block and zeros; every timestep's hidden
// state goes through the linear head and the predictions are summed.  For the
// candidates of decision i all timesteps before i are the same, so the recurrence over
// the committed prefix is kept per problem (cell state, the fed-back h folded into the
// gate pre-activations of the next step, the head's sum so far) and advanced by one
// step at every commit.  A candidate then costs one cell step on its own features plus
// one step per stage still unscheduled; for those the input part of the gates does not
// depend on the candidate either and comes from a per-problem table.
#include <type_traits>

#include "vf_internal.h"

namespace {

#include "vf_sched_dev.h"
#include "vf_score_dev.h"
#include "vf_layer_dev.h"

// fp32 blob of the model: W_ih[4H][64], W_hh[4H][H], b_ih[4H], b_hh[4H], w_head[H], b_head
struct SeqWeights {
  const float *Wih, *Whh, *bih, *bhh, *wh, *bh;
  int H;
};

__device__ __forceinline__ float wave_sum(float v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// G[b][t][r] = b_ih[r] + b_hh[r] + sum_{k<16} W_ih[r][k] x_k, x = the normalised intrinsic
// block of stage t: the input part of the gates of a stage that is not scheduled yet.
__global__ __launch_bounds__(256) void k_seq_tables(const int32_t *intr, SeqWeights sw, size_t n_bt, float *G) {
  const int H4 = 4 * sw.H;
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n_bt * (size_t)H4) return;
  const size_t bt = i / H4;
  const int r = (int)(i % H4);
  float acc = 0.0f;
#pragma unroll
  for (int k = 0; k < 16; ++k)
    acc = fmaf(bf16_val(sw.Wih[(size_t)r * 64 + k]), bf16_val(plog2_dev(intr[bt * 16 + k])), acc);
  G[i] = acc + sw.bih[r] + sw.bhh[r];
}

// the recurrence before the first stage: h = c = 0, so the gates start from the biases
__global__ __launch_bounds__(256) void k_seq_reset(SeqWeights sw, int B, float *hfb, float *cpre, float *P,
                                                   float *hsum) {
  const int H = sw.H;
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < (size_t)B * H) { hfb[i] = 0.0f; cpre[i] = 0.0f; }
  if (i < (size_t)B * 4 * H) P[i] = sw.bih[i % (4 * H)] + sw.bhh[i % (4 * H)];
  if (i < (size_t)B) hsum[i] = 0.0f;
}

// One cell step per problem on the vector committed for `stage`; then the part of the
// next step's gates that comes from the new h.  A problem whose schedule has ended
// keeps its state (it has no candidates any more).  With sel_idx (beam search) slot b
// of the dst set continues the recurrence of its parent slot sel_idx[b] / Mpad of the
// src set; slots past the sel_n[0] survivors are dead and left alone.
struct SeqState {
  float *hfb, *cpre, *P, *hsum;  // [B][H] (bf16 values), [B][H], [B][4H], [B]
};

constexpr int SEQ_PB = 4;  // problems per workgroup of k_seq_advance: they share the weight reads

// [W_ih | W_hh] transposed and rounded: WT[k][r], k over the 64 inputs then the H hidden
// units, r over the 4H gate rows, so that thread r of a block reads its row coalesced.
__global__ __launch_bounds__(256) void k_pack_seqT(SeqWeights sw, float *WT) {
  const int H = sw.H, H4 = 4 * H;
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (size_t)(64 + H) * H4) return;
  const int k = (int)(i / H4), r = (int)(i % H4);
  WT[i] = bf16_val(k < 64 ? sw.Wih[(size_t)r * 64 + k] : sw.Whh[(size_t)r * H + (k - 64)]);
}

struct SeqAdvance {
  Tables t;
  int stage;
  SeqWeights sw;
  const float *WT;
  SeqState src, dst;
  const int32_t *sel_idx, *sel_n;
  int64_t Mpad;
  int B;
};
struct SeqAdvanceShared {
  float x[SEQ_PB][64], z[SEQ_PB][1024], hn[SEQ_PB][256], hraw[SEQ_PB][256];
  int from_s[SEQ_PB], mode_s[SEQ_PB];  // 0: leave alone, 1: carry the state over, 2: one cell step
};
// A workgroup of 1024: problems b0 .. b0 + SEQ_PB - 1.
__device__ __forceinline__ void seq_advance(const SeqAdvance &a, SeqAdvanceShared &sh, int b0) {
  const Tables &t = a.t;
  const SeqWeights &sw = a.sw;
  const SeqState &src = a.src, &dst = a.dst;
  const float *const WT = a.WT;
  const int32_t *const sel_idx = a.sel_idx, *const sel_n = a.sel_n;
  const int64_t Mpad = a.Mpad;
  const int stage = a.stage, B = a.B;
  auto &x = sh.x;
  auto &z = sh.z;
  auto &hn = sh.hn, &hraw = sh.hraw;
  auto &from_s = sh.from_s, &mode_s = sh.mode_s;
  const int tid = threadIdx.x, lane = tid & 63;
  const int H = sw.H, H4 = 4 * H, S = t.S;
  if (tid < SEQ_PB) {
    const int b = b0 + tid;
    int mode = 0, from = b;
    if (b < B) {
      const bool survivor = !sel_idx || b < sel_n[0];  // beam search: slots past the survivors are dead
      if (survivor) {
        if (sel_idx) from = (int)((int64_t)sel_idx[b] / Mpad);
        const bool live = t.cids[(size_t)b * S + stage] >= 0;
        mode = live ? 2 : (src.cpre != dst.cpre ? 1 : 0);
      }
    }
    from_s[tid] = from;
    mode_s[tid] = mode;
  }
  __syncthreads();
  for (int i = tid; i < SEQ_PB * 64; i += 1024) {
    const int pb = i / 64, k = i % 64;
    x[pb][k] = mode_s[pb] == 2 ? bf16_val(plog2_dev(t.cf[((size_t)(b0 + pb) * S + stage) * 64 + k])) : 0.0f;
  }
  __syncthreads();
  // gate pre-activations: thread r owns row r for the block's problems
  if (tid < H4) {
    float acc[SEQ_PB];
#pragma unroll
    for (int pb = 0; pb < SEQ_PB; ++pb) acc[pb] = 0.0f;
#pragma unroll 16
    for (int k = 0; k < 64; ++k) {
      const float wv = WT[(size_t)k * H4 + tid];
#pragma unroll
      for (int pb = 0; pb < SEQ_PB; ++pb) acc[pb] = fmaf(wv, x[pb][k], acc[pb]);
    }
#pragma unroll
    for (int pb = 0; pb < SEQ_PB; ++pb)
      if (mode_s[pb] == 2) z[pb][tid] = src.P[(size_t)from_s[pb] * H4 + tid] + acc[pb];
  }
  __syncthreads();
  for (int i = tid; i < SEQ_PB * H; i += 1024) {
    const int pb = i / H, u = i % H, b = b0 + pb, from = from_s[pb];
    if (mode_s[pb] == 2) {
      float cn = src.cpre[(size_t)from * H + u];
      const float h = lstm_cell(z[pb][u], z[pb][H + u], z[pb][2 * H + u], z[pb][3 * H + u], cn);
      dst.cpre[(size_t)b * H + u] = cn;
      hraw[pb][u] = h;
      hn[pb][u] = bf16_val(h);
      dst.hfb[(size_t)b * H + u] = hn[pb][u];
    } else if (mode_s[pb] == 1) {
      dst.cpre[(size_t)b * H + u] = src.cpre[(size_t)from * H + u];
      dst.hfb[(size_t)b * H + u] = src.hfb[(size_t)from * H + u];
    }
  }
  __syncthreads();
  // the head's prediction for this timestep: one wave per problem, fixed order
  if (tid < SEQ_PB * 64) {
    const int pb = tid / 64;
    if (mode_s[pb] == 2) {
      float v = 0.0f;
      for (int u = lane; u < H; u += 64) v = fmaf(bf16_val(sw.wh[u]), hraw[pb][u], v);
      v = wave_sum(v);
      if (lane == 0) dst.hsum[b0 + pb] = src.hsum[from_s[pb]] + v + sw.bh[0];
    } else if (mode_s[pb] == 1 && lane == 0) {
      dst.hsum[b0 + pb] = src.hsum[from_s[pb]];
    }
  }
  // the h part of the next step's gates
  if (tid < H4) {
    float acc[SEQ_PB];
#pragma unroll
    for (int pb = 0; pb < SEQ_PB; ++pb) acc[pb] = 0.0f;
#pragma unroll 16
    for (int k = 0; k < H; ++k) {
      const float wv = WT[(size_t)(64 + k) * H4 + tid];
#pragma unroll
      for (int pb = 0; pb < SEQ_PB; ++pb) acc[pb] = fmaf(wv, hn[pb][k], acc[pb]);
    }
    const float bias = sw.bih[tid] + sw.bhh[tid];
#pragma unroll
    for (int pb = 0; pb < SEQ_PB; ++pb) {
      if (mode_s[pb] == 2) dst.P[(size_t)(b0 + pb) * H4 + tid] = bias + acc[pb];
      else if (mode_s[pb] == 1) dst.P[(size_t)(b0 + pb) * H4 + tid] = src.P[(size_t)from_s[pb] * H4 + tid];
    }
  }
}
__global__ __launch_bounds__(1024) void k_seq_advance(SeqAdvance a) {
  __shared__ SeqAdvanceShared sh;
  seq_advance(a, sh, blockIdx.x * SEQ_PB);
}

// The valid candidates of decision (problem b, stage), in ascending id order:
// list[b][0..count[b]).  The recurrent network costs one cell step per remaining stage and
// candidate, so the scoring kernel works on this dense list instead of the id range, where
// valid and invalid ids are interleaved.  Also fills the masked score array (nullable)
// with +inf: the scorer then only writes the candidates' entries.
__global__ __launch_bounds__(1024) void k_seq_compact(const uint32_t *decpack, uint32_t M, int64_t Mpad, int32_t *list,
                                                      int32_t *count, float *scores) {
  __shared__ DecPack pk;
  __shared__ int wsum[16];
  __shared__ int base;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (tid < VF_DECPACK_DWORDS) reinterpret_cast<uint32_t *>(&pk)[tid] = decpack[(size_t)b * VF_DECPACK_DWORDS + tid];
  if (tid == 0) base = 0;
  __syncthreads();
  for (uint32_t c0 = 0; c0 < (uint32_t)Mpad; c0 += 1024u) {
    const uint32_t cid = c0 + tid;
    bool ok = false;
    if (cid < M && !range_closed(pk.d, pk.sp, c0, c0 + 1024u < M ? c0 + 1024u : M)) {
      uint32_t dec;
      ok = eval_candidate<false>(pk.d, pk.sp, cid, dec, nullptr);
    }
    if (scores && cid < (uint32_t)Mpad) scores[(size_t)b * Mpad + cid] = __builtin_inff();
    const unsigned long long m = __ballot(ok);
    if (lane == 0) wsum[w] = __popcll(m);
    __syncthreads();
    int off = base;
    for (int k = 0; k < w; ++k) off += wsum[k];
    if (ok) list[(size_t)b * Mpad + off + __popcll(m & ((1ull << lane) - 1ull))] = (int32_t)cid;
    __syncthreads();
    if (tid == 0) {
      int tot = 0;
      for (int k = 0; k < 16; ++k) tot += wsum[k];
      base += tot;
    }
    __syncthreads();
  }
  if (tid == 0) count[b] = base;
}

struct SeqDev {
  int H, S;
  const uint16_t *w_pack;  // [unit tile][k step][gate][lane][8]; 4 k-steps of x, then H/16 of h
  const float *aux;        // b_ih + b_hh [4H], head vector [H] (bf16 values), head bias
  const float *G;          // [B][S][4H]
  const float *P;          // [B][4H]
  const float *cpre;       // [B][H]
  const float *hsum;       // [B]
  const uint32_t *decpack; // [B][VF_DECPACK_DWORDS]
  const int32_t *list;     // [B][Mpad] valid candidate ids of the decision, ascending
  const int32_t *count;    // [B]
  int64_t Mpad;
  unsigned long long *stat;
};

// Workgroup = NC consecutive entries of the valid-candidate list of decision `stage` of
// problem blockIdx.y: featurize them, one cell step on their features from the problem's prefix state, one
// step per later stage, the head's sum, the tile's first minimum.  Wave w owns hidden
// units 32w..32w+31 (their four gate row tiles); c lives in registers, h goes through
// LDS as bf16, double-buffered; the weight fragments of a step are one contiguous stream
// per wave, kept PD k-steps ahead in a register ring that wraps at the end of the step;
// the per-step gate biases of the problem are staged through LDS one step ahead.
template <int NC, int PD>
__global__ __launch_bounds__(512) void k_seq_step(SeqDev md, int stage, int64_t M, float *scores, int64_t ld_scores,
                                                  float *pval, int32_t *pidx, NoiseArgs na) {
  constexpr int CT = NC / 32;
  constexpr int XLD = 72;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int H = md.H, S = md.S, H4 = 4 * H, hld = H + 8;
  uint16_t *xs = reinterpret_cast<uint16_t *>(smem);                    // [NC][XLD]
  uint16_t *hs = xs + (size_t)NC * XLD;                                 // [2][NC][hld]
  float *gls = reinterpret_cast<float *>(hs + (size_t)2 * NC * hld);    // [2][4H]
  float *red = gls + 2 * H4;                                            // [8][NC]
  float *whs = red + 8 * NC;                                            // [H]
  int32_t *okf = reinterpret_cast<int32_t *>(whs + H);                  // [NC]
  int32_t *cids = okf + NC;                                             // [NC] candidate id of each column
  __shared__ DecPack pk;

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.y, nparts = gridDim.x;
  const int64_t n0 = (int64_t)blockIdx.x * NC;
  const size_t slot = (size_t)b * nparts + blockIdx.x;

  if (tid < VF_DECPACK_DWORDS)
    reinterpret_cast<uint32_t *>(&pk)[tid] = md.decpack[(size_t)b * VF_DECPACK_DWORDS + tid];
  __syncthreads();

  const int nvalid = md.count[b];
  if (n0 >= nvalid) {
    // past the end of the list: nothing for the network to do
    if (tid == 0) {
      pval[slot] = __builtin_inff();
      pidx[slot] = -1;
    }
    return;
  }
  // four threads per candidate, each producing 16 of the 64 core rows
  if (tid < NC) cids[tid] = (n0 + tid) < nvalid ? md.list[(size_t)b * md.Mpad + n0 + tid] : -1;
  if (tid < 4 * NC) {
    const int n = tid % NC, part = tid / NC;
    const bool inb = (n0 + n) < nvalid;
    const uint32_t cid = inb ? (uint32_t)md.list[(size_t)b * md.Mpad + n0 + n] : 0u;
    int32_t core[64];
    uint32_t dec;
    // the parts a thread does not store are dead code in its copy of the evaluation
    auto put = [&](const int32_t *v, int row0) {
      uint4 q0, q1;
      q0.x = pack_bf16(plog2_dev(v[0]), plog2_dev(v[1]));
      q0.y = pack_bf16(plog2_dev(v[2]), plog2_dev(v[3]));
      q0.z = pack_bf16(plog2_dev(v[4]), plog2_dev(v[5]));
      q0.w = pack_bf16(plog2_dev(v[6]), plog2_dev(v[7]));
      q1.x = pack_bf16(plog2_dev(v[8]), plog2_dev(v[9]));
      q1.y = pack_bf16(plog2_dev(v[10]), plog2_dev(v[11]));
      q1.z = pack_bf16(plog2_dev(v[12]), plog2_dev(v[13]));
      q1.w = pack_bf16(plog2_dev(v[14]), plog2_dev(v[15]));
      if (!inb) q0 = q1 = make_uint4(0u, 0u, 0u, 0u);
      uint4 *dst = reinterpret_cast<uint4 *>(xs + (size_t)n * XLD + row0);
      dst[0] = q0;
      dst[1] = q1;
    };
    if (part == 0) {
      // evaluated for padding columns too: core must be defined before put reads it
      const bool okc = eval_candidate<true>(pk.d, pk.sp, cid, dec, core);
      okf[n] = inb && okc;
      put(core, 0);
    } else if (part == 1) {
      eval_candidate<true>(pk.d, pk.sp, cid, dec, core);
      put(core + 16, 16);
    } else if (part == 2) {
      eval_candidate<true>(pk.d, pk.sp, cid, dec, core);
      put(core + 32, 32);
    } else {
      eval_candidate<true>(pk.d, pk.sp, cid, dec, core);
      put(core + 48, 48);
    }
  }

  const bool active = w < H / 32;
  const int wu = active ? w : 0;  // idle waves shadow tile 0 but never store
  const int ksh = H / 16, ksteps = 4 + ksh;
  // the wave's weight stream (4 k-steps of x part, then the h part): base in scalar registers,
  // 16 bytes per lane, fragment i at byte 1024 i
  const __amdgpu_buffer_rsrc_t ws = stream_rsrc(reinterpret_cast<const uint4 *>(md.w_pack) + (size_t)wu * ksteps * 4 * 64);
  const int voff = 16 * lane;
  int wstep = PD;  // the k-step of the stream that refills the next slot
  uint4 ring[PD][4];
#pragma unroll
  for (int j = 0; j < PD; ++j)
#pragma unroll
    for (int g = 0; g < 4; ++g) ring[j][g] = stream_load(ws, voff, j * 4 + g);

  for (int i = tid; i < H4; i += 512) gls[i] = md.P[(size_t)b * H4 + i];
  for (int i = tid; i < H; i += 512) whs[i] = md.aux[H4 + i];
  floatx16 cst[CT];
  float vsum[CT];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 cv = *reinterpret_cast<const float4 *>(md.cpre + (size_t)b * H + wu * 32 + 4 * (lane >> 5) + 8 * q);
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      cst[c][4 * q + 0] = cv.x; cst[c][4 * q + 1] = cv.y;
      cst[c][4 * q + 2] = cv.z; cst[c][4 * q + 3] = cv.w;
    }
  }
#pragma unroll
  for (int c = 0; c < CT; ++c) vsum[c] = 0.0f;
  __syncthreads();

  const int rowoff = (lane & 31), koff = 8 * (lane >> 5);
  for (int t = stage; t < S; ++t) {
    const int k = t - stage;
    // the next step's biases, fetched now, parked in LDS after this step's contraction
    const bool fetch_g = (t + 1 < S) && tid < H;
    float4 gnext = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (fetch_g) gnext = reinterpret_cast<const float4 *>(md.G + ((size_t)b * S + t + 1) * H4)[tid];

    // the step's gate biases (staged in LDS one step ahead) are the addends of the first k-step:
    // gate by gate, so that one bias vector is in registers at a time
    const float *bias = gls + (size_t)(k & 1) * H4;
    floatx16 acc[4][CT];

    if (active) {  // (waves without units of their own only keep the barriers company)
    const uint16_t *src = (k == 0) ? xs : hs + (size_t)(k & 1) * NC * hld;
    const int ld = (k == 0) ? XLD : hld;
    const int nsteps = (k == 0) ? 4 : ksh;
    {
      const uint16_t *brow = src + (size_t)rowoff * ld + koff;
      uint4 bcur[CT];
#pragma unroll
      for (int c = 0; c < CT; ++c) bcur[c] = *reinterpret_cast<const uint4 *>(brow + (size_t)c * 32 * ld);
      auto round = [&](int s0, auto startc) __attribute__((always_inline)) {
        constexpr bool starts = decltype(startc)::value;
        if (s0 + PD >= nsteps) wstep = 4;  // the next step's first fragments (always an h step)
#pragma unroll
        for (int j = 0; j < PD; ++j) {
          if constexpr (starts) {
            if (j == 0) {
              int boff = wu * 32 + 4 * (lane >> 5);
              asm volatile("" : "+v"(boff));  // (read afresh every step, not kept across them)
#pragma unroll
              for (int g = 0; g < 4; ++g) {
                floatx16 bg;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                  const float4 bv = *reinterpret_cast<const float4 *>(bias + g * H + boff + 8 * q);
                  bg[4 * q + 0] = bv.x; bg[4 * q + 1] = bv.y; bg[4 * q + 2] = bv.z; bg[4 * q + 3] = bv.w;
                }
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                  acc[g][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                      __builtin_bit_cast(bf16x8, ring[0][g]), __builtin_bit_cast(bf16x8, bcur[c]), bg, 0, 0, 0);
                  if (g == 3) bcur[c] = *reinterpret_cast<const uint4 *>(brow + (size_t)c * 32 * ld + 16);
                }
                ring[0][g] = stream_load(ws, voff, wstep * 4 + g);
              }
              continue;
            }
          }
          // column by column; every operand register is refilled in place behind the last product
          // that reads it: a column's activation fragment with the next k-step's (one k-step
          // past the end stays inside the row's padding or the next row), a weight fragment
          // with the one PD k-steps ahead
#pragma unroll
          for (int i = 0; i < 4 * CT; ++i) {
            const int c = i / 4, g = i % 4;
            acc[g][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                __builtin_bit_cast(bf16x8, ring[j][g]), __builtin_bit_cast(bf16x8, bcur[c]), acc[g][c], 0, 0, 0);
            if (g == 3) bcur[c] = *reinterpret_cast<const uint4 *>(brow + (size_t)c * 32 * ld + (s0 + j + 1) * 16);
            if (c == CT - 1) ring[j][g] = stream_load(ws, voff, (wstep + j) * 4 + g);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        wstep += PD;
      };
      round(0, vf_tag<true>{});
      for (int s0 = PD; s0 < nsteps; s0 += PD) round(s0, vf_tag<false>{});
    }
    uint16_t *hout = hs + (size_t)((k + 1) & 1) * NC * hld;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int u0 = wu * 32 + 4 * (lane >> 5) + 8 * q;
      const float4 whv = *reinterpret_cast<const float4 *>(whs + u0);
      const float whq[4] = {whv.x, whv.y, whv.z, whv.w};
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        float hv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int j = 4 * q + e;
          float cn = cst[c][j];
          hv[e] = lstm_cell(acc[0][c][j], acc[1][c][j], acc[2][c][j], acc[3][c][j], cn);
          cst[c][j] = cn;
          vsum[c] = fmaf(whq[e], hv[e], vsum[c]);
        }
        uint2 pkd;
        pkd.x = pack_bf16(hv[0], hv[1]);
        pkd.y = pack_bf16(hv[2], hv[3]);
        *reinterpret_cast<uint2 *>(hout + (size_t)(c * 32 + (lane & 31)) * hld + u0) = pkd;
      }
    }
    }
    if (fetch_g) reinterpret_cast<float4 *>(gls + (size_t)((k + 1) & 1) * H4)[tid] = gnext;
    __syncthreads();  // h_t and the next step's biases are in place
  }

#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const float v = vsum[c] + __shfl_xor(vsum[c], 32);
    if (lane < 32) red[w * NC + c * 32 + lane] = active ? v : 0.0f;
  }
  __syncthreads();
  if (tid < NC) {
    float s = md.hsum[b] + (float)(S - stage) * md.aux[H4 + H];
#pragma unroll
    for (int g = 0; g < 8; ++g) s += red[g * NC + tid];
    const bool ok = okf[tid] != 0;
    const int32_t cid = cids[tid];
    if (scores && ok) scores[(size_t)b * ld_scores + cid] = s;
    if (na.eps != 0.0f) s = add_noise(na, s, b, cid);
    float v = __builtin_inff();
    int32_t c = -1;
    if (ok && s < v) { v = s; c = cid; }
    wave_min(v, c);
    if (md.stat) {
      const int nok = __popcll(__ballot(ok));
      if (lane == 0) {
        atomicAdd(&md.stat[0], (unsigned long long)nok);
        atomicAdd(&md.stat[1], (unsigned long long)nok);
      }
    }
    if (tid == 0) {
      pval[slot] = v;
      pidx[slot] = c;
    }
  }
}

// The weights of k_seq_step_held and k_seq_step_wide: out[32 units][step][row tile][lane][8], steps = k-steps
// of h of the first 16 units ("pass 0"), of the other 16, then the four k-steps of x of either half; row
// tile 0 holds gate i of the 16 units in rows 0..15 and gate f in rows 16..31, row tile 1 the gates g and o.
__global__ __launch_bounds__(256) void k_pack_seq_wide(SeqWeights sw, uint16_t *out) {
  const int H = sw.H, ksh = H / 16, steps = 2 * ksh + 8;
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= H / 32 * steps * 1024) return;
  const int e = i & 7, lane = (i >> 3) & 63, r = (i >> 9) & 1, step = (i >> 10) % steps, w = (i >> 10) / steps;
  const bool of_x = step >= 2 * ksh;
  const int at = of_x ? step - 2 * ksh : step, per = of_x ? 4 : ksh, ps = at / per, s = at % per;
  const int row = lane & 31, gate = 2 * r + (row >> 4), unit = w * 32 + 16 * ps + (row & 15);
  const int k = s * 16 + 8 * (lane >> 5) + e;
  const float v = of_x ? sw.Wih[(size_t)(gate * H + unit) * 64 + k] : sw.Whh[(size_t)(gate * H + unit) * H + k];
  out[i] = (uint16_t)bf16_bits(v);
}

// ---- networks whose recurrent weights fit the registers of one workgroup (H <= 192)

// Opens decision `stage` of problem blockIdx.y for the two scorers below: the ordered list of its valid
// candidates, their number, and each one's 64 normalised features as a row of bfloat16.  The
// evaluation runs at full occupancy here, and none of its registers is taken from
// the scorers, which keep their weights there from one tile to the next.  Also: +inf into the masked score
// array (nullable), no minimum into the parts behind the last tile.  The list comes from the validity
// rules, not from a scan over the ids (one workgroup per problem, 10 us): 8 us for one problem, 18 for 64.
// The first `nadv` workgroups do something else: the prefix's step at the commit in front of this decision
// (seq_advance), which needs nothing of this and takes as long, so that the two make one launch (schedules of
// one problem of 20 layers, H = 32 0.70 -> 0.57 ms, 256 1.56 -> 1.51).
constexpr int SEQ_OPEN = 256;  // candidates per workgroup, four threads each
__global__ __launch_bounds__(1024) void k_seq_open(const uint32_t *decpack, uint32_t M, int64_t Mpad, int32_t *list, int32_t *count,
                                                   uint16_t *rows, float *scores, float *pval, int32_t *pidx, int nparts, int tile,
                                                   int nadv, SeqAdvance adv) {
  __shared__ union {
    struct {
      DecPack pk;
      EvalTabs tabs;
      OpenScratch os;
    } o;
    SeqAdvanceShared a;
  } sh;
  if ((int)blockIdx.x < nadv) {
    seq_advance(adv, sh.a, (int)blockIdx.x * SEQ_PB);
    return;
  }
  DecPack &pk = sh.o.pk;
  EvalTabs &tabs = sh.o.tabs;
  OpenScratch &os = sh.o.os;
  const int per = (int)(Mpad / SEQ_OPEN), at = (int)blockIdx.x - nadv, b = at / per, chunk = at - b * per;
  const int tid = threadIdx.x, lane = tid & 63, n = tid & (SEQ_OPEN - 1);
  const int part = __builtin_amdgcn_readfirstlane(tid / SEQ_OPEN);
  const int64_t k = (int64_t)chunk * SEQ_OPEN + n;
  if (tid < VF_DECPACK_DWORDS) reinterpret_cast<uint32_t *>(&pk)[tid] = decpack[(size_t)b * VF_DECPACK_DWORDS + tid];
  if (scores && part == 3) scores[(size_t)b * Mpad + k] = __builtin_inff();
  __syncthreads();
  fill_evaltabs(tabs, pk.d, pk.sp);
  if (tid >= 1015) list_factors(pk, os, tid - 1015);
  __syncthreads();
  if (tid < 64) list_pairs(pk, os, lane);
  __syncthreads();
  const int have = os.ncand;
  if (chunk == 0) {
    if (tid == 0) count[b] = have;
    for (int i = (have + tile - 1) / tile + tid; i < nparts; i += 1024) {
      pval[(size_t)b * nparts + i] = __builtin_inff();
      pidx[(size_t)b * nparts + i] = -1;
    }
  }
  if (k >= have) return;
  int pos_r[12];
#pragma unroll
  for (int j = 0; j < 12; ++j) pos_r[j] = j < os.npairs ? os.pos[j] : 0x7fffffff;
  const Digits g = unpack_digits(list_entry(pk, os, pos_r, (int)k, 1.0f / (float)pk.sp.nperm, 1.0f / (float)pk.sp.nvec));
  int32_t core[64];
  // sixteen rows of two 16-byte stores (what a thread does not store is dead code in its copy)
  auto put = [&](int row0) __attribute__((always_inline)) {
    uint4 *dst = reinterpret_cast<uint4 *>(rows + ((size_t)b * Mpad + k) * 64 + row0);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int32_t *v = core + row0 + 8 * q;
      uint4 o;
      o.x = pack_bf16(plog2_dev(v[0]), plog2_dev(v[1]));
      o.y = pack_bf16(plog2_dev(v[2]), plog2_dev(v[3]));
      o.z = pack_bf16(plog2_dev(v[4]), plog2_dev(v[5]));
      o.w = pack_bf16(plog2_dev(v[6]), plog2_dev(v[7]));
      dst[q] = o;
    }
  };
  if (part == 0) {
    eval_digits<true>(pk.d, pk.sp, g, &tabs, core);
    list[(size_t)b * Mpad + k] = (int32_t)id_of(pk.sp, g);
    put(0);
  } else if (part == 1) {
    eval_digits<true>(pk.d, pk.sp, g, &tabs, core);
    put(16);
  } else if (part == 2) {
    eval_digits<true>(pk.d, pk.sp, g, &tabs, core);
    put(32);
  } else {
    eval_digits<true>(pk.d, pk.sp, g, &tabs, core);
    put(48);
  }
}

// A workgroup's share of the tiles of NC list entries of all problems, in problem-major order: tiles
// [t_begin, t_end), the first one being tile `tile` of problem `b` (every thread of the NW waves gets
// the same; wsum: NW words of LDS, at: two).  false: no tile.
template <int NW, int NC>
__device__ __forceinline__ bool seq_share(const int32_t *count, int B, int tid, int lane, int w, int32_t *wsum, int32_t *at,
                                          int &t_begin, int &t_end) {
  constexpr int NT = 64 * NW;
  const int per = (B + NT - 1) / NT;  // a thread counts `per` consecutive problems
  int mine = 0;
  for (int q = 0; q < per; ++q) {
    const int b = tid * per + q;
    if (b < B) mine += (count[b] + NC - 1) / NC;
  }
  int upto = mine;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int o = __shfl_up(upto, off);
    if (lane >= off) upto += o;
  }
  if (lane == 63) wsum[w] = upto;
  __syncthreads();
  int total = 0;
#pragma unroll
  for (int q = 0; q < NW; ++q) {
    if (q == w) upto += total;
    total += wsum[q];
  }
  t_begin = (int)((int64_t)blockIdx.x * total / gridDim.x);
  t_end = (int)((int64_t)(blockIdx.x + 1) * total / gridDim.x);
  if (t_begin >= t_end) return false;
  if (t_begin >= upto - mine && t_begin < upto) {
    // the thread whose problems hold the first tile
    int b = tid * per, first = upto - mine;
    for (;;) {
      const int n = (count[b] + NC - 1) / NC;
      if (t_begin < first + n) break;
      first += n;
      ++b;
    }
    at[0] = b;
    at[1] = t_begin - first;
  }
  return true;
}

// The end of a tile, by one wave: the head's predictions of the tile's columns (red: [NW][NC], the waves'
// parts), the scores if they are wanted, the tile's first minimum.
template <int NW, int NC>
__device__ __forceinline__ void seq_tile_end(const SeqDev &md, const float *red, float constant, int b, int n0, int nvalid, int lane,
                                             float *scores, int64_t ld_scores, float *pval, int32_t *pidx, size_t slot,
                                             const NoiseArgs &na) {
  const bool ok = lane < NC && n0 + lane < nvalid;
  const int32_t cid = ok ? md.list[(size_t)b * md.Mpad + n0 + lane] : -1;
  float s = md.hsum[b] + constant;
#pragma unroll
  for (int g = 0; g < NW; ++g) s += red[g * NC + (lane & (NC - 1))];
  if (scores && ok) scores[(size_t)b * ld_scores + cid] = s;
  if (na.eps != 0.0f) s = add_noise(na, s, b, cid);
  float v = __builtin_inff();
  int32_t c = -1;
  if (ok && s < v) { v = s; c = cid; }
  wave_min(v, c);
  if (md.stat) {
    const int nok = __popcll(__ballot(ok));
    if (lane == 0) {
      atomicAdd(&md.stat[0], (unsigned long long)nok);
      atomicAdd(&md.stat[1], (unsigned long long)nok);
    }
  }
  if (lane == 0) {
    pval[slot] = v;
    pidx[slot] = c;
  }
}

// Cell states of a wave's unit tile `u` of 16 at the problem's prefix: a lane has units
// 8 q + 4 (lane / 32) + e.
__device__ __forceinline__ void seq_state(float (&cst)[8], const float *cpre, int u, int lane) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const float4 cv = *reinterpret_cast<const float4 *>(cpre + u * 16 + 8 * q + 4 * (lane >> 5));
    cst[4 * q + 0] = cv.x; cst[4 * q + 1] = cv.y; cst[4 * q + 2] = cv.z; cst[4 * q + 3] = cv.w;
  }
}

// LDS of k_seq_step_held and k_seq_step_wide: weights, h buffers, gate biases, head, the waves' predictions.
template <int KS, int NW, int NC, int LK>
struct SeqHeldLds {
  static constexpr int H = 16 * KS, HLD = H + 8;
  uint4 w[KS * LK * 128 + 1];                        // [unit tile][LK][2][64]
  __attribute__((aligned(16))) uint16_t h[2][NC * HLD];
  __attribute__((aligned(16))) float g[2][4 * H];    // this step's gate biases and the next one's
  __attribute__((aligned(16))) float wh[H];
  float red[NW * NC];
  int32_t wsum[NW], at[2];
};

// The candidates that k_seq_open listed, one cell step on their own features and one per later stage,
// H = 16 KS <= 192 hidden units.  A workgroup holds all of W_hh and goes through its share of the tiles of
// 32 candidates: wave w has the four gates of units 16 w .. 16 w + 15, RK k-steps of its weights in
// registers and the others in LDS, so that a step takes nothing from memory but the next step's gate
// biases.  (Streaming W_hh out of L2 for every step, in tiles of 96 with 32 units per wave, left one wave of
// eight at work for H = 32, and a wave waits for its fragments longer than it computes.)  What bounds a
// step now is the vector work of the gates, 28 instructions per cell: a wave by itself issues one
// every six to seven cycles, so a SIMD wants several - 8, 4 and 2 workgroups per compute unit for H = 32,
// 64 and 96, each at its own place in a step, so that one's gates run under another's products.
// Schedules of 20 ResNet-18-shaped layers of 4096 ids (each problem its own widths and resolution), with
// W_hh streamed and now: 64 problems H = 32 5.52 -> 1.75 ms, 64 4.90 -> 2.16, 128 6.45 -> 4.36, 192 12.4 -> 7.8;
// one problem 1.15 -> 0.56, 1.21 -> 0.61, 1.36 -> 0.83, 2.01 -> 1.16 ms (in all; the opening of a decision and the
// prefix's step have become cheaper as well).
template <int KS, int WPE, int RK>
__global__ __launch_bounds__(KS * 64, WPE) void k_seq_step_held(SeqDev md, const uint16_t *w_wide, const uint16_t *rows, int stage, int B,
                                                          float *scores, int64_t ld_scores, float *pval, int32_t *pidx, int nparts,
                                                          NoiseArgs na) {
  constexpr int H = 16 * KS, NT = 64 * KS, NC = 32, LK = KS - RK;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  SeqHeldLds<KS, KS, NC, LK> &sh = *reinterpret_cast<SeqHeldLds<KS, KS, NC, LK> *>(smem);
  constexpr int HLD = H + 8;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = md.S;
  int t_begin, t_end;
  if (!seq_share<KS, NC>(md.count, B, tid, lane, w, sh.wsum, sh.at, t_begin, t_end)) return;

  const __amdgpu_buffer_rsrc_t ws = stream_rsrc(w_wide);
  const int voff = 16 * lane, base = (w >> 1) * (2 * KS + 8);
  const int hfrag = (base + (w & 1) * KS) * 2, xfrag = (base + 2 * KS + 4 * (w & 1)) * 2;
  uint4 *const wl = sh.w + w * LK * 128 + lane;
  bf16x8 wr[RK][2];
#pragma unroll
  for (int s = 0; s < KS; ++s)
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const uint4 f = stream_load(ws, voff, hfrag + s * 2 + r);
      if (s < RK) wr[s < RK ? s : 0][r] = __builtin_bit_cast(bf16x8, f);
      else wl[((s - RK) * 2 + r) * 64] = f;
    }
  for (int i = tid; i < H; i += NT) sh.wh[i] = md.aux[4 * H + i];
  const float bhead = md.aux[5 * H];
  __syncthreads();
  int b = __builtin_amdgcn_readfirstlane(sh.at[0]), tile = __builtin_amdgcn_readfirstlane(sh.at[1]);
  const int u0 = 16 * w + 4 * (lane >> 5);  // the lane's units: u0 + 8 q + e

  for (int t = t_begin; t < t_end; ++t, ++tile) {
    int nvalid = md.count[b];
    while (tile * NC >= nvalid) {
      ++b;
      tile = 0;
      nvalid = md.count[b];
    }
    const int n0 = tile * NC;
    // (a ragged tile's last rows are whatever is there: their columns are dropped at the end)
    const uint4 *xrow = reinterpret_cast<const uint4 *>(rows + ((size_t)b * md.Mpad + n0 + (lane & 31)) * 64) + (lane >> 5);
    if (tid < H) reinterpret_cast<float4 *>(sh.g[0])[tid] = reinterpret_cast<const float4 *>(md.P + (size_t)b * 4 * H)[tid];
    float cst[1][8], vsum[1] = {0.0f};
    seq_state(cst[0], md.cpre + (size_t)b * H, w, lane);
    __syncthreads();
    auto step = [&](int st, auto firstc) __attribute__((always_inline)) {
      constexpr bool first = decltype(firstc)::value;
      const int k = st - stage;
      // the next step's biases, fetched now, parked in LDS after this step's gates
      const bool fetch_g = st + 1 < S && tid < H;
      float4 gnext = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if (fetch_g) gnext = reinterpret_cast<const float4 *>(md.G + ((size_t)b * S + st + 1) * 4 * H)[tid];
      const float *bias = sh.g[k & 1] + u0;
      floatx16 acc[2][1];
      if constexpr (first) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          bf16x8 a[2], bv[1];
#pragma unroll
          for (int r = 0; r < 2; ++r) a[r] = __builtin_bit_cast(bf16x8, stream_load(ws, voff, xfrag + s * 2 + r));
          bv[0] = __builtin_bit_cast(bf16x8, xrow[2 * s]);
          lstm_products<1>(acc, s == 0, bias, H, a, bv);
          if (s == 1) __builtin_amdgcn_sched_barrier(0);
        }
      } else {
        const uint16_t *bb = sh.h[k & 1] + (lane & 31) * HLD + 8 * (lane >> 5);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          bf16x8 a[2], bv[1];
          bv[0] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(bb + s * 16));
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            if (s < RK) a[r] = wr[s < RK ? s : 0][r];
            else a[r] = __builtin_bit_cast(bf16x8, wl[((s - RK) * 2 + r) * 64]);
          }
          lstm_products<1>(acc, s == 0, bias, H, a, bv);
        }
      }
      lstm_gates<1>(acc, cst, vsum, sh.wh + u0, sh.h[(k + 1) & 1] + (lane & 31) * HLD + u0, 0);
      if (fetch_g) reinterpret_cast<float4 *>(sh.g[(k + 1) & 1])[tid] = gnext;
      __syncthreads();  // h and the next step's biases are in place
    };
    step(stage, vf_tag<true>{});
    for (int st = stage + 1; st < S; ++st) step(st, vf_tag<false>{});

    vsum[0] += __shfl_xor(vsum[0], 32);
    if (lane < 32) sh.red[w * NC + lane] = vsum[0];
    __syncthreads();
    if (w == 0)
      seq_tile_end<KS, NC>(md, sh.red, (float)(S - stage) * bhead, b, n0, nvalid, lane, scores, ld_scores, pval, pidx,
                           (size_t)b * nparts + tile, na);
    // (red is written again behind the next tile's first barrier; g[0] and the h buffers were last read in
    // front of the barrier that ended the last step)
  }
}

// The same for H = 224 and 256: W_hh (401 and 512 KB) is more than a compute unit holds.  A wave has 32
// units in two passes of 16; of a pass's KS k-steps RK stay in registers, LK in LDS, the others stream
// out of L2 through a ring of two, spread evenly between them.  Tiles are of 32 candidates (CT = 1) or, where
// there are enough of them, 64: the stream then serves twice as many.  On its SIMD a wave of the first
// four (group A) shares the vector unit and the matrix core with one of the others (group B), and a
// step has four phases with a barrier behind each, in which one has its products while the other has
// its gates:
//   A: rest of products 0, gates 0 | products 1 | gates 1    | next step's products 0 as far as h is there
//   B: products 0                  | gates 0    | products 1 | gates 1
// (A's last phase leaves out the units that B's last gates are about to write.)  What bounds it: a phase
// is as long as its gates, which take a single wave 1700 cycles for 8 x 64 cells with products beside
// them, where the products take 1000 to 1400; without the phases both waves contract at the same time
// and the second one does its gates alone (+3 %).  Holding more of the weights or more waves in flight
// both want the registers of the other.  The schedules above, H = 256: 64 problems 13.7 -> 11.0 ms (before: tiles of
// 96, all weights streamed), 8: 2.87 -> 2.42, one: 2.23 -> 1.49.
template <int KS, int CT, int RK, int LK>
struct SeqWidePlan {
  static constexpr int NW = KS / 2, SK = KS - RK - LK;
  static constexpr int LATE = NW - 4;  // unit tiles that are written last: pass 1 of waves 4..
  // the order of the k-steps (unit tiles): those tiles last
  static constexpr int order(int i) {
    return i < KS - LATE ? (i < 8 ? i : 8 + 2 * (i - 8)) : 9 + 2 * (i - (KS - LATE));
  }
  static constexpr bool streamed(int i) { return (i + 1) * SK / KS > i * SK / KS; }
  static constexpr int stream_index(int i) { return i * SK / KS; }      // of a streamed place in the order
  static constexpr int held_index(int i) { return i - i * SK / KS; }    // of any other: < RK registers, else LDS
  static constexpr int stream_step(int j) { return order(((j + 1) * KS + SK - 1) / SK - 1); }
};
template <int KS, int CT, int RK, int LK>
__global__ __launch_bounds__(KS * 32, 2) void k_seq_step_wide(SeqDev md, const uint16_t *w_wide, const uint16_t *rows, int stage, int B,
                                                         float *scores, int64_t ld_scores, float *pval, int32_t *pidx, int nparts,
                                                         NoiseArgs na) {
  using Plan = SeqWidePlan<KS, CT, RK, LK>;
  constexpr int H = 16 * KS, NW = Plan::NW, NT = 64 * NW, NC = 32 * CT, SK = Plan::SK, PD = 2, HLD = H + 8;
  static_assert(NW > 4 && NW <= 8 && SK >= PD, "two groups of waves, a stream");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  SeqHeldLds<KS, NW, NC, LK> &sh = *reinterpret_cast<SeqHeldLds<KS, NW, NC, LK> *>(smem);
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = md.S;
  int t_begin, t_end;
  if (!seq_share<NW, NC>(md.count, B, tid, lane, w, sh.wsum, sh.at, t_begin, t_end)) return;

  const __amdgpu_buffer_rsrc_t ws = stream_rsrc(w_wide);
  const int voff = 16 * lane, hfrag = w * (2 * KS + 8) * 2, xfrag = hfrag + 4 * KS;  // (pass 1: KS, or 4, k-steps on)
  uint4 *const wl = sh.w + w * 2 * LK * 128 + lane;
  bf16x8 wr[2][RK][2], ring[PD][2];
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int i = 0; i < KS; ++i)
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        if (Plan::streamed(i)) continue;
        const uint4 f = stream_load(ws, voff, hfrag + (p * KS + Plan::order(i)) * 2 + r);
        const int at = Plan::held_index(i);
        if (at < RK) wr[p][at < RK ? at : 0][r] = __builtin_bit_cast(bf16x8, f);
        else wl[((p * LK + at - RK) * 2 + r) * 64] = f;
      }
#pragma unroll
  for (int j = 0; j < PD; ++j)
#pragma unroll
    for (int r = 0; r < 2; ++r) ring[j][r] = __builtin_bit_cast(bf16x8, stream_load(ws, voff, hfrag + Plan::stream_step(j) * 2 + r));
  for (int i = tid; i < H; i += NT) sh.wh[i] = md.aux[4 * H + i];
  const float bhead = md.aux[5 * H];
  __syncthreads();
  int b = __builtin_amdgcn_readfirstlane(sh.at[0]), tile = __builtin_amdgcn_readfirstlane(sh.at[1]);

  for (int t = t_begin; t < t_end; ++t, ++tile) {
    int nvalid = md.count[b];
    while (tile * NC >= nvalid) {
      ++b;
      tile = 0;
      nvalid = md.count[b];
    }
    const int n0 = tile * NC;
    // (a ragged tile's last rows are whatever is there: their columns are dropped at the end)
    const uint4 *xrow = reinterpret_cast<const uint4 *>(rows + ((size_t)b * md.Mpad + n0 + (lane & 31)) * 64) + (lane >> 5);
    if (tid < H) reinterpret_cast<float4 *>(sh.g[0])[tid] = reinterpret_cast<const float4 *>(md.P + (size_t)b * 4 * H)[tid];
    float cst[2][CT][8], vsum[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      vsum[c] = 0.0f;
      seq_state(cst[0][c], md.cpre + (size_t)b * H, 2 * w, lane);
      seq_state(cst[1][c], md.cpre + (size_t)b * H, 2 * w + 1, lane);
    }
    __syncthreads();

    floatx16 acc[2][CT];
    // products of pass p of the tile's first step: the candidates' own features
    auto products_x = [&](int p) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        bf16x8 a[2], bv[CT];
#pragma unroll
        for (int r = 0; r < 2; ++r) a[r] = __builtin_bit_cast(bf16x8, stream_load(ws, voff, xfrag + (4 * p + s) * 2 + r));
#pragma unroll
        for (int c = 0; c < CT; ++c) bv[c] = __builtin_bit_cast(bf16x8, xrow[c * 32 * 8 + 2 * s]);
        lstm_products<CT>(acc, s == 0, sh.g[0] + 32 * w + 16 * p + 4 * (lane >> 5), H, a, bv);
        if (s & 1) __builtin_amdgcn_sched_barrier(0);
      }
    };
    // products of pass p of step k, places [i0, i1) of the order
    auto products_h = [&](int p, int k, int i0, int i1) __attribute__((always_inline)) {
      const uint16_t *bb = sh.h[k & 1] + (lane & 31) * HLD + 8 * (lane >> 5);
      const float *bias = sh.g[k & 1] + 32 * w + 16 * p + 4 * (lane >> 5);
      bf16x8 bv[CT], al[2];  // a place's activations, and its weights where they come from LDS
      auto fetch = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < CT; ++c)
          bv[c] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(bb + c * 32 * HLD + Plan::order(i) * 16));
        if (!Plan::streamed(i) && Plan::held_index(i) >= RK) {
#pragma unroll
          for (int r = 0; r < 2; ++r) al[r] = __builtin_bit_cast(bf16x8, wl[((p * LK + Plan::held_index(i) - RK) * 2 + r) * 64]);
        }
      };
      fetch(i0);
#pragma unroll
      for (int i = i0; i < i1; ++i) {
        bf16x8 a[2], bc[CT];
        const int j = Plan::stream_index(i), at = Plan::held_index(i), slot = (p * SK + j) % PD;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          if (Plan::streamed(i)) a[r] = ring[slot][r];
          else if (at < RK) a[r] = wr[p][at < RK ? at : 0][r];
          else a[r] = al[r];
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) bc[c] = bv[c];
        if (i + 1 < i1) fetch(i + 1);  // (under this place's products)
        __builtin_amdgcn_sched_barrier(0);
        lstm_products<CT>(acc, i == 0, bias, H, a, bc);
        if (Plan::streamed(i)) {
          // the slot takes the streamed place PD further on: of this pass, or of the other one
          const int n = j + PD;
          const int step = n < SK ? p * KS + Plan::stream_step(n < SK ? n : 0) : (p ^ 1) * KS + Plan::stream_step(n < SK ? 0 : n - SK);
#pragma unroll
          for (int r = 0; r < 2; ++r) ring[slot][r] = __builtin_bit_cast(bf16x8, stream_load(ws, voff, hfrag + step * 2 + r));
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    auto gates = [&](int p, int k) __attribute__((always_inline)) {
      const int u0 = 32 * w + 16 * p + 4 * (lane >> 5);
      lstm_gates<CT>(acc, cst[p], vsum, sh.wh + u0, sh.h[(k + 1) & 1] + (lane & 31) * HLD + u0, 32 * HLD);
    };
    if (w < 4) {
      products_x(0);
      for (int k = 0; k < S - stage; ++k) {
        // the next step's biases (a float4 per thread of this group), fetched now, parked in LDS behind the gates
        const bool more = k + 1 < S - stage, fetch_g = more && tid < H;
        float4 gnext = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (fetch_g) gnext = reinterpret_cast<const float4 *>(md.G + ((size_t)b * S + stage + k + 1) * 4 * H)[tid];
        if (k > 0) products_h(0, k, KS - Plan::LATE, KS);
        gates(0, k);
        __syncthreads();
        if (k > 0) products_h(1, k, 0, KS);
        else products_x(1);
        __syncthreads();
        gates(1, k);
        if (fetch_g) reinterpret_cast<float4 *>(sh.g[(k + 1) & 1])[tid] = gnext;
        __syncthreads();
        if (more) products_h(0, k + 1, 0, KS - Plan::LATE);
        __syncthreads();
      }
    } else {
      for (int k = 0; k < S - stage; ++k) {
        if (k > 0) products_h(0, k, 0, KS);
        else products_x(0);
        __syncthreads();
        gates(0, k);
        __syncthreads();
        if (k > 0) products_h(1, k, 0, KS);
        else products_x(1);
        __syncthreads();
        gates(1, k);
        __syncthreads();
      }
    }
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const float v = vsum[c] + __shfl_xor(vsum[c], 32);
      if (lane < 32) sh.red[w * NC + c * 32 + lane] = v;
    }
    __syncthreads();
    if (w == 0)
      seq_tile_end<NW, NC>(md, sh.red, (float)(S - stage) * bhead, b, n0, nvalid, lane, scores, ld_scores, pval, pidx,
                           (size_t)b * nparts + tile, na);
  }
}

SeqWeights weights_of(const vf_ctx *c) {
  const int H = c->model.dims[1];
  SeqWeights sw;
  sw.H = H;
  sw.Wih = c->pm.w_f32;
  sw.Whh = sw.Wih + (size_t)4 * H * 64;
  sw.bih = sw.Whh + (size_t)4 * H * H;
  sw.bhh = sw.bih + 4 * H;
  sw.wh = sw.bhh + 4 * H;
  sw.bh = sw.wh + H;
  return sw;
}

SeqState state_of(const vf_ctx *c, int set) {
  SeqState s;
  s.hfb = c->d_seq_h[set]; s.cpre = c->d_seq_c[set]; s.P = c->d_seq_P[set]; s.hsum = c->d_seq_hs[set];
  return s;
}

}  // namespace

bool vfk_seq_model(const vf_ctx *c) {
  return c->has_model && c->model.kind == VF_LSTM && c->model.dtype == VF_BF16 && c->model.dims[0] == 64 &&
         c->pm.w_f32 != nullptr;
}

void vfk_seq_free(vf_ctx *c) {
  void *ps[] = {c->d_seq_G, c->d_seq_h[0], c->d_seq_h[1], c->d_seq_c[0], c->d_seq_c[1],
                c->d_seq_P[0], c->d_seq_P[1], c->d_seq_hs[0], c->d_seq_hs[1], c->d_seq_list, c->d_seq_count, c->d_seq_rows};
  for (void *p : ps)
    if (p) (void)hipFree(p);
  c->d_seq_G = nullptr;
  c->d_seq_list = nullptr;
  c->d_seq_count = nullptr;
  c->d_seq_rows = nullptr;
  for (int k = 0; k < 2; ++k) c->d_seq_h[k] = c->d_seq_c[k] = c->d_seq_P[k] = c->d_seq_hs[k] = nullptr;
  c->seq_stage = -1;
  c->seq_pending = 0;
  c->seq_cur = 0;
}

// The scorer for networks of H hidden units: its workgroups per compute unit, threads, LDS, candidates
// per tile.  many: more than about one round of tiles.  At H = 128 two workgroups of 128 registers then
// are better than one of all, above 192 tiles of 64.  Schedules as above, not many / many: H = 128 4
// problems 0.89 / 1.11 ms, 8: 1.15 / 1.18, 12: 1.41 / 1.35, 16: 1.64 / 1.59, 64: 4.88 / 4.36; H = 224 8: 1.76 / 1.97, 12:
// 2.47 / 2.43, 16: 2.67 / 2.82, 64: 8.42 / 7.96; H = 256 8: 2.46 / 2.54, 12: 3.08 / 2.82, 16: 3.75 / 3.77, 64: 12.3 / 11.4.
struct HeldKernel {
  void (*fn)(SeqDev, const uint16_t *, const uint16_t *, int, int, float *, int64_t, float *, int32_t *, int, NoiseArgs);
  int per_cu, threads, tile;
  size_t lds;
};
template <int KS, int WPE, int RK>
static HeldKernel held_kernel(int per_cu) {
  return {k_seq_step_held<KS, WPE, RK>, per_cu, KS * 64, 32, sizeof(SeqHeldLds<KS, KS, 32, KS - RK>)};
}
template <int KS, int CT, int RK, int LK>
static HeldKernel wide_kernel() {
  return {k_seq_step_wide<KS, CT, RK, LK>, 1, KS * 32, 32 * CT, sizeof(SeqHeldLds<KS, KS / 2, 32 * CT, LK>)};
}
static HeldKernel held_kernel_of(int H, bool many) {
  switch (H / 32) {
    case 1: return held_kernel<2, 4, 2>(8);
    case 2: return held_kernel<4, 4, 4>(4);
    case 3: return held_kernel<6, 3, 6>(2);
    case 4: return many ? held_kernel<8, 4, 5>(2) : held_kernel<8, 2, 8>(1);
    case 5: return held_kernel<10, 3, 8>(1);
    case 6: return held_kernel<12, 3, 9>(1);
    case 7: return many ? wide_kernel<14, 2, 1, 3>() : wide_kernel<14, 1, 5, 4>();
    default: return many ? wide_kernel<16, 2, 1, 2>() : wide_kernel<16, 1, 5, 3>();
  }
}

// The step of the prefix at the commit of `stage`.  how: 1 in place, 2 from the parents' set to the other one.
static SeqAdvance advance_of(const vf_ctx *c, int stage, int how) {
  SeqAdvance a;
  a.t = tables_of(c);
  a.stage = stage;
  a.sw = weights_of(c);
  a.WT = c->pm.w_seqT;
  a.src = state_of(c, c->seq_cur);
  a.dst = how == 2 ? state_of(c, c->seq_cur ^ 1) : a.src;
  a.sel_idx = how == 2 ? c->d_sel_idx : nullptr;
  a.sel_n = how == 2 ? c->d_sel_n : nullptr;
  a.Mpad = (int64_t)c->Mpad;
  a.B = c->B;
  return a;
}

// Tables and prefix state of the recurrence for the context's pipeline, model and
// committed prefix: built on first use, rebuilt after anything but a commit changed them.
int vfk_seq_sync(vf_ctx *c, int stage) {
  const int H = c->model.dims[1], B = c->B, S = c->S;
  const SeqWeights sw = weights_of(c);
  hipStream_t st = c->stream;
  if (!c->d_seq_G) {
    struct { float **p; size_t n; } want[] = {
        {&c->d_seq_G, (size_t)B * S * 4 * H},
        {&c->d_seq_h[0], (size_t)B * H}, {&c->d_seq_h[1], (size_t)B * H},
        {&c->d_seq_c[0], (size_t)B * H}, {&c->d_seq_c[1], (size_t)B * H},
        {&c->d_seq_P[0], (size_t)B * 4 * H}, {&c->d_seq_P[1], (size_t)B * 4 * H},
        {&c->d_seq_hs[0], (size_t)B}, {&c->d_seq_hs[1], (size_t)B}};
    bool ok = true;
    for (auto &wt : want) ok = ok && hipMalloc((void **)wt.p, wt.n * sizeof(float)) == hipSuccess;
    ok = ok && hipMalloc((void **)&c->d_seq_list, (size_t)B * c->Mpad * 4) == hipSuccess;
    ok = ok && hipMalloc((void **)&c->d_seq_count, (size_t)B * 4) == hipSuccess;
    if (!ok) {
      (void)hipGetLastError();
      vfk_seq_free(c);
      return VF_ENOMEM;
    }
    if (hipMalloc((void **)&c->d_seq_rows, (size_t)B * c->Mpad * 64 * sizeof(uint16_t)) != hipSuccess) {
      (void)hipGetLastError();  // (without memory for the rows the scorers below evaluate the candidates themselves)
      c->d_seq_rows = nullptr;
    }
    const size_t n = (size_t)B * S * 4 * H;
    hipLaunchKernelGGL(k_seq_tables, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, c->d_intr, sw,
                       (size_t)B * S, c->d_seq_G);
    VF_HIP(c, hipGetLastError());
    if (!c->pm.w_seqT) {
      const size_t nw = (size_t)(64 + H) * 4 * H;
      if (hipMalloc((void **)&c->pm.w_seqT, nw * sizeof(float)) != hipSuccess) {
        (void)hipGetLastError();
        vfk_seq_free(c);
        return VF_ENOMEM;
      }
      hipLaunchKernelGGL(k_pack_seqT, dim3((unsigned)((nw + 255) / 256)), dim3(256), 0, st, sw, c->pm.w_seqT);
      VF_HIP(c, hipGetLastError());
    }
    if (!c->pm.w_seq_wide) {
      // (without memory for this second form every step runs in tiles of 64, see vfk_seq_step)
      const size_t nv = (size_t)H / 32 * (2 * (H / 16) + 8) * 1024;
      if (hipMalloc((void **)&c->pm.w_seq_wide, nv * sizeof(uint16_t)) != hipSuccess) {
        (void)hipGetLastError();
        c->pm.w_seq_wide = nullptr;
      } else {
        hipLaunchKernelGGL(k_pack_seq_wide, dim3((unsigned)((nv + 255) / 256)), dim3(256), 0, st, sw, c->pm.w_seq_wide);
        VF_HIP(c, hipGetLastError());
      }
    }
    c->seq_stage = -1;
  }
  if (c->seq_stage == stage && !c->seq_pending) return VF_OK;
  if (c->seq_pending && c->seq_stage >= 0 && c->seq_stage + 1 == stage) return VF_OK;  // (the caller's to do)
  c->seq_cur = 0;
  const size_t n = (size_t)B * 4 * H;
  const SeqState s0 = state_of(c, 0);
  hipLaunchKernelGGL(k_seq_reset, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, sw, B, s0.hfb, s0.cpre, s0.P,
                     s0.hsum);
  VF_HIP(c, hipGetLastError());
  c->seq_pending = 0;
  for (int t = 0; t < stage; ++t) {
    hipLaunchKernelGGL(k_seq_advance, dim3((unsigned)((B + SEQ_PB - 1) / SEQ_PB)), dim3(1024), 0, st, advance_of(c, t, 1));
    VF_HIP(c, hipGetLastError());
  }
  c->seq_stage = stage;
  return VF_OK;
}

// After the commit of `stage`: one more step of every problem's prefix recurrence.  It is left for the
// launch that opens the call's next decision (vfk_seq_step); behind its last one vfk_seq_flush does it.
int vfk_seq_advance(vf_ctx *c, int stage) {
  if (c->seq_stage == stage) c->seq_pending = 1;  // (not in step: rebuilt at the next use)
  return VF_OK;
}

// beam search: slot j of the new layer continues the recurrence of its parent slot
int vfk_seq_advance_beam(vf_ctx *c, int stage) {
  if (c->seq_stage == stage) c->seq_pending = 2;
  return VF_OK;
}

static void advanced(vf_ctx *c) {
  if (c->seq_pending == 2) c->seq_cur ^= 1;
  c->seq_stage += 1;
  c->seq_pending = 0;
}

// A step that was left undone, by itself: at the end of a call, and before anything it reads changes (the
// survivors of a beam).
int vfk_seq_flush(vf_ctx *c) {
  if (!c->seq_pending || c->seq_stage < 0 || !c->d_seq_G) return VF_OK;
  hipLaunchKernelGGL(k_seq_advance, dim3((unsigned)((c->B + SEQ_PB - 1) / SEQ_PB)), dim3(1024), 0, c->stream,
                     advance_of(c, c->seq_stage, c->seq_pending));
  VF_HIP(c, hipGetLastError());
  advanced(c);
  return VF_OK;
}

// V of every candidate state of decision `stage` of every problem: per-tile minima into
// the partial arrays, optionally the masked scores [B][ld_scores].
int vfk_seq_step(vf_ctx *c, int stage, float *scores, int64_t ld_scores, int noise_stage, int *nparts_out) {
  int rc = vfk_seq_sync(c, stage);
  if (rc != VF_OK) return rc;
  rc = vfk_prepare(c, stage);
  if (rc != VF_OK) return rc;
  const int H = c->model.dims[1];
  int ncu = 256;
  (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, c->device);
  // (a third of the ids is valid, as a rule: three rounds of ids in tiles of 64)
  const HeldKernel hk = held_kernel_of(H, (c->M + 63) / 64 * c->B >= 3 * (int64_t)ncu);
  const bool held = c->pm.w_seq_wide && c->d_seq_rows && c->Mpad / SEQ_OPEN * c->B < (1 << 21);  // (a launch has less than 2^32 threads)
  const int NC = held ? hk.tile : 64;
  const int nparts = (int)((c->M + NC - 1) / NC);
  rc = vfk_ensure_parts(c, (size_t)nparts * c->B);
  if (rc != VF_OK) return rc;
  if (!held) {
    rc = vfk_seq_flush(c);
    if (rc != VF_OK) return rc;
  }
  SeqAdvance adv = {};
  const int nadv = c->seq_pending ? (c->B + SEQ_PB - 1) / SEQ_PB : 0;
  if (nadv) adv = advance_of(c, c->seq_stage, c->seq_pending);
  const SeqState s = state_of(c, c->seq_pending == 2 ? c->seq_cur ^ 1 : c->seq_cur);  // behind that step
  SeqDev md;
  md.H = H; md.S = c->S; md.w_pack = c->pm.w_pack; md.aux = c->pm.aux;
  md.G = c->d_seq_G; md.P = s.P; md.cpre = s.cpre; md.hsum = s.hsum;
  md.decpack = c->d_decpack;
  md.list = c->d_seq_list; md.count = c->d_seq_count; md.Mpad = c->Mpad;
  md.stat = c->profiling ? c->d_stat : nullptr;
  NoiseArgs na;
  na.eps = noise_stage >= 0 ? c->noise_eps : 0.0f;
  na.k0 = (uint32_t)c->noise_seed; na.k1 = (uint32_t)(c->noise_seed >> 32);
  na.stage = noise_stage; na.first_rollout = c->noise_first;
  *nparts_out = nparts;
  if (held) {
    {
      vf_prof_scope prof(c, VF_PROF_FEATURIZE);
      hipLaunchKernelGGL(k_seq_open, dim3((unsigned)nadv + (unsigned)(c->Mpad / SEQ_OPEN) * (unsigned)c->B), dim3(1024), 0, c->stream,
                         c->d_decpack, (uint32_t)c->M, (int64_t)c->Mpad, c->d_seq_list, c->d_seq_count, c->d_seq_rows, scores,
                         c->d_pval, c->d_pidx, nparts, hk.tile, nadv, adv);
      VF_HIP(c, hipGetLastError());
    }
    if (nadv) advanced(c);
    vf_prof_scope prof(c, VF_PROF_SCORE);
    VF_HIP(c, hipFuncSetAttribute((const void *)hk.fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)hk.lds));
    const int64_t most = (int64_t)nparts * c->B, fit = (int64_t)hk.per_cu * ncu;
    hipLaunchKernelGGL(hk.fn, dim3((unsigned)(most < fit ? most : fit)), dim3(hk.threads), hk.lds, c->stream, md,
                       (const uint16_t *)c->pm.w_seq_wide, (const uint16_t *)c->d_seq_rows, stage, c->B, scores, ld_scores,
                       c->d_pval, c->d_pidx, nparts, na);
    VF_HIP(c, hipGetLastError());
    return VF_OK;
  }
  hipLaunchKernelGGL(k_seq_compact, dim3((unsigned)c->B), dim3(1024), 0, c->stream, c->d_decpack, (uint32_t)c->M,
                     (int64_t)c->Mpad, c->d_seq_list, c->d_seq_count, scores);
  VF_HIP(c, hipGetLastError());
  const int hld = H + 8;
  const size_t smem = (size_t)NC * 72 * 2 + (size_t)2 * NC * hld * 2 + (size_t)2 * 4 * H * 4 + (size_t)8 * NC * 4 +
                      (size_t)H * 4 + (size_t)2 * NC * 4;
  {
    vf_prof_scope prof(c, VF_PROF_SCORE);
    void (*kern)(SeqDev, int, int64_t, float *, int64_t, float *, int32_t *, NoiseArgs) = k_seq_step<64, 2>;
    VF_HIP(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    hipLaunchKernelGGL(kern, dim3((unsigned)nparts, (unsigned)c->B), dim3(512), smem, c->stream, md, stage, c->M,
                       scores, ld_scores, c->d_pval, c->d_pidx, na);
    VF_HIP(c, hipGetLastError());
  }
  return VF_OK;
}
