// bf16 fast path of one aggregation level on gfx950 (paper Section 2.1: a cross-attention layer
// reduces the channel tokens of a patch to one token; Section 3.2: one layer per channel group).
//
//   k_scores_mfma     raw scores of every token against the query-folded key weights (MFMA)
//   k_softmax_alpha   softmax of the scores over the members of each group
//   k_vagg_mfma       value projection GEMM whose epilogue takes the softmax-weighted sum over
//                     the channels of the group, so that the projected values never leave the CU
//   k_product_dl      plain per-group products: output projections, their gradients, and the weight-only product
//                     Wv We[c] (value projection folded into the tokenizer weights)
//   k_scores_pixels*, k_compose_score_weights*   first-level scores straight from the pixels
//   k_tokenize_ws, k_tokenize_mfma               the per-channel tokenizer (paper Section 2.1)
//   k_tokenize_reduce_ring, k_tokenize_mix_*, k_tokenize_attend_wide   tokenizer fused with the first level
//                     (linear level of D-CHAG-L, or attention level with folded value weights): no tokens in HBM
//
// The large products share one core: 256x256 block tile, 8 wavefronts (2 x 4), 16x16x32 bf16
// MFMA, K staged in 64-element slices of four slots, two stages, each slot refilled by direct-to-LDS
// global loads of 128-byte row segments (no register staging; L2 delivers 128-byte segments at
// about twice the rate of 64-byte ones) and read with conflict-free swizzled or transposing LDS reads.
//
// Softmax weights are exchanged between the kernels in the layout
//   alpha[b][k][cl][head][n]   (n fastest, pitch Np = N rounded up to 32; cl < gpad = g rounded up to 8)
// with zeros for the padding members cl >= size of group k.
#pragma once
#include "dchag_dev.h"
#include "k_mfma.h"

namespace dchag {

typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// Wait until at most N vector-memory operations of this wavefront are outstanding
// (gfx9 s_waitcnt immediate: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[5:4] at [15:14]).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Each lane's 16 bytes of a wave-wide direct-to-LDS load land at lds_base + 16 * lane (lds_base is wave-uniform).
// Written as an asm statement on purpose: the compiler files the builtin under "flat access that may touch LDS and
// global memory", and while one is pending it turns every counted wait of the wavefront into a wait for zero, which
// serialises the LDS fragment reads of the GEMM loops.  The kernels order these loads themselves (wait_vmcnt + barrier
// before the stage is read; nothing outstanding when the block retires), so the compiler need not know them; the
// memory clobber keeps it from moving LDS or global accesses across the statement.
__device__ __forceinline__ void load16_to_lds(const void* src, void* lds_base) {
  const unsigned lds_off = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(lptr_t)lds_base);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_off), "v"(src) : "memory", "m0");
}

// LDS stages hold rows of 64 bf16 (128 bytes = 8 chunks of 16 bytes).  Chunk c of row r sits at chunk
// position c ^ ((r >> 1) & 7): the 16 consecutive rows a quarter-wavefront reads at one logical chunk
// then fall into 16 different 16-byte bank groups (64 banks x 4 bytes), so ds_read_b128 is conflict-free.
__device__ __forceinline__ int swz_chunk(int row) { return (row >> 1) & 7; }

constexpr int kGemmBM = 256, kGemmBN = 256, kGemmBK = 64, kGemmStages = 2;
constexpr int kGemmStageBytes = (kGemmBM + kGemmBN) * kGemmBK * 2;             // 64 KiB
constexpr int kGemmRingBytes = kGemmStages * kGemmStageBytes;                  // 128 KiB

// ---------------------------------------------------------------------------------------------
// Weight-only prep of attention levels (paper Section 2.1's cross-attention layer; the learned query is fixed, so its
// projection and its product with the key weights depend on the weights alone), one launch for any number of levels:
//   Q[k][i]    = sum_j Wq[k][i][j] query[k][j] + bq[k][i]
//   M[k][a][d] = (1 / sqrt(dh)) sum_{i in head a} Wk[k][i][d] Q[k][i]      (the key bias shifts every score of a softmax
//                                                                          equally and is dropped)
// so that the score of token z for head a is z . M[k][a][:].  grid (heads, all groups of all levels, column shares),
// block 256: a block of (head a, group k) first forms the dh entries of Q of its head (a wavefront per row of Wq, the
// rows dealt round-robin), leaves them in LDS (and, the first share, in Qp), then sums the dh rows of Wk of that head
// into its share of M's columns (fixed summation order).  Writes M as fp32 (Mf) and, where asked, bf16 (Mb) and
// transposed fp32 MfT[G][D][heads].  Requires dh % 4 == 0 and (D / shares) % 8 == 0.  Dynamic LDS: dh + 1536 floats.
// ---------------------------------------------------------------------------------------------
struct KeyPrepLevel {
  const void *query, *Wq, *bq, *Wk;
  float *Qp, *Mf, *MfT;
  bf16* Mb;
  int g_first;                     // index of this level's first group in the launch's group axis
};
constexpr int kKeyPrepMaxLevels = 16;
struct KeyPrepArgs {
  int n_levels;
  KeyPrepLevel lv[kKeyPrepMaxLevels];
};

template <typename T>
__global__ __launch_bounds__(256) void k_query_keys(int D, int heads, KeyPrepArgs args) {
  typedef T vec8 __attribute__((ext_vector_type(8), aligned(16)));
  extern __shared__ float qs[];                          // [dh] projected query of the head, then [3][512] partial sums
  const int a = blockIdx.x;
  int l = 0;
  while (l + 1 < args.n_levels && (int)blockIdx.y >= args.lv[l + 1].g_first) ++l;     // uniform over the block
  const KeyPrepLevel& P = args.lv[l];
  const T *Wq = static_cast<const T*>(P.Wq), *Wk = static_cast<const T*>(P.Wk), *bq = static_cast<const T*>(P.bq);
  const int k = blockIdx.y - P.g_first;
  const int dh = D / heads;
  float* part = qs + dh;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const T* q = static_cast<const T*>(P.query) + (size_t)k * D;
  const size_t row0 = (size_t)k * D + (size_t)a * dh;
  // Q of this head: wavefront w takes rows w, w + 4, ..., eight of them at a time so that their loads are in flight
  // together (every block of a head computes all of Q_a: the second block's reads come out of L2)
  for (int r0 = wave; r0 < dh; r0 += 32) {
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int j = lane * 8; j < D; j += kWave * 8) {
      const vec8 qv = *reinterpret_cast<const vec8*>(q + j);
      vec8 wv[8];
#pragma unroll
      for (int t = 0; t < 8; ++t)
        wv[t] = *reinterpret_cast<const vec8*>(Wq + (row0 + min(r0 + 4 * t, dh - 1)) * D + j);
#pragma unroll
      for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[t] += to_f32(wv[t][e]) * to_f32(qv[e]);
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const float v = wave_sum(acc[t]);
      const int r = r0 + 4 * t;
      if (lane == 0 && r < dh) {
        const float qv = v + (bq ? to_f32(bq[row0 + r]) : 0.f);
        if (blockIdx.z == 0) P.Qp[row0 + r] = qv;
        qs[r] = qv;
      }
    }
  }
  __syncthreads();
  // M of this head, this block's share of the columns: a lane takes eight adjacent columns (16-byte loads, eight rows
  // in flight), wavefront w the w-th quarter of the head's rows; the four partial sums meet in LDS in that order
  const float scale = rsqrtf((float)dh);
  const int qrows = dh / 4;
  const int cper = D / gridDim.z, cbeg = blockIdx.z * cper, cend = cbeg + cper;
  for (int c0 = cbeg; c0 < cend; c0 += 512) {
    const int d0 = c0 + lane * 8;
    const bool live = d0 < cend;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (live) {
      const T* w = Wk + (row0 + (size_t)wave * qrows) * D + d0;
      const float* qh = qs + wave * qrows;
#pragma unroll 8
      for (int r = 0; r < qrows; ++r) {
        const vec8 v = *reinterpret_cast<const vec8*>(w + (size_t)r * D);
        const float qr = qh[r];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += to_f32(v[e]) * qr;
      }
    }
    if (wave > 0) {
#pragma unroll
      for (int e = 0; e < 8; ++e) part[(wave - 1) * 512 + lane * 8 + e] = acc[e];
    }
    __syncthreads();
    if (wave == 0 && live) {
      const size_t o = ((size_t)k * heads + a) * D + d0;
      bf16x8 b8;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        acc[e] = (((acc[e] + part[lane * 8 + e]) + part[512 + lane * 8 + e]) + part[1024 + lane * 8 + e]) * scale;
        b8[e] = (bf16)acc[e];
      }
      *reinterpret_cast<f32x4*>(P.Mf + o) = f32x4{acc[0], acc[1], acc[2], acc[3]};
      *reinterpret_cast<f32x4*>(P.Mf + o + 4) = f32x4{acc[4], acc[5], acc[6], acc[7]};
      if (P.Mb) *reinterpret_cast<bf16x8*>(P.Mb + o) = b8;
      if (P.MfT) {
#pragma unroll
        for (int e = 0; e < 8; ++e) P.MfT[((size_t)k * D + d0 + e) * heads + a] = acc[e];
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------------
// Scores.  S[b][k][cl][head][n] = z[b, c, n, :] . Mb[k][head][:]   (c = k*g + cl)
// grid (ceil(N/16), G * ceil(g/4), B), block 256: a block takes 16 patches x 4 channels of one group; its
// four wavefronts each take a quarter of D (operands straight from global memory: 16 rows x 64 bytes per
// load for the tokens, the folded keys come from L2), and the partial 16x16 blocks meet in LDS in a
// fixed order.  The kernel is bound by the HBM read of the tokens (2*D bytes per token).
// Requires D % 128 == 0.
// ---------------------------------------------------------------------------------------------
template <int NB>   // head blocks of 16 (heads padded to 16 * NB)
__global__ __launch_bounds__(256) void k_scores_mfma(int Cin, int N, int D, int heads, int g, int gpad, int Np,
                                                     const bf16* __restrict__ z, const bf16* __restrict__ Mb,
                                                     float* __restrict__ S) {
  __shared__ float part[3][4 * NB * 4][64];
  const int qch = (g + 3) / 4;                         // channel quads per group
  const int k = blockIdx.y / qch, cq = blockIdx.y % qch;
  const int G = gridDim.y / qch;
  const int b = blockIdx.z, n0 = blockIdx.x * 16;
  const int c0 = k * g;
  const int gk = min(g, Cin - c0);                     // members of this group
  if (cq * 4 >= gk) return;                            // uniform: nothing in this quad
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, lq = lane >> 4;
  const int kq = D / 4, kbeg = wave * kq;
  const int n = min(n0 + l16, N - 1);

  const bf16* zrow[4];
  const bf16* mrow[NB];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    zrow[i] = z + (((size_t)b * Cin + c0 + min(cq * 4 + i, gk - 1)) * N + n) * D + kbeg + lq * 8;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
    mrow[nb] = Mb + ((size_t)k * heads + min(nb * 16 + l16, heads - 1)) * D + kbeg + lq * 8;

  f32x4 acc[4][NB];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[i][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int ks = 0; ks < kq; ks += 32) {
    bf16x8 bfr[NB], af[4];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      bfr[nb] = *reinterpret_cast<const bf16x8*>(mrow[nb] + ks);
      if (nb * 16 + l16 >= heads) bfr[nb] = bf16x8{};
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) af[i] = *reinterpret_cast<const bf16x8*>(zrow[i] + ks);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        acc[i][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bfr[nb], acc[i][nb], 0, 0, 0);
  }
  if (wave > 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int e = 0; e < 4; ++e) part[wave - 1][(i * NB + nb) * 4 + e][lane] = acc[i][nb][e];
  }
  __syncthreads();
  if (wave == 0) {
    // 16x16 accumulator block: lane holds head (lane % 16), patches 4 * (lane / 16) + 0..3
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int cl = cq * 4 + i;
      if (cl >= gk) continue;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int head = nb * 16 + l16;
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int slot = (i * NB + nb) * 4 + e;
          v[e] = acc[i][nb][e] + part[0][slot][lane] + part[1][slot][lane] + part[2][slot][lane];
        }
        if (head < heads) {
          float* dst = S + ((((size_t)b * G + k) * gpad + cl) * heads + head) * Np + n0 + lq * 4;
          *reinterpret_cast<f32x4*>(dst) = v;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Scores, group-resident form of the kernel above for D = 128 * KI (KI even): a block takes 16 patches and a
// run of whole channel quads of ONE group, so each wavefront loads its quarter of the folded keys once into
// registers (KI * NB operand fragments) and then only streams tokens; the token loads of the next 32-feature
// step are in flight while the current one is multiplied.  The four partial 16x16 blocks of a quad meet in
// LDS (two buffers, one barrier per quad) and wavefront w adds up and stores channel w of the quad, always in
// the order of the wavefronts.  grid (ceil(N/16), G * qsplit, B), block 256; part = blockIdx.y % qsplit takes
// quads [part * qper, (part + 1) * qper) of its group.  Bound by the HBM read of the tokens.
// ---------------------------------------------------------------------------------------------
template <int NB, int KI>
__global__ __launch_bounds__(256) void k_scores_group(int Cin, int N, int heads, int g, int gpad, int Np, int qsplit,
                                                      int qper, const bf16* __restrict__ z,
                                                      const bf16* __restrict__ Mb, float* __restrict__ S) {
  // one step = one 16-byte load per lane = 32 features of one channel; a quad takes 4 * KI steps, channel after
  // channel, so that a wavefront streams 16 rows x (D / 4) contiguous bytes of one channel before it moves on
  constexpr int STEPS = 4 * KI;
  constexpr int NBUF = STEPS < 8 ? STEPS : 8;            // NBUF - 1 loads in flight per lane
  constexpr int PD = NBUF - 1;
  static_assert(STEPS % NBUF == 0, "the fragment buffers rotate with the step index");
  constexpr int D = KI * 128;
  __shared__ float part[2][4][4][NB * 4][64];           // [buffer][source wavefront][channel of the quad]
  const int k = blockIdx.y / qsplit, prt = blockIdx.y % qsplit;
  const int G = gridDim.y / qsplit;
  const int b = blockIdx.z, n0 = blockIdx.x * 16;
  const int c0 = k * g;
  const int gk = min(g, Cin - c0);
  const int q_end = min((gk + 3) / 4, (prt + 1) * qper);
  const int q_begin = prt * qper;
  if (q_begin >= q_end) return;                          // uniform over the block
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, lq = lane >> 4;
  const int n = min(n0 + l16, N - 1);
  const int koff = wave * (D / 4) + lq * 16;
  // features of step ks (same for tokens and keys): the two steps of a pair read the two 16-byte halves of a
  // lane's 32 bytes, so that the four lanes of a row cover one 128-byte line with two back-to-back loads
  auto kstep = [](int ks) { return (ks >> 1) * 64 + (ks & 1) * 8; };

  bf16x8 bfr[KI][NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const bf16* mrow = Mb + ((size_t)k * heads + min(nb * 16 + l16, heads - 1)) * D + koff;
#pragma unroll
    for (int ks = 0; ks < KI; ++ks) {
      bfr[ks][nb] = *reinterpret_cast<const bf16x8*>(mrow + kstep(ks));
      if (nb * 16 + l16 >= heads) bfr[ks][nb] = bf16x8{};
    }
  }
  // tokens of channel cl of this group, this lane's patch and feature offset; members past the end of a
  // short group re-read the last member (their scores are never stored)
  const bf16* zb = z + (((size_t)b * Cin + c0) * N + n) * D + koff;
  const size_t cstride = (size_t)N * D;
  auto zptr = [&](int cl) { return zb + (size_t)min(cl, gk - 1) * cstride; };

  bf16x8 af[NBUF];
#pragma unroll
  for (int t = 0; t < PD; ++t) af[t] = *reinterpret_cast<const bf16x8*>(zptr(q_begin * 4 + t / KI) + kstep(t % KI));
  for (int q = q_begin; q < q_end; ++q) {
    const bf16* cur[4];
    const bf16* nxt[4];
    const int qn = min(q + 1, q_end - 1);                // past the last quad: re-read it (in bounds, unused)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      cur[i] = zptr(q * 4 + i);
      nxt[i] = zptr(qn * 4 + i);
    }
    f32x4 acc[4][NB];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[i][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
      const int tp = t + PD;                             // the step whose load is issued now
      af[tp % NBUF] = (tp < STEPS) ? *reinterpret_cast<const bf16x8*>(cur[tp / KI] + kstep(tp % KI))
                                   : *reinterpret_cast<const bf16x8*>(nxt[(tp - STEPS) / KI] + kstep((tp - STEPS) % KI));
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        acc[t / KI][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[t % NBUF], bfr[t % KI][nb], acc[t / KI][nb], 0, 0, 0);
    }
    const int pb = (q - q_begin) & 1;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int e = 0; e < 4; ++e) part[pb][wave][i][nb * 4 + e][lane] = acc[i][nb][e];
    __syncthreads();
    // 16x16 accumulator block: lane holds head (lane % 16), patches 4 * (lane / 16) + 0..3
    const int cl = q * 4 + wave;
    if (cl < gk) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int head = nb * 16 + l16;
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          v[e] = ((part[pb][0][wave][nb * 4 + e][lane] + part[pb][1][wave][nb * 4 + e][lane]) +
                  part[pb][2][wave][nb * 4 + e][lane]) + part[pb][3][wave][nb * 4 + e][lane];
        if (head < heads) {
          float* dst = S + ((((size_t)b * G + k) * gpad + cl) * heads + head) * Np + n0 + lq * 4;
          *reinterpret_cast<f32x4*>(dst) = v;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Scores and softmax in one kernel, for heads <= 16 and D % 256 == 0: a block takes 32 patches and ALL members
// of one group, so the raw scores stay in LDS and only the softmax weights are written (128-byte runs).
// The folded keys of the group sit in LDS (rows padded by 16 bytes: conflict-free ds_read_b128).  Wavefront w
// streams whole token rows of members w, w + 8, ...: per step two 16-row fragments (patches 0..15 and 16..31,
// 64 contiguous bytes per row and load) that share one key fragment, with the loads of the next seven steps in
// flight; no cross-wavefront reduction is needed.  After one barrier thread (head, patch) takes the softmax
// over the members and writes alpha, zeros for padding members and padding patches.
// grid (Np / 32, G, B), block 512, dynamic LDS 16 * (2 D + 16) + gpad * 2048 bytes.
// Bound by the HBM read of the tokens.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(512) void k_scores_softmax(int Cin, int N, int D, int heads, int g, int gpad, int Np,
                                                        const bf16* __restrict__ z, const bf16* __restrict__ Mb,
                                                        float* __restrict__ alpha) {
  constexpr int NBUF = 8, PD = NBUF - 1;                 // PD steps of loads in flight per lane and fragment
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int krow = D * 2 + 16;                           // bytes of one padded key row
  float* sc = reinterpret_cast<float*>(smem + 16 * krow);   // [gpad][16 heads][32 patches]
  const int k = blockIdx.y, G = gridDim.y, b = blockIdx.z, n0 = blockIdx.x * 32;
  const int c0 = k * g;
  const int gk = min(g, Cin - c0);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, lq = lane >> 4;
  const int KF = D / 32;

  for (int idx = threadIdx.x; idx < 16 * (D / 8); idx += 512) {
    const int head = idx / (D / 8), c = idx % (D / 8);
    bf16x8 v = {};
    if (head < heads) v = *reinterpret_cast<const bf16x8*>(Mb + ((size_t)k * heads + head) * D + c * 8);
    *reinterpret_cast<bf16x8*>(smem + head * krow + c * 16) = v;
  }
  __syncthreads();

  if (wave < gk) {
    const bf16* zb0 = z + (((size_t)b * Cin + c0) * N + min(n0 + l16, N - 1)) * D + lq * 8;
    const bf16* zb1 = z + (((size_t)b * Cin + c0) * N + min(n0 + 16 + l16, N - 1)) * D + lq * 8;
    const size_t cstride = (size_t)N * D;
    const unsigned char* kfrag = smem + l16 * krow + lq * 16;
    const int last = wave + ((gk - 1 - wave) / 8) * 8;     // this wavefront's last member
    bf16x8 a0[NBUF], a1[NBUF];
#pragma unroll
    for (int t = 0; t < PD; ++t) {
      a0[t] = *reinterpret_cast<const bf16x8*>(zb0 + (size_t)wave * cstride + t * 32);
      a1[t] = *reinterpret_cast<const bf16x8*>(zb1 + (size_t)wave * cstride + t * 32);
    }
    for (int cl = wave; cl < gk; cl += 8) {
      const size_t co = (size_t)cl * cstride;
      const size_t no = (size_t)min(cl + 8, last) * cstride - (size_t)KF * 32;   // past the end: re-read (unused)
      f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
      for (int tb = 0; tb < KF; tb += NBUF) {
#pragma unroll
        for (int u = 0; u < NBUF; ++u) {
          const int t = tb + u, tp = t + PD;               // tp: the step whose loads are issued now
          const size_t off = (tp < KF ? co : no) + (size_t)tp * 32;
          a0[(u + PD) % NBUF] = *reinterpret_cast<const bf16x8*>(zb0 + off);
          a1[(u + PD) % NBUF] = *reinterpret_cast<const bf16x8*>(zb1 + off);
          const bf16x8 kf = *reinterpret_cast<const bf16x8*>(kfrag + t * 64);
          acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0[u], kf, acc0, 0, 0, 0);
          acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1[u], kf, acc1, 0, 0, 0);
        }
      }
      // 16x16 accumulator block: lane holds head (lane % 16), patches 4 * (lane / 16) + 0..3
      *reinterpret_cast<f32x4*>(&sc[(cl * 16 + l16) * 32 + lq * 4]) = acc0;
      *reinterpret_cast<f32x4*>(&sc[(cl * 16 + l16) * 32 + 16 + lq * 4]) = acc1;
    }
  }
  __syncthreads();
  const int head = threadIdx.x >> 5, patch = threadIdx.x & 31;
  if (head >= heads) return;
  const int n = n0 + patch;
  const size_t stride = (size_t)heads * Np;
  float* p = alpha + ((((size_t)b * G + k) * gpad) * heads + head) * Np + n;
  if (n >= N) {                                            // pitch padding: never scored, weight zero
    for (int cl = 0; cl < gpad; ++cl) p[cl * stride] = 0.f;
    return;
  }
  const float* s = sc + head * 32 + patch;
  float mx = -INFINITY;
  for (int cl = 0; cl < gk; ++cl) mx = fmaxf(mx, s[cl * 512]);
  float den = 0.f;
  for (int cl = 0; cl < gk; ++cl) den += __expf(s[cl * 512] - mx);
  const float inv = 1.f / den;
  for (int cl = 0; cl < gk; ++cl) p[cl * stride] = __expf(s[cl * 512] - mx) * inv;
  for (int cl = gk; cl < gpad; ++cl) p[cl * stride] = 0.f;
}

// ---------------------------------------------------------------------------------------------
// In-place softmax over the members of a group: S[b][k][0..gk)[head][n] -> alpha, zeros for cl >= gk.
// grid (ceil(Np/256), heads, B*G), block 256; one thread per (b, k, head, n).
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_softmax_alpha(int Cin, int N, int heads, int g, int gpad, int G, int Np,
                                                       float* __restrict__ S) {
  const int n = blockIdx.x * 256 + threadIdx.x;
  if (n >= Np) return;
  const int head = blockIdx.y;
  const int k = blockIdx.z % G;
  const int gk = min(g, Cin - k * g);
  const size_t stride = (size_t)heads * Np;
  float* p = S + ((size_t)blockIdx.z * gpad * heads + head) * Np + n;
  if (n >= N) {                                          // pitch padding: never scored, weight zero
    for (int cl = 0; cl < gpad; ++cl) p[cl * stride] = 0.f;
    return;
  }
  if (gk <= 32) {
    // the whole group in registers: all loads of the thread are in flight together, one pass over memory each way
    // (same arithmetic and order as the loop below)
    float v[32];
#pragma unroll
    for (int cl = 0; cl < 32; ++cl) v[cl] = cl < gk ? p[cl * stride] : -INFINITY;
    float mx = -INFINITY;
#pragma unroll
    for (int cl = 0; cl < 32; ++cl) mx = fmaxf(mx, v[cl]);
    float den = 0.f;
#pragma unroll
    for (int cl = 0; cl < 32; ++cl)
      if (cl < gk) den += __expf(v[cl] - mx);
    const float inv = 1.f / den;
#pragma unroll
    for (int cl = 0; cl < 32; ++cl)
      if (cl < gk) p[cl * stride] = __expf(v[cl] - mx) * inv;
    for (int cl = gk; cl < gpad; ++cl) p[cl * stride] = 0.f;
    return;
  }
  float mx = -INFINITY;
  for (int cl = 0; cl < gk; ++cl) mx = fmaxf(mx, p[cl * stride]);
  float den = 0.f;
  for (int cl = 0; cl < gk; ++cl) den += __expf(p[cl * stride] - mx);
  const float inv = 1.f / den;
  for (int cl = 0; cl < gk; ++cl) p[cl * stride] = __expf(p[cl * stride] - mx) * inv;
  for (int cl = gk; cl < gpad; ++cl) p[cl * stride] = 0.f;
}

// ---------------------------------------------------------------------------------------------
// The 256 x 256 x 64 core of the large products (k_vagg_mfma, k_product_dl).
//
// Instruction: v_mfma_f32_16x16x32.  These kernels run into the card's power limit, so what counts is the work done per joule:
// a loop of nothing but products on normally distributed operands reaches 1.93 PFLOP/s with 16x16x32 and 1.35 with
// 32x32x16 (2.45 and 1.65 on constant operands; 256 x 8 wavefronts, a 128 x 64 tile each).
//
// Eight wavefronts (2 x 4).  A stage of the ring holds one slice of 64 contraction elements as four slots of 16 KiB (128
// rows x 128 bytes, swizzled): A0, A1 (tile rows 0..127, 128..255) and B0, B1; two stages.  Wavefront (wm, wn) owns rows
// [64 wm, +64) of BOTH A slots and columns [32 wn, +32) of BOTH B slots, so that a slice is four phases of sixteen
// products, one per pair of slots: (A0,B0) (A0,B1) (A1,B1) (A1,B0).  Each phase reads the fragments of ONE slot,
// the one whose first use comes next (B1, A1, the next slice's A0, the next slice's B0): after the phase's barrier that slot
// holds nothing anybody needs and takes its rows of the slice after the next one.  So seven slots (112 KiB) are on their
// way at any time and a load has seven phases (1.75 slices) to arrive; a stage handed over as a whole leaves it one slice.
// The barrier of a phase sits in front of its last products, which cover it; every wait is a counted one (vmcnt 12: all but
// the six youngest slots).
// ---------------------------------------------------------------------------------------------
constexpr int kSlotBytes = 128 * 128;                    // A stages at 0 and 2 slots, B stages at 4 and 6 slots
enum CoreSlot { kSlotA0 = 0, kSlotA1 = 1, kSlotB0 = 4, kSlotB1 = 5 };

// A copy that the compiler knows nothing about: what is computed from it is computed where it is used.  The fragments and
// sums need every register of the loops, so what a loop needs rarely is formed again instead of being kept (lane_id: the lane's
// number, from no register at all).
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}
__device__ __forceinline__ int lane_id() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

struct CoreLane {
  int wave, wm, wn;
  int a_ad, b_ad;                                        // byte of this lane's first fragment in A0 / B0, stage 0
  template <class OA, class OB>
  __device__ __forceinline__ void init() {
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform: lives in a scalar register
    wm = wave >> 2;
    wn = wave & 3;
    a_ad = OA::base(wm * 64, lane_id());
    b_ad = 4 * kSlotBytes + OB::base(wn * 32, lane_id());
  }
  // Wavefront w fills rows 16 w + 8 u + lane / 8 (u = 0, 1) of a RowOperand's slot; the byte of the chunk that belongs there:
  static __device__ __forceinline__ int ld_chunk(int lane, int u) { return ((lane & 7) ^ swz_chunk(u * 8 + (lane >> 3))) * 16; }
};

// 16 bytes a lane from base + voff (base wave-uniform) to lds_off + 16 * lane; an asm statement for the reason given at
// load16_to_lds.
__device__ __forceinline__ void load16_to_lds_at(const void* base, unsigned voff, unsigned lds_off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_off), "v"(voff), "s"(base) : "memory", "m0");
}

struct CoreFrags {
  bf16x8 a0[4][2], a1[4][2], bx[2][2], by[2][2];         // [block][k-step]; bx / by: B0 / B1 of an even slice, B1 / B0 of an odd one
};
typedef f32x4 CoreAcc[2][4][2][2];                       // [A slot][block of 16 rows][B slot][block of 16 columns]

// How an operand lies in its slots, and how a fragment (16 of its rows or columns x 32 contraction elements, eight to a lane)
// of block blk and k-step kk is read; base: the lane's address for block 0 and k-step 0 of the wavefront's part of slot 0.
//
// RowOperand: rows of 64 contraction elements, 128 rows a slot.  k-step kk flips bit 6 of the address (its chunk is
// (4 kk + lane / 16) ^ swizzle).
struct RowOperand {
  static __device__ __forceinline__ int base(int part, int lane) {
    const int l16 = lane & 15;
    return (part + l16) * 128 + ((lane >> 4) ^ swz_chunk(l16)) * 16;         // part: a multiple of 16
  }
  static __device__ __forceinline__ bf16x8 frag(const unsigned char* smem, int ad, int blk, int kk, int imm) {
    return *reinterpret_cast<const bf16x8*>(smem + (opaque(ad) ^ (kk * 64)) + imm + blk * 2048);
  }
};
// ColOperand: the contraction index runs over the rows, PITCH / 2 of the operand's columns to a row (128 columns and all 64
// contraction elements a slot, or 64 columns of two matrices).  ds_read_b64_tr_b16 transposes on the way: lane l of 16 names
// four columns (l % 4) of contraction row l / 4 and receives column l of the four rows; two of them make the lane's eight
// elements.  The chunk swizzle is twice f(row), f one of PITCH / 32 values, so that the eight rows (0..3 and 8..11, 4..7 and
// 12..15) that half a wavefront reads at one pair of chunks lie in different banks; block blk flips bits 5 and 6.
template <int PITCH>
struct ColOperand {
  static __device__ __forceinline__ int swz(int row) {
    return PITCH == 256 ? ((row & 3) | ((row >> 3) & 1) << 2) * 2 : (((row >> 1) & 1) | ((row >> 3) & 1) << 1) * 2;
  }
  static __device__ __forceinline__ int base(int part, int lane) {
    const int l16 = lane & 15, row = (lane >> 4) * 8 + (l16 >> 2);
    const int first = PITCH == 256 ? 0 : (part >> 6) * 64 * 128, col = PITCH == 256 ? part : part & 63;
    return first + row * PITCH + (((col >> 3) + ((l16 & 3) >> 1)) ^ swz(row)) * 16 + (l16 & 1) * 8;
  }
  static __device__ __forceinline__ bf16x8 frag(const unsigned char* smem, int ad, int blk, int kk, int imm) {
    typedef __attribute__((ext_vector_type(4))) short s16x4;
    typedef __attribute__((ext_vector_type(8))) short s16x8;
    typedef __attribute__((address_space(3))) s16x4* tptr;
    const unsigned char* p = smem + (opaque(ad) ^ (blk * 32)) + imm + kk * 32 * PITCH;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tptr)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tptr)(p + 4 * PITCH));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
};

// One phase: c += a x b over the slice; the reads of the next phase's slot (NR of them, rd(t)) behind the first products,
// the hand-over (wait, barrier) in front of the last four, the loads behind the third of these: the matrix units then start again right behind
// the barrier, on either wavefront of a SIMD, instead of behind the loads' address and m0 instructions.  (Loads right behind the barrier, us, value
// product: 64 members x 64 patches, D 1024 (8 workgroups) 166 -> 150; 256 items of 4 chunks 105 -> 100; 1024 items 407 -> 392.  Loads behind the
// first, second, fourth of the four: 158, 153, 150 of the first.)  SWAP multiplies b x a, which leaves the transposed block: a
// lane then holds one tile row and four adjacent columns.
template <bool FIRST, bool SWAP, int NR, int HA, int HB, class Read, class Issue>
__device__ __forceinline__ void core_phase(CoreAcc& acc, const bf16x8 (&a)[4][2], const bf16x8 (&b)[2][2], Read rd, Issue issue) {
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int m = 0; m < 16; ++m) {
    const int kk = m >> 3, i = (m >> 1) & 3, j = m & 1;
    f32x4& c = acc[HA][i][HB][j];
    if (m == 12) {
      __builtin_amdgcn_s_waitcnt((12 & 15) | (0 << 14) | (7 << 4) | (0 << 8));   // vmcnt(12) lgkmcnt(0)
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    }
    if (SWAP) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j][kk], a[i][kk], FIRST && kk == 0 ? zero : c, 0, 0, 0);
    else c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i][kk], b[j][kk], FIRST && kk == 0 ? zero : c, 0, 0, 0);
    if (m < 8) {
#pragma unroll
      for (int t = m * NR / 8; t < (m + 1) * NR / 8; ++t) rd(t);
    }
    if (m == 14) issue();
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Slice of stage S (0 even, 1 odd).  issue(slot constant): the next pair of loads of that slot (see CoreSlot).  In stage 1 the
// roles of bx and by are exchanged.  held(slot, fragments): called once a slice with all fragments of A0, and of A1.
template <bool FIRST, bool SWAP, int S, class OA, class OB, class Issue, class Held>
__device__ __forceinline__ void core_slice(CoreAcc& acc, CoreFrags& f, const unsigned char* smem, const CoreLane& L, Issue issue,
                                           Held held) {
  bf16x8 (&b0)[2][2] = S ? f.by : f.bx;
  bf16x8 (&b1)[2][2] = S ? f.bx : f.by;
  constexpr int here = S * 2 * kSlotBytes, next = (S ^ 1) * 2 * kSlotBytes;
  core_phase<FIRST, SWAP, 4, 0, 0>(acc, f.a0, b0,
      [&](int t) { b1[t & 1][t >> 1] = OB::frag(smem, L.b_ad, t & 1, t >> 1, here + kSlotBytes); },
      [&]() { issue(kSlotB1 + 2 * S); });
  held(0, f.a0);
  core_phase<FIRST, SWAP, 8, 0, 1>(acc, f.a0, b1,
      [&](int t) { f.a1[t & 3][t >> 2] = OA::frag(smem, L.a_ad, t & 3, t >> 2, here + kSlotBytes); },
      [&]() { issue(kSlotA1 + 2 * S); });
  core_phase<FIRST, SWAP, 8, 1, 1>(acc, f.a1, b1,
      [&](int t) { f.a0[t & 3][t >> 2] = OA::frag(smem, L.a_ad, t & 3, t >> 2, next); },
      [&]() { issue(kSlotA0 + 2 * (S ^ 1)); });
  held(1, f.a1);
  core_phase<FIRST, SWAP, 4, 1, 0>(acc, f.a1, b0,
      [&](int t) { b1[t & 1][t >> 1] = OB::frag(smem, L.b_ad, t & 1, t >> 1, next); },
      [&]() { issue(kSlotB0 + 2 * (S ^ 1)); });
}

// Fills the ring and reads the first slice's A0 and B0.  Slots are issued in the order A0 B0 B1 A1 of slice 0, of slice 1,
// then A0 B0 of slice 2; the phases go on with B1 A1 A0 B0 ...
template <class OA, class OB, class Issue>
__device__ __forceinline__ void core_prologue(CoreFrags& f, const unsigned char* smem, const CoreLane& L, Issue issue) {
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    issue(kSlotA0 + 2 * s);
    issue(kSlotB0 + 2 * s);
    issue(kSlotB1 + 2 * s);
    issue(kSlotA1 + 2 * s);
  }
  wait_vmcnt<12>();
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int t = 0; t < 8; ++t) f.a0[t & 3][t >> 2] = OA::frag(smem, L.a_ad, t & 3, t >> 2, 0);
#pragma unroll
  for (int t = 0; t < 4; ++t) f.bx[t & 1][t >> 1] = OB::frag(smem, L.b_ad, t & 1, t >> 1, 0);
  __builtin_amdgcn_s_waitcnt((10 & 15) | (0 << 14) | (7 << 4) | (0 << 8));       // vmcnt(10) lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  issue(kSlotA0);
  issue(kSlotB0);
  __builtin_amdgcn_sched_barrier(0);
}

// ---------------------------------------------------------------------------------------------
// Value projection with the channel aggregation in its epilogue:
//   O[b,k,n,o] = sum_{cl < gk} alpha[b][k][cl][head(o)][n] * (z[b, k*g + cl, n, :] . Wv[k][o][:]) + bv[k][o]
// Work item (decoded by TileWork with m = patch tile): group k, batch b, 32 patches, 256 columns; the group
// is walked in chunks of 8 channels.  Tile row 128 h + 64 wm + 16 i + l holds channel 4h + i of the chunk, patch
// 16*wm + l, so wavefront (wm, wn) sees all 8 channels of ITS 16 patches, a channel to a block of rows: the weighted
// sum over the channels stays inside the wavefront's registers and no cross-wavefront merge is needed.
// The kernel is persistent: workgroup L takes items L/8, L/8 + slots, ... of its XCD's contiguous
// range, and the ring keeps prefetching across chunk and item boundaries.
// Requires D % 256 == 0, dh = D / heads a multiple of 32, and 256 % dh == 0 or dh % 256 == 0.
// Held down by the card's power limit where the chip is full: at 512 channels, D 1024, B 4, N 256 790 us with the matrix units busy 73 % of the
// cycles at 1.88 GHz (a library product of as many flops: 674 us, 88 % at 1.76 GHz; 32x32x16 instructions and whole stages before:
// 865 us, 68 % at 1.79 GHz).  Its loads alone take 519 us, its products and LDS reads without loads 683.
// WIDE: 64-bit addresses for the softmax weights, whose eight channels of a chunk lie heads Np floats apart (host: vagg_wide).  It spills a
// register, which the narrow one does not: level of 4 x 1000 channels, 300 patches, D 256 451 us instead of 441.
// Dynamic LDS: ring (128 KiB) + 3 alpha tiles of 8 * NHS * 32 floats, used round-robin by chunk.
// ---------------------------------------------------------------------------------------------
struct VaggItem {
  int k, b, n0, o0, c0, gk, nch, h0, ch0, split;
};

template <bool WIDE>
__global__ __launch_bounds__(512) void k_vagg_mfma(int Cin, int N, int D, int heads, int g, int gpad, int G, int Np,
                                                   TileWork tw, int slots, const bf16* __restrict__ z,
                                                   const bf16* __restrict__ Wv, const bf16* __restrict__ bv,
                                                   const float* __restrict__ alpha, bf16* __restrict__ O, int S,
                                                   float* __restrict__ Opart) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int KT = D / kGemmBK;                            // a multiple of 4: every chunk starts in stage 0
  const int dh = D / heads;
  const int NHS = dh >= kGemmBN ? 1 : kGemmBN / dh;      // heads inside a 256-column slice
  const int nhs_log = __builtin_ctz(NHS);                // dh is 32, 64, 128 or a multiple of 256: NHS is a power of two
  const int hsh = 8 - nhs_log;                           // log2 of the columns of a head inside the slice
  unsigned char* alds = smem + kGemmRingBytes;           // 3 tiles of [8][NHS][32] floats
  const int atile = 8 * NHS * 32 * 4;

  // this workgroup's items: w = xcd * per + t * slots + slot, t = 0, 1, ...
  const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
  const int per = (tw.total + kXcds - 1) / kXcds;
  const int xcd_end = min((xcd + 1) * per, tw.total);
  auto item_of = [&](int t, VaggItem& it) -> bool {
    const int w = xcd * per + t * slots + slot;
    if (w >= xcd_end) return false;
    int pt, nt;
    it.split = w % S;                                    // the group's chunks are dealt to S items (S <= chunks of any group)
    tw.decode_linear(w / S, it.k, it.b, pt, nt);
    it.n0 = pt * 32;
    it.o0 = nt * kGemmBN;
    it.c0 = it.k * g;
    it.gk = min(g, Cin - it.c0);
    const int nch = (it.gk + 7) / 8;
    it.ch0 = it.split * nch / S;
    it.nch = (it.split + 1) * nch / S - it.ch0;
    it.h0 = it.o0 / dh;
    return true;
  };

  CoreLane L;
  L.init<RowOperand, RowOperand>();
  const unsigned smem_off = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(lptr_t)smem);
  const unsigned wave_off = smem_off + L.wave * 2048;    // this wavefront's 16 rows of a slot

  // ---- issue side: the wavefront's 16 rows of slot A_h are channel 4h + w % 4 of the chunk, patches 16 (w / 4) .. + 15 ----
  VaggItem ic, nx;                                       // the item that is multiplied, and the next chunk's
  if (!item_of(0, ic)) return;                           // uniform: the whole workgroup has nothing to do
  struct Src {
    const bf16 *a0, *a1, *b0, *b1;                       // origins of a chunk's tile in its running slice, per slot
    const float* al;                                     // its softmax weights
    int n0;
  } run, nxt;
  const long nd = (long)N * D;                           // elements of a channel
  auto source = [&](const VaggItem& it, int chunk, Src& s) {
    const int cl = (it.ch0 + chunk) * 8;
    const bf16* zb = z + ((size_t)it.b * Cin * N + it.n0) * D;
    s.a0 = zb + (size_t)(it.c0 + min(cl + (L.wave & 3), it.gk - 1)) * N * D;
    s.a1 = zb + (size_t)(it.c0 + min(cl + (L.wave & 3) + 4, it.gk - 1)) * N * D;
    s.b0 = Wv + ((size_t)it.k * D + it.o0 + L.wave * 16) * D;
    s.b1 = s.b0 + (size_t)128 * D;
    s.al = alpha + ((((size_t)it.b * G + it.k) * gpad + cl) * heads + it.h0) * Np + it.n0;
    s.n0 = it.n0;
  };
  unsigned a_off[2];                                     // byte of a lane's 16 behind those origins
  auto patch_rows = [&](int n0) {
    const int lane = lane_id();
#pragma unroll
    for (int u = 0; u < 2; ++u)
      a_off[u] = (unsigned)(min(n0 + 16 * (L.wave >> 2) + u * 8 + (lane >> 3), N - 1) - n0) * D * 2 + L.ld_chunk(lane, u);
  };
  const int b_off = (lane_id() >> 3) * D * 2 + L.ld_chunk(lane_id(), 0);  // eight rows further: bit 6 (the chunk's) flips, 16 D bytes
  source(ic, 0, nxt);
  run = nxt;
  patch_rows(run.n0);
  int ki = 0, gci = 0;                                   // slices issued of the chunk, running chunk count (alpha buffer)
  auto issue = [&](int sl) {                             // sl: a constant once inlined
    const unsigned dst = wave_off + sl * kSlotBytes;
    const int kind = sl & ~2;
    if (sl == kSlotA0 && ki == 0 && L.wave < NHS) {      // entering a chunk (its slices are even in number): its softmax weights
      const int l = lane_id(), sgm = L.wave * 8 + (l >> 3);   // segment = (channel of the chunk, head of the slice)
      const unsigned row = (unsigned)((sgm >> nhs_log) * heads + (sgm & (NHS - 1)));
      if constexpr (WIDE) load16_to_lds(run.al + (size_t)row * Np + (l & 7) * 4, alds + (gci % 3) * atile + L.wave * 1024);
      else load16_to_lds_at(run.al, (row * Np + (l & 7) * 4) * 4, smem_off + kGemmRingBytes + (gci % 3) * atile + L.wave * 1024);
    }
    const bf16*& p = kind == kSlotA0 ? run.a0 : kind == kSlotA1 ? run.a1 : kind == kSlotB0 ? run.b0 : run.b1;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (kind == kSlotA0 || kind == kSlotA1) load16_to_lds_at(p, a_off[u], dst + u * 1024);
      else load16_to_lds_at(p + (size_t)u * 8 * D, opaque(b_off) ^ (u * 64), dst + u * 1024);
    }
    p += kGemmBK;
    if (sl == kSlotA1 + 2) {                             // the last slot of an odd slice
      ki += 2;
      if (ki == KT) {
        ki = 0;
        ++gci;
        run = nxt;
        patch_rows(run.n0);
      }
    }
  };

  // ---- compute side ----
  auto nothing = [](int, const bf16x8 (&)[4][2]) {};
  CoreFrags f;
  core_prologue<RowOperand, RowOperand>(f, smem, L, issue);
  f32x4 o[2][2];
#pragma unroll
  for (int j = 0; j < 4; ++j) o[j >> 1][j & 1] = f32x4{0.f, 0.f, 0.f, 0.f};
  int t = 0, chunk = 0, gcc = 0;
  for (;;) {
    nx = ic;
    int nchunk = chunk + 1;
    bool more = true;
    if (nchunk == ic.nch) {
      nchunk = 0;
      more = item_of(++t, nx);                           // past the last item: this one again, loaded and not used
    }
    if (nchunk == 0) source(nx, nchunk, nxt);
    else {                                               // the same rows of eight channels further (D 256, 2 workgroups: 51.6 -> 50.1 us)
      const int cl = (ic.ch0 + nchunk) * 8, was = cl - 8;
      const int s0 = min(cl + (L.wave & 3), ic.gk - 1) - min(was + (L.wave & 3), ic.gk - 1);
      const int s1 = min(cl + (L.wave & 3) + 4, ic.gk - 1) - min(was + (L.wave & 3) + 4, ic.gk - 1);
      nxt.a0 += s0 * nd;
      nxt.a1 += s1 * nd;
      nxt.al += (size_t)8 * heads * Np;
    }
    {
      CoreAcc acc;
      core_slice<true, false, 0, RowOperand, RowOperand>(acc, f, smem, L, issue, nothing);
      core_slice<false, false, 1, RowOperand, RowOperand>(acc, f, smem, L, issue, nothing);
      for (int kt = 2; kt < KT; kt += 2) {
        core_slice<false, false, 0, RowOperand, RowOperand>(acc, f, smem, L, issue, nothing);
        core_slice<false, false, 1, RowOperand, RowOperand>(acc, f, smem, L, issue, nothing);
      }
      // o += alpha * acc over the 8 channels of the chunk
      const float* al = reinterpret_cast<const float*>(alds + (gcc % 3) * atile) + 16 * L.wm + 4 * (lane_id() >> 4);
#pragma unroll
      for (int hb = 0; hb < 2; ++hb) {
        const float* ap = al + ((hb * 128 + L.wn * 32) >> hsh) * 32;   // head inside the slice: dh divides 256 or is a multiple of it
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const f32x4 a4 = *reinterpret_cast<const f32x4*>(ap + c * NHS * 32);
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[hb][j][e] += a4[e] * acc[c >> 2][c & 3][hb][j][e];
        }
      }
    }
    ++gcc;
    if (nchunk != 0) {
      chunk = nchunk;
      continue;
    }
    const size_t first = S == 1 ? (((size_t)ic.b * G + ic.k) * N) * D
                                : ((((size_t)ic.split * tw.nb + ic.b) * G + ic.k) * N) * D;   // S > 1: partial sums, added up by k_vagg_merge
    // lane (l16, lq): patches 4 lq + e of the wavefront's 16, columns 128 hb + 32 wn + 16 j + l16.  One mask a patch and one choice of the
    // target; offsets opaque, so that none is formed ahead and kept in a register through the loops.  (A mask and a choice an element, two bytes
    // a store: 3 x 559 channels of 42 in groups of 13, D 256, level 72.2 -> 70.8 us; 80 channels of 512 in groups of 8, D 512, 65.0 -> 63.6.)
    const int lane = lane_id(), row = 4 * (lane >> 4), left = N - ic.n0 - 16 * L.wm;
    const size_t origin = first + (size_t)(ic.n0 + 16 * L.wm) * D + ic.o0 + L.wn * 32;
    const int at = opaque(row * D + (lane & 15));
    if (S > 1) {
      float* P = Opart + origin + at;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (row + e < left) {
#pragma unroll
          for (int j = 0; j < 4; ++j) P[(size_t)e * D + (j >> 1) * 128 + (j & 1) * 16] = o[j >> 1][j & 1][e];
        }
    } else {
      float bias[4] = {0.f, 0.f, 0.f, 0.f};
      if (bv) {
        const bf16* bp = bv + (size_t)ic.k * D + ic.o0 + L.wn * 32 + opaque(lane & 15);
#pragma unroll
        for (int j = 0; j < 4; ++j) bias[j] = (float)bp[(j >> 1) * 128 + (j & 1) * 16];
      }
      bf16* P = O + origin + at;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (row + e < left) {
#pragma unroll
          for (int j = 0; j < 4; ++j) P[(size_t)e * D + (j >> 1) * 128 + (j & 1) * 16] = (bf16)(o[j >> 1][j & 1][e] + bias[j]);
        }
    }
    if (!more) break;
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j >> 1][j & 1] = f32x4{0.f, 0.f, 0.f, 0.f};
    ic = nx;
    chunk = 0;
  }
  wait_vmcnt<0>();                                       // nothing may still target LDS when the block retires
}

// O[b,k,n,:] = sum over the S partial sums of k_vagg_mfma + bv[k][:], in a fixed order.  One thread per 4 columns.
__global__ __launch_bounds__(256) void k_vagg_merge(long quads, int S, int G, int N, int D, long per_split,
                                                    const float* __restrict__ Opart, const bf16* __restrict__ bv,
                                                    bf16* __restrict__ O) {
  const long q = (long)blockIdx.x * 256 + threadIdx.x;
  if (q >= quads) return;
  const long i = q * 4;                                  // ((b * G + k) * N + n) * D + col
  const int col = (int)(i % D);
  const int k = (int)((i / ((long)N * D)) % G);
  f32x4 acc = *reinterpret_cast<const f32x4*>(Opart + i);
  for (int sidx = 1; sidx < S; ++sidx) acc += *reinterpret_cast<const f32x4*>(Opart + sidx * per_split + i);
  bf16x4 out;
#pragma unroll
  for (int e = 0; e < 4; ++e) out[e] = (bf16)(acc[e] + (bv ? (float)bv[(size_t)k * D + col + e] : 0.f));
  *reinterpret_cast<bf16x4*>(O + i) = out;
}

// ---------------------------------------------------------------------------------------------
// Batched bf16 products on the same core, persistent over 256 x 256 tiles of the (group k, batch b, row tile, column tile)
// order as k_vagg_mfma is over its items; the operands of each instruction are exchanged, so that a lane ends with one row and
// four adjacent columns of a block, trades with lane ^ 16 and stores 16 bytes at a time (16 stores a lane for its tile).
//   kProductLinear   C[r][o] = sum_j A[r][j] B[k][o][j] + bias[k][o] (+ rowadd[r][o])      an output projection
//   kProductBack     C[r][j] = sum_o A[r][o] B[k][o][j]                                     the gradient at its input
//   kProductWeights  C[k][i][j] = sum_{b,n} A[b,k,n,i] B[b,k,n,j], rowsum[k][i] = sum_{b,n} A[b,k,n,i]
//                                                                                            its weight and bias gradients
//   kProductFold     C[c][o][kk] = sum_d A[k][o][d] B[c][d][kk], 64 kk, k = c / g           value weights into the tokenizer's
//   kProductImage    image[b][c][pixel kk of patch n] = sum_d A[c][d][kk] B[b,k,n][d]        pixel gradients of a linear first level
//   kProductOuter    P[c, kk][d] = sum_{b,n} u[b,c,n,kk] B[b,k,n][d], u: the 8 x 8 patches of the image A, which leaves as the linear
//                    first level's gradients (see k_linear_outer)
// us, 512 bands, 4 x 256 patches, D 1024, 128 x 256 tiles of pair_loop before: Outer 129 and 37 for the copies it read / 116 (of it
// about 55 for its epilogue, which moves 200 MB), Image 88 / 60.
// The last two have tile rows (member, pixel), a member to a wavefront and slot, and multiply in plain order: a lane holds one column
// and four adjacent pixels a block.  Outer reads its patches straight from the image, 16 bytes a lane (the eight pixel rows of two
// members are the 16 chunks of a slot's row).
// Rows of A of a group may be ragged (Linear, Back: loads clamped, stores masked); every other extent is a multiple of 256,
// of 64 kt slices of the contraction kt is even and at least 4, and every row is 16-byte aligned (host).  An operand whose
// contraction index is its row index is read by the transposing LDS reads (ColOperand): no transposed copy, no 2-byte reads.
// Bound by the card's power limit where there are many tiles (the clock falls to 1.7 to 1.9 GHz) and by the last round of tiles.
// One workgroup a tile, 2-byte stores and 32x32x16 instructions before, this after: 640 tiles of 16 slices (10 groups x 4096
// rows, D 1024) 117 -> 91 us, 256 tiles 46 -> 37, 1008 tiles of 32 slices (63 x 512 rows, D 2048) 294 -> 236; against the general
// 128 x 128 product kernel: Back 640 tiles 142 -> 86, 256 tiles 62 -> 34; Weights 160 tiles of 64 slices 214 -> 103, 256 of
// 16 slices 70 -> 38.  Fold, eight 2-byte LDS reads a fragment before: 512 channels, D 1024 81 -> 61, 1000 channels, D 2048 550 -> 413.
// Dynamic LDS: the ring (128 KiB).
// ---------------------------------------------------------------------------------------------
enum ProductKind { kProductLinear, kProductBack, kProductWeights, kProductFold, kProductImage, kProductOuter };
struct ProductArgs {
  const bf16 *A, *B, *bias, *rowadd;
  bf16 *C, *rowsum;
  long a_sb, a_sk, b_sb, b_sk, c_sb, c_sk;               // strides of a batch element and of a group
  int lda, ldb, ldc, ldbias;                             // row strides; elements of bias / rowsum a group
  RowBlocks rb;                                          // Linear, Back: rows of a group
  int kt, segs;                                          // slices of a segment of the contraction, and segments (batch elements)
  int C_all, g;                                          // Fold, Image, Outer: channels, channels of a group
  int H, W, pw, N;                                       // Image, Outer: image, patches of a row and in all
  unsigned pw_magic;                                     // ceil(2^32 / pw): n / pw is the upper half of n * pw_magic
  const bf16 *We, *be, *ce, *mix;                        // Outer: the operands and results of its epilogue
  const float* S;
  bf16 *dWe, *dtok, *dmix, *dbias, *Ws;
  TileWork tw;
  int slots;                                             // workgroups an XCD
};

// The tile of Image or Outer: block (h, i, hb, j), lane (l16, lq), register e: member 4 mt + 2 h + wm of the group, pixel 16 i + 4 lq + e,
// column 256 nt + 128 hb + 32 wn + 16 j + l16.  Blocks 2 q and 2 q + 1 trade with lane ^ 16: lane row lq then holds the eight
// pixels from 16 (2 q + lq % 2) + 8 (lq / 2) on, one row of the patch.
template <bool OUTER>
__device__ __forceinline__ void store_pixels(const ProductArgs& p, const CoreAcc& acc, const CoreLane& L, int k, int b, int mt,
                                             int nt) {
  typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
  typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
  const int lane = lane_id(), l16 = lane & 15, lq = lane >> 4;
  const int c0 = k * p.g, gk = min(p.g, p.C_all - c0);
  auto join = [](const bf16x4& x, const bf16x4& y) {
    const u32x2 a = __builtin_bit_cast(u32x2, x), c = __builtin_bit_cast(u32x2, y);
    const auto s0 = __builtin_amdgcn_permlane16_swap(a[0], c[0], false, false);
    const auto s1 = __builtin_amdgcn_permlane16_swap(a[1], c[1], false, false);
    return u32x4{s0[0], s1[0], s0[1], s1[1]};
  };
#pragma unroll
  for (int hb = 0; hb < 2; ++hb) {
    const int col0 = nt * kGemmBN + hb * 128 + L.wn * 32 + l16;
    if constexpr (!OUTER) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int n = col0 + j * 16, pi = __umulhi(n, p.pw_magic);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int cl = mt * 4 + 2 * h + L.wm;
          if (cl >= gk) continue;                          // uniform
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            bf16x4 v[2];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
              for (int e = 0; e < 4; ++e) v[t][e] = (bf16)acc[h][2 * q + t][hb][j][e];
            const u32x4 o = join(v[0], v[1]);
            const int row = 2 * (2 * q + (lq & 1)) + (lq >> 1);
            if (n < p.N)
              *reinterpret_cast<u32x4*>(p.C + (((size_t)b * p.C_all + c0 + cl) * p.H + pi * 8 + row) * p.W + (n - pi * p.pw) * 8) = o;
          }
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        // what a block of columns reads, asked for before its first store: one load at a time cost a round trip each
        const int col = col0 + j * 16;
        const float sv = p.S[(size_t)k * p.ldb + col];
        u32x4 w8[2][2];
        float sm[2], bias[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const size_t cd = (size_t)(c0 + min(mt * 4 + 2 * h + L.wm, gk - 1)) * p.ldb + col;
#pragma unroll
          for (int q = 0; q < 2; ++q)
            w8[h][q] = *reinterpret_cast<const u32x4*>(p.We + cd * 64 + (2 * q + (lq & 1)) * 16 + (lq >> 1) * 8);
          sm[h] = (float)p.mix[cd];
          bias[h] = (p.be ? (float)p.be[cd] : 0.f) + (p.ce ? (float)p.ce[cd] : 0.f);
        }
        if (p.dbias && mt == 0 && L.wm == 0 && lq == 0) p.dbias[(size_t)k * p.ldb + col] = (bf16)sv;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int cl = mt * 4 + 2 * h + L.wm;
          if (cl >= gk) continue;                          // uniform
          const size_t cd = (size_t)(c0 + cl) * p.ldb + col;
          float dot = 0.f;
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const u32x4 v8 = w8[h][q];
            const auto s0 = __builtin_amdgcn_permlane16_swap(v8[0], v8[2], false, false);   // the trade is its own inverse
            const auto s1 = __builtin_amdgcn_permlane16_swap(v8[1], v8[3], false, false);
            const bf16x4 w[2] = {__builtin_bit_cast(bf16x4, u32x2{s0[0], s1[0]}), __builtin_bit_cast(bf16x4, u32x2{s0[1], s1[1]})};
            bf16x4 gw[2], ws[2];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const float pv = acc[h][2 * q + t][hb][j][e];
                dot += (float)w[t][e] * pv;
                gw[t][e] = (bf16)(sm[h] * pv);
                ws[t][e] = (bf16)((float)w[t][e] * sm[h]);
              }
            const size_t at = cd * 64 + (2 * q + (lq & 1)) * 16 + (lq >> 1) * 8;
            if (p.Ws) *reinterpret_cast<u32x4*>(p.Ws + at) = join(ws[0], ws[1]);
            if (p.dWe) *reinterpret_cast<u32x4*>(p.dWe + at) = join(gw[0], gw[1]);
          }
          dot += __shfl_xor(dot, 16, kWave);
          dot += __shfl_xor(dot, 32, kWave);
          if (lq == 0) {
            if (p.dmix) p.dmix[cd] = (bf16)(dot + bias[h] * sv);
            if (p.dtok) p.dtok[cd] = (bf16)(sm[h] * sv);
          }
        }
      }
    }
  }
}

template <int KIND>
__global__ __launch_bounds__(512) void k_product_dl(ProductArgs p) {
  constexpr bool FOLD = KIND == kProductFold, IMAGE = KIND == kProductImage, OUTER = KIND == kProductOuter;
  constexpr bool A_COL = KIND == kProductWeights || OUTER, SWAP = !IMAGE && !OUTER;
  typedef std::conditional_t<A_COL, ColOperand<256>, std::conditional_t<IMAGE, ColOperand<128>, RowOperand>> OA;
  typedef std::conditional_t<FOLD, ColOperand<128>, std::conditional_t<KIND == kProductLinear || IMAGE, RowOperand, ColOperand<256>>> OB;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
  const int per = (p.tw.total + kXcds - 1) / kXcds;
  const int xcd_end = min((xcd + 1) * per, p.tw.total);
  struct Item {
    int k, b, mt, nt;
  };
  auto item_of = [&](int& t, Item& it) -> bool {         // the first item from the t-th on that has rows (Fold: channels)
    for (;; ++t) {
      const int w = xcd * per + t * p.slots + slot;
      if (w >= xcd_end) return false;
      p.tw.decode_linear(w, it.k, it.b, it.mt, it.nt);
      if (FOLD || OUTER ? (FOLD ? it.nt : it.mt) * 4 < min(p.g, p.C_all - it.k * p.g) : A_COL || it.mt * kGemmBM < p.rb.rows_of(it.k)) return true;
    }
  };

  CoreLane L;
  L.init<OA, OB>();
  const unsigned wave_off = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(lptr_t)smem) + L.wave * 2048;

  Item ic, nx;                                           // the tile that is multiplied, and the next segment's
  int t = 0;
  if (!item_of(t, ic)) return;                           // uniform: the whole workgroup has nothing to do
  struct Src {
    const bf16 *a, *b0, *b1;                             // origins of a segment's tile in its running slice (b1: slot B1)
    int rows;                                            // rows of A behind the tile's first (Outer: members of the group)
    int first;                                           // Outer: the tile's first member
    const bf16* a1;                                      // Image: a and a1 are this wavefront's 16 of a member's rows in slots A0 and A1
  } run, nxt;
  auto source = [&](const Item& it, int seg, Src& s) {
    s.a = p.A + seg * p.a_sb + it.b * p.a_sb + it.k * p.a_sk;
    if (OUTER) {
      s.first = it.mt * 4;
      s.rows = min(p.g, p.C_all - it.k * p.g);
      s.b0 = p.B + seg * p.b_sb + it.k * p.b_sk + it.nt * kGemmBN + (size_t)L.wave * 8 * p.ldb;
      s.b1 = s.b0 + 128;
      return;
    }
    if (IMAGE) {                                         // a slot is two members, of which the last of the group repeats
      const int last = min(p.g, p.C_all - it.k * p.g) - 1, m = it.mt * 4 + (L.wave >> 2);
      s.a1 = s.a + (size_t)min(m + 2, last) * p.lda * 64 + (L.wave & 3) * 16 * 64;
      s.a += (size_t)min(m, last) * p.lda * 64 + (L.wave & 3) * 16 * 64;
    } else if (A_COL) s.a += it.mt * kGemmBM + (size_t)L.wave * 8 * p.lda;
    else s.a += (size_t)it.mt * kGemmBM * p.lda;
    s.rows = FOLD || A_COL ? 256 : p.rb.rows_of(it.k) - it.mt * kGemmBM;
    if (FOLD) {
      const int c0 = it.k * p.g, last = min(p.g, p.C_all - c0) - 1, q = it.nt * 4 + (L.wave >> 2);
      const int in = (L.wave & 3) * 16 * 64;             // a wavefront's 16 of a channel's 64 contraction rows
      s.b0 = p.B + (c0 + min(q, last)) * p.b_sk + in;    // a missing channel of the four repeats the last one; not stored
      s.b1 = p.B + (c0 + min(q + 2, last)) * p.b_sk + in;
    } else {
      s.b0 = p.B + seg * p.b_sb + it.b * p.b_sb + it.k * p.b_sk;
      if (IMAGE) {
        s.b0 += ((size_t)it.nt * kGemmBN + L.wave * 16) * p.ldb;
        s.b1 = s.b0 + (it.nt * kGemmBN + 128 < p.N ? (size_t)128 * p.ldb : 0);   // half a tile of patches: the half again
        return;
      } else if (KIND == kProductLinear) s.b0 += ((size_t)it.nt * kGemmBN + L.wave * 16) * p.ldb;
      else s.b0 += it.nt * kGemmBN + (size_t)L.wave * 8 * p.ldb;
      s.b1 = s.b0 + (KIND == kProductLinear ? (size_t)128 * p.ldb : 128);
    }
  };
  // Byte of a lane's 16 behind those origins.  RowOperand: row lane / 8 and the chunk that belongs there; eight rows further bit 6
  // (the chunk's) flips.  ColOperand<256>: contraction row lane / 16, four rows further nothing changes.
  auto col_off = [&](int ld) {
    const int lane = lane_id(), row = L.wave * 8 + (lane >> 4);
    return (lane >> 4) * ld * 2 + ((lane & 15) ^ ColOperand<256>::swz(row)) * 16;
  };
  // Outer: the part of a chunk's place in the image that its patch does not change, per slot: member and pixel row.
  unsigned a_off[2][2];
  auto a_rows = [&](const Src& s) {
    const int lane = lane_id();
    if (OUTER) {
      const int lc = (lane & 15) ^ ColOperand<256>::swz(L.wave * 8 + (lane >> 4));
#pragma unroll
      for (int h = 0; h < 2; ++h)
        a_off[h][0] = (unsigned)(min(s.first + 2 * h + (lc >> 3), s.rows - 1) * p.H + (lc & 7)) * p.W * 2;
    } else if (A_COL) {
      a_off[0][0] = col_off(p.lda);
    } else if (IMAGE) {
      a_off[0][0] = (lane >> 3) * 128 + ((lane & 7) ^ ColOperand<128>::swz(lane >> 3)) * 16;
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int row = h * 128 + L.wave * 16 + u * 8 + (lane >> 3);
          a_off[h][u] = (unsigned)min(row, s.rows - 1) * p.lda * 2 + L.ld_chunk(lane, u);
        }
    }
  };
  int b_off;
  if (FOLD) b_off = (lane_id() >> 3) * 128 + ((lane_id() & 7) ^ ColOperand<128>::swz(lane_id() >> 3)) * 16;
  else if (KIND == kProductLinear || IMAGE) b_off = (lane_id() >> 3) * p.ldb * 2 + L.ld_chunk(lane_id(), 0);
  else b_off = col_off(p.ldb);
  source(ic, 0, run);
  a_rows(run);
  int ki = 0;                                            // slices issued of the segment
  auto issue = [&](int sl) {                             // sl: a constant once inlined
    const unsigned dst = wave_off + sl * kSlotBytes;
    const int kind = sl & ~2;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (kind == kSlotA0 || kind == kSlotA1) {
        const int h = kind == kSlotA1;
        if (OUTER) {
          const int n = (ki + ((sl & 2) >> 1)) * 64 + L.wave * 8 + u * 4 + (lane_id() >> 4), pi = __umulhi(n, p.pw_magic);
          load16_to_lds_at(run.a, a_off[h][0] + (unsigned)(pi * p.W + n - pi * p.pw) * 16, dst + u * 1024);
        } else if (IMAGE) load16_to_lds_at((h ? run.a1 : run.a) + u * 8 * 64, opaque(a_off[0][0]) ^ (u * 64), dst + u * 1024);
        else if (A_COL) load16_to_lds_at(run.a + h * 128 + (size_t)u * 4 * p.lda, a_off[0][0], dst + u * 1024);
        else load16_to_lds_at(run.a, a_off[h][u], dst + u * 1024);
      } else {
        const bf16* s = kind == kSlotB1 ? run.b1 : run.b0;
        if (FOLD) load16_to_lds_at(s + u * 8 * 64, opaque(b_off) ^ (u * 64), dst + u * 1024);
        else if (KIND == kProductLinear || IMAGE) load16_to_lds_at(s + (size_t)u * 8 * p.ldb, opaque(b_off) ^ (u * 64), dst + u * 1024);
        else load16_to_lds_at(s + (size_t)u * 4 * p.ldb, b_off, dst + u * 1024);
      }
    }
    if (kind == kSlotA1) {                               // the last slot of a slice
      if (!OUTER) run.a += A_COL ? (size_t)64 * p.lda : IMAGE ? 64 * 64 : 64;
      if (IMAGE) run.a1 += 64 * 64;
      const size_t bs = FOLD ? 64 * 64 : KIND == kProductLinear || IMAGE ? 64 : (size_t)64 * p.ldb;
      run.b0 += bs;
      run.b1 += bs;
      if (sl & 2) {
        ki += 2;
        if (ki == p.kt) {
          ki = 0;
          run = nxt;
          a_rows(run);
        }
      }
    }
  };

  CoreFrags f;
  CoreAcc acc;
  // Row sums of A (Weights, tiles of the first columns): wavefront wn adds up block wn of both slots, by products with ones.
  f32x4 rs[2];
  bool sums = false;
  auto held = [&](int h, const bf16x8 (&a)[4][2]) {
    if (KIND == kProductWeights && sums) {
      bf16x8 ones;
#pragma unroll
      for (int e = 0; e < 8; ++e) ones[e] = (bf16)1.f;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (L.wn == i) {                                 // uniform
#pragma unroll
          for (int kk = 0; kk < 2; ++kk) rs[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, a[i][kk], rs[h], 0, 0, 0);
        }
    }
  };
  core_prologue<OA, OB>(f, smem, L, issue);
  int seg = 0;
  for (;;) {
    nx = ic;
    int nseg = seg + 1;
    bool more = true;
    if (nseg == p.segs) {
      nseg = 0;
      ++t;
      more = item_of(t, nx);
      if (!more) nx = ic;                                // past the last tile: this one again, loaded and not used
    }
    source(nx, nseg, nxt);
    int kt = 0;
    if (seg == 0) {
      if (KIND == kProductWeights) {
        sums = p.rowsum && ic.nt == 0;
        rs[0] = rs[1] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      core_slice<true, SWAP, 0, OA, OB>(acc, f, smem, L, issue, held);
      core_slice<false, SWAP, 1, OA, OB>(acc, f, smem, L, issue, held);
      kt = 2;
    }
    for (; kt < p.kt; kt += 2) {
      core_slice<false, SWAP, 0, OA, OB>(acc, f, smem, L, issue, held);
      core_slice<false, SWAP, 1, OA, OB>(acc, f, smem, L, issue, held);
    }
    if (nseg != 0) {
      seg = nseg;
      continue;
    }
    if constexpr (!SWAP) {
      store_pixels<OUTER>(p, acc, L, ic.k, ic.b, ic.mt, ic.nt);
      if (!more) break;
      ic = nx;
      seg = 0;
      continue;
    }
    // block (h, i, hb, j), lane (l16, lq), register e: row 128 h + 64 wm + 16 i + l16, column 128 hb + 32 wn + 16 j + 4 lq + e
    const int l16 = lane_id() & 15, lq = lane_id() >> 4;
    const int o0 = ic.nt * kGemmBN, r0 = ic.mt * kGemmBM;
    const int rows = FOLD || A_COL ? 256 : p.rb.rows_of(ic.k) - r0;
    if (KIND == kProductWeights && sums && lq == 0) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        p.rowsum[(size_t)ic.k * p.ldbias + r0 + h * 128 + L.wm * 64 + L.wn * 16 + l16] = (bf16)rs[h][0];
    }
    bf16* Cb = p.C + ic.b * p.c_sb + ic.k * p.c_sk + (size_t)r0 * p.ldc + (FOLD ? (size_t)ic.nt * 4 * p.ldc * p.lda : o0);
    const int left = FOLD ? min(p.g, p.C_all - ic.k * p.g) - ic.nt * 4 : 4;      // channels from the tile's first on
#pragma unroll
    for (int hb = 0; hb < 2; ++hb) {
      const int col = hb * 128 + L.wn * 32;
      f32x4 bq[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        bq[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (KIND == kProductLinear && p.bias) {
          const bf16x4 v = *reinterpret_cast<const bf16x4*>(p.bias + (size_t)ic.k * p.ldbias + o0 + col + 16 * j + 4 * lq);
#pragma unroll
          for (int e = 0; e < 4; ++e) bq[j][e] = (float)v[e];
        }
      }
#pragma unroll
      for (int hi = 0; hi < 8; ++hi) {
        const int row = (hi >> 2) * 128 + L.wm * 64 + (hi & 3) * 16 + l16;
        const bool in = row < rows && (!FOLD || (col >> 6) < left);
        typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
        typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
        u32x2 w[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          f32x4 v = acc[hi >> 2][hi & 3][hb][j] + bq[j];
          if (KIND == kProductLinear && p.rowadd && in) {
            const bf16x4 ra = *reinterpret_cast<const bf16x4*>(p.rowadd + (size_t)(r0 + row) * p.ldc + o0 + col + 16 * j + 4 * lq);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += (float)ra[e];
          }
          bf16x4 q;
#pragma unroll
          for (int e = 0; e < 4; ++e) q[e] = (bf16)v[e];
          w[j] = __builtin_bit_cast(u32x2, q);
        }
        // lane rows 0 and 2 (of 16) keep block 0 and take the next row's columns of it; rows 1 and 3 the same of block 1
        const auto s0 = __builtin_amdgcn_permlane16_swap(w[0][0], w[1][0], false, false);
        const auto s1 = __builtin_amdgcn_permlane16_swap(w[0][1], w[1][1], false, false);
        bf16* dst = FOLD ? Cb + (size_t)(col >> 6) * p.ldc * p.lda + (size_t)row * p.ldc + (col & 63) : Cb + (size_t)row * p.ldc + col;
        if (in) *reinterpret_cast<u32x4*>(dst + (lq & 1) * 16 + (lq >> 1) * 8) = u32x4{s0[0], s1[0], s0[1], s1[1]};
      }
    }
    if (!more) break;
    ic = nx;
    seg = 0;
  }
  wait_vmcnt<0>();                                       // no load may still target LDS when the block retires
}

// The token biases under the same fold (weight-only):  fb[c][o] = sum_d (be[c][d] + ce[c][d]) * Wv[k][o][d],  k = c / g;
// either vector may be absent.  grid (D / 64, G), block 256: 64 rows o of Wv (16 a wavefront) against the group's members, 16 MB a
// pass; slices of 64 d of the rows and of both vectors by direct-to-LDS loads, three slices ahead.  Bound by the read of Wv.  Blocks start
// at different slices (the rows of all of them are multiples of 4 KB apart, which meets few channels).  be and ce, and the two halves of
// a slice, have sums of their own, added up at the end.  63 groups of 16, D 2048 (528 MB): 112 us (operands straight to
// registers, 64 bytes of a row to a lane: 171); 16 of 32, D 1024: 14 (17.5); 10 of 8: 9 (10).  Requires D % 256 == 0 and 16-byte aligned rows.
template <int MB>
__global__ __launch_bounds__(256) void k_fold_token_bias(int C, int D, int g, const bf16* __restrict__ Wv,
                                                         const bf16* __restrict__ be, const bf16* __restrict__ ce,
                                                         bf16* __restrict__ fb) {
  constexpr int ST = 4, WB = 64 * 128, VB = 16 * MB * 128, STAGE = WB + 2 * VB, L = 2 + MB;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[ST * STAGE];
  const int k = blockIdx.y, o0 = blockIdx.x * 64;
  const int c0 = k * g, gk = min(g, C - c0), KT = D / 64;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, lq = lane >> 4;
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(lptr_t)smem);
  const bf16* W0 = Wv + ((size_t)k * D + o0) * D;
  // a load brings 8 rows: two of Wv's to a wavefront, and MB of the vectors' (wavefronts 0 and 1: be, 2 and 3: ce)
  unsigned w_off[2], v_off[MB];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = (wave * 2 + i) * 8 + (lane >> 3);
    w_off[i] = (unsigned)row * (unsigned)D * 2 + ((lane & 7) ^ swz_chunk(row)) * 16;
  }
  const bf16* vec = wave < 2 ? be : ce;
  const int w_ad = RowOperand::base(wave * 16, lane), v_ad = RowOperand::base(0, lane);
  for (int cb = 0; cb < gk; cb += 16 * MB) {
    const bf16* V0 = vec + (size_t)(c0 + cb) * D;
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int row = ((wave & 1) * MB + i) * 8 + (lane >> 3);
      v_off[i] = (unsigned)min(row, gk - cb - 1) * (unsigned)D * 2 + ((lane & 7) ^ swz_chunk(row)) * 16;
    }
    int ki = blockIdx.x % KT, is = 0;
    auto issue = [&]() {
      const unsigned dst = lds0 + is * STAGE;
#pragma unroll
      for (int i = 0; i < 2; ++i) load16_to_lds_at(W0 + ki * 64, w_off[i], dst + (wave * 2 + i) * 1024);
#pragma unroll
      for (int i = 0; i < MB; ++i)                        // an absent vector's rows are never read: Wv's stand in for them
        load16_to_lds_at(vec ? V0 + ki * 64 : W0 + ki * 64, vec ? v_off[i] : w_off[0], dst + WB + (wave * MB + i) * 1024);
      is = (is + 1) % ST;
      ki = ki == KT - 1 ? 0 : ki + 1;
    };
    f32x4 acc[2][2][MB];
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int j = 0; j < MB; ++j) acc[v][kk][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < ST - 1; ++s)
      if (s < KT) issue();
    for (int s = 0; s < KT; ++s) {
      // slice s has landed (this wavefront's share; two behind it may stay in flight), every wavefront is done with slice s - 1
      const int behind = KT - 1 - s;                      // uniform
      if (behind >= 2) wait_vmcnt<2 * L>();
      else if (behind == 1) wait_vmcnt<L>();
      else wait_vmcnt<0>();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      if (s + ST - 1 < KT) issue();
      const unsigned char* st = smem + s % ST * STAGE;
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const bf16x8 w = RowOperand::frag(st, w_ad, 0, kk, 0);
#pragma unroll
        for (int j = 0; j < MB; ++j) {
          if (be) acc[0][kk][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, RowOperand::frag(st + WB, v_ad, j, kk, 0), acc[0][kk][j], 0, 0, 0);
          if (ce)
            acc[1][kk][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, RowOperand::frag(st + WB + VB, v_ad, j, kk, 0), acc[1][kk][j], 0, 0, 0);
        }
      }
    }
    // block j: member 16 j + l16, rows 4 lq + e of the wavefront's 16
#pragma unroll
    for (int j = 0; j < MB; ++j)
      if (cb + j * 16 + l16 < gk) {
        typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
        bf16x4_t out;
#pragma unroll
        for (int e = 0; e < 4; ++e) out[e] = (bf16)((acc[0][0][j][e] + acc[0][1][j][e]) + (acc[1][0][j][e] + acc[1][1][j][e]));
        *reinterpret_cast<bf16x4_t*>(fb + (size_t)(c0 + cb + j * 16 + l16) * D + o0 + wave * 16 + lq * 4) = out;
      }
    __syncthreads();                                      // the next pass fills the stages again
  }
}

// ---------------------------------------------------------------------------------------------
// Level-1 scores straight from the pixels.  The tokenizer is linear, so the score of token
// t = We[c] u + be[c] + ce[c] against the folded key M[k][a] is
//   t . M[k][a] = u . (We[c]^T M[k][a]) + (be[c] + ce[c]) . M[k][a]
// k_compose_score_weights builds the weight-only pieces  Ms[c][a][kk] = sum_d M[k][a][d] We[c][d][kk]
// and cs[c][a] = sum_d M[k][a][d] (be[c][d] + ce[c][d]) in fp32 (k = c / g);
// k_scores_pixels then scores every (channel, patch) with a p*p-long dot product per head.
// ---------------------------------------------------------------------------------------------
// grid (C), block 256.  The channel's tokenizer weights and the transposed folded key MfT[G][D][heads]
// stream through LDS in blocks of DQ rows of d (full-width 16-byte loads); outputs are tiled 4 heads x 4
// pixels, lane l of every wavefront owns tiles l, l+64, ... (TPL of them) and wavefront w sums the
// rows d = w (mod 4) of a block; the four partial sums meet in LDS in a fixed order.  Writes fp32 Ms,
// its bf16 copy Msb (the MFMA operand of k_scores_pixels) and cs.
// Requires heads % 4 == 0, pp % 8 == 0, DQ % 4 == 0, D % DQ == 0.
// Dynamic LDS: DQ * (pp * 2 + heads * 4 + 4) bytes, then 3 * TPL * 64 * 20 floats.
template <int TPL>
__global__ __launch_bounds__(256) void k_compose_score_weights(int D, int heads, int pp, int g, int DQ,
                                                               const float* __restrict__ MfT,
                                                               const bf16* __restrict__ We, const bf16* __restrict__ be,
                                                               const bf16* __restrict__ ce, float* __restrict__ Ms,
                                                               bf16* __restrict__ Msb, float* __restrict__ cs) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16* w_s = reinterpret_cast<bf16*>(smem);                                   // [DQ][pp]
  float* m_s = reinterpret_cast<float*>(smem + (size_t)DQ * pp * 2);           // [DQ][heads]
  float* b_s = m_s + (size_t)DQ * heads;                                       // [DQ]
  float* part = b_s + DQ;                                                      // [3][TPL*20][64]
  const int c = blockIdx.x, k = c / g;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kq_n = pp / 4, aq_n = heads / 4, ntiles = kq_n * aq_n;
  const float* M = MfT + (size_t)k * D * heads;
  const bf16* Wc = We + (size_t)c * D * pp;
  float acc[TPL][16], cacc[TPL][4];
  int kq[TPL], aq[TPL];
#pragma unroll
  for (int t = 0; t < TPL; ++t) {
    const int tile = lane + t * 64;
    kq[t] = tile < ntiles ? tile % kq_n : -1;
    aq[t] = tile < ntiles ? tile / kq_n : 0;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) cacc[t][e] = 0.f;
  }
  for (int d0 = 0; d0 < D; d0 += DQ) {
    __syncthreads();
    for (int idx = tid; idx < DQ * pp / 8; idx += 256)
      reinterpret_cast<bf16x8*>(w_s)[idx] = reinterpret_cast<const bf16x8*>(Wc + (size_t)d0 * pp)[idx];
    for (int idx = tid; idx < DQ * heads / 4; idx += 256)
      reinterpret_cast<f32x4*>(m_s)[idx] = reinterpret_cast<const f32x4*>(M + (size_t)d0 * heads)[idx];
    for (int idx = tid; idx < DQ; idx += 256) {
      float bsum = 0.f;
      if (be) bsum += (float)be[(size_t)c * D + d0 + idx];
      if (ce) bsum += (float)ce[(size_t)c * D + d0 + idx];
      b_s[idx] = bsum;
    }
    __syncthreads();
#pragma unroll 4
    for (int d = wave; d < DQ; d += 4) {
      const float bsum = b_s[d];
#pragma unroll
      for (int t = 0; t < TPL; ++t) {
        if (kq[t] < 0) continue;
        const f32x4 m4 = *reinterpret_cast<const f32x4*>(m_s + (size_t)d * heads + aq[t] * 4);
        const bf16x4 w4 = *reinterpret_cast<const bf16x4*>(w_s + (size_t)d * pp + kq[t] * 4);
#pragma unroll
        for (int a = 0; a < 4; ++a) {
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[t][a * 4 + q] += m4[a] * (float)w4[q];
          cacc[t][a] += m4[a] * bsum;
        }
      }
    }
  }
  if (wave > 0) {
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
#pragma unroll
      for (int e = 0; e < 16; ++e) part[((wave - 1) * TPL * 20 + t * 20 + e) * 64 + lane] = acc[t][e];
#pragma unroll
      for (int e = 0; e < 4; ++e) part[((wave - 1) * TPL * 20 + t * 20 + 16 + e) * 64 + lane] = cacc[t][e];
    }
  }
  __syncthreads();
  if (wave == 0) {
    float* Mo = Ms + (size_t)c * heads * pp;
    bf16* Mbo = Msb + (size_t)c * heads * pp;
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
      if (kq[t] < 0) continue;
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const int head = aq[t] * 4 + a;
        f32x4 v4;
        bf16x4 b4;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int e = a * 4 + q;
          v4[q] = acc[t][e] + part[((0 * TPL + t) * 20 + e) * 64 + lane] + part[((1 * TPL + t) * 20 + e) * 64 + lane] +
                  part[((2 * TPL + t) * 20 + e) * 64 + lane];
          b4[q] = (bf16)v4[q];
        }
        *reinterpret_cast<f32x4*>(Mo + (size_t)head * pp + kq[t] * 4) = v4;
        *reinterpret_cast<bf16x4*>(Mbo + (size_t)head * pp + kq[t] * 4) = b4;
        if (kq[t] == 0) {
          const int e = 16 + a;
          cs[(size_t)c * heads + head] = cacc[t][a] + part[((0 * TPL + t) * 20 + e) * 64 + lane] +
                                         part[((1 * TPL + t) * 20 + e) * 64 + lane] +
                                         part[((2 * TPL + t) * 20 + e) * 64 + lane];
        }
      }
    }
  }
}

// The same weights on 16x16x32 MFMA for pp = 16, 32, 64 or 128 (NKB = pp / 8 blocks of 8 pixels) and group sizes that
// are multiples of CPB = 16 / NKB: a block takes CPB channels of one group, its four wavefronts a quarter of D each.
// A fragments: the fp32 folded key rows Mf[k][head][d] split in two bf16 parts (nothing of them is lost); B fragments:
// a lane reads 8 rows d x 8 adjacent pixels of We[c] (16 bytes per row) and transposes them in registers, which gives
// it the fragments (column = channel l16 / NKB, pixel 8 (l16 % NKB) + j; d = 8 (lane / 16) ..) of eight products
// j = 0..7.  The bias part takes two more products per step (be and ce as they are: column = channel).  The partial
// blocks of the wavefronts meet in LDS in a fixed order.  grid (ceil(C / CPB)), block 256.  D % 128 == 0.
__device__ __forceinline__ void split_hi_lo(const f32x4& x0, const f32x4& x1, bf16x8& hi, bf16x8& lo) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    hi[i] = (bf16)x0[i];
    lo[i] = (bf16)(x0[i] - (float)hi[i]);
    hi[4 + i] = (bf16)x1[i];
    lo[4 + i] = (bf16)(x1[i] - (float)hi[4 + i]);
  }
}

template <int HB>   // blocks of 16 heads (heads <= 16 HB)
__global__ __launch_bounds__(256) void k_compose_score_weights_mfma(int C, int D, int heads, int pp, int g,
                                                                    const float* __restrict__ Mf,
                                                                    const bf16* __restrict__ We,
                                                                    const bf16* __restrict__ be,
                                                                    const bf16* __restrict__ ce, float* __restrict__ Ms,
                                                                    bf16* __restrict__ Msb, float* __restrict__ cs) {
  __shared__ f32x4 part[3][HB][9][64];
  const int nkb = pp / 8, cpb = 16 / nkb;
  const int c0 = blockIdx.x * cpb, k = c0 / g;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, lq = lane >> 4;
  const int csub = l16 / nkb, kkb = l16 % nkb;
  const int c = min(c0 + csub, C - 1);                   // a short last block: its repeats are not written
  const int cbias = min(c0 + l16, C - 1);                // the channel this lane supplies in the bias products
  const bf16* wsrc = We + (size_t)c * D * pp + kkb * 8;
  const int dq = D / 4;
  f32x4 acc[HB][8], bacc[HB];
#pragma unroll
  for (int hb = 0; hb < HB; ++hb) {
    bacc[hb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[hb][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  for (int d0 = wave * dq; d0 < (wave + 1) * dq; d0 += 32) {
    const int d = d0 + 8 * lq;                           // this lane's 8 steps of the contraction
    bf16x8 mhi[HB], mlo[HB];
#pragma unroll
    for (int hb = 0; hb < HB; ++hb) {
      const float* mp = Mf + ((size_t)k * heads + min(16 * hb + l16, heads - 1)) * D + d;
      split_hi_lo(*reinterpret_cast<const f32x4*>(mp), *reinterpret_cast<const f32x4*>(mp + 4), mhi[hb], mlo[hb]);
    }
    bf16x8 rows[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) rows[i] = *reinterpret_cast<const bf16x8*>(wsrc + (size_t)(d + i) * pp);
    bf16x8 bev = {}, cev = {};
    if (l16 < cpb) {
      if (be) bev = *reinterpret_cast<const bf16x8*>(be + (size_t)cbias * D + d);
      if (ce) cev = *reinterpret_cast<const bf16x8*>(ce + (size_t)cbias * D + d);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      bf16x8 col;
#pragma unroll
      for (int i = 0; i < 8; ++i) col[i] = rows[i][j];
#pragma unroll
      for (int hb = 0; hb < HB; ++hb) {
        acc[hb][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(mhi[hb], col, acc[hb][j], 0, 0, 0);
        acc[hb][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(mlo[hb], col, acc[hb][j], 0, 0, 0);
      }
    }
#pragma unroll
    for (int hb = 0; hb < HB; ++hb) {
      bacc[hb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(mhi[hb], bev, bacc[hb], 0, 0, 0);
      bacc[hb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(mlo[hb], bev, bacc[hb], 0, 0, 0);
      bacc[hb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(mhi[hb], cev, bacc[hb], 0, 0, 0);
      bacc[hb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(mlo[hb], cev, bacc[hb], 0, 0, 0);
    }
  }
  if (wave > 0) {
#pragma unroll
    for (int hb = 0; hb < HB; ++hb) {
#pragma unroll
      for (int j = 0; j < 8; ++j) part[wave - 1][hb][j][lane] = acc[hb][j];
      part[wave - 1][hb][8][lane] = bacc[hb];
    }
  }
  __syncthreads();
  if (wave != 0) return;
  // accumulator block: lane holds column l16, rows (heads) 4 lq + r
#pragma unroll
  for (int hb = 0; hb < HB; ++hb) {
    f32x4 tot[9];
#pragma unroll
    for (int j = 0; j < 8; ++j) tot[j] = acc[hb][j] + part[0][hb][j][lane] + part[1][hb][j][lane] + part[2][hb][j][lane];
    tot[8] = bacc[hb] + part[0][hb][8][lane] + part[1][hb][8][lane] + part[2][hb][8][lane];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int head = 16 * hb + 4 * lq + r;
      if (head >= heads) continue;
      if (c0 + csub < C) {
        const size_t o = ((size_t)(c0 + csub) * heads + head) * pp + kkb * 8;
        *reinterpret_cast<f32x4*>(Ms + o) = f32x4{tot[0][r], tot[1][r], tot[2][r], tot[3][r]};
        *reinterpret_cast<f32x4*>(Ms + o + 4) = f32x4{tot[4][r], tot[5][r], tot[6][r], tot[7][r]};
        bf16x8 b8;
#pragma unroll
        for (int j = 0; j < 8; ++j) b8[j] = (bf16)tot[j][r];
        *reinterpret_cast<bf16x8*>(Msb + o) = b8;
      }
      if (l16 < cpb && c0 + l16 < C) cs[(size_t)(c0 + l16) * heads + head] = tot[8][r];
    }
  }
}

// Level-1 scores on MFMA: S[b][k][cl][head][n] = u[b,c,n][:] . Msb[c][head][:] + cs[c][head].
// grid (ceil(N/128), C, B), block 256: wavefront w scores 32 patches of channel c against up to 32 heads
// with one 32x32x16 MFMA per 16 pixels.  A lane's operand (8 consecutive pixels of a patch) is one
// 16-byte load when p % 8 == 0, two 8-byte loads when p == 4.  Requires heads <= 32, pp % 16 == 0.
__global__ __launch_bounds__(256) void k_scores_pixels(int C, int H, int W, int p, int heads, int g, int gpad, int G,
                                                       int Np, const bf16* __restrict__ x,
                                                       const bf16* __restrict__ Msb, const float* __restrict__ cs,
                                                       float* __restrict__ S) {
  const int pp = p * p, pw = W / p, N = (H / p) * pw;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, lhi = lane >> 5;
  const int c = blockIdx.y, b = blockIdx.z, k = c / g, cl = c % g;
  const int n0 = blockIdx.x * 128 + wave * 32;
  if (n0 >= N) return;
  const int n = min(n0 + l32, N - 1);
  const int pi = n / pw, pj = n % pw;
  const bf16* img = x + ((size_t)b * C + c) * H * W + (size_t)(pi * p) * W + pj * p;
  const bf16* mrow = Msb + ((size_t)c * heads + min(l32, heads - 1)) * pp;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  for (int kc = lhi; kc < pp / 8; kc += 2) {            // 8-pixel chunk of the patch
    bf16x8 a;
    if (p == 4) {
      const bf16x4 lo = *reinterpret_cast<const bf16x4*>(img + (size_t)(2 * kc) * W);
      const bf16x4 hi = *reinterpret_cast<const bf16x4*>(img + (size_t)(2 * kc + 1) * W);
#pragma unroll
      for (int e = 0; e < 4; ++e) { a[e] = lo[e]; a[4 + e] = hi[e]; }
    } else {
      const int r = (kc * 8) / p, s0 = (kc * 8) % p;
      a = *reinterpret_cast<const bf16x8*>(img + (size_t)r * W + s0);
    }
    bf16x8 m = *reinterpret_cast<const bf16x8*>(mrow + kc * 8);
    if (l32 >= heads) m = bf16x8{};
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, m, acc, 0, 0, 0);
  }
  if (l32 < heads) {
    const float add = cs[(size_t)c * heads + l32];
    float* dst = S + ((((size_t)b * G + k) * gpad + cl) * heads + l32) * Np + n0 + 4 * lhi;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = acc[4 * q + e] + add;
      *reinterpret_cast<f32x4*>(dst + 8 * q) = v;
    }
  }
}

// The same scores with the softmax over the group in the same kernel, for groups whose scores of 32 patches fit LDS
// (size of the group x heads x 33 floats): grid (ceil(N/32), G, B), block 256.  The wavefronts take the group's
// channels in turn (the products of k_scores_pixels) and leave the scores in LDS as [member][head][patch, pitch 33];
// then every (head, patch) is normalised over the members in the order and with the arithmetic of k_softmax_alpha,
// and the weights are written in the layout of the forward kernels (alpha_f[b][k][cl][head][n], zeros for padding
// members and the pitch) and / or token-major (alpha_tm[b,c,n,head]), whichever pointer is given.
// PP: pixels per patch when known at compile time (16 or 64: a channel's operand loads are then issued together, and
// those of the wavefront's next channel while the current one is multiplied), 0 for any other patch size.
template <int PP>
__global__ __launch_bounds__(256) void k_scores_pixels_softmax(int C, int H, int W, int p, int heads, int g, int gpad,
                                                               int G, int Np, const bf16* __restrict__ x,
                                                               const bf16* __restrict__ Msb,
                                                               const float* __restrict__ cs,
                                                               float* __restrict__ alpha_f,
                                                               float* __restrict__ alpha_tm) {
  extern __shared__ __attribute__((aligned(16))) float sc[];       // [gk][heads][33]
  const int pp = PP ? PP : p * p, pw = W / p, N = (H / p) * pw;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, lhi = lane >> 5;
  const int k = blockIdx.y, b = blockIdx.z;
  const int c0 = k * g, gk = min(g, C - c0);
  const int n0 = blockIdx.x * 32;
  const int n = min(n0 + l32, N - 1);
  const int pi = n / pw, pj = n % pw;
  const size_t img_off = (size_t)(pi * p) * W + pj * p;
  // one 8-pixel chunk of this lane's patch of channel c, and the matching chunk of the composed score weights
  auto load_a = [&](int c, int kc) -> bf16x8 {
    const bf16* img = x + ((size_t)b * C + c) * H * W + img_off;
    bf16x8 a;
    if (p == 4) {
      const bf16x4 lo = *reinterpret_cast<const bf16x4*>(img + (size_t)(2 * kc) * W);
      const bf16x4 hi = *reinterpret_cast<const bf16x4*>(img + (size_t)(2 * kc + 1) * W);
#pragma unroll
      for (int e = 0; e < 4; ++e) { a[e] = lo[e]; a[4 + e] = hi[e]; }
    } else {
      const int r = (kc * 8) / p, s0 = (kc * 8) % p;
      a = *reinterpret_cast<const bf16x8*>(img + (size_t)r * W + s0);
    }
    return a;
  };
  auto load_m = [&](int c, int kc) -> bf16x8 {
    bf16x8 m = *reinterpret_cast<const bf16x8*>(Msb + ((size_t)c * heads + min(l32, heads - 1)) * pp + kc * 8);
    if (l32 >= heads) m = bf16x8{};
    return m;
  };
  auto leave = [&](int cl, const f32x16& acc) {          // lane: head l32, patches 8 (r / 4) + 4 lhi + r % 4
    if (l32 < heads) {
      const float add = cs[(size_t)(c0 + cl) * heads + l32];
      float* dst = sc + ((size_t)cl * heads + l32) * 33 + 4 * lhi;
#pragma unroll
      for (int r = 0; r < 16; ++r) dst[8 * (r >> 2) + (r & 3)] = acc[r] + add;
    }
  };
  if constexpr (PP > 0) {
    constexpr int NIT = PP / 16;                         // chunks per lane half
    bf16x8 a0[NIT], m0[NIT], a1[NIT], m1[NIT];
    auto fetch = [&](int cl, bf16x8 (&a)[NIT], bf16x8 (&m)[NIT]) {
#pragma unroll
      for (int t = 0; t < NIT; ++t) {
        a[t] = load_a(c0 + cl, lhi + 2 * t);
        m[t] = load_m(c0 + cl, lhi + 2 * t);
      }
    };
    auto product = [&](int cl, const bf16x8 (&a)[NIT], const bf16x8 (&m)[NIT]) {
      f32x16 acc;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
      for (int t = 0; t < NIT; ++t) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[t], m[t], acc, 0, 0, 0);
      leave(cl, acc);
    };
    int cl = wave;
    if (cl < gk) fetch(cl, a0, m0);
    while (cl < gk) {
      if (cl + 4 < gk) fetch(cl + 4, a1, m1);
      product(cl, a0, m0);
      cl += 4;
      if (cl >= gk) break;
      if (cl + 4 < gk) fetch(cl + 4, a0, m0);
      product(cl, a1, m1);
      cl += 4;
    }
  } else {
    for (int cl = wave; cl < gk; cl += 4) {
      f32x16 acc;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = 0.f;
      for (int kc = lhi; kc < pp / 8; kc += 2)           // 8-pixel chunk of the patch
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(load_a(c0 + cl, kc), load_m(c0 + cl, kc), acc, 0, 0, 0);
      leave(cl, acc);
    }
  }
  __syncthreads();
  for (int pr = threadIdx.x; pr < heads * 32; pr += 256) {         // (head, patch), patch fastest
    float* col = sc + (size_t)(pr >> 5) * 33 + (pr & 31);
    const int stride = heads * 33;
    float mx = -INFINITY;
    for (int cl = 0; cl < gk; ++cl) mx = fmaxf(mx, col[cl * stride]);
    float den = 0.f;
    for (int cl = 0; cl < gk; ++cl) den += __expf(col[cl * stride] - mx);
    const float inv = 1.f / den;
    for (int cl = 0; cl < gk; ++cl) col[cl * stride] = __expf(col[cl * stride] - mx) * inv;
  }
  __syncthreads();
  if (alpha_f) {
    for (int idx = threadIdx.x; idx < gpad * heads * 8; idx += 256) {       // four patches per thread: 16-byte stores
      const int quad = idx & 7, head = (idx >> 3) % heads, cl = (idx >> 3) / heads;
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        v[e] = (cl < gk && n0 + 4 * quad + e < N) ? sc[((size_t)cl * heads + head) * 33 + 4 * quad + e] : 0.f;
      *reinterpret_cast<f32x4*>(alpha_f + ((((size_t)b * G + k) * gpad + cl) * heads + head) * Np + n0 + 4 * quad) = v;
    }
  }
  if (alpha_tm) {
    const int hq = heads / 4;                            // heads % 4 == 0: four heads per thread, 16-byte stores
    for (int idx = threadIdx.x; idx < gk * 32 * hq; idx += 256) {
      const int h4 = idx % hq, patch = (idx / hq) & 31, cl = idx / (hq * 32);
      if (n0 + patch < N) {
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = sc[((size_t)cl * heads + 4 * h4 + e) * 33 + patch];
        *reinterpret_cast<f32x4*>(alpha_tm + (((size_t)b * C + c0 + cl) * N + n0 + patch) * heads + 4 * h4) = v;
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Tokenizer on MFMA (paper Section 2.1: every patch of every channel is embedded on its own by
// that channel's convolution, kernel = stride = patch):
//   tokens[b,c,n,d] = sum_k u[b,c,n][k] * We[c][d][k] + be[c][d] + ce[c][d],   k = p*p pixels of the patch
// grid (ceil(N/128), C, B), block 256.  The block gathers its 128 patches into LDS (rows of p*p bf16,
// padded by 16 bytes), then every wavefront sweeps 64-column slices: 4 x 2 MFMA blocks whose two
// column blocks interleave (block j holds columns 2*lane+j), so that a lane owns two adjacent
// outputs per row and half a wavefront stores 128 contiguous bytes.
// Requires p*p % 16 == 0, p*p <= 256, D % 64 == 0.  The kernel is HBM-write bound.
// ---------------------------------------------------------------------------------------------
// KSS = p*p / 16 when that is 1, 2 or 4 (the weight fragments of the next column slice are then fetched while
// the current slice is multiplied and stored), 0 for any other patch size (fragments fetched step by step).
template <int KSS>
__global__ __launch_bounds__(256, 2) void k_tokenize_mfma(int C, int H, int W, int p, int D, const bf16* __restrict__ x,
                                                       const bf16* __restrict__ We, const bf16* __restrict__ be,
                                                       const bf16* __restrict__ ce, bf16* __restrict__ tokens) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  const int pp = p * p, pw = W / p, N = (H / p) * pw;
  const int KS = KSS ? KSS : pp / 16;
  const int rbp = pp * 2 + 16;                           // padded bytes per patch row
  const int n0 = blockIdx.x * 128, c = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, lhi = lane >> 5;
  const bf16* img = x + ((size_t)b * C + c) * H * W;

  // gather: 4 pixels (8 bytes) at a time, eight pieces of a thread in flight; p % 4 == 0 keeps every piece inside one patch
  // row.  (One piece after another, 32 round trips to memory for 16 x 16 patches: 39 us for 2 x 77 channels of 135, D 384.)
  const int pieces = pp / 4, prow = p / 4;
  for (int i0 = tid; i0 < 128 * pieces; i0 += 8 * 256) {
    bf16x4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int idx = i0 + u * 256, t = idx / pieces, q = idx % pieces, n = n0 + t;
      v[u] = bf16x4{};
      if (idx < 128 * pieces && n < N)
        v[u] = *reinterpret_cast<const bf16x4*>(img + (size_t)((n / pw) * p + q / prow) * W + (n % pw) * p + (q % prow) * 4);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int idx = i0 + u * 256;
      if (idx < 128 * pieces) *reinterpret_cast<bf16x4*>(smem + (idx / pieces) * rbp + (idx % pieces) * 8) = v[u];
    }
  }
  __syncthreads();

  const bf16* Wc = We + (size_t)c * D * pp;
  // uniform tile base + per-lane byte offset (the two half-wavefronts sit 4 rows apart); a tile spans at most
  // 128 rows of 2 D bytes, so 32-bit offsets do
  typedef __attribute__((address_space(1))) unsigned char gbyte_t;
  typedef __attribute__((address_space(1))) bf16x2 gbf16x2_t;
  gbyte_t* tbase = (gbyte_t*)(tokens + (((size_t)b * C + c) * N + n0) * D);
  const unsigned rowb = (unsigned)D * 2;
  const int nlim = N - n0 - 4 * lhi;                     // rows of this lane's half that are inside the image
  const bool full = n0 + 128 <= N;                       // uniform: no row of the tile is outside

  constexpr int NF = KSS ? KSS : 1;
  bf16x8 bfrag[NF][2];                                   // weight fragments of the slice about to be multiplied
  if (KSS) {
    // a wavefront whose first slice lies past D (D < 256) never enters the loop below: it preloads slice 0 instead,
    // so that no read leaves We
    const int colp = wave * 64 < D ? wave * 64 : 0;
    const bf16* wrow = Wc + (size_t)(colp + 2 * l32) * pp + lhi * 8;
#pragma unroll
    for (int kk = 0; kk < NF; ++kk)
#pragma unroll
      for (int j = 0; j < 2; ++j) bfrag[kk][j] = *reinterpret_cast<const bf16x8*>(wrow + (size_t)j * pp + kk * 16);
  }
  const unsigned rowb5 = 5 * rowb;
  for (int col0 = wave * 64; col0 < D; col0 += 256) {
    f32x16 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    const int d0 = col0 + 2 * l32;
    if (KSS) {
#pragma unroll
      for (int kk = 0; kk < NF; ++kk) {
        bf16x8 af[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          af[i] = *reinterpret_cast<const bf16x8*>(smem + (i * 32 + l32) * rbp + (kk * 2 + lhi) * 16);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfrag[kk][j], acc[i][j], 0, 0, 0);
      }
      // fetch the slice after this one while this one is stored (the last slice fetches itself again:
      // in bounds, unused)
      const int coln = col0 + 256 < D ? col0 + 256 : col0;
      const bf16* wrow = Wc + (size_t)(coln + 2 * l32) * pp + lhi * 8;
#pragma unroll
      for (int kk = 0; kk < NF; ++kk)
#pragma unroll
        for (int j = 0; j < 2; ++j) bfrag[kk][j] = *reinterpret_cast<const bf16x8*>(wrow + (size_t)j * pp + kk * 16);
    } else {
      const bf16* wrow = Wc + (size_t)d0 * pp + lhi * 8;
      for (int kk = 0; kk < KS; ++kk) {
        bf16x8 bfr[2], af[4];
#pragma unroll
        for (int j = 0; j < 2; ++j) bfr[j] = *reinterpret_cast<const bf16x8*>(wrow + (size_t)j * pp + kk * 16);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          af[i] = *reinterpret_cast<const bf16x8*>(smem + (i * 32 + l32) * rbp + (kk * 2 + lhi) * 16);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
      }
    }
    float add0 = 0.f, add1 = 0.f;
    if (be) { add0 += (float)be[(size_t)c * D + d0]; add1 += (float)be[(size_t)c * D + d0 + 1]; }
    if (ce) { add0 += (float)ce[(size_t)c * D + d0]; add1 += (float)ce[(size_t)c * D + d0 + 1]; }
    // rows of a lane in register order: 0 1 2 3 8 9 10 11 16 ... (steps of 1, 1, 1, 5 rows).  The row pointer
    // is uniform and walks in scalar registers; the asm keeps the compiler from precomputing all 64 of them
    // outside the slice loop (which costs more registers than there are).
    const unsigned lane_off = (unsigned)(4 * lhi * D + d0) * 2;
    gbyte_t* rowp = tbase;
    asm volatile("" : "+s"(rowp));
    if (full) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          bf16x2 pk;
          pk[0] = (bf16)(acc[i][0][r] + add0);
          pk[1] = (bf16)(acc[i][1][r] + add1);
          *(gbf16x2_t*)(rowp + lane_off) = pk;
          rowp += (r & 3) == 3 ? rowb5 : rowb;
        }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int rr = i * 32 + 8 * (r >> 2) + (r & 3);  // uniform row index inside the tile
          if (rr < nlim) {
            bf16x2 pk;
            pk[0] = (bf16)(acc[i][0][r] + add0);
            pk[1] = (bf16)(acc[i][1][r] + add1);
            *(gbf16x2_t*)(rowp + lane_off) = pk;
          }
          rowp += (r & 3) == 3 ? rowb5 : rowb;
        }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Tokenizer on MFMA, weight-stationary form for p*p = 16 * KSS, KSS in {1, 2, 4}, D % 256 == 0 (same result
// as k_tokenize_mfma).  grid (D / 256, C, TS), block 256: wavefront w of block (x, c, z) owns the 64 columns
// 256 x + 64 w .. + 63 of channel c, loads their weight fragments ONCE and then walks the 128-patch tiles
// [z * per, (z + 1) * per) of the B * ceil(N / 128) tiles of its channel.  The patches of the next tile are
// fetched into registers while the current tile is multiplied and stored, and handed over through one of two
// LDS buffers (one barrier per tile).  Dynamic LDS: 2 * 128 * (p*p*2 + 16) bytes.  HBM-write bound.
// ---------------------------------------------------------------------------------------------
template <int KSS>
__global__ __launch_bounds__(256, 2) void k_tokenize_ws(int B, int C, int H, int W, int p, int D, int per,
                                                        const bf16* __restrict__ x, const bf16* __restrict__ We,
                                                        const bf16* __restrict__ be, const bf16* __restrict__ ce,
                                                        bf16* __restrict__ tokens) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  typedef __attribute__((address_space(1))) unsigned char gbyte_t;
  typedef __attribute__((address_space(1))) bf16x2 gbf16x2_t;
  constexpr int pp = 16 * KSS, pieces = pp / 4;          // 8-byte pieces per patch
  constexpr int rbp = pp * 2 + 16;                       // padded bytes per patch row
  constexpr int NG = 128 * pieces / 256;                 // pieces a thread gathers per tile
  const int pw = W / p, N = (H / p) * pw;
  const int ntile = (N + 127) / 128, T = B * ntile;
  const int c = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, lhi = lane >> 5;
  const int d0 = blockIdx.x * 256 + wave * 64 + 2 * l32;   // this lane's two adjacent columns
  const int t_begin = blockIdx.z * per, t_end = min(T, t_begin + per);
  if (t_begin >= t_end) return;                          // uniform over the block

  bf16x8 bfrag[KSS][2];
  {
    const bf16* wrow = We + ((size_t)c * D + d0) * pp + lhi * 8;
#pragma unroll
    for (int kk = 0; kk < KSS; ++kk)
#pragma unroll
      for (int j = 0; j < 2; ++j) bfrag[kk][j] = *reinterpret_cast<const bf16x8*>(wrow + (size_t)j * pp + kk * 16);
  }
  float add0 = 0.f, add1 = 0.f;
  if (be) { add0 += (float)be[(size_t)c * D + d0]; add1 += (float)be[(size_t)c * D + d0 + 1]; }
  if (ce) { add0 += (float)ce[(size_t)c * D + d0]; add1 += (float)ce[(size_t)c * D + d0 + 1]; }

  // gather of tile t: piece idx = tid + 256 * i covers patch idx / pieces, pixels 4 * (idx % pieces) .. + 3
  bf16x4 gv[NG];
  auto fetch = [&](int t) {
    const int b = t / ntile, n0 = (t % ntile) * 128;
    const bf16* img = x + ((size_t)b * C + c) * H * W;
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const int idx = tid + 256 * i;
      const int tp = idx / pieces, q = idx % pieces;
      const int r = (q * 4) / p, s0 = (q * 4) % p;
      const int n = n0 + tp;
      gv[i] = bf16x4{};
      if (n < N) {
        const int pi = n / pw, pj = n % pw;
        gv[i] = *reinterpret_cast<const bf16x4*>(img + (size_t)(pi * p + r) * W + pj * p + s0);
      }
    }
  };
  auto stash = [&](int buf) {
    unsigned char* u = smem + buf * 128 * rbp;
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const int idx = tid + 256 * i;
      *reinterpret_cast<bf16x4*>(u + (idx / pieces) * rbp + (idx % pieces) * 8) = gv[i];
    }
  };
  fetch(t_begin);
  stash(0);
  __syncthreads();

  const unsigned rowb = (unsigned)D * 2, rowb5 = 5 * rowb;
  const unsigned lane_off = (unsigned)(4 * lhi * D + d0) * 2;
  for (int t = t_begin; t < t_end; ++t) {
    const int cur = (t - t_begin) & 1;
    if (t + 1 < t_end) fetch(t + 1);
    const unsigned char* u = smem + cur * 128 * rbp;
    f32x16 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < KSS; ++kk) {
      bf16x8 af[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        af[i] = *reinterpret_cast<const bf16x8*>(u + (i * 32 + l32) * rbp + (kk * 2 + lhi) * 16);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfrag[kk][j], acc[i][j], 0, 0, 0);
    }
    // rows of a lane in register order: 0 1 2 3 8 9 10 11 16 ... (steps of 1, 1, 1, 5 rows); the row pointer
    // is uniform and walks in scalar registers (the asm keeps it from being expanded into 64 precomputed ones)
    const int b = t / ntile, n0 = (t % ntile) * 128;
    gbyte_t* rowp = (gbyte_t*)(tokens + (((size_t)b * C + c) * N + n0) * D);
    asm volatile("" : "+s"(rowp));
    if (n0 + 128 <= N) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          bf16x2 pk;
          pk[0] = (bf16)(acc[i][0][r] + add0);
          pk[1] = (bf16)(acc[i][1][r] + add1);
          *(gbf16x2_t*)(rowp + lane_off) = pk;
          rowp += (r & 3) == 3 ? rowb5 : rowb;
        }
    } else {
      const int nlim = N - n0 - 4 * lhi;                 // rows of this lane's half that are inside the image
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int rr = i * 32 + 8 * (r >> 2) + (r & 3);
          if (rr < nlim) {
            bf16x2 pk;
            pk[0] = (bf16)(acc[i][0][r] + add0);
            pk[1] = (bf16)(acc[i][1][r] + add1);
            *(gbf16x2_t*)(rowp + lane_off) = pk;
          }
          rowp += (r & 3) == 3 ? rowb5 : rowb;
        }
    }
    if (t + 1 < t_end) stash(cur ^ 1);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------------
// Tokenizer fused with a linear first level (D-CHAG-L: paper Section 2.1 tokenization, Sections 3.2/3.3
// linear partial aggregation): the tokens of a group are mixed as they are produced and never reach HBM,
//   y[b,k,n,d] = sum_{cl < gk} w[k][cl][d] * (We[c] u[b,c,n] + be[c] + ce[c])[d] + bias[k][d],   c = k*g + cl.
// grid (ceil(N/64) * (D/256), G, B), block 256: 64 patches x 256 columns x all members of one group.
// Wavefront w owns columns 64 w .. 64 w + 63 of the block's slice as 2 x 2 MFMA blocks (the two column
// blocks interleave as in k_tokenize_mfma).  Members are pipelined: while member cl is multiplied, scaled by
// its weight of the lane's column and added up in registers, the 64 patches and the weight fragments of member
// cl + 1 are already on their way (patches through registers into the other of two LDS buffers, one barrier
// per member).  p*p = 16 * KSS, KSS in {1, 4}; D % 256 == 0.  Dynamic LDS: 2 * 64 * (p*p*2 + 16) bytes.
// ---------------------------------------------------------------------------------------------
template <int KSS>
__global__ __launch_bounds__(256, 2) void k_tokenize_mix_mfma(int C, int H, int W, int p, int D, int g,
                                                              const bf16* __restrict__ x, const bf16* __restrict__ We,
                                                              const bf16* __restrict__ be, const bf16* __restrict__ ce,
                                                              const bf16* __restrict__ wmix,
                                                              const bf16* __restrict__ bias, bf16* __restrict__ y) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  constexpr int pp = 16 * KSS, pieces = pp / 4;
  constexpr int rbp = pp * 2 + 16;
  constexpr int NG = (64 * pieces + 255) / 256;          // 8-byte pieces a thread gathers per member
  const int pw = W / p, N = (H / p) * pw;
  const int ns_n = D / 256;
  const int n0 = (blockIdx.x / ns_n) * 64, col_base = (blockIdx.x % ns_n) * 256;
  const int k = blockIdx.y, b = blockIdx.z, G = gridDim.y;
  const int c0 = k * g, gk = min(g, C - c0);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, lhi = lane >> 5;
  const int d0 = col_base + wave * 64 + 2 * l32;         // this lane's two adjacent columns

  // what member cl needs: its patches (gv), its weight fragments (bfrag) and four per-column scalars
  bf16x4 gv[NG];
  bf16x8 bfrag[KSS][2];
  float w0, w1, a0, a1;
  // source offsets of this thread's pieces inside a channel image (-1: patch outside the image)
  int goff[NG];
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    const int idx = tid + 256 * i;
    const int t = idx / pieces, q = idx % pieces;
    const int r = (q * 4) / p, s0 = (q * 4) % p;
    const int n = n0 + t;
    goff[i] = (idx < 64 * pieces && n < N) ? ((n / pw) * p + r) * W + (n % pw) * p + s0 : -1;
  }
  auto fetch = [&](int cl) {
    const int c = c0 + cl;
    const bf16* img = x + ((size_t)b * C + c) * H * W;
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      gv[i] = bf16x4{};
      if (goff[i] >= 0) gv[i] = *reinterpret_cast<const bf16x4*>(img + goff[i]);
    }
    const bf16* wrow = We + ((size_t)c * D + d0) * pp + lhi * 8;
#pragma unroll
    for (int kk = 0; kk < KSS; ++kk)
#pragma unroll
      for (int j = 0; j < 2; ++j) bfrag[kk][j] = *reinterpret_cast<const bf16x8*>(wrow + (size_t)j * pp + kk * 16);
    w0 = (float)wmix[((size_t)k * g + cl) * D + d0];
    w1 = (float)wmix[((size_t)k * g + cl) * D + d0 + 1];
    a0 = 0.f;
    a1 = 0.f;
    if (be) { a0 += (float)be[(size_t)c * D + d0]; a1 += (float)be[(size_t)c * D + d0 + 1]; }
    if (ce) { a0 += (float)ce[(size_t)c * D + d0]; a1 += (float)ce[(size_t)c * D + d0 + 1]; }
  };
  auto stash = [&](int buf) {
    unsigned char* u = smem + buf * 64 * rbp;
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const int idx = tid + 256 * i;
      if (idx < 64 * pieces) *reinterpret_cast<bf16x4*>(u + (idx / pieces) * rbp + (idx % pieces) * 8) = gv[i];
    }
  };

  f32x16 o[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[i][j][r] = 0.f;
  float cst0 = 0.f, cst1 = 0.f;                          // patch-independent part: sum_c w * (be + ce) + bias

  fetch(0);
  stash(0);
  __syncthreads();
  for (int cl = 0; cl < gk; ++cl) {
    const unsigned char* u = smem + (cl & 1) * 64 * rbp;
    // this member's operands move to their own registers; the next member's loads start right away
    bf16x8 bcur[KSS][2];
#pragma unroll
    for (int kk = 0; kk < KSS; ++kk)
#pragma unroll
      for (int j = 0; j < 2; ++j) bcur[kk][j] = bfrag[kk][j];
    const float cw0 = w0, cw1 = w1;
    cst0 += w0 * a0;
    cst1 += w1 * a1;
    if (cl + 1 < gk) fetch(cl + 1);
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      f32x16 acc0 = zero, acc1 = zero;                   // two independent chains: row block i, both column blocks
#pragma unroll
      for (int kk = 0; kk < KSS; ++kk) {
        const bf16x8 af = *reinterpret_cast<const bf16x8*>(u + (i * 32 + l32) * rbp + (kk * 2 + lhi) * 16);
        acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, bcur[kk][0], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, bcur[kk][1], acc1, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        o[i][0][r] += cw0 * acc0[r];
        o[i][1][r] += cw1 * acc1[r];
      }
    }
    if (cl + 1 < gk) stash((cl + 1) & 1);
    __syncthreads();
  }
  if (bias) { cst0 += (float)bias[(size_t)k * D + d0]; cst1 += (float)bias[(size_t)k * D + d0 + 1]; }
  bf16* ybase = y + (((size_t)b * G + k) * N + n0) * D;
  const int lane_off = 4 * lhi * D + d0;
  const int nlim = N - n0 - 4 * lhi;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int rr = i * 32 + 8 * (r >> 2) + (r & 3);
      if (rr < nlim) {
        bf16x2 pk;
        pk[0] = (bf16)(o[i][0][r] + cst0);
        pk[1] = (bf16)(o[i][1][r] + cst1);
        *reinterpret_cast<bf16x2*>(ybase + (size_t)rr * D + lane_off) = pk;
      }
    }
}

// The same with 128 patches x 256 columns per workgroup of eight wavefronts (wavefront w: columns 32 w .. 32 w + 31,
// 4 row blocks): every workgroup re-reads the tokenizer weights of its members and gathers their pixels once per column
// slice, so the larger patch tile halves the weight traffic at the same pixel traffic.  grid (ceil(N/128) * (D/256), G, B),
// block 512.  Dynamic LDS: 2 * 128 * (p*p*2 + 16) bytes.
template <int KSS>
__global__ __launch_bounds__(512) void k_tokenize_mix_wide(int C, int H, int W, int p, int D, int g,
                                                              const bf16* __restrict__ x, const bf16* __restrict__ We,
                                                              const bf16* __restrict__ be, const bf16* __restrict__ ce,
                                                              const bf16* __restrict__ wmix,
                                                              const bf16* __restrict__ bias, bf16* __restrict__ y) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  constexpr int pp = 16 * KSS, pieces = pp / 4;
  constexpr int rbp = pp * 2 + 16;
  constexpr int PB = 128;                                // patches per workgroup
  constexpr int NG = (PB * pieces + 511) / 512;          // 8-byte pieces a thread gathers per member
  const int pw = W / p, N = (H / p) * pw;
  const int ns_n = D / 256;
  const int n0 = (blockIdx.x / ns_n) * PB, col_base = (blockIdx.x % ns_n) * 256;
  const int k = blockIdx.y, b = blockIdx.z, G = gridDim.y;
  const int c0 = k * g, gk = min(g, C - c0);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, lhi = lane >> 5;
  const int d0 = col_base + wave * 32 + l32;             // this lane's column

  // what member cl needs: its patches (gv), its weight fragments (bfrag) and four per-column scalars
  bf16x4 gv[NG];
  bf16x8 bfrag[KSS];
  float w0, a0;
  // source offsets of this thread's pieces inside a channel image (-1: patch outside the image)
  int goff[NG];
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    const int idx = tid + 512 * i;
    const int t = idx / pieces, q = idx % pieces;
    const int r = (q * 4) / p, s0 = (q * 4) % p;
    const int n = n0 + t;
    goff[i] = (idx < PB * pieces && n < N) ? ((n / pw) * p + r) * W + (n % pw) * p + s0 : -1;
  }
  auto fetch = [&](int cl) {
    const int c = c0 + cl;
    const bf16* img = x + ((size_t)b * C + c) * H * W;
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      gv[i] = bf16x4{};
      if (goff[i] >= 0) gv[i] = *reinterpret_cast<const bf16x4*>(img + goff[i]);
    }
    const bf16* wrow = We + ((size_t)c * D + d0) * pp + lhi * 8;
#pragma unroll
    for (int kk = 0; kk < KSS; ++kk) bfrag[kk] = *reinterpret_cast<const bf16x8*>(wrow + kk * 16);
    w0 = (float)wmix[((size_t)k * g + cl) * D + d0];
    a0 = 0.f;
    if (be) a0 += (float)be[(size_t)c * D + d0];
    if (ce) a0 += (float)ce[(size_t)c * D + d0];
  };
  auto stash = [&](int buf) {
    unsigned char* u = smem + buf * PB * rbp;
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const int idx = tid + 512 * i;
      if (idx < PB * pieces) *reinterpret_cast<bf16x4*>(u + (idx / pieces) * rbp + (idx % pieces) * 8) = gv[i];
    }
  };

  f32x16 o[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[i][r] = 0.f;
  float cst0 = 0.f;                                      // patch-independent part: sum_c w * (be + ce) + bias

  fetch(0);
  stash(0);
  __syncthreads();
  for (int cl = 0; cl < gk; ++cl) {
    const unsigned char* u = smem + (cl & 1) * PB * rbp;
    // this member's operands move to their own registers; the next member's loads start right away
    bf16x8 bcur[KSS];
#pragma unroll
    for (int kk = 0; kk < KSS; ++kk) bcur[kk] = bfrag[kk];
    const float cw0 = w0;
    cst0 += w0 * a0;
    if (cl + 1 < gk) fetch(cl + 1);
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; i += 2) {
      f32x16 acc0 = zero, acc1 = zero;                   // two independent chains: row blocks i and i + 1
#pragma unroll
      for (int kk = 0; kk < KSS; ++kk) {
        const bf16x8 af0 = *reinterpret_cast<const bf16x8*>(u + (i * 32 + l32) * rbp + (kk * 2 + lhi) * 16);
        const bf16x8 af1 = *reinterpret_cast<const bf16x8*>(u + ((i + 1) * 32 + l32) * rbp + (kk * 2 + lhi) * 16);
        acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af0, bcur[kk], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af1, bcur[kk], acc1, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        o[i][r] += cw0 * acc0[r];
        o[i + 1][r] += cw0 * acc1[r];
      }
    }
    if (cl + 1 < gk) stash((cl + 1) & 1);
    __syncthreads();
  }
  if (bias) cst0 += (float)bias[(size_t)k * D + d0];
  bf16* ybase = y + (((size_t)b * G + k) * N + n0) * D;
  const int lane_off = 4 * lhi * D + d0;
  const int nlim = N - n0 - 4 * lhi;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int rr = i * 32 + 8 * (r >> 2) + (r & 3);
      if (rr < nlim) ybase[(size_t)rr * D + lane_off] = (bf16)(o[i][r] + cst0);
    }
}

// The attention form of k_tokenize_mix_wide (cross-attention first level with the value projection folded into the
// tokenizer weights: Wf[c] = Wv[k] We[c], v1 = Wv be, v2 = Wv ce), for the shapes the ring kernel below does not take
// (16 pixels per patch, heads of 32 columns, unaligned images):
//   y[b,k,n,d] = sum_{cl < gk} alpha[b][k][cl][head(d)][n] * (Wf[c] u[b,c,n] + v1[c] + v2[c])[d] + bias[k][d].
// The member's constant enters as the MFMA's C operand; its softmax weights (NHS heads x 128 patches, fp32) travel with
// the patches through registers into LDS.  Requires (D / heads) % 32 == 0 and 256 % dh == 0 or dh % 256 == 0.
// Dynamic LDS: 2 * 128 * (p*p*2 + 16) + 2 * NHS * 512 bytes.
template <int KSS>
__global__ __launch_bounds__(512) void k_tokenize_attend_wide(int C, int H, int W, int p, int D, int g, int heads,
                                                              int gpad, int Np, const bf16* __restrict__ x,
                                                              const bf16* __restrict__ Wf, const bf16* __restrict__ v1,
                                                              const bf16* __restrict__ v2,
                                                              const float* __restrict__ alpha,
                                                              const bf16* __restrict__ bias, bf16* __restrict__ y) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int pp = 16 * KSS, pieces = pp / 4;
  constexpr int rbp = pp * 2 + 16;
  constexpr int PB = 128;                                // patches per workgroup
  constexpr int NG = (PB * pieces + 511) / 512;          // 8-byte pieces a thread gathers per member
  const int pw = W / p, N = (H / p) * pw;
  const int ns_n = D / 256;
  const int n0 = (blockIdx.x / ns_n) * PB, col_base = (blockIdx.x % ns_n) * 256;
  const int k = blockIdx.y, b = blockIdx.z, G = gridDim.y;
  const int c0 = k * g, gk = min(g, C - c0);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, lhi = lane >> 5;
  const int d0 = col_base + wave * 32 + l32;             // this lane's column
  const int dh = D / heads, nhs = dh >= 256 ? 1 : 256 / dh, h0 = col_base / dh;
  const int hrel = (col_base + wave * 32) / dh - h0;     // the wavefront's 32 columns lie in one head
  unsigned char* alds = smem + 2 * PB * rbp;             // [2][nhs][128] floats

  bf16x4 gv[NG];
  bf16x8 bfrag[KSS];
  f32x4 av = {0.f, 0.f, 0.f, 0.f};
  float a0;
  int goff[NG];
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    const int idx = tid + 512 * i;
    const int t = idx / pieces, q = idx % pieces;
    const int r = (q * 4) / p, s0 = (q * 4) % p;
    const int n = n0 + t;
    goff[i] = (idx < PB * pieces && n < N) ? ((n / pw) * p + r) * W + (n % pw) * p + s0 : -1;
  }
  // thread t < 32 nhs fetches the weights of head h0 + t / 32 for patches n0 + 4 (t % 32) .. + 3
  const float* asrc = alpha + ((((size_t)b * G + k) * gpad) * heads + h0 + min(tid >> 5, nhs - 1)) * Np +
                      min(n0 + 4 * (tid & 31), Np - 4);
  auto fetch = [&](int cl) {
    const int c = c0 + cl;
    const bf16* img = x + ((size_t)b * C + c) * H * W;
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      gv[i] = bf16x4{};
      if (goff[i] >= 0) gv[i] = *reinterpret_cast<const bf16x4*>(img + goff[i]);
    }
    const bf16* wrow = Wf + ((size_t)c * D + d0) * pp + lhi * 8;
#pragma unroll
    for (int kk = 0; kk < KSS; ++kk) bfrag[kk] = *reinterpret_cast<const bf16x8*>(wrow + kk * 16);
    a0 = 0.f;
    if (v1) a0 += (float)v1[(size_t)c * D + d0];
    if (v2) a0 += (float)v2[(size_t)c * D + d0];
    if (tid < 32 * nhs) av = *reinterpret_cast<const f32x4*>(asrc + (size_t)cl * heads * Np);
  };
  auto stash = [&](int buf) {
    unsigned char* u = smem + buf * PB * rbp;
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const int idx = tid + 512 * i;
      if (idx < PB * pieces) *reinterpret_cast<bf16x4*>(u + (idx / pieces) * rbp + (idx % pieces) * 8) = gv[i];
    }
    if (tid < 32 * nhs) *reinterpret_cast<f32x4*>(alds + buf * nhs * 512 + tid * 16) = av;
  };

  f32x16 o[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[i][r] = 0.f;

  fetch(0);
  stash(0);
  __syncthreads();
  for (int cl = 0; cl < gk; ++cl) {
    const unsigned char* u = smem + (cl & 1) * PB * rbp;
    const float* al = reinterpret_cast<const float*>(alds + (cl & 1) * nhs * 512 + hrel * 512) + 4 * lhi;
    bf16x8 bcur[KSS];
#pragma unroll
    for (int kk = 0; kk < KSS; ++kk) bcur[kk] = bfrag[kk];
    const float cb = a0;
    if (cl + 1 < gk) fetch(cl + 1);
    const f32x16 init = {cb, cb, cb, cb, cb, cb, cb, cb, cb, cb, cb, cb, cb, cb, cb, cb};
#pragma unroll
    for (int i = 0; i < 4; i += 2) {
      f32x16 acc0 = init, acc1 = init;                   // two independent chains: row blocks i and i + 1
#pragma unroll
      for (int kk = 0; kk < KSS; ++kk) {
        const bf16x8 af0 = *reinterpret_cast<const bf16x8*>(u + (i * 32 + l32) * rbp + (kk * 2 + lhi) * 16);
        const bf16x8 af1 = *reinterpret_cast<const bf16x8*>(u + ((i + 1) * 32 + l32) * rbp + (kk * 2 + lhi) * 16);
        acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af0, bcur[kk], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af1, bcur[kk], acc1, 0, 0, 0);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 w0 = *reinterpret_cast<const f32x4*>(al + i * 32 + 8 * q);
        const f32x4 w1 = *reinterpret_cast<const f32x4*>(al + (i + 1) * 32 + 8 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          o[i][4 * q + e] += w0[e] * acc0[4 * q + e];
          o[i + 1][4 * q + e] += w1[e] * acc1[4 * q + e];
        }
      }
    }
    if (cl + 1 < gk) stash((cl + 1) & 1);
    __syncthreads();
  }
  const float add = bias ? (float)bias[(size_t)k * D + d0] : 0.f;
  bf16* ybase = y + (((size_t)b * G + k) * N + n0) * D;
  const int lane_off = 4 * lhi * D + d0;
  const int nlim = N - n0 - 4 * lhi;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int rr = i * 32 + 8 * (r >> 2) + (r & 3);
      if (rr < nlim) ybase[(size_t)rr * D + lane_off] = (bf16)(o[i][r] + add);
    }
}

// ---------------------------------------------------------------------------------------------
// Tokenizer fused with the first aggregation level, operands streamed through a three-stage LDS ring
// (8 x 8 patches only: a patch and a weight row are both one 128-byte LDS row).  Two forms:
//   ATT = false (D-CHAG-L, paper Sections 3.2/3.3: linear partial aggregation)
//     y[b,k,n,d] = sum_cl wmix[k][cl][d] * (Wt[c] u[b,c,n] + v1[c] + v2[c])[d] + bias[k][d]
//   ATT = true (cross-attention level, paper Section 2.1, with the value projection folded into the tokenizer
//     weights: Wt[c] = Wv[k] We[c], v1 = Wv be, v2 = Wv ce; exact because the softmax weights sum to one)
//     y[b,k,n,d] = sum_cl alpha[b][k][cl][head(d)][n] * (Wt[c] u[b,c,n] + v1[c] + v2[c])[d] + bias[k][d]
// c = k*g + cl; u = the 64 pixels of patch n; alpha laid out [B][G][gpad][heads][Np] (fp32).
// Workgroup = 128 patches x 256 columns x all members of one group; wavefront (wm, wn) of 2 x 4 owns 64 patches x
// 64 columns as 2 x 2 MFMA blocks.  One ring stage = one member: its 128 patches (16 KiB, gathered from the image
// 16 bytes per lane), its 256 weight rows (32 KiB) and 4 KiB of per-member vectors (per-column scalars, softmax
// weights of the slice's heads), all by direct-to-LDS loads issued two members ahead; one barrier per member.
// Workgroups are dealt to the XCDs in contiguous ranges of the (k, b, patch tile, column slice) order, so the
// workgroups that share a member's weights or a patch tile meet in one L2.
// With S > 1 the members of a group are dealt to S workgroups per tile (few groups: not enough tiles to fill the
// chip otherwise); each writes its fp32 partial sums to ypart [S][B][G][N][D] and k_vagg_merge adds them and the bias.
// Requires D % 256 == 0, W % 8 == 0, 16-byte aligned x; ATT: (D / heads) % 64 == 0 and 256 % dh == 0 or dh % 256 == 0.
// Dynamic LDS: kRedLdsBytes.
// ---------------------------------------------------------------------------------------------
// Workgroup shapes of k_tokenize_reduce_ring.  CFG 0: 128 patches x 256 columns, 8 wavefronts (2 x 4) of 64 x 64, three
// stages, one workgroup per compute unit.  CFG 1: 128 x 128, 4 wavefronts (2 x 2) of 64 x 64, two stages, two workgroups
// per compute unit (the one taken: 0.107 against 0.114 ms at the headline shape; 64 x 128 with wavefronts of 64 x 32,
// three workgroups per compute unit, was slower than both: 0.127 ms).
template <int CFG>
struct RedCfg {
  static constexpr int kPatches = 128;
  static constexpr int WM = kPatches / 64, WN = CFG == 1 ? 2 : 4, TN = 2;
  static constexpr int kWaves = WM * WN, kThreads = kWaves * 64, kCols = WN * TN * 32;
  static constexpr int kABytes = kPatches * 128, kBBytes = kCols * 128, kXBytes = 4096;
  static constexpr int kStageBytes = kABytes + kBBytes + kXBytes;           // 52 or 36 KiB
  static constexpr int kStages = CFG == 0 ? 3 : 2;
  static constexpr int kPerCu = CFG + 1;                                    // workgroups per compute unit
  static constexpr int kLdsBytes = kStages * kStageBytes;                   // 156 or 72 KiB
};

template <bool ATT, int CFG>
__global__ __launch_bounds__(RedCfg<CFG>::kThreads, RedCfg<CFG>::kPerCu) void k_tokenize_reduce_ring(
    int C, int H, int W, int D, int g, int G, int heads, int gpad, int Np, TileWork tw, const bf16* __restrict__ x,
    const bf16* __restrict__ Wt, const bf16* __restrict__ wmix, const bf16* __restrict__ v1,
    const bf16* __restrict__ v2, const float* __restrict__ alpha, const bf16* __restrict__ bias, bf16* __restrict__ y,
    int S, float* __restrict__ ypart) {
  typedef RedCfg<CFG> Cfg;
  constexpr int WN = Cfg::WN, TN = Cfg::TN, kRedPatches = Cfg::kPatches;
  constexpr int kRedCols = Cfg::kCols, kRedABytes = Cfg::kABytes, kRedBBytes = Cfg::kBBytes;
  constexpr int kRedStageBytes = Cfg::kStageBytes, NS = Cfg::kStages;
  constexpr int AL = kRedPatches / 8 / Cfg::kWaves;      // A loads per wavefront and member
  constexpr int BL = kRedCols / 8 / Cfg::kWaves;         // B loads per wavefront and member
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int k, b, pt, cs, split;
  {
    // position w of the (k, b, patch tile, column slice, split) order; each XCD takes a contiguous range of it
    const int total = tw.total * S, per = (total + kXcds - 1) / kXcds;
    const int w = (blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
    if ((int)(blockIdx.x / kXcds) >= per || w >= total) return;   // uniform: the whole workgroup leaves
    split = w % S;
    tw.decode_linear(w / S, k, b, pt, cs);
  }
  const int pw = W / 8, N = (H / 8) * pw;
  const size_t HW = (size_t)H * W;
  const int n0 = pt * kRedPatches, col_base = cs * kRedCols;
  // this workgroup's members of the group: the S workgroups of a tile share them out evenly
  const int gfull = min(g, C - k * g);
  const int m_lo = split * gfull / S, gk = (split + 1) * gfull / S - m_lo;
  const int c0 = k * g + m_lo;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN, l32 = lane & 31, lhi = lane >> 5;
  const int wcol = wn * TN * 32;                         // first column of this wavefront inside the slice
  const int dh = D / heads;

  // ---- issue side: per-lane sources of this wavefront's loads of one member ----
  const bf16* a_src[AL];
  const bf16* b_src[BL];
#pragma unroll
  for (int i = 0; i < AL; ++i) {
    const int row = wave * (AL * 8) + i * 8 + (lane >> 3);
    const int n = min(n0 + row, N - 1);                  // rows past the image repeat its last patch; never stored
    const int q = (lane & 7) ^ swz_chunk(row);           // logical chunk = pixel row of the patch
    a_src[i] = x + ((size_t)b * C + c0) * HW + (size_t)((n / pw) * 8 + q) * W + (n % pw) * 8;
  }
#pragma unroll
  for (int i = 0; i < BL; ++i) {
    const int row = wave * (BL * 8) + i * 8 + (lane >> 3);
    const int q = (lane & 7) ^ swz_chunk(row);
    b_src[i] = Wt + ((size_t)c0 * D + col_base + row) * 64 + q * 8;
  }
  // The stage's vectors: four per-column vectors of kCols bf16 each (ATT: v1, v2, -, -; else wmix, v1, v2, -) in the
  // first half, filled by the first wavefront(s), 64 / (kCols / 8) vectors per load; in the second half the softmax
  // weights of the slice's heads (kPatches floats each), 64 / (kPatches / 4) heads per load of the next wavefront(s).
  constexpr int LPV = kRedCols / 8, VPI = 64 / LPV, NVW = 4 / VPI;
  constexpr int AOFF = Cfg::kXBytes / 2, LPH = kRedPatches / 4, HPI = 64 / LPH, HB = kRedPatches * 4;
  constexpr int NAW = (kRedCols / 64 + HPI - 1) / HPI;   // heads are at least 64 columns wide
  const unsigned char* e_src = reinterpret_cast<const unsigned char*>(Wt);   // absent vector: any valid 16 bytes
  size_t e_step = 0;
  bool extra = false;
  int e_slot = 0;
  if (wave < NVW && (!ATT || wave == 0)) {
    extra = true;
    e_slot = wave * 1024;
    const int vi = wave * VPI + lane / LPV, lv = lane % LPV;
    const bf16* v = ATT ? (vi == 0 ? v1 : (vi == 1 ? v2 : nullptr)) : (vi == 0 ? wmix : (vi == 1 ? v1 : (vi == 2 ? v2 : nullptr)));
    if (v) {
      const size_t row0 = (!ATT && vi == 0) ? (size_t)k * g + m_lo : (size_t)c0;
      e_src = reinterpret_cast<const unsigned char*>(v + row0 * D + col_base + 8 * lv);
      e_step = (size_t)D * 2;
    }
  } else if (ATT && wave >= NVW && wave < NVW + NAW) {
    extra = true;
    e_slot = AOFF + (wave - NVW) * 1024;
    const int nhs = dh >= kRedCols ? 1 : kRedCols / dh;
    const int head = col_base / dh + min(HPI * (wave - NVW) + lane / LPH, nhs - 1);
    e_src = reinterpret_cast<const unsigned char*>(alpha + ((((size_t)b * G + k) * gpad + m_lo) * heads + head) * Np +
                                                   min(n0 + 4 * (lane % LPH), Np - 4));
    e_step = (size_t)heads * Np * 4;
  }
  extra = __builtin_amdgcn_readfirstlane(extra);
  e_slot = __builtin_amdgcn_readfirstlane(e_slot);
  const size_t b_step = (size_t)D * 64;
  auto issue = [&](int stage) {
    unsigned char* st = smem + stage * kRedStageBytes;
#pragma unroll
    for (int i = 0; i < AL; ++i) {
      load16_to_lds(a_src[i], st + (wave * AL + i) * 1024);
      a_src[i] += HW;
    }
#pragma unroll
    for (int i = 0; i < BL; ++i) {
      load16_to_lds(b_src[i], st + kRedABytes + (wave * BL + i) * 1024);
      b_src[i] += b_step;
    }
    if (extra) {
      load16_to_lds(e_src, st + kRedABytes + kRedBBytes + e_slot);
      e_src += e_step;
    }
  };

  // ---- compute side ----
  const int a_base = (wm * 64 + l32) * 128, b_base = kRedABytes + (wcol + l32) * 128;
  int ck[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) ck[kk] = ((kk * 2 + lhi) ^ swz_chunk(l32)) * 16;
  const int xoff = kRedABytes + kRedBBytes;
  constexpr int VB = kRedCols * 2;                       // bytes of one per-column vector
  const int colj = (wcol + l32) * 2;                     // byte offset of this lane's first column in a vector
  const int hrel = ATT ? (col_base + wcol) / dh - col_base / dh : 0;

  const unsigned short mask1 = v1 ? 0xFFFF : 0, mask2 = v2 ? 0xFFFF : 0;
  f32x16 o[2][TN];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[i][j][r] = 0.f;
  float cst[TN];                                         // ATT = false: patch-independent part sum_c w * (v1 + v2)
#pragma unroll
  for (int j = 0; j < TN; ++j) cst[j] = 0.f;

  if constexpr (NS == 3) {
    // Three stages, a member to each, handed over as a whole.  The barrier sits behind the
    // member's third k-step: by then every fragment of the member is in registers (its last k-step's, its softmax
    // weights / mixing weights too), so the barrier hands its stage to member m + 3 and the next member over to
    // everyone; the fragments of the next member's first k-step are read right behind the barrier and the member's last
    // four products and its scaling into the running sum cover their latency.  Loads run two members ahead.
    struct F2 {
      bf16x8 a[2], b[TN];
    };
    auto read2 = [&](F2& f, const unsigned char* st, int kk) {
#pragma unroll
      for (int i = 0; i < 2; ++i) f.a[i] = *reinterpret_cast<const bf16x8*>(st + a_base + i * 4096 + ck[kk]);
#pragma unroll
      for (int j = 0; j < TN; ++j) f.b[j] = *reinterpret_cast<const bf16x8*>(st + b_base + j * 4096 + ck[kk]);
    };
    f32x16 acc[2][TN];
    auto mfma2 = [&](const F2& f) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[i], f.b[j], acc[i][j], 0, 0, 0);
    };
    auto mfma2_from = [&](const F2& f, const float (&c)[TN]) {       // a member starts from its per-column constant
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const f32x16 init = {c[j], c[j], c[j], c[j], c[j], c[j], c[j], c[j], c[j], c[j], c[j], c[j], c[j], c[j], c[j], c[j]};
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[i], f.b[j], init, 0, 0, 0);
      }
    };
    auto pin = [&]() {                                     // a fragment read behind each of the step's four products
#pragma unroll
      for (int t = 0; t < 2 + TN; ++t) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto vectors_of = [&](const unsigned char* st, float (&vb)[TN], float (&wj)[TN]) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const unsigned char* xs = st + xoff + colj + j * 64;
        auto column_value = [&](int slot, unsigned short mask) {
          const unsigned short raw = *reinterpret_cast<const unsigned short*>(xs + slot * VB) & mask;
          return (float)__builtin_bit_cast(bf16, raw);
        };
        if (ATT) {
          wj[j] = 1.f;
          vb[j] = column_value(0, mask1) + column_value(1, mask2);
        } else {
          wj[j] = column_value(0, 0xFFFF);
          vb[j] = column_value(1, mask1) + column_value(2, mask2);
        }
      }
    };
    if (gk == 0) return;                                   // uniform (the host never deals more shares than members)
    issue(0);
    if (gk > 1) issue(1);
    if (gk > 1) {
      if (extra) wait_vmcnt<AL + BL + 1>();
      else wait_vmcnt<AL + BL>();
    } else {
      wait_vmcnt<0>();
    }
    __builtin_amdgcn_s_barrier();
    if (gk > 2) issue(2);
    F2 f0, f1;
    float vb[TN], wj[TN], vbn[TN], wjn[TN];
    f32x4 areg[2][4];                                      // softmax weights of the member's rows (ATT)
    read2(f0, smem, 0);
    vectors_of(smem, vb, wj);
    int sc = 0;
    for (int m = 0; m < gk; ++m) {
      const unsigned char* st = smem + sc * kRedStageBytes;
      __builtin_amdgcn_sched_barrier(0);
      read2(f1, st, 1);
      if (ATT) mfma2_from(f0, vb);
      else {
        const float zero[TN] = {};
        mfma2_from(f0, zero);
      }
      pin();
      read2(f0, st, 2);
      mfma2(f1);
      pin();
      read2(f1, st, 3);
      mfma2(f0);
      pin();
      if (ATT) {
        const float* al = reinterpret_cast<const float*>(st + xoff + AOFF + hrel * HB) + wm * 64 + 4 * lhi;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q) areg[i][q] = *reinterpret_cast<const f32x4*>(al + i * 32 + 8 * q);
      }
      // member m + 1 has landed (this wavefront's share; member m + 2's loads may stay in flight) and every read of
      // member m's stage is in registers
      if (m + 2 < gk) {
        if (extra) wait_vmcnt<AL + BL + 1>();
        else wait_vmcnt<AL + BL>();
        __builtin_amdgcn_s_waitcnt((7 << 4) | (63 & 15) | ((63 >> 4) << 14));   // lgkmcnt(0), vmcnt untouched
      } else {
        __builtin_amdgcn_s_waitcnt(0);
      }
      __builtin_amdgcn_s_barrier();
      if (m + 3 < gk) issue(sc);                           // member m + 3 -> the stage just released
      sc = sc == 2 ? 0 : sc + 1;
      const unsigned char* sn = smem + sc * kRedStageBytes;
      __builtin_amdgcn_sched_barrier(0);
      read2(f0, sn, 0);                                    // past the last member: a stale stage, read and not used
      vectors_of(sn, vbn, wjn);
      mfma2(f1);
      __builtin_amdgcn_sched_barrier(0);
      if (ATT) {
        // rows of accumulator register r: 8 (r / 4) + 4 lhi + r % 4 of the block
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
              for (int e = 0; e < 4; ++e) o[i][j][4 * q + e] += areg[i][q][e] * acc[i][j][4 * q + e];
      } else {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[i][j][r] += wj[j] * acc[i][j][r];
#pragma unroll
        for (int j = 0; j < TN; ++j) cst[j] += wj[j] * vb[j];
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        vb[j] = vbn[j];
        wj[j] = wjn[j];
      }
    }
    wait_vmcnt<0>();
  } else {
#pragma unroll
  for (int s0 = 0; s0 < NS - 1; ++s0)
    if (gk > s0) issue(s0);
  int sc = 0, si = NS - 1;
  for (int m = 0; m < gk; ++m) {
    // member m has landed (this wavefront's share: with three stages the loads of member m + 1 may stay in flight) ...
    if (NS == 3 && m + 1 < gk) {
      if (extra) wait_vmcnt<AL + BL + 1>();
      else wait_vmcnt<AL + BL>();
    } else {
      wait_vmcnt<0>();
    }
    // ... and for everyone; all wavefronts are done with member m - 1, whose stage takes member m + NS - 1
    __builtin_amdgcn_s_barrier();
    if (m + NS - 1 < gk) issue(si);
    si = si == NS - 1 ? 0 : si + 1;
    const unsigned char* st = smem + sc * kRedStageBytes;
    sc = sc == NS - 1 ? 0 : sc + 1;

    // per-column vectors of this member, read without a branch: an absent vector's slot holds arbitrary bytes, which the
    // mask turns into +0 (a branch per vector would put one LDS round trip after the other in front of the products)
    float vb[TN];                                        // per-column constant of this member: v1 + v2
    float wj[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const unsigned char* xs = st + xoff + colj + j * 64;
      auto column_value = [&](int slot, unsigned short mask) {
        const unsigned short raw = *reinterpret_cast<const unsigned short*>(xs + slot * VB) & mask;
        return (float)__builtin_bit_cast(bf16, raw);
      };
      if (ATT) {
        wj[j] = 1.f;
        vb[j] = column_value(0, mask1) + column_value(1, mask2);
      } else {
        wj[j] = column_value(0, 0xFFFF);
        vb[j] = column_value(1, mask1) + column_value(2, mask2);
      }
    }
    // Row block i = 0 first, then i = 1: while the matrix pipe works on the second block the vector ALUs scale the
    // first into the running sum (the two instruction streams are interleaved below, one MFMA per four FMAs).
    f32x16 acc[2][TN];
    bf16x8 bfr[4][TN], af[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      af[kk] = *reinterpret_cast<const bf16x8*>(st + a_base + ck[kk]);
#pragma unroll
      for (int j = 0; j < TN; ++j) bfr[kk][j] = *reinterpret_cast<const bf16x8*>(st + b_base + j * 4096 + ck[kk]);
    }
    const float* al = reinterpret_cast<const float*>(st + xoff + AOFF + hrel * HB) + wm * 64 + 4 * lhi;
    auto product = [&](int i) {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          if (kk == 0) {
            // the accumulation starts from the member's per-column constant (ATT) or from zero
            const float c = ATT ? vb[j] : 0.f;
            const f32x16 init = {c, c, c, c, c, c, c, c, c, c, c, c, c, c, c, c};
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[kk], bfr[kk][j], init, 0, 0, 0);
          } else {
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[kk], bfr[kk][j], acc[i][j], 0, 0, 0);
          }
        }
    };
    auto scale_in = [&](int i) {
      if (ATT) {
        // rows of accumulator register r: 8 (r / 4) + 4 lhi + r % 4 of the block
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 a4 = *reinterpret_cast<const f32x4*>(al + i * 32 + 8 * q);
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[i][j][4 * q + e] += a4[e] * acc[i][j][4 * q + e];
        }
      } else {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[i][j][r] += wj[j] * acc[i][j][r];
      }
    };
    product(0);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) af[kk] = *reinterpret_cast<const bf16x8*>(st + a_base + 4096 + ck[kk]);
    __builtin_amdgcn_sched_barrier(0);
    product(1);
    scale_in(0);
#pragma unroll
    for (int t = 0; t < 4 * TN; ++t) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
      __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);   // four vector-ALU instructions
    }
    __builtin_amdgcn_sched_barrier(0);
    scale_in(1);
    if (!ATT) {
#pragma unroll
      for (int j = 0; j < TN; ++j) cst[j] += wj[j] * vb[j];
    }
  }
  }

  const size_t yoff = (((size_t)b * G + k) * N + n0 + wm * 64) * D + col_base + wcol + l32;
  const int nlim = N - n0 - wm * 64 - 4 * lhi;           // rows of this lane's half that are inside the image
  if (S > 1) {                                           // partial sum over this workgroup's members; k_vagg_merge adds them up
    float* pbase = ypart + (size_t)split * tw.nb * G * N * D + yoff;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int rr = i * 32 + 8 * (r >> 2) + (r & 3);
          if (rr < nlim) pbase[(size_t)(rr + 4 * lhi) * D + j * 32] = o[i][j][r] + cst[j];
        }
    return;
  }
  bf16* ybase = y + yoff;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int col = col_base + wcol + j * 32 + l32;
    const float add = cst[j] + (bias ? (float)bias[(size_t)k * D + col] : 0.f);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rr = i * 32 + 8 * (r >> 2) + (r & 3);
        if (rr < nlim) ybase[(size_t)(rr + 4 * lhi) * D + j * 32] = (bf16)(o[i][j][r] + add);
      }
  }
}

}  // namespace dchag
