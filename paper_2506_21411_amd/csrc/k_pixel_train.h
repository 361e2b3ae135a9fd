// Training step of an attention first level from the pixels (bf16, 4 x 4 or 8 x 8 patches): forward with the value
// projection folded into the tokenizer weights, and a reverse step in which neither the channel tokens nor their
// gradients nor the per-head averages exist.  Paper Section 2.1 (tokenizer, cross-attention), Section 3.3 (the module is
// trained through; its backward is local).
//
// A first-level token is linear in the patch, z[c] = We[c] u[c] + tb[c] (tb = be + ce), and its value is
// V[c] = Wf[c] u[c] + fb[c] with Wf[c] = Wv We[c], fb[c] = Wv tb[c].  Given d_o (the gradient at the heads before the output
// projection), with a(d) the head of column d:
//   dalpha[c,a] = sum_{d in a} d_o[d] V[c][d]                    ds = softmax Jacobian of dalpha
//   du[c]       = Wf[c]^T (alpha[c,a(.)] d_o) + sum_a ds[c,a] Ms[c][a]          (Ms[c][a] = We[c]^T M_a, the score weights)
//   E[c]        = sum_n (alpha[c,a(.)] d_o) (x) u[c]  [D, pp]    e[c] = sum_n alpha[c,a(.)] d_o  [D]
//   F[c]        = sum_n ds[c,.] (x) u[c]  [heads, pp]            f[c] = sum_n ds[c,.]
//   dWv         = sum_c E[c] We[c]^T + e[c] (x) tb[c]            r_a  = sum_c We[c] F[c]_a + f[c]_a tb[c]   (key path)
//   dWe[c]      = Wv^T E[c] + sum_a M_a (x) F[c]_a               dtb[c] = Wv^T e[c] + sum_a M_a f[c]_a
// Every sum over patches contracts against 16 or 64 pixels instead of D columns, and the two D x D factors meet weight-sized
// operands: 4 products of the tokenizer's size and 3 of the value fold's, where the route through the tokens streams
// tokens, averages, their gradients and the token gradients (about ten passes over B C N D elements).
// Rounded to bf16 on the way: Wf, fb, alpha u per member and the finished sums E and e (F, f and ds go on as hi + lo parts, sums are
// fp32), where the route through the tokens rounds tokens, per-head averages, their gradients and the token gradients.  Against
// float64 the errors of the first level's gradients are the smaller ones here (64 bands in groups of 16: dWv 4.9e-3 / 5.2e-3, dx 5.0e-3 /
// 5.5e-3).
//
// All products run on one loop (pair_loop): tiles of 128 x 256 or 256 x 128 outputs, eight wavefronts of 64 x 64, contraction in
// slices of 64 through three 48-KiB stages that are filled by direct-to-LDS loads two slices ahead.  The barrier sits behind a
// slice's third k-step, when all its fragments are in registers: it frees the slice's stage and hands the next slice over, whose
// first fragments are read under the last products.  (128 x 128 tiles with two stages and two workgroups per compute unit
// waited for each slice's loads: the value-weight gradient of 512 bands took 262 us, 3.5 us a slice.)
#pragma once
#include "k_fused.h"
#include "k_train.h"

namespace dchag {

constexpr int kPairTileBytes = 384 * 128;                 // rows of both operands, 128 bytes each
constexpr int kPairExtraBytes = 4096;                     // k_pixel_outer: softmax weights of a slice
constexpr int kPairStageBytes = kPairTileBytes + kPairExtraBytes, kPairLdsBytes = 3 * kPairStageBytes;

// Sizes of a pixel-route first level.  Np: alpha / ds pitch (N to 32); NT: pitch of n-contiguous operands (N to 64);
// gq: members a contraction over (member, pixel) runs over (g, or g to a multiple of 4 for 16 pixels); gp: g to 32;
// RE: rows (member, pixel) then one row per member, gq pp + gp;  KE: gq pp + 2 gp (the member columns twice: be, ce).
struct PixelDims {
  int B, C, N, D, g, G, heads, gpad, Np, NT, gq, gp, RE, KE, H, W;
};

template <int WM>   // wavefronts along the tile's rows: 2 (128 x 256) or 4 (256 x 128)
struct PairLane {
  static constexpr int WN = 8 / WM, ROWS = 64 * WM, COLS = 64 * WN;
  static constexpr int AL = ROWS / 64, BL = COLS / 64;      // loads per wavefront and slice
  int lane, wave, wm, wn, l32, lhi, a_base, b_base;
  int ck[4];
  __device__ __forceinline__ void init() {
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    wm = wave / WN;
    wn = wave % WN;
    l32 = lane & 31;
    lhi = lane >> 5;
    a_base = (wm * 64 + l32) * 128;
    b_base = ROWS * 128 + (wn * 64 + l32) * 128;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) ck[kk] = ((kk * 2 + lhi) ^ swz_chunk(l32)) * 16;
  }
  // load i of this wavefront fills row (A: 8 AL wave + 8 i + lane / 8; B likewise) with its chunk chunk(row)
  __device__ __forceinline__ int row_a(int i) const { return wave * (8 * AL) + i * 8 + (lane >> 3); }
  __device__ __forceinline__ int row_b(int i) const { return wave * (8 * BL) + i * 8 + (lane >> 3); }
  __device__ __forceinline__ int chunk(int row) const { return (lane & 7) ^ swz_chunk(row); }
  __device__ __forceinline__ void read(const unsigned char* st, int kk, bf16x8 (&a)[2], bf16x8 (&b)[2]) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      a[i] = *reinterpret_cast<const bf16x8*>(st + a_base + i * 4096 + ck[kk]);
      b[i] = *reinterpret_cast<const bf16x8*>(st + b_base + i * 4096 + ck[kk]);
    }
  }
  __device__ __forceinline__ void fill(const bf16* const (&a)[AL], const bf16* const (&b)[BL], unsigned char* st) const {
#pragma unroll
    for (int i = 0; i < AL; ++i) load16_to_lds(a[i], st + (wave * AL + i) * 1024);
#pragma unroll
    for (int i = 0; i < BL; ++i) load16_to_lds(b[i], st + ROWS * 128 + (wave * BL + i) * 1024);
  }
};

// issue(s, stage) starts the loads of slice s, step(s, kk, a, b, stage) takes the fragments of its k-step kk (stage: where the
// slice lies; not to be read by step 3, which runs after the stage has been handed back), post(s) runs behind them.
template <int WM, class Issue, class Step, class Post>
__device__ __forceinline__ void pair_loop(unsigned char* smem, int begin, int end, const PairLane<WM>& L, Issue issue,
                                          Step step, Post post) {
  constexpr int LD = PairLane<WM>::AL + PairLane<WM>::BL;  // a wavefront with further loads waits for a few more
  if (begin >= end) return;
  issue(begin, smem);
  if (begin + 1 < end) {
    issue(begin + 1, smem + kPairStageBytes);
    wait_vmcnt<LD>();
  } else {
    wait_vmcnt<0>();
  }
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  if (begin + 2 < end) issue(begin + 2, smem + 2 * kPairStageBytes);
  bf16x8 a0[2], b0[2], a1[2], b1[2];
  L.read(smem, 0, a0, b0);
  int sc = 0;
  for (int s = begin; s < end; ++s) {
    const unsigned char* st = smem + sc * kPairStageBytes;
    L.read(st, 1, a1, b1);
    __builtin_amdgcn_sched_barrier(0);
    step(s, 0, a0, b0, st);
    __builtin_amdgcn_sched_barrier(0);
    L.read(st, 2, a0, b0);
    __builtin_amdgcn_sched_barrier(0);
    step(s, 1, a1, b1, st);
    __builtin_amdgcn_sched_barrier(0);
    L.read(st, 3, a1, b1);
    __builtin_amdgcn_sched_barrier(0);
    step(s, 2, a0, b0, st);
    __builtin_amdgcn_sched_barrier(0);
    // slice s + 1 has landed (this wavefront's share; the loads of slice s + 2 may stay in flight) and this slice's reads are
    // in registers
    if (s + 2 < end) wait_vmcnt<LD>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_s_waitcnt((7 << 4) | (63 & 15) | ((63 >> 4) << 14));       // lgkmcnt(0), vmcnt untouched
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (s + 3 < end) issue(s + 3, smem + sc * kPairStageBytes);                 // the stage just released
    sc = sc == 2 ? 0 : sc + 1;
    L.read(smem + sc * kPairStageBytes, 0, a0, b0);        // past the last slice: a stale stage, read and not used
    __builtin_amdgcn_sched_barrier(0);
    step(s, 3, a1, b1, st);
    post(s);
    __builtin_amdgcn_sched_barrier(0);
  }
}

__device__ __forceinline__ void zero_acc(f32x16 (&acc)[2][2]) {
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
}
__device__ __forceinline__ void pair_products(f32x16 (&acc)[2][2], const bf16x8 (&a)[2], const bf16x8 (&b)[2]) {
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
}

// Four adjacent rows of a column (a register quad of an accumulator block: lane = column) as two packed words.
struct Quad { unsigned w[2]; };
__device__ __forceinline__ Quad pack_quad(const bf16x4& v) { return __builtin_bit_cast(Quad, v); }

// Rows of two quads q, q + 1 dealt so that a lane holds eight adjacent rows, lanes 0 .. 31 those of quad q (rows 0 .. 7), lanes
// 32 .. 63 those of quad q + 1 (rows 8 .. 15): 16-byte accesses where rows are contiguous, half as many.
__device__ __forceinline__ bf16x8 join_quads(const bf16x4& a, const bf16x4& b) {
  typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
  typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
  const Quad x = pack_quad(a), y = pack_quad(b);
  const u32x2 s0 = __builtin_amdgcn_permlane32_swap(x.w[0], y.w[0], false, false);
  const u32x2 s1 = __builtin_amdgcn_permlane32_swap(x.w[1], y.w[1], false, false);
  return __builtin_bit_cast(bf16x8, u32x4{s0[0], s1[0], s0[1], s1[1]});
}
// The inverse: eight adjacent rows of a column (lanes as above) to the quads of the accumulator layout.
__device__ __forceinline__ void split_quads(const bf16x8& v, bf16x4& a, bf16x4& b) {
  typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
  typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
  const u32x4 w = __builtin_bit_cast(u32x4, v);
  const u32x2 s0 = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
  const u32x2 s1 = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
  a = __builtin_bit_cast(bf16x4, u32x2{s0[0], s1[0]});
  b = __builtin_bit_cast(bf16x4, u32x2{s0[1], s1[1]});
}
// A quad of rows x four adjacent columns (four adjacent lanes) transposed: lane l of the four holds row l, columns 0 .. 3, so that
// a row leaves in 8-byte pieces instead of 2-byte ones.
__device__ __forceinline__ bf16x4 transpose_quad(const bf16x4& v, int lane) {
  const Quad q = pack_quad(v);
  const bool b1 = lane & 2, b0 = lane & 1;
  const unsigned send = b1 ? q.w[0] : q.w[1];
  const unsigned recv = (unsigned)__builtin_amdgcn_update_dpp(0, (int)send, kDppSwapHalves, 0xF, 0xF, true);
  const unsigned x = b1 ? recv : q.w[0], y = b1 ? q.w[1] : recv;      // this lane's two rows of column l & 1, and of that + 2
  const unsigned xp = (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, kDppSwapPairs, 0xF, 0xF, true);
  const unsigned yp = (unsigned)__builtin_amdgcn_update_dpp(0, (int)y, kDppSwapPairs, 0xF, 0xF, true);
  Quad o;
  o.w[0] = b0 ? (xp >> 16) | (x & 0xFFFF0000u) : (x & 0xFFFFu) | (xp << 16);
  o.w[1] = b0 ? (yp >> 16) | (y & 0xFFFF0000u) : (y & 0xFFFFu) | (yp << 16);
  return __builtin_bit_cast(bf16x4, o);
}

// Column block j of a wavefront's 64 rows (member, pixel) from `row` on, lane = patch n, into the image: 16 rows are two 8-pixel rows
// of a patch (8 x 8: a lane each) or a whole 4 x 4 patch.
template <int PP>
__device__ __forceinline__ void store_patch(const PixelDims& d, int b, int c0, int gk, int n, int row, int j,
                                            const f32x16 (&acc)[2][2], int lhi, bf16* __restrict__ dx) {
  constexpr int P = PP == 64 ? 8 : 4;
  const int pw = d.W / P, pi = n / pw, pj = n % pw;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r0 = row + i * 32 + 16 * h, cl = r0 / PP, k0 = r0 % PP;
      if (cl >= gk) continue;                              // uniform over the wavefront
      bf16x4 v[2];
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q >> 2][q & 3] = (bf16)acc[i][j][8 * h + q];
      const bf16x8 v8 = join_quads(v[0], v[1]);
      if (n >= d.N) continue;
      bf16* dst = dx + (((size_t)b * d.C + c0 + cl) * d.H + pi * P) * d.W + pj * P;
      if (PP == 64) {
        *reinterpret_cast<bf16x8*>(dst + (size_t)(k0 / 8 + lhi) * d.W) = v8;
      } else {
#pragma unroll
        for (int q = 0; q < 2; ++q) *reinterpret_cast<bf16x4*>(dst + (size_t)(2 * q + lhi) * d.W) = v[q];
      }
    }
}

// ---------------------------------------------------------------------------------------
// out[batch][c][r] = in[batch][r][c], zeros for R <= r < RT.  A wavefront takes a 64 x 64 tile: a lane reads eight rows of
// one 8-column chunk (128 contiguous bytes per row and eight lanes), transposes the 8 x 8 block in registers and writes
// eight 16-byte pieces (again 128 bytes per eight lanes).  Cc % 8 == 0, RT % 8 == 0.  grid (row tiles, column tiles / 4,
// batch), block 256.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_transpose(int R, int RT, int Cc, const bf16* __restrict__ in,
                                                   bf16* __restrict__ out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r0 = blockIdx.x * 64 + (lane & 7) * 8, c0 = (blockIdx.y * 4 + wave) * 64 + (lane >> 3) * 8;
  if (c0 >= Cc || r0 >= RT) return;
  const bf16* src = in + (size_t)blockIdx.z * R * Cc + c0;
  bf16* dst = out + (size_t)blockIdx.z * Cc * RT + r0;
  bf16x8 v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    v[i] = bf16x8{};
    if (r0 + i < R) v[i] = *reinterpret_cast<const bf16x8*>(src + (size_t)(r0 + i) * Cc);
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    bf16x8 t;
#pragma unroll
    for (int i = 0; i < 8; ++i) t[i] = v[i][e];
    *reinterpret_cast<bf16x8*>(dst + (size_t)(c0 + e) * RT) = t;
  }
}

// ---------------------------------------------------------------------------------------
// Patches with the patch index contiguous, UT[b,c,kk,n] (pitch NT, zeros past N), and for 4 x 4 patches also (where asked for) member-major
// patch rows Ug[b,k,n,(member, pixel)] (pitch gq * 16, zeros for missing members).  A lane takes eight patches x eight
// pixels of one channel.  8 x 8 patches: eight lanes load 128 contiguous bytes of an image row and trade patches through LDS (each
// lane its own eight patches, 128 bytes, overran the L1 by the time the line's last 16 were wanted: 512 bands, 67 MB each way, 38 -> 25 us).  grid (ceil(NT/64), ceil(G gq pp/8 / 32), B), block 256.
// ---------------------------------------------------------------------------------------
template <int P>
__global__ __launch_bounds__(256) void k_pixel_rows(PixelDims d, const bf16* __restrict__ x, bf16* __restrict__ UT,
                                                    bf16* __restrict__ Ug) {
  constexpr int CH = P * P / 8;                            // 8-pixel chunks of a patch
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, b = blockIdx.z;
  const int n0 = blockIdx.x * 64 + (lane & 7) * 8;
  const int q = (blockIdx.y * 4 + wave) * 8 + (lane >> 3);  // (group, member of gq, chunk)
  const int m = q / CH, kc = q % CH, k = m / d.gq, cl = m % d.gq;
  if (k >= d.G) return;
  const int c = k * d.g + cl;
  const bool live = cl < min(d.g, d.C - k * d.g);
  const int pw = d.W / P;
  const bf16* img = x + ((size_t)b * d.C + min(c, d.C - 1)) * d.H * d.W;
  bf16x8 v[8];
  if constexpr (P == 8) {
    __shared__ bf16x8 st[4][512];
    const int o = lane & 7;
    bf16x8* row = st[wave] + (lane >> 3) * 64;              // the 64 patches of this lane's pixel row
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      v[i] = bf16x8{};
      const int n = blockIdx.x * 64 + i * 8 + o;
      if (live && n < d.N) v[i] = *reinterpret_cast<const bf16x8*>(img + (size_t)((n / pw) * 8 + kc) * d.W + (n % pw) * 8);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) row[i * 8 + (o ^ i)] = v[i];
    asm volatile("" ::: "memory");                          // the wavefront's own LDS accesses stay in order
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = row[o * 8 + (i ^ o)];
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      v[i] = bf16x8{};
      const int n = n0 + i;
      if (live && n < d.N) {
        const int pi = n / pw, pj = n % pw;
        const bf16x4 lo = *reinterpret_cast<const bf16x4*>(img + (size_t)(pi * 4 + 2 * kc) * d.W + pj * 4);
        const bf16x4 hi = *reinterpret_cast<const bf16x4*>(img + (size_t)(pi * 4 + 2 * kc + 1) * d.W + pj * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[i][e] = lo[e]; v[i][4 + e] = hi[e]; }
      }
      if (Ug && n < d.N)
        *reinterpret_cast<bf16x8*>(Ug + (((size_t)b * d.G + k) * d.N + n) * (d.gq * 16) + cl * 16 + kc * 8) = v[i];
    }
  }
  if (!live) return;
  bf16* dst = UT + (((size_t)b * d.C + c) * (P * P) + kc * 8) * d.NT + n0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    bf16x8 t;
#pragma unroll
    for (int i = 0; i < 8; ++i) t[i] = v[i][e];
    *reinterpret_cast<bf16x8*>(dst + (size_t)e * d.NT) = t;
  }
}

// ---------------------------------------------------------------------------------------
// Small weight-only operands of the reverse step, one thread per element of a (group, column j) row:
//   M2[k][j][64]: the folded keys of column j, heads 0 .. 31 (zeros past `heads`), twice (they meet F's hi and lo parts)
//   X[k][j][XE]:  for 4 x 4 patches the tokenizer rows We[c][j][:] of the group's members (pitch 16, zeros for missing ones),
//                 then be[c][j] of the members (gp entries, zeros past the group) and ce[c][j] likewise; XE = (16 gq) + 2 gp
// grid (ceil(D (64 + XE) / 256), G), block 256.
// ---------------------------------------------------------------------------------------
template <int PP>
__global__ __launch_bounds__(256) void k_pixel_prep(PixelDims d, const float* __restrict__ Mf, const bf16* __restrict__ We,
                                                    const bf16* __restrict__ be, const bf16* __restrict__ ce,
                                                    bf16* __restrict__ M2, bf16* __restrict__ X) {
  const int XW = PP == 16 ? d.gq * 16 : 0, XE = XW + 2 * d.gp, row = 64 + XE;
  const int k = blockIdx.y, gk = min(d.g, d.C - k * d.g);
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long)d.D * row) return;
  const int j = (int)(idx / row), t = (int)(idx % row);
  if (t < 64) {
    const int a = t & 31;
    M2[((size_t)k * d.D + j) * 64 + t] = (bf16)(a < d.heads ? Mf[((size_t)k * d.heads + a) * d.D + j] : 0.f);
    return;
  }
  const int q = t - 64;
  bf16 v = (bf16)0.f;
  if (q < XW) {
    if (q / 16 < gk) v = We[((size_t)(k * d.g + q / 16) * d.D + j) * 16 + q % 16];
  } else {
    const int cl = (q - XW) % d.gp;
    const bf16* src = q - XW < d.gp ? be : ce;
    if (src && cl < gk) v = src[(size_t)(k * d.g + cl) * d.D + j];
  }
  X[((size_t)k * d.D + j) * XE + q] = v;
}

// ---------------------------------------------------------------------------------------
// Value fold of 4 x 4 patches in three layouts: Wf[c][o][kk], WfT[c][kk][o] = sum_j WeT[c][kk][j] Wv[k][o][j] (WeT: the
// tokenizer weights transposed) and member-major rows Wg[k][o][(member, pixel)] (pitch 16 gq, zeros for missing members).
// Tile rows: (member, pixel), tile columns: o.  (8 x 8 patches: k_product_dl<kProductFold> and a transposing copy,
// 0.09 against 0.134 ms for 512 bands.)
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(512) void k_pixel_fold(PixelDims d, TileWork tw, const bf16* __restrict__ WeT,
                                                       const bf16* __restrict__ Wv, bf16* __restrict__ Wf,
                                                       bf16* __restrict__ WfT, bf16* __restrict__ Wg) {
  constexpr int PP = 16;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int k, b, mt, nt;
  if (!tw.decode(blockIdx.x, k, b, nt, mt)) return;        // row tiles fastest: they share the rows of Wv
  const int c0 = k * d.g, gk = min(d.g, d.C - c0), D = d.D;
  PairLane<2> L;
  L.init();
  const bf16 *pa[2], *pb[4];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = L.row_a(i);
    pa[i] = WeT + ((size_t)c0 * PP + min(mt * 128 + row, gk * PP - 1)) * D + L.chunk(row) * 8;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = L.row_b(i);
    pb[i] = Wv + ((size_t)k * D + nt * 256 + row) * D + L.chunk(row) * 8;
  }
  f32x16 acc[2][2];
  zero_acc(acc);
  pair_loop<2>(
      smem, 0, D / 64, L,
      [&](int, unsigned char* st) {
        L.fill(pa, pb, st);
#pragma unroll
        for (int i = 0; i < 2; ++i) pa[i] += 64;
#pragma unroll
        for (int i = 0; i < 4; ++i) pb[i] += 64;
      },
      [&](int, int, const bf16x8 (&a)[2], const bf16x8 (&bb)[2], const unsigned char*) { pair_products(acc, a, bb); },
      [](int) {});
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int o = nt * 256 + L.wn * 64 + j * 32 + L.l32;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r0 = mt * 128 + L.wm * 64 + i * 32 + 8 * q + 4 * L.lhi, cl = r0 / PP, kk = r0 % PP;
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (bf16)acc[i][j][4 * q + e];
        if (cl < gk) {
          *reinterpret_cast<bf16x4*>(Wf + ((size_t)(c0 + cl) * D + o) * PP + kk) = v;
#pragma unroll
          for (int e = 0; e < 4; ++e) WfT[((size_t)c0 * PP + r0 + e) * D + o] = v[e];
        }
        if (cl < d.gq)
          *reinterpret_cast<bf16x4*>(Wg + ((size_t)k * D + o) * (d.gq * 16) + r0) = cl < gk ? v : bf16x4{};
      }
  }
}

// ---------------------------------------------------------------------------------------
// d alpha: tile rows are value columns, tile columns patches, a slice is one member (64 pixels) or four (16): the member's
// values V = Wf[c] u + fb[c] stay in the accumulators, meet d_o (held in registers: lane = patch) and are summed over the
// columns of the head.  dal[b][k][member][piece][n], pieces of min(dh, 64) columns (k_pixel_jacobian adds a head's pieces).
// ---------------------------------------------------------------------------------------
template <int PP, bool H32>   // H32: heads of 32 columns (two pieces per wavefront)
__global__ __launch_bounds__(512) void k_pixel_dalpha(PixelDims d, TileWork tw, const bf16* __restrict__ x,
                                                         const bf16* __restrict__ Wf, const bf16* __restrict__ fb,
                                                         const bf16* __restrict__ d_o, float* __restrict__ dal) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int k, b, mt, nt;
  if (!tw.decode(blockIdx.x, k, b, nt, mt)) return;        // nt: patches, mt: columns (fastest: they share the patches)
  constexpr int MS = PP == 64 ? 1 : 4;                     // members of a slice
  const int c0 = k * d.g, gk = min(d.g, d.C - c0), D = d.D, N = d.N;
  PairLane<4> L;
  L.init();
  const bf16 *pa[4], *pb[2];
  const size_t sa = PP == 64 ? (size_t)D * 64 : 64, sb = PP == 64 ? (size_t)d.H * d.W : 64;   // advance per slice
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = L.row_a(i), ch = L.chunk(row) * 8;
    pa[i] = PP == 64 ? Wf + ((size_t)c0 * D + mt * 256 + row) * 64 + ch
                     : Wf + ((size_t)k * D + mt * 256 + row) * (d.gq * 16) + ch;
  }
  const int pw = d.W / 8;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = L.row_b(i), ch = L.chunk(row), n = min(nt * 128 + row, N - 1);
    pb[i] = PP == 64 ? x + ((size_t)b * d.C + c0) * sb + (size_t)((n / pw) * 8 + ch) * d.W + (n % pw) * 8   // chunk: pixel row
                     : x + (((size_t)b * d.G + k) * N + n) * (d.gq * 16) + ch * 8;
  }
  const int slices = (gk + MS - 1) / MS;                   // 16 pixels: rows of 16 gq pixels, gq a multiple of 4
  const int dcol = mt * 256 + L.wm * 64 + 4 * L.lhi;       // first of this lane's columns of d_o
  float dv[2][2][16];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int n = min(nt * 128 + L.wn * 64 + j * 32 + L.l32, N - 1);
    const bf16* p = d_o + (((size_t)b * d.G + k) * N + n) * D + dcol;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bf16x4 v = *reinterpret_cast<const bf16x4*>(p + i * 32 + 8 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) dv[i][j][4 * q + e] = (float)v[e];
      }
  }
  const int PC = H32 ? D / 32 : D / 64;                    // pieces of all heads
  const int piece0 = H32 ? (mt * 256 + L.wm * 64) / 32 : (mt * 256 + L.wm * 64) / 64;
  const int n_out = nt * 128 + L.wn * 64 + L.lhi * 32 + L.l32;
  float* out = dal + ((((size_t)b * d.G + k) * d.gpad) * PC + piece0) * d.Np + n_out;
  auto finish = [&](int m, const f32x16 (&acc)[2][2]) {
    float s[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        s[i][j] = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[i][j] += acc[i][j][r] * dv[i][j][r];
      }
    if (!H32) {
#pragma unroll
      for (int j = 0; j < 2; ++j) s[0][j] += s[1][j];
    }
#pragma unroll
    for (int i = 0; i < (H32 ? 2 : 1); ++i) {
      // half 0 keeps block 0's sum and half 1 block 1's: one exchange, 64 adjacent patches stored
      const float give = L.lhi ? s[i][0] : s[i][1], keep = L.lhi ? s[i][1] : s[i][0];
      const float v = keep + __shfl_xor(give, 32, kWave);
      if (n_out < d.Np) out[((size_t)m * PC + i) * d.Np] = v;
    }
  };
  // The folded token bias of a slice's members (256 columns each) travels with the slice: for a vector load of its own the
  // compiler waits until NO load is in flight, the next slices' included (512 bands: 159 us like that, 107 us like this).
  f32x16 init[2], acc[2][2];
  bf16x4 fbl[2][4];                                        // bias of the member about to be multiplied
  const bool bias_wave = fb && L.wave < (MS + 1) / 2;      // two members' columns per load
  const int bm = L.wave * 2 + (L.lane >> 5);
  auto read_fb = [&](const unsigned char* st, int t) {
    const bf16* p = reinterpret_cast<const bf16*>(st + kPairTileBytes + t * 512) + L.wm * 64 + 4 * L.lhi;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) fbl[i][q] = fb ? *reinterpret_cast<const bf16x4*>(p + i * 32 + 8 * q) : bf16x4{};
  };
  pair_loop<4>(
      smem, 0, slices, L,
      [&](int s, unsigned char* st) {
        L.fill(pa, pb, st);
#pragma unroll
        for (int i = 0; i < 4; ++i) pa[i] += sa;
#pragma unroll
        for (int i = 0; i < 2; ++i) pb[i] += sb;
        if (bias_wave)
          load16_to_lds(fb + (size_t)(c0 + min(s * MS + bm, gk - 1)) * D + mt * 256 + (L.lane & 31) * 8,
                        st + kPairTileBytes + L.wave * 1024);
      },
      [&](int s, int kk, const bf16x8 (&a)[2], const bf16x8 (&bb)[2], const unsigned char* st) {
        if (PP == 16 && s * MS + kk >= gk) return;         // uniform
        if (PP == 16 || kk == 0) {
          if (kk == 0) read_fb(st, 0);
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
              for (int e = 0; e < 4; ++e) init[i][4 * q + e] = (float)fbl[i][q][e];
          if (PP == 16 && kk < 3) read_fb(st, kk + 1);     // step 3 must not read the stage
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], bb[j], PP == 16 || kk == 0 ? init[i] : acc[i][j], 0, 0, 0);
        if (PP == 16) finish(s * MS + kk, acc);
      },
      [&](int s) {
        if (PP == 64) finish(s, acc);
      });
}

// ---------------------------------------------------------------------------------------
// ds[c] = alpha[c] (dalpha[c] - sum_c' alpha[c'] dalpha[c']) per (b, k, head, patch), in place on the first of the head's
// `ppc` pieces of dal (layouts of k_pixel_dalpha and alpha_f; zero where alpha is: past N).  grid (ceil(Np/64), heads / 4,
// B G), block 256: a wavefront per head, lanes = patches.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_pixel_jacobian(PixelDims d, int ppc, const float* __restrict__ alpha,
                                                        float* __restrict__ dal) {
  const int n = blockIdx.x * 64 + (threadIdx.x & 63), a = blockIdx.y * 4 + (threadIdx.x >> 6);
  if (n >= d.Np || a >= d.heads) return;
  const int k = blockIdx.z % d.G, gk = min(d.g, d.C - k * d.g);
  const size_t as = (size_t)d.heads * d.Np, ds = (size_t)d.heads * ppc * d.Np;
  const float* al = alpha + ((size_t)blockIdx.z * d.gpad * d.heads + a) * d.Np + n;
  float* da = dal + ((size_t)blockIdx.z * d.gpad * d.heads * ppc + (size_t)a * ppc) * d.Np + n;
  auto total = [&](int cl) {
    float v = da[cl * ds];
    for (int t = 1; t < ppc; ++t) v += da[cl * ds + (size_t)t * d.Np];
    return v;
  };
  float dot = 0.f;
  if (gk <= 32) {                                          // the whole group in registers
    float av[32], dv[32];
#pragma unroll
    for (int cl = 0; cl < 32; ++cl) {
      av[cl] = cl < gk ? al[cl * as] : 0.f;
      dv[cl] = cl < gk ? total(cl) : 0.f;
    }
#pragma unroll
    for (int cl = 0; cl < 32; ++cl) dot += av[cl] * dv[cl];
#pragma unroll
    for (int cl = 0; cl < 32; ++cl)
      if (cl < gk) da[cl * ds] = av[cl] * (dv[cl] - dot);
    return;
  }
  for (int cl = 0; cl < gk; ++cl) dot += al[cl * as] * total(cl);
  for (int cl = 0; cl < gk; ++cl) da[cl * ds] = al[cl * as] * (total(cl) - dot);
}

// ---------------------------------------------------------------------------------------
// Pixel gradients: tile rows (member, pixel), tile columns patches, the contraction runs over the columns of d_o in slices
// of 64; a slice's product is scaled by the softmax weight of (member, head, patch) into the running sum (lane = patch).  The
// key path sum_a ds[c,a] Ms[c][a] starts the sum off (ds as hi + lo bf16 parts).  A lane ends up with four adjacent
// pixels of a patch row and stores them straight into the image.
// ---------------------------------------------------------------------------------------
template <int PP, bool H32, int WM>   // WM = 4: 256 rows x 128 patches; 2: 128 rows (groups of few pixels) x 256 patches
__global__ __launch_bounds__(512) void k_pixel_dx(PixelDims d, TileWork tw, int ppc, const bf16* __restrict__ WfT,
                                                     const bf16* __restrict__ d_o, const float* __restrict__ alpha,
                                                     const float* __restrict__ ds, const bf16* __restrict__ Msb,
                                                     bf16* __restrict__ dx) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int k, b, mt, nt;
  if (!tw.decode(blockIdx.x, k, b, nt, mt)) return;        // nt: patches, mt: rows (fastest: they share the rows of d_o)
  constexpr int MB = PP == 64 ? 1 : 4;                     // members of a wavefront's 64 rows
  constexpr int HH = H32 ? 2 : 1;
  const int c0 = k * d.g, gk = min(d.g, d.C - c0), D = d.D, N = d.N, dh = D / d.heads;
  typedef PairLane<WM> Lane;
  if (mt * Lane::ROWS >= gk * PP) return;                  // uniform: a short last group has fewer rows
  Lane L;
  L.init();
  const bf16 *pa[Lane::AL], *pb[Lane::BL];
#pragma unroll
  for (int i = 0; i < Lane::AL; ++i) {
    const int row = L.row_a(i);
    pa[i] = WfT + ((size_t)c0 * PP + min(mt * Lane::ROWS + row, gk * PP - 1)) * D + L.chunk(row) * 8;
  }
#pragma unroll
  for (int i = 0; i < Lane::BL; ++i) {
    const int row = L.row_b(i);
    pb[i] = d_o + (((size_t)b * d.G + k) * N + min(nt * Lane::COLS + row, N - 1)) * D + L.chunk(row) * 8;
  }
  const int cl0 = (mt * Lane::ROWS + L.wm * 64) / PP;      // this wavefront's first member
  int nn[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) nn[j] = min(nt * Lane::COLS + L.wn * 64 + j * 32 + L.l32, d.Np - 1);
  f32x16 o[2][2];
  zero_acc(o);
  // key path
  const int HP = d.heads * ppc;
#pragma unroll
  for (int m = 0; m < MB; ++m) {
    const int cl = min(cl0 + m, gk - 1);
    const float* dp = ds + (((size_t)b * d.G + k) * d.gpad + cl) * HP * d.Np;
    for (int a0 = 0; a0 < d.heads; a0 += 16) {
      bf16x8 dhi[2], dlo[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        f32x4 v0, v1;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int a = a0 + 8 * L.lhi + i;
          const float v = a < d.heads ? dp[(size_t)a * ppc * d.Np + nn[j]] : 0.f;
          if (i < 4) v0[i] = v; else v1[i - 4] = v;
        }
        split_bf16(v0, v1, dhi[j], dlo[j]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if (PP == 16 && i != m / 2) continue;              // 16 pixels: row block i holds members 2 i and 2 i + 1
        const int kk = PP == 64 ? i * 32 + L.l32 : L.l32 & 15;
        const bool mine = PP == 64 || (L.l32 >> 4) == (m & 1);
        bf16x8 mv;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const int a = a0 + 8 * L.lhi + t;
          mv[t] = (mine && a < d.heads) ? Msb[((size_t)(c0 + cl) * d.heads + a) * PP + kk] : (bf16)0.f;
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          o[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(mv, dhi[j], o[i][j], 0, 0, 0);
          o[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(mv, dlo[j], o[i][j], 0, 0, 0);
        }
      }
    }
  }
  // Softmax weights of a slice's head(s).  64 pixels: segments [head][member of the tile][patch of the tile] in the stage (see
  // k_pixel_dalpha); 16 pixels: a tile holds 8 or 16 members, too many for the stage, and few slices: vector loads.
  float al[HH][MB][2];
  constexpr int TMB = Lane::ROWS / 64, LPS = Lane::COLS / 4;   // 64-pixel members of a tile, lanes of one segment
  constexpr int SEGS = HH * TMB, WSEG = 64 / LPS;              // segments of a slice, per load
  const int sg = L.wave * WSEG + L.lane / LPS;
  const bool alpha_wave = PP == 64 && L.wave < SEGS / WSEG;
  const float* asrc = alpha + (((size_t)b * d.G + k) * d.gpad + min(mt * TMB + sg % TMB, d.gpad - 1)) * d.heads * d.Np +
                      min(nt * Lane::COLS + (L.lane % LPS) * 4, d.Np - 4);
  auto from_memory = [&](int s) {
#pragma unroll
    for (int hh = 0; hh < HH; ++hh)
#pragma unroll
      for (int m = 0; m < MB; ++m) {
        const int head = (s * 64 + hh * 32) / dh, cl = min(cl0 + m, d.gpad - 1);
        const float* p = alpha + ((((size_t)b * d.G + k) * d.gpad + cl) * d.heads + head) * d.Np;
#pragma unroll
        for (int j = 0; j < 2; ++j) al[hh][m][j] = p[nn[j]];
      }
  };
  f32x16 acc[2][2];
  auto scale_in = [&](int hh) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[i][j][r] += al[hh][PP == 64 ? 0 : 2 * i + (r >> 3)][j] * acc[i][j][r];
  };
  pair_loop<WM>(
      smem, 0, D / 64, L,
      [&](int s, unsigned char* st) {
        L.fill(pa, pb, st);
#pragma unroll
        for (int i = 0; i < Lane::AL; ++i) pa[i] += 64;
#pragma unroll
        for (int i = 0; i < Lane::BL; ++i) pb[i] += 64;
        if (alpha_wave)
          load16_to_lds(asrc + (size_t)((s * 64 + sg / TMB * 32) / dh) * d.Np, st + kPairTileBytes + L.wave * 1024);
      },
      [&](int s, int kk, const bf16x8 (&a)[2], const bf16x8 (&bb)[2], const unsigned char* st) {
        if (kk == 0) {
          if (PP == 64) {
            const float* p = reinterpret_cast<const float*>(st + kPairTileBytes) + L.wm * Lane::COLS + L.wn * 64 + L.l32;
#pragma unroll
            for (int hh = 0; hh < HH; ++hh)
#pragma unroll
              for (int j = 0; j < 2; ++j) al[hh][0][j] = p[hh * TMB * Lane::COLS + j * 32];
          } else {
            from_memory(s);
          }
        }
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (H32 && kk == 2) scale_in(0);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], bb[j], kk % (4 / HH) == 0 ? zero : acc[i][j], 0, 0, 0);
      },
      [&](int) { scale_in(HH - 1); });
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int n = nt * Lane::COLS + L.wn * 64 + j * 32 + L.l32;
    store_patch<PP>(d, b, c0, gk, n, mt * Lane::ROWS + L.wm * 64, j, o, L.lhi, dx);
  }
}

// ---------------------------------------------------------------------------------------
// E: tile rows (member, pixel), tile columns the columns d of d_o, the contraction runs over all patches (n contiguous: UT,
// dOT) in slices of 64.  The softmax weight depends on the contraction index, so it is multiplied into the pixel fragments
// (fp32, rounded once to bf16 as the token gradients it replaces were); the weights of a slice -- (member of the tile,
// wavefront column) segments of 64 patches -- travel with the slice through LDS (as vector loads, the same 16 bytes for every
// lane of a half-wavefront, they saturated the L1 return path: 430 us for 512 bands).
// Leaves E with (member, pixel) contiguous, Er[k][d][KE], and with d contiguous, ET[k][row][d]; with splits > 1 (few tiles)
// fp32 partial sums part[split][k][row][d] for k_pixel_outer_merge.
// ---------------------------------------------------------------------------------------
template <int PP>
__device__ __forceinline__ void store_outer(const PixelDims& d, int k, int r0, int col, const bf16x4& v,
                                            bf16* __restrict__ Er, bf16* __restrict__ ET) {
  if (r0 >= d.gq * PP) return;
  *reinterpret_cast<bf16x4*>(Er + ((size_t)k * d.D + col) * d.KE + r0) = v;
#pragma unroll
  for (int e = 0; e < 4; ++e) ET[((size_t)k * d.RE + r0 + e) * d.D + col] = v[e];
}
template <int PP, bool H32>
__global__ __launch_bounds__(512) void k_pixel_outer(PixelDims d, TileWork tw, int splits, const bf16* __restrict__ UT,
                                                        const bf16* __restrict__ dOT, const float* __restrict__ alpha,
                                                        bf16* __restrict__ Er, bf16* __restrict__ ET,
                                                        float* __restrict__ part) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int k, sp, mt, nt;
  if (!tw.decode(blockIdx.x, k, sp, nt, mt)) return;       // sp: split; mt: rows (fastest: they share the rows of dOT)
  constexpr int HH = H32 ? 2 : 1;                          // heads of a wavefront's 64 columns
  // 64 pixels: the weights of a slice in its stage, segments [member (2)][32- or 64-column piece of the tile][64 patches];
  // 16 pixels: a tile holds eight members, too many for the stage and few slices in all, so vector loads one slice ahead
  constexpr int NHT = 4 * HH, NSEG = 2 * NHT;
  static_assert(NSEG * 256 <= kPairExtraBytes, "the softmax weights of a slice do not fit the stage");
  const int c0 = k * d.g, gk = min(d.g, d.C - c0), D = d.D, dh = D / d.heads, rows = d.gq * PP;
  typedef PairLane<2> Lane;
  Lane L;
  L.init();
  const bf16 *pa[2], *pb[4];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = L.row_a(i);
    pa[i] = UT + ((size_t)c0 * PP + min(mt * 128 + row, gk * PP - 1)) * d.NT + L.chunk(row) * 8;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = L.row_b(i);
    pb[i] = dOT + ((size_t)k * D + nt * 256 + row) * d.NT + L.chunk(row) * 8;
  }
  const int nsl = d.NT / 64, total = d.B * nsl;
  const int s_begin = (int)((long)sp * total / splits), s_end = (int)((long)(sp + 1) * total / splits);
  // wavefront w < NSEG / 4 loads segments 4 w .. 4 w + 3
  const int seg = L.wave * 4 + (L.lane >> 4), sm = seg / NHT, sh = seg % NHT;
  const int scl = min(mt * 2 + sm, d.gpad - 1), shead = min((nt * 256 + sh * (256 / NHT)) / dh, d.heads - 1);
  const float* asrc = alpha + (((size_t)k * d.gpad + scl) * d.heads + shead) * d.Np;
  const size_t asb = (size_t)d.G * d.gpad * d.heads * d.Np;
  // 64 pixels: where this lane's weights lie in a stage; 16 pixels: its row of weights (block i, first head)
  const int aoff = kPairTileBytes + (L.wm * NHT + L.wn * HH) * 256 + L.lhi * 32;
  const float* arow[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int cl = min((mt * 128 + L.wm * 64 + i * 32 + L.l32) / PP, d.gpad - 1);
    arow[i] = alpha + (((size_t)k * d.gpad + cl) * d.heads + (nt * 256 + L.wn * 64) / dh) * d.Np + 8 * L.lhi;
  }
  struct W8 { f32x4 lo, hi; };
  W8 nxt[2][4];                                            // 16 pixels: block, k-step of the next slice (one head)
  auto from_memory = [&](int s, int hh, int i, int kk) {
    const int b = s / nsl, n = (s % nsl) * 64 + 16 * kk;
    const float* p = arow[i] + b * asb + (size_t)hh * d.Np + (n + 8 * L.lhi < d.Np ? n : 0);   // past the pitch: zero pixels
    return W8{*reinterpret_cast<const f32x4*>(p), *reinterpret_cast<const f32x4*>(p + 4)};
  };
  auto from_stage = [&](const unsigned char* st, int hh, int kk) {
    const unsigned char* p = st + aoff + hh * 256 + kk * 64;
    return W8{*reinterpret_cast<const f32x4*>(p), *reinterpret_cast<const f32x4*>(p + 16)};
  };
  if (PP == 16 && !H32 && s_begin < s_end) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) nxt[i][kk] = from_memory(s_begin, 0, i, kk);
  }
  W8 last[HH];                                             // 64 pixels: weights of a slice's last k-step
  f32x16 acc[2][2];
  zero_acc(acc);
  pair_loop<2>(
      smem, s_begin, s_end, L,
      [&](int s, unsigned char* st) {
        const int b = s / nsl, n0 = (s % nsl) * 64;
        const size_t oa = (size_t)b * d.C * PP * d.NT + n0, ob = (size_t)b * d.G * D * d.NT + n0;
        const bf16 *qa[2], *qb[4];
#pragma unroll
        for (int i = 0; i < 2; ++i) qa[i] = pa[i] + oa;
#pragma unroll
        for (int i = 0; i < 4; ++i) qb[i] = pb[i] + ob;
        L.fill(qa, qb, st);
        if (PP == 64 && L.wave < NSEG / 4)                 // past the pitch: any finite weight (the pixels are zero there)
          load16_to_lds(asrc + b * asb + min(n0 + (L.lane & 15) * 4, d.Np - 4), st + kPairTileBytes + L.wave * 1024);
      },
      [&](int s, int kk, const bf16x8 (&a)[2], const bf16x8 (&bb)[2], const unsigned char* st) {
#pragma unroll
        for (int hh = 0; hh < HH; ++hh) {
          bf16x8 sc[2];
          W8 w{};
          if (PP == 64) w = kk == 3 ? last[hh] : from_stage(st, hh, kk);
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            if (PP == 16) w = H32 ? from_memory(s, hh, i, kk) : nxt[i][kk];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              sc[i][e] = (bf16)((float)a[i][e] * w.lo[e]);
              sc[i][4 + e] = (bf16)((float)a[i][4 + e] * w.hi[e]);
            }
            if (PP == 16 && !H32 && s + 1 < s_end) nxt[i][kk] = from_memory(s + 1, 0, i, kk);
          }
          if (PP == 64 && kk == 2) last[hh] = from_stage(st, hh, 3);
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
              if (!H32 || j == hh)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sc[i], bb[j], acc[i][j], 0, 0, 0);
        }
      },
      [](int) {});
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int col = nt * 256 + L.wn * 64 + j * 32 + L.l32;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r0 = mt * 128 + L.wm * 64 + i * 32 + 8 * q + 4 * L.lhi;
        if (splits > 1) {
          if (r0 < rows)
#pragma unroll
            for (int e = 0; e < 4; ++e) part[(((size_t)sp * d.G + k) * rows + r0 + e) * D + col] = acc[i][j][4 * q + e];
        } else {
          bf16x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = (bf16)acc[i][j][4 * q + e];
          store_outer<PP>(d, k, r0, col, v, Er, ET);
        }
      }
  }
}

// Adds the partial sums of k_pixel_outer up in a fixed order.  A thread takes four adjacent rows of one column.
// grid (D / 64, ceil(gq pp / 16), G), block 256.
template <int PP>
__global__ __launch_bounds__(256) void k_pixel_outer_merge(PixelDims d, int splits, const float* __restrict__ part,
                                                           bf16* __restrict__ Er, bf16* __restrict__ ET) {
  const int k = blockIdx.z, col = blockIdx.x * 64 + (threadIdx.x & 63), r0 = blockIdx.y * 16 + (threadIdx.x >> 6) * 4;
  if (r0 >= d.gq * PP) return;
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  for (int sp = 0; sp < splits; ++sp)
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += part[(((size_t)sp * d.G + k) * (d.gq * PP) + r0 + e) * d.D + col];
  store_outer<PP>(d, k, r0, col, bf16x4{(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]}, Er, ET);
}

// e[c][d] = sum_n alpha[c,a(d),n] d_o[n,d] (softmax weights as hi + lo bf16 parts), rows behind the pixels' rows of ET and the
// two member columns of Er; zeros for members a group lacks.  A block takes 32 columns d (inside one head) and 32 members,
// its eight wavefronts the patches in steps of 16, merged in LDS in a fixed order.  grid (D / 32, gp / 32, G), block 512.
template <int PP>
__global__ __launch_bounds__(512) void k_pixel_member_sums(PixelDims d, const float* __restrict__ alpha,
                                                           const bf16* __restrict__ dOT, bf16* __restrict__ Er,
                                                           bf16* __restrict__ ET) {
  __shared__ float part[8][16][64];
  const int k = blockIdx.z, d0 = blockIdx.x * 32, m0 = blockIdx.y * 32, gk = min(d.g, d.C - k * d.g);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, lhi = lane >> 5;
  const int head = d0 / (d.D / d.heads), cl = min(m0 + l32, gk - 1);
  const bool live = m0 + l32 < gk;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  const int per = d.Np / 16, steps = d.B * per;
#pragma unroll 4
  for (int s = wave; s < steps; s += 8) {
    const int b = s / per, n = (s % per) * 16 + 8 * lhi;
    const float* p = alpha + ((((size_t)b * d.G + k) * d.gpad + cl) * d.heads + head) * d.Np + n;
    f32x4 v0 = *reinterpret_cast<const f32x4*>(p), v1 = *reinterpret_cast<const f32x4*>(p + 4);
    if (!live) v0 = v1 = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 hi, lo;
    split_bf16(v0, v1, hi, lo);
    const bf16x8 o = *reinterpret_cast<const bf16x8*>(dOT + (((size_t)b * d.G + k) * d.D + d0 + l32) * d.NT + n);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hi, o, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo, o, acc, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) part[wave][r][lane] = acc[r];
  __syncthreads();
  for (int idx = threadIdx.x; idx < 1024; idx += 512) {
    const int r = idx >> 6, ln = idx & 63, m = m0 + 8 * (r >> 2) + 4 * (ln >> 5) + (r & 3), col = d0 + (ln & 31);
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w) v += part[w][r][ln];
    const int row = d.gq * PP + m;
    ET[((size_t)k * d.RE + row) * d.D + col] = (bf16)v;
    bf16* er = Er + ((size_t)k * d.D + col) * d.KE + row;
    er[0] = er[d.gp] = (bf16)v;
  }
}

// ---------------------------------------------------------------------------------------
// F and f, as hi + lo bf16 parts in the two layouts the products below read: Fr[k][row][KE] with rows 0 .. 31 the heads'
// hi parts and 32 .. 63 their lo parts, FT[k][(member, pixel) / member row][64] with the same 64 as columns.  One block
// per (member, group), eight wavefronts over the patches (16 a step), partial blocks merged in LDS in a fixed order.
// grid (gp, G), block 512, dynamic LDS 8 (NB 4096 + 256) bytes.
// ---------------------------------------------------------------------------------------
template <int PP>
__global__ __launch_bounds__(512) void k_pixel_key_sums(PixelDims d, int ppc, const float* __restrict__ ds,
                                                        const bf16* __restrict__ UT, bf16* __restrict__ Fr,
                                                        bf16* __restrict__ FT) {
  constexpr int NB = PP == 64 ? 2 : 1;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  float (*part)[NB][16][64] = reinterpret_cast<float (*)[NB][16][64]>(smem);
  float (*fpart)[64] = reinterpret_cast<float (*)[64]>(smem + 8 * NB * 4096);
  const int cl = blockIdx.x, k = blockIdx.y, c0 = k * d.g, gk = min(d.g, d.C - c0);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, lhi = lane >> 5;
  const bool live = cl < gk;
  f32x16 acc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
  float fs = 0.f;
  if (live) {
    const int per = d.Np / 16, steps = d.B * per;
    const int head = min(l32, d.heads - 1);
    const bool hv = l32 < d.heads;
#pragma unroll 4
    for (int s = wave; s < steps; s += 8) {
      const int b = s / per, n = (s % per) * 16 + 8 * lhi;
      const float* dp = ds + ((((size_t)b * d.G + k) * d.gpad + cl) * d.heads + head) * ppc * d.Np + n;
      f32x4 v0 = *reinterpret_cast<const f32x4*>(dp), v1 = *reinterpret_cast<const f32x4*>(dp + 4);
      if (!hv) v0 = v1 = f32x4{0.f, 0.f, 0.f, 0.f};
      fs += ((v0[0] + v0[1]) + (v0[2] + v0[3])) + ((v1[0] + v1[1]) + (v1[2] + v1[3]));
      bf16x8 hi, lo;
      split_bf16(v0, v1, hi, lo);
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int kk = PP == 64 ? j * 32 + l32 : l32 & 15;
        const bf16x8 u = *reinterpret_cast<const bf16x8*>(UT + (((size_t)b * d.C + c0 + cl) * PP + kk) * d.NT + n);
        acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hi, u, acc[j], 0, 0, 0);
        acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo, u, acc[j], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) part[wave][j][r][lane] = acc[j][r];
  fpart[wave][lane] = fs;
  __syncthreads();
  const int rows = d.gq * PP;
  bf16* fr = Fr + (size_t)k * 64 * d.KE;
  if (cl < d.gq) {
    // thread: (block j, register r, lane) -> head 8 (r / 4) + 4 (lane / 32) + r % 4, pixel 32 j + lane % 32
    for (int idx = threadIdx.x; idx < NB * 16 * 64; idx += 512) {
      const int ln = idx & 63, r = (idx >> 6) & 15, j = idx >> 10;
      const int a = 8 * (r >> 2) + 4 * (ln >> 5) + (r & 3), kk = j * 32 + (ln & 31);
      if (kk >= PP) continue;
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < 8; ++w) v += part[w][j][r][ln];
      const bf16 hi = (bf16)v, lo = (bf16)(v - (float)hi);
      const int row = cl * PP + kk;
      fr[(size_t)a * d.KE + row] = hi;
      fr[(size_t)(32 + a) * d.KE + row] = lo;
      FT[((size_t)k * d.RE + row) * 64 + a] = hi;
      FT[((size_t)k * d.RE + row) * 64 + 32 + a] = lo;
    }
  }
  if (threadIdx.x < 32) {
    const int a = threadIdx.x;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w) v += fpart[w][a] + fpart[w][a + 32];
    const bf16 hi = (bf16)v, lo = (bf16)(v - (float)hi);
    const int row = rows + cl;
    fr[(size_t)a * d.KE + row] = fr[(size_t)a * d.KE + row + d.gp] = hi;
    fr[(size_t)(32 + a) * d.KE + row] = fr[(size_t)(32 + a) * d.KE + row + d.gp] = lo;
    FT[((size_t)k * d.RE + row) * 64 + a] = hi;
    FT[((size_t)k * d.RE + row) * 64 + 32 + a] = lo;
  }
}

// ---------------------------------------------------------------------------------------
// Tokenizer gradients: tile rows (member, pixel) then member rows, tile columns j;  D / 64 slices of ET against the
// transposed value weights, one slice of FT against the folded keys (M2).  dWe[c][j][kk], dtb[c][j]; either may be NULL.
// ---------------------------------------------------------------------------------------
template <int PP>
__global__ __launch_bounds__(512) void k_pixel_dwe(PixelDims d, TileWork tw, const bf16* __restrict__ ET,
                                                      const bf16* __restrict__ FT, const bf16* __restrict__ WvT,
                                                      const bf16* __restrict__ M2, bf16* __restrict__ dWe,
                                                      bf16* __restrict__ dtb) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int k, b, mt, nt;
  if (!tw.decode(blockIdx.x, k, b, nt, mt)) return;
  const int c0 = k * d.g, gk = min(d.g, d.C - c0), D = d.D, rows = d.gq * PP;
  PairLane<2> L;
  L.init();
  const bf16 *pa[2], *pb[4], *xa[2], *xb[4];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = L.row_a(i), ch = L.chunk(row) * 8;
    const size_t ra = (size_t)k * d.RE + min(mt * 128 + row, d.RE - 1);
    pa[i] = ET + ra * D + ch;
    xa[i] = FT + ra * 64 + ch;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = L.row_b(i), ch = L.chunk(row) * 8;
    const size_t rb = (size_t)k * D + nt * 256 + row;
    pb[i] = WvT + rb * D + ch;
    xb[i] = M2 + rb * 64 + ch;
  }
  const int KT = D / 64;
  f32x16 acc[2][2];
  zero_acc(acc);
  pair_loop<2>(
      smem, 0, KT + 1, L,
      [&](int s, unsigned char* st) {
        if (s == KT) {
          L.fill(xa, xb, st);
          return;
        }
        L.fill(pa, pb, st);
#pragma unroll
        for (int i = 0; i < 2; ++i) pa[i] += 64;
#pragma unroll
        for (int i = 0; i < 4; ++i) pb[i] += 64;
      },
      [&](int, int, const bf16x8 (&a)[2], const bf16x8 (&bb)[2], const unsigned char*) { pair_products(acc, a, bb); },
      [](int) {});
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int col = nt * 256 + L.wn * 64 + j * 32 + L.l32;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int r0 = mt * 128 + L.wm * 64 + i * 32 + 16 * h;    // 16 rows: of one member, or all behind the pixels' rows
        bf16x4 v[2];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q >> 2][q & 3] = (bf16)acc[i][j][8 * h + q];
        if (r0 < rows) {
          const int cl = r0 / PP;
          const bf16x8 v8 = join_quads(v[0], v[1]);
          if (dWe && cl < gk)
            *reinterpret_cast<bf16x8*>(dWe + ((size_t)(c0 + cl) * D + col) * PP + r0 % PP + 8 * L.lhi) = v8;
        } else if (dtb) {
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const int m = r0 - rows + 8 * (q >> 2) + 4 * L.lhi + (q & 3);
            if (m < gk) dtb[(size_t)(c0 + m) * D + col] = v[q >> 2][q & 3];
          }
        }
      }
  }
}

// ---------------------------------------------------------------------------------------
// Value-weight gradient (KEYS = false): tile rows the D rows of Er, tile columns j, the contraction runs over (member, pixel)
// (slices of We, or of X's rows for 16 pixels) and then over the members (be, ce).  KEYS = true: the same with the 64 rows of
// Fr, the contraction dealt to `splits` blocks (a row tile of its own would be a third round of tiles at 512 bands): the
// hi and lo rows added, r[k][split][head][j] in fp32.
// ---------------------------------------------------------------------------------------
template <int PP, bool KEYS>
__global__ __launch_bounds__(512) void k_pixel_dwv(PixelDims d, TileWork tw, int splits, const bf16* __restrict__ Er,
                                                      const bf16* __restrict__ Fr, const bf16* __restrict__ We,
                                                      const bf16* __restrict__ X, bf16* __restrict__ dWv,
                                                      float* __restrict__ r) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int k, b, mt, nt;
  if (!tw.decode(blockIdx.x, k, b, mt, nt)) return;
  const int c0 = k * d.g, gk = min(d.g, d.C - c0), D = d.D;
  typedef PairLane<2> Lane;
  Lane L;
  L.init();
  const int XE = (PP == 16 ? d.gq * 16 : 0) + 2 * d.gp;
  const bf16 *pa[2], *pb[4], *xb[4];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = L.row_a(i), ch = L.chunk(row) * 8;
    pa[i] = KEYS ? Fr + ((size_t)k * 64 + min(row, 63)) * d.KE + ch : Er + ((size_t)k * D + mt * 128 + row) * d.KE + ch;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = L.row_b(i), ch = L.chunk(row) * 8;
    pb[i] = We + ((size_t)c0 * D + nt * 256 + row) * 64 + ch;
    xb[i] = X + ((size_t)k * D + nt * 256 + row) * XE + ch;
  }
  const int KM = PP == 64 ? d.g : 0, KT = d.KE / 64;       // slices whose right operand is We itself; all slices
  const int s_begin = KEYS ? (int)((long)b * KT / splits) : 0, s_end = KEYS ? (int)((long)(b + 1) * KT / splits) : KT;
  f32x16 acc[2][2];
  zero_acc(acc);
  pair_loop<2>(
      smem, s_begin, s_end, L,
      [&](int s, unsigned char* st) {
        const bf16 *qa[2], *qb[4];
#pragma unroll
        for (int i = 0; i < 2; ++i) qa[i] = pa[i] + s * 64;
        // members a short group lacks meet zeros of Er / Fr: any row will do
        const size_t ob = s < KM ? (size_t)min(s, gk - 1) * D * 64 : (size_t)(s - KM) * 64;
#pragma unroll
        for (int i = 0; i < 4; ++i) qb[i] = (s < KM ? pb[i] : xb[i]) + ob;
        L.fill(qa, qb, st);
      },
      [&](int, int, const bf16x8 (&a)[2], const bf16x8 (&bb)[2], const unsigned char*) { pair_products(acc, a, bb); },
      [](int) {});
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int col = nt * 256 + L.wn * 64 + j * 32 + L.l32;
    if (KEYS) {
      if (L.wm) continue;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int a = 8 * (q >> 2) + 4 * L.lhi + (q & 3);
        if (a < d.heads) r[(((size_t)k * splits + b) * d.heads + a) * D + col] = acc[0][j][q] + acc[1][j][q];
      }
      continue;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int row = mt * 128 + L.wm * 64 + i * 32 + 8 * (q >> 2) + 4 * L.lhi + (q & 3);
        dWv[((size_t)k * D + row) * D + col] = (bf16)acc[i][j][q];
      }
  }
}

// ---------------------------------------------------------------------------------------
// Reverse step of a LINEAR first level from the pixels (formulas at k_linear_first_grads), both products on pair_loop: 4 x 4 patches, and
// the counts that linear_products_ok refuses (where it accepts, k_product_dl's Outer and Image take 176 us instead of the 252 below).
// k_linear_outer: P[(member, pixel)][d] = sum_n u[n] dy[n][d] over all patches (UT, dyT: patch index contiguous), tile rows
// (member, pixel), columns d; P stays in the accumulators and leaves as dWe = mix P, dmix = sum_pixels We P + (be + ce) S,
// dtok_bias = mix S, dbias = S and the scaled weights WsT[(member, pixel)][d] = mix We that k_linear_dx contracts dy with.
// Any gradient pointer may be NULL.  512 bands, 4 x 256 patches, D 1024: the per-channel products (1024 x 64 outputs each, operands
// transposed in registers on every load), the pass over P and two copies between image and patch rows took 430 us; these kernels and
// the two transposes before them take 252 (k_linear_outer 129, of which about 40 for the weights and gradients its epilogue moves;
// k_linear_dx 88; transposes 11 + 25).
// ---------------------------------------------------------------------------------------
template <int PP>
__global__ __launch_bounds__(512) void k_linear_outer(PixelDims d, TileWork tw, const bf16* __restrict__ UT,
                                                      const bf16* __restrict__ dyT, const float* __restrict__ S,
                                                      const bf16* __restrict__ We, const bf16* __restrict__ be,
                                                      const bf16* __restrict__ ce, const bf16* __restrict__ mix,
                                                      bf16* __restrict__ dWe, bf16* __restrict__ dtok_bias,
                                                      bf16* __restrict__ dmix, bf16* __restrict__ dbias,
                                                      bf16* __restrict__ WsT) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int k, b, mt, nt;
  if (!tw.decode(blockIdx.x, k, b, nt, mt)) return;        // mt: rows (fastest: they share the rows of dyT)
  const int c0 = k * d.g, gk = min(d.g, d.C - c0), D = d.D, rows = gk * PP;
  if (mt * 128 >= rows) return;                            // uniform: a short last group has fewer rows
  PairLane<2> L;
  L.init();
  const bf16 *pa[2], *pb[4];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = L.row_a(i);
    pa[i] = UT + ((size_t)c0 * PP + min(mt * 128 + row, rows - 1)) * d.NT + L.chunk(row) * 8;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = L.row_b(i);
    pb[i] = dyT + ((size_t)k * D + nt * 256 + row) * d.NT + L.chunk(row) * 8;
  }
  const int nsl = d.NT / 64;
  f32x16 acc[2][2];
  zero_acc(acc);
  pair_loop<2>(
      smem, 0, d.B * nsl, L,
      [&](int s, unsigned char* st) {
        const int bb = s / nsl, n0 = (s % nsl) * 64;
        const size_t oa = (size_t)bb * d.C * PP * d.NT + n0, ob = (size_t)bb * d.G * D * d.NT + n0;
        const bf16 *qa[2], *qb[4];
#pragma unroll
        for (int i = 0; i < 2; ++i) qa[i] = pa[i] + oa;
#pragma unroll
        for (int i = 0; i < 4; ++i) qb[i] = pb[i] + ob;
        L.fill(qa, qb, st);
      },
      [&](int, int, const bf16x8 (&a)[2], const bf16x8 (&bb)[2], const unsigned char*) { pair_products(acc, a, bb); },
      [](int) {});
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int col = nt * 256 + L.wn * 64 + j * 32 + L.l32;
    const float sv = S[(size_t)k * D + col];
    if (dbias && mt == 0 && L.wm == 0 && L.lhi == 0) dbias[(size_t)k * D + col] = (bf16)sv;
    float dot = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) {                        // 16 rows: of one member
        const int r0 = mt * 128 + L.wm * 64 + i * 32 + 16 * h, cl = r0 / PP;
        if (cl >= gk) continue;                            // uniform over the wavefront
        const size_t cd = (size_t)(c0 + cl) * D + col;
        const float sm = (float)mix[cd];
        const int k0 = r0 % PP;                            // pixels k0 .. k0 + 15: quads 2 h and 2 h + 1 of the block
        bf16x4 w[2], gw[2];
        split_quads(*reinterpret_cast<const bf16x8*>(We + cd * PP + k0 + 8 * L.lhi), w[0], w[1]);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          bf16x4 t;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float pv = acc[i][j][8 * h + 4 * q + e];
            dot += (float)w[q][e] * pv;
            gw[q][e] = (bf16)(sm * pv);
            t[e] = (bf16)((float)w[q][e] * sm);
          }
          if (WsT) {
            const int kk = k0 + 8 * q + 4 * L.lhi + (L.lane & 3);
            *reinterpret_cast<bf16x4*>(WsT + ((size_t)(c0 + cl) * PP + kk) * D + (col & ~3)) = transpose_quad(t, L.lane);
          }
        }
        const bf16x8 g8 = join_quads(gw[0], gw[1]);
        if (dWe) *reinterpret_cast<bf16x8*>(dWe + cd * PP + k0 + 8 * L.lhi) = g8;
        if (PP == 16 || (i == 1 && h == 1)) {              // the member's last rows
          dot += __shfl_xor(dot, 32, kWave);
          if (L.lhi == 0) {
            float bias = 0.f;
            if (be) bias += (float)be[cd];
            if (ce) bias += (float)ce[cd];
            if (dmix) dmix[cd] = (bf16)(dot + bias * sv);
            if (dtok_bias) dtok_bias[cd] = (bf16)(sm * sv);
          }
          dot = 0.f;
        }
      }
  }
}

// dx[b,c,pixel of patch n] = sum_d WsT[(c, pixel)][d] dy[b,k,n][d], written into the image.  Tile rows (member, pixel), columns
// patches.
template <int PP, int WM>
__global__ __launch_bounds__(512) void k_linear_dx(PixelDims d, TileWork tw, const bf16* __restrict__ WsT,
                                                   const bf16* __restrict__ dy, bf16* __restrict__ dx) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int k, b, mt, nt;
  if (!tw.decode(blockIdx.x, k, b, nt, mt)) return;        // nt: patches, mt: rows (fastest: they share the rows of dy)
  const int c0 = k * d.g, gk = min(d.g, d.C - c0), D = d.D, N = d.N, rows = gk * PP;
  typedef PairLane<WM> Lane;
  if (mt * Lane::ROWS >= rows) return;                     // uniform
  Lane L;
  L.init();
  const bf16 *pa[Lane::AL], *pb[Lane::BL];
#pragma unroll
  for (int i = 0; i < Lane::AL; ++i) {
    const int row = L.row_a(i);
    pa[i] = WsT + ((size_t)c0 * PP + min(mt * Lane::ROWS + row, rows - 1)) * D + L.chunk(row) * 8;
  }
#pragma unroll
  for (int i = 0; i < Lane::BL; ++i) {
    const int row = L.row_b(i);
    pb[i] = dy + (((size_t)b * d.G + k) * N + min(nt * Lane::COLS + row, N - 1)) * D + L.chunk(row) * 8;
  }
  f32x16 acc[2][2];
  zero_acc(acc);
  pair_loop<WM>(
      smem, 0, D / 64, L,
      [&](int, unsigned char* st) {
        L.fill(pa, pb, st);
#pragma unroll
        for (int i = 0; i < Lane::AL; ++i) pa[i] += 64;
#pragma unroll
        for (int i = 0; i < Lane::BL; ++i) pb[i] += 64;
      },
      [&](int, int, const bf16x8 (&a)[2], const bf16x8 (&bb)[2], const unsigned char*) { pair_products(acc, a, bb); },
      [](int) {});
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int n = nt * Lane::COLS + L.wn * 64 + j * 32 + L.l32;
    store_patch<PP>(d, b, c0, gk, n, mt * Lane::ROWS + L.wm * 64, j, acc, L.lhi, dx);
  }
}

}  // namespace dchag
