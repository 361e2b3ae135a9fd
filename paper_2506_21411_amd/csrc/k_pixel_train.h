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
//
// All products run on one loop: tiles of 128 x 128 x 64, four wavefronts (2 x 2) of 64 x 64, two 32-KiB stages filled by
// direct-to-LDS loads one slice ahead, two workgroups per compute unit (the shape whose ring kernel measured within 3 % of
// the larger ones at a third of the code), so one workgroup's load round trip hides under the other's products.
#pragma once
#include "k_fused.h"
#include "k_train.h"

namespace dchag {

constexpr int kPairStageBytes = 256 * 128, kPairLdsBytes = 2 * kPairStageBytes;

// Sizes of a pixel-route first level.  Np: alpha / ds pitch (N to 32); NT: pitch of n-contiguous operands (N to 64);
// gq: members a contraction over (member, pixel) runs over (g, or g to a multiple of 4 for 16 pixels); gp: g to 32;
// RE: rows (member, pixel) then one row per member, gq pp + gp;  KE: gq pp + 2 gp (the member columns twice: be, ce).
struct PixelDims {
  int B, C, N, D, g, G, heads, gpad, Np, NT, gq, gp, RE, KE, H, W;
};

struct PairLane {
  int lane, wave, wm, wn, l32, lhi, a_base, b_base;
  int ck[4];
  __device__ __forceinline__ void init() {
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    wm = wave >> 1;
    wn = wave & 1;
    l32 = lane & 31;
    lhi = lane >> 5;
    a_base = (wm * 64 + l32) * 128;
    b_base = 128 * 128 + (wn * 64 + l32) * 128;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) ck[kk] = ((kk * 2 + lhi) ^ swz_chunk(l32)) * 16;
  }
  // load i of this wavefront fills tile row 32 wave + 8 i + lane / 8 with its chunk chunk(row)
  __device__ __forceinline__ int row(int i) const { return wave * 32 + i * 8 + (lane >> 3); }
  __device__ __forceinline__ int chunk(int row) const { return (lane & 7) ^ swz_chunk(row); }
  __device__ __forceinline__ void read(const unsigned char* st, int kk, bf16x8 (&a)[2], bf16x8 (&b)[2]) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      a[i] = *reinterpret_cast<const bf16x8*>(st + a_base + i * 4096 + ck[kk]);
      b[i] = *reinterpret_cast<const bf16x8*>(st + b_base + i * 4096 + ck[kk]);
    }
  }
  __device__ __forceinline__ void fill(const bf16* const (&a)[4], const bf16* const (&b)[4], unsigned char* st) const {
#pragma unroll
    for (int i = 0; i < 4; ++i) load16_to_lds(a[i], st + wave * 4096 + i * 1024);
#pragma unroll
    for (int i = 0; i < 4; ++i) load16_to_lds(b[i], st + 128 * 128 + wave * 4096 + i * 1024);
  }
};

// issue(s, stage) starts the loads of slice s, compute(s, stage) multiplies it.
template <class Issue, class Compute>
__device__ __forceinline__ void pair_loop(unsigned char* smem, int begin, int end, Issue issue, Compute compute) {
  if (begin >= end) return;
  issue(begin, smem);
  for (int s = begin; s < end; ++s) {
    wait_vmcnt<0>();                                       // slice s has landed (this wavefront's share) ...
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();                          // ... and for everyone; slice s - 1's stage is free
    asm volatile("" ::: "memory");
    if (s + 1 < end) issue(s + 1, smem + ((s + 1 - begin) & 1) * kPairStageBytes);
    compute(s, smem + ((s - begin) & 1) * kPairStageBytes);
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
__device__ __forceinline__ void pair_products(f32x16 (&acc)[2][2], const unsigned char* st, const PairLane& L) {
  bf16x8 a[4][2], b[4][2];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) L.read(st, kk, a[kk], b[kk]);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk][i], b[kk][j], acc[i][j], 0, 0, 0);
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
// Patches with the patch index contiguous, UT[b,c,kk,n] (pitch NT, zeros past N), and for 4 x 4 patches also member-major
// patch rows Ug[b,k,n,(member, pixel)] (pitch gq * 16, zeros for missing members).  A lane takes eight patches x eight
// pixels of one channel.  grid (ceil(NT/64), ceil(G gq pp/8 / 32), B), block 256.
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
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    v[i] = bf16x8{};
    const int n = n0 + i;
    if (live && n < d.N) {
      const int pi = n / pw, pj = n % pw;
      if (P == 8) {
        v[i] = *reinterpret_cast<const bf16x8*>(img + (size_t)(pi * 8 + kc) * d.W + pj * 8);
      } else {
        const bf16x4 lo = *reinterpret_cast<const bf16x4*>(img + (size_t)(pi * 4 + 2 * kc) * d.W + pj * 4);
        const bf16x4 hi = *reinterpret_cast<const bf16x4*>(img + (size_t)(pi * 4 + 2 * kc + 1) * d.W + pj * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[i][e] = lo[e]; v[i][4 + e] = hi[e]; }
      }
    }
    if (P == 4 && n < d.N)
      *reinterpret_cast<bf16x8*>(Ug + (((size_t)b * d.G + k) * d.N + n) * (d.gq * 16) + cl * 16 + kc * 8) = v[i];
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
//   ones[n]:      1 for n < N, 0 up to NT
// grid (ceil(D (64 + XE) / 256), G), block 256.
// ---------------------------------------------------------------------------------------
template <int PP>
__global__ __launch_bounds__(256) void k_pixel_prep(PixelDims d, const float* __restrict__ Mf, const bf16* __restrict__ We,
                                                    const bf16* __restrict__ be, const bf16* __restrict__ ce,
                                                    bf16* __restrict__ M2, bf16* __restrict__ X, bf16* __restrict__ ones) {
  const int XW = PP == 16 ? d.gq * 16 : 0, XE = XW + 2 * d.gp, row = 64 + XE;
  const int k = blockIdx.y, gk = min(d.g, d.C - k * d.g);
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  if (k == 0)
    for (long i = idx; i < d.NT; i += (long)gridDim.x * 256) ones[i] = (bf16)(i < d.N ? 1.f : 0.f);
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
// Value fold in both layouts: Wf[c][o][kk] and WfT[c][kk][o] = sum_j WeT[c][kk][j] Wv[k][o][j] (WeT: the tokenizer weights
// transposed); for 4 x 4 patches also member-major rows Wg[k][o][(member, pixel)] (pitch 16 gq, zeros for missing members).
// Tile rows: (member, pixel), tile columns: o.
// ---------------------------------------------------------------------------------------
template <int PP>
__global__ __launch_bounds__(256, 2) void k_pixel_fold(PixelDims d, TileWork tw, const bf16* __restrict__ WeT,
                                                       const bf16* __restrict__ Wv, bf16* __restrict__ Wf,
                                                       bf16* __restrict__ WfT, bf16* __restrict__ Wg) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int k, b, mt, nt;
  if (!tw.decode(blockIdx.x, k, b, nt, mt)) return;        // row tiles fastest: they share the rows of Wv
  const int c0 = k * d.g, gk = min(d.g, d.C - c0), D = d.D;
  PairLane L;
  L.init();
  const bf16 *pa[4], *pb[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = L.row(i), ch = L.chunk(row) * 8;
    pa[i] = WeT + ((size_t)c0 * PP + min(mt * 128 + row, gk * PP - 1)) * D + ch;
    pb[i] = Wv + ((size_t)k * D + nt * 128 + row) * D + ch;
  }
  f32x16 acc[2][2];
  zero_acc(acc);
  pair_loop(
      smem, 0, D / 64,
      [&](int, unsigned char* st) {
        L.fill(pa, pb, st);
#pragma unroll
        for (int i = 0; i < 4; ++i) { pa[i] += 64; pb[i] += 64; }
      },
      [&](int, const unsigned char* st) { pair_products(acc, st, L); });
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int o = nt * 128 + L.wn * 64 + j * 32 + L.l32;
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
        if (PP == 16 && cl < d.gq)
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
__global__ __launch_bounds__(256, 2) void k_pixel_dalpha(PixelDims d, TileWork tw, const bf16* __restrict__ x,
                                                         const bf16* __restrict__ Wf, const bf16* __restrict__ fb,
                                                         const bf16* __restrict__ d_o, float* __restrict__ dal) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int k, b, mt, nt;
  if (!tw.decode(blockIdx.x, k, b, nt, mt)) return;        // nt: patches, mt: columns (fastest: they share the patches)
  constexpr int MS = PP == 64 ? 1 : 4;                     // members of a slice
  const int c0 = k * d.g, gk = min(d.g, d.C - c0), D = d.D, N = d.N;
  PairLane L;
  L.init();
  const bf16 *pa[4], *pb[4];
  size_t sa, sb;                                           // advance per slice
  if (PP == 64) {
    const int pw = d.W / 8;
    sa = (size_t)D * 64;
    sb = (size_t)d.H * d.W;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = L.row(i), ch = L.chunk(row), n = min(nt * 128 + row, N - 1);
      pa[i] = Wf + ((size_t)c0 * D + mt * 128 + row) * 64 + ch * 8;
      pb[i] = x + ((size_t)b * d.C + c0) * sb + (size_t)((n / pw) * 8 + ch) * d.W + (n % pw) * 8;   // chunk = pixel row
    }
  } else {
    sa = sb = 64;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = L.row(i), ch = L.chunk(row), n = min(nt * 128 + row, N - 1);
      pa[i] = Wf + ((size_t)k * D + mt * 128 + row) * (d.gq * 16) + ch * 8;
      pb[i] = x + (((size_t)b * d.G + k) * N + n) * (d.gq * 16) + ch * 8;
    }
  }
  const int slices = (gk + MS - 1) / MS;
  // 16 pixels: a slice of 64 runs past the row's end when 16 gq is no multiple of 64 -- it is: gq is a multiple of 4
  const int dcol = mt * 128 + L.wm * 64 + 4 * L.lhi;       // first of this lane's columns of d_o
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
  bf16x4 fbn[2][4];                                        // folded token bias of the next member, this lane's rows
  auto fetch_fb = [&](int m) {
    const bf16* p = fb + (size_t)(c0 + min(m, gk - 1)) * D + dcol;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) fbn[i][q] = fb ? *reinterpret_cast<const bf16x4*>(p + i * 32 + 8 * q) : bf16x4{};
  };
  fetch_fb(0);
  const int PC = H32 ? D / 32 : D / 64;                    // pieces of all heads
  const int piece0 = H32 ? (mt * 128 + L.wm * 64) / 32 : (mt * 128 + L.wm * 64) / 64;
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
  pair_loop(
      smem, 0, slices,
      [&](int, unsigned char* st) {
        L.fill(pa, pb, st);
#pragma unroll
        for (int i = 0; i < 4; ++i) { pa[i] += sa; pb[i] += sb; }
      },
      [&](int s, const unsigned char* st) {
        bf16x8 a[4][2], bb[4][2];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) L.read(st, kk, a[kk], bb[kk]);
#pragma unroll
        for (int t = 0; t < MS; ++t) {
          const int m = s * MS + t;
          if (MS > 1 && m >= gk) break;                    // uniform
          f32x16 init[2];
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
              for (int e = 0; e < 4; ++e) init[i][4 * q + e] = (float)fbn[i][q][e];
          fetch_fb(m + 1);
          f32x16 acc[2][2];
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              if (PP == 64) {
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0][i], bb[0][j], init[i], 0, 0, 0);
#pragma unroll
                for (int kk = 1; kk < 4; ++kk)
                  acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk][i], bb[kk][j], acc[i][j], 0, 0, 0);
              } else {
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[t][i], bb[t][j], init[i], 0, 0, 0);
              }
            }
          finish(m, acc);
        }
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
template <int PP, bool H32>
__global__ __launch_bounds__(256, 2) void k_pixel_dx(PixelDims d, TileWork tw, int ppc, const bf16* __restrict__ WfT,
                                                     const bf16* __restrict__ d_o, const float* __restrict__ alpha,
                                                     const float* __restrict__ ds, const bf16* __restrict__ Msb,
                                                     bf16* __restrict__ dx) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int k, b, mt, nt;
  if (!tw.decode(blockIdx.x, k, b, nt, mt)) return;        // nt: patches, mt: rows (fastest: they share the rows of d_o)
  constexpr int P = PP == 64 ? 8 : 4, MB = PP == 64 ? 1 : 4;   // members of a wavefront's 64 rows
  constexpr int HH = H32 ? 2 : 1;
  const int c0 = k * d.g, gk = min(d.g, d.C - c0), D = d.D, N = d.N, dh = D / d.heads;
  if (mt * 128 >= gk * PP) return;                         // uniform: a short last group has fewer rows
  PairLane L;
  L.init();
  const bf16 *pa[4], *pb[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = L.row(i), ch = L.chunk(row) * 8;
    pa[i] = WfT + ((size_t)c0 * PP + min(mt * 128 + row, gk * PP - 1)) * D + ch;
    pb[i] = d_o + (((size_t)b * d.G + k) * N + min(nt * 128 + row, N - 1)) * D + ch;
  }
  const int cl0 = (mt * 128 + L.wm * 64) / PP;             // this wavefront's first member
  int nn[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) nn[j] = min(nt * 128 + L.wn * 64 + j * 32 + L.l32, d.Np - 1);
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
  // softmax weights of the next slice's head(s)
  float aln[HH][MB][2];
  auto fetch_alpha = [&](int s) {
#pragma unroll
    for (int hh = 0; hh < HH; ++hh)
#pragma unroll
      for (int m = 0; m < MB; ++m) {
        const int head = min((s * 64 + hh * 32) / dh, d.heads - 1), cl = min(cl0 + m, d.gpad - 1);
        const float* p = alpha + ((((size_t)b * d.G + k) * d.gpad + cl) * d.heads + head) * d.Np;
#pragma unroll
        for (int j = 0; j < 2; ++j) aln[hh][m][j] = p[nn[j]];
      }
  };
  fetch_alpha(0);
  pair_loop(
      smem, 0, D / 64,
      [&](int, unsigned char* st) {
        L.fill(pa, pb, st);
#pragma unroll
        for (int i = 0; i < 4; ++i) { pa[i] += 64; pb[i] += 64; }
      },
      [&](int s, const unsigned char* st) {
        float al[HH][MB][2];
#pragma unroll
        for (int hh = 0; hh < HH; ++hh)
#pragma unroll
          for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int j = 0; j < 2; ++j) al[hh][m][j] = aln[hh][m][j];
        fetch_alpha(s + 1);
        bf16x8 a[4][2], bb[4][2];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) L.read(st, kk, a[kk], bb[kk]);
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int hh = 0; hh < HH; ++hh) {
          f32x16 acc[2][2];
          constexpr int KS = 4 / HH;
#pragma unroll
          for (int kk = 0; kk < KS; ++kk)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
              for (int j = 0; j < 2; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[hh * KS + kk][i], bb[hh * KS + kk][j],
                                                                   kk == 0 ? zero : acc[i][j], 0, 0, 0);
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
              for (int r = 0; r < 16; ++r) o[i][j][r] += al[hh][PP == 64 ? 0 : 2 * i + (r >> 3)][j] * acc[i][j][r];
        }
      });
  const int pw = d.W / P;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int n = nt * 128 + L.wn * 64 + j * 32 + L.l32;
    if (n >= N) continue;
    const int pi = n / pw, pj = n % pw;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r0 = mt * 128 + L.wm * 64 + i * 32 + 8 * q + 4 * L.lhi, cl = r0 / PP, kk = r0 % PP;
        if (cl >= gk) continue;
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (bf16)o[i][j][4 * q + e];
        *reinterpret_cast<bf16x4*>(dx + (((size_t)b * d.C + c0 + cl) * d.H + pi * P + kk / P) * d.W + pj * P + kk % P) = v;
      }
  }
}

// ---------------------------------------------------------------------------------------
// E and e: tile rows (member, pixel) then one row per member (its "pixel" is 1), tile columns the columns d of d_o, the
// contraction runs over all patches (n contiguous: UT, dOT) in slices of 64.  The softmax weight depends on the contraction
// index, so it is multiplied into the pixel fragments (fp32, rounded once to bf16 as the token gradients it replaces were).
// Leaves E with (member, pixel) contiguous, Er[k][d][KE] (the member columns twice), and with d contiguous, ET[k][row][d];
// with splits > 1 (few tiles) fp32 partial sums part[split][k][row][d] for k_pixel_outer_merge.
// ---------------------------------------------------------------------------------------
template <int PP>
__device__ __forceinline__ void store_outer(const PixelDims& d, int k, int r0, int col, const bf16x4& v,
                                            bf16* __restrict__ Er, bf16* __restrict__ ET) {
  const int rows = d.gq * PP;
  if (r0 >= d.RE) return;
  bf16* er = Er + ((size_t)k * d.D + col) * d.KE + r0;
  *reinterpret_cast<bf16x4*>(er) = v;
  if (r0 >= rows) *reinterpret_cast<bf16x4*>(er + d.gp) = v;
#pragma unroll
  for (int e = 0; e < 4; ++e) ET[((size_t)k * d.RE + r0 + e) * d.D + col] = v[e];
}

template <int PP, bool H32>
__global__ __launch_bounds__(256, 2) void k_pixel_outer(PixelDims d, TileWork tw, int splits, const bf16* __restrict__ UT,
                                                        const bf16* __restrict__ ones, const bf16* __restrict__ dOT,
                                                        const float* __restrict__ alpha, bf16* __restrict__ Er,
                                                        bf16* __restrict__ ET, float* __restrict__ part) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int k, sp, mt, nt;
  if (!tw.decode(blockIdx.x, k, sp, nt, mt)) return;       // sp: split; mt: rows (fastest: they share the rows of dOT)
  constexpr int HH = H32 ? 2 : 1;
  const int c0 = k * d.g, gk = min(d.g, d.C - c0), D = d.D, dh = D / d.heads, rows = d.gq * PP;
  PairLane L;
  L.init();
  const bf16 *pa[4], *pb[4];
  bool is_one[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = L.row(i), ch = L.chunk(row) * 8, r = mt * 128 + row;
    is_one[i] = r >= rows;
    pa[i] = is_one[i] ? ones + ch : UT + ((size_t)c0 * PP + min(r, gk * PP - 1)) * d.NT + ch;
    pb[i] = dOT + ((size_t)k * D + nt * 128 + row) * d.NT + ch;
  }
  const int nsl = d.NT / 64, total = d.B * nsl;
  const int s_begin = (int)((long)sp * total / splits), s_end = (int)((long)(sp + 1) * total / splits);
  // softmax weights: this lane's row of block i belongs to member cl[i]
  int acl[2];
  bool alive[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = mt * 128 + L.wm * 64 + i * 32 + L.l32;
    const int cl = r < rows ? r / PP : r - rows;
    alive[i] = cl < gk;
    acl[i] = min(cl, gk - 1);
  }
  const int head0 = (nt * 128 + L.wn * 64) / dh;
  f32x4 av[2][4][2];                                       // block, k-step, half of the 8 patches
  auto fetch_alpha = [&](int s, int hh) {
    const int b = s / nsl, n = (s % nsl) * 64 + 8 * L.lhi;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float* p = alpha + ((((size_t)b * d.G + k) * d.gpad + acl[i]) * d.heads + head0 + hh) * d.Np;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const bool in = alive[i] && n + 16 * kk < d.Np;
        const int nk = in ? n + 16 * kk : 0;
        const f32x4 v0 = *reinterpret_cast<const f32x4*>(p + nk), v1 = *reinterpret_cast<const f32x4*>(p + nk + 4);
        const f32x4 z = {0.f, 0.f, 0.f, 0.f};
        av[i][kk][0] = in ? v0 : z;
        av[i][kk][1] = in ? v1 : z;
      }
    }
  };
  f32x16 acc[2][2];
  zero_acc(acc);
  if (s_begin < s_end && !H32) fetch_alpha(s_begin, 0);
  pair_loop(
      smem, s_begin, s_end,
      [&](int s, unsigned char* st) {
        const int b = s / nsl, n0 = (s % nsl) * 64;
        const size_t oa = (size_t)b * d.C * PP * d.NT + n0, ob = (size_t)b * d.G * D * d.NT + n0;
        const bf16 *qa[4], *qb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          qa[i] = pa[i] + (is_one[i] ? (size_t)n0 : oa);
          qb[i] = pb[i] + ob;
        }
        L.fill(qa, qb, st);
      },
      [&](int s, const unsigned char* st) {
        bf16x8 a[4][2], bb[4][2];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) L.read(st, kk, a[kk], bb[kk]);
#pragma unroll
        for (int hh = 0; hh < HH; ++hh) {
          if (H32) fetch_alpha(s, hh);
          bf16x8 sc[4][2];
#pragma unroll
          for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
              for (int e = 0; e < 8; ++e) sc[kk][i][e] = (bf16)((float)a[kk][i][e] * av[i][kk][e >> 2][e & 3]);
          if (!H32 && s + 1 < s_end) fetch_alpha(s + 1, 0);
#pragma unroll
          for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
              for (int j = 0; j < 2; ++j)
                if (!H32 || j == hh)
                  acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sc[kk][i], bb[kk][j], acc[i][j], 0, 0, 0);
        }
      });
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int col = nt * 128 + L.wn * 64 + j * 32 + L.l32;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r0 = mt * 128 + L.wm * 64 + i * 32 + 8 * q + 4 * L.lhi;
        if (splits > 1) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (r0 + e < d.RE) part[(((size_t)sp * d.G + k) * d.RE + r0 + e) * D + col] = acc[i][j][4 * q + e];
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
// grid (D / 64, ceil(RE / 16), G), block 256.
template <int PP>
__global__ __launch_bounds__(256) void k_pixel_outer_merge(PixelDims d, int splits, const float* __restrict__ part,
                                                           bf16* __restrict__ Er, bf16* __restrict__ ET) {
  const int k = blockIdx.z, col = blockIdx.x * 64 + (threadIdx.x & 63), r0 = blockIdx.y * 16 + (threadIdx.x >> 6) * 4;
  if (r0 >= d.RE) return;
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  for (int sp = 0; sp < splits; ++sp)
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += part[(((size_t)sp * d.G + k) * d.RE + r0 + e) * d.D + col];
  store_outer<PP>(d, k, r0, col, bf16x4{(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]}, Er, ET);
}

// ---------------------------------------------------------------------------------------
// F and f, as hi + lo bf16 parts in the two layouts the products below read: Fr[k][row][KE] with rows 0 .. 31 the heads'
// hi parts and 32 .. 63 their lo parts, FT[k][(member, pixel) / member row][64] with the same 64 as columns.  One block
// per (member, group), four wavefronts over the patches (16 a step), partial blocks merged in LDS in a fixed order.
// grid (gp, G), block 256.
// ---------------------------------------------------------------------------------------
template <int PP>
__global__ __launch_bounds__(256) void k_pixel_key_sums(PixelDims d, int ppc, const float* __restrict__ ds,
                                                        const bf16* __restrict__ UT, bf16* __restrict__ Fr,
                                                        bf16* __restrict__ FT) {
  constexpr int NB = PP == 64 ? 2 : 1;
  __shared__ float part[4][NB][16][64];
  __shared__ float fpart[4][64];
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
    for (int s = wave; s < steps; s += 4) {
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
    for (int idx = threadIdx.x; idx < NB * 16 * 64; idx += 256) {
      const int ln = idx & 63, r = (idx >> 6) & 15, j = idx >> 10;
      const int a = 8 * (r >> 2) + 4 * (ln >> 5) + (r & 3), kk = j * 32 + (ln & 31);
      if (kk >= PP) continue;
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) v += part[w][j][r][ln];
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
    for (int w = 0; w < 4; ++w) v += fpart[w][a] + fpart[w][a + 32];
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
__global__ __launch_bounds__(256, 2) void k_pixel_dwe(PixelDims d, TileWork tw, const bf16* __restrict__ ET,
                                                      const bf16* __restrict__ FT, const bf16* __restrict__ WvT,
                                                      const bf16* __restrict__ M2, bf16* __restrict__ dWe,
                                                      bf16* __restrict__ dtb) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int k, b, mt, nt;
  if (!tw.decode(blockIdx.x, k, b, nt, mt)) return;
  const int c0 = k * d.g, gk = min(d.g, d.C - c0), D = d.D, rows = d.gq * PP;
  PairLane L;
  L.init();
  const bf16 *pa[4], *pb[4], *xa[4], *xb[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = L.row(i), ch = L.chunk(row) * 8;
    const size_t ra = (size_t)k * d.RE + min(mt * 128 + row, d.RE - 1), rb = (size_t)k * D + nt * 128 + row;
    pa[i] = ET + ra * D + ch;
    pb[i] = WvT + rb * D + ch;
    xa[i] = FT + ra * 64 + ch;
    xb[i] = M2 + rb * 64 + ch;
  }
  const int KT = D / 64;
  f32x16 acc[2][2];
  zero_acc(acc);
  pair_loop(
      smem, 0, KT + 1,
      [&](int s, unsigned char* st) {
        if (s == KT) {
          L.fill(xa, xb, st);
          return;
        }
        L.fill(pa, pb, st);
#pragma unroll
        for (int i = 0; i < 4; ++i) { pa[i] += 64; pb[i] += 64; }
      },
      [&](int, const unsigned char* st) { pair_products(acc, st, L); });
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int col = nt * 128 + L.wn * 64 + j * 32 + L.l32;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r0 = mt * 128 + L.wm * 64 + i * 32 + 8 * q + 4 * L.lhi;
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (bf16)acc[i][j][4 * q + e];
        if (r0 < rows) {
          const int cl = r0 / PP;
          if (dWe && cl < gk) *reinterpret_cast<bf16x4*>(dWe + ((size_t)(c0 + cl) * D + col) * PP + r0 % PP) = v;
        } else if (dtb) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (r0 - rows + e < gk) dtb[(size_t)(c0 + r0 - rows + e) * D + col] = v[e];
        }
      }
  }
}

// ---------------------------------------------------------------------------------------
// Value-weight gradient and key-path sums: tile rows the D rows of Er then the 64 rows of Fr, tile columns j, the
// contraction runs over (member, pixel) (slices of We, or of X's rows for 16 pixels) and then over the members (be, ce).
// dWv[k][d][j] (or NULL) and r[k][head][j] = its hi + lo rows, fp32.
// ---------------------------------------------------------------------------------------
template <int PP>
__global__ __launch_bounds__(256, 2) void k_pixel_dwv(PixelDims d, TileWork tw, const bf16* __restrict__ Er,
                                                      const bf16* __restrict__ Fr, const bf16* __restrict__ We,
                                                      const bf16* __restrict__ X, bf16* __restrict__ dWv,
                                                      float* __restrict__ r) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int k, b, mt, nt;
  if (!tw.decode(blockIdx.x, k, b, mt, nt)) return;
  const int c0 = k * d.g, gk = min(d.g, d.C - c0), D = d.D;
  const bool tail = mt * 128 >= D;                         // the tile of Fr's rows
  if (tail ? !r : !dWv) return;                            // uniform
  PairLane L;
  L.init();
  const int XE = (PP == 16 ? d.gq * 16 : 0) + 2 * d.gp;
  const bf16 *pa[4], *pb[4], *xb[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = L.row(i), ch = L.chunk(row) * 8;
    pa[i] = tail ? Fr + ((size_t)k * 64 + min(row, 63)) * d.KE + ch : Er + ((size_t)k * D + mt * 128 + row) * d.KE + ch;
    pb[i] = We + ((size_t)c0 * D + nt * 128 + row) * 64 + ch;
    xb[i] = X + ((size_t)k * D + nt * 128 + row) * XE + ch;
  }
  const int KM = PP == 64 ? d.g : 0, KT = d.KE / 64;       // slices whose right operand is We itself; all slices
  f32x16 acc[2][2];
  zero_acc(acc);
  pair_loop(
      smem, 0, KT,
      [&](int s, unsigned char* st) {
        if (s < KM) {
          L.fill(pa, pb, st);
          if (s + 1 < gk)                                  // members a short group lacks meet zeros of Er: any row will do
#pragma unroll
            for (int i = 0; i < 4; ++i) pb[i] += (size_t)D * 64;
        } else {
          L.fill(pa, xb, st);
#pragma unroll
          for (int i = 0; i < 4; ++i) xb[i] += 64;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) pa[i] += 64;
      },
      [&](int, const unsigned char* st) { pair_products(acc, st, L); });
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int col = nt * 128 + L.wn * 64 + j * 32 + L.l32;
    if (tail) {
      if (L.wm) continue;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int a = 8 * (q >> 2) + 4 * L.lhi + (q & 3);
        if (a < d.heads) r[((size_t)k * d.heads + a) * D + col] = acc[0][j][q] + acc[1][j][q];
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

}  // namespace dchag
