// Shape-generic kernels of the weight-folded forward and of the backward pass (any D, any group
// size, fp32 or bf16 storage, fp32 arithmetic).  Paper Section 2.1 (cross-attention aggregation),
// Section 3.3 (the module is trained through; its backward is the reverse of its forward).
//
// Notation: z[b,c,n,:] input tokens of a level, alpha[b,c,n,a] softmax weight of member c for head a,
// u[b,k,n,a,:] = sum_c alpha[b,c,n,a] z[b,c,n,:] (the group's tokens averaged per head),
// o = concatenated heads before the output projection, M[k][a][:] the query folded into the key
// weights.  Since the weights of a softmax sum to one,
//   o_a = sum_c alpha[c,a] (Wv z[c] + bv)_a = (Wv_a u_a) + bv_a ,
// so the value projection can run once per (group, patch, head) on u instead of once per member.
#pragma once
#include "dchag_dev.h"
#include "k_mfma.h"

namespace dchag {

// ---------------------------------------------------------------------------------------
// Strided batched matrix product, fp32 FMA, 64x64 tiles:
//   C(m,n) = scale * sum_kk A(m,kk) * B(kk,n) (+ bias[n])
// over a batch (b, k, a) = (batch element, group, head); with reduce_b the sum also runs over b
// (a contraction over token rows that are split in one block per batch element).
// ragged = 1: M of group k is rows_of(k); ragged = 2: K of group k is rows_of(k).
// grid (ceil(N/64), ceil(M/64), batch), block 256.
// ---------------------------------------------------------------------------------------
struct GemmOperand {
  long sb, sk, sa;   // offset per batch element, group, head
  long s0, s1;       // strides of the operand's two indices: A(m,kk), B(kk,n), C(m,n)
};
struct GemmDesc {
  int M, N, K;
  int nb, nk, na;
  int reduce_b;
  int ragged, ragged_total, ragged_nominal;
  GemmOperand A, Bm, C;
  long bias_sk, bias_sa;
  float scale;
  long rs_sk, rs_sa;   // k_gemm_mfma with a transposed A: optional row sums of A over the contraction, per (k, a)
  int c_vec;           // k_gemm_mfma: C rows are contiguous and 16-byte aligned, N % 8 == 0: store whole 16-byte chunks
  const void* rowadd;  // optional [M][N] addend of C's type, the same for every batch item (k_gemm_mfma, k_gemm_f32)
};

template <typename TA, typename TB, typename TC>
__global__ __launch_bounds__(256) void k_gemm_generic(GemmDesc d, const TA* __restrict__ A, const TB* __restrict__ Bm,
                                                      const TB* __restrict__ bias, TC* __restrict__ C) {
  __shared__ float As[16][64 + 1];
  __shared__ float Bs[16][64 + 1];
  int z = blockIdx.z;
  const int a = z % d.na;
  z /= d.na;
  const int k = z % d.nk;
  const int b0 = d.reduce_b ? 0 : z / d.nk;
  const int b1 = d.reduce_b ? d.nb : b0 + 1;
  int M = d.M, K = d.K;
  if (d.ragged) {
    int left = d.ragged_total - k * d.ragged_nominal;
    left = left < d.ragged_nominal ? left : d.ragged_nominal;
    if (d.ragged == 1) M = left; else K = left;
  }
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  if (m0 >= M) return;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;
  const bool a_kfast = d.A.s1 == 1, b_kfast = d.Bm.s0 == 1;
  for (int b = b0; b < b1; ++b) {
    const TA* Ab = A + d.A.sb * b + d.A.sk * k + d.A.sa * a;
    const TB* Bb = Bm + d.Bm.sb * b + d.Bm.sk * k + d.Bm.sa * a;
    for (int k0 = 0; k0 < K; k0 += 16) {
      for (int idx = threadIdx.x; idx < 64 * 16; idx += 256) {
        const int mm = a_kfast ? idx >> 4 : idx & 63, kk = a_kfast ? idx & 15 : idx >> 6;
        As[kk][mm] = (m0 + mm < M && k0 + kk < K) ? to_f32(Ab[d.A.s0 * (m0 + mm) + d.A.s1 * (k0 + kk)]) : 0.f;
        const int nn = b_kfast ? idx >> 4 : idx & 63, kb = b_kfast ? idx & 15 : idx >> 6;
        Bs[kb][nn] = (n0 + nn < d.N && k0 + kb < K) ? to_f32(Bb[d.Bm.s0 * (k0 + kb) + d.Bm.s1 * (n0 + nn)]) : 0.f;
      }
      __syncthreads();
#pragma unroll
      for (int kk = 0; kk < 16; ++kk) {
        float av[4], bv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) av[i] = As[kk][ty * 4 + i];
#pragma unroll
        for (int j = 0; j < 4; ++j) bv[j] = Bs[kk][tx * 4 + j];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] += av[i] * bv[j];
      }
      __syncthreads();
    }
  }
  TC* Cb = C + d.C.sb * b0 + d.C.sk * k + d.C.sa * a;
  const TB* bs = bias ? bias + d.bias_sk * k + d.bias_sa * a : nullptr;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + ty * 4 + i;
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + tx * 4 + j;
      if (n < d.N) Cb[d.C.s0 * m + d.C.s1 * n] = from_f32<TC>(acc[i][j] * d.scale + (bs ? to_f32(bs[n]) : 0.f));
    }
  }
}

// ---------------------------------------------------------------------------------------
// Softmax over the members of a group, in place on the scores S[B,Cin,N,heads] (fp32).
// One thread per (b, k, n, head).
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_softmax_group(int Cin, int N, int heads, int g, int G, long total,
                                                       float* __restrict__ S) {
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;     // ((b * G + k) * N + n) * heads + a
  if (idx >= total) return;
  const int a = (int)(idx % heads);
  long t = idx / heads;
  const int n = (int)(t % N);
  t /= N;
  const int k = (int)(t % G), b = (int)(t / G);
  const int c0 = k * g, c1 = min(c0 + g, Cin);
  float* s = S + (((size_t)b * Cin) * N + n) * heads + a;
  const size_t cs = (size_t)N * heads;
  float mx = -INFINITY;
  for (int c = c0; c < c1; ++c) mx = fmaxf(mx, s[c * cs]);
  float den = 0.f;
  for (int c = c0; c < c1; ++c) den += __expf(s[c * cs] - mx);
  const float inv = 1.f / den;
  for (int c = c0; c < c1; ++c) s[c * cs] = __expf(s[c * cs] - mx) * inv;
}

// Reverse of the softmax, in place on dalpha:  ds[c] = alpha[c] * (dalpha[c] - sum_c' alpha[c'] dalpha[c']).
__global__ __launch_bounds__(256) void k_softmax_group_backward(int Cin, int N, int heads, int g, int G, long total,
                                                                const float* __restrict__ alpha,
                                                                float* __restrict__ dalpha) {
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  const int a = (int)(idx % heads);
  long t = idx / heads;
  const int n = (int)(t % N);
  t /= N;
  const int k = (int)(t % G), b = (int)(t / G);
  const int c0 = k * g, c1 = min(c0 + g, Cin);
  const size_t base = (((size_t)b * Cin) * N + n) * heads + a, cs = (size_t)N * heads;
  float dot = 0.f;
  for (int c = c0; c < c1; ++c) dot += alpha[base + c * cs] * dalpha[base + c * cs];
  for (int c = c0; c < c1; ++c) dalpha[base + c * cs] = alpha[base + c * cs] * (dalpha[base + c * cs] - dot);
}

// ---------------------------------------------------------------------------------------
// Scores, softmax over the group and the weighted sums of a level in one launch, for the shapes that the bf16 kernels of
// k_fused.h do not take (fp32; D % 256 != 0):
//   s[c,a] = z[c] . M[k][a],  alpha = softmax over c,  and with VALUES  O[d] = sum_c alpha[c,a(d)] V[c][d],
//   otherwise  u[a][:] = sum_c alpha[c,a] z[c][:]  (alpha is also written, token-major [b,c,n,a], where asked).
// A block takes PN patches of a group.  Scores on v_mfma_f32_16x16x4_f32: 16 members x 16 heads; a lane loads four adjacent
// columns of its row, each the k-step of a product of its own (both operands in the same order, so the contraction is complete),
// in four sums; the wavefronts deal the columns among them by sixteens and the patches share the keys.  The partial scores meet in
// LDS in a fixed order, where the weights stay; eight lanes share a softmax.
// The separate kernels (scores, of which a product uses 8 of its 64 columns, a softmax, sums) took, us: fp32, D 512, 8 heads, 512
// patches, 10 groups of 8: 75, here 46 (168 MB: 3.7 TB/s); its upper level, 10 members: 34, 11.5; bf16, D 384, 6 heads, 2 x 135
// patches, 8 groups of 10: 54, 18; its upper level: 23, 7.  Eight patches a block left most compute units idle there (30 and 23).
// grid (ceil(N/PN), G, B), block 256, dynamic LDS 4 * PN * min(g, Cin) * hp floats, hp = heads to a multiple of 8.
// ---------------------------------------------------------------------------------------
template <typename T, bool VALUES, int PN>
__global__ __launch_bounds__(256) void k_level_generic(int Cin, int N, int D, int heads, int hp, int g, const T* __restrict__ z,
                                                       const float* __restrict__ Mf, const T* __restrict__ V,
                                                       float* __restrict__ alpha, T* __restrict__ out) {
  typedef T vec4 __attribute__((ext_vector_type(4)));
  extern __shared__ __attribute__((aligned(16))) float sc[];   // [wavefront][patch][member][head], then the weights in part 0
  const int n0 = blockIdx.x * PN, k = blockIdx.y, b = blockIdx.z, G = gridDim.y;
  const int c0 = k * g, gk = min(g, Cin - c0), live = min(PN, N - n0);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, lq = lane >> 4;
  const int pitch = gk * hp, total = PN * pitch;
  const size_t cs = (size_t)N * D;
  const T* zb = z + ((size_t)b * Cin + c0) * cs + (size_t)n0 * D;
  for (int m0 = 0; m0 < gk; m0 += 16)
    for (int a0 = 0; a0 < heads; a0 += 16) {
      const T* zp = zb + min(m0 + l16, gk - 1) * cs + lq * 4;
      const float* mp = Mf + ((size_t)k * heads + min(a0 + l16, heads - 1)) * D + lq * 4;
      f32x4 acc[PN][4];
#pragma unroll
      for (int p = 0; p < PN; ++p)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[p][e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
      for (int j = wave * 16; j < D; j += 64) {
        vec4 zv[PN] = {};
        f32x4 mv = {0.f, 0.f, 0.f, 0.f};
        if (j + lq * 4 < D) {                                // D % 8 == 0: the last 16 columns may be 8
#pragma unroll
          for (int p = 0; p < PN; ++p) zv[p] = *reinterpret_cast<const vec4*>(zp + (size_t)min(p, live - 1) * D + j);
          mv = *reinterpret_cast<const f32x4*>(mp + j);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int p = 0; p < PN; ++p)
            acc[p][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(to_f32(zv[p][e]), mv[e], acc[p][e], 0, 0, 0);
      }
      // lane: head l16, register r: member 4 lq + r
#pragma unroll
      for (int p = 0; p < PN; ++p) {
        const f32x4 s = (acc[p][0] + acc[p][1]) + (acc[p][2] + acc[p][3]);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = m0 + lq * 4 + r;
          if (m < gk && a0 + l16 < hp) sc[wave * total + p * pitch + m * hp + a0 + l16] = s[r];
        }
      }
    }
  __syncthreads();
  for (int i = tid; i < total; i += 256) sc[i] = (sc[i] + sc[total + i]) + (sc[2 * total + i] + sc[3 * total + i]);
  __syncthreads();
  for (int i = tid >> 3; i < live * hp; i += 32) {           // eight lanes a (patch, head); past `heads`: finite, not used
    const int p = i / hp, a = i % hp, sub = tid & 7;
    float* w = sc + p * pitch + a;
    float mx = -INFINITY, den = 0.f;
    for (int m = sub; m < gk; m += 8) mx = fmaxf(mx, w[m * hp]);
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o, kWave));
    for (int m = sub; m < gk; m += 8) {
      const float v = __expf(w[m * hp] - mx);
      w[m * hp] = v;
      den += v;
    }
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) den += __shfl_xor(den, o, kWave);
    const float inv = 1.f / den;
    for (int m = sub; m < gk; m += 8) {
      const float v = w[m * hp] * inv;
      w[m * hp] = v;
      if (alpha && a < heads) alpha[(((size_t)b * Cin + c0 + m) * N + n0 + p) * heads + a] = v;
    }
  }
  __syncthreads();
  const int quads = D / 4, dh = D / heads;
  for (int i = tid; i < live * quads; i += 256) {
    const int p = i / quads, d0 = (i % quads) * 4;
    const float* w = sc + p * pitch;
    if (VALUES) {
      const T* vp = V + ((size_t)b * Cin + c0) * cs + (size_t)(n0 + p) * D + d0;
      int a[4];
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = (d0 + e) / dh;
#pragma unroll 4
      for (int m = 0; m < gk; ++m) {
        const vec4 v = *reinterpret_cast<const vec4*>(vp + m * cs);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += w[m * hp + a[e]] * to_f32(v[e]);
      }
      vec4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = from_f32<T>(acc[e]);
      *reinterpret_cast<vec4*>(out + (((size_t)b * G + k) * N + n0 + p) * D + d0) = o;
    } else {
      const T* zp = zb + (size_t)p * D + d0;
      T* up = out + (((size_t)b * G + k) * N + n0 + p) * heads * D + d0;
      for (int a0 = 0; a0 < heads; a0 += 8) {
        f32x4 acc[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int m = 0; m < gk; ++m) {
          const vec4 v = *reinterpret_cast<const vec4*>(zp + m * cs);
          const f32x4 w0 = *reinterpret_cast<const f32x4*>(w + m * hp + a0), w1 = *reinterpret_cast<const f32x4*>(w + m * hp + a0 + 4);
#pragma unroll
          for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              acc[t][e] += w0[t] * to_f32(v[e]);
              acc[4 + t][e] += w1[t] * to_f32(v[e]);
            }
        }
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          if (a0 + t >= heads) break;
          vec4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = from_f32<T>(acc[t][e]);
          *reinterpret_cast<vec4*>(up + (size_t)(a0 + t) * D) = o;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// Per-head weighted token sums:  u[b,k,n,a,:] = sum_{c in group k} alpha[b,c,n,a] * z[b,c,n,:]
// grid (N, G, B), block 256; a thread owns columns d = tid, tid + 256, .. and HMAX heads at a time.
// ---------------------------------------------------------------------------------------
template <typename T, int HMAX>
__global__ __launch_bounds__(256) void k_head_sums(int Cin, int N, int D, int heads, int g,
                                                   const float* __restrict__ alpha, const T* __restrict__ z,
                                                   T* __restrict__ u) {
  __shared__ float al[32][HMAX];
  const int n = blockIdx.x, k = blockIdx.y, b = blockIdx.z, G = gridDim.y;
  const int c0 = k * g, c1 = min(c0 + g, Cin);
  for (int a0 = 0; a0 < heads; a0 += HMAX) {
    for (int d0 = 0; d0 < D; d0 += 256) {
      const int dcol = d0 + threadIdx.x;
      float acc[HMAX];
#pragma unroll
      for (int a = 0; a < HMAX; ++a) acc[a] = 0.f;
      for (int cb = c0; cb < c1; cb += 32) {
        __syncthreads();
        for (int idx = threadIdx.x; idx < 32 * HMAX; idx += 256) {
          const int cc = idx / HMAX, a = idx % HMAX;
          al[cc][a] = (cb + cc < c1 && a0 + a < heads)
                          ? alpha[(((size_t)b * Cin + cb + cc) * N + n) * heads + a0 + a] : 0.f;
        }
        __syncthreads();
        if (dcol < D) {
          const int cn = min(32, c1 - cb);
          for (int cc = 0; cc < cn; ++cc) {
            const float zv = to_f32(z[(((size_t)b * Cin + cb + cc) * N + n) * D + dcol]);
#pragma unroll
            for (int a = 0; a < HMAX; ++a) acc[a] += al[cc][a] * zv;
          }
        }
      }
      if (dcol < D) {
#pragma unroll
        for (int a = 0; a < HMAX; ++a)
          if (a0 + a < heads) u[((((size_t)b * G + k) * N + n) * heads + a0 + a) * D + dcol] = from_f32<T>(acc[a]);
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// dalpha[b,c,n,a] = w[b,k,n,a,:] . z[b,c,n,:]      (w = Wv_a^T do_a, the gradient at u_a)
// The value bias adds the same amount to every member of a group and cancels in the softmax
// Jacobian, so it is left out.  One wave per token; grid ceil(T/4), block 256.
// ---------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void k_dalpha(long T_total, int Cin, int N, int D, int heads, int g, int G,
                                                const T* __restrict__ z, const T* __restrict__ w,
                                                float* __restrict__ dalpha) {
  const long tok = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (tok >= T_total) return;
  const int n = (int)(tok % N);
  const int c = (int)((tok / N) % Cin);
  const int b = (int)(tok / ((long)N * Cin));
  const int k = c / g;
  const T* zr = z + (size_t)tok * D;
  const T* wr = w + (((size_t)b * G + k) * N + n) * heads * D;
  for (int a = 0; a < heads; ++a) {
    float acc = 0.f;
    for (int j = lane; j < D; j += kWave) acc += to_f32(zr[j]) * to_f32(wr[(size_t)a * D + j]);
    acc = wave_sum(acc);
    if (lane == 0) dalpha[(size_t)tok * heads + a] = acc;
  }
}

// ---------------------------------------------------------------------------------------
// Gradient at the input tokens of an attention level:
//   dz[b,c,n,:] = sum_a alpha[b,c,n,a] * w[b,k,n,a,:]  +  ds[b,c,n,a] * M[k][a][:]
// (value path and key path).  grid (Cin, N, B), block 256.
// ---------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void k_dz_attention(int Cin, int N, int D, int heads, int g, int G,
                                                      const float* __restrict__ alpha, const float* __restrict__ ds,
                                                      const T* __restrict__ w, const float* __restrict__ Mf,
                                                      T* __restrict__ dz) {
  const int c = blockIdx.x, n = blockIdx.y, b = blockIdx.z;
  const int k = c / g;
  const size_t tok = ((size_t)b * Cin + c) * N + n;
  const float* al = alpha + tok * heads;
  const float* dsr = ds + tok * heads;
  const T* wr = w + (((size_t)b * G + k) * N + n) * heads * D;
  const float* mr = Mf + (size_t)k * heads * D;
  for (int j = threadIdx.x; j < D; j += 256) {
    float acc = 0.f;
    for (int a = 0; a < heads; ++a) acc += al[a] * to_f32(wr[(size_t)a * D + j]) + dsr[a] * mr[(size_t)a * D + j];
    dz[tok * D + j] = from_f32<T>(acc);
  }
}

// ---------------------------------------------------------------------------------------
// The two kernels above, fp32, by groups: w[b,k,n] is read once for all members of its group instead of once per member.
// k_dalpha_group: one wavefront per (b, k, n), 16 members x 16 heads a tile on v_mfma_f32_16x16x4f32 (a lane's 16-byte load feeds
// four of them: any assignment of features to contraction steps serves as long as both operands share it), the softmax Jacobian
// over the members behind it: ds[c,a] = alpha[c,a] (dalpha[c,a] - sum_c' alpha[c',a] dalpha[c',a]).  Groups of up to 16 MT.
// 64 features are added up in four chains of 16 and then to the sum (one chain over D lost precision against a wavefront-wide sum).
// grid ceil(B G N / 4), block 256.  D % 16 == 0.  Bound by the read of w and z (80 variables, 512 patches, D 512, 8 heads: 168 MB;
// 37 us, one wavefront per token and a softmax pass 137 + 7).
// ---------------------------------------------------------------------------------------
template <int MT>
__global__ __launch_bounds__(256) void k_dalpha_group(long items, int Cin, int N, int D, int heads, int g, int G,
                                                      const float* __restrict__ z, const float* __restrict__ w,
                                                      const float* __restrict__ alpha, float* __restrict__ ds) {
  const long item = (long)blockIdx.x * 4 + (threadIdx.x >> 6);     // (b * G + k) * N + n
  if (item >= items) return;
  const int lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
  const int n = (int)(item % N), k = (int)((item / N) % G), b = (int)(item / ((long)N * G));
  const int c0 = k * g, gk = min(g, Cin - c0);
  const size_t cstride = (size_t)N * D;
  const float* zb = z + (((size_t)b * Cin + c0) * N + n) * D + lq * 4;
  for (int a0 = 0; a0 < heads; a0 += 16) {
    const float* wr = w + ((size_t)item * heads + min(a0 + l16, heads - 1)) * D + lq * 4;
    const float* zr[MT];
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      zr[mt] = zb + (size_t)min(mt * 16 + l16, gk - 1) * cstride;
      acc[mt] = zero;
    }
    for (int t = 0; t < D; t += 64) {                              // four steps of 16 per trip, loads first
      f32x4 wf[4], zf[MT][4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int tt = min(t + q * 16, D - 16);
        wf[q] = *reinterpret_cast<const f32x4*>(wr + tt);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) zf[mt][q] = *reinterpret_cast<const f32x4*>(zr[mt] + tt);
      }
      f32x4 trip[MT][4];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (t + q * 16 < D) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
              trip[mt][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(zf[mt][q][e], wf[q][e], q ? trip[mt][e] : zero, 0, 0, 0);
        }
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[mt] += (trip[mt][0] + trip[mt][1]) + (trip[mt][2] + trip[mt][3]);
    }
    // accumulator block: lane holds head lane % 16, members 4 (lane / 16) + 0..3 of the tile
    float al[MT][4];
    float dot = 0.f;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int cl = mt * 16 + lq * 4 + r;
        al[mt][r] = (cl < gk && a0 + l16 < heads)
                        ? alpha[(((size_t)b * Cin + c0 + cl) * N + n) * heads + a0 + l16] : 0.f;
        dot += al[mt][r] * acc[mt][r];
      }
    dot += __shfl_xor(dot, 16, kWave);
    dot += __shfl_xor(dot, 32, kWave);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int cl = mt * 16 + lq * 4 + r;
        if (cl < gk && a0 + l16 < heads)
          ds[(((size_t)b * Cin + c0 + cl) * N + n) * heads + a0 + l16] = al[mt][r] * (acc[mt][r] - dot);
      }
  }
}

// k_dz_group: a block takes PN patches of one (b, k); an item is (patch, 4 columns), its HB head rows of w and of the keys in registers,
// the members' weights and score gradients broadcast from LDS.  heads <= HB, D % 4 == 0.  grid (ceil(N/PN), G, B), block 256,
// dynamic LDS PN g 2 HB floats.  Bound by the read of w and the write of dz (same shape: 168 MB; 28 us, a block per token 137).
template <int HB, int PN>
__global__ __launch_bounds__(256) void k_dz_group(int Cin, int N, int D, int heads, int g, const float* __restrict__ alpha,
                                                  const float* __restrict__ ds, const float* __restrict__ w,
                                                  const float* __restrict__ Mf, float* __restrict__ dz) {
  extern __shared__ __attribute__((aligned(16))) float wt[];       // [patch][member][alpha HB, ds HB]
  const int k = blockIdx.y, b = blockIdx.z, G = gridDim.y, n0 = blockIdx.x * PN;
  const int c0 = k * g, gk = min(g, Cin - c0);
  for (int idx = threadIdx.x; idx < PN * gk * HB; idx += 256) {
    const int a = idx % HB, t = idx / HB, p = t % PN, cl = t / PN;
    const bool live = a < heads && n0 + p < N;
    const size_t o = (((size_t)b * Cin + c0 + cl) * N + min(n0 + p, N - 1)) * heads + min(a, heads - 1);
    float* q = wt + ((size_t)p * gk + cl) * 2 * HB + a;
    q[0] = live ? alpha[o] : 0.f;
    q[HB] = live ? ds[o] : 0.f;
  }
  __syncthreads();
  const int DC = D / 4;
  for (int it = threadIdx.x; it < PN * DC; it += 256) {
    const int d0 = (it % DC) * 4, p = it / DC, n = n0 + p;
    if (n >= N) break;
    const float* wr = w + ((((size_t)b * G + k) * N + n) * heads) * D + d0;
    const float* mr = Mf + (size_t)k * heads * D + d0;
    f32x4 wv[HB], mv[HB];
#pragma unroll
    for (int a = 0; a < HB; ++a) {
      wv[a] = mv[a] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (a < heads) {
        wv[a] = *reinterpret_cast<const f32x4*>(wr + (size_t)a * D);
        mv[a] = *reinterpret_cast<const f32x4*>(mr + (size_t)a * D);
      }
    }
    float* out = dz + (((size_t)b * Cin + c0) * N + n) * D + d0;
    for (int cl = 0; cl < gk; ++cl) {
      const f32x4* q = reinterpret_cast<const f32x4*>(wt + ((size_t)p * gk + cl) * 2 * HB);
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < HB / 4; ++t) {
        const f32x4 al = q[t], dv = q[HB / 4 + t];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[e] += al[a] * wv[t * 4 + a][e] + dv[a] * mv[t * 4 + a][e];
      }
      *reinterpret_cast<f32x4*>(out + (size_t)cl * N * D) = acc;
    }
  }
}

// ---------------------------------------------------------------------------------------
// Column sums over the rows of every group:  out[k][i] = sum_b sum_{r < rows_of(k)} X[first_row(b,k) + r][i]
// grid (ceil(D/64), G), block 1024: a block owns 64 columns; lane l of a wavefront takes the 4 columns 4 (l % 16) .. of
// row 4 wave + l / 16 and every 64th row after it (one 8- or 16-byte load per row); the four row groups of a
// wavefront meet by lane exchange, the 16 wavefronts in LDS, both in a fixed order.  D % 4 == 0.
template <typename T, typename TO>
__global__ __launch_bounds__(1024) void k_colsum(int B, int D, RowBlocks rb, const T* __restrict__ X,
                                                 TO* __restrict__ out) {
  typedef __attribute__((ext_vector_type(4))) T vec4;
  __shared__ float part[16][64];
  const int k = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int cg = lane & 15, rs = lane >> 4;               // 4 columns of the block's 64; row wave * 4 + rs, then every 64th
  const int i = blockIdx.x * 64 + cg * 4;
  const int rows = rb.rows_of(k);
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  if (i < D)
    for (int b = 0; b < B; ++b) {
      const T* xb = X + (size_t)rb.first_row(b, k) * D + i;
      for (int r = wave * 4 + rs; r < rows; r += 64) {
        const vec4 v = *reinterpret_cast<const vec4*>(xb + (size_t)r * D);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += to_f32(v[e]);
      }
    }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    acc[e] += __shfl_xor(acc[e], 16, kWave);
    acc[e] += __shfl_xor(acc[e], 32, kWave);
  }
  if (rs == 0) {
#pragma unroll
    for (int e = 0; e < 4; ++e) part[wave][cg * 4 + e] = acc[e];
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    const int ii = blockIdx.x * 64 + threadIdx.x;
    float sum = 0.f;
#pragma unroll
    for (int w16 = 0; w16 < 16; ++w16) sum += part[w16][threadIdx.x];
    if (ii < D) out[(size_t)k * D + ii] = from_f32<TO>(sum);
  }
}

// ---------------------------------------------------------------------------------------
// Everything of the key and query path that belongs to one row i of a level's weights (a(i): its head, r[k][a][:]: the sum over
// the group's tokens of ds[.,a] * z):
//   dWk[k][i][:] = scale Qp[k][i] r[k][a(i)][:]      dQ[k][i] = scale sum_j Wk[k][i][j] r[k][a(i)][j]
//   dWq[k][i][:] = dQ[k][i] query[k][:]              dbq[k][i] = dQ[k][i]       dbk[k][i] = 0
// A wavefront (a block of its own: a level of one group then reaches every compute unit) takes four rows of a head, V adjacent
// columns a lane: r is read once for the four.  Any output may be NULL; dQ NULL: no query path.  One launch where there were four
// (zeros, dWk, dQ and dbq, dWq), each of them a few us for one group: D 1024, bf16, one group 26 -> 8 us, 16 groups 45 -> 21 (bound
// by the 134 MB it moves: 6.3 TB/s).
// Requires D % V == 0 and 16-byte aligned rows.  grid (heads ceil(dh / 4), G), block 64.
// ---------------------------------------------------------------------------------------
template <typename T, int V>
__global__ __launch_bounds__(64) void k_key_query_grads(int D, int heads, float scale, const T* __restrict__ Wk,
                                                        const T* __restrict__ query, const float* __restrict__ Qp,
                                                        const float* __restrict__ r, float* __restrict__ dQ, T* __restrict__ dWk,
                                                        T* __restrict__ dWq, T* __restrict__ dbk, T* __restrict__ dbq) {
  typedef T vec __attribute__((ext_vector_type(V)));
  typedef float fvec __attribute__((ext_vector_type(V)));
  const int lane = threadIdx.x, dh = D / heads, quads = (dh + 3) / 4;
  const int k = blockIdx.y, a = blockIdx.x / quads, first = (blockIdx.x % quads) * 4;
  const size_t i0 = (size_t)k * D + (size_t)a * dh + first;
  const int rows = min(4, dh - first);
  const float* rv = r + ((size_t)k * heads + a) * D;
  float q[4], acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 4; ++t) q[t] = Qp[i0 + min(t, rows - 1)] * scale;
  for (int j = lane * V; j < D; j += kWave * V) {
    const fvec c = *reinterpret_cast<const fvec*>(rv + j);
    if (dQ) {
      vec w[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) w[t] = *reinterpret_cast<const vec*>(Wk + (i0 + min(t, rows - 1)) * D + j);
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int e = 0; e < V; ++e) acc[t] += to_f32(w[t][e]) * c[e];
    }
    if (dWk) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        vec o;
#pragma unroll
        for (int e = 0; e < V; ++e) o[e] = from_f32<T>(q[t] * c[e]);
        if (t < rows) *reinterpret_cast<vec*>(dWk + (i0 + t) * D + j) = o;
      }
    }
  }
  if (dbk && lane < rows) dbk[i0 + lane] = from_f32<T>(0.f);
  if (!dQ) return;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    acc[t] = wave_sum(acc[t]) * scale;
    if (lane == t && t < rows) {
      dQ[i0 + t] = acc[t];
      if (dbq) dbq[i0 + t] = from_f32<T>(acc[t]);
    }
  }
  if (!dWq) return;
  for (int j = lane * V; j < D; j += kWave * V) {
    const vec c = *reinterpret_cast<const vec*>(query + (size_t)k * D + j);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      vec o;
#pragma unroll
      for (int e = 0; e < V; ++e) o[e] = from_f32<T>(acc[t] * to_f32(c[e]));
      if (t < rows) *reinterpret_cast<vec*>(dWq + (i0 + t) * D + j) = o;
    }
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_fill_zero(long n, T* __restrict__ out) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i < n) out[i] = from_f32<T>(0.f);
}

// dquery[k][j] = sum_i Wq[k][i][j] * dQ[k][i].  grid (ceil(D/64), G), block 1024: a block owns 64 columns; lane l of a
// wavefront takes the 4 columns 4 (l % 16) .. of row 4 wave + l / 16 and every 64th row after it, eight of them in flight (one group of
// D 1024: 10.5 -> 6.3 us); the four row groups of a wavefront meet by lane exchange, the 16 wavefronts in LDS, both in a fixed order.  Requires D % 4 == 0.
template <typename T>
__global__ __launch_bounds__(1024) void k_query_input_grad(int D, const T* __restrict__ Wq,
                                                           const float* __restrict__ dQ, T* __restrict__ dquery) {
  __shared__ float part[16][64];
  const int k = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int cg = lane & 15, rs = lane >> 4;
  const int j = blockIdx.x * 64 + cg * 4;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  if (j < D) {
    const T* w = Wq + (size_t)k * D * D + j;
    const float* dq = dQ + (size_t)k * D;
    typedef T vec __attribute__((ext_vector_type(4)));
    int i = wave * 4 + rs;
    for (; i + 7 * 64 < D; i += 8 * 64) {                          // eight rows in flight
      vec v[8];
      float q[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        v[t] = *reinterpret_cast<const vec*>(w + (size_t)(i + 64 * t) * D);
        q[t] = dq[i + 64 * t];
      }
#pragma unroll
      for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += to_f32(v[t][e]) * q[t];
    }
    for (; i < D; i += 64) {
      const vec v = *reinterpret_cast<const vec*>(w + (size_t)i * D);
      const float q = dq[i];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += to_f32(v[e]) * q;
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    acc[e] += __shfl_xor(acc[e], 16, kWave);
    acc[e] += __shfl_xor(acc[e], 32, kWave);
  }
  if (rs == 0) {
#pragma unroll
    for (int e = 0; e < 4; ++e) part[wave][cg * 4 + e] = acc[e];
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    const int jj = blockIdx.x * 64 + threadIdx.x;
    float sum = 0.f;
#pragma unroll
    for (int w16 = 0; w16 < 16; ++w16) sum += part[w16][threadIdx.x];
    if (jj < D) dquery[(size_t)k * D + jj] = from_f32<T>(sum);
  }
}

// ---------------------------------------------------------------------------------------
// Patches as rows:  patches[b,c,n,kk] = pixel kk (row by row) of patch n of x[b,c]   and the reverse
// scatter of patch rows back into an image.  One thread per run of V adjacent pixels of one patch row
// (V divides p: both sides of the copy are V contiguous elements).  `total` counts runs.
// ---------------------------------------------------------------------------------------
template <typename T, int V, bool TO_IMAGE>
__global__ __launch_bounds__(256) void k_patch_rows(long total, int H, int W, int p, T* __restrict__ img,
                                                    T* __restrict__ patches) {
  typedef __attribute__((ext_vector_type(V))) T vec;
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;      // run index in [B*C, H, W / V]
  if (idx >= total) return;
  const int wv = W / V;
  const int wx = (int)(idx % wv) * V;
  long t = idx / wv;
  const int hy = (int)(t % H);
  const long bc = t / H;
  const int pw = W / p, pp = p * p;
  const int n = (hy / p) * pw + wx / p, kk = (hy % p) * p + wx % p;
  const size_t pi = ((size_t)bc * (H / p) * pw + n) * pp + kk;
  const size_t ii = ((size_t)bc * H + hy) * W + wx;
  if (V == 1) {
    if (TO_IMAGE) img[ii] = patches[pi];
    else patches[pi] = img[ii];
  } else {
    if (TO_IMAGE) *reinterpret_cast<vec*>(img + ii) = *reinterpret_cast<const vec*>(patches + pi);
    else *reinterpret_cast<vec*>(patches + pi) = *reinterpret_cast<const vec*>(img + ii);
  }
}

// ---------------------------------------------------------------------------------------
// Linear (D-CHAG-L) level, backward:   y[b,k,n,d] = sum_cl w[k][cl][d] z[b,k*g+cl,n,d] + bias[k][d]
//   dz[b,c,n,d] = w[k][cl][d] * dy[b,k,n,d]                       grid ceil(total/256), one thread per element
//   dw[k][cl][d] = sum_{b,n} dy[b,k,n,d] * z[b,k*g+cl,n,d]        grid (ceil(D/64), G*g), block 256 (waves split rows)
// Members a short last group does not have get a zero weight gradient.
// ---------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void k_channel_mix_dz(long total, int Cin, int N, int D, int g, int G,
                                                        const T* __restrict__ w, const T* __restrict__ dy,
                                                        T* __restrict__ dz) {
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;      // ((b * Cin + c) * N + n) * D + d
  if (idx >= total) return;
  const int d = (int)(idx % D);
  long t = idx / D;
  const int n = (int)(t % N);
  t /= N;
  const int c = (int)(t % Cin), b = (int)(t / Cin);
  const int k = c / g, cl = c % g;
  dz[idx] = from_f32<T>(to_f32(w[((size_t)k * g + cl) * D + d]) * to_f32(dy[(((size_t)b * G + k) * N + n) * D + d]));
}

template <typename T>
__global__ __launch_bounds__(256) void k_channel_mix_dw(int B, int Cin, int N, int D, int g, int G,
                                                        const T* __restrict__ z, const T* __restrict__ dy,
                                                        T* __restrict__ dw) {
  __shared__ float part[3][64];
  const int kc = blockIdx.y;
  const int k = kc / g, cl = kc % g, c = k * g + cl;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int d = blockIdx.x * 64 + lane;
  float acc = 0.f;
  if (d < D && c < Cin)
    for (int b = 0; b < B; ++b) {
      const T* zb = z + (((size_t)b * Cin + c) * N) * D + d;
      const T* yb = dy + (((size_t)b * G + k) * N) * D + d;
      for (int n = wave; n < N; n += 4) acc += to_f32(zb[(size_t)n * D]) * to_f32(yb[(size_t)n * D]);
    }
  if (wave > 0) part[wave - 1][lane] = acc;
  __syncthreads();
  if (wave == 0 && d < D) dw[(size_t)kc * D + d] = from_f32<T>(acc + part[0][lane] + part[1][lane] + part[2][lane]);
}

// The same two kernels for D % 8 == 0 and 16-byte aligned tensors, 8 adjacent columns per thread.
template <typename T>
__device__ __forceinline__ void load8(const T* p, float (&v)[8]) {
  if constexpr (sizeof(T) == 2) {
    const bf16x8 x = *reinterpret_cast<const bf16x8*>(p);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (float)x[e];
  } else {
    const f32x4 x0 = *reinterpret_cast<const f32x4*>(p), x1 = *reinterpret_cast<const f32x4*>(p + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) { v[e] = x0[e]; v[4 + e] = x1[e]; }
  }
}
template <typename T>
__device__ __forceinline__ void store8(T* p, const float (&v)[8]) {
  if constexpr (sizeof(T) == 2) {
    bf16x8 x;
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = (bf16)v[e];
    *reinterpret_cast<bf16x8*>(p) = x;
  } else {
    *reinterpret_cast<f32x4*>(p) = f32x4{v[0], v[1], v[2], v[3]};
    *reinterpret_cast<f32x4*>(p + 4) = f32x4{v[4], v[5], v[6], v[7]};
  }
}

// dz: grid (ceil(N / 16), Cin, B), block 256: thread t takes the columns 8 (t % (D/8)) .. of every (256 / (D/8))-th
// patch of the block's 16 when D <= 2048, and walks the columns otherwise; the mixing weights stay in registers.
template <typename T>
__global__ __launch_bounds__(256) void k_channel_mix_dz_vec(int Cin, int N, int D, int g, int G,
                                                            const T* __restrict__ w, const T* __restrict__ dy,
                                                            T* __restrict__ dz) {
  const int c = blockIdx.y, b = blockIdx.z, k = c / g, cl = c % g;
  const int n0 = blockIdx.x * 16, n1 = min(n0 + 16, N);
  const int d8 = D / 8;
  const T* wr = w + ((size_t)k * g + cl) * D;
  const T* yb = dy + (((size_t)b * G + k) * N) * D;
  T* zb = dz + (((size_t)b * Cin + c) * N) * D;
  for (int ch = threadIdx.x; ch < 16 * d8; ch += 256) {            // chunk: (patch of the tile, 8 columns)
    const int n = n0 + ch / d8, d = (ch % d8) * 8;
    if (n >= n1) break;
    float wv[8], yv[8];
    load8(wr + d, wv);
    load8(yb + (size_t)n * D + d, yv);
#pragma unroll
    for (int e = 0; e < 8; ++e) yv[e] *= wv[e];
    store8(zb + (size_t)n * D + d, yv);
  }
}

// dw: grid (ceil(D / 1024), G * g), block 256: 128 threads cover 1024 columns, the two halves of the block take the
// even and the odd rows (b, n) and meet in LDS.
template <typename T>
__global__ __launch_bounds__(256) void k_channel_mix_dw_vec(int B, int Cin, int N, int D, int g, int G,
                                                            const T* __restrict__ z, const T* __restrict__ dy,
                                                            T* __restrict__ dw) {
  __shared__ float part[128][9];
  const int kc = blockIdx.y;
  const int k = kc / g, cl = kc % g, c = k * g + cl;
  const int t = threadIdx.x & 127, half = threadIdx.x >> 7;
  const int d = blockIdx.x * 1024 + t * 8;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const bool live = d < D && c < Cin;
  if (live) {
    const long rows = (long)B * N;
#pragma unroll 4
    for (long r = half; r < rows; r += 2) {
      const int b = (int)(r / N), n = (int)(r % N);
      float zv[8], yv[8];
      load8(z + (((size_t)b * Cin + c) * N + n) * D + d, zv);
      load8(dy + (((size_t)b * G + k) * N + n) * D + d, yv);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += zv[e] * yv[e];
    }
  }
  if (half == 1) {
#pragma unroll
    for (int e = 0; e < 8; ++e) part[t][e] = acc[e];
  }
  __syncthreads();
  if (half == 0 && d < D) {                                        // members a short last group lacks: zero
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += part[t][e];
    store8(dw + (size_t)kc * D + d, acc);
  }
}

// ---------------------------------------------------------------------------------------
// Gradients of a linear first level and of the tokenizer below it without the tokens (bf16).  With
//   P[c][d][kk] = sum_{b,n} dy[b,k(c),n,d] * patch[b,c,n,kk]   (one product per channel)   and   S[k][d] = sum_{b,n} dy
// the token t[c] = We[c] patch + be[c] + ce[c] and the mixing weight s[c] give
//   dmix[c][d]      = sum_{b,n} t[c][d] dy[d]  = sum_kk We[c][d][kk] P[c][d][kk] + (be + ce)[c][d] S[k][d]
//   dWe[c][d][kk]   = s[c][d] P[c][d][kk]          dtok_bias[c][d] = s[c][d] S[k][d]
// and the pixel gradient is dy times the scaled weights  Ws[c][d][kk] = We[c][d][kk] s[c][d], which this kernel also
// writes.  One thread per 8 pixels of a (c, d) row, pp / 8 threads per row (a power of two <= 64), rows summed by
// lane exchange.  grid ceil(C D (pp/8) / 256), block 256.  Any output pointer may be NULL.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_linear_first_grads(long chunks, int C, int D, int pp, int g,
                                                            const float* __restrict__ P, const float* __restrict__ S,
                                                            const bf16* __restrict__ We, const bf16* __restrict__ be,
                                                            const bf16* __restrict__ ce, const bf16* __restrict__ mix,
                                                            bf16* __restrict__ dWe, bf16* __restrict__ dtok_bias,
                                                            bf16* __restrict__ dmix, bf16* __restrict__ Ws) {
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;           // ((c * D + d) * (pp / 8) + chunk)
  const int cpr = pp / 8;
  const bool live = idx < chunks;
  const long row = (live ? idx : chunks - 1) / cpr;                // c * D + d
  const int ch = (int)((live ? idx : chunks - 1) % cpr);
  const int c = (int)(row / D), d = (int)(row % D);
  const int k = c / g;
  const float s = (float)mix[(size_t)c * D + d];                   // mixing weights are [G * g][D], member c = k g + cl
  const size_t o = (size_t)row * pp + ch * 8;
  const bf16x8 w8 = *reinterpret_cast<const bf16x8*>(We + o);
  float dot = 0.f;
  if (P) {
    const f32x4 p0 = *reinterpret_cast<const f32x4*>(P + o), p1 = *reinterpret_cast<const f32x4*>(P + o + 4);
    bf16x8 g8;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      dot += (float)w8[e] * p0[e] + (float)w8[4 + e] * p1[e];
      g8[e] = (bf16)(s * p0[e]);
      g8[4 + e] = (bf16)(s * p1[e]);
    }
    if (dWe && live) *reinterpret_cast<bf16x8*>(dWe + o) = g8;
  }
  if (Ws && live) {
    bf16x8 v;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (bf16)((float)w8[e] * s);
    *reinterpret_cast<bf16x8*>(Ws + o) = v;
  }
  for (int off = 1; off < cpr; off <<= 1) dot += __shfl_xor(dot, off, kWave);     // the cpr threads of a row are adjacent lanes
  if (live && ch == 0) {
    const float sv = S[(size_t)k * D + d];
    if (dmix) {
      float bias = 0.f;
      if (be) bias += (float)be[(size_t)c * D + d];
      if (ce) bias += (float)ce[(size_t)c * D + d];
      dmix[(size_t)c * D + d] = (bf16)(dot + bias * sv);
    }
    if (dtok_bias) dtok_bias[(size_t)c * D + d] = (bf16)(s * sv);
  }
}

}  // namespace dchag

// =======================================================================================
// bf16 MFMA kernels of the folded forward and of the backward
// =======================================================================================
namespace dchag {

// ---------------------------------------------------------------------------------------
// Strided batched matrix product on bf16 MFMA (32x32x16, fp32 accumulation), BM x BN x 64 tiles,
// four wavefronts (WM x WN), operands staged through XOR-swizzled LDS rows of 64 contraction elements.
// Same contract as k_gemm_generic (GemmDesc), restricted to:
//   no ragged K, every operand has one unit stride, 16-byte aligned rows (so K % 8 == 0 where an operand's unit stride
//   is the contraction index).  k_gemm_ring takes what has whole 16-byte pieces throughout; here are the fp32 results and, of the bf16
//   ones, heads whose columns are no multiple of 8.
//   A last slice of fewer than 64 steps is filled up with zeros: the contraction over 135
//   patches of a 384-wide model (a weight gradient, 8 groups) takes 8 us here against 75 us on the fp32-FMA kernel that
//   used to take every K that is no multiple of 64.  Only EXTRA instances carry that code and the row addend (with both in
//   every instance a training step of whole slices took 2.93 ms instead of 2.75).
// An operand whose unit stride is the contraction index is copied chunk by chunk (AT / BT = false);
// one whose unit stride is its row index m (or n) is read as 8 x 8 blocks (8 contraction steps x 8
// rows), transposed in registers and written as whole 16-byte LDS chunks (AT / BT = true; threads
// 0 .. BM-1 take A's blocks, the last BN threads B's).
// With a transposed A the kernel can also write the sums of A's rows over the whole contraction (all batch
// elements when reduce_b is set): the bias gradients that go with a weight gradient, at no extra pass over A.
// grid (ceil(N/BN), ceil(M/BM), batch), block 256, dynamic LDS 2 x (BM + BN) x 128 bytes.
// ---------------------------------------------------------------------------------------
template <int BM, int BN, int WM, int WN, bool AT, bool BT, bool EXTRA, typename TC>
__global__ __launch_bounds__(256) void k_gemm_mfma(GemmDesc d, const bf16* __restrict__ A, const bf16* __restrict__ Bm,
                                                   const bf16* __restrict__ bias, TC* __restrict__ C,
                                                   TC* __restrict__ rowsum) {
  static_assert(WM * WN == 4 && BM % (WM * 32) == 0 && BN % (WN * 32) == 0 && BM <= 128 && BN <= 128, "tile");
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  constexpr int A_CH = BM * 8 / 256, B_CH = BN * 8 / 256;          // 16-byte chunks per thread and stage (copied)
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16x8* As = reinterpret_cast<bf16x8*>(smem);           // [2][BM * 8]
  bf16x8* Bs = As + 2 * BM * 8;                           // [2][BN * 8]
  int z = blockIdx.z;
  const int a = z % d.na;
  z /= d.na;
  const int k = z % d.nk;
  const int b0 = d.reduce_b ? 0 : z / d.nk;
  const int b1 = d.reduce_b ? d.nb : b0 + 1;
  int M = d.M;
  if (d.ragged == 1) {
    const int left = d.ragged_total - k * d.ragged_nominal;
    M = left < d.ragged_nominal ? left : d.ragged_nominal;
  }
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  if (m0 >= M) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int l32 = lane & 31, lhi = lane >> 5;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  bf16x8 a_reg[AT ? 8 : A_CH], b_reg[BT ? 8 : B_CH];
  const int KT = (d.K + 63) / 64;
  const int steps = (b1 - b0) * KT;
  const int tb = tid - (256 - BN);                          // B's transposing threads: tb >= 0

  // optional by-product with a transposed A: rsum[r] collects sum over the contraction of A(row 8 mc + r, .)
  // for this thread's share of the contraction steps (only the blocks of the first column tile do it)
  const bool want_rs = AT && rowsum != nullptr && blockIdx.x == 0;
  float rsum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  auto load_tail = [&](const bf16* Ab, const bf16* Bb, int k0) {
    const bf16x8 zero = {};
    if (!AT) {
#pragma unroll
      for (int i = 0; i < A_CH; ++i) {
        const int idx = tid + i * 256, gr = min(m0 + (idx >> 3), M - 1), kk = k0 + (idx & 7) * 8;
        a_reg[i] = kk < d.K ? *reinterpret_cast<const bf16x8*>(Ab + d.A.s0 * gr + kk) : zero;
      }
    } else if (tid < BM) {
      const int gm = min(m0 + (tid % (BM / 8)) * 8, M - 8), kk = k0 + (tid / (BM / 8)) * 8;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        a_reg[i] = kk + i < d.K ? *reinterpret_cast<const bf16x8*>(Ab + d.A.s1 * (kk + i) + gm) : zero;
    }
    if (!BT) {
#pragma unroll
      for (int i = 0; i < B_CH; ++i) {
        const int idx = tid + i * 256, gr = min(n0 + (idx >> 3), d.N - 1), kk = k0 + (idx & 7) * 8;
        b_reg[i] = kk < d.K ? *reinterpret_cast<const bf16x8*>(Bb + d.Bm.s1 * gr + kk) : zero;
      }
    } else if (tb >= 0) {
      const int gn = min(n0 + (tb % (BN / 8)) * 8, d.N - 8), kk = k0 + (tb / (BN / 8)) * 8;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        b_reg[i] = kk + i < d.K ? *reinterpret_cast<const bf16x8*>(Bb + d.Bm.s0 * (kk + i) + gn) : zero;
    }
  };
  auto load = [&](int s) {
    const int b = b0 + s / KT, k0 = (s % KT) * 64;
    const bf16* Ab = A + d.A.sb * b + d.A.sk * k + d.A.sa * a;
    const bf16* Bb = Bm + d.Bm.sb * b + d.Bm.sk * k + d.Bm.sa * a;
    if (EXTRA && k0 + 64 > d.K) {                            // uniform: the ragged last slice, zeros past the end
      load_tail(Ab, Bb, k0);
      return;
    }
    if (!AT) {
#pragma unroll
      for (int i = 0; i < A_CH; ++i) {
        const int idx = tid + i * 256, row = idx >> 3, ch = idx & 7;
        const int gr = min(m0 + row, M - 1);
        a_reg[i] = *reinterpret_cast<const bf16x8*>(Ab + d.A.s0 * gr + k0 + ch * 8);
      }
    } else if (tid < BM) {
      const int mc = tid % (BM / 8), kc = tid / (BM / 8);  // 8 rows m0 + 8 mc .., contraction steps k0 + 8 kc ..
      const int gm = min(m0 + mc * 8, M - 8);
#pragma unroll
      for (int i = 0; i < 8; ++i) a_reg[i] = *reinterpret_cast<const bf16x8*>(Ab + d.A.s1 * (k0 + kc * 8 + i) + gm);
    }
    if (!BT) {
#pragma unroll
      for (int i = 0; i < B_CH; ++i) {
        const int idx = tid + i * 256, row = idx >> 3, ch = idx & 7;
        const int gr = min(n0 + row, d.N - 1);
        b_reg[i] = *reinterpret_cast<const bf16x8*>(Bb + d.Bm.s1 * gr + k0 + ch * 8);
      }
    } else if (tb >= 0) {
      const int nc = tb % (BN / 8), kc = tb / (BN / 8);
      const int gn = min(n0 + nc * 8, d.N - 8);
#pragma unroll
      for (int i = 0; i < 8; ++i) b_reg[i] = *reinterpret_cast<const bf16x8*>(Bb + d.Bm.s0 * (k0 + kc * 8 + i) + gn);
    }
  };
  auto store = [&](int buf) {
    bf16x8* Ad = As + buf * BM * 8;
    bf16x8* Bd = Bs + buf * BN * 8;
    if (!AT) {
#pragma unroll
      for (int i = 0; i < A_CH; ++i) {
        const int idx = tid + i * 256, row = idx >> 3, ch = idx & 7;
        Ad[lds_slot<1>(row, ch)] = a_reg[i];
      }
    } else if (tid < BM) {
      const int mc = tid % (BM / 8), kc = tid / (BM / 8);
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        bf16x8 v;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = a_reg[i][r];
        Ad[lds_slot<1>(mc * 8 + r, kc)] = v;
        if (want_rs) {
#pragma unroll
          for (int i = 0; i < 8; ++i) rsum[r] += (float)a_reg[i][r];
        }
      }
    }
    if (!BT) {
#pragma unroll
      for (int i = 0; i < B_CH; ++i) {
        const int idx = tid + i * 256, row = idx >> 3, ch = idx & 7;
        Bd[lds_slot<1>(row, ch)] = b_reg[i];
      }
    } else if (tb >= 0) {
      const int nc = tb % (BN / 8), kc = tb / (BN / 8);
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        bf16x8 v;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = b_reg[i][r];
        Bd[lds_slot<1>(nc * 8 + r, kc)] = v;
      }
    }
  };

  load(0);
  store(0);
  __syncthreads();
  for (int s = 0; s < steps; ++s) {
    const int cur = s & 1;
    if (s + 1 < steps) load(s + 1);
    const bf16x8* Ac = As + cur * BM * 8;
    const bf16x8* Bc = Bs + cur * BN * 8;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      bf16x8 af[TM], bfr[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) af[i] = Ac[lds_slot<1>(wm * (BM / WM) + i * 32 + l32, kk * 2 + lhi)];
#pragma unroll
      for (int j = 0; j < TN; ++j) bfr[j] = Bc[lds_slot<1>(wn * (BN / WN) + j * 32 + l32, kk * 2 + lhi)];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
    }
    if (s + 1 < steps) store(cur ^ 1);
    __syncthreads();
  }

  if (AT && rowsum != nullptr && blockIdx.x == 0) {       // block-uniform: the eight shares of a row meet in LDS
    float* part = reinterpret_cast<float*>(smem);         // [8 shares][BM rows]; the stages are no longer read
    if (tid < BM) {
      const int mc = tid % (BM / 8), kc = tid / (BM / 8);
#pragma unroll
      for (int r = 0; r < 8; ++r) part[kc * BM + mc * 8 + r] = rsum[r];
    }
    __syncthreads();
    if (tid < BM && m0 + tid < M) {
      float sum = 0.f;
#pragma unroll
      for (int kc = 0; kc < 8; ++kc) sum += part[kc * BM + tid];
      rowsum[d.rs_sk * k + d.rs_sa * a + m0 + tid] = from_f32<TC>(sum);
    }
  }

  // 32x32 accumulator block: lane holds column (lane % 32); register r holds row 8 (r / 4) + 4 (lane / 32) + r % 4
  TC* Cb = C + d.C.sb * b0 + d.C.sk * k + d.C.sa * a;
  const bf16* bs = bias ? bias + d.bias_sk * k + d.bias_sa * a : nullptr;
  const TC* radd = EXTRA ? static_cast<const TC*>(d.rowadd) : nullptr;
  if (sizeof(TC) == 2 && d.c_vec) {
    // the tile goes through LDS (the stages are no longer read) so that rows leave in 16-byte chunks:
    // a lane's accumulator column is 2 bytes wide, a row of the tile up to 256 bytes
    constexpr int PITCH = BN + 8;                          // bf16 elements; 16 extra bytes keep the row starts apart
    bf16* tile = reinterpret_cast<bf16*>(smem);
    __syncthreads();                                      // (also orders the row-sum scratch before this reuse)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int nl = wn * (BN / WN) + j * 32 + l32;
      const float bv = (bs && n0 + nl < d.N) ? (float)bs[n0 + nl] : 0.f;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int ml = wm * (BM / WM) + i * 32 + 8 * (r >> 2) + 4 * lhi + (r & 3);
          float v = acc[i][j][r] * d.scale + bv;
          if (radd && m0 + ml < M && n0 + nl < d.N) v += to_f32(radd[(size_t)(m0 + ml) * d.N + n0 + nl]);
          tile[ml * PITCH + nl] = (bf16)v;
        }
    }
    __syncthreads();
    for (int idx = tid; idx < BM * (BN / 8); idx += 256) {
      const int ml = idx / (BN / 8), ch = idx % (BN / 8);
      const int m = m0 + ml, n = n0 + ch * 8;
      if (m < M && n < d.N)
        *reinterpret_cast<bf16x8*>(reinterpret_cast<bf16*>(Cb) + d.C.s0 * m + n) =
            *reinterpret_cast<const bf16x8*>(tile + ml * PITCH + ch * 8);
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = n0 + wn * (BN / WN) + j * 32 + l32;
    if (n >= d.N) continue;
    const float bv = bs ? (float)bs[n] : 0.f;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = m0 + wm * (BM / WM) + i * 32 + 8 * (r >> 2) + 4 * lhi + (r & 3);
        if (m < M)
          Cb[d.C.s0 * m + d.C.s1 * n] =
              from_f32<TC>(acc[i][j][r] * d.scale + bv + (radd ? to_f32(radd[(size_t)m * d.N + n]) : 0.f));
      }
  }
}

__device__ __align__(16) const bf16 kZeroPiece[8] = {};                 // what stands past the end of a contraction

// ---------------------------------------------------------------------------------------
// The products of k_gemm_mfma where every row is 16-byte aligned, transposed extents multiples of 8 and C's rows whole 16-byte pieces
// (host): the same contract (bias, row addend, scale, ragged M, sums over batch elements, row sums of a transposed A, a last slice of
// fewer than 64 steps), with slices brought in by direct-to-LDS loads, ST - 1 of them ahead, 16x16x32 instructions and transposing LDS reads
// (RowOperand, ColOperand of the large products).  k_gemm_mfma stages through registers one slice ahead and transposes there.  Before / after,
// us, D 1024: one group, 1024 rows: dWo 22 / 10, d_o 16.5 / 9, dWv 24 / 13.5, w 17 / 14, output projection (the 128 x 128 ring it had)
// 16.5 / 10; one group, 4096 rows: dWo 75 / 29, dWv 82 / 39, d_o 24 / 17; eight groups of 512 rows, D 2048, u Wv: 103 / 90.
// Four wavefronts (WM x WN).  Products are taken as B^T A^T: a lane holds one row and four adjacent columns a block, trades with lane ^ 16
// and stores 16 bytes.  ST: 4 stages while there is at most a tile to a compute unit, 2 otherwise (two or more blocks to a unit).
// grid (ceil(N/BN), ceil(M/BM), batch), block 256, dynamic LDS ST (BM + BN) 128 bytes.
// ---------------------------------------------------------------------------------------
template <int BM, int BN, int WM, int WN, bool AT, bool BT, int ST>
__global__ __launch_bounds__(256) void k_gemm_ring(GemmDesc d, const bf16* __restrict__ A, const bf16* __restrict__ Bm,
                                                   const bf16* __restrict__ bias, bf16* __restrict__ C, bf16* __restrict__ rowsum) {
  typedef std::conditional_t<AT, ColOperand<BM * 2>, RowOperand> OA;
  typedef std::conditional_t<BT, ColOperand<BN * 2>, RowOperand> OB;
  constexpr int TM = BM / WM / 16, TN = BN / WN / 16, AL = BM / 32, BL = BN / 32, STAGE = (BM + BN) * 128;
  static_assert(WM * WN == 4 && TN % 2 == 0 && (BM == 64 || BM == 128) && (BN == 64 || BN == 128), "tile");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int z = blockIdx.z;
  const int a = z % d.na;
  z /= d.na;
  const int k = z % d.nk;
  const int b0 = d.reduce_b ? 0 : z / d.nk;
  const int nb = d.reduce_b ? d.nb : 1;
  int M = d.M;
  if (d.ragged == 1) {
    const int left = d.ragged_total - k * d.ragged_nominal;
    M = left < d.ragged_nominal ? left : d.ragged_nominal;
  }
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  if (m0 >= M) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN, l16 = lane & 15, lq = lane >> 4;
  const int KT = (d.K + 63) / 64, steps = nb * KT;

  // Loads of an operand: R / 8 of 1 KiB, R / 32 to a wavefront.  Row r of the operand (T false): 8 rows a load; step of the slice
  // (T true): 1024 / (2 R) steps a load.  off: byte of a lane's 16 behind the tile's origin, the same for every slice.
  auto offsets = [&](auto op, bool T, int R, int r0, int ext, long srow, long sk, unsigned* off, int n) {
#pragma unroll
    for (int i = 0; i < n; ++i) {
      const int ld = wave * n + i;
      if (!T) {
        const int row = ld * 8 + (lane >> 3);
        off[i] = (unsigned)min(row, ext - 1 - r0) * (unsigned)srow * 2 + ((lane & 7) ^ swz_chunk(row)) * 16;
      } else {
        const int cpr = R / 8, row = ld * (64 / cpr) + lane / cpr;       // chunks a step, step of the slice
        const int col = min(((lane % cpr) ^ decltype(op)::swz(row)) * 8, ext - 8 - r0);
        off[i] = (unsigned)row * (unsigned)sk * 2 + col * 2;
      }
    }
  };
  struct NoSwz { static __device__ __forceinline__ int swz(int) { return 0; } };
  typedef std::conditional_t<AT, ColOperand<BM * 2>, NoSwz> SA;
  typedef std::conditional_t<BT, ColOperand<BN * 2>, NoSwz> SB;
  unsigned a_off[AL], b_off[BL];
  offsets(SA{}, AT, BM, m0, M, d.A.s0, d.A.s1, a_off, AL);
  offsets(SB{}, BT, BN, n0, d.N, d.Bm.s1, d.Bm.s0, b_off, BL);
  const bf16* Ab = A + d.A.sb * b0 + d.A.sk * k + d.A.sa * a + d.A.s0 * m0;
  const bf16* Bb = Bm + d.Bm.sb * b0 + d.Bm.sk * k + d.Bm.sa * a + d.Bm.s1 * n0;
  const bf16 *pa = Ab, *pb = Bb;
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(lptr_t)smem);
  int ki = 0, is = 0;
  // A load of a segment's last, shorter slice: 16 bytes past the contraction's end come from the zeros instead.  at: the first
  // contraction element of a lane's 16 bytes.
  auto tail = [&](const bf16* base, unsigned off, int at, int dst) {
    const bf16* src = at < d.K ? reinterpret_cast<const bf16*>(reinterpret_cast<const char*>(base) + off) : kZeroPiece;
    load16_to_lds(src, smem + dst);
  };
  auto first_of = [&](bool T, int R, int ld) {             // contraction element of a lane's 16 bytes in load ld of a slice
    return ki * 64 + (T ? ld * (512 / R) + lane / (R / 8) : ((lane & 7) ^ swz_chunk(ld * 8 + (lane >> 3))) * 8);
  };
  auto issue = [&]() {
    const unsigned dst = lds0 + is * STAGE;
    if (ki == KT - 1 && d.K % 64) {                        // uniform
#pragma unroll
      for (int i = 0; i < AL; ++i) tail(pa, a_off[i], first_of(AT, BM, wave * AL + i), is * STAGE + (wave * AL + i) * 1024);
#pragma unroll
      for (int i = 0; i < BL; ++i)
        tail(pb, b_off[i], first_of(BT, BN, wave * BL + i), is * STAGE + BM * 128 + (wave * BL + i) * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < AL; ++i) load16_to_lds_at(pa, a_off[i], dst + (wave * AL + i) * 1024);
#pragma unroll
      for (int i = 0; i < BL; ++i) load16_to_lds_at(pb, b_off[i], dst + BM * 128 + (wave * BL + i) * 1024);
    }
    is = is == ST - 1 ? 0 : is + 1;
    pa += AT ? d.A.s1 * 64 : 64;
    pb += BT ? d.Bm.s0 * 64 : 64;
    if (++ki == KT) {                                      // the next batch element of the sum
      ki = 0;
      Ab += d.A.sb;
      Bb += d.Bm.sb;
      pa = Ab;
      pb = Bb;
    }
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // row sums of A: wavefront column wn takes the blocks i = wn, wn + WN, .. of its rows, by products with ones
  constexpr int RS = (TM + WN - 1) / WN;
  f32x4 rs[RS];
#pragma unroll
  for (int i = 0; i < RS; ++i) rs[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  const bool want_rs = AT && rowsum != nullptr && blockIdx.x == 0;
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (bf16)1.f;

  const int a_ad = OA::base(wm * (BM / WM), lane), b_ad = BM * 128 + OB::base(wn * (BN / WN), lane);
#pragma unroll
  for (int s = 0; s < ST - 1; ++s)
    if (s < steps) issue();
  int sc = 0;
  for (int s = 0; s < steps; ++s) {
    // slice s has landed (this wavefront's share; the ST - 2 behind it may stay in flight), every wavefront is done with slice s - 1
    const int behind = min(steps - 1 - s, ST - 2);         // uniform
    if (behind >= 2) wait_vmcnt<2 * (AL + BL)>();
    else if (behind == 1) wait_vmcnt<AL + BL>();
    else wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (s + ST - 1 < steps) issue();
    const unsigned char* st = smem + sc * STAGE;
    sc = sc == ST - 1 ? 0 : sc + 1;
    bf16x8 af[2][TM], bfr[2][TN];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
      for (int i = 0; i < TM; ++i) af[kk][i] = OA::frag(st, a_ad, i, kk, 0);
#pragma unroll
      for (int j = 0; j < TN; ++j) bfr[kk][j] = OB::frag(st, b_ad, j, kk, 0);
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[kk][j], af[kk][i], acc[i][j], 0, 0, 0);
      if (want_rs) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
          if (i % WN == wn) rs[i / WN] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, af[kk][i], rs[i / WN], 0, 0, 0);
      }
    }
  }
  // block (i, j): row 16 i + l16, columns 16 j + 4 lq + e
  if (want_rs && lq == 0) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = m0 + wm * (BM / WM) + i * 16 + l16;
      if (i % WN == wn && m < M) rowsum[d.rs_sk * k + d.rs_sa * a + m] = (bf16)rs[i / WN][0];
    }
  }
  bf16* Cb = C + d.C.sb * b0 + d.C.sk * k + d.C.sa * a;
  const bf16* radd = static_cast<const bf16*>(d.rowadd);
  const bf16* bs = bias ? bias + d.bias_sk * k + d.bias_sa * a : nullptr;
#pragma unroll
  for (int jj = 0; jj < TN / 2; ++jj) {
    const int col = n0 + wn * (BN / WN) + jj * 32;
    f32x4 bq[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      bq[j] = f32x4{0.f, 0.f, 0.f, 0.f};
      const int c = col + 16 * j + 4 * lq;
      if (bs && c < d.N) {
        const bf16x4 v = *reinterpret_cast<const bf16x4*>(bs + c);
#pragma unroll
        for (int e = 0; e < 4; ++e) bq[j][e] = (float)v[e];
      }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
      typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
      u32x2 w[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        f32x4 v = acc[i][2 * jj + j] * d.scale + bq[j];
        const int mr = m0 + wm * (BM / WM) + i * 16 + l16, cr = col + 16 * j + 4 * lq;
        if (radd && mr < M && cr < d.N) {
          const bf16x4 ra = *reinterpret_cast<const bf16x4*>(radd + (size_t)mr * d.N + cr);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] += (float)ra[e];
        }
        bf16x4 q;
#pragma unroll
        for (int e = 0; e < 4; ++e) q[e] = (bf16)v[e];
        w[j] = __builtin_bit_cast(u32x2, q);
      }
      // lane rows 0 and 2 (of 16) keep block 2 jj and take the next row's columns of it; rows 1 and 3 the same of block 2 jj + 1
      const auto s0 = __builtin_amdgcn_permlane16_swap(w[0][0], w[1][0], false, false);
      const auto s1 = __builtin_amdgcn_permlane16_swap(w[0][1], w[1][1], false, false);
      const int m = m0 + wm * (BM / WM) + i * 16 + l16, c = col + (lq & 1) * 16 + (lq >> 1) * 8;
      if (m < M && c < d.N) *reinterpret_cast<u32x4*>(Cb + d.C.s0 * m + c) = u32x4{s0[0], s1[0], s0[1], s1[1]};
    }
  }
}

// ---------------------------------------------------------------------------------------
// The same products in single precision: 64 x 64 tiles on v_mfma_f32_32x32x2_f32 (fp32 operands and accumulation, twice
// the rate of unpacked vector FMAs), contraction in slices of 32, four wavefronts (2 x 2) of 32 x 32.  Takes the whole
// GemmDesc contract (ragged M or K, any strides with one unit stride per operand, any alignment) plus a row addend.
//   Rows of 32 contraction steps lie in LDS with a pitch of 36 floats (16-byte reads of 32 rows hit every bank group
//   evenly); a lane reads four steps at once, half 0 of the wavefront steps 8 s .. 8 s + 3 and half 1 the next four, and
//   feeds them to four products (both operands pair the steps the same way, so the contraction is complete).
//   An operand whose unit stride is the contraction index is copied in 16-byte pieces, one whose unit stride is its row
//   index is read as 4 x 4 blocks and transposed in registers.  Two slices are in flight in registers ahead of the
//   one being multiplied: what bounded the FMA kernels it replaces was a load round trip per 16 steps (2 to 3 us each;
//   24 us for a product over 128 steps).
//   A slice is added up on its own and then to the sum of the slices: chains of 32 and K / 32 instead of K.  One chain has the
//   error of the FMA kernels, more than the wavefront-wide sums that the scores had (outputs 1.18 times the error over 40 drawn
//   calls, up to 1.44); with slices 0.51 times (0.86 at most), for 1 % of a training step of 80 variables (947 -> 960 us; adding the
//   last slice under the next one's products takes 16 registers more and 1018 us).
//   split > 1: the contraction is dealt to `split` blocks, block t takes slices [t, t + 1) * per of it and writes its own
//   partial result at offset split_stride * t (per batch item); bias and addend are then not applied.
// grid (ceil(N/64), ceil(M/64), batch * split), block 256.
// ---------------------------------------------------------------------------------------
template <bool AT, bool BT>
__global__ __launch_bounds__(256) void k_gemm_f32(GemmDesc d, int va, int vb, int split, long split_stride,
                                                  const float* __restrict__ A, const float* __restrict__ Bm,
                                                  const float* __restrict__ bias, float* __restrict__ C) {
  constexpr int PITCH = 36;
  __shared__ __attribute__((aligned(16))) float As[2][64 * PITCH];
  __shared__ __attribute__((aligned(16))) float Bs[2][64 * PITCH];
  int z = blockIdx.z;
  const int part = z % split;
  z /= split;
  const int a = z % d.na;
  z /= d.na;
  const int k = z % d.nk;
  const int b0 = d.reduce_b ? 0 : z / d.nk;
  const int b1 = d.reduce_b ? d.nb : b0 + 1;
  int M = d.M, K = d.K;
  if (d.ragged) {
    int left = d.ragged_total - k * d.ragged_nominal;
    left = left < d.ragged_nominal ? left : d.ragged_nominal;
    if (d.ragged == 1) M = left; else K = left;
  }
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  if (m0 >= M) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, lhi = lane >> 5;
  const int KT = (K + 31) / 32;
  const int per = ((b1 - b0) * KT + split - 1) / split;
  const int s_begin = part * per, s_end = min(s_begin + per, (b1 - b0) * KT);

  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 acc = zero;

  // one operand's share of a slice in registers: four 16-byte pieces (row-fast operands: a 4 x 4 block; others: two pieces)
  auto load_op = [&](bool T, int vec, const float* P, long srow, long sk, int r0, int R, int k0, int t, f32x4 (&reg)[4]) {
    if (!T) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int idx = tid + i * 256, row = r0 + (idx >> 3), kk = k0 + (idx & 7) * 4;
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        if (row < R) {
          const float* p = P + srow * row + kk;
          if (vec && kk + 4 <= K) v = *reinterpret_cast<const f32x4*>(p);
          else
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (kk + e < K) v[e] = p[e];
        }
        reg[i] = v;
      }
    } else if (t >= 0 && t < 128) {                         // 16 row blocks x 8 blocks of four steps
      const int row = r0 + (t & 15) * 4, kb = k0 + (t >> 4) * 4;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        if (kb + i < K) {
          const float* p = P + sk * (kb + i) + row;
          if (vec && row + 4 <= R) v = *reinterpret_cast<const f32x4*>(p);
          else
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (row + e < R) v[e] = p[e];
        }
        reg[i] = v;
      }
    }
  };
  auto store_op = [&](bool T, float* S, int t, const f32x4 (&reg)[4]) {
    if (!T) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int idx = tid + i * 256;
        *reinterpret_cast<f32x4*>(S + (idx >> 3) * PITCH + (idx & 7) * 4) = reg[i];
      }
    } else if (t >= 0 && t < 128) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        *reinterpret_cast<f32x4*>(S + ((t & 15) * 4 + e) * PITCH + (t >> 4) * 4) =
            f32x4{reg[0][e], reg[1][e], reg[2][e], reg[3][e]};
    }
  };
  const int ta = tid, tb = BT && AT ? tid - 128 : tid;
  f32x4 ar[2][4], br[2][4];                                  // the two slices in flight
  auto load = [&](int s, f32x4 (&ra)[4], f32x4 (&rb)[4]) {
    const int b = b0 + s / KT, k0 = (s % KT) * 32;
    load_op(AT, va, A + d.A.sb * b + d.A.sk * k + d.A.sa * a, d.A.s0, d.A.s1, m0, M, k0, ta, ra);
    load_op(BT, vb, Bm + d.Bm.sb * b + d.Bm.sk * k + d.Bm.sa * a, d.Bm.s1, d.Bm.s0, n0, d.N, k0, tb, rb);
  };
  auto multiply = [&](int buf) {
    const float* Ap = As[buf] + (wm * 32 + l32) * PITCH + lhi * 4;
    const float* Bp = Bs[buf] + (wn * 32 + l32) * PITCH + lhi * 4;
    f32x16 slice = zero;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 av = *reinterpret_cast<const f32x4*>(Ap + q * 8), bv = *reinterpret_cast<const f32x4*>(Bp + q * 8);
#pragma unroll
      for (int e = 0; e < 4; ++e) slice = __builtin_amdgcn_mfma_f32_32x32x2f32(av[e], bv[e], slice, 0, 0, 0);
    }
    acc += slice;
  };
  // slice s goes to LDS buffer s & 1 one step before it is multiplied; its registers then take slice s + 2
  auto step = [&](int s, int buf, f32x4 (&ra)[4], f32x4 (&rb)[4]) {   // ra, rb: slice s + 1's registers
    if (s + 1 < s_end) {
      store_op(AT, As[buf ^ 1], ta, ra);
      store_op(BT, Bs[buf ^ 1], tb, rb);
      if (s + 3 < s_end) load(s + 3, ra, rb);
    }
    multiply(buf);
    __syncthreads();
  };
  if (s_begin < s_end) {
    load(s_begin, ar[0], br[0]);
    if (s_begin + 1 < s_end) load(s_begin + 1, ar[1], br[1]);
    store_op(AT, As[0], ta, ar[0]);
    store_op(BT, Bs[0], tb, br[0]);
    if (s_begin + 2 < s_end) load(s_begin + 2, ar[0], br[0]);
    __syncthreads();
    for (int s = s_begin; s < s_end; s += 2) {
      step(s, 0, ar[1], br[1]);
      if (s + 1 < s_end) step(s + 1, 1, ar[0], br[0]);
    }
  }
  // lane: column l32, register r: row 8 (r / 4) + 4 (lane / 32) + r % 4
  const int n = n0 + wn * 32 + l32;
  if (n >= d.N) return;
  float* Cb = C + d.C.sb * b0 + d.C.sk * k + d.C.sa * a + split_stride * part;
  const float bv = bias && split == 1 ? bias[d.bias_sk * k + d.bias_sa * a + n] : 0.f;
  const float* radd = split == 1 ? static_cast<const float*>(d.rowadd) : nullptr;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = m0 + wm * 32 + 8 * (r >> 2) + 4 * lhi + (r & 3);
    if (m < M) Cb[d.C.s0 * m + d.C.s1 * n] = acc[r] * d.scale + bv + (radd ? radd[(size_t)m * d.N + n] : 0.f);
  }
}

// ---------------------------------------------------------------------------------------
// The same products where every row is 16-byte aligned, every contraction a multiple of 32 and the extent of an operand whose
// unit stride is its row index a multiple of 4 (host): the same tiles, instructions and order of sums, with the slices brought in by
// direct-to-LDS loads two slices ahead (three 16-KiB stages, three blocks to a compute unit).  What the kernel above waits for is
// itself: 64-bit addresses, range checks and register copies of every piece.  640 blocks of 16 slices 41 .. 46 -> 34 .. 35 us (60 % of
// the matrix units' time), with two transposed operands 55 -> 34; 64 blocks 21 .. 26 -> 16.
//   A slice of an operand whose unit stride is the contraction index is 64 rows of 128 bytes, chunks swizzled as in the bf16
//   kernels (lane l of 32 reads 16 bytes of row l, half h of the wavefront steps 8 q + 4 h ..).  One whose unit stride is its
//   row index is 32 steps of 64 rows, 256 bytes each, read four bytes a lane; the two halves of a wavefront read steps four
//   apart, so every second four steps have the halves of their 256 bytes exchanged and the 64 lanes meet 64 banks.
//   Four sets of wavefronts a block with a quarter of the slices each (few tiles) gained a tenth at 64 blocks of 16 slices (16 -> 15
//   us) and lost as much at four slices, and tiles dealt to the XCDs by rows changed nothing: neither is kept.
// grid (ceil(N/64), ceil(M/64), batch * split), block 256.
// ---------------------------------------------------------------------------------------
template <bool AT, bool BT>
__global__ __launch_bounds__(256) void k_gemm_f32_ring(GemmDesc d, int split, long split_stride, const float* __restrict__ A,
                                                       const float* __restrict__ Bm, const float* __restrict__ bias,
                                                       float* __restrict__ C) {
  constexpr int STAGE = 16384, OPB = 8192;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[3 * STAGE];
  int z = blockIdx.z;
  const int part = z % split;
  z /= split;
  const int a = z % d.na;
  z /= d.na;
  const int k = z % d.nk;
  const int b0 = d.reduce_b ? 0 : z / d.nk;
  const int b1 = d.reduce_b ? d.nb : b0 + 1;
  int M = d.M, K = d.K;
  if (d.ragged) {
    int left = d.ragged_total - k * d.ragged_nominal;
    left = left < d.ragged_nominal ? left : d.ragged_nominal;
    if (d.ragged == 1) M = left; else K = left;
  }
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  if (m0 >= M) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, lhi = lane >> 5;
  const int KT = K / 32;
  const int per = ((b1 - b0) * KT + split - 1) / split;
  const int s_begin = part * per, s_end = min(s_begin + per, (b1 - b0) * KT);

  // loads 2 w and 2 w + 1 of an operand's eight (1 KiB each): rows 8 i .. 8 i + 7, or steps 4 i .. 4 i + 3
  auto offsets = [&](bool T, int r0, int R, long srow, long sk, unsigned (&off)[2]) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int i = wave * 2 + u;
      if (!T) {
        const int row = i * 8 + (lane >> 3);
        off[u] = (unsigned)min(row, R - 1 - r0) * (unsigned)srow * 4 + ((lane & 7) ^ swz_chunk(row)) * 16;
      } else {
        const int col = min(((lane & 15) ^ (8 * (i & 1))) * 4, R - 4 - r0);
        off[u] = (unsigned)(i * 4 + (lane >> 4)) * (unsigned)sk * 4 + col * 4;
      }
    }
  };
  unsigned a_off[2], b_off[2];
  offsets(AT, m0, M, d.A.s0, d.A.s1, a_off);
  offsets(BT, n0, d.N, d.Bm.s1, d.Bm.s0, b_off);
  const float* Ab = A + d.A.sk * k + d.A.sa * a + d.A.s0 * m0;
  const float* Bb = Bm + d.Bm.sk * k + d.Bm.sa * a + d.Bm.s1 * n0;
  int ib = b0 + s_begin / KT, ik = s_begin % KT;             // batch element and slice of the next loads
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(lptr_t)smem) + wave * 2048;
  int is = 0;
  auto issue = [&]() {
    const float* pa = Ab + d.A.sb * ib + (AT ? d.A.s1 * 32 : 32) * (long)ik;
    const float* pb = Bb + d.Bm.sb * ib + (BT ? d.Bm.s0 * 32 : 32) * (long)ik;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      load16_to_lds_at(pa, a_off[u], lds0 + is * STAGE + u * 1024);
      load16_to_lds_at(pb, b_off[u], lds0 + is * STAGE + OPB + u * 1024);
    }
    is = is == 2 ? 0 : is + 1;
    if (++ik == KT) {
      ik = 0;
      ++ib;
    }
  };
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 acc = zero;
  // steps 8 q + 4 lhi + e, e = 0 .. 3, of this lane's row
  auto read = [&](bool T, const unsigned char* st, int w, int q, float (&v)[4]) {
    if (!T) {
      const int row = w * 32 + l32;
      const f32x4 t = *reinterpret_cast<const f32x4*>(st + row * 128 + ((2 * q + lhi) ^ swz_chunk(row)) * 16);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = t[e];
    } else {
      const unsigned char* p = st + (8 * q + 4 * lhi) * 256 + ((w * 32 + l32) ^ (32 * lhi)) * 4;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = *reinterpret_cast<const float*>(p + e * 256);
    }
  };
  if (s_begin < s_end) issue();
  if (s_begin + 1 < s_end) issue();
  int sc = 0;
  for (int s = s_begin; s < s_end; ++s) {
    // slice s has landed (this wavefront's share; slice s + 1 may stay in flight), and every wavefront is done with slice s - 1
    if (s + 1 < s_end) wait_vmcnt<4>();
    else wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (s + 2 < s_end) issue();
    const unsigned char* st = smem + sc * STAGE;
    sc = sc == 2 ? 0 : sc + 1;
    float av[4][4], bv[4][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      read(AT, st, wm, q, av[q]);
      read(BT, st + OPB, wn, q, bv[q]);
    }
    f32x16 slice = zero;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) slice = __builtin_amdgcn_mfma_f32_32x32x2f32(av[q][e], bv[q][e], slice, 0, 0, 0);
    acc += slice;
  }
  // lane: column l32, register r: row 8 (r / 4) + 4 (lane / 32) + r % 4
  const int n = n0 + wn * 32 + l32;
  if (n >= d.N) return;
  float* Cb = C + d.C.sb * b0 + d.C.sk * k + d.C.sa * a + split_stride * part;
  const float bv = bias && split == 1 ? bias[d.bias_sk * k + d.bias_sa * a + n] : 0.f;
  const float* radd = split == 1 ? static_cast<const float*>(d.rowadd) : nullptr;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = m0 + wm * 32 + 8 * (r >> 2) + 4 * lhi + (r & 3);
    if (m < M) Cb[d.C.s0 * m + d.C.s1 * n] = acc[r] * d.scale + bv + (radd ? radd[(size_t)m * d.N + n] : 0.f);
  }
}

// ---------------------------------------------------------------------------------------
// Softmax weights from the layout of the forward kernels, alpha_f[b][k][cl][head][n] (pitch Np, gpad
// members per group), to token-major alpha[b,c,n,head].  One thread per output element.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_alpha_token_major(long total, int Cin, int N, int heads, int g, int gpad,
                                                           int G, int Np, const float* __restrict__ alpha_f,
                                                           float* __restrict__ alpha) {
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;      // ((b * Cin + c) * N + n) * heads + a
  if (idx >= total) return;
  const int a = (int)(idx % heads);
  long t = idx / heads;
  const int n = (int)(t % N);
  t /= N;
  const int c = (int)(t % Cin), b = (int)(t / Cin);
  const int k = c / g, cl = c % g;
  alpha[idx] = alpha_f[((((size_t)b * G + k) * gpad + cl) * heads + a) * Np + n];
}

// ---------------------------------------------------------------------------------------
// Per-head weighted token sums, bf16, D % 4 == 0:
//   u[b,k,n,a,:] = sum_{c in group k} alpha[b,c,n,a] * z[b,c,n,:]
// grid (N, G, B), block 256: a thread owns 4 adjacent columns (and every 1024th after them) and
// keeps one fp32 sum per head; the group's weights for this patch sit in LDS.  Bound by the read
// of z (2 D bytes per token) and the write of u.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_head_sums_bf16(int Cin, int N, int D, int heads, int g,
                                                        const float* __restrict__ alpha, const bf16* __restrict__ z,
                                                        bf16* __restrict__ u) {
  extern __shared__ __attribute__((aligned(16))) float al[];      // [gk][16]: the weights of one block of 16 heads
  const int n = blockIdx.x, k = blockIdx.y, b = blockIdx.z, G = gridDim.y;
  const int c0 = k * g, gk = min(g, Cin - c0);
  const size_t cstride = (size_t)N * D;
  for (int a0 = 0; a0 < heads; a0 += 16) {                        // more than 16 heads: z is walked once per block
    __syncthreads();
    for (int idx = threadIdx.x; idx < gk * 16; idx += 256) {
      const int cl = idx >> 4, a = a0 + (idx & 15);
      al[idx] = a < heads ? alpha[(((size_t)b * Cin + c0 + cl) * N + n) * heads + a] : 0.f;
    }
    __syncthreads();
    for (int d0 = threadIdx.x * 4; d0 < D; d0 += 1024) {
      const bf16* zp = z + (((size_t)b * Cin + c0) * N + n) * D + d0;
      float acc[16][4];
#pragma unroll
      for (int a = 0; a < 16; ++a)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[a][e] = 0.f;
      int cl = 0;
      for (; cl + 4 <= gk; cl += 4) {
        bf16x4 zv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) zv[i] = *reinterpret_cast<const bf16x4*>(zp + (size_t)(cl + i) * cstride);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f32x4* ar = reinterpret_cast<const f32x4*>(al + (cl + i) * 16);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 av = ar[q];
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
              for (int e = 0; e < 4; ++e) acc[q * 4 + a][e] += av[a] * (float)zv[i][e];
          }
        }
      }
      for (; cl < gk; ++cl) {
        const bf16x4 zv = *reinterpret_cast<const bf16x4*>(zp + (size_t)cl * cstride);
#pragma unroll
        for (int a = 0; a < 16; ++a)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[a][e] += al[cl * 16 + a] * (float)zv[e];
      }
      bf16* up = u + ((((size_t)b * G + k) * N + n) * heads + a0) * D + d0;
#pragma unroll
      for (int a = 0; a < 16; ++a)
        if (a0 + a < heads) {
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = (bf16)acc[a][e];
          *reinterpret_cast<bf16x4*>(up + (size_t)a * D) = o;
        }
    }
  }
}

// ---------------------------------------------------------------------------------------
// Scores, softmax and per-head weighted token sums of a level whose tokens are in HBM, in one kernel (bf16, D % 256 == 0,
// heads <= 16 NB):
//   alpha[b,c,n,a] = softmax over the group's members c of z[b,c,n,:] . M[k][a][:]       (token-major)
//   u[b,k,n,a,:]   = sum_c alpha[b,c,n,a] z[b,c,n,:]
// A block owns PN patches of one (b, k).  Scores: a wavefront contracts its quarter of the D features on 16x16x32 MFMA (16
// members x 16 heads a tile, the key fragments shared by the PN patches), the quarters meet in LDS.  Softmax: a wavefront per
// (patch, 16 heads), four lanes to a head.  Sums: an item is (patch, HB heads, 4 columns), fp32, members in order; the tokens come
// a second time from the L2.  Replaces four launches (scores, softmax, re-layout, sums) whose weights went through HBM twice:
// bound by the read of z and the write of u, at small sizes by the launch itself (128 patches, 10 members, D 256: the whole
// served call went from 55 to 44 us).
// grid (ceil(N/PN), G, B), block 256, dynamic LDS level_sums_lds(PN, NB, g).
// ---------------------------------------------------------------------------------------
constexpr size_t level_sums_lds(int PN, int NB, int g) { return (size_t)PN * NB * (4096 + 64 * (size_t)g); }

template <int NB, int PN, int HB>
__global__ __launch_bounds__(256) void k_level_sums(int Cin, int N, int D, int heads, int g, const bf16* __restrict__ z,
                                                    const bf16* __restrict__ Mb, float* __restrict__ alpha,
                                                    bf16* __restrict__ u) {
  constexpr int HS = NB * 16;                                     // pitch of a member's weights
  extern __shared__ __attribute__((aligned(16))) float lds[];
  float* part = lds;                                              // [source wavefront][patch, head block, register][lane]
  float* sc = lds + 4 * PN * NB * 256;                            // [patch][member][HS]
  const int k = blockIdx.y, b = blockIdx.z, G = gridDim.y, n0 = blockIdx.x * PN;
  const int c0 = k * g, gk = min(g, Cin - c0);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, lq = lane >> 4;
  const size_t cstride = (size_t)N * D;
  const bf16* zg = z + ((size_t)b * Cin + c0) * cstride;
  const int koff = wave * (D / 4) + lq * 16;                      // two steps take the halves of a lane's 32 bytes
  const bf16* mrow[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) mrow[nb] = Mb + ((size_t)k * heads + min(nb * 16 + l16, heads - 1)) * D + koff;
  for (int m0 = 0; m0 < gk; m0 += 16) {
    const bf16* zp[PN];
#pragma unroll
    for (int p = 0; p < PN; ++p)
      zp[p] = zg + (size_t)min(m0 + l16, gk - 1) * cstride + (size_t)min(n0 + p, N - 1) * D + koff;
    f32x4 acc[PN][NB];
#pragma unroll
    for (int p = 0; p < PN; ++p)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[p][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
    for (int f = 0; f < D / 4; f += 64) {
      bf16x8 zf[PN][2], mf[NB][2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int p = 0; p < PN; ++p) zf[p][h] = *reinterpret_cast<const bf16x8*>(zp[p] + f + 8 * h);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) mf[nb][h] = *reinterpret_cast<const bf16x8*>(mrow[nb] + f + 8 * h);
      }
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int p = 0; p < PN; ++p)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
            acc[p][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zf[p][h], mf[nb][h], acc[p][nb], 0, 0, 0);
    }
    if (m0) __syncthreads();                                      // the last tile's partial blocks have been read
#pragma unroll
    for (int p = 0; p < PN; ++p)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int e = 0; e < 4; ++e) part[((wave * PN + p) * NB + nb) * 256 + e * 64 + lane] = acc[p][nb][e];
    __syncthreads();
    // accumulator block: lane holds head lane % 16, members 4 (lane / 16) + 0..3; wavefront e adds up register e
    const int cl = m0 + lq * 4 + wave;
    if (cl < gk) {
#pragma unroll
      for (int p = 0; p < PN; ++p)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const float* q = part + (p * NB + nb) * 256 + wave * 64 + lane;
          constexpr int S = PN * NB * 256;
          sc[(p * gk + cl) * HS + nb * 16 + l16] = ((q[0] + q[S]) + q[2 * S]) + q[3 * S];
        }
    }
  }
  __syncthreads();
  for (int it = wave; it < PN * NB; it += 4) {
    const int p = it / NB, a = (it % NB) * 16 + l16, n = n0 + p;
    float* s = sc + (size_t)p * gk * HS + a;
    float mx = -INFINITY;
    for (int cl = lq; cl < gk; cl += 4) mx = fmaxf(mx, s[cl * HS]);
    mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
    mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
    float den = 0.f;
    for (int cl = lq; cl < gk; cl += 4) den += __expf(s[cl * HS] - mx);
    den += __shfl_xor(den, 16, kWave);
    den += __shfl_xor(den, 32, kWave);
    const float inv = 1.f / den;
    for (int cl = lq; cl < gk; cl += 4) {
      const float v = __expf(s[cl * HS] - mx) * inv;
      s[cl * HS] = v;
      if (n < N && a < heads) alpha[(((size_t)b * Cin + c0 + cl) * N + n) * heads + a] = v;
    }
  }
  __syncthreads();
  const int DC = D / 4, items = PN * (HS / HB) * DC;              // DC % 64 == 0: a wavefront shares patch and heads
  for (int it = threadIdx.x; it < items; it += 256) {
    const int d0 = (it % DC) * 4, t = it / DC, a0 = (t % (HS / HB)) * HB, p = t / (HS / HB), n = n0 + p;
    if (n >= N || a0 >= heads) continue;
    const bf16* zp = zg + (size_t)n * D + d0;
    const float* al = sc + (size_t)p * gk * HS + a0;
    float acc[HB][4];
#pragma unroll
    for (int a = 0; a < HB; ++a)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[a][e] = 0.f;
    auto add = [&](int cl, const bf16x4& zv) {
      const f32x4* ar = reinterpret_cast<const f32x4*>(al + (size_t)cl * HS);
#pragma unroll
      for (int q = 0; q < HB / 4; ++q) {
        const f32x4 av = ar[q];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[q * 4 + a][e] += av[a] * (float)zv[e];
      }
    };
    int cl = 0;
    for (; cl + 4 <= gk; cl += 4) {
      bf16x4 zv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) zv[i] = *reinterpret_cast<const bf16x4*>(zp + (size_t)(cl + i) * cstride);
#pragma unroll
      for (int i = 0; i < 4; ++i) add(cl + i, zv[i]);
    }
    for (; cl < gk; ++cl) add(cl, *reinterpret_cast<const bf16x4*>(zp + (size_t)cl * cstride));
    bf16* up = u + ((((size_t)b * G + k) * N + n) * heads + a0) * D + d0;
#pragma unroll
    for (int a = 0; a < HB; ++a)
      if (a0 + a < heads) {
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (bf16)acc[a][e];
        *reinterpret_cast<bf16x4*>(up + (size_t)a * D) = o;
      }
  }
}

// ---------------------------------------------------------------------------------------
// d alpha and the softmax Jacobian in one kernel (bf16, D % 32 == 0, group size <= 16 MT):
//   dalpha[c,a] = w[b,k,n,a,:] . z[b,c,n,:]            (16x16x32 MFMA: 16 members x 16 heads per block)
//   ds[c,a]     = alpha[c,a] * (dalpha[c,a] - sum_c' alpha[c',a] dalpha[c',a])
// One wavefront per (b, k, n): its A fragments are 16 member rows of z (64 contiguous bytes per row and
// step), its B fragments the head rows of w at this patch.  Accumulator block: lane holds head lane % 16,
// members 4 (lane / 16) + 0..3 of the tile.  grid ceil(B G N / 4), block 256.  Heads beyond 16 take
// further passes.  ds is written token-major [B,Cin,N,heads] like alpha.
// ---------------------------------------------------------------------------------------
template <int MT>
__global__ __launch_bounds__(256) void k_dalpha_softmax_mfma(long items, int Cin, int N, int D, int heads, int g,
                                                             int G, const bf16* __restrict__ z,
                                                             const bf16* __restrict__ w,
                                                             const float* __restrict__ alpha,
                                                             float* __restrict__ ds) {
  const long item = (long)blockIdx.x * 4 + (threadIdx.x >> 6);     // (b * G + k) * N + n
  if (item >= items) return;
  const int lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
  const int n = (int)(item % N);
  const int k = (int)((item / N) % G), b = (int)(item / ((long)N * G));
  const int c0 = k * g, gk = min(g, Cin - c0);
  const size_t cstride = (size_t)N * D;
  const bf16* zb = z + (((size_t)b * Cin + c0) * N + n) * D + lq * 8;
  for (int a0 = 0; a0 < heads; a0 += 16) {
    const int head = min(a0 + l16, heads - 1);
    const bf16* wr = w + ((size_t)item * heads + head) * D + lq * 8;
    const bf16* zr[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) zr[mt] = zb + (size_t)min(mt * 16 + l16, gk - 1) * cstride;
    f32x4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int t = 0; t < D; t += 128) {                             // four steps of 32 per trip, loads first
      bf16x8 wf[4], zf[MT][4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int tt = min(t + q * 32, D - 32);
        wf[q] = *reinterpret_cast<const bf16x8*>(wr + tt);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) zf[mt][q] = *reinterpret_cast<const bf16x8*>(zr[mt] + tt);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (t + q * 32 < D) {
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zf[mt][q], wf[q], acc[mt], 0, 0, 0);
        }
    }
    // softmax Jacobian over the members (registers and the four lane groups of a head)
    float al[MT][4];
    float dot = 0.f;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int cl = mt * 16 + lq * 4 + r;
        al[mt][r] = (cl < gk && a0 + l16 < heads)
                        ? alpha[(((size_t)b * Cin + c0 + cl) * N + n) * heads + a0 + l16] : 0.f;
        dot += al[mt][r] * acc[mt][r];
      }
    dot += __shfl_xor(dot, 16, kWave);
    dot += __shfl_xor(dot, 32, kWave);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int cl = mt * 16 + lq * 4 + r;
        if (cl < gk && a0 + l16 < heads)
          ds[(((size_t)b * Cin + c0 + cl) * N + n) * heads + a0 + l16] = al[mt][r] * (acc[mt][r] - dot);
      }
  }
}

// ---------------------------------------------------------------------------------------
// The same for groups of any size (the flat single-layer baseline has one group of all channels), bf16, D % 32 == 0:
// one block of four wavefronts per (b, k, n).  The wavefronts take the tiles of 16 members in turn (16x16x32 MFMA as
// above, the head rows of w re-read from L1 per tile) and leave d alpha of the whole group in LDS; then the sums
// sum_c alpha dalpha per head are formed in a fixed order and ds is written.  grid B G N, block 256, dynamic LDS
// (16 ceil(g/16) + 17) * 16 floats.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_dalpha_softmax_group(int Cin, int N, int D, int heads, int g, int G,
                                                              const bf16* __restrict__ z, const bf16* __restrict__ w,
                                                              const float* __restrict__ alpha, float* __restrict__ ds) {
  extern __shared__ __attribute__((aligned(16))) float sm[];       // da[16 ntile][16], red[16][16], dot[16]
  const long item = blockIdx.x;                                    // (b * G + k) * N + n
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, lq = lane >> 4;
  const int n = (int)(item % N);
  const int k = (int)((item / N) % G), b = (int)(item / ((long)N * G));
  const int c0 = k * g, gk = min(g, Cin - c0);
  const int ntile = (gk + 15) / 16;
  float* da = sm;
  float* red = sm + ntile * 256;
  float* dot = red + 256;
  const size_t cstride = (size_t)N * D;
  const bf16* zb = z + (((size_t)b * Cin + c0) * N + n) * D + lq * 8;
  const float* ab = alpha + (((size_t)b * Cin + c0) * N + n) * heads;   // member cl: + cl * N * heads
  float* dsb = ds + (((size_t)b * Cin + c0) * N + n) * heads;
  const size_t astride = (size_t)N * heads;
  for (int a0 = 0; a0 < heads; a0 += 16) {
    const int head = min(a0 + l16, heads - 1);
    const bf16* wr = w + ((size_t)item * heads + head) * D + lq * 8;
    for (int tile = wave; tile < ntile; tile += 4) {
      const bf16* zr = zb + (size_t)min(tile * 16 + l16, gk - 1) * cstride;
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
      for (int t = 0; t < D; t += 128) {                           // four steps of 32 per trip, loads first
        bf16x8 wf[4], zf[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int tt = min(t + q * 32, D - 32);
          wf[q] = *reinterpret_cast<const bf16x8*>(wr + tt);
          zf[q] = *reinterpret_cast<const bf16x8*>(zr + tt);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (t + q * 32 < D) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zf[q], wf[q], acc, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) da[(tile * 16 + lq * 4 + r) * 16 + l16] = acc[r];   // lane: head l16, members 4 lq + r
    }
    __syncthreads();
    {
      const int hd = threadIdx.x & 15, part = threadIdx.x >> 4;
      float p = 0.f;
      if (a0 + hd < heads)
        for (int cl = part; cl < gk; cl += 16) p += ab[(size_t)cl * astride + a0 + hd] * da[cl * 16 + hd];
      red[part * 16 + hd] = p;
    }
    __syncthreads();
    if (threadIdx.x < 16) {
      float sum = 0.f;
#pragma unroll
      for (int part = 0; part < 16; ++part) sum += red[part * 16 + threadIdx.x];
      dot[threadIdx.x] = sum;
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < gk * 16; idx += 256) {
      const int cl = idx >> 4, hd = idx & 15;
      if (a0 + hd < heads)
        dsb[(size_t)cl * astride + a0 + hd] = ab[(size_t)cl * astride + a0 + hd] * (da[idx] - dot[hd]);
    }
    __syncthreads();                                               // the next block of heads overwrites da
  }
}

// ---------------------------------------------------------------------------------------
// Gradient at the input tokens and the key-path sums, bf16, heads <= 16, D % 4 == 0:
//   dz[b,c,n,:]   = sum_a alpha[b,c,n,a] * w[b,k,n,a,:] + ds[b,c,n,a] * M[k][a][:]
//   rpart[b,k,t][a][:] = sum over the PT patches of tile t and the members c of  ds[b,c,n,a] * z[b,c,n,:]
// grid (n_tiles * ceil(D / (4 NT)), G, B), n_tiles = ceil(N/PT), block NT = D / 4 to a multiple of 64, at most 256: a thread owns 4
// adjacent columns, keeps the HB rows (heads to 8 or 16)
// of M and (per patch) of w for them in registers, and walks the members.  The softmax weights and ds of
// the whole tile of PT patches sit in LDS (dynamic, 2 * PT * g * HB floats).  The partial sums are added up in a fixed
// order by k_sum_partials.  (16 rows and 256 threads whatever the shape: 6 heads and D 384 used a seventh of the arithmetic.)
// ---------------------------------------------------------------------------------------
template <int HB>
__global__ __launch_bounds__(256) void k_dz_rpart_bf16(int Cin, int N, int D, int heads, int g, int n_tiles, int PT,
                                                       const float* __restrict__ alpha, const float* __restrict__ ds,
                                                       const bf16* __restrict__ z, const bf16* __restrict__ w,
                                                       const bf16* __restrict__ Mb, bf16* __restrict__ dz,
                                                       float* __restrict__ rpart) {
  extern __shared__ __attribute__((aligned(16))) float sm[];       // al[PT][g][HB], then dsv[PT][g][HB]
  const int tile = blockIdx.x % n_tiles, cb = blockIdx.x / n_tiles;
  const int k = blockIdx.y, b = blockIdx.z, G = gridDim.y;
  const int c0 = k * g, gk = min(g, Cin - c0);
  const int n0 = tile * PT, np = min(PT, N - n0);
  float* al = sm;
  float* dsv = sm + PT * g * HB;
  for (int idx = threadIdx.x; idx < np * gk * HB; idx += blockDim.x) {
    const int a = idx % HB, cl = (idx / HB) % gk, pi = (idx / HB) / gk;
    const size_t src = (((size_t)b * Cin + c0 + cl) * N + n0 + pi) * heads + a;
    al[(pi * g + cl) * HB + a] = a < heads ? alpha[src] : 0.f;
    dsv[(pi * g + cl) * HB + a] = a < heads ? ds[src] : 0.f;
  }
  __syncthreads();
  const int d0 = (cb * blockDim.x + threadIdx.x) * 4;
  if (d0 >= D) return;
  float mr[HB][4], racc[HB][4];
#pragma unroll
  for (int a = 0; a < HB; ++a) {
    bf16x4 mv = {};
    if (a < heads) mv = *reinterpret_cast<const bf16x4*>(Mb + ((size_t)k * heads + a) * D + d0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      mr[a][e] = (float)mv[e];
      racc[a][e] = 0.f;
    }
  }
  const size_t cstride = (size_t)N * D;
  for (int pi = 0; pi < np; ++pi) {
    const int n = n0 + pi;
    float wr[HB][4];
    const bf16* wp = w + ((((size_t)b * G + k) * N + n) * heads) * D + d0;
#pragma unroll
    for (int a = 0; a < HB; ++a) {
      bf16x4 wv = {};
      if (a < heads) wv = *reinterpret_cast<const bf16x4*>(wp + (size_t)a * D);
#pragma unroll
      for (int e = 0; e < 4; ++e) wr[a][e] = (float)wv[e];
    }
    const bf16* zp = z + (((size_t)b * Cin + c0) * N + n) * D + d0;
    bf16* dzp = dz + (((size_t)b * Cin + c0) * N + n) * D + d0;
    bf16x4 znext = *reinterpret_cast<const bf16x4*>(zp);
    for (int cl = 0; cl < gk; ++cl) {
      const bf16x4 zv = znext;
      if (cl + 1 < gk) znext = *reinterpret_cast<const bf16x4*>(zp + (size_t)(cl + 1) * cstride);
      const f32x4* ar = reinterpret_cast<const f32x4*>(al + (pi * g + cl) * HB);
      const f32x4* dr = reinterpret_cast<const f32x4*>(dsv + (pi * g + cl) * HB);
      float acc[4] = {0.f, 0.f, 0.f, 0.f};
      float zf[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) zf[e] = (float)zv[e];
#pragma unroll
      for (int q = 0; q < HB / 4; ++q) {
        const f32x4 av = ar[q], dv = dr[q];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            acc[e] += av[a] * wr[q * 4 + a][e] + dv[a] * mr[q * 4 + a][e];
            racc[q * 4 + a][e] += dv[a] * zf[e];
          }
      }
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (bf16)acc[e];
      *reinterpret_cast<bf16x4*>(dzp + (size_t)cl * cstride) = o;
    }
  }
  float* rp = rpart + ((((size_t)b * G + k) * n_tiles + tile) * heads) * D + d0;
#pragma unroll
  for (int a = 0; a < HB; ++a)
    if (a < heads) *reinterpret_cast<f32x4*>(rp + (size_t)a * D) = f32x4{racc[a][0], racc[a][1], racc[a][2], racc[a][3]};
}

// ---------------------------------------------------------------------------------------
// The same two results as two kernels for D % 256 == 0 (bf16, heads <= 32): the token gradients on MFMA
// (reads w, writes dz) and the key-path sums on the vector ALUs (reads z); neither needs the other's stream.
//
// k_dz_mfma:  dz[b, c0 + m, n, :] = [alpha | ds](m, 0..31) . [w ; M](0..31, :)   one 32x32x16 product per 32
// columns, alpha and ds split in two bf16 parts each (hi + lo) so that the fp32 softmax weights lose nothing.
// A wavefront owns 256 columns, lane l the four columns 4 l .. 4 l + 3 of them: it loads the 16 head rows of
// w (per patch) and of M (once) for its columns, packs them into 8-head chunks and swaps one chunk per column
// with lane l ^ 32, which gives both half-wavefronts the B fragments (column, heads 8 (l / 32) ..) of the eight
// 32-column tiles {4 (j + 32 half) + e : j < 32}.  Accumulator block (half, e): lane holds column
// 4 (l % 32 + 32 half) + e, register r member 8 (r / 4) + 4 (l / 32) + r % 4: four blocks give a lane four
// adjacent columns of a member row (one 8-byte store).  The A fragments (member row, 8 heads) come straight
// from the token-major alpha / ds.  grid (n_tiles * ceil(D/1024), G, B), block 256, pt patches per block.
// ---------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(4))) int i32x4;

// B fragments of the eight column tiles from 16 rows (heads) of a [heads][D] bf16 matrix at this lane's 4 columns.
template <bool LAST_USE = false>   // LAST_USE: streaming loads (the rows are not needed in the caches afterwards)
__device__ __forceinline__ void head_row_frags(const bf16* __restrict__ base, int D, int heads, int lhi,
                                               bf16x8 (&frag)[2][4]) {
  bf16x4 rows[16];
#pragma unroll
  for (int a = 0; a < 16; ++a) {
    rows[a] = bf16x4{};
    if (a < heads) {                                               // heads: rows that exist from base on
      const bf16x4* src = reinterpret_cast<const bf16x4*>(base + (size_t)a * D);
      rows[a] = LAST_USE ? __builtin_nontemporal_load(src) : *src;
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    bf16x8 c0, c1;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      c0[i] = rows[i][e];
      c1[i] = rows[8 + i][e];
    }
    const i32x4 v0 = __builtin_bit_cast(i32x4, c0), v1 = __builtin_bit_cast(i32x4, c1);
    i32x4 own, snd, rcv;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      own[q] = lhi ? v1[q] : v0[q];                      // the chunk this half-wavefront multiplies for its own columns
      snd[q] = lhi ? v0[q] : v1[q];                      // the chunk the other half needs for these columns
      rcv[q] = __shfl_xor(snd[q], 32, kWave);
    }
    const bf16x8 o8 = __builtin_bit_cast(bf16x8, own), r8 = __builtin_bit_cast(bf16x8, rcv);
    frag[0][e] = lhi ? r8 : o8;                          // tile of the lower half's columns
    frag[1][e] = lhi ? o8 : r8;                          // tile of the upper half's columns
  }
}

__device__ __forceinline__ void split_bf16(const f32x4& x0, const f32x4& x1, bf16x8& hi, bf16x8& lo) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    hi[i] = (bf16)x0[i];
    lo[i] = (bf16)(x0[i] - (float)hi[i]);
    hi[4 + i] = (bf16)x1[i];
    lo[4 + i] = (bf16)(x1[i] - (float)hi[4 + i]);
  }
}

template <int HB>   // blocks of 16 heads (heads <= 16 HB): the contraction runs over 2 HB steps of 16
__global__ __launch_bounds__(256, 3 - HB) void k_dz_mfma(int Cin, int N, int D, int heads, int g, int n_tiles, int pt,
                                                         const float* __restrict__ alpha, const float* __restrict__ ds,
                                                         const bf16* __restrict__ w, const bf16* __restrict__ Mb,
                                                         bf16* __restrict__ dz) {
  const int tile = blockIdx.x % n_tiles, cb = blockIdx.x / n_tiles;
  const int k = blockIdx.y, b = blockIdx.z, G = gridDim.y;
  const int c0 = k * g, gk = min(g, Cin - c0);
  const int n0 = tile * pt, np = min(pt, N - n0);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, lhi = lane >> 5;
  const int col0 = cb * 1024 + wave * 256;
  if (col0 >= D) return;
  const int d0 = col0 + 4 * lane;
  bf16x8 mfrag[HB][2][4];
#pragma unroll
  for (int hb = 0; hb < HB; ++hb)
    head_row_frags(Mb + ((size_t)k * heads + 16 * hb) * D + d0, D, heads - 16 * hb, lhi, mfrag[hb]);
  const size_t cstride = (size_t)N * D;
  const f32x4 z4 = {0.f, 0.f, 0.f, 0.f};
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const bool h8 = heads % 8 == 0;                        // then a lane's 8 heads are two aligned 16-byte loads
  for (int pi = 0; pi < np; ++pi) {
    const int n = n0 + pi;
    bf16x8 wfrag[HB][2][4];
#pragma unroll
    for (int hb = 0; hb < HB; ++hb)
      head_row_frags(w + ((((size_t)b * G + k) * N + n) * heads + 16 * hb) * D + d0, D, heads - 16 * hb, lhi, wfrag[hb]);
    for (int m0 = 0; m0 < gk; m0 += 32) {
      const int row = m0 + l32;
      bf16x8 ahi[HB], alo[HB], dhi[HB], dlo[HB];
#pragma unroll
      for (int hb = 0; hb < HB; ++hb) {
        const int h0 = 16 * hb + 8 * lhi;                // this lane's 8 heads of the block
        const size_t src = (((size_t)b * Cin + c0 + min(row, gk - 1)) * N + n) * heads + h0;
        f32x4 a0 = z4, a1 = z4, e0 = z4, e1 = z4;
        if (row < gk) {
          if (h8) {
            if (h0 < heads) {
              a0 = *reinterpret_cast<const f32x4*>(alpha + src);
              a1 = *reinterpret_cast<const f32x4*>(alpha + src + 4);
              e0 = *reinterpret_cast<const f32x4*>(ds + src);
              e1 = *reinterpret_cast<const f32x4*>(ds + src + 4);
            }
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              if (h0 + i < heads) { a0[i] = alpha[src + i]; e0[i] = ds[src + i]; }
              if (h0 + 4 + i < heads) { a1[i] = alpha[src + 4 + i]; e1[i] = ds[src + 4 + i]; }
            }
          }
        }
        split_bf16(a0, a1, ahi[hb], alo[hb]);
        split_bf16(e0, e1, dhi[hb], dlo[hb]);
      }
      auto tiles_of_half = [&](int half) {
        f32x16 acc[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc[e] = zero;
#pragma unroll
          for (int hb = 0; hb < HB; ++hb) {
            acc[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ahi[hb], wfrag[hb][half][e], acc[e], 0, 0, 0);
            acc[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(alo[hb], wfrag[hb][half][e], acc[e], 0, 0, 0);
            acc[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dhi[hb], mfrag[hb][half][e], acc[e], 0, 0, 0);
            acc[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dlo[hb], mfrag[hb][half][e], acc[e], 0, 0, 0);
          }
        }
        bf16* dzp = dz + (((size_t)b * Cin + c0) * N + n) * D + col0 + 4 * (l32 + 32 * half);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int m = m0 + 8 * (r >> 2) + 4 * lhi + (r & 3);
          if (m < gk) {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (bf16)acc[e][r];
            *reinterpret_cast<bf16x4*>(dzp + (size_t)m * cstride) = o;
          }
        }
      };
      tiles_of_half(0);
      tiles_of_half(1);
    }
  }
}

// ---------------------------------------------------------------------------------------
// The whole reverse step at the tokens of one level in one kernel (bf16, heads <= 16, D % 256 == 0, D <= 1024 CB,
// group size <= 16 MT <= 32), so that a patch's token rows and its w rows are fetched from HBM once (their second
// use, a few microseconds later in the same workgroup, finds them in L2) and ds never leaves the compute unit:
//   ds as in k_dalpha_softmax_mfma;  rpart[b,k,t][a][:] = sum over the pt patches of tile t and the members c of
//   ds[b,c,n,a] * z[b,c,n,:]  (the partial sums k_sum_partials adds up);  dz as in k_dz_mfma.
// grid (n_tiles, G, B), block 512, PP patches (one) per round of barriers:
//   d alpha   all eight wavefronts, each an eighth of D; the partial 16x16 blocks meet in LDS in a fixed order, the
//             first PP wavefronts apply the Jacobian (one patch each) and leave the softmax weights and ds in LDS;
//   sums      wavefronts 0..3, wavefront w columns 256 w .. 256 w + 255 (of each block of 1024 columns): ds^T (heads x 32 members, split in two
//             bf16 parts) times the 32 member rows on 16x16x32 MFMA; a lane reads 8 members x 8 adjacent columns
//             (16 bytes per row) and transposes them in registers, which gives it the B fragments (column
//             8 (lane % 16) + j, members 8 (lane / 16) ..) of eight products j = 0..7; accumulator (half, j): lane
//             holds column 128 half + 8 (lane % 16) + j, heads 4 (lane / 16) + r;
//   dz        wavefronts 4..7, wavefront 4 + w the same columns: the body of k_dz_mfma, A fragments from LDS.
// The two roles are separate loops (same barriers), so neither carries the other's accumulators.
// ---------------------------------------------------------------------------------------
template <int MT, int CB>   // CB: blocks of 1024 columns (D <= 1024 CB)
__global__ __launch_bounds__(512) void k_tokens_backward_fused(int Cin, int N, int D, int heads, int g, int pt,
                                                               const bf16* __restrict__ z, const bf16* __restrict__ w,
                                                               const float* __restrict__ alpha,
                                                               const bf16* __restrict__ Mb, bf16* __restrict__ dz,
                                                               float* __restrict__ rpart) {
  constexpr int PP = 1;                                            // patches per round of barriers (2: no faster)
  __shared__ f32x4 part[8][PP][MT][64];
  __shared__ float dsv[2][PP][32][17];                             // [round parity][patch][member][head], padded rows
  __shared__ float alv[2][PP][32][17];                             // the softmax weights, same layout
  const int tile = blockIdx.x, n_tiles = gridDim.x, k = blockIdx.y, b = blockIdx.z, G = gridDim.y;
  const int c0 = k * g, gk = min(g, Cin - c0);
  const int n0 = tile * pt, np = min(pt, N - n0);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, lq = lane >> 4, l32 = lane & 31, lhi = lane >> 5;
  const size_t cstride = (size_t)N * D;
  const int kq = D / 8;                                            // this wavefront's share of the contraction
  const int col0 = (wave & 3) * 256;                               // this wavefront's columns of the sums / of dz
  const int head = min(l16, heads - 1);
  const bf16* zg = z + (((size_t)b * Cin + c0) * N + n0) * D;      // member 0 of the group at the tile's first patch
  const size_t item0 = ((size_t)b * G + k) * N + n0;
  for (int i = threadIdx.x; i < 2 * PP * 32 * 17; i += 512) {      // members beyond 16 MT stay zero
    (&dsv[0][0][0][0])[i] = 0.f;
    (&alv[0][0][0][0])[i] = 0.f;
  }
  __syncthreads();

  // partial d alpha of patches pi .. pi + PP - 1 (past the tile's end: its last patch again, never used)
  auto dalpha_partial = [&](int pi) {
    const bf16* wr[PP];
    const bf16* zr[PP][MT];
    f32x4 acc[PP][MT];
#pragma unroll
    for (int q = 0; q < PP; ++q) {
      const int pq = min(pi + q, np - 1);
      wr[q] = w + ((item0 + pq) * heads + head) * D + wave * kq + lq * 8;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        zr[q][mt] = zg + (size_t)pq * D + (size_t)min(mt * 16 + l16, gk - 1) * cstride + wave * kq + lq * 8;
        acc[q][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
    for (int t = 0; t < kq; t += 128) {                            // four steps of 32 per trip, loads first
      bf16x8 wf[PP][4], zf[PP][MT][4];
#pragma unroll
      for (int q = 0; q < PP; ++q)
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
          const int tt = min(t + s4 * 32, kq - 32);
          wf[q][s4] = *reinterpret_cast<const bf16x8*>(wr[q] + tt);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) zf[q][mt][s4] = *reinterpret_cast<const bf16x8*>(zr[q][mt] + tt);
        }
#pragma unroll
      for (int q = 0; q < PP; ++q)
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4)
          if (t + s4 * 32 < kq) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
              acc[q][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zf[q][mt][s4], wf[q][s4], acc[q][mt], 0, 0, 0);
          }
    }
#pragma unroll
    for (int q = 0; q < PP; ++q)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) part[wave][q][mt][lane] = acc[q][mt];
  };
  // Wavefront q < PP applies the Jacobian of patch pi + q.  It fetches the softmax weights of that patch before its
  // share of d alpha, so that they have arrived when the others wait (lane: head l16, members 4 lq + r of each tile).
  auto fetch_alpha = [&](int pi, float (&al)[MT][4]) {
    const int n = n0 + min(pi + wave, np - 1);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int cl = mt * 16 + lq * 4 + r;
        al[mt][r] = (cl < gk && l16 < heads) ? alpha[(((size_t)b * Cin + c0 + cl) * N + n) * heads + l16] : 0.f;
      }
  };
  auto jacobian = [&](int par, const float (&al)[MT][4]) {
    float da[MT][4];
    float dot = 0.f;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      f32x4 tot = part[0][wave][mt][lane];
#pragma unroll
      for (int v = 1; v < 8; ++v) tot += part[v][wave][mt][lane];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        da[mt][r] = tot[r];
        dot += al[mt][r] * tot[r];
      }
    }
    dot += __shfl_xor(dot, 16, kWave);
    dot += __shfl_xor(dot, 32, kWave);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int cl = mt * 16 + lq * 4 + r;
        dsv[par][wave][cl][l16] = al[mt][r] * (da[mt][r] - dot);   // 0 for padding members and heads
        alv[par][wave][cl][l16] = al[mt][r];
      }
  };
  // Per round of PP patches: every wavefront writes its partial blocks, barrier, wavefronts 0 .. PP-1 fill the tables
  // of the round's parity, barrier, the roles read them.  The next round writes the other parity, and `part` only
  // after every wavefront has passed the second barrier of this one.
  if (wave < 4) {
    f32x4 racc[CB][2][8];
#pragma unroll
    for (int cbk = 0; cbk < CB; ++cbk)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 8; ++j) racc[cbk][h][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int pi = 0, par = 0; pi < np; pi += PP, par ^= 1) {
      float al[MT][4];
      if (wave < PP) fetch_alpha(pi, al);
      dalpha_partial(pi);
      __syncthreads();
      if (wave < PP) jacobian(par, al);
      __syncthreads();
      for (int q = 0; q < PP && pi + q < np; ++q) {
        f32x4 v0, v1;                                              // ds of head l16 at members 8 lq .. 8 lq + 7
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          v0[i] = dsv[par][q][8 * lq + i][l16];
          v1[i] = dsv[par][q][8 * lq + 4 + i][l16];
        }
        bf16x8 dhi, dlo;
        split_bf16(v0, v1, dhi, dlo);
#pragma unroll
        for (int cbk = 0; cbk < CB; ++cbk) {
          const int colc = col0 + 1024 * cbk;
          if (colc >= D) continue;
          const bf16* zc = zg + (size_t)(pi + q) * D + colc + 8 * l16;
          constexpr int HL = CB == 1 ? 2 : 1;                      // halves of 128 columns fetched together
#pragma unroll
          for (int h0 = 0; h0 < 2; h0 += HL) {
            bf16x8 rows[HL][8];
#pragma unroll
            for (int h = 0; h < HL; ++h)
#pragma unroll
              for (int i = 0; i < 8; ++i)
                rows[h][i] = __builtin_nontemporal_load(            // second and last use of the row
                    reinterpret_cast<const bf16x8*>(zc + (size_t)min(8 * lq + i, gk - 1) * cstride + 128 * (h0 + h)));
#pragma unroll
            for (int h = 0; h < HL; ++h)
#pragma unroll
              for (int j = 0; j < 8; ++j) {
                bf16x8 col;
#pragma unroll
                for (int i = 0; i < 8; ++i) col[i] = rows[h][i][j];
                racc[cbk][h0 + h][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dhi, col, racc[cbk][h0 + h][j], 0, 0, 0);
                racc[cbk][h0 + h][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dlo, col, racc[cbk][h0 + h][j], 0, 0, 0);
              }
          }
        }
      }
    }
#pragma unroll
    for (int cbk = 0; cbk < CB; ++cbk) {
      const int colc = col0 + 1024 * cbk;
      if (colc >= D) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int a = 4 * lq + r;
        if (a < heads) {
          float* rp = rpart + ((((size_t)b * G + k) * n_tiles + tile) * heads + a) * D + colc + 8 * l16;
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            *reinterpret_cast<f32x4*>(rp + 128 * h) =
                f32x4{racc[cbk][h][0][r], racc[cbk][h][1][r], racc[cbk][h][2][r], racc[cbk][h][3][r]};
            *reinterpret_cast<f32x4*>(rp + 128 * h + 4) =
                f32x4{racc[cbk][h][4][r], racc[cbk][h][5][r], racc[cbk][h][6][r], racc[cbk][h][7][r]};
          }
        }
      }
    }
  } else {
    const int d0c = col0 + 4 * lane;                               // this lane's 4 columns (of each column block)
    bf16x8 mfrag[CB][2][4];
#pragma unroll
    for (int cbk = 0; cbk < CB; ++cbk)
      if (col0 + 1024 * cbk < D)
        head_row_frags(Mb + ((size_t)k * heads) * D + d0c + 1024 * cbk, D, heads, lhi, mfrag[cbk]);
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int pi = 0, par = 0; pi < np; pi += PP, par ^= 1) {
      dalpha_partial(pi);
      __syncthreads();
      __syncthreads();
      for (int q = 0; q < PP && pi + q < np; ++q) {
        f32x4 a0, a1, e0, e1;                                      // member row l32, heads 8 lhi .. 8 lhi + 7
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          a0[i] = alv[par][q][l32][8 * lhi + i];
          a1[i] = alv[par][q][l32][8 * lhi + 4 + i];
          e0[i] = dsv[par][q][l32][8 * lhi + i];
          e1[i] = dsv[par][q][l32][8 * lhi + 4 + i];
        }
        bf16x8 ahi, alo, ehi, elo;
        split_bf16(a0, a1, ahi, alo);
        split_bf16(e0, e1, ehi, elo);
#pragma unroll
        for (int cbk = 0; cbk < CB; ++cbk) {
          const int colc = col0 + 1024 * cbk;
          if (colc >= D) continue;
          bf16x8 wfrag[2][4];
          head_row_frags<true>(w + ((item0 + pi + q) * heads) * D + d0c + 1024 * cbk, D, heads, lhi, wfrag);
          auto tiles_of_half = [&](int half) {
            f32x16 acc[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              acc[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ahi, wfrag[half][e], zero, 0, 0, 0);
              acc[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(alo, wfrag[half][e], acc[e], 0, 0, 0);
              acc[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ehi, mfrag[cbk][half][e], acc[e], 0, 0, 0);
              acc[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(elo, mfrag[cbk][half][e], acc[e], 0, 0, 0);
            }
            bf16* dzp = dz + (((size_t)b * Cin + c0) * N + n0 + pi + q) * D + colc + 4 * (l32 + 32 * half);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const int m = 8 * (r >> 2) + 4 * lhi + (r & 3);
              if (m < gk) {
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (bf16)acc[e][r];
                // streaming store: dz is not read again here, and the rows to come back from L2 are z's and w's
                __builtin_nontemporal_store(o, reinterpret_cast<bf16x4*>(dzp + (size_t)m * cstride));
              }
            }
          };
          tiles_of_half(0);
          tiles_of_half(1);
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// k_rpart_bf16:  rpart[b,k,t][a][:] = sum over the pt patches of tile t and the members c of ds[b,c,n,a] * z[b,c,n,:]
// grid (n_tiles * ceil(D/1024), G, B), block 256: a thread owns 4 adjacent columns and one fp32 sum per head;
// ds of the whole tile sits in LDS (dynamic, pt * g * 16 floats).
// ---------------------------------------------------------------------------------------
template <int HB>   // blocks of 16 heads, heads <= 16 HB
__global__ __launch_bounds__(256) void k_rpart_bf16(int Cin, int N, int D, int heads, int g, int n_tiles, int pt,
                                                    const float* __restrict__ ds, const bf16* __restrict__ z,
                                                    float* __restrict__ rpart) {
  extern __shared__ __attribute__((aligned(16))) float dsv[];      // [np * gk rows in (patch, member) order][16 heads]
  const int tile = blockIdx.x % n_tiles, cb = blockIdx.x / n_tiles;
  const int k = blockIdx.y, b = blockIdx.z, G = gridDim.y;
  const int c0 = k * g, gk = min(g, Cin - c0);
  const int n0 = tile * pt, np = min(pt, N - n0);
  const int rows = np * gk;
  const int d0 = cb * 1024 + threadIdx.x * 4;
#pragma unroll
  for (int hb = 0; hb < HB; ++hb) {                                // more than 16 heads: one pass over z per block of 16
    const int a0 = 16 * hb;
    if (HB > 1) __syncthreads();
    for (int idx = threadIdx.x; idx < rows * 16; idx += 256) {
      const int a = a0 + (idx & 15), cl = (idx >> 4) % gk, pi = (idx >> 4) / gk;
      dsv[idx] = a < heads ? ds[(((size_t)b * Cin + c0 + cl) * N + n0 + pi) * heads + a] : 0.f;
    }
    __syncthreads();
    if (d0 >= D) continue;
    float racc[16][4];
  #pragma unroll
    for (int a = 0; a < 16; ++a)
  #pragma unroll
      for (int e = 0; e < 4; ++e) racc[a][e] = 0.f;
    const size_t cstride = (size_t)N * D;
    const bf16* zb = z + (((size_t)b * Cin + c0) * N + n0) * D + d0;
    // the rows of the tile are walked eight at a time, the next eight already in flight while these are summed
    int pcl = 0, ppi = 0;                                  // (member, patch) of the next row to fetch
    bf16x4 cur[8], nxt[8];
    auto fetch = [&](bf16x4 (&buf)[8]) {
  #pragma unroll
      for (int i = 0; i < 8; ++i) {
        buf[i] = bf16x4{};
        if (ppi < np) buf[i] = *reinterpret_cast<const bf16x4*>(zb + (size_t)ppi * D + (size_t)pcl * cstride);
        if (++pcl == gk) { pcl = 0; ++ppi; }
      }
    };
    fetch(cur);
    for (int base = 0; base < rows; base += 8) {
      fetch(nxt);                                          // past the end: nothing is loaded
  #pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (base + i < rows) {
          const f32x4* dr = reinterpret_cast<const f32x4*>(dsv + (base + i) * 16);
  #pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 dv = dr[q];
  #pragma unroll
            for (int a = 0; a < 4; ++a)
  #pragma unroll
              for (int e = 0; e < 4; ++e) racc[q * 4 + a][e] += dv[a] * (float)cur[i][e];
          }
        }
      }
  #pragma unroll
      for (int i = 0; i < 8; ++i) cur[i] = nxt[i];
    }
    float* rp = rpart + ((((size_t)b * G + k) * n_tiles + tile) * heads + a0) * D + d0;
  #pragma unroll
    for (int a = 0; a < 16; ++a)
      if (a0 + a < heads) *reinterpret_cast<f32x4*>(rp + (size_t)a * D) = f32x4{racc[a][0], racc[a][1], racc[a][2], racc[a][3]};
  }
}

// ---------------------------------------------------------------------------------------
// k_rpart_mfma: the same partial sums on 16x16x32 MFMA for D % 256 == 0 (bf16, heads <= 16 HB), as in
// k_tokens_backward_fused: per patch and block of 32 members, ds^T (16 heads x 32 members, hi + lo bf16 parts) times
// the 32 member rows; a lane reads 8 members x 8 adjacent columns and transposes them in registers.
// grid (n_tiles * ceil(D/1024), G, B), block 256: wavefront w owns columns 1024 cb + 256 w .. + 255.  ds of the whole
// tile sits in LDS (dynamic, pt * g * 16 HB floats, rows in (patch, member) order).
// ---------------------------------------------------------------------------------------
template <int HB>
__global__ __launch_bounds__(256, 2) void k_rpart_mfma(int Cin, int N, int D, int heads, int g, int n_tiles, int pt,
                                                       const float* __restrict__ ds, const bf16* __restrict__ z,
                                                       float* __restrict__ rpart) {
  extern __shared__ __attribute__((aligned(16))) float dsv[];      // [np * gk rows][16 HB heads]
  constexpr int HP = 16 * HB;
  const int tile = blockIdx.x % n_tiles, cb = blockIdx.x / n_tiles;
  const int k = blockIdx.y, b = blockIdx.z, G = gridDim.y;
  const int c0 = k * g, gk = min(g, Cin - c0);
  const int n0 = tile * pt, np = min(pt, N - n0);
  const int rows = np * gk;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, lq = lane >> 4;
  const int col0 = cb * 1024 + wave * 256;
  for (int idx = threadIdx.x; idx < rows * HP; idx += 256) {
    const int a = idx % HP, cl = (idx / HP) % gk, pi = (idx / HP) / gk;
    dsv[idx] = a < heads ? ds[(((size_t)b * Cin + c0 + cl) * N + n0 + pi) * heads + a] : 0.f;
  }
  __syncthreads();
  if (col0 >= D) return;
  f32x4 racc[HB][2][8];
#pragma unroll
  for (int hb = 0; hb < HB; ++hb)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < 8; ++j) racc[hb][h][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const size_t cstride = (size_t)N * D;
  const bf16* zb = z + (((size_t)b * Cin + c0) * N + n0) * D + col0 + 8 * l16;
  for (int pi = 0; pi < np; ++pi)
    for (int m0 = 0; m0 < gk; m0 += 32) {                          // members m0 + 8 lq .. + 7 are this lane's
      bf16x8 dhi[HB], dlo[HB];
#pragma unroll
      for (int hb = 0; hb < HB; ++hb) {
        f32x4 v0, v1;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int cl = m0 + 8 * lq + i;
          const float v = cl < gk ? dsv[(pi * gk + cl) * HP + 16 * hb + l16] : 0.f;
          if (i < 4) v0[i] = v; else v1[i - 4] = v;
        }
        split_bf16(v0, v1, dhi[hb], dlo[hb]);
      }
      bf16x8 zr[2][8];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < 8; ++i)
          zr[h][i] = *reinterpret_cast<const bf16x8*>(zb + (size_t)pi * D + (size_t)min(m0 + 8 * lq + i, gk - 1) * cstride +
                                                     128 * h);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          bf16x8 col;
#pragma unroll
          for (int i = 0; i < 8; ++i) col[i] = zr[h][i][j];
#pragma unroll
          for (int hb = 0; hb < HB; ++hb) {
            racc[hb][h][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dhi[hb], col, racc[hb][h][j], 0, 0, 0);
            racc[hb][h][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dlo[hb], col, racc[hb][h][j], 0, 0, 0);
          }
        }
    }
#pragma unroll
  for (int hb = 0; hb < HB; ++hb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int a = 16 * hb + 4 * lq + r;
      if (a < heads) {
        float* rp = rpart + ((((size_t)b * G + k) * n_tiles + tile) * heads + a) * D + col0 + 8 * l16;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          *reinterpret_cast<f32x4*>(rp + 128 * h) =
              f32x4{racc[hb][h][0][r], racc[hb][h][1][r], racc[hb][h][2][r], racc[hb][h][3][r]};
          *reinterpret_cast<f32x4*>(rp + 128 * h + 4) =
              f32x4{racc[hb][h][4][r], racc[hb][h][5][r], racc[hb][h][6][r], racc[hb][h][7][r]};
        }
      }
    }
}

// r[k][i] = sum_b sum_t rpart[b][k][t][i]   (i over heads * D), fixed order.  grid (ceil(per/64), G), block 1024:
// 64 adjacent i per block, the sixteen wavefronts take every sixteenth partial (four in flight each) and meet in LDS.
__global__ __launch_bounds__(1024) void k_sum_partials(int B, int G, int n_tiles, long per, const float* __restrict__ rpart,
                                                       float* __restrict__ r) {
  __shared__ float part[15][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long i = (long)blockIdx.x * 64 + lane;
  const int k = blockIdx.y;
  float acc = 0.f;
  if (i < per)
    for (int b = 0; b < B; ++b) {
      const float* src = rpart + (((size_t)b * G + k) * n_tiles) * per + i;
      int t = wave;
      for (; t + 48 < n_tiles; t += 64) {
        const float v0 = src[(size_t)t * per], v1 = src[(size_t)(t + 16) * per], v2 = src[(size_t)(t + 32) * per],
                    v3 = src[(size_t)(t + 48) * per];
        acc += v0;
        acc += v1;
        acc += v2;
        acc += v3;
      }
      for (; t < n_tiles; t += 16) acc += src[(size_t)t * per];
    }
  if (wave > 0) part[wave - 1][lane] = acc;
  __syncthreads();
  if (wave == 0 && i < per) {
#pragma unroll
    for (int w = 0; w < 15; ++w) acc += part[w][lane];
    r[(size_t)k * per + i] = acc;
  }
}

}  // namespace dchag
