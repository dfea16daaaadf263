// refine64.hpp - fp32 validation mode: the refined keys' cross-attention
// logits in fp64.
//
// With QK-norm the logits are d_l * cos(q, k) (App. A, cross-attention), so a
// relative rounding of 1e-7 in q~ or k~ moves the heaviest keys' weights by
// about d_l * 1e-7 ~ 1e-4, the size of the fp32 mode's whole error budget.
// The flash pass therefore keeps its fp32 logits for the bulk of the keys,
// and for the refined keys (those carrying nearly all of a latent's mass)
// the logit is recomputed from the fp32 inputs with every step in fp64:
//   q = RoPE_c(l2n(RMSNorm(Z) W_Q^T + b_Q), p_q)      dgemm + q64_finalize
//   k = RoPE_c(l2n(X_n W_K^T + b_K), p_n),  X_n = [R(-p_n) K_n ; V_n]
//   logit = s * log2(e) * q . k                          refine64
// The result is handed to the merge as the difference to the logit the flash
// pass used, so the weight swap 2^(fp32 logit - M) -> 2^(exact - M) keeps
// full precision (the logits themselves are ~1e3 in log2 units).
#pragma once
#include "common.hpp"

namespace still {

// inv_freq[j] = base^(-2j / w), j < w/2 (the RoPE frequencies of width w)
static __global__ void inv_freq64_kernel(double base, int w, double* __restrict__ out) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j < w / 2) out[j] = pow(base, -2.0 * (double)j / (double)w);
}

// In place: each (row, head c) slice of width dc of Q, holding Z W_Q^T (fp64
// products and sums of the fp32 Z and W_Q, dgemm_kernel), becomes
// RoPE_c(q~ / max(||q~||, eps)) at the row's latent position, with
// q~ = r Z W_Q^T + b and r the row's RMS factor, formed here in fp64.  One
// wave per slice.
static __global__ __launch_bounds__(256) void q64_finalize_kernel(double* __restrict__ Q, const float* __restrict__ Z,
                                                           const float* __restrict__ bias, long rows, int nc, int dc,
                                                           int D, int t, const double* __restrict__ pq,
                                                           const double* __restrict__ invf, double rms_eps,
                                                           double l2_eps) {
  const long s = blockIdx.x * 4L + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (s >= rows * nc) return;
  const long row = s / nc;
  const int c = (int)(s - row * nc);
  double* q = Q + row * ((long)nc * dc) + (long)c * dc;
  const float* z = Z + row * D;
  double zz = 0.0;
  for (int k = lane; k < D; k += 64) zz = fma((double)z[k], (double)z[k], zz);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) zz += __shfl_xor(zz, o);
  const double rms = 1.0 / sqrt(zz / (double)D + rms_eps);
  auto qt = [&](int j) -> double { return fma(rms, q[j], bias ? (double)bias[(long)c * dc + j] : 0.0); };
  double ss = 0.0;
  for (int j = lane; j < dc; j += 64) {
    const double v = qt(j);
    ss = fma(v, v, ss);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  const double inv = 1.0 / fmax(sqrt(ss), l2_eps);
  const double p = pq[row % t];
  const int hh = dc / 2;
  for (int j = lane; j < hh; j += 64) {
    double sn, cs;
    sincos(p * invf[j], &sn, &cs);
    const double a = qt(j) * inv, b = qt(j + hh) * inv;
    q[j] = a * cs - b * sn;
    q[j + hh] = b * cs + a * sn;
  }
}

struct Refine64Args {
  const float* K;        // [H][N][d] RoPE'd keys
  const float* V;        // [H][N][d] values
  const double* pos;     // [N] key positions
  const double* invf_b;  // [d/2] base-model RoPE frequencies
  const double* invf_c;  // [dc/2] compactor RoPE frequencies
  const float* W;        // [nc*dc][2d] W_K
  const float* bias;     // [nc*dc] b_K or NULL
  const double* Q;       // [H*t][nc*dc] normalised, rotated q (q64_finalize)
  const int* ridx;       // [H*nc][t*R] key of each slot
  const float* rval;     // [H*nc][t*R] fp32 logit of the flash pass (log2 units)
  const int* crow;       // [H*nc][t*R] compacted list: row -> slot
  const int* count;      // [H*nc]
  float2* rpart;         // [H*nc][t*R]: .x = exact logit - fp32 logit
  long N;
  int H, t, R, nc, dc, d;
  double scale_log2, l2_eps;
  int ntile;             // row tiles of BM per list in the grid (workgroups loop past it)
};

// Workgroup = BM candidate rows of one (h, c) list (32, or 16 at D = 256 where
// the fp64 rows fill the LDS).  Their X rows are built in fp64 in LDS (base
// RoPE un-rotation with fp64 angles); the key projection runs on the fp64
// matrix instructions (lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16]
// of a 16 x 4 and a 4 x 16 step, and holds C[l / 16 + 4 v][l % 16] in register
// pair v), wave w taking every fourth chunk of 16 RoPE pairs.  The pairing of
// contraction indices is free: in a block of 16, lane group l / 16 takes
// indices 4 (l / 16) + s at step s, so that W_K streams as 16-byte loads from
// L2 and X as 16-byte LDS reads, with no staging and no barrier in the loop.
// The epilogue of a chunk adds the bias and accumulates the sum of squares and
// the dot product of the rotated key with q.  It is bound by the matrix pipe
// (16 instructions of 64 cycles per block of 16 indices and 32 rows); 4096
// keys, 256 latents, 8 x 8 heads of width 1024: 2.28 ms with fp64 FMAs from
// W_K staged in LDS, 0.50 ms now.
template <int D>
__global__ __launch_bounds__(256) void refine64_kernel(Refine64Args a) {
  constexpr int BM = D > 128 ? 16 : 32, MT = BM / 16, D2 = 2 * D, LX = D2 + 2;
  typedef double f64x4_t __attribute__((ext_vector_type(4)));
  typedef double f64x2_t __attribute__((ext_vector_type(2)));
  __shared__ __attribute__((aligned(16))) double Xs[BM][LX];
  __shared__ double sdot[4][BM], sss[4][BM];
  __shared__ int2 rinfo[BM];   // (key, latent)
  __shared__ int rslot[BM];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int nb = a.H * a.nc;
  const int b = blockIdx.x % nb, rt0 = blockIdx.x / nb;
  const int h = b / a.nc, c = b - h * a.nc;
  const int cnt = a.count[b];
  const int TR = a.t * a.R;
  const int hh = a.dc / 2, hd = D / 2;
  const long Ec = (long)a.nc * a.dc;
  for (int rt = rt0; rt * BM < cnt; rt += a.ntile) {
    const int r0 = rt * BM;
    __syncthreads();   // previous tile's LDS reads done
    if (tid < BM) {
      int key = 0, lat = 0, slot = -1;
      if (r0 + tid < cnt) {
        slot = a.crow[(long)b * TR + r0 + tid];
        key = max(a.ridx[(long)b * TR + slot], 0);
        lat = slot / a.R;
      }
      rinfo[tid] = make_int2(key, lat);
      rslot[tid] = slot;
    }
    __syncthreads();
    // X rows: [R(-p) K ; V] in fp64
    for (int e = tid; e < BM * hd; e += 256) {
      const int rr = e / hd, j = e - rr * hd;
      const long n = rinfo[rr].x;
      const float* kr = a.K + ((long)h * a.N + n) * D;
      const float* vr = a.V + ((long)h * a.N + n) * D;
      double sn, cs;
      sincos(a.pos[n] * a.invf_b[j], &sn, &cs);
      const double k0 = kr[j], k1 = kr[j + hd];
      Xs[rr][j] = k0 * cs + k1 * sn;
      Xs[rr][j + hd] = k1 * cs - k0 * sn;
      Xs[rr][D + j] = vr[j];
      Xs[rr][D + j + hd] = vr[j + hd];
    }
    __syncthreads();
    // this lane's candidates: rows 16 m + lk + 4 v
    double dot[MT][4], ss[MT][4];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int v = 0; v < 4; ++v) dot[m][v] = ss[m][v] = 0.0;
    for (int p0 = 16 * w; p0 < hh; p0 += 64) {   // dc is a multiple of 128: whole chunks
      const int j = p0 + li;                      // this lane's pair
      const float* w0 = a.W + ((long)c * a.dc + j) * D2 + 4 * lk;
      const float* w1 = w0 + (long)hh * D2;
      f64x4_t acc[MT][2];
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int u = 0; u < 2; ++u) acc[m][u] = f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
      for (int k0 = 0; k0 < D2; k0 += 16) {
        const f32x4 b0 = *(const f32x4*)(w0 + k0), b1 = *(const f32x4*)(w1 + k0);
        double x[MT][4];
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          const f64x2_t* xp = (const f64x2_t*)&Xs[16 * m + li][k0 + 4 * lk];
          const f64x2_t x0 = xp[0], x1 = xp[1];
          x[m][0] = x0.x;
          x[m][1] = x0.y;
          x[m][2] = x1.x;
          x[m][3] = x1.y;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int m = 0; m < MT; ++m) {
            acc[m][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[m][s], (double)b0[s], acc[m][0], 0, 0, 0);
            acc[m][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[m][s], (double)b1[s], acc[m][1], 0, 0, 0);
          }
      }
      const double bias0 = a.bias ? (double)a.bias[(long)c * a.dc + j] : 0.0;
      const double bias1 = a.bias ? (double)a.bias[(long)c * a.dc + j + hh] : 0.0;
      const double invf = a.invf_c[j];
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int2 ri = rinfo[16 * m + lk + 4 * v];
          const double* qrow = a.Q + ((long)h * a.t + ri.y) * Ec + (long)c * a.dc;
          const double v0 = acc[m][0][v] + bias0, v1 = acc[m][1][v] + bias1;
          ss[m][v] = fma(v0, v0, fma(v1, v1, ss[m][v]));
          double sn, cs;
          sincos(a.pos[ri.x] * invf, &sn, &cs);
          dot[m][v] += (v0 * cs - v1 * sn) * qrow[j] + (v1 * cs + v0 * sn) * qrow[j + hh];
        }
    }
    // over the 16 lanes (pairs) of a group, then over the waves
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) {
          dot[m][v] += __shfl_xor(dot[m][v], o);
          ss[m][v] += __shfl_xor(ss[m][v], o);
        }
        if (li == 0) {
          sdot[w][16 * m + lk + 4 * v] = dot[m][v];
          sss[w][16 * m + lk + 4 * v] = ss[m][v];
        }
      }
    __syncthreads();
    if (tid < BM && rslot[tid] >= 0) {
      const double d = (sdot[0][tid] + sdot[1][tid]) + (sdot[2][tid] + sdot[3][tid]);
      const double q = (sss[0][tid] + sss[1][tid]) + (sss[2][tid] + sss[3][tid]);
      const long sl = (long)b * TR + rslot[tid];
      const double logit = a.scale_log2 * d / fmax(sqrt(q), a.l2_eps);
      a.rpart[sl] = make_float2((float)(logit - (double)a.rval[sl]), 0.f);
    }
  }
}

}  // namespace still
