// attn.hpp - flash-style latent -> cache cross-attention (one KV head h, one
// cross head c per grid row), split over the key axis.
//
// For a tile of TT latents and a key range, stream key blocks of NB keys:
//   S^T = K_blk Q^T              (contraction over the head width, MFMA)
//   logits = S^T * rk[key] * rq[lat] * s * log2(e)   (QK-norm folded in)
//   online softmax over keys (running max m, running sum l per latent)
//   O^T += X_blk^T P^T           (contraction over the block's keys, MFMA)
// and write the un-normalised partial (O, m, l) of the key range.  The value
// projection W_V is applied afterwards to the merged O = P X (exact
// re-association of P (X W_V)).
//
// Orientation: keys are MFMA rows and latents MFMA columns in the first
// product, so every lane owns one latent and the softmax statistics stay in
// the lane; the S^T accumulator is then already a valid B operand of the
// second product once the block's keys are read from X^T in the matching
// (permuted) order.
#pragma once
#include <type_traits>

#include "common.hpp"

namespace still {

struct AttnArgs {
  const void* q;     // [H*t][nc*dc]  rotated, un-normalised queries (CT)
  long ldq;
  const float* rq;   // [H*t][nc]     1 / max(||q~||, eps)
  const void* k;     // rotated, un-normalised keys (CT): fp32 kernel [H*N][nc*dc] (row stride ldk),
  long ldk;          //   fp16 kernel the fragment-tiled layout (ktile_off) with npad keys per head
  const float* rk;   // [H*N][nc]
  const void* xt;    // X^T (CT), zero beyond N: fp32 kernel [H][2d][ldxt], fp16 kernel tiled (xtile_off)
  long ldxt;
  long npad;         // fp16 kernel: keys per head in the tiled layouts (a multiple of 256)
  long xfeat, xcoff; // fp16 kernel: features per KV head in the tiled values and the first
                     //   feature of head c at c * xcoff (cross-attention: 2d and 0, every head
                     //   reads all of X; self-attention: n_s * d_s and d_s, one value slice per head)
  float* opart;      // [S][H*nc][t][2d]
  float* mpart;      // [S][H*nc][t]
  float* lpart;      // [S][H*nc][t]
  int H, N, t, nc, dc, d2;
  float scale_log2;  // logit scale * log2(e)
  int keys_per_split;
  // candidates of the logit refinement
  float* cval;       // fp32 kernel: [S][H*nc][t][ncand] largest logits seen (log2 units) ...
  int* cidx;         // ... and their key indices (-1 = none): 2 TOPK list entries (one list per
                     // lane half), then up to ATT_OVF overflow entries
  float2* cand;      // fp16 kernel: [S][H*nc][t][XATT_NBK][ccap] (logit, key index as bits)
  int ccap;          // XATT_CAP or XATT_CAP_SPLIT
  int* ocnt;         // fp32 kernel: [S][H*nc][t] overflow entries; fp16 kernel: [S][H*nc][t][XATT_NBK] entries
};

// Capacity of the candidate lists per (split, latent row).  Keys enter while
// they are within the margin of the running maximum, so early blocks can add
// keys that a later, larger maximum leaves outside the margin; the capacity is
// sized for that (a cache of 32-fold duplicated rows writes several hundred
// entries to some rows).
// fp32 kernel: overflow entries, in-margin keys that a full register list
// rejects or evicts.
constexpr int ATT_OVF = 1536;
// (The fp16 kernel's lists: common.hpp.)

template <class CT, int TT, int NB, int DK, int D2, int TOPK>
__global__ __launch_bounds__(256) void cross_attn_kernel(AttnArgs a) {
  typedef Mma<CT> MM;
  typedef typename MM::frag frag;
  constexpr int E = MM::E;
  static_assert(E == 4, "fp32 operands");
  constexpr int PAD = 16 / sizeof(CT);
  constexpr int LQ = DK + PAD;           // Q/K stage row stride
  constexpr int LX = NB + PAD;           // X^T block row stride
  constexpr int KT = NB / 32;            // key tiles per block
  constexpr int FT = D2 / 32;            // feature tiles
  constexpr int QV = TT * DK / E / 256;  // stage vectors per thread
  constexpr int KVv = NB * DK / E / 256;
  constexpr int XV = D2 * NB / E / 256;
  static_assert(TT == 128, "4 waves x 32 latents");
  static_assert(QV >= 1 && KVv >= 1 && XV >= 1, "tile sizes");

  __shared__ __attribute__((aligned(16))) CT Qs[2][TT * LQ];
  __shared__ __attribute__((aligned(16))) CT Ks[2][NB * LQ];
  __shared__ __attribute__((aligned(16))) CT Xs[D2 * LX];
  __shared__ float rks[NB];
  __shared__ int ovn[TT];   // overflow entries of each latent row

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, lg = lane >> 5;
  const int hc = blockIdx.y, h = hc / a.nc, c = hc - h * a.nc;
  const int t0 = blockIdx.x * TT;
  const int split = blockIdx.z;
  const int nbeg = split * a.keys_per_split;
  const int nend = min(a.N, nbeg + a.keys_per_split);

  const CT* qbase = (const CT*)a.q + (long)h * a.t * a.ldq + (long)c * a.dc;
  const CT* kbase = (const CT*)a.k + (long)h * a.N * a.ldk + (long)c * a.dc;
  const CT* xtb = (const CT*)a.xt + (long)h * a.d2 * a.ldxt;
  const float* rkb = a.rk + (long)h * a.N * a.nc + c;

  const int my_lat = t0 + wave * 32 + l32;
  const float rq = my_lat < a.t ? a.rq[((long)h * a.t + my_lat) * a.nc + c] : 0.f;
  const float qscale = rq * a.scale_log2;
  if (tid < TT) ovn[tid] = 0;   // read after the first block's barriers
  constexpr int NCAND = 2 * (TOPK > 0 ? TOPK : 1) + ATT_OVF;   // list entries per (split, row)
  const long crow_ = ((long)split * a.H * a.nc + hc) * a.t + my_lat;

  f32x16 o[FT];
#pragma unroll
  for (int f = 0; f < FT; ++f) o[f] = zero16();
  float m_run = -INFINITY, l_run = 0.f;
  // top-TOPK keys of this lane's half of the key range, by logit (descending)
  float tv[TOPK > 0 ? TOPK : 1];
  int ti[TOPK > 0 ? TOPK : 1];
#pragma unroll
  for (int q = 0; q < (TOPK > 0 ? TOPK : 1); ++q) {
    tv[q] = -INFINITY;
    ti[q] = -1;
  }

  frag rq_[QV], rk_[KVv], rx[XV];
  auto load_qk = [&](int n0, int d0) {
#pragma unroll
    for (int i = 0; i < QV; ++i) {
      const int v = tid + i * 256, r = v / (DK / E), kk = (v % (DK / E)) * E;
      const int lat = t0 + r;
      rq_[i] = lat < a.t ? *(const frag*)(qbase + (long)lat * a.ldq + d0 + kk) : zero_frag<CT>();
    }
#pragma unroll
    for (int i = 0; i < KVv; ++i) {
      const int v = tid + i * 256, r = v / (DK / E), kk = (v % (DK / E)) * E;
      const int n = n0 + r;
      rk_[i] = n < nend ? *(const frag*)(kbase + (long)n * a.ldk + d0 + kk) : zero_frag<CT>();
    }
  };
  auto store_qk = [&](int buf) {
#pragma unroll
    for (int i = 0; i < QV; ++i) {
      const int v = tid + i * 256, r = v / (DK / E), kk = (v % (DK / E)) * E;
      *(frag*)&Qs[buf][r * LQ + kk] = rq_[i];
    }
#pragma unroll
    for (int i = 0; i < KVv; ++i) {
      const int v = tid + i * 256, r = v / (DK / E), kk = (v % (DK / E)) * E;
      *(frag*)&Ks[buf][r * LQ + kk] = rk_[i];
    }
  };
  auto load_x = [&](int n0) {
#pragma unroll
    for (int i = 0; i < XV; ++i) {
      const int v = tid + i * 256, f = v / (NB / E), kk = (v % (NB / E)) * E;
      rx[i] = *(const frag*)(xtb + (long)f * a.ldxt + n0 + kk);   // padded: always in bounds
    }
  };

  const int nd = a.dc / DK;
  for (int n0 = nbeg; n0 < nend; n0 += NB) {
    // ---- S^T = K_blk Q^T over the head width
    f32x16 s[KT];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) s[kt] = zero16();
    load_x(n0);
    load_qk(n0, 0);
    store_qk(0);
    __syncthreads();
    for (int di = 0; di < nd; ++di) {
      const int cur = di & 1;
      if (di + 1 < nd) load_qk(n0, (di + 1) * DK);
#pragma unroll
      for (int ks = 0; ks < DK / (2 * E); ++ks) {
        const frag bq = *(const frag*)&Qs[cur][(wave * 32 + l32) * LQ + ks * 2 * E + lg * E];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
          const frag ak = *(const frag*)&Ks[cur][(kt * 32 + l32) * LQ + ks * 2 * E + lg * E];
          MM::mma(s[kt], ak, bq);
        }
      }
      if (di + 1 < nd) store_qk(cur ^ 1);
      __syncthreads();
    }
    // ---- stage X^T block and the key norms
#pragma unroll
    for (int i = 0; i < XV; ++i) {
      const int v = tid + i * 256, f = v / (NB / E), kk = (v % (NB / E)) * E;
      *(frag*)&Xs[f * LX + kk] = rx[i];
    }
    if (tid < NB) {
      const int n = n0 + tid;
      rks[tid] = n < nend ? rkb[(long)n * a.nc] : 0.f;
    }
    __syncthreads();

    // ---- online softmax (lane owns latent my_lat; keys in registers)
    float mx = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int kl = kt * 32 + 8 * (j >> 2) + 4 * lg + (j & 3);
        float x = s[kt][j] * rks[kl] * qscale;
        x = (n0 + kl < nend) ? x : -INFINITY;
        s[kt][j] = x;
        mx = fmaxf(mx, x);
        if constexpr (TOPK > 0) {
          // keys within REFINE_MARGIN of the running maximum enter the lane's
          // sorted list; the entry a full list pushes out, or the key itself
          // when it does not enter, goes to the row's overflow list if it is
          // still in the margin (padding rows past t take none)
          const float cut = fmaxf(m_run, mx) - REFINE_MARGIN;
          if (x > cut && my_lat < a.t) {
            auto overflow = [&](float ov, int ok) {
              const int slot = atomicAdd(&ovn[wave * 32 + l32], 1);
              if (slot < ATT_OVF) {
                a.cval[crow_ * NCAND + 2 * TOPK + slot] = ov;
                a.cidx[crow_ * NCAND + 2 * TOPK + slot] = ok;
              }
            };
            if (x > tv[TOPK - 1]) {
              const float ev = tv[TOPK - 1];
              const int ek = ti[TOPK - 1];
              float v = x;
              int id = n0 + kl;
              bool moved = false;   // entries after the insertion point shift (exact ties too)
#pragma unroll
              for (int q = 0; q < TOPK; ++q) {
                const bool gt = moved || v > tv[q];
                const float tvq = tv[q];
                const int tiq = ti[q];
                tv[q] = gt ? v : tvq;
                ti[q] = gt ? id : tiq;
                v = gt ? tvq : v;
                id = gt ? tiq : id;
                moved = gt;
              }
              if (ek >= 0 && ev > cut) overflow(ev, ek);
            } else {
              overflow(x, n0 + kl);
            }
          }
        }
      }
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float m_new = fmaxf(m_run, mx);
    const float alpha = (m_new == -INFINITY) ? 1.f : exp2f(m_run - m_new);
    float psum = 0.f;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const float p = (m_new == -INFINITY) ? 0.f : exp2f(s[kt][j] - m_new);
        s[kt][j] = p;
        psum += p;
      }
    psum += __shfl_xor(psum, 32);
    l_run = l_run * alpha + psum;
    m_run = m_new;
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
      for (int j = 0; j < 16; ++j) o[f][j] *= alpha;

    // ---- O^T += X^T P^T
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        frag bp;
#pragma unroll
        for (int e = 0; e < 4; ++e) bp[e] = s[kt][4 * qd + e];
        const int key0 = kt * 32 + 8 * qd + 4 * lg;     // keys key0..+3
#pragma unroll
        for (int f = 0; f < FT; ++f) {
          const frag ax = *(const frag*)&Xs[(f * 32 + l32) * LX + key0];
          MM::mma(o[f], ax, bp);
        }
      }
    }
  }

  // ---- write the partial (O un-normalised, m, l) of this key range
  if (my_lat < a.t) {
    const long row = ((long)split * a.H * a.nc + hc) * a.t + my_lat;
    float* op = a.opart + row * a.d2;
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
      for (int j = 0; j < 16; ++j) op[f * 32 + 8 * (j >> 2) + 4 * lg + (j & 3)] = o[f][j];
    if (lg == 0) {
      a.mpart[row] = m_run;
      a.lpart[row] = l_run;
    }
    if constexpr (TOPK > 0) {
#pragma unroll
      for (int q = 0; q < TOPK; ++q) {
        a.cval[row * NCAND + lg * TOPK + q] = tv[q];
        a.cidx[row * NCAND + lg * TOPK + q] = ti[q];
      }
      if (lg == 0) a.ocnt[row] = min(ovn[wave * 32 + l32], ATT_OVF);
    }
  }
}

}  // namespace still

namespace still {

// ---------------------------------------------------------------------------
// fp16 cross-attention.  Workgroup = TT latents x one key range of one
// (KV head, cross head) pair; 4 waves, one per SIMD (512 registers each).
// Key blocks of KB = 128 KT keys; wave w owns keys [32 KT w, 32 KT (w + 1))
// of a block in the QK product (32 KT keys x TT latents per wave) and output
// features [w D2 / 4, (w + 1) D2 / 4) in the P.X product.
//
// What bounds it is the delivery of MFMA operands into the CU, so the tile is
// as large as the register file allows: the logit and the output accumulators
// together fill 384 of a lane's 512 registers, half of the logits (KT = 4) or
// all of them (KT = 2) in vector registers, the rest in accumulation registers.
// One layer, 8 x 8 heads, 8192 keys x 1024 latents of width 1024 (D2 = 256):
// 1.62 ms with 256-key blocks and compiler-placed accumulators, 1.50 now (916
// TFLOP/s); 9216 keys of width 2048 (D2 = 512): 4.32 ms with 64-latent tiles,
// 3.20 now (966).  Listing the candidates costs 0.12 ms of the 1.50; with every
// operand in the CU's L1 it would run at 1.24 PFLOP/s.
//   D2 = 256: 128 latents x 512 keys (KT = 4);  D2 = 512: 128 x 256 (KT = 2);
//   up to 64 latents in all: 64 x 512.
//   QK: S^T[key][lat] over the head width, in chunks of QC = 64 (one barrier
//       per chunk).  Q chunks are copied straight from global memory into a
//       ring of four LDS stages (direct loads, issued three chunks ahead of
//       use), and each step's Q fragments are read one step ahead of the
//       MFMAs that use them.  K fragments come from the tiled layout straight
//       into a ring of KR steps of registers: a fragment is reloaded as soon
//       as its MFMAs are issued (the next block's first steps are loaded over the
//       last P.X steps of a block).
//   softmax: logit (log2 units) = S * rk[key] * qs[lat] with qs = rq * scale
//       * log2(e) (the query side of the QK-norm and the logit scale: one
//       factor per lane and latent tile); per-latent block maxima combined
//       over the 4 waves through LDS; P (fp16) to LDS [lat][key], 256 keys
//       (64 of every wave) at a time.
//   P.X: O^T[feat][lat] += X^T[feat][key] P^T[key][lat]; X^T fragments from
//       the tiled layout through a ring of XR key steps, P from LDS.
// Keys past the range end (only in its last block) are masked by an additive
// -inf: their tiled k slots must hold finite values (the launches zero them,
// zero_ktile_tail_kernel).  A block may reach past the npad keys of the tiled
// layouts (multiples of 256): its tile indices are clamped to the last tile,
// whose values are finite and whose weights are masked.  The grid is 1-D,
// ordered so that the t tiles of one (pair, split) are consecutive workgroups
// of one XCD and read the same keys through its L2.
// ---------------------------------------------------------------------------

// Accumulators kept in accumulation registers named outright: tile T is
// a[16 T .. 16 T + 15].  Left to the compiler, 384 accumulator registers do not
// fit: it moves whole tiles through scratch memory.  The kernel's own values
// stay in the vector registers (the build fails if the compiler uses an
// accumulation register there, build.py), so nothing but these statements
// touches them; being volatile they keep their order.  Where the vector
// registers do not suffice the compiler spills to scratch memory, inside the
// loop over key blocks: about 28 registers at 128 latents x 512 keys, one or two
// at 128 x 256 x 512 features with candidates, none elsewhere
// (tests/test_attn_registers.py).  These transfers count as memory operations in
// the waits below, which then wait for more than they need, never for less.
// The compiler looks for no hazards in inline assembly: the s_nop in front
// covers operands that a vector instruction wrote just before, acc_settle()
// goes between the last MFMA or accumulator write and the first read of
// another kind.
template <int T> __device__ __forceinline__ void acc_mfma(const half8& a, const half8& b) {
  asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_f16 a[%2:%3], %0, %1, a[%2:%3]" ::"v"(a), "v"(b), "n"(16 * T), "n"(16 * T + 15));
}
template <int T> __device__ __forceinline__ void acc_mfma_first(const half8& a, const half8& b) {   // on zero
  asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_f16 a[%2:%3], %0, %1, 0" ::"v"(a), "v"(b), "n"(16 * T), "n"(16 * T + 15));
}
template <int R> __device__ __forceinline__ float acc_read() {
  float x;
  asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(x) : "n"(R));
  return x;
}
template <int R> __device__ __forceinline__ void acc_write(float x) {
  asm volatile("s_nop 1\n\tv_accvgpr_write_b32 a[%0], %1" ::"n"(R), "v"(x));
}
__device__ __forceinline__ void acc_settle() { asm volatile("s_nop 15\n\ts_nop 15"); }
// No value of the compiler's lives in an accumulation register across this
// point: called in every loop and pass over the accumulators.
#define STILL_A10(d) "a" #d "0", "a" #d "1", "a" #d "2", "a" #d "3", "a" #d "4", "a" #d "5", "a" #d "6", "a" #d "7", "a" #d "8", "a" #d "9"
__device__ __forceinline__ void acc_reserve() {
  asm volatile("" ::: "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", STILL_A10(1), STILL_A10(2), STILL_A10(3),
               STILL_A10(4), STILL_A10(5), STILL_A10(6), STILL_A10(7), STILL_A10(8), STILL_A10(9), STILL_A10(10),
               STILL_A10(11), STILL_A10(12), STILL_A10(13), STILL_A10(14), STILL_A10(15), STILL_A10(16), STILL_A10(17),
               STILL_A10(18), STILL_A10(19), STILL_A10(20), STILL_A10(21), STILL_A10(22), STILL_A10(23), STILL_A10(24),
               "a250", "a251", "a252", "a253", "a254", "a255");
}
#undef STILL_A10

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>)
template <int N, int I = 0, class F> __device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// Fragment loads through a buffer descriptor: one constant offset register
// per lane, the fragment's byte offset in a scalar register.  The descriptor
// spans 4 GiB; callers stay in bounds.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, -1, 0x00027000);
}
__device__ __forceinline__ half8 buf_load_frag(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
  return __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, 0));
}

// Where a wave finds its fragments.  One head's keys and values can span more
// than the 4 GiB of an offset, so the bases are formed in 64 bits: K of a key
// block from the wave's first key tile in it (tile0, clamped to the last tile;
// up to four tiles of 64 dc bytes follow: dc below 2^24), X^T from the wave's
// first feature tile (up to four of 64 npad bytes: npad below 2^24).  Bases in
// halfs from the head's first, offsets in bytes from the base.
__host__ __device__ __forceinline__ unsigned xatt_ktile0(unsigned n, unsigned ktlast) {
  return (n >> 5) < ktlast ? n >> 5 : ktlast;
}
__host__ __device__ __forceinline__ long xatt_kbase(unsigned tile0, unsigned ksteps) { return (long)tile0 * ksteps * 512; }
__host__ __device__ __forceinline__ unsigned xatt_koff(unsigned tile0, unsigned ktlast, unsigned kt, unsigned ksteps,
                                                       unsigned js) {
  return ((kt < ktlast - tile0 ? kt : ktlast - tile0) * ksteps + js) * 1024u;
}
__host__ __device__ __forceinline__ long xatt_xbase(unsigned ft0, unsigned nsteps) { return (long)ft0 * nsteps * 512; }
__host__ __device__ __forceinline__ unsigned xatt_xoff(unsigned f, unsigned nsteps, unsigned ns) {
  return (f * nsteps + (ns < nsteps - 1 ? ns : nsteps - 1)) * 1024u;
}

template <int TT, int D2, bool TRACK, int KT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void xattn_f16_kernel(AttnArgs a) {
  constexpr int NW = 4, NT = 256, KW = 32 * KT, KB = NW * KW;
  constexpr int LT = TT / 32;            // latent tiles
  constexpr int FW = D2 / NW;            // output features per wave
  constexpr int FT = FW / 32;            // feature tiles per wave
  constexpr int KV = KT < 2 ? KT : 2;    // key tiles per wave with logits in vector registers
  constexpr int OT = LT * FT;            // accumulation registers: output tiles lt * FT + f, then the other logits
  constexpr int QC = 64, NS = QC / 16;   // Q chunk width, k steps per chunk
  constexpr int KR = 4;                  // K ring depth (steps)
  constexpr int NQS = 4, QAHEAD = 3;     // Q stages; chunks between a stage's loads and its use
  constexpr int QI = TT / 8 / NW;        // Q stage loads per wave and chunk (8 rows of 128 bytes each)
  constexpr int PB = 256, NH = KB / PB;  // keys per P.X pass, passes per block
  constexpr int LP = PB + 8;             // P row stride (halfs)
  static_assert(XATT_NBK == 2 * NW && XATT_CAP < 256, "one candidate list per wave and lane half");
  static_assert(XATT_CAP_SPLIT >= 32 * KT, "room for a block's candidates and as many again");
  constexpr int XR = FT >= 4 ? 2 : 4;    // X^T ring depth (key steps of 16)
  constexpr int PS = PB / 16;            // key steps per P.X pass
  constexpr int RKI = KB / NT;           // key norms loaded per thread and block
  static_assert(FT >= 1 && QI >= 1 && TT % (8 * NW) == 0 && KT % 2 == 0 && OT + LT * (KT - KV) <= 16, "tile sizes");

  __shared__ __attribute__((aligned(16))) f16 Qs[NQS][TT * QC];   // rows of 8 swizzled 16-byte units
  __shared__ __attribute__((aligned(16))) f16 Ps[TT * LP];
  __shared__ float red_m[TT][NW], red_l[TT][NW];
  __shared__ __attribute__((aligned(16))) float rks[2][KB];   // key norm factors (0 past the range end)
  __shared__ __attribute__((aligned(16))) float kbs[2][KB];   // key mask: 0, or -inf past the range end
  __shared__ float qsl[TT];   // qs of each latent row (read in the softmax, not held in registers)
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave index (uniform)
  const int lane_ = lane;

  const int ntt = (a.t + TT - 1) / TT, HC = a.H * a.nc;
  const int total = gridDim.x;
  int L = blockIdx.x;
  if ((total & 7) == 0) L = (L & 7) * (total >> 3) + (L >> 3);
  const int S = total / (ntt * HC);
  const int tt = L % ntt, rest = L / ntt;
  const int split = rest % S, hc = rest / S;
  const int h = hc / a.nc, c = hc - h * a.nc;
  const int t0 = tt * TT;
  const int nbeg = split * a.keys_per_split;
  const int nend = min(a.N, nbeg + a.keys_per_split);

  const f16* qb = (const f16*)a.q + (long)h * a.t * a.ldq + (long)c * a.dc;
  const f16* kb = (const f16*)a.k + (long)hc * a.npad * a.dc;
  const f16* xtb = (const f16*)a.xt + ((long)h * a.xfeat + (long)c * a.xcoff) * a.npad;
  const float* rkb = a.rk + (long)h * a.N * a.nc + c;
  const unsigned ksteps = (unsigned)(a.dc >> 4);   // width steps of one key tile
  const unsigned nsteps = (unsigned)(a.npad >> 4); // key steps of one feature tile
  const unsigned ktlast = (unsigned)(a.npad >> 5) - 1;
  const __amdgpu_buffer_rsrc_t xrsrc = buf_rsrc(xtb + xatt_xbase((unsigned)(FW / 32 * w), nsteps));
  const unsigned voff = 16u * (unsigned)lane;

  float m_run[LT], l_run[LT];
#pragma unroll
  for (int lt = 0; lt < LT; ++lt) {
    m_run[lt] = -INFINITY;
    l_run[lt] = 0.f;
  }
  if (tid < TT) {
    const int lat = min(t0 + tid, a.t - 1);   // rows past t: any positive factor
    qsl[tid] = a.rq[((long)h * a.t + lat) * a.nc + c] * a.scale_log2;
  }
  // Candidate keys for the logit refinement: every key whose logit lies within
  // REFINE_MARGIN of the running maximum goes to a list of its latent's bucket
  // (wave, lane half), which only this lane writes; keys below that can never
  // be selected.  A list without room for another block's candidates (16 KT)
  // keeps the entries that reach the mean of 32 of them and of these, if they
  // are still too many, the larger of every pair (i, i + half): its largest keys
  // stay whatever comes before and after them.  Keys below that mean enter no
  // more: where all keys lie within the margin the scattered stores of the
  // entries would take longer than the products (32768 keys, 256 latents, 8 x 8
  // heads, logits scaled by 1, whole layer: 15.5 ms with lists of 512 that only
  // halve, 13.0 now).  ncand[lt]: entries (low 8 bits) and that mean, rounded
  // down (-inf before the first time).
  unsigned ncand[LT];
#pragma unroll
  for (int lt = 0; lt < LT; ++lt) ncand[lt] = 0xff800000u;
  const __amdgpu_buffer_rsrc_t crsrc =   // the lists of the tile's first row
      buf_rsrc(TRACK ? a.cand + (((long)split * HC + hc) * a.t + t0) * (XATT_NBK * a.ccap) : nullptr);
  acc_reserve();
  static_for<16 * OT>([&](auto r) { acc_write<decltype(r)::value>(0.f); });

  // Q chunk staging: wave instruction i fills rows [8 b, 8 b + 8) of a stage
  // (b = i NW + w, 1 KB); lane l writes unit l % 8 of row 8 b + l / 8 and so
  // reads the global unit that the swizzle puts there.  Rows past t read the
  // last row: their logits are finite and never reach a stored output.
  // The loads are issued from inline assembly: the compiler, seeing direct
  // loads among the register loads of the K ring, would wait for all of them
  // before each use of a K fragment.  It still counts the K-ring loads, and
  // so over-waits by at most the stage loads issued after them; the waits
  // for the stages are explicit (chunk_barrier).
  // The row offsets are computed at each use from two registers: held in
  // registers of their own they do not fit beside the accumulators, and a
  // reload in front of the chunk loop is waited for in every chunk.
  int qrow = t0 + 8 * w + (lane >> 3);   // (the swizzle is the same for every i: rows 32 apart)
  const unsigned qcol = 16u * (unsigned)((lane & 7) ^ lds_swz<8>(8 * w + (lane >> 3)));
  auto dma_q = [&](int stage, int d0) {
    const f16* qd = qb + d0;   // uniform: base in scalar registers
    asm volatile("" : "+v"(qrow));
#pragma unroll
    for (int i = 0; i < QI; ++i) {
      const unsigned qoff = (unsigned)min(qrow + 8 * NW * i, a.t - 1) * (2u * (unsigned)a.ldq) + qcol;   // bytes, below 2^32
      const unsigned m0v = (unsigned)(size_t)(__attribute__((address_space(3))) f16*)&Qs[stage][(i * NW + w) * 512];
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                   :: "v"(qoff), "s"(qd), "s"(m0v) : "memory", "m0");
    }
  };
  // Q fragment of latent tile lt, 16-column step js, from a stage
  auto q_frag = [&](int stage, int lt, int js) -> half8 {
    const int r = 32 * lt + (lane & 31);
    return *(const half8*)&Qs[stage][r * QC + 8 * ((2 * js + (lane >> 5)) ^ lds_swz<8>(r))];
  };
  // Chunks are numbered across blocks (g): chunk g uses stage g % NQS and Q
  // columns [(g % nch) QC, +QC); it issues the loads of chunk g + QAHEAD into
  // the stage that chunk g - 1 released, and its last step reads the first
  // fragments of chunk g + 1.  So at the barrier that ends chunk g the loads
  // of chunk g + 2 must have landed: they were issued at the start of chunk
  // g - 1, followed by the K-ring loads of chunk g - 1 and the stage and
  // K-ring loads of chunk g (more at block boundaries); loads return in
  // order.  The asm statements also keep the compiler from moving memory
  // accesses across the barriers.
  static_assert(NQS == 4 && QAHEAD == 3, "the stage ring and the wait count go together");
  constexpr int QWAIT = NS * KT + QI + NS * KT, QWAIT_LAST = QWAIT - KR * KT;   // (the last chunk reloads fewer)
  static_assert(QWAIT <= 63, "vmcnt range");
  // the first chunk's barrier: the loads after the previous block's last stage load are at least
  static_assert((NS - KR) * KT + NH * PS * FT + KR * KT + QI + NS * KT >= QWAIT, "wait count across blocks");
  auto chunk_barrier = [&]() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(QWAIT) : "memory");
  };
  auto chunk_barrier_last = [&]() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(QWAIT_LAST) : "memory");
  };
  // this wave's LDS traffic has completed, then all waves meet (stage loads
  // may still be in flight)
  auto lds_barrier = [&]() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };
  // the wave's K fragments: of the block at n0 (k_block), its key tile kt, width step js
  unsigned ktile0 = xatt_ktile0((unsigned)(nbeg + KW * w), ktlast);
  __amdgpu_buffer_rsrc_t krsrc = buf_rsrc(kb + xatt_kbase(ktile0, ksteps));
  auto k_block = [&](int n0) {
    ktile0 = xatt_ktile0((unsigned)(n0 + KW * w), ktlast);
    krsrc = buf_rsrc(kb + xatt_kbase(ktile0, ksteps));
  };
  auto load_k = [&](int kt, int js) -> half8 {
    return buf_load_frag(krsrc, voff, xatt_koff(ktile0, ktlast, (unsigned)kt, ksteps, (unsigned)js));
  };
  // X^T fragment of this wave's feature tile f, key step ns (absolute)
  auto load_x = [&](int f, int ns) -> half8 {
    return buf_load_frag(xrsrc, voff, xatt_xoff((unsigned)f, nsteps, (unsigned)ns));
  };
  // key step ps of pass hf of the block at n0: pass hf covers keys
  // [64 hf, 64 hf + 64) of every wave
  auto x_step = [&](int n0, int hf, int ps) -> int { return ((n0 + 64 * hf) >> 4) + (KW / 16) * (ps >> 2) + (ps & 3); };
  auto load_rk = [&](int n) -> float {   // unmasked (branch-free load)
    return rkb[(long)min(n, nend - 1) * a.nc];
  };

  const int nch = a.dc / QC;   // a.dc is a multiple of 2 QC (checked on the host), nch >= 2
  half8 kr[KR][KT];
  half8 xr[XR][FT];
  half8 qf[2][LT];
  int g = 0, qn = QAHEAD % nch;   // chunk number; Q chunk of chunk g + QAHEAD
  int rbuf = 0;
  // prologue: Q chunks 0 .. QAHEAD-1, key norms and K ring of the first block
#pragma unroll
  for (int c = 0; c < QAHEAD; ++c) dma_q(c, (c % nch) * QC);
#pragma unroll
  for (int j = 0; j < KR; ++j)
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) kr[j][kt] = load_k(kt, j);
#pragma unroll
  for (int i = 0; i < RKI; ++i) {
    const int n = nbeg + tid + NT * i;
    const float v = load_rk(n);
    rks[0][tid + NT * i] = n < nend ? v : 0.f;
    kbs[0][tid + NT * i] = n < nend ? 0.f : -INFINITY;
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

  for (int n0 = nbeg; n0 < nend; n0 += KB) {
    const bool next_block = n0 + KB < nend;   // uniform
    f32x16 s[LT * KV];   // [lt * KV + kt], kt < KV; the other tiles: accumulation tile OT + lt * (KT - KV) + kt - KV

    // ---- S^T = K_blk Q^T over the head width.  A chunk runs its MFMAs on the
    // Q chunk in LDS and the K ring while it loads the next stages: the Q
    // chunk QAHEAD chunks on and, into each K fragment right after its last
    // use, the step KR steps on (none past the block's last step).  Each step reads the next step's Q fragments (the
    // next chunk's first ones in the last step) before its own MFMAs;
    // scheduling barriers keep that order and spread the loads over the chunk.
    auto qk_chunk = [&](auto first, auto last, int ch) {
      dma_q((g + QAHEAD) & (NQS - 1), qn * QC);
      const int sc = g & (NQS - 1), sn = (g + 1) & (NQS - 1);
#pragma unroll
      for (int j = 0; j < NS; ++j) {
        if (!(decltype(last)::value && j + 1 == NS)) {
#pragma unroll
          for (int lt = 0; lt < LT; ++lt)
            qf[(j + 1) & 1][lt] = q_frag(j + 1 < NS ? sc : sn, lt, j + 1 < NS ? j + 1 : 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        acc_reserve();
        static_for<KT>([&](auto ktc) {
          constexpr int kt = decltype(ktc)::value;
          static_for<LT>([&](auto ltc) {
            constexpr int lt = decltype(ltc)::value;
            const half8 &ak = kr[j % KR][kt], &bq = qf[j & 1][lt];
            if constexpr (kt < KV) {
              f32x16& c = s[lt * KV + kt];
              c = __builtin_amdgcn_mfma_f32_32x32x16_f16(ak, bq, decltype(first)::value && j == 0 ? zero16() : c, 0, 0, 0);
            } else if (decltype(first)::value && j == 0) {
              acc_mfma_first<OT + lt * (KT - KV) + kt - KV>(ak, bq);
            } else {
              acc_mfma<OT + lt * (KT - KV) + kt - KV>(ak, bq);
            }
          });
          if (!(decltype(last)::value && j + KR >= NS)) kr[j % KR][kt] = load_k(kt, ch * NS + j + KR);
          __builtin_amdgcn_sched_barrier(0);
        });
      }
      ++g;
      qn = qn + 1 == nch ? 0 : qn + 1;
    };
#pragma unroll
    for (int lt = 0; lt < LT; ++lt) qf[0][lt] = q_frag(g & (NQS - 1), lt, 0);
    qk_chunk(std::true_type{}, std::false_type{}, 0);
    chunk_barrier();
    for (int ch = 1; ch + 1 < nch; ++ch) {
      qk_chunk(std::false_type{}, std::false_type{}, ch);
      chunk_barrier();
    }
    {  // last chunk, with the next block's key norms (selected after the
       // chunk: an earlier use would wait for their loads in front of the
       // chunk's stage loads)
      float rk_raw[RKI];
#pragma unroll
      for (int i = 0; i < RKI; ++i) rk_raw[i] = load_rk(n0 + KB + tid + NT * i);
      qk_chunk(std::false_type{}, std::true_type{}, nch - 1);
#pragma unroll
      for (int i = 0; i < RKI; ++i) {
        const int nn = n0 + KB + tid + NT * i;
        rks[rbuf ^ 1][tid + NT * i] = nn < nend ? rk_raw[i] : 0.f;
        kbs[rbuf ^ 1][tid + NT * i] = nn < nend ? 0.f : -INFINITY;
      }
      chunk_barrier_last();
    }
    acc_settle();
    acc_reserve();
    // the lane indices anew: addresses derived from them below are computed
    // here each time and not kept in registers through the QK product
    int l32 = lane_, lg = lane_ >> 5;
    asm volatile("" : "+v"(l32), "+v"(lg));
    l32 &= 31;
    // X^T ring for the block's P.X (arrives during the softmax)
#pragma unroll
    for (int i = 0; i < XR; ++i)
#pragma unroll
      for (int f = 0; f < FT; ++f) xr[i][f] = load_x(f, x_step(n0, 0, i));

    // ---- softmax: x = S * rk + kb: kb = -inf masks the keys past the range
    // end without a select (their tiled k slots are finite, and fma with a
    // zero addend is exactly the product); logit (log2 units) = x * qs[lt]
    // (qs > 0, so block maxima of x scale to those of the logits); one pass
    // for the block maxima, one for the probabilities
    const float* rkc = rks[rbuf];
    const float* kbc = kbs[rbuf];
    // x of the four keys of rows [8 jq, 8 jq + 4) + 4 lg of tile kt, for every latent tile
    auto key4 = [&](int kt, int jq, float (&rk)[4], float (&kb)[4]) {
      const int kl = KW * w + 32 * kt + 8 * jq + 4 * lg;
      const float4 r4 = *(const float4*)&rkc[kl];
      const float4 b4 = *(const float4*)&kbc[kl];
      rk[0] = r4.x; rk[1] = r4.y; rk[2] = r4.z; rk[3] = r4.w;
      kb[0] = b4.x; kb[1] = b4.y; kb[2] = b4.z; kb[3] = b4.w;
    };
    float lmx[LT][KT], qs[LT], alpha[LT], mref[LT];
#pragma unroll
    for (int lt = 0; lt < LT; ++lt) {
      qs[lt] = qsl[32 * lt + l32];
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) lmx[lt][kt] = -INFINITY;
    }
    // logit register j of tile (lt, kt)
    auto sval = [&](auto ltc, auto ktc, auto jc) -> float {
      constexpr int lt = decltype(ltc)::value, kt = decltype(ktc)::value, j = decltype(jc)::value;
      if constexpr (kt < KV) return s[lt * KV + kt][j];
      else return acc_read<16 * (OT + lt * (KT - KV) + kt - KV) + j>();
    };
    static_for<KT>([&](auto ktc) {
      static_for<4>([&](auto jqc) {
        constexpr int kt = decltype(ktc)::value, jq = decltype(jqc)::value;
        float rk[4], kb[4];
        key4(kt, jq, rk, kb);
        static_for<LT>([&](auto ltc) {
          static_for<4>([&](auto uc) {
            constexpr int lt = decltype(ltc)::value, u = decltype(uc)::value;
            lmx[lt][kt] = fmaxf(lmx[lt][kt], fmaf(sval(ltc, ktc, std::integral_constant<int, 4 * jq + u>{}), rk[u], kb[u]));
          });
          // computed here, not sunk to its first use with the logits kept until then
          asm volatile("" : "+v"(lmx[decltype(ltc)::value][kt]));
        });
        acc_reserve();
        __builtin_amdgcn_sched_barrier(0);
      });
    });
#pragma unroll
    for (int lt = 0; lt < LT; ++lt) {
      float mx = lmx[lt][0];
#pragma unroll
      for (int kt = 1; kt < KT; ++kt) mx = fmaxf(mx, lmx[lt][kt]);
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      if (lg == 0) red_m[32 * lt + l32][w] = mx * qs[lt];
    }
    lds_barrier();
#pragma unroll
    for (int lt = 0; lt < LT; ++lt) {
      const int li = 32 * lt + l32;
      float mb = red_m[li][0];
#pragma unroll
      for (int u = 1; u < NW; ++u) mb = fmaxf(mb, red_m[li][u]);
      const float m_new = fmaxf(m_run[lt], mb);
      mref[lt] = (m_new == -INFINITY) ? 0.f : m_new;   // all keys masked so far: every p is 0
      alpha[lt] = __builtin_amdgcn_exp2f(m_run[lt] - mref[lt]);   // m_run = -inf -> 0 (o, l are 0 then)
      m_run[lt] = m_new;
    }
    if constexpr (TRACK) {
      // Candidates: most 32 x 32 tiles have none and are passed by, then most
      // groups of four.  Padding rows past t (their last row's logits) take
      // none.
      typedef int i32x2 __attribute__((ext_vector_type(2)));
      static_for<LT>([&](auto ltc) {
        constexpr int lt = decltype(ltc)::value;
        const int li = 32 * lt + l32;
        int n = (int)(ncand[lt] & 0xffu);
        const float cut = t0 + li < a.t ? fmaxf(m_run[lt] - REFINE_MARGIN, __uint_as_float(ncand[lt] & ~0xffu)) : INFINITY;
        static_for<KT>([&](auto ktc) {
          constexpr int kt = decltype(ktc)::value;
          if (!__any(lmx[lt][kt] * qs[lt] > cut)) return;
          acc_reserve();
          asm volatile("" : "+v"(lg));   // (norms and masks are read anew, not kept from the pass before)
          const int slot0 = (li * XATT_NBK + 2 * w + lg) * a.ccap, k0 = n0 + KW * w + 32 * kt + 4 * lg;
          static_for<4>([&](auto jqc) {
            constexpr int jq = decltype(jqc)::value;
            float rk[4], kb[4], v[4];
            key4(kt, jq, rk, kb);
            static_for<4>([&](auto uc) {
              constexpr int u = decltype(uc)::value;
              v[u] = fmaf(sval(ltc, ktc, std::integral_constant<int, 4 * jq + u>{}), rk[u], kb[u]) * qs[lt];
            });
            if (__any(fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])) > cut)) {
#pragma unroll
              for (int u = 0; u < 4; ++u) {
                if (v[u] > cut) {
                  const i32x2 e = {__float_as_int(v[u]), k0 + 8 * jq + u};
                  __builtin_amdgcn_raw_buffer_store_b64(e, crsrc, 8 * (slot0 + n), 0, 0);
                  ++n;
                }
              }
            }
          });
        });
        ncand[lt] = (ncand[lt] & ~0xffu) | (unsigned)n;
        const int most = a.ccap - 16 * KT;
        if (__any(n > most)) {
          constexpr int NB = 8;   // entries loaded at a time
          n = n > most ? n : 0;
          const int at = 8 * (li * XATT_NBK + 2 * w + lg) * a.ccap;
          float sum = 0.f, top = -INFINITY;
#pragma unroll 1
          for (int i = 0; i < (n ? 32 : 0); i += NB) {   // (no list, no access: rows past t have no memory)
            float x[NB];
#pragma unroll
            for (int q = 0; q < NB; ++q)
              x[q] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(crsrc, at + 8 * ((i + q) * n >> 5), 0, 0));
#pragma unroll
            for (int q = 0; q < NB; ++q) {
              sum += x[q];
              top = fmaxf(top, x[q]);
            }
          }
          const float mean = fminf(sum * (1.f / 32), top);
          int kept = 0;
#pragma unroll 1
          for (int i = 0; i < n; i += NB) {   // (kept <= i: no entry is overwritten before it is read)
            i32x2 e[NB];
#pragma unroll
            for (int q = 0; q < NB; ++q)   // (past the last entry: the last one again)
              e[q] = __builtin_bit_cast(i32x2, __builtin_amdgcn_raw_buffer_load_b64(crsrc, at + 8 * min(i + q, n - 1), 0, 0));
#pragma unroll
            for (int q = 0; q < NB; ++q)
              if (i + q < n && __int_as_float(e[q].x) >= mean) {
                __builtin_amdgcn_raw_buffer_store_b64(e[q], crsrc, at + 8 * kept, 0, 0);
                ++kept;
              }
          }
          if (__any(kept > most)) {
            const int m = kept > most ? kept : 0, half = (m + 1) / 2;
#pragma unroll 1
            for (int i = 0; i + half < m; i += NB) {
              float own[NB];
              i32x2 other[NB];
#pragma unroll
              for (int q = 0; q < NB; ++q) {
                const int p = at + 8 * min(i + q, m - half - 1);
                own[q] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(crsrc, p, 0, 0));
                other[q] = __builtin_bit_cast(i32x2, __builtin_amdgcn_raw_buffer_load_b64(crsrc, p + 8 * half, 0, 0));
              }
#pragma unroll
              for (int q = 0; q < NB; ++q)
                if (__int_as_float(other[q].x) > own[q])
                  __builtin_amdgcn_raw_buffer_store_b64(other[q], crsrc, at + 8 * min(i + q, m - half - 1), 0, 0);
            }
            kept = m ? half : kept;
          }
          if (n) {   // (every entry is above the mean before, but for its rounding)
            const unsigned u = __float_as_uint(mean), down = mean < 0.f ? u + 0xffu : u;
            ncand[lt] = (down & ~0xffu) | (unsigned)kept;
          }
        }
      });
    }
    // rescale O for the latents whose maximum grew (rare after the first
    // blocks)
    static_for<LT>([&](auto ltc) {
      constexpr int lt = decltype(ltc)::value;
      if (__any(alpha[lt] != 1.f)) {
        static_for<16 * FT>([&](auto rc) {
          constexpr int r = 16 * FT * lt + decltype(rc)::value;
          acc_write<r>(acc_read<r>() * alpha[lt]);
        });
      }
    });
    float psum[LT];
#pragma unroll
    for (int lt = 0; lt < LT; ++lt) psum[lt] = 0.f;

    if (next_block) k_block(n0 + KB);   // (every K load of this block has been issued)
    static_for<NH>([&](auto hfc) {
      constexpr int hf = decltype(hfc)::value;
      // ---- probabilities of the pass's keys
      if (hf > 0) lds_barrier();   // every wave has read the previous pass's P
      asm volatile("" : "+v"(lg));
      static_for<2>([&](auto k2c) {
        static_for<4>([&](auto jqc) {
          constexpr int k2 = decltype(k2c)::value, kt = 2 * hf + k2, jq = decltype(jqc)::value;
          float rk[4], kb[4];
          key4(kt, jq, rk, kb);
          static_for<LT>([&](auto ltc) {
            constexpr int lt = decltype(ltc)::value;
            half4 pv;
            static_for<4>([&](auto uc) {
              constexpr int u = decltype(uc)::value;
              const float x = fmaf(sval(ltc, std::integral_constant<int, kt>{}, std::integral_constant<int, 4 * jq + u>{}),
                                   rk[u], kb[u]);
              const float p = __builtin_amdgcn_exp2f(fmaf(x, qs[lt], -mref[lt]));
              psum[lt] += p;
              pv[u] = (f16)p;
            });
            asm volatile("" : "+v"(psum[lt]));
            *(half4*)&Ps[(32 * lt + l32) * LP + 64 * w + 32 * k2 + 8 * jq + 4 * lg] = pv;
          });
          acc_reserve();
          __builtin_amdgcn_sched_barrier(0);
        });
      });
      if (hf + 1 == NH) {
#pragma unroll
        for (int lt = 0; lt < LT; ++lt) {
          const float ps = psum[lt] + __shfl_xor(psum[lt], 32);
          if (lg == 0) red_l[32 * lt + l32][w] = ps;
        }
      }
      lds_barrier();

      // ---- O^T += X^T P^T over the pass's keys, 16 at a time (the next
      // step's P fragments read before this step's MFMAs)
      half8 pf[2][LT];
#pragma unroll
      for (int lt = 0; lt < LT; ++lt) pf[0][lt] = *(const half8*)&Ps[(32 * lt + l32) * LP + 8 * lg];
#pragma unroll
      for (int ps = 0; ps < PS; ++ps) {
        if (ps + 1 < PS) {
#pragma unroll
          for (int lt = 0; lt < LT; ++lt)
            pf[(ps + 1) & 1][lt] = *(const half8*)&Ps[(32 * lt + l32) * LP + 16 * (ps + 1) + 8 * lg];
        }
        __builtin_amdgcn_sched_barrier(0);
        acc_reserve();
        static_for<FT>([&](auto fc) {
          constexpr int f = decltype(fc)::value;
          static_for<LT>([&](auto ltc) {
            constexpr int lt = decltype(ltc)::value;
            acc_mfma<lt * FT + f>(xr[ps % XR][f], pf[ps & 1][lt]);
          });
          if (ps + XR < PS) xr[ps % XR][f] = load_x(f, x_step(n0, hf, ps + XR));
          else if (hf + 1 < NH) xr[ps % XR][f] = load_x(f, x_step(n0, hf + 1, ps + XR - PS));
          else {   // the next block's first K fragments, as X^T fragments retire (of this block again at the
                   // very end: loaded, never used)
#pragma unroll
            for (int i = KR * KT * ((ps + XR - PS) * FT + f) / (XR * FT); i < KR * KT * ((ps + XR - PS) * FT + f + 1) / (XR * FT); ++i)
              kr[i / KT][i % KT] = load_k(i % KT, i / KT);
          }
          __builtin_amdgcn_sched_barrier(0);
        });
      }
    });
#pragma unroll
    for (int lt = 0; lt < LT; ++lt) {
      const int li = 32 * lt + l32;
      float lb = 0.f;
#pragma unroll
      for (int u = 0; u < NW; ++u) lb += red_l[li][u];
      l_run[lt] = l_run[lt] * alpha[lt] + lb;
    }
    rbuf ^= 1;
  }

  // stage loads of chunks past the end may still be in flight: they land
  // before the workgroup's LDS is released
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  acc_settle();
  acc_reserve();
  const int l32 = lane & 31, lg = lane >> 5;

  // ---- partial (O un-normalised, m, l) of this key range
  static_for<LT>([&](auto ltc) {
    constexpr int lt = decltype(ltc)::value;
    const int lat = t0 + 32 * lt + l32;
    const long row = ((long)split * HC + hc) * a.t + min(lat, a.t - 1);
    float* op = a.opart + row * a.d2;
    static_for<FT * 4>([&](auto ic) {   // (accumulators read by whole waves, rows past t not stored)
      constexpr int f = decltype(ic)::value / 4, jq = decltype(ic)::value % 4, r = 16 * (lt * FT + f) + 4 * jq;
      const f32x4 v = {acc_read<r>(), acc_read<r + 1>(), acc_read<r + 2>(), acc_read<r + 3>()};
      if (lat < a.t) *(f32x4*)&op[FW * w + 32 * f + 8 * jq + 4 * lg] = v;
    });
    if (lat >= a.t) return;
    if (w == 0 && lg == 0) {
      a.mpart[row] = m_run[lt];
      a.lpart[row] = l_run[lt];
    }
    if constexpr (TRACK) a.ocnt[row * XATT_NBK + 2 * w + lg] = (int)(ncand[lt] & 0xffu);
  });
}

}  // namespace still
