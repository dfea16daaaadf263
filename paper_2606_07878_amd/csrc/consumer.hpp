// consumer.hpp - attention of base-model queries over a compacted cache
// followed by an uncompacted suffix, with the optional per-entry bias of the
// compact part (Appendix B, bias semantics in attention):
//   out = sum_j exp(s_j) v_j / sum_j exp(s_j),
//   s_j = scale q.C_k[j] + beta[j]  (j < t),   s_j = scale q.K[j - t]  (suffix).
// Decode-shaped (a few query rows per KV head): one wave per (KV head, key
// split), register-resident; more rows: the fp32 matrix instructions.  Online
// softmax over the chunks of a split; splits merged by a second kernel.  fp32
// arithmetic.
#pragma once
#include "common.hpp"
#include "misc.hpp"

namespace still {

constexpr int ATTEND_MAX_ROWS = 32;   // group * n_queries
// Rows per KV head up to which the register-resident decode kernel is taken
// instead of the matrix one (us per call with its merge, decode / matrix, bf16
// unless said).  2 rows: 8 heads x 1088 keys of width 256 11.2 / 16.0, x 65600
// 110 / 118.  4 rows over few keys in all, 8 heads of width 128: x 1024 keys
// 10.3 / 10.6, x 1536 (the line) 11.3 / 10.9, x 4096 13.3 / 11.0, x 131136 152 /
// 114; of width 256: x 1536 13.4 / 16.5, x 2048 14.7 / 16.7, x 3072 22.2 / 17.4;
// 2 heads x 6144 17.9 / 17.2; of width 64 the matrix kernel throughout (x 512
// 10.0 / 8.2).  8 rows over still fewer, rows of 512 bytes and more, 8 heads: width
// 256 x 256 keys (the line) 14.0 / 16.1, x 384 16.8 / 16.2, x 1088 29.8 / 16.7; fp32
// width 256 x 256 12.4 / 15.8, x 512 15.8 / 15.9; fp32 width 128 x 256 10.2 / 10.8, x
// 384 11.4 / 10.9.
inline __host__ __device__ int attend_decode_rows(int d, int esize, int heads, long keys) {
  if (d * esize >= 512 && heads * keys <= 2048) return 8;
  return d >= 128 && heads * keys <= 12288 ? 4 : 2;
}
// 16-byte loads of a decode chunk per lane and operand, for a kernel of up to rb rows
inline __host__ __device__ constexpr int attend_decode_nit(int rb) { return rb <= 4 ? 8 : 4; }
constexpr int ATTEND_KC = 32;         // keys per chunk of the matrix kernel

struct ConsumerArgs {
  const void* q;        // [H*group][nq][D]
  const void* ck;       // [H][t][D]
  const void* cv;
  const float* beta;    // [H][t] or NULL
  const void* k;        // [H][S][D] suffix keys (RoPE'd), may be NULL when S = 0
  const void* v;
  void* out;            // [H*group][nq][D]
  float* opart;         // [splits][H][R][D]
  float* mpart;         // [splits][H][R]
  float* lpart;
  int H, group, nq, t, S, causal, splits, cps;   // cps: chunks per split
  float scale;
  const double* qpos;   // [nq] logical query positions, or NULL (q as given)
  double theta;         // base RoPE theta when qpos is set
};

// Rotation angle of feature pair jh (< d/2) at position pos, reduced to
// [-pi, pi] in fp64 before the fp32 sine and cosine (positions reach 1e5+).
__device__ __forceinline__ void rope_angle(double pos, int jh, int d, double theta, float& c, float& s) {
  const double inv = pow(theta, -2.0 * jh / d);
  double phi = pos * inv;
  phi -= 6.283185307179586 * rint(phi * 0.15915494309189535);
  sincosf((float)phi, &s, &c);
}

// 16-byte pieces as a native vector: plain loads and stores (a HIP uint4 copy
// lowers to memcpy, which keeps a staged array in scratch memory)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <class T> __device__ __forceinline__ void unpack16(const u32x4& u, float (&o)[16 / sizeof(T)]);
template <> __device__ __forceinline__ void unpack16<bf16>(const u32x4& u, float (&o)[8]) {
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    o[2 * i] = __uint_as_float(w[i] << 16);
    o[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}
template <> __device__ __forceinline__ void unpack16<float>(const u32x4& u, float (&o)[4]) {
  o[0] = __uint_as_float(u.x);
  o[1] = __uint_as_float(u.y);
  o[2] = __uint_as_float(u.z);
  o[3] = __uint_as_float(u.w);
}

// Chunk c of KV head h: chunks [0, nck) cover the compact rows, [nck, nck + nsk)
// the suffix rows; a chunk never straddles the two, so its base pointer and row
// count are wave-uniform.
struct AttendChunk {
  const char* kbase;   // row 0 of this part's keys for head h
  const char* vbase;
  int j0, rows;        // first row of the chunk within the part, rows in the part
  bool compact;
};

template <class IT, int D, int KC>
__device__ __forceinline__ AttendChunk attend_chunk(const ConsumerArgs& a, int h, int c) {
  constexpr long ROWB = (long)D * sizeof(IT);
  const int nck = (a.t + KC - 1) / KC;
  AttendChunk k;
  k.compact = c < nck;
  k.rows = k.compact ? a.t : a.S;
  k.j0 = (k.compact ? c : c - nck) * KC;
  const long hoff = (long)h * k.rows * ROWB;
  k.kbase = (const char*)(k.compact ? a.ck : a.k) + hoff;
  k.vbase = (const char*)(k.compact ? a.cv : a.v) + hoff;
  return k;
}

// ---------------------------------------------------------------------------
// More query rows (prefill-shaped calls, several heads per KV head): both products on the fp32 matrix
// instructions (operands and sums in fp32, as given), TR = 16 or 32 query rows
// (rows past R are zero queries, never stored).  A workgroup is 4 waves; wave w
// takes chunks c0 + w, c0 + w + 4, ... of the split's chunks of 32 keys.
//   S^T[key][row]: keys are MFMA rows, query rows columns, so a lane owns one
//   query row and the softmax statistics stay in the lane.  Lane group lg of
//   key l reads 16-byte pieces LG i + lg of the key's row: the pairing of
//   contraction indices is free, so the pieces feed the product as loaded,
//   against the query row in LDS.
//   O^T[feature][row]: accumulator register j of S^T holds the keys
//   row(j, lg), the B operand of one P.V step; lane l reads the D / TR
//   consecutive features [l D / TR, ..) of that key's V row, one per output
//   tile, so the V rows are read whole and nothing is exchanged.
// V of a chunk is loaded ahead of its logits and K of the next one ahead of
// the softmax (rows up to 512 bytes).  The waves' partials are combined in LDS.
// A chunk of 32 keys costs 8192 cycles of the matrix pipe at 32 rows and
// D = 128, 4.6 TB/s of bf16 keys and values over the chip: about what memory
// delivers.  32 rows over a 655-entry prefix and a 4099-token suffix (8 heads,
// d = 128): 143 us with FMAs from LDS-resident queries, one wave per split; 21 us.
// ---------------------------------------------------------------------------
constexpr int ATTEND_WAVES = 4;

template <int TR> struct AttendMma;
template <> struct AttendMma<32> {
  typedef f32x16 acc;
  static __device__ __forceinline__ void mma(acc& c, float a, float b) {
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
};
template <> struct AttendMma<16> {
  typedef f32x4 acc;
  static __device__ __forceinline__ void mma(acc& c, float a, float b) {
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

// B bytes at p (B-byte aligned, B = 4, 8 or a multiple of 16) into words
template <int B> __device__ __forceinline__ void load_words(const char* p, uint32_t (&w)[B / 4]) {
  if constexpr (B == 4) {
    w[0] = *(const uint32_t*)p;
  } else if constexpr (B == 8) {
    const uint2 u = *(const uint2*)p;
    w[0] = u.x;
    w[1] = u.y;
  } else {
#pragma unroll
    for (int i = 0; i < B / 16; ++i) {
      const u32x4 u = ((const u32x4*)p)[i];
#pragma unroll
      for (int e = 0; e < 4; ++e) w[4 * i + e] = u[e];
    }
  }
}
template <class IT> __device__ __forceinline__ float word_elem(const uint32_t* w, int e) {
  if constexpr (sizeof(IT) == 4) return __uint_as_float(w[e]);
  else return __uint_as_float(e & 1 ? w[e >> 1] & 0xffff0000u : w[e >> 1] << 16);
}

// dynamic LDS: q rows fp32 [TR][D + 4], later the combined output rows | per-wave key bias [4][KC] | m, l [4][TR]
template <int D, int TR>
inline size_t attend_lds_bytes() {
  return sizeof(float) * ((size_t)TR * (D + 4) + ATTEND_WAVES * ATTEND_KC + 2 * ATTEND_WAVES * TR);
}

template <class IT, int D, int TR>
__global__ __launch_bounds__(64 * ATTEND_WAVES) void attend_rows_kernel(ConsumerArgs a) {
  typedef AttendMma<TR> MM;
  constexpr int KC = ATTEND_KC, LG = 64 / TR, CR = TR * TR / 64, NKT = KC / TR;
  constexpr int ROWB = D * (int)sizeof(IT), EPP = 16 / (int)sizeof(IT), NP = ROWB / 16 / LG;
  constexpr int FPT = D / TR, VB = FPT * (int)sizeof(IT), LQ = D + 4;
  constexpr bool AHEAD = ROWB <= 512;
  constexpr int NA0 = TR == 16 ? 8 : 4, NA = NP < NA0 ? NP : NA0;   // partial sums of a logit
  static_assert(NP >= NA && NKT >= 1 && CR % 4 == 0, "tile shape");
  extern __shared__ float4 attend_smem[];
  float* qs = (float*)attend_smem;                     // [TR][LQ]
  float* kbias = qs + TR * LQ;                         // [waves][KC]: bias of a chunk's keys
  float* wm = kbias + ATTEND_WAVES * KC;               // [waves][TR]
  float* wl = wm + ATTEND_WAVES * TR;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l = lane % TR, lg = lane / TR;
  const int split = blockIdx.x, h = blockIdx.y, R = a.group * a.nq;
  const int nchunks = (a.t + KC - 1) / KC + (a.S + KC - 1) / KC;
  const int c0 = split * a.cps, c1 = min(nchunks, c0 + a.cps);   // this split's chunks [c0, c1)
  {  // query rows g*nq + i of KV head h are contiguous: 16-byte pieces, fp32 in LDS, rows past R zero
    const u32x4* qh = (const u32x4*)((const IT*)a.q + (long)h * R * D);
    for (int pc = tid; pc < TR * (D / EPP); pc += 64 * ATTEND_WAVES) {
      const int r = pc / (D / EPP), x = (pc - r * (D / EPP)) * EPP;
      float f[EPP];
#pragma unroll
      for (int e = 0; e < EPP; ++e) f[e] = 0.f;
      if (r < R) unpack16<IT>(qh[pc], f);
#pragma unroll
      for (int e = 0; e < EPP; e += 4) *(float4*)&qs[r * LQ + x + e] = make_float4(f[e], f[e + 1], f[e + 2], f[e + 3]);
    }
  }
  __syncthreads();
  if (a.qpos) {  // RoPE of the query rows at their logical positions (rotate-half pairs): one angle for the group's heads
    constexpr int HD = D / 2;
    for (int e = tid; e < a.nq * HD; e += 64 * ATTEND_WAVES) {
      const int i = e / HD, j = e % HD;
      float c, sn;
      rope_angle(a.qpos[i], j, D, a.theta, c, sn);
      for (int r = i; r < R; r += a.nq) {
        const float x0 = qs[r * LQ + j], x1 = qs[r * LQ + j + HD];
        qs[r * LQ + j] = x0 * c - x1 * sn;
        qs[r * LQ + j + HD] = x1 * c + x0 * sn;
      }
    }
    __syncthreads();
  }

  typename MM::acc o[FPT];
#pragma unroll
  for (int f = 0; f < FPT; ++f)
#pragma unroll
    for (int j = 0; j < CR; ++j) o[f][j] = 0.f;
  float m = -INFINITY, ls = 0.f;
  const int lim = a.causal ? a.S - a.nq + l % a.nq : 0x7fffffff;   // row g*nq+i sees suffix rows <= S-nq+i
  auto key_of = [&](int kt, int j) { return kt * TR + 4 * LG * (j >> 2) + 4 * lg + (j & 3); };   // within the chunk

  u32x4 kp[NKT][NP];
  auto load_k = [&](const AttendChunk& ch) {
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt) {
      const u32x4* kr = (const u32x4*)(ch.kbase + (long)min(ch.j0 + kt * TR + l, ch.rows - 1) * ROWB);
#pragma unroll
      for (int i = 0; i < NP; ++i) kp[kt][i] = kr[LG * i + lg];
    }
  };
  auto load_bias = [&](const AttendChunk& ch) -> float {   // lane = key (KC of them)
    const int jl = ch.j0 + lane % KC;
    return jl < ch.rows && ch.compact && a.beta ? a.beta[(long)h * a.t + jl] : 0.f;
  };
  float bias = 0.f;
  if (AHEAD && c0 + w < c1) {
    const AttendChunk ch = attend_chunk<IT, D, KC>(a, h, c0 + w);
    load_k(ch);
    bias = load_bias(ch);
  }
  for (int c = c0 + w; c < c1; c += ATTEND_WAVES) {
    const AttendChunk ch = attend_chunk<IT, D, KC>(a, h, c);
    uint32_t vr[NKT * CR][VB / 4];
    auto load_v = [&]() {
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
        for (int j = 0; j < CR; ++j)
          load_words<VB>(ch.vbase + (long)min(ch.j0 + key_of(kt, j), ch.rows - 1) * ROWB + l * VB, vr[kt * CR + j]);
    };
    if constexpr (AHEAD) {
      load_v();
    } else {
      load_k(ch);
      bias = load_bias(ch);
    }
    // ---- logits, summed in NA parts (shorter chains of fp32 additions)
    typename MM::acc s[NKT], sp[NKT][NA];
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
      for (int q = 0; q < NA; ++q)
#pragma unroll
        for (int j = 0; j < CR; ++j) sp[kt][q][j] = 0.f;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      float qv[EPP];
#pragma unroll
      for (int e = 0; e < EPP; e += 4) {
        const float4 u = *(const float4*)&qs[l * LQ + (LG * i + lg) * EPP + e];
        qv[e] = u.x;
        qv[e + 1] = u.y;
        qv[e + 2] = u.z;
        qv[e + 3] = u.w;
      }
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt) {
        float kv[EPP];
        unpack16<IT>(kp[kt][i], kv);
#pragma unroll
        for (int e = 0; e < EPP; ++e) MM::mma(sp[kt][i * NA / NP], kv[e], qv[e]);
      }
    }
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
      for (int j = 0; j < CR; ++j)
      {
#pragma unroll
        for (int st = 1; st < NA; st *= 2)
#pragma unroll
          for (int q = 0; q + st < NA; q += 2 * st) sp[kt][q][j] += sp[kt][q + st][j];
        s[kt][j] = sp[kt][0][j];
      }
    if (lane < KC) kbias[w * KC + lane] = bias;   // (this wave's slot; read back below in program order)
    if constexpr (AHEAD) {
      if (c + ATTEND_WAVES < c1) {
        const AttendChunk nx = attend_chunk<IT, D, KC>(a, h, c + ATTEND_WAVES);
        load_k(nx);
        bias = load_bias(nx);
      }
    } else {
      load_v();
    }
    __builtin_amdgcn_wave_barrier();
    // ---- online softmax: this lane's row, its keys of the chunk
    float cm = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
      for (int jq = 0; jq < CR / 4; ++jq) {
        const float4 b = *(const float4*)&kbias[w * KC + key_of(kt, 4 * jq)];
        const float bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int jl = ch.j0 + key_of(kt, 4 * jq) + u;
          const bool ok = jl < ch.rows && (ch.compact || jl <= lim);
          s[kt][4 * jq + u] = ok ? s[kt][4 * jq + u] * a.scale + bv[u] : -INFINITY;
          cm = fmaxf(cm, s[kt][4 * jq + u]);
        }
      }
#pragma unroll
    for (int off = TR; off < 64; off <<= 1) cm = fmaxf(cm, __shfl_xor(cm, off));
    const float mn = fmaxf(m, cm);
    const float mref = mn == -INFINITY ? 0.f : mn;
    float cs = 0.f;
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
      for (int j = 0; j < CR; ++j) {
        s[kt][j] = expf(s[kt][j] - mref);
        cs += s[kt][j];
      }
#pragma unroll
    for (int off = TR; off < 64; off <<= 1) cs += __shfl_xor(cs, off);
    const float al = expf(m - mref);
    ls = ls * al + cs;
    m = mn;
    // ---- P.V of the chunk, half of its keys in each of two sums, then added
    // to the running (rescaled) sums: chains of 16 keys, not of all keys
#pragma unroll
    for (int f = 0; f < FPT; ++f) {
      typename MM::acc pv[2];
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int j = 0; j < CR; ++j) pv[q][j] = 0.f;
#pragma unroll
      for (int i = 0; i < NKT * CR / 2; ++i)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int x = q * (NKT * CR / 2) + i;
          MM::mma(pv[q], word_elem<IT>(vr[x], f), s[x / CR][x % CR]);
        }
#pragma unroll
      for (int j = 0; j < CR; ++j) o[f][j] = fmaf(o[f][j], al, pv[0][j] + pv[1][j]);
    }
  }
  // ---- combine the waves (each lane holds its row's m, l and features l' FPT + f,
  // l' = row(j, lg) of the accumulator) and write the split's partial rows
  if (lane < TR) {
    wm[w * TR + l] = m;
    wl[w * TR + l] = ls;
  }
  __syncthreads();   // (also: every wave has read the query rows)
  float M = wm[l];
#pragma unroll
  for (int i = 1; i < ATTEND_WAVES; ++i) M = fmaxf(M, wm[i * TR + l]);
  const float Mref = M == -INFINITY ? 0.f : M;
  const float sc = expf(m - Mref);
  for (int i = 0; i < ATTEND_WAVES; ++i) {
    if (w == i) {
#pragma unroll
      for (int j = 0; j < CR; ++j) {
        float* dst = &qs[l * LQ + (4 * LG * (j >> 2) + 4 * lg + (j & 3)) * FPT];
#pragma unroll
        for (int f = 0; f < FPT; ++f) dst[f] = i == 0 ? o[f][j] * sc : dst[f] + o[f][j] * sc;
      }
    }
    __syncthreads();
  }
  const long base = ((long)split * a.H + h) * R;
  for (int e = tid; e < R * (D / 4); e += 64 * ATTEND_WAVES) {
    const int r = e / (D / 4), x = (e - r * (D / 4)) * 4;
    *(float4*)(a.opart + (base + r) * D + x) = *(const float4*)&qs[r * LQ + x];
  }
  if (tid < R) {   // (tid < TR: lane tid of wave 0 owns row tid, so M and Mref are that row's)
    float L = 0.f;
#pragma unroll
    for (int i = 0; i < ATTEND_WAVES; ++i) L += expf(wm[i * TR + tid] - Mref) * wl[i * TR + tid];
    a.mpart[base + tid] = M;
    a.lpart[base + tid] = L;
  }
}

// ---------------------------------------------------------------------------
// Decode-shaped attention (R <= 8 query rows per KV head), no LDS in the chunk
// loop.  A key row is PPR 16-byte pieces; LPK = PPR lanes share one key (lane
// piece pl = lane % LPK holds features [pl*EPP, (pl+1)*EPP)), KPI = 64 / LPK
// keys are read per instruction, NIT instructions make a chunk of KC keys.
// Each lane keeps its slice of every query row in registers; a dot product is
// the lane's EPP-term partial summed over its LPK lanes by DPP row operations
// and, past 16 lanes, shuffles.  The lane then holds the probability of its own
// key, so P.V accumulates o[r][its features] without any exchange; the KPI key
// slots are summed once per split.
// ---------------------------------------------------------------------------
template <class IT, int D, int RB>
struct DecodeTile {
  static constexpr int PPR = D * (int)sizeof(IT) / 16;
  static constexpr int LPK = PPR;
  static constexpr int KPI = 64 / LPK;
  static constexpr int EPP = 16 / (int)sizeof(IT);
  static constexpr int NIT = attend_decode_nit(RB);
  static constexpr int KC = NIT * KPI;
  static_assert(LPK >= 8 && LPK <= 64, "lanes per key");
};

// sum over aligned groups of N lanes (N in 8, 16, 32, 64); every lane gets its group's sum
template <int N>
__device__ __forceinline__ float group_sum(float x) {
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, false));   // xor 1
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4E, 0xF, 0xF, false));   // xor 2
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x141, 0xF, 0xF, false));  // half-row mirror
  if constexpr (N >= 16)
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x140, 0xF, 0xF, false));  // row mirror
  if constexpr (N >= 32) x += __shfl_xor(x, 16);
  if constexpr (N >= 64) x += __shfl_xor(x, 32);
  return x;
}

// combine over the key slots: lanes l, l ^ LPK, l ^ 2 LPK, ... (same piece position)
template <int LPK>
__device__ __forceinline__ float slots_max(float x) {
#pragma unroll
  for (int off = LPK; off < 64; off <<= 1) x = fmaxf(x, __shfl_xor(x, off));
  return x;
}
template <int LPK>
__device__ __forceinline__ float slots_sum(float x) {
#pragma unroll
  for (int off = LPK; off < 64; off <<= 1) x += __shfl_xor(x, off);
  return x;
}

template <class IT, int D, int RB>
struct DecodeStage {
  u32x4 k[DecodeTile<IT, D, RB>::NIT];
  u32x4 v[DecodeTile<IT, D, RB>::NIT];
  float b[DecodeTile<IT, D, RB>::NIT];
};

template <class IT, int D, int RB>
__device__ __forceinline__ void decode_load(const ConsumerArgs& a, const AttendChunk& ch, int h, int lane,
                                            DecodeStage<IT, D, RB>& st) {
  using TL = DecodeTile<IT, D, RB>;
  constexpr long ROWB = (long)D * sizeof(IT);
  const int g = lane / TL::LPK, pl = lane % TL::LPK;
#pragma unroll
  for (int it = 0; it < TL::NIT; ++it) {
    const int jl = min(ch.j0 + it * TL::KPI + g, ch.rows - 1);
    st.k[it] = ((const u32x4*)(ch.kbase + jl * ROWB))[pl];
    st.v[it] = ((const u32x4*)(ch.vbase + jl * ROWB))[pl];
    st.b[it] = (ch.compact && a.beta) ? a.beta[(long)h * a.t + jl] : 0.f;
  }
}

template <class IT, int D, int RB>
__global__ __launch_bounds__(64) void attend_decode_kernel(ConsumerArgs a) {
  using TL = DecodeTile<IT, D, RB>;
  constexpr int EPP = TL::EPP, NIT = TL::NIT;
  const int lane = threadIdx.x, g = lane / TL::LPK, pl = lane % TL::LPK;
  const int split = blockIdx.x, h = blockIdx.y, R = a.group * a.nq;
  const int nck = (a.t + TL::KC - 1) / TL::KC;
  const int nchunks = nck + (a.S + TL::KC - 1) / TL::KC;
  const int c0 = split * a.cps, c1 = min(nchunks, c0 + a.cps);
  auto chunk = [&](int c) {
    AttendChunk k;
    k.compact = c < nck;
    k.rows = k.compact ? a.t : a.S;
    k.j0 = (k.compact ? c : c - nck) * TL::KC;
    const long hoff = (long)h * k.rows * D * (long)sizeof(IT);
    k.kbase = (const char*)(k.compact ? a.ck : a.k) + hoff;
    k.vbase = (const char*)(k.compact ? a.cv : a.v) + hoff;
    return k;
  };

  DecodeStage<IT, D, RB> cur, nxt;
  decode_load<IT, D, RB>(a, chunk(c0), h, lane, cur);
  // the lane's slice of every query row (rows past R repeat row R-1 and are never stored)
  float qv[RB][EPP];
  int lim[RB];
  {
    const IT* qh = (const IT*)a.q + (long)h * R * D;
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const int rr = min(r, R - 1);
      unpack16<IT>(((const u32x4*)(qh + (long)rr * D))[pl], qv[r]);
      lim[r] = a.causal ? a.S - a.nq + rr % a.nq : 0x7fffffff;   // row g*nq+i sees suffix rows <= S-nq+i
    }
    if (a.qpos) {  // RoPE at the logical positions: the pair partner of feature j sits LPK/2 lanes away
      const bool upper = pl >= TL::LPK / 2;
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const double pos = a.qpos[min(r, R - 1) % a.nq];
#pragma unroll
        for (int e = 0; e < EPP; ++e) {
          const float other = __shfl_xor(qv[r][e], TL::LPK / 2);
          float c, sn;
          rope_angle(pos, (pl % (TL::LPK / 2)) * EPP + e, D, a.theta, c, sn);
          qv[r][e] = upper ? qv[r][e] * c + other * sn : qv[r][e] * c - other * sn;
        }
      }
    }
  }
  float m[RB], l[RB], o[RB][EPP];
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    m[r] = -INFINITY;
    l[r] = 0.f;
#pragma unroll
    for (int e = 0; e < EPP; ++e) o[r][e] = 0.f;
  }
  for (int c = c0; c < c1; ++c) {
    const AttendChunk ch = chunk(c);
    decode_load<IT, D, RB>(a, chunk(min(c + 1, c1 - 1)), h, lane, nxt);   // one chunk ahead, in bounds
    float lg[NIT][RB];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      float kv[EPP];
      unpack16<IT>(cur.k[it], kv);
      const int jl = ch.j0 + it * TL::KPI + g;
      const bool valid = jl < ch.rows;
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        float d = 0.f;
#pragma unroll
        for (int e = 0; e < EPP; ++e) d += qv[r][e] * kv[e];
        d = group_sum<TL::LPK>(d);
        const bool ok = valid && (ch.compact || jl <= lim[r]);
        lg[it][r] = ok ? d * a.scale + cur.b[it] : -INFINITY;
      }
    }
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      float cm = lg[0][r];
#pragma unroll
      for (int it = 1; it < NIT; ++it) cm = fmaxf(cm, lg[it][r]);
      cm = slots_max<TL::LPK>(cm);
      const float mn = fmaxf(m[r], cm);
      const float mref = mn == -INFINITY ? 0.f : mn;
      float cs = 0.f;
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        lg[it][r] = expf(lg[it][r] - mref);
        cs += lg[it][r];
      }
      cs = slots_sum<TL::LPK>(cs);   // lanes of one slot hold the same keys: sum over the slots
      const float al = expf(m[r] - mref);
      l[r] = l[r] * al + cs;
      m[r] = mn;
#pragma unroll
      for (int e = 0; e < EPP; ++e) o[r][e] *= al;
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      float vv[EPP];
      unpack16<IT>(cur.v[it], vv);
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int e = 0; e < EPP; ++e) o[r][e] += lg[it][r] * vv[e];
    }
    cur = nxt;
  }
  // sum the key slots; lanes of slot 0 write the split's partial rows
  const long base = ((long)split * a.H + h) * R;
#pragma unroll
  for (int r = 0; r < RB; ++r) {
#pragma unroll
    for (int e = 0; e < EPP; ++e) o[r][e] = slots_sum<TL::LPK>(o[r][e]);
    if (r < R && g == 0) {
      float* op = a.opart + (base + r) * D + pl * EPP;
#pragma unroll
      for (int e = 0; e < EPP; e += 4) *(float4*)(op + e) = make_float4(o[r][e], o[r][e + 1], o[r][e + 2], o[r][e + 3]);
      if (pl == 0) {
        a.mpart[base + r] = m[r];
        a.lpart[base + r] = l[r];
      }
    }
  }
}

// out[row] = sum_s exp(m_s - M) O_s / sum_s exp(m_s - M) l_s.  One block of
// ATTEND_MERGE_WAVES waves per (row, KV head): wave w takes splits w, w + W,
// ...; every lane holds FPL features; the waves' maxima, sums and rows are
// combined through LDS.
constexpr int ATTEND_MERGE_WAVES = 8;

template <class IT, int D>
__global__ __launch_bounds__(64 * ATTEND_MERGE_WAVES) void attend_merge_kernel(ConsumerArgs a) {
  constexpr int FPL = D / 64, W = ATTEND_MERGE_WAVES;
  __shared__ float red[W];
  __shared__ float racc[W][D];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int r = blockIdx.x, h = blockIdx.y, R = a.group * a.nq;
  const long stride = (long)a.H * R;   // between consecutive splits
  const long b0 = (long)h * R + r;
  float M = -INFINITY;
  for (int s = threadIdx.x; s < a.splits; s += 64 * W) M = fmaxf(M, a.mpart[s * stride + b0]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
  if (lane == 0) red[wv] = M;
  __syncthreads();
  M = red[0];
#pragma unroll
  for (int i = 1; i < W; ++i) M = fmaxf(M, red[i]);
  const float mref = M == -INFINITY ? 0.f : M;
  float L = 0.f, acc[FPL];
#pragma unroll
  for (int u = 0; u < FPL; ++u) acc[u] = 0.f;
#pragma unroll 4
  for (int s = wv; s < a.splits; s += W) {
    const long b = s * stride + b0;
    const float w = expf(a.mpart[b] - mref);
    L += w * a.lpart[b];
    const float* op = a.opart + b * D + lane * FPL;
#pragma unroll
    for (int u = 0; u < FPL; ++u) acc[u] += w * op[u];
  }
#pragma unroll
  for (int u = 0; u < FPL; ++u) racc[wv][lane * FPL + u] = acc[u];
  __syncthreads();
  if (lane == 0) red[wv] = L;   // every lane of a wave holds the same L
  __syncthreads();
  if (wv == 0) {
    float Lt = 0.f;
#pragma unroll
    for (int i = 0; i < W; ++i) Lt += red[i];
    const float inv = Lt > 0.f ? 1.f / Lt : 0.f;
    IT* dst = (IT*)a.out + b0 * D + lane * FPL;
#pragma unroll
    for (int u = 0; u < FPL; ++u) {
      float v = 0.f;
#pragma unroll
      for (int i = 0; i < W; ++i) v += racc[i][lane * FPL + u];
      dst[u] = from_f32<IT>(v * inv);
    }
  }
}

// beta[h][i] = shape(Z_out[h*t + i] . w_beta), Z_out = Z or RMSNorm(Z); one wave per row.
struct BetaShape {
  float beta_max;     // > 0: beta_max * tanh(beta / beta_max)
  float offset;       // added last (mass matching: log(N / t) + log_x; else 0)
};

template <class WT>
__global__ __launch_bounds__(256) void beta_kernel(const float* __restrict__ Z, const WT* __restrict__ w,
                                                   long rows, int D, int final_norm, float eps, BetaShape sh,
                                                   float* __restrict__ beta) {
  const long row = blockIdx.x * 4L + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= rows) return;
  const float* z = Z + row * D;
  float dot = 0.f, ss = 0.f;
  for (int i = lane; i < D; i += 64) {
    dot += z[i] * to_f32(w[i]);
    ss += z[i] * z[i];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    dot += __shfl_xor(dot, o);
    ss += __shfl_xor(ss, o);
  }
  if (lane == 0) {
    float b = final_norm ? dot / sqrtf(ss / (float)D + eps) : dot;
    if (sh.beta_max > 0.f) b = sh.beta_max * tanhf(b / sh.beta_max);
    beta[row] = b + sh.offset;
  }
}

}  // namespace still
