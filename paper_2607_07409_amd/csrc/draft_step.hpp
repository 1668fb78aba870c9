// One DeLS-Spec draft block per sequence (Algorithm 1, the decoding loop) as a chain of
// launches per draft position j, for heads that are drafted with as they are and for prepared ones
// where the persistent kernel is the slower route:
//
//   k_gates   tokens u_j (argmax keys of position j-1), x = E[u_j], GRU cell -> h
//             (k_gates_rows: up to four sequences; k_gates_folded: a prepared head)
//   k_rank    rho = SiLU(W_rank h); further workgroups write the results of position j-1
//   k_vocab   l_S = W_vocab rho, fused with the long logits, online LSEs, top-2; one argmax
//             key and one partial per (sequence, workgroup)
//
// and k_finish for the last position.  A Markov head (rho = E_M[u_j]) needs k_vocab alone: every
// workgroup gets the tokens and stages their rows itself.  The decoded token never leaves the
// device and no launch waits for another one beyond the order of the stream.
//
// The products run on the matrix cores (those of the GRU cell and of W_rank from five sequences on), 16
// weight rows by 16 sequences at a time, with float32 accuracy (V = 151,936, d = 4,096, H = 1,024, r = 256, 32
// sequences, 16 positions in bf16: 739 us a block; one wave per weight row with vector instructions, four
// sequences at a time, took 10.5 ms, and its error against float64 was larger): a float32 activation is split
// exactly into three bf16 values of 8 significant bits (bf16 heads, v_mfma_f32_16x16x32_bf16), or multiplied as
// it is (float32 heads, v_mfma_f32_16x16x4_f32).  Products of bf16 values are exact and the sums are float32.
#pragma once
#include <atomic>

#include "dels_internal.hpp"

namespace dls {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;   // arrays of it stay in registers
// LDS is read and written through pointers of its own address space: through a generic pointer the
// compiler may merge an access with one of global memory into a FLAT access.
typedef __attribute__((address_space(3))) u32x4_t lds_u32x4;
typedef __attribute__((address_space(3))) f32x4_t lds_f32x4;
typedef __attribute__((address_space(3))) float lds_float;
__device__ __forceinline__ u32x4_t vec(uint4 v) { return u32x4_t{v.x, v.y, v.z, v.w}; }
__device__ __forceinline__ uint4 unvec(u32x4_t v) { return make_uint4(v.x, v.y, v.z, v.w); }
// LDS of a wave alone: accesses before are ordered before those after, for all its lanes
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

constexpr int kST = 512;             // threads per workgroup
constexpr int kSW = kST / 64;
constexpr int kUnits = 5;            // hidden units per gates workgroup: 15 of 16 operand rows
constexpr int kPairRows = 32;        // vocabulary rows a wave multiplies at a time (two operand tiles)

// Statistics of one (sequence, workgroup) beside its argmax key.
struct StepPart {
  float lm, ls, sm, ss, fm, fs, t2;
};

// argmax key: orderable fused value over the complement of its index (equal values: lowest index)
__device__ __forceinline__ uint64_t step_key(float t1, int i1) {
  t1 += 0.0f;   // -0 -> +0, so that equal values compare equal
  const uint32_t u = __float_as_uint(t1);
  const uint32_t o = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ((uint64_t)o << 32) | (uint32_t)~(uint32_t)i1;
}
__device__ __forceinline__ int step_key_index(uint64_t k) { return (int)~(uint32_t)k; }
__device__ __forceinline__ float step_key_value(uint64_t k) {
  const uint32_t o = (uint32_t)(k >> 32);
  return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}
__device__ __forceinline__ uint64_t u64_max(uint64_t a, uint64_t b) { return a > b ? a : b; }
template <int N>
__device__ __forceinline__ uint64_t u64_ror(uint64_t v) {   // within each row of 16 lanes
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, 0x120 + N, 0xf, 0xf, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), 0x120 + N, 0xf, 0xf, false);
  return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t wave_u64_max(uint64_t k) {
  k = u64_max(k, u64_ror<8>(k));
  k = u64_max(k, u64_ror<4>(k));
  k = u64_max(k, u64_ror<2>(k));
  k = u64_max(k, u64_ror<1>(k));
  {
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)k, (uint32_t)k, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(k >> 32), (uint32_t)(k >> 32), false, false);
    k = u64_max(((uint64_t)hi[0] << 32) | lo[0], ((uint64_t)hi[1] << 32) | lo[1]);
  }
  {
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)k, (uint32_t)k, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(k >> 32), (uint32_t)(k >> 32), false, false);
    k = u64_max(((uint64_t)hi[0] << 32) | lo[0], ((uint64_t)hi[1] << 32) | lo[1]);
  }
  return k;
}

// ----------------------------------------------------------------------------------
// Matrix-core operands.  One 16-byte piece per lane is one operand chunk of KCH columns:
// lane l holds row (or sequence) l % 16, columns KCH c + NP (l / 16) .. + NP - 1.  For float32
// the four values of a piece feed four 16x16x4 products, whose column order both operands share.
// ----------------------------------------------------------------------------------
template <typename T> struct Op;
template <> struct Op<bf16_t> {
  static constexpr int KCH = 32, NP = 8, SPL = 3;
  __device__ __forceinline__ static f32x4_t mma(uint4 a, uint4 b, f32x4_t c) {
    union { uint4 u; bf16x8_t v; } x, y;
    x.u = a;
    y.u = b;
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.v, y.v, c, 0, 0, 0);
  }
  // x = s[0] + s[1] + s[2] exactly: 8 significant bits each (truncated, so that no remainder
  // changes sign or grows).  An infinity keeps its value in s[0] alone.
  __device__ __forceinline__ static void split(const float* x, uint4* s) {
    uint32_t p[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t u[2][3];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const float v = x[2 * i + e];
        const uint32_t h = __float_as_uint(v) & 0xffff0000u;
        const float r1 = fabsf(v) < INFINITY ? v - __uint_as_float(h) : 0.f;
        const uint32_t m = __float_as_uint(r1) & 0xffff0000u;
        u[e][0] = h;
        u[e][1] = m;
        u[e][2] = __float_as_uint(r1 - __uint_as_float(m));
      }
#pragma unroll
      for (int q = 0; q < 3; ++q) p[q][i] = (u[0][q] >> 16) | (u[1][q] & 0xffff0000u);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) s[q] = make_uint4(p[q][0], p[q][1], p[q][2], p[q][3]);
  }
};
template <> struct Op<float> {
  static constexpr int KCH = 16, NP = 4, SPL = 1;
  __device__ __forceinline__ static f32x4_t mma(uint4 a, uint4 b, f32x4_t c) {
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
    return c;
  }
  __device__ __forceinline__ static void split(const float* x, uint4* s) {
    s[0] = make_uint4(__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(x[3]));
  }
};
__device__ __forceinline__ uint4 sel4(bool p, uint4 v) {
  return make_uint4(p ? v.x : 0u, p ? v.y : 0u, p ? v.z : 0u, p ? v.w : 0u);
}
// one piece of a float32 activation row (zeros unless ok), split for products with weights of type WT
template <typename WT>
__device__ __forceinline__ void act_split(const float4* v, bool ok, uint4* s) {
  float x[Op<WT>::NP];
#pragma unroll
  for (int i = 0; i < Op<WT>::NP / 4; ++i) {
    x[4 * i] = ok ? v[i].x : 0.f;
    x[4 * i + 1] = ok ? v[i].y : 0.f;
    x[4 * i + 2] = ok ? v[i].z : 0.f;
    x[4 * i + 3] = ok ? v[i].w : 0.f;
  }
  Op<WT>::split(x, s);
}
// NB chunks c .. (below c1) of a weight row and of MT float32 activation rows: loaded in one go,
// then acc[m] += their products.  Pieces past the range are zeros in both operands.
template <typename WT, int MT, int NB>
struct ActBatch {
  using O = Op<WT>;
  static constexpr int NF = O::NP / 4;
  u32x4_t w[NB];
  f32x4_t x[MT][NB][NF];
  __device__ __forceinline__ void load(const WT* wr, const float* const* xr, int K, int c, int c1, int g) {
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int kk = (c + i) * O::KCH + g * O::NP;
      const int k = c + i < c1 && kk < K ? kk : 0;
      w[i] = *reinterpret_cast<const u32x4_t*>(wr + k);
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int f = 0; f < NF; ++f) x[m][i][f] = *reinterpret_cast<const f32x4_t*>(xr[m] + k + 4 * f);
    }
  }
  __device__ __forceinline__ void use(int K, int c, int c1, int g, f32x4_t* acc) {
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const bool ok = c + i < c1 && (c + i) * O::KCH + g * O::NP < K;
      const uint4 wi = sel4(ok, make_uint4(w[i].x, w[i].y, w[i].z, w[i].w));
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        float4 v[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) v[f] = make_float4(x[m][i][f].x, x[m][i][f].y, x[m][i][f].z, x[m][i][f].w);
        uint4 s[O::SPL];
        act_split<WT>(v, ok, s);
#pragma unroll
        for (int e = O::SPL - 1; e >= 0; --e) acc[m] = O::mma(wi, s[e], acc[m]);
      }
    }
  }
};

// the tokens decoded at the position before: the largest of a sequence's G <= kMaxG keys, or the
// caller's token of the first position
struct TokenSource {
  const uint64_t* keys;     // [batch][G], or NULL: last
  const int32_t* last;
  int G;
};
// Keys of the wave's sequences b0 + wave, b0 + wave + kSW, ..: every load is issued before the
// first is waited for.
template <int NS>
struct TokenKeys {
  uint64_t k[NS][kMaxG / 64];
};
template <int NS>
__device__ __forceinline__ void load_keys(const TokenSource& ts, int b0, int batch, int wave, int lane,
                                          TokenKeys<NS>& tk) {
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int b = min(b0 + wave + s * kSW, batch - 1);
    if (ts.keys) {
#pragma unroll
      for (int i = 0; i < kMaxG / 64; ++i) tk.k[s][i] = ts.keys[(size_t)b * ts.G + min(lane + 64 * i, ts.G - 1)];
    } else {
      tk.k[s][0] = (uint32_t)~(uint32_t)ts.last[b];
#pragma unroll
      for (int i = 1; i < kMaxG / 64; ++i) tk.k[s][i] = 0;
    }
  }
}
template <int NS>
__device__ __forceinline__ void merge_keys(const TokenKeys<NS>& tk, int V, int wave, int lane, int* s_tok) {
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    uint64_t k = tk.k[s][0];
#pragma unroll
    for (int i = 1; i < kMaxG / 64; ++i) k = u64_max(k, tk.k[s][i]);
    const int t = step_key_index(wave_u64_max(k));
    if (lane == 0) s_tok[wave + s * kSW] = (unsigned)t < (unsigned)V ? t : 0;   // out of range, or every value -inf
  }
}

// ----------------------------------------------------------------------------------
// The results of one position: the G keys and parts of a sequence, merged by one workgroup.
// ----------------------------------------------------------------------------------
struct FinishArgs {
  const uint64_t* keys;
  const StepPart* parts;
  int G, j, B, batch;
  float wl, al;
  int long_only;
  int32_t* out_tokens;
  dls_row_stats* out_stats;
  Sampler smp;
  const dls_row_uncertainty* unc;
  const uint32_t* hdr;   // header of the workspace (prepared heads): a set error word gives sentinels
};
__device__ __forceinline__ void finish_row(const FinishArgs& f, int b, Partial* sh) {
  if (f.hdr && f.hdr[1] != 0u) {   // uniform
    if (threadIdx.x == 0) {
      const float nan = __builtin_nanf("");
      f.out_tokens[(size_t)b * f.B + f.j] = -1;
      if (f.out_stats) f.out_stats[(size_t)b * f.B + f.j] = dls_row_stats{nan, nan, nan, nan, nan, nan};
    }
    return;
  }
  Partial P = partial_empty();
  for (int i = threadIdx.x; i < f.G; i += kST) {
    const uint64_t k = f.keys[(size_t)b * f.G + i];
    const StepPart s = f.parts[(size_t)b * f.G + i];
    Partial Q;
    Q.L = {s.lm, s.ls};
    Q.S = {s.sm, s.ss};
    Q.F = {s.fm, s.fs};
    Q.t1 = step_key_value(k);
    Q.i1 = step_key_index(k);
    Q.t2 = s.t2;
    Q.pad = 0;
    P = partial_merge(P, Q);
  }
  P = block_merge(P, sh, kSW);
  if (threadIdx.x == 0) {
    int32_t t;
    const int ti = P.i1 == 0x7fffffff ? 0 : P.i1;
    const float alb = f.unc ? f.al * f.unc[(size_t)b * f.B + f.j].gate : f.al;
    finalize_row(P, f.wl, alb, f.long_only != 0, &t, f.out_stats ? f.out_stats + (size_t)b * f.B + f.j : nullptr,
                 nullptr, f.smp.inv_temp != 0.f ? gumbel_at(f.smp, b, f.j, ti) : 0.f, f.smp.temp);
    f.out_tokens[(size_t)b * f.B + f.j] = t;
  }
}
// the row of a further workgroup of the vocabulary launch
__device__ __forceinline__ void finish_extra(const FinishArgs& f, int G, Partial* sh) {
  const int row = (int)((blockIdx.x - G) * gridDim.y + blockIdx.y);
  if (row < f.batch) finish_row(f, row, sh);
}
// The block's last launch also clears what its launches wrote into the workspace (float32 state, keys and
// partials): the persistent kernel takes a word of a workspace for its own by the tag in its upper
// half, and its words of another batch or block length lie where these lay.  About 18 KB a sequence.
struct ClearArgs {
  float *h0, *h1, *rho;   // [batch][H], [batch][H], [batch][r]; NULL: a head without them
  int H, r;
  uint64_t* keys;         // [sets][batch][G]
  StepPart* parts;
  int sets;
};
__global__ __launch_bounds__(kST) void k_finish(FinishArgs f, ClearArgs c) {
  __shared__ Partial sh[kSW];
  const size_t b = blockIdx.x;
  finish_row(f, (int)b, sh);
  __syncthreads();
  const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
  if (c.h0) {
    for (int i = threadIdx.x; i < c.H / 4; i += kST) {
      reinterpret_cast<float4*>(c.h0 + b * c.H)[i] = z;
      reinterpret_cast<float4*>(c.h1 + b * c.H)[i] = z;
    }
    for (int i = threadIdx.x; i < c.r / 4; i += kST) reinterpret_cast<float4*>(c.rho + b * c.r)[i] = z;
  }
  for (int s = 0; s < c.sets; ++s) {
    const size_t o = ((size_t)s * f.batch + b) * f.G;
    uint32_t* p = reinterpret_cast<uint32_t*>(c.parts + o);
    for (int i = threadIdx.x; i < f.G; i += kST) c.keys[o + i] = 0ull;
    for (int i = threadIdx.x; i < f.G * (int)(sizeof(StepPart) / 4); i += kST) p[i] = 0u;
  }
}

// ----------------------------------------------------------------------------------
// GRU cell.  A workgroup owns kUnits hidden units (15 gate rows of W_ih and W_hh: one operand
// tile) and 16 MT sequences; its eight waves take an eighth of the columns each and
// add their partial products in a fixed order.
// ----------------------------------------------------------------------------------
template <typename WT>
struct GatesArgs {
  const WT *emb, *w_ih, *w_hh;
  int d, H, V, batch;
  TokenSource ts;
  const float* h_in;
  int h_zero;
  float* h_out;
};
template <typename WT, int MT>
__global__ __launch_bounds__(kST, 2) void k_gates(GatesArgs<WT> a) {
  using O = Op<WT>;
  constexpr int NW = 16, NX = MT > 1 ? 4 : 8;   // chunks of W_ih and of x in flight
  constexpr int NH = MT > 2 ? 2 : 4;            // chunks of W_hh and h
  __shared__ int s_tok[16 * MT];
  __shared__ f32x4_t red[kSW][MT][64];    // rows of r and z: input + recurrent; of n: input
  __shared__ f32x4_t redn[kSW][MT][32];   // rows 8 to 15: recurrent (rows of n: 10 to 14)
  static_assert(kUnits * 3 <= 16 && kUnits * 2 >= 8, "operand rows of the n gate lie in the upper half");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 15, g = lane >> 4;
  const int b0 = blockIdx.y * 16 * MT;
  const int d = a.d, H = a.H;
  const int u0 = blockIdx.x * kUnits;
  const int q = min(n / kUnits, 2), unit = min(u0 + n % kUnits, H - 1);   // row n of the operand tile
  f32x4_t ax[MT], ah[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) ax[m] = ah[m] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  TokenKeys<2 * MT> tk;
  load_keys(a.ts, b0, a.batch, wave, lane, tk);
  asm volatile("" ::: "memory");
  // everything that does not depend on the tokens is asked for while their keys are on the way
  const int nch = (H + O::KCH - 1) / O::KCH;
  const int ch0 = nch * wave / kSW, ch1 = nch * (wave + 1) / kSW;
  const WT* wh = a.w_hh + (size_t)(q * H + unit) * H;
  const float* hr[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) hr[m] = a.h_in + (size_t)min(b0 + 16 * m + n, a.batch - 1) * H;
  ActBatch<WT, MT, NH> hb;
  if (!a.h_zero) hb.load(wh, hr, H, ch0, ch1, g);
  const int ncx = (d + O::KCH - 1) / O::KCH;
  const int cx0 = ncx * wave / kSW, cx1 = ncx * (wave + 1) / kSW;
  const WT* wx = a.w_ih + (size_t)(q * H + unit) * d;
  auto col = [&](int c) {   // first column of the lane's piece of chunk c (0 past the wave's range)
    const int k = c * O::KCH + g * O::NP;
    return c < cx1 && k < d ? k : 0;
  };
  uint4 w[NW];
  auto load_wx = [&](int c) {
#pragma unroll
    for (int i = 0; i < NW; ++i) w[i] = *reinterpret_cast<const uint4*>(wx + col(c + i));
  };
  load_wx(cx0);
  asm volatile("" ::: "memory");
  merge_keys(tk, a.V, wave, lane, s_tok);
  __syncthreads();
  const WT* xr[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) xr[m] = a.emb + (size_t)s_tok[16 * m + n] * d;
  uint4 x[MT][NX];
  auto load_x = [&](int c) {
#pragma unroll
    for (int i = 0; i < NX; ++i)
#pragma unroll
      for (int m = 0; m < MT; ++m) x[m][i] = *reinterpret_cast<const uint4*>(xr[m] + col(c + i));
  };
  load_x(cx0);
  asm volatile("" ::: "memory");
  if (!a.h_zero) {
    hb.use(H, ch0, ch1, g, ah);
    for (int c = ch0 + NH; c < ch1; c += NH) {
      hb.load(wh, hr, H, c, ch1, g);
      hb.use(H, c, ch1, g, ah);
    }
  }
  for (int c = cx0; c < cx1; c += NW) {
    if (c > cx0) load_wx(c);
#pragma unroll
    for (int h = 0; h < NW / NX; ++h) {
      if (c + h * NX < cx1) {
        if (c > cx0 || h) load_x(c + h * NX);
#pragma unroll
        for (int i = 0; i < NX; ++i) {
          const int ci = c + h * NX + i;
          const bool ok = ci < cx1 && ci * O::KCH + g * O::NP < d;
          const uint4 wi = sel4(ok, w[h * NX + i]);
#pragma unroll
          for (int m = 0; m < MT; ++m) ax[m] = O::mma(wi, sel4(ok, x[m][i]), ax[m]);
        }
      }
    }
  }
  // D layout: lane 16 (row / 4) + column holds row % 4 of its four values
#pragma unroll
  for (int m = 0; m < MT; ++m) {
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wave][m][lane][e] = 4 * g + e < 2 * kUnits ? ax[m][e] + ah[m][e] : ax[m][e];
    if (lane >= 32) redn[wave][m][lane - 32] = ah[m];
  }
  __syncthreads();
  for (int i = tid; i < 16 * MT * kUnits; i += kST) {
    const int s = i % (16 * MT), u = i / (16 * MT);
    const int b = b0 + s;
    if (b >= a.batch || u0 + u >= H) continue;
    const float hp = a.h_zero ? 0.f : a.h_in[(size_t)b * H + u0 + u];
    float sx[3], sn = 0.f;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      const int row = e * kUnits + u;
      const int l = 16 * (row >> 2) + (s & 15);
      sx[e] = 0.f;
#pragma unroll
      for (int v = 0; v < kSW; ++v) {
        sx[e] += red[v][s >> 4][l][row & 3];
        if (e == 2) sn += redn[v][s >> 4][l - 32][row & 3];
      }
    }
    const float rg = sigmoidf_(sx[0]), zg = sigmoidf_(sx[1]);
    const float ng = tanhf_(sx[2] + rg * sn);
    a.h_out[(size_t)b * H + u0 + u] = (1.f - zg) * ng + zg * hp;
  }
}

// GRU cell of up to four sequences, where a sixteenth to a quarter of the matrix cores' columns would count: one
// wave per hidden unit reads its six weight rows in memory order, 1 KB per instruction, those of W_ih kU
// pieces ahead of the tokens and of their use.  k_gates reads 16 rows at the same columns per instruction, which
// meet in one memory channel where the row length is a large power of two.  us a block of 16 positions by k_gates and
// k_rank and by the row kernels (batch 1 / 4): d = 4,096, H = 1,024, V = 151,936, r = 256, bf16 530 / 545 and
// 496 / 555; d = 4,096, H = 512, float32 554 / 566 and 365 / 422; d = 16,384, H = 64, float32 1,070 / 1,168 and
// 416 / 628; d = 512, H = 4,096, bf16 1,050 / 1,096 and 497 / 634; d = 128, H = 256, bf16 329 / 338 and 259 / 295.
constexpr int kRT = 256;
template <typename WT, int NB>
__global__ __launch_bounds__(kRT) void k_gates_rows(GatesArgs<WT> a) {
  constexpr int N = Op<WT>::NP, kU = 4;
  __shared__ int s_tok[kRT / 64];
  static_assert(NB <= kRT / 64, "a wave merges the keys of one sequence");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int d = a.d, H = a.H;
  const int k = min((int)blockIdx.x * (kRT / 64) + wave, H - 1);   // past H: the last unit again, not stored
  TokenKeys<1> tk;
  load_keys(a.ts, 0, a.batch, wave, lane, tk);
  asm volatile("" ::: "memory");
  float acc[4][NB];   // r, z, n from x, n from h
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[0][b] = acc[1][b] = acc[2][b] = acc[3][b] = 0.f;
  auto fma_row = [&](float& s, uint4 w, const float* x) {
    float wv[N];
    Chunk<WT>::widen(w, wv);
#pragma unroll
    for (int i = 0; i < N; ++i) s = __builtin_fmaf(wv[i], x[i], s);
  };
  const int np = d / N, nh = H / N;
  uint4 w[3][kU];
  auto load_w = [&](const WT* m, int cols, int n, int p) {   // pieces p + lane, + 64, ..
#pragma unroll
    for (int u = 0; u < kU; ++u)
#pragma unroll
      for (int q = 0; q < 3; ++q)
        w[q][u] = *reinterpret_cast<const uint4*>(m + (size_t)(q * H + k) * cols + (size_t)min(p + u * 64 + lane, n - 1) * N);
  };
  load_w(a.w_ih, d, np, 0);
  asm volatile("" ::: "memory");
  merge_keys(tk, a.V, wave, lane, s_tok);
  __syncthreads();
  const WT* xr[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) xr[b] = a.emb + (size_t)s_tok[b] * d;
  for (int p = 0; p < np; p += 64 * kU) {
    uint4 x[NB][kU];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int u = 0; u < kU; ++u) x[b][u] = *reinterpret_cast<const uint4*>(xr[b] + (size_t)min(p + u * 64 + lane, np - 1) * N);
    uint4 c[3][kU];
#pragma unroll
    for (int u = 0; u < kU; ++u)
#pragma unroll
      for (int q = 0; q < 3; ++q) c[q][u] = w[q][u];
    if (p + 64 * kU < np) load_w(a.w_ih, d, np, p + 64 * kU);
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      if (p + u * 64 + lane < np) {   // not the clamped pieces: a zero would not take an infinite weight out
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          float xv[N];
          Chunk<WT>::widen(x[b][u], xv);
#pragma unroll
          for (int q = 0; q < 3; ++q) fma_row(acc[q][b], c[q][u], xv);
        }
      }
    }
  }
  if (!a.h_zero) {
    const WT* u0 = a.w_hh + (size_t)k * H;
#pragma unroll 2
    for (int p = lane; p < nh; p += 64) {
      uint4 u[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) u[q] = *reinterpret_cast<const uint4*>(u0 + (size_t)q * H * H + (size_t)p * N);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const float* hp = a.h_in + (size_t)min(b, a.batch - 1) * H + (size_t)p * N;
        float hv[N];
#pragma unroll
        for (int i = 0; i < N; ++i) hv[i] = hp[i];
        fma_row(acc[0][b], u[0], hv);
        fma_row(acc[1][b], u[1], hv);
        fma_row(acc[3][b], u[2], hv);
      }
    }
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) {
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q][b] = wave_sum(acc[q][b]);
    if (lane == 0 && b < a.batch && (int)blockIdx.x * (kRT / 64) + wave < H) {
      const float rg = sigmoidf_(acc[0][b]), zg = sigmoidf_(acc[1][b]);
      const float ng = tanhf_(acc[2][b] + rg * acc[3][b]);
      const float hp = a.h_zero ? 0.f : a.h_in[(size_t)b * H + k];
      a.h_out[(size_t)b * H + k] = (1.f - zg) * ng + zg * hp;
    }
  }
}

// A prepared buffer of another head sets the error word, whatever it held (as the persistent kernel does).
template <typename WT>   // bf16_t
__global__ void k_check_prepared(const PreparedHeader* prep, PreparedHeader ex, uint32_t* hdr) {
  const bool same = prep->magic == ex.magic && prep->V == ex.V && prep->d == ex.d && prep->H == ex.H && prep->r == ex.r &&
                    prep->emb == ex.emb && prep->w_ih == ex.w_ih && prep->w_hh == ex.w_hh && prep->w_vocab == ex.w_vocab;
  if (!same) hdr[1] = kErrPrepared;
}

// GRU cell of a prepared head: the input products come from the folded table, W_hh in operand
// order.  A workgroup owns 16 hidden units (three operand tiles) and 16 sequences; the waves take
// an eighth of the columns each.  Bound by latency: the keys of the position before, the rows of T
// from HBM; W_hh and h are on their way meanwhile.
struct FoldedArgs {
  const float* T;
  const uint4* whh;
  int H, V, batch;
  TokenSource ts;
  const float* h_in;
  int h_zero;
  float* h_out;
};
template <typename WT>   // bf16_t: a template, so that only the units of bf16 heads hold it
__global__ __launch_bounds__(kST, 2) void k_gates_folded(FoldedArgs a) {
  using O = Op<WT>;
  constexpr int NB = 4;   // chunks in flight
  __shared__ int s_tok[16];
  __shared__ f32x4_t red[kSW][3][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 15, g = lane >> 4;
  const int b0 = blockIdx.y * 16, H = a.H, nc = H / 32;
  TokenKeys<2> tk;
  load_keys(a.ts, b0, a.batch, wave, lane, tk);
  asm volatile("" ::: "memory");
  const int c0 = nc * wave / kSW, c1 = nc * (wave + 1) / kSW;
  const u32x4_t* wp = reinterpret_cast<const u32x4_t*>(a.whh) + (size_t)blockIdx.x * 3 * nc * 64 + lane;
  const float* hr = a.h_in + (size_t)min(b0 + n, a.batch - 1) * H + 8 * g;
  f32x4_t acc[3];
  acc[0] = acc[1] = acc[2] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  u32x4_t w[3][NB];
  f32x4_t x[NB][2];
  auto load = [&](int c) {
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int ci = min(c + i, nc - 1);
#pragma unroll
      for (int q = 0; q < 3; ++q) w[q][i] = wp[((size_t)q * nc + ci) * 64];
      x[i][0] = *reinterpret_cast<const f32x4_t*>(hr + 32 * ci);
      x[i][1] = *reinterpret_cast<const f32x4_t*>(hr + 32 * ci + 4);
    }
  };
  if (!a.h_zero) load(c0);
  const int u = tid & 15, s = tid >> 4, b = b0 + s, unit = blockIdx.x * 16 + u;   // tid < 256
  const bool mine = tid < 256 && b < a.batch;
  const float hp = mine && !a.h_zero ? a.h_in[(size_t)b * H + unit] : 0.f;
  asm volatile("" ::: "memory");
  merge_keys(tk, a.V, wave, lane, s_tok);
  __syncthreads();
  float gi[3] = {0.f, 0.f, 0.f};
  if (mine) {
#pragma unroll
    for (int q = 0; q < 3; ++q) gi[q] = a.T[(size_t)s_tok[s] * 3 * H + q * H + unit];
  }
  if (!a.h_zero) {
    for (int c = c0; c < c1; c += NB) {
      if (c > c0) load(c);
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        if (c + i < c1) {   // wave-uniform
          const float4 v[2] = {make_float4(x[i][0].x, x[i][0].y, x[i][0].z, x[i][0].w),
                               make_float4(x[i][1].x, x[i][1].y, x[i][1].z, x[i][1].w)};
          uint4 sp[O::SPL];
          act_split<WT>(v, true, sp);
#pragma unroll
          for (int e = O::SPL - 1; e >= 0; --e)
#pragma unroll
            for (int q = 0; q < 3; ++q)
              acc[q] = O::mma(make_uint4(w[q][i].x, w[q][i].y, w[q][i].z, w[q][i].w), sp[e], acc[q]);
        }
      }
    }
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) red[wave][q][lane] = acc[q];
  __syncthreads();
  if (mine) {
    const int l = 16 * (u >> 2) + s;
    float gh[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      gh[q] = 0.f;
#pragma unroll
      for (int v = 0; v < kSW; ++v) gh[q] += red[v][q][l][u & 3];
    }
    const float rg = sigmoidf_(gi[0] + gh[0]), zg = sigmoidf_(gi[1] + gh[1]);
    const float ng = tanhf_(gi[2] + rg * gh[2]);
    a.h_out[(size_t)b * H + unit] = (1.f - zg) * ng + zg * hp;
  }
}

// ----------------------------------------------------------------------------------
// rho = SiLU(W_rank h), 16 rank rows by 16 sequences per workgroup (columns split over the
// waves); the workgroups after them write the results of the position before (fin.batch of
// them, none at the first position).
// ----------------------------------------------------------------------------------
template <typename WT>
struct RankArgs {
  const WT* w_rank;
  int H, r, batch, tiles;   // tiles = ceil(r / 16) * ceil(batch / 16)
  const float* h;
  float* rho;
};
template <typename WT>
__global__ __launch_bounds__(kST) void k_rank(RankArgs<WT> a, FinishArgs fin) {
  using O = Op<WT>;
  __shared__ f32x4_t red[kSW][64];
  __shared__ Partial sh[kSW];
  if ((int)blockIdx.x >= a.tiles) {
    finish_row(fin, blockIdx.x - a.tiles, sh);
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 15, g = lane >> 4;
  const int rt = (a.r + 15) >> 4;
  const int r0 = (blockIdx.x % rt) * 16, b0 = (blockIdx.x / rt) * 16;
  const WT* wr = a.w_rank + (size_t)min(r0 + n, a.r - 1) * a.H;
  const float* hr = a.h + (size_t)min(b0 + n, a.batch - 1) * a.H;
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
  const int nc = (a.H + O::KCH - 1) / O::KCH;
  const int c0 = nc * wave / kSW, c1 = nc * (wave + 1) / kSW;
  for (int c = c0; c < c1; c += 4) {
    ActBatch<WT, 1, 4> hb;
    hb.load(wr, &hr, a.H, c, c1, g);
    hb.use(a.H, c, c1, g, &acc);
  }
  red[wave][lane] = acc;
  __syncthreads();
  if (tid < 256) {
    const int row = tid & 15, s = tid >> 4;
    const int l = 16 * (row >> 2) + s;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < kSW; ++w) v += red[w][l][row & 3];
    if (b0 + s < a.batch && r0 + row < a.r) a.rho[(size_t)(b0 + s) * a.r + r0 + row] = siluf_(v);
  }
}

// The same for a few sequences (batch <= NB): one wave per rank row.
template <typename WT, int NB>
__global__ __launch_bounds__(kST) void k_rank_rows(RankArgs<WT> a, FinishArgs fin) {
  constexpr int N = Op<WT>::NP;
  __shared__ Partial sh[kSW];
  if ((int)blockIdx.x >= a.tiles) {   // tiles = ceil(r / kSW)
    finish_row(fin, blockIdx.x - a.tiles, sh);
    return;
  }
  const int lane = threadIdx.x & 63, i = blockIdx.x * kSW + (threadIdx.x >> 6);
  if (i >= a.r) return;
  const WT* wr = a.w_rank + (size_t)i * a.H;
  float acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[b] = 0.f;
#pragma unroll 4
  for (int p = lane; p < a.H / N; p += 64) {
    float w[N];
    Chunk<WT>::load(wr + (size_t)p * N, w);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const float* hp = a.h + (size_t)min(b, a.batch - 1) * a.H + (size_t)p * N;
#pragma unroll
      for (int e = 0; e < N; ++e) acc[b] = __builtin_fmaf(w[e], hp[e], acc[b]);
    }
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const float s = wave_sum(acc[b]);
    if (lane == 0 && b < a.batch) a.rho[(size_t)b * a.r + i] = siluf_(s);
  }
}

// ----------------------------------------------------------------------------------
// Vocabulary head and fusion.
// ----------------------------------------------------------------------------------
template <typename WT, typename LT>
struct VocabArgs {
  const WT* w_vocab;
  const uint4* wv;               // the same in operand order (a prepared head), or NULL
  int V, r, batch, G, np;        // np = ceil(V / kPairRows)
  const float* rho;              // RNN head
  const WT* e_m;                 // Markov head (then ts holds the tokens)
  TokenSource ts;
  const LT* L;                   // row of sequence 0 at this position
  size_t bstride;
  const float* prior;
  float wl, al, be;
  int long_only;
  int j, B;
  Sampler smp;
  const dls_row_uncertainty* unc;
  uint64_t* keys;
  StepPart* parts;
  int stats;                     // log-sum-exps are wanted
  int finish;                    // the results of the position before are written by: 0 nobody, 1 the workgroups,
                                 // at their end, 2 further workgroups (blockIdx.x >= G)
};

struct __attribute__((packed, aligned(2))) Raw16 { uint32_t x, y, z, w; };
// eight consecutive long logits (any alignment of the element type)
__device__ __forceinline__ void load8(const bf16_t* p, uint4* o) {
  const Raw16 v = *reinterpret_cast<const Raw16*>(p);
  o[0] = make_uint4(v.x, v.y, v.z, v.w);
}
struct __attribute__((packed, aligned(4))) Raw32 { uint32_t v[8]; };
__device__ __forceinline__ void load8(const float* p, uint4* o) {
  const Raw32 v = *reinterpret_cast<const Raw32*>(p);
  o[0] = make_uint4(v.v[0], v.v[1], v.v[2], v.v[3]);
  o[1] = make_uint4(v.v[4], v.v[5], v.v[6], v.v[7]);
}
__device__ __forceinline__ void widen8(const uint4* o, float* x, bf16_t) { Chunk<bf16_t>::widen(o[0], x); }
__device__ __forceinline__ void widen8(const uint4* o, float* x, float) {
  Chunk<float>::widen(o[0], x);
  Chunk<float>::widen(o[1], x + 4);
}

// one lane's running statistics of one sequence (finite-start log-sum-exps)
__device__ __forceinline__ void push8(Lse& a, const float* x) {
  const float m = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
  lse_fold_fin<8>(a, x, m);
}

// a finite-start state without an entry becomes the empty one (a NaN sum is kept)
__device__ __forceinline__ void close_lse(Lse& a) { a.m = a.s == 0.f ? -INFINITY : a.m; }

// The same for a sum of exp2(x log2(e) + neg), neg = -m log2(e) rounded: the rounding is taken out of the sum
// (of magnitudes where it is small beside 1).
__device__ __forceinline__ void close_ref(Lse& a, float neg) {
  if (fabsf(a.m) < 1.0e6f) a.s *= fast_exp2(-__builtin_fmaf(a.m, kLog2e, neg));
  close_lse(a);
}

template <int N>
struct PermN {   // N consecutive lanes
  template <typename F>
  __device__ __forceinline__ void each(F f) const {
#pragma unroll
    for (int m = N / 2; m >= 1; m >>= 1) f(m);
  }
  __device__ __forceinline__ float operator()(float v, int m) const { return __shfl_xor(v, m); }
  __device__ __forceinline__ int i(int v, int m) const { return __shfl_xor(v, m); }
};
struct Perm4Rows {   // lanes l, l ^ 16, l ^ 32, l ^ 48
  template <typename F>
  __device__ __forceinline__ void each(F f) const {
    f(32);
    f(16);
  }
  __device__ __forceinline__ float operator()(float v, int m) const { return __shfl_xor(v, m); }
  __device__ __forceinline__ int i(int v, int m) const { return __shfl_xor(v, m); }
};

// r above 256: the activations of 16 MT sequences stay in LDS as operands, and KCB chunks of a pair
// of tiles are loaded at a time (nkb rounds cover r).
template <typename WT, typename LT, int MT, int KCB, int SPL, bool SAMPLE>
__global__ __launch_bounds__(kST, 2) void k_vocab_any(VocabArgs<WT, LT> a, FinishArgs fin, int nkb) {
  using O = Op<WT>;
  constexpr int NL = sizeof(LT) == 2 ? 1 : 2;   // 16-byte pieces of eight long logits
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ int s_tok[16 * MT];
  if ((int)blockIdx.x >= a.G) {
    finish_extra(fin, a.G, reinterpret_cast<Partial*>(smem));
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 15, g = lane >> 4;
  const int b0 = blockIdx.y * 16 * MT;
  const int V = a.V, r = a.r;
  const int gw = blockIdx.x * kSW + wave, tw = a.G * kSW;
  const int p0 = (int)((int64_t)a.np * gw / tw), p1 = (int)((int64_t)a.np * (gw + 1) / tw);

  // Rows of a pair: lane row n of tile i is vocabulary row 32 p + 8 (n / 4) + 4 i + n % 4, so that
  // a lane's results (rows 4g + e of both tiles) are the eight consecutive entries 32 p + 8 g + ..
  struct Pair {
    uint4 A[2][KCB];
    uint4 L[MT][NL];
  };
  auto load_w = [&](Pair& t, int p, int kb) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = min(kPairRows * p + 8 * (n >> 2) + 4 * i + (n & 3), V - 1);
      const WT* wr = a.w_vocab + (size_t)row * r;
#pragma unroll
      for (int c = 0; c < KCB; ++c) {
        const int k = (kb * KCB + c) * O::KCH + g * O::NP;
        t.A[i][c] = *reinterpret_cast<const uint4*>(wr + (k < r ? k : 0));
      }
    }
  };
  auto load_pair = [&](Pair& t, int p) {
    if (p >= p1) return;
    if (kPairRows * (p + 1) <= V) {
#pragma unroll
      for (int m = 0; m < MT; ++m)
        load8(a.L + (size_t)min(b0 + 16 * m + n, a.batch - 1) * a.bstride + kPairRows * p + 8 * g, t.L[m]);
    }
    if (!a.long_only) load_w(t, p, 0);
  };
  const bool rfull = r == nkb * KCB * O::KCH;
  Pair t0;

  // activations of the 16 MT sequences as operands in LDS: [m][chunk][split][lane] of 16 bytes.
  // Loads return in order: the activations are asked for before the weights, which then arrive
  // while the operands are staged.
  lds_u32x4* s_b = (lds_u32x4*)smem;
  const int kc = nkb * KCB;
  auto put = [&](int i, const uint4* o) {
    const int s = i / (kc * 4), pc = i % (kc * 4);
#pragma unroll
    for (int e = 0; e < SPL; ++e)
      s_b[(((s >> 4) * kc + (pc >> 2)) * SPL + e) * 64 + 16 * (pc & 3) + (s & 15)] = vec(o[e]);
  };
  auto piece_ok = [&](int i) { return (i % (kc * 4)) * O::NP < r && b0 + i / (kc * 4) < a.batch; };
  auto piece_col = [&](int i) { return (i % (kc * 4)) * O::NP < r ? (i % (kc * 4)) * O::NP : 0; };
  constexpr int NQ = (16 * MT * KCB * 4 + kST - 1) / kST, NF = O::NP / 4;   // pieces per thread of one round
  const int pieces = a.long_only ? 0 : 16 * MT * kc * 4;
  if (!a.long_only && a.e_m) {
    TokenKeys<2 * MT> tk;
    load_keys(a.ts, b0, a.batch, wave, lane, tk);
    asm volatile("" ::: "memory");
    load_pair(t0, p0);
    asm volatile("" ::: "memory");
    merge_keys(tk, V, wave, lane, s_tok);
    __syncthreads();
    for (int i = tid; i < pieces; i += kST) {
      const uint4 o = sel4(piece_ok(i), *reinterpret_cast<const uint4*>(a.e_m + (size_t)s_tok[i / (kc * 4)] * r + piece_col(i)));
      put(i, &o);
    }
  } else {
    float4 v[NQ][NF];
    const float* rho0 = a.rho;
    if (!a.long_only) {
#pragma unroll
      for (int qi = 0; qi < NQ; ++qi) {
        const int i = min(tid + qi * kST, pieces - 1);
        const float* row = rho0 + (size_t)min(b0 + i / (kc * 4), a.batch - 1) * r + piece_col(i);
#pragma unroll
        for (int f = 0; f < NF; ++f) v[qi][f] = *reinterpret_cast<const float4*>(row + 4 * f);
      }
      asm volatile("" ::: "memory");
    }
    load_pair(t0, p0);
    if (!a.long_only) {
      asm volatile("" ::: "memory");
#pragma unroll
      for (int qi = 0; qi < NQ; ++qi) {
        const int i = tid + qi * kST;
        uint4 o[O::SPL];
        act_split<WT>(v[qi], i < pieces && piece_ok(i), o);
        if (i < pieces) put(i, o);
      }
      for (int i = tid + NQ * kST; i < pieces; i += kST) {   // r > 256 (bf16) or 128 (float32)
        const float* row = rho0 + (size_t)min(b0 + i / (kc * 4), a.batch - 1) * r + piece_col(i);
        float4 t[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) t[f] = *reinterpret_cast<const float4*>(row + 4 * f);
        uint4 o[O::SPL];
        act_split<WT>(t, piece_ok(i), o);
        put(i, o);
      }
    }
  }
  __syncthreads();

  Partial P[MT];
  float alb[MT], beb[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    P[m] = partial_empty();
    P[m].L.m = P[m].S.m = P[m].F.m = kFinMin;
    const int b = min(b0 + 16 * m + n, a.batch - 1);
    const float gt = a.unc ? a.unc[(size_t)b * a.B + a.j].gate : 1.f;
    alb[m] = a.al * gt;
    beb[m] = a.be * gt;
  }

  auto process = [&](Pair& t, int p) {
    const int v0 = kPairRows * p + 8 * g;
    const bool whole = kPairRows * (p + 1) <= V;   // uniform
    float pr[8];
    if (whole && a.prior) {
#pragma unroll
      for (int e = 0; e < 8; ++e) pr[e] = a.prior[v0 + e];
    }
    uint4 lraw[MT][NL];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int i = 0; i < NL; ++i) lraw[m][i] = t.L[m][i];
    f32x4_t acc[MT][2];
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[m][0] = acc[m][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (!a.long_only) {
      for (int kb = 0; kb < nkb; ++kb) {
        if (kb) load_w(t, p, kb);
        if (!rfull) {   // columns past r: zero in both operands
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int c = 0; c < KCB; ++c) t.A[i][c] = sel4((kb * KCB + c) * O::KCH + g * O::NP < r, t.A[i][c]);
        }
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          const lds_u32x4* sb = s_b + (m * kc + kb * KCB) * SPL * 64 + lane;
#pragma unroll
          for (int c = 0; c < KCB; ++c)
#pragma unroll
            for (int e = SPL - 1; e >= 0; --e) {
              const uint4 bb = unvec(sb[(c * SPL + e) * 64]);
              acc[m][0] = O::mma(t.A[0][c], bb, acc[m][0]);
              acc[m][1] = O::mma(t.A[1][c], bb, acc[m][1]);
            }
        }
      }
    }
    load_pair(t, p + 1);   // in flight during the fold
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      float x[8], s[8], f[8];
      const int b = b0 + 16 * m + n;
      if (whole) {
        widen8(lraw[m], x, LT());
      } else {
        const LT* lr = a.L + (size_t)min(b, a.batch - 1) * a.bstride;
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = to_f32(lr[min(v0 + e, V - 1)]);
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        s[e] = acc[m][e >> 2][e & 3];
        f[e] = a.wl == 0.f ? 0.f : a.wl * x[e];
      }
      if (!a.long_only) {
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = __builtin_fmaf(alb[m], s[e], f[e]);
        if (a.prior) {
#pragma unroll
          for (int e = 0; e < 8; ++e) f[e] = minus_weighted(f[e], beb[m], whole ? pr[e] : a.prior[min(v0 + e, V - 1)]);
        }
      }
      if (SAMPLE) {
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] *= a.smp.inv_temp;
      }
      if (!whole) {   // entries past the vocabulary (lanes past the batch repeat its last sequence)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const bool in = v0 + e < V;
          x[e] = in ? x[e] : -INFINITY;
          s[e] = in ? s[e] : -INFINITY;
          f[e] = in ? f[e] : -INFINITY;
        }
      }
      push8(P[m].L, x);
      if (!a.long_only) push8(P[m].S, s);
      push8(P[m].F, f);
      if (SAMPLE) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint4 w4 = philox_row(a.smp, b, a.j, v0 + 4 * h);
          f[4 * h] += gumbel_from_word(w4.x);
          f[4 * h + 1] += gumbel_from_word(w4.y);
          f[4 * h + 2] += gumbel_from_word(w4.z);
          f[4 * h + 3] += gumbel_from_word(w4.w);
        }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) top2_push(P[m], f[e], v0 + e);
    }
  };
  for (int p = p0; p < p1; ++p) process(t0, p);

  // merge: the four row groups of a wave, then the eight waves through LDS
  __syncthreads();
  Partial* sp = reinterpret_cast<Partial*>(smem);   // [wave][16 MT]
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    close_lse(P[m].L);
    close_lse(P[m].S);
    close_lse(P[m].F);
    const Partial Q = allred_partial(P[m], Perm4Rows{});
    if (g == 0) sp[wave * 16 * MT + 16 * m + n] = Q;
  }
  __syncthreads();
  for (int i = tid; i < 16 * MT * kSW; i += kST) {   // whole waves
    const int s = i >> 3, w = i & 7;
    const Partial Q = allred_partial(sp[w * 16 * MT + s], PermN<8>{});
    if (w == 0 && b0 + s < a.batch) {
      const size_t o = (size_t)(b0 + s) * a.G + blockIdx.x;
      a.keys[o] = step_key(Q.t1, Q.i1);
      a.parts[o] = StepPart{Q.L.m, Q.L.s, Q.S.m, Q.S.s, Q.F.m, Q.F.s, Q.t2};
    }
  }
  if (a.finish == 1 && blockIdx.y == 0) {   // uniform; G >= batch
    __syncthreads();
    if ((int)blockIdx.x < a.batch) finish_row(fin, blockIdx.x, sp);
  }
}

// ----------------------------------------------------------------------------------
// Vocabulary head for r <= 256.  Every wave keeps the activations of one tile of 16 sequences in
// registers as operands (KC chunks of SPL values) and folds one vocabulary tile of 16 rows at a
// time.  MT tiles of sequences share a workgroup: wave w serves sequence tile w % MT and, of the
// NSTR = 8 / MT vocabulary tiles of a step, tile w / MT.
//
// The stream of weights bounds the loop, so each weight is loaded once per workgroup, PD steps
// ahead and in memory order (whole kilobytes per instruction: 6.3 TB/s of a 78 MB matrix that is
// read over and over, against 5.2 TB/s for operand-shaped loads of 16 rows by 64 bytes), and turned
// into operands through LDS.  Every other position runs through the steps backwards, so that the
// end of the matrix is still in L2 (7.9 TB/s).
//
// LDS slot of a piece (row m of the tile, piece pc of the row): 16 pc + (m ^ pc % 16), so that
// neither the row-wise stores nor the operand-wise reads meet in a bank.
// ----------------------------------------------------------------------------------
template <typename LT> struct Four;
template <> struct Four<bf16_t> {   // four consecutive long logits at any alignment of their type
  struct __attribute__((packed, aligned(2))) raw { uint32_t x, y; };
  typedef uint2 type;
  __device__ __forceinline__ static type load(const bf16_t* p) {
    const raw v = *reinterpret_cast<const raw*>(p);
    return make_uint2(v.x, v.y);
  }
  __device__ __forceinline__ static void widen(type v, float* x) {
    x[0] = bf16_lo(v.x);
    x[1] = bf16_hi(v.x);
    x[2] = bf16_lo(v.y);
    x[3] = bf16_hi(v.y);
  }
};
template <> struct Four<float> {
  struct __attribute__((packed, aligned(4))) raw { float x, y, z, w; };
  typedef float4 type;
  __device__ __forceinline__ static type load(const float* p) {
    const raw v = *reinterpret_cast<const raw*>(p);
    return make_float4(v.x, v.y, v.z, v.w);
  }
  __device__ __forceinline__ static void widen(type v, float* x) {
    x[0] = v.x;
    x[1] = v.y;
    x[2] = v.z;
    x[3] = v.w;
  }
};
// weighted(w, x) in one instruction: w x, and 0 where w is 0, whatever x (-inf masks and NaN included)
__device__ __forceinline__ float mul_weight(float w, float x) {
  float r;
  asm("v_mul_legacy_f32 %0, %1, %2" : "=v"(r) : "s"(w), "v"(x));
  return r;
}
constexpr int kPriorTiles = 128;   // tiles of prior entries a workgroup keeps in LDS (8 KB)
template <int MT, int KC>
struct VocabPlan {
  static constexpr int NSTR = kSW / MT;                           // tiles per step
  static constexpr int NP = NSTR * KC / kSW;                      // 16-byte pieces per thread and step
  // Steps in flight, as deep as pays: none of these spills, and one or two steps more do (12 to 60
  // registers) without being faster where they do not.  us a block at V = 151,936, H = 1,024, r = 256 in bf16, these
  // and 2, 3, 6, 8: prepared batch 64 651 and 676, sampled 756 and 783, batch 32 515 and 529; unprepared
  // batch 32 361 and 392, 1 263 and 269 (8 positions).  r = 128, H = 512, batch 64: 554 and 581.
  static constexpr int PD = NP >= 8 ? 1 : NP >= 4 ? 2 : 4;
  static constexpr int kTile = KC * 64;                           // pieces of a tile in LDS
  static constexpr int kBufs = MT == 1 ? 1 : 2;                   // a wave alone needs no second buffer
  static constexpr size_t kLds = (size_t)kBufs * NSTR * kTile * 16;
  static constexpr size_t act(int spl) { return (size_t)MT * KC * spl * 1024; }
};

// PACKED: the weights are in operand order already (KC chunks a tile), else rows of r columns.
// STATS: with the log-sum-exps; a call for tokens alone goes without (prepared heads, where it matters beside the
// persistent kernel, which does so too: batch 64 at V = 151,936, r = 256 590 us a block, with them 676; a uniform branch
// instead costs sampled calls with statistics 3%).
template <typename WT, typename LT, int MT, int KC, int SPL, bool SAMPLE, bool PACKED, bool STATS>
__global__ __launch_bounds__(kST, 2) void k_vocab(VocabArgs<WT, LT> a, FinishArgs fin) {
  using O = Op<WT>;
  using PL = VocabPlan<MT, KC>;
  constexpr int NSTR = PL::NSTR, NP = PL::NP, PD = PL::PD, NF = O::NP / 4, kTile = PL::kTile;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ int s_tok[16 * MT];
  if ((int)blockIdx.x >= a.G) {
    finish_extra(fin, a.G, reinterpret_cast<Partial*>(smem));
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, g = lane >> 4;
  const int b0 = blockIdx.y * 16 * MT;
  const int V = a.V, r = a.r, pr = r / O::NP;   // pieces of a row
  const uint32_t nt = (uint32_t)(V + 15) >> 4;
  const int T0 = (int)(nt * blockIdx.x / (uint32_t)a.G), T1 = (int)(nt * (blockIdx.x + 1) / (uint32_t)a.G);
  const int steps = (T1 - T0 + NSTR - 1) / NSTR;
  const int mt = wave % MT, str = wave / MT;
  const int b = b0 + 16 * mt + n, bc = min(b, a.batch - 1);
  const LT* lrow = a.L + (size_t)bc * a.bstride;
  lds_u32x4* s_w = (lds_u32x4*)smem;
  const bool rev = (a.j & 1) != 0;

  // Pieces of a step are dealt out in memory order: with MT = 1 a wave takes its own tile, else the
  // workgroup the whole step.  Row and column of piece p from a reciprocal: exact for p < 4096 and
  // pr <= 64 (p times its error stays below 2^18).
  const uint32_t recip = ((1u << 18) + (uint32_t)pr - 1) / (uint32_t)pr;
  static_assert(kST * NP <= 4096 || MT == 1, "pieces of a step");
  auto piece = [&](int q) { return MT == 1 ? q * 64 + lane : q * kST + tid; };
  const int tile_pieces = PACKED ? kTile : 16 * pr;
  const int wbase = MT == 1 ? str * tile_pieces : 0;
  const int last = PACKED ? (int)nt * kTile - 1 : (V - 1) * pr + pr - 1;
  const u32x4_t* wsrc = PACKED ? reinterpret_cast<const u32x4_t*>(a.wv) : reinterpret_cast<const u32x4_t*>(a.w_vocab);
  u32x4_t w[PD][NP];
  typename Four<LT>::type lg[PD];
  auto load_step = [&](int u, int i) {
    if (i >= steps) return;   // uniform
    const int ii = rev ? steps - 1 - i : i;
    const int first = (T0 + ii * NSTR) * tile_pieces;
#pragma unroll
    for (int q = 0; q < NP; ++q)   // past the matrix: its last piece, for rows that are not folded
      w[u][q] = wsrc[min(first + wbase + piece(q), last)];
    const int t = T0 + ii * NSTR + str;
    if (16 * t + 16 <= V) lg[u] = Four<LT>::load(lrow + 16 * t + 4 * g);
  };

  // Activations as operands, [sequence tile][chunk][split][lane] in LDS and from there into
  // registers.  Loads return in order: they are asked for before the weights, which then arrive
  // while the operands are made.
  // The workgroup's slice of the prior goes to LDS with them.
  constexpr int NA = (MT * KC * 64 + kST - 1) / kST;
  lds_float* s_prior = (lds_float*)(smem + PL::kLds);
  const bool staged = a.prior != nullptr;   // the slice fits: T1 - T0 + NSTR <= kPriorTiles
  float pv0[kPriorTiles * 16 / kST];
  if (staged) {
#pragma unroll
    for (int q = 0; q < kPriorTiles * 16 / kST; ++q) pv0[q] = a.prior[min(16 * T0 + tid + q * kST, V - 1)];
  }
  lds_u32x4* s_a = (lds_u32x4*)smem;
  uint4 act[KC][SPL];
  {
    auto put = [&](int i, const uint4* o) {   // piece i: sequence i / (4 KC), piece i % (4 KC) of its row
      const int s = i / (4 * KC), pc = i % (4 * KC);
#pragma unroll
      for (int e = 0; e < SPL; ++e) s_a[(((s >> 4) * KC + (pc >> 2)) * SPL + e) * 64 + 16 * (pc & 3) + (s & 15)] = vec(o[e]);
    };
    if (a.e_m) {
      TokenKeys<2 * MT> tk;
      load_keys(a.ts, b0, a.batch, wave, lane, tk);
      asm volatile("" ::: "memory");
#pragma unroll
      for (int u = 0; u < PD / 2; ++u) load_step(u, u);
      asm volatile("" ::: "memory");
      merge_keys(tk, V, wave, lane, s_tok);
      __syncthreads();
      uint4 v[NA];
#pragma unroll
      for (int q = 0; q < NA; ++q) {
        const int i = min(tid + q * kST, MT * KC * 64 - 1), pc = i % (4 * KC);
        v[q] = sel4(pc < pr, *reinterpret_cast<const uint4*>(a.e_m + ((size_t)s_tok[i / (4 * KC)] * pr + (pc < pr ? pc : 0)) * O::NP));
      }
      asm volatile("" ::: "memory");
#pragma unroll
      for (int u = PD / 2; u < PD; ++u) load_step(u, u);
      asm volatile("" ::: "memory");
#pragma unroll
      for (int q = 0; q < NA; ++q)
        if (tid + q * kST < MT * KC * 64) put(tid + q * kST, &v[q]);
    } else {
      float4 v[NA][NF];
#pragma unroll
      for (int q = 0; q < NA; ++q) {
        const int i = min(tid + q * kST, MT * KC * 64 - 1), pc = i % (4 * KC);
        const float* row = a.rho + ((size_t)min(b0 + i / (4 * KC), a.batch - 1) * pr + (pc < pr ? pc : 0)) * O::NP;
#pragma unroll
        for (int f = 0; f < NF; ++f) v[q][f] = *reinterpret_cast<const float4*>(row + 4 * f);
      }
      asm volatile("" ::: "memory");
#pragma unroll
      for (int u = 0; u < PD; ++u) load_step(u, u);
      asm volatile("" ::: "memory");
#pragma unroll
      for (int q = 0; q < NA; ++q) {
        const int i = tid + q * kST;
        uint4 o[O::SPL];
        act_split<WT>(v[q], i % (4 * KC) < pr, o);
        if (i < MT * KC * 64) put(i, o);
      }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < KC; ++c)
#pragma unroll
      for (int e = 0; e < SPL; ++e) act[c][e] = unvec(s_a[((mt * KC + c) * SPL + e) * 64 + lane]);
    __syncthreads();
    if (staged) {
#pragma unroll
      for (int q = 0; q < kPriorTiles * 16 / kST; ++q) s_prior[tid + q * kST] = pv0[q];
      __syncthreads();
    }
    if (pr < 4 * KC) {   // columns past r: zero in both operands
      for (int i = tid; i < (int)(PL::kLds / 16); i += kST) s_w[i] = u32x4_t{0u, 0u, 0u, 0u};
      __syncthreads();
    }
  }

  Partial P = partial_empty();
  P.L.m = P.S.m = P.F.m = kFinMin;
  const float gate = a.unc ? a.unc[(size_t)bc * a.B + a.j].gate : 1.f;
  const float alb = a.al * gate, beb = a.be * gate;
  const bool no_prior = beb == 0.f;   // the term is absent, masks included

  // The entries of the step before (long, short, fused; -inf past the vocabulary and the call) are
  // folded while the matrix cores work on this one.  The sums are rescaled to the running maxima as the
  // entries are made, by the difference of the rounded references that the entries use, and the rounding of the
  // last one is taken out at the end.  References that lag (moved only when a value lies 40 above them) saved 3% of a
  // batch-64 block, but left the exponents of the entries that count six bits short after the point.
  float x[4], s[4], f[4];
  int vp = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) x[e] = s[e] = f[e] = -INFINITY;
  float nl = -kFinMin * kLog2e, ns = nl, nf = nl;   // minus the references, base 2
  auto max4 = [](const float* v) { return fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])); };
  auto add4 = [](Lse& a, float neg, const float* v) {
    const float e0 = fast_exp2(__builtin_fmaf(v[0], kLog2e, neg)), e1 = fast_exp2(__builtin_fmaf(v[1], kLog2e, neg));
    const float e2 = fast_exp2(__builtin_fmaf(v[2], kLog2e, neg)), e3 = fast_exp2(__builtin_fmaf(v[3], kLog2e, neg));
    a.s += (e0 + e1) + (e2 + e3);
  };
  auto move_ref = [](Lse& a, float& neg, float m) {   // to the maximum with m
#pragma clang fp contract(off)   // n - neg as a fused product would miss 0 by the rounding of n
    a.m = fmaxf(a.m, m);
    const float n = -a.m * kLog2e;
    a.s *= fast_exp2(n - neg);   // exactly 1 while the maximum stays
    neg = n;
  };
  auto fold = [&]() {
    if (STATS) {
      add4(P.L, nl, x);
      add4(P.S, ns, s);
      add4(P.F, nf, f);
    }
    float y[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = f[e];
    if (SAMPLE) {
      const uint4 w4 = philox_row(a.smp, b, a.j, vp);
      y[0] += gumbel_from_word(w4.x);
      y[1] += gumbel_from_word(w4.y);
      y[2] += gumbel_from_word(w4.z);
      y[3] += gumbel_from_word(w4.w);
    }
    // top two of the four, then of the lane: tiles come in falling order of their index when rev,
    // where an equal value replaces the one before
    float m1 = -INFINITY, m2 = -INFINITY;
    int mi = 0x7fffffff;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      m2 = __builtin_amdgcn_fmed3f(y[e], m1, m2);
      const bool above = y[e] > m1;
      mi = above ? vp + e : mi;
      m1 = above ? y[e] : m1;
    }
    const bool up = (m1 > P.t1) | (rev & (m1 == P.t1));
    P.t2 = up ? fmaxf(P.t1, m2) : fmaxf(P.t2, m1);
    P.i1 = up ? mi : P.i1;
    P.t1 = up ? m1 : P.t1;
  };
  auto tile = [&](int t, const lds_u32x4* sb, typename Four<LT>::type lcur) {
    uint4 A[KC];
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      const int pc = 4 * c + g;
      A[c] = unvec(sb[PACKED ? c * 64 + lane : 16 * pc + (n ^ (pc & 15))]);
    }
    f32x4_t acc[SPL];
#pragma unroll
    for (int e = 0; e < SPL; ++e) acc[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < KC; ++c)
#pragma unroll
      for (int e = SPL - 1; e >= 0; --e) acc[e] = O::mma(A[c], act[c][e], acc[e]);
    fold();
    vp = 16 * t + 4 * g;
    Four<LT>::widen(lcur, x);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s[e] = SPL == 3 ? (acc[SPL - 1][e] + acc[SPL / 2][e]) + acc[0][e] : acc[0][e];
      f[e] = __builtin_fmaf(alb, s[e], mul_weight(a.wl, x[e]));
    }
    if (a.prior) {   // uniform
      const f32x4_t pv = *(const lds_f32x4*)(s_prior + vp - 16 * T0);
      const float pe[4] = {pv.x, pv.y, pv.z, pv.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) f[e] = __builtin_fmaf(-beb, no_prior ? 0.f : pe[e], f[e]);
    }
    if (SAMPLE) {
#pragma unroll
      for (int e = 0; e < 4; ++e) f[e] *= a.smp.inv_temp;
    }
    if (16 * t + 16 > V || t >= T1) {   // uniform: the last tile of the vocabulary, or none
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int v = vp + e;
        const bool in = v < V && t < T1;
        const int vc = min(v, V - 1);
        x[e] = to_f32(lrow[vc]);
        f[e] = __builtin_fmaf(alb, s[e], mul_weight(a.wl, x[e]));
        if (a.prior) f[e] = minus_weighted(f[e], beb, a.prior[vc]);
        if (SAMPLE) f[e] *= a.smp.inv_temp;
        x[e] = in ? x[e] : -INFINITY;
        s[e] = in ? s[e] : -INFINITY;
        f[e] = in ? f[e] : -INFINITY;
      }
    }
    if (STATS) {
      move_ref(P.L, nl, max4(x));
      move_ref(P.S, ns, max4(s));
      move_ref(P.F, nf, max4(f));
    }
  };
  auto step = [&](int u, int i) {
    const int t = T0 + (rev ? steps - 1 - i : i) * NSTR + str;
    if (MT == 1) wave_lds_order();   // the operands of the step before are read
    lds_u32x4* buf = s_w + (PL::kBufs == 1 ? 0 : (i & 1) * NSTR * kTile);
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      if (PACKED) {
        buf[(MT == 1 ? str * kTile : 0) + piece(q)] = w[u][q];
        continue;
      }
      const uint32_t row = __umul24(piece(q), recip) >> 18;
      const int pc = piece(q) - (int)row * pr;
      if (row < 16 * (MT == 1 ? 1 : NSTR))
        buf[((MT == 1 ? str : 0) + (row >> 4)) * kTile + 16 * pc + ((row ^ pc) & 15)] = w[u][q];
    }
    const typename Four<LT>::type lcur = lg[u];
    load_step(u, i + PD);
    if (MT > 1) __syncthreads();
    else wave_lds_order();
    tile(t, buf + str * kTile, lcur);
  };
  for (int i = 0; i < steps; i += PD) {
#pragma unroll
    for (int u = 0; u < PD; ++u)
      if (i + u < steps) step(u, i + u);
  }
  fold();

  // merge: the four row groups of a wave, then the NSTR waves of a sequence tile through LDS
  close_ref(P.L, nl);
  close_ref(P.S, ns);
  close_ref(P.F, nf);
  P = allred_partial(P, Perm4Rows{});
  __syncthreads();
  Partial* sp = reinterpret_cast<Partial*>(smem);   // [str][16 MT]
  if (g == 0) sp[str * 16 * MT + 16 * mt + n] = P;
  __syncthreads();
  if (tid < 128) {   // 128 partials: whole waves
    const int s = tid / NSTR;
    const Partial Q = allred_partial(sp[(tid % NSTR) * 16 * MT + s], PermN<NSTR>{});
    if (tid % NSTR == 0 && b0 + s < a.batch) {
      const size_t o = (size_t)(b0 + s) * a.G + blockIdx.x;
      a.keys[o] = step_key(Q.t1, Q.i1);
      a.parts[o] = StepPart{Q.L.m, Q.L.s, Q.S.m, Q.S.s, Q.F.m, Q.F.s, Q.t2};
    }
  }
  if (a.finish == 1 && blockIdx.y == 0) {   // uniform; G >= batch
    __syncthreads();
    if ((int)blockIdx.x < a.batch) finish_row(fin, blockIdx.x, sp);
  }
}

// The dynamic LDS limit of a kernel is raised to the maximum once per device (a per-call
// attribute change costs microseconds of host time).
template <auto Kern>
hipError_t raise_lds_limit(size_t lds) {
  if (lds <= 64 * 1024) return hipSuccess;
  static std::atomic<uint64_t> raised{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev < 64 ? (uint64_t)1 << dev : 0;
  if (!bit || !(raised.load(std::memory_order_acquire) & bit)) {
    e = hipFuncSetAttribute((const void*)Kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kMaxLds - 1024));
    if (e != hipSuccess) return e;
    raised.fetch_or(bit, std::memory_order_acq_rel);
  }
  return hipSuccess;
}

inline size_t vocab_lds(int MT, int kc, int spl) {
  return std::max((size_t)MT * kc * spl * 1024, (size_t)kSW * 16 * MT * sizeof(Partial));
}

template <typename WT, typename LT, int MT, int SPL, bool SAMPLE>
hipError_t launch_vocab_any(const VocabArgs<WT, LT>& a, const FinishArgs& fin, int nkb, dim3 grid, hipStream_t st) {
  auto kern = k_vocab_any<WT, LT, MT, 8, SPL, SAMPLE>;
  const size_t lds = vocab_lds(MT, nkb * 8, SPL);
  hipError_t e = raise_lds_limit<k_vocab_any<WT, LT, MT, 8, SPL, SAMPLE>>(lds);
  if (e != hipSuccess) return e;
  kern<<<grid, kST, lds, st>>>(a, fin, nkb);
  return hipGetLastError();
}

template <typename WT, typename LT, int MT, int KC, int SPL, bool SAMPLE, bool PACKED, bool STATS>
hipError_t launch_vocab_s(const VocabArgs<WT, LT>& a, const FinishArgs& fin, dim3 grid, hipStream_t st) {
  auto kern = k_vocab<WT, LT, MT, KC, SPL, SAMPLE, PACKED, STATS>;
  // the final merge takes 128 partials
  const size_t lds = std::max({VocabPlan<MT, KC>::kLds + (a.prior ? kPriorTiles * 64 : 0), VocabPlan<MT, KC>::act(SPL),
                               128 * sizeof(Partial)});
  hipError_t e = raise_lds_limit<k_vocab<WT, LT, MT, KC, SPL, SAMPLE, PACKED, STATS>>(lds);
  if (e != hipSuccess) return e;
  kern<<<grid, kST, lds, st>>>(a, fin);
  return hipGetLastError();
}

template <typename WT, typename LT, int MT, int KC, int SPL, bool SAMPLE, bool PACKED>
hipError_t launch_vocab_k(const VocabArgs<WT, LT>& a, const FinishArgs& fin, dim3 grid, hipStream_t st) {
  if constexpr (PACKED) {
    if (!a.stats) return launch_vocab_s<WT, LT, MT, KC, SPL, SAMPLE, PACKED, false>(a, fin, grid, st);
  }
  return launch_vocab_s<WT, LT, MT, KC, SPL, SAMPLE, PACKED, true>(a, fin, grid, st);
}

template <typename WT, typename LT, int SPL, bool SAMPLE>
hipError_t launch_vocab(VocabArgs<WT, LT> a, const FinishArgs& fin, hipStream_t st) {
  constexpr int K1 = 128 / Op<WT>::KCH, K2 = 256 / Op<WT>::KCH;   // chunks of 128 and of 256 columns
  const int mt = (a.batch + 15) / 16;
  // k_vocab_any also takes the rows without short logits and a prior whose slice of a workgroup exceeds
  // its room in LDS
  const bool wide_prior = a.prior && (a.V + 15) / 16 / a.G + 1 + kSW > kPriorTiles;
  const bool any = a.r > 256 || a.long_only || wide_prior;
  // as many tiles of 16 sequences per workgroup as the call has, at most four: the weights are
  // read once per workgroup row
  const int MT = mt == 1 ? 1 : (mt == 2 || any) ? 2 : 4;
  dim3 grid((unsigned)a.G, (unsigned)((mt + MT - 1) / MT));
  // A workgroup writes one row of results at its end.  Where CUs are idle, or sequences more than
  // workgroups, further workgroups do (Markov head, 48 sequences, V = 2,053 with its 17 workgroups: 389 us a
  // block with three rows after one another, 195 with a workgroup for each).
  if (a.finish && (a.batch > a.G || a.G * (int)grid.y + a.batch <= kMaxG)) {
    a.finish = 2;
    grid.x += ((unsigned)a.batch + grid.y - 1) / grid.y;
  }
  if (any) {
    const int nkb = (a.r + 8 * Op<WT>::KCH - 1) / (8 * Op<WT>::KCH);
    return MT == 1 ? launch_vocab_any<WT, LT, 1, SPL, SAMPLE>(a, fin, nkb, grid, st)
                   : launch_vocab_any<WT, LT, 2, SPL, SAMPLE>(a, fin, nkb, grid, st);
  }
#define DLS_VOCAB(MT, PACKED)                                                          \
  return a.r <= 128 ? launch_vocab_k<WT, LT, MT, K1, SPL, SAMPLE, PACKED>(a, fin, grid, st) \
                    : launch_vocab_k<WT, LT, MT, K2, SPL, SAMPLE, PACKED>(a, fin, grid, st)
  if constexpr (sizeof(WT) == 2) {
    if (a.wv) {   // prepared heads come with r = 128 or 256 and more than 16 sequences (a Markov head: 32)
      if constexpr (SPL > 1) {
        if (MT == 2) DLS_VOCAB(2, true);
      }
      DLS_VOCAB(4, true);
    }
  }
  if (MT == 1) DLS_VOCAB(1, false);
  if (MT == 2) DLS_VOCAB(2, false);
  DLS_VOCAB(4, false);
#undef DLS_VOCAB
}

}  // namespace

// The launches of one block (WT: head type, LT: long-logit type), instantiated one pair and
// decoding mode per translation unit.
template <typename WT, typename LT, bool SAMPLE>
hipError_t launch_step(const DraftArgs& a, hipStream_t st) {
  const dls_local_head& hd = a.head;
  const int batch = a.batch, B = a.B, V = hd.V, H = hd.H, r = hd.r;
  const bool markov = hd.kind == DLS_HEAD_MARKOV;
  char* ws = a.ws;
  float* hc = (float*)(ws + a.lay.off_h0);   // current state
  float* hn = (float*)(ws + a.lay.off_h1);   // next state
  float* rho = (float*)(ws + a.lay.off_rho);
  const int G = a.lay.groups;
  const size_t per = (size_t)batch * G;
  uint64_t* keys = (uint64_t*)(ws + a.lay.off_part);
  // a Markov head's launches read the partials of the position before while they write: two sets
  StepPart* parts = (StepPart*)(keys + (markov ? 2 : 1) * per);
  const bool literal = (a.f.flags & DLS_FIRST_ROW_LONG_ONLY) != 0;
  hipError_t e;

  auto al_of = [&](int j) { return a.alphas ? a.alphas[j] : a.f.alpha; };
  auto set_of = [&](int j) { return markov ? (size_t)(j & 1) * per : (size_t)0; };
  auto finish_of = [&](int j) {
    FinishArgs f;
    f.keys = keys + set_of(j);
    f.parts = parts + set_of(j);
    f.G = G;
    f.j = j;
    f.B = B;
    f.batch = batch;
    f.wl = a.f.w_long;
    f.al = al_of(j);
    f.long_only = literal && j == 0;
    f.out_tokens = a.out_tokens;
    f.out_stats = a.out_stats;
    f.smp = a.smp;
    f.unc = a.unc;
    f.hdr = a.hdr;
    return f;
  };
  if constexpr (sizeof(WT) == 2) {   // prepared heads are bf16
    if (a.prep) k_check_prepared<WT><<<1, 1, 0, st>>>(a.prep, *a.expect, a.hdr);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  bool first_head_step = true;
  for (int j = 0; j < B; ++j) {
    const bool long_only = literal && j == 0;
    const bool rows = !a.T && batch <= 4;   // see k_gates_rows
    TokenSource ts;
    ts.keys = j ? keys + set_of(j - 1) : nullptr;
    ts.last = a.last_token;
    ts.G = G;
    const FinishArgs fin = finish_of(j ? j - 1 : 0);
    if (!long_only && !markov) {
      if constexpr (sizeof(WT) == 2) {
        if (a.T) {
          FoldedArgs fa;
          fa.T = a.T;
          fa.whh = a.whh;
          fa.H = H;
          fa.V = V;
          fa.batch = batch;
          fa.ts = ts;
          fa.h_in = hc;
          fa.h_zero = first_head_step;
          fa.h_out = hn;
          k_gates_folded<WT><<<dim3((unsigned)(H / 16), (unsigned)((batch + 15) / 16)), kST, 0, st>>>(fa);
        }
      }
      if (!a.T) {
        GatesArgs<WT> ga;
        ga.emb = (const WT*)hd.emb;
        ga.w_ih = (const WT*)hd.w_ih;
        ga.w_hh = (const WT*)hd.w_hh;
        ga.d = hd.d;
        ga.H = H;
        ga.V = V;
        ga.batch = batch;
        ga.ts = ts;
        ga.h_in = hc;
        ga.h_zero = first_head_step;
        ga.h_out = hn;
        const unsigned gx = (unsigned)((H + kUnits - 1) / kUnits);
        const unsigned gr = (unsigned)((H + kRT / 64 - 1) / (kRT / 64));
        if (batch == 1) k_gates_rows<WT, 1><<<gr, kRT, 0, st>>>(ga);
        else if (batch == 2) k_gates_rows<WT, 2><<<gr, kRT, 0, st>>>(ga);
        else if (batch <= 4) k_gates_rows<WT, 4><<<gr, kRT, 0, st>>>(ga);
        else if (batch <= 16) k_gates<WT, 1><<<dim3(gx, 1), kST, 0, st>>>(ga);
        else if (batch <= 32) k_gates<WT, 2><<<dim3(gx, 1), kST, 0, st>>>(ga);
        else k_gates<WT, 4><<<dim3(gx, (unsigned)((batch + 63) / 64)), kST, 0, st>>>(ga);
      }
      if ((e = hipGetLastError()) != hipSuccess) return e;
      RankArgs<WT> ra;
      ra.w_rank = (const WT*)hd.w_rank;
      ra.H = H;
      ra.r = r;
      ra.batch = batch;
      ra.tiles = ((r + 15) / 16) * ((batch + 15) / 16);
      ra.h = hn;
      ra.rho = rho;
      if (rows) ra.tiles = (r + kSW - 1) / kSW;
      const unsigned gk = (unsigned)(ra.tiles + (j ? batch : 0));
      if (!rows) k_rank<WT><<<gk, kST, 0, st>>>(ra, fin);
      else if (batch == 1) k_rank_rows<WT, 1><<<gk, kST, 0, st>>>(ra, fin);
      else if (batch == 2) k_rank_rows<WT, 2><<<gk, kST, 0, st>>>(ra, fin);
      else k_rank_rows<WT, 4><<<gk, kST, 0, st>>>(ra, fin);
      if ((e = hipGetLastError()) != hipSuccess) return e;
      std::swap(hc, hn);
      first_head_step = false;
    }
    VocabArgs<WT, LT> va;
    va.w_vocab = (const WT*)hd.w_vocab;
    va.wv = a.wv;
    va.V = V;
    va.r = r;
    va.batch = batch;
    va.G = G;
    va.np = (V + kPairRows - 1) / kPairRows;
    va.rho = rho;
    va.e_m = markov ? (const WT*)hd.emb : nullptr;
    va.ts = ts;
    va.L = (const LT*)a.long_logits + (size_t)j * V;
    va.bstride = (size_t)B * V;
    va.prior = a.prior;
    va.wl = a.f.w_long;
    va.al = al_of(j);
    va.be = a.prior ? (a.betas ? a.betas[j] : a.f.beta) : 0.f;
    va.long_only = long_only;
    va.j = j;
    va.B = B;
    va.smp = a.smp;
    va.unc = a.unc;
    va.keys = keys + set_of(j);
    va.parts = parts + set_of(j);
    va.stats = a.out_stats != nullptr;
    va.finish = markov && j;
    e = markov ? launch_vocab<WT, LT, 1, SAMPLE>(va, fin, st) : launch_vocab<WT, LT, Op<WT>::SPL, SAMPLE>(va, fin, st);
    if (e != hipSuccess) return e;
  }
  ClearArgs ca;
  ca.h0 = markov ? nullptr : hc;
  ca.h1 = hn;
  ca.rho = rho;
  ca.H = H;
  ca.r = r;
  ca.keys = keys;
  ca.parts = parts;
  ca.sets = markov ? 2 : 1;
  k_finish<<<batch, kST, 0, st>>>(finish_of(B - 1), ca);
  return hipGetLastError();
}

}  // namespace dls
