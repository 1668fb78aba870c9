// A whole draft block of a small head in one launch: one workgroup per sequence runs every
// position (Algorithm 1) by itself, with no hand-off to another workgroup.
//
// A chain of launches costs a few microseconds per launch and position whatever a head's size; one
// CU reads about 100 KB of weights per microsecond from L2.  A head of up to kSmallBytes of weights
// (read once per position) is drafted here where small_head expects less time than of the chain: at V = 1024,
// d = H = r = 64 in float32 (368 KB) 43 us for four positions, by the chain 67.
//
// Sixteen lanes share a weight row (16-byte pieces, a DPP sum over the row of lanes), float32
// throughout.  In the vocabulary phase a group of sixteen lanes takes sixteen rows at a time and lane
// i keeps the result of row i, so that the fusion and the statistics run on all lanes.
#include "dels_internal.hpp"

namespace dls {

namespace {

constexpr int kTh = 1024;
constexpr int kWv = kTh / 64;
constexpr int kGrp = kTh / 16;   // groups of sixteen lanes

template <int N>
__device__ __forceinline__ float ror_add(float v) {   // v + the value N lanes further in the row of 16
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xf, 0xf, false));
}
// sum over the row of 16 lanes, in every lane
__device__ __forceinline__ float row_sum(float v) { return ror_add<1>(ror_add<2>(ror_add<4>(ror_add<8>(v)))); }

template <typename WT>
__device__ __forceinline__ float dot_piece(const WT* w, const float* x) {
  constexpr int N = Chunk<WT>::N;
  float a[N], s = 0.f;
  Chunk<WT>::load(w, a);
#pragma unroll
  for (int i = 0; i < N; ++i) s = __builtin_fmaf(a[i], x[i], s);
  return s;
}

__device__ __forceinline__ uint64_t small_key(float t1, int i1) {
  const uint32_t u = __float_as_uint(t1 + 0.0f);   // -0 -> +0, so that equal values compare equal
  const uint32_t o = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ((uint64_t)o << 32) | (uint32_t)~(uint32_t)i1;
}

struct Xor16 {   // sixteen consecutive lanes
  template <typename F>
  __device__ __forceinline__ void each(F f) const {
    f(8);
    f(4);
    f(2);
    f(1);
  }
  __device__ __forceinline__ float operator()(float v, int m) const { return __shfl_xor(v, m); }
  __device__ __forceinline__ int i(int v, int m) const { return __shfl_xor(v, m); }
};

struct SmallArgs {
  int d, H, r, V, B, markov, literal;
  const int32_t* last;
  const float* prior;
  float wl;
  float al[64], be[64];
  int32_t* out_tokens;
  dls_row_stats* out_stats;
  Sampler smp;
  const dls_row_uncertainty* unc;
};

template <typename WT, typename LT, bool SAMPLE>
__global__ __launch_bounds__(kTh) void k_small(SmallArgs a, const WT* __restrict__ emb, const WT* __restrict__ w_ih,
                                               const WT* __restrict__ w_hh, const WT* __restrict__ w_rank,
                                               const WT* __restrict__ w_vocab, const LT* __restrict__ L) {
  constexpr int N = Chunk<WT>::N;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int d = a.d, H = a.H, r = a.r, V = a.V, B = a.B;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int sub = tid & 15, grp = tid >> 4;
  Partial* s_part = reinterpret_cast<Partial*>(smem);                      // [B][kWv]
  uint64_t* s_key = reinterpret_cast<uint64_t*>(s_part + (size_t)B * kWv);  // [2][kWv]
  float* s_x = reinterpret_cast<float*>(s_key + 2 * kWv);                   // d
  float* s_h = s_x + d;                                                     // [2][H]
  float* s_rho = s_h + 2 * H;                                               // r
  for (int i = tid; i < H; i += kTh) s_h[i] = 0.f;
  int tok = a.literal ? 0 : a.last[b];
  int cur = 0;   // the half of s_h that holds the state
  for (int j = 0; j < B; ++j) {
    const bool long_only = a.literal && j == 0;
    if (!long_only) {
      const WT* er = emb + (size_t)((unsigned)tok < (unsigned)V ? tok : 0) * (a.markov ? r : d);
      if (a.markov) {
        for (int i = tid; i < r; i += kTh) s_rho[i] = to_f32(er[i]);
      } else {
        for (int i = tid; i < d; i += kTh) s_x[i] = to_f32(er[i]);
        __syncthreads();
        const float* hc = s_h + cur * H;
        float* hn = s_h + (cur ^ 1) * H;
        for (int k = grp; k < H; k += kGrp) {   // a hidden unit per group
          float ar = 0.f, az = 0.f, ax = 0.f, ah = 0.f;
          for (int c = sub; c < d / N; c += 16) {
            ar += dot_piece(w_ih + (size_t)k * d + c * N, s_x + c * N);
            az += dot_piece(w_ih + (size_t)(H + k) * d + c * N, s_x + c * N);
            ax += dot_piece(w_ih + (size_t)(2 * H + k) * d + c * N, s_x + c * N);
          }
          for (int c = sub; c < H / N; c += 16) {
            ar += dot_piece(w_hh + (size_t)k * H + c * N, hc + c * N);
            az += dot_piece(w_hh + (size_t)(H + k) * H + c * N, hc + c * N);
            ah += dot_piece(w_hh + (size_t)(2 * H + k) * H + c * N, hc + c * N);
          }
          const float rg = sigmoidf_(row_sum(ar)), zg = sigmoidf_(row_sum(az));
          const float ng = tanhf_(row_sum(ax) + rg * row_sum(ah));
          if (sub == 0) hn[k] = (1.f - zg) * ng + zg * hc[k];
        }
        cur ^= 1;
        __syncthreads();
        for (int i = grp; i < r; i += kGrp) {   // a rank row per group
          float s = 0.f;
          for (int c = sub; c < H / N; c += 16) s += dot_piece(w_rank + (size_t)i * H + c * N, hn + c * N);
          s = row_sum(s);
          if (sub == 0) s_rho[i] = siluf_(s);
        }
      }
      __syncthreads();
    }
    const LT* lrow = L + ((size_t)b * B + j) * V;
    const float g = a.unc ? a.unc[(size_t)b * B + j].gate : 1.f;
    const float alb = a.al[j] * g, beb = a.be[j] * g;
    Partial P = partial_empty();
    P.L.m = P.S.m = P.F.m = kFinMin;
    for (int v0 = grp * 16; v0 < V; v0 += kGrp * 16) {
      const int v = v0 + sub;
      const bool in = v < V;
      const float x = in ? to_f32(lrow[v]) : -INFINITY;
      float f = weighted(a.wl, x);
      if (!long_only) {
        const float pv = a.prior && in ? a.prior[v] : 0.f;
        float s = 0.f;
        const int nc = r / N;
        for (int c0 = 0; c0 < nc; c0 += 16) {   // sixteen pieces of sixteen rows
          const int c = min(c0 + sub, nc - 1);
          float p[16];
#pragma unroll
          for (int u = 0; u < 16; ++u) {
            p[u] = dot_piece(w_vocab + (size_t)min(v0 + u, V - 1) * r + c * N, s_rho + c * N);
            p[u] = c0 + sub < nc ? p[u] : 0.f;
          }
#pragma unroll
          for (int u = 0; u < 16; ++u) {
            const float t = row_sum(p[u]);
            s += sub == u ? t : 0.f;
          }
        }
        f = __builtin_fmaf(alb, s, f);
        if (a.prior) f = minus_weighted(f, beb, pv);
        s = in ? s : -INFINITY;
        lse_fold_fin<1>(P.S, &s, s);
      }
      if (SAMPLE) f *= a.smp.inv_temp;
      f = in ? f : -INFINITY;
      lse_fold_fin<1>(P.L, &x, x);
      lse_fold_fin<1>(P.F, &f, f);
      if (SAMPLE && in) f += gumbel_at(a.smp, b, j, v);
      top2_push(P, f, v);
    }
    // the token first: the next position waits for it
    uint64_t k = small_key(P.t1, P.i1);
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
      const uint64_t o = __shfl_xor((unsigned long long)k, m);
      k = o > k ? o : k;
    }
    if (lane == 0) s_key[(j & 1) * kWv + wave] = k;
    P.L.m = P.L.s == 0.f ? -INFINITY : P.L.m;   // a state without an entry is empty (a NaN sum is kept)
    P.S.m = P.S.s == 0.f ? -INFINITY : P.S.m;
    P.F.m = P.F.s == 0.f ? -INFINITY : P.F.m;
    P = allred_partial(P, WaveXor{});
    if (lane == 0) s_part[j * kWv + wave] = P;
    __syncthreads();
    k = s_key[(j & 1) * kWv];
#pragma unroll
    for (int w = 1; w < kWv; ++w) {
      const uint64_t o = s_key[(j & 1) * kWv + w];
      k = o > k ? o : k;
    }
    tok = (int)~(uint32_t)k;
    tok = tok == 0x7fffffff ? 0 : tok;   // every value -inf: the first index
  }
  // results: sixteen lanes per position
  for (int j0 = 0; j0 < B; j0 += kGrp) {
    const int j = j0 + grp;
    const Partial P = allred_partial(s_part[min(j, B - 1) * kWv + sub], Xor16{});
    if (j < B && sub == 0) {
      int32_t t;
      const int ti = P.i1 == 0x7fffffff ? 0 : P.i1;
      const float alb = a.unc ? a.al[j] * a.unc[(size_t)b * B + j].gate : a.al[j];
      finalize_row(P, a.wl, alb, a.literal && j == 0, &t, a.out_stats ? a.out_stats + (size_t)b * B + j : nullptr,
                   nullptr, SAMPLE ? gumbel_at(a.smp, b, j, ti) : 0.f, a.smp.temp);
      a.out_tokens[(size_t)b * B + j] = t;
    }
  }
}

template <typename WT, typename LT>
hipError_t launch_small_t(const DraftArgs& a, const SmallArgs& s, size_t lds, hipStream_t st) {
  auto kern = s.smp.inv_temp != 0.f ? k_small<WT, LT, true> : k_small<WT, LT, false>;
  kern<<<a.batch, kTh, lds, st>>>(s, (const WT*)a.head.emb, (const WT*)a.head.w_ih, (const WT*)a.head.w_hh,
                                  (const WT*)a.head.w_rank, (const WT*)a.head.w_vocab, (const LT*)a.long_logits);
  return hipGetLastError();
}

constexpr size_t kSmallBytes = (size_t)1 << 20;

size_t small_lds(const dls_local_head& h, int32_t B) {
  return (size_t)B * kWv * sizeof(Partial) + 2 * kWv * 8 + ((size_t)h.d + 2 * h.H + h.r) * 4;
}

}  // namespace

// At most kSmallBytes of weights per position, vectors and partials within 64 KiB of LDS, and a shorter position
// here than in the chain, both in tenths of a microsecond.  Here every sixteen pieces of a row (16 bytes a lane) of
// the 64 units, 64 rank rows or 1,024 vocabulary rows at a time are a round; the chain's launches take longer for
// more sequences and for float32.  Fitted to both over 480 calls (V 64 to 8,192, d to 8,192, H to 400, r 8 to 512, 1
// to 256 sequences); the route it takes is within 5% of the better one for 471 of them and within 10% for all.
// us a block of 16 positions in bf16 at batch 1, here and by the chain: V = 3,072, d = H = r = 64 265 and 261; V =
// 6,000 431 and 261; V = 60,000, d = H = r = 8 3,210 and 271; V = 64, d = r = 8, H = 400 363 and 249; Markov, r = 64,
// V = 256 106 and 106, V = 1,024 130 and 113; 64 sequences: V = 6,000 442 and 507, Markov, V = 1,024 132 and 198.
bool small_head(const dls_local_head& h, int32_t batch, int32_t B) {
  const bool f32 = h.dtype != DLS_BF16, markov = h.kind == DLS_HEAD_MARKOV;
  const size_t rnn = markov ? 0 : (size_t)3 * h.H * (h.d + h.H) + (size_t)h.r * h.H;
  if ((rnn + (size_t)h.V * h.r) * (f32 ? 4 : 2) > kSmallBytes || small_lds(h, B) > 64 * 1024) return false;
  const int lanes = f32 ? 64 : 128;   // columns of sixteen pieces
  auto rounds = [&](int n) { return (n + lanes - 1) / lanes; };
  int here = rounds(h.r) * (10 + (int)((int64_t)30 * h.V / 1024));
  if (!markov) here += 30 + (h.H + 63) / 64 * (20 + 3 * (rounds(h.d) + rounds(h.H))) + (h.r + 63) / 64 * rounds(h.H);
  if (f32) here = here * 4 / 5;
  int chain = markov ? (batch <= 16 ? 25 : batch <= 32 ? 65 : 90) + (h.r > 256 ? 40 : 0)
                     : (batch <= 4 ? 180 : batch <= 16 ? 195 : batch <= 32 ? 235 : 305) + h.d / (batch <= 4 ? 400 : 128);
  if (f32) chain = chain * 17 / 10;
  return here <= chain;
}

hipError_t launch_small(const DraftArgs& a, hipStream_t st) {
  const dls_local_head& h = a.head;
  SmallArgs s;
  s.d = h.d;
  s.H = h.H;
  s.r = h.r;
  s.V = h.V;
  s.B = a.B;
  s.markov = h.kind == DLS_HEAD_MARKOV;
  s.literal = (a.f.flags & DLS_FIRST_ROW_LONG_ONLY) != 0;
  s.last = a.last_token;
  s.prior = a.prior;
  s.wl = a.f.w_long;
  for (int j = 0; j < 64; ++j) {
    s.al[j] = j < a.B && a.alphas ? a.alphas[j] : a.f.alpha;
    s.be[j] = !a.prior ? 0.f : (j < a.B && a.betas ? a.betas[j] : a.f.beta);
  }
  s.out_tokens = a.out_tokens;
  s.out_stats = a.out_stats;
  s.smp = a.smp;
  s.unc = a.unc;
  const size_t lds = small_lds(h, a.B);
  if (h.dtype == DLS_BF16)
    return a.long_dtype == DLS_BF16 ? launch_small_t<bf16_t, bf16_t>(a, s, lds, st) : launch_small_t<bf16_t, float>(a, s, lds, st);
  return a.long_dtype == DLS_BF16 ? launch_small_t<float, bf16_t>(a, s, lds, st) : launch_small_t<float, float>(a, s, lds, st);
}

}  // namespace dls
