// Flag-masked causal prefill attention (Eq. 2 under the mask of Eq. 5), over COMPACTED keys: dispatch, and the fp32
// kernel.
//
// Because the cache keeps surviving rows in token order, the keys visible to query j are exactly the first
// cnt[j] cache rows of its KV head (cnt = exclusive prefix count of the flags) plus the query's own k_j, v_j.
// So the kernels are causal flash attention over a shorter key sequence with the per-query boundary cnt[j], and
// the own-token term is folded in as the initial state of the online softmax (which also keeps every running
// maximum finite).  The work is (1 - evicted fraction) of dense causal attention for any flag pattern; tiles
// that hold only evicted keys do not exist.  bf16 (head dimension 128 or 64) runs on the kernel of ag_prefill_bf16.hip,
// fp32 on the kernel below.
#include "ag_internal.h"

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kEmptyMax = -3.40282347e+38f;  // maximum before any key: the least finite number, no score lies below it

// exclusive prefix count of the keep flags at token j of one unit
__device__ __forceinline__ int cnt_at(const uint64_t *__restrict__ words, const int32_t *__restrict__ bo, int j) {
  const uint64_t w = words[j >> 6];
  return bo[j >> 6] + __popcll(w & ((1ull << (j & 63)) - 1ull));
}

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
template <int N> struct fvec { typedef __attribute__((__vector_size__(N * sizeof(float)))) float type; };

__device__ __forceinline__ float over_kg_max(float x) {  // over the four lanes that share lane % 16
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float over_kg_sum(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// fp32 on v_mfma_f32_16x16x4_f32 (products and sums in 32 bits): a workgroup owns 16 queries of one head, its waves take the
// 16-key tiles of the compacted rows in turn and their states meet in LDS at the end -- short prompts are bound by the
// length of one wave's chain, so the keys are what is split.  Lane = (query q = lane % 16, group kg = lane / 16).
//   S^T = K Q^T: four consecutive features per load feed four MFMAs (element e of every lane's 16 bytes is feature
//     16 t + 4 kg + e of step e), so K and Q come in 16-byte pieces straight from memory, no LDS.
//   O^T = V^T P^T: step r takes the keys 4 kg + r, which is where S^T's accumulator has the weights (p[r] is the B operand
//     as it stands); its A operand, row m of column tile e, is V[key][VW m + e (+ 16 VW half)], so a lane again loads
//     VW consecutive features and a row leaves memory whole.  A lane ends up with 4 VW consecutive output features.
// The query's own token starts the state of the last wave, the evicted tokens of a recent-token window are added lane by
// lane (a row that a query does not see is not read for it, whatever it holds).  In a tile that some query sees only
// in part, values that are not finite are kept out of the product and added lane by lane where they are seen.
// 128 tokens, 4 heads of 64: 22.4 us with one wave per query on the vector ALU.
template <int D, int NW>
__global__ __launch_bounds__(64 * NW) void ag_prefill_f32_kernel(const float *__restrict__ q, const float *__restrict__ k,
                                                                 const float *__restrict__ v,
                                                                 const uint64_t *__restrict__ words,
                                                                 const int32_t *__restrict__ blk_off,
                                                                 const float *__restrict__ kc, const float *__restrict__ vc,
                                                                 const int64_t *__restrict__ row_off, int L, int Hq,
                                                                 int Hkv, int nw, float qscale, int n_recent,
                                                                 float *__restrict__ out) {
  constexpr int VW = D >= 64 ? 4 : 2;        // features per lane and V load
  constexpr int VH = D / (16 * VW);          // V loads per row
  constexpr int KT = D / 16;                 // 16-byte pieces per lane of a K or Q row
  typedef typename fvec<VW>::type vvec;
  __shared__ float st[NW][16][D + 4];        // merge states: max, sum, -, -, o[0..D)
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, kg = lane >> 4;
  const int j0 = (int)(gridDim.x - 1 - blockIdx.x) * 16;  // longest rows first
  const int bh = blockIdx.y, b = bh / Hq, head = bh - b * Hq;
  const int u = b * Hkv + head / (Hq / Hkv);
  const int j = min(j0 + col, L - 1);
  const uint64_t *wu = words + (size_t)u * nw;
  const int32_t *bo = blk_off + (size_t)u * (nw + 1);
  const int64_t ro = row_off[u];
  const int cap_u = (int)min(row_off[u + 1] - ro, (int64_t)L);  // kept tokens beyond it found no room in the cache
  const int cnt = min(cnt_at(wu, bo, j), cap_u);
  const int cnt_lo = min(cnt_at(wu, bo, j0), cap_u), cnt_hi = min(cnt_at(wu, bo, min(j0 + 15, L - 1)), cap_u);
  const float *Kc = kc + (size_t)ro * D, *Vc = vc + (size_t)ro * D;

  f32x4 qf[KT];
  {
    const float *qr = q + ((size_t)bh * L + j) * D + 4 * kg;
#pragma unroll
    for (int t = 0; t < KT; ++t) qf[t] = *reinterpret_cast<const f32x4 *>(qr + 16 * t);
  }
  float m = kEmptyMax, l = 0.f;
  float o[VH][4][VW];  // o[h][r][e]: feature 16 VW h + VW (4 kg + r) + e of query col
#pragma unroll
  for (int h = 0; h < VH; ++h)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int e = 0; e < VW; ++e) o[h][r][e] = 0.f;

  // one more key for this lane's query: row t of the uncompacted k, v, if `see`; alone: it is the only one, and weighs 1
  // whatever its score is (a score that overflowed to -infinity counts as the least finite one elsewhere)
  auto add_row = [&](int t, bool see, bool alone) {
    const float *kr = k + ((size_t)u * L + t) * D + 4 * kg, *vr = v + ((size_t)u * L + t) * D + 4 * VW * kg;
    float s = 0.f;
    if (see) {
#pragma unroll
      for (int i = 0; i < KT; ++i) {
        const f32x4 x = *reinterpret_cast<const f32x4 *>(kr + 16 * i);
#pragma unroll
        for (int e = 0; e < 4; ++e) s = fmaf(qf[i][e], x[e], s);
      }
    }
    s = over_kg_sum(s) * qscale;  // (the four lanes of a query agree on `see`)
    s = alone ? 0.f : (s < kEmptyMax ? kEmptyMax : s);
    if (see) {
      const float mn = fmaxf(m, s), alpha = exp2f(m - mn), p = exp2f(s - mn);
      m = mn;
      l = l * alpha + (kg == 0 ? p : 0.f);  // (summed over the groups at the end)
#pragma unroll
      for (int h = 0; h < VH; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const vvec x = *reinterpret_cast<const vvec *>(vr + 16 * VW * h + VW * r);
#pragma unroll
          for (int e = 0; e < VW; ++e) o[h][r][e] = fmaf(p, x[e], o[h][r][e] * alpha);
        }
    }
  };
  if (wave == NW - 1) add_row(j, true, cnt == 0 && (n_recent == 1 || j == 0));
  for (int i = 1 + wave; i < n_recent; i += NW) {
    const int t = j - i;
    bool see = t >= 0;
    if (see) see = !(((wu[t >> 6] >> (t & 63)) & 1ull) && cnt_at(wu, bo, t) < cap_u);  // (else a cache row already)
    if (__any(see)) add_row(max(t, 0), see, false);
  }

  const int n_tiles = (cnt_hi + 15) / 16;
  for (int tile = wave; tile < n_tiles; tile += NW) {
    const int c0 = tile * 16;
    f32x4 kf[KT];
    vvec vf[4][VH];
    {
      const float *kr = Kc + (size_t)min(c0 + col, cnt_hi - 1) * D + 4 * kg;
#pragma unroll
      for (int t = 0; t < KT; ++t) kf[t] = *reinterpret_cast<const f32x4 *>(kr + 16 * t);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float *vr = Vc + (size_t)min(c0 + 4 * kg + r, cnt_hi - 1) * D + VW * col;
#pragma unroll
        for (int h = 0; h < VH; ++h) vf[r][h] = *reinterpret_cast<const vvec *>(vr + 16 * VW * h);
      }
    }
    f32x4 s2[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) s2[e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[t][e], qf[t][e], s2[e & 1], 0, 0, 0);
    const f32x4 sc = s2[0] + s2[1];  // sc[r]: key 4 kg + r
    const bool part = c0 + 16 > cnt_lo;  // (uniform) some query sees only some of the keys
    float p[4], mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p[r] = sc[r] * qscale;
      if (part && c0 + 4 * kg + r >= cnt) p[r] = -INFINITY;
      mx = fmaxf(mx, p[r]);
    }
    const float mn = fmaxf(m, over_kg_max(mx));
    const float alpha = exp2f(m - mn);
    m = mn;
    l *= alpha;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p[r] = exp2f(p[r] - mn);
      l += p[r];
    }
    bool odd = false;
    if (part) {  // 0 times what a query does not see would be NaN: values that are not finite wait ...
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int h = 0; h < VH; ++h)
#pragma unroll
          for (int e = 0; e < VW; ++e)
            if ((__float_as_uint(vf[r][h][e]) & 0x7f800000u) == 0x7f800000u) { odd = true; vf[r][h][e] = 0.f; }
      odd = __any(odd);
    }
#pragma unroll
    for (int h = 0; h < VH; ++h)
#pragma unroll
      for (int e = 0; e < VW; ++e) {
        f32x4 acc = {o[h][0][e] * alpha, o[h][1][e] * alpha, o[h][2][e] * alpha, o[h][3][e] * alpha};
#pragma unroll
        for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][h][e], p[r], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) o[h][r][e] = acc[r];
      }
    if (odd) {  // ... and are added one by one where they are seen
#pragma unroll 1
      for (int i = 0; i < 16; ++i) {
        const float mine = i & 2 ? (i & 1 ? p[3] : p[2]) : (i & 1 ? p[1] : p[0]);
        const float w = __shfl(mine, 16 * (i >> 2) + col, 64);
        if (c0 + i >= cnt) continue;
        const float *vr = Vc + (size_t)(c0 + i) * D + 4 * VW * kg;
#pragma unroll
        for (int h = 0; h < VH; ++h)
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int e = 0; e < VW; ++e) {
              const float x = vr[16 * VW * h + VW * r + e];
              if ((__float_as_uint(x) & 0x7f800000u) == 0x7f800000u) o[h][r][e] = fmaf(w, x, o[h][r][e]);
            }
      }
    }
  }
  l = over_kg_sum(l);
  float *mine = st[wave][col];
  if (kg == 0) { mine[0] = m; mine[1] = l; }
#pragma unroll
  for (int h = 0; h < VH; ++h)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      vvec x;
#pragma unroll
      for (int e = 0; e < VW; ++e) x[e] = o[h][r][e];
      *reinterpret_cast<vvec *>(mine + 4 + 16 * VW * h + VW * (4 * kg + r)) = x;
    }
  __syncthreads();
  // thread -> four features of a query
  for (int i = threadIdx.x; i < 16 * (D / 4); i += 64 * NW) {
    const int qq = i / (D / 4), d = 4 * (i % (D / 4));
    if (j0 + qq >= L) continue;
    float M = kEmptyMax, Ls = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, st[w][qq][0]);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float f = exp2f(st[w][qq][0] - M);
      Ls = fmaf(f, st[w][qq][1], Ls);
      const f32x4 x = *reinterpret_cast<const f32x4 *>(&st[w][qq][4 + d]);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = fmaf(f, x[e], acc[e]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] /= Ls;
    *reinterpret_cast<f32x4 *>(out + ((size_t)bh * L + j0 + qq) * D + d) = acc;
  }
}

}  // namespace

bool ag_prefill_supported(ag_dtype dt, int D, int G) {
  if (!(G == 1 || G == 2 || G == 4 || G == 8)) return false;
  return dt == AG_BF16 ? (D == 64 || D == 128) : (D == 32 || D == 64 || D == 128 || D == 256);
}

hipError_t ag_launch_prefill(ag_ctx *ctx, hipStream_t s, const void *q, const void *k, const void *v,
                             const uint64_t *words, const int32_t *blk_off, int B, int L, int Hq, int Hkv, int D,
                             ag_dtype dt, float scale, int n_recent, const void *kc, const void *vc,
                             const int64_t *row_off, void *out, const ag_pf_plan &plan, float *part) {
  const int nw = ag_nwords(L);
  const float qscale = scale * kLog2e;
  if (dt == AG_BF16)
    return ag_launch_prefill_bf16(s, q, k, v, words, blk_off, B, L, Hq, Hkv, D, qscale, n_recent, kc, vc, row_off, out,
                                  plan, part, false, ag_time_kernel(ctx, AG_K_PREFILL));
  ag_tick(ctx, AG_K_PREFILL, s);
  {
    const dim3 grid((L + 15) / 16, B * Hq);
#define AG_PF32(DD, NWV)                                                                                              \
  hipLaunchKernelGGL((ag_prefill_f32_kernel<DD, NWV>), grid, dim3(64 * NWV), 0, s, (const float *)q, (const float *)k,  \
                     (const float *)v, words, blk_off, (const float *)kc, (const float *)vc, row_off, L, Hq, Hkv, nw,    \
                     qscale, n_recent, (float *)out)
    if (D == 32) AG_PF32(32, 4); else if (D == 64) AG_PF32(64, 4); else if (D == 128) AG_PF32(128, 4); else AG_PF32(256, 2);
#undef AG_PF32
  }
  ag_tock(ctx, AG_K_PREFILL, s);
  return hipGetLastError();
}
