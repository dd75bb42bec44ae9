// Decode attention over ragged per-(batch, KV head) caches (Sec. 3.1, decoding stage), one launch per step.
//
// A step reads every cached K and V row once: large batches are bound by HBM, small ones by the number of dependent
// round trips.  The kernel therefore does everything in one launch -- it builds its own work list from len[] (no host
// read-back), streams the rows, merges, takes in the new token and appends it -- and hands data between workgroups only
// where a unit is too long for one.
//   * Work is counted in tiles of 32 rows of one unit; a wave takes every NW-th tile of its workgroup's segment, so the
//     waves run without a barrier until their segment ends.  The new token's own key and value (the diagonal of
//     Eq. 5) and the slots of the recent-token ring are extra tiles in front of a unit's cache rows.
//   * bf16 runs on MFMA: K and V rows go from memory to the wave's own LDS by direct loads (whole 256-byte rows; the next
//     tile's K is requested as soon as this tile's fragments are read, its V after the second product, so 8 to 16 KiB per
//     wave are always in flight and no register holds them), S^T = K q^T and O^T = V^T p^T for all G query heads of the
//     group at once.  p enters the second product as a bf16 pair (high part + remainder, two MFMAs): the weights keep 16
//     bits, as a 32-bit product would.  fp32 caches run on the vector ALU.
//   * Segments (what a workgroup works on between two merges) are chosen on the device.  If the whole step gives every
//     workgroup at most one segment -- a unit of up to 4 rounds of its waves stays whole, a longer one is cut into
//     pieces of two rounds -- a unit's pieces meet once; otherwise the tiles of all units are laid end to end and cut
//     into equal ranges, one per workgroup, and only the units at the cuts cross workgroups.
//   * A unit inside one workgroup is finished there, through LDS.  The pieces of a longer one are stored as records
//     (written through, complete before the arrival is counted); the piece that arrives last merges them in order.
#include <algorithm>
#include <atomic>
#include <mutex>

#include "ag_internal.h"

// Scratch of ag_decode_attn_static, the entry point for callers that cannot allocate: the records that the pieces of a
// unit exchange live here instead of in a context's workspace.  One copy per GPU, held until the
// process ends.  In host code this name is only a stand-in for the symbol; the device address comes from
// hipGetSymbolAddress (ag_static_scratch below) and is what every launch receives.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

constexpr int kChunk = 128;      // cache rows per record of scratch space (ag_decode_scratch_bytes)
constexpr int kTileRows = 32;    // rows a wave takes at a time
constexpr int kFewUnits = 256;   // up to here 8 waves per workgroup and one workgroup per CU: a unit's rows are spread over
                                 // as many waves as LDS can feed; beyond, 4 waves and two workgroups per CU, so that one
                                 // streams while the other merges
constexpr float kEmptyMax = -1.0e30f;  // reference maximum before any row (finite on purpose)
constexpr float kLog2e = 1.4426950408889634f;

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float nt_f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
#define AG_LDS __attribute__((address_space(3)))

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  const f32x2 x = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
}

__device__ __forceinline__ void to_bf16(float x, uint16_t *o) {  // round to nearest even
  uint32_t u = __float_as_uint(x);
  u += 0x7fffu + ((u >> 16) & 1u);
  *o = (uint16_t)(u >> 16);
}

// 16 bytes that may (loose) lie at any even address
__device__ __forceinline__ uint4 chunk16(const uint8_t *p, bool loose) {
  if (!loose) return *reinterpret_cast<const uint4 *>(p);
  const uint16_t *h = reinterpret_cast<const uint16_t *>(p);
  auto two = [&](int i) { return (uint32_t)h[i] | ((uint32_t)h[i + 1] << 16); };
  return make_uint4(two(0), two(2), two(4), two(6));
}
__device__ __forceinline__ void put16(uint8_t *p, const uint4 &x, bool loose) {
  if (!loose) {
    *reinterpret_cast<uint4 *>(p) = x;
    return;
  }
  uint16_t *h = reinterpret_cast<uint16_t *>(p);
  const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) { h[2 * i] = (uint16_t)w[i]; h[2 * i + 1] = (uint16_t)(w[i] >> 16); }
}
// a pair of floats written through to memory / read past the caches (see ag_internal.h on data between workgroups)
__device__ __forceinline__ void put_pair(float *p, float a, float b) {
  __hip_atomic_store(reinterpret_cast<uint64_t *>(p), (uint64_t)__float_as_uint(a) | ((uint64_t)__float_as_uint(b) << 32),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ float2 get_pair(const float *p) {
  const uint64_t x = __hip_atomic_load(reinterpret_cast<const uint64_t *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  return make_float2(__uint_as_float((uint32_t)x), __uint_as_float((uint32_t)(x >> 32)));
}

template <int CTRL> __device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}
// Sum over aligned groups of LPR lanes; every lane of the group gets the sum.
template <int LPR> __device__ __forceinline__ float group_sum(float x) {
  x += dpp<0xB1>(x);                           // quad_perm [1,0,3,2]
  x += dpp<0x4E>(x);                           // quad_perm [2,3,0,1]
  if (LPR >= 8) x += dpp<0x141>(x);            // row_half_mirror
  if (LPR >= 16) x += dpp<0x140>(x);           // row_mirror
  if (LPR >= 32) x += __shfl_xor(x, 16, 64);
  if (LPR >= 64) x += __shfl_xor(x, 32, 64);
  return x;
}

// ---------------------------------------------------------------------------------------------------------
// LDS address key of row r of a wave's tile: the row's 16-byte chunk c lies at position c ^ key(r).  Among 16
// consecutive rows all keys differ (K fragments: 16 rows, one chunk), and among the 8 rows that a transposing V read
// serves together all pairs of chunks differ.  (D = 64: a row covers half of the banks, odd rows the other half.)
template <int D> __device__ __forceinline__ int tile_key(int r) {
  return D == 128 ? (((r & 7) << 1) | ((r >> 3) & 1)) : ((((r >> 1) & 3) << 1) | ((r >> 3) & 1));
}

// What a tile reads: rows row0 .. row0 + 31 of k and v; those whose bit in `vis` is clear are not seen (wave-uniform).
struct dec_tile {
  const void *k, *v;  // first row of the array the tile belongs to
  uint32_t bytes;     // cache rows: size of the array (rows past its end read as zeros)
  int row0;
  uint32_t vis;
  bool extra;         // new token or ring: rows whose bit is clear are not even read (they may hold anything)
};

// ---- bf16: one wave's pass over its tiles on MFMA -----------------------------------------------------------
// Lane = (query head q = lane % 16, key group kg = lane / 16); heads q >= G are zero columns.
template <int D, int G> struct wave_bf16 {
  static constexpr int kRowB = D * 2, CPR = kRowB / 16, RPI = 64 / CPR;  // RPI rows per load instruction
  static constexpr int NL = kTileRows / RPI;                             // load instructions per tile and operand
  static constexpr int kWaveB = 2 * kTileRows * kRowB;                   // the wave's LDS: K tile, V tile
  static constexpr int kStates = 1, kStateF = D + 4;                     // merge states a wave leaves, floats per head
  static constexpr int KS = D / 32, DT = D / 16;
  bf16x8 qf[KS];
  f32x4 o[DT];
  float m, l;
  int ld_off[NL], k_off[KS], v_off[DT];
  uint32_t lds_addr;
  AG_LDS uint8_t *lds;
  int lane, kg, col;

  __device__ __forceinline__ void init(AG_LDS uint8_t *mem, int lane_) {
    lane = lane_; kg = lane >> 4; col = lane & 15;
    lds = mem;
    lds_addr = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)mem);
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int r = RPI * i + lane / CPR;
      ld_off[i] = r * kRowB + (((lane % CPR) ^ tile_key<D>(r)) << 4);
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) k_off[ks] = col * kRowB + (((4 * ks + kg) ^ tile_key<D>(col)) << 4);
    const int vr = 4 * kg + (col >> 2);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      v_off[dt] = vr * kRowB + (((2 * dt + ((col & 3) >> 1)) ^ tile_key<D>(vr)) << 4) + (col & 1) * 8;
  }
  // q: the G query rows of the unit
  __device__ __forceinline__ void begin(const uint16_t *q) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      uint4 x = make_uint4(0, 0, 0, 0);
      if (col < G) x = *reinterpret_cast<const uint4 *>(q + (size_t)col * D + 32 * ks + 8 * kg);
      qf[ks] = __builtin_bit_cast(bf16x8, x);
    }
    m = kEmptyMax; l = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // Cache rows of one operand straight into LDS; rows past the array arrive as zeros.  Every cached row is read once per
  // step: non-temporal, so that the stream does not push the small hot data (queries, lengths, records) out of the caches.
  __device__ __forceinline__ void load(const dec_tile &t, const void *base, uint32_t dst) {
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, t.bytes, 0x00020000);
    const int soff = t.row0 * kRowB;
#pragma unroll
    for (int i = 0; i < NL; ++i)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                   :: "s"(dst + i * RPI * kRowB), "v"(ld_off[i]), "s"(rsrc), "s"(soff) : "memory");
  }
  // The new token's row or ring slots, through registers: only the visible rows are read, the others become zeros.
  __device__ __forceinline__ void load_extra(const dec_tile &t, bool loose) {
    uint4 x[2][NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const bool see = (t.vis >> (RPI * i + lane / CPR)) & 1u;
#pragma unroll
      for (int kv = 0; kv < 2; ++kv) {
        x[kv][i] = make_uint4(0, 0, 0, 0);
        if (see) x[kv][i] = chunk16(static_cast<const uint8_t *>(kv ? t.v : t.k) + (size_t)t.row0 * kRowB + ld_off[i], loose);
      }
    }
#pragma unroll
    for (int kv = 0; kv < 2; ++kv)
#pragma unroll
      for (int i = 0; i < NL; ++i)
        *reinterpret_cast<AG_LDS u32x4 *>(lds + (kv * kTileRows + i * RPI) * kRowB + lane * 16) =
            u32x4{x[kv][i].x, x[kv][i].y, x[kv][i].z, x[kv][i].w};
  }
  __device__ __forceinline__ void load_k(const dec_tile &t) { load(t, t.k, lds_addr); }
  __device__ __forceinline__ void load_v(const dec_tile &t) { load(t, t.v, lds_addr + kTileRows * kRowB); }

  // tiles first, first + step, ... < last of the segment; get(i) describes tile i
  // (a tile that is not cache rows can only be a wave's first: there are fewer of them than waves)
  template <typename GET> __device__ __forceinline__ void run(int first, int last, int step, float qscale, bool loose, GET &&get) {
    if (first >= last) return;
    dec_tile t = get(first);
    if (t.extra) {
      load_extra(t, loose);
    } else {
      load_k(t);
      load_v(t);
    }
    // the query's loads are waited for here, once: the compiler would otherwise put a wait for everything into the loop
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[ks]));
    for (int i = first; i < last; i += step) {
      const bool more = i + step < last;
      const uint32_t vis = t.vis;
      if (more) t = get(i + step);
      asm volatile("s_waitcnt vmcnt(%0)" :: "n"(NL) : "memory");  // K has landed (V, requested after it, may not have)
      bf16x8 kf[2][KS];
#pragma unroll
      for (int sub = 0; sub < 2; ++sub)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          kf[sub][ks] = *reinterpret_cast<const AG_LDS bf16x8 *>(lds + sub * 16 * kRowB + k_off[ks]);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (more) load_k(t);
      f32x4 s[2];
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) {
        s[sub] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) s[sub] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[sub][ks], qf[ks], s[sub], 0, 0, 0);
      }
      // s[sub][r]: key 16 sub + 4 kg + r, head col
      float p[8], mx = -INFINITY;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        p[e] = s[e >> 2][e & 3] * qscale;
        if (vis != 0xffffffffu && !((vis >> (16 * (e >> 2) + 4 * kg + (e & 3))) & 1u)) p[e] = -INFINITY;
        mx = fmaxf(mx, p[e]);
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float m_new = fmaxf(m, mx);
      const float alpha = __builtin_amdgcn_exp2f(m - m_new);
      if (__any(m_new != m)) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[dt] *= alpha;
      }
      m = m_new;
      l *= alpha;
      float lo[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        p[e] = __builtin_amdgcn_exp2f(p[e] - m);
        l += p[e];
      }
      uint4 ph = make_uint4(pack2(p[0], p[1]), pack2(p[2], p[3]), pack2(p[4], p[5]), pack2(p[6], p[7]));
      const uint32_t hw[4] = {ph.x, ph.y, ph.z, ph.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        lo[2 * e] = p[2 * e] - __uint_as_float(hw[e] << 16);
        lo[2 * e + 1] = p[2 * e + 1] - __uint_as_float(hw[e] & 0xffff0000u);
      }
      const uint4 pl = make_uint4(pack2(lo[0], lo[1]), pack2(lo[2], lo[3]), pack2(lo[4], lo[5]), pack2(lo[6], lo[7]));
      if (more)
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"(NL) : "memory");  // V has landed (the next K may not have)
      else
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      bf16x8 vf[DT];  // row d = 16 dt + col of V^T, keys 4 kg + 0..3 and 16 + 4 kg + 0..3
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const AG_LDS uint8_t *base = lds + kTileRows * kRowB + v_off[dt];
        const bf16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((AG_LDS bf16x4 *)base);
        const bf16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((AG_LDS bf16x4 *)(base + 16 * kRowB));
        vf[dt] = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (more) load_v(t);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[dt], __builtin_bit_cast(bf16x8, ph), o[dt], 0, 0, 0);
        o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[dt], __builtin_bit_cast(bf16x8, pl), o[dt], 0, 0, 0);
      }
    }
  }
  // the wave's state into its LDS: per head [max, sum, -, -, o[0..D)]
  __device__ __forceinline__ void leave(AG_LDS float *st) {
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    if (col < G) {
      AG_LDS float *h = st + col * kStateF;
      if (kg == 0) { h[0] = m; h[1] = l; }
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) *reinterpret_cast<AG_LDS f32x4 *>(h + 4 + 16 * dt + 4 * kg) = o[dt];
    }
  }
};

// ---- fp32: one wave's pass on the vector ALU; each group of LPR lanes owns one row per load -------------------
template <int D, int G> struct wave_f32 {
  static constexpr int EPL = 4, LPR = D / EPL, GPW = 64 / LPR;   // lanes per row, rows per load
  static constexpr int NIT = kTileRows / GPW;                    // loads that cover a tile
  static constexpr int UN = (G <= 2 ? 8 : 4) < NIT ? (G <= 2 ? 8 : 4) : NIT;  // rows in flight per lane group
  static constexpr int kStates = GPW, kStateF = D + 4;
  static constexpr int kWaveB = GPW * G * kStateF * 4;
  float4 qr[G];
  float m[G], l[G], acc[G][EPL];
  int grp, seg;
  __device__ __forceinline__ void init(AG_LDS uint8_t *, int lane) { grp = lane / LPR; seg = lane % LPR; }
  __device__ __forceinline__ void begin(const float *q) {
#pragma unroll
    for (int gg = 0; gg < G; ++gg) {
      qr[gg] = reinterpret_cast<const float4 *>(q + (size_t)gg * D)[seg];
      m[gg] = kEmptyMax; l[gg] = 0.f;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[gg][e] = 0.f;
    }
  }
  template <typename GET> __device__ __forceinline__ void run(int first, int last, int step, float qscale, bool, GET &&get) {
    for (int i = first; i < last; i += step) {
      const dec_tile t = get(i);
      const nt_f32x4 *K = reinterpret_cast<const nt_f32x4 *>(t.k) + (size_t)t.row0 * LPR + seg;
      const nt_f32x4 *V = reinterpret_cast<const nt_f32x4 *>(t.v) + (size_t)t.row0 * LPR + seg;
      for (int it0 = 0; it0 < NIT; it0 += UN) {
        nt_f32x4 kk[UN], vv[UN];
        bool ok[UN];
#pragma unroll
        for (int j = 0; j < UN; ++j) {
          const int r = (it0 + j) * GPW + grp;
          ok[j] = (t.vis >> r) & 1u;
          kk[j] = vv[j] = nt_f32x4{0.f, 0.f, 0.f, 0.f};
          if (ok[j]) {
            kk[j] = __builtin_nontemporal_load(K + (size_t)r * LPR);
            vv[j] = __builtin_nontemporal_load(V + (size_t)r * LPR);
          }
        }
#pragma unroll
        for (int gg = 0; gg < G; ++gg) {
          float s[UN], mn = m[gg];
#pragma unroll
          for (int j = 0; j < UN; ++j) {
            float d = qr[gg].x * kk[j][0];
            d = fmaf(qr[gg].y, kk[j][1], d);
            d = fmaf(qr[gg].z, kk[j][2], d);
            d = fmaf(qr[gg].w, kk[j][3], d);
            d = group_sum<LPR>(d) * qscale;
            s[j] = ok[j] ? d : -INFINITY;
            mn = fmaxf(mn, s[j]);
          }
          const float alpha = exp2f(m[gg] - mn);
          m[gg] = mn;
          l[gg] *= alpha;
#pragma unroll
          for (int e = 0; e < EPL; ++e) acc[gg][e] *= alpha;
#pragma unroll
          for (int j = 0; j < UN; ++j) {
            const float p = exp2f(s[j] - mn);
            l[gg] += p;
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[gg][e] = fmaf(p, vv[j][e], acc[gg][e]);
          }
        }
      }
    }
  }
  __device__ __forceinline__ void leave(AG_LDS float *st) {
#pragma unroll
    for (int gg = 0; gg < G; ++gg) {
      AG_LDS float *h = st + (grp * G + gg) * kStateF;
      if (seg == 0) { h[0] = m[gg]; h[1] = l[gg]; }
#pragma unroll
      for (int e = 0; e < EPL; ++e) h[4 + seg * EPL + e] = acc[gg][e];
    }
  }
};
template <typename T, int D, int G> struct wave_of;
template <int D, int G> struct wave_of<uint16_t, D, G> { typedef wave_bf16<D, G> type; };
template <int D, int G> struct wave_of<float, D, G> { typedef wave_f32<D, G> type; };

struct dec_args {
  const void *q, *k_new, *v_new;
  const uint8_t *new_flags;
  void *kc, *vc;
  int32_t *idx;
  const int64_t *row_off;
  int32_t *len;
  void *out;
  float *rec;           // records [id][G][D + 2]: o, max, sum
  int32_t *tickets;     // [U] pieces of a unit that have stored their record; zero between launches
  int32_t *arrived;     // [1] workgroups that have read len[]; zero between launches
  int32_t *d_err;
  int U, pos, max_wgs;  // max_wgs: workgroups the equal-range split may use (two records each)
  float qscale;
  bool loose;           // k_new, v_new, the ring or out are not 16-byte aligned: they are accessed by elements
  ag_ring_dev ring;
};

template <typename T, int D, int G, int NW>
__global__ __launch_bounds__(64 * NW, 2) void ag_decode_kernel(dec_args a) {
  typedef typename wave_of<T, D, G>::type wave_t;
  constexpr int NT = 64 * NW, SF = wave_t::kStateF;
  constexpr int kPieceTiles = 2 * NW, kWholeTiles = 4 * NW;
  constexpr int CPT = (int)(D * sizeof(T) / 16);  // 16-byte chunks per row
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  int32_t *s_len = reinterpret_cast<int32_t *>(smem + NW * wave_t::kWaveB);  // [U] valid rows; top bit: the unit has room
  __shared__ int32_t w_tiles[NW], w_items[NW], s_start[2], s_last;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int U = a.U;
  const bool has_ring = a.ring.k != nullptr;
  const int extra = 1 + (has_ring ? (a.ring.n + kTileRows - 1) / kTileRows : 0);

  // ---- the work list: tiles per unit, and the pieces they would be cut into ----
  const int per = (U + NT - 1) / NT;
  const int u0 = min(U, tid * per), u1 = min(U, u0 + per);
  auto tiles_of = [&](int n) { return extra + (n + kTileRows - 1) / kTileRows; };
  auto pieces_of = [&](int t) { return t <= kWholeTiles ? 1 : (t + kPieceTiles - 1) / kPieceTiles; };
  int my_tiles = 0, my_items = 0;
  for (int u = u0; u < u1; ++u) {
    const int64_t cap = a.row_off[u + 1] - a.row_off[u];
    const int n_raw = a.len[u];
    const int n = n_raw < 0 ? 0 : (n_raw < cap ? n_raw : (int)cap);
    s_len[u] = n | (n < cap ? 0x80000000 : 0);
    const int t = tiles_of(n);
    my_tiles += t;
    my_items += pieces_of(t);
  }
  int inc_t = my_tiles, inc_i = my_items;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(inc_t, o, 64), i = __shfl_up(inc_i, o, 64);
    if (lane >= o) { inc_t += t; inc_i += i; }
  }
  if (lane == 63) { w_tiles[wave] = inc_t; w_items[wave] = inc_i; }
  __syncthreads();  // (every thread's reads of len[] are complete here: the scan has consumed them)
  // The lengths may only change once every workgroup has read them: the workgroup that arrives last does it, at its end.
  int order = 0;
  if (tid == 0) order = __hip_atomic_fetch_add(a.arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  int base_t = inc_t - my_tiles, base_i = inc_i - my_items, total_t = 0, total_i = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    if (w < wave) { base_t += w_tiles[w]; base_i += w_items[w]; }
    total_t += w_tiles[w];
    total_i += w_items[w];
  }
  const bool by_piece = total_i <= (int)gridDim.x;
  const int wg = blockIdx.x;
  // equal ranges of tiles: at most max_wgs of them
  const int quota = by_piece ? 0 : (total_t + min((int)gridDim.x, a.max_wgs) - 1) / min((int)gridDim.x, a.max_wgs);
  const int x = by_piece ? wg : wg * quota;  // the piece or the tile this workgroup starts at
  const bool idle = by_piece ? x >= total_i : x >= total_t;
  if (!idle) {
    const int base = by_piece ? base_i : base_t;
    if (base <= x && x < base + (by_piece ? my_items : my_tiles)) {  // exactly one thread
      int at = base, u = u0;
      for (;; ++u) {
        const int t = tiles_of(s_len[u] & 0x7fffffff), n = by_piece ? pieces_of(t) : t;
        if (x < at + n) break;
        at += n;
      }
      s_start[0] = u;
      s_start[1] = x - at;  // piece or tile inside the unit
    }
  }
  __syncthreads();

  wave_t wv;
  AG_LDS uint8_t *my_lds = (AG_LDS uint8_t *)smem + wave * wave_t::kWaveB;
  wv.init(my_lds, lane);
  int left = idle ? 0 : by_piece ? 1 : min(quota, total_t - x);  // tiles (or the one piece) still to do
  int u = idle ? 0 : s_start[0], sub = idle ? 0 : s_start[1], at = x;
  while (left > 0) {
    u = __builtin_amdgcn_readfirstlane(u);
    const int sl = __builtin_amdgcn_readfirstlane(s_len[u]);
    const int n = sl & 0x7fffffff;
    const int T_u = tiles_of(n);
    int t0, t1, rec0 = 0, n_rec, my_rec;  // tiles [t0, t1) of the unit; the unit's records and this one's number
    if (by_piece) {
      n_rec = pieces_of(T_u);
      my_rec = sub;
      t0 = (int)((int64_t)T_u * sub / n_rec);
      t1 = (int)((int64_t)T_u * (sub + 1) / n_rec);
      rec0 = wg - sub;
      left = 0;
    } else {
      t0 = sub;
      t1 = min(T_u, t0 + left);
      left -= t1 - t0;
      const int first = at - t0;  // the unit's first tile, counted over all units
      at += t1 - t0;
      const int g0 = first / quota, g1 = (first + T_u - 1) / quota;
      n_rec = g1 - g0 + 1;
      my_rec = wg - g0;
      rec0 = g0;
    }
    const int64_t ro = a.row_off[u];
    const T *kn = static_cast<const T *>(a.k_new) + (size_t)u * D, *vn = static_cast<const T *>(a.v_new) + (size_t)u * D;
    const bool first_piece = t0 == 0;  // this workgroup takes the new token in
    // requested now, used at the segment's end
    uint4 new_row = make_uint4(0, 0, 0, 0);
    bool keep_new = true;
    if (first_piece) {
      if (tid < 2 * CPT) new_row = chunk16(reinterpret_cast<const uint8_t *>(tid < CPT ? kn : vn) + 16 * (tid % CPT), a.loose);
      keep_new = a.new_flags == nullptr || a.new_flags[u] != 0;
    }
    uint64_t ring_vis = 0;
    if (has_ring && t0 < extra) {  // evicted tokens of the window: the kept ones are cache rows already
      bool see = false;
      if (lane < a.ring.n) {
        const int p = a.ring.pos[(size_t)u * a.ring.n + lane];
        see = p < a.pos && p > a.pos - a.ring.n && a.ring.flags[(size_t)u * a.ring.n + lane] == 0;
      }
      ring_vis = __ballot(see);
    }
    wv.begin(static_cast<const T *>(a.q) + (size_t)u * G * D);
    const T *K = static_cast<const T *>(a.kc) + (size_t)ro * D, *V = static_cast<const T *>(a.vc) + (size_t)ro * D;
    wv.run(t0 + wave, t1, NW, a.qscale, a.loose, [&](int i) {
      if (i >= extra) {
        const int r = (i - extra) * kTileRows;
        return dec_tile{K, V, (uint32_t)n * (uint32_t)(D * sizeof(T)), r, n - r >= 32 ? 0xffffffffu : (1u << (n - r)) - 1u, false};
      }
      if (i == 0) return dec_tile{kn, vn, (uint32_t)(D * sizeof(T)), 0, 1u, true};
      const size_t ring0 = (size_t)u * a.ring.n * D;
      return dec_tile{static_cast<const T *>(a.ring.k) + ring0, static_cast<const T *>(a.ring.v) + ring0,
                      (uint32_t)a.ring.n * (uint32_t)(D * sizeof(T)), (i - 1) * kTileRows,
                      (uint32_t)(ring_vis >> (32 * (i - 1))), true};
    });
    wv.leave((AG_LDS float *)my_lds);
    __syncthreads();

    // ---- merge the waves' states; thread -> (head, two neighbouring columns) ----
    const int n_states = min(NW, t1 - t0) * wave_t::kStates;
    auto state = [&](int sI) {
      return (AG_LDS float *)((AG_LDS uint8_t *)smem + (sI / wave_t::kStates) * wave_t::kWaveB) + (sI % wave_t::kStates) * G * SF;
    };
    auto store_out = [&](int gg, int d, float o0, float o1) {
      T *dst = static_cast<T *>(a.out) + ((size_t)u * G + gg) * D + d;
      if constexpr (sizeof(T) == 2) {
        uint16_t lo, hi;
        to_bf16(o0, &lo);
        to_bf16(o1, &hi);
        if (a.loose) {
          dst[0] = lo;
          dst[1] = hi;
        } else {
          *reinterpret_cast<uint32_t *>(dst) = (uint32_t)lo | ((uint32_t)hi << 16);
        }
      } else {
        *reinterpret_cast<float2 *>(dst) = make_float2(o0, o1);
      }
    };
    auto rec_at = [&](int k) {  // record of piece k of this unit
      const int id = by_piece ? rec0 + k : 2 * (rec0 + k) + (k == 0 ? 1 : 0);
      return a.rec + (size_t)id * G * (D + 2);
    };
    for (int e = tid; e < G * D / 2; e += NT) {
      const int gg = e / (D / 2), d = 2 * (e - gg * (D / 2));
      float M = kEmptyMax;
      for (int sI = 0; sI < n_states; ++sI) M = fmaxf(M, state(sI)[gg * SF]);
      float L = 0.f, A0 = 0.f, A1 = 0.f;
      for (int sI = 0; sI < n_states; ++sI) {
        const AG_LDS float *h = state(sI) + gg * SF;
        const float w = exp2f(h[0] - M);
        L = fmaf(w, h[1], L);
        A0 = fmaf(w, h[4 + d], A0);
        A1 = fmaf(w, h[5 + d], A1);
      }
      if (n_rec == 1) {
        store_out(gg, d, A0 / L, A1 / L);
      } else {
        float *r = rec_at(my_rec) + gg * (D + 2);
        put_pair(r + d, A0, A1);
        if (d == 0) put_pair(r + D, M, L);
      }
    }
    if (n_rec > 1) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's part of the record is in memory
      __syncthreads();
      if (tid == 0)
        s_last = __hip_atomic_fetch_add(&a.tickets[u], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_rec - 1;
      __syncthreads();
      if (s_last) {  // all pieces are there: add them in order
        if (tid == 0) a.tickets[u] = 0;  // ready for the next launch
        for (int e = tid; e < G * D / 2; e += NT) {
          const int gg = e / (D / 2), d = 2 * (e - gg * (D / 2));
          float M = kEmptyMax, L = 0.f, A0 = 0.f, A1 = 0.f;
          for (int k0 = 0; k0 < n_rec; k0 += 8) {
            float2 ml[8], o[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const float *r = rec_at(min(k0 + j, n_rec - 1)) + gg * (D + 2);
              ml[j] = get_pair(r + D);
              o[j] = get_pair(r + d);
            }
            float M_new = M;
#pragma unroll
            for (int j = 0; j < 8; ++j) M_new = fmaxf(M_new, ml[j].x);
            const float keep = exp2f(M - M_new);
            M = M_new;
            L *= keep; A0 *= keep; A1 *= keep;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const float w = k0 + j < n_rec ? exp2f(ml[j].x - M) : 0.f;
              L = fmaf(w, ml[j].y, L);
              A0 = fmaf(w, o[j].x, A0);
              A1 = fmaf(w, o[j].y, A1);
            }
          }
          store_out(gg, d, A0 / L, A1 / L);
        }
      }
    }
    if (first_piece) {  // the new token: its cache row (nobody reads past len in this launch) and its ring slot
      if (keep_new && sl < 0) {
        if (tid < 2 * CPT) reinterpret_cast<uint4 *>(static_cast<T *>(tid < CPT ? a.kc : a.vc) + (size_t)(ro + n) * D)[tid % CPT] = new_row;
        if (tid == 0) a.idx[ro + n] = a.pos;
      } else if (keep_new && tid == 0) {
        atomicOr(a.d_err, 1);
      }
      if (has_ring) {  // slot pos % n_recent held position pos - n_recent, which no query sees any more
        const size_t slot = (size_t)u * a.ring.n + (size_t)(a.pos % a.ring.n);
        if (tid < 2 * CPT)
          put16(reinterpret_cast<uint8_t *>(static_cast<T *>(tid < CPT ? a.ring.k : a.ring.v) + slot * D) + 16 * (tid % CPT), new_row, a.loose);
        if (tid == 0) {
          a.ring.flags[slot] = keep_new ? 1 : 0;
          a.ring.pos[slot] = a.pos;
        }
      }
    }
    __syncthreads();  // the states have been read: the next segment may load over them
    ++u;
    sub = 0;
  }
  // ---- the last workgroup to have read the lengths counts the appended rows ----
  if (tid == 0) s_last = order == (int)gridDim.x - 1;
  __syncthreads();
  if (!s_last) return;
  for (int v = u0; v < u1; ++v)
    if (s_len[v] < 0 && (a.new_flags == nullptr || a.new_flags[v] != 0)) a.len[v] = (s_len[v] & 0x7fffffff) + 1;
  if (tid == 0) *a.arrived = 0;
}

// After prefilling: the ring takes the last min(L, n_recent) prompt tokens of every unit (kept or not); the other
// slots are marked empty.  One workgroup per unit, one wave per token slot in turn.
template <typename T>
__global__ __launch_bounds__(256) void ag_ring_fill_kernel(const T *__restrict__ k, const T *__restrict__ v,
                                                           const uint8_t *__restrict__ flags, int L, int D, int pos0,
                                                           ag_ring_dev ring) {
  const int u = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int w = wave; w < ring.n; w += 4) {
    // slot w holds the position p with p % n == w among the last n positions before pos0 + L, if it is a prompt token
    const int end = pos0 + L;                                   // first position after the prompt
    const int p = end - 1 - ((end - 1 - w) % ring.n + ring.n) % ring.n;  // largest p < end with p % n == w
    const int t = p - pos0;
    const size_t slot = (size_t)u * ring.n + w;
    if (t >= 0 && t < L && p >= 0) {
      for (int d = lane; d < D; d += 64) {
        static_cast<T *>(ring.k)[slot * D + d] = k[((size_t)u * L + t) * D + d];
        static_cast<T *>(ring.v)[slot * D + d] = v[((size_t)u * L + t) * D + d];
      }
      if (lane == 0) { ring.flags[slot] = flags[(size_t)u * L + t] != 0; ring.pos[slot] = p; }
    } else if (lane == 0) {
      ring.flags[slot] = 1;
      ring.pos[slot] = kRingEmpty;
    }
  }
}

int64_t max_records(int units, int64_t cache_rows) { return cache_rows / kChunk + units; }

template <typename T, int D, int G, int NW>
hipError_t launch_nw(ag_ctx *ctx, hipStream_t s, dec_args a, int64_t total_rows, int64_t records) {
  typedef typename wave_of<T, D, G>::type wave_t;
  const size_t shmem = (size_t)NW * wave_t::kWaveB + (size_t)a.U * 4;
  // one workgroup per CU (8 waves) or two (4 waves); no more than the step can have pieces
  const int64_t pieces = a.U + total_rows / (2 * NW * kTileRows) + 1;
  const int blocks = (int)std::min<int64_t>(NW == 8 ? ctx->num_cu : 2 * ctx->num_cu, pieces);
  a.max_wgs = (int)std::max<int64_t>(1, std::min<int64_t>(records / 2, blocks));
  if (shmem > 48 * 1024) {
    static std::atomic<size_t> allowed[64];  // per device: the largest size asked for so far
    std::atomic<size_t> &most = allowed[ctx->device & 63];
    if (most.load(std::memory_order_relaxed) < shmem) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&ag_decode_kernel<T, D, G, NW>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
      if (e != hipSuccess) return e;
      most.store(shmem, std::memory_order_relaxed);
    }
  }
  // (both timing ids report this launch: the merge is part of it)
  ag_tick(ctx, AG_K_DECODE_MERGE, s);
  AG_LAUNCH(ag_time_kernel(ctx, AG_K_DECODE_PARTIAL), (ag_decode_kernel<T, D, G, NW>), dim3(blocks), dim3(64 * NW), shmem, s, a);
  ag_tock(ctx, AG_K_DECODE_MERGE, s);
  return hipGetLastError();
}

template <typename T, int D, int G>
hipError_t launch_t(ag_ctx *ctx, hipStream_t s, dec_args a, int64_t total_rows, ws_cursor &ws) {
  const int64_t records = max_records(a.U, total_rows);
  a.rec = ws.take<float>((size_t)records * G * (D + 2));
  if (!ws.ok) return hipSuccess;
  return a.U <= kFewUnits ? launch_nw<T, D, G, 8>(ctx, s, a, total_rows, records) : launch_nw<T, D, G, 4>(ctx, s, a, total_rows, records);
}

template <typename T, int D>
hipError_t launch_g(int G, ag_ctx *ctx, hipStream_t s, const dec_args &a, int64_t total_rows, ws_cursor &ws) {
  switch (G) {
    case 1: return launch_t<T, D, 1>(ctx, s, a, total_rows, ws);
    case 2: return launch_t<T, D, 2>(ctx, s, a, total_rows, ws);
    case 4: return launch_t<T, D, 4>(ctx, s, a, total_rows, ws);
    case 8: return launch_t<T, D, 8>(ctx, s, a, total_rows, ws);
  }
  return hipErrorInvalidValue;
}

}  // namespace

// Records: one per 128 cache rows and one per unit cover what the kernel can cut (see launch_nw).
size_t ag_ws_decode_bytes(int units, int G, int D, int64_t cache_rows) {
  const int64_t records = max_records(units, cache_rows);
  return ag_align256((size_t)(units + 1) * 4) + 2 * ag_align256((size_t)records * G * 4) +
         ag_align256((size_t)records * G * D * 4);
}

// Device address of this GPU's copy of `scratch`, looked up once per device (with that device current) and kept.
hipError_t ag_static_scratch(int device, char **ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static char *known[kMaxDevices];
  *ptr = nullptr;
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!known[device]) {
    hipError_t e = hipSetDevice(device);
    if (e != hipSuccess) return e;
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    known[device] = static_cast<char *>(p);
  }
  *ptr = known[device];
  return hipSuccess;
}

bool ag_decode_supported(ag_dtype dt, int D, int G, int units) {
  if (units > kDecodeMaxUnits) return false;
  if (!(G == 1 || G == 2 || G == 4 || G == 8)) return false;
  return dt == AG_BF16 ? (D == 64 || D == 128) : (D == 64 || D == 128);
}

hipError_t ag_launch_decode(ag_ctx *ctx, hipStream_t s, const void *q, const void *k_new, const void *v_new,
                            const uint8_t *new_flags, int pos, int B, int Hq, int Hkv, int D, ag_dtype dt,
                            float scale, void *kc, void *vc, int32_t *idx, const int64_t *row_off, int32_t *len,
                            int64_t total_rows, void *out, ws_cursor &ws, ag_ring_dev ring) {
  dec_args a;
  a.q = q; a.k_new = k_new; a.v_new = v_new; a.new_flags = new_flags;
  a.kc = kc; a.vc = vc; a.idx = idx; a.row_off = row_off; a.len = len; a.out = out;
  a.rec = nullptr; a.tickets = ctx->decode_tickets; a.arrived = ctx->decode_tickets + kDecodeMaxUnits; a.d_err = ctx->d_err;
  a.U = B * Hkv; a.pos = pos; a.max_wgs = 1;
  a.qscale = scale * kLog2e;
  a.loose = dt == AG_BF16 && (((uintptr_t)k_new | (uintptr_t)v_new | (uintptr_t)out | (uintptr_t)ring.k | (uintptr_t)ring.v) & 15) != 0;
  a.ring = ring;
#define AG_DEC(T, DD) return launch_g<T, DD>(Hq / Hkv, ctx, s, a, total_rows, ws)
  if (dt == AG_BF16) {
    if (D == 64) AG_DEC(uint16_t, 64);
    if (D == 128) AG_DEC(uint16_t, 128);
  } else {
    if (D == 64) AG_DEC(float, 64);
    if (D == 128) AG_DEC(float, 128);
  }
#undef AG_DEC
  return hipErrorInvalidValue;
}

hipError_t ag_launch_ring_fill(hipStream_t s, const void *k, const void *v, const uint8_t *flags, int units, int L,
                               int D, ag_dtype dt, int pos0, ag_ring_dev ring) {
  if (dt == AG_BF16)
    hipLaunchKernelGGL(ag_ring_fill_kernel<uint16_t>, dim3(units), dim3(256), 0, s, (const uint16_t *)k,
                       (const uint16_t *)v, flags, L, D, pos0, ring);
  else
    hipLaunchKernelGGL(ag_ring_fill_kernel<float>, dim3(units), dim3(256), 0, s, (const float *)k, (const float *)v,
                       flags, L, D, pos0, ring);
  return hipGetLastError();
}
