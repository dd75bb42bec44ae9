// Decode attention over ragged per-(batch, KV head) caches (Sec. 3.1, decoding stage), one launch per step.
//
// A step reads every cached K and V row once: large batches are bound by HBM, small ones by the number of dependent
// round trips.  The kernel therefore does everything in one launch -- it builds its own work list from len[] (no host
// read-back), streams the rows, merges, takes in the new token and appends it -- and hands data between workgroups only
// where a unit is too long for one.
//   * Work is counted in tiles of 32 rows (fp32: mostly 16) of one unit; a wave takes every NW-th tile of its workgroup's segment, so the
//     waves run without a barrier until their segment ends.  The slots of the recent-token ring are extra tiles in front
//     of a unit's cache rows; the new token's own key and value (the diagonal of Eq. 5) are the state one wave starts from.
//   * bf16 runs on MFMA: K and V rows go from memory to the wave's own LDS by direct loads (whole rows; the next tile's K
//     is requested as soon as this tile's fragments are read, its V after the second product's, so 8 to 16 KiB per
//     wave are always in flight and no register holds them), S^T = K q^T and O^T = V^T p^T for all G query heads of the
//     group at once.  p enters the second product as three bf16 numbers whose sum it is (three MFMAs): the weights keep
//     their 24 bits, as in a 32-bit product.  Measured against 64 bits over 64 units of up to 2000 rows, rms error over rms
//     sum of p |v|: 0.9e-8 to 1.0e-8, as with products and sums on the vector ALU; with two bf16 numbers 3e-7.  (Third number:
//     0.35 us per step of 8 units of up to 777 rows, nothing where memory is the bound.)  fp32 caches run on the vector ALU.
//   * Segments (what a workgroup works on between two merges) are chosen on the device.  If the whole step gives every
//     workgroup at most one segment -- a unit of up to 2 rounds of its waves (kWholeRounds) stays whole, a longer one is cut into the
//     smallest pieces that fit the launch -- a unit's pieces meet once; otherwise the tiles of all units are laid end to end and cut
//     into equal ranges, one per workgroup, and only the units at the cuts cross workgroups.  More than kFewUnits units of a
//     few rounds each are given to four, two or one wave each instead, all at once.
//   * A unit inside one workgroup is finished there, through LDS.  The pieces of a longer one are stored as records
//     (written through, complete before the arrival is counted); the piece that arrives last merges them in order.
//   * A short step costs instructions as much as memory round trips (two waves share a SIMD, so each vector instruction of
//     the straight-line path is 8 cycles): up to 128 units every wave builds the work list in its own registers, without
//     LDS and barriers, and all addresses are one XOR away from a base.
#include <algorithm>
#include <atomic>
#include <mutex>
#include <type_traits>

#include "ag_internal.h"

// Scratch of ag_decode_attn_static, the entry point for callers that cannot allocate: the records that the pieces of a
// unit exchange live here instead of in a context's workspace.  One copy per GPU, held until the
// process ends.  In host code this name is only a stand-in for the symbol; the device address comes from
// hipGetSymbolAddress (ag_static_scratch below) and is what every launch receives.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

constexpr int kChunk = 128;      // cache rows per record of scratch space (ag_decode_scratch_bytes)
// Up to here 8 waves per workgroup and one workgroup per CU: a unit's rows are spread over as many waves as LDS can feed; beyond,
// 4 waves and two workgroups per CU, so that one streams while the other merges.  (160 to 256 units on 8 waves: whole workgroups
// for short units, 256 of up to 100 rows 10.9 us against 7.2 on 4; equal ranges for long ones, 224 of up to 700 rows 20.8 against
// 12.6.  128 units are level.  fp32, four heads of 128 per unit: 160 units of up to 500 rows 17.7 us on 8 waves, 24.7 on 4; 256 of
// up to 30 rows 10.9 and 9.1, of up to 1000 rows 40.1 and 38.7.)
template <typename T> constexpr int kFewUnits = sizeof(T) == 2 ? 128 : 192;
// Reference maximum before any row: the least finite number, so that no state that holds a row is below it (differences of
// maxima stay numbers or become -infinity, of which the exponential is 0).
constexpr float kEmptyMax = -3.40282347e+38f;
constexpr int kArriveSplit = 64; // workgroups (of 4 waves) from which their arrivals are counted at several addresses
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
// the first 16 bits of two words, lo's in the lower half
__device__ __forceinline__ uint32_t high_halves(uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x07060302u); }

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
template <int D> __device__ __forceinline__ constexpr int tile_key(int r) {
  return D == 128 ? (((r & 7) << 1) | ((r >> 3) & 1)) : ((((r >> 1) & 3) << 1) | ((r >> 3) & 1));
}

// Reductions over the four lanes that share lane % 16 (v_permlane*_swap: a register exchange, no LDS round trip)
__device__ __forceinline__ float kg_max(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float kg_sum(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// The maximum that the state of the new token's own key starts from.  Alone (no cache row, no ring slot seen) its weight is 1
// whatever its score is; a score that overflowed to -infinity counts as the least finite one; NaN stays NaN.
__device__ __forceinline__ float own_max(float s, bool alone) { return alone ? 0.f : (s < kEmptyMax ? kEmptyMax : s); }

// What a tile reads: up to 32 rows of k and v; those whose bit in `vis` is clear are not seen (wave-uniform).
struct dec_tile {
  const void *k, *v;  // the tile's first row (64-bit addresses: a unit's rows may span more than the 4 GiB a descriptor can)
  uint32_t bytes;     // cache rows: size of the rows that exist (the others read as zeros)
  uint32_t vis;
  bool ring;          // ring slots: rows whose bit is clear are not even read (they may hold anything)
};

// ---- bf16: one wave's pass over its tiles on MFMA -----------------------------------------------------------
// Lane = (query head q = lane % 16, key group kg = lane / 16); heads q >= G are zero columns.  EVEN: the caches start at an
// even address that is no multiple of 16; their rows go through registers (direct loads into LDS are not used for those).
template <int D, int G, bool EVEN> struct wave_bf16 {
  static constexpr int kTileRows = 32;                                   // rows a wave takes at a time
  static constexpr int kRowB = D * 2, CPR = kRowB / 16, RPI = 64 / CPR;  // RPI rows per load instruction
  static constexpr int NL = kTileRows / RPI;                             // load instructions per tile and operand
  static constexpr int kWaveB = 2 * kTileRows * kRowB;                   // the wave's LDS: K tile, V tile
  static constexpr int kStateF = D + 4;                                  // floats per head of the state a wave leaves
  // rounds of the workgroup's waves up to which a unit stays whole, and up to which it is left to a team (see the kernel)
  static constexpr int kWholeRounds = kRowB >= 256 ? 2 : 4, kTeamRounds = 8;
  static constexpr int KS = D / 32, DT = D / 16;
  bf16x8 qf[KS];
  f32x4 o[DT];
  float m, l;
  int ld_base, k_base, v_base;  // every offset below is one of these XOR a constant (rows only add constants)
  uint32_t lds_addr;
  AG_LDS uint8_t *lds;
  int lane, kg, col;

  // load instruction i, lane (row lr = lane / CPR of its RPI rows, position lane % CPR) fetches chunk
  // (lane % CPR) ^ key(RPI i + lr) of that row; key(RPI i + lr) = key(lr) ^ key(RPI i)
  __device__ __forceinline__ int ld_off(int i) const { return ld_base ^ (tile_key<D>(RPI * i) << 4); }
  // K fragment (A of S^T), k-step ks: row col (+ 16), chunk 4 ks + kg
  __device__ __forceinline__ int k_off(int ks) const { return k_base ^ (ks << 6); }
  // V fragment (A of O^T) by transposing read: rows 4 kg + 0..3 (+ 16), columns 16 dt + 0..15
  __device__ __forceinline__ int v_off(int dt) const { return v_base ^ (dt << 5); }

  __device__ __forceinline__ void init(AG_LDS uint8_t *mem, int lane_) {
    lane = lane_; kg = lane >> 4; col = lane & 15;
    lds = mem;
    lds_addr = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)mem);
    const int lr = lane / CPR, vr = 4 * kg + (col >> 2);
    ld_base = lr * kRowB + (((lane % CPR) ^ tile_key<D>(lr)) << 4);
    k_base = col * kRowB + ((kg ^ tile_key<D>(col)) << 4);
    v_base = vr * kRowB + ((((col & 3) >> 1) ^ tile_key<D>(vr)) << 4) + (col & 1) * 8;
    m = kEmptyMax; l = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // Cache rows of one operand straight into LDS; rows past the array arrive as zeros.  Every cached row is read once per
  // step: non-temporal, so that the stream does not push the small hot data (queries, lengths, records) out of the caches.
  __device__ __forceinline__ void load(const dec_tile &t, const void *base, int to) {
    const uint64_t at = (uint64_t)base;  // (wave-uniform, as the loads need it; said explicitly)
    const uint64_t base_s = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)at) |
                            ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(at >> 32)) << 32);
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void *)base_s, 0, __builtin_amdgcn_readfirstlane(t.bytes), 0x00020000);
    if constexpr (EVEN) {
      u32x4 x[NL];
#pragma unroll
      for (int i = 0; i < NL; ++i) x[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, ld_off(i) + i * RPI * kRowB, 0, 0);
#pragma unroll
      for (int i = 0; i < NL; ++i) *reinterpret_cast<AG_LDS u32x4 *>(lds + to + i * RPI * kRowB + lane * 16) = x[i];
      return;
    }
    const uint32_t dst = lds_addr + to;
#pragma unroll
    for (int i = 0; i < NL; ++i)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                   :: "s"(dst + i * RPI * kRowB), "v"(ld_off(i)), "s"(rsrc), "s"(i * RPI * kRowB) : "m0", "memory");
  }
  __device__ __forceinline__ void load_k(const dec_tile &t) { load(t, t.k, 0); }
  __device__ __forceinline__ void load_v(const dec_tile &t) { load(t, t.v, kTileRows * kRowB); }
  // Ring slots, through registers: only the visible rows are read, the others become zeros.
  __device__ __forceinline__ void load_ring(const dec_tile &t, bool loose) {
    uint4 x[2][NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const bool see = (t.vis >> (RPI * i + lane / CPR)) & 1u;
#pragma unroll
      for (int kv = 0; kv < 2; ++kv) {
        x[kv][i] = make_uint4(0, 0, 0, 0);
        if (see)
          x[kv][i] = chunk16(static_cast<const uint8_t *>(kv ? t.v : t.k) + i * RPI * kRowB + ld_off(i), loose);
      }
    }
#pragma unroll
    for (int kv = 0; kv < 2; ++kv)
#pragma unroll
      for (int i = 0; i < NL; ++i)
        *reinterpret_cast<AG_LDS u32x4 *>(lds + (kv * kTileRows + i * RPI) * kRowB + lane * 16) =
            u32x4{x[kv][i].x, x[kv][i].y, x[kv][i].z, x[kv][i].w};
  }

  // Tiles first, first + step, ... < last of the segment; get(i) describes tile i.  q: the G query rows of the unit.
  // own: start from the new token's key and value instead of from nothing; alone: nothing else is seen (see own_max).
  // (a ring tile can only be a wave's first: there are no more of them than waves)
  template <typename GET>
  __device__ __forceinline__ void run(const uint16_t *q, int first, int last, int step, float qscale, bool own, bool alone,
                                      const uint16_t *k_new, const uint16_t *v_new, bool loose, GET &&get) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      uint4 x = make_uint4(0, 0, 0, 0);
      if (col < G) x = *reinterpret_cast<const uint4 *>(q + (size_t)col * D + 32 * ks + 8 * kg);
      qf[ks] = __builtin_bit_cast(bf16x8, x);
    }
    uint4 kn[KS];
    uint2 vn[DT];
    if (own) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kn[ks] = chunk16(reinterpret_cast<const uint8_t *>(k_new + 32 * ks + 8 * kg), loose);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const uint16_t *v = v_new + 16 * dt + 4 * kg;
        if (!loose) vn[dt] = *reinterpret_cast<const uint2 *>(v);
        else vn[dt] = make_uint2((uint32_t)v[0] | ((uint32_t)v[1] << 16), (uint32_t)v[2] | ((uint32_t)v[3] << 16));
      }
    }
    dec_tile t = get(first);
    if (first < last) {
      if (t.ring) {
        load_ring(t, loose);
      } else {
        load_k(t);
        load_v(t);
      }
    }
    // the query's loads are waited for here, once: the compiler would otherwise put a wait for everything into the loop
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[ks]));
    if (own) {
      float s = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const uint4 qa = __builtin_bit_cast(uint4, qf[ks]);
        s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, qa.x), __builtin_bit_cast(bf16x2, kn[ks].x), s, false);
        s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, qa.y), __builtin_bit_cast(bf16x2, kn[ks].y), s, false);
        s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, qa.z), __builtin_bit_cast(bf16x2, kn[ks].z), s, false);
        s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, qa.w), __builtin_bit_cast(bf16x2, kn[ks].w), s, false);
      }
      m = own_max(kg_sum(s) * qscale, alone);
      l = kg == 0 ? 1.f : 0.f;  // (summed over the key groups at the end)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
        o[dt] = f32x4{__uint_as_float(vn[dt].x << 16), __uint_as_float(vn[dt].x & 0xffff0000u),
                      __uint_as_float(vn[dt].y << 16), __uint_as_float(vn[dt].y & 0xffff0000u)};
    }
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
          kf[sub][ks] = *reinterpret_cast<const AG_LDS bf16x8 *>(lds + sub * 16 * kRowB + k_off(ks));
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (more) load_k(t);
      f32x4 s[2];
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) {
        // (two sums of half as many terms: one of all four k-steps doubles the weights' error against 64 bits)
        f32x4 h2[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) h2[ks & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[sub][ks], qf[ks], h2[ks & 1], 0, 0, 0);
        s[sub] = h2[0] + h2[1];
      }
      // s[sub][r]: key 16 sub + 4 kg + r, head col
      float p[8], mx = -INFINITY;
#pragma unroll
      for (int e = 0; e < 8; ++e) p[e] = s[e >> 2][e & 3] * qscale;
      if (vis != 0xffffffffu) {
        const uint32_t mine = vis >> (4 * kg);
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (!((mine >> (16 * (e >> 2) + (e & 3))) & 1u)) p[e] = -INFINITY;
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) mx = fmaxf(mx, p[e]);
      const float m_new = fmaxf(m, kg_max(mx));
      if (__any(m_new != m)) {
        const float alpha = __builtin_amdgcn_exp2f(m - m_new);
        l *= alpha;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[dt] *= alpha;
        m = m_new;
      }
      // p = the sum of three bf16 numbers, exactly: each takes the first 8 bits of a number just below what is left (so that
      // something is left, down to the last: where p is not 0 all three are positive, and an infinite value comes out of the
      // three products with the same sign, as it would of one).
      uint32_t pw[3][8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        p[e] = __builtin_amdgcn_exp2f(p[e] - m);
        l += p[e];
        float rest = p[e];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          pw[i][e] = __builtin_elementwise_sub_sat(__float_as_uint(rest), 1u);  // (its first 16 bits)
          rest -= __uint_as_float(pw[i][e] & 0xffff0000u);
        }
        pw[2][e] = __float_as_uint(rest);  // (its last 16 bits are 0)
      }
      uint4 pt[3];
#pragma unroll
      for (int i = 0; i < 3; ++i)
        pt[i] = make_uint4(high_halves(pw[i][0], pw[i][1]), high_halves(pw[i][2], pw[i][3]), high_halves(pw[i][4], pw[i][5]),
                           high_halves(pw[i][6], pw[i][7]));
      if (more)
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"(NL) : "memory");  // V has landed (the next K may not have)
      else
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      bf16x8 vf[DT];  // row d = 16 dt + col of V^T, keys 4 kg + 0..3 and 16 + 4 kg + 0..3
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const AG_LDS uint8_t *base = lds + kTileRows * kRowB + v_off(dt);
        const bf16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((AG_LDS bf16x4 *)base);
        const bf16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((AG_LDS bf16x4 *)(base + 16 * kRowB));
        vf[dt] = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (more) load_v(t);
#pragma unroll
      for (int i = 2; i >= 0; --i)  // (the small parts first)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
          o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[dt], __builtin_bit_cast(bf16x8, pt[i]), o[dt], 0, 0, 0);
    }
  }
  // the wave's state into its LDS: per head [max, sum, -, -, o[0..D)]
  __device__ __forceinline__ void leave(AG_LDS float *st) {
    l = kg_sum(l);
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
  // A round of 16 rows per wave takes up to 5 us (eight heads of 128: 64 products of 128 terms per lane group, and the next loads wait
  // behind them), so tiles are what one batch of loads covers and little of a round is left over.  8 units of up to 500 rows, four
  // and eight heads of 128 per unit: 21.3 and 34.9 us a step with tiles of 32 rows and units whole up to two rounds, 11.2 and 15.7
  // with these; one head of 64 (32-row tiles): up to 1000 rows 7.5 whole up to two rounds, 9.6 up to four.  Teams: 256 units of up
  // to 186 rows (three rounds), four and eight heads of 128: 14.8 and 22.0 us at once, 24.1 and 36.5 in equal ranges; at 8 (4) rounds
  // about level; one head of 128 at 16 rounds 32.4 at once, 27.5 in ranges.
  static constexpr int UN = G <= 2 ? 8 : 4;                      // rows in flight per lane group
  static constexpr int kTileRows = UN * GPW > 16 ? UN * GPW : 16;
  static constexpr int kWholeRounds = G * D >= 256 ? 1 : 2, kTeamRounds = G * D >= 1024 ? 4 : 8;
  static constexpr int NIT = kTileRows / GPW;                    // loads that cover a tile
  static constexpr int kStateF = D + 4;
  static constexpr int kWaveB = G * kStateF * 4;
  float4 qr[G];
  float m[G], l[G], acc[G][EPL];
  int grp, seg;
  __device__ __forceinline__ void init(AG_LDS uint8_t *, int lane) {
    grp = lane / LPR; seg = lane % LPR;
#pragma unroll
    for (int gg = 0; gg < G; ++gg) {
      m[gg] = kEmptyMax; l[gg] = 0.f;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[gg][e] = 0.f;
    }
  }
  __device__ __forceinline__ float score(const float4 &q, const nt_f32x4 &k, float qscale) {
    float d = q.x * k[0];
    d = fmaf(q.y, k[1], d);
    d = fmaf(q.z, k[2], d);
    return group_sum<LPR>(fmaf(q.w, k[3], d)) * qscale;
  }
  template <typename GET>
  __device__ __forceinline__ void run(const float *q, int first, int last, int step, float qscale, bool own, bool alone,
                                      const float *k_new, const float *v_new, bool, GET &&get) {
#pragma unroll
    for (int gg = 0; gg < G; ++gg) qr[gg] = reinterpret_cast<const float4 *>(q + (size_t)gg * D)[seg];
    if (own) {
      const nt_f32x4 kn = reinterpret_cast<const nt_f32x4 *>(k_new)[seg], vn = reinterpret_cast<const nt_f32x4 *>(v_new)[seg];
#pragma unroll
      for (int gg = 0; gg < G; ++gg) {
        const float s = own_max(score(qr[gg], kn, qscale), alone);
        if (grp == 0) {
          m[gg] = s; l[gg] = 1.f;
#pragma unroll
          for (int e = 0; e < EPL; ++e) acc[gg][e] = vn[e];
        }
      }
    }
    for (int i = first; i < last; i += step) {
      const dec_tile t = get(i);
      const nt_f32x4 *K = reinterpret_cast<const nt_f32x4 *>(t.k) + seg;
      const nt_f32x4 *V = reinterpret_cast<const nt_f32x4 *>(t.v) + seg;
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
            const float d = score(qr[gg], kk[j], qscale);
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
    for (int gg = 0; gg < G; ++gg) {  // the lane groups' states first
      float M = m[gg];
#pragma unroll
      for (int o = LPR; o < 64; o <<= 1) M = fmaxf(M, __shfl_xor(M, o, 64));
      const float w = exp2f(m[gg] - M);
      l[gg] *= w;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[gg][e] *= w;
#pragma unroll
      for (int o = LPR; o < 64; o <<= 1) {
        l[gg] += __shfl_xor(l[gg], o, 64);
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[gg][e] += __shfl_xor(acc[gg][e], o, 64);
      }
      if (grp == 0) {
        AG_LDS float *h = st + gg * kStateF;
        if (seg == 0) { h[0] = M; h[1] = l[gg]; }
        *reinterpret_cast<AG_LDS f32x4 *>(h + 4 + seg * EPL) = f32x4{acc[gg][0], acc[gg][1], acc[gg][2], acc[gg][3]};
      }
    }
  }
};
template <typename T, int D, int G, bool EVEN> struct wave_of;
template <int D, int G, bool EVEN> struct wave_of<uint16_t, D, G, EVEN> { typedef wave_bf16<D, G, EVEN> type; };
template <int D, int G, bool EVEN> struct wave_of<float, D, G, EVEN> { typedef wave_f32<D, G> type; };

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
  int32_t *arrived;     // [kDecodeArriveInts] workgroups that have read len[] (see arrive); zero between launches
  int32_t *d_err;
  int U, pos, max_wgs;  // max_wgs: workgroups the equal-range split may use (two records each)
  int team;             // waves per unit where every unit can have its own (4-wave workgroups; else unused)
  float qscale;
  bool loose;           // k_new, v_new, the ring or out are not 16-byte aligned: they are accessed by elements
  ag_ring_dev ring;
};

// exclusive prefix sum over the wave's lanes (x: the lane's own value); total = the wave's sum
__device__ __forceinline__ int wave_prefix(int x, int &total) {
  int y = x;
  y += __builtin_amdgcn_update_dpp(0, y, 0x111, 0xf, 0xf, false);  // row_shr:1, 2, 4, 8: prefix inside each row of 16
  y += __builtin_amdgcn_update_dpp(0, y, 0x112, 0xf, 0xf, false);
  y += __builtin_amdgcn_update_dpp(0, y, 0x114, 0xf, 0xf, false);
  y += __builtin_amdgcn_update_dpp(0, y, 0x118, 0xf, 0xf, false);
  y += __builtin_amdgcn_update_dpp(0, y, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
  y += __builtin_amdgcn_update_dpp(0, y, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
  total = __builtin_amdgcn_readlane(y, 63);
  return y - x;
}

template <typename T, int D, int G, int NW, bool EVEN>
__global__ __launch_bounds__(64 * NW, 2) void ag_decode_kernel(dec_args a) {
  typedef typename wave_of<T, D, G, EVEN>::type wave_t;
  constexpr int NT = 64 * NW, SF = wave_t::kStateF;
  constexpr int kTileRows = wave_t::kTileRows, kWholeTiles = wave_t::kWholeRounds * NW;
  constexpr int CPT = (int)(D * sizeof(T) / 16);  // 16-byte chunks per row
  constexpr bool kRegs = NW == 8;                 // the work list lives in registers (at most kFewUnits units)
  constexpr int UPL = kFewUnits<T> / 64;             // ... that many units per lane: unit 64 j + lane
  // The arguments lie in three cache lines of memory that may be far away: all of them are requested here, in one trip,
  // instead of one line after the other as the code below comes to need them.
  asm volatile("" :: "s"(a.q), "s"(a.len), "s"(a.U), "s"(a.ring.n));
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  int32_t *s_len = reinterpret_cast<int32_t *>(smem + NW * wave_t::kWaveB);  // (!kRegs) [U] valid rows; top bit: room
  __shared__ int32_t w_sum[NW][2], s_start[2], s_last;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int U = a.U, wg = blockIdx.x;
  const bool has_ring = a.ring.k != nullptr;
  const int extra = has_ring ? (a.ring.n + kTileRows - 1) / kTileRows : 0;

  // ---- the work list: tiles per unit (at least one), and the pieces it is cut into ----
  int piece = NW;  // tiles per piece: `rounds` rounds of the workgroup's waves
  uint32_t piece_inv = (uint32_t)((1ull << 32) / NW);  // ceil(2^32 / piece): x / piece for x piece < 2^32
  auto tiles_of = [&](int n) { return max(1, extra + (int)((unsigned)(n + kTileRows - 1) / kTileRows)); };
  auto pieces_of = [&](int t) { return t <= max(kWholeTiles, piece) ? 1 : (int)__umulhi((uint32_t)(t + piece - 1), piece_inv); };
  auto read_len = [&](int u, int64_t &r0) {  // valid rows of unit u, top bit set if another one fits
    r0 = a.row_off[u];
    const int64_t cap = a.row_off[u + 1] - r0;
    const int n_raw = a.len[u];
    const int n = n_raw < 0 ? 0 : (n_raw < cap ? n_raw : (int)cap);
    return n | (n < cap ? (int)0x80000000 : 0);
  };
  int sl_r[kRegs ? UPL : 1];       // kRegs: this lane's units
  int64_t ro_r[kRegs ? UPL : 1];
  const int per = (U + NT - 1) / NT, u0 = min(U, tid * per), u1 = min(U, u0 + per);  // !kRegs: this thread's units
  int total_t = 0, total_i = 0, u = 0, sub = 0, team = NW, quota = 0, x = 0;
  bool by_piece, idle;
  // The lengths may only change once every workgroup has read them.  Each one counts its arrival when all its waves have
  // (4 waves: after the barrier below; 8 waves, which need no barrier before their first merge: after that), and the one
  // that arrives last counts the appended rows, at its end.
  // At one address that takes 19 ns per workgroup, one after the other, which is the tail of a short step with one for every
  // unit (264 units of up to 186 rows: 13.8 -> 9.4 us, 512: 14.9 -> 10.8): there they count at kDecodeArriveGroups addresses,
  // and the last ones of those at one more.  With 8 waves, which count late and are fewer, the second trip costs more than it
  // saves (64 units of up to 300 rows: 8.1 us, with it 9.1).
  const int groups = !kRegs && (int)gridDim.x >= kArriveSplit ? kDecodeArriveGroups : 1;
  int order = -1;  // (thread 0) place of this workgroup among those that count where it does
  auto arrive = [&] {
    order = __hip_atomic_fetch_add(a.arrived + (groups == 1 ? 0 : kDecodeArriveStride * (1 + wg % kDecodeArriveGroups)), 1,
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  if constexpr (kRegs) {
    int base_t[UPL], base_i[UPL], cnt_t[UPL], cnt_i[UPL];
#pragma unroll
    for (int j = 0; j < UPL; ++j) {
      sl_r[j] = 0; ro_r[j] = 0;
      if (64 * j < U && 64 * j + lane < U) sl_r[j] = read_len(64 * j + lane, ro_r[j]);
    }
#pragma unroll
    for (int j = 0; j < UPL; ++j) {
      base_t[j] = cnt_t[j] = 0;
      if (64 * j < U) {
        int sum_t;
        cnt_t[j] = 64 * j + lane < U ? tiles_of(sl_r[j] & 0x7fffffff) : 0;
        base_t[j] = total_t + wave_prefix(cnt_t[j], sum_t);
        total_t += sum_t;
      }
    }
    // The smallest pieces that the launch has workgroups for: the rounds of an even spread if they fit, else what is sure
    // to.  A round costs a workgroup about 1 us (what one CU's LDS keeps in flight), the meeting of a unit's pieces about
    // as much, so units of up to two rounds of 16 KiB stay whole.  Measured on 8 units of up to 777 rows of 256 bytes:
    // 7.9 us per step in pieces of one round, 8.4 us whole; rows of 128 bytes: 8.2 us and 7.4 us.
    const int grid = gridDim.x;
    bool last_try = false;
    int rounds = 1;
    if (total_t > NW * grid) rounds = (int)((unsigned)(total_t + NW * grid - 1) / (unsigned)(NW * grid));
    for (;;) {
      if (rounds > 1) {
        piece = rounds * NW;
        piece_inv = 0xffffffffu / (unsigned)piece + 1u;
      }
      total_i = 0;
#pragma unroll
      for (int j = 0; j < UPL; ++j) {
        base_i[j] = cnt_i[j] = 0;
        if (64 * j < U) {
          int sum_i;
          cnt_i[j] = 64 * j + lane < U ? pieces_of(cnt_t[j]) : 0;
          base_i[j] = total_i + wave_prefix(cnt_i[j], sum_i);
          total_i += sum_i;
        }
      }
      if (total_i <= grid || last_try || U >= grid) break;
      rounds = max(rounds, (int)((unsigned)(total_t + NW * (grid - U) - 1) / (unsigned)(NW * (grid - U))));
      last_try = true;
    }
    // ... unless there are so many units that the remainders of their last pieces weigh more than equal ranges cost
    by_piece = total_i <= grid && (rounds <= 2 || 4 * U <= grid);
    if (!by_piece) {
      const int wgs = min((int)gridDim.x, a.max_wgs);
      quota = (int)((unsigned)(total_t + wgs - 1) / (unsigned)wgs);
    }
    x = by_piece ? wg : wg * quota;  // the piece or the tile this workgroup starts at
    idle = by_piece ? x >= total_i : x >= total_t;
#pragma unroll
    for (int j = 0; j < UPL; ++j)
      if (64 * j < U) {
        const int bi = base_i[j], bt = base_t[j], ci = cnt_i[j], ct = cnt_t[j];
        const int b = by_piece ? bi : bt, c = by_piece ? ci : ct;
        const uint64_t hit = __ballot(b <= x && x < b + c);  // at most one unit
        if (hit) {
          const int at = __builtin_ctzll(hit);
          u = 64 * j + at;
          sub = x - __builtin_amdgcn_readlane(b, at);  // piece or tile inside the unit
        }
      }
  } else {
    int my_t = 0, max_t = 0;
    for (int v = u0; v < u1; ++v) {
      int64_t r0;
      const int sl = read_len(v, r0), t = tiles_of(sl & 0x7fffffff);
      s_len[v] = sl;
      my_t += t;
      max_t = max(max_t, t);
    }
    int sum_t;
    const int pre = wave_prefix(my_t, sum_t);
    for (int o = 32; o > 0; o >>= 1) max_t = max(max_t, __shfl_xor(max_t, o, 64));
    if (lane == 0) { w_sum[wave][0] = sum_t; w_sum[wave][1] = max_t; }
    __syncthreads();
    if (tid == 0) arrive();
    int base = pre;
    max_t = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      if (w < wave) base += w_sum[w][0];
      total_t += w_sum[w][0];
      max_t = max(max_t, w_sum[w][1]);
    }
    // Every unit at once, on a.team waves each, if none of them takes longer than 8 (kTeamRounds) rounds of those: then one pass
    // (no merges, or one of two or four waves) is cheaper than several units one after the other on the whole workgroup.
    // (6 rounds of 16 KiB where a few CUs would get a second unit and the others wait for them: 264 units of up to 1000 rows
    // of 256 bytes 22.4 us at once, 20.5 in equal ranges; from 300 units on the launch is even enough.)
    const int most = sizeof(T) == 2 && D == 128 && 2 * U > (int)gridDim.x && 16 * U <= 9 * (int)gridDim.x ? 6 : wave_t::kTeamRounds;
    by_piece = (int64_t)U * a.team <= (int64_t)gridDim.x * NW && max_t <= most * a.team && (!has_ring || a.ring.n <= 32 * a.team);
    if (by_piece) {
      team = a.team;
      u = wg * (NW / team) + wave / team;
      idle = wg * (NW / team) >= U;
    } else {
      const int wgs = min((int)gridDim.x, a.max_wgs);
      quota = (int)((unsigned)(total_t + wgs - 1) / (unsigned)wgs);
      x = wg * quota;
      idle = x >= total_t;
      if (base <= x && x < base + my_t) {  // exactly one thread, if x < total_t
        int at = base, v = u0;
        for (;; ++v) {
          const int t = tiles_of(s_len[v] & 0x7fffffff);
          if (x < at + t) break;
          at += t;
        }
        s_start[0] = v;
        s_start[1] = x - at;
      }
      __syncthreads();
      if (!idle) { u = s_start[0]; sub = s_start[1]; }
    }
  }

  // (in a team of fewer waves than the workgroup: lanes and waves of the team)
  const int wt = team == NW ? wave : wave & (team - 1), tt = wt * 64 + lane;
  AG_LDS uint8_t *my_lds = (AG_LDS uint8_t *)smem + wave * wave_t::kWaveB;
  AG_LDS uint8_t *team_lds = (AG_LDS uint8_t *)smem + (wave - wt) * wave_t::kWaveB;
  int left = idle || by_piece ? 0 : min(quota, total_t - x);  // tiles still to do
  int at = x;
  // One segment: a whole unit or a piece of it (PIECE, at most one per workgroup or team), or the next part of the
  // workgroup's range.  Two copies of the code: the one for pieces is straight-line, without the loop whose invariants the
  // compiler would compute, and spill, in front of it (a third of a short step; 60 to 77 scalar registers are spilled still).
  auto segment = [&](auto piece_mode) {
    constexpr bool PIECE = decltype(piece_mode)::value;
    u = __builtin_amdgcn_readfirstlane(u);
    const bool mine = kRegs || u < U;  // (a team past the last unit only takes part in the barriers)
    int sl = 0;
    int64_t ro = 0;
    if constexpr (kRegs) {
#pragma unroll
      for (int j = 0; j < UPL; ++j)
        if ((u >> 6) == j) {
          sl = __builtin_amdgcn_readlane(sl_r[j], u & 63);
          ro = (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)ro_r[j], u & 63) |
                         ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(ro_r[j] >> 32), u & 63) << 32));
        }
    } else if (mine) {
      sl = __builtin_amdgcn_readfirstlane(s_len[u]);
      ro = a.row_off[u];
    }
    const int n = sl & 0x7fffffff;
    const int T_u = tiles_of(n);
    int t0 = 0, t1 = mine ? T_u : 0, rec0 = 0, n_rec = 1, my_rec = 0;  // tiles [t0, t1) of the unit; its records, this one's number
    if constexpr (PIECE && kRegs) {
      n_rec = pieces_of(T_u);
      my_rec = sub;
      rec0 = wg - sub;
      if (n_rec > 1) {
        t0 = sub * piece;
        t1 = min(T_u, t0 + piece);
      }
    }
    if constexpr (!PIECE) {
      t0 = sub;
      t1 = min(T_u, t0 + left);
      left -= t1 - t0;
      const int first = at - t0;  // the unit's first tile, counted over all units
      at += t1 - t0;
      if (t0 > 0 || t1 < T_u) {   // a unit at one of the cuts
        const int g0 = (int)((unsigned)first / (unsigned)quota), g1 = (int)((unsigned)(first + T_u - 1) / (unsigned)quota);
        n_rec = g1 - g0 + 1;
        my_rec = wg - g0;
        rec0 = g0;
      }
    }
    const T *kn = static_cast<const T *>(a.k_new) + (size_t)u * D, *vn = static_cast<const T *>(a.v_new) + (size_t)u * D;
    const bool first_piece = mine && t0 == 0;  // this workgroup takes the new token in
    // requested now, used at the segment's end
    uint4 new_row = make_uint4(0, 0, 0, 0);
    int new_flag = 1;
    if (first_piece && tt < 2 * CPT) {
      new_row = chunk16(reinterpret_cast<const uint8_t *>(tt < CPT ? kn : vn) + 16 * (tt % CPT), a.loose);
      if (a.new_flags) new_flag = a.new_flags[u];
    }
    uint64_t ring_vis = 0;
    if (has_ring && t0 < extra && mine) {  // evicted tokens of the window: the kept ones are cache rows already
      bool see = false;
      if (lane < a.ring.n) {
        const int p = a.ring.pos[(size_t)u * a.ring.n + lane];
        const uint8_t f = a.ring.flags[(size_t)u * a.ring.n + lane];
        see = p < a.pos && p > a.pos - a.ring.n && f == 0;
      }
      ring_vis = __ballot(see);
    }
    const T *K = static_cast<const T *>(a.kc) + (size_t)ro * D, *V = static_cast<const T *>(a.vc) + (size_t)ro * D;
    wave_t wv;
    wv.init(my_lds, lane);
    // the wave that never has more tiles than another one takes the new token
    const bool own = first_piece && wt == team - 1;
    if (t0 + wt < t1 || own)
      wv.run(static_cast<const T *>(a.q) + (size_t)u * G * D, t0 + wt, t1, team, a.qscale, own, n == 0 && ring_vis == 0, kn, vn, a.loose, [&](int i) {
        if (i >= extra) {
          const int64_t r = (int64_t)(i - extra) * kTileRows;
          const int have = max(0, min(kTileRows, (int)(n - r)));
          return dec_tile{K + r * D, V + r * D, (uint32_t)have * (uint32_t)(D * sizeof(T)),
                          have == kTileRows ? 0xffffffffu : (1u << have) - 1u, false};
        }
        const size_t ring0 = ((size_t)u * a.ring.n + (size_t)i * kTileRows) * D;
        return dec_tile{static_cast<const T *>(a.ring.k) + ring0, static_cast<const T *>(a.ring.v) + ring0, 0u,
                        (uint32_t)(ring_vis >> (kTileRows * i)), true};
      });
    wv.leave((AG_LDS float *)my_lds);
    __syncthreads();
    if (kRegs && tid == 0 && (PIECE || order < 0)) arrive();

    // ---- merge the waves' states (every wave of the team left one); thread -> (head, two neighbouring columns) ----
    auto store_out = [&](int gg, int d, float A0, float A1, float L) {
      T *dst = static_cast<T *>(a.out) + ((size_t)u * G + gg) * D + d;
      if constexpr (sizeof(T) == 2) {
        const float inv = 1.f / L;
        const uint32_t two = pack2(A0 * inv, A1 * inv);
        if (a.loose) {
          dst[0] = (uint16_t)two;
          dst[1] = (uint16_t)(two >> 16);
        } else {
          *reinterpret_cast<uint32_t *>(dst) = two;
        }
      } else {
        *reinterpret_cast<float2 *>(dst) = make_float2(A0 / L, A1 / L);
      }
    };
    auto rec_at = [&](int k) {  // record of piece k of this unit
      const int id = PIECE ? rec0 + k : 2 * (rec0 + k) + (k == 0 ? 1 : 0);
      return a.rec + (size_t)id * G * (D + 2);
    };
    auto merge = [&](int e, auto waves) {
      constexpr int NS = decltype(waves)::value;
      const int gg = e / (D / 2), d = 2 * (e - gg * (D / 2));
      const AG_LDS float *h = (const AG_LDS float *)team_lds + gg * SF;
      constexpr int WF = wave_t::kWaveB / 4;
      float M = kEmptyMax, L = 0.f, A0 = 0.f, A1 = 0.f, ms[NS], ls[NS], o0[NS], o1[NS];
#pragma unroll
      for (int w = 0; w < NS; ++w) {
        ms[w] = h[w * WF];
        ls[w] = h[w * WF + 1];
        o0[w] = h[w * WF + 4 + d];
        o1[w] = h[w * WF + 5 + d];
      }
#pragma unroll
      for (int w = 0; w < NS; ++w) M = fmaxf(M, ms[w]);
#pragma unroll
      for (int w = 0; w < NS; ++w) {
        const float f = __builtin_amdgcn_exp2f(ms[w] - M);
        L = fmaf(f, ls[w], L);
        A0 = fmaf(f, o0[w], A0);
        A1 = fmaf(f, o1[w], A1);
      }
      if (n_rec == 1) {
        store_out(gg, d, A0, A1, L);
      } else {
        float *r = rec_at(my_rec) + gg * (D + 2);
        put_pair(r + d, A0, A1);
        if (d == 0) put_pair(r + D, M, L);
      }
    };
    if constexpr (kRegs || !PIECE) {
      for (int e = tid; e < G * D / 2; e += NT) merge(e, std::integral_constant<int, NW>{});
    } else if (mine) {
      if (team == 4)
        for (int e = tt; e < G * D / 2; e += 256) merge(e, std::integral_constant<int, 4>{});
      else if (team == 2)
        for (int e = tt; e < G * D / 2; e += 128) merge(e, std::integral_constant<int, 2>{});
      else
        for (int e = tt; e < G * D / 2; e += 64) merge(e, std::integral_constant<int, 1>{});
    }
    if ((kRegs || !PIECE) && n_rec > 1) {
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
            const float keep = __builtin_amdgcn_exp2f(M - M_new);
            M = M_new;
            L *= keep; A0 *= keep; A1 *= keep;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              if (k0 + j >= n_rec) break;  // (not weight 0: a record may hold infinities)
              const float w = __builtin_amdgcn_exp2f(ml[j].x - M);
              L = fmaf(w, ml[j].y, L);
              A0 = fmaf(w, o[j].x, A0);
              A1 = fmaf(w, o[j].y, A1);
            }
          }
          store_out(gg, d, A0, A1, L);
        }
      }
    }
    if (first_piece && tt < 2 * CPT) {  // the new token: its cache row (nobody reads past len in this launch) and its ring slot
      if (new_flag != 0 && sl < 0) {
        put16(reinterpret_cast<uint8_t *>(static_cast<T *>(tt < CPT ? a.kc : a.vc) + (size_t)(ro + n) * D) + 16 * (tt % CPT), new_row, EVEN);
        if (tt == 0) a.idx[ro + n] = a.pos;
      } else if (new_flag != 0 && tt == 0) {
        atomicOr(a.d_err, 1);
      }
      if (has_ring) {  // slot pos % n_recent held position pos - n_recent, which no query sees any more
        const size_t slot = (size_t)u * a.ring.n + (size_t)(a.pos % a.ring.n);
        put16(reinterpret_cast<uint8_t *>(static_cast<T *>(tt < CPT ? a.ring.k : a.ring.v) + slot * D) + 16 * (tt % CPT), new_row, a.loose);
        if (tt == 0) {
          a.ring.flags[slot] = new_flag != 0 ? 1 : 0;
          a.ring.pos[slot] = a.pos;
        }
      }
    }
    ++u;
    sub = 0;
  };
  if (by_piece) {
    if (!idle) segment(std::true_type{});
  } else {
    while (left > 0) {
      segment(std::false_type{});
      if (left > 0) __syncthreads();  // the states have been read: the next segment may load over them
    }
  }
  // ---- the last workgroup to arrive counts the appended rows ----
  __syncthreads();
  if (tid == 0) {
    if (kRegs && order < 0) arrive();
    int last = (int)gridDim.x - 1;
    if (groups > 1) {
      const int mine = ((int)gridDim.x - wg % kDecodeArriveGroups + kDecodeArriveGroups - 1) / kDecodeArriveGroups;  // that count with this one
      order = order == mine - 1 ? __hip_atomic_fetch_add(a.arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : -1;
      last = kDecodeArriveGroups - 1;
    }
    s_last = order == last;
  }
  __syncthreads();
  if (!s_last) return;
  if constexpr (kRegs) {
    if (wave == 0)
#pragma unroll
      for (int j = 0; j < UPL; ++j)
        if (64 * j + lane < U && sl_r[j] < 0 && (a.new_flags == nullptr || a.new_flags[64 * j + lane] != 0))
          a.len[64 * j + lane] = (sl_r[j] & 0x7fffffff) + 1;
  } else {
    for (int v0 = tid; v0 < U; v0 += 4 * NT) {  // (four flags requested together: this is the tail of the step)
      uint8_t f[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) f[j] = a.new_flags ? a.new_flags[min(v0 + j * NT, U - 1)] : (uint8_t)1;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (v0 + j * NT < U && f[j] != 0 && s_len[v0 + j * NT] < 0) a.len[v0 + j * NT] = (s_len[v0 + j * NT] & 0x7fffffff) + 1;
    }
  }
  if (tid <= kDecodeArriveGroups) a.arrived[kDecodeArriveStride * tid] = 0;
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

template <typename T, int D, int G, int NW, bool EVEN>
hipError_t launch_nw(ag_ctx *ctx, hipStream_t s, dec_args a, int64_t total_rows, int64_t records) {
  typedef typename wave_of<T, D, G, EVEN>::type wave_t;
  const size_t shmem = (size_t)NW * wave_t::kWaveB + (NW == 8 ? 0 : (size_t)a.U * 4);
  // one workgroup per CU (8 waves) or two (4 waves); no more than the step can have pieces, nor than there are records (a piece's
  // record has the number of its workgroup)
  const int64_t pieces = std::min<int64_t>(a.U + total_rows / (NW * wave_t::kTileRows) + 1, records);
  const int blocks = (int)std::min<int64_t>(NW == 8 ? ctx->num_cu : 2 * ctx->num_cu, pieces);
  a.max_wgs = (int)std::max<int64_t>(1, std::min<int64_t>(records / 2, blocks));
  for (a.team = NW; a.team > 1 && (int64_t)a.U * a.team > (int64_t)blocks * NW;) a.team /= 2;
  // The limit is raised once per device, to what the largest step needs: a limit that followed the size of each call could be
  // lowered by one thread under another one's launch.
  constexpr size_t kMost = (size_t)NW * wave_t::kWaveB + (NW == 8 ? 0 : (size_t)kDecodeMaxUnits * 4);
  if (kMost > 48 * 1024) {
    static std::atomic<bool> allowed[64];
    if (!allowed[ctx->device & 63].load(std::memory_order_relaxed)) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&ag_decode_kernel<T, D, G, NW, EVEN>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMost);
      if (e != hipSuccess) return e;
      allowed[ctx->device & 63].store(true, std::memory_order_relaxed);
    }
  }
  // (both timing ids report this launch: the merge is part of it)
  ag_tick(ctx, AG_K_DECODE_MERGE, s);
  AG_LAUNCH(ag_time_kernel(ctx, AG_K_DECODE_PARTIAL), (ag_decode_kernel<T, D, G, NW, EVEN>), dim3(blocks), dim3(64 * NW), shmem, s, a);
  ag_tock(ctx, AG_K_DECODE_MERGE, s);
  return hipGetLastError();
}

template <typename T, int D, int G>
hipError_t launch_t(ag_ctx *ctx, hipStream_t s, dec_args a, int64_t total_rows, ws_cursor &ws) {
  const int64_t records = max_records(a.U, total_rows);
  a.rec = ws.take<float>((size_t)records * G * (D + 2));
  if (!ws.ok) return hipSuccess;
  if constexpr (sizeof(T) == 2)
    if ((((uintptr_t)a.kc | (uintptr_t)a.vc) & 15) != 0)
      return a.U <= kFewUnits<T> ? launch_nw<T, D, G, 8, true>(ctx, s, a, total_rows, records) : launch_nw<T, D, G, 4, true>(ctx, s, a, total_rows, records);
  return a.U <= kFewUnits<T> ? launch_nw<T, D, G, 8, false>(ctx, s, a, total_rows, records) : launch_nw<T, D, G, 4, false>(ctx, s, a, total_rows, records);
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
