// The paper's main Attention-Gate module (Sec. 3.3, Eq. 3): a small multi-head attention MHA' in front of the
// gate's output projection,
//     Q', K', V' = X W'        (d -> h' heads of d'_k each)
//     A          = causal softmax attention per head over the whole prompt (no eviction inside the gate)
//     logits     = concat_heads(A) W^{O'} + bias     -> flags as in ag_gate (Eq. 4)
// Three stages, all bf16 with fp32 accumulation, d'_k = 128:
//   1. ag_proj_gemm_kernel: X [tokens, d] . W_qkv [d, 3 h' 128] on v_mfma_f32_32x32x16_bf16, written head-major
//      ([3][B, h', L, 128]) so that stage 2 reads it like any Q/K/V.
//   2. the tuned D = 128 prefill kernel with every token kept: the "compacted" rows of a head are then its K'/V'
//      themselves, so no copy is made; the output is written token-major [B, L, h' 128], the feature layout of
//   3. the gate kernels of ag_gate.hip with d_in = h' 128 and W_g = W^{O'}.
#include <string.h>

#include <algorithm>
#include <atomic>

#include "ag_internal.h"

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2;
#define AG_LDS __attribute__((address_space(3)))

constexpr int kDh = 128;  // head size

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  const f32x2 x = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
}

// COMPACT (the layer's own K/V projection, N = 2 * hp * 128: K columns, then V columns): besides the two full tensors
// -- every token needs its own k, v for the diagonal of Eq. 5 -- a tile also writes the rows of its kept tokens straight
// into the ragged cache, at the position the flag scan gives them (words / blk_off: 64-bit keep masks and their exclusive
// prefix counts), so the compaction pass and its re-read of K and V disappear.  The K tiles also write idx, the tile with
// a sequence's first token and a K head's first column writes len.
struct ag_proj_compact {
  const uint64_t *words;    // [units, nw]
  const int32_t *blk_off;   // [units, nw + 1]
  const int64_t *row_off;   // [units + 1]
  uint16_t *kc, *vc;        // cache rows
  int32_t *idx, *len, *d_err;
  int nw, pos0;
};

// C^T[n, m] = sum_k W[k, n] X[m, k]: the A operand is W^T (transposing LDS reads of the row-major W tile), the B
// operand is X^T (16-byte LDS reads of the row-major X tile), so a lane ends up with 4 consecutive output columns
// of one token.
//   x [M, K] bf16 row-major, w [K, N] bf16 row-major, K % 64 == 0, N % 128 == 0, N = (3 or 2) * hp * 128.
//   out: tensors [B, hp, L, 128] back to back; token m = b * L + t.
// A workgroup computes BM tokens x BN columns with WM x WN waves, each a block of 32-row MFMA tiles.  The operands stream
// through a ring of ST stages of BK k-steps, loaded straight into LDS ST - 1 stages ahead; one barrier per stage.
// What bounds it is LDS first: per 16 k-steps a wave reads (TM + TN) KiB for TM TN MFMAs of 32 cycles, so with 64 x 64 per
// wave (TM = TN = 2) the reads alone fill all of LDS's 128 bytes a cycle at the full MFMA rate; 64 x 128 per wave needs 96
// and the loads' own writes 31.  And under that load the chip's power: the vendor library's 8192^3 product reaches
// 1.24 PFLOP/s here.
// KS = 2: two waves share each block of MFMA tiles, each taking half of the 16-k slabs of a stage; their sums meet at the end.  A
// workgroup that has its CU to itself then has two waves per SIMD (one with 128 x 64 tiles, which would leave half of the SIMDs empty),
// and one issues while the other waits for LDS or the barrier, with no more LDS reads than one wave would make (K = 4096, 1536
// columns: 2000 tokens 39.8 -> 32.3 us, 4096 tokens 55.2 -> 51.2).  A sum over k is two fp32 sums added at the end instead of one, so last
// bits of the bf16 results differ from the other tiles'; against 64 bits neither is better: the gate module's logits, 22 inputs of 100 to
// 6000 tokens, K = 2048 and 4096, are off by 3.3956e-3 (2-norm) in the mean without pairs and by 3.3954e-3 with.
template <int BM_, int BN_, int WM_, int WN_, int BK_, int ST_, int KS_ = 1> struct proj_cfg {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, BK = BK_, ST = ST_, KS = KS_;
  static constexpr int NT = 64 * WM * WN * KS, TM = BM / WM / 32, TN = BN / WN / 32;
  static constexpr int XRow = BK * 2, WRow = BN * 2;             // bytes per LDS row of the X and W tiles
  static constexpr int XTile = BM * XRow, WTile = BK * WRow, Stage = XTile + WTile;
  static constexpr int XL = XTile / 1024 / (NT / 64), WL = WTile / 1024 / (NT / 64);  // load instructions per wave and stage
  static constexpr int Lds = ST * Stage > BM * WRow ? ST * Stage : BM * WRow;
  static_assert(KS == 1 || (KS == 2 && TM == 2 && ST > 2 && BK / 16 % 4 == 0 && Lds >= NT * TN * 64), "the waves of a pair exchange half of their sums");
  static_assert(XTile % (1024 * (NT / 64)) == 0 && WTile % (1024 * (NT / 64)) == 0, "whole load instructions per wave");
  // swizzle keys (chunks of 16 bytes): X rows of 64, 128 or 256 bytes, W rows of 128 bytes or more
  static __device__ __forceinline__ int xkey(int r) { return BK == 32 ? (r >> 2) & 3 : BK == 64 ? (r >> 1) & 7 : r & 15; }
  static __device__ __forceinline__ int wkey(int r) {
    // rows of a multiple of 256 bytes start at the same bank; others alternate between the two halves of the banks
    return WRow % 256 == 0 ? ((r & 3) << 2) | ((r >> 2) & 3) : ((r >> 1) & 1) << 2;
  }
};

template <typename CFG, bool COMPACT>
__global__ __launch_bounds__(CFG::NT, 2) void ag_proj_gemm_kernel(const uint16_t *__restrict__ x, const uint16_t *__restrict__ w,
                                                               int64_t M, int K, int N, int L, int hp,
                                                               uint16_t *__restrict__ out, ag_proj_compact cp, int m_tiles,
                                                               int n_tiles) {
  constexpr int BM = CFG::BM, BN = CFG::BN, BK = CFG::BK, ST = CFG::ST, TM = CFG::TM, TN = CFG::TN, NT = CFG::NT;
  constexpr int XRow = CFG::XRow, WRow = CFG::WRow, XL = CFG::XL, WL = CFG::WL;
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wave % CFG::WN, wm = wave / CFG::WN % CFG::WM;
  // (the compiler does not know the number of waves: said as a constant where a wave has its tiles to itself, or the slabs' LDS offsets
  // are computed in the loop -- 64 x 64 tiles, K = 4096, 64 tokens: 16.1 us instead of 15.3)
  const int kq = CFG::KS == 1 ? 0 : wave / (CFG::WN * CFG::WM);
  const int col = lane & 31, kb = lane >> 5;
  // Workgroup -> tile: workgroup i runs on XCD i % 8.  An XCD takes a contiguous part of the tile list, which walks groups
  // of 8 token tiles column by column, so that the tiles in flight on it share W and X panels in its L2.
  const int tiles = m_tiles * n_tiles, per_xcd = (tiles + 7) >> 3;
  const int t_id = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per_xcd || t_id >= tiles) return;
  const int grp = t_id / (8 * n_tiles), in_g = t_id - grp * 8 * n_tiles, gm = min(8, m_tiles - 8 * grp);
  const int n0 = (in_g / gm) * BN;
  const int64_t m0 = (int64_t)(8 * grp + in_g % gm) * BM;

  // ---- tile loaders (global -> LDS without registers); the swizzle is applied on the global side ----
  const int64_t rows_left = M - m0;  // rows of x that exist from m0 on (>= 1); rows past the end arrive as zeros
  const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void *)(x + (size_t)m0 * K), 0, (int)min((int64_t)BM, rows_left) * K * 2, 0x00020000);
  const __amdgpu_buffer_rsrc_t w_rsrc =
      __builtin_amdgcn_make_buffer_rsrc((void *)(w + n0), 0, (int)(((size_t)K * N - n0) * 2), 0x00020000);
  constexpr int XC = XRow / 16, WC = WRow / 16;  // chunks per row
  int xoff[XL], woff[WL];
#pragma unroll
  for (int i = 0; i < XL; ++i) {
    const int r = (wave * XL + i) * (64 / XC) + lane / XC;
    xoff[i] = r * K * 2 + (((lane % XC) ^ CFG::xkey(r)) << 4);
  }
#pragma unroll
  for (int i = 0; i < WL; ++i) {  // piece p of the tile, 64 pieces per instruction: row p / WC, position p % WC
    const int p = (wave * WL + i) * 64 + lane, r = p / WC, c = p % WC;
    woff[i] = r * N * 2 + ((c ^ CFG::wkey(r)) << 4);
  }
  const uint32_t lds0 = (uint32_t)(size_t)((AG_LDS uint8_t *)smem);
  auto issue = [&](int t, int buf) {  // stage t -> ring position buf
    const int xs = t * BK * 2, ws = t * BK * N * 2;
    const uint32_t base = lds0 + buf * CFG::Stage;
#pragma unroll
    for (int i = 0; i < XL; ++i)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                   :: "s"(base + (wave * XL + i) * 1024), "v"(xoff[i]), "s"(x_rsrc), "s"(xs) : "m0", "memory");
#pragma unroll
    for (int i = 0; i < WL; ++i)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                   :: "s"(base + CFG::XTile + (wave * WL + i) * 1024), "v"(woff[i]), "s"(w_rsrc), "s"(ws) : "m0", "memory");
  };

  // ---- loop-invariant LDS offsets of this lane's fragments ----
  // B operand (X^T): lane (token col, k half kb), slab sl: 16 bytes at row (wm TM + mt) 32 + col, chunk 2 sl + kb
  // (the key only depends on the row mod 32, so the slab and the row tile are an XOR and an addition)
  const int x_row = wm * TM * 32 + col;
  const int x_base = x_row * XRow + ((kb ^ CFG::xkey(x_row)) << 4);
  // A operand (W^T) by transposing reads: 16-lane group gl covers columns 16 (gl % 2) + 0..15 of a 32-column
  // sub-tile and k half gl / 2; lane i supplies the address of row 8 (gl / 2) + i / 4 (+ 4), columns 4 (i % 4) .. +3
  const int gl = lane >> 4, li = lane & 15;
  int w_off[TN][2];
#pragma unroll
  for (int nt = 0; nt < TN; ++nt)
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) {
      const int r = 8 * (gl >> 1) + (li >> 2) + 4 * h2;                        // row inside a 16-k slab
      const int c = 4 * (wn * TN + nt) + 2 * (gl & 1) + ((li & 3) >> 1);        // 16-byte chunk of the row
      w_off[nt][h2] = CFG::XTile + r * WRow + ((c ^ CFG::wkey(r)) << 4) + (li & 1) * 8;
    }

  f32x16 acc[TN][TM];
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;

  // ST > 2: the fragments of one 16-k slab are read from LDS while the MFMAs of the slab before it run, also across a stage's end:
  // after a barrier the first MFMAs find their operands in registers.  For that the NEXT stage must have landed at every
  // barrier, and a stage's place in the ring is free after the barrier that follows its last slab.
  constexpr int NS = BK / 16 / CFG::KS, NM = TN * TM, RPM = (2 * TN + TM + NM - 1) / NM;  // slabs per stage, MFMAs per slab, reads per MFMA
  const int T = K / BK;
  bf16x8 fa[2][TN], fb[2][TM];
  auto read = [&](const AG_LDS uint8_t *S, int sl, bf16x8 (&a)[TN], bf16x8 (&b)[TM]) {
#pragma unroll
    for (int nt = 0; nt < TN; ++nt) {
      // wkey only depends on the row inside the slab (r & 15), so the slab base can be added afterwards
      const AG_LDS uint8_t *base = S + 16 * sl * WRow;
      const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((AG_LDS bf16x4 *)(base + w_off[nt][0]));
      const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((AG_LDS bf16x4 *)(base + w_off[nt][1]));
      a[nt] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
#pragma unroll
    for (int mt = 0; mt < TM; ++mt) b[mt] = *reinterpret_cast<const AG_LDS bf16x8 *>(S + (x_base ^ (sl << 5)) + mt * 32 * XRow);
  };
  if constexpr (ST == 2) {
    // Two stages: what one workgroup waits for, the other one of its CU covers, and with half the barriers and no fragments
    // held ahead the two together are faster than two of the pipelined loop below.
    issue(0, 0);
    for (int t = 0; t < T; ++t) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's share of stage t has landed
      __syncthreads();                                  // ... and everyone's; stage t - 1 is fully read
      if (t + 1 < T) issue(t + 1, (t + 1) & 1);
      const AG_LDS uint8_t *S = (const AG_LDS uint8_t *)smem + (t & 1) * CFG::Stage;
#pragma unroll
      for (int sl = 0; sl < NS; ++sl) {
        read(S, sl, fa[0], fb[0]);
#pragma unroll
        for (int nt = 0; nt < TN; ++nt)
#pragma unroll
          for (int mt = 0; mt < TM; ++mt)
            acc[nt][mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0][nt], fb[0][mt], acc[nt][mt], 0, 0, 0);
      }
    }
  } else {
#pragma unroll
    for (int t = 0; t < ST; ++t)
      if (t < T) issue(t, t);
    if (T > ST - 1) asm volatile("s_waitcnt vmcnt(%0)" :: "n"((ST - 2) * (XL + WL)) : "memory");  // stages 0 and 1 have landed
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const int sl0 = kq * NS;  // this wave's first slab of a stage
    read((const AG_LDS uint8_t *)smem, sl0, fa[0], fb[0]);
    int buf = 0;
    for (int t = 0; t < T; ++t) {
      const AG_LDS uint8_t *S = (const AG_LDS uint8_t *)smem + buf * CFG::Stage;
      const int nxt = buf + 1 == ST ? 0 : buf + 1;
      const AG_LDS uint8_t *Sn = (const AG_LDS uint8_t *)smem + nxt * CFG::Stage;
#pragma unroll
      for (int sl = 0; sl < NS; ++sl) {
        const int cur = sl & 1;
        if (sl + 1 < NS) read(S, sl0 + sl + 1, fa[cur ^ 1], fb[cur ^ 1]);
        else read(Sn, sl0, fa[cur ^ 1], fb[cur ^ 1]);  // (after the last stage: stale bytes that nothing uses)
#pragma unroll
        for (int nt = 0; nt < TN; ++nt)
#pragma unroll
          for (int mt = 0; mt < TM; ++mt)
            acc[nt][mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[cur][nt], fb[cur][mt], acc[nt][mt], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < NM; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x100, RPM, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
      }
      // this wave's share of stage t + 2 has landed (t + 3 .. may be on their way) ...
      if (t + ST - 1 < T) asm volatile("s_waitcnt vmcnt(%0)" :: "n"((ST - 3) * (XL + WL)) : "memory");
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();  // ... and everyone's; stage t is fully read
      if (t + ST < T) issue(t + ST, buf);
      buf = nxt;
    }
  }

  // ---- epilogue: acc[nt][mt][r] = C[token m0 + 32 (wm TM + mt) + col][n0 + 32 (wn TN + nt) + 8 (r/4) + 4 kb + r%4] ----
  // A lane owns 4-column pieces of its tokens, so it would store scattered 8-byte pieces; the tile is laid out in the (now
  // unused) ring instead, 16-byte chunks XOR-swizzled with the row, and leaves in whole rows, to the output and, for a
  // kept token, to its cache row.
  __syncthreads();  // every wave is done with the last stage
  AG_LDS uint8_t *ost = (AG_LDS uint8_t *)smem;
  if constexpr (CFG::KS == 2) {  // a pair of waves: each hands the other half of its sums over and finishes token tile kq
    AG_LDS f32x4 *give = (AG_LDS f32x4 *)smem + (size_t)wave * TN * 256 + lane;
    AG_LDS f32x4 *take = (AG_LDS f32x4 *)smem + (size_t)(wave ^ (CFG::WM * CFG::WN)) * TN * 256 + lane;
#pragma unroll
    for (int nt = 0; nt < TN; ++nt)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        f32x4 g;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float a = acc[nt][0][4 * r4 + e], b = acc[nt][1][4 * r4 + e];
          g[e] = kq ? a : b;
          acc[nt][0][4 * r4 + e] = kq ? b : a;
        }
        give[(nt * 4 + r4) * 64] = g;
      }
    __syncthreads();
#pragma unroll
    for (int nt = 0; nt < TN; ++nt)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const f32x4 g = take[(nt * 4 + r4) * 64];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[nt][0][4 * r4 + e] += g[e];
      }
    __syncthreads();
  }
  constexpr int KM = WC % 16 == 0 ? 15 : 7;  // chunk bits that the row is mixed into
#pragma unroll
  for (int mt = 0; mt < TM / CFG::KS; ++mt) {
    const int row = 32 * (wm * TM + mt + kq) + col;  // (kq = 0 where a wave has its tiles to itself)
#pragma unroll
    for (int nt = 0; nt < TN; ++nt)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const f32x16 &c = acc[nt][mt];
        const u32x2 val = {pack2(c[4 * r4 + 0], c[4 * r4 + 1]), pack2(c[4 * r4 + 2], c[4 * r4 + 3])};
        *reinterpret_cast<AG_LDS u32x2 *>(ost + row * WRow + (((4 * (wn * TN + nt) + r4) ^ (row & KM)) << 4) + 8 * kb) = val;
      }
  }
  const int hd = hp * kDh;
  // COMPACT: the cache row of every (token, head) of the tile, -1 for none; looked up by all threads at once
  constexpr int NH = (BN + kDh - 1) / kDh;  // heads of a tile, which starts at one or lies inside one
  __shared__ int32_t dest[COMPACT ? BM * NH : 1];
  if (COMPACT) {
    for (int i = tid; i < BM * NH; i += NT) {
      const int row = i / NH, nh = n0 + (i % NH) * kDh, which = nh / hd, head = (nh - which * hd) / kDh;
      const int64_t m = m0 + row;
      int32_t to = -1;
      if (m < M) {
        const int64_t b = m / L;
        const int tt = (int)(m - b * L), u = (int)b * hp + head;
        const uint64_t word = cp.words[(size_t)u * cp.nw + (tt >> 6)];
        const int pre = cp.blk_off[(size_t)u * (cp.nw + 1) + (tt >> 6)];
        const int64_t r0 = cp.row_off[u], cap = cp.row_off[u + 1] - r0;
        const bool writes = which == 0 && nh % kDh == 0;  // K tile with the head's first column: idx, len and the error word
        if ((word >> (tt & 63)) & 1ull) {
          const int c = pre + __popcll(word & ((1ull << (tt & 63)) - 1ull));
          if (c < cap) {
            to = (int32_t)(r0 + c);
            if (writes) cp.idx[to] = cp.pos0 + tt;
          } else if (writes) {
            atomicOr(cp.d_err, 1);  // the row is dropped, nothing is written out of bounds
          }
        }
        if (writes && tt == 0) {  // the sequence's first token: the unit's length
          const int kept = cp.blk_off[(size_t)u * (cp.nw + 1) + cp.nw];
          cp.len[u] = (int)(kept < cap ? kept : cap);
        }
      }
      dest[i] = to;
    }
  }
  __syncthreads();  // a row's pieces come from several waves
  constexpr int RPI = NT / WC;  // rows per pass of the workgroup
  const int chunk = tid % WC, n = n0 + 8 * chunk;                       // this thread's 8 columns, the same in every pass
  const int which = n / hd, head = (n - which * hd) / kDh, d = n % kDh;  // which tensor, which head, which feature
  uint16_t *const out_h = out + (size_t)which * M * hd + (size_t)head * L * kDh + d;
  int64_t b = m0 / L;
  int tt = (int)(m0 - b * L) + tid / WC;  // sequence and position of this thread's row
  for (int row = tid / WC; row < BM; row += RPI, tt += RPI) {
    if (m0 + row >= M) break;
    while (tt >= L) { tt -= L; ++b; }
    const u32x4 val = *reinterpret_cast<const AG_LDS u32x4 *>(ost + row * WRow + ((chunk ^ (row & KM)) << 4));
    *reinterpret_cast<u32x4 *>(out_h + ((size_t)b * hp * L + tt) * kDh) = val;
    if (COMPACT) {
      const int32_t to = dest[row * NH + (n - n0) / kDh];
      if (to >= 0) *reinterpret_cast<u32x4 *>((which == 0 ? cp.kc : cp.vc) + (size_t)to * kDh + d) = val;
    }
  }
}

template <typename CFG, bool COMPACT>
hipError_t launch_proj(ag_ctx *ctx, hipStream_t s, const void *x, const void *w, int64_t M, int K, int N, int L, int hp, void *out,
                       const ag_proj_compact &cp) {
  if (CFG::Lds > 48 * 1024) {
    static std::atomic<bool> allowed[64];  // said once per device
    if (!allowed[ctx->device & 63].load(std::memory_order_relaxed)) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&ag_proj_gemm_kernel<CFG, COMPACT>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, CFG::Lds);
      if (e != hipSuccess) return e;
      allowed[ctx->device & 63].store(true, std::memory_order_relaxed);
    }
  }
  const int m_tiles = (int)((M + CFG::BM - 1) / CFG::BM), n_tiles = N / CFG::BN;
  const unsigned blocks = (unsigned)(((int64_t)m_tiles * n_tiles + 7) / 8 * 8);
  AG_LAUNCH(ag_time_kernel(ctx, AG_K_MHA_PROJ), (ag_proj_gemm_kernel<CFG, COMPACT>), dim3(blocks), dim3(CFG::NT), CFG::Lds, s,
            (const uint16_t *)x, (const uint16_t *)w, M, K, N, L, hp, (uint16_t *)out, cp, m_tiles, n_tiles);
  return hipGetLastError();
}

// The tile for a product: the one whose rounds of workgroups take the least time, from what a round of each takes on this chip.
// (All seven tiles timed at 354 products -- 64 to 8200 tokens, 384 to 8192 columns, K = 1024, 2048 and 4096 -- the choice is within
// 2 %, 0.3 us, of the fastest at each, 0.02 % in the mean; at 117 others, drawn at random after the costs were set, within 3.4 %, 0.45 us,
// and 0.08 %.)
//   256 x 256: 1.13 PFLOP/s where there are tiles for whole rounds (8192 tokens x 8192 columns: 446 us; with 128 x 128
//              tiles, which LDS bounds, 526); one tile takes 80 us.
//   128 x 128: 1.0 PFLOP/s with two workgroups on every CU, and fills the chip from a quarter of the columns x tokens on.  In
//              two stages of 64 k-steps; in four of 32, with the fragments read ahead, it is slower as soon as CUs hold two of
//              them (1536 columns: 2900 tokens 67 us against 49, 8192 tokens 114 against 102).
//   128 x 192: 1536 columns (three tensors of four heads) in whole rounds where 128 x 128 leaves a rest.
//   128 x 192, 128 x 128, 128 x 64 with KS = 2 and 160, 128 or 96 KB of stages, one workgroup on a CU: where the tiles do not
//              fill the chip more than once (1536 columns: 3000 tokens 48.0 -> 42.3 us, 2000 tokens 39.8 -> 32.3, 1000 tokens
//              28.9 -> 24.3); a second round loses to two workgroups per CU (2700 tokens in 264 tiles of 128 x 128: 64.6 against
//              48.5).  With three stages instead of four a load has too little time (2000 tokens: 40.6).
//   64 x 64  : few tokens, where one tile's chain of stages is the time: 128 k-steps per barrier (64 to 300 tokens: 40 -> 16 us).
typedef proj_cfg<256, 256, 2, 4, 32, 4> cfg_256x256;
typedef proj_cfg<128, 128, 2, 2, 64, 2> cfg_128x128;
typedef proj_cfg<128, 192, 2, 2, 32, 4> cfg_128x192;
typedef proj_cfg<64, 64, 2, 2, 128, 4> cfg_64x64;
typedef proj_cfg<128, 192, 2, 2, 64, 4, 2> cfg_128x192_k2;
typedef proj_cfg<128, 128, 2, 2, 64, 4, 2> cfg_128x128_k2;
typedef proj_cfg<128, 64, 2, 1, 64, 4, 2> cfg_128x64_k2;

// A round's time ends with its slowest CU: `few` tiles take as long as one, `one` workgroup on every CU a little longer (the
// clock falls with the number of busy CUs), and as soon as some CUs hold two workgroups the round takes what those take,
// `second`, up to `full` with two on every CU (per_cu == 1: there is no second).  us at K = 4096, beside a part per round that
// does not grow with K.
struct proj_cost {
  int per_cu;
  float few, one, second, full, fixed;
};
float proj_time(int64_t M, int N, int K, int bm, int bn, int num_cu, const proj_cost &c) {
  const int64_t tiles = (M + bm - 1) / bm * (N / bn), slots = (int64_t)c.per_cu * num_cu, rounds = tiles / slots, last = tiles - rounds * slots;
  float t = (float)rounds * c.full;
  if (last > num_cu) t += c.second + (c.full - c.second) * (float)(last - num_cu) / (float)num_cu;
  else if (last > 0) {
    const float busy = (float)last / (float)num_cu;
    t += c.few + (c.one - c.few) * busy * busy * busy;
  }
  return t * (float)K / 4096.f + c.fixed * (float)(rounds + (last > 0));
}

struct proj_tile {
  int bm, bn, bk, ks;
  proj_cost cost;
};
constexpr proj_tile kProjTiles[] = {  // of two that take the same time the first
    {64, 64, 128, 1, {1, 12.f, 13.6f, 0.f, 13.f, 2.8f}},
    {256, 256, 32, 1, {1, 74.f, 106.f, 0.f, 106.f, 7.f}},
    {128, 64, 64, 2, {1, 19.f, 21.f, 0.f, 21.f, 5.f}},
    {128, 128, 64, 2, {1, 25.5f, 29.f, 0.f, 31.f, 6.f}},
    {128, 192, 32, 1, {2, 43.5f, 48.5f, 65.f, 86.f, 5.5f}},
    {128, 192, 64, 2, {1, 33.f, 42.f, 0.f, 42.f, 7.f}},
    {128, 128, 64, 1, {2, 34.f, 39.f, 43.5f, 57.f, 4.5f}},
};

const proj_tile &pick_proj_tile(int64_t M, int N, int K, bool compact, int num_cu) {
  const proj_tile *best = nullptr;
  float least = 0.f;
  for (const proj_tile &t : kProjTiles) {
    // (a tile that starts inside a head and ends in the next is not made for the compaction's look-up of cache rows)
    if (N % t.bn || K % t.bk || (compact && t.bn > kDh && t.bn % kDh)) continue;
    const float us = proj_time(M, N, K, t.bm, t.bn, num_cu, t.cost);
    if (!best || us < least) best = &t, least = us;
  }
  return *best;  // 128 x 128 always fits
}

template <bool COMPACT>
hipError_t launch_proj_any(ag_ctx *ctx, hipStream_t s, const void *x, const void *w, int64_t M, int K, int N, int L, int hp, void *out,
                           const ag_proj_compact &cp) {
  const proj_tile &t = pick_proj_tile(M, N, K, COMPACT, ctx->num_cu);
#define AG_PROJ(CFG) \
  if (t.bm == CFG::BM && t.bn == CFG::BN && t.ks == CFG::KS) return launch_proj<CFG, COMPACT>(ctx, s, x, w, M, K, N, L, hp, out, cp)
  AG_PROJ(cfg_64x64);
  AG_PROJ(cfg_256x256);
  AG_PROJ(cfg_128x64_k2);
  AG_PROJ(cfg_128x128_k2);
  if constexpr (!COMPACT) {
    AG_PROJ(cfg_128x192);
    AG_PROJ(cfg_128x192_k2);
  }
  AG_PROJ(cfg_128x128);
#undef AG_PROJ
  return hipErrorInvalidValue;
}

}  // namespace

extern "C" ag_status ag_probe_projection_tile(int64_t tokens, int K, int columns, int compaction, int num_cu, int tile[3]) {
  if (!tile || tokens < 1 || K < 64 || K % 64 || columns < kDh || columns % kDh || num_cu < 1) return AG_EINVAL;
  const proj_tile &t = pick_proj_tile(tokens, columns, K, compaction != 0, num_cu);
  tile[0] = t.bm;
  tile[1] = t.bn;
  tile[2] = t.ks;
  return AG_OK;
}

size_t ag_ws_gate_mha_bytes(int B, int L, int d_model, int hp, int H_f) {
  (void)d_model;
  const size_t tokens = (size_t)B * L;
  const int units = B * hp;
  ws_cursor count{nullptr, ~size_t(0) >> 1, 0, true};
  ag_pf_plan plan;
  float *part;
  ag_prefill_bf16_plan(1024, B, L, hp, hp, 128, count, &plan, &part);
  return 3 * ag_align256(tokens * hp * kDh * 2)      // Q', K', V'
         + ag_align256(tokens * hp * kDh * 2)        // attention output = gate features
         + ag_ws_scan_bytes(units, L) + ag_align256((size_t)(units + 1) * 8) + count.off +
         ag_ws_gate_bytes((int64_t)tokens, hp * kDh, H_f, AG_BF16) + 4096;
}

hipError_t ag_launch_gate_mha(ag_ctx *ctx, hipStream_t s, const void *x, int B, int L, int d_model, const void *w_qkv,
                              int hp, const void *w_o, const float *bias, int H_f, float thr, int n_sink, float scale,
                              float *logits, uint8_t *flags, ws_cursor &ws) {
  const int64_t tokens = (int64_t)B * L;
  const int units = B * hp, N = 3 * hp * kDh;
  const size_t per = (size_t)tokens * hp * kDh;
  uint16_t *qkv = ws.take<uint16_t>(3 * per);
  uint16_t *feat = ws.take<uint16_t>(per);
  // (not used since the attention needs no scan; it stays in the sum, so that a workspace that was refused as too small still is)
  (void)ws.take<char>(ag_ws_scan_bytes(units, L) + ag_align256((size_t)(units + 1) * 8));
  ag_pf_plan plan;
  float *part = nullptr;
  ag_prefill_bf16_plan(ctx->num_cu, B, L, hp, hp, 128, ws, &plan, &part);
  if (!ws.ok) return hipSuccess;  // caller reports AG_EWORKSPACE

  hipError_t e = launch_proj_any<false>(ctx, s, x, w_qkv, tokens, d_model, N, L, hp, qkv, ag_proj_compact{});
  if (e != hipSuccess) return e;
  // Every token is kept: the compacted rows of a head are its K', V' rows themselves, no flag scan is needed, and the lengths
  // of the items are known here: chunks as the scan would plan them, a little above the average tiles per workgroup slot.
  // (The scan and the slab offsets were 4.7 us each in front of 42 us of attention, 4096 tokens x 4 heads.)
  plan.order = plan.chunk_tiles = nullptr;
  if (plan.n_split > 1) {
    plan.tickets = ctx->prefill_tickets;
    const int n_qt = plan.n_items / plan.n_hy;
    auto tiles_of = [&](int t) { return (std::min((t + 1) * plan.BM, L) + 63) / 64; };
    int64_t total = 0;
    for (int t = 0; t < n_qt; ++t) total += tiles_of(t);
    total *= plan.n_hy;
    plan.chunk_tiles_all = std::max({(int)((total * 23 / 20 + plan.slots - 1) / plan.slots), (plan.max_tiles + plan.n_split - 1) / plan.n_split, 8});
  }
  e = ag_launch_prefill_bf16(s, qkv, qkv + per, qkv + 2 * per, nullptr, nullptr, B, L, hp, hp, 128, scale * 1.4426950408889634f,
                             1, qkv + per, qkv + 2 * per, nullptr, feat, plan, part, /*out_token_major=*/true,
                             ag_time_kernel(ctx, AG_K_MHA_ATTN));
  if (e != hipSuccess) return e;
  return ag_launch_gate(ctx, s, feat, AG_BF16, B, L, hp * kDh, w_o, bias, H_f, thr, n_sink, logits, flags, ws);
}

// K/V projection with the compaction in its epilogue.  k_out and v_out must be one allocation of two
// [B, Hkv, L, 128] tensors back to back (k first).
size_t ag_ws_project_compact_bytes(int units, int L) {
  return ag_ws_scan_bytes(units, L) + 4096;
}

hipError_t ag_launch_project_compact(ag_ctx *ctx, hipStream_t s, const void *x, int B, int L, int d_model,
                                     const void *w_kv, int Hkv, const uint8_t *flags, int pos0, void *kv_out,
                                     void *kc, void *vc, int32_t *idx, const int64_t *row_off, int32_t *len,
                                     ws_cursor &ws) {
  const int64_t tokens = (int64_t)B * L;
  const int units = B * Hkv, nw = ag_nwords(L), N = 2 * Hkv * kDh;
  uint64_t *words = ws.take<uint64_t>((size_t)units * nw);
  int32_t *blk_off = ws.take<int32_t>((size_t)units * (nw + 1));
  if (!ws.ok) return hipSuccess;  // caller reports AG_EWORKSPACE
  hipError_t e = ag_launch_flag_scan(ctx, s, flags, units, L, words, blk_off, nullptr);
  if (e != hipSuccess) return e;
  const ag_proj_compact cp{words, blk_off, row_off, (uint16_t *)kc, (uint16_t *)vc, idx, len, ctx->d_err, nw, pos0};
  return launch_proj_any<true>(ctx, s, x, w_kv, tokens, d_model, N, L, Hkv, kv_out, cp);
}
