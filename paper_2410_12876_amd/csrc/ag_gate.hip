// Gate (Eq. 3, Eq. 4): features [tokens, d_in] x W [d_in, H_f] -> logits -> keep flags.
//
// The product is a skinny GEMM (N = H_f <= 32) whose cost is reading the features once from HBM.  One launch does
// everything: a workgroup of 8 waves owns a tile of tokens, each wave a slice of the features; the 8 partial tiles are
// added in wave order through LDS (so logits and flags are reproducible run to run), then bias, threshold, logits and the
// head-major flags.  bf16 runs on MFMA: a wave fetches its feature rows as whole 128-byte lines, handed to the MFMA layout
// through LDS, and takes the matching W fragments either from W as stored, transposed on the way through LDS, or (H_f not
// a multiple of 4, or W not 16-byte aligned) from a pre-packed copy.  ag_norm_gate_kernel fuses the normalisation of the
// input in as well.
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
#define AG_LDS __attribute__((address_space(3)))

constexpr int kNP = 32;  // padded head count (MFMA N)

// Swizzle key of row r of a wave's 32 x 128-byte hand-over buffer: the 16-byte piece p of the row is stored at
// position p ^ xkey(r).  Rows alternate between the two halves of the 64 banks, so the 16 lanes that LDS serves
// together (2 whole rows on the writing side, 16 rows at one piece index on the reading side) need 8 different
// keys among rows of equal parity: bits 1..3 of the row.
__device__ __forceinline__ int xkey(int r) { return (r >> 1) & 7; }

// W [d_in, H_f] bf16 -> the B fragments of v_mfma_f32_16x16x32_bf16: piece ((chunk * 2 + step) * 2 + column tile) * 64 + lane
// of 8 elements, lane = (col = lane % 16, kg = lane / 16), element j = W[chunk * 64 + step * 32 + kg * 8 + j][16 tile + col]
// (0 for columns >= H_f).
__global__ void ag_gate_pack_w(const uint16_t *__restrict__ w, int d_in, int H_f, uint16_t *__restrict__ wp) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;  // one packed element
  if (i >= d_in * kNP) return;
  const int j = i & 7, lane = (i >> 3) & 63, nt = (i >> 9) & 1, step = (i >> 10) & 1, chunk = i >> 11;
  const int n = 16 * nt + (lane & 15);
  const int kk = chunk * 64 + step * 32 + (lane >> 4) * 8 + j;
  wp[i] = n < H_f ? w[(size_t)kk * H_f + n] : (uint16_t)0;
}

// ---- One 64-feature chunk of W, from the 4 x 16 bytes per lane it is loaded as to MFMA fragments ---------------------
// RAW: W as the caller stores it ([d_in, H_f] row-major, H_f a multiple of 4, 16-byte aligned): lane l loads pieces l,
// l + 64, ... of the chunk's 8 H_f; they go to the wave's 4 KiB of LDS and come back through the transposing read, which
// hands lane (col, kg) the rows 32 step + 8 kg + 0..7 of column 16 tile + col.  (Columns >= H_f read whatever lies there;
// they only reach output columns that are never stored.)  Otherwise the pieces are ag_gate_pack_w's fragments already.
template <bool RAW> struct w_chunk {
  int H_f, n_u4, tr_off[2];
  AG_LDS uint8_t *st;
  __device__ __forceinline__ void init(int H_f_, int lane, AG_LDS uint8_t *stage) {
    H_f = H_f_; n_u4 = 8 * H_f; st = stage;
    const int col = lane & 15, row = 8 * (lane >> 4) + (col >> 2);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) tr_off[nt] = row * (H_f * 2) + min(16 * nt + 4 * (col & 3), H_f - 4) * 2;
  }
  __device__ __forceinline__ void load(uint4 (&b)[4], const uint4 *__restrict__ wp, int chunk, int lane) const {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if (RAW) {
        if (s == 0 || s * 64 < n_u4) b[s] = wp[(size_t)chunk * n_u4 + min(s * 64 + lane, n_u4 - 1)];
      } else {
        b[s] = wp[((size_t)chunk * 4 + s) * 64 + lane];
      }
    }
  }
  // the chunk's pieces -> LDS (RAW; between two wave_syncs)
  __device__ __forceinline__ void stage(const uint4 (&b)[4], int lane) const {
    if (RAW) {
#pragma unroll
      for (int s = 0; s < 4; ++s)
        if (s * 64 < n_u4 && s * 64 + lane < n_u4)
          *reinterpret_cast<AG_LDS u32x4 *>(st + (s * 64 + lane) * 16) = u32x4{b[s].x, b[s].y, b[s].z, b[s].w};
    }
  }
  __device__ __forceinline__ bf16x8 frag(const uint4 (&b)[4], int step, int nt) const {
    if (!RAW) return __builtin_bit_cast(bf16x8, b[2 * step + nt]);
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((AG_LDS bf16x4 *)(st + tr_off[nt] + (32 * step) * (H_f * 2)));
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((AG_LDS bf16x4 *)(st + tr_off[nt] + (32 * step + 4) * (H_f * 2)));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  }
};
// lanes of one wave exchange data through LDS
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Bias, threshold, logits [tokens, H_f] and head-major flags of a tile of 16 tokens from the 8 waves' partial tiles
// red(w, row, head), by 512 threads; bias_h: the bias of head threadIdx.x % 32 (see gate_bias).  Token and sequence of a row follow from the tile's first token by counting, not by a division each.
template <typename RED>
__device__ __forceinline__ void gate_epilogue(RED &&red, uint8_t (&fl)[kNP][16], uint32_t tok0, uint32_t tokens, int L, int H_f,
                                              float bias_h, float thr, int n_sink,
                                              float *__restrict__ logits, uint8_t *__restrict__ flags) {
  const uint32_t b0 = tok0 / (uint32_t)L, t0 = tok0 - b0 * (uint32_t)L;  // (uniform)
  auto place = [&](int rw, uint32_t &b, uint32_t &t) {
    b = b0; t = t0 + rw;
    while (t >= (uint32_t)L) { t -= L; ++b; }
  };
  {
    const int rw = threadIdx.x >> 5, h = threadIdx.x & 31;  // thread -> (token row, head)
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w) v += red(w, rw, h);
    const uint32_t tk = tok0 + rw;
    if (h < H_f && tk < tokens) {
      uint32_t b, t;
      place(rw, b, t);
      const float val = v + bias_h;
      if (logits) logits[(size_t)tk * H_f + h] = val;
      fl[h][rw] = (val > thr || (int)t < n_sink) ? 1 : 0;
    }
  }
  __syncthreads();
  const int h = threadIdx.x >> 4, rw = threadIdx.x & 15;
  if (h < H_f && tok0 + rw < tokens) {
    uint32_t b, t;
    place(rw, b, t);
    flags[((size_t)b * H_f + h) * L + t] = fl[h][rw];
  }
}

__device__ __forceinline__ float gate_bias(const float *__restrict__ bias, int H_f) {
  return bias[min((int)(threadIdx.x & 31), H_f - 1)];
}

constexpr int kFusedWaves = 8;

// One tile of 16 tokens per workgroup: launches of a few tiles per CU at most (and any with more than 4096 features).  A
// small launch is one round of loads, and what bounds it is the one CU's memory path (64 bytes a cycle: 16 rows of features
// and ALL of W for every workgroup, 384 KiB at 4096 x 32 features, 2.7 us) and the LDS behind it, not HBM.  Hence
// v_mfma_f32_16x16x32_bf16 (a 32-row MFMA would read every x fragment twice), chunks processed in the order they arrive
// while the later ones are on their way, no column tile beyond H_f, and W's first touch spread over the chip: the
// workgroups of an XCD each request other 8 KiB of W's first 256 (all of it at 4096 x 32 features) before anything else, so
// that they are in their L2 when 32 of them want them at once; without that its lines queue behind the features of the whole
// launch.
template <bool RAW, int PF>  // PF = chunks a wave keeps in flight
__global__ __launch_bounds__(64 * kFusedWaves, 2) void ag_gate16_kernel(
    const uint16_t *__restrict__ x, const uint4 *__restrict__ wp, uint32_t tokens, int d_in, int L, int H_f,
    const float *__restrict__ bias, float thr, int n_sink, float *__restrict__ logits, uint8_t *__restrict__ flags) {
  // [wave][6 KiB]: a chunk of W (64 rows), then a chunk of the 16 feature rows; afterwards the wave's partial tile
  __shared__ __attribute__((aligned(16))) uint8_t mem[kFusedWaves][6144];
  __shared__ uint8_t fl[kNP][16];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, kg = lane >> 4;
  const int lr = lane >> 3, lp = lane & 7;  // row within a group of 8 and 16-byte piece of the memory-side layout
  const uint32_t tok0 = blockIdx.x * 16;
  const int nchunks = d_in / 64;
  const float bias_h = gate_bias(bias, H_f);
  AG_LDS uint8_t *wst = (AG_LDS uint8_t *)mem[wave], *xst = wst + 4096;
  w_chunk<RAW> wc;
  wc.init(H_f, lane, wst);
  {
    // (into the wave's W buffer, which is first written after its own loads, which come later, have arrived; pieces past
    // the end of W are not requested)
    const __amdgpu_buffer_rsrc_t w_rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void *)wp, 0, (uint32_t)d_in * (uint32_t)(RAW ? H_f : kNP) * 2u, 0x00020000);
    const uint32_t dst = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)wst);
    const int off = (((blockIdx.x >> 3) & 31) * 512 + threadIdx.x) * 16;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(dst), "v"(off), "s"(w_rsrc) : "m0", "memory");
  }
  const int rows = (int)min(16u, tokens - tok0);
  const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void *)(x + (size_t)tok0 * d_in), 0, (uint32_t)rows * (uint32_t)d_in * 2u, 0x00020000);
  int row_off[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) row_off[i] = min(8 * i + lr, rows - 1) * d_in * 2 + lp * 16;
  const bool two = H_f > 16;
  f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
  for (int c0 = wave; c0 < nchunks; c0 += kFusedWaves * PF) {
    u32x4 a[PF][2];
    uint4 b[PF][4];
#pragma unroll
    for (int p = 0; p < PF; ++p) {
      const int c = min(c0 + kFusedWaves * p, nchunks - 1);
      wc.load(b[p], wp, c, lane);
#pragma unroll
      for (int i = 0; i < 2; ++i) a[p][i] = __builtin_amdgcn_raw_buffer_load_b128(x_rsrc, row_off[i], c * 128, 0);
    }
#pragma unroll
    for (int p = 0; p < PF; ++p)
      if (c0 + kFusedWaves * p < nchunks) {
        wave_sync();  // the previous chunk's fragments have been read
        wc.stage(b[p], lane);
#pragma unroll
        for (int i = 0; i < 2; ++i)
          *reinterpret_cast<AG_LDS u32x4 *>(xst + (8 * i + lr) * 128 + ((lp ^ xkey(8 * i + lr)) << 4)) = a[p][i];
        wave_sync();  // the chunk is there for every lane
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const bf16x8 af = *reinterpret_cast<const AG_LDS bf16x8 *>(xst + col * 128 + (((4 * s + kg) ^ xkey(col)) << 4));
#pragma unroll
          for (int nt = 0; nt < 2; ++nt)
            if (nt == 0 || two) acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, wc.frag(b[p], s, nt), acc[nt], 0, 0, 0);
        }
      }
  }
  // acc[nt][r] is (token 4 kg + r, head 16 nt + col)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (a wave without a chunk: its request for W has landed)
  wave_sync();
  float(*red)[6144 / 4] = reinterpret_cast<float(*)[6144 / 4]>(mem);
#pragma unroll
  for (int nt = 0; nt < 2; ++nt)
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave][(4 * kg + r) * 32 + 16 * nt + col] = acc[nt][r];
  __syncthreads();
  gate_epilogue([&](int w, int row, int h) { return red[w][row * 32 + h]; }, fl, tok0, tokens, L, H_f, bias_h, thr, n_sink, logits, flags);
}

// Many tokens, d_in <= 8 waves x NCH x 64 features: one persistent workgroup per CU walks the 16-token tiles.  A wave keeps the
// fragments of its NCH chunks of W in registers for the whole launch (16 each: no second read of W, no transposition per
// tile), and the features stream through a ring of kRing 2-KiB chunks per wave, loaded straight into LDS: as soon as a
// chunk's fragments are read, the chunk kRing further on -- of the same tile or of a later one -- is requested into its
// place, so the memory system always sees 8 x kRing x 2 KiB per CU, also while a tile's partial sums are added and its
// flags written.  32768 tokens x 4096 features x 32 heads: 62 us (4.3 TB/s) with tiles loaded, staged and finished one
// after the other by two workgroups per CU.
constexpr int kRing = 6;
template <bool RAW, int NCH>
__global__ __launch_bounds__(64 * kFusedWaves, 2) void ag_gate_stream_kernel(
    const uint16_t *__restrict__ x, const uint4 *__restrict__ wp, uint32_t tokens, int d_in, int L, int H_f,
    const float *__restrict__ bias, float thr, int n_sink, float *__restrict__ logits, uint8_t *__restrict__ flags) {
  // [wave][kRing x 2 KiB] ring of feature chunks, then [wave][4 KiB]: W staging before the loop, partial tiles in it
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  __shared__ uint8_t fl[kNP][16];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, kg = lane >> 4;
  const int lr = lane >> 3, lp = lane & 7;
  const int nchunks = d_in / 64, mine = (nchunks - wave + kFusedWaves - 1) / kFusedWaves;  // this wave's chunks (may be 0)
  const int tiles = (int)((tokens + 15) / 16), stride = gridDim.x;
  AG_LDS uint8_t *ring = (AG_LDS uint8_t *)smem + wave * (kRing * 2048);
  AG_LDS uint8_t *wst = (AG_LDS uint8_t *)smem + kFusedWaves * kRing * 2048 + wave * 4096;
  const uint32_t ring_addr = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)ring);
  int row_off[2];  // load instruction i, lane: row 8 i + lr, piece lp ^ key(row), to position lp
#pragma unroll
  for (int i = 0; i < 2; ++i) row_off[i] = (8 * i + lr) * d_in * 2 + ((lp ^ xkey(8 * i + lr)) << 4);
  // the wave's stream: chunk p of tile blockIdx.x + j * stride; (it, ip) is the next one to request
  uint32_t it = blockIdx.x;
  int ip = 0, slot_in = 0;
  auto request = [&]() {
    if (it < (uint32_t)tiles && mine > 0) {
      const uint32_t t0 = it * 16, rows = min(16u, tokens - t0);  // (rows past the last token arrive as zeros)
      const __amdgpu_buffer_rsrc_t rsrc =
          __builtin_amdgcn_make_buffer_rsrc((void *)(x + (size_t)t0 * d_in), 0, rows * (uint32_t)d_in * 2u, 0x00020000);
      const uint32_t dst = ring_addr + slot_in * 2048;
      const int soff = (wave + kFusedWaves * ip) * 128;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" :: "s"(dst), "v"(row_off[0]), "s"(rsrc), "s"(soff) : "m0", "memory");
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" :: "s"(dst + 1024), "v"(row_off[1]), "s"(rsrc), "s"(soff) : "m0", "memory");
      slot_in = slot_in + 1 == kRing ? 0 : slot_in + 1;
      if (++ip == mine) { ip = 0; it += stride; }
    }
  };
  // W first, as fragments in registers
  bf16x8 wf[NCH][2][2];
  {
    w_chunk<RAW> wc;
    wc.init(H_f, lane, wst);
    uint4 b[NCH][4];
#pragma unroll
    for (int p = 0; p < NCH; ++p) wc.load(b[p], wp, min(wave + kFusedWaves * p, nchunks - 1), lane);
#pragma unroll
    for (int p = 0; p < NCH; ++p) {
      wave_sync();
      wc.stage(b[p], lane);
      wave_sync();
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
          wf[p][s][nt] = wc.frag(b[p], s, nt);
          asm volatile("" : "+v"(wf[p][s][nt]));
        }
    }
  }
  float bias_h = gate_bias(bias, H_f);
  asm volatile("" : "+v"(bias_h));  // loaded here: a wait for it inside the loop would be one for the whole ring
  for (int i = 0; i < kRing; ++i) request();
  int slot = 0, done = 0;
  const int total = mine * (((int)tiles - (int)blockIdx.x + stride - 1) / stride);
  float *red = reinterpret_cast<float *>(smem + kFusedWaves * kRing * 2048);
  for (int tile = blockIdx.x; tile < tiles; tile += stride) {
    f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int p = 0; p < NCH; ++p)
      if (p < mine) {
        // two requests per chunk; the kRing - 1 later ones may still be on their way
        if (done + kRing <= total) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * (kRing - 1)) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const AG_LDS uint8_t *xst = ring + slot * 2048;
        bf16x8 af[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) af[s] = *reinterpret_cast<const AG_LDS bf16x8 *>(xst + col * 128 + (((4 * s + kg) ^ xkey(col)) << 4));
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        slot = slot + 1 == kRing ? 0 : slot + 1;
        ++done;
        request();
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int nt = 0; nt < 2; ++nt) acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[s], wf[p][s][nt], acc[nt], 0, 0, 0);
      }
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave * 1024 + (4 * kg + r) * 32 + 16 * nt + col] = acc[nt][r];
    __syncthreads();
    // (its barrier comes after the partial tiles have been read: the next tile's may be written)
    gate_epilogue([&](int w, int row, int h) { return red[w * 1024 + row * 32 + h]; }, fl, (uint32_t)tile * 16, tokens, L, H_f, bias_h, thr,
                  n_sink, logits, flags);
  }
}

// RMS normalisation fused with the gate: x = h / sqrt(mean_c h^2 + eps) * g, rounded once to bf16, written out for
// the projections that follow, and multiplied by W from the same registers, so the gate costs no second read of x.
// One workgroup of 8 waves per 32 tokens.  Wave w owns the 64-feature chunks w, w + 8, ... (at most NCH of
// them: d_in <= 4096 with 32-token tiles, <= 8192 with 16-token tiles) of all rows of the tile and keeps them in registers for the whole kernel, so all loads of the tile are
// in flight at once.  A chunk is one 128-byte line per row; a load or store instruction moves 8 whole lines (lane
// -> row 8 i + lane / 8, 16-byte piece lane % 8).  The squares are summed per lane, over the 8 lanes of a row and
// then over the waves through LDS in wave order.  After the scaling the chunk is stored from the same registers
// and handed through a 4 KiB LDS buffer of the wave (pieces XOR-swizzled with the row: no bank conflicts on either
// side) to the MFMA's A layout, lane (token col, group kg) holding features s*32 + kg*8 .. +7 for step s.  That
// layout, the W fragments and the order of the MFMAs (chunks ascending per wave, then the waves in order) are
// those of ag_gate, so the logits are those ag_gate gives on the stored x bit for bit.
template <bool RAW, int TOK, int NCH>  // NCH = chunks a wave holds: d_in <= 8 waves x NCH x 64 features
__global__ __launch_bounds__(64 * kFusedWaves, TOK == 16 ? 2 : 1) void ag_norm_gate_kernel(
    const uint16_t *h, const uint16_t *__restrict__ g, float eps, const uint4 *__restrict__ wp,
    int64_t tokens, int d_in, int L, int H_f, const float *__restrict__ bias, float thr, int n_sink,
    uint16_t *x_out, float *__restrict__ logits, uint8_t *__restrict__ flags) {
  // [wave][4 KiB]: the wave's hand-over buffer (chunk of x, then chunk of W), afterwards its 32 x 32 fp32 partial tile
  __shared__ __attribute__((aligned(16))) uint8_t wst[kFusedWaves][2][4096];
  __shared__ __attribute__((aligned(16))) uint16_t g_l[kFusedWaves * NCH * 64];
  __shared__ float ssq_l[kFusedWaves][32];
  __shared__ uint8_t fl[kNP][16];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // scalar: chunk offsets stay in SGPRs
  constexpr int NI = TOK / 8;  // load / store instructions per chunk: 8 rows each
  const int col = lane & 15, kg = lane >> 4;
  constexpr int MT = TOK / 16;  // 16-token tiles of the MFMA
  const int lr = lane >> 3, lp = lane & 7;  // row within a group of 8 and 16-byte piece of the memory-side layout
  const int64_t tok0 = (int64_t)blockIdx.x * TOK;
  const int nchunks = d_in / 64;
  // The tile's rows through buffer descriptors: a load or store is one per-lane offset plus a scalar chunk offset.
  // Rows past the last token are read as the last token's row again and never stored.
  const int rows = (int)min((int64_t)TOK, tokens - tok0);
  const uint32_t tile_bytes = (uint32_t)rows * (uint32_t)d_in * 2u;
  const __amdgpu_buffer_rsrc_t h_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(h + (size_t)tok0 * d_in), 0, tile_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(x_out + (size_t)tok0 * d_in), 0, tile_bytes, 0x00020000);
  int row_off[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) row_off[i] = min(8 * i + lr, rows - 1) * d_in * 2 + lp * 16;
  auto to_u4 = [](u32x4 v) { return make_uint4(v[0], v[1], v[2], v[3]); };
  uint4 a[NCH][NI];
#pragma unroll
  for (int p = 0; p < NCH; ++p) {
    const int c = min(wave + kFusedWaves * p, nchunks - 1);
#pragma unroll
    for (int i = 0; i < NI; ++i) a[p][i] = to_u4(__builtin_amdgcn_raw_buffer_load_b128(h_rsrc, row_off[i], c * 128, 0));
  }
  // W, requested two chunks ahead of its use
  w_chunk<RAW> wc;
  wc.init(H_f, lane, (AG_LDS uint8_t *)wst[wave][1]);
  auto load_w = [&](uint4 (&bw)[4], int p) { wc.load(bw, wp, min(wave + kFusedWaves * p, nchunks - 1), lane); };
  uint4 b[3][4];
  load_w(b[0], 0);
  load_w(b[1], 1);
  // the normalisation weights: 16 bytes per thread and round cover 4096 of them
  for (int i = (int)threadIdx.x * 8; i < d_in; i += 64 * kFusedWaves * 8)
    *reinterpret_cast<uint4 *>(&g_l[i]) = *reinterpret_cast<const uint4 *>(g + i);

  float ssq[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) ssq[i] = 0.f;
#pragma unroll
  for (int p = 0; p < NCH; ++p)
    if (wave + kFusedWaves * p < nchunks) {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const uint32_t wd[4] = {a[p][i].x, a[p][i].y, a[p][i].z, a[p][i].w};
        // two squares per instruction, on the packed pair as it is (v_dot2_f32_bf16, fp32 sum)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          ssq[i] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, wd[e]), __builtin_bit_cast(bf16x2, wd[e]), ssq[i], false);
      }
    }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    ssq[i] += __shfl_xor(ssq[i], 1, 64);
    ssq[i] += __shfl_xor(ssq[i], 2, 64);
    ssq[i] += __shfl_xor(ssq[i], 4, 64);
    if (lp == 0) ssq_l[wave][8 * i + lr] = ssq[i];
  }
  __syncthreads();  // (also publishes g_l)
  float r[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < kFusedWaves; ++w) tot += ssq_l[w][8 * i + lr];
    r[i] = 1.f / sqrtf(tot / (float)d_in + eps);
  }

  AG_LDS uint8_t *xst = (AG_LDS uint8_t *)wst[wave][0];
  const float bias_h = gate_bias(bias, H_f);
  const bool two = H_f > 16;
  f32x4 acc[MT][2];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) acc[mt][0] = acc[mt][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int p = 0; p < NCH; ++p) {
    __builtin_amdgcn_sched_barrier(0);  // one chunk at a time: interleaving them costs more registers than it hides
    if (p + 2 < NCH) load_w(b[(p + 2) % 3], p + 2);
    const bool valid = wave + kFusedWaves * p < nchunks;  // wave-uniform
    const int c = wave + kFusedWaves * p;
    if (valid) {
      const uint4 gw = *reinterpret_cast<const uint4 *>(&g_l[c * 64 + lp * 8]);
      const uint32_t gd[4] = {gw.x, gw.y, gw.z, gw.w};
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const uint32_t hd[4] = {a[p][i].x, a[p][i].y, a[p][i].z, a[p][i].w};
        uint32_t xd[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float lo = (__uint_as_float(hd[e] << 16) * r[i]) * __uint_as_float(gd[e] << 16);
          const float hi = (__uint_as_float(hd[e] & 0xffff0000u) * r[i]) * __uint_as_float(gd[e] & 0xffff0000u);
          const f32x2 pr = {lo, hi};
          xd[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2));
        }
        const u32x4 xv = {xd[0], xd[1], xd[2], xd[3]};
        if (8 * i + lr < rows) __builtin_amdgcn_raw_buffer_store_b128(xv, x_rsrc, row_off[i], c * 128, 0);
        *reinterpret_cast<AG_LDS u32x4 *>(xst + (8 * i + lr) * 128 + ((lp ^ xkey(8 * i + lr)) << 4)) = xv;
      }
    }
    uint4(&bw)[4] = b[p % 3];
    wc.stage(bw, lane);
    wave_sync();  // the chunk's x rows and W rows are there for every lane
    if (valid) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        bf16x8 af[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          af[mt] = *reinterpret_cast<const AG_LDS bf16x8 *>(xst + (16 * mt + col) * 128 + (((4 * s + kg) ^ xkey(16 * mt + col)) << 4));
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
          if (nt == 0 || two) {
            const bf16x8 wf = wc.frag(bw, s, nt);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[mt], wf, acc[mt][nt], 0, 0, 0);
          }
      }
    }
    wave_sync();  // both buffers have been read
  }
  float(*red)[32][32] = reinterpret_cast<float(*)[32][32]>(wst);
  __syncthreads();  // (red[w] is not wave w's own buffer)
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int r16 = 0; r16 < 4; ++r16) red[wave][16 * mt + 4 * kg + r16][16 * nt + col] = acc[mt][nt][r16];
  __syncthreads();
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    if (mt > 0) __syncthreads();  // (the flags of the first 16 rows have left)
    gate_epilogue([&](int w, int row, int hh) { return red[w][16 * mt + row][hh]; }, fl, (uint32_t)tok0 + 16 * mt, (uint32_t)tokens, L, H_f,
                  bias_h, thr, n_sink, logits, flags);
  }
}

// fp32: v_mfma_f32_16x16x4_f32 on tiles of 16 tokens, the features split over the 8 waves.  A lane's operand elements are
// four consecutive features (one 16-byte load of x, four rows of W), used by four MFMAs: the order of the features in the
// sum is free.  Launches of this path are small: one round of loads and the reduction are its time (128 tokens x 256
// features: 22 us with one thread per logit and a second kernel for the threshold).
__global__ __launch_bounds__(64 * kFusedWaves) void ag_gate_f32_kernel(const float *__restrict__ x, const float *__restrict__ w,
                                                                       uint32_t tokens, int d_in, int L, int H_f,
                                                                       const float *__restrict__ bias, float thr, int n_sink,
                                                                       float *__restrict__ logits, uint8_t *__restrict__ flags) {
  __shared__ float red[kFusedWaves][16][32];
  __shared__ uint8_t fl[kNP][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = lane & 15, kg = lane >> 4;
  const uint32_t tok0 = blockIdx.x * 16;
  const float *xr = x + (size_t)min(tok0 + col, tokens - 1) * d_in;
  const float bias_h = gate_bias(bias, H_f);
  f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
  const bool two = H_f > 16;
  const int n0 = min(col, H_f - 1), n1 = min(16 + col, H_f - 1);  // (columns past H_f: computed, never stored)
  for (int k0 = 16 * wave; k0 < d_in; k0 += 16 * kFusedWaves) {
    const int k = k0 + 4 * kg;
    float xa[4], wa[4], wb[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool in = k + j < d_in;
      const int kk = in ? k + j : d_in - 1;
      xa[j] = in ? xr[kk] : 0.f;
      wa[j] = in ? w[(size_t)kk * H_f + n0] : 0.f;
      wb[j] = two && in ? w[(size_t)kk * H_f + n1] : 0.f;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[j], wa[j], acc[0], 0, 0, 0);
      if (two) acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[j], wb[j], acc[1], 0, 0, 0);
    }
  }
#pragma unroll
  for (int nt = 0; nt < 2; ++nt)
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave][4 * kg + r][16 * nt + col] = acc[nt][r];
  __syncthreads();
  gate_epilogue([&](int v, int row, int h) { return red[v][row][h]; }, fl, tok0, tokens, L, H_f, bias_h, thr, n_sink, logits, flags);
}

}  // namespace

// (the pre-packed copy of W; the rest of the size is from the time when partial sums went through the workspace and is kept,
// so that a workspace that was sufficient, or too small, stays so)
size_t ag_ws_gate_bytes(int64_t tokens, int d_in, int H_f, ag_dtype dt) {
  (void)H_f;
  const int64_t tokens_pad = (tokens + 63) / 64 * 64;
  const size_t part = ag_align256((size_t)16 * tokens_pad * kNP * sizeof(float));
  const size_t pack = dt == AG_BF16 ? ag_align256((size_t)d_in * kNP * 2) : 0;
  return part + pack;
}

hipError_t ag_launch_gate(ag_ctx *ctx, hipStream_t s, const void *feat, ag_dtype dt, int B, int L, int d_in,
                          const void *w, const float *bias, int H_f, float thr, int n_sink, float *logits,
                          uint8_t *flags, ws_cursor &ws) {
  const int64_t tokens = (int64_t)B * L;
  if (tokens > 0xffffffffll - 64) return hipErrorInvalidValue;
  const dim3 block(64 * kFusedWaves);
  if (dt != AG_BF16) {
    AG_LAUNCH(ag_time_kernel(ctx, AG_K_GATE), ag_gate_f32_kernel, dim3((unsigned)((tokens + 15) / 16)), block, 0, s, (const float *)feat,
              (const float *)w, (uint32_t)tokens, d_in, L, H_f, bias, thr, n_sink, logits, flags);
    return hipGetLastError();
  }
  // W as stored when its rows can be moved and transposed in 8- and 16-byte pieces
  const bool raw_w = H_f % 4 == 0 && (reinterpret_cast<uintptr_t>(w) & 15) == 0;
  uint16_t *wp = !raw_w ? ws.take<uint16_t>((size_t)d_in * kNP) : nullptr;
  if (!ws.ok) return hipSuccess;  // caller reports AG_EWORKSPACE
  if (!raw_w) {
    const int n = d_in * kNP;
    hipLaunchKernelGGL(ag_gate_pack_w, dim3((n + 255) / 256), dim3(256), 0, s, (const uint16_t *)w, d_in, H_f, wp);
  }
  const uint4 *wv = (const uint4 *)(raw_w ? w : wp);
  const int64_t tiles = (tokens + 15) / 16;
  const int per_wave = (d_in / 64 + kFusedWaves - 1) / kFusedWaves;  // 64-feature chunks per wave
  const ag_evpair ev = ag_time_kernel(ctx, AG_K_GATE);
  // From two tiles per CU on, and as far as a wave's part of W fits its registers, tiles stream through one workgroup per CU.
  // (Its loads go straight into LDS, 16 bytes a lane: features that are not so aligned go through registers, below.)
  if (tiles >= 2 * ctx->num_cu && per_wave <= 8 && (reinterpret_cast<uintptr_t>(feat) & 15) == 0) {
    const size_t shmem = (size_t)kFusedWaves * (kRing * 2048 + 4096);
#define AG_GATE_STREAM(RAWV, NCHV)                                                                                    \
  do {                                                                                                                \
    static std::atomic<bool> allowed[64];  /* more than 64 KiB of LDS: said once per device */                         \
    if (!allowed[ctx->device & 63].load(std::memory_order_relaxed)) {                                                  \
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&ag_gate_stream_kernel<RAWV, NCHV>),      \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);                \
      if (e != hipSuccess) return e;                                                                                   \
      allowed[ctx->device & 63].store(true, std::memory_order_relaxed);                                                \
    }                                                                                                                  \
    AG_LAUNCH(ev, (ag_gate_stream_kernel<RAWV, NCHV>), dim3(ctx->num_cu), block, shmem, s, (const uint16_t *)feat, wv, (uint32_t)tokens, \
              d_in, L, H_f, bias, thr, n_sink, logits, flags);                                                          \
  } while (0)
#define AG_GATE_STREAM_N(RAWV)                                                                                        \
  do {                                                                                                                \
    if (per_wave <= 1) AG_GATE_STREAM(RAWV, 1); else if (per_wave <= 2) AG_GATE_STREAM(RAWV, 2);                        \
    else if (per_wave <= 4) AG_GATE_STREAM(RAWV, 4); else AG_GATE_STREAM(RAWV, 8);                                      \
  } while (0)
    if (raw_w) AG_GATE_STREAM_N(true); else AG_GATE_STREAM_N(false);
#undef AG_GATE_STREAM_N
#undef AG_GATE_STREAM
    return hipGetLastError();
  }
#define AG_GATE16(RAWV, PFV)                                                                                          \
  AG_LAUNCH(ev, (ag_gate16_kernel<RAWV, PFV>), dim3((unsigned)tiles), block, 0, s, (const uint16_t *)feat, wv, (uint32_t)tokens, d_in, L, \
            H_f, bias, thr, n_sink, logits, flags)
#define AG_GATE16_N(RAWV)                                                                                             \
  do {                                                                                                                \
    if (per_wave <= 1) AG_GATE16(RAWV, 1); else if (per_wave <= 2) AG_GATE16(RAWV, 2);                                  \
    else if (per_wave <= 4) AG_GATE16(RAWV, 4); else AG_GATE16(RAWV, 8);                                                \
  } while (0)
  if (raw_w) AG_GATE16_N(true); else AG_GATE16_N(false);  // (every chunk of a wave in flight, up to 8)
#undef AG_GATE16_N
#undef AG_GATE16
  return hipGetLastError();
}

hipError_t ag_launch_norm_gate(ag_ctx *ctx, hipStream_t s, const void *h, int B, int L, int d_in, const void *g,
                               float eps, const void *w, const float *bias, int H_f, float thr, int n_sink,
                               void *x_out, float *logits, uint8_t *flags, ws_cursor &ws) {
  const int64_t tokens = (int64_t)B * L;
  const bool raw_w = H_f % 4 == 0 && (reinterpret_cast<uintptr_t>(w) & 15) == 0;
  uint16_t *wp = raw_w ? nullptr : ws.take<uint16_t>((size_t)d_in * kNP);
  if (!ws.ok) return hipSuccess;  // caller reports AG_EWORKSPACE
  if (!raw_w) {
    const int n = d_in * kNP;
    hipLaunchKernelGGL(ag_gate_pack_w, dim3((n + 255) / 256), dim3(256), 0, s, (const uint16_t *)w, d_in, H_f, wp);
  }
  // tiles of 16 tokens while 32-token tiles would leave CUs without a workgroup (measured at 4096 features: 4096
  // tokens 17.8 us against 22.0 us; from 8192 tokens on the 32-token tiles are 5-10 % faster); rows of more than
  // 4096 features always take them, with 16 chunks per wave (the same registers as 32 tokens x 8 chunks)
  const bool wide = d_in > 4096;
  const bool tok16 = wide || (tokens + 31) / 32 < ctx->num_cu;
  const dim3 grid((unsigned)((tokens + (tok16 ? 15 : 31)) / (tok16 ? 16 : 32))), block(64 * kFusedWaves);
  const ag_evpair ev = ag_time_kernel(ctx, AG_K_NORM_GATE);
#define AG_NORM_GATE(RAWV, TOKV, NCHV, WPTR)                                                                              \
  AG_LAUNCH(ev, (ag_norm_gate_kernel<RAWV, TOKV, NCHV>), grid, block, 0, s, (const uint16_t *)h, (const uint16_t *)g, eps, \
            (const uint4 *)(WPTR), tokens, d_in, L, H_f, bias, thr, n_sink, (uint16_t *)x_out, logits, flags)
  if (raw_w) {
    if (wide) AG_NORM_GATE(true, 16, 16, w); else if (tok16) AG_NORM_GATE(true, 16, 8, w); else AG_NORM_GATE(true, 32, 8, w);
  } else {
    if (wide) AG_NORM_GATE(false, 16, 16, wp); else if (tok16) AG_NORM_GATE(false, 16, 8, wp); else AG_NORM_GATE(false, 32, 8, wp);
  }
#undef AG_NORM_GATE
  return hipGetLastError();
}
