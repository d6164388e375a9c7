// Products of a few rows (routing prefixes of a few documents) in bf16, without operands in LDS.  Bound by dependent launches, by
// the latency of memory and by what one compute unit streams from beyond its L2 (44 GB/s measured): a block's products are spread over as
// many workgroups as read whole 64-byte pieces of the weights' rows, and every wave has its loads in flight at once.
//   rows_product_kernel   32 rows x 32 columns a workgroup, seven waves along K: the q | k | v and the up-projection (32 x 896 -> 2688 and
//                         3584: 6.5 and 6.2 - 7.6 us in the fitted 32 x 64 tile, 5.7 and 6.3 here; 32 x 256 -> 768 and 1024: 1.5 us less each)
//   attn_out_kernel       attention of two heads over up to 32 positions, and their rows of the output projection for 64 columns: a plane of
//                         the sum over heads that the LayerNorm behind adds.  Every column's workgroup repeats the attention: it is
//                         shorter than the launch it replaces (32 x 14 heads x 64 -> 896: 3.1 + 6.2 us and a gap, 4.2 here; 256 rows of 896
//                         features 534 -> 500 us with it).
// One document through 12 blocks of 896 419 -> 351 us.  Left out, measured: a workgroup per head that takes its columns of q | k | v
// too, and one per 128 hidden columns for the whole MLP: 459 KB of weights a workgroup are 10 us of streaming, 472 us.
// Weights go from memory into registers as pieces of rows: a lane takes COLS adjacent columns of eight K and turns them into COLS B
// fragments of v_mfma_f32_16x16x32_bf16, tile t holding columns COLS c + t.
#include <algorithm>
#include <type_traits>

#include "gemm_common.h"
#include "kernels.h"

namespace dipaco {

namespace {

constexpr int SF_ROWS = 32;   // rows of a workgroup

// 32 of K x 16 COLS columns; lane (c = l % 16, g = l / 16): columns COLS c .. of the eight K that k_of(g, j) names
template <int COLS> struct Unit {
  static_assert(COLS == 2 || COLS == 4, "4 or 8 bytes a load");
  uint32_t w[8][COLS / 2];
  __device__ __forceinline__ void load_row(int j, const bf16* p) {
    if constexpr (COLS == 2) w[j][0] = *reinterpret_cast<const uint32_t*>(p);
    else { const uint2 x = *reinterpret_cast<const uint2*>(p); w[j][0] = x.x; w[j][1] = x.y; }
  }
  // rows k0 + 8 g + j of W.  K rows and columns beyond the matrix re-read the last ones: the A fragments are zero there, such columns
  // are not used.  Wave-uniform bases and 32-bit lane offsets (a matrix has less than 2^31 elements)
  __device__ __forceinline__ void load(const bf16* __restrict__ W, int ldw, int k0, int K, int col0, int cols, int lane) {
    const uint32_t col = min(col0 + COLS * (lane & 15), cols - COLS);
    if (k0 + 32 <= K) {   // uniform
      const uint32_t off = 8 * (lane >> 4) * (uint32_t)ldw + col;
#pragma unroll
      for (int j = 0; j < 8; ++j) load_row(j, W + (size_t)(k0 + j) * ldw + off);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) load_row(j, W + ((uint32_t)min(k0 + 8 * (lane >> 4) + j, K - 1) * (uint32_t)ldw + col));
    }
  }
  template <int t> __device__ __forceinline__ bf16x8 frag() const {
    auto pair = [&](int p) { return __builtin_amdgcn_perm(w[2 * p + 1][t / 2], w[2 * p][t / 2], (t & 1) ? 0x07060302u : 0x05040100u); };
    return __builtin_bit_cast(bf16x8, make_uint4(pair(0), pair(1), pair(2), pair(3)));
  }
};

// ---- weights of a later launch -----------------------------------------------------------------------------------
// A product of a few rows waits for its weights, 1.5 us of a launch of 5 when they come from memory, and the launches before it leave half
// of the compute units idle.  So these have workgroups behind their own that read a word of every 128-byte line of the weights that a
// product one to three launches on will read, each XCD those of its own workgroups: lines stay in an XCD's L2 over the end of a kernel.  One
// document through 12 blocks of 896, weights from memory 386 -> 332 us, with the last pass's still in the 256 MB cache 331 -> 326; lines
// dealt to any XCD 347 and 346.  More documents have more workgroups of their own and gain less: from memory 3 | 4 | 6 | 8 documents 436 -> 422 | 450 ->
// 432 | 523 -> 499 | 594 -> 562, level at 2 and from 12 on; from the last-level cache 1 - 2 % at 3 - 8, level from 12 on, and 2 documents 344 -> 348.  Up to
// 384 wide level (a pass's weights stay in the L2s), 512 wide 1 | 4 documents from memory 327 -> 303 | 339 -> 332.  The output projection's
// weights, whose loads run under the attention, gain nothing from it (334).
// Item v of that product's `items` (dealt to the XCDs in contiguous ranges) reads piece v / items_per_piece.  The launch's size comes as an
// argument: gridDim and blockDim bring 256 bytes of hidden ones, which a process whose host writes arguments slowly shows (issuing the 75 launches
// of a pass, 12 blocks of 256: 270 us with them, 253 so; in others 200 both ways).
template <int THREADS> __device__ __forceinline__ void touch(const WeightTiles& w, int block, int part, int parts) {
  const int x = block % N_XCD, per = w.items / N_XCD, rem = w.items % N_XCD;
  const int first = x * per + min(x, rem), last = first + per + (x < rem) - 1;
  if (last < first) return;
  const int p0 = first / w.items_per_piece, lines = (last / w.items_per_piece - p0 + 1) * w.piece_rows;
  for (int i = part * THREADS + (int)threadIdx.x; i < lines; i += parts * THREADS) {
    const int q = i / w.piece_rows, piece = p0 + q, row_block = piece / w.pieces_n;
    const int row = row_block * w.piece_rows + (i - q * w.piece_rows), col = 128 * (piece - row_block * w.pieces_n);
    if (row < w.rows && col < w.row_bytes) (void)*reinterpret_cast<const volatile uint32_t*>(static_cast<const char*>(w.base) + (size_t)row * w.row_bytes + col);
  }
}
// workgroups of `threads` for it, a line a thread
static int touch_blocks(const WeightTiles& w, int threads) {
  if (!w.items) return 0;
  const int lines = ((w.items + N_XCD - 1) / N_XCD / w.items_per_piece + 1) * w.piece_rows;
  return N_XCD * ((lines + threads - 1) / threads);
}

// ---- C[rows, N] = x[rows, K] W[K, N] + bias, GELU -----------------------------------------------------------------
constexpr int RP_WAVES = 7, RP_COLS = 32, RP_AHEAD = 4;
constexpr int RP_LD = RP_COLS + 4;   // floats between rows of the waves' sums

template <bool GELU>
__global__ void __launch_bounds__(RP_WAVES * WAVE) rows_product_kernel(const bf16* __restrict__ x, const bf16* __restrict__ W,
                                                                       const bf16* __restrict__ bias, bf16* __restrict__ out, int n_rows, int N, int K,
                                                                       int tiles, int blocks, WeightTiles ahead) {
  if ((int)blockIdx.x >= tiles) return touch<RP_WAVES * WAVE>(ahead, blockIdx.x, ((int)blockIdx.x - tiles) / N_XCD, (blocks - tiles) / N_XCD);
  __shared__ __attribute__((aligned(16))) float red[RP_WAVES][SF_ROWS][RP_LD];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  // neighbouring columns on one XCD: a 128-byte line of the weights holds two workgroups' columns, and each XCD that reads it fetches all of it
  const int tile = xcd_contiguous(blockIdx.x, tiles), row_tiles = (n_rows + SF_ROWS - 1) / SF_ROWS, tile_n = tile / row_tiles;
  const int n0 = tile_n * RP_COLS, row0 = (tile - tile_n * row_tiles) * SF_ROWS, rows = min(SF_ROWS, n_rows - row0);
  const int steps = (K + 31) / 32, s1 = (wave + 1) * steps / RP_WAVES;
  const int row = tid >> 3, col = 4 * (tid & 7);   // of the output: 256 threads of four columns each
  const bool on = row < rows && n0 + col < N;
  bf16x4 bi = {};
  if (on) bi = *reinterpret_cast<const bf16x4*>(bias + n0 + col);
  f32x4 acc[2][2];
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int t = 0; t < 2; ++t) acc[rb][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  uint32_t x_off[2];   // rows beyond the last re-read it
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) x_off[rb] = (uint32_t)((row0 + min(16 * rb + c, rows - 1)) * K + 8 * g);
  for (int s = wave * steps / RP_WAVES; s < s1; s += RP_AHEAD) {
    Unit<2> u[RP_AHEAD];
    uint4 a[RP_AHEAD][2];
#pragma unroll
    for (int i = 0; i < RP_AHEAD; ++i)
      if (s + i < s1) {
        const int k = 32 * (s + i);
        u[i].load(W, N, k, K, n0, N, lane);
        const int over = max(0, k + 8 * g + 8 - K);   // K is a multiple of 8: 0, or all of the lane's eight lie beyond it
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
          const uint4 v = *reinterpret_cast<const uint4*>(x + (x_off[rb] + (uint32_t)(k - over)));
          const uint32_t m = over ? 0u : 0xffffffffu;
          a[i][rb] = make_uint4(v.x & m, v.y & m, v.z & m, v.w & m);
        }
      }
#pragma unroll
    for (int i = 0; i < RP_AHEAD; ++i)
      if (s + i < s1) {
        const bf16x8 b[2] = {u[i].frag<0>(), u[i].frag<1>()};
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
          for (int t = 0; t < 2; ++t)
            acc[rb][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[i][rb]), b[t], acc[rb][t], 0, 0, 0);
      }
  }
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      *reinterpret_cast<float2*>(&red[wave][16 * rb + 4 * g + e][2 * c]) = make_float2(acc[rb][0][e], acc[rb][1][e]);
  __syncthreads();
  if (!on) return;
  float4 s = *reinterpret_cast<const float4*>(&red[0][row][col]);
#pragma unroll
  for (int w = 1; w < RP_WAVES; ++w) {   // in order
    const float4 v = *reinterpret_cast<const float4*>(&red[w][row][col]);
    s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
  }
  float v[4] = {s.x + (float)bi[0], s.y + (float)bi[1], s.z + (float)bi[2], s.w + (float)bi[3]};
  bf16x4 y;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float unused;
    y[i] = (bf16)(GELU ? gelu_with_grad_t<bf16>(v[i], unused) : v[i]);
  }
  *reinterpret_cast<bf16x4*>(out + (size_t)(row0 + row) * N + n0 + col) = y;
}

// ---- attention of two heads and their rows of the output projection ----------------------------------------------------
constexpr int AO_DH = 64, AO_HEADS = 2;
constexpr int AO_K = AO_HEADS * AO_DH, AO_STEPS = AO_K / 32;
constexpr int AO_ATT = 2 * AO_HEADS, AO_WAVES = AO_ATT + AO_STEPS;   // waves of 16 queries and a head; of 32 of K
constexpr int AO_ROW = 2 * AO_K + 16;   // bytes between rows of the heads' output
constexpr int AO_LD = 64 + 4;

// qkv [B S, 3 A] -> planes [ceil(H / 2)][B S, d]
__global__ void __launch_bounds__(AO_WAVES * WAVE) attn_out_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ w_o,
                                                                   float* __restrict__ planes, int S, int H, int d, int docs, int tiles,
                                                                   int blocks, WeightTiles ahead) {
  if ((int)blockIdx.x >= tiles) return touch<AO_WAVES * WAVE>(ahead, blockIdx.x, ((int)blockIdx.x - tiles) / N_XCD, (blocks - tiles) / N_XCD);
  __shared__ __attribute__((aligned(16))) char o_[SF_ROWS * AO_ROW];
  __shared__ __attribute__((aligned(16))) float red[AO_STEPS][SF_ROWS][AO_LD];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4, A = H * AO_DH;
  const int item = xcd_contiguous(blockIdx.x, tiles), piece = item / docs, doc = item - piece * docs, cols = (d + 63) / 64, plane = piece / cols;
  const int n0 = (piece - plane * cols) * 64, head0 = plane * AO_HEADS;
  if (wave < AO_ATT) {   // the arithmetic of attn_fwd_short_mfma<64>: probabilities rounded to bf16, sums of the rounded
    const int head = head0 + (wave >> 1), query = 16 * (wave & 1) + c;
    char* const o_row = o_ + query * AO_ROW + 2 * AO_DH * (wave >> 1);
    if (head < H) {
      const long ld = 3L * A;
      const bf16* const base = qkv + (long)doc * S * ld + head * AO_DH;
      uint4 qf[2], kf[2][2];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        qf[s] = *reinterpret_cast<const uint4*>(base + min(query, S - 1) * ld + 32 * s + 8 * g);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) kf[kb][s] = *reinterpret_cast<const uint4*>(base + A + min(16 * kb + c, S - 1) * ld + 32 * s + 8 * g);
      }
      Unit<4> v;   // V^T as A fragments; its keys in the order in which a lane holds a query's scores
#pragma unroll
      for (int j = 0; j < 8; ++j) v.load_row(j, base + 2 * A + min(16 * (j >> 2) + 4 * g + (j & 3), S - 1) * ld + 4 * c);
      f32x4 st[2];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        st[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 2; ++s)
          st[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[kb][s]), __builtin_bit_cast(bf16x8, qf[s]), st[kb], 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (16 * kb + 4 * g + e > query) st[kb][e] = -INFINITY;
      }
      float mx = fmaxf(fmaxf(fmaxf(st[0][0], st[0][1]), fmaxf(st[0][2], st[0][3])), fmaxf(fmaxf(st[1][0], st[1][1]), fmaxf(st[1][2], st[1][3])));
      mx = fmaxf(mx, __shfl_xor(mx, 16, WAVE));
      mx = fmaxf(mx, __shfl_xor(mx, 32, WAVE));
      constexpr float sc = 0.125f * 1.4426950408889634f;   // 1 / sqrt(64), base-2 exponentials
      const float top = mx * sc;
      bf16x8 p;
      float l = 0.f;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          p[4 * kb + e] = (bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(st[kb][e], sc, -top));
          l += (float)p[4 * kb + e];
        }
      l += __shfl_xor(l, 16, WAVE);
      l += __shfl_xor(l, 32, WAVE);
      const float scale = 1.0f / l;
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      const f32x4 ot[4] = {__builtin_amdgcn_mfma_f32_16x16x32_bf16(v.frag<0>(), p, zero, 0, 0, 0),
                           __builtin_amdgcn_mfma_f32_16x16x32_bf16(v.frag<1>(), p, zero, 0, 0, 0),
                           __builtin_amdgcn_mfma_f32_16x16x32_bf16(v.frag<2>(), p, zero, 0, 0, 0),
                           __builtin_amdgcn_mfma_f32_16x16x32_bf16(v.frag<3>(), p, zero, 0, 0, 0)};
#pragma unroll
      for (int e = 0; e < 4; ++e) {   // row 4 g + e of tile t is head column 4 (4 g + e) + t
        const bf16x4 y = {(bf16)(ot[0][e] * scale), (bf16)(ot[1][e] * scale), (bf16)(ot[2][e] * scale), (bf16)(ot[3][e] * scale)};
        *reinterpret_cast<bf16x4*>(o_row + 2 * (16 * g + 4 * e)) = y;
      }
    } else {   // an odd number of heads: the second one counts as zero
#pragma unroll
      for (int e = 0; e < 4; ++e) *reinterpret_cast<uint2*>(o_row + 2 * (16 * g + 4 * e)) = make_uint2(0, 0);
    }
    __syncthreads();
  } else {
    const int s = wave - AO_ATT;
    Unit<4> w;   // in flight over the attention
    w.load(w_o, d, head0 * AO_DH + 32 * s, A, n0, d, lane);
    __syncthreads();
    const bf16x8 b[4] = {w.frag<0>(), w.frag<1>(), w.frag<2>(), w.frag<3>()};
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(o_ + (16 * rb + c) * AO_ROW + 64 * s + 16 * g);
      f32x4 acc[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[t], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        *reinterpret_cast<float4*>(&red[s][16 * rb + 4 * g + e][4 * c]) = make_float4(acc[0][e], acc[1][e], acc[2][e], acc[3][e]);
    }
  }
  __syncthreads();
  const int row = tid >> 4, col = 4 * (tid & 15);   // 512 threads of four columns each
  if (row >= S || n0 + col >= d) return;
  float4 y = *reinterpret_cast<const float4*>(&red[0][row][col]);
#pragma unroll
  for (int s = 1; s < AO_STEPS; ++s) {
    const float4 v = *reinterpret_cast<const float4*>(&red[s][row][col]);
    y.x += v.x; y.y += v.y; y.z += v.z; y.w += v.w;
  }
  *reinterpret_cast<float4*>(planes + ((size_t)(plane * docs + doc) * S + row) * d + n0 + col) = y;
}

}  // namespace

// Workgroups of up to three quarters of the compute units: 2 x 32 x 896 -> 2688 (168) is ahead of the fitted tile, 3 x 32 (252) behind it
bool small_product_takes(int rows, int N, int K) {
  return rows <= SMALL_FORWARD_ROWS && K >= 256 && (long)((N + RP_COLS - 1) / RP_COLS) * ((rows + SF_ROWS - 1) / SF_ROWS) <= 192;
}
// Every document's workgroups read W_o again, so it is their number that the rule bounds, however short the documents are.  Features of
// B x S tokens with two launches -> this one, us: d_model 896, 14 heads (98 workgroups a document): 8 x 32 271 -> 254, 16 x 16 266 -> 265, 32 x
// 8 263 -> 294, 256 x 1 275 -> 683; 512, 8 heads (32): 32 x 8 136 -> 135, 64 x 4 135 -> 148; 256, 4 heads (8): 128 x 2 122 -> 107, 256 x 1 121 -> 119.
constexpr long AO_MOST = 1024;
int attn_out_most_planes(int H, int d_head) {
  const int planes = (H + AO_HEADS - 1) / AO_HEADS;
  return d_head == AO_DH && planes >= 2 && planes <= 8 ? planes : 0;
}
int attn_out_planes(int B, int S, int H, int d_head, int d) {
  const int planes = attn_out_most_planes(H, d_head);
  return S <= SF_ROWS && (long)B * S <= SMALL_FORWARD_ROWS && (long)((d + 63) / 64) * planes * B <= AO_MOST ? planes : 0;
}

WeightTiles small_product_weights(const bf16* W, int rows, int N, int K) {   // two tiles' columns a line
  const int row_tiles = (rows + SF_ROWS - 1) / SF_ROWS, tiles = (N + RP_COLS - 1) / RP_COLS;
  return WeightTiles{W, 2 * N, K, tiles * row_tiles, 2 * row_tiles, K, (tiles + 1) / 2};
}
dipaco_status launch_small_product(const bf16* x, const bf16* W, const bf16* bias, bf16* out, int rows, int N, int K, bool gelu, const WeightTiles& ahead,
                                   hipStream_t s) {
  const int tiles = (N + RP_COLS - 1) / RP_COLS * ((rows + SF_ROWS - 1) / SF_ROWS);
  const int grid = tiles + touch_blocks(ahead, RP_WAVES * WAVE);
  if (gelu) rows_product_kernel<true><<<grid, RP_WAVES * WAVE, 0, s>>>(x, W, bias, out, rows, N, K, tiles, grid, ahead);
  else rows_product_kernel<false><<<grid, RP_WAVES * WAVE, 0, s>>>(x, W, bias, out, rows, N, K, tiles, grid, ahead);
  DIPACO_LAUNCH_CHECK();
  return DIPACO_OK;
}

dipaco_status launch_attn_out(const bf16* qkv, const bf16* w_o, float* planes, int B, int S, int H, int d, const WeightTiles& ahead, hipStream_t s) {
  const int tiles = (d + 63) / 64 * ((H + AO_HEADS - 1) / AO_HEADS) * B;
  const int grid = tiles + touch_blocks(ahead, AO_WAVES * WAVE);
  attn_out_kernel<<<grid, AO_WAVES * WAVE, 0, s>>>(qkv, w_o, planes, S, H, d, B, tiles, grid, ahead);
  DIPACO_LAUNCH_CHECK();
  return DIPACO_OK;
}

}  // namespace dipaco
