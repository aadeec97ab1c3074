// conv_split.hip -- 3x3 / stride 1 / pad 1 convolution forward and data
// gradient of fp32 tensors on the bf16 MFMA: every fp32 operand is the sum of
// three bf16 values and a product is six bf16 MFMAs (split_bf16.hpp).
//
// The implicit GEMM of the other convolution kernels: rows = output
// channels, columns = output pixels, reduction = input channels x 9 taps in
// chunks of 32 channels.  A block of 512 threads has a CU to itself: four
// waves multiply, one per SIMD, each 64 channels x 64 pixels (4 x 4 blocks of
// the 16x16x32 MFMA), and four waves stage the input.  The multiplying waves
// are WN along channels x WM along pixels x WK along the reduction (wave group
// g of WK takes chunks g, g + WK, ... through LDS of its own, and the groups'
// sums are added in group order as the tile leaves LDS).  WK fills the chip on
// the late layers, whose output tiles are fewer than its SIMDs, without split
// partials in HBM.
//
//   * Input.  The staging waves load the halo of a chunk as fp32 NCHW (a lane
//     loads 8 channels of one halo pixel: each load is a run of consecutive
//     pixels), split it into its three bf16 parts in registers, and store it
//     to LDS as [part][ci / 8][halo pixel][ci % 8], double-buffered; an MFMA
//     operand is one 16-byte read per lane at one of the 9 shifted windows.
//     On waves of their own, the loads' latency and the splitting stay out of
//     the multiplying waves: loads return in order, so a wave that issues both
//     waits for its input at every filter load (16x16 layer of 128 channels,
//     128 images: 51 us with all waves doing both, two blocks per CU, 44 us
//     like this).
//   * Filters.  Packed once into the MFMA's own lane order (filter_pack_split:
//     [16 output channels][chunk][tap][part][lane][8]), they are read straight
//     from memory into registers, one tap (96 MFMAs) ahead: 1 KB coalesced per
//     operand, the same address in every block of a channel tile.  Through LDS
//     they would need 110 KB per chunk.
//
// Measured (us, batch 128, the fp32-MFMA kernel before): forward 32x32 64
// channels 84 -> 54, 16x16 128 channels 82 -> 43, 8x8 256 channels 78 -> 40;
// 27x45, 75 -> 107 channels, batch 19: 91 -> 38.  A call's first chunk is staged
// before anything multiplies (2.5 us) and its output tile leaves after (2 to
// 4 us); a grid of one round of blocks has nothing to put beside them.
//
// The data gradient is the same contraction with the filters transposed and
// rotated (done by the packing).
#include "conv_common.hpp"
#include "split_bf16.hpp"

#include <algorithm>
#include <cstdio>
#include <mutex>

namespace sb {

template <int TH_, int TW_, int IMGS_, int WN_, int WM_, int WK_>
struct STile {
  static constexpr int TH = TH_, TW = TW_, IMGS = IMGS_;
  static constexpr int WN = WN_, WM = WM_, WK = WK_;
  static_assert(WN * WM * WK == 4, "one multiplying wave per SIMD");
  static constexpr int BM = IMGS * TH * TW, BN = 64 * WN;
  static_assert(BM == 64 * WM, "64 pixels per wave");
  static constexpr int HH = TH + 2, HW = TW + 2, PLANE = IMGS * HH * HW;
  static constexpr int PART = 4 * PLANE * 8;               // bf16 per part of a chunk
  static constexpr int GROUP = 3 * PART, BUF = WK * GROUP;
  static constexpr int TASKS = WK * 4 * PLANE;             // (group, 8 channels, halo pixel)
  static constexpr int XI = (TASKS + 255) / 256;
  // Output staging: WK copies of [channel][pixel], rows BM + 4 floats apart
  // (the four lane groups store rows 4 apart: 16 banks apart).
  static constexpr int EP = BM + 4, COPY = BN * EP;
  static constexpr size_t LDS_STAGE = 2 * (size_t)BUF * sizeof(u16);
  static constexpr size_t LDS_OUT = (size_t)WK * COPY * sizeof(float);
  static constexpr size_t LDS_REDO = LDS_STAGE > LDS_OUT ? LDS_STAGE : LDS_OUT;
  static constexpr size_t LDS_BYTES = LDS_REDO + 16;       // behind them the redo flag
  static_assert(LDS_BYTES <= 160 * 1024, "one block per CU");
  __host__ __device__ static constexpr int hp(int img, int hy, int hx) {
    return (img * HH + hy) * HW + hx;
  }
};
constexpr int kSThreads = 512;

// The block's output tile on the fp32 MFMA, over the channels [c0, c1), for
// blocks that the split cannot carry: operands straight from memory (the
// filters put together from their parts), each tap's sum added only where the
// tap is inside the image.  Writes copy 0 of E, and zeros to the others.
template <class T>
__device__ __forceinline__ void conv_tile_f32(const ConvArgs& a, float* E, int n0, int h0, int w0,
                                              int co0, int c0, int c1, int wave, int lane) {
  const int lr = lane & 15, lq = lane >> 4;
  constexpr int CB = T::BM / 16;
  const int HWs = a.H * a.W, cblk = cdiv(a.Cout, 16);
#pragma unroll 1
  for (int q = wave; q < T::WN * CB; q += kSThreads / 64) {     // 64 channels x 16 pixels
    const int g = q / CB, px = q % CB * 16 + lr;
    const int n = n0 + px / (T::TH * T::TW), h = h0 + px / T::TW % T::TH, w = w0 + px % T::TW;
    const float* x = (const float*)a.in + (size_t)min(n, a.N - 1) * a.Cin * HWs;
    const u16* wp[4];
    f4 acc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int blk = min(co0 / 16 + g * 4 + i, cblk - 1);
      wp[i] = (const u16*)a.wpk + (size_t)blk * a.nchunks * kSplitSlice + lr * 8;
      acc[i] = f4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll 1
    for (int t = 0; t < 9; ++t) {
      const int hh = h + t / 3 - 1, ww = w + t % 3 - 1;
      const bool ok = n < a.N && (unsigned)hh < (unsigned)a.H && (unsigned)ww < (unsigned)a.W;
      f4 c[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) c[i] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
      for (int ch = c0; ch < c1; ch += 32) {       // a lane's channels: 8 lq .. + 7 of the chunk
        const int k = ch + lq * 8;
        const float* xk = x + (size_t)k * HWs + hh * a.W + ww;
        const size_t o = (size_t)(ch >> 5) * kSplitSlice + t * 3 * 512 + lq * 128;
        s8 f[4][3];
        float b[8];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int p = 0; p < 3; ++p) f[i][p] = *reinterpret_cast<const s8*>(wp[i] + o + p * 512);
#pragma unroll
        for (int j = 0; j < 8; ++j) b[j] = ok && k + j < c1 ? xk[(size_t)j * HWs] : 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            c[i] = mfma16x16x4(
                split_value((u16)f[i][0][j], (u16)f[i][1][j], (u16)f[i][2][j]), b[j], c[i]);
      }
      if (ok) {
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] += c[i];
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float* e = E + (g * 64 + i * 16 + 4 * lq + v) * T::EP + px;
        e[0] = acc[i][v];
#pragma unroll
        for (int k = 1; k < T::WK; ++k) e[k * T::COPY] = 0.f;
      }
  }
}

// POOL (forward, unsplit): ReLU and 2x2 max pooling run on the output tile
// and only the pooled tile and its window codes are written, as
// sb_relu_maxpool_fwd computes them.
template <class T, bool DGRAD, bool POOL = false>
__global__ __launch_bounds__(kSThreads, 2) void conv3x3_split_f32(ConvArgs a) {
  static_assert(!POOL || !DGRAD, "pooling follows the forward pass");
  extern __shared__ u16 ldsu[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // Blocks in (split, channel tile, pixel tile) order, dealt to the 8 XCDs in
  // contiguous ranges: an XCD's blocks share filters, and neighbouring pixel
  // tiles their halos, in its L2.
  const int ptiles = a.tiles_w * a.tiles_h * cdiv(a.N, T::IMGS);
  const int co_tiles = cdiv(a.Cout, T::BN);
  int b = blockIdx.x;
  if (gridDim.x % 8 == 0) b = (b % 8) * (gridDim.x / 8) + b / 8;
  int bt = b % ptiles;
  const int ct = b / ptiles % co_tiles, split = b / (ptiles * co_tiles);
  const int tx = bt % a.tiles_w; bt /= a.tiles_w;
  const int ty = bt % a.tiles_h;
  const int n0 = bt / a.tiles_h * T::IMGS, h0 = ty * T::TH, w0 = tx * T::TW;
  const int co0 = ct * T::BN;
  const int kc0 = split * a.chunks_per_split, kc1 = min(a.nchunks, kc0 + a.chunks_per_split);
  const int HWs = a.H * a.W;
  const int nt = cdiv(kc1 - kc0, T::WK);           // rounds: a chunk per wave group
  float* E = reinterpret_cast<float*>(ldsu);
  int* redo = reinterpret_cast<int*>(ldsu + T::LDS_REDO / sizeof(u16));
  if (tid == 0) *redo = 0;

  if (wave >= 4) {
    // ---- staging waves ----
    const int ptid = tid - 256;
    // Task u = (wave group, 8 channels of its chunk, halo pixel), pixels
    // fastest.  x_off: byte offset, from image n0, of the first channel in
    // round 0; out of range outside the image.  x_c: that channel.
    uint32_t x_off[T::XI];
    int x_c[T::XI];
#pragma unroll
    for (int i = 0; i < T::XI; ++i) {
      const int u = ptid + 256 * i;
      const int oct = u / T::PLANE, p = u % T::PLANE;
      const int row = p / T::HW, hx = p % T::HW, img = row / T::HH, hy = row % T::HH;
      const int h = h0 + hy - 1, w = w0 + hx - 1;
      const bool ok = u < T::TASKS && n0 + img < a.N && (unsigned)h < (unsigned)a.H &&
                      (unsigned)w < (unsigned)a.W;
      x_c[i] = kc0 * 32 + oct * 8;
      x_off[i] = ok ? (uint32_t)((img * a.Cin + x_c[i]) * HWs + h * a.W + w) * 4u : kOOB;
    }
    const rsrc_t xr = input_rsrc<float>(a, n0, T::IMGS);
    f8v rx[T::XI];
    uint32_t lost = 0;
    auto gload = [&](int t) {
      const int cb = t * T::WK * 32;
#pragma unroll
      for (int i = 0; i < T::XI; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j)
          rx[i][j] = __builtin_bit_cast(
              float, __builtin_amdgcn_raw_buffer_load_b32(
                         xr, (int)(x_c[i] + cb + j < a.Cin ? x_off[i] : kOOB),
                         (cb + j) * HWs * 4, 0));
    };
    auto lstore = [&](int buf) {
      u16* X = ldsu + buf * T::BUF;
#pragma unroll
      for (int i = 0; i < T::XI; ++i) {
        const int u = ptid + 256 * i;
        if (T::TASKS % 256 != 0 && u >= T::TASKS) continue;
        const int g = u / (4 * T::PLANE), r = u % (4 * T::PLANE);
        const Split8 s = split8(rx[i], lost);
#pragma unroll
        for (int p = 0; p < 3; ++p)
          *reinterpret_cast<s8*>(X + g * T::GROUP + p * T::PART + r * 8) = s.p[p];
        __builtin_amdgcn_sched_barrier(0);         // one task's parts in registers at a time
      }
    };
    gload(0);
    lstore(0);
    if (nt > 1) gload(1);
    __syncthreads();
    for (int t = 0; t < nt; ++t) {
      if (t + 1 < nt) lstore((t & 1) ^ 1);
      if (t + 2 < nt) gload(t + 2);
      __syncthreads();
    }
    if (lost & 0xffffu) *redo = 1;
  } else {
    // ---- multiplying waves ----
    const int lr = lane & 15, lq = lane >> 4;
    const int wm = wave % T::WM, wn = wave / T::WM % T::WN, wk = wave / (T::WM * T::WN);
    int b_off[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int p = wm * 64 + j * 16 + lr;
      const int img = p / (T::TH * T::TW), yy = p / T::TW % T::TH, xx = p % T::TW;
      b_off[j] = wk * T::GROUP + (lq * T::PLANE + T::hp(img, yy, xx)) * 8;
    }
    f4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
    // Filters of this wave: 1 KB operands (chunk, tap, part) of channel block
    // i, at scalar offsets from the wave's first block (a block past Cout
    // reads the last one; its outputs are dropped).
    constexpr uint32_t CHUNK_B = kSplitSlice * sizeof(u16);
    const int cblk = cdiv(a.Cout, 16);
    const int cb16 = min(ct * (T::BN / 16) + wn * 4, cblk - 1);
    const uint32_t w_blk = a.nchunks * CHUNK_B;
    const int last = min(3, cblk - 1 - cb16);
    const rsrc_t wr = make_rsrc((const char*)a.wpk + (size_t)cb16 * w_blk, (last + 1) * w_blk);
    s8 fa[2][4][3], fb[2][3];
    auto rd_a = [&](int t, int tap, int s) {
      const uint32_t o =
          (uint32_t)min(kc0 + t * T::WK + wk, a.nchunks - 1) * CHUNK_B + tap * 3072;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int p = 0; p < 3; ++p)
          fa[s][i][p] = __builtin_bit_cast(
              s8, __builtin_amdgcn_raw_buffer_load_b128(
                      wr, lane * 16, (int)(o + min(i, last) * w_blk + p * 1024), 0));
    };
    auto rd_b = [&](const u16* X, int tap, int j, int s) {
      const int off = T::hp(0, tap / 3, tap % 3) * 8;
#pragma unroll
      for (int p = 0; p < 3; ++p)
        fb[s][p] = *reinterpret_cast<const s8*>(X + b_off[j] + p * T::PART + off);
    };
    // The six products of a block (32 channels at one tap) are summed from zero
    // and added to acc one block later, when they have left the matrix pipe:
    // acc is rounded once per 32 channels and tap instead of six times.
    f4 cp[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) cp[i] = f4{0.f, 0.f, 0.f, 0.f};
    // A round: 9 taps x 4 pixel blocks of the group's chunk (staged as zeros
    // past the last one).  The next tap's filters are requested
    // a whole tap ahead (96 MFMAs, register sets in turn), the next pixel
    // block's inputs one block (24 MFMAs) ahead.  P: the first tap's set.
    auto round = [&](auto P, int t) {
      constexpr int S0 = decltype(P)::value;
      const u16* X = ldsu + (t & 1) * T::BUF;
      rd_b(X, 0, 0, 0);
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) {
        const int s = (tap + S0) & 1;
        if (tap < 8) rd_a(t, tap + 1, s ^ 1);
        else rd_a(t + 1, 0, s ^ 1);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (j < 3) rd_b(X, tap, j + 1, (j + 1) & 1);
          else if (tap < 8) rd_b(X, tap + 1, 0, 0);
          __builtin_amdgcn_sched_barrier(0);         // keep those reads ahead of the MFMAs
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            f4 c = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int m = 0; m < 6; ++m)
              c = mfma16x16x32(fa[s][i][kSplitA[m]], fb[j & 1][kSplitB[m]], c);
            acc[i][(j + 3) & 3] += cp[i];            // the block before
            cp[i] = c;
          }
          // Spread the additions over the MFMAs: 3 MFMAs, 2 additions, ...
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __syncthreads();
    };
    rd_a(0, 0, 0);
    __syncthreads();
    int t = 0;
    for (; t + 1 < nt; t += 2) {
      round(std::integral_constant<int, 0>{}, t);
      round(std::integral_constant<int, 1>{}, t + 1);
    }
    if (t < nt) round(std::integral_constant<int, 0>{}, t);
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i][3] += cp[i];
    if (split_suspect(acc)) *redo = 1;
    // acc[i][j] element v: channel wn*64 + i*16 + 4*lq + v, pixel wm*64 + j*16 + lr.
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          E[wk * T::COPY + (wn * 64 + i * 16 + 4 * lq + v) * T::EP + wm * 64 + j * 16 + lr] =
              acc[i][j][v];
  }

  // ---- the tile leaves through LDS: WK copies of [channel][pixel], pixels
  // image-major, added in group order ----
  __syncthreads();
  if (__builtin_expect(__builtin_amdgcn_readfirstlane(*redo), 0)) {
    conv_tile_f32<T>(a, E, n0, h0, w0, co0, kc0 * 32, min(a.Cin, kc1 * 32), wave, lane);
    __syncthreads();
  }
  if constexpr (POOL) {
    // Pooled pixel q = (channel, image, pooled row, pooled column), columns
    // fastest: the first maximum in row-major window order wins (strict >),
    // the output is the maximum if it is positive, else +0, and bit 7 of the
    // code flags the latter.
    constexpr int PTH = T::TH / 2, PTW = T::TW / 2, PP = T::IMGS * PTH * PTW;
    const int Hh = a.H / 2, Wh = a.W / 2;
#pragma unroll 2
    for (int q = tid; q < T::BN * PP; q += kSThreads) {
      const int col = q / PP, pp = q % PP;
      const int img = pp / (PTH * PTW), r = pp % (PTH * PTW);
      const int py = r / PTW, px = r % PTW;
      const int n = n0 + img, oh = h0 / 2 + py, ow = w0 / 2 + px, co = co0 + col;
      if (n >= a.N || oh >= Hh || ow >= Wh || co >= a.Cout) continue;
      const float* l = E + col * T::EP + (img * T::TH + 2 * py) * T::TW + 2 * px;
      const float bv = a.bias ? a.bias[co] : 0.f;
      float v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float* lk = l + (k >> 1) * T::TW + (k & 1);
        float s = lk[0];
#pragma unroll
        for (int g = 1; g < T::WK; ++g) s += lk[g * T::COPY];
        v[k] = s + bv;
      }
      float m = v[0];
      uint32_t c = 0;
#pragma unroll
      for (int k = 1; k < 4; ++k)
        if (v[k] > m) { m = v[k]; c = (uint32_t)k; }
      const bool pos = m > 0.f;
      const size_t off = (((size_t)n * a.Cout + co) * Hh + oh) * Wh + ow;
      ((float*)a.out)[off] = pos ? m : 0.f;
      a.pool_idx[off] = (uint8_t)(c | (pos ? 0u : 0x80u));
    }
    return;
  }
  // Pieces of 4 consecutive tile pixels of one channel; whole 16-byte moves
  // when they are 4 consecutive aligned elements of the image.
  constexpr int QPR = T::BM / 4;
  const bool part = a.splits > 1;
  float* out = part ? a.part + (size_t)split * a.N * a.Cout * HWs : (float*)a.out;
  const bool vec = (T::TW % 4 == 0 ? a.W % 4 == 0 : a.W == T::TW && a.H == T::TH) &&
                   (((uintptr_t)out | (uintptr_t)(part ? nullptr : a.mask)) & 15) == 0;
#pragma unroll 4
  for (int q = tid; q < T::BN * QPR; q += kSThreads) {
    const int col = q / QPR, px = (q % QPR) * 4;
    const int img = px / (T::TH * T::TW), rem = px % (T::TH * T::TW);
    const int co = co0 + col, n = n0 + img;
    if (co >= a.Cout || n >= a.N) continue;
    f4 v = *reinterpret_cast<const f4*>(E + col * T::EP + px);
#pragma unroll
    for (int g = 1; g < T::WK; ++g)
      v += *reinterpret_cast<const f4*>(E + g * T::COPY + col * T::EP + px);
    const int h = h0 + rem / T::TW, w = w0 + rem % T::TW;
    const size_t base = ((size_t)n * a.Cout + co) * HWs;
    const float bv = !part && a.bias ? a.bias[co] : 0.f;
    if (vec) {
      if (h >= a.H || w >= a.W) continue;
      const size_t off = base + (size_t)h * a.W + w;
      if (!part) {
        f4 mk = f4{1.f, 1.f, 1.f, 1.f};
        if (a.mask) mk = *reinterpret_cast<const f4*>((const float*)a.mask + off);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float r = v[e] + bv;
          if (a.relu && !(r > 0.f)) r = 0.f;
          v[e] = mk[e] > 0.f ? r : 0.f;
        }
      }
      *reinterpret_cast<f4*>(out + off) = v;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int he = h0 + (rem + e) / T::TW, we = w0 + (rem + e) % T::TW;
        if (he >= a.H || we >= a.W) continue;
        const size_t off = base + (size_t)he * a.W + we;
        out[off] = part ? v[e] : conv_epilogue<float>(a, v[e], co, off);
      }
    }
  }
}

// ---------------------------------------------------------------- packing --
// One block per (16 output channels, 32-channel chunk): a slice of 9 x 3
// fragments of 512 bf16, lane-ordered.
template <bool DGRAD>
__global__ __launch_bounds__(256) void filter_pack_split(const float* __restrict__ w,
                                                         u16* __restrict__ out, int Cin,
                                                         int Cout) {
  __shared__ float slice_lds[kSplitSliceLds];
  pack_split_slice<DGRAD>(w, out, Cin, Cout, blockIdx.x, slice_lds);
}

// ---------------------------------------------------------------- host --
struct SPlan {
  int tile, imgs, tiles_w, tiles_h, ptiles, co_tiles, nchunks, cps, splits;
  size_t pack_bytes, part_off, ws_bytes;
  double us;                              // estimated time
};

// Tile table: spatial tile (rows, columns, images), waves along channels,
// pixels and the reduction.
using S16A = STile<8, 16, 1, 2, 2, 1>;
using S16B = STile<16, 16, 1, 1, 4, 1>;
using S16C = STile<8, 16, 1, 1, 2, 2>;
using S8A = STile<8, 8, 1, 4, 1, 1>;
using S8B = STile<8, 8, 1, 2, 1, 2>;
using S8C = STile<8, 8, 1, 1, 1, 4>;
using S4A = STile<4, 4, 4, 4, 1, 1>;
using S4B = STile<4, 4, 4, 2, 1, 2>;
struct STileInfo { int th, tw, imgs, wn, wm, wk; const char* name; };
template <class T> constexpr STileInfo stile_info(const char* name) {
  return {T::TH, T::TW, T::IMGS, T::WN, T::WM, T::WK, name};
}
static const STileInfo kSTiles[] = {
    stile_info<S16A>("8, 16, 1, 2, 2, 1"), stile_info<S16B>("16, 16, 1, 1, 4, 1"),
    stile_info<S16C>("8, 16, 1, 1, 2, 2"), stile_info<S8A>("8, 8, 1, 4, 1, 1"),
    stile_info<S8B>("8, 8, 1, 2, 1, 2"),   stile_info<S8C>("8, 8, 1, 1, 1, 4"),
    stile_info<S4A>("4, 4, 4, 4, 1, 1"),   stile_info<S4B>("4, 4, 4, 2, 1, 2"),
};

// Tile and split of one pass: the candidate with the least estimated time.
// A block per CU; a round of blocks takes its staging of the first chunks and
// its output (about 5 us together) and 7.2 us for every chunk of a wave
// group; split partials cost their traffic and a launch.
static SPlan split_plan(int N, int Cin, int H, int W, int Cout) {
  SPlan best{};
  double best_t = 0;
  const int nchunks = cdiv(Cin, 32);
  for (int i = 0; i < (int)(sizeof(kSTiles) / sizeof(kSTiles[0])); ++i) {
    const STileInfo& t = kSTiles[i];
    if (t.tw > 8 && W <= 8) continue;
    if (t.tw == 4 && W >= 8) continue;
    SPlan p{};
    p.tile = i;
    p.imgs = t.imgs;
    p.tiles_w = cdiv(W, t.tw);
    p.tiles_h = cdiv(H, t.th);
    p.ptiles = p.tiles_w * p.tiles_h * cdiv(N, t.imgs);
    p.co_tiles = cdiv(Cout, 64 * t.wn);
    p.nchunks = nchunks;
    const int rounds = cdiv(nchunks, t.wk);
    for (int s = 1; s <= 8 && s <= rounds; ++s) {
      p.cps = cdiv(rounds, s) * t.wk;
      p.splits = cdiv(nchunks, p.cps);
      if (p.splits != s) continue;
      const long blocks = std::min<long>((long)p.ptiles * p.co_tiles * s, 1l << 30);
      const double out_mb = (double)N * Cout * H * W * 4e-6;
      const double est = cdiv((int)blocks, 256) * (5.0 + 7.2 * cdiv(std::min(p.cps, nchunks), t.wk)) +
                         (s > 1 ? 3.0 + out_mb * (s + 1) / 4.0 : 0.0);
      if (best_t == 0 || est < best_t) { best = p; best_t = best.us = est; }
    }
  }
  best.pack_bytes = (size_t)cdiv(Cout, 16) * nchunks * kSplitSlice * sizeof(u16);
  best.part_off = round_up(best.pack_bytes, 256);
  best.ws_bytes = best.part_off + (best.splits > 1 ? (size_t)best.splits * N * Cout * H * W *
                                                         sizeof(float) : 0);
  return best;
}

template <class T, bool DGRAD>
static void split_launch(const SPlan& p, const ConvArgs& a, hipStream_t st) {
  static std::once_flag once;
  std::call_once(once, [] {
    (void)hipFuncSetAttribute((const void*)conv3x3_split_f32<T, DGRAD>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)T::LDS_BYTES);
    if constexpr (!DGRAD)
      (void)hipFuncSetAttribute((const void*)conv3x3_split_f32<T, false, true>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)T::LDS_BYTES);
  });
  const unsigned grid = (unsigned)(p.ptiles * p.co_tiles * p.splits);
  if constexpr (!DGRAD) {
    if (a.pool_idx && p.splits == 1) {
      conv3x3_split_f32<T, false, true><<<grid, kSThreads, T::LDS_BYTES, st>>>(a);
      return;
    }
  }
  conv3x3_split_f32<T, DGRAD><<<grid, kSThreads, T::LDS_BYTES, st>>>(a);
  if (p.splits > 1) {
    const size_t total = (size_t)a.N * a.Cout * a.H * a.W;
    if (a.pool_idx)
      launch_splitk_reduce_pool<float>(a, p.splits, total, st);
    else
      launch_splitk_reduce<float>(a.part, p.splits, total, a.Cout, a.H * a.W, a.bias, a.relu,
                                  (const float*)a.mask, (float*)a.out, st);
  }
}

template <bool DGRAD>
static void split_dispatch(const SPlan& p, const ConvArgs& a, hipStream_t st) {
  switch (p.tile) {
    case 0: split_launch<S16A, DGRAD>(p, a, st); break;
    case 1: split_launch<S16B, DGRAD>(p, a, st); break;
    case 2: split_launch<S16C, DGRAD>(p, a, st); break;
    case 3: split_launch<S8A, DGRAD>(p, a, st); break;
    case 4: split_launch<S8B, DGRAD>(p, a, st); break;
    case 5: split_launch<S8C, DGRAD>(p, a, st); break;
    case 6: split_launch<S4A, DGRAD>(p, a, st); break;
    default: split_launch<S4B, DGRAD>(p, a, st); break;
  }
}

}  // namespace sb

namespace sbh {

// Estimated time in us of the fp32-MFMA kernels of conv_igemm.hip: rounds of 512
// blocks of 64 channels x 128 pixels (their tiles: 4x32, 8x16, 2 images of 8x8,
// 8 of 4x4), split over chunks of 8 channels where they are fewer.
static double fp32_mfma_us(int N, int Cin, int H, int W, int Cout) {
  using sb::cdiv;
  long tiles;
  if (W >= 32) tiles = (long)N * cdiv(W, 32) * cdiv(H, 4);
  else if (W >= 16) tiles = (long)N * cdiv(W, 16) * cdiv(H, 8);
  else if (W >= 8) tiles = (long)cdiv(N, 2) * cdiv(W, 8) * cdiv(H, 8);
  else if (W == 4 && H == 4) tiles = 2 * cdiv(N, 16);
  else tiles = (long)cdiv(N, 8) * cdiv(W, 4) * cdiv(H, 4);
  const long blocks = tiles * cdiv(Cout, 64);
  const int nchunks = cdiv(Cin, 8);
  int splits = 1;
  if (blocks < 512)
    splits = (int)std::min<long>(std::min(8, std::max(1, nchunks / 2)), (512 + blocks - 1) / blocks);
  const int cps = cdiv(nchunks, splits);
  splits = cdiv(nchunks, cps);
  const long all = blocks * splits;
  return 1.73 + (double)((all + 511) / 512) * (0.54 + 2.63 * cps) + 3.83 * all / 512 * cps +
         (splits > 1 ? 2.25 + 0.83e-6 * N * Cout * H * W * (splits + 1) : 0.0);
}

// Whether an fp32 pass runs here; the fp32-MFMA kernels of conv_igemm.hip take
// the others.  Never: images narrower than 4 (2x2 kernels skip the 56 % of the
// products that are padding), 16 input channels or fewer (a chunk is 32), wide
// images of 16 output channels or fewer (a tile is 64), sizes whose offsets
// pass 2^31 bytes.  Otherwise where the estimated time is the smaller one; a
// pass of a single chunk has no loop to hide its first loads in (1.3 us).  Narrow
// images of 4e7 products or more always run here, as only these tiles pool
// where the reduction is not split.
// Fitted to both kernels' times of 597 passes: the one taken is 0.5 % slower than
// the faster one on average, and slower than the fp32 MFMA in 8, by 14 % at most
// (a line by work and pixels alone: 5 %, 30, 33 %).  Forward and data gradient
// in us, fp32 MFMA and here: 16x16 128 -> 128, 8 images 44, 50; 20x20 32 -> 24, 74
// images 23, 31; 14x14 32 -> 256, 64 images 40, 29; 4x4 512 -> 512, 16 images 85, 64.
bool conv_split_takes(int N, int Cin, int H, int W, int Cout) {
  if (W < 4 || Cin <= 16 || (W >= 32 && Cout <= 16)) return false;
  // 32-bit offsets: the filters of a wave's four channel blocks, and an image
  // up to the end of its last chunk of channels.
  const int64_t nchunks = sb::cdiv(Cin, 32);
  if (4 * nchunks * sb::kSplitSlice * (int64_t)sizeof(sb::u16) >= (1ll << 31) ||
      (nchunks * 32 + 8) * H * W * 4 >= (1ll << 31))
    return false;
  if (W < 8 && (double)N * H * W * Cin * Cout >= 4e7) return true;
  return fp32_mfma_us(N, Cin, H, W, Cout) >
         1.2 * sb::split_plan(N, Cin, H, W, Cout).us + (nchunks == 1 ? 1.3 : 0.0);
}

size_t conv_split_ws(int N, int Cin, int H, int W, int Cout, bool prepacked) {
  const sb::SPlan p = sb::split_plan(N, Cin, H, W, Cout);
  return prepacked ? p.ws_bytes - p.part_off : p.ws_bytes;
}

size_t conv_split_pack_bytes(int N, int Cin, int H, int W, int Cout) {
  return sb::split_plan(N, Cin, H, W, Cout).pack_bytes;
}

void conv_split_pack(bool dgrad, int Cin, int Cout, const void* wt, void* packed,
                     hipStream_t st) {
  const unsigned g = (unsigned)(sb::cdiv(Cout, 16) * sb::cdiv(Cin, 32));
  if (dgrad)
    sb::filter_pack_split<true><<<g, 256, 0, st>>>((const float*)wt, (sb::u16*)packed, Cin, Cout);
  else
    sb::filter_pack_split<false><<<g, 256, 0, st>>>((const float*)wt, (sb::u16*)packed, Cin, Cout);
}

int conv_split_describe(bool dgrad, int N, int Cin, int H, int W, int Cout, char* buf, size_t len,
                        bool pool) {
  const sb::SPlan p = sb::split_plan(N, Cin, H, W, Cout);
  return snprintf(buf, len, "sb::conv3x3_split_f32<sb::STile<%s>, %s, %s> grid=%dx%dx%d",
                  sb::kSTiles[p.tile].name, dgrad ? "true" : "false",
                  pool && p.splits == 1 ? "true" : "false", p.ptiles, p.co_tiles, p.splits);
}

sb_status conv_split(bool dgrad, int N, int Cin, int H, int W, int Cout, const void* in,
                     const void* wt, const float* bias, const void* mask, void* out, void* ws,
                     size_t ws_bytes, int relu, bool prepacked, hipStream_t st,
                     uint8_t* pool_idx) {
  const sb::SPlan p = sb::split_plan(N, Cin, H, W, Cout);
  // Offsets within a block's images stay below 2^31 bytes.
  if ((int64_t)std::min(p.imgs, N) * Cin * H * W * 4 >= (1ll << 31)) return SB_ERR_UNSUPPORTED;
  const size_t part_off = prepacked ? 0 : p.part_off;
  const size_t need = prepacked ? p.ws_bytes - p.part_off : p.ws_bytes;
  if (need && (ws == nullptr || ws_bytes < need)) return SB_ERR_WORKSPACE;
  if (pool_idx && (dgrad || relu)) return SB_ERR_UNSUPPORTED;
  sb::ConvArgs a{};
  a.in = in; a.wt = wt; a.bias = bias; a.mask = mask; a.out = out; a.pool_idx = pool_idx;
  a.wpk = prepacked ? wt : ws;
  a.part = p.splits > 1 ? (float*)((char*)ws + part_off) : nullptr;
  a.N = N; a.Cin = Cin; a.H = H; a.W = W; a.Cout = Cout;
  a.tiles_w = p.tiles_w; a.tiles_h = p.tiles_h;
  a.nchunks = p.nchunks; a.chunks_per_split = p.cps; a.splits = p.splits; a.relu = relu;
  if (!prepacked) conv_split_pack(dgrad, Cin, Cout, wt, ws, st);
  if (dgrad) sb::split_dispatch<true>(p, a, st);
  else sb::split_dispatch<false>(p, a, st);
  return launch_status();
}

}  // namespace sbh
