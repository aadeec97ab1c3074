// conv_wgrad_split.hip -- 3x3 / stride 1 / pad 1 convolution weight and bias
// gradients of fp32 tensors on the bf16 MFMA, every fp32 operand split in
// three bf16 parts (split_bf16.hpp):
//   dw[k,c,r,s] = sum_{n,h,w} x[n,c,h+r-1,w+s-1] * dy[n,k,h,w]
//   db[k]       = sum_{n,h,w} dy[n,k,h,w]
//
// GEMM view: rows = output channels k, columns = input channels c at each of
// the 9 taps, reduction = pixels.  A block of 512 threads has a CU to itself
// and owns 64 k x 16 c x 9 taps over a contiguous range of 128-pixel tiles:
// four waves stage the next tile while four multiply, each the block's whole
// output for 32 of the tile's pixels (one 16x16x32 MFMA step: 4 x 9 blocks of
// 16 k x 16 c, 216 MFMAs).  The four waves' sums are added in wave order
// through LDS at the end, so a block writes 37 KB of partials for its share of
// the pixels, a fourth of what four waves with output blocks of their own
// would (all accumulators of the chip are 38 MB).
//
// Rounding.  The MFMA drops low bits always in one direction, so the local
// sums of 32 pixels are off by a little with the same sign and over 1e5 pixels
// that adds up (dw of 128 images of 32x32 against 64 bits: 4.4e-7, on the fp32
// MFMA 4.0e-7).  dy is therefore negated for the odd waves' pixels as it is
// staged, and their sums are subtracted: the shares cancel (1.2e-7).  (Flipped
// as the multiplying waves read it, their registers spill: 193 -> 213 us for a
// 32x32 layer's three passes.)
//
//   * Staging: a lane loads 8 channels of 4 consecutive pixels as fp32 NCHW
//     (16-byte loads where rows are whole aligned quads), splits them, and
//     stores each pixel as three 16-byte pieces [part][channel / 8][pixel]
//     [channel % 8]; the x tile is a halo, zero outside the image, so a tap is
//     a constant offset.
//   * An MFMA lane needs 8 consecutive pixels of one channel: two LDS
//     transpose loads (ds_read_b64_tr_b16), each over 4 pixels x 16 channels,
//     at any pixel offset, so no shifted copies.
//   * The staging waves of the first column tile's blocks add up the dy values
//     they load: the bias gradient.
//
// Measured (us, batch 128, the fp32-MFMA kernel before): 32x32 64 -> 64 channels
// 97 -> 59, 16x16 128 channels 92 -> 54, 8x8 256 channels 87 -> 56, 4x4 512
// channels 68 -> 53; 27x45, 75 -> 107 channels, batch 19: 79 -> 53.  With 4-byte
// staging loads, 48 a lane and tile, the loads bound it (95 us at 16x16).  The
// check for lost bits, one instruction in twelve of the split, costs large layers
// of few output channels 4 to 6 % (128 images of 16x16, 512 -> 32: 93 -> 98).
//
// The pixels are split over blocks when the output tiles do not fill the 256
// CUs; each split writes its sums to the workspace and they are added in split
// order.  No atomics: repeated calls give the same bits.
#include "split_bf16.hpp"

#include <algorithm>
#include <cstdio>
#include <mutex>
#include <type_traits>

namespace sb {

struct WsArgs {
  const float* x;        // [N][C][H][W]
  const float* dy;       // [N][K][H][W]
  float* dw;             // [K][C][3][3]
  float* db;             // [K] or null
  float* part;           // split partials: [splits][K*C*9 + K] (dw, then db)
  int N, C, H, W, K;
  int tiles_w, tiles_h, ptiles, tiles_per_split, c_tiles, splits;
};

template <int TH_, int TW_, int IMGS_>
struct WsTile {
  static constexpr int TH = TH_, TW = TW_, IMGS = IMGS_, BP = IMGS * TH * TW;
  static_assert(BP == 128 && TW % 4 == 0, "128 pixels, groups of 4 within a row");
  static constexpr int BK = 64, BC = 16;
  static constexpr int HH = TH + 2, HW = TW + 2, PLANE = IMGS * HH * HW;
  // Pixels per 8-channel plane in LDS: 4 modulo 16 (64 bytes), so the two
  // planes of a transpose load lie in different banks.
  static constexpr int DPL = BP + 4, XPL = (PLANE + 15) / 16 * 16 + 4;
  static constexpr int DPART = 8 * DPL * 8, XPART = 2 * XPL * 8;     // bf16
  static constexpr int LDS_DY = 3 * DPART, BUF = LDS_DY + 3 * XPART;
  // Staging tasks of 8 channels: dy quads of 4 pixels (one per staging lane),
  // x quads of 4 interior halo columns, single pixels of the two edge columns.
  static_assert(BK / 8 * BP / 4 == 256, "a dy quad per lane");
  static constexpr int XQ = 2 * IMGS * HH * (TW / 4), XE = 2 * IMGS * HH * 2;
  static_assert(XQ <= 256 && XE <= 256, "at most one of each per lane");
  // Block output in LDS: 4 copies of 64 rows of 16 c x 9 taps, then db.
  static constexpr int RP = BC * 9 + 4, COPY = BK * RP;
  static constexpr size_t LDS_STAGE = 2 * (size_t)BUF * sizeof(u16);
  static constexpr size_t LDS_OUT = (4 * COPY + 64) * sizeof(float);
  static constexpr size_t LDS_REDO = LDS_STAGE > LDS_OUT ? LDS_STAGE : LDS_OUT;
  static constexpr size_t LDS_BYTES = LDS_REDO + 16;   // behind them the redo flag
  static_assert(LDS_BYTES <= 160 * 1024, "one block per CU");
  __host__ __device__ static constexpr int hp(int p) {   // halo pixel of tile pixel p at tap (0, 0)
    return (p / (TH * TW) * HH + p / TW % TH) * HW + p % TW;
  }
};

typedef short v4s __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4s lds_v4s;

__device__ __forceinline__ s8 tr8(const u16* lo, const u16* hi) {
  const v4s a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)lo);
  const v4s b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)hi);
  return s8{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
}

// The block's output on the fp32 MFMA, over the pixel tiles [pt0, pt1), for
// blocks that the split cannot carry: operands straight from memory, a pixel
// taking part in a tap only where both are inside the image.  Wave w has 16 k
// (w % 4) and every second tile; a lane has 4 consecutive pixels of a row and
// the 3 x 6 window of x around them.  Writes copies 0 and 2 of E, which are
// added, and zeros to the others.
template <class T>
__device__ __forceinline__ void wgrad_tile_f32(const WsArgs& a, float* E, int k0, int c0, int pt0,
                                               int pt1, int wave, int lane) {
  const int lr = lane & 15, lq = lane >> 4;
  const int k = k0 + (wave & 3) * 16 + lr, c = c0 + lr;
  const int HWs = a.H * a.W;
  f4 acc[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int pt = pt0 + (wave >> 2); pt < pt1; pt += 2) {
    const int tx = pt % a.tiles_w, ty = pt / a.tiles_w % a.tiles_h, tn = pt / a.tiles_w / a.tiles_h;
#pragma unroll 2
    for (int q = 0; q < T::BP; q += 16) {
      const int p = q + lq * 4;
      const int n = tn * T::IMGS + p / (T::TH * T::TW);
      const int h = ty * T::TH + p / T::TW % T::TH, w = tx * T::TW + p % T::TW;
      const bool in = n < a.N && h < a.H;
      const float* dp = a.dy + ((size_t)n * a.K + k) * HWs + h * a.W + w;
      const float* xp = a.x + ((size_t)n * a.C + c) * HWs + h * a.W + w;
      float d[4], x[3][6];
#pragma unroll
      for (int e = 0; e < 4; ++e) d[e] = in && w + e < a.W && k < a.K ? dp[e] : 0.f;
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int e = 0; e < 6; ++e)
          x[r][e] = in && c < a.C && (unsigned)(h + r - 1) < (unsigned)a.H &&
                            (unsigned)(w + e - 1) < (unsigned)a.W
                        ? xp[(r - 1) * a.W + e - 1] : 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int t = 0; t < 9; ++t) {
          const bool ok = in && w + e < a.W && (unsigned)(h + t / 3 - 1) < (unsigned)a.H &&
                          (unsigned)(w + e + t % 3 - 1) < (unsigned)a.W;
          acc[t] = mfma16x16x4(ok ? d[e] : 0.f, ok ? x[t / 3][e + t % 3] : 0.f, acc[t]);
        }
    }
  }
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      float* e = E + (wave >> 2) * 2 * T::COPY + ((wave & 3) * 16 + 4 * lq + v) * T::RP + lr * 9 + t;
      e[0] = acc[t][v];
      e[T::COPY] = 0.f;
    }
}

// VEC: rows are whole aligned quads (W a multiple of 4, 16-byte tensors), so a
// quad of one channel is one 16-byte load.
// The work of block b of the layer `a`; the kernels below pick both.
template <class T, bool VEC>
__device__ __forceinline__ void wgrad_split_block(const WsArgs& a, int b) {
  extern __shared__ u16 ldsu[];
  float* E = reinterpret_cast<float*>(ldsu);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int k_tiles = cdiv(a.K, T::BK);
  const int ct = b % a.c_tiles, kt = b / a.c_tiles % k_tiles, split = b / (a.c_tiles * k_tiles);
  const int c0 = ct * T::BC, k0 = kt * T::BK;
  const int pt0 = split * a.tiles_per_split, pt1 = min(a.ptiles, pt0 + a.tiles_per_split);
  const int nt = pt1 - pt0;
  const bool do_db = a.db != nullptr && ct == 0;
  const int HWs = a.H * a.W;
  const size_t wsz = (size_t)a.K * a.C * 9;
  int* redo = reinterpret_cast<int*>(ldsu + T::LDS_REDO / sizeof(u16));
  if (tid == 0) *redo = 0;

  if (wave >= 4) {
    // ---- staging waves ----
    const int ptid = tid - 256;
    // dy quad: 8 channels doct = ptid / 32, tile pixels 4 (ptid % 32) .. +3.
    const int doct = ptid >> 5, dp = (ptid & 31) * 4;
    const int dimg = dp / (T::TH * T::TW), dyy = dp / T::TW % T::TH, dxx = dp % T::TW;
    const int d_rel = (dimg * a.K + k0 + doct * 8) * HWs + dyy * a.W + dxx;
    const int d_lds = (doct * T::DPL + dp) * 8;
    const uint32_t dneg = dp & 32 ? 0x80000000u : 0u;      // odd waves' pixels: negated
    // x quad: lanes from 0 up; x edge pixel: lanes from 255 down.
    const int qrow = ptid % (T::IMGS * T::HH * (T::TW / 4)) / (T::TW / 4);
    const int qoct = ptid / (T::IMGS * T::HH * (T::TW / 4));
    const int qx = ptid % (T::TW / 4) * 4, qimg = qrow / T::HH, qy = qrow % T::HH - 1;
    const bool q_on = ptid < T::XQ;
    const int q_rel = (qimg * a.C + c0 + qoct * 8) * HWs + qy * a.W + qx;
    const int q_lds = T::LDS_DY + (qoct * T::XPL + qrow * T::HW + qx + 1) * 8;
    const int et = 255 - ptid, erow = et / 2 % (T::IMGS * T::HH);
    const int eoct = et / (2 * T::IMGS * T::HH), ex = et % 2 ? T::TW : -1;
    const int eimg = erow / T::HH, ey = erow % T::HH - 1;
    const bool e_on = et < T::XE;
    const int e_rel = (eimg * a.C + c0 + eoct * 8) * HWs + ey * a.W + ex;
    const int e_lds = T::LDS_DY + (eoct * T::XPL + erow * T::HW + ex + 1) * 8;
    const int dch = min(8, a.K - k0 - doct * 8);           // live channels of each task
    const int qch = min(8, a.C - c0 - qoct * 8), ech = min(8, a.C - c0 - eoct * 8);
    f4 rd[8], rq[8];
    uint32_t lost = 0;
    f8v re, dbs = f8v{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // Quad of channel j at byte offset off (+ j planes): its first `cols`
    // columns are in the image (all or none if VEC).
    auto quad = [&](rsrc_t r, uint32_t off, int cols, int j) {
      const int so = j * HWs * 4;
      if constexpr (VEC) {
        return __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(
                                          r, (int)(cols > 0 ? off : kOOB), so, 0));
      } else {
        f4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          v[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                               r, (int)(e < cols ? off + 4 * e : kOOB), so, 0));
        return v;
      }
    };
    auto gload = [&](int t) {
      const int pt = pt0 + t;
      const int tx = pt % a.tiles_w, q = pt / a.tiles_w, ty = q % a.tiles_h, tn = q / a.tiles_h;
      const int n0 = tn * T::IMGS, h0 = ty * T::TH, w0 = tx * T::TW, cnt = min(T::IMGS, a.N - n0);
      const rsrc_t dr = make_rsrc(a.dy + (size_t)n0 * a.K * HWs, (uint32_t)(cnt * a.K * HWs) * 4u);
      const rsrc_t xr = make_rsrc(a.x + (size_t)n0 * a.C * HWs, (uint32_t)(cnt * a.C * HWs) * 4u);
      const int base = h0 * a.W + w0;
      const int dcol = dimg < cnt && h0 + dyy < a.H ? a.W - w0 - dxx : 0;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        rd[j] = quad(dr, (uint32_t)(d_rel + base) * 4u, j < dch ? dcol : 0, j);
      const int qcol = q_on && qimg < cnt && (unsigned)(h0 + qy) < (unsigned)a.H ? a.W - w0 - qx : 0;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        rq[j] = quad(xr, (uint32_t)(q_rel + base) * 4u, j < qch ? qcol : 0, j);
      const bool eok = e_on && eimg < cnt && (unsigned)(h0 + ey) < (unsigned)a.H &&
                       (unsigned)(w0 + ex) < (unsigned)a.W;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        re[j] = __builtin_bit_cast(
            float, __builtin_amdgcn_raw_buffer_load_b32(
                       xr, (int)(eok && j < ech ? (uint32_t)(e_rel + base) * 4u : kOOB),
                       j * HWs * 4, 0));
    };
    auto neg = [&](float v) { return __uint_as_float(__float_as_uint(v) ^ dneg); };
    auto put = [&](u16* at, int part, f8v v) {
      const Split8 s = split8(v, lost);
#pragma unroll
      for (int p = 0; p < 3; ++p) *reinterpret_cast<s8*>(at + p * part) = s.p[p];
      __builtin_amdgcn_sched_barrier(0);           // one pixel's parts in registers at a time
    };
    auto lstore = [&](int buf) {
      u16* B = ldsu + buf * T::BUF;
      if (do_db) {
#pragma unroll
        for (int j = 0; j < 8; ++j) dbs[j] += (rd[j][0] + rd[j][1]) + (rd[j][2] + rd[j][3]);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
        put(B + d_lds + e * 8, T::DPART, f8v{neg(rd[0][e]), neg(rd[1][e]), neg(rd[2][e]),
                                             neg(rd[3][e]), neg(rd[4][e]), neg(rd[5][e]),
                                             neg(rd[6][e]), neg(rd[7][e])});
      if (q_on) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          put(B + q_lds + e * 8, T::XPART, f8v{rq[0][e], rq[1][e], rq[2][e], rq[3][e],
                                               rq[4][e], rq[5][e], rq[6][e], rq[7][e]});
      }
      if (e_on) put(B + e_lds, T::XPART, re);
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
    if (do_db) {
      // The 32 lanes of a channel group hold its pixels.
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        float v = dbs[j];
#pragma unroll
        for (int m = 16; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
        if ((lane & 31) == 0) E[4 * T::COPY + doct * 8 + j] = v;
      }
    }
  } else {
    // ---- multiplying waves: pixels wave*32 .. +31 of the tile ----
    const int lr = lane & 15, lq = lane >> 4;
    // Transpose loads: lane s of a 16-lane group points at channels 4 (s % 4)
    // .. +3 of the group's pixel s / 4 (second load: of pixel 4 + s / 4).
    const int ca = lr & 3, pj = wave * 32 + lq * 8 + (lr >> 2);
    const int d_off = ((ca >> 1) * T::DPL + pj) * 8 + (ca & 1) * 4;
    const int x_lo = ((ca >> 1) * T::XPL + T::hp(pj)) * 8 + (ca & 1) * 4;
    const int x_hi = ((ca >> 1) * T::XPL + T::hp(pj + 4)) * 8 + (ca & 1) * 4;
    f4 acc[4][9], cp[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      cp[i] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < 9; ++t) acc[i][t] = f4{0.f, 0.f, 0.f, 0.f};
    }
    s8 fa[4][3], fb[2][3];
    __syncthreads();
    for (int t = 0; t < nt; ++t) {
      const u16* D = ldsu + (t & 1) * T::BUF;
      const u16* X = D + T::LDS_DY;
      auto rd_b = [&](int tap, int s) {
        const int off = (tap / 3 * T::HW + tap % 3) * 8;
#pragma unroll
        for (int p = 0; p < 3; ++p)
          fb[s][p] = tr8(X + p * T::XPART + x_lo + off, X + p * T::XPART + x_hi + off);
      };
      rd_b(0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          const u16* q = D + p * T::DPART + 2 * i * T::DPL * 8 + d_off;
          fa[i][p] = tr8(q, q + 4 * 8);
        }
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) {
        if (tap < 8) rd_b(tap + 1, (tap + 1) & 1);
        __builtin_amdgcn_sched_barrier(0);         // keep those reads ahead of the MFMAs
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          f4 c = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int m = 0; m < 6; ++m)
            c = mfma16x16x32(fa[i][kSplitA[m]], fb[tap & 1][kSplitB[m]], c);
          acc[i][(tap + 8) % 9] += cp[i];          // the tap before
          cp[i] = c;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i][8] += cp[i];
    if (split_suspect(acc)) *redo = 1;
    // acc[i][t] element v: row i*16 + 4*lq + v, channel lr, tap t.
    float* R = E + wave * T::COPY;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) R[(i * 16 + 4 * lq + v) * T::RP + lr * 9 + t] = acc[i][t][v];
  }
  __syncthreads();
  if (__builtin_expect(__builtin_amdgcn_readfirstlane(*redo), 0)) {
    wgrad_tile_f32<T>(a, E, k0, c0, pt0, pt1, wave, lane);
    __syncthreads();
  }

  // ---- the block's 64 k x (16 c x 9 taps), rows contiguous in dw ----
  float* dst = a.splits == 1 ? a.dw : a.part + (size_t)split * (wsz + a.K);
  constexpr int QPR = T::BC * 9 / 4;
  const int cw = min(T::BC, a.C - c0) * 9;           // live columns
  const bool vec = (a.C * 9) % 4 == 0 && cw % 4 == 0 &&
                   (((uintptr_t)dst + (size_t)c0 * 9 * sizeof(float)) & 15) == 0;
#pragma unroll 1
  for (int q = tid; q < T::BK * QPR; q += 512) {
    const int row = q / QPR, col = (q % QPR) * 4, k = k0 + row;
    if (k >= a.K || col >= cw) continue;
    f4 v = *reinterpret_cast<const f4*>(E + row * T::RP + col);
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const f4 u = *reinterpret_cast<const f4*>(E + w * T::COPY + row * T::RP + col);
      if (w & 1) v -= u;
      else v += u;
    }
    float* o = dst + (size_t)k * a.C * 9 + (size_t)c0 * 9 + col;
    if (vec) {
      *reinterpret_cast<f4*>(o) = v;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (col + e < cw) o[e] = v[e];
    }
  }
  if (do_db && tid < T::BK && k0 + tid < a.K)
    (a.splits == 1 ? a.db : dst + wsz)[k0 + tid] = E[4 * T::COPY + tid];
}

// Blocks in (split, k tile, c tile) order, dealt to the 8 XCDs in contiguous
// ranges: the blocks of a split read the same pixel tiles through one L2.
__device__ __forceinline__ int ws_deal(int b, int nb) {
  return nb % 8 == 0 ? (b % 8) * (nb / 8) + b / 8 : b;
}

template <class T, bool VEC>
__global__ __launch_bounds__(512, 2) void conv3x3_wgrad_split(WsArgs a) {
  wgrad_split_block<T, VEC>(a, ws_deal(blockIdx.x, gridDim.x));
}

// Weight gradients of up to kWsMany layers that take the same kernel, in one
// launch: layer i owns the blocks first[i] .. first[i+1]-1 and numbers them as
// its own grid would be.  A layer's grid is about one block per CU, so the
// next layer's blocks start on the CUs that finish first instead of after the
// last block and a launch.
constexpr int kWsMany = 4;
struct WsMany {
  WsArgs a[kWsMany];
  int first[kWsMany + 1];
  int n;
};

template <class T, bool VEC>
__global__ __launch_bounds__(512, 2) void conv3x3_wgrad_split_many(WsMany m) {
  const int blk = blockIdx.x;
  int i = 0;
  while (i + 1 < m.n && blk >= m.first[i + 1]) ++i;
  const int nb = m.first[i + 1] - m.first[i], b = blk - m.first[i];
  wgrad_split_block<T, VEC>(m.a[i], m.first[i] % 8 == 0 ? ws_deal(b, nb) : b);
}

// ---------------------------------------------------------------- host --
struct WsPlan {
  int tile, imgs, tiles_w, tiles_h, ptiles, k_tiles, c_tiles, tps, splits;
  size_t ws_bytes;
};

using Ws16 = WsTile<8, 16, 1>;
using Ws8 = WsTile<8, 8, 2>;
using Ws4 = WsTile<4, 4, 8>;
struct WsTileInfo { int th, tw, imgs; const char* name; };
static const WsTileInfo kWsTiles[] = {{8, 16, 1, "8, 16, 1"}, {8, 8, 2, "8, 8, 2"},
                                      {4, 4, 8, "4, 4, 8"}};

// The tile that pads the images least (the larger one if equal: less halo),
// then the split with the least estimated time: a block per CU takes about 5 us
// for its first tile and its output and 1.8 us a tile; split partials cost
// their traffic and a launch.  Partials stay within the scratch array of
// sb_conv3x3_bwd_weight_noalloc, so that call takes every shape this kernel does.
static WsPlan ws_plan(int N, int C, int H, int W, int K) {
  WsPlan p{};
  long least = 0;
  for (int i = 0; i < 3; ++i) {
    const WsTileInfo& t = kWsTiles[i];
    const long n = (long)cdiv(W, t.tw) * cdiv(H, t.th) * cdiv(N, t.imgs);
    // A tile's images have to stay below 2^31 bytes.
    if (i > 0 && (int64_t)std::min(t.imgs, N) * std::max(C, K) * H * W * 4 >= (1ll << 31)) continue;
    if (i == 0 || n < least) {
      least = n;
      p.tile = i;
      p.imgs = t.imgs;
      p.tiles_w = cdiv(W, t.tw);
      p.tiles_h = cdiv(H, t.th);
    }
  }
  p.ptiles = (int)least;
  p.k_tiles = cdiv(K, 64);
  p.c_tiles = cdiv(C, 16);
  const long blocks = (long)p.k_tiles * p.c_tiles;
  double best = 0;
  const double dw_mb = (double)K * C * 36e-6;
  for (int s = 1; s <= 256 && s <= p.ptiles; ++s) {
    const int tps = cdiv(p.ptiles, s);
    if (cdiv(p.ptiles, tps) != s) continue;
    if (s > 1 && (size_t)s * ((size_t)K * C * 9 + K) * sizeof(float) > SB_NOALLOC_SCRATCH_BYTES)
      break;
    const double est = (double)cdiv((int)std::min<long>(blocks * s, 1l << 30), 256) *
                           (5.0 + 1.8 * tps) +
                       (s > 1 ? 1.5 + dw_mb * (2 * s + 1) / 4.0 : 0.0);
    if (best == 0 || est < best) {
      best = est;
      p.tps = tps;
      p.splits = s;
    }
  }
  p.ws_bytes = p.splits > 1 ? (size_t)p.splits * ((size_t)K * C * 9 + K) * sizeof(float) : 0;
  return p;
}

template <class T, bool VEC>
static void ws_launch(const WsPlan& p, const WsArgs& a, hipStream_t st) {
  static std::once_flag once;
  std::call_once(once, [] {
    (void)hipFuncSetAttribute((const void*)conv3x3_wgrad_split<T, VEC>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)T::LDS_BYTES);
  });
  conv3x3_wgrad_split<T, VEC>
      <<<(unsigned)(p.k_tiles * p.c_tiles * p.splits), 512, T::LDS_BYTES, st>>>(a);
}
static bool ws_vec(int W, const void* x, const void* dy) {
  return W % 4 == 0 && (((uintptr_t)x | (uintptr_t)dy) & 15) == 0;
}
template <class T>
static void ws_launch(const WsPlan& p, const WsArgs& a, hipStream_t st) {
  if (ws_vec(a.W, a.x, a.dy)) ws_launch<T, true>(p, a, st);
  else ws_launch<T, false>(p, a, st);
}

template <class T, bool VEC>
static void ws_launch_many(const WsMany& m, hipStream_t st) {
  static std::once_flag once;
  std::call_once(once, [] {
    (void)hipFuncSetAttribute((const void*)conv3x3_wgrad_split_many<T, VEC>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)T::LDS_BYTES);
  });
  conv3x3_wgrad_split_many<T, VEC><<<(unsigned)m.first[m.n], 512, T::LDS_BYTES, st>>>(m);
}

static WsArgs ws_args(const WsPlan& p, int N, int C, int H, int W, int K, const void* x,
                      const void* dy, float* dw, float* db, void* ws) {
  WsArgs a{};
  a.x = (const float*)x; a.dy = (const float*)dy; a.dw = dw; a.db = db;
  a.part = p.splits > 1 ? (float*)ws : nullptr;
  a.N = N; a.C = C; a.H = H; a.W = W; a.K = K;
  a.tiles_w = p.tiles_w; a.tiles_h = p.tiles_h; a.ptiles = p.ptiles;
  a.tiles_per_split = p.tps; a.c_tiles = p.c_tiles; a.splits = p.splits;
  return a;
}

}  // namespace sb

namespace sbh {

void conv_wgrad_reduce(const float* part, int splits, int K, int C, float* dw, float* db,
                       hipStream_t st);

// Whether an fp32 weight gradient runs here: at least 8 input channels (the
// narrow kernels flatten fewer), images at least 4 wide, 4x4 ones at least 8 (a
// tile), and enough work, which is counted as the fp32 MFMA would do it: u =
// padded pixels (tiles of 2x32, 4x16, 8x8, or 4 images of 4x4) x 64-channel tiles x
// 16-channel tiles.  From 1.65e7 on, from 1.5e7 on narrow images: of 678 layers
// of 3e5 to 2e8 products 9 are then slower than on the fp32 MFMA, by 17 % at most
// (55 images of 36x36, 32 -> 64: 61 us, 72), where a line at 7e6 products or none had 70
// (12 images of 8x8, 72 -> 24: u = 3.9e6, 9.5 us on the fp32 MFMA, 11.9 here; 5 of
// 28x36, 64 -> 16: 2.3e7, 20.7 and 12.9; 4 of 4x4, 512 -> 512: 7.0 and 11.3).  The
// fp32 MFMA's 4x4 kernel wastes less on few channels, so 4x4 images also need
// 1.4e7 products (128 of them, 128 -> 24, 6.3e6: 9.5 and 12.6).
bool conv_wgrad_split_takes(int N, int C, int H, int W, int K) {
  using sb::cdiv;
  if (C < 8 || W < 4 || (W == 4 && H == 4 && N < 8)) return false;
  long tiles;
  if (W >= 32) tiles = (long)N * cdiv(W, 32) * cdiv(H, 2);
  else if (W >= 16) tiles = (long)N * cdiv(W, 16) * cdiv(H, 4);
  else if (W >= 8) tiles = (long)N * cdiv(W, 8) * cdiv(H, 8);
  else tiles = (long)cdiv(N, 4) * cdiv(W, 4) * cdiv(H, 4);
  const double u = (double)tiles * 64 * (cdiv(K, 64) * 64.0) * (cdiv(C, 16) * 16.0);
  return u >= (W < 8 ? 1.5e7 : 1.65e7) && (H != 4 || W != 4 || 16.0 * N * C * K >= 1.4e7);
}

size_t conv_wgrad_split_ws(int N, int C, int H, int W, int K) {
  return sb::ws_plan(N, C, H, W, K).ws_bytes;
}

int conv_wgrad_split_describe(int N, int C, int H, int W, int K, char* buf, size_t len) {
  const sb::WsPlan p = sb::ws_plan(N, C, H, W, K);
  return snprintf(buf, len, "sb::conv3x3_wgrad_split<sb::WsTile<%s>, %s> grid=%dx1x%d",
                  sb::kWsTiles[p.tile].name, W % 4 == 0 ? "true" : "false", p.k_tiles * p.c_tiles, p.splits);
}

sb_status conv_wgrad_split(int N, int C, int H, int W, int K, const void* x, const void* dy,
                           float* dw, float* db, void* ws, size_t ws_bytes, hipStream_t st) {
  const sb::WsPlan p = sb::ws_plan(N, C, H, W, K);
  // Buffer ranges: one tile's images of x and of dy.
  if ((int64_t)std::min(p.imgs, N) * std::max(C, K) * H * W * 4 >= (1ll << 31))
    return SB_ERR_UNSUPPORTED;
  if (p.ws_bytes > 0 && (ws == nullptr || ws_bytes < p.ws_bytes)) return SB_ERR_WORKSPACE;
  const sb::WsArgs a = sb::ws_args(p, N, C, H, W, K, x, dy, dw, db, ws);
  switch (p.tile) {
    case 0: sb::ws_launch<sb::Ws16>(p, a, st); break;
    case 1: sb::ws_launch<sb::Ws8>(p, a, st); break;
    default: sb::ws_launch<sb::Ws4>(p, a, st); break;
  }
  if (p.splits > 1) conv_wgrad_reduce(a.part, p.splits, K, C, dw, db, st);
  return launch_status();
}

// Batch key (0..5) of a layer that runs here: layers on the same instantiation
// of the kernel above share a key; -1 for a layer that the kernel refuses.
int conv_wgrad_split_key(int N, int C, int H, int W, int K, const void* x, const void* dy) {
  const sb::WsPlan p = sb::ws_plan(N, C, H, W, K);
  if ((int64_t)std::min(p.imgs, N) * std::max(C, K) * H * W * 4 >= (1ll << 31)) return -1;
  return p.tile * 2 + (sb::ws_vec(W, x, dy) ? 1 : 0);
}

// n (1..4) layers with one batch key on one launch: the same partials,
// reductions and results as n single calls.  shape[i] = {N, C, H, W, K};
// ws[i] / ws_bytes[i]: layer i's own workspace region.
sb_status conv_wgrad_split_group(int n, const int (*shape)[5], const void* const* x,
                                 const void* const* dy, float* const* dw, float* const* db,
                                 void* const* ws, const size_t* ws_bytes, hipStream_t st) {
  if (n < 1 || n > sb::kWsMany) return SB_ERR_INVALID_ARG;
  sb::WsPlan p[sb::kWsMany];
  sb::WsMany m{};
  m.n = n;
  int key = -1, total = 0;
  for (int i = 0; i < n; ++i) {
    const int N = shape[i][0], C = shape[i][1], H = shape[i][2], W = shape[i][3],
              K = shape[i][4];
    if (!conv_wgrad_split_takes(N, C, H, W, K)) return SB_ERR_INVALID_ARG;
    const int k = conv_wgrad_split_key(N, C, H, W, K, x[i], dy[i]);
    if (k < 0 || (i > 0 && k != key)) return SB_ERR_INVALID_ARG;
    key = k;
    p[i] = sb::ws_plan(N, C, H, W, K);
    if (p[i].ws_bytes > 0 && (ws[i] == nullptr || ws_bytes[i] < p[i].ws_bytes))
      return SB_ERR_WORKSPACE;
    m.a[i] = sb::ws_args(p[i], N, C, H, W, K, x[i], dy[i], dw[i], db ? db[i] : nullptr, ws[i]);
    m.first[i] = total;
    total += p[i].k_tiles * p[i].c_tiles * p[i].splits;
  }
  for (int i = n; i <= sb::kWsMany; ++i) m.first[i] = total;
  switch (key) {
    case 0: sb::ws_launch_many<sb::Ws16, false>(m, st); break;
    case 1: sb::ws_launch_many<sb::Ws16, true>(m, st); break;
    case 2: sb::ws_launch_many<sb::Ws8, false>(m, st); break;
    case 3: sb::ws_launch_many<sb::Ws8, true>(m, st); break;
    case 4: sb::ws_launch_many<sb::Ws4, false>(m, st); break;
    default: sb::ws_launch_many<sb::Ws4, true>(m, st); break;
  }
  for (int i = 0; i < n; ++i)
    if (p[i].splits > 1)
      conv_wgrad_reduce(m.a[i].part, p[i].splits, m.a[i].K, m.a[i].C, m.a[i].dw, m.a[i].db, st);
  return launch_status();
}

}  // namespace sbh
