// fc.hip -- FC column shard forward and backward (sec. 3.1: a LINEAR layer
// split to 1/K of its outputs, run on the batch the modulo layer gathers;
// its backward yields this shard's partial gradient over the full input).
//
//   forward   Y   = X * W_sh (+ b) (ReLU)       [m x ns] = [m x kin][kin x ns]
//   backward  dXp = G * W_sh^T                  [m x kin]
//             dW  = (dW +) X^T * G              [kin x ns]
//             db  = (db +) column sums of G     [ns]
// with G = dY, or dY * [mask > 0] (ReLU of this shard's output).
//
// One GEMM kernel on the bf16 MFMA (gemm_split below) serves the three
// products.  fp32 operands are split in three bf16 parts (split_bf16.hpp, six
// MFMAs per product); bf16 operands are their own first part, so their products
// are exact with one MFMA, and y and dx_partial are rounded to nearest-even on
// store.  Sums, dW and db are fp32.  The backward's bias gradient is added up
// inside the dW product.  Tile shapes and reduction splits are chosen per shape
// (gemm_plan).
#include "split_bf16.hpp"

#include <algorithm>
#include <type_traits>
#include <mutex>

namespace sb {

// ---------------------------------------------------------------------------
// GEMM core.  C = epi(A * B) with A [M x K], B [K x N].  Blocks of 512 threads,
// one or two a CU: four waves stage, four multiply (2 x 2, each BM/2 x BN/2
// as 16 x 16 blocks of the 16x16x32 MFMA).
//
// A stage is 8*KO of the reduction, kept in LDS as [part][k / 8][row][k % 8] for
// both operands whatever their layout in memory, so an MFMA operand is one
// 16-byte read per lane.  A staging lane makes two 16-byte pieces (8 k of a row)
// of each operand per stage, or two of one operand (64 x 64 tiles of 32 k: two
// waves stage A, two B):
//   * contiguous along k ("K-contiguous"): two pieces of 8 consecutive elements;
//   * contiguous along its rows: 8 k of two adjacent rows, transposed in
//     registers.
// The ReLU mask of dY is applied there.  Out-of-range offsets read 0 (raw buffer
// loads), so ragged edges need no branches.  Three stages are in LDS: while
// stage t is multiplied, t + 2 is stored and t + 3 loaded, and t + 1 is already
// readable, so the operands of the next 32 k are in registers before a stage
// ends: with two stages each of these short rounds (1536 matrix cycles) would
// start by waiting for LDS.
//
// A long reduction over few output tiles is split over `splits` ranges of k;
// each split writes fp32 partials [split][M][N] and gemm_splitk_epilogue sums
// them in a fixed order.  Blocks are numbered split-major and dealt to the 8
// XCDs in contiguous ranges of that order, so the blocks one XCD runs share
// operand slices in its L2.
//
// colsum (the FC bias gradient): the staging waves of the first row tile's
// blocks add up the B values they stage.
//
// A tile leaves through LDS; a thread's pieces share their columns, so the bias
// is loaded once and several pieces are under way at a time (one by one, each
// waiting for its bias, they cost 1024 x 2048 outputs of 128 k 3 us of 16.6).
//
// Measured (512 x 4096 x 1024 fp32 shard, forward and backward): 132 us with
// the fp32 MFMA kernels before, 104 like this; the staging waves' loads and
// vector ALU bound it (dW product 34 us: 25 without the loads, 30 without the
// splitting, 27 with one MFMA in six).
constexpr int kGThreads = 512, kGLocal = 4;

// LOC: bf16 products are summed inside the MFMA over kGLocal steps of 32 k and
// then added to the accumulators (split ones always are, after every step).
template <int BM_, int BN_, int KO_, int NP_, bool LOC_>
struct GemmTile {
  static constexpr int BM = BM_, BN = BN_, KO = KO_, NP = NP_;
  static constexpr bool LOC = LOC_;
  static constexpr int RB = BM / 32, CB = BN / 32;          // 16 x 16 blocks per wave
  static_assert(BM == BN && (BM * KO == 512 || BM * KO == 256), "two pieces per staging lane");
  // Staging lanes of an operand: all of them, or two waves for A and two for B.
  static constexpr int LANES = BM * KO / 2;
  // 8-k planes 4 rows apart modulo 16: the planes that neighbouring lanes write
  // start in different banks.
  static constexpr int APL = BM + 4, BPL = BN + 4;
  static constexpr int APART = KO * APL * 8, BPART = KO * BPL * 8;
  static constexpr int LDS_A = NP * APART, STAGE = LDS_A + NP * BPART;   // bf16
  static constexpr int EP = BN + 4;                         // output tile row pitch (floats)
  static constexpr size_t LDS_STAGES = 3 * (size_t)STAGE * sizeof(u16);
  static constexpr size_t LDS_OUT = ((size_t)BM * EP + BN * KO) * sizeof(float);
  static constexpr size_t LDS_REDO = LDS_STAGES > LDS_OUT ? LDS_STAGES : LDS_OUT;
  static constexpr size_t LDS_BYTES = LDS_REDO + 16;        // behind them the redo flag
  static_assert(LDS_BYTES <= 160 * 1024, "one block per CU");
};

struct GemmArgs {
  const void* a; int lda;              // A element (m,k): A_KC ? a[m*lda+k] : a[k*lda+m]
  const void* amask;                   // optional mask, same layout/stride as a
  const void* b; int ldb;              // B element (k,n): B_KC ? b[n*ldb+k] : b[k*ldb+n]
  const void* bmask;
  void* c; int ldc;                    // C[m*ldc + n] (type CE), or fp32 partials
  int M, N, K;
  int mt, nt, splits, k_per_split;
  const float* bias; int relu; int accumulate;
  float* colsum; int colsum_acc;       // column sums of B (k < K), or null
};

// One operand's staging: two pieces of 8 k per lane.  ROWS x 8*KO elements of
// an operand whose rows start at r0; [kb, ke) the block's range of k.
template <int ROWS, int KO, int PL, int PART, int NP, bool KC, bool VEC, class E, bool MASK>
struct GStage {
  f8v v[2], m[2];
  int row[2], oct[2];
  int ld, rows;
  __device__ __forceinline__ void init(int ld_, int rows_, int r0, int ptid) {
    ld = ld_;
    rows = rows_;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if (KC) {                                    // piece u: k octet fastest
        const int u = ptid + ROWS * KO / 2 * i;
        oct[i] = u % KO;
        row[i] = r0 + u / KO;
      } else {                                     // rows 2p, 2p + 1
        oct[i] = ptid / (ROWS / 2);
        row[i] = r0 + ptid % (ROWS / 2) * 2 + i;
      }
    }
  }
  __device__ __forceinline__ void load_one(rsrc_t r, int k0, int ke, f8v (&d)[2]) {
    if constexpr (KC) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int k = k0 + oct[i] * 8;
        const uint32_t off = (uint32_t)(row[i] * ld + k) * (uint32_t)sizeof(E);
        const bool ok = row[i] < rows;
        if constexpr (VEC) {                       // whole groups of 4
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const f4 t = BufLoad<E>::four(r, ok && k + 4 * q < ke ? off + 4 * q * sizeof(E) : kOOB);
#pragma unroll
            for (int e = 0; e < 4; ++e) d[i][4 * q + e] = t[e];
          }
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            d[i][e] = BufLoad<E>::one(r, ok && k + e < ke ? off + e * sizeof(E) : kOOB);
        }
      }
    } else {
      const int k = k0 + oct[0] * 8;
      const uint32_t off = (uint32_t)(k * ld + row[0]) * (uint32_t)sizeof(E);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t o = off + (uint32_t)(e * ld) * (uint32_t)sizeof(E);
        const bool ok = k + e < ke;
        if constexpr (VEC && sizeof(E) == 4) {     // both rows or neither
          typedef uint32_t u2 __attribute__((ext_vector_type(2)));
          const u2 t = __builtin_bit_cast(
              u2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)(ok && row[0] < rows ? o : kOOB), 0, 0));
          d[0][e] = __uint_as_float(t[0]);
          d[1][e] = __uint_as_float(t[1]);
        } else if constexpr (VEC) {
          const uint32_t t =
              __builtin_amdgcn_raw_buffer_load_b32(r, (int)(ok && row[0] < rows ? o : kOOB), 0, 0);
          d[0][e] = __uint_as_float(t << 16);
          d[1][e] = __uint_as_float(t & 0xffff0000u);
        } else {
          d[0][e] = BufLoad<E>::one(r, ok && row[0] < rows ? o : kOOB);
          d[1][e] = BufLoad<E>::one(r, ok && row[1] < rows ? o + (uint32_t)sizeof(E) : kOOB);
        }
      }
    }
  }
  __device__ __forceinline__ void load(rsrc_t r, rsrc_t rm, int k0, int ke) {
    load_one(r, k0, ke, v);
    if constexpr (MASK) load_one(rm, k0, ke, m);
  }
  // Stores the pieces; r0 as in init.  Leaves the (masked) values in v; lost as
  // in split_pair.
  __device__ __forceinline__ void store(u16* S, int r0, uint32_t& lost) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if constexpr (MASK) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[i][e] = m[i][e] > 0.f ? v[i][e] : 0.f;
      }
      u16* at = S + (oct[i] * PL + row[i] - r0) * 8;
      if constexpr (NP == 1) {                     // bf16 values: exact
        u32x4 h;
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = f32x2_to_bf16x2(v[i][2 * e], v[i][2 * e + 1]);
        *reinterpret_cast<s8*>(at) = __builtin_bit_cast(s8, h);
      } else {
        const Split8 s = split8(v[i], lost);
#pragma unroll
        for (int p = 0; p < 3; ++p) *reinterpret_cast<s8*>(at + p * PART) = s.p[p];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
};

// The block's (row tile, column tile, split) from its linear id: dealt to
// the 8 XCDs in contiguous ranges of the split-major order when the grid is
// a multiple of 8 blocks.
__device__ __forceinline__ void gemm_block(const GemmArgs& g, int& mtile, int& ntile, int& split) {
  const int nb = g.mt * g.nt * g.splits;
  int h = blockIdx.x;
  if (nb % 8 == 0) h = (h % 8) * (nb / 8) + h / 8;
  const int tiles = g.mt * g.nt;
  split = h / tiles;
  const int t = h - split * tiles;
  mtile = t / g.nt;
  ntile = t - mtile * g.nt;
}

// The block's output tile on the fp32 MFMA, over k in [k0, k1), for blocks
// that the split cannot carry: operands straight from memory.  A wave has 16
// rows and BM * BN / 2048 blocks of 16 columns.
template <class T, bool A_KC, bool B_KC, bool AMK, bool BMK>
__device__ __forceinline__ void gemm_tile_f32(const GemmArgs& g, float* O, int m0, int n0, int k0,
                                              int k1, int wave, int lane) {
  constexpr int RBT = T::BM / 16, NB = T::BM * T::BN / 2048;
  const int lr = lane & 15, lq = lane >> 4;
  const int rb = wave % RBT, cb = wave / RBT * NB, m = m0 + rb * 16 + lr;
  const float *A = (const float*)g.a, *B = (const float*)g.b;
  const float *MA = (const float*)g.amask, *MB = (const float*)g.bmask;
  f4 acc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) acc[j] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
  for (int kk = k0; kk < k1; kk += 4) {
    const int k = kk + lq;
    const size_t ao = A_KC ? (size_t)m * g.lda + k : (size_t)k * g.lda + m;
    const bool aok = m < g.M && k < k1 && (!AMK || MA[ao] > 0.f);
    const float av = aok ? A[ao] : 0.f;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int n = n0 + (cb + j) * 16 + lr;
      const size_t bo = B_KC ? (size_t)n * g.ldb + k : (size_t)k * g.ldb + n;
      const bool bok = n < g.N && k < k1 && (!BMK || MB[bo] > 0.f);
      acc[j] = mfma16x16x4(av, bok ? B[bo] : 0.f, acc[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) O[(rb * 16 + 4 * lq + v) * T::EP + (cb + j) * 16 + lr] = acc[j][v];
}

template <class T, bool A_KC, bool B_KC, bool VEC, class E, class CE, bool AMK, bool BMK>
__global__ __launch_bounds__(kGThreads, T::LANES == 256 ? 2 : 4) void gemm_split(GemmArgs g) {
  extern __shared__ u16 ldsu[];
  float* O = reinterpret_cast<float*>(ldsu);
  constexpr int KS = T::KO * 8;                    // k per stage
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int mtile, ntile, split;
  gemm_block(g, mtile, ntile, split);
  const int m0 = mtile * T::BM, n0 = ntile * T::BN;
  const int kb = split * g.k_per_split;
  const int ke = min(g.K, kb + g.k_per_split);
  const int nk = ke > kb ? cdiv(ke - kb, KS) : 0;
  const bool do_colsum = g.colsum != nullptr && mtile == 0;
  int* redo = reinterpret_cast<int*>(ldsu + T::LDS_REDO / sizeof(u16));
  if (tid == 0) *redo = 0;

  if (wave >= 4) {
    // ---- staging waves ----
    const int ptid = tid - 256;
    // Whole operand tensors (the host keeps them below 2^31 bytes).
    const size_t a_elems = A_KC ? (size_t)(g.M - 1) * g.lda + g.K : (size_t)(g.K - 1) * g.lda + g.M;
    const size_t b_elems = B_KC ? (size_t)(g.N - 1) * g.ldb + g.K : (size_t)(g.K - 1) * g.ldb + g.N;
    const rsrc_t ra = make_rsrc(g.a, (uint32_t)(a_elems * sizeof(E)));
    const rsrc_t rb = make_rsrc(g.b, (uint32_t)(b_elems * sizeof(E)));
    const rsrc_t ram = make_rsrc(AMK ? g.amask : g.a, (uint32_t)(a_elems * sizeof(E)));
    const rsrc_t rbm = make_rsrc(BMK ? g.bmask : g.b, (uint32_t)(b_elems * sizeof(E)));
    using StageA = GStage<T::BM, T::KO, T::APL, T::APART, T::NP, A_KC, VEC, E, AMK>;
    using StageB = GStage<T::BN, T::KO, T::BPL, T::BPART, T::NP, B_KC, VEC, E, BMK>;
    uint32_t lost = 0;
    float cs[2] = {0.f, 0.f};                      // column sums of this lane's two rows of B
    auto load_a = [&](StageA& q, int t) { q.load(ra, ram, kb + t * KS, ke); };
    auto load_b = [&](StageB& q, int t) { q.load(rb, rbm, kb + t * KS, ke); };
    auto store_a = [&](StageA& q, int t) { q.store(ldsu + t % 3 * T::STAGE, m0, lost); };
    auto store_b = [&](StageB& q, int t) {
      q.store(ldsu + t % 3 * T::STAGE + T::LDS_A, n0, lost);
      if (!B_KC && do_colsum) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
          cs[i] += ((q.v[i][0] + q.v[i][1]) + (q.v[i][2] + q.v[i][3])) +
                   ((q.v[i][4] + q.v[i][5]) + (q.v[i][6] + q.v[i][7]));
      }
    };
    // load0 / store0: the first stage through registers of its own, so that the
    // first two loads are in flight at once.  A stage past the end loads zeros.
    auto pipeline = [&](auto&& load0, auto&& store0, auto&& load, auto&& store) {
      if (nk > 1) {
        load0(0);
        load(1);
        store0(0);
        store(1);
      } else {
        load(0);
        store(0);
      }
      if (nk > 2) load(2);
      __syncthreads();
      for (int t = 0; t < nk; ++t) {
        if (t + 2 < nk) store(t + 2);
        if (t + 3 < nk) load(t + 3);
        __syncthreads();
      }
    };
    auto put_sums = [&](const StageB& q) {         // [octet][row] after the output tile
      if (!B_KC && do_colsum) {
#pragma unroll
        for (int i = 0; i < 2; ++i) O[T::BM * T::EP + q.oct[i] * T::BN + q.row[i] - n0] = cs[i];
      }
    };
    if constexpr (T::LANES == 256) {
      StageA a;
      StageB b;
      a.init(g.lda, g.M, m0, ptid);
      b.init(g.ldb, g.N, n0, ptid);
      StageA a0 = a;
      StageB b0 = b;
      pipeline([&](int t) { load_a(a0, t); load_b(b0, t); },
               [&](int t) { store_a(a0, t); store_b(b0, t); },
               [&](int t) { load_a(a, t); load_b(b, t); },
               [&](int t) { store_a(a, t); store_b(b, t); });
      put_sums(b);
    } else if (wave < 6) {
      StageA a;
      a.init(g.lda, g.M, m0, ptid);
      StageA a0 = a;
      pipeline([&](int t) { load_a(a0, t); }, [&](int t) { store_a(a0, t); },
               [&](int t) { load_a(a, t); }, [&](int t) { store_a(a, t); });
    } else {
      StageB b;
      b.init(g.ldb, g.N, n0, ptid - T::LANES);
      StageB b0 = b;
      pipeline([&](int t) { load_b(b0, t); }, [&](int t) { store_b(b0, t); },
               [&](int t) { load_b(b, t); }, [&](int t) { store_b(b, t); });
      put_sums(b);
    }
    if (T::NP == 3 && (lost & 0xffffu)) *redo = 1;
  } else {
    // ---- multiplying waves ----
    const int lr = lane & 15, lq = lane >> 4;
    const int wm = wave & 1, wn = wave >> 1;
    const int a_off = (lq * T::APL + wm * (T::BM / 2) + lr) * 8;
    const int b_off = T::LDS_A + (lq * T::BPL + wn * (T::BN / 2) + lr) * 8;
    f4 acc[T::RB][T::CB], cp[T::RB];
#pragma unroll
    for (int i = 0; i < T::RB; ++i) {
      cp[i] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < T::CB; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
    }
    constexpr int LI = T::LOC ? T::RB : 1, LJ = T::LOC ? T::CB : 1;
    f4 loc[LI][LJ];
#pragma unroll
    for (int i = 0; i < LI; ++i)
#pragma unroll
      for (int j = 0; j < LJ; ++j) loc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
    auto add_local = [&]() {
#pragma unroll
      for (int i = 0; i < LI; ++i)
#pragma unroll
        for (int j = 0; j < LJ; ++j) {
          acc[i][j] += loc[i][j];
          loc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
        }
    };
    s8 fa[2][T::RB][T::NP], fb[2][T::NP];
    auto rd_a = [&](const u16* S, int step, int s) {
#pragma unroll
      for (int i = 0; i < T::RB; ++i)
#pragma unroll
        for (int p = 0; p < T::NP; ++p)
          fa[s][i][p] = *reinterpret_cast<const s8*>(S + a_off + p * T::APART +
                                                     (step * 4 * T::APL + i * 16) * 8);
    };
    auto rd_b = [&](const u16* S, int step, int j, int s) {
#pragma unroll
      for (int p = 0; p < T::NP; ++p)
        fb[s][p] = *reinterpret_cast<const s8*>(S + b_off + p * T::BPART +
                                                (step * 4 * T::BPL + j * 16) * 8);
    };
    constexpr int STEPS = T::KO / 4;               // 32-k steps per stage
    static_assert(T::CB % 2 == 0, "column blocks alternate two register sets");
    // One 32-k step out of register set P, the next step's operands read
    // meanwhile (from S2 if it is in the next stage).
    auto step = [&](auto P, const u16* S, const u16* S2, int q, int q2) {
      constexpr int s = decltype(P)::value;
      rd_a(S2, q2, s ^ 1);
#pragma unroll
      for (int j = 0; j < T::CB; ++j) {
        if (j + 1 < T::CB) rd_b(S, q, j + 1, (j + 1) & 1);
        else rd_b(S2, q2, 0, 0);
        __builtin_amdgcn_sched_barrier(0);         // keep those reads ahead of the MFMAs
#pragma unroll
        for (int i = 0; i < T::RB; ++i) {
          if constexpr (T::LOC) {
            loc[i][j] = mfma16x16x32(fa[s][i][0], fb[j & 1][0], loc[i][j]);
          } else if constexpr (T::NP == 1) {
            acc[i][j] = mfma16x16x32(fa[s][i][0], fb[j & 1][0], acc[i][j]);
          } else {
            f4 c = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int m = 0; m < 6; ++m)
              c = mfma16x16x32(fa[s][i][kSplitA[m]], fb[j & 1][kSplitB[m]], c);
            acc[i][(j + T::CB - 1) % T::CB] += cp[i];   // the block before
            cp[i] = c;
          }
        }
        if constexpr (T::NP == 3) {
#pragma unroll
          for (int r = 0; r < 2 * T::RB; ++r) {
            __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    __syncthreads();
    rd_a(ldsu, 0, 0);
    rd_b(ldsu, 0, 0, 0);
    auto stage = [&](auto P, int t) {
      constexpr int s0 = decltype(P)::value;
      const u16* S = ldsu + t % 3 * T::STAGE;
      const u16* S2 = ldsu + (t + 1) % 3 * T::STAGE;   // past the end: stale, unused
      if constexpr (STEPS == 1) {
        step(std::integral_constant<int, s0>{}, S, S2, 0, 0);
      } else {
        static_assert(STEPS == 1 || STEPS == 2, "one or two steps per stage");
        step(std::integral_constant<int, s0>{}, S, S, 0, 1);
        step(std::integral_constant<int, s0 ^ 1>{}, S, S2, 1, 0);
      }
      if (T::LOC && (t + 1) % (kGLocal / STEPS) == 0) add_local();
      __syncthreads();
    };
    int t = 0;
    for (; t + 1 < nk; t += 2) {
      stage(std::integral_constant<int, 0>{}, t);
      stage(std::integral_constant<int, STEPS & 1>{}, t + 1);
    }
    if (t < nk) stage(std::integral_constant<int, 0>{}, t);
#pragma unroll
    for (int i = 0; i < T::RB; ++i) acc[i][T::CB - 1] += cp[i];
    if constexpr (T::LOC) add_local();
    if (T::NP == 3 && split_suspect(acc)) *redo = 1;
    // acc[i][j] element v: row wm*BM/2 + 16 i + 4 lq + v, column wn*BN/2 + 16 j + lr.
#pragma unroll
    for (int i = 0; i < T::RB; ++i)
#pragma unroll
      for (int j = 0; j < T::CB; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          O[(wm * (T::BM / 2) + 16 * i + 4 * lq + v) * T::EP + wn * (T::BN / 2) + 16 * j + lr] =
              acc[i][j][v];
  }
  __syncthreads();
  if constexpr (T::NP == 3) {                      // bf16 products are exact
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(*redo), 0)) {
      gemm_tile_f32<T, A_KC, B_KC, AMK, BMK>(g, O, m0, n0, kb, ke, wave, lane);
      __syncthreads();
    }
  }

  if (do_colsum && tid < T::BN && n0 + tid < g.N) {
    float s = 0.f;
#pragma unroll
    for (int o = 0; o < T::KO; ++o) s += O[T::BM * T::EP + o * T::BN + tid];
    float* cs = g.colsum + (g.splits > 1 ? (size_t)split * g.N : 0);   // this split's partials
    cs[n0 + tid] = g.colsum_acc ? cs[n0 + tid] + s : s;
  }
  const bool partial = g.splits > 1;
  float* part = partial ? (float*)g.c + (size_t)split * g.M * g.ldc : nullptr;
  CE* dst = (CE*)g.c;
  const bool vec4 = g.N % 4 == 0 && g.ldc % 4 == 0 &&
                    ((uintptr_t)(partial ? (void*)part : g.c) &
                     (partial ? 15 : 4 * sizeof(CE) - 1)) == 0;
  // A thread's quads share their columns.
  static_assert(kGThreads % (T::BN / 4) == 0, "one column quad per thread");
  const int c = tid % (T::BN / 4) * 4, n = n0 + c;
  if (n >= g.N) return;
  f4 bias = f4{0.f, 0.f, 0.f, 0.f};
  if (!partial && g.bias) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (n + e < g.N) bias[e] = g.bias[n + e];
  }
#pragma unroll 4
  for (int r = tid / (T::BN / 4); r < T::BM; r += kGThreads / (T::BN / 4)) {
    const int m = m0 + r;
    if (m >= g.M) break;
    f4 v = *reinterpret_cast<const f4*>(O + r * T::EP + c);
    const size_t o = (size_t)m * g.ldc + n;
    if (!partial) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] += bias[e];
        if (g.relu && !(v[e] > 0.f)) v[e] = 0.f;
      }
    }
    if (vec4) {
      if (partial) {
        *reinterpret_cast<f4*>(part + o) = v;
      } else {
        if (g.accumulate) v += Elem<CE>::load4(dst + o);
        Elem<CE>::store4(dst + o, v);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (n + e >= g.N) continue;
        if (partial) part[o + e] = v[e];
        else Elem<CE>::store(dst, o + e, g.accumulate ? v[e] + Elem<CE>::load(dst, o + e) : v[e]);
      }
    }
  }
}

// out[m, n] = epi(sum_s part[s][m][n]): + bias[n], ReLU, + out (accumulate),
// rounded to the output type CE.  Four consecutive outputs per thread when
// N is a multiple of 4; the splits are summed in order, in fours or
// eights (16 splits round 4 times at the size of the sum instead of 16).  The
// blocks past the output add up the splits' column sums csum [splits][N] (db).
template <class CE>
__global__ __launch_bounds__(256) void gemm_splitk_epilogue(
    const float* __restrict__ part, int splits, int M, int N, CE* __restrict__ out, int ldo,
    const float* __restrict__ bias, int relu, int accumulate, const float* __restrict__ csum,
    float* __restrict__ db, int db_accumulate) {
  const size_t stride = (size_t)M * N;
  const size_t blocks = (stride + 1023) / 1024;
  if (blockIdx.x >= blocks) {
    const int n = (int)(blockIdx.x - blocks) * 256 + threadIdx.x;
    if (n >= N) return;
    float v = 0.f;
    int s = 0;
    for (; s + 4 <= splits; s += 4)
      v += (csum[(size_t)s * N + n] + csum[(size_t)(s + 1) * N + n]) +
           (csum[(size_t)(s + 2) * N + n] + csum[(size_t)(s + 3) * N + n]);
    for (; s < splits; ++s) v += csum[(size_t)s * N + n];
    db[n] = db_accumulate ? db[n] + v : v;
    return;
  }
  const size_t i4 = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i4 >= stride) return;
  if (N % 4 == 0) {
    f4 v = f4{0.f, 0.f, 0.f, 0.f};
    int s = 0;
    for (; s + 4 <= splits; s += 4) {              // four loads in flight
      f4 p[4];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        p[q] = *reinterpret_cast<const f4*>(part + (size_t)(s + q) * stride + i4);
      v += (p[0] + p[1]) + (p[2] + p[3]);
    }
    for (; s < splits; ++s) v += *reinterpret_cast<const f4*>(part + (size_t)s * stride + i4);
    const int m = (int)(i4 / N), n = (int)(i4 - (size_t)m * N);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float x = v[e];
      if (bias) x += bias[n + e];
      if (relu && !(x > 0.f)) x = 0.f;
      const size_t o = (size_t)m * ldo + n + e;
      if (accumulate) x += Elem<CE>::load(out, o);
      Elem<CE>::store(out, o, x);
    }
    return;
  }
  for (int e = 0; e < 4; ++e) {
    const size_t i = i4 + e;
    if (i >= stride) return;
    const int m = (int)(i / N), n = (int)(i - (size_t)m * N);
    float x = 0.f;
    int s = 0;
    for (; s + 8 <= splits; s += 8) {              // eight loads in flight
      float p[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) p[q] = part[(size_t)(s + q) * stride + i];
      x += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
    }
    for (; s < splits; ++s) x += part[(size_t)s * stride + i];
    if (bias) x += bias[n];
    if (relu && !(x > 0.f)) x = 0.f;
    const size_t o = (size_t)m * ldo + n;
    if (accumulate) x += Elem<CE>::load(out, o);
    Elem<CE>::store(out, o, x);
  }
}

// Tile shape and split of one GEMM: the least estimated time over 128x128 and
// 64x64 block tiles and 1 to 32 ranges of k.
//   * A 64x64 tile stages 32 k at a time in fp32, so that two blocks share a CU
//     and one's first loads and output run beside the other's products: 1024 x
//     2048 outputs of 128 k 13.1 -> 9.8 us, 4096 x 512 of 128 k 13.2 -> 10.4.
//     Two K-contiguous operands of element loads stay with 64 k and one block
//     (479 x 741 outputs of 1859 k: 56.9 us, with 32 k 61.3), bf16 too, whose
//     blocks are small enough (512 x 4096 of 1024 k: 22.4 us, with 32 k 28.3).
//   * Costs in us: `block` for a block's first stages and output, `k32` for 32
//     k, `elems` times as much (X W, dY W^T, X^T dY) where rows allow element
//     loads alone; blocks that share a CU take `alone` of the loop's time where
//     one has it to itself; split partials a launch, `each`, and their traffic,
//     `odd` times as much where outputs are added one by one.
// Fitted to 15000 timings of the three products of 104 shards under forced plans
// in both types; fp32 splits have to save 1.7 us more, since a caller that does
// not capture its calls is bound by launches (K = 2 modulo iterations of 128
// rows: 78 launches and 545 us, 70 and 517 without the splits that save less; a
// bf16 shard of 200 x 1500 x 700 rather needs them, 31 us and 35).  The plan taken
// is 0.8 (bf16) or 1.4 % slower than the best one on average, 19 % at most, where
// one block a CU at the same cost for all operands lost 4 % (fp32) and 12 %
// (bf16), up to 2.1 times.
struct GemmPlan { int bm, ko, mt, nt, splits, kps; size_t ws_bytes; };
struct GemmCost { double block[2], k32[2], elems[2][3], alone, split, each, tb_s, odd; };
static const GemmCost kGCost[2] = {
    {{3.44, 1.35}, {1.74, 1.08}, {{0.63, 1.28, 1.61}, {0.88, 1.17, 1.61}},       // fp32
     0.68, 3.86, 0.11, 5.61, 1.58},
    {{3.69, 1.30}, {0.95, 0.63}, {{1.28, 1.47, 2.17}, {1.37, 1.65, 2.91}},       // bf16
     0.72, 2.50, 0.13, 5.24, 3.5}};

// ak, bk: A, B contiguous along k; aligned: their rows allow vector staging.
static GemmPlan gemm_plan(int M, int N, int K, int esize, bool ak, bool bk, bool aligned) {
  const bool b16 = esize == 2;
  const GemmCost& c = kGCost[b16];
  const double traffic = (double)M * N * 4e-6 / c.tb_s * (N % 4 ? c.odd : 1.0);
  GemmPlan best{};
  double best_t = 0;
  for (int i = 0; i < 2; ++i) {
    const int bm = i == 0 ? 128 : 64, ko = i == 1 && (b16 || (ak && bk && !aligned)) ? 8 : 4;
    const int ks = ko * 8;                                   // k per stage
    const double elems = aligned ? 1.0 : c.elems[i][ak ? (bk ? 1 : 0) : 2];
    const int mt = cdiv(M, bm), nt = cdiv(N, bm), ktiles = cdiv(K, ks);
    const double k32 = c.k32[i] * elems * ks / 32;
    const int64_t tiles = (int64_t)mt * nt;
    for (int s = 1; s <= 32 && s <= ktiles; ++s) {
      const double parts = s > 1 ? c.split + c.each * s + traffic * (2 * s + 1) : 0.0;
      if (s > 1 && parts >= best_t) break;                   // and more with every split
      const int tps = cdiv(ktiles, s);
      if (cdiv(ktiles, tps) != s) continue;
      const bool two = b16 ? bm == 64 || tps * ks <= 32 * kGLocal : bm == 64 && ko == 4;
      const int64_t blocks = tiles * s, rest = blocks & (two ? 511 : 255);
      const double loop = k32 * tps;
      const double all = c.block[i] + loop, alone = c.block[i] + (two ? c.alone : 1.0) * loop;
      const double est = parts + (double)(blocks >> (two ? 9 : 8)) * all +
                         (rest == 0 ? 0.0 : rest <= 256 ? alone : all);
      if (best_t == 0 || est < best_t) {
        best_t = est;
        best = GemmPlan{bm, ko, mt, nt, s, tps * ks, 0};
      }
    }
  }
  // Each split's output, then each split's column sums (db of the dW product).
  best.ws_bytes = best.splits > 1 ? (size_t)best.splits * ((size_t)M * N + N) * sizeof(float) : 0;
  return best;
}

// Vector staging: K-contiguous operands in groups of 4 elements along k,
// row-contiguous ones in pairs of rows.
static bool vec_dims(int ld, int contiguous_extent, bool kc) {
  const int n = kc ? 4 : 2;
  return ld % n == 0 && contiguous_extent % n == 0;
}
template <class E>
static bool vec_ok(const void* p, int ld, int contiguous_extent, bool kc) {
  return ((uintptr_t)p & ((kc ? 4 : 2) * sizeof(E) - 1)) == 0 &&
         vec_dims(ld, contiguous_extent, kc);
}

// The plan of a product with operands of these layouts; it does not depend on
// the tensors' addresses, which the workspace query does not know.
static GemmPlan product_plan(int M, int N, int K, int lda, bool ak, int ldb, bool bk, int esize) {
  return gemm_plan(M, N, K, esize, ak, bk,
                   vec_dims(lda, ak ? K : M, ak) && vec_dims(ldb, bk ? K : N, bk));
}

template <class T, bool AK, bool BK, bool VEC, class E, class CE, bool AMK, bool BMK>
static void gemm_launch_t(const GemmPlan& p, const GemmArgs& g, hipStream_t st) {
  static std::once_flag once;
  std::call_once(once, [] {
    (void)hipFuncSetAttribute((const void*)gemm_split<T, AK, BK, VEC, E, CE, AMK, BMK>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)T::LDS_BYTES);
  });
  gemm_split<T, AK, BK, VEC, E, CE, AMK, BMK>
      <<<(unsigned)(p.mt * p.nt * p.splits), kGThreads, T::LDS_BYTES, st>>>(g);
}

template <bool AK, bool BK, bool VEC, class E, class CE, bool AMK, bool BMK>
static void gemm_launch_m(const GemmPlan& p, const GemmArgs& g, hipStream_t st) {
  constexpr int NP = sizeof(E) == 2 ? 1 : 3;
  constexpr bool B16 = NP == 1;
  // The MFMA drops low bits always in one direction, so long bf16 sums are
  // taken out of it every 128 k (dW of 1024 rows against 64 bits 1.4e-7 with all
  // of them inside, 7e-8 like this, 1.1e-7 on the fp32 MFMA).  Shorter ones
  // stay inside on the large tile: 119 registers instead of 183 leave room
  // for two blocks a CU (dW of 84 rows, 6787 x 692: 18.6 us instead of 21.8).
  if (p.bm == 128) {
    if (B16 && p.kps > 32 * kGLocal)
      gemm_launch_t<GemmTile<128, 128, 4, NP, B16>, AK, BK, VEC, E, CE, AMK, BMK>(p, g, st);
    else
      gemm_launch_t<GemmTile<128, 128, 4, NP, false>, AK, BK, VEC, E, CE, AMK, BMK>(p, g, st);
    return;
  }
  constexpr bool WIDE = B16 || (AK && BK && !VEC);   // where the plan may stage 64 k at a time
  if constexpr (!B16) {
    if (!WIDE || p.ko == 4) {
      gemm_launch_t<GemmTile<64, 64, 4, NP, false>, AK, BK, VEC, E, CE, AMK, BMK>(p, g, st);
      return;
    }
  }
  if constexpr (WIDE)
    gemm_launch_t<GemmTile<64, 64, 8, NP, B16>, AK, BK, VEC, E, CE, AMK, BMK>(p, g, st);
}

// The masks are template arguments, so that no load or store of the
// staging carries a branch.  The library's products mask only dY: the A
// operand of the data-gradient product (both operands K-contiguous) or
// the B operand of the weight-gradient product (neither).
template <bool AK, bool BK, bool VEC, class E, class CE>
static void gemm_launch(const GemmPlan& p, const GemmArgs& g, hipStream_t st) {
  if constexpr (AK && BK) {
    if (g.amask) { gemm_launch_m<AK, BK, VEC, E, CE, true, false>(p, g, st); return; }
  }
  if constexpr (!AK && !BK) {
    if (g.bmask) { gemm_launch_m<AK, BK, VEC, E, CE, false, true>(p, g, st); return; }
  }
  gemm_launch_m<AK, BK, VEC, E, CE, false, false>(p, g, st);
}

// C (ldc) = epi(A * B): the GEMM applies the epilogue itself when the
// reduction is not split; otherwise it writes per-split partial sums to the
// workspace and gemm_splitk_epilogue adds them in order and applies it.
// colsum (may be null): column sums of B, likewise.  p: the product's plan.
template <bool AK, bool BK, class E, class CE>
static sb_status gemm_run(GemmArgs g, const GemmPlan& p, float* ws, size_t ws_bytes,
                          hipStream_t st) {
  // Masks exist only where gemm_launch instantiates them.
  if ((g.amask && !(AK && BK)) || (g.bmask && (AK || BK))) return SB_ERR_UNSUPPORTED;
  if (p.ws_bytes > 0 && (!ws || ws_bytes < p.ws_bytes)) return SB_ERR_WORKSPACE;
  // Buffer ranges cover whole operands.
  const int64_t a_elems = AK ? (int64_t)(g.M - 1) * g.lda + g.K : (int64_t)(g.K - 1) * g.lda + g.M;
  const int64_t b_elems = BK ? (int64_t)(g.N - 1) * g.ldb + g.K : (int64_t)(g.K - 1) * g.ldb + g.N;
  const int64_t es = (int64_t)sizeof(E);
  if (a_elems * es >= (1ll << 31) || b_elems * es >= (1ll << 31)) return SB_ERR_UNSUPPORTED;
  g.mt = p.mt; g.nt = p.nt; g.splits = p.splits; g.k_per_split = p.kps;
  const bool vec = vec_ok<E>(g.a, g.lda, AK ? g.K : g.M, AK) &&
                   vec_ok<E>(g.b, g.ldb, BK ? g.K : g.N, BK) &&
                   (!g.amask || vec_ok<E>(g.amask, g.lda, AK ? g.K : g.M, AK)) &&
                   (!g.bmask || vec_ok<E>(g.bmask, g.ldb, BK ? g.K : g.N, BK));
  CE* out = (CE*)g.c;
  const int ldo = g.ldc;
  const float* bias = g.bias;
  const int relu = g.relu, accumulate = g.accumulate;
  float* colsum = g.colsum;
  const int colsum_acc = g.colsum_acc;
  const bool split = p.splits > 1;
  if (split) {
    g.c = ws; g.ldc = g.N;
    g.bias = nullptr; g.relu = 0; g.accumulate = 0;
    if (colsum) g.colsum = ws + (size_t)p.splits * g.M * g.N;
    g.colsum_acc = 0;
  }
  if (vec) gemm_launch<AK, BK, true, E, CE>(p, g, st);
  else gemm_launch<AK, BK, false, E, CE>(p, g, st);
  if (split) {
    const size_t total = (size_t)g.M * g.N;
    const unsigned blocks = (unsigned)((total + 1023) / 1024) + (colsum ? cdiv(g.N, 256) : 0);
    gemm_splitk_epilogue<CE><<<blocks, 256, 0, st>>>(ws, p.splits, g.M, g.N, out, ldo, bias, relu,
                                                     accumulate, g.colsum, colsum, colsum_acc);
  }
  return SB_OK;
}

}  // namespace sb

using namespace sb;

static sb_status fc_check(const sb_fc_desc* d) {
  if (!d) return SB_ERR_INVALID_ARG;
  if (d->m <= 0 || d->k_in <= 0 || d->n_shard <= 0) return SB_ERR_INVALID_ARG;
  if (d->ldx < d->k_in || d->ldy < d->n_shard) return SB_ERR_INVALID_ARG;
  if (d->flags & ~SB_FUSE_RELU) return SB_ERR_INVALID_ARG;
  if (d->dtype != SB_F32 && d->dtype != SB_BF16) return SB_ERR_INVALID_ARG;
  return SB_OK;
}

// The plans of the three products: Y, dX partial, dW.
static GemmPlan plan_y(const sb_fc_desc* d) {
  return product_plan(d->m, d->n_shard, d->k_in, d->ldx, true, d->n_shard, false,
                      (int)sbh::dsize(d->dtype));
}
static GemmPlan plan_dx(const sb_fc_desc* d) {
  return product_plan(d->m, d->k_in, d->n_shard, d->ldy, true, d->n_shard, true,
                      (int)sbh::dsize(d->dtype));
}
static GemmPlan plan_dw(const sb_fc_desc* d) {
  return product_plan(d->k_in, d->n_shard, d->m, d->ldx, false, d->ldy, false,
                      (int)sbh::dsize(d->dtype));
}

extern "C" size_t sb_fc_workspace_bytes(const sb_fc_desc* d, int pass) {
  if (fc_check(d) != SB_OK) return (size_t)-1;
  if (pass == SB_FC_FWD) return plan_y(d).ws_bytes;
  if (pass == SB_FC_BWD)   // dX partial, then dW: the two share the workspace
    return std::max(plan_dx(d).ws_bytes, plan_dw(d).ws_bytes);
  return (size_t)-1;
}

// Forward on operands of type E (fp32, or bf16 bits with a bf16 output).
template <class E>
static sb_status fc_fwd_run(const sb_fc_desc* d, const GemmPlan& p, const void* x, const void* w,
                            const float* b, void* y, void* ws, size_t ws_bytes, hipStream_t st) {
  GemmArgs g{};
  g.a = x; g.lda = d->ldx; g.amask = nullptr;
  g.b = w; g.ldb = d->n_shard; g.bmask = nullptr;
  g.c = y; g.ldc = d->ldy;
  g.M = d->m; g.N = d->n_shard; g.K = d->k_in;
  g.bias = b; g.relu = (d->flags & SB_FUSE_RELU) ? 1 : 0; g.accumulate = 0;
  return gemm_run<true, false, E, E>(g, p, (float*)ws, ws_bytes, st);
}

extern "C" sb_status sb_fc_shard_fwd(const sb_fc_desc* d, const void* x, const void* w,
                                     const float* b, void* y, void* ws, size_t ws_bytes,
                                     void* stream) {
  sb_status s = fc_check(d);
  if (s != SB_OK) return s;
  if (!x || !w || !y) return SB_ERR_INVALID_ARG;
  const size_t es = d->dtype == SB_BF16 ? 2 : 4;
  size_t xb = ((size_t)(d->m - 1) * d->ldx + d->k_in) * es;
  size_t yb = ((size_t)(d->m - 1) * d->ldy + d->n_shard) * es;
  size_t wb = (size_t)d->k_in * d->n_shard * es;
  if (sbh::overlaps(y, yb, x, xb) || sbh::overlaps(y, yb, w, wb) ||
      sbh::overlaps(y, yb, b, b ? d->n_shard * sizeof(float) : 0))
    return SB_ERR_INVALID_ARG;
  // The workspace (split partials) must not overlap any operand.
  const GemmPlan p = plan_y(d);
  const size_t need = p.ws_bytes;
  if (need > 0 && (sbh::overlaps(ws, need, x, xb) || sbh::overlaps(ws, need, w, wb) ||
                   sbh::overlaps(ws, need, y, yb) ||
                   sbh::overlaps(ws, need, b, b ? d->n_shard * sizeof(float) : 0)))
    return SB_ERR_INVALID_ARG;
  hipStream_t st = sbh::stream_of(stream);
  s = d->dtype == SB_BF16 ? fc_fwd_run<u16>(d, p, x, w, b, y, ws, ws_bytes, st)
                          : fc_fwd_run<float>(d, p, x, w, b, y, ws, ws_bytes, st);
  if (s != SB_OK) return s;
  return sbh::launch_status();
}

// Backward on operands of type E: dx_partial has type E, dW and db fp32.
// db is added up inside the dW product.
template <class E>
static sb_status fc_bwd_run(const sb_fc_desc* d, const GemmPlan& px, const GemmPlan& pw,
                            const void* x, const void* w, const void* dy, const void* mask,
                            void* dxp, float* dw, float* db, int accumulate, void* ws,
                            size_t ws_bytes, hipStream_t st) {
  sb_status s;
  if (dxp) {
    GemmArgs g{};
    g.a = dy; g.lda = d->ldy; g.amask = mask;
    g.b = w; g.ldb = d->n_shard; g.bmask = nullptr;
    g.c = dxp; g.ldc = d->ldx;
    g.M = d->m; g.N = d->k_in; g.K = d->n_shard;
    s = gemm_run<true, true, E, E>(g, px, (float*)ws, ws_bytes, st);
    if (s != SB_OK) return s;
  }
  GemmArgs g{};
  g.a = x; g.lda = d->ldx; g.amask = nullptr;
  g.b = dy; g.ldb = d->ldy; g.bmask = mask;
  g.c = dw; g.ldc = d->n_shard;
  g.M = d->k_in; g.N = d->n_shard; g.K = d->m;
  g.accumulate = accumulate;
  g.colsum = db; g.colsum_acc = accumulate;
  return gemm_run<false, false, E, float>(g, pw, (float*)ws, ws_bytes, st);
}

extern "C" sb_status sb_fc_shard_bwd(const sb_fc_desc* d, const void* x, const void* w,
                                     const void* dy, const void* mask, void* dxp, float* dw,
                                     float* db, int accumulate, void* ws, size_t ws_bytes,
                                     void* stream) {
  sb_status s = fc_check(d);
  if (s != SB_OK) return s;
  if (d->flags != 0) return SB_ERR_INVALID_ARG;
  if (!x || !w || !dy || !dw) return SB_ERR_INVALID_ARG;
  if (accumulate != 0 && accumulate != 1) return SB_ERR_INVALID_ARG;
  const size_t es = d->dtype == SB_BF16 ? 2 : 4;
  size_t xb = ((size_t)(d->m - 1) * d->ldx + d->k_in) * es;
  size_t yb = ((size_t)(d->m - 1) * d->ldy + d->n_shard) * es;
  size_t wb = (size_t)d->k_in * d->n_shard * es;
  size_t dwb = (size_t)d->k_in * d->n_shard * sizeof(float);
  size_t dbb = (size_t)d->n_shard * sizeof(float);
  const void* ins[4] = {x, w, dy, mask};
  size_t insb[4] = {xb, wb, yb, mask ? yb : 0};
  void* outs[3] = {dxp, dw, db};
  size_t outsb[3] = {dxp ? xb : 0, dwb, db ? dbb : 0};
  for (int o = 0; o < 3; ++o) {
    for (int i = 0; i < 4; ++i)
      if (sbh::overlaps(outs[o], outsb[o], ins[i], insb[i])) return SB_ERR_INVALID_ARG;
    for (int o2 = o + 1; o2 < 3; ++o2)
      if (sbh::overlaps(outs[o], outsb[o], outs[o2], outsb[o2])) return SB_ERR_INVALID_ARG;
  }
  const GemmPlan px = plan_dx(d), pw = plan_dw(d);
  const size_t need = std::max(px.ws_bytes, pw.ws_bytes);
  if (need > 0 && (!ws || ws_bytes < need)) return SB_ERR_WORKSPACE;
  // The workspace (split partials) must not overlap any operand.
  if (need > 0) {
    for (int i = 0; i < 4; ++i)
      if (sbh::overlaps(ws, need, ins[i], insb[i])) return SB_ERR_INVALID_ARG;
    for (int o = 0; o < 3; ++o)
      if (sbh::overlaps(ws, need, outs[o], outsb[o])) return SB_ERR_INVALID_ARG;
  }
  hipStream_t st = sbh::stream_of(stream);
  s = d->dtype == SB_BF16
          ? fc_bwd_run<u16>(d, px, pw, x, w, dy, mask, dxp, dw, db, accumulate, ws, ws_bytes, st)
          : fc_bwd_run<float>(d, px, pw, x, w, dy, mask, dxp, dw, db, accumulate, ws, ws_bytes, st);
  if (s != SB_OK) return s;
  return sbh::launch_status();
}
