// fp32 GEMM on the matrix units (gfx950):
//   C[i, j] = sum_k A(i, k) * B(j, k)  (+ epilogue), fp32 products and sums.
//
// v_mfma_f32_32x32x2_f32 multiplies and adds in fp32 at twice the rate of the
// vector unit's FMA (256 against 128 FLOP per clock and CU), so it serves the
// parity path without giving up precision (error against 64 bits of the mid
// LSTM's gradients 1.3e-6 before and after).  A product of 4096 x 2048 x 4096
// takes 645 us here (107 TFLOP/s, matrix units 73% busy) against 1490 us on a
// vector-FMA engine with scalar loads; the LSTM forward's 256 x 4096 x 2048
// 51 us against 215.
//
// Block tile 128 x 128 (4 waves of 64 x 64) where that gives every CU a
// block, else 64 x 64 (4 waves of 32 x 32: four times the blocks); K tile 32.
// Operands go through registers to a double-buffered LDS stage.  A 32 x 32 x
// 2 product holds its unit for 64 clocks, so all else of a K tile is issued
// between products of the same wave (scheduling groups): the loads of tile r
// + 1 during the first runs of 8 k of tile r, the LDS stores of r + 1 during
// the third, then the barrier, and the first fragments of r + 1 are read
// during the last.  (With the loads ahead of the products and the stores
// after them the weight gradient took 697 us, and 776 us while every
// fragment read was waited for.)
//
// LDS layout follows the operand: K-contiguous rows as [row][k] (rows padded
// by 4 floats: a fragment is one 16-byte read, 16 rows fall on 16 distinct
// bank groups); I-contiguous rows as [k][i] (a fragment is four 4-byte reads
// of 32 consecutive floats).  Within a run of 8 k, lanes 0..31 hold k = 0..3
// and lanes 32..63 k = 4..7, so product e of the run takes k = e and 4 + e.
#pragma once

#include "gemm_dma.h"

namespace o5 {

namespace f32e {

constexpr int NT = 256;
constexpr int kBK = 32;  // k per stage

// four consecutive floats with 4-byte alignment (one 16-byte load)
typedef float f4u_t __attribute__((ext_vector_type(4), aligned(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4_t load4(const float* p) { return *reinterpret_cast<const f4u_t*>(p); }

// Read (with stride 0) where an operand has no row mask.
__device__ const uint8_t kNoMask = 0;

// Per-thread state of one operand's ROWS x BK tile.  load() issues the loads
// of the tile at k0 with every index clamped into range and every choice of
// source a select, so no load waits behind a branch or another load; store()
// zeroes what lies outside the matrix or under the row mask and writes the
// LDS stage.  VEC: every source's extent along its contiguous index is a
// multiple of 4, so a chunk is one 16-byte load; else four 4-byte loads.
template <class L, int ROWS, int BK, bool VEC>
struct Op;

template <int ROWS, int BK, bool VEC>
struct Op<KRows2<float>, ROWS, BK, VEC> {
  static constexpr int kStage = ROWS * (BK + 4);  // floats
  static constexpr int kPer = ROWS * BK / 4 / NT;
  static_assert(ROWS * BK / 4 % NT == 0, "tile/threads mismatch");
  const float* b0[kPer];
  const float* b1[kPer];  // the second source's row, offset by -K0
  bool row_ok[kPer], keep1[kPer];
  f4_t r[kPer];

  __device__ __forceinline__ static int row(int tid, int u) { return (tid + u * NT) / (BK / 4); }
  __device__ __forceinline__ static int kc(int tid, int u) { return (tid + u * NT) % (BK / 4) * 4; }

  __device__ __forceinline__ void init(const KRows2<float>& l, int row0, int tid) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int i = row0 + row(tid, u);
      row_ok[u] = i < l.rows;
      const size_t ic = row_ok[u] ? i : 0;
      keep1[u] = row_ok[u] && !(l.mask1 != nullptr && l.mask1[ic] != 0);
      b0[u] = l.p0 + ic * l.ld0;
      b1[u] = l.p1 != nullptr ? l.p1 + ic * l.ld1 - l.K0 : b0[u];
    }
  }
  __device__ __forceinline__ void load(const KRows2<float>& l, int k0, int tid) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int k = k0 + kc(tid, u);
      if constexpr (VEC) {
        const int c = min(k, l.K - 4);
        r[u] = load4((c < l.K0 ? b0[u] : b1[u]) + c);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int c = min(k + q, l.K - 1);
          r[u][q] = (c < l.K0 ? b0[u] : b1[u])[c];
        }
      }
    }
  }
  __device__ __forceinline__ void store(const KRows2<float>& l, int k0, float* lds, int tid) const {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int k = k0 + kc(tid, u);
      f4_t v = r[u];
      if constexpr (VEC) {
        if (k >= l.K || !(k < l.K0 ? row_ok[u] : keep1[u])) v = f4_t{0.0f, 0.0f, 0.0f, 0.0f};
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (k + q >= l.K || !(k + q < l.K0 ? row_ok[u] : keep1[u])) v[q] = 0.0f;
      }
      *reinterpret_cast<f4_t*>(lds + row(tid, u) * (BK + 4) + kc(tid, u)) = v;
    }
  }
  // k run s (8 k) of the 32-row block at row0
  __device__ __forceinline__ static f4_t frag(const float* lds, int row0, int lane, int s) {
    return *reinterpret_cast<const f4_t*>(lds + (row0 + (lane & 31)) * (BK + 4) + 8 * s + 4 * (lane >> 5));
  }
};

template <int ROWS, int BK, bool VEC>
struct Op<ICols2<float>, ROWS, BK, VEC> {
  static constexpr int kPitch = ROWS + 4;
  static constexpr int kStage = BK * kPitch;
  static constexpr int kPer = ROWS * BK / 4 / NT;
  static constexpr int kC = VEC ? 1 : 4;  // columns with a source of their own per chunk
  // row k of the chunk's (column's) source starts at (k < sw ? pa : pb) +
  // k * ld; columns past the matrix repeat its last ones
  const float* pa[kPer][kC];
  const float* pb[kPer][kC];
  int ld[kPer][kC], sw[kPer][kC];
  const uint8_t* mask;
  int mstride, row0;
  f4_t r[kPer];
  uint32_t mb[kPer];  // the row's mask byte as read

  __device__ __forceinline__ static int kr(int tid, int u) { return (tid + u * NT) / (ROWS / 4); }
  __device__ __forceinline__ static int ic(int tid, int u) { return (tid + u * NT) % (ROWS / 4) * 4; }

  __device__ __forceinline__ void init(const ICols2<float>& l, int row0_, int tid) {
    row0 = row0_;
    mask = l.mask1 != nullptr ? l.mask1 : &kNoMask;
    mstride = l.mask1 != nullptr ? 1 : 0;
#pragma unroll
    for (int u = 0; u < kPer; ++u)
#pragma unroll
      for (int q = 0; q < kC; ++q) {
        const int i = VEC ? min(row0 + ic(tid, u), l.I - 4) : min(row0 + ic(tid, u) + q, l.I - 1);
        const bool second = i >= l.I0;
        const int c = second ? i - l.I0 : i;
        pa[u][q] = (second ? l.p1a : l.p0) + c;
        pb[u][q] = second ? l.p1b + c - static_cast<ptrdiff_t>(l.kswitch) * l.ld1 : l.p0 + c;
        ld[u][q] = second ? l.ld1 : l.ld0;
        sw[u][q] = second ? l.kswitch : 0x7fffffff;
      }
  }
  __device__ __forceinline__ void load(const ICols2<float>& l, int k0, int tid) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int k = min(k0 + kr(tid, u), l.K - 1);
      // (a global load by its address space: the choice between the mask and
      // its stand-in hides that from the compiler, and a generic load would
      // make every LDS wait cover it)
      mb[u] = *(const __attribute__((address_space(1))) uint8_t*)(mask + static_cast<size_t>(k) * mstride);
#pragma unroll
      for (int q = 0; q < kC; ++q) {
        const float* p = (k < sw[u][q] ? pa[u][q] : pb[u][q]) + static_cast<size_t>(k) * ld[u][q];
        if constexpr (VEC)
          r[u] = load4(p);
        else
          r[u][q] = *p;
      }
    }
  }
  __device__ __forceinline__ void store(const ICols2<float>& l, int k0, float* lds, int tid) const {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const bool kin = k0 + kr(tid, u) < l.K;
      f4_t v = r[u];
      if constexpr (VEC) {
        const int i = row0 + ic(tid, u);
        if (!kin || i >= l.I || (i >= l.I0 && mb[u] != 0u)) v = f4_t{0.0f, 0.0f, 0.0f, 0.0f};
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int i = row0 + ic(tid, u) + q;
          if (!kin || i >= l.I || (i >= l.I0 && mb[u] != 0u)) v[q] = 0.0f;
        }
      }
      *reinterpret_cast<f4_t*>(lds + kr(tid, u) * kPitch + ic(tid, u)) = v;
    }
  }
  __device__ __forceinline__ static f4_t frag(const float* lds, int row0, int lane, int s) {
    const float* p = lds + (8 * s + 4 * (lane >> 5)) * kPitch + row0 + (lane & 31);
    f4_t v;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = p[q * kPitch];
    return v;
  }
};

inline bool vec_ok(const KRows2<float>& l) { return l.K % 4 == 0 && l.K0 % 4 == 0; }
inline bool vec_ok(const ICols2<float>& l) { return l.I % 4 == 0 && l.I0 % 4 == 0; }

}  // namespace f32e

template <int BT, bool VEC, class AL, class BL, class Epi>
__global__ void __launch_bounds__(f32e::NT) gemm_f32_mfma(AL al, BL bl, Epi epi, int M, int N, int K,
                                                          int ktiles_per_split) {
  using namespace f32e;
  static_assert(BT == 128 || BT == 64, "block tile 128 x 128 or 64 x 64");
  constexpr int BK = kBK;
  static_assert(BK == 32, "four runs of 8 k per stage");
  constexpr int MB = BT / 64;  // 32 x 32 blocks per wave and direction (2 x 2 waves)
  using OA = Op<AL, BT, BK, VEC>;
  using OB = Op<BL, BT, BK, VEC>;
  __shared__ __attribute__((aligned(16))) float as[2][OA::kStage];
  __shared__ __attribute__((aligned(16))) float bs[2][OB::kStage];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave >> 1) * (BT / 2), wn0 = (wave & 1) * (BT / 2);
  int tm, tn;
  xcd_tile(blockIdx.x, (M + BT - 1) / BT, (N + BT - 1) / BT, tm, tn);
  const int m0 = tm * BT, n0 = tn * BT;
  const int split = blockIdx.z;
  const int kt0 = split * ktiles_per_split;
  const int kt1 = min((K + BK - 1) / BK, kt0 + ktiles_per_split);

  f32x16_t acc[MB][MB];
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.0f;

  if (kt0 < kt1) {
    OA oa;
    OB ob;
    oa.init(al, m0, tid);
    ob.init(bl, n0, tid);
    oa.load(al, kt0 * BK, tid);
    ob.load(bl, kt0 * BK, tid);
    oa.store(al, kt0 * BK, as[0], tid);
    ob.store(bl, kt0 * BK, bs[0], tid);
    __syncthreads();
    f4_t af[2][MB], bf[2][MB];
    auto read = [&](int st, int s, int f) {
#pragma unroll
      for (int a = 0; a < MB; ++a) af[f][a] = OA::frag(as[st], wm0 + 32 * a, lane, s);
#pragma unroll
      for (int b = 0; b < MB; ++b) bf[f][b] = OB::frag(bs[st], wn0 + 32 * b, lane, s);
    };
    // the products of run s, with everything else of the region between them
    auto products = [&](int f) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int a = 0; a < MB; ++a)
#pragma unroll
          for (int b = 0; b < MB; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[f][a][q], bf[f][b][q], acc[a][b], 0, 0, 0);
      dma::unroll<0, 4 * MB * MB>([&](auto) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one product
        __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);  // vector ALU
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // global load
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);  // LDS reads
        __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);  // LDS write
      });
      __builtin_amdgcn_sched_barrier(0);
    };
    if (kt1 - kt0 == 1) {
      // a single K tile: only the runs of 8 that hold a k (a weight gradient of
      // 5 rows, 4096 x 4096: 28.0 us with all four, 20.2 so; the vector-FMA engine
      // before it, with its K tile of 16, took 22.6)
      const int runs = min(4, (K - kt0 * BK + 7) / 8);
      for (int s = 0; s < runs; ++s) {
        read(0, s, 0);
        products(0);
      }
    } else {
      read(0, 0, 0);
      for (int kt = kt0; kt < kt1; ++kt) {
        const int st = (kt - kt0) & 1;
        // (past the last tile the loads repeat it and the stage is not read)
        const int kn = min(kt + 1, kt1 - 1) * BK;
        __builtin_amdgcn_sched_barrier(0);
        oa.load(al, kn, tid);
        ob.load(bl, kn, tid);
        read(st, 1, 1);
        products(0);
        read(st, 2, 0);
        products(1);
        read(st, 3, 1);
        oa.store(al, kn, as[st ^ 1], tid);
        ob.store(bl, kn, bs[st ^ 1], tid);
        products(0);
        __syncthreads();
        read(st ^ 1, 0, 0);
        products(1);
      }
    }
  }
  store_acc<MB, MB>(epi, acc, m0 + wm0, n0 + wn0, lane, split, M, N, m0 + BT <= M && n0 + BT <= N);
}

// 128 x 128 tiles where they give every CU a block; a 64 x 64 grid otherwise.
inline bool f32_big_tile(long long M, long long N) { return ((M + 127) / 128) * ((N + 127) / 128) >= 256; }

// Output tiles of an M x N product.
inline long long f32_tiles(long long M, long long N) {
  const int t = f32_big_tile(M, N) ? 128 : 64;
  return ((M + t - 1) / t) * ((N + t - 1) / t);
}

template <class AL, class BL, class Epi>
inline void launch_gemm_f32(const AL& al, const BL& bl, const Epi& epi, int M, int N, int K, int splits,
                            hipStream_t s) {
  const int nkt = (K + f32e::kBK - 1) / f32e::kBK;
  const int kps = (nkt + splits - 1) / splits;
  const dim3 grid(static_cast<unsigned>(f32_tiles(M, N)), 1, splits);
  const bool vec = f32e::vec_ok(al) && f32e::vec_ok(bl);
  auto kernel = f32_big_tile(M, N) ? (vec ? gemm_f32_mfma<128, true, AL, BL, Epi> : gemm_f32_mfma<128, false, AL, BL, Epi>)
                                   : (vec ? gemm_f32_mfma<64, true, AL, BL, Epi> : gemm_f32_mfma<64, false, AL, BL, Epi>);
  hipLaunchKernelGGL(kernel, grid, dim3(f32e::NT), 0, s, al, bl, epi, M, N, K, kps);
}

}  // namespace o5
