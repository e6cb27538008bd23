// One recurrent step of the LSTM in one launch, for small and middle batches
// (and every batch in fp32): the step's product and its cell.
//
//   forward   a = [x_t | h~_{t-1}] . [W_x | W_h]^T + b, then the cell
//   backward  R = [P_t | dG_{t+1}] . [W | W_h^T]^T, then the gate gradients
//             (P, W only where the heads' gradient comes in factored form)
//
// A block owns 16 MF batch rows x 16 hidden units (forward: their four gates,
// 64 columns) or 16 MF rows x 16 NF units (backward) for the whole reduction,
// so no partial sum goes through HBM and the cell needs no second launch.
// Its 4 waves split K: wave w takes the 128-byte pieces w, w + 4, ... of
// every row, so the block reads 512 bytes of each row at a time.  A wave copies
// its pieces straight to LDS (buffer loads, 8 rows x 128 bytes each: whole
// cache lines, four consecutive lanes in one) into a ring of its own, so the
// loop has no barrier; it reads the MFMA fragments (v_mfma_f32_16x16x32_bf16,
// or v_mfma_f32_16x16x4_f32) and refills the stage before it multiplies.  The
// 4 partial tiles meet once in LDS, are added in wave order, and the same
// threads finish the cell.  (Fragments loaded from memory straight into
// registers, 16 rows x 64 bytes with consecutive lanes on different rows,
// took 22.8 us for a bf16 step of B = 256, D = H = 1024;
// this form takes 11.7, the product and cell as two launches took 36.)
//
// Tiles are dealt so that an XCD holds all row blocks of a run of units: its
// share of the weights is read into its L2 once per step.
#pragma once

#include "gemm_kk.h"

namespace o5 {

namespace step {

constexpr int NW = 4;
constexpr int NT = NW * 64;
constexpr int PIECE = 128;          // bytes of a row per piece: a cache line
constexpr int HALVES = PIECE / 64;  // MFMA k steps per piece
constexpr int CPR = PIECE / 16;     // 16-byte chunks per stage row
constexpr int RPC = 1024 / PIECE;   // rows per copy
constexpr int UNITS = 16;           // hidden units per block (forward)

typedef float f4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void mma(const uint4& a, const uint4& b, f4_t& c, const uint16_t*) {
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0,
                                              0);
}
__device__ __forceinline__ void mma(const uint4& a, const uint4& b, f4_t& c, const float*) {
  const f4_t x = __builtin_bit_cast(f4_t, a), y = __builtin_bit_cast(f4_t, b);
#pragma unroll
  for (int q = 0; q < 4; ++q) c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[q], y[q], c, 0, 0, 0);
}

// 16-byte chunk c of stage row r is stored at slot c ^ (r / (256 / PIECE)) %
// CPR: the 16 rows of a fragment read fall on 16 distinct 16-byte bank groups.
__device__ __forceinline__ int slot(int r, int c) { return c ^ ((r / (256 / PIECE)) % CPR); }

// One operand of F 16-row fragments with two sources along K: source 0 holds
// pieces [0, n0), source 1 the rest up to n.  A lane's byte offset into each
// source is fixed (copy q of a piece moves stage rows 8 q .. 8 q + 7); a row
// that reads zeros has an offset past the buffer.
template <int F>
struct Operand {
  kk::rsrc_t r0, r1;
  uint32_t v0[HALVES * F], v1[HALVES * F];
  int n0, n;

  // rows [0, rows) of ld0 / ld1 bytes; row(r) gives the source row of stage
  // row r and whether it is masked in source 1
  template <class Row>
  __device__ __forceinline__ void init(const void* p0, const void* p1, uint32_t rows, uint32_t ld0, uint32_t ld1,
                                       int n0_, int n_, int lane, Row&& row) {
    n0 = n0_;
    n = n_;
    r0 = kk::make_rsrc(p0, rows * ld0);
    r1 = kk::make_rsrc(p1, rows * ld1);
#pragma unroll
    for (int q = 0; q < HALVES * F; ++q) {
      const int r = RPC * q + lane / CPR;
      const uint32_t c = slot(r, lane % CPR) * 16;
      bool masked = false;
      const uint32_t sr = row(r, masked);
      v0[q] = sr < rows ? sr * ld0 + c : kk::kOutOfRange;
      v1[q] = sr < rows && !masked ? sr * ld1 + c : kk::kOutOfRange;
    }
  }
  // copy q of piece u, to the stage at LDS address `lds` (past the last
  // piece: zeros, nothing read)
  __device__ __forceinline__ void issue_one(int u, uint32_t lds, int q) const {
    const bool s0 = u < n0;
    kk::rsrc_t rs = s0 ? r0 : r1;
    if (u >= n) rs.z = 0;
    const uint32_t soff = static_cast<uint32_t>(s0 ? u : u - n0) * PIECE;
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(s0 ? v0[q] : v1[q]),
                 "s"(rs), "s"(soff), "s"(lds + q * 1024)
                 : "memory", "m0");
  }
  // fragment f, half q (64 bytes) of the piece in `stage`
  __device__ __forceinline__ static uint4 read(const char* stage, int f, int q, int lane) {
    const int r = 16 * f + (lane & 15);
    return *reinterpret_cast<const uint4*>(stage + r * PIECE + slot(r, q * 4 + (lane >> 4)) * 16);
  }
};

// LDS bytes of the rings of the waves.
template <int NA, int NB, int NST>
constexpr size_t ring_bytes() {
  return static_cast<size_t>(NW) * NST * (NA + NB) * 16 * PIECE;
}

// acc[a][b] += this wave's pieces of the NA x NB fragments' product, through
// NST stages of the wave's own.  While the products of piece i run from
// registers, piece i + NST is copied into the stage that piece i was read out
// of (the first half of the products) and the fragments of piece i + 1 are
// read (the second half); scheduling barriers keep one copy or read between
// products, so a wave alone on its SIMD overlaps the three (31.6 against 33.1
// us one after the other for B = 256, D = H = 2048 in bf16).  Measured
// slower: pieces of 64 bytes in twice the stages (half lines: 40 us), two
// waves with twice the stages each (44 us).
template <typename E, int NST, int NA, int NB>
__device__ __forceinline__ void k_loop(const Operand<NA>& oa, const Operand<NB>& ob, char* smem, int wave, int lane,
                                       f4_t (&acc)[NA][NB]) {
  constexpr int STAGE = (NA + NB) * 16 * PIECE;
  constexpr int COPIES = HALVES * (NA + NB);  // per stage; also the fragment reads per piece
  constexpr int MM = HALVES * NA * NB;        // products per piece (of one k step each)
  static_assert(MM % 2 == 0, "halves of a piece's products");
  char* mine = smem + wave * NST * STAGE;
  const uint32_t l0 = static_cast<uint32_t>(reinterpret_cast<size_t>((__attribute__((address_space(3))) char*)mine));
  const int cnt = (oa.n - wave + NW - 1) / NW;  // this wave's pieces (may be <= 0)
  uint4 fa[2][HALVES][NA], fb[2][HALVES][NB];
  auto issue_one = [&](int i, int st, int c) {
    if (c < HALVES * NA)
      oa.issue_one(wave + i * NW, l0 + st, c);
    else
      ob.issue_one(wave + i * NW, l0 + st + NA * 16 * PIECE, c - HALVES * NA);
  };
  // read c of a piece's fragments: those of k step 0 first
  auto read_one = [&](const char* st, int f, int c) {
    const int q = c / (NA + NB), k = c % (NA + NB);
    if (k < NB)
      fb[f][q][k] = Operand<NB>::read(st + NA * 16 * PIECE, k, q, lane);
    else
      fa[f][q][k - NB] = Operand<NA>::read(st, k - NB, q, lane);
  };
  auto product = [&](int f, int m) {
    const int q = m / (NA * NB), a = m / NB % NA, b = m % NB;
    mma(fa[f][q][a], fb[f][q][b], acc[a][b], static_cast<const E*>(nullptr));
  };
  if (cnt <= 0) return;
#pragma unroll
  for (int s = 0; s < NST; ++s)
#pragma unroll
    for (int c = 0; c < COPIES; ++c) issue_one(s, s * STAGE, c);
  dma::vm_wait<(NST - 1) * COPIES>();
#pragma unroll
  for (int c = 0; c < COPIES; ++c) read_one(mine, 0, c);
  int st = 0;  // byte offset of piece i's stage
  auto step = [&](int i, auto F) {
    constexpr int f = decltype(F)::value;
    const int nx = st + STAGE == NST * STAGE ? 0 : st + STAGE;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // piece i is read out: its stage is free
    __builtin_amdgcn_sched_barrier(0);
    dma::unroll<0, MM / 2>([&](auto M) {
      constexpr int m = decltype(M)::value;
      product(f, m);
      dma::unroll<m * COPIES / (MM / 2), (m + 1) * COPIES / (MM / 2)>(
          [&](auto C) { issue_one(i + NST, st, decltype(C)::value); });
      __builtin_amdgcn_sched_barrier(0);
    });
    dma::vm_wait<(NST - 1) * COPIES>();  // piece i + 1 has landed
    const char* np = mine + nx;
    dma::unroll<0, MM / 2>([&](auto M) {
      constexpr int m = decltype(M)::value;
      product(f, MM / 2 + m);
      dma::unroll<m * COPIES / (MM / 2), (m + 1) * COPIES / (MM / 2)>(
          [&](auto C) { read_one(np, f ^ 1, decltype(C)::value); });
      __builtin_amdgcn_sched_barrier(0);
    });
    st = nx;
  };
  // (an odd count takes one piece of zeros more: a tail of its own would cost
  // accumulator moves in every iteration)
  for (int i = 0; i < cnt; i += 2) {
    step(i, std::integral_constant<int, 0>{});
    step(i + 1, std::integral_constant<int, 1>{});
  }
  dma::vm_wait<0>();  // no copy outlives the loop
}

// Leaves the wave's accumulators in red [NW][16 NA][PITCH] (fragment layout:
// lane holds column lane % 16, element e row 4 (lane / 16) + e).
template <int NA, int NB, int PITCH>
__device__ __forceinline__ void park(const f4_t (&acc)[NA][NB], float* red, int wave, int lane) {
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        red[(wave * 16 * NA + 16 * a + 4 * (lane >> 4) + e) * PITCH + 16 * b + (lane & 15)] = acc[a][b][e];
}

// The waves' partial sums of (row, col), in wave order.
template <int ROWS, int PITCH>
__device__ __forceinline__ float gather(const float* red, int row, int col) {
  float v[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) v[w] = red[(w * ROWS + row) * PITCH + col];
  float s = v[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) s += v[w];
  return s;
}

// Row block and column block of a linear block id: each XCD takes all row
// blocks of a contiguous run of column blocks.
__device__ __forceinline__ void tile_of(int id, int nrow, int ncol, int& rb, int& cb) {
  if ((ncol & 7) == 0) {
    const int slot = id >> 3;
    rb = slot % nrow;
    cb = (id & 7) * (ncol >> 3) + slot / nrow;
  } else {
    rb = id % nrow;
    cb = id / nrow;
  }
}

// Stages per wave for F fragments of both operands.
template <int F>
constexpr int stages() {
  constexpr int lds = 160 * 1024 / (NW * F * 16 * PIECE);
  constexpr int wait = 63 / (HALVES * F) + 1;  // (NST - 1) stages' copies within vmcnt's range
  constexpr int fit = lds < wait ? lds : wait;
  return fit < 6 ? fit : 6;
}

// Forward step.  Grid: cdiv(B, 16 MF) * (H / 16) blocks.
template <typename E, int MF>
__global__ void __launch_bounds__(NT, 1) lstm_step_fwd(int B, int D, int H, const E* __restrict__ x,
                                                       const E* __restrict__ h_prev, const E* __restrict__ Wx,
                                                       const E* __restrict__ Wh, const float* __restrict__ bias,
                                                       const float* __restrict__ c_prev,
                                                       const uint8_t* __restrict__ reset_t, E* __restrict__ h_out,
                                                       float* __restrict__ c_out, E* __restrict__ gates_out) {
  constexpr int ROWS = 16 * MF, PITCH = 4 * UNITS + 4;
  constexpr int EPT = ROWS * UNITS / NT;  // elements per thread
  constexpr int NST = stages<MF + 4>();
  constexpr size_t RED = sizeof(float) * NW * ROWS * PITCH;
  constexpr size_t RING = ring_bytes<MF, 4, NST>();
  __shared__ __attribute__((aligned(1024))) char smem[RED > RING ? RED : RING];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int rb, cb;
  tile_of(blockIdx.x, (B + ROWS - 1) / ROWS, H / UNITS, rb, cb);
  const int m0 = rb * ROWS, u0 = cb * UNITS;
  constexpr int EPP = PIECE / sizeof(E);
  const uint32_t ldx = D * sizeof(E), ldh = H * sizeof(E);

  Operand<MF> oa;
  Operand<4> ob;
  oa.init(x, h_prev, B, ldx, ldh, D / EPP, (D + H) / EPP, lane, [&](int r, bool& masked) {
    const int row = m0 + r;
    masked = reset_t != nullptr && row < B && reset_t[row] != 0;
    return static_cast<uint32_t>(row);
  });
  ob.init(Wx, Wh, 4 * H, ldx, ldh, D / EPP, (D + H) / EPP, lane,
          [&](int r, bool&) { return static_cast<uint32_t>((r >> 4) * H + u0 + (r & 15)); });
  // what the cell needs, requested ahead of the product (reset flags as bytes)
  float cp[EPT], bs[4];
  const int uc = tid & (UNITS - 1);
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const size_t row = min(m0 + (tid >> 4) + i * (NT / UNITS), B - 1);
    cp[i] = c_prev[row * H + u0 + uc];
  }
#pragma unroll
  for (int g = 0; g < 4; ++g) bs[g] = bias[g * H + u0 + uc];

  f4_t acc[MF][4];
#pragma unroll
  for (int a = 0; a < MF; ++a)
#pragma unroll
    for (int g = 0; g < 4; ++g) acc[a][g] = f4_t{0.0f, 0.0f, 0.0f, 0.0f};
  k_loop<E, NST>(oa, ob, smem, wave, lane, acc);
  float* red = reinterpret_cast<float*>(smem);
  __syncthreads();  // every wave is done with its ring
  park<MF, 4, PITCH>(acc, red, wave, lane);
  __syncthreads();

#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int r = (tid >> 4) + i * (NT / UNITS);
    const int row = m0 + r;
    if (row >= B) continue;
    float p[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) p[g] = gather<ROWS, PITCH>(red, r, g * UNITS + uc) + bs[g];
    const float cpv = (reset_t != nullptr && reset_t[row] != 0) ? 0.0f : cp[i];
    const float ig = sigmoid_f(p[0]), fg = sigmoid_f(p[1]), gg = tanh_f(p[2]), og = sigmoid_f(p[3]);
    const float c = fg * cpv + ig * gg;
    const size_t hj = static_cast<size_t>(row) * H + u0 + uc;
    c_out[hj] = c;
    h_out[hj] = elem<E>::from_f32(og * tanh_f(c));
    if (gates_out != nullptr) {
      E* gp = gates_out + static_cast<size_t>(row) * 4 * H + u0 + uc;
      gp[0] = elem<E>::from_f32(ig);
      gp[H] = elem<E>::from_f32(fg);
      gp[2 * H] = elem<E>::from_f32(gg);
      gp[3 * H] = elem<E>::from_f32(og);
    }
  }
}

// Backward step t: the recurrent product over source 0 (the factored heads'
// gradient: P_t [B][ldp] against Wf [H][ldp]; K0 = 0 without) and source 1
// (dG_{t+1} [B][4H] against W_h^T [H][4H]; absent where dG_next is null), the
// rows under reset_next zero in source 1; then the cell as lstm_bwd_cell.
// Grid: (time-padded rows / (16 MF)) * (H / (16 NF)) blocks; a block past B
// writes the zeros of its padding columns.  Partial column sums of dG go to
// row rb * ROWS / 32 of db_part (one row per 32 batch rows).
template <typename E, int MF, int NF>
__global__ void __launch_bounds__(NT, 1) lstm_step_bwd(
    int B, int Bp, int H, const E* __restrict__ P, const E* __restrict__ Wf, int K0, const E* __restrict__ dG_next,
    const E* __restrict__ WhT, const uint8_t* __restrict__ reset_next, const float* __restrict__ dh_t,
    const float* __restrict__ dh_extra, const float* dc_in, float* dc_out, const E* __restrict__ gates_t,
    const float* __restrict__ c_t, const float* __restrict__ c_prev, const uint8_t* __restrict__ reset_t,
    E* __restrict__ dG_t, float* __restrict__ db_part, int db_accumulate, E* __restrict__ dGT, size_t ldt, int col0) {
  constexpr int ROWS = 16 * MF, COLS = 16 * NF, PITCH = COLS + 4;
  constexpr int RG = NT / COLS;         // row groups: a thread takes rows rg, rg + RG, ...
  constexpr int EPT = ROWS / RG;        // rows per thread
  constexpr int TP = ROWS + 8;          // row pitch of the transposed tile (bf16)
  static_assert(EPT >= 1 && ROWS % 32 == 0 && 4 * COLS <= NT, "whole rows of db_part, a thread per column and gate");
  constexpr int NST = stages<MF + NF>();
  constexpr size_t RED = sizeof(float) * NW * ROWS * PITCH;
  constexpr size_t SUMS = sizeof(float) * RG * 4 * COLS;
  constexpr size_t TQ = sizeof(E) == 2 ? sizeof(uint16_t) * 4 * COLS * TP : 0;
  constexpr size_t RING = ring_bytes<MF, NF, NST>();
  constexpr size_t SMEM = RED > RING ? RED : RING;
  static_assert(SUMS + TQ <= SMEM, "the epilogue's arrays reuse the ring");
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];
  float* red = reinterpret_cast<float*>(smem);
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int rb, cb;
  tile_of(blockIdx.x, Bp / ROWS, H / COLS, rb, cb);
  const int m0 = rb * ROWS, j0 = cb * COLS;
  const int G = 4 * H;

  f4_t acc[MF][NF];
#pragma unroll
  for (int a = 0; a < MF; ++a)
#pragma unroll
    for (int b = 0; b < NF; ++b) acc[a][b] = f4_t{0.0f, 0.0f, 0.0f, 0.0f};
  if (m0 < B) {
    constexpr int EPP = PIECE / sizeof(E);
    const uint32_t ld0 = K0 * sizeof(E), ld1 = G * sizeof(E);
    const int n = (K0 + (dG_next != nullptr ? G : 0)) / EPP;
    Operand<MF> oa;
    Operand<NF> ob;
    oa.init(P, dG_next, B, ld0, ld1, K0 / EPP, n, lane, [&](int r, bool& masked) {
      const int row = m0 + r;
      masked = reset_next != nullptr && row < B && reset_next[row] != 0;
      return static_cast<uint32_t>(row);
    });
    ob.init(Wf, WhT, H, ld0, ld1, K0 / EPP, n, lane, [&](int r, bool&) { return static_cast<uint32_t>(j0 + r); });
    k_loop<E, NST>(oa, ob, smem, wave, lane, acc);
  }

  // the cell's inputs, requested before the partial sums meet
  const int jc = tid % COLS, rg = tid / COLS;
  const int j = j0 + jc;
  float dhv[EPT], exv[EPT], dcv[EPT], ctv[EPT], cpv[EPT], gin[EPT][4];
  bool rt[EPT];
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int bc = min(m0 + rg + i * RG, B - 1);
    const size_t hj = static_cast<size_t>(bc) * H + j;
    const size_t gj = static_cast<size_t>(bc) * G + j;
    dhv[i] = dh_t != nullptr ? dh_t[hj] : 0.0f;
    exv[i] = dh_extra != nullptr ? dh_extra[hj] : 0.0f;
    dcv[i] = dc_in != nullptr ? dc_in[hj] : 0.0f;
#pragma unroll
    for (int g = 0; g < 4; ++g) gin[i][g] = elem<E>::to_f32(gates_t[gj + g * static_cast<size_t>(H)]);
    ctv[i] = c_t[hj];
    cpv[i] = c_prev[hj];
    rt[i] = reset_t != nullptr && reset_t[bc] != 0;
  }
  __syncthreads();  // every wave is done with its ring
  park<MF, NF, PITCH>(acc, red, wave, lane);
  __syncthreads();
  float rec[EPT];
#pragma unroll
  for (int i = 0; i < EPT; ++i) rec[i] = gather<ROWS, PITCH>(red, rg + i * RG, jc);
  __syncthreads();  // the partial sums' memory is free

  float* sums = reinterpret_cast<float*>(smem);              // [RG][4][COLS]
  uint16_t* tq = reinterpret_cast<uint16_t*>(smem + SUMS);   // [4 COLS][TP]
  float sd[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int r = rg + i * RG, b = m0 + r;
    float d[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (b < B) {
      const float dh = dhv[i] + exv[i] + rec[i];
      const float ig = gin[i][0], fg = gin[i][1], gg = gin[i][2], og = gin[i][3];
      const float tc = tanh_f(ctv[i]);
      const float keep = rt[i] ? 0.0f : 1.0f;
      const float dc = dcv[i] + dh * og * (1.0f - tc * tc);
      d[0] = dc * gg * ig * (1.0f - ig);
      d[1] = dc * (keep * cpv[i]) * fg * (1.0f - fg);
      d[2] = dc * ig * (1.0f - gg * gg);
      d[3] = dh * tc * og * (1.0f - og);
      dc_out[static_cast<size_t>(b) * H + j] = keep * dc * fg;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        dG_t[static_cast<size_t>(b) * G + g * static_cast<size_t>(H) + j] = elem<E>::from_f32(d[g]);
        sd[g] += d[g];
      }
    }
    if constexpr (sizeof(E) == 2) {
#pragma unroll
      for (int g = 0; g < 4; ++g) tq[(g * COLS + jc) * TP + r] = f32_to_bf16_bits(d[g]);
    }
  }
#pragma unroll
  for (int g = 0; g < 4; ++g) sums[(rg * 4 + g) * COLS + jc] = sd[g];
  __syncthreads();
  if (tid < 4 * COLS) {
    const int g = tid / COLS, jl = tid % COLS;
    float s = 0.0f;
#pragma unroll
    for (int q = 0; q < RG; ++q) s += sums[(q * 4 + g) * COLS + jl];
    float* p = db_part + static_cast<size_t>(m0 / 32) * G + g * static_cast<size_t>(H) + j0 + jl;
    *p = db_accumulate ? *p + s : s;  // the same block owns this entry at every step
    if (!db_accumulate) {
#pragma unroll
      for (int q = 1; q < ROWS / 32; ++q) p[static_cast<size_t>(q) * G] = 0.0f;
    }
  }
  if constexpr (sizeof(E) == 2) {
    constexpr int CPR = ROWS / 8;  // 16-byte pieces per transposed row
    for (int e = tid; e < 4 * COLS * CPR; e += NT) {
      const int u = e / CPR, c = e % CPR;
      const uint4 v = *reinterpret_cast<const uint4*>(tq + u * TP + 8 * c);
      *reinterpret_cast<uint4*>(dGT + (static_cast<size_t>(u / COLS) * H + j0 + u % COLS) * ldt + col0 + m0 + 8 * c) = v;
    }
  }
}

// Every operand lies within the 32-bit byte offsets of the copies.
inline bool offsets_fit(size_t esize, int B, int D, int H) {
  const size_t lim = size_t{1} << 31;
  return 4 * static_cast<size_t>(H) * D * esize < lim && 4 * static_cast<size_t>(H) * H * esize < lim &&
         static_cast<size_t>(B) * D * esize < lim && 4 * static_cast<size_t>(B) * H * esize < lim;
}

}  // namespace step

// Row fragments per block of the forward step: the tallest tile that still
// gives every CU a block (a taller tile reads the weights fewer times).
inline int step_fwd_mf(int B, int H) {
  for (int mf = 4; mf > 1; mf /= 2)
    if (static_cast<long long>((B + 16 * mf - 1) / (16 * mf)) * (H / step::UNITS) >= 256) return mf;
  return 1;
}

template <typename E>
inline void launch_step_fwd(int B, int D, int H, const E* x, const E* h_prev, const E* Wx, const E* Wh,
                            const float* bias, const float* c_prev, const uint8_t* reset_t, E* h, float* c, E* gates,
                            hipStream_t s) {
  const int mf = step_fwd_mf(B, H);
  auto kernel = mf == 4 ? step::lstm_step_fwd<E, 4> : mf == 2 ? step::lstm_step_fwd<E, 2> : step::lstm_step_fwd<E, 1>;
  const unsigned blocks = static_cast<unsigned>((B + 16 * mf - 1) / (16 * mf)) * (H / step::UNITS);
  hipLaunchKernelGGL(kernel, dim3(blocks), dim3(step::NT), 0, s, B, D, H, x, h_prev, Wx, Wh, bias, c_prev, reset_t, h,
                     c, gates);
}

}  // namespace o5
