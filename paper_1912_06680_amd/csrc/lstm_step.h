// One recurrent step of the LSTM in one launch, for small and middle batches
// (in fp32 for most shapes): the step's product and its cell.
//
//   forward   a = [x_t | h~_{t-1}] . [W_x | W_h]^T + b, then the cell
//   backward  R = [P_t | dG_{t+1}] . [W | W_h^T]^T, then the gate gradients
//             (P, W only where the heads' gradient comes in factored form)
//
// A block owns 16 to 64 batch rows x 16 hidden units (forward: their four
// gates, 64 columns) or T x T rows and units (backward) for the whole reduction,
// so no partial sum goes through HBM and the cell needs no second launch.
// Its 4 waves split K into 128-byte pieces of every row.  A wave copies
// its pieces straight to LDS (buffer loads, 8 rows x 128 bytes each: whole
// cache lines, four consecutive lanes in one) into a ring of its own, so the
// loop has no barrier; it reads the MFMA fragments (v_mfma_f32_32x32x16_bf16,
// or v_mfma_f32_16x16x4_f32) and refills the stage while it multiplies.  The
// partial tiles meet once in LDS, are added in order, and the same threads
// finish the cell.  In bf16 the K ranges of the partial sums and the order
// within them are those of the separate product (gemm_plan.h), so a shape's
// results do not depend, to the bit, on which of the two paths serves it; in
// fp32 wave w takes pieces w, w + 4, ....  (Fragments loaded from memory straight into
// registers, 16 rows x 64 bytes with consecutive lanes on different rows,
// took 22.8 us for a bf16 step of B = 256, D = H = 1024;
// this form takes 12.5, the product and cell as two launches took 36.)
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
constexpr int CPR = PIECE / 16;     // 16-byte chunks per stage row
constexpr int RPC = 1024 / PIECE;   // rows per copy
constexpr int UNITS = 16;           // hidden units per block (forward)

typedef float f4_t __attribute__((ext_vector_type(4)));

// The fragments of a type: R rows (or columns) per block of the accumulator,
// STEPS 16-byte reads per lane and piece, and where an accumulator element
// lies (lane -> column, lane and element -> row).
template <typename E>
struct Frag;
template <>
struct Frag<uint16_t> {  // 32 x 32 x 16: two chunks per step, one per half wave
  static constexpr int R = 32, STEPS = 4, N = 16;
  typedef f32x16_t acc_t;
  __device__ __forceinline__ static int chunk(int s, int lane) { return 2 * s + (lane >> 5); }
  __device__ __forceinline__ static int row(int e, int lane) { return 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3); }
  __device__ __forceinline__ static void mma(const uint4& a, const uint4& b, acc_t& c) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0,
                                                0, 0);
  }
};
template <>
struct Frag<float> {  // 16 x 16 x 4, four times: four chunks per step, one per quarter wave
  static constexpr int R = 16, STEPS = 2, N = 4;
  typedef f4_t acc_t;
  __device__ __forceinline__ static int chunk(int s, int lane) { return 4 * s + (lane >> 4); }
  __device__ __forceinline__ static int row(int e, int lane) { return 4 * (lane >> 4) + e; }
  __device__ __forceinline__ static void mma(const uint4& a, const uint4& b, acc_t& c) {
    const f4_t x = __builtin_bit_cast(f4_t, a), y = __builtin_bit_cast(f4_t, b);
#pragma unroll
    for (int q = 0; q < 4; ++q) c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[q], y[q], c, 0, 0, 0);
  }
};

// 16-byte chunk c of stage row r is stored at slot c ^ (r / 2) % 8: 16 rows
// read at one chunk fall on 16 distinct 16-byte bank groups.
__device__ __forceinline__ int slot(int r, int c) { return c ^ ((r >> 1) & 7); }

// One operand of ROWS stage rows with two sources along K: source 0 holds
// pieces [0, n0), source 1 the rest up to n.  A lane's byte offset into each
// source is fixed (copy q of a piece moves stage rows 8 q .. 8 q + 7); a row
// that reads zeros has an offset past the buffer.
template <int ROWS>
struct Operand {
  static constexpr int COPIES = ROWS / RPC;
  kk::rsrc_t r0, r1;
  uint32_t v0[COPIES], v1[COPIES];
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
    for (int q = 0; q < COPIES; ++q) {
      const int r = RPC * q + lane / CPR;
      const uint32_t c = slot(r, lane % CPR) * 16;
      bool masked = false;
      const uint32_t sr = row(r, masked);
      v0[q] = sr < rows ? sr * ld0 + c : kk::kOutOfRange;
      v1[q] = sr < rows && !masked ? sr * ld1 + c : kk::kOutOfRange;
    }
  }
  // copy q of piece u, to the stage at LDS address `lds` (no such piece:
  // zeros, nothing read)
  __device__ __forceinline__ void issue_one(int u, uint32_t lds, int q) const {
    const bool none = u < 0 || u >= n;
    const bool s0 = none || u < n0;
    kk::rsrc_t rs = s0 ? r0 : r1;
    if (none) rs.z = 0;  // an empty buffer: every offset reads zero
    const uint32_t soff = none ? 0u : static_cast<uint32_t>(s0 ? u : u - n0) * PIECE;
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(s0 ? v0[q] : v1[q]),
                 "s"(rs), "s"(soff), "s"(lds + q * 1024)
                 : "memory", "m0");
  }
};

// Fragment f, step s of the piece in `stage`.
template <typename E>
__device__ __forceinline__ uint4 read_frag(const char* stage, int f, int s, int lane) {
  const int r = Frag<E>::R * f + (lane & (Frag<E>::R - 1));
  return *reinterpret_cast<const uint4*>(stage + r * PIECE + slot(r, Frag<E>::chunk(s, lane)) * 16);
}

// The pieces of one wave: up to two runs (each a partial sum of its own), run
// q the cnt[q] pieces first[q], first[q] + stride, ....
struct Runs {
  int first[2], cnt[2], stride;
  // piece i of the wave, run 0 padded to an even count; -1: zeros
  __device__ __forceinline__ int at(int i) const {
    const int pad = (cnt[0] + 1) & ~1;
    const int q = i < pad ? 0 : 1;
    const int k = i - (q ? pad : 0);
    return k < cnt[q] ? first[q] + k * stride : -1;
  }
};

// The K ranges of a wave: S partial sums of kps pieces each, the wave's own
// first and, beyond NW, its second; S = 0: one run of every NW-th piece.
__device__ __forceinline__ Runs runs_of(int S, int kps, int n, int wave) {
  Runs r;
  if (S == 0) {
    r.stride = NW;
    r.first[0] = wave;
    r.cnt[0] = max(0, (n - wave + NW - 1) / NW);
    r.first[1] = r.cnt[1] = 0;
  } else {
    r.stride = 1;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int sp = wave + q * NW;
      r.first[q] = sp * kps;
      r.cnt[q] = sp < S ? max(0, min(n, (sp + 1) * kps) - sp * kps) : 0;
    }
  }
  return r;
}

// acc[q][a][b] = the products of the wave's run q, through NST stages of the
// wave's own.  While the products of piece i run from registers, piece i +
// NST is copied into the stage that piece i was read out of (the first half
// of the products) and the fragments of piece i + 1 are read (the second
// half); scheduling barriers keep one copy or read between products, so a
// wave alone on its SIMD overlaps the three (31.6 against 33.1 us one after
// the other for B = 256, D = H = 2048 in bf16).  Measured slower: pieces of 64
// bytes in twice the stages (half lines: 40 us), two waves with twice the
// stages each (44 us).
template <typename E, int NST, int RA, int RB, int Q>
__device__ __forceinline__ void k_loop(const Operand<RA>& oa, const Operand<RB>& ob, const Runs& runs, char* smem,
                                       int wave, int lane,
                                       typename Frag<E>::acc_t (&acc)[Q][RA / Frag<E>::R][RB / Frag<E>::R]) {
  typedef Frag<E> F;
  constexpr int NA = RA / F::R, NB = RB / F::R;
  constexpr int STAGE = (RA + RB) * PIECE;
  constexpr int COPIES = Operand<RA>::COPIES + Operand<RB>::COPIES;  // per stage
  constexpr int READS = F::STEPS * (NA + NB);                        // per piece
  constexpr int HALF = F::STEPS * NA * NB / 2;                       // products per half piece
  char* mine = smem + wave * NST * STAGE;
  const uint32_t l0 = static_cast<uint32_t>(reinterpret_cast<size_t>((__attribute__((address_space(3))) char*)mine));
  uint4 fa[2][F::STEPS][NA], fb[2][F::STEPS][NB];
  auto issue_one = [&](int u, int st, int c) {
    if (c < Operand<RA>::COPIES)
      oa.issue_one(u, l0 + st, c);
    else
      ob.issue_one(u, l0 + st + RA * PIECE, c - Operand<RA>::COPIES);
  };
  // read c of a piece's fragments: those of step 0 first
  auto read_one = [&](const char* st, int f, int c) {
    const int s = c / (NA + NB), k = c % (NA + NB);
    if (k < NB)
      fb[f][s][k] = read_frag<E>(st + RA * PIECE, k, s, lane);
    else
      fa[f][s][k - NB] = read_frag<E>(st, k - NB, s, lane);
  };
  // piece i of the wave.  With one run per wave (fp32) every NW-th piece, past
  // the end of which there is none: two runs' arithmetic between the products cost
  // 6 us of a mid pass's 1640 (B = 256, D = H = 1024, 32 steps)
  auto piece = [&](int i) { return Q == 1 ? runs.first[0] + i * runs.stride : runs.at(i); };
  const int total = ((runs.cnt[0] + 1) & ~1) + runs.cnt[1];
  if (total <= 0) return;
#pragma unroll
  for (int s = 0; s < NST; ++s) {
    const int u = piece(s);
#pragma unroll
    for (int c = 0; c < COPIES; ++c) issue_one(u, s * STAGE, c);
  }
  dma::vm_wait<(NST - 1) * COPIES>();
#pragma unroll
  for (int c = 0; c < READS; ++c) read_one(mine, 0, c);
  int st = 0;  // byte offset of piece i's stage
  dma::unroll<0, Q>([&](auto QI) {
    constexpr int q = decltype(QI)::value;
    auto product = [&](int f, int m) {
      const int s = m / (NA * NB), a = m / NB % NA, b = m % NB;
      F::mma(fa[f][s][a], fb[f][s][b], acc[q][a][b]);
    };
    auto step = [&](int i, auto FI) {
      constexpr int f = decltype(FI)::value;
      const int nx = st + STAGE == NST * STAGE ? 0 : st + STAGE;
      const int u = piece(i + NST);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // piece i is read out: its stage is free
      __builtin_amdgcn_sched_barrier(0);
      dma::unroll<0, HALF>([&](auto M) {
        constexpr int m = decltype(M)::value;
        product(f, m);
        dma::unroll<m * COPIES / HALF, (m + 1) * COPIES / HALF>([&](auto C) { issue_one(u, st, decltype(C)::value); });
        __builtin_amdgcn_sched_barrier(0);
      });
      dma::vm_wait<(NST - 1) * COPIES>();  // piece i + 1 has landed
      const char* np = mine + nx;
      dma::unroll<0, HALF>([&](auto M) {
        constexpr int m = decltype(M)::value;
        product(f, HALF + m);
        dma::unroll<m * READS / HALF, (m + 1) * READS / HALF>([&](auto C) { read_one(np, f ^ 1, decltype(C)::value); });
        __builtin_amdgcn_sched_barrier(0);
      });
      st = nx;
    };
    // (an odd count takes one piece of zeros more: a tail of its own would
    // cost accumulator moves in every iteration)
    const int i0 = q == 0 ? 0 : (runs.cnt[0] + 1) & ~1;
    for (int i = i0; i < i0 + runs.cnt[q]; i += 2) {
      step(i, std::integral_constant<int, 0>{});
      step(i + 1, std::integral_constant<int, 1>{});
    }
  });
  dma::vm_wait<0>();  // no copy outlives the loop
}

template <typename A, int Q, int NA, int NB>
__device__ __forceinline__ void zero_acc(A (&acc)[Q][NA][NB]) {
#pragma unroll
  for (int q = 0; q < Q; ++q)
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[q][a][b] = A{};
}

// Leaves the accumulators of the wave's runs below S in red [S][RA][PITCH].
template <typename E, int RA, int PITCH, int Q, int NA, int NB>
__device__ __forceinline__ void park(const typename Frag<E>::acc_t (&acc)[Q][NA][NB], float* red, int S, int wave,
                                     int lane) {
  typedef Frag<E> F;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int sp = wave + q * NW;
    if (sp >= S) continue;
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int e = 0; e < F::N; ++e) {
          const int row = F::R * a + F::row(e, lane);
          if (row < RA) red[(sp * RA + row) * PITCH + F::R * b + (lane & (F::R - 1))] = acc[q][a][b][e];
        }
  }
}

// s + the first S of the MAXS partial sums of (row, col), in order (all are
// read, so no read waits behind a branch; those from S on are not used).
template <int MAXS, int RA, int PITCH>
__device__ __forceinline__ float gather(float s, const float* red, int S, int row, int col) {
  float v[MAXS];
#pragma unroll
  for (int w = 0; w < MAXS; ++w) v[w] = red[(w * RA + row) * PITCH + col];
#pragma unroll
  for (int w = 0; w < MAXS; ++w) s = w < S ? s + v[w] : s;
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

// Stages per wave for ROWS stage rows of both operands.
template <int ROWS>
constexpr int stages() {
  constexpr int lds = 160 * 1024 / (NW * ROWS * PIECE);
  constexpr int wait = 63 / (ROWS / RPC) + 1;  // (NST - 1) stages' copies within vmcnt's range
  constexpr int fit = lds < wait ? lds : wait;
  return fit < 6 ? fit : 6;
}

// LDS bytes of the four rings, or of the partial sums of Q runs per wave.
template <int RA, int RB, int NST, int PITCH, int Q>
constexpr size_t smem_bytes() {
  constexpr size_t ring = static_cast<size_t>(NW) * NST * (RA + RB) * PIECE;
  constexpr size_t red = sizeof(float) * NW * Q * RA * PITCH;
  return ring > red ? ring : red;
}

// Read (with stride 0) where there are no reset flags.
__device__ const uint8_t kNoReset = 0;

// Forward step.  Grid: cdiv(B, ROWS) * (H / 16) blocks.  S partial sums of
// kps pieces each (bf16), or S = 0 (fp32).
template <typename E, int ROWS>
__global__ void __launch_bounds__(NT, 1) lstm_step_fwd(int B, int D, int H, int S, int kps, const E* __restrict__ x,
                                                       const E* __restrict__ h_prev, const E* __restrict__ Wx,
                                                       const E* __restrict__ Wh, const float* __restrict__ bias,
                                                       const float* __restrict__ c_prev,
                                                       const uint8_t* __restrict__ reset_t, E* __restrict__ h_out,
                                                       float* __restrict__ c_out, E* __restrict__ gates_out) {
  constexpr int COLS = 4 * UNITS, PITCH = COLS + 4;
  constexpr int Q = sizeof(E) == 2 ? 2 : 1;
  constexpr int EPT = ROWS * UNITS / NT;  // elements per thread
  constexpr int NST = stages<ROWS + COLS>();
  __shared__ __attribute__((aligned(1024))) char smem[smem_bytes<ROWS, COLS, NST, PITCH, Q>()];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int rb, cb;
  tile_of(blockIdx.x, (B + ROWS - 1) / ROWS, H / UNITS, rb, cb);
  const int m0 = rb * ROWS, u0 = cb * UNITS;
  constexpr int EPP = PIECE / sizeof(E);
  const uint32_t ldx = D * sizeof(E), ldh = H * sizeof(E);
  const int n = (D + H) / EPP;

  Operand<ROWS> oa;
  Operand<COLS> ob;
  oa.init(x, h_prev, B, ldx, ldh, D / EPP, n, lane, [&](int r, bool& masked) {
    const int row = m0 + r;
    masked = reset_t != nullptr && row < B && reset_t[row] != 0;
    return static_cast<uint32_t>(row);
  });
  ob.init(Wx, Wh, 4 * H, ldx, ldh, D / EPP, n, lane,
          [&](int r, bool&) { return static_cast<uint32_t>((r >> 4) * H + u0 + (r & 15)); });
  // what the cell needs, requested ahead of the product
  float cp[EPT], bs[4];
  const int uc = tid & (UNITS - 1);
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const size_t row = min(m0 + (tid >> 4) + i * (NT / UNITS), B - 1);
    cp[i] = c_prev[row * H + u0 + uc];
  }
#pragma unroll
  for (int g = 0; g < 4; ++g) bs[g] = bias[g * H + u0 + uc];

  typename Frag<E>::acc_t acc[Q][ROWS / Frag<E>::R][COLS / Frag<E>::R];
  zero_acc(acc);
  k_loop<E, NST>(oa, ob, runs_of(S, kps, n, wave), smem, wave, lane, acc);
  float* red = reinterpret_cast<float*>(smem);
  __syncthreads();  // every wave is done with its ring
  const int sums = Q == 1 ? NW : S;
  park<E, ROWS, PITCH>(acc, red, sums, wave, lane);
  __syncthreads();

#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int r = (tid >> 4) + i * (NT / UNITS);
    const int row = m0 + r;
    if (row >= B) continue;
    float p[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) p[g] = gather<Q * NW, ROWS, PITCH>(bs[g], red, sums, r, g * UNITS + uc);
    const float cpv = (reset_t != nullptr && reset_t[row] != 0) ? 0.0f : cp[i];
    const float ig = sigmoid_f(p[0]), fg = sigmoid_f(p[1]), gg = tanh_f(p[2]), og = sigmoid_f(p[3]);
    const float c = fg * cpv + ig * gg;
    const float h = og * tanh_f(c);
    const size_t hj = static_cast<size_t>(row) * H + u0 + uc;
    c_out[hj] = c;
    h_out[hj] = elem<E>::from_f32(h);
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
// Grid: (time-padded rows / T) * (H / T) blocks of T x T; a block past B
// writes the zeros of its padding columns.  Partial column sums of dG go to
// row rb * T / 32 of db_part (one row per 32 batch rows).  S, kps as in the
// forward step.
template <typename E, int T>
__global__ void __launch_bounds__(NT, 1) lstm_step_bwd(
    int B, int Bp, int H, int S, int kps, const E* __restrict__ P, const E* __restrict__ Wf, int K0,
    const E* __restrict__ dG_next, const E* __restrict__ WhT, const uint8_t* __restrict__ reset_next, const float* __restrict__ dh_t,
    const float* __restrict__ dh_extra, const float* dc_in, float* dc_out, const E* __restrict__ gates_t,
    const float* __restrict__ c_t, const float* __restrict__ c_prev, const uint8_t* __restrict__ reset_t,
    E* __restrict__ dG_t, float* __restrict__ db_part, int db_accumulate, E* __restrict__ dGT, size_t ldt, int col0) {
  constexpr int PITCH = T + 4;
  constexpr int Q = sizeof(E) == 2 ? 2 : 1;
  // Row groups: a thread takes EPT rows of one column.  In bf16 adjacent ones,
  // whose dG pairs up as in lstm_bwd_cell (the same column sums); in fp32 every
  // RG-th, so that a batch smaller than the tile is spread over the groups (a
  // tiny optimizer step, 8 rows: 259 us against 277 with adjacent rows).
  constexpr int RG = NT / T;
  constexpr int EPT = T / RG;
  constexpr bool kPairs = sizeof(E) == 2;
  constexpr int PER_SUM = kPairs ? 2 : 32 / RG;  // rows of a thread in one partial column sum
  constexpr int SLOTS = 32 / PER_SUM;            // such sums per 32 rows
  constexpr int TP = T + 8;    // row pitch of the transposed tile (bf16)
  static_assert(T % 32 == 0 && EPT % PER_SUM == 0 && 4 * T <= NT, "whole rows of db_part, whole sums, a thread per sum");
  constexpr int NST = stages<2 * T>();
  constexpr size_t SMEM = smem_bytes<T, T, NST, PITCH, Q>();
  constexpr size_t SUMS = sizeof(float) * (T / 32) * SLOTS * 4 * T;
  constexpr size_t TQ = sizeof(E) == 2 ? sizeof(uint16_t) * 4 * T * TP : 0;
  static_assert(SUMS + TQ <= SMEM, "the epilogue's arrays reuse the ring");
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];
  float* red = reinterpret_cast<float*>(smem);
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int rb, cb;
  tile_of(blockIdx.x, Bp / T, H / T, rb, cb);
  const int m0 = rb * T, j0 = cb * T;
  const int G = 4 * H;

  typename Frag<E>::acc_t acc[Q][T / Frag<E>::R][T / Frag<E>::R];
  zero_acc(acc);
  if (m0 < B) {
    constexpr int EPP = PIECE / sizeof(E);
    const uint32_t ld0 = K0 * sizeof(E), ld1 = G * sizeof(E);
    const int n = (K0 + (dG_next != nullptr ? G : 0)) / EPP;
    Operand<T> oa, ob;
    oa.init(P, dG_next, B, ld0, ld1, K0 / EPP, n, lane, [&](int r, bool& masked) {
      const int row = m0 + r;
      masked = reset_next != nullptr && row < B && reset_next[row] != 0;
      return static_cast<uint32_t>(row);
    });
    ob.init(Wf, WhT, H, ld0, ld1, K0 / EPP, n, lane, [&](int r, bool&) { return static_cast<uint32_t>(j0 + r); });
    k_loop<E, NST>(oa, ob, runs_of(S, kps, n, wave), smem, wave, lane, acc);
  }

  // the cell's inputs, requested before the partial sums meet
  const int jc = tid % T, rg = tid / T;
  const int j = j0 + jc;
  auto row_of = [&](int i) { return kPairs ? rg * EPT + i : rg + i * RG; };
  float dhv[EPT], exv[EPT], dcv[EPT], ctv[EPT], cpv[EPT], gin[EPT][4];
  bool rt[EPT];
  // (absent reset flags read a zero byte: behind a branch each flag's load was
  // waited for before the next row's loads went out, 0.5 us a step)
  const uint8_t* rtp = reset_t != nullptr ? reset_t : &kNoReset;
  const int rts = reset_t != nullptr ? 1 : 0;
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int bc = min(m0 + row_of(i), B - 1);
    const size_t hj = static_cast<size_t>(bc) * H + j;
    const size_t gj = static_cast<size_t>(bc) * G + j;
    dhv[i] = dh_t != nullptr ? dh_t[hj] : 0.0f;
    exv[i] = dh_extra != nullptr ? dh_extra[hj] : 0.0f;
    dcv[i] = dc_in != nullptr ? dc_in[hj] : 0.0f;
#pragma unroll
    for (int g = 0; g < 4; ++g) gin[i][g] = elem<E>::to_f32(gates_t[gj + g * static_cast<size_t>(H)]);
    ctv[i] = c_t[hj];
    cpv[i] = c_prev[hj];
    rt[i] = rtp[bc * rts] != 0;
  }
  __syncthreads();  // every wave is done with its ring
  const int sums_n = Q == 1 ? NW : S;
  park<E, T, PITCH>(acc, red, sums_n, wave, lane);
  __syncthreads();
  float rec[EPT];
#pragma unroll
  for (int i = 0; i < EPT; ++i) rec[i] = gather<Q * NW, T, PITCH>(0.0f, red, sums_n, row_of(i), jc);
  __syncthreads();  // the partial sums' memory is free

  float* sums = reinterpret_cast<float*>(smem);             // [T / 32][SLOTS][4][T]
  uint16_t* tq = reinterpret_cast<uint16_t*>(smem + SUMS);  // [4 T][TP]
  float sd[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int r = row_of(i), b = m0 + r;
    float d[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (b < B) {
      float dh = dhv[i];
      if (dh_extra != nullptr) dh = dh + exv[i];
      dh = dh + rec[i];
      const float ig = gin[i][0], fg = gin[i][1], gg = gin[i][2], og = gin[i][3];
      const float tc = tanh_f(ctv[i]);
      const float dc = dcv[i] + dh * og * (1.0f - tc * tc);
      d[0] = dc * gg * ig * (1.0f - ig);
      d[1] = dc * (rt[i] ? 0.0f : cpv[i]) * fg * (1.0f - fg);
      d[2] = dc * ig * (1.0f - gg * gg);
      d[3] = dh * tc * og * (1.0f - og);
      dc_out[static_cast<size_t>(b) * H + j] = rt[i] ? 0.0f : dc * fg;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        dG_t[static_cast<size_t>(b) * G + g * static_cast<size_t>(H) + j] = elem<E>::from_f32(d[g]);
        sd[g] += d[g];
      }
    }
    if constexpr (sizeof(E) == 2) {
#pragma unroll
      for (int g = 0; g < 4; ++g) tq[(g * T + jc) * TP + r] = f32_to_bf16_bits(d[g]);
    }
    if (i % PER_SUM == PER_SUM - 1) {  // the rows of a partial sum are done
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        sums[((kPairs ? r >> 1 : (r >> 5) * SLOTS + rg) * 4 + g) * T + jc] = sd[g];
        sd[g] = 0.0f;
      }
    }
  }
  __syncthreads();
  if (tid < 4 * T) {
    const int g = tid / T, jl = tid % T;
#pragma unroll
    for (int k = 0; k < T / 32; ++k) {
      float s = 0.0f;
#pragma unroll
      for (int q = 0; q < SLOTS; ++q) s += sums[((k * SLOTS + q) * 4 + g) * T + jl];
      float* p = db_part + static_cast<size_t>(m0 / 32 + k) * G + g * static_cast<size_t>(H) + j0 + jl;
      *p = db_accumulate ? *p + s : s;  // the same block owns this entry at every step
    }
  }
  if constexpr (sizeof(E) == 2) {
    constexpr int CPT = T / 8;  // 16-byte pieces per transposed row
    for (int e = tid; e < 4 * T * CPT; e += NT) {
      const int u = e / CPT, c = e % CPT;
      const uint4 v = *reinterpret_cast<const uint4*>(tq + u * TP + 8 * c);
      *reinterpret_cast<uint4*>(dGT + (static_cast<size_t>(u / T) * H + j0 + u % T) * ldt + col0 + m0 + 8 * c) = v;
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

// Rows per block of the forward step: the tallest tile that still gives every
// CU a block (a taller tile reads the weights fewer times).
template <typename E>
inline int step_fwd_rows(int B, int H) {
  for (int rows = 64; rows > step::Frag<E>::R; rows /= 2)
    if (static_cast<long long>((B + rows - 1) / rows) * (H / step::UNITS) >= 256) return rows;
  return step::Frag<E>::R;
}

// S, kps: the K split of the separate product (bf16), 0 in fp32.
template <typename E>
inline void launch_step_fwd(int B, int D, int H, int S, int kps, const E* x, const E* h_prev, const E* Wx, const E* Wh,
                            const float* bias, const float* c_prev, const uint8_t* reset_t, E* h, float* c, E* gates,
                            hipStream_t s) {
  const int rows = step_fwd_rows<E>(B, H);
  auto kernel = rows == 64 ? step::lstm_step_fwd<E, 64> : step::lstm_step_fwd<E, 32>;
  if constexpr (sizeof(E) == 4)
    if (rows == 16) kernel = step::lstm_step_fwd<E, 16>;
  const unsigned blocks = static_cast<unsigned>((B + rows - 1) / rows) * (H / step::UNITS);
  hipLaunchKernelGGL(kernel, dim3(blocks), dim3(step::NT), 0, s, B, D, H, S, kps, x, h_prev, Wx, Wh, bias, c_prev,
                     reset_t, h, c, gates);
}

}  // namespace o5
