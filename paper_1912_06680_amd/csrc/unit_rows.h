// The loss rows of a batch with a unit-selection head, in one pass over the
// unit embeddings: the head's logits <q, E[n, u]>, every head's softmax, the
// PPO row, dL/dz, and dq = sum_u dz_u E[n, u].
//
// Bound by the embeddings (N nk d elements; 464 MB of the 566 MB that a call
// must move at N = 9600, nk = 189, d = 128 in bf16): a block takes one row at a
// time and every thread keeps its 16-byte chunks of E[n] in registers from the
// logits to dq, so the row is read once.  Chunks t, t + 256, ... of the row
// belong to thread t, so its position t % (d / 8) within a unit never changes
// and the d / 8 chunks of a unit sit on consecutive lanes.  What a row costs is
// latency (a chain of loads, reductions and six barriers), so registers decide:
// 127 with 12 chunks of bf16 let 4 blocks share a CU.  With the chunks' fp32
// values kept from the logits to dq it took 231 registers, 2 blocks and 259 us;
// now 124 us (3.8 TB/s of embeddings) at the sizes above, against 265 us for the
// three kernels it replaces (logits 109, rows 55, dq 101).  Each block walks rows
// n, n + grid, ... and keeps its column sums in registers.
#pragma once

#include "heads.h"
#include "reduce.h"

namespace o5 {

constexpr int kUrThreads = 256;
constexpr int kUrMaxD = 512;
constexpr int kUrStat = 8;

// 16 bytes of a buffer; beyond its end they read as 0.
template <typename V>
__device__ __forceinline__ V buffer16(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}

// 8 consecutive embedding values, held as loaded.
template <typename E>
struct Chunk8;
template <>
struct Chunk8<uint16_t> {
  uint4 v;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, int off) { v = buffer16<uint4>(r, off); }
  // Makes the converted values of get() before and after it separate, so that
  // the chunk stays in its 4 registers in between.
  __device__ __forceinline__ void keep() { asm("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w)); }
  __device__ __forceinline__ void get(float (&f)[8]) const {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      f[2 * k] = __uint_as_float(w[k] << 16);
      f[2 * k + 1] = __uint_as_float(w[k] & 0xffff0000u);
    }
  }
};
template <>
struct Chunk8<float> {
  float4 a, b;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, int off) {
    a = buffer16<float4>(r, off);
    b = buffer16<float4>(r, off + 16);
  }
  __device__ __forceinline__ void keep() {}
  __device__ __forceinline__ void get(float (&f)[8]) const {
    f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
    f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
  }
};

struct UnitRowsArgs {
  int N, A1, S, Sq, d, dp, kext;  // S, Sq: partial sums of the logits and the query
  const float* zpart;             // [S][N][A1]
  const float* bp;
  const float* qpart;  // [Sq][N][d]
  const float* bq;
  const int32_t* act;
  const float* logp_old;
  const float* adv;
  const float* ret;
  const uint8_t* mask;
  const uint8_t* avail;
  HeadsMeta hm;
  float clip_eps, vf_coef, ent_coef, invN;
  float* dz;        // fp32: [N][A1], and dq [N][d]
  float* dq;
  uint16_t* pair;   // bf16: row n = [hi (ldh) | lo (ldh)]: A1p columns of dz, then dp of dq
  int A1p, ldh;
  float* part;      // [grid][A1 + kUrStat + d] column sums of dz, row statistics, column sums of dq
};

__device__ __forceinline__ void store_pair(uint16_t* row, int ldh, int c, float v) {
  const uint16_t hb = f32_to_bf16_bits(v);
  row[c] = hb;
  row[ldh + c] = f32_to_bf16_bits(v - bf16_bits_to_f32(hb));
}

template <int N, typename F>
__device__ __forceinline__ void each(F f) {
#pragma unroll
  for (int i = 0; i < N; ++i) f(i);
}

// Waves per SIMD that a chunk array of this size leaves room for.
constexpr int ur_waves(int regs) { return regs <= 48 ? 4 : regs <= 64 ? 3 : 2; }

// CH: chunks per thread, at least nk (d / 8) / 256; CPT, DPT: logit columns
// and embedding columns per thread.
template <typename E, int CH, int CPT, int DPT>
__global__ void __launch_bounds__(kUrThreads, ur_waves(CH * static_cast<int>(sizeof(E)) * 2 + (CPT > 1 ? 16 : 0)))
    unit_rows(UnitRowsArgs g, const E* __restrict__ emb) {
  constexpr int NWV = kUrThreads / 64;
  __shared__ float zs[kMaxA1];  // logits, then dL/dz
  __shared__ uint8_t avs[kMaxA1];
  __shared__ float qs[kUrMaxD], dqr[NWV][kUrMaxD], st[kUrStat];  // st: thread 0's
  __shared__ float hd_mx[kMaxHeads], hd_inv[kMaxHeads], hd_zbar[kMaxHeads], hd_lp[kMaxHeads], hd_ent[kMaxHeads];
  __shared__ int hd_act[kMaxHeads], hd_use[kMaxHeads];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int A1 = g.A1, A = g.hm.A, K = g.hm.K, d = g.d;
  const int e0 = g.hm.off[g.kext], nk = g.hm.off[g.kext + 1] - e0;
  const int C = d >> 3, jc = t & (C - 1), lc = __builtin_ctz(C);
  const int chunks = nk << lc;
  const size_t zstride = static_cast<size_t>(g.N) * A1, qstride = static_cast<size_t>(g.N) * d;
  const int W = A1 + kUrStat + d;
  // the head of each column this thread owns (t, t + 256, ...); -1: the value
  // column and beyond
  int head[CPT];
#pragma unroll
  for (int i = 0; i < CPT; ++i) {
    const int c = t + i * kUrThreads;
    head[i] = -1;
    for (int k = 0; k < K; ++k)
      if (c >= g.hm.off[k] && c < g.hm.off[k + 1]) head[i] = k;
  }
  float csum[CPT] = {}, qsum[DPT] = {};
  if (t < kUrStat) st[t] = 0.0f;

  for (int n = blockIdx.x; n < g.N; n += gridDim.x) {
    // (chunks past the row's end read as 0)
    const __amdgpu_buffer_rsrc_t row = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<E*>(emb + static_cast<size_t>(n) * nk * d), 0, chunks * 8 * static_cast<int>(sizeof(E)), 0x00020000);
    Chunk8<E> ch[CH];
#pragma unroll
    for (int i = 0; i < CH; ++i) ch[i].load(row, (t + i * kUrThreads) * 8 * static_cast<int>(sizeof(E)));
    // (the head this wave takes first; read here, used after two barriers)
    const int act0 = wave < K ? g.act[static_cast<size_t>(n) * K + wave] : 0;
    const float lpo = g.logp_old[n], Ad = g.adv[n], R = g.ret[n];
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int c = t + i * kUrThreads;
      if (c < A1 && head[i] != g.kext) {
        zs[c] = add_parts<4>(g.bp[c], g.zpart + static_cast<size_t>(n) * A1 + c, g.S, zstride);
      }
      if (c < A) avs[c] = g.avail != nullptr ? g.avail[static_cast<size_t>(n) * A + c] : static_cast<uint8_t>(1);
    }
#pragma unroll
    for (int i = 0; i < DPT; ++i) {
      const int j = t + i * kUrThreads;
      if (j < d) {
        qs[j] = add_parts<4>(g.bq[j], g.qpart + static_cast<size_t>(n) * d + j, g.Sq, qstride);
      }
    }
    __syncthreads();
    {  // the unit head's logits
      float qv[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) qv[k] = qs[jc * 8 + k];
      float s[CH];
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        float f[8];
        ch[i].get(f);
        ch[i].keep();
        s[i] = 0.0f;
#pragma unroll
        for (int k = 0; k < 8; ++k) s[i] += qv[k] * f[k];
      }
      // the unit's C lanes: swaps within 4, then within the 16 of a row, then across rows
      if (C > 1) each<CH>([&](int i) { s[i] += dpp<0xB1>(0.0f, s[i]); });
      if (C > 2) each<CH>([&](int i) { s[i] += dpp<0x4E>(0.0f, s[i]); });
      if (C > 4) each<CH>([&](int i) { s[i] += dpp<0x141>(0.0f, s[i]); });   // row_half_mirror
      if (C > 8) each<CH>([&](int i) { s[i] += dpp<0x140>(0.0f, s[i]); });   // row_mirror
      if (C > 16) each<CH>([&](int i) { s[i] += __shfl_xor(s[i], 16, 64); });
      if (C > 32) each<CH>([&](int i) { s[i] += __shfl_xor(s[i], 32, 64); });
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        const int c = t + i * kUrThreads;
        if (c < chunks && jc == 0) zs[e0 + (c >> lc)] = s[i];
      }
    }
    __syncthreads();
    // heads: wave w takes heads w, w + 4, ..., lanes over the head's columns
    for (int k = wave; k < K; k += NWV) {
      const int o = g.hm.off[k], n_k = g.hm.off[k + 1] - o;
      float m = -INFINITY;
#pragma unroll 1
      for (int a = lane; a < n_k; a += 64)
        if (avs[o + a]) m = fmaxf(m, zs[o + a]);
      m = wave_max(m);
      float se = 0.0f, sz = 0.0f;
#pragma unroll 1
      for (int a = lane; a < n_k; a += 64)
        if (avs[o + a]) {
          const float z = zs[o + a], e = expf(z - m);
          se += e;
          sz += e * z;
        }
      se = wave_sum(se);
      sz = wave_sum(sz);
      const bool some = se > 0.0f;  // the maximum contributes e = 1
      const float lse = some ? m + logf(se) : 0.0f, zb = some ? sz / se : 0.0f;
      const int ak = k == wave ? act0 : g.act[static_cast<size_t>(n) * K + k];
      const bool use = some && (g.mask == nullptr || g.mask[static_cast<size_t>(n) * K + k] != 0);
      const int sel = o + min(max(ak, 0), n_k - 1);
      if (lane == 0) {
        hd_mx[k] = m;
        hd_inv[k] = some ? 1.0f / se : 0.0f;
        hd_zbar[k] = zb;
        hd_lp[k] = use ? (avs[sel] ? zs[sel] - lse : -INFINITY) : 0.0f;
        hd_ent[k] = use ? lse - zb : 0.0f;
        hd_act[k] = o + ak;
        hd_use[k] = use;
      }
    }
    __syncthreads();
    // the row, by every thread alike
    float logpi = 0.0f, ent = 0.0f;
#pragma unroll 1
    for (int k = 0; k < K; ++k)
      if (hd_use[k]) {
        logpi += hd_lp[k];
        ent += hd_ent[k];
      }
    const float dlog = logpi - lpo;
    const float ratio = expf(dlog);
    const float rc = fminf(fmaxf(ratio, 1.0f - g.clip_eps), 1.0f + g.clip_eps);
    const float surr = fminf(ratio * Ad, rc * Ad);
    const float verr = zs[A] - R;
    const bool flow = (Ad >= 0.0f && ratio <= 1.0f + g.clip_eps) || (Ad < 0.0f && ratio >= 1.0f - g.clip_eps);
    const float gl = flow ? -ratio * Ad * g.invN : 0.0f;
    const float es = g.ent_coef * g.invN;
    if (t == 0) {
      const float row_loss = -surr + g.vf_coef * verr * verr - g.ent_coef * ent;
      st[0] += surr;
      st[1] += verr * verr;
      st[2] += ent;
      st[3] += fabsf(ratio - 1.0f) > g.clip_eps ? 1.0f : 0.0f;
      st[4] += expm1f(dlog) - dlog;  // (r - 1) - log r without the cancellation in r - 1
      st[5] += ratio;
      st[6] += isfinite(row_loss) ? 0.0f : 1.0f;
    }
    __syncthreads();  // every thread has read the value's logit
    uint16_t* prow = g.pair != nullptr ? g.pair + static_cast<size_t>(n) * 2 * g.ldh : nullptr;
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int c = t + i * kUrThreads;
      const int k = head[i];
      float v = 0.0f;
      if (c == A) v = 2.0f * g.vf_coef * verr * g.invN;
      if (k >= 0 && hd_use[k] && avs[c]) {
        const float z = zs[c];
        const float p = expf(z - hd_mx[k]) * hd_inv[k];
        v = gl * ((c == hd_act[k] ? 1.0f : 0.0f) - p) + es * p * (z - hd_zbar[k]);
      }
      if (k >= 0 && k == g.kext) {
        zs[c] = v;
        v = 0.0f;  // these logits do not depend on Wp, bp
      }
      csum[i] += v;
      if (c < A1 && g.dz != nullptr) g.dz[static_cast<size_t>(n) * A1 + c] = v;
      if (prow != nullptr && c < g.A1p) store_pair(prow, g.ldh, c, v);
    }
    __syncthreads();
    {  // dq: this thread's chunk over the units it holds, then the wave's, then the block's
      float acc[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        const int c = t + i * kUrThreads;
        const float gz = c < chunks ? zs[e0 + (c >> lc)] : 0.0f;
        float f[8];
        ch[i].get(f);
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] += gz * f[k];
      }
      for (int w = C; w < 64; w <<= 1)
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] += __shfl_xor(acc[k], w, 64);
      if (lane < C) {
#pragma unroll
        for (int k = 0; k < 8; ++k) dqr[wave][jc * 8 + k] = acc[k];
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < DPT; ++i) {
      const int j = t + i * kUrThreads;
      float v = 0.0f;
      if (j < d) {
#pragma unroll
        for (int w = 0; w < NWV; ++w) v += dqr[w][j];
        qsum[i] += v;
        if (g.dq != nullptr) g.dq[static_cast<size_t>(n) * d + j] = v;
      }
      if (prow != nullptr && j < g.dp) store_pair(prow, g.ldh, g.A1p + j, v);
    }
  }
  float* part = g.part + static_cast<size_t>(blockIdx.x) * W;
#pragma unroll
  for (int i = 0; i < CPT; ++i)
    if (t + i * kUrThreads < A1) part[t + i * kUrThreads] = csum[i];
  if (t == 0) {
    for (int q = 0; q < kUrStat; ++q) part[A1 + q] = st[q];
  }
#pragma unroll
  for (int i = 0; i < DPT; ++i)
    if (t + i * kUrThreads < d) part[A1 + kUrStat + t + i * kUrThreads] = qsum[i];
}

// Blocks: at most four per CU.
inline int unit_rows_grid(int N) { return N < 1024 ? N : 1024; }

// Chunks per thread that a row of nk units of width d needs; a row that needs
// more than 16 takes the two-pass kernels of unit.hip.
inline int unit_rows_chunks(int nk, int d) { return (nk * (d / 8) + kUrThreads - 1) / kUrThreads; }
inline bool unit_rows_fits(int nk, int d) { return unit_rows_chunks(nk, d) <= 16; }

template <typename E, int CH>
inline void launch_unit_rows_c(const UnitRowsArgs& g, const E* emb, hipStream_t s) {
  const dim3 grid(unit_rows_grid(g.N)), block(kUrThreads);
  if (g.A1p <= kUrThreads && g.d <= kUrThreads)  // one column per thread: fewer registers
    hipLaunchKernelGGL((unit_rows<E, CH, 1, 1>), grid, block, 0, s, g, emb);
  else
    hipLaunchKernelGGL((unit_rows<E, CH, kMaxA1 / kUrThreads, kUrMaxD / kUrThreads>), grid, block, 0, s, g, emb);
}

template <typename E>
inline void launch_unit_rows(const UnitRowsArgs& g, const E* emb, int nk, hipStream_t s) {
  const int ch = unit_rows_chunks(nk, g.d);
  if (ch <= 4)
    launch_unit_rows_c<E, 4>(g, emb, s);
  else if (ch <= 12)
    launch_unit_rows_c<E, 12>(g, emb, s);
  else
    launch_unit_rows_c<E, 16>(g, emb, s);
}

}  // namespace o5
