// The probe linear (Sec. 3.2) and the fused head scoring (Sec. 3.3) for fp32 operands, on the fp32 matrix
// instruction (v_mfma_f32_16x16x4_f32: fp32 products and sums throughout).
//
// fp32 calls are small (the 256-wide configuration at 768 rows is typical), so a call is bound by the latency of
// its launches and of the loads inside them: one preparation launch, one for the side columns, one for the
// products; operands are requested a whole K slab (64 or 128 columns) at a time, and the tiles shrink until the
// chip has work.  At 768 x 256 x 256 (r = 4) and a 512-row head, on the vector ALU before -> now (kernel trace): side
// columns 28 -> 7 us, products 42 -> 7, head 42 -> 8, preparation four launches -> one; linear and scoring 134 -> 31.
//
// An output element is summed in an order that depends on the input width alone, so its bits do not depend on
// the batch, the tile size or the load width.
#include "zo_device.hpp"
#include "zo_internal.hpp"

namespace zo {
namespace {

// acc = A[m0 ..][:] B[t0 ..][:]^T for a TM x TN tile, WR x WC waves.  MFMA rows are the rows of A (output features,
// vocabulary), MFMA columns the rows of B (tokens): lane l holds rows 4*(l/16) + v of column l%16.  A lane reads
// four neighbouring k-values of its row at once (16 bytes) and hands them to four instructions, so k-values
// {i, 4+i, 8+i, 12+i} of a block of 16 meet in instruction i.  LDS rows are padded by 16 bytes: the 16 rows of a
// fragment read fall on different banks.
// kVec: rows and K come in whole aligned groups of four (16-byte loads); otherwise element by element.
template <int TM, int TN, int WR, int WC, int KC>
struct TileF32 {
  static constexpr int kThreads = WR * WC * 64;
  static constexpr int RB = TM / WR / 16, CB = TN / WC / 16;
  static constexpr int kPitch = KC + 4;
  static constexpr int kLdsFloats = (TM + TN) * kPitch;
  static constexpr int kQuads = (TM + TN) * (KC / 4) / kThreads;   // 16-byte pieces of a slab per thread
  static_assert((TM + TN) * (KC / 4) % kThreads == 0, "whole pieces per thread");

  template <bool kVec>
  __device__ static __forceinline__ void multiply(const float* __restrict__ A, int64_t lda, int M, int m0,
                                                  const float* __restrict__ B, int64_t ldb, int N, int n0, int K,
                                                  float* lds, f32x4 (&acc)[RB][CB]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wr = wave / WC, wc = wave % WC;
    f32x4 piece[kQuads];
    auto load = [&](int k0) {
#pragma unroll
      for (int e = 0; e < kQuads; ++e) {
        const int q = tid + e * kThreads;
        const int row = q / (KC / 4), k = k0 + (q % (KC / 4)) * 4;
        const bool isA = row < TM;
        const int r = isA ? m0 + row : n0 + row - TM;
        const float* src = isA ? A + (int64_t)r * lda : B + (int64_t)r * ldb;
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        if (r < (isA ? M : N)) {
          if constexpr (kVec) {
            if (k < K) v = *reinterpret_cast<const f32x4*>(src + k);
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (k + i < K) v[i] = src[k + i];
          }
        }
        piece[e] = v;
      }
    };
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) acc[rb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float* fragA = lds + (wr * (TM / WR) + (lane & 15)) * kPitch + (lane >> 4) * 4;
    const float* fragB = lds + (TM + wc * (TN / WC) + (lane & 15)) * kPitch + (lane >> 4) * 4;
    load(0);
    for (int k0 = 0; k0 < K; k0 += KC) {
      if (k0 > 0) __syncthreads();   // every wave is done with the previous slab
#pragma unroll
      for (int e = 0; e < kQuads; ++e) {
        const int q = tid + e * kThreads;
        *reinterpret_cast<f32x4*>(lds + (q / (KC / 4)) * kPitch + (q % (KC / 4)) * 4) = piece[e];
      }
      __syncthreads();
      if (k0 + KC < K) load(k0 + KC);   // the next slab travels under this one's products
#pragma unroll
      for (int kb = 0; kb < KC / 16; ++kb) {
        if (k0 + kb * 16 >= K) break;
        f32x4 a[RB], b[CB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) a[rb] = *reinterpret_cast<const f32x4*>(fragA + rb * 16 * kPitch + kb * 16);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) b[cb] = *reinterpret_cast<const f32x4*>(fragB + cb * 16 * kPitch + kb * 16);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
              acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[rb][i], b[cb][i], acc[rb][cb], 0, 0, 0);
      }
    }
  }
};

bool whole_quads(const void* a, int64_t lda, const void* b, int64_t ldb, int K) {
  return (((uintptr_t)a | (uintptr_t)b) & 15u) == 0 && lda % 4 == 0 && ldb % 4 == 0 && K % 4 == 0;
}

// Tside[t, :] = [ s_t eps X[t,:] V_{k_t} | X[t,:] Vb ]; zero where the row has no such term.  One wave per (row,
// 8 columns): the lanes share the input columns, then the eight sums are folded across the wave.
__global__ __launch_bounds__(256) void k_side_f32(ProbeF32Args p) {
  const int NC = p.r + p.R;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int j0 = blockIdx.y * 8;
  if (t >= p.T) return;
  const int s = p.tok_seq[t];
  const int kind = p.seq_kind[s];
  const float* x = p.X + (int64_t)t * p.ldx;
  float acc[8] = {};
  // a group of eight may hold direction columns, bank columns, or both
  const float* src[8];
  int64_t pitch[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int j = j0 + e;
    src[e] = nullptr;
    pitch[e] = 0;
    if (j < p.r) {
      if (kind >= 0) { src[e] = p.Vf + (int64_t)kind * p.n * p.r + j; pitch[e] = p.r; }
    } else if (j < NC && kind >= kKindCentre) {
      src[e] = p.Vb + (j - p.r);
      pitch[e] = p.R_cap;
    }
  }
  for (int i = lane; i < p.n; i += 64) {
    const float xi = x[i];
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (src[e]) acc[e] = fmaf(xi, src[e][(int64_t)i * pitch[e]], acc[e]);
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) acc[e] += __shfl_xor(acc[e], o);
  }
  const float scale = kind >= 0 ? p.seq_scale[s] : 0.0f;
#pragma unroll
  for (int e = 0; e < 8; ++e)
    if (lane == e && j0 + e < NC) p.Tside[(int64_t)t * NC + j0 + e] = j0 + e < p.r ? acc[e] * scale : acc[e];
}

template <class C, int TM, int TN, int WC, bool kVec>
__global__ __launch_bounds__(C::kThreads) void k_probe_f32(ProbeF32Args p) {
  __shared__ __attribute__((aligned(16))) float lds[C::kLdsFloats];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m0 = blockIdx.x * TM, t0 = blockIdx.y * TN;
  f32x4 acc[C::RB][C::CB];
  C::template multiply<kVec>(p.W, p.ldw, p.m, m0, p.X, p.ldx, p.T, t0, p.n, lds, acc);
  const int NC = p.r + p.R;
#pragma unroll
  for (int cb = 0; cb < C::CB; ++cb) {
    const int t = t0 + (wave % WC) * (C::CB * 16) + cb * 16 + (lane & 15);
    if (t >= p.T) continue;
    int kind = kKindForeground;
    if (p.has_side) kind = p.seq_kind[p.tok_seq[t]];
#pragma unroll
    for (int rb = 0; rb < C::RB; ++rb) {
      const int o = m0 + (wave / WC) * (C::RB * 16) + rb * 16 + 4 * (lane >> 4);   // four neighbouring features
      if (o >= p.m) continue;
      float y[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = acc[rb][cb][e];
      if (kind >= kKindCentre) {   // foreground rows skip the side state entirely
        const float* ts = p.Tside + (int64_t)t * NC;
        float side[4] = {0.f, 0.f, 0.f, 0.f};
        int64_t at[4];   // rows past the end repeat the last one (not stored)
#pragma unroll
        for (int e = 0; e < 4; ++e) at[e] = min(o + e, p.m - 1);
#pragma unroll 4
        for (int jj = 0; jj < p.R; ++jj) {
          const float x = ts[p.r + jj];
#pragma unroll
          for (int e = 0; e < 4; ++e) side[e] = fmaf(x, p.P[at[e] * p.R_cap + jj], side[e]);
        }
        if (kind >= 0) {
          const float* u = p.Uf + (int64_t)kind * p.m * p.r;
#pragma unroll 4
          for (int jj = 0; jj < p.r; ++jj) {
            const float x = ts[jj];
#pragma unroll
            for (int e = 0; e < 4; ++e) side[e] = fmaf(x, u[at[e] * p.r + jj], side[e]);
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] += side[e];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (p.bias) y[e] += p.bias[min(o + e, p.m - 1)];
        if (p.act == 1) y[e] = fmaxf(y[e], 0.0f);
      }
      if (p.act == 2) {   // (gate, up) pairs of adjacent output features -> one output column each (m is even)
#pragma unroll
        for (int e = 0; e < 4; e += 2)
          if (o + e < p.m) p.Y[(int64_t)t * p.ldy + ((o + e) >> 1)] = y[e] / (1.0f + expf(-y[e])) * y[e + 1];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (o + e < p.m) p.Y[(int64_t)t * p.ldy + o + e] = y[e];
      }
    }
  }
}

// Tokens in groups of TN against 64 vocabulary rows per workgroup; per (vocabulary tile, token): max logit,
// sum exp(z - max) and, where the target falls in the tile, the target logit.
template <class C, int TN, bool kVec>
__global__ __launch_bounds__(C::kThreads) void k_head_f32(HeadScoreF32Args p) {
  constexpr int WR = 4;   // one wave per 16 vocabulary rows, whatever the tile: a token's sums are merged in one order
  __shared__ __attribute__((aligned(16))) float lds[C::kLdsFloats];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4;
  const int v0 = blockIdx.x * kHeadTileF32, t0 = blockIdx.y * TN;
  f32x4 acc[C::RB][C::CB];
  C::template multiply<kVec>(p.Wh, p.ldw, p.vocab, v0, p.H, p.ldh, p.T, t0, p.d, lds, acc);
  __syncthreads();   // the operand slabs are done with: their memory holds the exchange between wave rows now
  float* s_max = lds;              // [WR][TN]
  float* s_sum = lds + WR * TN;    // [WR][TN]
  const int vbase = v0 + wave * (C::RB * 16);
#pragma unroll
  for (int cb = 0; cb < C::CB; ++cb) {
    const int tl = cb * 16 + (lane & 15);
    float mx = -INFINITY;
#pragma unroll
    for (int rb = 0; rb < C::RB; ++rb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (vbase + rb * 16 + 4 * g + v >= p.vocab) acc[rb][cb][v] = -INFINITY;
        mx = fmaxf(mx, acc[rb][cb][v]);
      }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    // (a wave whose rows all lie past the end of the vocabulary has no finite maximum: its sum is zero)
    const float ref = mx == -INFINITY ? 0.0f : mx;
    float sum = 0.0f;
#pragma unroll
    for (int rb = 0; rb < C::RB; ++rb)
#pragma unroll
      for (int v = 0; v < 4; ++v) sum += expf(acc[rb][cb][v] - ref);
    sum += __shfl_xor(sum, 16);
    sum += __shfl_xor(sum, 32);
    if (g == 0) { s_max[wave * TN + tl] = mx; s_sum[wave * TN + tl] = sum; }
    const int t = t0 + tl;
    if (t < p.T) {
      const int loc = p.targets[t] - vbase;
      if (loc >= 0 && loc < C::RB * 16 && ((loc >> 2) & 3) == g) {
        float z = 0.0f;
#pragma unroll
        for (int rb = 0; rb < C::RB; ++rb)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if ((loc >> 4) * 4 + (loc & 3) == rb * 4 + v) z = acc[rb][cb][v];
        p.tgt_logit[t] = z;
      }
    }
  }
  __syncthreads();
  const int t = t0 + threadIdx.x;
  if (threadIdx.x < TN && t < p.T) {
    float M = s_max[threadIdx.x];
#pragma unroll
    for (int w = 1; w < WR; ++w) M = fmaxf(M, s_max[w * TN + threadIdx.x]);
    const float ref = M == -INFINITY ? 0.0f : M;
    float S = 0.0f;
#pragma unroll
    for (int w = 0; w < WR; ++w) S += s_sum[w * TN + threadIdx.x] * expf(s_max[w * TN + threadIdx.x] - ref);
    p.part_max[(int64_t)blockIdx.x * p.T + t] = M;
    p.part_sum[(int64_t)blockIdx.x * p.T + t] = S;
  }
}

int64_t tiles(int rows, int tm, int cols, int tn) { return (int64_t)((rows + tm - 1) / tm) * ((cols + tn - 1) / tn); }

}  // namespace

hipError_t launch_probe_f32(const ProbeF32Args& a, hipStream_t st) {
  if (a.T == 0 || a.m == 0) return hipSuccess;
  if (a.has_side) {
    const hipError_t e = launch_probe_prep_f32(a.batch, a.eps, a.tabs, a.tensor_id, a.m, a.n, a.r, a.Uf, a.Vf, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_side_f32, dim3((a.T + 3) / 4, (a.r + a.R + 7) / 8), dim3(256), 0, st, a);
  }
  const bool vec = whole_quads(a.X, a.ldx, a.W, a.ldw, a.n);
  // 64x64 tiles when they give every compute unit one, 32x32 (a longer K slab, four times the workgroups) otherwise
  if (tiles(a.m, 64, a.T, 64) >= compute_units()) {
    using C = TileF32<64, 64, 2, 2, 64>;
    const dim3 grid((a.m + 63) / 64, (a.T + 63) / 64);
    if (vec) hipLaunchKernelGGL((k_probe_f32<C, 64, 64, 2, true>), grid, dim3(C::kThreads), 0, st, a);
    else hipLaunchKernelGGL((k_probe_f32<C, 64, 64, 2, false>), grid, dim3(C::kThreads), 0, st, a);
  } else {
    using C = TileF32<32, 32, 2, 2, 128>;
    const dim3 grid((a.m + 31) / 32, (a.T + 31) / 32);
    if (vec) hipLaunchKernelGGL((k_probe_f32<C, 32, 32, 2, true>), grid, dim3(C::kThreads), 0, st, a);
    else hipLaunchKernelGGL((k_probe_f32<C, 32, 32, 2, false>), grid, dim3(C::kThreads), 0, st, a);
  }
  return hipGetLastError();
}

int head_vocab_tiles_f32(int vocab) { return (vocab + kHeadTileF32 - 1) / kHeadTileF32; }

hipError_t launch_head_score_f32(const HeadScoreF32Args& a, hipStream_t st) {
  if (a.T == 0) return hipSuccess;
  const bool vec = whole_quads(a.H, a.ldh, a.Wh, a.ldw, a.d);
  static_assert(kHeadTileF32 == 64, "vocabulary rows per workgroup");
  if (tiles(a.vocab, 64, a.T, 64) >= compute_units()) {
    using C = TileF32<64, 64, 4, 1, 64>;
    const dim3 grid((a.vocab + 63) / 64, (a.T + 63) / 64);
    if (vec) hipLaunchKernelGGL((k_head_f32<C, 64, true>), grid, dim3(C::kThreads), 0, st, a);
    else hipLaunchKernelGGL((k_head_f32<C, 64, false>), grid, dim3(C::kThreads), 0, st, a);
  } else {   // fewer tokens per workgroup
    using C = TileF32<64, 16, 4, 1, 128>;
    const dim3 grid((a.vocab + 63) / 64, (a.T + 15) / 16);
    if (vec) hipLaunchKernelGGL((k_head_f32<C, 16, true>), grid, dim3(C::kThreads), 0, st, a);
    else hipLaunchKernelGGL((k_head_f32<C, 16, false>), grid, dim3(C::kThreads), 0, st, a);
  }
  return hipGetLastError();
}

}  // namespace zo
