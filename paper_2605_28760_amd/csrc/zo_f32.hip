// The probe linear (Sec. 3.2) and the fused head scoring (Sec. 3.3) for fp32 operands, on the fp32 matrix
// instruction (v_mfma_f32_16x16x4_f32: fp32 products and sums throughout).
//
// fp32 calls are small (the 256-wide configuration at 768 rows is typical), so a call is bound by the latency of
// its launches and of the loads inside them: the side columns ride along with the products in one launch where they are few,
// and have a preparation launch and one of their own otherwise; operands are requested a whole K slab (64 or 128 columns) at
// a time, and the tiles shrink until the chip has work.  At 768 x 256 x 256 (r = 4) and a 512-row head: probe linear 16.4 us in
// three launches (3, 7 and 7) -> 11 in one, linear and scoring 31 -> 26 (kernel trace; on the vector ALU 134).
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

  // side: what further waves of the workgroup multiply with the rows of B in the same walk over K (SideF32 below, or NoSide:
  // there are none).
  template <bool kVec, class Side>
  __device__ static __forceinline__ void multiply(const float* __restrict__ A, int64_t lda, int M, int m0,
                                                  const float* __restrict__ B, int64_t ldb, int N, int n0, int K,
                                                  float* lds, f32x4 (&acc)[RB][CB], Side& side) {
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
    if constexpr (Side::kWaves > 0) {
      if (wave >= WR * WC) {   // the side waves: a walk of their own through the same barriers
        side.walk(K, lds + TM * kPitch);
        return;
      }
    }
    load(0);
    if constexpr (Side::kWaves > 0) __syncthreads();   // (their tables)
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

struct NoSide {
  static constexpr int kWaves = 0;
};

// The side columns of a tile's tokens, computed by four more waves of the tile's own workgroup: rows of [V_0 | V_1 | .. | Vb]^T,
// 16 to a block, meet the slabs of X that the products use.  V is drawn from its seeds slab by slab (a Philox block holds four
// neighbouring entries of V), Vb is read; a block of the result is X [V or Vb] of the tile's tokens, and a token takes
// the block of its own direction.  The waves of the products are waiting for their operands most of the time (one wave per
// SIMD), so what these waves add is hidden but for their start: done by the same waves it took 12.4 us instead of 11.
constexpr int kFusedBlocks = 3;      // 16-column blocks at most
constexpr int kFusedColumns = 16 * kFusedBlocks;
constexpr int kFusedTable = 1024;    // sequences and candidates at most (their tables sit in LDS)

// LDS of a fused tile, in words: the operand slabs, the side operand's slab, U of the tile's features, the side columns of
// its tokens, the tokens' kinds, the seeds, and the batch's tables.
template <class C, int TM, int TN>
struct FusedLds {
  int rows, u, cols, kinds, seeds, cu, cand, dir, sign, end;
  __host__ __device__ explicit FusedLds(const ProbeF32Args& p) {
    const int K = p.batch.K, blocks = K * ((p.r + 15) / 16) + (p.R + 15) / 16;
    rows = C::kLdsFloats;
    u = rows + blocks * 16 * C::kPitch;
    cols = u + K * TM * p.r;
    kinds = cols + TN * (p.r + p.R);
    seeds = (kinds + TN + 1) & ~1;   // 64-bit: [K] of U, [K] of V
    cu = seeds + 4 * K;
    cand = cu + p.batch.S + 1;
    dir = cand + p.batch.S;
    sign = dir + p.batch.C;
    end = sign + p.batch.C;
  }
};

// Products of 16 side columns and 16 rows of X over the input width: two chains of two instructions (eight products) per 16
// columns, the sums of 32 columns added, and these in double precision.  One chain over the width, the instruction's own accumulation,
// was further from 64-bit sums than a wave's 64 partial sums had been: relative error of the term alone, rank 4, at 64 / 256 / 2048 /
// 16384 columns 0.8, 0.9, 1.3, 3.0e-7 (64 partial sums); 1.5, 2.9, 8.0, 23e-7 (one chain); 0.8e-7 throughout (this).  It costs a
// fused call up to 1.5 %, 0.4 us of 28.  (Every 16 columns in double: no closer, and twice that.  The last columns are
// taken by blocks, as 64 at a time 5285 rows of 81 columns took 0.6 us more, linear and scoring 31.6 instead of 31.0.)
template <int kTogether>   // blocks of 16 columns whose instructions may overlap, two or four: one takes 16 registers
struct SideSum {
  double sum[4] = {0.0, 0.0, 0.0, 0.0};

  // a, x: a lane's four values of the 16-column block b (zeros past the end); left: columns up to the end
  template <class A, class X>
  __device__ __forceinline__ void add(int left, A a, X x) {
#pragma unroll
    for (int b0 = 0; b0 < 4; b0 += kTogether) {
      if (b0 > 0 && b0 * 16 >= left) break;
      f32x4 block[kTogether];
#pragma unroll
      for (int j = 0; j < kTogether; ++j) {
        const f32x4 va = a(b0 + j), vx = x(b0 + j), zero = {0.f, 0.f, 0.f, 0.f};
        f32x4 lo = __builtin_amdgcn_mfma_f32_16x16x4f32(va[0], vx[0], zero, 0, 0, 0);
        f32x4 hi = __builtin_amdgcn_mfma_f32_16x16x4f32(va[2], vx[2], zero, 0, 0, 0);
        lo = __builtin_amdgcn_mfma_f32_16x16x4f32(va[1], vx[1], lo, 0, 0, 0);
        hi = __builtin_amdgcn_mfma_f32_16x16x4f32(va[3], vx[3], hi, 0, 0, 0);
        block[j] = lo + hi;
      }
      // (summed here: left alone, the sums are put off and their operands take 130 registers more)
#pragma unroll
      for (int j = 0; j < kTogether; ++j) asm volatile("" : "+v"(block[j]));
#pragma unroll
      for (int j = 0; j < kTogether; j += 2)
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] += (double)(block[j][e] + block[j + 1][e]);
    }
  }
  __device__ __forceinline__ f32x4 total() const { return f32x4{(float)sum[0], (float)sum[1], (float)sum[2], (float)sum[3]}; }
};

template <class C, int TM, int TN, int KC>
struct SideF32 {
  static constexpr int kWaves = 4, kThreads = kWaves * 64;
  static constexpr int kItems = (kFusedBlocks * (TN / 16) + kWaves - 1) / kWaves;   // (block of columns, 16 tokens) pairs of a wave
  const ProbeF32Args& p;
  const int m0, t0;
  const FusedLds<C, TM, TN> at;
  float* const lds;
  float* const rows;             // [blocks * 16][kPitch]
  const int rb, n_blocks;        // blocks of a direction, of all directions and the bank

  __device__ __forceinline__ SideF32(const ProbeF32Args& args, float* mem, int first_m, int first_t)
      : p(args), m0(first_m), t0(first_t), at(args), lds(mem), rows(mem + at.rows), rb((args.r + 15) / 16),
        n_blocks(args.batch.K * ((args.r + 15) / 16) + (args.R + 15) / 16) {}

  // four neighbouring entries of a factor stream
  __device__ __forceinline__ f32x4 draw(uint64_t seed, uint32_t stream, uint64_t block) const {
    const uint4 w = factor_block(seed, stream, block);
    float z0, z1, z2, z3;
    box_muller(w.x, w.y, z0, z1);
    box_muller(w.z, w.w, z2, z3);
    return f32x4{z0, z1, z2, z3};
  }

  // columns k0 .. k0 + KC of the side operand; with the first, U of the tile's features
  __device__ __forceinline__ void fill(int tid, int k0) {
    const int K = p.batch.K, n_here = min(KC, p.n - k0);
    const uint64_t* seeds = reinterpret_cast<const uint64_t*>(lds + at.seeds);
    float* bank = rows + K * rb * 16 * C::kPitch;
    constexpr int U = 8;   // values of Vb asked for together
    for (int e0 = tid; e0 < KC * p.R; e0 += kThreads * U) {
      float v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * kThreads, i = e / p.R, j = e - i * p.R;
        v[u] = i < n_here ? p.Vb[(int64_t)(k0 + i) * p.R_cap + j] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * kThreads, i = e / p.R, j = e - i * p.R;
        if (i < KC) bank[j * C::kPitch + i] = v[u];
      }
    }
    const int v_dir = KC * p.r / 4, u_dir = TM * p.r / 4;   // Philox blocks: k0 r and m0 r are multiples of 4
    const int n_v = v_dir * K, total = n_v + (k0 == 0 ? u_dir * K : 0);
    for (int q = tid; q < total; q += kThreads) {
      const bool is_v = q < n_v;
      const int q0 = is_v ? q : q - n_v, per_dir = is_v ? v_dir : u_dir;
      const int d = q0 / per_dir, blk = q0 - d * per_dir;
      const f32x4 z = draw(seeds[is_v ? K + d : d], is_v ? p.tensor_id | 1u : p.tensor_id & ~1u, (uint64_t)(is_v ? k0 : m0) * p.r / 4 + blk);
      if (is_v) {
        int i = blk * 4 / p.r, j = blk * 4 - i * p.r;
        float* dst = rows + d * rb * 16 * C::kPitch;
#pragma unroll
        for (int l = 0; l < 4; ++l) {
          dst[j * C::kPitch + i] = i < n_here ? z[l] : 0.f;
          if (++j == p.r) { j = 0; ++i; }
        }
      } else {
#pragma unroll
        for (int l = 0; l < 4; ++l) lds[at.u + q0 * 4 + l] = z[l];
      }
    }
  }

  // The side waves' part of TileF32::multiply (slab_x: the slab's rows of X); leaves the tokens' columns and kinds in LDS.
  __device__ __forceinline__ void walk(int n, const float* slab_x) {
    const BatchDev& b = p.batch;
    const int tid = threadIdx.x - C::kThreads, lane = tid & 63, wave = tid >> 6;
    int* words = reinterpret_cast<int*>(lds);
    {   // every table in one round trip
      uint64_t* seeds = reinterpret_cast<uint64_t*>(lds + at.seeds);
      for (int e = tid; e <= b.S; e += kThreads) {
        words[at.cu + e] = b.cu[e];
        if (e < b.S) words[at.cand + e] = b.seq_cand[e];
      }
      for (int e = tid; e < b.C; e += kThreads) {
        words[at.dir + e] = b.cand_dir[e];
        lds[at.sign + e] = b.cand_sign[e];
      }
      if (tid < b.K) {
        seeds[tid] = b.seed[tid];
        seeds[b.K + tid] = b.seed_v ? b.seed_v[tid] : b.seed[tid];
      }
      // rows that pad a block stay zero
      for (int row = wave; row < n_blocks * 16; row += kWaves) {
        const bool bank = row >= b.K * rb * 16;
        if (bank ? row - b.K * rb * 16 >= p.R : row % (rb * 16) >= p.r)
          for (int k = lane; k < KC; k += 64) rows[row * C::kPitch + k] = 0.f;
      }
    }
    __syncthreads();
    SideSum<TM == 32 ? 2 : 4> sum[kItems];
    for (int k0 = 0; k0 < n; k0 += KC) {
      if (k0 > 0) __syncthreads();
      fill(tid, k0);
      __syncthreads();
#pragma unroll
      for (int i = 0; i < kItems; ++i) {
        const int item = i * kWaves + wave, blk = item / (TN / 16), cb = item % (TN / 16);
        if (blk >= n_blocks) break;
        const float* fa = rows + (blk * 16 + (lane & 15)) * C::kPitch + (lane >> 4) * 4;
        const float* fb = slab_x + (cb * 16 + (lane & 15)) * C::kPitch + (lane >> 4) * 4;
#pragma unroll
        for (int k64 = 0; k64 < KC; k64 += 64) {
          if (k0 + k64 >= n) break;
          sum[i].add(n - k0 - k64, [&](int b) { return *reinterpret_cast<const f32x4*>(fa + k64 + b * 16); },
                     [&](int b) { return *reinterpret_cast<const f32x4*>(fb + k64 + b * 16); });
        }
      }
    }
    // a token's kind and scale, then its columns
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      const int item = i * kWaves + wave, blk = item / (TN / 16), cb = item % (TN / 16);
      const int tl = cb * 16 + (lane & 15), t = t0 + tl;
      int kind = kKindForeground;
      float scale = 0.f;
      if (t < p.T) {
        int lo = 0, hi = b.S;   // the last sequence that starts at or before the row
        while (hi - lo > 1) {
          const int mid = (lo + hi) >> 1;
          if (words[at.cu + mid] <= t) lo = mid; else hi = mid;
        }
        candidate_kind(words[at.cand + lo], b.C, b.K, p.eps, words + at.dir, lds + at.sign, kind, scale);
      }
      if (blk == 0) words[at.kinds + tl] = kind;
      if (blk >= n_blocks) break;
      const int d = blk / rb;   // direction of the block, or past them the bank
      const bool bank = d >= b.K;
      const int j0 = (bank ? blk - b.K * rb : blk - d * rb) * 16 + 4 * (lane >> 4);
      if (bank ? kind < kKindCentre : kind != d) continue;
      const f32x4 acc = sum[i].total();
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (j0 + e < (bank ? p.R : p.r)) lds[at.cols + tl * (p.r + p.R) + (bank ? p.r : 0) + j0 + e] = bank ? acc[e] : acc[e] * scale;
    }
  }
};

bool whole_quads(const void* a, int64_t lda, const void* b, int64_t ldb, int K) {
  return (((uintptr_t)a | (uintptr_t)b) & 15u) == 0 && lda % 4 == 0 && ldb % 4 == 0 && K % 4 == 0;
}

// Tside[t, :] = [ s_t eps X[t,:] V_{k_t} | X[t,:] Vb ] where the row has such a term, for the calls whose side columns do not
// ride along with the products (f32_side_rides_along).  A wave per 16 rows, 16 columns and direction among the rows (the first
// kSideDirs; further ones follow in turn), operands straight from memory, 256 columns of X asked for together: such a call is
// a chain of round trips.  Linear and scoring, a wave per row and 8 columns on the vector ALU -> this: 3671 rows, 632 wide, 8 + 33
// columns 225 -> 128 us; 2010 rows, 258 wide, four directions, 1 + 33 columns 80 -> 67; 252 rows, 366 wide, 8 + 33 46 -> 42.5.
// Summed as in SideF32: the same bits.
constexpr int kSideDirs = 4;

template <bool kVec>
__global__ __launch_bounds__(64, 2) void k_side_f32(ProbeF32Args p) {
  constexpr int U = 16;                  // blocks of 16 columns of X per trip
  const int NC = p.r + p.R, rb = (p.r + 15) / 16;
  const int lane = threadIdx.x, g = lane >> 4, col = lane & 15;
  const int t = blockIdx.x * 16 + col;   // this lane's row of X, and column of the result
  const bool dir = (int)blockIdx.y < rb;
  const int j0 = dir ? blockIdx.y * 16 : ((int)blockIdx.y - rb) * 16;
  const int j = j0 + col;                // this lane's column of V or Vb
  const int s = p.tok_seq[min(t, p.T - 1)];
  const int kind = t < p.T ? p.seq_kind[s] : kKindForeground;
  const float* x = p.X + (int64_t)min(t, p.T - 1) * p.ldx;
  uint64_t left = __ballot(dir ? kind >= 0 : kind >= kKindCentre);
  for (int nth = 0; left; ++nth) {
    int k = 0;
    uint64_t mine = left;
    if (dir) {   // the rows of one direction
      k = __builtin_amdgcn_readlane(kind, __ffsll((unsigned long long)left) - 1);
      mine = __ballot(kind == k);
    }
    left &= ~mine;
    if (nth % kSideDirs != (int)blockIdx.z) continue;
    const float* v = dir ? p.Vf + (int64_t)k * p.n * p.r + min(j, p.r - 1) : p.Vb + min(j, p.R - 1);
    const int64_t pitch = dir ? p.r : p.R_cap;
    const bool real = j < (dir ? p.r : p.R);
    SideSum<2> sum;
    for (int k0 = 0; k0 < p.n; k0 += 16 * U) {
      f32x4 a[U], b[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int at = k0 + u * 16 + g * 4;
        if constexpr (kVec) {
          b[u] = *reinterpret_cast<const f32x4*>(x + min(at, p.n - 4));
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) b[u][i] = x[min(at + i, p.n - 1)];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) a[u][i] = v[min(at + i, p.n - 1) * pitch];
      }
      // (the loads all go out before the first product: left alone they are moved behind the ends of the row they may be past)
#pragma unroll
      for (int u = 0; u < U; ++u) asm volatile("" : "+v"(a[u]), "+v"(b[u]));
#pragma unroll
      for (int u = 0; u < U; u += 4) {
        if (k0 + u * 16 >= p.n) break;
        auto in = [&](int at, bool also, const f32x4& v) {   // what lies past the end of the row, or of the columns, counts as zero
          f32x4 z;
#pragma unroll
          for (int i = 0; i < 4; ++i) z[i] = also && at + i < p.n ? v[i] : 0.f;
          return z;
        };
        sum.add(p.n - k0 - u * 16, [&](int blk) { return in(k0 + (u + blk) * 16 + g * 4, real, a[u + blk]); },
                [&](int blk) { return in(k0 + (u + blk) * 16 + g * 4, true, b[u + blk]); });
      }
    }
    if ((mine >> lane) & 1) {
      const float scale = dir ? p.seq_scale[s] : 1.0f;
      const f32x4 acc = sum.total();
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int jj = j0 + 4 * g + e;
        if (jj < (dir ? p.r : p.R)) p.Tside[(int64_t)t * NC + (dir ? jj : p.r + jj)] = acc[e] * scale;
      }
    }
  }
}

// kFused: the call's one launch.  Four more waves look up the tile's tokens' sequences, draw the factors it needs and
// compute its tokens' side columns along with the products; otherwise these come from memory (k_probe_prep_f32, k_side_f32).
template <class C, int TM, int TN, int WC, int KC, bool kVec, bool kFused>
__global__ __launch_bounds__(C::kThreads + (kFused ? 256 : 0)) void k_probe_f32(ProbeF32Args p) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m0 = blockIdx.x * TM, t0 = blockIdx.y * TN;
  const int NC = p.r + p.R;
  f32x4 acc[C::RB][C::CB];
  const float* s_u = nullptr;      // [direction][TM][r]
  const float* s_side = nullptr;   // [TN][NC]
  const int* s_kind = nullptr;
  if constexpr (kFused) {
    SideF32<C, TM, TN, KC> side(p, lds, m0, t0);
    C::template multiply<kVec>(p.W, p.ldw, p.m, m0, p.X, p.ldx, p.T, t0, p.n, lds, acc, side);
    __syncthreads();
    if (wave >= C::kThreads / 64) return;
    s_u = lds + side.at.u;
    s_side = lds + side.at.cols;
    s_kind = reinterpret_cast<const int*>(lds + side.at.kinds);
  } else {
    NoSide none;
    C::template multiply<kVec>(p.W, p.ldw, p.m, m0, p.X, p.ldx, p.T, t0, p.n, lds, acc, none);
  }
#pragma unroll
  for (int cb = 0; cb < C::CB; ++cb) {
    const int tl = (wave % WC) * (C::CB * 16) + cb * 16 + (lane & 15), t = t0 + tl;
    if (t >= p.T) continue;
    int kind = kKindForeground;
    if constexpr (kFused) kind = s_kind[tl];
    else if (p.has_side) kind = p.seq_kind[p.tok_seq[t]];
#pragma unroll
    for (int rb = 0; rb < C::RB; ++rb) {
      const int o = m0 + (wave / WC) * (C::RB * 16) + rb * 16 + 4 * (lane >> 4);   // four neighbouring features
      if (o >= p.m) continue;
      float y[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = acc[rb][cb][e];
      if (kind >= kKindCentre) {   // foreground rows skip the side state entirely
        const float* ts = kFused ? s_side + tl * NC : p.Tside + (int64_t)t * NC;
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
          const float* u = kFused ? s_u + ((int64_t)kind * TM + (o - m0)) * p.r : p.Uf + (int64_t)kind * p.m * p.r;
#pragma unroll 4
          for (int jj = 0; jj < p.r; ++jj) {
            const float x = ts[jj];
#pragma unroll
            for (int e = 0; e < 4; ++e) side[e] = fmaf(x, u[(kFused ? e : at[e]) * p.r + jj], side[e]);
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
  NoSide none;
  C::template multiply<kVec>(p.Wh, p.ldw, p.vocab, v0, p.H, p.ldh, p.T, t0, p.d, lds, acc, none);
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

// Whether a call's side columns ride along with its products, in one launch.  (No result depends on it.)  It saves two launches,
// 4 to 7 us; every tile draws and multiplies the columns of all directions, whichever its tokens have, and converts the
// bank's.  That has to stay under the products: the line is drawn by tiles per compute unit (one at least) x input columns x
// drawn and bank columns (read one by one: twice), lower with more blocks of 16; beyond two tiles of 64x64 per unit, or the tiles
// of 32x32 that are resident by their LDS, the start of a tile's side waves shows as well.  Linear and scoring of a layer, us, one
// launch / three: one block: 1024 rows, 256 wide (product 1024) 24.1 / 28.7; 510, 621 (7762) 79.2 / 85.9; 3168, 585 (11426) 118.4 / 126.8;
// 4096, 640, 2.5 tiles of 64x64 90.5 / 84.6; 4096, 1024, 4 tiles 157 / 138; 8192, 2048 1028 / 758.  Two: 1024, 256 (4096) 26.3 / 29.6; 424, 472
// with 4 + 8 columns (9440) 35.4 / 37.7; 4516, 381 (10144) 115 / 122; 1024, 256 with 16 + 16 (12288) 29.6 / 31.0, 4096, 256 47.5 / 45.5;
// 2048, 640 (12800) 74.4 / 69.3; 1024, 640 (25600) 62.8 / 50.2; 2048, 1024 with 16 + 16 (98304) 136 / 105.  Three: 510, 398 (4776) 57.4 /
// 61.1; 594, 304 (7296) 33.4 / 32.7; 558, 436 (10464) 56.9 / 53.8; 597, 488 (20862) 58.8 / 44.4; 4096, 640 (102400) 164 / 101.  Four: 872, 344
// 66.8 / 57.7.  Inputs without columns go the other way: the factors are drawn with the slabs of X, of which there are none.
bool f32_side_rides_along(int T, int m, int n, int r, int R, int K, int S, int C) {
  constexpr int64_t kLimit[kFusedBlocks + 1] = {12000, 12000, 10200, 5500};
  const int64_t blocks = (int64_t)K * ((r + 15) / 16) + (R + 15) / 16, cus = compute_units();
  if (n == 0 || blocks > kFusedBlocks || r + R > kFusedColumns || S > kFusedTable || C > kFusedTable) return false;
  ProbeF32Args a{};
  a.r = r; a.R = R; a.batch.K = K; a.batch.S = S; a.batch.C = C;
  int64_t n_tiles = tiles(m, 64, T, 64), most = 2 * cus;
  if (n_tiles < cus) {
    n_tiles = tiles(m, 32, T, 32);
    most = cus * (160 * 1024 / (int64_t)(sizeof(float) * FusedLds<TileF32<32, 32, 2, 2, 128>, 32, 32>(a).end));
  }
  return n_tiles <= most && (n_tiles < cus ? cus : n_tiles) * n * (K * r + 2 * R) <= kLimit[blocks] * cus;
}

template <int TM, int TN, int KC, bool kVec, bool kFused>
static hipError_t launch_probe_f32_tile(const ProbeF32Args& a, hipStream_t st) {
  using C = TileF32<TM, TN, 2, 2, KC>;
  size_t lds = sizeof(float) * C::kLdsFloats;
  if constexpr (kFused) {
    lds = sizeof(float) * FusedLds<C, TM, TN>(a).end;
    static std::atomic<bool> configured[kMaxDevices];
    const hipError_t ec = once_per_device(configured, [] {
      return hipFuncSetAttribute((const void*)k_probe_f32<C, TM, TN, 2, KC, kVec, true>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    });
    if (ec != hipSuccess) return ec;
  }
  hipLaunchKernelGGL((k_probe_f32<C, TM, TN, 2, KC, kVec, kFused>), dim3((a.m + TM - 1) / TM, (a.T + TN - 1) / TN), dim3(C::kThreads + (kFused ? 256 : 0)), (unsigned)lds, st, a);
  return hipGetLastError();
}

hipError_t launch_probe_f32(const ProbeF32Args& a, hipStream_t st) {
  if (a.T == 0 || a.m == 0) return hipSuccess;
  // 64x64 tiles when they give every compute unit one, 32x32 (a longer K slab, four times the workgroups) otherwise
  const bool large = tiles(a.m, 64, a.T, 64) >= compute_units();
  const bool fused = a.has_side && f32_side_rides_along(a.T, a.m, a.n, a.r, a.R, a.batch.K, a.batch.S, a.batch.C);
  const bool vec = whole_quads(a.X, a.ldx, a.W, a.ldw, a.n);
  if (a.has_side && !fused) {
    const hipError_t e = launch_probe_prep_f32(a.batch, a.eps, a.tabs, a.tensor_id, a.m, a.n, a.r, a.Uf, a.Vf, st);
    if (e != hipSuccess) return e;
    const dim3 grid((a.T + 15) / 16, (a.r + 15) / 16 + (a.R + 15) / 16, a.batch.K < 1 ? 1 : a.batch.K < kSideDirs ? a.batch.K : kSideDirs);
    if (vec && a.n > 0) hipLaunchKernelGGL(k_side_f32<true>, grid, dim3(64), 0, st, a);
    else hipLaunchKernelGGL(k_side_f32<false>, grid, dim3(64), 0, st, a);
  }
  if (large) {
    if (fused) return vec ? launch_probe_f32_tile<64, 64, 64, true, true>(a, st) : launch_probe_f32_tile<64, 64, 64, false, true>(a, st);
    return vec ? launch_probe_f32_tile<64, 64, 64, true, false>(a, st) : launch_probe_f32_tile<64, 64, 64, false, false>(a, st);
  }
  if (fused) return vec ? launch_probe_f32_tile<32, 32, 128, true, true>(a, st) : launch_probe_f32_tile<32, 32, 128, false, true>(a, st);
  return vec ? launch_probe_f32_tile<32, 32, 128, true, false>(a, st) : launch_probe_f32_tile<32, 32, 128, false, false>(a, st);
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
