// What joins the probe linears of a decoder block during a candidate's scoring pass
// (Sec. 2.2: a query is a teacher-forced scoring pass under the candidate's weights;
// Sec. 3.1: packed variable-length sequences): residual sum + normalisation, and causal
// self-attention over each packed sequence.  None of it has perturbed parameters, so it is
// the same for every candidate and takes no candidate table.
//
//   k_add_norm_bf16 / k_add_norm_any   h = x + res, y = LayerNorm(h) or RMSNorm(h); one wave per row,
//                                      the row stays in registers between the passes (HBM-bound)
//   k_attention_bf16                   online-softmax attention on 16x16x32 bf16 MFMA, head_dim 128
//   k_attention_f32                    plain fp32 attention on the vector ALU (any head_dim <= 256)
//   k_qk_norm_rope_*                   per-head RMS norm of queries and keys + rotary embedding, in place
//                                      (the Qwen3 family; its gated MLP is an epilogue of the probe linear)
#include <type_traits>

#include "zo_device.hpp"
#include "zo_internal.hpp"

namespace zo {
namespace {

typedef __attribute__((address_space(3))) void lds_void;

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ void block_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// ------------------------------------------------------------------ add + norm

constexpr int kNormWaves = 4;   // waves per workgroup, one row each at a time
// Workgroups resident per CU, by what a row of that many chunks takes in registers.
constexpr int norm_wgs_per_cu(int chunks) { return chunks <= 2 ? 8 : chunks <= 4 ? 7 : chunks <= 6 ? 5 : chunks <= 8 ? 4 : chunks <= 12 ? 3 : 2; }

// bf16 rows with d % 8 == 0 and d <= kChunks * 512: lane l owns the 8 elements starting at
// (c*64 + l)*8 of chunk c.  Exact two-pass moments in fp32 on the register copy of the row.
// The grid is one resident round of waves that stride through the rows; gamma and beta are staged once per
// workgroup in LDS (re-reading them per row from L2 would move four times the bytes of the
// row itself), in the order the lanes read them: the two 16-byte halves of a lane's 8 values
// sit in separate planes so that consecutive lanes read consecutive 16-byte words.
//
// All of a row's loads are under way at once.  (Chunk by chunk, with a wait and a store between,
// a wave had two loads in flight, and a row took as many trips to memory as it has chunks: 528 rows
// of 5120, where a wave has one row, took 15.0 us for the norm and the residual sum, now 12.8.)
template <int kChunks, bool kRes>
__global__ __launch_bounds__(kNormWaves* kWave, norm_wgs_per_cu(kChunks)) void k_add_norm_bf16(NormArgs a) {
  __shared__ __attribute__((aligned(16))) float s_gamma[kChunks * 512];
  __shared__ __attribute__((aligned(16))) float s_beta[kChunks * 512];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (a.Y) {
    for (int e = threadIdx.x * 4; e < a.d; e += kNormWaves * kWave * 4) {
      const int at = (e >> 9) * 512 + ((e >> 2) & 1) * 256 + ((e & 511) >> 3) * 4;
      *reinterpret_cast<float4*>(&s_gamma[at]) = *reinterpret_cast<const float4*>(a.gamma + e);
      *reinterpret_cast<float4*>(&s_beta[at]) =
          a.beta ? *reinterpret_cast<const float4*>(a.beta + e) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();
  }
  const float inv_d = 1.0f / (float)a.d;
  // A row is one window of d values: what a lane asks for past its end reads as zero, what it writes there is dropped.
  auto window = [&](const void* base, int64_t ld, int row) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)((bf16_t*)base + (int64_t)row * ld), 0, a.d * 2, 0x00020000);
  };
  const int stride = gridDim.x * kNormWaves;
  for (int row = blockIdx.x * kNormWaves + __builtin_amdgcn_readfirstlane(wave); row < a.T; row += stride) {
    u32x4 hv[kChunks];   // the row as it is normalised: bf16 values
    u32x4 xv[kChunks], rv[kChunks];
    {
      const __amdgpu_buffer_rsrc_t wx = window(a.X, a.ldx, row), wr = window(kRes ? a.R : a.X, kRes ? a.ldr : a.ldx, row);
#pragma unroll
      for (int c = 0; c < kChunks; ++c) {   // (all requested before the first is looked at)
        xv[c] = __builtin_amdgcn_raw_buffer_load_b128(wx, lane * 16 + c * 1024, 0, 0);
        if constexpr (kRes) rv[c] = __builtin_amdgcn_raw_buffer_load_b128(wr, lane * 16 + c * 1024, 0, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    float sum = 0.f, sumsq = 0.f;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t p = xv[c][i];
        // the sum is stored as bf16, and it is that stored value which is normalised
        if constexpr (kRes)
          p = pack_bf16x2(__uint_as_float(p << 16) + __uint_as_float(rv[c][i] << 16),
                          __uint_as_float(p & 0xFFFF0000u) + __uint_as_float(rv[c][i] & 0xFFFF0000u));
        hv[c][i] = p;
        const float lo = __uint_as_float(hv[c][i] << 16), hi = __uint_as_float(hv[c][i] & 0xFFFF0000u);
        sum += lo + hi;
        sumsq += lo * lo + hi * hi;
      }
      __builtin_amdgcn_sched_barrier(0);   // (a chunk's operands make room for the chunk)
    }
    if (kRes && a.Hsum) {
      const __amdgpu_buffer_rsrc_t wh = window(a.Hsum, a.ldh, row);
#pragma unroll
      for (int c = 0; c < kChunks; ++c) __builtin_amdgcn_raw_buffer_store_b128(hv[c], wh, lane * 16 + c * 1024, 0, 0);
    }
    if (!a.Y) continue;
    // (the row stays packed: its values in fp32, kept from pass to pass, would take the registers of the next row's loads)
    auto packed_again = [&]() {
#pragma unroll
      for (int c = 0; c < kChunks; ++c) asm volatile("" : "+v"(hv[c]));
    };
    packed_again();
    float mean = 0.f, rstd;
    if (a.kind == 0) {
      mean = wave_sum(sum) * inv_d;
      float dev = 0.f;
#pragma unroll
      for (int c = 0; c < kChunks; ++c)
        if ((c * kWave + lane) * 8 < a.d) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float lo = __uint_as_float(hv[c][i] << 16) - mean, hi = __uint_as_float(hv[c][i] & 0xFFFF0000u) - mean;
            dev += lo * lo;
            dev += hi * hi;
          }
        }
      rstd = 1.0f / sqrtf(wave_sum(dev) * inv_d + a.eps);
    } else {
      rstd = 1.0f / sqrtf(wave_sum(sumsq) * inv_d + a.eps);
    }
    packed_again();
    const __amdgpu_buffer_rsrc_t wy = window(a.Y, a.ldy, row);
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      const float4 g0 = *reinterpret_cast<const float4*>(&s_gamma[c * 512 + lane * 4]);
      const float4 g1 = *reinterpret_cast<const float4*>(&s_gamma[c * 512 + 256 + lane * 4]);
      const float4 b0 = *reinterpret_cast<const float4*>(&s_beta[c * 512 + lane * 4]);
      const float4 b1 = *reinterpret_cast<const float4*>(&s_beta[c * 512 + 256 + lane * 4]);
      float v[8];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[2 * i] = (__uint_as_float(hv[c][i] << 16) - mean) * rstd;
        v[2 * i + 1] = (__uint_as_float(hv[c][i] & 0xFFFF0000u) - mean) * rstd;
      }
      u32x4 o;
      o[0] = pack_bf16x2(v[0] * g0.x + b0.x, v[1] * g0.y + b0.y);
      o[1] = pack_bf16x2(v[2] * g0.z + b0.z, v[3] * g0.w + b0.w);
      o[2] = pack_bf16x2(v[4] * g1.x + b1.x, v[5] * g1.y + b1.y);
      o[3] = pack_bf16x2(v[6] * g1.z + b1.z, v[7] * g1.w + b1.w);
      __builtin_amdgcn_raw_buffer_store_b128(o, wy, lane * 16 + c * 1024, 0, 0);
      __builtin_amdgcn_sched_barrier(0);   // (gamma and beta of one chunk at a time)
    }
  }
}

__device__ __forceinline__ float ld_elem(const float* p, int64_t i) { return p[i]; }
__device__ __forceinline__ float ld_elem(const bf16_t* p, int64_t i) { return bf16_to_f32(p[i]); }
__device__ __forceinline__ float st_round(float*, float v) { return v; }
__device__ __forceinline__ float st_round(bf16_t*, float v) { return bf16_round(v); }
__device__ __forceinline__ void st_elem(float* p, int64_t i, float v) { p[i] = v; }
__device__ __forceinline__ void st_elem(bf16_t* p, int64_t i, float v) { p[i] = f32_to_bf16(v); }

// Any width and either storage type: one wave per row, the row is re-read from memory per pass.
// A lane reads back only elements it wrote itself, so Hsum may alias X.
template <typename Tio>
__global__ __launch_bounds__(kNormWaves* kWave) void k_add_norm_any(NormArgs a) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = blockIdx.x * kNormWaves + wave;
  if (row >= a.T) return;
  const Tio* x = (const Tio*)a.X + (int64_t)row * a.ldx;
  const Tio* res = a.R ? (const Tio*)a.R + (int64_t)row * a.ldr : nullptr;
  Tio* hs = a.Hsum ? (Tio*)a.Hsum + (int64_t)row * a.ldh : nullptr;
  const bool stored = res && hs;
  float sum = 0.f, sumsq = 0.f;
  for (int e = lane; e < a.d; e += kWave) {
    float h = ld_elem(x, e);
    if (res) h = st_round((Tio*)nullptr, h + ld_elem(res, e));
    if (stored) st_elem(hs, e, h);
    sum += h;
    sumsq += h * h;
  }
  if (!a.Y) return;
  auto value = [&](int e) {
    if (stored) return ld_elem((const Tio*)hs, e);
    float h = ld_elem(x, e);
    if (res) h = st_round((Tio*)nullptr, h + ld_elem(res, e));
    return h;
  };
  const float inv_d = 1.0f / (float)a.d;
  float mean = 0.f, rstd;
  if (a.kind == 0) {
    mean = wave_sum(sum) * inv_d;
    float dev = 0.f;
    for (int e = lane; e < a.d; e += kWave) {
      const float t = value(e) - mean;
      dev += t * t;
    }
    rstd = 1.0f / sqrtf(wave_sum(dev) * inv_d + a.eps);
  } else {
    rstd = 1.0f / sqrtf(wave_sum(sumsq) * inv_d + a.eps);
  }
  Tio* y = (Tio*)a.Y + (int64_t)row * a.ldy;
  for (int e = lane; e < a.d; e += kWave)
    st_elem(y, e, (value(e) - mean) * rstd * a.gamma[e] + (a.beta ? a.beta[e] : 0.f));
}

// ------------------------------------------------------------------ attention, fp32

// Largest i with cu[i] <= t (cu[0] = 0 <= t < cu[S]): the sequence that holds row t.
__device__ __forceinline__ int seq_of_row(const int32_t* cu, int S, int t) {
  int lo = 0, hi = S;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (cu[mid] <= t) lo = mid; else hi = mid - 1;
  }
  return lo;
}

constexpr int kAttnF32MaxDh = 256;

// One wave per (row, head): scores in two passes (maximum, then weights), values accumulated
// with lanes over the head dimension.
__global__ __launch_bounds__(kWave) void k_attention_f32(AttnArgs a) {
  __shared__ float s_q[kAttnF32MaxDh];
  __shared__ float s_p[kWave];
  const int lane = threadIdx.x;
  const int t = blockIdx.x, h = blockIdx.y, g = h / a.group;
  const int dh = a.dh;
  const int a0 = a.cu[seq_of_row(a.cu, a.S, t)];
  const int nkeys = t - a0 + 1;
  const float* q = (const float*)a.Q + (int64_t)t * a.ldq + h * dh;
  const float* Kb = (const float*)a.K + (int64_t)a0 * a.ldk + g * dh;
  const float* Vb = (const float*)a.V + (int64_t)a0 * a.ldv + g * dh;
  for (int d = lane; d < dh; d += kWave) s_q[d] = q[d];
  __syncthreads();
  auto score = [&](int j) {
    const float* k = Kb + (int64_t)j * a.ldk;
    float s = 0.f;
    for (int d = 0; d < dh; ++d) s += s_q[d] * k[d];
    return s * a.scale;
  };
  float mx = -INFINITY;
  for (int j = lane; j < nkeys; j += kWave) mx = fmaxf(mx, score(j));
  mx = wave_max(mx);
  float acc[kAttnF32MaxDh / kWave] = {0.f, 0.f, 0.f, 0.f};
  float lsum = 0.f;
  for (int base = 0; base < nkeys; base += kWave) {
    const int j = base + lane;
    const float p = j < nkeys ? expf(score(j) - mx) : 0.f;
    lsum += p;
    s_p[lane] = p;
    __syncthreads();
    const int cnt = min(kWave, nkeys - base);
    for (int jj = 0; jj < cnt; ++jj) {
      const float pj = s_p[jj];
      const float* v = Vb + (int64_t)(base + jj) * a.ldv;
#pragma unroll
      for (int c = 0; c < kAttnF32MaxDh / kWave; ++c)
        if (lane + c * kWave < dh) acc[c] += pj * v[lane + c * kWave];
    }
    __syncthreads();
  }
  const float inv = 1.0f / wave_sum(lsum);
  float* o = (float*)a.O + (int64_t)t * a.ldo + h * dh;
#pragma unroll
  for (int c = 0; c < kAttnF32MaxDh / kWave; ++c)
    if (lane + c * kWave < dh) o[lane + c * kWave] = acc[c] * inv;
}

// ------------------------------------------------------------------ attention, bf16 MFMA

constexpr int kBQ = 128;            // query rows per workgroup (32 per wave)
constexpr int kBKV = 64;            // keys per step
constexpr int kDh = 128;            // head dimension of this kernel
constexpr int kAttnWaves = 4;
constexpr int kKStage = kBKV * kDh * 2;   // 16 KiB: keys x head dim, 256-byte rows
constexpr int kVStage = kBKV * kDh * 2;   // 16 KiB: keys x head dim, 256-byte rows

// Swizzle keys: the 16-byte chunk c of row `row` of a stage is stored at chunk c ^ key (both stages have 256-byte
// rows, so the same chunk of any two rows lies on the same banks).
// Keys are read 16 rows at a time, {8*(i/4) + i%4 : i < 16} plus a multiple of 4 and of 32: sixteen different keys.
__device__ __forceinline__ int swz_k(int row) { return (row & 3) | (((row >> 3) & 3) << 2); }
// Values are read transposed, 8 bytes of each of four neighbouring chunks (the lower half of the even ones, the upper of
// the odd ones, or the other way round) of eight rows at a time, {0..3, 8..11} plus a multiple of 4 and of 16: with bit 1 of
// the key zero no two of the 32 pieces share a bank.
__device__ __forceinline__ int swz_v(int row) { return (row & 1) | (((row >> 1) & 1) << 2) | (((row >> 3) & 1) << 3); }

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((address_space(3))) const char lds_cchar;

// Finds the (sequence, query block) pair behind slot w: sequences are walked 64 at a time and a
// wave-wide prefix sum of their block counts locates the slot.  Every wave of the workgroup
// computes the same answer.  Returns false when w is past the last pair.
__device__ __forceinline__ bool find_query_block(const int32_t* cu, int S, int w, int lane, int& seq, int& qb) {
  int base = 0;
  for (int s0 = 0; s0 < S; s0 += kWave) {
    const int i = s0 + lane;
    const int nb = i < S ? (cu[i + 1] - cu[i] + kBQ - 1) / kBQ : 0;
    // inclusive scan in the vector ALU: within rows of 16 lanes, then row 0 into 1, 2 into 3, then lane 31 into rows 2, 3
    int inc = nb;
    inc += __builtin_amdgcn_update_dpp(0, inc, 0x111, 0xf, 0xf, true);
    inc += __builtin_amdgcn_update_dpp(0, inc, 0x112, 0xf, 0xf, true);
    inc += __builtin_amdgcn_update_dpp(0, inc, 0x114, 0xf, 0xf, true);
    inc += __builtin_amdgcn_update_dpp(0, inc, 0x118, 0xf, 0xf, true);
    inc += __builtin_amdgcn_update_dpp(0, inc, 0x142, 0xa, 0xf, false);
    inc += __builtin_amdgcn_update_dpp(0, inc, 0x143, 0xc, 0xf, false);
    const int excl = base + inc - nb;
    const unsigned long long hit = __ballot(w >= excl && w < excl + nb);
    if (hit) {
      const int src = __ffsll((long long)hit) - 1;
      seq = s0 + src;
      qb = w - __builtin_amdgcn_readlane(excl, src);
      return true;
    }
    base += __builtin_amdgcn_readlane(inc, kWave - 1);
  }
  return false;
}

// Causal attention of one (sequence, head, block of 128 query rows).
//
// Both products are computed transposed so that every per-query quantity lives in the lane that
// owns that query's column: S^T = K Q^T (A = keys from LDS, B = queries held in registers) and
// O^T = V^T P^T (A = transposed values from LDS, B = the weights just computed).  In the 16x16
// result layout lane l holds column l%16 (a query) and rows 4*(l/16)+v; the 16 A-rows of a key
// tile are chosen as {8*(i/4) + i%4} (+4 for the second tile of a pair), so that over a pair
// of tiles a lane holds 8 consecutive keys: exactly the k-group it must supply as B operand of the
// second product.  The running maximum, the rescaling factor and the normaliser are then per-lane
// scalars and P never leaves registers.
//
// Keys and values go global->LDS directly (the swizzle is applied on the source address), 64 keys per
// step, two stages: the loads of step j+1 are issued when step j starts.  Values are transposed by the
// LDS read itself (ds_read_b64_tr_b16: the 16 lanes of a group name four rows of 16 columns, and lane j
// receives column j); which columns a tile holds is chosen so that over a pair of tiles a lane ends up with
// eight neighbouring ones, one 16-byte store (8-byte stores: 128 sequences of 128 rows, 40 heads, 162 us;
// 16-byte stores 146).  Rows past the end of the sequence repeat its last row and are always masked by the
// causal test.
//
// A query's arithmetic is its own: the maximum is that of the keys it sees in whole steps, raised in every
// step in which it grows, the normaliser is the fp32 sum of the fp32 weights, and nothing another row of
// the tile holds enters it, so a row has the same bits whatever follows it in its sequence.  (A
// maximum that lags until a row of the tile exceeds it by a factor of two, the scale in the exponent's
// multiply-add and a normaliser summed from the rounded weights by one more matrix instruction, 32 keys per
// step, take 398 us where this takes 428, but tie rows to their neighbours and sum in 16 bits.)
//
// Long sequences are bound by instruction issue between the two products: the matrix core leaves two
// issue slots of four cycles free per matrix instruction, an exponential takes two of them, any other
// vector instruction one.  So what a step need not do it skips: only the step that meets the diagonal masks,
// its second 32 keys are multiplied only if some row sees them, the output is rescaled only when the maximum of
// some query grows (the factors are exactly one otherwise), and fragment addresses are constants of the stage.
// 8 sequences of 2048 rows, 40 heads: 547 us (values through registers, every step masked and rescaled) -> 428
// (803 TFLOP/s of causal work); 14144 ragged rows of up to 512, 32 heads over 8: 134 -> 109 us, bound by the
// latency of a workgroup's start and its few steps; 128 sequences of 128 rows: 150 -> 146, near the bandwidth of its
// 671 MB.  Sequences of a few rows are bound by how many workgroups are resident, two per compute unit (128 of up
// to 30 rows, 40 heads: 50 -> 40; the 32-key form above, three per unit, 28).  Three waves per SIMD with 64 keys (168
// registers, one stage of keys or values, a second barrier per step) spill and take 440 to 490 us, and 35 on the short.

// Largest of the four lanes l, l ^ 16, l ^ 32, l ^ 48 (the lanes that share a query), in the vector ALU.
__device__ __forceinline__ float column_max(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const uint32_t v = __float_as_uint(fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1])));
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

__global__ __launch_bounds__(kAttnWaves* kWave, 2) void k_attention_bf16(AttnArgs a) {
  // [2] stages of keys, [2] stages of values.  (Dynamic: with named arrays the compiler tracks which of them a
  // direct-to-LDS load writes and waits for the next step's loads before it reads this step's stage.)
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  char* const s_k = lds;
  char* const s_v = lds + 2 * kKStage;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  int seq, qb;
  // One-dimensional grid, heads fastest: the query heads that share a key/value head run next to each other
  // (ragged Qwen3-shaped batch: 187 -> 166 us).  Slots are taken from the last: the grid is an upper bound, the
  // slots past the last query block leave at once, and within a sequence the blocks with the most keys start first.
  const int slot_id = gridDim.x / a.n_heads - 1 - blockIdx.x / a.n_heads;
  if (!find_query_block(a.cu, a.S, slot_id, lane, seq, qb)) return;
  const int h = blockIdx.x % a.n_heads, kvh = h / a.group;
  seq = __builtin_amdgcn_readfirstlane(seq);
  qb = __builtin_amdgcn_readfirstlane(qb);
  const int row_a = a.cu[seq], row_b = a.cu[seq + 1];       // the sequence is rows [row_a, row_b)
  const int q0 = row_a + qb * kBQ;
  const int q_last = min(q0 + kBQ, row_b) - 1;
  const int n_steps = (q_last - row_a) / kBKV + 1;
  const int wq0 = q0 + wave * 32;                            // this wave's first query row
  const bool wave_valid = wq0 < row_b;

  const bf16_t* Kh = (const bf16_t*)a.K + kvh * kDh;
  const bf16_t* Vh = (const bf16_t*)a.V + kvh * kDh;

  // ---- loads: load i of a wave fills the 1 KiB block wave*4 + i of a stage = 4 rows.  A whole step's offsets are the
  // same for every step (the base advances); rows past the end of the sequence repeat its last row.
  auto issue = [&](int step, int slot) __attribute__((always_inline)) {
    const int j0 = row_a + step * kBKV;
    const int last_rel = min(row_b - 1 - j0, kBKV - 1);
    const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc((void*)(Kh + (int64_t)j0 * a.ldk), 0,
                                                                        (last_rel * (int)a.ldk + kDh) * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc((void*)(Vh + (int64_t)j0 * a.ldv), 0,
                                                                        (last_rel * (int)a.ldv + kDh) * 2, 0x00020000);
    char* dk = s_k + slot * kKStage + wave * 4096;
    char* dv = s_v + slot * kVStage + wave * 4096;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = wave * 16 + 4 * i + (lane >> 4);
      const uint32_t off = (uint32_t)min(row, last_rel) * (uint32_t)(a.ldk * 2) + ((lane & 15) ^ swz_k(row)) * 16;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (lds_void*)(dk + i * 1024), 16, (int)off, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = wave * 16 + 4 * i + (lane >> 4);
      const uint32_t off = (uint32_t)min(row, last_rel) * (uint32_t)(a.ldv * 2) + ((lane & 15) ^ swz_v(row)) * 16;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (lds_void*)(dv + i * 1024), 16, (int)off, 0, 0, 0);
    }
  };
  issue(0, 0);

  // ---- queries: B fragments, lane (r16, g) holds Q[row r16 of tile qt][32 ks + 8 g .. + 8].
  bf16x8 qf[2][4];
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    const int qrow = min(wq0 + qt * 16 + r16, row_b - 1);
    const bf16_t* qp = (const bf16_t*)a.Q + (int64_t)qrow * a.ldq + h * kDh + g * 8;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) qf[qt][ks] = load_frag(qp + ks * 32);
  }
  const float sl2 = a.scale * 1.4426950408889634f;   // scores are kept in base-2 units

  // ---- fragment addresses: they differ between fragments by constants that leave the swizzle alone (4 rows, whole
  // stages) or by chunks (an exclusive or)
  const int k_row = 8 * (r16 >> 2) + (r16 & 3);
  const uint32_t k_off = k_row * 256 + ((g ^ swz_k(k_row)) << 4);
  // values: lane i of a group names row (key) 8 g + i/4 and four columns of chunk i%4 of a block of 32: in tile 2 dp the
  // first four of an even chunk and the last four of an odd one, in tile 2 dp + 1 the others
  const int v_row = 8 * g + (r16 >> 2);
  const uint32_t v_off = v_row * 256 + (((r16 & 3) ^ swz_v(v_row)) << 4) + (r16 & 1) * 8;

  f32x4 oacc[8][2];   // [head-dim tile][query tile]
#pragma unroll
  for (int dt = 0; dt < 8; ++dt)
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) oacc[dt][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run[2] = {-INFINITY, -INFINITY};
  float l_run[2] = {0.f, 0.f};   // this lane's share of the normaliser

  const char* kp[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) kp[ks] = s_k + (k_off ^ (ks << 6));
  uint32_t vp[8];   // LDS addresses
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) vp[dt] = (uint32_t)(uintptr_t)(lds_cchar*)s_v + (v_off ^ (uint32_t)((dt >> 1) << 6 | (dt & 1) << 3));
  typedef f32x4 Scores[2][2][2];   // [32 keys][half][query tile]; lane (g, r16): query r16, keys 32 tp + 8 g + 4 hf + v
  // The wave's 32 rows face the 32 keys of block n_diag: every block before it is whole, the ones after are not seen.
  const int n_diag = wave_valid ? (wq0 - row_a) / 32 : -1;
  auto attend = [&](int step, auto slot_c) __attribute__((always_inline)) {
    // (a score is rounded before the maximum is taken off: contracted or not must not be the compiler's choice)
#pragma clang fp contract(off)
    constexpr int slot = decltype(slot_c)::value;
    const bool both = step * 2 < n_diag;   // false: the step's second 32 keys lie past every query
    Scores s;
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int tp = 0; tp < 2; ++tp) {
      if (tp == 1 && !both) {
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
          for (int qt = 0; qt < 2; ++qt) s[tp][hf][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
        break;
      }
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        bf16x8 kf[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) kf[ks] = *reinterpret_cast<const bf16x8*>(kp[ks] + slot * kKStage + tp * 8192 + 4 * hf * 256);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
          for (int qt = 0; qt < 2; ++qt)
            s[tp][hf][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks], qf[qt][ks], ks == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : s[tp][hf][qt], 0, 0, 0);
      }
    }
    __builtin_amdgcn_s_setprio(0);
#pragma unroll
    for (int tp = 0; tp < 2; ++tp)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) s[tp][hf][qt] *= sl2;
    if (step * 2 + 1 >= n_diag) {   // some key lies past some query
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
        const int last = min(wq0 + qt * 16 + r16, row_b - 1) - (row_a + step * kBKV) - 8 * g;   // the last key this query sees
#pragma unroll
        for (int tp = 0; tp < 2; ++tp)
#pragma unroll
          for (int hf = 0; hf < 2; ++hf)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (32 * tp + 4 * hf + v > last) s[tp][hf][qt][v] = -INFINITY;
      }
    }
    bf16x8 pf[2][2];   // [query tile][32 keys]
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
      float mx = -INFINITY;
#pragma unroll
      for (int tp = 0; tp < 2; ++tp)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
          for (int v = 0; v < 4; ++v) mx = fmaxf(mx, s[tp][hf][qt][v]);
      float alpha = 1.0f;
      if (__any(mx > m_run[qt])) {   // (otherwise every factor is one)
        const float m = fmaxf(column_max(mx), m_run[qt]);
        alpha = __builtin_amdgcn_exp2f(m_run[qt] - m);
        m_run[qt] = m;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) oacc[dt][qt] *= alpha;
      }
      float psum = 0.f;
#pragma unroll
      for (int tp = 0; tp < 2; ++tp) {
        float p[8];
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            p[hf * 4 + v] = __builtin_amdgcn_exp2f(s[tp][hf][qt][v] - m_run[qt]);
            psum += p[hf * 4 + v];
          }
        u32x4 packed = {pack_bf16x2(p[0], p[1]), pack_bf16x2(p[2], p[3]), pack_bf16x2(p[4], p[5]), pack_bf16x2(p[6], p[7])};
        pf[qt][tp] = __builtin_bit_cast(bf16x8, packed);
      }
      l_run[qt] = __builtin_fmaf(l_run[qt], alpha, psum);
    }
    // ---- O^T += V^T P^T
#pragma unroll
    for (int tp = 0; tp < 2; ++tp) {
      if (tp == 1 && !both) break;
#pragma unroll
      for (int d4 = 0; d4 < 8; d4 += 4) {
        // (waits in the block itself: before a read through the builtin the compiler waits for every direct-to-LDS load
        // in flight, the next step's included)
        constexpr int kAt = slot * kVStage;
        s16x4 t[8];
        asm volatile(
            "ds_read_b64_tr_b16 %0, %8 offset:%12\n ds_read_b64_tr_b16 %1, %8 offset:%13\n"
            "ds_read_b64_tr_b16 %2, %9 offset:%12\n ds_read_b64_tr_b16 %3, %9 offset:%13\n"
            "ds_read_b64_tr_b16 %4, %10 offset:%12\n ds_read_b64_tr_b16 %5, %10 offset:%13\n"
            "ds_read_b64_tr_b16 %6, %11 offset:%12\n ds_read_b64_tr_b16 %7, %11 offset:%13\n"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]), "=&v"(t[4]), "=&v"(t[5]), "=&v"(t[6]), "=&v"(t[7])
            : "v"(vp[d4]), "v"(vp[d4 + 1]), "v"(vp[d4 + 2]), "v"(vp[d4 + 3]), "n"(kAt + tp * 8192), "n"(kAt + tp * 8192 + 4 * 256)
            : "memory");
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const bf16x8 vf = __builtin_bit_cast(bf16x8, __builtin_shufflevector(t[2 * d], t[2 * d + 1], 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
          for (int qt = 0; qt < 2; ++qt)
            oacc[d4 + d][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf[qt][tp], oacc[d4 + d][qt], 0, 0, 0);
        }
        __builtin_amdgcn_s_setprio(0);
      }
    }
  };
  // Two stages: while step s is worked on, s + 1 is landing.
  auto one_step = [&](int step, auto slot_c) __attribute__((always_inline)) {
    constexpr int slot = decltype(slot_c)::value;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    block_barrier();   // the step's loads have landed for every wave, and every wave is done with the stage of step - 1
    if (step + 1 < n_steps) issue(step + 1, slot ^ 1);
    if (step * 2 <= n_diag) attend(step, slot_c);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  };
  for (int step = 0; step < n_steps; step += 2) {
    one_step(step, std::integral_constant<int, 0>{});
    if (step + 1 < n_steps) one_step(step + 1, std::integral_constant<int, 1>{});
  }

  if (!wave_valid) return;
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    float l = l_run[qt];
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    const float inv = 1.0f / l;
    const int qrow = wq0 + qt * 16 + r16;
    if (qrow < row_b) {
      bf16_t* o = (bf16_t*)a.O + (int64_t)qrow * a.ldo + h * kDh + g * 8;
#pragma unroll
      for (int dp = 0; dp < 4; ++dp) {
        const f32x4 x = oacc[2 * dp][qt], y = oacc[2 * dp + 1][qt];
        const u32x2 xp = {pack_bf16x2(x[0] * inv, x[1] * inv), pack_bf16x2(x[2] * inv, x[3] * inv)};
        const u32x2 yp = {pack_bf16x2(y[0] * inv, y[1] * inv), pack_bf16x2(y[2] * inv, y[3] * inv)};
        const u32x2 lo = (g & 1) ? yp : xp, hi = (g & 1) ? xp : yp;   // chunk g of the block: its first and last four columns
        *reinterpret_cast<u32x4*>(o + dp * 32) = u32x4{lo[0], lo[1], hi[0], hi[1]};
      }
    }
  }
}

// ------------------------------------------------------------------ per-head q/k norm + rotary embedding

// Rotation angle of pair i (of dh/2) at position pos: pos * theta^(-2i/dh).
__device__ __forceinline__ float rope_angle(float log2_theta, int i, int dh, int pos) {
  return (float)pos * exp2f(-(float)(2 * i) / (float)dh * log2_theta);
}

// bf16, head dimension 128, in place.  One wave per token, four heads at a time: the 16 lanes of a head
// hold elements 4j..4j+3 and their rotation partners 64+4j..64+4j+3 (j = lane % 16), so the per-head sum
// of squares is four shuffles and the rotation is lane-local.  The token's position and the four
// (cos, sin) pairs of a lane depend on neither the head nor on queries versus keys: they are computed
// once per token, under the first loads.  Heads 0..H-1 are queries, H..H+Hkv-1 keys.
__global__ __launch_bounds__(256) void k_qk_norm_rope_bf16(QkRopeArgs a) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= a.T) return;
  const int heads = a.n_heads + a.n_kv_heads;
  const int groups = (heads + 3) >> 2;
  const int j = lane & 15, hh = lane >> 4;
  auto row_of = [&](int head) -> bf16_t* {
    return head < a.n_heads ? (bf16_t*)a.Q + (int64_t)t * a.ldq + head * 128
                            : (bf16_t*)a.K + (int64_t)t * a.ldk + (head - a.n_heads) * 128;
  };
  auto load = [&](int grp, uint2& lo, uint2& hi) {
    const int head = grp * 4 + hh;
    lo = hi = make_uint2(0u, 0u);
    if (head < heads) {
      const bf16_t* row = row_of(head);
      lo = *reinterpret_cast<const uint2*>(row + 4 * j);
      hi = *reinterpret_cast<const uint2*>(row + 64 + 4 * j);
    }
  };
  uint2 lo, hi;
  load(0, lo, hi);
  float cs[4] = {1.f, 1.f, 1.f, 1.f}, sn[4] = {0.f, 0.f, 0.f, 0.f};
  if (a.theta > 0.f) {
    const int pos = t - a.cu[seq_of_row(a.cu, a.S, t)];
    const float l2t = log2f(a.theta);
#pragma unroll
    for (int e = 0; e < 4; ++e) sincosf(rope_angle(l2t, 4 * j + e, 128, pos), &sn[e], &cs[e]);
  }
  float4 gq0 = make_float4(1.f, 1.f, 1.f, 1.f), gq1 = gq0, gk0 = gq0, gk1 = gq0;
  if (a.gamma_q) {
    gq0 = *reinterpret_cast<const float4*>(a.gamma_q + 4 * j);
    gq1 = *reinterpret_cast<const float4*>(a.gamma_q + 64 + 4 * j);
    gk0 = *reinterpret_cast<const float4*>(a.gamma_k + 4 * j);
    gk1 = *reinterpret_cast<const float4*>(a.gamma_k + 64 + 4 * j);
  }
  for (int grp = 0; grp < groups; ++grp) {
    uint2 nlo, nhi;
    if (grp + 1 < groups) load(grp + 1, nlo, nhi);   // the next four heads travel under this group's arithmetic
    const int head = grp * 4 + hh;
    const bool is_q = head < a.n_heads;
    float x[8];   // [0..3] first half, [4..7] partners
    x[0] = __uint_as_float(lo.x << 16); x[1] = __uint_as_float(lo.x & 0xFFFF0000u);
    x[2] = __uint_as_float(lo.y << 16); x[3] = __uint_as_float(lo.y & 0xFFFF0000u);
    x[4] = __uint_as_float(hi.x << 16); x[5] = __uint_as_float(hi.x & 0xFFFF0000u);
    x[6] = __uint_as_float(hi.y << 16); x[7] = __uint_as_float(hi.y & 0xFFFF0000u);
    if (a.gamma_q) {
      float ss = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) ss += x[e] * x[e];
#pragma unroll
      for (int o = 8; o >= 1; o >>= 1) ss += __shfl_xor(ss, o);
      const float rstd = 1.0f / sqrtf(ss * (1.0f / 128.0f) + a.eps);
      const float4 g0 = is_q ? gq0 : gk0, g1 = is_q ? gq1 : gk1;
      x[0] *= rstd * g0.x; x[1] *= rstd * g0.y; x[2] *= rstd * g0.z; x[3] *= rstd * g0.w;
      x[4] *= rstd * g1.x; x[5] *= rstd * g1.y; x[6] *= rstd * g1.z; x[7] *= rstd * g1.w;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float p = x[e], q = x[4 + e];
      x[e] = p * cs[e] - q * sn[e];
      x[4 + e] = q * cs[e] + p * sn[e];
    }
    if (head < heads) {
      bf16_t* row = row_of(head);
      *reinterpret_cast<uint2*>(row + 4 * j) = make_uint2(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]));
      *reinterpret_cast<uint2*>(row + 64 + 4 * j) = make_uint2(pack_bf16x2(x[4], x[5]), pack_bf16x2(x[6], x[7]));
    }
    lo = nlo;
    hi = nhi;
  }
}

// Any even head dimension up to 256 and either storage type: one wave per (token, head), lane l holds the
// pairs l and l + 64.  With fp32 storage the angle is formed in double precision, so that positions in the
// thousands still give angles good to fp32 rounding.
template <typename Tio>
__global__ __launch_bounds__(256) void k_qk_norm_rope_any(QkRopeArgs a) {
  const int lane = threadIdx.x & 63;
  const int heads = a.n_heads + a.n_kv_heads;
  const int64_t item = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (item >= (int64_t)a.T * heads) return;
  const int t = (int)(item / heads), head = (int)(item % heads);
  const bool is_q = head < a.n_heads;
  const int dh = a.dh, half = dh >> 1;
  Tio* row = is_q ? (Tio*)a.Q + (int64_t)t * a.ldq + head * dh : (Tio*)a.K + (int64_t)t * a.ldk + (head - a.n_heads) * dh;
  float lo[2], hi[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int i = lane + c * kWave;
    lo[c] = i < half ? ld_elem(row, i) : 0.f;
    hi[c] = i < half ? ld_elem(row, half + i) : 0.f;
  }
  if (a.gamma_q) {
    const float ss = wave_sum(lo[0] * lo[0] + hi[0] * hi[0] + lo[1] * lo[1] + hi[1] * hi[1]);
    const float rstd = 1.0f / sqrtf(ss / (float)dh + a.eps);
    const float* gam = is_q ? a.gamma_q : a.gamma_k;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int i = lane + c * kWave;
      if (i < half) { lo[c] *= rstd * gam[i]; hi[c] *= rstd * gam[half + i]; }
    }
  }
  if (a.theta > 0.f) {
    const int pos = t - a.cu[seq_of_row(a.cu, a.S, t)];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int i = lane + c * kWave;
      if (i >= half) continue;
      float sn, cs;
      if (sizeof(Tio) == 4) {
        double dsn, dcs;
        sincos((double)pos * exp2(-(double)(2 * i) / (double)dh * log2((double)a.theta)), &dsn, &dcs);
        sn = (float)dsn; cs = (float)dcs;
      } else {
        sincosf(rope_angle(log2f(a.theta), i, dh, pos), &sn, &cs);
      }
      const float p = lo[c], q = hi[c];
      lo[c] = p * cs - q * sn;
      hi[c] = q * cs + p * sn;
    }
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int i = lane + c * kWave;
    if (i < half) { st_elem(row, i, lo[c]); st_elem(row, half + i, hi[c]); }
  }
}

}  // namespace

hipError_t launch_qk_norm_rope(const QkRopeArgs& a, hipStream_t st) {
  if (a.T == 0 || (!a.gamma_q && !(a.theta > 0.f))) return hipSuccess;
  const int heads = a.n_heads + a.n_kv_heads;
  auto aligned = [](const void* p, int64_t ld) { return ((uintptr_t)p & 7u) == 0 && ld % 4 == 0; };
  const bool fast = a.bf16 && a.dh == 128 && aligned(a.Q, a.ldq) && aligned(a.K, a.ldk) &&
                    (((uintptr_t)a.gamma_q | (uintptr_t)a.gamma_k) & 15u) == 0;
  if (fast) {
    k_qk_norm_rope_bf16<<<dim3((unsigned)((a.T + 3) / 4)), 256, 0, st>>>(a);
  } else {
    const int64_t items = (int64_t)a.T * heads;
    if (a.bf16) k_qk_norm_rope_any<bf16_t><<<dim3((unsigned)((items + 3) / 4)), 256, 0, st>>>(a);
    else k_qk_norm_rope_any<float><<<dim3((unsigned)((items + 3) / 4)), 256, 0, st>>>(a);
  }
  return hipGetLastError();
}

hipError_t launch_add_norm(const NormArgs& a, hipStream_t st) {
  if (a.T == 0 || a.d == 0) return hipSuccess;
  const dim3 block(kNormWaves * kWave);
  auto aligned = [](const void* p, int64_t ld) { return p == nullptr || (((uintptr_t)p & 15u) == 0 && ld % 8 == 0); };
  const bool fast = a.bf16 && a.d % 8 == 0 && a.d <= 8192 && aligned(a.X, a.ldx) && aligned(a.R, a.ldr) &&
                    aligned(a.Hsum, a.ldh) && aligned(a.Y, a.ldy) && ((uintptr_t)a.gamma & 15u) == 0 &&
                    ((uintptr_t)a.beta & 15u) == 0;
  if (!fast) {
    const dim3 grid((a.T + kNormWaves - 1) / kNormWaves);
    if (a.bf16) k_add_norm_any<bf16_t><<<grid, block, 0, st>>>(a);
    else k_add_norm_any<float><<<grid, block, 0, st>>>(a);
    return hipGetLastError();
  }
  // One round of workgroups: as many as are resident at once (registers and the LDS copy of gamma and
  // beta allow norm_wgs_per_cu per CU), each wave striding through the rows.  More, smaller
  // workgroups re-stage gamma and beta more often and leave a partial last round; equal shares of
  // consecutive rows leave workgroups out whenever the rows don't divide (6240 rows of 5120 are 3 per
  // wave on 520 of 768 workgroups: norm and sum with the attention between 96.6 us, strided 90.5).
  const int cus = compute_units();
  const int per_round = cus * norm_wgs_per_cu((a.d + 511) / 512), all = (a.T + kNormWaves - 1) / kNormWaves;
  const dim3 grid(all < per_round ? all : per_round);
  auto launch = [&](auto chunks) {
    constexpr int kChunks = decltype(chunks)::value;
    if (a.R) k_add_norm_bf16<kChunks, true><<<grid, block, 0, st>>>(a);
    else k_add_norm_bf16<kChunks, false><<<grid, block, 0, st>>>(a);
  };
  switch ((a.d + 1023) / 1024) {   // (one chunk at most is empty: an empty one costs as much as another, 5 % of 2474 rows of 5120)
    case 1: launch(std::integral_constant<int, 2>{}); break;
    case 2: launch(std::integral_constant<int, 4>{}); break;
    case 3: launch(std::integral_constant<int, 6>{}); break;
    case 4: launch(std::integral_constant<int, 8>{}); break;
    case 5: launch(std::integral_constant<int, 10>{}); break;
    case 6: launch(std::integral_constant<int, 12>{}); break;
    case 7: launch(std::integral_constant<int, 14>{}); break;
    default: launch(std::integral_constant<int, 16>{}); break;
  }
  return hipGetLastError();
}

int attention_f32_max_head_dim() { return kAttnF32MaxDh; }
int attention_bf16_head_dim() { return kDh; }

hipError_t launch_attention(const AttnArgs& a, hipStream_t st) {
  if (a.T == 0 || a.S == 0 || a.n_heads == 0) return hipSuccess;
  if (a.bf16) {
    const dim3 grid(((a.T + kBQ - 1) / kBQ + a.S) * a.n_heads);
    k_attention_bf16<<<grid, kAttnWaves * kWave, 2 * (kKStage + kVStage), st>>>(a);
  } else {
    const dim3 grid(a.T, a.n_heads);
    k_attention_f32<<<grid, kWave, 0, st>>>(a);
  }
  return hipGetLastError();
}

}  // namespace zo
