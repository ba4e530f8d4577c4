// The probe linear (Sec. 3.2) for batches that leave most of the chip idle when cut into 256x256 tiles: the
// same arithmetic on smaller output tiles, from 32x32 to 160x256, one tile per workgroup.
//
// Such a call is bound by how fast the operands reach the compute units, not by the matrix cores: the weight
// matrix comes once from HBM and every workgroup pulls its rows of both operands from L2.  The kernel
// therefore keeps several K stages in flight per workgroup (direct-to-LDS loads into a ring of S stages), and
// for the smallest tiles a stage is 256 columns wide, so that a load instruction covers two rows of 512
// contiguous bytes instead of eight of 128: row pitches of 4096 elements and their multiples put the same
// columns of all rows on the same memory channels.
//
// Every output element is accumulated by the same chain of v_mfma_f32_16x16x32_bf16 as in the large kernel
// (side K tiles, then the base columns in ascending order, C = +0 first), so which kernel a call takes does
// not show in its results: a row's bits do not depend on how many other rows are in the batch.
#include <type_traits>

#include "zo_device.hpp"
#include "zo_internal.hpp"

namespace zo {
namespace {

typedef __attribute__((address_space(3))) void lds_void;

// silu(gate) * up (activation 2)
__device__ __forceinline__ float silu_mul(float gate, float up) { return gate / (1.0f + __expf(-gate)) * up; }

// Tile of TM weight rows x TN tokens; WR x WC waves, each (TM/WR) x (TN/WC); K stages of KC columns; ring of S.
// An LDS row of a stage is KC*2 bytes in 16-byte chunks; chunk c of row `row` is stored at c ^ key(row), which
// spreads the 16 rows of a fragment read over all banks.
template <int TM_, int TN_, int WR_, int WC_, int KC_, int S_>
struct SmallTile {
  static constexpr int TM = TM_, TN = TN_, WR = WR_, WC = WC_, KC = KC_, S = S_;
  static constexpr int kWaves = WR * WC;
  static constexpr int RB = TM / WR / 16, CB = TN / WC / 16;
  static constexpr int CPR = KC / 8;                          // 16-byte chunks per row
  static constexpr int kRowBytes = KC * 2;
  static constexpr int kStage = (TM + TN) * kRowBytes;
  // direct-to-LDS loads of 1 KiB, neighbouring blocks of the A part, then of the B part, of a stage; where the A part does not
  // come out even over the waves, they are dealt in turn and the last waves repeat the last block
  static constexpr int kBlocksA = TM * kRowBytes / 1024, kBlocksB = TN * kRowBytes / 1024;
  static constexpr int kLoadsA = (kBlocksA + kWaves - 1) / kWaves, kLoadsB = kBlocksB / kWaves;
  static constexpr int kLoads = kLoadsA + kLoadsB;            // of a wave per stage
  static constexpr int kLds = S * kStage;
  static constexpr int kSideTiles = KC / kTileK;              // side K tiles per stage
  static_assert(TM * kRowBytes % 1024 == 0 && TN * kRowBytes % (1024 * kWaves) == 0, "whole loads");
  static_assert((S - 1) * kLoads <= 63, "the load counter holds 6 bits");
  static_assert(kLds <= 160 * 1024, "LDS of a compute unit");
  static_assert(kTileN % TN == 0, "a token tile of this kernel lies inside one tile of the side tables");
  __device__ static int key(int row) { return KC == 64 ? (row >> 1) & 7 : row & 15; }
};

template <class C, bool kSide, bool kOutBf16, bool kGate, bool kBias>
__global__ __launch_bounds__(C::kWaves * 64, 1) void k_probe_gemm_small(ProbeGemmArgs p, int n_tm, int n_tn) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wr = wave / C::WC, wc = wave % C::WC;
  const int r16 = lane & 15, g = lane >> 4;

  // Workgroup -> tile.  Consecutive workgroup ids land on consecutive XCDs; an XCD takes a contiguous range of
  // weight rows and all token tiles of them next to each other, so a weight row is fetched into one L2 only.
  const int per_xcd = gridDim.x / 8;
  const int pos = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (pos >= n_tm * n_tn) return;
  const int tm = pos / n_tn, tn = pos - tm * n_tn;
  const int m0 = tm * C::TM, t0 = tn * C::TN;

  // side K tiles of the token tile
  TileHdr h{0, 0, 0, 0};
  int tr = 0;   // row of t0 in the 256-row tile of the side tables
  if constexpr (kSide) {
    h = p.tile_hdr[t0 / kTileN];
    h.kt0 = __builtin_amdgcn_readfirstlane(h.kt0);
    h.n_slots = __builtin_amdgcn_readfirstlane(h.n_slots);
    h.n_bank_kt = __builtin_amdgcn_readfirstlane(h.n_bank_kt);
    h.slot0 = __builtin_amdgcn_readfirstlane(h.slot0);
    tr = t0 % kTileN;
  }
  const int n_dir_kt = (h.n_slots + 1) >> 1;
  const int n_side = n_dir_kt + h.n_bank_kt;
  const int n_side_st = (n_side + C::kSideTiles - 1) / C::kSideTiles;
  const int n_st = n_side_st + (p.n + C::KC - 1) / C::KC;

  // Load j of a wave fills a 1 KiB block of the A part, then of the B part, of a stage; lane i lands at byte 16 i of it.
  // Rows past the end of a matrix repeat its last row (never stored), columns past the end of a row in its last stage are
  // whatever follows (never multiplied; the windows bound every access).
  constexpr int kRowsPerLoad = 64 / C::CPR;
  const int lrow = lane / C::CPR, lchunk = lane % C::CPR;
  auto block_of = [&](int j) {
    if (j >= C::kLoadsA) return wave * C::kLoadsB + j - C::kLoadsA;
    return C::kBlocksA % C::kWaves == 0 ? wave * C::kLoadsA + j : min(j * C::kWaves + wave, C::kBlocksA - 1);
  };
  uint32_t off[C::kLoads];
#pragma unroll
  for (int j = 0; j < C::kLoads; ++j) {
    const bool isA = j < C::kLoadsA;
    const int row = block_of(j) * kRowsPerLoad + lrow;
    const int ch = lchunk ^ C::key(row);
    const int r = isA ? min(row, p.m - 1 - m0) : min(row, p.T - 1 - t0);
    off[j] = __umul24((uint32_t)r, (uint32_t)(isA ? p.ldw : p.ldx) * 2u) + ch * 16;
  }
  const int64_t bytesA = ((int64_t)(p.m - m0 - 1) * p.ldw + p.n) * 2;
  const int64_t bytesB = ((int64_t)(p.T - t0 - 1) * p.ldx + p.n) * 2;
  const __amdgpu_buffer_rsrc_t rA = __builtin_amdgcn_make_buffer_rsrc((void*)(p.W + (int64_t)m0 * p.ldw), 0,
                                                                      (int)min(bytesA, (int64_t)0x7FFFFFFF), 0x00020000);
  const __amdgpu_buffer_rsrc_t rB = __builtin_amdgcn_make_buffer_rsrc((void*)(p.X + (int64_t)t0 * p.ldx), 0,
                                                                      (int)min(bytesB, (int64_t)0x7FFFFFFF), 0x00020000);
  auto dst_of = [&](int slot, int j) {
    const bool isA = j < C::kLoadsA;
    return lds + slot * C::kStage + (isA ? 0 : C::TM * C::kRowBytes) + block_of(j) * 1024;
  };
  auto issue_some = [&](int st, int slot, int first, int end) __attribute__((always_inline)) {
    const int soff = st * C::kRowBytes;
#pragma unroll
    for (int j = first; j < end; ++j) {
      if (j < C::kLoadsA) __builtin_amdgcn_raw_ptr_buffer_load_lds(rA, (lds_void*)dst_of(slot, j), 16, (int)off[j], soff, 0, 0);
      else __builtin_amdgcn_raw_ptr_buffer_load_lds(rB, (lds_void*)dst_of(slot, j), 16, (int)off[j], soff, 0, 0);
    }
  };
  auto issue_base = [&](int st, int slot) { issue_some(st, slot, 0, C::kLoads); };
  // Side stage st: the side K tiles st * kSideTiles ..; 64-column K tile q of the token tile is a direction
  // tile (columns 0-31 from slot 2q, 32-63 from slot 2q+1 of the U image) or a bank tile, and pool K tile
  // kt0 + q on the token side.  Lanes past the last K tile repeat it (their k-steps are not multiplied).
  const __amdgpu_buffer_rsrc_t rU = __builtin_amdgcn_make_buffer_rsrc((void*)p.Uimg, 0, (int)p.uimg_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rP = __builtin_amdgcn_make_buffer_rsrc((void*)p.Pimg, 0, (int)p.pimg_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rXs = __builtin_amdgcn_make_buffer_rsrc((void*)p.Xs, 0, (int)p.xs_bytes, 0x00020000);
  auto issue_side = [&](int st, int slot) {
    // the U image blocks behind this lane's chunks (table reads first, so that they are waited for once)
    int e[C::kLoadsA];
    if (n_dir_kt > 0) {
#pragma unroll
      for (int j = 0; j < C::kLoadsA; ++j) {
        const int ch = lchunk ^ C::key(block_of(j) * kRowsPerLoad + lrow);
        e[j] = p.tile_slots[h.slot0 + min(2 * (st * C::kSideTiles + (ch >> 3)) + ((ch >> 2) & 1), h.n_slots - 1)];
      }
    } else {
#pragma unroll
      for (int j = 0; j < C::kLoadsA; ++j) e[j] = 0;
    }
#pragma unroll
    for (int j = 0; j < C::kLoads; ++j) {
      const bool isA = j < C::kLoadsA;
      const int row = block_of(j) * kRowsPerLoad + lrow;
      const int ch = lchunk ^ C::key(row);
      const int q = min(st * C::kSideTiles + (ch >> 3), n_side - 1);
      if (!isA) {
        const int src = ((h.kt0 + q) * kTileN + tr + row) * (kTileK * 2) + (ch & 7) * 16;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rXs, (lds_void*)dst_of(slot, j), 16, src, 0, 0, 0);
      } else if (q < n_dir_kt) {   // (lanes of one load may go either way: a lane lands at its own 16 bytes)
        const int src = (e[j] * p.m_img + m0 + row) * 64 + (ch & 3) * 16;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rU, (lds_void*)dst_of(slot, j), 16, src, 0, 0, 0);
      } else {
        const int src = ((q - n_dir_kt) * p.m_img + m0 + row) * 128 + (ch & 7) * 16;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rP, (lds_void*)dst_of(slot, j), 16, src, 0, 0, 0);
      }
    }
  };
  auto issue = [&](int st, int slot) {
    if (kSide && st < n_side_st) issue_side(st, slot);
    else issue_base(st - n_side_st, slot);
  };

  f32x4 acc[C::RB][C::CB];
#pragma unroll
  for (int rb = 0; rb < C::RB; ++rb)
#pragma unroll
    for (int cb = 0; cb < C::CB; ++cb) acc[rb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};

  // fragment reads: lane l holds row l%16, k-values 8*(l/16) .. +7 of the k-step
  const uint32_t aRow = (uint32_t)(wr * (C::TM / C::WR) + r16) * C::kRowBytes;
  const uint32_t bRow = (uint32_t)(C::TM * C::kRowBytes) + (uint32_t)(wc * (C::TN / C::WC) + r16) * C::kRowBytes;
  const uint32_t lane_chunk = (uint32_t)(g ^ C::key(r16)) << 4;   // (a fragment's rows start at a multiple of 16)
  bf16x8 fa[2][C::RB], fb[2][C::CB];
  auto load_frags = [&](int set, const char* s, int ks) __attribute__((always_inline)) {
    const uint32_t c = lane_chunk ^ (uint32_t)(ks << 6);
#pragma unroll
    for (int cb = 0; cb < C::CB; ++cb) fb[set][cb] = *(const bf16x8*)(s + bRow + cb * 16 * C::kRowBytes + c);
#pragma unroll
    for (int rb = 0; rb < C::RB; ++rb) fa[set][rb] = *(const bf16x8*)(s + aRow + rb * 16 * C::kRowBytes + c);
  };
  auto mfmas = [&](int set) __attribute__((always_inline)) {
#pragma unroll
    for (int rb = 0; rb < C::RB; ++rb)
#pragma unroll
      for (int cb = 0; cb < C::CB; ++cb)
        acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[set][rb], fb[set][cb], acc[rb][cb], 0, 0, 0);
  };
  auto wait_loads = [&](auto out_c) __attribute__((always_inline)) {   // until at most `out` loads of this wave are outstanding
    constexpr int out = decltype(out_c)::value;
    static_assert(out <= 63, "the counter holds 6 bits");
    __builtin_amdgcn_s_waitcnt((out & 15) | ((out >> 4) << 14) | (7 << 4) | (15 << 8));
  };

  // Memory returns in order: a stage has landed when no more loads are outstanding than the newer stages have.
  // (A side stage may have issued more: waiting for fewer than are out is only stricter.)
#pragma unroll
  for (int st = 0; st < C::S; ++st)
    if (st < n_st) issue(st, st);
  if (n_st >= C::S) wait_loads(std::integral_constant<int, (C::S - 1) * C::kLoads>{});
  else wait_loads(std::integral_constant<int, 0>{});
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  load_frags(0, lds, 0);
  int slot = 0, st = 0;
  if constexpr (C::KC == 64) {
    // Stages of two k-steps.  First the side stages whose successor S ahead is a side stage too: a few, and their loads are
    // three times as many instructions with the addresses.
    if constexpr (kSide) {
      for (; st + C::S < n_side_st; ++st) {
        const int next = slot == C::S - 1 ? 0 : slot + 1;
        load_frags(1, lds + slot * C::kStage, 1);
        __builtin_amdgcn_sched_barrier(0);
        mfmas(0);
        __builtin_amdgcn_sched_barrier(0);
        wait_loads(std::integral_constant<int, (C::S - 2) * C::kLoads>{});
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        issue_side(st + C::S, slot);
        load_frags(0, lds + next * C::kStage, 0);
        __builtin_amdgcn_sched_barrier(0);
        mfmas(1);
        __builtin_amdgcn_sched_barrier(0);
        slot = next;
      }
    }
    // Then every stage whose successor is one of base columns: loads and fragment reads are spread through the products, one
    // after each group of them: a wave that issues its loads in one burst stands at the memory pipeline's queue (5120 x 20480 at
    // 1560 tokens on 160x256 tiles 387 -> 350 us, on 128x128 565 -> 493; with more side stages than the ring has, 200 bank columns or
    // 24 directions, 5120 x 20480 at 1552 tokens on 160x256 460 -> 410, 5120 x 5120 at 480 on 128x128 75 -> 60).
    auto spread = [&](auto n_loads_c) __attribute__((always_inline)) {
      constexpr int n_loads = decltype(n_loads_c)::value, n = C::RB * C::CB, n_reads = C::RB + C::CB;
#pragma unroll
      for (int i = 0; i < n; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
#pragma unroll
        for (int e = n_reads * i / n; e < n_reads * (i + 1) / n; ++e) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // LDS read
#pragma unroll
        for (int e = n_loads * i / n; e < n_loads * (i + 1) / n; ++e) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // load
      }
    };
    for (; st + C::S < n_st; ++st) {
      const int next = slot == C::S - 1 ? 0 : slot + 1;
      __builtin_amdgcn_sched_barrier(0);
      load_frags(1, lds + slot * C::kStage, 1);
      mfmas(0);
      spread(std::integral_constant<int, 0>{});
      __builtin_amdgcn_sched_barrier(0);
      wait_loads(std::integral_constant<int, (C::S - 2) * C::kLoads>{});
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      issue_base(st + C::S - n_side_st, slot);
      load_frags(0, lds + next * C::kStage, 0);
      mfmas(1);
      spread(std::integral_constant<int, C::kLoads>{});
      __builtin_amdgcn_sched_barrier(0);
      slot = next;
    }
  }
  for (; st < n_st; ++st) {
    const char* s = lds + slot * C::kStage;
    const int next = slot == C::S - 1 ? 0 : slot + 1;
    const int cols = (kSide && st < n_side_st) ? (n_side - st * C::kSideTiles) * kTileK : p.n - (st - n_side_st) * C::KC;
    // every k-step but the stage's last: the next one's fragments are read under this one's products
    constexpr int kSteps = C::KC / 32;
    // Stages of four and eight k-steps: the slot of the stage before takes its successor S ahead a few loads per k-step (all at
    // once after the barrier: one prompt pair through 4096 x 4096 27.7 us instead of 26.7, 44 rows through 5120 x 20480 96 instead of 92).
    const bool late = kSteps > 2 && st > 0 && st - 1 + C::S < n_st && (!kSide || st - 1 + C::S >= n_side_st);
    const int before = slot == 0 ? C::S - 1 : slot - 1;
    if (kSteps > 2 && late && cols >= C::KC) {
#pragma unroll
      for (int ks = 0; ks + 1 < kSteps; ++ks) {
        load_frags((ks + 1) & 1, s, ks + 1);
        issue_some(st - 1 + C::S - n_side_st, before, C::kLoads * ks / (kSteps - 1), C::kLoads * (ks + 1) / (kSteps - 1));
        __builtin_amdgcn_sched_barrier(0);
        mfmas(ks & 1);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else if (kSteps == 2 || cols >= C::KC) {
      if (late) issue_base(st - 1 + C::S - n_side_st, before);
#pragma unroll
      for (int ks = 0; ks + 1 < kSteps; ++ks) {
        load_frags((ks + 1) & 1, s, ks + 1);
        __builtin_amdgcn_sched_barrier(0);
        mfmas(ks & 1);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {   // a side stage or a last stage of fewer columns (whole K tiles of 64)
      if (late) issue_base(st - 1 + C::S - n_side_st, before);
      int ks = 0;
      for (; ks + 2 < cols / 32; ks += 2) {
        load_frags(1, s, ks + 1);
        mfmas(0);
        load_frags(0, s, ks + 2);
        mfmas(1);
      }
      load_frags(1, s, ks + 1);
      mfmas(0);
    }
    // The stage's last k-step multiplies what is already in registers: once every wave has read its fragments
    // the slot can take the stage S ahead, and the next stage's first fragments are read under the products.
    // (Only side stages of more than two k-steps: the others are taken above.)
    if (st + C::S <= n_st) wait_loads(std::integral_constant<int, (C::S - 2) * C::kLoads>{});
    else wait_loads(std::integral_constant<int, 0>{});
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (kSteps > 2 && kSide && st + C::S < n_side_st) issue_side(st + C::S, slot);
    if (st + 1 < n_st) load_frags(0, lds + next * C::kStage, 0);
    __builtin_amdgcn_sched_barrier(0);
    mfmas(1);
    __builtin_amdgcn_sched_barrier(0);
    slot = next;
  }

  // D block (rb, cb): out feature = 16 rb + 4 g + v, token = 16 cb + r16 of the wave's part of the tile
  const bool relu = p.act == 1;
#pragma unroll
  for (int cb = 0; cb < C::CB; ++cb) {
    const int t = t0 + wc * (C::TN / C::WC) + cb * 16 + r16;
    if (t >= p.T) continue;
#pragma unroll
    for (int rb = 0; rb < C::RB; ++rb) {
      const int o = m0 + wr * (C::TM / C::WR) + rb * 16 + 4 * g;
      if (o >= p.m) continue;
      float y[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        y[e] = acc[rb][cb][e];
        if constexpr (kBias) y[e] += p.bias[min(o + e, p.m - 1)];
      }
      if constexpr (kGate) {   // m is even (a multiple of 16 with bf16 output): a pair is inside or outside as a whole
        const float lo = silu_mul(y[0], y[1]), hi = silu_mul(y[2], y[3]);
        if constexpr (kOutBf16) {
          *(uint32_t*)((bf16_t*)p.Y + (int64_t)t * p.ldy + (o >> 1)) = pack_bf16x2(lo, hi);
        } else {
          float* Y = (float*)p.Y + (int64_t)t * p.ldy + (o >> 1);
          Y[0] = lo;
          if (o + 2 < p.m) Y[1] = hi;
        }
      } else {
        // ReLU as a select on the sign, which lets a NaN through
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = (relu && y[e] < 0.0f) ? 0.0f : y[e];
        if constexpr (kOutBf16) {   // m % 8 == 0: four features are inside or outside as a whole
          *(uint2*)((bf16_t*)p.Y + (int64_t)t * p.ldy + o) = make_uint2(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]));
        } else {
          float* Y = (float*)p.Y + (int64_t)t * p.ldy + o;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (o + e < p.m) Y[e] = y[e];
        }
      }
    }
  }
}

template <class C, bool kSide, bool kOutBf16, bool kGate, bool kBias>
hipError_t launch_small(const ProbeGemmArgs& a, hipStream_t st) {
  static std::atomic<bool> configured[kMaxDevices];
  const hipError_t ec = once_per_device(configured, [] {
    return hipFuncSetAttribute((const void*)k_probe_gemm_small<C, kSide, kOutBf16, kGate, kBias>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, C::kLds);
  });
  if (ec != hipSuccess) return ec;
  const int n_tm = (a.m + C::TM - 1) / C::TM, n_tn = (a.T + C::TN - 1) / C::TN;
  const int grid = (n_tm * n_tn + 7) / 8 * 8;
  hipLaunchKernelGGL((k_probe_gemm_small<C, kSide, kOutBf16, kGate, kBias>), dim3(grid), dim3(C::kWaves * 64), C::kLds, st, a, n_tm, n_tn);
  return hipGetLastError();
}

template <class C, bool kSide, bool kOutBf16>
hipError_t launch_act(const ProbeGemmArgs& a, hipStream_t st) {
  if (a.act == 2)
    return a.bias ? launch_small<C, kSide, kOutBf16, true, true>(a, st) : launch_small<C, kSide, kOutBf16, true, false>(a, st);
  return a.bias ? launch_small<C, kSide, kOutBf16, false, true>(a, st) : launch_small<C, kSide, kOutBf16, false, false>(a, st);
}

template <class C>
hipError_t launch_tile(const ProbeGemmArgs& a, hipStream_t st) {
  if (a.has_side) return a.out_bf16 ? launch_act<C, true, true>(a, st) : launch_act<C, true, false>(a, st);
  return a.out_bf16 ? launch_act<C, false, true>(a, st) : launch_act<C, false, false>(a, st);
}

// Tiles and their time per 64 columns of K for one round of workgroups (one per compute unit), in units of
// 10 ns, measured on a 4096-row layer at 4096 and 12288 columns and on a 5120 x 20480 layer (16 .. 1536
// tokens, weights from HBM; a 256x256 tile of the large kernel: 163, half of one: 82).  The more of a tile's
// operands are shared, the less time per element; the smaller the tile, the more compute units have one.
enum { kT32x32, kT32x64, kT64x32, kT64x64, kT64x128, kT128x64, kT128x128, kTiles, kT160x128 = kTiles, kT160x256, kAllTiles };
constexpr struct { int tm, tn, cost; } kTileCost[kAllTiles] = {
    {32, 32, 17}, {32, 64, 20}, {64, 32, 23}, {64, 64, 28}, {64, 128, 43}, {128, 64, 43}, {128, 128, 57}, {160, 128, 66}, {160, 256, 110}};
constexpr int kCostWhole = 163, kCostHalf = 82;

int64_t up(int64_t a, int64_t b) { return (a + b - 1) / b; }
int64_t tile_cost(int T, int m, int tile) {   // tile -1: the 256x256 kernel
  const int64_t cus = compute_units();
  if (tile >= 0) return up(up(m, kTileCost[tile].tm) * up(T, kTileCost[tile].tn), cus) * kTileCost[tile].cost;
  const int64_t whole = up(m, kTileM) * up(T, kTileN), rem = whole % cus;
  return whole / cus * kCostWhole + (rem == 0 ? 0 : (rem <= cus / 2 ? kCostHalf : kCostWhole));
}

}  // namespace

// The tile of up to 128 weight rows that finishes the call soonest by the costs above, or -1 when the 256x256 kernel does.
// (Which one is taken does not enter the result.)  GEMM alone, before -> after, us: 4096 x 4096 at 96 tokens
// 45 -> 14, at 384 45 -> 24, at 768 45 -> 34; 5120 x 20480 at 32 tokens 207 -> 56, at 512 259 -> 193;
// 1024 x 3072 at 1475 tokens 36 -> 19; from about 1500 tokens at 4096 rows up the large kernel is faster than any of these
// (not than the tiles of 160 rows, below).
int small_gemm_tile(int T, int m) {
  int best = -1;
  for (int i = 0; i < kTiles; ++i)
    if (tile_cost(T, m, i) < tile_cost(T, m, best)) best = i;
  return best;
}

// The same with the two tiles of 160 weight rows, for calls of some hundred to some thousand rows whose 256x256 tiles leave part of
// the chip idle in their only round, or most of it in the second.  Their time per round depends more than that of the others
// on how full the round is, so they have to be 5 % ahead.  Whole calls, us, 256x256 -> 160x256: 5120 x 20480 at 1560 tokens
// 497 -> 350, at 1980 538 -> 389; 5120 x 5120 at 1740 128 -> 106; 4096 x 4096 at 2300 116 -> 92; 6144 x 4096 at 3300 180 -> 172
// (two rounds each); 20480 x 5120 at 1300 279 -> 299 (three for two: not taken).  160x128: 5120 x 5120 at 900 81 -> 71.
int gemm_tile(int T, int m) {
  int best = small_gemm_tile(T, m);
  const int64_t cost = tile_cost(T, m, best);
  for (int i = kTiles; i < kAllTiles; ++i)
    if (tile_cost(T, m, i) * 20 < cost * 19 && (best < kTiles || tile_cost(T, m, i) < tile_cost(T, m, best))) best = i;
  return best;
}

hipError_t launch_probe_gemm_small(const ProbeGemmArgs& a, int tile, hipStream_t st) {
  switch (tile) {
    case kT32x32: return launch_tile<SmallTile<32, 32, 2, 2, 256, 4>>(a, st);
    case kT32x64: return launch_tile<SmallTile<32, 64, 2, 2, 256, 3>>(a, st);
    case kT64x32: return launch_tile<SmallTile<64, 32, 2, 2, 256, 3>>(a, st);
    case kT64x64: return launch_tile<SmallTile<64, 64, 4, 2, 128, 4>>(a, st);
    case kT64x128: return launch_tile<SmallTile<64, 128, 2, 4, 64, 3>>(a, st);
    case kT128x64: return launch_tile<SmallTile<128, 64, 4, 2, 128, 3>>(a, st);
    case kT160x128: return launch_tile<SmallTile<160, 128, 2, 4, 64, 4>>(a, st);
    case kT160x256: return launch_tile<SmallTile<160, 256, 2, 4, 64, 3>>(a, st);
    default: return launch_tile<SmallTile<128, 128, 2, 4, 64, 4>>(a, st);
  }
}

}  // namespace zo
