// Preparation kernels: factor generation (Philox4x32-10 + Box-Muller; the
// seed-regenerated directions of Sec. 2.2 with the N(0,1) entries of Sec. 3.3),
// packing indices of the variable-length batch (Sec. 3.1) and the operand
// images the matrix-core kernels consume.
#include "zo_device.hpp"
#include "zo_internal.hpp"

namespace zo {

// ---- raw words / standalone factor fill ------------------------------------------
__global__ void k_philox_words(uint64_t seed, uint32_t tensor_id, uint64_t first_block,
                               int64_t n_blocks, uint4* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_blocks) return;
  out[i] = factor_block(seed, tensor_id, first_block + (uint64_t)i);
}

__global__ void k_factor_fill(uint64_t seed, uint32_t tensor_id, int64_t n_elems, int bf16, void* out) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q * 4 >= n_elems) return;
  const uint4 w = factor_block(seed, tensor_id, (uint64_t)q);
  float z[4];
  box_muller(w.x, w.y, z[0], z[1]);
  box_muller(w.z, w.w, z[2], z[3]);
#pragma unroll
  for (int l = 0; l < 4; ++l) {
    const int64_t e = q * 4 + l;
    if (e < n_elems) {
      if (bf16) ((bf16_t*)out)[e] = f32_to_bf16(z[l]);
      else ((float*)out)[e] = z[l];
    }
  }
}

hipError_t launch_philox_words(uint64_t seed, uint32_t tensor_id, uint64_t first_block,
                               int64_t n_blocks, uint32_t* out, hipStream_t st) {
  if (n_blocks == 0) return hipSuccess;
  const int64_t grid = (n_blocks + 255) / 256;
  hipLaunchKernelGGL(k_philox_words, dim3((unsigned)grid), dim3(256), 0, st, seed, tensor_id, first_block,
                     n_blocks, (uint4*)out);
  return hipGetLastError();
}

hipError_t launch_factor_fill(uint64_t seed, uint32_t tensor_id, int64_t rows, int r, int bf16,
                              void* out, hipStream_t st) {
  const int64_t n = rows * r;
  if (n == 0) return hipSuccess;
  const int64_t blocks = (n + 3) / 4;
  hipLaunchKernelGGL(k_factor_fill, dim3((unsigned)((blocks + 255) / 256)), dim3(256), 0, st, seed,
                     tensor_id, n, bf16, out);
  return hipGetLastError();
}

// ---- packing indices -----------------------------------------------------------------
// tok_seq[t] = largest s with cu[s] <= t (empty sequences share an offset with
// their successor; the last of them is the one that owns row t).
__device__ __forceinline__ int seq_of_row(const int32_t* cu, int S, int t) {
  int lo = 0, hi = S;  // invariant: cu[lo] <= t, answer in [lo, hi)
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (cu[mid] <= t) lo = mid; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ void tok_index_at(const BatchDev& b, int t, int32_t* tok_seq, int32_t* tok_cand) {
  if (t >= b.T) return;
  const int s = seq_of_row(b.cu, b.S, t);
  if (tok_seq) tok_seq[t] = s;
  if (tok_cand) tok_cand[t] = b.seq_cand[s];
}

__global__ void k_tok_index(BatchDev b, int32_t* tok_seq, int32_t* tok_cand) {
  tok_index_at(b, blockIdx.x * blockDim.x + threadIdx.x, tok_seq, tok_cand);
}

hipError_t launch_tok_index(const BatchDev& b, int32_t* tok_seq, int32_t* tok_cand, hipStream_t st) {
  if (b.T == 0) return hipSuccess;
  hipLaunchKernelGGL(k_tok_index, dim3((b.T + 255) / 256), dim3(256), 0, st, b, tok_seq, tok_cand);
  return hipGetLastError();
}

// Exclusive prefix sum of one value per thread over a block of 1024 threads, of which only the first n have one (n is the same
// in every thread); *total = the sum.  Up to 64 values are the first wave's own affair (0.4 us less); the other waves get 0.
__device__ __forceinline__ int block_scan_1024(int v, int n, int* s_wave, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int u = __shfl_up(incl, off);
    if (lane >= off) incl += u;
  }
  if (n <= 64) {
    *total = __shfl(incl, 63);
    return incl - v;
  }
  __syncthreads();   // the previous scan's totals have been read
  if (lane == 63) s_wave[wave] = incl;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    const int x = s_wave[w];
    before += w < wave ? x : 0;
    all += x;
  }
  *total = all;
  return before + incl - v;
}

// Per-sequence kind / scale and the list of side-down work items (chunks of at most item_rows rows of one sequence).
// One workgroup; sequences are scanned in blocks of 1024 so the item order follows the row order.  This workgroup and the
// one of the token tiles below are the longest chains of a preparation launch of a small batch (the images are there after 2
// to 3 us), so they run side by side, each reading the batch's tables for itself: one after the other, with a thread per
// tile, they took 5.2 us of a prompt pair, 7.4 of 34 sequences on 6 tiles.
__device__ __forceinline__ void seq_tables_block(const BatchDev& b, float eps, const SeqTables& t) {
  __shared__ int s_wave[16];
  const int tid = threadIdx.x;
  int carry = 0;
  for (int base = 0; base < b.S; base += 1024) {
    const int s = base + tid;
    int row0 = 0, len = 0, kind = kKindForeground, nchunk = 0;
    float scale = 0.0f;
    if (s < b.S) {
      row0 = b.cu[s];
      const int next = b.cu[s + 1];
      const int c = b.seq_cand[s];
      len = max(next - row0, 0);
      candidate_kind(c, b.C, b.K, eps, b.cand_dir, b.cand_sign, kind, scale);
      t.seq_kind[s] = kind;
      t.seq_scale[s] = scale;
      // (a foreground sequence has no side term: no items, none of its rows is read by the side-down pass)
      nchunk = kind == kKindForeground ? 0 : (len + t.item_rows - 1) / t.item_rows;
    }
    int total;
    const int first = carry + block_scan_1024(nchunk, min(b.S - base, 1024), s_wave, &total);
    for (int j = 0; j < nchunk; ++j) {
      if (first + j < t.max_items) {
        SideItem it;
        it.row0 = row0 + j * t.item_rows;
        it.nrows = min(t.item_rows, len - j * t.item_rows);
        it.kind = kind;
        it.scale = scale;
        t.items[first + j] = it;
      }
    }
    carry += total;
  }
  if (tid == 0) t.n_items[0] = min(carry, t.max_items);
}

// Largest s in [0, S) with cu[s] <= t, found by a wave: a 64th of the range per step.
__device__ __forceinline__ int wave_seq_of_row(const int32_t* cu, int S, int t, int lane) {
  int base = 0, n = S;
  while (n > 1) {
    const int step = (n + 63) >> 6, at = lane * step;
    const int k = max(__popcll(__ballot(at < n && cu[base + min(at, n - 1)] <= t)) - 1, 0);
    base += k * step;
    n = min(step, n - k * step);
  }
  return base;
}

// The side K tiles of every token tile of the bf16 GEMM.  A tile's slot list names the distinct directions of the
// sequences that intersect it, in order of first appearance, SPD slots each.  One workgroup.  Where a tile's slots lie needs
// no knowledge of the tiles before it: with s the first sequence of tile i, at most s + i (tile, sequence) intersections do.
//
// Up to kFewTiles tiles are taken one by a wave, whose lanes share the searches and the sequences: the shortest chain.  A
// wave needs 0.4 us and more for a tile, so with more tiles (kMany) a thread searches for each, and walks its sequences too
// unless a tile has many of them (with more than 64 directions, fewer: each is looked up in the tile's list).  Linears of 64 x
// 64, us, a wave for each tile / a thread: up to 64 directions, 36 tiles of 8 sequences 16.5 / 16.8; 64 of 1 24.0 / 21.6, of 8 20.7 /
// 19.8, of 16 20.4 / 21.5; 128 of 16 28.4 / 26.7, of 32 30.4 / 32.9; 512 of one sequence in four 63 / 42.6, of 32 90 / 76, of 64 98 /
// 108; 1024 of 16 160 / 99; beyond 64 directions, 64 of 8 24.2 / 25.3; 128 of 8 30.2 / 27.8, of 16 36.5 / 39.4; 1024 of 16 232 / 171,
// of 64 585 / 1052.  (The chain of a small call is in a kernel of its own: beside this code it took 0.4 us longer.)
constexpr int kFewTiles = 32;

template <bool kMany>
__device__ __forceinline__ void tile_tables_block(const BatchDev& b, const SeqTables& t) {
  constexpr int kCached = kMany ? 4096 : 1024;   // sequences whose bounds and kinds are kept in LDS
  __shared__ int s_wave[16], s_cu[kCached + 1], s_kind[kCached];
  __shared__ int s_tile[1024], s_slot0[1024];   // directions of a tile (bit 31: it holds a candidate's row), its first slot
  __shared__ int s_dirs[16][kTileN];    // a wave's tile: the directions met so far
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool cached = b.S <= kCached;
  auto kind_of = [&](int s) {
    int kind;
    float scale;
    candidate_kind(b.seq_cand[s], b.C, b.K, 1.0f, b.cand_dir, b.cand_sign, kind, scale);
    return kind;
  };
  auto keep = [&](int s) {
    s_cu[s] = b.cu[s];
    if (s == b.S - 1) s_cu[b.S] = b.cu[b.S];
    s_kind[s] = kind_of(s);
  };
  if constexpr (kMany) {
    for (int s = tid; cached && s < b.S; s += 1024) keep(s);
  } else {
    if (cached && tid < b.S) keep(tid);
  }
  __syncthreads();
  const int32_t* cu = cached ? s_cu : b.cu;
  const int per_tile = min(b.K, kTileN);
  const bool by_sequence = (int64_t)t.n_tn + b.S <= (int64_t)t.n_tn * per_tile;   // (which of the two bounds slot_cap is)
  int kt_carry = 0;
  for (int base = 0; base < t.n_tn; base += 1024) {
    const int n_here = min(t.n_tn - base, 1024);
    const int tn_own = base + tid;   // a thread's tile: its first and last sequence
    int s_first = 0, s_last = 0;
    bool by_wave = true;
    if constexpr (kMany) {
      if (tid < n_here) {
        const int t0 = tn_own * kTileN;
        s_first = seq_of_row(cu, b.S, t0);
        s_last = seq_of_row(cu, b.S, min(b.T, t0 + kTileN) - 1);
        s_slot0[tid] = s_first;
        s_tile[tid] = s_last;
      }
      const int most = b.K > 64 ? min(n_here / 12, 20) : min(n_here / 6 + 1, 60);
      by_wave = __syncthreads_or(s_last - s_first >= most);
    }
    if (by_wave) {
      // the wave's lanes look at 64 of the tile's sequences at a time and tell one by one which bring a direction
      for (int i = wave; i < n_here; i += 16) {
        const int tn = base + i, t0 = tn * kTileN, t1 = min(b.T, t0 + kTileN);
        const int first = kMany ? __builtin_amdgcn_readfirstlane(s_slot0[i]) : wave_seq_of_row(cu, b.S, t0, lane);
        const int last = kMany ? __builtin_amdgcn_readfirstlane(s_tile[i]) : wave_seq_of_row(cu, b.S, t1 - 1, lane);
        const int slot0 = (by_sequence ? first + tn : tn * per_tile) * t.SPD;
        int q = 0;
        bool any = false;
        for (int s0 = first; s0 <= last; s0 += 64) {
          const int s = min(s0 + lane, last);
          const bool rows = s0 + lane <= last && min(cu[s + 1], t1) > max(cu[s], t0);
          const int kind = rows ? (cached ? s_kind[s] : kind_of(s)) : kKindForeground;
          any |= __ballot(kind >= kKindCentre) != 0;
          uint64_t left = __ballot(kind >= 0);
          for (int j = 0; j < (s0 > first ? q : 0); ++j) left &= ~__ballot(kind == s_dirs[wave][j]);
          uint64_t first_of = 0;   // lanes whose sequence brings a direction
          while (left) {
            const int at = __ffsll((unsigned long long)left) - 1;
            first_of |= 1ull << at;
            left &= ~__ballot(kind == __builtin_amdgcn_readlane(kind, at));
          }
          const int nth = q + __popcll(first_of & ((1ull << lane) - 1ull));
          if (((first_of >> lane) & 1) && slot0 + (nth + 1) * t.SPD <= t.slot_cap) {   // (the cap is a bound)
            s_dirs[wave][nth] = kind;
            for (int blk = 0; blk < t.SPD; ++blk) t.tile_slots[slot0 + nth * t.SPD + blk] = kind * t.SPD + blk;
          }
          q += __popcll(first_of);
        }
        if (lane == 0) {
          s_tile[i] = q | (any ? 1 << 31 : 0);
          s_slot0[i] = slot0;
        }
      }
    } else if (tid < n_here) {
      const int t0 = tn_own * kTileN, t1 = min(b.T, t0 + kTileN);
      const int slot0 = (by_sequence ? s_first + tn_own : tn_own * per_tile) * t.SPD;
      int q = 0;
      bool any = false;
      uint64_t met = 0;   // directions met so far, when there are at most 64
      for (int s = s_first; s <= s_last; ++s) {
        if (min(cu[s + 1], t1) <= max(cu[s], t0)) continue;   // no row of s in this tile
        const int kind = cached ? s_kind[s] : kind_of(s);
        any |= kind >= kKindCentre;
        if (kind < 0) continue;
        bool seen = false;
        if (b.K <= 64) {
          seen = (met >> kind) & 1;
          met |= 1ull << kind;
        } else {
          for (int j = 0; j < q && !seen; ++j) seen = t.tile_slots[slot0 + j * t.SPD] == kind * t.SPD;
        }
        if (!seen && slot0 + (q + 1) * t.SPD <= t.slot_cap) {
          for (int blk = 0; blk < t.SPD; ++blk) t.tile_slots[slot0 + q * t.SPD + blk] = kind * t.SPD + blk;
          ++q;
        }
      }
      s_tile[tid] = q | (any ? 1 << 31 : 0);
      s_slot0[tid] = slot0;
    }
    __syncthreads();
    const int tn = base + tid, met = tid < n_here ? s_tile[tid] : 0;   // (n_here <= 64: only the first wave's scan counts)
    const int n_slots = (met & 0x7FFFFFFF) * t.SPD, n_bank = met < 0 ? t.RpT : 0;
    const int n_kt = tid < n_here ? (n_slots + 1) / 2 + n_bank : 0;
    int total;
    const int kt0 = kt_carry + block_scan_1024(n_kt, n_here, s_wave, &total);
    kt_carry += total;
    if (tid < n_here) {
      TileHdr h;
      h.kt0 = kt0; h.n_slots = n_slots; h.n_bank_kt = n_bank; h.slot0 = s_slot0[tid];
      const bool fits = kt0 + n_kt <= t.kt_cap;
      if (!fits) { h.n_slots = 0; h.n_bank_kt = 0; }   // cannot happen: the caps are bounds
      t.tile_hdr[tn] = h;
      for (int j = 0; fits && j < n_kt; ++j) t.kt_tile[kt0 + j] = tn;
    }
    __syncthreads();   // s_tile is written again
  }
  if (tid == 0) t.n_items[1] = min(kt_carry, t.kt_cap);
}

// ---- operand images ----------------------------------------------------------------------
// Four consecutive columns c0 .. c0+3 of row i of a [rows x r] factor: entries c >= r are zero.
// Entry (i, c) is element e = i*r + c of the stream, i.e. lane e%4 of block e/4; the four entries
// come out of one block when r is a multiple of 4 and out of two neighbouring blocks otherwise.
__device__ __forceinline__ void factor_quad(uint64_t seed, uint32_t tid, int64_t i, int r, int c0, float (&z)[4]) {
  const uint64_t e0 = (uint64_t)i * r + c0;
  float v[8];
  {
    const uint4 w = factor_block(seed, tid, e0 >> 2);
    box_muller(w.x, w.y, v[0], v[1]);
    box_muller(w.z, w.w, v[2], v[3]);
  }
  const int lane0 = (int)(e0 & 3);
  if (lane0 != 0) {
    const uint4 w = factor_block(seed, tid, (e0 >> 2) + 1);
    box_muller(w.x, w.y, v[4], v[5]);
    box_muller(w.z, w.w, v[6], v[7]);
  } else {
    v[4] = v[5] = v[6] = v[7] = 0.0f;
  }
#pragma unroll
  for (int l = 0; l < 4; ++l) {
    float x = 0.0f;
#pragma unroll
    for (int t = 0; t < 8; ++t) x = (t == lane0 + l) ? v[t] : x;   // register select, no indexing
    z[l] = c0 + l < r ? x : 0.0f;
  }
}

// idx = (a * per_a) + b * inner + c with b * inner + c < per_a and c < inner.  32-bit divisions when the numbers
// allow (a 64-bit division costs more instructions than the normals a thread generates).
__device__ __forceinline__ void split3(int64_t idx, int64_t per_a, int inner, int& a, int& b, int& c) {
  if (idx < (1ll << 31) && per_a < (1ll << 31)) {
    const uint32_t x = (uint32_t)idx, pa = (uint32_t)per_a;
    const uint32_t qa = x / pa, rem = x - qa * pa;
    const uint32_t qb = rem / (uint32_t)inner;
    a = (int)qa; b = (int)qb; c = (int)(rem - qb * (uint32_t)inner);
  } else {
    const int64_t qa = idx / per_a, rem = idx - qa * per_a;
    const int64_t qb = rem / inner;
    a = (int)qa; b = (int)qb; c = (int)(rem - qb * inner);
  }
}

// idx runs over [K][m_img][SPD * 4]: one thread writes eight neighbouring entries of a row of U (16 bytes) into
// the image [K * SPD][m_img][32]; rows >= m and columns >= r are zero
__device__ __forceinline__ void image_U_at(const BatchDev& b, int64_t idx, uint32_t tid_u, int m, int m_img, int r, int SPD,
                                           bf16_t* Uimg) {
  const int groups = SPD * 4;
  const int64_t per_dir = (int64_t)m_img * groups;
  if (idx >= per_dir * b.K) return;
  int k, i, c0;
  split3(idx, per_dir, groups, k, i, c0);
  c0 *= 8;
  float z[2][4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  if (i < m && c0 < r) {
    factor_quad(b.seed[k], tid_u, i, r, c0, z[0]);
    if (c0 + 4 < r) factor_quad(b.seed[k], tid_u, i, r, c0 + 4, z[1]);
  }
  *reinterpret_cast<u32x4*>(Uimg + (((int64_t)k * SPD + (c0 >> 5)) * m_img + i) * 32 + (c0 & 31)) =
      u32x4{pack_bf16x2(z[0][0], z[0][1]), pack_bf16x2(z[0][2], z[0][3]), pack_bf16x2(z[1][0], z[1][1]), pack_bf16x2(z[1][2], z[1][3])};
}

// Where entry i of row c of a transposed factor (V^T or Vb^T, rows padded to blocks of 16) lives: row-major, or in
// the order of the side-down matrix instruction's operands (frag_major): [block of 16 rows][32 columns][lane][8], lane =
// row % 16 + 16 * (column / 8 % 4).  Entries i .. i+7 of a multiple of 8 are neighbours either way.
__device__ __forceinline__ int64_t transposed_at(int c, int i, int n, bool frag_major) {
  return frag_major ? ((int64_t)(c >> 4) * (n >> 5) + (i >> 5)) * 512 + ((c & 15) + ((i >> 3) & 3) * 16) * 8 + (i & 7)
                    : (int64_t)c * n + i;
}

// idx runs over [K][RP/4][n/2]: one thread writes entries i, i+1 of four neighbouring rows of V^T (n is even)
__device__ __forceinline__ void image_Vt_at(const BatchDev& b, int64_t idx, uint32_t tid_v, int n, int r, int RP, bool frag_major,
                                            bf16_t* Vt) {
  const int quads = RP >> 2, half = n >> 1;
  const int64_t per_dir = (int64_t)half * quads;
  if (idx >= per_dir * b.K) return;
  int k, c0, i;
  split3(idx, per_dir, half, k, c0, i);
  c0 *= 4;
  i *= 2;
  float z[2][4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  if (c0 < r) {
    const uint64_t seed = b.seed_v ? b.seed_v[k] : b.seed[k];
    factor_quad(seed, tid_v, i, r, c0, z[0]);
    factor_quad(seed, tid_v, i + 1, r, c0, z[1]);
  }
  bf16_t* dst = Vt + (int64_t)k * RP * n;
#pragma unroll
  for (int l = 0; l < 4; ++l) *reinterpret_cast<uint32_t*>(dst + transposed_at(c0 + l, i, n, frag_major)) = pack_bf16x2(z[0][l], z[1][l]);
}

// idx runs over [n/8][Rp]: one thread writes entries i .. i+7 of one row of Vb^T in operand order (neighbouring threads
// read neighbouring columns of Vb and write neighbouring 16 bytes); columns >= R_used are zero
__device__ __forceinline__ void image_Vb_frag_at(int64_t idx, const float* Vb, int R_cap, int R_used, int Rp, int n, bf16_t* Vbt) {
  if (idx >= (int64_t)(n >> 3) * Rp) return;
  const int i = (int)(idx / Rp) * 8, j = (int)(idx % Rp);
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = j < R_used ? Vb[(int64_t)(i + e) * R_cap + j] : 0.0f;
  *reinterpret_cast<u32x4*>(Vbt + transposed_at(j, i, n, true)) =
      u32x4{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
}

// idx runs over [m_img][RpT * 8]: one thread writes eight neighbouring entries (16 bytes) of the image [RpT][m_img][64]
// of P; rows >= m and columns >= R_used are zero
__device__ __forceinline__ void image_P_at(int64_t idx, const float* P, int R_cap, int R_used, int RpT, int m, int m_img,
                                           bf16_t* Pimg) {
  const int groups = RpT * 8;
  if (idx >= (int64_t)m_img * groups) return;
  int zero, i, j;
  split3(idx, (int64_t)m_img * groups, groups, zero, i, j);
  j *= 8;
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (i < m) {
    const float* src = P + (int64_t)i * R_cap + j;
    if (j + 8 <= R_used && ((uintptr_t)src & 15u) == 0) {
      const float4 a = reinterpret_cast<const float4*>(src)[0], c = reinterpret_cast<const float4*>(src)[1];
      v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = c.x; v[5] = c.y; v[6] = c.z; v[7] = c.w;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (j + e < R_used) v[e] = src[e];
    }
  }
  *reinterpret_cast<u32x4*>(Pimg + ((int64_t)(j >> 6) * m_img + i) * 64 + (j & 63)) =
      u32x4{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
}

// ---- everything an fp32 probe linear prepares, in one launch ----------------------------------
// Four consecutive entries 4q .. 4q+3 of a factor stream (one Philox block) of direction k into out[k][rows*r].
// idx runs over [K][ceil(rows*r/4)].
__device__ __forceinline__ void factor_f32_at(const BatchDev& b, const uint64_t* seeds, int64_t idx, uint32_t tid, int rows,
                                              int r, float* out) {
  const int64_t per_dir = (int64_t)rows * r, quads = (per_dir + 3) / 4;
  if (idx >= quads * b.K) return;
  const int k = (int)(idx / quads);
  const int64_t q = idx - (int64_t)k * quads;
  const uint4 w = factor_block(seeds[k], tid, (uint64_t)q);
  float z[4];
  box_muller(w.x, w.y, z[0], z[1]);
  box_muller(w.z, w.w, z[2], z[3]);
#pragma unroll
  for (int l = 0; l < 4; ++l)
    if (q * 4 + l < per_dir) out[(int64_t)k * per_dir + q * 4 + l] = z[l];
}

// Block roles, in order: [sequence tables: 1] [token -> sequence map] [U] [V].
__global__ __launch_bounds__(1024) void k_probe_prep_f32(BatchDev b, float eps, SeqTables t, uint32_t tensor_id, int m, int n,
                                                         int r, float* Uf, float* Vf, int nb_tok, int nb_U) {
  int blk = blockIdx.x;
  if (blk == 0) { seq_tables_block(b, eps, t); return; }
  blk -= 1;
  if (blk < nb_tok) { tok_index_at(b, blk * 1024 + threadIdx.x, t.tok_seq, nullptr); return; }
  blk -= nb_tok;
  if (blk < nb_U) { factor_f32_at(b, b.seed, (int64_t)blk * 1024 + threadIdx.x, tensor_id & ~1u, m, r, Uf); return; }
  blk -= nb_U;
  factor_f32_at(b, b.seed_v ? b.seed_v : b.seed, (int64_t)blk * 1024 + threadIdx.x, tensor_id | 1u, n, r, Vf);
}

hipError_t launch_probe_prep_f32(const BatchDev& b, float eps, const SeqTables& t, uint32_t tensor_id, int m, int n, int r,
                                 float* Uf, float* Vf, hipStream_t st) {
  auto blocks = [&](int rows) { return (int)(((((int64_t)rows * r + 3) / 4) * b.K + 1023) / 1024); };
  const int nb_tok = (b.T + 1023) / 1024, nb_U = blocks(m), nb_V = blocks(n);
  hipLaunchKernelGGL(k_probe_prep_f32, dim3(1 + nb_tok + nb_U + nb_V), dim3(1024), 0, st, b, eps, t, tensor_id, m, n, r, Uf,
                     Vf, nb_tok, nb_U);
  return hipGetLastError();
}

// ---- everything a bf16 probe linear prepares before its side-down pass, in one launch ------
// Block roles, in order: [sequence tables: 1] [token tiles: 1] [token -> sequence map] [U image] [V^T image]
// [P image] [Vb^T image: 32x32 transposing tiles, or 16-byte pieces in operand order].  The pieces do not depend on one another.
struct ProbePrepArgs {
  BatchDev b; float eps; SeqTables tabs;
  uint32_t tensor_id; int m, n, r, RP, Rp, m_img;
  const float* P; const float* Vb; int R_cap, R_used;
  bf16_t* Uimg; bf16_t* Vt; bf16_t* Pimg; bf16_t* Vbt;
  int nb_tok, nb_U, nb_Vt, nb_P, nb_Vbt, vbt_tiles_n;
};

template <bool kMany>   // more than kFewTiles token tiles
__global__ __launch_bounds__(1024) void k_probe_prep(ProbePrepArgs a) {
  int blk = blockIdx.x;
  if (blk == 0) { seq_tables_block(a.b, a.eps, a.tabs); return; }
  if (blk == 1) { tile_tables_block<kMany>(a.b, a.tabs); return; }
  blk -= 2;
  if (blk < a.nb_tok) { tok_index_at(a.b, blk * 1024 + threadIdx.x, a.tabs.tok_seq, nullptr); return; }
  blk -= a.nb_tok;
  if (blk < a.nb_U) { image_U_at(a.b, (int64_t)blk * 1024 + threadIdx.x, a.tensor_id & ~1u, a.m, a.m_img, a.r, a.tabs.SPD, a.Uimg); return; }
  blk -= a.nb_U;
  if (blk < a.nb_Vt) { image_Vt_at(a.b, (int64_t)blk * 1024 + threadIdx.x, a.tensor_id | 1u, a.n, a.r, a.RP, a.tabs.frag_major, a.Vt); return; }
  blk -= a.nb_Vt;
  if (blk < a.nb_P) { image_P_at((int64_t)blk * 1024 + threadIdx.x, a.P, a.R_cap, a.R_used, a.tabs.RpT, a.m, a.m_img, a.Pimg); return; }
  blk -= a.nb_P;
  if (a.tabs.frag_major) { image_Vb_frag_at((int64_t)blk * 1024 + threadIdx.x, a.Vb, a.R_cap, a.R_used, a.Rp, a.n, a.Vbt); return; }
  // Vbt[j][i] = Vb[i][j], one 32x32 tile per block, coalesced on both sides
  __shared__ float tile[32][33];
  const int i0 = (blk % a.vbt_tiles_n) * 32, j0 = (blk / a.vbt_tiles_n) * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  {
    const int i = i0 + ty, j = j0 + tx;
    tile[ty][tx] = (i < a.n && j < a.R_used) ? a.Vb[(int64_t)i * a.R_cap + j] : 0.0f;
  }
  __syncthreads();
  {
    const int j = j0 + ty, i = i0 + tx;
    if (j < a.Rp && i < a.n) a.Vbt[(int64_t)j * a.n + i] = f32_to_bf16(tile[tx][ty]);
  }
}

hipError_t launch_probe_prep_bf16(const BatchDev& b, float eps, const SeqTables& tabs, uint32_t tensor_id, int m,
                                  int n, int r, int RP, int Rp, const float* P, const float* Vb, int R_cap,
                                  int R_used, int m_img, uint16_t* Uimg, uint16_t* Vt, uint16_t* Pimg, uint16_t* Vbt,
                                  hipStream_t st) {
  ProbePrepArgs a;
  a.b = b; a.eps = eps; a.tabs = tabs; a.tensor_id = tensor_id; a.m = m; a.n = n; a.r = r; a.RP = RP; a.Rp = Rp;
  a.P = P; a.Vb = Vb; a.R_cap = R_cap; a.R_used = R_used; a.Uimg = Uimg; a.Vt = Vt; a.Pimg = Pimg; a.Vbt = Vbt;
  a.m_img = m_img;
  auto blocks = [](int64_t n_elems) { return (int)((n_elems + 1023) / 1024); };
  a.nb_tok = blocks(b.T);
  a.nb_U = blocks((int64_t)b.K * m_img * (tabs.SPD * 4));
  a.nb_Vt = blocks((int64_t)b.K * (n / 2) * (RP / 4));
  a.nb_P = Rp > 0 ? blocks((int64_t)m_img * tabs.RpT * 8) : 0;
  a.vbt_tiles_n = (n + 31) / 32;
  a.nb_Vbt = Rp == 0 ? 0 : tabs.frag_major ? blocks((int64_t)(n / 8) * Rp) : a.vbt_tiles_n * ((Rp + 31) / 32);
  const int64_t total = 2 + (int64_t)a.nb_tok + a.nb_U + a.nb_Vt + a.nb_P + a.nb_Vbt;
  if (tabs.n_tn > kFewTiles) hipLaunchKernelGGL(k_probe_prep<true>, dim3((unsigned)total), dim3(1024), 0, st, a);
  else hipLaunchKernelGGL(k_probe_prep<false>, dim3((unsigned)total), dim3(1024), 0, st, a);
  return hipGetLastError();
}

// ---- device-resident schedule of the multi-step loop (Sec. 3.2) ---------------------------
__global__ __launch_bounds__(256) void k_schedule_step(SchedDev* s, int nu, int n_blocks, int K, uint64_t base_u,
                                                       uint64_t base_v, uint64_t* seed_u, uint64_t* seed_v) {
  const int64_t t = s->next_step;
  __syncthreads();   // every thread has read the step number before thread 0 advances it
  const int64_t interval = t / nu;
  for (int j = threadIdx.x; j < K; j += blockDim.x) {
    seed_u[j] = base_u + (uint64_t)t * (uint64_t)K + (uint64_t)j;
    seed_v[j] = base_v + (uint64_t)interval * (uint64_t)K + (uint64_t)j;
  }
  if (threadIdx.x == 0) {
    s->step = t;
    s->interval = (int32_t)interval;
    s->block = (int32_t)(interval % n_blocks);
    s->append = (t % nu == 0) ? 1 : 0;
    s->reserved = 0;
    s->next_step = t + 1;
  }
}

hipError_t launch_schedule_step(SchedDev* s, int nu, int n_blocks, int K, uint64_t base_u, uint64_t base_v,
                                uint64_t* seed_u, uint64_t* seed_v, hipStream_t st) {
  hipLaunchKernelGGL(k_schedule_step, dim3(1), dim3(256), 0, st, s, nu, n_blocks, K, base_u, base_v, seed_u, seed_v);
  return hipGetLastError();
}

}  // namespace zo
