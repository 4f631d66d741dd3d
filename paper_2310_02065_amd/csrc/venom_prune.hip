// One-shot magnitude pruning of a dense fp16 matrix to V:N:M (paper section 3: per V x M block keep
// the four most significant columns, then per row the two most meaningful of those four) and the
// masses the energy metric of section 5 is made of.
//
// "Most significant" is read as the column's L1 mass over the V rows; ties go to the smaller
// index.  Every fp16 is an integer multiple of 2^-24, so magnitudes are handled as integers in
// that unit (Inf and NaN count as 2^40, above any finite value): the masses are exact, no
// summation order exists, and the mask is a pure function of the bits.
#include "venom_internal.h"

namespace venom {

constexpr int kPruneMaxCols = 1024;   // columns (groups x M) one workgroup looks at

__device__ __forceinline__ unsigned long long magnitude_units(uint16_t bits) {
  const unsigned e = (bits >> 10) & 31u, f = bits & 1023u;
  if (e == 0) return f;
  if (e == 31) return 1ull << 40;
  return (unsigned long long)(1024u + f) << (e - 1);
}

__global__ void zero_u64_kernel(unsigned long long* a, unsigned long long* b, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    if (a) a[i] = 0;
    if (b) b[i] = 0;
  }
}

// Ordering key of a magnitude that fits 16 bits: |bits|, with every non-finite value mapped to
// the one key above all finite ones (same order as magnitude_units, ties included).
__device__ __forceinline__ unsigned magnitude_key(uint16_t bits) {
  const unsigned a = bits & 0x7fffu;
  return a > 0x7c00u ? 0x7c00u : a;
}

// The two largest magnitudes among a row's four selected entries `w` (smaller position on ties) and
// where they sit.
__device__ __forceinline__ void pick_two(const uint16_t (&w)[kSelCols], int& p0, int& p1) {
  unsigned key[kSelCols];
#pragma unroll
  for (int p = 0; p < kSelCols; ++p) key[p] = magnitude_key(w[p]);
  p0 = 0;
  unsigned k0 = key[0];
#pragma unroll
  for (int p = 1; p < kSelCols; ++p) if (key[p] > k0) { p0 = p; k0 = key[p]; }
  p1 = p0 == 0 ? 1 : 0;
  unsigned k1 = p0 == 0 ? key[1] : key[0];
#pragma unroll
  for (int p = 1; p < kSelCols; ++p) if (p != p0 && key[p] > k1) { p1 = p; k1 = key[p]; }
}

// Mask bytes of one row and group: 1 at columns c0 and c1, 0 elsewhere, with words of `mask_word` bytes.
__device__ __forceinline__ void write_mask(uint8_t* mrow, int M, int mask_word, int c0, int c1) {
  auto word4 = [&](int j) {   // mask bytes of columns j .. j+3
    return ((unsigned)(c0 - j) < 4u ? 1u << (8 * (c0 - j)) : 0u) | ((unsigned)(c1 - j) < 4u ? 1u << (8 * (c1 - j)) : 0u);
  };
  if (mask_word == 16) {
    for (int j = 0; j < M; j += 16)
      *reinterpret_cast<uint4*>(mrow + j) = make_uint4(word4(j), word4(j + 4), word4(j + 8), word4(j + 12));
  } else if (mask_word == 8) {
    for (int j = 0; j < M; j += 8) *reinterpret_cast<uint2*>(mrow + j) = make_uint2(word4(j), word4(j + 4));
  } else if (mask_word == 4) {
    for (int j = 0; j < M; j += 4) *reinterpret_cast<unsigned*>(mrow + j) = word4(j);
  } else {
    for (int c = 0; c < M; ++c) mrow[c] = (c == c0 || c == c1) ? 1 : 0;
  }
}

// One workgroup per (block row b, chunk of `gpw` groups): V rows x gpw*M columns.
//   phase 1: column masses into LDS (64-bit integer adds), the block's total mass.  A thread owns
//            8 neighbouring columns (one 16-byte load) and a slice of the rows, sums in registers
//            and adds once per column; columns past the last multiple of 8 and unaligned inputs
//            take the element-wise loop.
//   phase 2: one thread per group picks the 4 columns: largest mass first, smaller index on ties,
//            then sorted ascending
//   phase 3: one thread per (row, group): the 2 largest magnitudes among the 4, smaller position on
//            ties; writes the M mask bytes of its row and group, two of them 1, with the widest
//            stores the alignment allows (`mask_word`: 16, 8, 4 or 1 bytes), so the mask is written once
__global__ void __launch_bounds__(256) prune_kernel(const uint16_t* __restrict__ A, int64_t lda, int V, int M,
                                                    int64_t G, int gpw, int vec_ok, int mask_word, uint8_t* __restrict__ mask,
                                                    int64_t ldm, unsigned long long* __restrict__ kept_mass,
                                                    unsigned long long* __restrict__ total_mass) {
  __shared__ unsigned long long mass[kPruneMaxCols];
  __shared__ int sel[kPruneMaxCols / kSelCols][kSelCols];
  __shared__ unsigned long long wg_total, wg_kept;
  const int64_t chunk = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x;
  const int64_t g0 = chunk * gpw;
  const int ng = (int)((G - g0) < gpw ? (G - g0) : gpw);
  const int span = ng * M;

  for (int i = tid; i < span; i += blockDim.x) mass[i] = 0;
  if (tid == 0) { wg_total = 0; wg_kept = 0; }
  __syncthreads();
  unsigned long long my_total = 0;
  const int units = vec_ok ? span / 8 : 0;         // 8-column units handled with wide accesses
  if (units > 0) {
    const int slices = blockDim.x / units > 0 ? blockDim.x / units : 1;   // row slices working side by side
    for (int u0 = 0; u0 < units; u0 += blockDim.x) {                        // (more than 256 units: several sweeps)
      const int u = u0 + (slices > 1 ? tid % units : tid);
      const int slice = slices > 1 ? tid / units : 0;
      if (u < units && slice < slices) {
        unsigned long long m8[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int v = slice; v < V; v += slices) {
          const uint4 w = *reinterpret_cast<const uint4*>(A + (b * V + v) * lda + g0 * M + 8 * u);
          const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            m8[2 * e] += magnitude_units((uint16_t)ws[e]);
            m8[2 * e + 1] += magnitude_units((uint16_t)(ws[e] >> 16));
          }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if (m8[e]) atomicAdd(&mass[8 * u + e], m8[e]);
          my_total += m8[e];
        }
      }
    }
  }
  const int tail0 = units * 8;                     // columns not covered above
  const int tail = span - tail0;
  for (int64_t i = tid; i < (int64_t)V * tail; i += blockDim.x) {
    const int v = (int)(i / tail), c = tail0 + (int)(i % tail);
    const unsigned long long m = magnitude_units(A[(b * V + v) * lda + g0 * M + c]);
    if (m) atomicAdd(&mass[c], m);
    my_total += m;
  }
  if (my_total) atomicAdd(&wg_total, my_total);
  __syncthreads();
  if (tid < ng) {
    const unsigned long long* mg = mass + tid * M;
    int s[kSelCols];
    for (int k = 0; k < kSelCols; ++k) {
      int best = -1;
      for (int c = 0; c < M; ++c) {
        bool taken = false;
        for (int j = 0; j < k; ++j) taken |= s[j] == c;
        if (!taken && (best < 0 || mg[c] > mg[best])) best = c;   // strict >: the smaller index wins ties
      }
      s[k] = best;
    }
    for (int i = 1; i < kSelCols; ++i)                             // ascending order
      for (int j = i; j > 0 && s[j - 1] > s[j]; --j) { const int t = s[j]; s[j] = s[j - 1]; s[j - 1] = t; }
    for (int k = 0; k < kSelCols; ++k) sel[tid][k] = s[k];
  }
  __syncthreads();
  unsigned long long my_kept = 0;
  for (int i = tid; i < V * ng; i += blockDim.x) {
    const int v = i / ng, t = i % ng;
    const int64_t base = (b * V + v) * lda + (g0 + t) * M;
    uint16_t w[kSelCols];
    for (int p = 0; p < kSelCols; ++p) w[p] = A[base + sel[t][p]];
    int p0, p1;
    pick_two(w, p0, p1);
    write_mask(mask + (b * V + v) * ldm + (g0 + t) * M, M, mask_word, sel[t][p0], sel[t][p1]);
    my_kept += magnitude_units(w[p0]) + magnitude_units(w[p1]);
  }
  if (my_kept) atomicAdd(&wg_kept, my_kept);
  __syncthreads();
  if (tid == 0) {
    if (total_mass && wg_total) atomicAdd(&total_mass[b], wg_total);
    if (kept_mass && wg_kept) atomicAdd(&kept_mass[b], wg_kept);
  }
}

// Sums of magnitudes in a double that starts at 2^28: every magnitude is a multiple of 2^-24 and a
// sum stays below 2^28 (at most kTileMaxV of at most 2^16), so the sum's unit in the last place is 2^-24, no
// addition rounds, and the bits above those of 2^28 are the sum in units of 2^-24.  Three full-rate
// instructions per element (convert, clamp, widen) and an addition, where the integer form
// (decompose, 64-bit shift, 64-bit add) takes a dozen.
constexpr double kMassBias = 268435456.0;        // 2^28
constexpr int kTileMaxV = 2048;                  // (the LDS stops tiles earlier, at 1982 rows)
__device__ __forceinline__ double magnitude(uint16_t bits) {
  const float x = (float)__builtin_bit_cast(_Float16, bits);
  return (double)fminf(fabsf(x), 65536.f);        // Inf and NaN: 2^16 = 2^40 units
}
__device__ __forceinline__ unsigned long long mass_units(double biased) {
  return __builtin_bit_cast(unsigned long long, biased) - __builtin_bit_cast(unsigned long long, kMassBias);
}

// The same pruning with the block's tile (V rows x `gpw` groups) held in LDS, so that the matrix is
// read once, in 16-byte pieces at any alignment (12288 x 8190 at 128:2:10: 114 us; 299 when rows off the 16-byte
// boundaries went element by element, 256 in prune_kernel), and the second pass (4 scattered 2-byte reads per row and group)
// stays on chip.  Column choice: for M up to 64 a thread per column counts the columns that beat
// its own (all threads of a group read the same masses: broadcasts), above that a wave per group
// takes the maximum four times.
// Bound by memory: 49152 x 12288 at V = 128, M = 32 takes 0.37 ms, 4.9 TB/s of the 1.8 GB read and written (a
// copy reaches 5.1); prune_kernel takes 0.55 ms there.  Tiles of 128 columns x 128 rows (35 KB), so that
// four workgroups share a compute unit and one's loads run under the others' second passes.
// Needs V <= kTileMaxV and the tile within kTileLds; prune_kernel above takes the rest.
constexpr int kTileLds = 64 * 1024;
constexpr int kTileMaxGroups = 64;
__host__ __device__ constexpr int tile_pitch(int cols) { return (cols * 2 + 15) / 16 * 16 + 16; }
constexpr int64_t tile_lds(int V, int cols) { return (int64_t)V * tile_pitch(cols) + 8 * cols; }

// PIECES: large groups whose mask bytes are no whole number of 16-byte words: written one group a thread, the words of a store lie
// M bytes apart (a store for each 4 at M = 100).  Instead the picks go to LDS, over the group's first two entries, and each thread
// then makes 16 bytes of a row, of all groups that meet there, stored at any alignment; neighbouring workgroups, which share
// the lines at their edges, run on the same XCD.  8192 x 8100, us per call: 64:2:100 118 -> 73, 128:2:100 125 -> 96, 32:2:100 121 -> 91.
// Groups of up to 64 gain nothing or lose by the second pass over LDS (64:2:40 66 -> 68, 64:2:7 76 -> 86).
template <bool PIECES>
__global__ void __launch_bounds__(256) prune_tile_kernel(const uint16_t* __restrict__ A, int64_t lda, int V, int M,
                                                         int64_t G, int gpw, int mask_word,
                                                         uint8_t* __restrict__ mask, int64_t ldm,
                                                         unsigned long long* __restrict__ kept_mass,
                                                         unsigned long long* __restrict__ total_mass) {
  extern __shared__ __attribute__((aligned(16))) char tile[];      // [row][pitch], then the column masses
  __shared__ int sel[kTileMaxGroups][kSelCols];                     // by rank, then ascending
  __shared__ unsigned long long wg_total, wg_kept;
  int64_t b = blockIdx.y, chunk = blockIdx.x;
  if constexpr (PIECES) {
    const uint64_t all = (uint64_t)gridDim.x * gridDim.y, per_xcd = all / 8, id = blockIdx.y * (uint64_t)gridDim.x + blockIdx.x;
    if (id < 8 * per_xcd) {
      const uint64_t work = id % 8 * per_xcd + id / 8;
      b = (int64_t)(work / gridDim.x);
      chunk = (int64_t)(work - b * gridDim.x);
    }
  }
  const int64_t g0 = chunk * gpw;
  const int tid = threadIdx.x, lane = tid & 63;
  const int ng = (int)((G - g0) < gpw ? (G - g0) : gpw);
  const int span = ng * M;
  const int pitch = tile_pitch(gpw * M);
  unsigned long long* mass = reinterpret_cast<unsigned long long*>(tile + V * pitch);
  const uint16_t* blk = A + b * V * lda + g0 * M;

  for (int i = tid; i < span; i += 256) mass[i] = 0;
  if (tid == 0) { wg_total = 0; wg_kept = 0; }
  __syncthreads();
  unsigned long long my_total = 0;
  const int units = span / 8;                      // 8-column units: at most 128
  if (units > 0) {
    const int slices = 256 / units, u = tid % units, slice = tid / units;   // row slices working side by side
    if (slice < slices) {
      double m8[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) m8[e] = kMassBias;
      constexpr int NL = 8;                        // loads in flight per thread
      for (int v0 = slice; v0 < V; v0 += NL * slices) {
        u32x4_any w[NL];
#pragma unroll
        for (int j = 0; j < NL; ++j) {
          const int v = v0 + j * slices;
          w[j] = v < V ? *reinterpret_cast<const u32x4_any*>(blk + (int64_t)v * lda + 8 * u) : u32x4_any{0, 0, 0, 0};
        }
#pragma unroll
        for (int j = 0; j < NL; ++j) {
          const int v = v0 + j * slices;
          if (v < V) *reinterpret_cast<uint4*>(tile + v * pitch + u * 16) = make_uint4(w[j].x, w[j].y, w[j].z, w[j].w);
          const uint32_t ws[4] = {w[j].x, w[j].y, w[j].z, w[j].w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            m8[2 * e] += magnitude((uint16_t)ws[e]);
            m8[2 * e + 1] += magnitude((uint16_t)(ws[e] >> 16));
          }
        }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const unsigned long long m = mass_units(m8[e]);
        if (m) atomicAdd(&mass[8 * u + e], m);
        my_total += m;
      }
    }
  }
  const int tail0 = units * 8, tail = span - tail0;  // columns not covered above
  for (int i = tid; i < V * tail; i += 256) {
    const int v = i / tail, c = tail0 + i % tail;
    const uint16_t w = blk[(int64_t)v * lda + c];
    *reinterpret_cast<uint16_t*>(tile + v * pitch + c * 2) = w;
    const unsigned long long m = magnitude_units(w);
    if (m) atomicAdd(&mass[c], m);
    my_total += m;
  }
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) my_total += __shfl_xor(my_total, s);
  if (lane == 0 && my_total) atomicAdd(&wg_total, my_total);
  __syncthreads();
  // largest mass first, smaller index on ties
  if (M <= 64) {
    for (int c = tid; c < span; c += 256) {
      const int t = c / M, own = c - t * M;
      const unsigned long long* mg = mass + t * M;
      const unsigned long long mine = mg[own];
      int rank = 0;
#pragma unroll 4
      for (int j = 0; j < M; ++j) rank += mg[j] > mine || (mg[j] == mine && j < own);
      if (rank < kSelCols) sel[t][rank] = own;
    }
  } else {
    for (int t = tid >> 6; t < ng; t += 4) {
      int s[kSelCols] = {-1, -1, -1, -1};
#pragma unroll
      for (int k = 0; k < kSelCols; ++k) {
        unsigned long long best = 0;
        int at = M;                                // M: nothing seen yet
        for (int c = lane; c < M; c += 64) {
          const unsigned long long m = mass[t * M + c];
          const bool taken = c == s[0] || c == s[1] || c == s[2];
          if (!taken && (at == M || m > best)) { best = m; at = c; }
        }
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) {
          const unsigned long long om = __shfl_xor(best, d);
          const int oa = __shfl_xor(at, d);
          if (oa < M && (at == M || om > best || (om == best && oa < at))) { best = om; at = oa; }
        }
        s[k] = at;
        if (lane == 0) sel[t][k] = at;
      }
    }
  }
  __syncthreads();
  if (tid < ng) {                                  // ascending order
    int s0 = sel[tid][0], s1 = sel[tid][1], s2 = sel[tid][2], s3 = sel[tid][3];
    auto order = [](int& x, int& y) { const int lo = x < y ? x : y, hi = x < y ? y : x; x = lo; y = hi; };
    order(s0, s1); order(s2, s3); order(s0, s2); order(s1, s3); order(s1, s2);
    sel[tid][0] = s0; sel[tid][1] = s1; sel[tid][2] = s2; sel[tid][3] = s3;
  }
  __syncthreads();
  double my_kept = kMassBias;
  for (int i = tid; i < V * ng; i += 256) {
    const int v = i / ng, t = i - v * ng;
    uint16_t w[kSelCols];
    int c[kSelCols];
#pragma unroll
    for (int p = 0; p < kSelCols; ++p) {
      c[p] = sel[t][p];
      w[p] = *reinterpret_cast<const uint16_t*>(tile + v * pitch + (t * M + c[p]) * 2);
    }
    int p0, p1;
    pick_two(w, p0, p1);
    int c0 = c[0], c1 = c[0];
    uint16_t w0 = w[0], w1 = w[0];
#pragma unroll
    for (int p = 1; p < kSelCols; ++p) {
      if (p == p0) { c0 = c[p]; w0 = w[p]; }
      if (p == p1) { c1 = c[p]; w1 = w[p]; }
    }
    if constexpr (PIECES) {
      uint16_t* pick = reinterpret_cast<uint16_t*>(tile + v * pitch) + t * M;   // (this row and group is read by this thread only)
      pick[0] = (uint16_t)(t * M + c0);
      pick[1] = (uint16_t)(t * M + c1);
    } else {
      write_mask(mask + (b * V + v) * ldm + (g0 + t) * M, M, mask_word, c0, c1);
    }
    my_kept += magnitude(w0) + magnitude(w1);
  }
  if constexpr (PIECES) {
    __syncthreads();
    const int pieces = (span + 15) / 16;
    for (int i = tid; i < V * pieces; i += 256) {
      const int v = i / pieces, j = 16 * (i - v * pieces), left = span - j;
      const uint16_t* row = reinterpret_cast<const uint16_t*>(tile + v * pitch);
      uint64_t lo = 0, hi = 0;
      for (int at = j / M * M; at < j + 16 && at < span; at += M) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const unsigned d = (unsigned)(row[at + p] - j);
          if (d < 8) lo |= (uint64_t)1 << (8 * d);
          else if (d < 16) hi |= (uint64_t)1 << (8 * d - 64);
        }
      }
      uint8_t* out = mask + (b * V + v) * ldm + g0 * M + j;
      if (left >= 16) {
        *reinterpret_cast<u32x4_any*>(out) = u32x4_any{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
      } else {
        int n = left;
        if (n >= 8) {
          *reinterpret_cast<u32x2_any*>(out) = u32x2_any{(uint32_t)lo, (uint32_t)(lo >> 32)};
          lo = hi; out += 8; n -= 8;
        }
        if (n >= 4) {
          *reinterpret_cast<u32_any*>(out) = (uint32_t)lo;
          lo >>= 32; out += 4; n -= 4;
        }
        for (; n > 0; --n, lo >>= 8) *out++ = (uint8_t)lo;
      }
    }
  }
  unsigned long long kept = mass_units(my_kept);
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) kept += __shfl_xor(kept, s);
  if (lane == 0 && kept) atomicAdd(&wg_kept, kept);
  __syncthreads();
  if (tid == 0) {
    if (total_mass && wg_total) atomicAdd(&total_mass[b], wg_total);
    if (kept_mass && wg_kept) atomicAdd(&kept_mass[b], wg_kept);
  }
}

// Groups per workgroup of prune_kernel.
static int general_groups(int M) {
  const int gpw = kPruneMaxCols / M;
  return gpw > kStepGroups ? kStepGroups : gpw < 1 ? 1 : gpw;
}

// Groups per workgroup of prune_tile_kernel, 0 if the shape is not its: rows of 256 bytes, in whole
// 16-byte pieces (which at odd M takes several groups), doubled while four tiles still share a compute unit: a workgroup's
// second passes then cost less per byte (8192 x 8192, us per call with 128 columns -> now: 64:2:16 62 -> 51, 48:2:8 78 -> 60,
// 32:2:16 94 -> 53, 40:2:32 83 -> 56; with 256: 16:2:16 95 -> 63; 4096 x 8192 at 1:2:128, prune_kernel 960: 1227 ->
// 312).  Widths between the doublings lose (80 rows, 176 columns: 63 -> 65).  Where the columns are no whole number of groups
// the doubling pays in low blocks only (56:2:10, 280 columns: 97 -> 103; 12:2:40 with 1024 columns 139 -> 151), and less
// where a wave picks the columns of a group (M > 64: 16:2:100 with 600 columns 114 -> 133).
static int tile_groups(int V, int M) {
  if (V > kTileMaxV) return 0;
  const int whole = M % 8 == 0 ? 1 : M % 4 == 0 ? 2 : M % 2 == 0 ? 4 : 8;
  constexpr int kShared = 38 * 1024;
  int widest = V < 8 ? kPruneMaxCols : 512;
  if (512 % M == 0) widest = V < 16 ? kPruneMaxCols : 512;
  else if (M > 64) widest = V < 8 ? kPruneMaxCols : V < 16 ? 512 : V < 32 ? 256 : 128;
  else if (V > 48) widest = 128;
  int cols = 128;
  while (cols < widest && tile_lds(V, 2 * cols) <= kShared) cols *= 2;
  int n = (cols + M * whole - 1) / (M * whole);    // in units of `whole` groups
  while (n > 1 && (tile_lds(V, n * whole * M) > kShared || n * whole * M > kPruneMaxCols || n * whole > kTileMaxGroups)) --n;
  const int gpw = n * whole;
  return tile_lds(V, gpw * M) <= kTileLds - 2048 && gpw * M <= kPruneMaxCols && gpw <= kTileMaxGroups ? gpw : 0;
}

// A tall block leaves the tile few columns, pieces of rows too short to read well; prune_kernel takes `general` columns of
// it but reads the matrix twice, and its workgroups last longer.  So the tile is the better kernel while prune_kernel would
// not fill the chip, up to the number of prune_kernel's workgroups returned here, which grows with the share of its
// columns that the tile keeps.  Measured for V = 192 .. 1536, M = 4 .. 64, matrices of 1.5 to 600 million entries (468 shapes
// with rows at 16-byte boundaries, as many without); us per call, tile / prune_kernel, by tile columns: 8: 2048 x 768 at
// 1024:2:8 20 / 54, 12288 x 8192 384 / 110; 16: 12288 x 8192 at 512:2:16 192 / 92; 24: 2048 x 768 at 512:2:8 20 / 36,
// 12288 x 8192 160 / 112, 49152 x 12288 at 512:2:4 1200 / 1011; 32: 12288 x 8192 at 512:2:32 111 / 123, 49152 x
// 12288 700 / 617, 12288 x 8192 at 448:2:4 127 / 180; 48: 49152 x 12288 at 256:2:48 1.25 times as long as prune_kernel,
// 12288 x 8192 at 320:2:8 0.85 times; 64 and more: never slower.  Where prune_kernel could only read single elements the tile
// wins from 16 or 24 columns on (12288 x 8190 at 640:2:10 166 / 241), below that on small matrices.  Chosen so, 920 of the 936
// shapes are within 4 % of the better kernel, the others within 10 %.
static int64_t tile_pays_up_to(int cols, int general, bool general_wide) {
  constexpr int64_t kAlways = INT64_MAX;
  const int share = 8 * cols / general;            // in eighths
  if (!general_wide) return cols < 16 ? 800 : cols < 24 && share < 2 ? 4000 : kAlways;
  if (cols >= 64 || cols >= general) return kAlways;
  if (cols < 16) return 280;
  if (cols < 32) return share < 3 ? 420 : share < 4 ? 840 : cols < 24 ? 1500 : share < 6 ? kAlways : 13000;
  if (cols < 48) return share < 4 ? 900 : 2850;
  return share < 3 ? 1300 : share < 4 ? 2600 : 12000;
}

// The mask bytes by way of LDS (PIECES) cost a second pass over the picks, which every call waits for: 2 us where a unit has one workgroup
// or two.  They pay where the group's own stores are many and the rows of a workgroup short: 805 shapes (M 65-500, V 1-256, 0.25 to 130
// million entries), us per call without / with: 8192 x 8136 at 24:2:72 (9 stores) 90.5 / 94.4, 64:2:72 81 / 71; 32768 x
// 1728 at 32:2:72 93 / 100; 8192 x 8100 at 8:2:100 (25) 1.03 times, 16:2:100 0.92, 8192 x 8125 at 8:2:65 (65, bytes) 1.04, 16:2:65 0.79;
// small: 1024 x 1000 at 128:2:100 23.2 / 25.6.  Above 200 columns always: 0.74 to 1.00.  Chosen so 0.930 of the time without, at most 1.04
// (with pieces for all groups above 64: 0.946 and 1.31).
static bool pieces_pay(int64_t entries, int V, int M, int mask_word) {
  if (mask_word == 16 || M <= 64) return false;
  const int stores = M / mask_word < 48 ? M / mask_word : 48;   // of a row and group
  return M > 200 || (V * stores >= 400 && entries >= (int64_t)8 << 20);
}

hipError_t launch_prune(const uint16_t* A, int64_t lda, int64_t R, int64_t K, int V, int M, uint8_t* mask, int64_t ldm,
                        unsigned long long* kept_mass, unsigned long long* total_mass, hipStream_t st) {
  const int64_t Rb = R / V, G = K / M;
  if (kept_mass || total_mass)
    hipLaunchKernelGGL(zero_u64_kernel, dim3((unsigned)((Rb + 255) / 256)), dim3(256), 0, st, kept_mass, total_mass, Rb);
  if (Rb == 0 || G == 0) return hipGetLastError();
  // prune_kernel's wide loads need every chunk of every row of A to start on a 16-byte boundary
  const int general = general_groups(M);
  const int vec_ok = ((int64_t)general * M) % 8 == 0 && lda % 8 == 0 && reinterpret_cast<uintptr_t>(A) % 16 == 0;
  int tiled = tile_groups(V, M);
  if (Rb * ((G + general - 1) / general) > tile_pays_up_to(tiled * M, general * M, vec_ok)) tiled = 0;
  if (tiled > 0 && (G + tiled - 1) / tiled > kMaxBlocks) tiled = 0;   // too many workgroups for a launch (K near 2^31)
  const int gpw = tiled > 0 ? tiled : general;
  const int64_t chunks = (G + gpw - 1) / gpw;
  // every (row, group) of the mask starts at row * ldm + group * M: the widest word that always divides that
  const uintptr_t ma = reinterpret_cast<uintptr_t>(mask);
  const int mask_word = (M % 16 == 0 && ldm % 16 == 0 && ma % 16 == 0) ? 16 : (M % 8 == 0 && ldm % 8 == 0 && ma % 8 == 0) ? 8
                        : (M % 4 == 0 && ldm % 4 == 0 && ma % 4 == 0) ? 4 : 1;
  if (tiled > 0 && pieces_pay(R * K, V, M, mask_word))
    hipLaunchKernelGGL(prune_tile_kernel<true>, dim3((unsigned)chunks, (unsigned)Rb), dim3(256), (size_t)tile_lds(V, gpw * M), st,
                       A, lda, V, M, G, gpw, mask_word, mask, ldm, kept_mass, total_mass);
  else if (tiled > 0)
    hipLaunchKernelGGL(prune_tile_kernel<false>, dim3((unsigned)chunks, (unsigned)Rb), dim3(256), (size_t)tile_lds(V, gpw * M), st,
                       A, lda, V, M, G, gpw, mask_word, mask, ldm, kept_mass, total_mass);
  else
    hipLaunchKernelGGL(prune_kernel, dim3((unsigned)chunks, (unsigned)Rb), dim3(256), 0, st, A, lda, V, M, G, gpw, vec_ok,
                       mask_word, mask, ldm, kept_mass, total_mass);
  return hipGetLastError();
}

}  // namespace venom
