// Format kernels: dense + mask -> canonical V:N:M arrays (section 3 of the paper), canonical ->
// the product kernel's packed copies, and packed -> dense (the format read backwards).
// Pure data movement: fp16 payloads are handled as 16-bit patterns and never interpreted.
#include <type_traits>

#include "venom_internal.h"

namespace venom {

Layout make_layout(int64_t R, int64_t K, int V, int M) {
  Layout L{};
  L.R = R; L.K = K; L.G = K / M; L.Rb = R / V;
  L.W = (L.G + 7) / 8;
  L.steps = (L.G + kStepGroups - 1) / kStepGroups;
  int Vp = V;                                       // block height of the packed copy
  if (M == kSelCols && R % (kMaxTiles * kTileRows) == 0) Vp = kMaxTiles * kTileRows;
  L.packed = (Vp % kTileRows) == 0 && Vp / kTileRows <= kMaxTiles;
  L.vt = L.packed ? Vp / kTileRows : 0;
  L.Rbp = L.packed ? R / Vp : 0;
  L.rec_bytes = (int64_t)L.vt * kTileValBytes + kTailBytes;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
  L.off_values = take((size_t)R * L.G * 2 * sizeof(uint16_t));
  L.off_columns = take((size_t)L.Rb * L.G * kSelCols * sizeof(uint16_t));
  L.off_meta = take((size_t)R * L.W * sizeof(uint32_t));
  if (L.packed) {
    L.off_arec = take((size_t)L.Rbp * L.steps * L.rec_bytes);
    L.off_rowidx = take((size_t)L.Rbp * L.steps * kStepRows * sizeof(int32_t));
  }
  L.off_status = take(8);
  L.total = off;
  return L;
}

// ---------------------------------------------------------------------------------------------
// Legality word: the smallest key wins, so the first offending block in row-major order is
// reported, the column rule before the row rule inside one block, and the first row for the
// row rule.  key = (block_linear << 24) | (kind << 23) | row_in_block; the word holds ~key, 0 if there is none.
// With a slot the word is one of the library's own, which is 0 between calls, and `found` is a word of host memory that the host
// has cleared and the first violation sets: a legal call then needs neither a kernel that clears the word nor a
// copy that fetches it, and only after a violation take_violation_kernel does both.
// us per call of the binding, without -> with it: venom_import of 512 x 1024 at 64:2:8 27.4 -> 23.3, of 8192 x 8192
// 51 -> 47; venom_compress of 4096 x 1024 at 128:2:16 35 -> 31.
// Without one (slot < 0) it is the workspace's.  A wave reports one violation, and none after the one that is known; the host
// is told once, by the wave that finds the word empty.  8192 x 8192 at 64:2:8, us per call with every group wrong, against a
// store to the host by each thread that finds a violation and a second run for its place: compression 602 -> 122,
// import 3804 -> 98; with one group wrong 163 -> 94 and 47 -> 59.
static __device__ unsigned long long violations[kLegalitySlots];

struct Legality {
  int slot;
  unsigned long long *found, *own;               // own: the workspace's word, used without a slot
};

__global__ void init_status_kernel(unsigned long long* status) { *status = 0; }

__global__ void take_violation_kernel(int slot, unsigned long long* to) {
  *reinterpret_cast<volatile unsigned long long*>(to) = violations[slot];
  violations[slot] = 0;
}

__device__ __forceinline__ void report(const Legality& l, unsigned long long key) {
  unsigned long long* word = l.slot >= 0 ? &violations[l.slot] : l.own;
  if (__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= ~key) return;
  if (atomicMax(word, ~key) == 0 && l.slot >= 0) *reinterpret_cast<volatile unsigned long long*>(l.found) = 1;
}

// ---------------------------------------------------------------------------------------------
// Where one (row, group) entry goes: the canonical arrays and, if the product kernel serves this
// shape, its packed copies.  A packed record of one (block row, k-step):
//   [V/32 tiles x 1024 B of values][512 B tail]
// values of a tile: 64 lanes x 8 halfs; lane = 32*h + i holds row 32*tile + i and the two kept
// values of groups 8*step + 4*h .. +3 -- the A operand of v_smfmac_f32_32x32x32_f16.
// tail: 64 lanes x 4 x uint16, entry [lane][tile] = the lane's four canonical nibbles for that tile
//       (a lane reads its 8 bytes with one LDS load; the matrix instruction picks the 16-bit field
//       with its ABID operand); the entries of tiles that do not exist are zero.
// rowidx: absolute row of B of every gathered row, [block row][k-step][32], entry 4*t + p of a step
// is (8*step + t)*M + column_loc[p]; groups past the end point at row 0 (their values are zero).
// The block height Vp of the packed copy differs from V only at M = 4, where all canonical block
// rows hold the same column ids.
struct FormatDst {
  uint32_t* values;
  uint16_t* columns;
  uint32_t* meta;
  char* arec;              // null: no packed copies
  int32_t* rowidx;
  int64_t G, W;            // groups per row, metadata words per row = k-steps
  int V, Vp, vt, M;
};

// Row `v` of canonical block row `cb` in the packed copy: its block row and the row inside it.
__device__ __forceinline__ void packed_row(const FormatDst& d, int64_t cb, int v, int64_t& rb, int& rr) {
  if (d.Vp == d.V) { rb = cb; rr = v; return; }
  const int64_t r = cb * d.V + v;                // M = 4: blocks of 128 rows
  rb = r / (kMaxTiles * kTileRows);
  rr = (int)(r % (kMaxTiles * kTileRows));
}

// Column ids of group g of block row cb, and the rows of B of group t of k-step w of packed block row rb.
__device__ __forceinline__ void emit_columns(const FormatDst& d, int64_t cb, int64_t g, ushort4 c) {
  *reinterpret_cast<ushort4*>(d.columns + (cb * d.G + g) * kSelCols) = c;
}
__device__ __forceinline__ void emit_rowidx(const FormatDst& d, int64_t rb, int64_t w, int t, ushort4 c) {
  const int64_t g = w * 8 + t;
  const int k0 = (int)(g * d.M);
  *reinterpret_cast<int4*>(d.rowidx + (rb * d.W + w) * kStepRows + 4 * t) =
      g < d.G ? make_int4(k0 + c.x, k0 + c.y, k0 + c.z, k0 + c.w) : make_int4(0, 0, 0, 0);
}
// The index word of row rr in the record `rec`: half h of the row's metadata word, one 2-byte store (a row
// of the first tile clears the fields of the tiles that do not exist).
__device__ __forceinline__ void emit_index_field(const FormatDst& d, char* rec, int rr, int h, uint32_t word) {
  const int tile = rr / kTileRows, i = rr % kTileRows;
  uint16_t* tail = reinterpret_cast<uint16_t*>(rec + d.vt * kTileValBytes) + (32 * h + i) * kMaxTiles;
  tail[tile] = (uint16_t)(word >> (16 * h));
  if (tile == 0)
    for (int e = d.vt; e < kMaxTiles; ++e) tail[e] = 0;
}
// The same for a whole lane 32*h + i at once, from the words of rows i, i+32, ...: one 8-byte store, where those
// words are at hand, in LDS.
__device__ __forceinline__ void emit_index(const FormatDst& d, char* rec, int i, int h, const uint32_t (&word)[kMaxTiles]) {
  uint32_t o[2] = {0, 0};
#pragma unroll
  for (int e = 0; e < kMaxTiles; ++e) o[e / 2] |= ((word[e] >> (16 * h)) & 0xffffu) << (16 * (e % 2));
  *reinterpret_cast<uint2*>(rec + d.vt * kTileValBytes + (32 * h + i) * 8) = make_uint2(o[0], o[1]);
}

// x of eight neighbouring lanes (0-7, 8-15, ...), combined; all lanes of the wave take part.
__device__ __forceinline__ uint32_t or_of_eight_lanes(uint32_t x) {
  x |= __builtin_amdgcn_mov_dpp(x, 0xb1, 0xf, 0xf, true);        // quads: 1 0 3 2
  x |= __builtin_amdgcn_mov_dpp(x, 0x4e, 0xf, 0xf, true);        // 2 3 0 1
  x |= __builtin_amdgcn_mov_dpp(x, 0x141, 0xf, 0xf, true);       // the mirrored half row: lane 7 - l
  return x;
}

// The non-zero bytes of a word as four bits.
__device__ __forceinline__ uint32_t nonzero_bits(uint32_t x) {
  const uint32_t top = (((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x) & 0x80808080u;   // bit 7 of every non-zero byte
  return ((top >> 7) * 0x10204080u) >> 28;       // byte e's flag to bit e
}

constexpr int kMaxM = 1024;
constexpr int kCompressWords = 4;                // most metadata words (8 groups each) one workgroup takes
constexpr int kCompressBits = 48 * 1024;         // most LDS for the mask bits of a workgroup's rows

// bytes per row of mask bits in LDS, with a word of padding
__host__ __device__ constexpr int bits_pitch(int wpw, int M) { return (wpw * M + 3) / 4 * 4 + 4; }

// Dense + mask -> canonical arrays and packed copies.  One workgroup per (block row b, `wpw` metadata
// words) = V rows x 8*wpw groups x M columns.
//   phase 1: the mask is read once, UB bytes at a time (16 or 8, at any alignment), and kept in LDS as one bit
//            per column and row; the bits of all rows together say which columns the block uses
//   phase 2: one thread per group picks the 4 columns: the used ones ascending, padded with the
//            smallest unused ids, sorted
//   phase 3: one thread per (row, group): positions kept inside the 4 selected columns, padded with
//            the smallest unused positions, sorted -> nibble; values copied as bits; canonical and
//            packed entries written together.  A thread keeps its group, so that only what depends on the row is
//            left in the loop, and the nibble comes from a table of the 16 sets of kept positions.
// NE: rows of phase 3 in flight per thread (the rule: launch_compress).  Bound by memory from M = 32 on: 49152 x 12288 (0.6 GB
// of mask, 1.2 GB of A -- the two kept values of 32 touch every 64-byte sector -- and 0.17 GB written) takes 0.39 ms, 5.0 TB/s; it was 0.40 ms with four rows in
// flight, 0.45 ms, and another 0.08 ms to pack in a second pass, when phase 3 fetched the mask bytes again one by one.  For
// smaller groups there are more entries than bytes to wait for, and eight rows in flight cost occupancy: 8192 x 8192 at 64:2:8,
// us per call with 2 / 4 / 8 rows 80.6 / 84.5 / 87.1.  Against an index computation for each entry: 128:2:4 135 -> 115, 64:2:8 83 -> 75,
// 64:2:16 71 -> 67, 128:2:40 68 -> 64.
// by_full, by_last: n / units = n * by >> 16 for n, units <= 256, for the loads of a row in all chunks of columns but the
// last, and in the last (a division in the kernel is 5 % of a workgroup with one row).
// bits_ok: the bits of V rows fit (48 KB of LDS: 49152 x 12288 at 1024:2:32 takes 464 us a call, more if phase 3 reads the
// mask again); otherwise (very tall blocks) it does.
// The block rows are taken from the last to the first: what wrote the mask (and read the matrix) went the other way, and
// left the ends of both in the memory-side cache.  ONCE (phase 1 is the mask's only reader, bits_ok): its loads
// are streamed, so that they leave that room to the matrix and the outputs.  us of venom_prune and
// venom_compress together, first to last and cached -> last to first -> streamed as well: 49152 x 12288 at 128:2:32 803 -> 784 ->
// 765, 12288 x 12288 at 256:2:8 278 -> 267 -> 263, 49152 x 2048 at 32:2:16 168 -> 158 -> 154, 16384 x 4096 at 128:2:16
// 116 -> 114 -> 113 (compression of one mask again and again, 66 instead of 65).
template <int UB, bool ONCE, int NE>
__global__ void __launch_bounds__(256) compress_kernel(const uint16_t* __restrict__ A, int64_t lda,
                                                       const uint8_t* __restrict__ mask, int64_t ldm, int wpw, int bits_ok,
                                                       unsigned by_full, unsigned by_last,
                                                       FormatDst d, Legality legality) {
  extern __shared__ __attribute__((aligned(16))) uint8_t bits[];   // [row][pitch]
  __shared__ uint32_t used[kCompressWords * 8 * kMaxM / 32 + 1];
  __shared__ ushort4 sel[kCompressWords * 8];
  __shared__ int cols_ok[kCompressWords * 8];
  __shared__ uint32_t words[kCompressWords][kMaxTiles * kTileRows];   // metadata words, if the packed copy has blocks of V rows
  const int V = d.V, M = d.M;
  const int64_t b = gridDim.y - 1 - blockIdx.y, w0 = (int64_t)blockIdx.x * wpw, g0 = w0 * 8;
  const int tid = threadIdx.x;
  const int nw = (int)((d.W - w0) < wpw ? (d.W - w0) : wpw);              // words of this workgroup that exist
  const int ng = (int)((d.G - g0) < 8 * nw ? (d.G - g0) : 8 * nw);        // groups that exist
  const int span = ng * M;
  const int pitch = bits_pitch(wpw, M);
  const uint8_t* mblk = mask + b * V * ldm + g0 * M;

  const int units = span / UB, tail0 = units * UB, tail = span - tail0;
  for (int i = tid; i < (span + 31) / 32 + 1; i += 256) used[i] = 0;
  if (bits_ok && tail > 0)                       // the columns of the byte loop are set bit by bit
    for (int i = tid; i < V * pitch / 4; i += 256) reinterpret_cast<uint32_t*>(bits)[i] = 0;
  __syncthreads();
  // row slices working side by side; no unit at all where a padded mask's last columns are fewer than a load takes
  const unsigned by_units = (int)blockIdx.x + 1 < (int)gridDim.x ? by_full : by_last;
  const int slices = units > 0 && units < 256 ? (int)(256 * by_units >> 16) : 1;
  for (int u0 = 0; u0 < units; u0 += 256) {                               // (more than 256 units: several sweeps)
    const int slice = slices > 1 ? (int)(tid * by_units >> 16) : 0;
    const int u = u0 + tid - slice * units;
    if (u < units && slice < slices) {
      uint32_t seen = 0;
      const uint8_t* p = mblk + UB * u;
      auto rows = [&](int v0, auto in_flight) {  // rows v0, v0 + slices, ..., their loads in flight together
        constexpr int NL = decltype(in_flight)::value;
        uint32_t x[NL][UB / 4];
#pragma unroll
        for (int j = 0; j < NL; ++j) {
          const int v = v0 + j * slices;
#pragma unroll
          for (int e = 0; e < UB / 4; ++e) x[j][e] = 0;
          if (v < V) {
            if constexpr (UB == 16) {
              const u32x4_any* src = reinterpret_cast<const u32x4_any*>(p + (int64_t)v * ldm);
              const u32x4_any q = ONCE ? __builtin_nontemporal_load(src) : *src;
              x[j][0] = q.x; x[j][1] = q.y; x[j][2] = q.z; x[j][3] = q.w;
            } else {
              const u32x2_any q = *reinterpret_cast<const u32x2_any*>(p + (int64_t)v * ldm);
              x[j][0] = q.x; x[j][1] = q.y;
            }
          }
        }
#pragma unroll
        for (int j = 0; j < NL; ++j) {
          const int v = v0 + j * slices;
          uint32_t m = 0;
#pragma unroll
          for (int e = 0; e < UB / 4; ++e) m |= nonzero_bits(x[j][e]) << (4 * e);
          seen |= m;
          if (bits_ok && v < V) {
            if constexpr (UB == 16) *reinterpret_cast<uint16_t*>(bits + v * pitch + 2 * u) = (uint16_t)m;
            else bits[v * pitch + u] = (uint8_t)m;
          }
        }
      };
      // short rows or few of them: one load each (1048576 x 32 at 128:2:8: 90 us a call with eight slots, 82 with one)
      if (V <= slices) rows(slice, std::integral_constant<int, 1>{});
      else
        for (int v0 = slice; v0 < V; v0 += 8 * slices) rows(v0, std::integral_constant<int, 8>{});
      if (seen) atomicOr(&used[u * UB / 32], seen << (u * UB % 32));
    }
  }
  for (int64_t i = tid; i < (int64_t)V * tail; i += 256) {
    const int v = (int)(i / tail), c = tail0 + (int)(i % tail);
    if (mblk[(int64_t)v * ldm + c]) {
      atomicOr(&used[c / 32], 1u << (c % 32));
      if (bits_ok) atomicOr(reinterpret_cast<uint32_t*>(bits + v * pitch + c / 32 * 4), 1u << (c % 32));
    }
  }
  __syncthreads();
  uint32_t first = ~0u;                          // key of this thread's first violation, groups counted from g0
  if (tid < ng) {
    int cnt = 0;
    int s[kSelCols] = {0, 0, 0, 0};
    auto bits32 = [&](int c) {                   // used flags of columns c .. c+31 of this group, zero past its end
      const int o = tid * M + c;
      const uint32_t x = (uint32_t)(((((unsigned long long)used[o / 32 + 1]) << 32) | used[o / 32]) >> (o % 32));
      return M - c >= 32 ? x : x & ((1u << (M - c)) - 1u);
    };
    for (int c = 0; c < M; c += 32) {
      uint32_t x = bits32(c);
      int n = cnt;
      cnt += __popc(x);
      for (; x != 0 && n < kSelCols; ++n, x &= x - 1) {
        const int id = c + __ffs(x) - 1;
#pragma unroll
        for (int p = 0; p < kSelCols; ++p) s[p] = p == n ? id : s[p];
      }
    }
    const bool ok = cnt <= kSelCols;
    if (!ok) first = (uint32_t)tid << 24;
    // pad with the smallest unused ids, keeping the list sorted
    for (int c = 0; cnt < kSelCols && c < M; ++c) {
      if ((bits32(c) & 1u) != 0) continue;
      int id = c;                                // bubble it into place
#pragma unroll
      for (int p = 0; p < kSelCols; ++p) {
        if (p < cnt && s[p] > id) { const int x = s[p]; s[p] = id; id = x; }
        else if (p == cnt) s[p] = id;
      }
      ++cnt;
    }
    cols_ok[tid] = ok;
    sel[tid] = make_ushort4((uint16_t)s[0], (uint16_t)s[1], (uint16_t)s[2], (uint16_t)s[3]);
  }
  __syncthreads();
  // one thread per (row, group): eight neighbouring lanes hold the eight nibbles of a metadata word and combine them with three
  // lane exchanges.  A thread keeps its group and goes from row to row, so all that depends on the group is done once.
  const int64_t rec_bytes = (int64_t)d.vt * kTileValBytes + kTailBytes;
  const int lanes = nw == 1 ? 3 : nw == 2 ? 4 : 5;                        // log2 of a row's lanes (of 32, three words leave eight idle)
  const int tg = tid & ((1 << lanes) - 1), dv = 256 >> lanes;
  const bool group_in = tg < ng, word_in = tg < 8 * nw;
  const ushort4 c4 = group_in ? sel[tg] : make_ushort4(0, 0, 0, 0);
  const uint64_t cols = (uint64_t)c4.x | (uint64_t)c4.y << 16 | (uint64_t)c4.z << 32 | (uint64_t)c4.w << 48;
  const bool legal_cols = group_in && cols_ok[tg];
  const int64_t w = w0 + (tg >> 3), g = g0 + tg;
  const int t = tg & 7, h = t >> 2;
  const uint16_t* acol = A + b * V * lda + g * M;
  uint32_t* vals = d.values + b * V * d.G + g;
  uint32_t* meta = d.meta + b * V * d.W + w;
  char* rec0 = d.arec == nullptr ? nullptr : d.arec + (b * d.W + w) * rec_bytes;   // (of this block, if the packed one is the same)
  const bool same_block = d.Vp == d.V;
  for (int base = 0; base < V; base += NE * dv) {
    uint32_t v01[NE], nib[NE];
#pragma unroll
    for (int j = 0; j < NE; ++j) {
      const int v = base + (tid >> lanes) + j * dv;
      nib[j] = 0; v01[j] = 0;
      if (v < V && group_in) {
        int kept = 0;                            // bit p: the row keeps selected column p
        if (bits_ok && M <= 32) {                // the group's bits in one word
          const uint32_t* row = reinterpret_cast<const uint32_t*>(bits + v * pitch) + tg * M / 32;
          const uint32_t x = (uint32_t)((((uint64_t)row[1] << 32) | row[0]) >> (tg * M % 32));
          kept = (x >> c4.x & 1) | (x >> c4.y & 1) << 1 | (x >> c4.z & 1) << 2 | (x >> c4.w & 1) << 3;
        } else if (bits_ok) {
#pragma unroll
          for (int p = 0; p < kSelCols; ++p) {
            const int col = tg * M + (int)(cols >> (16 * p) & 0xffff);
            kept |= ((bits[v * pitch + col / 8] >> (col % 8)) & 1) << p;
          }
        } else {                                 // four loads in flight (one after the other: 1351 instead of 1029 us
          const uint8_t* mrow = mblk + (int64_t)v * ldm + tg * M;   // for 49152 x 12288 at 8192:2:8)
          const uint8_t m0 = mrow[c4.x], m1 = mrow[c4.y], m2 = mrow[c4.z], m3 = mrow[c4.w];
          kept = (m0 != 0) | (m1 != 0) << 1 | (m2 != 0) << 2 | (m3 != 0) << 3;
        }
        if (legal_cols && __popc(kept) > 2) {
          const uint32_t key = (uint32_t)tg << 24 | 1u << 23 | (uint32_t)v;
          first = first < key ? first : key;
        }
        // the nibble p0 | p1 << 2: the first two kept positions, padded with the smallest unused ones, sorted; of `kept` = 0 .. 15
        constexpr uint64_t kNibbles = 0x498e4dcc49884444ull;
        const uint32_t n = (uint32_t)(kNibbles >> (4 * kept)) & 15u, p0 = n & 3u, p1 = n >> 2;
        const uint16_t* arow = acol + (int64_t)v * lda;
        const uint32_t a0 = kept >> p0 & 1 ? arow[cols >> (16 * p0) & 0xffff] : 0u;
        const uint32_t a1 = kept >> p1 & 1 ? arow[cols >> (16 * p1) & 0xffff] : 0u;
        v01[j] = a0 | (a1 << 16);
        nib[j] = n << (4 * t);
      }
    }
#pragma unroll
    for (int j = 0; j < NE; ++j) {
      const int v = base + (tid >> lanes) + j * dv;
      const uint32_t word = or_of_eight_lanes(nib[j]);
      if (v < V && word_in) {
        if (group_in) vals[v * d.G] = v01[j];
        if (t == 0) meta[v * d.W] = word;
        if (v == 0 && group_in) emit_columns(d, b, g, c4);
        if (d.arec != nullptr) {
          int64_t rb = b;
          int rr = v;
          char* rec = rec0;
          if (!same_block) {
            packed_row(d, b, v, rb, rr);
            rec = d.arec + (rb * d.W + w) * rec_bytes;
          }
          *reinterpret_cast<uint32_t*>(rec + (rr / kTileRows) * kTileValBytes + (32 * h + rr % kTileRows) * 16 + (t & 3) * 4) = v01[j];
          if (t == 0 && same_block) words[tg >> 3][v] = word;
          else if ((t & 3) == 0 && !same_block) emit_index_field(d, rec, rr, h, word);   // (the packed block's other rows are elsewhere)
          if (rr == 0) emit_rowidx(d, rb, w, t, c4);
        }
      }
    }
  }
  if (__ballot(first != ~0u) != 0) {
    for (int m = 1; m < 64; m *= 2) {
      const uint32_t other = __shfl_xor(first, m);
      first = first < other ? first : other;
    }
    if (tid % 64 == 0) report(legality, ((unsigned long long)(b * d.G + g0) << 24) + first);
  }
  if (d.arec == nullptr || d.Vp != d.V) return;
  __syncthreads();
  for (int i = tid; i < nw * 64; i += 256) {
    const int k = i / 64, l = i % 64;
    uint32_t word[kMaxTiles];
#pragma unroll
    for (int e = 0; e < kMaxTiles; ++e) word[e] = e < d.vt ? words[k][32 * e + l % 32] : 0u;
    emit_index(d, d.arec + (b * d.W + w0 + k) * rec_bytes, l % 32, l / 32, word);
  }
}

// Canonical arrays from outside -> the workspace: checked, copied and packed in one pass (the handle
// is only handed out if the check found nothing).  One thread per row and half metadata word = 4 groups: 16 bytes
// of values, one 16-byte slot of the packed record.  TILES: 32-row tiles of a packed block row; a workgroup takes 4 words of all
// of them, the loads of all rows in flight together: it reads rows of 128 bytes and completes the 128-byte lines of the
// records, their index words by way of LDS (two bytes a row and tile: workgroups of one tile each wrote parts of the same lines
// from several XCDs).  SPLIT: a workgroup takes one tile after all (the rule: launch_import).  TILES = 0, no packed records:
// 2^wbits words of 128 >> wbits rows, 32 of 4 where there are as many; a row that starts inside a line then shares far fewer lines
// with workgroups of other XCDs (4096 x 8190 at 1:2:7, us per call: 81 with 4 words, 60 with 32, three copies and a check 72).
// Checked is what the gather and the matrix instruction rely on -- column ids strictly increasing
// and below M (once per block), the two m-indices of a nibble ordered idx0 < idx1, unused nibbles of
// the last metadata word zero.
// 8192 x 8192, us per call of the binding (20 of them the launch and the wait), the same arrays again, one tile a workgroup ->
// all: 64:2:8 (120 MB in and out) 48.2 -> 46.0, 128:2:8 47.1 -> 44.7, 64:2:16 37.0 -> 34.0, 64:2:7 63.2 -> 59.4; three copies, the check and the packing by themselves
// took 90 us at 64:2:8.
template <int TILES, bool SPLIT>
__global__ void __launch_bounds__(256) import_kernel(const u32_any* __restrict__ values, const u16_any* __restrict__ columns,
                                                     const u32_any* __restrict__ meta, int64_t R, int wbits, FormatDst d,
                                                     Legality legality) {
  constexpr bool PACKED = TILES > 0, GATHER = PACKED && !SPLIT;   // GATHER: the index words go through LDS
  constexpr int NT = PACKED ? TILES : 1;
  __shared__ uint32_t words[GATHER ? 4 : 1][NT * kTileRows];
  if constexpr (PACKED) wbits = 2;
  const int64_t wq = (d.W + (1 << wbits) - 1) >> wbits;
  const int rows = PACKED ? NT * kTileRows : 128 >> wbits;   // of the workgroup
  const int64_t rblk = blockIdx.x / wq, wblk = blockIdx.x - rblk * wq;
  const int64_t rb = SPLIT ? rblk / d.vt : rblk;   // packed block row
  const int t0 = SPLIT ? (int)(rblk - rb * d.vt) : 0;
  const int u = threadIdx.x & ((2 << wbits) - 1), h = u & 1, i = threadIdx.x >> (wbits + 1);
  const int64_t w = (wblk << wbits) + (u >> 1), r0 = rblk * rows + i;
  const bool in = w < d.W && r0 < R;               // (R is a multiple of a packed block's rows)
  const int64_t g = w * 8 + 4 * h;
  const int ng = !in || g >= d.G ? 0 : d.G - g < 4 ? (int)(d.G - g) : 4;  // groups of the half word that exist
  uint32_t word[NT], x[NT][4];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int64_t r = r0 + t * kTileRows;
    word[t] = in ? (uint32_t)meta[r * d.W + w] : 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e) x[t][e] = 0;
    const u32_any* src = values + r * d.G + g;
    if (ng == 4) {                                 // wide also where G is no multiple of 4 (rows start at any word)
      const u32x4_any q = *reinterpret_cast<const u32x4_any*>(src);
      x[t][0] = q.x; x[t][1] = q.y; x[t][2] = q.z; x[t][3] = q.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < ng) x[t][e] = src[e];
    }
  }
  bool bad = false;
  const int64_t cb0 = rblk * rows / d.V;           // canonical block row of the workgroup's first row: a scalar division
  const int first = (int)(rblk * rows - cb0 * d.V);
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (!in) continue;
    const int64_t r = r0 + t * kTileRows;
    uint32_t* dst = d.values + r * d.G + g;
    if (ng == 4) {
      *reinterpret_cast<u32x4_word*>(dst) = u32x4_word{x[t][0], x[t][1], x[t][2], x[t][3]};
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < ng) dst[e] = x[t][e];
    }
    if (h == 0) d.meta[r * d.W + w] = word[t];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t nib = (word[t] >> (16 * h + 4 * e)) & 0xfu;
      bad = bad || (e < ng ? (nib & 3u) >= (nib >> 2) : nib != 0);
    }
    const int rr = (t0 + t) * kTileRows + i;       // row of the packed block row
    if constexpr (PACKED) {
      char* rec = d.arec + (rb * d.W + w) * ((int64_t)d.vt * kTileValBytes + kTailBytes);
      *reinterpret_cast<uint4*>(rec + (t0 + t) * kTileValBytes + (32 * h + i) * 16) = make_uint4(x[t][0], x[t][1], x[t][2], x[t][3]);
      if (SPLIT) emit_index_field(d, rec, rr, h, word[t]);
      else if (h == 0) words[u >> 1][rr] = word[t];
    }
    const int v0 = first + t * kTileRows + i, down = v0 >= d.V ? v0 / d.V : 0, v = v0 - down * d.V;
    const int64_t cb = cb0 + down;
    const bool ids = PACKED && rr == 0;
    if (v == 0 || ids) {
      for (int e = 0; e < 4; ++e) {
        ushort4 c = make_ushort4(0, 0, 0, 0);
        if (e < ng) {
          const u16_any* cp = columns + (cb * d.G + g + e) * kSelCols;
          c = make_ushort4(cp[0], cp[1], cp[2], cp[3]);
          bad = bad || !(c.x < c.y && c.y < c.z && c.z < c.w && c.w < d.M);
          if (v == 0) emit_columns(d, cb, g + e, c);
        }
        if (ids) emit_rowidx(d, rb, w, 4 * h + e, c);
      }
    }
  }
  const unsigned long long lanes = __ballot(bad);
  if (bad && (lanes & ((1ull << threadIdx.x % 64) - 1)) == 0) report(legality, 0);   // (which one it is nobody asks)
  if constexpr (GATHER) {
    __syncthreads();
    const int k = threadIdx.x / 64, l = threadIdx.x % 64;
    const int64_t wk = (wblk << wbits) + k;
    if (wk < d.W) {
      uint32_t tiles[kMaxTiles];
#pragma unroll
      for (int e = 0; e < kMaxTiles; ++e) tiles[e] = e < NT ? words[k][32 * e + l % 32] : 0u;
      emit_index(d, d.arec + (rb * d.W + wk) * ((int64_t)d.vt * kTileValBytes + kTailBytes), l % 32, l / 32, tiles);
    }
  }
}

// Exact quotients of values below 2^31 by a divisor of at least 2: n / divisor = n * mul >> (31 + shift).
struct Divisor { uint32_t mul; int shift; };
static Divisor make_divisor(uint32_t d) {
  int l = 1;
  while ((1ull << l) < d) ++l;
  return {(uint32_t)(((1ull << (31 + l)) + d - 1) / d), l};
}
__device__ __forceinline__ uint32_t divide(uint32_t n, Divisor d) { return __umulhi(n, d.mul) >> (d.shift - 1); }

// packed -> dense.  A workgroup expands 32 rows (one tile of a block row) x 256 columns; a thread owns 8 neighbouring
// columns of four rows.  The NG groups that its columns can touch -- one where M is a multiple of 8, three at M = 5, else two
// (the first column is a multiple of 8, so at M = 6 at most the fifth of its group) -- are the same in every row, and so is
// what a nibble means there: of its two values, which bytes go to which of the four output words.  That is tabulated in LDS, as
// byte selectors for each of the six nibbles, while the loads of all four rows are in flight; then each row and group takes an
// index word, the two values, one LDS read and four byte permutations, and each row one 16-byte store at any alignment.
// ALL: M = 4, where every column is kept and a thread's two groups share an index word and an 8-byte pair of values.  PAIRS: M
// below 16, where most threads have two groups: neighbours, whose values lie side by side and whose index word is the same, unless
// the second starts a new half of the k-step.  STREAM: rows on 16-byte boundaries: stores past the caches, as nothing reads the
// lines again here and streamed they leave at the rate of a linear fill.  Other rows have their stores merged to whole lines in
// the L2, so neighbouring workgroups run on the same XCD.  Bound by the writes, below M = 16 by the number of loads.
// us per call (the same records and output again), positions compared in every row (some 40 instructions a row and group), one group at
// a time, all streamed -> now: 8192 x 8192 at 64:2:8 35 -> 31, at 64:2:16 29 -> 25, 49152 x 12288 at 128:2:32 210 -> 200 (6.5 TB/s; with others
// each time 274 -> 243); rows on no 16-byte boundary:
// 8192 x 8100 at 64:2:100 47 -> 24 (streamed 41), 8192 x 8180 at 64:2:20 50 -> 32, 8192 x 8190 at 64:2:10 50 -> 34 and at 64:2:7 67 -> 49
// (one group at a time 60).  The entries of a chunk staged in LDS by wide loads: 64:2:8 39, 64:2:7 65.
template <int NG, bool ALL, bool PAIRS, bool STREAM>
__global__ void __launch_bounds__(256) decompress_kernel(const char* __restrict__ arec,
                                                         const int32_t* __restrict__ rowidx, int64_t K, int M, Divisor by_M,
                                                         int64_t steps, int vt, int chunks, int64_t rt0,
                                                         uint16_t* __restrict__ A, int64_t lda) {
  __shared__ uint4 select[NG][16][32];                           // [group of the thread's columns][nibble][thread of a row]
  unsigned work = blockIdx.x;
  if constexpr (!STREAM) {
    const unsigned per_xcd = gridDim.x / 8;
    if (work < 8 * per_xcd) work = work % 8 * per_xcd + work / 8;
  }
  const unsigned rtl = work / (unsigned)chunks;
  const unsigned chunk = work - rtl * (unsigned)chunks;
  const int64_t rt = rt0 + rtl;                                  // 32-row tile of the matrix
  const int64_t b = rt / vt;
  const int tile = (int)(rt - b * vt);
  const unsigned cx = threadIdx.x & 31;
  const unsigned k = chunk * 256 + cx * 8;
  const bool inside = k < K;
  const int i0 = threadIdx.x >> 5;                               // rows i0, i0 + 8, ...
  const unsigned rec_bytes = (unsigned)(vt * kTileValBytes + kTailBytes);
  const char* recs = arec + b * steps * rec_bytes;
  const unsigned end = K - k < 8 ? (unsigned)K : k + 8;
  const unsigned g0 = divide(k, by_M);
  constexpr int NI = 4;                                          // rows per thread
  int4 ids[NG];
  uint32_t word[NG][NI] = {}, v01[NG][NI] = {};
  bool in[NG];
#pragma unroll
  for (int q = 0; q < NG; ++q) {
    const unsigned g = g0 + q, s = g / 8, t = g % 8;
    in[q] = inside && (q == 0 || g * (unsigned)M < end);         // (a group that starts past the columns may not exist)
    ids[q] = make_int4(0, 0, 0, 0);
    if (!in[q]) continue;
    if constexpr (ALL) ids[q] = make_int4((int)(4 * g), (int)(4 * g + 1), (int)(4 * g + 2), (int)(4 * g + 3));
    else ids[q] = *reinterpret_cast<const int4*>(rowidx + (b * steps + s) * kStepRows + 4 * t);
    if (PAIRS && q == 1 && t % 4 != 0) continue;                 // came with the group before
    const char* rec = recs + (int64_t)s * rec_bytes;
    const char* val = rec + tile * kTileValBytes + (32 * (t / 4) + i0) * 16 + (t % 4) * 4;
    const char* idx = rec + vt * kTileValBytes + (32 * (t / 4) + i0) * 8 + tile * 2;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      if constexpr (ALL || PAIRS) {
        if (ALL && q > 0) continue;
        // (the word after a group's values is in the record also where no group follows: another row's, or the tail)
        const u32x2_any pair = *reinterpret_cast<const u32x2_any*>(val + j * 128);
        word[q][j] = *reinterpret_cast<const uint16_t*>(idx + j * 64);
        v01[q][j] = pair.x;
        if (q == 0) { v01[1 % NG][j] = pair.y; word[1 % NG][j] = word[0][j]; }
      } else {
        word[q][j] = *reinterpret_cast<const uint16_t*>(idx + j * 64);
        v01[q][j] = *reinterpret_cast<const uint32_t*>(val + j * 128);
      }
    }
  }
  if (i0 < 6) {                                                  // the six nibbles p0 | p1 << 2 with p0 < p1
    const int p1 = i0 == 0 ? 1 : i0 < 3 ? 2 : 3, p0 = i0 - p1 * (p1 - 1) / 2;
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      const int4 ri = ids[q];
      auto pick = [&](int p) { return (unsigned)(p == 0 ? ri.x : p == 1 ? ri.y : p == 2 ? ri.z : ri.w) - k; };
      const unsigned c0 = pick(p0), c1 = pick(p1);               // outside 0 .. 7: not in this thread's columns
      uint32_t o[4];
#pragma unroll
      for (unsigned e = 0; e < 4; ++e) {                         // selector 0x0c: a zero byte
        const uint32_t lo = in[q] && c0 == 2 * e ? 0x0100u : in[q] && c1 == 2 * e ? 0x0302u : 0x0c0cu;
        const uint32_t hi = in[q] && c0 == 2 * e + 1 ? 0x0100u : in[q] && c1 == 2 * e + 1 ? 0x0302u : 0x0c0cu;
        o[e] = lo | hi << 16;
      }
      select[q][p0 | p1 << 2][cx] = make_uint4(o[0], o[1], o[2], o[3]);
    }
  }
  __syncthreads();
  if (!inside) return;
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    uint32_t o[4] = {0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      const uint32_t nib = in[q] ? word[q][j] >> (4 * ((g0 + q) % 4)) & 15u : 4u;
      const uint4 s = select[q][nib][cx];
      o[0] |= __builtin_amdgcn_perm(0u, v01[q][j], s.x);
      o[1] |= __builtin_amdgcn_perm(0u, v01[q][j], s.y);
      o[2] |= __builtin_amdgcn_perm(0u, v01[q][j], s.z);
      o[3] |= __builtin_amdgcn_perm(0u, v01[q][j], s.w);
    }
    uint16_t* row = A + (rt * kTileRows + i0 + 8 * j) * lda + k;
    if (end - k == 8) {
      if constexpr (STREAM) __builtin_nontemporal_store(u32x4_any{o[0], o[1], o[2], o[3]}, reinterpret_cast<u32x4_any*>(row));
      else *reinterpret_cast<u32x4_any*>(row) = u32x4_any{o[0], o[1], o[2], o[3]};
    } else {
#pragma unroll
      for (unsigned e = 0; e < 8; ++e)
        if (k + e < K) row[e] = (uint16_t)(o[e / 2] >> (16 * (e % 2)));
    }
  }
}

static FormatDst format_dst(const venom_handle& h) {
  const Layout& L = h.lay;
  FormatDst d{};
  d.values = reinterpret_cast<uint32_t*>(h.ws + L.off_values);
  d.columns = reinterpret_cast<uint16_t*>(h.ws + L.off_columns);
  d.meta = reinterpret_cast<uint32_t*>(h.ws + L.off_meta);
  d.arec = L.packed ? h.ws + L.off_arec : nullptr;
  d.rowidx = L.packed ? reinterpret_cast<int32_t*>(h.ws + L.off_rowidx) : nullptr;
  d.G = L.G; d.W = L.W;
  d.V = h.V; d.Vp = L.packed ? L.vt * kTileRows : h.V; d.vt = L.vt; d.M = h.M;
  return d;
}

hipError_t launch_import(const uint16_t* values, const uint16_t* columns, const uint32_t* meta, const venom_handle& h,
                         hipStream_t st, int slot, unsigned long long* found) {
  const Layout& L = h.lay;
  const Legality legality{slot, found, reinterpret_cast<unsigned long long*>(h.ws + L.off_status)};
  if (slot < 0) hipLaunchKernelGGL(init_status_kernel, dim3(1), dim3(1), 0, st, legality.own);
  if (L.R > 0 && L.G > 0) {
    // 4 words of a packed block row where there are packed records; otherwise longer pieces of fewer rows, as the rows are
    int wbits = 2;
    while (!L.packed && wbits < 5 && (1 << wbits) < L.W) ++wbits;
    const int64_t words = (L.W + (1 << wbits) - 1) >> wbits;
    // One tile a workgroup where there are fewer than three workgroups for each of 256 units: 8192 x 8192 at 128:2:64 (256 of them)
    // 27.3 whole, 25.7 split; at 128:2:20 (832) 35.2 and 36.3.  Also blocks of three and four tiles of 2^24 groups or more (64 MB of
    // values), whose 96 or 128 rows at once the memory takes more slowly, with other arrays each time or the same: 8192 x 8192 at
    // 128:2:4 85 whole, 79 split, 24576 x 12288 at 128:2:8 148 and 143, 49152 x 12288 at 128:2:16 153 and 147; below that the same arrays
    // again are faster whole, others slower (8192 x 8192 at 128:2:8 44.4 and 47.1, 57 and 54), and two tiles are faster whole (49152 x 12288 at
    // 64:2:8 282 and 299).  And packed blocks that are not the canonical ones (M = 4), where the rows of a thread lie in
    // several of those: 8192 x 8192 at 32:2:4 97 and 83, 1:2:4 193 and 177.
    const bool split = L.vt > 1 && (words * L.Rbp < 768 || (L.vt > 2 && L.R * L.G >= (int64_t)1 << 24) || h.V != L.vt * kTileRows);
    const int64_t rows = !L.packed ? 128 >> wbits : split ? kTileRows : L.vt * kTileRows;
    auto fn = L.vt == 0 ? import_kernel<0, false> : split ? import_kernel<1, true> : L.vt == 1 ? import_kernel<1, false>
              : L.vt == 2 ? import_kernel<2, false> : L.vt == 3 ? import_kernel<3, false> : import_kernel<4, false>;
    hipLaunchKernelGGL(fn, dim3((unsigned)(words * ((L.R + rows - 1) / rows))), dim3(256), 0, st,
                       reinterpret_cast<const u32_any*>(values), columns, meta, L.R, wbits, format_dst(h), legality);
  }
  return hipGetLastError();
}

hipError_t launch_compress(const uint16_t* A, int64_t lda, const uint8_t* mask, int64_t ldm, const venom_handle& h,
                           hipStream_t st, int slot, unsigned long long* found) {
  const Layout& L = h.lay;
  const Legality legality{slot, found, reinterpret_cast<unsigned long long*>(h.ws + L.off_status)};
  if (slot < 0) hipLaunchKernelGGL(init_status_kernel, dim3(1), dim3(1), 0, st, legality.own);
  if (L.R > 0 && L.G > 0) {
    // as many words per workgroup as leave eight workgroups per compute unit (rows of `values` are then written in
    // longer pieces) and the mask bits within LDS
    int wpw = kCompressWords;
    while (wpw > 1 && (((L.W + wpw - 1) / wpw) * L.Rb < 2048 || (int64_t)h.V * bits_pitch(wpw, h.M) > 16 * 1024)) wpw /= 2;
    const int64_t bit_bytes = (int64_t)h.V * bits_pitch(wpw, h.M);
    const int bits_ok = bit_bytes <= kCompressBits;
    const size_t lds = bits_ok ? (size_t)bit_bytes : 0;
    const dim3 grid((unsigned)((L.W + wpw - 1) / wpw), (unsigned)L.Rb);
    auto by = [](int64_t n) { return n > 0 ? (unsigned)((65535 + n) / n) : 0u; };
    // every chunk of columns in whole loads, fewer than 8 columns left over at the end of a row
    const int64_t chunk = (int64_t)8 * wpw * h.M, last = L.K - (grid.x - 1) * chunk;
    const int ub = chunk % 16 == 0 && L.K % 16 < 8 ? 16 : 8;
    auto of = [&](auto ne) {
      constexpr int NE = decltype(ne)::value;
      return ub == 8 ? compress_kernel<8, false, NE> : bits_ok ? compress_kernel<16, true, NE> : compress_kernel<16, false, NE>;
    };
    // A thread has V * wpw / 32 rows in phase 3, and rows that it does not have cost their instructions all the same: eight in flight
    // where there are three or more.  With 2 / 8, us per call: 49152 x 12288 at 1:2:32 1690 / 2579 (wpw = 4), 8:2:32 351 / 410,
    // 24:2:32 363 / 359, 32:2:32 409 / 392; 32768 x 768 at 64:2:32 36.3 / 40.8 (wpw = 1), 96:2:32 36.1 / 37.7, 128:2:32 36.6 / 37.8.
    auto fn = h.M >= 32 && (int64_t)h.V * wpw >= 96 ? of(std::integral_constant<int, 8>{}) : of(std::integral_constant<int, 2>{});
    hipLaunchKernelGGL(fn, grid, dim3(256), lds, st, A, lda, mask, ldm, wpw, bits_ok, by(chunk / ub), by(last / ub), format_dst(h),
                       legality);
  }
  return hipGetLastError();
}

hipError_t launch_take_violation(int slot, unsigned long long* to, hipStream_t st) {
  hipLaunchKernelGGL(take_violation_kernel, dim3(1), dim3(1), 0, st, slot, to);
  return hipGetLastError();
}

// The canonical arrays out of the workspace, all three in one launch: each workgroup copies 16 KB of one of them, 16
// bytes a thread and access, at any alignment of the destination, streamed.  Three asynchronous copies cost the host 5 us
// each, and two of them move next to nothing.  us per call of the binding, copies -> now: 49152 x 12288 at
// 128:2:32 (86 MB) 36 -> 29 (30 with cached stores), 16384 x 4096 at 128:2:4 32 -> 23, 512 x 1024 at 64:2:8 18 -> 13.5.
struct CopyList { const char* src[3]; char* dst[3]; int64_t bytes[3]; unsigned first[3]; };   // first workgroup of each
constexpr int kCopyUnits = 4;                        // 16-byte pieces per thread
constexpr int64_t kCopyBytes = 256 * 16 * kCopyUnits;

__global__ void __launch_bounds__(256) export_kernel(CopyList l) {
  const int k = blockIdx.x >= l.first[2] ? 2 : blockIdx.x >= l.first[1] ? 1 : 0;
  const char* src = k == 0 ? l.src[0] : k == 1 ? l.src[1] : l.src[2];
  char* dst = k == 0 ? l.dst[0] : k == 1 ? l.dst[1] : l.dst[2];
  const int64_t bytes = k == 0 ? l.bytes[0] : k == 1 ? l.bytes[1] : l.bytes[2];
  const int64_t at = (int64_t)(blockIdx.x - (k == 0 ? l.first[0] : k == 1 ? l.first[1] : l.first[2])) * kCopyBytes + threadIdx.x * 16;
  u32x4_any x[kCopyUnits];
#pragma unroll
  for (int j = 0; j < kCopyUnits; ++j) {
    const int64_t o = at + j * 4096;
    if (o + 16 <= bytes) x[j] = *reinterpret_cast<const u32x4_any*>(src + o);
  }
#pragma unroll
  for (int j = 0; j < kCopyUnits; ++j) {
    const int64_t o = at + j * 4096;
    if (o + 16 <= bytes) __builtin_nontemporal_store(x[j], reinterpret_cast<u32x4_any*>(dst + o));
    else
      for (int64_t e = o; e < bytes; e += 4)         // (the arrays are whole words)
        *reinterpret_cast<u32_any*>(dst + e) = *reinterpret_cast<const u32_any*>(src + e);
  }
}

hipError_t launch_export(const venom_handle& h, void* values, void* columns, void* meta, hipStream_t st) {
  const Layout& L = h.lay;
  CopyList l{{h.ws + L.off_values, h.ws + L.off_columns, h.ws + L.off_meta},
             {static_cast<char*>(values), static_cast<char*>(columns), static_cast<char*>(meta)},
             {values ? L.R * L.G * 4 : 0, columns ? L.Rb * L.G * 8 : 0, meta ? L.R * L.W * 4 : 0},
             {0, 0, 0}};
  unsigned blocks = 0;
  for (int k = 0; k < 3; ++k) {
    l.first[k] = blocks;
    blocks += (unsigned)((l.bytes[k] + kCopyBytes - 1) / kCopyBytes);
  }
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(export_kernel, dim3(blocks), dim3(256), 0, st, l);
  return hipGetLastError();
}

template <bool STREAM>
static auto decompress_of(int M) {
  return M % 8 == 0 ? decompress_kernel<1, false, false, STREAM> : M == 4 ? decompress_kernel<2, true, false, STREAM>
         : M == 5 ? decompress_kernel<3, false, true, STREAM> : M < 16 ? decompress_kernel<2, false, true, STREAM>
         : decompress_kernel<2, false, false, STREAM>;
}

hipError_t launch_decompress(const venom_handle& h, uint16_t* A, int64_t lda, hipStream_t st) {
  const Layout& L = h.lay;
  if (L.R == 0 || L.K == 0) return hipSuccess;
  const int64_t chunks = (L.K + 255) / 256;
  const bool aligned = reinterpret_cast<uintptr_t>(A) % 16 == 0 && lda % 8 == 0;
  auto fn = aligned ? decompress_of<true>(h.M) : decompress_of<false>(h.M);
  // Six workgroups a unit (24 KB of LDS each) and not eight, where whole lines are streamed: more reads and stores in flight at once
  // slow the memory down.  us per call with 8 / 6, cold (other records and output each time) and hot: 49152 x 12288 at 128:2:8 318 / 295 and
  // 318 / 296 (before the table, at whose pace there were fewer: 299), 128:2:16 285 / 245 and 202 / 195, 128:2:20 354 / 338, 128:2:32
  // 264 / 243, 24576 x 12288 at 128:2:10 179 / 173, 8192 x 8192 at 64:2:8 38.0 / 35.4 and 31.2 / 30.7.  Not above M = 64, where little is
  // read (49152 x 12288 at 128:2:128 198 / 205), nor for merged stores (8192 x 8100 at 64:2:100 38 / 42), nor where all run in three or
  // four rounds (4032 x 4096 at 96:2:16 11.4 / 12.5); M = 5 has six anyway.
  const size_t tables = (size_t)(h.M % 8 == 0 ? 1 : h.M == 5 ? 3 : 2) * 8 * 1024;
  const size_t lds = aligned && h.M <= 64 && L.R / kTileRows * chunks >= 24 * 256 ? 24 * 1024 - tables : 0;
  // a launch holds fewer than 2^32 threads, 256 per workgroup however few columns there are: tall narrow matrices
  // take several
  const int64_t tiles = L.R / kTileRows, most = kMaxBlocks / chunks;
  for (int64_t rt0 = 0; rt0 < tiles; rt0 += most) {
    const int64_t n = tiles - rt0 < most ? tiles - rt0 : most;
    hipLaunchKernelGGL(fn, dim3((unsigned)(n * chunks)), dim3(256), lds, st, h.ws + L.off_arec,
                       reinterpret_cast<const int32_t*>(h.ws + L.off_rowidx), L.K, h.M, make_divisor((uint32_t)h.M), L.steps,
                       L.vt, (int)chunks, rt0, A, lda);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace venom
