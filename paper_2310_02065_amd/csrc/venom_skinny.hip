// The product with at most 32 columns, and the layer with at most 32 tokens: decoding, small batches.  A tile of spmm_kernel
// would be mostly padding there, and its k-steps, one barrier each, a chain that a call waits for; the bound is the stream of A,
// each record of it read once, or for a small matrix the launch.  So:
//   * a workgroup owns RT of the 32-row tiles of a block row and NP waves deal out its k-steps, wave w taking steps w,
//     w + NP, ...: each wave reads whole records two of its k-steps ahead, straight into the operand registers (the packed
//     order is the operand's), and there is no barrier until the end, where the partial sums meet in LDS, in a fixed order;
//   * the B operand has one 32-column tile.  A product's waves gather the 32 rows of the k-step, 64 bytes each, into LDS of
//     their own and read them transposed.  A layer's may take them from X itself, [token][k]: the wave stages the 8*M
//     columns of the k-step for every token, and the gather is a 2-byte LDS read at any column, so that X is not transposed
//     by a kernel before: 3.5 us less for M/4 times the bytes of X.
// Measured, us per call, spmm_kernel's 64-column tile (and the transposition) -> now, the same call again: 8192 x 8192 x 16 at
// 128:2:16 11.6 -> 6.7, as a layer 14.9 -> 9.4; 96 x 13552 x 32 at 96:2:8 (one block row) 28 -> 10; 1024 x 1024 x 8 at 128:2:8 6.0 -> 4.4,
// as a layer 9.4 -> 5.9; the layer of 49152 x 12288 with 16 tokens, bias and GELU at 128:2:32 (85 MB of records) 22.6 -> 20.1, with
// other weights and activations each time 24.8 -> 22.3.
#include <atomic>
#include <cmath>

#include "venom_device.h"

namespace venom {

struct SkinnyParams {
  const char* arec;        // packed A stream, as for spmm_kernel
  const int32_t* rowidx;
  const char* src;         // X (tokens x K) or B (K x columns), fp16
  void* out;               // token-major [column][row] for a layer, else [row][column]
  int64_t ldo, rec_bytes;
  uint32_t ld_bytes;       // of src: everything lies within 2^32 bytes of it
  int cols;                // tokens or columns, at most 32
  int K, M, G, steps, nbr;
  const _Float16* bias;
  int act;
  int token_major;         // a product: the layout of out
};

constexpr int kSkinnyCols = 32;
// bytes of LDS in which a wave stages X for a k-step, with a spare piece
__host__ __device__ constexpr int skinny_window(int cols, int M) { return cols * (M | 1) * 16 + 16; }

// VT: 32-row tiles per block row; RT: those of a workgroup; NP: phases, the waves that deal out its k-steps; GB: block rows per
// workgroup, NP waves each, whose waves of one phase share the window of X (all waves then keep in step, two windows in turn);
// XJ: 16-byte pieces of X that a lane stages per k-step and block row (0: a product, B is gathered from memory), all of them
// loaded: those past the last token are the first piece again.
// Registers for two waves per SIMD, enough but for pairs of block rows of 128 with 16 pieces, which spill 7 of them (32 bytes a lane); three
// records ahead instead of two measured the same.
template <int VT, int RT, int NP, int GB, int XJ, bool OUT_F32>
__global__ void __launch_bounds__(NP * GB * 64, 2) skinny_kernel(SkinnyParams p) {
  constexpr bool TOKENS = XJ > 0;
  static_assert(GB == 1 || (RT == VT && NP == 4 && TOKENS), "block rows share X");
  constexpr int PA = 2;                            // records on the way ahead of the one in work
  extern __shared__ __attribute__((aligned(16))) char skinny_lds[];
  const int lane = threadIdx.x & 63, h = lane >> 5, col = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int phase = GB == 1 ? wave : wave % NP, member = GB == 1 ? 0 : wave / NP;
  int br = RT == VT ? blockIdx.x * GB + member : blockIdx.x / (VT / RT);
  const bool exists = GB == 1 || br < p.nbr;
  if (GB > 1 && !exists) br = p.nbr - 1;           // (an odd block row at the end: its second half goes along, and stores nothing)
  const int t0 = RT == VT ? 0 : (blockIdx.x % (VT / RT)) * RT;
  const char* recs = p.arec + (int64_t)br * p.steps * p.rec_bytes;
  const int32_t* ids = p.rowidx + (int64_t)br * p.steps * kStepRows;

  // lane offsets as 32-bit values that are only widened where they are used: a load then takes them beside a scalar base
  auto at = [](const char* base, uint32_t off) {
    asm("" : "+v"(off));
    return base + off;
  };
  half8 av[PA + 1][RT];
  uint32_t ix[PA + 1][(RT + 1) / 2];               // tiles t and t + 1 of a word
  int id[PA + 1][TOKENS ? 1 : 2];                  // a layer: lane l < 32 has row id l of the k-step; a product: rows l/4, 16 + l/4
  auto load_a = [&](int slot, int s) {
    const char* row_ids = reinterpret_cast<const char*>(ids + (int64_t)s * kStepRows);
    id[slot][0] = *reinterpret_cast<const int*>(at(row_ids, (TOKENS ? col : lane >> 2) * 4));
    if constexpr (!TOKENS) id[slot][1] = *reinterpret_cast<const int*>(at(row_ids + 64, (lane >> 2) * 4));
    const char* rec = recs + (int64_t)s * p.rec_bytes;
#pragma unroll
    for (int t = 0; t < RT; ++t) av[slot][t] = *reinterpret_cast<const half8*>(at(rec + (t0 + t) * kTileValBytes, lane * 16));
    const char* tail = at(rec + VT * kTileValBytes + 2 * t0, lane * 8);
    if constexpr (RT == 1) ix[slot][0] = *reinterpret_cast<const uint16_t*>(tail);
    else if constexpr (RT == 2) ix[slot][0] = *reinterpret_cast<const uint32_t*>(tail);
    else {
      const uint2 w = *reinterpret_cast<const uint2*>(tail);
      ix[slot][0] = w.x;
      ix[slot][1] = w.y;
    }
  };

  // ---- the layer's X: a k-step's window is 8 * M columns, M pieces of 16 bytes a token; piece q = lane + 64 j is the (q % M)-th
  // of token q / M
  const int pieces = p.M, pitch = (pieces | 1) * 16;   // an odd number of 16-byte units: tokens on different banks
  // ---- LDS: a layer's waves hold the offsets of a k-step's rows, one area for each wave, and the windows, one for each wave, or
  // two for each phase where the waves of several block rows share them; a product's waves the 32 gathered rows, 64 bytes each
  constexpr int kArea = TOKENS ? 128 : kStepRows * 64;
  char* offs = skinny_lds + wave * kArea;
  const int window = skinny_window(p.cols, p.M);
  char* win = skinny_lds + NP * GB * kArea + (GB == 1 ? wave : 2 * phase) * window;
  int flip = GB == 1 ? 0 : window;                 // from the window in use to the other one
  constexpr int XN = TOKENS ? XJ / GB : 2;
  uint32_t xoff[XN], xlds[XN];
  u32x4_any xr[XN];
  if constexpr (TOKENS) {
#pragma unroll
    for (int j = 0; j < XN; ++j) {
      const int q = lane + 64 * (j + XN * member), tok = q / pieces, c = q - tok * pieces;
      const bool in = tok < p.cols;                // past the last token: the first piece again, to the spare one
      xoff[j] = in ? (uint32_t)tok * p.ld_bytes + c * 16 : 0u;
      xlds[j] = in ? tok * pitch + c * 16 : p.cols * pitch;
    }
  } else xoff[0] = (lane & 3) * 8 < p.cols ? (lane & 3) * 16 : 0u;   // (columns past the last: any others, never stored)
  // What a wave has put into LDS its other lanes read, as other types: nothing in the language keeps that order, so the compiler
  // is told (the hardware runs a wave's LDS accesses in order).
  auto lds_in_order = []() { asm volatile("" ::: "memory"); };
  auto load_x = [&](int s) {                       // a whole window
    const char* base = p.src + (int64_t)s * (16 * pieces);
#pragma unroll
    for (int j = 0; j < XN; ++j) xr[j] = *reinterpret_cast<const u32x4_any*>(at(base, xoff[j]));
  };
  auto put_x = [&]() {
    lds_in_order();                                // after the reads of the last k-step
#pragma unroll
    for (int j = 0; j < XN; ++j) *reinterpret_cast<uint4*>(win + xlds[j]) = make_uint4(xr[j].x, xr[j].y, xr[j].z, xr[j].w);
  };
  auto stage_end = [&](int s) {                    // the columns that are left, and nothing past the end of a row
    const char* base = p.src + (int64_t)s * (16 * pieces);
    const int n = p.K - s * 8 * p.M, wide = n >> 3;   // pieces that are there as a whole; pieces past them are not read later
#pragma unroll
    for (int j = 0; j < XN; ++j) {
      const int q = lane + 64 * (j + XN * member), tok = q / pieces, c = q - tok * pieces;
      if (tok < p.cols && c < wide) xr[j] = *reinterpret_cast<const u32x4_any*>(at(base, xoff[j]));
      else xr[j] = u32x4_any{0, 0, 0, 0};
    }
    uint32_t rest[7];                              // the last columns: lane l's token
#pragma unroll
    for (int e = 0; e < 7; ++e)
      rest[e] = lane < p.cols && e < (n & 7) ? *reinterpret_cast<const u16_any*>(at(base, lane * p.ld_bytes + wide * 16 + 2 * e)) : 0;
    put_x();
    lds_in_order();                                // zeros of other lanes lie where these go
    if (lane < p.cols)
#pragma unroll
      for (int e = 0; e < 7; ++e)
        if (e < (n & 7)) *reinterpret_cast<uint16_t*>(win + lane * pitch + wide * 16 + 2 * e) = (uint16_t)rest[e];
  };

  // ---- a product's rows: lane l loads 16 bytes of rows l/4 and 16 + l/4, which lie in LDS as [row][32 columns]
  auto load_rows = [&](int slot) {
#pragma unroll
    for (int j = 0; j < 2; ++j) xr[j] = *reinterpret_cast<const u32x4_any*>(at(p.src, (uint32_t)id[slot][TOKENS ? 0 : j] * p.ld_bytes + xoff[0]));
  };
  auto put_rows = [&]() {
    lds_in_order();
#pragma unroll
    for (int j = 0; j < 2; ++j) *reinterpret_cast<uint4*>(offs + j * 1024 + lane * 16) = make_uint4(xr[j].x, xr[j].y, xr[j].z, xr[j].w);
  };

  // ---- the B operand of a k-step: lane half h holds, of column `col`, the 4 rows of groups 2h, 2h + 1, 4 + 2h and 5 + 2h.
  // A product: transposing LDS reads, as in spmm_kernel.  A layer: the offsets of the 32 rows go through LDS, where each half
  // reads its own, and the halfs come from the window.
  const uint32_t my_row = (col < p.cols ? col : 0) * pitch;   // (lanes past the last column: any of them, never stored)
  auto operand = [&](int row_id, int s) {
    half16 b;
    if constexpr (TOKENS) {
      const int c0 = row_id - s * 8 * p.M;         // (groups past the end have row 0: any column of the window)
      if (lane < kStepRows) *reinterpret_cast<uint32_t*>(offs + 4 * lane) = 2u * (c0 > 0 ? c0 : 0);
      lds_in_order();
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        const uint4 o = *reinterpret_cast<const uint4*>(offs + 16 * (4 * (cb >> 1) + (cb & 1) + 2 * h));
        const uint32_t oe[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) b[4 * cb + e] = *reinterpret_cast<const _Float16*>(win + (my_row + oe[e]));
      }
    } else {
      lds_in_order();
      const int blk = lane >> 4, i = lane & 15;
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        const int row = 4 * (4 * (cb >> 1) + 2 * (blk >> 1) + (cb & 1)) + (i >> 2);
        const short4v piece = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (LDS_PTR(short4v))(offs + row * 64 + (blk & 1) * 32 + (i & 3) * 8));
        const half4 ph = __builtin_bit_cast(half4, piece);
        b[4 * cb + 0] = ph[0]; b[4 * cb + 1] = ph[1]; b[4 * cb + 2] = ph[2]; b[4 * cb + 3] = ph[3];
      }
    }
    return b;
  };
  auto clear_absent = [&](half16& b, int s) {      // groups past the end: their values are zero, but 0 x Inf is not
    const int left = p.G - 8 * s;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (4 * (cb >> 1) + (cb & 1) + 2 * h >= left) b[4 * cb + e] = (_Float16)0.f;
  };

  floatx16 acc[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;

  auto multiply = [&](int slot, const half16& b) {
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      if (t & 1) acc[t] = smfmac<1>(av[slot][t], b, acc[t], (int)ix[slot][t >> 1]);
      else acc[t] = smfmac<0>(av[slot][t], b, acc[t], (int)ix[slot][t >> 1]);
    }
  };
  // The k-steps with all their groups, without a branch: near the end the streams fetch their last k-step again.
  const int whole = p.G / 8;
  const int mine = whole > phase ? (whole - phase + NP - 1) / NP : 0;
  int n = GB == 1 ? mine : (whole + NP - 1) / NP;  // (where windows are shared all waves keep in step)
  const int last = mine > 0 ? phase + (mine - 1) * NP : 0;
  int s = phase;
  auto at_most_last = [&](int x) { return x < last ? x : last; };
  auto step = [&](int slot, int next_slot) {
    const int s1 = at_most_last(s + NP), s2 = at_most_last(s + PA * NP);
    if constexpr (TOKENS) put_x();
    else put_rows();
    if constexpr (XN > 8) __builtin_amdgcn_sched_barrier(0);   // (registers for one window, not two)
    if constexpr (TOKENS) load_x(s1);
    else load_rows((slot + 1) % (PA + 1));
    load_a(next_slot, s2);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (GB > 1) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const half16 b = operand(id[slot][0], s);
    if (GB == 1 || s < whole) multiply(slot, b);
    __builtin_amdgcn_sched_barrier(0);             // (or the loads of three steps are hoisted into registers that do not exist)
    s += NP;
    if constexpr (GB > 1) { win += flip; flip = -flip; }
  };
  if (n > 0) {
    if constexpr (TOKENS) load_x(at_most_last(s));
    load_a(0, at_most_last(s));
#pragma unroll
    for (int k = 1; k < PA; ++k) load_a(k, at_most_last(s + k * NP));
    if constexpr (!TOKENS) load_rows(0);
    for (; n > PA; n -= PA + 1)
#pragma unroll
      for (int k = 0; k <= PA; ++k) step(k, (k + PA) % (PA + 1));
#pragma unroll
    for (int k = 0; k < PA; ++k)
      if (k < n) step(k, (k + PA) % (PA + 1));
  }
  if (p.steps > whole) {                           // the last k-step, where G is no multiple of 8: one phase's
    const bool ours = phase == whole % NP;
    if (ours) {
      load_a(0, whole);
      if constexpr (TOKENS) stage_end(whole);      // (to the window that nobody has read since the last barrier)
      else { load_rows(0); put_rows(); }
    }
    // each wave of the phase has staged its share of the window
    if constexpr (GB > 1) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (ours) {
      half16 b = operand(id[0][0], whole);
      clear_absent(b, whole);
      multiply(0, b);
    }
  }

  // ---- the partial sums of the waves, halved until four are left, then summed by one wave per tile
  float4* red = reinterpret_cast<float4*>(skinny_lds) + member * (4 * RT * 256);
  auto put = [&](int slot, int t) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      red[(slot * 4 + q) * 64 + lane] = make_float4(acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]);
  };
  auto add = [&](int slot, int t) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 x = red[(slot * 4 + q) * 64 + lane];
      acc[t][4 * q] += x.x; acc[t][4 * q + 1] += x.y; acc[t][4 * q + 2] += x.z; acc[t][4 * q + 3] += x.w;
    }
  };
  __syncthreads();                                 // the windows are done with
#pragma unroll
  for (int m = NP; m > 4; m /= 2) {
    if (phase >= m / 2 && phase < m)
#pragma unroll
      for (int t = 0; t < RT; ++t) put((phase - m / 2) * RT + t, t);
    __syncthreads();
    if (phase < m / 2)
#pragma unroll
      for (int t = 0; t < RT; ++t) add(phase * RT + t, t);
    __syncthreads();
  }
  if (phase < 4)
#pragma unroll
    for (int t = 0; t < RT; ++t)
      if (t != phase) put(phase * RT + t, t);
  __syncthreads();
  if (phase >= RT || !exists) return;
  floatx16 sum;
#pragma unroll
  for (int t = 0; t < RT; ++t)
    if (t == phase) sum = acc[t];
#pragma unroll
  for (int w = 0; w < 4; ++w)
    if (w != phase) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 x = red[((w * RT + phase) * 4 + q) * 64 + lane];
        sum[4 * q] += x.x; sum[4 * q + 1] += x.y; sum[4 * q + 2] += x.z; sum[4 * q + 3] += x.w;
      }
    }

  // ---- element v of the tile sits at row 8*(v/4) + 4*h + v%4, column lane%32
  const int64_t row0 = ((int64_t)br * VT + t0 + phase) * kTileRows + 4 * h;
  if (col >= p.cols) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float o[4];
    half4 b4 = {};
    if (p.bias) b4 = *reinterpret_cast<const half4*>(p.bias + row0 + 8 * q);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o[e] = sum[4 * q + e];
      if (p.bias) o[e] += (float)b4[e];
      if (p.act == VENOM_ACT_GELU) o[e] = gelu_by_definition<OUT_F32>(o[e]);
      else if (p.act == VENOM_ACT_GELU_TANH) o[e] = gelu_tanh_form(o[e]);
    }
    if (TOKENS || p.token_major) {
      const int64_t at = (int64_t)col * p.ldo + row0 + 8 * q;
      if constexpr (OUT_F32) *reinterpret_cast<float4*>(reinterpret_cast<float*>(p.out) + at) = make_float4(o[0], o[1], o[2], o[3]);
      else *reinterpret_cast<half4*>(reinterpret_cast<_Float16*>(p.out) + at) = half4{(_Float16)o[0], (_Float16)o[1], (_Float16)o[2], (_Float16)o[3]};
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t at = (row0 + 8 * q + e) * p.ldo + col;
        if constexpr (OUT_F32) reinterpret_cast<float*>(p.out)[at] = o[e];
        else reinterpret_cast<_Float16*>(p.out)[at] = (_Float16)o[e];
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
constexpr int kSkinnyPieces = 16;            // most pieces of X that a lane stages

template <int VT, int FORM, int XJ>
static void (*skinny_of(bool f32))(SkinnyParams) {
  constexpr int RT = FORM == kSplit ? 1 : VT, NP = FORM == kSplit ? 8 : 4, GB = FORM == kPair ? 2 : 1;
  return f32 ? skinny_kernel<VT, RT, NP, GB, XJ, true> : skinny_kernel<VT, RT, NP, GB, XJ, false>;
}
// a product is served split or whole, a layer that reads X itself split or by pairs
template <int VT>
static void (*skinny_of(int form, int xj, bool f32))(SkinnyParams) {
  if (xj == 0) return form == kSplit ? skinny_of<VT, kSplit, 0>(f32) : skinny_of<VT, kWhole, 0>(f32);
  if (form == kSplit) return xj == 8 ? skinny_of<VT, kSplit, 8>(f32) : skinny_of<VT, kSplit, 16>(f32);
  return xj == 8 ? skinny_of<VT, kPair, 8>(f32) : skinny_of<VT, kPair, 16>(f32);
}

// Whether the kernel can serve: sizes, 32-bit offsets into B or X, and a launch of fewer than 2^32 threads, 512 for each tile at most
// (spmm_kernel's grid does not grow with the matrix)
static bool skinny_can(const Layout& L, int64_t ld, int64_t cols, bool tokens) {
  if (!L.packed || L.R == 0 || L.steps == 0 || cols < 1 || cols > kSkinnyCols) return false;
  if (L.K >= (int64_t)1 << 24 || L.Rbp * L.vt >= (int64_t)1 << 23 || ld >= (int64_t)1 << 31) return false;
  return 2 * (tokens ? (cols - 1) * ld + L.K : (L.K - 1) * ld + cols) < (int64_t)1 << 32;
}

// A product: single tiles where whole block rows leave the chip idle: 5888 x 8640 x 32 at 128:2:16 8.5 whole, 5.7 split; 9472 x
// 2896 x 8 at 64:2:16 4.6 both; 17664 x 6112 x 8 at 128:2:16 8.7 whole, 14.8 split (each tile gathers its rows of B again).
static bool split_pays(int64_t tiles, int cus) { return tiles * 64 < 75 * (int64_t)cus; }

// Many block rows of 128 keep spmm_kernel's units busy, whose loads bypass the registers: 49152 x 12288 x 16 at 128:2:32 16.8
// there, 17.5 here; 24448 x 14320 x 32 at 128:2:20 15.9 and 16.6; up to 64 rows it is slower there, too (19648 x 4704 x 32 at
// 64:2:32 7.6 and 5.8)
static bool tile_serves(const Layout& L, int cus) { return L.vt == kMaxTiles && L.Rbp * 64 >= 50 * (int64_t)cus; }

int skinny_product(const venom_handle& h, int64_t ld, int64_t cols, int cus) {
  const Layout& L = h.lay;
  if (!skinny_can(L, ld, cols, false) || tile_serves(L, cus)) return -1;
  return split_pays(L.Rbp * L.vt, cus) ? kSplit : kWhole;
}

// Pieces of X that a lane loads per k-step (the needed ones or copies of the first): two instantiations.
static int staged_pieces(int64_t tokens, int M) { return tokens * M <= 64 * 8 ? 8 : kSkinnyPieces; }
static int layer_lds(int64_t tokens, int M) { return 8 * (128 + skinny_window((int)tokens, M)); }

// A layer: X read in place, split or by pairs of block rows, or transposed and then a product.  The expected times are fits to
// 8250 random shapes (R 64-49152, K 64-16000, 8-32 tokens, M 4-128; rms error 5 to 7 %): `load` workgroups per unit, `rounds` of
// them, one at a time (pairs of single tiles with 8 staged pieces: two, if their LDS leaves room, `starts`), `spw` k-steps per wave.
// On 2750 others the choice is 0.7 % slower than the best on average, and takes 0.74 of the time of transposition and 64-column tiles, 1.14 times
// at most and more than 1.05 in one of 300.  (Fits to 240 shapes, with the needed pieces in the place of the loaded ones and no
// rounds of pairs, took these also for many block rows of few k-steps: 35712 x 896 with 16 tokens at 32:2:64 10.8 -> 18.3 us, now
// 7.3.)  Reading in place counts 5 % less, as on an idle GPU a second launch costs more than among others.
static int layer_form(const Layout& L, int64_t ldx, int64_t tokens, int M, int cus) {
  if (!skinny_can(L, ldx, tokens, true) || tokens * M > 64 * kSkinnyPieces) return -1;
  const int64_t tiles = L.Rbp * L.vt, pairs = (L.Rbp + 1) / 2;
  const float steps = (float)L.steps, vt = (float)L.vt, end = L.G % kStepGroups ? 1.f : 0.f;
  const float staged = (float)staged_pieces(tokens, M), pieces = (float)(tokens * M) / 64.f;
  const float records = (float)(4.5e-6 * (double)L.R * (double)L.G) - 20.f, more = records > 0.f ? records : 0.f;   // MB over 20
  const float x_mb = (float)(2e-6 * (double)tokens * (double)L.K);
  auto rounds_of = [&](int64_t wgs, int64_t resident) { return (float)((wgs + resident * cus - 1) / (resident * cus)); };
  struct Shape { float load, rounds, spw; };
  auto shape = [&](int64_t wgs, int waves) {
    return Shape{(float)wgs / (float)cus, rounds_of(wgs, 1), (float)((L.steps + waves - 1) / waves)};
  };
  const Shape s = shape(tiles, 8), w = shape(L.Rbp, 4), p = shape(pairs, 4);
  const float starts = rounds_of(pairs, L.vt == 1 && staged <= 8.f && layer_lds(tokens, M) <= 80 * 1024 ? 2 : 1);
  const float split = 2.83f + s.rounds * (1.19f + .0455f * staged + s.spw * (.027f + .0727f * staged)) +
                      s.load * steps * (.0114f + .0055f * pieces) + .196f * s.spw + .405f * end;
  const float pair = 2.3f + starts * (2.57f + .0164f * staged + .1485f * p.spw) + p.rounds * p.spw * (.0435f * staged + .1167f * vt) +
                     p.load * (.0086f * steps * pieces + .23f * vt) + .445f * end;
  const float first = split_pays(tiles, cus)
      ? 6.2f + s.load * (.11f + .01f * steps) + s.spw * (.0793f + .2625f * s.rounds) + .36f * x_mb + .822f * sqrtf(x_mb) + .0448f * more + .388f * end
      : tile_serves(L, cus)
      ? 7.12f + 1.126f * w.rounds + w.load * .0287f * steps * vt + w.spw * (.0435f + .1577f * w.rounds) + .329f * sqrtf(x_mb) + .395f * end
      : 5.88f + .345f * vt + w.load * .0289f * steps * vt + w.spw * (.0229f + .1187f * w.rounds) + 1.664f * x_mb + .013f * more + .4185f * end;
  if (split <= pair) return split < 1.05f * first ? kSplit : -1;
  return pair < 1.05f * first ? kPair : -1;
}

struct Rows { const void* at; uintptr_t bytes, pitch; };   // of a row, and from one to the next

// Whether two matrices of as many rows have bytes in common: from the first to the last, gaps between rows included, but for
// matrices side by side in the rows of one buffer.
static bool overlap(const Rows& a, const Rows& b, int64_t rows) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a.at), y = reinterpret_cast<uintptr_t>(b.at), gaps = (uintptr_t)(rows - 1);
  if (x >= y + gaps * b.pitch + b.bytes || y >= x + gaps * a.pitch + a.bytes) return false;
  if (a.pitch != b.pitch) return true;
  const uintptr_t behind = y >= x ? (y - x) % a.pitch : (a.pitch - (x - y) % a.pitch) % a.pitch;   // where in a row of a one of b starts
  return behind < a.bytes || behind + b.bytes > a.pitch;
}

// An output over X stays with the transposition, which has read all of X before the product starts: a workgroup here reads
// every column of X to the end of its run, when others have long stored their features.
int skinny_layer(const venom_handle& h, const void* X, int64_t ldx, int64_t tokens, const void* Y, int64_t ldy, int dtype, int cus) {
  const int form = layer_form(h.lay, ldx, tokens, h.M, cus);
  const uintptr_t size = dtype == 1 ? 4 : 2;
  const Rows x{X, 2 * (uintptr_t)h.K, 2 * (uintptr_t)ldx}, y{Y, size * (uintptr_t)h.R, size * (uintptr_t)ldy};
  return form < 0 || overlap(x, y, tokens) ? -1 : form;
}

venom_status_t launch_skinny(const venom_handle& h, int form, const void* src, int64_t ld, int64_t cols, const void* bias, int act,
                             void* out, int64_t ldo, int dtype, bool in_place, bool token_major, hipStream_t st) {
  const Layout& L = h.lay;
  if (!skinny_can(L, ld, cols, in_place) || (in_place && cols * h.M > 64 * kSkinnyPieces)) return VENOM_ERR_UNSUPPORTED;
  if (form != kSplit && form != (in_place ? kPair : kWhole)) return VENOM_ERR_UNSUPPORTED;
  SkinnyParams p{};
  p.arec = h.ws + L.off_arec;
  p.rowidx = reinterpret_cast<const int32_t*>(h.ws + L.off_rowidx);
  p.src = static_cast<const char*>(src);
  p.out = out;
  p.ldo = ldo; p.rec_bytes = L.rec_bytes;
  p.ld_bytes = (uint32_t)(2 * ld);
  p.cols = (int)cols;
  p.K = (int)h.K; p.M = h.M; p.G = (int)L.G; p.steps = (int)L.steps; p.nbr = (int)L.Rbp;
  p.bias = static_cast<const _Float16*>(bias);
  p.act = act;
  p.token_major = token_major;
  const int xj = in_place ? staged_pieces(cols, h.M) : 0;
  const bool f32 = dtype == 1;
  auto fn = L.vt == 1 ? skinny_of<1>(form, xj, f32) : L.vt == 2 ? skinny_of<2>(form, xj, f32)
            : L.vt == 3 ? skinny_of<3>(form, xj, f32) : skinny_of<4>(form, xj, f32);
  const int rt = form == kSplit ? 1 : L.vt, gb = form == kPair ? 2 : 1, waves = form == kWhole ? 4 : 8;
  const int staged = in_place ? layer_lds(cols, h.M) : waves * kStepRows * 64, sums = 4 * rt * gb * 4096;
  const int lds = staged > sums ? staged : sums;
  if (lds > 64 * 1024) {
    // opting in to more than 64 KB of dynamic LDS is a per-function attribute, set once per device, to the most that any call
    // needs (two threads racing here both set the same attribute: harmless)
    constexpr int kMost = 160 * 1024;
    static std::atomic<bool> opted_in[kMaxTiles][3][2][2][kMaxDevices] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return VENOM_ERR_HIP;
    const bool cached = dev >= 0 && dev < kMaxDevices;
    std::atomic<bool>* done = cached ? &opted_in[L.vt - 1][form][xj == kSkinnyPieces][f32][dev] : nullptr;
    if (!done || !done->load(std::memory_order_acquire)) {
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, kMost) != hipSuccess)
        return VENOM_ERR_HIP;
      if (done) done->store(true, std::memory_order_release);
    }
  }
  hipLaunchKernelGGL(fn, dim3((unsigned)((L.Rbp + gb - 1) / gb * (L.vt / rt))), dim3(64 * waves), lds, st, p);
  return hipGetLastError() == hipSuccess ? VENOM_OK : VENOM_ERR_HIP;
}

}  // namespace venom
