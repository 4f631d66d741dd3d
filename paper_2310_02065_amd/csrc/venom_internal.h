// Internal declarations shared by the library's translation units (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "venom.h"

namespace venom {

constexpr int kSelCols = 4;    // columns kept per V x M block (section 3)
constexpr int kTileRows = 32;  // rows of one matrix-instruction tile (v_smfmac_f32_32x32x32_f16)
constexpr int kStepGroups = 8; // groups of M columns consumed per k-step: 8 groups x 4 columns = 32
constexpr int kStepRows = kStepGroups * kSelCols;  // gathered rows of B per k-step
constexpr int kTileValBytes = 1024;                // packed values of one 32-row tile for one k-step
constexpr int kMaxTiles = 4;                       // the product kernel serves V = 32, 64, 96, 128
constexpr int kTailBytes = 512;                    // record tail: the index words, 64 lanes x 4 tiles x 16 bits
constexpr int kMaxDevices = 16;    // devices whose per-device launch state is cached
constexpr int64_t kMaxBlocks = (1 << 24) - 1;      // most workgroups of 256 threads along x: a launch holds fewer than
                                                   // 2^32 threads there

// Words of arrays that come from outside at any address: global accesses need no alignment on this target, and the
// compiler emits the same single loads for these types as for the aligned ones.
typedef uint32_t u32_any __attribute__((aligned(1)));
typedef uint16_t u16_any __attribute__((aligned(1)));
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(1)));
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t u32x4_word __attribute__((ext_vector_type(4), aligned(4)));

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Where each array lives inside the caller's workspace (byte offsets, all 256-byte aligned).
struct Layout {
  int64_t R, K, G, Rb, W;  // G = K/M groups per row, Rb = R/V block rows, W = ceil(G/8) meta words per row
  int64_t steps;           // k-steps = ceil(G/8)
  int vt;                  // 32-row tiles per block row of the PACKED copy (its block height / 32)
  int64_t Rbp;             // block rows of the packed copy: R / (32 * vt).  Its block height is V, except at
                           // M = 4, where every block selects all four columns, V plays no role in the arrays,
                           // and the copy is packed 128 rows high whenever R allows
  int64_t rec_bytes;       // bytes of one (block row, k-step) record of the packed A stream
  bool packed;             // the kernel's packed copies exist (block height 32, 64, 96 or 128)
  size_t off_values, off_columns, off_meta;      // canonical
  size_t off_arec, off_rowidx;                   // packed for the kernel
  size_t off_status;                             // 8-byte legality word
  size_t total;
};

Layout make_layout(int64_t R, int64_t K, int V, int M);

}  // namespace venom

struct venom_handle {
  int64_t R, K;
  int V, N, M;
  venom::Layout lay;
  char* ws;  // borrowed device pointer
};

namespace venom {

// ---- format kernels (venom_format.hip)
// The legality word: ~key of the first violation, 0 if there is none.  Without a slot it is the workspace's, for the host
// to fetch.  With one (below kLegalitySlots, one call at a time) the library's: `found`, a word of host memory that holds 0,
// is non-zero after a violation, and then launch_take_violation brings the word to the host and clears it.
constexpr int kLegalitySlots = 64;
hipError_t launch_compress(const uint16_t* A, int64_t lda, const uint8_t* mask, int64_t ldm, const venom_handle& h,
                           hipStream_t st, int slot = -1, unsigned long long* found = nullptr);
// checks, copies and packs canonical arrays; the word says whether everything was well formed, not what was not
hipError_t launch_import(const uint16_t* values, const uint16_t* columns, const uint32_t* meta, const venom_handle& h,
                         hipStream_t st, int slot = -1, unsigned long long* found = nullptr);
hipError_t launch_take_violation(int slot, unsigned long long* to, hipStream_t st);
hipError_t launch_decompress(const venom_handle& h, uint16_t* A, int64_t lda, hipStream_t st);
// copies the canonical arrays (null: not that one) to memory of the handle's device, at any address
hipError_t launch_export(const venom_handle& h, void* values, void* columns, void* meta, hipStream_t st);

// ---- pruning (venom_prune.hip)
hipError_t launch_prune(const uint16_t* A, int64_t lda, int64_t R, int64_t K, int V, int M, uint8_t* mask, int64_t ldm,
                        unsigned long long* kept_mass, unsigned long long* total_mass, hipStream_t st);

// ---- product kernels (venom_spmm.hip)
int spmm_variant_count();
const char* spmm_variant_name(int v);
// returns VENOM_OK / VENOM_ERR_UNSUPPORTED / VENOM_ERR_HIP
// tokens_major != 0: C is written transposed (C[column][row], leading dimension ldc counts rows of A)
venom_status_t launch_spmm(const venom_handle& h, const void* B, int64_t ldb, int64_t Ccols, const void* bias, int act,
                           void* C, int64_t ldc, int c_dtype, int tokens_major, int variant, hipStream_t st);
// Compute units of the current device, 0 if they cannot be found out.
int compute_units();
// The same for at most 32 columns (venom_skinny.hip), where skinny_product or skinny_layer gives a form for it (else -1): a workgroup
// takes a block row (products), one 32-row tile of it, or two block rows (layers that read X in place).
enum SkinnyForm { kWhole, kSplit, kPair };
int skinny_product(const venom_handle& h, int64_t ld, int64_t cols, int cus);
int skinny_layer(const venom_handle& h, const void* X, int64_t ldx, int64_t tokens, const void* Y, int64_t ldy, int dtype, int cus);
// in_place: src is X, tokens x K, else B; token_major: as above
venom_status_t launch_skinny(const venom_handle& h, int form, const void* src, int64_t ld, int64_t cols, const void* bias, int act,
                             void* out, int64_t ldo, int dtype, bool in_place, bool token_major, hipStream_t st);
// register-only loop of 2:4 matrix instructions, for the measured instruction peak (grid = one workgroup of 8 waves per
// compute unit x 2)
hipError_t launch_smfmac_probe(int iters, float* sink, hipStream_t st);
// out_bytes: of the layer's output, which follows
hipError_t launch_transpose_tokens(const uint16_t* X, int64_t ldx, int64_t tokens, int64_t K, uint16_t* BT, int64_t ldbt,
                                   int64_t out_bytes, hipStream_t st);

}  // namespace venom
