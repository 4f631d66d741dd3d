// The format and pruning kernels and their launch code, compiled for the CPU, behind C entries.
#include "hip/hip_runtime.h"

namespace venom {
// dynamic LDS of the kernels (64 KB per workgroup)
__attribute__((aligned(16))) thread_local uint8_t bits[64 * 1024];
__attribute__((aligned(16))) thread_local char tile[64 * 1024];
}  // namespace venom

#include "venom_format.hip"
#include "venom_prune.hip"

static venom_handle handle(int64_t R, int64_t K, int V, int M, void* ws) {
  return {R, K, V, 2, M, venom::make_layout(R, K, V, M), static_cast<char*>(ws)};
}

extern "C" {
void host_dry_run(int on) { emu::dry_run = on != 0; emu::launches = emu::blocks = 0; }
uint64_t host_launches(void) { return emu::launches; }
uint64_t host_blocks(void) { return emu::blocks; }
size_t host_workspace_bytes(int64_t R, int64_t K, int V, int M) { return venom::make_layout(R, K, V, M).total; }
// each returns the launch's status; `legal` receives the key of the first violation, ~0 if there is none
int host_compress(const uint16_t* A, int64_t lda, const uint8_t* mask, int64_t ldm, int64_t R, int64_t K, int V, int M,
                  void* ws, uint64_t* legal) {
  const venom_handle h = handle(R, K, V, M, ws);
  const int e = venom::launch_compress(A, lda, mask, ldm, h, nullptr);
  if (!emu::dry_run) *legal = ~*reinterpret_cast<uint64_t*>(h.ws + h.lay.off_status);
  return e;
}
int host_import(const uint16_t* values, const uint16_t* columns, const uint32_t* meta, int64_t R, int64_t K, int V, int M,
                void* ws, uint64_t* legal) {
  const venom_handle h = handle(R, K, V, M, ws);
  const int e = venom::launch_import(values, columns, meta, h, nullptr);
  if (!emu::dry_run) *legal = ~*reinterpret_cast<uint64_t*>(h.ws + h.lay.off_status);
  return e;
}
// the same with a legality slot: `found` as the kernels leave it, `legal` as taken from the slot, and taken once more
int host_compress_with_slot(const uint16_t* A, int64_t lda, const uint8_t* mask, int64_t ldm, int64_t R, int64_t K, int V,
                            int M, void* ws, int slot, unsigned long long* found, unsigned long long* legal) {
  const int e = venom::launch_compress(A, lda, mask, ldm, handle(R, K, V, M, ws), nullptr, slot, found);
  for (int k = 0; k < 2; ++k) {
    venom::launch_take_violation(slot, legal + k, nullptr);
    legal[k] = ~legal[k];
  }
  return e;
}
int host_import_with_slot(const uint16_t* values, const uint16_t* columns, const uint32_t* meta, int64_t R, int64_t K, int V,
                          int M, void* ws, int slot, unsigned long long* found, unsigned long long* legal) {
  const int e = venom::launch_import(values, columns, meta, handle(R, K, V, M, ws), nullptr, slot, found);
  for (int k = 0; k < 2; ++k) {
    venom::launch_take_violation(slot, legal + k, nullptr);
    legal[k] = ~legal[k];
  }
  return e;
}
void host_export(int64_t R, int64_t K, int V, int M, const char* ws, uint16_t* values, uint16_t* columns, uint32_t* meta) {
  const venom::Layout L = venom::make_layout(R, K, V, M);
  __builtin_memcpy(values, ws + L.off_values, (size_t)R * L.G * 4);
  __builtin_memcpy(columns, ws + L.off_columns, (size_t)L.Rb * L.G * 8);
  __builtin_memcpy(meta, ws + L.off_meta, (size_t)R * L.W * 4);
}
int host_decompress(int64_t R, int64_t K, int V, int M, void* ws, uint16_t* A, int64_t lda) {
  return venom::launch_decompress(handle(R, K, V, M, ws), A, lda, nullptr);
}
int host_prune(const uint16_t* A, int64_t lda, int64_t R, int64_t K, int V, int M, uint8_t* mask, int64_t ldm,
               uint64_t* kept, uint64_t* total) {
  return venom::launch_prune(A, lda, R, K, V, M, mask, ldm, reinterpret_cast<unsigned long long*>(kept),
                             reinterpret_cast<unsigned long long*>(total), nullptr);
}
}
