// The product kernel: C = A . B with A in V:N:M form (paper section 4: stage 1 loads column-loc,
// the gathered rows of B and the A tile; stage 2 runs the 2:4 matrix instruction; stage 3 stores
// the output through on-chip memory).  Written for gfx950:
//   * the 2:4 inner pattern maps onto v_smfmac_f32_32x32x32_f16: A operand = 8 kept halfs per lane
//     (row = lane%32, four groups), 16 index bits per lane (= four canonical nibbles), B operand =
//     16 halfs per lane (column = lane%32, four groups x the 4 selected rows);
//   * a workgroup owns V x (64*NC) blocks of C (BS_r = V as in the paper, so every gathered row of
//     B serves all V rows); a k-step is 8 groups = 32 gathered rows of B;
//   * the workgroup is split by role.  NC CONSUMER waves each own a 64-column strip (on the 64-column
//     tile two or three waves share the one strip, a part of its rows each): they only read
//     LDS (transposing reads ds_read_b64_tr_b16 build the B operand, plain reads fetch the packed
//     values and index words) and issue matrix instructions.  Four PRODUCER waves, one per SIMD,
//     only move data, by direct-to-LDS loads.  A SIMD issues one wave-wide 16-byte load (1 KB) per
//     ~69 cycles whatever the rest of the compute unit does (measured), so the loads of a k-step --
//     the gathered rows of B, the packed A record, the row ids -- are dealt round-robin over the
//     four producers: every SIMD's share of the vector-memory issue rate is used;
//   * the loads are issued from inline assembly and retired with exact `s_waitcnt vmcnt(n)` counts
//     (loads retire in order per wave); one s_barrier per k-step hands filled stages to the
//     consumers and drained ones back;
//   * the consumers run one k-step behind the loads and refill each operand register from the new
//     stage right after its last use, so no LDS latency sits between two barriers;
//   * workgroups are persistent (one per compute unit): the k-steps of all tiles of a workgroup
//     form one sequence, so the load pipeline runs on across tile boundaries while the consumers
//     store their output;
//   * each XCD (one L2 each) walks a contiguous range of the column-tile-major tile list, so its
//     workgroups share the gathered rows of one slab of B through that L2.
#include <atomic>
#include <type_traits>

#include "venom_device.h"

namespace venom {

struct SpmmParams {
  const char* arec;        // packed A stream, one record per (block row, k-step)
  const int32_t* rowidx;   // absolute B row of every gathered row, [block row][k-step][32]
  const char* B;           // fp16, row-major
  void* C;
  int64_t ldb_bytes, ldc, Ccols, rec_bytes;
  int steps;
  int nbr, nct;            // block rows, column tiles
  int cgroup;              // the tile list goes through groups of this many column tiles, block row by block row
  int per_xcd;             // ceil(nbr*nct / 8)
  int stream_out;          // nonzero: non-temporal stores of C
  int serpentine;          // nonzero: a workgroup's odd tiles run their k-steps backwards, so the end of the
                           // slab of B that the last tile left in L2 is where the next one starts
  int pad_row0;            // first gathered row of a tile's LAST k-step that lies past the end of K (32: none)
  const _Float16* bias;    // one entry per row of C, or null
  int act;                 // venom_activation_t
};

constexpr int kNumXcd = 8;
constexpr int kProducers = 4;        // producer waves per workgroup: one per SIMD
constexpr int kRidSlots = 16;        // row-id ring: 128 bytes per k-step

// ---- direct-to-LDS loads and their retirement, outside the compiler's wait-count bookkeeping.
// LDS destination of lane l is lds_addr + l*16; M0 carries lds_addr and needs one wait state
// before the load reads it.
// The global address is a wave-uniform 64-bit base (SGPR pair) plus an unsigned 32-bit byte offset
// per lane, so address generation costs one vector instruction per load.
__device__ __forceinline__ void dma16(const char* base, uint32_t lane_off, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_off), "s"(base), "s"(lds_addr)
               : "memory");
}
__device__ __forceinline__ void dma4(const char* base, uint32_t lane_off, uint32_t lds_addr) {  // lane l -> lds_addr + 4*l
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(lane_off), "s"(base), "s"(lds_addr)
               : "memory");
}
// wait until at most n of this wave's loads are outstanding, 0 <= n <= MAXN.  The count is an immediate
// of the instruction, hence the cascade.
template <int MAXN>
__device__ __forceinline__ void wait_loads(int n) {
  static_assert(MAXN <= 63, "vmcnt is a 6-bit counter");
  if (n >= MAXN) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(MAXN) : "memory");
  else if constexpr (MAXN > 0) wait_loads<MAXN - 1>(n);
}
__device__ __forceinline__ void barrier_only() { asm volatile("s_barrier" ::: "memory"); }
// the same once every LDS access of this wave has completed
__device__ __forceinline__ void lgkm_drained_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// 16-byte slot swizzle of gathered row rho inside its LDS row.  The four rows a lane block reads at
// once lie ROW_BYTES apart; a row of 128 bytes is half the banks, so there only every second row has
// to move (and a row has 8 slots, not 16 or more).
template <int ROW_BYTES>
__device__ __forceinline__ int slot_swizzle(int rho) {
  return ROW_BYTES == 128 ? 4 * ((rho >> 1) & 1) : 4 * (rho & 3);
}

// This workgroup's share of the tile list.  The grid holds one workgroup per compute unit (the
// host sizes it) and every workgroup walks several tiles: starting a wide workgroup that owns most
// of the LDS costs microseconds, and a persistent one can keep its load pipeline full across tile
// boundaries.  Consecutive workgroup ids land on different XCDs; each XCD takes a contiguous
// range of the column-tile-major list, so the workgroups of one XCD sweep the same slab of B and
// a gathered row is fetched from beyond the L2 once for the workgroups that reach it while it is
// resident (measured: all of them while the workgroups run in lock-step, fewer once they drift).
struct TileWalk {
  int base, first, stride, count;
  __device__ __forceinline__ void locate(const SpmmParams& p, int t, int& ct, int& br) const {
    const int work = base + first + t * stride;
    const int group = work / (p.nbr * p.cgroup), rest = work - group * (p.nbr * p.cgroup);
    if (p.cgroup == 1) { ct = group; br = rest; return; }
    const int left = p.nct - group * p.cgroup, width = left < p.cgroup ? left : p.cgroup;   // (the last group may be narrower)
    br = rest / width;
    ct = group * p.cgroup + rest - br * width;
  }
};

// MODE 0: the plain product; 1: fused bias / activation; 2: the same with C written transposed
// (token-major), straight from the accumulators; 3: token-major fp16 through LDS with 16-byte
// stores (needs the output and its leading dimension 16-byte aligned).  Separate instantiations:
// the plain kernel carries none of the epilogue code, and one kernel holding both token-major
// paths behind a run-time branch does not compile (the compiler then keeps the producers' scalar
// operands in vector registers).
// KS: k-steps of a stage, which one barrier hands over (1 or 2); NS: stages of the B ring; NA: stages of records in the A ring.
// D: barriers after which a consumed stage returns to the producers.  The consumers read stage g
// between barriers g and g+1 but use what they read only after barrier g+1.  D = 2: they do not
// wait for those reads before barrier g+1, so the stage stays theirs until barrier g+2 and the
// loads run NS-2 k-steps ahead.  D = 1: they drain their reads before every barrier and the loads
// run NS-1 k-steps ahead.
// NR: consumer waves that share a 64-column strip, each owning VT/NR of its tile rows.  1 for the wide
// tiles.  The 64-column tile has a single strip: one wave would need 8 matrix instructions (256
// cycles) per k-step while its 8.5 KB arrive in ~190, so the strip's rows are split over two or three waves.
//
// Waves per SIMD that the registers are kept low enough for: four where a workgroup has at most eight waves with at most 64
// accumulators each (two 32-row tiles), five for ten waves of 32, so that two workgroups share a unit if their LDS
// allows it; three for the others.
constexpr int simd_waves(int VT, int NC, int NR) {
  return VT / NR == 1 && NC * NR == 6 ? 5 : VT / NR <= 2 && NC * NR <= 4 ? 4 : 3;
}

template <int VT, int NC, int NR, int KS, int NS, int NA, int D, bool OUT_F32, int MODE>
__global__ void __launch_bounds__((NC * NR + kProducers) * 64, simd_waves(VT, NC, NR)) spmm_kernel(SpmmParams p) {
  static_assert(NC == 1 || NC == 2 || NC == 4 || NC == 8, "64-column strips per workgroup");
  static_assert(VT % NR == 0, "the tile rows divide evenly over the waves of a strip");
  static_assert(D == 1 || D == 2, "barriers between the hand-over of a stage and its return");
  constexpr bool EPI = MODE != 0;
  constexpr int FENCE = MODE == 1 && NC * NR <= 4 ? 4 : 2;   // activations evaluated together (3072 x 768 x 4096 at
                                                   // 64:2:8 with GELU 19.3 -> 18.6 us with four; no registers for that elsewhere)
  static_assert(VT >= 1 && VT <= kMaxTiles, "32-row tiles per block row");
  constexpr int NP = kProducers;
  constexpr int CONS = NC * NR;                    // consumer waves
  constexpr int RT = VT / NR;                      // 32-row tiles a consumer wave accumulates
  constexpr int CT = 2;                            // 32-column tiles a consumer wave accumulates
  constexpr int WCOLS = 32 * CT;                   // columns of C per consumer wave
  constexpr int BSC = WCOLS * NC;                  // columns of C per workgroup
  constexpr int ROW_BYTES = 2 * BSC;               // one gathered row of B in LDS
  constexpr int RPI = 1024 / ROW_BYTES;            // rows written by one wave-wide 16-byte load
  constexpr int LPR = 64 / RPI;                    // lanes (= 16-byte slots) per row
  constexpr int SROWS = KS * kStepRows;            // gathered rows of B in a stage of KS k-steps
  constexpr int NI = SROWS / RPI;                  // B loads per stage (4 * NC a k-step)
  constexpr int CB = NI / NP;                      // ... per producer
  static_assert(NI % NP == 0, "the B loads of a k-step divide evenly over the producers");
  constexpr int STEP_BYTES = kStepRows * ROW_BYTES;
  constexpr int B_BYTES = KS * STEP_BYTES;
  constexpr int REC = VT * kTileValBytes + kTailBytes;       // one A record
  constexpr int T_OFF = VT * kTileValBytes;        // record tail: index words
  constexpr int ARING = NS * B_BYTES;              // LDS: [B ring][A ring][row-id ring]
  constexpr int RIDRING = ARING + NA * KS * REC;
  constexpr int RID_BYTES = SROWS * 4;             // row ids of a stage
  constexpr int NJ = VT + 1;                       // A loads per k-step: VT value blocks + the tail
  constexpr int PB = NS - D;                       // k-steps the B stream runs ahead
  constexpr int PA = NA - D;                       // k-steps the A stream runs ahead
  constexpr int RA = 2 * PB + 2 > PA ? 2 * PB + 2 : PA;   // k-steps the row-id stream runs ahead: the ids of step g+PB+1
                                                   // are then older, in their producer's load queue, than its loads
                                                   // of step g, and the stream ends no later than the records
  static_assert(PB >= 1 && PA >= PB, "a record is issued no later than the B rows of its k-step");
  static_assert(kRidSlots >= PB + 2, "a row-id slot is rewritten only after its last reader");
  static_assert(RA <= kRidSlots, "the row ids of the start-up fit the ring");
  constexpr bool OWN_STG = NR > 1;                 // the consumers' output staging: the drained stage, or its own LDS
  constexpr int STG = RIDRING + kRidSlots * RID_BYTES;
  static_assert(OWN_STG || CONS * 32 * WCOLS * 2 <= B_BYTES, "the output staging of all consumers fits one B stage");

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(LDS_PTR(char))smem;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  TileWalk tw;
  {
    const int xcd = blockIdx.x % kNumXcd;
    tw.base = xcd * p.per_xcd;
    tw.first = blockIdx.x / kNumXcd;
    tw.stride = gridDim.x / kNumXcd;
    int lim = p.nbr * p.nct - tw.base;
    if (lim > p.per_xcd) lim = p.per_xcd;
    tw.count = lim > tw.first ? (lim - tw.first + tw.stride - 1) / tw.stride : 0;
  }
  if (tw.count == 0) return;                       // the whole workgroup leaves together
  // All k-steps of all tiles of this workgroup form one sequence g = 0 .. G-1; the rings and the
  // barriers are indexed by g, so the loads of the next tile start while this one is finishing.
  // Barriers, in order: one before the first step (the first row ids are on chip), one per step
  // ("step g is complete in LDS, step g-D is consumed"), and one more after the last step of each
  // tile, after which the consumers stage their output in the B stage they have just drained.
  // (KS = 2: "step" in the following is a stage of two k-steps, which one barrier hands over; the last stage of a tile
  // has one where the k-steps are odd, `odd`, and its second half holds copies that nobody multiplies)
  const int S = KS == 1 ? p.steps : (p.steps + 1) / 2;
  const bool odd = KS == 2 && (p.steps & 1);
  const int G = tw.count * S;

  if (wave >= CONS) {
    // ========================================================================= producers
    // Iteration i (after barrier i) issues, in this order: the row ids of step i+RA, this
    // producer's part of record i+PA, its part of the B rows of step i+PB.  Before barrier g the
    // producer needs its loads of step g and of record g landed (and the row ids of step g+PB):
    // all of them are at least as old as its B loads of step g, so it waits until only the loads
    // of the PB-1 iterations issued since then are outstanding.
    __builtin_amdgcn_s_setprio(3);                 // their few instructions go ahead of the consumers'
    auto produce = [&](auto pj_const) {
      constexpr int PJ = decltype(pj_const)::value;
      constexpr int CA = PJ < KS * NJ ? (KS * NJ - PJ + NP - 1) / NP : 0;   // A loads per stage: loads PJ, PJ+NP, ...
      constexpr int CR = PJ == NP - 1 ? 1 : 0;                    // the row ids travel with the last producer
      constexpr int L = CA + CR + CB;
      static_assert((PB - 1) * L <= 63, "load counts fit the 6-bit counter");
      // A producer is never ahead of the barrier it is about to meet: every instruction of its loop
      // body lengthens the k-step (a wave issues nothing else while the address unit takes one of
      // its loads, ~70 cycles, and instructions between two loads are not hidden behind them:
      // measured).  So the streams advance by plain increments, ring positions wrap by compare and
      // select, and everything that depends on the tile is recomputed in a branch taken once per tile.
      // For the same reason the loop that runs most k-steps (`runs` below) is taken without a branch between its
      // loads: it covers the iterations in which no stream comes to the end of its tile.  A k-step of a 64-column
      // tile takes 0.12 us in it (one tile alone on the chip, operands in L2) and 0.20 us in a loop that tests
      // the four streams each time round.
      const uint32_t lane_off = lane * 16;
      using checked = std::false_type;             // tags of the streams' steps: the tile may end with it / it does not
      using inside = std::true_type;
      int ct, br;
      // ---- record stream: record pointer, LDS slot address, k-steps left in its tile
      tw.locate(p, 0, ct, br);
      const char* a_ptr = p.arec + (int64_t)br * p.steps * p.rec_bytes;
      int64_t a_inc = KS * p.rec_bytes;
      bool a_back = false;
      uint32_t a_lds = lds0 + ARING;
      int a_left = S, a_t = 0;
      auto next_record = [&](auto inside_tile) {
        const bool single = !decltype(inside_tile)::value && odd && a_left == (a_back ? S : 1);   // a stage of one k-step
        const char* second = single ? a_ptr : a_ptr + p.rec_bytes;
#pragma unroll
        for (int l = PJ; l < KS * NJ; l += NP) {
          const int a = l % NJ;
          const char* rec = l < NJ ? a_ptr : second;
          const uint32_t to = a_lds + l / NJ * REC;
          if (a < VT) dma16(rec + a * 1024, lane_off, to + a * 1024);
          else if (lane < kTailBytes / 16) dma16(rec + T_OFF, lane_off, to + T_OFF);   // the 512-byte tail: half a wave
        }
        a_ptr += a_inc;
        a_lds = a_lds + KS * REC == lds0 + ARING + NA * KS * REC ? lds0 + ARING : a_lds + KS * REC;
        if constexpr (decltype(inside_tile)::value) return;
        if (--a_left == 0) {
          a_left = S;
          if (++a_t < tw.count) {
            tw.locate(p, a_t, ct, br);
            const bool back = p.serpentine && (a_t & 1);       // odd tiles run their k-steps backwards
            a_back = back;
            a_inc = back ? -KS * p.rec_bytes : KS * p.rec_bytes;
            a_ptr = p.arec + ((int64_t)br * p.steps + (back ? (S - 1) * KS : 0)) * p.rec_bytes;
          }
        }
      };
      // ---- row-id stream (producer NP-1 only)
      const char* r_ptr = reinterpret_cast<const char*>(p.rowidx) + (int64_t)br * p.steps * (kStepRows * 4);
      int r_inc = RID_BYTES;
      uint32_t r_lds = lds0 + RIDRING;
      int r_left = S, r_t = 0;
      auto end_of_rowids = [&]() {                 // the stream has come to the end of its tile
        r_left = S;
        if (++r_t < tw.count) {
          int ct2, br2;
          tw.locate(p, r_t, ct2, br2);
          const bool back = p.serpentine && (r_t & 1);
          r_inc = back ? -RID_BYTES : RID_BYTES;
          r_ptr = reinterpret_cast<const char*>(p.rowidx) +
                  ((int64_t)br2 * p.steps + (back ? (S - 1) * KS : 0)) * (kStepRows * 4);
        } else {                                   // past the last one it stays on its last k-step: ids nobody reads,
          r_ptr -= r_inc;                          // so that an iteration has the same loads while records are left
          r_inc = 0;
        }
      };
      auto next_rowids = [&](auto inside_tile) {
        // (a stage of one k-step fetches 128 bytes past it, too: other ids or, after the last, what follows them in the workspace)
        if (lane < SROWS) dma4(r_ptr, lane * 4, r_lds);
        r_ptr += r_inc;
        r_lds = r_lds + RID_BYTES == lds0 + RIDRING + kRidSlots * RID_BYTES ? lds0 + RIDRING : r_lds + RID_BYTES;
        if constexpr (decltype(inside_tile)::value) return;
        if (--r_left == 0) end_of_rowids();
      };
      // ---- B stream.  Load q of this producer is load number PJ + NP*q of the k-step; it covers
      // rows (that number)*RPI .. +RPI-1; lane l writes 16-byte slot l%LPR of row l/LPR and fetches
      // the XOR-swizzled chunk of the gathered row.  A lane reads the id of its row from the row-id
      // ring (one LDS read per load, all of them before the record loads so that their latency is
      // covered) and forms the byte offset with one multiply-add (the host checks the 24-bit ranges).
      int chunk_col[CB];                           // first column of this lane's chunk inside the tile
#pragma unroll
      for (int q = 0; q < CB; ++q) {
        const int rho = (PJ + NP * q) * RPI + lane / LPR;
        chunk_col[q] = ((lane % LPR) ^ slot_swizzle<ROW_BYTES>(rho)) * 8;
      }
      uint32_t ld_col[CB];
      auto set_tile = [&](int t) {
        int ct3, br3;
        tw.locate(p, t, ct3, br3);
#pragma unroll
        for (int q = 0; q < CB; ++q) {
          int64_t col = (int64_t)ct3 * BSC + chunk_col[q];
          if (col + 8 > p.Ccols) col = p.Ccols - 8;  // past the edge: any in-bounds data, never stored
          ld_col[q] = (uint32_t)(col * 2);
        }
      };
      const int rowsel = lane / LPR;               // which of the RPI rows of a load this lane writes
      const uint32_t ldb24 = (uint32_t)p.ldb_bytes;
      uint32_t b_lds = lds0 + PJ * 1024;           // this producer's first row in the stage it fills next
      const char* rid_rd = smem + RIDRING + rowsel * 4;   // this lane's entry of the ring slot it reads next
      int b_left = S, b_t = 0;
      set_tile(0);
      int rid[CB];
      auto read_rowids = [&](auto inside_tile) {
        // (a stage of one k-step: its rows once more)
        const bool single = !decltype(inside_tile)::value && odd && b_left == ((p.serpentine && (b_t & 1)) ? S : 1);
        const int again = single ? kStepRows * 4 : 0;
#pragma unroll
        for (int q = 0; q < CB; ++q)
          rid[q] = *reinterpret_cast<const int*>(rid_rd + (PJ + NP * q) * RPI * 4 - (q >= CB / KS ? again : 0));
        rid_rd = rid_rd + RID_BYTES == smem + RIDRING + rowsel * 4 + kRidSlots * RID_BYTES
                     ? smem + RIDRING + rowsel * 4 : rid_rd + RID_BYTES;
      };
      auto next_rows = [&](auto inside_tile) {
        uint32_t off[CB];
#pragma unroll
        for (int q = 0; q < CB; ++q)   // row id x bytes per row + this lane's column bytes, one instruction
          asm("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(off[q]) : "v"(rid[q]), "s"(ldb24), "v"(ld_col[q]));
#pragma unroll
        for (int q = 0; q < CB; ++q) dma16(p.B, off[q], b_lds + q * (NP * 1024));
        b_lds = b_lds + B_BYTES == lds0 + PJ * 1024 + NS * B_BYTES ? lds0 + PJ * 1024 : b_lds + B_BYTES;
        if constexpr (decltype(inside_tile)::value) return;
        if (--b_left == 0) {
          b_left = S;
          if (++b_t < tw.count) set_tile(b_t);
        }
      };
      // start-up: the row ids of the first RA steps, then what iterations -PA .. -1 would have issued
      // (the records that run ahead of the rows do not wait for the ids)
      auto first_records = [&]() {
        for (int i = -PA; i < -PB; ++i)
          if (i + PA < G) next_record(checked{});
      };
      if constexpr (CR != 0) {
        const int n0 = S < RA ? S : RA, k0 = p.steps < KS * RA ? p.steps : KS * RA;   // those of the first tile: eight k-steps a load
#pragma unroll
        for (int q = 0; 8 * q < KS * RA; ++q) {
          const int s = 8 * q + lane / 8;
          if (s < k0) dma16(r_ptr, s * (kStepRows * 4) + lane % 8 * 16, r_lds + q * 1024);
        }
        r_ptr += n0 * RID_BYTES;
        r_lds = n0 == kRidSlots ? r_lds : r_lds + n0 * RID_BYTES;
        r_left -= n0;
        if (r_left == 0) end_of_rowids();
        for (int j = n0; j < RA && j < G; ++j) next_rowids(checked{});
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      } else first_records();
      barrier_only();                              // the first row ids are on chip
      if constexpr (CR != 0) first_records();
      for (int i = -PB; i < 0; ++i) {
        if (i + PA < G) next_record(checked{});
        if (i + PB < G) { read_rowids(checked{}); next_rows(checked{}); }
      }
      const bool ragged = p.pad_row0 < kStepRows;  // K/M is not a multiple of 8
      int c_left = S, c_t = 0;               // k-steps left in the tile the consumers are on / that tile
      // One iteration: the loads of step g have landed, barrier, the next loads.  RECORDS, ROWS: these
      // streams are still inside the sequence.  `waited` waits for the loads of step g.
      auto iteration = [&](int g, auto records, auto rows, auto waited) {
        waited();
        if (ragged && c_left == ((p.serpentine && (c_t & 1)) ? S : 1)) {
          // The last k-step of a tile when K/M is not a multiple of 8: its trailing groups do not
          // exist.  Their values are zero, but 0 x Inf is not, so the rows gathered for them (row 0
          // of B, a valid address that keeps the load count exact) are overwritten with zeros once
          // they have landed; every producer cleans the rows it loaded itself.
          char* stage = smem + (g % NS) * B_BYTES;
#pragma unroll
          for (int q = 0; q < CB; ++q)             // (the rows of the last k-step: the second of its stage, or the first and only)
            if ((PJ + NP * q) * RPI + rowsel >= p.pad_row0 + (KS == 2 && !odd ? kStepRows : 0))
              *reinterpret_cast<uint4*>(stage + (PJ + NP * q) * 1024 + lane * 16) = make_uint4(0, 0, 0, 0);
          lgkm_drained_barrier();
        } else barrier_only();
        // after barrier g the consumers are done with stage g-D and record g-D
        if constexpr (decltype(rows)::value) read_rowids(checked{});
        if constexpr (decltype(records)::value) {
          if constexpr (CR != 0) next_rowids(checked{});
          next_record(checked{});
        }
        if constexpr (decltype(rows)::value) next_rows(checked{});
        if (--c_left == 0) { c_left = S; ++c_t; barrier_only(); }
      };
      // How many iterations from the next on, at most n, do not end a tile of any of the streams
      // (the first k-step of a tile, where the ragged end of a backward tile lies, is left to the checked one).
      const bool any_runs = S > 4;           // (shorter tiles end a stream in all of them)
      auto runs = [&](int n, bool records) {
        if (!any_runs) return 0;
        if (odd && (b_left == S || (records && a_left == S))) return 0;   // (the first stage of a backward tile has one k-step)
        n = n < b_left - 1 ? n : b_left - 1;
        n = n < c_left - 1 ? n : c_left - 1;
        if (records) {
          n = n < a_left - 1 ? n : a_left - 1;
          if constexpr (CR != 0) n = n < r_left - 1 ? n : r_left - 1;
        }
        return ragged && c_left == S ? 0 : n;
      };
      // The loads of step g are those of iteration g-PB: step g is there when only those of the PB-1
      // iterations since are outstanding.  While records are left these are L each (the start-up
      // issued no row ids beside the first records and rows), after that at least CB.
      int g = 0;
      while (g + PA < G) {
        iteration(g, std::true_type{}, std::true_type{}, [&]() {
          if (CR != 0 && g < PB - 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((PB - 1) * (CA + CB)) : "memory");
          else asm volatile("s_waitcnt vmcnt(%0)" ::"n"((PB - 1) * L) : "memory");
        });
        ++g;
        if (g < PB - 1) continue;
        int n = runs(G - PA - g, true);
        if (n <= 0) continue;
        g += n; a_left -= n; b_left -= n; c_left -= n;
        if constexpr (CR != 0) r_left -= n;
        do {
          asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((PB - 1) * L) : "memory");
          read_rowids(inside{});
          if constexpr (CR != 0) next_rowids(inside{});
          next_record(inside{});
          next_rows(inside{});
        } while (--n > 0);
      }
      while (g + PB < G) {
        iteration(g, std::false_type{}, std::true_type{},
                  []() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"((PB - 1) * CB) : "memory"); });
        ++g;
        int n = runs(G - PB - g, false);
        if (n <= 0) continue;
        g += n; b_left -= n; c_left -= n;
        do {
          asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((PB - 1) * CB) : "memory");
          read_rowids(inside{});
          next_rows(inside{});
        } while (--n > 0);
      }
      for (; g < G; ++g)
        iteration(g, std::false_type{}, std::false_type{}, [&]() { wait_loads<(PB - 1) * CB>((G - 1 - g) * CB); });
    };
    switch (wave - CONS) {
      case 0: produce(std::integral_constant<int, 0>{}); break;
      case 1: produce(std::integral_constant<int, 1>{}); break;
      case 2: produce(std::integral_constant<int, 2>{}); break;
      default: produce(std::integral_constant<int, 3>{}); break;
    }
  } else {
    // ========================================================================= consumers
    // Transposing LDS reads that build the B operand.  Sub-read cb of a 32-column tile: lane block
    // blk = lane/16 reads group t = 4*(cb/2) + 2*(blk/2) + cb%2, 16-column window 2*tile + blk%2;
    // inside the block lane i reads row 4*t + i/4, 8-byte piece i%4.
    const int wc = NR == 1 ? wave : wave % NC;     // this wave's strip
    const int wr = NR == 1 ? 0 : wave / NC;        // ... and its share of the strip's tile rows
    int rd_off[CT][4];
    {
      const int blk = lane >> 4, i = lane & 15, e = i >> 2, c8 = i & 3;
#pragma unroll
      for (int tc = 0; tc < CT; ++tc)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
          const int t = 4 * (cb >> 1) + 2 * (blk >> 1) + (cb & 1);
          const int rho = 4 * t + e;
          const int win = (wc * CT + tc) * 2 + (blk & 1);
          const int slot = (2 * win + (c8 >> 1)) ^ slot_swizzle<ROW_BYTES>(rho);
          rd_off[tc][cb] = rho * ROW_BYTES + slot * 16 + (c8 & 1) * 8;
        }
    }
    floatx16 acc[RT][CT];
    half16 bf[CT];                                 // the wave's two 32-column B operands of one k-step
    uint32_t ixw[2];                               // index words of tile rows (0,1) and (2,3): 2 x 16 bits each
    half8 av[RT];                                  // the A operands of one k-step
    auto read_a = [&](const char* sa, int t) {
      av[t] = *reinterpret_cast<const half8*>(sa + (wr * RT + t) * kTileValBytes + lane * 16);
    };
    auto read_b = [&](const char* sb, int tc) {
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        const short4v piece = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(short4v))(sb + rd_off[tc][cb]));
        const half4 ph = __builtin_bit_cast(half4, piece);
        bf[tc][4 * cb + 0] = ph[0]; bf[tc][4 * cb + 1] = ph[1]; bf[tc][4 * cb + 2] = ph[2]; bf[tc][4 * cb + 3] = ph[3];
      }
    };
    auto read_ix = [&](const char* sa, int half) {
      if constexpr (NR > 1 && RT == 1) ixw[0] = *reinterpret_cast<const uint16_t*>(sa + T_OFF + lane * 8 + 2 * wr);
      else ixw[half] = *reinterpret_cast<const uint32_t*>(sa + T_OFF + lane * 8 + 4 * (wr * (RT / 2) + half));
    };
    auto mma = [&](int t, int tc) {
      const int ix = (int)ixw[t >> 1];
      if (t & 1) acc[t][tc] = smfmac<1>(av[t], bf[tc], acc[t][tc], ix);
      else acc[t][tc] = smfmac<0>(av[t], bf[tc], acc[t][tc], ix);
    };
    // after tile row t of the LAST column pass nothing reads av[t] any more, and an index word is
    // free after the last tile row that uses it
    auto refill_after = [&](const char* sa, int t) {
      read_a(sa, t);
      if ((t & 1) == 1 || t == RT - 1) read_ix(sa, t >> 1);
    };
    // In iteration g (after barrier g: stage g and record g are complete) a wave multiplies step
    // g-1 from registers, one column tile after the other, and refills every operand register from
    // stage g as soon as its last matrix instruction has been issued.
    int b_slot = 0, a_slot = 0;
    barrier_only();                                // (the producers' start-up barrier)
    for (int t = 0; t < tw.count; ++t) {
#pragma unroll
      for (int tr = 0; tr < RT; ++tr)
#pragma unroll
        for (int tc = 0; tc < CT; ++tc)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[tr][tc][v] = 0.f;

      const char* sb = smem;
      const char* sa = smem;
      auto advance = [&]() {
        sb = smem + b_slot * B_BYTES;
        sa = smem + ARING + a_slot * (KS * REC);
        b_slot = (b_slot + 1) % NS;
        a_slot = a_slot + 1 == NA ? 0 : a_slot + 1;
      };
      // first k-step of the tile: only fetch (same order of reads as in the steady state)
      barrier_only();
      advance();
      read_b(sb, 0);
#pragma unroll
      for (int tr = 0; tr < RT; ++tr) refill_after(sa, tr);
      read_b(sb, 1);
      // multiplies a k-step from registers and refills them with the next one, at (nb, na)
      auto k_step = [&](const char* nb, const char* na) {
#pragma unroll
        for (int tc = 0; tc < CT; ++tc) {
#pragma unroll
          for (int tr = 0; tr < RT; ++tr) {
            mma(tr, tc);
            if (tc == CT - 1) refill_after(na, tr);
            __builtin_amdgcn_sched_barrier(0);
          }
          read_b(nb, tc);
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      const bool back = KS == 2 && p.serpentine && (t & 1);
      if (KS == 2 && !(odd && (back || S == 1))) k_step(sb + STEP_BYTES, sa + REC);   // the first stage's second k-step
      for (int s = 1; s < S; ++s) {
        if constexpr (D == 1) lgkm_drained_barrier();   // my reads of the last stage are over; this one is complete
        else barrier_only();                            // stage s and record s are complete
        // (the next matrix instruction may wait for this wave's reads, and the narrow tiles' k-steps are short: they
        // arrive at the barrier first.  On the wide ones it is issued while the wave waits there)
        if constexpr (NC <= 2) __builtin_amdgcn_sched_barrier(0);
        advance();
        k_step(sb, sa);
        if (KS == 2 && !(odd && !back && s == S - 1)) k_step(sb + STEP_BYTES, sa + REC);
      }
#pragma unroll
      for (int tc = 0; tc < CT; ++tc)
#pragma unroll
        for (int tr = 0; tr < RT; ++tr) mma(tr, tc);
      lgkm_drained_barrier();                      // every consumer has drained the last B stage

      // ---- stage 3: registers -> (LDS) -> global.  Accumulator element v of a 32x32 tile sits
      // at row 8*(v/4) + 4*(lane/32) + v%4, column lane%32.
      // everything below is per-tile work: its index arithmetic starts from a lane id computed here,
      // so that none of it is hoisted out of the tile loop into registers the k-loop needs
      int ln;
      asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(ln));
      int ct, br;
      tw.locate(p, t, ct, br);
      const int64_t row0 = ((int64_t)br * VT + wr * RT) * 32;
      const int64_t col0 = (int64_t)ct * BSC + wc * WCOLS;
      // fused epilogue (the layer's bias, one per output row, then the activation), in fp32 on
      // the accumulators, one 32-row tile at a time right before it is stored: a ln holds rows
      // 8j + 4*(ln/32) + 0..3 of the tile
      auto finish = [&](int tr, int tc_lo = 0, int tc_hi = CT) {   // column tiles tc_lo .. tc_hi-1 of tile row tr
        if constexpr (!EPI) return;                // the plain product compiles without any of this
        if (p.bias) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const half4 b4 = *reinterpret_cast<const half4*>(p.bias + row0 + tr * 32 + 8 * j + 4 * (ln >> 5));
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
              for (int tc = tc_lo; tc < tc_hi; ++tc) acc[tr][tc][4 * j + i] += (float)b4[i];
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        // (scheduling fences keep the evaluations from being interleaved by the dozen: their
        // temporaries would push accumulators out of registers, for the whole kernel)
        if (p.act == VENOM_ACT_GELU) {
#pragma unroll
          for (int tc = tc_lo; tc < tc_hi; ++tc)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
              acc[tr][tc][v] = gelu_by_definition<OUT_F32>(acc[tr][tc][v]);
              if (v % FENCE == FENCE - 1) __builtin_amdgcn_sched_barrier(0);
            }
        } else if (p.act == VENOM_ACT_GELU_TANH) {
#pragma unroll
          for (int tc = tc_lo; tc < tc_hi; ++tc)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
              acc[tr][tc][v] = gelu_tanh_form(acc[tr][tc][v]);
              if (v % FENCE == FENCE - 1) __builtin_amdgcn_sched_barrier(0);
            }
        }
      };
      if constexpr (MODE >= 2) {
        // Token-major output Y[token][feature] = C transposed: a lane owns one column of C (a token)
        // and, per 32-row tile, four runs of 4 consecutive rows (features).
        auto direct = [&]() {
          // each run is one 8-byte (fp16) or 16-byte (fp32) store straight from the accumulators;
          // the two half-waves write neighbouring runs
#pragma unroll
          for (int tr = 0; tr < RT; ++tr) {
            finish(tr);
#pragma unroll
            for (int tc = 0; tc < CT; ++tc) {
              const int64_t tok = col0 + tc * 32 + (ln & 31);
              if (tok < p.Ccols) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                  const int64_t feat = row0 + tr * 32 + 8 * q + 4 * (ln >> 5);
                  if constexpr (OUT_F32) {
                    typedef float f32x4 __attribute__((ext_vector_type(4)));
                    const f32x4 o = {acc[tr][tc][4 * q], acc[tr][tc][4 * q + 1], acc[tr][tc][4 * q + 2], acc[tr][tc][4 * q + 3]};
                    *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(p.C) + tok * p.ldc + feat) = o;
                  } else {
                    const half4 o = {(_Float16)acc[tr][tc][4 * q], (_Float16)acc[tr][tc][4 * q + 1],
                                     (_Float16)acc[tr][tc][4 * q + 2], (_Float16)acc[tr][tc][4 * q + 3]};
                    *reinterpret_cast<half4*>(reinterpret_cast<_Float16*>(p.C) + tok * p.ldc + feat) = o;
                  }
                }
              }
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        };
        if constexpr (OUT_F32 || MODE == 2) {
          direct();
        } else {
          // fp16: the 8-byte runs of FT tile rows go through this wave's 4 KB of the drained stage
          // as [token][32*FT features] and leave as 16-byte stores, 64*FT contiguous bytes per
          // token (a full 128-byte line when the block height allows pairs of tile rows).  The
          // 8-byte slots of a staged row are XOR-swizzled by the token so that neighbouring tokens,
          // whose rows lie 64*FT bytes apart, use different banks.
          constexpr int FT = RT % 2 == 0 ? 2 : 1;  // 32-row tiles per pass
          constexpr int RB = 64 * FT;              // bytes of a staged token row
          constexpr int LPT = RB / 16;             // lanes (16-byte chunks) per token row
          constexpr int TPI = 64 / LPT;            // tokens per wave-wide read
          constexpr int SH = FT == 2 ? 1 : 2;      // tokens 2^SH apart share a bank group
          char* stg = (OWN_STG ? smem + STG : const_cast<char*>(sb)) + wave * 4096;
          _Float16* Y = reinterpret_cast<_Float16*>(p.C);
          const int h = ln >> 5;
#pragma unroll
          for (int trg = 0; trg < RT / FT; ++trg) {
#pragma unroll
            for (int ps = 0; ps < FT; ++ps) {      // FT = 2: one column tile per pass; FT = 1: both in one pass
#pragma unroll
              for (int trr = 0; trr < FT; ++trr) {   // the epilogue of exactly what this pass stores
                if constexpr (FT == 2) finish(trg * FT + trr, ps, ps + 1);
                else finish(trg * FT + trr);
              }
#pragma unroll
              for (int tc = (FT == 2 ? ps : 0); tc < (FT == 2 ? ps + 1 : CT); ++tc) {
                const int t = (FT == 2 ? 0 : tc * 32) + (ln & 31);
                const int sw = 2 * ((t >> SH) & (LPT - 1));
#pragma unroll
                for (int trr = 0; trr < FT; ++trr)
#pragma unroll
                  for (int q = 0; q < 4; ++q) {
                    const int tr = trg * FT + trr;
                    const half4 o = {(_Float16)acc[tr][tc][4 * q], (_Float16)acc[tr][tc][4 * q + 1],
                                     (_Float16)acc[tr][tc][4 * q + 2], (_Float16)acc[tr][tc][4 * q + 3]};
                    const int slot = trr * 8 + 2 * q + h;
                    *reinterpret_cast<half4*>(stg + t * RB + ((slot ^ sw) * 8)) = o;
                  }
              }
#pragma unroll
              for (int i = 0; i < (64 / FT) / TPI; ++i) {
                const int tt = i * TPI + ln / LPT, c = ln % LPT;
                const uint4 val = *reinterpret_cast<const uint4*>(stg + tt * RB + ((c ^ ((tt >> SH) & (LPT - 1))) * 16));
                const int64_t tok = col0 + (FT == 2 ? ps * 32 : 0) + tt;
                if (tok < p.Ccols) {
                  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
                  const u32x4 v4 = {val.x, val.y, val.z, val.w};
                  *reinterpret_cast<u32x4*>(Y + tok * p.ldc + row0 + trg * FT * 32 + c * 8) = v4;
                }
              }
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      } else if constexpr (OUT_F32) {
        float* Cf = reinterpret_cast<float*>(p.C);
#pragma unroll
        for (int tr = 0; tr < RT; ++tr) {
          finish(tr);
#pragma unroll
          for (int tc = 0; tc < CT; ++tc) {
            const int64_t col = col0 + tc * 32 + (ln & 31);
            if (col < p.Ccols) {
#pragma unroll
              for (int v = 0; v < 16; ++v) {
                const int64_t row = row0 + tr * 32 + 8 * (v >> 2) + 4 * (ln >> 5) + (v & 3);
                Cf[row * p.ldc + col] = acc[tr][tc][v];
              }
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
        // One 32-row tile of the wave's columns at a time through this wave's share of the drained
        // stage (the producers refill that stage only after the next barrier).  A staged row is
        // 2*WCOLS bytes; its 16-byte chunks are XOR-swizzled by bit 2 of the row so that the two
        // half-waves, which write rows r and r+4, use different banks.
        constexpr int SROW = 2 * WCOLS;            // bytes of a staged row
        constexpr int LPS = SROW / 16;             // lanes (16-byte chunks) per staged row
        constexpr int SWZ = LPS / 2;               // chunk distance that changes the bank group
        char* stg = (OWN_STG ? smem + STG : const_cast<char*>(sb)) + wave * (32 * SROW);
        _Float16* Ch = reinterpret_cast<_Float16*>(p.C);
        const int chunk = ln % LPS, rsub = ln / LPS;
        const int64_t col = col0 + chunk * 8;
#pragma unroll
        for (int tr = 0; tr < RT; ++tr) {
          finish(tr);
#pragma unroll
          for (int tc = 0; tc < CT; ++tc) {
            if constexpr (CONS <= 4) {
              // two rows of this lane's column leave as two columns of one row, half as many LDS writes: the pair of rows is
              // rounded into a word, and an even lane takes the first row of its own and its neighbour's, an odd lane the second
              // (3072 x 768 x 4096 at 64:2:8 14.1 -> 13.6 us, 4096 x 1024 x 16384 on v128_c128d 42.3 -> 40.6, the same call again:
              // with other operands each time 67, where v128_c512 takes 56 and is chosen; with eight waves and 128 accumulators a lane
              // it costs registers: with GELU 65.5 -> 68.8)
              const int c = tc * 32 + (ln & 30);
              const uint32_t pick = ln & 1 ? 0x07060302u : 0x01000504u;   // bytes: 0-3 the neighbour's, 4-7 its own
#pragma unroll
              for (int v = 0; v < 16; v += 2) {
                const int r = 8 * (v >> 2) + 4 * (ln >> 5) + (v & 3) + (ln & 1);
                const int sw = ((c >> 3) ^ (SWZ * ((r >> 2) & 1)));
                const half2 rows = {(_Float16)acc[tr][tc][v], (_Float16)acc[tr][tc][v + 1]};   // one rounding, nearest-even
                const uint32_t own = __builtin_bit_cast(uint32_t, rows);
                const uint32_t other = __builtin_amdgcn_mov_dpp(own, 0xb1, 0xf, 0xf, true);    // lanes 1 0 3 2
                *reinterpret_cast<uint32_t*>(stg + r * SROW + sw * 16 + (c & 7) * 2) = __builtin_amdgcn_perm(own, other, pick);
              }
            } else {
              const int c = tc * 32 + (ln & 31);
#pragma unroll
              for (int v = 0; v < 16; ++v) {
                const int r = 8 * (v >> 2) + 4 * (ln >> 5) + (v & 3);
                const int sw = ((c >> 3) ^ (SWZ * ((r >> 2) & 1)));
                *reinterpret_cast<_Float16*>(stg + r * SROW + sw * 16 + (c & 7) * 2) =
                    (_Float16)acc[tr][tc][v];      // one rounding, nearest-even
              }
            }
          }
#pragma unroll
          for (int i = 0; i < 32 / (64 / LPS); ++i) {
            const int r = i * (64 / LPS) + rsub;
            const uint4 val = *reinterpret_cast<const uint4*>(stg + r * SROW + ((chunk ^ (SWZ * ((r >> 2) & 1))) * 16));
            if (col < p.Ccols) {
              typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
              u32x4* dst = reinterpret_cast<u32x4*>(Ch + (row0 + tr * 32 + r) * p.ldc + col);
              const u32x4 v4 = {val.x, val.y, val.z, val.w};
              // streaming stores keep C out of the L2 that holds the slab of B; they drain more
              // slowly, so the host asks for them only where the output is a small share of the traffic
              if (p.stream_out) __builtin_nontemporal_store(v4, dst);
              else *dst = v4;
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// What a call takes with a variant, in us: `launch`; for each tile that the busiest unit walks `tile`, and `k_step` for each
// of its k-steps; and as the units compete for the L2s and the memory behind them, `chip_tile` and `chip_step` for each tile
// and k-step that a unit has on average, and `fill_step` for each k-step of a tile by the share of the units in use.
struct TileCost { float launch, k_step, tile, chip_step, chip_tile, fill_step; };

struct Variant {
  const char* name;
  int V;       // block height it serves
  int bsc;     // columns per workgroup
  int threads;
  int lds;     // dynamic LDS bytes
  int share;   // workgroups that share a compute unit
  TileCost cost;
  void (*fn[2][4])(SpmmParams);   // [fp32 output][mode]
};

template <int VT, int NC, int NR, int KS, int NS, int NA>
constexpr int lds_bytes() {   // B ring, A ring, row-id ring, output staging (4 KB a wave) where it does not reuse a B stage
  return KS * (NS * kStepRows * 128 * NC + NA * (VT * kTileValBytes + kTailBytes) + kRidSlots * kStepRows * 4) +
         (NR > 1 ? NC * NR * 4096 : 0);
}

#define VARIANT(NAME, VT, NC, NR, KS, NS, NA, ...)                                                          \
  { NAME, (VT) * 32, 64 * (NC), 64 * ((NC) * (NR) + kProducers), lds_bytes<VT, NC, NR, KS, NS, NA>(),        \
    simd_waves(VT, NC, NR) >= 4 && lds_bytes<VT, NC, NR, KS, NS, NA>() <= 80 * 1024 ? 2 : 1, { __VA_ARGS__ }, \
    { { spmm_kernel<VT, NC, NR, KS, NS, NA, kD, false, 0>, spmm_kernel<VT, NC, NR, KS, NS, NA, kD, false, 1>, \
        spmm_kernel<VT, NC, NR, KS, NS, NA, kD, false, 2>, spmm_kernel<VT, NC, NR, KS, NS, NA, kD, false, 3> }, \
      { spmm_kernel<VT, NC, NR, KS, NS, NA, kD, true, 0>, spmm_kernel<VT, NC, NR, KS, NS, NA, kD, true, 1>,   \
        spmm_kernel<VT, NC, NR, KS, NS, NA, kD, true, 2>, spmm_kernel<VT, NC, NR, KS, NS, NA, kD, true, 2> } } }

constexpr int kD = 2;   // barriers between the hand-over of a stage and its return (1 and 2 measure the same)
// Rows per wave and ring depths, as measured (us per call).  V = 128: two waves per strip up to 256 columns
// (2048 x 1520 x 7896 at 128:2:20 with 256 columns 17.5, one wave 19.9).  "d" has rings shallow enough for a second
// workgroup on the unit, whose k-loop runs while the first one stores: better with few k-steps a tile, worse with many
// (16384 x 1024 x 512 at 128:2:8 13.9 against 14.5, 1024 x 16000 x 4096 at 128:2:40 20.4 against 17.8).  At V = 64 and 32
// the accumulators allow that with 256 columns (3072 x 768 x 4096 at 64:2:8 14.6, one workgroup with deeper rings 15.3).
// More stages than these cost start-up and gain nothing.
// KS: k-steps per stage.  A k-step of a narrow tile is barrier, row-id read and two or three loads a producer, one after the
// other (262 cycles with 64 columns, V = 128, of which no part waits for memory); two k-steps a barrier deal 19 loads over four
// producers where one deals 10, so that none has three while others have two, and meet half as often.  us per call, one -> two,
// V = 128: 8192 x 8192 x 64 at 2:16 12.0 -> 10.3 (64 columns), 12.4 -> 11.1 (128), x 256 13.3 -> 12.4; 3072 x 4096 x 256 at 96:2:8 12.0 -> 9.7
// (64), 14.3 -> 11.9 (128); 2048 x 4096 x 256 at 64:2:8 10.6 -> 8.6; 1024 x 4096 x 256 at 32:2:8 9.9 -> 8.3.  With 256 columns the loads
// take most of a k-step and two of them leave rings too short (8192 x 8192 x 256 18.4 -> 26.3); at V = 64 and 128 columns the second
// workgroup of the unit would go (2048 x 1000 x 2048 at 64:2:10 9.0 -> 10.9).
static const Variant kVariants[] = {
    VARIANT("v128_c512", 4, 8, 1, 1, 4, 6, 2.629f, .262f, 5.781f, .261f, 2.889f, 0.f),
    VARIANT("v128_c256", 4, 4, 2, 1, 5, 6, 3.285f, .248f, 2.159f, .073f, 2.764f, 0.f),
    VARIANT("v128_c128", 4, 2, 2, 2, 4, 4, 3.985f, .113f, 1.433f, .093f, .803f, 0.f),
    VARIANT("v128_c128d", 4, 2, 2, 1, 4, 6, 4.448f, .168f, .818f, .04f, .992f, 0.f),
    VARIANT("v128_c64", 4, 1, 2, 2, 4, 4, 4.681f, .103f, .764f, .014f, .518f, 0.f),
    VARIANT("v96_c512", 3, 8, 1, 1, 4, 6, 3.049f, .312f, 4.218f, .173f, 1.88f, .006f),
    VARIANT("v96_c256", 3, 4, 1, 1, 5, 6, 4.83f, .196f, .883f, .091f, 2.513f, .003f),
    VARIANT("v96_c128", 3, 2, 3, 2, 4, 4, 3.298f, .131f, .73f, .057f, 1.378f, 0.f),
    VARIANT("v96_c128d", 3, 2, 3, 1, 4, 4, 3.96f, .159f, .362f, .012f, 1.053f, .023f),
    VARIANT("v96_c64", 3, 1, 3, 2, 4, 4, 3.344f, .072f, .732f, .029f, .304f, .069f),
    VARIANT("v64_c512", 2, 8, 1, 1, 4, 10, 3.309f, .288f, 2.153f, .128f, 2.933f, 0.f),
    VARIANT("v64_c256", 2, 4, 1, 1, 5, 6, 3.927f, .152f, .874f, .106f, 1.158f, 0.f),
    VARIANT("v64_c256d", 2, 4, 1, 1, 4, 4, 4.121f, .173f, .412f, .053f, 1.52f, .021f),
    VARIANT("v64_c128", 2, 2, 2, 1, 5, 6, 3.671f, .146f, .354f, .017f, .676f, 0.f),
    VARIANT("v64_c64", 2, 1, 2, 2, 4, 4, 3.396f, .102f, .736f, .01f, .244f, .006f),
    VARIANT("v32_c512", 1, 8, 1, 1, 4, 10, 3.965f, .279f, .824f, .056f, 2.184f, .008f),
    VARIANT("v32_c256", 1, 4, 1, 1, 6, 10, 2.943f, .16f, 1.161f, .043f, .537f, .014f),
    VARIANT("v32_c256d", 1, 4, 1, 1, 4, 6, 3.529f, .16f, .519f, .033f, .372f, .041f),
    VARIANT("v32_c128", 1, 2, 1, 2, 4, 4, 3.45f, .093f, .775f, .052f, .05f, .003f),
    VARIANT("v32_c64", 1, 1, 1, 2, 4, 4, 2.57f, .081f, .765f, 0.f, .062f, .035f),
};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);

int spmm_variant_count() { return kNumVariants; }
const char* spmm_variant_name(int v) { return (v >= 0 && v < kNumVariants) ? kVariants[v].name : nullptr; }

// The variant of block height V with the smallest expected time.  Narrow tiles spread a small product over more units and
// have shorter k-steps (us of one tile alone on the chip, V = 128: 0.35 / 0.20 / 0.12 / 0.10 for 512 / 256 / 128 / 64 columns,
// the last two with two k-steps a barrier: 36.5 / 20.5 / 12.5 / 8.5 KB); wide ones read the records of A less often and load the
// chip's fabric less; the columns that pad C to whole tiles and a last round with few tiles cost as much as full ones.  The constants of TileCost are fits to the
// times of all variants over 4478 random shapes (R 64-49152, K 256-16000, C 40-16384, M 4-128, up to 6e10 FLOP) in four output
// forms (plain, with bias and GELU, that in fp32, and token-major): least squares of the relative error, from there on random steps
// on three quarters of them that make the chosen variant's time over the best one's smaller.  On the others the chosen variant is
// slower than the best by 0.5 to 0.9 % on average and 32 % at most, and the calls take 0.935 (V = 96) to 0.964 of the time of the tiles with
// one k-step a barrier, chosen by constants of their own.
static int pick_variant(int V, int64_t Ccols, int64_t nbr, int64_t steps, int cus) {
  int best = -1;
  float best_time = 0.f;
  for (int i = 0; i < kNumVariants; ++i) {
    const Variant& v = kVariants[i];
    if (v.V != V) continue;
    const TileCost& c = v.cost;
    const int64_t tiles = nbr * ((Ccols + v.bsc - 1) / v.bsc);
    const float s = (float)steps, most = (float)((tiles + cus - 1) / cus), mean = (float)tiles / (float)cus;
    const float time = c.launch + most * (c.k_step * s + c.tile) + mean * (c.chip_step * s + c.chip_tile) +
                       (mean < 1.f ? mean : 1.f) * c.fill_step * s;
    if (best < 0 || time < best_time) { best = i; best_time = time; }
  }
  return best;
}

// How many column tiles the workgroups of an XCD take side by side.  `resident` tiles are in work there together: one
// column of them shares the rows of one slab of B but needs as many block rows of A; `c` columns need a c-th of the
// records and c slabs.  With a 64-column slab the records are most of what the XCD fetches: 8192 x 8192 x 256 at 128:2:16
// (64 x 4 tiles, 32 per XCD: 10.5 MB with one column, 6.8 with two) 15.4 -> 13.4 us, 16384 x 1024 x 512 at 128:2:8 on
// this tile 16.8 -> 14.6.  Where the fetch shrinks by less than a quarter nothing is gained (4096 x 4096 x 1024 at
// 128:2:16 12.3 -> 12.6), nor where the XCD's L2 holds the records (3072 x 768 x 4096 at 64:2:8 23 -> 25), nor on
// the wider tiles (49152 x 12288 x 2048 at 128:2:32 228 -> 230).
static int column_group(const Layout& L, int bsc, int64_t nbr, int64_t nct, int64_t resident) {
  if (bsc != 64) return 1;
  auto records = [&](int c) {
    const int64_t rows = (resident + c - 1) / c;
    return (double)(rows < nbr ? rows : nbr) * (double)L.steps * (double)L.rec_bytes;
  };
  auto fetched = [&](int c) { return records(c) + (double)c * 2.0 * bsc * (double)L.K; };
  int best = 1;
  for (int c = 2; c <= 4 && c <= nct; c *= 2)
    if (records(best) > 3e6 && fetched(c) < 0.75 * fetched(best)) best = c;
  return best;
}

int compute_units() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  static std::atomic<int> cu_count[kMaxDevices] = {};   // per device, filled on first use
  const bool cached = dev >= 0 && dev < kMaxDevices;
  int cus = cached ? cu_count[dev].load(std::memory_order_relaxed) : 0;
  if (cus == 0) {
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (cached) cu_count[dev].store(cus, std::memory_order_relaxed);
  }
  return cus;
}

venom_status_t launch_spmm(const venom_handle& h, const void* B, int64_t ldb, int64_t Ccols, const void* bias, int act,
                           void* C, int64_t ldc, int c_dtype, int tokens_major, int variant, hipStream_t st) {
  const Layout& L = h.lay;
  if (!L.packed) return VENOM_ERR_UNSUPPORTED;
  if (L.R == 0 || Ccols == 0) return VENOM_OK;
  if (L.steps == 0) return VENOM_ERR_UNSUPPORTED;  // K = 0: there is no k-step to run the pipeline on
  const int Vp = L.vt * kTileRows;                 // block height of the packed copy
  const int cus = compute_units();
  if (cus < kNumXcd) return VENOM_ERR_HIP;
  // gather offsets are formed as row * ldb_bytes + column bytes in 32 bits with a 24-bit multiply
  if (h.K >= ((int64_t)1 << 24) || ldb * 2 >= ((int64_t)1 << 24) || h.K * ldb * 2 >= ((int64_t)1 << 32))
    return VENOM_ERR_UNSUPPORTED;
  if (variant < 0) {
    const int form = skinny_product(h, ldb, Ccols, cus);
    if (form >= 0) return launch_skinny(h, form, B, ldb, Ccols, bias, act, C, ldc, c_dtype, false, tokens_major != 0, st);
  }
  if (variant < 0) variant = pick_variant(Vp, Ccols, L.Rbp, L.steps, cus);
  if (variant < 0 || variant >= kNumVariants || kVariants[variant].V != Vp) return VENOM_ERR_UNSUPPORTED;
  const Variant& var = kVariants[variant];
  SpmmParams p{};
  p.arec = h.ws + L.off_arec;
  p.rowidx = reinterpret_cast<const int32_t*>(h.ws + L.off_rowidx);
  p.B = reinterpret_cast<const char*>(B);
  p.C = C;
  p.ldb_bytes = ldb * 2; p.ldc = ldc; p.Ccols = Ccols; p.rec_bytes = L.rec_bytes;
  p.steps = (int)L.steps;
  p.bias = reinterpret_cast<const _Float16*>(bias);
  p.act = act;
  p.serpentine = 1;
  p.pad_row0 = (L.G % kStepGroups) ? (int)(L.G % kStepGroups) * kSelCols : kStepRows;
  p.stream_out = L.steps >= 32;   // measured: +3 % at 48 k-steps per tile, -20 % at 8
  const int64_t nct = (Ccols + var.bsc - 1) / var.bsc;
  const int64_t nbr = L.Rbp;
  const int64_t total = nct * nbr;
  if (total > (int64_t)1 << 30 || L.steps > (int64_t)1 << 24) return VENOM_ERR_UNSUPPORTED;
  p.nbr = (int)nbr; p.nct = (int)nct;
  p.per_xcd = (int)((total + kNumXcd - 1) / kNumXcd);
  // one resident workgroup per compute unit (two where the tile is small enough to share a unit);
  // each walks per_xcd / (grid / 8) tiles
  const int64_t resident_per_xcd = (int64_t)(cus / kNumXcd) * var.share;
  const int64_t wg_per_xcd = p.per_xcd < resident_per_xcd ? p.per_xcd : resident_per_xcd;
  p.cgroup = column_group(L, var.bsc, p.nbr, p.nct, wg_per_xcd);
  const unsigned grid = (unsigned)(wg_per_xcd * kNumXcd);
  // a workgroup numbers the k-steps of all its tiles with one 32-bit counter
  if ((p.per_xcd + wg_per_xcd - 1) / wg_per_xcd * L.steps >= ((int64_t)1 << 30)) return VENOM_ERR_UNSUPPORTED;
  // token-major fp16 output takes the staged path when 16-byte stores are possible
  const bool wide = tokens_major && c_dtype == 0 && reinterpret_cast<uintptr_t>(C) % 16 == 0 && ldc % 8 == 0;
  const int epi = tokens_major ? (wide ? 3 : 2) : ((bias != nullptr || act != VENOM_ACT_NONE) ? 1 : 0);
  auto fn = var.fn[c_dtype == 1 ? 1 : 0][epi];
  if (var.lds > 64 * 1024) {
    // opting in to more than 64 KB of dynamic LDS is a per-function attribute (set once per device)
    // (two threads racing here both set the same attribute: harmless)
    static std::atomic<bool> opted_in[kNumVariants][8][kMaxDevices] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return VENOM_ERR_HIP;
    const bool cached = dev >= 0 && dev < kMaxDevices;
    if (!cached || !opted_in[variant][4 * c_dtype + epi][dev].load(std::memory_order_acquire)) {
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                              var.lds) != hipSuccess)
        return VENOM_ERR_HIP;
      if (cached) opted_in[variant][4 * c_dtype + epi][dev].store(true, std::memory_order_release);
    }
  }
  hipLaunchKernelGGL(fn, dim3(grid), dim3(var.threads), var.lds, st, p);
  return hipGetLastError() == hipSuccess ? VENOM_OK : VENOM_ERR_HIP;
}

// ---------------------------------------------------------------------------------------------
// The 2:4 matrix instruction alone: every wave issues `iters` x 8 independent instructions on
// register operands (pseudo-random fp16 values, so the multipliers toggle as they do on real data).
// Timed by the caller, it gives the instruction peak this GPU sustains at the clock it holds under
// that load: iters * 8 * 32768 useful FLOP per wave, 8 waves x 2 workgroups per compute unit.
__global__ void __launch_bounds__(512) smfmac_probe_kernel(int iters, float* sink) {
  const unsigned lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  unsigned x = (blockIdx.x * 8 + wave) * 64 + lane;
  auto next_half = [&]() {
    x = x * 1664525u + 1013904223u;
    return (_Float16)((float)((x >> 9) & 0xfff) * (1.f / 2048.f) - 1.f);      // in [-1, 1)
  };
  half8 a; half16 b;
  for (int e = 0; e < 8; ++e) a[e] = next_half();
  for (int e = 0; e < 16; ++e) b[e] = next_half();
  const int idx = 0x4e944e94 ^ (int)((lane & 1) * 0x00900090);                 // legal nibbles only
  floatx16 acc[8] = {};
  for (int i = 0; i < iters; ++i) {
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = smfmac<0>(a, b, acc[j], idx);
  }
  float s = 0.f;
  for (int j = 0; j < 8; ++j) s += acc[j][0];
  if (s == 12345.678f) sink[0] = s;              // keeps the loop alive; practically never true
}

hipError_t launch_smfmac_probe(int iters, float* sink, hipStream_t st) {
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(smfmac_probe_kernel, dim3(2 * cus), dim3(512), 0, st, iters, sink);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Activations as a linear layer holds them, X[token][k], to the K x tokens row-major operand the
// gather wants: 64 x 64 tiles through LDS, 4-byte accesses on both sides.
__global__ void __launch_bounds__(256) transpose_tokens_kernel(const uint16_t* __restrict__ X, int64_t ldx, int64_t tokens,
                                                               int64_t K, uint16_t* __restrict__ BT, int64_t ldbt) {
  __shared__ uint16_t tile[64][66];                // [k][token], padded
  const int64_t k0 = (int64_t)blockIdx.x * 64, tok0 = (int64_t)blockIdx.y * 64;
  const int pair = threadIdx.x & 31, sub = threadIdx.x >> 5;
  for (int r = sub; r < 64; r += 8) {               // r: token inside the tile, pair: two k
    const int64_t tok = tok0 + r, k = k0 + 2 * pair;
    uint16_t a = 0, b = 0;
    if (tok < tokens) {
      if (k + 1 < K && ((reinterpret_cast<uintptr_t>(X + tok * ldx + k) & 3) == 0)) {
        const uint32_t w = *reinterpret_cast<const uint32_t*>(X + tok * ldx + k);
        a = (uint16_t)w; b = (uint16_t)(w >> 16);
      } else {
        if (k < K) a = X[tok * ldx + k];
        if (k + 1 < K) b = X[tok * ldx + k + 1];
      }
    }
    tile[2 * pair][r] = a;
    tile[2 * pair + 1][r] = b;
  }
  __syncthreads();
  for (int r = sub; r < 64; r += 8) {               // r: k inside the tile, pair: two tokens
    const int64_t k = k0 + r, tok = tok0 + 2 * pair;
    if (k < K && tok < ldbt) {                       // ldbt is even and >= tokens: pad columns get zeros
      const uint32_t w = (uint32_t)tile[r][2 * pair] | ((uint32_t)tile[r][2 * pair + 1] << 16);
      *reinterpret_cast<uint32_t*>(BT + k * ldbt + tok) = w;
    }
  }
}

// The same with 16-byte accesses on both sides, for X, BT and both leading dimensions 16-byte
// aligned and K a multiple of 8: a thread loads 8 consecutive k of a token, the tile sits in LDS as
// [token][k] with rows of 136 bytes (so that the column reads below spread over the banks), and a
// thread gathers 8 consecutive tokens of one k for its store; 8 lanes write 128 contiguous bytes.
// STREAM: X is read past the caches, which leaves them to BT.  (Tiles of 128 tokens, with four loads a thread, are slower:
// layer of 4096 x 1024 x 16384 tokens 71.5 -> 73 us, with transposing LDS reads 75.)
template <bool STREAM>
__global__ void __launch_bounds__(256) transpose_tokens_wide_kernel(const uint16_t* __restrict__ X, int64_t ldx,
                                                                    int64_t tokens, int64_t K,
                                                                    uint16_t* __restrict__ BT, int64_t ldbt) {
  constexpr int kPitch = 136;                      // bytes per token row in LDS
  __shared__ __attribute__((aligned(16))) char tile[64 * kPitch];
  const int64_t k0 = (int64_t)blockIdx.x * 64, tok0 = (int64_t)blockIdx.y * 64;
  const int c = threadIdx.x & 7, r = threadIdx.x >> 3;
#pragma unroll
  for (int j = 0; j < 2; ++j) {                    // token r + 32j, k chunk c
    const int64_t tok = tok0 + r + 32 * j, k = k0 + 8 * c;
    uint4 w = make_uint4(0, 0, 0, 0);
    if (tok < tokens && k < K) {
      typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
      const u32x4* src = reinterpret_cast<const u32x4*>(X + tok * ldx + k);
      if constexpr (STREAM) {
        const u32x4 q = __builtin_nontemporal_load(src);
        w = make_uint4(q.x, q.y, q.z, q.w);
      } else {
        const u32x4 q = *src;
        w = make_uint4(q.x, q.y, q.z, q.w);
      }
    }
    uint2* dst = reinterpret_cast<uint2*>(tile + (r + 32 * j) * kPitch + c * 16);
    dst[0] = make_uint2(w.x, w.y);
    dst[1] = make_uint2(w.z, w.w);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 2; ++j) {                    // k row r + 32j, token chunk c
    const int kr = r + 32 * j;
    const int64_t k = k0 + kr, tok = tok0 + 8 * c;
    uint32_t o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t lo = *reinterpret_cast<const uint16_t*>(tile + (8 * c + 2 * e) * kPitch + kr * 2);
      const uint32_t hi = *reinterpret_cast<const uint16_t*>(tile + (8 * c + 2 * e + 1) * kPitch + kr * 2);
      o[e] = lo | (hi << 16);
    }
    if (k < K && tok < ldbt) *reinterpret_cast<uint4*>(BT + k * ldbt + tok) = make_uint4(o[0], o[1], o[2], o[3]);
  }
}

hipError_t launch_transpose_tokens(const uint16_t* X, int64_t ldx, int64_t tokens, int64_t K, uint16_t* BT, int64_t ldbt,
                                   int64_t out_bytes, hipStream_t st) {
  if (tokens == 0 || K == 0) return hipSuccess;
  if (reinterpret_cast<uintptr_t>(X) % 16 == 0 && reinterpret_cast<uintptr_t>(BT) % 16 == 0 && ldx % 8 == 0 &&
      ldbt % 8 == 0 && K % 8 == 0) {
    // X, its copy and the output against the 256 MB memory-side cache.  Where they exceed it, X is not found there when
    // the layer is called again, and its reads only take room from the copy.  Where they take more than half and the output is
    // at least twice X, that holds as soon as other buffers come in between (activations and output of three
    // layers in turn), and little is lost if they do not (the same buffers again and again); with a smaller output more is.
    // us per call, cached / streamed, the same buffers and three in turn: 8192 x 8192 x 8192 tokens (403 MB) 223 / 205, 224 / 206;
    // 4096 x 1024 x 16384 (201) 49.0 / 51.2, 54.9 / 51.1; 8192 x 1024 x 8192 (168) 45.8 / 46.1, 49.5 / 46.4; 2048 x 2048 x 16384 (201)
    // 50.9 / 56.7, 59.3 / 56.9; 512 x 6144 x 8192 (210) 49.8 / 53.9, 53.2 / 53.8; 512 x 4096 x 8192 (143) 35.5 / 38.7, 38.5 / 38.7.
    const int64_t x_bytes = tokens * K * 2, all = 2 * x_bytes + out_bytes;
    const bool streamed = all > (int64_t)256 << 20 || (all > (int64_t)128 << 20 && out_bytes >= 2 * x_bytes);
    auto fn = streamed ? transpose_tokens_wide_kernel<true> : transpose_tokens_wide_kernel<false>;
    hipLaunchKernelGGL(fn, dim3((unsigned)((K + 63) / 64), (unsigned)((ldbt + 63) / 64)), dim3(256),
                       0, st, X, ldx, tokens, K, BT, ldbt);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(transpose_tokens_kernel, dim3((unsigned)((K + 63) / 64), (unsigned)((ldbt + 63) / 64)), dim3(256), 0,
                     st, X, ldx, tokens, K, BT, ldbt);
  return hipGetLastError();
}

}  // namespace venom
