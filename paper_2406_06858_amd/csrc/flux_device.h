// Device-side building blocks of the fused tensor-parallel GEMM kernels (gfx950 / CDNA4).
//
// One templated kernel serves the three entry points; what differs is the prologue
// (AllGather-GEMM reads A from the chunk sources and stores the gathered matrix on the way, or waits on
// signals, paper Alg. 2) and the epilogue (GEMM-ReduceScatter adds the peer partial tiles and writes
// each row into its owner's slice, paper Alg. 1).
//
// Mapping to the hardware:
//   * bf16 inputs, v_mfma_f32_16x16x32_bf16, fp32 accumulators kept in registers;
//   * A tile [BM][BK] and B tile [BK][BN] staged in LDS with XOR-swizzled 16-byte slots;
//     A fragments are read with ds_read_b128, B fragments (B is [K,N] row-major, so a lane
//     needs 8 consecutive k of one column) with the transposing ds_read_b64_tr_b16;
//   * direct global-to-LDS loads of the slabs ahead while this one is multiplied;
//   * the accumulators go through LDS once in the epilogue so that every lane owns 8
//     consecutive columns of a row (of fp32 partials twice 4): peer partials are read and outputs
//     written 16 B per lane and instruction, 128..512 B contiguous per row.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include <type_traits>
#include <utility>
#include "flux.h"

namespace flux {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;

// ---- workspace layout (bytes) -------------------------------------------------------------
constexpr size_t WS_STATUS_OFF = 0;        // uint32 code, uint32 detail
constexpr size_t WS_DONE_OFF = 16;         // uint32: workgroups that are past their signal wait
constexpr size_t WS_STARTED_OFF = 32;      // uint32: copy-driver workgroups that have started
constexpr size_t WS_CALLSEQ_OFF = 48;      // uint32: calls without a copy kernel that have completed on this workspace
constexpr size_t WS_COUNTER_OFF = 256;     // uint32 per communication tile (copy kernel arrivals)
constexpr int MAX_COMM_TILES = 1024;
constexpr size_t WS_TILECNT_OFF = WS_COUNTER_OFF + 4 * MAX_COMM_TILES;   // split-K arrival counters
constexpr int MAX_SPLITK_TILES = 4096;
// Counter of the st-th K-cut tile.  Neighbouring tiles' counters lie 256 bytes apart: atomics on one memory channel queue
// up behind each other, tens of nanoseconds each, and the parts of all tiles arrive at about the same time.
__host__ __device__ constexpr int sk_counter_index(int st) { return (st % 64) * (MAX_SPLITK_TILES / 64) + st / 64; }
// Workgroups past their signal wait are counted in two levels: workgroup b adds to leaf b mod
// DONE_LEAVES, whoever completes a leaf adds to the root (WS_DONE_OFF).  Hundreds of additions to one
// address queue up behind each other (tens of nanoseconds each), and every workgroup waits for its
// own to come back.  The leaves lie in different memory channels.
constexpr int DONE_LEAVES = 32;
constexpr size_t DONE_LEAF_STRIDE = 256;
constexpr size_t WS_DONELEAF_OFF = WS_TILECNT_OFF + 4 * MAX_SPLITK_TILES;
constexpr size_t WS_HEADER_BYTES = WS_DONELEAF_OFF + DONE_LEAVES * DONE_LEAF_STRIDE;
// After the header: AllGather piece claims (uint32 per communication tile and piece), then the
// split-K partials.
constexpr int MAX_COPY_PIECES = 256;       // pieces per communication tile = copy-driver workgroups

// ---- TileCoord (paper Sec. 4.1) -----------------------------------------------------------
// The host builds `m_order`: the order in which m-tiles are scheduled (slice by slice after
// the local rank for ReduceScatter, chunk by chunk in arrival order for AllGather).  Ascending
// workgroup ids walk that order in bands of `band_h` m-tiles times all n-tiles, m fastest.
// Workgroups are dealt round-robin to the accelerator dies, so with n_xcd > 1 the in-band index
// is regrouped to give every die a contiguous run of the band (shared panels stay in its L2).
// With at most 16 m-tiles the order also sits in `order4`, four bits per position: a kernel then
// has its tile after the first fetch of its arguments, not after a second, dependent one into the
// table (about a microsecond at the start of every workgroup).
struct TileMap {
  int32_t tiles_m, tiles_n, band_h, n_xcd;
  int32_t packed;
  int32_t peers_first;       // reduce-scatter: every second column (1) or row (2) of tiles adds its peers ahead of its main loop (see sum_peers_first)
  uint64_t order4;
};

// `m_order`: the table, read where the order is not packed.
__host__ __device__ inline void tile_coord(const TileMap& tm, const uint16_t* m_order, int block, int& mt, int& nt) {
  const int band_sz = tm.band_h * tm.tiles_n;
  const int band = block / band_sz;
  int q = block - band * band_sz;
  if (tm.n_xcd > 1 && band_sz % tm.n_xcd == 0) q = (q % tm.n_xcd) * (band_sz / tm.n_xcd) + q / tm.n_xcd;
  const int i = band * tm.band_h + q % tm.band_h;
  nt = q / tm.band_h;
  mt = tm.packed ? (int)((tm.order4 >> (4 * i)) & 15) : (int)m_order[i];
}

enum : int { EPI_PLAIN = 0, EPI_RS = 1 };
// What a kernel does about A ahead of its main loop: nothing; wait for the signals of its rows of the gathered matrix (Alg. 2);
// or read A from the chunk sources themselves, and move the chunks into the gathered matrix beside its products.
enum : int { PRO_NONE = 0, PRO_WAIT = 1, PRO_CHUNKS = 2 };

// Kernel arguments.  A workgroup's first fetches from the argument block miss the scalar cache one
// 64-byte line after the other, a quarter of a microsecond each, before its first load can be
// issued: the scalars sit together at the front, grouped by who needs them (every kernel; the signal
// wait; the transfer; split-K and the reduce-scatter epilogue), and the arrays come last.  What every workgroup reads
// ahead of its first operand load fills the first two lines exactly (asserted below).  With the tile map behind the arrays
// a field added anywhere pushed it across one more line; us per launched call, map in a line behind the arrays / across
// two / here: rs 128 x 256 x 256 fp32, 2 ranks, 7.04 / 7.22 / 6.29, rs 64 x 8192 x 3584, 8 ranks, - / 19.7 / 18.9.
struct GemmArgs {
  // ---- every kernel: two lines ----
  const __bf16* A;           // [M,K]
  const __bf16* B;           // [K,N]
  void* C;                   // [M,N] of out dtype (plain epilogue)
  int32_t M, N, K;
  int32_t R, rank, S;        // S = M / R
  int32_t lda, ldb, ldc;     // row pitches in elements: A (the gathered matrix); B; C and the out slices (peer partials are packed)
  int32_t b_is_nk;           // B is [N,K] (the kernels built for that layout are launched)
  // K split: the first `full_tiles` tiles (in TileCoord order) are computed by one workgroup
  // each; every one of the remaining `split_tiles` tiles by `split_k` workgroups that each take
  // `k_per_split` of K.  A uniform split has full_tiles = 0; splitting only the tiles of the last,
  // partly filled round of the grid keeps all CUs busy to the end.
  int32_t full_tiles, split_tiles;
  int32_t split_k, k_per_split;   // k_per_split is a multiple of BK
  TileMap tm;
  flux_trace_record_t* trace;     // tile trace, one record per workgroup; null: none
  int32_t write_only;        // 1: reduce-scatter epilogue without the reduction (Write branch of Alg. 1);
                             // 2: no peers are read, the tile is added to the slice with atomic additions
  int32_t partial_f32;
  // ---- all-gather prologue: the signal wait ----
  uint32_t* signals;
  uint32_t* done_counter;
  uint32_t* status;
  unsigned long long timeout_ticks;
  int32_t rows_per_signal;
  int32_t n_signals, sig_local_lo, sig_local_hi;   // local communication tiles: [lo, hi)
  // the transfer: pieces of communication tiles are claimed and moved by this grid's workgroups
  // and/or a copy kernel (outs[] then holds the chunk sources, A is the gathered matrix);
  // copy_pieces = 0: the grid moves nothing and only waits (hipMemcpyAsync driver, or R = 1)
  int32_t copy_pieces;       // pieces per communication tile
  // No driver at all (copy_owner_wgs > 0): piece g (counted over the remote communication tiles in
  // transfer order, tile j lying in the chunk at position j / ctpc of copy_order4) belongs to
  // workgroup g % copy_owner_wgs of this grid, which moves it before it looks at its own signals.
  int32_t copy_owner_wgs;
  int32_t copy_eager;        // waiting workgroups take pieces even while the whole driver is running
  int32_t acquire_l2;        // the gathered rows may share cache lines across communication tiles: full acquire after the wait
  // The driver is a copy engine or library copy that takes no pieces (copy_pieces = 0): a workgroup
  // that has waited this long (100 MHz ticks; 0: never) fetches the rows of its own tile itself.
  uint32_t self_serve_ticks;
  // ---- the transfer ----
  uint32_t* copy_claims;     // [n_signals][copy_pieces], a piece is taken when it holds copy_call_id
  uint32_t* copy_counters;   // [n_signals] pieces finished
  uint32_t* copy_call_seq;
  uint32_t* started_counter;
  unsigned long long copy_order4;   // chunk of position i in bits [4i, 4i+4)
  unsigned long long copy_tile_vec;   // 16-byte vectors per communication tile
  uint32_t copy_call_id;     // 0: take the id from copy_call_seq (calls without a copy kernel)
  int32_t copy_driver_wgs;   // workgroups of the copy kernel launched beside this grid (0: none)
  int32_t copy_n_tiles;
  // The rank's own chunk lies in a buffer of its own and is moved by the grid too, ahead of the remote ones (copy_n_tiles
  // counts it, its tiles come first).  Its signals are preset, so a tile of it has arrived when its word in copy_counters
  // reads copy_pieces.  (See tile_arrived.)
  int32_t copy_local;
  // The last copy_defer_tiles remote communication tiles of the transfer order are not moved before
  // the signal wait: the workgroups of the first round carry them inside their main loops (piece w
  // of each such tile by workgroup w, copy_defer_steps 16-byte vectors per thread and tile).
  int32_t copy_defer_tiles;
  int32_t copy_defer_steps;
  // ... and with copy_pace_ticks != 0 they stand for a link: the i-th tile of the transfer order is
  // counted in no earlier than (i + 1) * copy_pace_ticks (100 MHz ticks) after the kernel started
  unsigned long long copy_pace_ticks;
  int32_t gather_local;      // A read from the chunk sources (see GatherOut): the rank's own chunk, too, lies in a buffer of its own
  // ---- split-K hand-over, reduce-scatter epilogue ----
  float* sk_partials;             // [split_k][split_tiles][BM*BN] fp32
  uint32_t* sk_counters;          // [tiles]
  int32_t sk_share;               // not 0: the parts of a tile share its final sum out among themselves (see SharedFinish), and wait so many
                                  // 100 MHz ticks for parts that have not started
  int32_t out_f32;
  uint32_t* tile_ready;           // reduce-scatter, Write branch: per output tile, producers that have written it; null: not kept
  int32_t persist_blocks;         // > 0: a grid of resident workgroups, workgroup b takes the blocks b, b + grid, ... below this
  uint32_t persist_delay_ticks;   // ... and every second group of eight starts this late (100 MHz ticks)
  // ---- arrays ----
  alignas(64) void* outs[FLUX_MAX_RANKS];
  const void* peers[FLUX_MAX_RANKS];   // the R-1 peer partials packed in ascending rank order
  uint16_t m_order[FLUX_MAX_M_TILES];  // order of the m-tiles, where it does not fit tm.order4
};
static_assert(alignof(GemmArgs) == 64 && offsetof(GemmArgs, partial_f32) + sizeof(int32_t) == 128, "every workgroup's arguments: the first two lines");

// The rank-indexed pointers (output slices, or chunk sources) go to LDS for dynamic indexing.  The
// second half of the array lies in another line of the argument block and is only touched when
// there are that many ranks.  Made visible to the other threads by the next workgroup barrier.
__device__ __forceinline__ void fill_lds_outs(const GemmArgs& a, void** lds_outs, int tid) {
  static_assert(FLUX_MAX_RANKS == 16, "two halves of eight");
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (tid == j) lds_outs[j] = a.outs[j];
  if (a.R > 8) {
#pragma unroll
    for (int j = 8; j < 16; ++j)
      if (tid == j) lds_outs[j] = a.outs[j];
  }
}

// workgroup id -> (tile in TileCoord order, K split index, is this tile split)
__device__ __forceinline__ void map_block(const GemmArgs& a, int b, int& tile, int& split, bool& is_split) {
  if (b < a.full_tiles) {
    tile = b; split = 0; is_split = false;
  } else {
    const int r = b - a.full_tiles;
    tile = a.full_tiles + r % a.split_tiles;
    split = r / a.split_tiles;
    is_split = a.split_k > 1;
  }
}

// ---- tile trace -------------------------------------------------------------------------------
// With a trace buffer every workgroup leaves one record: which tile and K part it computed, on which
// die and compute unit, and the 100 MHz wall clock at four points (kernel entry, past the signal
// wait, main loop done, epilogue stores acknowledged).  Thread 0 writes; without a buffer the cost
// is one scalar test per point.
enum : int { TRACE_START = 0, TRACE_READY = 1, TRACE_MAIN_END = 2, TRACE_END = 3 };

__device__ __forceinline__ void trace_begin(const GemmArgs& a, int tile, int mt, int nt, int split, bool is_split, int vb = -1) {
  if (a.trace == nullptr || threadIdx.x != 0) return;
  const uint32_t b = vb < 0 ? blockIdx.x : (uint32_t)vb;
  flux_trace_record_t* r = a.trace + b;
  r->block = b;
  r->m_tile = (uint32_t)mt;
  r->n_tile = (uint32_t)nt;
  r->k_part = (uint32_t)split | (is_split ? 0x10000u : 0u);
  r->die = __builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) ;       // XCC_ID, bits [3:0]
  r->hw_id = __builtin_amdgcn_s_getreg(4 | (0 << 6) | (31 << 11));      // HW_ID, all 32 bits
  r->tile = (uint32_t)tile;
  r->reserved = 0;
  const uint64_t t = wall_clock64();
  r->t_start = t; r->t_ready = t; r->t_main_end = t; r->t_end = t;
}

__device__ __forceinline__ void trace_stamp(const GemmArgs& a, int point, int vb = -1) {
  if (a.trace == nullptr) return;
  if (point == TRACE_END) __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's stores are acknowledged
  if (threadIdx.x != 0) return;
  flux_trace_record_t* r = a.trace + (vb < 0 ? blockIdx.x : (uint32_t)vb);
  const uint64_t t = wall_clock64();
  if (point == TRACE_READY) r->t_ready = t;
  if (point <= TRACE_MAIN_END) r->t_main_end = t;
  r->t_end = t;
}

// ---- LDS swizzles ---------------------------------------------------------------------------
// A tile: rows of BK bf16 = BK/8 slots of 16 B; slot s of row r is stored at slot s ^ fA(r).
// LDS has 64 banks of 4 B and answers a ds_read_b128 in four passes of 16 lanes that are not consecutive: lanes 0-3,
// 12-15 and 20-27 together, then 4-11, 16-19 and 28-31, and the same for the upper half (measured: which two lanes get in each
// other's way).  A fragment's lanes are rows i = 0..15 of slot q, the next sixteen the same rows of slot q + 1 (q even), so a
// pass holds every row once, half of them with the lowest slot bit flipped.  128-byte rows fill half of the banks: the eight
// rows of one parity must land in eight different slots, and s ^ (row & 7) does that.  (With bit 3 of the row mixed in as
// well, right for sixteen consecutive lanes, every read took two turns: 6.0 against 3.1 cycles per instruction.)
template <int SLOTS>
__device__ __forceinline__ int swz_a(int row) {
  return row & (SLOTS - 1);
}
// B tile: rows of BN bf16 (one k each).  The transposing read answers 32 lanes per pass: 32 bytes of each of the rows k..k+3
// and k+8..k+11, whose pitch is a multiple of all banks (or, 64 columns, half of it).  Bits 0, 1 and 3 of k pick the 32-byte bank
// group.  (Without bit 3 the two sets of four rows got in each other's way: 3.1 against 2.1 cycles per instruction.)
template <int SLOTS>
__device__ __forceinline__ int swz_b(int k) {
  const int kk = k & 3;
  return ((kk << 2) ^ (kk << 1) ^ ((k >> 2) & 2)) & (SLOTS - 1);
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  f32x2 v = {lo, hi};
  bf16x2 h = __builtin_convertvector(v, bf16x2);   // round-to-nearest-even
  return __builtin_bit_cast(uint32_t, h);
}

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

// Streaming (non-temporal) 16-byte accesses for data touched exactly once: peer partials and
// outputs must not push the A/B panels, which are re-read many times, out of the L2.
// All of them are addresses of device memory.  Where the type says so (global_u32x4) an access counts as one to memory alone; of a
// pointer that was kept in LDS the compiler does not know it and makes flat accesses, which a wait for an LDS read then waits
// for too.  st_out16 says where that is wanted.
typedef __attribute__((address_space(1))) u32x4 global_u32x4;
__device__ __forceinline__ u32x4 ld_stream(const void* p) { return __builtin_nontemporal_load((const global_u32x4*)p); }
__device__ __forceinline__ uint4 ld_stream16(const void* p) {
  const u32x4 v = ld_stream(p);
  return make_uint4(v[0], v[1], v[2], v[3]);
}
template <bool FLAT = false>
__device__ __forceinline__ void st_stream16(void* p, const uint4& v) {
  const u32x4 d = {v.x, v.y, v.z, v.w};
  if (FLAT) __builtin_nontemporal_store(d, static_cast<u32x4*>(p));
  else __builtin_nontemporal_store(d, (global_u32x4*)p);
}

// 16-byte store at device scope: written through this die's L2, so that a reader on another
// accelerator die needs no write-back of the whole L2 to see it.
__device__ __forceinline__ void store_through(uint4* p, const u32x4& d) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1" : : "v"(p), "v"(d) : "memory");
}
// Output vectors: streamed, or written through when a consumer may read the tile as soon as its ready
// counter moves (`through`, uniform).
// FLAT: a wave does not read on from LDS before its stores are out.  Behind reads of peers, where every unit reads and writes all
// the memory gives, that is faster (us, flat / global: rs 8192x12288x1536 424 / 438, 512x8192x1024 37.9 / 39.6, 1024x4096x2048 44.4 / 46.3;
// the other side: 1496x5112x3400 86.1 / 85.2); without peers waiting costs (the end of a 256x256 tile 9.0 / 7.6).
template <bool FLAT>
__device__ __forceinline__ void st_out16(void* p, const uint4& v, bool through) {
  if (through) store_through(static_cast<uint4*>(p), u32x4{v.x, v.y, v.z, v.w});
  else st_stream16<FLAT>(p, v);
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// B_NK: B is given as [N,K] (row n holds the K values of output column n, the layout of a linear
// layer's weight).  Its tile then sits in LDS like A's (rows of BK values, the same slot swizzle) and a
// fragment is one 16-byte read per lane, as for A, instead of two transposing reads.
// NA, NB: slabs of A and of B that LDS holds; A may have one more.
template <int BM_, int BN_, int BK_, int WAVES_M_, int WAVES_N_, int NA_, int NB_, int OCC_, bool B_NK_ = false>
struct TileCfg {
  static constexpr int BM = BM_, BN = BN_, BK = BK_, WAVES_M = WAVES_M_, WAVES_N = WAVES_N_;
  static constexpr int NA = NA_, NB = NB_, OCC = OCC_;
  static constexpr bool B_NK = B_NK_;
  static constexpr int NT = WAVES_M * WAVES_N * 64;
  static constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;
  static constexpr int MI = WTM / 16, NI = WTN / 16;       // 16x16 blocks of a wave's tile
  static constexpr int A_SLOTS = BK / 8, B_SLOTS = BN / 8;
  static constexpr int A_BYTES = BM * BK * 2, B_BYTES = BK * BN * 2;
  static constexpr int RING_BYTES = NA * A_BYTES + NB * B_BYTES;   // the A slabs, then the B slabs
  static constexpr int EP_STRIDE = WTN + 8;                       // floats; 4 rows apart = 128 B off
  static constexpr int EP_BYTES = WAVES_M * WAVES_N * 32 * EP_STRIDE * 4;
  static_assert(BM % (WAVES_M * 32) == 0 && BN % (WAVES_N * 32) == 0 && BK % 32 == 0, "tile shape");
  static_assert(B_SLOTS >= 8, "BN >= 64");
  static_assert(NB >= 2 && (NA == NB || NA == NB + 1), "the order of the loads (MmaPipe)");

  // LDS of a workgroup: the ring, over it (once the main loop is done) the epilogue's staging area, and a few words that the
  // workgroup shares (SharedWords).  Where the ring takes all of a compute unit's LDS the words lie over the slab that is asked
  // for last, by the main loop, and behind the staging area after it.
  static constexpr int LDS_MAX = 160 * 1024;
  static constexpr int WORDS_BYTES = 256;
  static constexpr int MAX_BYTES = RING_BYTES > EP_BYTES ? RING_BYTES : EP_BYTES;
  static constexpr bool WORDS_IN_RING = MAX_BYTES + WORDS_BYTES > LDS_MAX / OCC;
  static constexpr int POOL_BYTES = WORDS_IN_RING ? MAX_BYTES : MAX_BYTES + WORDS_BYTES;
  static constexpr int WORDS_AT = WORDS_IN_RING ? (NA - 1) * A_BYTES : MAX_BYTES;   // before and in the main loop
  static constexpr int WORDS_AT_TAIL = WORDS_IN_RING ? MAX_BYTES - WORDS_BYTES : MAX_BYTES;   // after it
  static_assert(!WORDS_IN_RING || (NA > NB && WORDS_AT_TAIL >= EP_BYTES), "room for the shared words");
};

struct SharedWords {
  void* outs[FLUX_MAX_RANKS];       // output slices (reduce-scatter) or chunk sources (all-gather), by rank
  int misc[4];
};

// f(0), f(1), ... f(N-1) with the index as a compile-time constant.
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// MFMA shape: 16x16x32, the A fragment held over a row of MFMAs.  With random operands the chip runs at its power
// limit, and this form takes less power than 32x32x16: MFMAs alone 2.0 against 1.75-1.8 PFLOP/s (2.4 for both on
// zeros).  Holding B instead and changing A every time costs 25 % of the rate even on zeros.
//
// The instruction is written out with its accumulator tied to an accumulation register: left to itself the compiler
// gives D and C different registers and shuffles hundreds of them around per slab.  It then does not know that
// the result takes a while: whoever reads the accumulators waits for them (mfma_results_settle).
__device__ __forceinline__ void mfma_in_place(f32x4& acc, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// The results of all MFMAs issued so far can be read (18 wait states are the most any of them takes).  The
// accumulators pass through, so that nothing that reads them can be moved in front.
template <int MI, int NI>
__device__ __forceinline__ void mfma_results_settle(f32x4 (&acc)[MI][NI]) {
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) asm volatile("" : "+a"(acc[mi][ni]));
}

// Store 8 consecutive output columns of one row into the owner's slice (GetOutput of Alg. 1) or
// into C, converting once.
template <int EPI, bool FLAT>
__device__ __forceinline__ void store_row8(const GemmArgs& a, void* const* lds_outs, int gm, int gn, const float (&v)[8]) {
  void* base;
  size_t o;
  const bool through = EPI == EPI_RS && a.tile_ready != nullptr;
  if (EPI == EPI_RS) {
    const int r = gm / a.S;
    base = lds_outs[r];
    o = (size_t)(gm - r * a.S) * a.ldc + gn;
  } else {
    base = a.C;
    o = (size_t)gm * a.ldc + gn;
  }
  if (a.out_f32) {
    float* q = static_cast<float*>(base) + o;
    st_out16<FLAT>(q, make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])), through);
    st_out16<FLAT>(q + 4, make_uint4(__float_as_uint(v[4]), __float_as_uint(v[5]), __float_as_uint(v[6]), __float_as_uint(v[7])), through);
  } else {
    uint4 w;
    w.x = pack_bf16x2(v[0], v[1]); w.y = pack_bf16x2(v[2], v[3]);
    w.z = pack_bf16x2(v[4], v[5]); w.w = pack_bf16x2(v[6], v[7]);
    st_out16<FLAT>(static_cast<__bf16*>(base) + o, w, through);
  }
}

// ... and 4 of them (fp32 partials: see piece_col).
template <int EPI, bool FLAT>
__device__ __forceinline__ void store_row4(const GemmArgs& a, void* const* lds_outs, int gm, int gn, const float* v) {
  const bool through = EPI == EPI_RS && a.tile_ready != nullptr;
  void* base = a.C;
  size_t o = (size_t)gm * a.ldc + gn;
  if (EPI == EPI_RS) {
    const int r = gm / a.S;
    base = lds_outs[r];
    o = (size_t)(gm - r * a.S) * a.ldc + gn;
  }
  if (a.out_f32) {
    st_out16<FLAT>(static_cast<float*>(base) + o, make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])), through);
  } else {
    // (fp32 partials are never asked for with counted-in tiles, whose peers are not read: no write-through form)
    typedef __attribute__((ext_vector_type(2))) unsigned int u32x2_;
    typedef __attribute__((address_space(1))) u32x2_ global_u32x2;
    const u32x2_ d = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
    __builtin_nontemporal_store(d, (global_u32x2*)(static_cast<__bf16*>(base) + o));
  }
}

// A lane's 8 columns of a row of a wave's tile: 8 in a row; of fp32 partials twice 4, so that an instruction reads (and writes) 16 bytes a
// lane without gaps: whole lines of 64 columns or more.  With 8 in a row an instruction takes every second 16 bytes of twice as many lines, and
// streamed lines were fetched twice: us, 8 in a row / twice 4, fp32, 8 ranks 512x1024x256 14.2 / 11.0, 512x12288x6144 126 / 113, 1496x5112x3400
// 124 / 115, 4096x4608x1536 189 / 176, 16 ranks 4096x4608x3584 386 / 344, 2 ranks 8192x6144x1536 203 / 181.
template <class C, bool PF32>
__device__ __forceinline__ int piece_col(int cc, int half) {
  return PF32 ? (half * (C::WTN / 8) + cc) * 4 : cc * 8 + half * 4;
}

// The peer partials of one tile as buffer resources based at the tile's origin (Reduce of Alg. 1
// reads them).  `a.peers` holds the R-1 peers in ascending rank order; a resource past that has no
// records, so its loads return zeros and every lane runs the same straight-line code: seven loads
// per 8-column piece, no branch and no pointer fetch between them.
struct PeerBufs {
  __amdgpu_buffer_rsrc_t r[FLUX_MAX_RANKS - 1];
};

__device__ __forceinline__ void make_peer_bufs(const GemmArgs& a, int m0, int n0, PeerBufs& pb) {
  const size_t tile_off = ((size_t)m0 * a.N + n0) * (a.partial_f32 ? 4 : 2);
#pragma unroll
  for (int j = 0; j < FLUX_MAX_RANKS - 1; ++j) {
    // (the address is the same in every lane; saying so keeps the resource in scalar registers)
    const uint64_t addr = reinterpret_cast<uint64_t>(a.peers[j]) + tile_off;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)addr), hi = __builtin_amdgcn_readfirstlane((uint32_t)(addr >> 32));
    unsigned char* base = reinterpret_cast<unsigned char*>(((uint64_t)hi << 32) | lo);
    pb.r[j] = __builtin_amdgcn_make_buffer_rsrc(base, 0, j < a.R - 1 ? 0x7fffffff : 0, 0x00027000);
  }
}

// The peers' rows of a small whole tile, asked for ahead of its main loop and held in registers until its end: a small call is a
// chain of memory round trips, and this one does not depend on the products.  NP peers (1, 3 or 7; absent ones read nothing, but cost
// an issue slot each; not streamed: half a line each, us, streamed / kept, 8 ranks 512x1024x256 9.0 / 7.6, 32x8192x384 9.4 / 7.9), where they fit ROOM
// vectors (with 14 instead of 6, and kept through a hand-over, the kernels of two workgroups per unit spilled: 5.9 us -> 6.6).
// us per call, peers behind the main loop / ahead of it: fp32, 2 ranks: 128x256x256 5.92 / 5.09 (5.1 to 5.8 on other machines, 4 to 10 % gained), 64x512x512 8.21 / 6.69, 512x1024x256 9.00 /
// 6.85; bf16: 2 ranks 2048x2048x1024 18.7 / 16.3, 4 ranks 512x3584x1536 14.7 / 13.7, 8 ranks 2048x1024x512 13.5 / 13.0; the other side:
// 64x512x512 7.8 / 8.0, 2048x1024x2048 20.5 / 20.8.
template <class C>
struct EarlyPeers {
  static constexpr int RPP = 512 / C::WTN;                 // rows per pass (see epilogue_block)
  static constexpr int PASSES = C::WTM / RPP;
  static constexpr bool SMALL = C::BM * C::BN < 128 * 128;
  static constexpr int ROOM = C::OCC == 1 ? 28 : 6;        // 112 or 24 registers
  u32x4 w[SMALL ? ROOM : 1];                               // pass by pass, peer by peer
  template <int NP, bool PF32>
  static constexpr __device__ int at(int pass, int j, int l) { return (pass * NP + j) * (PF32 ? 2 : 1) + l; }
  template <int NP, bool PF32>
  static constexpr bool fits() { return SMALL && PASSES * NP * (PF32 ? 2 : 1) <= ROOM; }

  // K-cut tiles never ask.  The compiler does not know it, and kept these registers through their hand-over, which then spilled in the kernels of
  // two workgroups per unit (8 to 28 bytes of scratch a lane; us, spilled / not: 128x256x256 fp32, 2 ranks, 5.16 / 5.12, 8 ranks 40x1000x2008
  // 9.33 / 9.09, 8x1000x1024 8.56 / 8.45, 136x1536x1536 [N,K] 9.03 / 8.92; the other side 72x1536x1536 8.22 / 8.29).  Called where a hand-over ends.
  __device__ __forceinline__ void forget() {
    if constexpr (SMALL)
#pragma unroll
      for (int i = 0; i < ROOM; ++i) asm volatile("" : "=v"(w[i]));
  }

  template <bool EDGE, int NP, bool PF32>
  __device__ __forceinline__ int ask_as(const GemmArgs& a, int m0, int n0, int lane, int wm, int wn) {
    if constexpr (fits<NP, PF32>()) {
      PeerBufs pb;
      make_peer_bufs(a, m0, n0, pb);
      const int cc = lane % (C::WTN / 8), rl = lane / (C::WTN / 8);
#pragma unroll
      for (int t = 0; t < PASSES; ++t) {
        const int row = wm * C::WTM + t * RPP + rl;
#pragma unroll
        for (int l = 0; l < (PF32 ? 2 : 1); ++l) {
          const int col = wn * C::WTN + piece_col<C, PF32>(cc, l);
          const bool ok = !EDGE || (m0 + row < a.M && n0 + col < a.N);
          const int voff = ok ? (int)(((uint32_t)row * (uint32_t)a.N + (uint32_t)col) * (PF32 ? 4u : 2u)) : (int)0x80000000;
#pragma unroll
          for (int j = 0; j < NP; ++j) w[at<NP, PF32>(t, j, l)] = __builtin_amdgcn_raw_buffer_load_b128(pb.r[j], voff, 0, 0);
        }
      }
      return NP;
    }
    return 0;
  }
  // Peers asked for: 1, 3, 7 or none.  (Uniform.)
  template <bool EDGE>
  __device__ __forceinline__ int ask(const GemmArgs& a, bool is_split, int m0, int n0, int lane, int wm, int wn) {
    if (is_split || a.write_only) return 0;
    if (a.R == 2) return a.partial_f32 ? ask_as<EDGE, 1, true>(a, m0, n0, lane, wm, wn) : ask_as<EDGE, 1, false>(a, m0, n0, lane, wm, wn);
    if (a.R <= 4) return a.partial_f32 ? ask_as<EDGE, 3, true>(a, m0, n0, lane, wm, wn) : ask_as<EDGE, 3, false>(a, m0, n0, lane, wm, wn);
    if (a.R <= 8) return a.partial_f32 ? ask_as<EDGE, 7, true>(a, m0, n0, lane, wm, wn) : ask_as<EDGE, 7, false>(a, m0, n0, lane, wm, wn);
    return 0;
  }
};

// One 32-row block of a wave's tile, already transposed into `ep`: every lane takes 8 consecutive
// columns of a row per pass.  With the reduce-scatter epilogue the peer loads of BATCH passes are
// issued together before any of them is used (PF32: fp32 partials, two 16-byte loads per peer);
// the peers are added in ascending rank order.
// EARLY: they are in `early` already, from pass `pass0` on.
template <class C, int EPI, bool EDGE, bool PF32, int BATCH, int NP, bool RESIDENT, bool EARLY>
__device__ __forceinline__ void epilogue_block(const GemmArgs& a, void* const* lds_outs, const float* ep, const PeerBufs& pb,
                                               int row_base, int col_base, int m0, int n0, int lane, const EarlyPeers<C>& early, int pass0) {
  constexpr int CH = C::WTN / 8;          // 8-column pieces per row of the wave tile
  constexpr int RPP = 64 / CH;            // rows per pass
  constexpr int NIT = 32 / RPP;
  constexpr int B = BATCH < NIT ? BATCH : NIT;
  constexpr int LPP = PF32 ? 2 : 1;
  // cache policy: streamed, not kept; but where an instruction reads half a line of a row, another wave has the other half.  (By the tile's
  // width alone: rows of peers or results that are no whole lines, N * size not a multiple of 128 bytes, share lines between
  // instructions and are streamed all the same.)
  constexpr int CACHE = C::WTN < 64 ? 0 : 2;
  static_assert(NIT % B == 0, "batch must divide the passes");
  const int cc = lane % CH, rl = lane / CH;
  // (A loop in the code too: unrolled, the ends of a 256x256 tile are 50 KB of instructions, and with the main loop they no longer fit
  // the instruction cache of 64 KB that two units share: us, unrolled / not, 4096x8192x3584 251 / 242.  On a resident grid, whose units are
  // out of step, unrolled is faster: 8192x12288x1536 428 / 436; and so is it with small tiles, whose code fits: 128x256x256 fp32 5.9 / 6.1.
  // Without peers to read: unrolled ahead in one round of tiles (ag 768x8192x1536 25.9 / 26.1, write-only 768x8192x1536 27.4 / 27.6), behind
  // in several (write-only 5440x8192x1536 156 / 145, 5336x4608x6144 277 / 272).)
  constexpr int UNROLL = RESIDENT || C::BM * C::BN < 128 * 128 ? NIT / B : 1;
#pragma unroll UNROLL
  for (int it0 = 0; it0 < NIT; it0 += B) {
    u32x4 w[B][NP > 0 ? NP : 1][LPP];
    bool ok[B][LPP];
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int row = row_base + (it0 + b) * RPP + rl;
#pragma unroll
      for (int l = 0; l < LPP; ++l) {
        const int col = col_base + piece_col<C, PF32>(cc, l);
        ok[b][l] = !EDGE || (m0 + row < a.M && n0 + col < a.N);
        if (EPI != EPI_RS) continue;
        // a lane outside the matrix gets an offset past the records: zeros, no memory access
        // (tile-relative: row < BM <= 256 and N < 2^21, so the byte offset stays below 2^31)
        const int voff = ok[b][l] ? (int)(((uint32_t)row * (uint32_t)a.N + (uint32_t)col) * (PF32 ? 4u : 2u)) : (int)0x80000000;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
          if constexpr (EARLY) w[b][j][l] = early.w[EarlyPeers<C>::template at<NP, PF32>(pass0 + it0 + b, j, l)];
          else w[b][j][l] = __builtin_amdgcn_raw_buffer_load_b128(pb.r[j], voff, 0, CACHE);
        }
      }
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int r = (it0 + b) * RPP + rl;
      const float4 x = *reinterpret_cast<const float4*>(ep + r * C::EP_STRIDE + piece_col<C, PF32>(cc, 0));
      const float4 y = *reinterpret_cast<const float4*>(ep + r * C::EP_STRIDE + piece_col<C, PF32>(cc, 1));
      float v[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
      if (EPI == EPI_RS) {
#pragma unroll
        for (int j = 0; j < NP; ++j) {
          if (PF32) {
#pragma unroll
            for (int e = 0; e < 4; ++e) { v[e] += __uint_as_float(w[b][j][0][e]); v[4 + e] += __uint_as_float(w[b][j][LPP - 1][e]); }
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) { v[2 * e] += bf16_lo(w[b][j][0][e]); v[2 * e + 1] += bf16_hi(w[b][j][0][e]); }
          }
        }
      }
      if constexpr (PF32) {
#pragma unroll
        for (int l = 0; l < LPP; ++l)
          if (ok[b][l]) store_row4<EPI, NP != 0>(a, lds_outs, m0 + row_base + r, n0 + col_base + piece_col<C, PF32>(cc, l), v + 4 * l);
      } else if (ok[b][0]) {
        store_row8<EPI, NP != 0>(a, lds_outs, m0 + row_base + r, n0 + col_base + cc * 8, v);
      }
    }
    // one batch of peer loads in flight at a time: left alone, the scheduler hoists the loads of
    // later batches up here too and has to spill accumulators to make room for them
    if (EPI == EPI_RS) __builtin_amdgcn_sched_barrier(0);
  }
}

// 32 rows of a wave's accumulators into its staging area (row-major): a lane of a 16x16 block holds four
// consecutive rows of one column.
template <class C>
__device__ __forceinline__ void stage_rows32(float* ep, const f32x4 (&acc)[C::MI][C::NI], int mb, int lane) {
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int ni = 0; ni < C::NI; ++ni)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        ep[(16 * s + 4 * (lane >> 4) + e) * C::EP_STRIDE + ni * 16 + (lane & 15)] = acc[2 * mb + s][ni][e];
  __builtin_amdgcn_wave_barrier();
}

// The whole epilogue of one wave: its accumulators pass through LDS 32 rows at a time.
template <class C, int EPI, bool EDGE, bool PF32, int BATCH, int NP, bool RESIDENT, bool EARLY = false>
__device__ __forceinline__ void epilogue_all(const GemmArgs& a, void* const* lds_outs, float* ep, f32x4 (&acc)[C::MI][C::NI],
                                             int m0, int n0, int lane, int wm, int wn, const EarlyPeers<C>& early = {}) {
  PeerBufs pb;
  if (EPI == EPI_RS && NP > 0 && !EARLY) make_peer_bufs(a, m0, n0, pb);
#pragma unroll
  for (int mb = 0; mb < C::WTM / 32; ++mb) {
    stage_rows32<C>(ep, acc, mb, lane);
    epilogue_block<C, EPI, EDGE, PF32, BATCH, NP, RESIDENT, EARLY>(a, lds_outs, ep, pb, wm * C::WTM + mb * 32, wn * C::WTN, m0, n0, lane,
                                                                   early, mb * (32 / EarlyPeers<C>::RPP));
    __builtin_amdgcn_wave_barrier();
  }
}

// The peers' rows ahead of the main loop: their sum (fp32, ascending rank) is what the accumulators start from, and the end
// of the tile only stores.  The way of epilogue_all backwards: 8 columns per lane -> LDS -> registers.
//
constexpr int PEERS_FIRST_AREA = 128 * 128;      // smallest tile
// Why: reading the peers takes a unit 32 us per 256x256 tile and 7 peers when half of the units do it, 44-50 when all do, and
// the workgroups of a grid all reach the end of their tiles at about the same time.  With half of the tiles
// (peers_first) reading their peers first, one half reads while the other multiplies, from the first tile on and whatever the number of
// rounds.  us per call, 8 ranks, every tile's peers behind its main loop / half of them ahead: 4096x8192x3584 256 / 224, 4096x8192x1536
// 167 / 142, 2048x8192x1024 74 / 61, 1024x8192x1024 42 / 33, 4096x12288x4608 435 / 401, 8192x12288x4608 833 / 797, 1496x5112x3400 85.1 / 84.4.
// 16 ranks: 2048x8192x3584 172 / 144, 1024x8192x1536 71 / 56, 4096x8192x1536 257 / 208, 4096x4608x3584 233 / 201, 832x4608x1448 44 / 38.
// (Four passes' loads in flight instead of two: the same.)
template <class C, bool EDGE, int NP>
__device__ __forceinline__ void sum_peers_first(const GemmArgs& a, float* ep, f32x4 (&acc)[C::MI][C::NI], int m0, int n0, int lane, int wm, int wn) {
  constexpr int CH = C::WTN / 8, RPP = 64 / CH, NIT = 32 / RPP, B = NP <= 3 ? 4 : 2;
  static_assert(NIT % B == 0);
  PeerBufs pb;
  make_peer_bufs(a, m0, n0, pb);
  const int cc = lane % CH, rl = lane / CH;
#pragma unroll
  for (int mb = 0; mb < C::WTM / 32; ++mb) {
#pragma unroll 1
    for (int it0 = 0; it0 < NIT; it0 += B) {
      u32x4 w[B][NP];
#pragma unroll
      for (int b = 0; b < B; ++b) {
        const int row = wm * C::WTM + mb * 32 + (it0 + b) * RPP + rl, col = wn * C::WTN + cc * 8;
        const bool ok = !EDGE || (m0 + row < a.M && n0 + col < a.N);
        const int voff = ok ? (int)(((uint32_t)row * (uint32_t)a.N + (uint32_t)col) * 2u) : (int)0x80000000;
#pragma unroll
        for (int j = 0; j < NP; ++j) w[b][j] = __builtin_amdgcn_raw_buffer_load_b128(pb.r[j], voff, 0, 2);
      }
#pragma unroll
      for (int b = 0; b < B; ++b) {
        float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NP; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) { v[2 * e] += bf16_lo(w[b][j][e]); v[2 * e + 1] += bf16_hi(w[b][j][e]); }
        float* const to = ep + ((it0 + b) * RPP + rl) * C::EP_STRIDE + cc * 8;
        *reinterpret_cast<float4*>(to) = make_float4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<float4*>(to + 4) = make_float4(v[4], v[5], v[6], v[7]);
      }
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int ni = 0; ni < C::NI; ++ni)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc[2 * mb + s][ni][e] = ep[(16 * s + 4 * (lane >> 4) + e) * C::EP_STRIDE + ni * 16 + (lane & 15)];
    __builtin_amdgcn_wave_barrier();
  }
}
// Which half follows from where a tile lies in the result, not from when it is visited: the bits of a result depend neither on the
// rank nor on the flags that change the order of visits.  Every second column of tiles, or, where a slice is two tiles high or more
// (a die then walks down the rows of a slice), every second row.  us, columns / rows: 1024x8192x1024 33.5 / 35.7, 16 ranks 1024x8192x1536
// 55.9 / 60.9, 1152x12288x2048 87.8 / 93.6, 768x12288x2048 66.4 / 72.1, but 1496x5112x3400 85.0 / 81.7; the other side, slices of two tiles
// or more: 4096x8192x3584 229.8 / 227.1, 8192x3584x1536 147.2 / 136.8, 8192x1536x6144 221.7 / 204.2, 4 ranks 4096x1536x4608 77.4 / 66.4.
// (Neighbours in both directions in turn is behind one of the two everywhere: tiles that share a panel of B or A part company.  By place in
// the order of visits, every second group of eight tiles: the same times where a slice's tiles fill the dies evenly, 3-10 % behind
// where they do not: 3000x3584x5120 150.4 / 137.4, 1280x4608x1536 39.2 / 35.7, 6144x3072x2048 133.5 / 123.9.)
template <class C, int EPI>
__device__ __forceinline__ bool takes_peers_first(const GemmArgs& a, int mt, int nt, bool is_split) {
  return EPI == EPI_RS && C::BM * C::BN >= PEERS_FIRST_AREA && a.tm.peers_first && !is_split && ((a.tm.peers_first == 2 ? mt : nt) & 1);
}

// ---- AllGather copy pieces --------------------------------------------------------------------
// A communication tile is moved in `pieces` pieces; piece w is what workgroup w of a grid of
// `pieces` workgroups of 256 threads touches in a grid-stride loop over 16-byte vectors.  The copy
// driver's workgroup w normally moves piece w of every tile; a GEMM workgroup that would otherwise
// only wait may take pieces nobody has claimed yet.  Either way the piece is claimed first (a
// compare-and-swap of the call's id into the piece's claim word), moved, and counted in; whoever
// counts in last sets the tile's signal (SetSignal of Alg. 3).

// DEPTH vectors per thread in flight (32 made the plain chunk copy slower: 60 against 24 us for 58.7 MB);
// the last batch is predicated, not walked one vector (one memory round trip) at a time.
//
// The sources are packed; the gathered matrix may have a row pitch.  Vector i of a communication
// tile then goes to row i / kv, place i % kv, counted from the tile's first row.
struct AggPitch {
  uint32_t kv, pitch_v;      // 16-byte vectors per row; from one row to the next
  __device__ __forceinline__ bool packed() const { return kv == pitch_v; }
};
__device__ __forceinline__ AggPitch agg_pitch(const GemmArgs& a) { return AggPitch{(uint32_t)a.K / 8u, (uint32_t)a.lda / 8u}; }
// first vector of communication tile f in the gathered matrix
__device__ __forceinline__ uint4* agg_tile(const GemmArgs& a, int f) {
  return reinterpret_cast<uint4*>(const_cast<__bf16*>(a.A)) + (unsigned long long)f * a.rows_per_signal * ((unsigned long long)a.lda / 8);
}
template <bool PITCHED>
__device__ __forceinline__ unsigned long long agg_index(const AggPitch& g, unsigned long long i) {
  if (!PITCHED) return i;
  const uint32_t j = (uint32_t)i;          // a tile has fewer than 2^28 vectors
  return (unsigned long long)(j / g.kv) * g.pitch_v + j % g.kv;
}

template <int DEPTH, bool PITCHED>
__device__ __forceinline__ void copy_piece_as(const uint4* __restrict__ src, uint4* __restrict__ dst, unsigned long long tile_vec,
                                              int piece, int pieces, int tid, const AggPitch& g) {
  const unsigned long long stride = (unsigned long long)pieces * 256;
  for (unsigned long long i = (unsigned long long)piece * 256 + tid; i < tile_vec; i += DEPTH * stride) {
    u32x4 v[DEPTH];
#pragma unroll
    for (int u = 0; u < DEPTH; ++u)
      if (i + u * stride < tile_vec) v[u] = ld_stream(src + i + u * stride);
#pragma unroll
    for (int u = 0; u < DEPTH; ++u)
      if (i + u * stride < tile_vec) store_through(dst + agg_index<PITCHED>(g, i + u * stride), v[u]);
  }
}
template <int DEPTH = 16>
__device__ __forceinline__ void copy_piece(const uint4* __restrict__ src, uint4* __restrict__ dst, unsigned long long tile_vec,
                                           int piece, int pieces, int tid, const AggPitch& g) {
  if (g.packed()) copy_piece_as<DEPTH, false>(src, dst, tile_vec, piece, pieces, tid, g);       // (uniform)
  else copy_piece_as<DEPTH, true>(src, dst, tile_vec, piece, pieces, tid, g);
}

// A piece of at most COPY_DEPTH * 256 vectors in two halves: the loads, and, once the piece is known
// to be the caller's, the stores.  The loads touch only the source, so they can be on their way
// while the claim is.
constexpr int COPY_DEPTH = 16;
__device__ __forceinline__ void load_piece(const uint4* __restrict__ src, unsigned long long tile_vec, int piece, int pieces,
                                           int tid, u32x4 (&v)[COPY_DEPTH]) {
  const unsigned long long stride = (unsigned long long)pieces * 256;
  const unsigned long long i = (unsigned long long)piece * 256 + tid;
#pragma unroll
  for (int u = 0; u < COPY_DEPTH; ++u) {
    v[u] = u32x4{0, 0, 0, 0};
    if (i + u * stride < tile_vec) v[u] = ld_stream(src + i + u * stride);
  }
}
template <bool PITCHED>
__device__ __forceinline__ void store_piece_as(uint4* __restrict__ dst, unsigned long long tile_vec, int piece, int pieces,
                                               int tid, const u32x4 (&v)[COPY_DEPTH], const AggPitch& g) {
  const unsigned long long stride = (unsigned long long)pieces * 256;
  const unsigned long long i = (unsigned long long)piece * 256 + tid;
#pragma unroll
  for (int u = 0; u < COPY_DEPTH; ++u)
    if (i + u * stride < tile_vec) store_through(dst + agg_index<PITCHED>(g, i + u * stride), v[u]);
}
__device__ __forceinline__ void store_piece(uint4* __restrict__ dst, unsigned long long tile_vec, int piece, int pieces,
                                            int tid, const u32x4 (&v)[COPY_DEPTH], const AggPitch& g) {
  if (g.packed()) store_piece_as<false>(dst, tile_vec, piece, pieces, tid, v, g);               // (uniform)
  else store_piece_as<true>(dst, tile_vec, piece, pieces, tid, v, g);
}

// true if the caller now owns the piece.  One exchange, one round trip: whoever swaps the call's id
// in first sees something else come back; anyone later swaps the id for itself.
__device__ __forceinline__ bool claim_piece(uint32_t* claim, uint32_t call_id) {
  return __hip_atomic_exchange(claim, call_id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != call_id;
}

// Communication tile f has arrived: its signal is set, or, for a tile of a local chunk that the grid moves (its signal is
// preset to 1 throughout), all of its pieces have been counted in.  The last workgroup past its wait clears those counts.
//
// The local chunk used to be put in place by a kernel of its own ahead of the grid: a launch, its drain and 400 KB..6 MB of
// copy that nothing overlapped with (ag 200 x 3584 x 8192 with the chunk in a buffer of its own: 39.5 us per call with it, 37.1
// with the grid moving it; 3000 x 3584 x 8192 185 -> 175 us).
__device__ __forceinline__ bool moved_local(const GemmArgs& a, int f) { return a.copy_local && f >= a.sig_local_lo && f < a.sig_local_hi; }
__device__ __forceinline__ bool tile_arrived(const GemmArgs& a, int f) {
  const bool local = moved_local(a, f);
  const uint32_t v = __hip_atomic_load(local ? a.copy_counters + f : a.signals + f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  return local ? v == (uint32_t)a.copy_pieces : v != 0u;
}
// `n` of the `pieces` pieces of tile f are in place (their stores acknowledged): count them in, set the signal if they were the
// tile's last.  One thread calls this.
__device__ __forceinline__ void count_pieces_in(uint32_t* counter, uint32_t* signal, int pieces, int n, bool local) {
  if (n == pieces) {
    // the whole tile was this workgroup's (a small transfer: one piece per tile): nobody else counts, no round trip
    if (local) __hip_atomic_store(counter, (uint32_t)pieces, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else __hip_atomic_store(signal, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  } else {
    const uint32_t prev = __hip_atomic_fetch_add(counter, (uint32_t)n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!local && prev + (uint32_t)n == (uint32_t)pieces) {
      __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next call
      __hip_atomic_store(signal, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
}

// After the stores of `n` pieces of one tile: wait until they are acknowledged, then count the pieces in.
// All threads of the workgroup call this.
__device__ __forceinline__ void finish_pieces(uint32_t* counter, uint32_t* signal, int pieces, int n, bool local = false) {
  __builtin_amdgcn_s_waitcnt(0x0F70);     // vmcnt(0): this wave's write-through stores are acknowledged
  __syncthreads();
  if (threadIdx.x == 0) count_pieces_in(counter, signal, pieces, n, local);
  // Callers loop: without a barrier here, this one-thread block and the one-thread block that
  // opens the caller's next iteration (a claim, a counter fetch) are adjacent across the back
  // edge, and the compiler has been seen to merge them into one divergent region that the other
  // lanes of the first wave skip on their way to the next iteration's barrier, which they then
  // reach without thread 0 (and read what it has not written yet).
  __syncthreads();
}

// The copy driver's workgroups count themselves in when they start: word 0 of `started` only ever
// grows.  Word 1 is what word 0 read before the current call's driver was launched; the last GEMM
// workgroup past its wait advances it by the driver's size for the next call (by then every driver
// workgroup of this call has been or will be counted, and the next call starts after the driver
// has finished).  Nothing is ever reset, so a workgroup that starts late cannot spoil a count.
__device__ __forceinline__ bool driver_fully_started(const uint32_t* started, int workgroups) {
  if (workgroups == 0) return false;
  const uint32_t total = __hip_atomic_load(started, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint32_t base = __hip_atomic_load(started + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return total - base >= (uint32_t)workgroups;
}

// The id that marks a piece as taken in this call.  With a copy kernel beside the grid the host
// hands out a fresh one per call.  Without, it is the number of such calls that have completed on
// this workspace (the last workgroup past its wait counts the call in, when every workgroup has
// read the old value: a workgroup only reads it before it is past its own wait), so a call
// recorded in a graph gets a new id on every replay.
__device__ __forceinline__ uint32_t transfer_call_id(const GemmArgs& a) {
  if (a.copy_call_id != 0u) return a.copy_call_id;
  return 0x80000000u | __hip_atomic_load(a.copy_call_seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// No driver: the first copy_owner_wgs workgroups of the grid share the transfer out among
// themselves by index, each moving its pieces in transfer order before it looks at its own
// signals, whatever its own tile needs.  A piece still goes through the claim table (one word per
// piece, so nobody contends), which lets any waiting workgroup take over the piece of an owner
// that has not been given a compute unit yet.  The first wave claims up to 64 pieces in one round
// trip and, when they have been moved, counts them in in another.  `lds` is 4 ints shared by the
// workgroup; `lds_srcs` holds the chunk sources by rank (written before, not yet synchronised).
__device__ __forceinline__ void transfer_own_pieces(const GemmArgs& a, int* lds, void* const* lds_srcs) {
  if ((int)blockIdx.x >= a.copy_owner_wgs) return;
  const int tid = threadIdx.x;
  const int ctpc = a.n_signals / a.R;
  const int total = (a.copy_n_tiles - a.copy_defer_tiles) * a.copy_pieces;
  const int G = a.copy_owner_wgs;
  if (total <= G && a.copy_tile_vec <= (unsigned long long)a.copy_pieces * 256 * COPY_DEPTH) {
    // A small transfer (decode): at most one piece per owner, moved in one pass.  Then the whole
    // call waits for a chain of memory round trips, so they overlap where they can: the piece is
    // loaded while the call's id and then the claim are on their way.
    const int g = (int)blockIdx.x;
    if (g >= total) return;
    __syncthreads();                       // lds_srcs
    const uint32_t call_id = transfer_call_id(a);
    const int j = g / a.copy_pieces, piece = g - j * a.copy_pieces;
    const int chunk = (int)((a.copy_order4 >> (4 * (j / ctpc))) & 15), t = j % ctpc;
    const int f = chunk * ctpc + t;
    const uint4* src = static_cast<const uint4*>(lds_srcs[chunk]) + (unsigned long long)t * a.copy_tile_vec;
    uint4* dst = agg_tile(a, f);
    u32x4 v[COPY_DEPTH];
    load_piece(src, a.copy_tile_vec, piece, a.copy_pieces, tid, v);
    if (tid == 0) lds[2] = claim_piece(a.copy_claims + (size_t)f * a.copy_pieces + piece, call_id) ? 1 : 0;
    __syncthreads();
    if (lds[2]) {
      store_piece(dst, a.copy_tile_vec, piece, a.copy_pieces, tid, v, agg_pitch(a));
      finish_pieces(a.copy_counters + f, a.signals + f, a.copy_pieces, 1, moved_local(a, f));
    }
    return;
  }
  const uint32_t call_id = transfer_call_id(a);
  for (int base = (int)blockIdx.x; base < total; base += 64 * G) {
    if (tid < 64) {
      const int g = base + tid * G;
      bool mine = false;
      if (g < total) {
        const int j = g / a.copy_pieces;
        const int f = (int)((a.copy_order4 >> (4 * (j / ctpc))) & 15) * ctpc + j % ctpc;
        mine = claim_piece(a.copy_claims + (size_t)f * a.copy_pieces + (g - j * a.copy_pieces), call_id);
      }
      const unsigned long long won = __ballot(mine);
      if (tid == 0) { lds[1] = (int)(uint32_t)won; lds[2] = (int)(uint32_t)(won >> 32); }
    }
    __syncthreads();
    const unsigned long long won = (unsigned long long)(uint32_t)lds[1] | ((unsigned long long)(uint32_t)lds[2] << 32);
    for (unsigned long long rest = won; rest != 0; rest &= rest - 1) {
      const int g = base + __builtin_ctzll(rest) * G;
      const int j = g / a.copy_pieces, piece = g - j * a.copy_pieces;
      const int chunk = (int)((a.copy_order4 >> (4 * (j / ctpc))) & 15), t = j % ctpc;
      const int f = chunk * ctpc + t;
      const uint4* src = static_cast<const uint4*>(lds_srcs[chunk]) + (unsigned long long)t * a.copy_tile_vec;
      copy_piece(src, agg_tile(a, f), a.copy_tile_vec, piece, a.copy_pieces, tid, agg_pitch(a));
    }
    // count the pieces in, all at once: lane l of the first wave for the piece it claimed
    __builtin_amdgcn_s_waitcnt(0x0F70);     // vmcnt(0): this wave's write-through stores are acknowledged
    __syncthreads();
    if (tid < 64 && ((won >> tid) & 1)) {
      const int g = base + tid * G;
      const int j = g / a.copy_pieces;
      const int f = (int)((a.copy_order4 >> (4 * (j / ctpc))) & 15) * ctpc + j % ctpc;
      count_pieces_in(a.copy_counters + f, a.signals + f, a.copy_pieces, 1, moved_local(a, f));
    }
    __syncthreads();
  }
}

// The transfer carried by the GEMM's own waves (Sec. 3.2: the tiles whose data has arrived compute
// while the rest is still on its way).  A workgroup of the first round owns piece `blockIdx.x` of
// every deferred communication tile and moves it in 16-byte vectors per thread, tile after tile in
// transfer order: inside its main loop two vectors per K slab (the loads at the end of a slab, the
// stores of what was loaded two slabs earlier at the start of one, so that neither is ever waited
// for), and in batches while it still waits for its own signals.  All addressing goes through
// buffer resources whose size is the tile's (or zero for a workgroup with nothing to move, a tile
// taken over by somebody else, or when all tiles are done), so a lane past the end, and everything
// such a workgroup issues, is dropped by the range check: the loops have one shape for every
// workgroup and no branch around a memory access.
// With a pace (the transfer stands for a link of a given rate) the data still moves as fast as the
// loops take it, but a tile is counted in, and so its signal set, no earlier than the link would
// have delivered it: tile number i of the transfer order (i + 1) * pace_ticks after the workgroup
// started (the workgroups of a first round start within a microsecond of each other).
struct SideCopy {
  __amdgpu_buffer_rsrc_t rs, rd;     // source chunk / its place in the gathered matrix, for the tile being loaded / stored
  uint32_t first, ld_off, st_off;    // this lane's first vector of a piece, next to load, next to store (byte offsets in the tile)
  uint32_t stride;                   // bytes between a lane's vectors
  int n_tiles, n_steps, pos0;        // deferred tiles; vectors per thread and tile; transfer position of the first of them
  int ld_t, ld_s, st_t, st_s;        // cursors: tile and step
  int fin_t;                         // tiles counted in so far
  uint32_t mine;                     // bit t: this workgroup claimed its piece of deferred tile t
  unsigned long long t0, pace;       // start clock; 100 MHz ticks per tile (0: unpaced)
  int* slot;                         // one int of LDS: whatever depends on the clock is decided by thread 0 and read from here

  // deferred tile t -> its signal index (= communication tile index in the gathered matrix) and chunk
  __device__ __forceinline__ void locate(const GemmArgs& a, int t, int& f, int& chunk, int& sub) const {
    const int ctpc = a.n_signals / a.R;
    const int pos = pos0 + t;
    chunk = (int)((a.copy_order4 >> (4 * (pos / ctpc))) & 15);
    sub = pos % ctpc;
    f = chunk * ctpc + sub;
  }
  __device__ __forceinline__ unsigned records(const GemmArgs& a, int t) const {
    return (t < n_tiles && ((mine >> t) & 1u)) ? (unsigned)(a.copy_tile_vec * 16ull) : 0u;
  }
  __device__ __forceinline__ void set_src(const GemmArgs& a, void* const* lds_srcs, int t) {
    int f = 0, chunk = 0, sub = 0;
    if (t < n_tiles) locate(a, t, f, chunk, sub);
    const uint64_t addr = reinterpret_cast<uint64_t>(lds_srcs[chunk]) + (unsigned long long)sub * a.copy_tile_vec * 16ull;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)addr), hi = __builtin_amdgcn_readfirstlane((uint32_t)(addr >> 32));
    rs = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(((uint64_t)hi << 32) | lo), 0, (int)records(a, t), 0x00027000);
  }
  __device__ __forceinline__ void set_dst(const GemmArgs& a, int t) {
    int f = 0, chunk = 0, sub = 0;
    if (t < n_tiles) locate(a, t, f, chunk, sub);
    unsigned char* base = reinterpret_cast<unsigned char*>(const_cast<__bf16*>(a.A)) + (unsigned long long)f * a.copy_tile_vec * 16ull;
    rd = __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)records(a, t), 0x00027000);
  }

  // Claims this workgroup's pieces (one exchange per deferred tile, all in one round trip) and sets
  // the cursors up.  `lds` is one int shared by the workgroup, kept for this object.  All threads call this.
  __device__ __forceinline__ void begin(const GemmArgs& a, int* lds, void* const* lds_srcs) {
    const int tid = threadIdx.x;
    slot = lds;
    t0 = wall_clock64();
    pace = a.copy_pace_ticks;
    n_tiles = 0; mine = 0u; n_steps = a.copy_defer_steps;
    pos0 = a.copy_n_tiles - a.copy_defer_tiles;
    if (a.copy_defer_tiles > 0 && (int)blockIdx.x < a.copy_pieces && (int)blockIdx.x < a.copy_owner_wgs) n_tiles = a.copy_defer_tiles;
    if (n_tiles > 0) {           // (uniform)
      if (tid < 64) {
        bool won = false;
        if (tid < n_tiles) {
          int f, chunk, sub;
          locate(a, tid, f, chunk, sub);
          won = claim_piece(a.copy_claims + (size_t)f * a.copy_pieces + blockIdx.x, transfer_call_id(a));
        }
        const unsigned long long w = __ballot(won);
        if (tid == 0) *lds = (int)(uint32_t)w;
      }
      __syncthreads();
      mine = (uint32_t)__builtin_amdgcn_readfirstlane(*lds);
      __syncthreads();
    }
    first = ((uint32_t)blockIdx.x * 256u + (uint32_t)tid) * 16u;
    stride = (uint32_t)a.copy_pieces * 256u * 16u;
    ld_off = st_off = first;
    ld_t = ld_s = st_t = st_s = 0;
    fin_t = 0;
    if (mine == 0u) fin_t = n_tiles = 0;
    set_src(a, lds_srcs, 0);
    set_dst(a, 0);
  }
  __device__ __forceinline__ bool pending() const { return fin_t < n_tiles; }         // something left to move or to count in
  __device__ __forceinline__ bool all_stored() const { return st_t >= n_tiles; }
  // Is there a tile whose stores are all issued and which may be counted in now?  Reads the clock:
  // different waves may get different answers, so only thread 0's counts (see maybe_finish).
  __device__ __forceinline__ bool due() const {
    if (fin_t >= st_t) return false;
    if (pace == 0ull) return st_t >= n_tiles;        // unpaced: everything is counted in together, at the end
    return wall_clock64() - t0 >= (unsigned long long)(pos0 + fin_t + 1) * pace;
  }
  __device__ __forceinline__ bool may_be_due() const { return fin_t < st_t && (pace != 0ull || st_t >= n_tiles); }   // (uniform)

  __device__ __forceinline__ u32x4 load(const GemmArgs& a, void* const* lds_srcs) {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)ld_off, 0, 2);      // streamed: not kept in the caches
    ld_off += stride;
    if (++ld_s == n_steps) { ld_s = 0; ld_off = first; set_src(a, lds_srcs, ++ld_t); }
    return v;
  }
  __device__ __forceinline__ void store(const GemmArgs& a, const u32x4& v) {
    __builtin_amdgcn_raw_buffer_store_b128(v, rd, (int)st_off, 0, 16);                 // device scope: written through the die's L2
    st_off += stride;
    if (++st_s == n_steps) { st_s = 0; st_off = first; set_dst(a, ++st_t); }
  }
  // Counts in the tiles that are due (see due()).  A tile whose last piece this was gets its signal
  // (SetSignal of Alg. 3).  All threads call this.
  __device__ __forceinline__ void finish(const GemmArgs& a) {
    __builtin_amdgcn_s_waitcnt(0x0F70);     // vmcnt(0): this wave's write-through stores are acknowledged
    __syncthreads();
    if (threadIdx.x == 0) {
      int upto = fin_t;
      const int stored = st_t < n_tiles ? st_t : n_tiles;
      if (pace == 0ull) {
        upto = stored;
      } else {
        const unsigned long long now = wall_clock64() - t0;
        while (upto < stored && now >= (unsigned long long)(pos0 + upto + 1) * pace) ++upto;
      }
      for (int t = fin_t; t < upto; ++t) {
        if (!((mine >> t) & 1u)) continue;
        int f, chunk, sub;
        locate(a, t, f, chunk, sub);
        count_pieces_in(a.copy_counters + f, a.signals + f, a.copy_pieces, 1, false);      // (deferred tiles are remote)
      }
      *slot = upto;
    }
    __syncthreads();
    fin_t = __builtin_amdgcn_readfirstlane(*slot);
    __syncthreads();                        // the slot is free again
  }
  // finish() if thread 0 finds a tile due.  All threads call this.
  __device__ __forceinline__ void maybe_finish(const GemmArgs& a) {
    if (!may_be_due()) return;
    __syncthreads();
    if (threadIdx.x == 0) *slot = due() ? 1 : 0;
    __syncthreads();
    const int go = __builtin_amdgcn_readfirstlane(*slot);
    __syncthreads();
    if (go) finish(a);
  }
  // While the workgroup has nothing else to do (it waits for its own signals, or its main loop is
  // over): a batch of vectors, loads first.  All threads call this.
  __device__ __forceinline__ void pump(const GemmArgs& a, void* const* lds_srcs) {
    constexpr int BATCH = 8;
    u32x4 v[BATCH];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) v[u] = load(a, lds_srcs);
#pragma unroll
    for (int u = 0; u < BATCH; ++u) store(a, v[u]);
  }
  // Everything that is left, now: the rest of the vectors, then the tiles as they become due.
  // All threads call this.
  __device__ __forceinline__ void drain(const GemmArgs& a, void* const* lds_srcs) {
    while (ld_t < n_tiles) pump(a, lds_srcs);
    while (pending()) {
      maybe_finish(a);
      if (pending()) __builtin_amdgcn_s_sleep(16);
    }
  }
};

// Are the signals covering rows [m0, m1) all set?  One poll by the first wave, the answer handed to
// everybody through `slot` (one int of LDS).  All threads call this.
__device__ __forceinline__ bool signals_all_set(const GemmArgs& a, int m0, int m1, int* slot) {
  const int f0 = m0 / a.rows_per_signal, f1 = (m1 - 1) / a.rows_per_signal;
  const int nf = f1 - f0 + 1;
  if (threadIdx.x < 64) {
    bool any = false;
    for (int base = 0; base < nf; base += 64) {
      const bool unset = base + (int)threadIdx.x < nf && !tile_arrived(a, f0 + base + (int)threadIdx.x);
      any = any || __ballot(unset) != 0ull;
    }
    if (threadIdx.x == 0) *slot = any ? 0 : 1;
  }
  __syncthreads();
  const int all = __builtin_amdgcn_readfirstlane(*slot);
  __syncthreads();
  return all != 0;
}

// WaitSignal (Alg. 2).  The first wave polls the signals covering rows [m0, m1) with coherent
// loads, one lane per signal; when all are set, the workgroup barrier hands that to the other waves.
// A workgroup that finds a signal missing
// and unclaimed pieces among the tiles it waits for claims and moves such pieces itself (at once;
// beside a paced driver only while part of that driver has not been given a compute unit), picking
// them by a hash that depends on its index so that the workgroups of a grid spread over the pieces
// instead of racing for the same one: without that, a mover that never gets a compute unit (the
// GEMM grid may have taken them all, and its waiting workgroups do not leave) would stall the grid
// for good.  Bounded: past `timeout_ticks` the tile is given up and the status block says so.  A
// workgroup never looks at the signals again after this, so the last workgroup of the grid to get
// here puts the signal array back into its preset state for the next call (the reset "after the
// GEMM" of Sec. 4.3, without a separate launch).
// `lds` is 4 ints shared by the workgroup; `lds_srcs` holds the chunk sources by rank.
__device__ __forceinline__ bool wait_signals(const GemmArgs& a, int m0, int m1, int* lds, void* const* lds_srcs) {
  const int tid = threadIdx.x;
  const int f0 = m0 / a.rows_per_signal, f1 = (m1 - 1) / a.rows_per_signal;
  const unsigned long long t0 = wall_clock64();
  enum : int { ARRIVED = 1, GIVE_UP = 2, HELP = 3, SELF_SERVE = 4 };
  const int nf = f1 - f0 + 1;
  // The search for a piece covers a window of at most 4096 pieces (12 index bits in the key below),
  // starting at the first tile whose signal is still missing, so it moves on as tiles complete.
  const int window_tiles = a.copy_pieces > 0 ? (4096 / a.copy_pieces < nf ? 4096 / a.copy_pieces : nf) : 0;
  uint32_t salt = (uint32_t)blockIdx.x * 0x9E3779B9u;      // varies per workgroup and per attempt
  int dead_w0 = -1;                                        // window start at which a search found nothing left to take
  bool ok = true;
  uint32_t call_id = 0u;                                   // fetched when a piece is first looked for
  bool have_call_id = false;
  for (;;) {
    if (tid < 64) {
      // the first wave polls, one signal per lane: one memory round trip per 64 signals, however
      // many the tile waits for (a decode tile waits for all of them)
      int st;
      int first_missing = 0;
      for (int polls = 0;; ++polls) {
        first_missing = -1;
        for (int base = 0; base < nf && first_missing < 0; base += 64) {
          const bool unset = base + tid < nf && !tile_arrived(a, f0 + base + tid);
          const unsigned long long missing = __ballot(unset);
          if (missing != 0) first_missing = f0 + base + __builtin_ctzll(missing);
        }
        if (first_missing < 0) { st = ARRIVED; break; }
        if (wall_clock64() - t0 > a.timeout_ticks) {
          if (tid == 0 && atomicCAS(a.status, 0u, (uint32_t)FLUX_ERR_TIMEOUT) == 0u) a.status[1] = (uint32_t)first_missing;
          st = GIVE_UP;
          break;
        }
        if (a.copy_pieces > 0 && first_missing != dead_w0 &&
            (a.copy_eager || (polls >= 8 && !driver_fully_started(a.started_counter, a.copy_driver_wgs)))) {
          st = HELP;
          break;
        }
        if (a.copy_pieces == 0 && a.self_serve_ticks != 0u && wall_clock64() - t0 > (unsigned long long)a.self_serve_ticks) {
          st = SELF_SERVE;
          break;
        }
        __builtin_amdgcn_s_sleep(16);
      }
      if (tid == 0) {
        lds[0] = st;
        lds[1] = 0x7fffffff;
        lds[3] = first_missing;
      }
    }
    __syncthreads();
    // (read as scalars: the compiler takes a value loaded from LDS for one that may differ between lanes,
    // and everything changed inside a loop left under such a value, like the transfer's cursors, with it)
    const int st = __builtin_amdgcn_readfirstlane(lds[0]);
    const int w0 = __builtin_amdgcn_readfirstlane(lds[3]);                // first tile of the search window
    __syncthreads();                    // everyone has read them before the first wave can write again
    if (st == ARRIVED) break;
    if (st == GIVE_UP) { ok = false; break; }
    if (st == SELF_SERVE) {
      // The transfers of a driver that takes no pieces (a library copy per tile with a stream write
      // of its signal) run as kernels of their own on this chip: when the grid's waiting workgroups
      // hold every compute unit, those kernels cannot start and the signals never come.  A workgroup
      // that has waited long enough therefore fetches the rows of its own tile from the chunk
      // sources itself and goes on without its signals.  The driver may write the same bytes to the
      // same places at the same time: harmless.  (The host puts the signals back after the join in
      // this form, since a driver that was overtaken sets some of them after the grid is done.)
      const unsigned long long vec_per_row = (unsigned long long)a.K / 8;
      const unsigned long long nvec = (unsigned long long)(m1 - m0) * vec_per_row;
      for (unsigned long long v = tid; v < nvec; v += 4 * blockDim.x) {
        u32x4 x[4];
        const uint4* src[4];
        uint4* dst[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const unsigned long long vv = v + (unsigned long long)u * blockDim.x;
          const int row = m0 + (int)((vv < nvec ? vv : 0) / vec_per_row);
          const unsigned long long col = (vv < nvec ? vv : 0) % vec_per_row;
          const int chunk = row / a.S;
          src[u] = static_cast<const uint4*>(lds_srcs[chunk]) + (unsigned long long)(row - chunk * a.S) * vec_per_row + col;
          dst[u] = reinterpret_cast<uint4*>(const_cast<__bf16*>(a.A)) + (unsigned long long)row * ((unsigned long long)a.lda / 8) + col;
          if (vv < nvec) x[u] = ld_stream(src[u]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (v + (unsigned long long)u * blockDim.x < nvec && src[u] != dst[u]) store_through(dst[u], x[u]);
      }
      __builtin_amdgcn_s_waitcnt(0x0F70);     // vmcnt(0): the stores are acknowledged
      __syncthreads();
      break;
    }
    // One of the unclaimed pieces among the tiles of the window, picked by a hash that differs per
    // workgroup and attempt: workgroups that wait for the same tiles then rarely go for the same
    // piece (taking "the first free one" would make them queue up behind each other).  A local
    // chunk that is in place already is not copied by anyone, its signals are preset.
    if (!have_call_id) { call_id = transfer_call_id(a); have_call_id = true; }
    const int wt = f1 - w0 + 1 < window_tiles ? f1 - w0 + 1 : window_tiles;
    const int total = wt * a.copy_pieces;
    salt = salt * 1664525u + 1013904223u;
    for (int i = tid; i < total; i += blockDim.x) {
      const int f = w0 + i / a.copy_pieces;
      if (!a.copy_local && f >= a.sig_local_lo && f < a.sig_local_hi) continue;
      if (__hip_atomic_load(a.copy_claims + (size_t)f * a.copy_pieces + i % a.copy_pieces, __ATOMIC_RELAXED,
                            __HIP_MEMORY_SCOPE_AGENT) != call_id) {
        const uint32_t h = ((uint32_t)i * 2654435761u) ^ salt;
        atomicMin(&lds[1], (int)(((h >> 14) << 12) | (uint32_t)i));   // 18 hash bits above the 12-bit index: below the "none" value
      }
    }
    __syncthreads();
    const int key = lds[1];
    if (key != 0x7fffffff) {
      const int i = key & 4095;
      const int f = w0 + i / a.copy_pieces, piece = i % a.copy_pieces;
      if (tid == 0) lds[2] = claim_piece(a.copy_claims + (size_t)f * a.copy_pieces + piece, call_id) ? 1 : 0;
      __syncthreads();
      if (lds[2]) {
        const int ctpc = a.n_signals / a.R;
        const uint4* src = static_cast<const uint4*>(lds_srcs[f / ctpc]) + (unsigned long long)(f % ctpc) * a.copy_tile_vec;
        copy_piece(src, agg_tile(a, f), a.copy_tile_vec, piece, a.copy_pieces, tid, agg_pitch(a));
        finish_pieces(a.copy_counters + f, a.signals + f, a.copy_pieces, 1, moved_local(a, f));
      }
    } else {
      dead_w0 = w0;                     // every piece of this window is in the hands of a workgroup that is running
    }
    __syncthreads();                    // lds[1], lds[2] are rewritten in the next round
  }
  if (tid == 0) {
    // Acquire.  The rows were written through to memory (write-through stores of a workgroup or of
    // the copy kernel, or a DMA engine) and acknowledged before their signal was set, and the poll
    // that saw the signal has returned, so loads issued from here on come after them.  What is
    // left to rule out is a stale copy in this die's L2 or this unit's L1.  Both are emptied when
    // a kernel starts, and nobody reads a row of the gathered matrix before its signal, so such a
    // copy can only exist if a cache line holds rows of two communication tiles.  Only then is
    // the die's L2 invalidated here: doing that costs one to two microseconds per workgroup and
    // throws out the operand panels the die's other workgroups are sharing.
    if (a.acquire_l2) __atomic_thread_fence(__ATOMIC_ACQUIRE);   // system scope
    else __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    // count this workgroup in: its leaf first, the root if that completed the leaf
    const uint32_t leaf = blockIdx.x % DONE_LEAVES;
    const uint32_t quota = (gridDim.x - leaf + DONE_LEAVES - 1) / DONE_LEAVES;
    const uint32_t leaves = gridDim.x < (uint32_t)DONE_LEAVES ? gridDim.x : (uint32_t)DONE_LEAVES;
    uint32_t* leaf_counter = a.done_counter + (WS_DONELEAF_OFF - WS_DONE_OFF + leaf * DONE_LEAF_STRIDE) / 4;
    bool last = false;
    if (__hip_atomic_fetch_add(leaf_counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == quota - 1) {
      __hip_atomic_store(leaf_counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next call
      last = __hip_atomic_fetch_add(a.done_counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == leaves - 1;
    }
    if (last) {
      for (int i = 0; i < a.n_signals; ++i)
        __hip_atomic_store(a.signals + i, (i >= a.sig_local_lo && i < a.sig_local_hi) ? 1u : 0u, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
      if (a.copy_local)
        for (int i = a.sig_local_lo; i < a.sig_local_hi; ++i)
          __hip_atomic_store(a.copy_counters + i, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (a.copy_pieces > 0 && a.copy_call_id == 0u)
        __hip_atomic_fetch_add(a.copy_call_seq, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (a.copy_driver_wgs > 0)
        __hip_atomic_fetch_add(a.started_counter + 1, (uint32_t)a.copy_driver_wgs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(a.done_counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  __syncthreads();
  return ok;
}

// Reduce by atomic additions on device memory (Sec. 4.2, "Reduce", first form): the owner's fp32 slice
// already holds what the other ranks have added; every element of the tile is added to it with one
// hardware addition that returns nothing.  The lanes of an instruction take consecutive columns of a
// row, so that an instruction touches two whole cache lines and not sixteen partial ones (with the
// eight-columns-per-lane layout of the other epilogues this form took five times as long).
template <class C, bool EDGE>
__device__ __forceinline__ void epilogue_all_atomic(const GemmArgs& a, void* const* lds_outs, float* ep, f32x4 (&acc)[C::MI][C::NI],
                                                    int m0, int n0, int lane, int wm, int wn) {
  constexpr int W = C::WTN < 64 ? C::WTN : 64;   // columns per instruction
  constexpr int RPI = 64 / W;                    // rows per instruction
  const int c_in = lane % W, r_in = lane / W;
#pragma unroll
  for (int mb = 0; mb < C::WTM / 32; ++mb) {
    stage_rows32<C>(ep, acc, mb, lane);
    for (int r0 = 0; r0 < 32; r0 += RPI) {
      const int r = r0 + r_in;
      const int gm = m0 + wm * C::WTM + mb * 32 + r;
      const int owner = gm / a.S;
      float* row = static_cast<float*>(lds_outs[owner]) + (size_t)(gm - owner * a.S) * a.ldc + n0 + wn * C::WTN;
#pragma unroll
      for (int c0 = 0; c0 < C::WTN; c0 += W) {
        const int c = c0 + c_in;
        if (!EDGE || (gm < a.M && n0 + wn * C::WTN + c < a.N)) unsafeAtomicAdd(row + c, ep[r * C::EP_STRIDE + c]);
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// ---- a K-cut tile finished by all of its parts --------------------------------------------------
// Left to the part that arrives last, the end of a K-cut tile is a chain of round trips of ONE workgroup (all parts' sums
// read back, then the peers' rows, batch after batch) at what one compute unit can pull, while the others are gone:
// 4-8 us of an 18 us kernel (64 x 8192 x 3584, 4 parts, 7 peers), 15 us of 38 (200 x 3584 x 8192, 9 parts).  Where all parts
// surely run at the same time (sk_share, decided on the host), each parks its sums, asks for the peers' rows of its
// share of the tile, waits for the other parts, and finishes that share: one round trip for the
// parts' sums, with the peers' rows already there.
// A share is a range of 16x32 blocks of the tile, numbered wave tile by wave tile; a wave takes one block at a time.
// The sum runs in split order, then peers in rank order, as ever: results do not depend on timing.
// us per call, last part -> shared: rs 64 x 8192 x 3584 24.0 -> 21.5, ag 200 x 3584 x 8192 49.8 -> 40.1, rs 1080 x 408 x 6144
// 48 -> 25, ag 8192 x 4608 x 12288 (its last round's 64 tiles in 4 parts) 754 -> 743.  (Asking for the next block's sums while
// a block is finished made the small calls 0.5-1 us slower: the code of a tail runs once, and every line of it is fetched.)
//
// A part that has not been given a compute unit yet (another kernel holds some) may be waiting for one of these.  So a part
// waits for the others only where all of them have started, and for those that have not about an eighth of the time of its
// main loop (sk_share, set on the host: nothing has to be kept through the main loop); a part that all others gave up on sums the tile alone, as if nothing were
// shared.  Waiting for every part up to the bound stalled calls beside a kernel that holds compute units for as long (us per
// call beside one that holds 4 / 32 / 128 units, every part waited for -> only started ones -> none ever: rs 64 x 2048 x 8192
// 54 / 54 / 72 -> 26 / 26 / 29 -> 23 / 24 / 28, ag 8 x 3584 x 8192 30 / 59 / 73 -> 31 / 31 / 36 -> 28 / 29 / 34).  The start is
// counted after the first slab is there: ahead of it, the addition's round trip comes first (+0.25 us).  The last round of a
// grid whose other tiles are whole is waited for up to the bound: its parts start as those tiles are finished, one by one
// (672 x 12288 x 1536 with 15 fp32 peers 168 us, 214 with the short wait).
//
// The tile's counter word: parts that have arrived in bits [4:0], parts that have seen all arrive in bits [9:5], parts
// that have started their main loop in bits [14:10], parts that gave up waiting in bits [31:16].  Who gives up leaves its
// share to the last to arrive, who reads in its own arrival whose those are.  The last to see the tile complete clears the
// word; every part's start has been counted by then (acknowledged ahead of its arrival).
constexpr uint32_t SK_COUNT = 31u, SK_SEEN_AT = 5, SK_STARTED_AT = 10, SK_GAVE_UP = 1u << 16;
constexpr int SK_SHARE_MAX = 16;                      // parts of a tile whose shares fit the word
static_assert(SK_SHARE_MAX <= 16, "a give-up bit per part, counts of up to 31");
constexpr uint32_t SK_WAIT_TICKS = 10000;             // 100 us: longest wait for a part that has started
constexpr uint32_t SK_START_TICKS = 50;               // 0.5 us: shortest wait for one that has not (a grid is not dispatched at once)

// This part has its first operands and enters its main loop.
__device__ __forceinline__ void part_started(const GemmArgs& a, int tile, int tid) {
  if (tid == 0)
    __hip_atomic_fetch_add(a.sk_counters + sk_counter_index(tile - a.full_tiles), 1u << SK_STARTED_AT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <class C, int EPI, bool EDGE, bool PF32, int NP>
struct SharedFinish {
  static constexpr int LPP = PF32 ? 2 : 1;            // 16-byte loads per peer and lane
  static constexpr int NPA = NP > 0 ? NP : 1;
  static constexpr int BLOCKS_W = C::MI * (C::NI / 2);          // 16x32 blocks of a wave tile
  static constexpr int BLOCKS = (C::NT / 64) * BLOCKS_W;
  static constexpr int STRIDE = 36;                   // floats per staged row: rows stay 16-byte aligned
  static_assert(C::NI % 2 == 0 && 16 * STRIDE <= 32 * C::EP_STRIDE, "a block is staged in a wave's part of the staging area");

  // where this lane's eight columns of block u lie (row and column within the tile)
  static __device__ __forceinline__ void place(int u, int lane, int& row, int& col) {
    const int w = u / BLOCKS_W, v = u % BLOCKS_W;
    row = (w / C::WAVES_N) * C::WTM + (v / (C::NI / 2)) * 16 + lane / 4;
    col = (w % C::WAVES_N) * C::WTN + (v % (C::NI / 2)) * 32 + (lane % 4) * 8;
  }
  // (Not streamed: a block's rows are 64 bytes of bf16, half a line, and another wave takes the other half.  us, streamed / kept: 4
  // layers of 64x8192x3584 with 7 peers 78.8 / 74.5.)
  static __device__ __forceinline__ void load_peers(const GemmArgs& a, const PeerBufs& pb, int u, int m0, int n0, int lane, u32x4 (&w)[NPA][LPP]) {
    int row, col;
    place(u, lane, row, col);
    const bool ok = !EDGE || (m0 + row < a.M && n0 + col < a.N);
    const int voff = ok ? (int)(((uint32_t)row * (uint32_t)a.N + (uint32_t)col) * (PF32 ? 4u : 2u)) : (int)0x80000000;
#pragma unroll
    for (int j = 0; j < NP; ++j)
#pragma unroll
      for (int l = 0; l < LPP; ++l) w[j][l] = __builtin_amdgcn_raw_buffer_load_b128(pb.r[j], voff + 16 * l, 0, 0);
  }
  static __device__ __forceinline__ void block(const GemmArgs& a, void* const* lds_outs, float* ep, int u, int st, int m0, int n0, int lane,
                                               const u32x4 (&w)[NPA][LPP]) {
    constexpr int SC1 = 16;
    constexpr int BLOCK_BYTES = C::BM * C::BN * 4;
    const int wv = u / BLOCKS_W, v = u % BLOCKS_W;
    const int mi = v / (C::NI / 2), ni = v % (C::NI / 2) * 2;
    const int off = ((mi * C::NI + ni) * C::NT + wv * 64 + lane) * 16;
    const bool past = EDGE && m0 + (wv / C::WAVES_N) * C::WTM + mi * 16 + 4 * (lane >> 4) >= a.M;    // (never parked)
    f32x4 sum[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    constexpr int PB = 8;                             // parts whose loads are out together
    for (int s0 = 0; s0 < a.split_k; s0 += PB) {
      u32x4 x[PB][2];
#pragma unroll
      for (int g = 0; g < PB; ++g) {
        const int s = s0 + g;
        const bool none = s >= a.split_k;
        float* part = a.sk_partials + ((size_t)(none ? 0 : s) * a.split_tiles + st) * (C::BM * C::BN);
        __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(part, 0, BLOCK_BYTES, 0x00027000);
#pragma unroll
        for (int i = 0; i < 2; ++i) x[g][i] = __builtin_amdgcn_raw_buffer_load_b128(r, none || past ? BLOCK_BYTES : off + i * C::NT * 16, 0, SC1);
      }
      __builtin_amdgcn_sched_barrier(0);              // all of them before the first is waited for
#pragma unroll
      for (int g = 0; g < PB; ++g)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) sum[i][e] += __uint_as_float(x[g][i][e]);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) ep[(4 * (lane >> 4) + e) * STRIDE + i * 16 + (lane & 15)] = sum[i][e];
    __builtin_amdgcn_wave_barrier();
    const float4 y = *reinterpret_cast<const float4*>(ep + (lane / 4) * STRIDE + (lane % 4) * 8);
    const float4 z = *reinterpret_cast<const float4*>(ep + (lane / 4) * STRIDE + (lane % 4) * 8 + 4);
    __builtin_amdgcn_wave_barrier();
    float o[8] = {y.x, y.y, y.z, y.w, z.x, z.y, z.z, z.w};
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      if (PF32) {
#pragma unroll
        for (int e = 0; e < 4; ++e) { o[e] += __uint_as_float(w[j][0][e]); o[4 + e] += __uint_as_float(w[j][LPP - 1][e]); }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) { o[2 * e] += bf16_lo(w[j][0][e]); o[2 * e + 1] += bf16_hi(w[j][0][e]); }
      }
    }
    int row, col;
    place(u, lane, row, col);
    if (!EDGE || (m0 + row < a.M && n0 + col < a.N)) store_row8<EPI, false>(a, lds_outs, m0 + row, n0 + col, o);
  }

  // Called by every part once its sums are parked and acknowledged.  `lds_misc`: two ints of the workgroup.  False: all others gave up, the tile is this part's alone (the caller sums it up).
  static __device__ __forceinline__ bool run(const GemmArgs& a, int* lds_misc, void* const* lds_outs, float* ep, int tile, int split,
                                             int m0, int n0, int tid, int lane, int wave) {
    const int st = tile - a.full_tiles, S = a.split_k;
    uint32_t* const word = a.sk_counters + sk_counter_index(st);
    constexpr int NW = C::NT / 64;
    PeerBufs pb;
    if (NP > 0) make_peer_bufs(a, m0, n0, pb);
    int u = BLOCKS * split / S + wave;
    const int u_end = BLOCKS * (split + 1) / S;
    u32x4 w[NPA][LPP];
    if (NP > 0 && u < u_end) load_peers(a, pb, u, m0, n0, lane, w);       // on their way during the wait
    // seen; whoever completes that clears the word for the next launch.  (A part that gives up counts too, in the same addition.)
    auto seen = [&](uint32_t and_gave_up) {
      const uint32_t prev = __hip_atomic_fetch_add(word, (1u << SK_SEEN_AT) + and_gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (((prev >> SK_SEEN_AT) & SK_COUNT) + 1u == (uint32_t)S) __hip_atomic_store(word, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return prev;
    };
    bool gave_up = false;
    if (tid == 0) {
      uint32_t extra = 0u;                            // parts whose shares fall to this one
      int mine = 1;
      const uint32_t prev = __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if ((prev & SK_COUNT) + 1u == (uint32_t)S) {
        extra = prev >> 16;
      } else {
        const uint32_t t0 = (uint32_t)wall_clock64();
        const uint32_t longest = a.timeout_ticks < SK_WAIT_TICKS ? (uint32_t)a.timeout_ticks : SK_WAIT_TICKS;
        const uint32_t unstarted = (uint32_t)a.sk_share < longest ? (uint32_t)a.sk_share : longest;
        for (;;) {
          const uint32_t now = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if ((now & SK_COUNT) == (uint32_t)S) break;
          const bool all_started = ((now >> SK_STARTED_AT) & SK_COUNT) == (uint32_t)S;
          if ((uint32_t)wall_clock64() - t0 > (all_started ? longest : unstarted)) {
            gave_up = true;
            mine = (seen(SK_GAVE_UP << split) & SK_COUNT) == (uint32_t)S;   // (all there after all: the last one did not see this part give up)
            break;
          }
          __builtin_amdgcn_s_sleep(1);
        }
      }
      lds_misc[0] = mine;
      lds_misc[1] = (int)extra;
    }
    __syncthreads();
    const int mine = __builtin_amdgcn_readfirstlane(lds_misc[0]);
    const uint32_t extra = (uint32_t)__builtin_amdgcn_readfirstlane(lds_misc[1]);
    if (tid == 0 && !gave_up) seen(0u);
    if (!mine) return true;
    if (extra == ((1u << S) - 1u - (1u << split))) return false;
    for (; u < u_end;) {
      block(a, lds_outs, ep, u, st, m0, n0, lane, w);
      u += NW;
      if (NP > 0 && u < u_end) load_peers(a, pb, u, m0, n0, lane, w);
    }
    if (extra != 0u)                                  // (all waves over all of the tile's blocks: a share may be less than one a wave)
      for (int x = wave; x < BLOCKS; x += NW) {
        const int owner = (S * (x + 1) - 1) / BLOCKS; // BLOCKS * owner / S <= x < BLOCKS * (owner + 1) / S
        if (((extra >> owner) & 1u) == 0u) continue;
        if (NP > 0) load_peers(a, pb, x, m0, n0, lane, w);
        block(a, lds_outs, ep, x, st, m0, n0, lane, w);
      }
    return true;
  }
};

// Everything after the main loop: the split-K hand-over (all but the last-arriving workgroup of
// a tile park their partial sums, the last one adds them up) and the epilogue, in which the
// accumulators pass through LDS once (per wave, 32 rows at a time) so that every lane ends up
// with 8 consecutive columns of one row.  `smem` must hold C::EP_BYTES and is free to reuse.
// MAX_NP: most peers there can be; PARTIALS: their type, 0 bf16, 1 fp32, -1 either.  (A resident kernel is built for up to 4 ranks or for more, and a type:
// with the code of both in one kernel 8192x12288x1536 of 8 ranks took 439 us instead of 422.  The other kernels of 256x256 tiles are built for a type, too, since
// their lanes have other columns for each; us, one kernel / by type, 8 ranks, bf16, masked edges: 4000x8192x1536 162.2 / 156.3, 3000x8192x3584 232.2 / 225.0, 2000x12288x6144
// 326.7 / 324.5; the other side: fp32 3000x8192x3584 316.9 / 319.3, tiles that divide 4096x8192x3584 the same; not 256x128 and 128x128 tiles: 760x8192x1000
// 35.3 / 38.2, 1104x4608x272 28.7 / 31.0, 552x4608x272 16.7 / 16.4.)
template <class C, int EPI, bool EDGE, bool RESIDENT, int MAX_NP = FLUX_MAX_RANKS - 1, int PARTIALS = -1>
__device__ __forceinline__ void gemm_tail(const GemmArgs& a, unsigned char* smem, int* lds_misc, void* const* lds_outs,
                                          f32x4 (&acc)[C::MI][C::NI], int tile, int split, bool is_split,
                                          int m0, int n0, int tid, int lane, int wave, int wm, int wn, bool peers_added,
                                          EarlyPeers<C>& early, int n_early, int vb = -1) {
  trace_stamp(a, TRACE_MAIN_END, vb);
  const bool partial_f32 = PARTIALS < 0 ? a.partial_f32 != 0 : PARTIALS != 0;
  // ---- split-K: all but the last-arriving workgroup of a tile park their partial sums ----
  if (is_split) {
    const int st = tile - a.full_tiles;            // index among the split tiles
    // Partials are stored and re-read with device-scope (sc1) accesses, which go through the
    // die's L2 to memory: the hand-over between workgroups on different dies then needs neither
    // an L2 write-back nor an L2 invalidate, only "my stores are acknowledged" before counting in.
    constexpr int SC1 = 16;                               // cache-policy bit: device scope
    constexpr int BLOCK_BYTES = C::BM * C::BN * 4;
    float* mine = a.sk_partials + ((size_t)split * a.split_tiles + st) * (C::BM * C::BN);
    __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(mine, 0, BLOCK_BYTES, 0x00027000);
    // layout inside a tile's partial block: [vector index][thread] -> coalesced 16-byte columns.
    // A vector holds four consecutive rows; with a ragged M (a decode tile of 8 rows in a
    // 32-row tile) the vectors that lie wholly past the last row are neither parked nor read back:
    // their offset is moved past the end of the block, where the range check of the buffer drops a
    // store and answers a load with zeros (a branch around them would make every load wait for
    // the one before).
    const int rows_valid = EDGE ? a.M - m0 - wm * C::WTM - 4 * (lane >> 4) : C::BM;
#pragma unroll
    for (int mi = 0; mi < C::MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < C::NI; ++ni) {
        const u32x4 v = {__float_as_uint(acc[mi][ni][0]), __float_as_uint(acc[mi][ni][1]),
                         __float_as_uint(acc[mi][ni][2]), __float_as_uint(acc[mi][ni][3])};
        const bool past = EDGE && mi * 16 >= rows_valid;
        __builtin_amdgcn_raw_buffer_store_b128(v, rm, past ? BLOCK_BYTES : ((mi * C::NI + ni) * C::NT + tid) * 16, 0, SC1);
      }
    __builtin_amdgcn_s_waitcnt(0x0F70);                   // vmcnt(0): stores acknowledged
    __syncthreads();
    if (a.sk_share) {                                     // (uniform)
      float* const ep = reinterpret_cast<float*>(smem) + wave * (32 * C::EP_STRIDE);
      bool finished;
      if (EPI != EPI_RS || a.write_only) finished = SharedFinish<C, EPI, EDGE, false, 0>::run(a, lds_misc, lds_outs, ep, tile, split, m0, n0, tid, lane, wave);
      else if (a.R <= 4) {
        if (partial_f32) finished = SharedFinish<C, EPI, EDGE, true, 3>::run(a, lds_misc, lds_outs, ep, tile, split, m0, n0, tid, lane, wave);
        else finished = SharedFinish<C, EPI, EDGE, false, 3>::run(a, lds_misc, lds_outs, ep, tile, split, m0, n0, tid, lane, wave);
      } else if (a.R <= 8) {
        if (partial_f32) finished = SharedFinish<C, EPI, EDGE, true, 7>::run(a, lds_misc, lds_outs, ep, tile, split, m0, n0, tid, lane, wave);
        else finished = SharedFinish<C, EPI, EDGE, false, 7>::run(a, lds_misc, lds_outs, ep, tile, split, m0, n0, tid, lane, wave);
      } else {
        if (partial_f32) finished = SharedFinish<C, EPI, EDGE, true, 15>::run(a, lds_misc, lds_outs, ep, tile, split, m0, n0, tid, lane, wave);
        else finished = SharedFinish<C, EPI, EDGE, false, 15>::run(a, lds_misc, lds_outs, ep, tile, split, m0, n0, tid, lane, wave);
      }
      if (finished) {
        trace_stamp(a, TRACE_END, vb);
        return;
      }
    } else {
      int* lds_last = lds_misc;
      if (tid == 0) {
        uint32_t* const word = a.sk_counters + sk_counter_index(st);
        const uint32_t prev = __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int last = prev == (uint32_t)(a.split_k - 1);
        if (last) __hip_atomic_store(word, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next launch
        *lds_last = last;
      }
      __syncthreads();
      trace_stamp(a, TRACE_END, vb);    // a workgroup that is not the tile's last ends here
      if (!*lds_last) return;
    }
    // The sum always runs over the parked partials in split order, whichever workgroup happens
    // to be last, so results do not depend on arrival timing.  (Keeping the own part in registers
    // and skipping its load was tried: no gain for 64x64 tiles, a loss for 64x128.)
#pragma unroll
    for (int mi = 0; mi < C::MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < C::NI; ++ni)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[mi][ni][e] = 0.f;
    // Sixteen or thirty-two loads are issued before the first is used.  Left to itself the compiler waits for
    // every vector before it requests the next (a memory round trip each: 17 us for the 256 KB of
    // two parts of a 256x128 tile); a branch around a load has the same effect, so parts past the
    // end are read as zeros through the buffer's range check instead.  A large tile takes its
    // vectors a batch at a time, part by part; a small one takes all vectors of several parts.
    constexpr int NVEC = C::MI * C::NI;                     // 16-byte vectors per thread and part
    constexpr int IN_FLIGHT = NVEC >= 32 ? 32 : 16;         // (32 is ahead for the large tiles, 16 for the small)
    constexpr int VB = NVEC < IN_FLIGHT ? NVEC : IN_FLIGHT; // vectors per batch within a part
    constexpr int PB = IN_FLIGHT / VB;                      // parts per batch
    static_assert(NVEC % VB == 0 && IN_FLIGHT % VB == 0, "batches divide the tile");
    for (int s0 = 0; s0 < a.split_k; s0 += PB) {
#pragma unroll
      for (int b0 = 0; b0 < NVEC; b0 += VB) {
        u32x4 v[PB][VB];
#pragma unroll
        for (int g = 0; g < PB; ++g) {
          const int s = s0 + g;
          const bool none = s >= a.split_k;                 // only with PB > 1
          float* other = a.sk_partials + ((size_t)(none ? 0 : s) * a.split_tiles + st) * (C::BM * C::BN);
          __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(other, 0, BLOCK_BYTES, 0x00027000);
#pragma unroll
          for (int i = 0; i < VB; ++i) {
            const int idx = b0 + i, mi = idx / C::NI;
            const bool past = none || (EDGE && mi * 16 >= rows_valid);
            v[g][i] = __builtin_amdgcn_raw_buffer_load_b128(ro, past ? BLOCK_BYTES : (idx * C::NT + tid) * 16, 0, SC1);
          }
        }
        __builtin_amdgcn_sched_barrier(0);                  // all of the batch's loads first
#pragma unroll
        for (int g = 0; g < PB; ++g)
#pragma unroll
          for (int i = 0; i < VB; ++i) {
            const int idx = b0 + i, mi = idx / C::NI, ni = idx % C::NI;
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[mi][ni][e] += __uint_as_float(v[g][i][e]);
          }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();
    early.forget();
  }

  // ---- epilogue: registers -> LDS (per wave, 32 rows at a time) -> 8 columns per lane ----
  float* ep = reinterpret_cast<float*>(smem) + wave * (32 * C::EP_STRIDE);
  // (the dtype and rank-count tests stay outside the loop over blocks: inside it, the accumulators
  // would no longer be kept in registers.  Up to 4 ranks, 3 peer loads per piece are issued, up to 8, 7, else 15:
  // loads from absent peers return zeros but still cost an issue slot and four registers each: us, 7 / 3 of them, 2 ranks 4096x8192x1536
  // 111.9 / 98.6, 4096x8192x3584 195 / 180, 1024x8192x1024 27.1 / 23.9, 512x12288x6144 92.2 / 87.7, 4 ranks 4096x8192x3584 211 / 189,
  // 8192x12288x1536 351 / 317, 1496x5112x3400 72.5 / 70.5; fp32 partials 2 ranks 4096x8192x3584 225 / 218.
  // Of 3 peers four passes' loads are out together: fp32, 2 ranks 8192x6144x1536 220 / 186 / 181 us with one / two / four.)
  constexpr int NP_ALL = FLUX_MAX_RANKS - 1, NP_8 = 7, NP_4 = 3;
  if (EPI == EPI_RS && a.write_only == 2) {
    epilogue_all_atomic<C, EDGE>(a, lds_outs, ep, acc, m0, n0, lane, wm, wn);
  } else if (EPI != EPI_RS || a.write_only || peers_added) {
    epilogue_all<C, EPI, EDGE, false, 2, 0, RESIDENT>(a, lds_outs, ep, acc, m0, n0, lane, wm, wn);
  } else if (EarlyPeers<C>::SMALL && n_early != 0) {
    auto finish = [&](auto np_, auto pf32_) {
      constexpr int NP = decltype(np_)::value;
      constexpr bool PF32 = decltype(pf32_)::value;
      if constexpr (EarlyPeers<C>::template fits<NP, PF32>())
        if (n_early == NP && partial_f32 == PF32) epilogue_all<C, EPI, EDGE, PF32, PF32 ? 1 : 2, NP, RESIDENT, true>(a, lds_outs, ep, acc, m0, n0, lane, wm, wn, early);
    };
    static_for<2>([&](auto pf32_) {
      constexpr std::bool_constant<decltype(pf32_)::value != 0> PF32;
      finish(std::integral_constant<int, 1>{}, PF32);
      finish(std::integral_constant<int, 3>{}, PF32);
      finish(std::integral_constant<int, 7>{}, PF32);
    });
  } else if (RESIDENT ? MAX_NP == NP_4 : a.R <= NP_4 + 1) {
    if (partial_f32) epilogue_all<C, EPI, EDGE, true, 4, NP_4, RESIDENT>(a, lds_outs, ep, acc, m0, n0, lane, wm, wn);
    else epilogue_all<C, EPI, EDGE, false, 4, NP_4, RESIDENT>(a, lds_outs, ep, acc, m0, n0, lane, wm, wn);
  } else if (a.R <= NP_8 + 1) {
    if (partial_f32) epilogue_all<C, EPI, EDGE, true, 1, NP_8, RESIDENT>(a, lds_outs, ep, acc, m0, n0, lane, wm, wn);
    else epilogue_all<C, EPI, EDGE, false, 2, NP_8, RESIDENT>(a, lds_outs, ep, acc, m0, n0, lane, wm, wn);
  } else {
    if (partial_f32) epilogue_all<C, EPI, EDGE, true, 1, NP_ALL, RESIDENT>(a, lds_outs, ep, acc, m0, n0, lane, wm, wn);
    else epilogue_all<C, EPI, EDGE, false, 1, NP_ALL, RESIDENT>(a, lds_outs, ep, acc, m0, n0, lane, wm, wn);
  }
  if (EPI == EPI_RS && a.tile_ready != nullptr) {
    // Producer side of the tile-ready handshake (Sec. 4.2, "Reduce", second form): the tile was written
    // through to memory; once every wave's stores are acknowledged, count this producer in.
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    if (tid == 0)
      __hip_atomic_fetch_add(a.tile_ready + (size_t)(m0 / C::BM) * a.tm.tiles_n + n0 / C::BN, 1u, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_SYSTEM);
  }
  trace_stamp(a, TRACE_END, vb);
}

// ---------------------------------------------------------------------------------------------
// Operand loads: global -> LDS without passing through registers.
//
// buffer_load_dwordx4 ... lds writes the 64 x 16 B a wave fetches to 1 KiB of consecutive LDS,
// so the swizzled layouts above are produced by permuting which 16 B each lane FETCHES:
//   A: one instruction = 8 rows x 128 B; lane i fills physical slot i%8 of row i/8 and fetches
//      logical slot (i%8) ^ swz_a(row);
//   B: one instruction = 1 KiB / (2*BN) k-rows; lane i fills physical slot i%B_SLOTS and
//      fetches logical slot (i%B_SLOTS) ^ swz_b(k).  Which rows are a wave's: those whose bits 0, 1 and 3, which swz_b looks
//      at, are the same in all of its instructions (wave_row, instr_row).
// Per K-slab only scalar offsets change (soffset), so the address arithmetic costs no vector
// instructions.
//
// EDGE (the tile does not divide the shape): a lane whose 16 bytes lie past the last row, past the last column of a
// [K,N] matrix, or past the end of K asks for an offset outside the records, which loads zeros and touches no memory:
// a compare and a select per load, between the MFMAs.  (The scalar offset takes no part in the hardware's range
// check, so the check alone would not do.)  Rows and columns past the end would only reach results that are not
// stored; K has to be padded with zeros on both sides.  Against a kernel that staged masked loads through
// registers: 3000 x 3584 x 8192 268 -> 186 us, 1496 x 5112 x 3400 with 8 ranks 119 -> 88 us, 200 x 3584 x 8192 58 -> 50 us.
// ---------------------------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void lds_void_t;

// A slab of A and one of B: where they start in K, and the matrices, or nothing in the place of a slab past the end (its
// loads touch no memory).
struct Slabs {
  __amdgpu_buffer_rsrc_t ra, rb;
  int ka, kb;
};

// CHUNKS: row i of A is row i % S of chunk source i / S, so every lane has a pointer per load of a slab (its rows of a tile lie in
// different chunks); a lane with nothing to fetch reads zero_vec instead.  Two additions per load, between the MFMAs: the main loop
// alone takes what it takes on a gathered matrix through buffer loads (4096x3584x8192 170 us, plain GEMM 173; with masks, 3000 rows, 166 / 160).
static __device__ const uint4 zero_vec = {0u, 0u, 0u, 0u};

// B_ONCE: B is streamed (see b_once in the host's plan).
template <class C, bool EDGE, bool CHUNKS = false, bool B_ONCE = false>
struct DmaLoader {
  static constexpr int NW = C::NT / 64;
  static constexpr int A_RPI = 8;                              // A rows per instruction (1 KiB of 128-byte rows)
  static constexpr int A_INSTR = C::BM / A_RPI / NW;           // per wave
  static constexpr int RPI = C::B_NK ? A_RPI : 512 / C::BN;    // B rows per instruction: k-rows of BN values, or ([N,K]) n-rows of BK
  static constexpr int B_INSTR = (C::B_NK ? C::BN : C::BK) / RPI / NW;   // per wave
  // first row of the p-th of a wave's instructions for B: wave_row(wave) + instr_row(p)
  static constexpr __device__ int wave_row(int wave) {
    if (C::B_NK || RPI == 8) return RPI * wave;
    return RPI == 4 ? 8 * (wave & 1) + 4 * (wave >> 1) : 2 * (wave & 1) + 8 * (wave >> 1);
  }
  static constexpr __device__ int instr_row(int p) {
    if (C::B_NK || RPI == 8) return p * RPI * NW;
    return RPI == 4 ? 16 * p : 4 * (p & 1) + 16 * (p >> 1);
  }
  static_assert(C::BK == 64, "A rows must be 128 B");
  static_assert(NW == 4 && (RPI == 2 || RPI == 4 || RPI == 8), "the swizzle must not depend on the instruction index");
  static_assert(C::BM % (A_RPI * NW) == 0 && (C::B_NK ? C::BN : C::BK) % (RPI * NW) == 0 && 512 % C::BN == 0, "loader shape");

  // Offsets into A and B are unsigned 32-bit byte offsets (a matrix has fewer than 2^31 elements, so
  // fewer than 2^32 bytes); the hardware adds the vector and the scalar part as unsigned numbers.
  uint32_t voff_a, voff_b;
  uint32_t K2, N2;               // row pitches in bytes
  uint32_t bytes_a, bytes_b;     // extents
  uint32_t lds_b;                // where this wave's rows of B begin in a slab in LDS
  // EDGE: how many of this lane's loads of A (and of an [N,K] B) have a row, the k of its vector in a slab, and the k of
  // its first vector of a [K,N] B (out of reach for a lane past the last column)
  int lim_a, lim_b, k_vec, k_row;
  uint64_t rows[CHUNKS ? A_INSTR : 1];
  static constexpr uint32_t OUTSIDE = 0xfffffff0u;      // a matrix has fewer than 2^31 elements

  __device__ __forceinline__ void init(const GemmArgs& a, int m0, int n0, int wave, int lane) {
    bytes_a = ((unsigned)(a.M - 1) * (unsigned)a.lda + (unsigned)a.K) * 2u;
    bytes_b = (C::B_NK ? (unsigned)(a.N - 1) * (unsigned)a.ldb + (unsigned)a.K : (unsigned)(a.K - 1) * (unsigned)a.ldb + (unsigned)a.N) * 2u;
    lds_b = (uint32_t)(wave_row(wave) * (1024 / RPI));
    const int r_in = lane / C::A_SLOTS, sp = lane % C::A_SLOTS;
    const int row = A_RPI * wave + r_in;
    if (EDGE) {
      k_vec = (sp ^ swz_a<C::A_SLOTS>(row)) * 8;
      lim_a = (a.M - m0 - row + A_RPI * NW - 1) / (A_RPI * NW);           // (not positive: none)
      if (C::B_NK) lim_b = (a.N - n0 - row + A_RPI * NW - 1) / (A_RPI * NW);
    }
    K2 = (uint32_t)a.lda * 2u;
    N2 = (uint32_t)a.ldb * 2u;
    voff_a = (uint32_t)(m0 + row) * K2 + ((uint32_t)(sp ^ swz_a<C::A_SLOTS>(row)) << 4);
    if constexpr (C::B_NK) {
      voff_b = (uint32_t)(n0 + row) * N2 + ((uint32_t)(sp ^ swz_a<C::A_SLOTS>(row)) << 4);      // as for A, rows of n
    } else {
      const int k_in = lane / C::B_SLOTS, spb = lane % C::B_SLOTS;
      const int k = wave_row(wave) + k_in;
      voff_b = (uint32_t)k * N2 + (uint32_t)n0 * 2u + ((uint32_t)(spb ^ swz_b<C::B_SLOTS>(k)) << 4);
      if (EDGE) k_row = n0 + (spb ^ swz_b<C::B_SLOTS>(k)) * 8 < a.N ? k : 0x40000000;
    }
  }

  // The lane's pointers into the chunk sources: `src` holds the one of chunk j in lane j.
  __device__ __forceinline__ void init_rows(const GemmArgs& a, uint64_t src, int m0, int wave, int lane) {
    static_assert(CHUNKS);
    const int sp = lane % C::A_SLOTS;
    const int chunk0 = m0 / a.S, in0 = m0 - chunk0 * a.S;              // (uniform)
    const float per_row = __builtin_amdgcn_rcpf((float)a.S);
#pragma unroll
    for (int d = 0; d < A_INSTR; ++d) {
      const int row = A_RPI * wave + lane / C::A_SLOTS + d * A_RPI * NW;
      const int x = in0 + row;
      // x / S: a tile touches one or two chunks, or x is below 2 * BM (exact in fp32: x + 1/2 is no closer than 1/2 to a multiple of S)
      const int q = a.S >= C::BM ? (x >= a.S ? 1 : 0) : (int)(((float)x + 0.5f) * per_row);
      const int chunk = chunk0 + q < a.R ? chunk0 + q : a.R - 1;        // (rows past the last are not loaded)
      const uint64_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(chunk * 4, (int)(uint32_t)src);
      const uint64_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(chunk * 4, (int)(uint32_t)(src >> 32));
      const uint32_t pitch = !a.gather_local && chunk == a.rank ? K2 : (uint32_t)a.K * 2u;       // (in place: the gathered matrix's)
      rows[d] = (lo | hi << 32) + (uint64_t)(uint32_t)(x - q * a.S) * pitch + ((uint32_t)(sp ^ swz_a<C::A_SLOTS>(row)) << 4);
    }
  }

  __device__ __forceinline__ Slabs slabs(const GemmArgs& a, bool there_a, int ka, bool there_b, int kb) const {
    return Slabs{__builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16*>(a.A), 0, (int)(there_a ? bytes_a : 0u), 0x00027000),
                 __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16*>(a.B), 0, (int)(there_b ? bytes_b : 0u), 0x00027000), ka, kb};
  }

  // the d-th (constant after unrolling) of this wave's loads of A / of B, into `slab` in LDS
  __device__ __forceinline__ void load_a(int d, const GemmArgs& a, const Slabs& s, unsigned char* slab, int wave) const {
    if constexpr (CHUNKS) {
      // (Slabs past the end, into places that nobody reads: of K, the last one again, or zeros; of a part of K, the next part's.  With the
      // part's own last slab there, whose lines the unit has just had, the same times: us, next part's / own, 8x3584x8192 16.68 / 16.75, 200x3584x8192
      // [N,K] 30.58 / 30.61, 512x3584x8192 44.35 / 44.11, 512x6144x12288 90.6 / 91.4.)
      const int ka = !EDGE && s.ka > a.K - C::BK ? a.K - C::BK : s.ka;
      uint64_t p = rows[d] + (uint32_t)ka * 2u;
      if (EDGE && !(d < (k_vec < a.K - s.ka ? lim_a : 0))) p = reinterpret_cast<uint64_t>(&zero_vec);
      typedef const __attribute__((address_space(1))) void* global_ptr;
      __builtin_amdgcn_global_load_lds((global_ptr)p, (lds_void_t*)(slab + (d * NW + wave) * 1024), 16, 0, 0);
      return;
    }
    const uint32_t v = !EDGE || d < (k_vec < a.K - s.ka ? lim_a : 0) ? voff_a : OUTSIDE;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(s.ra, (lds_void_t*)(slab + (d * NW + wave) * 1024), 16, (int)v,
                                             (int)((uint32_t)s.ka * 2u + (uint32_t)(d * A_RPI * NW) * K2), 0, 0);
  }
  __device__ __forceinline__ void load_b(int d, const GemmArgs& a, const Slabs& s, unsigned char* slab) const {
    const bool in = !EDGE || (C::B_NK ? d < (k_vec < a.K - s.kb ? lim_b : 0) : k_row < a.K - s.kb - instr_row(d));
    lds_void_t* const to = (lds_void_t*)(slab + instr_row(d) * (1024 / RPI) + lds_b);
    const int v = (int)(in ? voff_b : OUTSIDE);
    const int from = (int)(C::B_NK ? (uint32_t)s.kb * 2u + (uint32_t)instr_row(d) * N2 : (uint32_t)(s.kb + instr_row(d)) * N2);
    if constexpr (B_ONCE) __builtin_amdgcn_raw_ptr_buffer_load_lds(s.rb, to, 16, v, from, 0, 2);
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(s.rb, to, 16, v, from, 0, 0);
  }

  // this wave's loads of the A part / the B part of one K-slab
  __device__ __forceinline__ void issue_a(const GemmArgs& a, const Slabs& s, unsigned char* slab, int wave) const {
#pragma unroll
    for (int d = 0; d < A_INSTR; ++d) load_a(d, a, s, slab, wave);
    // keep the loads where they are written: scheduled late they would be issued just before
    // the wait for them, and nothing would overlap
    __builtin_amdgcn_sched_barrier(0);
  }
  __device__ __forceinline__ void issue_b(const GemmArgs& a, const Slabs& s, unsigned char* slab) const {
#pragma unroll
    for (int d = 0; d < B_INSTR; ++d) load_b(d, a, s, slab);
    __builtin_amdgcn_sched_barrier(0);
  }
};

typedef __attribute__((address_space(3))) unsigned char lds_byte_t;
__device__ __forceinline__ uint32_t lds_address(const unsigned char* p) {
  return (uint32_t)reinterpret_cast<uintptr_t>((const lds_byte_t*)p);
}

// A fragment as its LDS reads leave it: one 16-byte read, or the two halves of a transposing read.  The halves are two
// values until their wait is over: joining them means whatever the register allocator makes of it, a copy included.
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
struct FragHalves { u32x2 lo, hi; };
__device__ __forceinline__ void frag_settle(bf16x8& f) { asm volatile("" : "+v"(f)); }
__device__ __forceinline__ void frag_settle(FragHalves& f) { asm volatile("" : "+v"(f.lo), "+v"(f.hi)); }
__device__ __forceinline__ bf16x8 frag_value(const bf16x8& f) { return f; }
__device__ __forceinline__ bf16x8 frag_value(const FragHalves& f) {
  const u32x4 w = {f.lo[0], f.lo[1], f.hi[0], f.hi[1]};
  return __builtin_bit_cast(bf16x8, w);
}

// All LDS reads issued so far have returned.  The fragments pass through it so that nothing that
// uses them can be moved in front of the wait.
template <int NA, int NB, class FA, class FB>
__device__ __forceinline__ void wait_lds_reads(FA (&af)[NA], FB (&bfr)[NB]) {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
  for (int i = 0; i < NA; ++i) frag_settle(af[i]);
#pragma unroll
  for (int i = 0; i < NB; ++i) frag_settle(bfr[i]);
}

template <int N>
__device__ __forceinline__ void wait_vm_at_most() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit field");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));   // expcnt and lgkmcnt: no wait
}

// Workgroup barrier that lets this wave's younger loads stay in flight.  The compiler puts a wait
// for ALL outstanding memory operations in front of every barrier instruction it can see, which
// would empty the pipeline once per slab; it does not look inside this one.  What the barrier has
// to order is covered by the counter wait placed before it.
__device__ __forceinline__ void barrier_keeping_loads_in_flight() {
  asm volatile("s_barrier" ::: "memory");
}

__device__ __forceinline__ void wait_vm0_and_barrier() {
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's LDS-bound loads have landed
  __syncthreads();
}

// The gathered matrix of a grid that reads A from the chunk sources: nothing waits for it, it is a result like C, and it is stored
// out of the slabs of A that lie in LDS for the products.  The tiles of a row of tiles share its rows out among themselves: the nt-th
// stores rows [nt * share, (nt + 1) * share) of every slab, one vector per thread (gather_fits; the parts of a tile cut along K each
// their slabs).
// us per pass, gathered first and waited for / read from the sources: 4 layers of 8x3584x8192 86.0 / 70.0 (the wait was 6.5 of a call's
// 17.6 us in the kernel), 4 of 200x3584x8192 150 / 119, 4096x3584x8192 192 / 177, 3000x3584x8192 180 / 173, 8192x4608x12288 694 / 657.  With sources,
// weights and results out of memory (buffers of 1.2 GB in turn), per call: 8x3584x8192 21.6 / 16.7, 200x3584x8192 [N,K] 37.3 / 29.1, 512x6144x12288 106.7 / 92.5,
// 1024x8192x7168, 2 ranks, 107.9 / 102.1, 2048x6144x6144, 4 ranks, 154.4 / 149.5, 4096x3584x5120 140.6 / 114.7, 3000x3584x8192 188.9 / 174.8, 5000x4608x3400
// 188.7 / 161.3, 8192x4608x12288 738 / 655; the other side, weights of 151 MB out of the Infinity Cache: 512x6144x12288 88.2 / 89.7.  The stores
// are 2-3 % of that (left out: 70.0 / 68.9, 183 / 179, 175.5 / 170, 676 / 664 on a slower chip); moving the chunks through registers, a load and a
// store per slab, costs 7 % (a load that goes to memory holds up the operand loads behind it: 184, 175, 680).
constexpr int GATHER_ROWS = 32;      // rows of a slab that 256 threads store
__host__ __device__ constexpr bool gather_fits(int bm, int tiles_n) { return (long long)GATHER_ROWS * tiles_n >= bm; }
template <class C, bool EDGE>
struct GatherOut {
  __amdgpu_buffer_rsrc_t r;
  uint32_t from, to;                 // this lane's vector: in a slab in LDS, in the gathered matrix
  int k_vec;
  u32x4 v;
  static_assert(C::NT == 256 && C::A_SLOTS == 8, "32 rows of 8 vectors");
  static constexpr uint32_t OUTSIDE = 0xfffffff0u;

  __device__ __forceinline__ void init(const GemmArgs& a, const unsigned char* slab0, int m0, int nt, int tid) {
    const int share = (C::BM + a.tm.tiles_n - 1) / a.tm.tiles_n;
    const int slot = tid % C::A_SLOTS, row = nt * share + tid / C::A_SLOTS, gm = m0 + row;
    const bool in_place = !a.gather_local && gm >= a.rank * a.S && gm < (a.rank + 1) * a.S;
    const bool mine = tid / C::A_SLOTS < share && row < C::BM && gm < a.M && !in_place;
    from = lds_address(slab0) + (uint32_t)(row & (C::BM - 1)) * (C::BK * 2) + ((uint32_t)(slot ^ swz_a<C::A_SLOTS>(row)) << 4);
    to = mine ? (uint32_t)gm * ((uint32_t)a.lda * 2u) + (uint32_t)slot * 16u : OUTSIDE;
    k_vec = slot * 8;
    const unsigned bytes = ((unsigned)(a.M - 1) * (unsigned)a.lda + (unsigned)a.K) * 2u;
    r = __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16*>(a.A), 0, (int)bytes, 0x00027000);
  }
  template <int SLAB>
  __device__ __forceinline__ void read() {
    constexpr int OFF = SLAB * C::A_BYTES;
    const uint32_t at = OFF >= 65536 ? from + 65536u : from;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(at), "n"(OFF % 65536));
  }
  __device__ __forceinline__ void settle() { asm volatile("" : "+v"(v)); }
  __device__ __forceinline__ void write(const GemmArgs& a, int k) {
    __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)(!EDGE || k_vec < a.K - k ? to : OUTSIDE), k * 2, 2);
  }
};

// The main loop of every kernel: K-slabs out of an LDS ring of NA slabs of A and NB of B, every memory instruction placed
// by hand between the MFMAs.  A wave issues in order and (with the large tile) has its SIMD to itself, so what it
// issues in a burst or waits for is time its matrix core stands still:
//   * a slab has two k-steps of 32; the fragments of the next k-step are read while the MFMAs of this one run,
//     one read per few MFMAs, also across the slab's end: the last k-step reads the first fragments of the
//     next slab;
//   * the one barrier per slab therefore sits at the start of the last k-step: by then the next slab has landed
//     (counter wait: loads land in issue order), and every wave has its last fragments of this slab in
//     registers, so this slab's place is free;
//   * from there on the wave's loads are dealt out over SPAN MFMAs: B of the slab NB ahead, which the next barrier but NB - 2
//     needs, and A of the slab NA ahead.
// An operand that leads (the 256x256 tile, whose two slabs of 64 KB leave 32 KB of LDS: a third slab of A): with two slabs of
// each nothing was in flight at the barrier, and a slab's 64 KB, asked for in one go, took 1.24 us to come out of an L2 without a
// single MFMA beside them, longer than the 1.05 us of its MFMAs.  A third slab keeps 32 to 96 KB on their way.  Plain GEMM, us,
// two slabs / three of A: 4096x4096x8192 on zeros (no power limit) 166 / 135, where the MFMAs and the LDS reads take 134 by
// themselves; N(0,1), operands from memory: 4096x3584x8192 204 / 178, 8192x4608x12288 846 / 727 (B as [N,K] 918 / 770),
// 8192x12288x4608 670 / 648; 4096x4096x12288 with one peer 334 / 293.
// What bounds it now: with operands from a cache the chip's power limit (4096x4096x8192 182-200 us on N(0,1), 135 on zeros;
// MFMAs alone 2.0 PFLOP/s), with a long K from memory the memory (8192x4608x12288: 740 us on zeros too).
// Placing reads and loads between 16x16x32 MFMAs, against a burst per k-step, a wait at the slab's end and 32x32x16: 8192^3 699
// against 799 us, 8192x12288x4608 611 / 691; of that the placement gives 5-6 %, the MFMA shape 8-9 %.
// Measured, not kept: bringing the lines of a slab 4 to 32 ahead to the L2 with a load of one word per line and workgroup
// (instead of the third slab: the same gain; with it, or with 256x128 tiles: slower, a line is a line for the unit's L1);
// starting each die's walk over K elsewhere (dies share lines in the Infinity Cache only while they walk in step: 176 -> 185 us,
// 3000 rows 185 -> 258); B's fourth slab of 256x128 tiles (147 / 168 us on zeros, nothing on the calls).
// The fragment reads are instructions the compiler cannot look into.  For every LDS read it can see, it works
// out by itself which of the direct-to-LDS loads in flight must land first, and gets that wrong on the safe side.
// Their addresses are a few registers per lane plus an immediate.  They are waited for in the k-step that issued
// them, so no register is waiting for data where the compiler is free to move registers around.
//
// B_FIRST (signal wait): B, which does not depend on a gathered A, is requested before the wait for all of the first
// slabs, A after it.  Without, the first slabs are requested one after the other, so that slab 0 does not have to
// wait for the B of the others (64 x 8192 x 3584: 0.5 us of 23).
template <class C, bool B_FIRST, bool EDGE, bool CHUNKS = false, bool B_ONCE = false>
struct MmaPipe {
  typedef DmaLoader<C, EDGE, CHUNKS, B_ONCE> Ld;
  static constexpr int NA = C::NA, NB = C::NB;
  static constexpr bool A_LEADS = NA > NB;                           // by one slab
  static constexpr int U = NA == NB ? NB : NA * NB;                   // slabs after which both rings are where they were
  static constexpr int KS = C::BK / 32;                              // k-steps per slab
  static_assert(KS == 2, "two fragment sets, one per k-step");
  static constexpr int G = C::MI * C::NI;                            // MFMAs per k-step
  static constexpr int NF = C::MI + C::NI;                           // fragments per k-step
  static constexpr int LA = Ld::A_INSTR, LB = Ld::B_INSTR, L = LA + LB;   // loads per slab and wave
  static constexpr int LX = A_LEADS ? LA : 0;                        // loads of A where it is a slab further ahead
  static constexpr int NBV = C::B_NK ? KS : C::NI;
  static constexpr int A_HI = (NA * C::A_BYTES + 65535) / 65536, B_HI = (NB * C::B_BYTES + 65535) / 65536;  // a read's immediate offset reaches 64 KB
  // Placement, in MFMAs.  (8192^3, of G = 64: within 1 % for SPREAD 40 to 62, BAR_AT 1 to 12.  Without an operand that leads SPAN
  // 64 to 96 are alike and 118 costs 3-6 %: the last loads have not landed at the wait.  With one they have a slab longer: 104 is
  // 1 % ahead of 88.)
  static constexpr int BAR_AT = G / 8;                               // MFMAs of the last k-step ahead of the barrier
  static constexpr int SPREAD = (G * 15 + 15) / 16;                  // the reads go with the first SPREAD MFMAs of a k-step
  static constexpr int SPAN = G * (NA != NB ? 13 : 11) / 8;           // the loads with the first SPAN MFMAs from the last k-step on
  static_assert(BAR_AT < SPREAD && SPREAD <= G && SPAN >= G && SPAN + LX <= 2 * G, "placement");
  // the d-th load goes with slot load_slot(d), counted from the start of the last k-step
  static constexpr int load_slot(int d) { return BAR_AT + d * (SPAN - BAR_AT) / L; }
  static constexpr int loads_before(int slot) { int n = 0; while (n < L && load_slot(n) < slot) ++n; return n; }
  static constexpr int reads_before(int slot, int from) { int n = 0; while (n < NF && from + n * (SPREAD - from) / NF < slot) ++n; return n; }
  static constexpr int L0 = loads_before(G);                         // loads that go with that last k-step

  // What a step's loads are.  WHOLE_RING: as above.  TWO_SLABS (of a ring of three slabs of A and two of B): A no further ahead
  // than B, in the first two places of A's ring.  SWITCH: the step after the last one of those.
  enum Mode { WHOLE_RING, TWO_SLABS, SWITCH };

  unsigned char* pool;
  uint32_t a[A_HI][KS], b[B_HI][NBV];
  typedef std::conditional_t<C::B_NK, bf16x8, FragHalves> FragB;
  bf16x8 af[2][C::MI];
  FragB bf[2][C::NI];
  GatherOut<C, EDGE> out;            // CHUNKS

  __device__ __forceinline__ unsigned char* slab_a(int i) const { return pool + i * C::A_BYTES; }
  __device__ __forceinline__ unsigned char* slab_b(int i) const { return pool + NA * C::A_BYTES + i * C::B_BYTES; }

  __device__ __forceinline__ void init(unsigned char* pool_, int wm, int wn, int lane) {
    pool = pool_;
    const uint32_t base_a = lds_address(pool), base_b = base_a + NA * C::A_BYTES;
    const int g = lane >> 4, i = lane & 15;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int q = ks * 4 + g;
      const int row = wm * C::WTM + i;
#pragma unroll
      for (int h = 0; h < A_HI; ++h) a[h][ks] = base_a + h * 65536u + row * (C::BK * 2) + ((q ^ swz_a<C::A_SLOTS>(row)) << 4);
      if constexpr (C::B_NK) {
        const int rn = wn * C::WTN + i;
#pragma unroll
        for (int h = 0; h < B_HI; ++h) b[h][ks] = base_b + h * 65536u + rn * (C::BK * 2) + ((q ^ swz_a<C::A_SLOTS>(rn)) << 4);
      }
    }
    if constexpr (!C::B_NK) {
#pragma unroll
      for (int ni = 0; ni < C::NI; ++ni) {
        const int k = 8 * g + (i >> 2);
        const int n = wn * C::WTN + ni * 16 + 4 * (i & 3);
#pragma unroll
        for (int h = 0; h < B_HI; ++h) b[h][ni] = base_b + h * 65536u + k * (C::BN * 2) + (((n >> 3) ^ swz_b<C::B_SLOTS>(k)) << 4) + ((n >> 2) & 1) * 8;
      }
    }
  }

  template <int OFF>
  static __device__ __forceinline__ bf16x8 read16(uint32_t base) {
    u32x4 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(base), "n"(OFF));
    return __builtin_bit_cast(bf16x8, v);
  }
  template <int OFF>
  static __device__ __forceinline__ u32x2 read_tr(uint32_t base) {
    u32x2 v;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(base), "n"(OFF));
    return v;
  }
  // fragment R (in the order the MFMAs want them) of k-step K out of A's slab SA / B's slab SB in LDS
  template <int SA, int SB, int K, int R>
  __device__ __forceinline__ void fetch() {
    constexpr bool IS_B = R >= 1 && R <= C::NI;
    constexpr int I = R == 0 ? 0 : (IS_B ? R - 1 : R - C::NI);
    if constexpr (!IS_B) {
      constexpr int OFF = SA * C::A_BYTES + I * 16 * C::BK * 2;
      af[K][I] = read16<OFF % 65536>(a[OFF / 65536][K]);
    } else if constexpr (C::B_NK) {
      constexpr int OFF = SB * C::B_BYTES + I * 16 * C::BK * 2;
      bf[K][I] = read16<OFF % 65536>(b[OFF / 65536][K]);
    } else {
      constexpr int LO = SB * C::B_BYTES + K * 32 * C::BN * 2, HI = LO + 4 * C::BN * 2;
      bf[K][I].lo = read_tr<LO % 65536>(b[LO / 65536][I]);
      bf[K][I].hi = read_tr<HI % 65536>(b[HI / 65536][I]);
    }
  }

  // Fills the pipeline: slabs 0 .. NB-2 requested, and A of slab NB-1 where it leads; then the first of the loads that a step
  // "-1" would deal out; the fragments of the first k-step read.  Slabs past the end are loads outside the records everywhere
  // (no memory access; A from the chunk sources has addresses instead: see load_a): every step issues the same number of loads,
  // which keeps the counter waits constants and the loop one shape.
  // (`two_slabs`: the steps that follow are of that mode.)
  __device__ __forceinline__ void request_b(const Ld& ld, const GemmArgs& ga, int k_begin, int KT) {
    static_assert(B_FIRST);
#pragma unroll
    for (int j = 0; j < NB - 1; ++j) ld.issue_b(ga, slab_pair(ld, ga, k_begin, j, j, KT), slab_b(j));
  }
  __device__ __forceinline__ void start(const Ld& ld, const GemmArgs& ga, int k_begin, int KT, int wave, bool two_slabs) {
#pragma unroll
    for (int j = 0; j < NB - 1; ++j) {
      const auto s = slab_pair(ld, ga, k_begin, j, j, KT);
      ld.issue_a(ga, s, slab_a(j), wave);
      if constexpr (!B_FIRST) ld.issue_b(ga, s, slab_b(j));
    }
    const auto s = slab_pair(ld, ga, k_begin, NB - 1, NB - 1, KT);
    constexpr int BEHIND = (NB - 2) * (B_FIRST ? LA : L) + L0;         // loads behind slab 0's, without the A that leads
    if (A_LEADS && two_slabs) {
      const auto w = window<TWO_SLABS>(ld, ga, k_begin, -1, KT);
#pragma unroll
      for (int d = 0; d < L0; ++d) load<TWO_SLABS>(ld, ga, w, d, NB - 1, wave);
      wait_vm_at_most<BEHIND>();                                      // slab 0 is there
    } else {
      if constexpr (A_LEADS) ld.issue_a(ga, s, slab_a(NB - 1), wave);
      const auto w = window<WHOLE_RING>(ld, ga, k_begin, -1, KT);
#pragma unroll
      for (int d = 0; d < L0; ++d) load<WHOLE_RING>(ld, ga, w, d, U - 1, wave);
      wait_vm_at_most<BEHIND + LX>();
    }
    barrier_keeping_loads_in_flight();
    static_for<NF>([&](auto r) { fetch<0, 0, 0, decltype(r)::value>(); });
    wait_lds_reads(af[0], bf[0]);
  }

  // slab ja of A and slab jb of B
  __device__ __forceinline__ Slabs slab_pair(const Ld& ld, const GemmArgs& ga, int k_begin, int ja, int jb, int KT) const {
    return ld.slabs(ga, ja < KT, k_begin + ja * C::BK, jb < KT, k_begin + jb * C::BK);
  }
  // What step kt (in place S of the unrolled loop) asks for from its barrier on, and the d-th of those loads: first the operand
  // that the next barrier needs.
  static constexpr Mode now(Mode m) { return m == TWO_SLABS ? TWO_SLABS : WHOLE_RING; }
  static constexpr Mode before(Mode m) { return m == WHOLE_RING ? WHOLE_RING : TWO_SLABS; }     // of the step ahead of it
  template <Mode MODE>
  __device__ __forceinline__ Slabs window(const Ld& ld, const GemmArgs& ga, int k_begin, int kt, int KT) const {
    return slab_pair(ld, ga, k_begin, kt + (MODE == TWO_SLABS ? NB : NA), kt + NB, KT);
  }
  template <Mode MODE>
  __device__ __forceinline__ void load(const Ld& ld, const GemmArgs& ga, const Slabs& w, int d, int S, int wave) const {
    const bool is_a = A_LEADS ? d >= LB : d < LA;
    if (is_a) ld.load_a(A_LEADS ? d - LB : d, ga, w, slab_a(S % (MODE == TWO_SLABS ? NB : NA)), wave);
    else ld.load_b(A_LEADS ? d : d - LA, ga, w, slab_b(S % NB));
  }

  // Slab kt, in place S of the unrolled loop: A in place S % NA (TWO_SLABS: S % NB) of its ring, B in S % NB.  VM_EXTRA: that
  // many younger memory operations, issued by before_wait(), may stay outstanding at the wait.
  template <int S, int VM_EXTRA, Mode MODE, class Hook>
  __device__ __forceinline__ void step(const Ld& ld, const GemmArgs& ga, int k_begin, int kt, int KT, int wave,
                                       f32x4 (&acc)[C::MI][C::NI], Hook&& before_wait) {
    constexpr int RA = MODE == TWO_SLABS ? NB : NA;
    constexpr int VM = (NB - 2) * L + (MODE == TWO_SLABS ? 0 : LX) + VM_EXTRA;
    // (the slab's offset goes into the loads' scalar operand: should the compiler ever take the loop
    // counter for a value that may differ between lanes, it would wrap every load into a loop over lanes)
    kt = __builtin_amdgcn_readfirstlane(kt);
    const auto rest = window<before(MODE)>(ld, ga, k_begin, kt - 1, KT), first = window<now(MODE)>(ld, ga, k_begin, kt, KT);
    static_for<KS>([&](auto ks_) {
      constexpr int ks = decltype(ks_)::value;
      constexpr bool LAST = ks == KS - 1;
      if constexpr (LAST) before_wait();
      if constexpr (CHUNKS && !LAST) out.template read<S % RA>();
      static_for<G>([&](auto g_) {
        constexpr int g = decltype(g_)::value;
        // (with the large tile every second row of MFMAs goes backwards: it begins with the B fragment that the row before ended with,
        // 1-2 % of 8192x4608x12288 and 8192x12288x4608 at the power limit; small tiles lose as much)
        constexpr int mi = g / C::NI, ni = G < 64 || mi % 2 == 0 ? g % C::NI : C::NI - 1 - g % C::NI;
        if constexpr (LAST && g == BAR_AT) {
          // slab kt+1 is there (this wave's part, then everyone's); this slab has been read by all
          if constexpr (B_FIRST && S < NB - 2) {
            // (slabs 0 .. NB-2 were requested as all of B, then all of A: behind slab kt+1's are the A parts of the
            // later ones of those, and what was requested since)
            if (kt == S) wait_vm_at_most<(NB - 3 - S) * LA + LX + (S + 1) * L + VM_EXTRA>();
            else wait_vm_at_most<VM>();
          } else {
            wait_vm_at_most<VM>();
          }
          barrier_keeping_loads_in_flight();
        }
        mfma_in_place(acc[mi][ni], af[ks][mi], frag_value(bf[ks][ni]));
        // (behind the barrier: a store is acknowledged in any order with loads, so the next wait must not find it too young)
        if constexpr (CHUNKS && LAST && g == BAR_AT) out.write(ga, k_begin + kt * C::BK);
        // this MFMA's loads [d0, d1) and fragment reads [r0, r1)
        constexpr int d0 = loads_before(LAST ? g : G + g), d1 = loads_before((LAST ? g : G + g) + 1);
#pragma unroll
        for (int d = d0; d < d1; ++d) {
          if constexpr (LAST) load<now(MODE)>(ld, ga, first, d, S, wave);
          else load<before(MODE)>(ld, ga, rest, d, S + U - 1, wave);
        }
        if constexpr (MODE == SWITCH && !LAST && g >= SPAN - G && g < SPAN - G + LA) load<WHOLE_RING>(ld, ga, window<WHOLE_RING>(ld, ga, k_begin, kt - 1, KT), LB + g - (SPAN - G), S + U - 1, wave);
        constexpr int r0 = reads_before(g, LAST ? BAR_AT : 0), r1 = reads_before(g + 1, LAST ? BAR_AT : 0);
        static_for<r1 - r0>([&](auto r_) {
          constexpr int r = r0 + decltype(r_)::value;
          if constexpr (LAST) fetch<(S + 1) % RA, (S + 1) % NB, 0, r>();
          else fetch<S % RA, S % NB, ks + 1, r>();
        });
        __builtin_amdgcn_sched_barrier(0);
      });
      wait_lds_reads(af[1 - ks], bf[1 - ks]);
      if constexpr (CHUNKS && !LAST) out.settle();
    });
  }

  // Slabs kt to the end: 0 after start(), or the next one after steps of TWO_SLABS (`two_slabs`), an even number of them.
  __device__ __forceinline__ void run(const Ld& ld, const GemmArgs& ga, int k_begin, int KT, int kt, int wave,
                                      f32x4 (&acc)[C::MI][C::NI], bool two_slabs) {
    if constexpr (A_LEADS && B_FIRST) {
      if (two_slabs) {
        // the first step asks for A a slab further ahead; from there on as if K began here
        if (kt < KT) step<0, 0, SWITCH>(ld, ga, k_begin, kt, KT, wave, acc, [] {});
        static_for<U - 1>([&](auto s_) {
          constexpr int S = decltype(s_)::value + 1;
          if (kt + S < KT) step<S, 0, WHOLE_RING>(ld, ga, k_begin, kt + S, KT, wave, acc, [] {});
        });
        kt += U;
      }
    }
    for (; kt + U <= KT; kt += U)
      static_for<U>([&](auto s_) {
        constexpr int S = decltype(s_)::value;
        step<S, 0, WHOLE_RING>(ld, ga, k_begin, kt + S, KT, wave, acc, [] {});
      });
    static_for<U - 1>([&](auto s_) {
      constexpr int S = decltype(s_)::value;
      if (kt + S < KT) step<S, 0, WHOLE_RING>(ld, ga, k_begin, kt + S, KT, wave, acc, [] {});
    });
    mfma_results_settle<C::MI, C::NI>(acc);
  }
};

// All of A asked for once, ahead of the main loop, in the order it lies in memory: the threads of the first round's workgroups take its
// 128-byte lines in turn, one word each, so that it is in the Infinity Cache when the slabs are loaded.  A slab is 128 bytes of every row, and
// rows a multiple of 2 KB apart put those into few of the memory's channels, slab after slab: A of 6 MB out of memory cost a call
// with 151 MB of weights as much as the weights did (512x12288x6144: 67 us with both in the cache, 82 with the weights
// out of memory, 91 with A out of memory, 93 with both).
// us in the kernel without / with, A in memory: 2 ranks 512x8192x5120 87.0 / 77.3, 1024x8192x7168 130.5 / 120.3, 256x8192x6144 64.3 / 59.7, 8 ranks
// 512x12288x6144 136.2 / 120.0; several rounds, 8 ranks 3000x3584x5120 182.9 / 164.3, 1400x8192x5120 194.9 / 166.5, 2048x4608x5120 148.8 / 137.1 (shared
// out over all workgroups, of which the later ones ask when A has gone by: 168.5, 170.0, 147.2).  An A that is in a cache, written by the
// kernel before, gains nothing and costs the requests: 76.6 / 77.3, 116.7 / 118.2, 58.4 / 59.5, 119.5 / 119.9; 156.9 / 159.5, 161.9 / 163.5, 132.0 / 133.0.
// Not taken (warm_a): other pitches (512x8192x3584 47.8 / 48.7, 1496x5112x3400 67.0 / 68.2), a multiple of 16 KB (1024x8192x8192
// 134.9 / 137.7; 512x12288x8192 113.8 / 111.7), few slabs (512x12288x3072 47.0 / 46.9), tiles other than 256x128 (64x8192x8192 33.9 / 34.6,
// 4096x8192x4096 224.7 / 228.6), a gathered A, which the same grid has just written, and an A read from the chunk sources (not measured:
// its rows are packed in up to 16 buffers).
constexpr int WARM_LOADS = 8;      // per thread
constexpr uint32_t WARM_BLOCKS = 256;   // workgroups of one round: one per compute unit
__device__ __forceinline__ bool warm_a(const GemmArgs& a, uint32_t lines, uint32_t at_once) {
  const uint32_t pitch = (uint32_t)a.lda * 2u;
  return blockIdx.x < WARM_BLOCKS && pitch % 2048u == 0u && pitch % 16384u != 0u && a.K >= 4096 && lines <= WARM_LOADS * at_once;
}
struct WarmA {
  uint32_t word[WARM_LOADS];
  __device__ __forceinline__ void ask(const GemmArgs& a, uint32_t bytes_a, int tid) {
    const uint32_t row_lines = ((uint32_t)a.K * 2u + 127u) / 128u, lines = (uint32_t)a.M * row_lines;
    const uint32_t at_once = (gridDim.x < WARM_BLOCKS ? gridDim.x : WARM_BLOCKS) * 256u;
    const bool warm = warm_a(a, lines, at_once);
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16*>(a.A), 0, (int)bytes_a, 0x00027000);
#pragma unroll
    for (int t = 0; t < WARM_LOADS; ++t) {
      word[t] = 0u;
      if (!warm || t * at_once >= lines) continue;         // (uniform)
      const uint32_t i = t * at_once + blockIdx.x * 256u + (uint32_t)tid, row = i / row_lines;
      const uint32_t off = i < lines ? row * ((uint32_t)a.lda * 2u) + (i - row * row_lines) * 128u : 0xfffffff0u;
      word[t] = __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0);
    }
  }
  __device__ __forceinline__ void drop() {
#pragma unroll
    for (int t = 0; t < WARM_LOADS; ++t) asm volatile("" : : "v"(word[t]));
  }
};

// EDGE: the tile does not divide M, N or K (see DmaLoader; the epilogue leaves rows and columns past the end out).
template <class C, int EPI, int PRO, bool EDGE, bool B_ONCE, int PARTIALS>
__global__ void __launch_bounds__(C::NT, C::OCC) gemm_kernel_dma(const GemmArgs a) {
  constexpr bool WAIT = PRO == PRO_WAIT, CHUNKS = PRO == PRO_CHUNKS;
  // the transfer inside the main loop (SideCopy) is asked of the kernel with two slabs of B and one workgroup per unit
  constexpr bool CARRY = WAIT && !EDGE && C::NB == 2 && C::OCC == 1;
  __shared__ __attribute__((aligned(1024))) unsigned char pool[C::POOL_BYTES];
  SharedWords* const words = reinterpret_cast<SharedWords*>(pool + C::WORDS_AT);
  int* const lds_misc = words->misc;
  void** const lds_outs = words->outs;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / C::WAVES_N, wn = wave % C::WAVES_N;
  uint64_t src = 0;
  if constexpr (CHUNKS) {
    // the chunk sources, one per lane: asked for at once, beside the fetch of everything else (the struct is the kernel's only argument)
    typedef const uint64_t __attribute__((address_space(4))) * SrcPtr;
    src = reinterpret_cast<const uint64_t*>((const unsigned char*)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(GemmArgs, outs))[lane & (FLUX_MAX_RANKS - 1)];
  }

  int tile, split;
  bool is_split;
  map_block(a, (int)blockIdx.x, tile, split, is_split);
  int mt, nt;
  tile_coord(a.tm, a.m_order, tile, mt, nt);
  const int m0 = mt * C::BM, n0 = nt * C::BN;
  trace_begin(a, tile, mt, nt, split, is_split);

  if (WAIT || (EPI == EPI_RS && !C::WORDS_IN_RING)) fill_lds_outs(a, lds_outs, tid);
  const int k_begin = is_split ? split * a.k_per_split : 0;
  const int k_end = (is_split && k_begin + a.k_per_split < a.K) ? k_begin + a.k_per_split : a.K;
  const int KT = (k_end - k_begin + C::BK - 1) / C::BK;

  typedef MmaPipe<C, WAIT, EDGE, CHUNKS, B_ONCE> Pipe;
  typename Pipe::Ld ld;
  ld.init(a, m0, n0, wave, lane);
  Pipe pipe;
  pipe.init(pool, wm, wn, lane);
  if constexpr (CHUNKS) {
    ld.init_rows(a, src, m0, wave, lane);
    pipe.out.init(a, pipe.slab_a(0), m0, nt, tid);
  }
  SideCopy side;
  if constexpr (WAIT) {
    const int m1 = (!EDGE || m0 + C::BM < a.M) ? m0 + C::BM : a.M;
    // First this workgroup's own pieces of the chunks: the whole grid waits for them.
    transfer_own_pieces(a, lds_misc, lds_outs);
    if constexpr (CARRY) {
      side.begin(a, lds_misc + 2, lds_outs);     // (also orders fill_lds_outs before the reads of lds_outs below)
      // A workgroup that has pieces to move and no data to compute on yet moves them in batches, and
      // counts tiles in as they become due, until its own signals are there (the main loop then
      // carries what is left) or its part of the transfer is done (then it waits like anybody else).
      while (side.pending() && !signals_all_set(a, m0, m1, lds_misc + 2)) {
        if (!side.all_stored()) side.pump(a, lds_outs);
        else __builtin_amdgcn_s_sleep(16);
        side.maybe_finish(a);
      }
    }
    // Then the weights, which do not depend on the gathered rows: their part of the first slabs is on its
    // way while the workgroup waits for its signals.
    pipe.request_b(ld, a, k_begin, KT);
    if (!wait_signals(a, m0, m1, lds_misc, lds_outs)) {
      // given up (a workgroup only gets to its wait with pieces left if its signals were there, so this
      // is for safety): the pieces it claimed still have to be moved, or their tiles' signals never come
      if constexpr (CARRY) {
        if (side.pending()) side.drain(a, lds_outs);
      }
      wait_vm_at_most<0>();        // nothing of this workgroup is left in flight towards its LDS
      trace_stamp(a, TRACE_END);
      return;
    }
    trace_stamp(a, TRACE_READY);
  }

  f32x4 acc[C::MI][C::NI];
#pragma unroll
  for (int mi = 0; mi < C::MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < C::NI; ++ni)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[mi][ni][e] = 0.f;
  const bool added = takes_peers_first<C, EPI>(a, mt, nt, is_split);       // (uniform)
  if constexpr (EPI == EPI_RS && C::BM * C::BN >= PEERS_FIRST_AREA) {
    if (added) {
      float* const ep = reinterpret_cast<float*>(pool) + wave * (32 * C::EP_STRIDE);
      if (a.R <= 4) sum_peers_first<C, EDGE, 3>(a, ep, acc, m0, n0, lane, wm, wn);
      else if (a.R <= 8) sum_peers_first<C, EDGE, 7>(a, ep, acc, m0, n0, lane, wm, wn);
      else sum_peers_first<C, EDGE, FLUX_MAX_RANKS - 1>(a, ep, acc, m0, n0, lane, wm, wn);
      __syncthreads();      // (the ring takes the place of other waves' staging areas)
    }
  }

  EarlyPeers<C> early;
  int n_early = 0;
  if constexpr (EPI == EPI_RS && EarlyPeers<C>::SMALL) n_early = early.template ask<EDGE>(a, is_split, m0, n0, lane, wm, wn);

  bool carries = false;
  if constexpr (CARRY) carries = side.pending();      // (uniform)
  constexpr bool WARM = PRO == PRO_NONE && C::BM == 256 && C::BN == 128;
  WarmA warm;
  if constexpr (WARM) warm.ask(a, ld.bytes_a, tid);
  pipe.start(ld, a, k_begin, KT, wave, carries);
  if constexpr (WARM) warm.drop();
  if (is_split && a.sk_share) part_started(a, tile, tid);
  int kt = 0;
  if constexpr (CARRY) {
    if (carries) {
      // With the transfer aboard (a workgroup of the first round with pieces to move; everybody else
      // runs the plain loop below): per slab two stores (of the vectors loaded two slabs ago) ahead of
      // the slab's operand loads and two loads right before the slab's wait.  "All but the two youngest
      // operations have completed" then means that the operand loads have landed (loads complete in
      // order, and those two are the youngest loads).  Thread 0 looks at the clock once per two slabs and
      // leaves word in LDS whether a tile is due to be counted in (a decision every wave must take
      // alike: finish() has barriers).  When the last tile is counted in, the plain loop takes over for the rest of K.
      // (The loop leaves A's last slab in LDS alone: the workgroup's shared words may lie there.)
      u32x4 dA0 = side.load(a, lds_outs), dA1 = side.load(a, lds_outs);
      u32x4 dB0 = side.load(a, lds_outs), dB1 = side.load(a, lds_outs);
      for (; kt + 2 <= KT && side.pending(); kt += 2) {
        side.store(a, dA0);
        side.store(a, dA1);
        pipe.template step<0, 2, Pipe::TWO_SLABS>(ld, a, k_begin, kt, KT, wave, acc, [&] {
          dA0 = side.load(a, lds_outs);
          dA1 = side.load(a, lds_outs);
        });
        side.store(a, dB0);
        side.store(a, dB1);
        bool look = false;
        pipe.template step<1, 2, Pipe::TWO_SLABS>(ld, a, k_begin, kt + 1, KT, wave, acc, [&] {
          look = side.may_be_due();       // (uniform)
          if (look) {
            if (tid == 0) *side.slot = side.due() ? 1 : 0;
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          }
          dB0 = side.load(a, lds_outs);
          dB1 = side.load(a, lds_outs);
        });
        if (look) {
          const int go = __builtin_amdgcn_readfirstlane(*side.slot);
          if (go) side.finish(a);           // (its barriers also keep the slot from being rewritten too early)
        }
      }
      if (side.pending()) {          // K is over before the transfer is: the vectors in flight first, then the rest
        side.store(a, dA0); side.store(a, dA1); side.store(a, dB0); side.store(a, dB1);
        side.ld_t = side.st_t; side.ld_s = side.st_s; side.ld_off = side.st_off;     // the loads start again where the stores are
        side.set_src(a, lds_outs, side.ld_t);
        side.drain(a, lds_outs);
      }
    }
  }
  pipe.run(ld, a, k_begin, KT, kt, wave, acc, carries);
  wait_vm0_and_barrier();        // the epilogue's staging area lies over slabs other waves may still be reading
  SharedWords* const tail_words = reinterpret_cast<SharedWords*>(pool + C::WORDS_AT_TAIL);
  if (EPI == EPI_RS && C::WORDS_IN_RING) {
    fill_lds_outs(a, tail_words->outs, tid);
    __syncthreads();
  }
  gemm_tail<C, EPI, EDGE, false, FLUX_MAX_RANKS - 1, PARTIALS>(a, pool, tail_words->misc, tail_words->outs, acc, tile, split, is_split, m0, n0, tid, lane, wave, wm, wn, added, early, n_early);
}

// The same kernel for reduce-scatter calls as a grid of resident workgroups, one per compute unit, each walking the block
// sequence with the grid's stride (block b, b + grid, ...: the order of Sec. 4.1 is kept, in time
// instead of in dispatch).
template <class C, int MAX_NP, int PARTIALS>
__global__ void __launch_bounds__(C::NT, C::OCC) gemm_kernel_dma_resident(const GemmArgs a_) {
  __shared__ __attribute__((aligned(1024))) unsigned char pool[C::POOL_BYTES];
  SharedWords* const words = reinterpret_cast<SharedWords*>(pool + C::WORDS_AT_TAIL);
  if (a_.persist_delay_ticks != 0 && ((blockIdx.x >> 3) & 1)) {
    const uint64_t t0 = wall_clock64();
    while (wall_clock64() - t0 < a_.persist_delay_ticks) __builtin_amdgcn_s_sleep(32);
  }
  const int n_blocks = a_.persist_blocks;
  for (int vb = (int)blockIdx.x; vb < n_blocks; vb += (int)gridDim.x) {
    // The argument block is read afresh for every block (the struct is the kernel's only argument and
    // lies at the start of the argument segment): fetched once before the loop, its hundred-odd scalars
    // would be kept in registers across the main loop, which has none to spare.
    typedef const GemmArgs __attribute__((address_space(4))) * ArgPtr;
    ArgPtr ap = (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(ap));
    const GemmArgs& a = *(const GemmArgs*)ap;
    // ... and so is everything a lane derives from its index (fragment addresses, load offsets)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / C::WAVES_N, wn = wave % C::WAVES_N;
    int tile, split;
    bool is_split;
    map_block(a, vb, tile, split, is_split);
    int mt, nt;
    tile_coord(a.tm, a.m_order, tile, mt, nt);
    const int m0 = mt * C::BM, n0 = nt * C::BN;
    trace_begin(a, tile, mt, nt, split, is_split, vb);
    const int k_begin = is_split ? split * a.k_per_split : 0;
    const int k_end = (is_split && k_begin + a.k_per_split < a.K) ? k_begin + a.k_per_split : a.K;
    const int KT = (k_end - k_begin) / C::BK;
    f32x4 acc[C::MI][C::NI];
#pragma unroll
    for (int mi = 0; mi < C::MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < C::NI; ++ni)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[mi][ni][e] = 0.f;
    DmaLoader<C, false> ld;
    ld.init(a, m0, n0, wave, lane);
    MmaPipe<C, false, false> pipe;
    pipe.init(pool, wm, wn, lane);
    pipe.start(ld, a, k_begin, KT, wave, false);
    if (is_split && a.sk_share) part_started(a, tile, tid);
    pipe.run(ld, a, k_begin, KT, 0, wave, acc, false);
    wait_vm0_and_barrier();
    fill_lds_outs(a, words->outs, tid);
    __syncthreads();
    EarlyPeers<C> none;
    gemm_tail<C, EPI_RS, false, true, MAX_NP, PARTIALS>(a, pool, words->misc, words->outs, acc, tile, split, is_split, m0, n0, tid, lane, wave, wm, wn, false, none, 0, vb);
    __syncthreads();      // the staging area and the shared words are the next block's
  }
}

}  // namespace flux
