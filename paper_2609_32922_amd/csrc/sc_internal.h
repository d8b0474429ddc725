// Internal definitions shared by the kernels and the host API of libscgemm.
//
// Data layout in device memory (all inside the caller's workspace):
//
//   status     one uint32 (bit 0: some L_i out of range), then one uint32: the longest
//              tile-pair cycle count of the call (256-row GEMM), then one uint32: nonzero
//              when some 256-row pair holds more row lengths that end inside a slot group
//              than the int8-chunk GEMM has masked tables (rslots; it then masks its
//              fragments), then one uint32: nonzero when a C-BSG call's tables serve.  Cleared
//              by k_draws (or k_schedule), or, int8-chunk GEMM, written by k_rprep
//   draws      rA[LBS], rB[LBS]                   uint32, comparator sequences (not with rgen)
//   CA         C-BSG only: CA[L][beta] = #{l < L : rA_l < beta}, uint16 [L_max+1][257]
//   plan       int8-chunk GEMM only: slot plans (see below), int4 {prefix, merged slots,
//              slots in all, 0} each, and their slots, uint2 [plan][LBS]
//   rtab       int8-chunk GEMM only: for each plan and 32-slot group G, the fp4 slot row of
//              every int8 byte for A and for B: uint4 [plan][LBS/32][2][256] (built once per
//              call, for the plans that some pair takes)
//   per batch entry b of A (batch entries):
//     perm[MT*BM]      sorted position -> original row (or -1 for padding)
//     Ls[MT*BM]        stream length at each sorted position
//     tileL[MT]        cycles the GEMM runs for row tile t: the longest L of the tile (of
//                      the tile pair with 256-row blocks), rounded up to 8
//     tileOff[MT]      word offset of tile t's planes inside Ap
//     pair[MT/2]       int8-chunk GEMM, in place of tileL and tileOff: int4 {longest, shortest
//                      length, distinct lengths, those not multiples of 32} of each 256-row
//                      pair (k_schedule), which k_rprep replaces with {32-slot groups, plan,
//                      slots the plan saves, slots of a row of L_max cycles}; then the batch
//                      entry's record {bad length, longest length rounded up to 8, bits of the
//                      plans its pairs take (two words)}
//     Ap               fp4 planes of A (or int8 chunks, below)
//   part       partial counts when GEMM tiles are split along the inner (element, cycle) range
//   units      vsplit only (k_rprep): the 256-row GEMM's work units {tile, first chunk step,
//              end chunk step, UNIT_PLAN * plan + partial index + 1 (0: none)} (int4), per tile {pieces, partial index
//              of piece 0} (int2), and per GEMM block the first of its units (uint32,
//              sk_slots + 1 of them)
//   per batch entry of B (1 if B is broadcast, else batch entries):
//     Bp               fp4 planes of B (or int8 chunks)
//
// Each stream bit is an fp4 (e2m1) value in {-1, 0, +1} ("nibble planes").  A slot is
// (octet o of 8 cycles, element quad dq of 4 elements) and holds 16 bytes: dword e =
// element 4*dq+e, nibble c = cycle 8*o+c, with value +1 (0x2), -1 (0xA) or 0.  Slots are
// ordered s = o * KQP + dq and each slot stores its 128 rows contiguously: A tile t is
// uint4 [Lloop/8 * KQP][128], B tile is uint4 [LBS/8 * KQP][128].  A row of length L has
// zero nibbles at cycles >= L.
//
// 256 x 256 GEMM blocks with comparator streams (rgen): no planes.  Ap and Bp hold the int8
// operands in 32-element chunks instead: pair t of 256 rows (A in the scheduler's order) is
// bytes [KC][256][32], byte e of row r of chunk c = element 32c + e, with -128 read as -127
// (the same comparator boundaries) and 0x80 (-128) marking an element >= K or a padding
// row.  The GEMM builds the fp4 fragments from them.
//
// 64-row blocks (tall): A's chunks a row tile each, bytes [KC][64][32]; B's as above, or with N <= 64 or
// 128 bytes [KC][64 or 128][32] (chunk_bits_b).
//
// N <= 128 with comparator streams (fused): no planes or chunks where streams are so short that laying
// them out costs more than it saves, or where they would not fit sc_gemm_noalloc's array or would add
// gigabytes (make_layout); the GEMM builds its fragments from the int8 rows themselves.
//
// A C-BSG call's tables (make_cbsg_layout): rows, chunks and partial sums of the int8-chunk GEMM in the
// memory of the planes, which are only written if the tables do not serve; the rest behind it all.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/scgemm.h"

static_assert(SC_KL_LIMIT == 8ll << 24, "K * L_max limit: MAX_SPLIT parts of 2^24 products");

namespace scg {

constexpr int BM = 128;          // rows of A per GEMM tile
constexpr int BN = 128;          // rows of B per GEMM tile
constexpr int LCH = 32;          // cycle granularity of the draw arrays and B's planes
constexpr uint32_t STATUS_BAD_LENGTH = 1u;
constexpr int DEFAULT_CUS = 256; // compute units of an MI355X, when no device can be queried
constexpr int MAX_SPLIT = 8;     // most parts a GEMM tile is split into along its inner range
constexpr int CBSG_L_MAX = 256;  // one period of the 8-bit Sobol sequences
constexpr int CA_COLS = 257;     // boundaries 0..256

constexpr int MSTEP = 8;         // cycles per octet (tile lengths padded to it)
constexpr int MSTAGE = 4;        // slots per LDS stage of the MFMA GEMM (2 MFMA k-steps)
constexpr int MFMA_BLOCKS_PER_CU = 2;   // resident 128-row MFMA GEMM blocks per CU (LDS bound)
constexpr double MFMA_QUAD_RATE = 1.1e13;  // products/s of one 256 x 256 GEMM block (one per CU)
constexpr double PART_BW = 3e12;           // bytes/s of writing and summing partial sums

// Estimated time of the 256-row GEMM with every tile split s ways (F = 0): the larger of
// the load per block slot and the longest unit, plus writing and summing the partial sums.  With
// one row length the units are equal and the load is whole rounds of them; with varying
// lengths the tiles come longest first, so the blocks fill in behind the long units and
// the load is the total over the CUs.  The host evaluates it with L_max, the GEMM kernels
// again with the longest tile pair of the call (both pick the same way among s).
__host__ __device__ inline double quad_split_time(int64_t tiles, int s, double perL, double Lmean,
                                                  double Lmax, bool one_length, int slots, double part_bytes) {
    const double avgT = perL * Lmean, maxT = perL * Lmax;
    const double load = one_length ? (double)((tiles * s + slots - 1) / slots) * avgT / s
                                   : (double)tiles * avgT / slots;
    const double red = s > 1 ? (double)tiles * (2 * s) * part_bytes / PART_BW + 5e-6 : 0.0;
    return (load > maxT / s ? load : maxT / s) + red;
}
// Slot plans of the int8-chunk GEMM.  The count of an element pair is a sum over cycles of
// zA_l zB_l, and cycle l's A bit is a function of the element's value alone: z = [n >= c],
// with n = q + 127 (bipolar) or |q| (unipolar) and c = the class of the draw r_l, the least n
// whose boundary lies above r_l.  There are only 254 (bipolar) or 127 (unipolar) classes, so
// cycles whose A draws share a class have the same A bit for every element, and their B bits
// can be added first: sum_l a b_l = a sum_l b_l.  The same holds with A and B swapped.  A slot
// is such a set of cycles; it holds +-1 (or 0) on one side and a sum of up to SLOT_CYCLES bits
// on the other, an integer of magnitude <= 4, which fp4 e2m1 represents exactly.  The cycles
// are edges between A classes and B classes, a slot takes the edges of one class, so the
// fewest slots are a minimum vertex cover: 88 of 128 cycles for bipolar streams, 140 of 256,
// 212 of 512, and 58 of 96, 90 of 192 for unipolar ones (means over seeds).  The sum over a
// slot's cycles is only right for rows that run all of them, so plan k covers the cycles
// below its prefix p_k, and cycle p_k + j keeps a slot of its own, S_k + j: a 256-row pair
// takes the plan with the largest prefix no longer than its shortest row, and a row of L >=
// p_k cycles ends after S_k + L - p_k slots.  Prefixes: multiples of pstep, and L_max.
//
// Large C-BSG calls whose rows all have L = L_max cycles take the same GEMM: A's bit of counter k is
// [k < c(n)], c(n) = #{l < L : class(rA_l) <= n}, so it is [n >= the (k + 1)-th smallest class of A's
// draws].  Bipolar: A holds sgn D_k = [k < c] - [k < L - c], the same at k and L - 1 - k, so the two
// share a slot: half the cycles.  The host cannot see the lengths, so it enqueues this path (first)
// and the planes path, and the one that does not serve returns at once.
constexpr int SLOT_CYCLES = 4;
constexpr int MAX_PLANS = 40;    // plans of a call (bits of the status words)
constexpr int PLAN_GROUPS = 512; // most (merged plan, group) tables of a call, 8 KiB each (the
                                 // plan of no cycle adds its L_max / 32: 640 in all at L_max = 4096)
constexpr int UNIT_PLAN = 1 << 24;   // a unit's partial index (below 2^22) and plan in one word

constexpr int TROWS = 64;        // rows of a block of k_tgemm
constexpr int64_t TALL_BYTES = 0x7FFFFFFC;   // largest output of a batch entry that k_tgemm decodes itself
constexpr int OCH = 8;           // octets per block of the nibble-plane generator
constexpr int RSLOTS = 4;        // int8-chunk GEMM: tables masked to a row length, per cycle group
constexpr int64_t MFMA_EXACT = 1ll << 24;   // products one fp32 accumulator sums exactly
// chunk steps whose counts fit int16: a step adds at most 32 x 32 products of magnitude 1 to a count
constexpr int64_t P16_STEPS = 32767 / (32 * 32);
constexpr int64_t RSTEP_EXACT = MFMA_EXACT / (32 * 32);   // int8-chunk GEMM chunk steps (32 cycles x
                                                          // 32 elements) one accumulator sums exactly
// Cost of a chunk step of the 256 x 64 int8-chunk GEMM in the work division, while all of a
// wave's row blocks run (RW1) and once only the first two do (RW2): half the MFMAs and two
// thirds of the table reads (measured on attention-V: 9/16 of a full step's time, against
// 8/16, 10/16 and 11/16).  The 256 x 256 blocks: a step of a group of 32 slots, and of a last
// group of at most 16 (half the MFMAs, the same number of wider-spread table reads)
constexpr int64_t RW1_WIDE = 8, RW2_WIDE = 5;
constexpr int64_t RW1_NARROW = 16, RW2_NARROW = 9;
// ... and once only the first one does (RW3: one A read and two MFMAs per k-step, beside two B
// reads; measured on attention-V: 5/16 against 3, 4, 7 and 9); the smallest of the three
constexpr int64_t RW3_NARROW = 5;
// The 256 x 64 blocks run two per CU, and the one dispatched first issues first: of the two
// ranges of a CU's pair of blocks, the first one's is RLEAD_NARROW / 16 longer than the
// average and the second one's as much shorter, so that both end together
constexpr int64_t RLEAD_NARROW = 4;

__host__ __device__ inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// comparator boundaries of an int8 value (bipolar, and unipolar magnitude).  -128 lies
// outside the quantiser's range; its boundaries equal those of -127 (0 bipolar, and a
// magnitude boundary at or above 256 unipolar: a one on every cycle), so the magnitude is
// capped at 127 and every boundary stays in [0, 256].
__device__ __forceinline__ int beta_bipolar(int q) { return (256 * (q + 127) + 127) / 254; }
__device__ __forceinline__ int beta_unipolar(int q) {
    const int a = q < 0 ? (q < -127 ? 127 : -q) : q;
    return (256 * a + 63) / 127;
}

__device__ __forceinline__ int wave_uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// classes of a draw r in [0, 255]: the least n = q + 127 (bipolar) or n = |q| (unipolar) whose
// boundary floor((256 n + 127) / 254) (floor((256 n + 63) / 127)) lies above r, so that
// [r < beta] = [n >= class]
__host__ __device__ inline int class_bipolar(int r) { return (254 * r + 127 + 255) >> 8; }
__host__ __device__ inline int class_unipolar(int r) { return (127 * r + 64 + 255) >> 8; }

// Inclusive scan across a 64-lane wave.
template <typename T>
__device__ __forceinline__ T wave_incl_scan(T v, int lane) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const T t = __shfl_up(v, o, 64);
        if (lane >= o) v += t;
    }
    return v;
}

// Exclusive scan over a block of NT threads; returns the block total in *total.
template <int NT, typename T>
__device__ T block_excl_scan(T v, T *total) {
    constexpr int NW = NT / 64;
    __shared__ T wsum[NW];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const T inc = wave_incl_scan(v, lane);
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    // (every thread adds up the waves before its own: NW <= 16 broadcast reads, no second scan)
    T base = 0, all = 0;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        const T x = wsum[k];
        if (k < w) base += x;
        all += x;
    }
    *total = all;
    __syncthreads();
    return base + inc - v;
}

template <typename T>
__device__ __forceinline__ T *ws_ptr(uint8_t *ws, size_t off) {
    return reinterpret_cast<T *>(ws + off);
}

struct Layout {
    int MT, NT;        // row tiles of A and B (NT rounded up to a multiple of mbn / 128, the
                       // B tiles one GEMM block takes)
    int LBS;           // cycle stride of B planes and length of draw arrays (L_max rounded to LCH)
    int nbB;           // batch entries of B planes (1 when B is broadcast)
    int KQP;           // element quads per octet, ceil(K/4) rounded up to 4
    int mbn;           // columns of B per GEMM block (256, or 128 when N <= 128)
    int fused;         // N <= 128, comparator streams, long A: the GEMM builds its fp4 fragments from
                       // the int8 operands (no planes or chunks in the workspace)
    int mbm;           // rows of A per GEMM block: 256 (row tiles taken in pairs that run at
                       // the pair's longest length; MT even) when mbn = 256 and MT > 1, else 128
    int rgen;          // 256-row GEMM with comparator streams: fragments built in the GEMM
                       // from int8 chunks and a per-group table (no planes)
    int tall;          // rgen in blocks of 64 rows x 128 tall columns (k_tgemm): columns of 32 per wave,
                       // 0 when the blocks have 256 rows
    int tshift, rtiles;    // rgen: rows of a tile (256, or 64 with tall) as a shift, and row tiles
    int cbsg;          // rgen: the tables of a C-BSG call whose rows all have L_max cycles (below)
    size_t off_skip;   // planes of such a call: a word that is nonzero when its tables serve (0: none)
    int halves;        // 256 x 256 blocks of rgen: a tile's last group of at most 16 slots runs half the MFMAs
    int narrow;        // rgen with N <= 64: blocks of 256 rows x 64 columns
    int rslots;        // rgen: tables masked to a row length per cycle group (0 when narrow)
    int KC;            // 32-element chunks per row, ceil(K/32)
    int cus;           // compute units of the device the call runs on
    int64_t words_per_L;   // plane words of one 128-row tile per cycle of its length
    int nplans, pstep;     // rgen: slot plans (1: every cycle has its own slot) and their spacing
    size_t off_rA, off_rB, off_status, off_CA, off_plan, off_pslots, off_rtab;
    size_t off_perm, off_Ls, off_tileL, off_tileOff, off_pair, off_Ap;
    size_t stride_batchA;          // bytes per A batch entry block
    size_t off_Bp;
    size_t stride_batchB;          // bytes per B batch entry block
    int S;             // splits of the inner range per GEMM tile (1 = no split)
    int Sleast;        // rgen: fewest parts that the tiles of a call with split tiles are run in
    int Smin;          // fewest splits that keep every part's fp32 sums exact (<= 2^24 products)
    int F;             // 256-row GEMM: tiles 0 .. F-1 run whole, tiles F.. in S parts each
    double q_perL, q_Lmean;   // 256-row GEMM split model: seconds per cycle of one tile, mean L
    int q_one;                // 256-row GEMM split model: all rows have one length
    int q_slots;              // 256-row GEMM split model: blocks that run at once
    double q_pbytes;          // 256-row GEMM split model: partial-sum bytes of one part (the
                              // columns a block computes: 256, or 64 with N <= 64)
    size_t off_part;   // partial counts of split tiles: [pieces][256 rows][pcols columns] int32
    int pcols;         // columns of a piece of partial counts: 256, or 64 for the 256 x 64 blocks
    int p16;           // int8-chunk GEMM split into parts of at most P16_STEPS chunk steps: the
                       // partial counts are int16 ([pieces][256 rows][pcols columns])
    int vsplit;        // int8-chunk GEMM with varying lengths: the tiles' chunk steps, end to
                       // end, are cut into sk_slots equal ranges, one per GEMM block (k_rprep)
    int sk_slots;      // vsplit: GEMM blocks, each running one range of the work
    size_t off_units, off_tinfo, off_slot;
    size_t total;
};

// Host-side layout computation for a device with `cus` compute units (no HIP calls).
// Returns false on overflow or when no split count up to MAX_SPLIT keeps the counts exact.
bool make_layout(const sc_gemm_desc &d, int cus, Layout *lay);
// The layout of a C-BSG call's tables behind its planes layout; false when it has none.
bool make_cbsg_layout(const sc_gemm_desc &d, int cus, const Layout &planes, Layout *lay);

// Kernel launchers (sc_kernels.hip).  All return hipSuccess or the launch error.
hipError_t launch_draws(uint64_t seed, int rng, int n, uint32_t *rA, uint32_t *rB,
                        uint8_t *bytes_out, int op_only, uint32_t *status, hipStream_t st);
// draws: also clear the status words and make the comparator sequences (one batch entry only);
// with rgen also the slot plans, with C-BSG planes also the table CA (from k_draws' sequences)
// planes (with the tables of a C-BSG call): the layout of its planes, for which the same launch
// writes all that k_draws and its own scheduler would, but the status words (k_rprep)
hipError_t launch_schedule(const sc_gemm_desc &d, const Layout &lay, const int32_t *L,
                           uint8_t *ws, bool draws, const Layout *planes, hipStream_t st);

// counting GEMM (sc_mfma.hip)
// Profiling events of the next launch_mgemm / launch_fgemm on this host thread (sc_gemm's
// prof_event_begin / end, NULL = none): its first kernel records begin when it starts and
// every kernel records end when it ends (the last one's stays), so the events time the GEMM
// kernels themselves, with no marker of their own in the stream.  gemm_events_taken() tells
// whether a kernel took them since set_gemm_events.
void set_gemm_events(hipEvent_t begin, hipEvent_t end);
bool gemm_events_taken();
hipError_t launch_mplanes(const sc_gemm_desc &d, const Layout &lay, const int8_t *A,
                          const int8_t *B, uint8_t *ws, hipStream_t st);
hipError_t launch_mgemm(const sc_gemm_desc &d, const Layout &lay, const float *sA, const float *sB,
                        float *out, int32_t *counts, uint8_t *ws, hipStream_t st);
hipError_t launch_fgemm(const sc_gemm_desc &d, const Layout &lay, const int8_t *A, const int8_t *B,
                        const float *sA, const float *sB, float *out, int32_t *counts, uint8_t *ws,
                        hipStream_t st);
hipError_t launch_rprep(const sc_gemm_desc &d, const Layout &lay, const int8_t *A, const int8_t *B,
                          uint8_t *ws, hipStream_t st);

// bytes of one batch entry of an operand from its first byte: (rows - 1) * ld + K
__host__ __device__ inline int64_t fused_extent(int rows, int64_t ld, int K) {
    return rows > 0 && K > 0 ? (int64_t)(rows - 1) * ld + K : 0;
}

// Where the scheduler of a C-BSG call's tables leaves what the planes path reads
struct PlanesOut {
    int MT, mbm, LBS;
    int64_t words_per_L;
    size_t off_perm, off_Ls, off_tileL, off_tileOff, off_rA, off_rB, off_CA, stride_batchA;
};

// cycles below which slot plan k merges (k < nplans), and the plan of a pair whose shortest row
// has L cycles
__host__ __device__ inline int plan_prefix(int k, int nplans, int pstep, int L_max) {
    return k == 0 ? 0 : k == nplans - 1 ? L_max : k * pstep;
}
__host__ __device__ inline int plan_of(int L, int nplans, int pstep, int L_max) {
    return nplans == 1 ? 0 : L >= L_max ? nplans - 1 : L / pstep;
}
// a kernel of the path (tables, or planes) that does not serve this C-BSG call
__device__ __forceinline__ bool not_serving(const Layout &lay, uint8_t *ws) {
    return (lay.cbsg && ws_ptr<uint32_t>(ws, lay.off_status)[3] == 0u) ||
           (lay.off_skip != 0 && *ws_ptr<uint32_t>(ws, lay.off_skip) != 0u);
}
// rows of a block of B's chunks as a shift (A's: Layout::tshift).  A function, as every kernel takes the
// layout as an argument: 8 bytes more of it (480 of arguments, not 472) cost a small call's launches 0.45 us
__host__ __device__ inline int chunk_bits_b(int tall, int N) {
    return !tall || N > 2 * TROWS ? 8 : N > TROWS ? 7 : 6;
}
// slots of a row of L cycles in a pair whose plan saves `save` slots and gives L_max `top` slots
// (top counts whole groups: the slots past the last cycle are zero)
__device__ __forceinline__ int slot_length(int L, int save, int top, int L_max) {
    return L <= 0 ? 0 : L >= L_max ? top : L - save;
}

// thresholds and ladder of the per-row length policy, passed by value to the kernel
struct MpParams {
    float tau[SC_MP_MAX_LEVELS];
    int32_t ladder[SC_MP_MAX_LEVELS];
    int32_t n;
};

// front end (sc_frontend.hip)
hipError_t launch_quantize(int batch, int rows, int K, const float *X, int64_t ldx, int64_t strideX,
                           int per_tensor, int8_t *Q, int64_t ldq, int64_t strideQ, float *scale,
                           float *rowmax, int64_t strideS, hipStream_t st);
hipError_t launch_mp_lengths(int batch, int M, const float *metric, int64_t strideM,
                             const MpParams &p, int32_t *L_out, int64_t strideL, hipStream_t st);

}  // namespace scg
