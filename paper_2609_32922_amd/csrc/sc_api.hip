// Host side of libscgemm: argument checks, workspace layout and the launch sequence.
// Every check runs before anything is enqueued; the library allocates nothing.
#include <limits.h>
#include <math.h>

#include <atomic>
#include <initializer_list>
#include <mutex>

#include "sc_internal.h"

namespace scg {

namespace {

// Slots that L cycles merge into (means over 40 seeds, rows all of length L; see the slot plans)
double mean_slots(double L, bool bipolar) {
    static const double at[] = {0, 32, 64, 96, 128, 192, 256, 384, 512, 1024, 4096};
    static const double bip[] = {0, 29, 52, 72, 88, 116, 140, 179, 212, 342, 1120};
    static const double uni[] = {0, 26, 44, 58, 70, 90, 106, 138, 172, 304, 1072};
    int k = 1;
    while (k < 10 && L > at[k]) ++k;
    const double *v = bipolar ? bip : uni, f = (L - at[k - 1]) / (at[k] - at[k - 1]);
    return v[k - 1] + f * (v[k] - v[k - 1]);
}

// What a layout is chosen by: estimated times (us) of the int8-chunk GEMM.  A chunk step of a 256 x
// 256 block (one per CU) takes 3.5, its first loads and decode 23 (10 for a part); one of a 64 x
// 128 C block 1.55, 2.15, 4.05, 5.5 for C = 1, 2, 4, 5 while two run on the CU and 1.4, 1.55, 2.7,
// 3.3 alone, its other costs 5 + 0.36 C and 1.7 a slot group; partial sums move at 5e6 bytes a us,
// and the launch that adds them up takes 4.3.  (Fitted to 75 shapes, 14 divisions each: over them
// the chosen division takes 1.005 times the best one's whole-call time on average, 1.18 at most.)
struct WorkShape {
    double batch, KC, gmean, gmax;   // 32-element chunks; 32-slot groups of the mean and the longest row
    int M, N, cus, Smin;
    bool one;                        // one row length
};
double est_parts(double pieces, double bytes) { return pieces * bytes * 2.0 / 5e6 + 4.3; }
double est_wide(const WorkShape &w) {
    const double tiles = w.batch * ((w.M + 255) / 256) * ((w.N + 255) / 256), n = w.KC * w.gmean, part = 256.0 * 256 * 4;
    if (!w.one) return tiles * (23 + 3.5 * n) / w.cus + 13 + est_parts(2.0 * w.cus, part) * (tiles > w.cus ? 0.5 : 1.0);
    double best = 1e30;
    for (int S = w.Smin; S <= MAX_SPLIT && (S == w.Smin || n / S >= 2); S *= 2) {
        const double t = S == 1 ? ceil(tiles / w.cus) * (23 + 3.5 * n)
                                : ceil(tiles * S / w.cus) * (10 + 3.5 * n / S) + est_parts(tiles * S, part);
        best = t < best ? t : best;
    }
    const double rest = fmod(tiles, w.cus);
    if (w.Smin == 1 && tiles > w.cus && rest > 0) {
        const double S = fmin(floor(w.cus / rest), MAX_SPLIT);
        best = fmin(best, floor(tiles / w.cus) * (23 + 3.5 * n) + 10 + 3.5 * n / S + (S > 1 ? est_parts(rest * S, part / 2) : 7));
    }
    return best;
}
double est_tall(const WorkShape &w, int C, int S) {
    const double step2 = C == 1 ? 1.55 : C == 2 ? 2.15 : C == 4 ? 4.05 : 5.5;
    const double step1 = C == 1 ? 1.4 : C == 2 ? 1.55 : C == 4 ? 2.7 : 3.3;
    const double units = w.batch * ((w.M + 63) / 64) * ((w.N + 128 * C - 1) / (128 * C)) * S;
    const double n = w.KC * w.gmean / S, fixed = 5 + 0.36 * C + 1.7 * ceil(w.gmean / S), slots = 2.0 * w.cus;
    const double two = fixed + n * step2, alone = fixed + n * step1;
    double t;
    if (w.one) {
        const double rest = fmod(units, slots);
        t = floor(units / slots) * two + (rest == 0 ? 0 : rest <= w.cus ? alone : two);
    } else {
        // (units go out longest first)
        t = units <= w.cus ? 0 : units / slots * two + 0.58 * two;
        t = fmax(t, fixed + w.KC * w.gmax / S * (units <= w.cus ? step1 : step2));
    }
    if (S > 1) t += est_parts(units, 64.0 * 128 * C * (w.KC * w.gmax / S <= P16_STEPS ? 2 : 4));
    return t;
}

// fewest chunk steps of a part of a 64-row tile
constexpr int TPART = 4;

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

// checked size arithmetic: returns false on overflow of size_t
bool mul_ok(size_t a, size_t b, size_t *r) {
    if (a != 0 && b > SIZE_MAX / a) return false;
    *r = a * b;
    return true;
}

}  // namespace

// Compute units of the current device (the width over which the GEMM's work is divided),
// cached per device; DEFAULT_CUS when no device can be queried (e.g. sizing a workspace on
// a host without a GPU).
static int device_cus() {
    static std::atomic<int> cache[64];
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) {
        (void)hipGetLastError();
        return DEFAULT_CUS;
    }
    if (dev < 64) {
        const int c = cache[dev].load(std::memory_order_relaxed);
        if (c > 0) return c;
    }
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
        (void)hipGetLastError();
        return DEFAULT_CUS;
    }
    if (dev < 64) cache[dev].store(n, std::memory_order_relaxed);
    return n;
}

// How much of the workspace a layout may spend: everything; slot plans of no cycle and of all cycles
// only; no slot plans; int8 chunks only where the 128-row kernels could not take their operands as they are
enum { LAY_FULL, LAY_TWO_PLANS, LAY_ONE_PLAN, LAY_LEAST };

// cbsg: of the tables of a C-BSG call (d's source is then taken as the LFSR); parts: fewer than MAX_SPLIT,
// 64-row blocks in at most so many parts (if exactness allows), or 256-row blocks (0); est: the estimated
// time that the blocks were chosen by
static bool layout_with(const sc_gemm_desc &d, int cus, int spend, bool cbsg, Layout *lay, int parts = MAX_SPLIT,
                        double *est = nullptr) {
    Layout l{};
    l.cbsg = cbsg;
    l.cus = cus > 0 ? cus : DEFAULT_CUS;
    l.KQP = (int)round_up((d.K + 3) / 4, 4);
    l.words_per_L = (int64_t)l.KQP * 64;
    l.MT = (d.M + BM - 1) / BM;
    l.NT = (d.N + BN - 1) / BN;
    const bool lfsr = d.rng == SC_RNG_LFSR32 || cbsg;
    const double Lmean = d.L_hint > 0 ? d.L_hint : d.L_max;
    const int KC = (d.K + 31) / 32;
    const bool one_length = Lmean >= d.L_max, long_tiles = (int64_t)KC * ((int64_t)(Lmean + 31) / 32) >= 16;
    // N <= 64 with comparator streams and M > 128: the int8-chunk GEMM in blocks of
    // 256 rows x 64 columns (the B side still laid out as one 256-row pair)
    l.narrow = lfsr && d.N <= 64 && d.M > BM;
    // comparator streams with few rows or columns, or short tiles with varying lengths
    // (attention heads): the int8-chunk GEMM in blocks of 64 rows
    const bool few = lfsr && !l.narrow && (d.M <= BM || d.N <= BN);
    // few columns and no chunks of A: k_fgemm takes the operands as they are (operand offsets must fit 31 bits)
    l.fused = few && spend == LAY_LEAST && d.N <= BN && fused_extent(d.M, d.lda, d.K) < INT_MAX - 4 &&
              fused_extent(d.N, d.ldb, d.K) < INT_MAX - 4;
    // Blocks of 64 rows x 128 C columns in S parts where that is estimated to take the least time:
    // few rows or columns, short tiles with varying lengths (attention heads), and shapes that
    // 256 x 256 blocks pad or fill the chip unevenly with.  Measured (us, 256-row blocks against
    // these): 48 x 768 x 3072 135 (128-row kernels, since gone) and 32; 197 x 768 x 3072 75 and 51;
    // 400 x 768 x 768 67 and 38; 128 heads of 577 x 64 x 577 412 and 199; and 6304 x 768 x 3072 375
    // and 429, 18464 x 1024 x 4096 2150 and 2280, where the 256-row blocks stay.
    WorkShape w{};
    w.batch = d.batch > 0 ? d.batch : 0;
    w.KC = KC;
    w.M = d.M;
    w.N = d.N;
    w.cus = l.cus;
    w.one = one_length;
    const bool bip = d.polarity == SC_BIPOLAR_XNOR;
    // (C-BSG: counters k and L - 1 - k share a slot, or nearly none of B's classes repeat up to 128)
    const double slots = !cbsg ? mean_slots(Lmean, bip) : bip ? (d.L_max + 1) / 2 : fmin(d.L_max, 127);
    w.gmean = ceil(slots / 32.0);
    w.gmax = one_length ? w.gmean : (d.L_max + 31) / 32;
    const int64_t rsteps = (int64_t)KC * ((d.L_max + 31) / 32);
    w.Smin = 1;
    while (rsteps > RSTEP_EXACT * w.Smin) w.Smin *= 2;
    // (few rows or columns: any number of parts, for every K x L_max of at most 2^27 products in
    // whole octets of cycles and 16-element steps)
    if (few) w.Smin = (int)((rsteps + RSTEP_EXACT - 1) / RSTEP_EXACT);
    if (few && round_up(d.L_max, MSTEP) * l.KQP * 4 > SC_KL_LIMIT) return false;
    if (w.Smin < 1) w.Smin = 1;
    // (an output past 31-bit offsets is decoded by the split-sum pass, so it takes parts)
    const bool far = ((int64_t)(d.M - 1) * d.ldo + d.N) * 4 > TALL_BYTES;
    if (far && few && w.Smin < 2) w.Smin = 2;
    int tallC = 0, tallS = 1;
    if (lfsr && !l.narrow && !l.fused && (few || (spend != LAY_LEAST && !far))) {
        double best = few || (parts > 0 && parts < MAX_SPLIT) ? 1e30 : est_wide(w);
        for (int c : {1, 2, 4, 5})
            for (int S = w.Smin; (few || parts > 0) && S <= (c == 5 ? 1 : w.Smin > parts ? w.Smin : parts); ++S) {
                if (S > w.Smin && w.KC * w.gmean / S < TPART) break;
                // (units are counted in 32 bits)
                if (w.batch * ((d.M + TROWS - 1) / TROWS) * ceil(d.N / (128.0 * c)) * S > INT_MAX) break;
                const double t = est_tall(w, c, S);
                if (t < best) {
                    best = t;
                    tallC = c;
                    tallS = S;
                }
            }
        if (est != nullptr) {
            // (without plans a slot is a cycle)
            if (spend == LAY_ONE_PLAN || (spend == LAY_TWO_PLANS && !one_length)) {
                w.gmean = ceil(Lmean / 32.0);
                w.gmax = (d.L_max + 31) / 32;
            }
            *est = tallC > 0 ? est_tall(w, tallC, tallS) : est_wide(w);
        }
    }
    const bool tall = tallC > 0;
    if (few && !tall && !l.fused) return false;
    l.mbn = (l.NT > 1 || l.narrow || tall) && !l.fused ? 2 * BN : BN;
    l.NT = (int)round_up(l.NT, l.mbn / BN);
    l.mbm = ((l.MT > 1 && l.mbn == 2 * BN) || tall) ? 2 * BM : BM;
    if (l.mbm == 2 * BM) l.MT = (int)round_up(l.MT, 2);
    // comparator streams: fragments from int8 chunks and a table of each slot group, so the
    // operands are read as bytes instead of as fp4 planes
    l.rgen = l.mbm == 2 * BM && lfsr;
    l.tshift = tall ? 6 : 8;
    l.rtiles = tall ? (d.M + TROWS - 1) / TROWS : l.MT / 2;
    const int bbits = chunk_bits_b(tallC, d.N);
    l.rslots = l.narrow || tall ? 0 : RSLOTS;
    l.halves = l.rgen && !l.narrow && !tall;
    l.KC = (d.K + 31) / 32;
    l.LBS = (int)round_up(d.L_max, LCH);
    l.nbB = (d.strideB == 0) ? 1 : d.batch;
    if (l.nbB < 1) l.nbB = 1;

    // the status word is always the first word of the workspace
    size_t off = 0;
    l.off_status = off;
    off = align256(off + 8 * 4);
    // (the int8-chunk GEMM's sequences are in its plans' slots)
    l.off_rA = off;
    if (!l.rgen) off = align256(off + (size_t)l.LBS * 4);
    l.off_rB = off;
    if (!l.rgen) off = align256(off + (size_t)l.LBS * 4);
    l.off_CA = off;
    if (!lfsr) off = align256(off + (size_t)(d.L_max + 1) * CA_COLS * 2);
    // Slot plans: while a tile's products sum to less than 2^24 in magnitude whatever slots hold
    // them (K x L_max; so every part is exact), and more than one group of 32 cycles exists.
    // At most 32 plans past the first, and at most PLAN_GROUPS tables of theirs (past the first's).
    l.nplans = 1;
    l.pstep = LCH;
    if (spend <= LAY_TWO_PLANS && !cbsg && l.rgen && l.LBS > 32 && (int64_t)l.KC * 32 * l.LBS < MFMA_EXACT) {
        const int n = spend == LAY_TWO_PLANS ? 1 : PLAN_GROUPS / (l.LBS / 32) < 32 ? PLAN_GROUPS / (l.LBS / 32) : 32;
        l.pstep = (int)round_up((d.L_max + n - 1) / n, 8);
        l.nplans = 1 + (d.L_max + l.pstep - 1) / l.pstep;
    }
    l.off_plan = off;
    if (l.rgen) off = align256(off + (size_t)l.nplans * 16);
    l.off_pslots = off;
    if (l.rgen) off = align256(off + (size_t)l.nplans * l.LBS * 8);
    l.off_rtab = off;
    if (l.rgen) off = align256(off + (size_t)l.nplans * (l.LBS / 32) * 512 * 16);

    // one A block per batch entry
    const size_t rowsA = (size_t)l.MT * BM;
    size_t a = 0, sz;
    l.off_perm = a;
    a = align256(a + rowsA * 4);
    l.off_Ls = a;
    a = align256(a + rowsA * 4);
    l.off_tileL = a;
    if (!l.rgen) a = align256(a + (size_t)l.MT * 4);
    l.off_tileOff = a;
    if (!l.rgen) a = align256(a + (size_t)l.MT * 8);
    l.off_pair = a;
    if (l.rgen) a = align256(a + (size_t)(l.rtiles + 1) * 16);
    l.off_Ap = a;
    // largest planes of one batch entry: every tile at L_max rounded up to an octet
    if (!mul_ok((size_t)l.MT * (size_t)l.words_per_L, (size_t)round_up(d.L_max, MSTEP) * 4, &sz))
        return false;
    if (l.fused) sz = 0;
    if (l.rgen && !mul_ok((size_t)l.rtiles << l.tshift, (size_t)l.KC * 32, &sz)) return false;
    a = align256(a + sz);
    l.stride_batchA = a;
    const size_t baseA = off;
    size_t totA;
    if (!mul_ok(a, (size_t)(d.batch > 0 ? d.batch : 0), &totA)) return false;
    off += totA;

    // one B block per distinct B batch entry
    const size_t rowsB = (size_t)l.NT * BN;
    size_t bb = 0;
    l.off_Bp = bb;
    if (!mul_ok((size_t)l.NT * (size_t)l.words_per_L, (size_t)l.LBS * 4, &sz)) return false;
    if (l.fused) sz = 0;
    if (l.rgen && !mul_ok(bbits < 8 ? (size_t)1 << bbits : rowsB, (size_t)l.KC * 32, &sz)) return false;
    bb = align256(bb + sz);
    l.stride_batchB = bb;
    const size_t baseB = off;
    size_t totB;
    if (!mul_ok(bb, (size_t)l.nbB, &totB)) return false;
    off += totB;

    // Exactness of the counts: a GEMM part sums its products into fp32 accumulators, which
    // stay exact integers while a part holds at most 2^24 products per output.  Units of the
    // inner range and products per unit of each GEMM: (32-cycle group, 32-element chunk) =
    // 1024 (int8-chunk GEMM); stage of 4 slots = 128 (fused GEMM); k-step of 2 slots = 64.
    // A part takes at most ceil(units / S) units, so S is at least Smin; the parts' int32
    // partial sums are then added exactly.
    const int64_t octs = round_up(d.L_max, MSTEP) / MSTEP;
    const int64_t units = l.rgen ? (int64_t)(l.LBS / 32) * l.KC
                                 : l.fused ? octs * (l.KQP / MSTAGE) : octs * (l.KQP / 2);
    const int64_t per_unit = l.rgen ? 32 * 32 : l.fused ? 128 : 64;
    l.Smin = 1;
    while (l.Smin <= MAX_SPLIT && (units + l.Smin - 1) / l.Smin * per_unit > MFMA_EXACT) l.Smin *= 2;
    if (few && tallC > 0) l.Smin = w.Smin;
    else if (l.Smin > MAX_SPLIT) return false;

    int64_t tiles = (int64_t)(d.batch > 0 ? d.batch : 0) * (l.MT / (l.mbm / BM)) * (l.NT / (l.mbn / BN));
    l.tall = tallC;
    if (tall) {
        tiles = (int64_t)(d.batch > 0 ? d.batch : 0) * l.rtiles * (((int64_t)d.N + 128 * tallC - 1) / (128 * tallC));
    }

    // Division of the GEMM tiles into work units.
    const bool quad = l.mbm == 2 * BM && !tall;
    // indivisible steps along the inner range per cycle (chunks of every 32-cycle group with rgen)
    const int kunits = l.rgen ? l.KC * (l.LBS / 32) : l.KQP / 2;
    const int smax = kunits > l.Smin ? kunits : l.Smin;
    // partial-sum bytes of one part (256-row blocks of N <= 64 compute 64 columns)
    const double tile_bytes = (double)l.mbm * (l.narrow ? 64 : l.mbn) * 4.0;
    l.S = l.Smin;
    l.F = 0;
    if (tall) {
        l.S = tallS;
    } else if (quad && tiles > 0) {
        // 256 x 256 tiles, one block per CU, taking whole tiles or parts of tiles
        // (quad_split_time).  Candidates: every tile split s ways (F = 0), or whole tiles in
        // full rounds with the tiles of a last partial round split to fill one round.  Split
        // counts are powers of two: units are dealt to the eight XCDs round-robin, so each
        // XCD then holds units of one k-range, whose operand slots its blocks read
        // together from its L2 (three-way splits measured slower than four-way).  With
        // F = 0 the GEMM kernels may lower s again with the actual longest tile pair
        // (measured: 6304 x 768 x 3072 with L in [16, 256], mean 64, longest 172: the GEMM
        // takes 0.49 ms split two ways against 0.61 ms three ways), never below Smin.
        // (the 64-column blocks of N <= 64 do a quarter of the work and run two per CU)
        l.q_perL = (double)l.mbm * (l.narrow ? 64 : l.mbn) * 4.0 * l.KQP / MFMA_QUAD_RATE;
        l.q_slots = l.narrow ? 2 * l.cus : l.cus;
        l.q_Lmean = Lmean;
        l.q_pbytes = tile_bytes;
        l.q_one = one_length;
        const double avgT = l.q_perL * Lmean, maxT = l.q_perL * d.L_max;
        double best = 0.0;
        for (int s = l.Smin; s <= MAX_SPLIT && s <= smax; s *= 2) {
            const double est = quad_split_time(tiles, s, l.q_perL, Lmean, d.L_max, l.q_one != 0, l.q_slots,
                                               l.q_pbytes);
            if (s == l.Smin || est < best * 0.97) {
                best = est;
                l.S = s;
            }
        }
        // (the tail's split fills the last round as closely as it can: its units are few
        // and short, so balance counts for more there than a shared k-range per XCD)
        const int64_t R = tiles % l.q_slots;
        int s2 = R > 0 ? (int)(l.q_slots / R) : 1;
        s2 = s2 > MAX_SPLIT ? MAX_SPLIT : s2;
        if (s2 > kunits) s2 = kunits;
        if (l.Smin == 1 && tiles >= l.q_slots && R > 0 && s2 > 1) {
            const double red = (double)R * (2 * s2) * tile_bytes / PART_BW + 5e-6;
            const double est = fmax((double)(tiles / l.q_slots) * avgT + avgT / s2, maxT) + red;
            if (est < best * 0.97) {
                best = est;
                l.F = (int)(tiles - R);
                l.S = s2;
            }
        }
        // (256 x 64 blocks: the last pair of each batch entry, if it holds at most half its rows, runs at
        // most half its row blocks (a step then 9/16 of a full one, 5/16 with at most 32 rows).  A last round
        // of such tiles alone stays whole while parts would save few steps: parts and the launch that
        // sums them cost 10 to 20 us, less for the fewer tiles of more parts.  Measured, whole against parts
        // (us): the compensator, 16 x 8224 rows, 3 steps saved, 65 and 68; 256 x 550 x 64 x 577 at L = 256,
        // 21 of 2 parts, 289 and 306; and 128 x 1099 x 64 x 577, 40 of 4 parts, 323 and 310; 64 x 2115 x
        // 64 x 256 at L = 512, 24 of 8 parts, 181 and 172)
        const double saved = w.KC * w.gmean * (d.M % 256 <= 32 ? RW3_NARROW : RW2_NARROW) / RW1_NARROW * (1.0 - 1.0 / l.S);
        if (l.F > 0 && l.narrow && d.M % 256 > 0 && d.M % 256 <= 128 && R <= (int64_t)d.batch * (l.NT / 2) &&
            saved <= (l.S > 4 ? 12 : 24))
            l.S = 1;
        if (l.S == 1) l.F = (int)tiles;
    } else if (tiles > 0 && kunits > 1) {
        // 128-row tiles: every tile split s ways.  Estimated time of split s: the busiest
        // slot (a resident block) runs ceil(units/slots) units of average work, plus the
        // excess of the heaviest unit over the average, plus, for s > 1, writing and summing
        // s partial tiles.  Units are dealt to the eight XCDs round-robin, so s is a power of
        // two: each XCD then keeps one k-range of its tiles, and its L2 serves that range to
        // all of them.  Rates are the measured order of magnitude: 4.8e12 products/s per
        // resident block (two per CU); partial sums at 3e12 B/s.
        const int slots = l.cus * MFMA_BLOCKS_PER_CU;
        const double rate = 4.8e12;
        const double per_L = (double)BM * l.mbn * 4.0 * l.KQP;
        double best = 0.0;
        for (int s = l.Smin; s <= MAX_SPLIT && s <= smax; s *= 2) {
            const int64_t nunits = tiles * s;
            const double avg_u = per_L * Lmean / s, max_u = per_L * d.L_max / s;
            const double gemm = ((double)((nunits + slots - 1) / slots) * avg_u + (max_u - avg_u)) / rate;
            const double red = s > 1 ? (double)tiles * (2 * s) * tile_bytes / 3e12 + 5e-6 : 0.0;
            if (s == l.Smin || gemm + red < best * 0.97) {
                best = gemm + red;
                l.S = s;
            }
        }
    }
    // Int8-chunk GEMM with varying lengths: the work of a tile follows its rows' lengths
    // (Sec. 4.1: the cost follows the sum of the l_i), known only on the device.  There the
    // tiles' chunk steps are laid end to end and cut into sk_slots equal ranges, one per GEMM
    // block (k_rprep): a tile inside a range runs whole, one that a cut crosses runs in
    // pieces that the split-sum pass adds.  A range holds at most RSTEP_EXACT steps, so every
    // whole tile and piece sums exactly.
    // (Short tiles, a few chunk steps each, keep the division below: their pieces' partial sums
    // and their in-GEMM decodes would cost as much as the steps; ViT-L/14 Q.K^T heads with
    // K = 64 took 0.61 ms cut into ranges against 0.41 ms split alike.)
    l.pcols = tall ? 128 * l.tall : l.narrow ? 64 : l.mbn;
    l.vsplit = quad && l.rgen && tiles > 0 && !l.q_one && long_tiles;
    l.off_units = off;
    int64_t pieces = quad ? (tiles - l.F) * (int64_t)l.S : tiles * (int64_t)l.S;
    if (l.vsplit) {
        // Ranges so many that no unit, a run of one tile's steps within a range, passes RSTEP_EXACT: any
        // number while a tile's own steps do not.  Longer tiles: k_rprep weighs a step at most w1 and at
        // least w2 and adds at most 7 w1 per tile for its decode and a minimum step: W <= w1 wmax, a range
        // costs T = ceil(W / sl) <= w1 wmax / sl + 1 (256 x 64 blocks: up to twice that) and holds at most
        // T / w2 + 1 steps.  The 256 x 256 blocks run no half groups there, so that w2 = w1.  (Lighter steps
        // in this rule, whatever the tile's length, grew the partial sums of long calls 1.6 times: 136 -> 217
        // GB for 406072 x 87105 x 5304 at L = 1579; a half group saves at most 3/8 of one of 17 or more.)
        const int64_t tsteps = (int64_t)l.KC * (l.LBS / 32), wmax = tiles * (tsteps + 7);
        if (tsteps > RSTEP_EXACT) l.halves = 0;
        const int64_t w1 = l.narrow ? RW1_NARROW : RW1_WIDE, w2 = l.narrow ? RW3_NARROW : w1;   // (w2: the lightest step)
        const int64_t den = (w2 * (RSTEP_EXACT - 2) - 1) / (l.narrow ? 2 : 1);
        int64_t sl = l.q_slots;
        if (tsteps > RSTEP_EXACT && w1 * wmax > sl * den) sl = (w1 * wmax + den - 1) / den;
        // (refused: a call that would fill 2^20 ranges, whether or not it needs as many)
        const int64_t refused = l.narrow ? w1 * wmax - den * (1 << 20) : wmax - (RSTEP_EXACT - 3) * (1 << 20);
        if (refused > 0) return false;
        l.sk_slots = (int)sl;
        l.F = 0;
        l.S = 1;
        off = align256(off + (size_t)(tiles + sl) * 16);
        l.off_tinfo = off;
        off = align256(off + (size_t)tiles * 8);
        l.off_slot = off;
        off = align256(off + (size_t)(sl + 1) * 4);
        // a cut inside a tile adds one piece to it and may make it a split tile: at most two
        // pieces per cut
        pieces = 2 * sl;
    }
    // Parts of the int8-chunk GEMM's split tiles of at most P16_STEPS chunk steps store int16
    // partial counts (half the partial-sum traffic).  A part of S has at most ceil(steps / S)
    // of a tile's steps; with F = 0 the GEMM may lower S to Smin.
    l.Sleast = tall || l.F > 0 ? l.S : l.Smin;
    if (l.rgen && !l.vsplit && l.S > 1) {
        const int64_t smin = l.Sleast;
        // (a step of a C-BSG call's slots, two cycles each, twice as much)
        const bool two = cbsg && bip;
        const int64_t steps = (int64_t)l.KC * (two ? ((d.L_max + 1) / 2 + 31) / 32 : l.LBS / 32);
        l.p16 = (steps + smin - 1) / smin <= P16_STEPS / (two ? 2 : 1);
    }
    l.off_part = off;
    if (pieces > 0 && (l.S > 1 || l.vsplit)) {
        size_t partb;
        // every piece is [mbm rows][pcols columns] of int32 (int16 with p16)
        if (!mul_ok((size_t)pieces, (size_t)(tall ? TROWS : l.mbm) * (size_t)l.pcols * (l.p16 ? 2 : 4), &partb)) return false;
        off = align256(off + partb);
    }

    // make every offset absolute for batch entry 0
    l.off_perm += baseA;
    l.off_Ls += baseA;
    l.off_tileL += baseA;
    l.off_tileOff += baseA;
    l.off_pair += baseA;
    l.off_Ap += baseA;
    l.off_Bp += baseB;
    l.total = off;
    *lay = l;
    return true;
}

// Most bytes that plans and chunks may add to a call's workspace.  An operand's chunks are as large as the
// operand (31 x at K = 1), so without a bound a call whose operands nearly fill the card would no longer
// fit it: 128 x 1272922 x 93 x 243 takes 1.3 GB in k_fgemm and 43 GB in chunks beside 263 GB of operands.
static constexpr size_t MOST_EXTRA = (size_t)8 << 30;
bool make_layout(const sc_gemm_desc &d, int cus, Layout *lay) {
    if (!layout_with(d, cus, LAY_FULL, false, lay)) return layout_with(d, cus, LAY_LEAST, false, lay);
    // Few columns and lengths of 8 cycles or less on average: k_fgemm runs octets of cycles, a quarter of the
    // 32-slot groups, and lays out no chunks, but at half the rate.  Taken where reading the operands (0.67 us a
    // MB), writing and reading A's chunks (0.39, padding rows too) and the fixed cost of 64-row blocks outweigh
    // its stages (16 elements of an octet; two blocks a CU), with a wider margin where lengths differ; or, many
    // rows, by A's chunks alone (1.1 us a MB).  Fitted to 3400 calls: 108 of them are 10 % slower than in
    // k_fgemm and 12 than in 64-row blocks (by A's chunks alone, which leaves out batches of few rows and of a
    // B each: 325 and 6).  (us, 64-row blocks against k_fgemm: 24589 x 116 x 1983 at L = 8 148 and 105;
    // 8 x 45067 x 87 x 3067 1524 and 1015; 564 x 79 x 128 x 378, a B each, at L = 7 93 and 67; 2196 x 114 x 71 24 and 32; lengths up
    // to 16 with a mean of 8, 40413 x 118 x 2959 262 and 182, 8 x 3811 x 79 x 1032 82 and 84.)
    const int Lmean = d.L_hint > 0 ? d.L_hint : d.L_max;
    Layout taken;
    const bool few_short =
        lay->tall && d.N <= BN && Lmean <= MSTEP && layout_with(d, cus, LAY_LEAST, false, &taken) && taken.fused;
    double rounds = 0, octets = 0, chunks = 0, operands = 0;
    if (few_short) {
        rounds = (double)d.batch * taken.MT * taken.S / (MFMA_BLOCKS_PER_CU * taken.cus);
        const double stages = (double)(taken.KQP / MSTAGE) / taken.S, longest = ceil((double)d.L_max / MSTEP);
        const double load = stages * (rounds <= 0.5 ? 1.0 : Lmean >= d.L_max ? ceil(rounds) : fmax(rounds, 1.0));
        octets = fmax(load * fmin(fmax((Lmean + 6.0) / MSTEP, 1.0), longest), stages * longest);
        chunks = (double)d.batch * lay->rtiles * lay->KC * (TROWS * 32 / 1e6);
        operands = ((double)d.batch * d.M + (double)lay->nbB * d.N) * d.K / 1e6;
        const double saved = 0.39 * chunks + 0.67 * operands + 2.5 * rounds;
        if (d.L_max <= MSTEP ? saved > 0.41 * octets + 5.2
                             : (d.L_max <= 2 * MSTEP && saved > 0.6 * octets + 15) ||
                                   (d.M > BM && 1.1 * chunks > 0.8 * load + 3 * rounds + 25))
            *lay = taken;
    }
    if (lay->total > MOST_EXTRA) {
        Layout least;
        if (layout_with(d, cus, LAY_LEAST, false, &least) && least.total < lay->total - MOST_EXTRA) *lay = least;
    }
    // A call that fits sc_gemm_noalloc's array in some layout keeps fitting it (sc_gemm_workspace_size reports
    // what both entry points use, so sc_gemm pays for it too): of those that fit, the one with the least
    // estimated time among fewer parts, fewer plans and no plans, or else the one without chunks.
    // (500 calls of up to 9000 rows, with 64 to 220 MiB in full: 1.06 times the full layout's time in the
    // middle, where going without plans at once took 1.68 times, as long as before there were any.  2200 x
    // 1024 x 1024 at L = 256: 66.6 MiB in 7 parts, 57.8 in 6)
    if (lay->total <= SC_NOALLOC_WORKSPACE_BYTES) return true;
    Layout best, l;
    double least_t = 1e30;
    auto consider = [&](int spend, int parts) {
        double t = 1e29;
        if (!layout_with(d, cus, spend, false, &l, parts, &t) || l.total > SC_NOALLOC_WORKSPACE_BYTES) return false;
        if (t < least_t) {
            best = l;
            least_t = t;
        }
        return true;
    };
    // (a call that fits neither without plans nor without chunks never did)
    if (!consider(LAY_ONE_PLAN, MAX_SPLIT) && !consider(LAY_LEAST, MAX_SPLIT)) return true;
    if (lay->off_part < SC_NOALLOC_WORKSPACE_BYTES) {
        int S = MAX_SPLIT - 1;
        if (lay->tall) {
            const double part = (double)(lay->total - lay->off_part) / lay->S;
            S = (int)fmin((SC_NOALLOC_WORKSPACE_BYTES - lay->off_part) / part, lay->S - 1);
        }
        while (S >= 1 && !consider(LAY_FULL, S)) --S;
    }
    if (lay->tall) consider(LAY_FULL, 0);
    if (!consider(LAY_TWO_PLANS, MAX_SPLIT)) consider(LAY_TWO_PLANS, 0);
    // (k_fgemm once more, beside what a smaller layout costs 64-row blocks of longer streams: estimated times
    // of both calls; 64-row blocks are overestimated, 1.2 to 1.7 times, k_fgemm by 0.75 to 1.2.  18 x 637 x 100 x
    // 4669 at L = 12 with a mean of 4: 175 us in the parts that fit and 103; 61 x 103 x 63 x 4915, L = 24: 116 and 140)
    if (few_short && taken.total <= SC_NOALLOC_WORKSPACE_BYTES &&
        0.68 * octets + 14.4 * rounds + 0.15 * operands + 22 < 0.62 * (least_t + 17 + 0.39 * chunks + 0.67 * operands))
        best = taken;
    *lay = best;
    return true;
}

// Products of a C-BSG call from which the tables are tried: there the launches that may return at
// once (two, about 5 us, beside the chunks' 7) are small against the planes' path (over 200 us).  And
// with more than an octet of cycles: a group of 32 slots costs four of them, and 55 calls of 4, 7 and 8
// cycles took up to 2.2 times as long from tables (13132 x 5516 x 768 four times at L = 4: 926 and 2034 us;
// at L = 12 23 calls took 0.65 to 1.18 times as long)
static constexpr double CBSG_TABLES = 4e11;
bool make_cbsg_layout(const sc_gemm_desc &d, int cus, const Layout &planes, Layout *lay) {
    if (d.rng != SC_RNG_SOBOL8_CBSG || d.batch < 1 || d.K < 1 || d.L_max <= MSTEP || (d.L_hint > 0 && d.L_hint < d.L_max) ||
        (double)d.batch * d.M * d.N * d.K * d.L_max < CBSG_TABLES)
        return false;
    if (round_up(d.K, 32) * round_up(d.L_max, 32) >= MFMA_EXACT || !layout_with(d, cus, LAY_FULL, true, lay) || !lay->rgen)
        return false;
    // The tables lie where the planes will if the tables do not serve: their rows and chunks of a batch entry
    // in that entry's planes (16 bytes and more an element quad and octet of cycles, against 4 and 8 a row), their
    // partial sums behind the last entry's, or in the planes path's; the rest, 100 KB at most, behind it all.
    // (Beside each other they added up to 8 GiB to calls that nearly fill the card.)
    Layout &t = *lay;
    const size_t small = t.off_perm, parts = t.total - t.off_part, rows = t.off_perm;
    const size_t roomA = planes.stride_batchA - (planes.off_Ap - planes.off_perm), roomB = planes.stride_batchB;
    if (t.vsplit || t.total > MOST_EXTRA || t.stride_batchA > roomA || t.stride_batchB > roomB) return false;
    for (size_t *o : {&t.off_perm, &t.off_Ls, &t.off_tileL, &t.off_tileOff, &t.off_pair, &t.off_Ap})
        *o += planes.off_Ap - rows;
    t.off_Bp = planes.off_Bp;
    if (parts <= roomB - t.stride_batchB)
        t.off_part = planes.off_Bp + (size_t)(planes.nbB - 1) * planes.stride_batchB + t.stride_batchB;
    else if (parts <= roomA - t.stride_batchA)
        t.off_part = planes.off_Ap + (size_t)(d.batch - 1) * planes.stride_batchA + t.stride_batchA;
    else
        t.off_part = planes.off_part;
    t.stride_batchA = planes.stride_batchA;
    t.stride_batchB = planes.stride_batchB;
    if (parts + small > SIZE_MAX - planes.total) return false;
    const size_t base = t.off_part + parts > planes.total ? t.off_part + parts : planes.total;
    for (size_t *o : {&t.off_rA, &t.off_rB, &t.off_status, &t.off_CA, &t.off_plan, &t.off_pslots, &t.off_rtab}) *o += base;
    t.off_units = t.off_tinfo = t.off_slot = base;      // (no range division)
    t.total = base + small;
    // a call whose planes fit sc_gemm_noalloc's array keeps fitting it
    return planes.total > SC_NOALLOC_WORKSPACE_BYTES || lay->total <= SC_NOALLOC_WORKSPACE_BYTES;
}

static int check_desc(const sc_gemm_desc *d) {
    if (d == nullptr) return SC_ERR_NULL;
    if (d->batch < 0 || d->M < 0 || d->N < 0 || d->K < 0 || d->K > SC_K_LIMIT) return SC_ERR_SHAPE;
    if (d->L_max < 1 || d->L_max > SC_L_MAX_LIMIT) return SC_ERR_LEN;
    // the counts stay exact: at most MAX_SPLIT parts of at most 2^24 products each
    if ((int64_t)d->K * d->L_max > SC_KL_LIMIT) return SC_ERR_SHAPE;
    if (d->polarity != SC_BIPOLAR_XNOR && d->polarity != SC_UNIPOLAR_AND_SM) return SC_ERR_POLARITY;
    if (d->rng != SC_RNG_LFSR32 && d->rng != SC_RNG_SOBOL8_CBSG) return SC_ERR_RNG;
    if (d->rng == SC_RNG_SOBOL8_CBSG && d->L_max > CBSG_L_MAX) return SC_ERR_LEN;
    if (d->L_hint < 0 || d->L_hint > d->L_max) return SC_ERR_LEN;
    if (d->reserved != 0) return SC_ERR_RESERVED;
    if (d->lda < d->K || d->ldb < d->K || d->ldo < d->N) return SC_ERR_STRIDE;
    if (d->strideA < 0 || d->strideB < 0 || d->strideO < 0 || d->strideSA < 0 || d->strideSB < 0 ||
        d->strideL < 0)
        return SC_ERR_STRIDE;
    // distinct batch entries must not overlap in the output: either each entry's block
    // lies before the next one (blocked), or the entries sit side by side in the columns
    // of one row stride (interleaved, e.g. per-head outputs of one token matrix)
    if (d->batch > 1 && d->M > 0 && d->N > 0) {
        const bool blocked = d->strideO >= (int64_t)(d->M - 1) * d->ldo + d->N;
        const bool interleaved = d->strideO >= d->N && (int64_t)(d->batch - 1) * d->strideO + d->N <= d->ldo;
        if (!blocked && !interleaved) return SC_ERR_STRIDE;
    }
    return SC_OK;
}

// Checks of one call (before anything is enqueued) and its workspace layout.
static int check_call(const sc_gemm_desc *desc, const int8_t *A, const float *sA, const int8_t *B,
                      const float *sB, const int32_t *L_per_row, const float *out, Layout *lay, Layout *tables) {
    const int rc = check_desc(desc);
    if (rc != SC_OK) return rc;
    const sc_gemm_desc &d = *desc;
    // a descriptor whose workspace cannot be laid out is refused as sc_gemm_workspace_size refuses it
    const int cus = device_cus();
    if (!make_layout(d, cus, lay)) return SC_ERR_SHAPE;
    if (make_cbsg_layout(d, cus, *lay, tables)) {
        lay->off_skip = tables->off_status + 3 * 4;
        lay->total = tables->total;
    } else {
        tables->rgen = 0;
    }
    // a pointer may be NULL only when the array it points to has no elements
    const bool anyM = d.batch > 0 && d.M > 0, anyN = d.batch > 0 && d.N > 0;
    if ((anyM && d.K > 0 && A == nullptr) || (anyN && d.K > 0 && B == nullptr) ||
        (anyM && (sA == nullptr || L_per_row == nullptr)) || (anyN && sB == nullptr) ||
        (anyM && anyN && out == nullptr))
        return SC_ERR_NULL;
    return SC_OK;
}

// The launch sequence of one call on workspace ws (lay.total bytes, 256-byte aligned); tables: of
// a C-BSG call whose rows may all have one length (rgen), or none
static int enqueue(const sc_gemm_desc &d, const Layout &lay, const Layout &tables, const int8_t *A, const float *sA,
                   const int8_t *B, const float *sB, const int32_t *L_per_row, float *out, int32_t *counts, uint8_t *ws,
                   hipStream_t st) {
    uint32_t *rA = reinterpret_cast<uint32_t *>(ws + lay.off_rA);
    // one batch entry with LFSR sequences: the scheduler's single block also clears the
    // status and makes the sequences (one launch fewer); otherwise k_draws does, first.  The
    // int8-chunk GEMM's scheduler and k_rprep write all that k_draws would
    const bool empty = d.batch == 0 || d.M == 0 || d.N == 0;
    const bool fuse = !empty && (lay.rgen || (d.batch == 1 && d.rng == SC_RNG_LFSR32));
    const bool try_tables = tables.rgen != 0 && !empty;
    hipError_t e = hipSuccess;
    // (the tables' first two launches also write what the planes path's first two would)
    if (try_tables && (launch_schedule(d, tables, L_per_row, ws, false, &lay, st) != hipSuccess ||
                       launch_rprep(d, tables, A, B, ws, st) != hipSuccess))
        return SC_ERR_HIP;
    if (!fuse && !try_tables) {
        // (the layout of an empty int8-chunk GEMM has no room for sequences: the status only)
        e = launch_draws(d.seed, d.rng, lay.rgen ? 0 : lay.LBS, rA, reinterpret_cast<uint32_t *>(ws + lay.off_rB), nullptr, -1,
                         reinterpret_cast<uint32_t *>(ws + lay.off_status), st);
        if (e != hipSuccess) return SC_ERR_HIP;
    }
    if (empty) return SC_OK;

    if (!try_tables && (e = launch_schedule(d, lay, L_per_row, ws, fuse, nullptr, st)) != hipSuccess) return SC_ERR_HIP;
    if (lay.rgen) {
        if ((e = launch_rprep(d, lay, A, B, ws, st)) != hipSuccess) return SC_ERR_HIP;
    } else if (!lay.fused) {
        if ((e = launch_mplanes(d, lay, A, B, ws, st)) != hipSuccess) return SC_ERR_HIP;
    }
    // the profiling events ride on the GEMM kernels' own dispatches (a marker of their own
    // in the stream left an idle gap of several microseconds after it); recorded as markers
    // only if no GEMM kernel was launched
    hipEvent_t ev0 = reinterpret_cast<hipEvent_t>(d.prof_event_begin);
    hipEvent_t ev1 = reinterpret_cast<hipEvent_t>(d.prof_event_end);
    set_gemm_events(ev0, ev1);
    e = lay.fused ? launch_fgemm(d, lay, A, B, sA, sB, out, counts, ws, st)
                  : launch_mgemm(d, lay, sA, sB, out, counts, ws, st);
    if (e == hipSuccess && try_tables) e = launch_mgemm(d, tables, sA, sB, out, counts, ws, st);
    const bool taken = gemm_events_taken();
    set_gemm_events(nullptr, nullptr);
    if (e != hipSuccess) return SC_ERR_HIP;
    if (!taken && ev0 != nullptr && hipEventRecord(ev0, st) != hipSuccess) return SC_ERR_HIP;
    if (!taken && ev1 != nullptr && hipEventRecord(ev1, st) != hipSuccess) return SC_ERR_HIP;
    return SC_OK;
}

// The workspace of sc_gemm_noalloc: a static device array, one copy per device, held until
// the process ends.  Host code never uses its name as an address: the device address of
// each device's copy is looked up once (hipGetSymbolAddress, with that device current) and
// kept per device.
static __device__ __align__(256) uint8_t scratch[SC_NOALLOC_WORKSPACE_BYTES];

static bool scratch_address(uint8_t **ptr) {
    constexpr int MAXDEV = 64;
    static std::mutex mu;
    static uint8_t *addr[MAXDEV] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAXDEV) return false;
    std::lock_guard<std::mutex> lock(mu);
    if (addr[dev] == nullptr) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr ||
            (reinterpret_cast<uintptr_t>(p) & 255u) != 0)
            return false;
        addr[dev] = static_cast<uint8_t *>(p);
    }
    *ptr = addr[dev];
    return true;
}

}  // namespace scg

using namespace scg;

extern "C" {

int sc_version(void) { return 10200; }

const char *sc_strerror(int code) {
    switch (code) {
        case SC_OK: return "SC_OK";
        case SC_ERR_NULL: return "SC_ERR_NULL: a required pointer is NULL";
        case SC_ERR_SHAPE: return "SC_ERR_SHAPE: bad batch/M/N/K (or K*L_max above 2^27)";
        case SC_ERR_LEN:
            return "SC_ERR_LEN: L_max outside [1, SC_L_MAX_LIMIT] ([1, 256] for C-BSG) or L_hint "
                   "outside [0, L_max]";
        case SC_ERR_POLARITY: return "SC_ERR_POLARITY: unknown polarity";
        case SC_ERR_RNG: return "SC_ERR_RNG: unknown rng or operand index";
        case SC_ERR_WORKSPACE: return "SC_ERR_WORKSPACE: workspace missing or too small";
        case SC_ERR_HIP: return "SC_ERR_HIP: a HIP call or kernel launch failed";
        case SC_ERR_DEVICE_STATUS: return "SC_ERR_DEVICE_STATUS: some L_i outside [0, L_max]";
        case SC_ERR_STRIDE: return "SC_ERR_STRIDE: a stride is too small or negative";
        case SC_ERR_RESERVED: return "SC_ERR_RESERVED: the reserved descriptor field is not 0";
        default: return "unknown status code";
    }
}

int sc_gemm_workspace_size(const sc_gemm_desc *desc, size_t *bytes) {
    if (bytes == nullptr) return SC_ERR_NULL;
    const int rc = check_desc(desc);
    if (rc != SC_OK) return rc;
    Layout lay, tables;
    const int cus = device_cus();
    if (!make_layout(*desc, cus, &lay)) return SC_ERR_SHAPE;
    *bytes = make_cbsg_layout(*desc, cus, lay, &tables) ? tables.total : lay.total;
    return SC_OK;
}

int sc_gemm(const sc_gemm_desc *desc, const int8_t *A, const float *sA, const int8_t *B,
            const float *sB, const int32_t *L_per_row, float *out, int32_t *counts, void *workspace,
            size_t workspace_bytes, void *stream) {
    Layout lay, tables;
    const int rc = check_call(desc, A, sA, B, sB, L_per_row, out, &lay, &tables);
    if (rc != SC_OK) return rc;
    if (workspace == nullptr || workspace_bytes < lay.total ||
        (reinterpret_cast<uintptr_t>(workspace) & 255u) != 0)
        return SC_ERR_WORKSPACE;
    return enqueue(*desc, lay, tables, A, sA, B, sB, L_per_row, out, counts, reinterpret_cast<uint8_t *>(workspace),
                   reinterpret_cast<hipStream_t>(stream));
}

int sc_gemm_noalloc(const sc_gemm_desc *desc, const int8_t *A, const float *sA, const int8_t *B,
                    const float *sB, const int32_t *L_per_row, float *out, int32_t *counts,
                    int32_t *status_out, void *stream) {
    Layout lay, tables;
    const int rc = check_call(desc, A, sA, B, sB, L_per_row, out, &lay, &tables);
    if (rc != SC_OK) return rc;
    if (lay.total > SC_NOALLOC_WORKSPACE_BYTES) return SC_ERR_WORKSPACE;
    uint8_t *ws = nullptr;
    if (!scratch_address(&ws)) return SC_ERR_HIP;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const int e = enqueue(*desc, lay, tables, A, sA, B, sB, L_per_row, out, counts, ws, st);
    if (e != SC_OK) return e;
    // the status word (offset 0 of every workspace) of this call, for the caller
    if (status_out != nullptr &&
        hipMemcpyAsync(status_out, ws, sizeof(int32_t), hipMemcpyDeviceToDevice, st) != hipSuccess)
        return SC_ERR_HIP;
    return SC_OK;
}

int sc_gemm_status(const void *workspace, void *stream) {
    if (workspace == nullptr) return SC_ERR_NULL;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (hipStreamSynchronize(st) != hipSuccess) return SC_ERR_HIP;
    uint32_t word = 0;
    if (hipMemcpy(&word, workspace, sizeof(word), hipMemcpyDeviceToHost) != hipSuccess)
        return SC_ERR_HIP;
    return (word & STATUS_BAD_LENGTH) ? SC_ERR_DEVICE_STATUS : SC_OK;
}

int sc_quantize(int32_t batch, int32_t rows, int32_t K, const float *X, int64_t ldx,
                int64_t strideX, int32_t per_tensor, int8_t *Q, int64_t ldq, int64_t strideQ,
                float *scale, float *rowmax, int64_t strideS, void *stream) {
    if (batch < 0 || rows < 0 || K < 0 || K > SC_K_LIMIT) return SC_ERR_SHAPE;
    if (per_tensor != 0 && per_tensor != 1) return SC_ERR_SHAPE;
    if (ldx < K || ldq < K || strideX < 0 || strideQ < 0 || strideS < 0) return SC_ERR_STRIDE;
    if (batch > 1 && rows > 0 && strideS < rows) return SC_ERR_STRIDE;
    if (batch == 0 || rows == 0) return SC_OK;
    if ((K > 0 && (X == nullptr || Q == nullptr)) || scale == nullptr) return SC_ERR_NULL;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (launch_quantize(batch, rows, K, X, ldx, strideX, per_tensor, Q, ldq, strideQ, scale, rowmax,
                        strideS, st) != hipSuccess)
        return SC_ERR_HIP;
    return SC_OK;
}

int sc_mp_lengths(int32_t batch, int32_t M, const float *metric, int64_t strideM,
                  const float *tau, const int32_t *ladder, int32_t n_levels, int32_t *L_out,
                  int64_t strideL, void *stream) {
    if (batch < 0 || M < 0) return SC_ERR_SHAPE;
    if (n_levels < 1 || n_levels > SC_MP_MAX_LEVELS) return SC_ERR_LEN;
    if (ladder == nullptr || (n_levels > 1 && tau == nullptr)) return SC_ERR_NULL;
    MpParams p{};
    p.n = n_levels;
    for (int k = 0; k < n_levels; ++k) {
        if (ladder[k] < 0 || ladder[k] > SC_L_MAX_LIMIT || (k > 0 && ladder[k] >= ladder[k - 1]))
            return SC_ERR_LEN;
        p.ladder[k] = ladder[k];
    }
    for (int k = 0; k + 1 < n_levels; ++k) {
        if (!(tau[k] >= 0.0f && tau[k] <= 1.0f) || (k > 0 && tau[k] > tau[k - 1])) return SC_ERR_LEN;
        p.tau[k] = tau[k];
    }
    if (strideM < 0 || strideL < 0 || (batch > 1 && M > 0 && (strideM < M || strideL < M)))
        return SC_ERR_STRIDE;
    if (batch == 0 || M == 0) return SC_OK;
    if (metric == nullptr || L_out == nullptr) return SC_ERR_NULL;
    if (launch_mp_lengths(batch, M, metric, strideM, p, L_out, strideL,
                          reinterpret_cast<hipStream_t>(stream)) != hipSuccess)
        return SC_ERR_HIP;
    return SC_OK;
}

int sc_comparator_sequence(uint64_t seed, int32_t op, int32_t rng, int32_t n, uint8_t *out,
                           void *stream) {
    if (out == nullptr) return SC_ERR_NULL;
    if ((op != 0 && op != 1) || (rng != SC_RNG_LFSR32 && rng != SC_RNG_SOBOL8_CBSG))
        return SC_ERR_RNG;
    if (n < 1 || n > (rng == SC_RNG_SOBOL8_CBSG ? CBSG_L_MAX : SC_L_MAX_LIMIT)) return SC_ERR_LEN;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (launch_draws(seed, rng, n, nullptr, nullptr, out, op, nullptr, st) != hipSuccess)
        return SC_ERR_HIP;
    return SC_OK;
}

}  // extern "C"
