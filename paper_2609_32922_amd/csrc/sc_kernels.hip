// HIP kernels of libscgemm for gfx950 (MI355X) that precede the counting GEMM of an SC
// GEMM call (the GEMM itself is in sc_mfma.hip).  All run on the caller's stream:
//   k_draws      comparator sequences r^A, r^B (Sec. 3.1 "Bitstream generation",
//                LFSR or scrambled Sobol-8 of Sec. A.1) -- one lane per cycle, the LFSR
//                through jump-ahead; it also clears the status words.  With one batch
//                entry and LFSR sequences k_schedule does both instead (one launch fewer),
//                and the int8-chunk GEMM needs neither
//   k_schedule   per-row length scheduler: validates L_i, counting-sorts rows by L
//                (descending) so that a 128-row tile runs for the longest length it
//                holds (Sec. 4.2: row i stops after its own l_i cycles; Sec. 4.1: the
//                cost grows with the sum of the l_i); with C-BSG planes one more block makes
//                CA[L][beta] = ones of A's stream in its first L cycles
//   k_schedule_plans  the same for the int8-chunk GEMM, with its slot plans beside it
#include "sc_internal.h"

namespace scg {

// ----------------------------------------------------------------------------
// comparator sequence
// ----------------------------------------------------------------------------
constexpr uint32_t kFeedback = 0x80200003u;   // x^32+x^22+x^2+x+1, Galois right-shift taps
constexpr uint32_t kPolyLow = 0x00400007u;    // the same polynomial minus x^32

constexpr uint32_t lfsr_step_ce(uint32_t s) { return (s >> 1) ^ ((s & 1u) ? kFeedback : 0u); }

// kJump.v[l] is the register state after 8*l steps from state 1.  A right-shift step
// multiplies the state polynomial by x^{-1} modulo p(x), so the state after 8*l steps
// from S_0 is S_0 * kJump.v[l] mod p(x): every cycle's draw is computed independently.
struct JumpTable {
    uint32_t v[SC_L_MAX_LIMIT];
};
constexpr JumpTable make_jump_table() {
    JumpTable t{};
    uint32_t s = 1u;
    for (int l = 0; l < SC_L_MAX_LIMIT; ++l) {
        t.v[l] = s;
        for (int k = 0; k < 8; ++k) s = lfsr_step_ce(s);
    }
    return t;
}
__constant__ JumpTable kJump = make_jump_table();

__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
    uint64_t z = x + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Product of two polynomials of degree < 32 modulo p(x), Horner from the top bit.
__device__ __forceinline__ uint32_t gf2_mulmod(uint32_t a, uint32_t b) {
    uint32_t acc = 0;
#pragma unroll
    for (int k = 31; k >= 0; --k) {
        acc = (acc << 1) ^ ((acc >> 31) ? kPolyLow : 0u);
        acc ^= ((a >> k) & 1u) ? b : 0u;
    }
    return acc;
}

// 8-bit Sobol direction numbers V_j = m_j 2^(8-j), j = 1..8: dimension 1 has m_j = 1;
// dimension 2 comes from the primitive polynomial x + 1, whose recurrence is
// m_j = m_{j-1} xor 2 m_{j-1} from m_1 = 1.
struct SobolDirs {
    uint32_t v[2][8];
};
constexpr SobolDirs make_sobol_dirs() {
    SobolDirs t{};
    uint32_t m = 1u;
    for (int j = 1; j <= 8; ++j) {
        t.v[0][j - 1] = 1u << (8 - j);
        if (j > 1) m = m ^ (m << 1);
        t.v[1][j - 1] = m << (8 - j);
    }
    return t;
}
__constant__ SobolDirs kSobol = make_sobol_dirs();

// Draw l of operand op (0: A, 1: B) of the comparator sequence.
__device__ __forceinline__ uint32_t draw_value(uint64_t seed, int rng, int op, int l) {
    const uint64_t h = splitmix64(2ull * seed + (uint64_t)op);
    uint32_t v = 0;
    if (rng == SC_RNG_SOBOL8_CBSG) {
        // point l (< 256) of dimension op + 1, digitally shifted by the top 8 bits of h
        v = (uint32_t)(h >> 56);
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if ((l >> j) & 1) v ^= kSobol.v[op][j];
    } else {
        uint32_t s0 = (uint32_t)(h >> 32);
        if (s0 == 0u) s0 = 1u;
        uint32_t s = gf2_mulmod(s0, kJump.v[l]);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            v = (v << 1) | (s & 1u);
            s = (s >> 1) ^ ((s & 1u) ? kFeedback : 0u);
        }
    }
    return v;
}

__global__ __launch_bounds__(256) void k_draws(uint64_t seed, int rng, int n, uint32_t *rA,
                                               uint32_t *rB, uint8_t *bytes_out, int op_only,
                                               uint32_t *status) {
    const int l = blockIdx.x * blockDim.x + threadIdx.x;
    const int op = op_only >= 0 ? op_only : (int)blockIdx.y;
    if (status != nullptr && l == 0 && blockIdx.y == 0) {
        status[0] = 0u;
        status[1] = 0u;   // longest tile pair of the call
        status[2] = 0u;   // (int8-chunk GEMM only; k_rprep writes it)
    }
    if (l >= n) return;
    const uint32_t v = draw_value(seed, rng, op, l);
    if (bytes_out != nullptr)
        bytes_out[l] = (uint8_t)v;
    else
        (op == 0 ? rA : rB)[l] = v;
}

hipError_t launch_draws(uint64_t seed, int rng, int n, uint32_t *rA, uint32_t *rB,
                        uint8_t *bytes_out, int op_only, uint32_t *status, hipStream_t st) {
    dim3 grid((unsigned)((n > 0 ? n : 1) + 255) / 256, op_only >= 0 ? 1u : 2u);
    hipLaunchKernelGGL(k_draws, grid, dim3(256), 0, st, seed, rng, n, rA, rB, bytes_out, op_only,
                       status);
    return hipGetLastError();
}

// CA[L][beta] = #{l < L : rA_l < beta} for L = 0..L_max, beta = 0..256 (one thread per
// boundary; L_max <= 256 draws staged in LDS)
__device__ __forceinline__ void cbsg_table_block(const uint32_t *rA, int L_max, uint16_t *__restrict__ CA,
                                                 uint32_t *r) {
    const int beta = threadIdx.x;
    for (int l = threadIdx.x; l < L_max; l += blockDim.x) r[l] = rA[l];
    __syncthreads();
    if (beta >= CA_COLS) return;
    uint32_t c = 0;
    for (int l = 0; l < L_max; ++l) {
        CA[(size_t)l * CA_COLS + beta] = (uint16_t)c;
        c += r[l] < (uint32_t)beta ? 1u : 0u;
    }
    CA[(size_t)L_max * CA_COLS + beta] = (uint16_t)c;
}

// ----------------------------------------------------------------------------
// per-row length scheduler (one 1024-thread block per batch entry)
// ----------------------------------------------------------------------------
// Adds 1 to hist[l] for every active lane and returns the lane's old value (its place
// in bucket l).  The lanes that share the first active lane's l take one LDS atomic
// together, the others one each: equal lengths (the common case) cost one atomic per
// wave instead of one per row, and mixed lengths cost what single atomics cost.
__device__ int wave_bucket_add(int *hist, int l, bool active) {
    const int lane = threadIdx.x & 63;
    const uint64_t act = __ballot(active);
    if (act == 0) return 0;
    const int leader = __ffsll((unsigned long long)act) - 1;
    const int lv = __builtin_amdgcn_readlane(l, leader);
    const bool mine = active && l == lv;
    const uint64_t grp = __ballot(mine);
    int base = 0;
    if (lane == leader) base = atomicAdd(&hist[lv], __popcll(grp));
    base = __builtin_amdgcn_readlane(base, leader);
    if (mine) return base + __popcll(grp & ((1ull << lane) - 1));
    return active ? atomicAdd(&hist[l], 1) : 0;
}

struct SchedLds {
    int hist[SC_L_MAX_LIMIT + 1], hstart[SC_L_MAX_LIMIT + 1], dpair[2048 + 1];
    int lmin, lmax;
    uint32_t bad, used[2];
};
// RGEN: of the int8-chunk GEMM.  There the block leaves what it found in its batch entry's record
// (bad length, longest row, plans taken) instead of adding to the status words, which k_rprep
// writes from all records: no launch has to clear them first.
template <bool RGEN>
__device__ __forceinline__ void schedule_block(const int32_t *__restrict__ L, int64_t strideL, int M, int L_max,
                                               const Layout &lay, uint8_t *ws, uint64_t seed, int rng, int ndraws,
                                               SchedLds &sh, const PlanesOut &po) {
    int *hist = sh.hist, *hstart = sh.hstart, *dpair = sh.dpair;
    int &lmin = sh.lmin, &lmax = sh.lmax;
    const int b = blockIdx.x, tid = threadIdx.x;
    uint8_t *wsb = ws + (size_t)b * lay.stride_batchA;
    int32_t *perm = ws_ptr<int32_t>(wsb, lay.off_perm);
    int32_t *Ls = ws_ptr<int32_t>(wsb, lay.off_Ls);
    int32_t *tileL = ws_ptr<int32_t>(wsb, lay.off_tileL);
    int64_t *tileOff = ws_ptr<int64_t>(wsb, lay.off_tileOff);
    uint32_t *status = RGEN ? &sh.bad : ws_ptr<uint32_t>(ws, lay.off_status);
    const int32_t *Lb = L + (size_t)b * strideL;

    // Up to SREG * 1024 rows the lengths are loaded once, all loads in flight together (issued
    // first, so that their latency overlaps the sequences and the clearing below), and kept in
    // registers for the scatter; longer batch entries loop (and load them twice).
    constexpr int SREG = 20;
    const bool cached = M <= SREG * 1024;
    int lv[SREG];
    if (cached) {
#pragma unroll
        for (int k = 0; k < SREG; ++k) {
            const int i = k * 1024 + tid;
            lv[k] = i < M ? Lb[i] : 0;
        }
    }
    if (!RGEN && ndraws > 0) {
        // one batch entry: this block also clears the status words and makes the comparator
        // sequences (the work of k_draws), before any of its own status updates
        if (tid == 0) {
            status[0] = 0u;
            status[1] = 0u;
            status[2] = 0u;
        }
        uint32_t *rA = ws_ptr<uint32_t>(ws, lay.off_rA), *rB = ws_ptr<uint32_t>(ws, lay.off_rB);
        for (int l = tid; l < ndraws; l += 1024) {
            rA[l] = draw_value(seed, rng, 0, l);
            rB[l] = draw_value(seed, rng, 1, l);
        }
    }
    for (int v = tid; v <= L_max; v += 1024) hist[v] = 0;
    if (tid == 0) {
        lmin = INT_MAX;
        lmax = INT_MIN;
        sh.bad = sh.used[0] = sh.used[1] = 0u;
    }
    __syncthreads();
    // the lengths held in registers: validated, and their range over the batch entry
    if (cached) {
        int lo = INT_MAX, hi = INT_MIN;
#pragma unroll
        for (int k = 0; k < SREG; ++k) {
            if (lv[k] < 0 || lv[k] > L_max) {
                atomicOr(status, STATUS_BAD_LENGTH);
                lv[k] = 0;
            }
            if (k * 1024 + tid < M) {
                lo = min(lo, lv[k]);
                hi = max(hi, lv[k]);
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            lo = min(lo, __shfl_xor(lo, o, 64));
            hi = max(hi, __shfl_xor(hi, o, 64));
        }
        if ((tid & 63) == 0) {
            atomicMin(&lmin, lo);
            atomicMax(&lmax, hi);
        }
        __syncthreads();
    }
    // One length for every row (M > 0): the sort keeps the row order, and the counts below
    // are set directly.
    const bool one = cached && M > 0 && lmin == lmax;
    if (one) {
        const int l = lmin;
        // as after the scatter of the general path: hist[v] = end and hstart[v] = start of
        // length v's run of sorted positions (lengths above l: empty runs at 0, below: at M)
        for (int v = tid; v <= L_max; v += 1024) {
            hist[v] = v <= l ? M : 0;
            hstart[v] = v < l ? M : 0;
        }
#pragma unroll
        for (int k = 0; k < SREG; ++k) {
            const int i = k * 1024 + tid;
            if (i < M) {
                perm[i] = i;
                Ls[i] = l;
            }
        }
    } else if (cached) {
#pragma unroll
        for (int k = 0; k < SREG; ++k)
            if (k * 1024 < M) wave_bucket_add(hist, lv[k], k * 1024 + tid < M);
    } else {
        for (int i0 = 0; i0 < M; i0 += 1024) {
            const int i = i0 + tid;
            int l = i < M ? Lb[i] : 0;
            if (l < 0 || l > L_max) {
                atomicOr(status, STATUS_BAD_LENGTH);
                l = 0;
            }
            wave_bucket_add(hist, l, i < M);
        }
    }
    __syncthreads();
    // start position of each length bucket, longest lengths first (also kept in hstart: the
    // scatter below moves hist[l] on to the end of l's run)
    int rcarry = 0;
    for (int c = 0; !one && c <= L_max; c += 1024) {
        const int idx = L_max - (c + tid);
        const int v = idx >= 0 ? hist[idx] : 0;
        int tot;
        const int ex = block_excl_scan<1024>(v, &tot);
        if (idx >= 0) {
            hist[idx] = rcarry + ex;
            hstart[idx] = rcarry + ex;
        }
        rcarry += tot;
        __syncthreads();
    }
    if (one) {
        // (done above)
    } else if (cached) {
#pragma unroll
        for (int k = 0; k < SREG; ++k) {
            const int i = k * 1024 + tid;
            if (k * 1024 >= M) break;
            const int pos = wave_bucket_add(hist, lv[k], i < M);
            if (i < M) {
                perm[pos] = i;
                Ls[pos] = lv[k];
            }
        }
    } else {
        for (int i0 = 0; i0 < M; i0 += 1024) {
            const int i = i0 + tid;
            int l = i < M ? Lb[i] : 0;
            if (l < 0 || l > L_max) l = 0;
            const int pos = wave_bucket_add(hist, l, i < M);
            if (i < M) {
                perm[pos] = i;
                Ls[pos] = l;
            }
        }
    }
    for (int p = M + tid; p < lay.MT * BM; p += 1024) {
        perm[p] = -1;
        Ls[p] = 0;
    }
    __syncthreads();
    // After the scatter hist[l] is the end of length l's run of sorted positions (runs in
    // order of decreasing length, ends non-increasing in l): the length at sorted position
    // p < M is the largest l whose run ends after p.
    auto length_at = [&](int p) {
        if (p >= M) return 0;
        int lo = 0, hi = L_max;   // hist[lo] > p holds (hist[0] = M)
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (hist[mid] > p) lo = mid;
            else hi = mid - 1;
        }
        return lo;
    };
    if (RGEN) {
        // Int8-chunk GEMM: each pair's longest and shortest length, which choose its slot plan,
        // and how many distinct lengths it meets (the GEMM keeps a table of A masked to each
        // row length that ends inside a group, rslots of them).  Rows are sorted, so a length is a
        // run [hstart[l], end) and adds one to every pair that the run meets (a difference array
        // over pairs, then a scan; lengths that are not multiples of 32 in the upper half);
        // end = hstart[l - 1] (runs in order of decreasing length).  Up to 2048 pairs per pass.
        int4 *pair = ws_ptr<int4>(wsb, lay.off_pair);
        const int npairs = lay.rtiles, sh8 = lay.tshift;      // (row tiles: 256 rows, or 64 with tall)
        for (int q0 = 0; q0 < npairs; q0 += 2048) {
            const int nq = min(npairs - q0, 2048);
            if (!one) {
                __syncthreads();
                for (int q = tid; q <= nq; q += 1024) dpair[q] = 0;
                __syncthreads();
                for (int l = 1 + tid; l <= L_max; l += 1024) {
                    const int start = hstart[l], end = hstart[l - 1];
                    if (end <= start) continue;
                    const int qa = max(start >> sh8, q0), qb = min((end - 1) >> sh8, q0 + nq - 1);
                    if (qa > qb) continue;
                    const int add = l % 32 != 0 ? 0x10001 : 1;
                    atomicAdd(&dpair[qa - q0], add);
                    atomicAdd(&dpair[qb + 1 - q0], -add);
                }
                __syncthreads();
            }
            int pc = 0;
            for (int c = 0; c < nq; c += 1024) {
                const int q = c + tid;
                int nd = lmin > 0 ? (lmin % 32 != 0 ? 0x10001 : 1) : 0;
                if (!one) {
                    int tot;
                    const int v = q < nq ? dpair[q] : 0;
                    nd = pc + block_excl_scan<1024>(v, &tot) + v;
                    pc += tot;
                }
                if (q >= nq) continue;
                const int p = (q0 + q) << sh8;
                const int hi = one ? lmin : length_at(p), lo = one ? lmin : length_at(min(p + (1 << sh8) - 1, M - 1));
                pair[q0 + q] = make_int4(hi, lo, nd & 0xFFFF, nd >> 16);
                const int k = plan_of(lo, lay.nplans, lay.pstep, L_max);
                atomicOr(&sh.used[k >> 5], 1u << (k & 31));
            }
        }
        __syncthreads();
        if (tid == 0)
            pair[npairs] = make_int4((int)sh.bad, (int)round_up(one ? lmin : length_at(0), MSTEP),
                                     lay.cbsg ? (one ? lmin : length_at(M - 1)) : (int)sh.used[0], (int)sh.used[1]);
        if (lay.cbsg) {
            // the planes path's rows (as above, in its own place) and tiles (as below)
            uint8_t *wsp = ws + (size_t)b * po.stride_batchA;
            for (int p = tid; p < po.MT * BM; p += 1024) {
                const bool in = p < lay.MT * BM;
                ws_ptr<int32_t>(wsp, po.off_perm)[p] = in ? perm[p] : -1;
                ws_ptr<int32_t>(wsp, po.off_Ls)[p] = in ? Ls[p] : 0;
            }
            int64_t carry = 0;
            for (int c = 0; c < po.MT; c += 1024) {
                const int t = c + tid, p = (po.mbm == 2 * BM ? (t & ~1) : t) * BM;
                const int tl = t >= po.MT || p >= M ? 0 : (int)round_up(one ? lmin : length_at(p), MSTEP);
                int64_t tot;
                const int64_t ex = block_excl_scan<1024>((int64_t)tl * po.words_per_L, &tot);
                if (t < po.MT) {
                    ws_ptr<int32_t>(wsp, po.off_tileL)[t] = tl;
                    ws_ptr<int64_t>(wsp, po.off_tileOff)[t] = carry + ex;
                }
                carry += tot;
            }
        }
    } else {
        // tile lengths (first sorted row of a tile holds its longest length; a pair of tiles
        // that one 256-row block takes runs at the pair's longest length) and the tiles' plane
        // offsets
        int64_t carry = 0;
        for (int c = 0; c < lay.MT; c += 1024) {
            const int t = c + tid;
            int tl = 0;
            if (t < lay.MT) {
                const int t0 = lay.mbm == 2 * BM ? (t & ~1) : t;
                tl = (int)round_up(length_at(t0 * BM), MSTEP);
                tileL[t] = tl;
            }
            int64_t tot;
            const int64_t ex = block_excl_scan<1024>((int64_t)tl * lay.words_per_L, &tot);
            if (t < lay.MT) tileOff[t] = carry + ex;
            carry += tot;
        }
    }
    // the first tile pair holds the batch entry's longest rows
    if (!RGEN && tid == 0 && lay.mbm == 2 * BM) atomicMax(status + 1, (uint32_t)round_up(length_at(0), MSTEP));
}

// ----------------------------------------------------------------------------
// slot plans of the int8-chunk GEMM (one 1024-thread block per plan)
// ----------------------------------------------------------------------------
// The cycles l < p of plan k are edges between the class of A's draw and the class of B's; the
// block covers them with few classes by leaf removal: while some class holds one live cycle,
// the class at that cycle's other end takes all of its own live cycles (all such classes at
// once; optimal as long as such classes are found, which is nearly always up to L = 256 bipolar
// or 192 unipolar: 2 to 5 rounds); when there is none, or after PLAN_ROUNDS rounds, A's classes
// take what is left (more rounds, or the fullest classes first, saved at most one slot of 212
// and none past L = 512).  A class with more than SLOT_CYCLES cycles takes several slots.  The
// order in which cycles take places in a class's slots does not matter: every sum is an exact
// integer.  (Latency: 16 waves around two barriers per round.)
struct PlanLds {
    int deg[512];                       // live cycles of each class: A's, then B's
    int mark[512];                      // the round in which the class was taken
    int cnt[512], base[512];            // cycles, and first slot, of each class
    uint32_t own[SC_L_MAX_LIMIT];       // slot: class | side << 8 | cycles << 9 | second class << 16
    uint32_t part[SC_L_MAX_LIMIT];      // slot: its cycles' classes on the other side, a byte each
    int wg[SC_L_MAX_LIMIT / 32];        // cycles of each group
    int leaf[8], left[8];               // per round: a class of one live cycle exists; cycles are left
    int wmax;
};
constexpr int PLAN_ROUNDS = 6;

__device__ __forceinline__ void plan_block(int k, const Layout &lay, int L_max, uint8_t *ws, uint64_t seed, bool bip,
                                           PlanLds &sh) {
    constexpr int EPT = SC_L_MAX_LIMIT / 1024;    // cycles per thread
    const int tid = threadIdx.x;
    const int p = lay.cbsg ? L_max : plan_prefix(k, lay.nplans, lay.pstep, L_max);
    const int rng = lay.cbsg ? SC_RNG_SOBOL8_CBSG : SC_RNG_LFSR32;
    uint2 *slots = ws_ptr<uint2>(ws, lay.off_pslots) + (size_t)k * lay.LBS;
    int ca[EPT], cb[EPT], rank[EPT];
    uint32_t live = 0u, onB = 0u;
    if (tid < 512) {
        sh.deg[tid] = 0;
        sh.mark[tid] = 0;
        sh.cnt[tid] = 0;
    }
    if (tid < SC_L_MAX_LIMIT / 32) sh.wg[tid] = 0;
    if (tid < 8) sh.leaf[tid] = sh.left[tid] = 0;
    for (int i = tid; i < p; i += 1024) sh.part[i] = 0xFFFFFFFFu;
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
        const int l = i * 1024 + tid;
        ca[i] = cb[i] = rank[i] = 0;
        if (l >= L_max) continue;
        const int ra = (int)draw_value(seed, rng, 0, l), rb = (int)draw_value(seed, rng, 1, l);
        ca[i] = bip ? class_bipolar(ra) : class_unipolar(ra);
        cb[i] = 256 + (bip ? class_bipolar(rb) : class_unipolar(rb));
        if (l < p) live |= 1u << i;
    }
    __syncthreads();
    if (lay.cbsg) {
        // A's classes in increasing order (L_max <= 256 draws, one per thread), B's beside them
        if (tid < L_max) sh.part[tid] = (uint32_t)ca[0];
        __syncthreads();
        if (tid < L_max) {
            int at = 0;
            for (int l = 0; l < L_max; ++l) at += (int)sh.part[l] < ca[0] || ((int)sh.part[l] == ca[0] && l < tid) ? 1 : 0;
            sh.own[at] = (uint32_t)ca[0];
            sh.own[CBSG_L_MAX + tid] = (uint32_t)(cb[0] - 256);
        }
        __syncthreads();
        if (bip) {
            // slot j: counters j and L - 1 - j, A = [n >= u] + [n >= v] - 1 there
            const int S = (L_max + 1) / 2, j = tid, e = L_max - 1 - tid;
            if (j < S)
                slots[j] = make_uint2(sh.own[e] | (j == e ? 1u : 2u) << 9 | sh.own[j] << 16,
                                      sh.own[CBSG_L_MAX + j] | (j == e ? 255u : sh.own[CBSG_L_MAX + e]) << 8 | 0xFFFF0000u);
            if (tid < 32 && S + tid < (int)round_up(S, 32)) slots[S + tid] = make_uint2(0u, 0xFFFFFFFFu);
            if (tid == 0) ws_ptr<int4>(ws, lay.off_plan)[k] = make_int4(L_max, S, S, 0);
            return;
        }
        if (tid < L_max) {
            ca[0] = (int)sh.own[tid];
            sh.part[tid] = 0xFFFFFFFFu;
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < EPT; ++i)
        if ((live >> i) & 1u) {
            atomicAdd(&sh.deg[ca[i]], 1);
            atomicAdd(&sh.deg[cb[i]], 1);
        }
    __syncthreads();
    static_assert(PLAN_ROUNDS <= 8, "a flag per round");
    for (int round = 0; round < PLAN_ROUNDS; ++round) {
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            if (!((live >> i) & 1u)) continue;
            const bool la = sh.deg[ca[i]] == 1, lb = sh.deg[cb[i]] == 1;
            if (la) sh.mark[cb[i]] = round + 1;
            else if (lb) sh.mark[ca[i]] = round + 1;
            if (la || lb) sh.leaf[round] = 1;
        }
        __syncthreads();
        const bool all = round == PLAN_ROUNDS - 1 || sh.leaf[round] == 0;
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            if (!((live >> i) & 1u)) continue;
            const bool b = !all && sh.mark[cb[i]] == round + 1;
            if (!all && !b && sh.mark[ca[i]] != round + 1) {
                sh.left[round] = 1;
                continue;
            }
            live &= ~(1u << i);
            if (b) onB |= 1u << i;
            atomicSub(&sh.deg[ca[i]], 1);
            atomicSub(&sh.deg[cb[i]], 1);
        }
        __syncthreads();
        if (sh.left[round] == 0) break;
    }
#pragma unroll
    for (int i = 0; i < EPT; ++i)
        if (i * 1024 + tid < p) rank[i] = atomicAdd(&sh.cnt[(onB >> i) & 1u ? cb[i] : ca[i]], 1);
    __syncthreads();
    int S;
    const int ex = block_excl_scan<1024>(tid < 512 ? (sh.cnt[tid] + SLOT_CYCLES - 1) / SLOT_CYCLES : 0, &S);
    if (tid < 512) sh.base[tid] = ex;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
        if (i * 1024 + tid >= p) continue;
        const bool b = (onB >> i) & 1u;
        const int v = b ? cb[i] : ca[i], o = b ? ca[i] : cb[i];
        const int slot = sh.base[v] + rank[i] / SLOT_CYCLES, j = rank[i] % SLOT_CYCLES;
        reinterpret_cast<uint8_t *>(&sh.part[slot])[j] = (uint8_t)(o & 255);
        if (j == 0) {
            const int n = min(SLOT_CYCLES, sh.cnt[v] - (rank[i] - j));
            sh.own[slot] = (uint32_t)(v & 255) * 0x10001u | (b ? 0x100u : 0u) | ((uint32_t)n << 9);
            if (lay.p16) atomicAdd(&sh.wg[slot / 32], n);
        }
    }
    __syncthreads();
    // int16 partial counts (Layout::p16): a part of n chunk steps holds counts of at most 32 n x
    // the heaviest group's cycles; where that could pass int16 the plan merges nothing
    if (lay.p16) {
        if (tid < 64) {
            int m = 32;      // (a group of cycles p.., one a slot; one shared with merged slots adds < 32)
#pragma unroll
            for (int i = 0; i < SC_L_MAX_LIMIT / 32 / 64; ++i) {
                const int G = i * 64 + tid, alone = S < p && G == S / 32 ? 32 - S % 32 : 0;
                m = max(m, sh.wg[G] + alone);
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, 64));
            if (tid == 0) sh.wmax = m;
        }
        __syncthreads();
        const int64_t smin = lay.Sleast;
        const int64_t steps = ((int64_t)lay.KC * ((S + L_max - p + 31) / 32) + smin - 1) / smin;
        if (steps * 32 * sh.wmax > 32767) S = p;
    }
    const bool merged = S < p;
    for (int i = tid; merged && i < S; i += 1024) slots[i] = make_uint2(sh.own[i], sh.part[i]);
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
        const int l = i * 1024 + tid;
        if (l < L_max && (l >= p || !merged))
            slots[S + l - p] = make_uint2((uint32_t)ca[i] * 0x10001u | (1u << 9), (uint32_t)(cb[i] - 256) | 0xFFFFFF00u);
    }
    const int T = S + L_max - p;
    if (tid < 32 && T + tid < (int)round_up(T, 32)) slots[T + tid] = make_uint2(0u, 0xFFFFFFFFu);
    if (tid == 0) ws_ptr<int4>(ws, lay.off_plan)[k] = make_int4(p, S, T, 0);
}

__global__ __launch_bounds__(1024) void k_schedule(const int32_t *__restrict__ L, int64_t strideL, int M, int L_max,
                                                   Layout lay, uint8_t *ws, uint64_t seed, int rng, int ndraws) {
    __shared__ SchedLds sh;
    if (rng == SC_RNG_SOBOL8_CBSG && blockIdx.x == gridDim.x - 1) {
        cbsg_table_block(ws_ptr<uint32_t>(ws, lay.off_rA), L_max, ws_ptr<uint16_t>(ws, lay.off_CA),
                         reinterpret_cast<uint32_t *>(sh.hist));
        return;
    }
    schedule_block<false>(L, strideL, M, L_max, lay, ws, seed, rng, ndraws, sh, PlanesOut{});
}

// Int8-chunk GEMM: blocks 0 .. batch-1 schedule a batch entry each, the rest make a slot plan each
union SchedPlanLds {
    SchedLds s;
    PlanLds p;
};
__global__ __launch_bounds__(1024) void k_schedule_plans(const int32_t *__restrict__ L, int64_t strideL, int batch,
                                                         int M, int L_max, Layout lay, uint8_t *ws, uint64_t seed,
                                                         int polarity, PlanesOut po) {
    __shared__ SchedPlanLds sh;
    if ((int)blockIdx.x < batch) {
        schedule_block<true>(L, strideL, M, L_max, lay, ws, seed, SC_RNG_LFSR32, 0, sh.s, po);
    } else if ((int)blockIdx.x - batch == lay.nplans) {
        // (C-BSG) the planes path's sequences and table CA
        uint32_t *rA = ws_ptr<uint32_t>(ws, po.off_rA), *rB = ws_ptr<uint32_t>(ws, po.off_rB);
        for (int l = threadIdx.x; l < po.LBS; l += 1024) {
            rA[l] = draw_value(seed, SC_RNG_SOBOL8_CBSG, 0, l);
            rB[l] = draw_value(seed, SC_RNG_SOBOL8_CBSG, 1, l);
        }
        __syncthreads();
        cbsg_table_block(rA, L_max, ws_ptr<uint16_t>(ws, po.off_CA), reinterpret_cast<uint32_t *>(sh.s.hist));
    } else plan_block((int)blockIdx.x - batch, lay, L_max, ws, seed, polarity == SC_BIPOLAR_XNOR, sh.p);
}

hipError_t launch_schedule(const sc_gemm_desc &d, const Layout &lay, const int32_t *L, uint8_t *ws,
                           bool draws, const Layout *planes, hipStream_t st) {
    if (lay.rgen) {
        PlanesOut po{};
        if (planes != nullptr) {
            po.MT = planes->MT;
            po.mbm = planes->mbm;
            po.LBS = planes->LBS;
            po.words_per_L = planes->words_per_L;
            po.off_perm = planes->off_perm;
            po.off_Ls = planes->off_Ls;
            po.off_tileL = planes->off_tileL;
            po.off_tileOff = planes->off_tileOff;
            po.off_rA = planes->off_rA;
            po.off_rB = planes->off_rB;
            po.off_CA = planes->off_CA;
            po.stride_batchA = planes->stride_batchA;
        }
        hipLaunchKernelGGL(k_schedule_plans, dim3((unsigned)(d.batch + lay.nplans + (lay.cbsg ? 1 : 0))), dim3(1024), 0,
                           st, L, d.strideL, d.batch, d.M, d.L_max, lay, ws, d.seed, d.polarity, po);
        return hipGetLastError();
    }
    if (draws && d.batch != 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_schedule, dim3((unsigned)d.batch + (d.rng == SC_RNG_SOBOL8_CBSG ? 1u : 0u)), dim3(1024), 0, st, L, d.strideL, d.M, d.L_max, lay, ws,
                       d.seed, d.rng, draws ? lay.LBS : 0);
    return hipGetLastError();
}

}  // namespace scg
