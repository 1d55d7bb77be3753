// kernels.h -- device data layout and kernel launchers of the solver.
//
// Layout in HBM per instance (all int32 unless noted; built by table_kernel):
//   T   [n][n]        folded upper-triangular matrix (input of the table build)
//   ML  [2A][64]      lane parts of the interaction rows M_int[v][s] = sum over
//                     set suffix bits t of T[v][A+t] (Sec. II-C: M_int =
//                     Q_ps U_B^T).  Lane `lane` owns columns s = j*64 + lane,
//                     j < MC (column-wise split, Sec. III-C.2), and the sum
//                     over the six lowest suffix bits depends on the lane
//                     only, the sum over the others on j only:
//                     M_int[v][j*64 + lane] = ML[v][lane] + MH[v][j].
//                     Rows A..2A-1 are the negated ones
//   EB  [64 MC]       suffix energies E_s(U_B) (Sec. III-A, preprocessing 2)
//                     Packed instances (tiers 4, 5) hold 2^(B-1) words: word c
//                     holds column c in its low 16 bits and column c + 2^(B-1)
//                     (suffix variable A set) in its high 16 bits, EB biased
//                     by kPackBias in each half and ML, MH words the sums of
//                     the two columns' parts (low + high 2^16, mod 2^32), so
//                     one 32-bit add moves both energies (see kPackSumLimit)
//   S   [A][64]       S[w][l] = T[min(l,w)][max(l,w)] for l != w < A, else 0:
//                     the prefix couplings, one lane per variable
//   K   [6][32]+[16]  (all instances' K tables are contiguous) tier-2 bound
//                     constants per 64-step super-block offset o and table
//                     (0: o < 32; 1: o >= 32, level-5 bit rising; 2: o >= 32,
//                     falling), entry o mod 32: rows 0..2 hold C2 = ELOW + D,
//                     rows 3..5 hold D, where D is the minimum over all 2^B
//                     columns of E_sd(o) - E_sd(super-block start) and ELOW
//                     the low-low coupling energy of the low pattern at o;
//                     then the minima of C2 over each bound-test segment
//                     (one a table; the other entries unused); then
//                     SL[64][5]: SL[w][t] = coupling of prefix variable w
//                     with the low variable A-1-t (0 when equal), so a flip
//                     of w moves the low fields by scalar loads only; then
//                     MH[2A][MC]: the column parts of the interaction rows
//                     (see ML), read by scalar loads
//   Qf  [n][n] fp32   caller's float32 Q (fp32 instances only, for rescoring)
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace qk {

constexpr int kWave = 64;
constexpr int kSuperLog = 6;          // unrolled super-block: 64 Gray steps
constexpr int kLowLevels = 5;         // Gray levels with static patterns in a super-block
constexpr int kPatterns = 1 << kLowLevels;
constexpr int kBlockWaves = 4;        // waves of a block that walks one instance alone
constexpr int kSegSteps = 32;         // steps per bound-test segment (measured
                                      // 3.7% faster than 16 at n = 44)
static_assert(kPatterns == kSegSteps, "a segment is a table of K");
constexpr int kKC2Min = 6 * kPatterns;   // min of C2 per (table, segment)
constexpr int kKBound = kKC2Min + 16;    // bound constants at the head of a K table (and
                                         // padding: a row of MH is a 64-byte line)
constexpr int kMaxCols = 16;          // words per lane (MC) of the widest variant
constexpr int kMaxVgprLevels = 12;    // at most Gray levels 0..11 keep their M_int row in VGPRs
constexpr int32_t kNoEnergy = 1 << 30;  // above every energy the walk can meet
constexpr int kMaxVars = 60;          // largest n the planner accepts
constexpr int kMaxPrefixRows = 60 - 6;   // A = n - B <= 60 - 6
constexpr int kKHigh = kKBound + kLowLevels * kWave;   // MH[2A][MC], after SL[w][t]
constexpr int kKTable = kKHigh + 2 * kMaxPrefixRows * kMaxCols;
// Packed walk (tiers 4 and 5, the int16 energies of Sec. IV-B "Data types"
// at two per 32-bit word).  Word = (E_lo + c + kPackBias) + (E_hi + c +
// kPackBias) 2^16 and a row word = m_lo + m_hi 2^16 (mod 2^32), with c the
// instance's shift below: the map is additive mod 2^32, so a
// 32-bit add of a row word adds m_lo and m_hi to the two halves however the
// intermediate carries fall, and a word decodes exactly whenever both biased
// halves lie in [0, 2^16).  The planner proves every chunk energy E_sd + c
// (c = Inst::pack_shift, a constant per instance) a signed 16-bit value from
// the exact extremes of E_sd over all prefixes and columns, and picks c so
// that the least biased half is 0.
constexpr int32_t kPackBias = 1 << 15;
constexpr int64_t kPackSumLimit = (int64_t(1) << 15) - 1;

// Wide words (a lone tier-2 walk): three shifted chunk energies, each in [0,
// 2^kWideBits), in a 64-bit word, whose add issues at half the rate of a 32-bit
// one: 3 energies in the time of 2.  The 16 columns of a lane are five such
// words and one plain one.  As with the packed words the map is additive mod
// 2^64, so a word decodes exactly whenever its energies lie in range, which
// their exact extremes prove.
constexpr int kWideBits = 21;
constexpr int kWideWords = 5;

struct ItemRes;

// An instance whose Q is prepared on the device (lone solve of a device
// pointer): the preparation's outcome, written by prepare_kernel.
constexpr int64_t kExactSumLimit = (int64_t(1) << 30) - 1;   // sum |T| bound of the int32 walk
constexpr int32_t kPrepOverflow = 1;    // int32 input with sum |T| above kExactSumLimit
constexpr int32_t kPrepNonFinite = 2;   // float32 input with a NaN or Inf
constexpr int32_t kPrepInternal = 3;    // scaled float32 matrix above the bound
struct PrepOut {
    int32_t status;      // 0, or kPrepOverflow / kPrepNonFinite / kPrepInternal
    int32_t p;           // fixed-point exponent (float32 input), else 0
    int64_t sum_abs;     // sum of |T_ij|, i <= j, of the int32 matrix solved
    double eps_q;        // per-state quantisation bound (float32 input), else 0
    int64_t hist_lo;     // top-k histogram: energy of bin 0's lower edge ...
    int32_t hist_shift;  // ... and the bin shift
    int32_t pad;
};

struct Inst {
    const int32_t *T;
    int32_t *ML;
    int32_t *EB;
    int32_t *S;
    int32_t *K;            // this instance's K table (kslot-th table of the K array)
    const float *Qf;
    ItemRes *res;          // this launch's item results: item g of the launch
                           // (item_begin <= g < item_end) that found a candidate
                           // writes res[g - item_begin] ...
    uint32_t *bits;        // ... and sets bit bit0 + (g - item_begin) of the
                           // instance's item bitmap (bit q <-> res record q of
                           // the instance; cleared by the table build), so the
                           // finish reads only records that were written
    uint64_t bit0;
    int n, A, B, L;
    int direct;            // 1: no walk, direct evaluation of all 2^n states
    int kslot;             // index of the K table in the launch's K array
    int packed;            // 1: ML, MH and EB in the packed 16-bit layout (tiers 4, 5)
    int32_t pack_shift;    // c added to every chunk energy in EB and taken
                           // off the prefix energy: tiers 4, 5 make every
                           // E_sd + c a signed 16-bit value, the int32 walk
                           // makes it non-negative (written by prepare_kernel
                           // for a device-prepared instance)
    int wide;              // 1: the lone walk runs on wide words (device-prepared: set
                           // in the image where the shape allows it, and cleared by
                           // prepare_kernel where the energies do not)
    uint64_t item_begin;   // this launch's walk-item range [item_begin, item_end)
    uint64_t item_end;
    uint64_t item_local0;  // the instance's own item number of launch item item_begin
    uint64_t n_items;      // item records of the instance (res[0 .. n_items), bitmap
                           // words bits[0 .. ceil(n_items / 32)))
    int32_t *gbest;        // best energy any wave has found for the instance
                           // (set by the table build)
    const PrepOut *prep;   // device-prepared instance: its preparation (an error
                           // makes the walk skip all items), else null
};

struct ItemRes {
    int32_t E;         // best energy accepted inside the item
    int32_t found;     // 1 (only items that found a candidate write a record)
    uint64_t row;      // prefix row (U_A row) of that chunk
};

// Top-k (k > 1) state of one walk launch over a single instance.  Each
// wave keeps, in listE / listR (its slot of k entries), the k smallest chunk
// keys (E_p + min over the chunk, prefix row) it has met; a chunk can belong to the instance's k smallest
// chunks only if its minimum is at most the largest E of any full list, so
// waves share that bound through gthr (atomic min).
struct TopkWalk {
    int32_t *listE;      // [waves][k] chunk minima
    uint64_t *listR;     // [waves][k] prefix rows of those chunks
    int32_t *listCount;  // [waves] entries used (written by every wave on exit)
    int32_t *gthr;       // shared bound, kNoEnergy before the walk
    uint32_t *hist;      // [kTopkBins] keys entered into any list, by energy bin, then
                         // [kWave] by kTopkFine bins (zeroed)
    int64_t hist_lo;     // energy of bin 0's lower edge (-sum|T|)
    int hist_shift;      // bin = (E - hist_lo) >> hist_shift
    int k;
    const PrepOut *prep; // device-prepared instance: hist_lo and hist_shift come
                         // from here instead (null otherwise)
};
constexpr int kTopkBins = 16384;
constexpr int kTopkFine = kTopkBins / kWave;
constexpr int kTopkLook = 8;   // entered keys of a wave per look at the counts

// One state of a top-k answer; the same layout as qubo_state_t.
struct TopkState {
    int64_t E;           // exact integer energy
    double E64;          // float64 rescore (fp32) or (double)E
    uint64_t index;      // U_N row
};

// Device buffers of the top-k finish of a single instance.
struct TopkBufs {
    TopkWalk walk;
    int waves;           // lists in walk.listE (walked instances)
    int32_t *candE;      // [waves * k] list entries <= the final bound, dense ...
    uint64_t *candR;
    int32_t *candN;      // [1] their number (zero before the finish)
    int32_t *chunkE;     // [k] the k smallest chunk keys, in no order ...
    uint64_t *chunkR;    // [k] ... and their prefix rows
    int32_t *chunkCount; // [0] chunks selected (min(k, chunks met)), [1] their largest key
    int32_t *stE;        // [k << B] (or [2^n] direct) candidate state energies
    uint64_t *stI;       // same, U_N rows
    int32_t *segCount;   // [0]: states kept by the rescan (2^n when direct)
    int32_t *selE;       // [k] the k smallest states, in no order
    uint64_t *selR;
    int32_t *selCount;   // [0] states selected, [1] their largest energy
    TopkState *out;      // [k] the states in order of (E, index)
};


struct FinalRes {
    int64_t E;         // exact integer energy of the answer
    uint64_t index;    // U_N row of the answer
    double E64;        // float64 rescore from Qf (fp32 instances)
    int32_t status;    // 0 ok, nonzero: self-check failure
    int32_t pad;
    uint64_t walk_ticks;   // from the end of instance 0's descents in the table build
                           // to the finish's start (k > 1: to the compaction's, the
                           // seed included), in ticks of the device's constant clock
};

// Where a top-k finish leaves its results: device or mapped host memory.
struct TopkResults {
    FinalRes *best;
    PrepOut *prep;       // the preparation's outcome, or null
    TopkState *topk;     // [k] answer (fp32: sorted by (E64, index))
};
constexpr int64_t kTopkBadState = INT64_MIN;   // E of a state whose energy did not verify

// Host image of a lone solve, read by the first kernel itself instead of by a
// copy ahead of it (a 4 us copy and a 10 us gap): `copy_bytes` of the mapped
// host block `src` go to `dst`, and the `zero_bytes` after them are cleared.
// src null: the image is in place.
struct Upload {
    const unsigned char *src;
    unsigned char *dst;
    uint32_t copy_bytes, zero_from, zero_bytes;
};

// Word of a walk launch's counters that holds its start (and, top-k, the word
// after it its end), in ticks of the device clock.
constexpr int kClockWord = 1;

// Fold, check and (float32) scale the caller's device matrix dQ (n x n,
// row-major, int32 or float32) into the instance's upper-triangular int32 T
// (d_T, n x n), exactly as the host planner does, and write the outcome to
// *d_prep and the walk's chunk-energy shift to d_inst->pack_shift (the
// descriptor's split A, B already set; int32 walk only).  On an input error
// T is left zero and the status says why.
hipError_t launch_prepare(const void *dQ, int n, int is_fp32, int32_t *d_T, PrepOut *d_prep,
                          Inst *d_inst, const Upload &up, hipStream_t stream);

// Item counters of one walk launch: kQueues of them, kQueueStride words apart.
// Wave b walks item b first, without a claim, and then claims from queue b mod
// kQueues, whose items are those of the same residue.  Atomics on one address
// complete one per 12.4 ns: a single counter kept the waves of a fresh grid
// (4096 at once) waiting for up to 50 us, and no walk could hand out items
// faster.  Workgroups go to the eight XCDs in turn, so a queue is an XCD's.
constexpr int kQueues = 8;
constexpr int kQueueStride = 32;
constexpr int kCounterWords = kQueues * kQueueStride;
// Where items are long (2^kStealSteps steps and more), a wave whose queue is
// empty takes items of the others: the XCDs do not run at one speed (queues
// left alone cost 1.2% at n = 44 and 2.5% on 4096 instances).  Shorter items
// end together anyway, and the tries would cost what they save.
constexpr int kStealSteps = 12;

// How the items of a walk launch are claimed.  A lone instance of kRunItems
// items and more hands out the first 85% of them in runs of four consecutive
// ones, which one set-up starts (2.1 us of a SIMD's time each), and the rest
// one by one, so that the waves end together.  Measured, with the items a
// quarter as long, against items of the old length without runs: n = 33 166
// -> 160 us, n = 34 315 -> 294, packed n = 36 610 -> 570, n = 36 1100 -> 1068,
// n = 38 4324 -> 4190.  Runs beyond 2^kRunMaxSteps steps gain nothing.
constexpr uint64_t kRunItems = uint64_t(1) << 15;
constexpr int kRunLog = 2;
constexpr int kRunMaxSteps = 14;
struct WalkClaims {
    uint64_t claims;     // claims in all: `runs` runs of 2^run_log consecutive items each,
    uint64_t runs;       // then the remaining items one by one (one instance only)
    int run_log;
    int others;          // queues a wave tries after its own (see kStealSteps)
};

// Builds ML, EB, S, K for every instance, clears each instance's item bitmap,
// sets its shared best (to the energy of greedy descents), and zeroes the item
// counters of n_groups walk launches (kCounterWords each).  With up.src (one
// instance) the descriptor and T are read there.
hipError_t launch_tables(const Inst *d_insts, int n_inst, unsigned long long *d_counters,
                         int n_groups, const Upload &up, hipStream_t stream);

// The same for n_inst instances whose host images ups[0 .. n_inst) (a mapped
// array) the build puts in place.
hipError_t launch_tables_upload(const Upload *ups, int n_inst, hipStream_t stream);

// Puts one host image in place.
hipError_t launch_upload(const Upload &up, hipStream_t stream);

// Persistent Gray walk over all items (d_counter: the launch's kCounterWords
// zeroed words, max_L: log2 of the longest item's steps); `waves` resident wavefronts.  d_k is
// the contiguous array of K tables (instance i's at insts[i].kslot*kKTable).
// Variant: mcols words per lane (B = 6 + log2 mcols, 7 + log2 mcols for
// tiers 4 and 5), the M_int rows of Gray levels below vgpr_levels cached in
// VGPRs (higher ones from L2), tier.
// Tiers 3 and 5 (top-k lists) need `tk` and exactly one instance; tiers 1,
// 2 and 4 ignore it (may be null).  wide (one instance): 1 walks it on wide
// words, 2 leaves that to its descriptor (both kernels are launched, and the
// one it does not name returns at once).
hipError_t launch_walk(int mcols, int vgpr_levels, int tier, const Inst *d_insts, int n_inst,
                       uint64_t total_items, int max_L, unsigned long long *d_counter,
                       const int32_t *d_k,
                       int waves, hipStream_t stream, const TopkWalk *tk = nullptr, int wide = 0);

// Two groups of one launch_walk each, on 16 columns and row cache "4", of tiers 2
// and 4, as one launch.
struct WalkPart {
    const Inst *d_insts;
    int n_inst;
    uint64_t total_items;
    int max_L;
    unsigned long long *d_counter;
};
hipError_t launch_walk_pair(const WalkPart &tier2, const WalkPart &tier4, const int32_t *d_k,
                            int waves, hipStream_t stream);

// Whether a (mcols, vgpr_levels) walk variant is compiled in, and whether
// its packed form (tiers 4 and 5: 2 mcols 64 suffix columns) is.
bool walk_variant_exists(int mcols, int vgpr_levels);
bool walk_packed_exists(int mcols, int vgpr_levels);

// Resident walk wavefronts per CU for a variant (occupancy query, >= 1);
int walk_occupancy(int mcols, int vgpr_levels, int tier);

// LDS bytes of one tier-3 wave's list scalars (its k entries are in listE /
// listR in global memory).
constexpr int kTopkMetaWords = 12 + kWave + kWave / 2;  // 64-bit words: scalars, queued keys
__host__ __device__ constexpr size_t topk_lds_bytes()
{
    return size_t(kTopkMetaWords) * 8;
}

// Seeds the shared top-k bound *d_gthr of one walked instance before its
// walk: the k-th smallest energy of up to 4096 states with distinct prefix
// rows near a local minimum (every walked chunk must be in the walk: full
// item range only).  Leaves *d_gthr unchanged when the instance has fewer
// such states than k.
hipError_t launch_topk_seed(const Inst *d_inst, int32_t *d_gthr, int k, hipStream_t stream);

// Top-k finish of one instance (descriptor d_inst, host copy hI): select the
// k smallest chunks of the walk lists, rescan them (or, direct, evaluate all
// 2^n states), select and sort the k smallest states, verify their energies
// and write the results (best's status 4: fewer than k states).
hipError_t launch_topk_finish(const Inst *d_inst, const Inst &hI, const TopkBufs &buf, int k,
                              const TopkResults &to, unsigned long long *d_counters,
                              hipStream_t stream);

// Per-instance reduction of item results (insts[i].res[0..n_items)), argmin
// rescan (or direct evaluation for tiny n) and float64 rescoring; one
// FinalRes per descriptor.  up.src (a direct instance, whose first kernel this
// is): the descriptor, T and Q are read there.  d_counters: the walk's (its
// start time), or null.  prep_out: receives the instance's preparation, or null.
hipError_t launch_finish(const Inst *d_insts, int n_inst, FinalRes *d_out, const Upload &up,
                         const unsigned long long *d_counters, PrepOut *prep_out,
                         hipStream_t stream);

}  // namespace qk
