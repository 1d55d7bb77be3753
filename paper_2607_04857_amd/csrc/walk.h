// walk.h -- the Gray-walk kernel template (Sec. III-B, Eq. incremental_update)
// and its per-variant launch helpers.  Each walk_*.hip file instantiates a
// few variants, so that the variants compile in parallel.
#pragma once

#include "kcommon.h"
#include "walk_variants.h"

namespace qk {

// ---------------------------------------------------------------- walk

// Wave-wide minimum for the tier-2 super-block base: DPP inside each row of
// 16 lanes, then row broadcasts, result in lane 63.
__device__ __forceinline__ int32_t wave_min_bcast(int32_t v)
{
    // lanes a DPP source leaves unwritten read INT32_MAX, the identity of min
    constexpr int32_t I = INT32_MAX;
    v = min(v, __builtin_amdgcn_update_dpp(I, v, 0xB1, 0xF, 0xF, false));   // quad_perm 1,0,3,2
    v = min(v, __builtin_amdgcn_update_dpp(I, v, 0x4E, 0xF, 0xF, false));   // quad_perm 2,3,0,1
    v = min(v, __builtin_amdgcn_update_dpp(I, v, 0x124, 0xF, 0xF, false));  // row_ror:4
    v = min(v, __builtin_amdgcn_update_dpp(I, v, 0x128, 0xF, 0xF, false));  // row_ror:8
    v = min(v, __builtin_amdgcn_update_dpp(I, v, 0x142, 0xA, 0xF, false));  // row_bcast:15
    v = min(v, __builtin_amdgcn_update_dpp(I, v, 0x143, 0xC, 0xF, false));  // row_bcast:31
    return __builtin_amdgcn_readlane(v, 63);
}

// TIER 1: the chunk minimum (v_min3 tree) is compared with the threshold at
//         every Gray step.
// TIER 2: each lane takes its chunk minimum lm0 once per 64-step
//         super-block; at offset o the chunk minimum is at least
//         W0 + D(o) (table K), W0 the wave minimum of lm0, so step o needs
//         only the scalar test W0 <= THR - D(o).  Each 32-step segment (a
//         half super-block: the level-5 flip separates the two) first tests
//         lm0 against an upper bound of its 32 thresholds (one vector
//         compare); only when a lane passes are W0 and the exact thresholds
//         formed and tested, step by step.
// TIER 4, 5: tiers 2 and 3 on the packed layout: each of the MC words of a
//         lane holds two chunk energies (columns c and c + 2^(B-1) of the
//         chunk), so one 32-bit add per word and step moves two states (Eq.
//         incremental_update at 16-bit precision); only the lane minimum
//         (packed 16-bit minima, then the unbiased smaller half) and the
//         prefix energy's shift differ.
// Where the rows of the frequent Gray levels live (levels below G are in
// VGPRs, except where LDS holds them; RC):
//  kRowsVgpr    VGPRs only
//  kRowsWave    levels 3 and 4 in LDS, a copy per wave (2 x MC x 64 dwords),
//               which leaves room for a fourth wave per SIMD
//  kRowsBlock   G = 4: levels 4 to 8 in LDS, one copy for the four waves of a
//               block, which all walk the launch's one instance (a copy per
//               wave has room for two rows).  Rows 0 and 1 are levels 4 and 5,
//               then come level 6's row and its negation, 7's and 8's: a
//               boundary flip of either direction is one code path.  Nearly
//               every flip then is one full-rate add per word: a row formed
//               from its parts takes a three-operand add, which issues at half
//               the rate (one on every boundary was 1.5% of the VALU work).
//               Measured: n = 44 walk 255.9 -> 254.6 ms, n = 33 and 36 equal.
//               A top-k walk holds what survives the list's call across the
//               super-block; with G = 4 that spilled 9 registers that each
//               half reloads, so its rows start at level 3 (n = 36 packed,
//               k = 100 walk 795 -> 725 us, n = 33 float32, k = 1024 320 -> 280,
//               n = 30, k = 4 57 -> 52).
//  kRowsWide    the chunk vector in wide words (kWideBits): the walk is bound
//               by its adds, and five 64-bit ones and one of 32 bits take 11
//               issue slots where 16 of 32 bits take 16.  As kRowsBlock, with
//               levels 0-2 in VGPRs and 3-8 in LDS, and every row as well as
//               its negation, since no 64-bit add subtracts: 128 VGPRs, and no
//               spill in the loop.  A boundary above level 8 forms its row from its parts
//               (1 in 8 of the boundaries).  Measured against kRowsBlock on the
//               same instances: n = 44 walk 254.6 -> 192.5 ms (169 ms at the
//               adds' full rate; 194 with level 9 in LDS and the plain words'
//               rows apart, which takes a second address register), n = 40
//               16.4 -> 12.4, n = 36 1.07 -> 0.85, n = 33 0.160 -> 0.139.
enum { kRowsVgpr = 0, kRowsWave = 1, kRowsBlock = 2, kRowsWide = 3 };
constexpr int kWideLow = 3;       // first Gray level of the wide rows in LDS
constexpr int kWideTop = 8;       // last one
constexpr int kWideRows = 2 * (kWideTop - kWideLow + 1);
// a row: its words, then the plain one in a slot of the same size (one address
// register for all): 36 KB in all, four blocks a CU
constexpr size_t kWideRowBytes = kWave * (kWideWords + 1) * sizeof(uint64_t);
constexpr int kBlockLow = 4;      // first Gray level of the block's rows,
constexpr int kBlockLowTopk = 3;  // of a top-k walk, which needs the VGPRs
constexpr int kBlockTop = 8;      // last one
// rows for first level G (plain up to level 5, then signed): 32 KB at MC = 16
// and G = 4, 36 KB at G = 3, four blocks a CU
constexpr int block_rows(int G) { return (kSuperLog - G) + 2 * (kBlockTop - kSuperLog + 1); }

template <int RC>
constexpr int walk_block_waves()
{
    return RC == kRowsBlock || RC == kRowsWide ? kBlockWaves : 1;
}
// Resident waves per SIMD each variant is register-allocated for: the full
// 12-level row cache fits 256 VGPRs (2 waves); the 8- and 6-level caches
// leave room for a third (MC=16) or a fourth (MC=8) wave.
template <int MC, int G, int RC = kRowsVgpr>
constexpr int walk_waves_per_simd()
{
    return RC != kRowsVgpr ? 4 : (G >= 12 ? (MC >= 16 ? 2 : (MC >= 8 ? 3 : 4)) : (G <= 5 ? 4 : (MC >= 16 ? 3 : 4)));
}
// (G = 6 and 8 with MC = 16 target 3 waves, G = 5 four; 8 and 5 spill a few
// values outside the unrolled steps.)

// Bytes of dynamic LDS ahead of the LDS rows (the lists of the block's waves,
// tiers 3 and 5), 16-aligned.
__host__ __device__ constexpr size_t lds_rows_offset(int tier, int waves)
{
    return (tier == 3 || tier == 5) ? (size_t(waves) * topk_lds_bytes() + 15) & ~size_t(15) : 0;
}
template <int MC, int G, int RC>
constexpr size_t lds_rows_bytes()
{
    constexpr int rows = RC == kRowsBlock ? block_rows(G) : RC == kRowsWave ? 2 : 0;
    if (RC == kRowsWide) return kWideRows * kWideRowBytes;
    return size_t(rows) * MC * kWave * sizeof(int32_t);
}

// ---- tier-3 list (top-k), one a wave.  Its scalars and the keys met in the
// current super-block live in dynamic LDS (kTopkMetaWords 64-bit words); its k
// entries (E and prefix row) live in global memory, at listE / listR + the
// wave's number * k, and entry p is written and read only by lane p % 64, so
// each lane reads its own earlier writes in program order and no fence is
// needed.  Only the rare candidate path touches the entries (from L2), and the
// LDS stays free for the row cache, so tier 3 runs the LDS row-cache variants
// at four waves per SIMD whatever k is.  No list state is held in registers,
// and the list code sits in functions that are not inlined, called at one
// place of the walk.
//   M[0] entries used  M[1] slot of the largest key  M[2] its E (kNoEnergy
//   until the list is full)  M[3] lowest shared bound seen  M[4] k
//   M[5] histogram bin shift  M[6] keys since the last look at the
//   counts  M[7] the list's number
//   P[0] the largest key's row  P[1] gthr  P[2] listE  P[3] listR
//   P[4] listCount  P[5] hist  P[6] hist_lo
//   (M = words 0..3 as int32, P = words 4..11, then the queue of keys met)
//
// Shared bound.  Every key that enters any wave's list is also counted in a
// device-wide histogram by energy bin.  Keys entered belong to distinct
// chunks (each chunk is walked once), so if the bins up to b hold at least k
// of them, at least k chunks have a key <= the upper edge of bin b, which
// therefore bounds the instance's k-th smallest chunk key: no chunk above it
// can be among the k smallest.  A wave that has entered kTopkLook keys
// recomputes that edge and lowers gthr; every wave's threshold is min(its own
// list's largest E when full, gthr as the wave last saw it).
extern __shared__ uint64_t tk_lds[];

__device__ __forceinline__ int tk_lane() { return int(threadIdx.x) % kWave; }
__device__ __forceinline__ uint64_t *tk_meta()
{
    return tk_lds + sread(int(threadIdx.x) / kWave) * kTopkMetaWords;
}
__device__ __forceinline__ int32_t *tk_M() { return reinterpret_cast<int32_t *>(tk_meta()); }
__device__ __forceinline__ uint64_t *tk_P() { return tk_meta() + 4; }
// the keys the wave has met in its current super-block: at most one a step
__device__ __forceinline__ uint64_t *tk_queueR() { return tk_meta() + 12; }
__device__ __forceinline__ int32_t *tk_queueE()
{
    return reinterpret_cast<int32_t *>(tk_queueR() + kWave);
}
// The wave's LDS accesses before this are done before those after it (they
// complete in order: this holds the compiler's order).
__device__ __forceinline__ void tk_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// this wave's k list entries in global memory
__device__ __forceinline__ int32_t *tk_E(int k)
{
    return reinterpret_cast<int32_t *>(sread64(tk_P()[2])) + size_t(sread(tk_M()[7])) * size_t(k);
}
__device__ __forceinline__ uint64_t *tk_R(int k)
{
    return reinterpret_cast<uint64_t *>(sread64(tk_P()[3])) + size_t(sread(tk_M()[7])) * size_t(k);
}
__device__ __forceinline__ int32_t *tk_gthr()
{
    return reinterpret_cast<int32_t *>(sread64(tk_P()[1]));
}

// list: the wave's number in the grid
__device__ __forceinline__ void tk_init(const TopkWalk &tk, int list)
{
    if (tk_lane() == 0) {
        int32_t *M = tk_M();
        uint64_t *P = tk_P();
        M[0] = 0;
        M[1] = 0;
        M[2] = kNoEnergy;
        M[3] = kNoEnergy;
        M[4] = tk.k;
        M[5] = tk.prep ? tk.prep->hist_shift : tk.hist_shift;
        M[6] = 0;
        M[7] = list;
        P[0] = 0;
        P[1] = reinterpret_cast<uint64_t>(tk.gthr);
        P[2] = reinterpret_cast<uint64_t>(tk.listE);
        P[3] = reinterpret_cast<uint64_t>(tk.listR);
        P[4] = reinterpret_cast<uint64_t>(tk.listCount);
        P[5] = reinterpret_cast<uint64_t>(tk.hist);
        P[6] = uint64_t(tk.prep ? tk.prep->hist_lo : tk.hist_lo);
    }
    tk_sync();
}

// Threshold at an item start: min(largest E of the full list, shared bound).
__device__ __noinline__ int32_t tk_threshold()
{
    int32_t *M = tk_M();
    const int32_t g = sread(__hip_atomic_load(tk_gthr(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    const int32_t gm = min(sread(M[3]), g);
    const int32_t t = min(sread(M[2]), gm);
    tk_sync();
    if (tk_lane() == 0) M[3] = gm;
    tk_sync();
    return t;
}

// Largest key (E, row) of the full list: store it and its slot, publish its
// E to the shared bound; returns that E.
__device__ int32_t tk_rescan(int k)
{
    tk_sync();              // lane 0's LDS scalar stores are visible to the wave
    const int lane = tk_lane();
    const int32_t *E = tk_E(k);
    const uint64_t *R = tk_R(k);
    int32_t mE = INT32_MIN;
    uint64_t mR = 0;
    int mP = 0;
    for (int p = lane; p < k; p += kWave) {
        const int32_t e = E[p];
        const uint64_t r = R[p];
        if (e > mE || (e == mE && r > mR)) {
            mE = e;
            mR = r;
            mP = p;
        }
    }
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) {
        const int32_t oE = __shfl_xor(mE, off, kWave);
        const uint64_t oR = __shfl_xor(mR, off, kWave);
        const int oP = __shfl_xor(mP, off, kWave);
        if (oE > mE || (oE == mE && oR > mR)) {
            mE = oE;
            mR = oR;
            mP = oP;
        }
    }
    mE = sread(mE);
    if (lane == 0) {
        int32_t *M = tk_M();
        M[1] = mP;
        M[2] = mE;
        M[3] = min(M[3], mE);
        tk_P()[0] = mR;
        if (mE < __hip_atomic_load(tk_gthr(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMin(tk_gthr(), mE);
    }
    return mE;
}

// Count this lane's key energy Ec in the shared histogram: two atomics that
// nothing waits for (at two levels, so that a look at the counts takes two
// loads).
__device__ __forceinline__ int tk_bin(int32_t E)
{
    const int64_t b = (int64_t(E) - int64_t(sread64(tk_P()[6]))) >> sread(tk_M()[5]);
    return int(b < 0 ? 0 : (b >= kTopkBins ? kTopkBins - 1 : b));
}
__device__ __forceinline__ void tk_count(int32_t Ec)
{
    uint32_t *hist = reinterpret_cast<uint32_t *>(sread64(tk_P()[5]));
    const int b = tk_bin(Ec);
    atomicAdd(&hist[b], 1u);
    atomicAdd(&hist[kTopkBins + b / kTopkFine], 1u);
}

// The shared bound from the counts: the upper edge of the first bin where the
// running count reaches k, by lanes over the coarse bins and then over the
// coarse bin's own (counts that are not there yet only leave it higher).
// Lowers gthr to it; returns gthr.
__device__ int32_t tk_bound(int k)
{
    uint32_t *hist = reinterpret_cast<uint32_t *>(sread64(tk_P()[5]));
    const int lane = tk_lane();
    auto count = [&](int at) {
        return __hip_atomic_load(&hist[at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // inclusive prefix sum over the wave
    auto prefix = [&](uint32_t c) {
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const uint32_t o = __shfl_up(c, off, kWave);
            if (lane >= off) c += o;
        }
        return c;
    };
    const int32_t gv = __hip_atomic_load(tk_gthr(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t c0 = count(kTopkBins + lane);
    const int32_t g = sread(gv);
    const uint32_t cum = prefix(c0);
    const uint64_t hit = __builtin_amdgcn_ballot_w64(cum >= uint32_t(k));
    if (hit == 0) return g;
    const int cb = int(__builtin_ctzll(hit));
    const uint32_t need = uint32_t(k) - uint32_t(__builtin_amdgcn_readlane(int32_t(cum - c0), cb));
    constexpr int kPer = kTopkFine / kWave;
    uint32_t f[kPer], sum = 0;
#pragma unroll
    for (int x = 0; x < kPer; x++) f[x] = count(cb * kTopkFine + kPer * lane + x);
#pragma unroll
    for (int x = 0; x < kPer; x++) f[x] = sum += f[x];
    const uint32_t before = prefix(sum) - sum;
    int past = 0;   // this lane's bins whose running count is below need
#pragma unroll
    for (int x = 0; x < kPer; x++) past += before + f[x] < need ? 1 : 0;
    const uint64_t fhit = __builtin_amdgcn_ballot_w64(past < kPer);
    int bin = (cb + 1) * kTopkFine - 1;
    if (fhit) {
        const int fl = int(__builtin_ctzll(fhit));
        bin = cb * kTopkFine + kPer * fl + __builtin_amdgcn_readlane(past, fl);
    }
    const int64_t edge =
        int64_t(sread64(tk_P()[6])) + (int64_t(bin + 1) << sread(tk_M()[5])) - 1;
    const int32_t T = edge > int64_t(kNoEnergy) ? kNoEnergy : int32_t(edge);
    if (lane == 0 && T < g) atomicMin(tk_gthr(), T);
    return min(T, g);
}

// Offer chunk key (Ec, rc) to the wave's list: append while it has room, else
// replace the largest key if (Ec, rc) is smaller.
__device__ void tk_insert(int32_t Ec, uint64_t rc)
{
    int32_t *M = tk_M();
    const int cnt = sread(M[0]);
    const int k = sread(M[4]);
    int pos = cnt;
    if (cnt >= k) {
        const int32_t lkth = sread(M[2]);
        const uint64_t lkR = sread64(tk_P()[0]);
        if (!(Ec < lkth || (Ec == lkth && rc < lkR))) return;
        pos = sread(M[1]);
    }
    tk_sync();
    if (tk_lane() == pos % kWave) {   // the lane that owns entry pos
        tk_E(k)[pos] = Ec;
        tk_R(k)[pos] = rc;
    }
    if (tk_lane() == 0) M[0] = max(cnt, pos + 1);
    tk_sync();
    if (pos + 1 == k || cnt >= k) (void)tk_rescan(k);
    if (tk_lane() == 0) tk_count(Ec);
}

// Enter the nq (1 .. 64) queued keys of a super-block into the wave's list and
// the counts; returns the new threshold.  Low keys lie close together in the
// walk, so the few thousand that enter come to some waves by the dozen, and
// those waves end the walk: with room in the list the lanes enter them side by
// side, and nothing in global memory is waited for except that a wave looks at
// the counts once in kTopkLook keys.  (An insertion at a time, with three
// replies and the counts awaited, had made the walk of n = 31, k = 1024 take
// 205 us and of n = 16, k = 1024, where every chunk enters, 117; now 128 and 35.)
__device__ __noinline__ int32_t tk_drain(int nq)
{
    int32_t *M = tk_M();
    const int32_t *qE = tk_queueE();
    const uint64_t *qR = tk_queueR();
    nq = sread(nq);
    tk_sync();
    const int cnt = sread(M[0]);
    const int k = sread(M[4]);
    const int lane = tk_lane();
    if (cnt + nq <= k) {
        const int j = (lane - cnt) & (kWave - 1);   // entry cnt + j is this lane's
        if (j < nq) {
            tk_E(k)[cnt + j] = qE[j];
            tk_R(k)[cnt + j] = qR[j];
            tk_count(qE[j]);
        }
        tk_sync();
        if (lane == 0) M[0] = cnt + nq;
        tk_sync();
        if (cnt + nq == k) (void)tk_rescan(k);
    } else {
        for (int j = 0; j < nq; j++) tk_insert(sread(qE[j]), sread64(qR[j]));
    }
    const int seen = sread(M[6]) + nq;
    int32_t g = sread(M[3]);
    if (seen >= kTopkLook) g = min(g, tk_bound(k));
    tk_sync();
    if (lane == 0) {
        M[3] = g;
        M[6] = seen >= kTopkLook ? 0 : seen;
    }
    tk_sync();
    return min(sread(M[2]), g);
}

// Publish the number of entries of the wave's list (the entries are already
// in listE / listR, at the wave's number * k).
__device__ __noinline__ void tk_flush()
{
    tk_sync();
    const int32_t *M = tk_M();
    const uint64_t *P = tk_P();
    const int cnt = sread(M[0]);
    if (tk_lane() == 0) reinterpret_cast<int32_t *>(sread64(P[4]))[M[7]] = cnt;
}

// TIER 3: tier 2's bound test against a top-k threshold instead of the best
//         energy: the wave keeps the k smallest chunk keys it has met (above).
// own: a wave's first claim is its own number's, and the queues' start past
// those (see claim).
template <int MC, int G, int TIER, int RC>
// (No __restrict__ here: on an inlined function's parameters it cost the lone
// kernels some forty SGPRs.)
__device__ __forceinline__ void walk_items(const Inst *insts, int n_inst, WalkClaims wc,
                                           unsigned long long *counter,
                                           const int32_t *kall, TopkWalk tk,
                                           bool own)
{
    static_assert(TIER >= 1 && TIER <= 5, "tier");
    static_assert(RC == kRowsBlock  ? G == kBlockLow || G == kBlockLowTopk
                  : RC == kRowsWide ? G == kWideLow && MC == 3 * kWideWords + 1 && (TIER == 2 || TIER == 3)
                                    : G >= kLowLevels && G <= kMaxVgprLevels,
                  "VGPR-resident levels");
    static_assert(RC != kRowsBlock || TIER >= 2, "no per-step exact walk over the block's rows");
    constexpr bool LR = RC == kRowsWave, BR = RC == kRowsBlock, WD = RC == kRowsWide;
    constexpr bool LONE = BR || WD;   // blocks of four waves over one instance
    constexpr int WPB = walk_block_waves<RC>();
    // packed layout (tiers 4 and 5) and the test it runs (2: best, 3: top-k)
    constexpr bool PK = TIER >= 4;
    constexpr int BT = PK ? TIER - 2 : TIER;
    constexpr int SEG = kSegSteps;   // steps per bound-test segment
    constexpr int NSEG = (1 << kSuperLog) / SEG;
    const int lane = int(threadIdx.x) % kWave;
    const uint32_t ulane = threadIdx.x % kWave;
    const int bwave = WPB > 1 ? sread(int(threadIdx.x) / kWave) : 0;   // this wave of the block
    // log2 of the words per lane, and the suffix bits of a chunk
    constexpr int JB = cx_ctz(MC), B = JB + (PK ? 7 : 6);
    // wide words: the chunk vector W, X and the rows of levels 0-2, both signs
    // (X's rows need one), in place of E and R
    uint64_t W[kWideWords], RW[WD ? kWideLow : 1][2][kWideWords];
    int32_t X = 0, RX[WD ? kWideLow : 1];
    auto pin_wide = [&]() {
#pragma unroll
        for (int k = 0; k < kWideWords; k++) asm("" : "+v"(W[k]));
        asm("" : "+v"(X));
    };
    // this lane's chunk minimum (packed: over both halves of every word)
    auto lane_min = [&](const int32_t(&e)[MC]) {
        if constexpr (WD) return wide_min(W, X);
        else if constexpr (PK) return tree_min_packed<MC>(e);
        else return tree_min<MC>(e);
    };
    // the rows in dynamic LDS, after the (tier-3) list
    int32_t *const ldsR = reinterpret_cast<int32_t *>(
        reinterpret_cast<char *>(tk_lds) + lds_rows_offset(TIER, WPB));

    int cur = -1;
    // the tables, addressed as global memory (uniform base + lane offset +
    // immediate), not through generic pointers
    const gint32 *ML = nullptr, *S = nullptr;
    int kbase = 0;                // this instance's K table: kall[kbase ...] (scalar loads)
    // word j of this lane in M_int's (signed) row v: its lane part, one load
    // per lane, plus its column part, a scalar load
    auto lrow = [&](int v) { return ML[v * kWave + ulane]; };
    auto hrow = [&](int v) {
        return *reinterpret_cast<const ivec<MC> *>(kall + (kbase + kKHigh + v * MC));
    };
    int A = 0;
    int32_t R[G][MC];        // M_int rows of Gray levels 0..G-1 (variable A-1-t)
    int32_t Smid = 0;          // couplings of the middle-level variable, one lane each
    int32_t SmidL[kLowLevels];  // couplings of the middle-level variable with the low ones
    int32_t CR[kPatterns];   // low-low coupling increments per pattern
    int32_t best = kNoEnergy;     // tier 3: the current top-k threshold
    uint64_t bestRow = ~0ull;

    if constexpr (BT == 3) tk_init(tk, int(blockIdx.x) * WPB + bwave);

    // the next claim of this wave's queue (kQueues), or, where it is empty, of
    // one of the next wc.others queues
    uint32_t queue = blockIdx.x % kQueues;
    auto claim = [&]() {
        for (int k = 0;; k++) {
            uint64_t c = 0;
            if (lane == 0) c = atomicAdd(counter + queue * kQueueStride, 1ull);
            // a queue's first items are the waves' own
            const uint64_t first = own ? (gridDim.x * WPB + kQueues - 1 - queue) / kQueues : 0;
            const uint64_t v = (sread64(c) + first) * kQueues + queue;
            if (v < wc.claims || k >= wc.others) return v;
            queue = (queue + 1) % kQueues;
        }
    };
    // wide words: add signed row `row` of the LDS rows to the chunk vector
    auto add_wide = [&](int row) {
        const uint64_t *r = reinterpret_cast<const uint64_t *>(
                                reinterpret_cast<const char *>(ldsR) + size_t(row) * kWideRowBytes) +
                            lane;
#pragma unroll
        for (int k = 0; k < kWideWords; k++) W[k] += r[k * kWave];
        X += int32_t(uint32_t(r[kWideWords * kWave]));
    };
    if constexpr (WD) {
        const Inst &I = insts[0];
        if (I.wide == 0) return;
        A = I.A;
        ML = to_global(I.ML);
        kbase = I.kslot * kKTable;
        auto words = [&](int row, uint64_t *w, int32_t *x) {
            const int32_t ml = lrow(row);
            const ivec<MC> mh = hrow(row);
#pragma unroll
            for (int k = 0; k < kWideWords; k++)
                w[k] = wide_word(ml + mh[3 * k], ml + mh[3 * k + 1], ml + mh[3 * k + 2]);
            *x = ml + mh[MC - 1];
        };
        for (int r = bwave; r < kWideRows; r += WPB) {
            const int t = kWideLow + r / 2;
            if (t >= A) continue;
            uint64_t w[kWideWords];
            int32_t x;
            words((r % 2 ? 2 * A : A) - 1 - t, w, &x);
            uint64_t *p = reinterpret_cast<uint64_t *>(reinterpret_cast<char *>(ldsR) +
                                                       size_t(r) * kWideRowBytes) +
                          lane;
#pragma unroll
            for (int k = 0; k < kWideWords; k++) p[k * kWave] = w[k];
            p[kWideWords * kWave] = uint32_t(x);
        }
        static_for<0, kWideLow>([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            words(A - 1 - t, RW[t][0], &RX[t]);
            int32_t x;
            words(2 * A - 1 - t, RW[t][1], &x);
        });
        __syncthreads();
    }
    if constexpr (BR) {
        // the block's rows, a wave filling every fourth one
        const Inst &I = insts[0];
        if (I.wide != 0) return;
        A = I.A;
        ML = to_global(I.ML);
        kbase = I.kslot * kKTable;
        for (int r = bwave; r < block_rows(G); r += WPB) {
            constexpr int plain = kSuperLog - G;
            const int t = r < plain ? G + r : kSuperLog + (r - plain) / 2;
            // M_int's or its negation's
            const int row = (r >= plain && (r - plain) % 2 ? 2 * A : A) - 1 - t;
            if (t >= A) continue;
            const int32_t ml = lrow(row);
            const ivec<MC> mh = hrow(row);
#pragma unroll
            for (int j = 0; j < MC; j++) ldsR[(r * MC + j) * kWave + lane] = ml + mh[j];
        }
        __syncthreads();
    }
    for (uint64_t v = own ? blockIdx.x * WPB + bwave : claim(); v < wc.claims; v = claim()) {
        // items [g, g + 2^run): a run of them for the first wc.runs claims
        const int run = v < wc.runs ? wc.run_log : 0;
        const uint64_t g = v < wc.runs ? v << wc.run_log : v + ((wc.runs << wc.run_log) - wc.runs);
        // instance owning item g: first k with item_end > g
        int lo = 0, hi = LONE ? 0 : n_inst - 1;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (insts[mid].item_end > g) hi = mid;
            else lo = mid + 1;
        }
        // (what only the item set-up and the rare paths use is read from the
        // descriptor where it is used, not held in registers)
        const Inst &I = insts[lo];
        if (lo != cur) {
            cur = lo;
            // a device-prepared instance whose input was refused walks no item
            if (I.prep && sread(I.prep->status) != 0) break;
            ML = to_global(I.ML);
            S = to_global(I.S);
            kbase = I.kslot * kKTable;
            A = I.A;
            static_for<0, WD ? 0 : G>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                const bool have = t < A;
                const int v = have ? A - 1 - t : 0;
                const int32_t ml = lrow(v);
                const ivec<MC> mh = hrow(v);
                if constexpr (LR && (t == 3 || t == 4)) {
                    // each lane writes and later reads only its own columns
#pragma unroll
                    for (int j = 0; j < MC; j++)
                        ldsR[(t - 3) * (MC * kWave) + j * kWave + lane] =
                            have ? ml + mh[j] : 0;
                } else {
#pragma unroll
                    for (int j = 0; j < MC; j++) R[t][j] = have ? ml + mh[j] : 0;
                }
            });
            Smid = S[size_t(A - 1 - kLowLevels) * kWave + ulane];
            static_for<0, kLowLevels>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                SmidL[t] = kall[kbase + kKBound + (A - 1 - kLowLevels) * kLowLevels + t];
            });
            // Sll(t,u): coupling of the low variables A-1-t and A-1-u
            int32_t Sll[kLowLevels][kLowLevels];
            static_for<0, kLowLevels>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                static_for<0, kLowLevels>([&](auto uc) {
                    constexpr int u = decltype(uc)::value;
                    // loads through the descriptor's generic pointers count as
                    // divergent; readfirstlane keeps these constants in SGPRs
                    Sll[t][u] = (t == u) ? 0 : sread(S[(A - 1 - u) * kWave + (A - 1 - t)]);
                });
            });
            CR[0] = 0;
            static_for<1, kPatterns>([&](auto pc) {
                constexpr int p = decltype(pc)::value;
                constexpr int t = cx_ctz(p);
                constexpr int pp = p & (p - 1);
                int32_t acc = 0;
                static_for<0, kLowLevels>([&](auto uc) {
                    constexpr int u = decltype(uc)::value;
                    if constexpr ((pp >> u) & 1) acc += Sll[t][u];
                });
                CR[p] = acc;
            });
            best = kNoEnergy;
            bestRow = ~0ull;
        }

        // Best energy found by any wave for this instance (published at the
        // end of each item), read while the set-up's other loads are in flight.
        int32_t g0 = kNoEnergy;
        if constexpr (BT != 3)
            g0 = __hip_atomic_load(I.gbest, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

        // ---- item set-up: state g(i0) from scratch
        const uint64_t qloc = g - I.item_begin + I.item_local0;   // the instance's item number
        const uint64_t i0 = qloc << I.L;
        const uint64_t sb0 = i0 >> kSuperLog;
        const uint64_t sbEnd = sb0 + (1ull << (I.L + run - kSuperLog));
        const uint64_t row0 = i0 ^ (i0 >> 1);

        // What bounds the set-up is latency: its loads are masked, not branched
        // over, and issued in groups, so that most of them share one L2 round
        // trip (one per set bit of the row had made an n = 33 walk 274 us
        // instead of 248).
        int32_t E[MC];
        {
            const gint32 *EB = to_global(I.EB);
#pragma unroll
            for (int j = 0; j < MC; j++) E[j] = EB[j * kWave + ulane];
        }
        // Chunk vector E_s + x_p M_int: M_int[v][s] sums T[v][A+t] over the set
        // suffix bits t of s, so x_p M_int[s] sums, over the same bits, the
        // suffix fields h_t = sum over the set prefix variables v of
        // T[v][A+t].  Lane 16 q + t adds up the rows v = q (mod 4).
        const gint32 *T = to_global(I.T);
        const int nT = I.n;
        int32_t F = T[min(lane, A - 1) * (nT + 1)];   // T[l][l], lane l < A
        F = lane < A ? F : 0;
        int32_t h = 0;
        for (int v0 = 0; v0 < A; v0 += 32) {
            int32_t x[8];
#pragma unroll
            for (int k = 0; k < 8; k++) {
                const int v = v0 + 4 * k + (lane >> 4);
                // (a lane without a row or a column reads another entry, masked below)
                x[k] = T[min(v, A - 1) * nT + A + min(lane & 15, B - 1)];
            }
#pragma unroll
            for (int k = 0; k < 8; k++) {
                const int v = v0 + 4 * k + (lane >> 4);
                const uint32_t on = uint32_t(row0 >> ((A - 1 - v) & 63)) & uint32_t(v < A);
                h += x[k] & -int32_t(on & 1u);
            }
        }
        h += __shfl_xor(h, 16, kWave);
        h += __shfl_xor(h, 32, kWave);
        {
            uint32_t lsum = 0;   // over the six bits of the lane
            static_for<0, 6>([&](auto uc) {
                constexpr int u = decltype(uc)::value;
                lsum += uint32_t(-((lane >> u) & 1) & __builtin_amdgcn_readlane(h, B - 1 - u));
            });
            uint32_t hsum[MC];   // over the bits of j
            hsum[0] = 0;
            static_for<1, MC>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                hsum[j] = hsum[j & (j - 1)] +
                          uint32_t(__builtin_amdgcn_readlane(h, B - 7 - cx_ctz(j)));
            });
            // packed: both columns of a word, the high one with variable A set
            const uint32_t top = PK ? uint32_t(__builtin_amdgcn_readlane(h, 0)) << 16 : 0u;
            if constexpr (PK) lsum *= 0x10001u;
            static_for<0, MC>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                const uint32_t hj = PK ? hsum[j] * 0x10001u + top : hsum[j];
                E[j] = int32_t(uint32_t(E[j]) + lsum + hj);
            });
        }
        // F: field of every prefix variable from the non-low ones (levels >=
        // kLowLevels, variables 0..A-1-kLowLevels), plus its diagonal; one
        // lane per variable.  Fb: the part from the variables before it, so
        // that the energy E_nl of the non-low prefix bits is the sum of Fb
        // over the set ones (a partial sum of T at every point).
        if constexpr (WD) {
#pragma unroll
            for (int k = 0; k < kWideWords; k++) W[k] = wide_word(E[3 * k], E[3 * k + 1], E[3 * k + 2]);
            X = E[MC - 1];
        }
        int32_t Fb = F;
        for (int w0 = 0; w0 <= A - 1 - kLowLevels; w0 += 16) {
            int32_t c[16];
#pragma unroll
            for (int k = 0; k < 16; k++) c[k] = S[min(w0 + k, A - 1) * kWave + ulane];
#pragma unroll
            for (int k = 0; k < 16; k++) {
                const int w = w0 + k;
                const int32_t on =
                    w <= A - 1 - kLowLevels ? -int32_t((row0 >> ((A - 1 - w) & 63)) & 1) : 0;
                F += c[k] & on;
                Fb += w < lane ? c[k] & on : 0;
            }
        }
        const bool lbit = lane <= A - 1 - kLowLevels && ((row0 >> (A - 1 - lane)) & 1);
        int32_t Enl = wave_sum(lbit ? Fb : 0);
        // the chunk energies carry the instance's shift c (packed: into the
        // 16-bit range; int32: non-negative), the prefix energy the opposite
        // one, so every sum is the true energy
        Enl -= I.pack_shift;
        Enl = sread(Enl);
        int32_t H[kLowLevels];
        static_for<0, kLowLevels>([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            H[t] = __builtin_amdgcn_readlane(F, A - 1 - t);
        });
        if constexpr (BT == 3) {
            best = tk_threshold();
        } else {
            // A chunk can improve the final answer only if its key is at most
            // the shared best.  (A chunk tying it with an unknown row is still
            // recorded: bestRow restarts at the largest row whenever the
            // shared value lowers best.)
            g0 = sread(g0);
            if (g0 < best) {
                best = g0;
                bestRow = ~0ull;
            }
        }

        // TIER 1: THR[p] = best - E_p(low pattern p): the chunk holds a
        // candidate when its minimum E_sd is <= THR of the current pattern.
        int32_t THR[kPatterns];
        auto build_thr = [&]() {
            THR[0] = best - Enl;
            static_for<1, kPatterns>([&](auto pc) {
                constexpr int p = decltype(pc)::value;
                constexpr int t = cx_ctz(p);
                constexpr int pp = p & (p - 1);
                THR[p] = THR[pp] - H[t] - CR[p];
            });
        };
        if constexpr (TIER == 1) build_thr();

        // A non-low prefix variable w flips (direction up: 0 -> 1); SLw[t] is
        // its coupling with the low variable A-1-t; Sd is its coupling
        // column with the sign of the flip applied.
        auto nonlow_flip = [&](int w, bool up, int32_t Sd, const int32_t *SLw) {
            const int32_t Fw = __builtin_amdgcn_readlane(F, w);
            Enl = up ? Enl + Fw : Enl - Fw;
            F += Sd;
            static_for<0, kLowLevels>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                H[t] = up ? H[t] + SLw[t] : H[t] - SLw[t];
            });
        };

        int32_t itemE = kNoEnergy;
        uint64_t itemRow = 0;
        int found = 0;
        int32_t W0 = 0;    // TIER 2: exact wave minimum at the super-block start
                           // (taken on the cold path only)
        int32_t lm0 = 0;   // TIER 2: this lane's chunk minimum at the super-block start
        int tab2 = 0;      // TIER 2: K table of the current segment (0 before the middle
                           // flip, 1 / 2 after it with level 5 rising / falling)

        // Candidate test at Gray step i with chunk minimum lm and threshold thr.
        auto candidate = [&](int32_t lm, int32_t thr, uint64_t i) {
            if (__builtin_amdgcn_ballot_w64(lm <= thr)) {
                const int32_t wmin = wave_min(lm);
                const int32_t Ec = wmin + (best - thr);   // + E_p
                const uint64_t rc = i ^ (i >> 1);
                if (Ec < best || (Ec == best && rc < bestRow)) {
                    const int32_t d = Ec - best;
                    best = Ec;
                    bestRow = rc;
                    itemE = Ec;
                    itemRow = rc;
                    found = 1;
                    if constexpr (TIER == 1) {
                        static_for<0, kPatterns>([&](auto pc) { THR[decltype(pc)::value] += d; });
                    }
                }
            }
        };

        // TIER 3 candidate: a chunk key (E_p + chunk minimum, row) at or below
        // the threshold waits in the wave's queue; the super-block's end enters
        // the queue into the wave's list and lowers the threshold.
        int nq = 0;
        auto candidate3 = [&](int32_t lm, int32_t thr, uint64_t i) {
            if (__builtin_amdgcn_ballot_w64(lm <= thr)) {
                const int32_t Ec = wave_min(lm) + (best - thr);
                if (lane == 0) {
                    tk_queueE()[nq] = Ec;
                    tk_queueR()[nq] = i ^ (i >> 1);
                }
                nq++;
            }
        };
        auto test = [&](int32_t lm, int32_t thr, uint64_t i) {
            if constexpr (BT == 3) candidate3(lm, thr, i);
            else candidate(lm, thr, i);
        };

        // Low flip of static level t (< kLowLevels) with static direction (Alg. 2:
        // E_sd += delta M_int[k]).
        auto low_flip = [&](auto tc, auto upc) {
            constexpr int t = decltype(tc)::value;
            constexpr bool up = decltype(upc)::value;
            if constexpr (WD) {
                if constexpr (t < kWideLow) {
#pragma unroll
                    for (int k = 0; k < kWideWords; k++) W[k] += RW[t][up ? 0 : 1][k];
                    X = up ? X + RX[t] : X - RX[t];
                } else {
                    add_wide(2 * (t - kWideLow) + (up ? 0 : 1));
                }
                pin_wide();
            } else if constexpr (LR && (t == 3 || t == 4)) {
#pragma unroll
                for (int j = 0; j < MC; j++) {
                    const int32_t r = ldsR[(t - 3) * (MC * kWave) + j * kWave + lane];
                    E[j] = up ? E[j] + r : E[j] - r;
                }
            } else if constexpr (BR && t >= G) {
#pragma unroll
                for (int j = 0; j < MC; j++) {
                    const int32_t r = ldsR[((t - G) * MC + j) * kWave + lane];
                    E[j] = up ? E[j] + r : E[j] - r;
                }
            } else {
#pragma unroll
                for (int j = 0; j < MC; j++) E[j] = up ? E[j] + R[t][j] : E[j] - R[t][j];
            }
            if constexpr (!WD) pin_vec<MC>(E);
        };
        // Flip of level kLowLevels in the middle of super-block sb (its
        // direction alternates between super-blocks).
        auto middle_flip = [&](uint64_t sb) {
            const bool up = (sb & 1) == 0;
            constexpr int tm = kLowLevels;
            if constexpr (WD) {
                add_wide(2 * (tm - kWideLow) + (up ? 0 : 1));
                pin_wide();
            } else if constexpr (BR) {
                int32_t r[MC];
#pragma unroll
                for (int j = 0; j < MC; j++) r[j] = ldsR[((tm - G) * MC + j) * kWave + lane];
                if (up) {
#pragma unroll
                    for (int j = 0; j < MC; j++) E[j] += r[j];
                } else {
#pragma unroll
                    for (int j = 0; j < MC; j++) E[j] -= r[j];
                }
            } else if constexpr (G > tm) {
                if (up) {
#pragma unroll
                    for (int j = 0; j < MC; j++) E[j] += R[tm][j];
                } else {
#pragma unroll
                    for (int j = 0; j < MC; j++) E[j] -= R[tm][j];
                }
            } else {
                const int ws = up ? A - 1 - tm : 2 * A - 1 - tm;
                const int32_t ml = lrow(ws);
                const ivec<MC> mh = hrow(ws);
#pragma unroll
                for (int j = 0; j < MC; j++) E[j] += ml + mh[j];
            }
            pin_vec<MC>(E);
            nonlow_flip(A - 1 - tm, up, up ? Smid : -Smid, SmidL);
            return up;
        };
        // Flip entering super-block sb + 1 (Gray level >= kSuperLog): its
        // signed row (M_int's or the negated one: one code path whatever the
        // direction) is `row`, and the lane part and coupling column of that
        // row are loaded a super-block ahead, which hides their latency (two
        // VGPRs; n = 44 walk 0.7% and n = 36 3% shorter than loading them
        // at the flip).
        struct Boundary {
            int w;
            bool up;
            int row;
            int32_t ml, sd;
        };
        auto boundary_load = [&](uint64_t sb) {
            Boundary b;
            const uint64_t ip1 = (sb + 1) << kSuperLog;
            const int t = __builtin_ctzll(ip1);
            b.up = ((ip1 >> (t + 1)) & 1) == 0;
            // (past the last super-block t can be A: any row will do there)
            b.w = max(A - 1 - t, 0);
            b.row = b.up ? b.w : b.w + A;
            b.ml = LONE ? 0 : lrow(b.row);
            b.sd = S[b.row * kWave + ulane];
            return b;
        };
        auto boundary_flip = [&](const Boundary &b) {
            bool done = false;
            static_for<kSuperLog, G>([&](auto tc) {
                constexpr int tt = decltype(tc)::value;
                if (b.w == A - 1 - tt) {
                    if (b.up) {
#pragma unroll
                        for (int j = 0; j < MC; j++) E[j] += R[tt][j];
                    } else {
#pragma unroll
                        for (int j = 0; j < MC; j++) E[j] -= R[tt][j];
                    }
                    done = true;
                }
            });
            if constexpr (WD) {
                const int t = A - 1 - b.w;
                if (__builtin_expect(t <= kWideTop, 1)) add_wide(2 * (t - kWideLow) + (b.up ? 0 : 1));
                if (t > kWideTop) {
                    const int32_t ml = lrow(b.row);
                    const ivec<MC> mh = hrow(b.row);
#pragma unroll
                    for (int k = 0; k < kWideWords; k++)
                        W[k] += wide_word(ml + mh[3 * k], ml + mh[3 * k + 1], ml + mh[3 * k + 2]);
                    X += ml + mh[MC - 1];
                }
                pin_wide();
            } else if constexpr (BR) {
                const int t = A - 1 - b.w;
                if (__builtin_expect(t <= kBlockTop, 1)) {
                    const int r0 = kSuperLog - G + 2 * (t - kSuperLog) + (b.up ? 0 : 1);
#pragma unroll
                    for (int j = 0; j < MC; j++) E[j] += ldsR[(r0 * MC + j) * kWave + lane];
                }
                // (an if of its own: as the other branch's else the chunk vector is
                // copied, 16 moves, where the two meet)
                if (t > kBlockTop) {
                    const int32_t ml = lrow(b.row);
                    const ivec<MC> mh = hrow(b.row);
#pragma unroll
                    for (int j = 0; j < MC; j++) E[j] += ml + mh[j];
                }
            } else if (!done) {
                const ivec<MC> mh = hrow(b.row);
#pragma unroll
                for (int j = 0; j < MC; j++) E[j] += b.ml + mh[j];
            }
            pin_vec<MC>(E);
            int32_t SLw[kLowLevels];
            static_for<0, kLowLevels>([&](auto tc) {
                constexpr int tt = decltype(tc)::value;
                SLw[tt] = kall[kbase + kKBound + b.w * kLowLevels + tt];
            });
            nonlow_flip(b.w, b.up, b.sd, SLw);
        };

        if constexpr (TIER == 1) {
            for (uint64_t sb = sb0; sb < sbEnd; sb++) {
                const Boundary next = boundary_load(sb);
                static_for<0, (1 << kSuperLog)>([&](auto oc) {
                    constexpr int o = decltype(oc)::value;
                    constexpr int pat = (o ^ (o >> 1)) & (kPatterns - 1);
                    candidate(tree_min<MC>(E), THR[pat], (sb << kSuperLog) | uint64_t(o));
                    if constexpr (o < (1 << kSuperLog) - 1) {
                        constexpr int t = cx_ctz(o + 1);
                        if constexpr (t < kLowLevels) {
                            constexpr bool up = ((((o + 1) ^ ((o + 1) >> 1)) >> t) & 1) != 0;
                            low_flip(std::integral_constant<int, t>{}, std::integral_constant<bool, up>{});
                        } else {
                            middle_flip(sb);
                            build_thr();
                        }
                    } else if (sb + 1 < sbEnd) {
                        boundary_flip(next);
                        build_thr();
                    }
                });
            }
        } else {
            // 32-bit trip count: a 64-bit compare would take the vector unit
            const uint32_t nsb = uint32_t(sbEnd - sb0);
            Boundary next = boundary_load(sb0);
            for (uint32_t ks = 0; ks < nsb; ks++) {
                const uint64_t sb = sb0 + ks;
                if (ks) {
                    boundary_flip(next);
                    next = boundary_load(sb);
                }
                lm0 = lane_min(E);
                tab2 = 0;
                // NSEG segments of SEG steps (tier 2: the two halves around
                // the level-5 flip), each with (cold) or without the per-step
                // bound tests; every step's chunk energies stay observable
                // through the (rarely taken) test, so each state gets its add
                static_for<0, NSEG>([&](auto sc) {
                    constexpr int h = decltype(sc)::value;
                    // the low flip after step o (none after the segment's last)
                    auto step_flip = [&](auto oc) {
                        constexpr int o2 = decltype(oc)::value;
                        constexpr int o = h * SEG + o2;
                        if constexpr (o2 < SEG - 1) {
                            constexpr int t = cx_ctz(o + 1);
                            constexpr bool up = ((((o + 1) ^ ((o + 1) >> 1)) >> t) & 1) != 0;
                            low_flip(std::integral_constant<int, t>{},
                                     std::integral_constant<bool, up>{});
                        }
                    };
                    // One scalar test for the segment: an upper bound of its SEG
                    // thresholds tp(o) = best - Enl - hs(o) - C2(o), since
                    // hs(o) >= sum_t min(0, H[t]) and C2(o) >= the segment's
                    // minimum of C2; any lane at or below it takes the cold
                    // path (the wave minimum W0 is formed only then)
                    int32_t tb = best - Enl - kall[kbase + kKC2Min + tab2];
                    static_for<0, kLowLevels>([&](auto tc) { tb -= min(0, H[decltype(tc)::value]); });
                    const bool cold = __builtin_amdgcn_ballot_w64(lm0 <= tb) != 0;
                    if (__builtin_expect(cold, 0)) {
                        // Exact tests, step by step: at offset o,
                        //   tp(o) = best - E_p(low pattern at o) - C2(o)
                        // (K table tab2), with hs = the sum of H[t] over the
                        // set low bits walked along the Gray sequence of
                        // patterns g(o) & 31 and best read afresh at every
                        // step (a candidate found earlier in the segment has
                        // lowered it).  Step o can hold a candidate only if
                        // W0 <= tp(o), and then holds one exactly when the
                        // chunk minimum is <= tp(o) + D(o) = best - E_p(o).
                        W0 = wave_min_bcast(lm0);
                        constexpr int o0 = h * SEG;
                        constexpr int p0 = (o0 ^ (o0 >> 1)) & (kPatterns - 1);
                        int32_t hs = 0;
                        static_for<0, kLowLevels>([&](auto tc) {
                            constexpr int t = decltype(tc)::value;
                            if constexpr ((p0 >> t) & 1) hs += H[t];
                        });
                        static_for<0, SEG>([&](auto oc) {
                            constexpr int o2 = decltype(oc)::value;
                            constexpr int o = o0 + o2;
                            if constexpr (o2 > 0) {
                                constexpr int pa0 = ((o - 1) ^ ((o - 1) >> 1)) & (kPatterns - 1);
                                constexpr int pa1 = (o ^ (o >> 1)) & (kPatterns - 1);
                                constexpr int t = cx_ctz(pa0 ^ pa1);
                                if constexpr (((pa1 >> t) & 1) != 0) hs += H[t];
                                else hs -= H[t];
                            }
                            const int32_t tp = (best - Enl) - hs -
                                               kall[kbase + tab2 * kPatterns + (o & (kPatterns - 1))];
                            if (W0 <= tp) {
                                const int32_t thr =
                                    tp + kall[kbase + (3 + tab2) * kPatterns + (o & (kPatterns - 1))];
                                test(lane_min(E), thr, (sb << kSuperLog) | uint64_t(o));
                            }
                            step_flip(oc);
                        });
                    } else {
                        static_for<0, SEG>([&](auto oc) { step_flip(oc); });
                    }
                    // the flip after the segment's last step: level 5 in the
                    // middle, a low level (static direction) between shorter
                    // segments, the boundary flip after the last
                    if constexpr (h == NSEG / 2 - 1) {
                        tab2 = middle_flip(sb) ? 1 : 2;
                    } else if constexpr (h < NSEG - 1) {
                        constexpr int o = (h + 1) * SEG;
                        constexpr int t = cx_ctz(o);
                        constexpr bool up = (((o ^ (o >> 1)) >> t) & 1) != 0;
                        low_flip(std::integral_constant<int, t>{}, std::integral_constant<bool, up>{});
                    }
                });
                if constexpr (BT == 3) {
                    if (__builtin_expect(nq != 0, 0)) {
                        best = sread(tk_drain(nq));
                        nq = 0;
                    }
                }
            }
        }

        if (BT != 3 && found && lane == 0) {
            // Only items that found a candidate leave a record, marked in the
            // instance's bitmap (the record and bitmap pointers are read from
            // the descriptor here, on this rare path, rather than held in
            // registers through the walk).
            ItemRes r;
            r.E = itemE;
            r.found = 1;
            r.row = itemRow;
            const uint64_t q = g - insts[cur].item_begin;
            insts[cur].res[q] = r;
            const uint64_t b = insts[cur].bit0 + q;
            atomicOr(insts[cur].bits + (b >> 5), 1u << (b & 31));
            // publish once per item: every wave starting an item of this
            // instance at once would otherwise contend on one address
            atomicMin(insts[cur].gbest, itemE);
        }
    }
    if constexpr (BT == 3) tk_flush();
}

template <int MC, int G, int TIER, int RC = kRowsVgpr>
__global__ __launch_bounds__(kWave *walk_block_waves<RC>(),
                             (walk_waves_per_simd<MC, G, RC>())) void walk_kernel(
    const Inst *__restrict__ insts, int n_inst, WalkClaims wc,
    unsigned long long *__restrict__ counter, const int32_t *__restrict__ kall, TopkWalk tk)
{
    walk_items<MC, G, TIER, RC>(insts, n_inst, wc, counter, kall, tk, true);
}

// The instances of tier 2 and then those of tier 4 in one launch: a wave that
// finds the first queues empty goes on to the second ones, so that the tail of
// the one (the time of an item, four waves to a SIMD) is filled by the other.
// 64 requests of n = 16..34, 13 of them float32, submitted at once: 1961 -> 1905 us.
// The two walks share one register allocation, and spill what they do alone (17
// VGPRs and 7 SGPRs each) side by side: 35 and 30.
template <int MC, int G, int RC>
__global__ __launch_bounds__(kWave, (walk_waves_per_simd<MC, G, RC>())) void walk_pair_kernel(
    const Inst *__restrict__ insts2, int n2, WalkClaims wc2, unsigned long long *__restrict__ counter2,
    const Inst *__restrict__ insts4, int n4, WalkClaims wc4, unsigned long long *__restrict__ counter4,
    const int32_t *__restrict__ kall)
{
    const TopkWalk none{};
    walk_items<MC, G, 2, RC>(insts2, n2, wc2, counter2, kall, none, true);
    walk_items<MC, G, 4, RC>(insts4, n4, wc4, counter4, kall, none, false);
}

template <int MC, int G, int RC>
static size_t walk_lds_bytes(int tier)
{
    return lds_rows_offset(tier, walk_block_waves<RC>()) + lds_rows_bytes<MC, G, RC>();
}

template <int MC, int G, int TIER, int RC>
static hipError_t launch_walk_tier(const WalkLaunch &w, const TopkWalk &tk)
{
    constexpr int WPB = walk_block_waves<RC>();
    hipLaunchKernelGGL((walk_kernel<MC, G, TIER, RC>), dim3((w.waves + WPB - 1) / WPB),
                       dim3(kWave * WPB), (walk_lds_bytes<MC, G, RC>(TIER)), w.stream, w.insts,
                       w.n_inst, w.claims, w.counter, w.k, tk);
    return hipGetLastError();
}

template <int MC, int G, int RC = kRowsVgpr>
static hipError_t launch_walk_g(const WalkLaunch &w)
{
    const TopkWalk none{};
    if constexpr (RC == kRowsBlock) {
        if (w.n_inst != 1) return hipErrorInvalidValue;
        if (w.tier == 2) return launch_walk_tier<MC, G, 2, RC>(w, none);
        if (w.tier == 4) return launch_walk_tier<MC, G, 4, RC>(w, none);
        if (!w.tk || w.tk->k < 2) return hipErrorInvalidValue;
        if (w.tier == 3) return launch_walk_tier<MC, kBlockLowTopk, 3, RC>(w, *w.tk);
        if (w.tier == 5) return launch_walk_tier<MC, kBlockLowTopk, 5, RC>(w, *w.tk);
    } else if constexpr (RC == kRowsWave && G == 6) {
        // (its top-k form would be a lone walk, over the block's rows)
        if (w.tier == 1) return launch_walk_tier<MC, G, 1, RC>(w, none);
        if (w.tier == 2) return launch_walk_tier<MC, G, 2, RC>(w, none);
        if (w.tier == 4) return launch_walk_tier<MC, G, 4, RC>(w, none);
    } else {
        if (w.tier == 1) return launch_walk_tier<MC, G, 1, RC>(w, none);
        if (w.tier == 2) return launch_walk_tier<MC, G, 2, RC>(w, none);
        if constexpr (MC >= 4)
            if (w.tier == 4) return launch_walk_tier<MC, G, 4, RC>(w, none);
        if (!w.tk || w.tk->k < 2 || w.n_inst != 1) return hipErrorInvalidValue;
        if (w.tier == 3) return launch_walk_tier<MC, G, 3, RC>(w, *w.tk);
        if constexpr (MC >= 4)
            if (w.tier == 5) return launch_walk_tier<MC, G, 5, RC>(w, *w.tk);
    }
    return hipErrorInvalidValue;
}

// Resident waves per CU (>= 1).
template <int MC, int G, int TIER, int RC>
static int occupancy_tier()
{
    constexpr int WPB = walk_block_waves<RC>();
    int blocks = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &blocks, walk_kernel<MC, G, TIER, RC>, kWave * WPB, walk_lds_bytes<MC, G, RC>(TIER));
    return e != hipSuccess || blocks < 1 ? 1 : blocks * WPB;
}

template <int MC, int G, int RC = kRowsVgpr>
static int occupancy_g(int tier)
{
    constexpr bool topk = RC != kRowsWave || G != 6;
    if constexpr (topk)
        if (tier == 3) return occupancy_tier<MC, G, 3, RC>();
    if (tier == 2) return occupancy_tier<MC, G, 2, RC>();
    if constexpr (MC >= 4) {
        if (tier == 4) return occupancy_tier<MC, G, 4, RC>();
        if constexpr (topk)
            if (tier == 5) return occupancy_tier<MC, G, 5, RC>();
    }
    return occupancy_tier<MC, G, 1, RC>();
}

}  // namespace qk
