// kernels.hip -- gfx950 kernels of the exhaustive dense-QUBO solver: the
// table build, the finish and the walk dispatch (the walk kernel itself is in
// walk.h, its variants in walk_*.hip).
//
// Method (paper Sec. II-III): split every state x = [x_p | x_s] into an
// A-bit prefix and a B-bit suffix.  For a fixed prefix the energies of all
// 2^B states of its chunk are (Sec. II-C, Eq. chunk_energy_final)
//     E(C_xp) = E_p(x_p) 1 + x_p M_int + E_s(U_B),   M_int = Q_ps U_B^T.
// Walking the prefixes in reflected Gray order (Sec. III-B) changes x_p by one
// bit k per step, so the suffix-dependent vector E_sd = x_p M_int + E_s moves
// by +-M_int[k] (Eq. incremental_update): one int32 add per state.
//
// MI355X mapping:
//  * one wavefront owns all 2^B columns of its chunk: lane l holds columns
//    s = j*64 + l (j < MC), i.e. E_sd lives in MC VGPRs per lane (column-wise
//    split, Sec. III-C.2, at lane granularity);
//  * the rows M_int[k] of the most frequently flipped Gray levels stay on
//    chip: by default levels 0-2 and 5 in VGPRs and 3-4 in LDS (8 KB per
//    wave), or, walking one instance alone, 0-3 in VGPRs and 4-8 in LDS (32 KB
//    per block of four waves), which fits 128 VGPRs and so four waves per
//    SIMD; other variants keep 5, 6, 8 or 12 levels in VGPRs; a lone instance
//    whose energies allow it walks three columns to a 64-bit word (kWideBits);
//    higher levels are formed when they
//    flip (level 6 once per 128 steps; level 5, in the 5-level variants, once
//    per 64) from the row's two parts: column j*64 + lane of a row is a sum
//    over the lane's bits plus a sum over the bits of j, so a row is one load
//    per lane, 2^B / 64 scalars and a three-operand add per word;
//  * wavefronts take work items (2^L consecutive Gray steps of the prefix,
//    the "straightforward" split of Sec. III-C.1 along the Gray index), the
//    first by its own number and the others from eight atomic counters, singly
//    or in runs (WalkClaims); the grid is persistent;
//  * the scalar unit keeps the prefix self-energy E_p: the walk is unrolled
//    over 64-step super-blocks in which the five lowest Gray levels follow a
//    static pattern and level 5 flips once, in the middle, so the flip
//    sequence is known at compile time and E_p of each low pattern follows
//    from SGPR fields refreshed only when a higher prefix bit flips;
//  * the candidate test "min over the chunk + E_p <= best" is, by default
//    (tier 2), a lower bound from one DPP wave minimum per super-block and a
//    per-offset table, tested against a cheap upper bound of the thresholds
//    once per 32 steps; exact per-step tests run only when that passes (tier
//    1 does the exact v_min3 test at every step).  Each step still updates
//    the chunk vector once (pinned, so the compiler cannot fold flips).  Ties
//    resolve to the lowest prefix row here and to the lowest suffix in the
//    final rescan, giving the lowest U_N index overall.
#include "kcommon.h"
#include "walk_variants.h"

namespace qk {

// ---------------------------------------------------------------- tables

// Greedy single-flip descents, one per wave (from the all-zero state for wave
// 0, from hashed states otherwise); the block's least energy becomes the
// instance's shared best.  Any
// state's energy is a valid threshold for the walk (the state's own chunk
// still passes it), and a local minimum of a dense QUBO is usually close to
// the global one, so walk waves start with a near-final threshold.
__device__ int32_t seed_best(const int32_t *S, int n, int wave)
{
    int32_t E;
    uint64_t xm;
    greedy_descent(S, n, uint32_t(wave), E, xm);
    return E;
}

// The upper triangle of T (n x n) as a symmetric matrix in LDS, by the whole
// block.  bus: T is a host image, read over the bus in 16-byte words (its
// region is 256-byte aligned; n = 36 build 22 -> 13 us); one entry a lane is
// faster from device memory, where the wide form's strided LDS writes weigh
// more (100 builds 12 us against 21).
__device__ void stage_symmetric(const int32_t *T, int n, int32_t *S, int tid, int threads, bool bus)
{
    const int nn = n * n;
    if (!bus) {
        for (int e = tid; e < nn; e += threads) {
            const int i = e / n, j = e % n;
            if (i > j) continue;
            const int32_t t = T[e];
            S[e] = t;
            S[j * n + i] = t;
        }
        return;
    }
    for (int e0 = 4 * tid; e0 < nn; e0 += 4 * threads) {
        int32_t t[4] = {0, 0, 0, 0};
        if (e0 + 4 <= nn) {
            *reinterpret_cast<int4 *>(t) = *reinterpret_cast<const int4 *>(T + e0);
        } else {
            for (int x = 0; x < nn - e0; x++) t[x] = T[e0 + x];
        }
        int i = e0 / n, j = e0 - i * n;
#pragma unroll
        for (int x = 0; x < 4; x++) {
            if (e0 + x < nn && i <= j) {
                S[i * n + j] = t[x];
                S[j * n + i] = t[x];
            }
            if (++j == n) {
                j = 0;
                i++;
            }
        }
    }
}

// The first kernel of a lone solve copies its host image (see Upload).
__device__ void upload(const Upload &up, int tid, int threads)
{
    const uint4 *src = reinterpret_cast<const uint4 *>(up.src);
    uint4 *dst = reinterpret_cast<uint4 *>(up.dst);
    for (uint32_t x = uint32_t(tid); x < up.copy_bytes / 16; x += uint32_t(threads)) dst[x] = src[x];
    uint4 *z = reinterpret_cast<uint4 *>(up.dst + up.zero_from);
    for (uint32_t x = uint32_t(tid); x < up.zero_bytes / 16; x += uint32_t(threads))
        z[x] = uint4{0, 0, 0, 0};
}

__global__ __launch_bounds__(256) void upload_kernel(Upload up)
{
    upload(up, int(blockIdx.x * blockDim.x + threadIdx.x), int(gridDim.x * blockDim.x));
}

// One block per (instance, part of its tables), blockIdx.x naming the part.
// Every part stages T in LDS first, as the symmetric matrix: everything below
// is sums of a few entries, so what bounds the build is latency, and no part
// waits for another.  M_int is never formed: its lane and column parts (ML,
// MH) are, and the bound constants have closed forms over the suffix bits.
// Measured: a lone build 9-16 us and 4096 batch instances 157 us; 60-92 us and
// 950 us when 8 blocks per instance wrote the whole M_int (2A x 2^B words) and
// reduced the bound constants over its columns.
enum { kPartSeed = 0, kPartK, kPartEB, kPartRows, kTableParts, kPartUpload = kTableParts };
constexpr int kTableThreads = 512;   // eight descents at once

__global__ __launch_bounds__(kTableThreads) void tables_kernel(
    const Inst *__restrict__ insts, unsigned long long *__restrict__ counters, int n_groups,
    Upload up, const Upload *__restrict__ ups)
{
    if (ups) up = ups[blockIdx.y];
    __shared__ int32_t sS[kMaxVars * kMaxVars];   // T made symmetric
    __shared__ int32_t sSeed;
    const int part = int(blockIdx.x);
    const int tid = int(threadIdx.x);
    if (part == kPartUpload) {
        upload(up, tid, kTableThreads);
        return;
    }
    const Inst I = up.src ? *reinterpret_cast<const Inst *>(up.src) : insts[blockIdx.y];
    const int32_t *T = up.src ? reinterpret_cast<const int32_t *>(
                                    reinterpret_cast<const unsigned char *>(I.T) - up.dst + up.src)
                              : I.T;
    if (part == kPartSeed && blockIdx.y == 0) {
        for (int c = tid; c < n_groups * kCounterWords; c += kTableThreads) counters[c] = 0;
    }
    if (part == kPartRows && I.bits) {   // no item has reported yet
        const uint64_t words = (I.n_items + 31) / 32;
        for (uint64_t w = uint64_t(tid); w < words; w += kTableThreads) I.bits[w] = 0u;
    }
    if (I.direct) return;
    const int n = I.n, A = I.A, B = I.B;
    stage_symmetric(T, n, sS, tid, kTableThreads, up.src != nullptr);
    if (tid == 0) sSeed = kNoEnergy;
    __syncthreads();
    const int MC = 1 << (I.packed ? B - 7 : B - 6);   // words per lane
    // Packed words: a part x shared by both columns is x in each half, and
    // the high column (c + 2^(B-1)) also has suffix variable A set.
    auto both = [&](int32_t x) { return I.packed ? uint32_t(x) * 0x10001u : uint32_t(x); };

    if (part == kPartSeed) {
        // (only when the walk covers every state: a restricted item range must
        // not start from an energy found outside it)
        if (I.item_local0 == 0 && I.n_items == (uint64_t(1) << (A - I.L))) {
            const int32_t E = seed_best(sS, n, tid / kWave);
            if (tid % kWave == 0) atomicMin(&sSeed, E);
        }
        __syncthreads();
        if (tid == 0) {
            *I.gbest = sSeed;
            if (n_groups > 0 && blockIdx.y == 0) counters[kClockWord] = wall_clock64();
        }
    } else if (part == kPartRows) {
        for (int e = tid; e < A * kWave; e += kTableThreads) {
            const int v = e / kWave, l = e % kWave;
            // the six lowest suffix bits of column j*64 + l are those of l:
            // bit u is suffix variable n-1-u
            int32_t m = 0;
#pragma unroll
            for (int u = 0; u < 6; u++) m += -((l >> u) & 1) & sS[v * n + n - 1 - u];
            const uint32_t w = both(m);
            I.ML[e] = int32_t(w);
            I.ML[A * kWave + e] = int32_t(0u - w);
            // prefix couplings, one lane per variable
            const int32_t c = (l < A && l != v) ? sS[v * n + l] : 0;
            I.S[e] = c;
            I.S[A * kWave + e] = -c;
        }
    } else if (part == kPartEB) {
        // E_s(U_B)[s] = sum_{t <= u, both set} T[A+t][A+u] (Sec. III-A, step
        // 2), s = (tid mod 256) + 256 hp: the low eight bits' energy and their
        // fields on the (at most three) high variables once per thread, then
        // one sum per high pattern hp.  Bit b of s is variable n-1-b.
        int32_t base = 0, h[3] = {0, 0, 0}, hh[3][3];
#pragma unroll
        for (int b = 0; b < 8; b++) {
            const int32_t mb = -((tid >> b) & 1);
            int32_t row = sS[(n - 1 - b) * n + n - 1 - b];
#pragma unroll
            for (int c = 0; c < b; c++) row += -((tid >> c) & 1) & sS[(n - 1 - b) * n + n - 1 - c];
            base += mb & row;
        }
#pragma unroll
        for (int x = 0; x < 3; x++) {
            const int r = n - 1 - (8 + x);   // n > 14: a row of T either way
            h[x] = sS[r * n + r];
#pragma unroll
            for (int b = 0; b < 8; b++) h[x] += -((tid >> b) & 1) & sS[r * n + n - 1 - b];
#pragma unroll
            for (int y = 0; y < x; y++) hh[x][y] = sS[r * n + n - 1 - (8 + y)];
        }
        auto esuf = [&](int hp) {
            int32_t e = base;
#pragma unroll
            for (int x = 0; x < 3; x++) {
                if (!((hp >> x) & 1)) continue;
                e += h[x];
#pragma unroll
                for (int y = 0; y < x; y++)
                    if ((hp >> y) & 1) e += hh[x][y];
            }
            return e;
        };
        const int NW = MC * kWave;
        for (int c = tid; c < NW; c += kTableThreads) {
            const int hp = c >> 8;
            if (I.packed) {
                const int32_t b = I.pack_shift + kPackBias;
                I.EB[c] = int32_t(uint32_t(esuf(hp) + b) +
                                  (uint32_t(esuf(hp + (1 << (B - 9))) + b) << 16));
            } else {
                I.EB[c] = esuf(hp) + I.pack_shift;
            }
        }
    } else {
        for (int e = tid; e < A * kLowLevels; e += kTableThreads) {
            const int w = e / kLowLevels, l = A - 1 - e % kLowLevels;
            I.K[kKBound + e] = l != w ? sS[w * n + l] : 0;
        }
        // column parts of M_int: bit u of j is suffix variable n-7-u
        for (int e = tid; e < A * MC; e += kTableThreads) {
            const int v = e / MC, j = e % MC;
            int32_t m = 0;
            for (int u = 0; (MC >> u) > 1; u++) m += -((j >> u) & 1) & sS[v * n + n - 7 - u];
            uint32_t w = both(m);
            if (I.packed) w += uint32_t(sS[v * n + A]) << 16;
            I.K[kKHigh + e] = int32_t(w);
            I.K[kKHigh + A * MC + e] = int32_t(0u - w);
        }
        // Tier-2 bound constants.  Inside a 64-step super-block the five lowest
        // Gray levels follow the static pattern p(o) = g(o) & 31 from 0, and the
        // level-5 bit moves once (by cm = +-1) at o = 32, so
        //   E_sd(o) - E_sd(0) = sum_{t<5} p_t(o) M[A-1-t] + [o >= 32] cm M[A-6].
        // D = its minimum over all 2^B columns, a lower bound of how far the
        // chunk minimum can fall from its value at the super-block start.  In
        // column s the difference is the sum over the set suffix bits u of
        //   c_u = sum_{t<5} p_t(o) T[A-1-t][A+u] + [o >= 32] cm T[A-6][A+u],
        // so its minimum over the columns is sum_u min(0, c_u).
        constexpr int NQ = 3 * kPatterns;
        __shared__ int32_t c2s[NQ];
        if (tid < NQ) {
            const int q = tid, tab = q / kPatterns, oo = q % kPatterns;
            const int cm = tab == 0 ? 0 : (tab == 1 ? 1 : -1);
            const int o = tab == 0 ? oo : kPatterns + oo;
            const int pat = (o ^ (o >> 1)) & (kPatterns - 1);
            int32_t d = 0;
            for (int u = A; u < n; u++) {
                int32_t c = cm * sS[(A - 1 - kLowLevels) * n + u];
#pragma unroll
                for (int t = 0; t < kLowLevels; t++) c += -((pat >> t) & 1) & sS[(A - 1 - t) * n + u];
                d += min(0, c);
            }
            int32_t elow = 0;   // couplings among the set low variables
#pragma unroll
            for (int t = 0; t < kLowLevels; t++)
#pragma unroll
                for (int u = t + 1; u < kLowLevels; u++)
                    elow += -((pat >> t) & (pat >> u) & 1) & sS[(A - 1 - u) * n + (A - 1 - t)];
            I.K[(3 + tab) * kPatterns + oo] = d;
            I.K[tab * kPatterns + oo] = elow + d;
            c2s[q] = elow + d;
        }
        __syncthreads();
        if (tid < 3) {   // min of C2 over each bound-test segment
            int32_t m = INT32_MAX;
            for (int oo = 0; oo < kPatterns; oo++) m = min(m, c2s[tid * kPatterns + oo]);
            I.K[kKC2Min + tid] = m;
        }
    }
}

// ---------------------------------------------------------------- prepare

// Canonicalisation of a lone instance held in device memory, with the host
// planner's arithmetic: fold T_ii = Q_ii, T_ij = Q_ij + Q_ji (i < j; the
// energy sums over all pairs); int32 input: sum |T| <= 2^30 - 1 proves every
// partial sum the walk forms exact in int32; float32 input: all entries
// finite, S = sum |T| in float64 accumulated i ascending then j ascending
// (the host's order, so the same S), p = the largest exponent with
// S 2^p <= 2^29, T~ = round-half-even(T 2^p).
// One block.  What bounds it is latency, so nothing of size n^2 runs on one
// thread: S's exponent comes from a parallel sum unless that is within its
// rounding of a power of two (then one thread adds in the host's order), and
// the least chunk energy from the column parts of M_int (as in the table
// build).  Measured: n = 27 float32 37 -> 11 us, n = 44 28 -> 12 us.
constexpr int kPrepThreads = 1024;
constexpr int kPrepWaves = kPrepThreads / kWave;

__device__ __forceinline__ int prep_scale_exponent(double S)
{
    // S = m 2^e, m in [0.5, 1): m 2^(e+p) <= 2^29 for e + p <= 29, and for
    // e + p = 30 exactly when m = 0.5
    if (!(S > 0.0)) return 0;
    int e = 0;
    const double m = frexp(S, &e);
    return (m == 0.5 ? 30 : 29) - e;
}

__global__ __launch_bounds__(kPrepThreads) void prepare_kernel(const void *__restrict__ dQ, int n,
                                                               int is_fp32, int32_t *__restrict__ T,
                                                               PrepOut *__restrict__ out,
                                                               Inst *__restrict__ inst, Upload up)
{
    __shared__ double sTd[kMaxVars * kMaxVars];   // folded float32 input in float64
    __shared__ int32_t sTi[kMaxVars * kMaxVars];  // the int32 T written to T
    __shared__ int32_t sML[kMaxPrefixRows][kWave];      // M_int's lane parts (see ML)
    __shared__ int32_t sMH[kMaxPrefixRows][kMaxCols];   // and column parts
    __shared__ double sW[kPrepWaves];
    __shared__ int sLo, sHi;
    __shared__ unsigned long long sSum;
    __shared__ int sNnz, sBad;
    __shared__ double sS;
    const int tid = int(threadIdx.x), nn = n * n;
    const Inst &hI = up.src ? *reinterpret_cast<const Inst *>(up.src) : *inst;
    const int A = hI.A, B = hI.B, direct = hI.direct, wide = hI.wide;
    if (up.src) upload(up, tid, kPrepThreads);
    if (tid == 0) {
        sSum = 0ull;
        sNnz = 0;
        sBad = 0;
        sLo = INT32_MAX;
        sHi = INT32_MIN;
    }
    __syncthreads();
    uint64_t mySum = 0;
    int myNnz = 0, myBad = 0;
    double myAbs = 0.0;
    if (!is_fp32) {
        const int32_t *q = static_cast<const int32_t *>(dQ);
        for (int e = tid; e < nn; e += kPrepThreads) {
            const int i = e / n, j = e % n;
            int32_t v = 0;
            if (i <= j) {
                const int64_t t = i == j ? int64_t(q[e]) : int64_t(q[e]) + int64_t(q[j * n + i]);
                mySum += uint64_t(t < 0 ? -t : t);
                v = int32_t(t);   // kept only if the bound holds (else T is zeroed)
            }
            T[e] = v;
            sTi[e] = v;
        }
    } else {
        const float *q = static_cast<const float *>(dQ);
        for (int e = tid; e < nn; e += kPrepThreads) {
            const int i = e / n, j = e % n;
            double t = 0.0;
            if (i <= j) {
                const double a = double(q[e]), b = i == j ? 0.0 : double(q[j * n + i]);
                if (!isfinite(a) || !isfinite(b)) myBad = 1;
                t = a + b;
                if (t != 0.0) myNnz++;
                myAbs += fabs(t);
            }
            sTd[e] = t;
        }
    }
    // wave sums first: one LDS atomic per wave
    mySum = uint64_t(wave_sum64(int64_t(mySum)));
    myNnz = wave_sum(myNnz);
    const bool anyBad = __builtin_amdgcn_ballot_w64(myBad != 0) != 0;
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) myAbs += __shfl_xor(myAbs, off, kWave);
    if (tid % kWave == 0) {
        if (mySum) atomicAdd(&sSum, (unsigned long long)mySum);
        if (myNnz) atomicAdd(&sNnz, myNnz);
        if (anyBad) atomicOr(&sBad, 1);
        sW[tid / kWave] = myAbs;
    }
    __syncthreads();
    int32_t status = 0;
    int p = 0;
    int64_t sum = 0;
    double eps = 0.0;
    if (!is_fp32) {
        sum = int64_t(sSum);
        if (sum > kExactSumLimit) status = kPrepOverflow;
    } else if (sBad) {
        status = kPrepNonFinite;
    } else {
        // S by a tree: any order of at most 1830 non-negative terms is within
        // 2^-41 of the exact sum, and so of the host's.  The exponents agree
        // unless a power of two lies between.
        double S = 0.0;
#pragma unroll
        for (int w = 0; w < kPrepWaves; w++) S += sW[w];
        p = prep_scale_exponent(S);
        const double off = ldexp(S, -40);
        if (prep_scale_exponent(S - off) != p || prep_scale_exponent(S + off) != p) {
            if (tid == 0) {
                double s = 0.0;
                for (int i = 0; i < n; i++)
                    for (int j = i; j < n; j++) s += fabs(sTd[i * n + j]);
                sS = s;
            }
            __syncthreads();
            p = prep_scale_exponent(sS);
        }
        uint64_t s2 = 0;
        for (int e = tid; e < nn; e += kPrepThreads) {
            const int64_t t = int64_t(rint(ldexp(sTd[e], p)));   // ties to even
            s2 += uint64_t(t < 0 ? -t : t);
            T[e] = int32_t(t);
            sTi[e] = int32_t(t);
        }
        s2 = uint64_t(wave_sum64(int64_t(s2)));
        if (tid % kWave == 0 && s2) atomicAdd(&sSum, (unsigned long long)s2);
        __syncthreads();
        sum = int64_t(sSum);
        if (sum > kExactSumLimit) status = kPrepInternal;
        eps = double(sNnz) * ldexp(1.0, -p - 1);
    }
    if (status != 0)
        for (int e = tid; e < nn; e += kPrepThreads) T[e] = 0;
    // The int32 walk's shift c = -(least chunk energy of the split): every
    // E_sd(s, x_p) = E_s(s) + sum_v x_v M[v][s] is at least E_s(s) + the
    // negative M[v][s], so the least is the minimum of that over the 2^B
    // columns s = j*64 + l (the host planner's rule; B <= 10 here); the largest
    // one decides whether the walk may use wide words.  All are partial sums of
    // T: int32.
    const bool walked = !direct && status == 0;
    const int JB = B - 6;
    if (walked) {
        for (int e = tid; e < A * kWave; e += kPrepThreads) {
            const int v = e / kWave, l = e % kWave;
            int32_t m = 0;
#pragma unroll
            for (int u = 0; u < 6; u++) m += -((l >> u) & 1) & sTi[v * n + n - 1 - u];
            sML[v][l] = m;
        }
        for (int e = tid; e < A * kMaxCols; e += kPrepThreads) {
            const int v = e / kMaxCols, j = e % kMaxCols;
            int32_t m = 0;
            for (int u = 0; u < JB; u++) m += -((j >> u) & 1) & sTi[v * n + n - 7 - u];
            sMH[v][j] = m;
        }
    }
    __syncthreads();
    if (walked) {
        // thread (j, l): column j*64 + l
        int32_t lo = INT32_MAX, hi = INT32_MIN;
        const int l = tid % kWave, j = tid / kWave;
        if (j < (1 << JB)) {
            const int s = tid;
            int32_t e = 0;
            for (int b = 0; b < B; b++) {
                const int r = (n - 1 - b) * n;
                int32_t row = sTi[r + n - 1 - b];
                for (int c = 0; c < b; c++) row += -((s >> c) & 1) & sTi[r + n - 1 - c];
                e += -((s >> b) & 1) & row;
            }
            lo = hi = e;
#pragma unroll 4
            for (int v = 0; v < A; v++) {
                const int32_t m = sML[v][l] + sMH[v][j];
                lo += min(0, m);
                hi += max(0, m);
            }
        }
        lo = wave_min(lo);
        hi = -1 - wave_min(-1 - hi);
        if (tid % kWave == 0) {
            atomicMin(&sLo, lo);
            atomicMax(&sHi, hi);
        }
    }
    __syncthreads();
    if (tid == 0) {
        const int64_t lo = walked ? int64_t(sLo) : 0;
        const bool fits = sum + (lo < 0 ? -lo : lo) <= kExactSumLimit;
        inst->pack_shift = fits ? int32_t(-lo) : 0;
        inst->wide = wide && walked && fits && int64_t(sHi) - lo < (int64_t(1) << kWideBits) ? 1 : 0;
        PrepOut o;
        o.status = status;
        o.p = status ? 0 : p;
        o.sum_abs = status ? 0 : sum;
        o.eps_q = status ? 0.0 : eps;
        int shift = 0;
        while (((2 * o.sum_abs) >> shift) >= kTopkBins) shift++;
        o.hist_lo = -o.sum_abs;
        o.hist_shift = shift;
        o.pad = 0;
        *out = o;
    }
}

// ---------------------------------------------------------------- finish

constexpr int kFinishThreads = 256;
constexpr int kFinishWaves = kFinishThreads / kWave;
constexpr int kDirectLow = 8;    // index bits of a direct instance held by the thread number
constexpr int kDirectHigh = 14 - kDirectLow;
static_assert((1 << kDirectLow) == kFinishThreads, "one low pattern per thread");

__device__ __forceinline__ uint32_t wave_umin(uint32_t v)
{
    return uint32_t(wave_min(int32_t(v ^ 0x80000000u))) ^ 0x80000000u;
}

// Lexicographic (E, index) minimum over the block, the same in every thread:
// DPP minima of the energy, then of the index words among the lanes that
// hold it, and the wave results through LDS (sE, sI: one slot per wave).
__device__ void block_lexmin(int32_t &E, uint64_t &I, int32_t *sE, uint64_t *sI)
{
    const int32_t m = wave_min(E);
    const uint32_t hi = E == m ? uint32_t(I >> 32) : ~0u;
    const uint32_t mh = wave_umin(hi);
    const uint32_t ml = wave_umin(E == m && hi == mh ? uint32_t(I) : ~0u);
    const int w = int(threadIdx.x) / kWave;
    __syncthreads();   // the slots may still be read from the last call
    if (int(threadIdx.x) % kWave == 0) {
        sE[w] = m;
        sI[w] = (uint64_t(mh) << 32) | ml;
    }
    __syncthreads();
    E = sE[0];
    I = sI[0];
#pragma unroll
    for (int k = 1; k < kFinishWaves; k++)
        if (sE[k] < E || (sE[k] == E && sI[k] < I)) {
            E = sE[k];
            I = sI[k];
        }
}

// One 256-thread block per instance.  What bounds it is the chain of short
// dependent steps (descriptor, T and records, block minimum, suffix fields,
// chunk minimum, check), so the steps are few, their loads are issued together
// ahead of the first barrier, and sums and minima go through DPP; four waves a
// block let eight blocks share a CU, which a batch needs.  Energies are
// partial sums of T and fit int32 (sum |T| <= 2^30 - 1).
// Measured, against 1024-thread blocks with the O(B^2) rescan per state and a
// serial gather of the rescore: n = 12 direct 29 -> 6.6 us, lone walked int32
// 17-21 -> 6.6-12 us, float32 31-50 -> 10-18 us; 1000 float32 instances 163 ->
// 16 us, 4096 int32 ones 184 -> 21 us.
__global__ __launch_bounds__(kFinishThreads) void finish_kernel(
    const Inst *__restrict__ insts, FinalRes *__restrict__ out, Upload up,
    const unsigned long long *__restrict__ counters, PrepOut *__restrict__ prep_out)
{
    const unsigned long long now = wall_clock64();
    __shared__ int32_t sE[kFinishWaves];
    __shared__ uint64_t sI[kFinishWaves];
    __shared__ int32_t sH[16];                    // suffix fields of the winning chunk
    __shared__ int32_t sFull[kFinishWaves];
    __shared__ int32_t sVar[kWave];               // the answer's set variables, ascending
    __shared__ int32_t sHigh[1 << kDirectHigh];   // direct: energies of the high patterns
    // T made symmetric, and later the float32 entries the rescore adds up
    __shared__ int32_t sS[kMaxVars * kMaxVars];
    Inst I = up.src ? *reinterpret_cast<const Inst *>(up.src) : insts[blockIdx.x];
    if (up.src) {   // T and Q of the host image
        I.T = reinterpret_cast<const int32_t *>(reinterpret_cast<const unsigned char *>(I.T) - up.dst +
                                                up.src);
        if (I.Qf)
            I.Qf = reinterpret_cast<const float *>(reinterpret_cast<const unsigned char *>(I.Qf) -
                                                   up.dst + up.src);
    }
    const int n = I.n, tid = int(threadIdx.x), w = tid / kWave, l = tid % kWave;
    stage_symmetric(I.T, n, sS, tid, kFinishThreads, false);
    int32_t bE = INT32_MAX;
    uint64_t bI = ~0ull;
    int32_t status = 0;
    if (I.direct) {
        __syncthreads();
        // Every state r = (high pattern) 2^low + tid, low = min(n, 8): the
        // energy of the low bits and their fields on the high variables once
        // per thread, then the high patterns in Gray order, one add each, plus
        // the pattern's own energy.  Bit b of r is variable n-1-b.
        const int low = n < kDirectLow ? n : kDirectLow, nh = n - low;
        auto S = [&](int b, int c) { return sS[(n - 1 - b) * n + n - 1 - c]; };
        if (tid < (1 << nh)) {
            int32_t e = 0;
            for (int x = 0; x < nh; x++) {
                int32_t row = S(low + x, low + x);
                for (int y = 0; y < x; y++) row += -((tid >> y) & 1) & S(low + x, low + y);
                e += -((tid >> x) & 1) & row;
            }
            sHigh[tid] = e;
        }
        int32_t base = 0, g[kDirectHigh];
        for (int b = 0; b < low; b++) {
            int32_t row = S(b, b);
            for (int c = 0; c < b; c++) row += -((tid >> c) & 1) & S(b, c);
            base += -((tid >> b) & 1) & row;
        }
#pragma unroll
        for (int x = 0; x < kDirectHigh; x++) {
            g[x] = 0;
            if (x < nh)
                for (int b = 0; b < low; b++) g[x] += -((tid >> b) & 1) & S(low + x, b);
        }
        __syncthreads();
        uint32_t bR = ~0u;
        if (tid < (1 << low)) {
            bE = base;
            bR = uint32_t(tid);
            int32_t e = base;
            static_for<1, (1 << kDirectHigh)>([&](auto pc) {
                constexpr int p = decltype(pc)::value, x = cx_ctz(p), pat = p ^ (p >> 1);
                if (p < (1 << nh)) {
                    e += ((pat >> x) & 1) ? g[x] : -g[x];
                    const int32_t E = e + sHigh[pat];
                    const uint32_t r = (uint32_t(pat) << low) | uint32_t(tid);
                    if (E < bE || (E == bE && r < bR)) {
                        bE = E;
                        bR = r;
                    }
                }
            });
        }
        bI = bR;
        block_lexmin(bE, bI, sE, sI);
    } else {
        const int A = I.A, B = I.B;
        const int NS = 1 << B, NW = I.packed ? NS / 2 : NS;
        // suffix energies of this thread's columns (words tid + 256 k)
        constexpr int kWords = kMaxCols * kWave / kFinishThreads;
        int32_t eb[kWords];
#pragma unroll
        for (int k = 0; k < kWords; k++) {
            const int c = tid + kFinishThreads * k;
            eb[k] = c < NW ? I.EB[c] : 0;
        }
        // the records of items whose bit is set (the others were never
        // written); each thread takes four consecutive bitmap words at a
        // time, loaded together before any is examined
        const uint64_t words = (I.n_items + 31) / 32;
        for (uint64_t w0 = uint64_t(tid) * 4; w0 < words; w0 += uint64_t(kFinishThreads) * 4) {
            uint32_t x[4];
#pragma unroll
            for (int k = 0; k < 4; k++) x[k] = w0 + k < words ? I.bits[w0 + k] : 0u;
#pragma unroll
            for (int k = 0; k < 4; k++) {
                while (x[k]) {
                    const uint32_t b = uint32_t(__builtin_ctz(x[k]));
                    x[k] &= x[k] - 1u;
                    const ItemRes r = I.res[(w0 + k) * 32 + b];
                    if (r.E < bE || (r.E == bE && r.row < bI)) {
                        bE = r.E;
                        bI = r.row;
                    }
                }
            }
        }
        block_lexmin(bE, bI, sE, sI);   // (its barriers also cover sS)
        const int32_t Estar = bE;
        const uint64_t rowstar = bI;
        if (Estar == INT32_MAX) {
            status = 2;   // no item reported a candidate
        } else {
            // Argmin reconstruction (ConstructState of Alg. 2): the lowest
            // suffix s of the minima of chunk rowstar.  With the prefix fixed,
            // E(row, s) = E_p(row) + E_s(s) + sum_{t in s} h_t (Sec. II-C),
            // h_t = sum over the set prefix variables v of T[v][A+t], so the
            // chunk's minima are those of E_s + sum h_t.  Wave w forms h_t for
            // t = w, w + 4, ..., one lane per prefix variable (A < 64).
            for (int t = w; t < B; t += kFinishWaves) {
                const bool on = l < A && ((rowstar >> ((A - 1 - l) & 63)) & 1);
                const int32_t h = wave_sum(on ? sS[(A + t) * n + l] : 0);
                if (l == 0) sH[t] = h;
            }
            __syncthreads();
            int32_t lowsum = 0;   // column bits 0..5 and 6, 7: tid's
#pragma unroll
            for (int b = 0; b < 8; b++)
                if (b < B) lowsum += -((tid >> b) & 1) & sH[B - 1 - b];
            int32_t mF = INT32_MAX;
            uint32_t mS = ~0u;
            auto offer = [&](int32_t es, uint32_t s) {
                int32_t f = es + lowsum;
#pragma unroll
                for (int b = 8; b < 11; b++)
                    if (b < B) f += -int32_t((s >> b) & 1) & sH[B - 1 - b];
                if (f < mF || (f == mF && s < mS)) {
                    mF = f;
                    mS = s;
                }
            };
#pragma unroll
            for (int k = 0; k < kWords; k++) {
                const int c = tid + kFinishThreads * k;
                if (c >= NW) continue;
                if (I.packed) {
                    offer(eb[k] & 0xffff, uint32_t(c));
                    offer(int32_t(uint32_t(eb[k]) >> 16), uint32_t(c + NW));
                } else {
                    offer(eb[k], uint32_t(c));
                }
            }
            uint64_t s64 = mS;
            block_lexmin(mF, s64, sE, sI);
            bI = (rowstar << B) | s64;
            // the winner evaluated in full from T must have the energy the
            // walk claimed: lane l adds up variable l's row, each wave a
            // quarter of it
            const bool on = l < n && ((bI >> ((n - 1 - l) & 63)) & 1);
            int32_t own = 0;
            for (int j = w; j < n; j += kFinishWaves) {
                const int32_t c = sS[j * n + (l < n ? l : 0)];
                own += (j >= l && ((bI >> (n - 1 - j)) & 1)) ? c : 0;
            }
            own = wave_sum(on ? own : 0);
            if (l == 0) sFull[w] = own;
            __syncthreads();
            int32_t full = 0;
#pragma unroll
            for (int k = 0; k < kFinishWaves; k++) full += sFull[k];
            if (full != Estar) status = 3;   // the walk claimed an energy the chunk lacks
        }
    }
    double E64 = double(bE);
    if (I.Qf && status == 0) {
        // float64 rescore from the caller's matrix, summed i ascending then j
        // ascending over the set variables: the entries are gathered side by
        // side, in that order, and one thread adds them up
        float *sQ = reinterpret_cast<float *>(sS);
        const int m = __builtin_popcountll(bI);
        // variable l is bit n-1-l: its rank counts the set bits above
        if (tid < n && ((bI >> (n - 1 - tid)) & 1))
            sVar[__builtin_popcountll((bI >> (n - 1 - tid)) >> 1)] = tid;
        __syncthreads();   // (and sS is done with)
        for (int e = w; e < m; e += kFinishWaves)
            if (l < m) sQ[e * m + l] = I.Qf[sVar[e] * n + sVar[l]];
        __syncthreads();
        if (tid == 0) {
            double s = 0.0;
#pragma unroll 8
            for (int e = 0; e < m * m; e++) s += double(sQ[e]);
            E64 = s;
        }
    }
    if (tid == 0) {
        FinalRes o;
        o.E = bE;
        o.index = bI;
        o.E64 = E64;
        o.status = status;
        o.pad = 0;
        o.walk_ticks = counters ? now - counters[kClockWord] : 0;
        out[blockIdx.x] = o;
        if (prep_out) *prep_out = *I.prep;
    }
}

// ---------------------------------------------------------------- launchers

hipError_t launch_prepare(const void *dQ, int n, int is_fp32, int32_t *d_T, PrepOut *d_prep,
                          Inst *d_inst, const Upload &up, hipStream_t stream)
{
    if (n < 1 || n > kMaxVars) return hipErrorInvalidValue;
    hipLaunchKernelGGL(prepare_kernel, dim3(1), dim3(kPrepThreads), 0, stream, dQ, n, is_fp32, d_T,
                       d_prep, d_inst, up);
    return hipGetLastError();
}

hipError_t launch_tables(const Inst *d_insts, int n_inst, unsigned long long *d_counters,
                         int n_groups, const Upload &up, hipStream_t stream)
{
    if (up.src && n_inst != 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(tables_kernel, dim3(up.src ? kTableParts + 1 : kTableParts, n_inst),
                       dim3(kTableThreads), 0, stream, d_insts, d_counters, n_groups, up,
                       static_cast<const Upload *>(nullptr));
    return hipGetLastError();
}

hipError_t launch_tables_upload(const Upload *ups, int n_inst, hipStream_t stream)
{
    hipLaunchKernelGGL(tables_kernel, dim3(kTableParts + 1, n_inst), dim3(kTableThreads), 0, stream,
                       static_cast<const Inst *>(nullptr), static_cast<unsigned long long *>(nullptr),
                       0, Upload{}, ups);
    return hipGetLastError();
}

hipError_t launch_upload(const Upload &up, hipStream_t stream)
{
    const uint32_t bytes = up.copy_bytes + up.zero_bytes;
    const int blocks = int(bytes / 16384 < 63 ? bytes / 16384 + 1 : 64);
    hipLaunchKernelGGL(upload_kernel, dim3(blocks), dim3(256), 0, stream, up);
    return hipGetLastError();
}

// Variants built: every MC with G = 12; MC = 8 and 16 with G = 8; MC = 16
// with G = 6 and 5, "4": G = 6 with levels 3 and 4 in LDS (levels 0-2 and 5
// in VGPRs, four waves per SIMD), and "3": G = 5 with levels 3 and 4 in LDS
// (levels 0-2 in VGPRs; every flip of level 5 or above reads its signed row
// from L2).
bool walk_packed_exists(int mcols, int vgpr_levels)
{
    return mcols >= 4 && walk_variant_exists(mcols, vgpr_levels);
}

bool walk_variant_exists(int mcols, int vgpr_levels)
{
    if (vgpr_levels == 12) return mcols == 1 || mcols == 2 || mcols == 4 || mcols == 8 || mcols == 16;
    if (vgpr_levels == 8) return mcols == 8 || mcols == 16;
    if (vgpr_levels == 6 || vgpr_levels == 5 || vgpr_levels == 4 || vgpr_levels == 3)
        return mcols == 16;
    return false;
}

int walk_occupancy(int mcols, int vgpr_levels, int tier)
{
    switch (vgpr_levels) {
    case 4: return tier == 3 || tier == 5 ? occupancy_walk_g4_topk(tier) : occupancy_walk_g6(true, tier);
    case 3: return occupancy_walk_g5(true, tier);
    case 6: return occupancy_walk_g6(false, tier);
    case 5: return occupancy_walk_g5(false, tier);
    case 8: return occupancy_walk_g8(mcols, tier);
    default:
        return mcols <= 4 ? occupancy_walk_g12(mcols, tier) : occupancy_walk_g12w(mcols, tier);
    }
}

hipError_t launch_walk_pair(const WalkPart &tier2, const WalkPart &tier4, const int32_t *d_k,
                            int waves, hipStream_t stream)
{
    auto part = [&](int tier, const WalkPart &p) {
        const WalkClaims wc{p.total_items, 0, 0, p.max_L >= kStealSteps ? kQueues - 1 : 0};
        return WalkLaunch{tier, p.d_insts, p.n_inst, wc, p.d_counter, d_k, waves, stream, nullptr};
    };
    return launch_walk_pair(part(2, tier2), part(4, tier4));
}

hipError_t launch_walk(int mcols, int vgpr_levels, int tier, const Inst *d_insts, int n_inst,
                       uint64_t total_items, int max_L, unsigned long long *d_counter,
                       const int32_t *d_k, int waves, hipStream_t stream, const TopkWalk *tk,
                       int wide)
{
    WalkClaims wc{total_items, 0, 0, max_L >= kStealSteps ? kQueues - 1 : 0};
    if (n_inst == 1 && total_items >= kRunItems && max_L + kRunLog <= kRunMaxSteps) {
        wc.run_log = kRunLog;
        wc.runs = (total_items >> kRunLog) * 17 / 20;
        wc.claims = wc.runs + (total_items - (wc.runs << kRunLog));
    }
    const WalkLaunch w{tier, d_insts, n_inst, wc, d_counter, d_k, waves, stream, tk};
    if (vgpr_levels == 6 || vgpr_levels == 5 || vgpr_levels == 4 || vgpr_levels == 3) {
        if (mcols != 16) return hipErrorInvalidValue;
        if (vgpr_levels == 4 && n_inst == 1 && tier >= 2) {
            if (wide && tier != 2 && tier != 3) return hipErrorInvalidValue;
            const hipError_t e = wide ? launch_walk_wide(w) : hipSuccess;
            return e != hipSuccess || wide == 1 ? e : launch_walk_g4(w);
        }
        if (wide) return hipErrorInvalidValue;
        if (vgpr_levels == 6 || vgpr_levels == 4) return launch_walk_g6(vgpr_levels == 4, w);
        return launch_walk_g5(vgpr_levels == 3, w);
    }
    if (vgpr_levels == 8) return launch_walk_g8(mcols, w);
    if (vgpr_levels != 12) return hipErrorInvalidValue;
    return mcols <= 4 ? launch_walk_g12(mcols, w) : launch_walk_g12w(mcols, w);
}

hipError_t launch_finish(const Inst *d_insts, int n_inst, FinalRes *d_out, const Upload &up,
                         const unsigned long long *d_counters, PrepOut *prep_out,
                         hipStream_t stream)
{
    if (up.src && n_inst != 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(finish_kernel, dim3(n_inst), dim3(kFinishThreads), 0, stream, d_insts, d_out,
                       up, d_counters, prep_out);
    return hipGetLastError();
}

}  // namespace qk
