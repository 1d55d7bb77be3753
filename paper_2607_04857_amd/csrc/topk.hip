// topk.hip -- the k lowest-energy states of one instance (k > 1).
//
// The paper's kernel returns the minimum; it names the k lowest energies as
// an extension (Sec. VI).  Here the answer is the k smallest (E, index)
// pairs, index = U_N row.  Let a chunk be the 2^B states of one prefix row
// and its key (E_p + min over the chunk, row).  The k smallest states lie in
// the k smallest chunks by key: if a chunk c holding one of them were not
// among those, k chunks with smaller keys would each hold a state smaller
// than it.  So:
//   1. the tier-3 walk leaves per-wave lists of candidate chunk keys that
//      together contain the k smallest chunks (kernels.hip);
//   2. compact the list entries at or below the final shared bound, and
//      select the k smallest chunk keys among them;
//   3. rescan those chunks: every state's energy from the tables,
//      E = E_p(row) + E_s(s) + x_p M_int[:, s] (Sec. II-C), keeping the
//      states at or below the largest selected chunk key (the k chunk minima
//      are k states at or below it, so the k-th smallest energy is too), or,
//      with fewer than k chunks, those at or below a bound that each block
//      finds for its own;
//   4. select the k smallest (E, index) among them;
//   5. put them in order, verify each energy from T, rescore fp32 instances
//      in float64 and sort those by (E64, index).
// Selection is an exact radix select on the energy (order-preserving
// unsigned key) and, where the k-th energy is tied, on the row/index among
// the tied entries; keys are unique (a row is walked once, an index occurs
// once), so exactly min(k, candidates) entries are kept.
#include "device_energy.h"
#include "kcommon.h"
#include "kernels.h"

namespace qk {

namespace {

constexpr int kSelThreads = 1024;   // also the largest k

struct SelArgs {
    const int32_t *E;          // dense candidates [0, *count * mult)
    const uint64_t *R;
    const int32_t *count;
    uint32_t mult;
    int k;
    int32_t *oE;               // [k] output, in no order
    uint64_t *oR;
    int32_t *oCount;           // [0] entries selected, [1] their largest energy
    int32_t *clear;            // set to 0 when done (a later kernel's counter), or null
};

__device__ __forceinline__ uint32_t ukey(int32_t e) { return uint32_t(e) ^ 0x80000000u; }

__device__ __forceinline__ bool key_less(int32_t ea, uint64_t ra, int32_t eb, uint64_t rb)
{
    return ea < eb || (ea == eb && ra < rb);
}

// Bin of the histogram where the running count reaches `need` (need <= the
// total), by the first wave: four bins a lane, one wave-wide prefix sum.  (One
// thread's walk over the 256 bins had taken 10 us a digit.)
__device__ void pick_bin(const uint32_t *hist, uint32_t need, uint32_t *bin, uint32_t *rest,
                         uint32_t *inbin)
{
    const int lane = int(threadIdx.x);
    if (lane >= kWave) return;
    uint32_t h[4], sum = 0;
#pragma unroll
    for (int x = 0; x < 4; x++) {
        h[x] = hist[4 * lane + x];
        sum += h[x];
    }
    uint32_t cum = sum;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t o = __shfl_up(cum, off, kWave);
        if (lane >= off) cum += o;
    }
    const uint64_t hit = __builtin_amdgcn_ballot_w64(cum >= need);
    if (hit == 0 || lane != int(__builtin_ctzll(hit))) return;
    cum -= sum;
    int x = 0;
    while (x < 3 && cum + h[x] < need) cum += h[x++];
    *bin = uint32_t(4 * lane + x);
    *rest = need - cum;
    *inbin = h[x];
}

// One block.  The energies are taken from their minimum, so that only the
// digits their spread occupies are counted, and up to kHeld entries a thread
// are read from memory once.  What bounds it is the chain of digits.  Nothing
// here needs the selected entries in order (the final kernel ranks them, on
// many blocks): with the 55 exchanges of a sort at the end, 2600 candidates
// with k = 1024 had taken 24 us, now 8, and a few hundred 6, now 5.
constexpr int kHeld = 4;

__global__ __launch_bounds__(kSelThreads) void topk_select_kernel(SelArgs a)
{
    __shared__ uint32_t hist[256];
    __shared__ uint32_t sh_pos, sh_bin, sh_rest, sh_in, sh_min, sh_max;
    const uint32_t tid = threadIdx.x;
    const uint32_t k = uint32_t(a.k);
    const uint32_t total = uint32_t(*a.count) * a.mult;
    const bool held = total <= kHeld * kSelThreads;

    int32_t hE[kHeld];
    uint64_t hR[kHeld];
#pragma unroll
    for (int x = 0; x < kHeld; x++) {
        const uint32_t i = tid + uint32_t(x) * kSelThreads;
        const bool on = held && i < total;
        hE[x] = on ? a.E[i] : INT32_MAX;
        hR[x] = on ? a.R[i] : ~0ull;
    }
    if (tid == 0) {
        sh_pos = 0;
        sh_min = ~0u;
        sh_max = 0;
    }
    __syncthreads();
    // visit every candidate: f(E, R)
    auto for_valid = [&](auto &&f) {
        if (held) {
#pragma unroll
            for (int x = 0; x < kHeld; x++)
                if (tid + uint32_t(x) * kSelThreads < total) f(hE[x], hR[x]);
        } else {
            for (uint32_t i = tid; i < total; i += kSelThreads) f(a.E[i], a.R[i]);
        }
    };

    const bool take_all = total <= k;
    uint32_t uk = 0xFFFFFFFFu;      // energy key of the k-th entry
    bool all_eq = true;             // take every entry whose key equals uk
    uint64_t rk = ~0ull;            // else those with R <= rk
    int32_t mn = INT32_MAX, mx = INT32_MIN;
    for_valid([&](int32_t e, uint64_t) {
        mn = min(mn, e);
        mx = max(mx, e);
    });
    mn = wave_min(mn);
    mx = -1 - wave_min(-1 - mx);   // max: ~ reverses the order
    if (tid % kWave == 0) {
        atomicMin(&sh_min, ukey(mn));
        atomicMax(&sh_max, ukey(mx));
    }
    __syncthreads();
    if (!take_all) {
        const uint32_t u0 = sh_min, spread = sh_max - u0;
        const int digits = spread ? (31 - __builtin_clz(spread)) / 8 : 0;
        uint32_t prefix = 0, mask = 0, need = k;
        for (int shift = 8 * digits; shift >= 0; shift -= 8) {
            for (uint32_t b = tid; b < 256; b += kSelThreads) hist[b] = 0;
            __syncthreads();
            for_valid([&](int32_t e, uint64_t) {
                const uint32_t u = ukey(e) - u0;
                if ((u & mask) == prefix) atomicAdd(&hist[(u >> shift) & 255u], 1u);
            });
            __syncthreads();
            pick_bin(hist, need, &sh_bin, &sh_rest, &sh_in);
            __syncthreads();
            prefix |= sh_bin << shift;
            mask |= 255u << shift;
            need = sh_rest;
        }
        uk = prefix + u0;
        all_eq = need == sh_in;     // every entry with energy key uk is kept
        if (!all_eq) {
            uint64_t rprefix = 0, rmask = 0;
            for (int shift = 56; shift >= 0; shift -= 8) {
                __syncthreads();
                for (uint32_t b = tid; b < 256; b += kSelThreads) hist[b] = 0;
                __syncthreads();
                for_valid([&](int32_t e, uint64_t r) {
                    if (ukey(e) == uk && (r & rmask) == rprefix)
                        atomicAdd(&hist[uint32_t(r >> shift) & 255u], 1u);
                });
                __syncthreads();
                pick_bin(hist, need, &sh_bin, &sh_rest, &sh_in);
                __syncthreads();
                rprefix |= uint64_t(sh_bin) << shift;
                rmask |= uint64_t(255) << shift;
                need = sh_rest;
            }
            rk = rprefix;
        }
    }
    // at most k entries
    for_valid([&](int32_t e, uint64_t r) {
        const uint32_t u = ukey(e);
        if (take_all || u < uk || (u == uk && (all_eq || r <= rk))) {
            const uint32_t p = atomicAdd(&sh_pos, 1u);
            if (p < k) {
                a.oE[p] = e;
                a.oR[p] = r;
            }
        }
    });
    __syncthreads();
    if (tid == 0) {
        a.oCount[0] = int32_t(min(sh_pos, k));
        a.oCount[1] = int32_t((take_all ? sh_max : uk) ^ 0x80000000u);
        if (a.clear) *a.clear = 0;
    }
}

// The walk lists, compacted: entries with E <= *bound of every wave's list,
// appended densely (one wave per list, wave-aggregated slots).
__global__ __launch_bounds__(256) void topk_compact_kernel(const int32_t *__restrict__ E,
                                                           const uint64_t *__restrict__ R,
                                                           const int32_t *__restrict__ listCount,
                                                           int nlists, int stride,
                                                           const int32_t *__restrict__ bound,
                                                           int32_t *__restrict__ oE,
                                                           uint64_t *__restrict__ oR,
                                                           int32_t *__restrict__ oN,
                                                           unsigned long long *__restrict__ counters)
{
    if (counters && blockIdx.x == 0 && threadIdx.x == 0) counters[kClockWord + 1] = wall_clock64();
    const int lane = int(threadIdx.x) & (kWave - 1);
    const int list = int(blockIdx.x) * (256 / kWave) + int(threadIdx.x) / kWave;
    if (list >= nlists) return;
    const int32_t bnd = *bound;
    const int c = listCount[list];
    for (int p0 = 0; p0 < c; p0 += kWave) {
        const int p = p0 + lane;
        const size_t x = size_t(list) * size_t(stride) + size_t(p);
        const bool keep = p < c && E[x] <= bnd;
        const uint64_t m = __builtin_amdgcn_ballot_w64(keep);
        if (!m) continue;
        int base = 0;
        if (lane == 0) base = atomicAdd(oN, int(__builtin_popcountll(m)));
        base = __builtin_amdgcn_readfirstlane(base);
        if (keep) {
            const int rank = int(__builtin_popcountll(m & ((1ull << lane) - 1)));
            oE[base + rank] = E[x];
            oR[base + rank] = R[x];
        }
    }
}

// Step 3: each wave rescans one chunk of rows[0 .. *rowCount) and its states
// with E <= the largest selected chunk key go to (stE, stI), densely (slots
// counted in *stCount, zeroed by the chunk select).  With fewer than k chunks
// selected (the instance has fewer than k chunks) the k-th smallest state may
// lie above every chunk minimum: each block then finds, by bisection on the
// value, the least bound with k of its own states (which bounds the instance's
// k-th smallest), so that hundreds of states of a chunk reach the select and not
// all (n = 18, k = 700: whole call 570 -> 167 us).  At most rc << B < k << B entries.
// A chunk's states follow from its suffix fields h_t = sum over the set prefix
// variables v of T[v][A+t]: E(row, s) = E_p + E_s(s) + sum_{t in s} h_t, E_s
// read from the walk's table.  One atomic per block of kRescanWaves chunks
// (they complete one per 12.4 ns).  Measured: 10 us for k = 1024
// at n = 31 and 7 us for k = 16 at n = 21 (27 and 13 us with a block per chunk,
// its rows summed one after another, and an atomic per wave and pass).
constexpr int kRescanWaves = 8;

__global__ __launch_bounds__(kRescanWaves *kWave) void topk_rescan_kernel(
    const Inst *__restrict__ inst, const uint64_t *__restrict__ rows,
    const int32_t *__restrict__ rowCount, int k,
    int32_t *__restrict__ stE, uint64_t *__restrict__ stI, int32_t *__restrict__ stCount)
{
    __shared__ int32_t sT[kMaxVars * kMaxVars];
    __shared__ int32_t sN[kRescanWaves], sLo[kRescanWaves], sHi[kRescanWaves], sBase;
    const Inst I = *inst;
    const int n = I.n, A = I.A, B = I.B;
    const int tid = int(threadIdx.x), lane = tid % kWave, w = tid / kWave;
    const int32_t rc = *rowCount;
    const int32_t b = int32_t(blockIdx.x) * kRescanWaves + w;
    if (int32_t(blockIdx.x) * kRescanWaves >= rc) return;
    for (int e = tid; e < n * n; e += kRescanWaves * kWave) sT[e] = I.T[e];
    int32_t bound = rowCount[1];   // the largest selected key
    const bool mine = b < rc;
    const uint64_t row = mine ? sread64(rows[b]) : 0;
    const int NW = I.packed ? (1 << B) / 2 : 1 << B, MC = NW / kWave;
    int32_t eb[kMaxCols];
#pragma unroll
    for (int j = 0; j < kMaxCols; j++) eb[j] = j < MC ? I.EB[j * kWave + lane] : 0;
    __syncthreads();
    auto set = [&](int v) { return ((row >> (A - 1 - v)) & 1) != 0; };
    // E_p: lane l adds up column l of the set prefix variables v <= l
    int32_t own = 0;
    for (int v = 0; v < A; v++)
        if (set(v)) own += (v <= lane && lane < A) ? sT[v * n + lane] : 0;
    const int32_t Ep = wave_sum(lane < A && set(lane < A ? lane : 0) ? own : 0);
    int32_t h = 0;   // lane t: h_t
    for (int v = 0; v < A; v++)
        if (set(v)) h += lane < B ? sT[v * n + A + lane] : 0;
    int32_t low = Ep;   // the lane's six column bits
#pragma unroll
    for (int u = 0; u < 6; u++) low += -((lane >> u) & 1) & __builtin_amdgcn_readlane(h, B - 1 - u);
    const int JB = I.packed ? B - 7 : B - 6;
    const int32_t top = __builtin_amdgcn_readlane(h, 0);   // packed: the high column's variable A
    // energies of the lane's words (packed: of both columns of a word)
    int32_t E[kMaxCols], E2[kMaxCols];
#pragma unroll
    for (int j = 0; j < kMaxCols; j++) {
        int32_t hj = 0;   // the bits of j
#pragma unroll
        for (int u = 0; u < 4; u++)
            if (u < JB && ((j >> u) & 1)) hj += __builtin_amdgcn_readlane(h, B - 7 - u);
        if (I.packed) {
            // E_s carries the walk's shift and the packed bias
            const int32_t base = low + hj - kPackBias - I.pack_shift;
            E[j] = base + (eb[j] & 0xffff);
            E2[j] = base + top + int32_t(uint32_t(eb[j]) >> 16);
        } else {
            E[j] = low + hj + eb[j] - I.pack_shift;
            E2[j] = 0;
        }
    }
    // this wave's states at or below e
    auto at_most = [&](int32_t e) {
        int32_t c = 0;
#pragma unroll
        for (int j = 0; j < kMaxCols; j++) {
            if (!mine || j >= MC) continue;
            c += __builtin_popcountll(__builtin_amdgcn_ballot_w64(E[j] <= e));
            if (I.packed) c += __builtin_popcountll(__builtin_amdgcn_ballot_w64(E2[j] <= e));
        }
        return c;
    };
    if (rc < k) {
        int32_t mn = INT32_MAX, mx = INT32_MIN;
#pragma unroll
        for (int j = 0; j < kMaxCols; j++) {
            if (!mine || j >= MC) continue;
            mn = min(mn, I.packed ? min(E[j], E2[j]) : E[j]);
            mx = max(mx, I.packed ? max(E[j], E2[j]) : E[j]);
        }
        mn = wave_min(mn);
        mx = -1 - wave_min(-1 - mx);
        if (lane == 0) {
            sLo[w] = mn;
            sHi[w] = mx;
        }
        __syncthreads();
        int64_t lo = INT32_MAX, hi = INT32_MIN;
        for (int x = 0; x < kRescanWaves; x++) {
            lo = min(lo, int64_t(sLo[x]));
            hi = max(hi, int64_t(sHi[x]));
        }
        // (a block with fewer than k states ends at its largest)
        while (lo < hi) {
            const int64_t mid = lo + (hi - lo) / 2;
            const int32_t c = at_most(int32_t(mid));
            __syncthreads();   // the last round's counts have been read
            if (lane == 0) sN[w] = c;
            __syncthreads();
            int32_t sum = 0;
#pragma unroll
            for (int x = 0; x < kRescanWaves; x++) sum += sN[x];
            if (sum >= k) hi = mid;
            else lo = mid + 1;
        }
        bound = int32_t(hi);
        __syncthreads();
    }
    const int32_t kept = at_most(bound);
    if (lane == 0) sN[w] = kept;
    __syncthreads();
    if (tid == 0) {
        int32_t sum = 0;
        for (int x = 0; x < kRescanWaves; x++) {
            const int32_t c = sN[x];
            sN[x] = sum;
            sum += c;
        }
        sBase = sum ? atomicAdd(stCount, sum) : 0;
    }
    __syncthreads();
    if (!mine) return;
    int32_t at = sBase + sN[w];
    auto offer = [&](int32_t e, uint32_t s) {
        const uint64_t m = __builtin_amdgcn_ballot_w64(e <= bound);
        if (e <= bound) {
            const int p = at + int(__builtin_popcountll(m & ((1ull << lane) - 1)));
            stE[p] = e;
            stI[p] = (row << B) | s;
        }
        at += int(__builtin_popcountll(m));
    };
#pragma unroll
    for (int j = 0; j < kMaxCols; j++) {
        if (j < MC) {
            offer(E[j], uint32_t(j * kWave + lane));
            if (I.packed) offer(E2[j], uint32_t(NW + j * kWave + lane));
        }
    }
}

// Step 3 for direct instances: every state.
__global__ __launch_bounds__(256) void topk_direct_kernel(const Inst *__restrict__ inst,
                                                          int32_t *__restrict__ stE,
                                                          uint64_t *__restrict__ stI,
                                                          int32_t *__restrict__ segCount)
{
    const Inst I = *inst;
    const uint32_t N = 1u << I.n;
    for (uint32_t r = blockIdx.x * blockDim.x + threadIdx.x; r < N; r += gridDim.x * blockDim.x) {
        stE[r] = int32_t(energy_int(I.T, I.n, r));
        stI[r] = r;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) segCount[0] = int32_t(N);
}

// Step 5: a block of sixteen waves per 64 states of the answer, a lane each in
// every wave.  A state's place is the number of selected keys below its own
// (each wave counts a sixteenth of them, broadcast from LDS), and its energy
// from T, a sixteenth of the rows a wave, must be the one the selection has.
// float32 instances are rescored in float64 and ordered by topk_order_kernel.
// A state whose energy differs goes out as kTopkBadState: out and best may be
// mapped host memory, where no atomic could raise a status (a copy of the
// results had cost 10-12 us).  Measured, with the selection left unordered: 8 us
// for k = 1024 at n = 31 and 3 us for k = 16 at n = 21 (16 and 9 us at one thread
// a state, of states that the selection had sorted).
constexpr int kFinalWaves = 16;

__global__ __launch_bounds__(kFinalWaves *kWave) void topk_final_kernel(
    const Inst *__restrict__ inst, const int32_t *__restrict__ selE,
    const uint64_t *__restrict__ selR, const int32_t *__restrict__ selCount, int k,
    TopkState *__restrict__ out, FinalRes *__restrict__ best,
    const unsigned long long *__restrict__ counters, const PrepOut *__restrict__ prep,
    PrepOut *__restrict__ prep_out)
{
    __shared__ int32_t sT[kMaxVars * kMaxVars];
    __shared__ float sQ[kMaxVars * kMaxVars];
    __shared__ int32_t sE[kSelThreads], sPlace[kWave], sSum[kWave];
    __shared__ uint64_t sR[kSelThreads];
    const Inst I = *inst;
    const int n = I.n;
    const int tid = int(threadIdx.x), lane = tid % kWave, w = tid / kWave;
    const int cnt = min(*selCount, k);
    for (int x = tid; x < cnt; x += kFinalWaves * kWave) {
        sE[x] = selE[x];
        sR[x] = selR[x];
    }
    for (int x = tid; x < n * n; x += kFinalWaves * kWave) {
        sT[x] = I.T[x];
        if (I.Qf) sQ[x] = I.Qf[x];
    }
    if (tid < kWave) sPlace[tid] = sSum[tid] = 0;
    __syncthreads();
    const int at = int(blockIdx.x) * kWave + lane;
    const bool on = at < cnt;
    const uint64_t idx = on ? sR[at] : 0;
    const int32_t e = on ? sE[at] : 0;
    int32_t place = 0;
    for (int x = w; x < cnt; x += kFinalWaves) place += key_less(sE[x], sR[x], e, idx) ? 1 : 0;
    int32_t sum = 0;   // a partial sum of T: within the int32 bound
    for (int i = w; i < n; i += kFinalWaves) {
        int32_t row = 0;
#pragma unroll 4
        for (int j = i; j < n; j++) row += -int32_t((idx >> (n - 1 - j)) & 1) & sT[i * n + j];
        sum += -int32_t((idx >> (n - 1 - i)) & 1) & row;
    }
    if (on) {
        atomicAdd(&sPlace[lane], place);
        atomicAdd(&sSum[lane], sum);
    }
    __syncthreads();
    if (w != 0) return;
    if (on) {
        TopkState o;
        o.E = sSum[lane] == e ? int64_t(e) : kTopkBadState;
        o.E64 = I.Qf ? energy_f64(sQ, n, idx) : double(e);
        o.index = idx;
        out[sPlace[lane]] = o;
        if (sPlace[lane] == 0) {
            best->E = o.E;
            best->index = idx;
            best->E64 = o.E64;
        }
    }
    if (at == 0) {
        best->walk_ticks = counters ? counters[kClockWord + 1] - counters[kClockWord] : 0;
        best->status = cnt < k ? 4 : 0;
        if (prep_out) *prep_out = *prep;
    }
}

// The integer order is exact for the scaled energies; float32 answers are
// reported by their float64 energies, in their own (E64, index) order.  (in and
// out are the same where the results stay in device memory: all of in is read
// before the first barrier.)
__global__ __launch_bounds__(kSelThreads) void topk_order_kernel(
    const int32_t *__restrict__ selCount, int k, const TopkState *in, TopkState *out,
    FinalRes *__restrict__ best)
{
    __shared__ double sF[kSelThreads];
    __shared__ uint64_t sI[kSelThreads];
    __shared__ int64_t sE[kSelThreads];
    const uint32_t tid = threadIdx.x;
    const int cnt = min(*selCount, k);
    uint32_t P = 1;
    while (P < uint32_t(cnt)) P <<= 1;
    const bool on = int(tid) < cnt;
    sF[tid] = on ? in[tid].E64 : __builtin_huge_val();
    sI[tid] = on ? in[tid].index : ~0ull;
    sE[tid] = on ? in[tid].E : 0;
    __syncthreads();
    for (uint32_t size = 2; size <= P; size <<= 1) {
        for (uint32_t st = size >> 1; st > 0; st >>= 1) {
            const uint32_t j = tid ^ st;
            if (tid < P && j > tid) {
                const bool asc = (tid & size) == 0;
                const bool jl = sF[j] < sF[tid] || (sF[j] == sF[tid] && sI[j] < sI[tid]);
                if (jl == asc) {
                    const double tf = sF[tid];
                    const uint64_t ti = sI[tid];
                    const int64_t te = sE[tid];
                    sF[tid] = sF[j];
                    sI[tid] = sI[j];
                    sE[tid] = sE[j];
                    sF[j] = tf;
                    sI[j] = ti;
                    sE[j] = te;
                }
            }
            __syncthreads();
        }
    }
    if (on) {
        TopkState o;
        o.E = sE[tid];
        o.E64 = sF[tid];
        o.index = sI[tid];
        out[tid] = o;
    }
    if (tid == 0 && cnt > 0) {
        best->E = sE[0];
        best->index = sI[0];
        best->E64 = sF[0];
    }
}

// ---------------------------------------------------------------- seed
// Upper bound of the k-th smallest chunk key, set as the shared bound before
// the walk (which then only lowers it).  Chunks of distinct prefix rows are
// distinct, and a state's energy bounds its own chunk's key from above, so
// the k-th smallest energy over states with k or more distinct prefix rows
// bounds the k-th smallest chunk key.  The states: a local minimum x* of
// eight greedy descents and the states that differ from it in one to four
// prefix variables (the first kSeedStates in order of the number of flips,
// each group in colex order).  Their energies follow from x*'s single-flip
// changes d_i and the couplings: flipping the set F changes E by
//   sum_{i in F} d_i + sum_{i<j in F} s_i s_j T_ij,   s_i = 1 - 2 x_i.
// Each thread numbers its four states by binary search over the binomials and
// keeps their energies in registers; the k-th smallest is found by bisection
// on the value, its counts taken by ballots.  Measured: 25 us at n = 31, k =
// 1024 and 14 us at n = 21 (506 and 78 us when every thread unranked by 64-bit
// division and scanned all energies for their range).
constexpr int kSeedThreads = 1024;
constexpr int kSeedPer = 4;
constexpr int kSeedStates = kSeedPer * kSeedThreads;
constexpr int kSeedDescents = 8;

__global__ __launch_bounds__(kSeedThreads) void topk_seed_kernel(const Inst *__restrict__ inst,
                                                                 int32_t *gthr, int k)
{
    const Inst &I = *inst;
    const int n = I.n, A = I.A;
    const int tid = int(threadIdx.x), lane = tid % kWave, wave = tid / kWave;
    constexpr int kWaves = kSeedThreads / kWave;
    __shared__ int32_t T[kMaxVars * kMaxVars];   // T made symmetric
    __shared__ int32_t C[5][kWave];              // C[p][v] = binomial(v, p)
    __shared__ int32_t wE[kSeedDescents];
    __shared__ uint64_t wX[kSeedDescents];
    __shared__ int32_t d[kWave];
    __shared__ int32_t sg[kWave];
    __shared__ int32_t wLo[kWaves], wHi[kWaves], wN[kWaves];

    for (int e = tid; e < n * n; e += kSeedThreads) {
        const int i = e / n, j = e % n;
        if (i > j) continue;
        const int32_t t = I.T[e];
        T[e] = t;
        T[j * n + i] = t;
    }
    if (tid < kWave) {   // v <= 60: within int32
        const int v = tid;
        C[0][v] = 1;
        C[1][v] = v;
        C[2][v] = v * (v - 1) / 2;
        C[3][v] = v * (v - 1) / 2 * (v - 2) / 3;
        C[4][v] = v < 4 ? 0 : v * (v - 1) / 2 * (v - 2) / 3 * (v - 3) / 4;
    }
    __syncthreads();
    // 1. the best local minimum of eight descents
    if (wave < kSeedDescents) {
        int32_t E;
        uint64_t xm;
        greedy_descent(T, n, uint32_t(wave), E, xm);
        if (lane == 0) {
            wE[wave] = E;
            wX[wave] = xm;
        }
    }
    __syncthreads();
    int32_t bE = wE[0];
    uint64_t xm = wX[0];
    for (int w = 1; w < kSeedDescents; w++)
        if (wE[w] < bE || (wE[w] == bE && wX[w] < xm)) {
            bE = wE[w];
            xm = wX[w];
        }
    // 2. single-flip changes and signs at x*, one thread per variable
    if (tid < n) {
        const int xl = int((xm >> tid) & 1);
        int32_t f = T[tid * n + tid];
        for (int j = 0; j < n; j++) f += (j != tid && ((xm >> j) & 1)) ? T[j * n + tid] : 0;
        d[tid] = xl ? -f : f;
        sg[tid] = xl ? -1 : 1;
    }
    // 3. the states with 0..4 prefix variables flipped
    int32_t total = 0;
    for (int p = 0; p <= 4; p++) total += C[p][A];
    const int M = min(total, kSeedStates);
    if (M < k) return;   // fewer distinct rows than k: no bound
    __syncthreads();
    int32_t Ec[kSeedPer];
    int32_t lo32 = INT32_MAX, hi32 = INT32_MIN;
#pragma unroll
    for (int q = 0; q < kSeedPer; q++) {
        const int c = tid + q * kSeedThreads;
        int32_t e = bE;
        if (c < M) {
            int p = 0, rank = c;
            while (rank >= C[p][A]) rank -= C[p++][A];
            // colex unranking: the largest x with C(x, r) <= rank, from r = p
            int v[4] = {0, 0, 0, 0};
#pragma unroll
            for (int r = 4; r >= 1; r--) {
                if (r > p) continue;
                int x = 0;
#pragma unroll
                for (int bit = 32; bit >= 1; bit >>= 1)
                    if (x + bit < A && C[r][x + bit] <= rank) x += bit;
                rank -= C[r][x];
                v[r - 1] = x;
            }
#pragma unroll
            for (int a = 0; a < 4; a++) {
                if (a >= p) continue;
                e += d[v[a]];
#pragma unroll
                for (int b = 0; b < a; b++) e += sg[v[b]] * sg[v[a]] * T[v[b] * n + v[a]];
            }
            lo32 = min(lo32, e);
            hi32 = max(hi32, e);
        }
        Ec[q] = c < M ? e : INT32_MAX;
    }
    lo32 = wave_min(lo32);
    hi32 = -1 - wave_min(-1 - hi32);
    if (lane == 0) {
        wLo[wave] = lo32;
        wHi[wave] = hi32;
    }
    __syncthreads();
    // 4. the k-th smallest of the M energies: the least value v with at
    //    least k energies <= v
    int64_t lo = wLo[0], hi = wHi[0];
    for (int w = 1; w < kWaves; w++) {
        lo = min(lo, int64_t(wLo[w]));
        hi = max(hi, int64_t(wHi[w]));
    }
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        const int32_t m32 = int32_t(mid);
        int cnt = 0;
#pragma unroll
        for (int q = 0; q < kSeedPer; q++)
            cnt += int(__builtin_popcountll(__builtin_amdgcn_ballot_w64(Ec[q] <= m32)));
        __syncthreads();   // the counts of the last round have been read
        if (lane == 0) wN[wave] = cnt;
        __syncthreads();
        int sum = 0;
#pragma unroll
        for (int w = 0; w < kWaves; w++) sum += wN[w];
        if (sum >= k) hi = mid;
        else lo = mid + 1;
    }
    if (tid == 0) atomicMin(gthr, int32_t(lo));
}

}  // namespace

hipError_t launch_topk_seed(const Inst *d_inst, int32_t *d_gthr, int k, hipStream_t stream)
{
    if (k < 2 || k > kSeedStates) return hipErrorInvalidValue;
    hipLaunchKernelGGL(topk_seed_kernel, dim3(1), dim3(kSeedThreads), 0, stream, d_inst, d_gthr, k);
    return hipGetLastError();
}

hipError_t launch_topk_finish(const Inst *d_inst, const Inst &hI, const TopkBufs &buf, int k,
                              const TopkResults &to, unsigned long long *d_counters,
                              hipStream_t stream)
{
    if (hI.direct) d_counters = nullptr;
    if (k < 2 || k > kSelThreads) return hipErrorInvalidValue;
    SelArgs st{};
    if (hI.direct) {
        const uint32_t N = 1u << hI.n;
        const uint32_t blocks = (N + 255) / 256;
        hipLaunchKernelGGL(topk_direct_kernel, dim3(blocks), dim3(256), 0, stream, d_inst, buf.stE,
                           buf.stI, buf.segCount);
        st.count = buf.segCount;     // 2^n
        st.mult = 1;
    } else {
        // the lists' entries at or below the final shared bound, densely
        const int lists_per_block = 256 / kWave;
        const int blocks = (buf.waves + lists_per_block - 1) / lists_per_block;
        if (blocks > 0)
            hipLaunchKernelGGL(topk_compact_kernel, dim3(blocks), dim3(256), 0, stream,
                               buf.walk.listE, buf.walk.listR, buf.walk.listCount, buf.waves, k,
                               buf.walk.gthr, buf.candE, buf.candR, buf.candN, d_counters);
        SelArgs ch{};
        ch.E = buf.candE;
        ch.R = buf.candR;
        ch.count = buf.candN;
        ch.mult = 1;
        ch.k = k;
        ch.oE = buf.chunkE;
        ch.oR = buf.chunkR;
        ch.oCount = buf.chunkCount;
        ch.clear = buf.segCount;     // [0]: the rescan's state counter
        hipLaunchKernelGGL(topk_select_kernel, dim3(1), dim3(kSelThreads), 0, stream, ch);
        hipLaunchKernelGGL(topk_rescan_kernel, dim3((k + kRescanWaves - 1) / kRescanWaves),
                           dim3(kRescanWaves * kWave), 0, stream, d_inst, buf.chunkR, buf.chunkCount,
                            k, buf.stE, buf.stI, buf.segCount);
        st.count = buf.segCount;     // states kept by the rescan, densely
        st.mult = 1;
    }
    st.E = buf.stE;
    st.R = buf.stI;
    st.k = k;
    st.oE = buf.selE;
    st.oR = buf.selR;
    st.oCount = buf.selCount;
    hipLaunchKernelGGL(topk_select_kernel, dim3(1), dim3(kSelThreads), 0, stream, st);
    hipLaunchKernelGGL(topk_final_kernel, dim3((k + kWave - 1) / kWave),
                       dim3(kFinalWaves * kWave), 0, stream, d_inst, buf.selE, buf.selR, buf.selCount, k, hI.Qf ? buf.out : to.topk,
                       to.best, d_counters, buf.walk.prep, to.prep);
    if (hI.Qf)
        hipLaunchKernelGGL(topk_order_kernel, dim3(1), dim3(kSelThreads), 0, stream, buf.selCount, k,
                           buf.out, to.topk, to.best);
    return hipGetLastError();
}

}  // namespace qk
