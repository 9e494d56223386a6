// Skip-gram with negative sampling for small minibatches (Train of
// Algorithm 1; Eq. (1)-(2)): P (K + 2) <= 8192 touches per minibatch, the
// shape of the 1,024-pair configurations.
//
// At that size a minibatch moves a few MB, so the per-minibatch launch chain
// of sgns.hip (ids, two scan passes, forward, two apply launches) is bound by
// launch and cache-flush latency, not by HBM.  Here the work splits in two:
//
//   plan    one workgroup per minibatch, many minibatches per launch.  It
//           draws the minibatch's node ids (walk reads, noise draws), sorts
//           its touches by (table, row) with a stable radix sort in LDS and
//           lists the rows' segments.  Touches of a row keep touch order,
//           which is pair order (pair, then slot), so no global atomics and
//           no per-row counters are needed.  Plans depend only on the walks
//           and the noise table, never on the embeddings.
//   update  one persistent cooperative launch for those minibatches.  Per
//           minibatch: the forward (gathers, FP64 dots, sigma, coefficients;
//           each out-touch's coefficient at its sorted position; the context
//           row copied for pairs with an out row touched more than once; rows
//           touched once in either table updated in place), a grid barrier,
//           the apply (one 16-lane group per segment of two or more touches
//           sums the row's terms and adds them once), and a grid barrier.
//           The apply reads the context copies, not the in-table, so in and
//           out rows are applied together.
//
// The arithmetic is that of sgns.hip term for term: rows of at most kChunk
// touches sum their FP64 terms sequentially in pair order, longer rows sum
// terms rounded onto the exact-sum grid, every stored value is rounded once.
// The two paths therefore give bit-identical tables.
//
// The workgroups exchange rows, coefficients, deltas and context copies
// through agent-scope relaxed accesses of 8 bytes instead of release and
// acquire fences, which write back and invalidate each XCD's whole L2 at every
// barrier (the rows are read once per minibatch, so the L2 held little of use).
// With the forward of sgns_forward.h, and hubs' segments shared by a workgroup,
// per minibatch of 1,024 pairs: R-MAT 2^20, d = 128, 17.3 -> 10.7 us (forward
// phase 4.0, first barrier 1.6, apply 1.1, second barrier 3.3: it waits for the
// workgroups that have segments); 1,000 nodes, d = 64, 18.8 -> 10.1.  A
// minibatch is two dependent trips to memory, the arithmetic between them and
// two barriers.
//
// The grid barrier is a flag per workgroup: each workgroup stores its barrier
// count to a flag on its own 128-byte line, and the first wave of every
// workgroup watches all the flags (one lane per flag).  Workgroup 0 gathering
// the flags and raising a go flag, and one shared atomic counter, whose
// same-address atomics serialise, were slower.  Workgroups and us per
// minibatch (R-MAT 2^20 / 1,000 nodes): 32 15.2 / 16.5, 64 11.9 / 12.6,
// 96 12.7 / 13.3, 128 12.8 / 13.5.  Every wait is
// bounded: one that exceeds kSpinLimit polls raises an abort flag that every
// workgroup checks, so every wave leaves the kernel, and the host reports the
// failure.
#include <algorithm>
#include <cmath>
#include <vector>

#include "common.h"
#include "noise.h"
#include "sgns_device.h"
#include "sgns_forward.h"

namespace felog {

// Values of one minibatch that the plan and update launches read.
struct MbDesc {
    int64_t vcol_base;     // offset of the minibatch's chunk in valid_cols
    uint32_t Wv;           // valid columns of the chunk
    uint32_t first_pair;   // first pair of the minibatch in its chunk
    uint32_t npairs;
    float lr;
    double grid_c;         // exact-sum grid constant of lr
};
static_assert(sizeof(MbDesc) == 32, "descriptor layout shared by host and device");

constexpr int kPlanThreads = 1024;
// touches a plan sorts in LDS: the persistent update's most, and twice that
// (136 KB of LDS) for planned launches
constexpr int kPlanMaxTouches = 2 * kSmallMaxTouches;
constexpr int32_t kPosMask = (1 << 30) - 1;
constexpr int32_t kSingleBit = 1 << 30;  // row touched once in the minibatch: the forward updates it
constexpr uint32_t kSpinLimit = 1u << 22;  // polls before a barrier wait gives up (seconds)
constexpr int kUpdThreads = 512;         // one workgroup per CU at two waves per SIMD
constexpr int kFlagStride = 32;          // 32-bit words between barrier flags (128 bytes)
constexpr int kDefaultUpdBlocks = 64;    // workgroups of the persistent launch by default

// ------------------------------------------------------------------- plan
struct PlanArgs {
    const int32_t* walks;          // step-major [L][W]
    int64_t W;
    const int32_t* vcols;
    const int32_t* slices;         // (j << 8) | slot
    int64_t id_base;
    int32_t window;
    uint64_t seed;
    NoiseTable noise;
    int32_t row_bits;              // n < 2^row_bits, at most 31
    const MbDesc* desc;            // [minibatches of the launch], or NULL: consecutive
                                   // minibatches of `pairs` pairs of one chunk, from `first`
    MbDesc first;
    uint32_t pairs, chunk_pairs;
    int32_t tmax;                  // touch slots per minibatch, P (K + 2)
    int2* tinfo;                   // [mb][tmax]: (row, sorted position | kSingleBit), -1 skipped
    int2* segs;                    // [mb][tmax / 2]: pack_seg of each segment, those of at
                                   // most kChunk touches from the front, the others from the
                                   // back
    uint16_t* spair;               // [mb][tmax]: pair of each sorted position
    uint32_t* meta;                // [mb][4]: segments of at most kChunk touches, longer ones,
                                   // out rows, out rows touched once
    unsigned long long* row_totals;// [3]: in rows, out rows, out rows touched once
};

// A segment: its row, and its first position (14 bits), its touches less one
// (14 bits) and its table in one word.
static_assert(kPlanMaxTouches <= 16384, "positions and touches of a segment take 14 bits");
__device__ __forceinline__ int2 pack_seg(int32_t row, uint32_t start, uint32_t len, uint32_t out)
{
    return make_int2(row, (int32_t)(start | ((len - 1u) << 14) | (out << 28)));
}
struct Seg {
    int32_t row, start, len;   // len 0: none
    bool out;
};
constexpr int32_t kNoSeg = -1;
__device__ __forceinline__ Seg unpack_seg(int2 s)
{
    if (s.x == kNoSeg) return Seg{0, 0, 0, false};
    return Seg{s.x, s.y & 16383, ((s.y >> 14) & 16383) + 1, (s.y >> 28) != 0};
}

// Plans of one launch: workgroups [start[j], start[j + 1]) plan the
// minibatches of job j (one model and corpus per job).
struct PlanBatch {
    PlanArgs job[kMaxBatchJobs];
    int32_t start[kMaxBatchJobs + 1];
    int32_t njobs;
};

constexpr int kPlanWaves = kPlanThreads / 64;
constexpr int kPlanBins = 256;                                // 8 key bits per sorting pass

// Sorts the workgroup's touches by the low `bits` of key, stably: pass by
// pass over 8 bits, every touch's new position is the number of touches
// before it in (digit, position) order.  Wave w holds positions
// [w R 64, (w + 1) R 64), one per lane and round, so counting a wave's rounds
// in turn keeps their order: a round finds each lane's peers of equal digit
// with eight ballots, and its first peer adds their number to the wave's bin.
// A bitonic network over the same 8,192 touches took 91 dependent passes
// through LDS (196 us of a one-minibatch plan).
template <int kPlanRounds>
__device__ __forceinline__ void sort_touches(uint32_t (&key)[kPlanRounds],
                                             uint32_t (&touch)[kPlanRounds], int R, int bits,
                                             uint32_t* skey, uint16_t* stouch,
                                             uint16_t (*bins)[kPlanBins], uint32_t* wave_sum)
{
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned long long lt = (1ull << lane) - 1ull;
    for (int shift = 0; shift < bits; shift += 8) {
        // (opaque, so that the rounds' addresses are not all kept across passes)
        uint32_t at0 = (uint32_t)(w * R * 64 + lane);
        asm volatile("" : "+v"(at0));
        for (int b = lane; b < kPlanBins; b += 64) bins[w][b] = 0;
        uint32_t rank[kPlanRounds];   // touches of the same digit before this one in the wave
#pragma unroll
        for (int r = 0; r < kPlanRounds; ++r) {
            rank[r] = 0;
            if (r < R) {
                const uint32_t d = (key[r] >> shift) & (kPlanBins - 1);
                unsigned long long peers = ~0ull;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const bool set = (d >> i) & 1u;
                    const unsigned long long m = __ballot(set);
                    peers &= set ? m : ~m;
                }
                const uint32_t before = bins[w][d];
                const uint32_t mine = (uint32_t)__popcll(peers & lt);
                rank[r] = before + mine;
                __builtin_amdgcn_wave_barrier();
                if (mine == 0) bins[w][d] = (uint16_t)(before + (uint32_t)__popcll(peers));
                __builtin_amdgcn_wave_barrier();
            }
            __builtin_amdgcn_sched_barrier(0);   // one round's ballots live at a time
        }
        __syncthreads();
        // thread b < 256: bin b's touches over the waves, then an exclusive scan over the bins
        uint32_t total = 0;
        if (threadIdx.x < kPlanBins) {
#pragma unroll
            for (int i = 0; i < kPlanWaves; ++i) {
                const uint32_t c = bins[i][threadIdx.x];
                bins[i][threadIdx.x] = (uint16_t)total;
                total += c;
            }
        }
        uint32_t incl = total;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(incl, off);
            if (lane >= off) incl += y;
        }
        if (threadIdx.x < kPlanBins && lane == 63) wave_sum[w] = incl;
        __syncthreads();
        if (threadIdx.x < kPlanBins) {
            uint32_t base = incl - total;
            for (int i = 0; i < w; ++i) base += wave_sum[i];
#pragma unroll
            for (int i = 0; i < kPlanWaves; ++i)
                bins[i][threadIdx.x] = (uint16_t)(bins[i][threadIdx.x] + base);
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kPlanRounds; ++r)
            if (r < R) {
                const uint32_t at = bins[w][(key[r] >> shift) & (kPlanBins - 1)] + rank[r];
                skey[at] = key[r];
                stouch[at] = (uint16_t)touch[r];
            }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kPlanRounds; ++r)
            if (r < R) {
                key[r] = skey[at0 + 64 * r];
                touch[r] = stouch[at0 + 64 * r];
            }
    }
}

template <int K, int MAXT>
__global__ __launch_bounds__(kPlanThreads) void sgns_plan_kernel(PlanBatch pb)
{
    constexpr int T = K + 2;
    constexpr int kPlanRounds = MAXT / kPlanThreads;   // most touches per thread
    int jb = 0;
    while (jb + 1 < pb.njobs && (int32_t)blockIdx.x >= pb.start[jb + 1]) ++jb;
    const PlanArgs& a = pb.job[jb];
    const uint32_t lb = blockIdx.x - (uint32_t)pb.start[jb];   // minibatch within the job's group
    __shared__ uint32_t skey[MAXT + 1];
    __shared__ uint16_t stouch[MAXT];
    __shared__ uint16_t bins[kPlanWaves][kPlanBins];
    __shared__ uint16_t seg_lo[MAXT / 2], seg_hi[MAXT / 2];
    __shared__ uint32_t wave_sum[kPlanWaves], wave_end[kPlanWaves];
    __shared__ uint32_t counts[5];   // rows, in rows, out rows touched once, segments of at most
                                     // kChunk touches, longer ones
    MbDesc d = a.first;
    if (a.desc) {
        d = a.desc[lb];
    } else {
        d.first_pair += lb * a.pairs;
        d.npairs = min(a.pairs, a.chunk_pairs - d.first_pair);
    }
    const uint32_t nt = d.npairs * T;       // nt <= MAXT (checked on the host)
    // rounds: as many as the minibatch needs, or all (with 16 conditional rounds
    // the arrays below do not stay in registers)
    const int R = MAXT > kSmallMaxTouches ? kPlanRounds
                                          : (int)((nt + kPlanThreads - 1) / kPlanThreads);
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int2* tinfo = a.tinfo + (int64_t)lb * a.tmax;
    int2* segs = a.segs + (int64_t)lb * (a.tmax / 2);
    uint16_t* spair = a.spair + (int64_t)lb * a.tmax;
    const int32_t* vcols = a.vcols + d.vcol_base;
    const uint32_t none = (2u << a.row_bits) - 1u;   // above every real key
    if (threadIdx.x < 5) counts[threadIdx.x] = 0;

    // 1. each touch's key, table << row_bits | row.  One thread per pair: its
    //    walk reads and its negatives' guide entries are in flight together
    //    (negative k of a pair: Philox(walk id, (j << 8) | slot, NEG | k / 2),
    //    words 2 (k mod 2) and 2 (k mod 2) + 1), then the cumulative weights.
    for (uint32_t t = nt + threadIdx.x; t < (uint32_t)R * kPlanThreads; t += kPlanThreads)
        skey[t] = none;
    for (uint32_t p = threadIdx.x; p < d.npairs; p += kPlanThreads) {
        const uint32_t gq = d.first_pair + p;
        const uint32_t sidx = gq / d.Wv;
        const uint32_t rank = gq - sidx * d.Wv;
        const int32_t js = a.slices[sidx];
        const int32_t col = vcols[rank];
        const int32_t j = js >> 8, s = js & 255;
        const int32_t off = s < a.window ? s - a.window : s - a.window + 1;
        const int32_t ctr = a.walks[(int64_t)j * a.W + col];
        const int32_t ctx = a.walks[(int64_t)(j + off) * a.W + col];
        const int64_t wid = a.id_base + col;
        uint64_t u[K];
        int32_t neg[K];
        Rand4 x{};
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if ((k & 1) == 0)
                x = philox4x32((uint32_t)wid, (uint32_t)(wid >> 32), (uint32_t)js,
                               kTagNeg | (uint32_t)(k >> 1), a.seed);
            u[k] = ((uint64_t)((k & 1) ? x.v[3] : x.v[1]) << 32) | ((k & 1) ? x.v[2] : x.v[0]);
            neg[k] = a.noise.guide[u[k] >> (64 - a.noise.bits)];
            u[k] = __umul64hi(u[k], a.noise.total);
        }
        uint64_t c[K];
#pragma unroll
        for (int k = 0; k < K; ++k) c[k] = a.noise.cdf[neg[k] + 1];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (c[k] <= u[k]) {
                ++neg[k];
                while (a.noise.cdf[neg[k] + 1] <= u[k]) ++neg[k];
            }
        }
        skey[p * T] = (uint32_t)ctx;
        skey[p * T + 1] = (1u << a.row_bits) | (uint32_t)ctr;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const bool skip = neg[k] == ctr;   // a negative equal to the centre is skipped
            skey[p * T + 2 + k] = skip ? none : (1u << a.row_bits) | (uint32_t)neg[k];
            if (skip) tinfo[p * T + 2 + k] = make_int2(-1, -1);
        }
    }
    __syncthreads();

    // 2. sort by (table, row), touches of a row in touch (pair, then slot) order
    uint32_t key[kPlanRounds], touch[kPlanRounds];
#pragma unroll
    for (int r = 0; r < kPlanRounds; ++r) {
        key[r] = none;
        touch[r] = 0;
        if (r < R) {
            touch[r] = (uint32_t)((w * R + r) * 64 + lane);
            key[r] = skey[touch[r]];
        }
    }
    __syncthreads();
    sort_touches(key, touch, R, a.row_bits + 1, skey, stouch, bins, wave_sum);

    // 3. a position is its row's first or last where its neighbour's key
    //    differs.  Rows touched once are updated by the forward; the k-th
    //    first and the k-th last position of the others bound segment k.
    //    In-table rows sort first.
    if (threadIdx.x == 0) skey[(uint32_t)R * kPlanThreads] = none;
    __syncthreads();
    const unsigned long long lt = (1ull << lane) - 1ull;
    uint32_t nfirst = 0, nlast = 0, c_seg = 0, c_in = 0, c_single = 0;
    uint32_t bits_first = 0, bits_last = 0;   // per round: this lane starts / ends a segment
#pragma unroll
    for (int r = 0; r < kPlanRounds; ++r)
        if (r < R) {
            const int i = (w * R + r) * 64 + lane;
            const bool real = key[r] != none;
            const bool first = real && (i == 0 || skey[i - 1] != key[r]);
            const bool last = real && skey[i + 1] != key[r];
            const bool out = (key[r] >> a.row_bits) != 0;
            if (real) {
                const uint32_t t = touch[r];
                const int32_t row = (int32_t)(key[r] & ((1u << a.row_bits) - 1u));
                tinfo[t] = make_int2(row, i | (first && last ? kSingleBit : 0));
                spair[i] = (uint16_t)(t / T);
            }
            c_seg += first ? 1u : 0u;
            c_in += first && !out ? 1u : 0u;
            c_single += first && last && out ? 1u : 0u;
            const bool f = first && !last, l = last && !first;
            bits_first |= (f ? 1u : 0u) << r;
            bits_last |= (l ? 1u : 0u) << r;
            nfirst += (uint32_t)__popcll(__ballot(f));
            nlast += (uint32_t)__popcll(__ballot(l));
        }
    if (c_seg) atomicAdd(&counts[0], c_seg);
    if (c_in) atomicAdd(&counts[1], c_in);
    if (c_single) atomicAdd(&counts[2], c_single);
    if (lane == 0) {
        wave_sum[w] = nfirst;
        wave_end[w] = nlast;
    }
    __syncthreads();
    uint32_t at_first = 0, at_last = 0, n_apply = 0;
#pragma unroll
    for (int i = 0; i < kPlanWaves; ++i) {
        at_first += i < w ? wave_sum[i] : 0u;
        at_last += i < w ? wave_end[i] : 0u;
        n_apply += wave_sum[i];
    }
#pragma unroll
    for (int r = 0; r < kPlanRounds; ++r)
        if (r < R) {
            const uint16_t i = (uint16_t)((w * R + r) * 64 + lane);
            const bool f = (bits_first >> r) & 1u, l = (bits_last >> r) & 1u;
            const unsigned long long mf = __ballot(f), ml = __ballot(l);
            if (f) seg_lo[at_first + (uint32_t)__popcll(mf & lt)] = i;
            if (l) seg_hi[at_last + (uint32_t)__popcll(ml & lt)] = i;
            at_first += (uint32_t)__popcll(mf);
            at_last += (uint32_t)__popcll(ml);
        }
    __syncthreads();
    // (the order of the lists does not matter: no two segments share a row)
    for (uint32_t q = threadIdx.x; q < n_apply; q += kPlanThreads) {
        const uint32_t f = seg_lo[q], x = skey[f], len = seg_hi[q] - f + 1u;
        const bool is_long = len > (uint32_t)kChunk;
        const uint32_t at = atomicAdd(&counts[is_long ? 4 : 3], 1u);
        segs[is_long ? (uint32_t)(a.tmax / 2) - 1u - at : at] =
            pack_seg((int32_t)(x & ((1u << a.row_bits) - 1u)), f, len, x >> a.row_bits);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t* m = a.meta + (int64_t)lb * 4;
        m[0] = counts[3];
        m[1] = counts[4];
        m[2] = counts[0] - counts[1];
        m[3] = counts[2];
        atomicAdd(&a.row_totals[0], (unsigned long long)counts[1]);
        atomicAdd(&a.row_totals[1], (unsigned long long)(counts[0] - counts[1]));
        atomicAdd(&a.row_totals[2], (unsigned long long)counts[2]);
    }
}

// ----------------------------------------------------------------- update
// One job's part of an update launch.
struct UpdJob {
    float* tin;
    float* tout;
    const MbDesc* desc;            // [nmb]
    const int2* tinfo;             // [nmb][tmax]
    const int2* segs;              // [nmb][tmax / 2]
    const uint32_t* meta;          // [nmb][4]
    const uint16_t* spair;         // [nmb][tmax]: pair of each sorted position
    double* gpos;                  // [tmax]: FP64 coefficient of each out-touch, by position
    float* dinp;                   // [P][D]: each pair's in-row delta, by sorted position
    float* ctxc;                   // [P][D]: each pair's context row at the minibatch start
    double* loss_part;             // [waves]
    int32_t tmax;
    int32_t nmb;
};

// An update launch over the minibatches of up to kMaxBatchJobs jobs (equal d
// and K): phase by phase, minibatch m of every job that has one.  The jobs'
// tables are distinct, so their minibatches share each phase and its
// barriers.
struct UpdArgs {
    UpdJob job[kMaxBatchJobs];
    int32_t njobs;
    int32_t nmb_max;               // largest nmb of the jobs
    uint32_t* flags;               // workgroup b's at [kFlagStride (1 + b)] (the first line is
                                   // unused); zero at the call's start
    uint32_t epoch0;               // barriers passed by earlier launches of the call
    int32_t* abort;
    unsigned long long* clocks;    // null, or [4]: device wall-clock ticks of the forward,
                                   // the first barrier, the apply and the second barrier,
                                   // summed over workgroups and minibatches
};

// Bounded wait until *p >= target; false (and the abort flag raised) when
// the wait gives up or another workgroup has raised it.
__device__ __forceinline__ bool wait_at_least(const uint32_t* p, uint32_t target, int32_t* abort)
{
    uint32_t polls = 0;
    while (__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
        if (++polls > kSpinLimit) {
            __hip_atomic_store(abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
        if ((polls & 255) == 0 && __hip_atomic_load(abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            return false;
        __builtin_amdgcn_s_sleep(1);
    }
    return true;
}

// Grid barrier.  What the workgroups exchange (table rows, coefficients,
// deltas, context copies) goes through agent-scope relaxed atomics, which no
// cache holds back, so a barrier needs only that every wave's accesses have
// completed before its workgroup's flag is raised.  A release and an acquire
// fence at agent scope write back and invalidate the whole L2 instead.
// Returns false when the launch is aborting (a wait exceeded its bound).
__device__ __forceinline__ bool grid_sync(const UpdArgs& a, uint32_t& epoch,
                                          unsigned long long* arrive)
{
    __shared__ int s_ok;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (arrive) *arrive = wall_clock64();   // every wave of the workgroup is here
    ++epoch;
    if (threadIdx.x == 0)
        __hip_atomic_store(&a.flags[kFlagStride * (1 + blockIdx.x)], epoch, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    // every workgroup's first wave watches every flag (lane l the flags of
    // workgroups l, l + 64, ...)
    if (threadIdx.x < 64) {
        bool ok = true;
        for (uint32_t b = threadIdx.x; b < gridDim.x; b += 64)
            ok = ok && wait_at_least(&a.flags[kFlagStride * (1 + b)], epoch, a.abort);
        const bool all_ok = __all(ok);
        if (threadIdx.x == 0) s_ok = all_ok;
    }
    __syncthreads();
    asm volatile("" ::: "memory");
    return s_ok != 0;
}

// Touch l of the pairs [q0, q0 + S H) of minibatch m, or -1.
template <int K>
__device__ __forceinline__ int2 touch_of(const UpdJob& J, int m, uint32_t np, uint32_t q0,
                                         uint32_t pairs)
{
    const int lane = threadIdx.x & 63;
    if (q0 < np && lane < (int)min(pairs, np - q0) * (K + 2))
        return J.tinfo[(int64_t)m * J.tmax + (int64_t)q0 * (K + 2) + lane];
    return make_int2(-1, -1);
}

// Forward of one batch of pairs of minibatch m, from pair q0; `touch` is
// touch_of those pairs.
template <int D, int K, int S, RowAccess A>
__device__ __forceinline__ void forward_pairs(const UpdJob& J, uint32_t npairs, uint32_t q0,
                                              int2 touch, double lr, double& lacc)
{
    using Batch = FwdBatch<D, K, S, A>;
    constexpr int T = K + 2, H = Batch::H, L = Batch::L, V = Batch::V;
    const int lane = threadIdx.x & 63;
    const uint32_t gl = lane & (L - 1);
    const int np = (int)min((uint32_t)(S * H), npairs - q0);
    const int32_t m_row = touch.x, m_code = touch.y;
    const unsigned long long single = __ballot(m_code >= 0 && (m_code & kSingleBit));
    const unsigned long long shared = __ballot(m_code >= 0 && !(m_code & kSingleBit));
    Batch bt;
    bt.load(J.tin, J.tout, m_row, 0, np);
    bt.coefficients(m_row, 0, np, lr, lacc);
    {
        // coefficients of the out-touches (not of the rows touched once)
        const int32_t code = __shfl(m_code, bt.touch);
        if (bt.mine && !(code & kSingleBit)) {
            double* gp = &J.gpos[code & kPosMask];
            if constexpr (A == kAgent)
                __hip_atomic_store(gp, bt.g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else
                *gp = bt.g;
        }
    }
#pragma unroll
    for (int b = 0; b < S; ++b) {
        const int p = b * H + (H == 2 ? lane >> 5 : 0);
        const bool live = p < np;
        const int src = (live ? p : 0) * T;
        double gk[K + 1];
#pragma unroll
        for (int k = 0; k <= K; ++k) gk[k] = bt.coef(b, k);
        // out rows touched once: row + g in[ctx] in FP64, rounded once
#pragma unroll
        for (int k = 0; k <= K; ++k) {
            if (live && bt.row[b][k] >= 0 && ((single >> (src + 1 + k)) & 1ull)) {
                f2* dst = reinterpret_cast<f2*>(J.tout + (int64_t)bt.row[b][k] * D);
#pragma unroll
                for (int i = 0; i < V; ++i)
                    store_row2<A>(row_at(dst, i * L + gl), bt.out_row(b, i, gk[k], bt.vo[b][k][i]));
            }
        }
        const int32_t pos_in = __shfl(m_code, src) & kPosMask;
        if (live) {
            // the context copy is read by the apply of the pair's out rows
            // touched more than once; an in row touched once is updated here
            // (its delta rounded to FP32 first, as the apply rounds the stored
            // delta), others store the delta
            const bool need_ctx = ((shared >> (src + 1)) & ((1ull << (K + 1)) - 1ull)) != 0;
            const bool in_single = (single >> src) & 1ull;
            f2 o[V];
            bt.in_delta(b, gk, o);
            if (need_ctx) {
                f2* cc = reinterpret_cast<f2*>(J.ctxc + (int64_t)(q0 + (uint32_t)p) * D);
#pragma unroll
                for (int i = 0; i < V; ++i) store_row2<A>(row_at(cc, i * L + gl), bt.vin[b][i]);
            }
            f2* dp = reinterpret_cast<f2*>(in_single ? J.tin + (int64_t)bt.ctx[b] * D
                                                     : J.dinp + (int64_t)pos_in * D);
#pragma unroll
            for (int i = 0; i < V; ++i) {
                f2 v = o[i];
                if (in_single)
                    v = f2{(float)((double)bt.vin[b][i].x + (double)o[i].x),
                           (float)((double)bt.vin[b][i].y + (double)o[i].y)};
                store_row2<A>(row_at(dp, i * L + gl), v);
            }
        }
    }
}

// Rows in flight per 16-lane group of an apply: 8 of up to 16 float2s per lane.
template <int D>
constexpr int apply_rows() { return D == 256 ? 4 : 8; }

// Coefficient of the out-touch at a sorted position.
template <RowAccess A>
__device__ __forceinline__ double load_coef(const double* p)
{
    if constexpr (A == kAgent)
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        return *p;
}

// Adds to acc the terms of touches [i0, i0 + R) of a 16-lane group's nb.
// g, src: in lane l of the group, touch l's coefficient and source row (out
// rows: its pair's context copy; in rows: 1 and the pair's delta).  No load is
// issued for slots past nb: pointing them at row 0 made every short segment
// read the same line, which queued in one memory channel.
template <int D, RowAccess A, int R, bool EXACT>
__device__ __forceinline__ void add_terms(const float* srcb, double g, int32_t src, int32_t i0,
                                          int32_t nb, double gc, double (&acc)[D / 16])
{
    constexpr int V = D / 32;        // float2s per lane and row
    const int g0 = threadIdx.x & 48, l16 = threadIdx.x & 15;
    f2 x[R][V];
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const int32_t rr = __shfl(src, g0 + min(i0 + u, 15));
        const f2* rp = reinterpret_cast<const f2*>(srcb + (int64_t)rr * D);
#pragma unroll
        for (int i = 0; i < V; ++i) x[u][i] = f2{0.0f, 0.0f};
        if (i0 + u < nb) {
#pragma unroll
            for (int i = 0; i < V; ++i) x[u][i] = load_row2<A>(rp + i * 16 + l16);
        }
    }
    double gg[R];
#pragma unroll
    for (int u = 0; u < R; ++u) gg[u] = __shfl(g, g0 + min(i0 + u, 15));
#pragma unroll
    for (int u = 0; u < R; ++u) {
        if (i0 + u >= nb) break;
#pragma unroll
        for (int i = 0; i < V; ++i) {
            if (EXACT) {
                // order-free: each term rounded onto the grid, sums exact
                acc[2 * i] += on_grid(gg[u] * (double)x[u][i].x, gc);
                acc[2 * i + 1] += on_grid(gg[u] * (double)x[u][i].y, gc);
            } else {
                // in rows: g = 1, and 1 * x + acc is exactly x + acc
                acc[2 * i] = fma(gg[u], (double)x[u][i].x, acc[2 * i]);
                acc[2 * i + 1] = fma(gg[u], (double)x[u][i].y, acc[2 * i + 1]);
            }
        }
    }
}

// Adds a segment's terms, in touch order, to its row: one 16-lane group, at
// most kChunk touches (none: len 0).  pair0: in lane l, the pair of touch l
// (out segments).  A whole wave per segment, with all 16 touches in flight,
// was slower (the apply 1.1 -> 3.2 us per workgroup on R-MAT 2^20, 2.9 -> 9.6
// on 1,000 nodes).
template <int D, RowAccess A>
__device__ __forceinline__ void apply_short(const UpdJob& J, const Seg& seg, int32_t pair0)
{
    constexpr int V = D / 32, R = apply_rows<D>();
    if (seg.len == 0) return;        // whole groups leave
    const int l16 = threadIdx.x & 15;
    f2* const table = reinterpret_cast<f2*>((seg.out ? J.tout : J.tin) + (int64_t)seg.row * D);
    f2 cur[V];
#pragma unroll
    for (int i = 0; i < V; ++i) cur[i] = load_row2<A>(table + i * 16 + l16);
    const double g = seg.out && l16 < seg.len ? load_coef<A>(&J.gpos[seg.start + l16]) : 1.0;
    const int32_t src = seg.out ? pair0 : seg.start + l16;
    double acc[2 * V];
#pragma unroll
    for (int e = 0; e < 2 * V; ++e) acc[e] = 0.0;
    for (int32_t i0 = 0; i0 < seg.len; i0 += R)
        add_terms<D, A, R, false>(seg.out ? J.ctxc : J.dinp, g, src, i0, seg.len, 0.0, acc);
#pragma unroll
    for (int i = 0; i < V; ++i)
        store_row2<A>(table + i * 16 + l16, f2{(float)((double)cur[i].x + acc[2 * i]),
                                               (float)((double)cur[i].y + acc[2 * i + 1])});
}

// A segment of more than kChunk touches: the whole workgroup, whose 16-lane
// groups take 16 touches each in turn.  The terms are rounded onto the
// exact-sum grid, so the groups' sums add up in any order.  A hub's segment
// (hundreds of touches of a 1,024-pair minibatch on a power-law graph of 700
// nodes) took one group 20 us.  part: NW D doubles of LDS.
template <int D, RowAccess A, int NW>
__device__ __forceinline__ void apply_long(const UpdJob& J, const uint16_t* sp, const Seg& seg,
                                           double gc, double* part)
{
    constexpr int V = D / 32, R = apply_rows<D>();
    const int lane = threadIdx.x & 63, l16 = lane & 15;
    f2* const table = reinterpret_cast<f2*>((seg.out ? J.tout : J.tin) + (int64_t)seg.row * D);
    f2 cur = f2{0.0f, 0.0f};
    if (threadIdx.x < D / 2) cur = load_row2<A>(table + threadIdx.x);
    double acc[2 * V];
#pragma unroll
    for (int e = 0; e < 2 * V; ++e) acc[e] = 0.0;
    for (int32_t b0 = (int32_t)(threadIdx.x >> 4) * 16; b0 < seg.len; b0 += NW * 64) {
        const int32_t nb = min(16, seg.len - b0), at = seg.start + b0 + l16;
        double g = 1.0;
        int32_t src = at;
        if (seg.out && l16 < nb) {
            g = load_coef<A>(&J.gpos[at]);
            src = sp[at];
        }
        for (int32_t i0 = 0; i0 < nb; i0 += R)
            add_terms<D, A, R, true>(seg.out ? J.ctxc : J.dinp, g, src, i0, nb, gc, acc);
    }
#pragma unroll
    for (int e = 0; e < 2 * V; ++e) acc[e] = xor_sum<32>(xor_sum<16>(acc[e]));
    double* mine = part + (threadIdx.x >> 6) * D;
    if (lane < 16)
#pragma unroll
        for (int i = 0; i < V; ++i) {
            mine[2 * (i * 16 + l16)] = acc[2 * i];
            mine[2 * (i * 16 + l16) + 1] = acc[2 * i + 1];
        }
    __syncthreads();
    if (threadIdx.x < D / 2) {
        double x = 0.0, y = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            x += part[w * D + 2 * threadIdx.x];
            y += part[w * D + 2 * threadIdx.x + 1];
        }
        store_row2<A>(table + threadIdx.x, f2{(float)((double)cur.x + x), (float)((double)cur.y + y)});
    }
    __syncthreads();
}

// Item `item` of minibatch m's apply: a long segment, or one short segment
// per 16-lane group.  Items [0, n_long) are the long ones.
template <int NW>
__device__ __forceinline__ int2 short_seg(const UpdJob& J, int m, uint32_t item)
{
    const uint32_t nshort = J.meta[(int64_t)m * 4], nlong = J.meta[(int64_t)m * 4 + 1];
    const uint32_t q = (item - nlong) * (NW * 4) + (threadIdx.x >> 4);
    return item >= nlong && q < nshort ? J.segs[(int64_t)m * (J.tmax / 2) + q] : make_int2(kNoSeg, 0);
}
__device__ __forceinline__ int32_t short_pair(const UpdJob& J, int m, const Seg& sd)
{
    const int l16 = threadIdx.x & 15;
    return sd.out && l16 < sd.len ? J.spair[(int64_t)m * J.tmax + sd.start + l16] : 0;
}

// Every item of minibatch m from `first` on.  ahead, pair0: short_seg and
// short_pair of the first item.
template <int D, RowAccess A, int NW>
__device__ __forceinline__ void apply_items(const UpdJob& J, int m, uint32_t first, uint32_t stride,
                                            int2 ahead, int32_t pair0, double gc, double* part)
{
    const uint32_t nshort = J.meta[(int64_t)m * 4], nlong = J.meta[(int64_t)m * 4 + 1];
    const uint32_t items = nlong + (nshort + NW * 4 - 1) / (NW * 4);
    for (uint32_t item = first; item < items; item += stride) {
        if (item < nlong) {
            const Seg sd = unpack_seg(J.segs[(int64_t)m * (J.tmax / 2) + (J.tmax / 2) - 1 - item]);
            apply_long<D, A, NW>(J, J.spair + (int64_t)m * J.tmax, sd, gc, part);
            continue;
        }
        if (item != first) {
            ahead = short_seg<NW>(J, m, item);
            pair0 = short_pair(J, m, unpack_seg(ahead));
        }
        apply_short<D, A>(J, unpack_seg(ahead), pair0);
    }
}

// Steps of pairs per forward batch of the persistent update: two pairs per
// wave, so that 1,024 pairs occupy every wave of the 64 workgroups.
template <int D, int K>
constexpr int upd_steps() { return D == 64 || fwd_max_steps(D, K) < 2 ? 1 : 2; }

template <int D, int K>
__global__ __launch_bounds__(kUpdThreads) void sgns_small_update_kernel(UpdArgs a)
{
    constexpr int S = upd_steps<D, K>();
    constexpr uint32_t G = S * FwdShape<D, K>::kHalves;   // pairs per wave at a time
    constexpr int NW = kUpdThreads / 64;
    __shared__ double part[NW * D];
    const int lane = threadIdx.x & 63;
    const uint32_t nw = gridDim.x * (blockDim.x >> 6);
    const uint32_t gw = blockIdx.x * (blockDim.x >> 6) +
                        (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t epoch = a.epoch0;
    double lacc = 0.0;
    // plan data of job 0's next phase, loaded a phase ahead: this lane's touch
    // of the wave's first batch (forward) and the group's first segment with
    // the pair of each of its first 16 positions (apply)
    const UpdJob& J0 = a.job[0];
    int2 pf_touch = J0.nmb > 0 ? touch_of<K>(J0, 0, J0.desc[0].npairs, gw * G, G)
                               : make_int2(-1, -1);
    // phase clocks (thread 0 of each workgroup, when asked for), kept in LDS:
    // [0..3] ticks of the phases summed over the launch's minibatches (added
    // to the totals once at the end), [4] phase start, [5] barrier arrival,
    // [6] first barrier's exit
    __shared__ unsigned long long s_clk[7];
    const bool clk = a.clocks != nullptr && threadIdx.x == 0;
    if (clk)
        for (int i = 0; i < 4; ++i) s_clk[i] = 0;
    for (int m = 0; m < a.nmb_max; ++m) {
        if (clk) s_clk[4] = wall_clock64();
        int2 pf_seg = make_int2(kNoSeg, 0);
        int32_t pf_pair = 0;
        if (m < J0.nmb) {
            pf_seg = short_seg<NW>(J0, m, blockIdx.x);
        }

        // ---- forward of every job's minibatch m: G pairs per wave at a time
        for (int j = 0; j < a.njobs; ++j) {
            const UpdJob& J = a.job[j];
            if (m >= J.nmb) continue;
            const uint32_t np = J.desc[m].npairs;
            const double lr = (double)J.desc[m].lr;
            for (uint32_t q0 = gw * G; q0 < np; q0 += nw * G)
                forward_pairs<D, K, S, kAgent>(
                    J, np, q0,
                    j == 0 && q0 == gw * G ? pf_touch : touch_of<K>(J, m, np, q0, G), lr, lacc);
            if (a.njobs > 1) {
                // each job's loss terms to its own partials
                const double l = wave_total(lacc);
                if (lane == 0) J.loss_part[gw] += l;
                lacc = 0.0;
            }
        }
        pf_pair = short_pair(J0, m, unpack_seg(pf_seg));
        if (!grid_sync(a, epoch, clk ? &s_clk[5] : nullptr)) break;
        if (clk) {
            s_clk[6] = wall_clock64();
            s_clk[0] += s_clk[5] - s_clk[4];
            s_clk[1] += s_clk[6] - s_clk[5];
        }

        // ---- apply: in and out rows together
        if (m + 1 < J0.nmb) pf_touch = touch_of<K>(J0, m + 1, J0.desc[m + 1].npairs, gw * G, G);
        for (int j = 0; j < a.njobs; ++j) {
            const UpdJob& J = a.job[j];
            if (m >= J.nmb) continue;
            int2 seg = pf_seg;
            int32_t pair = pf_pair;
            if (j > 0) {
                seg = short_seg<NW>(J, m, blockIdx.x);
                pair = short_pair(J, m, unpack_seg(seg));
            }
            apply_items<D, kAgent, NW>(J, m, blockIdx.x, gridDim.x, seg, pair, J.desc[m].grid_c,
                                       part);
        }
        if (!grid_sync(a, epoch, clk ? &s_clk[5] : nullptr)) break;
        if (clk) {
            s_clk[2] += s_clk[5] - s_clk[6];
            s_clk[3] += wall_clock64() - s_clk[5];
        }
    }
    if (clk)
        for (int i = 0; i < 4; ++i) atomicAdd(&a.clocks[i], s_clk[i]);
    if (a.njobs == 1) {
        lacc = wave_total(lacc);
        if (lane == 0) J0.loss_part[gw] += lacc;
    }
}

// ------------------------------------------------- planned launches
// One minibatch's forward and apply as launches of their own, for callers that
// want no persistent launch (update path 1, serving jobs on streams of their
// own): two launches per minibatch with the plans of many made ahead, where
// ids, two scan passes, forward and two applies were six.  Jobs of 700 to
// 1,400 nodes (d = 64, K = 5, P = 1,024 and 2,048, one stream): 37 -> 14 us per
// minibatch, of which plans of ten minibatches per launch are 3 to 5.5.  Taken
// up to the 16,384 touches a plan sorts in LDS.
template <int D, int K>
__global__ __launch_bounds__(256) void sgns_planned_forward_kernel(UpdJob J, int32_t m,
                                                                   uint32_t npairs, float lr)
{
    constexpr uint32_t H = FwdShape<D, K>::kHalves;
    const uint32_t gw = blockIdx.x * 4 + (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t q0 = gw * H;
    if (q0 >= npairs) return;
    double lacc = 0.0;
    forward_pairs<D, K, 1, kPlain>(J, npairs, q0, touch_of<K>(J, m, npairs, q0, H), (double)lr,
                                   lacc);
    lacc = wave_total(lacc);
    if ((threadIdx.x & 63) == 0) J.loss_part[gw] += lacc;
}

template <int D>
__global__ __launch_bounds__(256) void sgns_planned_apply_kernel(UpdJob J, int32_t m, double gc)
{
    __shared__ double part[4 * D];
    const int2 seg = short_seg<4>(J, m, blockIdx.x);
    apply_items<D, kPlain, 4>(J, m, blockIdx.x, gridDim.x, seg, short_pair(J, m, unpack_seg(seg)),
                              gc, part);
}

__global__ void zero_words_kernel(uint32_t* p, int32_t n)
{
    for (int32_t i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0u;
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
// At d = 64 the persistent update is taken up to K = 14.  Beyond that planned
// launches are as fast or faster: us per minibatch of the persistent update and
// of planned launches, 8,192 touches, 1,000 nodes and R-MAT 2^18: K = 14 11.9 and
// 12.1, 11.3 and 11.7; K = 15 12.1 and 12.0, 11.6 and 11.5; K = 17 12.5 and 12.2,
// 12.1 and 11.5; K = 20 13.1 and 12.7, 12.9 and 12.2.
static bool persistent_pays(int d, int K) { return d > 64 || K <= 14; }

bool small_path_applies(const Model& m, const felog_train_params& p)
{
    return m.precision == FELOG_PREC_FP32 && m.ctx->sgns_path == 0 &&
           p.minibatch_pairs * (p.negatives + 2) <= kSmallMaxTouches && p.negatives <= 20 &&
           persistent_pays(m.dim, p.negatives);
}

// Minibatches per plan / update launch pair: the launches' fixed costs spread
// over 64 minibatches are under 1% of their time, and the plans stay small.
int64_t small_minibatches_per_launch() { return 64; }

// Bytes of one minibatch's plan (take_small_buffers), and of the buffers beside
// the plans.
static uint64_t plan_bytes(int64_t T) { return (uint64_t)(8 + 4 + 2) * T + 16; }
static uint64_t pair_buffer_bytes(int64_t P, int K, int d)
{
    return 8 * (uint64_t)(P * (K + 2)) + 2 * 4 * (uint64_t)P * d;
}

// Device bytes the small-minibatch update holds for minibatches of P pairs
// and K negatives at dimension d, over a call of B minibatches.
uint64_t small_path_bytes(int64_t P, int K, int d, int64_t B, int num_cus)
{
    const uint64_t G = (uint64_t)small_minibatches_per_launch();
    const uint64_t blocks = (uint64_t)std::max(kDefaultUpdBlocks, num_cus);
    return 2 * G * plan_bytes(P * (K + 2)) + pair_buffer_bytes(P, K, d) +
           32 * (uint64_t)std::max<int64_t>(B, 1) + 4 * kFlagStride * (blocks + 2) +
           8 * blocks * (kUpdThreads / 64) + 64;
}

template <int D, int K>
static void* update_kernel_ptr()
{
    return reinterpret_cast<void*>(&sgns_small_update_kernel<D, K>);
}

template <int D>
static void* update_kernel_d(int K)
{
    switch (K) {
#define FELOG_CASE(k) \
    case k: return update_kernel_ptr<D, k>();
        FELOG_CASE(1) FELOG_CASE(2) FELOG_CASE(3) FELOG_CASE(4) FELOG_CASE(5) FELOG_CASE(6)
        FELOG_CASE(7) FELOG_CASE(8) FELOG_CASE(9) FELOG_CASE(10) FELOG_CASE(11) FELOG_CASE(12)
        FELOG_CASE(13) FELOG_CASE(14) FELOG_CASE(15) FELOG_CASE(16) FELOG_CASE(17)
        FELOG_CASE(18) FELOG_CASE(19) FELOG_CASE(20)
#undef FELOG_CASE
        default: fail(FELOG_EUNSUPPORTED, "negatives = %d not supported", K);
    }
}

static void* update_kernel(int D, int K)
{
    if (D == 64) return update_kernel_d<64>(K);
    if (D == 128) return update_kernel_d<128>(K);
    return update_kernel_d<256>(K);
}

static void launch_plan(int K, int nblocks, const PlanBatch& pb, hipStream_t s)
{
    const bool wide = pb.job[0].tmax > kSmallMaxTouches;   // one job per such launch
    switch (K) {
#define FELOG_CASE(k)                                                                          \
    case k:                                                                                    \
        if (wide)                                                                              \
            hipLaunchKernelGGL((sgns_plan_kernel<k, kPlanMaxTouches>), dim3(nblocks),          \
                               dim3(kPlanThreads), 0, s, pb);                                  \
        else                                                                                   \
            hipLaunchKernelGGL((sgns_plan_kernel<k, kSmallMaxTouches>), dim3(nblocks),         \
                               dim3(kPlanThreads), 0, s, pb);                                  \
        break;
        FELOG_CASE(1) FELOG_CASE(2) FELOG_CASE(3) FELOG_CASE(4) FELOG_CASE(5) FELOG_CASE(6)
        FELOG_CASE(7) FELOG_CASE(8) FELOG_CASE(9) FELOG_CASE(10) FELOG_CASE(11) FELOG_CASE(12)
        FELOG_CASE(13) FELOG_CASE(14) FELOG_CASE(15) FELOG_CASE(16) FELOG_CASE(17)
        FELOG_CASE(18) FELOG_CASE(19) FELOG_CASE(20)
#undef FELOG_CASE
        default: fail(FELOG_EUNSUPPORTED, "negatives = %d not supported", K);
    }
    FELOG_HIP(hipGetLastError());
}

// Model-owned buffers of the planned paths, grown on demand: plans of `plans`
// minibatches (two sets of a launch group: the plans of group i + 1 are
// written while the update of group i reads set i mod 2), the out-touch
// coefficients, and each pair's in-row delta and context copy.
static void take_small_buffers(Model& m, int64_t P, int32_t tmax, int64_t plans)
{
    Ctx& c = *m.ctx;
    const int D = m.dim;
    if (m.sm_tmax < tmax || m.sm_G < plans) {
        const int64_t t = std::max<int64_t>(m.sm_tmax, tmax), g = std::max<int64_t>(m.sm_G, plans);
        m.sm_tmax = m.sm_G = 0;   // an allocation that fails leaves no stale capacity
        m.sm_tinfo.alloc(&c, sizeof(int2) * t * g);
        m.sm_segs.alloc(&c, sizeof(int2) * (t / 2) * g);
        m.sm_meta.alloc(&c, sizeof(uint32_t) * 4 * g);
        m.sm_spair.alloc(&c, sizeof(uint16_t) * t * g);
        m.sm_gpos.alloc(&c, sizeof(double) * t);
        m.sm_tmax = t;
        m.sm_G = g;
    }
    if (m.sm_pairs < P || m.sm_dim != D) {
        const int64_t n = std::max<int64_t>(m.sm_pairs, P);
        m.sm_pairs = 0;
        m.sm_dinp.alloc(&c, sizeof(float) * n * D);
        m.sm_ctxc.alloc(&c, sizeof(float) * n * D);
        m.sm_pairs = n;
        m.sm_dim = D;
    }
}

void drop_plans(Model& m)
{
    for (DevBuf* b : {&m.sm_tinfo, &m.sm_segs, &m.sm_meta, &m.sm_spair, &m.sm_gpos, &m.sm_dinp,
                      &m.sm_ctxc})
        b->release();
    m.sm_tmax = m.sm_G = m.sm_pairs = 0;
}

// Leaves the plans that the persistent update needs, or one for each of a
// planned launch's two sets.
void shrink_plans(Model& m)
{
    const int64_t t = m.sm_keep_tmax, g = m.sm_keep_G;
    if (m.sm_tmax * m.sm_G <= t * g) return;
    m.sm_tmax = m.sm_G = 0;
    for (DevBuf* b : {&m.sm_tinfo, &m.sm_segs, &m.sm_meta, &m.sm_spair, &m.sm_gpos}) b->release();
    try {
        take_small_buffers(m, m.sm_pairs, (int32_t)t, g);
    } catch (const Error& e) {
        if (e.code != FELOG_ENOMEM) throw;   // (they are taken on the next use)
        (void)hipGetLastError();
        clear_error();
    }
}

static void small_buffers(Model& m, int64_t P, int32_t tmax, int64_t plans)
{
    try {
        take_small_buffers(m, P, tmax, plans);
    } catch (const Error& e) {
        if (e.code != FELOG_ENOMEM) throw;
        // once more, for this call's sizes only and with the id sets of larger
        // minibatches given back
        (void)hipGetLastError();
        clear_error();
        shrink_id_sets(m);
        drop_plans(m);
        take_small_buffers(m, P, tmax, plans);
    }
}

// Plan arguments of a training call (plan set 0; the caller offsets them).
static PlanArgs plan_args(Model& m, Walks& w, const felog_train_params& p,
                          const int32_t* d_slices, int32_t tmax)
{
    PlanArgs pa{};
    pa.walks = w.data.as<int32_t>();
    pa.W = w.W;
    pa.vcols = w.valid_cols.as<int32_t>();
    pa.slices = d_slices;
    pa.id_base = w.id_base;
    pa.window = p.window;
    pa.seed = p.seed;
    pa.noise = NoiseTable{m.cdf.as<uint64_t>(), m.guide.as<int32_t>(), m.total_weight,
                          m.guide_bits};
    pa.row_bits = 1;
    while (((int64_t)1 << pa.row_bits) <= m.g->n) ++pa.row_bits;
    pa.tmax = tmax;
    pa.tinfo = m.sm_tinfo.as<int2>();
    pa.segs = m.sm_segs.as<int2>();
    pa.spair = m.sm_spair.as<uint16_t>();
    pa.meta = m.sm_meta.as<uint32_t>();
    pa.row_totals = m.row_totals.as<unsigned long long>();
    return pa;
}

// Descriptors of minibatches [first_mb, end); *last_chunk gets the chunk of
// the last minibatch of each launch group of G, *pairs the pair count.
static std::vector<MbDesc> mb_descs(const Walks& w, const felog_train_params& p,
                                    const TrainSchedule& sch, int64_t first_mb, int64_t end,
                                    int64_t G, std::vector<size_t>* last_chunk, int64_t* pairs)
{
    const int64_t P = p.minibatch_pairs;
    const double lr0 = (double)p.lr_start, lr1 = (double)p.lr_end;
    std::vector<MbDesc> desc((size_t)std::max<int64_t>(1, end - first_mb));
    size_t chunk = 0;
    *pairs = 0;
    for (int64_t b = first_mb; b < end; ++b) {
        while (chunk + 1 < sch.chunk_first_mb.size() && sch.chunk_first_mb[chunk + 1] <= b) ++chunk;
        const int64_t first = (b - sch.chunk_first_mb[chunk]) * P;
        const int64_t np = std::min<int64_t>(P, sch.chunk_pairs[chunk] - first);
        MbDesc& d = desc[(size_t)(b - first_mb)];
        d.vcol_base = sch.chunk_valid_base[chunk];
        d.Wv = (uint32_t)w.chunk_valid[chunk];
        d.first_pair = (uint32_t)first;
        d.npairs = (uint32_t)np;
        const double lr = lr0 - (lr0 - lr1) * (double)b / (double)std::max<int64_t>(1, sch.B - 1);
        d.lr = (float)lr;
        d.grid_c = d.lr > 0.0f ? std::ldexp(1.5, std::ilogb(d.lr) + 17) : 1.5;
        *pairs += np;
        if (last_chunk && ((b - first_mb) % G == G - 1 || b == end - 1)) last_chunk->push_back(chunk);
    }
    return desc;
}

// Workgroups of a persistent update launch: the context's choice (default 64),
// capped at what is resident at once (the launch is cooperative).
int small_update_blocks(const Ctx& c, int D, int K)
{
    int per_cu = 0;
    FELOG_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, update_kernel(D, K),
                                                           kUpdThreads, 0));
    FELOG_REQUIRE(per_cu >= 1, "the update kernel does not fit a compute unit");
    const int64_t max_blocks = (int64_t)per_cu * c.num_cus;
    const int64_t want = c.sgns_blocks > 0 ? c.sgns_blocks : kDefaultUpdBlocks;
    return (int)std::max<int64_t>(1, std::min(want, max_blocks));
}

// ------------------------------------------------------- shared launches
// A training call of one model (one job) run inside launches shared with
// other jobs: plans and updates of the jobs' next launch groups together.
// Its plans run on the model's own stream one launch group ahead of the
// shared updates, in two buffer sets (group g uses set g mod 2): the plan of
// group g waits for the update of group g - 2, the update of group g for the
// plan of group g.
struct SmallJob {
    Model* m = nullptr;
    Walks* w = nullptr;
    felog_train_params p{};
    TrainSchedule sch;
    DevBuf slices, ddesc, loss;
    int K = 0, D = 0;
    int32_t tmax = 0;
    int64_t next = 0;        // first minibatch not yet updated
    int64_t planned = 0;     // first minibatch whose plan is not launched
    int64_t end = 0, pairs = 0;
    int nwaves = 0;
    PlanArgs pa{};
    UpdJob uj{};
    hipEvent_t plan_done[2] = {nullptr, nullptr};
    hipEvent_t upd_done[2] = {nullptr, nullptr};
    ~SmallJob()
    {
        for (hipEvent_t e : {plan_done[0], plan_done[1], upd_done[0], upd_done[1]})
            if (e) (void)hipEventDestroy(e);
    }
};

void SmallJobDeleter::operator()(SmallJob* j) const { delete j; }

// Plan arguments of a job's launch group starting at minibatch b (set b / G mod 2).
static PlanArgs group_plan(const SmallJob& j, int64_t b)
{
    const int64_t G = small_minibatches_per_launch();
    const int64_t set = (b / G) & 1;
    PlanArgs pl = j.pa;
    pl.desc = j.ddesc.as<MbDesc>() + b;
    pl.tinfo = j.pa.tinfo + set * G * j.tmax;
    pl.segs = j.pa.segs + set * G * (j.tmax / 2);
    pl.spair = j.pa.spair + set * G * j.tmax;
    pl.meta = j.pa.meta + set * G * 4;
    return pl;
}

// Launches the plan of the job's next unplanned launch group on its model's stream.
static void plan_next_group(SmallJob& j)
{
    const int64_t G = small_minibatches_per_launch();
    if (j.planned >= j.end) return;
    const int64_t g = j.planned / G;
    const int set = (int)(g & 1);
    hipStream_t js = j.m->ctx->stream;
    if (g >= 2) FELOG_HIP(hipStreamWaitEvent(js, j.upd_done[set], 0));
    const int nmb = (int)std::min<int64_t>(G, j.end - j.planned);
    PlanBatch pb{};
    pb.job[0] = group_plan(j, j.planned);
    pb.start[0] = 0;
    pb.start[1] = nmb;
    pb.njobs = 1;
    launch_plan(j.K, nmb, pb, js);
    FELOG_HIP(hipEventRecord(j.plan_done[set], js));
    j.planned += nmb;
}

bool small_job_fits(const Model& m, const felog_train_params& p)
{
    return m.precision == FELOG_PREC_FP32 && p.negatives <= 20 &&
           p.minibatch_pairs * (p.negatives + 2) <= kSmallMaxTouches &&
           (m.dim == 64 || m.dim == 128 || m.dim == 256) && persistent_pays(m.dim, p.negatives);
}

SmallJobPtr small_job_begin(Model& m, Walks& w, const felog_train_params& p, int nblocks)
{
    Ctx& c = *m.ctx;
    FELOG_REQUIRE(small_job_fits(m, p), "the job does not fit the shared persistent update");
    SmallJobPtr j(new SmallJob);
    j->m = &m;
    j->w = &w;
    j->p = p;
    j->sch = train_schedule(w, p);
    j->K = p.negatives;
    j->D = m.dim;
    j->tmax = (int32_t)(p.minibatch_pairs * (p.negatives + 2));
    j->end = j->sch.B;
    j->nwaves = nblocks * (kUpdThreads / 64);
    small_buffers(m, p.minibatch_pairs, j->tmax, 2 * small_minibatches_per_launch());
    const std::vector<int32_t> sl = train_slices(w.L, p.window);
    j->slices.alloc(&c, sizeof(int32_t) * std::max<size_t>(sl.size(), 1));
    if (!sl.empty())
        FELOG_HIP(hipMemcpyAsync(j->slices.ptr, sl.data(), sizeof(int32_t) * sl.size(),
                                 hipMemcpyHostToDevice, c.stream));
    const std::vector<MbDesc> desc =
        mb_descs(w, p, j->sch, 0, j->end, small_minibatches_per_launch(), nullptr, &j->pairs);
    j->ddesc.alloc(&c, sizeof(MbDesc) * desc.size());
    FELOG_HIP(hipMemcpyAsync(j->ddesc.ptr, desc.data(), sizeof(MbDesc) * desc.size(),
                             hipMemcpyHostToDevice, c.stream));
    j->loss.alloc(&c, sizeof(double) * j->nwaves);
    FELOG_HIP(hipMemsetAsync(j->loss.ptr, 0, j->loss.bytes, c.stream));
    FELOG_HIP(hipMemsetAsync(m.row_totals.ptr, 0, sizeof(uint64_t) * 3, c.stream));
    j->pa = plan_args(m, w, p, j->slices.as<int32_t>(), j->tmax);
    j->uj.tin = m.tin.as<float>();
    j->uj.tout = m.tout.as<float>();
    j->uj.tmax = j->tmax;
    j->uj.gpos = m.sm_gpos.as<double>();
    j->uj.dinp = m.sm_dinp.as<float>();
    j->uj.ctxc = m.sm_ctxc.as<float>();
    j->uj.loss_part = j->loss.as<double>();
    for (hipEvent_t* e : {&j->plan_done[0], &j->plan_done[1], &j->upd_done[0], &j->upd_done[1]})
        FELOG_HIP(hipEventCreateWithFlags(e, hipEventDisableTiming));
    c.sync();   // the buffers are ready before another stream uses them
    plan_next_group(*j);
    return j;
}

int small_job_dim(const SmallJob& j) { return j.D; }
int small_job_negatives(const SmallJob& j) { return j.K; }
bool small_job_done(const SmallJob& j) { return j.next >= j.end; }

void small_batch_init(SmallBatchCtl& ctl, Ctx& c, int nblocks)
{
    ctl.nblocks = nblocks;
    ctl.epoch = 0;
    ctl.words.alloc(&c, sizeof(uint32_t) * kFlagStride * (nblocks + 2));
    hipLaunchKernelGGL(zero_words_kernel, dim3(1), dim3(256), 0, c.stream,
                       ctl.words.as<uint32_t>(), (int32_t)(ctl.words.bytes / sizeof(uint32_t)));
    FELOG_HIP(hipGetLastError());
    c.sync();
}

void small_jobs_step(const std::vector<SmallJob*>& jobs, SmallBatchCtl& ctl, hipStream_t s)
{
    FELOG_REQUIRE(!jobs.empty() && jobs.size() <= (size_t)kMaxBatchJobs,
                  "a shared launch takes 1 to %d jobs", kMaxBatchJobs);
    const int K = jobs[0]->K, D = jobs[0]->D;
    const int64_t G = small_minibatches_per_launch();
    UpdArgs u{};
    int nmb_max = 0;
    for (size_t i = 0; i < jobs.size(); ++i) {
        SmallJob& j = *jobs[i];
        FELOG_REQUIRE(j.K == K && j.D == D && !small_job_done(j),
                      "jobs of a shared launch need equal d and K and minibatches left");
        FELOG_REQUIRE(j.nwaves == ctl.nblocks * (kUpdThreads / 64),
                      "job prepared for another grid size");
        if (j.planned == j.next) plan_next_group(j);
        const int set = (int)((j.next / G) & 1);
        FELOG_HIP(hipStreamWaitEvent(s, j.plan_done[set], 0));
        const int nmb = (int)std::min<int64_t>(G, j.end - j.next);
        const PlanArgs pl = group_plan(j, j.next);
        UpdJob uj = j.uj;
        uj.desc = pl.desc;
        uj.tinfo = pl.tinfo;
        uj.segs = pl.segs;
        uj.spair = pl.spair;
        uj.meta = pl.meta;
        uj.nmb = nmb;
        u.job[i] = uj;
        nmb_max = std::max(nmb_max, nmb);
    }
    u.njobs = (int32_t)jobs.size();
    u.nmb_max = nmb_max;
    u.flags = ctl.words.as<uint32_t>();
    u.abort = reinterpret_cast<int32_t*>(u.flags + (int64_t)kFlagStride * (ctl.nblocks + 1));
    u.epoch0 = ctl.epoch;
    void* args[] = {&u};
    FELOG_HIP(hipLaunchCooperativeKernel(update_kernel(D, K), dim3(ctl.nblocks), dim3(kUpdThreads),
                                         args, 0, s));
    ctl.epoch += 2u * (uint32_t)nmb_max;
    for (SmallJob* jp : jobs) {
        SmallJob& j = *jp;
        const int set = (int)((j.next / G) & 1);
        FELOG_HIP(hipEventRecord(j.upd_done[set], s));
        j.next += std::min<int64_t>(G, j.end - j.next);
        // the next group's plan beside this update, on the job's stream
        if (j.planned == j.next) plan_next_group(j);
    }
}

bool small_batch_aborted(SmallBatchCtl& ctl, hipStream_t s)
{
    int32_t aborted = 0;
    const int32_t* abort =
        reinterpret_cast<const int32_t*>(ctl.words.as<uint32_t>() + (int64_t)kFlagStride * (ctl.nblocks + 1));
    FELOG_HIP(hipMemcpyAsync(&aborted, abort, sizeof aborted, hipMemcpyDeviceToHost, s));
    FELOG_HIP(hipStreamSynchronize(s));
    return aborted != 0;
}

void small_job_end(SmallJob& j, hipStream_t s, felog_train_stats* stats)
{
    Model& m = *j.m;
    launch_loss_reduce(j.loss.as<double>(), j.nwaves, m.loss_out.as<double>(), s);
    double loss = 0.0;
    unsigned long long rows[3] = {0, 0, 0};
    FELOG_HIP(hipMemcpyAsync(&loss, m.loss_out.ptr, sizeof loss, hipMemcpyDeviceToHost, s));
    FELOG_HIP(hipMemcpyAsync(rows, m.row_totals.ptr, sizeof rows, hipMemcpyDeviceToHost, s));
    FELOG_HIP(hipStreamSynchronize(s));
    if (stats) {
        *stats = felog_train_stats{};
        stats->minibatches = j.end;
        stats->pairs = j.pairs;
        stats->minibatches_total = j.sch.B;
        stats->loss = loss;
        stats->rows_in = (int64_t)rows[0];
        stats->rows_out = (int64_t)rows[1];
        stats->rows_out_single = (int64_t)rows[2];
        stats->path = 1;
    }
}

void train_minibatches_small(Model& m, Walks& w, const felog_train_params& p,
                             const TrainSchedule& sch, const int32_t* d_slices, int64_t first_mb,
                             int64_t end, felog_train_stats* stats)
{
    Ctx& c = *m.ctx;
    const int K = p.negatives;
    const int D = m.dim;
    const int64_t P = p.minibatch_pairs;
    const int32_t tmax = (int32_t)(P * (K + 2));
    FELOG_REQUIRE(tmax <= kSmallMaxTouches, "minibatch of %lld pairs is too large for the "
                  "small-minibatch update", (long long)P);
    FELOG_REQUIRE(D == 64 || D == 128 || D == 256, "dim %d not supported", D);
    const int64_t G = small_minibatches_per_launch();
    void* kern = update_kernel(D, K);
    const int nblocks = small_update_blocks(c, D, K);
    const int nwaves = nblocks * (kUpdThreads / 64);

    // control words: barrier flags (an unused line, then one per workgroup,
    // each on its own 128-byte line), the abort flag on the next line, then
    // the loss partials, one per wave, and the four phase-clock sums
    const int64_t ctl_words = (int64_t)kFlagStride * (nblocks + 2);
    DevBuf ctl;
    ctl.alloc(&c, sizeof(uint32_t) * ctl_words + sizeof(double) * nwaves +
                      sizeof(unsigned long long) * 4);
    uint32_t* flags = ctl.as<uint32_t>();
    int32_t* abort = reinterpret_cast<int32_t*>(flags + (int64_t)kFlagStride * (nblocks + 1));
    double* loss_part = reinterpret_cast<double*>(flags + ctl_words);
    unsigned long long* clocks = reinterpret_cast<unsigned long long*>(loss_part + nwaves);
    hipLaunchKernelGGL(zero_words_kernel, dim3(1), dim3(256), 0, c.stream, flags,
                       (int32_t)(ctl.bytes / sizeof(uint32_t)));
    FELOG_HIP(hipMemsetAsync(m.row_totals.ptr, 0, sizeof(uint64_t) * 3, c.stream));

    // every minibatch's descriptor, uploaded once for the call
    std::vector<size_t> last_chunk;   // chunk of the last minibatch of each launch
    int64_t pairs = 0;
    const std::vector<MbDesc> desc = mb_descs(w, p, sch, first_mb, end, G, &last_chunk, &pairs);
    DevBuf ddesc;
    ddesc.alloc(&c, sizeof(MbDesc) * desc.size());
    FELOG_HIP(hipMemcpyAsync(ddesc.ptr, desc.data(), sizeof(MbDesc) * desc.size(),
                             hipMemcpyHostToDevice, c.stream));

    const HoldScratch hold(m);
    small_buffers(m, P, tmax, 2 * G);
    m.sm_keep_tmax = m.sm_keep_G == 2 * G ? std::max<int64_t>(m.sm_keep_tmax, tmax) : tmax;
    m.sm_keep_G = 2 * G;
    const PlanArgs pa = plan_args(m, w, p, d_slices, tmax);
    UpdJob uj{};
    uj.tin = m.tin.as<float>();
    uj.tout = m.tout.as<float>();
    uj.tmax = tmax;
    uj.gpos = m.sm_gpos.as<double>();
    uj.dinp = m.sm_dinp.as<float>();
    uj.ctxc = m.sm_ctxc.as<float>();
    uj.loss_part = loss_part;

    // Plans run on the context's second stream one launch group ahead of the
    // updates: plan(i) waits for update(i - 2) (its buffer set), update(i)
    // waits for plan(i).  pipe_ev: [0] start, [1 + set] plan done,
    // [3 + set] update done.
    c.ensure_aux();
    hipStream_t ps = c.aux;
    FELOG_HIP(hipEventRecord(c.pipe_ev[0], c.stream));
    FELOG_HIP(hipStreamWaitEvent(ps, c.pipe_ev[0], 0));
    size_t gated = 0;
    const bool timing = c.timing_every > 0 && !c.timing_pool.empty();
    const size_t tslots = c.timing_pool.size() / 4;
    std::vector<int64_t> slot_nmb(tslots, 0);
    double ms_plan = 0.0, ms_update = 0.0;
    int64_t timed = 0, timed_mb = 0;
    auto harvest = [&](size_t slot) {
        hipEvent_t* e = &c.timing_pool[4 * slot];
        FELOG_HIP(hipEventSynchronize(e[3]));
        float a0 = 0.0f, a1 = 0.0f;
        FELOG_HIP(hipEventElapsedTime(&a0, e[0], e[1]));
        FELOG_HIP(hipEventElapsedTime(&a1, e[2], e[3]));
        ms_plan += a0;
        ms_update += a1;
        ++timed;
        timed_mb += slot_nmb[slot];
        slot_nmb[slot] = 0;
    };
    uint32_t epoch = 0;
    FELOG_HIP(hipEventRecord(c.ev0, c.stream));
    for (int64_t g0 = first_mb, li = 0; g0 < end; g0 += G, ++li) {
        const int64_t g1 = std::min(end, g0 + G);
        const int nmb = (int)(g1 - g0);
        const int set = (int)(li & 1);
        hipEvent_t* e = nullptr;
        if (timing) {
            const size_t slot = (size_t)(li % (int64_t)tslots);
            if (slot_nmb[slot]) harvest(slot);
            slot_nmb[slot] = nmb;
            e = &c.timing_pool[4 * slot];
        }
        // plan of group li, on the second stream
        if (li >= 2) FELOG_HIP(hipStreamWaitEvent(ps, c.pipe_ev[3 + set], 0));
        // the walks of the launch's chunks must be written
        while (gated <= last_chunk[(size_t)li] && gated < w.chunk_ready.size())
            FELOG_HIP(hipStreamWaitEvent(ps, w.chunk_ready[gated++], 0));
        PlanArgs pl = pa;
        pl.desc = ddesc.as<MbDesc>() + (g0 - first_mb);
        pl.tinfo = pa.tinfo + (int64_t)set * G * tmax;
        pl.segs = pa.segs + (int64_t)set * G * (tmax / 2);
        pl.spair = pa.spair + (int64_t)set * G * tmax;
        pl.meta = pa.meta + (int64_t)set * G * 4;
        PlanBatch pb{};
        pb.job[0] = pl;
        pb.start[0] = 0;
        pb.start[1] = nmb;
        pb.njobs = 1;
        if (e) FELOG_HIP(hipEventRecord(e[0], ps));
        launch_plan(K, nmb, pb, ps);
        if (e) FELOG_HIP(hipEventRecord(e[1], ps));
        FELOG_HIP(hipEventRecord(c.pipe_ev[1 + set], ps));
        // update of group li, on the context's stream
        FELOG_HIP(hipStreamWaitEvent(c.stream, c.pipe_ev[1 + set], 0));
        UpdArgs u{};
        u.job[0] = uj;
        u.job[0].desc = pl.desc;
        u.job[0].tinfo = pl.tinfo;
        u.job[0].segs = pl.segs;
        u.job[0].spair = pl.spair;
        u.job[0].meta = pl.meta;
        u.job[0].nmb = nmb;
        u.njobs = 1;
        u.nmb_max = nmb;
        u.flags = flags;
        u.abort = abort;
        u.epoch0 = epoch;
        u.clocks = timing ? clocks : nullptr;
        void* args[] = {&u};
        if (e) FELOG_HIP(hipEventRecord(e[2], c.stream));
        FELOG_HIP(hipLaunchCooperativeKernel(kern, dim3(nblocks), dim3(kUpdThreads), args, 0,
                                             c.stream));
        if (e) FELOG_HIP(hipEventRecord(e[3], c.stream));
        FELOG_HIP(hipEventRecord(c.pipe_ev[3 + set], c.stream));
        epoch += 2u * (uint32_t)nmb;
    }
    if (timing)
        for (size_t slot = 0; slot < tslots; ++slot)
            if (slot_nmb[slot]) harvest(slot);
    launch_loss_reduce(loss_part, nwaves, m.loss_out.as<double>(), c.stream);
    FELOG_HIP(hipEventRecord(c.ev1, c.stream));
    double loss = 0.0;
    unsigned long long rows[3] = {0, 0, 0};
    int32_t aborted = 0;
    unsigned long long ticks[4] = {0, 0, 0, 0};
    FELOG_HIP(hipMemcpyAsync(&loss, m.loss_out.ptr, sizeof loss, hipMemcpyDeviceToHost, c.stream));
    FELOG_HIP(hipMemcpyAsync(rows, m.row_totals.ptr, sizeof rows, hipMemcpyDeviceToHost, c.stream));
    FELOG_HIP(hipMemcpyAsync(&aborted, abort, sizeof aborted, hipMemcpyDeviceToHost, c.stream));
    if (timing)
        FELOG_HIP(hipMemcpyAsync(ticks, clocks, sizeof ticks, hipMemcpyDeviceToHost, c.stream));
    c.sync();
    FELOG_HIP(hipStreamSynchronize(ps));
    FELOG_REQUIRE(!aborted, "small-minibatch update: a grid barrier wait exceeded its bound");
    float ms = 0.0f;
    FELOG_HIP(hipEventElapsedTime(&ms, c.ev0, c.ev1));
    if (stats) {
        *stats = felog_train_stats{};
        stats->minibatches = end - first_mb;
        stats->pairs = pairs;
        stats->minibatches_total = sch.B;
        stats->loss = loss;
        stats->ms = ms;
        stats->rows_in = (int64_t)rows[0];
        stats->rows_out = (int64_t)rows[1];
        stats->rows_out_single = (int64_t)rows[2];
        stats->path = 1;
        stats->timed_launches = timed;
        stats->timed_minibatches = timed_mb;
        stats->ms_prep = ms_plan;
        stats->ms_update = ms_update;
        stats->update_blocks = nblocks;
        if (timing && end > first_mb) {
            int khz = 0;   // device wall-clock rate
            FELOG_HIP(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, c.device));
            const double per = (double)nblocks * (double)(end - first_mb) * (double)khz / 1e3;
            for (int i = 0; i < 4; ++i)
                stats->us_phase[i] = khz > 0 ? (double)ticks[i] / per : 0.0;
        }
    }
}

// ---------------------------------------------------- planned launches, host
template <int D>
static void launch_planned_forward_d(int K, const UpdJob& J, int32_t m, uint32_t np, float lr,
                                     hipStream_t s)
{
    const uint32_t per_block = 4 * (D == 64 ? 2 : 1);   // pairs
    const dim3 grid((np + per_block - 1) / per_block);
    switch (K) {
#define FELOG_CASE(k)                                                                            \
    case k:                                                                                      \
        hipLaunchKernelGGL((sgns_planned_forward_kernel<D, k>), grid, dim3(256), 0, s, J, m, np, lr); \
        break;
        FELOG_CASE(1) FELOG_CASE(2) FELOG_CASE(3) FELOG_CASE(4) FELOG_CASE(5) FELOG_CASE(6)
        FELOG_CASE(7) FELOG_CASE(8) FELOG_CASE(9) FELOG_CASE(10) FELOG_CASE(11) FELOG_CASE(12)
        FELOG_CASE(13) FELOG_CASE(14) FELOG_CASE(15) FELOG_CASE(16) FELOG_CASE(17)
        FELOG_CASE(18) FELOG_CASE(19) FELOG_CASE(20)
#undef FELOG_CASE
        default: fail(FELOG_EUNSUPPORTED, "negatives = %d not supported", K);
    }
}

// Trains [first_mb, end) with planned launches; false (nothing done) when the
// minibatches are too large for a plan or the context's budget or the card
// has no room for the plans of one.
bool train_minibatches_planned(Model& m, Walks& w, const felog_train_params& p,
                               const TrainSchedule& sch, const int32_t* d_slices,
                               int64_t first_mb, int64_t end, felog_train_stats* stats)
{
    Ctx& c = *m.ctx;
    const int K = p.negatives, D = m.dim;
    const int64_t P = p.minibatch_pairs;
    if (m.precision != FELOG_PREC_FP32 || K > 20 || P * (K + 2) > kPlanMaxTouches) return false;
    const int32_t tmax = (int32_t)(P * (K + 2));
    const int64_t B = std::max<int64_t>(1, end - first_mb);
    // launch groups: one set of plans when everything is on one stream
    const int64_t sets = c.single_stream ? 1 : 2;
    int64_t G = std::min<int64_t>(small_minibatches_per_launch(), B);
    if (c.budget) {
        uint64_t held = 0;   // plan buffers of earlier calls, which a larger set replaces
        for (const DevBuf* b : {&m.sm_tinfo, &m.sm_segs, &m.sm_meta, &m.sm_spair, &m.sm_gpos,
                                &m.sm_dinp, &m.sm_ctxc})
            held += b->bytes;
        const uint64_t room = c.budget + held - std::min(c.budget + held, c.in_use);
        const uint64_t fixed = pair_buffer_bytes(P, K, D) + 8 * ((uint64_t)P + 1) + 4096;
        if (room < fixed + sets * plan_bytes(tmax)) return false;
        G = std::min<int64_t>(G, (int64_t)((room - fixed) / (sets * plan_bytes(tmax))));
        if (m.sm_tmax < tmax || m.sm_G < sets * G || m.sm_pairs < P) drop_plans(m);
    }
    const int64_t side = D == 64 ? 2 : 1;
    const int64_t nwaves = (P + side - 1) / side;
    DevBuf loss_part;
    const HoldScratch hold(m);
    try {
        loss_part.alloc(&c, sizeof(double) * nwaves);
        small_buffers(m, P, tmax, sets * G);
        if (m.sm_keep_G <= 2) {
            m.sm_keep_tmax = std::max<int64_t>(m.sm_keep_tmax, tmax);
            m.sm_keep_G = 2;
        }
    } catch (const Error& e) {
        if (e.code != FELOG_ENOMEM) throw;
        (void)hipGetLastError();
        clear_error();
        drop_plans(m);
        return false;
    }
    int64_t pairs = 0;
    const std::vector<MbDesc> desc = mb_descs(w, p, sch, first_mb, end, G, nullptr, &pairs);
    // launch groups: up to G consecutive minibatches of one chunk
    struct Group {
        int64_t first, end;
        size_t chunk;
    };
    std::vector<Group> groups;
    {
        size_t chunk = 0;
        for (int64_t b = first_mb; b < end;) {
            while (chunk + 1 < sch.chunk_first_mb.size() && sch.chunk_first_mb[chunk + 1] <= b) ++chunk;
            int64_t e = std::min(end, b + G);
            if (chunk + 1 < sch.chunk_first_mb.size())
                e = std::min<int64_t>(e, sch.chunk_first_mb[chunk + 1]);
            groups.push_back(Group{b, e, chunk});
            b = e;
        }
    }
    FELOG_HIP(hipMemsetAsync(loss_part.ptr, 0, loss_part.bytes, c.stream));
    FELOG_HIP(hipMemsetAsync(m.row_totals.ptr, 0, sizeof(uint64_t) * 3, c.stream));
    const PlanArgs pa = plan_args(m, w, p, d_slices, tmax);
    UpdJob uj{};
    uj.tin = m.tin.as<float>();
    uj.tout = m.tout.as<float>();
    uj.tmax = tmax;
    uj.gpos = m.sm_gpos.as<double>();
    uj.dinp = m.sm_dinp.as<float>();
    uj.ctxc = m.sm_ctxc.as<float>();
    uj.loss_part = loss_part.as<double>();
    // a segment has two touches or more, and each table row at most one segment
    const int64_t segs = std::min<int64_t>(tmax / 2 + 1, 2 * (int64_t)m.g->n);
    const int64_t items = (segs + 15) / 16 + std::min<int64_t>(tmax / kChunk, segs);
    const dim3 agrid((uint32_t)std::min<int64_t>(items, (int64_t)c.num_cus));

    // plans of group i + 1 on the second stream beside group i, as in the
    // persistent path (pipe_ev: [0] start, [1 + set] plan done, [3 + set]
    // group done)
    c.ensure_aux();
    hipStream_t ps = c.aux;
    FELOG_HIP(hipEventRecord(c.pipe_ev[0], c.stream));
    if (ps != c.stream) FELOG_HIP(hipStreamWaitEvent(ps, c.pipe_ev[0], 0));
    size_t gated = 0;
    // sampled timing: per timed minibatch [0, 1] around its group's plan
    // launch (one launch for the group's minibatches, each timed one counts
    // its share), [2] before its forward, [3] after it, [5] after its apply
    const int every = c.timing_every;
    const size_t pool = c.timing_pool.size() / kTimingEvents;
    size_t next_slot = 0, used_slots = 0;
    int64_t timed = 0;
    double ms_prep = 0.0, ms_fwd = 0.0, ms_apply = 0.0;
    std::vector<double> slot_share(pool, 0.0);   // 1 / minibatches of the group, by slot
    std::vector<hipEvent_t> plan_ev;             // two per group that has a timed minibatch
    struct PlanEvents {
        std::vector<hipEvent_t>& v;
        ~PlanEvents()
        {
            for (hipEvent_t e : v) (void)hipEventDestroy(e);
        }
    } plan_ev_guard{plan_ev};
    std::vector<size_t> slot_plan(pool, 0);
    auto harvest = [&](size_t slot) {
        hipEvent_t* e = &c.timing_pool[kTimingEvents * slot];
        FELOG_HIP(hipEventSynchronize(e[5]));
        float a0 = 0.0f, f = 0.0f, ap = 0.0f;
        FELOG_HIP(hipEventElapsedTime(&a0, plan_ev[slot_plan[slot]], plan_ev[slot_plan[slot] + 1]));
        FELOG_HIP(hipEventElapsedTime(&f, e[2], e[3]));
        FELOG_HIP(hipEventElapsedTime(&ap, e[3], e[5]));
        ms_prep += a0 * slot_share[slot];
        ms_fwd += f;
        ms_apply += ap;
        ++timed;
    };
    FELOG_HIP(hipEventRecord(c.ev0, c.stream));
    auto plan_group = [&](size_t li) {
        const Group& gr = groups[li];
        const int64_t set = (int64_t)li % sets;
        const int nmb = (int)(gr.end - gr.first);
        if (ps != c.stream && li >= 2) FELOG_HIP(hipStreamWaitEvent(ps, c.pipe_ev[3 + set], 0));
        while (gated <= gr.chunk && gated < w.chunk_ready.size())
            FELOG_HIP(hipStreamWaitEvent(ps, w.chunk_ready[gated++], 0));
        PlanBatch pb{};
        pb.job[0] = pa;
        pb.job[0].first = desc[(size_t)(gr.first - first_mb)];
        pb.job[0].pairs = (uint32_t)P;
        pb.job[0].chunk_pairs = (uint32_t)sch.chunk_pairs[gr.chunk];
        pb.job[0].tinfo += set * G * tmax;
        pb.job[0].segs += set * G * (tmax / 2);
        pb.job[0].spair += set * G * tmax;
        pb.job[0].meta += set * G * 4;
        pb.start[1] = nmb;
        pb.njobs = 1;
        if (every > 0) {
            hipEvent_t e[2] = {nullptr, nullptr};
            for (hipEvent_t& x : e) {
                FELOG_HIP(hipEventCreate(&x));
                plan_ev.push_back(x);
            }
            FELOG_HIP(hipEventRecord(e[0], ps));
            launch_plan(K, nmb, pb, ps);
            FELOG_HIP(hipEventRecord(e[1], ps));
        } else {
            launch_plan(K, nmb, pb, ps);
        }
        FELOG_HIP(hipEventRecord(c.pipe_ev[1 + set], ps));
    };
    if (!groups.empty()) plan_group(0);
    for (size_t li = 0; li < groups.size(); ++li) {
        const int64_t set = (int64_t)li % sets, g0 = groups[li].first, g1 = groups[li].end;
        if (sets == 2 && li + 1 < groups.size()) plan_group(li + 1);
        if (ps != c.stream) FELOG_HIP(hipStreamWaitEvent(c.stream, c.pipe_ev[1 + set], 0));
        UpdJob J = uj;
        J.tinfo = pa.tinfo + set * G * tmax;
        J.segs = pa.segs + set * G * (tmax / 2);
        J.spair = pa.spair + set * G * tmax;
        J.meta = pa.meta + set * G * 4;
        for (int64_t b = g0; b < g1; ++b) {
            const MbDesc& d = desc[(size_t)(b - first_mb)];
            const int32_t mm = (int32_t)(b - g0);
            hipEvent_t* e = nullptr;
            if (every > 0 && pool > 0 && (b - first_mb) % every == 0) {
                if (used_slots == pool) harvest(next_slot);
                else ++used_slots;
                e = &c.timing_pool[kTimingEvents * next_slot];
                slot_share[next_slot] = 1.0 / (double)(g1 - g0);
                slot_plan[next_slot] = 2 * li;
                next_slot = (next_slot + 1) % pool;
            }
            if (e) FELOG_HIP(hipEventRecord(e[2], c.stream));
            if (D == 64) launch_planned_forward_d<64>(K, J, mm, d.npairs, d.lr, c.stream);
            else if (D == 128) launch_planned_forward_d<128>(K, J, mm, d.npairs, d.lr, c.stream);
            else launch_planned_forward_d<256>(K, J, mm, d.npairs, d.lr, c.stream);
            if (e) FELOG_HIP(hipEventRecord(e[3], c.stream));
            if (D == 64)
                hipLaunchKernelGGL(sgns_planned_apply_kernel<64>, agrid, dim3(256), 0, c.stream, J, mm, d.grid_c);
            else if (D == 128)
                hipLaunchKernelGGL(sgns_planned_apply_kernel<128>, agrid, dim3(256), 0, c.stream, J, mm, d.grid_c);
            else
                hipLaunchKernelGGL(sgns_planned_apply_kernel<256>, agrid, dim3(256), 0, c.stream, J, mm, d.grid_c);
            if (e) FELOG_HIP(hipEventRecord(e[5], c.stream));
        }
        FELOG_HIP(hipGetLastError());
        FELOG_HIP(hipEventRecord(c.pipe_ev[3 + set], c.stream));
        if (sets == 1 && li + 1 < groups.size()) plan_group(li + 1);
    }
    launch_loss_reduce(loss_part.as<double>(), nwaves, m.loss_out.as<double>(), c.stream);
    FELOG_HIP(hipGetLastError());
    FELOG_HIP(hipEventRecord(c.ev1, c.stream));
    double loss = 0.0;
    unsigned long long rows[3] = {0, 0, 0};
    FELOG_HIP(hipMemcpyAsync(&loss, m.loss_out.ptr, sizeof loss, hipMemcpyDeviceToHost, c.stream));
    FELOG_HIP(hipMemcpyAsync(rows, m.row_totals.ptr, sizeof rows, hipMemcpyDeviceToHost, c.stream));
    c.sync();
    if (ps != c.stream) FELOG_HIP(hipStreamSynchronize(ps));
    for (size_t k = 0; k < used_slots; ++k) harvest((next_slot + pool - used_slots + k) % pool);
    float ms = 0.0f;
    FELOG_HIP(hipEventElapsedTime(&ms, c.ev0, c.ev1));
    if (stats) {
        *stats = felog_train_stats{};
        stats->minibatches = end - first_mb;
        stats->pairs = pairs;
        stats->minibatches_total = sch.B;
        stats->loss = loss;
        stats->ms = ms;
        stats->rows_in = (int64_t)rows[0];
        stats->rows_out = (int64_t)rows[1];
        stats->rows_out_single = (int64_t)rows[2];
        stats->timed_launches = timed;
        stats->timed_minibatches = timed;
        stats->ms_forward = ms_fwd;
        stats->ms_apply = ms_apply;
        stats->ms_apply_first = ms_apply;
        stats->ms_prep = ms_prep;
    }
    return true;
}

}  // namespace felog
