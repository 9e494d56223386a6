// The SGNS forward of a batch of pairs in one wave, shared by the update paths
// (sgns.hip, sgns_small.hip).
//
// A wave takes B pairs per step side by side in its registers: every row of a
// pair is spread over all 64 lanes (d >= 128; at d = 64 over 32, and the wave
// holds two pairs at a time).  So a pair's row numbers are wave-uniform and
// its addresses scalar, all B (K + 2) row reads are in flight before the first
// is used, and the B (K + 1) dots are reduced together: each halving step of
// the butterfly over the lanes also halves the number of values, and each lane
// ends with one dot.  The lanes evaluate their dots' sigma and loss at the
// same time, one FP64 exponential for the whole batch, and the coefficients
// return to all lanes as scalars.
//
// Arithmetic of a dot (all paths): FP64, one fused chain over elements 4 j ..
// 4 j + 3 (and at d = 256 on over 128 + 4 j .. 131 + 4 j) for each j, then the
// butterfly over the 32 (16) chains.  A chain's elements lie in two lanes, so
// it passes between them by DPP; each lane's own sum and one more butterfly
// step would take four instructions less per dot, but the order is part of the
// result: minibatches of summed updates can be unstable enough (16,384 pairs
// on 20,000 nodes) to grow the last bit of one dot into the tables' leading
// digits.
#pragma once

#include "sgns_device.h"
#include "wave.h"

namespace felog {

typedef float f2 __attribute__((ext_vector_type(2)));

// Most steps of pairs a batch takes: at most 4, its rows in at most 64
// registers, its touches in one lane each, its dots in the lanes of a row.
constexpr int fwd_max_steps(int D, int K)
{
    const int halves = D == 64 ? 2 : 1, lanes = 64 / halves, v = D / (2 * lanes);
    int b = 4;
    while (b > 1 &&
           (b * (K + 2) * v * 2 > 64 || b * halves * (K + 2) > 64 || b * (K + 1) > lanes))
        --b;
    return b;
}

template <int D, int K>
struct FwdShape {
    static constexpr int kHalves = D == 64 ? 2 : 1;   // pairs side by side
    static constexpr int kLanes = 64 / kHalves;       // lanes per row
    static constexpr int kV = D / (2 * kLanes);       // float2s per lane and row
    static constexpr int kT = K + 2;                  // touches per pair
};

// Sums of n values over the odd ones of L lanes, value by value: after the call
// v[0] of a lane is the sum of value lane_value(lane).
template <int N, int X, int A>
__device__ __forceinline__ void reduce_values(double (&v)[A])
{
    if constexpr (X == 1) {
        // the sums are in the odd lanes: the even ones take their first half
        constexpr int H = (N + 1) / 2;
        const bool odd = (__lane_id() & 1) != 0;
#pragma unroll
        for (int j = 0; j < H; ++j) {
            const double even = from_xor<1>(v[j]);
            v[j] = odd ? v[j + H < N ? j + H : j] : even;
        }
    } else {
        constexpr int H = (N + 1) / 2;
#pragma unroll
        for (int j = 0; j < H; ++j)
            v[j] = j + H < N ? pair_sums<X>(v[j], v[j + H < N ? j + H : j]) : xor_sum<X>(v[j]);
        reduce_values<H, X / 2>(v);
    }
}

// A lane (of L) that holds value v of N after reduce_values.
template <int N, int L>
constexpr int value_lane(int v)
{
    int lane = 0, n = N;
    for (int x = L / 2; x > 0; x /= 2) {
        const int h = (n + 1) / 2;
        if (n > 1 && v >= h) {
            lane |= x;
            v -= h;
        }
        n = h;
    }
    return lane;
}

// The value a lane holds; `first` is false in lanes that repeat another's.
template <int N, int X>
__device__ __forceinline__ int lane_value(int lane, bool& first)
{
    if constexpr (X == 0) {
        first = true;
        return 0;
    } else {
        constexpr int H = (N + 1) / 2;
        const int v = lane_value<H, X / 2>(lane, first);
        const bool up = (lane & X) != 0;
        const bool has = v + H < N;
        first = first && (!up || has);
        return up && has ? v + H : v;
    }
}

// Row accesses.  kPlain: cached.  kStream: stores with the nontemporal hint.
// kAgent: agent-scope relaxed atomics of 8 bytes, which neither hit nor leave
// lines in caches that other compute units do not see.
enum RowAccess { kPlain, kStream, kAgent };

// Element `at` of a row: a scalar row address plus a 32-bit lane offset where
// the row is wave-uniform.
__device__ __forceinline__ const f2* row_at(const f2* row, uint32_t at)
{
    return reinterpret_cast<const f2*>(reinterpret_cast<const char*>(row) + at * (uint32_t)sizeof(f2));
}
__device__ __forceinline__ f2* row_at(f2* row, uint32_t at)
{
    return reinterpret_cast<f2*>(reinterpret_cast<char*>(row) + at * (uint32_t)sizeof(f2));
}

template <RowAccess A>
__device__ __forceinline__ f2 load_row2(const f2* p)
{
    if constexpr (A == kAgent) {
        const unsigned long long x = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p),
                                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return __builtin_bit_cast(f2, x);
    } else {
        return *p;
    }
}
template <RowAccess A>
__device__ __forceinline__ void store_row2(f2* p, f2 v)
{
    if constexpr (A == kAgent)
        __hip_atomic_store(reinterpret_cast<unsigned long long*>(p),
                           __builtin_bit_cast(unsigned long long, v), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    else if constexpr (A == kStream)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

// One batch of S steps (S kHalves pairs, from pair `base` of the wave's np).
template <int D, int K, int S, RowAccess A>
struct FwdBatch {
    using Sh = FwdShape<D, K>;
    static constexpr int H = Sh::kHalves, L = Sh::kLanes, V = Sh::kV, T = Sh::kT;
    static constexpr int N = S * (K + 1);   // dots per half
    static_assert(N <= L && S * H * T <= 64, "a batch's dots and touches fit the lanes");

    int32_t ctx[S], row[S][K + 1];   // of this lane's pair (scalars when H == 1)
    f2 vin[S][V], vo[S][K + 1][V];
    double g;        // this lane's coefficient: touch `touch` of the wave's lanes
    int touch;       // m_row lane of the touch this lane evaluates
    bool mine;       // this lane is the one that stands for that touch

    // value of m in the lane that holds touch r of the pair of step b (this half's)
    static __device__ __forceinline__ int32_t of_pair(int32_t m, int p0, int p1, int r)
    {
        const int32_t a = __builtin_amdgcn_readlane(m, p0 * T + r);
        if constexpr (H == 1) return a;
        const int32_t c = __builtin_amdgcn_readlane(m, p1 * T + r);
        return (threadIdx.x & 32) ? c : a;
    }

    // Reads the batch's rows.  m_row: lane l holds the row of touch l of the
    // wave's pairs (-1 skipped).  Pairs past the last repeat it; they get zero
    // coefficients and store nothing.
    __device__ __forceinline__ void load(const float* tin, const float* tout, int32_t m_row,
                                         int base, int np)
    {
        const uint32_t gl = threadIdx.x & (L - 1);
#pragma unroll
        for (int b = 0; b < S; ++b) {
            const int p0 = min(base + b * H, np - 1), p1 = min(base + b * H + 1, np - 1);
            ctx[b] = of_pair(m_row, p0, p1, 0);
            const f2* ri = reinterpret_cast<const f2*>(tin + (int64_t)ctx[b] * D);
#pragma unroll
            for (int i = 0; i < V; ++i) vin[b][i] = load_row2<A>(row_at(ri, i * L + gl));
#pragma unroll
            for (int k = 0; k <= K; ++k) {
                row[b][k] = of_pair(m_row, p0, p1, 1 + k);
                // a skipped negative equals the centre: that row is read in its place
                const int32_t r = k > 0 && row[b][k] < 0 ? row[b][0] : row[b][k];
                const f2* ro = reinterpret_cast<const f2*>(tout + (int64_t)r * D);
#pragma unroll
                for (int i = 0; i < V; ++i) vo[b][k][i] = load_row2<A>(row_at(ro, i * L + gl));
            }
        }
    }

    // Dots and coefficients: g0 = lr (1 - sigma(s0)), gk = -lr sigma(sk) and 0
    // for a skipped negative, FP64.  The loss terms, -log sigma(s0) and
    // -log sigma(-sk), are added to lacc in FP64.
    __device__ __forceinline__ void coefficients(int32_t m_row, int base, int np, double lr,
                                                 double& lacc)
    {
        const int lane = threadIdx.x & 63;
        // a touch is skipped rarely: its row is cleared off the common path
        const int first = base * T, past = min(base + S * H, np) * T;
        if (__ballot(m_row < 0 && lane >= first && lane < past) != 0) {
#pragma unroll
            for (int b = 0; b < S; ++b)
#pragma unroll
                for (int k = 1; k <= K; ++k)
                    if (row[b][k] < 0)
#pragma unroll
                        for (int i = 0; i < V; ++i) vo[b][k][i] = f2{0.0f, 0.0f};
        }
        double s[N];
#pragma unroll
        for (int b = 0; b < S; ++b)
#pragma unroll
            for (int k = 0; k <= K; ++k) {
                // each chain: the even lane's elements, then the odd lane's
                double acc = 0.0;
#pragma unroll
                for (int i = 0; i < V; ++i)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        if (i + h > 0) acc = from_xor<1>(acc);
                        acc = fma((double)vin[b][i].x, (double)vo[b][k][i].x, acc);
                        acc = fma((double)vin[b][i].y, (double)vo[b][k][i].y, acc);
                    }
                s[b * (K + 1) + k] = acc;
            }
        reduce_values<N, L / 2>(s);
        // the FP64 copies of the rows are not kept across the exponential
#pragma unroll
        for (int b = 0; b < S; ++b)
#pragma unroll
            for (int i = 0; i < V; ++i) {
                asm volatile("" : "+v"(vin[b][i]));
#pragma unroll
                for (int k = 0; k <= K; ++k) asm volatile("" : "+v"(vo[b][k][i]));
            }
        bool one;
        const int v = lane_value<N, L / 2>(lane & (L - 1), one);
        const int b = v / (K + 1), k = v - b * (K + 1);
        const int p = base + b * H + (H == 2 ? lane >> 5 : 0);
        touch = min(p, np - 1) * T + 1 + k;
        const int32_t target = __shfl(m_row, touch);   // every lane takes part
        const bool ok = p < np && target >= 0;
        mine = one && ok;
        const double dk = s[0];
        const SigmaTerms t = sigma_terms(dk);
        g = k == 0 ? lr * (1.0 - t.sigma) : -lr * t.sigma;
        if (!ok) g = 0.0;
        if (mine) lacc += fmax(k == 0 ? -dk : dk, 0.0) + (double)t.l1p;
    }

    // Coefficient of touch k of the pair of step b, in every lane of its half.
    __device__ __forceinline__ double coef(int b, int k) const
    {
        const int l = value_lane<N, L>(b * (K + 1) + k);
        const double a = read_lane(g, l);
        if constexpr (H == 1) return a;
        const double c = read_lane(g, l + 32);
        return (threadIdx.x & 32) ? c : a;
    }

    // sum_k g_k out[t_k] of the pair of step b, rounded to FP32 once.
    __device__ __forceinline__ void in_delta(int b, const double (&gk)[K + 1], f2 (&o)[V]) const
    {
#pragma unroll
        for (int i = 0; i < V; ++i) {
            double x = gk[0] * (double)vo[b][0][i].x, y = gk[0] * (double)vo[b][0][i].y;
#pragma unroll
            for (int k = 1; k <= K; ++k) {
                x = fma(gk[k], (double)vo[b][k][i].x, x);
                y = fma(gk[k], (double)vo[b][k][i].y, y);
            }
            o[i] = f2{(float)x, (float)y};
        }
    }

    // out[t_k] + g_k in[ctx] (from: the row, or zero), rounded to FP32 once.
    __device__ __forceinline__ f2 out_row(int b, int i, double gk, f2 from) const
    {
        return f2{(float)fma(gk, (double)vin[b][i].x, (double)from.x),
                  (float)fma(gk, (double)vin[b][i].y, (double)from.y)};
    }
};

}  // namespace felog
