// Embedding initialisation and the negative-sampling noise distribution
// Pn(u) of Eq. (2).
//
// Pn(u) ~ c_u^0.75, where c is a node's degree or its occurrence count in a
// walk corpus.  Weights are integers, W_u = floor(2^16 * sqrt(c) * sqrt(sqrt(c)))
// in IEEE double (sqrt and multiply correctly rounded), so the cumulative
// weights are exact and a draw is the exact inverse CDF of a 64-bit uniform:
// u = floor(x * T / 2^64), answer = the node whose interval [cdf[i], cdf[i+1])
// holds u.  A guide table (Chen & Asau's indexed search) over the top bits of
// x gives a starting node no larger than the answer, from which a short
// forward scan finds it: O(1) expected reads per draw.
#include <algorithm>

#include "common.h"
#include "noise.h"

namespace felog {

// in[v][c] = ((x >> 8) * 2^-24 - 0.5) / d, x = word c mod 4 of Philox(v, c/4, 0, INIT).
__global__ void init_tables_kernel(float* __restrict__ tin, int32_t n, int32_t d, uint64_t seed)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;   // one thread per 4 entries
    int64_t quads = (int64_t)n * (d / 4);
    if (i >= quads) return;
    int64_t v = i / (d / 4);
    uint32_t c4 = (uint32_t)(i - v * (d / 4));
    Rand4 r = philox4x32((uint32_t)v, (uint32_t)(v >> 32), c4, kTagInit, seed);
    float4 o;
    const float inv = 1.0f / 16777216.0f;
    o.x = ((float)(r.v[0] >> 8) * inv - 0.5f) / (float)d;
    o.y = ((float)(r.v[1] >> 8) * inv - 0.5f) / (float)d;
    o.z = ((float)(r.v[2] >> 8) * inv - 0.5f) / (float)d;
    o.w = ((float)(r.v[3] >> 8) * inv - 0.5f) / (float)d;
    reinterpret_cast<float4*>(tin)[i] = o;
}

void launch_init_tables(Model& m, uint64_t seed)
{
    Ctx& c = *m.ctx;
    int64_t quads = (int64_t)m.g->n * (m.dim / 4);
    hipLaunchKernelGGL(init_tables_kernel, dim3((quads + 255) / 256), dim3(256), 0, c.stream,
                       m.tin.as<float>(), m.g->n, m.dim, seed);
    FELOG_HIP(hipGetLastError());
    FELOG_HIP(hipMemsetAsync(m.tout.ptr, 0, sizeof(float) * (size_t)m.g->n * m.dim, c.stream));
}

__global__ void degree_counts_kernel(const int64_t* indptr, int32_t n, uint32_t* counts)
{
    int32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n) counts[v] = (uint32_t)(indptr[v + 1] - indptr[v]);
}

void launch_degree_counts(Graph& g, uint32_t* d_counts)
{
    Ctx& c = *g.ctx;
    hipLaunchKernelGGL(degree_counts_kernel, dim3((g.n + 255) / 256), dim3(256), 0, c.stream,
                       g.indptr.as<int64_t>(), g.n, d_counts);
    FELOG_HIP(hipGetLastError());
}

// Occurrences of each node in a walk corpus, and of the padding (integer sums:
// order-free).
//
// Device-scope atomics meet beyond the XCDs' L2s and run at 10 to 45 G/s, a
// fiftieth of the rate at which the corpus can be read.  A workgroup therefore
// counts one range of nodes over one part of the corpus in LDS: the corpus is
// read once per range (the ranges of a part are on one XCD and share its L2),
// and the parts' counts are stored and summed without atomics.  41.9 M positions
// over 2^17 nodes: 2.36 ms -> 64 us, and 17 us for the sum.
constexpr int kCountRange = 40960;        // counters of a workgroup: all of a CU's LDS
constexpr int kCountThreads = 1024;
constexpr int kCountInFlight = 4;         // 16-byte loads of a thread
// The time grows with the ranges (104 M positions over 1.3 M nodes, 32 ranges,
// where a part is an eighth of the corpus: 0.99 ms against 3.03 by atomics);
// beyond 32 the parts no longer fill the XCDs.  At 2^20 positions the atomics
// take 118 us and the parts 16 plus the allocation of their counts.
constexpr int kCountRangesMax = 32;
constexpr int64_t kCountPositionsMin = (int64_t)1 << 20;
// Fewest parts: with 26 ranges of 2^20 nodes and one part of 4.2 M positions, 26
// workgroups take 250 us; 32-bit atomics take 50, 160 for twice the positions and
// 390 for four times, where four parts take 250 (the codec's 64-bit atomics 240,
// 380 and 650).
template <class T>
constexpr int64_t count_parts_min() { return sizeof(T) == 8 ? 2 : 4; }

// Adds a workgroup's paddings: one atomic, for they all meet at one address
// (4 ns each).  s: a word per wave; below 2^32 paddings in a workgroup.
__device__ __forceinline__ void add_pads(unsigned long long* pads, uint32_t mine, uint32_t* s)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (uint32_t i = 1; i < blockDim.x / 64; ++i) mine += s[i];
        if (mine) atomicAdd(pads, (unsigned long long)mine);
    }
}

template <class T>
__global__ __launch_bounds__(256) void node_counts_kernel(const int32_t* __restrict__ data,
                                                          int64_t total, T* counts,
                                                          unsigned long long* pads)
{
    __shared__ uint32_t waves[4];
    uint32_t mine = 0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * 256) {
        const int32_t v = data[i];
        if (v >= 0) atomicAdd(&counts[v], (T)1);
        else ++mine;
    }
    if (pads) add_pads(pads, mine, waves);
}

// Block r * parts + p: the nodes [r * range, (r + 1) * range) over positions
// [p * span, (p + 1) * span), span a multiple of 4; data is 16-byte aligned.
__global__ __launch_bounds__(kCountThreads) void node_count_parts_kernel(
    const int32_t* __restrict__ data, int64_t total, int64_t span, int32_t parts, int32_t n,
    int32_t range, uint32_t* __restrict__ out, unsigned long long* pads)
{
    __shared__ uint32_t cnt[kCountRange];
    const int32_t part = (int32_t)(blockIdx.x % (uint32_t)parts);
    const int32_t lo = (int32_t)(blockIdx.x / (uint32_t)parts) * range;
    const uint32_t width = (uint32_t)min(range, n - lo);
    for (uint32_t i = threadIdx.x; i < width; i += kCountThreads) cnt[i] = 0;
    __syncthreads();
    const int64_t begin = (int64_t)part * span, end = min(begin + span, total);
    uint32_t mine = 0;
    auto count = [&](int32_t v) {
        const uint32_t at = (uint32_t)v - (uint32_t)lo;   // a padding -1 is beyond every width
        if (at < width) atomicAdd(&cnt[at], 1u);
        mine += v < 0 ? 1u : 0u;
    };
    const int64_t quads = end > begin ? (end - begin) >> 2 : 0;
    const int4* rows = reinterpret_cast<const int4*>(data + begin);
    for (int64_t q0 = threadIdx.x; q0 < quads; q0 += kCountInFlight * kCountThreads) {
        int4 v[kCountInFlight];
#pragma unroll
        for (int u = 0; u < kCountInFlight; ++u)
            v[u] = rows[min(q0 + u * kCountThreads, quads - 1)];
#pragma unroll
        for (int u = 0; u < kCountInFlight; ++u)
            if (q0 + u * kCountThreads < quads) {
                count(v[u].x);
                count(v[u].y);
                count(v[u].z);
                count(v[u].w);
            }
    }
    for (int64_t i = begin + 4 * quads + threadIdx.x; i < end; i += kCountThreads) count(data[i]);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < width; i += kCountThreads)
        out[(int64_t)part * n + lo + i] = cnt[i];
    if (pads && lo == 0) {
        __syncthreads();
        add_pads(pads, mine, cnt);
    }
}

template <class T>
__global__ __launch_bounds__(256) void node_count_sum_kernel(const uint32_t* __restrict__ in,
                                                             int32_t parts, int32_t n, T* counts)
{
    const int32_t v = blockIdx.x * 256 + threadIdx.x;
    if (v >= n) return;
    T s = 0;
    for (int32_t p = 0; p < parts; ++p) s += in[(int64_t)p * n + v];
    counts[v] = s;
}

template <class T>
void launch_node_counts(const Walks& w, T* counts, unsigned long long* pads, DevBuf& buf)
{
    Ctx& c = *w.g->ctx;
    const int32_t n = w.g->n;
    const int64_t total = w.W * (int64_t)w.L;
    const int32_t* data = w.data.as<int32_t>();
    if (pads) FELOG_HIP(hipMemsetAsync(pads, 0, sizeof *pads, c.stream));
    const int64_t ranges = (n + kCountRange - 1) / (int64_t)kCountRange;
    if (total >= kCountPositionsMin && ranges <= kCountRangesMax) {
        // one workgroup per CU; a multiple of 8 parts puts a part's ranges on
        // one XCD; the parts' counts take at most a quarter of the corpus
        int64_t parts = std::min<int64_t>(c.num_cus / ranges, total / (4 * (int64_t)n));
        parts = parts >= 8 ? parts / 8 * 8 : parts;
        // a part's counts fit 32 bits
        if (parts >= count_parts_min<T>() && total / parts < ((int64_t)1 << 32) - 4 &&
            try_alloc(buf, &c, sizeof(uint32_t) * (size_t)(parts * n))) {
            const int32_t range = (int32_t)((n + ranges - 1) / ranges);
            const int64_t span = ((total + parts - 1) / parts + 3) / 4 * 4;
            hipLaunchKernelGGL(node_count_parts_kernel, dim3((uint32_t)(ranges * parts)),
                               dim3(kCountThreads), 0, c.stream, data, total, span, (int32_t)parts,
                               n, range, buf.as<uint32_t>(), pads);
            hipLaunchKernelGGL(node_count_sum_kernel<T>, dim3((n + 255) / 256), dim3(256), 0,
                               c.stream, buf.as<uint32_t>(), (int32_t)parts, n, counts);
            FELOG_HIP(hipGetLastError());
            return;
        }
    }
    FELOG_HIP(hipMemsetAsync(counts, 0, sizeof(T) * n, c.stream));
    if (total == 0) return;
    const int64_t blocks = std::min<int64_t>((total + 255) / 256, (int64_t)c.num_cus * 16);
    hipLaunchKernelGGL(node_counts_kernel<T>, dim3(blocks), dim3(256), 0, c.stream, data, total,
                       counts, pads);
    FELOG_HIP(hipGetLastError());
}

void launch_corpus_counts(const Walks& w, uint32_t* d_counts, DevBuf& work)
{
    launch_node_counts<uint32_t>(w, d_counts, nullptr, work);
}

void launch_symbol_counts(const Walks& w, unsigned long long* d_counts,
                          unsigned long long* d_pads)
{
    DevBuf work;
    launch_node_counts<unsigned long long>(w, d_counts, d_pads, work);
    if (work.ptr) w.g->ctx->sync();   // before it is given back
}

// W_u = floor(2^16 * sqrt(c) * sqrt(sqrt(c))).
__global__ void noise_weights_kernel(const uint32_t* counts, int32_t n, uint64_t* w)
{
    int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double c = (double)counts[i];
    double s = __dsqrt_rn(c);
    double t = __dsqrt_rn(s);
    double x = __dmul_rn(s, t);
    w[i] = (uint64_t)__dmul_rn(x, 65536.0);
}

// Inclusive scan of 64-bit weights into cdf[1..n] (cdf[0] = 0), three passes.
__global__ __launch_bounds__(256) void block_sums_u64(const uint64_t* w, int32_t n,
                                                      uint64_t* sums)
{
    __shared__ uint64_t lds[256];
    int64_t base = (int64_t)blockIdx.x * 2048 + threadIdx.x * 8;
    uint64_t acc = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k)
        if (base + k < n) acc += w[base + k];
    lds[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) lds[threadIdx.x] += lds[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[blockIdx.x] = lds[0];
}

__global__ __launch_bounds__(256) void scan_sums_u64(uint64_t* sums, int64_t nb)
{
    // one block: exclusive scan in place, total written to sums[nb]
    __shared__ uint64_t lds[256];
    uint64_t carry = 0;
    for (int64_t s = 0; s < nb; s += 256) {
        int64_t i = s + threadIdx.x;
        uint64_t v = i < nb ? sums[i] : 0;
        lds[threadIdx.x] = v;
        __syncthreads();
        for (int off = 1; off < 256; off <<= 1) {
            uint64_t add = threadIdx.x >= off ? lds[threadIdx.x - off] : 0;
            __syncthreads();
            lds[threadIdx.x] += add;
            __syncthreads();
        }
        if (i < nb) sums[i] = carry + lds[threadIdx.x] - v;
        uint64_t tot = lds[255];
        __syncthreads();
        carry += tot;
    }
    if (threadIdx.x == 0) sums[nb] = carry;
}

__global__ __launch_bounds__(256) void finish_cdf_u64(const uint64_t* w, int32_t n,
                                                      const uint64_t* offsets, uint64_t* cdf)
{
    __shared__ uint64_t lds[256];
    int64_t base = (int64_t)blockIdx.x * 2048 + threadIdx.x * 8;
    uint64_t vals[8];
    uint64_t acc = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        vals[k] = base + k < n ? w[base + k] : 0;
        acc += vals[k];
    }
    lds[threadIdx.x] = acc;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        uint64_t add = threadIdx.x >= off ? lds[threadIdx.x - off] : 0;
        __syncthreads();
        lds[threadIdx.x] += add;
        __syncthreads();
    }
    uint64_t run = offsets[blockIdx.x] + lds[threadIdx.x] - acc;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        if (base + k < n) {
            run += vals[k];
            cdf[base + k + 1] = run;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) cdf[0] = 0;
}

// guide[b] = first node whose interval reaches past the smallest u of bucket b.
__global__ void guide_kernel(const uint64_t* cdf, int32_t n, int32_t bits, uint64_t total,
                             int32_t* guide)
{
    int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= (int64_t)1 << bits) return;
    uint64_t x = (uint64_t)b << (64 - bits);
    uint64_t u = __umul64hi(x, total);
    int32_t lo = 0, hi = n - 1;
    while (lo < hi) {
        int32_t mid = lo + (hi - lo) / 2;
        if (cdf[mid + 1] > u) hi = mid; else lo = mid + 1;
    }
    guide[b] = lo;
}

// Room for a new table; training is refused until build_guide has ended.
static void alloc_cdf(Model& m)
{
    m.have_noise = false;
    const size_t bytes = sizeof(uint64_t) * ((size_t)m.g->n + 1);
    if (m.cdf.bytes != bytes) m.cdf.alloc(m.ctx, bytes);
}

// guide table of m.cdf (n + 1 entries, total > 0)
static void build_guide(Model& m, uint64_t total)
{
    Ctx& c = *m.ctx;
    const int32_t n = m.g->n;
    int32_t bits = 1;
    while (bits < 31 && ((int64_t)1 << bits) < n) ++bits;
    m.guide_bits = bits;
    m.total_weight = total;
    const size_t bytes = sizeof(int32_t) * ((size_t)1 << bits);
    if (m.guide.bytes != bytes) m.guide.alloc(&c, bytes);
    hipLaunchKernelGGL(guide_kernel, dim3((((int64_t)1 << bits) + 255) / 256), dim3(256), 0,
                       c.stream, m.cdf.as<uint64_t>(), n, bits, total, m.guide.as<int32_t>());
    FELOG_HIP(hipGetLastError());
    c.sync();
    m.have_noise = true;
}

void set_noise_cdf(Model& m, const uint64_t* host_cdf)
{
    Ctx& c = *m.ctx;
    const int32_t n = m.g->n;
    FELOG_REQUIRE(host_cdf[0] == 0, "a noise table starts at 0");
    for (int32_t i = 0; i < n; ++i)
        FELOG_REQUIRE(host_cdf[i + 1] >= host_cdf[i], "the noise table decreases at node %d", i);
    FELOG_REQUIRE(host_cdf[n] > 0, "the noise distribution is empty (every weight is zero)");
    alloc_cdf(m);
    FELOG_HIP(hipMemcpyAsync(m.cdf.ptr, host_cdf, sizeof(uint64_t) * (n + 1),
                             hipMemcpyHostToDevice, c.stream));
    build_guide(m, host_cdf[n]);
}

void build_noise_from_counts(Model& m, const uint32_t* d_counts, DevBuf& w)
{
    Ctx& c = *m.ctx;
    int32_t n = m.g->n;
    // the weights go where the counts of parts were (a large block given back and
    // another taken can cost 300 us), but no budget pays for more than they need
    if (w.bytes < sizeof(uint64_t) * n || c.budget) {
        if (w.ptr) c.sync();
        w.alloc(&c, sizeof(uint64_t) * n);
    }
    hipLaunchKernelGGL(noise_weights_kernel, dim3((n + 255) / 256), dim3(256), 0, c.stream,
                       d_counts, n, w.as<uint64_t>());
    FELOG_HIP(hipGetLastError());
    int64_t nb = (n + 2047) / 2048;
    DevBuf sums;
    sums.alloc(&c, sizeof(uint64_t) * (nb + 1));
    hipLaunchKernelGGL(block_sums_u64, dim3(nb), dim3(256), 0, c.stream, w.as<uint64_t>(), n,
                       sums.as<uint64_t>());
    hipLaunchKernelGGL(scan_sums_u64, dim3(1), dim3(256), 0, c.stream, sums.as<uint64_t>(), nb);
    FELOG_HIP(hipGetLastError());
    uint64_t total = 0;
    FELOG_HIP(hipMemcpyAsync(&total, sums.as<uint64_t>() + nb, sizeof total,
                             hipMemcpyDeviceToHost, c.stream));
    c.sync();
    // (the model keeps the table that it has)
    FELOG_REQUIRE(total > 0, "the noise distribution is empty (every count is zero)");
    alloc_cdf(m);
    hipLaunchKernelGGL(finish_cdf_u64, dim3(nb), dim3(256), 0, c.stream, w.as<uint64_t>(), n,
                       sums.as<uint64_t>(), m.cdf.as<uint64_t>());
    FELOG_HIP(hipGetLastError());
    build_guide(m, total);
}

}  // namespace felog
