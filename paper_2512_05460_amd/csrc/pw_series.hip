// Binary64 reference quantities on the device: the truncated series (Lemma 2.3)
// and the mixing factor (section 2.1).
//
// The series h_L = sum_{i <= L} P^i v_0 is formed by h <- v_0 + P h: one matrix
// of columns instead of three (the term, the next term, the running sum), and
// with v_0's two entries a column known to the kernel one gather and one write
// per step. Errors do not grow with the number of terms added as they do in
// the running sum (measured against long double: at most the sum's).
#include <algorithm>

#include "pw_internal.hpp"

namespace pw {

// Neighbour ids, 4 bytes or packed in 3 (8 bytes of padding follow).
struct RowTables {
    const uint32_t* rp;
    const uint32_t* col;
    const uint32_t* col24;
    __device__ __forceinline__ uint32_t at(uint32_t i) const
    {
        if (!col24) return col[i];
        uint32_t v;
        __builtin_memcpy(&v, reinterpret_cast<const char*>(col24) + (size_t)i * 3u, 4);
        return v & 0xFFFFFFu;
    }
};

// V columns that a lane sums at once: two are a 16-byte load.
template <int V>
struct Cols {
    double v[V];
    __device__ __forceinline__ void add(const Cols& o)
    {
#pragma unroll
        for (int i = 0; i < V; ++i) v[i] += o.v[i];
    }
};

template <int V>
__device__ __forceinline__ Cols<V> load_cols(const double* p)
{
    typedef double f64x2 __attribute__((ext_vector_type(2)));
    Cols<V> r;
    if constexpr (V == 2) {
        const f64x2 w = *reinterpret_cast<const f64x2*>(p);
        r.v[0] = w.x;
        r.v[1] = w.y;
    } else {
        r.v[0] = *p;
    }
    return r;
}

// Sum of columns c .. c + V of H (C columns a row) over entries b + slot,
// b + slot + slots, ... < e: four loads in flight, four partial sums in a fixed
// order.
template <int C, int V>
__device__ __forceinline__ Cols<V> row_part(const RowTables& g, const double* H, uint32_t b, uint32_t e, uint32_t slot,
                                            uint32_t slots, uint32_t c)
{
    Cols<V> a0{}, a1{}, a2{}, a3{};
    uint32_t i = b + slot;
    for (; i + 3u * slots < e; i += 4u * slots) {
        const uint32_t u0 = g.at(i), u1 = g.at(i + slots), u2 = g.at(i + 2u * slots), u3 = g.at(i + 3u * slots);
        const Cols<V> v0 = load_cols<V>(H + (size_t)u0 * C + c), v1 = load_cols<V>(H + (size_t)u1 * C + c);
        const Cols<V> v2 = load_cols<V>(H + (size_t)u2 * C + c), v3 = load_cols<V>(H + (size_t)u3 * C + c);
        a0.add(v0);
        a1.add(v1);
        a2.add(v2);
        a3.add(v3);
    }
    if (i < e) a0.add(load_cols<V>(H + (size_t)g.at(i) * C + c));
    if (i + slots < e) a1.add(load_cols<V>(H + (size_t)g.at(i + slots) * C + c));
    if (i + 2u * slots < e) a2.add(load_cols<V>(H + (size_t)g.at(i + 2u * slots) * C + c));
    a0.add(a1);
    a2.add(a3);
    a0.add(a2);
    return a0;
}

template <int kCtrl>
__device__ __forceinline__ double dpp_add(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), kCtrl, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), kCtrl, 0xF, 0xF, false);
    return v + __hiloint2double(hi, lo);
}
// the sum over a lane's group of four, or of 16, in every lane of it
__device__ __forceinline__ double quad_sum(double v)
{
    return dpp_add<0x4E>(dpp_add<0xB1>(v));  // quad_perm 1 0 3 2, then 2 3 0 1
}
__device__ __forceinline__ double row_sum16(double v)
{
    return dpp_add<0x140>(dpp_add<0x141>(quad_sum(v)));  // mirrored halves of 8, then of 16
}

// the sum over the wave in every lane
__device__ __forceinline__ double wave_sum(double v)
{
    v = row_sum16(v);
    v += __shfl_xor(v, 16);
    return v + __shfl_xor(v, 32);
}

// One value per thread summed over the threads of each column (thread t has
// column t % C) in a fixed tree; the sums are in threads 0 .. C-1.
template <int C>
__device__ __forceinline__ double block_columns(double v, double* lds)
{
    lds[threadIdx.x] = v;
    __syncthreads();
    for (uint32_t w = 128; w >= (uint32_t)C; w >>= 1) {
        if (threadIdx.x < w) lds[threadIdx.x] += lds[threadIdx.x + w];
        __syncthreads();
    }
    const double s = lds[threadIdx.x & (C - 1)];
    __syncthreads();
    return s;
}

// ---------------------------------------------------------------------------
// Truncated series on any graph. The columns are cut into slabs of C (16 where
// there are that many), each slab an n x C matrix of its own, and consecutive
// work groups take consecutive slabs, so that every XCD works on few slabs and
// its 4 MB L2 holds their often-read rows. The step is bound by the gather of
// nnz x 8 Q bytes, by L2 misses first: a row of 16 columns is one 128-byte line,
// all of which is used. A lane owns V columns of a row (two: 16-byte loads; P lanes
// share the neighbours where C or the graph is small), and rows of more than kHubDegree
// neighbours, which would keep their wave for long after the others have ended,
// get a work group each.
// Chung-Lu-like graph, n = 1e5, 1e6 entries, 64 columns, a step: 417 us as one
// wave per row over 64-column rows; 63 us so (slabs of 8: 80 us, of 32: 63 us;
// 8,192 waves looping over the rows instead of a wave a row: 91 us).
// ---------------------------------------------------------------------------
template <int C, int P, int V>
__global__ __launch_bounds__(256) void series_step_kernel(RowTables g, uint32_t n, const uint32_t* hubs, uint32_t nhub,
                                                          uint32_t sbits, uint32_t slabs, const SeriesSeeds* seeds,
                                                          const double* H, double* Y)
{
    __shared__ double lds[256];
    constexpr uint32_t kColLanes = C / V, kLanes = kColLanes * P, kRowsAtOnce = 256u / kLanes;
    const uint32_t slab = blockIdx.x & ((1u << sbits) - 1u);
    if (slab >= slabs) return;  // the whole work group (of three slabs)
    const uint32_t c = (threadIdx.x & (kColLanes - 1u)) * V, q = slab * C + c;
    uint32_t s[V], t[V];
    double vs[V], vt[V];
#pragma unroll
    for (int i = 0; i < V; ++i) {
        s[i] = seeds->s[q + i];
        t[i] = seeds->t[q + i];
        vs[i] = seeds->vs[q + i];
        vt[i] = seeds->vt[q + i];
    }
    H += (size_t)slab * n * C;
    Y += (size_t)slab * n * C;
    auto finish = [&](uint32_t row, const Cols<V>& sum, uint32_t d) {
#pragma unroll
        for (int i = 0; i < V; ++i) {
            double y = sum.v[i] / (double)d;
            if (row == s[i]) y += vs[i];
            if (row == t[i]) y += vt[i];
            Y[(size_t)row * C + c + i] = y;
        }
    };
    const uint32_t item = blockIdx.x >> sbits;
    if (item < nhub) {
        const uint32_t row = hubs[item], b = g.rp[row], e = g.rp[row + 1];
        Cols<V> sum = row_part<C, V>(g, H, b, e, threadIdx.x / kColLanes, 256u / kColLanes, c);
#pragma unroll
        for (int i = 0; i < V; ++i) sum.v[i] = block_columns<kColLanes>(sum.v[i], lds);
        if (threadIdx.x < kColLanes) finish(row, sum, e - b);
    } else {
        const uint32_t row = (item - nhub) * kRowsAtOnce + threadIdx.x / kLanes;
        if (row >= n) return;  // (all lanes of a row leave together, here and below)
        const uint32_t b = g.rp[row], e = g.rp[row + 1];
        if (e - b > kHubDegree) return;
        Cols<V> sum = row_part<C, V>(g, H, b, e, (threadIdx.x / kColLanes) & (P - 1u), P, c);
        for (uint32_t off = kColLanes; off < kLanes; off <<= 1) {
#pragma unroll
            for (int i = 0; i < V; ++i) sum.v[i] += __shfl_xor(sum.v[i], (int)off);
        }
        if ((threadIdx.x & (kLanes - 1u) & ~(kColLanes - 1u)) == 0u) finish(row, sum, e - b);
    }
}

// v_0; and the seeds left in memory for the steps, whose launches are a
// microsecond each longer with 1.5 KB of arguments.
template <int C>
__global__ __launch_bounds__(256) void series_start_kernel(uint32_t n, uint32_t sbits, uint32_t slabs, SeriesSeeds seeds,
                                                           double* H, SeriesSeeds* kept)
{
    if (blockIdx.x == 0 && threadIdx.x < 64u) {
        kept->s[threadIdx.x] = seeds.s[threadIdx.x];
        kept->t[threadIdx.x] = seeds.t[threadIdx.x];
        kept->vs[threadIdx.x] = seeds.vs[threadIdx.x];
        kept->vt[threadIdx.x] = seeds.vt[threadIdx.x];
    }
    const uint32_t slab = blockIdx.x & ((1u << sbits) - 1u), item = blockIdx.x >> sbits;
    const uint32_t c = threadIdx.x & (C - 1u), q = slab * C + c;
    const uint32_t row = item * (256u / C) + threadIdx.x / C;
    if (row >= n || slab >= slabs) return;
    H[((size_t)slab * n + row) * C + c] = row == seeds.s[q] ? seeds.vs[q] : row == seeds.t[q] ? seeds.vt[q] : 0.0;
}

// ||h||^2 and 1^T h of each column in a fixed order: kSeriesParts row ranges,
// then (second kernel) one work group a column.
template <int C>
__global__ __launch_bounds__(256) void series_sums_kernel(uint32_t n, uint32_t sbits, uint32_t slabs, const double* H,
                                                          double* part)
{
    __shared__ double lds[256];
    const uint32_t slab = blockIdx.x & ((1u << sbits) - 1u), item = blockIdx.x >> sbits;
    const uint32_t c = threadIdx.x & (C - 1u);
    if (slab >= slabs) return;
    double sq = 0.0, lin = 0.0;
    for (uint32_t row = item * (256u / C) + threadIdx.x / C; row < n; row += kSeriesParts * (256u / C)) {
        const double h = H[((size_t)slab * n + row) * C + c];
        sq += h * h;
        lin += h;
    }
    sq = block_columns<C>(sq, lds);
    lin = block_columns<C>(lin, lds);
    if (threadIdx.x < C) {
        double* p = part + ((size_t)(slab * C + c) * kSeriesParts + item) * 2;
        p[0] = sq;
        p[1] = lin;
    }
}

__global__ __launch_bounds__(256) void series_finish_kernel(uint32_t n, const double* part, double* beta)
{
    __shared__ double lds[256];
    const double* p = part + (size_t)blockIdx.x * kSeriesParts * 2;
    double sq = 0.0, lin = 0.0;
    for (uint32_t i = threadIdx.x; i < kSeriesParts; i += 256u) {
        sq += p[2 * i];
        lin += p[2 * i + 1];
    }
    sq = block_columns<1>(sq, lds);
    lin = block_columns<1>(lin, lds);
    if (threadIdx.x == 0) beta[blockIdx.x] = sq - lin * lin / (double)n;
}

template <int C, int P, int V>
static hipError_t series_on(const RowTables& g, uint32_t n, const uint32_t* hubs, uint32_t nhub, uint32_t sbits,
                            uint32_t Q, int32_t L, const SeriesSeeds& seeds, double* H, double* Y, double* part,
                            double* beta, hipStream_t st)
{
    const uint32_t per = 256u / (C / V * P), rows = (n + per - 1) / per, all = (n + 256u / C - 1) / (256u / C);
    const uint32_t slabs = series_slabs(Q);
    const dim3 block(256);
    SeriesSeeds* kept = reinterpret_cast<SeriesSeeds*>(part + (size_t)C * slabs * kSeriesParts * 2);
    hipLaunchKernelGGL((series_start_kernel<C>), dim3(all << sbits), block, 0, st, n, sbits, slabs, seeds, H, kept);
    for (int32_t i = 0; i < L; ++i) {
        hipLaunchKernelGGL((series_step_kernel<C, P, V>), dim3((rows + nhub) << sbits), block, 0, st, g, n, hubs, nhub, sbits,
                           slabs, kept, H, Y);
        std::swap(H, Y);
    }
    hipLaunchKernelGGL((series_sums_kernel<C>), dim3(kSeriesParts << sbits), block, 0, st, n, sbits, slabs, H, part);
    hipLaunchKernelGGL(series_finish_kernel, dim3(Q), block, 0, st, n, part, beta);
    return hipGetLastError();
}

// Rows (of all slabs) up to which a row's lanes are a wave or half of one: with
// fewer rows than that, lanes of their own for a row's columns alone leave most of
// the device idle and a long row's reads one after another. A step (a
// microsecond of it since saved in the launch) at n = 3,000, 62 neighbours a row,
// 1, 8 and 16 columns: 5.1, 6.6, 7.0 us so, 6.3, 10.9, 12.3 else; n = 10,000, 10 a
// row, 48 columns 18.2 so, 15.8 else.
constexpr uint32_t kSeriesWaveRows = 8000;

uint32_t series_columns(uint32_t Q)
{
    return Q > 8 ? 16 : Q > 4 ? 8 : Q > 2 ? 4 : Q;
}

uint32_t series_slabs(uint32_t Q)
{
    return (Q + series_columns(Q) - 1) / series_columns(Q);
}

hipError_t launch_series(const uint32_t* rp, const uint32_t* col, const uint32_t* col24, uint32_t n,
                         const uint32_t* hubs, uint32_t nhub, uint32_t Q, int32_t L, const SeriesSeeds& seeds, double* H,
                         double* Y, double* part, double* beta, hipStream_t st)
{
    const RowTables g{rp, col, col24};
    uint32_t sbits = 0;
    while ((1u << sbits) < series_slabs(Q)) ++sbits;
    auto on = [&](auto narrow, auto wave) {
        return ((uint64_t)n << sbits) > kSeriesWaveRows ? narrow(g, n, hubs, nhub, sbits, Q, L, seeds, H, Y, part, beta, st)
                                                           : wave(g, n, hubs, nhub, sbits, Q, L, seeds, H, Y, part, beta, st);
    };
    switch (series_columns(Q)) {
    case 1: return on(series_on<1, 4, 1>, series_on<1, 64, 1>);
    case 2: return on(series_on<2, 4, 2>, series_on<2, 32, 1>);
    case 4: return on(series_on<4, 2, 2>, series_on<4, 16, 1>);
    case 8: return on(series_on<8, 1, 2>, series_on<8, 16, 2>);
    default: return on(series_on<16, 1, 2>, series_on<16, 8, 2>);
    }
}

// ---------------------------------------------------------------------------
// Truncated series on a small graph: one work group a pair runs all L steps
// with the column (two copies in turn) and the adjacency in LDS, so a step costs
// one barrier instead of a launch, and the instructions of one CU bound it: a
// read, an add and half an unpacking per neighbour. Rows of up to kShort
// neighbours take a lane, which keeps their ids in registers (they are the same
// in every step), in descending order of their length so that a wave's rows
// need equally many reads; longer rows take 16 lanes that read the ids from LDS
// and add up by DPP.
// n = 1,000, 6,000 entries, 3 pairs, L = 200: 815 us as 200 launches, the kernel 333
// us with four lanes a row (more instructions for the sums than for the reads), 212
// us of a call's 245 so.
// ---------------------------------------------------------------------------
constexpr uint32_t kLaneRows = kSeriesSmallNodes / 1024, kShort = kSeriesShortRow;

__global__ __launch_bounds__(1024) void series_small_kernel(const uint4* tab, uint32_t nrow, uint32_t idw, uint32_t n,
                                                            int32_t L, const SeriesPair* pairs, double* beta)
{
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ uint32_t count[kShort + 1], place[kShort + 1];  // rows of kShort, kShort - 1, ... neighbours, then long ones
    double* h = reinterpret_cast<double*>(lds);                            // n doubles, now and next
    double* next = h + n;
    uint4* t4 = reinterpret_cast<uint4*>(lds + ((16u * n + 15u) & ~15u));
    const uint32_t* rows = reinterpret_cast<const uint32_t*>(t4);          // row offset | degree << 16
    const uint16_t* ids = reinterpret_cast<const uint16_t*>(rows + nrow);  // 4 x neighbour id
    uint16_t* order = reinterpret_cast<uint16_t*>(const_cast<uint32_t*>(rows) + nrow + idw);  // rows by length, long ones last
    for (uint32_t i = threadIdx.x; i < (nrow + idw) / 4u; i += 1024u) t4[i] = tab[i];
    const SeriesPair pr = pairs[blockIdx.x];
    for (uint32_t x = threadIdx.x; x < n; x += 1024u) h[x] = x == pr.s ? pr.vs : x == pr.t ? pr.vt : 0.0;
    if (threadIdx.x <= kShort) count[threadIdx.x] = 0u;
    __syncthreads();
    auto class_of = [&](uint32_t x) {
        const uint32_t d = rows[x] >> 16;
        return d > kShort ? kShort : kShort - d;
    };
    for (uint32_t x = threadIdx.x; x < n; x += 1024u) atomicAdd(&count[class_of(x)], 1u);
    __syncthreads();
    if (threadIdx.x <= kShort) {
        uint32_t at = 0;
        for (uint32_t c = 0; c < threadIdx.x; ++c) at += count[c];
        place[threadIdx.x] = at;
    }
    __syncthreads();
    for (uint32_t x = threadIdx.x; x < n; x += 1024u) order[atomicAdd(&place[class_of(x)], 1u)] = (uint16_t)x;
    __syncthreads();
    const uint32_t nl = count[kShort], ns = n - nl;
    // this lane's rows: kept: 8 x the ids, two a word; have: how many; most: the
    // most that a lane of the wave has; 1/d
    uint32_t kept[kLaneRows][kShort / 2], have[kLaneRows], most[kLaneRows], mine[kLaneRows];
    double inv[kLaneRows];
#pragma unroll
    for (uint32_t k = 0; k < kLaneRows; ++k) {
        const uint32_t i = threadIdx.x + 1024u * k, x = i < ns ? order[i] : n;
        const uint32_t w = x < n ? rows[x] : 0u, b = w & 0xFFFFu;
        mine[k] = x;
        have[k] = w >> 16;
        inv[k] = have[k] ? 1.0 / (double)have[k] : 0.0;
        most[k] = 0u;
#pragma unroll
        for (uint32_t j = 0; j < kShort; ++j) {
            const uint32_t id = j < have[k] ? 2u * ids[b + j] : 0u;
            kept[k][j / 2] = j & 1u ? kept[k][j / 2] | id << 16 : id;
            if (__ballot(j < have[k])) most[k] = j + 1u;
        }
    }
    // a 16-lane group's first long row: 1/d (a division each step for further ones; the
    // same product for both, since which rows come first differs from run to run)
    const uint32_t long0 = threadIdx.x / 16u < nl ? order[ns + threadIdx.x / 16u] : n;
    const double linv = long0 < n ? 1.0 / (double)(rows[long0] >> 16) : 0.0;
    auto at = [&](uint32_t byte) { return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(h) + byte); };
    auto seeded = [&](uint32_t x, double v) { return x == pr.s ? v + pr.vs : x == pr.t ? v + pr.vt : v; };
    for (int32_t step = 0; step < L; ++step) {
#pragma unroll
        for (uint32_t k = 0; k < kLaneRows; ++k) {
            if (most[k] == 0u) continue;  // wave-uniform, as below
            double a = 0.0, b = 0.0;
#pragma unroll
            for (uint32_t j = 0; j < kShort; j += 2) {
                if (j >= most[k]) break;
                const double v = at(kept[k][j / 2] & 0xFFFFu), w = at(kept[k][j / 2] >> 16);
                a += j < have[k] ? v : 0.0;
                b += j + 1u < have[k] ? w : 0.0;
            }
            if (mine[k] < n) next[mine[k]] = seeded(mine[k], (a + b) * inv[k]);
        }
        for (uint32_t i = threadIdx.x / 16u; i < nl; i += 64u) {
            const uint32_t x = order[ns + i], w = rows[x], e = (w & 0xFFFFu) + (w >> 16);
            double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
            for (uint32_t j = (w & 0xFFFFu) + (threadIdx.x & 15u); j < e; j += 64u) {
                a0 += at(2u * ids[j]);
                if (j + 16u < e) a1 += at(2u * ids[j + 16u]);
                if (j + 32u < e) a2 += at(2u * ids[j + 32u]);
                if (j + 48u < e) a3 += at(2u * ids[j + 48u]);
            }
            const double s = row_sum16((a0 + a1) + (a2 + a3));
            if ((threadIdx.x & 15u) == 0u) next[x] = seeded(x, s * (x == long0 ? linv : 1.0 / (double)(w >> 16)));
        }
        __syncthreads();
        double* t = h;
        h = next;
        next = t;
    }
    double sq = 0.0, lin = 0.0;
    for (uint32_t x = threadIdx.x; x < n; x += 1024u) {
        sq += h[x] * h[x];
        lin += h[x];
    }
    __syncthreads();
    double* red = reinterpret_cast<double*>(lds);  // the tables are done with: 1,024 pairs of sums
    red[threadIdx.x] = sq;
    red[1024u + threadIdx.x] = lin;
    __syncthreads();
    for (uint32_t w = 512; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            red[threadIdx.x] += red[threadIdx.x + w];
            red[1024u + threadIdx.x] += red[1024u + threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) beta[blockIdx.x] = red[0] - red[1024] * red[1024] / (double)n;
}

size_t series_small_bytes(uint32_t nrow, uint32_t idw, uint32_t n)
{
    return std::max<size_t>(4ull * (nrow + idw) + 18ull * n + 16, 16384);
}

hipError_t launch_series_small(const uint4* tab, uint32_t nrow, uint32_t idw, uint32_t n, uint32_t Q, int32_t L,
                               const SeriesPair* pairs, double* beta, hipStream_t st)
{
    const size_t bytes = series_small_bytes(nrow, idw, n);
    const hipError_t e = hipFuncSetAttribute((const void*)series_small_kernel,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSignLdsMost);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(series_small_kernel, dim3(Q), dim3(1024), bytes, st, tab, nrow, idw, n, L, pairs, beta);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Spectral radius of P off the stationary direction: power iteration on the
// symmetric N = D^{-1/2} A D^{-1/2} (same spectrum as P), whose top eigenvector
// is phi = sqrt(d / nnz). With y = N x the next x is (y - (phi.y) phi) / |.|,
// whose norm sqrt(y.y - (phi.y)^2) is the estimate. Kept is w = y / sqrt(d),
// which needs no root: with c = (phi.y) / sqrt(nnz),
//   w'_x = (sum_{u ~ x} w_u - d_x c) / (norm d_x),
//   phi.y' = sum_x d_x w'_x / sqrt(nnz),   y'.y' = sum_x d_x w'_x^2.
// So an iteration is one launch: every work group first adds up the sums that
// the work groups of the launch before left (in their fixed order; the end of
// a launch is the only wait needed), gathers its rows and leaves its own. (One work group reducing for
// all behind a counter cost 60 us an iteration: each work group's fence writes
// its XCD's L2 back.) Rows take four lanes, those above kHubDegree a wave.
// n = 1e5, 1e6 entries: 33.6 us an iteration in five launches (24.3 us of them
// one wave a row, held by the longest rows), 14.0 us so.
// ---------------------------------------------------------------------------

// {c, norm} from the sums that `count` work groups left in part.
__device__ __forceinline__ void lambda_scalars(const double* part, uint32_t count, double nnz, double* lds, double* c,
                                               double* norm)
{
    double a = 0.0, b = 0.0;
    for (uint32_t i = threadIdx.x; i < count; i += 1024u) {
        a += part[2 * i];
        b += part[2 * i + 1];
    }
    a = wave_sum(a);
    b = wave_sum(b);
    const uint32_t wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63u) == 0u) {
        lds[2 * wave] = a;
        lds[2 * wave + 1] = b;
    }
    __syncthreads();
    a = b = 0.0;
    for (uint32_t w = 0; w < 16u; ++w) {
        a += lds[2 * w];
        b += lds[2 * w + 1];
    }
    __syncthreads();
    const double dot = a / sqrt(nnz);
    *c = dot / sqrt(nnz);
    *norm = sqrt(fmax(b - dot * dot, 0.0));
}

// a work group's sums into part[blockIdx.x]
__device__ __forceinline__ void lambda_leave(double dw, double dw2, double* part, double* lds)
{
    dw = wave_sum(dw);
    dw2 = wave_sum(dw2);
    const uint32_t wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63u) == 0u) {
        lds[2 * wave] = dw;
        lds[2 * wave + 1] = dw2;
    }
    __syncthreads();
    if (threadIdx.x < 2u) {
        double s = 0.0;
        for (uint32_t w = 0; w < 16u; ++w) s += lds[2 * w + threadIdx.x];
        part[2 * blockIdx.x + threadIdx.x] = s;
    }
}

// the start: y a counter-based vector (the SplitMix64 output function of seed +
// i times the golden-ratio increment, mapped to [-1/2, 1/2))
__global__ __launch_bounds__(1024) void lambda_start_kernel(RowTables g, uint32_t n, uint64_t seed, double* W,
                                                            double* part)
{
    __shared__ double lds[32];
    double dw = 0.0, dw2 = 0.0;
    for (uint32_t i = blockIdx.x * 1024u + threadIdx.x; i < n; i += gridDim.x * 1024u) {
        uint64_t z = seed + (uint64_t)(i + 1) * 0x9E3779B97F4A7C15ull;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        z ^= z >> 31;
        const double y = (double)(z >> 11) * 0x1p-53 - 0.5, d = (double)(g.rp[i + 1] - g.rp[i]);
        W[i] = y / sqrt(d);
        dw += sqrt(d) * y;
        dw2 += y * y;
    }
    lambda_leave(dw, dw2, part, lds);
}

__global__ __launch_bounds__(1024) void lambda_step_kernel(RowTables g, uint32_t n, double nnz, const uint32_t* hubs,
                                                           uint32_t nhub, const double* W, double* Y,
                                                           const double* part_in, uint32_t count, double* part)
{
    __shared__ double lds[32];
    constexpr uint32_t kLanes = 4;
    const uint32_t lane = threadIdx.x & 63u;
    double c, norm, dw = 0.0, dw2 = 0.0;
    lambda_scalars(part_in, count, nnz, lds, &c, &norm);
    auto finish = [&](uint32_t row, double sum, uint32_t deg) {
        const double d = (double)deg;
        const double w = norm > 0.0 ? (sum - d * c) / (norm * d) : 0.0;
        Y[row] = w;
        dw += d * w;
        dw2 += d * w * w;
    };
    // each wave takes hub rows, then 16 rows at a time
    const uint32_t items = nhub + (n + 15u) / 16u;
    for (uint32_t item = blockIdx.x + gridDim.x * (threadIdx.x >> 6); item < items; item += gridDim.x * 16u) {
        if (item < nhub) {
            const uint32_t row = hubs[item], b = g.rp[row], e = g.rp[row + 1];
            const double s = wave_sum(row_part<1, 1>(g, W, b, e, lane, 64u, 0u).v[0]);
            if (lane == 0u) finish(row, s, e - b);
        } else {
            const uint32_t row = (item - nhub) * 16u + lane / kLanes;
            const uint32_t b = row < n ? g.rp[row] : 0u, e = row < n ? g.rp[row + 1] : 0u;
            if (row < n && e - b <= kHubDegree) {
                const double s = quad_sum(row_part<1, 1>(g, W, b, e, lane & (kLanes - 1u), kLanes, 0u).v[0]);
                if ((lane & (kLanes - 1u)) == 0u) finish(row, s, e - b);
            }
        }
    }
    lambda_leave(dw, dw2, part, lds);
}

__global__ __launch_bounds__(1024) void lambda_finish_kernel(const double* part, uint32_t count, double nnz, double* out)
{
    __shared__ double lds[32];
    double c, norm;
    lambda_scalars(part, count, nnz, lds, &c, &norm);
    if (threadIdx.x == 0) *out = norm;
}

hipError_t launch_lambda(const uint32_t* rp, const uint32_t* col, const uint32_t* col24, uint32_t n, uint32_t nnz,
                         const uint32_t* hubs, uint32_t nhub, int32_t iters, uint64_t seed, double* W, double* Y,
                         double* part, double* lambda, hipStream_t st)
{
    const RowTables g{rp, col, col24};
    const dim3 block(1024);
    const uint32_t start = std::min<uint32_t>((n + 1023) / 1024, kLambdaBlocks);
    const uint32_t grid = std::min<uint32_t>((nhub + (n + 15) / 16 + 15) / 16, kLambdaBlocks);
    double* sums[2] = {part, part + 2 * kLambdaBlocks};  // one read while the other is written
    hipLaunchKernelGGL(lambda_start_kernel, dim3(start), block, 0, st, g, n, seed, W, sums[0]);
    for (int32_t it = 0; it < iters; ++it) {
        hipLaunchKernelGGL(lambda_step_kernel, dim3(grid), block, 0, st, g, n, (double)nnz, hubs, nhub, W, Y,
                           sums[it & 1], it ? grid : start, sums[(it + 1) & 1]);
        std::swap(W, Y);
    }
    hipLaunchKernelGGL(lambda_finish_kernel, dim3(1), block, 0, st, sums[iters & 1], grid, (double)nnz, lambda);
    return hipGetLastError();
}

}  // namespace pw
