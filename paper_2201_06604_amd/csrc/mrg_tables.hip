// mrg_tables.hip -- the Monte-Carlo Fisher test consumer of the streams
// (Section 4): random contingency tables with fixed margins, one stream per
// table, entries drawn in row-major order by inversion of their conditional
// hypergeometric distributions, one uniform per free entry.
//
// Each entry is sampled by hyper_search (mrg_hyper.h), or by the definition
// itself, hyper_invert, where the search's bounds do not decide.
//
// One lane owns one table.  Trip counts depend on the margins, so lanes of a
// wave diverge; both kernels therefore run one flat loop over a table's
// entries, and what a lane indexes by column lives in LDS.
#include <hip/hip_runtime.h>

#include <cmath>
#include <mutex>
#include <vector>

#include "mrg_engine.h"
#include "mrg_hyper.h"
#include "mrg_internal.h"
#include "mrg_math.h"

namespace mrg355 {

constexpr int kTableBlock = 256;
constexpr float kTableOverhead = 20.0f;  // of an inversion, in units of a total's square root

// log(n!) for n <= kTableMaxTotal: lgamma(n+1) in long double on the host,
// rounded to double, uploaded once per device (ensure_logfact).  Every entry
// of a valid table is at most its grand total, so the index is in range.
__device__ double g_logfact[kTableMaxTotal + 1];

struct LogFactGlobal {
    __device__ __forceinline__ double operator()(int k) const { return g_logfact[k]; }
};

// The first kLdsFact of them in LDS, for tables whose grand total is below it.
// A lane's arguments are its own, so a read of the global table takes the
// address unit a cycle per lane (64 a wave, nine reads an inversion), an LDS
// read about four.
constexpr int kLdsFact = 1024;
struct LogFactLds {
    const double* tab;
    __device__ __forceinline__ double operator()(int k) const { return tab[k]; }
};

// One I x J table of grand total `total` with row totals row(i) and column
// totals col(j), which are used up: take(i, j, x) receives every entry in
// row-major order.  Returns -sum log(n_ij!) summed in that order.  The engine
// advances (I-1)(J-1) steps.
//
// One loop over the entries, the row's end handled inside it: with a loop over
// rows around a loop over columns a wave of mixed shapes ran the product of
// the largest row and column counts among its lanes.
template <typename Engine, typename LogFact, typename Row, typename Col, typename Take>
__device__ __forceinline__ double sample_table(Engine& e, double norm, LogFact lf, int total, int I, int J, Row row,
                                               Col col, Take take) {
    const typename Engine::Regs kr;
    double stat = 0.0;
    int i = 0, j = 0;
    int left = total;  // units left in rows i..I-1
    int n = I > 1 ? row(0) : 0, Np = left;
    double lfN = lf(Np);
    // determined entries: the row's last is what the row has left
    auto row_end = [&]() {
        take(i, J - 1, n);
        stat -= lf(n);
        col(J - 1) -= n;
        left -= row(i);
        ++i;
        j = 0;
        n = row(i);
        Np = left;
    };
    if (J == 1)
        while (i < I - 1) row_end();
    const int entries = (I - 1) * (J - 1);
    for (int k = 0; k < entries; ++k) {
        const double u = to_f64(e.step_rot(kr)) * norm;
        const int K = col(j);
        int x = hyper_search(u, Np, K, n, lfN, lf);
        if (x < 0) x = hyper_invert(u, Np, K, n);
        take(i, j, x);
        stat -= lf(x);
        n -= x;
        Np -= K;
        col(j) = K - x;
        if (++j == J - 1) {
            row_end();
            lfN = lf(Np);
        }
    }
    for (int c = 0; c < J; ++c) {  // the last row is what the columns have left
        const int x = col(c);
        take(I - 1, c, x);
        stat -= lf(x);
    }
    return stat;
}

// The scale 1/(m1+1) of generator G.
template <int G>
__device__ __forceinline__ constexpr double norm_of() {
    return G == kGen32k3a ? kNorm : kNorm31;
}

// Tables of shape I[t] x J[t] (<= 5 x 5) with margins rows[t][5], cols[t][5],
// table t from stream t; outputs tabs[t][5][5] (zero padded) and stats[t]
// (optional).  A table whose shape is out of range or whose margins are
// negative, differ in total or total more than kTableMaxTotal gets zeros and a
// NaN statistic, and its stream is left as it was (the checks also bound every
// loop).
struct TablesArgs {
    uint32_t* streams;
    uint64_t n;
    const int32_t *I, *J, *rows, *cols;
    int32_t* tabs;
    double* stats;
    uint32_t window;  // tables per block: kTableBlock or kTableWindow
};

constexpr int kTabWords = 25;
constexpr uint32_t kTableWindow = 2 * kTableBlock;
constexpr int kBuckets = 64;

// The grand total of a table whose shape and margins are valid, else -1.
template <typename T>
__device__ __forceinline__ int checked_total(int I, int J, const T* row, const T* col) {
    if (!(I >= 1 && I <= 5 && J >= 1 && J <= 5)) return -1;
    int64_t rs = 0, cs = 0;
    bool ok = true;
    for (int i = 0; i < I; ++i) {
        ok = ok && row[i] >= 0;
        rs += row[i];
    }
    for (int j = 0; j < J; ++j) {
        ok = ok && col[j] >= 0;
        cs += col[j];
    }
    return ok && rs == cs && rs <= kTableMaxTotal ? static_cast<int>(rs) : -1;
}

// Table t of valid total `total`: entries through take(i, j, x).
template <int G, typename LogFact, typename Row, typename Col, typename Take>
__device__ __forceinline__ double one_table(const TablesArgs& a, uint64_t t, int total, LogFact lf, Row row, Col col,
                                            Take take) {
    uint32_t* rec = a.streams + t * 18;
    uint32_t x[6];
#pragma unroll
    for (int w = 0; w < 6; ++w) x[w] = rec[w];
    F64EngineOf<G> e;
    e.load(x);
    const double stat = sample_table(e, norm_of<G>(), lf, total, a.I[t], a.J[t], row, col, take);
    e.save(x);
#pragma unroll
    for (int w = 0; w < 6; ++w) rec[w] = x[w];
    return stat;
}

// A block takes a window of consecutive tables.  A table makes (I-1)(J-1)
// inversions, 1 to 16, each over a range that grows like the square root of the
// table's total, and a wave runs as long as its longest lane; so the block first
// orders its tables by the estimate (I-1)(J-1) (kTableOverhead + sqrt(total))
// in 64 buckets (a counting sort in LDS: the order within a bucket does not
// matter, every table has its own stream and output), and its waves then take
// groups of 64 neighbours in that order, longest first, until none is left: with
// one group a wave, the waves of the short tables left their place empty until
// the block's longest was done.
//
// Where all margins of the window are below kLdsFact and so is every total,
// everything an inversion reads lies in LDS: margins (read from global memory in
// whole lines; a lane's own lie 20 bytes from its neighbour's), logarithms, and
// a group's entries, written out as whole tables.  Any other window reads its
// margins and logarithms and writes its entries where they are.
//
// Bound by VALU issue (68% busy) and by lanes that wait for the longest search
// of their wave (68% of lanes active).  10^6 tables of the 2x2..5x5 mix of
// totals 5..200: 1648 us with two passes over each range and divisions, 363
// with the search, 205 with one loop over the entries, 185 with logarithms in
// LDS, 181 with groups taken longest first.  Four waves a SIMD (128 registers,
// 12 bytes of the general case spilled) against three: 181 against 203 us.
template <int G>
__global__ void __launch_bounds__(kTableBlock) __attribute__((amdgpu_waves_per_eu(4)))
tables_kernel(TablesArgs a) {
    constexpr int kWaves = kTableBlock / 64;
    __shared__ double fact_lds[kLdsFact];
    __shared__ uint16_t row_lds[kTableWindow * 5], col_lds[kTableWindow * 5];
    __shared__ uint32_t tab_lds[kWaves][64 * kTabWords / 2];  // 16-bit entries; 5 column totals a lane in the other case
    __shared__ uint16_t order[kTableWindow];
    __shared__ uint32_t start[kBuckets + 1];
    __shared__ uint32_t next_group;
    const uint64_t base = static_cast<uint64_t>(blockIdx.x) * a.window;
    const uint32_t here = a.n - base < a.window ? static_cast<uint32_t>(a.n - base) : a.window;
    const uint32_t me = threadIdx.x, lane = me & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(me >> 6);
    uint32_t high = 0;  // 16 bits and more of any margin (negative ones too)
    for (uint32_t k = me; k < here * 5; k += kTableBlock) {
        const uint32_t r = static_cast<uint32_t>(a.rows[base * 5 + k]), c = static_cast<uint32_t>(a.cols[base * 5 + k]);
        high |= (r | c) >> 15;
        row_lds[k] = static_cast<uint16_t>(r);
        col_lds[k] = static_cast<uint16_t>(c);
    }
    if (me <= kBuckets) start[me] = 0;
    if (me == 0) next_group = 0;
    bool small = __syncthreads_or(static_cast<int>(high)) == 0;
    uint32_t key[kTableWindow / kTableBlock];  // buckets of this thread's tables (0 for those refused: they stop at once)
    int most = 0;
#pragma unroll
    for (uint32_t q = 0; q < kTableWindow / kTableBlock; ++q) {
        const uint32_t k = me + q * kTableBlock;
        key[q] = 0;
        if (k >= here) continue;
        const uint64_t t = base + k;
        const int It = a.I[t], Jt = a.J[t];
        const int total = small ? checked_total(It, Jt, row_lds + k * 5, col_lds + k * 5)
                                : checked_total(It, Jt, a.rows + t * 5, a.cols + t * 5);
        most = total > most ? total : most;
        if (total >= 0) {
            const float est = static_cast<float>((It - 1) * (Jt - 1)) *
                              (kTableOverhead + __builtin_sqrtf(static_cast<float>(total)));
            key[q] = static_cast<uint32_t>(fminf(est * (1.0f / 16.0f), kBuckets - 1.0f));
        }
        key[q] = kBuckets - 1 - key[q];  // longest first
        atomicAdd(&start[key[q] + 1], 1u);
    }
    small = __syncthreads_or(most >= kLdsFact) == 0 && small;
    if (me == 0)
        for (int c = 1; c <= kBuckets; ++c) start[c] += start[c - 1];  // start[c] = tables in buckets below c
    if (small)
        for (uint32_t k = me; k < kLdsFact; k += kTableBlock) fact_lds[k] = g_logfact[k];
    else
        for (uint32_t k = me; k < here * kTabWords; k += kTableBlock) a.tabs[base * kTabWords + k] = 0;
    __syncthreads();  // orders the zeros before the entries too
#pragma unroll
    for (uint32_t q = 0; q < kTableWindow / kTableBlock; ++q) {
        const uint32_t k = me + q * kTableBlock;
        if (k < here) order[atomicAdd(&start[key[q]], 1u)] = static_cast<uint16_t>(k);
    }
    __syncthreads();
    for (;;) {  // every lane executes the atomic, with 1 on lane 0 only: wave-uniform
        const uint32_t g = __builtin_amdgcn_readfirstlane(atomicAdd(&next_group, lane == 0 ? 1u : 0u));
        if (g * 64 >= here) break;
        const uint32_t in_group = here - g * 64 < 64 ? here - g * 64 : 64;
        const uint32_t k = lane < in_group ? order[g * 64 + lane] : 0;
        const uint64_t t = base + k;
        double stat = __builtin_nan("");
        if (small) {
            uint32_t* words = tab_lds[wave];
            for (uint32_t w = lane; w < 64 * kTabWords / 2; w += 64) words[w] = 0;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            uint16_t* tabs16 = reinterpret_cast<uint16_t*>(words);
            if (lane < in_group) {
                const uint16_t* row = row_lds + k * 5;
                uint16_t* col = col_lds + k * 5;
                uint16_t* out = tabs16 + lane * kTabWords;
                const int total = checked_total(a.I[t], a.J[t], row, col);
                if (total >= 0)
                    stat = one_table<G>(
                        a, t, total, LogFactLds{fact_lds}, [=](int i) { return static_cast<int>(row[i]); },
                        [=](int j) -> uint16_t& { return col[j]; },
                        [=](int i, int j, int x) { out[i * 5 + j] = static_cast<uint16_t>(x); });
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            for (uint32_t w = lane; w < in_group * kTabWords; w += 64) {
                const uint32_t l = w / kTabWords;
                a.tabs[(base + order[g * 64 + l]) * kTabWords + (w - l * kTabWords)] = tabs16[w];
            }
        } else if (lane < in_group) {
            int32_t* col = reinterpret_cast<int32_t*>(tab_lds[wave]) + lane * 5;
            const int32_t *row = a.rows + t * 5, *c = a.cols + t * 5;
            int32_t* out = a.tabs + t * kTabWords;
            const int total = checked_total(a.I[t], a.J[t], row, c);
            if (total >= 0) {
                for (int j = 0; j < a.J[t]; ++j) col[j] = c[j];
                stat = one_table<G>(
                    a, t, total, LogFactGlobal{}, [=](int i) { return row[i]; }, [=](int j) -> int32_t& { return col[j]; },
                    [=](int i, int j, int x) { out[i * 5 + j] = x; });
            }
        }
        if (a.stats && lane < in_group) a.stats[t] = stat;
    }
}

// The count is cleared by a kernel, not a memset, so the launch can be
// captured in a graph.
__global__ void fisher_clear_kernel(unsigned long long* count) { *count = 0; }

struct FisherArgs {
    uint32_t* streams;
    uint64_t B;
    int I, J;
    int32_t r[kFisherMaxDim], c[kFisherMaxDim];
    double threshold;      // observed statistic / (1 + 64 eps)
    unsigned long long* count;
    double* stats;
};

// Replicate b < B of the observed table's margins from stream b; counts the
// replicates whose statistic is <= threshold (one atomic per wave; every
// lane executes it, with the wave's count on lane 0 and 0 elsewhere).  Column
// totals lie in LDS (as registers they cost 32 of them and a wave a SIMD).
// Bound by VALU issue, 92% busy at 666 instructions an entry of a wave, three
// quarters of them the search's loop: 12 x 12 of 12,912 counts, 2^20 replicates,
// 29.9 -> 2.35 ms.
template <int G>
__global__ void __launch_bounds__(kTableBlock) fisher_kernel(FisherArgs a) {
    extern __shared__ int32_t fisher_cols[];  // a.J * kTableBlock
    const uint64_t b = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const uint32_t lane = threadIdx.x & 63;
    bool hit = false;
    if (b < a.B) {
        int32_t* col = fisher_cols + threadIdx.x;  // column j's remaining total at col[j * kTableBlock]
        int total = 0;
        for (int j = 0; j < a.J; ++j) {
            col[j * kTableBlock] = a.c[j];
            total += a.c[j];
        }
        uint32_t* rec = a.streams + b * 18;
        uint32_t x[6];
#pragma unroll
        for (int w = 0; w < 6; ++w) x[w] = rec[w];
        F64EngineOf<G> e;
        e.load(x);
        const double stat = sample_table(e, norm_of<G>(), LogFactGlobal{}, total, a.I, a.J, [&](int i) { return a.r[i]; },
                                         [=](int j) -> int32_t& { return col[j * kTableBlock]; },
                                         [](int, int, int) {});
        hit = stat <= a.threshold;
        if (a.stats) a.stats[b] = stat;
        e.save(x);
#pragma unroll
        for (int w = 0; w < 6; ++w) rec[w] = x[w];
    }
    const unsigned long long wave_hits = __popcll(__ballot(hit));
    atomicAdd(a.count, lane == 0 ? wave_hits : 0ull);
}

double host_log_factorial(int64_t k) {
    int sign = 0;
    return static_cast<double>(lgammal_r(static_cast<long double>(k) + 1.0L, &sign));
}

// One upload of the log-factorial table per device, before the first table
// launch there (synchronous; a launch captured in a graph needs one call
// made beforehand on the device).
hipError_t ensure_logfact() {
    static std::mutex mu;
    static std::vector<char> ready;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lk(mu);
    if (static_cast<size_t>(dev) < ready.size() && ready[dev]) return hipSuccess;
    static std::vector<double> host;
    if (host.empty()) {
        host.resize(kTableMaxTotal + 1);
        for (int64_t k = 0; k <= kTableMaxTotal; ++k)
            host[k] = host_log_factorial(k);
    }
    e = hipMemcpyToSymbol(HIP_SYMBOL(g_logfact), host.data(), host.size() * sizeof(double));
    if (e != hipSuccess) return e;
    if (ready.size() <= static_cast<size_t>(dev)) ready.resize(dev + 1, 0);
    ready[dev] = 1;
    return hipSuccess;
}

hipError_t launch_tables(int gen, uint32_t* streams, uint64_t n, const int32_t* I, const int32_t* J,
                         const int32_t* rows, const int32_t* cols, int32_t* tabs, double* stats, hipStream_t s) {
    if (hipError_t e = ensure_logfact()) return e;
    // windows of two groups a wave once they fill the chip (about four blocks a
    // CU), of one below that
    TablesArgs a{streams, n, I, J, rows, cols, tabs, stats, kTableBlock};
    if (n >= kTableWindow * 1024ull) a.window = kTableWindow;
    const dim3 grid(static_cast<unsigned>((n + a.window - 1) / a.window));
    if (gen == kGen32k3a) hipLaunchKernelGGL(tables_kernel<kGen32k3a>, grid, dim3(kTableBlock), 0, s, a);
    else hipLaunchKernelGGL(tables_kernel<kGen31k3p>, grid, dim3(kTableBlock), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_fisher(int gen, uint32_t* streams, uint64_t B, int I, int J, const int32_t* r, const int32_t* c,
                         double threshold, unsigned long long* count, double* stats, hipStream_t s) {
    FisherArgs a{};
    a.streams = streams;
    a.B = B;
    a.I = I;
    a.J = J;
    for (int k = 0; k < kFisherMaxDim; ++k) {
        a.r[k] = k < I ? r[k] : 0;
        a.c[k] = k < J ? c[k] : 0;
    }
    a.threshold = threshold;
    a.count = count;
    a.stats = stats;
    if (B) {
        if (hipError_t e = ensure_logfact()) return e;
    }
    hipLaunchKernelGGL(fisher_clear_kernel, dim3(1), dim3(1), 0, s, count);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || B == 0) return e;
    const dim3 grid(static_cast<unsigned>((B + kTableBlock - 1) / kTableBlock));
    const size_t lds = static_cast<size_t>(J) * kTableBlock * sizeof(int32_t);  // J <= 32: 32 KB at most
    if (gen == kGen32k3a) hipLaunchKernelGGL(fisher_kernel<kGen32k3a>, grid, dim3(kTableBlock), lds, s, a);
    else hipLaunchKernelGGL(fisher_kernel<kGen31k3p>, grid, dim3(kTableBlock), lds, s, a);
    return hipGetLastError();
}

}  // namespace mrg355
