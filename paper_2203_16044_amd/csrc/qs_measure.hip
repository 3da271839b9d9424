// Measurement, sampling and reset (the simulator's intermediate measurement, Sec. II-A and Sec. I: the state
// vector gives the outcome probabilities directly, and a measured state collapses onto the observed outcome).
//
//  * qs_measure: one FP64 pass yields P0 and P1 (the probability mass with the qubit's bit 0 / 1), the outcome is
//    decided in FP64 from a caller-supplied uniform u, and one more pass keeps the amplitudes of the observed outcome,
//    scaled by 1/sqrt(P_outcome), and zeroes the others.
//  * qs_sample: the state is cut into chunks of 2048 amplitudes (one wave each); each chunk's FP64 mass is reduced
//    from coalesced loads, a deterministic two-level scan turns the chunk masses into an inclusive prefix, and each
//    shot (one wave) finds its chunk by a 64-ary search and its index by two wave scans over the chunk's probabilities
//    held in LDS. Shot k returns the smallest index i whose cumulative mass exceeds u_k x total mass, up to the
//    rounding of the sums; where there is mass, an index without it is never returned.
#include <cmath>
#include <cstring>

#include "qs_internal.h"

namespace {

constexpr int kMeasBlocks = 2048;  // partial pairs fit the state's reduction scratch (2 x 2048 <= 4096)
constexpr int kChunkLog = 11;      // 2048 amplitudes per sampling chunk
constexpr int kTile = 2048;        // chunk masses scanned per workgroup (256 threads x 8)
constexpr size_t kSampleKeep = (size_t)64 << 20;  // sampling scratch a state keeps between calls
constexpr int64_t kDirectShots = 1 << 15;  // shots whose uniforms and indices cross the bus inside the kernel

// 16-byte vector v of a state holds P amplitudes from index P v on (P = 1 complex128, 2 complex64). Whether an
// amplitude's bit q is set depends on the vector alone, except for complex64, q = 0: there the vector's two halves are
// the two outcomes.
template <class R> struct MVec;
template <> struct MVec<double> { typedef double T __attribute__((ext_vector_type(2))); };
template <> struct MVec<float> { typedef float T __attribute__((ext_vector_type(4))); };

// Per-block FP64 masses of the amplitudes whose bit q is 0 and 1 (grid-stride over 16-byte vectors, four loads in
// flight per thread, then an LDS tree in fixed order).
template <class R>
__global__ __launch_bounds__(256) void k_measure_partials(const typename MVec<R>::T *__restrict__ psi, uint64_t nvec,
                                                          int q, double *__restrict__ partials)
{
    using V = typename MVec<R>::T;
    constexpr int U = 4;
    __shared__ double r0[256], r1[256];
    double a0 = 0.0, a1 = 0.0;
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    auto add = [&](const V &x, uint64_t v) {
        if constexpr (sizeof(R) == 8) {
            const double p = x.x * x.x + x.y * x.y;
            const bool one = (v >> q) & 1;
            a0 += one ? 0.0 : p;
            a1 += one ? p : 0.0;
        } else {
            const double p = (double)x.x * (double)x.x + (double)x.y * (double)x.y;
            const double r = (double)x.z * (double)x.z + (double)x.w * (double)x.w;
            if (q == 0) {
                a0 += p;
                a1 += r;
            } else {
                const bool one = (v >> (q - 1)) & 1;
                a0 += one ? 0.0 : p + r;
                a1 += one ? p + r : 0.0;
            }
        }
    };
    uint64_t v = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    for (; v + (U - 1) * stride < nvec; v += U * stride) {
        V x[U];
#pragma unroll
        for (int j = 0; j < U; ++j)
            x[j] = psi[v + j * stride];
#pragma unroll
        for (int j = 0; j < U; ++j)
            add(x[j], v + j * stride);
    }
    for (; v < nvec; v += stride)
        add(psi[v], v);
    r0[threadIdx.x] = a0;
    r1[threadIdx.x] = a1;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            r0[threadIdx.x] += r0[threadIdx.x + w];
            r1[threadIdx.x] += r1[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        partials[2 * blockIdx.x] = r0[0];
        partials[2 * blockIdx.x + 1] = r1[0];
    }
}

// s + c <- (s + c) + v, the rounding error of s + v kept in c (Knuth's two-sum).
__device__ __forceinline__ void two_sum(double &s, double &c, double v)
{
    const double t = s + v;
    const double z = t - s;
    c += (s - (t - z)) + (v - z);
    s = t;
}

// What a measurement decided (device memory; P0 and P1 also go to the host).
struct MeasResult {
    double P0, P1;
    double scale;  // 1 / sqrt(mass of the outcome)
    int outcome;   // 0 or 1; -1: the state has no finite nonzero mass (it is then left as it is)
};

// Sum the partial pairs in a fixed order (compensated: each of 128 threads per outcome its share, then a tree) and
// decide the outcome: 1 iff u (P0 + P1) < P1. One workgroup; what bounds it is the latency of one round of loads and
// of seven tree steps, then the write to the host (2,048 pairs: 6 us; one thread per outcome walking all of them in
// sequence took 209 us).
__global__ __launch_bounds__(256) void k_measure_decide(const double *__restrict__ partials, int nb, double u,
                                                        MeasResult *__restrict__ result, double *__restrict__ host)
{
    __shared__ double ss[256], sc[256];
    const int t = threadIdx.x, o = t & 1;
    double s = 0.0, c = 0.0;
    for (int b = t >> 1; b < nb; b += 128)
        two_sum(s, c, partials[2 * b + o]);
    ss[t] = s;
    sc[t] = c;
    __syncthreads();
    for (int w = 128; w > 1; w >>= 1) {  // t and t + w hold the same outcome
        if (t < w) {
            two_sum(s, c, ss[t + w]);
            c += sc[t + w];
            ss[t] = s;
            sc[t] = c;
        }
        __syncthreads();
    }
    if (t == 0) {
        const double P0 = ss[0] + sc[0], P1 = ss[1] + sc[1], tot = P0 + P1;
        const bool ok = tot > 0.0 && tot <= 1.7976931348623157e308;
        const int out = u * tot < P1 ? 1 : 0;
        result->P0 = P0;
        result->P1 = P1;
        result->scale = 1.0 / sqrt(out ? P1 : P0);
        result->outcome = ok ? out : -1;
        host[0] = P0;
        host[1] = P1;
    }
}

// Keep the amplitudes of the observed outcome, scaled in FP64; zero the others (not read, but for complex64, q = 0,
// where both outcomes share each vector).
template <class R>
__global__ __launch_bounds__(256) void k_collapse(typename MVec<R>::T *__restrict__ psi, uint64_t nvec, int q,
                                                  const MeasResult *__restrict__ result)
{
    using V = typename MVec<R>::T;
    const int outcome = result->outcome;
    if (outcome < 0)
        return;
    const double scale = result->scale;
    for (uint64_t v = (uint64_t)blockIdx.x * 256 + threadIdx.x; v < nvec; v += (uint64_t)gridDim.x * 256) {
        V x;
        if constexpr (sizeof(R) == 8) {
            x = V{0, 0};
            if ((int)((v >> q) & 1) == outcome) {
                x = psi[v];
                x.x *= scale;
                x.y *= scale;
            }
        } else {
            x = V{0, 0, 0, 0};
            if (q == 0 || (int)((v >> (q - 1)) & 1) == outcome) {
                x = psi[v];
                x.x = (R)((double)x.x * scale);
                x.y = (R)((double)x.y * scale);
                x.z = (R)((double)x.z * scale);
                x.w = (R)((double)x.w * scale);
                if (q == 0) {
                    if (outcome)
                        x.x = x.y = 0;
                    else
                        x.z = x.w = 0;
                }
            }
        }
        psi[v] = x;
    }
}

// Wave-inclusive scan of one FP64 value per lane (Hillis-Steele, 6 steps, the same order on every call).
__device__ __forceinline__ double wave_incl_scan(double x)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const double y = __shfl_up(x, d, 64);
        if (lane >= d)
            x += y;
    }
    return x;
}

// The 16-byte vectors of a chunk are read in lane order (whole lines per load), eight in flight per lane. fn(j, x) takes
// vector j of the chunk (amplitudes P j .. P j + P - 1 of it).
template <class R, class F>
__device__ __forceinline__ void chunk_vectors(const typename MVec<R>::T *__restrict__ pv, int nv, F fn)
{
    using V = typename MVec<R>::T;
    constexpr int U = 8;
    int j = threadIdx.x & 63;
    for (; j + (U - 1) * 64 < nv; j += U * 64) {
        V x[U];
#pragma unroll
        for (int t = 0; t < U; ++t)
            x[t] = pv[j + 64 * t];
#pragma unroll
        for (int t = 0; t < U; ++t)
            fn(j + 64 * t, x[t]);
    }
    for (; j < nv; j += 64)
        fn(j, pv[j]);
}

// One wave per chunk: its mass, each lane's share summed in order, then a butterfly over the lanes. Bound by the read
// of the state: 27 qubits complex128 (2 GiB) 0.366 ms = 5.9 TB/s, against 2.24 ms with 64 consecutive amplitudes per
// lane (every load instruction of a wave touched 64 lines).
template <class R>
__global__ __launch_bounds__(256) void k_chunk_mass(const typename MVec<R>::T *__restrict__ psi, int nv,
                                                    uint64_t nchunks, double *__restrict__ mass)
{
    using V = typename MVec<R>::T;
    const uint64_t c = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (c >= nchunks)
        return;  // whole waves leave together
    double s = 0.0;
    chunk_vectors<R>(psi + c * (uint64_t)nv, nv, [&](int, const V &x) {
        s += (double)x.x * (double)x.x + (double)x.y * (double)x.y;
        if constexpr (sizeof(R) == 4)
            s += (double)x.z * (double)x.z + (double)x.w * (double)x.w;
    });
#pragma unroll
    for (int d = 32; d > 0; d >>= 1)
        s += __shfl_xor(s, d, 64);
    if ((threadIdx.x & 63) == 0)
        mass[c] = s;
}

// Level 1 of the prefix scan: each workgroup scans a tile of kTile masses (8 sequential per thread, then the threads' runs
// joined two by two) into tile-local inclusive prefixes, in place, and writes the tile total, its last prefix. Where two
// runs join, the left one's last prefix is added to every prefix of the right one, so that the prefix never falls and
// stays exactly where a chunk has no mass: a target cannot meet an empty chunk. (Prefixes and thread sums added up in
// different orders rise and fall by a rounding at such chunks.)
__global__ __launch_bounds__(256) void k_scan_tile(double *__restrict__ io, uint64_t len,
                                                   double *__restrict__ totals)
{
    __shared__ double last[256];  // each thread's last prefix
    const int t = threadIdx.x;
    const uint64_t base = (uint64_t)blockIdx.x * kTile + (uint64_t)t * 8;
    double v[8];
    double run = 0.0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        v[j] = base + j < len ? io[base + j] : 0.0;
        run += v[j];
        v[j] = run;
    }
    last[t] = run;
    __syncthreads();
    for (int d = 1; d < 256; d <<= 1) {  // read: threads with bit d clear; written: threads with it set
        if (t & d) {
            const double left = last[(t & ~(2 * d - 1)) + d - 1];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                v[j] += left;
            last[t] = v[7];
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (base + j < len)
            io[base + j] = v[j];
    if (t == 255)
        totals[blockIdx.x] = v[7];
}

// Level 2: the tile totals become exclusive tile offsets, totals[ntiles] their sum. The additions run in sequence (so
// that a tile's offset is bit for bit the last prefix of the tile before it and the prefix never falls); what is
// parallel is the traffic: 2048 totals at a time pass through LDS.
__global__ __launch_bounds__(256) void k_scan_totals(double *__restrict__ totals, uint64_t ntiles)
{
    __shared__ double sh[2048];
    __shared__ double carry;
    if (threadIdx.x == 0)
        carry = 0.0;
    for (uint64_t t0 = 0; t0 < ntiles; t0 += 2048) {
        const int cnt = (int)(ntiles - t0 < 2048 ? ntiles - t0 : 2048);
        for (int i = threadIdx.x; i < cnt; i += 256)
            sh[i] = totals[t0 + i];
        __syncthreads();
        if (threadIdx.x == 0) {
            double run = carry;
            for (int i = 0; i < cnt; ++i) {
                const double x = sh[i];
                sh[i] = run;
                run += x;
            }
            carry = run;
        }
        __syncthreads();
        for (int i = threadIdx.x; i < cnt; i += 256)
            totals[t0 + i] = sh[i];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        totals[ntiles] = carry;
}

// Level 3: add each tile's offset.
__global__ __launch_bounds__(256) void k_scan_add(double *__restrict__ out, uint64_t len,
                                                  const double *__restrict__ offs)
{
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < len && i >= (uint64_t)kTile)
        out[i] += offs[i / kTile];
}

// One wave per shot, one wave per workgroup (16.5 KB of LDS). total = incl[last]; target = u x total; the chunk is the
// smallest c with incl[c] > target (or, when rounding puts the target at the total, the smallest c with
// incl[c] >= total), found by a 64-ary search: three rounds of loads for 2^18 chunks where a binary search waits for
// eighteen. The chunk's probabilities go to LDS (kept when the wave's next shot falls into the same chunk); lane l sums
// the chunk/64 consecutive ones of sub-block l, a wave scan of the sums finds the sub-block, a wave scan of its
// elements the index. If rounding leaves no index above the residual, the last index with nonzero mass is taken. Every
// returned index lies in [0, dim) and, where the state has any mass, has mass. Bound by the search's and the chunk's
// load latency: 4,096 shots at 27 qubits 33 us (153 us with a binary search and strided loads).
template <class R>
__global__ __launch_bounds__(64) void k_sample(const typename MVec<R>::T *__restrict__ psi, int chunk, int nv, int per,
                                               uint64_t nchunks, const double *__restrict__ incl,
                                               const double *__restrict__ u, int64_t nshots, int64_t *__restrict__ out,
                                               double *__restrict__ total_out)
{
    using V = typename MVec<R>::T;
    constexpr int P = sizeof(R) == 8 ? 1 : 2;
    __shared__ double p[(1 << kChunkLog) + (1 << kChunkLog) / 32];  // element i at i + i / 32: lanes on distinct banks
    auto at = [](int i) { return i + (i >> 5); };
    const int lane = threadIdx.x;
    const double total = incl[nchunks - 1];
    if (blockIdx.x == 0 && lane == 0)
        *total_out = total;
    uint64_t held = nchunks;  // the chunk in LDS
    for (int64_t shot = blockIdx.x; shot < nshots; shot += gridDim.x) {
        const double target = u[shot] * total;
        const bool clamp = !(target < total);
        uint64_t lo = 0, len = nchunks;  // the chunk is in [lo, lo + len)
        while (len > 1) {
            const uint64_t step = (len + 63) / 64, last = lo + len - 1;
            const uint64_t pos = lo + (lane + 1) * step - 1;
            const double x = incl[pos < last ? pos : last];
            const bool right = pos < last && (clamp ? x < total : x <= target);
            const int k = __ffsll(~__ballot(right)) - 1;  // lane 63 is never right
            lo += k * step;
            len = last - lo + 1 < step ? last - lo + 1 : step;
        }
        const uint64_t c = lo;
        const double r = target - (c > 0 ? incl[c - 1] : 0.0);
        if (c != held) {
            lds_barrier();
            chunk_vectors<R>(psi + c * (uint64_t)nv, nv, [&](int j, const V &x) {
                p[at(P * j)] = (double)x.x * (double)x.x + (double)x.y * (double)x.y;
                if constexpr (P == 2)
                    p[at(P * j + 1)] = (double)x.z * (double)x.z + (double)x.w * (double)x.w;
            });
            lds_barrier();
            held = c;
        }
        double mine = 0.0;
        for (int j = 0; j < per; ++j)
            if (lane * per + j < chunk)
                mine += p[at(lane * per + j)];
        const double sc = wave_incl_scan(mine);
        const unsigned long long above = __ballot(!clamp && sc > r && mine > 0.0);
        const unsigned long long nonzero = __ballot(mine > 0.0);
        const int pick = above ? __ffsll(above) - 1 : nonzero ? 63 - __clzll(nonzero) : 0;
        // every lane takes part in both shuffles (a lane inactive in a shuffle gives undefined values to its readers)
        const double prev = __shfl_up(sc, 1, 64);
        const double before = __shfl(lane > 0 ? prev : 0.0, pick, 64);
        const double rr = r - before;
        const int e = pick * per + lane;
        const double x = lane < per && e < chunk ? p[at(e)] : 0.0;
        const double acc = wave_incl_scan(x);
        const unsigned long long hit = __ballot(above != 0 && acc > rr && x > 0.0);
        const unsigned long long some = __ballot(x > 0.0);
        const int sel = hit ? __ffsll(hit) - 1 : some ? 63 - __clzll(some) : 0;
        if (lane == 0)
            out[shot] = (int64_t)(c * (uint64_t)chunk) + pick * per + sel;
    }
}

template <class R>
hipError_t measure_r(void *psi, uint64_t dim, int q, double u, double *partials, MeasResult *result, double *host,
                     hipEvent_t decided, hipStream_t s)
{
    using V = typename MVec<R>::T;
    const uint64_t nvec = sizeof(R) == 8 ? dim : dim / 2;
    uint64_t nb = (dim + 256 * 16 - 1) / (256 * 16);
    if (nb > (uint64_t)kMeasBlocks)
        nb = kMeasBlocks;
    hipLaunchKernelGGL((k_measure_partials<R>), dim3((unsigned)nb), dim3(256), 0, s, (const V *)psi, nvec, q,
                       partials);
    hipLaunchKernelGGL(k_measure_decide, dim3(1), dim3(256), 0, s, (const double *)partials, (int)nb, u, result, host);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess)
        e = hipEventRecord(decided, s);
    if (e != hipSuccess)
        return e;
    uint64_t grid = (nvec + 255) / 256;
    if (grid > ((uint64_t)1 << 20))
        grid = (uint64_t)1 << 20;
    hipLaunchKernelGGL((k_collapse<R>), dim3((unsigned)grid), dim3(256), 0, s, (V *)psi, nvec, q,
                       (const MeasResult *)result);
    return hipGetLastError();
}

struct SampleGeom {
    uint64_t chunk, nchunks, ntiles;
    int per;
};

SampleGeom sample_geom(uint64_t dim)
{
    SampleGeom g;
    g.chunk = dim < ((uint64_t)1 << kChunkLog) ? dim : ((uint64_t)1 << kChunkLog);
    g.per = (int)(g.chunk >= 64 ? g.chunk / 64 : 1);
    g.nchunks = dim / g.chunk;
    g.ntiles = (g.nchunks + kTile - 1) / kTile;
    return g;
}

template <class R>
hipError_t sample_r(const void *psi, const SampleGeom &g, double *incl, double *tiles, const double *u, int64_t nshots,
                    int64_t *out, double *total, hipStream_t s)
{
    using V = typename MVec<R>::T;
    const int nv = (int)(g.chunk * sizeof(R) * 2 / 16);
    hipLaunchKernelGGL((k_chunk_mass<R>), dim3((unsigned)((g.nchunks + 3) / 4)), dim3(256), 0, s, (const V *)psi, nv,
                       g.nchunks, incl);
    hipLaunchKernelGGL(k_scan_tile, dim3((unsigned)g.ntiles), dim3(256), 0, s, incl, g.nchunks, tiles);
    if (g.ntiles > 1) {  // one tile's prefixes are the whole prefix
        hipLaunchKernelGGL(k_scan_totals, dim3(1), dim3(256), 0, s, tiles, g.ntiles);
        hipLaunchKernelGGL(k_scan_add, dim3((unsigned)((g.nchunks + 255) / 256)), dim3(256), 0, s, incl, g.nchunks,
                           (const double *)tiles);
    }
    // a wave per shot up to 64 waves per CU's worth of workgroups, then several shots per wave
    uint64_t grid = (uint64_t)qs_cu_count() * 64;
    if (grid > (uint64_t)nshots)
        grid = (uint64_t)nshots;
    hipLaunchKernelGGL((k_sample<R>), dim3((unsigned)grid), dim3(64), 0, s, (const V *)psi, (int)g.chunk, nv, g.per,
                       g.nchunks, (const double *)incl, u, nshots, out, total);
    return hipGetLastError();
}

// The collapse is enqueued behind the decision, which the GPU takes itself; the host waits for the decision alone and
// is free to enqueue what follows while the collapse runs.
int measure_impl(qs_state *st, int qubit, double u, int *outcome, double *prob_one)
{
    const uint64_t dim = (uint64_t)1 << st->n;
    double *partials = st->red;
    MeasResult *result = reinterpret_cast<MeasResult *>(st->red + 2 * kMeasBlocks + 4);
    QS_HIP(st->dtype == QS_C128 ? measure_r<double>(st->psi, dim, qubit, u, partials, result, st->hresult,
                                                    st->hresult_ev, st->stream)
                                : measure_r<float>(st->psi, dim, qubit, u, partials, result, st->hresult,
                                                   st->hresult_ev, st->stream));
    QS_HIP(hipEventSynchronize(st->hresult_ev));
    const double P0 = st->hresult[0], P1 = st->hresult[1], tot = P0 + P1;
    if (!(tot > 0.0) || !std::isfinite(tot))
        return qs_fail(QS_EINVAL, "qs_measure: the state has no finite nonzero mass (%g)", tot);
    if (outcome)
        *outcome = (u * tot < P1) ? 1 : 0;
    if (prob_one)
        *prob_one = P1 / tot;
    return QS_OK;
}

}  // namespace

extern "C" {

QS_API int qs_measure(qs_state *st, int qubit, double u, int *outcome, double *prob_one)
{
    qs_clear_error();
    if (!st || !outcome)
        return qs_fail(QS_EINVAL, "qs_measure: NULL argument");
    if (qubit < 0 || qubit >= st->n)
        return qs_fail(QS_EINVAL, "qs_measure: qubit %d outside [0, %d)", qubit, st->n);
    if (!(u >= 0.0 && u < 1.0))
        return qs_fail(QS_EINVAL, "qs_measure: u = %g outside [0, 1)", u);
    if (st->red_cap < 2 * (size_t)kMeasBlocks + 8)
        return qs_fail(QS_EUNSUPPORTED, "qs_measure: reduction scratch too small");
    return measure_impl(st, qubit, u, outcome, prob_one);
}

QS_API int qs_reset(qs_state *st, int qubit, double u, int *outcome)
{
    qs_clear_error();
    int out = 0;
    if (int rc = qs_measure(st, qubit, u, &out, nullptr))
        return rc;
    if (out) {
        static const double X[8] = {0, 0, 1, 0, 1, 0, 0, 0};
        const int t = qubit;
        if (int rc = qs_apply_gate(st, &t, 1, X))
            return rc;
    }
    if (outcome)
        *outcome = out;
    return QS_OK;
}

QS_API int qs_sample(qs_state *st, int64_t nshots, const double *u, int64_t *out)
{
    qs_clear_error();
    if (!st || (nshots > 0 && (!u || !out)))
        return qs_fail(QS_EINVAL, "qs_sample: NULL argument");
    if (nshots < 0 || nshots > ((int64_t)1 << 30))
        return qs_fail(QS_EINVAL, "qs_sample: nshots = %lld outside [0, 2^30]", (long long)nshots);
    for (int64_t k = 0; k < nshots; ++k)
        if (!(u[k] >= 0.0 && u[k] < 1.0))
            return qs_fail(QS_EINVAL, "qs_sample: u[%lld] = %g outside [0, 1)", (long long)k, u[k]);
    if (nshots == 0)
        return QS_OK;
    const uint64_t dim = (uint64_t)1 << st->n;
    const SampleGeom g = sample_geom(dim);
    // scratch: chunk masses turned into their prefix, tile totals (+ total); for many shots also uniforms and outputs
    const bool direct = nshots <= kDirectShots;
    const size_t nd = g.nchunks + g.ntiles + 1;
    const size_t bytes = (nd + 1) * sizeof(double) + (direct ? 0 : (size_t)nshots * (sizeof(double) + sizeof(int64_t)));
    char *buf = qs_scratch(st, bytes);
    if (!buf)
        return QS_ENOMEM;
    double *incl = (double *)buf;
    double *tiles = incl + g.nchunks;
    const double *du = nullptr;
    int64_t *dout = nullptr;
    char *host = nullptr;
    hipError_t e = hipSuccess;
    if (direct) {  // few shots: the kernel reads the uniforms from and writes the indices to pinned host memory
        host = qs_ring_host(st, (size_t)nshots * (sizeof(double) + sizeof(int64_t)));
        if (!host)
            return QS_EDEVICE;
        std::memcpy(host, u, (size_t)nshots * sizeof(double));
        du = (const double *)host;
        dout = (int64_t *)(host + (size_t)nshots * sizeof(double));
    } else {
        double *d = tiles + g.ntiles + 2;
        e = hipMemcpyAsync(d, u, (size_t)nshots * sizeof(double), hipMemcpyHostToDevice, st->stream);
        du = d;
        dout = (int64_t *)(d + nshots);
    }
    if (e == hipSuccess)
        e = st->dtype == QS_C128 ? sample_r<double>(st->psi, g, incl, tiles, du, nshots, dout, st->hresult, st->stream)
                                 : sample_r<float>(st->psi, g, incl, tiles, du, nshots, dout, st->hresult, st->stream);
    if (e == hipSuccess && !direct)
        e = hipMemcpyAsync(out, dout, (size_t)nshots * sizeof(int64_t), hipMemcpyDeviceToHost, st->stream);
    if (e == hipSuccess)
        e = hipStreamSynchronize(st->stream);
    if (bytes > kSampleKeep)
        qs_scratch_drop(st);
    if (e != hipSuccess)
        return qs_hip_fail(e, "qs_sample");
    const double total = st->hresult[0];
    if (direct)
        std::memcpy(out, host + (size_t)nshots * sizeof(double), (size_t)nshots * sizeof(int64_t));
    // a state without finite nonzero mass has no distribution: its indices are meaningless
    if (!(total > 0.0) || !std::isfinite(total))
        return qs_fail(QS_EINVAL, "qs_sample: the state has no finite nonzero mass (%g)", total);
    return QS_OK;
}

}  // extern "C"
