// Dense k-qubit blocks (k = 4, 5, 6) on the matrix cores (gfx950 MFMA).
//
// A k-qubit gate (Sec. II-A, Eq. 4 generalised) is the product Y = U X of the 2^k x 2^k matrix U with the
// 2^k x G matrix X whose columns are the amplitude groups (members = target-bit patterns). It is run as the
// real product Y' = A' X' with interleaved (re, im) rows:
//   A'[2a+0][2b+0] = Re U[a][b]   A'[2a+0][2b+1] = -Im U[a][b]
//   A'[2a+1][2b+0] = Im U[a][b]   A'[2a+1][2b+1] =  Re U[a][b]
// on 16x16x4 MFMA tiles (FP64 for complex128, FP32 with FP32 accumulation for complex64). Such a tile adds its four
// products one by one, each a fused multiply-add rounded once (compared bit for bit with a chain of FMAs on gfx950), so
// the order of a sum is the order of its contraction indices: k = 5, 6 take the real parts of four members, then their
// imaginary parts, even and odd quads of members in accumulators of their own; k = 4 takes, member by member, the two
// products of an output's component in the order of the register kernels (its own component first for the imaginary
// part), so that its results are theirs bit for bit.
//
// Work split: a persistent workgroup of 4 waves walks column tiles of 16 CT consecutive groups, 16 KiB of amplitudes
// each (8 on small states). Such a tile's amplitudes are the patterns of the targets and of the lowest free qubits, so in address order
// they are whole cache lines whichever the targets are: they are loaded and stored in that order, 16 bytes a lane, and
// find their (member, group) place in LDS by a bit permutation formed once per thread. Each wave keeps its slice of A'
// in registers for the whole launch. While a tile is multiplied the next one's loads are in flight in registers; the
// products go through a second LDS buffer back into address order.
//
// What bounds it (27 qubits): HBM for k = 4 and 5 (k = 5 complex128 0.68 ms = 6.3 TB/s, complex64 0.34 ms = 6.2 TB/s;
// k = 4, which from HBM comes here with targets or controls inside a line, 0.74 to 0.87 and 0.37 to 0.43 ms), the matrix
// cores for k = 6 (complex128 1.14 ms = 60 TFLOP/s, busy 77 % of the cycles at 2.1 GHz; complex64 0.56 ms = 124 TFLOP/s).
// Tiles of 16 groups with each lane storing its own accumulators took 0.92 and 1.21 ms (k = 5, 6 complex128), 0.65 and
// 0.73 ms (complex64); the register kernel on those sets for k = 4 0.84-1.34 and 0.42-1.02 ms.
#include "qs_internal.h"

namespace {

// Lane layouts of the 16x16x4 MFMAs (both types): lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16].
// The accumulator differs: lane l, register r holds D[4 (l / 16) + r][l % 16] for FP32 but
// D[l / 16 + 4 r][l % 16] for FP64 (measured on gfx950). Tile row i of A' is therefore assigned to the
// (member, component) pair that makes registers (0, 1) and (2, 3) of every lane two complete (re, im) pairs:
// members 2 (l / 16) and 2 (l / 16) + 1 of the tile.
template <class R> struct MF;
template <> struct MF<double> {
    using C2 = double2;
    typedef double acc_t __attribute__((ext_vector_type(4)));
    typedef double vec_t __attribute__((ext_vector_type(2)));
    static __device__ __forceinline__ acc_t mma(double a, double b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    // tile row i = l/16 + 4 r  ->  member 2 (i % 4) + (i / 8), component (i / 4) % 2
    static __device__ __forceinline__ int row_member(int i) { return 2 * (i & 3) + (i >> 3); }
    static __device__ __forceinline__ int row_comp(int i) { return (i >> 2) & 1; }
    static __device__ __forceinline__ int acc_row(int kq, int r) { return kq + 4 * r; }  // tile row of register r
};
template <> struct MF<float> {
    using C2 = float2;
    typedef float acc_t __attribute__((ext_vector_type(4)));
    typedef float vec_t __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ acc_t mma(float a, float b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    // tile row i = 4 (l/16) + r  ->  member i / 2, component i % 2
    static __device__ __forceinline__ int row_member(int i) { return i >> 1; }
    static __device__ __forceinline__ int row_comp(int i) { return i & 1; }
    static __device__ __forceinline__ int acc_row(int kq, int r) { return 4 * kq + r; }
};

// A tile's amplitudes in address order: bit b of the running index sits at state bit gpos[b] and moves the LDS place by
// slot[b] (exclusive or): the place of (member m, group c) is 16 m + ((c % 16) ^ (m % 16)) + 16 D (c / 16), so that lanes
// that differ in member bits, in group bits or in both fall on distinct banks.
constexpr int kMaxTileBits = 11;
struct TileMap {
    int bits;
    int gpos[kMaxTileBits];
    uint32_t slot[kMaxTileBits];
};

// PAIR (complex64): two amplitudes next to each other per 16-byte access; else one amplitude per access (complex64: a
// control on qubit 0). NT: non-temporal accesses. WHOLE: every tile has all its groups; else the state has one tile of
// fewer (the loop has no conditions on its accesses then, so that a wave waits for its loads and not for the stores
// behind them).
template <class R, int K, int CT, bool PAIR, bool NT, bool WHOLE>
__global__ __launch_bounds__(256) void k_dense_mfma(typename MF<R>::C2 *__restrict__ psi, uint64_t ntiles,
                                                    uint64_t ngroups, InsBits ins, TileMap tm, const R *__restrict__ U)
{
    using C2 = typename MF<R>::C2;
    using acc_t = typename MF<R>::acc_t;
    constexpr int D = 1 << K;             // members per group
    constexpr int ROWS = D / 8;           // 16-row tiles of A'
    constexpr bool SPLIT = K == 4;        // a row tile holds one component of 16 members (else both of 8)
    constexpr int RW = SPLIT ? 1 : ROWS < 4 ? ROWS : 4;  // waves side by side over them, the others over the columns
    constexpr int CW = 4 / RW;
    constexpr int RT = ROWS / RW;         // row tiles and column tiles of a wave
    constexpr int CTW = CT / CW;
    constexpr int KT = D / 4;             // member quads along the contraction; each quad feeds 2 MFMAs
    constexpr int P = PAIR ? 2 : 1;
    constexpr int E = 16 * CT * D;        // amplitudes of a tile
    constexpr int LPT = E / P / 256;      // accesses per thread
    constexpr int LB = __builtin_ctz(E / P) - 8;
    constexpr int PB = P - 1;             // bit of the running index that the pair takes
    static_assert(CT % CW == 0 && LPT == 1 << LB, "tile shape");
    typedef R pair_t __attribute__((ext_vector_type(2 * P)));
    __shared__ C2 tile[2][E];

    const int tid = threadIdx.x;
    const int lane = tid & 63, w = tid >> 6;
    const int j = lane & 15, kq = lane >> 4;
    const int wr = w % RW, wc = w / RW;

    // this wave's slice of A': lane (i + 16 kk) holds A'[row i of the tile][contraction index kk of the step]
    R afr[RT][KT][2];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            if constexpr (SPLIT) {  // row tile rt: component rt of member row; step c: members 4 t + 2 c, 4 t + 2 c + 1
                const int ao = j;
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const int ai = 4 * t + 2 * c + (kq >> 1);
                    const R ur = U[2 * (ao * D + ai)], ui = U[2 * (ao * D + ai) + 1];
                    afr[rt][t][c] = (kq & 1) == 0 ? ur : rt == 0 ? -ui : ui;
                }
            } else {
                const int ao = (wr * RT + rt) * 8 + MF<R>::row_member(j);  // output member of tile row j
                const int co = MF<R>::row_comp(j);
                const int ai = 4 * t + kq;
                const R ur = U[2 * (ao * D + ai)], ui = U[2 * (ao * D + ai) + 1];
                afr[rt][t][0] = co == 0 ? ur : ui;   // multiplies Re x[ai]
                afr[rt][t][1] = co == 0 ? -ui : ur;  // multiplies Im x[ai]
            }
        }
    }
    // this thread's amplitudes of every tile: running index (tid + 256 it) P
    uint64_t own = 0;
    uint32_t place = 0;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const uint32_t bit = (tid >> b) & 1u;
        own |= (uint64_t)bit << tm.gpos[b + PB];
        place ^= bit ? tm.slot[b + PB] : 0u;
    }
    uint64_t hoff[LB];
    uint32_t hplace[LB];
#pragma unroll
    for (int b = 0; b < LB; ++b) {
        hoff[b] = (uint64_t)1 << tm.gpos[8 + b + PB];
        hplace[b] = tm.slot[8 + b + PB];
    }
    auto off_of = [&](int it) { return blk_hi<LB>(hoff, it); };
    auto place_of = [&](int it) {
        uint32_t p = place;
#pragma unroll
        for (int b = 0; b < LB; ++b)
            p ^= (it >> b) & 1 ? hplace[b] : 0u;
        return p;
    };
    // a state of fewer groups than a tile has columns: places of groups past the last hold nothing
    auto there = [&](uint32_t p) {
        const uint32_t m = (p >> 4) % D, c = ((p & 15u) ^ (m & 15u)) + 16u * (p / (16u * D));
        return c < ngroups;
    };
    auto load = [&](const C2 *at) -> pair_t {
        const pair_t *q = reinterpret_cast<const pair_t *>(at);
        if constexpr (NT)
            return __builtin_nontemporal_load(q);
        else
            return *q;
    };
    auto put = [&](C2 *t, uint32_t p, const pair_t &v) {
        t[p] = C2{v[0], v[1]};
        if constexpr (P == 2)
            t[p ^ tm.slot[0]] = C2{v[2], v[3]};
    };

    const uint64_t G = gridDim.x;
    // k = 6 is bound by the matrix cores and loses by it (28 qubits 2255 us against 2207); k = 4, SU(4) layers on 27 qubits,
    // 861 us a pass, so 820
    auto at = [&](uint64_t t) { return NT && K < 6 ? (uint64_t)xcd_runs((uint32_t)t, ntiles) : t; };
    uint64_t T = blockIdx.x;
    if (T >= ntiles)
        return;
    pair_t pre[LPT];
    uint64_t base = qs_ins0(at(T) * (16 * CT), ins);
#pragma unroll
    for (int it = 0; it < LPT; ++it) {
        pre[it] = pair_t(0);
        if (WHOLE || there(place_of(it)))
            pre[it] = load(psi + (base | own | off_of(it)));
    }
#pragma unroll
    for (int it = 0; it < LPT; ++it)
        put(tile[0], place_of(it), pre[it]);
    lds_barrier();
    for (;;) {
        const uint64_t Tn = T + G;
        const bool more = WHOLE && Tn < ntiles;  // uniform
        const uint64_t nbase = qs_ins0(at(more ? Tn : T) * (16 * CT), ins);
        if (more) {
#pragma unroll
            for (int it = 0; it < LPT; ++it)
                pre[it] = load(psi + (nbase | own | off_of(it)));
        }
        // consecutive MFMAs go to different row and column tiles, so that none waits for the one before it
        constexpr int NA = SPLIT ? 1 : 2;
        acc_t acc[RT][CTW][NA];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int ct = 0; ct < CTW; ++ct)
#pragma unroll
                for (int e = 0; e < NA; ++e)
                    acc[rt][ct][e] = acc_t{0, 0, 0, 0};
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            C2 bv[CTW][NA == 1 ? 2 : 1];
#pragma unroll
            for (int ct = 0; ct < CTW; ++ct) {
                const C2 *col = tile[0] + (wc * CTW + ct) * 16 * D;
                if constexpr (SPLIT) {
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const int m = 4 * t + 2 * c + (kq >> 1);
                        const C2 x = col[16 * m + (j ^ (m & 15))];
                        // row tile 0 takes x then y of a member, row tile 1 y then x
                        bv[ct][c].x = kq & 1 ? x.y : x.x;
                        bv[ct][c].y = kq & 1 ? x.x : x.y;
                    }
                } else {
                    const int m = 4 * t + kq;
                    bv[ct][0] = col[16 * m + (j ^ (m & 15))];
                }
            }
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int ct = 0; ct < CTW; ++ct)
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) {
                        const C2 x = bv[ct][SPLIT ? c : 0];
                        const bool im = SPLIT ? rt == 1 : c == 1;
                        acc_t &a = acc[rt][ct][SPLIT ? 0 : t & 1];
                        a = MF<R>::mma(afr[rt][t][c], im ? x.y : x.x, a);
                    }
        }
#pragma unroll
        for (int ct = 0; ct < CTW; ++ct) {
            C2 *t = tile[1] + (wc * CTW + ct) * 16 * D;
            if constexpr (SPLIT) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {  // the lane's members, both components
                    const int a0 = MF<R>::acc_row(kq, r);
                    t[16 * a0 + (j ^ (a0 & 15))] = C2{acc[0][ct][0][r], acc[1][ct][0][r]};
                }
            } else {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    const int a0 = (wr * RT + rt) * 8 + 2 * kq;  // accumulators: members a0 (re, im), a0 + 1 (re, im)
                    const acc_t s = acc[rt][ct][0] + acc[rt][ct][NA - 1];
                    t[16 * a0 + (j ^ (a0 & 15))] = C2{s[0], s[1]};
                    t[16 * (a0 + 1) + (j ^ ((a0 + 1) & 15))] = C2{s[2], s[3]};
                }
            }
        }
        lds_barrier();  // the products are in place, and nobody reads the tile any more
#pragma unroll
        for (int it = 0; it < LPT; ++it) {
            const uint32_t p = place_of(it);
            pair_t v;
            const C2 a = tile[1][p];
            v[0] = a.x;
            v[1] = a.y;
            if constexpr (P == 2) {
                const C2 b = tile[1][p ^ tm.slot[0]];
                v[2] = b.x;
                v[3] = b.y;
            }
            if (WHOLE || there(p)) {
                pair_t *q = reinterpret_cast<pair_t *>(psi + (base | own | off_of(it)));
                if constexpr (NT)
                    __builtin_nontemporal_store(v, q);
                else
                    *q = v;
            }
        }
        if (!more)
            break;
#pragma unroll
        for (int it = 0; it < LPT; ++it)
            put(tile[0], place_of(it), pre[it]);
        T = Tn;
        base = nbase;
        lds_barrier();
    }
}

template <class R, int K, int CT, bool PAIR>
hipError_t mfma_p(void *psi, uint64_t ngroups, const InsBits &ins, const TileMap &tm, const void *U, bool nt,
                  hipStream_t s)
{
    using C2 = typename MF<R>::C2;
    const uint64_t ntiles = ngroups > 16 * CT ? ngroups / (16 * CT) : 1;
    uint64_t grid = (uint64_t)qs_cu_count() * qs_tunables().mfma_wg_per_cu;
    if (grid > ntiles)
        grid = ntiles;
    const dim3 g((unsigned)grid), b(256);
    if (ngroups < 16 * CT)
        hipLaunchKernelGGL((k_dense_mfma<R, K, CT, PAIR, false, false>), g, b, 0, s, (C2 *)psi, ntiles, ngroups, ins,
                           tm, (const R *)U);
    else if (nt)
        hipLaunchKernelGGL((k_dense_mfma<R, K, CT, PAIR, true, true>), g, b, 0, s, (C2 *)psi, ntiles, ngroups, ins,
                           tm, (const R *)U);
    else
        hipLaunchKernelGGL((k_dense_mfma<R, K, CT, PAIR, false, true>), g, b, 0, s, (C2 *)psi, ntiles, ngroups, ins,
                           tm, (const R *)U);
    return hipGetLastError();
}

template <class R, int K, int CT>
hipError_t mfma_ct(void *psi, uint64_t ngroups, const InsBits &ins, const TPos &tp, const void *U, hipStream_t s)
{
    constexpr int D = 1 << K, CB = 4 + __builtin_ctz(CT);
    TileMap tm{};
    tm.bits = K + CB;
    uint64_t tmask = 0, taken = 0;
    for (int t = 0; t < K; ++t)
        tmask |= (uint64_t)1 << tp.tpos[t];
    for (int i = 0; i < ins.np; ++i)
        taken |= ins.lowmask[i] + 1;
    bool low_control = false;
    for (int p = 0, b = 0, m = 0, c = 0; b < tm.bits; ++p) {  // ascending positions: targets and the lowest free ones
        const bool target = (tmask >> p) & 1;
        if (!target && ((taken >> p) & 1)) {
            low_control = low_control || p < (sizeof(R) == 8 ? 3 : 4);
            continue;
        }
        if (!target && c >= CB)
            continue;
        tm.gpos[b] = p;
        if (target) {
            tm.slot[b] = (16u << m) | (m < 4 ? 1u << m : 0u);
            ++m;
        } else {
            tm.slot[b] = c < 4 ? 1u << c : (uint32_t)(16 * D) << (c - 4);
            ++c;
        }
        ++b;
    }
    // non-temporal where whole lines stream from HBM (27 qubits, k = 5 complex128: 682 us against 700, complex64 344
    // against 359), not on states the caches hold (22 qubits, k = 4 complex128: 28 us against 24)
    const bool nt = !low_control && qs_streams((ngroups << K) * sizeof(typename MF<R>::C2)) && qs_tunables().nontemporal;
    if constexpr (sizeof(R) == 4)
        if (!(taken & ~tmask & 1))
            return mfma_p<R, K, CT, true>(psi, ngroups, ins, tm, U, nt, s);
    return mfma_p<R, K, CT, false>(psi, ngroups, ins, tm, U, nt, s);
}

template <class R, int K>
hipError_t mfma_k(void *psi, uint64_t ngroups, const InsBits &ins, const TPos &tp, const void *U, hipStream_t s)
{
    constexpr int CT = (sizeof(R) == 8 ? 1 : 2) << (6 - K);  // 16 KiB of amplitudes
    // Fewer tiles than compute units: half as large, since one tile is each workgroup's whole work (16 qubits, k = 6
    // complex64 9.2 us, so 7.8; k = 5 complex128 5.6 and 4.8).
    if constexpr (K > 4 && CT > 1)
        if (ngroups < 16 * CT * (uint64_t)qs_cu_count())
            return mfma_ct<R, K, CT / 2>(psi, ngroups, ins, tp, U, s);
    return mfma_ct<R, K, CT>(psi, ngroups, ins, tp, U, s);
}

}  // namespace

hipError_t launch_dense_mfma(int dtype, int k, void *psi, uint64_t ngroups, const InsBits &ins, const TPos &tp,
                             const void *U_dev, hipStream_t s)
{
    if (dtype == QS_C128) {
        switch (k) {
        case 4: return mfma_k<double, 4>(psi, ngroups, ins, tp, U_dev, s);
        case 5: return mfma_k<double, 5>(psi, ngroups, ins, tp, U_dev, s);
        case 6: return mfma_k<double, 6>(psi, ngroups, ins, tp, U_dev, s);
        default: return hipErrorInvalidValue;
        }
    }
    switch (k) {
    case 4: return mfma_k<float, 4>(psi, ngroups, ins, tp, U_dev, s);
    case 5: return mfma_k<float, 5>(psi, ngroups, ins, tp, U_dev, s);
    case 6: return mfma_k<float, 6>(psi, ngroups, ins, tp, U_dev, s);
    default: return hipErrorInvalidValue;
    }
}
