// Plain gate kernels of libqs for gfx950 (CDNA4, wave64).
//
// Every kernel is one in-place pass over the amplitudes it touches (HBM-bound): the gate rule of Sec. II-A,
// Eq. 4 applied to 2^k-member groups, the fused-swap permutation of Sec. III-D, and the FP64 probability /
// norm reduction. Group members are located by inserting zero bits at the (sorted) target and control
// positions of a group counter ("bit insert"); consecutive threads take consecutive counters, so every
// member stream is a coalesced 16-byte-per-lane stream whenever its bit positions are not the lowest ones.
#include "qs_internal.h"

#include <algorithm>
#include <type_traits>

namespace {

template <class R> struct CT;
template <> struct CT<double> { using T = double2; };
template <> struct CT<float> { using T = float2; };

__device__ __forceinline__ uint64_t ins0(uint64_t g, const InsBits &s) { return qs_ins0(g, s); }

template <int K> __device__ __forceinline__ uint64_t member_off(int a, const TPos &tp)
{
    return qs_member_off<K>(a, tp);
}

// Loads/stores with an optional non-temporal hint (the nontemporal builtins need native vector types).
template <class T> struct NativeVec;
template <> struct NativeVec<double2> { typedef double type __attribute__((ext_vector_type(2))); };
template <> struct NativeVec<float2> { typedef float type __attribute__((ext_vector_type(2))); };

template <class T> __device__ __forceinline__ T ld(const T *p, int nt)
{
    if (!nt)
        return *p;
    using N = typename NativeVec<T>::type;
    const N v = __builtin_nontemporal_load(reinterpret_cast<const N *>(p));
    T r;
    r.x = v.x;
    r.y = v.y;
    return r;
}
template <class T> __device__ __forceinline__ void st(T *p, T v, int nt)
{
    if (!nt) {
        *p = v;
        return;
    }
    using N = typename NativeVec<T>::type;
    N w;
    w.x = v.x;
    w.y = v.y;
    __builtin_nontemporal_store(w, reinterpret_cast<N *>(p));
}

// ---------------------------------------------------------------------------------------------------------
// dense k-qubit gate, k <= 3 (and k = 4 where it streams whole lines, dense_k): the group's 2^k members live in
// registers; U comes from kernel arguments, for k = 4 from device memory through uniform (scalar) loads.
// ---------------------------------------------------------------------------------------------------------
template <class R, int K> struct MatByVal {
    R v[2 << (2 * K)];
    __device__ __forceinline__ R re(int i) const { return v[2 * i]; }
    __device__ __forceinline__ R im(int i) const { return v[2 * i + 1]; }
};
template <class R> struct MatByPtr {
    const R *__restrict__ p;
    __device__ __forceinline__ R re(int i) const { return p[2 * i]; }
    __device__ __forceinline__ R im(int i) const { return p[2 * i + 1]; }
};

// ---------------------------------------------------------------------------------------------------------
// 1-qubit gate whose target lies inside a wave's contiguous span (complex128: q < 6; complex64: q < 7). Every lane
// streams one 16-byte vector (one complex128 amplitude, or two adjacent complex64 ones) with full-width coalesced
// non-temporal loads and stores, and takes its pair partner from lane ^ 2^t by a cross-lane shuffle (complex64,
// q = 0: the partner is the other half of the lane's own vector). Each lane computes the outputs of its own
// amplitudes: a member with bit q = 0 gets U00 a + U01 b, with bit q = 1 gets U10 b + U11 a (b: the partner).
// The vector count is a multiple of 64 and so is the grid stride, so whole waves run the loop together.
// ---------------------------------------------------------------------------------------------------------
template <class R> struct LaneVec;
template <> struct LaneVec<double> { typedef double T __attribute__((ext_vector_type(2))); };
template <> struct LaneVec<float> { typedef float T __attribute__((ext_vector_type(4))); };

template <class R>
__device__ __forceinline__ void pair_out(R ar, R ai, R br, R bi, int bit, const MatByVal<R, 1> &m, R &outr, R &outi)
{
    // bit 0: U00 a + U01 b; bit 1: U11 a + U10 b
    const int ia = bit ? 3 : 0, ib = bit ? 2 : 1;
    const R ur = m.re(ia), ui = m.im(ia), vr = m.re(ib), vi = m.im(ib);
    outr = fma(ur, ar, fma(-ui, ai, fma(vr, br, -vi * bi)));
    outi = fma(ur, ai, fma(ui, ar, fma(vr, bi, vi * br)));
}

template <class R, bool NT>
__global__ __launch_bounds__(256) void k_dense1_lane(typename LaneVec<R>::T *__restrict__ psi, uint64_t nvec, int q,
                                                     MatByVal<R, 1> m)
{
    using V = typename LaneVec<R>::T;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < nvec; v += stride) {
        const V x = NT ? __builtin_nontemporal_load(psi + v) : psi[v];
        V y;
        if constexpr (sizeof(R) == 8) {
            const int d = 1 << q;
            const R pr = __shfl_xor(x.x, d, 64), pi = __shfl_xor(x.y, d, 64);
            const int bit = (int)((v >> q) & 1);
            R o0, o1;
            pair_out<R>(x.x, x.y, pr, pi, bit, m, o0, o1);
            y.x = o0;
            y.y = o1;
        } else {
            if (q == 0) {
                R o0, o1, o2, o3;
                pair_out<R>(x.x, x.y, x.z, x.w, 0, m, o0, o1);
                pair_out<R>(x.z, x.w, x.x, x.y, 1, m, o2, o3);
                y.x = o0;
                y.y = o1;
                y.z = o2;
                y.w = o3;
            } else {
                const int d = 1 << (q - 1);
                const R p0 = __shfl_xor(x.x, d, 64), p1 = __shfl_xor(x.y, d, 64);
                const R p2 = __shfl_xor(x.z, d, 64), p3 = __shfl_xor(x.w, d, 64);
                const int bit = (int)((v >> (q - 1)) & 1);
                R o0, o1, o2, o3;
                pair_out<R>(x.x, x.y, p0, p1, bit, m, o0, o1);
                pair_out<R>(x.z, x.w, p2, p3, bit, m, o2, o3);
                y.x = o0;
                y.y = o1;
                y.z = o2;
                y.w = o3;
            }
        }
        if constexpr (NT)
            __builtin_nontemporal_store(y, psi + v);
        else
            psi[v] = y;
    }
}

template <class R, int K, int G, class MS>
__global__ __launch_bounds__(256) void k_dense(typename CT<R>::T *__restrict__ psi, uint64_t ngroups, InsBits ins,
                                               TPos tp, MS ms, int nt)
{
    using C2 = typename CT<R>::T;
    constexpr int D = 1 << K;
    uint64_t off[D];
#pragma unroll
    for (int a = 0; a < D; ++a)
        off[a] = member_off<K>(a, tp);
    const uint64_t bs = blockDim.x;
    const uint64_t stride = (uint64_t)gridDim.x * bs * G;
    for (uint64_t g0 = (uint64_t)blockIdx.x * bs * G + threadIdx.x; g0 < ngroups; g0 += stride) {
        C2 x[G][D];
        uint64_t base[G];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            uint64_t g = g0 + j * bs;
            base[j] = ins0(g < ngroups ? g : 0, ins);
            if (g < ngroups) {
#pragma unroll
                for (int a = 0; a < D; ++a)
                    x[j][a] = ld(psi + base[j] + off[a], nt);
            }
        }
#pragma unroll
        for (int j = 0; j < G; ++j) {
            if (g0 + j * bs < ngroups) {
#pragma unroll
                for (int a = 0; a < D; ++a) {
                    R yr = 0, yi = 0;
#pragma unroll
                    for (int b = 0; b < D; ++b) {
                        const R ur = ms.re(a * D + b), ui = ms.im(a * D + b);
                        yr = fma(ur, x[j][b].x, yr);
                        yr = fma(-ui, x[j][b].y, yr);
                        yi = fma(ur, x[j][b].y, yi);
                        yi = fma(ui, x[j][b].x, yi);
                    }
                    C2 y;
                    y.x = yr;
                    y.y = yi;
                    st(psi + base[j] + off[a], y, nt);
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------------------
// monomial ("permutation") gates: member a <- phase(a) * member src(a); pure moves, bit-exact.
// ---------------------------------------------------------------------------------------------------------
template <class C2> __device__ __forceinline__ C2 apply_phase(C2 x, int ph)
{
    C2 y;
    if (ph == 0) {
        y = x;
    } else if (ph == 1) {  // i * x
        y.x = -x.y;
        y.y = x.x;
    } else if (ph == 2) {  // -x
        y.x = -x.x;
        y.y = -x.y;
    } else {  // -i * x
        y.x = x.y;
        y.y = -x.x;
    }
    return y;
}

template <class R, int K, int G>
__global__ __launch_bounds__(256) void k_perm(typename CT<R>::T *__restrict__ psi, uint64_t ngroups, InsBits ins,
                                              TPos tp, PermTable pt, int nt)
{
    using C2 = typename CT<R>::T;
    constexpr int D = 1 << K;
    const uint64_t bs = blockDim.x;
    const uint64_t stride = (uint64_t)gridDim.x * bs * G;
    for (uint64_t g0 = (uint64_t)blockIdx.x * bs * G + threadIdx.x; g0 < ngroups; g0 += stride) {
        C2 v[G][D];
        uint64_t base[G];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            uint64_t g = g0 + j * bs;
            base[j] = ins0(g < ngroups ? g : 0, ins);
            if (g < ngroups) {
#pragma unroll
                for (int a = 0; a < D; ++a)
                    if ((pt.moving >> a) & 1)
                        v[j][a] = ld(psi + base[j] + member_off<K>(pt.src[a], tp), nt);
            }
        }
#pragma unroll
        for (int j = 0; j < G; ++j) {
            if (g0 + j * bs < ngroups) {
#pragma unroll
                for (int a = 0; a < D; ++a)
                    if ((pt.moving >> a) & 1)
                        st(psi + base[j] + member_off<K>(a, tp), apply_phase(v[j][a], pt.phase[a]), nt);
            }
        }
    }
}

// Lane-order form of a monomial op over Q for states where every 128-byte line holds amplitudes it changes (a CZ or
// controlled phase on qubits inside the line, a CNOT or Toffoli with a control there): a wave streams 64 consecutive
// 16-byte vectors (one complex128 amplitude or two complex64 ones per lane, LB = 6 or 7 in-wave index bits) for each
// of the 2^H combinations of the out-of-wave qubits of Q, so every access is a whole line in lane order, and each
// output takes its source from the lane, vector slot and member the move table names, by cross-lane reads. Which
// source feeds an output depends only on the lane, so it is worked out once per thread.
template <class R, int H, bool NT>
__global__ __launch_bounds__(256) void k_perm_lanes(typename LaneVec<R>::T *__restrict__ psi, uint64_t nchunks,
                                                    InsBits ins_h, PermLanes pl)
{
    using V = typename LaneVec<R>::T;
    constexpr int P = sizeof(R) == 8 ? 1 : 2;  // amplitudes per 16-byte vector
    constexpr int LB = sizeof(R) == 8 ? 6 : 7;  // in-wave index bits
    constexpr int M = 1 << H;                   // members per lane
    const int lane = threadIdx.x & 63;
    uint64_t hoff[M];
    int sl[M][P], sp[M][P], sm[M][P], ph[M][P];
    {
        int hpos[2] = {0, 0}, nh = 0;
        for (int u = 0; u < pl.nq; ++u)
            if (pl.qpos[u] >= LB)
                hpos[nh++] = pl.qpos[u];
#pragma unroll
        for (int m = 0; m < M; ++m) {
            hoff[m] = 0;
            for (int j = 0; j < H; ++j)
                hoff[m] |= (uint64_t)((m >> j) & 1) << hpos[j];
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const int iw = lane * P + p;
                int a = 0;
                for (int u = 0, j = 0; u < pl.nq; ++u)
                    a |= (pl.qpos[u] < LB ? (iw >> pl.qpos[u]) & 1 : (m >> j++) & 1) << u;
                const int sa = pl.src[a];
                int siw = iw, smem = 0;
                for (int u = 0, j = 0; u < pl.nq; ++u) {
                    const int bit = (sa >> u) & 1;
                    if (pl.qpos[u] < LB)
                        siw = (siw & ~(1 << pl.qpos[u])) | (bit << pl.qpos[u]);
                    else
                        smem |= bit << j++;
                }
                sl[m][p] = siw / P;
                sp[m][p] = siw % P;
                sm[m][p] = smem;
                ph[m][p] = pl.phase[a];
            }
        }
    }
    const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const uint64_t nwaves = ((uint64_t)gridDim.x * blockDim.x) >> 6;
    for (uint64_t c = wave; c < nchunks; c += nwaves) {
        const uint64_t base = qs_ins0(c << LB, ins_h) / P + lane;  // vector index of member 0
        V v[M];
#pragma unroll
        for (int m = 0; m < M; ++m)
            v[m] = NT ? __builtin_nontemporal_load(psi + base + hoff[m] / P) : psi[base + hoff[m] / P];
#pragma unroll
        for (int m = 0; m < M; ++m) {
            V y;
#pragma unroll
            for (int p = 0; p < P; ++p) {
                // the source vector of every candidate member, read from the source lane; keep the named one
                R re = 0, im = 0;
#pragma unroll
                for (int cm = 0; cm < M; ++cm) {
                    R w[2 * P];
#pragma unroll
                    for (int e = 0; e < 2 * P; ++e)
                        w[e] = __shfl(v[cm][e], sl[m][p], 64);
                    if (cm == sm[m][p]) {
                        if constexpr (P == 1) {
                            re = w[0];
                            im = w[1];
                        } else {
                            re = sp[m][p] ? w[2] : w[0];
                            im = sp[m][p] ? w[3] : w[1];
                        }
                    }
                }
                typename CT<R>::T z;
                z.x = re;
                z.y = im;
                z = apply_phase(z, ph[m][p]);
                y[2 * p] = z.x;
                y[2 * p + 1] = z.y;
            }
            if constexpr (NT)
                __builtin_nontemporal_store(y, psi + base + hoff[m] / P);
            else
                psi[base + hoff[m] / P] = y;
        }
    }
}

// ---------------------------------------------------------------------------------------------------------
// diagonal gates
// ---------------------------------------------------------------------------------------------------------
// Streaming diagonals, one 16-byte vector (one complex128 amplitude, two complex64 ones) per thread. cls: 4 bits per
// entry, 0: untouched (entry exactly 1), 1: negate (exactly -1), 2: multiply.
template <class R> struct DiagSmall {  // k <= 2: entries and classes in kernel arguments, selected, never indexed
    R re[4], im[4];
    uint32_t cls;
};

template <class R> __device__ __forceinline__ void diag_apply(R &x, R &y, uint32_t cls, R dr, R di)
{
    const R r = fma(dr, x, -di * y), i = fma(dr, y, di * x);
    x = cls == 2 ? r : cls == 1 ? -x : x;
    y = cls == 2 ? i : cls == 1 ? -y : y;
}

// Bound by HBM. The entries come from scalar registers by selection: indexed by the lane they were loads of their own,
// in front of the amplitude's. 27 qubits, RZ: complex128 659 us against 740, complex64 328 against
// 411; 23 qubits 37 against 47 and 20 against 27.
template <class R, int K, bool NT>
__global__ __launch_bounds__(256) void k_diag_small(typename LaneVec<R>::T *__restrict__ psi, uint64_t nvec,
                                                    int t0, int t1, DiagSmall<R> ds)
{
    using V = typename LaneVec<R>::T;
    constexpr int P = sizeof(R) == 8 ? 1 : 2;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < nvec; v += stride) {
        uint32_t cl[P];
        bool b0[P], b1[P];
#pragma unroll
        for (int h = 0; h < P; ++h) {
            const uint64_t i = v * P + h;
            b0[h] = (i >> t0) & 1;
            b1[h] = K == 2 && ((i >> t1) & 1);
            cl[h] = (ds.cls >> (4 * ((int)b0[h] + 2 * (int)b1[h]))) & 15u;
        }
        if (!(cl[0] | cl[P - 1]))
            continue;
        V x = NT ? __builtin_nontemporal_load(psi + v) : psi[v];
#pragma unroll
        for (int h = 0; h < P; ++h) {
            R dr = b0[h] ? ds.re[1] : ds.re[0], di = b0[h] ? ds.im[1] : ds.im[0];
            if constexpr (K == 2) {
                dr = b1[h] ? (b0[h] ? ds.re[3] : ds.re[2]) : dr;
                di = b1[h] ? (b0[h] ? ds.im[3] : ds.im[2]) : di;
            }
            R re = x[2 * h], im = x[2 * h + 1];
            diag_apply(re, im, cl[h], dr, di);
            x[2 * h] = re;
            x[2 * h + 1] = im;
        }
        if constexpr (NT)
            __builtin_nontemporal_store(x, psi + v);
        else
            psi[v] = x;
    }
}

// k >= 3: the 2^k entries (in the compute precision) and classes come from a table: for k <= 6 in the kernel's own
// arguments (through the staging ring two copies a gate made a 3-qubit diagonal on 21 qubits take 29 us; 9 us now),
// beyond in device memory. The index bits above a block's vectors are the block's: they are gathered on the scalar unit.
// 27 qubits, 3 targets: complex128 676 us against 746, complex64 369 against 606. full: no entry is 1, and the loads need
// not wait for their class; otherwise an amplitude whose entry is 1 is not accessed.
template <class R> struct DiagTable {
    R d[128];
    uint8_t cls[64];
};
template <class R, bool NT>
__device__ __forceinline__ void diag_stream(typename LaneVec<R>::T *__restrict__ psi, uint64_t nvec, const DiagArgs &da,
                                            const R *d, const uint8_t *cls, int full)
{
    using V = typename LaneVec<R>::T;
    constexpr int P = sizeof(R) == 8 ? 1 : 2;
    constexpr int LB = P == 1 ? 8 : 9;  // index bits within a block's vectors
    const uint32_t low = threadIdx.x * P;
    for (uint64_t b = blockIdx.x; b * 256 < nvec; b += gridDim.x) {
        const uint64_t v = b * 256 + threadIdx.x;
        if (v >= nvec)
            return;
        V x;
        if (full)
            x = NT ? __builtin_nontemporal_load(psi + v) : psi[v];
        uint32_t ab = 0, a0 = 0, a1 = 0;
        for (int q = 0; q < da.k; ++q) {
            const int t = da.t[q];
            if (t >= LB) {
                ab |= (uint32_t)((b * 256 * P >> t) & 1) << q;
            } else {
                a0 |= ((low >> t) & 1u) << q;
                a1 |= (((low | 1u) >> t) & 1u) << q;
            }
        }
        const uint32_t a[2] = {ab | a0, ab | a1};
        if (full) {
#pragma unroll
            for (int h = 0; h < P; ++h) {
                R re = x[2 * h], im = x[2 * h + 1];
                diag_apply(re, im, cls[a[h]], d[2 * a[h]], d[2 * a[h] + 1]);
                x[2 * h] = re;
                x[2 * h + 1] = im;
            }
            if constexpr (NT)
                __builtin_nontemporal_store(x, psi + v);
            else
                psi[v] = x;
            continue;
        }
        typename CT<R>::T *amp = reinterpret_cast<typename CT<R>::T *>(psi + v);
#pragma unroll
        for (int h = 0; h < P; ++h) {
            const uint32_t c = cls[a[h]];
            if (!c)
                continue;
            typename CT<R>::T z = ld(amp + h, NT);
            diag_apply(z.x, z.y, c, d[2 * a[h]], d[2 * a[h] + 1]);
            st(amp + h, z, NT);
        }
    }
}
template <class R, bool NT>
__global__ __launch_bounds__(256) void k_diag_args(typename LaneVec<R>::T *__restrict__ psi, uint64_t nvec, DiagArgs da,
                                                   DiagTable<R> tab, int full)
{
    diag_stream<R, NT>(psi, nvec, da, tab.d, tab.cls, full);
}
template <class R, bool NT>
__global__ __launch_bounds__(256) void k_diag_table(typename LaneVec<R>::T *__restrict__ psi, uint64_t nvec, DiagArgs da,
                                                    const R *__restrict__ d, const uint8_t *__restrict__ cls,
                                                    int full)
{
    diag_stream<R, NT>(psi, nvec, da, d, cls, full);
}

struct SparseArgs {
    int m;
    DiagSparseEntry e[kMaxSparseDiag];
};

// Only the subspaces whose pattern has an entry != 1 are visited: blockIdx.y selects the pattern.
template <class R, int G, bool NT>
__global__ __launch_bounds__(256) void k_diag_sparse(typename CT<R>::T *__restrict__ psi, uint64_t nsub,
                                                     InsBits ins, SparseArgs sa)
{
    using C2 = typename CT<R>::T;
    const DiagSparseEntry &e = sa.e[blockIdx.y];
    const uint64_t bs = blockDim.x;
    const uint64_t stride = (uint64_t)gridDim.x * bs * G;
    for (uint64_t g0 = (uint64_t)blockIdx.x * bs * G + threadIdx.x; g0 < nsub; g0 += stride) {
        C2 x[G];
        uint64_t idx[G];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            const uint64_t g = g0 + j * bs;
            idx[j] = ins0(g < nsub ? g : 0, ins) | e.orm;
            if (g < nsub)
                x[j] = ld(psi + idx[j], NT);
        }
#pragma unroll
        for (int j = 0; j < G; ++j) {
            if (g0 + j * bs >= nsub)
                continue;
            C2 y;
            if (e.cls == 1) {
                y.x = -x[j].x;
                y.y = -x[j].y;
            } else {
                const R dr = (R)e.re, di = (R)e.im;
                y.x = fma(dr, x[j].x, -di * x[j].y);
                y.y = fma(dr, x[j].y, di * x[j].x);
            }
            st(psi + idx[j], y, NT);
        }
    }
}

// ---------------------------------------------------------------------------------------------------------
// fused-swap (Sec. III-D, Listing 1): sigma exchanges bits [lo, lo+s) with [hi, hi+s), lo + s <= hi.
// Index layout: | top | A = bits [hi, hi+s) | mid | B = bits [lo, lo+s) | e = bits [0, lo) |.
// ---------------------------------------------------------------------------------------------------------
__device__ __forceinline__ uint64_t sigma_bits(uint64_t i, int lo, int hi, uint64_t smask)
{
    return fsw_sigma(i, lo, hi, smask);
}

// Generic form: one thread per index; the member of each moved pair with the smaller index does the swap.
template <class C2>
__global__ __launch_bounds__(256) void k_fswap_pairs(C2 *__restrict__ psi, uint64_t dim, int lo, int hi, uint64_t smask)
{
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < dim;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t j = sigma_bits(i, lo, hi, smask);
        if (j > i) {
            const C2 a = psi[i], b = psi[j];
            psi[i] = b;
            psi[j] = a;
        }
    }
}

// Run form (runs of at least 256 bytes, or one 128-byte line with s <= 4): thread -> (outer, pair a > b, element e);
// the runs (A=a, B=b) and (A=b, B=a) are exchanged with coalesced 16-byte lanes along e.
template <class C2>
__global__ __launch_bounds__(256) void k_fswap_runs(C2 *__restrict__ psi, uint64_t total, int lo, int hi, int s,
                                                    uint64_t npairs)
{
    for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
         t += (uint64_t)gridDim.x * blockDim.x) {
        uint64_t i1, i2;
        fsw_runs_pair(t, lo, hi, s, npairs, i1, i2);
        const C2 x1 = psi[i1], x2 = psi[i2];
        psi[i1] = x2;
        psi[i2] = x1;
    }
}

// LDS form (runs too short for the direct form): a workgroup exchanges the sub-tile pair (I, J) / (J, I) of one
// 2^s x 2^s tile (rows A, contiguous columns B of 2^lo-amplitude runs) through LDS; I == J transposes in
// place. Rows are read and written as contiguous (B, e) segments.
template <class C2, int TS>
__global__ __launch_bounds__(256) void k_fswap_lds(C2 *__restrict__ psi, uint64_t nwork, int lo, int hi, int s,
                                                   int ntile, uint64_t npairs_t)
{
    constexpr int T = 1 << TS;
    const int E = 1 << lo;
    const int row = T * E;         // amplitudes per sub-tile row
    const int rstride = row + 1;   // padded LDS row
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C2 *X = reinterpret_cast<C2 *>(smem_raw);
    C2 *Y = X + (size_t)T * rstride;
    const int nel = T * row;
    (void)ntile;
    for (uint64_t w = blockIdx.x; w < nwork; w += gridDim.x) {
        uint64_t I, J, common;
        fsw_lds_item(w, lo, hi, s, npairs_t, I, J, common);
        // X: rows A in I-range, columns B in J-range.  Y: rows A in J-range, columns B in I-range.
        for (int u = threadIdx.x; u < nel; u += blockDim.x) {
            const int ra = u / row, rc = u % row;  // rc = cb * E + e
            X[ra * rstride + rc] = psi[fsw_lds_x(common, I, J, ra, rc, lo, hi, TS)];
            if (I != J)
                Y[ra * rstride + rc] = psi[fsw_lds_y(common, I, J, ra, rc, lo, hi, TS)];
        }
        lds_barrier();
        for (int u = threadIdx.x; u < nel; u += blockDim.x) {
            const int ra = u / row, rc = u % row;
            const int cb = rc / E, e = rc % E;
            // position (A = I*T + ra, B = J*T + cb) receives the old value at (A = J*T + cb, B = I*T + ra)
            if (I != J) {
                psi[fsw_lds_x(common, I, J, ra, rc, lo, hi, TS)] = Y[cb * rstride + ra * E + e];
                psi[fsw_lds_y(common, I, J, ra, rc, lo, hi, TS)] = X[cb * rstride + ra * E + e];
            } else if (ra != cb) {
                psi[fsw_lds_x(common, I, J, ra, rc, lo, hi, TS)] = X[cb * rstride + ra * E + e];
            }
        }
        lds_barrier();
    }
}

// Wide-row form for runs the direct form does not take, whose 2^s x 2^s tile fits 32 KiB. With x low "mid" bits carried along, the segment
// (mid_low, B, e) for fixed A is contiguous: 2^(x+s+lo) amplitudes (kilobytes). A workgroup loads the 2^s rows
// A = a of one work item with coalesced 16-byte lanes into LDS and writes every row b back with the element at
// (mid_low, B = a, e) taken from row a at (mid_low, B = b, e): 2^x independent 2^s x 2^s transposes at once.
// Fixed points (a == b) share cache lines with moved amplitudes at these sizes and are rewritten unchanged.
template <class C2>
__global__ __launch_bounds__(256) void k_fswap_wide(C2 *__restrict__ psi, uint64_t nwork, int lo, int hi, int s,
                                                    int x)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C2 *X = reinterpret_cast<C2 *>(smem_raw);
    const int R = 1 << (x + s + lo);  // amplitudes per row
    const int RP = R + 1;             // padded LDS row
    const int nel = (1 << s) * R;
    for (uint64_t w = blockIdx.x; w < nwork; w += gridDim.x) {
        const uint64_t base = fsw_wide_base(w, lo, hi, s, x);
        for (int u = threadIdx.x; u < nel; u += blockDim.x) {
            uint64_t g;
            int a, c;
            fsw_wide_load(base, u, lo, hi, s, x, g, a, c);
            X[a * RP + c] = psi[g];
        }
        lds_barrier();
        for (int u = threadIdx.x; u < nel; u += blockDim.x) {
            uint64_t g;
            int a, cs;
            fsw_wide_store(base, u, lo, hi, s, x, g, a, cs);
            psi[g] = X[a * RP + cs];
        }
        lds_barrier();
    }
}

// ---------------------------------------------------------------------------------------------------------
// probabilities, norm, scale, init
// ---------------------------------------------------------------------------------------------------------
__device__ __forceinline__ void kahan_add(double &s, double &c, double v)
{
    const double y = v - c;
    const double t = s + y;
    c = (t - s) - y;
    s = t;
}

// out[i] = |a_i|^2 (FP64); partials[blockIdx.x] = compensated sum of this block's share, reduced in a fixed order. Each
// lane streams 16-byte vectors (one complex128 amplitude or two complex64 ones), four in flight, a block's four next to
// each other so that the resident blocks sweep one contiguous window. Bound by HBM: norm alone at 29 qubits complex128
// 1.27 ms = 6.8 TB/s, with probabilities 2.25 ms = 5.7 TB/s (one amplitude per lane and grid stride: 1.78 and 2.76 ms).
// NT, non-temporal loads and stores: faster from 256 MiB of state on (25 qubits complex128 with probabilities 130 us
// against 150), slower where the caches hold the state (23 qubits: 35 against 30).
template <class R, bool NT>
__global__ __launch_bounds__(256) void k_probs(const typename LaneVec<R>::T *__restrict__ psi, uint64_t nvec,
                                               double *__restrict__ out, double *__restrict__ partials)
{
    using V = typename LaneVec<R>::T;
    typedef double D2 __attribute__((ext_vector_type(2), aligned(8)));  // out is any array of doubles
    constexpr int U = 4;
    __shared__ double red[256];
    double s = 0.0, c = 0.0;
    auto get = [&](uint64_t v) -> V {
        if constexpr (NT)
            return __builtin_nontemporal_load(psi + v);
        else
            return psi[v];
    };
    auto one = [&](const V &x, uint64_t v) {
        const double p = (double)x.x * (double)x.x + (double)x.y * (double)x.y;
        if constexpr (sizeof(R) == 8) {
            if (out) {
                if constexpr (NT)
                    __builtin_nontemporal_store(p, out + v);
                else
                    out[v] = p;
            }
            kahan_add(s, c, p);
        } else {
            const double q = (double)x.z * (double)x.z + (double)x.w * (double)x.w;
            if (out) {
                if constexpr (NT)
                    __builtin_nontemporal_store(D2{p, q}, reinterpret_cast<D2 *>(out) + v);
                else
                    reinterpret_cast<D2 *>(out)[v] = D2{p, q};
            }
            kahan_add(s, c, p);
            kahan_add(s, c, q);
        }
    };
    const uint64_t stride = (uint64_t)gridDim.x * 256 * U;
    for (uint64_t v = (uint64_t)blockIdx.x * 256 * U + threadIdx.x; v < nvec; v += stride) {
        if (v + (U - 1) * 256 < nvec) {
            V x[U];
#pragma unroll
            for (int j = 0; j < U; ++j)
                x[j] = get(v + j * 256);
#pragma unroll
            for (int j = 0; j < U; ++j)
                one(x[j], v + j * 256);
        } else {
            for (uint64_t w = v; w < nvec; w += 256)
                one(get(w), w);
        }
    }
    red[threadIdx.x] = s - c;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        partials[blockIdx.x] = red[0];
}

// *result = the sum of the partials in a fixed order; also to pinned host memory where `host` is given.
__global__ __launch_bounds__(256) void k_sum_partials(const double *__restrict__ partials, int nb,
                                                      double *__restrict__ result, double *__restrict__ host)
{
    __shared__ double red[256];
    double s = 0.0, c = 0.0;
    for (int i = threadIdx.x; i < nb; i += blockDim.x)
        kahan_add(s, c, partials[i]);
    red[threadIdx.x] = s - c;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        *result = red[0];
        if (host)
            *host = red[0];
    }
}

// One 16-byte vector per thread, factor and products in FP64. 27 qubits: complex128 653 us against 797, complex64 330
// against 352 with one amplitude per thread and step.
template <class R, bool NT>
__global__ __launch_bounds__(256) void k_scale(typename LaneVec<R>::T *__restrict__ psi, uint64_t nvec, double f,
                                               const double *__restrict__ norm_dev)
{
    using V = typename LaneVec<R>::T;
    const double ff = norm_dev ? 1.0 / sqrt(*norm_dev) : f;
    for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < nvec;
         v += (uint64_t)gridDim.x * blockDim.x) {
        V x = NT ? __builtin_nontemporal_load(psi + v) : psi[v];
#pragma unroll
        for (int e = 0; e < (int)(16 / sizeof(R)); ++e)
            x[e] = (R)((double)x[e] * ff);
        if constexpr (NT)
            __builtin_nontemporal_store(x, psi + v);
        else
            psi[v] = x;
    }
}

// One 16-byte vector per thread (up to 2^31 threads): the write front is contiguous. 27 qubits complex128 314 us =
// 6.85 TB/s, against 375 us with eight vectors per thread a grid apart.
template <class R>
__global__ __launch_bounds__(256) void k_init_zero(typename LaneVec<R>::T *__restrict__ psi, uint64_t nvec)
{
    using V = typename LaneVec<R>::T;
    for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < nvec;
         v += (uint64_t)gridDim.x * blockDim.x) {
        V x;
#pragma unroll
        for (int e = 0; e < (int)(16 / sizeof(R)); ++e)
            x[e] = 0;
        if (v == 0)
            x[0] = 1;
        psi[v] = x;
    }
}

// ---------------------------------------------------------------------------------------------------------
// bandwidth probes
// ---------------------------------------------------------------------------------------------------------
template <int G>
__global__ __launch_bounds__(256) void k_probe_copy(double2 *__restrict__ dst, const double2 *__restrict__ src,
                                                    uint64_t nw)
{
    const uint64_t bs = blockDim.x;
    for (uint64_t i0 = (uint64_t)blockIdx.x * bs * G + threadIdx.x; i0 < nw; i0 += (uint64_t)gridDim.x * bs * G) {
        double2 v[G];
#pragma unroll
        for (int j = 0; j < G; ++j)
            if (i0 + j * bs < nw)
                v[j] = src[i0 + j * bs];
#pragma unroll
        for (int j = 0; j < G; ++j)
            if (i0 + j * bs < nw)
                dst[i0 + j * bs] = v[j];
    }
}

// In-place pass: every 16-byte word is read, scaled by a runtime factor and written back (one word per thread,
// non-temporal), the access pattern of a gate pass with the arithmetic removed.
__global__ __launch_bounds__(256) void k_probe_rmw(double2 *__restrict__ buf, uint64_t nw, double f)
{
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nw; i += (uint64_t)gridDim.x * blockDim.x) {
        double2 v = ld(buf + i, 1);
        v.x *= f;
        v.y *= f;
        st(buf + i, v, 1);
    }
}

// Grid for a grid-stride loop over `work` items at `per_block` items per block. Streaming gate kernels run best
// with one item per thread and a grid that covers the work in a single sweep; the cap keeps the total thread
// count at or below 2^31 (the grid-stride loop covers anything larger).
unsigned grid_for(uint64_t work, uint64_t per_block)
{
    uint64_t b = (work + per_block - 1) / per_block;
    const uint64_t cap = (uint64_t)1 << 23;
    if (b > cap)
        b = cap;
    if (b == 0)
        b = 1;
    return (unsigned)b;
}

}  // namespace

Tunables &qs_tunables()
{
    static Tunables t;
    return t;
}

// =============================================================================================================
// launchers
// =============================================================================================================
hipError_t launch_init_zero(int dtype, void *psi, uint64_t dim, hipStream_t s)
{
    const uint64_t nvec = dtype == QS_C128 ? dim : dim / 2;
    const unsigned g = grid_for(nvec, 256);
    if (dtype == QS_C128)
        hipLaunchKernelGGL(k_init_zero<double>, dim3(g), dim3(256), 0, s, (LaneVec<double>::T *)psi, nvec);
    else
        hipLaunchKernelGGL(k_init_zero<float>, dim3(g), dim3(256), 0, s, (LaneVec<float>::T *)psi, nvec);
    return hipGetLastError();
}

namespace {
// Non-temporal accesses help where whole cache lines are touched; when a target sits inside a 128-byte line the members of
// a group share lines across load instructions, so the loads go through the cache instead. A control inside a line halves
// the lines: no gain on cached states (20 qubits complex128, controlled 1-qubit gate: 6.2 us, non-temporal 8.2).
template <class R> int nt_for(const TPos &tp, int k, uint64_t ngroups, const InsBits &ins)
{
    constexpr int line_bits = sizeof(typename CT<R>::T) == 16 ? 3 : 4;
    const uint64_t bytes = (ngroups << ins.np) * sizeof(typename CT<R>::T);
    const bool low_control = (ins.orm & ((1u << line_bits) - 1)) != 0;
    if (!(low_control ? qs_streams(bytes) : qs_streams_lines(bytes)))
        return 0;
    for (int j = 0; j < k; ++j)
        if (tp.tpos[j] < line_bits)
            return 0;
    return qs_tunables().nontemporal;
}

template <class R, int K>
hipError_t dense_k(void *psi, uint64_t ngroups, const InsBits &ins, const TPos &tp, const double *Uh, const void *Ud,
                   hipStream_t s)
{
    using C2 = typename CT<R>::T;
    struct {
        int dense_gpt, nontemporal;
    } tu{qs_tunables().dense_gpt.load(), nt_for<R>(tp, K, ngroups, ins)};
    const int bs = 256;
    if constexpr (K <= 3) {
        MatByVal<R, K> m;
        for (int i = 0; i < (2 << (2 * K)); ++i)
            m.v[i] = (R)Uh[i];
        if constexpr (K == 1) {
            // a plain 1-qubit gate (no controls) whose partner lies inside the wave: the lane-exchange form
            const uint64_t dim = ngroups * 2;
            const uint64_t nvec = sizeof(R) == 8 ? dim : dim / 2;
            if (ins.np == 1 && ins.orm == 0 &&
                qs_dense1_in_lanes(sizeof(R) == 8 ? QS_C128 : QS_C64, __builtin_ctzll(dim), tp.tpos[0])) {
                using V = typename LaneVec<R>::T;
                if (qs_streams_lines(nvec * 16))
                    hipLaunchKernelGGL((k_dense1_lane<R, true>), dim3(grid_for(nvec, bs)), dim3(bs), 0, s, (V *)psi,
                                       nvec, tp.tpos[0], m);
                else
                    hipLaunchKernelGGL((k_dense1_lane<R, false>), dim3(grid_for(nvec, bs)), dim3(bs), 0, s, (V *)psi,
                                       nvec, tp.tpos[0], m);
                return hipGetLastError();
            }
        }
        if (K <= 2 && tu.dense_gpt == 4) {
            hipLaunchKernelGGL((k_dense<R, K, 4, MatByVal<R, K>>), dim3(grid_for(ngroups, bs * 4)), dim3(bs), 0, s,
                               (C2 *)psi, ngroups, ins, tp, m, tu.nontemporal);
        } else if (K <= 2 && tu.dense_gpt == 2) {
            hipLaunchKernelGGL((k_dense<R, K, 2, MatByVal<R, K>>), dim3(grid_for(ngroups, bs * 2)), dim3(bs), 0, s,
                               (C2 *)psi, ngroups, ins, tp, m, tu.nontemporal);
        } else {
            hipLaunchKernelGGL((k_dense<R, K, 1, MatByVal<R, K>>), dim3(grid_for(ngroups, bs)), dim3(bs), 0, s,
                               (C2 *)psi, ngroups, ins, tp, m, tu.nontemporal);
        }
    } else {
        // k = 4 from HBM with no target or control inside a 128-byte line: groups in registers, which depend less on where
        // the targets lie than the tiles do (27 qubits complex128, targets 5 9 13 20: 765 us against 929, 4 8 15 24: 763
        // against 814, 10 12 17 23: 766 against 699; SU(4) layers in 4-qubit blocks 770 against 820 a pass; complex64,
        // targets 5 9 10 26: 367 against 402, 4 13 14 26: 366 and 368). In cache (24 qubits complex128: 111 against 95,
        // complex64 54 and 39), with low targets (0 6 11 22 complex128: 860 against 743) and with low controls (5 13 14 26
        // controlled by 1: 1157 against 884, complex64 572 against 424) the tiles are the better form.
        if constexpr (K == 4) {
            constexpr int line_bits = sizeof(R) == 8 ? 3 : 4;
            if (qs_streams((ngroups << ins.np) * sizeof(C2)) && tp.tpos[0] >= line_bits &&
                !(ins.orm & ((1u << line_bits) - 1))) {
                hipLaunchKernelGGL((k_dense<R, 4, 1, MatByPtr<R>>), dim3(grid_for(ngroups, bs)), dim3(bs), 0, s, (C2 *)psi,
                                   ngroups, ins, tp, MatByPtr<R>{(const R *)Ud}, tu.nontemporal);
                return hipGetLastError();
            }
        }
        return launch_dense_mfma(std::is_same<R, double>::value ? QS_C128 : QS_C64, K, psi, ngroups, ins, tp, Ud, s);
    }
    return hipGetLastError();
}

template <class R>
hipError_t dense_r(int k, void *psi, uint64_t ngroups, const InsBits &ins, const TPos &tp, const double *Uh,
                   const void *Ud, hipStream_t s)
{
    switch (k) {
    case 1: return dense_k<R, 1>(psi, ngroups, ins, tp, Uh, Ud, s);
    case 2: return dense_k<R, 2>(psi, ngroups, ins, tp, Uh, Ud, s);
    case 3: return dense_k<R, 3>(psi, ngroups, ins, tp, Uh, Ud, s);
    case 4: return dense_k<R, 4>(psi, ngroups, ins, tp, Uh, Ud, s);
    case 5: return dense_k<R, 5>(psi, ngroups, ins, tp, Uh, Ud, s);
    case 6: return dense_k<R, 6>(psi, ngroups, ins, tp, Uh, Ud, s);
    default: return hipErrorInvalidValue;
    }
}

template <class R, int K>
hipError_t perm_k(void *psi, uint64_t ngroups, const InsBits &ins, const TPos &tp, const PermTable &pt, hipStream_t s)
{
    using C2 = typename CT<R>::T;
    constexpr int G = 1;
    hipLaunchKernelGGL((k_perm<R, K, G>), dim3(grid_for(ngroups, 256 * G)), dim3(256), 0, s, (C2 *)psi, ngroups, ins,
                       tp, pt, nt_for<R>(tp, K, ngroups, ins));
    return hipGetLastError();
}

template <class R>
hipError_t perm_r(int k, void *psi, uint64_t ngroups, const InsBits &ins, const TPos &tp, const PermTable &pt,
                  hipStream_t s)
{
    switch (k) {
    case 1: return perm_k<R, 1>(psi, ngroups, ins, tp, pt, s);
    case 2: return perm_k<R, 2>(psi, ngroups, ins, tp, pt, s);
    case 3: return perm_k<R, 3>(psi, ngroups, ins, tp, pt, s);
    case 4: return perm_k<R, 4>(psi, ngroups, ins, tp, pt, s);
    case 5: return perm_k<R, 5>(psi, ngroups, ins, tp, pt, s);
    case 6: return perm_k<R, 6>(psi, ngroups, ins, tp, pt, s);
    default: return hipErrorInvalidValue;
    }
}
}  // namespace

hipError_t launch_dense(int dtype, int k, void *psi, uint64_t ngroups, const InsBits &ins, const TPos &tp,
                        const double *U_host_sorted, const void *U_dev, hipStream_t s)
{
    return dtype == QS_C128 ? dense_r<double>(k, psi, ngroups, ins, tp, U_host_sorted, U_dev, s)
                            : dense_r<float>(k, psi, ngroups, ins, tp, U_host_sorted, U_dev, s);
}

hipError_t launch_perm(int dtype, int k, void *psi, uint64_t ngroups, const InsBits &ins, const TPos &tp,
                       const PermTable &pt, hipStream_t s)
{
    return dtype == QS_C128 ? perm_r<double>(k, psi, ngroups, ins, tp, pt, s)
                            : perm_r<float>(k, psi, ngroups, ins, tp, pt, s);
}

hipError_t launch_perm_lanes(int dtype, void *psi, int n, const PermLanes &pl, hipStream_t s)
{
    const int LB = dtype == QS_C128 ? 6 : 7;
    int h = 0;
    uint64_t hmask = 0;
    for (int u = 0; u < pl.nq; ++u)
        if (pl.qpos[u] >= LB) {
            ++h;
            hmask |= (uint64_t)1 << pl.qpos[u];
        }
    if (pl.nq < 1 || pl.nq > 6 || h > 2 || n < LB + h)
        return hipErrorInvalidValue;
    const InsBits ins_h = qs_make_ins(hmask, 0);
    const uint64_t nchunks = (uint64_t)1 << (n - LB - h);
    const unsigned g = grid_for(nchunks * 64, 256);
    const bool nt = qs_streams(((uint64_t)1 << n) * amp_bytes(dtype));
    auto go = [&](auto kernel, auto *p) {
        hipLaunchKernelGGL(kernel, dim3(g), dim3(256), 0, s, p, nchunks, ins_h, pl);
        return hipGetLastError();
    };
    if (dtype == QS_C128) {
        auto *p = (LaneVec<double>::T *)psi;
        switch (2 * h + nt) {
        case 0: return go(k_perm_lanes<double, 0, false>, p);
        case 1: return go(k_perm_lanes<double, 0, true>, p);
        case 2: return go(k_perm_lanes<double, 1, false>, p);
        case 3: return go(k_perm_lanes<double, 1, true>, p);
        case 4: return go(k_perm_lanes<double, 2, false>, p);
        default: return go(k_perm_lanes<double, 2, true>, p);
        }
    }
    auto *p = (LaneVec<float>::T *)psi;
    switch (2 * h + nt) {
    case 0: return go(k_perm_lanes<float, 0, false>, p);
    case 1: return go(k_perm_lanes<float, 0, true>, p);
    case 2: return go(k_perm_lanes<float, 1, false>, p);
    case 3: return go(k_perm_lanes<float, 1, true>, p);
    case 4: return go(k_perm_lanes<float, 2, false>, p);
    default: return go(k_perm_lanes<float, 2, true>, p);
    }
}

namespace {
template <class R, bool NT>
hipError_t diag_r(void *psi_, uint64_t dim, const DiagArgs &da, const double *d, const void *d_dev, const uint8_t *cls,
                  hipStream_t s)
{
    using V = typename LaneVec<R>::T;
    V *psi = (V *)psi_;
    const uint64_t nvec = sizeof(R) == 8 ? dim : dim / 2;
    const dim3 g(grid_for(nvec, 256)), b(256);
    const int D = 1 << da.k;
    const int full = std::find(cls, cls + D, 0) == cls + D;
    if (da.k <= 2) {
        DiagSmall<R> ds{};
        for (int a = 0; a < D; ++a) {
            ds.re[a] = (R)d[2 * a];
            ds.im[a] = (R)d[2 * a + 1];
            ds.cls |= (uint32_t)cls[a] << (4 * a);
        }
        if (da.k == 1)
            hipLaunchKernelGGL((k_diag_small<R, 1, NT>), g, b, 0, s, psi, nvec, da.t[0], 0, ds);
        else
            hipLaunchKernelGGL((k_diag_small<R, 2, NT>), g, b, 0, s, psi, nvec, da.t[0], da.t[1], ds);
    } else if (da.k <= 6) {
        DiagTable<R> tab;
        for (int a = 0; a < 2 * D; ++a)
            tab.d[a] = (R)d[a];
        for (int a = 0; a < D; ++a)
            tab.cls[a] = cls[a];
        hipLaunchKernelGGL((k_diag_args<R, NT>), g, b, 0, s, psi, nvec, da, tab, full);
    } else {
        const R *dd = (const R *)d_dev;
        hipLaunchKernelGGL((k_diag_table<R, NT>), g, b, 0, s, psi, nvec, da, dd, (const uint8_t *)(dd + 2 * D),
                           full);
    }
    return hipGetLastError();
}
}  // namespace

hipError_t launch_diag_full(int dtype, void *psi, uint64_t dim, const DiagArgs &da, const double *d, const void *d_dev,
                            const uint8_t *cls, hipStream_t s)
{
    const bool nt = qs_streams(dim * amp_bytes(dtype));
    if (dtype == QS_C128)
        return nt ? diag_r<double, true>(psi, dim, da, d, d_dev, cls, s)
                  : diag_r<double, false>(psi, dim, da, d, d_dev, cls, s);
    return nt ? diag_r<float, true>(psi, dim, da, d, d_dev, cls, s)
              : diag_r<float, false>(psi, dim, da, d, d_dev, cls, s);
}

hipError_t launch_diag_sparse(int dtype, void *psi, uint64_t nsub, const InsBits &ins, int m,
                              const DiagSparseEntry *ent, hipStream_t s)
{
    if (m < 1 || m > kMaxSparseDiag)
        return hipErrorInvalidValue;
    SparseArgs sa{};
    sa.m = m;
    for (int i = 0; i < m; ++i)
        sa.e[i] = ent[i];
    const int G = 1;
    const dim3 grid(grid_for(nsub, 256 * G), m), b(256);
    const bool nt = qs_streams((nsub << ins.np) * amp_bytes(dtype));
    if (dtype == QS_C128) {
        if (nt)
            hipLaunchKernelGGL((k_diag_sparse<double, G, true>), grid, b, 0, s, (double2 *)psi, nsub, ins, sa);
        else
            hipLaunchKernelGGL((k_diag_sparse<double, G, false>), grid, b, 0, s, (double2 *)psi, nsub, ins, sa);
    } else {
        if (nt)
            hipLaunchKernelGGL((k_diag_sparse<float, G, true>), grid, b, 0, s, (float2 *)psi, nsub, ins, sa);
        else
            hipLaunchKernelGGL((k_diag_sparse<float, G, false>), grid, b, 0, s, (float2 *)psi, nsub, ins, sa);
    }
    return hipGetLastError();
}

namespace {
template <class C2>
hipError_t fswap_t(void *psi_, int n, int lo, int hi, int s_, hipStream_t s)
{
    C2 *psi = (C2 *)psi_;
    const FswPlan f = fsw_plan(n, lo, hi, s_, (int)sizeof(C2));
    const unsigned g = (unsigned)(f.nwork < (1u << 20) ? f.nwork : (1u << 20));
    switch (f.form) {
    case FSW_RUNS:
        hipLaunchKernelGGL(k_fswap_runs<C2>, dim3(grid_for(f.nwork, 256)), dim3(256), 0, s, psi, f.nwork, lo, hi, s_,
                           f.npairs);
        break;
    case FSW_WIDE:
        hipLaunchKernelGGL(k_fswap_wide<C2>, dim3(g), dim3(256), f.shm, s, psi, f.nwork, lo, hi, s_, f.x);
        break;
    case FSW_LDS: {
        const int ntile = 1 << (s_ - f.ts);
        switch (f.ts) {
        case 2: hipLaunchKernelGGL((k_fswap_lds<C2, 2>), dim3(g), dim3(256), f.shm, s, psi, f.nwork, lo, hi, s_, ntile, f.npairs); break;
        case 3: hipLaunchKernelGGL((k_fswap_lds<C2, 3>), dim3(g), dim3(256), f.shm, s, psi, f.nwork, lo, hi, s_, ntile, f.npairs); break;
        case 4: hipLaunchKernelGGL((k_fswap_lds<C2, 4>), dim3(g), dim3(256), f.shm, s, psi, f.nwork, lo, hi, s_, ntile, f.npairs); break;
        default: hipLaunchKernelGGL((k_fswap_lds<C2, 5>), dim3(g), dim3(256), f.shm, s, psi, f.nwork, lo, hi, s_, ntile, f.npairs); break;
        }
        break;
    }
    default:
        hipLaunchKernelGGL(k_fswap_pairs<C2>, dim3(grid_for(f.nwork, 256)), dim3(256), 0, s, psi, f.nwork, lo, hi,
                           ((uint64_t)1 << s_) - 1);
        break;
    }
    return hipGetLastError();
}
}  // namespace

namespace {
// A fused-swap within the lowest index bits: 32 KiB of consecutive amplitudes per workgroup, read and written as
// 16-byte vectors, permuted in LDS. (As tiles of 2^s x 2^s runs it left a workgroup as little as 64 bytes: qubits 1 and 2
// of 27, complex64, 5741 us; 362 this way, as any swap of the kind. With more to a tile it moved 8 bytes a lane: 509.) The slots of higher bits
// are folded onto the banks, in pairs for complex64, so that a transposition's columns are spread over them.
template <class R> struct FswTile;
template <> struct FswTile<double> { static constexpr int B = 11; };
template <> struct FswTile<float> { static constexpr int B = 12; };
template <class R> __device__ __forceinline__ uint32_t fsw_slot(uint32_t i)
{
    return sizeof(R) == 8 ? i ^ (((i >> 4) ^ (i >> 8)) & 15u) : i ^ (((i >> 5) ^ (i >> 9)) & 30u);
}
template <class R, bool NT>
__global__ __launch_bounds__(256) void k_fswap_tile(typename LaneVec<R>::T *__restrict__ psi, int lo, int hi, uint32_t sm)
{
    using V = typename LaneVec<R>::T;
    using C2 = typename CT<R>::T;
    constexpr int P = sizeof(R) == 8 ? 1 : 2, N = 1 << FswTile<R>::B, PER = N / P / 256;
    __shared__ __align__(16) C2 s[N];
    V *p = psi + (uint64_t)blockIdx.x * (N / P);
    V x[PER];
#pragma unroll
    for (int it = 0; it < PER; ++it) {
        const V *a = p + threadIdx.x + 256 * it;
        x[it] = NT ? __builtin_nontemporal_load(a) : *a;
    }
#pragma unroll
    for (int it = 0; it < PER; ++it)
        *reinterpret_cast<V *>(&s[fsw_slot<R>((threadIdx.x + 256 * it) * P)]) = x[it];
    __syncthreads();
#pragma unroll
    for (int it = 0; it < PER; ++it) {
        const uint32_t i = (threadIdx.x + 256 * it) * P;
#pragma unroll
        for (int h = 0; h < P; ++h) {
            const C2 z = s[fsw_slot<R>((uint32_t)fsw_sigma(i + h, lo, hi, sm))];
            x[it][2 * h] = z.x;
            x[it][2 * h + 1] = z.y;
        }
        V *a = p + i / P;
        if constexpr (NT)
            __builtin_nontemporal_store(x[it], a);
        else
            *a = x[it];
    }
}
template <class R> hipError_t fswap_tile(void *psi, int n, int lo, int hi, int s_, hipStream_t s)
{
    using V = typename LaneVec<R>::T;
    const dim3 g((unsigned)((uint64_t)1 << (n - FswTile<R>::B))), b(256);
    const uint32_t sm = (1u << s_) - 1u;
    if (qs_streams(((uint64_t)1 << n) * sizeof(typename CT<R>::T)))
        hipLaunchKernelGGL((k_fswap_tile<R, true>), g, b, 0, s, (V *)psi, lo, hi, sm);
    else
        hipLaunchKernelGGL((k_fswap_tile<R, false>), g, b, 0, s, (V *)psi, lo, hi, sm);
    return hipGetLastError();
}
}  // namespace

// Swaps within one line and the lowest bits go tile by tile (from lo on that is a whole line, moving the exchanged runs
// alone is less; complex128 states streaming from HBM only up to bit 6: 27 qubits, lo 0, s 3, hi 3 1189 us against 789,
// but s 4, hi 4 725 against 787). Where tiles are at most 64 (17 qubits, complex64 18) the wide-row form, whose work items of
// 2^(hi + s) amplitudes are up to 1024, is faster (16 qubits, lo 0, s 4, hi 4: tiles 2.6 us, rows 2.3, complex64 2.6 and
// 2.1; with more items the tiles are, 17 qubits, lo 0, s 1, hi 4: 2.7 against 3.4, as with larger ones, lo 1, s 5, hi 6:
// 2.7 against 4.4). Complex64 swaps that leave bit 0 alone move pairs of amplitudes, as complex128 amplitudes of a state of
// one qubit less: 16 bytes a lane (27 qubits, lo 1 to 3, hi far above: 510 us, so 380; 25 qubits, in cache, 84 and 65).
// Whole lines streaming from HBM are the exception: 8 bytes a lane are 5 to 10 % faster (27 qubits, lo 4, s 1: 178 and 195).
hipError_t launch_fused_swap(int dtype, void *psi, int n, int lo, int hi, int s_, hipStream_t s)
{
    const int span = hi + s_;
    const bool rows = n <= (dtype == QS_C128 ? 17 : 18) && span >= 3 && span <= 9 && n - span <= 10;
    if (dtype == QS_C128)
        return lo < 3 && span <= (qs_streams((uint64_t)16 << n) ? 6 : FswTile<double>::B) && n >= FswTile<double>::B && !rows
                   ? fswap_tile<double>(psi, n, lo, hi, s_, s)
                   : fswap_t<double2>(psi, n, lo, hi, s_, s);
    if (lo < 4 && span <= FswTile<float>::B && n >= FswTile<float>::B)
        return rows ? fswap_t<float2>(psi, n, lo, hi, s_, s) : fswap_tile<float>(psi, n, lo, hi, s_, s);
    if (lo >= 1 && (lo < 4 || !qs_streams((uint64_t)8 << n)))
        return fswap_t<double2>(psi, n - 1, lo - 1, hi - 1, s_, s);
    return fswap_t<float2>(psi, n, lo, hi, s_, s);
}

int probs_blocks(uint64_t dim)
{
    uint64_t b = (dim + 256 * 16 - 1) / (256 * 16);
    if (b > 1024)  // one wave of blocks on 256 compute units: 2 to 8 % faster than 4096 blocks
        b = 1024;
    return (int)(b ? b : 1);
}

hipError_t launch_probs(int dtype, const void *psi, uint64_t dim, double *out, double *partials, int nblocks,
                        double *result, hipStream_t s, double *host)
{
    if (nblocks == 1 && result && !host)
        partials = result;  // the one partial sum is the result
    const bool nt = dim * amp_bytes(dtype) >= ((uint64_t)256 << 20);
    const dim3 g(nblocks), b(256);
    if (dtype == QS_C128) {
        using V = LaneVec<double>::T;
        if (nt)
            hipLaunchKernelGGL((k_probs<double, true>), g, b, 0, s, (const V *)psi, dim, out, partials);
        else
            hipLaunchKernelGGL((k_probs<double, false>), g, b, 0, s, (const V *)psi, dim, out, partials);
    } else {
        using V = LaneVec<float>::T;
        if (nt)
            hipLaunchKernelGGL((k_probs<float, true>), g, b, 0, s, (const V *)psi, dim / 2, out, partials);
        else
            hipLaunchKernelGGL((k_probs<float, false>), g, b, 0, s, (const V *)psi, dim / 2, out, partials);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !result || partials == result)
        return e;
    return launch_sum_partials(partials, nblocks, result, s, host);
}

hipError_t launch_sum_partials(const double *partials, int nb, double *result, hipStream_t s, double *host)
{
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, s, partials, nb, result, host);
    return hipGetLastError();
}

namespace {
template <class R> hipError_t scale_r(void *psi, uint64_t dim, double f, const double *norm_dev, hipStream_t s)
{
    using V = typename LaneVec<R>::T;
    const uint64_t nvec = sizeof(R) == 8 ? dim : dim / 2;
    const dim3 g(grid_for(nvec, 256)), b(256);
    if (qs_streams(nvec * 16))
        hipLaunchKernelGGL((k_scale<R, true>), g, b, 0, s, (V *)psi, nvec, f, norm_dev);
    else
        hipLaunchKernelGGL((k_scale<R, false>), g, b, 0, s, (V *)psi, nvec, f, norm_dev);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_scale(int dtype, void *psi, uint64_t dim, double f, hipStream_t s)
{
    return dtype == QS_C128 ? scale_r<double>(psi, dim, f, nullptr, s) : scale_r<float>(psi, dim, f, nullptr, s);
}

hipError_t launch_scale_dev(int dtype, void *psi, uint64_t dim, const double *norm_dev, hipStream_t s)
{
    return dtype == QS_C128 ? scale_r<double>(psi, dim, 0.0, norm_dev, s) : scale_r<float>(psi, dim, 0.0, norm_dev, s);
}

hipError_t launch_probe_copy(void *dst, const void *src, size_t bytes, hipStream_t s)
{
    const uint64_t nw = bytes / 16;
    constexpr int G = 4;
    hipLaunchKernelGGL(k_probe_copy<G>, dim3(grid_for(nw, 256 * G)), dim3(256), 0, s, (double2 *)dst,
                       (const double2 *)src, nw);
    return hipGetLastError();
}

hipError_t launch_probe_rmw(void *buf, size_t bytes, hipStream_t s)
{
    const uint64_t nw = bytes / 16;
    hipLaunchKernelGGL(k_probe_rmw, dim3(grid_for(nw, 256)), dim3(256), 0, s, (double2 *)buf, nw, 1.0);
    return hipGetLastError();
}
