// Circuits on states that fit one workgroup's LDS: every operation of a circuit, in order, in one launch.
//
// Gate by gate, a state of a few thousand amplitudes costs one launch per operation (2.8 to 3.8 us each, of which the
// kernel computes for a fraction). Here one workgroup loads the state into LDS, applies the operations one after
// another, each a pass over LDS with a workgroup barrier behind it, and writes the state back: 195 operations on 10
// qubits (complex128) take 45 us against about 620 as 195 launches. What bounds an operation is the instructions a
// wave issues for it (0.2 to 0.3 us up to 10 qubits), at 12 the LDS traffic as well.
//
// The circuit travels as a program: records of 32 bytes, those of 1- and 2-qubit gates followed by their matrix, packed
// into 8 KiB chunks that the kernel brings into the scalar cache one at a time; larger matrices and tables lie in a
// pool behind them. The program is formed once per circuit and precision, on the host, and goes to the device through
// the runs' ring of the state with each run.
//
// Arithmetic per operation is that of the one-pass kernels, rounding for rounding (1-qubit gates the lane-exchange form
// takes there in its order, matrix entries otherwise in FMA chains in ascending column order, 5 and 6 targets complex64
// in the order of the matrix-core tiles), so that complex64 results are the single calls' bit for bit; monomial gates
// with entries 1, -1, i, -i and fused-swaps are pure moves; diagonal entries 1 leave amplitudes untouched, -1 flips
// signs.
#include <algorithm>
#include <cstring>

#include "qs_internal.h"

namespace {

enum : uint32_t {
    OP_END,     // end of the program
    OP_NEXT,    // end of a chunk
    OP_DENSE11, // two 1-qubit gates on different qubits, the first then the second, in one pass
    OP_DENSE1,  // 1-qubit gate
    OP_MOVE1,   // monomial 1-qubit gate (X, CNOT, Toffoli, Y ...)
    OP_DIAG2,   // diagonal on at most 2 qubits
    OP_DENSE2,
    OP_MOVE2,
    OP_SWAP,
    OP_DIAG,    // more targets
    OP_DENSE,
    OP_MOVE
};

// Entry codes of diagonals: untouched, sign flip, multiply, multiply by i or -i as a move.
enum : uint32_t { D_ONE, D_NEG, D_MUL, D_I, D_MINUS_I };

struct Rec {
    uint32_t kind_size;  // kind, and the record's length in 16-byte units with its matrix << 8
    uint32_t cmask;      // control bits
    uint32_t tmask;      // target bits
    uint32_t k;          // targets
    uint64_t pos;        // target positions, 4 bits each; swap: lo, hi, s, 8 bits each
    uint32_t table;      // moves and diagonals on at most 2 targets: 4 bits per member (source and phase, or code); one
                         // target: the second position repeats the first, so that members 0 and 3 are named; 1-qubit
                         // gates: bits 0 and 1, the first and second gate in the lane-exchange order
    uint32_t off;        // byte offset of the matrix or table in the pool
};
static_assert(sizeof(Rec) == 32, "program record");

constexpr size_t kChunk = 8192;             // bytes: half of the scalar cache
constexpr size_t kTail = sizeof(Rec) + 64;  // what a chunk ends with: a record, read as if a matrix followed

template <class R> struct ST;
template <> struct ST<double> { using C2 = double2; };
template <> struct ST<float> { using C2 = float2; };

template <class C2> __device__ __forceinline__ C2 turn(C2 x, uint32_t ph)  // i^ph x, exactly
{
    C2 y = x;
    if (ph == 1) {
        y.x = -x.y;
        y.y = x.x;
    } else if (ph == 2) {
        y.x = -x.x;
        y.y = -x.y;
    } else if (ph == 3) {
        y.x = x.y;
        y.y = -x.x;
    }
    return y;
}

__device__ __forceinline__ uint32_t insert0(uint32_t g, uint32_t p)
{
    const uint32_t lo = g & ((1u << p) - 1u);
    return ((g ^ lo) << 1) | lo;
}

// bits of i at the k positions in pos (4 bits each), packed, and back
__device__ __forceinline__ uint32_t gather_bits(uint32_t i, uint64_t pos, uint32_t k)
{
    uint32_t a = 0;
    for (uint32_t j = 0; j < k; ++j)
        a |= ((i >> ((pos >> (4 * j)) & 15u)) & 1u) << j;
    return a;
}
__device__ __forceinline__ uint32_t scatter_bits(uint32_t a, uint64_t pos, uint32_t k)
{
    uint32_t i = 0;
    for (uint32_t j = 0; j < k; ++j)
        i |= ((a >> j) & 1u) << ((pos >> (4 * j)) & 15u);
    return i;
}

template <class C2, class R> __device__ __forceinline__ void mul_add(R &yr, R &yi, R ur, R ui, const C2 &x)
{
    yr = fma(ur, x.x, yr);
    yr = fma(-ui, x.y, yr);
    yi = fma(ur, x.y, yi);
    yi = fma(ui, x.x, yi);
}

// lane: in the order of the lane-exchange kernel (own member's products last), else column by column.
template <class C2, class R> __device__ __forceinline__ void pair_gate(C2 &a, C2 &b, const R *u, bool lane)
{
    C2 y{0, 0}, z{0, 0};
    if (lane) {
        y.x = fma(u[0], a.x, fma(-u[1], a.y, fma(u[2], b.x, -u[3] * b.y)));
        y.y = fma(u[0], a.y, fma(u[1], a.x, fma(u[2], b.y, u[3] * b.x)));
        z.x = fma(u[6], b.x, fma(-u[7], b.y, fma(u[4], a.x, -u[5] * a.y)));
        z.y = fma(u[6], b.y, fma(u[7], b.x, fma(u[4], a.y, u[5] * a.x)));
        a = y;
        b = z;
        return;
    }
    mul_add(y.x, y.y, u[0], u[1], a);
    mul_add(y.x, y.y, u[2], u[3], b);
    mul_add(z.x, z.y, u[4], u[5], a);
    mul_add(z.x, z.y, u[6], u[7], b);
    a = y;
    b = z;
}

// The program is read through the scalar cache (constant address space): a record and its matrix take two or three
// instructions and no vector registers. With one or two waves per SIMD an operation costs its instruction count, about
// five cycles each, so that what a wave does per record counts as much as what it does per amplitude: records read
// from LDS as uniform vectors made a run of 195 operations 55 us long instead of 45, handed out by v_readlane 72.
typedef const __attribute__((address_space(4))) uint32_t *cwords;
typedef uint32_t words8 __attribute__((ext_vector_type(8), aligned(4)));
typedef uint32_t words16 __attribute__((ext_vector_type(16), aligned(4)));
struct Fetched {  // a record and the first 64 bytes of its matrix
    words8 h;
    words16 m;
};
__device__ __forceinline__ Fetched fetch(cwords w)
{
    Fetched f;
    f.h = *(const __attribute__((address_space(4))) words8 *)w;
    f.m = *(const __attribute__((address_space(4))) words16 *)(w + 8);
    return f;
}
template <int N> __device__ __forceinline__ void reals(const words16 &m, double *u)
{
#pragma unroll
    for (int e = 0; e < N; ++e)
        u[e] = __builtin_bit_cast(double, (uint64_t)m[2 * e] | (uint64_t)m[2 * e + 1] << 32);
}
template <int N> __device__ __forceinline__ void reals(const words16 &m, float *u)
{
#pragma unroll
    for (int e = 0; e < N; ++e) {
        const uint32_t x = m[e];  // a value: the cast of a vector's element in place takes element 0
        u[e] = __builtin_bit_cast(float, x);
    }
}
template <class R, int N> __device__ __forceinline__ void reals_at(cwords w, R *u)
{
    typedef const __attribute__((address_space(4))) R *creals;
    creals m = (creals)w;
#pragma unroll
    for (int e = 0; e < N; ++e)
        u[e] = m[e];
}

// Bring 64-byte lines [0, lines) at w into the scalar cache, each wave its share, so that the records' loads hit.
__device__ __forceinline__ void warm(cwords w, uint32_t lines, uint32_t wave, uint32_t waves)
{
    for (uint32_t l = wave; l < lines; l += 8 * waves) {
        uint32_t x[8];
#pragma unroll
        for (uint32_t j = 0; j < 8; ++j)
            x[j] = w[16 * (l + j * waves < lines ? l + j * waves : l)];
        asm volatile("" ::"s"(x[0]), "s"(x[1]), "s"(x[2]), "s"(x[3]), "s"(x[4]), "s"(x[5]), "s"(x[6]), "s"(x[7]));
    }
}

// PER: amplitudes of a thread (the state has at most PER blockDim.x of them). An operation that moves amplitudes
// between threads reads its sources into registers, waits for the others, and writes; gates and moves on more than two
// qubits write their results to the state's place in device memory instead and read them back.
template <class R, int PER>
__global__ __launch_bounds__(1024) void k_small(typename ST<R>::C2 *__restrict__ psi, uint32_t dim,
                                                const char *__restrict__ prog, uint32_t bytes,
                                                const char *__restrict__ pool)
{
    using C2 = typename ST<R>::C2;
    extern __shared__ __align__(16) unsigned char smem[];
    C2 *s = reinterpret_cast<C2 *>(smem);
    const uint32_t tid = threadIdx.x, NT = blockDim.x;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int Q4 = PER >= 4 ? PER / 4 : 1;
    {
        C2 x[PER];
#pragma unroll
        for (int it = 0; it < PER; ++it)
            x[it] = psi[tid + it * NT < dim ? tid + it * NT : 0];
#pragma unroll
        for (int it = 0; it < PER; ++it)
            if (tid + it * NT < dim)
                s[tid + it * NT] = x[it];
    }
    for (uint32_t c0 = 0; c0 < bytes; c0 += kChunk) {
        cwords w = (cwords)(prog + c0);
        warm(w, (bytes - c0 < kChunk ? bytes - c0 : (uint32_t)kChunk) / 64, wave, NT / 64);
        lds_barrier();
        Fetched nf = fetch(w);
        while ((nf.h[0] & 255u) > OP_NEXT) {
            const Fetched f = nf;
            const uint32_t ks = f.h[0], kind = ks & 255u;
            const uint32_t cmask = f.h[1], tmask = f.h[2], k = f.h[3], table = f.h[6];
            const uint64_t pos = (uint64_t)f.h[4] | (uint64_t)f.h[5] << 32;
            const uint32_t p0 = f.h[4] & 15u, p1 = (f.h[4] >> 4) & 15u;
            const char *own = pool + f.h[7];
            cwords mat = w + 8;
            w += (ks >> 8) * 4;
            nf = fetch(w);  // one operation ahead (the program ends with slack for it)
            if (kind <= OP_DENSE1) {
                R u[16];
                reals<8>(f.m, u);
                if (kind == OP_DENSE11) {
                    if constexpr (sizeof(R) == 8)
                        reals_at<R, 8>(mat + 16, u + 8);
                    else
                        reals<16>(f.m, u);
                    const uint32_t lo = p0 < p1 ? p0 : p1, hi = p0 < p1 ? p1 : p0;
                    const uint32_t o0 = 1u << p0, o1 = 1u << p1;
                    const bool l0 = table & 1u, l1 = table & 2u;
#pragma unroll
                    for (int it = 0; it < Q4; ++it) {
                        const uint32_t g = tid + it * NT, i = insert0(insert0(g, lo), hi);
                        if (g < dim / 4) {
                            C2 a = s[i], b = s[i | o0], c = s[i | o1], d = s[i | o0 | o1];
                            pair_gate(a, b, u, l0);
                            pair_gate(c, d, u, l0);
                            pair_gate(a, c, u + 8, l1);
                            pair_gate(b, d, u + 8, l1);
                            s[i] = a;
                            s[i | o0] = b;
                            s[i | o1] = c;
                            s[i | o0 | o1] = d;
                        }
                    }
                } else {
#pragma unroll
                    for (int it = 0; it < PER / 2; ++it) {
                        const uint32_t g = tid + it * NT, i = insert0(g, p0);
                        if (g < dim / 2 && (i & cmask) == cmask) {
                            C2 a = s[i], b = s[i | tmask];
                            pair_gate(a, b, u, table & 1u);
                            s[i] = a;
                            s[i | tmask] = b;
                        }
                    }
                }
            } else if (kind <= OP_DIAG2) {
                if (kind == OP_MOVE1) {
                    const bool plain = (table & 0xccu) == 0;
#pragma unroll
                    for (int it = 0; it < PER / 2; ++it) {
                        const uint32_t g = tid + it * NT, i = insert0(g, p0);
                        if (g < dim / 2 && (i & cmask) == cmask) {
                            const C2 a = s[i], b = s[i | tmask];
                            if (plain) {
                                s[i] = b;
                                s[i | tmask] = a;
                            } else {
                                const bool x = table & 1u;  // exchanged
                                s[i] = turn(x ? b : a, (table >> 2) & 3u);
                                s[i | tmask] = turn(x ? a : b, (table >> 6) & 3u);
                            }
                        }
                    }
                } else {
                    R m[8];
                    reals<8>(f.m, m);
#pragma unroll
                    for (int it = 0; it < PER; ++it) {
                        const uint32_t i = tid + it * NT;
                        if (i < dim) {
                            const uint32_t b0 = (i >> p0) & 1u, b1 = (i >> p1) & 1u;
                            const uint32_t what = (table >> (4 * (b0 | b1 << 1))) & 15u;
                            const bool hi = k == 2 && b1;  // entries selected, not indexed
                            const R dr = hi ? (b0 ? m[6] : m[4]) : (b0 ? m[2] : m[0]);
                            const R di = hi ? (b0 ? m[7] : m[5]) : (b0 ? m[3] : m[1]);
                            const C2 x = s[i];
                            C2 y;
                            y.x = fma(dr, x.x, -di * x.y);
                            y.y = fma(dr, x.y, di * x.x);
                            if (what != D_MUL)
                                y = turn(x, what == D_ONE ? 0u : what == D_NEG ? 2u : what == D_I ? 1u : 3u);
                            s[i] = y;
                        }
                    }
                }
            } else if (kind == OP_DENSE2) {
                const uint32_t o0 = 1u << p0, o1 = 1u << p1;
                R m[32];
                reals_at<R, 32>(mat, m);
#pragma unroll
                for (int it = 0; it < Q4; ++it) {
                    const uint32_t g = tid + it * NT, i = insert0(insert0(g, p0), p1);
                    if (g < dim / 4 && (i & cmask) == cmask) {
                        const C2 x[4] = {s[i], s[i | o0], s[i | o1], s[i | o0 | o1]};
                        C2 y[4];
#pragma unroll
                        for (int a = 0; a < 4; ++a) {
                            y[a] = C2{0, 0};
#pragma unroll
                            for (int b = 0; b < 4; ++b)
                                mul_add(y[a].x, y[a].y, m[2 * (4 * a + b)], m[2 * (4 * a + b) + 1], x[b]);
                        }
                        s[i] = y[0];
                        s[i | o0] = y[1];
                        s[i | o1] = y[2];
                        s[i | o0 | o1] = y[3];
                    }
                }
            } else if (kind <= OP_SWAP) {
                const int lo = (int)(pos & 255u), hi = (int)((pos >> 8) & 255u);
                const uint32_t sm = (1u << ((pos >> 16) & 255u)) - 1u;
                C2 y[PER];
#pragma unroll
                for (int it = 0; it < PER; ++it) {
                    const uint32_t i = tid + it * NT;
                    uint32_t src, ph = 0;
                    if (kind == OP_SWAP) {
                        src = (uint32_t)fsw_sigma(i, lo, hi, sm);
                    } else {
                        const uint32_t a = ((i >> p0) & 1u) | ((i >> p1) & 1u) << 1, e = table >> (4 * a);
                        const bool on = (i & cmask) == cmask;
                        src = on ? (i & ~tmask) | (e & 1u) << p0 | ((e >> 1) & 1u) << p1 : i;
                        ph = on ? (e >> 2) & 3u : 0u;
                    }
                    y[it] = turn(s[i < dim ? src : 0], ph);
                }
                lds_barrier();
#pragma unroll
                for (int it = 0; it < PER; ++it)
                    if (tid + it * NT < dim)
                        s[tid + it * NT] = y[it];
            } else if (kind == OP_DIAG) {
                const R *d = reinterpret_cast<const R *>(own);
                const uint8_t *codes = reinterpret_cast<const uint8_t *>(own + (sizeof(C2) << k));
                for (uint32_t i = tid; i < dim; i += NT) {
                    const uint32_t a = gather_bits(i, pos, k), what = codes[a];
                    if (what == D_ONE)
                        continue;
                    const C2 x = s[i];
                    C2 y;
                    if (what == D_MUL) {
                        const R dr = d[2 * a], di = d[2 * a + 1];
                        y.x = fma(dr, x.x, -di * x.y);
                        y.y = fma(dr, x.y, di * x.x);
                    } else {
                        y = turn(x, what == D_NEG ? 2u : what == D_I ? 1u : 3u);
                    }
                    s[i] = y;
                }
            } else {  // OP_DENSE, OP_MOVE
                const R *U = reinterpret_cast<const R *>(own);
                const uint8_t *tab = reinterpret_cast<const uint8_t *>(own);
                for (uint32_t i = tid; i < dim; i += NT) {
                    C2 y = s[i];
                    if ((i & cmask) == cmask) {
                        const uint32_t a = gather_bits(i, pos, k), base = i & ~tmask;
                        if (kind == OP_MOVE) {
                            y = turn(s[base | scatter_bits(tab[a], pos, k)], tab[64 + a]);
                        } else {
                            const R *row = U + ((size_t)a << (k + 1));
                            uint32_t sub = 0;  // the members' offsets, ascending
                            y = C2{0, 0};
                            if (sizeof(R) == 4 && k >= 5) {
                                // four members' real parts, then their imaginary parts; quads alternate between sums
                                C2 odd{0, 0};
                                for (uint32_t b = 0; b < (1u << k); b += 4) {
                                    C2 x[4];
#pragma unroll
                                    for (int e = 0; e < 4; ++e) {
                                        x[e] = s[base | sub];
                                        sub = (sub - tmask) & tmask;
                                    }
                                    C2 acc = b & 4u ? odd : y;
#pragma unroll
                                    for (int e = 0; e < 4; ++e) {
                                        acc.x = fma(row[2 * (b + e)], x[e].x, acc.x);
                                        acc.y = fma(row[2 * (b + e) + 1], x[e].x, acc.y);
                                    }
#pragma unroll
                                    for (int e = 0; e < 4; ++e) {
                                        acc.x = fma(-row[2 * (b + e) + 1], x[e].y, acc.x);
                                        acc.y = fma(row[2 * (b + e)], x[e].y, acc.y);
                                    }
                                    if (b & 4u)
                                        odd = acc;
                                    else
                                        y = acc;
                                }
                                y.x += odd.x;
                                y.y += odd.y;
                            } else {
#pragma unroll 4
                                for (uint32_t b = 0; b < (1u << k); ++b) {
                                    mul_add(y.x, y.y, row[2 * b], row[2 * b + 1], s[base | sub]);
                                    sub = (sub - tmask) & tmask;
                                }
                            }
                        }
                    }
                    psi[i] = y;
                }
                __syncthreads();
                for (uint32_t i = tid; i < dim; i += NT)
                    s[i] = psi[i];
            }
            lds_barrier();
        }
    }
    for (uint32_t i = tid; i < dim; i += NT)
        psi[i] = s[i];
}

// Room for a record of `units` 16-byte units and the record that ends its chunk.
char *take(SmallProgram &P, uint32_t units)
{
    const size_t need = 16 * (size_t)units + kTail;
    if (P.chunks.empty() || P.used + need > kChunk) {
        if (!P.chunks.empty()) {
            Rec r{};
            r.kind_size = OP_NEXT;
            std::memcpy(&P.chunks[P.chunks.size() - kChunk + P.used], &r, sizeof r);
        }
        P.chunks.resize(P.chunks.size() + kChunk, 0);  // zeros: OP_END
        P.used = 0;
    }
    char *p = &P.chunks[P.chunks.size() - kChunk + P.used];
    P.used += 16 * (size_t)units;
    return p;
}

uint32_t pool_take(SmallProgram &P, size_t bytes)
{
    const size_t at = P.pool.size();
    P.pool.resize(at + ((bytes + 15) & ~(size_t)15), 0);
    return (uint32_t)at;
}

void put_reals(char *to, const double *v, size_t n, int dtype)
{
    if (dtype == QS_C128) {
        std::memcpy(to, v, n * sizeof(double));
    } else {
        for (size_t i = 0; i < n; ++i) {
            const float f = (float)v[i];
            std::memcpy(to + i * sizeof f, &f, sizeof f);
        }
    }
}

size_t real_bytes(int dtype) { return amp_bytes(dtype) / 2; }

void emit(SmallProgram &P, Rec r, uint32_t kind, const double *inl, size_t nreal)
{
    const uint32_t units = 2 + (uint32_t)((nreal * real_bytes(P.dtype) + 15) / 16);
    P.last_dense1 = SIZE_MAX;
    r.kind_size = kind | units << 8;
    char *p = take(P, units);
    std::memcpy(p, &r, sizeof r);
    if (nreal)
        put_reals(p + sizeof r, inl, nreal, P.dtype);
}

// A 1-qubit gate right behind another one on a different qubit: both in one pass over the state.
bool join_dense1(SmallProgram &P, const Rec &r, const double *U)
{
    const size_t at = P.last_dense1, mat = 8 * real_bytes(P.dtype);
    if (at == SIZE_MAX || P.used + mat + kTail > kChunk)
        return false;
    char *p = &P.chunks[P.chunks.size() - kChunk + at];
    Rec first;
    std::memcpy(&first, p, sizeof first);
    if (first.tmask == r.tmask)
        return false;
    first.kind_size = OP_DENSE11 | (uint32_t)(2 + 2 * mat / 16) << 8;
    first.tmask |= r.tmask;
    first.table |= r.table << 1;
    first.k = 2;
    first.pos |= r.pos << 4;
    std::memcpy(p, &first, sizeof first);
    put_reals(p + sizeof first + mat, U, 8, P.dtype);
    P.used += mat;
    P.last_dense1 = SIZE_MAX;
    return true;
}

void add_diag(SmallProgram &P, const int *t, int k, const double *d)
{
    const int D = 1 << k;
    std::vector<uint8_t> code(D);
    int m = 0;
    bool phases = true;
    for (int a = 0; a < D; ++a) {
        const double re = d[2 * a], im = d[2 * a + 1];
        code[a] = re == 1.0 && im == 0.0 ? D_ONE : re == -1.0 && im == 0.0 ? D_NEG : D_MUL;
        m += code[a] != D_ONE;
        phases = phases && (code[a] != D_MUL || (re == 0.0 && (im == 1.0 || im == -1.0)));
    }
    if (m == 0)
        return;
    if (phases && m < D && k <= QS_MAX_K)  // as in qs_apply_diag: i and -i are moves where every entry is a phase
        for (int a = 0; a < D; ++a)
            if (code[a] == D_MUL)
                code[a] = d[2 * a + 1] == 1.0 ? D_I : D_MINUS_I;
    Rec r{};
    r.k = (uint32_t)k;
    for (int j = 0; j < k; ++j) {
        r.tmask |= 1u << t[j];
        r.pos |= (uint64_t)t[j] << (4 * j);
    }
    if (k <= 2) {
        for (int a = 0; a < 4; ++a)
            r.table |= (uint32_t)code[k == 1 ? a & 1 : a] << (4 * a);
        if (k == 1)
            r.pos |= r.pos << 4;
        emit(P, r, OP_DIAG2, d, 2 * (size_t)D);
        return;
    }
    r.off = pool_take(P, amp_bytes(P.dtype) * D + D);
    put_reals(&P.pool[r.off], d, 2 * (size_t)D, P.dtype);
    std::memcpy(&P.pool[r.off + amp_bytes(P.dtype) * D], code.data(), D);
    emit(P, r, OP_DIAG, nullptr, 0);
}

}  // namespace

void qs_small_add_diag(SmallProgram &P, const int *t, int k, const double *d)
{
    add_diag(P, t, k, d);
}

void qs_small_add_matrix(SmallProgram &P, const int *t, int k, const int *c, int nc, const double *U)
{
    const int D = 1 << k;
    if (nc == 0 && qs_is_diagonal(U, k)) {
        std::vector<double> d((size_t)2 * D);
        for (int a = 0; a < D; ++a) {
            d[2 * a] = U[2 * (a * D + a)];
            d[2 * a + 1] = U[2 * (a * D + a) + 1];
        }
        add_diag(P, t, k, d.data());
        return;
    }
    TPos tp{};
    int perm[QS_MAX_DIAG_K];
    qs_sort_targets(t, k, tp, perm);
    std::vector<double> Us;
    qs_permute_matrix(U, k, perm, Us);
    Rec r{};
    r.k = (uint32_t)k;
    for (int j = 0; j < k; ++j) {
        r.tmask |= 1u << tp.tpos[j];
        r.pos |= (uint64_t)tp.tpos[j] << (4 * j);
    }
    for (int j = 0; j < nc; ++j)
        r.cmask |= 1u << c[j];
    PermTable pt;
    if (qs_monomial_table(Us, k, pt)) {
        if (!pt.moving)
            return;  // identity
        if (k <= 2) {
            for (int a = 0; a < D; ++a)
                r.table |= (uint32_t)(pt.src[a] | pt.phase[a] << 2) << (4 * a);
            emit(P, r, k == 1 ? OP_MOVE1 : OP_MOVE2, nullptr, 0);
        } else {
            r.off = pool_take(P, 128);
            std::memcpy(&P.pool[r.off], pt.src, 64);
            std::memcpy(&P.pool[r.off + 64], pt.phase, 64);
            emit(P, r, OP_MOVE, nullptr, 0);
        }
        return;
    }
    if (k <= 2) {
        if (k == 1 && nc == 0)
            r.table = qs_dense1_in_lanes(P.dtype, P.n, tp.tpos[0]) ? 1 : 0;
        if (k == 1 && nc == 0 && join_dense1(P, r, Us.data()))
            return;
        emit(P, r, k == 1 ? OP_DENSE1 : OP_DENSE2, Us.data(), Us.size());
        if (k == 1 && nc == 0)
            P.last_dense1 = P.used - 16 * (size_t)(2 + (8 * real_bytes(P.dtype)) / 16);
        return;
    }
    r.off = pool_take(P, Us.size() * real_bytes(P.dtype));
    put_reals(&P.pool[r.off], Us.data(), Us.size(), P.dtype);
    emit(P, r, OP_DENSE, nullptr, 0);
}

void qs_small_add_swap(SmallProgram &P, int p, int q, int s)
{
    Rec r{};
    r.pos = (uint64_t)std::min(p, q) | (uint64_t)std::max(p, q) << 8 | (uint64_t)s << 16;
    emit(P, r, OP_SWAP, nullptr, 0);
}

namespace {
template <class R, int PER>
hipError_t launch_per(qs_state *st, uint32_t dim, int nt, const char *prog, uint32_t bytes, const char *pool)
{
    using C2 = typename ST<R>::C2;
    if (hipError_t e = qs_allow_lds((const void *)k_small<R, PER>, sizeof(C2) << kSmallQubits))
        return e;
    hipLaunchKernelGGL((k_small<R, PER>), dim3(1), dim3(nt), (size_t)dim * sizeof(C2), st->stream, (C2 *)st->psi, dim,
                       prog, bytes, pool);
    return hipGetLastError();
}

template <class R> hipError_t launch_r(qs_state *st, const char *prog, uint32_t bytes, const char *pool)
{
    const uint32_t dim = 1u << st->n;
    // two amplitudes per thread as far as 1024 threads go (100 operations on 10 qubits: 35.5 us with 512 threads, 37.7
    // with 256)
    const int nt = (int)std::min<uint32_t>(1024, std::max<uint32_t>(64, dim / 2));
    switch ((dim + nt - 1) / nt) {
    case 1:
    case 2: return launch_per<R, 2>(st, dim, nt, prog, bytes, pool);
    case 4: return launch_per<R, 4>(st, dim, nt, prog, bytes, pool);
    default: return hipErrorInvalidValue;
    }
}
}  // namespace

int qs_small_run(qs_state *st, const SmallProgram &P)
{
    if (P.chunks.empty())
        return QS_OK;
    // the last chunk goes as far as what ends it (whole cache lines, as the kernel reads them)
    const size_t bytes = (P.chunks.size() - kChunk + P.used + kTail + 63) & ~(size_t)63;
    RingUse use;
    char *h = qs_ring_host(st, bytes + P.pool.size(), &use);
    if (!h)
        return QS_EDEVICE;
    std::memcpy(h, P.chunks.data(), bytes);
    if (!P.pool.empty())
        std::memcpy(h + bytes, P.pool.data(), P.pool.size());
    char *d = qs_ring_upload(st, h, bytes + P.pool.size(), use);
    if (!d)
        return QS_EDEVICE;
    QS_HIP(st->dtype == QS_C128 ? launch_r<double>(st, d, (uint32_t)bytes, d + bytes)
                                : launch_r<float>(st, d, (uint32_t)bytes, d + bytes));
    return QS_OK;
}
