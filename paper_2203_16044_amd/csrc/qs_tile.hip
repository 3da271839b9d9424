// Plain runs of circuits on states beyond one workgroup's LDS: consecutive operations in one pass over the state.
//
// Gate by gate, an operation streams the whole state through the compute units for a few operations per amplitude. Here
// the operations of a circuit are taken in order, and as many in a row as act on the qubits of one tile (4,096
// complex128 or 8,192 complex64 amplitudes: the lowest qubits, for whole 128-byte lines, and any others) go in one pass:
// every workgroup loads one tile into registers, 16 amplitudes per thread, applies the operations, and writes it back.
// Diagonals and controls may name any qubit: outside the tile their bits are the workgroup's.
//
// Within a pass the operations are grouped, in order, into stages of at most 4 target qubits, which the 16 amplitudes
// of a thread differ in; between stages the tile goes through LDS. The order of the operations is never changed and the
// arithmetic of each is that of the one-pass kernels, rounding for rounding (1-qubit gates the lane-exchange form takes
// there in its order, otherwise FMA chains in ascending column order), so results are the single calls' bit for bit.
//
// A pass is bound by HBM up to about 16 1-qubit gates (complex128, 26 qubits: 0.40 ms with 4, 0.43 with 16, 0.55 with
// 32; complex64, 27 qubits: 0.36, 0.54 and 0.98) and by the multiply-adds beyond: 4 waves a SIMD from different tiles
// keep loads and arithmetic going at once. On small states an operation costs its instructions and the branches to them
// (14 qubits: 0.4 us each). Circuits of U3, CZ, RZ and Toffoli layers, 3 layers: 28 qubits complex128 20.3 ms against
// 268 gate by gate, complex64 12.5 against 142; 20 qubits 177 us against 888; 14 qubits 86 us against 448.
//
// Operations with more than two targets to mix, and fused-swaps, stay calls of their own, as do runs whose operations
// together would cost less than a pass, and whole circuits whose passes save less than the copy of their records costs.
#include <algorithm>
#include <cstring>

#include "qs_internal.h"

namespace {

enum : uint32_t {
    OP_END,    // end of the pass
    OP_STAGE,  // the next stage's positions
    OP_DENSE1,
    OP_MOVE1,  // monomial 1-qubit gate
    OP_DENSE2,
    OP_MOVE2,
    OP_DIAG,   // diagonal on at most 2 qubits
    OP_DIAGK   // more targets
};
// Entry codes of diagonals: untouched, sign flip, multiply, multiply by i or -i as a move.
enum : uint32_t { D_ONE, D_NEG, D_MUL, D_I, D_MINUS_I };
// Diagonals: every entry multiplies / every entry is 1 or -1.
enum : uint32_t { F_ALL_MUL = 1, F_SIGNS = 2, F_LANE = 4, F_DIRECT = 8 };

constexpr int kW = 4, kM = 1 << kW;  // positions of a stage, amplitudes of a thread
constexpr uint32_t kOuter = 64, kReg = 128, kNone = 255;  // a bit of the index: tile position, outer qubit, register bit

struct Rec {
    uint32_t head;   // kind, length in 16-byte units << 8, form << 16, flags << 24
    uint32_t cloc;   // controls: tile positions
    uint32_t creg;   // controls: register bits
    uint32_t table;  // moves and diagonals on at most 2 targets: 4 bits per member (source and phase, or code)
    uint64_t cout;   // controls: outer qubits; a stage: its qubits, 8 bits each
    uint32_t pos;    // a stage: its tile positions, 8 bits each, ascending; a diagonal: its two bits, 8 bits each
    uint32_t k;      // diagonals on more qubits: targets
};
static_assert(sizeof(Rec) == 32, "program record");
constexpr size_t kTail = sizeof(Rec) + 64;     // what a pass's records end with: a record, read as if a matrix followed
constexpr size_t kPassBytes = 12288;           // of records: of a 16 KiB scalar cache
constexpr size_t kSlabBytes = (size_t)2 << 20; // of records uploaded at once: half the ring they go through

template <class R> struct TT;
template <> struct TT<double> {
    using C2 = double2;
    static constexpr int B = 12, LB = 3;  // tile bits, bits within a 128-byte line
};
template <> struct TT<float> {
    using C2 = float2;
    static constexpr int B = 13, LB = 4;
};

struct TileMap {  // tile position -> qubit, as runs: off(i) = sum over runs of (i & mask) << shift
    int nruns;
    uint32_t mask[TT<float>::B];
    int shift[TT<float>::B];
};

__device__ __forceinline__ double pick(bool c, double a, double b) { return c ? a : b; }
__device__ __forceinline__ float pick(bool c, float a, float b) { return c ? a : b; }
template <class C2> __device__ __forceinline__ C2 pick(bool c, const C2 &a, const C2 &b)  // by value: no address taken
{
    const auto ax = a.x, ay = a.y, bx = b.x, by = b.y;
    return C2{c ? ax : bx, c ? ay : by};
}

__device__ __forceinline__ double flip(double x, uint32_t sign)  // sign: 0 or 0x80000000
{
    return __hiloint2double(__double2hiint(x) ^ (int)sign, __double2loint(x));
}
__device__ __forceinline__ float flip(float x, uint32_t sign) { return __uint_as_float(__float_as_uint(x) ^ sign); }
template <class C2> __device__ __forceinline__ C2 turn(const C2 &x, uint32_t ph)  // i^ph x, exactly
{
    return C2{flip(pick(ph & 1u, x.y, x.x), (ph + 1u) << 30 & 0x80000000u),
              flip(pick(ph & 1u, x.x, x.y), ph << 30 & 0x80000000u)};
}

template <class C2, class R> __device__ __forceinline__ void mul_add(R &yr, R &yi, R ur, R ui, const C2 &x)
{
    yr = fma(ur, x.x, yr);
    yr = fma(-ui, x.y, yr);
    yi = fma(ur, x.y, yi);
    yi = fma(ui, x.x, yi);
}

// The addend of a final product lives on past it, so that the product is a three-operand instruction into the register
// of the amplitude it replaces: accumulated in place of the addend, all 16 amplitudes of an operation end up in a second
// set of registers and are moved back.
template <class R> __device__ __forceinline__ void outlive(const R &t) { asm volatile("" ::"v"(t)); }

// LANE: in the order of the lane-exchange kernel (own member's products last), else column by column.
template <bool LANE, class C2, class R> __device__ __forceinline__ void pair_gate(C2 &a, C2 &b, const R *u)
{
    C2 y{0, 0}, z{0, 0}, v, w;
    if constexpr (LANE) {
        y.x = fma(-u[1], a.y, fma(u[2], b.x, -u[3] * b.y));
        y.y = fma(u[1], a.x, fma(u[2], b.y, u[3] * b.x));
        z.x = fma(-u[7], b.y, fma(u[4], a.x, -u[5] * a.y));
        z.y = fma(u[7], b.x, fma(u[4], a.y, u[5] * a.x));
        v.x = fma(u[0], a.x, y.x);
        v.y = fma(u[0], a.y, y.y);
        w.x = fma(u[6], b.x, z.x);
        w.y = fma(u[6], b.y, z.y);
    } else {
        mul_add(y.x, y.y, u[0], u[1], a);
        mul_add(z.x, z.y, u[4], u[5], a);
        y.x = fma(u[2], b.x, y.x);
        y.y = fma(u[2], b.y, y.y);
        z.x = fma(u[6], b.x, z.x);
        z.y = fma(u[6], b.y, z.y);
        v.x = fma(-u[3], b.y, y.x);
        v.y = fma(u[3], b.x, y.y);
        w.x = fma(-u[7], b.y, z.x);
        w.y = fma(u[7], b.x, z.y);
    }
    outlive(y.x);
    outlive(y.y);
    outlive(z.x);
    outlive(z.y);
    a = v;
    b = w;
}

// The program is read through the scalar cache (constant address space).
typedef const __attribute__((address_space(4))) uint32_t *cwords;
typedef uint32_t words8 __attribute__((ext_vector_type(8), aligned(4)));
typedef uint32_t words16 __attribute__((ext_vector_type(16), aligned(4)));
__device__ __forceinline__ words8 fetch(cwords w) { return *(const __attribute__((address_space(4))) words8 *)w; }
__device__ __forceinline__ words16 fetch16(cwords w) { return *(const __attribute__((address_space(4))) words16 *)w; }
__device__ __forceinline__ void reals8(const words16 &m, double *u)
{
#pragma unroll
    for (int e = 0; e < 8; ++e)
        u[e] = __builtin_bit_cast(double, (uint64_t)m[2 * e] | (uint64_t)m[2 * e + 1] << 32);
}
__device__ __forceinline__ void reals8(const words16 &m, float *u)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
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

__device__ __forceinline__ uint32_t insert0(uint32_t g, uint32_t p)
{
    const uint32_t lo = g & ((1u << p) - 1u);
    return ((g ^ lo) << 1) | lo;
}
// The LDS slot (8 bytes) of tile index i: the higher bits folded onto those within the banks (linear over xor).
__device__ __forceinline__ uint32_t slot(uint32_t i) { return i ^ ((i >> 5) & 31u) ^ ((i >> 10) & 31u); }
__device__ __forceinline__ uint64_t spread(uint32_t i, const TileMap &map)
{
    uint64_t off = 0;
    for (int r = 0; r < map.nruns; ++r)
        off |= (uint64_t)(i & map.mask[r]) << map.shift[r];
    return off;
}

// A bit of the index for a thread (not a register bit).
__device__ __forceinline__ uint32_t index_bit(uint32_t what, uint32_t i0, uint64_t base)
{
    if (what < kOuter)
        return (i0 >> what) & 1u;
    return what < kReg ? (uint32_t)(base >> (what - kOuter)) & 1u : 0u;
}

// A value that the compiler neither computes ahead nor shares between cases: one at a time in registers.
template <class C2> __device__ __forceinline__ void pin(C2 &z) { asm volatile("" : "+v"(z.x), "+v"(z.y)); }

// Members (r, r | 1 << J) of a thread's amplitudes.
template <int J, bool LANE, class C2, class R>
__device__ __forceinline__ void dense1(C2 (&x)[kM], const R *u)
{
#pragma unroll
    for (int r = 0; r < kM; ++r)
        if (!((r >> J) & 1)) {
            pair_gate<LANE>(x[r], x[r | 1 << J], u);
            pin(x[r]);
            pin(x[r | 1 << J]);
        }
}
template <int J, class C2, class R>
__device__ __forceinline__ void dense1_ctrl(C2 (&x)[kM], const R *u, bool on, uint32_t creg)
{
#pragma unroll
    for (int r = 0; r < kM; ++r)
        if (!((r >> J) & 1) && (r & creg) == creg) {
            C2 a = x[r], b = x[r | 1 << J];
            pair_gate<false>(a, b, u);
            x[r] = pick(on, a, x[r]);
            x[r | 1 << J] = pick(on, b, x[r | 1 << J]);
            pin(x[r]);
            pin(x[r | 1 << J]);
        }
}
// JC: a control on register bit JC (-1: none), with or without others on lanes
template <int J, int JC, class C2> __device__ __forceinline__ void exchange(C2 (&x)[kM], bool on)
{
#pragma unroll
    for (int r = 0; r < kM; ++r)
        if (!((r >> J) & 1) && (JC < 0 || ((r >> (JC & 3)) & 1))) {
            const C2 a = x[r], b = x[r | 1 << J];
            x[r] = pick(on, b, a);
            x[r | 1 << J] = pick(on, a, b);
            pin(x[r]);
            pin(x[r | 1 << J]);
        }
}
template <int J, class C2>
__device__ __forceinline__ void move1(C2 (&x)[kM], uint32_t table, bool on, uint32_t creg)
{
    if ((table & 0xccu) == 0) {  // no phases
        if (creg == 0)
            return exchange<J, -1>(x, on);
        if (J != 0 && creg == 1u)
            return exchange<J, 0>(x, on);
        if (J != 1 && creg == 2u)
            return exchange<J, 1>(x, on);
        if (J != 2 && creg == 4u)
            return exchange<J, 2>(x, on);
        if (J != 3 && creg == 8u)
            return exchange<J, 3>(x, on);
    }
    const bool ex = table & 1u;
#pragma unroll
    for (int r = 0; r < kM; ++r)
        if (!((r >> J) & 1)) {
            const bool go = on & ((r & creg) == creg);
            C2 a = x[r], b = x[r | 1 << J];
            pin(a);
            pin(b);
            x[r] = pick(go, turn(pick(ex, b, a), (table >> 2) & 3u), a);
            x[r | 1 << J] = pick(go, turn(pick(ex, a, b), (table >> 6) & 3u), b);
        }
}
// Group by group, row by row: a row of the matrix is all that scalar registers hold at a time.
template <int J0, int J1, class R, class C2>
__device__ __forceinline__ void dense2(C2 (&x)[kM], cwords mat, bool on, uint32_t creg)
{
    constexpr int O[4] = {0, 1 << J0, 1 << J1, 1 << J0 | 1 << J1};
#pragma unroll
    for (int r = 0; r < kM; ++r)
        if (!(r & O[3])) {
            const bool go = on & ((r & creg) == creg);
            C2 y[4];
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                R m[8];
                reals_at<R, 8>(mat + a * (8 * sizeof(R) / 4), m);
                y[a] = C2{0, 0};
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    mul_add(y[a].x, y[a].y, m[2 * b], m[2 * b + 1], x[r | O[b]]);
            }
#pragma unroll
            for (int a = 0; a < 4; ++a)
                x[r | O[a]] = pick(go, y[a], x[r | O[a]]);
#pragma unroll
            for (int a = 0; a < 4; ++a)
                pin(x[r | O[a]]);
        }
}
template <int J0, int J1, class C2>
__device__ __forceinline__ void move2(C2 (&x)[kM], uint32_t table, bool on, uint32_t creg)
{
#pragma unroll
    for (int r = 0; r < kM; ++r)
        if (!((r >> J0) & 1) && !((r >> J1) & 1)) {
            const bool go = on & ((r & creg) == creg);
            const int e[4] = {r, r | 1 << J0, r | 1 << J1, r | 1 << J0 | 1 << J1};
            C2 y[4];
#pragma unroll
            for (int a = 0; a < 4; ++a)
                pin(x[e[a]]);
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const uint32_t src = (table >> (4 * a)) & 3u;
                y[a] = turn(pick(src & 2u, pick(src & 1u, x[e[3]], x[e[2]]), pick(src & 1u, x[e[1]], x[e[0]])),
                            (table >> (4 * a + 2)) & 3u);
            }
#pragma unroll
            for (int a = 0; a < 4; ++a)
                x[e[a]] = pick(go, y[a], x[e[a]]);
        }
}

template <class C2, class R> __device__ __forceinline__ void times(C2 &x, R dr, R di)
{
    const R t0 = -di * x.y, t1 = di * x.x;
    x.x = fma(dr, x.x, t0);
    x.y = fma(dr, x.y, t1);
    outlive(t0);
    outlive(t1);
}
template <class C2, class R> __device__ __forceinline__ void entry(C2 &x, R dr, R di, uint32_t code)
{
    C2 y = x;
    times(y, dr, di);
    x = pick(code == D_MUL, y, turn(x, (0x31020u >> (4 * code)) & 3u));  // i^0, i^2, -, i^1, i^3
}
// Member bits of amplitude r: J0 >= 0, register bit J0 is index bit 0 (otherwise the thread's b0), J1 likewise.
template <int J0, int J1, class C2, class R>
__device__ __forceinline__ void diag(C2 (&x)[kM], const R *m, uint32_t table, uint32_t flags, uint32_t b0, uint32_t b1)
{
    // the entries that differ over the thread's amplitudes, selected once per thread
    constexpr int N0 = J0 >= 0 ? 2 : 1, N1 = J1 >= 0 ? 2 : 1;
    R dr[4], di[4];
    uint32_t code[4];
#pragma unroll
    for (int v1 = 0; v1 < N1; ++v1)
#pragma unroll
        for (int v0 = 0; v0 < N0; ++v0) {
            const uint32_t s0 = J0 >= 0 ? v0 : b0, s1 = J1 >= 0 ? v1 : b1;
            dr[v0 + 2 * v1] = pick(s1, pick(s0, m[6], m[4]), pick(s0, m[2], m[0]));
            di[v0 + 2 * v1] = pick(s1, pick(s0, m[7], m[5]), pick(s0, m[3], m[1]));
            code[v0 + 2 * v1] = (table >> (4 * (s0 | s1 << 1))) & 15u;
        }
    if (flags & F_ALL_MUL) {
#pragma unroll
        for (int r = 0; r < kM; ++r) {
            const int a = (J0 >= 0 ? (r >> (J0 & 3)) & 1 : 0) | (J1 >= 0 ? ((r >> (J1 & 3)) & 1) << 1 : 0);
            times(x[r], dr[a], di[a]);
            pin(x[r]);
        }
    } else if (flags & F_SIGNS) {
#pragma unroll
        for (int r = 0; r < kM; ++r) {
            const int a = (J0 >= 0 ? (r >> (J0 & 3)) & 1 : 0) | (J1 >= 0 ? ((r >> (J1 & 3)) & 1) << 1 : 0);
            x[r] = C2{flip(x[r].x, code[a] << 31), flip(x[r].y, code[a] << 31)};  // D_NEG = 1
            pin(x[r]);
        }
    } else {
#pragma unroll
        for (int r = 0; r < kM; ++r) {
            const int a = (J0 >= 0 ? (r >> (J0 & 3)) & 1 : 0) | (J1 >= 0 ? ((r >> (J1 & 3)) & 1) << 1 : 0);
            entry(x[r], dr[a], di[a], code[a]);
            pin(x[r]);
        }
    }
}

// One pass: tile blockIdx.x. outer inserts the tile's qubits into the tile number.
template <class R, bool NT>
__global__ __launch_bounds__(1 << (TT<R>::B - kW)) void k_tile(typename TT<R>::C2 *__restrict__ psi, InsBits outer,
                                                             TileMap map, const char *__restrict__ prog,
                                                             uint32_t bytes)
{
    using C2 = typename TT<R>::C2;
    constexpr uint32_t T = 1u << (TT<R>::B - kW);
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t tid = threadIdx.x;
    const uint64_t base = qs_ins0(NT ? xcd_runs(blockIdx.x, gridDim.x) : blockIdx.x, outer);
    C2 *const p = psi + base;
    cwords w = (cwords)prog;
    C2 x[kM];
    uint32_t i0;          // the thread's tile index, register bits 0
    uint32_t at, qubits;  // the stage's positions and their qubits, 8 bits each
    uint32_t flags;
    words8 f = fetch(w);
    auto begin = [&](const words8 &g) {
        at = g[6];
        qubits = g[4];
        flags = g[0] >> 24;
        i0 = tid;
#pragma unroll
        for (int j = 0; j < kW; ++j)
            i0 = insert0(i0, (at >> (8 * j)) & 255u);
    };
    auto slot_at = [&](uint32_t where, uint32_t s0, int r) {
#pragma unroll
        for (int j = 0; j < kW; ++j)
            if ((r >> j) & 1)
                s0 ^= slot(1u << ((where >> (8 * j)) & 255u));
        return s0;
    };
    auto off_of = [&](int r) {
        uint64_t o = 0;
#pragma unroll
        for (int j = 0; j < kW; ++j)
            if ((r >> j) & 1)
                o |= (uint64_t)1 << ((qubits >> (8 * j)) & 255u);
        return o;
    };
    auto get = [&](uint64_t off) {
        typedef typename NT2<R>::type V;
        const V *a = reinterpret_cast<const V *>(p + off);
        const V v = NT ? __builtin_nontemporal_load(a) : *a;
        return C2{v.x, v.y};
    };
    auto put = [&](uint64_t off, const C2 &z) {
        typedef typename NT2<R>::type V;
        V *a = reinterpret_cast<V *>(p + off);
        V v = {z.x, z.y};
        if constexpr (NT)
            __builtin_nontemporal_store(v, a);
        else
            *a = v;
    };
    // The amplitudes from the slots `from` to the slots `to` of other threads. The first were the thread's own.
    auto through_lds = [&](auto from, auto to) {
        if constexpr (sizeof(R) == 8) {
            R *s = reinterpret_cast<R *>(smem);
#pragma unroll
            for (int r = 0; r < kM; ++r)
                s[from(r)] = x[r].x;
            lds_barrier();
#pragma unroll
            for (int r = 0; r < kM; ++r)
                x[r].x = s[to(r)];
            lds_barrier();
#pragma unroll
            for (int r = 0; r < kM; ++r)
                s[from(r)] = x[r].y;
            lds_barrier();
#pragma unroll
            for (int r = 0; r < kM; ++r)
                x[r].y = s[to(r)];
        } else {
            C2 *s = reinterpret_cast<C2 *>(smem);
#pragma unroll
            for (int r = 0; r < kM; ++r)
                s[from(r)] = x[r];
            lds_barrier();
#pragma unroll
            for (int r = 0; r < kM; ++r)
                x[r] = s[to(r)];
        }
    };
    const uint32_t line = slot(tid);
    auto in_lines = [&](int r) { return line ^ slot((uint32_t)r * T); };
    begin(f);
    if (flags & F_DIRECT) {  // whole lines over the lanes
        const uint64_t t0 = spread(i0, map);
#pragma unroll
        for (int r = 0; r < kM; ++r)
            x[r] = get(t0 | off_of(r));
        warm(w, (bytes + 63) / 64, __builtin_amdgcn_readfirstlane(tid >> 6), T / 64);
    } else {
        const uint64_t t0 = spread(tid, map);
#pragma unroll
        for (int r = 0; r < kM; ++r)
            x[r] = get(t0 | spread(r * T, map));
        warm(w, (bytes + 63) / 64, __builtin_amdgcn_readfirstlane(tid >> 6), T / 64);
        const uint32_t s0 = slot(i0);
        through_lds(in_lines, [&](int r) { return slot_at(at, s0, r); });
    }
    w += (f[0] >> 8 & 255u) * 4;
    f = fetch(w);
    while ((f[0] & 255u) != OP_END) {
        const uint32_t head = f[0], kind = head & 255u, form = head >> 16 & 255u, fl = head >> 24;
        const uint32_t cloc = f[1], creg = f[2], table = f[3];
        const uint64_t cout = (uint64_t)f[4] | (uint64_t)f[5] << 32;
        const words8 g = f;
        cwords mat = w + 8;
        const words16 gm = fetch16(mat);
        w += (head >> 8 & 255u) * 4;
        f = fetch(w);  // one operation ahead (the program ends with slack for it)
        if (kind == OP_STAGE) {
            const uint32_t s0 = slot(i0), at0 = at;
            begin(g);
            const uint32_t s1 = slot(i0);
            through_lds([&](int r) { return slot_at(at0, s0, r); }, [&](int r) { return slot_at(at, s1, r); });
            continue;
        }
        if (kind < OP_DIAG) {
            if ((base & cout) != cout)
                continue;
            const bool on = (i0 & cloc) == cloc;
            if (kind == OP_DENSE1) {
                R u[8];
                reals8(gm, u);
                if (!(cloc | creg)) {
                    if (fl & F_LANE) {
                        switch (form) {
                        case 0: dense1<0, true>(x, u); break;
                        case 1: dense1<1, true>(x, u); break;
                        case 2: dense1<2, true>(x, u); break;
                        default: dense1<3, true>(x, u); break;
                        }
                    } else {
                        switch (form) {
                        case 0: dense1<0, false>(x, u); break;
                        case 1: dense1<1, false>(x, u); break;
                        case 2: dense1<2, false>(x, u); break;
                        default: dense1<3, false>(x, u); break;
                        }
                    }
                } else if (__ballot(on)) {
                    switch (form) {
                    case 0: dense1_ctrl<0>(x, u, on, creg); break;
                    case 1: dense1_ctrl<1>(x, u, on, creg); break;
                    case 2: dense1_ctrl<2>(x, u, on, creg); break;
                    default: dense1_ctrl<3>(x, u, on, creg); break;
                    }
                }
            } else if (!__ballot(on)) {
            } else if (kind == OP_MOVE1) {
                switch (form) {
                case 0: move1<0>(x, table, on, creg); break;
                case 1: move1<1>(x, table, on, creg); break;
                case 2: move1<2>(x, table, on, creg); break;
                default: move1<3>(x, table, on, creg); break;
                }
            } else if (kind == OP_DENSE2) {
                switch (form) {
                case 0: dense2<0, 1, R>(x, mat, on, creg); break;
                case 1: dense2<0, 2, R>(x, mat, on, creg); break;
                case 2: dense2<0, 3, R>(x, mat, on, creg); break;
                case 3: dense2<1, 2, R>(x, mat, on, creg); break;
                case 4: dense2<1, 3, R>(x, mat, on, creg); break;
                default: dense2<2, 3, R>(x, mat, on, creg); break;
                }
            } else {
                switch (form) {
                case 0: move2<0, 1>(x, table, on, creg); break;
                case 1: move2<0, 2>(x, table, on, creg); break;
                case 2: move2<0, 3>(x, table, on, creg); break;
                case 3: move2<1, 2>(x, table, on, creg); break;
                case 4: move2<1, 3>(x, table, on, creg); break;
                default: move2<2, 3>(x, table, on, creg); break;
                }
            }
        } else if (kind == OP_DIAG) {
            // the host has put a register bit first, and two of them in ascending order
            const uint32_t b0 = index_bit(g[6] & 255u, i0, base), b1 = index_bit(g[6] >> 8 & 255u, i0, base);
            R m[8];
            reals8(gm, m);
            switch (form) {
            case 0: diag<-1, -1>(x, m, table, fl, b0, b1); break;
            case 1: diag<0, -1>(x, m, table, fl, b0, b1); break;
            case 2: diag<1, -1>(x, m, table, fl, b0, b1); break;
            case 3: diag<2, -1>(x, m, table, fl, b0, b1); break;
            case 4: diag<3, -1>(x, m, table, fl, b0, b1); break;
            case 5: diag<0, 1>(x, m, table, fl, b0, b1); break;
            case 6: diag<0, 2>(x, m, table, fl, b0, b1); break;
            case 7: diag<0, 3>(x, m, table, fl, b0, b1); break;
            case 8: diag<1, 2>(x, m, table, fl, b0, b1); break;
            case 9: diag<1, 3>(x, m, table, fl, b0, b1); break;
            default: diag<2, 3>(x, m, table, fl, b0, b1); break;
            }
        } else {
            // behind the record: the k bits' places (a word each), the entries, their codes (a byte each)
            const uint32_t k = g[7];
            uint32_t a0 = 0, c[kW] = {0, 0, 0, 0};
            for (uint32_t j = 0; j < k; ++j) {
                const uint32_t what = mat[j];
                if (what >= kReg) {
#pragma unroll
                    for (int q = 0; q < kW; ++q)
                        c[q] |= what == kReg + q ? 1u << j : 0u;
                } else {
                    a0 |= index_bit(what, i0, base) << j;
                }
            }
            const R *d = reinterpret_cast<const R *>((const uint32_t *)(mat + 16));
            const uint8_t *codes = reinterpret_cast<const uint8_t *>(d + ((size_t)2 << k));
#pragma unroll
            for (int r = 0; r < kM; ++r) {
                const uint32_t a = a0 | (r & 1 ? c[0] : 0u) | (r & 2 ? c[1] : 0u) | (r & 4 ? c[2] : 0u) |
                                   (r & 8 ? c[3] : 0u);
                entry(x[r], d[2 * a], d[2 * a + 1], codes[a]);
                if (r % 4 == 3)
                    __builtin_amdgcn_sched_barrier(0);  // not all the loads at once: registers
                pin(x[r]);
            }
        }
    }
    if (flags & F_DIRECT) {
        const uint64_t t0 = spread(i0, map);
#pragma unroll
        for (int r = 0; r < kM; ++r)
            put(t0 | off_of(r), x[r]);
    } else {
        const uint32_t s0 = slot(i0);
        through_lds([&](int r) { return slot_at(at, s0, r); }, in_lines);
        const uint64_t t0 = spread(tid, map);
#pragma unroll
        for (int r = 0; r < kM; ++r)
            put(t0 | spread(r * T, map), x[r]);
    }
}

// ---------------------------------------------------------------------------------------------------------
// forming the program
// ---------------------------------------------------------------------------------------------------------
int tile_bits(int dtype) { return dtype == QS_C128 ? TT<double>::B : TT<float>::B; }
int line_bits(int dtype) { return dtype == QS_C128 ? TT<double>::LB : TT<float>::LB; }
size_t real_bytes(int dtype) { return amp_bytes(dtype) / 2; }

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

size_t inline_bytes(const TileOp &o, int dtype)
{
    if (o.kind != OP_DIAGK)
        return o.m.size() * real_bytes(dtype);
    return 64 + o.m.size() * real_bytes(dtype) + o.code.size();
}
size_t units_of(const TileOp &o, int dtype) { return 2 + (inline_bytes(o, dtype) + 15) / 16; }

// Microseconds of an operation as a call of its own: its launch or the share of the lines it reads and rewrites, whichever
// takes longer (dense 2-qubit gates one after the other).
double call_us(const TileProgram &P, const TileOp &o)
{
    const double lines = 2e-6 * o.share * (double)(((uint64_t)1 << P.n) * amp_bytes(P.dtype)) / 6.4;
    if (o.kind == OP_DENSE2)
        return 3.0 + lines;
    return std::max(3.0, 1.0 + lines);
}
// ... and of a pass over the whole state with these operations' arithmetic.
double pass_us(const TileProgram &P, const std::vector<TileOp> &ops)
{
    const double amps = (double)((uint64_t)1 << P.n), bytes = amps * amp_bytes(P.dtype);
    double us = 6.0 + 2e-6 * bytes / (qs_streams((uint64_t)bytes) ? 5.5 : 8.0);
    for (const TileOp &o : ops)
        us += (o.kind == OP_DENSE2 ? 1.2 : 0.4) +
              amps * (o.kind == OP_DENSE2 ? 16 : o.kind == OP_DENSE1 ? 8 : o.kind == OP_DIAGK ? 24 : 4) / 2.2e7;
    return us;
}
// The copy of the records in front of the first pass, once a run: what all passes together have to save. Microseconds of
// a run as passes and as calls, and, waited for, on 16 qubits complex128: 5 U3 gates 14.6 (25.2) and 13.7 (23.6), 6 14.6
// (25.5) and 16.3 (25.9); dense 2-qubit gates 5 17.3 (27.3) and 15.6 (26.9), 8 22.1 (32.9) and 24.4 (49.5). On 20: 3 U3
// gates 19.1 and 15.2, 4 20.1 and 21.8.
constexpr double kUploadUs = 7.0;

void flush(TileProgram &P)
{
    std::vector<TileOp> ops;
    ops.swap(P.open);
    uint64_t L = P.open_qubits;
    P.open_qubits = 0;
    P.open_bytes = 0;
    if (ops.empty())
        return;
    double calls = 0;
    for (const TileOp &o : ops)
        calls += call_us(P, o);
    const double saved = calls - pass_us(P, ops);
    if (saved <= 0) {
        for (const TileOp &o : ops)
            P.steps.push_back(TileStep{o.raw, 0, 0, 0});
        return;
    }
    P.saved_us += saved;
    const int B = tile_bits(P.dtype), LB = line_bits(P.dtype);
    for (int q = 0; __builtin_popcountll(L) < B; ++q)
        L |= (uint64_t)1 << q;
    int local[64];
    int qubit[16], nb = 0;
    for (int q = 0; q < 64; ++q) {
        local[q] = -1;
        if ((L >> q) & 1) {
            local[q] = nb;
            qubit[nb++] = q;
        }
    }
    // stages: operations in order, at most kW positions to mix
    std::vector<uint32_t> masks;
    std::vector<size_t> first;
    for (size_t i = 0; i < ops.size(); ++i) {
        uint32_t need = 0;
        for (int j = 0; j < ops[i].nt; ++j)
            need |= 1u << local[ops[i].t[j]];
        if (masks.empty() || __builtin_popcount(masks.back() | need) > kW) {
            masks.push_back(0);
            first.push_back(i);
        }
        masks.back() |= need;
    }
    const size_t at = P.prog.size();
    auto emit = [&](const Rec &r, size_t extra) {
        const size_t o = P.prog.size();
        P.prog.resize(o + 16 * (2 + (extra + 15) / 16), 0);
        std::memcpy(&P.prog[o], &r, sizeof r);
        return &P.prog[o + sizeof r];
    };
    size_t stage = 0;
    int reg[64];  // qubit -> register bit of the present stage
    uint64_t regs = 0;
    for (size_t i = 0; i < ops.size(); ++i) {
        if (stage < first.size() && first[stage] == i) {
            uint32_t m = masks[stage++];
            for (int j = B - 1; __builtin_popcount(m) < kW; --j)  // fill up with the highest: whole lines over the lanes
                m |= 1u << j;
            Rec r{};
            r.head = OP_STAGE | 2u << 8 | (m & ((1u << LB) - 1u) ? 0u : F_DIRECT << 24);
            regs = 0;
            int nr = 0;
            for (int j = 0; j < B; ++j)
                if ((m >> j) & 1) {
                    r.pos |= (uint32_t)j << (8 * nr);
                    r.cout |= (uint64_t)qubit[j] << (8 * nr);
                    regs |= (uint64_t)1 << qubit[j];
                    reg[qubit[j]] = nr++;
                }
            emit(r, 0);
        }
        const TileOp &o = ops[i];
        Rec r{};
        for (int q = 0; q < P.n; ++q)
            if ((o.cmask >> q) & 1) {
                if ((regs >> q) & 1)
                    r.creg |= 1u << reg[q];
                else if (local[q] >= 0)
                    r.cloc |= 1u << local[q];
                else
                    r.cout |= (uint64_t)1 << q;
            }
        auto place = [&](int q) -> uint32_t {
            return (regs >> q) & 1 ? kReg + reg[q] : local[q] >= 0 ? (uint32_t)local[q] : kOuter + q;
        };
        static const int pair[4][4] = {{0, 0, 1, 2}, {0, 0, 3, 4}, {0, 0, 0, 5}, {0, 0, 0, 0}};
        uint32_t form = 0, flags = o.flags;
        r.table = o.table;
        std::vector<double> m = o.m;
        if (o.kind == OP_DENSE1 || o.kind == OP_MOVE1) {
            form = reg[o.t[0]];
        } else if (o.kind == OP_DENSE2 || o.kind == OP_MOVE2) {
            form = pair[reg[o.t[0]]][reg[o.t[1]]];  // targets ascending, so register bits too
        } else if (o.kind == OP_DIAG) {
            uint32_t w0 = place(o.d[0]), w1 = o.k == 2 ? place(o.d[1]) : kNone;
            // a register bit first, two of them ascending
            if (o.k == 2 && w1 >= kReg && (w0 < kReg || w1 < w0)) {
                std::swap(w0, w1);
                std::swap(m[2], m[4]);
                std::swap(m[3], m[5]);
                r.table = (o.table & 0xf00fu) | (o.table & 0xf0u) << 4 | (o.table & 0xf00u) >> 4;
            }
            const bool r0 = w0 >= kReg && w0 != kNone, r1 = w1 >= kReg && w1 != kNone;
            if (r0 && r1) {
                form = 5 + pair[w0 - kReg][w1 - kReg];
            } else if (r0) {
                form = 1 + (w0 - kReg);
            }
            r.pos = w0 | w1 << 8;
        } else {
            r.k = (uint32_t)o.k;
        }
        const size_t extra = inline_bytes(o, P.dtype);
        r.head = o.kind | (uint32_t)units_of(o, P.dtype) << 8 | form << 16 | flags << 24;
        char *to = emit(r, extra);
        if (o.kind == OP_DIAGK) {
            for (int j = 0; j < o.k; ++j) {
                const uint32_t what = place(o.d[j]);
                std::memcpy(to + 4 * j, &what, 4);
            }
            put_reals(to + 64, m.data(), m.size(), P.dtype);
            std::memcpy(to + 64 + m.size() * real_bytes(P.dtype), o.code.data(), o.code.size());
        } else if (!m.empty()) {
            put_reals(to, m.data(), m.size(), P.dtype);
        }
    }
    emit(Rec{}, kTail - sizeof(Rec));  // OP_END
    while (P.prog.size() % 64)
        P.prog.resize(P.prog.size() + 16, 0);
    P.steps.push_back(TileStep{-1, L, at, P.prog.size() - at});
}

void add(TileProgram &P, TileOp &&o)
{
    uint64_t need = 0;
    for (int j = 0; j < o.nt; ++j)
        need |= (uint64_t)1 << o.t[j];
    const int B = tile_bits(P.dtype);
    const uint64_t low = ((uint64_t)1 << line_bits(P.dtype)) - 1;
    const size_t bytes = 16 * (units_of(o, P.dtype) + 2);  // with a stage of its own
    if (__builtin_popcountll(P.open_qubits | low | need) > B || P.open_bytes + bytes + kTail + 64 > kPassBytes)
        flush(P);
    P.open_qubits |= low | need;
    P.open_bytes += bytes;
    P.open.push_back(std::move(o));
}

// The share of a state's 128-byte lines in which index bits `fixed` (one value each) hold for some amplitude.
double share_of(const TileProgram &P, uint64_t fixed)
{
    return 1.0 / (double)((uint64_t)1 << __builtin_popcountll(fixed >> line_bits(P.dtype)));
}

void add_diag(TileProgram &P, int raw, const int *t, int k, const double *d)
{
    const int D = 1 << k;
    TileOp o;
    o.raw = raw;
    o.code.resize(D);
    int m = 0;
    bool phases = true, muls = true, signs = true;
    for (int a = 0; a < D; ++a) {
        const double re = d[2 * a], im = d[2 * a + 1];
        o.code[a] = re == 1.0 && im == 0.0 ? D_ONE : re == -1.0 && im == 0.0 ? D_NEG : D_MUL;
        m += o.code[a] != D_ONE;
        phases = phases && (o.code[a] != D_MUL || (re == 0.0 && (im == 1.0 || im == -1.0)));
        muls = muls && o.code[a] == D_MUL;
        signs = signs && o.code[a] != D_MUL;
    }
    if (m == 0)
        return;
    if (phases && m < D && k <= QS_MAX_K)  // as in qs_apply_diag: i and -i are moves where every entry is a phase
        for (int a = 0; a < D; ++a)
            if (o.code[a] == D_MUL)
                o.code[a] = d[2 * a + 1] == 1.0 ? D_I : D_MINUS_I;
    uint64_t tm = 0;
    for (int j = 0; j < k; ++j) {
        tm |= (uint64_t)1 << t[j];
        o.d[j] = t[j];
    }
    o.k = k;
    o.share = std::min(1.0, m * share_of(P, tm));
    o.m.assign(d, d + 2 * D);
    if (k <= 2) {
        o.kind = OP_DIAG;
        o.flags = muls ? F_ALL_MUL : signs ? F_SIGNS : 0;
        for (int a = 0; a < 4; ++a)
            o.table |= (uint32_t)o.code[k == 1 ? a & 1 : a] << (4 * a);
        o.m.resize(8, 0.0);
        if (k == 1)
            for (int e = 0; e < 4; ++e)
                o.m[4 + e] = o.m[e];
        o.code.clear();
    } else {
        o.kind = OP_DIAGK;
    }
    add(P, std::move(o));
}

}  // namespace

bool qs_tile_fits(int n, int dtype) { return n >= tile_bits(dtype); }

void qs_tile_add_call(TileProgram &P, int raw)
{
    flush(P);
    P.steps.push_back(TileStep{raw, 0, 0, 0});
}

void qs_tile_add_diag(TileProgram &P, int raw, const int *t, int k, const double *d)
{
    if (k > 6) {  // the records are to fit the scalar cache
        qs_tile_add_call(P, raw);
        return;
    }
    add_diag(P, raw, t, k, d);
}

void qs_tile_add_matrix(TileProgram &P, int raw, const int *t, int k, const int *c, int nc, const double *U)
{
    const int D = 1 << k;
    if (nc == 0 && qs_is_diagonal(U, k)) {
        std::vector<double> d((size_t)2 * D);
        for (int a = 0; a < D; ++a) {
            d[2 * a] = U[2 * (a * D + a)];
            d[2 * a + 1] = U[2 * (a * D + a) + 1];
        }
        add_diag(P, raw, t, k, d.data());
        return;
    }
    if (k > 2) {
        qs_tile_add_call(P, raw);
        return;
    }
    TPos tp{};
    int perm[QS_MAX_DIAG_K];
    qs_sort_targets(t, k, tp, perm);
    std::vector<double> Us;
    qs_permute_matrix(U, k, perm, Us);
    TileOp o;
    o.raw = raw;
    o.nt = o.k = k;
    for (int j = 0; j < k; ++j)
        o.t[j] = tp.tpos[j];
    for (int j = 0; j < nc; ++j)
        o.cmask |= (uint64_t)1 << c[j];
    o.share = share_of(P, o.cmask);
    PermTable pt;
    if (qs_monomial_table(Us, k, pt)) {
        if (!pt.moving)
            return;  // identity
        for (int a = 0; a < D; ++a)
            o.table |= (uint32_t)(pt.src[a] | pt.phase[a] << 2) << (4 * a);
        o.kind = k == 1 ? OP_MOVE1 : OP_MOVE2;
    } else {
        o.kind = k == 1 ? OP_DENSE1 : OP_DENSE2;
        if (k == 1 && nc == 0 && qs_dense1_in_lanes(P.dtype, P.n, o.t[0]))
            o.flags = F_LANE;
        o.m = std::move(Us);
    }
    add(P, std::move(o));
}

void qs_tile_finish(TileProgram &P)
{
    flush(P);
    for (const TileStep &s : P.steps)
        P.calls += s.raw >= 0;
    if (P.saved_us <= kUploadUs) {
        P.steps.clear();
        P.prog.clear();
    }
}

namespace {
template <class R> hipError_t launch_tile(qs_state *st, const TileStep &step, const char *prog)
{
    using C2 = typename TT<R>::C2;
    constexpr int B = TT<R>::B;
    TileMap map{};
    for (int q = 0, j = 0; j < B; ++q) {
        if (!((step.qubits >> q) & 1))
            continue;
        if (!map.nruns || map.shift[map.nruns - 1] != q - j) {
            map.shift[map.nruns] = q - j;
            map.mask[map.nruns++] = 0;
        }
        map.mask[map.nruns - 1] |= 1u << j;
        ++j;
    }
    const InsBits outer = qs_make_ins(step.qubits, 0);
    const size_t lds = (size_t)8 << B;
    const dim3 grid((unsigned)((uint64_t)1 << (st->n - B))), block(1u << (B - kW));
    const uint32_t bytes = (uint32_t)step.bytes;
    auto go = [&](auto kernel) {
        if (hipError_t e = qs_allow_lds((const void *)kernel, lds))
            return e;
        hipLaunchKernelGGL(kernel, grid, block, lds, st->stream, (C2 *)st->psi, outer, map, prog, bytes);
        return hipGetLastError();
    };
    return qs_streams(((uint64_t)1 << st->n) * sizeof(C2)) ? go(k_tile<R, true>) : go(k_tile<R, false>);
}
}  // namespace

// Upload the records of as many passes from step `i` on as make a slab; `end` receives the first step beyond.
int qs_tile_upload(qs_state *st, const TileProgram &P, size_t i, size_t *end, const char **dev)
{
    size_t total = 0, lo = 0, hi = 0;
    size_t j = i;
    for (; j < P.steps.size(); ++j) {
        const TileStep &s = P.steps[j];
        const size_t more = s.raw < 0 ? s.bytes : 0;
        if (total && total + more > kSlabBytes)
            break;
        total += more;
        if (s.raw < 0) {
            if (!hi)
                lo = s.at;
            hi = s.at + s.bytes;
        }
    }
    *end = j;
    if (!hi)
        return QS_OK;
    RingUse use;
    char *h = qs_ring_host(st, hi - lo, &use);
    if (!h)
        return QS_EDEVICE;
    std::memcpy(h, P.prog.data() + lo, hi - lo);
    const char *d = qs_ring_upload(st, h, hi - lo, use);
    if (!d)
        return QS_EDEVICE;
    *dev = d - lo;
    return QS_OK;
}

int qs_tile_pass(qs_state *st, const TileStep &step, const char *dev)
{
    QS_HIP(st->dtype == QS_C128 ? launch_tile<double>(st, step, dev + step.at)
                                : launch_tile<float>(st, step, dev + step.at));
    return QS_OK;
}
