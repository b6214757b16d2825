// A run of gates in one pass over the state. A workgroup holds a tile of
// 2^T amplitudes (the values of T chosen qubits, the lowest ones always
// among them so that every access moves whole 128-byte lines) in registers,
// 16 amplitudes per thread, applies every gate of the pass to it and writes
// it back: the state is read and written once for all of them, where a sweep
// per fused block moves it for each block of up to six qubits.
//
// A pass is a sequence of stages (passes.cpp). In a stage four of the tile's
// qubits index a thread's 16 registers, so a gate on one or two of them is
// arithmetic between registers with its matrix in scalar operands. Between
// stages the tile goes through LDS, which makes four other qubits the
// register qubits. Diagonal gates and the controls of other gates need no
// register qubit, nor even a qubit of the tile: they depend on index bits
// alone, which a thread knows.
//
// Complex64 states are computed in FP64 between the exchanges. The
// compiler's packed FP32 is off, so FP32 and FP64 multiply-adds issue at the
// same rate here, and a value is rounded once per stage, not once per gate.
//
// What bounds it: the FP64 arithmetic (eight multiplies and multiply-adds per
// amplitude and general one-qubit gate, four where its phases have joined the
// diagonal gates around it) on complex64 states, that and the memory on
// complex128 ones; workgroups on a compute unit hide one behind the other.
// Against fused block sweeps, programs of random layers: 28 qubits complex128
// in blocks of up to four 143 -> 32.2 ms, 25 qubits in blocks of up to six
// 44.3 -> 4.4 ms, 27 qubits complex64 in blocks of up to six 29.5 -> 13.9 ms.
#include "qs_internal.h"
#include "tile.h"
#include "tile_dev.h"

namespace qs {
namespace {

using namespace tiledev;

typedef const uint64_t __attribute__((address_space(4))) *Words;   // uniform loads
typedef uint64_t Head __attribute__((ext_vector_type(kTileAhead), aligned(8)));

struct TileGeom {
    int pos[kTileBitsMax];   // absolute tile bit positions, ascending
    int n_stages;
};

__device__ __forceinline__ double as_double(uint64_t w) { return __longlong_as_double((long long)w); }

// One-qubit gate on the pair of amplitudes p, q, in place: the last
// multiply-add of each sum overwrites an input that nothing reads any more.
// Written out, because every path through the operation loop has to leave
// the tile in the same registers; from plain expressions the compiler makes
// new values on each path, merges them by copies and spills. CLS: the
// matrix's register class, scalar or the thread's own.
#define QS_PAIR(CLS)                                                                                      \
    double ur, ui, vr, vi;                                                                                \
    asm("v_mul_f64 %4, %8, %0\n\t"                                                                        \
        "v_mul_f64 %5, %8, %1\n\t"                                                                        \
        "v_mul_f64 %6, %12, %0\n\t"                                                                       \
        "v_mul_f64 %7, %12, %1\n\t"                                                                       \
        "v_fma_f64 %4, -%9, %1, %4\n\t"                                                                   \
        "v_fma_f64 %5, %9, %0, %5\n\t"                                                                    \
        "v_fma_f64 %6, -%13, %1, %6\n\t"                                                                  \
        "v_fma_f64 %7, %13, %0, %7\n\t"                                                                   \
        "v_fma_f64 %4, %10, %2, %4\n\t"                                                                   \
        "v_fma_f64 %5, %10, %3, %5\n\t"                                                                   \
        "v_fma_f64 %6, %14, %2, %6\n\t"                                                                   \
        "v_fma_f64 %7, %15, %2, %7\n\t"                                                                   \
        "v_fma_f64 %0, -%11, %3, %4\n\t"                                                                  \
        "v_fma_f64 %1, %11, %2, %5\n\t"                                                                   \
        "v_fma_f64 %2, -%15, %3, %6\n\t"                                                                  \
        "v_fma_f64 %3, %14, %3, %7"                                                                       \
        : "+v"(pr), "+v"(pi), "+v"(qr), "+v"(qi), "=&v"(ur), "=&v"(ui), "=&v"(vr), "=&v"(vi)              \
        : CLS(m[0]), CLS(m[1]), CLS(m[2]), CLS(m[3]), CLS(m[4]), CLS(m[5]), CLS(m[6]), CLS(m[7]))

__device__ __forceinline__ void pair(double &pr, double &pi, double &qr, double &qi, const double (&m)[8])
{
    QS_PAIR("s");
}

__device__ __forceinline__ void cpair(double &pr, double &pi, double &qr, double &qi, const double (&m)[8])
{
    QS_PAIR("v");
}

// Amplitude x times a phase f, in place: the thread's own, or (uphase) one
// that all threads share.
#define QS_PHASE(CLS)                                                                                     \
    double u, v;                                                                                          \
    asm("v_mul_f64 %2, %5, %1\n\t"                                                                        \
        "v_mul_f64 %3, %5, %0\n\t"                                                                        \
        "v_fma_f64 %0, %4, %0, -%2\n\t"                                                                   \
        "v_fma_f64 %1, %4, %1, %3"                                                                        \
        : "+v"(xr), "+v"(xi), "=&v"(u), "=&v"(v)                                                          \
        : CLS(fr), CLS(fi))

__device__ __forceinline__ void phase(double &xr, double &xi, double fr, double fi) { QS_PHASE("v"); }

__device__ __forceinline__ void uphase(double &xr, double &xi, double fr, double fi) { QS_PHASE("s"); }

// Flips the sign of x where the top bit of f is set: hi ^ (f & top).
__device__ __forceinline__ void flip(double &x, uint32_t f, uint32_t top)
{
    uint32_t hi = uint32_t(__double2hiint(x));
    asm("v_bitop3_b32 %0, %0, %1, %2 bitop3:0x78" : "+v"(hi) : "v"(f), "s"(top));
    x = __hiloint2double(int(hi), __double2loint(x));
}

__device__ __forceinline__ void matrix2(double (&m)[8], Words w)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) m[i] = as_double(w[i]);
}

template <int B>
__device__ __forceinline__ void dense1(double (&xr)[16], double (&xi)[16], Words w)
{
    double m[8];
    matrix2(m, w);
#pragma unroll
    for (int j = 0; j < 16; ++j)
        if (!((j >> B) & 1)) pair(xr[j], xi[j], xr[j | (1 << B)], xi[j | (1 << B)], m);
}

// Real matrix on register bit B: what is left of a unitary once its phases
// have joined the diagonal gates around it. Half the multiply-adds of a
// complex one.
template <int B>
__device__ __forceinline__ void rotate1(double (&xr)[16], double (&xi)[16], const Head &w)
{
    const double a = as_double(w[1]), b = as_double(w[2]), c = as_double(w[3]), d = as_double(w[4]);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        if ((j >> B) & 1) continue;
        const int k = j | (1 << B);
        double t0, t1, t2, t3;
        asm("v_mul_f64 %4, %10, %0\n\t"
            "v_mul_f64 %5, %10, %1\n\t"
            "v_mul_f64 %6, %9, %2\n\t"
            "v_mul_f64 %7, %9, %3\n\t"
            "v_fma_f64 %0, %8, %0, %6\n\t"
            "v_fma_f64 %1, %8, %1, %7\n\t"
            "v_fma_f64 %2, %11, %2, %4\n\t"
            "v_fma_f64 %3, %11, %3, %5"
            : "+v"(xr[j]), "+v"(xi[j]), "+v"(xr[k]), "+v"(xi[k]), "=&v"(t0), "=&v"(t1), "=&v"(t2), "=&v"(t3)
            : "s"(a), "s"(b), "s"(c), "s"(d));
    }
}

// The same as dense1 where controls match: `on` says whether the thread's index bits
// do, bit j of `amps` whether register j's do. A thread whose bits do not
// match multiplies by the identity, exactly: a branch on `on` would make the
// compiler copy the tile on every path around it.
template <int B>
__device__ __forceinline__ void cdense1(double (&xr)[16], double (&xi)[16], Words w, bool on, uint32_t amps)
{
    double m[8];
    matrix2(m, w);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        asm("" : "+s"(m[i]));   // keeps the load out of the condition: a branch around it
        m[i] = on ? m[i] : (i == 0 || i == 6 ? 1.0 : 0.0);
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        if ((j >> B) & 1) continue;
        const int k = j | (1 << B);
        if ((amps >> j) & 1) cpair(xr[j], xi[j], xr[k], xi[k], m);
    }
}

// Exchanges two values where the mask is all ones (zero: leaves them).
__device__ __forceinline__ void exchange(double &a, double &b, uint32_t mask)
{
    uint32_t al = uint32_t(__double2loint(a)), ah = uint32_t(__double2hiint(a));
    uint32_t bl = uint32_t(__double2loint(b)), bh = uint32_t(__double2hiint(b)), t;
    asm("v_xor_b32 %2, %0, %1\n\tv_and_b32 %2, %2, %3\n\tv_xor_b32 %0, %0, %2\n\tv_xor_b32 %1, %1, %2"
        : "+v"(al), "+v"(bl), "=&v"(t) : "v"(mask));
    asm("v_xor_b32 %2, %0, %1\n\tv_and_b32 %2, %2, %3\n\tv_xor_b32 %0, %0, %2\n\tv_xor_b32 %1, %1, %2"
        : "+v"(ah), "+v"(bh), "=&v"(t) : "v"(mask));
    a = __hiloint2double(int(ah), int(al));
    b = __hiloint2double(int(bh), int(bl));
}

// (Controlled) X on register bit B: moves, no arithmetic.
template <int B>
__device__ __forceinline__ void xswap(double (&xr)[16], double (&xi)[16], bool on, uint32_t amps)
{
    const uint32_t mask = on ? ~0u : 0u;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        if ((j >> B) & 1) continue;
        const int k = j | (1 << B);
        if ((amps >> j) & 1) {
            exchange(xr[j], xr[k], mask);
            exchange(xi[j], xi[k], mask);
        }
    }
}

// Two-qubit gate on register bits B0 < B1 (local index bit 0 = B0).
template <int B0, int B1>
__device__ __forceinline__ void dense2(double (&xr)[16], double (&xi)[16], Words m)
{
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        if (((j >> B0) & 1) || ((j >> B1) & 1)) continue;
        const int at[4] = {j, j | (1 << B0), j | (1 << B1), j | (1 << B0) | (1 << B1)};
        double vr[4], vi[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            double sr = 0.0, si = 0.0;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double mr = as_double(m[2 * (4 * r + c)]), mi = as_double(m[2 * (4 * r + c) + 1]);
                sr = fma(-mi, xi[at[c]], fma(mr, xr[at[c]], sr));
                si = fma(mi, xr[at[c]], fma(mr, xi[at[c]], si));
            }
            vr[r] = sr;
            vi[r] = si;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            asm("v_mov_b64 %0, %1" : "+v"(xr[at[r]]) : "v"(vr[r]));
            asm("v_mov_b64 %0, %1" : "+v"(xi[at[r]]) : "v"(vi[r]));
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Calls f<B0, B1> for the pair number q in (0,1) (0,2) (0,3) (1,2) (1,3) (2,3).
#define QS_PAIR_CASES(f, q, ...)                     \
    switch (q) {                                     \
    case 0: f<0, 1>(__VA_ARGS__); break;             \
    case 1: f<0, 2>(__VA_ARGS__); break;             \
    case 2: f<0, 3>(__VA_ARGS__); break;             \
    case 3: f<1, 2>(__VA_ARGS__); break;             \
    case 4: f<1, 3>(__VA_ARGS__); break;             \
    default: f<2, 3>(__VA_ARGS__); break;            \
    }
#define QS_BIT_CASES(f, b, ...)                      \
    switch (b) {                                     \
    case 0: f<0>(__VA_ARGS__); break;                \
    case 1: f<1>(__VA_ARGS__); break;                \
    case 2: f<2>(__VA_ARGS__); break;                \
    default: f<3>(__VA_ARGS__); break;               \
    }

// Diagonal gates. First the phases that depend on register bits alone, as
// one factor per register, multiplied together by the planner. Then signs:
// every term flips the amplitudes of its register mask where the thread's
// index bits match, gathered in one 16-bit mask per thread. Then groups of
// phases that change the same registers: their product is formed once per
// thread, then multiplied in.
__device__ __forceinline__ void diagonal(double (&xr)[16], double (&xi)[16], uint32_t h, Words pc, uint64_t idx)
{
    const int nsign = int(h >> 8) & 0xfff, ngroup = int(h >> 20) & 0xfff;
    if ((h >> 6) & 1) {
#pragma unroll
        for (int j = 0; j < 16; ++j) uphase(xr[j], xi[j], as_double(pc[2 * j]), as_double(pc[2 * j + 1]));
        pc += 32;
    }
    if (nsign) {
        uint32_t s = 0;
        for (int i = 0; i < nsign; ++i) {
#pragma unroll
            for (int k = 0; k < kTileSigns; ++k) {
                const uint32_t amps = uint32_t(pc[3 * k + 2]);   // read first: a load under a condition is a branch
                s ^= (idx & pc[3 * k]) == pc[3 * k + 1] ? amps : 0u;
            }
            pc += 3 * kTileSigns;
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) {   // all 16: a branch around each costs more
            const uint32_t f = s << (31 - j);
            flip(xr[j], f, 0x80000000u);
            flip(xi[j], f, 0x80000000u);
        }
    }
    for (int g = 0; g < ngroup; ++g) {
        const uint32_t amps = uint32_t(pc[0]) & 0xffff;
        const int nt = int(pc[0] >> 16);
        double fr = as_double(pc[1]), fi = as_double(pc[2]);
        pc += 3;
        for (int i = 0; i < nt; ++i) {
            const bool on = (idx & pc[0]) == pc[1];
            const double pr = as_double(pc[2]), pi = as_double(pc[3]);
            const double r = fma(-pi, fi, pr * fr), q = fma(pi, fr, pr * fi);
            fr = on ? r : fr;
            fi = on ? q : fi;
            pc += 4;
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            if ((amps >> j) & 1) {
                phase(xr[j], xi[j], fr, fi);
            }
        }
    }
}

template <typename S, int T, bool NT>
__global__ __launch_bounds__(1 << (T - 4), 4) void k_tile_pass(typename V2<S>::T *__restrict__ psi,
                                                              const uint64_t *__restrict__ words, TileGeom tg)
{
    using N2 = typename V2<S>::N;
    __shared__ __align__(16) char lds[8 << T];
    const uint32_t tid = threadIdx.x;
    uint64_t base = xcd_order<uint64_t, 64>(blockIdx.x, gridDim.x);
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const int p = tg.pos[i];
        base = ((base >> p) << (p + 1)) | (base & ((1ull << p) - 1));
    }
    Words pc = (Words)words;
    Layout<T> L;
    L.set(base, pc[0], pc[1], pc[2], tid);
    double xr[16], xi[16];
    {
        const N2 *p = reinterpret_cast<const N2 *>(psi) + L.idx;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            N2 v;
            if constexpr (NT) v = __builtin_nontemporal_load(p + L.off(j));
            else v = p[L.off(j)];
            xr[j] = double(v.x);
            xi[j] = double(v.y);
        }
    }
    for (int st = 0;; ++st) {
        int nops = int(pc[2] >> 32);
        pc += 3;
        Head cur = *(const Head __attribute__((address_space(4))) *)pc;
        for (; nops > 0; --nops) {
            // the next operation's first words are on their way while this
            // one runs
            const uint64_t h = cur[0];
            const Words op = pc + 1;
            pc += h >> 32;
            const Head next = *(const Head __attribute__((address_space(4))) *)pc;
            const int type = int(h) & 7, arg = int(h >> 3) & 7;
            if (type == kTileRotate) {
                QS_BIT_CASES(rotate1, arg, xr, xi, cur)
            } else if (type == kTileDiag) {
                diagonal(xr, xi, uint32_t(h), op, L.idx);
            } else if (type == kTileDense1) {
                QS_BIT_CASES(dense1, arg, xr, xi, op)
            } else if (type == kTileDense2) {
                QS_PAIR_CASES(dense2, arg, xr, xi, op)
            } else {
                const bool on = (L.idx & cur[1]) == cur[2];
                const uint32_t amps = uint32_t(h >> 8) & 0xffff;
                if (type == kTileX) {
                    QS_BIT_CASES(xswap, arg, xr, xi, on, amps)
                } else {
                    QS_BIT_CASES(cdense1, arg, xr, xi, op + 2, on, amps)
                }
            }
            cur = next;
        }
        if (st + 1 >= tg.n_stages) break;
        Layout<T> M;
        M.set(base, pc[0], pc[1], pc[2], tid);
        exchange_tile<S, T>(xr, xi, lds, L, M);
        L = M;
    }
    N2 *p = reinterpret_cast<N2 *>(psi) + L.idx;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const N2 v = {S(xr[j]), S(xi[j])};
        if constexpr (NT) __builtin_nontemporal_store(v, p + L.off(j));
        else p[L.off(j)] = v;
    }
}

template <typename S, int T>
void launch(qs_state *h, const uint64_t *words, const TileGeom &tg, bool nt)
{
    auto *psi = static_cast<typename V2<S>::T *>(h->psi);
    const dim3 grid(unsigned(h->dim() >> T)), block(1u << (T - 4));
    if (nt) hipLaunchKernelGGL((k_tile_pass<S, T, true>), grid, block, 0, h->stream, psi, words, tg);
    else hipLaunchKernelGGL((k_tile_pass<S, T, false>), grid, block, 0, h->stream, psi, words, tg);
}

}  // namespace

int launch_tile_pass(qs_state *h, const TilePass &p, const uint64_t *dwords)
{
    if (p.T > h->n || (h->dim() >> p.T) > 0x7fffffffull)
        return fail(QS_EUNSUPPORTED, "tile of %d qubits on a %d-qubit state", p.T, h->n);
    TileGeom tg;
    for (int i = 0; i < kTileBitsMax; ++i) tg.pos[i] = i < p.T ? p.pos[i] : 0;
    tg.n_stages = p.n_stages;
    const uint64_t *w = dwords + p.word0;
    // past the last-level cache (28 qubits complex128: 32.5 ms, 33.0 without)
    const bool nt = h->dim() * h->amp_bytes() > (size_t(256) << 20);
    const bool d = h->dtype == QS_C128;
    switch (p.T) {
    case 10: d ? launch<double, 10>(h, w, tg, nt) : launch<float, 10>(h, w, tg, nt); break;
    case 11: d ? launch<double, 11>(h, w, tg, nt) : launch<float, 11>(h, w, tg, nt); break;
    case 12: d ? launch<double, 12>(h, w, tg, nt) : launch<float, 12>(h, w, tg, nt); break;
    default: return fail(QS_EUNSUPPORTED, "tile of %d qubits", p.T);
    }
    QS_HIP(hipGetLastError());
    return QS_OK;
}

}  // namespace qs
