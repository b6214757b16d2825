// FFT passes over digits of up to 10 bits on tiles held in registers
// (the decomposition is fft.hip's: a pass transforms one digit of the field).
//
// A workgroup owns a tile of 2^E amplitudes: the digit's values times
// 2^(E - r) columns, the bits that are lowest in the destination. 16
// amplitudes sit in each thread's registers. The digit is transformed four
// bits at a time from its top (radix 16 in registers, decimation in
// frequency) with an exchange through LDS after each step, the last step
// taking the one to four bits that are left; its other registers hold the
// top bits of the digit that the step before put out, so that the register
// number is always the top four bits of the output digit. Lanes run along
// the lowest source bits on the load and along the lowest destination bits
// on the store: both move whole 128-byte lines, also on a final pass, which
// reverses the digits' order.
//
// Twiddles: each thread forms its own roots by FP64 sincospi on exponents
// that are reduced in integers; a value's twiddle is the product of two.
// Complex64 tiles are computed in FP64 between loads, exchanges and stores:
// without packed FP32 that is the same number of instructions.
//
// What bounds it: memory on complex128 states, the arithmetic on complex64
// ones (72 % busy on digits of 9 bits). Tiles of 2^12 amplitudes leave four
// workgroups of four waves to a compute unit, tiles of 2^13 (digits whose
// lines need them: 9 and 10 bits in complex64, 10 in complex128) two of eight
// waves, so loads of one tile overlap with the arithmetic of others, without
// the persistent loop and prefetch that the 10-bit register tiles of fft.hip
// need at one workgroup per unit.
#include "fft_tile.h"

#include <algorithm>

#include "fft_dev.h"
#include "tile_dev.h"

namespace qs {
namespace {

using namespace tiledev;

constexpr int kMaxTile = 13;

struct Geom {
    int nrest;                   // bits outside the tile: their places in the source and the destination
    uint8_t src[40], dst[40];
    uint64_t lay[3][3];          // layouts of the load, the middle step and the store
    int cb;                      // column bits: tile bits 0 .. cb - 1, the digit above them
    int dig_lo, r;
    int tw_bits, krest_lo, krest_bits;   // pass twiddle (tw_bits 0: none)
    int inverse;
    double scale;
};

using C = double2;

__device__ __forceinline__ C mul(C a, C b) { return C{fma(-a.y, b.y, a.x * b.x), fma(a.y, b.x, a.x * b.y)}; }

// exp(2 pi i u / 16) d, u < 8
template <int U>
__device__ __forceinline__ C turn(C d)
{
    constexpr double c1 = 0.92387953251128675613, s1 = 0.38268343236508977173, h = 0.70710678118654752440;
    if constexpr (U == 0) return d;
    else if constexpr (U == 4) return C{-d.y, d.x};
    else if constexpr (U == 2) return C{h * (d.x - d.y), h * (d.x + d.y)};
    else if constexpr (U == 6) return C{-h * (d.x + d.y), h * (d.x - d.y)};
    else {
        constexpr double cs = U == 1 ? c1 : U == 3 ? s1 : U == 5 ? -s1 : -c1;
        constexpr double sn = U == 1 ? s1 : U == 3 ? c1 : U == 5 ? c1 : s1;
        return C{cs * d.x - sn * d.y, cs * d.y + sn * d.x};
    }
}

// Natural-order DFT of the 2^K registers x[o + s i], i < 2^K.
template <int K, int H, int I>
__device__ __forceinline__ void level(double (&xr)[16], double (&xi)[16], int o, int s)
{
    if constexpr (I < H) {
#pragma unroll
        for (int b = 0; b < (1 << K); b += 2 * H) {
            const int p = o + s * (b + I), q = o + s * (b + I + H);
            const double ar = xr[p], ai = xi[p], br = xr[q], bi = xi[q];
            xr[p] = ar + br;
            xi[p] = ai + bi;
            const C d = turn<I *(8 / H)>(C{ar - br, ai - bi});
            xr[q] = d.x;
            xi[q] = d.y;
        }
        level<K, H, I + 1>(xr, xi, o, s);
    }
}

template <int K, int H = (1 << K) / 2>
__device__ __forceinline__ void dft(double (&xr)[16], double (&xi)[16], int o, int s)
{
    if constexpr (H >= 1) {
        level<K, H, 0>(xr, xi, o, s);
        dft<K, H / 2>(xr, xi, o, s);
    } else {
#pragma unroll
        for (int l = 0; l < (1 << K); ++l) {
            int v = 0;
#pragma unroll
            for (int b = 0; b < K; ++b) v |= ((l >> b) & 1) << (K - 1 - b);
            if (v > l) {
                const double r = xr[o + s * l], i = xi[o + s * l];
                xr[o + s * l] = xr[o + s * v];
                xi[o + s * l] = xi[o + s * v];
                xr[o + s * v] = r;
                xi[o + s * v] = i;
            }
        }
    }
}

__device__ __forceinline__ C root(uint64_t num, int bits)
{
    double sn, cs;
    sincospi(__builtin_ldexp(double(num), 1 - bits), &sn, &cs);
    return C{cs, sn};
}

__device__ __forceinline__ void times(double &xr, double &xi, C p)
{
    const double r = xr;
    xr = fma(-p.y, xi, p.x * r);
    xi = fma(p.y, r, p.x * xi);
}

// x[k] times exp(2 pi i (e0 + k e) / 2^bits). Complex128: as the product of
// the factors of k mod 4 (with e0) and of k / 4, every one a root of its own;
// powers by repeated squaring double their error with each squaring (24-qubit
// transform: 1.2e-15 against 6.7e-16 for the same time). Complex64, where
// that error is far below a rounding: powers, a tenth faster.
template <typename S, bool START>
__device__ __forceinline__ void turns(double (&xr)[16], double (&xi)[16], uint64_t e0, uint64_t e, int bits)
{
    const uint64_t m = (1ull << bits) - 1;
    C a[4];
    if constexpr (sizeof(S) == 8) {
#pragma unroll
        for (int i = START ? 0 : 1; i < 4; ++i) a[i] = root((e0 + uint64_t(i) * e) & m, bits);
    } else {
        a[1] = root(e & m, bits);
        a[2] = mul(a[1], a[1]);
        a[3] = mul(a[2], a[1]);
    }
    C b{1, 0}, w4{1, 0};
    if constexpr (sizeof(S) == 4) {
        w4 = mul(a[2], a[2]);
        if constexpr (START) {
            a[0] = root(e0 & m, bits);
#pragma unroll
            for (int i = 1; i < 4; ++i) a[i] = mul(a[i], a[0]);
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (j) {
            if constexpr (sizeof(S) == 8) b = root((uint64_t(4 * j) * e) & m, bits);
            else b = j == 1 ? w4 : mul(b, w4);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (!START && i == 0) {
                if (j) times(xr[4 * j], xi[4 * j], b);
            } else {
                times(xr[4 * j + i], xi[4 * j + i], j ? mul(a[i], b) : a[i]);
            }
        }
    }
}

// STEPS register steps; the last takes LAST bits of the digit, the others
// four each.
template <typename S, int STEPS, int LAST>
__global__ __launch_bounds__(512, 4) void k_fft_tile(const typename V2<S>::T *__restrict__ src,
                                                    typename V2<S>::T *__restrict__ dst, Geom g)
{
    using N2 = typename V2<S>::N;
    constexpr int R = 4 * (STEPS - 1) + LAST;
    extern __shared__ __align__(16) char lds[];
    const uint32_t tid = threadIdx.x;
    const uint32_t b = blockIdx.x, n = gridDim.x;
    const uint32_t tile = n % 8 ? b : (b % 8) * (n / 8) + b / 8;   // an eighth of the tiles per XCD
    uint64_t from = 0, to = 0;
    for (int i = 0; i < g.nrest; ++i) {
        const uint64_t bit = (tile >> i) & 1;
        from |= bit << g.src[i];
        to |= bit << g.dst[i];
    }
    Layout<kMaxTile> L;
    L.set(from, g.lay[0][0], g.lay[0][1], g.lay[0][2], tid);
    double xr[16], xi[16];
    {
        const N2 *p = reinterpret_cast<const N2 *>(src) + L.idx;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const N2 v = p[L.off(j)];
            xr[j] = double(v.x);
            xi[j] = double(v.y);
        }
    }
    // an inverse transform is the forward one of the conjugates, conjugated
    const double s0 = g.inverse ? -1.0 : 1.0;
#pragma unroll
    for (int j = 0; j < 16; ++j) xi[j] *= s0;
#pragma unroll
    for (int st = 0; st + 1 < STEPS; ++st) {
        const int low = R - 4 * (st + 1);   // digit bits below this step's
        dft<4>(xr, xi, 0, 1);
        const uint32_t lo = (L.e >> g.cb) & ((1u << low) - 1);
        turns<S, false>(xr, xi, 0, lo, low + 4);
        const uint64_t *w = g.lay[st + 2 == STEPS ? 2 : 1];
        Layout<kMaxTile> M;
        M.set(st + 2 == STEPS ? to : from, w[0], w[1], w[2], tid);
        exchange_tile<S>(xr, xi, lds, L, M);
        L = M;
    }
    if constexpr (STEPS == 1) {
        // nothing moves: the store's places in the layout of the load
        L.set(to, g.lay[2][0], g.lay[2][1], g.lay[2][2], tid);
    }
    constexpr int X = 4 - LAST;             // register bits that are not this step's
#pragma unroll
    for (int o = 0; o < (1 << X); ++o) dft<LAST>(xr, xi, o, 1 << X);
    if (g.tw_bits) {
        const uint64_t k = (L.idx >> g.krest_lo) & ((1ull << g.krest_bits) - 1);
        const uint64_t l = (L.idx >> g.dig_lo) & ((1ull << R) - 1);
        turns<S, true>(xr, xi, k * l, k << (R - 4), g.tw_bits);
    }
    // scale and conjugation in every pass: a branch around either makes the
    // compiler copy the tile (28 qubits: 6.7 against 5.5 ms)
    N2 *p = reinterpret_cast<N2 *>(dst) + L.idx;
    const double sr = g.scale, si = g.inverse ? -g.scale : g.scale;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const N2 v = {S(xr[j] * sr), S(xi[j] * si)};
        p[L.off(j)] = v;
    }
}

template <typename S, int STEPS, int LAST>
void launch(hipStream_t s, const void *src, void *dst, const Geom &g, int E, uint32_t tiles)
{
    using T = typename V2<S>::T;
    hipLaunchKernelGGL((k_fft_tile<S, STEPS, LAST>), dim3(tiles), dim3(1u << (E - 4)), STEPS > 1 ? size_t(8) << E : 0,
                       s, static_cast<const T *>(src), static_cast<T *>(dst), g);
}

template <typename S>
void launch_r(hipStream_t s, const void *src, void *dst, const Geom &g, int E, uint32_t tiles)
{
    switch (g.r) {
    case 1: launch<S, 1, 1>(s, src, dst, g, E, tiles); break;
    case 2: launch<S, 1, 2>(s, src, dst, g, E, tiles); break;
    case 3: launch<S, 1, 3>(s, src, dst, g, E, tiles); break;
    case 4: launch<S, 1, 4>(s, src, dst, g, E, tiles); break;
    case 5: launch<S, 2, 1>(s, src, dst, g, E, tiles); break;
    case 6: launch<S, 2, 2>(s, src, dst, g, E, tiles); break;
    case 7: launch<S, 2, 3>(s, src, dst, g, E, tiles); break;
    case 8: launch<S, 2, 4>(s, src, dst, g, E, tiles); break;
    case 9: launch<S, 3, 1>(s, src, dst, g, E, tiles); break;
    default: launch<S, 3, 2>(s, src, dst, g, E, tiles); break;
    }
}

// A few bit positions, on the stack: a launch between two passes allocates
// nothing that could fail.
struct Bits {
    int v[64], n = 0;
    void push_back(int b) { v[n++] = b; }
    int size() const { return n; }
    int *begin() { return v; }
    int *end() { return v + n; }
    const int *begin() const { return v; }
    const int *end() const { return v + n; }
    int operator[](int i) const { return v[i]; }
};

}  // namespace

bool fft_tile_applies(int n, const fftdev::PassArgs &pa)
{
    // digits of fewer than four bits with a pass twiddle come from a tuned
    // digit width only
    return n >= 10 && pa.r <= 10 && (pa.r >= 4 || !pa.tw_bits);
}

int launch_fft_tile(qs_state *h, const fftdev::PassArgs &pa, const void *src, void *dst)
{
    const int n = h->n, r = pa.r;
    const int line = h->dtype == QS_C128 ? 3 : 4;   // bits inside 128 bytes
    // 2^12 amplitudes, or 2^13 where a line's worth of columns needs it
    const int E = std::min(n, r + line > 12 ? 13 : 12);
    Geom g;
    std::fill_n(&g.lay[0][0], 9, 0);
    g.r = r;
    g.cb = E - r;
    g.dig_lo = pa.dig_lo;
    g.tw_bits = pa.tw_bits;
    g.krest_lo = pa.krest_lo;
    g.krest_bits = pa.krest_bits;
    g.inverse = pa.sgn < 0;
    g.scale = pa.scale;
    // destination of every source bit, digit included (its output bits take
    // its places; a final pass reverses the digits' order)
    int dest[64];
    for (int q = 0; q < n; ++q) dest[q] = q;
    if (pa.final_pass)
        for (int d = 0; d < pa.ndig; ++d)
            for (int i = 0; i < pa.dw[d]; ++i) dest[pa.dpos[d] + i] = pa.q_lo + pa.doff[d] + i;
    Bits other, cols, rest;
    for (int q = 0; q < n; ++q)
        if (q < pa.dig_lo || q >= pa.dig_lo + r) other.push_back(q);
    std::sort(other.begin(), other.end(), [&](int a, int b) { return dest[a] < dest[b]; });
    for (int i = 0; i < other.size(); ++i) (i < g.cb ? cols : rest).push_back(other[i]);
    std::sort(rest.begin(), rest.end());
    g.nrest = rest.size();
    for (int i = 0; i < g.nrest; ++i) {
        g.src[i] = uint8_t(rest[i]);
        g.dst[i] = uint8_t(dest[rest[i]]);
    }
    // Tile bit t < cb: column t. Tile bit cb + p: digit place p; after a step
    // over places [p, p + 4) these hold four bits of the output digit, whose
    // first step's bits are the lowest.
    const int steps = (r + 3) / 4, last = r - 4 * (steps - 1);
    auto out_bit = [&](int p) {   // output digit bit at place p after all steps
        for (int s = 0; s < steps; ++s) {
            const int w = s + 1 < steps ? 4 : last, lo = s + 1 < steps ? r - 4 * (s + 1) : 0;
            if (p >= lo && p < lo + w) return 4 * s + (p - lo);
        }
        return 0;
    };
    auto src_of = [&](int t) { return t < g.cb ? cols[t] : pa.dig_lo + (t - g.cb); };
    auto dst_of = [&](int t) { return t < g.cb ? dest[cols[t]] : dest[pa.dig_lo + out_bit(t - g.cb)]; };
    // lay[i]: register tile bits regs (lowest first), thread bits ordered by
    // address inside a line, then so that the low five differ modulo 5 (LDS
    // banks), then by address
    auto lay = [&](int i, const Bits &regs, auto &&addr) {
        Bits thr, order;
        for (int t = 0; t < E; ++t)
            if (std::find(regs.begin(), regs.end(), t) == regs.end()) thr.push_back(t);
        std::sort(thr.begin(), thr.end(), [&](int a, int b) { return addr(a) < addr(b); });
        uint32_t cls = 0;
        for (int t : thr) {
            if (order.size() >= 5) break;
            if (addr(t) < line || !((cls >> (t % 5)) & 1)) {
                cls |= 1u << (t % 5);
                order.push_back(t);
            }
        }
        for (int t : thr)
            if (std::find(order.begin(), order.end(), t) == order.end()) order.push_back(t);
        for (int k = 0; k < E - 4; ++k) {
            g.lay[i][0] |= uint64_t(order[k]) << (4 * k);
            g.lay[i][1] |= uint64_t(addr(order[k])) << (6 * k);
        }
        for (int b = 0; b < 4; ++b) {
            g.lay[i][0] |= uint64_t(regs[b]) << (4 * (kMaxTile - 4 + b));
            g.lay[i][2] |= uint64_t(addr(regs[b])) << (6 * b);
        }
    };
    Bits top, mid, fin;
    if (steps == 1) {
        // columns fill the registers below the digit
        for (int t = E - 4; t < E; ++t) top.push_back(t);
        fin = top;
    } else {
        for (int b = 0; b < 4; ++b) top.push_back(g.cb + r - 4 + b);
        for (int b = 0; b < 4; ++b) mid.push_back(g.cb + r - 8 + b);
        const int before = r - 4 * (steps - 1);   // lowest place of the step before the last
        for (int b = last; b < 4; ++b) fin.push_back(g.cb + before + b);
        for (int b = 0; b < last; ++b) fin.push_back(g.cb + b);
    }
    lay(0, top, src_of);
    if (steps == 3) lay(1, mid, src_of);
    if (steps == 1) {
        // the store keeps the load's thread bits: nothing is exchanged
        g.lay[2][0] = g.lay[0][0];
        for (int k = 0; k < E - 4; ++k) g.lay[2][1] |= uint64_t(dst_of(int(g.lay[0][0] >> (4 * k)) & 15)) << (6 * k);
        for (int b = 0; b < 4; ++b) g.lay[2][2] |= uint64_t(dst_of(top[b])) << (6 * b);
    } else {
        lay(2, fin, dst_of);
    }
    const uint64_t tiles = h->dim() >> E;
    if (tiles > 0x7fffffffull) return fail(QS_EUNSUPPORTED, "FFT tile count too large");
    if (h->dtype == QS_C128) launch_r<double>(h->stream, src, dst, g, E, uint32_t(tiles));
    else launch_r<float>(h->stream, src, dst, g, E, uint32_t(tiles));
    QS_HIP(hipGetLastError());
    return QS_OK;
}

}  // namespace qs
