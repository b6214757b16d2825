// Measurement quantities read directly off the state (Sec. III-D): the
// whole distribution or an expectation value in one pass, no sampling of
// repeated runs. Probabilities are |alpha_i|^2 (Sec. II). All accumulation
// is FP64, also for FP32 states. Partial sums are combined in a fixed order
// so repeated calls give identical results.
#include "qs_internal.h"

#include <algorithm>
#include <cmath>
#include <mutex>

namespace qs {
namespace {

constexpr int kThreads = 256;
constexpr int kReduceBlocks = 2048;

template <typename R> struct V2;
template <> struct V2<double> { using T = double2; };
template <> struct V2<float> { using T = float2; };

__device__ __forceinline__ double wave_sum(double v)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Sum over the block in a fixed order; result valid in thread 0.
__device__ __forceinline__ double block_sum(double v, double *sh)
{
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) sh[wave] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < kThreads / 64; ++w) t += sh[w];
    __syncthreads();
    return t;
}

template <typename R>
__global__ __launch_bounds__(kThreads) void k_norm2(const typename V2<R>::T *__restrict__ psi,
                                                    uint64_t dim, double *__restrict__ partial)
{
    __shared__ double sh[kThreads / 64];
    double s = 0.0;
    for (uint64_t i = uint64_t(blockIdx.x) * kThreads + threadIdx.x; i < dim;
         i += uint64_t(gridDim.x) * kThreads) {
        const double x = double(psi[i].x), y = double(psi[i].y);
        s = fma(x, x, fma(y, y, s));
    }
    s = block_sum(s, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// <psi|P|psi> for a Pauli string: P|i> = c_i |i ^ f>, f = x|y,
// c_i = i^{|y|} (-1)^{popcount(i & (y|z))}. For f != 0 the pair (i, i^f) is
// visited once through its member with the top bit of f clear, and both
// terms conj(psi_{i^f}) c_i psi_i and conj(psi_i) c_{i^f} psi_{i^f} are
// added; the common factor i^{|y|} is applied on the host.
template <typename R>
__global__ __launch_bounds__(kThreads) void k_pauli(const typename V2<R>::T *__restrict__ psi,
                                                    uint64_t n_items, uint64_t f, int hbit,
                                                    uint64_t sgn_mask, double *__restrict__ partial)
{
    __shared__ double sh[kThreads / 64];
    double sre = 0.0, sim = 0.0;
    for (uint64_t g = uint64_t(blockIdx.x) * kThreads + threadIdx.x; g < n_items;
         g += uint64_t(gridDim.x) * kThreads) {
        if (f == 0) {
            const double x = double(psi[g].x), y = double(psi[g].y);
            const double p = fma(x, x, y * y);
            sre += (__popcll(g & sgn_mask) & 1) ? -p : p;
            continue;
        }
        const uint64_t i = ((g >> hbit) << (hbit + 1)) | (g & ((1ull << hbit) - 1));
        const uint64_t j = i ^ f;
        const double ar = double(psi[i].x), ai = double(psi[i].y);
        const double br = double(psi[j].x), bi = double(psi[j].y);
        const double si = (__popcll(i & sgn_mask) & 1) ? -1.0 : 1.0;
        const double sj = (__popcll(j & sgn_mask) & 1) ? -1.0 : 1.0;
        // conj(b) * a * si + conj(a) * b * sj
        const double cr = br * ar + bi * ai;  // Re(conj(b) a) = Re(conj(a) b)
        const double ci = br * ai - bi * ar;  // Im(conj(b) a) = -Im(conj(a) b)
        sre += (si + sj) * cr;
        sim += (si - sj) * ci;
    }
    sre = block_sum(sre, sh);
    sim = block_sum(sim, sh);
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = sre;
        partial[2 * blockIdx.x + 1] = sim;
    }
}

// Fixed-order sums over `count` tuples of width W, valid in thread 0. The
// columns are read together, in one pass over the tuples: an expectation of a
// 24-qubit complex64 state 35.9 -> 35.3 us, of 20 qubits 19.1 -> 18.4, of 14
// (few tuples) 16.6 -> 16.4 from call to result. Kernel traces do not resolve
// it (4.1 us before and after).
template <int W>
__device__ __forceinline__ void finish_sums(const double *__restrict__ partial, int count, double (&s)[W])
{
    __shared__ double sh[W][kThreads / 64];
#pragma unroll
    for (int c = 0; c < W; ++c) s[c] = 0.0;
#pragma unroll 8
    for (int i = threadIdx.x; i < count; i += kThreads)
#pragma unroll
        for (int c = 0; c < W; ++c) s[c] += partial[size_t(i) * W + c];
#pragma unroll
    for (int c = 0; c < W; ++c) s[c] = block_sum(s[c], sh[c]);
}

// out may be mapped host memory
template <int W>
__global__ __launch_bounds__(kThreads) void k_finish(const double *__restrict__ partial, int count,
                                                     double *__restrict__ out)
{
    double s[W];
    finish_sums<W>(partial, count, s);
    if (threadIdx.x == 0)
#pragma unroll
        for (int c = 0; c < W; ++c) out[c] = s[c];
}

struct QArgs {
    int m;
    int q[20];
};

__device__ __forceinline__ uint32_t outcome_of(uint64_t i, const QArgs &qa)
{
    uint32_t o = 0;
    for (int r = 0; r < qa.m; ++r) o |= uint32_t((i >> qa.q[r]) & 1) << r;
    return o;
}

// An item is 16 bytes of the state: one complex128 or two neighbouring
// complex64 amplitudes. A thread of k_hist has kAhead items in flight.
constexpr int kAheadBits = 2, kAhead = 1 << kAheadBits;
template <typename R> struct Item;
template <> struct Item<double> {
    static constexpr int bits = 0;
    double2 a;
    __device__ __forceinline__ void load(const void *psi, uint64_t g) { a = static_cast<const double2 *>(psi)[g]; }
    __device__ __forceinline__ double re(int) const { return a.x; }
    __device__ __forceinline__ double im(int) const { return a.y; }
};
template <> struct Item<float> {
    static constexpr int bits = 1;
    float4 a;
    __device__ __forceinline__ void load(const void *psi, uint64_t g) { a = static_cast<const float4 *>(psi)[g]; }
    __device__ __forceinline__ double re(int h) const { return double(h ? a.z : a.x); }
    __device__ __forceinline__ double im(int h) const { return double(h ? a.w : a.y); }
};

// Marginals. A wave reads rows of 64 items (the state's low bits); its high
// measured bits are fixed, and it walks the values of the unmeasured high
// bits in one of `splits` ranges, each lane adding up its own items. At the
// end the lanes are summed over the unmeasured low bits. So every read is a
// whole row, nothing is atomic, and the order of every sum is fixed. Waves
// that share their outcomes (splits > 1) write rows of partial sums.
// Workgroup histograms in LDS, which this replaces, left the columns of up to
// 2048 rows to a few workgroups, and above 12 qubits one thread read all of
// an outcome's amplitudes. 24 qubits complex64, 10 measured: 522 -> 27 us; 27
// qubits complex128, 13 measured: 13.6 -> 0.40 ms a call.
// 16 waves per CU; 32 and 64, with twice and four times the partial rows, are
// within 3% of it on 28 to 30 qubits.
constexpr int kHistWaveBits = 12;
struct HistArgs {
    uint64_t hi_meas, hi_rest;   // masks of item index bits above the row
    int hi_count;                // measured bits above the row
    int low_meas;                // mask of measured bits of an amplitude's place in the row
    uint64_t steps;              // unmeasured high values per wave
    int splits;
    int row;                     // items in a row: 64, or all of a smaller state
};

__device__ __forceinline__ uint64_t spread(uint64_t x, uint64_t mask)
{
    uint64_t o = 0;
    for (; mask && x; mask &= mask - 1, x >>= 1)
        if (x & 1) o |= mask & (~mask + 1);
    return o;
}

template <typename R>
__global__ __launch_bounds__(kThreads) void k_hist(const void *__restrict__ psi, QArgs qa, HistArgs ha,
                                                   double *__restrict__ partial)
{
    constexpr int B = Item<R>::bits, H = 1 << B;
    const int lane = threadIdx.x & 63;
    const uint64_t wave = uint64_t(blockIdx.x) * (kThreads / 64) + (threadIdx.x >> 6);
    const uint64_t hi = wave & ((1ull << ha.hi_count) - 1), split = wave >> ha.hi_count;
    if (split >= uint64_t(ha.splits)) return;   // whole waves; no barrier below
    const uint64_t row0 = spread(hi, ha.hi_meas) | uint64_t(min(lane, ha.row - 1));
    uint64_t x = spread(split * ha.steps, ha.hi_rest);
    double s[H];
#pragma unroll
    for (int h = 0; h < H; ++h) s[h] = 0.0;
    // next value of the unmeasured bits: carries run through the other bits
    auto next = [&]() { x = ((x | ~ha.hi_rest) + 1) & ha.hi_rest; };
    auto add = [&](const Item<R> &v) {
#pragma unroll
        for (int h = 0; h < H; ++h) s[h] = fma(v.re(h), v.re(h), fma(v.im(h), v.im(h), s[h]));
    };
    uint64_t t = 0;
    for (; t + kAhead <= ha.steps; t += kAhead) {
        Item<R> v[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            v[u].load(psi, row0 | x);
            next();
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) add(v[u]);
    }
    for (; t < ha.steps; ++t) {
        Item<R> v;
        v.load(psi, row0 | x);
        next();
        add(v);
    }
    if (lane >= ha.row) {
#pragma unroll
        for (int h = 0; h < H; ++h) s[h] = 0.0;
    }
    if (H == 2 && !(ha.low_meas & 1)) {
        s[0] += s[H - 1];
        s[H - 1] = 0.0;
    }
    for (int b = 0; b < 6; ++b)
        if (!((ha.low_meas >> (b + B)) & 1))
#pragma unroll
            for (int h = 0; h < H; ++h) s[h] += __shfl_xor(s[h], 1 << b, 64);
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const int low = (lane << B) | h;
        if (low & ~ha.low_meas) continue;       // the sum's first lane writes it
        const uint64_t i = (spread(hi, ha.hi_meas) << B) | uint64_t(low);
        partial[(split << qa.m) + outcome_of(i, qa)] = s[h];
    }
}

// Column sums of the partial rows, up to 64 outcomes per workgroup: the
// threads of an outcome take its rows in turn, then halve their sums in LDS.
constexpr int kColThreads = 1024;
__global__ __launch_bounds__(kColThreads) void k_hist_cols(const double *__restrict__ partial, int rows, int M,
                                                           double *__restrict__ p)
{
    __shared__ double sh[kColThreads];
    const int cols = min(M, 64), t = threadIdx.x, o = int(blockIdx.x) * cols + (t & (cols - 1));
    double s = 0.0;
#pragma unroll 4
    for (int r = t / cols; r < rows; r += kColThreads / cols) s += partial[size_t(r) * M + o];
    sh[t] = s;
    for (int half = kColThreads / 2; half >= cols; half >>= 1) {
        __syncthreads();
        if (t < half) sh[t] += sh[t + half];
    }
    if (t < cols) p[o] = sh[t];
}

// Inclusive prefix sum of p (single workgroup, fixed order): each thread
// scans a contiguous chunk, chunk totals are scanned serially.
__global__ __launch_bounds__(kThreads) void k_cdf(const double *__restrict__ p, int M,
                                                  double *__restrict__ cdf)
{
    __shared__ double tot[kThreads];
    const int chunk = (M + kThreads - 1) / kThreads;
    const int lo = threadIdx.x * chunk, hi = min(M, lo + chunk);
    double s = 0.0;
    for (int o = lo; o < hi; ++o) s += p[o];
    tot[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double run = 0.0;
        for (int t = 0; t < kThreads; ++t) {
            const double v = tot[t];
            tot[t] = run;
            run += v;
        }
    }
    __syncthreads();
    double run = tot[threadIdx.x];
    for (int o = lo; o < hi; ++o) {
        run += p[o];
        cdf[o] = run;
    }
}

// Smallest o with cdf[o] > u * total (binary search).
__global__ void k_sample(const double *__restrict__ cdf, int M, const double *__restrict__ u,
                         int shots, uint64_t *__restrict__ out)
{
    const int s = blockIdx.x * kThreads + threadIdx.x;
    if (s >= shots) return;
    const double target = u[s] * cdf[M - 1];
    int lo = 0, hi = M - 1;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (cdf[mid] > target) hi = mid;
        else lo = mid + 1;
    }
    out[s] = uint64_t(lo);
}

// Project onto the first shot's outcome and rescale by 1/sqrt(p) (read on
// the device). Items outside the outcome are written, not read.
template <typename R>
__global__ __launch_bounds__(kThreads) void k_collapse(void *__restrict__ psi, uint64_t n_items, QArgs qa,
                                                       const uint64_t *__restrict__ outcome,
                                                       const double *__restrict__ p)
{
    constexpr int B = Item<R>::bits, H = 1 << B;
    const uint32_t o = uint32_t(outcome[0]);
    const double sc = 1.0 / sqrt(p[o]);
    uint64_t mask = 0, vals = 0;
    for (int r = 0; r < qa.m; ++r) {
        mask |= 1ull << qa.q[r];
        vals |= uint64_t((o >> r) & 1) << qa.q[r];
    }
    for (uint64_t g = uint64_t(blockIdx.x) * kThreads + threadIdx.x; g < n_items;
         g += uint64_t(gridDim.x) * kThreads) {
        Item<R> v;
        if ((g & (mask >> B)) == vals >> B) {
            v.load(psi, g);
        } else {
            v.a = {};
        }
        double re[H], im[H];
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const bool on = (uint64_t(h) & mask & (H - 1)) == (vals & (H - 1));
            re[h] = on ? v.re(h) * sc : 0.0;
            im[h] = on ? v.im(h) * sc : 0.0;
        }
        if constexpr (B == 0) static_cast<double2 *>(psi)[g] = double2{re[0], im[0]};
        else static_cast<float4 *>(psi)[g] = float4{float(re[0]), float(im[0]), float(re[H - 1]), float(im[H - 1])};
    }
}

template <typename R>
__global__ void k_gather_amps(const typename V2<R>::T *__restrict__ psi,
                              const uint64_t *__restrict__ idx, int count,
                              typename V2<R>::T *__restrict__ out)
{
    const int t = blockIdx.x * kThreads + threadIdx.x;
    if (t < count) out[t] = psi[idx[t]];
}

// Fixed-order final sum of the Pauli partials (as k_finish), times
// i^{popcount(y)} (y_pow = popcount(y) mod 4), written to device memory.
__global__ __launch_bounds__(kThreads) void k_finish_pauli(const double *__restrict__ partial, int count, int y_pow,
                                                           double *__restrict__ out)
{
    double s[2];
    finish_sums<2>(partial, count, s);
    if (threadIdx.x == 0) {
        double r = s[0], im = s[1];
        switch (y_pow) {
        case 0: break;
        case 1: { const double t = r; r = -im; im = t; break; }
        case 2: r = -r; im = -im; break;
        default: { const double t = r; r = im; im = -t; break; }
        }
        out[0] = r;
        out[1] = im;
    }
}

// Scratch of the allocation-free expectation (qs_expectation_noalloc): the
// per-block partial sums of one Pauli expectation, two doubles for each of
// at most kReduceBlocks blocks (32 KiB). Each GPU holds one copy from the
// library's load until the process ends; calls that overlap on one GPU race
// on it. Host code reaches it only through the per-device address that
// hipGetSymbolAddress returns (the array's name is a host-side stand-in).
constexpr size_t kNoAllocDoubles = 2 * size_t(kReduceBlocks);
static __device__ __align__(256) double scratch[kNoAllocDoubles];

constexpr int kMaxDevices = 64;

// Device address of `scratch` on `device`, resolved once per device with
// that device current.
int scratch_address(int device, double **out)
{
    static std::mutex mu;
    static double *addr[kMaxDevices] = {};
    if (device < 0 || device >= kMaxDevices) return fail(QS_EUNSUPPORTED, "device %d outside [0, %d)", device, kMaxDevices);
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[device]) {
        int cur = -1;
        QS_HIP(hipGetDevice(&cur));
        if (cur != device) QS_HIP(hipSetDevice(device));
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (cur != device) (void)hipSetDevice(cur);
        if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        if (!p) return fail(QS_EDEVICE, "no device address for the expectation scratch");
        addr[device] = static_cast<double *>(p);
    }
    *out = addr[device];
    return QS_OK;
}

unsigned red_grid(uint64_t items)
{
    uint64_t b = (items + kThreads - 1) / kThreads;
    return unsigned(std::max<uint64_t>(1, std::min<uint64_t>(b, kReduceBlocks)));
}

// The last kernel writes the result straight to host memory (pinned and
// coherent, so it is there when the stream is idle); a copy took 3.3 us more.
int finish_to_host(qs_state *h, int count, int w, double *out)
{
    if (int rc = ensure_host_out(h, sizeof(double) * size_t(w))) return rc;
    hipLaunchKernelGGL(w == 1 ? k_finish<1> : k_finish<2>, dim3(1), dim3(kThreads), 0, h->stream, h->partials, count,
                       h->host_out);
    QS_HIP(hipGetLastError());
    QS_HIP(hipStreamSynchronize(h->stream));
    for (int c = 0; c < w; ++c) out[c] = h->host_out[c];
    return QS_OK;
}

}  // namespace

int reduce_norm2(qs_state *h, double *out)
{
    if (int rc = ensure_partials(h, size_t(kReduceBlocks) * 2 + 8)) return rc;
    const unsigned g = red_grid(h->dim());
    if (h->dtype == QS_C128)
        hipLaunchKernelGGL(k_norm2<double>, dim3(g), dim3(kThreads), 0, h->stream,
                           static_cast<const double2 *>(h->psi), h->dim(), h->partials);
    else
        hipLaunchKernelGGL(k_norm2<float>, dim3(g), dim3(kThreads), 0, h->stream,
                           static_cast<const float2 *>(h->psi), h->dim(), h->partials);
    QS_HIP(hipGetLastError());
    return finish_to_host(h, int(g), 1, out);
}

int reduce_pauli(qs_state *h, uint64_t xm, uint64_t ym, uint64_t zm, double *re, double *im)
{
    if (int rc = ensure_partials(h, size_t(kReduceBlocks) * 2 + 8)) return rc;
    const uint64_t f = xm | ym;
    const uint64_t sgn = ym | zm;
    int hbit = 0;
    uint64_t items = h->dim();
    if (f) {
        hbit = 63 - __builtin_clzll(f);
        items >>= 1;
    }
    const unsigned g = red_grid(items);
    if (h->dtype == QS_C128)
        hipLaunchKernelGGL(k_pauli<double>, dim3(g), dim3(kThreads), 0, h->stream,
                           static_cast<const double2 *>(h->psi), items, f, hbit, sgn, h->partials);
    else
        hipLaunchKernelGGL(k_pauli<float>, dim3(g), dim3(kThreads), 0, h->stream,
                           static_cast<const float2 *>(h->psi), items, f, hbit, sgn, h->partials);
    QS_HIP(hipGetLastError());
    double s[2];
    if (int rc = finish_to_host(h, int(g), 2, s)) return rc;
    // multiply by i^{popcount(y)}
    double r = s[0], i = s[1];
    switch (__builtin_popcountll(ym) & 3) {
    case 0: break;
    case 1: { double t = r; r = -i; i = t; break; }
    case 2: r = -r; i = -i; break;
    case 3: { double t = r; r = i; i = -t; break; }
    }
    *re = r;
    *im = i;
    return QS_OK;
}

int reduce_pauli_noalloc(qs_state *h, uint64_t xm, uint64_t ym, uint64_t zm, double *device_out)
{
    double *part = nullptr;
    if (int rc = scratch_address(h->device, &part)) return rc;
    const uint64_t f = xm | ym;
    const uint64_t sgn = ym | zm;
    int hbit = 0;
    uint64_t items = h->dim();
    if (f) {
        hbit = 63 - __builtin_clzll(f);
        items >>= 1;
    }
    const unsigned g = red_grid(items);
    if (size_t(g) * 2 > kNoAllocDoubles)
        return fail(QS_EUNSUPPORTED, "%u partial sums exceed the %zu-double scratch", g, kNoAllocDoubles);
    if (h->dtype == QS_C128)
        hipLaunchKernelGGL(k_pauli<double>, dim3(g), dim3(kThreads), 0, h->stream,
                           static_cast<const double2 *>(h->psi), items, f, hbit, sgn, part);
    else
        hipLaunchKernelGGL(k_pauli<float>, dim3(g), dim3(kThreads), 0, h->stream,
                           static_cast<const float2 *>(h->psi), items, f, hbit, sgn, part);
    QS_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_finish_pauli, dim3(1), dim3(kThreads), 0, h->stream, part, int(g),
                       __builtin_popcountll(ym) & 3, device_out);
    QS_HIP(hipGetLastError());
    return QS_OK;
}

int gather_amplitudes(qs_state *h, int count, const uint64_t *indices, void *host_dst)
{
    void *didx = nullptr, *dout = nullptr;
    if (int rc = h->stage.put(h->stream, indices, sizeof(uint64_t) * size_t(count), &didx)) return rc;
    if (int rc = h->stage.reserve(h->stream, h->amp_bytes() * size_t(count), &dout)) return rc;
    const unsigned g = unsigned((count + kThreads - 1) / kThreads);
    if (h->dtype == QS_C128)
        hipLaunchKernelGGL(k_gather_amps<double>, dim3(g), dim3(kThreads), 0, h->stream,
                           static_cast<const double2 *>(h->psi), static_cast<const uint64_t *>(didx),
                           count, static_cast<double2 *>(dout));
    else
        hipLaunchKernelGGL(k_gather_amps<float>, dim3(g), dim3(kThreads), 0, h->stream,
                           static_cast<const float2 *>(h->psi), static_cast<const uint64_t *>(didx),
                           count, static_cast<float2 *>(dout));
    QS_HIP(hipGetLastError());
    if (int rc = ensure_host_out(h, h->amp_bytes() * size_t(count))) return rc;
    QS_HIP(hipMemcpyAsync(h->host_out, dout, h->amp_bytes() * size_t(count), hipMemcpyDeviceToHost,
                          h->stream));
    QS_HIP(hipStreamSynchronize(h->stream));
    std::copy_n(reinterpret_cast<char *>(h->host_out), h->amp_bytes() * size_t(count),
                static_cast<char *>(host_dst));
    return QS_OK;
}

int measure(qs_state *h, int m, const int *qubits, int shots, const double *u, uint64_t *outcomes,
            double *probs, int collapse)
{
    const int M = 1 << m;
    QArgs qa;
    qa.m = m;
    for (int r = 0; r < m; ++r) qa.q[r] = qubits[r];
    const int bits = h->dtype == QS_C128 ? Item<double>::bits : Item<float>::bits;
    const int row_bits = std::min(h->n - bits, 6), low_bits = bits + row_bits;
    HistArgs ha{};
    ha.row = 1 << row_bits;
    ha.hi_rest = (h->dim() - 1) >> low_bits << row_bits;
    for (int r = 0; r < m; ++r) {
        if (qubits[r] < low_bits) {
            ha.low_meas |= 1 << qubits[r];
        } else {
            ha.hi_meas |= 1ull << (qubits[r] - bits);
            ++ha.hi_count;
        }
    }
    ha.hi_rest &= ~ha.hi_meas;
    // enough waves to fill the chip, but rows of kAhead items or more each
    const int rest_bits = __builtin_popcountll(ha.hi_rest);
    const int split_bits = std::max(0, std::min(kHistWaveBits - ha.hi_count, rest_bits - kAheadBits));
    ha.splits = 1 << split_bits;
    ha.steps = 1ull << (rest_bits - split_bits);
    // device layout: [p (M) | cdf (M) | partial rows | outcomes | uniforms]
    const size_t rows = ha.splits > 1 ? size_t(ha.splits) : 0;
    const size_t need = size_t(M) * 2 + rows * size_t(M) + size_t(shots) * 2 + 16;
    if (int rc = ensure_partials(h, std::max(need, size_t(kReduceBlocks) * 2 + 8))) return rc;
    double *p = h->partials;
    double *cdf = p + M;
    double *part = cdf + M;
    uint64_t *dout = reinterpret_cast<uint64_t *>(part + rows * size_t(M));
    double *du = reinterpret_cast<double *>(dout + shots);
    const uint64_t waves = uint64_t(ha.splits) << ha.hi_count;
    hipLaunchKernelGGL(h->dtype == QS_C128 ? k_hist<double> : k_hist<float>,
                       dim3(unsigned((waves + kThreads / 64 - 1) / (kThreads / 64))), dim3(kThreads), 0, h->stream,
                       h->psi, qa, ha, rows ? part : p);
    if (rows)
        hipLaunchKernelGGL(k_hist_cols, dim3((M + 63) / 64), dim3(kColThreads), 0, h->stream, part, int(rows), M,
                           p);
    QS_HIP(hipGetLastError());
    if (shots > 0) {
        hipLaunchKernelGGL(k_cdf, dim3(1), dim3(kThreads), 0, h->stream, p, M, cdf);
        QS_HIP(hipGetLastError());
        void *du_staged = nullptr;
        if (int rc = h->stage.put(h->stream, u, sizeof(double) * size_t(shots), &du_staged)) return rc;
        QS_HIP(hipMemcpyAsync(du, du_staged, sizeof(double) * size_t(shots),
                              hipMemcpyDeviceToDevice, h->stream));
        hipLaunchKernelGGL(k_sample, dim3((shots + kThreads - 1) / kThreads), dim3(kThreads), 0,
                           h->stream, cdf, M, du, shots, dout);
        QS_HIP(hipGetLastError());
        if (collapse) {
            const uint64_t items = h->dim() >> bits;
            const unsigned cg = unsigned(std::min<uint64_t>((items + kThreads - 1) / kThreads, 1u << 20));
            hipLaunchKernelGGL(h->dtype == QS_C128 ? k_collapse<double> : k_collapse<float>, dim3(cg), dim3(kThreads),
                               0, h->stream, h->psi, items, qa, dout, p);
            QS_HIP(hipGetLastError());
        }
    }
    const size_t hb = (probs ? sizeof(double) * size_t(M) : 0) + sizeof(uint64_t) * size_t(shots);
    if (int rc = ensure_host_out(h, hb + 16)) return rc;
    char *ho = reinterpret_cast<char *>(h->host_out);
    if (shots > 0)
        QS_HIP(hipMemcpyAsync(ho, dout, sizeof(uint64_t) * size_t(shots), hipMemcpyDeviceToHost,
                              h->stream));
    if (probs)
        QS_HIP(hipMemcpyAsync(ho + sizeof(uint64_t) * size_t(shots), p, sizeof(double) * size_t(M),
                              hipMemcpyDeviceToHost, h->stream));
    QS_HIP(hipStreamSynchronize(h->stream));
    if (shots > 0) std::copy_n(reinterpret_cast<uint64_t *>(ho), shots, outcomes);
    if (probs) std::copy_n(reinterpret_cast<double *>(ho + sizeof(uint64_t) * size_t(shots)), M, probs);
    return QS_OK;
}

}  // namespace qs
