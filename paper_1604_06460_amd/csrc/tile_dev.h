// Device code that the gate passes (tile.hip) and the FFT passes
// (fft_tile.hip) share: a tile of 2^T amplitudes, 16 in each thread's
// registers, and its exchange through LDS.
#pragma once

#include "qs_internal.h"

namespace qs {
namespace tiledev {

template <typename S> struct V2;
template <> struct V2<double> {
    using T = double2;
    typedef double N __attribute__((ext_vector_type(2)));
};
template <> struct V2<float> {
    using T = float2;
    typedef float N __attribute__((ext_vector_type(2)));
};

// LDS slot of tile element e. Linear over XOR, so the slot of a thread's
// register j is the thread's slot XOR a uniform constant; bits p, p + 5 and
// p + 10 of e choose the same pair of banks, and the planner gives the low
// lane bits tile bits that differ modulo 5.
__device__ __forceinline__ uint32_t slot(uint32_t e) { return e ^ ((e >> 5) & 31) ^ ((e >> 10) & 31); }

// Layout of a stage: where the thread's bits and the register bits sit in
// the tile (LDS slots) and in the state (index bits).
// T: tile bits; words: see tile.h, with the register bits' places after those
// of T - 4 thread bits. A tile of fewer bits has its register bits there too:
// thread bits that its workgroup does not have are zero.
template <int T>
struct Layout {
    uint32_t e;         // the thread's tile bits (register bits zero)
    uint64_t idx;       // its index bits in the state
    uint32_t sl;        // LDS byte offset of register 0
    uint32_t rs[4];     // XOR of that by register bit b
    uint64_t ro[4];     // index bit of register bit b
    __device__ __forceinline__ void set(uint64_t base, uint64_t w0, uint64_t w1, uint64_t w2, uint32_t tid)
    {
        e = 0;
        uint64_t a = base;
#pragma unroll
        for (int i = 0; i < T - 4; ++i) {
            const uint32_t b = (tid >> i) & 1;
            e |= b << ((w0 >> (4 * i)) & 15);
            a |= uint64_t(b) << ((w1 >> (6 * i)) & 63);
        }
        idx = a;
        sl = 8 * slot(e);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            rs[b] = 8 * slot(1u << ((w0 >> (4 * (T - 4 + b))) & 15));
            ro[b] = 1ull << ((w2 >> (6 * b)) & 63);
        }
    }
    __device__ __forceinline__ uint32_t at(uint32_t first, int j) const
    {
        return first ^ ((j & 1 ? rs[0] : 0) ^ (j & 2 ? rs[1] : 0) ^ (j & 4 ? rs[2] : 0) ^ (j & 8 ? rs[3] : 0));
    }
    __device__ __forceinline__ uint64_t off(int j) const
    {
        return (j & 1 ? ro[0] : 0) + (j & 2 ? ro[1] : 0) + (j & 4 ? ro[2] : 0) + (j & 8 ? ro[3] : 0);
    }
};

// The tile from the registers of layout L to those of layout M, through
// 8 * 2^T bytes of LDS.
template <typename S, int T>
__device__ __forceinline__ void exchange_tile(double (&xr)[16], double (&xi)[16], char *lds, const Layout<T> L,
                                              const Layout<T> M)
{
    // the thread's offsets are opaque per half-exchange: the compiler
    // would keep all 32 of them in registers and spill the tile
    auto write = [&](auto &&put) {
        uint32_t first = L.sl;
        asm volatile("" : "+v"(first));
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 16; ++j) put(lds + L.at(first, j), j);
    };
    auto read = [&](auto &&get) {
        uint32_t first = M.sl;
        asm volatile("" : "+v"(first));
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 16; ++j) get(lds + M.at(first, j), j);
    };
    if constexpr (sizeof(S) == 8) {
        // real parts, then imaginary parts: half the LDS, so that two
        // workgroups (T = 13) share a compute unit
        write([&](char *p, int j) { *reinterpret_cast<double *>(p) = xr[j]; });
        read([&](char *p, int j) { xr[j] = *reinterpret_cast<double *>(p); });
        write([&](char *p, int j) { *reinterpret_cast<double *>(p) = xi[j]; });
        read([&](char *p, int j) { xi[j] = *reinterpret_cast<double *>(p); });
    } else {
        write([&](char *p, int j) { *reinterpret_cast<float2 *>(p) = float2{float(xr[j]), float(xi[j])}; });
        read([&](char *p, int j) {
            const float2 v = *reinterpret_cast<float2 *>(p);
            xr[j] = double(v.x);
            xi[j] = double(v.y);
        });
    }
}

}  // namespace tiledev
}  // namespace qs
