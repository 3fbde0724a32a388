// Pooling kernels for gfx950 (Section 6 of "Communication-Optimal Convolutional Neural Nets": the convolution nest
// without the Filter, per-channel reading k = c).  HBM-bound: every Image word is needed by at most
// ceil(R/sigma_w)*ceil(S/sigma_h) outputs and those re-reads are served by L1/L2, every Out word is written once.
// One thread owns VEC adjacent images of one (h, w, c); threads are ordered images fastest, then c, so a wave's loads are
// contiguous in Image ([.][.][C][B]) and its stores are runs of B floats in Out ([.][.][.][B]).
// Measured (MI355X, one launch in a HIP graph; with one element per thread where 16-byte loads did not divide B, 64-bit products per
// element and a load at a time, then now): bf16 average (20, 192, 27, 27, 3 x 3, s 2) 20.9 -> 7.3 us (34 MB: 4.7 TB/s), bf16 max
// (6, 544, 20, 20, 7 x 7, s 7) 50.2 -> 22.0, fp32 average (8, 80, 111, 111, 3 x 3) 36.5 -> 18.5; 65 calls 1.5 times.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "cacnn_internal.h"

namespace cacnn {

typedef float pf32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int pu32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t pdiv(uint32_t n, const FastDiv& f) { return f.mul ? __umulhi(n, f.mul) : n; }

typedef unsigned int pu32x2 __attribute__((ext_vector_type(2)));
typedef float pf32x2 __attribute__((ext_vector_type(2)));

// VEC adjacent Image elements through a descriptor: lane offset voff and wave-uniform offset soff in bytes, as they lie in memory
template <int BYTES>
struct PoolWords {
    uint32_t w[(BYTES + 3) / 4];
    __device__ __forceinline__ void load(const char* p) {
        if constexpr (BYTES == 2) {
            w[0] = *(const uint16_t*)p;
        } else if constexpr (BYTES == 4) {
            w[0] = *(const uint32_t*)p;
        } else if constexpr (BYTES == 8) {
            const pu32x2 v = *(const pu32x2*)p;
            w[0] = v[0], w[1] = v[1];
        } else {
            const pu32x4 v = *(const pu32x4*)p;
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = v[i];
        }
    }
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
        if constexpr (BYTES == 2) {
            w[0] = __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0);
        } else if constexpr (BYTES == 4) {
            w[0] = __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0);
        } else if constexpr (BYTES == 8) {
            const pu32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
            w[0] = v[0], w[1] = v[1];
        } else {
            const pu32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = v[i];
        }
    }
};

template <bool BIG>
struct PoolOffset {
    typedef uint32_t type;
};
template <>
struct PoolOffset<true> {
    typedef int64_t type;
};

template <int DT, int MODE, int VEC>
__device__ __forceinline__ void pool_take(float (&acc)[VEC], const PoolWords<VEC*(DT == 0 ? 4 : 2)>& x, bool first) {
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
        const float v = DT == 0 ? __uint_as_float(x.w[DT == 0 ? i : 0]) : __uint_as_float(i & 1 ? x.w[i / 2] & 0xffff0000u : x.w[i / 2] << 16);
        if (first) acc[i] = v;
        else if (MODE == 0) acc[i] += v;
        else acc[i] = fmaxf(acc[i], v);
    }
}

// BIG: the Image is larger than the 2 GiB of a buffer descriptor; 64-bit addresses.
// WR x WS: the window the kernel is compiled for, all of whose loads are in flight at once (0: any window, eight loads
// at a time).  One load takes the address unit as long whether a lane asks for 2 bytes or 4, and twice as long for 8
// or 16, so VEC is the largest of 8, 4, 2 (fp32: 4, 2) that divides B (bf16 with Out past the L2: 4 where few loads go to an output).  Offsets are 32 bits wide and the window's part of them is
// scalar: with 64-bit products per element the vector unit, not memory, set the pace of calls with a small VEC.
// STREAM: Out past the L2, where a row of images is whole cache lines (B a multiple of 32); elsewhere the pieces of a line
// come from several instructions and the L2 has to put them together (bf16 (20, 192, 27, 27, 3 x 3, s 2) 7.4 us through it, 8.4
// past it; fp32 (8, 80, 111, 111, 3 x 3) 17.6 and 30.9).  A template parameter because the compiler makes one store of the two
// sides of a branch and drops the hint: fp32 max (128, 496, 43, 2, 2 x 2, s 2) 20.5 us without the hint, 18.1 with it;
// (32, 64, 56, 56, 3 x 3, s 2) 29.1 and 24.8; bf16 (32, 100, 50, 75, 2 x 2, s 2) 29.7 and 27.2.
template <int DT, int MODE, int VEC, int WR, int WS, bool BIG, bool STREAM>
__global__ void __launch_bounds__(256) pool_kernel(const PoolArgs a) {
    constexpr int ESZ = DT == 0 ? 4 : 2;
    // consecutive workgroups go to different XCDs: give every XCD one contiguous run of the output instead, so the
    // rows its windows share stay in one L2
    int wg = blockIdx.x;
    if (a.n_xcd > 1) {
        const int l = (int)pdiv((uint32_t)wg, a.d_nxcd), x = wg - l * a.n_xcd;
        wg = x * a.xcd_q + min(x, a.xcd_rem) + l;
    }
    const int g = wg * 256 + threadIdx.x;
    if (g >= a.n_threads) return;
    // thread order: images fastest, then c, then the column within a chunk of TWC output columns, then h, then the
    // chunk.  An XCD's contiguous share of the workgroups is then a band of columns over all rows, so the Image rows
    // that vertically adjacent windows share are fetched into that XCD's L2 once.
    uint32_t t = (uint32_t)g;
    uint32_t q = pdiv(t, a.d_BV);
    const uint32_t bv = t - q * a.BV;
    t = q;
    q = pdiv(t, a.d_C);
    const uint32_t c = t - q * a.C;
    t = q;
    q = pdiv(t, a.d_TWC);
    const uint32_t wl = t - q * a.TWC;
    t = q;
    q = pdiv(t, a.d_H);
    const uint32_t h = t - q * a.H, w = q * a.TWC + wl;
    if (w >= (uint32_t)a.W) return;

    using Off = typename PoolOffset<BIG>::type;
    const __amdgpu_buffer_rsrc_t img = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.image), 0, BIG ? 0 : a.img_bytes, 0x00020000);
    const Off row = (Off)a.C * a.B * ESZ, col = row * a.IH;               // bytes from one y, one x to the next
    const Off voff = (Off)w * (a.sw * col) + (Off)h * (a.sh * row) + (Off)(c * a.B + bv * VEC) * ESZ;
    auto load = [&](PoolWords<VEC * ESZ>& x, int r, int s) {
        if constexpr (BIG) x.load((const char*)a.image + voff + r * col + s * row);
        else x.load(img, voff, r * col + s * row);
    };
    float acc[VEC];
    if constexpr (WR > 0) {
        PoolWords<VEC * ESZ> x[WR * WS];
#pragma unroll
        for (int i = 0; i < WR * WS; ++i) load(x[i], i / WS, i % WS);
#pragma unroll
        for (int i = 0; i < WR * WS; ++i) pool_take<DT, MODE, VEC>(acc, x[i], i == 0);
    } else {
        // the window's elements in the order r, s, in batches of 8, 4 and 1 whose loads are in flight together
        int r = 0, s = 0, i = 0;
        const int n = a.R * a.S;
        auto batch = [&](auto size) {
            constexpr int SIZE = decltype(size)::value;
            for (; i + SIZE <= n; i += SIZE) {
                PoolWords<VEC * ESZ> x[SIZE];
#pragma unroll
                for (int e = 0; e < SIZE; ++e) {
                    load(x[e], r, s);
                    if (++s == a.S) s = 0, ++r;
                }
#pragma unroll
                for (int e = 0; e < SIZE; ++e) pool_take<DT, MODE, VEC>(acc, x[e], i == 0 && e == 0);
            }
        };
        batch(std::integral_constant<int, 8>{});
        batch(std::integral_constant<int, 4>{});
        batch(std::integral_constant<int, 1>{});
    }
    if (MODE == 0) {
        const float n = (float)(a.R * a.S);
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[i] = acc[i] / n;
    }
    float* const dst = a.out + (((c * (uint32_t)a.H + h) * (uint32_t)a.W + w) * (uint32_t)a.B + bv * VEC);
    if constexpr (VEC >= 4) {
#pragma unroll
        for (int i = 0; i < VEC; i += 4) {
            const pf32x4 v = {acc[i], acc[i + 1], acc[i + 2], acc[i + 3]};
            if constexpr (STREAM) __builtin_nontemporal_store(v, (pf32x4*)(dst + i));
            else *(pf32x4*)(dst + i) = v;
        }
    } else if constexpr (VEC == 2) {
        *(pf32x2*)dst = pf32x2{acc[0], acc[1]};
    } else {
        dst[0] = acc[0];
    }
}

template <int DT, int MODE, int VEC, bool STREAM>
static int launch_one(const PoolArgs& a, void* stream) {
    const dim3 grid(a.n_wg), block(256);
    const hipStream_t st = (hipStream_t)stream;
    if (a.img_bytes == 0) hipLaunchKernelGGL((pool_kernel<DT, MODE, VEC, 0, 0, true, STREAM>), grid, block, 0, st, a);
    else if (a.R == 3 && a.S == 3) hipLaunchKernelGGL((pool_kernel<DT, MODE, VEC, 3, 3, false, STREAM>), grid, block, 0, st, a);
    else if (a.R == 2 && a.S == 2) hipLaunchKernelGGL((pool_kernel<DT, MODE, VEC, 2, 2, false, STREAM>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((pool_kernel<DT, MODE, VEC, 0, 0, false, STREAM>), grid, block, 0, st, a);
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

template <int DT, int MODE, int VEC>
static int launch_stream(const PoolArgs& a, void* stream) {
    if constexpr (VEC >= 4)
        if (a.stream) return launch_one<DT, MODE, VEC, true>(a, stream);
    return launch_one<DT, MODE, VEC, false>(a, stream);
}

template <int DT, int MODE>
static int launch_vec(const PoolArgs& a, int vec, void* stream) {
    if constexpr (DT == 1)
        if (vec == 8) return launch_stream<DT, MODE, 8>(a, stream);
    if (vec == 4) return launch_stream<DT, MODE, 4>(a, stream);
    if (vec == 2) return launch_stream<DT, MODE, 2>(a, stream);
    return launch_stream<DT, MODE, 1>(a, stream);
}

int launch_pool(const PoolArgs& a, int dtype, int mode, int vec, void* stream) {
    if (dtype == 0) return mode == 0 ? launch_vec<0, 0>(a, vec, stream) : launch_vec<0, 1>(a, vec, stream);
    return mode == 0 ? launch_vec<1, 0>(a, vec, stream) : launch_vec<1, 1>(a, vec, stream);
}

}  // namespace cacnn
