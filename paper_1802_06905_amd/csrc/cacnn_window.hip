// gfx950 bf16 kernels that keep the window of a tile's positions in LDS: the Image is staged as it lies in memory, a box of columns x and rows
// y with all their channels, and every filter tap reads its operands out of the same box.  They are for the first layers of a
// network, whose C * S rows per filter column are few and whose filters are large: the flattened kernels stage the Image once per tap there, in
// runs of 16 to 64 bytes; here a word comes once per tile, in runs of a whole column, which is what Section 4.3's small-filter reuse
// amounts to inside LDS.
//
// A tile is KT output channels and WN * NB * 32 columns, TW x TH positions (powers of two) of TB images.  The box is nx = sigma_w (TW - 1) + R
// by ny = sigma_h (TH - 1) + S positions; LDS holds its rows of TB images in the order of the Image, [x][y][c].  For a position at (w, h) of the
// tile and a filter column r, the contraction indices (s, c) are S * C consecutive rows from ((sigma_w w + r) ny + sigma_h h) C on,
// so the contraction is cut into chunks of 8 rows (the last of a column moved back to end with it, and masked), and an MFMA operand is two
// transposing LDS reads of four rows each at a lane's own position: nothing is decoded in the loop, any filter and strides will do.
// A workgroup keeps its Filter tile in LDS and walks position tiles, one box ahead (bufs = 2), or takes one tile (bufs = 1).
//
// Data goes to LDS by buffer loads with LDS destination, 64 lanes x 16 bytes each, which are in flight under the products (cacnn_lds_load.h).
//
// Measured (us, flattened kernel before): (16, 3, 64, 112, 112, 7 x 7, s 2) 19.6 -> 15.8, 32 images 33.4 -> 29.5, (128, 3, 32, 89, 89, 5 x 5, s 2)
// 56.7 -> 30.9, (256, 3, 16, 98, 98, 5 x 5) 81.2 -> 42.2.  What is left is Out, 51 MB of the first one's 56, the 1.7 us before the first product (the
// Filter tile, the lanes' places in the box), and a last round of tiles that is not full.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cacnn_internal.h"
#include "cacnn_lds_load.h"

namespace cacnn {

typedef float wf32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int wu32x4 __attribute__((ext_vector_type(4)));
typedef short ws16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 wbf16x8 __attribute__((ext_vector_type(8)));
#define WIN_LDS(T) __attribute__((address_space(3))) T
struct __attribute__((packed, aligned(2))) WinBytes16 {
    wu32x4 v;
};

// a descriptor of the `left` bytes from p on: loads beyond them return zeros
__device__ __forceinline__ i32x4 window_rsrc(const char* p, uint32_t left) {
    const uint64_t a = (uint64_t)p;
    i32x4 d;
    d[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    d[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32) & 0xffff);
    d[2] = __builtin_amdgcn_readfirstlane((int)left);
    d[3] = 0x00020000;
    return d;
}
__device__ __forceinline__ void window_loads_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

template <int MB, int NB, int WM, int WN, int TB, bool STREAM>
__global__ void __launch_bounds__(WM* WN * 64) conv_window_kernel(const WindowArgs a) {
    constexpr int THREADS = WM * WN * 64, WAVES = WM * WN, KT = WM * MB * 32, ROW = TB * 2;
    static_assert(TB == 8 || TB == 16 || TB == 32, "window kernel: images of a tile");
    extern __shared__ __align__(16) char s_mem[];
    const uint32_t lds = (uint32_t)(uintptr_t)(WIN_LDS(char)*)s_mem;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int j = lane & 31, g = lane >> 5, i16 = lane & 15, jhalf = (lane >> 4) & 1;

    // this workgroup's tile of output channels and first tile of positions; others follow at a distance of t_step
    const uint32_t t0 = xcd_order(blockIdx.x, a.xcd_q, a.xcd_rem);
    uint32_t tk, tn;
    {
        const uint32_t q = flat_div(t0, a.d_inner), i = t0 - q * a.inner;
        tk = a.k_inner ? i : q;
        tn = a.k_inner ? q : i;
    }
    const uint32_t k0 = tk * KT;
    struct Tile {
        uint32_t b0, h0, w0;
    };
    auto tile_at = [&](uint32_t t) {                   // images fastest, then rows, then columns
        const uint32_t q = flat_div(t, a.d_tb), w = flat_div(q, a.d_th);
        return Tile{(t - q * a.tiles_b) * TB, (q - w * a.tiles_h) << a.th_shift, w << a.tw_shift};
    };

    // 8 rows of zeros, for the chunks that make the number of steps even
    const uint32_t zeros = lds + a.zeros + (i16 >> 2) * ROW;
    if (tid < 8 * ROW / 16) *(wu32x4*)(s_mem + a.zeros + tid * 16) = wu32x4{0, 0, 0, 0};

    // ---- staging: the lane's places in the box
    uint32_t ioff[kWindowItems];
#pragma unroll
    for (int i = 0; i < kWindowItems; ++i) {
        const uint32_t item = (wave + i * WAVES) * 64 + lane, row = item / (TB / 8), piece = item % (TB / 8);
        const uint32_t x = flat_div(row, a.d_plane);
        ioff[i] = row < a.rows ? x * a.img_x + (row - x * a.plane) * (a.B * 2) + piece * 16 : 0x80000000u;
    }
    auto fetch = [&](Tile t, uint32_t dst) {
        const uint32_t org = t.w0 * a.img_w + t.h0 * a.img_h + t.b0 * 2;
        const i32x4 d = window_rsrc((const char*)a.image + org, a.img_bytes - org);
#pragma unroll
        for (int i = 0; i < kWindowItems; ++i)
            if (i < (int)a.img_items) load_to_lds_unseen(d, ioff[i], dst + (wave + i * WAVES) * 1024);
    };

    // ---- multiplication
    wf32x16 acc[MB][NB];
    auto clear = [&] {
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[m][n][v] = 0.f;
    };
    // the lane's row and four images (columns 4 (i16 % 4).. of a half block) of chunk 0 at its position
    uint32_t xl[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        const uint32_t col = (wn * NB + n) * 32 + jhalf * 16 + (i16 & 3) * 4, p = col / TB, b = col % TB;
        const uint32_t w = p & ((1u << a.tw_shift) - 1), h = p >> a.tw_shift;
        xl[n] = ((w * a.sw * a.plane + h * a.sh * a.C) + (i16 >> 2)) * ROW + b * 2;
    }
    const uint32_t al = ((wm * MB * 32 + j) * a.UP + g) * 16;
    auto multiply = [&](uint32_t img, uint32_t flt) {
        const uint32_t r0 = flat_div(g, a.d_TC);
        uint32_t i = g - r0 * a.TC, off = img + r0 * a.off_r + i * (8 * ROW), fa = flt + al, u = g;
        wu32x4 A[2][MB], X[2][NB], keep[2];
        auto load = [&](int set) {
#pragma unroll
            for (int m = 0; m < MB; ++m) A[set][m] = *(WIN_LDS(wu32x4)*)(uintptr_t)(fa + m * 32 * a.UP * 16);
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                // (chunks behind the last one: zeros for both operands)
                const uint32_t p = u < a.U ? xl[n] + off - (i + 1 == a.TC ? a.back * ROW : 0u) : zeros;
                const ws16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((WIN_LDS(ws16x4)*)(uintptr_t)p);
                const ws16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((WIN_LDS(ws16x4)*)(uintptr_t)(p + 4 * ROW));
                X[set][n] = __builtin_bit_cast(wu32x4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
            const uint32_t drop = i + 1 == a.TC ? a.back : 0u;
#pragma unroll
            for (uint32_t d = 0; d < 4; ++d) keep[set][d] = (2 * d >= drop ? 0xffffu : 0u) | (2 * d + 1 >= drop ? 0xffff0000u : 0u);
            fa += 32;
            u += 2;
            i += a.adv_i;
            off += a.adv_off;
            if (i >= a.TC) {
                i -= a.TC;
                off += a.wrap_off;
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto products = [&](int set) {
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int d = 0; d < 4; ++d) X[set][n][d] &= keep[set][d];
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int n = 0; n < NB; ++n)
                    acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(wbf16x8, A[set][m]), __builtin_bit_cast(wbf16x8, X[set][n]), acc[m][n], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
        // A step's operands are read under the products of the step before.  (An even number of steps, without a way out in
        // between: with one the compiler moved all accumulators to other registers and back for every tile.)
        load(0);
        for (uint32_t st = 0; st < a.steps; st += 2) {
            load(1);
            products(0);
            load(0);
            products(1);
        }
    };

    // MFMA D layout: lane j + 32 g holds rows 8 (v / 4) + 4 g + v % 4 of column j.  A row's address is scalar, the lane's offset 32 bits.
    auto store = [&](Tile t) {
        const uint32_t kw = k0 + wm * MB * 32;
        const int rows = (int)(a.K - kw) - 4 * g;          // of the wave's, from the lane's first on
        const bool whole = kw + MB * 32 <= a.K;
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            const uint32_t col = (wn * NB + n) * 32 + j, p = col / TB, b = t.b0 + col % TB;
            const uint32_t w = t.w0 + (p & ((1u << a.tw_shift) - 1)), h = t.h0 + (p >> a.tw_shift);
            if (w < a.W && h < a.H && b < a.B) {
                const uint32_t off = (4 * g * a.N + (h * a.W + w) * a.B + b) * 4;
#pragma unroll
                for (int m = 0; m < MB; ++m)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int row = m * 32 + (v >> 2) * 8 + (v & 3);
                        float* const dst = (float*)((char*)(a.out + (int64_t)(kw + row) * a.N) + off);
                        if (whole || row < rows) {
                            if constexpr (STREAM) __builtin_nontemporal_store(acc[m][n][v], dst);
                            else *dst = acc[m][n][v];
                        }
                    }
            }
        }
    };

    const uint32_t flt = lds, img0 = lds + a.flt_lds;
    uint32_t next = tn;
    Tile t = tile_at(next);
    fetch(t, img0);
    // the Filter tile: chunks of 8 of the S * C elements of an output channel's column r, the last of a column moved back to end with it and
    // without the elements that the chunk before it has as well; zeros behind the last chunk and beyond K
    constexpr int AT_ONCE = 4;
    for (uint32_t first = tid; first < KT * a.UP; first += AT_ONCE * THREADS) {
        wu32x4 v[AT_ONCE];
        uint32_t drop[AT_ONCE];
#pragma unroll
        for (int q = 0; q < AT_ONCE; ++q) {
            const uint32_t item = first + q * THREADS, k = flat_div(item, a.d_UP), u = item - k * a.UP, r = flat_div(u, a.d_TC), i = u - r * a.TC;
            const bool in = k < KT && k0 + k < a.K && u < a.U;
            const uint32_t back = i + 1 == a.TC ? a.back : 0u;
            drop[q] = in ? back : 8u;
            v[q] = ((const WinBytes16*)((const char*)a.filter + (in ? (k0 + k) * a.flt_k + r * a.flt_tap + i * 16 - back * 2 : 0u)))->v;
        }
#pragma unroll
        for (int q = 0; q < AT_ONCE; ++q) {
            if (first + q * THREADS < KT * a.UP) {
#pragma unroll
                for (uint32_t d = 0; d < 4; ++d) v[q][d] &= (2 * d >= drop[q] ? 0xffffu : 0u) | (2 * d + 1 >= drop[q] ? 0xffff0000u : 0u);
                *(wu32x4*)(s_mem + (first + q * THREADS) * 16) = v[q];
            }
        }
    }
    window_loads_done();
    __syncthreads();
    for (uint32_t buf = 0;; buf ^= 1) {
        const Tile now = t;
        next += a.t_step;
        const bool more = next < a.tiles_n;
        if (more) {
            t = tile_at(next);
            fetch(t, img0 + (buf ^ 1) * a.img_lds);
        }
        clear();
        multiply(img0 + buf * a.img_lds, flt);
        if (!more) {
            store(now);
            return;
        }
        // (the loads of the next box, and this wave's stores of the tile before, which had these products' time)
        window_loads_done();
        __syncthreads();
        store(now);
    }
}

template <int MB, int NB, int WM, int WN, int TB, bool STREAM>
static int launch_window_as(const WindowArgs& a, int grid, size_t lds, void* stream) {
    auto kernel = conv_window_kernel<MB, NB, WM, WN, TB, STREAM>;
    if (lds > 64 * 1024) {
        static OncePerDevice once;
        int device = -1;
        if (hipGetDevice(&device) != hipSuccess || !once(device, [&] {
                return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) == hipSuccess;
            })) {
            (void)hipGetLastError();
            return 1;
        }
    }
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(WM * WN * 64), lds, (hipStream_t)stream, a);
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

// Out past the L2 where every store writes whole halves of cache lines
template <int MB, int NB, int WM, int WN, int TB>
static int launch_window(const WindowArgs& a, int grid, size_t lds, void* stream) {
    if constexpr (TB >= 16)
        if (a.B % TB == 0 && (TB == 32 || a.B == 16) && a.N % 32 == 0 && reinterpret_cast<uintptr_t>(a.out) % 64 == 0)
            return launch_window_as<MB, NB, WM, WN, TB, true>(a, grid, lds, stream);
    return launch_window_as<MB, NB, WM, WN, TB, false>(a, grid, lds, stream);
}

#define CACNN_WINDOW(MB, NB, WM, WN, TB) \
    {{MB, NB, WM, WN, TB}, launch_window<MB, NB, WM, WN, TB>}
// blocks of 32 output channels and of 32 columns of one wave; waves along output channels and columns; images of a tile.  (Tiles of 32 x 256:
// over 79 first layers of 10 us and more 1.07 of the time of the best of this and 64 x 128, 64 x 256 by four and by eight waves, 32 x 128 in the
// geometric mean; each of those alone 1.15 to 1.23.)
static const WindowVariant g_window[] = {
    CACNN_WINDOW(1, 2, 1, 4, 8),
    CACNN_WINDOW(1, 2, 1, 4, 16),
    CACNN_WINDOW(1, 2, 1, 4, 32),
};

int num_window() { return (int)(sizeof(g_window) / sizeof(g_window[0])); }
const WindowVariant& window_variant(int i) { return g_window[i]; }

}  // namespace cacnn
