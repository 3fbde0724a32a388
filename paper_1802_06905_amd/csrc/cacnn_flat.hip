// gfx950 kernels with flattened positions: the convolution as one matrix product Out[K x N] = Filter[K x Q] * Window[Q x N]
// with N = H*W*B positions and Q = R*S*C contraction indices, for problems that the tiled kernels (cacnn_kernels.hip) leave
// mostly idle or cannot stage: few images, batches and channel counts that 16-byte items do not divide, few outputs.
//
// Out[k] is N consecutive words and Filter[k] is Q consecutive elements whatever the sizes are.  A window element's place is
// a sum, base(position) + r * row(r) + (s*C + c) * B, because y and c are neighbouring axes of the Image: so a lane keeps
// the offset of its position, the step through the contraction is a scalar or one shared vector add, nothing is padded
// and nothing is decoded in the loop.  Positions are cut into tiles wherever they end: 32 columns of an MFMA block are 32
// positions (or 32 groups of images) in a row, whatever B, W and H are.
//
// Two kernels.  The first takes every operand from global memory (L1 and L2 hold the windows' overlap) straight to the
// registers of the wave that multiplies it, several steps ahead, with no barrier.  It is bound by the compute unit's
// address unit: a load whose 64 lanes fall into many cache lines takes about a clock for each of them, which is why a lane
// loads several images at once where it can.  The second stages both operands in LDS with loads that
// run along memory, so that the address unit sees each byte of a tile once (it moves 64 bytes a clock then) instead of once
// per wave in pieces of 32 bytes: 1.2 to 3 times faster for bf16, whose products are short, level for fp32.
// Where there are few tiles the waves of a workgroup divide the contraction and add up in LDS at the end.
//
// Measured against the kernels that ran these calls before (one launch, MI355X; direct, then staged):
//   fp32 (5, 30, 50, 27, 19, 5 x 5)         109.7 -> 11.3 / 9.3 us       bf16 (1, 128, 128, 28, 28, 3 x 3)    46.0 -> 6.8 / 5.0 us
//   bf16 (16, 3, 64, 112, 112, 7 x 7, s 2)  349 -> 28.1 / 20.4 us        bf16 (3, 367, 237, 15, 15, 3 x 3)   310 -> 53 / 22.8 us
// (the first of the second row runs on cacnn_window.hip now, 16.2 us)
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cacnn_internal.h"

namespace cacnn {

typedef float ff32x16 __attribute__((ext_vector_type(16)));
typedef float ff32x4 __attribute__((ext_vector_type(4)));
typedef float ff32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int fu32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int fu32x2 __attribute__((ext_vector_type(2)));
typedef short fs16x4 __attribute__((ext_vector_type(4)));
#define FLAT_LDS(T) __attribute__((address_space(3))) T
typedef __bf16 fbf16x8 __attribute__((ext_vector_type(8)));

// BYTES bytes (2, 4, 8 or 16) at any element-aligned address: base is wave-uniform, off the lane's
typedef unsigned short fu16;
struct __attribute__((packed, aligned(2))) Bytes4 {
    uint32_t v;
};
struct __attribute__((packed, aligned(2))) Bytes8 {
    fu32x2 v;
};
struct __attribute__((packed, aligned(2))) Bytes16 {
    fu32x4 v;
};
struct __attribute__((packed, aligned(4))) Out2 {
    ff32x2 v;
};
struct __attribute__((packed, aligned(4))) Out4 {
    ff32x4 v;
};
template <int BYTES>
__device__ __forceinline__ void load_at(uint32_t* to, const char* base, uint32_t off) {
    if constexpr (BYTES == 2) {
        to[0] = *(const fu16*)(base + off);
    } else if constexpr (BYTES == 4) {
        to[0] = ((const Bytes4*)(base + off))->v;
    } else if constexpr (BYTES == 8) {
        const fu32x2 v = ((const Bytes8*)(base + off))->v;
        to[0] = v[0], to[1] = v[1];
    } else {
        const fu32x4 v = ((const Bytes16*)(base + off))->v;
        to[0] = v[0], to[1] = v[1], to[2] = v[2], to[3] = v[3];
    }
}

// the same through a buffer descriptor: the scalar offset soff costs no vector instruction
template <int BYTES>
__device__ __forceinline__ void load_image(uint32_t* to, __amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    if constexpr (BYTES == 2) {
        to[0] = __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0);
    } else if constexpr (BYTES == 4) {
        to[0] = __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0);
    } else if constexpr (BYTES == 8) {
        const fu32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
        to[0] = v[0], to[1] = v[1];
    } else {
        const fu32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
        to[0] = v[0], to[1] = v[1], to[2] = v[2], to[3] = v[3];
    }
}

// The exchange of partial sums at the end of a tile: rows of a block per round, and the LDS it takes
template <int MB, int NG, int IPL, int TILES, int WK>
struct FlatReduce {
    static constexpr int bytes(int vs) { return TILES * WK * IPL * vs * 256; }
    static constexpr int VS = bytes(16) <= (MB * NG == 1 ? 65536 : 32768) ? 16 : bytes(8) <= 32768 ? 8 : 4;
    static constexpr int ROUNDS = MB * NG * (16 / VS);
    static constexpr int BUF = bytes(VS) / 4;                       // floats of one buffer
    static constexpr size_t BYTES = WK == 1 ? 0 : (size_t)(ROUNDS > 1 ? 2 : 1) * bytes(VS);
};

// Hands a wave's sums (NG groups of IPL column blocks) to store(m, group, row, IPL values); with WK > 1 the partial sums of the
// WK waves of a tile first meet in LDS, VS rows of a block at a time, in two buffers: a buffer is written again two rounds later,
// when every wave has passed the barrier in between and so has read it.
template <int MB, int NG, int IPL, int TILES, int WK, class Store>
__device__ __forceinline__ void flat_write_out(float* s_red, ff32x16 (&acc)[MB][NG * IPL], int wave, int wk, int lane, Store store) {
    using Lay = FlatReduce<MB, NG, IPL, TILES, WK>;
    if constexpr (WK == 1) {
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int v = 0; v < 16; ++v)
#pragma unroll
                for (int p = 0; p < NG; ++p) {
                    float o[IPL];
#pragma unroll
                    for (int q = 0; q < IPL; ++q) o[q] = acc[m][p * IPL + q][v];
                    store(m, p, v, o);
                }
    } else {
        constexpr int VS = Lay::VS, SLOT = IPL * VS * 64;
        float* const grp = s_red + (size_t)(wave / WK) * WK * SLOT + lane;
        int buf = 0;
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int p = 0; p < NG; ++p)
#pragma unroll
                for (int v0 = 0; v0 < 16; v0 += VS) {
                    float* const slot = grp + buf * Lay::BUF;
#pragma unroll
                    for (int v = 0; v < VS; ++v)
#pragma unroll
                        for (int q = 0; q < IPL; ++q) slot[wk * SLOT + (v * IPL + q) * 64] = acc[m][p * IPL + q][v0 + v];
                    __syncthreads();
                    for (int v = wk; v < VS; v += WK) {
                        float o[IPL];
#pragma unroll
                        for (int q = 0; q < IPL; ++q) {
                            float s = 0.f;
#pragma unroll
                            for (int w = 0; w < WK; ++w) s += slot[w * SLOT + (v * IPL + q) * 64];
                            o[q] = s;
                        }
                        store(m, p, v0 + v, o);
                    }
                    buf ^= 1;
                }
    }
}

// A lane holds IM adjacent images of a position and loads them one contraction index at a time.
// SHORT: a filter row (T = S*C indices) is shorter than a chunk, which is one r then; only the T elements that exist are loaded, the
// others stay zero.
// AHEAD: steps whose loads are in flight.  0, for short rows and for waves of one step at most: every load is of a step that is
// multiplied.  The loop of the longer contractions fetches up to 2 AHEAD - 1 steps beyond the last one, and with those and a short row's
// last element repeated up to the end of the chunk, a 1 x 1 layer of one channel took up to 64 times the loads it needs: fp32
// (1, 2, 2, 1059, 1059, 7 x 1) 415 -> 44 us, bf16 (1, 3, 81, 821, 821, 1 x 1) 664 -> 102, (4, 2, 192, 37, 37, 1 x 1) 10.8 -> 4.1, and with
// whole chunks fp32 (7, 4, 136, 90, 39, 1 x 1) 10.8 -> 7.2, bf16 (3, 8, 176, 8, 8, 1 x 1) 5.3 -> 2.6.
template <int DT, int MB, int NG, int IM, int WM, int WN, int WK, int AHEAD, bool SHORT>
__global__ void __launch_bounds__(WM* WN* WK * 64) conv_flat_kernel(const FlatArgs a) {
    constexpr int ESZ = DT == 0 ? 4 : 2, CH = 16 / ESZ;
    static_assert(IM == 1 || IM == 2 || IM == 4, "flat kernel: images per lane that one load and one store take");
    static_assert(!SHORT || AHEAD == 0, "flat kernel: short rows have no steps ahead");
    constexpr int NB = NG * IM;                        // column blocks per wave
    constexpr int LW = (IM * ESZ + 3) / 4;             // dwords of one Image load
    constexpr int D = AHEAD ? AHEAD : 1;               // steps of operands in registers
    extern __shared__ __align__(16) float s_red[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave % WK, wm = (wave / WK) % WM, wn = wave / (WK * WM);
    const int j = lane & 31, g = lane >> 5;

    const uint32_t t = xcd_order(blockIdx.x, a.xcd_q, a.xcd_rem);
    uint32_t tk, tn;
    {
        const uint32_t q = flat_div(t, a.d_inner), i = t - q * a.inner;
        tk = a.k_inner ? i : q;
        tn = a.k_inner ? q : i;
    }
    const uint32_t k0 = (tk * WM + wm) * (MB * 32), q0 = (tn * WN + wn) * (NG * 32);

    uint32_t aoff[MB], boff[NG], opos[NG];
    int skip[NG];                                      // images of the lane that its left neighbour has as well; IM: nothing to store
#pragma unroll
    for (int m = 0; m < MB; ++m) aoff[m] = min(k0 + m * 32 + j, a.K - 1) * a.flt_row;
#pragma unroll
    for (int p = 0; p < NG; ++p) {
        const uint32_t q = min(q0 + p * 32 + j, a.groups - 1);
        const uint32_t hw = flat_div(q, a.d_G), first = (q - hw * a.G) * IM;
        const uint32_t b = min(first, a.B - IM);
        const uint32_t h = flat_div(hw, a.d_W), w = hw - h * a.W;
        boff[p] = w * a.img_w + h * a.img_h + b * ESZ;
        opos[p] = hw * a.B + b;
        skip[p] = q0 + p * 32 + j < a.groups ? (int)(first - b) : IM;
    }

    const uint32_t eoff = a.B * ESZ;                   // bytes from one contraction index to the next
    const __amdgpu_buffer_rsrc_t rimg = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.image), 0, a.img_bytes, 0x00020000);

    // this wave's steps, and this half-wave's chunk of the next step to fetch
    const uint32_t s_begin = min(wk * a.steps_per_wave, a.steps), s_end = min(s_begin + a.steps_per_wave, a.steps);
    const uint32_t u_end = min(2 * s_end, a.U);
    uint32_t u = 2 * s_begin + g;
    const uint32_t r = flat_div(u, a.d_TC);
    uint32_t tc = u - r * a.TC;
    uint32_t foff = r * a.flt_r + tc * 16, ioff = r * a.img_r + tc * a.img_chunk;

    uint32_t A[D][MB][SHORT ? CH : 4];
    uint32_t X[D][NG][CH][LW];
    uint32_t lo[D];

    auto fetch = [&](int d) {
        const bool last = tc + 1 == a.TC, out = u >= u_end;
        uint32_t fo = foff, io = ioff;
        lo[d] = 0;
        if (!SHORT) {
            if (last) fo -= a.back * ESZ, io -= a.back * eoff, lo[d] = a.back;
        }
        if (out) fo = 0, io = 0, lo[d] = CH;
#pragma unroll
        for (int m = 0; m < MB; ++m) {
            if constexpr (SHORT) {
#pragma unroll
                for (int e = 0; e < CH; ++e)
                    if ((uint32_t)e < a.T) load_at<ESZ>(A[d][m] + e, (const char*)a.filter + e * ESZ, aoff[m] + fo);
            } else {
                load_at<16>(A[d][m], (const char*)a.filter, aoff[m] + fo);
            }
        }
#pragma unroll
        for (int p = 0; p < NG; ++p) {
            const uint32_t vo = boff[p] + io;
#pragma unroll
            for (int e = 0; e < CH; ++e)
                if (!SHORT || (uint32_t)e < a.T) load_image<IM * ESZ>(X[d][p][e], rimg, vo, e * eoff);
        }
        // the half-wave's chunk of the next step lies two chunks further on
        u += 2;
        tc += a.adv_tc;
        foff += a.adv_flt;
        ioff += a.adv_img;
        if (tc >= a.TC) {
            tc -= a.TC;
            foff += a.wrap_flt;
            ioff += a.wrap_img;
        }
    };

    ff32x16 acc[MB][NB];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[m][n][v] = 0.f;

    auto multiply = [&](int d) {
        const bool mask = __any(lo[d] != 0);
        fu32x4 av[MB], bv[NB];
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int i = 0; i < 4; ++i) av[m][i] = SHORT && DT == 1 ? A[d][m][2 * i] | (A[d][m][(2 * i + 1) % (SHORT ? CH : 4)] << 16) : A[d][m][i];
#pragma unroll
        for (int p = 0; p < NG; ++p)
#pragma unroll
            for (int q = 0; q < IM; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t v;
                    if constexpr (DT == 0) v = X[d][p][i % CH][q % LW];
                    else v = __builtin_amdgcn_perm(X[d][p][(2 * i + 1) % CH][q / 2 % LW], X[d][p][2 * i % CH][q / 2 % LW], q & 1 ? 0x07060302u : 0x05040100u);
                    bv[p * IM + q][i] = v;
                }
        if (mask) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t keep;
                if constexpr (DT == 0) {
                    keep = (uint32_t)i >= lo[d] ? 0xffffffffu : 0u;
                } else {
                    keep = ((uint32_t)(2 * i) >= lo[d] ? 0x0000ffffu : 0u) |
                           ((uint32_t)(2 * i + 1) >= lo[d] ? 0xffff0000u : 0u);
                }
#pragma unroll
                for (int m = 0; m < MB; ++m) av[m][i] &= keep;
#pragma unroll
                for (int n = 0; n < NB; ++n) bv[n][i] &= keep;
            }
        }
        if constexpr (DT == 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int m = 0; m < MB; ++m)
#pragma unroll
                    for (int n = 0; n < NB; ++n)
                        acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(av[m][e]), __uint_as_float(bv[n][e]),
                                                                         acc[m][n], 0, 0, 0);
        } else {
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int n = 0; n < NB; ++n)
                    acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(fbf16x8, av[m]),
                                                                        __builtin_bit_cast(fbf16x8, bv[n]), acc[m][n], 0, 0, 0);
        }
    };

    if constexpr (SHORT) {
#pragma unroll
        for (int e = 0; e < CH; ++e) {
#pragma unroll
            for (int m = 0; m < MB; ++m) A[0][m][e] = 0;
#pragma unroll
            for (int p = 0; p < NG; ++p)
#pragma unroll
                for (int i = 0; i < LW; ++i) X[0][p][e][i] = 0;
        }
    }
    if constexpr (AHEAD == 0) {
        for (uint32_t s = s_begin; s < s_end; ++s) {
            fetch(0);
            multiply(0);
        }
    } else {
        // D steps of loads are in flight; the order of the loads is kept (left alone, the compiler mixes the steps of the
        // first group, and then waits for nearly all of them before the first product of every group)
#pragma unroll
        for (int d = 0; d < D; ++d) {
            fetch(d);
            __builtin_amdgcn_sched_barrier(0);
        }
        for (uint32_t s = s_begin; s < s_end; s += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                multiply(d);
                fetch(d);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    // (the fetches beyond the last step are of the first chunk, cached, and masked)
    // MFMA D layout: lane j + 32 g holds rows 8 (v / 4) + 4 g + v % 4 of column j
    auto store = [&](int m, int p, int v, const float (&o)[IM]) {
        const uint32_t k = k0 + m * 32 + (v >> 2) * 8 + g * 4 + (v & 3);
        if (k >= a.K) return;
        float* const dst = a.out + (int64_t)k * a.N + opos[p];
        if (skip[p] == 0) {
            if constexpr (IM == 4) ((Out4*)dst)->v = ff32x4{o[0], o[1], o[2], o[3]};
            else if constexpr (IM == 2) ((Out2*)dst)->v = ff32x2{o[0], o[1]};
            else dst[0] = o[0];
        } else {
#pragma unroll
            for (int i = 1; i < IM; ++i)
                if (i >= skip[p]) dst[i] = o[i];
        }
    };
    flat_write_out<MB, NG, IM, WM * WN, WK>(s_red, acc, wave, wk, lane, store);
}

template <int DT, int MB, int NG, int IM, int WM, int WN, int WK, int D, bool SHORT>
static int launch_flat_one(const FlatArgs& a, int grid, void* stream) {
    constexpr size_t lds = FlatReduce<MB, NG, IM, WM * WN, WK>::BYTES;
    static_assert(lds <= 64 * 1024, "flat kernel: partial sums fit the LDS that a launch gets without asking");
    auto kernel = conv_flat_kernel<DT, MB, NG, IM, WM, WN, WK, D, SHORT>;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(WM * WN * WK * 64), lds, (hipStream_t)stream, a);
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

template <int DT, int MB, int NG, int IM, int WM, int WN, int WK, int D>
static int launch_flat_shape(const FlatArgs& a, int grid, void* stream) {
    if (a.T < (DT == 0 ? 4u : 8u)) return launch_flat_one<DT, MB, NG, IM, WM, WN, WK, 0, true>(a, grid, stream);
    if (a.steps_per_wave <= 1) return launch_flat_one<DT, MB, NG, IM, WM, WN, WK, 0, false>(a, grid, stream);
    return launch_flat_one<DT, MB, NG, IM, WM, WN, WK, D, false>(a, grid, stream);
}

// ---------------------------------------------------------------------------------------------------------------
// The same product with both operands staged in LDS, NCH chunks of the contraction at a time.  Loads go through registers
// (16-byte loads at any element alignment, zeroed where a chunk is shorter) two stages ahead.  A stage always multiplies
// all of its steps, the zeros of a last, shorter one included: a way out between the steps kept the compiler from reading
// ahead (4 to 8 % of the time), and a second copy of the steps for whole stages cost as much in code as it gained.
// IM > 0: the tile's columns are groups of IM adjacent images; LDS holds one row of columns per contraction index.
// IM < 0: the columns are positions with all of their -IM images; LDS holds a position's chunks as they lie in memory.
template <int DT, int MB, int NBW, int IM, int WM, int WN, int WK, int NCH>
struct FlatLds {
    static constexpr int ESZ = DT == 0 ? 4 : 2, CH = 16 / ESZ, THREADS = WM * WN * WK * 64;
    static constexpr bool RUN = IM < 0;
    static constexpr int IPL = RUN ? -IM : IM, NB = RUN ? NBW * IPL : NBW;
    static constexpr int KT = WM * MB * 32, COLS = WN * NBW * 32;   // columns (RUN: positions) of the tile
    static constexpr int GROUPS = RUN ? COLS : COLS / IPL;
    static constexpr int FP = NCH + 1;                              // 16-byte units of a Filter row, odd: conflict-free reads
    static constexpr int FLT_BYTES = KT * FP * 16;
    // bytes of an Image row.  Positions: an odd number of 16-byte units.  bf16 columns: four rows' 64-byte pieces, which a
    // transposing read takes at once, lie in different banks; fp32 columns: rows four apart differ by 32 banks.
    static constexpr int ROW = RUN ? ((NCH * IPL) | 1) * 16 : DT == 0 ? COLS * 4 + 32 : COLS * 2 + (COLS == 32 ? 0 : 64);
    static constexpr int IMG_BYTES = (RUN ? COLS : NCH * CH) * ROW;
    static constexpr int BUF = FLT_BYTES + IMG_BYTES;
    static constexpr int NF = KT * NCH / THREADS;                   // Filter items per thread and stage
    static constexpr int RPP = RUN ? THREADS / NCH : THREADS / GROUPS;   // positions / contraction indices per pass
    static constexpr int NI = RUN ? COLS / RPP : NCH * CH / RPP;    // Image items (RUN: of IPL loads each)
    static constexpr int LW = RUN ? 4 : IPL * ESZ / 4;              // dwords of one Image load
    static constexpr int STEPS = NCH / 2 / WK;                      // steps of two chunks per wave and stage
    using Red = FlatReduce<MB, NBW, RUN ? IPL : 1, WM * WN, WK>;
    static constexpr size_t LDS = 2 * BUF > (int)Red::BYTES ? (size_t)2 * BUF : Red::BYTES;
    static_assert(NF * THREADS == KT * NCH && NF >= 1, "flat LDS kernel: whole Filter items per thread");
    static_assert(RUN ? NI * RPP == COLS && NI >= 1 : (NI * RPP == NCH * CH && RPP % CH == 0 && NI >= 1), "flat LDS kernel: whole Image items per thread");
    static_assert(STEPS >= 1 && STEPS * 2 * WK == NCH, "flat LDS kernel: whole steps per wave");
    static_assert(LDS <= 160 * 1024, "flat LDS kernel: LDS size");
};

// STREAM: Out past the L2, only where every store instruction writes whole halves of cache lines; elsewhere the L2 has to put the pieces
// together.  One launch, buffers in rotation, through the L2 and past it: bf16 (16, 3, 64, 112, 112, 7 x 7, s 2) 21.4 and 20.6
// us, 32 images 48.2 and 36.8, (32, 3, 64, 112, 112, 3 x 3, s 2) 37.2 and 24.1, fp32 (12, 3, 16, 112, 112, 3 x 3, s 2) 12.5 and 11.9; of
// pieces of lines, bf16 (20, 3, 64, 111, 111, 3 x 3, s 2) 21.7 and 33.0, (12, 64, 256, 57, 55, 1 x 1) 14.9 and 19.0.  A template
// parameter because the compiler makes one ordinary store of the two sides of a branch.
constexpr int OUT_CACHED = 0, OUT_STREAMED = 1, OUT_SPLIT = 2;

// OUT_SPLIT: the contraction of a tile is divided over a.parts workgroups, for calls whose tiles leave most compute units idle while each of
// the few at work walks a long contraction.  Every workgroup leaves its sums in the device's scratch memory and counts itself; the one
// that comes last adds all of them, in the order of the parts (the result does not depend on which one that is), and writes Out.  No
// workgroup waits for another.  The scratch belongs to one launch at a time: the host makes such launches on the null stream alone.  Fitted to
// such launches, the exchange costs 1.7 us, 0.25 us a part and the sums at 2.7 TB/s; fp32 (1, 784, 64, 3, 12, 3 x 3) 42.2 -> 8.8 us, bf16 (72, 976,
// 16, 5, 5, 3 x 3, s 2) 27.8 -> 11.7.
__device__ float g_split_sums[kSplitWords];
__device__ unsigned int g_split_arrived[kSplitTiles];      // zero between launches: the workgroup that comes last clears its tile's

template <int DT, int MB, int NBW, int IM, int WM, int WN, int WK, int NCH, int OUT, class Args>
__global__ void __launch_bounds__(WM* WN* WK * 64) conv_flat_lds_kernel(const Args a) {
    using GEO = FlatLds<DT, MB, NBW, IM, WM, WN, WK, NCH>;
    constexpr int ESZ = GEO::ESZ, CH = GEO::CH, IPL = GEO::IPL, NB = GEO::NB, NF = GEO::NF, NI = GEO::NI, LW = GEO::LW;
    constexpr int THREADS = GEO::THREADS, RPP = GEO::RPP;
    constexpr bool RUN = GEO::RUN;
    constexpr int LE = RUN ? IPL : 1;                  // loads per Image item
    constexpr int NS = RUN ? 1 : NI;                   // chunks that a thread's Image items belong to
    extern __shared__ __align__(16) char s_mem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave % WK, wm = (wave / WK) % WM, wn = wave / (WK * WM);
    const int j = lane & 31, g = lane >> 5;

    uint32_t t = xcd_order(blockIdx.x, a.xcd_q, a.xcd_rem), part = 0;
    if constexpr (OUT == OUT_SPLIT) {
        part = flat_div(t, a.d_tiles);
        t -= part * a.tiles;
    }
    uint32_t tk, tn;
    {
        const uint32_t q = flat_div(t, a.d_inner), i = t - q * a.inner;
        tk = a.k_inner ? i : q;
        tn = a.k_inner ? q : i;
    }
    const uint32_t k0 = tk * GEO::KT, q0 = tn * GEO::GROUPS;
    auto position = [&](uint32_t q, uint32_t& img, uint32_t& pos, int& skip) {
        const uint32_t qc = min(q, a.groups - 1);
        const uint32_t hw = RUN ? qc : flat_div(qc, a.d_G), first = RUN ? 0 : (qc - hw * a.G) * IPL;
        const uint32_t b = RUN ? 0 : min(first, a.B - IPL);
        const uint32_t h = flat_div(hw, a.d_W), w = hw - h * a.W;
        img = w * a.img_w + h * a.img_h + b * ESZ;
        pos = hw * a.B + b;
        skip = q < a.groups ? (int)(first - b) : IPL;
    };

    // ---- staging: a thread's items, fixed but for the chunk that they move on to with every stage
    struct Chunk {
        uint32_t u, tc, flt, img;
    };
    auto chunk_at = [&](uint32_t u) {
        const uint32_t r = flat_div(u, a.d_TC), tc = u - r * a.TC;
        return Chunk{u, tc, r * a.flt_r + tc * 16, r * a.img_r + tc * a.img_chunk};
    };
    auto advance = [&](Chunk& c) {
        c.u += NCH;
        c.tc += a.adv_tc;
        c.flt += a.adv_flt;
        c.img += a.adv_img;
        if (c.tc >= a.TC) {
            c.tc -= a.TC;
            c.flt += a.wrap_flt;
            c.img += a.wrap_img;
        }
    };
    // this workgroup's stages, and the chunk behind its last one
    int stages = (int)((a.U + NCH - 1) / NCH);
    uint32_t u_first = 0, u_end = a.U;
    if constexpr (OUT == OUT_SPLIT) {
        u_first = part * a.part_stages * NCH;
        stages = min((int)a.part_stages, stages - (int)(part * a.part_stages));
        u_end = min(a.U, u_first + stages * NCH);
    }
    const uint32_t eoff = a.B * ESZ;
    const int fc = tid % NCH, fr = tid / NCH;
    uint32_t aoff[NF];
#pragma unroll
    for (int i = 0; i < NF; ++i) aoff[i] = min(k0 + fr + i * (THREADS / NCH), a.K - 1) * a.flt_row;
    Chunk fch = chunk_at(u_first + fc), ich[NS];
    const int ig = RUN ? 0 : tid % GEO::GROUPS, ir = RUN ? fr : tid / GEO::GROUPS;
    uint32_t boff[RUN ? NI : 1];
    {
        uint32_t pos;
        int skip;
        if constexpr (RUN) {
#pragma unroll
            for (int i = 0; i < NI; ++i) position(q0 + ir + i * RPP, boff[i], pos, skip);
            ich[0] = fch;
        } else {
            position(q0 + ig, boff[0], pos, skip);
#pragma unroll
            for (int i = 0; i < NI; ++i) ich[i] = chunk_at(u_first + ir / CH + i * (RPP / CH));
        }
    }
    const int ie = ir % CH;                            // (columns) the item's contraction index inside its chunk

    uint32_t F[2][NF][4], X[2][NI][LE][LW], flo[2], ilo[2][NS];
    auto fetch = [&](int set) {
        {
            const bool out = fch.u >= u_end, last = fch.tc + 1 == a.TC;
            flo[set] = out ? CH : last ? a.back : 0;
            const uint32_t fo = out ? 0 : last ? fch.flt - a.back * ESZ : fch.flt;
#pragma unroll
            for (int i = 0; i < NF; ++i) load_at<16>(F[set][i], (const char*)a.filter, aoff[i] + fo);
            if constexpr (RUN) {
                const uint32_t io = out ? 0 : last ? fch.img - a.back * eoff : fch.img;
                ilo[set][0] = flo[set];
#pragma unroll
                for (int i = 0; i < NI; ++i)
#pragma unroll
                    for (int e = 0; e < LE; ++e) load_at<16>(X[set][i][e], (const char*)a.image + e * 16, boff[i] + io);
            }
            advance(fch);
        }
        if constexpr (!RUN) {
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const bool out = ich[i].u >= u_end, last = ich[i].tc + 1 == a.TC;
                ilo[set][i] = out ? CH : last ? a.back : 0;
                const uint32_t io = out ? 0 : (last ? ich[i].img - a.back * eoff : ich[i].img) + ie * eoff;
                load_at<LW * 4>(X[set][i][0], (const char*)a.image, boff[0] + io);
                advance(ich[i]);
            }
        }
    };
    // elements [0, lo) of a chunk are zeros for both operands: a chunk beyond the last one, and the elements of the last chunk
    // of a filter row that the chunk before it has as well
    auto put = [&](int set, char* buf) {
        uint32_t any = flo[set];
#pragma unroll
        for (int i = 0; i < NS; ++i) any |= ilo[set][i];
        if (__any(any != 0)) {
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const uint32_t lo = flo[set];
                const uint32_t keep = DT == 0 ? ((uint32_t)d >= lo ? ~0u : 0u)
                                              : ((uint32_t)(2 * d) >= lo ? 0xffffu : 0u) | ((uint32_t)(2 * d + 1) >= lo ? 0xffff0000u : 0u);
#pragma unroll
                for (int i = 0; i < NF; ++i) F[set][i][d] &= keep;
            }
            if constexpr (RUN) {
                const uint32_t lo = flo[set] * IPL;
#pragma unroll
                for (int e = 0; e < LE; ++e)
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        const uint32_t f = DT == 0 ? e * 4 + d : e * 8 + 2 * d;
                        const uint32_t keep = DT == 0 ? (f >= lo ? ~0u : 0u) : (f >= lo ? 0xffffu : 0u) | (f + 1 >= lo ? 0xffff0000u : 0u);
#pragma unroll
                        for (int i = 0; i < NI; ++i) X[set][i][e][d] &= keep;
                    }
            } else {
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    const uint32_t keep = (uint32_t)ie >= ilo[set][i] ? ~0u : 0u;
#pragma unroll
                    for (int d = 0; d < LW; ++d) X[set][i][0][d] &= keep;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < NF; ++i)
            *(fu32x4*)(buf + ((fr + i * (THREADS / NCH)) * GEO::FP + fc) * 16) = fu32x4{F[set][i][0], F[set][i][1], F[set][i][2], F[set][i][3]};
        char* const img = buf + GEO::FLT_BYTES;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            if constexpr (RUN) {
#pragma unroll
                for (int e = 0; e < LE; ++e)
                    *(fu32x4*)(img + (ir + i * RPP) * GEO::ROW + (fc * IPL + e) * 16) = fu32x4{X[set][i][e][0], X[set][i][e][1], X[set][i][e][2], X[set][i][e][3]};
            } else if constexpr (LW == 4) {
                *(fu32x4*)(img + (ir + i * RPP) * GEO::ROW + ig * 16) = fu32x4{X[set][i][0][0], X[set][i][0][1 % LW], X[set][i][0][2 % LW], X[set][i][0][3 % LW]};
            } else {
                *(fu32x2*)(img + (ir + i * RPP) * GEO::ROW + ig * 8) = fu32x2{X[set][i][0][0], X[set][i][0][1 % LW]};
            }
        }
    };

    // ---- multiplication
    ff32x16 acc[MB][NB];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[m][n][v] = 0.f;
    const int i16 = lane & 15, jhalf = (lane >> 4) & 1;
    auto read_step = [&](const char* buf, int st, fu32x4 (&av)[MB], fu32x4 (&bv)[NB]) {
        const char* const ap = buf + ((wm * MB * 32 + j) * GEO::FP + g) * 16;
        const char* const img = buf + GEO::FLT_BYTES;
#pragma unroll
        for (int m = 0; m < MB; ++m) av[m] = *(const fu32x4*)(ap + m * 32 * GEO::FP * 16 + st * 32);
        if constexpr (RUN) {
#pragma unroll
            for (int p = 0; p < NBW; ++p) {
                const char* const xp = img + ((wn * NBW + p) * 32 + j) * GEO::ROW + (2 * st + g) * IPL * 16;
                fu32x4 x[IPL];
#pragma unroll
                for (int e = 0; e < IPL; ++e) x[e] = *(const fu32x4*)(xp + e * 16);
#pragma unroll
                for (int q = 0; q < IPL; ++q)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if constexpr (DT == 0) {
                            bv[p * IPL + q][i] = x[(i * IPL + q) / 4][(i * IPL + q) % 4];
                        } else {
                            const int e0 = 2 * i * IPL + q, e1 = e0 + IPL;
                            bv[p * IPL + q][i] = IPL == 1 ? x[0][i]
                                                          : __builtin_amdgcn_perm(x[e1 / 8][e1 / 2 % 4], x[e0 / 8][e0 / 2 % 4],
                                                                                  (e1 & 1 ? 0x07060000u : 0x05040000u) | (e0 & 1 ? 0x0302u : 0x0100u));
                        }
                    }
            }
        } else if constexpr (DT == 0) {
            const char* const xp = img + (2 * st + g) * CH * GEO::ROW + (wn * NBW * 32 + j) * 4;
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int e = 0; e < 4; ++e) bv[n][e] = *(const uint32_t*)(xp + e * GEO::ROW + n * 128);
        } else {
            // the transposing read: four rows (contraction indices) of 16 columns to a lane per column
            const char* const xp = img + (16 * st + 8 * g + (i16 >> 2)) * GEO::ROW + wn * NBW * 64 + jhalf * 32 + (i16 & 3) * 8;
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                const fs16x4 l = __builtin_amdgcn_ds_read_tr16_b64_v4i16((FLAT_LDS(fs16x4)*)(xp + n * 64));
                const fs16x4 h = __builtin_amdgcn_ds_read_tr16_b64_v4i16((FLAT_LDS(fs16x4)*)(xp + 4 * GEO::ROW + n * 64));
                bv[n] = __builtin_bit_cast(fu32x4, __builtin_shufflevector(l, h, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        }
    };
    auto mfma_step = [&](const fu32x4 (&av)[MB], const fu32x4 (&bv)[NB]) {
        if constexpr (DT == 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int m = 0; m < MB; ++m)
#pragma unroll
                    for (int n = 0; n < NB; ++n)
                        acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(av[m][e]), __uint_as_float(bv[n][e]), acc[m][n], 0, 0, 0);
        } else {
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int n = 0; n < NB; ++n)
                    acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(fbf16x8, av[m]), __builtin_bit_cast(fbf16x8, bv[n]), acc[m][n], 0, 0, 0);
        }
    };
    // The operands of AHEAD steps are read before the first of their products: left alone, the compiler reads a step's operands
    // right in front of its products and waits for them every time.
    constexpr int FIT = 32 / ((MB + NB) * 4), AHEAD = FIT < 1 ? 1 : FIT < GEO::STEPS ? FIT : GEO::STEPS;
    auto multiply = [&](const char* buf) {
#pragma unroll
        for (int s0 = 0; s0 < GEO::STEPS; s0 += AHEAD) {
            fu32x4 av[AHEAD][MB], bv[AHEAD][NB];
#pragma unroll
            for (int s = 0; s < AHEAD; ++s)
                if (s0 + s < GEO::STEPS) read_step(buf, (s0 + s) * WK + wk, av[s], bv[s]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < AHEAD; ++s)
                if (s0 + s < GEO::STEPS) mfma_step(av[s], bv[s]);
        }
    };

    // Stage s is multiplied out of buffer s % 2 while the loads of stages s + 1 and s + 2 are in flight or in registers; a
    // buffer is written again after the barrier that every wave reaches behind its reads of it.  All waves run the same
    // number of stages.
    char* const buf0 = s_mem;
    char* const buf1 = s_mem + GEO::BUF;
    auto keep_order = [] {
        // (neither the compiler's passes nor its scheduler may move loads past this point)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    fetch(0);
    keep_order();
    fetch(1);
    keep_order();
    put(0, buf0);
    keep_order();
    fetch(0);
    keep_order();
    __syncthreads();
    // (no way out of the middle of the loop: the compiler would count loads as if the second half could be followed by the first
    // half's wait, and wait for the younger of the two sets there as well)
    int s = 0;
    for (; s + 2 < stages; s += 2) {
        multiply(buf0);
        put(1, buf1);
        keep_order();
        fetch(1);
        keep_order();
        __syncthreads();
        multiply(buf1);
        put(0, buf0);
        keep_order();
        fetch(0);
        keep_order();
        __syncthreads();
    }
    multiply(buf0);
    if (s + 1 < stages) {
        put(1, buf1);
        __syncthreads();
        multiply(buf1);
    }

    // ---- Out
    constexpr int SI = RUN ? IPL : 1;                  // images of a lane's column block group
    uint32_t opos[NBW];
    int skip[NBW];
#pragma unroll
    for (int p = 0; p < NBW; ++p) {
        uint32_t img;
        const uint32_t col = (wn * NBW + p) * 32 + j;
        position(q0 + (RUN ? col : col / IPL), img, opos[p], skip[p]);
        if (!RUN) {
            opos[p] += col % IPL;
            skip[p] = (int)(col % IPL) < skip[p];
        }
    }
    auto store = [&](int m, int p, int v, const float (&o)[SI]) {
        const uint32_t k = k0 + (wm * MB + m) * 32 + (v >> 2) * 8 + g * 4 + (v & 3);
        if (k >= a.K || skip[p]) return;
        float* const dst = a.out + (int64_t)k * a.N + opos[p];
        if constexpr (OUT == OUT_STREAMED) {
            __builtin_nontemporal_store(o[0], dst);
        } else if constexpr (SI == 4) {
            ((Out4*)dst)->v = ff32x4{o[0], o[1], o[2], o[3]};
        } else if constexpr (SI == 2 || SI == 6) {
#pragma unroll
            for (int i = 0; i < SI; i += 2) ((Out2*)(dst + i))->v = ff32x2{o[i], o[i + 1]};
        } else {
#pragma unroll
            for (int i = 0; i < SI; ++i) dst[i] = o[i];
        }
    };
    if constexpr (WK > 1) __syncthreads();             // the buffers become the exchange area of the partial sums
    if constexpr (OUT == OUT_SPLIT) {
        constexpr uint32_t ROWS = WM * MB * WN * NBW * 16, TILE = ROWS * SI * 64;     // rows of 64 lanes' sums, words of a part
        float* const mine = g_split_sums + (size_t)(t * a.parts + part) * TILE;
        auto row_of = [&](int m, int p, int v) { return (((wm * MB + m) * (WN * NBW) + wn * NBW + p) * 16 + v) * (SI * 64) + lane; };
        flat_write_out<MB, NBW, SI, WM * WN, WK>((float*)s_mem, acc, wave, wk, lane, [&](int m, int p, int v, const float (&o)[SI]) {
#pragma unroll
            for (int i = 0; i < SI; ++i) __hip_atomic_store(mine + row_of(m, p, v) + i * 64, o[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        });
        // The sums pass through stores and loads of the device's scope, which the L2s of the XCDs do not keep; a wave's stores have arrived
        // when it has waited for them.  (A device-scope fence would write back and invalidate an L2: 10 to 60 us in such a launch.)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        unsigned int* const last = (unsigned int*)s_mem;
        if (tid == 0) {
            *last = __hip_atomic_fetch_add(&g_split_arrived[t], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == a.parts;
            if (*last) __hip_atomic_store(&g_split_arrived[t], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (!*last) return;
        float* const sums = g_split_sums + (size_t)t * a.parts * TILE;
        // rows divided over the waves of a column of them as above; the loads of a part are in flight together
        float o[MB][NBW][16 / WK][SI];
        auto each_row = [&](auto f) {
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int p = 0; p < NBW; ++p)
#pragma unroll
                    for (int v = 0; v < 16 / WK; ++v) f(m, p, v);
        };
        each_row([&](int m, int p, int v) {
#pragma unroll
            for (int i = 0; i < SI; ++i) o[m][p][v][i] = 0.f;
        });
#pragma unroll 4
        for (uint32_t q = 0; q < a.parts; ++q)
            each_row([&](int m, int p, int v) {
#pragma unroll
                for (int i = 0; i < SI; ++i) 
                    o[m][p][v][i] += __hip_atomic_load(sums + (size_t)q * TILE + row_of(m, p, v * WK + wk) + i * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            });
        each_row([&](int m, int p, int v) { store(m, p, v * WK + wk, o[m][p][v]); });
    } else {
        flat_write_out<MB, NBW, SI, WM * WN, WK>((float*)s_mem, acc, wave, wk, lane, store);
    }
}

template <int DT, int MB, int NBW, int IM, int WM, int WN, int WK, int NCH, int OUT, class Args>
static int launch_flat_lds_as(const Args& a, int grid, void* stream) {
    using GEO = FlatLds<DT, MB, NBW, IM, WM, WN, WK, NCH>;
    auto kernel = conv_flat_lds_kernel<DT, MB, NBW, IM, WM, WN, WK, NCH, OUT, Args>;
    if constexpr (GEO::LDS > 64 * 1024) {
        static OncePerDevice once;
        int device = -1;
        if (hipGetDevice(&device) != hipSuccess || !once(device, [&] {
                return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) == hipSuccess;
            })) {
            (void)hipGetLastError();
            return 1;
        }
    }
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(GEO::THREADS), GEO::LDS, (hipStream_t)stream, a);
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

// Out is streamed where the 32 columns of a block are one run of 128 bytes: a lane stores one image and none that another has (B a
// multiple of IM), the rows of Out are whole lines, and Out starts at a multiple of 64 bytes, half a line.  At other addresses,
// past the L2 and through it: bf16 (32, 3, 64, 112, 112, 7 x 7, s 2) 54.4 and 49.5 us, (32, 3, 64, 112, 112, 3 x 3, s 2) 51.3 and 39.2,
// (64, 30, 64, 56, 56, 3 x 3) 28.3 and 30.6; 64 bytes beyond a line 40.3 and 49.9, 31.8 and 39.1, 26.4 and 30.3.
template <int DT, int MB, int NBW, int IM, int WM, int WN, int WK, int NCH>
static int launch_flat_lds(const FlatArgs& a, int grid, void* stream) {
    if constexpr (IM >= -1)
        if (a.B % (IM > 0 ? IM : 1) == 0 && a.N % 32 == 0 && reinterpret_cast<uintptr_t>(a.out) % 64 == 0)
            return launch_flat_lds_as<DT, MB, NBW, IM, WM, WN, WK, NCH, OUT_STREAMED>(a, grid, stream);
    return launch_flat_lds_as<DT, MB, NBW, IM, WM, WN, WK, NCH, OUT_CACHED>(a, grid, stream);
}

template <int DT, int MB, int NBW, int IM, int WM, int WN, int WK, int NCH>
static int launch_flat_split(const FlatSplitArgs& a, int grid, void* stream) {
    return launch_flat_lds_as<DT, MB, NBW, IM, WM, WN, WK, NCH, OUT_SPLIT>(a, grid, stream);
}

// blocks of output channels, groups of images per wave; images per lane; waves along k, positions, contraction; steps ahead.
// (The configurations that the cost estimate in cacnn_host.cpp picks from: chosen from 490 by leaving out, one after the
// other, what made its picks on 390 layers of all sizes worse by least; on 330 others the best of these is within 0.3 % of the
// best of all that were left then.)
#define CACNN_FLAT(DT, MB, NG, IM, WM, WN, WK, D) \
    {{DT, MB, NG, IM, WM, WN, WK, 0}, launch_flat_shape<DT, MB, NG, IM, WM, WN, WK, D>, nullptr}

#define CACNN_FLAT_LDS(DT, MB, NBW, IM, WM, WN, WK, NCH) \
    {{DT, MB, NBW, IM, WM, WN, WK, NCH}, launch_flat_lds<DT, MB, NBW, IM, WM, WN, WK, NCH>, launch_flat_split<DT, MB, NBW, IM, WM, WN, WK, NCH>}

static const FlatVariant g_flat[] = {
    // fp32
    CACNN_FLAT(0, 1, 1, 1, 1, 1, 4, 4),
    CACNN_FLAT(0, 1, 1, 2, 1, 4, 1, 4),
    CACNN_FLAT(0, 1, 1, 4, 1, 4, 1, 4),
    CACNN_FLAT(0, 1, 1, 4, 2, 1, 2, 4),
    CACNN_FLAT(0, 1, 1, 4, 2, 2, 1, 4),
    CACNN_FLAT_LDS(0, 1, 1, 2, 1, 1, 4, 8),
    CACNN_FLAT_LDS(0, 1, 1, 2, 1, 1, 8, 32),
    CACNN_FLAT_LDS(0, 1, 1, 4, 1, 1, 4, 8),
    CACNN_FLAT_LDS(0, 1, 1, 4, 1, 1, 8, 32),
    CACNN_FLAT_LDS(0, 1, 1, 4, 1, 2, 4, 16),
    CACNN_FLAT_LDS(0, 1, 1, 4, 1, 4, 1, 8),
    CACNN_FLAT_LDS(0, 1, 1, 4, 2, 1, 4, 16),
    CACNN_FLAT_LDS(0, 1, 1, 4, 2, 2, 1, 8),
    CACNN_FLAT_LDS(0, 1, 1, 4, 4, 2, 1, 8),
    CACNN_FLAT_LDS(0, 1, 2, 4, 2, 2, 1, 8),
    CACNN_FLAT_LDS(0, 2, 2, 4, 2, 2, 1, 8),
    CACNN_FLAT_LDS(0, 1, 1, -1, 1, 1, 4, 16),
    CACNN_FLAT_LDS(0, 1, 1, -1, 1, 1, 8, 32),
    CACNN_FLAT_LDS(0, 1, 1, -1, 2, 2, 1, 8),
    CACNN_FLAT_LDS(0, 1, 1, -2, 1, 1, 4, 8),
    CACNN_FLAT_LDS(0, 1, 1, -2, 1, 1, 8, 32),
    CACNN_FLAT_LDS(0, 1, 1, -3, 1, 1, 4, 8),
    // bf16
    CACNN_FLAT(1, 1, 1, 1, 1, 1, 4, 4),
    CACNN_FLAT(1, 1, 2, 1, 1, 1, 4, 3),
    CACNN_FLAT(1, 1, 2, 2, 1, 4, 1, 3),
    CACNN_FLAT(1, 2, 2, 2, 1, 4, 1, 3),
    CACNN_FLAT(1, 1, 1, 4, 1, 1, 4, 4),
    CACNN_FLAT_LDS(1, 1, 1, 4, 1, 1, 4, 8),
    CACNN_FLAT_LDS(1, 1, 1, 4, 1, 1, 8, 32),
    CACNN_FLAT_LDS(1, 1, 1, 4, 2, 1, 4, 16),
    CACNN_FLAT_LDS(1, 1, 1, 4, 2, 2, 1, 8),
    CACNN_FLAT_LDS(1, 1, 2, 4, 4, 2, 1, 8),
    CACNN_FLAT_LDS(1, 1, 1, 8, 1, 1, 4, 8),
    CACNN_FLAT_LDS(1, 1, 1, 8, 1, 1, 8, 32),
    CACNN_FLAT_LDS(1, 1, 1, 8, 1, 4, 1, 8),
    CACNN_FLAT_LDS(1, 1, 1, 8, 2, 2, 1, 8),
    CACNN_FLAT_LDS(1, 1, 1, 8, 2, 4, 1, 8),
    CACNN_FLAT_LDS(1, 1, 1, 8, 4, 2, 1, 8),
    CACNN_FLAT_LDS(1, 1, 2, 8, 4, 2, 1, 8),
    CACNN_FLAT_LDS(1, 2, 2, 8, 2, 2, 1, 8),
    CACNN_FLAT_LDS(1, 2, 2, 8, 2, 4, 1, 8),
    CACNN_FLAT_LDS(1, 1, 1, -1, 1, 1, 4, 8),
    CACNN_FLAT_LDS(1, 1, 1, -1, 1, 1, 8, 32),
    CACNN_FLAT_LDS(1, 1, 1, -1, 2, 2, 1, 8),
    CACNN_FLAT_LDS(1, 1, 1, -2, 1, 1, 4, 8),
    CACNN_FLAT_LDS(1, 1, 1, -2, 1, 1, 8, 32),
    CACNN_FLAT_LDS(1, 1, 1, -2, 4, 2, 1, 8),
    CACNN_FLAT_LDS(1, 1, 1, -3, 1, 1, 4, 8),
    CACNN_FLAT_LDS(1, 1, 1, -3, 1, 1, 8, 16),
    CACNN_FLAT_LDS(1, 1, 1, -3, 4, 1, 1, 8),
    CACNN_FLAT_LDS(1, 1, 1, -4, 1, 1, 8, 16),
    CACNN_FLAT_LDS(1, 1, 1, -4, 4, 1, 1, 8),
    CACNN_FLAT_LDS(1, 1, 1, -5, 1, 1, 8, 16),
    CACNN_FLAT_LDS(1, 1, 1, -6, 1, 1, 8, 16),
    CACNN_FLAT_LDS(1, 1, 1, -7, 1, 1, 4, 8),
};

int num_flat() { return (int)(sizeof(g_flat) / sizeof(g_flat[0])); }
const FlatVariant& flat_variant(int i) { return g_flat[i]; }

}  // namespace cacnn
