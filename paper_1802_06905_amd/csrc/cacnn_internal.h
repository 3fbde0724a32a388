// Internal interface between the host planner/dispatcher (cacnn_host.cpp) and the gfx950 kernels
// (cacnn_kernels.hip).  Not part of the public ABI.
#ifndef CACNN_INTERNAL_H
#define CACNN_INTERNAL_H

#include <stddef.h>
#include <stdint.h>

#include <atomic>

namespace cacnn {

// What cacnn_torch.cpp takes on trust of the library: the problem's layout and the signatures of cacnn_internal_conv_forward_sized and
// cacnn_internal_pool_forward_sized.  To be raised with any of them; a module and a library that differ are not used together.
constexpr int kSizedInterface = 1;

// Set-up that a process needs once for each device: done(device, set_up) calls set_up() until it has succeeded there.  A failure is not
// remembered; threads that come at the same time may both set up.
struct OncePerDevice {
    std::atomic<uint64_t> devices{0};
    template <class SetUp>
    bool operator()(int device, SetUp set_up) {
        const uint64_t bit = device >= 0 && device < 64 ? 1ull << device : 0;
        if (devices.load(std::memory_order_acquire) & bit) return true;
        if (!set_up()) return false;
        devices.fetch_or(bit, std::memory_order_release);
        return true;
    }
};

// Division of small unsigned numbers by a run-time constant with one multiply-high.
// Exact for n * d < 2^32 (the staged-tile indices it is used on are bounded by the LDS size).
struct FastDiv {
    uint32_t mul;  // floor(2^32 / d) + 1, or 0 when d == 1
    uint32_t d;
};

inline FastDiv make_fastdiv(uint32_t d) {
    FastDiv f;
    f.d = d;
    f.mul = (d <= 1) ? 0u : (uint32_t)((0x100000000ull / d) + 1ull);
    return f;
}

// Geometry of one compiled kernel variant: the workgroup's Out tile is KT output channels by a position tile of
// TB images x TW output columns x TH output rows, flattened as n = (h_l*TW + w_l)*TB + b_l and cut into MFMA
// column blocks of 32.  WM x WN wavefronts; each owns MBLK x NBLK MFMA tiles of 32x32.
struct VariantInfo {
    const char* name;
    int dtype;  // cacnn_dtype
    int WM, WN, MBLK, NBLK, TB, TW, TH;
    // 0: one workgroup per Out tile, staging and MFMA alternate (works for every shape and alignment).
    // 1: persistent workgroups walk a list of (tile, contraction slice) units; the next unit's Image and Filter
    //    words are fetched into registers while the current one is multiplied, LDS is double-buffered.
    //    Needs 16-byte-legal operands and a slice that fits MAXI/MAXF staging items per thread.
    // 2: as 1, with twice the waves: half of them only stage (two units ahead), the other half only multiply.
    int pipelined;
    int MAXI, MAXF;
    int occ;    // workgroups of this kernel one compute unit can hold at once, as far as registers go
    int reuse_r;  // > 0: filter-row reuse path compiled for exactly this many taps per contraction tile (sigma_w = 1);
                  // -4: fp32 kernel with the 16-byte-fragment LDS layout (c-slices in multiples of 4 channels)
    float tune;   // measured time of this variant relative to what the planner's cost model predicts (1 = as modelled)
    // fixed-geometry kernels: the only contraction tile (c-slice, b_r, b_s) the kernel was compiled for (0 = any)
    // and the staged Image rows sigma_h*(TH-1)+b_s it assumes
    int fx_ct = 0, fx_br = 0, fx_bs = 0, fx_ys = 0;
    int fx_sw = 1, fx_sh = 1;   // the strides it assumes
    int fx_lds = 0;             // the fixed-geometry kernels' own LDS layout, bytes (they all have one)
    // measured on MI355X with every CU busy: microseconds per unit (tile and contraction slice) of one workgroup, and the
    // fixed part of a launch (first loads, last Out tile, dispatch); the planner prices these kernels with them
    float fx_unit_us = 0.f, fx_fixed_us = 0.f;
    int fx_whole = 0;           // 1: with its own LDS layout, the kernel takes a tile's whole contraction as one unit (C == fx_ct, S == fx_bs)
    int fx_ragged = 0;          // 1: W, H and K need not be multiples of the tile (the kernel masks its Out stores); 2: nor B
    int fx_calib_cus = 0;       // > 0 (bf16): the busy compute units fx_unit_us was measured with.  The chip's bf16 MFMA rate is
                                // power-limited, so a unit takes longer the more compute units work at once
    int fx_any_stride = 0;      // 1 (1 x 1 filters): any strides; a tile stages exactly the TW x TH positions its outputs read
    int fx_tail8 = 0;           // 0: C = 0 mod fx_ct; 1: the instance for C a multiple of 8 but not of fx_ct (the last c-slice partly
                                // filled); 2 (fp32): any C that is a multiple of 4
    int KT() const { return WM * MBLK * 32; }
    int NT() const { return TB * TW * TH; }
    int threads() const { return WM * WN * (pipelined == 2 ? 128 : 64); }
    int staging_threads() const { return WM * WN * 64; }
    bool f32v4() const { return reuse_r == -4; }
    int cgran() const { return dtype == 0 ? (f32v4() ? 4 : 1) : 16; }  // contraction granularity of the c-slice
};

// Everything a kernel needs, passed by value.
struct KernelArgs {
    const void* image;
    const void* filter;
    float* out;
    int32_t B, C, K, W, H, R, S, sw, sh, IW, IH;
    int32_t bR, bS, CT;       // contraction tile: r-range, s-range, c-slice (CT multiple of cgran)
    int32_t XS, YS;           // staged Image extents: sw*(TW-1)+bR, sh*(TH-1)+bS
    int32_t xpitch, ypitch;   // LDS pitches of the staged Image tile (fp32: floats; bf16: 16-byte units)
    int32_t fpitch;           // LDS pitch of one Filter row (one k), in elements
    int32_t QE;               // fp32: per-r contraction length bS*CT rounded up to even
    int32_t img_lds_elems;    // fp32: floats before the Filter tile; bf16: 16-byte units before it
    int32_t zero_off;         // fp32: offset (floats) of a zeroed row of 64 floats inside the Image region
    int32_t tiles_k, tiles_b, tiles_w, tiles_h;
    int32_t vec_img, vec_flt; // 1 = 16-byte global loads are legal for this operand
    FastDiv d_CT, d_YS, d_bS, d_bR, d_C8, d_RS, d_XS, d_C4;
    // pipelined kernels only
    int32_t n_tiles;          // Out tiles in the whole problem (all kernels)
    int32_t n_xcd;            // XCDs the dispatcher deals workgroups to (8 on MI355X); 1 = no remapping
    int32_t b_group;          // consecutive b-tiles whose Image rows share 128-byte lines (divides tiles_b)
    int32_t xcd_q, xcd_rem;   // n_tiles = n_xcd * xcd_q + xcd_rem
    // the tile list is k_groups blocks of grp tiles; inside a block the kpg k-tiles of the group are the fastest index
    // (k_groups = 1: the whole list is one block with all tiles_k k-tiles fastest); d_tk divides by kpg
    int32_t k_groups, kpg, grp;
    int32_t pos_fastest;      // 1: inside a block the position tiles of a k-tile are the fastest index, the k-tile the slowest
    int32_t npos;             // position tiles per block, grp / kpg
    FastDiv d_npos;           // its reciprocal
    FastDiv d_nxcd, d_tk, d_bg, d_tw, d_th;   // reciprocals of n_xcd, tiles_k, b_group, tiles_w, tiles_h
    int32_t img_items, flt_items;   // 16-byte staging items per slice
    int32_t img_buf, flt_buf; // size of one LDS buffer of each operand (fp32: floats; bf16: 16-byte units)
    int32_t flt_off;          // where the Filter buffers start (same unit)
    int32_t flt_resident;     // 1 = the Filter tile is the same for every unit of a workgroup: staged once
};

typedef int (*LaunchFn)(const KernelArgs& a, int grid, size_t lds_bytes, void* stream);

struct Variant {
    VariantInfo info;
    LaunchFn launch;
};

// Division of any n < 2^31 by a run-time constant: one multiply-high and a shift, exact.
struct FlatDiv {
    uint32_t mul;    // floor(2^(31 + l) / d) + 1 with l = ceil(log2 d), or 0 when d == 1
    uint32_t shift;  // l - 1
};

inline FlatDiv make_flatdiv(uint32_t d) {
    FlatDiv f = {0u, 0u};
    if (d <= 1) return f;
    uint32_t l = 0;
    while ((1ull << l) < d) ++l;
    f.mul = (uint32_t)((1ull << (31 + l)) / d + 1ull);
    f.shift = l - 1;
    return f;
}

constexpr uint32_t flat_div(uint32_t n, FlatDiv d) {
    return d.mul ? (uint32_t)(((uint64_t)n * d.mul) >> 32) >> d.shift : n;
}

// The tile of a workgroup of these kernels: the dispatcher deals workgroups to the 8 XCDs in turn, and every XCD gets one contiguous run
// of the tile list, q tiles and one more for the first rem of them.  The count is fixed, unlike that of the box tiles' order: on a
// device with fewer XCDs every tile is still taken once, in another order.  With the count as an argument (a division: 0.08 us of the
// 2.6 us of the smallest launches; a shift and a mask: two instructions more) two staged configurations, bf16 with 8 images per lane
// on 64 x 128 tiles and fp32 with 4 on 32 x 64, took 1.01 to 1.02 times as long in most of four builds.
constexpr uint32_t kFlatXcds = 8;
constexpr uint32_t xcd_order(uint32_t workgroup, uint32_t q, uint32_t rem) {
    const uint32_t l = workgroup / kFlatXcds, x = workgroup % kFlatXcds;
    return x * q + (x < rem ? x : rem) + l;
}

// The kernels with flattened positions (cacnn_flat.hip).  Out is a K x N matrix, N = H*W*B.  The contraction is cut
// into chunks of 16 bytes of the Filter (8 bf16 or 4 fp32 consecutive (s, c) of one filter column r).
struct FlatArgs {
    const void* image;
    const void* filter;
    float* out;
    uint32_t N, K, B, W;
    uint32_t G, groups;                 // groups of images per position, groups in all (H*W*G): one per lane
    uint32_t T, TC, U;                  // S*C; chunks per r; chunks in all, R*TC
    uint32_t back;                      // elements by which the last chunk of an r reaches beyond T (it is moved back by them)
    uint32_t steps, steps_per_wave;     // steps of two chunks; those of one of the waves that share a tile
    uint32_t img_w, img_h;              // Image bytes from one output column / row to the next
    uint32_t img_r, img_chunk;          // ... from one r to the next, from one chunk to the next
    uint32_t flt_row, flt_r;            // Filter bytes from one output channel / one r to the next
    uint32_t adv_tc, adv_flt, adv_img;  // from a chunk to the one that is fetched next in its place (2 or NCH further on)
    uint32_t wrap_flt, wrap_img;        // correction when that passes the end of an r
    int32_t img_bytes;
    uint32_t inner, k_inner;            // tile list: the fastest index, its length; 1: the k-tiles, 0: the position tiles
    uint32_t xcd_q, xcd_rem;
    FlatDiv d_G, d_W, d_TC, d_inner;
};
// A launch whose workgroups share a tile's contraction: parts of part_stages LDS stages each (the last may be shorter).
struct FlatSplitArgs : FlatArgs {
    uint32_t parts, part_stages, tiles;
    FlatDiv d_tiles;
};
// What the device's scratch memory for them holds: tiles, and words of partial sums.
constexpr uint32_t kSplitTiles = 4096, kSplitWords = 2u << 20;
struct FlatInfo {
    int dtype;          // cacnn_dtype
    int MB, NG;         // blocks of 32 of one wave: output channels, groups of images
    int IM;             // > 0: images a lane holds; < 0: all of that many, loaded in runs along the contraction
    int WM, WN, WK;     // waves along output channels, along positions, along the contraction
    int NCH;            // 0: operands straight from global memory (IM > 0); else chunks per LDS stage, and NG counts blocks of columns
    int threads() const { return WM * WN * WK * 64; }
    int KT() const { return WM * MB * 32; }
    int GT() const { return WN * NG * 32 / (NCH && IM > 0 ? IM : 1); }   // groups of images per tile
    int words() const { return KT() * WN * NG * 32 * (NCH && IM > 0 ? 1 : IM < 0 ? -IM : IM); }   // outputs of a tile
};
struct FlatVariant {
    FlatInfo info;
    int (*launch)(const FlatArgs& a, int grid, void* stream);
    int (*launch_split)(const FlatSplitArgs& a, int grid, void* stream);   // null: operands straight from global memory
};
int num_flat();
const FlatVariant& flat_variant(int i);

// The bf16 kernels that keep a tile's window in LDS (cacnn_window.hip).  Offsets and strides in bytes.
struct WindowArgs {
    const void* image;
    const void* filter;
    float* out;
    uint32_t N, K, B, C, W, H, sw, sh;
    uint32_t img_bytes;
    uint32_t img_x, img_w, img_h;                 // Image: one x, output column, output row further on
    uint32_t flt_k, flt_tap;                      // Filter: one output channel, one r further on
    uint32_t tw_shift, th_shift;                  // log2 of a tile's output columns / rows
    uint32_t tiles_b, tiles_h, tiles_n;           // position tiles along b and h, and in all
    uint32_t inner, k_inner, xcd_q, xcd_rem;      // tile list, as in FlatArgs
    uint32_t t_step;                              // position tiles from one of a workgroup's to the next
    uint32_t plane, rows;                         // rows of TB images in the box: of one x, in all
    uint32_t TC, U, UP, steps, back;              // chunks of one r, in all; those of a Filter row in LDS; steps; rows by which the last chunk of an r is moved back
    uint32_t off_r, adv_i, adv_off, wrap_off;     // LDS bytes from one r to the next; from a chunk to the one two further on
    uint32_t img_items;                           // 1 KiB pieces of the box that every wave loads
    uint32_t img_lds, flt_lds, zeros;             // LDS bytes of a box and of the Filter tile; where the zeros are
    FlatDiv d_inner, d_tb, d_th, d_plane, d_UP, d_TC;
};
constexpr int kWindowItems = 8;                   // 1 KiB pieces of the box that one wave loads, at most
struct WindowInfo {
    int MB, NB, WM, WN, TB;
    int threads() const { return WM * WN * 64; }
    int KT() const { return WM * MB * 32; }
    int cols() const { return WN * NB * 32; }
};
struct WindowVariant {
    WindowInfo info;
    int (*launch)(const WindowArgs& a, int grid, size_t lds, void* stream);
};
int num_window();
const WindowVariant& window_variant(int i);

// Pooling (cacnn_pool.hip): everything the kernel needs, by value.
struct PoolArgs {
    const void* image;
    float* out;
    int32_t B, C, W, H, R, S, sw, sh, IH;
    int32_t BV;               // groups of VEC adjacent images per (x, y, c): B / VEC
    int32_t TWC;              // output columns per chunk (the last chunk may overhang W)
    int32_t n_threads;        // chunks * H * TWC * C * BV
    int32_t n_wg, n_xcd, xcd_q, xcd_rem;   // workgroups, and the XCD remapping of their order
    int32_t img_bytes;        // size of the Image; 0: 2 GiB or more
    int32_t stream;           // 1: Out is stored past the caches
    FastDiv d_BV, d_C, d_TWC, d_H, d_nxcd;
};
// dtype: cacnn_dtype; mode: cacnn_pool_mode; vec: images per thread (1, 2, 4, bf16 also 8). 0 = launched.
int launch_pool(const PoolArgs& a, int dtype, int mode, int vec, void* stream);

// Measurement kernels (cacnn_probe.hip).  0 = launched.
int launch_mfma_probe(int dtype, const void* operands, float* sink, int iters, int grid, void* stream);
int launch_copy_probe(const void* src, void* dst, size_t bytes, int grid, void* stream);
int launch_lds_fill_probe(const void* src, uint32_t window, int iters, float* sink, int grid, void* stream);
int launch_mfma_and_fill_probe(int tile, const void* operands, const void* src, uint32_t window, int mfma_iters, int fill_iters,
                               int lds_reads, int barrier, float* sink, int grid, void* stream);

// Defined in cacnn_kernels.hip.
int num_variants();
const Variant& variant(int i);

}  // namespace cacnn
#endif
