// Host side of the cacnn C ABI: Theorem 1's bound, the tiling linear program of Section 5, the Appendix A case
// analysis, the gfx950 tile planner, argument validation and the launch dispatcher.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <list>
#include <memory>
#include <mutex>
#include <unordered_map>
#include <vector>

#include "../../include/cacnn.h"
#include "cacnn_internal.h"

using namespace cacnn;

namespace {

#include "cacnn_closed_form_table.inc"

const cacnn_machine kDefaultMachine = {160 * 1024, 512 * 1024, 256};

bool valid_problem(const cacnn_problem* p) {
    const int64_t v[9] = {p->B, p->C, p->K, p->W, p->H, p->R, p->S, p->sigma_w, p->sigma_h};
    for (int64_t x : v)
        if (x < 1) return false;
    return true;
}

// product with overflow detection; returns false on overflow past lim
bool mul_check(int64_t a, int64_t b, int64_t lim, int64_t* out) {
    if (a != 0 && b > lim / a) return false;
    *out = a * b;
    return true;
}

// ------------------------------------------------------------------------------------------------------------
// Section 5: the linear program over l_x = log_M(tile size of x), x in (b,c,k,w,h,r',r'',s',s'').
// maximise sum l_x  s.t.  l >= 0, each tile within its loop bound, Out / Filter / Image footprints <= M, the Image
// footprint (b_w + b_r')(b_h + b_s') being bounded term by term.  All right-hand sides are >= 0, so the slack basis
// is feasible and a plain primal simplex (Bland's rule) suffices.
struct LpSolution {
    double l[9];
    double log_volume;
};

// M_out, M_flt, M_img: the words the Out, Filter and Image tiles may occupy (the paper's LP has one M for all three; the
// gfx950 budget has accumulator registers for Out and LDS for the other two).  l[] and log_volume are logarithms to base
// `base`.
LpSolution solve_tiling_lp(const cacnn_problem& p, double M_out, double M_flt, double M_img, double base) {
    const int n = 9;
    enum { b_, c_, k_, w_, h_, r1_, r2_, s1_, s2_ };
    const double lnM = std::log(base);
    auto lg = [&](double x) { return std::log(x) / lnM; };
    const double sw = (double)std::min(p.sigma_w, p.R), sh = (double)std::min(p.sigma_h, p.S);

    std::vector<std::vector<double>> A;
    std::vector<double> rhs;
    auto row = [&](std::initializer_list<int> vars, double r) {
        std::vector<double> a(n, 0.0);
        for (int v : vars) a[v] += 1.0;
        A.push_back(a);
        rhs.push_back(std::max(r, 0.0));
    };
    row({b_}, lg((double)p.B));
    row({c_}, lg((double)p.C));
    row({k_}, lg((double)p.K));
    row({w_}, lg((double)p.W));
    row({h_}, lg((double)p.H));
    row({r2_}, lg(sw));
    row({s2_}, lg(sh));
    row({r1_}, lg((double)p.R) - lg(sw));
    row({s1_}, lg((double)p.S) - lg(sh));
    row({b_, k_, w_, h_}, lg(M_out));                    // Out tile
    row({c_, k_, r1_, r2_, s1_, s2_}, lg(M_flt));        // Filter tile
    row({b_, c_, w_, h_, r2_, s2_}, lg(M_img));          // Image tile, four products
    row({b_, c_, w_, s1_, r2_, s2_}, lg(M_img));
    row({b_, c_, r1_, h_, r2_, s2_}, lg(M_img));
    row({b_, c_, r1_, s1_, r2_, s2_}, lg(M_img));

    const int m = (int)A.size();
    // tableau: m rows x (n + m + 1) columns, objective row last; maximise sum x  <=>  reduced costs start at -1
    const int cols = n + m + 1;
    std::vector<std::vector<double>> T(m + 1, std::vector<double>(cols, 0.0));
    std::vector<int> basis(m);
    for (int i = 0; i < m; ++i) {
        for (int jx = 0; jx < n; ++jx) T[i][jx] = A[i][jx];
        T[i][n + i] = 1.0;
        T[i][cols - 1] = rhs[i];
        basis[i] = n + i;
    }
    for (int jx = 0; jx < n; ++jx) T[m][jx] = -1.0;
    const double eps = 1e-12;
    for (int iter = 0; iter < 10000; ++iter) {
        int enter = -1;
        for (int jx = 0; jx < n + m; ++jx)
            if (T[m][jx] < -1e-10) {
                enter = jx;  // Bland: lowest index
                break;
            }
        if (enter < 0) break;
        int leave = -1;
        double best = 0.0;
        for (int i = 0; i < m; ++i) {
            if (T[i][enter] > eps) {
                const double ratio = T[i][cols - 1] / T[i][enter];
                if (leave < 0 || ratio < best - 1e-14 || (std::fabs(ratio - best) <= 1e-14 && basis[i] < basis[leave])) {
                    leave = i;
                    best = ratio;
                }
            }
        }
        if (leave < 0) break;  // unbounded: cannot happen, every variable is capped
        const double piv = T[leave][enter];
        for (int jx = 0; jx < cols; ++jx) T[leave][jx] /= piv;
        for (int i = 0; i <= m; ++i) {
            if (i == leave) continue;
            const double f = T[i][enter];
            if (f != 0.0)
                for (int jx = 0; jx < cols; ++jx) T[i][jx] -= f * T[leave][jx];
        }
        basis[leave] = enter;
    }
    LpSolution s;
    for (int jx = 0; jx < n; ++jx) s.l[jx] = 0.0;
    for (int i = 0; i < m; ++i)
        if (basis[i] < n) s.l[basis[i]] = std::max(0.0, T[i][cols - 1]);
    s.log_volume = 0.0;
    for (int jx = 0; jx < n; ++jx) s.log_volume += s.l[jx];
    return s;
}

LpSolution solve_tiling_lp(const cacnn_problem& p, double M) { return solve_tiling_lp(p, M, M, M, M); }

// Appendix A, Theorem 2 (strides 1): which leaf of the decision tree the shape falls in.
int appendix_a_case(const cacnn_problem& p, double M) {
    if (p.sigma_w != 1 || p.sigma_h != 1) return 0;
    const double img = (double)p.C * p.H * p.W * p.B, flt = (double)p.K * p.C * p.R * p.S,
                 out = (double)p.K * p.H * p.W * p.B;
    if (std::min(img, std::min(flt, out)) <= M) {
        // Case 1, by which arrays exceed M (the sub-cases of the proof of the Case 1 lemma)
        const bool bi = img > M, bf = flt > M, bo = out > M;
        const double hwb = (double)p.H * p.W * p.B;
        if (!bi && !bf && !bo) return 11;
        if (bi && !bf && !bo) return 12;
        if (bo && !bf && !bi) return 13;
        if (bf && !bi && !bo) return (double)p.K * p.C <= M ? 14 : 15;
        if (bi && bo) return 16;
        if (bi && bf) return (double)p.K >= hwb ? 17 : 18;
        return (double)p.C >= hwb ? 19 : 110;
    }
    const double RS = (double)p.R * p.S, BHW = (double)p.B * p.H * p.W;
    if (RS >= M) return 21;
    if (M * RS >= BHW * BHW) return 221;
    if ((double)std::min(p.C, p.K) >= std::sqrt(M / RS)) return 2221;
    return 2222;
}

void bound_terms(const cacnn_problem& p, double M, cacnn_bound* out) {
    const double sw = (double)std::min(p.sigma_w, p.R), sh = (double)std::min(p.sigma_h, p.S);
    const double B = (double)p.B, C = (double)p.C, K = (double)p.K, W = (double)p.W, H = (double)p.H, R = (double)p.R,
                 S = (double)p.S;
    out->term[0] = B * K * W * H;
    out->term[1] = sw * sh * B * C * W * H;
    out->term[2] = C * K * R * S;
    out->term[3] = B * C * K * W * H * R * S / M;
    out->term[4] = B * C * K * W * H * std::sqrt(R * S * sw * sh / M);
    out->argmax = 0;
    for (int i = 1; i < 5; ++i)
        if (out->term[i] > out->term[out->argmax]) out->argmax = i;
    out->bound = out->term[out->argmax];
}

// Section 7: Theorem 1's terms with the Image replicated over the a_K groups of output channels and the Filter over
// the a_B a_W a_H groups of positions.
void parallel_terms(const cacnn_problem& p, double M, int64_t ab, int64_t ak, int64_t aw, int64_t ah, cacnn_bound* out) {
    bound_terms(p, M, out);
    out->term[1] *= (double)ak;
    out->term[2] *= (double)ab * (double)aw * (double)ah;
    out->argmax = 0;
    for (int i = 1; i < 5; ++i)
        if (out->term[i] > out->term[out->argmax]) out->argmax = i;
    out->bound = out->term[out->argmax];
}

// ------------------------------------------------------------------------------------------------------------
// gfx950 tile geometry for one (variant, contraction tile)

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
int64_t round_up(int64_t a, int64_t b) { return ceil_div(a, b) * b; }

struct Geometry {
    int CT, bR, bS, XS, YS, xpitch, ypitch, fpitch, QE, img_lds_elems, zero_off;
    int64_t lds_bytes;
    // pipelined variants
    int img_items, flt_items, img_buf, flt_buf, flt_off, flt_resident;
    int64_t n_slices;
    bool legal;   // the variant can run this geometry (staging items fit, packed fields fit)
};

Geometry make_geometry(const VariantInfo& v, const cacnn_problem& p, int CT, int bR, int bS, bool vec_img) {
    Geometry g;
    std::memset(&g, 0, sizeof(g));
    g.legal = true;
    g.CT = CT;
    g.bR = bR;
    g.bS = bS;
    {
        // Extents first, in 64 bits: a stride can be anything up to 2^31, and everything below is 32-bit arithmetic on
        // products of these.  A tile whose staged Image range or Filter tile cannot fit twice the largest LDS is refused
        // here; past this check every factor and every product of them stays below 2^20.
        // (a 1 x 1 kernel that takes any strides stages the positions its outputs read, not the range between them)
        const int64_t XS = v.fx_any_stride ? v.TW : p.sigma_w * (int64_t)(v.TW - 1) + bR,
                      YS = v.fx_any_stride ? v.TH : p.sigma_h * (int64_t)(v.TH - 1) + bS;
        const double esz0 = v.dtype == CACNN_F32 ? 4.0 : 2.0, cap = 2.0 * 160.0 * 1024.0;
        if (XS < 1 || YS < 1 || (double)XS * (double)YS * (double)CT * (double)v.TB * esz0 > cap ||
            (double)v.KT() * (double)bR * (double)bS * (double)CT * esz0 > cap) {
            g.legal = false;
            g.lds_bytes = INT64_MAX;
            return g;
        }
        g.XS = (int)XS;
        g.YS = (int)YS;
    }
    const int64_t Cpad = round_up(p.C, v.cgran());
    g.n_slices = ceil_div(p.R, bR) * ceil_div(p.S, bS) * ceil_div(Cpad, CT);
    g.flt_resident = (g.n_slices == 1 && ceil_div(p.K, v.KT()) == 1 && v.fx_ct == 0) ? 1 : 0;
    const int nbuf_f = g.flt_resident ? 1 : 2;
    if (v.fx_lds > 0) {
        // a fixed-geometry kernel: its own LDS layout, contraction tile and strides, a shape the tiles divide exactly
        g.lds_bytes = v.fx_lds;
        g.img_items = g.flt_items = 1;
        g.legal = CT == v.fx_ct && bR == v.fx_br && bS == v.fx_bs && g.YS == v.fx_ys &&
                  (v.fx_any_stride || (p.sigma_w == v.fx_sw && p.sigma_h == v.fx_sh)) &&
                  // (the kernels compiled for 1 x 1 filters take any filter one tap at a time)
                  (p.R == bR || (v.fx_any_stride && bR == 1)) && p.S % bS == 0 &&
                  (v.fx_tail8 == 2 ? p.C % 4 == 0 : v.fx_tail8 ? (p.C % CT != 0 && p.C % 8 == 0) : p.C % CT == 0) && vec_img &&
                  (v.fx_ragged == 2 || p.B % v.TB == 0) &&
                  (v.fx_ragged || (p.W % v.TW == 0 && p.H % v.TH == 0 && p.K % v.KT() == 0));
        if (v.fx_whole && (p.S != bS || p.C != CT)) g.legal = false;
        // staged words are addressed by 32-bit byte offsets from the unit's origin
        const double esz = v.dtype == CACNN_F32 ? 4.0 : 2.0;
        const double IHd = (double)(p.sigma_h * (p.H - 1) + p.S);
        const double reach = v.fx_any_stride ? (double)p.sigma_w * v.TW + (double)p.R : (double)(g.XS + 1);
        if (reach * IHd * (double)p.C * (double)p.B * esz >= 2147483648.0) g.legal = false;
        if ((double)(v.KT() + 1) * (double)p.R * (double)p.S * (double)p.C * esz >= 2147483648.0) g.legal = false;
        return g;
    }
    if (v.dtype == CACNN_F32 && v.f32v4()) {
        // 16-byte units: four consecutive contraction indices of one position
        const int G = CT / 4;
        g.ypitch = G * v.TB;
        const int base = g.YS * g.ypitch;
        int pad = 0;
        if (v.TB < 32) {
            // eight neighbouring staging lanes (b-quads fastest, then x) must land in eight different 16-byte slots
            const int want = v.TB >= 16 ? 2 : 1;
            while (((base + pad) & 7) != want) ++pad;
        }
        g.xpitch = base + pad;
        g.QE = (int)round_up((int64_t)bS * CT, 8);
        int f4 = bR * g.QE / 4;
        if ((f4 & 1) == 0) f4 += 1;     // odd count of 16-byte units: conflict-free A fragments
        g.fpitch = 4 * f4;
        g.img_buf = g.XS * g.xpitch;
        g.zero_off = 2 * g.img_buf;
        g.flt_off = g.zero_off + 32;
        g.flt_buf = v.KT() * f4;
        g.lds_bytes = 16ll * (g.flt_off + (int64_t)nbuf_f * g.flt_buf);
        g.img_items = g.XS * g.YS * G * (v.TB / 4);
        g.flt_items = v.KT() * bR * bS * G;
        g.legal = vec_img && v.TB % 4 == 0 && CT % 4 == 0 && (g.flt_resident || p.C % 4 == 0);
    } else if (v.dtype == CACNN_F32) {
        g.ypitch = CT * v.TB;
        int base = g.YS * g.ypitch;
        int pad = 0;
        if (v.TB < 32) {
            // spread the position groups of one MFMA column block over the 32 LDS banks: sigma_w * xpitch = TB (mod 32)
            int best = -1;
            for (int t = 0; t < 64; ++t) {
                if (vec_img && ((base + t) % 4) != 0) continue;
                if (best < 0) best = t;
                if (((int64_t)p.sigma_w * (base + t)) % 32 == v.TB % 32) {
                    best = t;
                    break;
                }
            }
            pad = best < 0 ? 0 : best;
        }
        g.xpitch = base + pad;
        g.QE = bS * CT + ((bS * CT) & 1);
        g.fpitch = bR * g.QE;
        if ((g.fpitch & 1) == 0) g.fpitch += 1;  // odd pitch: the 32 rows of an A fragment hit 32 different banks
        if (!v.pipelined) {
            g.zero_off = g.XS * g.xpitch;
            g.img_lds_elems = (int)round_up(g.zero_off + 64, 4);
            g.lds_bytes = 4ll * (g.img_lds_elems + (int64_t)v.KT() * g.fpitch);
        } else {
            g.img_buf = (int)round_up((int64_t)g.XS * g.xpitch, 4);
            g.zero_off = 2 * g.img_buf;
            g.flt_off = g.zero_off + 64;
            g.flt_buf = (int)round_up((int64_t)v.KT() * g.fpitch, 4);
            g.lds_bytes = 4ll * (g.flt_off + (int64_t)nbuf_f * g.flt_buf);
            g.img_items = g.XS * g.YS * CT * (v.TB / 4);
            g.flt_items = v.KT() * bR * bS * (CT / 4);
            g.legal = vec_img && v.TB % 4 == 0 && (g.flt_resident || (CT % 4 == 0 && p.C % 4 == 0));
        }
    } else {
        const int C8 = CT / 8;
        int f8 = bR * bS * C8;          // Filter row in 16-byte units; odd count keeps 16-byte reads conflict-free
        if ((f8 & 1) == 0) f8 += 1;
        g.fpitch = f8 * 8;
        g.ypitch = C8 * v.TB;           // 16-byte units, [c/8][b][8 c]
        g.xpitch = g.YS * g.ypitch;
        if (!v.pipelined) {
            g.img_lds_elems = g.XS * g.xpitch;
            g.lds_bytes = 16ll * g.img_lds_elems + 2ll * v.KT() * g.fpitch;
        } else {
            g.img_buf = g.XS * g.xpitch;
            g.flt_off = 2 * g.img_buf;
            g.flt_buf = v.KT() * f8;
            g.lds_bytes = 16ll * (g.flt_off + (int64_t)nbuf_f * g.flt_buf);
            g.img_items = g.XS * g.YS * C8 * (v.TB / 8);    // 8 channels x 8 images each
            g.flt_items = v.KT() * bR * bS * C8;
            g.legal = vec_img && v.TB % 8 == 0 && (g.flt_resident || p.C % 8 == 0);
        }
    }
    if (v.reuse_r > 0 && (bR != v.reuse_r || p.sigma_w != 1)) g.legal = false;
    if (v.pipelined) {
        const int64_t thr = v.staging_threads();
        if (g.img_items > v.MAXI * thr || (!g.flt_resident && g.flt_items > v.MAXF * thr)) g.legal = false;
        if (g.XS > 1023 || g.YS > 1023 || CT > 1023 || bR > 127 || bS > 127 || v.KT() > 256) g.legal = false;
        // staging items are addressed by 32-bit byte offsets from the unit's origin
        const double esz = v.dtype == CACNN_F32 ? 4.0 : 2.0;
        const double IHd = (double)(p.sigma_h * (p.H - 1) + p.S);
        const double reach = v.fx_any_stride ? (double)p.sigma_w * v.TW + 1.0 : (double)(g.XS + 1);
        if (reach * IHd * (double)p.C * (double)p.B * esz >= 2147483648.0) g.legal = false;
        if ((double)(v.KT() + 1) * (double)p.R * (double)p.S * (double)p.C * esz >= 2147483648.0) g.legal = false;
    }
    return g;
}

struct Choice {
    int variant = -1;
    Geometry g{};
    double cost = 0.0;
    int64_t n_wg = 0;
    double words = 0.0;       // words staged from global memory by the whole grid
    double img_words = 0.0;   // the Image part of them
    // the cost model's terms for the chosen geometry, in CU cycles: tiles per CU, MFMA time, staging time and
    // contraction slices per tile, Out drain
    double terms[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
};

// words staged from global memory by the whole grid for one variant/geometry, clipped to the arrays
double staged_words(const VariantInfo& v, const cacnn_problem& p, const Geometry& g, double* image_words) {
    const int64_t tiles_k = ceil_div(p.K, v.KT()), tiles_b = ceil_div(p.B, v.TB), tiles_w = ceil_div(p.W, v.TW),
                  tiles_h = ceil_div(p.H, v.TH);
    const int64_t IW = p.sigma_w * (p.W - 1) + p.R, IH = p.sigma_h * (p.H - 1) + p.S;
    double sum_x = 0.0, sum_y = 0.0;
    for (int64_t r0 = 0; r0 < p.R; r0 += g.bR)
        for (int64_t tw = 0; tw < tiles_w; ++tw) {
            const int64_t lo = p.sigma_w * tw * v.TW + r0;
            sum_x += (double)std::max<int64_t>(0, std::min<int64_t>(IW, lo + g.XS) - lo);
        }
    for (int64_t s0 = 0; s0 < p.S; s0 += g.bS)
        for (int64_t th = 0; th < tiles_h; ++th) {
            const int64_t lo = p.sigma_h * th * v.TH + s0;
            sum_y += (double)std::max<int64_t>(0, std::min<int64_t>(IH, lo + g.YS) - lo);
        }
    const double image = (double)tiles_k * sum_x * sum_y * (double)p.C * (double)p.B;
    const double filter = (double)tiles_b * tiles_w * tiles_h * (double)p.K * p.R * p.S * p.C;
    if (image_words) *image_words = image;
    return image + filter;
}

bool vec_img_ok(const VariantInfo& v, const cacnn_problem& p) {
    const int vi = v.dtype == CACNN_F32 ? 4 : 8;
    return v.TB % vi == 0 && p.B % vi == 0;
}

// Cost model in CU cycles: MFMA issue time of one wavefront plus the staging time of the workgroup, times the
// number of workgroups a compute unit has to run.  Staging overlaps MFMA only when two workgroups share a CU.
// Coefficients of the generic kernels' cost model (see evaluate): cycles per MFMA-pipe cycle, per staging cycle, per
// contraction slice, per Out-drain cycle, and the constant part of a launch.
struct ModelCoef {
    double mfma, stage, slice, drain, fixed;
};

const ModelCoef& model_coef(const VariantInfo& v) {
    static const ModelCoef one_tile_bf16 = {4.926, 1.741, 7.1, 0.02466, 17060.0};
    static const ModelCoef one_tile_f32 = {2.459, 2.334, 8696.0, 0.1144, 1322.0};
    static const ModelCoef pipe_bf16 = {2.696, 0.0, 5385.0, 0.0928, 15510.0};
    static const ModelCoef pipe3_bf16 = {1.525, 0.0, 4127.0, 0.0, 27740.0};
    static const ModelCoef pipe_f32 = {1.667, 0.0, 6584.0, 0.1336, 4643.0};
    static const ModelCoef ws_bf16 = {2.236, 0.0, 2918.0, 0.0, 24020.0};
    static const ModelCoef ws3_bf16 = {1.358, 0.0, 1926.0, 0.0, 34050.0};
    static const ModelCoef ws_f32 = {1.514, 0.0, 2807.0, 0.2543, 11870.0};
    static const ModelCoef ws4_f32 = {1.284, 0.0, 5212.0, 0.2865, 7469.0};
    const bool f32 = v.dtype == CACNN_F32;
    if (v.pipelined == 0) return f32 ? one_tile_f32 : one_tile_bf16;
    if (v.pipelined == 1) return f32 ? pipe_f32 : (v.reuse_r > 0 ? pipe3_bf16 : pipe_bf16);
    return f32 ? (v.f32v4() ? ws4_f32 : ws_f32) : (v.reuse_r > 0 ? ws3_bf16 : ws_bf16);
}

bool evaluate(int vi, const cacnn_problem& p, const cacnn_machine& mach, Choice* best) {
    const VariantInfo& v = variant(vi).info;
    // fp32 slices in multiples of 4 channels keep the 16-byte Filter loads legal
    const int gran = (v.dtype == CACNN_F32 && p.C % 4 == 0) ? 4 : v.cgran();   // v.cgran() is 4 for the v4 layout
    const int Cpad = (int)std::min<int64_t>(round_up(p.C, gran), 1 << 20);
    // candidate contraction tiles: every even split of the (padded) channel range, and halvings of the s and r ranges
    std::vector<int> cts;
    for (int d = 1; d <= 64; ++d) {
        const int ct = (int)round_up(ceil_div(Cpad, d), gran);
        if (cts.empty() || cts.back() != ct) cts.push_back(ct);
        if (ct == gran) break;
    }
    if (v.fx_ct > 0) cts.assign(1, v.fx_ct);      // a fixed-geometry kernel has one c-slice (it may exceed a small C)
    const bool vimg = vec_img_ok(v, p);
    bool found = false;
    const int64_t tiles_k = ceil_div(p.K, v.KT()), tiles_b = ceil_div(p.B, v.TB), tiles_w = ceil_div(p.W, v.TW),
                  tiles_h = ceil_div(p.H, v.TH);
    int64_t n_wg = 0, t = 0;
    if (!mul_check(tiles_k, tiles_b, INT32_MAX, &t) || !mul_check(t, tiles_w, INT32_MAX, &t) ||
        !mul_check(t, tiles_h, INT32_MAX, &n_wg))
        return false;
    const double ebytes = v.dtype == CACNN_F32 ? 4.0 : 2.0;
    // global runs shorter than 32 bytes along b waste the rest of each 32-byte sector
    const double run_bytes = (double)std::min<int64_t>(v.TB, p.B) * ebytes;
    const double waste = std::max(1.0, 32.0 / run_bytes);
    for (int bR = (int)std::min<int64_t>(p.R, 1 << 12); bR >= 1; bR = (bR + 1) / 2 == bR ? 0 : (bR + 1) / 2) {
        for (int bS = (int)std::min<int64_t>(p.S, 1 << 12); bS >= 1; bS = (bS + 1) / 2 == bS ? 0 : (bS + 1) / 2) {
            for (int ct : cts) {
                const Geometry g = make_geometry(v, p, ct, bR, bS, vimg);
                if (!g.legal || g.lds_bytes > mach.lds_bytes) continue;
                double img_words = 0.0;
                const double words = staged_words(v, p, g, &img_words);
                // Cost model, in compute-unit cycles, for the generic kernels.  Four quantities of the launch:
                //   t_mfma   MFMA pipe time of one wavefront for one Out tile (64 cycles per fp32 32x32x2, 32 per bf16
                //            32x32x16);
                //   t_stage  staged bytes of the tile at 16 B/clk (runs shorter than 32 bytes along b waste the rest of
                //            each sector);
                //   n_ctiles contraction slices per tile (each costs a barrier and exposed latency);
                //   t_out    the Out tile draining to HBM at ~1 TB/s for the whole chip;
                // and per_cu, the Out tiles a compute unit runs one after the other.  The launch time is a non-negative
                // linear combination of them plus a constant, with one set of coefficients per kernel family, fitted
                // (least squares on the relative error) to the measured launch times of every generic variant on 28
                // calibration layers (bench.py --planner-sweep calibration).
                // (a kernel that reuses Image fragments over three taps r runs a last r-slice of fewer taps at the cost of a
                // whole one)
                const double r_run = v.reuse_r > 0 ? (double)round_up(p.R, v.reuse_r) : (double)p.R;
                const double ksteps = v.dtype != CACNN_F32 ? r_run * p.S * (Cpad / 16)
                                      : v.f32v4()          ? (double)p.R * (double)round_up((int64_t)p.S * Cpad, 8) / 2.0
                                                           : (double)p.R * ceil_div((int64_t)p.S * Cpad, 2);
                const double t_mfma = (v.dtype == CACNN_F32 ? 64.0 : 32.0) * v.MBLK * v.NBLK * ksteps;
                const double t_stage = (img_words * waste + (words - img_words)) * ebytes / (double)n_wg / 16.0;
                const double n_ctiles = (double)g.n_slices;
                const double t_out = (double)v.KT() * v.NT() * 4.0 * waste * (double)mach.num_cu / 1.0e12 * 2.4e9;
                const ModelCoef& mc = model_coef(v);
                const double per_cu = (double)ceil_div(n_wg, mach.num_cu);
                double cost = per_cu * (mc.mfma * t_mfma + mc.stage * t_stage + mc.slice * n_ctiles) +
                              mc.drain * t_out / std::max(1.0, std::min(per_cu, 4.0)) + mc.fixed;
                // the fixed-geometry kernels run one schedule: priced by what a unit was measured to take
                if (v.fx_unit_us > 0.f) {
                    double rounds = per_cu;
                    if (v.fx_calib_cus > 0) {
                        // the bf16 MFMA rate is the chip's (its power-managed clock), not the compute unit's: measured, a unit
                        // takes 1.13 to 1.2 times as long on 256 busy compute units as on 224 or 196, and 0.72 to 0.8 times
                        // on 128; (n / n_calibration)^0.8, not below 0.75, is within a few per cent of those.  Full rounds of
                        // tiles run on all compute units, the last round on what is left.
                        auto scale = [&](double busy) { return std::max(0.75, std::pow(busy / (double)v.fx_calib_cus, 0.8)); };
                        const int64_t full = n_wg / mach.num_cu, rest = n_wg % mach.num_cu;
                        rounds = (double)full * scale((double)mach.num_cu) + (rest ? scale((double)rest) : 0.0);
                    }
                    // a compute unit that runs several tiles one after the other pays, for each one after the first, the
                    // empty pipeline at the tile's start and the stores at its end (about 2 us, measured on 1 x 1 layers
                    // of 1 to 4 units per tile); the first tile's share is in the variant's fixed time
                    const double tile_us = v.fx_calib_cus > 0 ? 2.0 * (per_cu - 1.0) : 0.0;
                    // (a bf16 kernel compiled for 1 x 1 filters that walks the taps of a larger filter: its units were
                    // measured to take 1.1 to 1.17 times a 1 x 1 layer's on 3 x 3 layers with strides 2)
                    const double taps = v.fx_calib_cus > 0 && v.fx_any_stride && (p.R > 1 || p.S > 1) ? 1.12 : 1.0;
                    cost = (rounds * n_ctiles * (double)v.fx_unit_us * taps + tile_us + (double)v.fx_fixed_us) * 2400.0;
                }
                if (best->variant < 0 || cost < best->cost) {
                    best->variant = vi;
                    best->g = g;
                    best->cost = cost;
                    best->n_wg = n_wg;
                    best->words = words;
                    best->img_words = img_words;
                    best->terms[0] = per_cu;
                    best->terms[1] = t_mfma;
                    best->terms[2] = t_stage;
                    best->terms[3] = n_ctiles;
                    best->terms[4] = t_out;
                }
                found = true;
            }
        }
    }
    return found;
}

// ------------------------------------------------------------------------------------------------------------
// The generic kernels' tile, sized from the Section 5 linear program at the gfx950 budget.  The paper bounds three
// tiles by one M; here the Out tile lives in accumulator registers (at most 7 MFMA blocks of 32 x 32 per multiplying
// wave, four such waves: 28672 words) and the Image and Filter tiles share the LDS, double-buffered, so each may take a
// quarter of it (the paper's own slack: per-array bounds instead of a bound on the sum).  The LP's optimum gives the
// Out tile's two extents k* and P* = b*w*h and says how much of the filter a contraction tile should cover; the compiled
// variant nearest to (k*, P*) in log distance is launched, where padding (tile extents beyond the problem's), an uneven
// or short tile count over the compute units (Section 7: divide the output over all processors) and the kernel family
// (measured ratios between the one-tile, pipelined and wave-specialised kernels on the same tile) add to the distance.
// The contraction tile is the one of largest volume b_c b_r b_s the LDS really holds, whole filter extents first as in
// the LP's optimum for R S << M (Appendix A, Case 2.2.2.1: b_R = R, b_S = S).
struct GpuLpTile {
    double k, P, c, r, s;
};

GpuLpTile solve_gpu_lp(const cacnn_problem& p, int dtype, const cacnn_machine& mach) {
    const double esz = dtype == CACNN_F32 ? 4.0 : 2.0;
    const double M_acc = 28672.0, M_lds = std::max(2.0, (double)mach.lds_bytes / (4.0 * esz));
    const LpSolution s = solve_tiling_lp(p, M_acc, M_lds, M_lds, std::exp(1.0));
    GpuLpTile t;
    t.k = std::exp(s.l[2]);
    t.P = std::exp(s.l[0] + s.l[3] + s.l[4]);
    t.c = std::exp(s.l[1]);
    t.r = std::exp(s.l[5] + s.l[6]);
    t.s = std::exp(s.l[7] + s.l[8]);
    return t;
}

bool evaluate_lp(int vi, const cacnn_problem& p, const cacnn_machine& mach, const GpuLpTile& lp, Choice* best) {
    const VariantInfo& v = variant(vi).info;
    const int gran = (v.dtype == CACNN_F32 && p.C % 4 == 0) ? 4 : v.cgran();
    const int Cpad = (int)std::min<int64_t>(round_up(p.C, gran), 1 << 20);
    const bool vimg = vec_img_ok(v, p);
    const int64_t tiles_k = ceil_div(p.K, v.KT()), tiles_b = ceil_div(p.B, v.TB), tiles_w = ceil_div(p.W, v.TW),
                  tiles_h = ceil_div(p.H, v.TH);
    int64_t n_wg = 0, t = 0;
    if (!mul_check(tiles_k, tiles_b, INT32_MAX, &t) || !mul_check(t, tiles_w, INT32_MAX, &t) ||
        !mul_check(t, tiles_h, INT32_MAX, &n_wg))
        return false;
    // the contraction tile of largest volume that is legal and fits: whole filter extents first, then the c-slice
    Geometry g_best{};
    double vol_best = -1.0;
    for (int bR = (int)std::min<int64_t>(p.R, 1 << 12); bR >= 1; bR = (bR + 1) / 2 == bR ? 0 : (bR + 1) / 2)
        for (int bS = (int)std::min<int64_t>(p.S, 1 << 12); bS >= 1; bS = (bS + 1) / 2 == bS ? 0 : (bS + 1) / 2)
            for (int d = 1; d <= 64; ++d) {
                const int ct = (int)round_up(ceil_div(Cpad, d), gran);
                const Geometry g = make_geometry(v, p, ct, bR, bS, vimg);
                if (g.legal && g.lds_bytes <= mach.lds_bytes) {
                    // volume, with a premium on covering the filter extents (the halo re-staging the LP's optimum avoids)
                    const double vol = (double)std::min<int64_t>(ct, p.C) * bR * bS * ((int64_t)bR * bS == p.R * p.S ? 4.0 : 1.0);
                    if (vol > vol_best) {
                        vol_best = vol;
                        g_best = g;
                    }
                    break;      // smaller c-slices of the same (b_r, b_s) only lose volume
                }
                if (ct == gran) break;
            }
    if (vol_best < 0.0) return false;
    const double ku = (double)std::min<int64_t>(v.KT(), p.K);
    const double Pu = (double)std::min<int64_t>(v.TB, p.B) * (double)std::min<int64_t>(v.TW, p.W) * (double)std::min<int64_t>(v.TH, p.H);
    double dist = std::fabs(std::log(ku / lp.k)) + std::fabs(std::log(Pu / lp.P));
    dist += std::log((double)v.KT() * v.NT() / (ku * Pu));                          // padded MFMA rows and columns
    // global runs along b shorter than a 64-byte half line use a fraction of every line they touch
    dist += std::log(std::max(1.0, 64.0 / ((double)std::min<int64_t>(v.TB, p.B) * (v.dtype == CACNN_F32 ? 4.0 : 2.0))));
    const int64_t resident = std::max<int64_t>(1, std::min<int64_t>(v.occ, mach.lds_bytes / std::max<int64_t>(1, g_best.lds_bytes)));
    const double slots = (double)mach.num_cu * (v.pipelined ? 1.0 : (double)resident);
    dist += std::log((double)ceil_div(n_wg, (int64_t)slots) * slots / (double)n_wg);    // idle or unevenly loaded compute units
    dist += v.pipelined == 2 ? 0.0 : (v.pipelined == 1 ? std::log(1.3) : std::log(2.5));  // kernel family
    dist += std::log((double)v.tune);
    if (best->variant < 0 || dist < best->cost) {
        best->variant = vi;
        best->g = g_best;
        best->cost = dist;
        best->n_wg = n_wg;
        best->words = staged_words(v, p, g_best, &best->img_words);
    }
    return true;
}

// Measured against the fastest of all variants (cacnn_tune) on sixteen mid-size and ragged layers, the LP-sized choice is
// 1.38x slower in the geometric mean (worst 2.1x) and the calibrated cycle model 1.34x (worst 2.5x): on problems this
// small what separates the variants is how well each kernel family keeps its pipeline full, which neither the LP nor
// the model prices well.  The cycle model stays the default; CACNN_PLANNER=lp selects the LP-sized choice.
bool planner_uses_lp() {
    static const bool lp = [] {
        const char* e = std::getenv("CACNN_PLANNER");
        return e && std::strcmp(e, "lp") == 0;
    }();
    return lp;
}

// workgroups launched: one per Out tile, or for the persistent kernels as many as the machine holds at once
int64_t launch_grid(const VariantInfo& v, const Geometry& g, int64_t n_tiles, const cacnn_machine& mach) {
    if (!v.pipelined) return n_tiles;
    const int64_t resident =
        std::max<int64_t>(1, std::min<int64_t>(v.occ, mach.lds_bytes / std::max<int64_t>(1, g.lds_bytes)));
    return std::min<int64_t>(n_tiles, mach.num_cu * resident);
}

// XCD count used for the tile remapping of the box tiles and of pooling; CACNN_XCDS=1 switches the remapping off (debugging aid)
int xcd_count() {
    static int n = [] {
        const char* e = std::getenv("CACNN_XCDS");
        const int v = e ? std::atoi(e) : 8;
        return v >= 1 && v <= 64 ? v : 8;
    }();
    return n;
}

// Section 7 with the XCDs as the processors and the arrays' real sizes: divide the XCDs into a_K groups of output
// channels and n_xcd / a_K ranges of positions; an XCD then fetches 1 / a_K of the Filter and the Image is fetched a_K
// times over all XCDs.  a_K must divide both the XCD count and the k-tile count (whole k-tiles per group).
int choose_xcd_split_k(const cacnn_problem& p, int dtype, int64_t tiles_k, int n_xcd) {
    const double esz = dtype == CACNN_F32 ? 4.0 : 2.0;
    const double img = (double)(p.sigma_w * (p.W - 1) + p.R) * (double)(p.sigma_h * (p.H - 1) + p.S) * (double)p.C *
                       (double)p.B * esz;
    const double flt = (double)p.K * p.R * p.S * p.C * esz;
    int best = 1;
    double best_bytes = img + (double)n_xcd * flt;
    for (int ak = 2; ak <= n_xcd; ak *= 2) {
        if (n_xcd % ak || tiles_k % ak) continue;
        const double bytes = (double)ak * img + (double)(n_xcd / ak) * flt;
        if (bytes < best_bytes) {
            best = ak;
            best_bytes = bytes;
        }
    }
    return best;
}

// ------------------------------------------------------------------------------------------------------------
// Two levels: the words the XCDs' L2s fetch for one way of laying out an XCD's run of tiles (a_K groups of k-tiles, walk
// order inside a group).  A model of the launch: workgroup i belongs to XCD i % n_xcd and takes the tiles at places
// i / n_xcd, i / n_xcd + grid / n_xcd, ... of its XCD's contiguous run of the tile list; an XCD's round n is every
// workgroup's n-th tile; a tile reads the Filter rows of its k-tile (one atom) and the Image columns of its position
// tile (one atom per input pixel and image group: all channels); an L2 keeps atoms in LRU order up to its size.
struct L2Machine {
    double words;      // one L2, in input words
    int n_xcd, cu_per_xcd;
};
constexpr L2Machine kDefaultL2Bytes = {4.0 * 1024.0 * 1024.0, 8, 32};

struct TileGeom {
    int KT, TB, TW, TH, b_group;
    int64_t grid;
};

int b_group_of(const VariantInfo& v, int dtype, int64_t tiles_b) {
    // b-tiles that read different pieces of the same 128-byte Image lines stay adjacent in the tile order
    const int64_t esz = dtype == CACNN_F32 ? 4 : 2;
    const int64_t want = std::max<int64_t>(1, 128 / (int64_t)(v.TB * esz));
    int g_b = 1;
    for (int d = 1; d <= tiles_b && d <= want; ++d)
        if (tiles_b % d == 0) g_b = d;
    return g_b;
}

// -1: not simulated (too large)
double l2_model_words(const cacnn_problem& p, const TileGeom& tg, int a_k, int walk, const L2Machine& m2) {
    const int64_t tk = ceil_div(p.K, tg.KT), tb = ceil_div(p.B, tg.TB), tw = ceil_div(p.W, tg.TW), th = ceil_div(p.H, tg.TH);
    const int64_t npos = tb * tw * th, n_tiles = tk * npos, kpg = tk / a_k;
    const int64_t IW = p.sigma_w * (p.W - 1) + p.R, IH = p.sigma_h * (p.H - 1) + p.S;
    const int64_t XS = p.sigma_w * (tg.TW - 1) + p.R, YS = p.sigma_h * (tg.TH - 1) + p.S;
    if ((double)n_tiles > 1.0e5) return -1.0;     // the walk costs about half a microsecond per tile and candidate
    const int64_t q = n_tiles / m2.n_xcd, rem = n_tiles % m2.n_xcd;
    const int64_t per_xcd = std::max<int64_t>(1, tg.grid / m2.n_xcd);
    double total = 0.0;
    std::vector<int64_t> atoms;
    for (int x = 0; x < m2.n_xcd; ++x) {
        const int64_t lo = x * q + std::min<int64_t>(x, rem), hi = lo + q + (x < rem ? 1 : 0);
        // LRU over atom ids: id < tk is the Filter atom of a k-tile, tk + position tile the Image footprint of that tile.
        // Position tiles that overlap in their halo are separate atoms: measured, an XCD's L2 serves a line to the
        // workgroups of one position tile (they fetch it in the same microsecond) but has turned it over before a
        // neighbouring position tile asks for it.
        std::list<std::pair<int64_t, double>> lru;
        std::unordered_map<int64_t, std::list<std::pair<int64_t, double>>::iterator> where;
        double used = 0.0;
        for (int64_t n0 = lo; n0 < hi; n0 += per_xcd) {
            atoms.clear();
            for (int64_t t = n0; t < std::min(hi, n0 + per_xcd); ++t) {
                const int64_t kg = t / (kpg * npos), tl = t - kg * kpg * npos;
                int64_t k_l, pos;
                if (walk == 0) {
                    k_l = tl % kpg;
                    pos = tl / kpg;
                } else {
                    pos = tl % npos;
                    k_l = tl / npos;
                }
                const int64_t b_lo = pos % tg.b_group, w_i = (pos / tg.b_group) % tw, h_i = (pos / (tg.b_group * tw)) % th,
                              b_i = (pos / (tg.b_group * tw * th)) * tg.b_group + b_lo;
                atoms.push_back(kg * kpg + k_l);
                atoms.push_back(tk + (b_i * tw + w_i) * th + h_i);
            }
            std::sort(atoms.begin(), atoms.end());
            atoms.erase(std::unique(atoms.begin(), atoms.end()), atoms.end());
            for (int64_t id : atoms) {
                auto it = where.find(id);
                if (it != where.end()) {
                    lru.splice(lru.end(), lru, it->second);
                    continue;
                }
                double sz;
                if (id < tk) {
                    sz = (double)std::min<int64_t>(tg.KT, p.K - id * tg.KT) * (double)p.R * p.S * p.C;
                } else {
                    const int64_t pt = id - tk, h_i = pt % th, w_i = (pt / th) % tw, b_i = pt / (th * tw);
                    const int64_t xs = std::min(IW, p.sigma_w * w_i * tg.TW + XS) - p.sigma_w * w_i * tg.TW,
                                  ys = std::min(IH, p.sigma_h * h_i * tg.TH + YS) - p.sigma_h * h_i * tg.TH;
                    sz = (double)std::min<int64_t>(tg.TB, p.B - b_i * tg.TB) * (double)p.C * (double)(xs * ys);
                }
                total += sz;
                lru.emplace_back(id, sz);
                where[id] = std::prev(lru.end());
                used += sz;
                while (used > m2.words && lru.size() > 1) {
                    used -= lru.front().second;
                    where.erase(lru.front().first);
                    lru.pop_front();
                }
            }
        }
    }
    return total + (double)p.K * p.H * p.W * p.B;
}

struct L2Choice {
    int a_k = 1, walk = 0, n = 0;
    int cand_a_k[8] = {0}, cand_walk[8] = {0};
    double cand_words[8] = {0.0};
    double words = 0.0;
};

L2Choice choose_l2_layout(const cacnn_problem& p, int dtype, const VariantInfo& v, int64_t grid, const L2Machine& m2) {
    L2Choice c;
    const int64_t tk = ceil_div(p.K, v.KT());
    TileGeom tg{v.KT(), v.TB, v.TW, v.TH, b_group_of(v, dtype, ceil_div(p.B, v.TB)), grid};
    const int64_t n_tiles = tk * ceil_div(p.B, v.TB) * ceil_div(p.W, v.TW) * ceil_div(p.H, v.TH);
    for (int ak = 1; ak <= m2.n_xcd && ak <= 8; ak *= 2) {
        if (m2.n_xcd % ak || tk % ak) continue;
        for (int walk = 0; walk < 2; ++walk) {
            // the walk order only differs when a group has several k-tiles; its decoding needs n_tiles * npos < 2^32
            if (walk == 1 && (tk / ak < 2 || (double)n_tiles * (double)(n_tiles / tk) >= 4294967296.0)) continue;
            const double w = l2_model_words(p, tg, ak, walk, m2);
            if (w < 0.0) {
                c = L2Choice();
                c.a_k = choose_xcd_split_k(p, dtype, tk, m2.n_xcd);
                return c;
            }
            c.cand_a_k[c.n] = ak;
            c.cand_walk[c.n] = walk;
            c.cand_words[c.n] = w;
            // a later layout must save more than the few per cent the model is off by on the measured layouts
            if (c.n == 0 || w < 0.97 * c.words) {
                c.words = w;
                c.a_k = ak;
                c.walk = walk;
            }
            ++c.n;
        }
    }
    return c;
}

int fill_plan(const cacnn_problem& p, int dtype, const cacnn_machine& mach, const Choice& ch, cacnn_plan* out) {
    const VariantInfo& v = variant(ch.variant).info;
    const double esz = dtype == CACNN_F32 ? 4.0 : 2.0;
    const double M = (double)mach.lds_bytes / esz;
    std::memset(out, 0, sizeof(*out));
    if (M > 1.0) {
        const LpSolution s = solve_tiling_lp(p, M);
        for (int i = 0; i < 9; ++i) out->lp_tile[i] = std::pow(M, s.l[i]);
        out->lp_volume = std::pow(M, s.log_volume);
        const double F = (double)p.B * p.C * p.K * p.W * p.H * p.R * p.S;
        out->lp_cost_words = F * M / out->lp_volume;
        cacnn_bound b;
        bound_terms(p, M, &b);
        out->bound_words = b.bound;
        out->paper_case = appendix_a_case(p, M);
    }
    out->variant = ch.variant;
    out->b_b = v.TB;
    out->b_c = ch.g.CT;
    out->b_k = v.KT();
    out->b_w = v.TW;
    out->b_h = v.TH;
    out->b_r = ch.g.bR;
    out->b_s = ch.g.bS;
    out->b_r2 = (int32_t)std::min<int64_t>(p.sigma_w, ch.g.bR);
    out->b_r1 = (int32_t)ceil_div(ch.g.bR, std::max<int64_t>(1, std::min<int64_t>(p.sigma_w, p.R)));
    out->b_s2 = (int32_t)std::min<int64_t>(p.sigma_h, ch.g.bS);
    out->b_s1 = (int32_t)ceil_div(ch.g.bS, std::max<int64_t>(1, std::min<int64_t>(p.sigma_h, p.S)));
    out->grid[0] = (int32_t)launch_grid(v, ch.g, ch.n_wg, mach);
    out->grid[1] = 1;
    out->grid[2] = 1;
    out->block = v.threads();
    out->lds_bytes_used = ch.g.lds_bytes;
    out->tile_volume = (double)v.TB * ch.g.CT * v.KT() * v.TW * v.TH * ch.g.bR * ch.g.bS;
    double staged = ch.words;
    // a kernel that takes a tile's whole contraction as one unit keeps its Filter tile while the output channels stay
    // the same: with one k-tile it is staged once per workgroup, not once per Out tile
    if (v.fx_whole && ceil_div(p.K, v.KT()) == 1)
        staged = ch.img_words + (double)out->grid[0] * (double)p.K * p.R * p.S * p.C;
    out->predicted_words = staged + (double)p.K * p.H * p.W * p.B;
    {
        L2Machine m2 = kDefaultL2Bytes;
        m2.words /= esz;
        m2.n_xcd = xcd_count();
        const L2Choice l2 = choose_l2_layout(p, dtype, v, out->grid[0], m2);
        out->xcd_split_k = l2.a_k;
        out->xcd_walk = l2.walk;
    }
    return CACNN_OK;
}

// per-array element counts must fit the kernels' 31-bit tile arithmetic
int validate_dims(const cacnn_problem& pr) {
    const cacnn_problem* p = &pr;
    const int64_t IW = p->sigma_w * (p->W - 1) + p->R, IH = p->sigma_h * (p->H - 1) + p->S;
    int64_t t;
    const int64_t lim = INT32_MAX;
    if (p->sigma_w > lim || p->sigma_h > lim || p->W > lim || p->H > lim || p->R > lim || p->S > lim ||
        IW > lim || IH > lim || IW < 1 || IH < 1)
        return CACNN_ERR_INVALID_ARG;
    if (!mul_check(IW, IH, lim, &t) || !mul_check(t, p->C, lim, &t) || !mul_check(t, p->B, lim, &t))
        return CACNN_ERR_INVALID_ARG;
    if (!mul_check(p->K, p->R, lim, &t) || !mul_check(t, p->S, lim, &t) || !mul_check(t, p->C, lim, &t))
        return CACNN_ERR_INVALID_ARG;
    if (!mul_check(p->K, p->H, lim, &t) || !mul_check(t, p->W, lim, &t) || !mul_check(t, p->B, lim, &t))
        return CACNN_ERR_INVALID_ARG;
    return CACNN_OK;
}

int plan_impl(const cacnn_problem* p, int dtype, const cacnn_machine* machine, cacnn_plan* out,
              bool allow_pipelined = true, double* model_us = nullptr) {
    if (!p || !out) return CACNN_ERR_NULL;
    if (!valid_problem(p)) return CACNN_ERR_INVALID_ARG;
    if (dtype != CACNN_F32 && dtype != CACNN_BF16_F32ACC) return CACNN_ERR_UNSUPPORTED;
    cacnn_machine mach = machine ? *machine : kDefaultMachine;
    if (mach.lds_bytes < 1024 || mach.num_cu < 1) return CACNN_ERR_INVALID_ARG;
    mach.lds_bytes = std::min<int64_t>(mach.lds_bytes, 160 * 1024);  // the kernels cannot address more
    {
        const int vrc = validate_dims(*p);
        if (vrc != CACNN_OK) return vrc;
    }
    Choice best;
    // Where a fixed-geometry kernel fits the problem and gives at least an eighth of the machine a tile, it has beaten
    // every generic kernel measured (by 2-3x on mid-size layers), and its cost above is a measurement while the
    // generic kernels' is a model: choose among those first.
    for (int vi = 0; vi < num_variants() && allow_pipelined; ++vi)
        if (variant(vi).info.dtype == dtype && variant(vi).info.fx_ct > 0) evaluate(vi, *p, mach, &best);
    // ... unless half or more of its tiles' outputs lie outside Out (fewer images than a tile holds, mostly): then the generic
    // kernels, which have tiles of 8 and 16 images, compete with it on the estimated time
    bool mostly_padding = false;
    if (best.variant >= 0) {
        const VariantInfo& bv = variant(best.variant).info;
        const double padded = (double)best.n_wg * bv.KT() * bv.NT();
        // (fp32: also where exactly half lie outside; the generic fp32 kernels' estimates are within 10 %, the bf16 ones' are
        // up to a third too low, and a half-empty bf16 tile was still the fastest on seven of seven such layers)
        const double useful = (double)p->B * p->K * p->W * p->H;
        mostly_padding = dtype == CACNN_F32 ? useful <= 0.5 * padded : useful < 0.5 * padded;
    }
    // ... or it is the fp32 kernel for 1 x 1 filters walking the taps of a larger filter, which re-stages the Image once
    // per tap: there the generic fp32 kernels, whose model is within 10 % of their measured times, win on some layers
    const bool f32_taps = best.variant >= 0 && dtype == CACNN_F32 && variant(best.variant).info.fx_any_stride && (p->R > 1 || p->S > 1);
    if (best.variant < 0 || best.n_wg * 8 < mach.num_cu || mostly_padding || f32_taps) {
        const bool use_lp = planner_uses_lp() && !((mostly_padding || f32_taps) && best.n_wg * 8 >= mach.num_cu);
        if (use_lp) best = Choice();
        // a bf16 fixed-geometry kernel that competes is given a head start of a quarter of its time: on such layers its
        // price was up to a quarter too high and the generic bf16 kernels' up to a quarter too low, and where the pick was
        // wrong the generic kernel lost up to 1.5 x, the fixed-geometry one 1.15 x
        const int fx_variant = best.variant;
        const double fx_cost = best.cost;
        if (fx_variant >= 0 && dtype != CACNN_F32) best.cost *= 0.75;
        const GpuLpTile lp = solve_gpu_lp(*p, dtype, mach);
        for (int vi = 0; vi < num_variants(); ++vi) {
            if (variant(vi).info.dtype != dtype) continue;
            if (variant(vi).info.pipelined && !allow_pipelined) continue;
            if (variant(vi).info.fx_ct > 0) continue;      // already in
            if (use_lp) evaluate_lp(vi, *p, mach, lp, &best);
            else evaluate(vi, *p, mach, &best);
        }
        if (best.variant == fx_variant && fx_variant >= 0) best.cost = fx_cost;
    }
    if (best.variant < 0) return CACNN_ERR_INVALID_ARG;  // nothing fits the given LDS size
    if (model_us) *model_us = best.cost / 2400.0;
    return fill_plan(*p, dtype, mach, best, out);
}

bool g_device_checked = false;
bool g_device_ok = false;
std::mutex g_mutex;

bool have_device() {
    std::lock_guard<std::mutex> lock(g_mutex);
    if (!g_device_checked) {
        int n = 0;
        const hipError_t e = hipGetDeviceCount(&n);
        if (e != hipSuccess) (void)hipGetLastError();
        g_device_ok = (e == hipSuccess && n > 0);
        g_device_checked = true;
    }
    return g_device_ok;
}

// layouts chosen by the two-level model for launches that name none, keyed by (problem, dtype, variant, grid): the model
// walks every tile of every candidate, which is host time a launch loop should pay once
struct LayoutEntry {
    cacnn_problem p;
    int dtype, vi;
    int64_t grid;
    int a_k, walk;
};
std::vector<LayoutEntry> g_layouts;

void cached_l2_layout(const cacnn_problem& p, int dtype, int vi, int64_t grid, const L2Machine& m2, int* a_k, int* walk) {
    {
        std::lock_guard<std::mutex> lock(g_mutex);
        for (const LayoutEntry& e : g_layouts)
            if (e.dtype == dtype && e.vi == vi && e.grid == grid && std::memcmp(&e.p, &p, sizeof(cacnn_problem)) == 0) {
                *a_k = e.a_k;
                *walk = e.walk;
                return;
            }
    }
    const L2Choice l2 = choose_l2_layout(p, dtype, variant(vi).info, grid, m2);
    *a_k = l2.a_k;
    *walk = l2.walk;
    std::lock_guard<std::mutex> lock(g_mutex);
    if (g_layouts.size() >= 64) g_layouts.erase(g_layouts.begin());
    g_layouts.push_back(LayoutEntry{p, dtype, vi, grid, l2.a_k, l2.walk});
}

// Tile-list decoding divides by launch constants with one multiply-high each, exact while dividend * divisor < 2^32; with the
// positions fastest one of the divisors is the number of position tiles of a block.
bool tile_list_in_range(const cacnn_problem& p, const VariantInfo& v, int walk, int split_k) {
    const double tk = (double)ceil_div(p.K, v.KT()), tw = (double)ceil_div(p.W, v.TW), th = (double)ceil_div(p.H, v.TH);
    const double n = tk * tw * th * (double)ceil_div(p.B, v.TB);
    if (n > 2147483647.0 || n * std::max(std::max(tk, tw), std::max(th, 64.0)) >= 4294967296.0) return false;
    return walk != 1 || split_k < 1 || n * (n / tk) < 4294967296.0;
}

// A launch of one of the two kinds of kernels but for its three pointers: everything that depends on the problem, the
// kernel and the operands' alignment alone.
struct Launch {
    const Variant* tiled = nullptr;
    const FlatVariant* flat = nullptr;
    const WindowVariant* window = nullptr;
    const FlatVariant* split = nullptr;     // what runs instead on the null stream: workgroups that share a tile's contraction
    KernelArgs a;
    FlatArgs f;
    FlatSplitArgs fs;
    WindowArgs w;
    int grid = 0, split_grid = 0;
    size_t lds = 0;
};

bool pointers_legal(int dtype, const void* image, const void* filter, const void* out) {
    const uintptr_t mask = dtype == CACNN_F32 ? 3 : 1;
    return ((reinterpret_cast<uintptr_t>(image) | reinterpret_cast<uintptr_t>(filter)) & mask) == 0 && reinterpret_cast<uintptr_t>(out) % 4 == 0;
}

bool aligned16(const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

template <class Args>
Args with_buffers(const Args& args, const void* image, const void* filter, void* out) {
    Args a = args;
    a.image = image;
    a.filter = filter;
    a.out = (float*)out;
    return a;
}

int fire(const Launch& l, const void* image, const void* filter, void* out, void* stream) {
    if (!have_device()) return CACNN_ERR_NO_DEVICE;
    int rc;
    if (l.split && !stream) rc = l.split->launch_split(with_buffers(l.fs, image, filter, out), l.split_grid, stream);
    else if (l.flat) rc = l.flat->launch(with_buffers(l.f, image, filter, out), l.grid, stream);
    else if (l.window) rc = l.window->launch(with_buffers(l.w, image, filter, out), l.grid, l.lds, stream);
    else rc = l.tiled->launch(with_buffers(l.a, image, filter, out), l.grid, l.lds, stream);
    return rc == 0 ? CACNN_OK : CACNN_ERR_LAUNCH;
}

int prepare_tiled(const cacnn_problem& p, int dtype, int vi, int CT, int bR, int bS, int split_k, int walk, bool aligned_img,
                  bool aligned_flt, Launch* out) {
    const Variant& var = variant(vi);
    const VariantInfo& v = var.info;
    const size_t esz = dtype == CACNN_F32 ? 4 : 2;
    const bool vimg = vec_img_ok(v, p) && aligned_img;
    const Geometry g = make_geometry(v, p, CT, bR, bS, vimg);
    if (!g.legal || g.lds_bytes > 160 * 1024 || g.lds_bytes < 1) return CACNN_ERR_UNSUPPORTED;
    if (v.pipelined && !aligned_flt && !g.flt_resident) return CACNN_ERR_UNSUPPORTED;

    KernelArgs& a = out->a;
    std::memset(&a, 0, sizeof(a));
    a.B = (int32_t)p.B;
    a.C = (int32_t)p.C;
    a.K = (int32_t)p.K;
    a.W = (int32_t)p.W;
    a.H = (int32_t)p.H;
    a.R = (int32_t)p.R;
    a.S = (int32_t)p.S;
    a.sw = (int32_t)p.sigma_w;
    a.sh = (int32_t)p.sigma_h;
    a.IW = (int32_t)(p.sigma_w * (p.W - 1) + p.R);
    a.IH = (int32_t)(p.sigma_h * (p.H - 1) + p.S);
    a.bR = g.bR;
    a.bS = g.bS;
    a.CT = g.CT;
    a.XS = g.XS;
    a.YS = g.YS;
    a.xpitch = g.xpitch;
    a.ypitch = g.ypitch;
    a.fpitch = g.fpitch;
    a.QE = g.QE;
    a.img_lds_elems = g.img_lds_elems;
    a.zero_off = g.zero_off;
    a.tiles_k = (int32_t)ceil_div(p.K, v.KT());
    a.tiles_b = (int32_t)ceil_div(p.B, v.TB);
    a.tiles_w = (int32_t)ceil_div(p.W, v.TW);
    a.tiles_h = (int32_t)ceil_div(p.H, v.TH);
    a.vec_img = vimg ? 1 : 0;
    if (dtype == CACNN_F32)
        a.vec_flt = (aligned_flt && p.C % 4 == 0 && g.CT % 4 == 0) ? 1 : 0;
    else
        a.vec_flt = (aligned_flt && p.C % 8 == 0) ? 1 : 0;
    a.d_CT = make_fastdiv((uint32_t)g.CT);
    a.d_YS = make_fastdiv((uint32_t)g.YS);
    a.d_bS = make_fastdiv((uint32_t)g.bS);
    a.d_bR = make_fastdiv((uint32_t)g.bR);
    a.d_RS = make_fastdiv((uint32_t)(g.bR * g.bS));
    a.d_XS = make_fastdiv((uint32_t)g.XS);
    a.d_C4 = make_fastdiv((uint32_t)std::max(1, g.CT / 4));
    if (dtype == CACNN_F32)
        a.d_C8 = make_fastdiv((uint32_t)(a.vec_flt ? g.CT / 4 : g.CT));
    else
        a.d_C8 = make_fastdiv((uint32_t)(g.CT / 8));
    int64_t grid = 0, t = 0;
    if (!mul_check(a.tiles_k, a.tiles_b, INT32_MAX, &t) || !mul_check(t, a.tiles_w, INT32_MAX, &t) ||
        !mul_check(t, a.tiles_h, INT32_MAX, &grid))
        return CACNN_ERR_INVALID_ARG;
    a.n_tiles = (int32_t)grid;
    a.n_xcd = xcd_count();
    {
        // b-tiles that read different pieces of the same 128-byte Image lines stay adjacent in the tile order
        const int64_t want = std::max<int64_t>(1, 128 / (int64_t)(v.TB * esz));
        int g_b = 1;
        for (int d = 1; d <= a.tiles_b && d <= want; ++d)
            if (a.tiles_b % d == 0) g_b = d;
        a.b_group = g_b;
    }
    if (!tile_list_in_range(p, v, walk, split_k)) return CACNN_ERR_INVALID_ARG;    // (before the layout is chosen, which walks the tiles)
    a.xcd_q = a.n_tiles / a.n_xcd;
    a.xcd_rem = a.n_tiles % a.n_xcd;
    a.d_nxcd = make_fastdiv((uint32_t)a.n_xcd);
    if (split_k == 0) {
        // no layout given: the two-level model's choice for this variant and grid
        L2Machine m2 = kDefaultL2Bytes;
        m2.words /= (double)esz;
        m2.n_xcd = a.n_xcd;
        cached_l2_layout(p, dtype, vi, launch_grid(v, g, grid, kDefaultMachine), m2, &split_k, &walk);
    }
    if (split_k < 1 || split_k > 8 || (split_k & (split_k - 1)) || a.tiles_k % split_k) return CACNN_ERR_INVALID_ARG;
    if (walk != 0 && walk != 1) return CACNN_ERR_INVALID_ARG;
    a.k_groups = split_k;
    a.kpg = a.tiles_k / split_k;
    a.grp = a.n_tiles / split_k;
    a.npos = a.grp / a.kpg;
    if (!tile_list_in_range(p, v, walk, split_k)) return CACNN_ERR_INVALID_ARG;    // (with the layout's walk)
    a.pos_fastest = walk;
    a.d_npos = make_fastdiv((uint32_t)a.npos);
    a.d_tk = make_fastdiv((uint32_t)a.kpg);
    a.d_bg = make_fastdiv((uint32_t)a.b_group);
    a.d_tw = make_fastdiv((uint32_t)a.tiles_w);
    a.d_th = make_fastdiv((uint32_t)a.tiles_h);
    a.img_items = g.img_items;
    a.flt_items = g.flt_items;
    a.img_buf = g.img_buf;
    a.flt_buf = g.flt_buf;
    a.flt_off = g.flt_off;
    a.flt_resident = g.flt_resident;
    out->tiled = &var;
    out->flat = out->split = nullptr;
    out->window = nullptr;
    out->grid = (int)launch_grid(v, g, grid, kDefaultMachine);
    out->lds = (size_t)g.lds_bytes;
    return CACNN_OK;
}

int launch_with(const cacnn_problem& p, int dtype, int vi, int CT, int bR, int bS, int split_k, int walk, const void* image,
                const void* filter, void* out, void* stream) {
    if (!pointers_legal(dtype, image, filter, out)) return CACNN_ERR_INVALID_ARG;
    Launch l;
    const int rc = prepare_tiled(p, dtype, vi, CT, bR, bS, split_k, walk, aligned16(image), aligned16(filter), &l);
    return rc != CACNN_OK ? rc : fire(l, image, filter, out, stream);
}

// ------------------------------------------------------------------------------------------------------------
// The kernels with flattened positions (cacnn_flat.hip): which of them takes a problem, what it costs, its launch.

// bytes of the Image that some output reads (strides beyond the filter's extent leave some out), of Filter and of Out
struct Bytes {
    double image, filter, out;
};
Bytes compulsory_bytes(const cacnn_problem& p, int dtype) {
    const double esz = dtype == CACNN_F32 ? 4.0 : 2.0;
    const double cols = (double)std::min(p.sigma_w * (p.W - 1) + p.R, p.W * p.R), rows = (double)std::min(p.sigma_h * (p.H - 1) + p.S, p.H * p.S);
    return {esz * (double)p.B * p.C * cols * rows, esz * (double)p.K * p.R * p.S * p.C, 4.0 * (double)p.K * p.H * p.W * p.B};
}

// the time that reading and writing them once takes at the rate of a large copy
double compulsory_us(const cacnn_problem& p, int dtype) {
    const Bytes b = compulsory_bytes(p, dtype);
    return (b.image + b.filter + b.out) / 4.6e6;
}

// ... and what a kernel takes that would need `us` with all data at hand: the larger of the two, and a quarter of the smaller
// that the other does not hide (fitted with the estimates below)
double with_copy_time(double us, const cacnn_problem& p, int dtype) {
    const double copy = compulsory_us(p, dtype);
    return std::max(us, copy) + 0.25 * std::min(us, copy);
}

// Whether a kernel with flattened positions takes the problem: enough images for the group a lane holds (or exactly the
// number it was compiled for, and a filter row of at least one 16-byte chunk), and Image and Filter within the 2 GiB
// that its 32-bit byte offsets reach, and a launch of fewer than 2^32 threads (its workgroups walk no list of tiles, there is one for each).
bool flat_fits(const cacnn_problem& p, int dtype, const FlatInfo& v) {
    const int esz = dtype == CACNN_F32 ? 4 : 2;
    if (v.dtype != dtype) return false;
    if (v.IM < 0 ? p.B != -v.IM : p.B < v.IM) return false;
    if (v.NCH && p.S * p.C * esz < 16) return false;
    const double IW = (double)(p.sigma_w * (p.W - 1) + p.R), IH = (double)(p.sigma_h * (p.H - 1) + p.S);
    const double groups = (double)p.H * (double)p.W * (double)(v.IM < 0 ? 1 : ceil_div(p.B, v.IM));
    if ((double)ceil_div(p.K, v.KT()) * std::ceil(groups / v.GT()) * v.threads() >= 4294967296.0) return false;
    return IW * IH * (double)p.C * (double)p.B * esz < 2147483648.0 && (double)p.K * p.R * p.S * p.C * esz < 2147483648.0;
}

// Estimated launch time in microseconds, from what bounds these kernels on MI355X: the address unit of a compute unit, through
// which every operand comes, the issue slots and MFMA pipes of its SIMDs, and the latency of a chain of steps or stages.
// The clocks of one 64-lane load, measured out of L1: at least 8.5 for 2 and 4 bytes a lane and 17.4 for 8 and 16 (that is
// the 64 bytes a clock L1 delivers), else about one for each separate run of bytes; runs that are not made of four
// neighbouring lanes cost more, and lanes whose address is no multiple of 4 bytes take about twice (8 bytes and less) to
// three times (16 bytes) as long.  The other constants are a least-squares fit to the launch times of all
// configurations on 330 layers drawn over all sizes: there the configuration with the smallest estimate takes 1.04 times as
// long as the fastest one in the geometric mean, and the estimate is within 14 % of the time (one standard deviation).
double load_clocks(int bytes, double run_bytes, bool aligned4, bool whole_quads) {
    const double floor_clk = bytes <= 4 ? 8.5 : 17.4, run_lanes = std::max(run_bytes / bytes, 1.0);
    const double odd = aligned4 || bytes == 2 ? 1.0 : bytes == 16 ? 3.0 : 1.8;
    const double clk = std::max(floor_clk, std::min(64.0, 48.0 / run_lanes)) * odd;
    return whole_quads || run_lanes >= 32.0 ? clk : std::max(clk, 40.0 - run_lanes);
}

// part_stages > 0: a tile's contraction is divided into parts of so many stages.  Sums leave in parallel and meet at the memory behind the L2s:
// 1.67 us, 0.245 us for every part that the last workgroup reads 16 rows a wave of, and the sums at 2.7 TB/s (fitted to 14000
// launches of 400 layers: 10 % (one standard deviation) where the time is within 1.5 of the layer's best).
double flat_us(const cacnn_problem& p, int dtype, const FlatInfo& v, int64_t part_stages = 0) {
    const bool f32 = dtype == CACNN_F32, run = v.IM < 0;
    const int esz = f32 ? 4 : 2, ch = 16 / esz, ipl = run ? -v.IM : v.IM;
    const int64_t T = p.S * p.C, chunks = p.R * ceil_div(T, ch);
    const int64_t groups = p.H * p.W * (run ? 1 : ceil_div(p.B, ipl));
    const int64_t stages_in_all = v.NCH ? ceil_div(chunks, v.NCH) : 0, parts = part_stages ? ceil_div(stages_in_all, part_stages) : 1;
    const double tiles = (double)ceil_div(p.K, v.KT()) * (double)ceil_div(groups, v.GT());
    const double per_cu = std::ceil(tiles * (double)parts / (double)kDefaultMachine.num_cu);
    const double waves = v.WM * v.WN * v.WK, simd_waves = std::ceil(waves / 4.0), mfma = f32 ? 256.0 : 32.0;   // of one block's step
    const double blocks = v.MB * v.NG * (run || !v.NCH ? ipl : 1);                                            // of one wave
    const bool flt_aligned = f32 || T % 2 == 0, img_aligned = f32 || (run ? p.C * p.B : p.B) % 2 == 0;
    double clk;
    if (T < ch) {
        // Filter rows shorter than a chunk: T loads for each operand and step, of which the waves share R / 2, nothing fetched ahead.  Fitted
        // on 1350 such layers: 18 % (one standard deviation), the pick is within 1.02 of the fastest.
        const int64_t steps = (chunks + 1) / 2, mine = ceil_div(steps, v.WK);
        const double busy = (double)(v.WM * v.WN * ceil_div(steps, mine));                                    // waves that have a step
        const double b_clk = load_clocks(ipl * esz, (double)(std::min<int64_t>(p.B, 32 * ipl) * esz), img_aligned, ipl == 4 || p.B % (4 * ipl) == 0);
        const double load = per_cu * busy * mine * T * (v.MB * 12.7 + v.NG * b_clk * 0.79);
        const double simd = per_cu * std::ceil(busy / 4.0) * mine * blocks * mfma, latency = mine * 1244.0;
        clk = std::sqrt(load * load + simd * simd + latency * latency);
        clk += per_cu * blocks * (v.WM * v.WN * 105.0 + (v.WK > 1 ? waves * 82.0 : 0.0));                     // Out
        return with_copy_time(clk / 2272.0, p, dtype) + 2.1;
    }
    if (!v.NCH) {
        const double mine = (double)ceil_div((chunks + 1) / 2, v.WK) + 1.0;                                   // steps of a wave
        const double a_clk = load_clocks(16, 32.0, flt_aligned, true);
        const double b_clk = ch * load_clocks(ipl * esz, (double)(std::min<int64_t>(p.B, 32 * ipl) * esz), img_aligned,
                                              ipl == 4 || p.B % (4 * ipl) == 0);
        const double load = per_cu * waves * mine * (v.MB * a_clk + v.NG * b_clk);
        const double simd = per_cu * simd_waves * mine * (blocks * mfma + 62.0), latency = (mine / 4.0 + 0.75) * 1020.0;
        clk = std::sqrt(load * load + simd * simd + latency * latency);
    } else {
        const double stages = (double)(part_stages ? part_stages : stages_in_all), cols = v.WN * v.NG * 32, kt = v.KT();
        const double steps = std::max(1, v.NCH / 2 / v.WK);                                                   // of a wave per stage
        const double flt_items = kt * v.NCH, img_items = run ? cols * v.NCH * ipl : (double)v.NCH * ch * v.GT();
        const double load = flt_items / 64.0 * load_clocks(16, (double)std::min<int64_t>(v.NCH * 16, T * esz), flt_aligned, true) +
                            img_items / 64.0 * (run ? load_clocks(16, (double)std::min<int64_t>(v.NCH * 16 * ipl, T * p.B * esz), img_aligned, true)
                                                    : load_clocks(ipl * esz, std::min((double)p.B, cols) * esz, img_aligned, true));
        const double simd = simd_waves * (steps * blocks * mfma + 66.0 * (flt_items + img_items) / (64.0 * waves));
        const double lds = (flt_items + (run ? img_items : v.NCH * ch * cols * esz / 16.0)) / 4.0 + waves * steps * (v.MB + blocks / v.MB) * 10.24;
        const double stage = std::sqrt(load * load + simd * simd + 0.063 * lds * lds);
        const double together = std::min(per_cu, std::max(1.0, std::min(2.0, std::floor(8.0 / waves))));      // workgroups that overlap
        const double busy = per_cu * stages * stage, latency = std::ceil(per_cu / together) * stages * 357.0;
        clk = std::sqrt(busy * busy + latency * latency) + 1000.0;
    }
    clk += per_cu * blocks * (v.WM * v.WN * 200.0 + (v.WK > 1 ? waves * 110.0 : 0.0));                        // Out
    double us = with_copy_time(clk / 2272.0, p, dtype) + 2.1;
    if (parts > 1) us += 1.67 + 0.245 * (double)parts * v.words() / (waves * 1024.0) + 1.5e-6 * tiles * (double)parts * v.words();
    return us;
}

// The flattened kernel with the smallest estimate, -1 if none takes the problem.
int choose_flat(const cacnn_problem& p, int dtype, double* us) {
    int best = -1;
    for (int i = 0; i < num_flat(); ++i) {
        const FlatInfo& v = flat_variant(i).info;
        if (!flat_fits(p, dtype, v)) continue;
        const double t = flat_us(p, dtype, v);
        if (best < 0 || t < *us) {
            best = i;
            *us = t;
        }
    }
    return best;
}

// The stages of a part and the number of parts when a tile's contraction is divided into `want` of them, as evenly as whole stages
// allow; 0 if it cannot be (the kernel stages nothing, there are too few stages or too many sums).
int split_parts(const cacnn_problem& p, int dtype, const FlatInfo& v, int64_t want, int64_t* part_stages) {
    if (!v.NCH || want < 2) return 0;
    const int64_t groups = p.H * p.W * (v.IM < 0 ? 1 : ceil_div(p.B, v.IM));
    const int64_t tiles = ceil_div(p.K, v.KT()) * ceil_div(groups, v.GT());
    const int64_t stages = ceil_div(p.R * ceil_div(p.S * p.C, dtype == CACNN_F32 ? 4 : 8), v.NCH);
    *part_stages = ceil_div(stages, want);
    const int64_t parts = ceil_div(stages, *part_stages);
    return parts >= 2 && tiles <= kSplitTiles && parts * tiles <= kSplitWords / v.words() ? (int)parts : 0;
}

// The kernel and the number of parts with the smallest estimate among launches whose workgroups share a tile's contraction, -1 if there is none
int choose_split(const cacnn_problem& p, int dtype, int only, int* best_parts, double* us) {
    static const int kParts[] = {2, 3, 4, 6, 8, 12, 16, 24, 32, 48};
    int best = -1;
    for (int i = only < 0 ? 0 : only; i < (only < 0 ? num_flat() : only + 1); ++i) {
        const FlatInfo& v = flat_variant(i).info;
        if (!v.NCH || !flat_fits(p, dtype, v)) continue;
        for (int want : kParts) {
            int64_t part_stages = 0;
            const int parts = split_parts(p, dtype, v, want, &part_stages);
            if (!parts) continue;
            const double t = flat_us(p, dtype, v, part_stages);
            if (best < 0 || t < *us) {
                best = i;
                *best_parts = parts;
                *us = t;
            }
        }
    }
    return best;
}

int prepare_flat(const cacnn_problem& p, int dtype, int fi, Launch* out) {
    const FlatVariant& var = flat_variant(fi);
    const FlatInfo& v = var.info;
    if (!flat_fits(p, dtype, v)) return CACNN_ERR_UNSUPPORTED;
    const int esz = dtype == CACNN_F32 ? 4 : 2, ch = 16 / esz;
    const int64_t T = p.S * p.C;
    const int64_t IW = p.sigma_w * (p.W - 1) + p.R, IH = p.sigma_h * (p.H - 1) + p.S;
    const int64_t img = IW * IH * p.C * p.B * esz, flt = p.K * p.R * T * esz;
    FlatArgs& a = out->f;
    std::memset(&a, 0, sizeof(a));
    a.N = (uint32_t)(p.H * p.W * p.B);
    a.K = (uint32_t)p.K;
    a.B = (uint32_t)p.B;
    a.W = (uint32_t)p.W;
    a.G = v.IM < 0 ? 1u : (uint32_t)ceil_div(p.B, v.IM);
    a.groups = (uint32_t)(p.H * p.W) * a.G;
    a.T = (uint32_t)T;
    a.TC = (uint32_t)ceil_div(T, ch);
    a.U = (uint32_t)p.R * a.TC;
    a.back = T % ch ? (uint32_t)(ch - T % ch) : 0u;
    a.steps = (a.U + 1) / 2;
    a.steps_per_wave = (a.steps + v.WK - 1) / v.WK;
    a.img_h = (uint32_t)(p.sigma_h * p.C * p.B * esz);
    a.img_r = (uint32_t)(IH * p.C * p.B * esz);
    a.img_w = (uint32_t)p.sigma_w * a.img_r;
    a.img_chunk = (uint32_t)(ch * p.B * esz);
    a.flt_r = (uint32_t)(T * esz);
    a.flt_row = (uint32_t)p.R * a.flt_r;
    const uint32_t adv = v.NCH ? v.NCH : 2;
    a.adv_tc = adv % a.TC;
    a.adv_flt = adv / a.TC * a.flt_r + a.adv_tc * 16u;
    a.adv_img = adv / a.TC * a.img_r + a.adv_tc * a.img_chunk;
    a.wrap_flt = a.flt_r - a.TC * 16u;
    a.wrap_img = a.img_r - a.TC * a.img_chunk;
    a.img_bytes = (int32_t)img;
    const int64_t tiles_k = ceil_div(p.K, v.KT()), tiles_n = ceil_div(a.groups, v.GT());
    const int64_t grid = tiles_k * tiles_n;
    a.k_inner = img >= flt ? 1u : 0u;
    a.inner = (uint32_t)(a.k_inner ? tiles_k : tiles_n);
    a.xcd_q = (uint32_t)grid / kFlatXcds;
    a.xcd_rem = (uint32_t)grid % kFlatXcds;
    a.d_G = make_flatdiv(a.G);
    a.d_W = make_flatdiv((uint32_t)p.W);
    a.d_TC = make_flatdiv(a.TC);
    a.d_inner = make_flatdiv(a.inner);
    out->flat = &var;
    out->split = nullptr;
    out->window = nullptr;
    out->tiled = nullptr;
    out->grid = (int)grid;
    return CACNN_OK;
}

int prepare_split(const cacnn_problem& p, int dtype, int fi, int want, Launch* out) {
    int64_t part_stages = 0;
    Launch l;
    if (prepare_flat(p, dtype, fi, &l) != CACNN_OK) return CACNN_ERR_UNSUPPORTED;
    const int parts = split_parts(p, dtype, l.flat->info, want, &part_stages);
    if (!parts) return CACNN_ERR_UNSUPPORTED;
    FlatSplitArgs& a = out->fs;
    static_cast<FlatArgs&>(a) = l.f;
    a.parts = (uint32_t)parts;
    a.part_stages = (uint32_t)part_stages;
    a.tiles = (uint32_t)l.grid;
    a.d_tiles = make_flatdiv(a.tiles);
    out->split = l.flat;
    out->split_grid = l.grid * parts;
    a.xcd_q = (uint32_t)out->split_grid / kFlatXcds;
    a.xcd_rem = (uint32_t)out->split_grid % kFlatXcds;
    return CACNN_OK;
}

int launch_flat(const cacnn_problem& p, int dtype, int fi, const void* image, const void* filter, void* out, void* stream) {
    if (!pointers_legal(dtype, image, filter, out)) return CACNN_ERR_INVALID_ARG;
    Launch l;
    const int rc = prepare_flat(p, dtype, fi, &l);
    return rc != CACNN_OK ? rc : fire(l, image, filter, out, stream);
}

// ------------------------------------------------------------------------------------------------------------
// The bf16 kernels that keep a tile's window in LDS (cacnn_window.hip).

struct WindowTile {
    int TW = 0, TH = 0;     // output columns and rows
    int bufs = 0;           // boxes in LDS: 2, workgroups walk position tiles, or 1, they take one each
};

// The launch of a window kernel with these tiles; CACNN_ERR_UNSUPPORTED where it does not take them.  Whole 16-byte items along b, filter
// columns of at least one chunk, Image, Filter and a row of Out within the 2 GiB of 32-bit offsets, the Filter tile and the boxes in LDS.
int prepare_window(const cacnn_problem& p, int wi, const WindowTile& t, Launch* out) {
    const WindowVariant& var = window_variant(wi);
    const WindowInfo& v = var.info;
    const int64_t IW = p.sigma_w * (p.W - 1) + p.R, IH = p.sigma_h * (p.H - 1) + p.S;
    const double img = 2.0 * (double)IW * (double)IH * (double)p.C * (double)p.B, flt = 2.0 * (double)p.K * p.R * p.S * p.C;
    if (p.B % 8 != 0 || p.S * p.C < 8 || img >= 2147483648.0 || flt >= 2147483648.0) return CACNN_ERR_UNSUPPORTED;
    if (20.0 * (double)p.H * (double)p.W * (double)p.B >= 2147483648.0) return CACNN_ERR_UNSUPPORTED;
    if (t.TW < 1 || t.TH < 1 || (t.TW & (t.TW - 1)) || (t.TH & (t.TH - 1)) || t.TW * t.TH * v.TB != v.cols()) return CACNN_ERR_UNSUPPORTED;
    const int64_t nx = p.sigma_w * (t.TW - 1) + p.R, ny = p.sigma_h * (t.TH - 1) + p.S, waves = v.threads() / 64;
    const double box = (double)nx * (double)ny * p.C * v.TB * 2.0, chunks = (double)p.R * (double)ceil_div(p.S * p.C, 8);
    if (box > 131072.0 || chunks * v.KT() * 16.0 > 131072.0) return CACNN_ERR_UNSUPPORTED;
    WindowArgs& a = out->w;
    std::memset(&a, 0, sizeof(a));
    a.N = (uint32_t)(p.H * p.W * p.B);
    a.K = (uint32_t)p.K;
    a.B = (uint32_t)p.B;
    a.C = (uint32_t)p.C;
    a.W = (uint32_t)p.W;
    a.H = (uint32_t)p.H;
    a.sw = (uint32_t)p.sigma_w;
    a.sh = (uint32_t)p.sigma_h;
    a.img_bytes = (uint32_t)img;
    a.img_x = (uint32_t)(IH * p.C * p.B * 2);
    a.img_w = (uint32_t)p.sigma_w * a.img_x;
    a.img_h = (uint32_t)(p.sigma_h * p.C * p.B * 2);
    a.flt_tap = (uint32_t)(p.S * p.C * 2);
    a.flt_k = (uint32_t)p.R * a.flt_tap;
    while ((1 << a.tw_shift) < t.TW) ++a.tw_shift;
    while ((1 << a.th_shift) < t.TH) ++a.th_shift;
    a.tiles_h = (uint32_t)ceil_div(p.H, t.TH);
    a.tiles_b = (uint32_t)ceil_div(p.B, v.TB);
    a.tiles_n = (uint32_t)ceil_div(p.W, t.TW) * a.tiles_h * a.tiles_b;
    a.plane = (uint32_t)(ny * p.C);
    a.rows = (uint32_t)nx * a.plane;
    a.TC = (uint32_t)ceil_div(p.S * p.C, 8);
    a.back = 8 * a.TC - (uint32_t)(p.S * p.C);
    a.U = (uint32_t)p.R * a.TC;
    a.steps = ((a.U + 1) / 2 + 1) & ~1u;
    a.UP = 2 * a.steps + 1;                     // odd: the rows that a read takes at once lie in different banks
    const uint32_t row = (uint32_t)v.TB * 2;
    a.off_r = a.plane * row;
    a.adv_i = 2 % a.TC;
    a.adv_off = 2 / a.TC * a.off_r + a.adv_i * 8 * row;
    a.wrap_off = a.off_r - a.TC * 8 * row;
    a.img_items = (uint32_t)ceil_div(ceil_div(a.rows * row, 1024), waves);
    a.img_lds = a.img_items * (uint32_t)waves * 1024;
    a.flt_lds = (uint32_t)ceil_div((int64_t)v.KT() * a.UP * 16, 1024) * 1024;
    a.zeros = a.flt_lds + (uint32_t)t.bufs * a.img_lds;
    out->lds = (size_t)a.zeros + 8 * row;
    if (a.img_items > kWindowItems || out->lds > 160 * 1024) return CACNN_ERR_UNSUPPORTED;
    const int64_t tiles_k = ceil_div(p.K, v.KT());
    int64_t walkers = a.tiles_n;                // workgroups of a tile of output channels
    if (t.bufs == 2) {
        const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(160 * 1024 / (int64_t)out->lds, 16 / waves));
        walkers = std::max<int64_t>(1, std::min<int64_t>(walkers, kDefaultMachine.num_cu * per_cu / tiles_k));
    }
    if ((double)tiles_k * (double)a.tiles_n * v.threads() >= 4294967296.0) return CACNN_ERR_UNSUPPORTED;
    a.t_step = (uint32_t)walkers;
    a.k_inner = img >= flt ? 1u : 0u;
    a.inner = (uint32_t)(a.k_inner ? tiles_k : walkers);
    out->grid = (int)(tiles_k * walkers);
    a.xcd_q = (uint32_t)out->grid / kFlatXcds;
    a.xcd_rem = (uint32_t)out->grid % kFlatXcds;
    a.d_inner = make_flatdiv(a.inner);
    a.d_tb = make_flatdiv(a.tiles_b);
    a.d_th = make_flatdiv(a.tiles_h);
    a.d_plane = make_flatdiv(a.plane);
    a.d_UP = make_flatdiv(a.UP);
    a.d_TC = make_flatdiv(a.TC);
    out->window = &var;
    out->tiled = nullptr;
    out->flat = out->split = nullptr;
    return CACNN_OK;
}

// The tile of a window kernel with `bufs` boxes whose position tiles stage the fewest words, of those that leave room for a second workgroup on the
// compute unit, and its launch; false where none does
bool pick_window_tile(const cacnn_problem& p, int wi, int bufs, WindowTile* pick, Launch* out) {
    const WindowInfo& v = window_variant(wi).info;
    WindowTile t;
    double words = 0.0;
    *pick = t;
    t.bufs = bufs;
    for (t.TW = v.cols() / v.TB; t.TW >= 1; t.TW /= 2) {
        t.TH = v.cols() / v.TB / t.TW;
        if (prepare_window(p, wi, t, out) != CACNN_OK || out->lds > 80 * 1024) continue;
        const double w = (double)out->w.tiles_n * (double)out->w.rows;
        if (!pick->TW || w < words) *pick = t, words = w;
    }
    return pick->TW && prepare_window(p, wi, *pick, out) == CACNN_OK;
}

// The window kernel of a first layer: few channels, and a batch of which every tile is whole rows of images (others, whose stores are pieces of
// cache lines, took up to 1.36 times as long as the flattened kernels).  One box per workgroup or two, whichever fills its last round of tiles
// better.  -1 where the flattened kernel's estimate is below 10 us (1.7 us are spent before the first product: 5.6 -> 7.3 us at (8, 3, 64, 56, 56, 7 x 7, s 2)), and, up to 22
// us, where less than 0.64 of the last round and of the tiles along k is filled ((128, 3, 48, 56, 24, 3 x 3) 10.6 -> 12.3 us).  Over 113 first layers of
// 8 us and more the time is 0.89 of the flattened kernels' in the geometric mean, 0.51 at best and 1.03 at worst.
int choose_window(const cacnn_problem& p, double flat_est, WindowTile* tile) {
    if (flat_est < 10.0 || p.C > 4 || (p.B % 32 != 0 && p.B != 16 && p.B != 8)) return -1;
    const int TB = (int)std::min<int64_t>(p.B, 32);
    int best = -1;
    double best_fill = 0.0;
    for (int i = 0; i < num_window(); ++i) {
        const WindowInfo& v = window_variant(i).info;
        if (v.TB != TB) continue;
        for (int bufs = 2; bufs >= 1; --bufs) {
            Launch l;
            WindowTile pick;
            if (!pick_window_tile(p, i, bufs, &pick, &l)) continue;
            // tiles per round of the workgroups that are resident together (launch_bounds: four waves a SIMD)
            const double resident = (double)kDefaultMachine.num_cu * (double)std::min<int64_t>(160 * 1024 / (int64_t)l.lds, 16 / (v.threads() / 64));
            const double rounds = bufs == 2 ? (double)l.w.tiles_n / l.w.t_step : (double)l.grid / resident;
            const double fill = rounds / std::ceil(rounds);
            if (best < 0 || fill > best_fill + 0.1) {       // (nearly level, two boxes are faster: (16, 3, 64, 112, 112, 7 x 7, s 2) 16.4 us with fills of 0.68, 17.9 with 0.77)
                best = i;
                best_fill = fill;
                *tile = pick;
            }
        }
    }
    if (best < 0) return -1;
    best_fill *= (double)p.K / (double)round_up(p.K, window_variant(best).info.KT());
    return best_fill < 0.64 && flat_est < 22.0 ? -1 : best;
}

// Launch cache of cacnn_conv_forward, keyed by (problem, dtype, alignment of the two operands): planning costs tens of
// microseconds and laying out a launch one, the launch itself two.  What is kept depends on the key alone, not on the buffers.
// An entry is never changed: a call holds on to its launch (a kilobyte, which it need not copy) while others come and go.
using LaunchPtr = std::shared_ptr<const Launch>;
struct PlanEntry {
    cacnn_problem p;
    int key;
    LaunchPtr launch;
};
std::vector<PlanEntry> g_plans;

int launch_key(int dtype, const void* image, const void* filter) {
    return dtype | (aligned16(image) ? 0 : 0x100) | (aligned16(filter) ? 0 : 0x200);
}

// One large fp32 image whose filter rows are shorter than a chunk (fewer than 4 channels of a 1 x 1 filter, a 3 x 3 one on a single
// channel): each lane's load takes 4 bytes from a place of its own, which the box tiles of 16 x 16 positions of one image do
// better where there are many positions.  (1, 1, 40, W, W, 1 x 1), box tiles and flattened: W = 180 6.1 and 4.6 us, 280 7.9 and
// 7.8, 340 9.3 and 10.2, 528 18.1 and 21.2; over 320 layers the flattened kernel takes 0.3 to 1.0 times as long up to 80 000 positions
// and 0.7 to 1.5 times, mostly more than 1.0, from 117 000 on.  Images that do not fill a
// box tile in one direction, a second image, and bf16: the flattened one is faster at every size measured.
bool boxes_for_short_rows(const cacnn_problem& p, int dtype) {
    return dtype == CACNN_F32 && p.B == 1 && p.S * p.C < 4 && p.W * p.H >= 100000 && std::min(p.W, p.H) >= 16;
}

// A flattened kernel takes the place of a fixed-geometry one where its estimate is below this share of the other's time: on 60 layers the
// flattened kernel was 1.2 to 4 times faster below 0.7 (layers that leave most compute units idle, taps of large
// filters), and between it and the break-even both sides won, by up to 1.5 times (1.27 for the fixed-geometry ones).
// The estimate knows nothing of windows read again from beyond the L2.  For bf16, whose products do not hide that, on Images of more than
// 100 MB it is too low by up to 2.2 times, the more the windows overlap and the larger the Image is than the last-level
// cache of 256 MB: (16, 888, 24, 126, 126, 3 x 3) 435 us and 571 flattened, (16, 1360, 3, 127, 127, 3 x 3) 562 and 978, (32, 152, 1, 151, 107,
// 1 x 7) 109 and 134.  The line there is fitted on 173 such layers and tried on 105 others: with 0.7 48 of these 278 take up to 1.74 times
// as long as on their fixed-geometry kernel, with this one 3, up to 1.16.  fp32 layers of these
// sizes: 0.24 to 0.87 times as long with 0.7.
double flat_margin(const cacnn_problem& p, int dtype) {
    const double image = 2.0 * (double)(p.sigma_w * (p.W - 1) + p.R) * (double)(p.sigma_h * (p.H - 1) + p.S) * (double)p.C * (double)p.B;
    if (dtype == CACNN_F32 || image < 100e6) return 0.7;
    const double overlap = std::max(1.0, (double)p.R / (double)p.sigma_w) * std::max(1.0, (double)p.S / (double)p.sigma_h);
    return std::min(0.7, 0.85 * std::pow(overlap * std::max(1.0, image / 256e6), -0.2));
}

// The two estimates compared as measurements correct them: whether the flattened kernel is expected to take less than a share of the
// fixed-geometry one's time.  The factors on either estimate are least-squares fits of the logarithm of time over estimate, on 1850
// layers of up to 250 MB whose plan is a fixed-geometry variant and whose flattened estimate is not below the margin above, all
// run on both: the planner's price is low by up to half where a launch is short, and by the more the larger
// Out's part of the words is; the flattened kernel's is low for large Images with overlapping windows.  At these shares (fp32 0.8, bf16 0.75) the
// time over all of them is 0.867 and 0.863 of the fixed-geometry kernels' in the geometric mean (the faster of the two each time:
// 0.829 and 0.795), and three take longer, by up to 1.19; at 0.83 and 0.8 it is 0.854 and 0.836, nine take up to 1.2 times as long and
// one of 4 us 1.45, at 0.9 44 do, up to 1.47 times.  fp32 (256, 32, 498, 81, 3, 1 x 1) 118 -> 41
// us, (128, 512, 64, 15, 15, 1 x 1, s 2) 49 -> 24, bf16 (256, 32, 16, 36, 43, 1 x 1) 27.9 -> 14.1, (8, 88, 96, 77, 77, 1 x 1, s 2) 28.6 -> 9.3.
// No size ends it; what is there for short launches levels off at 60 us, which 123 of those 1850 exceed.  So it holds beyond the layers it was
// fitted on: of 5700 others of 150 MB to 5 GB and up to 200 GFLOP (bf16 2 TFLOP), 800 of them large bf16 Images with overlapping windows, 469 fp32
// and 17 bf16 layers beyond 250 MB or 7.6 (59.2) GFLOP are given to the flattened kernel by this comparison alone, and take 0.58 and 0.61 of the
// fixed-geometry kernels' time in the geometric mean, 1.03 at worst: fp32 (256, 32, 498, W, 3, 1 x 1) at W = 155, 170 224 and 242 -> 74 and 88 us, (40, 88,
// 1860, 44, 17, 1 x 1, s 2) 211 -> 125, bf16 (16, 192, 80, 251, 251, 1 x 1) 276 -> 180.  Not for the stem's own kernel, which none of these has.
bool flat_beats_fixed(const cacnn_problem& p, int dtype, const VariantInfo& v, double flat_est, double tiled_est) {
    if (v.fx_whole) return false;
    const Bytes b = compulsory_bytes(p, dtype);
    const double total = b.image + b.filter + b.out, depth = (double)p.C * p.R * p.S;
    const double overlap = std::max(1.0, (double)p.R / (double)p.sigma_w) * std::max(1.0, (double)p.S / (double)p.sigma_h);
    auto over = [](double x, double unit) { return std::max(0.0, std::log(x / unit)); };
    const double one = p.R * p.S == 1 ? 1.0 : 0.0, taps = v.fx_br == 1 && v.fx_bs == 1 && !one ? 1.0 : 0.0, copy = total / 4.6e6, out = b.out / total;
    const double log_tiled = std::log(std::min(tiled_est, 60.0)), log_flat = std::log(std::min(flat_est, 60.0)), deep = over(depth, 128.0), wide = over((double)p.K, 64.0);
    const double narrow = over(32.0, (double)p.C), batch = std::min(1.0, (double)p.B / 64.0), large = over(b.image, 16e6), lap = std::log(overlap);
    const double tc = copy / tiled_est, fc = copy / flat_est;
    const bool f32 = dtype == CACNN_F32;
    const double tiled_fix = f32 ? 0.218 + 0.084 * one + (0.112 + 0.138 * one) * tc + 0.141 * out - 0.071 * log_tiled + 0.020 * taps + 0.012 * narrow - 0.067 * deep + 0.035 * batch
                                 : 0.480 + 0.060 * one + (0.016 - 0.133 * one) * tc - 0.108 * out - 0.107 * log_tiled - 0.092 * taps + 0.092 * narrow + 0.012 * deep - 0.025 * batch;
    const double flat_fix = f32 ? 0.112 - 0.010 * lap - 0.088 * fc - 0.042 * log_flat + (0.009 + 0.061 * lap) * large - 0.008 * one + 0.218 * out + (0.026 + 0.014 * one) * deep - 0.016 * wide
                                : 0.052 - 0.012 * lap - 0.211 * fc - 0.018 * log_flat + (0.035 + 0.042 * lap) * large - 0.144 * one + 0.166 * out + (0.040 + 0.065 * one) * deep + 0.024 * wide;
    return flat_est * std::exp(flat_fix) < (f32 ? 0.8 : 0.75) * tiled_est * std::exp(tiled_fix);
}

// Workgroups share a tile's contraction where the estimate of that is below the other kernel's by this factor: with 1.0 15 of 400 layers
// take up to 1.22 times as long as undivided, with 1.2 one (1.05 times), and the time over all 400 is 0.888 of the undivided one, against 0.882.
// fp32 (1, 784, 64, 3, 12, 3 x 3) 42.2 -> 8.8 us, (4, 464, 156, 10, 7, 3 x 3) 30.6 -> 12.6, bf16 (3, 859, 480, 42, 5, 3 x 3, s 2) 41.5 ->
// 28.5, (72, 976, 16, 5, 5, 3 x 3, s 2) 27.8 -> 11.7
constexpr double kSplitMargin = 1.2;

// What cacnn_conv_forward launches: the planned variant or a kernel with flattened positions.  A generic variant
// gives way to a flattened kernel that takes the problem, but for the case above: on 1500 layers whose plan was a generic variant, large and
// small ones and all those where the two estimates are near each other, the flattened kernel took 0.02 to 1.0 times as long.  A fixed-geometry
// variant, whose price is a measurement, gives way below flat_margin.
int plan_route(const cacnn_problem& p, int dtype, bool aligned_img, bool aligned_flt, Launch* out) {
    double tiled_us = 0.0, flat_est = 0.0;
    // the pipelined kernels need 16-byte aligned operands; a misaligned call is planned without them
    cacnn_plan plan;
    const int rc = plan_impl(&p, dtype, nullptr, &plan, aligned_img && aligned_flt, &tiled_us);
    if (rc != CACNN_OK) return rc;
    if (!planner_uses_lp()) {
        const int fi = choose_flat(p, dtype, &flat_est);
        // (a call whose plan cannot be launched is refused, as it would be without the flattened kernels)
        const VariantInfo& v = variant(plan.variant).info;
        const double tiled_est = with_copy_time(tiled_us - 2.1, p, dtype) + 2.1;
        if (fi >= 0 && tile_list_in_range(p, v, plan.xcd_walk, plan.xcd_split_k) &&
            (v.fx_ct == 0 ? !boxes_for_short_rows(p, dtype)
                          : flat_est < flat_margin(p, dtype) * tiled_est || flat_beats_fixed(p, dtype, v, flat_est, tiled_est))) {
            WindowTile tile;
            const int wi = dtype != CACNN_F32 && aligned_img ? choose_window(p, flat_est, &tile) : -1;
            if (wi >= 0 && prepare_window(p, wi, tile, out) == CACNN_OK) return CACNN_OK;
            const int frc = prepare_flat(p, dtype, fi, out);
            int parts = 0;
            double split_est = 0.0;
            const int si = frc == CACNN_OK ? choose_split(p, dtype, -1, &parts, &split_est) : -1;
            if (si >= 0 && split_est * kSplitMargin < flat_est) (void)prepare_split(p, dtype, si, parts, out);
            return frc;
        }
    }
    return prepare_tiled(p, dtype, plan.variant, plan.b_c, plan.b_r, plan.b_s, plan.xcd_split_k, plan.xcd_walk, aligned_img, aligned_flt, out);
}

LaunchPtr lookup_plan(const cacnn_problem& p, int key) {
    std::lock_guard<std::mutex> lock(g_mutex);
    for (const PlanEntry& e : g_plans)
        if (e.key == key && std::memcmp(&e.p, &p, sizeof(cacnn_problem)) == 0) return e.launch;
    return nullptr;
}

LaunchPtr store_plan(const cacnn_problem& p, int key, const Launch& launch) {
    LaunchPtr kept = std::make_shared<const Launch>(launch);
    std::lock_guard<std::mutex> lock(g_mutex);
    for (PlanEntry& e : g_plans)
        if (e.key == key && std::memcmp(&e.p, &p, sizeof(cacnn_problem)) == 0) return e.launch = kept;
    if (g_plans.size() >= 64) g_plans.erase(g_plans.begin());
    g_plans.push_back(PlanEntry{p, key, kept});
    return kept;
}

// the launch of a call with these operands, remembered or planned now
int route(const cacnn_problem& p, int dtype, const void* image, const void* filter, LaunchPtr* out) {
    const int key = launch_key(dtype, image, filter);
    *out = lookup_plan(p, key);
    if (*out) return CACNN_OK;
    Launch launch;
    const int rc = plan_route(p, dtype, aligned16(image), aligned16(filter), &launch);
    if (rc == CACNN_OK) *out = store_plan(p, key, launch);
    return rc;
}

}  // namespace

extern "C" {

int cacnn_lower_bound(const cacnn_problem* problem, double M_words, cacnn_bound* out) {
    if (!problem || !out) return CACNN_ERR_NULL;
    if (!valid_problem(problem) || !(M_words > 0.0) || !std::isfinite(M_words)) return CACNN_ERR_INVALID_ARG;
    bound_terms(*problem, M_words, out);
    return CACNN_OK;
}

int cacnn_tile_plan(const cacnn_problem* problem, int dtype, const cacnn_machine* machine, cacnn_plan* out) {
    return plan_impl(problem, dtype, machine, out);
}

int cacnn_conv_forward(const cacnn_problem* problem, int dtype, const void* image, const void* filter, void* out,
                       void* hip_stream) {
    if (!problem || !image || !filter || !out) return CACNN_ERR_NULL;
    if (dtype != CACNN_F32 && dtype != CACNN_BF16_F32ACC) return CACNN_ERR_UNSUPPORTED;
    LaunchPtr launch;
    const int rc = route(*problem, dtype, image, filter, &launch);
    if (rc != CACNN_OK) return rc;
    if (!pointers_legal(dtype, image, filter, out)) return CACNN_ERR_INVALID_ARG;
    return fire(*launch, image, filter, out, hip_stream);
}

int cacnn_conv_forward_with_plan(const cacnn_problem* problem, int dtype, const cacnn_plan* plan, const void* image,
                                 const void* filter, void* out, void* hip_stream) {
    if (!problem || !plan || !image || !filter || !out) return CACNN_ERR_NULL;
    if (dtype != CACNN_F32 && dtype != CACNN_BF16_F32ACC) return CACNN_ERR_UNSUPPORTED;
    if (!valid_problem(problem)) return CACNN_ERR_INVALID_ARG;
    const int rc = validate_dims(*problem);
    if (rc != CACNN_OK) return rc;
    if (plan->variant < 0 || plan->variant >= num_variants()) return CACNN_ERR_UNSUPPORTED;
    const VariantInfo& v = variant(plan->variant).info;
    if (v.dtype != dtype) return CACNN_ERR_UNSUPPORTED;
    if (plan->b_c < 1 || plan->b_r < 1 || plan->b_s < 1) return CACNN_ERR_INVALID_ARG;
    const int64_t Cpad = round_up(problem->C, v.cgran());
    // (a fixed-geometry kernel's c-slice is its own, also where it exceeds a small C)
    const int CT = v.fx_ct > 0 && plan->b_c == v.fx_ct ? v.fx_ct : (int)std::min<int64_t>(round_up(plan->b_c, v.cgran()), Cpad);
    const int bR = (int)std::min<int64_t>(plan->b_r, problem->R);
    const int bS = (int)std::min<int64_t>(plan->b_s, problem->S);
    if (plan->xcd_split_k < 0) return CACNN_ERR_INVALID_ARG;
    return launch_with(*problem, dtype, plan->variant, CT, bR, bS, plan->xcd_split_k, plan->xcd_walk, image, filter, out, hip_stream);
}

int cacnn_parallel_bound(const cacnn_problem* problem, double M_words, const cacnn_division* a, cacnn_bound* out) {
    if (!problem || !a || !out) return CACNN_ERR_NULL;
    if (!valid_problem(problem) || !(M_words > 0.0) || !std::isfinite(M_words)) return CACNN_ERR_INVALID_ARG;
    const cacnn_problem& p = *problem;
    if (a->a_b < 1 || a->a_k < 1 || a->a_w < 1 || a->a_h < 1 || a->a_b > p.B || a->a_k > p.K || a->a_w > p.W ||
        a->a_h > p.H)
        return CACNN_ERR_INVALID_ARG;
    parallel_terms(p, M_words, a->a_b, a->a_k, a->a_w, a->a_h, out);
    return CACNN_OK;
}

int cacnn_work_division(const cacnn_problem* problem, double M_words, int32_t p_count, cacnn_division* out_a,
                        cacnn_bound* out_bound) {
    if (!problem || !out_a || !out_bound) return CACNN_ERR_NULL;
    if (!valid_problem(problem) || !(M_words > 0.0) || !std::isfinite(M_words) || p_count < 1 || p_count > 4096)
        return CACNN_ERR_INVALID_ARG;
    const cacnn_problem& p = *problem;
    bool have = false;
    int64_t best_prod = 0;
    double best_rep = 0.0;
    cacnn_division best_a = {1, 1, 1, 1};
    cacnn_bound best_b;
    std::memset(&best_b, 0, sizeof(best_b));
    // every admissible division, in lexicographic order (so the first of equals is the lexicographically smallest)
    for (int64_t ab = 1; ab <= std::min<int64_t>(p.B, p_count); ++ab)
        for (int64_t ak = 1; ak <= std::min<int64_t>(p.K, p_count / ab); ++ak)
            for (int64_t aw = 1; aw <= std::min<int64_t>(p.W, p_count / (ab * ak)); ++aw)
                for (int64_t ah = 1; ah <= std::min<int64_t>(p.H, p_count / (ab * ak * aw)); ++ah) {
                    cacnn_bound b;
                    parallel_terms(p, M_words, ab, ak, aw, ah, &b);
                    const int64_t prod = ab * ak * aw * ah;
                    const double rep = b.term[1] + b.term[2];
                    const bool better = !have || prod > best_prod ||
                                        (prod == best_prod && (b.bound < best_b.bound ||
                                                               (b.bound == best_b.bound && rep < best_rep)));
                    if (better) {
                        have = true;
                        best_prod = prod;
                        best_rep = rep;
                        best_b = b;
                        best_a = cacnn_division{(int32_t)ab, (int32_t)ak, (int32_t)aw, (int32_t)ah};
                    }
                }
    *out_a = best_a;
    *out_bound = best_b;
    return CACNN_OK;
}

int cacnn_tune(const cacnn_problem* problem, int dtype, const void* image, const void* filter, void* out, void* hip_stream,
               cacnn_plan* out_plan) {
    if (!problem || !image || !filter || !out) return CACNN_ERR_NULL;
    if (dtype != CACNN_F32 && dtype != CACNN_BF16_F32ACC) return CACNN_ERR_UNSUPPORTED;
    if (!valid_problem(problem)) return CACNN_ERR_INVALID_ARG;
    {
        const int vrc = validate_dims(*problem);
        if (vrc != CACNN_OK) return vrc;
    }
    if (!have_device()) return CACNN_ERR_NO_DEVICE;
    const bool aligned = aligned16(image) && aligned16(filter);
    const int key = launch_key(dtype, image, filter);
    hipStream_t stream = (hipStream_t)hip_stream;
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return CACNN_ERR_LAUNCH;
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return CACNN_ERR_LAUNCH;
    }
    // every kernel variant that accepts the problem, each with the contraction tile the cost model likes best for it
    Choice best;
    float best_ms = 0.f;
    int status = CACNN_ERR_UNSUPPORTED;
    // warm-up launches, then timed ones; < 0: could not be launched or timed
    auto time_ms = [&](auto launch) {
        constexpr int WARM = 2, TIMED = 5;
        for (int i = 0; i < WARM + TIMED; ++i)
            if ((i == WARM && hipEventRecord(e0, stream) != hipSuccess) || launch() != CACNN_OK) return -1.f;
        float ms = 0.f;
        if (hipEventRecord(e1, stream) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
            hipEventElapsedTime(&ms, e0, e1) != hipSuccess) {
            status = CACNN_ERR_LAUNCH;
            return -1.f;
        }
        return ms;
    };
    for (int vi = 0; vi < num_variants(); ++vi) {
        const VariantInfo& v = variant(vi).info;
        if (v.dtype != dtype || (v.pipelined && !aligned)) continue;
        Choice c;
        if (!evaluate(vi, *problem, kDefaultMachine, &c)) continue;
        const float ms = time_ms([&] {
            return launch_with(*problem, dtype, vi, c.g.CT, c.g.bR, c.g.bS, 0, 0, image, filter, out, hip_stream);
        });
        if (ms < 0.f) continue;
        if (best.variant < 0 || ms < best_ms) {
            best = c;
            best_ms = ms;
        }
    }
    // ... and every kernel with flattened positions
    int flat = -1;
    for (int i = 0; i < num_flat() && best.variant >= 0; ++i) {
        if (!flat_fits(*problem, dtype, flat_variant(i).info)) continue;
        const float ms = time_ms([&] { return launch_flat(*problem, dtype, i, image, filter, out, hip_stream); });
        if (ms >= 0.f && ms < best_ms) {
            flat = i;
            best_ms = ms;
        }
    }
    // ... and every window kernel with one box and with two, each on the tile that stages the fewest words
    int window = -1;
    WindowTile window_tile;
    for (int i = 0; i < 2 * num_window() && best.variant >= 0 && dtype != CACNN_F32 && aligned16(image); ++i) {
        WindowTile t;
        Launch l;
        if (!pick_window_tile(*problem, i / 2, 2 - i % 2, &t, &l)) continue;
        const float ms = time_ms([&] { return fire(l, image, filter, out, hip_stream); });
        if (ms >= 0.f && ms < best_ms) {
            window = i / 2;
            window_tile = t;
            best_ms = ms;
        }
    }
    // ... and those whose workgroups share the contraction, each with the number of parts that the estimate likes best
    int split = -1, split_parts = 0;
    for (int i = 0; i < num_flat() && best.variant >= 0 && !hip_stream; ++i) {
        int parts = 0;
        double us = 0.0;
        Launch l;
        if (choose_split(*problem, dtype, i, &parts, &us) < 0 || prepare_split(*problem, dtype, i, parts, &l) != CACNN_OK) continue;
        const float ms = time_ms([&] { return fire(l, image, filter, out, nullptr); });
        if (ms >= 0.f && ms < best_ms) {
            split = i;
            split_parts = parts;
            best_ms = ms;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (best.variant < 0) return status;
    cacnn_plan plan;
    const int rc = fill_plan(*problem, dtype, kDefaultMachine, best, &plan);
    if (rc != CACNN_OK) return rc;
    Launch launch;
    const int lrc = window >= 0 ? prepare_window(*problem, window, window_tile, &launch)
                    : flat >= 0 ? prepare_flat(*problem, dtype, flat, &launch)
                                : prepare_tiled(*problem, dtype, plan.variant, plan.b_c, plan.b_r, plan.b_s, plan.xcd_split_k, plan.xcd_walk,
                                                aligned16(image), aligned16(filter), &launch);
    if (lrc != CACNN_OK) return lrc;
    if (split >= 0) (void)prepare_split(*problem, dtype, split, split_parts, &launch);
    // (the entry is one for all streams: tuned on another one, where they cannot be timed, the null stream keeps those that it had)
    LaunchPtr before;
    if (hip_stream && route(*problem, dtype, image, filter, &before) == CACNN_OK && before->split) {
        launch.split = before->split;
        launch.split_grid = before->split_grid;
        launch.fs = before->fs;
    }
    store_plan(*problem, key, launch);
    if (out_plan) *out_plan = plan;
    return CACNN_OK;
}

int cacnn_plan_variant(const cacnn_problem* problem, int dtype, int variant_index, cacnn_plan* out, double* model_us,
                       double* model_terms) {
    if (!problem || !out) return CACNN_ERR_NULL;
    if (!valid_problem(problem)) return CACNN_ERR_INVALID_ARG;
    if (dtype != CACNN_F32 && dtype != CACNN_BF16_F32ACC) return CACNN_ERR_UNSUPPORTED;
    if (variant_index < 0 || variant_index >= num_variants() || variant(variant_index).info.dtype != dtype)
        return CACNN_ERR_UNSUPPORTED;
    {
        const int vrc = validate_dims(*problem);
        if (vrc != CACNN_OK) return vrc;
    }
    Choice c;
    if (!evaluate(variant_index, *problem, kDefaultMachine, &c)) return CACNN_ERR_UNSUPPORTED;
    if (model_us) *model_us = c.cost / 2400.0;
    if (model_terms)
        for (int i = 0; i < 5; ++i) model_terms[i] = c.terms[i];
    return fill_plan(*problem, dtype, kDefaultMachine, c, out);
}

int cacnn_two_level_plan(const cacnn_problem* problem, int dtype, const cacnn_machine* machine,
                         const cacnn_machine_l2* machine_l2, cacnn_l2_plan* out) {
    if (!problem || !out) return CACNN_ERR_NULL;
    cacnn_plan plan;
    const int rc = plan_impl(problem, dtype, machine, &plan);
    if (rc != CACNN_OK) return rc;
    const cacnn_problem& p = *problem;
    const double esz = dtype == CACNN_F32 ? 4.0 : 2.0;
    L2Machine m2 = kDefaultL2Bytes;
    if (machine_l2) {
        if (machine_l2->l2_bytes < 1024 || machine_l2->n_xcd < 1 || machine_l2->n_xcd > 8 ||
            (machine_l2->n_xcd & (machine_l2->n_xcd - 1)) || machine_l2->cu_per_xcd < 1)
            return CACNN_ERR_INVALID_ARG;
        m2.words = (double)machine_l2->l2_bytes;
        m2.n_xcd = machine_l2->n_xcd;
        m2.cu_per_xcd = machine_l2->cu_per_xcd;
    }
    m2.words /= esz;
    std::memset(out, 0, sizeof(*out));
    const double M = m2.words;
    const LpSolution s = solve_tiling_lp(p, M);
    for (int i = 0; i < 9; ++i) out->lp_tile[i] = std::pow(M, s.l[i]);
    out->lp_volume = std::pow(M, s.log_volume);
    out->lp_cost_words = (double)p.B * p.C * p.K * p.W * p.H * p.R * p.S * M / out->lp_volume;
    cacnn_bound b;
    bound_terms(p, M, &b);
    out->bound_words = b.bound;
    // the LP's tile rounded to whole LDS tiles
    auto whole = [](double lp, int tile, int64_t extent) {
        const int64_t n = std::max<int64_t>(1, (int64_t)std::floor(lp / tile + 0.5));
        return (int32_t)std::min<int64_t>(n * tile, round_up(extent, tile));
    };
    out->l2_tile_b = whole(out->lp_tile[0], plan.b_b, p.B);
    out->l2_tile_k = whole(out->lp_tile[2], plan.b_k, p.K);
    out->l2_tile_w = whole(out->lp_tile[3], plan.b_w, p.W);
    out->l2_tile_h = whole(out->lp_tile[4], plan.b_h, p.H);
    const VariantInfo& v = variant(plan.variant).info;
    const int64_t grid = machine_l2 ? std::min<int64_t>(plan.grid[0], (int64_t)m2.n_xcd * m2.cu_per_xcd) : plan.grid[0];
    const L2Choice l2 = choose_l2_layout(p, dtype, v, grid, m2);
    out->a_k = l2.a_k;
    out->walk = l2.walk;
    out->n_candidates = l2.n;
    for (int i = 0; i < l2.n; ++i) {
        out->cand_a_k[i] = l2.cand_a_k[i];
        out->cand_walk[i] = l2.cand_walk[i];
        out->cand_words[i] = l2.cand_words[i];
    }
    out->chosen_words = l2.words;
    {
        // Section 7 for the chosen a_K, the positions divided over the remaining processors: images, then rows, then columns
        int64_t rest = m2.n_xcd / l2.a_k, ab = 1, ah = 1, aw = 1;
        for (int64_t* a : {&ab, &ah, &aw}) {
            const int64_t extent = a == &ab ? p.B : (a == &ah ? p.H : p.W);
            while (*a * 2 <= std::min<int64_t>(rest, extent)) *a *= 2;
            rest /= *a;
        }
        cacnn_bound pb;
        parallel_terms(p, M, ab, l2.a_k, aw, ah, &pb);
        out->parallel_bound_words = pb.bound;
    }
    return CACNN_OK;
}

int cacnn_pool_lower_bound(const cacnn_problem* problem, double M_words, cacnn_pool_bound* out) {
    if (!problem || !out) return CACNN_ERR_NULL;
    if (!valid_problem(problem) || !(M_words > 0.0) || !std::isfinite(M_words)) return CACNN_ERR_INVALID_ARG;
    const cacnn_problem& p = *problem;
    const double sw = (double)std::min(p.sigma_w, p.R), sh = (double)std::min(p.sigma_h, p.S);
    const double bkwh = (double)p.B * p.K * p.W * p.H, bcwh = (double)p.B * p.C * p.W * p.H;
    out->term[0] = bkwh;
    out->term[1] = sw * sh * bcwh;
    out->term[2] = bkwh * (double)p.C * p.R * p.S / M_words;
    out->argmax = 0;
    for (int i = 1; i < 3; ++i)
        if (out->term[i] > out->term[out->argmax]) out->argmax = i;
    out->bound = out->term[out->argmax];
    return CACNN_OK;
}

// What a pooling call launches; CACNN_OK, or why it is refused.
static int prepare_pool(const cacnn_problem& p, int dtype, const void* image, const void* out, PoolArgs* args, int* images) {
    {
        // element counts of Image and Out within the kernel's 32-bit indexing
        const int64_t lim = INT32_MAX;
        if (p.sigma_w > lim || p.sigma_h > lim || p.W > lim || p.H > lim || p.R > lim || p.S > lim) return CACNN_ERR_INVALID_ARG;
        const int64_t IW = p.sigma_w * (p.W - 1) + p.R, IH = p.sigma_h * (p.H - 1) + p.S;
        int64_t t;
        if (IW > lim || IH > lim || !mul_check(IW, IH, lim, &t) || !mul_check(t, p.C, lim, &t) || !mul_check(t, p.B, lim, &t))
            return CACNN_ERR_INVALID_ARG;
        if (!mul_check(p.K, p.H, lim, &t) || !mul_check(t, p.W, lim, &t) || !mul_check(t, p.B, lim, &t))
            return CACNN_ERR_INVALID_ARG;
    }
    const size_t esz = dtype == CACNN_F32 ? 4 : 2;
    if (reinterpret_cast<uintptr_t>(image) % esz || reinterpret_cast<uintptr_t>(out) % 4) return CACNN_ERR_INVALID_ARG;
    const int full = dtype == CACNN_F32 ? 4 : 8;
    // images per thread: as many as one load takes (16 bytes) or the largest power of two below that divides B
    int vec = full;
    while (vec > 1 && (p.B % vec || reinterpret_cast<uintptr_t>(image) % (vec * esz) || reinterpret_cast<uintptr_t>(out) % std::min(16, vec * 4)))
        vec /= 2;
    PoolArgs& a = *args;
    std::memset(&a, 0, sizeof(a));
    a.image = image;
    a.out = (float*)const_cast<void*>(out);
    a.B = (int32_t)p.B;
    a.C = (int32_t)p.C;
    a.W = (int32_t)p.W;
    a.H = (int32_t)p.H;
    a.R = (int32_t)p.R;
    a.S = (int32_t)p.S;
    a.sw = (int32_t)p.sigma_w;
    a.sh = (int32_t)p.sigma_h;
    a.IH = (int32_t)(p.sigma_h * (p.H - 1) + p.S);
    a.BV = (int32_t)(p.B / vec);
    a.n_xcd = xcd_count();
    a.TWC = (int32_t)ceil_div(p.W, a.n_xcd);              // one band of output columns per XCD
    const int64_t chunks = ceil_div(p.W, a.TWC);
    int64_t n = 0;
    // The reciprocal divisions in the kernel are exact while dividend * divisor < 2^32.  The limit is that of a thread per
    // 16-byte load, or per image where those do not divide B, whatever the images per thread are.
    const int64_t groups = vec == full ? p.B / full : p.B;
    if (!mul_check(p.H, chunks * a.TWC, INT32_MAX, &n) || !mul_check(n, p.C, INT32_MAX, &n) || !mul_check(n, groups, INT32_MAX, &n) ||
        (double)n * (double)std::max<int64_t>(std::max<int64_t>(groups, p.C), std::max<int64_t>(p.H, 64)) >= 4294967296.0)
        return CACNN_ERR_INVALID_ARG;
    // Where a row of images is whole cache lines the kernel stores past the L2, and a thread's 8 floats would reach memory in two
    // instructions of half lines each: 4 images per thread then, whose stores are contiguous (bf16 (32, 100, 50, 75, 2 x 2, s 2)
    // 27.6 us with 8, 24.7 with 4; (128, 64, 56, 56, 3 x 3, s 2) 75.2 and 74.0), where the thread count still fits the limit.  With 4 there are
    // twice the loads, though, and where windows overlap and are read from the caches these set the pace: so windows of at most five
    // elements, or with at most 9/4 reads of an element.  With 8 and with 4: (64, 13, 98, 98, 7 x 7) 33.9 and 49.0 us, (256, 399, 2, 50, 7 x 8, s 1 2)
    // 150 and 164, (32, 291, 18, 18, 7 x 7) 19.7 and 21.3, (32, 118, 70, 70, 3 x 3) 23.5 and 25.0; (64, 138, 20, 20, 2 x 1) 5.3 and 4.6; over
    // 500 calls the choice loses 1.012 to the better of both in the geometric mean (always 4: 1.06).  Where Out itself does not start on half a line
    // ordinary stores and these win in turn, by up to 1.16 times: it is stored past the L2 there too.
    a.stream = p.B % 32 == 0;
    const double overlap = std::max(1.0, (double)p.R / (double)p.sigma_w) * std::max(1.0, (double)p.S / (double)p.sigma_h);
    const bool few_loads = p.R * p.S <= 5 || overlap <= 2.25;
    if (a.stream && few_loads && vec == 8 && n * 2 <= INT32_MAX &&
        (double)n * 2.0 * (double)std::max<int64_t>(std::max<int64_t>(groups * 2, p.C), std::max<int64_t>(p.H, 64)) < 4294967296.0) {
        vec = 4;
        a.BV = (int32_t)(p.B / vec);
    }
    n = n / groups * a.BV;
    a.n_threads = (int32_t)n;
    a.n_wg = (int32_t)ceil_div(n, 256);
    const double img_bytes = (double)(p.sigma_w * (p.W - 1) + p.R) * (double)(p.sigma_h * (p.H - 1) + p.S) * (double)p.C * (double)p.B * (double)esz;
    a.img_bytes = img_bytes < 2147483648.0 ? (int32_t)img_bytes : 0;
    a.xcd_q = a.n_wg / a.n_xcd;
    a.xcd_rem = a.n_wg % a.n_xcd;
    a.d_BV = make_fastdiv((uint32_t)a.BV);
    a.d_C = make_fastdiv((uint32_t)a.C);
    a.d_TWC = make_fastdiv((uint32_t)a.TWC);
    a.d_H = make_fastdiv((uint32_t)a.H);
    a.d_nxcd = make_fastdiv((uint32_t)a.n_xcd);
    *images = vec;
    return CACNN_OK;
}

int cacnn_pool_forward(const cacnn_problem* problem, int dtype, int mode, const void* image, void* out,
                       void* hip_stream) {
    if (!problem || !image || !out) return CACNN_ERR_NULL;
    if (dtype != CACNN_F32 && dtype != CACNN_BF16_F32ACC) return CACNN_ERR_UNSUPPORTED;
    if (mode != CACNN_POOL_AVG && mode != CACNN_POOL_MAX) return CACNN_ERR_UNSUPPORTED;
    if (!valid_problem(problem) || problem->K != problem->C) return CACNN_ERR_INVALID_ARG;
    PoolArgs a;
    int images = 0;
    const int rc = prepare_pool(*problem, dtype, image, out, &a, &images);
    if (rc != CACNN_OK) return rc;
    if (!have_device()) return CACNN_ERR_NO_DEVICE;
    return launch_pool(a, dtype, mode, images, hip_stream) == 0 ? CACNN_OK : CACNN_ERR_LAUNCH;
}

int cacnn_probe_mfma(int dtype, const void* operands, float* sink, int32_t iters, int64_t* mfma_issued, void* hip_stream) {
    if (!operands || !sink || !mfma_issued) return CACNN_ERR_NULL;
    if (dtype != CACNN_F32 && dtype != CACNN_BF16_F32ACC) return CACNN_ERR_UNSUPPORTED;
    if (iters < 1 || iters > (1 << 24) || reinterpret_cast<uintptr_t>(operands) % 16 || reinterpret_cast<uintptr_t>(sink) % 4)
        return CACNN_ERR_INVALID_ARG;
    if (!have_device()) return CACNN_ERR_NO_DEVICE;
    const int grid = kDefaultMachine.num_cu;
    *mfma_issued = (int64_t)grid * 4 * iters * 42;
    return launch_mfma_probe(dtype, operands, sink, iters, grid, hip_stream) == 0 ? CACNN_OK : CACNN_ERR_LAUNCH;
}

int cacnn_probe_lds_fill(const void* src, size_t window_bytes, float* sink, int32_t iters, void* hip_stream, int64_t* bytes_moved) {
    if (!src || !sink || !bytes_moved) return CACNN_ERR_NULL;
    if (window_bytes < 65536 || window_bytes > (1ull << 30) || (window_bytes & (window_bytes - 1)) || iters < 1 ||
        iters > (1 << 20) || reinterpret_cast<uintptr_t>(src) % 16)
        return CACNN_ERR_INVALID_ARG;
    if (!have_device()) return CACNN_ERR_NO_DEVICE;
    const int grid = kDefaultMachine.num_cu;
    *bytes_moved = (int64_t)grid * 4 * 12 * 1024 * iters;
    return launch_lds_fill_probe(src, (uint32_t)window_bytes, iters, sink, grid, hip_stream) == 0 ? CACNN_OK : CACNN_ERR_LAUNCH;
}

int cacnn_probe_mfma_and_fill(const void* operands, const void* src, size_t window_bytes, float* sink, int32_t mfma_iters,
                              int32_t fill_iters, void* hip_stream) {
    return cacnn_probe_mfma_and_fill_on((int32_t)kDefaultMachine.num_cu, 0, 0, operands, src, window_bytes, sink, mfma_iters,
                                        fill_iters, hip_stream);
}

int cacnn_probe_mfma_and_fill_on(int32_t compute_units, int32_t tile, int32_t mode, const void* operands, const void* src,
                                 size_t window_bytes, float* sink, int32_t mfma_iters, int32_t fill_iters, void* hip_stream) {
    if (!operands || !src || !sink) return CACNN_ERR_NULL;
    // mode: bit 0 = operands read from LDS, bit 1 = a workgroup barrier per iteration (equal iteration counts only)
    if (compute_units < 1 || compute_units > kDefaultMachine.num_cu || mode < 0 || mode > 3 || (tile != 0 && tile != 1))
        return CACNN_ERR_INVALID_ARG;
    if ((mode & 2) && mfma_iters != fill_iters) return CACNN_ERR_INVALID_ARG;
    if (window_bytes < 65536 || window_bytes > (32u << 20) || (window_bytes & (window_bytes - 1)) || mfma_iters < 0 ||
        fill_iters < 0 || mfma_iters > (1 << 20) || fill_iters > (1 << 20) || (mfma_iters == 0 && fill_iters == 0) ||
        reinterpret_cast<uintptr_t>(src) % 16 || reinterpret_cast<uintptr_t>(operands) % 16)
        return CACNN_ERR_INVALID_ARG;
    if (!have_device()) return CACNN_ERR_NO_DEVICE;
    return launch_mfma_and_fill_probe(tile, operands, src, (uint32_t)window_bytes, mfma_iters, fill_iters, mode & 1, (mode >> 1) & 1, sink, compute_units,
                                      hip_stream) == 0
               ? CACNN_OK
               : CACNN_ERR_LAUNCH;
}

int cacnn_probe_copy(const void* src, void* dst, size_t bytes, void* hip_stream) {
    if (!src || !dst) return CACNN_ERR_NULL;
    if (bytes == 0 || bytes % 16 || reinterpret_cast<uintptr_t>(src) % 16 || reinterpret_cast<uintptr_t>(dst) % 16)
        return CACNN_ERR_INVALID_ARG;
    if (!have_device()) return CACNN_ERR_NO_DEVICE;
    return launch_copy_probe(src, dst, bytes, kDefaultMachine.num_cu * 8, hip_stream) == 0 ? CACNN_OK : CACNN_ERR_LAUNCH;
}

// Section 5.1: the tabulated closed form.  theta is clamped into the tabulated box first; a region is a set of faces
// a.theta <= b with integer coefficients, its form nine integer rows over a common denominator.
int cacnn_closed_form_tiling(const cacnn_problem* p, double M, cacnn_closed_form* out) {
    if (!p || !out) return CACNN_ERR_NULL;
    if (!valid_problem(p) || !(M > 1.0)) return CACNN_ERR_INVALID_ARG;
    std::memset(out, 0, sizeof(*out));
    const double lnM = std::log(M);
    auto lg = [&](int64_t v) { return std::log((double)v) / lnM; };
    double th[9] = {lg(p->B), lg(p->C), lg(p->K), lg(p->W), lg(p->H), lg(p->R), lg(p->S), lg(p->sigma_w), lg(p->sigma_h)};
    for (int i = 0; i < 5; ++i) th[i] = std::min(th[i], 1.0);
    for (int i = 0; i < 2; ++i) {       // (R, sigma_w), (S, sigma_h): the LP sees min(sigma, extent) and extent / sigma
        double sg = std::min(th[7 + i], th[5 + i]);
        const double rest = std::min(th[5 + i] - sg, 1.0);
        sg = std::min(sg, 1.0);
        th[7 + i] = sg;
        th[5 + i] = sg + rest;
    }
    int best = 0;
    double best_v = std::numeric_limits<double>::infinity();
    for (int r = 0; r < kClosedFormRegions; ++r) {
        double worst = -std::numeric_limits<double>::infinity();
        for (int f = kClosedFormRegion[r][0]; f < kClosedFormRegion[r][0] + kClosedFormRegion[r][1]; ++f) {
            double v = -(double)kClosedFormFace[f][9];
            for (int j = 0; j < 9; ++j) v += (double)kClosedFormFace[f][j] * th[j];
            worst = std::max(worst, v);
        }
        if (worst < best_v) {
            best_v = worst;
            best = r;
        }
        if (worst <= 1e-12) break;
    }
    const int form = kClosedFormRegion[best][2];
    out->region = best;
    out->n_regions = kClosedFormRegions;
    double sum = 0.0;
    for (int i = 0; i < 9; ++i) {
        double v = (double)kClosedFormNum[form][i][9];
        for (int j = 0; j < 9; ++j) v += (double)kClosedFormNum[form][i][j] * th[j];
        v /= (double)kClosedFormDen[form];
        out->theta[i] = th[i];
        out->l[i] = std::max(v, 0.0);
        out->tile[i] = std::pow(M, out->l[i]);
        sum += out->l[i];
    }
    // how far l is from satisfying the LP's rows (the same rows solve_tiling_lp builds)
    {
        const double* l = out->l;
        const double rows[15] = {l[0] - th[0], l[1] - th[1], l[2] - th[2], l[3] - th[3], l[4] - th[4], l[6] - th[7], l[8] - th[8],
                                 l[5] - (th[5] - th[7]), l[7] - (th[6] - th[8]),
                                 l[0] + l[2] + l[3] + l[4] - 1.0, l[1] + l[2] + l[5] + l[6] + l[7] + l[8] - 1.0,
                                 l[0] + l[1] + l[3] + l[4] + l[6] + l[8] - 1.0, l[0] + l[1] + l[3] + l[7] + l[6] + l[8] - 1.0,
                                 l[0] + l[1] + l[5] + l[4] + l[6] + l[8] - 1.0, l[0] + l[1] + l[5] + l[7] + l[6] + l[8] - 1.0};
        double worst = 0.0;
        for (double v : rows) worst = std::max(worst, v);
        out->worst_violation = worst;
    }
    out->log_volume = sum;
    out->volume = std::pow(M, sum);
    const double F = (double)p->B * p->C * p->K * p->W * p->H * p->R * p->S;
    out->cost_words = F * M / out->volume;
    cacnn_bound b;
    bound_terms(*p, M, &b);
    out->bound_words = b.bound;
    return CACNN_OK;
}

// The two calls for the binding's tensors: element counts instead of a check in the interpreter.  CACNN_ERR_INVALID_ARG if a buffer
// is shorter than the problem needs (nothing is enqueued).
static bool holds(const cacnn_problem& p, int64_t image_elems, int64_t filter_elems, int64_t out_elems) {
    if (!valid_problem(&p) || validate_dims(p) != CACNN_OK) return false;
    return image_elems >= (p.sigma_w * (p.W - 1) + p.R) * (p.sigma_h * (p.H - 1) + p.S) * p.C * p.B &&
           filter_elems >= p.K * p.R * p.S * p.C && out_elems >= p.K * p.H * p.W * p.B;
}
int cacnn_internal_conv_forward_sized(const cacnn_problem* problem, int dtype, const void* image, int64_t image_elems, const void* filter,
                                      int64_t filter_elems, void* out, int64_t out_elems, void* hip_stream) {
    if (!problem || !holds(*problem, image_elems, filter_elems, out_elems)) return CACNN_ERR_INVALID_ARG;
    return cacnn_conv_forward(problem, dtype, image, filter, out, hip_stream);
}
int cacnn_internal_pool_forward_sized(const cacnn_problem* problem, int dtype, int mode, const void* image, int64_t image_elems, void* out,
                                      int64_t out_elems, void* hip_stream) {
    if (!problem || problem->K != problem->C || !holds(*problem, image_elems, INT64_MAX, out_elems)) return CACNN_ERR_INVALID_ARG;
    return cacnn_pool_forward(problem, dtype, mode, image, out, hip_stream);
}
int cacnn_internal_sized_interface(void) { return kSizedInterface; }
// Which kernel cacnn_conv_forward launches for a problem and operands at these addresses (of which the alignment alone matters):
// {0: a variant with box tiles, 1: a flattened kernel, 2: a window kernel; its index; workgroups; threads of one}.  Nothing is enqueued.
int cacnn_internal_route(const cacnn_problem* problem, int dtype, const void* image, const void* filter, int32_t* four) {
    if (!problem || !four) return CACNN_ERR_NULL;
    if (dtype != CACNN_F32 && dtype != CACNN_BF16_F32ACC) return CACNN_ERR_UNSUPPORTED;
    LaunchPtr launch;
    const int rc = route(*problem, dtype, image, filter, &launch);
    if (rc != CACNN_OK) return rc;
    const Launch& l = *launch;
    four[0] = l.window ? 2 : l.flat ? 1 : 0;
    four[1] = l.window ? (int32_t)(l.window - &window_variant(0)) : l.flat ? (int32_t)(l.flat - &flat_variant(0)) : (int32_t)(l.tiled - &variant(0));
    four[2] = l.grid;
    four[3] = l.window ? l.window->info.threads() : l.flat ? l.flat->info.threads() : l.tiled->info.threads();
    return CACNN_OK;
}
// {kernel; parts; workgroups} where cacnn_conv_forward launches, on the null stream, workgroups that share a tile's contraction; else zeros
int cacnn_internal_route_split(const cacnn_problem* problem, int dtype, const void* image, const void* filter, int32_t* three) {
    if (!problem || !three) return CACNN_ERR_NULL;
    if (dtype != CACNN_F32 && dtype != CACNN_BF16_F32ACC) return CACNN_ERR_UNSUPPORTED;
    LaunchPtr launch;
    const int rc = route(*problem, dtype, image, filter, &launch);
    if (rc != CACNN_OK) return rc;
    const Launch& l = *launch;
    three[0] = l.split ? (int32_t)(l.split - &flat_variant(0)) : 0;
    three[1] = l.split ? (int32_t)l.fs.parts : 0;
    three[2] = l.split ? l.split_grid : 0;
    return CACNN_OK;
}
// Images per thread of a pooling call with operands at these addresses, 0 if it is refused
int cacnn_internal_pool_images(const cacnn_problem* problem, int dtype, const void* image, const void* out) {
    PoolArgs a;
    int images = 0;
    if (!problem || !valid_problem(problem) || problem->K != problem->C || (dtype != CACNN_F32 && dtype != CACNN_BF16_F32ACC)) return 0;
    return prepare_pool(*problem, dtype, image, out, &a, &images) == CACNN_OK ? images : 0;
}
int cacnn_internal_flat_count(void) { return num_flat(); }
int cacnn_internal_flat_info(int i, int32_t* eight) {
    if (i < 0 || i >= num_flat() || !eight) return CACNN_ERR_INVALID_ARG;
    const FlatInfo& v = flat_variant(i).info;
    const int32_t x[8] = {v.dtype, v.MB, v.NG, v.IM, v.WM, v.WN, v.WK, v.NCH};
    std::memcpy(eight, x, sizeof(x));
    return CACNN_OK;
}
double cacnn_internal_flat_us(const cacnn_problem* p, int dtype, int i) {
    return p && i >= 0 && i < num_flat() && flat_fits(*p, dtype, flat_variant(i).info) ? flat_us(*p, dtype, flat_variant(i).info) : -1.0;
}
int cacnn_internal_flat_forward(const cacnn_problem* problem, int dtype, int index, const void* image, const void* filter, void* out,
                                void* hip_stream) {
    if (!problem || !image || !filter || !out) return CACNN_ERR_NULL;
    if (dtype != CACNN_F32 && dtype != CACNN_BF16_F32ACC) return CACNN_ERR_UNSUPPORTED;
    if (!valid_problem(problem)) return CACNN_ERR_INVALID_ARG;
    const int rc = validate_dims(*problem);
    if (rc != CACNN_OK) return rc;
    if (index < 0 || index >= num_flat()) return CACNN_ERR_UNSUPPORTED;
    return launch_flat(*problem, dtype, index, image, filter, out, hip_stream);
}
// The same kernel with the contraction of a tile divided into about `parts` parts, on the null stream
int cacnn_internal_split_forward(const cacnn_problem* problem, int dtype, int index, int parts, const void* image, const void* filter, void* out) {
    if (!problem || !image || !filter || !out) return CACNN_ERR_NULL;
    if (dtype != CACNN_F32 && dtype != CACNN_BF16_F32ACC) return CACNN_ERR_UNSUPPORTED;
    if (!valid_problem(problem) || validate_dims(*problem) != CACNN_OK) return CACNN_ERR_INVALID_ARG;
    if (index < 0 || index >= num_flat()) return CACNN_ERR_UNSUPPORTED;
    if (!pointers_legal(dtype, image, filter, out)) return CACNN_ERR_INVALID_ARG;
    Launch l;
    const int rc = prepare_split(*problem, dtype, index, parts, &l);
    return rc != CACNN_OK ? rc : fire(l, image, filter, out, nullptr);
}

int cacnn_internal_window_count(void) { return num_window(); }
// {blocks of 32 output channels and of 32 columns of a wave; waves along either; images of a tile}
int cacnn_internal_window_info(int i, int32_t* five) {
    if (i < 0 || i >= num_window() || !five) return CACNN_ERR_INVALID_ARG;
    const WindowInfo& v = window_variant(i).info;
    const int32_t x[5] = {v.MB, v.NB, v.WM, v.WN, v.TB};
    std::memcpy(five, x, sizeof(x));
    return CACNN_OK;
}
// A window kernel with tiles of TW columns and `bufs` boxes, bf16
int cacnn_internal_window_forward(const cacnn_problem* problem, int index, int TW, int bufs, const void* image, const void* filter, void* out,
                                  void* hip_stream) {
    if (!problem || !image || !filter || !out) return CACNN_ERR_NULL;
    if (!valid_problem(problem) || validate_dims(*problem) != CACNN_OK) return CACNN_ERR_INVALID_ARG;
    if (index < 0 || index >= num_window() || TW < 1 || bufs < 1 || bufs > 2) return CACNN_ERR_UNSUPPORTED;
    const WindowInfo& v = window_variant(index).info;
    if (!pointers_legal(CACNN_BF16_F32ACC, image, filter, out)) return CACNN_ERR_INVALID_ARG;
    if (!aligned16(image)) return CACNN_ERR_UNSUPPORTED;
    WindowTile t;
    t.TW = TW;
    t.TH = v.cols() / v.TB / TW;
    t.bufs = bufs;
    Launch l;
    const int rc = prepare_window(*problem, index, t, &l);
    return rc != CACNN_OK ? rc : fire(l, image, filter, out, hip_stream);
}

int cacnn_variant_count(void) { return num_variants(); }

const char* cacnn_variant_name(int i) {
    if (i < 0 || i >= num_variants()) return nullptr;
    return variant(i).info.name;
}

const char* cacnn_status_string(int status) {
    switch (status) {
        case CACNN_OK: return "ok";
        case CACNN_ERR_NULL: return "null pointer argument";
        case CACNN_ERR_INVALID_ARG: return "invalid argument";
        case CACNN_ERR_UNSUPPORTED: return "unsupported dtype, variant or plan";
        case CACNN_ERR_LAUNCH: return "kernel launch failed";
        case CACNN_ERR_NO_DEVICE: return "no usable GPU";
        default: return "unknown status";
    }
}

}  // extern "C"
