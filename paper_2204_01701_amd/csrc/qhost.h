// qhost.h -- host-side planning shared by the library's translation units:
// descriptor checks (Geom), tile-configuration and split-K plans, workspace
// sizes, and the launchers each kernel family's translation unit defines.
// Nothing here touches tensor data or allocates device memory.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdlib>

#include "qlayer.h"
#include "qargs.h"
#include "qdevice.h"
#include "qconv_aux.h"
#include "qconv_depthwise.h"
#include "qconv_fwd_smallc.h"
#include "qconv_fwd_narrow.h"

namespace ql {
namespace host {

// Device address of the 16 zero bytes masked-off DMA lanes read (qlayer_api.hip).
const void *zero_page();


constexpr int kNumCUs = 256;         // MI355X compute units
constexpr size_t kAlign = 256;
constexpr long long kMaxElems = (1LL << 31) - 1;  // 32-bit element offsets in the kernels
constexpr size_t kMaxSplitBytes = 128ull << 20;  // cap on split-K partial sums (written + read once)
// Cap on a pass's padded copies (Geom::pad_bwd_data, pad_bwd_weight): what X alone
// can take within 32-bit element offsets in fp32, so the forward's copy is always
// below.  Beyond it the register-staged kernels take the tensors as they are.  A
// bound on memory and not a line of speed: 24 x 512 x 512 maps, 20 -> 60 channels, 3 x 3,
// bf16, input and weight gradient 18.8 and 9.5 ms as they are, 3.3 and 1.8 padded (2.4 GB
// of copies); a cap of 2 GiB cost such layers four fifths of their speed.
constexpr size_t kMaxPadBytes = 8192ull << 20;
// Split-K cost model, in units of one K step of one workgroup alone on a CU:
// a CU holding two co-resident workgroups finishes both in kSharedRound steps
// per step each (the second one hides the first one's latency), and one unit
// of time moves about kBytesPerStep bytes of partial sums through HBM.
constexpr double kSharedRound = 1.25;
// ... for the forward kernels, whose second workgroup on a CU adds less (measured on
// the 4 x 4 VGG-16 layers: two splits of 256 workgroups beat four of 512)
constexpr double kSharedRoundFwd = 1.6;
constexpr double kBytesPerStep = 3.2e6;
constexpr double kReduceSteps = 6.0;  // the reduction kernel's launch and ramp
// An fp32 K step takes about three times a bf16 one (the fp32 MFMA rate), so
// the partial sums' traffic and the reduction cost a third as many steps.
// Measured on 18 fp32 shapes with the factor at 1, 1.5, 2, 3, 4, 6: from 1 to 3
// the forward of 64 -> 64 channels, 256 x 8 x 8 maps, 3 x 3, goes from 64 to 40
// us, 32 -> 64 at stride 2 from 37 to 26, the input gradient of 128 -> 128,
// 16 x 14 x 14 maps, 1 x 1, from 32 to 24; above 3 the weight gradients slow down.
// That is one per weighted term: the types with fewer terms run as many fewer MFMAs.
// A workgroup of two pipelines (one per CU) on the two halves of its K range:
// the cost of a K step of each pipeline, in the units above.  The two
// pipelines share the workgroup's barriers, which costs them some of the
// latency hiding of two independent workgroups (measured on the VGG-16
// weight gradients: 1.5 reproduces which of the two kernels is faster on
// every layer).
constexpr double kPipeRound = 1.5;
// A K step of the 8-wave workgroup with the 128-channel tile (one per CU, twice
// the MFMAs of a 64-channel step), in the same units (measured on the same
// layers: 1.2 reproduces where it is the fastest of the three kernels).
constexpr double kFatStep = 1.2;
// A tile's ramp (first loads, epilogue) in K steps, for the choice between tiles;
// the split counts are searched without it.  Fitted on 1200 layers of random
// sizes timed in every tile: weight gradients in the tile chosen 0.4 % slower than in
// the best (geometric mean; 1.0 % without the ramps, 13 of 630 bf16 layers more than 6 %
// slower than before the 64 x 64 tile was weighed at all, 4 with them), fp32 input
// gradients 0.5 % (1.1 %), fp32 forwards 0.2 %.
constexpr double kBwRamp = 8.0, kBwRampSmall = 4.0, kSmallStep = 0.9;  // weight gradient; its 64 x 64 tile (and that tile's step)
constexpr double kBdRampF32 = 1.0, kFwdRampF32 = 0.5;

// Tuning override: QLAYER_<NAME>=<int> replaces a planner choice (for sweeps).
inline int env_override(const char *name, int dflt) {
    const char *v = std::getenv(name);
    if (!v || !*v) return dflt;
    return std::atoi(v);
}

inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }
inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline int cdiv(long long a, long long b) { return (int)((a + b - 1) / b); }

struct Geom {
    int N, C, H, W, O, KH, KW, SH, SW, PH, PW, HO, WO;
    ql_dtype dt;
    int ne;  // neuron type (NEURON_*)
    bool dw; // depthwise (groups == C == O)
    int om() const { return om_of_neuron(ne); }
    int terms() const { return om_terms(om()); }
    size_t esize() const { return dt == QL_BF16 ? 2 : 4; }
    int vec() const { return dt == QL_BF16 ? 8 : 4; }
    // Channel counts that are not a multiple of the 16-byte vector: the tensors
    // that the pipelined kernels read in 16-byte vectors along those channels
    // are copied zero-padded to whole vectors (cpad() input, opad() output
    // channels), where the copies stay within the 32-bit element offsets.  The
    // register-staged kernels that take such rows as they are load one element
    // at a time.  us per pass (fwd, input gradient, weight gradient), as they
    // are against padded, the copies included: 50 x 27 x 27 maps, 60 -> 100
    // channels, 3 x 3, bf16 197, 368, 318 against 40, 66, 54; a dense layer of
    // 128 rows, 512 -> 10, bf16 10, 12, 30 against 10, 8, 10; 32 x 28 x 28
    // maps, 51 -> 51 channels, 3 x 3, fp32 89, 113, 104 against 72, 74, 80.
    // Not for layers of a few million flops and less, where a pass is about the
    // launches and the copy is one more (a dense layer of 4 rows, 16 -> 73,
    // called from Python: 38 us for the three passes as it is, 45 padded); few
    // input channels (below two vectors) are always padded in the forward, as one
    // copied vector per pixel and tap is what the pipelined kernels need there.
    int cpad() const { return (C + vec() - 1) / vec() * vec(); }
    int opad() const { return (O + vec() - 1) / vec() * vec(); }
    double flops() const { return 2.0 * terms() * N * HO * WO * KH * KW * (double)C * O; }  // of a pass
    bool pad_pays() const { return 6.0 * N * HO * WO * KH * KW * (double)C * O >= 2e6; }  // (counted at three terms)
    bool few_c() const { return C < 2 * vec(); }
    bool pad_c_fits() const {
        return C % vec() != 0 && (long long)N * H * W * cpad() <= kMaxElems && 3LL * O * KH * KW * cpad() <= kMaxElems;
    }
    bool pad_o_fits() const {
        return O % vec() != 0 && (long long)N * HO * WO * opad() <= kMaxElems && 3LL * C * KH * KW * opad() <= kMaxElems;
    }
    // Bytes of the copies: of X, and of the neuron's output-side maps (G, T_a, T_b).
    size_t pad_x_bytes() const { return (size_t)N * H * W * cpad() * esize(); }
    size_t pad_maps_bytes() const { return om_gmaps(om()) * ((size_t)N * HO * WO * opad() * esize()); }
    // Where the filter reads less than a tenth of the pixels that the copy of X
    // moves: not if the copy is large and the layer's work is not (1 x 1 / 4,
    // 227 x 60 x 60 maps, 204 -> 116, bf16: forward 112 us as it is, 171 padded).
    bool pad_x_skips() const {
        const double bytes = (double)pad_x_bytes();
        return 10.0 * KH * KW * HO * WO < (double)H * W && bytes > 3e7 && flops() < 64 * bytes;
    }
    // The passes' lines, from 5000 layers of random sizes timed both ways (for each
    // line the geometric mean of time as it is over time padded, below and above).
    // Forward: a reduction of one K step of the pipelined kernels onto 16
    // channels or fewer is as fast in the register-staged kernel (175 x 22 x 22, 25 -> 6,
    // 1 x 1, bf16: 13.5 us, 14.5 padded).  The types with fewer matrix products
    // gain less from the fp32 pipeline: only a reduction of 48 to 256, or 1 GFLOP
    // (0.76 up to 48, 1.0 to 1.15 up to 256, 0.96 above; 1.35 from 1 GFLOP).
    bool pad_fwd() const {
        if (!pad_c_fits() || few_c()) return pad_c_fits();
        if (!pad_pays() || pad_x_skips()) return false;
        const int K = KH * KW * C;
        if (dt == QL_BF16 || ne == NEURON_QUADRA) return K > 64 / (int)esize() || O > 16;
        return flops() >= 1e9 || (K > 48 && K <= 256);
    }
    // Input gradient: where the reduction over the output channels is a step or
    // two, the copies cost what they save on all but the proposed neuron in
    // bf16 (dense 1612 x 308 -> 10, T2, fp32: 8.3 us, 12.7 padded; 104 x 35 x 35, 48 -> 14, 1 x 1 / 2,
    // fp32: 26.5, 36.5; bf16, other types, 0.91 to 1.0 below, 1.8 above; fp32, proposed
    // neuron, 0.89 to 1.08 and 1.3 to 2; other types 0.73 to 0.93 and 1.0 to 1.55).
    bool pad_bwd_data() const {
        if (!pad_o_fits() || !pad_pays()) return false;
        const bool s1 = SH == 1 && SW == 1;
        const int K = KH * KW * O;
        const long long px = (long long)N * H * W;
        const double bytes = (double)pad_maps_bytes();
        if (pad_maps_bytes() > kMaxPadBytes) return false;
        if (dt == QL_BF16)
            return ne == NEURON_QUADRA || K > 40 || flops() >= 5e7 || (C <= 64 && (!s1 || px >= 4096));
        if (ne == NEURON_QUADRA) return C <= 32 || (!(K <= 48 && bytes > 3.3e5 && s1) && !(K <= 16 && bytes > 3e6));
        return K > 40 && (flops() >= 1e9 || !s1 || px >= 2048 || C <= 64);
    }
    // Weight gradient: the fp32 pipelined kernels gain little over the
    // register-staged one and take a copy and a reduction more, so in fp32 only
    // from 0.3 GFLOP or 20000 pixels (64 -> 5, 8 x 6 x 6 maps, 3 x 3: 10.5 us as it is, 15.6
    // padded; 0.68 to 0.94 below, 1.05 to 1.45 above), the narrow kernel from 32 MFLOP
    // (0.84 to 1.05 and 0.98 to 3.7).
    bool pad_bwd_weight(bool narrow) const {
        if (!(C % vec() == 0 || pad_c_fits()) || !(O % vec() == 0 || pad_o_fits())) return false;
        const bool offc = C % vec() != 0, offo = O % vec() != 0;
        if (!offc && !offo) return false;
        if (offo || !few_c()) {
            if (!pad_pays() || (offc && pad_x_skips())) return false;
            if ((offc ? pad_x_bytes() : 0) + (offo ? pad_maps_bytes() : 0) > kMaxPadBytes) return false;
        }
        if (dt == QL_BF16 || (narrow && offc && few_c() && !offo)) return true;
        return flops() >= (narrow ? 3.2e7 : 3e8) || (long long)N * HO * WO >= 20000;
    }
};

// Length of a K step in the split model's units (see kReduceSteps).
inline double step_scale(const Geom &g) { return g.dt == QL_F32 ? g.terms() : 1.0; }

inline ql_status make_geom(const ql_conv_desc *d, Geom &g) {
    if (!d) return QL_EINVAL;
    if (d->n <= 0 || d->c <= 0 || d->h <= 0 || d->w <= 0 || d->o <= 0 || d->kh <= 0 || d->kw <= 0)
        return QL_EINVAL;
    if (d->stride_h < 1 || d->stride_w < 1 || d->pad_h < 0 || d->pad_w < 0) return QL_EINVAL;
    if (d->dtype != QL_F32 && d->dtype != QL_BF16) return QL_EINVAL;
    if ((int)d->neuron < NEURON_QUADRA || (int)d->neuron > NEURON_T24) return QL_EINVAL;
    const long long eh = (long long)d->h + 2LL * d->pad_h - d->kh;
    const long long ew = (long long)d->w + 2LL * d->pad_w - d->kw;
    if (eh < 0 || ew < 0) return QL_EINVAL;  // empty output
    g.N = d->n; g.C = d->c; g.H = d->h; g.W = d->w; g.O = d->o; g.KH = d->kh; g.KW = d->kw;
    g.SH = d->stride_h; g.SW = d->stride_w; g.PH = d->pad_h; g.PW = d->pad_w;
    g.HO = (int)(eh / d->stride_h + 1);
    g.WO = (int)(ew / d->stride_w + 1);
    g.dt = d->dtype;
    g.ne = (int)d->neuron;
    if (d->groups != 0 && d->groups != 1 && d->groups != d->c) return QL_EUNSUPPORTED;
    g.dw = d->groups == d->c && d->c > 1;
    if (g.dw && d->o != d->c) return QL_EINVAL;  // one output channel per group
    if (g.dw && 3LL * d->kh * d->kw * kDwCB * 4 > 64 * 1024) return QL_EUNSUPPORTED;  // filters staged in LDS
    if (g.dw && g.ne == NEURON_T24) return QL_EUNSUPPORTED;  // (the depthwise kernels cover types 0-4)
    // the shortcut of T4 + identity adds input channel o at the same pixel
    if (g.ne == NEURON_T4I && (g.C != g.O || g.HO != g.H || g.WO != g.W)) return QL_EINVAL;
    const long long nx = (long long)g.N * g.H * g.W * g.C;
    const long long ny = (long long)g.N * g.HO * g.WO * g.O;
    const long long nw = (long long)g.O * g.KH * g.KW * g.C;
    if (nx > kMaxElems || ny > kMaxElems || 3 * nw > kMaxElems || g.H + 2LL * g.PH > kMaxElems ||
        g.W + 2LL * g.PW > kMaxElems)
        return QL_EUNSUPPORTED;
    return QL_OK;
}

inline ql_status linear_geom(const ql_linear_desc *d, Geom &g) {
    if (!d) return QL_EINVAL;
    ql_conv_desc c{d->batch, d->in, 1, 1, d->out, 1, 1, 1, 1, 0, 0, d->dtype, d->neuron, 1};
    return make_geom(&c, g);
}

// Split-K planning.  The workgroups run in rounds of kNumCUs * slots (slots =
// workgroups one CU can hold at once); the split count minimises the modelled
// time: K steps per split times the rounds' cost, plus the traffic of the
// partial sums and the reduction.  A count that leaves a few CUs with a second
// workgroup in the last round costs a whole shared round, which the search
// avoids.  At least min_stages K steps per split, at most kMaxSplitBytes of
// partial sums (bytes_per_split each).  Returns the modelled time, a ramp of
// `ramp` steps per round added.
inline double plan_splits(int tiles, int stages_total, int min_stages, size_t bytes_per_split, int slots, int &splits,
                          int &sps, double step_scale, size_t max_bytes = kMaxSplitBytes, int pipes = 1,
                          double shared_round = kSharedRound, double step_cost = 1.0, double ramp = 0.0) {
    const int cap_bytes = (int)std::max<size_t>(1, max_bytes / std::max<size_t>(bytes_per_split, 1));
    const int s_max = std::max(1, std::min(stages_total / std::max(min_stages, 1), cap_bytes));
    double best = 0.0, cost = 0.0;
    splits = 1;
    // Each partition once, by its K steps per split: cdiv(stages_total, per - 1) is
    // the next count whose splits are shorter (at most 2 sqrt(stages_total) of
    // them; the callers plan on every call).
    for (int s = 1, per = stages_total; s <= s_max; s = cdiv(stages_total, per - 1)) {
        per = cdiv(stages_total, s);
        const int eff = s;
        const long long wgs = (long long)tiles * eff;
        const long long round = (long long)kNumCUs * std::max(slots, 1);
        const long long full = wgs / round, rest = wgs % round;
        double rounds = (double)full * (slots > 1 ? shared_round : 1.0);
        if (rest > 0) rounds += rest > kNumCUs ? shared_round : 1.0;
        double t = per * rounds * step_cost;
        if (pipes > 1) {
            rounds = (double)(full + (rest > 0));
            t = (double)cdiv(per, pipes) * rounds * kPipeRound;
        }
        if (eff > 1) t += ((double)eff * bytes_per_split * 2.0 / kBytesPerStep + kReduceSteps) / step_scale;
        if (s == 1 || t < best) {
            best = t;
            cost = t + ramp * rounds;
            splits = eff;
        }
        if (per == 1) break;
    }
    sps = cdiv(stages_total, splits);
    splits = cdiv(stages_total, sps);
    return cost;
}

// Taps (r, q) in bounds for output position pos = (oh, ow): a bit mask.
inline uint32_t tap_mask(const Geom &g, int pos) {
    const int oh = pos / g.WO, ow = pos % g.WO;
    const int h0 = oh * g.SH - g.PH, w0 = ow * g.SW - g.PW;
    uint32_t m = 0;
    for (int r = 0; r < g.KH; ++r)
        for (int q = 0; q < g.KW; ++q)
            if (h0 + r >= 0 && h0 + r < g.H && w0 + q >= 0 && w0 + q < g.W) m |= 1u << (r * g.KW + q);
    return m;
}

// Position-major pixel order (column m = position m / N of image m % N): the
// most in-bounds taps of any pixel tile of `bcol` columns (the union over
// the positions it spans).
inline int pm_max_taps(const Geom &g, int bcol, long long M) {
    int best = 0;
    for (long long m0 = 0; m0 < M; m0 += bcol) {
        const long long m1 = std::min(M, m0 + bcol) - 1;
        uint32_t u = 0;
        for (long long pos = m0 / g.N; pos <= m1 / g.N; ++pos) u |= tap_mask(g, (int)pos);
        best = std::max(best, __builtin_popcount(u));
    }
    return best;
}

// Whether to use the position-major order: forced by `env` (0 / 1), else on
// padded maps of at most 4 positions (2 x 2 maps of a 3 x 3 filter: every
// position has 4 taps in bounds).  Measured on larger maps (4 x 4, 8 x 8),
// the order is slower: the interior positions keep every tap, so their tiles
// bound the kernel's time, and a tile of one position no longer re-reads the
// X rows its neighbouring pixels share across taps from the caches.
inline bool pm_default(const Geom &g, int env) {
    if (env >= 0) return env != 0;
    return g.HO * g.WO <= 4 && (g.PH > 0 || g.PW > 0);
}

// Input gradient at stride 1: the taps (r, q) whose output pixel
// (h + PH - r, w + PW - q) lies in the map, for input position pos = h W + w.
inline uint32_t bd_tap_mask(const Geom &g, int pos) {
    const int h = pos / g.W, w = pos % g.W;
    uint32_t u = 0;
    for (int r = 0; r < g.KH; ++r)
        for (int q = 0; q < g.KW; ++q)
            if (h + g.PH - r >= 0 && h + g.PH - r < g.HO && w + g.PW - q >= 0 && w + g.PW - q < g.WO)
                u |= 1u << (r * g.KW + q);
    return u;
}

// The most taps any pixel tile of bcol position-major columns keeps.
inline int bd_pm_max_taps(const Geom &g, int bcol, long long M) {
    int best = 0;
    for (long long m0 = 0; m0 < M; m0 += bcol) {
        const long long m1 = std::min(M, m0 + bcol) - 1;
        uint32_t u = 0;
        for (long long pos = m0 / g.N; pos <= m1 / g.N; ++pos) u |= bd_tap_mask(g, (int)pos);
        best = std::max(best, __builtin_popcount(u));
    }
    return best;
}

// ---------------------------------------------------------------------------
// Forward planning.
// ---------------------------------------------------------------------------
// Pipelined forward tile configurations (rows = output channels per term,
// columns = output pixels; per-wave tile in parentheses; 4 waves unless noted):
//   0: 128 x 128 (32 x 128), 1: 64 x 256 (32 x 128), 2: 128 x 128 (64 x 64), 3: 64 x 128 (32 x 64),
//   4: 128 x 256 (32 x 128, 8 waves), 5: 128 x 256 (64 x 64, 8 waves), 6: as 4 with four LDS stages,
//   7: 32 x 128 (32 x 32).
// Larger workgroup tiles move fewer bytes through the vector-memory address
// path per MFMA: 32768 (1/BCOL + 1/(3 BR)) bytes.
constexpr int kFwdCfgs = 8;
constexpr int kFwdBR[kFwdCfgs] = {128, 64, 128, 64, 128, 128, 128, 32};
constexpr int kFwdBCOL[kFwdCfgs] = {128, 256, 128, 128, 256, 256, 256, 128};
// Workgroups one CU holds at once (limited by LDS stages and registers).
constexpr int kFwdSlots[kFwdCfgs] = {1, 1, 1, 2, 1, 1, 1, 2};

// Images that one launch of a narrow kernel addresses: its buffer loads take 32-bit
// byte offsets, with those from 2^31 on meaning "zero".  Larger layers are launched
// in equal groups of that many images; 0 where a single image is too large (the
// tiled kernels, whose addresses have 64 bits, take such a layer).
inline int narrow_images(const Geom &g, int C, int O) {
    const long long image = std::max((long long)g.H * g.W * C, (long long)g.HO * g.WO * O) * (long long)g.esize();
    const long long most = std::min<long long>(g.N, env_override("QLAYER_NARROW_BYTES", 0x7fffffff) / image);
    return most > 0 ? cdiv(g.N, cdiv(g.N, most)) : 0;
}

// Waves of the narrow kernels (a multiple of the four per workgroup): one per
// 16-pixel block up to three per SIMD, then more blocks per wave.
inline int narrow_waves(long long pixels) {
    const long long waves = std::min<long long>(std::max<long long>(1, cdiv(pixels, 16)), 3LL * 4 * kNumCUs);
    return (int)(cdiv(waves, 4) * 4);
}

// A K step of a tile configuration relative to the 64 x 128 tile's, for the
// split model: in fp32 the MFMAs bound a step, in bf16 its copies and their
// latency do, so a smaller tile saves less there.
constexpr double kFwdStepBf16[kFwdCfgs] = {1.0, 1.0, 1.0, 1.0, 1.0, 1.0, 1.0, 0.85};
constexpr double kFwdStepF32[kFwdCfgs] = {1.0, 1.0, 1.0, 1.0, 1.0, 1.0, 1.0, 0.55};

struct FwdPlan {
    int cfg;  // pipelined: index into kFwd*; generic: 0: 128 x 128, 1: 64 x 128
    int BR, BCOL, KE, slots;
    int row_tiles, col_tiles, splits, sps, stages_total;
    bool veck;
    bool smallc;  // KH KW C + bias columns <= 32, 32 or 64 output channels: qconv_fwd_smallc_kernel, no workspace
    bool narrow;  // at most 16 output channels, short J: qconv_fwd_narrow_kernel (OB row blocks, NCH chunks)
    int ob, nch, ni;  // ... NI images per launch
    bool ksplit;  // small outputs: qconv_fwd_ksplit_kernel (tiles of 3 x 16 krb rows by 16 kcb pixels, K split by waves)
    int krb, kcb;
    int stat_parts;  // partial sums of the epilogue statistics the kernel writes (fused path)
    bool ca;  // channel-aligned K steps (C a multiple of KE, at most 32 taps): every step within one tap
    bool pm;  // position-major pixel order, K steps of padding-only taps skipped (FwdArgs)
    bool pad;                      // X and W_t zero-padded to Cp channels first
    int Cp;
    size_t xpad_bytes, wpad_bytes;  // workspace: [X padded][W_a, W_b, W_c padded][split partials][X o X]
    size_t part_bytes;
    size_t xsq_bytes;               // T2 with 16-byte channel vectors: X o X formed once by a pre-pass
    size_t ws_bytes;
};

inline FwdPlan plan_fwd(const Geom &g) {
    FwdPlan p{};
    const int bias_cols = g.dt == QL_BF16 ? smallc_bias_cols<uint16_t>() : smallc_bias_cols<float>();
    if (g.ne == NEURON_QUADRA && g.C * g.KH * g.KW + bias_cols <= kSmallcK && (g.O == 32 || g.O == 64) &&
        env_override("QLAYER_FWD_SMALLC", 1) != 0) {
        p.smallc = true;
        p.splits = 1;
        return p;
    }
    p.pad = g.pad_fwd();
    p.Cp = p.pad ? g.cpad() : g.C;
    const int M = g.N * g.HO * g.WO, K = g.KH * g.KW * p.Cp;
    p.veck = p.Cp % g.vec() == 0;
    if (p.pad) {
        p.xpad_bytes = align_up((size_t)g.N * g.H * g.W * p.Cp * g.esize());
        p.wpad_bytes = align_up((size_t)g.O * g.KH * g.KW * p.Cp * g.esize());
    }
    // Narrow layers: the weight fragments of all three terms (3 OB NCH runs of
    // 16 bytes per lane) stay in registers for the whole kernel.
    p.ob = cdiv(g.O, 16);
    p.nch = cdiv(K, 4 * g.vec());
    // (one 16-channel row block: two measured slower than the tiled kernel on the
    // 16 -> 32-channel stride-2 layer of a CIFAR ResNet)
    if (p.veck && g.ne == NEURON_QUADRA && g.O % 4 == 0 && p.ob == 1 && p.nch <= 9 &&
        narrow_images(g, p.Cp, g.O) > 0 && env_override("QLAYER_FWD_NARROW", 1) != 0) {
        p.narrow = true;
        p.splits = 1;
        p.KE = 64 / (int)g.esize();
        p.ni = narrow_images(g, p.Cp, g.O);
        for (int n = 0; n < g.N; n += p.ni) p.stat_parts += narrow_waves((long long)std::min(p.ni, g.N - n) * g.HO * g.WO);
        p.ws_bytes = p.xpad_bytes + 3 * p.wpad_bytes;
        return p;
    }
    const int cfg_env = env_override("QLAYER_FWD_CFG", -1), min_stages = env_override("QLAYER_FWD_MINSTAGES", 4);
    if (p.veck) {
        // 8-wave 128 x 256 tiles where there are enough of them to fill the GPU several times,
        // else the 64 x 128 or the 32 x 128 tile by the split model (below)
        const bool big = g.O >= 128 && (long long)cdiv(g.O, 128) * cdiv(M, 256) >= 4 * kNumCUs;
        // (the 8-wave tile with four stages where the filter has several taps: measured 3 % faster on
        // the N=64, 256-channel 56 x 56 layer, and no faster on the dense layer)
        p.cfg = cfg_env >= 0 ? cfg_env : (big ? (g.KH * g.KW > 1 ? 6 : 4) : 3);
        if (p.cfg < 0 || p.cfg >= kFwdCfgs || g.ne != NEURON_QUADRA) p.cfg = 3;  // (the other types: tile 3 only)
        p.BR = kFwdBR[p.cfg];
        p.BCOL = kFwdBCOL[p.cfg];
        p.slots = kFwdSlots[p.cfg];
    } else {
        p.cfg = g.O <= 64 || g.ne != NEURON_QUADRA ? 1 : 0;
        p.BR = p.cfg == 0 ? 128 : 64;
        p.BCOL = 128;
        p.slots = 1;
    }
    p.KE = 64 / (int)g.esize();
    p.row_tiles = cdiv(g.O, p.BR);
    p.col_tiles = cdiv(M, p.BCOL);
    p.stat_parts = p.col_tiles;
    p.stages_total = cdiv(K, p.KE);
    // Position-major order where the maps are small, so that many taps of a
    // position lie in the padding: the splits are planned for the pixel tile
    // with the most in-bounds taps.  It needs channel-aligned K steps.  Without
    // it they are on by default in fp32 only: in bf16 they measured slower than
    // the per-lane (r, q, c) addresses (the VGG-16 and CIFAR ResNet layers with
    // 32 to 512 channels and the 256-channel 56 x 56 layer, 2 to 20 %), in fp32
    // 2 to 3 % faster (the ResNet layers with 32 and 64 channels).
    const int ca_env = env_override("QLAYER_FWD_CA", -1);
    const bool pm_want = pm_default(g, env_override("QLAYER_FWD_POSMAJ", -1));
    p.ca = p.veck && p.Cp % p.KE == 0 && g.KH * g.KW <= 32 &&
           (ca_env >= 0 ? ca_env != 0 : (pm_want || g.dt == QL_F32));
    p.pm = p.ca && pm_want;
    int kst = p.stages_total;
    if (p.pm) kst = pm_max_taps(g, p.BCOL, M) * (p.Cp / p.KE);
    auto fill = [&](int cfg) {
        p.cfg = cfg;
        p.BR = kFwdBR[cfg];
        p.BCOL = kFwdBCOL[cfg];
        p.slots = kFwdSlots[cfg];
        p.row_tiles = cdiv(g.O, p.BR);
        p.col_tiles = cdiv(M, p.BCOL);
        p.stat_parts = p.col_tiles;
        return plan_splits(p.row_tiles * p.col_tiles, kst, min_stages, (size_t)3 * M * g.O * 4, p.slots, p.splits,
                           p.sps, step_scale(g), kMaxSplitBytes, 1, kSharedRoundFwd,
                           (g.dt == QL_F32 ? kFwdStepF32 : kFwdStepBf16)[cfg], g.dt == QL_F32 ? kFwdRampF32 : 0.0);
    };
    // The 32-row tile where it leaves fewer empty rows or, on small outputs, fewer
    // idle CUs.  us per call (64-row against 32-row): 32 -> 32 channels, 256 x 16 x
    // 16 maps, 3 x 3, fp32 67 against 39, bf16 14.9 against 12.3; 96 -> 96, 128 x 14 x 14,
    // fp32 165 against 121, bf16 25.5 against 29.4; 64 -> 64, 256 x 8 x 8, bf16 14.1
    // against 12.5.  (BCOL is the same, so kst holds for both.)
    if (p.veck && p.cfg == 3 && g.ne == NEURON_QUADRA && cfg_env < 0) {
        const double t7 = fill(7), t3 = fill(3);
        if (t7 < t3) fill(7);
    } else if (p.veck) {
        fill(p.cfg);
    } else {
        plan_splits(p.row_tiles * p.col_tiles, kst, min_stages, (size_t)3 * M * g.O * 4, p.slots, p.splits, p.sps,
                    step_scale(g), kMaxSplitBytes, 1, kSharedRoundFwd);
    }
    // Where these tiles would split K over workgroups (small outputs: the 4 x 4
    // and 2 x 2 maps of a CIFAR VGG-16), the in-workgroup K split of
    // qconv_fwd_ksplit.h instead: tiles small enough to fill the GPU, no
    // partial sums in HBM.  (32-bit byte offsets into X and the weights.)
    // By default only where each wave's K range is at most 768 in bf16 (on
    // longer K the tiled kernel's split-K measured faster: the 512-channel
    // 4 x 4 layers, 1152 per wave, 52 against 47 us per call), 1152 in fp32
    // (the longest measured: the same layers, 215 against 228 us).  In bf16 up to
    // 1024 where there are at most 80 of the 64 x 128 tiles, whether or not they
    // would split (448 -> 256 channels, 3 x 9 x 9 maps, 3 x 3: 24.1 us tiled, 14.3 here;
    // a dense layer of 1024 rows, 512 -> 512: 12.7, 9.5; 32 -> 64, 4 x 20 x 20: 9.7, 6.4).
    // Past one workgroup per CU only from 128 to 768 per wave (1 x 1, 2 x 49 x 49, 32 -> 128,
    // 304 of them: 7.1 us tiled, 8.2 here; dense 911 x 3488 -> 320, 300 of them: 27.3, 32.8;
    // by the size of the reduction, below 512, from 512 to 3072 and above, time here over time tiled
    // 1.03, 0.78 and 1.10 on 60 layers).
    // In fp32, whose tiles' MFMAs outweigh the split's traffic, above 320 per wave
    // only with at least 88 workgroups of its own (time here over time tiled on 90
    // layers of random sizes: 1.14 to 1.46 below, 0.91 above; 64 -> 544, 3 x 8 x 8, 5 x 5,
    // 102 of them: 27.1 us here, 36.0 tiled; 448 -> 256, 3 x 9 x 9, 3 x 3, 64 of them: 55.8, 39.4).
    const int ks_env = env_override("QLAYER_FWD_KSPLIT", -1);
    const int ks_k = (pm_want ? pm_max_taps(g, 64, M) : g.KH * g.KW) * p.Cp;
    auto ks_default = [&]() {
        if (p.cfg != 3 && p.cfg != 7) return false;
        if (g.dt == QL_F32)
            return p.splits > 1 && ks_k <= 4 * 1152 && (ks_k <= 4 * 320 || cdiv(g.O, 16) * cdiv(M, 64) >= 88);
        if (p.splits > 1 && ks_k <= 4 * 768) return true;
        const int wide = cdiv(g.O, 32) * cdiv(M, 64);  // workgroups (of the larger tile where they fill the GPU)
        const bool one_each = (wide >= kNumCUs ? wide : cdiv(g.O, 16) * cdiv(M, 64)) <= kNumCUs;
        return cfg_env < 0 && cdiv(g.O, 64) * cdiv(M, 128) <= 80 &&
               (one_each ? ks_k <= 4 * 1024 : ks_k >= 4 * 128 && ks_k <= 4 * 768);
    };
    if (p.veck && g.ne == NEURON_QUADRA && g.O % 4 == 0 && p.Cp % p.KE == 0 && g.KH * g.KW <= 32 &&
        (long long)g.N * g.H * g.W * p.Cp * (long long)g.esize() < (1LL << 31) &&
        (long long)g.O * K * (long long)g.esize() < (1LL << 31) &&
        (ks_env >= 0 ? ks_env != 0 : ks_default())) {
        // the larger tile where its count fills the GPU, else the smaller one (or as forced)
        constexpr int kKsRB[3] = {2, 1, 2}, kKsCB[3] = {4, 4, 2};
        int t = cdiv(g.O, 32) * cdiv(M, 64) >= kNumCUs ? 0 : 1;
        t = env_override("QLAYER_FWD_KSPLIT_TILE", t);
        if (t < 0 || t > 2) t = 1;
        p.ksplit = true;
        p.krb = kKsRB[t];
        p.kcb = kKsCB[t];
        p.pm = pm_want;
        p.row_tiles = cdiv(g.O, 16 * p.krb);
        p.col_tiles = cdiv(M, 16 * p.kcb);
        p.splits = 1;
        p.sps = p.stages_total;
        p.stat_parts = p.col_tiles * p.kcb;
        p.ws_bytes = p.xpad_bytes + 3 * p.wpad_bytes;
        return p;
    }
    p.part_bytes = p.splits > 1 ? align_up((size_t)p.splits * 3 * M * g.O * sizeof(float)) : 0;
    p.xsq_bytes = g.ne == NEURON_T2 && p.veck ? align_up((size_t)g.N * g.H * g.W * p.Cp * g.esize()) : 0;
    p.ws_bytes = p.xpad_bytes + 3 * p.wpad_bytes + p.part_bytes + p.xsq_bytes;
    return p;
}

// ---------------------------------------------------------------------------
// Input-gradient planning.  Workspace: transposed weights, then split partials.
// ---------------------------------------------------------------------------
// Pipelined input-gradient tile configurations (rows = input channels,
// columns = input pixels):  0: 128 x 128, 1: 64 x 128, 2: 128 x 64, 3: 128 x 128
// with the four waves side by side (each 128 x 32: half the prologue
// products per MFMA of configuration 0), 5: 64 x 128 with the waves side by
// side (each 64 x 32: half the products per MFMA of configuration 1).
// 6: 32 x 128, the waves side by side.
constexpr int kBdCfgs = 7;
constexpr int kBdBR[kBdCfgs] = {128, 64, 128, 128, 256, 64, 32};
constexpr int kBdBCOL[kBdCfgs] = {128, 128, 64, 128, 256, 128, 128};  // 4: the wide kernel (8 waves, 16-channel K steps)

// K steps relative to the 64 x 128 tile's (see kFwdStepBf16).
constexpr double kBdStepBf16[kBdCfgs] = {1.3, 1.0, 1.0, 1.3, 1.0, 1.0, 0.9};
constexpr double kBdStepF32[kBdCfgs] = {2.0, 1.0, 1.0, 1.9, 1.0, 1.0, 0.6};

struct BwdDataPlan {
    int cfg;  // pipelined: index into kBd*; generic: 0: 128 x 128, 1: 64 x 128
    int BR, BCOL, KE, slots;  // slots: one workgroup per CU (the LDS ring takes 144 KB)
    int row_tiles, col_tiles, splits, sps, stages_total;
    bool veck, s1;
    bool natw;    // weights read untransposed through natural LDS tiles (bf16, C % 8 == 0)
    bool smallc;  // C <= 4: per-pixel partial sums by MFMA, then a gather over the taps
    bool narrow;  // at most 16 input channels, short K: qconv_bwd_data_narrow_kernel (CB row blocks, NCH chunks)
    int cb, nch, ni;  // ... NI images per launch
    bool ca, pm;  // channel-aligned K steps; position-major order with taps skipped (BwdDataArgs)
    int order;  // block order of the split-K grid (tile_coord)
    int fused_rb; // ... stride 1: both steps in one kernel, bands of fused_rb input rows (0: two kernels)
    size_t fused_smem;
    int njb;      // ... 32-column blocks of (r, q, c)
    size_t smem;  // ... LDS of the weight fragments
    bool pad;     // G, T_a, T_b (and the transposed weights) zero-padded to Op output channels first
    int Op;
    size_t wt_bytes, gpad_bytes, part_bytes, ws_bytes;  // workspace: [weights][G, T_a, T_b padded][split partials]
};

// At stride > 1 the kernels split the input pixels into phases (BwdPhase), one
// per stride offset: the most taps and the most pixels of any phase.
inline void bwd_phase_extents(const Geom &g, int &taps, int &pixels) {
    taps = cdiv(g.KH, g.SH) * cdiv(g.KW, g.SW);
    pixels = g.N * cdiv(g.H, g.SH) * cdiv(g.W, g.SW);
}

// Whether a strided layer takes the phases: up to kMaxPhases, or one for each
// wave of the narrow kernel, always.  Past that where their tiles (at least one
// per phase, its ramp priced at four K steps) and K steps, spread over the CUs,
// take no longer than the register-staged kernel, in which every pixel meets
// every tap and a step takes about four times as long.  us per call in the
// register-staged kernel and by phases, bf16: 16 x 16 patches at stride 16, 32 x 224 x 224
// maps of 8 channels -> 768, 1190000 and 963; 3 x 3 at stride 100, 2 x 300 x 300, 64 ->
// 64, 513 and 72; 1 x 1 at stride 32, 4 x 128 x 128, 64 -> 64, 29 and 10.
inline bool bwd_phased(const Geom &g, int Op) {
    const long long P = (long long)g.SH * g.SW, M = (long long)g.N * g.H * g.W;
    if (P <= std::max(kMaxPhases, narrow_waves(M))) return true;
    int taps, pixels;
    bwd_phase_extents(g, taps, pixels);
    const long long tiles = cdiv(pixels, 128), whole = cdiv(M, 128);
    const long long steps = (long long)g.KH * g.KW * cdiv(Op, 64 / (int)g.esize());
    auto rounds = [](long long work) { return (work + kNumCUs - 1) / kNumCUs; };
    return P <= (1 << 20) / tiles &&
           4 * rounds(P * tiles) + rounds(tiles * steps) <= 4 * (4 * rounds(whole) + rounds(whole * steps));
}

inline BwdDataPlan plan_bwd_data(const Geom &g) {
    BwdDataPlan p{};
    {
        const int J = g.KH * g.KW * g.C;  // columns (r, q, c) of the partial sums
        p.njb = cdiv(J, 32);
        p.smem = (size_t)3 * p.njb * (g.O / (2 * g.vec())) * 64 * 16;
        p.smallc = g.C <= 4 && g.O % (2 * g.vec()) == 0 && p.njb <= 2 && p.smem <= 64 * 1024 &&
                   g.ne == NEURON_QUADRA && env_override("QLAYER_BWD_DATA_SMALLC", 1) != 0;
        if (p.smallc) {
            // fused (stride 1): LDS holds the weights and the partial sums of RB + KH - 1
            // output rows; at most 64 KB, so that two workgroups share a CU
            int rb = env_override("QLAYER_BWD_DATA_FUSED_RB", 8);  // (0: the two kernels)
            if (g.SH == 1 && g.SW == 1 && p.njb == 1 && rb > 0) {
                for (; rb >= 1; --rb) {
                    const size_t lds = p.smem + (size_t)(rb + g.KH - 1) * g.WO * kFusedPitch * sizeof(float);
                    if (lds <= 64 * 1024) {
                        p.fused_rb = rb;
                        p.fused_smem = lds;
                        break;
                    }
                }
            }
            p.ws_bytes = p.fused_rb ? 0 : align_up((size_t)g.N * g.HO * g.WO * J * sizeof(float));
            return p;
        }
    }
    p.s1 = g.SH == 1 && g.SW == 1;
    const bool phases = !p.s1 && bwd_phased(g, g.opad());
    p.pad = g.pad_bwd_data() && (p.s1 || phases);  // (the register-staged kernel takes the maps as they are)
    p.Op = p.pad ? g.opad() : g.O;
    if (p.pad) p.gpad_bytes = align_up((size_t)g.N * g.HO * g.WO * p.Op * g.esize());
    const size_t gpads = om_gmaps(g.om()) * p.gpad_bytes;
    const int M = g.N * g.H * g.W;
    int taps = g.KH * g.KW, phase_pixels = M;  // of one phase (stride 1: the whole map)
    if (phases) bwd_phase_extents(g, taps, phase_pixels);
    const int K = taps * p.Op;
    p.veck = p.Op % g.vec() == 0 && (p.s1 || phases);
    // Narrow layers: the transposed weight runs of all three terms stay in registers.
    p.cb = cdiv(g.C, 16);
    p.nch = cdiv(K, 4 * g.vec());
    if (p.veck && g.ne == NEURON_QUADRA && g.C % 4 == 0 && p.cb == 1 && p.nch <= 9 &&
        (p.s1 || (long long)g.SH * g.SW <= std::max(kMaxPhases, narrow_waves(M))) &&  // (a wave per phase)
        narrow_images(g, g.C, p.Op) > 0 && env_override("QLAYER_BWD_DATA_NARROW", 1) != 0) {
        p.narrow = true;
        p.ni = narrow_images(g, g.C, p.Op);
        p.splits = 1;
        p.wt_bytes = align_up(3 * (size_t)p.Op * g.KH * g.KW * g.C * g.esize());
        p.ws_bytes = p.wt_bytes + gpads;
        return p;
    }
    p.natw = p.veck && !p.pad && g.dt == QL_BF16 && g.C % 8 == 0;
    // the wide kernel: bf16, natural weight tiles, stride 1, 16-channel K steps within one tap
    const bool wide_ok = p.natw && p.s1 && g.O % 16 == 0 && g.KH * g.KW <= 32;
    // (measured: faster where its 256 x 256 tiles fill the GPU at least twice, as on
    // the dense layer and the N=64, 256-channel 56 x 56 layer; on the small maps of
    // VGG-16 the 4-wave tiles win, the wide kernel's 8 waves run their product
    // arithmetic in step)
    const bool wide = wide_ok && g.C >= 256 && (long long)cdiv(g.C, 256) * cdiv(M, 256) >= 2 * kNumCUs;
    const int cfg_env = env_override("QLAYER_BWD_DATA_CFG", -1);
    if (p.veck) {
        p.cfg = cfg_env >= 0 ? cfg_env : (wide ? 4 : (g.C > 64 ? 3 : 5));
        if (p.cfg >= kBdCfgs || (p.cfg == 4 && !wide_ok)) p.cfg = 0;
        if (g.ne != NEURON_QUADRA) p.cfg = g.C > 64 ? 3 : 5;  // (the other types: tiles 3 and 5 only)
    } else {
        p.cfg = g.C <= 64 || g.ne != NEURON_QUADRA ? 1 : 0;
        p.BR = p.cfg == 0 ? 128 : 64;
        p.BCOL = 128;
    }
    p.KE = p.cfg == 4 && p.veck ? 16 : 64 / (int)g.esize();
    p.slots = 1;
    // (register-staged kernel at stride > 1: every pixel meets every tap)
    const bool phased = p.veck && phases;
    p.stages_total = cdiv(p.veck ? K : g.KH * g.KW * p.Op, p.KE);
    // Channel-aligned K steps (each within one tap) in the 4-wave kernels, and
    // with them, on small padded maps, the position-major order that skips
    // the taps whose output pixel lies outside the map for every position of
    // a pixel tile (the proposed neuron: 5 of 9 taps on a 2 x 2 map).
    const bool ca_ok = p.natw && p.cfg != 4 && g.O % p.KE == 0 && g.KH * g.KW <= 32;
    const int ca_env = env_override("QLAYER_BWD_DATA_CA", -1);
    p.pm = ca_ok && ca_env != 0 && p.s1 && g.ne == NEURON_QUADRA &&
           pm_default(g, env_override("QLAYER_BWD_DATA_POSMAJ", -1));
    const int min_stages = env_override("QLAYER_BWD_DATA_MINSTAGES", 4);
    auto fill = [&](int cfg) {
        p.cfg = cfg;
        if (p.veck) {
            p.BR = kBdBR[cfg];
            p.BCOL = kBdBCOL[cfg];
        }
        p.row_tiles = cdiv(g.C, p.BR);
        p.col_tiles = phased ? g.SH * g.SW * cdiv(phase_pixels, p.BCOL) : cdiv(M, p.BCOL);
        int kst = p.stages_total;
        if (p.pm) kst = bd_pm_max_taps(g, p.BCOL, M) * (g.O / p.KE);
        return plan_splits(p.row_tiles * p.col_tiles, kst, min_stages, (size_t)M * g.C * 4, p.slots, p.splits, p.sps,
                           step_scale(g), kMaxSplitBytes, 1, kSharedRound,
                           p.veck ? (g.dt == QL_F32 ? kBdStepF32 : kBdStepBf16)[cfg] : 1.0,
                           g.dt == QL_F32 ? kBdRampF32 : 0.0);
    };
    // The tile by the split model: smaller tiles where they leave fewer empty rows
    // or idle CUs.  us per call: 128 -> 128 channels, 32 x 14 x 14 maps, 1 x 1, bf16 8.8
    // in 128 x 128 tiles, 7.0 in 128 x 64, fp32 26.0, 16.2 in 32 x 128; 272 -> 16, 8 x 14 x
    // 14, 3 x 3, bf16 10.0, 7.0 in 32 x 128; 32 -> 32, 256 x 16 x 16, 3 x 3, fp32 81 in 64 x
    // 128, 52 in 32 x 128, bf16 22.6, 20.2.
    double best = fill(p.cfg);
    if (p.veck && p.cfg != 4 && g.ne == NEURON_QUADRA && cfg_env < 0) {
        int pick = p.cfg;
        for (int cfg : {3, 2, 5, 6}) {
            if (g.C <= 64 && cfg < 5) continue;  // (128-row tiles: half empty)
            // (maps of four pixels: 416 -> 64 channels, 209 x 2 x 2, 5 x 5, 14.5 us in 128 x 64, 17.5 in 32 x 128)
            if (g.C > 64 && cfg >= 5 && p.pm) continue;
            const double t = fill(cfg);
            if (t < best) {
                best = t;
                pick = cfg;
            }
        }
        fill(pick);
    }
    // The 64- and 32-row tiles keep the per-lane addresses, which interleave with
    // the MFMAs (64 -> 64 channels, 3 x 3, bf16: 128 x 32 x 32 maps 65.7 against 70.4 us
    // with channel-aligned steps, 256 x 8 x 8 maps 16.3 against 18.3).
    p.ca = ca_ok && ca_env != 0 && (p.pm || ca_env == 1 || (p.cfg != 5 && p.cfg != 6));
    // Block order of the split grid: tile-major (each XCD's blocks share pixel
    // tiles: their rows of G, T_a, T_b once, all of the weights) where G, T_a,
    // T_b are at least the weight bytes (M >= C KH KW), split-major otherwise
    // (each XCD reads its K range of the weights and all of G, T_a, T_b).
    // Measured on the VGG-16 layers at batch 128 (bitwise the same results in
    // every order): the 128 -> 256 8 x 8 layer reads 44 instead of 115 MB per
    // call from beyond the L2s and runs 34.0 -> 33.1 us; on the 4 x 4 layers
    // tile-major read twice the bytes (142 against 72 MB per call on 512 ->
    // 512) for at most 1 us, and on the 2 x 2 layers it was 1 us slower.
    {
        const int dflt = (long long)M >= (long long)g.C * g.KH * g.KW ? 1 : 0;
        p.order = p.splits > 1 ? env_override("QLAYER_BWD_DATA_ORDER", dflt) : 0;
        if (p.order < 0 || p.order > 2) p.order = 0;
    }
    p.wt_bytes = p.natw ? 0 : align_up(3 * (size_t)p.Op * g.KH * g.KW * g.C * g.esize());
    p.part_bytes = p.splits > 1 ? align_up((size_t)p.splits * M * g.C * sizeof(float)) : 0;
    p.ws_bytes = p.wt_bytes + gpads + p.part_bytes;
    return p;
}

// ---------------------------------------------------------------------------
// Weight-gradient planning.  Workspace: dW partials, then db partials.
// ---------------------------------------------------------------------------
// Pipelined (bf16) weight-gradient tile configurations (rows = k', columns =
// output channels per term):  0: 128 x 64, 1: 128 x 128, 2: 64 x 64.
// (3: the 128 x 64 tile of the 16 x 16 x 32 kernel, qconv_bwd_weight16.h;
// 4: the same with two pipelines per 8-wave workgroup; 5: its 128 x 128 tile,
// eight waves side by side in one pipeline)
constexpr int kBwCfgs = 6;
constexpr int kBwBKP[kBwCfgs] = {128, 128, 64, 128, 128, 128};
constexpr int kBwBO[kBwCfgs] = {64, 128, 64, 64, 64, 128};
constexpr int kBwSlots[kBwCfgs] = {2, 1, 2, 2, 1, 1};  // workgroups one CU holds at once
constexpr int kBwThreads[kBwCfgs] = {256, 256, 256, 256, 512, 512};
constexpr int kBwPipes[kBwCfgs] = {1, 1, 1, 1, 2, 1};  // pipelines per workgroup (K halves)

struct BwdWeightPlan {
    bool narrow;  // KH KW C <= 144: qconv_bwd_weight_narrow_kernel (NF fragments, NOB 16-channel slices)
    bool few;     // a few-channel layer on the padded copy of X (refused where its scratch does not fit)
    int nf, nob, ni;  // ... NI images per launch
    int cfg;   // pipelined path only
    bool pipe; // bf16 and vectorizable: pipelined kernel; otherwise the generic one
    int BKP, BO, KE, slots;
    int row_tiles, col_tiles, splits, sps, stages_total;
    bool veck;
    bool padc, pado;  // X zero-padded to Cp, G, T_a, T_b to Op channels first (pipelined paths only)
    int Cp, Op;
    // workspace: [X padded][G, T_a, T_b padded][dW partials][db partials]
    size_t xpad_bytes, gpad_bytes, dw_bytes, db_bytes, ws_bytes;
    // splits of the narrow kernel's launch on the images from n on
    int narrow_splits(const Geom &g, int n) const {
        return cdiv(cdiv((long long)std::min(ni, g.N - n) * g.HO * g.WO, g.dt == QL_BF16 ? 32 : 16), sps);
    }
};

// max_split_bytes: cap on the dW partial sums (the no-allocation entry point
// plans for its fixed scratch array).  may_pad: whether channel counts off the
// 16-byte vector may take padded copies (else the register-staged kernel).
inline BwdWeightPlan plan_bwd_weight(const Geom &g, size_t max_split_bytes = kMaxSplitBytes, bool may_pad = true) {
    BwdWeightPlan p{};
    // the narrow kernel: rows k' of at most 144 (after the channel padding)
    const bool f32_pipe = g.ne == NEURON_QUADRA && env_override("QLAYER_BWD_WEIGHT_F32_PIPE", 1) != 0;
    may_pad = may_pad && (g.dt == QL_BF16 || f32_pipe);
    // (wider layers, up to 64 channels, in 16-channel slices, one per workgroup row of the
    // grid: by default in fp32, where the 16 -> 32-channel stride-2 CIFAR ResNet layer
    // measured 37 against 66 us per call; in bf16 it and the VGG-16 stem were no faster)
    const int narrow_max_o = env_override("QLAYER_BWD_WEIGHT_NARROW_MAXO", g.dt == QL_F32 ? 64 : 16);
    const size_t bytes_per_split = (size_t)3 * g.O * g.KH * g.KW * g.C * 4;
    const int most_splits = (int)std::min<size_t>(0x7fffffff, std::max<size_t>(1, max_split_bytes / bytes_per_split));
    auto narrow_dims = [&](int Cp, int Op) {
        const int ni = narrow_images(g, Cp, Op);
        return ni > 0 && cdiv(g.N, ni) <= most_splits && g.ne == NEURON_QUADRA &&
               (Op <= 16 || (Op % 16 == 0 && Op <= narrow_max_o)) && Cp % g.vec() == 0 && Op % g.vec() == 0 &&
               cdiv(g.KH * g.KW * Cp, 16) <= 9 &&
               env_override("QLAYER_BWD_WEIGHT_NARROW", 1) != 0;
    };
    const bool pad = may_pad && g.pad_bwd_weight(narrow_dims(g.cpad(), g.opad()));
    p.padc = pad && g.C % g.vec() != 0;
    p.pado = pad && g.O % g.vec() != 0;
    p.Cp = p.padc ? g.cpad() : g.C;
    p.Op = p.pado ? g.opad() : g.O;
    p.veck = p.Cp % g.vec() == 0 && p.Op % g.vec() == 0;
    const bool narrow_shape = narrow_dims(p.Cp, p.Op);
    const int M = g.N * g.HO * g.WO, KP = g.KH * g.KW * p.Cp, KPO = g.KH * g.KW * g.C;
    // pipelined kernels: bf16 every neuron type; fp32 the proposed neuron (the 16 x 16 kernel's fp32 form)
    p.pipe = p.veck && (g.dt == QL_BF16 || f32_pipe);
    if (p.padc) p.xpad_bytes = align_up((size_t)g.N * g.H * g.W * p.Cp * g.esize());
    if (p.pado) p.gpad_bytes = align_up((size_t)M * p.Op * g.esize());
    const size_t pads = p.xpad_bytes + om_gmaps(g.om()) * p.gpad_bytes;
    p.KE = 64 / (int)g.esize();
    p.stages_total = cdiv(M, p.KE);
    // At least two K steps per split (small outputs with few pixels leave most
    // CUs idle otherwise: 64 -> 64 channels, 8 x 8 x 8 maps, 3 x 3, in fp32 35 us
    // at a floor of 16, 18 at 4, 16 at 2; no change on the VGG-16 layers).  The
    // generic kernel's steps are latency-bound: down to one step each (the
    // 64 -> 10 head of a CIFAR ResNet at batch 256, 53 -> 17 us).
    const int min_stages = env_override("QLAYER_BWD_WEIGHT_MINSTAGES", p.pipe ? 2 : 1);
    // Narrow layers: the whole gradient of a 16-channel slice is one tile; about
    // one workgroup per CU in all down to one K step per wave, two per CU from
    // four steps per wave, the partial sums within max_split_bytes.  (16 -> 16
    // channels, 3 x 3, us at four steps per wave everywhere and now: 64 x 16 x 16
    // maps fp32 22.6 -> 17.8, bf16 18.6 -> 15.1; 16 x 8 x 8 maps fp32 22.4 -> 14.)
    // Below 16 splits the reduction adds them one after the other in each thread,
    // 2 us and 0.3 for each, which few steps do not pay for: there the count that
    // the measured step times make the fastest, one included.  (us at one step
    // per wave and now, bf16: 3 -> 16, 3 x 3, 4 x 9 x 9 maps 14.9, 13.2; 16 -> 16, 1 x 1,
    // 768 pixels 7.9, 6.7; 8 -> 8, 3 x 3, 1024 pixels 12.3, 11.4.)
    p.nf = cdiv(KP, 16);
    p.few = p.padc && !p.pado && g.C < 2 * g.vec() && (g.dt == QL_BF16 || narrow_shape);
    if (narrow_shape) {
        p.narrow = true;
        p.nob = cdiv(p.Op, 16);
        p.ni = narrow_images(g, p.Cp, p.Op);
        p.stages_total = cdiv((long long)p.ni * g.HO * g.WO, g.dt == QL_BF16 ? 32 : 16);  // of one launch
        int splits = std::max(cdiv(p.stages_total, 16), std::min(cdiv(kNumCUs, p.nob), cdiv(p.stages_total, 4)));
        splits = std::min(std::max(1, 2 * kNumCUs / p.nob), splits);
        if (splits < 16) {
            const double step = g.dt == QL_BF16 ? 0.1 * p.nf + 0.3 : 0.22 * p.nf + 0.25;  // us, one step of a wave
            double best = step * cdiv(p.stages_total, 4);
            const int most = splits;
            splits = 1;
            for (int s = 2; s <= most; ++s) {
                const double t = step * cdiv(p.stages_total, 4 * s) + 2.0 + 0.3 * s;
                if (t < best) {
                    best = t;
                    splits = s;
                }
            }
        }
        splits = env_override("QLAYER_BWD_WEIGHT_NARROW_SPLITS", splits);
        splits = std::max(1, std::min(splits, most_splits / cdiv(g.N, p.ni)));
        p.sps = cdiv(p.stages_total, splits);
        p.splits = 0;
        for (int n = 0; n < g.N; n += p.ni) p.splits += p.narrow_splits(g, n);
        if (p.splits > 1) {
            p.dw_bytes = align_up((size_t)p.splits * 3 * g.O * KPO * sizeof(float));
            p.db_bytes = align_up((size_t)p.splits * 3 * g.O * sizeof(float));
        }
        p.ws_bytes = pads + p.dw_bytes + p.db_bytes;
        return p;
    }
    auto fill = [&](int cfg) {
        p.cfg = cfg;
        p.BKP = p.pipe ? kBwBKP[cfg] : 128;
        p.BO = p.pipe ? kBwBO[cfg] : 64;
        p.slots = p.pipe ? kBwSlots[cfg] : 1;
        p.row_tiles = cdiv(KP, p.BKP);
        p.col_tiles = cdiv(g.O, p.BO);
        return plan_splits(p.row_tiles * p.col_tiles, p.stages_total, min_stages, bytes_per_split, p.slots, p.splits,
                           p.sps, step_scale(g), max_split_bytes, kBwPipes[cfg], kSharedRound, cfg == 5 ? kFatStep : cfg == 2 ? kSmallStep : 1.0, cfg == 2 ? kBwRampSmall : kBwRamp);
    };
    if (p.pipe && g.ne == NEURON_QUADRA) {
        // the 16 x 16 x 32 kernel: four waves on a 64-channel tile, two such pipelines per
        // workgroup, or eight waves on a 128-channel tile, whichever the model finds fastest
        const int forced = env_override("QLAYER_BWD_WEIGHT_CFG", -1);
        if (forced >= (g.dt == QL_BF16 ? 0 : 3) && forced < kBwCfgs) {  // (fp32: configurations 3-5 only)
            fill(forced);
        } else {
            // the 128-channel tile only where it has no empty columns
            const double t3 = fill(3), t4 = fill(4);  // (declarators initialise in order)
            const double t5 = g.O % 128 == 0 ? fill(5) : 1e30;
            int best = t5 < t3 && t5 < t4 ? 5 : (t4 < t3 ? 4 : 3);
            // the 64 x 64 tile of the 32 x 32 kernel on small outputs, where its ramp is
            // the shortest (32 -> 64 channels, 4 x 20 x 20 maps, 3 x 3: 11.1 against 13.9 us;
            // 256 -> 256, 2 x 4 x 4: 6.0 against 7.8)
            const double t2 = g.dt == QL_BF16 ? fill(2) : 1e30;
            if (t2 < std::min(t3, std::min(t4, t5))) best = 2;
            fill(best);
        }
    } else {
        fill(0);  // the other neuron types and fp32: the 128 x 64 tile
    }
    if (p.splits > 1) {
        p.dw_bytes = align_up((size_t)p.splits * 3 * g.O * KPO * sizeof(float));
        p.db_bytes = align_up((size_t)p.splits * 3 * g.O * sizeof(float));
    }
    p.ws_bytes = pads + p.dw_bytes + p.db_bytes;
    return p;
}

inline ql_status hip_status() {
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? QL_OK : QL_EHIP;
}

inline int grid_1d(long long total) {
    long long b = (total + kThreads - 1) / kThreads;
    return (int)std::max(1LL, std::min(b, 8LL * kNumCUs));
}

// One tensor of a zero-padding pass (qconv_pad_rows_kernel): `rows` rows of c
// channels of T into dst, padded to whole 16-byte vectors.
template <typename T>
inline void pad_segment(PadSegments &sg, int &n, const void *src, void *dst, long long rows, int c) {
    const int nv = cdiv(c, Elem<T>::VEC);
    sg.src[n] = src;
    sg.dst[n] = dst;
    sg.total[n] = (uint32_t)(rows * nv);
    sg.c[n] = c;
    sg.fd_nv[n] = make_fastdiv(nv);
    ++n;
}
template <typename T>
inline ql_status launch_pad(const PadSegments &sg, int n, hipStream_t st) {
    uint32_t most = 0;
    int c = sg.c[0];  // the channel count of every tensor, if they agree and it is below one vector
    for (int i = 0; i < n; ++i) {
        most = std::max(most, sg.total[i]);
        if (sg.c[i] != c || sg.c[i] >= Elem<T>::VEC) c = 0;
    }
    const dim3 grid(grid_1d(most), n), block(kThreads);
#define QL_PAD_SHORT(C)                                                                                   \
    case C:                                                                                               \
        if constexpr (C < Elem<T>::VEC) {                                                                 \
            hipLaunchKernelGGL((qconv_pad_short_rows_kernel<T, C>), grid, block, 0, st, sg);              \
            return hip_status();                                                                          \
        }                                                                                                 \
        break
    switch (c) {
        QL_PAD_SHORT(1);
        QL_PAD_SHORT(2);
        QL_PAD_SHORT(3);
        QL_PAD_SHORT(4);
        QL_PAD_SHORT(5);
        QL_PAD_SHORT(6);
        QL_PAD_SHORT(7);
        default: break;
    }
#undef QL_PAD_SHORT
    hipLaunchKernelGGL((qconv_pad_rows_kernel<T>), grid, block, 0, st, sg);
    return hip_status();
}

// ---------------------------------------------------------------------------
// Launch helpers, one per kernel family, dispatching the template instances.
// ---------------------------------------------------------------------------
// Whether launch_fwd's kernel writes Y through its staged epilogue, the path
// that gathers the epilogue statistics itself (qconv_fwd.h).
inline bool fwd_stats_fused(const Geom &g, const FwdPlan &p) {
    if (p.narrow || p.ksplit) return true;
    if (p.smallc || !p.veck || p.splits != 1 || g.O % (16 / (int)g.esize()) != 0) return false;
    const int ns = (g.ne == NEURON_QUADRA && (p.cfg == 4 || p.cfg == 5)) ? 3 : 4;
    return fwd_staged_fits(p.BR, p.BCOL, ns, (int)g.esize());
}

// ---------------------------------------------------------------------------
// Depthwise layers (groups == C == O): direct kernels of qconv_depthwise.h.
// 3 x 3 filters at stride 1 or 2 take the column kernels (the input gradient
// at stride 2 the gathering one); other shapes take the generic kernels.
// ---------------------------------------------------------------------------
// Rows per thread of the column kernels (chosen by measurement on the N=64,
// C=256, 56x56 layer: the configurations that fit the registers without spilling).
constexpr int kDwRowsFwd = 4, kDwRowsBd = 4, kDwRowsBw = 2;

struct DwPlan {
    bool fast;             // 3 x 3 kernels for this pass
    bool col;              // column kernel (else the gathering input-gradient kernel)
    int V;                 // channels per thread (8 or 4)
    bool vec;              // C % V == 0: vector loads
    int lanes, lsh, tiles; // channel lanes per pixel, log2, channel slices
    int R;                 // column kernels: rows per thread
    bool rows;             // row kernels (forward, input gradient at stride 1): segments of `seg` rows
    int seg;
    long long items;       // work items: columns, or input pixels for the gathering kernel
    int ng, iwid;          // column kernels: row groups per image, columns per row
    int ct, tg;            // generic kernels: channel tiles of kDwCB, tap groups of 9
    int splits, pps;       // weight gradient: splits and work items per split
    int grid;              // 3 x 3 forward / input gradient: workgroups (tiles x blocks per slice)
    size_t ws_bytes;
};

inline int dw_lanes(int C, int V, int most = 8) {
    int l = 1;
    while (l < most && l * V < C) l *= 2;
    return l;
}

// Channel lanes of the row kernels, 4 channels each: 64, or on layers of several
// slices the count of 64, 32 and 16 (a cache line in bf16) that leaves the fewest
// lanes of the last slice empty.  Of 280 channels in slices of 256 nearly half
// are: 133 x 33 x 33 maps, bf16, forward 182 us in 64 lanes, 115 in 16 (160 in the
// column kernels), input gradient 285, 124 (186); 288 channels, 114 x 54 x 54, stride
// 2, fp32 forward 209, 120 (150).
inline int dw_row_lanes(int C) {
    int best = dw_lanes(C, 4, 64);
    for (int l = 32; C > 256 && l >= 16; l /= 2)
        if (cdiv(C, l * 4) * l < cdiv(C, best * 4) * best) best = l;
    return best;
}

// Columns per thread of the row kernels: as many as the registers take.
inline int dw_row_cols(const Geom &g, int pass) {
    return pass == 0 ? (g.SH == 1 ? 4 : 2) : (g.dt == QL_BF16 ? 4 : 2);
}

// pass: 0 forward, 1 input gradient, 2 weight gradient
inline DwPlan plan_dw(const Geom &g, int pass) {
    DwPlan p{};
    const int taps = g.KH * g.KW;
    // (the 3 x 3 kernels address each tensor with 32-bit buffer offsets)
    const long long xbytes = (long long)g.N * g.H * g.W * g.C * g.esize();
    const long long pbytes = (long long)g.N * g.HO * g.WO * g.C * g.esize();
    p.fast = g.KH == 3 && g.KW == 3 && g.SH == g.SW && g.SH <= 2 && xbytes < (1LL << 31) && pbytes < (1LL << 31);
    p.col = p.fast && (pass != 1 || g.SH == 1);
    // bf16 channel vectors: 16 bytes for the gathering input gradient, else 8
    // (the column kernels' registers; the weight gradient's 27 V accumulators)
    p.V = (g.dt == QL_BF16 && g.C % 8 == 0 && pass == 1 && !p.col) ? 8 : 4;
    p.vec = g.C % p.V == 0;
    p.lanes = dw_lanes(g.C, p.V);
    p.lsh = p.lanes == 1 ? 0 : (p.lanes == 2 ? 1 : (p.lanes == 4 ? 2 : 3));
    p.tiles = cdiv(g.C, p.lanes * p.V);
    p.ct = cdiv(g.C, kDwCB);
    p.tg = cdiv(taps, 9);
    p.R = pass == 0 ? kDwRowsFwd : (pass == 1 ? kDwRowsBd : kDwRowsBw);
    const int rows = pass == 1 ? g.H : g.HO;
    p.iwid = pass == 1 ? g.W : g.WO;
    p.ng = cdiv(rows, p.R);
    p.items = p.col ? (long long)g.N * p.ng * p.iwid : (long long)g.N * (pass == 1 ? g.H * g.W : g.HO * g.WO);
    const int PL = kThreads / p.lanes;
    // The row kernels on large maps: a segment of rows per thread, as many segments
    // per column as make the fewest row steps of a workgroup slot (the rounds
    // times a segment's rows and halo), where at least three quarters of the
    // resident workgroups get a segment of 14 rows or more.  With less work than
    // that a thread's rows are a serial chain, about 2 us each alone on a SIMD, and
    // the column kernels' shorter items win (bf16 forward and input gradient, us,
    // row against column kernels: 64 x 56 x 56 maps of 256 channels 115, 114 against
    // 170, 213; 128 x 32 x 32 of 32 channels 26.4, 25.2 against 14.3, 14.2).
    // (T2 moves a third of the proposed neuron's bytes per product, and reads X again at
    // every store of the input gradient: in bf16 its column kernels are the faster ones,
    // 352 channels, 151 x 56 x 56 maps, 334 us against 482, 176 channels, 158 x 47 x 47, 170 against 174.)
    const int rows_env = env_override("QLAYER_DW_ROWS", -1);
    const bool t2 = g.ne == NEURON_T2 && g.dt == QL_BF16 && rows_env != 1;
    if (p.col && p.vec && pass != 2 && rows_env != 0 && !t2) {
        const int lanes = dw_row_lanes(g.C), tiles = cdiv(g.C, lanes * 4), ncg = cdiv(p.iwid, dw_row_cols(g, pass));
        const bool three = pass == 0 ? g.dt == QL_BF16 : g.dt == QL_F32;  // 4-wave workgroups per CU by registers
        const int slots = kNumCUs * (three ? 3 : 2);
        long long best = 0;
        int seg = 0, wgs = 0;
        for (int ns = 1; ns <= std::max(1, rows / 14); ++ns) {
            const int sg = cdiv(rows, ns);
            const int n = cdiv((long long)g.N * ncg * cdiv(rows, sg), kThreads / lanes) * tiles;
            const long long cost = (long long)cdiv(n, slots) * (sg + 2);
            if (!seg || cost < best) {
                best = cost;
                seg = sg;
                wgs = n;
            }
        }
        if (rows_env == 1 || (seg >= 14 && 4LL * wgs >= 3LL * slots)) {
            p.rows = true;
            p.lanes = lanes;
            p.lsh = __builtin_ctz(lanes);
            p.tiles = tiles;
            p.iwid = ncg;
            p.seg = seg;
            p.ng = cdiv(rows, seg);
            p.items = (long long)g.N * p.ng * ncg;
            p.grid = std::max(1, std::min(cdiv(p.items, kThreads / lanes), cdiv(slots, tiles))) * tiles;
            return p;
        }
    }
    if (pass != 2) {
        const int chunks = cdiv(p.items, PL);
        const int target = env_override("QLAYER_DW_BLOCKS", 2 * kNumCUs);
        p.grid = p.fast ? std::max(1, std::min(chunks, cdiv(target, p.tiles))) * p.tiles : 0;
        return p;
    }
    // weight gradient: about 2 workgroups per CU, at least 4 items per lane and split
    const long long blocks_per_split = p.fast ? p.tiles : (long long)p.ct * p.tg;
    const int lanes_px = p.fast ? PL : kDwPL;
    p.splits = std::max(1, std::min(cdiv(env_override("QLAYER_DW_BW_BLOCKS", 2 * kNumCUs), blocks_per_split),
                                    cdiv(p.items, (long long)lanes_px * 4)));
    p.pps = cdiv(p.items, p.splits);
    p.splits = cdiv(p.items, p.pps);
    if (p.splits > 1) p.ws_bytes = align_up((size_t)p.splits * 3 * g.C * (taps + 1) * sizeof(float));
    return p;
}

inline DwArgs dw_args(const Geom &g, const DwPlan &p) {
    DwArgs a{};
    a.N = g.N; a.C = g.C; a.H = g.H; a.W = g.W; a.KH = g.KH; a.KW = g.KW;
    a.SH = g.SH; a.SW = g.SW; a.PH = g.PH; a.PW = g.PW; a.HO = g.HO; a.WO = g.WO;
    a.neuron = g.ne;
    a.J = 3 * g.C * (g.KH * g.KW + 1);
    a.lanes = p.lanes; a.lsh = p.lsh; a.tiles = p.tiles;
    a.ng = p.ng; a.iwid = p.iwid; a.seg = p.seg;
    a.fd_howo = make_fastdiv(g.HO * g.WO);
    a.fd_wo = make_fastdiv(g.WO);
    a.fd_hw = make_fastdiv(g.H * g.W);
    a.fd_w = make_fastdiv(g.W);
    a.fd_sh = make_fastdiv(g.SH);
    a.fd_sw = make_fastdiv(g.SW);
    a.fd_item = make_fastdiv(p.ng * p.iwid);
    a.fd_iw = make_fastdiv(p.iwid);
    a.xbytes = (int)std::min<long long>((long long)g.N * g.H * g.W * g.C * g.esize(), INT32_MAX);
    a.pbytes = (int)std::min<long long>((long long)g.N * g.HO * g.WO * g.C * g.esize(), INT32_MAX);
    return a;
}


// ---------------------------------------------------------------------------
// Launchers, one translation unit per kernel family (qlaunch_*.hip): the
// kernels of a call on `st`, dispatched on the dtype.
// ---------------------------------------------------------------------------
ql_status run_fwd(const Geom &g, const FwdPlan &p, const void *x, const void *wa, const void *wb, const void *wc,
                  const float *ba, const float *bb, const float *bc, void *y, void *ta, void *tb, void *ws,
                  const EpiArgs &epi, float *stat_part, hipStream_t st);
// The small-output forward (qlaunch_fwd_ksplit.hip, its own translation unit:
// compiled with the MFMA accumulators in VGPRs) with the arguments run_fwd set up.
template <typename T>
ql_status launch_fwd_ksplit(const FwdPlan &p, const FwdArgs &a, bool ep, hipStream_t st);
ql_status run_bwd_data(const Geom &g, const BwdDataPlan &p, const void *gy, const void *ta, const void *tb,
                       const void *xin, const void *wa, const void *wb, const void *wc, void *dx, void *ws,
                       hipStream_t st);
ql_status run_bwd_weight(const Geom &g, const BwdWeightPlan &p, const void *x, const void *gy, const void *ta,
                         const void *tb, float *dwa, float *dwb, float *dwc, float *dba, float *dbb, float *dbc,
                         void *ws, hipStream_t st);
ql_status run_dw_fwd(const Geom &g, const void *x, const void *const *w, const float *const *b, void *y, void *ta,
                     void *tb, const EpiArgs &epi, hipStream_t st);
ql_status run_dw_bwd_data(const Geom &g, const void *gy, const void *ta, const void *tb, const void *const *w,
                          void *dx, hipStream_t st);
ql_status run_dw_bwd_weight(const Geom &g, const DwPlan &p, const void *x, const void *gy, const void *ta,
                            const void *tb, float *const *dw, float *const *db, void *ws, hipStream_t st);

}  // namespace host
}  // namespace ql

