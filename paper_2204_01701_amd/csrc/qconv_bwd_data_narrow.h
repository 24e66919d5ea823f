// qconv_bwd_data_narrow.h -- input gradient of the quadratic convolution
// layer (arXiv 2204.01701, section 4.3, eq:SD) for narrow layers: at most 16
// input channels and a short reduction K = KH * KW * O (the 16-channel stages
// of a CIFAR ResNet), where the tiled kernels spend most of their time on
// per-tile overhead:
//
//   dX[n,h,w,c] = sum_t sum_{o,r,q} W_t[o,r,q,c] G_t[n,(h+p-r)/s,(w+p-q)/s,o]
//   G_a = G o T_b,  G_b = G o T_a,  G_c = G
//
// As in qconv_fwd_narrow.h both MFMA operands arrive in registers straight
// from global memory, in 16-byte runs of the reduction index k = (tap, o):
//   - A (rows = input channels c): the transposed weights W_t^T[c][tap][o],
//     in which a run of o within one tap is contiguous; the three terms'
//     runs are loaded once per wave and stay in registers;
//   - B (columns = input pixels): for input pixel (n, h, w) and tap (r, q)
//     the output pixel ((h + p - r) / s, (w + p - q) / s) when it exists
//     (zero otherwise), whose runs of G, T_a and T_b are contiguous in NHWC;
//     the products G o T_b and G o T_a are formed in fp32 on the run and
//     rounded once to the element type (as in the tiled kernels' prologue);
//   - the 16 x 16 accumulator puts input pixel l % 16 and channels
//     4 (l / 16) .. +4 in lane l: dX of a block is one contiguous run of 16
//     NHWC rows.
// Each wave takes every (waves)-th block of 16 input pixels.  At stride > 1 it
// takes blocks of one phase (BwdPhase), whose taps alone are its reduction
// and its weight runs, and the waves are shared out among the phases by
// their taps (16 -> 32 channels, 256 x 32 x 32 maps, 3 x 3 at stride 2, whose
// phases of 1, 2, 2 and 4 taps fit where the 9 taps did not: fp32 290 us in the
// tiled kernel, 41 us here; bf16 43 and 20).
#pragma once

#include "qargs.h"
#include "qdevice.h"
#include "qconv_fwd_narrow.h"
#include "qpipe.h"

namespace ql {

// CB: 16-channel row blocks (C <= 16 CB, C a multiple of 4).  NCH: reduction
// chunks (K <= NCH narrow_chunk).  S1: stride 1.  O (and so every run) is a
// multiple of the run length.
template <typename T, int CB, int NCH, bool S1>
__global__ __launch_bounds__(kThreads, 2) void qconv_bwd_data_narrow_kernel(const BwdDataArgs a) {
    constexpr int VEC = Elem<T>::VEC;
    constexpr int CK = narrow_chunk<T>();
    const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
    const uint32_t gbytes = (uint32_t)(a.N * a.HO * a.WO * a.O) * (uint32_t)sizeof(T);
    const __amdgpu_buffer_rsrc_t grs[3] = {raw_rsrc(a.gy, gbytes), raw_rsrc(a.ta, gbytes), raw_rsrc(a.tb, gbytes)};

    // This wave's phase, its rank among the phase's waves and their number: wave
    // u of every a.units belongs to the phase with unit_end[phase - 1] <= u < unit_end[phase]
    // (past kMaxPhases phases: to phase u).
    const int nw = gridDim.x * (kThreads / 64);
    const int wid = blockIdx.x * (kThreads / 64) + wave_id();
    int phase = 0, rank = wid, ranks = nw;
    if constexpr (!S1) {
        const int round = wid / a.units, u = wid - round * a.units;
        int at = u, n = 1;
        const int nph = a.SH * a.SW;
        if (nph <= 8) {  // (fixed indices: a walk down the list waits for the scalar cache at each entry)
            at = 0;
            n = a.units;
#pragma unroll
            for (int i = 7; i >= 0; --i) {
                const bool past = (i < nph) & (u >= a.unit_end[i]);
                phase += past;
                at = max(at, past ? (int)a.unit_end[i] : 0);
                n = i < nph && !past ? (int)a.unit_end[i] : n;
            }
            n -= at;
        } else if (nph <= kMaxPhases) {
            while (u >= a.unit_end[phase]) ++phase;  // (u < units = the last phase's end)
            at = phase ? a.unit_end[phase - 1] : 0;
            n = a.unit_end[phase] - at;
        } else {
            phase = u;
        }
        rank = round * n + u - at;
        ranks = (nw / a.units) * n + min(max(nw % a.units - at, 0), n);
    }
    const BwdPhase ph = S1 ? BwdPhase(a.H, a.W, a.KH, a.KW, a.PH, a.PW)
                           : BwdPhase(phase, a.H, a.W, a.KH, a.KW, a.PH, a.PW, a.fd_sh, a.fd_sw);
    const RunDiv dqp(S1 ? 1 : ph.qp), dwp(S1 ? 1 : ph.wp), dhw(S1 ? 1 : ph.hp * ph.wp);
    const int K = S1 ? a.K : ph.rp * ph.qp * a.O;
    const int mp = S1 ? a.M : a.N * ph.hp * ph.wp;

    // This lane's reduction runs: k = CK ch + VEC lg .. + VEC, the phase's tap
    // (ri, qi), first channel o; kw: the run in the whole filter's row.
    int kr[NCH], kq[NCH], ko[NCH], kw[NCH];
    bool kin[NCH];
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
        const int k = CK * ch + VEC * lg;
        kin[ch] = k < K;
        const int tap = kin[ch] ? (int)fdiv((uint32_t)k, a.fd_o) : 0;
        ko[ch] = k - tap * a.O;
        kr[ch] = S1 ? (int)fdiv((uint32_t)tap, a.fd_kw) : (int)dqp.div((uint32_t)tap);
        kq[ch] = tap - kr[ch] * (S1 ? a.KW : ph.qp);
        kw[ch] = S1 ? k : ((ph.r0 + a.SH * kr[ch]) * a.KW + ph.q0 + a.SW * kq[ch]) * a.O + ko[ch];
    }
    // The three terms' transposed weight runs: row c = 16 cb + li (zero past C or K).
    v4u wf[3][CB][NCH];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        const __amdgpu_buffer_rsrc_t wrs = raw_rsrc(a.wt[t], (uint32_t)(a.C * a.K) * (uint32_t)sizeof(T));
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const int c = 16 * cb + li;
#pragma unroll
            for (int ch = 0; ch < NCH; ++ch) {
                wf[t][cb][ch] = narrow_run<T>(wrs, c * a.K + kw[ch], (c < a.C) & kin[ch]);
            }
        }
    }

    T *__restrict__ dx = static_cast<T *>(a.dx);
    const int nblk = (mp + 15) / 16;
    for (int b = rank; b < nblk; b += ranks) {
        // this lane's input pixel (B column): image n, position (h, w) of the phase
        const int m = 16 * b + li;
        const bool pok = m < mp;
        const int pp = pok ? m : mp - 1;
        int n, h, w, p;
        if constexpr (S1) {
            n = (int)fdiv((uint32_t)pp, a.fd_hw);
            const int rem = pp - n * a.H * a.W;
            h = (int)fdiv((uint32_t)rem, a.fd_w);
            w = rem - h * a.W;
            p = m;
        } else {
            n = (int)dhw.div((uint32_t)pp);
            const int rem = pp - n * ph.hp * ph.wp;
            h = (int)dwp.div((uint32_t)rem);
            w = rem - h * ph.wp;
            p = (n * a.H + ph.h0 + a.SH * h) * a.W + ph.w0 + a.SW * w;
        }
        const int nbase = n * a.HO * a.WO;
        f32x4n_t acc[CB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) acc[cb] = f32x4n_t{0.0f, 0.0f, 0.0f, 0.0f};
        // Chunks in groups of GC: a group's runs are all loaded before its products.
        // (A phase's taps may end early, so a long reduction takes small groups there: the
        // layer of the header in fp32 42 us in pairs, 55 in fours; all at once where they
        // fit: 16 -> 8 channels of the same maps 23 us in fp32, 29 in pairs.)
        constexpr int GC = NCH <= 5 ? NCH : (S1 ? (NCH + 1) / 2 : 2);
#pragma unroll
        for (int c0 = 0; c0 < NCH; c0 += GC) {
            if (!S1 && CK * c0 >= K) continue;  // (wave-uniform: past the phase's taps)
            v4u run[GC][3];  // of G, T_a, T_b
#pragma unroll
            for (int u = 0; u < GC && c0 + u < NCH; ++u) {
                const int ch = c0 + u;
                if (!S1 && GC > 2 && CK * ch >= K) continue;
                // the output pixel tap (r, q) of this input pixel reads, if any
                const int oh = h + ph.oh0 - kr[ch], ow = w + ph.ow0 - kq[ch];
                const bool ok = pok & kin[ch] & ((unsigned)oh < (unsigned)a.HO) & ((unsigned)ow < (unsigned)a.WO);
                const int off = (nbase + oh * a.WO + ow) * a.O + ko[ch];
#pragma unroll
                for (int t = 0; t < 3; ++t) run[u][t] = narrow_run<T>(grs[t], off, ok);
            }
#pragma unroll
            for (int u = 0; u < GC && c0 + u < NCH; ++u) {
                const int ch = c0 + u;
                if (!S1 && GC > 2 && CK * ch >= K) continue;
                v4u ga, gb;
                prologue_frag<T>(run[u][0], run[u][1], run[u][2], ga, gb);
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    narrow_mfma<T>(wf[0][cb][ch], ga, acc[cb]);
                    narrow_mfma<T>(wf[1][cb][ch], gb, acc[cb]);
                    narrow_mfma<T>(wf[2][cb][ch], run[u][0], acc[cb]);
                }
            }
        }
        if (pok) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                const int c = 16 * cb + 4 * lg;
                if (c < a.C)
                    store4<T>(dx + (size_t)p * a.C + c, acc[cb][0], acc[cb][1], acc[cb][2], acc[cb][3]);
            }
        }
    }
}

}  // namespace ql
