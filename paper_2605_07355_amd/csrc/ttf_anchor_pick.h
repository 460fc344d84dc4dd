// The anchor rule evaluated on the device from what the frame-sum kernels leave in the workspace: the guess
// from the guess channels, and the exact rule from the per-slice shares.  Shared by the kernels that choose
// an anchor in their prologue.
#pragma once

#include "ttf_device.h"
#include "ttf_internal.h"

namespace ttf {
namespace {

constexpr int kAnchorGiven = -2;   // "fixed_anchor" value: the anchor of every clip is already in anchor_index

// Anchor guess, step 2: the anchor rule evaluated on the guess channels alone (fp64 from the fp32
// sums of step 1), by all NWV waves of a block together (every thread must call it; it synchronises
// the block).  The guess is trusted when its score beats the runner-up's by at least kGuessMinGap and
// no score is NaN; the search then runs against it before the exact rule has been evaluated, and the
// exact rule (from sums the search produces on the side) confirms it or triggers a second search.
// Returns the guessed frame (lowest k on ties) and whether it is trusted, to every thread.
constexpr double kGuessMinGap = 0.1;
template <int NWV, int UN>                              // UN: frames in flight per wave
__device__ __forceinline__ void guess_pick_block(const float* __restrict__ guess_sum, int b, int F, int parts,
                                                 int& guess, bool& trusted)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const size_t fstride = (size_t)parts * kGuessChannels;
    const float* gs = guess_sum + (size_t)b * F * fstride + lane * 4;
    // this lane's four guess channels of frame k: its parts added in order
    auto load4 = [&](int k) {
        float4 v = *reinterpret_cast<const float4*>(gs + (size_t)k * fstride);
        for (int pp = 1; pp < parts; ++pp) {
            const float4 q = *reinterpret_cast<const float4*>(gs + (size_t)k * fstride + (size_t)pp * kGuessChannels);
            v.x += q.x; v.y += q.y; v.z += q.z; v.w += q.w;
        }
        return v;
    };
    __shared__ double gsh[NWV][kGuessChannels];
    __shared__ double s_best[NWV], s_second[NWV];
    __shared__ int s_arg[NWV], s_nan[NWV];
    __shared__ int s_out[2];
    // clips of up to NWV*UN frames: every wave's frames stay in its registers for the second pass
    const bool resident = F <= NWV * UN;
    float4 v[UN];
    double gp[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k0 = wave; k0 < F; k0 += NWV * UN) {
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int k = k0 + NWV * u;
            v[u] = float4{0.f, 0.f, 0.f, 0.f};
            if (k < F) v[u] = load4(k);
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            gp[0] += (double)v[u].x; gp[1] += (double)v[u].y; gp[2] += (double)v[u].z; gp[3] += (double)v[u].w;
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) gsh[wave][lane * 4 + e] = gp[e];
    __syncthreads();
    double g[4], vv = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        double t = gsh[0][lane * 4 + e];
#pragma unroll
        for (int w = 1; w < NWV; ++w) t += gsh[w][lane * 4 + e];
        g[e] = t;
        vv += t * t;
    }
    vv = wave_sum(vv);
    double best = -1.0e300, second = -1.0e300;          // wave-uniform running top two of this wave's frames
    int arg = 0x7fffffff, nan = 0;
    for (int k0 = wave; k0 < F; k0 += NWV * UN) {       // ascending k per wave: strict > keeps the lowest on ties
        if (!resident) {
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int k = k0 + NWV * u;
                v[u] = float4{0.f, 0.f, 0.f, 0.f};
                if (k < F) v[u] = load4(k);
            }
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int k = k0 + NWV * u;
            const double xv[4] = {(double)v[u].x, (double)v[u].y, (double)v[u].z, (double)v[u].w};
            double uv = 0.0, uu = 0.0;
#pragma unroll
            for (int e = 0; e < 4; ++e) { uv += xv[e] * g[e]; uu += xv[e] * xv[e]; }
            uv = wave_sum(uv);
            uu = wave_sum(uu);
            const double den = sqrt(uu) * sqrt(vv);
            const double score = den > 0.0 ? uv / den : 0.0;
            if (k < F) {                                // wave-uniform
                if (!(score == score)) nan = 1;
                if (score > best) { second = best; best = score; arg = k; }
                else if (score > second) second = score;
            }
        }
    }
    if (lane == 0) { s_best[wave] = best; s_second[wave] = second; s_arg[wave] = arg; s_nan[wave] = nan; }
    __syncthreads();
    if (threadIdx.x == 0) {
        double bb = -1.0e300, sec = -1.0e300;
        int aa = 0x7fffffff, nn = 0;
        for (int w = 0; w < NWV; ++w) {
            nn |= s_nan[w];
            if (s_best[w] > bb || (s_best[w] == bb && s_arg[w] < aa)) {
                sec = fmax(sec, bb);
                bb = s_best[w];
                aa = s_arg[w];
            } else {
                sec = fmax(sec, s_best[w]);
            }
            sec = fmax(sec, s_second[w]);
        }
        s_out[0] = aa == 0x7fffffff ? 0 : aa;
        s_out[1] = (!nn && aa != 0x7fffffff && (F == 1 || bb - sec >= kGuessMinGap)) ? 1 : 0;
    }
    __syncthreads();
    guess = s_out[0];
    trusted = s_out[1] != 0;
}

// Arg max over k of cos(frame_sum_k, clip_sum), assembled in fp64 from the per-slice shares
// (slices added in order); 0 when a norm is 0.  Computed by one wave, every lane gets the result;
// lowest k on ties; frame 0 if every score is NaN.
__device__ __forceinline__ int pick_anchor(const double* __restrict__ score_part,
                                           const double* __restrict__ clip_part, int b, int F, int S, int lane)
{
    double vv = 0.0;
#pragma unroll 8
    for (int s = 0; s < S; ++s) vv += clip_part[(size_t)b * S + s];
    double best = -1.0e300;
    int arg = 0x7fffffff;
    for (int k = lane; k < F; k += 64) {                // ascending k per lane: strict > keeps the lowest
        double uv = 0.0, uu = 0.0;
#pragma unroll 8
        for (int s = 0; s < S; ++s) {
            const double2 o = *reinterpret_cast<const double2*>(score_part + (((size_t)b * S + s) * F + k) * 2);
            uv += o.x;
            uu += o.y;
        }
        const double den = sqrt(uu) * sqrt(vv);
        const double score = den > 0.0 ? uv / den : 0.0;
        if (score > best) { best = score; arg = k; }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        const double ob = __shfl_xor(best, m, 64);
        const int oa = __shfl_xor(arg, m, 64);
        if (ob > best || (ob == best && oa < arg)) { best = ob; arg = oa; }
    }
    return arg == 0x7fffffff ? 0 : arg;
}

}  // namespace
}  // namespace ttf
