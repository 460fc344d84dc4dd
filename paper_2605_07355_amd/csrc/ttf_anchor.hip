// Anchor frame selection (Section 3, "Anchor Frame Selection"):
//   a* = argmax_k cos( (1/N) sum_i x_{k,i} , (1/(FN)) sum_{k',i} x_{k',i} )
// The cosine does not change when either argument is scaled, so the kernels work with plain
// sums: frame sums in fp32 (one streaming pass over X, the only large read of this stage),
// everything after that in fp64 on [B,F,C] numbers.  The last kernel of the stage picks the arg
// max (lowest k on ties) and computes 1/||x_{a,j}|| for the anchor tokens, which the window
// search uses as the anchor half of every cosine denominator.
#include <algorithm>
#include <type_traits>

#include "ttf_anchor_pick.h"
#include "ttf_internal.h"

namespace ttf {
namespace {

// One block = one frame x one slice of 64*V channels x one of `parts` runs of rows (whole rounds of 16 rows
// but for the last run).  Wave w adds rows w, w+4, ... of the run; the four partial sums are combined through
// LDS in wave order, so the result is order-stable, and stored as share `part` of the frame:
// out[frame][part][C].  Bound by HBM on large inputs and by latency where there are few blocks.  R rows are
// in flight per wave, and none behind a guard of its own: a load under a guard is waited for before the next
// one is issued.  Kernel alone, eight guarded rows -> four plain ones: B64 F32 16x16 C256 76 -> 45 us (6.0
// TB/s), B16 F32 16x16 C4000 196 -> 178, B1 F64 14x14 C2048 26 -> 12.  Eight plain ones pay for fp32 rows in at
// most 256 blocks (sums and their addition, four -> eight: B1 F4 28x16 C912 20.0 -> 17.3, B1 F20 22x23 C272
// 25.6 -> 22.6; 612 blocks, B9 F34 32x32 C320: 75 -> 86).
// `spec` (may be null): per clip {guessed anchor, guess trusted, ...}; clips with a trusted guess get
// their exact sums from the search and are skipped here.  Blocks from keep_from on, the last to run, leave
// their rows in the Infinity Cache for the search (kept_share()).
template <typename T, int V, int R>
__global__ __launch_bounds__(256) void k_frame_sums(const T* __restrict__ x, float* __restrict__ out,
                                                    int N, int C, int F, int parts, const int32_t* __restrict__ spec,
                                                    unsigned keep_from)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const size_t frame = blockIdx.x / parts;
    const bool keep = blockIdx.y * gridDim.x + blockIdx.x >= keep_from;   // (block-uniform)
    const int run = blockIdx.x % parts;
    if (spec && spec[4 * (frame / F) + 1]) return;
    const int c0 = (blockIdx.y * 64 + lane) * V;
    const int per = ((N + parts - 1) / parts + 15) / 16 * 16;
    const int lo = run * per, hi = min(N, lo + per);
    __shared__ float part[4][64 * V];
    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.f;
    if (c0 < C) {
        const T* base = x + frame * (size_t)N * C + c0;
        int i = lo + wave;
        auto add_rows = [&](auto count) {
            constexpr int n = decltype(count)::value;
            RowVec<T, V> r[n];
            if (keep) {
#pragma unroll
                for (int u = 0; u < n; ++u) r[u].template load<false>(base + (size_t)(i + 4 * u) * C);
            } else {
#pragma unroll
                for (int u = 0; u < n; ++u) r[u].template load<true>(base + (size_t)(i + 4 * u) * C);
            }
#pragma unroll
            for (int u = 0; u < n; ++u) {
#pragma unroll
                for (int e = 0; e < V; ++e) acc[e] += r[u].v[e];
            }
            i += 4 * n;
        };
        while (i + 4 * (R - 1) < hi) add_rows(std::integral_constant<int, R>{});
        while (i + 12 < hi) add_rows(std::integral_constant<int, 4>{});
        while (i < hi) add_rows(std::integral_constant<int, 1>{});
    }
#pragma unroll
    for (int e = 0; e < V; ++e) part[wave][lane * V + e] = acc[e];
    __syncthreads();
    if (wave == 0 && c0 < C) {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const int q = lane * V + e;
            out[blockIdx.x * (size_t)C + c0 + e] = ((part[0][q] + part[1][q]) + part[2][q]) + part[3][q];
        }
    }
}

// The same sums for rows that are whole 4 KiB slabs: a block owns one frame and one slab, every
// thread its 16 bytes of the slab for all N rows (eight rows in flight), so the four waves of a block
// read 4 KiB of one row together and no cross-wave sum is needed.
template <typename T, int V>
__global__ __launch_bounds__(256) void k_frame_sums_slab(const T* __restrict__ x, float* __restrict__ frame_sum,
                                                         int N, int C, int F, const int32_t* __restrict__ spec, unsigned keep_from)
{
    const size_t frame = blockIdx.x;
    const bool keep = blockIdx.y * gridDim.x + blockIdx.x >= keep_from;   // (block-uniform)
    if (spec && spec[4 * (frame / F) + 1]) return;
    const int c0 = (blockIdx.y * 256 + threadIdx.x) * V;
    const T* base = x + frame * (size_t)N * C + c0;
    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.f;
    int i = 0;
    for (; i + 8 <= N; i += 8) {
        RowVec<T, V> r[8];
        if (keep) {
#pragma unroll
            for (int u = 0; u < 8; ++u) r[u].template load<false>(base + (size_t)(i + u) * C);
        } else {
#pragma unroll
            for (int u = 0; u < 8; ++u) r[u].template load<true>(base + (size_t)(i + u) * C);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
#pragma unroll
            for (int e = 0; e < V; ++e) acc[e] += r[u].v[e];
        }
    }
    for (; i < N; ++i) {
        RowVec<T, V> r0;
        r0.template load<true>(base + (size_t)i * C);
#pragma unroll
        for (int e = 0; e < V; ++e) acc[e] += r0.v[e];
    }
#pragma unroll
    for (int e = 0; e < V; ++e) frame_sum[frame * (size_t)C + c0 + e] = acc[e];
}

// Per clip and 256-channel slice, in fp64: the clip sum g = sum_k frame_sum[k] (k ascending inside
// each of sixteen interleaved groups, groups added in order), then for every frame the slice's share
// of <frame_sum_k, g> and |frame_sum_k|^2, and the slice's share of |g|^2.  The cosine of the
// anchor rule is assembled from these shares by pick_anchor().
// STRIPS: a frame sum is not stored as such but as `strips` partial sums (one per run of the grid, as the
// walking search writes them, or of rows, as k_frame_sums: fs[k][strip][C]); they are added in ascending
// order (fp32) as they are loaded.  UN: frames in flight per wave.
template <int UN, bool STRIPS>
__device__ __forceinline__ void anchor_partials_body(const float* __restrict__ fs, double* __restrict__ score_part,
                                                     double* __restrict__ clip_part, size_t b, int slice, int fg,
                                                     int F, int C, int S, int FG, int strips, double (*gsh)[256])
{
    // Long clips: FG blocks share a (clip, slice); each forms the clip sum itself (frame sums come
    // from L2) and scores its own run of frames, so that few clips still fill the chip.
    constexpr int NWV = 16;                             // waves per block
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int per = (F + FG - 1) / FG;                  // frames scored by one block
    const int k_lo = fg * per, k_hi = min(F, k_lo + per);
    const size_t fstride = STRIPS ? (size_t)strips * C : (size_t)C;   // floats between consecutive frames
    int c[4];
    bool ok[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        c[e] = slice * 256 + lane * 4 + e;             // four consecutive channels per lane: one 16-byte load
        ok[e] = c[e] < C;
    }
    // this lane's four channels of one frame sum: one 16-byte load when the row allows it
    const bool vec = (C % 4 == 0) && ok[3];
    auto load4 = [&](const float* row, float* out) {
        if constexpr (STRIPS) {                        // (C % 4 == 0 on this path: always 16-byte loads)
            if (!ok[3]) return;                        // the last slice may reach beyond C
            for (int s0 = 0; s0 < strips; s0 += 8) {
                float4 q[8];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (s0 + u < strips) q[u] = *reinterpret_cast<const float4*>(row + (size_t)(s0 + u) * C + c[0]);
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (s0 + u < strips) { out[0] += q[u].x; out[1] += q[u].y; out[2] += q[u].z; out[3] += q[u].w; }
            }
        } else if (vec) {
            const float4 q = *reinterpret_cast<const float4*>(row + c[0]);
            out[0] = q.x; out[1] = q.y; out[2] = q.z; out[3] = q.w;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (ok[e]) out[e] = row[c[e]];
        }
    };
    // short clips: every wave's frames fit its registers, so the second pass re-uses the first's loads
    const bool resident = F <= NWV * UN && FG == 1;
    float v[UN][4];
    double gp[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k0 = wave; k0 < F; k0 += NWV * UN) {
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int k = k0 + NWV * u;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[u][e] = 0.f;
            if (k < F) load4(fs + (size_t)k * fstride, v[u]);
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
#pragma unroll
            for (int e = 0; e < 4; ++e) gp[e] += (double)v[u][e];
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) gsh[wave][lane * 4 + e] = gp[e];
    __syncthreads();
    double g[4], vv = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int q = lane * 4 + e;
        double t = gsh[0][q];
#pragma unroll
        for (int w = 1; w < NWV; ++w) t += gsh[w][q];
        g[e] = t;
        vv += t * t;
    }
    vv = wave_sum(vv);
    if (threadIdx.x == 0 && fg == 0) clip_part[b * S + slice] = vv;
    for (int k0 = k_lo + wave; k0 < k_hi; k0 += NWV * UN) {
        if (!resident) {
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int k = k0 + NWV * u;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[u][e] = 0.f;
                if (k < k_hi) load4(fs + (size_t)k * fstride, v[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int k = k0 + NWV * u;
            double uv = 0.0, uu = 0.0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double x = (double)v[u][e];
                uv += x * g[e];
                uu += x * x;
            }
            uv = wave_sum(uv);
            uu = wave_sum(uu);
            if (lane == 0 && k < k_hi) {
                double* o = score_part + ((b * S + slice) * (size_t)F + k) * 2;
                o[0] = uv;
                o[1] = uu;
            }
        }
    }
}

// MIXED: clips with a trusted anchor guess (spec[b][1]) have their frame sums in parts
// (strip_sum [B,F,strips,C], frame_sum itself for a single part), the other clips in frame_sum [B,F,C];
// otherwise every clip in frame_sum, or (spec null, strip_sum given) every clip as the shares that
// k_frame_sums leaves in strip_sum.
template <bool MIXED>
__global__ __launch_bounds__(1024) void k_anchor_partials(const float* __restrict__ frame_sum,
                                                         double* __restrict__ score_part,
                                                         double* __restrict__ clip_part, int F, int C, int S,
                                                         int FG, int strips, const float* __restrict__ strip_sum,
                                                         const int32_t* __restrict__ spec)
{
    const int fg = blockIdx.x % FG;
    const int slice = (blockIdx.x / FG) % S;
    const size_t b = blockIdx.x / FG / S;
    __shared__ double gsh[16][256];
    if (MIXED && (!spec || spec[4 * b + 1] != 0))        // block-uniform
        anchor_partials_body<2, true>(strip_sum + b * (size_t)F * strips * C, score_part, clip_part, b, slice, fg, F,
                                      C, S, FG, strips, gsh);
    else
        anchor_partials_body<8, false>(frame_sum + b * (size_t)F * C, score_part, clip_part, b, slice, fg, F, C, S, FG,
                                       1, gsh);
}

// Partial sums -> frame sums for the clips with a trusted anchor guess (grids in many runs per
// frame: a plain streaming reduction ahead of k_anchor_partials<false> keeps the chip full, where the
// fused form has too few blocks).  Block (frame, 1024-channel slab): thread t adds its four channels
// over the strips in ascending order, eight loads in flight.
__global__ __launch_bounds__(256) void k_reduce_strips(const float* __restrict__ strip_sum,
                                                       float* __restrict__ frame_sum,
                                                       const int32_t* __restrict__ spec, int F, int C, int strips)
{
    const size_t frame = blockIdx.x;
    if (!spec[4 * (frame / F) + 1]) return;             // this clip's frame sums come from k_frame_sums
    const int c = (blockIdx.y * 256 + threadIdx.x) * 4;
    if (c >= C) return;
    const float* row = strip_sum + frame * (size_t)strips * C + c;
    float4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < strips; s0 += 8) {
        float4 q[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (s0 + u < strips) q[u] = *reinterpret_cast<const float4*>(row + (size_t)(s0 + u) * C);
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (s0 + u < strips) { acc.x += q[u].x; acc.y += q[u].y; acc.z += q[u].z; acc.w += q[u].w; }
    }
    *reinterpret_cast<float4*>(frame_sum + frame * (size_t)C + c) = acc;
}

// Anchor guess, step 1: sums over the tokens of a frame of the kGuessChannels guess channels only
// (kGuessSegments runs of 64 channels per token row).  Block (frame, part) covers tokens part*per ..
// (part+1)*per - 1: thread t reads 16-byte piece t%P of the guess channels of its tokens t/P, t/P + 256/P, ...
// (P = 32 pieces of bf16, 64 of fp32 rows); the token groups are added through LDS in order.  The parts
// of a frame are added by guess_pick_block.
template <typename T>
__global__ __launch_bounds__(256) void k_guess_sums(const T* __restrict__ x, float* __restrict__ guess_sum,
                                                    int N, int C, int parts)
{
    constexpr int V = 16 / (int)sizeof(T), SEG = kGuessSegChannels / V, P = kGuessSegments * SEG, G = 256 / P;
    const size_t frame = blockIdx.x / parts;
    const int part = blockIdx.x % parts;
    const int per = (N + parts - 1) / parts;
    const int n_lo = part * per, n_hi = min(N, n_lo + per);
    const int ts = threadIdx.x / P, q = threadIdx.x % P;
    const int ch = guess_segment_start(C, q / SEG) + (q % SEG) * V;
    const T* base = x + frame * (size_t)N * C + ch;
    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.f;
    for (int i0 = n_lo + ts; i0 < n_hi; i0 += 8 * G) {
        RowVec<T, V> r[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + G * u;
            if (i < n_hi) r[u].template load<true>(base + (size_t)i * C);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (i0 + G * u < n_hi) {
#pragma unroll
                for (int e = 0; e < V; ++e) acc[e] += r[u].v[e];
            }
        }
    }
    __shared__ float part_s[G][kGuessChannels];
#pragma unroll
    for (int e = 0; e < V; ++e) part_s[ts][q * V + e] = acc[e];
    __syncthreads();
    float t = part_s[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < G; ++w) t += part_s[w][threadIdx.x];
    guess_sum[(size_t)blockIdx.x * kGuessChannels + threadIdx.x] = t;
}

// Batch-tied anchor (tied-batch mode): the frame whose anchor score, averaged over the B clips
// (fp64), is largest; lowest k on ties.  A fixed frame is simply broadcast.  One workgroup of 16
// waves: wave w adds the scores of clips w, w+16, ... (ascending) for 64 frames at a time, wave 0
// adds the 16 partial sums in wave order and keeps the running arg max; the shared index is
// written to every entry of anchor_index.
__global__ __launch_bounds__(1024) void k_tied_anchor(const double* __restrict__ score_part,
                                                      const double* __restrict__ clip_part,
                                                      int32_t* __restrict__ anchor_index, int B, int F, int S,
                                                      int fixed_anchor)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __shared__ double part[16][64];
    __shared__ int s_arg;
    int arg = fixed_anchor;
    if (fixed_anchor < 0) {
        double best = -1.0e300;
        arg = 0x7fffffff;
        for (int k0 = 0; k0 < F; k0 += 64) {
            const int k = k0 + lane;
            double acc = 0.0;
            for (int b = wave; b < B && k < F; b += 16) {
                double vv = 0.0, uv = 0.0, uu = 0.0;
#pragma unroll 8
                for (int s = 0; s < S; ++s) {
                    vv += clip_part[(size_t)b * S + s];
                    const double2 o = *reinterpret_cast<const double2*>(score_part + (((size_t)b * S + s) * F + k) * 2);
                    uv += o.x;
                    uu += o.y;
                }
                const double den = sqrt(uu) * sqrt(vv);
                acc += den > 0.0 ? uv / den : 0.0;
            }
            part[wave][lane] = acc;
            __syncthreads();
            if (wave == 0 && k < F) {
                double sum = part[0][lane];
#pragma unroll
                for (int w = 1; w < 16; ++w) sum += part[w][lane];
                const double score = sum / (double)B;
                if (score > best) { best = score; arg = k; }   // ascending k per lane: strict > keeps the lowest
            }
            __syncthreads();
        }
        if (wave == 0) {
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) {
                const double ob = __shfl_xor(best, m, 64);
                const int oa = __shfl_xor(arg, m, 64);
                if (ob > best || (ob == best && oa < arg)) { best = ob; arg = oa; }
            }
            if (arg == 0x7fffffff) arg = 0;
            if (lane == 0) s_arg = arg;
        }
        __syncthreads();
        arg = s_arg;
    }
    for (int b = threadIdx.x; b < B; b += 1024) anchor_index[b] = arg;
}

// Picks the anchor of clip b (arg max of frame_score, lowest k on ties, or the fixed frame),
// publishes it, and writes 1/||x_{a,j}|| for the anchor tokens.  One wave per anchor token.
template <typename T, int V>
__global__ __launch_bounds__(256) void k_anchor_norms(const T* __restrict__ x, const T* __restrict__ ext_anchor,
                                                      const double* __restrict__ score_part,
                                                      const double* __restrict__ clip_part,
                                                      int32_t* __restrict__ anchor_index,
                                                      float* __restrict__ anchor_inv,
                                                      int F, int N, int C, int S, int fixed_anchor, int groups)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int b = blockIdx.x / groups;
    const int j = (blockIdx.x % groups) * 4 + wave;
    // the anchor is a frame of x (fixed, picked here, or already chosen: kAnchorGiven), or frame b
    // of ext_anchor (published as -1)
    const int a = ext_anchor ? -1
                : fixed_anchor >= 0 ? fixed_anchor
                : fixed_anchor == kAnchorGiven ? anchor_index[b]
                                               : pick_anchor(score_part, clip_part, b, F, S, lane);
    if (fixed_anchor != kAnchorGiven && blockIdx.x % groups == 0 && threadIdx.x == 0) anchor_index[b] = a;
    if (j >= N) return;
    const T* row = (ext_anchor ? ext_anchor + (size_t)b * N * C : x + ((size_t)b * F + a) * N * C) + (size_t)j * C;
    float ss = 0.f;
    for (int c = lane * V; c < C; c += 64 * V) {
        RowVec<T, V> r;
        r.load(row + c);
#pragma unroll
        for (int e = 0; e < V; ++e) ss = fmaf(r.v[e], r.v[e], ss);
    }
    ss = wave_sum(ss);
    if (lane == 0) anchor_inv[(size_t)b * N + j] = ss > 0.f ? 1.0f / sqrtf(ss) : 0.f;
}

// Matrix-core path.  One workgroup (8 waves) per anchor tile of 16 tokens: picks the anchor,
// writes the anchor-frame rows of the per-token outputs (never fused, all keep bits set), reads
// the tile once with coalesced loads (lane l: chunk l%4 of token l/4), accumulates squared
// norms, permutes every 16x64-byte block into MFMA operand order (lane = token + 16*chunk) and
// stores it as one contiguous KiB: anchor_frag[b][tile][K-step][lane][8 bf16].
// PAD: the grid is Wg <= 16*CT tokens wide; a tile is 16 columns of one grid row, columns at and
// beyond Wg are padding (zero fragments, inverse norm 0), and tiles are numbered row * CT + column
// tile.  Without PAD a tile is 16 consecutive flat tokens (the same thing when Wg == 16*CT).
template <bool PAD>
__global__ __launch_bounds__(512) void k_anchor_prepare(const uint16_t* __restrict__ x,
                                                        const uint16_t* __restrict__ ext_anchor,
                                                        const double* __restrict__ score_part,
                                                        const double* __restrict__ clip_part,
                                                        int32_t* __restrict__ anchor_index,
                                                        float* __restrict__ anchor_inv,
                                                        uint16_t* __restrict__ anchor_frag,
                                                        int32_t* __restrict__ fuse_map, float* __restrict__ best_sim,
                                                        int32_t* __restrict__ best_idx, uint16_t* __restrict__ keep16,
                                                        int F, int N, int C, int S, int fixed_anchor, int tiles,
                                                        int Wg, int CT)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int b = blockIdx.x / tiles, tile = blockIdx.x % tiles;
    // the anchor is a frame of x (fixed, picked here, or already chosen: kAnchorGiven), or frame b
    // of ext_anchor (published as -1)
    const int a = ext_anchor ? -1
                : fixed_anchor >= 0 ? fixed_anchor
                : fixed_anchor == kAnchorGiven ? anchor_index[b]
                                               : pick_anchor(score_part, clip_part, b, F, S, lane);
    if (fixed_anchor != kAnchorGiven && tile == 0 && threadIdx.x == 0) anchor_index[b] = a;
    // flat index of the tile's first token, and how many of its 16 columns exist
    const int first = PAD ? (tile / CT) * Wg + 16 * (tile % CT) : 16 * tile;
    const int ncol = PAD ? min(16, Wg - 16 * (tile % CT)) : 16;
    if (a >= 0 && fuse_map && (int)threadIdx.x < ncol) {     // anchor tokens are always retained
        const size_t o = ((size_t)b * F + a) * N + first + threadIdx.x;
        fuse_map[o] = -1;
        if (best_sim) best_sim[o] = 1.0f;
        if (best_idx) best_idx[o] = first + (int)threadIdx.x;
        if (!PAD && threadIdx.x == 0) keep16[o / 16] = 0xffffu;
    }
    const int KS = (C + 31) / 32;
    const uint16_t* frame = ext_anchor ? ext_anchor + (size_t)b * N * C : x + ((size_t)b * F + a) * N * C;
    const bool real = (lane >> 2) < ncol;                    // this lane's token exists (padding reads the tile's first)
    const uint16_t* src = frame + (size_t)(first + (real ? lane >> 2 : 0)) * C + (lane & 3) * 8;
    uint16_t* dst = anchor_frag + ((size_t)b * tiles + tile) * (size_t)KS * 512 + lane * 8;
    const int bperm = (4 * (lane & 15) + (lane >> 4)) * 4;
    float nn = 0.f;
    constexpr int UN = 8;                                   // K-steps in flight per wave
    for (int k0 = wave; k0 < KS; k0 += 8 * UN) {
        uint4 v[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int ks = k0 + 8 * u;
            if (ks < KS) {
                // (the last K-step of tail_channels() rows ends on pieces past the row: zeros)
                v[u] = uint4{0u, 0u, 0u, 0u};
                if (ks * 32 + (lane & 3) * 8 < C) v[u] = *reinterpret_cast<const uint4*>(src + (size_t)ks * 32);
                if (PAD && !real) v[u] = uint4{0u, 0u, 0u, 0u};
            }
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int ks = k0 + 8 * u;
            if (ks < KS) {
                uint32_t r[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bf16x2 p = __builtin_bit_cast(bf16x2, r[e]);
                    nn = __builtin_amdgcn_fdot2_f32_bf16(p, p, nn, false);
                    r[e] = (uint32_t)__builtin_amdgcn_ds_bpermute(bperm, (int)r[e]);
                }
                *reinterpret_cast<uint4*>(dst + (size_t)ks * 512) = uint4{r[0], r[1], r[2], r[3]};
            }
        }
    }
    nn += __shfl_xor(nn, 1, 64);
    nn += __shfl_xor(nn, 2, 64);
    __shared__ float part[8][16];
    if ((lane & 3) == 0) part[wave][lane >> 2] = nn;
    __syncthreads();
    if (threadIdx.x < 16) {
        float ss = part[0][threadIdx.x], inv;
        if (PAD && C % 32 != 0) {
            // rows that end inside a K-step: eight shares and inverse root rounded once each, so that the
            // similarities are no less exact than the wave-per-token kernels' (relative error against 64 bits at
            // C 776 and 4072: theirs 7.4e-8 and 9.1e-8; here with fp32 shares and root 7.7e-8 and 8.2e-8, so 7.2e-8
            // and 7.3e-8)
            double sum = (double)ss;
#pragma unroll
            for (int w = 1; w < 8; ++w) sum += (double)part[w][threadIdx.x];
            ss = (float)sum;                                 // (overflows as the fp32 sum does)
            inv = (float)(1.0 / sqrt((double)ss));
        } else {
#pragma unroll
            for (int w = 1; w < 8; ++w) ss += part[w][threadIdx.x];
            inv = 1.0f / sqrtf(ss);
        }
        anchor_inv[((size_t)b * tiles + tile) * 16 + threadIdx.x] = ss > 0.f ? inv : 0.f;
    }
}

// The anchor guessed from the sums over the guess channels, one workgroup per clip.  Bound by the fp64 sums over the
// lanes, two for each of a wave's UN frames, real or not: 32 frames of 16 clips with four a wave 7.9 us,
// with eight 9.8, on 16 waves with eight 12.9.
template <int UN>
__global__ __launch_bounds__(512) void k_guess_pick(const float* __restrict__ guess_sum, int32_t* __restrict__ spec, int F,
                                                    int parts)
{
    int a;
    bool trusted;
    guess_pick_block<8, UN>(guess_sum, (int)blockIdx.x, F, parts, a, trusted);
    if (threadIdx.x == 0) {
        int32_t* o = spec + 4 * blockIdx.x;
        o[0] = a;
        o[1] = trusted ? 1 : 0;
        o[2] = o[3] = 0;
    }
}

// Matrix-core path for fp32 tokens.  As k_anchor_prepare, but the anchor frame is stored as three
// bf16 planes (hi, mid, lo pieces of every value) per tile and K-step of 32 channels:
// anchor_frag[b][tile][K-step][plane][lane][8 bf16], 3 KiB per tile and K-step.  Inside a K-step the
// operand lane (token n, group g) holds channels 4g..4g+3 and 16+4g..16+4g+3: the order in which two
// coalesced 16-byte loads per lane (lane l: token l/4, floats 4(l%4).. of each 64-byte half) arrive
// after one lane permutation.  The search splits and orders its source fragments the same way.
template <bool PAD>
__global__ __launch_bounds__(512) void k_anchor_prepare_f32(const float* __restrict__ x,
                                                            const float* __restrict__ ext_anchor,
                                                            const double* __restrict__ score_part,
                                                            const double* __restrict__ clip_part,
                                                            int32_t* __restrict__ anchor_index,
                                                            float* __restrict__ anchor_inv,
                                                            uint16_t* __restrict__ anchor_frag,
                                                            int32_t* __restrict__ fuse_map,
                                                            float* __restrict__ best_sim,
                                                            int32_t* __restrict__ best_idx,
                                                            uint16_t* __restrict__ keep16, int F, int N, int C, int S,
                                                            int fixed_anchor, int tiles, int Wg, int CT)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int b = blockIdx.x / tiles, tile = blockIdx.x % tiles;
    const int a = ext_anchor ? -1
                : fixed_anchor >= 0 ? fixed_anchor
                : fixed_anchor == kAnchorGiven ? anchor_index[b]
                                               : pick_anchor(score_part, clip_part, b, F, S, lane);
    if (fixed_anchor != kAnchorGiven && tile == 0 && threadIdx.x == 0) anchor_index[b] = a;
    const int first = PAD ? (tile / CT) * Wg + 16 * (tile % CT) : 16 * tile;
    const int ncol = PAD ? min(16, Wg - 16 * (tile % CT)) : 16;
    if (a >= 0 && fuse_map && (int)threadIdx.x < ncol) {     // anchor tokens are always retained
        const size_t o = ((size_t)b * F + a) * N + first + threadIdx.x;
        fuse_map[o] = -1;
        if (best_sim) best_sim[o] = 1.0f;
        if (best_idx) best_idx[o] = first + (int)threadIdx.x;
        if (!PAD && threadIdx.x == 0) keep16[o / 16] = 0xffffu;
    }
    const int KS = C / 32;
    const float* frame = ext_anchor ? ext_anchor + (size_t)b * N * C : x + ((size_t)b * F + a) * N * C;
    const bool real = (lane >> 2) < ncol;                    // this lane's token exists (padding reads the tile's first)
    const float* src = frame + (size_t)(first + (real ? lane >> 2 : 0)) * C + (lane & 3) * 4;
    uint16_t* dst = anchor_frag + ((size_t)b * tiles + tile) * (size_t)KS * 1536 + lane * 8;
    const int bperm = (4 * (lane & 15) + (lane >> 4)) * 4;
    float nn = 0.f;
    constexpr int UN = 4;                                   // K-steps in flight per wave
    for (int k0 = wave; k0 < KS; k0 += 8 * UN) {
        uint4 v[UN][2];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int ks = k0 + 8 * u;
            if (ks < KS) {
                v[u][0] = *reinterpret_cast<const uint4*>(src + (size_t)ks * 32);
                v[u][1] = *reinterpret_cast<const uint4*>(src + (size_t)ks * 32 + 16);
                if (PAD && !real) v[u][0] = v[u][1] = uint4{0u, 0u, 0u, 0u};
            }
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int ks = k0 + 8 * u;
            if (ks < KS) {
                uint32_t r[8] = {v[u][0].x, v[u][0].y, v[u][0].z, v[u][0].w, v[u][1].x, v[u][1].y, v[u][1].z, v[u][1].w};
                float f[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float t = __builtin_bit_cast(float, r[e]);
                    nn = fmaf(t, t, nn);
                    f[e] = __builtin_bit_cast(float, (uint32_t)__builtin_amdgcn_ds_bpermute(bperm, (int)r[e]));
                }
                uint32_t hi[4], mid[4], lo[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) split_bf16x3(f[2 * e], f[2 * e + 1], hi[e], mid[e], lo[e]);
                uint16_t* o = dst + (size_t)ks * 1536;
                *reinterpret_cast<uint4*>(o) = uint4{hi[0], hi[1], hi[2], hi[3]};
                *reinterpret_cast<uint4*>(o + 512) = uint4{mid[0], mid[1], mid[2], mid[3]};
                *reinterpret_cast<uint4*>(o + 1024) = uint4{lo[0], lo[1], lo[2], lo[3]};
            }
        }
    }
    nn += __shfl_xor(nn, 1, 64);
    nn += __shfl_xor(nn, 2, 64);
    __shared__ float part[8][16];
    if ((lane & 3) == 0) part[wave][lane >> 2] = nn;
    __syncthreads();
    if (threadIdx.x < 16) {
        float ss = part[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < 8; ++w) ss += part[w][threadIdx.x];
        anchor_inv[((size_t)b * tiles + tile) * 16 + threadIdx.x] = ss > 0.f ? 1.0f / sqrtf(ss) : 0.f;
    }
}

template <typename F>
hipError_t by_layout(const ttf_params& p, F&& f)
{
    // 16-byte vector loads need rows that start 16-byte aligned: C*sizeof(T) % 16 == 0.
    if (p.dtype == TTF_BF16) {
        if (p.C % 8 == 0) return f(bf16_t{}, std::integral_constant<int, 8>{});
        return f(bf16_t{}, std::integral_constant<int, 1>{});
    }
    if (p.C % 4 == 0) return f(float{}, std::integral_constant<int, 4>{});
    return f(float{}, std::integral_constant<int, 1>{});
}

}  // namespace

// Rows whose 16-byte pieces one block of k_frame_sums_slab sums over a whole frame.
static bool frame_sums_by_slab(const ttf_params& p)
{
    const int V = p.dtype == TTF_BF16 ? 8 : 4;
    return p.C % (256 * V) == 0 && (size_t)p.B * p.F * (p.C / (256 * V)) >= 512;
}

// Runs of rows a frame is cut into by k_frame_sums, of at least 32 rows each: as many as make no more than 512
// blocks, two for every CU; two where one run each would leave most CUs a block and some two (257 to 384 blocks);
// whole frames beyond.  Sums and their addition together, us, by blocks without runs: 128 (B4 F16 16x16 C1024)
// 22 / two 16 / four 14 / eight 14.6; 240 (B1 F40 32x32 C3000) 58 / two 46 / four 51; 340 (B5 F34 24x24 C1024) 42 /
// two 39 / three 40; 384 (B4 F32 16x16 C1504) 27 / two 24 / three 26; 400 (B4 F50 24x24 C960) 43 / two 47.5 / three 46;
// 512 (B4 F64 16x16 C1024) 29.6 / two 31.2; 612 (B9 F34 32x32 C320 fp32) 72 / two 82.
// The shares stand in the anchor's fragment copy, which is written after the anchor has been chosen, so
// they have to fit there (short clips and long rows may get fewer).  Row lengths of whole 16-byte pieces
// only: k_anchor_partials adds the shares with 16-byte loads.
static int frame_sum_parts(const ttf_params& p, const Workspace& w)
{
    const int V = p.dtype == TTF_BF16 ? 8 : 4;
    if (p.C % V != 0 || frame_sums_by_slab(p)) return 1;
    const size_t blocks = (size_t)p.B * p.F * ((p.C + 64 * V - 1) / (64 * V));
    const size_t share = (size_t)p.B * p.F * p.C * sizeof(float);
    size_t parts = blocks <= 256 ? std::min<size_t>(8, 512 / blocks) : (blocks <= 384 ? 2 : 1);
    parts = std::min<size_t>(parts, (size_t)p.H * p.W / 32);
    parts = std::min<size_t>(parts, w.frag_bytes / share);
    if (parts < 2) return 1;
    const size_t N = (size_t)p.H * p.W, per = align_up((N + parts - 1) / parts, 16);
    return (int)((N + per - 1) / per);                       // (no run is empty)
}

hipError_t launch_frame_sums(const ttf_params& p, const void* x, const Workspace& w, bool skip_trusted, double kept,
                             hipStream_t s)
{
    const int N = p.H * p.W;
    const int32_t* spec = skip_trusted ? w.spec : nullptr;
    auto keep_from = [&](dim3 g) { return (unsigned)((double)g.x * g.y * (1.0 - kept)); };
    return by_layout(p, [&](auto tag, auto vtag) {
        using T = decltype(tag);
        constexpr int V = decltype(vtag)::value;
        if (V > 1 && frame_sums_by_slab(p)) {
            dim3 slabs((unsigned)(p.B * p.F), (unsigned)(p.C / (256 * V)));
            k_frame_sums_slab<T, V><<<slabs, 256, 0, s>>>(static_cast<const T*>(x), w.frame_sum, N, p.C, p.F, spec,
                                                          keep_from(slabs));
            return hipGetLastError();
        }
        // (beside a speculative search the fragment copy is in use: no parts)
        const int parts = skip_trusted ? 1 : frame_sum_parts(p, w);
        float* out = parts > 1 ? reinterpret_cast<float*>(w.anchor_frag) : w.frame_sum;
        dim3 grid((unsigned)(p.B * p.F * parts), (unsigned)((p.C + 64 * V - 1) / (64 * V)));
        auto go = [&](auto kernel) {
            kernel<<<grid, 256, 0, s>>>(static_cast<const T*>(x), out, N, p.C, p.F, parts, spec, keep_from(grid));
            return hipGetLastError();
        };
        if constexpr (sizeof(T) == 4 && V > 1) {
            if ((size_t)grid.x * grid.y <= 256) return go(k_frame_sums<T, V, 8>);
        }
        return go(k_frame_sums<T, V, 4>);
    });
}

hipError_t launch_anchor_scores(const ttf_params& p, const Workspace& w, const float* strip_sum, int strips, hipStream_t s)
{
    const int S = (p.C + 255) / 256;
    // runs of at least 32 frames, and no more blocks than fill the chip a few times
    int FG = 1;
    while (FG < 16 && (size_t)S * p.B * FG < 512 && p.F >= 64 * FG) FG *= 2;
    const unsigned grid = (unsigned)((size_t)S * p.B * FG);
    const bool mixed = strip_sum != nullptr;
    if (mixed && strips > 8) {
        k_reduce_strips<<<dim3((unsigned)(p.B * p.F), (unsigned)((p.C + 1023) / 1024)), 256, 0, s>>>(
            strip_sum, w.frame_sum, w.spec, p.F, p.C, strips);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const int parts = mixed ? 1 : frame_sum_parts(p, w);
    if (parts > 1)
        k_anchor_partials<true><<<grid, 1024, 0, s>>>(w.frame_sum, w.score_part, w.clip_part, p.F, p.C, S, FG, parts,
                                                      reinterpret_cast<const float*>(w.anchor_frag), nullptr);
    else if (mixed && strips <= 8)
        k_anchor_partials<true><<<grid, 1024, 0, s>>>(w.frame_sum, w.score_part, w.clip_part, p.F, p.C, S, FG, strips,
                                                      strip_sum, w.spec);
    else
        k_anchor_partials<false><<<grid, 1024, 0, s>>>(w.frame_sum, w.score_part, w.clip_part, p.F, p.C, S, FG, 1,
                                                       nullptr, nullptr);
    return hipGetLastError();
}

// Frame sums over the guess channels only (w.guess_sum), from which the anchor is guessed.
hipError_t launch_guess_sums(const ttf_params& p, const void* x, const Workspace& w, hipStream_t s)
{
    const int parts = guess_parts(p);
    auto go = [&](auto tag) {
        using T = decltype(tag);
        k_guess_sums<T><<<(unsigned)(p.B * p.F * parts), 256, 0, s>>>(static_cast<const T*>(x), w.guess_sum, p.H * p.W, p.C,
                                                                      parts);
        return hipGetLastError();
    };
    return p.dtype == TTF_BF16 ? go(bf16_t{}) : go(float{});
}

hipError_t launch_guess_pick(const ttf_params& p, const Workspace& w, hipStream_t s)
{
    if (p.F <= 32) k_guess_pick<4><<<(unsigned)p.B, 512, 0, s>>>(w.guess_sum, w.spec, p.F, guess_parts(p));
    else k_guess_pick<8><<<(unsigned)p.B, 512, 0, s>>>(w.guess_sum, w.spec, p.F, guess_parts(p));
    return hipGetLastError();
}

int fixed_frame(const ttf_params& p)
{
    if (p.anchor_mode != TTF_ANCHOR_FIXED) return -1;
    return p.anchor_index < 0 ? p.anchor_index + p.F : p.anchor_index;
}

hipError_t launch_tied_anchor(const ttf_params& p, const Workspace& w, int32_t* anchor_index, hipStream_t s)
{
    k_tied_anchor<<<1, 1024, 0, s>>>(w.score_part, w.clip_part, anchor_index, p.B, p.F, (p.C + 255) / 256,
                                     fixed_frame(p));
    return hipGetLastError();
}

hipError_t launch_anchor_norms(const ttf_params& p, const void* x, const void* ext_anchor, const Workspace& w,
                               int32_t* anchor_index, bool anchor_given, hipStream_t s)
{
    const int N = p.H * p.W;
    const int groups = (N + 3) / 4;
    const int fixed = anchor_given ? kAnchorGiven : fixed_frame(p);
    return by_layout(p, [&](auto tag, auto vtag) {
        using T = decltype(tag);
        constexpr int V = decltype(vtag)::value;
        k_anchor_norms<T, V><<<(unsigned)(p.B * groups), 256, 0, s>>>(
            static_cast<const T*>(x), static_cast<const T*>(ext_anchor), w.score_part, w.clip_part, anchor_index,
            w.anchor_inv, p.F, N, p.C,
            (p.C + 255) / 256, fixed, groups);
        return hipGetLastError();
    });
}

hipError_t launch_anchor_prepare_mfma(const ttf_params& p, const void* x, const void* ext_anchor, const Workspace& w,
                                      int32_t* anchor_index, int32_t* fuse_map, float* best_sim,
                                      int32_t* best_idx, bool anchor_given, hipStream_t s)
{
    const int N = p.H * p.W;
    const int fixed = anchor_given ? kAnchorGiven : fixed_frame(p);
    const bool pad = mfma_search_padded(p);
    const int CT = (p.W + 15) / 16;                          // column tiles per grid row
    const int tiles = pad ? p.H * CT : N / 16;
    auto go = [&](auto kernel) {
        kernel<<<(unsigned)(p.B * tiles), 512, 0, s>>>(static_cast<const uint16_t*>(x),
                                                       static_cast<const uint16_t*>(ext_anchor), w.score_part,
                                                       w.clip_part, anchor_index, w.anchor_inv, w.anchor_frag, fuse_map,
                                                       best_sim, best_idx, reinterpret_cast<uint16_t*>(w.keep_bits),
                                                       p.F, N, p.C, (p.C + 255) / 256, fixed, tiles, p.W, CT);
        return hipGetLastError();
    };
    return pad ? go(k_anchor_prepare<true>) : go(k_anchor_prepare<false>);
}

hipError_t launch_anchor_prepare_mfma_f32(const ttf_params& p, const void* x, const void* ext_anchor,
                                          const Workspace& w, int32_t* anchor_index, int32_t* fuse_map,
                                          float* best_sim, int32_t* best_idx, bool anchor_given, hipStream_t s)
{
    const int N = p.H * p.W;
    const int fixed = anchor_given ? kAnchorGiven : fixed_frame(p);
    const bool pad = !mfma_f32_aligned(p);
    const int CT = (p.W + 15) / 16;                          // column tiles per grid row
    const int tiles = pad ? p.H * CT : N / 16;
    auto go = [&](auto kernel) {
        kernel<<<(unsigned)(p.B * tiles), 512, 0, s>>>(static_cast<const float*>(x), static_cast<const float*>(ext_anchor),
                                                       w.score_part, w.clip_part, anchor_index, w.anchor_inv,
                                                       w.anchor_frag, fuse_map, best_sim, best_idx,
                                                       reinterpret_cast<uint16_t*>(w.keep_bits), p.F, N, p.C,
                                                       (p.C + 255) / 256, fixed, tiles, p.W, CT);
        return hipGetLastError();
    };
    return pad ? go(k_anchor_prepare_f32<true>) : go(k_anchor_prepare_f32<false>);
}

}  // namespace ttf
