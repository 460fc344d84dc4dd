// Internal declarations of the TTF library for gfx950: workspace layout and the launch
// functions behind ttf_compress.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "ttf.h"

namespace ttf {

constexpr int kWave = 64;

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// A launch may not have 2^32 threads or more: the most blocks of up to 256 threads.  Kernels that take
// a block per row are launched with at most this many blocks and walk on by the grid size.
constexpr size_t kMaxBlocks256 = (1u << 24) - 1;

// Lets `kernel` use `bytes` of dynamic LDS.  The limit is a property of the function on a device, so it
// is raised once (per function, device and size reached) and not on every launch.
hipError_t allow_dynamic_lds(const void* kernel, size_t bytes);
// fp32 tokens on the matrix cores (ttf_search_mfma_f32.hip): can this problem take them; is its grid one
// whose keep words the search writes itself (exactly 16 or 32 wide, whole 64-token words)
bool mfma_search_f32_supported(const ttf_params& p, int frames);   // `frames` searched per clip
bool mfma_f32_aligned(const ttf_params& p);

// Share of an input whose reads by the frame sums or the walk leave it in the caches for the kernel that reads it next; the
// search that follows walks (`walks`), or runs on the matrix cores (`mfma`), or neither.
double kept_share(const ttf_params& p, bool walks, bool mfma);

// Device scratch carved out of the caller's workspace.  All sections are 256-byte aligned.
struct Workspace {
    float*    frame_sum;     // [B,F,C]  sum over the N tokens of every frame (anchor rule, inner sum)
    double*   score_part;    // [B,S,F,2] per 256-channel slice: <frame sum, clip sum> and |frame sum|^2
    double*   clip_part;     // [B,S]    per slice: |clip sum|^2          (S = ceil(C/256))
    float*    anchor_inv;    // [B,NP]   1/||x_{a,j}|| of every anchor token (0 for a zero token); NP = token count
                             //          of the grid with rows padded to whole 16-column tiles (N when W % 16 == 0)
    uint16_t* anchor_frag;   // [B,NP/16,ceil(C/32),64,8] bf16 anchor frame in MFMA fragment order (matrix-core path);
                             // scratch of the walking search
    uint64_t* keep_bits;     // [B,F,NW] bit i%64 of word i/64 set iff token i is kept (NW=ceil(N/64))
    int32_t*  frame_base;    // [B,F]    output row of the first kept token of every frame
    int32_t*  src_row;       // [B*F*N]  input token (flat over clips and frames) that output row r copies
    // Speculative anchor (single pass over the input, see ttf_api.hip); sized 0 where it cannot apply
    float*    guess_sum;     // [B,F,P,kGuessChannels] frame sums over the guess channels only, in P = guess_parts()
                             // shares (one per run of tokens)
    int32_t*  spec;          // [B,4]    guessed anchor, guess trusted (1/0), unused
    float*    strip_sum;     // room for [B,F,spec_strips(),C] floats: frame sums per run of the grid and window
                             // products of the walking search (walk_scratch())
    size_t    frag_bytes;    // size of anchor_frag; until the anchor is chosen it holds the frame-sum shares
    size_t    strip_bytes;   // size of strip_sum
    bool      tail;          // anchor_frag holds the whole last K-step of tail_channels() rows
    size_t    bytes;
};

// Channels the anchor guess looks at: kGuessSegments runs of kGuessSegChannels channels, run j starting
// at channel (2j+1)*C/(2*kGuessSegments) rounded down to a multiple of kGuessSegChannels.
constexpr int kGuessSegments = 4;
constexpr int kGuessSegChannels = 64;
constexpr int kGuessChannels = kGuessSegments * kGuessSegChannels;
__host__ __device__ inline int guess_segment_start(int C, int j)
{
    return (int)(((long long)(2 * j + 1) * C / (2 * kGuessSegments)) / kGuessSegChannels * kGuessSegChannels);
}
// The guess sums of a frame are formed by this many blocks, each over a run of the frame's tokens (more
// blocks for big grids, so that few frames still fill the chip), and added when the guess is picked.
inline int guess_parts(const ttf_params& p)
{
    const long long n = (long long)p.H * p.W;
    return n >= 2048 ? 8 : (n >= 1024 ? 4 : (n >= 256 ? 2 : 1));   // (16x16 grids: 23 -> 16 us with two)
}
// Strips of 32 cells per frame: grids 16 or 32 wide N/32; two grid rows per strip up to 16 columns, one row per strip
// up to 32, ceil(column tiles / 2) per row beyond.  Measures the room for the search's sums and products.
inline long long spec_strips(const ttf_params& p)
{
    const bool aligned = (p.W == 16 && p.H % 4 == 0) || (p.W == 32 && p.H % 2 == 0);
    if (aligned) return (long long)p.H * p.W / 32;
    if (p.W <= 16) return (p.H + 1) / 2;
    return (long long)p.H * (((p.W + 15) / 16 + 1) / 2);
}
// Shapes the speculative anchor path exists for: bf16, C % 128 == 0, grids whose tokens fill at least 70 % of
// such strips (12..16, 23..32, 45..64 columns, ...), with at least 1024 channels, so that the guess
// channels are a small part of a row.  The radius is not looked at (the workspace must not depend on it).
inline bool speculation_shape(const ttf_params& p)
{
    if (p.dtype != TTF_BF16 || p.C % 128 != 0 || p.C < 1024 || p.F < 2) return false;
    return 10ll * p.H * p.W >= 7ll * 32 * spec_strips(p);
}
// ... and fp32 tokens in whole 32-channel K-steps with windows up to 3x3, whose sums, products and guess all stand in
// the fragment section.
inline bool speculation_possible(const ttf_params& p)
{
    if (p.dtype == TTF_F32) return p.C % 32 == 0 && p.C >= 1024 && p.F >= 2 && p.r <= 1;
    return speculation_shape(p);
}

// bf16 rows that are whole 16-byte pieces but not whole 32-channel K-steps: the matrix-core kernels end
// on a K-step whose missing channels count as zero.  From 768 channels on: much shorter rows keep the
// wave-per-token kernels, whose sums are then the more exact ones (relative error of the similarities against
// 64 bits, matrix cores over wave-per-token, the same within 0.02 for every radius and column layout: C 264
// 1.06, 360 1.07, 520 0.97, 744 0.96, 776 0.96, 872 0.94, 1016 0.82, 2040 0.85, 4072 0.81).
inline bool tail_channels(const ttf_params& p)
{
    return p.dtype == TTF_BF16 && p.C % 32 != 0 && p.C % 8 == 0 && p.C >= 768;
}

// tail: with room for the whole last K-step of tail_channels() rows in the anchor's fragment copy.
// Without it the workspace is a little smaller and such rows take the general kernels (callers whose
// workspace is that small: the fixed one, or one sized for the rows as they are; calls without a search).
inline Workspace carve(const ttf_params& p, void* base, bool tail = true)
{
    const size_t B = p.B, F = p.F, N = (size_t)p.H * p.W, C = p.C, NW = (N + 63) / 64;
    const size_t NP = (size_t)p.H * ((p.W + 15) / 16) * 16;   // grid rows padded to whole 16-column tiles
    size_t off = 0;
    auto take = [&](size_t n) { size_t o = off; off = align_up(off + n, 256); return o; };
    const size_t o_fs = take(B * F * C * sizeof(float));
    const size_t S = (C + 255) / 256;
    const size_t o_sp = take(B * S * F * 2 * sizeof(double));
    const size_t o_cp = take(B * S * sizeof(double));
    const size_t o_ai = take(B * NP * sizeof(float));
    // anchor frame in fragment order: bf16 as is, fp32 as three bf16 planes (where the matrix-core path can run)
    const bool whole = tail && tail_channels(p);
    const size_t o_af = take(p.dtype == TTF_BF16 ? B * NP * (whole ? align_up(C, 32) : C) * sizeof(uint16_t)
                                                 : (C % 32 == 0 ? 3 * B * NP * C * sizeof(uint16_t) : 0));
    const size_t o_kb = take(B * F * NW * sizeof(uint64_t));
    const size_t o_fb = take(B * F * sizeof(int32_t));
    const size_t o_sr = take(B * F * N * sizeof(int32_t));
    const bool spec = speculation_shape(p);
    const size_t o_gs = take(spec ? B * F * guess_parts(p) * kGuessChannels * sizeof(float) : 0);
    const size_t o_sp2 = take(spec ? B * 4 * sizeof(int32_t) : 0);
    const size_t o_ss = take(spec ? B * F * (size_t)spec_strips(p) * C * sizeof(float) : 0);
    char* c = static_cast<char*>(base);
    Workspace w;
    w.frame_sum   = reinterpret_cast<float*>(c + o_fs);
    w.score_part  = reinterpret_cast<double*>(c + o_sp);
    w.clip_part   = reinterpret_cast<double*>(c + o_cp);
    w.anchor_inv  = reinterpret_cast<float*>(c + o_ai);
    w.anchor_frag = reinterpret_cast<uint16_t*>(c + o_af);
    w.keep_bits   = reinterpret_cast<uint64_t*>(c + o_kb);
    w.frame_base  = reinterpret_cast<int32_t*>(c + o_fb);
    w.src_row     = reinterpret_cast<int32_t*>(c + o_sr);
    w.guess_sum   = reinterpret_cast<float*>(c + o_gs);
    w.spec        = reinterpret_cast<int32_t*>(c + o_sp2);
    w.strip_sum   = reinterpret_cast<float*>(c + o_ss);
    w.frag_bytes = o_kb - o_af;
    w.strip_bytes = off - o_ss;
    w.tail = whole;
    w.bytes = off;
    return w;
}

// Stage launchers.  Each enqueues on `s` and returns the launch status.
// `skip_trusted`: clips with a trusted anchor guess (w.spec) are left out.  `kept`: share of the input left in the
// Infinity Cache.
hipError_t launch_frame_sums(const ttf_params& p, const void* x, const Workspace& w, bool skip_trusted, double kept,
                             hipStream_t s);
// Per-slice shares of the anchor scores from w.frame_sum; with strip_sum [B,F,strips,C]: from there for the clips
// with a trusted anchor guess.
hipError_t launch_anchor_scores(const ttf_params& p, const Workspace& w, const float* strip_sum, int strips, hipStream_t s);
// The anchor guessed from w.guess_sum: w.spec[b] = {guess, trusted, 0, 0}.
hipError_t launch_guess_pick(const ttf_params& p, const Workspace& w, hipStream_t s);
// Frame sums over the guess channels only (w.guess_sum).
hipError_t launch_guess_sums(const ttf_params& p, const void* x, const Workspace& w, hipStream_t s);
// `ext_anchor` (here and below): nullptr when the anchor is a frame of x; otherwise the anchor
// frames [B,N,C] of a segment, in which case anchor_index is written as -1 and every frame of x
// is a source frame.
// `anchor_given`: the anchor of every clip is already in anchor_index (tied-batch mode); it is
// read, not chosen.
hipError_t launch_anchor_norms(const ttf_params& p, const void* x, const void* ext_anchor, const Workspace& w,
                               int32_t* anchor_index, bool anchor_given, hipStream_t s);
// Matrix-core path: anchor choice, inverse norms, the anchor frame re-laid in fragment order, and
// the anchor-frame rows of fuse_map / best_sim / best_idx / keep bits.
hipError_t launch_anchor_prepare_mfma(const ttf_params& p, const void* x, const void* ext_anchor, const Workspace& w,
                                      int32_t* anchor_index, int32_t* fuse_map, float* best_sim,
                                      int32_t* best_idx, bool anchor_given, hipStream_t s);
// The same for fp32 tokens: the anchor frame as three bf16 planes per tile and K-step.
hipError_t launch_anchor_prepare_mfma_f32(const ttf_params& p, const void* x, const void* ext_anchor,
                                          const Workspace& w, int32_t* anchor_index, int32_t* fuse_map,
                                          float* best_sim, int32_t* best_idx, bool anchor_given, hipStream_t s);
bool mfma_search_supported(const ttf_params& p);   // grids exactly 16 or 32 wide with whole keep words
bool mfma_search_padded(const ttf_params& p);      // every other grid (tile rows padded to 16 columns)
bool tail_search_pays(const ttf_params& p, int frames);   // tail_channels() rows: large enough for them
hipError_t launch_window_search(const ttf_params& p, const void* x, const void* ext_anchor, const Workspace& w,
                                const int32_t* anchor_index, int32_t* fuse_map, float* best_sim,
                                int32_t* best_idx, float* win_sim, hipStream_t s);
// Search by workgroups that walk whole frames (ttf_search_walk.hip): how it is dealt to workgroups, and its
// scratch, which lies in the sections strip_sum and anchor_frag.
struct WalkPlan {
    bool ok;                 // the kernels can run this problem
    bool patch;              // tiles are 4x4 patches, not runs of a grid row
    int nk;                  // shares of the channels
    int lines;               // column strips of the grid
    int lsegs, ysegs;        // runs of strips, and runs of rows, dealt to different workgroups
    int groups, nf;          // frame groups of nf frames
    double tiles;            // time of a workgroup, in tiles
};
struct WalkDeal {
    int lsegs, ysegs, groups, nf;   // as in WalkPlan
};
// The guessed anchor: microseconds that it saves where every clip has a clear guess, and that it costs where it is dropped, and how
// many clips have to have a clear one for any to be taken.
struct GuessCost {
    double saves, dropped;
    int min_trusted;
};
struct WalkScratch {
    float* part;             // [nk][B*F*N][(2r+1)^2 + 1]
    float* norm_part;        // [nk][B*N]
    float* strip_sum;        // [B*F][lsegs*ysegs][C], where sums are kept (frame_sum for a single run)
    float* guess_sum;        // the sections of the same names (in the fragment section for fp32 tokens)
    int32_t* spec;
};
WalkPlan walk_plan(const ttf_params& p, int frames, bool sums);
GuessCost guess_cost(const ttf_params& p, const WalkPlan& first, const WalkPlan& again);
bool walk_scratch(const ttf_params& p, const Workspace& w, const WalkPlan& plan, bool sums, WalkScratch& scratch);
// Whether a problem with a workspace of ttf_workspace_size() bytes is searched so (ttf_api.hip).
bool search_walks(const ttf_params& p, bool external_anchor);
// How many of its clips have to have a clear guess for their anchors to be guessed, with the setting `mode` of
// ttf_set_speculation(); -1: the anchors are not guessed.
int search_guesses(const ttf_params& p, int mode);
// mode 0: anchor external, fixed, given or picked from the scores.  1: clips with a trusted guess, every frame,
// with sums; fewer such clips than min_trusted lose their mark.  2: clips whose guess the
// exact rule refutes, and those without one; dealt as in `all` where no clip has a trusted guess.
hipError_t launch_search_walk(const ttf_params& p, const void* x, const void* ext_anchor, const Workspace& w,
                              const WalkPlan& plan, const WalkPlan& all, const WalkScratch& scratch, int32_t* anchor_index,
                              bool anchor_given, int mode, int min_trusted, hipStream_t s);
// Similarities, arg max, gate and keep words from the walk's products (win_sim: tied-batch mode, see k_tie).
hipError_t launch_walk_finish(const ttf_params& p, const Workspace& w, const WalkPlan& plan, const WalkScratch& scratch,
                              const int32_t* anchor_index, int32_t* fuse_map, float* best_sim, int32_t* best_idx,
                              float* win_sim, hipStream_t s);
int fixed_frame(const ttf_params& p);              // the fixed anchor frame, or -1 for the automatic rule
// Keep words rebuilt from the fuse map (for searches whose work units do not line up with keep words).
hipError_t launch_pack_keep(const ttf_params& p, const int32_t* fuse_map, const int32_t* anchor_index,
                            const Workspace& w, hipStream_t s);
// Output row offsets; launches nothing where the emission counts them itself.
hipError_t launch_offsets_scan(const ttf_params& p, const Workspace& w, const int32_t* anchor_index,
                               int32_t* kept_count, int32_t* row_offsets, bool tied, hipStream_t s);
// Output rows, ids and -- where launch_offsets_scan leaves that to it -- kept_count and row_offsets.
hipError_t launch_emit_rows(const ttf_params& p, const void* x, const Workspace& w, const int32_t* anchor_index,
                            int32_t* kept_count, int32_t* row_offsets, void* tokens_out, int32_t* pos_ids,
                            int32_t* src_index, int frame_offset, bool tied, hipStream_t s);

// Tied-batch mode.  Workspace behind the common sections: every window similarity of every
// element, and the two row offsets of the shared mask.
struct TiedWorkspace {
    Workspace base;
    float*    win_sim;       // [B,F,(2r+1)^2,N]
    int32_t*  row_offsets;   // [2]
    size_t    bytes;
};
inline TiedWorkspace carve_tied(const ttf_params& p, void* base, bool tail = true)
{
    TiedWorkspace t;
    t.base = carve(p, base, tail);
    const size_t K = (size_t)(2 * p.r + 1) * (2 * p.r + 1);
    const size_t o_ws = t.base.bytes;
    const size_t o_ro = align_up(o_ws + (size_t)p.B * p.F * p.H * p.W * K * sizeof(float), 256);
    char* c = static_cast<char*>(base);
    t.win_sim = reinterpret_cast<float*>(c + o_ws);
    t.row_offsets = reinterpret_cast<int32_t*>(c + o_ro);
    t.bytes = o_ro + 256;
    return t;
}
// The shared anchor (batch-mean score, or the fixed frame) written to every entry of anchor_index.
hipError_t launch_tied_anchor(const ttf_params& p, const Workspace& w, int32_t* anchor_index, hipStream_t s);
// Shared offset, per-element s^, united keep mask (keep bits [F,NW] at the start of w.keep_bits).
hipError_t launch_tie(const ttf_params& p, const Workspace& w, const float* win_sim, const int32_t* anchor_index,
                      int32_t* fuse_map, float* best_sim, int32_t* best_idx, float* mean_sim, hipStream_t s);

// Restoration: map from every original token to the compressed row that stands for it, and the
// gather that rebuilds the full layout.
hipError_t launch_restore_map(const ttf_params& p, const int32_t* fuse_map, const int32_t* row_offsets,
                              const int32_t* src_index, int32_t* restore_map, hipStream_t s);
hipError_t launch_restore_rows(const ttf_params& p, const void* tokens, long long rows,
                               const int32_t* restore_map, void* restored, hipStream_t s);
// Adaptive threshold: exact order statistic of the source similarities per clip, and the gate
// redone from stored similarities (fills fuse_map and the keep bits).
// keep_fraction = 1 - requested fused fraction (double); the rank is formed per clip on the device,
// from the clip's own number of source tokens.
hipError_t launch_select_threshold(const ttf_params& p, const float* best_sim, const int32_t* anchor_index,
                                   double keep_fraction, float* thresholds, hipStream_t s);
hipError_t launch_regate(const ttf_params& p, const Workspace& w, const float* best_sim, const int32_t* best_idx,
                         const int32_t* anchor_index, const float* thresholds, int32_t* fuse_map, hipStream_t s);

}  // namespace ttf
