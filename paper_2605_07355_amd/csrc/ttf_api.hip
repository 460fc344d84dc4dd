// C ABI of the TTF library: argument checks, workspace carving, the launch sequence of
// Section 3 (anchor selection -> window search + gate -> offsets -> row emission) and the
// optional per-stage event timing.  Nothing here allocates device memory.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <utility>

#include "ttf_internal.h"

namespace ttf {

hipError_t launch_window_search_generic(const ttf_params& p, const void* x, const void* ext_anchor, const Workspace& w,
                                        const int32_t* anchor_index, int32_t* fuse_map, float* best_sim,
                                        int32_t* best_idx, float* win_sim, hipStream_t s);

hipError_t launch_window_search_mfma(const ttf_params& p, const void* x, bool external_anchor, const Workspace& w,
                                     const int32_t* anchor_index, int32_t* fuse_map, float* best_sim,
                                     int32_t* best_idx, float* win_sim, hipStream_t s);
hipError_t launch_window_search_mfma_f32(const ttf_params& p, const void* x, bool external_anchor, const Workspace& w,
                                         const int32_t* anchor_index, int32_t* fuse_map, float* best_sim,
                                         int32_t* best_idx, float* win_sim, hipStream_t s);

// bf16 and fp32 tokens with r <= 2 and C % 32 == 0 take the matrix-core kernels (grids exactly 16 or 32
// wide with whole keep words the aligned ones, every other grid the padded-tile ones), bf16 tokens also with
// the channel counts of tail_channels() where the workspace has room for them (`tail`) and it pays for the
// frames that are walked (all of them against an external anchor, all but the anchor otherwise); larger
// radii and other channel counts take the general wave-per-token kernel.  The environment variable
// TTF_SEARCH=general, read once per process, forces the general kernels (for comparisons).
static bool forced_general()
{
    static const bool general = [] {
        const char* force = std::getenv("TTF_SEARCH");
        return force && std::strcmp(force, "general") == 0;
    }();
    return general;
}

bool use_mfma_path(const ttf_params& p, bool tail, bool external_anchor)
{
    const int frames = external_anchor ? p.F : p.F - 1;      // (a segment takes the search of the clip it equals)
    if (forced_general() || (tail_channels(p) && !(tail && tail_search_pays(p, frames)))) return false;
    return mfma_search_supported(p) || mfma_search_padded(p) || mfma_search_f32_supported(p, frames);
}

// Anchor preparation of the matrix-core path for the element type at hand (fp32: three bf16 planes).
hipError_t launch_anchor_prepare_any(const ttf_params& p, const void* x, const void* ext_anchor, const Workspace& w,
                                     int32_t* anchor_index, int32_t* fuse_map, float* best_sim, int32_t* best_idx,
                                     bool anchor_given, hipStream_t s)
{
    if (p.dtype == TTF_F32)
        return launch_anchor_prepare_mfma_f32(p, x, ext_anchor, w, anchor_index, fuse_map, best_sim, best_idx,
                                              anchor_given, s);
    return launch_anchor_prepare_mfma(p, x, ext_anchor, w, anchor_index, fuse_map, best_sim, best_idx, anchor_given,
                                      s);
}

hipError_t launch_window_search(const ttf_params& p, const void* x, const void* ext_anchor, const Workspace& w,
                                const int32_t* anchor_index, int32_t* fuse_map, float* best_sim,
                                int32_t* best_idx, float* win_sim, hipStream_t s)
{
    if (use_mfma_path(p, w.tail, ext_anchor != nullptr)) {
        if (p.dtype == TTF_F32)
            return launch_window_search_mfma_f32(p, x, ext_anchor != nullptr, w, anchor_index, fuse_map, best_sim,
                                                 best_idx, win_sim, s);
        return launch_window_search_mfma(p, x, ext_anchor != nullptr, w, anchor_index, fuse_map, best_sim, best_idx,
                                         win_sim, s);
    }
    return launch_window_search_generic(p, x, ext_anchor, w, anchor_index, fuse_map, best_sim, best_idx, win_sim, s);
}

// Whether the search walks whole frames (ttf_search_walk.hip).  Its workgroups are few
// and long, so it starts slower and streams faster; against the kernels above it also does without the launch that
// copies the anchor frame, and adds the one that forms the similarities.  Where the lines lie (whole calls, bf16,
// r 0..2, 130 random shapes; time of the kernels above over the walk's):
//   tile rows padded to 16 columns, C >= 1024: 0.99 to 2.2 at every size (B1 F23 9x14 C1792 54.2 / 33.8 us, B1 F5 32x23
//     C4096 r2 106 / 48.5, B8 F59 10x16 C2048 216 / 189); shorter rows 0.91 to 1.14.  Without the anchor rule, whose sums leave
//     the end of the input in the cache, C < 1536 also 0.90 to 1.27 with the 5x5 window and up to 16 columns (40 segments and tied
//     batches, 1.04 on average; segment B4 F135 14x14 C1152 85 / 94, tied B8 F23 18x14 C1088 94 / 103): one rule for all calls.
//   aligned 16- and 32-wide grids: 0.78 to 0.97 on small calls (B1 F10 16x16 C2048 27.2 / 34.8, B1 F32 32x32 C1024 58 /
//     67), 1.0 to 1.3 from 96 MiB on (B6 F17 16x16 C3584 111 / 103, B4 F20 16x16 C3584 r0 95 / 83), with three strips in a row of
//     32 from 160 MiB (B2 F6 32x32 C2048 53 / 61, B5 F9 32x32 C3072 172 / 145); the 5x5 window from 24 MiB (B5 F14 16x16
//     C1792 68.5 / 59.0), and rows whose K-steps do not divide over the waves there from 32 MiB (B2 F15 16x16 C2624 61.1 / 49.8).
//   the 5x5 window, 16 wide: 0.95 to 1.2 from 24 to 64 MiB (85 shapes; B4 F5 88x16 C1280 75 / 65, segment B2 F9 48x16 C2304 37 /
//     44), but up to 48 MiB not where the walk makes fewer than 256 workgroups of such a problem: 102 shapes 0.96 on average, 0.80 to
//     1.26 (segment B2 F17 24x16 C1024 25 / 29, B1 F10 48x16 C2048 38 / 45); with 256 28 shapes 1.01 (C 3072 and 4096 0.98 to 1.2).
//     Grids of two rows fill half of every patch, and whole strips of the kernels above: C < 1536 from 32 MiB
//     0.75 to 0.98 (segment B64 F40 2x16 C1024 66 / 88, B32 F24 2x12 C1152 37 / 42), longer rows from 96 MiB 0.88 to 1.03
//     (B64 F24 2x14 C1536 61 / 69), below 1.0 to 1.4.
// fp32 tokens, windows up to 3x3 (90 shapes): against the matrix-core search 1.02 to 2.8 from C 1024 on (B3 F7 16x21 C1024
//   73 / 50 us, B2 F21 16x13 C4096 264 / 94, B16 F14 16x16 C3072 387 / 314), 0.84 to 1.57 below; against the wave-per-token
//   search of small problems from 32 MiB and C 768 on 0.97 to 1.9 (B1 F12 16x16 C3072 64 / 48), below 32 MiB 0.6 to 1.4.
//   Rows of 32 cells are three strips of 11: arithmetic for 33 of every 48 cells only.  From 480 MiB on that bounds them where the
//   32-channel groups do not divide over the waves either (B1 F33 64x32 C3424, 107 groups over 32 waves, 503 / 539; B8 F33 32x32 C832
//   526 / 551; B8 F17 16x32 C3200 tied 519 / 540); where they do 0.99 to 1.13 (B1 F73 32x32 C3584 583 / 518), below 480 MiB 0.93 to 2.3
//   (B2 F17 32x32 C2560 230 / 246, segment B2 F33 16x32 C3104 237 / 199).
static bool use_walk(const ttf_params& p, const Workspace& w, bool mfma, bool external_anchor, WalkPlan& plan,
                     WalkScratch& scratch)
{
    const int frames = external_anchor ? p.F : p.F - 1;      // (a segment takes the search of the clip it equals)
    const size_t mib = ((size_t)p.B * frames * p.H * p.W * p.C * (p.dtype == TTF_BF16 ? 2 : 4)) >> 20;
    if (p.dtype == TTF_F32) {
        if (forced_general() || !((mfma && p.C >= 1024) || (p.C >= 768 && mib >= 32))) return false;
        const int groups = p.C / 32, waves = 8 * ((groups + 31) / 32);
        if (p.W == 32 && p.r == 1 && mfma_f32_aligned(p) && mib >= 480 && 100 * groups < 85 * waves * ((groups + waves - 1) / waves))
            return false;
    } else {
        if (!mfma || p.C < 1024) return false;
        if (mfma_search_supported(p) &&
            mib < (size_t)(p.r == 2 ? 24 : (p.C % 256 != 0 ? 32 : (p.W == 32 && p.r == 1 ? 160 : 96))))
            return false;
    }
    if (p.r == 2 && p.H == 2 && p.C < 2048 && mib >= (size_t)(p.C < 1536 ? 32 : 96)) return false;
    plan = walk_plan(p, frames, false);
    if (!plan.ok) return false;
    if (p.r == 2 && p.W == 16 && p.C < 2560 && mfma_search_supported(p) && mib < 48 &&
        (size_t)p.B * plan.nk * plan.groups * plan.lsegs * plan.ysegs < 256)
        return false;
    // The products of all frames have to fit the workspace at once.  A segment's workspace is that of F frames, its
    // clip's that of F + 1: asked is whether they fit the clip's, where there is less room for a frame.
    ttf_params clip = p;
    clip.F = frames + 1;
    WalkScratch fits{};
    return walk_scratch(clip, carve(clip, nullptr), plan, false, fits) && walk_scratch(p, w, plan, false, scratch);
}

// Inputs, or the end of a pass over larger ones, are left in the Infinity Cache (256 MiB): plain
// loads instead of non-temporal ones, for a little more than fits where the input does not.
// B2 F256 16x16 C4096 (1 GiB): frame sums 161 us either way and the search behind them 174 -> 162, with 1 GiB of plain
// loads 179 and 162; B4 F32 16x16 C4096 (256 MiB): sums 42.8 -> 41.5, search 47.8 -> 44.6, row copy 33.8 -> 29.9.  Searches
// that read with plain loads themselves (`walks` false) push out the end of a larger input before they reach it: there
// it costs (B2 F256 32x23 C384, 276 MiB: sums 44 -> 50, whole call 278 -> 295).
// The wave-per-token search gains by it too from 16 MiB on (90 shapes, 2 to 20 %).  Below, where most of the input still stands
// in some XCD's L2 when the search starts, it can be slower: kernel 34.5 -> 46 us, B1 F4 14x16 C4096 fp32.  (That it comes with
// the plain loads is measured; that it is the lines in other XCDs' L2s is a guess.)  From 6 to 16 MiB a call takes 0.89 to 1.34
// times what it takes with non-temporal loads (118 shapes, mean 1.006; fp32 B1 F3 16x14 C4096 52 / 68, B1 F7 32x16 C896 r 3
// 70 / 78, but B2 F2 14x32 C2048 59.5 / 53), on less there is no difference.
double kept_share(const ttf_params& p, bool walks, bool mfma)
{
    const double bytes = (double)p.B * p.F * p.H * p.W * p.C * (p.dtype == TTF_BF16 ? 2 : 4);
    const double mib = 1 << 20;
    if (!walks && !mfma && bytes < 16 * mib) return 0.0;
    if (!walks) return bytes <= 256 * mib ? 1.0 : 0.0;
    return bytes <= 320 * mib ? 1.0 : 320 * mib / bytes;
}

bool search_walks(const ttf_params& p, bool external_anchor)
{
    const Workspace w = carve(p, nullptr);
    WalkPlan plan{};
    WalkScratch scratch{};
    return use_walk(p, w, use_mfma_path(p, w.tail, external_anchor), external_anchor, plan, scratch);
}

// Speculative anchor: -1 never, 1 whenever the shape allows, 0 where it is expected to pay (two-pass / with the guess below, us):
//  * inputs of 256 MiB and more;
//  * clips of 12 to 128 frames.  Shorter ones clear the trust gap too seldom (B32 F4 16x16 C4096 150 / 177, none of 32;
//    B16 F12 203 / 163 and B16 F15 242 / 195, all of 16), longer ones hardly ever.
//  * clips of more than 64 frames are as often of several scenes, which have no clear guess, as of one, and neither is known
//    before the call: there the guess has to save half as much again as one that is dropped costs, by guess_cost().  One
//    scene, then scenes of 32 frames: B8 F128 16x16 C4096 968 / 672 and 1351 / 1398, B16 F66 16x16 C2048 489 / 422 and 602 / 647,
//    B8 F72 16x16 C4096 r 0 494 / 403 and 639 / 674; not where that is not expected: B4 F100 24x24 C2048 408 / 378 and 552 / 593,
//    B3 F117 9x16 C3584 184 / 172 and 236 / 268, B14 F84 20x28 C1024 r 0 595 / 560 and 766 / 845.
//  * where the model of the two ways, guess_cost(), has it save anything;
//  * fp32 on grids of one strip: with sums it is bound by its arithmetic, which strips of 11 cells do not fill (B6 F32
//    16x32 C2048 449 / 478, B16 F32 16x16 C4096 944 / 749).
// Where too few clips of a batch have a clear guess, all are dropped on the device (min_trusted): B8 F20 24x24 C2048, 6 of 8
// clear, 195 two-pass, 290 with the guesses, 226 with them dropped; B16 F32 16x16 C4096, 4 of 16, 561 / 683 / 591.
constexpr unsigned long long kSpeculationMinBytes = 256ull << 20;
constexpr int kSpeculationMinFrames = 12, kSpeculationSceneFrames = 64, kSpeculationMaxFrames = 128;

// Whether the anchor of a clip that walks (use_walk()) is guessed first, and the deal and scratch of the walk that
// then keeps sums.  Only such clips: one that took the walk beside a guess and another search without one would have
// the bits of its similarities depend on the setting.
// `plan` comes as that of use_walk(), the search without a guess, and goes as that of the walk beside one.
static bool use_guess(const ttf_params& p, const Workspace& w, bool mfma, int mode, WalkPlan& plan, WalkScratch& scratch,
                      int& min_trusted)
{
    if (p.anchor_mode != TTF_ANCHOR_AUTO || !mfma || !speculation_possible(p) || mode < 0) return false;
    if (mode == 0) {
        const unsigned long long bytes = (unsigned long long)p.B * p.F * p.H * p.W * p.C * (p.dtype == TTF_BF16 ? 2ull : 4ull);
        if (bytes < kSpeculationMinBytes || p.F < kSpeculationMinFrames || p.F > kSpeculationMaxFrames ||
            (p.dtype == TTF_F32 && p.W > 16))
            return false;
    }
    const WalkPlan with_sums = walk_plan(p, p.F, true);
    WalkScratch its{};
    if (!with_sums.ok || !walk_scratch(p, w, with_sums, true, its)) return false;
    min_trusted = 0;                                         // (forced: however few)
    if (mode == 0) {
        const GuessCost cost = guess_cost(p, with_sums, plan);
        if (cost.saves < (p.F > kSpeculationSceneFrames ? 1.5 * cost.dropped : 0.0)) return false;
        min_trusted = cost.min_trusted;
    }
    plan = with_sums;
    scratch = its;
    return true;
}

int search_guesses(const ttf_params& p, int mode)
{
    const Workspace w = carve(p, nullptr);
    const bool mfma = use_mfma_path(p, w.tail, false);
    WalkPlan plan{};
    WalkScratch scratch{};
    int min_trusted = 0;
    return use_walk(p, w, mfma, false, plan, scratch) && use_guess(p, w, mfma, mode, plan, scratch, min_trusted) ? min_trusted : -1;
}

hipError_t allow_dynamic_lds(const void* kernel, size_t bytes)
{
    static std::mutex mutex;
    static std::map<std::pair<const void*, int>, size_t> granted;   // (function, device) -> bytes allowed so far
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mutex);
    size_t& have = granted[{kernel, dev}];
    if (bytes <= have) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) have = bytes;
    return e;
}

namespace {

thread_local int g_last_hip_error = 0;

std::atomic<int> g_speculation{0};

// Event sets for stage timing: `slots` sets of TTF_NUM_STAGES+1 events, used round-robin by
// successive profiled calls so that a benchmark can time many calls and read them afterwards.
struct Profile {
    int slots = 0;                 // 0 = profiling off
    int created = 0;               // event sets that exist
    long long calls = 0;           // profiled calls since enabling
    hipEvent_t ev[TTF_PROFILE_MAX_SLOTS][TTF_NUM_STAGES + 1];
};
thread_local Profile g_prof;

ttf_status check_params(const ttf_params* p)
{
    if (!p) return TTF_ERR_INVALID_ARG;
    if (p->B < 1 || p->F < 1 || p->H < 1 || p->W < 1 || p->C < 1) return TTF_ERR_INVALID_ARG;
    const long long tokens = (long long)p->B * p->F * p->H * p->W;
    if ((long long)p->H * p->W >= (1ll << 31) || tokens >= (1ll << 31)) return TTF_ERR_INVALID_ARG;
    if (p->C > (1 << 21)) return TTF_ERR_INVALID_ARG;       // keeps every launch grid inside HIP limits
    // every launch stays below 2^32 threads: the densest grids take a 256-thread block per 16 tokens of a
    // frame rounded up to whole 64-token keep words, or per 4 anchor tokens
    if ((long long)p->B * p->F * (((long long)p->H * p->W + 63) / 64) * 64 >= (1ll << 25)) return TTF_ERR_INVALID_ARG;
    if (p->r < 0) return TTF_ERR_INVALID_ARG;
    if (!std::isfinite(p->t)) return TTF_ERR_INVALID_ARG;
    if (p->anchor_mode != TTF_ANCHOR_AUTO && p->anchor_mode != TTF_ANCHOR_FIXED) return TTF_ERR_INVALID_ARG;
    if (p->anchor_mode == TTF_ANCHOR_FIXED && (p->anchor_index < -p->F || p->anchor_index >= p->F))
        return TTF_ERR_INVALID_ARG;
    if (p->dtype != TTF_BF16 && p->dtype != TTF_F32) return TTF_ERR_UNSUPPORTED;
    return TTF_OK;
}

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

}  // namespace
}  // namespace ttf

using namespace ttf;

extern "C" {

ttf_status ttf_workspace_size(const ttf_params* params, size_t* bytes)
{
    if (!bytes) return TTF_ERR_INVALID_ARG;
    const ttf_status st = check_params(params);
    if (st != TTF_OK) return st;
    *bytes = carve(*params, nullptr).bytes;
    return TTF_OK;
}

// The launch sequence behind ttf_compress (ext_anchor == nullptr) and ttf_compress_segment.
static ttf_status run_pass(const ttf_params* params, const void* features, const void* ext_anchor,
                           int frame_offset, void* workspace, size_t workspace_bytes, const ttf_outputs* out,
                           void* hip_stream)
{
    const ttf_status st = check_params(params);
    if (st != TTF_OK) return st;
    if (!features || !workspace || !out) return TTF_ERR_INVALID_ARG;
    if (!out->tokens_out || !out->pos_ids || !out->src_index || !out->row_offsets || !out->kept_count ||
        !out->anchor_index || !out->fuse_map)
        return TTF_ERR_INVALID_ARG;
    if (!aligned(features, 16) || !aligned(out->tokens_out, 16) || !aligned(workspace, 256))
        return TTF_ERR_UNSUPPORTED;
    if (ext_anchor && !aligned(ext_anchor, 16)) return TTF_ERR_UNSUPPORTED;

    ttf_params p = *params;
    p.r = std::min(p.r, std::max(p.H, p.W));                 // beyond the grid = whole grid
    Workspace w = carve(p, workspace);
    if (workspace_bytes < w.bytes) w = carve(p, workspace, false);
    if (workspace_bytes < w.bytes) return TTF_ERR_WORKSPACE_TOO_SMALL;
    const bool mfma = use_mfma_path(p, w.tail, ext_anchor != nullptr);
    const bool pick = !ext_anchor && p.anchor_mode == TTF_ANCHOR_AUTO;       // the automatic anchor rule runs

    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    Profile& prof = g_prof;
    const bool timing = prof.slots > 0;
    hipEvent_t* ev = timing ? prof.ev[prof.calls % prof.slots] : nullptr;
    hipError_t e = hipSuccess;
    int stage = 0;
    auto mark = [&]() {
        if (timing && e == hipSuccess) e = hipEventRecord(ev[stage], s);
        ++stage;
    };
#define TTF_STEP(call)                 \
    do {                               \
        if (e == hipSuccess) e = (call); \
    } while (0)

    // The automatic anchor rule needs the sum of every frame, i.e. a pass over the whole input before
    // the search can start.  Large inputs on the matrix-core path avoid that pass: the rule is
    // first evaluated on a few channels only (4 x 128 bytes of every token row); where that guess wins
    // clearly the search runs against it at once and adds up, on the side, the exact sums of every
    // frame it reads.  The exact rule is then evaluated from those sums: it confirms the
    // guess (the usual case: nothing else to do) or refutes it, and then the clip's search is repeated
    // against the exact anchor.  A clip whose guess is not clear-cut sits out the first search; its
    // frame sums are then formed the two-pass way and it is searched with the refuted clips.  Either way
    // every output is what the exact rule gives.
    WalkPlan plan{};
    WalkScratch scratch{};
    const bool walk = use_walk(p, w, mfma, ext_anchor != nullptr, plan, scratch);
    const WalkPlan again = plan;
    int min_trusted = 0;
    const bool spec = walk && pick &&
                      use_guess(p, w, mfma, g_speculation.load(std::memory_order_relaxed), plan, scratch, min_trusted);
    if (spec) {
        w.guess_sum = scratch.guess_sum;
        w.spec = scratch.spec;
    }

    mark();                                                    // start of stage 0
    if (spec) TTF_STEP(launch_guess_sums(p, features, w, s));
    else if (pick) TTF_STEP(launch_frame_sums(p, features, w, false, kept_share(p, walk, mfma), s));
    mark();
    if (pick && !spec) TTF_STEP(launch_anchor_scores(p, w, nullptr, 0, s));
    mark();
    if (spec) TTF_STEP(launch_guess_pick(p, w, s));
    else if (!walk && mfma)                                    // (a walking search picks the anchor and forms its norms)
        TTF_STEP(launch_anchor_prepare_any(p, features, ext_anchor, w, out->anchor_index, out->fuse_map,
                                           out->best_sim, out->best_idx, false, s));
    else if (!walk) TTF_STEP(launch_anchor_norms(p, features, ext_anchor, w, out->anchor_index, false, s));
    mark();
    if (walk) {
        TTF_STEP(launch_search_walk(p, features, ext_anchor, w, plan, plan, scratch, out->anchor_index, false, spec ? 1 : 0,
                                    min_trusted, s));
        if (!spec)
            TTF_STEP(launch_walk_finish(p, w, plan, scratch, out->anchor_index, out->fuse_map, out->best_sim, out->best_idx,
                                        nullptr, s));
    } else {
        TTF_STEP(launch_window_search(p, features, ext_anchor, w, out->anchor_index, out->fuse_map, out->best_sim,
                                      out->best_idx, nullptr, s));
    }
    mark();
    if (spec) {
        TTF_STEP(launch_frame_sums(p, features, w, true, kept_share(p, true, mfma), s));     // clips without a trusted guess only
        TTF_STEP(launch_anchor_scores(p, w, scratch.strip_sum, plan.lsegs * plan.ysegs, s));
        TTF_STEP(launch_search_walk(p, features, nullptr, w, plan, again, scratch, out->anchor_index, false, 2, 0, s));
        TTF_STEP(launch_walk_finish(p, w, plan, scratch, out->anchor_index, out->fuse_map, out->best_sim, out->best_idx,
                                    nullptr, s));
    }
    mark();
    TTF_STEP(launch_offsets_scan(p, w, out->anchor_index, out->kept_count, out->row_offsets, false, s));
    mark();
    TTF_STEP(launch_emit_rows(p, features, w, out->anchor_index, out->kept_count, out->row_offsets, out->tokens_out,
                              out->pos_ids, out->src_index, frame_offset, false, s));
    mark();                                                    // end of the last stage
    if (out->host_counts) {
        TTF_STEP(hipMemcpyAsync(out->host_counts, out->kept_count, sizeof(int32_t) * p.B,
                                hipMemcpyDeviceToHost, s));
        TTF_STEP(hipMemcpyAsync(out->host_counts + p.B, out->row_offsets, sizeof(int32_t) * (p.B + 1),
                                hipMemcpyDeviceToHost, s));
    }
#undef TTF_STEP
    if (e != hipSuccess) {
        g_last_hip_error = static_cast<int>(e);
        return TTF_ERR_HIP;
    }
    if (timing) ++prof.calls;
    return TTF_OK;
}

ttf_status ttf_compress(const ttf_params* params, const void* features, void* workspace,
                        size_t workspace_bytes, const ttf_outputs* out, void* hip_stream)
{
    return run_pass(params, features, nullptr, 0, workspace, workspace_bytes, out, hip_stream);
}

// Workspace of ttf_compress_static.  In host code this name is only a handle for the runtime's symbol
// lookup, never a device address: host code uses the pointer hipGetSymbolAddress returns for the
// current device (every GPU holds its own copy of the array at its own address).
static __device__ __align__(256) unsigned char scratch[TTF_STATIC_WORKSPACE_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};   // device address of `scratch` per device, looked up once
}  // namespace

ttf_status ttf_compress_static(const ttf_params* params, const void* features, const ttf_outputs* out,
                               void* hip_stream)
{
    const ttf_status st = check_params(params);
    if (st != TTF_OK) return st;
    if (!features || !out) return TTF_ERR_INVALID_ARG;
    if (carve(*params, nullptr, false).bytes > (size_t)TTF_STATIC_WORKSPACE_BYTES) return TTF_ERR_WORKSPACE_TOO_SMALL;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess && (dev < 0 || dev >= kMaxDevices)) e = hipErrorInvalidDevice;
    void* ptr = nullptr;
    if (e == hipSuccess) {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        if (!g_scratch_ptr[dev]) {
            void* found = nullptr;
            e = hipGetSymbolAddress(&found, HIP_SYMBOL(scratch));
            if (e == hipSuccess && !found) e = hipErrorInvalidSymbol;
            if (e == hipSuccess) g_scratch_ptr[dev] = found;
        }
        ptr = g_scratch_ptr[dev];
    }
    if (e != hipSuccess) {
        g_last_hip_error = static_cast<int>(e);
        return TTF_ERR_HIP;
    }
    return run_pass(params, features, nullptr, 0, ptr, (size_t)TTF_STATIC_WORKSPACE_BYTES, out, hip_stream);
}

ttf_status ttf_compress_segment(const ttf_params* params, const void* features, const void* anchor_frame,
                                int32_t frame_offset, void* workspace, size_t workspace_bytes,
                                const ttf_outputs* out, void* hip_stream)
{
    if (!anchor_frame) return TTF_ERR_INVALID_ARG;
    if (params && (long long)frame_offset + params->F > 0x7fffffffll) return TTF_ERR_INVALID_ARG;
    return run_pass(params, features, anchor_frame, frame_offset, workspace, workspace_bytes, out, hip_stream);
}

// Largest radius of the tied-batch mode: its workspace keeps all (2r+1)^2 similarities per token.
static constexpr int kTiedMaxRadius = 3;

ttf_status ttf_tied_workspace_size(const ttf_params* params, size_t* bytes)
{
    if (!bytes) return TTF_ERR_INVALID_ARG;
    const ttf_status st = check_params(params);
    if (st != TTF_OK) return st;
    if (params->r > kTiedMaxRadius) return TTF_ERR_UNSUPPORTED;
    *bytes = carve_tied(*params, nullptr).bytes;
    return TTF_OK;
}

ttf_status ttf_compress_tied(const ttf_params* params, const void* features, void* workspace,
                             size_t workspace_bytes, const ttf_tied_outputs* out, void* hip_stream)
{
    const ttf_status st = check_params(params);
    if (st != TTF_OK) return st;
    if (!features || !workspace || !out) return TTF_ERR_INVALID_ARG;
    if (!out->tokens_out || !out->pos_ids || !out->src_index || !out->kept_count || !out->anchor_index ||
        !out->fuse_map)
        return TTF_ERR_INVALID_ARG;
    if (params->r > kTiedMaxRadius) return TTF_ERR_UNSUPPORTED;
    if (!aligned(features, 16) || !aligned(out->tokens_out, 16) || !aligned(workspace, 256))
        return TTF_ERR_UNSUPPORTED;
    const ttf_params& p = *params;
    TiedWorkspace tw = carve_tied(p, workspace);
    if (workspace_bytes < tw.bytes) tw = carve_tied(p, workspace, false);
    if (workspace_bytes < tw.bytes) return TTF_ERR_WORKSPACE_TOO_SMALL;
    const Workspace& w = tw.base;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    hipError_t e = hipSuccess;
#define TTF_STEP(call)                 \
    do {                               \
        if (e == hipSuccess) e = (call); \
    } while (0)
    WalkPlan plan{};
    WalkScratch scratch{};
    const bool mfma = use_mfma_path(p, w.tail, false), walk = use_walk(p, w, mfma, false, plan, scratch);
    if (p.anchor_mode == TTF_ANCHOR_AUTO) {
        TTF_STEP(launch_frame_sums(p, features, w, false, kept_share(p, walk, mfma), s));
        TTF_STEP(launch_anchor_scores(p, w, nullptr, 0, s));
    }
    TTF_STEP(launch_tied_anchor(p, w, out->anchor_index, s));
    if (walk) {
        TTF_STEP(launch_search_walk(p, features, nullptr, w, plan, plan, scratch, out->anchor_index, true, 0, 0, s));
        TTF_STEP(launch_walk_finish(p, w, plan, scratch, out->anchor_index, nullptr, nullptr, nullptr, tw.win_sim, s));
    } else {
        if (mfma)
            TTF_STEP(launch_anchor_prepare_any(p, features, nullptr, w, out->anchor_index, nullptr, nullptr, nullptr,
                                               true, s));
        else TTF_STEP(launch_anchor_norms(p, features, nullptr, w, out->anchor_index, true, s));
        TTF_STEP(launch_window_search(p, features, nullptr, w, out->anchor_index, nullptr, nullptr, nullptr,
                                      tw.win_sim, s));
    }
    TTF_STEP(launch_tie(p, w, tw.win_sim, out->anchor_index, out->fuse_map, out->best_sim, out->best_idx,
                        out->mean_sim, s));
    TTF_STEP(launch_offsets_scan(p, w, out->anchor_index, out->kept_count, tw.row_offsets, true, s));
    TTF_STEP(launch_emit_rows(p, features, w, out->anchor_index, out->kept_count, tw.row_offsets, out->tokens_out,
                              out->pos_ids, out->src_index, 0, true, s));
    if (out->host_counts)
        TTF_STEP(hipMemcpyAsync(out->host_counts, out->kept_count, sizeof(int32_t), hipMemcpyDeviceToHost, s));
#undef TTF_STEP
    if (e != hipSuccess) {
        g_last_hip_error = static_cast<int>(e);
        return TTF_ERR_HIP;
    }
    return TTF_OK;
}

ttf_status ttf_restore_map(const ttf_params* params, const int32_t* fuse_map, const int32_t* row_offsets,
                           const int32_t* src_index, int32_t* restore_map, void* hip_stream)
{
    const ttf_status st = check_params(params);
    if (st != TTF_OK) return st;
    if (!fuse_map || !row_offsets || !src_index || !restore_map) return TTF_ERR_INVALID_ARG;
    const hipError_t e = launch_restore_map(*params, fuse_map, row_offsets, src_index, restore_map,
                                            static_cast<hipStream_t>(hip_stream));
    if (e != hipSuccess) {
        g_last_hip_error = static_cast<int>(e);
        return TTF_ERR_HIP;
    }
    return TTF_OK;
}

ttf_status ttf_restore(const ttf_params* params, const void* tokens, int64_t rows,
                       const int32_t* restore_map, void* restored, void* hip_stream)
{
    const ttf_status st = check_params(params);
    if (st != TTF_OK) return st;
    if (!tokens || !restore_map || !restored || rows < 0) return TTF_ERR_INVALID_ARG;
    if (!aligned(tokens, 16) || !aligned(restored, 16)) return TTF_ERR_UNSUPPORTED;
    const hipError_t e = launch_restore_rows(*params, tokens, rows, restore_map, restored,
                                             static_cast<hipStream_t>(hip_stream));
    if (e != hipSuccess) {
        g_last_hip_error = static_cast<int>(e);
        return TTF_ERR_HIP;
    }
    return TTF_OK;
}

ttf_status ttf_decode_alignment(int64_t l_prime, int64_t text_tokens, int64_t step,
                                int64_t* l_pre, int64_t* position, int64_t* mask_length)
{
    if (l_prime < 0 || text_tokens < 0 || step < 0) return TTF_ERR_INVALID_ARG;
    const int64_t pre = l_prime + text_tokens;
    if (l_pre) *l_pre = pre;
    if (position) *position = pre + step;
    if (mask_length) *mask_length = pre + step + 1;
    return TTF_OK;
}

ttf_status ttf_select_threshold(const ttf_params* params, const float* best_sim,
                                const int32_t* anchor_index, float fused_fraction,
                                float* thresholds, void* hip_stream)
{
    const ttf_status st = check_params(params);
    if (st != TTF_OK) return st;
    if (!best_sim || !anchor_index || !thresholds) return TTF_ERR_INVALID_ARG;
    if (!(fused_fraction >= 0.0f && fused_fraction <= 1.0f)) return TTF_ERR_INVALID_ARG;
    const hipError_t e = launch_select_threshold(*params, best_sim, anchor_index, 1.0 - (double)fused_fraction,
                                                 thresholds,
                                                 static_cast<hipStream_t>(hip_stream));
    if (e != hipSuccess) {
        g_last_hip_error = static_cast<int>(e);
        return TTF_ERR_HIP;
    }
    return TTF_OK;
}

ttf_status ttf_regate(const ttf_params* params, const void* features, const float* thresholds,
                      void* workspace, size_t workspace_bytes, const ttf_outputs* out, void* hip_stream)
{
    const ttf_status st = check_params(params);
    if (st != TTF_OK) return st;
    if (!features || !workspace || !out) return TTF_ERR_INVALID_ARG;
    if (!out->tokens_out || !out->pos_ids || !out->src_index || !out->row_offsets || !out->kept_count ||
        !out->anchor_index || !out->fuse_map || !out->best_sim || !out->best_idx)
        return TTF_ERR_INVALID_ARG;
    if (!aligned(features, 16) || !aligned(out->tokens_out, 16) || !aligned(workspace, 256))
        return TTF_ERR_UNSUPPORTED;
    const ttf_params& p = *params;
    const Workspace w = carve(p, workspace, false);
    if (workspace_bytes < w.bytes) return TTF_ERR_WORKSPACE_TOO_SMALL;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    hipError_t e = launch_regate(p, w, out->best_sim, out->best_idx, out->anchor_index, thresholds,
                                 out->fuse_map, s);
    if (e == hipSuccess)
        e = launch_offsets_scan(p, w, out->anchor_index, out->kept_count, out->row_offsets, false, s);
    if (e == hipSuccess)
        e = launch_emit_rows(p, features, w, out->anchor_index, out->kept_count, out->row_offsets, out->tokens_out,
                             out->pos_ids, out->src_index, 0, false, s);
    if (e == hipSuccess && out->host_counts) {
        e = hipMemcpyAsync(out->host_counts, out->kept_count, sizeof(int32_t) * p.B, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess)
            e = hipMemcpyAsync(out->host_counts + p.B, out->row_offsets, sizeof(int32_t) * (p.B + 1),
                               hipMemcpyDeviceToHost, s);
    }
    if (e != hipSuccess) {
        g_last_hip_error = static_cast<int>(e);
        return TTF_ERR_HIP;
    }
    return TTF_OK;
}

ttf_status ttf_search_route(const ttf_params* params, int* route)
{
    if (!route) return TTF_ERR_INVALID_ARG;
    const ttf_status st = check_params(params);
    if (st != TTF_OK) return st;
    ttf_params p = *params;
    p.r = std::min(p.r, std::max(p.H, p.W));                 // (as ttf_compress)
    const bool mfma = use_mfma_path(p, true, false), walk = search_walks(p, false);
    *route = !mfma && !walk                 ? TTF_ROUTE_GENERAL
           : p.dtype == TTF_F32             ? TTF_ROUTE_MFMA_F32
           : mfma_search_supported(p)       ? TTF_ROUTE_MFMA_BF16
                                            : TTF_ROUTE_MFMA_BF16_PADDED;
    return TTF_OK;
}

ttf_status ttf_set_speculation(int mode)
{
    if (mode < -1 || mode > 1) return TTF_ERR_INVALID_ARG;
    g_speculation.store(mode, std::memory_order_relaxed);
    return TTF_OK;
}

const char* ttf_status_string(ttf_status status)
{
    switch (status) {
        case TTF_OK: return "ok";
        case TTF_ERR_INVALID_ARG: return "invalid argument";
        case TTF_ERR_UNSUPPORTED: return "unsupported dtype or alignment";
        case TTF_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
        case TTF_ERR_HIP: return "HIP runtime error";
    }
    return "unknown status";
}

int ttf_last_hip_error(void) { return g_last_hip_error; }

ttf_status ttf_profile_enable(int slots)
{
    Profile& prof = g_prof;
    if (slots < 0 || slots > TTF_PROFILE_MAX_SLOTS) return TTF_ERR_INVALID_ARG;
    for (; prof.created < slots; ++prof.created) {
        for (int i = 0; i <= TTF_NUM_STAGES; ++i) {
            const hipError_t e = hipEventCreate(&prof.ev[prof.created][i]);
            if (e != hipSuccess) {
                for (int j = 0; j < i; ++j) (void)hipEventDestroy(prof.ev[prof.created][j]);
                g_last_hip_error = static_cast<int>(e);
                return TTF_ERR_HIP;
            }
        }
    }
    prof.slots = slots;
    prof.calls = 0;
    return TTF_OK;
}

ttf_status ttf_profile_read(int call, float* ms_out, int n)
{
    Profile& prof = g_prof;
    if (!ms_out || n < 0 || prof.slots <= 0) return TTF_ERR_INVALID_ARG;
    if (call < 0 || call >= prof.calls || call < prof.calls - prof.slots) return TTF_ERR_INVALID_ARG;
    hipEvent_t* ev = prof.ev[call % prof.slots];
    hipError_t e = hipEventSynchronize(ev[TTF_NUM_STAGES]);
    for (int i = 0; i < n && i < TTF_NUM_STAGES && e == hipSuccess; ++i)
        e = hipEventElapsedTime(&ms_out[i], ev[i], ev[i + 1]);
    if (e != hipSuccess) {
        g_last_hip_error = static_cast<int>(e);
        return TTF_ERR_HIP;
    }
    return TTF_OK;
}

const char* ttf_stage_name(int stage)
{
    static const char* names[TTF_NUM_STAGES] = {"frame_sums", "anchor_scores", "anchor_norms", "window_search",
                                                "anchor_verify", "offsets_scan", "emit_rows"};
    return (stage >= 0 && stage < TTF_NUM_STAGES) ? names[stage] : "";
}

}  // extern "C"
