// Window search of large inputs: workgroups that walk whole frames (Section 3, "Pointwise Matching
// with Local Window Search" and "Threshold Gating").
//
// What bounds it is how the token rows stream out of HBM.  A workgroup that keeps the products of many
// tiles in registers has to read its rows a few hundred bytes at a time (k_search_mfma: 128 rows, 512
// bytes of each per pass, 5.3 TB/s); the same bytes read as 4 KiB runs of consecutive rows come at 6.7.
// Here a workgroup therefore owns a share of the channels (eight waves x KW K-steps of 32) of a column strip
// of up to 16 cells in a group of frames, and walks down the rows of the grid: per row one anchor tile and
// the source tiles of its frames, every tile 16 consecutive tokens.  A tile is finished before the next
// begins, so its products need (2r+1) accumulators only, and the registers hold the window instead: the
// anchor tiles of rows y-r .. y+r in MFMA operand order, read straight from the anchor frame, one new tile
// per row.  The shares of the channels meet in a small array of window products per token (part), and
// k_walk_finish turns them into similarities.
//
//  * Tokens go from memory to LDS without passing the registers (global_load_lds), each wave through a ring of
//    its own: groups of two K-steps (128 bytes of each of the 16 rows: whole cache lines; 64-byte pieces
//    ran at 5.7 TB/s), four groups deep, 64 KiB in flight per workgroup.  The ring runs across tiles,
//    rows and frames, so the stream never drains; a wave waits for its own loads only.
//  * Pieces of a row are stored at position (piece ^ row / 2), which spreads the 16 rows that an operand
//    read touches over all LDS banks.
//  * The products of the eight waves are added through LDS, double-buffered, one barrier per tile; every wave adds
//    and stores those of two tokens (only the band of the products that the window needs).
//  * A strip of a grid wider than 16 is 16 - 2r cells wide at most, so that its window lies in one anchor tile.
//  * Plain loads leave a line in the Infinity Cache and stream slower than non-temporal ones (whole walk plain 193
//    us, non-temporal 173, B2 F256 16x16 C4096).  Only the last tiles of a workgroup are read that way, for the row copy
//    (323 -> 302 us); not beside a guess, where fewer rows are kept than that pays for.
//  * SPEC (the anchor may be a guess): every frame is walked and its sums over the strip are kept, 16 channels
//    a register: two MFMAs per K-step against 0/1 matrices that pick 16 of the 32 channels leave four tokens
//    of one channel in a lane.
//  * fp32 tokens: a group is one K-step, every value cut into three bf16 planes as it is used (the window holds the
//    planes), six plane products per MFMA of the bf16 form.  Norms and sums are plain fp32: eight channels of a token in a
//    lane, sums by exchanging halves inside a row of 16 lanes until two lanes hold one channel.  Bound by the
//    arithmetic and its latency: B16 F32 16x16 C4096 (2 GiB) 380 us plain (452 for k_search_mfma_f32), 487 with sums, which
//    save the 322 us of k_frame_sums_slab; eight frames a workgroup instead of four 522 -> 502 when that was tried.
// Kernel alone, bf16, against the kernels it replaces there: B16 F32 16x16 C4096 with sums 248 -> 180 us (5.9 TB/s of
// tokens), 14x14 218 -> 152, B2 F256 16x16 C4096 189 -> 174 (162 behind frame sums that leave the Infinity Cache warm), B4
// F64 32x32 C4096 r 2 with sums 596 -> 496.  With everything but the loads taken out the first runs no faster
// (179), so it is the walk through memory that is left; of the last 64 us are the stores of the window products and
// 60 the reduction (rows of 11 cells instead of patches: 575, twice the products and 1.5 times the tiles).
// Tried: fragments read one group ahead (187 against 181), twice the groups in flight (no change).
#include "ttf_anchor_pick.h"
#include "ttf_internal.h"
#include "ttf_search_tile.h"

#include <algorithm>

namespace ttf {
namespace {

constexpr int kWalkWaves = 8;
constexpr int kWalkGroups = 4;                               // groups of a tile per wave, at most
constexpr int kWalkGroup = 2048;                             // bytes of a group: 16 rows x 128 (two K-steps of 32 bf16
                                                             // channels, or one of 32 fp32 channels)

// Most frames of a workgroup that keeps sums: what fits the registers beside the window (fp32: one register for a group's
// 32 channels, four for 64 of bf16).
template <typename E, int RAD>
constexpr int spec_frames() { return sizeof(E) == 4 ? 8 : (RAD == 2 ? 2 : 4); }

struct WalkArgs {
    const char* x;
    const char* ext_anchor;                                  // external anchor frames, or null
    const double* score_part;
    const double* clip_part;
    int32_t* anchor_index;
    int32_t* spec;
    float* part;                                             // [nk][B*F*N][K+1] window products, squared norm
    float* norm_part;                                        // [nk][B*N] squared norms of the anchor tokens
    float* strip_sum;                                        // [B*F][strips*ysegs][C]
    int B, F, H, W, C, S;
    int nk, lines;
    WalkDeal deal, all;                                      // `all`: mode 2, where no clip has a trusted guess
    int fixed_anchor, mode;
    int min_trusted;                                         // mode 1: with fewer trusted guesses than this none is taken
    int keep_from;                                           // of 256 parts of a workgroup's tiles, the first left in the cache
};

// LDS reads of two fragments are complete and no longer need their ring slot.
__device__ __forceinline__ void settle(u32x4& a, u32x4& b) { asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a), "+v"(b)::"memory"); }
template <int N>
__device__ __forceinline__ void wait_loads()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// 64 lanes x 16 bytes from base + off (per lane) to LDS at lds + 16 * lane.  No register receives the data; the
// ring's readers wait on vmcnt.  m0 holds the LDS address; it is a reserved register that the compiler sets right before
// each use of its own and keeps nothing in, so it need not (and, being reserved, cannot) be named as clobbered.
template <bool STREAM>
__device__ __forceinline__ void load_to_lds(const char* base, uint32_t off, uint32_t lds)
{
    if constexpr (STREAM)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds), "v"(off), "s"(base) : "memory");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base) : "memory");
}

// A value from another lane of the row of 16 (the DPP control names which).
template <int DPP_CTRL>
__device__ __forceinline__ float row_move(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), DPP_CTRL, 0xf, 0xf, true));
}

// B operand that picks 16 of the 32 channels of a K-step: E_h[k][n] = 1 iff k == 16h + n (operand order: lane
// n + 16g holds rows k = 8g .. 8g+7 of column n).  A tile times E_h is its tokens x channels 16h .. 16h+15 in
// the MFMA result layout, i.e. a lane then holds four TOKENS of one channel.
__device__ __forceinline__ bf16x8 channel_picker(int h, int lane)
{
    const int n = lane & 15, g = lane >> 4;
    const bool mine = g == 2 * h + (n >> 3);
    const int e = n & 7;
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = (mine && (e >> 1) == i) ? ((e & 1) ? 0x3F800000u : 0x00003F80u) : 0u;
    return __builtin_bit_cast(bf16x8, w);
}

// The tiles of a search and the window that the registers hold for one.
//  Rows (PATCH false): a tile is up to 16 cells of one grid row, its window 2r+1 anchor tiles, the rows y-r .. y+r
//   with the cells r to either side; the next tile is the row below, whose window needs one new anchor tile.
//  Patches (PATCH true): a tile is 4x4 cells (token 4 * column + row).  Its window of (4+2r) x (4+2r) cells is 2+r
//   anchor tiles of two rows each (anchor n: column n % (4+2r), row n / (4+2r)); the next tile lies four rows
//   below, and its window needs two new ones.
template <int RAD, bool PATCH>
struct Tiles {
    static constexpr int NP = 2 * RAD + 1, KK = NP * NP;
    static constexpr int SPAN = 4 + 2 * RAD;                 // anchor columns that four neighbouring tokens look at
    static constexpr int NT = PATCH ? 2 + RAD : NP;          // anchor tiles of a window
    static constexpr int NEW = PATCH ? 2 : 1;                // ... that the next tile does not share
    static constexpr int STEP = PATCH ? 4 : 1;               // grid rows of a tile
    static constexpr int RING = RAD == 2 ? 6 : 8;            // groups in flight per wave
    // Lanes of a product tile that hold values of windows, and the 16-byte words that its share of the reduction
    // takes (a few more, so that the values of a token come from different banks).
    static constexpr int BAND = PATCH ? 8 * NP + 2 : 4 * SPAN + 4;
    static constexpr int RED = NT * BAND + 16;               // words per wave: the products, and the diagonal of the tile
                                                             // against itself
    static constexpr size_t LDS = kWalkWaves * (RING * kWalkGroup + 2 * RED * 16);
    static_assert(LDS <= 160 * 1024, "LDS of a CU");
};

// mode 0: the anchor is external, fixed, given in anchor_index or picked here; the source frames are walked.
// mode 1 (SPEC): clips with a trusted guess, every frame walked.  mode 2: the exact rule; clips whose
// guess it confirms are left out, the others walked as in mode 0.  (Units are made of the clips to search alone, so
// that a few of them still meet all XCDs.)
template <typename E, int RAD, bool PATCH, bool SPEC>
__global__ __launch_bounds__(kWalkWaves * 64, 2) void k_search_walk(const WalkArgs A)
{
    using T = Tiles<RAD, PATCH>;
    constexpr int NP = T::NP, KK = T::KK, NT = T::NT, NEW = T::NEW, STEP = T::STEP, FRS = spec_frames<E, RAD>(), GM = kWalkGroups;
    constexpr bool F32 = sizeof(E) == 4;
    constexpr int PL = F32 ? 3 : 2;                          // fragments of a group: three bf16 planes, or two K-steps
    constexpr int SL = F32 ? 1 : 4;                          // registers of a group's sums
    extern __shared__ u32x4 lds_mem[];
    char* const ring = reinterpret_cast<char*>(lds_mem);
    f32x4* const red = reinterpret_cast<f32x4*>(ring + kWalkWaves * T::RING * kWalkGroup);   // [2][wave][RED]

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = lane & 15, g = lane >> 4;
    const int H = A.H, W = A.W, N = H * W, F = A.F;
    // The clips to search (mode 2: up to kPickClips, whose anchors the waves pick between them; more clips pick their
    // own below and leave where there is nothing to do, and so do all where no guess is left: the picks of all clips ahead of
    // the walk took B16 F66 16x16 C2048 187 us for the 172 of a search without a guess), and how many units they make.
    bool guessed = A.mode != 2;
    for (int b0 = 0; !guessed && b0 < A.B; b0 += 64)
        guessed = __ballot(b0 + lane < A.B && A.spec[4 * min(b0 + lane, A.B - 1) + 1] != 0) != 0;
    const WalkDeal deal = guessed ? A.deal : A.all;
    const int per_clip = deal.groups * deal.lsegs * deal.ysegs * A.nk;
    constexpr int kPickClips = 32;
    int32_t* const picked = reinterpret_cast<int32_t*>(red); // [2][kPickClips] exact anchor, search again
    const bool choose = A.mode == 1 || (A.mode == 2 && guessed && A.B <= kPickClips);
    if (A.mode == 2 && choose) {
        for (int c = wave; c < A.B; c += kWalkWaves) {
            const int exact = pick_anchor(A.score_part, A.clip_part, c, F, A.S, lane);
            if (lane == 0) {
                picked[c] = exact;
                picked[kPickClips + c] = A.spec[4 * c + 1] == 0 || A.spec[4 * c] != exact;
                if (blockIdx.x == 0) A.anchor_index[c] = exact;
            }
        }
        __syncthreads();
    }
    auto flags = [&](int b0) {                               // of the 64 clips from b0 on
        const int bb = b0 + lane;
        bool mine = false;
        if (bb < A.B) mine = A.mode == 1 ? A.spec[4 * bb + 1] != 0 : picked[kPickClips + bb] != 0;
        return (uint64_t)__ballot(mine);
    };
    int clips = A.B;
    if (choose) {
        clips = 0;
        for (int b0 = 0; b0 < A.B; b0 += 64) clips += __popcll(flags(b0));
        if (A.mode == 1 && clips < A.min_trusted) {
            // No guess is taken (guess_cost()): the marks go, for this launch and those behind it.  A workgroup
            // that counts some of them gone comes to the same answer.
            if (blockIdx.x == 0) {
                for (int c = threadIdx.x; c < A.B; c += kWalkWaves * 64) A.spec[4 * c + 1] = 0;
            }
            return;
        }
    }
    // Workgroups are dealt to the XCDs round robin; every XCD gets one contiguous run of the units, in
    // which the frame groups of one (clip, strip, channel share) are neighbours: their anchor rows are read
    // from HBM once and then come from that XCD's L2.
    int u;
    {
        const int U = clips * per_clip, xcd = (int)blockIdx.x & 7, nth = (int)blockIdx.x >> 3;
        if (nth >= (U >> 3) + (xcd < (U & 7) ? 1 : 0)) return;   // (workgroup-uniform)
        u = xcd * (U >> 3) + min(xcd, U & 7) + nth;
    }
    const int grp = u % deal.groups; u /= deal.groups;
    const int seg = u % (deal.lsegs * deal.ysegs); u /= deal.lsegs * deal.ysegs;
    const int share = u % A.nk;
    int b = u / A.nk;
    if (choose) {                                            // the b-th clip of those to search
        int left_out = b, b0 = 0;
        uint64_t set = flags(0);
        while (left_out >= (int)__popcll(set)) {
            left_out -= (int)__popcll(set);
            b0 += 64;
            set = flags(b0);
        }
        for (; left_out > 0; --left_out) set &= set - 1;
        b = b0 + __ffsll((unsigned long long)set) - 1;
    }

    int a;
    if (A.mode == 0) {
        a = A.ext_anchor ? -1
          : A.fixed_anchor >= 0 ? A.fixed_anchor
          : A.fixed_anchor == kAnchorGiven ? A.anchor_index[b]
                                           : pick_anchor(A.score_part, A.clip_part, b, F, A.S, lane);
    } else if (A.mode == 1) {
        a = A.spec[4 * b];
    } else {
        a = choose ? picked[b] : pick_anchor(A.score_part, A.clip_part, b, F, A.S, lane);
    }
    a = __builtin_amdgcn_readfirstlane(a);
    if ((A.mode == 0 ? A.fixed_anchor != kAnchorGiven : A.mode == 2 && !choose) && grp + seg + share == 0 && threadIdx.x == 0)
        A.anchor_index[b] = a;
    if (A.mode == 2) {
        if (!choose && A.spec[4 * b + 1] != 0 && A.spec[4 * b] == a) return;   // confirmed: searched already
        __syncthreads();                                     // `picked` is read: its place is free
    }

    // the unit's part of the grid: column strips line_lo .. line_hi-1, tiles step_lo .. step_hi-1 of each
    const int line_lo = (int)((long long)A.lines * (seg / deal.ysegs) / deal.lsegs);
    const int line_hi = (int)((long long)A.lines * (seg / deal.ysegs + 1) / deal.lsegs);
    const int all_steps = (H + STEP - 1) / STEP;
    const int step_lo = (int)((long long)all_steps * (seg % deal.ysegs) / deal.ysegs);
    const int step_hi = (int)((long long)all_steps * (seg % deal.ysegs + 1) / deal.ysegs);
    // first cell and width of a strip; rows of grids wider than 16 keep a margin of r for the window
    const int margin = PATCH || A.lines == 1 ? 0 : RAD;
    const int strip_w = W / A.lines, wide_strips = W % A.lines;      // (the first strips are a cell wider where need be)
    auto strip_x = [&](int line) { return PATCH ? 4 * line : line * strip_w + min(line, wide_strips); };
    // frames of the group: cnt slots from k0, the anchor left out where it is not walked
    const int walked = (SPEC || a < 0) ? F : F - 1;
    const int skip = (SPEC || a < 0) ? 0x7fffffff : a;
    const int k0 = grp * deal.nf;
    const int cnt = min(deal.nf, walked - k0);
    if (cnt <= 0) return;                                    // (one frame, the anchor: nothing to walk)
    // channels of this wave: groups q_lo .. q_lo+gq-1 of 128 bytes
    const int total_groups = A.C / (128 / (int)sizeof(E));
    const int q_lo = (int)((long long)total_groups * (share * kWalkWaves + wave) / (kWalkWaves * A.nk));
    const int gq = (int)((long long)total_groups * (share * kWalkWaves + wave + 1) / (kWalkWaves * A.nk)) - q_lo;
    const size_t row_bytes = (size_t)A.C * sizeof(E);
    const size_t frame_bytes = (size_t)N * row_bytes;
    const char* const src_frames = A.x + (size_t)b * F * frame_bytes + (size_t)q_lo * 128;
    const char* const anchor_frame = (a < 0 ? A.ext_anchor + (size_t)b * frame_bytes + (size_t)q_lo * 128
                                            : src_frames + (size_t)a * frame_bytes);

    // lane l of load i of a group fills piece l of its KiB: row 8i + l/8 of the tile, stored piece l%8
    const int lrow = lane >> 3;
    const uint32_t piece0 = (uint32_t)((lane & 7) ^ (lane >> 4)) * 16, piece1 = piece0 ^ 64;
    // operand lane (token m, channels 8g..8g+7) of K-step j of a group
    const uint32_t rd0 = (uint32_t)((m >> 3) * 1024 + ((m & 7) * 8 + (g ^ (m >> 1))) * 16), rd1 = rd0 ^ 64;
    const uint32_t ring_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)ring + (uint32_t)wave * (T::RING * kWalkGroup);
    const char* const my_ring = ring + wave * (T::RING * kWalkGroup);

    // The stream of tiles, in the order they are used: for every strip the anchor tiles of the first window but the
    // new ones, then for every step the NEW anchor tiles and the source tiles of the frames.  The state below
    // belongs to the loads, which run ahead of the use by up to RING groups.  l_e < 0: tiles ahead of the strip's
    // first step; 0 .. NEW-1: the new anchor tiles; NEW + f: frame f.
    int left = (line_hi - line_lo) * (NT - NEW + (step_hi - step_lo) * (NEW + cnt)) * gq;   // groups not yet used
    int to_load = left;                                      // groups not yet requested
    int l_line = line_lo, l_step = step_lo, l_e = NEW - NT, l_q = 0, l_slot = 0;
    const char* l_base;
    uint32_t l_off0, l_off1;
    bool l_keep = false;
    auto locate = [&]() {                                    // addresses of the tile at the load state
        // cells outside the grid read the nearest cell inside (their products are masked, their sums weighted 0)
        auto cell = [&](int y, int x) {
            return (uint32_t)(min(max(y, 0), H - 1) * W + min(max(x, 0), W - 1)) * (uint32_t)row_bytes;
        };
        const int x0 = strip_x(l_line);
        if (l_e < NEW) {
            const int c = NT - NEW + NEW * (l_step - step_lo) + l_e;
            l_base = anchor_frame;
            if constexpr (PATCH) {
                const int y = STEP * step_lo + 2 * c - RAD;
                l_off0 = cell(y + lrow / T::SPAN, x0 - RAD + lrow % T::SPAN) + piece0;
                l_off1 = cell(y + min((lrow + 8) / T::SPAN, 1), x0 - RAD + (lrow + 8) % T::SPAN) + piece1;
            } else {
                const int y = step_lo + c - RAD;
                l_off0 = cell(y, x0 - margin + lrow) + piece0;
                l_off1 = cell(y, x0 - margin + lrow + 8) + piece1;
            }
        } else {
            const int k = k0 + l_e - NEW + (k0 + l_e - NEW >= skip ? 1 : 0);
            l_base = src_frames + (size_t)k * frame_bytes;
            if constexpr (!SPEC)
                l_keep = ((l_line - line_lo) * (step_hi - step_lo) + l_step - step_lo) * 256 >=
                         (line_hi - line_lo) * (step_hi - step_lo) * A.keep_from;
            if constexpr (PATCH) {
                l_off0 = cell(STEP * l_step + (lrow & 3), x0 + (lrow >> 2)) + piece0;
                l_off1 = cell(STEP * l_step + (lrow & 3), x0 + 2 + (lrow >> 2)) + piece1;
            } else {
                const int last = strip_x(l_line + 1) - 1;
                l_off0 = cell(l_step, min(x0 + lrow, last)) + piece0;
                l_off1 = cell(l_step, min(x0 + lrow + 8, last)) + piece1;
            }
        }
    };
    locate();
    auto request = [&]() {
        if (to_load == 0) return;
        --to_load;
        const uint32_t d = ring_lds + (uint32_t)l_slot * kWalkGroup;
        if (l_e < NEW) {
            load_to_lds<false>(l_base, l_off0, d);
            load_to_lds<false>(l_base, l_off1, d + 1024);
        } else {
            if (l_keep) {
                load_to_lds<false>(l_base, l_off0, d);
                load_to_lds<false>(l_base, l_off1, d + 1024);
            } else {
                load_to_lds<true>(l_base, l_off0, d);
                load_to_lds<true>(l_base, l_off1, d + 1024);
            }
        }
        l_slot = l_slot + 1 == T::RING ? 0 : l_slot + 1;
        l_base += 128;
        if (++l_q == gq) {
            l_q = 0;
            if (++l_e == NEW + cnt) {
                l_e = 0;
                if (++l_step == step_hi) {
                    l_step = step_lo;
                    l_e = NEW - NT;
                    ++l_line;
                }
            }
            locate();
        }
    };
    for (int i = 0; i < T::RING; ++i) request();

    int slot = 0;
    // the two K-steps of the next group, in operand order; its ring slot is filled again at once
    auto take = [&](u32x4& f0, u32x4& f1) {
        if (left >= T::RING) wait_loads<2 * (T::RING - 1)>();
        else wait_loads<0>();                                // (the last groups: nothing is requested behind them)
        const char* s = my_ring + slot * kWalkGroup;
        f0 = *reinterpret_cast<const u32x4*>(s + rd0);
        f1 = *reinterpret_cast<const u32x4*>(s + rd1);
        settle(f0, f1);
        slot = slot + 1 == T::RING ? 0 : slot + 1;
        --left;
        request();
    };
    bf16x8 win[NT][GM][PL];                                  // the window of the tile
#pragma unroll
    for (int q = 0; q < NT; ++q) {
#pragma unroll
        for (int gi = 0; gi < GM; ++gi) {
#pragma unroll
            for (int e = 0; e < PL; ++e) win[q][gi][e] = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
        }
    }
    float sum[SPEC ? FRS : 1][GM][SL];
    bf16x8 pick0, pick1;
    if constexpr (SPEC) {
        pick0 = channel_picker(0, lane);
        pick1 = channel_picker(1, lane);
#pragma unroll
        for (int f = 0; f < FRS; ++f) {
#pragma unroll
            for (int gi = 0; gi < GM; ++gi) {
#pragma unroll
                for (int e = 0; e < SL; ++e) sum[f][gi][e] = 0.f;
            }
        }
    }
    // A finished tile has 16 x (KK + 1) numbers worth adding up over the waves: the (2r+1)^2 products of every
    // token with its window, and its squared norm (the diagonal of the tile against itself).  Wave w adds
    // those of tokens 2w and 2w + 1, a lane each.
    constexpr int PER = 2 * (KK + 1);
    static_assert(PER <= 64, "a lane per value");
    const bool adds = lane < PER;
    const int vt = 2 * wave + (lane >= KK + 1 ? 1 : 0), ve = lane >= KK + 1 ? lane - (KK + 1) : lane;
    const int vy = ve / NP, vx = ve % NP;                    // cell of the window
    int v_slot, my_slot;                                     // where the value lies, and where this lane's products go
    bool in_band;
    if constexpr (PATCH) {
        const int row = (vt & 3) + vy, span = m % T::SPAN - g;
        v_slot = (row >> 1) * T::BAND + ((vt >> 2) * 2 + (row & 1)) * NP + vx;
        in_band = m < 2 * T::SPAN && span >= 0 && span < NP;
        my_slot = (g * 2 + m / T::SPAN) * NP + span;
    } else {
        v_slot = vy * T::BAND + (vt >> 2) * T::SPAN + (vt & 3) + vx;
        my_slot = m - (4 * g - RAD + margin);
        in_band = my_slot >= 0 && my_slot < T::SPAN;
        my_slot += g * T::SPAN;
    }
    const bool on_diagonal = (m >> 2) == g;
    const float* const red_in = reinterpret_cast<const float*>(red) + (!adds ? 0 : (ve < KK ? v_slot : NT * T::BAND + vt) * 4 + (vt & 3));
    f32x4* const red_out = red + (in_band ? my_slot : 0);
    int buf = 0;
    // The shares are read behind the barrier and added and stored in the middle of the next tile, when they have
    // long arrived.
    float pend[kWalkWaves];
    float* pend_out = nullptr;
    auto fetch_shares = [&](float* out) {
        lds_barrier();
        pend_out = adds ? out : nullptr;
        const float* r = red_in + buf * (kWalkWaves * T::RED * 4);
#pragma unroll
        for (int w = 0; w < kWalkWaves; ++w) pend[w] = r[w * (T::RED * 4)];
        buf ^= 1;
    };
    auto store_shares = [&]() {
        if (pend_out) *pend_out = ((pend[0] + pend[1]) + (pend[2] + pend[3])) + ((pend[4] + pend[5]) + (pend[6] + pend[7]));
        pend_out = nullptr;
    };
    float* const part_out = A.part + ((size_t)share * A.B * F * N + (size_t)b * F * N) * (KK + 1) + ve;
    // fp32: the fragments of a group as bf16 planes, and this lane's share of the tokens' squared norms
    auto planes = [&](const u32x4 (&fr)[2], bf16x8 (&pl)[PL], float& nn) {
        const uint32_t r[8] = {fr[0][0], fr[0][1], fr[0][2], fr[0][3], fr[1][0], fr[1][1], fr[1][2], fr[1][3]};
        uint32_t w[3][4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float v0 = __builtin_bit_cast(float, r[2 * e]), v1 = __builtin_bit_cast(float, r[2 * e + 1]);
            nn = fmaf(v1, v1, fmaf(v0, v0, nn));
            uint32_t h, mi, l;
            split_bf16x3(v0, v1, h, mi, l);
            w[0][e] = h; w[1][e] = mi; w[2][e] = l;
        }
#pragma unroll
        for (int e = 0; e < PL; ++e) pl[e] = __builtin_bit_cast(bf16x8, uint4{w[e][0], w[e][1], w[e][2], w[e][3]});
    };
    // ... summed over the lanes that share a token and put where the diagonal of a tile's products stands
    auto put_norm = [&](size_t mine, float nn) {
        nn += __shfl_xor(nn, 16, 64);
        nn += __shfl_xor(nn, 32, 64);
        if (on_diagonal) reinterpret_cast<float*>(red + mine + NT * T::BAND + m)[m & 3] = nn;
    };
    auto source_tile = [&](int f, int line, int step, float (&tile_sum)[GM][SL]) {
        const int x0 = strip_x(line), x1 = min(strip_x(line + 1), W);
        f32x4 acc[NT + 1];
        float nn = 0.f;
#pragma unroll
        for (int q = 0; q <= NT; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
        float weight[4];                                     // SPEC: rows of the tile that hold no cell of their own count zero
#pragma unroll
        for (int j = 0; j < 4; ++j)
            weight[j] = (PATCH ? STEP * step + j < H && x0 + g < W : x0 + 4 * g + j < x1) ? 1.0f : 0.0f;
        const bool full = !PATCH && x1 - x0 == 16;
        const bool own = PATCH ? STEP * step + (m & 3) < H && x0 + (m >> 2) < W : x0 + m < x1;
#pragma unroll
        for (int gi = 0; gi < GM; ++gi) {
            if (gi < gq) {                                   // wave-uniform
                u32x4 fr[2];
                take(fr[0], fr[1]);
                if (gi == 0) store_shares();
                if constexpr (F32) {
                    bf16x8 pl[PL];
                    planes(fr, pl, nn);
                    // six of the nine products of the planes, the smallest first
                    constexpr int SP[6] = {2, 0, 1, 1, 0, 0}, WP[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
                    for (int term = 0; term < 6; ++term) {
#pragma unroll
                        for (int q = 0; q < NT; ++q)
                            acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pl[SP[term]], win[q][gi][WP[term] % PL], acc[q], 0, 0, 0);
                    }
                    if constexpr (SPEC) {
                        // a lane's eight channels over the 16 tokens (the lanes of its row): halves are exchanged until
                        // two lanes hold one channel
                        const uint32_t r[8] = {fr[0][0], fr[0][1], fr[0][2], fr[0][3], fr[1][0], fr[1][1], fr[1][2], fr[1][3]};
                        float v[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e) v[e] = __builtin_bit_cast(float, r[e]);
                        if (!full) {                         // (wave-uniform)
#pragma unroll
                            for (int e = 0; e < 8; ++e) v[e] = own ? v[e] : 0.f;
                        }
                        float h[4], q2[2];
#pragma unroll
                        for (int e = 0; e < 4; ++e) h[e] = ((m & 8) ? v[e + 4] : v[e]) + row_move<0x128>((m & 8) ? v[e] : v[e + 4]);
#pragma unroll
                        for (int e = 0; e < 2; ++e) q2[e] = ((m & 4) ? h[e + 2] : h[e]) + row_move<0x141>((m & 4) ? h[e] : h[e + 2]);
                        const float o = ((m & 2) ? q2[1] : q2[0]) + row_move<0x4E>((m & 2) ? q2[0] : q2[1]);
                        tile_sum[gi][0] += o + row_move<0xB1>(o);
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const bf16x8 av = __builtin_bit_cast(bf16x8, fr[j]);
#pragma unroll
                        for (int q = 0; q < NT; ++q)
                            acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, win[q][gi][j], acc[q], 0, 0, 0);
                        acc[NT] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, av, acc[NT], 0, 0, 0);
                        if constexpr (SPEC) {
                            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
                            const f32x4 d0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, pick0, zero, 0, 0, 0);
                            const f32x4 d1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, pick1, zero, 0, 0, 0);
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                tile_sum[gi][2 * j % SL] = fmaf(d0[e], weight[e], tile_sum[gi][2 * j % SL]);
                                tile_sum[gi][(2 * j + 1) % SL] = fmaf(d1[e], weight[e], tile_sum[gi][(2 * j + 1) % SL]);
                            }
                        }
                    }
                }
            }
        }
        const size_t mine = (size_t)(buf * kWalkWaves + wave) * T::RED;
        if (in_band) {
#pragma unroll
            for (int q = 0; q < NT; ++q) red_out[mine + q * T::BAND] = acc[q];
        }
        if constexpr (F32) put_norm(mine, nn);
        else if (on_diagonal) red[mine + NT * T::BAND + m] = acc[NT];
        const int k = k0 + f + (k0 + f >= skip ? 1 : 0);
        const int y = PATCH ? STEP * step + (vt & 3) : step, xc = x0 + (PATCH ? vt >> 2 : vt);
        fetch_shares(y < H && xc < x1 ? part_out + ((size_t)k * N + y * W + xc) * (KK + 1) : nullptr);
    };
    auto anchor_tile = [&](int line, int c, bf16x8 (&tile)[GM][PL]) {
        f32x4 norm = {0.f, 0.f, 0.f, 0.f};
        float nn = 0.f;
#pragma unroll
        for (int gi = 0; gi < GM; ++gi) {
            if (gi < gq) {
                u32x4 fr[2];
                take(fr[0], fr[1]);
                if constexpr (F32) {
                    planes(fr, tile[gi], nn);
                } else {
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const bf16x8 av = __builtin_bit_cast(bf16x8, fr[j]);
                        tile[gi][j] = av;
                        norm = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, av, norm, 0, 0, 0);
                    }
                }
            }
        }
        if (grp == 0) {                                      // one frame group publishes the anchor's norms
            store_shares();
            const size_t mine = (size_t)(buf * kWalkWaves + wave) * T::RED;
            if constexpr (F32) put_norm(mine, nn);
            else if (on_diagonal) red[mine + NT * T::BAND + m] = norm;
            const int y = STEP * step_lo - RAD + (PATCH ? 2 * c + vt / T::SPAN : c);
            const int xc = strip_x(line) + (PATCH ? vt % T::SPAN - RAD : vt - margin);
            fetch_shares(ve == KK && (!PATCH || vt < 2 * T::SPAN) && y >= 0 && y < H && xc >= 0 && xc < W
                             ? A.norm_part + ((size_t)share * A.B + b) * N + y * W + xc : nullptr);
        }
    };

    for (int line = line_lo; line < line_hi; ++line) {
#pragma unroll
        for (int q = 0; q + NEW < NT; ++q) anchor_tile(line, q, win[q + NEW]);
        for (int step = step_lo; step < step_hi; ++step) {
#pragma unroll
            for (int q = 0; q + NEW < NT; ++q) {
#pragma unroll
                for (int gi = 0; gi < GM; ++gi) {
#pragma unroll
                    for (int e = 0; e < PL; ++e) win[q][gi][e] = win[q + NEW][gi][e];
                }
            }
#pragma unroll
            for (int e = 0; e < NEW; ++e) anchor_tile(line, NT - NEW + NEW * (step - step_lo) + e, win[NT - NEW + e]);
            if constexpr (SPEC && F32) {
                for (int f = 0; f < cnt; ++f) {
                    float add[GM][SL] = {};
                    source_tile(f, line, step, add);
#pragma unroll
                    for (int e = 0; e < FRS; ++e) {
                        if (e == f) {                        // (wave-uniform)
#pragma unroll
                            for (int gi = 0; gi < GM; ++gi) sum[e][gi][0] += add[gi][0];
                        }
                    }
                }
            } else if constexpr (SPEC) {
                source_tile(0, line, step, sum[0]);
                if (cnt > 1) source_tile(1, line, step, sum[1]);
                if constexpr (FRS > 2) {
                    if (cnt > 2) source_tile(2, line, step, sum[2]);
                    if (cnt > 3) source_tile(3, line, step, sum[3]);
                }
            } else {
                for (int f = 0; f < cnt; ++f) source_tile(f, line, step, sum[0]);
            }
        }
    }
    store_shares();
    if constexpr (SPEC) {
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int f = 0; f < FRS; ++f) {
            if (f < cnt) {
                float* out = A.strip_sum + (((size_t)b * F + k0 + f) * (deal.lsegs * deal.ysegs) + seg) * A.C + (size_t)q_lo * (128 / sizeof(E));
#pragma unroll
                for (int gi = 0; gi < GM; ++gi) {
                    if (gi < gq) {
                        if constexpr (F32) {
                            // (pieces g and 4 + g of the group: channels 4g .. and 16 + 4g ..)
                            if (!(m & 1)) out[gi * 32 + ((m & 8) ? 16 : 0) + 4 * g + ((m >> 1) & 3)] = sum[f][gi][0];
                        } else {
                            // a lane holds four tokens' worth of channel m (and 16 + m) of a K-step: the four groups of
                            // lanes are added by an fp32 MFMA against ones; 256 bytes per frame and group
                            float total[2];
#pragma unroll
                            for (int j = 0; j < 2; ++j) {
                                const f32x4 r0 = __builtin_amdgcn_mfma_f32_16x16x4f32(1.0f, sum[f][gi][2 * j % SL], zero, 0, 0, 0);
                                const f32x4 r1 = __builtin_amdgcn_mfma_f32_16x16x4f32(1.0f, sum[f][gi][(2 * j + 1) % SL], zero, 0, 0, 0);
                                total[j] = (g & 1) ? r1[0] : r0[0];
                            }
                            out[gi * 64 + lane] = lane < 32 ? total[0] : total[1];
                        }
                    }
                }
            }
        }
    }
}

// The similarities, arg max, gate and keep words from the window products (one wave per keep word, a lane per
// token): the shares of the channels are added in order, candidates are met in ascending order of their
// index, and a NaN wins no comparison.  ALL (tied-batch mode): every similarity of the window is stored to
// win_sim[b][k][cell of the window][i] instead.
// The quotient is formed in 64 bits and rounded once: relative error of the similarities against 64 bits, 30 fp32 shapes
// of 34 to 80 MiB, 5.6e-8 to 7.0e-8 (with fp32 roots and products 7.6e-8 to 8.9e-8; the wave-per-token search that small
// fp32 problems took before 7.5e-8 to 8.6e-8).  Its time is that of the loads: no difference on 14 shapes.
template <int RAD, bool ALL>
__global__ __launch_bounds__(256) void k_walk_finish(const float* __restrict__ part, const float* __restrict__ norm_part,
                                                     const int32_t* __restrict__ anchor_index,
                                                     int32_t* __restrict__ fuse_map, float* __restrict__ best_sim,
                                                     int32_t* __restrict__ best_idx, uint64_t* __restrict__ keep_bits,
                                                     float* __restrict__ win_sim, int B, int F, int H, int W, int NW,
                                                     int nk, float t, size_t words)
{
    constexpr int NP = 2 * RAD + 1, KK = NP * NP;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const size_t wd = (size_t)blockIdx.x * 4 + wave;
    if (wd >= words) return;
    const int N = H * W;
    const size_t frame = wd / NW;
    const int b = (int)(frame / F), k = (int)(frame % F);
    const int i = (int)(wd % NW) * 64 + lane;
    const bool real = i < N;
    const size_t tok = frame * (size_t)N + i;
    const int a = anchor_index[b];
    if (k == a) {                                            // (wave-uniform)
        if constexpr (!ALL) {
            if (real) {
                fuse_map[tok] = -1;
                if (best_sim) best_sim[tok] = 1.0f;
                if (best_idx) best_idx[tok] = i;
            }
            const uint64_t bits = __ballot(real);
            if (lane == 0) keep_bits[wd] = bits;
        }
        return;
    }
    float best = kNegInf;
    int arg = -1;
    if (real) {
        const size_t tokens = (size_t)B * F * N;
        const int y = i / W, xc = i % W;
        float v[KK + 1];
        const float* p = part + tok * (KK + 1);
#pragma unroll
        for (int e = 0; e <= KK; ++e) v[e] = p[e];
        for (int s = 1; s < nk; ++s) {
            p += tokens * (KK + 1);
#pragma unroll
            for (int e = 0; e <= KK; ++e) v[e] += p[e];
        }
#pragma unroll
        for (int dy = -RAD; dy <= RAD; ++dy) {
#pragma unroll
            for (int dx = -RAD; dx <= RAD; ++dx) {
                const int yy = y + dy, xx = xc + dx, cell = (dy + RAD) * NP + dx + RAD;
                if (yy >= 0 && yy < H && xx >= 0 && xx < W) {
                    const int ja = yy * W + xx;
                    float ss = norm_part[(size_t)b * N + ja];
                    for (int s = 1; s < nk; ++s) ss += norm_part[((size_t)s * B + b) * N + ja];
                    const double den2 = (double)v[KK] * (double)ss;
                    const float sim = (float)((double)v[cell] * (den2 > 0.0 ? rsqrt(den2) : 0.0));
                    if constexpr (ALL) {
                        win_sim[(frame * KK + cell) * (size_t)N + i] = sim;
                    } else if (sim > best) {
                        best = sim;
                        arg = ja;
                    }
                }
            }
        }
    }
    if constexpr (!ALL) {
        const bool fused = best > t;                         // keep = 1[s^ <= t]
        if (real) {
            fuse_map[tok] = fused ? arg : -1;
            if (best_sim) best_sim[tok] = best;
            if (best_idx) best_idx[tok] = arg;
        }
        const uint64_t bits = __ballot(real && !fused);
        if (lane == 0) keep_bits[wd] = bits;
    }
}

}  // namespace

// Rounds that this many workgroups take, one per CU at a time.  The last one may not fill the chip; half of its time is
// that of its CUs, half that of the memory (B4 F32 16x16 C4096: 64 / 128 / 256 workgroups 102 / 64 / 46 us).
static double deal_rounds(double units)
{
    const double whole = (double)((long long)units / 256), rest = units - 256 * whole;
    return whole + (rest > 0 ? 0.5 + 0.5 * rest / 256 : 0.0);
}

// How the walk is dealt to workgroups (one per CU at a time).  `frames` are walked per clip.
WalkPlan walk_plan(const ttf_params& p, int frames, bool sums)
{
    WalkPlan w{};
    const int piece = p.dtype == TTF_BF16 ? 64 : 32;         // channels of a group
    const int groups_all = p.C / piece;
    if (p.r > (p.dtype == TTF_BF16 ? 2 : 1) || p.C % piece != 0 || groups_all < kWalkWaves || frames < 1) return w;
    if ((unsigned long long)p.H * p.W * p.C * (128 / piece) >= (1ull << 32)) return w;   // (32-bit offsets inside a frame)
    w.patch = p.r == 2;
    w.nk = (groups_all + kWalkWaves * kWalkGroups - 1) / (kWalkWaves * kWalkGroups);
    w.lines = w.patch ? (p.W + 3) / 4 : (p.W <= 16 ? 1 : (p.W + 15 - 2 * p.r) / (16 - 2 * p.r));
    const int steps = w.patch ? (p.H + 3) / 4 : p.H, fresh = w.patch ? 2 : 1, held = w.patch ? p.r : 2 * p.r;
    // Time of a deal in tiles: a workgroup starts up (two tiles' time), reads the anchor tiles of its run (which
    // come from L2: a third each) and its source tiles.
    // Frame sums are stored per run of the grid: as many runs as leave the products room.
    const long long products = (long long)w.nk * ((2 * p.r + 1) * (2 * p.r + 1) + 1) * p.H * p.W;
    long long most_runs = !sums ? 1 << 20 : p.dtype == TTF_F32 ? 2 : std::max(1ll, spec_strips(p) - (products + p.C - 1) / p.C);
    if (sums && most_runs > 1) {
        WalkPlan all_runs = w;
        all_runs.lsegs = (int)most_runs;
        all_runs.ysegs = 1;
        WalkScratch room{};
        if (!walk_scratch(p, carve(p, nullptr), all_runs, true, room)) most_runs = 1;
    }
    const bool in_cache = (double)p.B * p.F * p.H * p.W * p.C * (p.dtype == TTF_BF16 ? 2 : 4) <= 256.0 * (1 << 20);
    double best = 1e300;
    const int most = !sums ? 32 : p.dtype == TTF_F32 ? spec_frames<float, 1>() : (p.r == 2 ? spec_frames<bf16_t, 2>() : spec_frames<bf16_t, 1>());
    auto deal = [&](int lsegs, int ysegs, double least_units) {   // the frame groups for these runs of the grid
        int last = 0;
        for (int want = 1; want <= most; ++want) {
            const int groups = (frames + want - 1) / want, nf = (frames + groups - 1) / groups;
            if (nf == last) continue;
            last = nf;
            const double units = (double)p.B * w.nk * groups * lsegs * ysegs;
            if (units < least_units || units * (kWalkWaves * 64) >= 4294967296.0) continue;   // (threads of a launch)
            const double lines = (w.lines + lsegs - 1) / lsegs, run = (steps + ysegs - 1) / ysegs;   // (of the longest)
            const double tiles = 2.0 + lines * (run * (nf + 0.35 * fresh) + 0.35 * held);
            const double time = tiles * deal_rounds(units);
            if (time < best) {
                best = time;
                w.tiles = tiles;
                w.nf = nf; w.groups = groups; w.lsegs = lsegs; w.ysegs = ysegs;
            }
        }
    };
    auto next_lsegs = [&](int lsegs) { return std::min(2 * lsegs, lsegs < w.lines ? w.lines : 2 * lsegs); };
    for (int lsegs = 1; lsegs <= w.lines; lsegs = next_lsegs(lsegs)) {
        for (int ysegs = 1; ysegs <= steps && (long long)lsegs * ysegs <= most_runs; ysegs *= 2) {
            // More than four runs only where fewer leave the chip empty, as on tall grids of few columns and frames: with
            // four, segment B1 F6 848x16 C1024 430 us / with as many as it takes 63 (tile-wise kernels 75), tied B1 F2 3428x16
            // C1152 2254 / 401 (457), fp32 tied B1 F2 2868x13 C896 2887 / 247 (486), B2 F10 116x16 C2048 r 0 125 / 81 (105).
            // Elsewhere short runs leave too little of a pass in the Infinity Cache (B2 F256 16x16 C4096, runs of two
            // rows: 669 -> 691).
            if (ysegs > 4 && (double)p.B * w.nk * frames * lsegs * (ysegs / 2) >= 1024) break;
            deal(lsegs, ysegs, 0.0);
        }
    }
    // Three, five and six runs where they fill the chip better by more than 5 %: grids of few tiles a column, which powers of two
    // cut unevenly (97 of 600 drawn shapes up to 700 MiB, 0.94 of the time on average, 0.81 to 1.03: segment B1 F68 20x16 C3200 r 2, five rows
    // of patches, 71 us on 184 workgroups of one run, 58 on 240 of five, tile-wise kernels 69; segment B1 F33 18x32 C2368 57 / 48.5 / 57;
    // less than 5 % 0.99 on average; fewer than 128 workgroups 1.00 to 1.03).  More than four beyond the Infinity Cache only where
    // two leave the chip empty.  Not with sums, whose number of runs is limited by their room.
    if (!sums) {
        best *= 0.95;
        for (int lsegs = 1; lsegs <= w.lines; lsegs = next_lsegs(lsegs)) {
            for (int ysegs : {3, 5, 6}) {
                if (ysegs > steps || (ysegs > 4 && !in_cache && (double)p.B * w.nk * frames * lsegs * 2 >= 1024)) break;
                deal(lsegs, ysegs, 128.0);
            }
        }
    }
    w.ok = best < 1e300;
    return w;
}

// What the guess saves where every clip has a clear one, and how many clips need one: beside unclear clips it saves
// their share of a read and costs two searches and a pass for frame sums that may each fill part of the chip.  B16 F32
// 16x16 C4096: walk with sums 180 us where all guesses are clear, 164 + 155 for sums without; with 12 clear ones of 16
// walks 151 + 114 and sums 84.  With fewer than min_trusted the guesses of all clips are dropped in the first walk.
// The times are those of the model of walk_plan(): a tile of 2048 (fp32 1024) channels takes 2.5 us (fp32 3.0, 5x5 window
// 2.8), with sums 1.04, 1.2 and 1.0 of that; the guess channels 5.5 TB/s, or 4 us for what a block has in flight; a pass for
// frame sums 6.6 TB/s, or 0.8 (few blocks) to 2.6 us (one on every CU) for every eight rows of a frame.  Measured ratio of
// taking the guesses to dropping them / the model's: B16 F32 16x16 C4096, 12 of 16 clear, 1.07 / 1.09; B8 F20 24x24 C2048,
// 6 of 8, 1.27 / 1.5; B128 F16 16x16 C2048, 124 of 128, 0.88 / 0.81; B32 F20 24x24 C2048, 31 of 32, 0.89 / 0.92.
// The launches beside them, and what the model leaves out of the 5x5 window, of few channels and of sums in many runs of
// the grid, are 10 to 70 us, fitted to 100 shapes of 256 MiB to 2 GiB.  Saved by the model / measured: B16 F32 16x16 C4096
// 113 / 115, B16 F64 16x16 C1024 12 / 15, B2 F64 32x32 C1024 -17 / -20, B23 F14 32x16 C2048 60 / 50, B9 F24 24x14 C2048 8 / 8,
// B5 F40 12x48 C2304 5 / -4; 5x5 window B4 F64 32x32 C4096 117 / 163, B4 F40 32x26 C1536 -65 / -60, B3 F64 27x16 C2304 -31 / -11;
// fp32 B16 F32 16x16 C4096 185 / 198, B7 F33 32x16 C1088 3 / 11; many runs B1 F32 200x16 C4096 53 / 48, B1 F64 64x64 C1024
// -16 / -12.
// A guess that is dropped costs the pass over its channels, the pick and a walk that does nothing: model / measured B16 F66
// 16x16 C2048 49 / 45, B8 F128 16x16 C4096 44 / 47, B30 F65 16x16 C1536 70 / 70, B3 F126 32x14 C4096 r 0 40 / 42, fp32 B4 F100 16x16
// C4096 43 / 43.
GuessCost guess_cost(const ttf_params& p, const WalkPlan& first, const WalkPlan& again)
{
    const bool f32 = p.dtype == TTF_F32;
    const double tile = (f32 ? 3.0 : (p.r == 2 ? 2.8 : 2.5)) * p.C / (first.nk * (f32 ? 1024.0 : 2048.0));
    const double with_sums = f32 ? 1.2 : (p.r == 2 ? 1.0 : 1.04);
    const double clip = (double)p.F * p.H * p.W * p.C * (f32 ? 4 : 2) / 6.6e6;
    const double units = (double)first.nk * first.groups * first.lsegs * first.ysegs;
    auto sums = [&](int n) {
        const double blocks = (double)n * p.F * p.C * (f32 ? 4 : 2) / 4096;
        return std::max(n * clip, std::min(p.B * clip, (double)p.H * p.W / 8 * (0.8 + 1.8 * std::min(1.0, blocks / 256))));
    };
    auto walk = [&](int n) { return tile * first.tiles * deal_rounds(units * n); };
    const double without = p.B * clip + tile * again.tiles * deal_rounds((double)p.B * again.nk * again.groups * again.lsegs * again.ysegs);
    GuessCost cost{};
    const int in_flight = f32 ? 32 : 64, rows = (p.H * p.W + guess_parts(p) - 1) / guess_parts(p);   // of a block of k_guess_sums
    const double guess = std::max(p.B * clip * 1.2 * kGuessChannels / p.C, 4.0 * ((rows + in_flight - 1) / in_flight));
    const double launches = f32 ? 10.0 : 20.0 + (p.F > 32 ? 8.0 : 0.0) + (p.C < 1536 ? 8.0 : 0.0) + (p.r == 2 ? 25.0 : 0.0) +
                                             (first.lsegs * first.ysegs > 8 ? 20.0 : 0.0);
    cost.saves = without - with_sums * walk(p.B) - guess - launches;
    cost.dropped = guess + 24.0;
    cost.min_trusted = p.B + 1;
    const int step = (p.B + 63) / 64;                        // (no more than 64 of the counts are looked at)
    for (int n = p.B; n > 0; n -= step) {
        const int rest = p.B - n;
        const double time = with_sums * walk(n) + (rest > 0 ? sums(rest) + walk(rest) : 0.0);
        if (time > without) break;
        cost.min_trusted = n;
    }
    return cost;
}

// The scratch of the walk in the strip-sum and fragment sections of the workspace, where they have room.
bool walk_scratch(const ttf_params& p, const Workspace& w, const WalkPlan& plan, bool sums, WalkScratch& scratch)
{
    const size_t tokens = (size_t)p.B * p.F * p.H * p.W, KK = (size_t)(2 * p.r + 1) * (2 * p.r + 1);
    char* base[2] = {reinterpret_cast<char*>(w.strip_sum), reinterpret_cast<char*>(w.anchor_frag)};
    size_t room[2] = {w.strip_bytes, w.frag_bytes};
    bool fits = true;
    auto take = [&](size_t floats) -> float* {
        const size_t n = align_up(floats * sizeof(float), 256);
        for (int i = 0; i < 2; ++i) {
            if (n > room[i]) continue;
            char* at = base[i];
            base[i] += n;
            room[i] -= n;
            return reinterpret_cast<float*>(at);
        }
        fits = false;
        return nullptr;
    };
    scratch.part = take(plan.nk * tokens * (KK + 1));
    // (sums of one run are whole frame sums and stand in their own section)
    const size_t runs = (size_t)plan.lsegs * plan.ysegs;
    scratch.strip_sum = !sums ? nullptr : (runs == 1 ? w.frame_sum : take((size_t)p.B * p.F * runs * p.C));
    scratch.norm_part = take((size_t)plan.nk * p.B * p.H * p.W);
    // the guess has sections of its own beside bf16 tokens
    scratch.guess_sum = w.guess_sum;
    scratch.spec = w.spec;
    if (sums && p.dtype == TTF_F32) {
        scratch.guess_sum = take((size_t)p.B * p.F * guess_parts(p) * kGuessChannels);
        scratch.spec = reinterpret_cast<int32_t*>(take((size_t)p.B * 4));
    }
    return fits;
}

hipError_t launch_search_walk(const ttf_params& p, const void* x, const void* ext_anchor, const Workspace& w,
                              const WalkPlan& plan, const WalkPlan& all, const WalkScratch& scratch, int32_t* anchor_index,
                              bool anchor_given, int mode, int min_trusted, hipStream_t s)
{
    WalkArgs a{};
    a.x = static_cast<const char*>(x);
    a.ext_anchor = static_cast<const char*>(ext_anchor);
    a.score_part = w.score_part;
    a.clip_part = w.clip_part;
    a.anchor_index = anchor_index;
    a.spec = w.spec;
    a.part = scratch.part;
    a.norm_part = scratch.norm_part;
    a.strip_sum = scratch.strip_sum;
    a.B = p.B; a.F = p.F; a.H = p.H; a.W = p.W; a.C = p.C; a.S = (p.C + 255) / 256;
    a.nk = plan.nk; a.lines = plan.lines;
    a.deal = {plan.lsegs, plan.ysegs, plan.groups, plan.nf};
    a.all = {all.lsegs, all.ysegs, all.groups, all.nf};
    a.fixed_anchor = anchor_given ? kAnchorGiven : fixed_frame(p);
    a.mode = mode;
    a.min_trusted = min_trusted;
    a.keep_from = 256 - (int)(256 * kept_share(p, true, true));
    auto units = [&](const WalkPlan& w) { return (size_t)p.B * w.nk * w.groups * w.lsegs * w.ysegs; };
    const unsigned grid = (unsigned)(mode == 2 ? std::max(units(plan), units(all)) : units(plan));
    auto go = [&](auto kernel, size_t lds) {
        const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kernel), lds);
        if (e != hipSuccess) return e;
        kernel<<<grid, kWalkWaves * 64, lds, s>>>(a);
        return hipGetLastError();
    };
    const bool sums = mode == 1;
#define TTF_WALK(E, RAD, PATCH) \
    (sums ? go(k_search_walk<E, RAD, PATCH, true>, Tiles<RAD, PATCH>::LDS) : go(k_search_walk<E, RAD, PATCH, false>, Tiles<RAD, PATCH>::LDS))
    if (p.dtype == TTF_F32) return p.r == 0 ? TTF_WALK(float, 0, false) : TTF_WALK(float, 1, false);
    return p.r == 0 ? TTF_WALK(bf16_t, 0, false) : (p.r == 1 ? TTF_WALK(bf16_t, 1, false) : TTF_WALK(bf16_t, 2, true));
#undef TTF_WALK
}

hipError_t launch_walk_finish(const ttf_params& p, const Workspace& w, const WalkPlan& plan, const WalkScratch& scratch,
                              const int32_t* anchor_index, int32_t* fuse_map, float* best_sim, int32_t* best_idx,
                              float* win_sim, hipStream_t s)
{
    const int NW = (p.H * p.W + 63) / 64;
    const size_t words = (size_t)p.B * p.F * NW;
    auto go = [&](auto kernel) {
        kernel<<<(unsigned)((words + 3) / 4), 256, 0, s>>>(scratch.part, scratch.norm_part, anchor_index, fuse_map, best_sim,
                                                           best_idx, w.keep_bits, win_sim, p.B, p.F, p.H, p.W, NW, plan.nk,
                                                           p.t, words);
        return hipGetLastError();
    };
    switch (p.r) {
        case 0: return win_sim ? go(k_walk_finish<0, true>) : go(k_walk_finish<0, false>);
        case 1: return win_sim ? go(k_walk_finish<1, true>) : go(k_walk_finish<1, false>);
        case 2: return win_sim ? go(k_walk_finish<2, true>) : go(k_walk_finish<2, false>);
    }
    return hipErrorInvalidValue;
}

}  // namespace ttf
