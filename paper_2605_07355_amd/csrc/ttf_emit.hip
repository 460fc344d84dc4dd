// Sequence compaction and positional alignment (Section 3: stacked X' = [anchor rows ; kept
// source rows], retention mask m_{k,i}, gather of X and P by I_keep, L' = N + P).
//
// The search leaves one keep bit per token.  Small and ordinary calls count the rows ahead of a run of
// keep words where they are needed (anchor frame first inside each clip, clips packed one after the
// other); on large ones, and for short rows, a single small block turns per-frame popcounts into output
// row offsets first.  Every kept row is copied bit-exactly, with its original (k, y, x) triple and flat index.
#include "ttf_device.h"
#include "ttf_internal.h"

namespace ttf {
namespace {

constexpr int kPlaceWords = 16;                // keep words per block of k_place_ids
// The forms of the row placement, us of a re-gating call with a third of the tokens kept (graph replays):
// k_place_rows / k_place_ids + k_copy_rows / scan + k_emit_ids + k_copy_rows.
//   256 words: 1 KiB rows 8.8 / 10.2 / 11.6, 4 KiB rows (64 MiB) 15.1 / 16.1 / 17.7, 8 KiB (128 MiB) 23.6 / 23.1 / 24.4;
//   384 words, 2 KiB rows (48 MiB): 14.7 / 14.5 / 16.0;  512 words, 2 KiB rows (64 MiB): 16.9 / 16.3 / 17.5;
//   1024 words, 1 KiB rows: 20.9 / 16.8 / 17.7.
// A wave of k_place_rows copies up to four rows one after the other, so rows have a limit too.  Re-gating 64 words of
// 6144-byte rows 11.7 / 12.1 / 13.6, 8704 bytes 14.4 / 13.8 / 14.8, 12 000 bytes 18.2 / 16.0 / 17.4, 4 words of 128 KiB
// rows 52 / 24 / 26.  Whole calls also lose a launch: segment B5 F5 9x21, 8704-byte fp32 rows 71.4 / 75.3 / 77.0, bf16
// 74.1 / 75.0 / 76.3; compress B4 F8 14x14, 7200 bytes 88.6 / 90.4 / 92.9, 9616 bytes 111.9 / 112.4 / 113.4, 10 400
// bytes 119.1 / 118.4 / 120.5; B1 F12 16x16, 12 288-byte bf16 rows 63.5 / 61.7 / 63.5.  (Rows that are not whole
// 16-byte pieces are copied by a wave each in every form.)
// Counting in every block of k_place_ids against the scan: 4096 words 39.4 / 41.7, 8192 69.3 / 73.0, 16384 131.6 /
// 137.0 (1 KiB rows); the line stands below the crossing, which was not met.
constexpr size_t kPlaceAllWords = 256;         // at most this many keep words: offsets, ids and rows in one launch
constexpr size_t kPlaceAllBytes = 64ull << 20; // ... and this much input
constexpr size_t kPlaceAllRow = 10240;         // ... in rows of whole 16-byte pieces of at most this length
constexpr size_t kPlaceIdsWords = 4096;        // at most this many: offsets and ids in one launch

// Exclusive scan over the sequence  [N, c(b,0), ..., c(b,F-1)]  for b = 0..B-1, where c(b,k) is
// the number of kept tokens of source frame k and 0 for the anchor frame.  The entry in front
// of each clip places its N anchor rows first.
__global__ __launch_bounds__(1024) void k_offsets_scan(const uint64_t* __restrict__ keep_bits,
                                                       const int32_t* __restrict__ anchor_index,
                                                       int32_t* __restrict__ frame_base,
                                                       int32_t* __restrict__ kept_count,
                                                       int32_t* __restrict__ row_offsets,
                                                       int B, int F, int N, int NW)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    __shared__ int wave_tot[16];
    __shared__ int carry_s;
    if (tid == 0) carry_s = 0;
    __syncthreads();
    const long long E = (long long)B * (F + 1);
    for (long long e0 = 0; e0 < E; e0 += 1024) {
        const long long e = e0 + tid;
        int v = 0, b = 0, s = 0, a = 0;
        if (e < E) {
            b = (int)(e / (F + 1));
            s = (int)(e % (F + 1));
            a = anchor_index[b];                       // < 0: the anchor frame is not part of the clip
            if (s == 0) {
                v = a < 0 ? 0 : N;
            } else if (s - 1 != a) {
                const uint64_t* kb = keep_bits + ((size_t)b * F + (s - 1)) * NW;
                for (int q = 0; q < NW; ++q) v += __popcll(kb[q]);
            }
        }
        int inc = v;                                   // inclusive scan inside the wave
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_up(inc, d, 64);
            if (lane >= d) inc += o;
        }
        if (lane == 63) wave_tot[wave] = inc;
        __syncthreads();
        int pre = carry_s;
        for (int q = 0; q < wave; ++q) pre += wave_tot[q];
        const int excl = pre + inc - v;
        if (e < E) {
            if (s == 0) {
                row_offsets[b] = excl;
                if (a >= 0) frame_base[(size_t)b * F + a] = excl;
            } else if (s - 1 != a) {
                frame_base[(size_t)b * F + (s - 1)] = excl;
            }
        }
        __syncthreads();
        if (tid == 1023) carry_s = excl + v;
        __syncthreads();
    }
    if (tid == 0) row_offsets[B] = carry_s;
    __syncthreads();
    for (int b = tid; b < B; b += 1024) kept_count[b] = row_offsets[b + 1] - row_offsets[b];
}

// One block = 16 tokens (a quarter of a 64-token keep word) of one frame; its kept tokens are dealt
// to the four waves by rank.  tied_rows > 0 (tied-batch mode): keep bits and frame bases are shared
// by all clips ([F,NW] and [F]), clip b writes its rows at row b*tied_rows + shared row, and only
// clip 0 writes the shared position ids and source indices.  Small blocks matter: a wave copies its rows one after the other, so
// the fewer rows per wave, the more copies are in flight across the chip.
template <int U>
__global__ __launch_bounds__(256) void k_emit_rows(const char* __restrict__ x,
                                                   const uint64_t* __restrict__ keep_bits,
                                                   const int32_t* __restrict__ frame_base,
                                                   char* __restrict__ tokens_out,
                                                   int32_t* __restrict__ pos_ids,
                                                   int32_t* __restrict__ src_index,
                                                   int F, int N, int W, int NW, size_t row_bytes, size_t cap,
                                                   int frame_offset, size_t tied_rows)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int quarter = blockIdx.x & 3;
    const int word = (blockIdx.x >> 2) % NW;
    const size_t frame = (blockIdx.x >> 2) / NW;
    const int k = (int)(frame % F);
    const size_t meta = tied_rows ? (size_t)k : frame;        // which frame's bits and base to use
    const size_t row0 = tied_rows ? (frame / F) * tied_rows : 0;
    const bool ids = !tied_rows || frame < (size_t)F;
    const uint64_t* kb = keep_bits + meta * (size_t)NW;
    const uint64_t wbits = kb[word];
    const uint64_t bits = wbits & (0xffffull << (16 * quarter));
    if (bits == 0) return;
    int before = frame_base[meta];
    for (int q = 0; q < word; ++q) before += __popcll(kb[q]);
    before += __popcll(wbits & ((1ull << (16 * quarter)) - 1ull));
    uint64_t rem = bits;
    for (int rank = 0; rem != 0; ++rank) {
        const int bit = __ffsll((unsigned long long)rem) - 1;
        rem &= rem - 1;
        if ((rank & 3) != wave) continue;
        const int i = word * 64 + bit;
        const size_t row = (size_t)before + rank;
        copy_row<U>(x + (frame * (size_t)N + i) * row_bytes, tokens_out + (row0 + row) * row_bytes, row_bytes, lane);
        if (ids && lane == 0) {
            pos_ids[row] = k + frame_offset;
            pos_ids[cap + row] = i / W;
            pos_ids[2 * cap + row] = i % W;
            src_index[row] = k * N + i;
        }
    }
}

// Rows placed ahead of a run of keep words, counted by the block itself from the keep words (no scan in
// front): the anchor frame's keep bits are all set, so the rows of every clip before b and of the words of
// clip b before `word` are their popcounts.  All 256 threads call it; every thread gets both counts.
__device__ __forceinline__ void count_rows_before(const uint64_t* __restrict__ keep_bits, size_t clip_word,
                                                  size_t word, int& clips, int& words)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __shared__ int part[2][4];
    int c = 0, m = 0;
    const size_t end = clip_word + word;
#pragma unroll 8
    for (size_t i = threadIdx.x; i < end; i += 256) {
        const int n = __popcll(keep_bits[i]);
        c += i < clip_word ? n : 0;
        m += i < clip_word ? 0 : n;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        c += __shfl_xor(c, d, 64);
        m += __shfl_xor(m, d, 64);
    }
    if (lane == 0) { part[0][wave] = c; part[1][wave] = m; }
    __syncthreads();
    clips = (part[0][0] + part[0][1]) + (part[0][2] + part[0][3]);
    words = (part[1][0] + part[1][1]) + (part[1][2] + part[1][3]);
}

// Output row of the first kept token of a keep word of frame k: `clips` rows of the clips before, `words`
// kept tokens of the clip's words before it (in flat order).  The anchor frame a comes first: its rows
// stand ahead of every frame before it, and its own words are full.
__device__ __forceinline__ int first_row(int clips, int words, int k, int a, int word_in_frame, int N)
{
    return clips + (k == a ? 64 * word_in_frame : (k < a ? words + N : words));
}

// Offsets, ids and rows in one launch, for calls of at most kPlaceAllWords keep words: there the copy is
// short and the two launches ahead of it (offsets, ids) take longer than their work.  Block = 16 tokens
// (a quarter of a keep word) of one frame, its kept tokens dealt to the four waves by rank; it counts the rows
// ahead of it itself (whole calls: B1 F4 8x8 C256 fp32 28.9 -> 23.8 us, segment
// of B1 F8 16x16 C4096 29.1 -> 24.4, B1 F32 16x16 C2048 50.5 -> 47.4).  Larger calls and longer rows keep the
// faster copy of k_copy_rows.  tied_rows as for k_emit_rows: blockIdx.y = clip, the mask is the shared one ([F,NW]).
//
// Blocks go round robin to the XCDs, and inside an XCD to its CUs.  Frames of at most 48 tokens: the quarter a block
// takes moves on with its word, so that the filled quarters meet every XCD.  Longer frames keep quarters in block
// order, the order of the wave-per-token search, whose rows then lie in the XCD's own L2 (B1 F4 28x16 C912 fp32, kernel
// alone: 6.1 us, with moving quarters 10.4).  Each 256 blocks are turned by five CUs against those before, so that anchor
// frames a power of two of words apart do not meet on one CU.  Re-gating, quarters in block order -> so: B64 F4 4x4,
// 8 KiB rows 26.2 -> 14.1 us, B4 F64 8x8, 4 KiB rows 18.9 -> 15.5.
template <int U>
__global__ __launch_bounds__(256) void k_place_rows(const char* __restrict__ x, const uint64_t* __restrict__ keep_bits,
                                                    const int32_t* __restrict__ anchor_index,
                                                    int32_t* __restrict__ kept_count, int32_t* __restrict__ row_offsets,
                                                    char* __restrict__ tokens_out, int32_t* __restrict__ pos_ids,
                                                    int32_t* __restrict__ src_index, int F, int N, int W, int NW,
                                                    size_t row_bytes, size_t cap, int frame_offset, size_t tied_rows)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned turn = (blockIdx.x | 255u) < gridDim.x ? 40u * (blockIdx.x >> 8) : 0u;
    const unsigned slot = (blockIdx.x & ~255u) | ((blockIdx.x + turn) & 255u);
    const int wd = (int)(slot >> 2);                         // keep word over all clips
    const int quarter = (int)((slot + (N <= 48 ? slot >> 3 : 0u)) & 3u);
    const int per_clip = F * NW;
    const int b = wd / per_clip, word = wd % per_clip;
    const int k = word / NW, q = word % NW;
    const bool ids = blockIdx.y == 0;
    const uint64_t wbits = keep_bits[wd];
    const bool last = word == per_clip - 1 && quarter == 3 && ids;   // this block closes the clip's counts
    uint64_t rem = wbits & (0xffffull << (16 * quarter));
    if (rem == 0 && !last) return;
    int clips, words;
    count_rows_before(keep_bits, (size_t)b * per_clip, word, clips, words);
    if (last && threadIdx.x == 0) {
        const int kept = words + __popcll(wbits);
        if (b == 0) row_offsets[0] = 0;
        row_offsets[b + 1] = clips + kept;
        kept_count[b] = kept;
    }
    const size_t frame = (tied_rows ? (size_t)blockIdx.y * F : (size_t)b * F) + k;
    const size_t row0 = blockIdx.y * tied_rows;
    const size_t first = (size_t)first_row(clips, words, k, anchor_index[b], q, N) +
                         __popcll(wbits & ((1ull << (16 * quarter)) - 1ull));
    for (int rank = 0; rem != 0; ++rank) {
        const int bit = __ffsll((unsigned long long)rem) - 1;
        rem &= rem - 1;
        if ((rank & 3) != wave) continue;
        const int i = q * 64 + bit;
        const size_t row = first + rank;
        copy_row<U>(x + (frame * (size_t)N + i) * row_bytes, tokens_out + (row0 + row) * row_bytes, row_bytes, lane);
        if (ids && lane == 0) {
            pos_ids[row] = k + frame_offset;
            pos_ids[cap + row] = i / W;
            pos_ids[2 * cap + row] = i % W;
            src_index[row] = k * N + i;
        }
    }
}

// Rows of 1 KiB and more are emitted in two steps, so that the copy runs in the shape a plain device
// copy is fastest in on this chip -- many small blocks, a whole block on one row, one or two 16-byte
// pieces per thread (measured on 1 GiB: 6.4-6.5 TB/s against 5.8 for eight pieces per lane in a
// loop) -- without launching blocks for fused tokens (a block per input token costs 0.17 ms of
// launches alone on 262 144 tokens of which 17 % are kept).
//
// Step 1: the offsets (row_offsets, kept_count), the ids of every kept token and, in src_row[r], the input
// token that output row r copies.  Block = kPlaceWords consecutive keep words of one clip, which counts the
// rows ahead of it itself from L2 instead of waiting for a scan kernel (figures above, at the constants).
// Tied-batch mode: the mask is the shared one, one clip.
__global__ __launch_bounds__(256) void k_place_ids(const uint64_t* __restrict__ keep_bits,
                                                   const int32_t* __restrict__ anchor_index,
                                                   int32_t* __restrict__ kept_count, int32_t* __restrict__ row_offsets,
                                                   int32_t* __restrict__ pos_ids, int32_t* __restrict__ src_index,
                                                   int32_t* __restrict__ src_row, int F, int N, int W, int NW,
                                                   int runs, size_t cap, int frame_offset)
{
    static_assert(kPlaceWords % 4 == 0 && kPlaceWords <= 64, "whole words per wave, one lane per word");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int per_clip = F * NW;
    const int b = blockIdx.x / runs, run = blockIdx.x % runs;
    const int w0 = run * kPlaceWords;
    const uint64_t* kb = keep_bits + (size_t)b * per_clip;
    int clips, words;
    count_rows_before(keep_bits, (size_t)b * per_clip, w0, clips, words);
    // kept tokens of the run's words: lane l holds word w0 + l, inclusive sums over the lanes
    const int n = (lane < kPlaceWords && w0 + lane < per_clip) ? __popcll(kb[w0 + lane]) : 0;
    int inc = n;
#pragma unroll
    for (int d = 1; d < kPlaceWords; d <<= 1) {
        const int o = __shfl_up(inc, d, 64);
        if (lane >= d) inc += o;
    }
    if (run == runs - 1 && threadIdx.x == kPlaceWords - 1) {
        if (b == 0) row_offsets[0] = 0;
        row_offsets[b + 1] = clips + words + inc;
        kept_count[b] = words + inc;
    }
    const int a = anchor_index[b];
    for (int u = wave; u < kPlaceWords && w0 + u < per_clip; u += 4) {   // wave-uniform
        const int ahead = words + __shfl(inc - n, u, 64);
        const int word = w0 + u, k = word / NW, q = word % NW;
        const uint64_t wbits = kb[word];
        if (((wbits >> lane) & 1ull) == 0) continue;
        const size_t row = (size_t)first_row(clips, ahead, k, a, q, N) + __popcll(wbits & ((1ull << lane) - 1ull));
        const int i = q * 64 + lane;
        pos_ids[row] = k + frame_offset;
        pos_ids[cap + row] = i / W;
        pos_ids[2 * cap + row] = i % W;
        src_index[row] = k * N + i;
        src_row[row] = (int32_t)(((size_t)b * F + k) * (size_t)N + i);
    }
}

// The same ids behind k_offsets_scan, one wave per keep word: calls of more than kPlaceIdsWords keep words.
// Tied-batch mode: `words` and the mask are the shared ones ([F,NW]); ids and src_row are those of one clip.
__global__ __launch_bounds__(256) void k_emit_ids(const uint64_t* __restrict__ keep_bits,
                                                  const int32_t* __restrict__ frame_base,
                                                  int32_t* __restrict__ pos_ids, int32_t* __restrict__ src_index,
                                                  int32_t* __restrict__ src_row, int F, int N, int W, int NW,
                                                  size_t words, size_t cap, int frame_offset)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const size_t wd = (size_t)blockIdx.x * 4 + wave;
    if (wd >= words) return;
    const int word = (int)(wd % NW);
    const size_t frame = wd / NW;
    const int k = (int)(frame % F);
    const uint64_t* kb = keep_bits + frame * (size_t)NW;
    const uint64_t wbits = kb[word];
    if (((wbits >> lane) & 1ull) == 0) return;
    int before = frame_base[frame];
    for (int q = 0; q < word; ++q) before += __popcll(kb[q]);
    const size_t row = (size_t)before + __popcll(wbits & ((1ull << lane) - 1ull));
    const int i = word * 64 + lane;
    pos_ids[row] = k + frame_offset;
    pos_ids[cap + row] = i / W;
    pos_ids[2 * cap + row] = i % W;
    src_index[row] = k * N + i;
    src_row[row] = (int32_t)(frame * (size_t)N + i);
}

// Step 2: block j copies output rows j, j + gridDim.x, ... below *total_rows.  blockIdx.y = clip in
// tied-batch mode (input tokens src_clip_stride apart, output rows dst_clip_stride apart), 0 otherwise.
__global__ __launch_bounds__(256) void k_copy_rows(const char* __restrict__ x, const int32_t* __restrict__ src_row,
                                                   const int32_t* __restrict__ total_rows,
                                                   char* __restrict__ tokens_out, size_t row_bytes,
                                                   size_t src_clip_stride, size_t dst_clip_stride)
{
    const int total = *total_rows;
    const int n = (int)(row_bytes / 16);
    const int step = (int)blockDim.x;
    const char* xs = x + blockIdx.y * src_clip_stride * row_bytes;
    char* out = tokens_out + blockIdx.y * dst_clip_stride * row_bytes;
    for (int r = blockIdx.x; r < total; r += gridDim.x) {
        const uint4* s = reinterpret_cast<const uint4*>(xs + (size_t)src_row[r] * row_bytes);
        uint4* d = reinterpret_cast<uint4*>(out + (size_t)r * row_bytes);
        int q = threadIdx.x;
        for (; q + step < n; q += 2 * step) {
            const uint4 v0 = load16_stream(s + q), v1 = load16_stream(s + q + step);
            store16_stream(d + q, v0);
            store16_stream(d + q + step, v1);
        }
        if (q < n) store16_stream(d + q, load16_stream(s + q));
    }
}

// How the rows of a call are placed.
enum class Placement { all, ids, scan };
constexpr size_t kRowBlockMin = 1024;          // shortest rows that k_copy_rows takes
inline Placement placement(const ttf_params& p, bool tied)
{
    const size_t words = (size_t)(tied ? 1 : p.B) * p.F * (((size_t)p.H * p.W + 63) / 64);
    const size_t row_bytes = (size_t)p.C * (p.dtype == TTF_BF16 ? 2 : 4);
    const size_t tokens_bytes = (size_t)p.B * p.F * p.H * p.W * row_bytes;
    if (tied && p.B > 65535) return Placement::scan;         // (clips ride on gridDim.y)
    const bool by_wave = row_bytes <= kPlaceAllRow || row_bytes % 16 != 0;
    if (words <= kPlaceAllWords && tokens_bytes <= kPlaceAllBytes && by_wave) return Placement::all;
    if (row_bytes % 16 == 0 && row_bytes >= kRowBlockMin && words <= kPlaceIdsWords) return Placement::ids;
    return Placement::scan;
}

}  // namespace

hipError_t launch_offsets_scan(const ttf_params& p, const Workspace& w, const int32_t* anchor_index,
                               int32_t* kept_count, int32_t* row_offsets, bool tied, hipStream_t s)
{
    const int N = p.H * p.W, NW = (N + 63) / 64;
    if (placement(p, tied) != Placement::scan) return hipSuccess;   // the emission counts for itself
    // tied-batch mode: one shared mask, i.e. the scan of a single clip
    k_offsets_scan<<<1, 1024, 0, s>>>(w.keep_bits, anchor_index, w.frame_base, kept_count, row_offsets,
                                      tied ? 1 : p.B, p.F, N, NW);
    return hipGetLastError();
}

hipError_t launch_emit_rows(const ttf_params& p, const void* x, const Workspace& w,
                            const int32_t* anchor_index, int32_t* kept_count, int32_t* row_offsets,
                            void* tokens_out, int32_t* pos_ids, int32_t* src_index, int frame_offset, bool tied,
                            hipStream_t s)
{
    const int N = p.H * p.W, NW = (N + 63) / 64;
    const size_t row_bytes = (size_t)p.C * (p.dtype == TTF_BF16 ? 2 : 4);
    const size_t tied_rows = tied ? (size_t)p.F * N : 0;
    const size_t cap = tied ? tied_rows : (size_t)p.B * p.F * N;  // length of one pos_ids plane
    const unsigned grid = (unsigned)((size_t)p.B * p.F * NW * 4);
    const char* xs = static_cast<const char*>(x);
    char* out = static_cast<char*>(tokens_out);
    const Placement place = placement(p, tied);
    if (place == Placement::all) {
        const unsigned blocks = (unsigned)((size_t)(tied ? 1 : p.B) * p.F * NW * 4);
        auto go = [&](auto kernel) {
            kernel<<<dim3(blocks, tied ? p.B : 1), 256, 0, s>>>(xs, w.keep_bits, anchor_index, kept_count, row_offsets, out,
                                                                pos_ids, src_index, p.F, N, p.W, NW, row_bytes, cap,
                                                                frame_offset, tied_rows);
            return hipGetLastError();
        };
        return row_bytes % 16 == 0 ? go(k_place_rows<16>) : (row_bytes % 4 == 0 ? go(k_place_rows<4>) : go(k_place_rows<2>));
    }
    if (row_bytes % 16 == 0 && row_bytes >= kRowBlockMin && (!tied || p.B <= 65535)) {   // (clips ride on gridDim.y)
        const size_t words = (size_t)(tied ? 1 : p.B) * p.F * NW;
        if (place == Placement::ids) {
            const int runs = (p.F * NW + kPlaceWords - 1) / kPlaceWords;
            k_place_ids<<<(unsigned)((tied ? 1 : p.B) * runs), 256, 0, s>>>(w.keep_bits, anchor_index, kept_count, row_offsets,
                                                                           pos_ids, src_index, w.src_row, p.F, N, p.W, NW,
                                                                           runs, cap, frame_offset);
        } else {
            k_emit_ids<<<(unsigned)((words + 3) / 4), 256, 0, s>>>(w.keep_bits, w.frame_base, pos_ids, src_index, w.src_row,
                                                                  p.F, N, p.W, NW, words, cap, frame_offset);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        // a quarter as many blocks as there could be rows: at the usual kept fractions every block has
        // one to four rows; 64 threads per KiB of row, at most 256
        const unsigned threads = (unsigned)(row_bytes >= 4096 ? 256 : row_bytes / 1024 * 64);
        const size_t want = (cap + 3) / 4;
        const unsigned blocks = (unsigned)(want < kMaxBlocks256 ? want : kMaxBlocks256);
        k_copy_rows<<<dim3(blocks, tied ? p.B : 1), threads, 0, s>>>(xs, w.src_row, row_offsets + (tied ? 1 : p.B), out, row_bytes,
                                                                     tied_rows, tied_rows);
        return hipGetLastError();
    }
    if (row_bytes % 16 == 0)
        k_emit_rows<16><<<grid, 256, 0, s>>>(xs, w.keep_bits, w.frame_base, out, pos_ids, src_index,
                                             p.F, N, p.W, NW, row_bytes, cap, frame_offset, tied_rows);
    else if (row_bytes % 4 == 0)
        k_emit_rows<4><<<grid, 256, 0, s>>>(xs, w.keep_bits, w.frame_base, out, pos_ids, src_index,
                                            p.F, N, p.W, NW, row_bytes, cap, frame_offset, tied_rows);
    else
        k_emit_rows<2><<<grid, 256, 0, s>>>(xs, w.keep_bits, w.frame_base, out, pos_ids, src_index,
                                            p.F, N, p.W, NW, row_bytes, cap, frame_offset, tied_rows);
    return hipGetLastError();
}

}  // namespace ttf
