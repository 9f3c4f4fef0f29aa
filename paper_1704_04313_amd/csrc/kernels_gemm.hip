// Gathered matrix generation + matrix multiplication + output update for gfx950.
//
// Section 3.1 of the paper assembles only the columns of the image matrix X that belong to
// output positions needing an update, multiplies them with the unchanged filter matrix K and
// writes the result (with the activation) over the stored output.  Here the three steps are one
// kernel: a workgroup owns BN output positions to recompute x BM output channels, builds the
// BN x 128-byte slices of the reduced X directly in LDS by gathering 16-byte channel units from
// the channel-contiguous input map, multiplies on the matrix cores and scatters bias + ReLU
// results straight into the stored map.  The reduced X never exists in HBM.
//
// Which positions: all of them in order (dense evaluation: nothing to wait for; reading an identity list
// cost every tile two dependent round trips to memory), from an index list, or -- for maps small enough to be held in LDS -- from the
// map itself.  Every workgroup then loads the map of positions to recompute (or the layer's
// change map, which it first dilates by the filter support), ranks it with popcounts and a scan,
// and picks the positions whose rank falls into its tile: the index extraction and the dilation
// of Section 3.1 without launches of their own.
//
// The workgroup has twelve waves with two roles.  The last four ("producers") compute gather
// addresses and issue the loads that bring the next K slices of both operands from global memory
// straight into LDS; the first eight ("consumers") only read LDS fragments and issue MFMAs
// (v_mfma_f32_16x16x32_bf16, float32 accumulation).  One producer and two consumer waves share each
// SIMD, so address arithmetic and global-load latency overlap the matrix pipeline instead of draining
// it once per slice, and while one consumer wave waits for its fragments the other keeps the pipeline
// fed (measured +2.5 % over one consumer wave per SIMD).
//
// float32 storage multiplies in bfloat16 parts.  A float32 is the exact sum of three bfloat16 (8 bits of
// its 24 each); of the nine products of parts the six down to 2^-24 of the leading one are formed, the
// leading one and the corrections in accumulators of their own.  The matrix unit takes 16 cycles for 32 k
// of a 16 x 16 tile in bfloat16 and 256 in float32, so six products cost 96: the float32 instruction bounded
// these layers at 151 TFLOP/s (measured for a plain product), 64->256 7x7 on 320x180 ran at 126 and
// runs at 218 TFLOP/s (736 -> 425 us), 16->64 7x7 on 640x360 at 105 and 178 (220 -> 130 us).  What bounds
// them now is the bfloat16 matrix rate that the card sustains on such data: 218 x 6 = 1 308 TFLOP/s, the
// plain library product of 8192 and 16384 rows reaches 1 120 to 1 340.  (Figures of single steps further down were
// taken when the step was made and say what it gave.)  The sums are
// more exact than before: 2.8e-7 against 7.1e-7 (2-norm, K = 3 136, against 64 bits), because 32 products
// enter the leading accumulator with one rounding instead of eight; with one accumulator for all
// six the error would be 8.1e-7.  Only a sum of a single nonzero product loses by the three products left
// out: up to 0.7 units of 2^-23 instead of half of one, 2 % more in the 2-norm.  The filter matrix is split
// once, when the state is created, and lies in memory in the order in which it is read; pixels are split in
// registers (3.5 instructions per value) in the shadow of the MFMAs.
//
// Layers of more than 32 channels whose workgroups sum up long ranges of K (halves_suit) take float16 halves and three
// products instead, half the matrix time and two thirds of the filter bytes: 64->256 7x7 on 320x180 407 -> 300 us (308
// TFLOP/s), on 80x60 50.6 -> 44.1, 256->256 3x3 on 160x120 122 -> 96, 512->512 3x3 on 80x60 117 -> 88; 16->64 7x7 on 640x360 131 ->
// 120, 64->64 5x5 on 400x300 133 -> 110, 96->64 3x3 on 640x480 181 -> 154; on pixels of one scale with errors no larger than the
// parts' (figures at kHalfRange), on others by the check of every sum (kHalfBits).  What bounds them is the split of the pixels, 3.5
// vector instructions a value that add to the MFMAs (one instruction less, without the scale: 5 % faster, and wrong for pixels far
// below their brightest neighbours), and the card's clock: on 64 streams the matrix unit is busy 48 % of the time in the
// 128-channel tile, at 1.9 GHz, and 27 % in the 64-channel one, which splits as much for half the MFMAs.
//
// Work distribution: one workgroup per compute unit.  Output tiles are dealt out whole as long
// as every workgroup gets one; the (tiles mod workgroups) left over are cut along K into
// equal iteration ranges, one per workgroup, so that all compute units finish together whatever
// the number of positions is.  A wave that computed only part of a sub-tile's K range stores its
// partial accumulators; the last wave to finish a sub-tile (an atomic ticket, nobody waits)
// adds all parts in ascending K order, which keeps results deterministic, and performs the
// output update.
//
// Layers with short filter-matrix rows and few output channels (a first layer on camera frames, 1x1
// layers) would spend such a launch filling and draining the ring; they run gemm_thin_kernel, in
// which every wave multiplies 16 positions by the whole reduction out of its own registers.
#include "kernels.h"

#include <cfloat>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <type_traits>

namespace cbk {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef floatx4 floatx4_a4 __attribute__((aligned(4))); // a 16-byte unit that starts at any 4-byte word
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short ushortx2 __attribute__((ext_vector_type(2)));

// Partial accumulators cross between workgroups that may sit on different XCDs (separate L2s).
// They are written and read with buffer instructions carrying the sc1 bit: write-through to, and
// read at, the level all XCDs share, so no cache-wide write-back or invalidate is needed.
static constexpr int kDeviceCoherent = 0x10; // cache-policy operand: sc1
__device__ __forceinline__ __amdgpu_buffer_rsrc_t slab_resource(const float *p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p), 0, bytes, 0x00020000);
}


static constexpr int BK = 32;       // K slice per pipeline stage: 128 bytes = 32 floats or 64 bfloat16,
                                    // i.e. 8 units of 16 bytes
static constexpr int KU = 8;        // units per slice
static constexpr int LDK = BK;      // LDS row pitch in 4-byte words: 128 bytes, no padding.  The eight 16-byte
                                    // units of a row are stored permuted (unit u of row r sits in slot
                                    // u ^ lds_swizzle(r)) so that the 16-lane groups of a ds_read_b128
                                    // (16 rows, one or two neighbouring units) and of a ds_write_b128 (two rows,
                                    // all units) each cover all 64 banks once
static constexpr int kConsWaves = 8;              // consumer waves per workgroup (two per SIMD)
static constexpr int kProdWaves = 4;              // producer waves (one per SIMD)
static constexpr int NPROD = 64 * kProdWaves;     // producer threads
static constexpr int kRP = NPROD / 8;             // tile rows staged per pass: eight threads (units) per row
static constexpr int NCONS = 64 * kConsWaves;     // consumer threads: waves 0 .. kConsWaves-1
static constexpr int NT = NCONS + NPROD;          // threads per workgroup
static constexpr int kEpiChunk = 4;       // accumulators whose replaced values are loaded together in the output update
static constexpr int kMinIters = 8;       // shortest K range worth giving to a workgroup
static constexpr int kMaxGrid = 1024;
// Big tiles are used from (workgroups / this) of them on.  128 channels of float32 split further where their K
// range is long enough to be cut for the other workgroups: the small tile reads LDS for longer than it
// multiplies (64->256 7x7, 98 slices, 4 800 positions: 60 us with 64-pixel tiles, 56 with 128; 64->128 5x5, 50
// slices, 99 tiles of 128 pixels 43.9 and 42.5).  Shorter ranges are better off in small tiles from half the
// workgroups down (64->128 3x3, 18 slices, 20 and 99 tiles: 14.7 and 24.9 us, in big ones 20.6 and 26.6; 128->128
// 1x1, 4 slices, 99 tiles 12.2 and 15.7; 128->128 3x3, 36 slices, 66 tiles 29.0 and 33.8).
__host__ __device__ inline int small_tile_factor(int dtype, int bm, int nk)
{
    return dtype == kF32 && bm == 128 && nk >= 48 ? 4 : 2;
}

// Whether a launch of that many big tiles (channel tile bm) of nk slices multiplies in halves: where the ranges of K that
// workgroups sum up are `range` slices long in the mean over the tiles.  Halves leave off the last of float32's 24 bits
// in a quarter of the values and the product of both second halves, 7.0e-8 of a sum whatever its length; the bfloat16 parts
// are exact but are rounded at the magnitude of the whole sum in every slice, 3.4e-8 sqrt(slices / 2).  Error against 64
// bits (2-norm, halves / parts, pixels of which half are zero): whole ranges of 20 slices 1.17e-7 / 1.10e-7, 22 1.18e-7 / 1.15e-7,
// 23 1.20e-7 / 1.20e-7, 24 1.23e-7 / 1.24e-7, 28 1.23e-7 / 1.36e-7, 36 1.20e-7 / 1.51e-7; 16->64 7x7 (24.5, eight sets of
// weights and pixels) 1.22e-7 / 1.23e-7; 64->256 7x7 (98) 1.43e-7 / 2.62e-7, in three ranges 1.27e-7 / 1.47e-7, in twelve
// 1.30e-7 / 0.95e-7.  So the line is where the errors meet; short ranges are latency, not multiplication (64->256 in
// twelve 19.1 / 20.4 us, the last 22.4 / 25.0).  Zero weights round nothing, so ranges are counted in the nonzero weights
// of the layer's sparsest row (64->256 7x7 with a quarter of them 1.32e-7 / 1.27e-7, with an eighth 1.30e-7 / 0.91e-7).
__host__ __device__ inline bool halves_suit(int bm, int tiles, int whole_rounds, int nk, int grid, int range)
{
    // only where the big tile is used at all: gemm_partial_bytes has no room for its partial sums elsewhere
    if (nk < range || tiles < 1 || (long long)tiles * small_tile_factor(kF32, bm, nk) < grid) return false;
    const int rem = tiles - whole_rounds * grid;
    if (rem == 0) return true;
    // as make_schedule cuts them: into equal parts, or evenly over all workgroups, which then cross from tile to tile
    const int most = nk / kMinIters > 1 ? nk / kMinIters : 1;
    int parts = grid / rem;
    if (parts > most) parts = most;
    const long long ranges = rem * parts * 8 < grid * 7 && rem * most >= grid ? grid + rem : rem * parts;
    return (tiles - rem) * (nk * ranges) + (long long)rem * rem * nk >= range * ranges * tiles;
}

static constexpr int kSelMaxWords = 2048; // largest selection map ranked in-kernel (131072 pixels)
static constexpr int kSelWordsPerThread = (kSelMaxWords + NT - 1) / NT;
static constexpr int kSelSlots = kSelMaxWords + kSelWordsPerThread; // LDS words per ranking array

// 16-byte-per-lane fragments that one slice of 16 filter rows consists of: bfloat16 storage two (the two
// halves of a slice's 64 k), float32 three (the bfloat16 parts of 32 k, see split_fragment) or, in halves, two.
static constexpr int kF32Halves = 2; // besides kF32 and kBF16: float32 storage, multiplied in halves (split_halves)
template <int DT>
static constexpr int kFilterParts = DT == kF32 ? 3 : 2;
template <int DT>
static constexpr int kStorage = DT == kBF16 ? kBF16 : kF32;
static constexpr int kFragBytes = 1024; // one fragment: 64 lanes x 16 bytes

// LDS of one tile shape: a ring of STAGES K slices of both operands, then pixel lists.
template <int DT, int BM, int BN, int STAGES>
struct TileSmem {
    static constexpr int a_floats = BN * LDK;
    static constexpr int b_floats = BM / 16 * kFilterParts<DT> * kFragBytes / 4;
    // Pixel lists: of the segment the consumers finish and of those that the slices after it belong to.
    // A segment has a slice at least; of the 64-channel tiles in float32 (rows of five slices or more, the
    // shorter ones are the thin kernel's) at most two can be that short in a row, and LDS has no room for more.
    static constexpr int lists = DT != kBF16 && BM == 64 && BN == 256 ? 3 : STAGES + 1;
    // with a list go the biases of its tile's channels
    static constexpr int list_words = BN + BM;
    static constexpr int tile_bytes = STAGES * (a_floats + b_floats) * 4 + lists * list_words * 4;
};
// LDS of a kernel instantiation (a big and a small tile shape share it): behind the larger of the
// two tiles the selection map's words, their exclusive ranks, and the wave totals of the scan.
template <int DT, int BM, int BNB, int SB, int BNS, int SS>
struct KernelSmem {
    static constexpr int tb = TileSmem<DT, BM, BNB, SB>::tile_bytes, ts = TileSmem<DT, BM, BNS, SS>::tile_bytes;
    static constexpr int sel_offset = ((tb > ts ? tb : ts) + 15) / 16 * 16;
    static constexpr int bytes = sel_offset + kSelSlots * 12 + 64;
    static_assert(bytes <= 160 * 1024, "a workgroup has 160 KiB of LDS");
};

// Selection-map mode: the words of the map and the rank of each word's first set bit, in LDS.
struct Selection {
    const uint64_t *words; // nullptr: list mode
    const int *rank; // of words behind the last: larger than any
    int top;         // the power of two below the number of words that steps of the search begin with, 0 for one word
};
__device__ __forceinline__ Selection make_selection(const GemmArgs &a, const uint64_t *words, const int *rank)
{
    return {words, rank, a.sel_ranked > 1 ? 1 << (31 - __builtin_clz(a.sel_ranked - 1)) : 0};
}

// Inclusive prefix sum over the 64 lanes of a wave with data-parallel-primitive moves: shifts by
// 1, 2, 4, 8 inside each row of 16 lanes, then lane 15 of a row into the next row (rows 1 and 3)
// and lane 31 into rows 2 and 3.  Lanes without a source add the zero given as the old value.
__device__ __forceinline__ int wave_inclusive_sum(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false); // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false); // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false); // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false); // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false); // row_bcast:15
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false); // row_bcast:31
    return x;
}

// Change maps with a byte per position hold 0 or 1 in each; two dot products gather eight of them into a byte.
__device__ __forceinline__ unsigned byte_flags(unsigned lo, unsigned hi)
{
    return __builtin_amdgcn_udot4(hi, 0x80402010u, __builtin_amdgcn_udot4(lo, 0x08040201u, 0u, false), false);
}
__device__ __forceinline__ unsigned byte_flags(const uint4 &v) { return byte_flags(v.x, v.y) | byte_flags(v.z, v.w) << 8; }

// A map of nw words (64 positions each; bytes: a byte per position) from global memory into LDS as a bitmap, kSelGuard
// zero words before and behind it.  All loads of a thread are under way together.  The caller synchronises.
static constexpr int kSelGuard = 2;
__device__ __forceinline__ void load_bitmap(const uint64_t *__restrict__ map, int bytes, int nw, uint64_t *sM)
{
    const int tid = threadIdx.x;
    if (tid < 2 * kSelGuard) sM[tid < kSelGuard ? tid : nw + tid] = 0ull;
    sM += kSelGuard;
    if (bytes) {
        constexpr int B = 5; // 61 440 positions in a round
        const uint4 *m16 = reinterpret_cast<const uint4 *>(map);
        unsigned short *s16 = reinterpret_cast<unsigned short *>(sM);
        const int n16 = nw * 4;
        for (int i0 = tid; i0 < n16; i0 += B * NT) {
            uint4 v[B];
#pragma unroll
            for (int j = 0; j < B; ++j)
                if (i0 + j * NT < n16) v[j] = m16[i0 + j * NT];
#pragma unroll
            for (int j = 0; j < B; ++j)
                if (i0 + j * NT < n16) s16[i0 + j * NT] = (unsigned short)byte_flags(v[j]);
        }
    } else {
        uint64_t v[kSelWordsPerThread];
#pragma unroll
        for (int j = 0; j < kSelWordsPerThread; ++j)
            if (tid + j * NT < nw) v[j] = map[tid + j * NT];
#pragma unroll
        for (int j = 0; j < kSelWordsPerThread; ++j)
            if (tid + j * NT < nw) sM[tid + j * NT] = v[j];
    }
}

// Dilation by the filter support (Section 3.1, second formula) for a stride-1 layer, from its change map (sC: bits
// in LDS behind the guard): the outputs x .. x + len - 1, at most 64, of output row qy of stream st.  The rows of the
// change map under them are OR-ed as windows of 96 bits, then the kw shifted copies of the window by
// doubling.  `lanes` lanes take a tap row each, in turn, from the one of number `first` on.
__device__ __forceinline__ uint64_t dilated_piece(const GemmArgs &a, const unsigned *sC, int st, int qy, int x, int len, int first,
                                                  int lanes)
{
    constexpr int R = 4; // rows read together
    const int xs = x - a.pad; // the window's first column
    const int bit = ((st * a.H + qy - a.pad) * a.W + xs) + kSelGuard * 64;
    unsigned w0 = 0, w1 = 0, w2 = 0;
    const int j0 = a.pad - qy > 0 ? a.pad - qy : 0; // tap rows j0 .. j0 + jn - 1 lie in the image
    const int j1 = a.H + a.pad - qy, jn = (j1 < a.kh ? j1 : a.kh) - j0;
#pragma unroll 1
    for (int jb = 0; jb < a.kh; jb += R * lanes) {
        unsigned m[R][4], sh[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int j = jb + first + r * lanes;
            // outside the image or behind the filter: the guard's zeros
            const int b = (unsigned)(j - j0) < (unsigned)jn ? bit + j * a.W : 0;
            sh[r] = b & 31;
#pragma unroll
            for (int d = 0; d < 4; ++d) m[r][d] = sC[(b >> 5) + d];
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            w0 |= __builtin_amdgcn_alignbit(m[r][1], m[r][0], sh[r]);
            w1 |= __builtin_amdgcn_alignbit(m[r][2], m[r][1], sh[r]);
            w2 |= __builtin_amdgcn_alignbit(m[r][3], m[r][2], sh[r]);
        }
    }
    // columns outside the image belong to other rows (pad < kw <= 16)
    auto first_bits = [](int n) { // the lowest n bits; all for n >= 32, none for n <= 0
        const int c = n < 0 ? 0 : (n > 32 ? 32 : n);
        return (unsigned)((1ull << c) - 1ull);
    };
    const int in = a.W - xs, before = xs < 0 ? -xs : 0;
    w0 = (w0 & first_bits(in)) >> before << before;
    w1 &= first_bits(in - 32);
    w2 &= first_bits(in - 64);
    int cover = 1; // the window's bits t .. t + cover - 1 are in bit t
#pragma unroll
    for (int q = 0; q < 4; ++q) { // kw <= 16
        const int sft = cover < a.kw - cover ? cover : a.kw - cover;
        w0 |= __builtin_amdgcn_alignbit(w1, w0, sft);
        w1 |= __builtin_amdgcn_alignbit(w2, w1, sft);
        w2 |= w2 >> sft;
        cover += sft;
    }
    return (uint64_t)(w1 & first_bits(len - 32)) << 32 | (w0 & first_bits(len));
}

// Word i of the map of outputs to recompute: inside one output row when rows begin on words (GemmArgs::dSelRow),
// else put together from pieces of rows.
__device__ __forceinline__ uint64_t dilated_word(const GemmArgs &a, const unsigned *sC, int i, int first, int lanes)
{
    const int Ho = a.dHo.d;
    if (a.dSelRow.d) {
        const int row = fast_div(i, a.dSelRow), x = (i - row * a.dSelRow.d) * 64;
        const int st = a.S > 1 ? fast_div(row, a.dHo) : 0;
        return dilated_piece(a, sC, st, row - st * Ho, x, a.Wo - x < 64 ? a.Wo - x : 64, first, lanes);
    }
    const int pos = i * 64, total = a.S * a.No;
    const int row = fast_div(pos, a.dWo);
    int x = pos - row * a.Wo, left = total - pos < 64 ? total - pos : 64, at = 0;
    int st = fast_div(row, a.dHo), qy = row - st * Ho;
    uint64_t word = 0;
#pragma unroll 1
    while (left > 0) {
        const int len = a.Wo - x < left ? a.Wo - x : left;
        word |= dilated_piece(a, sC, st, qy, x, len, first, lanes) << at;
        at += len;
        left -= len;
        x = 0;
        if (++qy == Ho) {
            qy = 0;
            ++st;
        }
    }
    return word;
}

// Word i of a map of a.sel_words words over all outputs, from words of which rows begin on words.
__device__ __forceinline__ uint64_t packed_word(const GemmArgs &a, const uint64_t *sW, int i)
{
    const int total = a.S * a.No, P = a.dSelRow.d;
    int pos = i * 64, at = 0, left = total - pos < 64 ? total - pos : 64;
    int row = fast_div(pos, a.dWo), x = pos - row * a.Wo;
    uint64_t word = 0;
    while (left > 0) {
        const int len = a.Wo - x < left ? a.Wo - x : left, q = x >> 6, sh = x & 63;
        uint64_t v = sW[row * P + q] >> sh;
        if (sh && q + 1 < P) v |= sW[row * P + q + 1] << (64 - sh);
        if (len < 64) v &= (1ull << len) - 1ull;
        word |= v << at;
        at += len;
        left -= len;
        x = 0;
        ++row;
    }
    return word;
}

// Brings the map of positions to recompute into LDS (sW) and ranks it: sRank[i] = number of
// selected positions in the words before word i.  Returns the number of selected positions.
// The map is either given (bits or bytes) or, sel_dilate != 0, derived here from the layer's change map (scratch:
// LDS that the tile ring will use later); the workgroups then share in writing it to a.upd_out for the kernels that
// follow.  All NT threads take part; thread t ranks `per` consecutive words, or 2^sh threads a word between them.
// Three barriers and one pass from the change map to the words: with a pass over rows, one over columns and
// words re-read for the ranking (seven barriers), 4 800 positions under a 7x7 filter took 4.1 us from the
// kernel's start to their number, 57 600 6.5 and 76 800 from bits 5.6; now 2.7, 4.7 and 4.5 (64->256 7x7 on 169 of
// 83 x 61 positions 22.2 -> 20.6 us, bfloat16 256->256 3x3 on a hundredth of 160 x 120 14.8 -> 13.5).
__device__ __forceinline__ int rank_selection(const GemmArgs &a, uint64_t *sW, int *sRank, int *sTot,
                                              uint64_t *scratch)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nw = a.sel_ranked, per = nw <= NT ? 1 : (nw <= 2 * NT ? 2 : 3);
    uint64_t w[kSelWordsPerThread];
    int sh = 0, i0 = per * tid;
    bool holds = true; // of the threads of a word, one holds it
    if (a.sel_dilate) {
        load_bitmap(a.sel_map, a.sel_bytes, a.sel_in_words, scratch);
        while (sh < 3 && (nw << (sh + 1)) <= NT && (1 << sh) < a.kh) ++sh;
        if (sh) i0 = tid >> sh;
        const int first = tid & ((1 << sh) - 1);
        holds = first == 0;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kSelWordsPerThread; ++j) w[j] = 0;
#pragma unroll 1
        for (int j = 0; j < per; ++j) { // one copy of the code
            const uint64_t d = i0 + j < nw ? dilated_word(a, reinterpret_cast<const unsigned *>(scratch), i0 + j, first, 1 << sh) : 0ull;
#pragma unroll
            for (int q = 0; q < kSelWordsPerThread; ++q) w[q] = q == j ? d : w[q];
        }
        if (sh) { // per == 1
            unsigned lo = (unsigned)w[0], hi = (unsigned)(w[0] >> 32);
            auto merge = [&](unsigned v, auto ctrl) { return v | (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, 0xf, 0xf, false); };
            lo = merge(lo, std::integral_constant<int, 0xB1>()); // lanes 1, 0, 3, 2 of each four
            hi = merge(hi, std::integral_constant<int, 0xB1>());
            if (sh > 1) {
                lo = merge(lo, std::integral_constant<int, 0x4E>()); // lanes 2, 3, 0, 1
                hi = merge(hi, std::integral_constant<int, 0x4E>());
            }
            if (sh > 2) {
                lo = merge(lo, std::integral_constant<int, 0x141>()); // of each eight in reverse
                hi = merge(hi, std::integral_constant<int, 0x141>());
            }
            w[0] = (uint64_t)hi << 32 | lo;
        }
    } else if (a.sel_bytes) { // through LDS: a thread's words of bytes lie far apart for loads
        load_bitmap(a.sel_map, 1, nw, scratch);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kSelWordsPerThread; ++j) w[j] = j < per && i0 + j < nw ? scratch[kSelGuard + i0 + j] : 0ull;
    } else {
#pragma unroll
        for (int j = 0; j < kSelWordsPerThread; ++j) w[j] = j < per && i0 + j < nw ? a.sel_map[i0 + j] : 0ull;
    }
    int c[kSelWordsPerThread], sum = 0;
#pragma unroll
    for (int j = 0; j < kSelWordsPerThread; ++j) {
        c[j] = holds ? __popcll(w[j]) : 0;
        sum += c[j];
    }
    const int incl = wave_inclusive_sum(sum);
    if (lane == 63) sTot[wave] = incl;
    __syncthreads();
    int before = 0, total = 0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) {
        const int t = sTot[i];
        if (i < wave) before += t;
        total += t;
    }
    int e = before + incl - sum;
#pragma unroll
    for (int j = 0; j < kSelWordsPerThread; ++j) {
        if (holds && j < per && i0 + j < nw) {
            sW[i0 + j] = w[j];
            sRank[i0 + j] = e;
        }
        e += c[j];
    }
    // the search reads ranks up to the next power of two
    for (int i = nw + tid; i < 2 * make_selection(a, sW, sRank).top; i += NT) sRank[i] = 0x7fffffff;
    __syncthreads();
    return total;
}

// This workgroup's share of a map derived by rank_selection, to a.upd_out for the kernels that follow; by the 64 lanes of a
// wave that the others do not wait for.
__device__ __forceinline__ void write_update_map(const GemmArgs &a, const uint64_t *sW)
{
    for (int i = (int)blockIdx.x + (int)gridDim.x * (int)(threadIdx.x & 63); i < a.sel_words; i += (int)gridDim.x * 64)
        a.upd_out[i] = a.Wo & 63 && a.dSelRow.d ? packed_word(a, sW, i) : sW[i];
}

// Channels ch .. ch + 3 of position g in the planar output.
__device__ __forceinline__ void store_planar(const GemmArgs &a, int g, int ch, const float4 &v)
{
    const int st = a.S > 1 ? fast_div(g, a.dNo) : 0;
    float *dst = a.planar + ((size_t)st * a.M + ch) * a.No + (g - st * a.No);
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (ch + e < a.M) dst[(size_t)e * a.No] = (&v.x)[e];
}
__device__ __forceinline__ float4 bf16_values(const uint2 &v)
{
    return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16),
                       __uint_as_float(v.y & 0xffff0000u));
}

// The position of rank r (0 <= r < number of selected positions) in a ranked selection map.
__device__ __forceinline__ int select_rank(const GemmArgs &a, const Selection &sel, int r)
{
    // the last word whose exclusive rank is <= r holds it: later words start at a higher rank,
    // and of the words sharing its rank it is the last (the others are empty)
    int w = 0;
    for (int step = sel.top; step; step >>= 1)
        if (sel.rank[w + step] <= r) w += step;
    const uint64_t word = sel.words[w];
    int k = r - sel.rank[w], pos = 0; // the k-th set bit of the word, counted from 0
    unsigned bits = (unsigned)word;
    const int low = __popc(bits);
    if (k >= low) {
        k -= low;
        bits = (unsigned)(word >> 32);
        pos = 32;
    }
#pragma unroll
    for (int sh = 16; sh; sh >>= 1) {
        const int c = __popc(bits & ((1u << sh) - 1u));
        const bool up = k >= c;
        k -= up ? c : 0;
        pos += up ? sh : 0;
        bits = up ? bits >> sh : bits;
    }
    if (!(a.Wo & 63 && a.dSelRow.d)) return w * 64 + pos;
    const int row = fast_div(w, a.dSelRow);
    return row * a.Wo + (w - row * a.dSelRow.d) * 64 + pos;
}

// The split of one launch's work over W workgroups; a pure function of its arguments.  32-bit
// arithmetic: W <= 1024 and the host refuses filter matrices of 2^20 slices or more, so
// rem * nk stays below 2^30.
struct Schedule {
    int tiles; // output tiles: pixel tiles x channel tiles (channel tile fastest)
    int whole; // rounds in which every workgroup takes one whole tile
    int rem;   // tiles left over, shared along K
    int wr;    // workgroups sharing the left-over tiles
    int iters; // rem * nk: K-slice iterations of the left-over tiles
    int q, r;  // iters = q * wr + r
};

// a / b for 0 <= a < 2^30, b >= 1 and quotients below 2^20: the estimate in float is off by one at most
// (the division that the compiler makes of an integer one takes about four times as long).
__device__ __forceinline__ int small_div(int a, int b)
{
    int q = (int)((float)a * __builtin_amdgcn_rcpf((float)b));
    const int r = a - q * b;
    if (r < 0) --q;
    if (r >= b) ++q;
    return __builtin_amdgcn_readfirstlane(q); // its arguments are the same for the whole workgroup
}

__device__ __forceinline__ Schedule make_schedule(int n, int bn, int mtiles, int nk, const FastDiv &dW)
{
    const int W = dW.d;
    Schedule s;
    s.tiles = ((n + bn - 1) / bn) * mtiles;
    s.whole = fast_div(s.tiles, dW);
    s.rem = s.tiles - s.whole * W;
    s.iters = s.rem * nk;
    // Cut every left-over tile into the same number of parts if that occupies at least 7/8 of
    // the workgroups (ranges then start on tile boundaries: one segment per workgroup); otherwise
    // deal the iterations out evenly over all workgroups.  Never make parts shorter than
    // kMinIters slices.
    const int max_parts = nk / kMinIters > 1 ? nk / kMinIters : 1;
    int wr = 1;
    if (s.rem > 0) {
        int p = small_div(W, s.rem);
        if (p > max_parts) p = max_parts;
        if (p < 1) p = 1;
        wr = s.rem * p;
        if (wr * 8 < W * 7 && s.rem * max_parts >= W) wr = W;
        if (wr > W) wr = W;
    }
    s.wr = wr;
    s.q = small_div(s.iters, wr);
    s.r = s.iters - s.q * wr;
    return s;
}

// First iteration of workgroup w's share: floor(iters * w / wr), and the workgroup owning an iteration.
__device__ __forceinline__ int share_begin(const Schedule &s, int w) { return s.q * w + small_div(s.r * w, s.wr); }

__device__ __forceinline__ int share_owner(const Schedule &s, int it)
{
    // estimate in float (off by one at most for these magnitudes), then settle exactly
    int w = (int)((float)it * (float)s.wr / (float)s.iters);
    if (w > s.wr - 1) w = s.wr - 1;
    if (w < 0) w = 0;
    while (w + 1 < s.wr && share_begin(s, w + 1) <= it) ++w;
    while (w > 0 && share_begin(s, w) > it) --w;
    return w;
}

__device__ __forceinline__ int lds_swizzle(int row) { return (row >> 1) & 7; }

// s_waitcnt vmcnt(N), everything else unconstrained (gfx9 encoding: vmcnt in bits 3:0 and 15:14).  What is
// waited for are loads and stores issued before it, on behalf of what comes behind it: the compiler must
// not move memory operations across in either direction, and the builtin alone does not say so.
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a six-bit counter");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
    asm volatile("" ::: "memory");
}

// The workgroup barrier as the direct-to-LDS producers execute it: the bare instruction.  The
// fences of __syncthreads() would make the wave wait for all of its loads in flight, which are
// exactly what has to stay in flight across the barrier; the one ordering the producers owe the
// consumers -- a slice has landed in LDS before the barrier that publishes it -- is the explicit
// wait_vmcnt in front of it, and the compiler must not move memory operations across either.
__device__ __forceinline__ void producer_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

typedef __attribute__((address_space(1))) const void *GlobalPtr;
typedef __attribute__((address_space(3))) void *LdsPtr;

// s_waitcnt lgkmcnt(0), everything else unconstrained; ordered like wait_vmcnt.
__device__ __forceinline__ void wait_lgkmcnt0()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);
    asm volatile("" ::: "memory");
}

// The workgroup barrier as the consumers execute it: their LDS reads are complete (the slice they read
// may be overwritten), stores to global memory need not be.
__device__ __forceinline__ void consumer_barrier()
{
    wait_lgkmcnt0();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The work of one workgroup: first whole tiles, then its share of the K ranges of the left-over ones.  A
// segment is a tile with the range of K slices to multiply.  Producers and consumers each walk it.
struct Segment {
    int tile, kc0, kc1, shared_j; // shared_j: index among the left-over tiles, or -1
};
struct Walk {
    Schedule sch;
    int W, nk, w;         // workgroups; slices per tile; this workgroup's number in the whole rounds
    int wsh;              // ... and among those that share the left-over tiles
    int it_begin, it_end; // its iterations of those
    int slices;           // K slices of all its segments
    int round, it;        // the cursor

    __device__ __forceinline__ bool next(const GemmArgs &a, Segment &s)
    {
        if (round < sch.whole) {
            s.tile = round * W + w;
            s.kc0 = 0;
            s.kc1 = nk;
            s.shared_j = -1;
            ++round;
            return true;
        }
        if (it >= it_end) return false;
        s.shared_j = fast_div(it, a.dNk);
        s.kc0 = it - s.shared_j * nk;
        const int left = it_end - it;
        s.kc1 = left < nk - s.kc0 ? s.kc0 + left : nk;
        s.tile = sch.whole * W + s.shared_j;
        it += s.kc1 - s.kc0;
        return true;
    }
};

// Producer waves: global_load_lds_dwordx4 moves 16 bytes per lane from global memory into LDS without
// passing through registers -- lane l of an instruction lands at the wave-uniform LDS base + 16 l, i.e.
// in slot l & 7 of row l >> 3 of eight consecutive rows -- so the producers only compute addresses.
// Wave pw covers rows 8 pw .. 8 pw + 7 of every pass of kRP rows; vf is the unit column this lane
// fetches (its slot with the row permutation undone).  The ring holds STAGES slices of all the
// workgroup's segments, one behind the other: slice t + STAGES - 1 is issued in iteration t into the
// slot that slice t - 1 occupied, and has to have landed by the barrier that ends iteration
// t + STAGES - 3 (the consumers read the first fragments of a slice one iteration early).  The loads of
// a wave complete in order, so "at most (STAGES - 3) slices' worth of instructions outstanding" means
// slice t + 2 is in LDS (the loads of a list entry or two in between make it wait for more, never for
// less).  The ring does not stop at a tile's end: while the consumers update the outputs of one tile or
// hand over its partial sums, the first slices of the next are on their way, found by the producers
// alone.  (With a prologue per tile, 2 us of list, addresses and a memory round trip in which
// nothing multiplies: bfloat16 64->128 3x3 at 320x240 31 us instead of 26, 128->128 44 instead of 39; float32
// 64->256 7x7 at 80x60 58 instead of 52, 128->128 3x3 at 320x240 143 instead of 128.)
// A producer's vector instructions are not hidden behind the MFMAs of the consumer waves on its SIMD, they
// add to them, so they are what is saved here.  Everything wave-uniform is computed on the scalar unit (the ring
// slot and the LDS destinations), loads take a 32-bit byte offset per lane from a scalar base, and per
// image-matrix row there remain, by what the layer allows (TAPS):
//   kTapUniform   The units per pixel are a multiple of the eight units of a slice, so a slice lies inside one filter
//                 tap and the tap is the same for all lanes (filters up to 32 wide, no higher than the map).  The base moves with the tap, a row keeps its lane's
//                 offset and one bit per tap column; a bit extraction makes the mask that selects between it and
//                 the zero unit: 14 vector instructions per slice of the 128-pixel tile instead of 50.
//   kTapPerLane   Any other, with maps up to 16000 x 16000: a lane per unit finds tap and offset of eight slices at
//                 once, to be fetched by a lane exchange; a row's test of both coordinates is one addition and one
//                 saturating subtraction of 16-bit pairs: 28 instead of 75, integer multiplications among them.
//   kTapGeneral   Maps of 4 GiB or longer sides: 64-bit addresses, tap and tests anew for every slice.
// bfloat16 64->64 3x3 at 640x480 53.5 -> 51.6 us, 512->512 3x3 at 80x60 38.9 -> 37.3, 16->64 7x7 at 640x360 55.1 -> 52.0;
// float32 64->256 7x7 at 320x180 420 -> 416, 96->100 5x5 at 101x37 27.0 -> 24.0.
template <int DT, int BM, int BN, int STAGES, int TAPS>
__device__ __forceinline__ void direct_producer(const GemmArgs &a, const int n, float *As, float *Bs, int *sU, const Selection &sel,
                                                Walk walk, int mtiles, int pw_)
{
    constexpr int PA = BN / kRP;                        // image-matrix rows per producer thread and slice
    constexpr int FB = BM / 16 * kFilterParts<DT>;      // filter fragments per slice
    constexpr int PB = (FB + kProdWaves - 1) / kProdWaves; // ... per wave (the last ones repeat others' when FB does not divide)
    constexpr int PS = PA + PB;                         // instructions per slice and wave
    constexpr int ASZ = BN * LDK, BSZ = FB * kFragBytes / 4;
    constexpr int NL = TileSmem<DT, BM, BN, STAGES>::lists;
    static_assert((STAGES - 3) * PS < 64, "outstanding loads must fit the counter");
    const int pw = __builtin_amdgcn_readfirstlane(pw_); // the wave's number among the producers, as a scalar
    const int lane = threadIdx.x & 63;
    const int r0 = pw * 8 + (lane >> 3);                // first row this lane stages
    // the hardware puts lane l's 16 bytes into slot l & 7 of row l >> 3 of the eight rows an
    // instruction covers, so the lane fetches the unit that belongs there
    const int vf = (lane & 7) ^ lds_swizzle(r0);
    const float *x = static_cast<const float *>(a.x);
    const unsigned lofs = lane * 16u;
    // General: a row's window origin, and its offset in words.  Otherwise: its offset in bytes, from bias words
    // before the map on (a uniform tap) or from the map's start, and the taps inside the image: the origin's row
    // and the columns' bits (uniform), or the origin's coordinates modulo 2^16.
    int iy0[PA], ix0[PA], base[PA];
    unsigned columns[PA], inside[PA]; // a uniform tap: bit i for column i, of the tap row in hand and in general
    int row_in_hand = -1;
    const int bias = a.pad * (a.W + 1) * a.pix_words;
    unsigned unit_tap = 0, unit_ofs = 0; // taps per lane: lane l's unit, of 64 units in eight slices
    int unit_slice = 0;
    const char *wtile = nullptr; // the channel tile's slices of the filter matrix, one behind the other as they lie in LDS
    Segment seg = {0, 0, 0, -1};
    int kc = 0, list = 0;
    // the next segment's positions: where this lane's rows start in the map, and the list for the consumers
    auto enter = [&]() {
        walk.next(a, seg);
        kc = seg.kc0;
        const int pt = small_div(seg.tile, mtiles), mt = seg.tile - pt * mtiles;
        wtile = static_cast<const char *>(DT == kF32Halves ? a.wt_halves : a.wt) + (size_t)mt * walk.nk * (FB * kFragBytes);
        // a lane per row of this wave: eight in each pass (one search of the ranks instead of one per pass)
        static_assert(PA <= 8, "the wave's rows fit its lanes");
        int *rows = sU + list * TileSmem<DT, BM, BN, STAGES>::list_words + pw * 8;
        // The biases travel like the slices that follow them (loads complete in order): loaded by the consumers, at
        // the end of a tile, they cost it a trip to memory of 0.3 to 0.8 us (bfloat16 128->128 3x3 at 320x240 37.5 ->
        // 36.4 us, 128->256 at 160x120, everything changed, 30.5 -> 29.3).
        if (pw * 64 < BM && lane < BM - pw * 64)
            __builtin_amdgcn_global_load_lds((GlobalPtr)(a.bias + mt * BM + pw * 64 + lane), (LdsPtr)(rows - pw * 8 + BN + pw * 64), 4, 0, 0);
        if (lane < 8 * PA) {
            const int row = (lane & 7) + kRP * (lane >> 3), u = pt * BN + pw * 8 + row;
            int g = -1;
            if (u < n) g = sel.words ? select_rank(a, sel, u) : (a.list ? a.list[u] : u);
            rows[row] = g;
        }
        __builtin_amdgcn_wave_barrier(); // written and read by this wave, in order
#pragma unroll
        for (int ps = 0; ps < PA; ++ps) {
            const int g = rows[(lane >> 3) + kRP * ps];
            if (g >= 0) {
                const int st = fast_div(g, a.dNo), q = g - st * a.No;
                const int qy = fast_div(q, a.dWo), qx = q - qy * a.Wo;
                iy0[ps] = qy * a.stride - a.pad;
                ix0[ps] = qx * a.stride - a.pad;
                base[ps] = ((st * a.H + iy0[ps]) * a.W + ix0[ps]) * a.pix_words;
            } else {
                iy0[ps] = -(1 << 28);
                ix0[ps] = -(1 << 28);
                base[ps] = 0;
            }
            if (TAPS == kTapUniform) {
                // columns lo .. hi - 1 of the window lie in the image, 0 <= lo < hi <= 32
                const int lo = ix0[ps] < 0 ? -ix0[ps] : 0, hi = a.W - ix0[ps] < a.kw ? a.W - ix0[ps] : a.kw;
                columns[ps] = g >= 0 ? (~0u >> ((32 - hi) & 31)) & (~0u << (lo & 31)) : 0u;
                base[ps] = g >= 0 ? (int)((unsigned)(base[ps] + bias + vf * 4) * 4u) : 0;
                row_in_hand = -1;
            }
            if (TAPS == kTapPerLane) {
                inside[ps] = g >= 0 ? (unsigned)iy0[ps] << 16 | ((unsigned)ix0[ps] & 0xffffu) : 0x80008000u;
                base[ps] = (int)((unsigned)base[ps] * 4u);
            }
        }
        list = list == NL - 1 ? 0 : list + 1;
        wait_lgkmcnt0(); // the list is in LDS before this wave's next barrier
    };
    // taps per lane: the units of slices kc .. kc + 7, one per lane
    auto unit_taps = [&]() {
        const int q = kc * KU + lane, tap = fast_div(q, a.dVin), cu = q - tap * a.dVin.d;
        const int tj = fast_div(tap, a.dKw), ti = tap - tj * a.kw;
        unit_tap = tj < a.kh ? (unsigned)tj << 16 | (unsigned)ti : 0x40004000u;
        unit_ofs = (unsigned)((tj * a.W + ti) * a.pix_words + cu * 4) * 4u;
        unit_slice = kc;
    };
    auto issue = [&](int slot) {
        if (kc == seg.kc1) {
            enter();
            if (TAPS == kTapPerLane) unit_taps();
        }
        float *A = As + slot * ASZ + pw * 8 * LDK, *B = Bs + slot * BSZ;
        if constexpr (TAPS == kTapUniform) {
            const int q = kc * KU, tap = fast_div(q, a.dVin), cu = q - tap * a.dVin.d;
            const int tj = fast_div(tap, a.dKw), ti = tap - tj * a.kw;
            const int off = (tj * a.W + ti) * a.pix_words + cu * 4 - bias;
            if (tj != row_in_hand) {
                row_in_hand = tj;
#pragma unroll
                for (int ps = 0; ps < PA; ++ps)
                    inside[ps] = tj < a.kh && (unsigned)(iy0[ps] + tj) < (unsigned)a.H ? columns[ps] : 0u;
            }
            const char *xt = reinterpret_cast<const char *>(x + off);
            const unsigned zero = (unsigned)(a.zero_word - off) * 4u;
#pragma unroll
            for (int ps = 0; ps < PA; ++ps) {
                const unsigned m = (unsigned)__builtin_amdgcn_sbfe((int)inside[ps], ti, 1);
                const unsigned ofs = ((unsigned)base[ps] & m) | (zero & ~m);
                __builtin_amdgcn_global_load_lds((GlobalPtr)(xt + ofs), (LdsPtr)(A + kRP * ps * LDK), 16, 0, 0);
            }
        } else if constexpr (TAPS == kTapPerLane) {
            if (kc - unit_slice >= 8 || kc < unit_slice) unit_taps();
            const int from = ((kc - unit_slice) * KU + vf) * 4;
            const unsigned tap = (unsigned)__builtin_amdgcn_ds_bpermute(from, (int)unit_tap);
            const unsigned ofs = (unsigned)__builtin_amdgcn_ds_bpermute(from, (int)unit_ofs);
            const unsigned zero = (unsigned)a.zero_word * 4u;
            const ushortx2 last = {(unsigned short)(a.W - 1), (unsigned short)(a.H - 1)};
#pragma unroll
            for (int ps = 0; ps < PA; ++ps) {
                const ushortx2 at = __builtin_bit_cast(ushortx2, inside[ps]) + __builtin_bit_cast(ushortx2, tap);
                const bool ok = __builtin_bit_cast(unsigned, __builtin_elementwise_sub_sat(at, last)) == 0u;
                const unsigned o = ok ? (unsigned)base[ps] + ofs : zero;
                __builtin_amdgcn_global_load_lds((GlobalPtr)(reinterpret_cast<const char *>(x) + o), (LdsPtr)(A + kRP * ps * LDK),
                                                 16, 0, 0);
            }
        } else {
            // tap of this lane's unit in slice kc: unit index -> (filter tap, channel unit) -> (j, i)
            const int q = kc * KU + vf;
            const int tap = fast_div(q, a.dVin), cu = q - tap * a.dVin.d;
            const int tj = fast_div(tap, a.dKw), ti = tap - tj * a.kw;
            const bool tv = tj < a.kh;
            const int off = (tj * a.W + ti) * a.pix_words + cu * 4;
#pragma unroll
            for (int ps = 0; ps < PA; ++ps) {
                const bool ok = tv && (unsigned)(iy0[ps] + tj) < (unsigned)a.H && (unsigned)(ix0[ps] + ti) < (unsigned)a.W;
                // outside the image (or no pixel in this row): the zero unit kept behind the map, so that the
                // load needs no predication
                const unsigned idx = ok ? (unsigned)(base[ps] + off) : (unsigned)a.zero_word;
                __builtin_amdgcn_global_load_lds((GlobalPtr)(x + idx), (LdsPtr)(A + kRP * ps * LDK), 16, 0, 0);
            }
        }
        const char *wslice = wtile + (size_t)kc * (FB * kFragBytes);
#pragma unroll
        for (int ps = 0; ps < PB; ++ps) {
            const int f = (pw + kProdWaves * ps) % FB;
            unsigned l = lofs;
            asm volatile("" : "+v"(l)); // its extension to 64 bits stays with the load, which takes a 32-bit lane offset as it is
            __builtin_amdgcn_global_load_lds((GlobalPtr)(wslice + f * kFragBytes + l), (LdsPtr)(B + f * (kFragBytes / 4)), 16, 0, 0);
        }
        ++kc;
    };
    // prologue: STAGES - 1 slices in flight, the first two landed
    const int slices = walk.slices;
#pragma unroll 1
    for (int d = 0; d < STAGES - 1; ++d)
        if (d < slices) issue(d);
    if (STAGES > 3 && STAGES - 2 < slices)
        wait_vmcnt<(STAGES - 3) * PS>();
    else
        wait_vmcnt<0>();
    producer_barrier();
    int slot = STAGES - 1; // ring slot of slice t + STAGES - 1
#pragma unroll 1
    for (int t = 0; t < slices; ++t) {
        const bool more = t + STAGES - 1 < slices;
        if (more) issue(slot);
        if (STAGES > 3 && more) // (three slices: nothing may stay in flight either way)
            wait_vmcnt<(STAGES - 3) * PS>();
        else
            wait_vmcnt<0>();
        slot = slot == STAGES - 1 ? 0 : slot + 1;
        producer_barrier();
    }
}

// A float32 as the sum of three bfloat16: hi = x rounded to 8 significant bits, mid = the rest rounded
// likewise, lo = what is left; 24 bits need no fourth.  Both differences are exact (the rest of a
// rounding to nearest has at most 16 significant bits, the next one at most 8), so hi + mid + lo is x
// itself from 2^-110 on.  Below, lo ends at the smallest bfloat16, 2^-133, and hi + mid + lo is x to half of
// that; sums in which this counts are formed again (GemmArgs::tiny_sum).  (Neither the dot product nor the
// matrix instruction flushes subnormal operands: measured.)
// Eight consecutive values of a lane become one 16-byte fragment of each part.
struct Parts {
    uintx4 hi, mid, lo;
};
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float minus_part(float x, unsigned pair, unsigned which)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, which), __builtin_bit_cast(bf16x2, pair), x, false);
}
__device__ __forceinline__ Parts split_fragment(const floatx4 x0, const floatx4 x1)
{
    // (-1, 0) and (0, -1) in scalar registers: as an inline constant the compiler writes the first as the
    // float -1, whose bits the instruction reads as (0, -1)
    unsigned first = 0x0000bf80u, second = 0xbf800000u;
    asm("" : "+s"(first));
    asm("" : "+s"(second));
    Parts p;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float a = i < 2 ? x0[2 * i] : x1[2 * i - 4], b = i < 2 ? x0[2 * i + 1] : x1[2 * i - 3];
        const unsigned h = bf16_pair(a, b);
        // a - hi(a): the two-element dot product with (-1, 0) and the float added takes a packed part as it is
        const float ra = minus_part(a, h, first), rb = minus_part(b, h, second);
        const unsigned m = bf16_pair(ra, rb);
        p.hi[i] = h;
        p.mid[i] = m;
        p.lo[i] = bf16_pair(minus_part(ra, m, first), minus_part(rb, m, second));
    }
    return p;
}

// float32 in halves: a value times a power of two as the sum of two float16 (11 bits each and the sign of the second: all
// but one of float32's 24), for the three products hi hi, hi lo and lo hi -- half of what the bfloat16 parts take.  The
// second is held times 2^kHalfLift, so that it does not end at the smallest float16, 2^-24, but at 2^-36 of where
// the first does: of a largest value between 2^13 and 2^15, values down to 2^-14 have all their bits, and what lies below is
// off by 2^-37 at most.  (Without the lift values below 2^-2 lost bits: a channel 2^-20 of its brightest neighbour,
// which its filter does not see, came out 4.4e-6 off, one of 2^-40 as zero.)  Three instructions per value: the scale, and
// v_fma_mix, which multiplies, subtracts and rounds at once, for each half.  The compiler does not know what the asm writes to;
// whoever multiplies the halves at once waits two cycles first.
static constexpr int kHalfLift = 12;
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
struct Halves {
    uintx4 hi, lo;
};
// scale: the power of two, times 2^kHalfLift
__device__ __forceinline__ Halves split_halves(const floatx4 x0, const floatx4 x1, const float scale)
{
    const float up = 1 << kHalfLift, down = 1.0f / (1 << kHalfLift);
    Halves p;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float a = (i < 2 ? x0[2 * i] : x1[2 * i - 4]) * scale, b = (i < 2 ? x0[2 * i + 1] : x1[2 * i - 3]) * scale;
        unsigned h, l;
        asm("v_fma_mixlo_f16 %0, %1, %3, 0\n\tv_fma_mixhi_f16 %0, %2, %3, 0" : "=&v"(h) : "v"(a), "v"(b), "s"(down));
        asm("v_fma_mixlo_f16 %0, -%4, %3, %1 op_sel_hi:[1,0,0]\n\tv_fma_mixhi_f16 %0, -%4, %3, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]"
            : "=&v"(l)
            : "v"(a), "v"(b), "s"(up), "v"(h));
        p.hi[i] = h;
        p.lo[i] = l;
    }
    return p;
}
// The largest magnitude of m and eight values (a NaN counts as nothing).
__device__ __forceinline__ float largest(float m, const floatx4 x0, const floatx4 x1)
{
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(x0[0]), "v"(x0[1]));
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(x0[2]), "v"(x0[3]));
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(x1[0]), "v"(x1[1]));
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(x1[2]), "v"(x1[3]));
    return m;
}
// A pixel's values are in lanes 16 apart: the largest of theirs.
__device__ __forceinline__ float pixel_largest(float m)
{
    m = fmaxf(m, __shfl_xor(m, 16));
    return fmaxf(m, __shfl_xor(m, 32));
}

// Where value (row, k) of a filter matrix in fragments lies, in bfloat16 values from its start; float32:
// its first part.
template <int DT>
__host__ __device__ inline size_t filter_fragment(int bm, int nk, int row, int k)
{
    constexpr int KS = DT == kBF16 ? 64 : 32; // k per slice
    const int mt = row / bm, ct = row % bm / 16, kc = k / KS, kk = k % KS;
    // float32: a lane's eight k are two units of four, 16 k apart; bfloat16: one unit of eight
    const int lk = DT == kF32 ? kk % 16 / 4 : kk / 8 % 4, e = DT == kF32 ? kk / 16 * 4 + kk % 4 : kk % 8;
    const int part = DT == kF32 ? 0 : kk / 32;
    return ((((size_t)mt * nk + kc) * (bm / 16) + ct) * kFilterParts<DT> + part) * (kFragBytes / 2) + (lk * 16 + row % 16) * 8 + e;
}

// float32 in halves: the exponent that a scale gives the largest value; the largest scale; the exponent of the largest value that
// it can have (half a unit of the last place of the first half is then 2^3, 2^15 when lifted); slices until leading sums are folded.
static constexpr int kHalfTop = 13, kHalfMostShift = 126 - kHalfLift, kHalfLimit = 15, kHalfChunk = 4;
// Sums that the halves' absolute errors may reach beyond 2^-kHalfBits of are formed again (gemm_halves_least).  That is if all of
// them have one sign; of either sign, they are a fiftieth of it or less.  Of pixels of one scale it is one sum in several millions: with 2^-18
// and 2^-20 64->256 7x7 on 320x180 takes 288 us, without any 290, with 2^-21 292.
static constexpr int kHalfBits = 20;

// Parts of a shared tile's sum that the finishing wave has under way, by its accumulators.
template <int ACC>
static constexpr int kPartsUnderWay = ACC <= 4 ? 4 : 2;

// Slices kc0 .. kc1 - 1 of TC channel tiles of a wave's sub-tile once more, multiplied by the float32 instruction
// straight from global memory (wt: their filter fragments of the first slice): for sums that the parts do not give.
// Where a value is infinite, not a number, or so near the largest float32 that its first part rounds to infinity, the
// products of parts are not those of the values (infinity less infinity, infinity times a part that is zero),
// and values below 2^-110 are not the sum of theirs, so the values themselves decide.  Filter values are put
// together from their parts; channels behind the last one of a packed pixel count as zero.  Bound by putting the
// filter values together, vector instructions that add to the MFMAs, so a value serves all pixels of the sub-tile,
// and by the loads, which are issued one group ahead; see the figures where it is called.
// FOLD: the products of two slices are added up before they join the sums, whose roundings are then as few as those of the
// halves that they replace.
template <int BM, int TP, int TC, bool FOLD>
__device__ __forceinline__ void plain_sums(const GemmArgs &a, int kc0, int kc1, const char *wt, const int *list, floatx4 (&sum)[TC][TP])
{
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane)); // nothing of this is computed ahead of the K loop and kept across it
    const int lrow = lane & 15, lk = lane >> 4;
    const float *x = static_cast<const float *>(a.x);
    int iy0[TP], ix0[TP], base[TP];
#pragma unroll
    for (int i = 0; i < TP; ++i) {
        const int g = list[i * 16 + lrow];
        const int st = fast_div(g < 0 ? 0 : g, a.dNo), q = g - st * a.No;
        const int qy = fast_div(g < 0 ? 0 : q, a.dWo), qx = q - qy * a.Wo;
        iy0[i] = g < 0 ? -(1 << 28) : qy * a.stride - a.pad;
        ix0[i] = g < 0 ? -(1 << 28) : qx * a.stride - a.pad;
        base[i] = g < 0 ? 0 : ((st * a.H + iy0[i]) * a.W + ix0[i]) * a.pix_words;
    }
#pragma unroll
    for (int j = 0; j < TC; ++j)
#pragma unroll
        for (int i = 0; i < TP; ++i) sum[j][i] = (floatx4){0.f, 0.f, 0.f, 0.f};
    floatx4 part[FOLD ? TC : 1][TP];
    auto &to = [&]() -> floatx4(&)[TC][TP] {
        if constexpr (FOLD)
            return part;
        else
            return sum;
    }();
    auto fold = [&] {
        if constexpr (FOLD) {
#pragma unroll
            for (int j = 0; j < TC; ++j)
#pragma unroll
                for (int i = 0; i < TP; ++i) {
                    sum[j][i] += part[j][i];
                    part[j][i] = (floatx4){0.f, 0.f, 0.f, 0.f};
                }
        }
    };
    if constexpr (FOLD) {
#pragma unroll
        for (int j = 0; j < TC; ++j)
#pragma unroll
            for (int i = 0; i < TP; ++i) part[j][i] = (floatx4){0.f, 0.f, 0.f, 0.f};
    }
    // G groups of four units are loaded together: a slice, as wide as loads come, or half of one where two tiles of
    // pixels would not leave two of channels their registers (with whole slices and one tile of channels 16->64
    // 7x7 on 640 x 900 positions that are all NaN 1190 us, now 1024; 64->32 5x5 on 320 x 240 197 and 167, with one NaN
    // 130 and 115).
    constexpr int G = TP == 1 ? 2 : 1;
    typedef typename std::conditional<G == 2, uint4, uint2>::type Part;
    struct Slice {
        floatx4 px[G][TP];
        Part w[TC][3];
        int c[G]; // channel of the units' first values
    };
    // units 4 G kc + lk and, of a whole slice, 4 more of the filter rows
    auto load = [&](Slice &v, int kc) {
#pragma unroll
        for (int h = 0; h < G; ++h) {
            const int unit = 4 * G * kc + 4 * h + lk, tap = fast_div(unit, a.dVin), cu = unit - tap * a.dVin.d;
            const int tj = fast_div(tap, a.dKw), ti = tap - tj * a.kw;
            const int off = (tj * a.W + ti) * a.pix_words + cu * 4;
            v.c[h] = cu * 4;
#pragma unroll
            for (int i = 0; i < TP; ++i) {
                const bool ok = tj < a.kh && (unsigned)(iy0[i] + tj) < (unsigned)a.H && (unsigned)(ix0[i] + ti) < (unsigned)a.W;
                v.px[h][i] = *reinterpret_cast<const floatx4_a4 *>(x + (ok ? (unsigned)(base[i] + off) : (unsigned)a.zero_word));
            }
        }
        const char *slice = wt + (size_t)((G == 2 ? kc : kc >> 1) - kc0) * (BM / 16 * 3 * kFragBytes) + lane * 16 + (G == 2 ? 0 : (kc & 1) * 8);
#pragma unroll
        for (int j = 0; j < TC; ++j)
#pragma unroll
            for (int p = 0; p < 3; ++p) v.w[j][p] = *reinterpret_cast<const Part *>(slice + (j * 3 + p) * kFragBytes);
    };
    // k = 16 G kc + 16 h + 4 lk + e in step (h, e)
    auto multiply = [&](const Slice &v) {
#pragma unroll
        for (int e = 0; e < 4 * G; ++e) {
            auto value = [&](int j, int p) { return bf16_value((unsigned short)((&v.w[j][p].x)[e >> 1] >> (e & 1 ? 16 : 0))); };
#pragma unroll
            for (int j = 0; j < TC; ++j)
#pragma unroll
                for (int i = 0; i < TP; ++i)
                    to[j][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                        __builtin_ldexpf(value(j, 0) + (value(j, 1) + value(j, 2)), -a.filter_exp),
                        v.c[e >> 2] + (e & 3) < a.pix_words ? v.px[e >> 2][i][e & 3] : 0.f, to[j][i], 0, 0, 0);
        }
    };
    Slice v0, v1;
    const int end = 2 / G * kc1;
    int kc = 2 / G * kc0;
    load(v0, kc);
#pragma unroll 1
    for (; kc + 1 < end; kc += 2) {
        load(v1, kc + 1);
        multiply(v0);
        load(v0, kc + 2 < end ? kc + 2 : kc);
        multiply(v1);
        fold();
    }
    if (kc < end) multiply(v0);
    fold();
}

// One such sum, of output position g and a row of the filter matrix (from its beginning, wt), by the whole wave: a unit per lane and
// step, in ascending order, the lanes' sums by halving.  (64->256 7x7 on 80x60 with one of them in the launch 44 us, without 42,
// by plain_sums 62.)
template <int BM>
__device__ __forceinline__ float plain_sum(const GemmArgs &a, int kc0, int kc1, const char *wt, int g, int row)
{
    const int lane = threadIdx.x & 63, nk = a.dNk.d;
    const float *x = static_cast<const float *>(a.x);
    const int st = fast_div(g < 0 ? 0 : g, a.dNo), q = g < 0 ? 0 : g - st * a.No, qy = fast_div(q, a.dWo), qx = q - qy * a.Wo;
    const int iy0 = g < 0 ? -(1 << 28) : qy * a.stride - a.pad, ix0 = qx * a.stride - a.pad;
    const int base = g < 0 ? 0 : ((st * a.H + iy0) * a.W + ix0) * a.pix_words;
    float sum = 0.f;
#pragma unroll 4
    for (int unit = kc0 * KU + lane; unit < kc1 * KU; unit += 64) {
        const int tap = fast_div(unit, a.dVin), cu = unit - tap * a.dVin.d;
        const int tj = fast_div(tap, a.dKw), ti = tap - tj * a.kw;
        const bool ok = tj < a.kh && (unsigned)(iy0 + tj) < (unsigned)a.H && (unsigned)(ix0 + ti) < (unsigned)a.W;
        const floatx4 px = *reinterpret_cast<const floatx4_a4 *>(
            x + (ok ? (unsigned)(base + (tj * a.W + ti) * a.pix_words + cu * 4) : (unsigned)a.zero_word));
        uint2 w[3];
#pragma unroll
        for (int p = 0; p < 3; ++p)
            w[p] = *reinterpret_cast<const uint2 *>(wt + filter_fragment<kF32>(BM, nk, row, unit * 4) * 2 + p * kFragBytes);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            auto value = [&](int p) { return bf16_value((unsigned short)((&w[p].x)[e >> 1] >> (e & 1 ? 16 : 0))); };
            sum = fmaf(__builtin_ldexpf(value(0) + (value(1) + value(2)), -a.filter_exp), cu * 4 + e < a.pix_words ? px[e] : 0.f, sum);
        }
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
    return sum;
}
// Sums of two channel tiles of a wave up to which they are formed one by one.
static constexpr int kFewSums = 16;

// BM x BN workgroup tile; the consumer waves are arranged WM (channels) x WN (pixels).
//
// LDS holds a ring of STAGES K slices.  In iteration kc the producers issue the loads of slice
// kc + STAGES - 1, while the consumers multiply slice kc and already read the first fragments of slice
// kc + 1, so the matrix pipeline keeps running across the one barrier per slice.  Pixel rows lie in LDS as
// they do in the map, their units permuted against bank conflicts; filter fragments lie as a wave
// reads them, 16 bytes per lane one lane behind the other, and arrive so from memory.
//
// Sub-tiles of the float32 shapes: a wave splits every pixel value it multiplies, so waves that share
// pixels repeat each other's work, and vector instructions are not hidden behind the MFMAs of either wave of
// a SIMD but add to them (a loop of this tile's 48 MFMAs per wave and slice takes 713 ns, with the fragment reads
// 806, with the splits of a 2 x 4 arrangement 994).  All channels of a 64-channel tile in one wave (1 x 8) took 136 us on
// 16->64 7x7 at 640x360 against 230 in a 2 x 4 arrangement; of a 128-channel tile, 64->256 7x7 at 320x180 418 us
// against 440, 256->256 3x3 at 160x120 127 against 131, although every wave then reads all filter fragments: LDS
// delivers 430 bytes per ns and compute unit, twice what that takes.
template <int DT, int BM, int BN, int WM, int WN, int STAGES>
__device__ __forceinline__ void gemm_gather_body(const GemmArgs &a, const int n, float *smem, const Selection sel)
{
    static_assert(WM * WN == kConsWaves, "one sub-tile per consumer wave");
    static_assert(STAGES >= 3, "ring depth");
    constexpr int TP = BN / WN / 16; // 16-pixel MFMA tiles per consumer wave
    constexpr int TC = BM / WM / 16; // 16-channel MFMA tiles per consumer wave
    constexpr int FP = kFilterParts<DT>;
    static_assert(BN % kRP == 0, "whole passes over the pixel rows");
    constexpr int ASZ = BN * LDK, BSZ = BM / 16 * FP * kFragBytes / 4;
    constexpr int SLAB = BM * BN; // floats of one partial-accumulator slab
    static_assert(TP >= 1 && TC >= 1, "tile too small");
    static_assert(BK == 32, "two 16-wide fragment groups per slice");
    static_assert(TC * TP * 4 * NCONS == SLAB, "a slab holds every consumer lane's accumulators");

    float *As = smem;                                     // [STAGES][BN][LDK]  gathered image-matrix slices
    float *Bs = smem + STAGES * ASZ;                      // [STAGES][BM/16][FP] filter fragments
    int *sU = reinterpret_cast<int *>(Bs + STAGES * BSZ); // [lists][BN + BM] pixels of a tile (-1: none), biases

    int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    const int mtiles = a.Mpad / BM;
    Walk walk;
    walk.nk = a.Kpad / (Unit<kStorage<DT>>::N * KU); // K slices
    walk.W = gridDim.x;
    walk.sch = make_schedule(n, BN, mtiles, walk.nk, a.dGrid);
    const Schedule &sch = walk.sch;
    if (sch.tiles == 0) return;
    // Workgroups are dealt round-robin over the 8 XCDs.  Number them so that each XCD works on a
    // contiguous range of tiles / iterations: neighbours share gathered pixels (channel tiles of
    // one pixel tile) or filter slices, and that sharing then happens inside one L2.
    walk.w = (int)(blockIdx.x & 7) * (walk.W >> 3) + (int)(blockIdx.x >> 3);
    const bool xcd_ranges = (sch.wr & 7) == 0;
    walk.wsh = xcd_ranges ? (int)(blockIdx.x & 7) * (sch.wr >> 3) + (int)(blockIdx.x >> 3)
                          : (int)blockIdx.x; // number inside the K-sharing group
    const bool sharing =
        sch.rem > 0 && (xcd_ranges ? (int)(blockIdx.x >> 3) < (sch.wr >> 3) : (int)blockIdx.x < sch.wr);
    walk.it_begin = sharing ? share_begin(sch, walk.wsh) : 0;
    walk.it_end = sharing ? share_begin(sch, walk.wsh + 1) : 0;
    walk.slices = sch.whole * walk.nk + walk.it_end - walk.it_begin;
    walk.round = 0;
    walk.it = walk.it_begin;
    if (walk.slices == 0) return;

    // Both roles execute the same number of barriers: one after the prologue, one per slice.
    if (wave >= kConsWaves) {
        if (a.taps_mode == kTapUniform)
            direct_producer<DT, BM, BN, STAGES, kTapUniform>(a, n, As, Bs, sU, sel, walk, mtiles, wave - kConsWaves);
        else if (a.taps_mode == kTapPerLane)
            direct_producer<DT, BM, BN, STAGES, kTapPerLane>(a, n, As, Bs, sU, sel, walk, mtiles, wave - kConsWaves);
        else
            direct_producer<DT, BM, BN, STAGES, kTapGeneral>(a, n, As, Bs, sU, sel, walk, mtiles, wave - kConsWaves);
        return;
    }

    const int wpx0 = (wave % WN) * (BN / WN);
    const int wch0 = (wave / WN) * (BM / WM);
    int lrow = lane & 15; // row of the 16-row operand tiles this lane feeds
    int lk = lane >> 4;   // k slot this lane feeds
    const int nk = walk.nk;
    int slot = 0; // ring slot of the slice in hand
    const int *list = sU;
    consumer_barrier();
    Segment seg;
    while (walk.next(a, seg)) {
        const int kc0 = seg.kc0, kc1 = seg.kc1, shared_j = seg.shared_j;
        const int pt = small_div(seg.tile, mtiles), mt = seg.tile - pt * mtiles;
        const bool partial = (kc1 - kc0) != nk;
        floatx4 acc[TC][TP];
        float unit[TP]; // float32 in halves: what a unit of scaled pixel values is, 0 for pixels of zeros
        {
#pragma unroll
            for (int j = 0; j < TC; ++j)
#pragma unroll
                for (int i = 0; i < TP; ++i) acc[j][i] = (floatx4){0.f, 0.f, 0.f, 0.f};
            // unit 4*kk + lk of this lane's pixel row, stored in slot (4*kk + lk) ^ swizzle
            const int u0 = (lk ^ lds_swizzle(lrow)) * 4;
            const float *A0 = As + (wpx0 + lrow) * LDK;
            const char *B0 = reinterpret_cast<const char *>(Bs) + wch0 / 16 * FP * kFragBytes + lane * 16;
            // Both operands of an MFMA hold eight k per lane, in the same order: D = (filter rows) x
            // (pixel columns), D[4*slot + r][lane%16] lands in this lane, i.e. four consecutive
            // channels of one pixel per accumulator.
            auto read_pixels = [&](int slot, int kk, int i) {
                return *reinterpret_cast<const floatx4 *>(A0 + slot * ASZ + (u0 ^ (kk * 16)) + i * 16 * LDK);
            };
            auto read_filter = [&](int slot, int j, int part) {
                return *reinterpret_cast<const uintx4 *>(B0 + slot * (BSZ * 4) + (j * FP + part) * kFragBytes);
            };
            auto mfma = [](const uintx4 w, const uintx4 x, const floatx4 c) {
                return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), c,
                                                               0, 0, 0);
            };
            // Operands stay alive to the end of a group of MFMAs.  Otherwise the register allocator puts the
            // result of an operand's last MFMA over that operand instead of over its own accumulator, and
            // the next MFMA of that accumulator has to wait for the result to be written: with two of sixteen
            // MFMAs like that 256->256 3x3 in bfloat16 took 42 us instead of 36, with a third of them float32
            // 256->256 3x3 131 instead of 122 and 16->64 7x7 at 640x360 133 instead of 127.
            auto keep = [](const uintx4 &v) { asm volatile("" ::"v"(v)); };
            // the wave feeding the matrix pipeline wins instruction-issue arbitration on its SIMD
            __builtin_amdgcn_s_setprio(3);
            if constexpr (DT == kBF16) {
                uintx4 af[2][TP], bf[2][TC];
                auto read_frags = [&](int set, int sl, int kk) {
#pragma unroll
                    for (int i = 0; i < TP; ++i) af[set][i] = __builtin_bit_cast(uintx4, read_pixels(sl, kk, i));
#pragma unroll
                    for (int j = 0; j < TC; ++j) bf[set][j] = read_filter(sl, j, kk);
                };
                auto multiply = [&](int set) {
#pragma unroll
                    for (int j = 0; j < TC; ++j)
#pragma unroll
                        for (int i = 0; i < TP; ++i) acc[j][i] = mfma(bf[set][j], af[set][i], acc[j][i]);
#pragma unroll
                    for (int j = 0; j < TC; ++j) keep(bf[set][j]);
#pragma unroll
                    for (int i = 0; i < TP; ++i) keep(af[set][i]);
                };
                read_frags(0, slot, 0);
                for (int kc = kc0; kc < kc1; ++kc) {
                    const int nslot = slot == STAGES - 1 ? 0 : slot + 1;
                    // The scheduling barriers pin the order "issue the LDS reads of the next fragment
                    // group, then the MFMAs of the current one", so that LDS latency and bandwidth
                    // are spent while the matrix pipeline is busy.
                    read_frags(1, slot, 1);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(0);
                    __builtin_amdgcn_sched_barrier(0);
                    // Also in the last iteration, where the slot holds nothing of use: under a condition
                    // the compiler, which counts outstanding LDS reads per path, would make the MFMAs
                    // below wait for these reads too.
                    read_frags(0, nslot, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(1);
                    __builtin_amdgcn_sched_barrier(0);
                    slot = nslot;
                    consumer_barrier();
                }
            } else if constexpr (DT == kF32Halves) {
                auto mfma_half = [](const uintx4 w, const uintx4 x, const floatx4 c) {
                    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(halfx8, w), __builtin_bit_cast(halfx8, x), c,
                                                                  0, 0, 0);
                };
                // float32 in halves: three of the four products, hi hi in the leading sums, the others in sums of their own.  The
                // matrix unit cuts addends off at 2^-24 of the largest (an error of 4.7e-8 of the sum per instruction, measured,
                // on float16 products of 22 bits; 3.4e-8 on bfloat16's 16), so the leading sums go to others every kHalfChunk
                // slices and begin again: their roundings are relative to four slices' sum, not to all.
                floatx4 lead[TC][TP], cor[TC][TP];
#pragma unroll
                for (int j = 0; j < TC; ++j)
#pragma unroll
                    for (int i = 0; i < TP; ++i) lead[j][i] = cor[j][i] = (floatx4){0.f, 0.f, 0.f, 0.f};
                Halves x0[TP], x1[TP]; // pixel fragments of two slices in turn
                uintx4 w[2][2];
                auto read_tile = [&](int set, int sl, int j) {
                    w[set][0] = read_filter(sl, j, 0);
                    w[set][1] = read_filter(sl, j, 1);
                };
                // The power of two that a pixel's values are multiplied with, from the largest in its first slice: that becomes
                // 2^kHalfTop to twice as much.  A slice with a value beyond 2^kHalfLimit has the sums so far folded and another
                // power from then on.  A power for each pixel: how bright its neighbours are is nothing to it.
                float scale[TP], most[TP]; // a power of two, with kHalfLift; the largest of this lane's values
                auto set_scale = [&] {
#pragma unroll
                    for (int i = 0; i < TP; ++i) {
                        const int shift = kHalfTop + 127 - (int)(__float_as_uint(pixel_largest(most[i])) >> 23);
                        scale[i] = __uint_as_float((unsigned)(127 + kHalfLift + (shift < kHalfMostShift ? shift : kHalfMostShift)) << 23);
                    }
                };
                auto unscale = [&](int i, int lift) { // one through the power of two, and through 2^lift
                    return __uint_as_float(((unsigned)(254 + kHalfLift - lift) << 23) - __float_as_uint(scale[i]));
                };
                auto fold = [&](floatx4(&from)[TC][TP], int lift) {
#pragma unroll
                    for (int j = 0; j < TC; ++j)
#pragma unroll
                        for (int i = 0; i < TP; ++i) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[j][i][e] = fmaf(from[j][i][e], unscale(i, lift), acc[j][i][e]);
                            from[j][i] = (floatx4){0.f, 0.f, 0.f, 0.f};
                        }
                };
                read_tile(0, slot, 0);
                {
                    floatx4 raw[TP][2];
#pragma unroll
                    for (int i = 0; i < TP; ++i) {
                        raw[i][0] = read_pixels(slot, 0, i);
                        raw[i][1] = read_pixels(slot, 1, i);
                        most[i] = largest(0.f, raw[i][0], raw[i][1]);
                    }
                    set_scale();
#pragma unroll
                    for (int i = 0; i < TP; ++i) x0[i] = split_halves(raw[i][0], raw[i][1], scale[i]);
                    asm volatile("s_nop 3");
                }
                auto step = [&](Halves(&x)[TP], Halves(&nx)[TP], const bool more) {
                    const int nslot = slot == STAGES - 1 ? 0 : slot + 1;
                    floatx4 raw[TP][2];
#pragma unroll
                    for (int j = 0; j < TC; ++j) {
                        if (j + 1 < TC)
                            read_tile((j + 1) & 1, slot, j + 1);
                        else
                            read_tile((j + 1) & 1, nslot, 0);
                        // pixel fragment i of the next slice is read a channel tile before it is split
#pragma unroll
                        for (int i = 0; i < TP; ++i) {
                            if (j == (i < TC - 1 ? i : (TC > 1 ? TC - 2 : 0))) {
                                raw[i][0] = read_pixels(nslot, 0, i);
                                raw[i][1] = read_pixels(nslot, 1, i);
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        const uintx4 *wj = w[j & 1];
#pragma unroll
                        for (int i = 0; i < TP; ++i) cor[j][i] = mfma_half(wj[1], x[i].hi, cor[j][i]);
#pragma unroll
                        for (int i = 0; i < TP; ++i) lead[j][i] = mfma_half(wj[0], x[i].hi, lead[j][i]);
#pragma unroll
                        for (int i = 0; i < TP; ++i) cor[j][i] = mfma_half(wj[0], x[i].lo, cor[j][i]);
                        keep(wj[0]);
                        keep(wj[1]);
#pragma unroll
                        for (int i = 0; i < TP; ++i) {
                            if (j < TC - 1) continue;
                            keep(x[i].hi);
                            keep(x[i].lo);
                        }
#pragma unroll
                        for (int i = 0; i < TP; ++i)
                            if (j == (i + 1 < TC ? i + 1 : TC - 1)) {
                                if (more) most[i] = largest(most[i], raw[i][0], raw[i][1]); // else the slot holds nothing of this tile
                                nx[i] = split_halves(raw[i][0], raw[i][1], scale[i]);
                            }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if constexpr (TC & 1) {
                        w[0][0] = w[1][0];
                        w[0][1] = w[1][1];
                    }
                    slot = nslot;
                    consumer_barrier();
                };
                int kc = kc0;
                for (;;) {
                    bool over = false;
#pragma unroll
                    for (int s = 0; s < kHalfChunk; ++s) {
                        if (s & 1)
                            step(x1, x0, kc + 1 < kc1);
                        else
                            step(x0, x1, kc + 1 < kc1);
                        bool beyond = false;
#pragma unroll
                        for (int i = 0; i < TP; ++i) beyond |= most[i] * scale[i] > (float)(1 << (kHalfLimit + kHalfLift));
                        over = __any(beyond);
                        if (++kc == kc1 || over) break;
                    }
                    fold(lead, 0);
                    if (kc == kc1) break;
                    if (__builtin_expect(over, 0)) { // the next slice needs another power of two
                        fold(cor, kHalfLift);
                        set_scale();
#pragma unroll
                        for (int i = 0; i < TP; ++i) x0[i] = split_halves(read_pixels(slot, 0, i), read_pixels(slot, 1, i), scale[i]);
                        asm volatile("s_nop 3");
                    }
                }
                fold(cor, kHalfLift);
#pragma unroll
                for (int j = 0; j < TC; ++j)
#pragma unroll
                    for (int i = 0; i < TP; ++i)
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[j][i][e] = __builtin_ldexpf(acc[j][i][e], -a.halves_exp);
#pragma unroll
                for (int i = 0; i < TP; ++i) unit[i] = pixel_largest(most[i]) > 0.f ? unscale(i, 0) : 0.f;
                // found anew rather than kept across the K loop, which needs all registers
                unsigned thread = threadIdx.x;
                asm volatile("" : "+v"(thread));
                lane = (int)thread & 63;
                lrow = lane & 15;
                lk = lane >> 4;
            } else {
                // float32: six of the nine products of parts, everything down to 2^-24 of the leading one.
                // Leading products and corrections have accumulators of their own: the corrections are
                // then summed at their own magnitude and do not round the leading sum again.
                floatx4 cor[TC][TP];
#pragma unroll
                for (int j = 0; j < TC; ++j)
#pragma unroll
                    for (int i = 0; i < TP; ++i) cor[j][i] = (floatx4){0.f, 0.f, 0.f, 0.f};
                Parts x0[TP], x1[TP]; // pixel fragments of two slices in turn
                uintx4 w[2][3];
#pragma unroll
                for (int p = 0; p < 3; ++p) w[0][p] = read_filter(slot, 0, p);
#pragma unroll
                for (int i = 0; i < TP; ++i) x0[i] = split_fragment(read_pixels(slot, 0, i), read_pixels(slot, 1, i));
                // One slice: while channel tile j is multiplied, the filter fragments of the next tile are
                // on their way from LDS and the next slice's pixels are read and split.
                auto step = [&](Parts(&x)[TP], Parts(&nx)[TP]) {
                    const int nslot = slot == STAGES - 1 ? 0 : slot + 1;
                    floatx4 raw[TP][2];
#pragma unroll
                    for (int j = 0; j < TC; ++j) {
#pragma unroll
                        for (int p = 0; p < 3; ++p)
                            w[(j + 1) & 1][p] = j + 1 < TC ? read_filter(slot, j + 1, p) : read_filter(nslot, 0, p);
                        // pixel fragment i of the next slice is read a channel tile before it is split
#pragma unroll
                        for (int i = 0; i < TP; ++i) {
                            if (j == (i < TC - 1 ? i : (TC > 1 ? TC - 2 : 0))) {
                                raw[i][0] = read_pixels(nslot, 0, i);
                                raw[i][1] = read_pixels(nslot, 1, i);
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        const uintx4 *wj = w[j & 1];
#pragma unroll
                        for (int i = 0; i < TP; ++i) acc[j][i] = mfma(wj[0], x[i].hi, acc[j][i]);
#pragma unroll
                        for (int i = 0; i < TP; ++i) cor[j][i] = mfma(wj[2], x[i].hi, cor[j][i]);
#pragma unroll
                        for (int i = 0; i < TP; ++i) cor[j][i] = mfma(wj[1], x[i].mid, cor[j][i]);
#pragma unroll
                        for (int i = 0; i < TP; ++i) cor[j][i] = mfma(wj[0], x[i].lo, cor[j][i]);
#pragma unroll
                        for (int i = 0; i < TP; ++i) cor[j][i] = mfma(wj[1], x[i].hi, cor[j][i]);
#pragma unroll
                        for (int i = 0; i < TP; ++i) cor[j][i] = mfma(wj[0], x[i].mid, cor[j][i]);
                        keep(wj[0]);
                        keep(wj[1]);
                        keep(wj[2]);
#pragma unroll
                        for (int i = 0; i < TP; ++i) {
                            if (j < TC - 1) continue;
                            keep(x[i].hi);
                            keep(x[i].mid);
                            keep(x[i].lo);
                        }
                        // ... in the shadow of that tile's MFMAs
#pragma unroll
                        for (int i = 0; i < TP; ++i)
                            if (j == (i + 1 < TC ? i + 1 : TC - 1)) nx[i] = split_fragment(raw[i][0], raw[i][1]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if constexpr (TC & 1) {
#pragma unroll
                        for (int p = 0; p < 3; ++p) w[0][p] = w[1][p];
                    }
                    slot = nslot;
                    consumer_barrier();
                };
                int kc = kc0;
                for (; kc + 1 < kc1; kc += 2) {
                    step(x0, x1);
                    step(x1, x0);
                }
                if (kc < kc1) step(x0, x1);
#pragma unroll
                for (int j = 0; j < TC; ++j)
#pragma unroll
                    for (int i = 0; i < TP; ++i)
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[j][i][e] = __builtin_ldexpf(acc[j][i][e] + cor[j][i][e], -a.filter_exp);
            }
            __builtin_amdgcn_s_setprio(0);
        }

        if constexpr (DT != kBF16) {
            // Sums that are not finite, and such small ones that parts below the smallest bfloat16 count
            // (GemmArgs::tiny_sum), are formed again from the values themselves, by each wave for its own K
            // range.  (x * 0 is zero for every finite x.)  A tile with such a sum takes two to five times as long:
            // 64->256 7x7 on 160 x 90 positions 115 us, with one NaN in the map 374, with nothing else in it 524; on
            // 20 x 20 21, 37 and 38; 16->64 7x7 on 640 x 900 289, 340 and 1024 (one lane per sum, product by product:
            // 11 150 us for that one NaN, 25 700 for the full map).  The 128-channel tile in a 2 x 4 arrangement of waves
            // took 428 us for the map of nothing else, as a filter value put together served two tiles of pixels, and 120
            // and 425 for the others.
            // In halves these are, of pixels that are not all zero, the sums below GemmArgs::halves_least or, looked at more
            // closely, what is stored behind the halves for their rows.
            float z = 0.f;
            unsigned least = ~0u;
            auto size = [](float v) { return (__float_as_uint(v) << 1) - 1u; }; // grows with |v|; largest for zero
            bool again = false;
#pragma unroll
            for (int i = 0; i < TP; ++i) {
                float lowest = __builtin_inff();
#pragma unroll
                for (int j = 0; j < TC; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        z = fmaf(acc[j][i][e], 0.f, z);
                        if constexpr (DT == kF32)
                            least = min(least, size(acc[j][i][e]));
                        else
                            lowest = fminf(lowest, fabsf(acc[j][i][e]));
                    }
                if constexpr (DT == kF32Halves) again |= lowest < __builtin_ldexpf(a.halves_least * unit[i], -a.halves_exp);
            }
            if constexpr (DT == kF32) again = least < a.tiny_sum;
            if (__builtin_expect(__any(z != 0.f || again), 0)) { // NaN compares unequal
                const char *wt = static_cast<const char *>(a.wt) +
                                 (((size_t)mt * nk + kc0) * (BM / 16) + wch0 / 16) * (3 * kFragBytes);
                // two channel tiles at a time: more would not leave their operands registers
                constexpr int CJ = TC % 2 == 0 ? 2 : 1;
                static_assert(TC % CJ == 0, "whole steps");
#pragma unroll 1
                for (int j0 = 0; j0 < TC; j0 += CJ) {
                    float4 row_least[CJ]; // of this lane's rows
                    // whether a sum does not stand
                    auto fails = [&](float v, int j, int i, int e) {
                        if constexpr (DT == kF32) return !(fabsf(v) < __builtin_inff()) || size(v) < a.tiny_sum;
                        const float t = __builtin_ldexpf((&row_least[j % CJ].x)[e] * unit[i], -a.halves_exp);
                        return !(fabsf(v) < __builtin_inff()) || fabsf(v) < t;
                    };
                    if constexpr (DT == kF32Halves) { // most often it is one sum of the tile
                        const float *row = static_cast<const float *>(a.wt_halves) + (size_t)a.Mpad * a.Kpad + mt * BM + wch0 + j0 * 16 + lk * 4;
#pragma unroll
                        for (int j = 0; j < CJ; ++j) row_least[j] = *reinterpret_cast<const float4 *>(row + j * 16);
                        static_assert(TP == 1, "sums are numbered by channel tile and channel");
                        unsigned failed = 0;
#pragma unroll
                        for (int j = 0; j < TC; ++j) {
                            if (j / CJ != j0 / CJ) continue;
#pragma unroll
                            for (int e = 0; e < 4; ++e) failed |= fails(acc[j][0][e], j, 0, e) ? 1u << (j % CJ * 4 + e) : 0u;
                        }
                        int count = 0;
#pragma unroll
                        for (int bit = 0; bit < CJ * 4; ++bit) count += __builtin_popcountll(__ballot(failed >> bit & 1));
                        if (count <= kFewSums) {
                            for (uint64_t lanes; (lanes = __ballot(failed != 0)) != 0;) {
                                const int from = __builtin_ctzll(lanes);
                                const int bit = __builtin_ctz(__builtin_amdgcn_readlane((int)failed, from));
                                const int g = __builtin_amdgcn_readfirstlane(list[wpx0 + (from & 15)]);
                                const float v = plain_sum<BM>(a, kc0, kc1, static_cast<const char *>(a.wt), g,
                                                              mt * BM + wch0 + (j0 + (bit >> 2)) * 16 + (from >> 4) * 4 + (bit & 3));
#pragma unroll
                                for (int j = 0; j < TC; ++j) {
                                    if (j / CJ != j0 / CJ) continue;
#pragma unroll
                                    for (int e = 0; e < 4; ++e)
                                        if (bit == j % CJ * 4 + e && lane == from) acc[j][0][e] = v;
                                }
                                if (lane == from) failed &= failed - 1;
                            }
                            continue;
                        }
                    }
                    floatx4 sum[CJ][TP];
                    plain_sums<BM, TP, CJ, DT == kF32Halves>(a, kc0, kc1, wt + j0 * (3 * kFragBytes), list + wpx0, sum);
#pragma unroll
                    for (int j = 0; j < TC; ++j) {
                        if (j / CJ != j0 / CJ) continue;
#pragma unroll
                        for (int i = 0; i < TP; ++i)
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                float v = acc[j][i][e];
                                asm("" : "+v"(v)); // compared anew: the results from above would all be kept in registers
                                if (fails(v, j, i, e)) acc[j][i][e] = sum[j % CJ][i][e];
                            }
                    }
                }
            }
        }

        // ---- a shared tile: store this K range's accumulators, take a ticket; the wave holding the last
        //      ticket of its sub-tile adds up all ranges (ascending K) and does the output update.  A
        //      sub-tile belongs to the same wave of every workgroup, so waves need no barrier for this:
        //      a wave's slab stores are complete (vmcnt(0)) before it takes its ticket.
        bool finish = true;
        if (partial) {
            const int t0 = shared_j * nk;
            const int w_first = share_owner(sch, t0);
            const int w_last = share_owner(sch, t0 + nk - 1);
            // slab 2*wsh + (0: first tile this workgroup touches, 1: a later one), register layout:
            // one float4 per lane and accumulator, consecutive lanes consecutive addresses
            const int first_j = fast_div(walk.it_begin, a.dNk);
            const __amdgpu_buffer_rsrc_t slab = slab_resource(
                a.partial + (size_t)(2 * walk.wsh + (shared_j == first_j ? 0 : 1)) * SLAB, SLAB * 4);
            const int ofs = wave * (TC * TP * kFragBytes) + lane * 16;
#pragma unroll
            for (int j = 0; j < TC; ++j)
#pragma unroll
                for (int i = 0; i < TP; ++i)
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uintx4, acc[j][i]), slab,
                                                           ofs + (j * TP + i) * kFragBytes, 0, kDeviceCoherent);
            // all of this wave's slab stores have reached the device-coherent level
            wait_vmcnt<0>();
            int *ticket = a.tickets + shared_j * kConsWaves + wave;
            int drawn = 0;
            if (lane == 0) drawn = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            drawn = __builtin_amdgcn_readfirstlane(drawn);
            asm volatile("" ::: "memory"); // the other waves' parts are read behind the ticket, not before it
            finish = drawn == w_last - w_first;
            if (finish) {
                if (lane == 0) *ticket = 0; // ready for the next launch
                // Sum the parts in ascending K order, whichever wave finishes (its own part is read back like the
                // others, which keeps the accumulators in one register set).  A part is a round trip to the level
                // that all XCDs share, half a microsecond, so several are under way: four for waves of up to four
                // accumulators (64->256 7x7 on 169 of 83 x 61 positions, 12 parts, 25.1 us with one, now 22.2; 64->256 on
                // 144 of 80 x 60 24.2 -> 21.8; bfloat16 512->512 3x3 on 64 17.8 -> 16.8), two for the big tiles (three:
                // 64->256 7x7 on 4 800 positions 64 -> 66 us).
#pragma unroll
                for (int j = 0; j < TC; ++j)
#pragma unroll
                    for (int i = 0; i < TP; ++i) acc[j][i] = (floatx4){0.f, 0.f, 0.f, 0.f};
                constexpr int D = kPartsUnderWay<TC * TP>;
                // the tile is the first one of every workgroup that shares it but the one that began before it
                const int first_slab = 2 * w_first + (share_begin(sch, w_first) < t0 ? 1 : 0);
#pragma unroll 1
                for (int ww = w_first; ww <= w_last; ww += D) {
                    floatx4 part[D][TC][TP];
#pragma unroll
                    for (int d = 0; d < D; ++d) {
                        // behind the last part: a buffer of no bytes, which reads as zeros
                        const int slab_index = ww + d == w_first ? first_slab : (ww + d > w_last ? 0 : 2 * (ww + d));
                        const __amdgpu_buffer_rsrc_t part_slab =
                            slab_resource(a.partial + (size_t)slab_index * SLAB, ww + d > w_last ? 0 : SLAB * 4);
#pragma unroll
                        for (int j = 0; j < TC; ++j)
#pragma unroll
                            for (int i = 0; i < TP; ++i)
                                part[d][j][i] = __builtin_bit_cast(
                                    floatx4, __builtin_amdgcn_raw_buffer_load_b128(part_slab, ofs + (j * TP + i) * kFragBytes, 0,
                                                                                   kDeviceCoherent));
                    }
#pragma unroll
                    for (int d = 0; d < D; ++d) {
#pragma unroll
                        for (int j = 0; j < TC; ++j)
#pragma unroll
                            for (int i = 0; i < TP; ++i) acc[j][i] += part[d][j][i];
                    }
                }
            }
        }

        // ---- output update: bias, activation, scatter to the stored map; optionally the change
        //      detection of the layer this map feeds (new value against the one it replaces)
        if (finish) {
            const bool detect = a.next_flags != nullptr && !a.next_force;
            bool changed[TP];
#pragma unroll
            for (int i = 0; i < TP; ++i) changed[i] = false;
            float4 bias[TC];
#pragma unroll
            for (int j = 0; j < TC; ++j) bias[j] = *reinterpret_cast<const float4 *>(list + BN + wch0 + j * 16 + lk * 4);
            // The values about to be replaced are loaded kEpiChunk accumulators at a time before the
            // stores of those accumulators (the compiler cannot move a load across a store to the
            // same map, and one round trip to memory per accumulator would line up at the very end
            // of the kernel).  Accumulator q covers channels of block q / TP at the positions of block q % TP.
            // (Eight accumulators in halves: two at a time, as four spill.)
            constexpr int CH = DT == kF32Halves && TC > 4 ? 2 : TC * TP < kEpiChunk ? TC * TP : kEpiChunk;
            static_assert((TC * TP) % CH == 0, "whole chunks");
#pragma unroll
            for (int q0 = 0; q0 < TC * TP; q0 += CH) {
                uintx4 replaced[CH];
                if (detect) {
#pragma unroll
                    for (int qq = 0; qq < CH; ++qq) {
                        const int j = (q0 + qq) / TP, i = (q0 + qq) % TP;
                        const int ch = mt * BM + wch0 + j * 16 + lk * 4;
                        const int g = list[wpx0 + i * 16 + lrow];
                        replaced[qq] = (uintx4){0u, 0u, 0u, 0u};
                        if (g >= 0 && ch < a.Ms) {
                            if constexpr (DT == kBF16) {
                                const uint2 v = *reinterpret_cast<const uint2 *>(static_cast<const unsigned short *>(a.out) +
                                                                                 (size_t)g * a.Ms + ch);
                                replaced[qq][0] = v.x;
                                replaced[qq][1] = v.y;
                            } else {
                                replaced[qq] = *reinterpret_cast<const uintx4 *>(static_cast<const float *>(a.out) +
                                                                                 (size_t)g * a.Ms + ch);
                            }
                        }
                    }
                }
#pragma unroll
                for (int qq = 0; qq < CH; ++qq) {
                    const int j = (q0 + qq) / TP, i = (q0 + qq) % TP;
                    const int ch = mt * BM + wch0 + j * 16 + lk * 4;
                    const float4 bv = bias[j];
                    const int g = list[wpx0 + i * 16 + lrow];
                    if (g >= 0 && ch < a.Ms) {
                        float4 o;
                        o.x = acc[j][i][0] + bv.x;
                        o.y = acc[j][i][1] + bv.y;
                        o.z = acc[j][i][2] + bv.z;
                        o.w = acc[j][i][3] + bv.w;
                        if (a.relu) {
                            o.x = fmaxf(o.x, 0.f);
                            o.y = fmaxf(o.y, 0.f);
                            o.z = fmaxf(o.z, 0.f);
                            o.w = fmaxf(o.w, 0.f);
                        }
                        if constexpr (DT == kBF16) {
                            // four consecutive bfloat16 channels: one 8-byte word
                            uint2 *dst = reinterpret_cast<uint2 *>(static_cast<unsigned short *>(a.out) +
                                                                   (size_t)g * a.Ms + ch);
                            uint2 nv;
                            nv.x = bf16_pair(o.x, o.y);
                            nv.y = bf16_pair(o.z, o.w);
                            if (detect) {
                                const uint2 ov = make_uint2(replaced[qq][0], replaced[qq][1]);
                                changed[i] |= fabsf(bf16_value(nv.x & 0xffff) - bf16_value(ov.x & 0xffff)) > a.next_tau ||
                                              fabsf(bf16_value(nv.x >> 16) - bf16_value(ov.x >> 16)) > a.next_tau ||
                                              fabsf(bf16_value(nv.y & 0xffff) - bf16_value(ov.y & 0xffff)) > a.next_tau ||
                                              fabsf(bf16_value(nv.y >> 16) - bf16_value(ov.y >> 16)) > a.next_tau;
                            }
                            *dst = nv;
                            const float4 r = bf16_values(nv);
                            acc[j][i] = (floatx4){r.x, r.y, r.z, r.w};
                        } else {
                            float4 *dst = reinterpret_cast<float4 *>(static_cast<float *>(a.out) + (size_t)g * a.Ms + ch);
                            if (detect) {
                                const float4 ov = make_float4(__uint_as_float(replaced[qq][0]), __uint_as_float(replaced[qq][1]),
                                                              __uint_as_float(replaced[qq][2]), __uint_as_float(replaced[qq][3]));
                                changed[i] |= fabsf(o.x - ov.x) > a.next_tau || fabsf(o.y - ov.y) > a.next_tau ||
                                              fabsf(o.z - ov.z) > a.next_tau || fabsf(o.w - ov.w) > a.next_tau;
                            }
                            *dst = o;
                            acc[j][i] = (floatx4){o.x, o.y, o.z, o.w};
                        }
                    }
                }
            }
            if (a.planar) {
#pragma unroll
                for (int i = 0; i < TP; ++i) {
                    const int g = list[wpx0 + i * 16 + lrow];
                    if (g < 0) continue;
#pragma unroll
                    for (int j = 0; j < TC; ++j)
                        store_planar(a, g, mt * BM + wch0 + j * 16 + lk * 4, make_float4(acc[j][i][0], acc[j][i][1], acc[j][i][2], acc[j][i][3]));
                }
            }
            if (a.next_flags) {
#pragma unroll
                for (int i = 0; i < TP; ++i) {
                    const int g = list[wpx0 + i * 16 + lrow];
                    int f = a.next_force ? 1 : (int)changed[i];
                    // the other channels of this pixel sit in the lanes 16, 32 and 48 further on
                    f |= __shfl_xor(f, 16);
                    f |= __shfl_xor(f, 32);
                    if (lk == 0 && f && g >= 0) a.next_flags[g] = 1;
                }
            }
        }
        constexpr int LW = TileSmem<DT, BM, BN, STAGES>::list_words;
        list = list == sU + (TileSmem<DT, BM, BN, STAGES>::lists - 1) * LW ? sU : list + LW;
    }
}

// The kernel: reads the list length (or ranks the selection map) and runs
// the tile shape that suits it -- BNB listed pixels per tile normally, BNS when even the deepest K
// split of the big tiles would leave compute units idle (short lists): small tiles then need no
// or fewer shared tiles, whose partial sums and reduction are pure overhead.
template <int DT, int BM, int BNB, int WMB, int WNB, int SB, int BNS, int WMS, int WNS, int SS>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu((NT + 255) / 256, (NT + 255) / 256))) void gemm_gather_kernel(GemmArgs a)
{
    extern __shared__ __align__(16) float smem[];
    Selection sel = {nullptr, nullptr, 0};
    int n;
    if (a.sel_words > 0) {
        char *base = reinterpret_cast<char *>(smem) + KernelSmem<DT, BM, BNB, SB, BNS, SS>::sel_offset;
        uint64_t *sW = reinterpret_cast<uint64_t *>(base);
        int *sRank = reinterpret_cast<int *>(base + kSelSlots * 8);
        n = rank_selection(a, sW, sRank, sRank + kSelSlots, reinterpret_cast<uint64_t *>(smem));
        sel = make_selection(a, sW, sRank);
        if (a.sel_dilate && threadIdx.x < 64) write_update_map(a, sW); // a consumer wave: the first slices are awaited
    } else {
        n = a.count ? *a.count : a.max_pixels;
    }
    const long long big_tiles = (long long)((n + BNB - 1) / BNB) * (a.Mpad / BM);
    if (big_tiles * small_tile_factor(kStorage<DT>, BM, a.dNk.d) >= (long long)gridDim.x)
        gemm_gather_body<DT, BM, BNB, WMB, WNB, SB>(a, n, smem, sel);
    else
        gemm_gather_body<DT, BM, BNS, WMS, WNS, SS>(a, n, smem, sel);
}

// The halves of a filter matrix from its bfloat16 parts, once per state: a thread eight values of a fragment, which lie
// alike.  (On the host this took 2 ms for the 0.8 million weights of 64->256 7x7, as long as all the rest of its creation.)
__global__ void make_halves_kernel(const uintx4 *__restrict__ wt, uintx4 *__restrict__ out, size_t n, int shift)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const size_t fragment = i >> 6, lane = i & 63;
    uintx4 part[3], hi, lo;
#pragma unroll
    for (int p = 0; p < 3; ++p) part[p] = wt[(fragment * 3 + p) * 64 + lane];
    typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        halfx2 h, l;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            auto value = [&](int p) { return bf16_value((unsigned short)(part[p][q] >> (16 * e))); };
            const float v = __builtin_ldexpf(value(0) + (value(1) + value(2)), shift);
            h[e] = (_Float16)v;
            l[e] = (_Float16)((v - (float)h[e]) * (1 << kHalfLift));
        }
        hi[q] = __builtin_bit_cast(unsigned, h);
        lo[q] = __builtin_bit_cast(unsigned, l);
    }
    out[fragment * 128 + lane] = hi;
    out[fragment * 128 + 64 + lane] = lo;
}

// float32 layers of more than 32 channels that have their filter matrix in halves too: a big tile in halves where sums are
// long, else as in the kernel above.
template <int BM, int BNB, int WMB, int WNB, int SB, int BNS, int WMS, int WNS, int SS, int BNH, int SH>
struct HalvesSmem {
    static constexpr int th = TileSmem<kF32Halves, BM, BNH, SH>::tile_bytes;
    static constexpr int other = KernelSmem<kF32, BM, BNB, SB, BNS, SS>::sel_offset;
    static constexpr int sel_offset = ((th > other ? th : other) + 15) / 16 * 16;
    static constexpr int bytes = sel_offset + kSelSlots * 12 + 64;
    static_assert(bytes <= 160 * 1024, "a workgroup has 160 KiB of LDS");
};
template <int BM, int BNB, int WMB, int WNB, int SB, int BNS, int WMS, int WNS, int SS, int BNH, int SH>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu((NT + 255) / 256, (NT + 255) / 256))) void gemm_halves_kernel(GemmArgs a)
{
    extern __shared__ __align__(16) float smem[];
    Selection sel = {nullptr, nullptr, 0};
    int n;
    if (a.sel_words > 0) {
        char *base = reinterpret_cast<char *>(smem) + HalvesSmem<BM, BNB, WMB, WNB, SB, BNS, WMS, WNS, SS, BNH, SH>::sel_offset;
        uint64_t *sW = reinterpret_cast<uint64_t *>(base);
        int *sRank = reinterpret_cast<int *>(base + kSelSlots * 8);
        n = rank_selection(a, sW, sRank, sRank + kSelSlots, reinterpret_cast<uint64_t *>(smem));
        sel = make_selection(a, sW, sRank);
        if (a.sel_dilate && threadIdx.x < 64) write_update_map(a, sW); // a consumer wave: the first slices are awaited
    } else {
        n = a.count ? *a.count : a.max_pixels;
    }
    const long long big_tiles = (long long)((n + BNB - 1) / BNB) * (a.Mpad / BM);
    const int half_tiles = (n + BNH - 1) / BNH * (a.Mpad / BM);
    if (big_tiles * small_tile_factor(kF32, BM, a.dNk.d) < (long long)gridDim.x)
        gemm_gather_body<kF32, BM, BNS, WMS, WNS, SS>(a, n, smem, sel);
    else if (halves_suit(BM, half_tiles, fast_div(half_tiles, a.dGrid), a.dNk.d, (int)gridDim.x, a.halves_range))
        gemm_gather_body<kF32Halves, BM, BNH, 1, 8, SH>(a, n, smem, sel);
    else
        gemm_gather_body<kF32, BM, BNB, WMB, WNB, SB>(a, n, smem, sel);
}

// ---- layers whose whole reduction fits a wave's registers ----------------------------------
//
// A filter-matrix row of at most kThinGroups * 4 units (256 floats, 512 bfloat16) and at most
// kThinChannels output channels: first layers on camera frames, 1x1 layers on few channels.  The
// tile pipeline above spends most of such a launch filling and draining its ring -- a tile has a
// handful of K slices -- so here a wave works alone: 16 listed positions x 16 channels x the whole
// reduction.  Lane (pixel l % 16, slot l / 16) gathers units slot, 4 + slot, 8 + slot ... of its pixel's
// image-matrix row straight into registers, all loads in flight at once, and feeds them to the
// matrix cores against filter fragments read from an LDS copy of the filter matrix (rows one unit
// apart in the banks).  No barrier after set-up: the three waves of a SIMD hide each other's
// gather latency.  The positions come from the ranked map (each lane finds its own position with
// a binary search over the ranks) or from the list.  Every sum is formed in ascending k by one
// wave, so results do not depend on the number of positions.
static constexpr int kThinGroups = 16;
static constexpr int kThinChannels = 64;
static constexpr int kThinMaxWork = 32;     // groups x channel tiles up to which this kernel is used
// Tiles of 16 positions per wave from which the taps are kept in registers: 3->16 7x7 on 1280x720 (19 a wave) 89 -> 78 us, on
// 1800x1600 264 -> 225, 256->16 1x1 on 640x480 71.6 -> 69; in bfloat16 49.9 -> 41, 151 -> 124 and 28.9 -> 29.7, 12->16 3x3 there 14.6 ->
// 13.5; fewer do not pay for putting them there (320x240, 1.6 a wave: 12.2 either way).
static constexpr int kThinManyFactor = 4;
static constexpr int kThinWholeFactor = 2; // tiles of 16 positions per wave from which a wave takes all channel tiles
static constexpr int kThinScratchBytes = (kSelMaxWords + 2 * kSelGuard) * 8;                   // front-end scratch
static constexpr int kThinFilterBytes = kThinChannels * (kThinGroups * 4 + 1) * 16;              // [Mpad][units + 1]
static constexpr int kThinTapBytes = kThinGroups * 4 * (int)sizeof(int2);
static constexpr int kThinSelOffset = kThinScratchBytes + kThinFilterBytes + kThinTapBytes;
static constexpr int kThinSmemBytes = kThinSelOffset + kSelSlots * 12 + 64;
static_assert(kThinSmemBytes <= 160 * 1024, "a workgroup has 160 KiB of LDS");

// One wave's share of the tiles: 16 positions x TC channel tiles of 16.  In program order per tile:
// find the next tile's positions, multiply the current tile (its gathers were issued a tile ago),
// issue the next tile's gathers into the registers the MFMAs have just read, update the outputs of
// the current tile -- so a tile's gather latency passes during the update before it and the search
// after it.
// MANY: launches of several tiles a wave, on maps below 4 GiB with sides up to 16000, keep the taps in registers, packed
// coordinates and byte offsets: a gather is five vector instructions and a load from a scalar base, instead of a tap from
// LDS, a dozen instructions and a 64-bit address.
template <int DT, int TC, bool MANY>
__device__ __forceinline__ void thin_tiles(const GemmArgs &a, const int n, const Selection &sel, const uintx4 *sB,
                                           const int2 *sTap, const int G, const int pitch)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int cgroups = (a.Mpad >> 4) / TC; // wave tiles per pixel tile: 1, 2 or 4
    const int cshift = cgroups == 1 ? 0 : (cgroups == 2 ? 1 : 2);
    const long long T = (long long)((n + 15) >> 4) << cshift; // wave tiles, channel group fastest
    const int W = gridDim.x;
    // workgroups are dealt round-robin over the 8 XCDs: number them so that each XCD gets a contiguous range
    const int w = (int)(blockIdx.x & 7) * (W >> 3) + (int)(blockIdx.x >> 3);
    const int t_begin = (int)(T * w / W), t_end = (int)(T * (w + 1) / W);
    const int lrow = lane & 15, lk = lane >> 4;
    const float *x = static_cast<const float *>(a.x);
    const bool detect = a.next_flags != nullptr && !a.next_force;

    struct Where {
        int g, iy0, ix0, base;
    };
    auto locate = [&](int t) {
        const int r = (t >> cshift) * 16 + lrow;
        Where p = {-1, -(1 << 28), -(1 << 28), 0};
        if (r < n) p.g = sel.words ? select_rank(a, sel, r) : (a.list ? a.list[r] : r);
        if (p.g >= 0) {
            const int st = fast_div(p.g, a.dNo), q = p.g - st * a.No;
            const int qy = fast_div(q, a.dWo), qx = q - qy * a.Wo;
            p.iy0 = qy * a.stride - a.pad;
            p.ix0 = qx * a.stride - a.pad;
            p.base = ((st * a.H + p.iy0) * a.W + p.ix0) * a.pix_words;
        }
        return p;
    };
    floatx4 ra[kThinGroups];
    uintx4 replaced[TC];
    constexpr int KT = MANY ? kThinGroups : 1;
    unsigned taps[KT], offsets[KT]; // of this lane's units
    if constexpr (MANY) {
#pragma unroll
        for (int gg = 0; gg < kThinGroups; ++gg) {
            const int2 tp = sTap[gg < G ? 4 * gg + lk : lk];
            taps[gg] = (tp.y >> 16) != 0 ? (unsigned)(tp.y & 0xff) << 16 | (unsigned)(tp.y >> 8 & 0xff) : 0x40004000u;
            offsets[gg] = (unsigned)tp.x * 4u;
        }
    }
    auto gather = [&](const Where &p, int cg) {
        if constexpr (MANY) {
            const unsigned at0 = p.g >= 0 ? (unsigned)p.iy0 << 16 | ((unsigned)p.ix0 & 0xffffu) : 0x80008000u;
            const unsigned origin = (unsigned)p.base * 4u, zero = (unsigned)a.zero_word * 4u;
            const ushortx2 last = {(unsigned short)(a.W - 1), (unsigned short)(a.H - 1)};
#pragma unroll
            for (int gg = 0; gg < kThinGroups; ++gg) {
                if (gg < G) {
                    const ushortx2 at = __builtin_bit_cast(ushortx2, at0) + __builtin_bit_cast(ushortx2, taps[MANY ? gg : 0]);
                    const bool ok = __builtin_bit_cast(unsigned, __builtin_elementwise_sub_sat(at, last)) == 0u;
                    const unsigned o = ok ? origin + offsets[MANY ? gg : 0] : zero;
                    ra[gg] = *reinterpret_cast<const floatx4_a4 *>(reinterpret_cast<const char *>(x) + o);
                }
            }
        }
#pragma unroll
        for (int gg = 0; gg < kThinGroups; ++gg) {
            if (!MANY && gg < G) {
                const int2 tp = sTap[4 * gg + lk];
                const int tj = tp.y & 0xff, ti = (tp.y >> 8) & 0xff;
                const bool ok = (tp.y >> 16) != 0 && (unsigned)(p.iy0 + tj) < (unsigned)a.H && (unsigned)(p.ix0 + ti) < (unsigned)a.W;
                // outside the image (or no pixel in this row): the zero unit kept behind the map
                const unsigned idx = ok ? (unsigned)(p.base + tp.x) : (unsigned)a.zero_word;
                ra[gg] = *reinterpret_cast<const floatx4_a4 *>(x + idx);
            }
        }
        // the values about to be replaced, for the change detection of the layer this map feeds
#pragma unroll
        for (int j = 0; j < TC; ++j) {
            const int ch = (cg * TC + j) * 16 + lk * 4;
            replaced[j] = (uintx4){0u, 0u, 0u, 0u};
            if (detect && p.g >= 0 && ch < a.Ms) {
                if constexpr (DT == kBF16) {
                    const uint2 v = *reinterpret_cast<const uint2 *>(static_cast<const unsigned short *>(a.out) + (size_t)p.g * a.Ms + ch);
                    replaced[j][0] = v.x;
                    replaced[j][1] = v.y;
                } else {
                    replaced[j] = *reinterpret_cast<const uintx4 *>(static_cast<const float *>(a.out) + (size_t)p.g * a.Ms + ch);
                }
            }
        }
    };

    int t = t_begin + wave;
    if (t >= t_end) return;
    Where cur = locate(t);
    gather(cur, t & (cgroups - 1));
    while (t < t_end) {
        const int tn = t + NT / 64;
        const bool more = tn < t_end;
        Where nxt = {-1, 0, 0, 0};
        if (more) nxt = locate(tn);
        const int cg = t & (cgroups - 1);
        // MFMA step s of group gg contracts k = 16 gg + 4 slot + s over the four slots (bfloat16: the
        // eight k of a unit at once); D[4 slot + i][pixel] lands in this lane: four consecutive channels
        floatx4 acc[TC];
#pragma unroll
        for (int j = 0; j < TC; ++j) acc[j] = (floatx4){0.f, 0.f, 0.f, 0.f};
        const uintx4 *brow = sB + (cg * TC * 16 + lrow) * pitch + lk;
#pragma unroll
        for (int gg = 0; gg < kThinGroups; ++gg) {
            if (gg < G) {
#pragma unroll
                for (int j = 0; j < TC; ++j) {
                    const uintx4 bq = brow[j * 16 * pitch + 4 * gg];
                    if constexpr (DT == kBF16) {
                        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, bq),
                                                                     __builtin_bit_cast(bf16x8, ra[gg]), acc[j], 0, 0, 0);
                    } else {
                        const floatx4 bf = __builtin_bit_cast(floatx4, bq);
#pragma unroll
                        for (int s = 0; s < 4; ++s) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bf[s], ra[gg][s], acc[j], 0, 0, 0);
                    }
                }
            }
        }
        uintx4 old[TC];
#pragma unroll
        for (int j = 0; j < TC; ++j) old[j] = replaced[j];
        if (more) gather(nxt, tn & (cgroups - 1));
        // output update: bias, activation, scatter to the stored map
        bool changed = false;
#pragma unroll
        for (int j = 0; j < TC; ++j) {
            const int ch = (cg * TC + j) * 16 + lk * 4;
            if (cur.g >= 0 && ch < a.Ms) {
                const float4 bv = *reinterpret_cast<const float4 *>(a.bias + ch);
                float4 o;
                o.x = acc[j][0] + bv.x;
                o.y = acc[j][1] + bv.y;
                o.z = acc[j][2] + bv.z;
                o.w = acc[j][3] + bv.w;
                if (a.relu) {
                    o.x = fmaxf(o.x, 0.f);
                    o.y = fmaxf(o.y, 0.f);
                    o.z = fmaxf(o.z, 0.f);
                    o.w = fmaxf(o.w, 0.f);
                }
                if constexpr (DT == kBF16) {
                    uint2 nv;
                    nv.x = bf16_pair(o.x, o.y);
                    nv.y = bf16_pair(o.z, o.w);
                    if (detect)
                        changed |= fabsf(bf16_value(nv.x & 0xffff) - bf16_value(old[j][0] & 0xffff)) > a.next_tau ||
                                   fabsf(bf16_value(nv.x >> 16) - bf16_value(old[j][0] >> 16)) > a.next_tau ||
                                   fabsf(bf16_value(nv.y & 0xffff) - bf16_value(old[j][1] & 0xffff)) > a.next_tau ||
                                   fabsf(bf16_value(nv.y >> 16) - bf16_value(old[j][1] >> 16)) > a.next_tau;
                    *reinterpret_cast<uint2 *>(static_cast<unsigned short *>(a.out) + (size_t)cur.g * a.Ms + ch) = nv;
                    if (a.planar) store_planar(a, cur.g, ch, bf16_values(nv));
                } else {
                    if (detect)
                        changed |= fabsf(o.x - __uint_as_float(old[j][0])) > a.next_tau ||
                                   fabsf(o.y - __uint_as_float(old[j][1])) > a.next_tau ||
                                   fabsf(o.z - __uint_as_float(old[j][2])) > a.next_tau ||
                                   fabsf(o.w - __uint_as_float(old[j][3])) > a.next_tau;
                    *reinterpret_cast<float4 *>(static_cast<float *>(a.out) + (size_t)cur.g * a.Ms + ch) = o;
                    if (a.planar) store_planar(a, cur.g, ch, o);
                }
            }
        }
        if (a.next_flags) {
            int f = a.next_force ? 1 : (int)changed;
            // the other channels of this pixel sit in the lanes 16, 32 and 48 further on
            f |= __shfl_xor(f, 16);
            f |= __shfl_xor(f, 32);
            if (lk == 0 && f && cur.g >= 0) a.next_flags[cur.g] = 1;
        }
        cur = nxt;
        t = tn;
    }
}

// MT: channel tiles of the layer (Mpad / 16).  A wave takes all of them for its 16 positions when
// there are enough positions to occupy every wave that way, else one each.  MANY: maps on which a launch may have
// kThinManyFactor tiles a wave; a kernel of its own, for the sake of the small launches' registers and code.
template <int DT, int MT, bool MANY>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu((NT + 255) / 256, (NT + 255) / 256))) void gemm_thin_kernel(GemmArgs a)
{
    extern __shared__ __align__(16) float smem[];
    char *lds = reinterpret_cast<char *>(smem);
    uintx4 *sB = reinterpret_cast<uintx4 *>(lds + kThinScratchBytes);
    int2 *sTap = reinterpret_cast<int2 *>(lds + kThinScratchBytes + kThinFilterBytes);
    const int tid = threadIdx.x;
    const int nu = a.Kpad / Unit<DT>::N; // units per filter-matrix row: a multiple of eight
    // Groups that are not padding to the last unit: rows are stored in whole slices of eight units, and a group costs a wave
    // a gather and four MFMAs per channel tile whatever it holds.  13 instead of 14 for 3->16 7x7, 3 instead of 4 for
    // 3->64 3x3: 264 -> 249 us on 64 maps of 320 x 240, 107 -> 104 on 1280 x 720; bfloat16 27.9 -> 26.6 on 640 x 480.
    const int G = (a.kh * a.kw * a.dVin.d + 3) >> 2, pitch = nu + 1;
    {
        const uintx4 *wt = static_cast<const uintx4 *>(a.wt);
        for (int i = tid; i < a.Mpad * nu; i += NT) {
            const int r = fast_div(i >> 3, a.dNk), u = i - r * nu;
            sB[r * pitch + u] = wt[i];
        }
        for (int i = tid; i < nu; i += NT) sTap[i] = a.taps[i];
    }
    Selection sel = {nullptr, nullptr, 0};
    int n;
    if (a.sel_words > 0) {
        uint64_t *sW = reinterpret_cast<uint64_t *>(lds + kThinSelOffset);
        int *sRank = reinterpret_cast<int *>(lds + kThinSelOffset + kSelSlots * 8);
        n = rank_selection(a, sW, sRank, sRank + kSelSlots, reinterpret_cast<uint64_t *>(lds));
        sel = make_selection(a, sW, sRank);
        if (a.sel_dilate && threadIdx.x >= NT - 64) write_update_map(a, sW); // the wave with the fewest tiles
    } else {
        n = a.count ? *a.count : a.max_pixels;
    }
    __syncthreads();
    const int tiles = (n + 15) >> 4, waves = (NT / 64) * (int)gridDim.x;
    if constexpr (MANY) {
        if (tiles >= kThinManyFactor * waves) {
            thin_tiles<DT, 1, true>(a, n, sel, sB, sTap, G, pitch);
            return;
        }
    }
    if constexpr (MT > 1) {
        if (tiles >= kThinWholeFactor * waves) {
            thin_tiles<DT, MT, false>(a, n, sel, sB, sTap, G, pitch);
            return;
        }
    }
    thin_tiles<DT, 1, false>(a, n, sel, sB, sTap, G, pitch);
}

// ---- 1x1 layers on pixels of one or two units ------------------------------------------------
//
// A handful of products per output: nothing for the matrix cores, whose operands would be padding for
// the most part (3->8: 3 of 32 k, 8 of 16 channels), and a chain of search, gather, MFMA and store per
// sixteen positions.  Here a thread owns one 16-byte unit of output channels, keeps its weights in
// registers and takes positions, kPointBatch at a time so that as many pixels are on their way at once;
// the threads of a position sit next to each other, so that a wave stores one contiguous run.
// Bound by HBM: 3->8 on 2048 x 2048, every position, 133 -> 34 us from a list (24 + 16 + 64 + 128 MB of
// list, frame values and outputs: 6 TB/s), 111 -> 31 in order; 3->64 on 1024 x 1024 102 -> 54, 8->64 there
// 108 -> 78, bfloat16 3->8 34 -> 12.
static constexpr int kPointBatch = 4;
static constexpr int kPointGroups = 512; // workgroups up to which a short list is spread out: one position per thread

template <int DT, int VIN>
__global__ __launch_bounds__(256) void gemm_point_kernel(GemmArgs a, int mshift)
{
    constexpr int E = Unit<DT>::N, B = kPointBatch;
    const int n = a.count ? *a.count : a.max_pixels;
    // A list shorter than the map leaves workgroups idle rather than threads with fewer positions than their weights
    // are worth loading for: 8->64 on a tenth of 1024 x 1024 positions 15 us, with all workgroups 21.9 (thin kernel
    // 15), 3->8 on 2048 x 2048 6.9 and 8.5 (17).  Up to kPointGroups it spreads out: with fewer positions than
    // that the compute units, not the weights, are what is short (8->64 on a hundredth 6.4 us otherwise, now 4.7).
    const long long one = (((long long)n << mshift) + 255) / 256; // workgroups for a position per thread
    const long long want = one <= kPointGroups ? one : (one <= (long long)kPointGroups * B ? kPointGroups : (one + B - 1) / B);
    const int groups = want < (long long)gridDim.x ? (int)want : (int)gridDim.x;
    if ((int)blockIdx.x >= groups) return;
    // a map without padding has the next pixel's values behind its channels
    const int C = DT == kBF16 ? VIN * E : (a.pix_words < VIN * E ? a.pix_words : VIN * E);
    const int m = (int)threadIdx.x & ((1 << mshift) - 1);
    const bool detect = a.next_flags != nullptr && !a.next_force;
    const float *x = static_cast<const float *>(a.x);
    uint4 *out = static_cast<uint4 *>(a.out);
    float w[E][VIN * E], bias[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const size_t row = (size_t)(m * E + e) * a.Kpad; // rows up to Mpad exist, zero beyond M
        bias[e] = a.bias[m * E + e];
#pragma unroll
        for (int c = 0; c < VIN * E; ++c)
            w[e][c] = DT == kBF16 ? bf16_value(static_cast<const unsigned short *>(a.wt)[row + c]) : static_cast<const float *>(a.wt)[row + c];
    }
    const int per = 256 >> mshift, step = groups * per; // positions per workgroup and pass
    for (long long r0 = (long long)blockIdx.x * per + ((int)threadIdx.x >> mshift); r0 < n; r0 += (long long)B * step) {
        int g[B];
        uint4 v[B][VIN], old[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const long long r = r0 + (long long)b * step;
            g[b] = r < n ? (a.list ? a.list[r] : (int)r) : -1;
        }
#pragma unroll
        for (int b = 0; b < B; ++b) {
            old[b] = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
            for (int u = 0; u < VIN; ++u) v[b][u] = old[b];
            if (g[b] < 0) continue;
#pragma unroll
            for (int u = 0; u < VIN; ++u)
                v[b][u] = __builtin_bit_cast(uint4, *reinterpret_cast<const floatx4_a4 *>(x + (size_t)g[b] * a.pix_words + u * 4));
            if (detect) old[b] = out[((size_t)g[b] << mshift) + m];
        }
#pragma unroll
        for (int b = 0; b < B; ++b) {
            if (g[b] < 0) continue;
            uint4 nv = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
            for (int e = 0; e < E; ++e) {
                float s = 0.f;
#pragma unroll
                for (int c = 0; c < VIN * E; ++c)
                    if (c < C) s = fmaf(Unit<DT>::get(v[b][c / E], c % E), w[e][c], s);
                s += bias[e];
                if (a.relu) s = fmaxf(s, 0.f);
                Unit<DT>::set(nv, e, s);
            }
            out[((size_t)g[b] << mshift) + m] = nv;
            // several threads of a position may store the same 1
            if (a.next_flags && (a.next_force || unit_exceeds<DT>(nv, old[b], a.next_tau))) a.next_flags[g[b]] = 1;
        }
    }
}

// Whether a launch goes to gemm_point_kernel: a 1x1 layer of few enough weights per output unit for
// registers (8 float32 or 8 bfloat16 values per pixel) and units of output that divide a wave, on a map too
// large to be ranked in the kernel.  That is a property of the layer alone, and has to be: the two kernels add
// a position's products in different orders, and the same layer must give the same bits whether its positions
// come from the map, from a list or are all of them.  (Maps that can be ranked are in the thin kernel's hands
// whichever way their positions come: in order, 3->8 on 320 x 240 takes 7.7 us there and 4.5 here.)  On
// 400 x 400 positions it takes 6 us for 3->8 (thin: 9.5) and 15 for 3->64 (21).  Two units of pixel into sixteen
// of output are 64 weights a thread, and pay from 2^19 positions on: 8->64 on 400 x 400 20.9 (20.3), 512 x 512
// 30 (27.7), 1024 x 1024 78 (112).
static bool gemm_is_point(const GemmArgs &a)
{
    const int units = a.Ms / elems_per_unit(a.dtype);
    return a.kh == 1 && a.kw == 1 && a.stride == 1 && a.pad == 0 && a.sel_words == 0 && a.max_pixels > kSelMaxWords * 64 &&
           a.dVin.d <= (a.dtype == kBF16 ? 1 : 2) && (units & (units - 1)) == 0 && a.Ms <= a.Mpad &&
           (a.dVin.d * units < 32 || a.max_pixels >= 1 << 19);
}

// The lone waves win as long as (groups of four units) x (channel tiles) stays at or below 32 -- beyond that
// a wave's chain of MFMAs per tile gets long and the big tiles' reuse of filter fragments pays.  Against the tile
// pipeline, float32, dense and with a tenth of the input changed, in us (thin / tiles): 3->16 7x7 on 320 x 240
// 13.1 / 20.4 and 11.9 / 13.5, on 1280 x 720 98.7 / 119 and 13.5 / 20.2, on 3840 x 2160 788 / 982 and 86 / 103;
// 5x5/2 3->32 on 640 x 480 23.0 / 24.8 and 5.8 / 7.4; 3x3 3->64 there 39.0 / 40.9 and 10.8 / 9.2; 3x3 16->32 on
// 320 x 240 25.8 / 26.3 and 11.2 / 11.7 (with three quarters changed 26.1 / 21.2, the largest loss found); 256->16
// 1x1 on 160 x 120 8.2 / 8.1 and 7.8 / 9.5, on 320 x 240 16.4 / 25.0 and 7.8 / 9.6.  bfloat16 3->16 7x7 on
// 1280 x 720 56 / 88 and 9.7 / 16.7.
static bool is_thin(int dtype, int Mpad, int Kpad)
{
    const int nu = Kpad / elems_per_unit(dtype);
    return nu <= kThinGroups * 4 && (Mpad == 16 || Mpad == 32 || Mpad == 64) && (nu / 4) * (Mpad / 16) <= kThinMaxWork;
}
static bool gemm_is_thin(const GemmArgs &a) { return is_thin(a.dtype, a.Mpad, a.Kpad); }

bool gemm_filter_in_fragments(int dtype, int Mpad, int Kpad) { return !is_thin(dtype, Mpad, Kpad); }

size_t gemm_filter_bytes(int dtype, int Mpad, int Kpad)
{
    return (size_t)Mpad * Kpad * (gemm_filter_in_fragments(dtype, Mpad, Kpad) && dtype == kF32 ? 6 : elem_bytes(dtype));
}

size_t gemm_filter_fragment(int dtype, int Mpad, int Kpad, int row, int k)
{
    const int ks = gemm_k_multiple(dtype);
    return dtype == kF32 ? filter_fragment<kF32>(gemm_channel_tile(Mpad), Kpad / ks, row, k)
                         : filter_fragment<kBF16>(gemm_channel_tile(Mpad), Kpad / ks, row, k);
}

// ---- host side --------------------------------------------------------------------------
bool gemm_filter_halves(const GemmArgs &a, int grid)
{
    if (a.dtype != kF32 || a.Mpad < 64 || gemm_is_thin(a)) return false;
    const int bm = gemm_channel_tile(a.M);
    const int tiles = (a.max_pixels + 127) / 128 * (a.Mpad / bm);
    return halves_suit(bm, tiles, tiles / grid, a.Kpad / gemm_k_multiple(kF32), grid, a.halves_range);
}

size_t gemm_halves_bytes(int Mpad, int Kpad) { return (size_t)Mpad * Kpad * 4 + (size_t)Mpad * 4; }

float gemm_halves_least(double magnitudes, int small)
{
    return (float)std::ldexp(magnitudes + std::ldexp((double)small, kHalfLimit), kHalfBits - 36);
}

hipError_t gemm_make_halves(hipStream_t st, const void *wt, void *wt_halves, int Mpad, int Kpad, int shift)
{
    if (!wt || !wt_halves || Mpad < 64 || Mpad % 16 || Kpad < 1 || Kpad % gemm_k_multiple(kF32)) return hipErrorInvalidValue;
    const size_t n = (size_t)Mpad * Kpad / 8;
    make_halves_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st>>>(static_cast<const uintx4 *>(wt), static_cast<uintx4 *>(wt_halves),
                                                                                n, shift);
    return hipGetLastError();
}

unsigned gemm_tiny_sum(int K, float largest_weight)
{
    const double t = std::ldexp((double)K * largest_weight, -110);
    const float f = t < FLT_MAX ? (float)t : FLT_MAX;
    unsigned u;
    memcpy(&u, &f, 4);
    return u ? (u << 1) - 1 : 0;
}

int gemm_k_multiple(int dtype) { return BK * 4 / elem_bytes(dtype); }

// How the producers of the tile kernel address image-matrix rows (direct_producer): with 32-bit byte offsets, and
// tests of tap rows and columns in 16 bits or as bits of a word, wherever the map allows it.
static int taps_mode(const GemmArgs &a)
{
    const long long pixels = (long long)a.S * a.N, above = (long long)a.pad * (a.W + 1);
    if ((pixels + above) * a.pix_words * 4 + 16 >= 1ll << 32) return kTapGeneral;
    // the zero unit must not lie before the window of the last tap, from which its offset is counted
    if (a.dVin.d % KU == 0 && a.kw <= 32 && pixels + above >= (long long)a.kh * a.W + a.kw) return kTapUniform;
    return a.H <= 16000 && a.W <= 16000 ? kTapPerLane : kTapGeneral;
}

// Words of a row in the ranking where rows begin with words of their own (GemmArgs::sel_ranked, dSelRow), else 0.  Words
// that run across rows are put together from a piece per row, one after the other, which takes longer than the more words
// of short rows do, as long as LDS holds them: 64->64 3x3 on 64 maps of 10 x 10 (100 words or 640) 17.8 and 14.5 us, 7x7
// 23.9 and 21.0, 3->16 3x3 on 400 of 5 x 5 (157 or 2000) 15.9 and 9.6, 64->64 7x7 on 600 of 3 x 3 37.6 and 26.5, on 2000 x 5
// 23.9 and 17.4, on 1000 x 65 16.9 and 16.4, on 83 x 61 15.8 and 14.6.
static int sel_row_words(const GemmArgs &a)
{
    if (a.sel_words <= 0 || !a.sel_dilate || a.Wo < 1) return 0;
    const long long per_row = (a.Wo + 63) / 64;
    return per_row * (a.max_pixels / a.Wo) <= kSelMaxWords ? (int)per_row : 0;
}

void gemm_set_divisors(GemmArgs &a)
{
    a.dNo = make_fastdiv(a.No > 0 ? a.No : 1);
    a.dWo = make_fastdiv(a.Wo > 0 ? a.Wo : 1);
    a.dHo = make_fastdiv(a.Wo > 0 && a.No >= a.Wo ? a.No / a.Wo : 1);
    const int nk = a.Kpad / gemm_k_multiple(a.dtype);
    a.dNk = make_fastdiv(nk > 0 ? nk : 1);
    a.dGrid = make_fastdiv(a.grid > 0 ? a.grid : 1);
    a.dVin = make_fastdiv(a.pix_words > 0 ? (a.pix_words + 3) / 4 : 1);
    a.dKw = make_fastdiv(a.kw > 0 ? a.kw : 1);
    a.taps_mode = taps_mode(a);
    const int per_row = sel_row_words(a);
    a.sel_ranked = per_row ? per_row * (a.max_pixels / a.Wo) : a.sel_words;
    a.dSelRow = per_row ? make_fastdiv(per_row) : FastDiv{0, 0, 0};
}

int gemm_select_max_words(void) { return kSelMaxWords; }

int gemm_channel_tile(int M)
{
    if (M <= 16) return 16;
    if (M <= 32) return 32;
    if (M <= 64) return 64;
    return 128;
}

// Pixels per big tile.  The 64-channel kernel takes 128 instead of 256 on maps of few positions, where
// 256-pixel tiles leave workgroups idle in the last round or most of them a third of a tile's K range.  The line
// lies higher for float32, whose slices carry six products per value and hide their loads at either
// width: 32->64 3x3 at 320x240 33.7 -> 28.1 us, 16->64 7x7 at 640x360 131.4 -> 131.0, and 6.90 -> 7.05 ms for
// two frames of 64 streams (1.2 million positions).  bfloat16, 16->64 7x7 at 640x360: 55.1 -> 57.7 us.
static int pixel_tile(int bm, int max_pixels, int dtype)
{
    if (bm == 128) return 128;
    return bm == 64 && max_pixels <= (dtype == kF32 ? 1 << 19 : 1 << 16) ? 128 : 256;
}

// One ticket counter per shared tile (fewer than the workgroup count) and wave; zero between launches.
size_t gemm_ticket_bytes(int grid) { return (size_t)grid * kConsWaves * sizeof(int); }

// Workgroups to launch: one per compute unit, fewer if even the longest list gives less work.
int gemm_grid(const GemmArgs &a, int compute_units)
{
    const int bm = gemm_channel_tile(a.M), bn = pixel_tile(bm, a.max_pixels, a.dtype);
    int W = compute_units & ~7;
    if (W < 8) W = 8;
    if (W > kMaxGrid) W = kMaxGrid;
    if (gemm_is_thin(a)) {
        // a workgroup per four wave tiles of 16 positions x 16 channels (one per SIMD: spreading a short
        // list over more compute units shortens the launch, 128->16 1x1 at 160x120: 6.6 -> 5.4 us)
        const long long wave_tiles = (long long)((a.max_pixels + 15) / 16) * (a.Mpad / 16);
        long long need = ((wave_tiles + 3) / 4 + 7) / 8 * 8;
        if (need < 8) need = 8;
        return (int)(need < W ? need : W);
    }
    const int nk = a.Kpad / gemm_k_multiple(a.dtype);
    const int parts = nk / kMinIters > 1 ? nk / kMinIters : 1;
    // with few pixels the small tile (64 pixels) is used: count those
    const long long big = (long long)((a.max_pixels + bn - 1) / bn) * (a.Mpad / bm);
    const long long tiles = big * small_tile_factor(a.dtype, bm, nk) >= W ? big : (long long)((a.max_pixels + 63) / 64) * (a.Mpad / bm);
    long long need = tiles >= W ? W : (tiles * parts + 7) / 8 * 8;
    if (need < 8) need = 8;
    return (int)(need < W ? need : W);
}

bool gemm_takes_halves(const GemmArgs &a, int n) // as gemm_halves_kernel
{
    const int bm = gemm_channel_tile(a.M), bn = pixel_tile(bm, a.max_pixels, a.dtype), nk = a.Kpad / gemm_k_multiple(kF32), mtiles = a.Mpad / bm;
    const int half_tiles = (n + 127) / 128 * mtiles;
    return gemm_filter_halves(a, a.grid) && (long long)((n + bn - 1) / bn) * mtiles * small_tile_factor(kF32, bm, nk) >= a.grid &&
           halves_suit(bm, half_tiles, half_tiles / a.grid, nk, a.grid, a.halves_range);
}

// Two slabs of partial sums per workgroup, of the tile shape that the launch uses.  That is the big one only if
// its tiles of the longest list come to the launch's workgroups / small_tile_factor, which on a map of few
// positions they do in launches of few workgroups alone.  (Fewer compute units never make for more workgroups.)
size_t gemm_partial_bytes(const GemmArgs &a, int compute_units)
{
    if (gemm_is_thin(a)) return 0;
    const int bm = gemm_channel_tile(a.M), bn = pixel_tile(bm, a.max_pixels, a.dtype), bns = bm == 16 ? 128 : 64;
    const long long grid = gemm_grid(a, compute_units);
    const long long big = (long long)((a.max_pixels + bn - 1) / bn) * (a.Mpad / bm) *
                          small_tile_factor(a.dtype, bm, a.Kpad / gemm_k_multiple(a.dtype));
    const long long wide = (big < grid ? big : grid) * bn, narrow = grid * bns;
    return 2 * sizeof(float) * bm * (size_t)(wide > narrow ? wide : narrow);
}

// storage type; BM; big tile (BN, WM, WN, ring slices); small tile (the same)
// float32 with halves: the same, then the tile in halves (BN, ring slices).  Of 64 channels it is 128 pixels on every map:
// 16->64 7x7 on 1200x1280 662 us, in parts 773; with 256 pixels 26 registers spilled (737 us where 128 took 613, before a pixel had
// a scale of its own).
#define CBK_HALVES(X)                                \
    X(64, 256, 1, 8, 3, 64, 2, 4, 5, 128, 5)         \
    X(64, 128, 1, 8, 4, 64, 2, 4, 5, 128, 5)         \
    X(128, 128, 1, 8, 3, 64, 2, 4, 4, 128, 4)
#define CBK_VARIANTS(X)                                  \
    X(kF32, 16, 256, 1, 8, 3, 128, 1, 8, 4)              \
    X(kF32, 32, 256, 1, 8, 3, 64, 2, 4, 4)               \
    X(kF32, 64, 256, 1, 8, 3, 64, 2, 4, 5)               \
    X(kF32, 64, 128, 1, 8, 4, 64, 2, 4, 5)               \
    X(kF32, 128, 128, 1, 8, 3, 64, 2, 4, 4)              \
    X(kBF16, 16, 256, 1, 8, 3, 128, 1, 8, 4)             \
    X(kBF16, 32, 256, 1, 8, 3, 64, 2, 4, 4)              \
    X(kBF16, 64, 256, 2, 4, 3, 64, 2, 4, 5)              \
    X(kBF16, 64, 128, 2, 4, 4, 64, 2, 4, 5)              \
    X(kBF16, 128, 128, 2, 4, 4, 64, 4, 2, 5)

#define X(DT_, BM_, BNB_, WMB_, WNB_, SB_, BNS_, WMS_, WNS_, SS_) \
    static_assert(BNS_ == (BM_ == 16 ? 128 : 64) && BNB_ >= BNS_, "gemm_partial_bytes counts on these tiles");
CBK_VARIANTS(X)
#undef X

// One channel tile only: wider layers gather less per MFMA (5x5/2 3->32 on 640x480 33.9 -> 34.5 us, 3x3 16->32 there 40.1 ->
// 40.7).
static bool thin_many(const GemmArgs &a)
{
    return a.Mpad == 16 && (a.max_pixels + 15) / 16 >= kThinManyFactor * (NT / 64) * a.grid && a.taps_mode != kTapGeneral &&
           a.H <= 16000 && a.W <= 16000;
}
// storage type; channel tiles; many tiles a wave
#define CBK_THIN(T)                                                      \
    T(kF32, 1, false) T(kF32, 1, true) T(kF32, 2, false) T(kF32, 4, false) \
    T(kBF16, 1, false) T(kBF16, 1, true) T(kBF16, 2, false) T(kBF16, 4, false)

hipError_t gemm_prepare(void)
{
    hipError_t e = hipSuccess;
#define X(DT_, BM_, BNB_, WMB_, WNB_, SB_, BNS_, WMS_, WNS_, SS_)                                                         \
    if (e == hipSuccess)                                                                                                  \
        e = hipFuncSetAttribute(                                                                                          \
            reinterpret_cast<const void *>(&gemm_gather_kernel<DT_, BM_, BNB_, WMB_, WNB_, SB_, BNS_, WMS_, WNS_, SS_>),  \
            hipFuncAttributeMaxDynamicSharedMemorySize, KernelSmem<DT_, BM_, BNB_, SB_, BNS_, SS_>::bytes);
    CBK_VARIANTS(X)
#undef X
#define X(...)                                                                                                                      \
    if (e == hipSuccess)                                                                                                            \
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_halves_kernel<__VA_ARGS__>), hipFuncAttributeMaxDynamicSharedMemorySize, \
                                HalvesSmem<__VA_ARGS__>::bytes);
    CBK_HALVES(X)
#undef X
#define T(DT_, MT_, MANY_)                                                                                         \
    if (e == hipSuccess)                                                                                           \
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_thin_kernel<DT_, MT_, MANY_>),                \
                                hipFuncAttributeMaxDynamicSharedMemorySize, kThinSmemBytes);
    CBK_THIN(T)
#undef T
    return e;
}

hipError_t gemm_gather(hipStream_t st, const GemmArgs &a, const Timing &tm)
{
    const int bm = gemm_channel_tile(a.M), bn = pixel_tile(bm, a.max_pixels, a.dtype);
    const int eu = elems_per_unit(a.dtype);
    if (a.Mpad % bm != 0 || a.Kpad % gemm_k_multiple(a.dtype) != 0 || a.Ms % eu != 0 || a.pix_words < 1 || !a.partial ||
        !a.tickets || a.grid < 8 || (a.grid & 7) || a.grid > kMaxGrid)
        return hipErrorInvalidValue;
    if (a.wt_halves && (a.dtype != kF32 || bm < 64 || gemm_is_thin(a))) return hipErrorInvalidValue;
    // the wide 64-channel tile in float32 counts on rows of four slices or more (TileSmem::lists); those it gets have five
    if (a.dtype == kF32 && bm == 64 && bn == 256 && !gemm_is_thin(a) && a.Kpad < 4 * gemm_k_multiple(kF32)) return hipErrorInvalidValue;
    // the divisors must belong to these arguments, and the schedule's 32-bit arithmetic must hold
    if (a.kh < 1 || a.kw < 1 || a.dKw.d != a.kw || a.dVin.d != (a.pix_words + 3) / 4) return hipErrorInvalidValue;
    if (a.dNo.d != a.No || a.dWo.d != a.Wo || a.dHo.d * a.Wo != a.No || a.dGrid.d != a.grid ||
        a.dNk.d != a.Kpad / gemm_k_multiple(a.dtype) || a.dNk.d >= (1 << 20))
        return hipErrorInvalidValue;
    // so must what else was derived from them: the ranking's room in LDS, where ranked words lie, the producers' 32-bit offsets
    const int per_row = sel_row_words(a);
    if (a.taps_mode != taps_mode(a) || a.dSelRow.d != per_row || a.sel_ranked != (per_row ? per_row * (a.max_pixels / a.Wo) : a.sel_words))
        return hipErrorInvalidValue;
    if (a.sel_words > 0 && a.sel_dilate &&
        (a.stride != 1 || a.kw > 16 || a.kw < 1 || a.kh < 1 || a.kh > 16 || !a.upd_out || a.S < 1 || a.sel_in_words < 1 ||
         a.sel_in_words > kSelMaxWords || (long long)a.sel_in_words * 64 < (long long)a.S * a.N || a.No % a.Wo != 0))
        return hipErrorInvalidValue;
    if (a.sel_words < 0 || a.sel_words > kSelMaxWords || (a.sel_words > 0 && !a.sel_map) ||
        (a.sel_words == 0 && !a.list != !a.count) || (long long)a.sel_words * 64 < a.max_pixels * (a.sel_words > 0))
        return hipErrorInvalidValue;
    if (gemm_is_thin(a) && gemm_is_point(a)) {
        if (a.planar) return hipErrorInvalidValue; // maps that may be ranked only
        int mshift = 0;
        while ((1 << mshift) < a.Ms / eu) ++mshift;
        long long grid = (((long long)a.max_pixels << mshift) + 256 * kPointBatch - 1) / (256 * kPointBatch);
        if (grid > 4096) grid = 4096;
        if (grid < 1) grid = 1;
#define P(DT_, V_)                                                                                           \
    if (a.dtype == DT_ && a.dVin.d == V_) {                                                                   \
        launch_kernel(tm, gemm_point_kernel<DT_, V_>, dim3((int)grid), dim3(256), 0, st, a, mshift);          \
        return hipGetLastError();                                                                            \
    }
        P(kF32, 1) P(kF32, 2) P(kBF16, 1)
#undef P
    }
    if (gemm_is_thin(a)) {
        const bool many = thin_many(a);
#define T(DT_, MT_, MANY_)                                                                                    \
    if (a.dtype == DT_ && a.Mpad == 16 * MT_ && many == MANY_) {                                               \
        launch_kernel(tm, gemm_thin_kernel<DT_, MT_, MANY_>, dim3(a.grid), dim3(NT), kThinSmemBytes, st, a);  \
        return hipGetLastError();                                                                             \
    }
        CBK_THIN(T)
#undef T
    }
    if (a.wt_halves) {
#define X(BM_, BNB_, ...)                                                                                                         \
    if (bm == BM_ && bn == BNB_) {                                                                                                \
        launch_kernel(tm, gemm_halves_kernel<BM_, BNB_, __VA_ARGS__>, dim3(a.grid), dim3(NT), (HalvesSmem<BM_, BNB_, __VA_ARGS__>::bytes), st, a); \
        return hipGetLastError();                                                                                                 \
    }
        CBK_HALVES(X)
#undef X
    }
#define X(DT_, BM_, BNB_, WMB_, WNB_, SB_, BNS_, WMS_, WNS_, SS_)                                                        \
    if (a.dtype == DT_ && bm == BM_ && bn == BNB_) {                                                                     \
        launch_kernel(tm, gemm_gather_kernel<DT_, BM_, BNB_, WMB_, WNB_, SB_, BNS_, WMS_, WNS_, SS_>, dim3(a.grid),      \
                      dim3(NT), (KernelSmem<DT_, BM_, BNB_, SB_, BNS_, SS_>::bytes), st, a);                             \
        return hipGetLastError();                                                                                        \
    }
    CBK_VARIANTS(X)
#undef X
    return hipErrorInvalidValue;
}

} // namespace cbk
