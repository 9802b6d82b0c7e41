// szi_internal.h -- structures shared by libszi's host code and its gfx950
// kernels.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "szi_limits.h"

namespace szi {

constexpr int kLutBits = 13;       // decode look-up table width (bits)
constexpr int kRangeBlocks = 2048; // partial min/max blocks per field
constexpr int kThreads = 256;      // threads per interpolation workgroup
constexpr int kEncBlockMax = 32;      // Huffman chunks per encode workgroup, at most
constexpr int kDecBlockChunks = 256;  // Huffman chunks per decode workgroup
constexpr int kWordPad = 8;        // allocated u32 past the end of every Huffman word array

// Static description of one field, written by the host before launch.
// Decode lanes per Huffman chunk: the encoder records where each of a
// chunk's kSubParts equal parts starts, and one lane decodes each part.
constexpr int kSubParts = 8;

struct FieldDesc {
    int32_t ndim;
    int32_t n[3];          // n[0] fastest; unused dims 1
    int32_t w[3];          // window; unused dims 1
    int32_t nwin[3];       // windows per dimension
    uint32_t wmag[2];      // floor(2^32 / m), m = nwin[0] and nwin[0] * nwin[1] (at most 2^32 - 1)
    int32_t na[3];         // anchors per dimension
    int32_t S, L, R;
    int32_t eb_mode;
    int32_t need_prof;
    int32_t interp[3];     // requested splines (AUTO allowed)
    int32_t order_req[3];  // requested order; order_req[0] < 0 = auto
    int32_t chunk;         // Huffman chunk
    double eb;
    double alpha_req;
    uint64_t npts;
    uint64_t chunk_base;   // first chunk of this field in a batch
    uint64_t tab_src;      // its code tables' offset in a batch's staged table region
    uint64_t nchunks;
    uint64_t n_outliers;
    uint64_t words_cap;    // capacity of words (encode)
    const float* in;       // compress input
    float* out;            // decompress output
    uint16_t* codes;
    float* anchors;
    uint32_t* hist;        // 2R bins
    // Huffman encode/decode
    const uint32_t* cbook; // per symbol: codeword << (32 - len) | len (0 without a code)
    uint32_t* words;
    uint16_t* chunk_bits;
    uint32_t* outlier_idx;
    float* outlier_val;
    const uint32_t* dtab;  // decode tables (see DecodeTables layout)
    unsigned long long* tot;  // compress: receives the field's words and non-zero words
    uint32_t* esec;        // compress: its words section with the zero words elided
    uint16_t* sub;         // per chunk kSubParts entries: its place, then the bits where its 2nd .. last eighth starts (or null)
};

// One pass of the interpolation (Sec. V-A: levels from stride S/2 to 1, one
// pass per dimension in the planned order), as the window kernels run it:
// the points of the pass lie on nlines lines along dimension d, numbered
// i0 + ne * i1 over the two other dimensions e < g (i1 = 0 in 2D); line
// (i0, i1) lies at coordinate i0 << she along e and i1 << shg along g.  Six
// words, so that the passes of a window (nine in 3D, eight in 2D) fit one
// register of a wave, a word a lane.
constexpr int kMaxPasses = 12;
struct PassDesc {
    uint32_t kind;             // d | spl << 2 | she << 4 | shg << 8
    uint32_t lines;            // nlines | ne << 16
    uint32_t magic;            // ceil(2^16 / ne): i1 = line * magic >> 16 (lines < 300)
    float el, ebx2, inv;       // level bound, 2 e_l, 1 / (2 e_l) (0 when e_l = 0)
};
constexpr int kPassWords = sizeof(PassDesc) / 4;
static_assert(kPassWords == 6 && 9 * kPassWords <= 64 && kMaxPasses * kPassWords >= 64,
              "a word per lane, and a wave's load stays inside the array");

// Per-field plan computed on the device from the range and the profile.
struct FieldPlan {
    float vmin, vmax;
    uint32_t nonfinite;
    int32_t status;        // 0 ok, -2 non-finite input
    double range, eps, e_abs;
    float e;
    int32_t levels;
    double alpha;
    float el[kMaxLevels];
    float ebx2[kMaxLevels];
    float inv[kMaxLevels];
    int32_t spline[3];
    int32_t order[3];
    double prof[3][3];     // [dim][linear, NAK, natural] L1 errors
    PassDesc pass[kMaxPasses];   // derived from order, spline and e_l
};

// Windows are handed to the interpolation kernels in groups of this many,
// one per wave of a workgroup; each field is padded to whole groups.
constexpr int kWinPerGroup = 4;

// Decode tables, one u32 array per field:
//   LUT, 1<<kLutBits u16 entries in (1<<kLutBits)/2 words: len << 11 | symbol
//                      for the codes of at most kLutBits bits (symbols < 2048;
//                      len 0 = longer code)
//   limit[kLmax+1]     limit[l]: the codes of length <= l, left-justified to
//                      kLmax bits, lie below it ((first + count) << (kLmax - l))
//   base[kLmax+1]      base[l]: position of length l among the sorted
//                      symbols minus the first code of length l
//   sorted symbols (nsym entries, by (length, symbol))
constexpr int kLutSymBits = 11;
constexpr int kDtLimit = (1 << kLutBits) / 2;
constexpr int kDtBase = kDtLimit + kLmax + 1;
constexpr int kDtSorted = kDtBase + kLmax + 1;
static_assert(2 * kMaxRadius <= (1 << kLutSymBits) && kLutBits < (1 << (16 - kLutSymBits)),
              "LUT entries hold a symbol and a length in 16 bits");
__host__ __device__ inline int dtab_words(int nsym) { return kDtSorted + nsym; }

// ---- launchers (k_plan.hip, k_interp.hip, k_huff.hip) ----
// range partials and, in one extra block per field, the profiling (Sec. V-C.1)
hipError_t launch_range(const FieldDesc* d_fields, FieldPlan* d_plans, int nfields,
                        float* d_part_min, float* d_part_max, uint32_t* d_part_bad,
                        hipStream_t st);
// zero: nzero words to clear (the encode's sums)
hipError_t launch_plan(const FieldDesc* d_fields, FieldPlan* d_plans, int nfields,
                       const float* d_part_min, const float* d_part_max,
                       const uint32_t* d_part_bad, uint32_t* zero, uint64_t nzero, hipStream_t st);
hipError_t launch_zero_hist(const FieldDesc* d_fields, int nfields, hipStream_t st);
// decompression prologue: block word counts, outlier scatter, pass descriptors
hipError_t launch_dec_prep(const FieldDesc* d_fields, FieldPlan* d_plans, int nfields,
                           const uint64_t* d_dboff, uint64_t nblocks, uint32_t* d_bsum,
                           hipStream_t st);
hipError_t launch_fill_u32(uint32_t* p, uint64_t n, uint32_t v, hipStream_t st);
// batches: every field's histogram into dst + f * stride, and every field's
// code tables from the staged region src (at tab_src) to its table block
// (the 16-byte-padded lengths before cbook)
hipError_t launch_gather_hist(const FieldDesc* d_fields, int nfields, uint32_t* dst,
                              uint32_t stride, hipStream_t st);
hipError_t launch_scatter_tables(const FieldDesc* d_fields, int nfields, const uint8_t* src,
                                 hipStream_t st);
// Launch shape of a window kernel; every shape gives the same results.
// variant 0: compiled for three waves per SIMD (168 VGPRs); variant 1: for
// four (128 VGPRs; 2D only, whose smaller blocks leave LDS for 16 windows
// per CU).  per_cu: persistent workgroups per CU, 0 = resident capacity.
struct LaunchShape {
    int variant = 0;
    int per_cu = 0;
};
constexpr int kShapeVariants = 2;
hipError_t launch_compress(int ndim, const FieldDesc* d_fields, const FieldPlan* d_plans,
                           const uint64_t* d_goff, uint64_t ngroups, int num_cus,
                           LaunchShape shape, int max_R, hipStream_t st);
// Fields of any anchor stride and window (block points <= kGenMaxBlock):
// the generic window kernels, geometry from the descriptors; block: the
// points of the launch's largest block.
hipError_t launch_compress_gen(const FieldDesc* d_fields, const FieldPlan* d_plans,
                               const uint64_t* d_goff, uint64_t ngroups, int num_cus, int max_R,
                               uint64_t block, hipStream_t st);
hipError_t launch_decompress_gen(const FieldDesc* d_fields, const FieldPlan* d_plans,
                                 const uint64_t* d_goff, uint64_t ngroups, int num_cus,
                                 uint64_t block, hipStream_t st);
hipError_t launch_decompress(int ndim, const FieldDesc* d_fields, const FieldPlan* d_plans,
                             const uint64_t* d_goff, uint64_t ngroups, int num_cus,
                             LaunchShape shape, hipStream_t st);
// Chunks per encode workgroup (a multiple of its four waves): 32 where that
// leaves eight workgroups a CU, fewer on smaller calls, where a workgroup's
// chunks follow each other with nothing beside them (64^3, 256 chunks: stats
// 10 -> 7 us and encode 18 -> 8 us with 4 instead of 32).
inline int enc_block_chunks(uint64_t chunks, int num_cus) {
    int ec = kEncBlockMax;
    while (ec > 4 && chunks < 8ull * (uint64_t)num_cus * (uint64_t)ec) ec /= 2;
    return ec;
}
// Sums over the encode blocks of a group: per block, and over every 2^shift
// of a field's blocks (its last ones, fewer than that, are not summed), so
// that a block finds what lies before it from at most 256 long sums and 63
// short ones, without a scan between the kernels.  The long sums are added to
// by atomics and start at zero (launch_plan clears them), each in a 128-byte
// line of its own: atomics on one line take 25 ns each, one after another
// (one counter per field had bounded the encode of 512^3, 4096 blocks, at
// 91 us; sums over 256 blocks cost 6 us at 100x500x500).  Those of field f of
// the group start at (boff[f] >> shift) + f, with a place to spare behind
// them.  Calls of more than 16384 blocks take sums over 256 blocks and scan
// them in place, a launch ahead of the kernels that read them, so that a block
// reads one of them and at most 255 short ones: added up by every block they
// cost the square of the size (1625^3 in chunks of 256, 2048 long sums:
// elision 3862 us, now 231, encode 6113, now 4315; in chunks of 1024 elision
// 215, now 68).  A launch takes 5 us (820^3, just above the line, elision 12
// us with 66 long sums added, now 17 of a call of 2200).
inline int enc_super_shift(uint64_t blocks) { return blocks <= 16384 ? 6 : 8; }
constexpr int kSuperLine = 32;   // words
struct EncSums {
    uint32_t* words;    // per block: Huffman words, outliers, non-zero words
    uint32_t* outs;
    uint32_t* nz;
    uint32_t* woff;     // per block: words of the field's earlier blocks
    uint32_t* sup;      // per 2^shift blocks: words, outliers
    uint32_t* supnz;    // per 2^shift blocks: non-zero words
    int shift;          // 6, or 8 with the long sums scanned
    __host__ __device__ bool scanned() const { return shift == 8; }
};
// A chunk's place, where its first part's bit offset (always 0) would be, so
// that a result's record costs no more than the offsets: units of kUnitChunks
// chunks (the decoder's), entry 0 of the unit's first two chunks the low and
// high half of the unit's first word, of the others the chunk's first word
// counted from there (the second chunk's follows from the first one's bits).
// A unit of one chunk has its high half past the field's last entry.
constexpr int kUnitChunks = 32;
static_assert(kUnitChunks * ((2048 * kLmax + 31) / 32) < 65536, "a unit's words count in 16 bits");
inline uint64_t sub_entries(uint64_t chunks) { return kSubParts * chunks + (chunks % kUnitChunks == 1 ? 1 : 0); }
// d_ccnt: per chunk its words, and its outliers above them (16 bits each)
hipError_t launch_huff_stats(const FieldDesc* d_fields, int nfields, const uint64_t* d_boff,
                             uint64_t nblocks, int chunk, int ec, uint32_t* d_ccnt, EncSums sums,
                             int max_nsym, hipStream_t st);
hipError_t launch_huff_encode(const FieldDesc* d_fields, int nfields, const uint64_t* d_boff,
                              uint64_t nblocks, int chunk, int ec, const uint32_t* d_ccnt, EncSums sums,
                              int max_nsym, hipStream_t st);
// Zero-word elision of the words that the encode left: into each field's
// esec (bitmap words, then the non-zero words; capacity (n_words + 31) / 32 +
// n_words) where that is shorter.
hipError_t launch_elide(const FieldDesc* d_fields, int nfields, const uint64_t* d_boff,
                        uint64_t nblocks, EncSums sums, hipStream_t st);
// The restore of an uploaded field's nw words from its elided section.
struct ElideField {
    uint32_t* words;
    uint32_t* sec;
    uint64_t nw;
};
// Restore tiles: 8192 words, or 2048 where there are few words (then four
// times the waves share them, each with one round of loads instead of four);
// the tile size only splits the work.
constexpr uint64_t kElideTileWords = 8192;
constexpr uint64_t kElideTileSmall = 2048;
inline uint64_t elide_tile_words(uint64_t words) {
    return words < (uint64_t)1024 * kElideTileSmall ? kElideTileSmall : kElideTileWords;
}
// Fields own the tiles [toff[f], toff[f + 1]) of tw words (a multiple of
// 2048); cnt and off (u32[ntiles], u64[ntiles + 1]) are scratch.
hipError_t launch_restore(const ElideField* d_e, int nf, const uint64_t* d_toff, uint64_t ntiles,
                          uint64_t tw, uint32_t* d_cnt, uint64_t* d_off, hipStream_t st);
// The kernel for the decode: eight lanes a chunk where every field has the
// encoder's offsets (kDecSplit), else one.
//
// With the offsets no prologue is launched: a result's plan holds its pass
// descriptors, and the decode scatters the outliers itself, a unit its share.
// Decode and prologue (an eighth as many workgroups as there are units)
// together, us, without / with it, by the share of outliers: 64^3 20 / 27 at
// 0.4 %, 21 / 33 at 1.7 %, 35 / 98 at 22 %; 256^3 40 / 50, 35 / 54, 55 / 171;
// 512^3 209 / 226, 220 / 249, 447 / 488; 64 fields of 64^3, one of them all
// outliers, 39 / 123.
//
// Without the offsets runs of symbols per look-up (kDecRuns) pay where the
// chip is not full of chains (a quarter of a decode block then has a CU of
// its own) and codes are short enough that several fit a look-up; their table
// costs about 10 us a call, which a chunk of 256 symbols wins back only with
// the shortest.  Plain against runs, us: 1024 symbols a chunk 91 / 43 at 1.05
// bits a symbol, 105 / 54 at 2.7, 120 / 88 at 4.8, 126 / 126 at 5.8; 512
// 50 / 30, 58 / 39, 67 / 57, 70 / 80; 256 30 / 26, 35 / 32, 39 / 45, 40 / 54.
enum DecodeKind { kDecSplit, kDecRuns, kDecPlain };
constexpr int kRunWaves = kDecBlockChunks / 64;
inline DecodeKind decode_kind(bool split, uint64_t nblocks, uint64_t words, uint64_t npts, int min_chunk,
                              int num_cus) {
    if (split) return kDecSplit;
    const uint64_t bits = min_chunk >= 512 ? 5 : 3;
    return kRunWaves * nblocks <= (uint64_t)num_cus && 32 * words <= bits * npts ? kDecRuns : kDecPlain;
}
// d_bsum: the word count of every decode block (launch_dec_prep), not read
// for kDecSplit
hipError_t launch_huff_decode(const FieldDesc* d_fields, int nfields, const uint64_t* d_dboff,
                              uint64_t nblocks, const uint32_t* d_bsum, int max_nsym, DecodeKind kind,
                              int num_cus, hipStream_t st);

// ---- the entry point that allocates nothing (noalloc.hip) ----
// Workspace of sz_decompress_noalloc: a static device array of this many
// bytes per GPU, holding the decoded quant-codes (2 bytes per point) and the
// call's descriptors; fields of up to kNoAllocMaxPoints points.
constexpr uint64_t kNoAllocMaxPoints = 1ull << 25;
constexpr uint64_t kNoAllocScratchBytes = 2 * kNoAllocMaxPoints + (1ull << 20);
// the device address of this GPU's workspace; called with device current
hipError_t noalloc_scratch(int device, void** ptr);
// up to kStageWordsMax u32 written to dst by a kernel that takes them as
// its argument
constexpr int kStageWordsMax = 896;
struct StageWords {
    uint32_t n;
    uint32_t w[kStageWordsMax];
};
hipError_t launch_stage_words(uint32_t* dst, const StageWords& a, hipStream_t st);

}  // namespace szi
