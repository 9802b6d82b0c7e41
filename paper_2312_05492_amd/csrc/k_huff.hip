// k_huff.hip -- chunked Huffman encode/decode with fused outlier compaction
// (Sec. VI-A) on gfx950.
//
// Encode: up to 32 consecutive chunks of one field per workgroup (4 wave64,
// one chunk per wave at a time, C/64 consecutive symbols per lane).
//   k_huff_stats   bit count and outlier count of every chunk; sums per
//                  workgroup block and per 64 blocks (large calls: per 256,
//                  scanned by k_scan_long)
//   k_huff_encode  chunk offsets = sums of the field's earlier blocks +
//                  in-block prefix; packs the codewords MSB-first through
//                  LDS and writes the outliers (index, original value) in
//                  ascending index order; sums of the non-zero words
//   k_elide        zero-word elision of the words, block by block
// Decode: kDecChunks chunks per decode block, kSubParts lanes per chunk from
// the bit offsets of its parts that the encoder records (one lane per chunk
// without them).
//   k_dec_prep     (k_plan.hip) ahead of the kernels without the offsets: word
//                  count of every decode block, outliers, pass descriptors
//   k_huff_decode8 (offsets at hand) persistent workgroups, eight lanes a
//                  chunk from its recorded first word and part offsets; it
//                  scatters the outliers for the replay
//   k_huff_decode1 (none) one lane a chunk; first words from the field's
//                  earlier block sums and an in-block scan
//   k_huff_decode_runs (none, few chunks of short codes) the same with up to
//                  four symbols a look-up
//                  All: a table-driven canonical decode from a two-word
//                  register window fed by a per-lane LDS word ring; whole
//                  lines stored at once
#include "dev_common.h"

namespace szi {

constexpr int kDecChunks = 256;
static_assert(kDecChunks == kDecBlockChunks,
              "the host sizes the decode grid with the same chunk count");

// The long sums of a field into what lies before each and, behind the last,
// their total: a workgroup a field.
template <int COLS>
__global__ __launch_bounds__(256) void k_scan_long(const uint64_t* __restrict__ boff, uint32_t* sup, int shift) {
    __shared__ uint32_t tot[4][COLS];
    const uint64_t b0 = boff[blockIdx.x];
    const uint32_t n = (uint32_t)((boff[blockIdx.x + 1] - b0) >> shift);
    SZI_G uint32_t* s = gp(sup) + ((b0 >> shift) + blockIdx.x) * kSuperLine;
    uint32_t before[COLS] = {};
    for (uint32_t i0 = 0; i0 <= n; i0 += 256) {
        const uint32_t i = i0 + threadIdx.x;
        uint32_t x[COLS], t[COLS];
#pragma unroll
        for (int c = 0; c < COLS; ++c) x[c] = wave_excl_scan(i < n ? s[(uint64_t)i * kSuperLine + c] : 0u, &t[c]);
        __syncthreads();
        if ((threadIdx.x & 63) == 0)
#pragma unroll
            for (int c = 0; c < COLS; ++c) tot[threadIdx.x >> 6][c] = t[c];
        __syncthreads();
#pragma unroll
        for (int c = 0; c < COLS; ++c) {
            uint32_t y = before[c] + x[c];
            for (uint32_t k = 0; k < 4; ++k) {
                if (k < threadIdx.x >> 6) y += tot[k][c];
                before[c] += tot[k][c];
            }
            if (i <= n) s[(uint64_t)i * kSuperLine + c] = y;
        }
    }
}

// Sum over the blocks [first, blk) of field f of one number a block or two
// (b, the second of a line of sup), by the 256 threads of a workgroup; red:
// 8 words of LDS, with a barrier inside.
__device__ __forceinline__ void sum_before(const uint32_t* __restrict__ a, const uint32_t* __restrict__ b,
                                           const uint32_t* __restrict__ sup, const EncSums& sums, int f,
                                           uint64_t first, uint64_t blk, uint32_t* red, uint32_t& ra,
                                           uint32_t& rb) {
    const int shift = sums.shift;
    const uint32_t nsup = (uint32_t)((blk - first) >> shift);
    const uint64_t sb0 = (first >> shift) + (uint32_t)f;
    uint32_t xa = 0, xb = 0;
    // scanned: the first thread reads the one behind them
    const uint32_t end = sums.scanned() ? nsup + 1u : nsup;
    for (uint32_t i = (sums.scanned() ? nsup : 0u) + threadIdx.x; i < end; i += 256) {
        xa += gp(sup)[(sb0 + i) * kSuperLine];
        if (b) xb += gp(sup)[(sb0 + i) * kSuperLine + 1];
    }
    const uint64_t i = first + ((uint64_t)nsup << shift) + threadIdx.x;   // fewer than 256 left
    if (i < blk) {
        xa += gp(a)[i];
        if (b) xb += gp(b)[i];
    }
    xa = wave_sum(xa);
    if (b) xb = wave_sum(xb);
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6] = xa;
        red[4 + (threadIdx.x >> 6)] = xb;
    }
    __syncthreads();
    ra = red[0] + red[1] + red[2] + red[3];
    rb = red[4] + red[5] + red[6] + red[7];
}
// the word of the long sum that block blk of field f, [first, end), belongs
// to, or -1 where the field ends before it is complete
__device__ __forceinline__ int64_t super_of(int shift, int f, uint64_t first, uint64_t end, uint64_t blk) {
    const uint64_t k = (blk - first) >> shift;
    return k < ((end - first) >> shift) ? (int64_t)(((first >> shift) + (uint32_t)f + k) * kSuperLine) : -1;
}

// symbols [s0, s0 + per) of the code array (all inside the field)
template <int PER>
__device__ __forceinline__ void load_syms(const SZI_G uint16_t* __restrict__ codes, uint64_t s0,
                                          uint32_t* sym) {
    if (PER >= 8) {
        const SZI_G vu4* p = reinterpret_cast<const SZI_G vu4*>(codes + s0);
#pragma unroll
        for (int k = 0; k < PER / 8; ++k) {
            const vu4 w = p[k];
            const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                sym[8 * k + 2 * j] = ww[j] & 0xFFFFu;
                sym[8 * k + 2 * j + 1] = ww[j] >> 16;
            }
        }
    } else {
        const vu2 w = *reinterpret_cast<const SZI_G vu2*>(codes + s0);
        sym[0] = w.x & 0xFFFFu;
        sym[1] = w.x >> 16;
        sym[2] = w.y & 0xFFFFu;
        sym[3] = w.y >> 16;
    }
}

template <int PER>
__device__ __forceinline__ void lane_syms(const FieldDesc& fd, uint64_t ch, int lane,
                                          uint32_t* sym, int& nsym_lane) {
    const uint64_t s0 = ch * (uint64_t)(PER * 64) + (uint64_t)lane * PER;
    if (s0 + PER <= fd.npts) {
        load_syms<PER>(gp(fd.codes), s0, sym);
        nsym_lane = PER;
    } else {
        nsym_lane = s0 < fd.npts ? (int)(fd.npts - s0) : 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) sym[k] = k < nsym_lane ? gp(fd.codes)[s0 + k] : 0u;
    }
}

template <int PER>
__global__ __launch_bounds__(256) void k_huff_stats(const FieldDesc* __restrict__ F, int nfields,
                                                    const uint64_t* __restrict__ boff, int ec,
                                                    uint32_t* ccnt, EncSums sums) {
    // the last blocks first: the codes written last may still lie in the
    // memory-side cache, and the encode then starts on those read last here
    // (512^3: 58 -> 56 us, encode 95 -> 91)
    const uint32_t blk = gridDim.x - 1u - blockIdx.x;
    extern __shared__ uint32_t cb[];
    __shared__ uint32_t sw[kEncBlockMax], so[kEncBlockMax];
    const int f = block_field(boff, nfields, blk);
    const FieldDesc& fd = F[f];
    const int nsym = 2 * fd.R;
    // per symbol its length, with 2^16 added for an outlier (code 0): the sum
    // over a chunk then holds its bits (< 2^16) and outliers (<= 2048)
    for (int s = threadIdx.x; s < nsym; s += blockDim.x)
        cb[s] = (gp(fd.cbook)[s] & 31u) + (s == 0 ? 0x10000u : 0u);
    __syncthreads();
    const uint64_t first = (blk - boff[f]) * (uint32_t)ec;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int j = wave; j < ec; j += 4) {
        const uint64_t ch = first + j;
        uint32_t words = 0, zeros = 0;
        if (ch < fd.nchunks) {   // uniform across the wave
            static_assert(PER * 64 * kLmax < 65536, "chunk bits fit 16 bits");
            uint32_t sym[PER];
            uint32_t bz = 0;
            if ((ch + 1) * (uint64_t)(PER * 64) <= fd.npts) {
                load_syms<PER>(gp(fd.codes), ch * (uint64_t)(PER * 64) + (uint64_t)lane * PER, sym);
#pragma unroll
                for (int k = 0; k < PER; ++k) bz += cb[sym[k]];
            } else {   // the field's last chunk
                int ns;
                lane_syms<PER>(fd, ch, lane, sym, ns);
#pragma unroll
                for (int k = 0; k < PER; ++k) bz += k < ns ? cb[sym[k]] : 0u;
            }
            bz = wave_sum(bz);
            const uint32_t bits = bz & 0xFFFFu;
            zeros = bz >> 16;
            words = (bits + 31) >> 5;
            if (lane == 0) {
                gp(fd.chunk_bits)[ch] = (uint16_t)bits;
                ccnt[fd.chunk_base + ch] = words | zeros << 16;
            }
        }
        if (lane == 0) {
            sw[j] = words;
            so[j] = zeros;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t a = 0, b = 0;
        for (int j = 0; j < ec; ++j) {
            a += sw[j];
            b += so[j];
        }
        sums.words[blk] = a;
        sums.outs[blk] = b;
        const int64_t sb = super_of(sums.shift, f, boff[f], boff[f + 1], blk);
        if (sb >= 0)   // words and outliers in one 64-bit addition (neither sum reaches 2^32)
            __hip_atomic_fetch_add(reinterpret_cast<SZI_G unsigned long long*>(gp(sums.sup) + sb),
                                   (unsigned long long)a | (unsigned long long)b << 32, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Exclusive scan of a u32 array of length n into u64 offsets (the upload's
// tile counts); one workgroup of 1024 threads, a contiguous run per thread:
// run sums, wave scans, the 16 wave totals through LDS (one barrier), then
// the run's offsets.  off[n] receives the total.  LONG = false takes runs of
// at most kRun (n <= 16384) in registers; LONG = true, longer runs kRun
// elements a round (the launcher chooses by n).
template <bool LONG>
__global__ __launch_bounds__(1024) void k_scan_blocks(const uint32_t* __restrict__ a, uint64_t n,
                                                      uint64_t* aoff) {
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const uint64_t per = (n + 1023) / 1024;
    const uint64_t beg = (uint64_t)t * per < n ? (uint64_t)t * per : n;
    const uint64_t end = beg + per < n ? beg + per : n;
    // runs of up to kRun elements sit in registers, all loads issued at once
    constexpr int kRun = 16;
    const bool regs = !LONG && per <= (uint64_t)kRun;   // LONG: runs of more than kRun
    uint32_t va[kRun];
    uint64_t sa = 0;
    if (regs) {
#pragma unroll
        for (int k = 0; k < kRun; ++k) {
            const uint64_t i = beg + k;
            va[k] = i < end ? a[i] : 0u;
        }
#pragma unroll
        for (int k = 0; k < kRun; ++k) sa += va[k];
    } else if (LONG) {
        for (uint64_t i0 = beg; i0 < end; i0 += kRun) {
#pragma unroll
            for (int k = 0; k < kRun; ++k) {
                const uint64_t i = i0 + k;
                va[k] = i < end ? a[i] : 0u;
            }
#pragma unroll
            for (int k = 0; k < kRun; ++k) sa += va[k];
        }
    }
    uint64_t xa = sa;   // inclusive scan over the wave's lanes
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t ya = __shfl_up(xa, o);
        if (lane >= o) xa += ya;
    }
    __shared__ uint64_t wa[16];
    if (lane == 63) wa[wave] = xa;
    __syncthreads();
    for (int k = 0; k < wave; ++k) xa += wa[k];
    uint64_t ra = xa - sa;
    if (regs) {
#pragma unroll
        for (int k = 0; k < kRun; ++k) {
            const uint64_t i = beg + k;
            if (i < end) aoff[i] = ra;
            ra += va[k];
        }
    } else if (LONG) {
        for (uint64_t i0 = beg; i0 < end; i0 += kRun) {
#pragma unroll
            for (int k = 0; k < kRun; ++k) {
                const uint64_t i = i0 + k;
                va[k] = i < end ? a[i] : 0u;
            }
#pragma unroll
            for (int k = 0; k < kRun; ++k) {
                const uint64_t i = i0 + k;
                if (i < end) aoff[i] = ra;
                ra += va[k];
            }
        }
    }
    if (t == 1023) aoff[n] = xa;
}

// Orders the LDS accesses of one wave around this point (a wave's LDS
// instructions execute in issue order, so only the compiler needs holding).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// LDS words of one wave's chunk buffer: the longest chunk, one word for the
// low part of its last code (zero when that code ends in its first word),
// and one for the symbols past a chunk's end (a zero code at the chunk's
// last bit, whose two ORs of zeros then land one word further).
__host__ __device__ constexpr int enc_chunk_words(int chunk) { return (chunk * kLmax + 31) / 32 + 2; }

// One wave per chunk, PER consecutive symbols per lane: the wave scans the
// lanes' bit counts, ORs every code MSB first into the chunk's words in LDS
// and copies them out contiguously.  The waves of a workgroup share only
// the code book, so they synchronise among their own lanes.  (Packing a
// lane's codes in registers with plain stores for the words it owns, and
// loading the next chunk ahead, were both slower.)
template <int PER>
__global__ __launch_bounds__(256) void k_huff_encode(const FieldDesc* __restrict__ F, int nfields,
                                                     const uint64_t* __restrict__ boff, int ec,
                                                     const uint32_t* __restrict__ ccnt, EncSums sums) {
    extern __shared__ uint32_t smem[];
    __shared__ uint32_t wnz[4], red[8];
    constexpr int C = PER * 64;
    constexpr int MCW = enc_chunk_words(C);
    const int f = block_field(boff, nfields, blockIdx.x);
    const FieldDesc& fd = F[f];
    const int nsym = 2 * fd.R;
    uint32_t* cb = smem;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint32_t* wbuf = smem + nsym + wave * MCW;
    for (int s = threadIdx.x; s < nsym; s += blockDim.x) cb[s] = gp(fd.cbook)[s];
    const uint64_t blk_local = blockIdx.x - boff[f];
    const uint64_t first = blk_local * (uint32_t)ec;
    // in-block exclusive prefix of the chunk word and outlier counts
    uint32_t cc = 0;
    if (lane < ec && first + lane < fd.nchunks) cc = ccnt[fd.chunk_base + first + lane];
    // words of the unit's earlier blocks
    const uint32_t inu = (uint32_t)(first % kUnitChunks) / (uint32_t)ec;
    uint32_t rel0 = (uint32_t)lane < inu ? gp(sums.words)[blockIdx.x - inu + lane] : 0u;
    uint32_t tw, to;
    const uint32_t pw = wave_excl_scan(cc & 0xFFFFu, &tw);
    const uint32_t po = wave_excl_scan(cc >> 16, &to);
    if (inu) rel0 = wave_sum(rel0);   // uniform
    // words and outliers of the field's earlier blocks; the barrier inside
    // also completes the code book in LDS
    uint32_t bw0, bo0;
    sum_before(sums.words, sums.outs, sums.sup, sums, f, boff[f], blockIdx.x, red, bw0, bo0);
    if (threadIdx.x == 0) sums.woff[blockIdx.x] = bw0;
    uint32_t nz = 0;   // non-zero words written, for the zero-word elision of the blob
    for (int j = wave; j < ec; j += 4) {
        const uint64_t ch = first + j;
        if (ch >= fd.nchunks) break;   // uniform across the wave
        uint32_t sym[PER], e[PER];
        int ns = PER;
        if ((ch + 1) * (uint64_t)C <= fd.npts) {   // uniform
            load_syms<PER>(gp(fd.codes), ch * (uint64_t)C + (uint64_t)lane * PER, sym);
#pragma unroll
            for (int k = 0; k < PER; ++k) e[k] = cb[sym[k]];
        } else {   // the field's last chunk: no bits past its end
            lane_syms<PER>(fd, ch, lane, sym, ns);
#pragma unroll
            for (int k = 0; k < PER; ++k) e[k] = k < ns ? cb[sym[k]] : 0u;
        }
        // bits (< 2^16 per chunk) in the low half, outliers in the high half
        // (looked for only where some lane holds one): one scan gives both
        // offsets
        static_assert(PER * 64 * kLmax < 65536, "chunk bits fit 16 bits");
        uint32_t bz = 0, least = sym[0];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            bz += e[k] & 31u;
            least = sym[k] < least ? sym[k] : least;
        }
        uint32_t om = 0u;   // the lane's outliers, a bit a symbol
        if (wave_any(least == 0u)) {
#pragma unroll
            for (int k = 0; k < PER; ++k) om |= (k < ns && sym[k] == 0u) ? 1u << k : 0u;
            bz += (uint32_t)__popc(om) << 16;
        }
        uint32_t tbz;
        const uint32_t pbz = wave_excl_scan(bz, &tbz);
        const uint32_t pos = pbz & 0xFFFFu, tb = tbz & 0xFFFFu;
        const uint32_t nw = (tb + 31) >> 5;
        for (uint32_t k = lane; k < nw; k += 64) wbuf[k] = 0;
        wave_lds_sync();
        {
            // every symbol ORs both words its code may touch, without
            // branches: the second takes the code's low part, zero when the
            // code ends in the first; a symbol past the chunk's end has the
            // zero entry (length 0, no bits) and ORs zeros.  The entry holds
            // the code from its top bit on, so each word is one shift by the
            // bit position (taken mod 32): ten vector instructions a symbol
            // where a 64-bit shift to the place took eighteen's time.
            uint32_t p = pos;
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const uint32_t c = e[k] & ~31u;
                uint32_t* w = wbuf + (p >> 5);
                atomicOr(w, c >> (p & 31u));
                atomicOr(w + 1, __builtin_amdgcn_alignbit(c, 0u, p));
                p += e[k] & 31u;
            }
        }
        wave_lds_sync();
        const uint64_t ow = (uint64_t)bw0 + (uint32_t)__builtin_amdgcn_readlane((int)pw, j);   // j is uniform
        for (uint32_t k = lane; k < nw; k += 64) {
            const uint32_t w = wbuf[k];
            nz += w != 0u;
            if (ow + k < fd.words_cap) gp(fd.words)[ow + k] = w;
        }
        if (fd.sub) {
            // the chunk's place and the decoder's starting bits of its 2nd ..
            // last eighth (symbol 8 k PER starts lane 8 k), as one 16-byte store
            static_assert(kSubParts == 8, "eight parts: lanes 8, 16, .., 56");
            uint32_t b[8];
            const uint32_t uw = bw0 - rel0;   // the unit's first word
            const uint32_t at = (uint32_t)ch % kUnitChunks;
            b[0] = at == 0u ? uw & 0xFFFFu : (at == 1u ? uw >> 16 : (uint32_t)ow - uw);
#pragma unroll
            for (int k = 1; k < 8; ++k) b[k] = (uint32_t)__builtin_amdgcn_readlane((int)pos, 8 * k);
            if (lane == 0) {
                *reinterpret_cast<SZI_G vu4*>(gp(fd.sub) + (uint64_t)kSubParts * ch) =
                    vu4{b[0] | (b[1] << 16), b[2] | (b[3] << 16), b[4] | (b[5] << 16), b[6] | (b[7] << 16)};
                if (at == 0u && ch + 1 == fd.nchunks)   // a unit of one chunk
                    gp(fd.sub)[(uint64_t)kSubParts * (ch + 1)] = (uint16_t)(uw >> 16);
            }
        }
        wave_lds_sync();
        if (tbz >> 16) {   // uniform: outliers in this chunk
            // their places are gathered where the words were, so that the
            // lanes take them in turn and loads and stores are coalesced (a
            // load and two stores a symbol, the lanes 64 bytes apart, ran the
            // L1 over: 256^3 with 64 % outliers 221 us, now 49; 512^3 with 1.7 %
            // 220, now 116, and 86, now 82, with next to none)
            uint16_t* list = reinterpret_cast<uint16_t*>(wbuf);
            static_assert(2 * C <= 4 * MCW, "a place a symbol");
            for (uint32_t zo = pbz >> 16; om != 0u; ++zo, om &= om - 1u)
                list[zo] = (uint16_t)(lane * PER + __builtin_ctz(om));
            wave_lds_sync();
            const uint64_t oo = (uint64_t)bo0 + (uint32_t)__builtin_amdgcn_readlane((int)po, j);
            const uint32_t s0 = (uint32_t)ch * (uint32_t)C;   // a field has fewer than 2^32 points
            // the histogram sized the list
            const uint64_t room = oo < fd.n_outliers ? fd.n_outliers - oo : 0u;
            const uint32_t no = room < (tbz >> 16) ? (uint32_t)room : tbz >> 16;
            const SZI_G float* in = gp(fd.in) + s0;
            SZI_G uint32_t* oi = gp(fd.outlier_idx) + oo;
            SZI_G float* ov = gp(fd.outlier_val) + oo;
#pragma unroll 4
            for (uint32_t i = lane; i < no; i += 64) {
                const uint32_t at = list[i];
                oi[i] = s0 + at;
                ov[i] = in[at];
            }
            wave_lds_sync();
        }
    }
    // one count per block, and one atomic for the long sum it belongs to
    nz = wave_sum(nz);
    if (lane == 0) wnz[wave] = nz;
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t t = wnz[0] + wnz[1] + wnz[2] + wnz[3];
        sums.nz[blockIdx.x] = t;
        const int64_t sb = super_of(sums.shift, f, boff[f], boff[f + 1], blockIdx.x);
        if (sb >= 0) gatomic_add(gp(sums.supnz) + sb, t);
    }
}

// One lane decodes one chunk: canonical decode with a 2^kLutBits table of
// u16 entries for short codes; a longer code's length comes from comparing
// the next bits with the per-length limits, without a loop or a
// data-dependent branch.  The next bits are a 32-bit window taken with one
// funnel shift from two words held in registers, w0:w1, at bit o of w0
// (1 <= o <= 32, so w1 is always whole and the window always has 32 valid
// bits; a lookup needs at most kLmax = 24).  When o passes 32 the words move
// up by one, w1 taking the next word, which every step has already read from
// the lane's ring, off the critical path of the table lookups.  The ring is
// 32 words per lane in LDS: once per group of 8 symbols every lane requests
// its next 8 words from global memory (two 16-byte loads, if the ring has
// room) and commits them to the ring one group later, so global loads sit at
// fixed points and their latency is covered by a group of decoding.  A group
// consumes at most 6 words and the ring always holds at least 7 ahead of the
// window.  Symbols leave 64 at a time per lane in eight back-to-back 16-byte
// stores.
//
// With Q = kSubParts (8) lanes per chunk, each lane decodes an eighth of
// the chunk's symbols from the word and bit that the encoder recorded for it
// (fd.sub: the chunk's place and the eighths' bit offsets, kept with a
// compressed result): eight times the independent
// chains, each an eighth as long (against four lanes a chunk, 1 % faster at
// rel 1e-3, 5 % at 1e-4 and 38 % on a 64^3 field), and no sums over the
// field's earlier words ahead of them.  A workgroup then covers an eighth of
// a decode block (kDecChunks chunks).  A field without offsets (an uploaded
// blob) is decoded by one lane a chunk, which finds its words from the word
// counts that the prologue summed.
//
// Where the time of eight lanes a chunk went at 512^3, rel 1e-3 (164 us, one
// workgroup per eighth of a decode block; timed with parts of the kernel left
// out): 61 us ahead of the first symbol (table, sums, offsets, words, one
// after another), 34 us for stores of 64 different lines an instruction, the
// rest the symbols.  So the eight lanes of a chunk exchange their 16-byte
// pieces, after which each store instruction writes eight whole lines, and
// the kernel is persistent: a workgroup fills its table once and its waves
// go through their chunks on their own, a chunk's offsets requested two ahead
// and its first words one ahead (142 us).
constexpr int kRing = 32;   // ring words per lane (power of 2)
// The table of the codes longer than the look-up table, where the length of
// the chain counts: 1024 entries over their part of the code space, so that a
// step where any lane of the wave holds one mostly takes one look-up more in
// place of ten compares and two look-ups (78 -> 69 us on a 100x150x200 field;
// in the eight-lane kernel 140.5 -> 139.4 us at 512^3 and 20.5 -> 21.7 on a
// 64^3 field, whose table costs more than it saves: not used there).  Nor
// where that part is so large (1/64 of the code space) that an entry would
// resolve few of the codes.
constexpr int kMidBits = 10;
constexpr uint32_t kMidShift = 8;

// Exchange among the eight lanes c, c + 8, .., c + 56 of a wave (all lanes
// active): lane c + 8 q's piece j becomes lane c + 8 j's piece q.
__device__ __forceinline__ void exchange8(vu4 (&p)[8]) {
#pragma unroll
    for (int d = 0; d < 4; ++d) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {   // lane bit 5 with piece bit 2
            const auto r = __builtin_amdgcn_permlane32_swap(p[i][d], p[i + 4][d], false, false);
            p[i][d] = r[0];
            p[i + 4][d] = r[1];
        }
#pragma unroll
        for (int i = 0; i < 6; ++i) {   // lane bit 4 with piece bit 1
            if (i & 2) continue;
            const auto r = __builtin_amdgcn_permlane16_swap(p[i][d], p[i + 2][d], false, false);
            p[i][d] = r[0];
            p[i + 2][d] = r[1];
        }
#pragma unroll
        for (int i = 0; i < 8; i += 2) {   // lane bit 3 with piece bit 0: rows rotated by 8, half of each kept
            constexpr int kRowRor8 = 0x128;
            const int a = (int)p[i][d], b = (int)p[i + 1][d];
            p[i][d] = (uint32_t)__builtin_amdgcn_update_dpp(a, b, kRowRor8, 0xF, 0xC, false);
            p[i + 1][d] = (uint32_t)__builtin_amdgcn_update_dpp(b, a, kRowRor8, 0xF, 0x3, false);
        }
    }
}

// The tables of a field in LDS: the look-up table at a fixed address (a
// look-up's address is then its index and an offset, with no base to add),
// the limits, bases and sorted symbols, sized by the radius, after it.
__device__ __forceinline__ void fill_tables(const FieldDesc& fd, uint32_t* lut32, uint32_t* tab_hi) {
    // the look-up table 16 bytes at a time, its four loads per lane in
    // flight together (word by word where the tables do not start on 16
    // bytes: odd radius), then the rest word by word
    const int tid = threadIdx.x, ntab = dtab_words(2 * fd.R);
    const SZI_G uint32_t* src = gp(fd.dtab);
    static_assert(kDtLimit % (4 * kDecChunks) == 0, "whole rounds of 16-byte copies");
    if (((uintptr_t)fd.dtab & 15u) == 0u) {
        const SZI_G vu4* s4 = reinterpret_cast<const SZI_G vu4*>(src);
        vu4* d4 = reinterpret_cast<vu4*>(lut32);
        vu4 v[kDtLimit / (4 * kDecChunks)];
#pragma unroll
        for (int j = 0; j < kDtLimit / (4 * kDecChunks); ++j) v[j] = s4[tid + j * kDecChunks];
#pragma unroll
        for (int j = 0; j < kDtLimit / (4 * kDecChunks); ++j) d4[tid + j * kDecChunks] = v[j];
    } else {
        for (int k = tid; k < kDtLimit; k += kDecChunks) lut32[k] = src[k];
    }
    for (int k = kDtLimit + tid; k < ntab; k += kDecChunks) tab_hi[k - kDtLimit] = src[k];
}

// Where a lane's symbols start in its field's words, and how far it may read.
struct LaneWords {
    const SZI_G uint32_t* words;   // from the 4-aligned word at or below the lane's first
    uint32_t first;                // the lane's first word, counted from there
    uint32_t b0;                   // and bit in it
    uint32_t cap;                  // words to request (0: none)
};
// wfirst: the chunk's first word; bits [bo, be0) of the chunk's cbits are
// the lane's.  Requests stop after the word that holds the lane's last bit
// (the ring may then hold stale words past it, which only fill a look-up's
// unused low bits) and never pass the field's words (the array has kWordPad
// words of slack, so the 8-word loads of the last request stay inside it).
// Stopping at the lane's own end saves a twentieth of decode time.
__device__ __forceinline__ LaneWords lane_words(const FieldDesc& fd, bool any, uint64_t wfirst, uint32_t bo,
                                                uint32_t be0, uint32_t cbits) {
    const uint64_t w0abs = wfirst + (bo >> 5);
    const uint64_t wbase = w0abs & ~(uint64_t)3;
    const uint32_t be = be0 < bo || be0 > cbits ? cbits : be0;   // a corrupt offset: the chunk's end
    const uint64_t wlim0 = wfirst + ((be + 31u) >> 5);
    const uint64_t wlim = wlim0 < fd.words_cap ? wlim0 : fd.words_cap;
    const uint64_t wleft = any && wlim > wbase ? wlim - wbase : 0;
    return LaneWords{gp((const uint32_t*)fd.words) + wbase, (uint32_t)(w0abs - wbase), bo & 31u,
                     wleft < (1u << 30) ? (uint32_t)wleft : (1u << 30)};
}
// the first 16 words of a lane
__device__ __forceinline__ void first_words(const LaneWords& l, vu4 (&w)[4]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = vu4{0u, 0u, 0u, 0u};
    if (l.cap > 0) {
        w[0] = *reinterpret_cast<const SZI_G vu4*>(l.words);
        w[1] = *reinterpret_cast<const SZI_G vu4*>(l.words + 4);
    }
    if (l.cap > 8) {
        w[2] = *reinterpret_cast<const SZI_G vu4*>(l.words + 8);
        w[3] = *reinterpret_cast<const SZI_G vu4*>(l.words + 12);
    }
}

// A lane's decoder.
constexpr uint32_t kLenMask = ~0u << 27;   // a u16 table entry's length, the entry in the high half
static_assert(kLutSymBits == 11 && kLmax < 32, "lengths in the top five bits");
struct LaneDec {
    const uint16_t* lut;
    const uint32_t* tab_hi;
    uint32_t* ring;      // the lane's ring: word i at ring[(i + rot) % kRing], rotated by 16-byte groups
    uint32_t rot;        // per lane so that lanes at the same position hit different banks
    uint32_t nsym;
    // scalar registers: the limits of the codes longer than the table, the
    // first of them (left-justified to kLmax bits) and their table's shift
    uint32_t lim[kLmax - kLutBits - 1];
    uint32_t long0, sh;
    const uint16_t* mid;   // used by some() only
    LaneWords l;
    uint32_t wr, rd;     // next word to request, next word to read from the ring (rot added)
    uint32_t w0, w1, nxw;   // the window's words, and the one the next move takes
    uint32_t left;       // 32 - o in the top five bits, o the window's first bit of w0:w1 (1 <= o <= 32)
    bool pend;           // words [pat, pat + 8) requested, in la and lb
    uint32_t pat;
    vu4 la, lb;

    __device__ __forceinline__ void tables(const FieldDesc& fd) {
        nsym = 2u * (uint32_t)fd.R;
#pragma unroll
        for (int k = kLutBits + 1; k < kLmax; ++k)
            lim[k - kLutBits - 1] = __builtin_amdgcn_readfirstlane(gp(fd.dtab)[kDtLimit + k]);
    }
    // The table of long codes, by the workgroup once fill_tables' are
    // visible: entry j for the codes at long0 + (j << sh), all of one length
    // and symbol where that length is at most kLmax - sh (they start at
    // multiples of their span, long0 at one of them all); length - kLutBits
    // above the symbol, 0: look further.
    __device__ __forceinline__ void fill_mid(const FieldDesc& fd, uint16_t* m) {
        mid = m;
        long0 = __builtin_amdgcn_readfirstlane(gp(fd.dtab)[kDtLimit + kLutBits]);
        const uint32_t span = (1u << kLmax) - long0;   // of the long codes
        const int bits = span > 1u ? 32 - __builtin_clz(span - 1u) : 0;
        sh = bits > kMidBits ? (uint32_t)(bits - kMidBits) : 0u;
        if (sh > kMidShift) return;
        for (uint32_t j = threadIdx.x; j < 1u << kMidBits; j += kDecChunks) {
            const uint32_t c = long0 + (j << sh);
            uint32_t e = 0u;
            if (c < 1u << kLmax) {
                uint32_t ln, sl;
                long_code(c << (32 - kLmax), ln, sl);
                if (ln <= (uint32_t)kLmax - sh) e = ((ln - (uint32_t)kLutBits) << kLutSymBits) | sl;
            }
            m[j] = (uint16_t)e;
        }
    }
    __device__ __forceinline__ uint32_t slot(uint32_t i) const { return i & (uint32_t)(kRing - 1); }   // rot added
    __device__ __forceinline__ void put(uint32_t at, vu4 a, vu4 b) {   // words [at, at + 8) into the ring
        *reinterpret_cast<vu4*>(ring + slot(at + rot)) = a;
        *reinterpret_cast<vu4*>(ring + slot(at + rot + 4u)) = b;
    }
    // starts on a lane's words: 16 into the ring, the window at bit b0 of
    // the first: the top of w1 (o = 32) or bit b0 of w0
    __device__ __forceinline__ void start(const LaneWords& lw, const vu4 (&w)[4]) {
        l = lw;
        put(0u, w[0], w[1]);
        put(8u, w[2], w[3]);
        wr = 16;
        rd = l.first + rot;
        w0 = 0u;
        if (l.b0 == 0u) {
            w1 = ring[slot(rd)];
            ++rd;
            left = 0u;
        } else {
            w0 = ring[slot(rd)];
            w1 = ring[slot(rd + 1u)];
            rd += 2;
            left = (32u - l.b0) << 27;
        }
        nxw = ring[slot(rd)];
        pend = false;
        pat = 0;
        la = lb = vu4{0u, 0u, 0u, 0u};
    }
    // a code longer than the table at the top of x: the length is one more
    // than the number of length limits at or below the next kLmax bits
    // (canonical codes grow with their length), then one look-up
    __device__ __forceinline__ void long_code(uint32_t x, uint32_t& ln, uint32_t& sl) const {
        const uint32_t w = x >> (32 - kLmax);
        ln = kLutBits + 1;
#pragma unroll
        for (int k = kLutBits + 1; k < kLmax; ++k) ln += w >= lim[k - kLutBits - 1] ? 1u : 0u;
        const uint32_t i = tab_hi[kDtBase - kDtLimit + ln] + (w >> (kLmax - ln));
        sl = tab_hi[kDtSorted - kDtLimit + (i < nsym ? i : 0u)];   // a corrupt stream stays inside
    }
    // the same for the lanes with lng, by the table of long codes first
    __device__ __forceinline__ void long_lookup(uint32_t x, bool lng, uint32_t& ln, uint32_t& sl) const {
        bool more = true;
        if (sh <= kMidShift) {
            const uint32_t e = mid[(((x >> (32 - kLmax)) - long0) >> sh) & ((1u << kMidBits) - 1u)];
            ln = (e >> kLutSymBits) + (uint32_t)kLutBits;
            sl = e & ((1u << kLutSymBits) - 1u);
            more = wave_any(lng && e < 1u << kLutSymBits);
        }
        if (more) long_code(x, ln, sl);
    }
    // up to four symbols from a table of runs (see k_huff_decode_runs), two a
    // word; returns their number
    __device__ __forceinline__ int some(const vu2* runs, vu2& sy) {
        const uint32_t x = __builtin_amdgcn_alignbit(w0, w1, left >> 27);
        const vu2 e = runs[x >> (32 - kLutBits)];
        constexpr uint32_t kSyms = ((1u << kLutSymBits) - 1u) * 0x10001u;
        uint32_t lo = e.x & kSyms, n = e.y >> (16 + kLutSymBits);
        uint32_t len = (e.x << 16) & kLenMask;
        if (wave_any(len == 0)) {
            const bool lng = len == 0;
            uint32_t ln, sl;
            long_lookup(x, lng, ln, sl);
            lo = lng ? sl : lo;
            n = lng ? 1u : n;
            len = lng ? ln << 27 : len;
        }
        move(len);
        sy = vu2{lo, e.y & kSyms};
        return (int)n;
    }
    __device__ __forceinline__ uint32_t one() {
        // bits [o, o + 32) of w0:w1 (the shift amount is 32 - o, taken mod 32)
        const uint32_t x = __builtin_amdgcn_alignbit(w0, w1, left >> 27);
        const uint32_t e = lut[x >> (32 - kLutBits)];
        // (one shift to the top for either kind of code: shifted each by
        // itself, an upload of long codes in chunks of 2048 took 418 us for 408)
        uint32_t len = e >> kLutSymBits, sym = e & ((1u << kLutSymBits) - 1u);
        if (wave_any(len == 0)) {
            uint32_t ln, sl;
            long_code(x, ln, sl);
            const bool lng = len == 0;
            sym = lng ? sl : sym;
            len = lng ? ln : len;
        }
        move(len << 27);
        return sym;
    }
    // len: a code's length in the top five bits.  Past the end of w0 the
    // words move up by one (length <= kLmax < 32): the subtraction's borrow
    // is the test, and nothing is brought back into range (with a signed bit
    // position, a compare and a correction, and the ring permuted by xor, the
    // decode took 129 us in place of 123 on the 24 x 1800x3600 batch, 141 in
    // place of 139 at 512^3).
    __device__ __forceinline__ void move(uint32_t len) {
        const bool t = left < len;
        left -= len;
        w0 = t ? w1 : w0;
        w1 = t ? nxw : w1;
        rd += t ? 1u : 0u;
        nxw = ring[slot(rd)];
    }
    // ahead of a group of up to 8 symbols: commit the previous request,
    // maybe request 8 more words
    __device__ __forceinline__ void refill() {
        if (pend) put(pat, la, lb);
        // the ring holds [rd, wr) and a request adds 8; the prefetched word
        // at rd is not overwritten because the ring keeps kRing - 8 >= 7
        pend = wr < l.cap && wr + rot + 8 - rd <= (uint32_t)kRing;
        if (pend) {
            pat = wr;
            la = *reinterpret_cast<const SZI_G vu4*>(l.words + wr);
            lb = *reinterpret_cast<const SZI_G vu4*>(l.words + wr + 4);
            wr += 8;
        }
    }
    __device__ __forceinline__ uint32_t two() {
        const uint32_t lo = one(), hi = one();
        return lo | (hi << 16);
    }
    __device__ __forceinline__ vu4 group8() {
        refill();
        vu4 pk;
        pk.x = two();
        pk.y = two();
        pk.z = two();
        pk.w = two();
        return pk;
    }
    // symbols [k, cnt) one store each
    __device__ __forceinline__ void tail(SZI_G uint16_t* out, int k, int cnt) {
#pragma unroll 1
        while (k < cnt) {
            refill();
            const int e = k + 8 < cnt ? k + 8 : cnt;
#pragma unroll 1
            for (; k < e; ++k) out[k] = (uint16_t)one();
        }
    }
};

// The first word of the chunk of thread tid of decode block blk of a field
// whose blocks start at first: the words of the field's earlier blocks (the
// sum of their word counts) and the block's exclusive scan of its chunks'
// word counts.  scan, pre: LDS, with a barrier inside.
__device__ __forceinline__ uint64_t first_word(uint32_t cbits, const uint32_t* __restrict__ bsum, uint64_t first,
                                               uint64_t blk, uint32_t* scan, uint64_t* pre) {
    const int tid = threadIdx.x;
    uint64_t pb = 0;
    for (uint64_t i = first + (uint64_t)tid; i < blk; i += kDecChunks) pb += bsum[i];
    for (int o = 32; o > 0; o >>= 1) pb += __shfl_xor(pb, o);
    uint32_t tot;
    const uint32_t wx = wave_excl_scan((cbits + 31) >> 5, &tot);
    if ((tid & 63) == 0) {
        scan[tid >> 6] = tot;
        pre[tid >> 6] = pb;
    }
    __syncthreads();
    uint64_t wfirst = wx;
    for (int k = 0; k < kDecChunks / 64; ++k) wfirst += pre[k];
    for (int k = 0; k < (tid >> 6); ++k) wfirst += scan[k];
    return wfirst;
}

// One lane a chunk, kDecChunks chunks a workgroup.
__global__ __launch_bounds__(kDecChunks) void k_huff_decode1(const FieldDesc* __restrict__ F, int nfields,
                                                             const uint64_t* __restrict__ boff,
                                                             const uint32_t* __restrict__ bsum) {
    __shared__ __align__(16) uint32_t rings[kDecChunks * kRing];
    __shared__ __align__(16) uint32_t lut32[kDtLimit];   // 2^kLutBits u16 entries
    __shared__ uint32_t scan[kDecChunks / 64];
    __shared__ uint64_t pre[kDecChunks / 64];
    extern __shared__ uint32_t tab_hi[];   // decode-table words kDtLimit .. dtab_words(nsym)
    const uint64_t pblk = blockIdx.x;
    const int f = block_field(boff, nfields, pblk);
    const FieldDesc& fd = F[f];
    const int tid = threadIdx.x;
    fill_tables(fd, lut32, tab_hi);
    LaneDec dec;
    dec.lut = reinterpret_cast<const uint16_t*>(lut32);
    dec.tab_hi = tab_hi;
    dec.ring = rings + tid * kRing;
    dec.rot = ((uint32_t)tid & (kRing / 4 - 1)) << 2;
    dec.tables(fd);
    const uint64_t ch = (pblk - boff[f]) * kDecChunks + (uint32_t)tid;
    const uint32_t cbits = ch < fd.nchunks ? (uint32_t)gp(fd.chunk_bits)[ch] : 0u;
    const uint64_t wfirst = first_word(cbits, bsum, boff[f], pblk, scan, pre);
    const uint64_t s0 = ch * (uint64_t)fd.chunk;
    const int cnt = s0 >= fd.npts ? 0 : (s0 + fd.chunk <= fd.npts ? fd.chunk : (int)(fd.npts - s0));
    if (cnt == 0) return;
    const LaneWords lw = lane_words(fd, true, wfirst, 0u, cbits, cbits);
    vu4 w[4];
    first_words(lw, w);
    dec.start(lw, w);
    SZI_G uint16_t* out = gp(fd.codes) + s0;
    int k = 0;
    // 64 symbols of a lane leave as eight back-to-back 16-byte stores, so
    // that a lane writes a whole 128-byte cache line at once (half lines
    // written far apart in time cost 15 % more decode time)
    if (((uintptr_t)fd.codes & 15u) == 0u) {   // s0 and k are multiples of 8
#pragma unroll 1
        for (; k + 64 <= cnt; k += 64) {
            vu4 p[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) p[j] = dec.group8();
            SZI_G vu4* o = reinterpret_cast<SZI_G vu4*>(out + k);
#pragma unroll
            for (int j = 0; j < 8; ++j) o[j] = p[j];
        }
    }
    dec.tail(out, k, cnt);
}

// One lane a chunk where the call has too few chunks to fill the chip, so
// that only the length of a lane's chain counts (about 0.1 us a step; spread
// over four times the CUs, one wave each, the plain kernel took 116 us in
// place of 117 on a 100x150x200 field): a look-up gives up to four
// symbols, from a table of runs that the workgroup makes out of the field's
// (u64 entries: four symbols of 16 bits, the run's length in bits above the
// first, its symbols' number above the last; 0 where the first code is longer
// than the table).  A workgroup is a quarter of a decode block, one wave of
// lanes (its scattered stores, a line each, then have a CU's memory pipe to
// themselves); the other three waves help with the table.
__global__ __launch_bounds__(kDecChunks) void k_huff_decode_runs(const FieldDesc* __restrict__ F, int nfields,
                                                                 const uint64_t* __restrict__ boff,
                                                                 const uint32_t* __restrict__ bsum) {
    __shared__ __align__(16) vu2 runs[1 << kLutBits];
    __shared__ __align__(16) uint32_t lut32[kDtLimit];   // 2^kLutBits u16 entries, then the rings
    __shared__ uint16_t mid[1 << kMidBits];
    __shared__ uint32_t scan[kDecChunks / 64];
    __shared__ uint64_t pre[kDecChunks / 64];
    extern __shared__ uint32_t tab_hi[];   // decode-table words kDtLimit .. dtab_words(nsym)
    static_assert(64 * kRing <= kDtLimit, "a wave's rings take the table's place");
    const uint64_t pblk = blockIdx.x / kRunWaves;
    const int part = (int)(blockIdx.x % kRunWaves);
    const int f = block_field(boff, nfields, pblk);
    const FieldDesc& fd = F[f];
    const int tid = threadIdx.x;
    fill_tables(fd, lut32, tab_hi);
    LaneDec dec;
    dec.lut = nullptr;
    dec.tab_hi = tab_hi;
    dec.ring = lut32 + (tid & 63) * kRing;
    dec.rot = ((uint32_t)tid & (kRing / 4 - 1)) << 2;
    dec.tables(fd);
    const uint64_t ch = (pblk - boff[f]) * kDecChunks + (uint32_t)tid;
    const uint32_t cbits = ch < fd.nchunks ? (uint32_t)gp(fd.chunk_bits)[ch] : 0u;
    const uint64_t wfirst = first_word(cbits, bsum, boff[f], pblk, scan, pre);
    const uint64_t s0 = ch * (uint64_t)fd.chunk;
    const bool mine = tid >> 6 == part && s0 < fd.npts;
    const int cnt = !mine ? 0 : (s0 + fd.chunk <= fd.npts ? fd.chunk : (int)(fd.npts - s0));
    const LaneWords lw = lane_words(fd, mine, wfirst, 0u, cbits, cbits);
    vu4 w[4];
    first_words(lw, w);
    dec.fill_mid(fd, mid);
    const uint16_t* lut = reinterpret_cast<const uint16_t*>(lut32);
#pragma unroll 4
    for (int i = tid; i < 1 << kLutBits; i += kDecChunks) {
        uint32_t sy[4] = {0u, 0u, 0u, 0u}, at = 0, n = 0;
        bool on = true;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t e = lut[((uint32_t)i << at) & ((1u << kLutBits) - 1u)], len = e >> kLutSymBits;
            on = on && len != 0u && at + len <= (uint32_t)kLutBits;
            sy[j] = on ? e & ((1u << kLutSymBits) - 1u) : 0u;
            at += on ? len : 0u;
            n += on ? 1u : 0u;
        }
        runs[i] = vu2{sy[0] | (at << kLutSymBits) | (sy[1] << 16),
                      sy[2] | (sy[3] << 16) | (n << (16 + kLutSymBits))};
    }
    static_assert(kLutBits < 1 << (16 - kLutSymBits), "a run's length fits above its first symbol");
    __syncthreads();
    if (cnt == 0) return;
    dec.start(lw, w);
    SZI_G uint16_t* out = gp(fd.codes) + s0;
    int k = 0;
    // a run is written whole, what is past its end over again by the next
    while (k + 32 <= cnt) {
        dec.refill();
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            vu2 sy;
            const int n = dec.some(runs, sy);
            *reinterpret_cast<SZI_G vu2a2*>(out + k) = sy;
            k += n;
        }
    }
#pragma unroll 1
    while (k < cnt) {
        dec.refill();
        vu2 sy;
        const int n = dec.some(runs, sy);
        out[k] = (uint16_t)sy.x;
        if (n > 1 && k + 1 < cnt) out[k + 1] = (uint16_t)(sy.x >> 16);
        if (n > 2 && k + 2 < cnt) out[k + 2] = (uint16_t)sy.y;
        if (n > 3 && k + 3 < cnt) out[k + 3] = (uint16_t)(sy.y >> 16);
        k += n;
    }
}

// Eight lanes a chunk.  A decode block is kUnits units of 32 chunks, eight a
// wave.  The G workgroups take the n units of one field in turn: hard places
// lie together (a field's last plane, predicted from one side, holds its long
// codes), and in runs of n / G one workgroup had them all (512^3 with 0.1 %
// spikes, long codes throughout: the last workgroup ended at 197 us, 99 in 100
// by 120; decode 209 us in runs, 160 in turn).  A batch's units go in runs
// [b n / G, (b + 1) n / G): a workgroup meets fewer fields, each a table to
// fill (in turn: 24 fields of 1800x3600 134 -> 146 us, 256 of 64^3 66 -> 78).
constexpr int kUnits = kSubParts;
static_assert(kUnits * kUnitChunks == kDecChunks && kUnitChunks == 32, "32 chunks a unit, eight lanes each");

__global__ __launch_bounds__(kDecChunks) void k_huff_decode8(const FieldDesc* __restrict__ F, int nfields,
                                                             const uint64_t* __restrict__ boff,
                                                             uint64_t units) {
    __shared__ __align__(16) uint32_t rings[kDecChunks * kRing];
    __shared__ __align__(16) uint32_t lut32[kDtLimit];   // 2^kLutBits u16 entries
    extern __shared__ uint32_t tab_hi[];   // decode-table words kDtLimit .. dtab_words(nsym)
    const int tid = threadIdx.x;
    const uint32_t q = ((uint32_t)tid >> 3) & 7u;   // the lane's part: eight lanes of a chunk lie 8 apart
    LaneDec dec;
    dec.lut = reinterpret_cast<const uint16_t*>(lut32);
    dec.tab_hi = tab_hi;
    dec.ring = rings + tid * kRing;
    dec.rot = ((uint32_t)tid & (kRing / 4 - 1)) << 2;
    // a unit as this lane sees it: its chunk's record
    struct Unit {
        int f;
        uint32_t ch;         // chunk of the field (fields have fewer than 2^32)
        uint32_t cbits;
        // entry q and the next of the chunk's record: where the part starts
        // and ends.  The first part starts at 0 and holds the chunk's place
        // instead; the last ends with the chunk, and its lanes 0, 1 and 2
        // hold the halves of the unit's first word and its first chunk's bits.
        uint32_t bo, be;
    };
    const uint32_t lane = (uint32_t)tid & 63u;
    auto request = [&](uint64_t u, Unit& n) SZI_INLINE {   // n.f: the field of the unit before
        while (u / kUnits >= boff[n.f + 1]) ++n.f;
        const FieldDesc& fd = F[n.f];
        n.ch = (uint32_t)(u - boff[n.f] * kUnits) * kUnitChunks + (uint32_t)(8 * (tid >> 6) + (tid & 7));
        n.cbits = n.bo = n.be = 0u;
        const SZI_G uint16_t* rec = gp((const uint16_t*)fd.sub);
        const SZI_G uint16_t* bits = gp((const uint16_t*)fd.chunk_bits);
        const uint32_t c0 = (uint32_t)(u - boff[n.f] * kUnits) * kUnitChunks;
        const SZI_G uint16_t* end = rec + ((uint64_t)kSubParts * n.ch + q + 1u);
        bool has = n.ch < fd.nchunks;
        if (has) {
            n.cbits = (uint32_t)bits[n.ch];
            n.bo = (uint32_t)rec[(uint64_t)kSubParts * n.ch + q];
        }
        if (q + 1u == (uint32_t)kSubParts) {
            has = lane < 59u && c0 < fd.nchunks;
            end = lane == 58u ? bits + c0 : rec + (uint64_t)kSubParts * (c0 + (lane & 1u));
        }
        if (has) n.be = (uint32_t)*end;
    };
    // a requested unit's words for the lane
    auto place = [&](const FieldDesc& fd, const Unit& n, bool any) SZI_INLINE {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)n.be, 56);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)n.be, 57);
        const uint32_t b0 = (uint32_t)__builtin_amdgcn_readlane((int)n.be, 58);
        const uint32_t rel = (uint32_t)__shfl((int)n.bo, (int)(lane & 7u));
        const uint32_t at = n.ch % kUnitChunks;
        const uint32_t wfirst = (lo | hi << 16) + (at == 0u ? 0u : (at == 1u ? (b0 + 31u) >> 5 : rel));
        return lane_words(fd, any, wfirst, q > 0u ? n.bo : 0u, q + 1u < (uint32_t)kSubParts ? n.be : 0xFFFFu,
                          n.cbits);
    };
    // symbols of the lane in a unit (none from a corrupt offset)
    auto symbols = [&](const FieldDesc& fd, const Unit& n, uint64_t& s0) SZI_INLINE {
        const int SC = fd.chunk / kSubParts;
        s0 = (uint64_t)n.ch * (uint32_t)fd.chunk + q * (uint32_t)SC;
        if (n.ch >= fd.nchunks || s0 >= fd.npts || (q > 0u && n.bo > n.cbits)) return 0;
        return s0 + SC <= fd.npts ? SC : (int)(fd.npts - s0);
    };
    const uint32_t step = nfields == 1 ? gridDim.x : 1u;
    uint64_t u = nfields == 1 ? blockIdx.x : (uint64_t)blockIdx.x * units / gridDim.x;
    const uint64_t ue = nfields == 1 ? units : ((uint64_t)blockIdx.x + 1) * units / gridDim.x;
    if (u >= ue) return;
    // the current unit's words and the next one's record are on their way
    Unit cu, nx;
    cu.f = block_field(boff, nfields, u / kUnits);
    request(u, cu);
    uint64_t s0;
    int cnt = symbols(F[cu.f], cu, s0);
    LaneWords lw = place(F[cu.f], cu, cnt > 0);
    vu4 w[4];
    first_words(lw, w);
    nx = cu;
    if (u + step < ue) request(u + step, nx);
    int tf = -1;   // the field whose tables are in LDS
    while (true) {
        const FieldDesc& fd = F[cu.f];
        if (cu.f != tf) {   // uniform over the workgroup
            if (tf >= 0) __syncthreads();
            fill_tables(fd, lut32, tab_hi);
            dec.tables(fd);
            __syncthreads();
            tf = cu.f;
        }
        dec.start(lw, w);
        {   // the unit's share of the field's outliers, into the output for the replay
            const uint64_t u0 = boff[cu.f] * kUnits, nu = boff[cu.f + 1] * kUnits - u0;
            for (uint64_t k = (u - u0) * kDecChunks + (uint32_t)tid; k < fd.n_outliers; k += nu * kDecChunks) {
                const uint32_t idx = gp(fd.outlier_idx)[k];
                if (idx < fd.npts) gp(fd.out)[idx] = gp(fd.outlier_val)[k];
            }
        }
        const int n = cnt;
        const uint64_t first = s0;
        const uint32_t ch = cu.ch;
        if (u + step < ue) {
            cu = nx;
            cnt = symbols(F[cu.f], cu, s0);
            lw = place(F[cu.f], cu, cnt > 0);
            first_words(lw, w);
            if (u + 2ull * step < ue) request(u + 2ull * step, nx);
        }
        int k = 0;
        // Symbols leave 64 at a time where every lane of the wave has them
        // (all but a field's last chunks): the eight lanes of a chunk
        // exchange their pieces, and store j writes the whole 128-byte line
        // of part j.
        if (((uintptr_t)fd.codes & 15u) == 0u) {
            const uint32_t SC = (uint32_t)fd.chunk / kSubParts;
            SZI_G uint16_t* cout = gp(fd.codes) + (uint64_t)ch * (uint32_t)fd.chunk + 8u * q;
#pragma unroll 1
            for (; !wave_any(k + 64 > n); k += 64) {
                vu4 p[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) p[j] = dec.group8();
                exchange8(p);
#pragma unroll
                for (int j = 0; j < 8; ++j) *reinterpret_cast<SZI_G vu4*>(cout + (uint32_t)j * SC + (uint32_t)k) = p[j];
            }
            // a wave that holds a field's end, or parts of fewer symbols
            // (chunks of 256): each lane its own, 16 bytes at a time (two at
            // a time a line of 5000 points took 20.6 us, now 16, in chunks of
            // 2048 36.8, now 27.8; 256^3 in chunks of 256 87, now 30)
            SZI_G uint16_t* out = gp(fd.codes) + first;
#pragma unroll 1
            for (; k + 8 <= n; k += 8) *reinterpret_cast<SZI_G vu4*>(out + k) = dec.group8();
        }
        dec.tail(gp(fd.codes) + first, k, n);
        if ((u += step) >= ue) break;
    }
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// ------------------------------------------------------- zero-word elision
// The de-redundancy step after Huffman coding (taking the place of the
// closed pass of Sec. VI-B): the words section becomes a bitmap of the
// non-zero words (bit k % 32 of bitmap word k / 32 for word k) followed by
// those words in order.
//
// One workgroup per encode block, whose words it elides: the non-zero words
// before it follow from the encode's sums, each wave counts a quarter of the
// block's words and then writes them.  Rounds of 64 words start at multiples
// of 64; the bitmap word of 32 words is written by the block that holds the
// first of them.  A field that would not get shorter is left alone from its
// totals.  (One launch in place of a count, a scan and a write over tiles:
// 64^3 13 -> 6 us, 512^3 14 -> 7, 24 climate fields 37 -> 24.)
__global__ __launch_bounds__(256) void k_elide(const FieldDesc* __restrict__ F, int nfields,
                                               const uint64_t* __restrict__ boff, EncSums sums) {
    __shared__ uint32_t red[8], cnt[4];
    const int f = block_field(boff, nfields, blockIdx.x);
    const FieldDesc& fd = F[f];
    const uint64_t bf = boff[f], be = boff[f + 1];
    uint32_t nz, before, none;
    sum_before(sums.nz, nullptr, sums.supnz, sums, f, bf, be, red, nz, none);
    const uint64_t nw = (uint64_t)sums.woff[be - 1] + sums.words[be - 1], nbm = (nw + 31) / 32;
    if (blockIdx.x == be - 1 && threadIdx.x == 0) {
        fd.tot[0] = nw;
        fd.tot[1] = nz;
    }
    if (nbm + nz >= nw) return;   // uniform: the field keeps its words
    __syncthreads();
    sum_before(sums.nz, nullptr, sums.supnz, sums, f, bf, blockIdx.x, red, before, none);
    const uint64_t w0 = sums.woff[blockIdx.x], w1 = w0 + sums.words[blockIdx.x];
    const uint64_t base = w0 & ~(uint64_t)63;
    const uint32_t rounds = (uint32_t)((w1 - base + 63) / 64), each = (rounds + 3) / 4;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t r0 = wave * each < rounds ? wave * each : rounds;
    const uint32_t r1 = r0 + each < rounds ? r0 + each : rounds;
    const SZI_G uint32_t* words = gp((const uint32_t*)fd.words);
    constexpr int kIn = 8;   // rounds of loads in flight
    uint32_t n = 0;
    for (uint32_t r = r0; r < r1; r += kIn) {
        uint32_t w[kIn];
#pragma unroll
        for (int k = 0; k < kIn; ++k) {   // unconditional loads, held inside the block's words
            const uint64_t i = base + (uint64_t)(r + k) * 64 + lane;
            w[k] = words[i < w1 ? i : w1 - 1];
        }
#pragma unroll
        for (int k = 0; k < kIn; ++k) {
            const uint64_t i = base + (uint64_t)(r + k) * 64 + lane;
            n += (uint32_t)__popcll(wave_ballot(r + k < r1 && i >= w0 && i < w1 && w[k] != 0u));
        }
    }
    if (lane == 0) cnt[wave] = n;
    __syncthreads();
    uint64_t at = nbm + before;
    for (uint32_t k = 0; k < wave; ++k) at += cnt[k];
    SZI_G uint32_t* sec = gp(fd.esec);
    for (uint32_t r = r0; r < r1; r += kIn) {
        uint32_t w[kIn];
#pragma unroll
        for (int k = 0; k < kIn; ++k) {   // past the block too, for its last bitmap word
            const uint64_t i = base + (uint64_t)(r + k) * 64 + lane;
            w[k] = words[i < nw ? i : nw - 1];
        }
#pragma unroll
        for (int k = 0; k < kIn; ++k) {
            const uint64_t i0 = base + (uint64_t)(r + k) * 64, i = i0 + lane;
            const bool live = r + k < r1;   // uniform
            const uint64_t all = wave_ballot(i < nw && w[k] != 0u);
            const bool mine = live && i >= w0 && i < w1 && w[k] != 0u;
            const uint64_t m = wave_ballot(mine);
            const uint64_t b = i0 + 32u * lane;   // lanes 0 and 1: the round's bitmap words
            if (live && lane < 2u && b >= w0 && b < w1) sec[b / 32] = (uint32_t)(all >> (32u * lane));
            if (mine) sec[at + lanes_below(m)] = w[k];
            at += (uint64_t)__popcll(m);
        }
    }
}

// The restore (upload of an elided blob) splits the words into tiles of tw
// words (8192, or 2048 where there are few), one wave per tile: counts of
// set bits, an exclusive scan of the tile counts (k_scan_blocks), then each
// tile's words in place.
static_assert(kElideTileWords % 2048 == 0 && kElideTileSmall % 2048 == 0,
              "a tile is whole rounds of 64 bitmap words");

__global__ __launch_bounds__(256) void k_restore_count(const ElideField* __restrict__ E, int nf,
                                                       const uint64_t* __restrict__ toff,
                                                       uint64_t ntiles, uint64_t tw, uint32_t* cnt) {
    // the wave's tile, uniform (so the field record and its pointers sit in
    // scalar registers, loaded once, not again before every word)
    const uint64_t tile = (uint64_t)blockIdx.x * 4 + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t lane = threadIdx.x & 63u;
    if (tile >= ntiles) return;
    const int f = block_field(toff, nf, tile);
    const ElideField& e = E[f];
    const uint64_t nbm = (e.nw + 31) / 32;
    const uint64_t w0 = (tile - toff[f]) * tw;
    const SZI_G uint32_t* sec = gp((const uint32_t*)e.sec);
    uint32_t n = 0;
    for (int j = 0; j < (int)(tw / 2048); ++j) {
        const uint64_t b = w0 / 32 + (uint64_t)j * 64 + lane;
        n += (uint32_t)__popc(b < nbm ? sec[b] : 0u);
    }
    n = wave_sum(n);
    if (lane == 0) cnt[tile] = n;
}

// restore: the words of a tile from the bitmap and the non-zero words
__global__ __launch_bounds__(256) void k_restore_write(const ElideField* __restrict__ E, int nf,
                                                       const uint64_t* __restrict__ toff,
                                                       uint64_t ntiles, uint64_t tw,
                                                       const uint64_t* __restrict__ off) {
    // the wave's tile, uniform (so the field record and its pointers sit in
    // scalar registers, loaded once, not again before every word)
    const uint64_t tile = (uint64_t)blockIdx.x * 4 + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t lane = threadIdx.x & 63u;
    if (tile >= ntiles) return;
    const int f = block_field(toff, nf, tile);
    const ElideField& e = E[f];
    const uint64_t nw = e.nw, nbm = (nw + 31) / 32;
    const uint64_t w0 = (tile - toff[f]) * tw;
    if (w0 >= nw) return;
    uint64_t at = nbm + (off[tile] - off[toff[f]]);
    const SZI_G uint32_t* sec = gp(e.sec);
#pragma unroll 4
    for (int it = 0; it < (int)(tw / 64); ++it) {
        const uint64_t i0 = w0 + (uint64_t)it * 64, i = i0 + lane;
        const uint32_t lo = i0 / 32 < nbm ? sec[i0 / 32] : 0u;
        const uint32_t hi = i0 / 32 + 1 < nbm ? sec[i0 / 32 + 1] : 0u;
        const uint64_t m = (uint64_t)lo | (uint64_t)hi << 32;
        const bool set = (m >> lane) & 1u;
        if (i < nw) gp(e.words)[i] = set ? sec[at + lanes_below(m)] : 0u;
        at += (uint64_t)__popcll(m);
    }
}

// ------------------------------------------------------- launchers
hipError_t launch_elide(const FieldDesc* d_fields, int nfields, const uint64_t* d_boff,
                        uint64_t nblocks, EncSums sums, hipStream_t st) {
    if (nblocks == 0) return hipSuccess;
    if (sums.scanned())
        hipLaunchKernelGGL(k_scan_long<1>, dim3((unsigned)nfields), dim3(256), 0, st, d_boff, sums.supnz, sums.shift);
    hipLaunchKernelGGL(k_elide, dim3((unsigned)nblocks), dim3(256), 0, st, d_fields, nfields, d_boff, sums);
    return hipGetLastError();
}

hipError_t launch_restore(const ElideField* d_e, int nf, const uint64_t* d_toff, uint64_t ntiles,
                          uint64_t tw, uint32_t* d_cnt, uint64_t* d_off, hipStream_t st) {
    if (ntiles == 0) return hipSuccess;
    if (tw == 0 || tw % 2048 != 0) return hipErrorInvalidValue;
    const dim3 g((unsigned)((ntiles + 3) / 4)), b(256);
    hipLaunchKernelGGL(k_restore_count, g, b, 0, st, d_e, nf, d_toff, ntiles, tw, d_cnt);
    if (ntiles > 16 * 1024)
        hipLaunchKernelGGL(k_scan_blocks<true>, dim3(1), dim3(1024), 0, st, d_cnt, ntiles, d_off);
    else
        hipLaunchKernelGGL(k_scan_blocks<false>, dim3(1), dim3(1024), 0, st, d_cnt, ntiles, d_off);
    hipLaunchKernelGGL(k_restore_write, g, b, 0, st, d_e, nf, d_toff, ntiles, tw, d_off);
    return hipGetLastError();
}

hipError_t launch_huff_stats(const FieldDesc* d_fields, int nfields, const uint64_t* d_boff,
                             uint64_t nblocks, int chunk, int ec, uint32_t* d_ccnt, EncSums sums,
                             int max_nsym, hipStream_t st) {
    if (nblocks == 0) return hipSuccess;
    if (ec < 4 || ec > kEncBlockMax || ec % 4 != 0) return hipErrorInvalidValue;
    const size_t lds = (size_t)max_nsym * sizeof(uint32_t);
    const dim3 g((unsigned)nblocks), b(256);
    switch (chunk) {
    case 256: hipLaunchKernelGGL(k_huff_stats<4>, g, b, lds, st, d_fields, nfields, d_boff, ec, d_ccnt, sums); break;
    case 512: hipLaunchKernelGGL(k_huff_stats<8>, g, b, lds, st, d_fields, nfields, d_boff, ec, d_ccnt, sums); break;
    case 1024: hipLaunchKernelGGL(k_huff_stats<16>, g, b, lds, st, d_fields, nfields, d_boff, ec, d_ccnt, sums); break;
    case 2048: hipLaunchKernelGGL(k_huff_stats<32>, g, b, lds, st, d_fields, nfields, d_boff, ec, d_ccnt, sums); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_huff_encode(const FieldDesc* d_fields, int nfields, const uint64_t* d_boff,
                              uint64_t nblocks, int chunk, int ec, const uint32_t* d_ccnt, EncSums sums,
                              int max_nsym, hipStream_t st) {
    if (nblocks == 0) return hipSuccess;
    if (ec < 4 || ec > kEncBlockMax || ec % 4 != 0) return hipErrorInvalidValue;
    const int mcw = enc_chunk_words(chunk);
    const size_t lds = ((size_t)max_nsym + 4 * (size_t)mcw) * sizeof(uint32_t);
    const dim3 g((unsigned)nblocks), b(256);
    if (sums.scanned())
        hipLaunchKernelGGL(k_scan_long<2>, dim3((unsigned)nfields), dim3(256), 0, st, d_boff, sums.sup, sums.shift);
    switch (chunk) {
    case 256: hipLaunchKernelGGL(k_huff_encode<4>, g, b, lds, st, d_fields, nfields, d_boff, ec, d_ccnt, sums); break;
    case 512: hipLaunchKernelGGL(k_huff_encode<8>, g, b, lds, st, d_fields, nfields, d_boff, ec, d_ccnt, sums); break;
    case 1024: hipLaunchKernelGGL(k_huff_encode<16>, g, b, lds, st, d_fields, nfields, d_boff, ec, d_ccnt, sums); break;
    case 2048: hipLaunchKernelGGL(k_huff_encode<32>, g, b, lds, st, d_fields, nfields, d_boff, ec, d_ccnt, sums); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}


hipError_t launch_huff_decode(const FieldDesc* d_fields, int nfields, const uint64_t* d_dboff,
                              uint64_t nblocks, const uint32_t* d_bsum, int max_nsym, DecodeKind kind,
                              int num_cus, hipStream_t st) {
    if (nblocks == 0) return hipSuccess;
    const size_t lds = (size_t)(dtab_words(max_nsym) - kDtLimit) *
                       sizeof(uint32_t);
    if (kind == kDecSplit) {
        // as many workgroups as are resident at once, but no more than units
        uint64_t grid = (uint64_t)num_cus * (uint64_t)resident_per_cu(k_huff_decode8, lds);
        if (grid > kUnits * nblocks) grid = kUnits * nblocks;
        hipLaunchKernelGGL(k_huff_decode8, dim3((unsigned)grid), dim3(kDecChunks), lds, st, d_fields, nfields,
                           d_dboff, kUnits * nblocks);
    } else if (kind == kDecRuns) {
        hipLaunchKernelGGL(k_huff_decode_runs, dim3((unsigned)(kRunWaves * nblocks)), dim3(kDecChunks), lds, st,
                           d_fields, nfields, d_dboff, d_bsum);
    } else {
        hipLaunchKernelGGL(k_huff_decode1, dim3((unsigned)nblocks), dim3(kDecChunks), lds, st, d_fields, nfields,
                           d_dboff, d_bsum);
    }
    return hipGetLastError();
}


}  // namespace szi
