// k_huff.hip -- chunked Huffman encode/decode with fused outlier compaction
// (Sec. VI-A) on gfx950.
//
// Encode: up to 32 consecutive chunks of one field per workgroup (4 wave64,
// one chunk per wave at a time, C/64 consecutive symbols per lane).
//   k_huff_stats   bit count and outlier count of every chunk; sums per
//                  workgroup block and per 64 blocks
//   k_huff_encode  chunk offsets = sums of the field's earlier blocks +
//                  in-block prefix; packs the codewords MSB-first through
//                  LDS and writes the outliers (index, original value) in
//                  ascending index order; sums of the non-zero words
//   k_elide        zero-word elision of the words, block by block
// Decode: kDecChunks chunks per decode block, kSubParts lanes per chunk from
// the bit offsets of its parts that the encoder records (one lane per chunk
// without them).
//   k_dec_prep     (k_plan.hip) word count of every decode block
//   k_huff_decode  sum of the field's earlier block sums and an in-block
//                  scan, then a table-driven canonical decode from a
//                  two-word register window fed by a per-lane LDS word
//                  ring; 64 symbols per lane stored at once
#include "dev_common.h"

namespace szi {

constexpr int kDecChunks = 256;
static_assert(kDecChunks == kDecBlockChunks,
              "the host sizes the decode grid with the same chunk count");

// Sum over the blocks [first, blk) of field f of one number a block or two
// (b, the second of a line of sup), by the 256 threads of a workgroup; red:
// 8 words of LDS, with a barrier inside.
__device__ __forceinline__ void sum_before(const uint32_t* __restrict__ a, const uint32_t* __restrict__ b,
                                           const uint32_t* __restrict__ sup, int shift, int f,
                                           uint64_t first, uint64_t blk, uint32_t* red, uint32_t& ra,
                                           uint32_t& rb) {
    const uint32_t nsup = (uint32_t)((blk - first) >> shift);
    const uint64_t sb0 = (first >> shift) + (uint32_t)f;
    uint32_t xa = 0, xb = 0;
    for (uint32_t i = threadIdx.x; i < nsup; i += 256) {
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
                                                    uint32_t* cwords, uint32_t* couts,
                                                    EncSums sums) {
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
                cwords[fd.chunk_base + ch] = words;
                couts[fd.chunk_base + ch] = zeros;
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

// Exclusive scan of a u32 array of length n into u64 offsets; one
// workgroup of 1024 threads, a contiguous run per thread: run sums, wave
// scans, the 16 wave totals through LDS (one barrier), then the run's
// offsets.  off[n] receives the total.  LONG = false takes runs of at
// most kRun (n <= 16384) in registers; LONG = true, longer runs kRun
// elements a round (the launchers choose by n).
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
        for (int k = 0; k < kRun; ++k) {
            sa += va[k];
        }
    } else if (LONG) {
        // longer runs (the LONG instance): kRun elements a round, their
        // loads issued together
        for (uint64_t i0 = beg; i0 < end; i0 += kRun) {
#pragma unroll
            for (int k = 0; k < kRun; ++k) {
                const uint64_t i = i0 + k;
                va[k] = i < end ? a[i] : 0u;
                }
#pragma unroll
            for (int k = 0; k < kRun; ++k) {
                sa += va[k];
                }
        }
    }
    uint64_t xa = sa;   // inclusive scans over the wave's lanes
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t ya = __shfl_up(xa, o);
        if (lane >= o) {
            xa += ya;
        }
    }
    __shared__ uint64_t wa[16];
    if (lane == 63) {
        wa[wave] = xa;
    }
    __syncthreads();
    for (int k = 0; k < wave; ++k) {
        xa += wa[k];
    }
    uint64_t ra = xa - sa;
    if (regs) {
#pragma unroll
        for (int k = 0; k < kRun; ++k) {
            const uint64_t i = beg + k;
            if (i < end) {
                aoff[i] = ra;
            }
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
                if (i < end) {
                    aoff[i] = ra;
                    }
                ra += va[k];
                }
        }
    }
    if (t == 1023) {
        aoff[n] = xa;
    }
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
                                                     const uint32_t* __restrict__ cwords,
                                                     const uint32_t* __restrict__ couts,
                                                     EncSums sums) {
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
    uint32_t cw = 0, co = 0;
    if (lane < ec && first + lane < fd.nchunks) {
        cw = cwords[fd.chunk_base + first + lane];
        co = couts[fd.chunk_base + first + lane];
    }
    uint32_t tw, to;
    const uint32_t pw = wave_excl_scan(cw, &tw);
    const uint32_t po = wave_excl_scan(co, &to);
    // words and outliers of the field's earlier blocks; the barrier inside
    // also completes the code book in LDS
    uint32_t bw0, bo0;
    sum_before(sums.words, sums.outs, sums.sup, sums.shift, f, boff[f], blockIdx.x, red, bw0, bo0);
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
        if (wave_any(least == 0u)) {
#pragma unroll
            for (int k = 0; k < PER; ++k) bz += (k < ns && sym[k] == 0u) ? 0x10000u : 0u;
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
        if (tbz >> 16) {   // uniform: outliers in this chunk
            uint32_t zo = pbz >> 16;
            const uint64_t oo = (uint64_t)bo0 + (uint32_t)__builtin_amdgcn_readlane((int)po, j);
            const uint64_t s0 = ch * (uint64_t)C + (uint64_t)lane * PER;
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                if (k < ns && sym[k] == 0) {
                    if (oo + zo < fd.n_outliers) {   // the histogram sized the list
                        gp(fd.outlier_idx)[oo + zo] = (uint32_t)(s0 + k);
                        gp(fd.outlier_val)[oo + zo] = gp(fd.in)[s0 + k];
                    }
                    ++zo;
                }
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
            // the decoder's starting bits of the chunk's eighths (symbol
            // 8 k PER starts lane 8 k), as one 16-byte store: 0, b1 .. b7
            static_assert(kSubParts == 8, "eight parts: lanes 8, 16, .., 56");
            uint32_t b[8];
            b[0] = 0u;
#pragma unroll
            for (int k = 1; k < 8; ++k) b[k] = (uint32_t)__builtin_amdgcn_readlane((int)pos, 8 * k);
            if (lane == 0) gp(fd.choff)[ch] = (uint32_t)ow;   // and the chunk's first word
            if (lane == 0)
                *reinterpret_cast<SZI_G vu4*>(gp(fd.sub) + (uint64_t)kSubParts * ch) =
                    vu4{b[0] | (b[1] << 16), b[2] | (b[3] << 16), b[4] | (b[5] << 16), b[6] | (b[7] << 16)};
        }
        wave_lds_sync();
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
// (fd.choff: the chunk's first word; fd.sub: the eighths' bit offsets, the
// first 0; both kept with a compressed result): eight times the independent
// chains, each an eighth as long (against four lanes a chunk, 1 % faster at
// rel 1e-3, 5 % at 1e-4 and 38 % on a 64^3 field), and no sums over the
// field's earlier words ahead of them.  A workgroup then covers an eighth of
// a decode block (kDecChunks chunks).  A field without offsets (an uploaded
// blob) is decoded by one lane a chunk, which finds its words from the word
// counts that the prologue summed.
//
// What a workgroup of eight lanes a chunk takes at 512^3, rel 1e-3 (164 us
// for 5.3 rounds of workgroups, before; timed with parts of the kernel left
// out): 61 us ahead of the first symbol (table, sums, offsets, words, one
// after another), 34 us for stores of 64 different lines an instruction, the
// rest the symbols.  So the words are requested before the table is filled,
// and eight lanes of a chunk exchange their 16-byte pieces, after which each
// store instruction writes eight whole lines (DECT us now).
constexpr int kRing = 32;   // ring words per lane (power of 2)

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

template <int Q>
__global__ __launch_bounds__(kDecChunks) void k_huff_decode(const FieldDesc* __restrict__ F,
                                                            int nfields,
                                                            const uint64_t* __restrict__ boff,
                                                            const uint32_t* __restrict__ bsum) {
    // the rings and the look-up table at fixed LDS addresses (a look-up's
    // address is then its index and an offset, with no base to add); the
    // limits, bases and sorted symbols, sized by the radius, after them
    __shared__ __align__(16) uint32_t rings[kDecChunks * kRing];
    __shared__ __align__(16) uint32_t lut32[kDtLimit];   // 2^kLutBits u16 entries
    __shared__ uint32_t scan[kDecChunks / 64];
    __shared__ uint64_t pre[kDecChunks / 64];
    extern __shared__ uint32_t tab_hi[];   // decode-table words kDtLimit .. dtab_words(nsym)
    static_assert(Q == 1 || Q == kSubParts, "one lane or kSubParts per chunk");
    constexpr int CPW = kDecChunks / Q;   // chunks per workgroup
    const uint64_t pblk = blockIdx.x / Q;   // the decode block
    const uint32_t part = blockIdx.x % Q;   // the workgroup's share of it
    const int f = block_field(boff, nfields, pblk);
    const FieldDesc& fd = F[f];
    const int nsym = 2 * fd.R;
    const int ntab = dtab_words(nsym);
    const uint16_t* lut = reinterpret_cast<const uint16_t*>(lut32);
    const int tid = threadIdx.x;
    auto fill_tables = [&]() SZI_INLINE {
        // the look-up table 16 bytes at a time, its four loads per lane in
        // flight together (word by word where the tables do not start on 16
        // bytes: odd radius), then the rest word by word
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
    };
    // length limits of the codes longer than the LUT, in scalar registers
    uint32_t lim[kLmax - kLutBits - 1];
#pragma unroll
    for (int l = kLutBits + 1; l < kLmax; ++l)
        lim[l - kLutBits - 1] = __builtin_amdgcn_readfirstlane(gp(fd.dtab)[kDtLimit + l]);
    // the lane's part of its chunk: eight lanes of a chunk lie 8 apart (exchange8)
    const uint32_t q = Q > 1 ? ((uint32_t)tid >> 3) & 7u : 0u;
    const uint64_t bfirst = (pblk - boff[f]) * kDecChunks;   // the decode block's first chunk
    const uint64_t ch = Q > 1 ? bfirst + part * CPW + (uint32_t)(8 * (tid >> 6) + (tid & 7)) : bfirst + (uint32_t)tid;
    const bool live = ch < fd.nchunks;
    const uint32_t cbits = live ? (uint32_t)gp(fd.chunk_bits)[ch] : 0u;
    const int C = fd.chunk;
    const int SC = C / Q;   // symbols per lane
    const uint64_t s0 = ch * (uint64_t)C + (uint64_t)(q * (uint32_t)SC);
    int cnt = !live || s0 >= fd.npts ? 0 : (s0 + SC <= fd.npts ? SC : (int)(fd.npts - s0));
    uint64_t wfirst = 0;               // the chunk's first word
    uint32_t bo = 0, be0 = cbits;      // the lane's bits of it
    if constexpr (Q > 1) {
        if (live) {
            wfirst = gp(fd.choff)[ch];
            if (q > 0u) bo = (uint32_t)gp(fd.sub)[(uint64_t)Q * ch + q];
            if (q + 1u < (uint32_t)Q) be0 = (uint32_t)gp(fd.sub)[(uint64_t)Q * ch + q + 1];
        }
        if (bo > cbits) cnt = 0;   // a corrupt offset: nothing to decode from it
    } else {
        // words of the field's earlier blocks (the sum of their word counts)
        // and the workgroup's exclusive scan of its chunks' word counts
        fill_tables();
        const uint32_t nw = (cbits + 31) >> 5;
        uint64_t pb = 0;
        for (uint64_t i = boff[f] + (uint64_t)tid; i < pblk; i += kDecChunks) pb += bsum[i];
        for (int o = 32; o > 0; o >>= 1) pb += __shfl_xor(pb, o);
        uint32_t tot;
        const uint32_t wx = wave_excl_scan(nw, &tot);
        if ((tid & 63) == 0) {
            scan[tid >> 6] = tot;
            pre[tid >> 6] = pb;
        }
        __syncthreads();
        for (int k = 0; k < kDecChunks / 64; ++k) wfirst += pre[k];
        for (int k = 0; k < (tid >> 6); ++k) wfirst += scan[k];
        wfirst += wx;
    }
    const uint64_t w0abs = wfirst + (bo >> 5);   // the lane's first word
    const uint32_t b0 = bo & 31u;                // and bit in it
    // word indices count from the 4-aligned word at or below the lane's
    // first; requests stop after the word that holds the lane's last bit
    // (where the next part starts, else the chunk's end; the ring may
    // then hold stale words past it, which only fill a look-up's unused
    // low bits) and never pass the field's words (the array has kWordPad
    // words of slack, so the 8-word loads of the last request stay inside
    // it).  Stopping at the lane's own end saves a twentieth of decode time.
    const uint64_t wbase = w0abs & ~(uint64_t)3;
    const SZI_G uint32_t* words = gp(fd.words) + wbase;
    const uint32_t be = be0 < bo || be0 > cbits ? cbits : be0;   // a corrupt offset: the chunk's end
    const uint64_t wlim0 = wfirst + ((be + 31u) >> 5);
    const uint64_t wlim = wlim0 < fd.words_cap ? wlim0 : fd.words_cap;
    const uint64_t wleft = wlim > wbase ? wlim - wbase : 0;
    const uint32_t wcap = cnt == 0 ? 0u : (wleft < (1u << 30) ? (uint32_t)wleft : (1u << 30));
    // the lane's ring: word i at ring[(i ^ sw) % kRing], the 16-byte groups
    // permuted per lane so that lanes at the same position hit different banks
    uint32_t* ring = rings + tid * kRing;
    const uint32_t sw = ((uint32_t)tid & (kRing / 4 - 1)) << 2;
    auto slot = [&](uint32_t i) SZI_INLINE { return (i ^ sw) & (uint32_t)(kRing - 1); };
    auto put = [&](uint32_t at, vu4 a, vu4 b) SZI_INLINE {   // words [at, at + 8) into the ring
        *reinterpret_cast<vu4*>(ring + slot(at)) = a;
        *reinterpret_cast<vu4*>(ring + slot(at + 4u)) = b;
    };
    uint32_t wr = 0;                              // next word to request
    uint32_t rd = (uint32_t)(w0abs - wbase);      // next word to read from the ring
    // prime the ring with 16 words
    {
        vu4 a = {0u, 0u, 0u, 0u}, b = a, c = a, d = a;
        if (wcap > 0) {
            a = *reinterpret_cast<const SZI_G vu4*>(words);
            b = *reinterpret_cast<const SZI_G vu4*>(words + 4);
        }
        if (wcap > 8) {
            c = *reinterpret_cast<const SZI_G vu4*>(words + 8);
            d = *reinterpret_cast<const SZI_G vu4*>(words + 12);
        }
        if (Q > 1) {   // the words are on their way; then the table
            fill_tables();
            __syncthreads();
        }
        if (!wave_any(cnt > 0)) return;   // uniform: a wave past the field's chunks
        put(0u, a, b);
        put(8u, c, d);
        wr = 16;
    }
    // the window starts at bit b0 of the first word: the top of w1 (o = 32,
    // held as nego = -o) or bit b0 of w0
    uint32_t w0 = 0u, w1;
    int32_t nego;
    if (b0 == 0u) {
        w1 = ring[slot(rd)];
        ++rd;
        nego = -32;
    } else {
        w0 = ring[slot(rd)];
        w1 = ring[slot(rd + 1u)];
        rd += 2;
        nego = -(int32_t)b0;
    }
    uint32_t nxw = ring[slot(rd)];   // the ring word the next move takes
    auto decode_one = [&]() SZI_INLINE -> uint32_t {
        // bits [o, o + 32) of w0:w1 (the shift amount is 32 - o, taken mod 32)
        const uint32_t x = __builtin_amdgcn_alignbit(w0, w1, (uint32_t)nego);
        const uint32_t e = lut[x >> (32 - kLutBits)];
        uint32_t len = e >> kLutSymBits, sym = e & ((1u << kLutSymBits) - 1u);
        if (wave_any(len == 0)) {
            // longer than the table: the length is one more than the number
            // of length limits at or below the next kLmax bits (canonical
            // codes grow with their length), then one look-up
            const uint32_t w = x >> (32 - kLmax);
            uint32_t ln = kLutBits + 1;
#pragma unroll
            for (int l = kLutBits + 1; l < kLmax; ++l) ln += w >= lim[l - kLutBits - 1] ? 1u : 0u;
            const uint32_t i = tab_hi[kDtBase - kDtLimit + ln] + (w >> (kLmax - ln));
            const uint32_t sl = tab_hi[kDtSorted - kDtLimit + (i < (uint32_t)nsym ? i : 0u)];   // a corrupt stream stays inside
            const bool lng = len == 0;
            sym = lng ? sl : sym;
            len = lng ? ln : len;
        }
        // o += len; past 32 the words move up by one (len <= kLmax < 32)
        nego -= (int32_t)len;
        const bool t = nego < -32;
        w0 = t ? w1 : w0;
        w1 = t ? nxw : w1;
        nego += t ? 32 : 0;
        rd += t ? 1u : 0u;
        nxw = ring[slot(rd)];
        return sym;
    };
    SZI_G uint16_t* out = gp(fd.codes) + s0;   // s0: a multiple of 64 symbols
    const bool vec = ((uintptr_t)fd.codes & 15u) == 0u;   // s0 and k are multiples of 8
    // a group: commit the previous request, maybe request 8 more words,
    // then decode up to 8 symbols
    bool pend = false;
    uint32_t pat = 0;
    vu4 la = {0u, 0u, 0u, 0u}, lb = la;
    auto refill = [&]() SZI_INLINE {
        if (pend) put(pat, la, lb);
        // the ring holds [rd, wr) and a request adds 8; the prefetched word
        // at rd is not overwritten because the ring keeps kRing - 8 >= 7
        pend = wr < wcap && wr + 8 - rd <= (uint32_t)kRing;
        if (pend) {
            pat = wr;
            la = *reinterpret_cast<const SZI_G vu4*>(words + wr);
            lb = *reinterpret_cast<const SZI_G vu4*>(words + wr + 4);
            wr += 8;
        }
    };
    auto group8 = [&]() SZI_INLINE -> vu4 {
        refill();
        vu4 pk;
        uint32_t lo, hi;
        lo = decode_one();
        hi = decode_one();
        pk.x = lo | (hi << 16);
        lo = decode_one();
        hi = decode_one();
        pk.y = lo | (hi << 16);
        lo = decode_one();
        hi = decode_one();
        pk.z = lo | (hi << 16);
        lo = decode_one();
        hi = decode_one();
        pk.w = lo | (hi << 16);
        return pk;
    };
    int k = 0;
    // Symbols leave 64 at a time.  Where every lane of the wave has them (all
    // but a field's last chunks) the eight lanes of a chunk exchange their
    // pieces: store j then writes the whole 128-byte line of part j.
    if (Q > 1 && vec) {
        SZI_G uint16_t* cout = gp(fd.codes) + ch * (uint64_t)C + 8u * q;
#pragma unroll 1
        for (; !wave_any(k + 64 > cnt); k += 64) {
            vu4 p[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) p[j] = group8();
            exchange8(p);
#pragma unroll
            for (int j = 0; j < 8; ++j)
                *reinterpret_cast<SZI_G vu4*>(cout + (uint32_t)(j * SC + k)) = p[j];
        }
    }
    // One lane a chunk: a lane's 64 symbols as eight back-to-back 16-byte
    // stores, so that it writes a whole line at once (half lines written far
    // apart in time cost 15 % more decode time).
    if (Q == 1 && vec) {
#pragma unroll 1
        for (; k + 64 <= cnt; k += 64) {
            vu4 p[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) p[j] = group8();
            SZI_G vu4* o = reinterpret_cast<SZI_G vu4*>(out + k);
#pragma unroll
            for (int j = 0; j < 8; ++j) o[j] = p[j];
        }
    }
#pragma unroll 1
    while (k < cnt) {
        refill();
        const int e = k + 8 < cnt ? k + 8 : cnt;
#pragma unroll 1
        for (; k < e; ++k) out[k] = (uint16_t)decode_one();
    }
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// restore = 0: non-zero words per tile of the words; 1: set bits per tile
// of the bitmap (the tile's 64 bitmap words)
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
    sum_before(sums.nz, nullptr, sums.supnz, sums.shift, f, bf, be, red, nz, none);
    const uint64_t nw = (uint64_t)sums.woff[be - 1] + sums.words[be - 1], nbm = (nw + 31) / 32;
    if (blockIdx.x == be - 1 && threadIdx.x == 0) {
        fd.tot[0] = nw;
        fd.tot[1] = nz;
    }
    if (nbm + nz >= nw) return;   // uniform: the field keeps its words
    __syncthreads();
    sum_before(sums.nz, nullptr, sums.supnz, sums.shift, f, bf, blockIdx.x, red, before, none);
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
                             uint64_t nblocks, int chunk, int ec, uint32_t* d_cwords,
                             uint32_t* d_couts, EncSums sums, int max_nsym, hipStream_t st) {
    if (nblocks == 0) return hipSuccess;
    if (ec < 4 || ec > kEncBlockMax || ec % 4 != 0) return hipErrorInvalidValue;
    const size_t lds = (size_t)max_nsym * sizeof(uint32_t);
    const dim3 g((unsigned)nblocks), b(256);
    switch (chunk) {
    case 256: hipLaunchKernelGGL(k_huff_stats<4>, g, b, lds, st, d_fields, nfields, d_boff, ec, d_cwords, d_couts, sums); break;
    case 512: hipLaunchKernelGGL(k_huff_stats<8>, g, b, lds, st, d_fields, nfields, d_boff, ec, d_cwords, d_couts, sums); break;
    case 1024: hipLaunchKernelGGL(k_huff_stats<16>, g, b, lds, st, d_fields, nfields, d_boff, ec, d_cwords, d_couts, sums); break;
    case 2048: hipLaunchKernelGGL(k_huff_stats<32>, g, b, lds, st, d_fields, nfields, d_boff, ec, d_cwords, d_couts, sums); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_huff_encode(const FieldDesc* d_fields, int nfields, const uint64_t* d_boff,
                              uint64_t nblocks, int chunk, int ec, const uint32_t* d_cwords,
                              const uint32_t* d_couts, EncSums sums, int max_nsym, hipStream_t st) {
    if (nblocks == 0) return hipSuccess;
    if (ec < 4 || ec > kEncBlockMax || ec % 4 != 0) return hipErrorInvalidValue;
    const int mcw = enc_chunk_words(chunk);
    const size_t lds = ((size_t)max_nsym + 4 * (size_t)mcw) * sizeof(uint32_t);
    const dim3 g((unsigned)nblocks), b(256);
    switch (chunk) {
    case 256: hipLaunchKernelGGL(k_huff_encode<4>, g, b, lds, st, d_fields, nfields, d_boff, ec, d_cwords, d_couts, sums); break;
    case 512: hipLaunchKernelGGL(k_huff_encode<8>, g, b, lds, st, d_fields, nfields, d_boff, ec, d_cwords, d_couts, sums); break;
    case 1024: hipLaunchKernelGGL(k_huff_encode<16>, g, b, lds, st, d_fields, nfields, d_boff, ec, d_cwords, d_couts, sums); break;
    case 2048: hipLaunchKernelGGL(k_huff_encode<32>, g, b, lds, st, d_fields, nfields, d_boff, ec, d_cwords, d_couts, sums); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}


hipError_t launch_huff_decode(const FieldDesc* d_fields, int nfields, const uint64_t* d_dboff,
                              uint64_t nblocks, const uint32_t* d_bsum, int max_nsym, int split,
                              hipStream_t st) {
    if (nblocks == 0) return hipSuccess;
    const size_t lds = (size_t)(dtab_words(max_nsym) - kDtLimit) *
                       sizeof(uint32_t);
    if (split)
        hipLaunchKernelGGL(k_huff_decode<kSubParts>, dim3((unsigned)(kSubParts * nblocks)), dim3(kDecChunks), lds, st,
                           d_fields, nfields, d_dboff, d_bsum);
    else
        hipLaunchKernelGGL(k_huff_decode<1>, dim3((unsigned)nblocks), dim3(kDecChunks), lds, st,
                           d_fields, nfields, d_dboff, d_bsum);
    return hipGetLastError();
}


}  // namespace szi
