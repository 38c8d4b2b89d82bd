// Small batches (up to 16 activation vectors) on the matrix cores while the weights stream by once.
//
// Decoding a weight costs the same vector work whether one or sixteen activation vectors use it, so from a
// handful of vectors on the multiply moves to v_mfma_f32_16x16x32_f16 and only the decode stays on the vector
// units.  A wavefront owns four adjacent 64-weight block columns (256 columns of K) and walks down the rows in
// groups of sixteen: lane (i, g) = (lane & 15, lane >> 4) holds block (row r0 + i, column kb0 + g).  MFMA step
// w takes weights 8w..8w+7 of each lane's block as A[i][8g..8g+7] and the matching eight activations of batch
// column j from lane (j, g) as B[8g..8g+7][j]; after eight steps D[i][j] is the product over the wavefront's
// 256 columns.  The activations of a lane never change (its block column is fixed), so they stay in 32
// registers, permuted once into the decoder's element order.  Weights are fully dequantized before the MFMA
// (the four blocks of a step have different scales): Eq.5 and Eq.2 of the paper with the single-rounded fp16
// fused multiply-add, i.e. exactly the values iflow_dequant produces.
// A workgroup is sixteen wavefronts = sixteen column groups = one 4096-column strip.  The grid is resident (at most one
// workgroup per compute unit) and a workgroup walks over groups of sixteen rows, strip by strip, with the strip's
// activations held in registers for all of them; the sixteen partial 16 x 16 tiles of a step are added up through LDS
// in a fixed order (so results do not vary from run to run), one sum per four groups: between two of them the wavefronts
// run freely.  (One per group, with a barrier each and the residual read behind it: 8 vectors with normalization and residual,
// 11008 x 4096, us before -> after: 3.5-bit 13.6 -> 12.2, 8-bit 21.2 -> 15.8, 28672 x 8192 41.7 -> 35.5 and 62.3 -> 51.2.)
#include "iflow_common.h"

namespace iflow {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// Raw bytes of a lane's 64 weights and their block header(s), per format.
template <int KIND> struct SmallRaw { uint32_t d[12]; uint32_t hdr[2]; };   // bit planes: up to 8 words of the low plane, then up to 4 of the high one
template <> struct SmallRaw<KIND_Q3H> { uint32_t d[8]; uint32_t hdr[2]; };   // (header in the spare bits of d)
template <> struct SmallRaw<KIND_Q4>  { uint32_t d[8]; uint32_t hdr[2]; };   // 32 code bytes
template <> struct SmallRaw<KIND_Q8>  { uint32_t d[16]; uint32_t hdr[2]; };  // 64 code bytes

// LDS of a workgroup: the activation staging area of each wavefront (eight batch rows of its 256 columns at a time,
// rows 528 bytes apart so that sixteen lanes reading 16 bytes each from eight different rows hit different banks) and each wavefront's
// partial 16 x 16 tiles of SMALL_ROUNDS rounds: 4 floats per lane, the four lane groups 16 floats further apart, so that the sums over
// them (sixteen rows of four vectors per wavefront) read 64 different banks; and the running sums of the rounds when a row spans several strips.
constexpr int SMALL_XROW = 528;
constexpr int SMALL_XBYTES = 16 * 8 * SMALL_XROW;
constexpr int SMALL_TILE = 4 * (64 + 16) - 16;
constexpr int SMALL_SETS = 2;                                 // register sets of weights in flight per wavefront
constexpr int SMALL_ROUNDS = 4;                               // rounds between two sums over the wavefronts (1024 threads = their outputs)
constexpr int SMALL_MAX_ROUNDS = 16;                          // rounds per workgroup when there is more than one strip
constexpr int SMALL_PART = SMALL_XBYTES + SMALL_ROUNDS * 16 * SMALL_TILE * 4;
constexpr int SMALL_LDS_BYTES = SMALL_PART + SMALL_MAX_ROUNDS * 256 * 4;
constexpr int SMALL_LDS_BYTES_OPS = SMALL_LDS_BYTES + 16 * 16 * 4;        // + the wavefronts' shares of sum x^2 per activation vector

// A grid of at most one workgroup per compute unit; workgroup b takes the groups of sixteen rows group0 + b,
// group0 + b + gridDim.x, ... below `ngroups` ("rounds").  Per strip the activations are loaded once, with loads
// in which neighbouring lanes read neighbouring addresses, turned through LDS into the operand layout and kept in
// registers for all rounds; the weights of the round after next are requested while a round is decoded.
// The modules of a decoder layer around the product, per activation vector (Section 2's module table: "rms" normalization,
// "silu" activation; Section 5: dynamic batching makes several vectors per step the served case): XOP = -1 none (the plain
// kernel), IFLOW_X_PLAIN (residual only), IFLOW_X_RMS_GAIN (v = fp16(x g) at the staging, sum x^2 per vector, the scalar
// 1/sqrt(mean + eps) at the store), IFLOW_X_SILU_MUL (v = fp16(silu(x) aux) at the staging, aux [batch][cols]); a residual
// [batch][rows] is added to the fp32 sum before its one rounding.
struct SmallOps {
    const uint16_t *aux;
    const uint16_t *residual;
    float eps;
};

// UPPER: more than eight vectors.  A kernel of its own for either case, because on a small matrix the second half's loads under a branch show (us, a
// branch / a kernel for each: 1024 x 1024 4-bit, blocks of 32, 9 vectors 5.55 / 5.32, 8 vectors 5.15 / 4.80; 4096 x 11008 3.5-bit, 9 vectors 13.4 / 12.7).
// LINES (8-bit formats): a load of codes takes the 256 consecutive bytes that the wavefront's columns have in a row, of four rows, and its staging rows turn them.  As the operand
// layout wants them, one load touches both lines of all sixteen rows for 16 bytes of every 64, four times over; where rows don't begin at multiples of 256
// bytes this costs most (us, a ring of matrices, 8 vectors: 9918 x 23680 67.6 -> 57.3, 998 x 25856 26.4 -> 22.5, 512 x 8192 7.5 -> 6.9, 11008 x 4096 14.8 -> 14.2, 28672 x 8192
// 49.2 -> 47.3; 36 shapes 0 to 16 % faster).  Up to SMALL_LINES_COLS columns, half of the sixteen wavefronts or more without any, the turn is what shows (1024 x 1024 4.7 -> 5.0, 16384 x 1088 10.4 -> 11.2,
// 2048 x 2048 5.4 -> 5.5; 4096 x 2752 6.2 -> 6.1): the loads stay as they were.  So do those of the other formats, which have 128 bytes and less per row (4-bit, 4096 x 4096 4.9 -> 5.2).
constexpr int64_t SMALL_LINES_COLS = 2048;

template <int F, int S, int XOP, bool UPPER, bool LINES>
__device__ __forceinline__ void gemm_small_body(const uint8_t *__restrict__ packed, const uint16_t *__restrict__ X,
                                                uint16_t *__restrict__ Y, int rows, int cols, int batch, int nbk64, int nstrips,
                                                int64_t header_offset, int group0, int ngroups, const SmallOps ops)
{
    typedef Fmt<F> T;
    constexpr int KIND = T::kind;
    constexpr int HPL = 64 / T::block;                        // block headers per lane (1, or 2 for the 32-wide formats)
    constexpr int WA = Planes<KIND>::WA, WB = Planes<KIND>::WB;       // bit-plane formats: a lane's 64 weights take 2 WA + 2 WB words
    constexpr int NWORDS = kind_has_planes(KIND) ? 2 * WA + 2 * WB : KIND == KIND_Q8 ? 16 : 8;
    // kernels that would keep some of the staging's and the sums' addresses in scratch memory all through the rounds
    constexpr bool TIGHT = KIND == KIND_Q8 || XOP == IFLOW_X_RMS_GAIN || XOP == IFLOW_X_SILU_MUL;
    extern __shared__ __align__(16) uint8_t lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i = lane & 15, g = lane >> 4;
    uint8_t *xst = lds + wave * (8 * SMALL_XROW);
    float *mine = reinterpret_cast<float *>(lds + SMALL_XBYTES) + wave * SMALL_TILE + lane * 4 + g * 16;   // + round * 16 tiles
    float *part = reinterpret_cast<float *>(lds + SMALL_PART);                        // [round][thread of its 256 outputs]
    const int first = group0 + (int)blockIdx.x;
    const int rounds = (ngroups - first + (int)gridDim.x - 1) / (int)gridDim.x;       // >= 1: the grid never exceeds the groups
    const int total = nstrips * rounds;                       // steps (strip, round) of this workgroup, strips outermost
    const int batches = (rounds + SMALL_ROUNDS - 1) / SMALL_ROUNDS, per_batch = (rounds + batches - 1) / batches;
    const bool carry = batches == 1;                          // every round keeps its slot: the strips add up there, one sum at the very end

    // weights of step k = (strip, round): the lane's 64 columns of row (group * 16 + i); steps past the end repeat the last one,
    // rows past the end the last row, dead column groups of a ragged strip the strip's first group: every load stays in bounds
    // The loads go out with four neighbouring lanes on one row (lane = 4 * row + column group: sixteen lanes touch four
    // 64-byte pieces instead of sixteen); round_body moves every word to the lane the MFMA layout wants it in.
    const int il = lane >> 2, gl = lane & 3;
    const int from = 4 * (4 * i + g);                         // ds_bpermute address of the lane that loaded block (i, g)
    // (LINES) where row r's 16-byte piece p is while it is turned: permuted by the row, so that the rows' same piece is in different banks
    auto turned = [&](int r, int p) { return reinterpret_cast<u32x4_t *>(xst + r * 256 + (p ^ r) * 16); };
    static_assert(8 * SMALL_XROW >= 16 * 256, "a step's codes fit where the activations were turned");
    auto load_step = [&](SmallRaw<KIND> &raw, int t, int r) {
        const bool beyond = t >= nstrips;                     // past the last step: every lane re-reads the matrix's first bytes
        if (beyond) { t = nstrips - 1; r = rounds - 1; }
        const int kb = t * 64 + wave * 4 + gl;
        const int kbc = kb < nbk64 ? kb : t * 64;
        const int n_t = min(64, nbk64 - t * 64);
        const int group = min(first + r * (int)gridDim.x, ngroups - 1);
        const int64_t row = min(group * 16 + il, rows - 1);
        if constexpr (KIND == KIND_Q3H) {                     // two planes of the strip, 16 bytes each
            const uint8_t *p0 = packed + row * ((int64_t)nbk64 * 32) + (int64_t)t * 2048 + (kbc & 63) * 16;
            const uint8_t *p1 = p0 + n_t * 16;
            if (beyond) { p0 = packed; p1 = packed; }
            const u32x4_t wa = *reinterpret_cast<const u32x4_t *>(p0);
            const u32x4_t wc = *reinterpret_cast<const u32x4_t *>(p1);
            raw.d[0] = wa.x; raw.d[1] = wa.y; raw.d[2] = wa.z; raw.d[3] = wa.w;
            raw.d[4] = wc.x; raw.d[5] = wc.y; raw.d[6] = wc.z; raw.d[7] = wc.w;
        } else if constexpr (kind_has_planes(KIND)) {         // low plane, high plane (each row-major over all rows), then the headers
            constexpr int ABYTES = 8 * WA, BBYTES = 8 * WB;   // bytes of a 64-weight block in each plane
            const uint8_t *pa = packed + row * ((int64_t)nbk64 * ABYTES) + (int64_t)kbc * ABYTES;
            const uint8_t *pb = packed + (int64_t)rows * nbk64 * ABYTES + row * ((int64_t)nbk64 * BBYTES) + (int64_t)kbc * BBYTES;
            if (beyond) { pa = packed; pb = packed; }
#pragma unroll
            for (int q = 0; q < ABYTES / 16; ++q) {
                const u32x4_t v = *reinterpret_cast<const u32x4_t *>(pa + (beyond ? 0 : q * 16));
                raw.d[4 * q] = v.x; raw.d[4 * q + 1] = v.y; raw.d[4 * q + 2] = v.z; raw.d[4 * q + 3] = v.w;
            }
            if constexpr (BBYTES == 16) {
                const u32x4_t v = *reinterpret_cast<const u32x4_t *>(pb);
                raw.d[2 * WA] = v.x; raw.d[2 * WA + 1] = v.y; raw.d[2 * WA + 2] = v.z; raw.d[2 * WA + 3] = v.w;
            } else if constexpr (BBYTES == 8) {
                const uint2 v = *reinterpret_cast<const uint2 *>(pb);
                raw.d[2 * WA] = v.x; raw.d[2 * WA + 1] = v.y;
            }
            const uint32_t *hp = reinterpret_cast<const uint32_t *>(packed + header_offset) + (beyond ? 0 : (row * nbk64 + kbc) * HPL);
#pragma unroll
            for (int h = 0; h < HPL; ++h) raw.hdr[h] = hp[h];
        } else {                                              // code bytes row-major, then the headers
            constexpr int BYTES = KIND == KIND_Q4 ? 32 : 64;
            if constexpr (LINES) {                            // load q: rows 4q .. 4q + 3
                int ln = lane;
                asm volatile("" : "+v"(ln));                  // (addresses worked out per step: the registers are needed in the rounds)
                const int kb_line = t * 64 + wave * 4 + (ln & 15) / 4;
                const uint8_t *line = packed + (int64_t)(kb_line < nbk64 ? kb_line : t * 64) * BYTES + (ln & 3) * 16;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int64_t row_q = min(group * 16 + q * 4 + (ln >> 4), rows - 1);
                    const u32x4_t v = *reinterpret_cast<const u32x4_t *>(beyond ? packed : line + row_q * ((int64_t)nbk64 * BYTES));
                    raw.d[4 * q] = v.x; raw.d[4 * q + 1] = v.y; raw.d[4 * q + 2] = v.z; raw.d[4 * q + 3] = v.w;
                }
            } else {
                const uint8_t *p0 = packed + row * ((int64_t)nbk64 * BYTES) + (int64_t)kbc * BYTES;
                if (beyond) p0 = packed;
#pragma unroll
                for (int q = 0; q < BYTES / 16; ++q) {
                    const u32x4_t v = *reinterpret_cast<const u32x4_t *>(p0 + (beyond ? 0 : q * 16));
                    raw.d[4 * q] = v.x; raw.d[4 * q + 1] = v.y; raw.d[4 * q + 2] = v.z; raw.d[4 * q + 3] = v.w;
                }
            }
            const uint32_t *hp = reinterpret_cast<const uint32_t *>(packed + header_offset) + (beyond ? 0 : (row * nbk64 + kbc) * HPL);
#pragma unroll
            for (int h = 0; h < HPL; ++h) raw.hdr[h] = hp[h];
        }
    };

    const half2_t m1025 = {(half_t)-1025.0f, (half_t)-1025.0f}, m1024 = {(half_t)-1024.0f, (half_t)-1024.0f};
    const half2_t m11 = {(half_t)-11.0f, (half_t)-11.0f};
    DecodeConstants constants;
    constants.open();
    half8_t xq[8];                                            // MFMA B operands of the current strip
    float ssq[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};  // (rms normalization) this lane's share of sum x^2 of the eight vectors it loads
    float *ssq_lds = reinterpret_cast<float *>(lds + SMALL_LDS_BYTES);                // [wavefront][vector]
    auto join = [](half2_t a, half2_t b, half2_t c, half2_t e) {
        return __builtin_bit_cast(half8_t, (u32x4_t){as_u32(a), as_u32(b), as_u32(c), as_u32(e)});
    };

    // one round: dequantize the lane's block, eight MFMA steps (on top of the earlier strips'), the tile to its slot
    auto round_body = [&](const SmallRaw<KIND> &raw, int slot, bool onto) {
        uint32_t d[NWORDS], hdr[2];
        if constexpr (LINES) {
            int ln = lane;
            asm volatile("" : "+v"(ln));
#pragma unroll
            for (int q = 0; q < 4; ++q) *turned(q * 4 + (ln >> 4), ln & 15) = (u32x4_t){raw.d[4 * q], raw.d[4 * q + 1], raw.d[4 * q + 2], raw.d[4 * q + 3]};
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();                  // (the wavefront's own rows: its LDS operations are served in order)
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const u32x4_t v = *turned(ln & 15, (ln >> 4) * 4 + q);
                d[4 * q] = v.x; d[4 * q + 1] = v.y; d[4 * q + 2] = v.z; d[4 * q + 3] = v.w;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();                  // the next round overwrites them
        } else {
#pragma unroll
            for (int w = 0; w < NWORDS; ++w) d[w] = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)raw.d[w]);
        }
        if (KIND != KIND_Q3H) {
#pragma unroll
            for (int h = 0; h < HPL; ++h) hdr[h] = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)raw.hdr[h]);
        }
        float4_t acc = {0.f, 0.f, 0.f, 0.f};
        if (onto) acc = *reinterpret_cast<const float4_t *>(mine + slot * (16 * SMALL_TILE));
        if constexpr (KIND == KIND_Q3H) {
            uint32_t h = d[0] & 0xC000C000u;                  // header from the spare bits of the eight words
#pragma unroll
            for (int w = 1; w < 8; ++w) h = (d[w] & 0xC000C000u) | (h >> 2);
            const half2_t so = as_h2(h);
            const half2_t s2 = {so.x, so.x}, o2 = {so.y, so.y};
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                half2_t wv[4];
#pragma unroll
                for (int hs = 0; hs < 2; ++hs) {              // slot s = 2w + hs: weights 4s .. 4s+3
                    const uint32_t hc = and_or(d[w] >> (7 * hs), 0x007F007Fu, constants.at0);
                    const half2_t q1 = q3h_high_digit(hc) + m1025;                    // floor(c/11), exact
                    const half2_t c = as_h2(hc) + m1024;                              // c, exact
                    const half2_t q2 = __builtin_elementwise_fma(q1, m11, c);         // c mod 11, exact
                    wv[2 * hs] = __builtin_elementwise_fma(q1, s2, o2);               // (w[4s], w[4s+2])   Eq.2, one rounding
                    wv[2 * hs + 1] = __builtin_elementwise_fma(q2, s2, o2);           // (w[4s+1], w[4s+3])
                }
                acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(join(wv[0], wv[1], wv[2], wv[3]), xq[w], acc, 0, 0, 0);
            }
        } else if constexpr (kind_has_planes(KIND) || KIND == KIND_Q4) {
            // eight weights at a time: the level's bits of both planes next to each other in an fp16 mantissa, then Eq.2
            constexpr int LA = KIND == KIND_Q4 ? 4 : WA, LB = KIND == KIND_Q4 ? 0 : WB;
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                const half2_t so = as_h2(hdr[HPL == 2 ? w >> 2 : 0]);
                const half2_t s2 = {so.x, so.x}, o2 = {so.y, so.y};
                const uint32_t lo = LA == 4 ? d[w] : d[w >> 1] >> (8 * (w & 1));
                const uint32_t hi = LB == 0 ? 0u : LB == 2 ? d[2 * LA + (w >> 1)] >> (8 * (w & 1)) : d[2 * LA + (w >> 2)] >> (4 * (w & 3));
                half2_t wv[4];
#pragma unroll
                for (int p = 0; p < 4; ++p) wv[p] = __builtin_elementwise_fma(plane_level<LA, LB>(lo, lo >> 8, hi, p, constants), s2, o2);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(join(wv[0], wv[1], wv[2], wv[3]), xq[w], acc, 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int w = 0; w < 8; ++w) {                     // words 2w, 2w + 1: bytes = weights 8w .. 8w+7
                const half2_t so = as_h2(hdr[HPL == 2 ? w >> 2 : 0]);
                const half2_t s2 = {so.x, so.x}, o2 = {so.y, so.y};
                half2_t wv[4];
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    wv[p] = __builtin_elementwise_fma(as_h2(__builtin_amdgcn_perm(0x64646464u, d[2 * w + (p >> 1)], p & 1 ? 0x04030402u : 0x04010400u)) + m1024, s2, o2);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(join(wv[0], wv[1], wv[2], wv[3]), xq[w], acc, 0, 0, 0);
            }
        }
        *reinterpret_cast<float4_t *>(mine + slot * (16 * SMALL_TILE)) = acc;      // register e of lane (j, g') is D[4g' + e][j]
    };

    // activations of strip t: batch rows x the wavefront's 256 columns -> lane (j, g) holds row j, columns 64g .. 64g+63
    auto stage = [&](int t) {
        int ln = lane;
        if constexpr (TIGHT) asm volatile("" : "+v"(ln));     // (addresses worked out per strip: the registers are needed in the rounds)
        const int kb = t * 64 + wave * 4 + g;
        const bool live = kb < nbk64;                         // ragged last strip: dead lanes add nothing (their activations are zeroed)
        int c = (t * 64 + wave * 4) * 64 + (ln & 31) * 8;
        if (c >= cols) c = 0;                                 // columns past the end: any valid address, the values are masked below
        // (uniform; where a module's arithmetic comes between the loads and the turn a constant is no better: silu up to 7 % slower, rms with sixteen
        // vectors up to 3 %)
        const bool upper = XOP == IFLOW_X_SILU_MUL || (XOP == IFLOW_X_RMS_GAIN && UPPER) ? batch > 8 : UPPER;
        u32x4_t va[4], vb[4] = {};                             // load q: batch rows 2q and 2q+1 (vb: 8+2q, 9+2q), 512 bytes each, lane by lane
#pragma unroll
        for (int q = 0; q < 4; ++q)
            va[q] = *reinterpret_cast<const u32x4_t *>(X + (int64_t)min(2 * q + (ln >> 5), batch - 1) * cols + c);
        if (upper)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                vb[q] = *reinterpret_cast<const u32x4_t *>(X + (int64_t)min(8 + 2 * q + (ln >> 5), batch - 1) * cols + c);
        if constexpr (XOP == IFLOW_X_RMS_GAIN) {
            // the lane's eight columns of every vector it loaded: x^2 summed (columns past the end and dead column groups
            // were redirected to column 0: they do not count), then v = fp16(x g), an exact product rounded once
            const bool counts = (t * 64 + wave * 4) * 64 + (ln & 31) * 8 < cols;
            const u32x4_t gv = *reinterpret_cast<const u32x4_t *>(ops.aux + c);
            const uint32_t gw[4] = {gv.x, gv.y, gv.z, gv.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t xa[4] = {va[q].x, va[q].y, va[q].z, va[q].w}, xb[4] = {vb[q].x, vb[q].y, vb[q].z, vb[q].w};
                float sa = 0.f, sb = 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    sa = __builtin_amdgcn_fdot2(as_h2(xa[e]), as_h2(xa[e]), sa, false);
                    xa[e] = as_u32(as_h2(xa[e]) * as_h2(gw[e]));
                    if constexpr (UPPER) {                    // (of zeros where there are no more than eight vectors)
                        sb = __builtin_amdgcn_fdot2(as_h2(xb[e]), as_h2(xb[e]), sb, false);
                        xb[e] = as_u32(as_h2(xb[e]) * as_h2(gw[e]));
                    }
                }
                ssq[q] += counts ? sa : 0.f;
                ssq[4 + q] += counts ? sb : 0.f;
                va[q] = (u32x4_t){xa[0], xa[1], xa[2], xa[3]};
                vb[q] = (u32x4_t){xb[0], xb[1], xb[2], xb[3]};
            }
            if (t == nstrips - 1) {
                // vector 2q + (ln >> 5) (and 8 + ...) over the wavefront's lanes: sum within each half of the wavefront
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    float v = row16_sum(ssq[q]);
                    v += __shfl_xor(v, 16);
                    if ((ln & 31) == 0) ssq_lds[wave * 16 + (q < 4 ? 2 * q : 8 + 2 * (q - 4)) + (ln >> 5)] = v;
                    ssq[q] = 0.f;
                }
            }
        } else if constexpr (XOP == IFLOW_X_SILU_MUL) {
            // v = fp16(silu(x) aux) in fp32 with the hardware exp and reciprocal, one rounding
            auto gate = [&](u32x4_t &v, int brow) {
                const u32x4_t av = *reinterpret_cast<const u32x4_t *>(ops.aux + (int64_t)min(brow, batch - 1) * cols + c);
                uint32_t xv[4] = {v.x, v.y, v.z, v.w};
                const uint32_t aw[4] = {av.x, av.y, av.z, av.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const half2_t xa = as_h2(xv[e]), xb = as_h2(aw[e]);
                    const float g0 = (float)xa.x, g1 = (float)xa.y;
                    const float v0 = g0 * __builtin_amdgcn_rcpf(1.0f + __expf(-g0)) * (float)xb.x;
                    const float v1 = g1 * __builtin_amdgcn_rcpf(1.0f + __expf(-g1)) * (float)xb.y;
                    const half2_t rv = {(half_t)v0, (half_t)v1};
                    xv[e] = as_u32(rv);
                }
                v = (u32x4_t){xv[0], xv[1], xv[2], xv[3]};
            };
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                // (uniform: the gate is most of a strip's work - with the staging below, two vectors, 4096 x 11008 4-bit 16.7 -> 9.9 us, nine, 1077 x 10432 8-bit 24.4 -> 18.2)
                if (2 * q < batch) gate(va[q], 2 * q + (ln >> 5));
                if (upper && 8 + 2 * q < batch) gate(vb[q], 8 + 2 * q + (ln >> 5));
            }
        }
        uint32_t n[32];
        auto turn = [&](const u32x4_t (&v)[4], bool mine) {     // eight batch rows through the staging rows
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<u32x4_t *>(xst + (2 * q + (ln >> 5)) * SMALL_XROW + (ln & 31) * 16) = v[q];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (mine) {
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const u32x4_t u = *reinterpret_cast<const u32x4_t *>(xst + (i & 7) * SMALL_XROW + g * 128 + q * 16);
                    n[4 * q] = u.x; n[4 * q + 1] = u.y; n[4 * q + 2] = u.z; n[4 * q + 3] = u.w;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();                  // the next turn overwrites the staging rows
        };
        // (Up to eight vectors: lanes 8 .. 15 of a group hold the first eight again, their columns of the result are not stored.  A lane reads the half that
        // is its own, instead of both with a select per register, and the zeros for dead column groups are made only where there are some: 190 -> 90
        // vector instructions a strip next to 150 to 220 of a step's decode; us, before -> after, 8 vectors with a residual: 4096 x 4096 4-bit 5.15 -> 4.6, 4096 x 11008
        // 8-bit 13.3 -> 12.8, 11008 x 4096 3.5-bit with rms 9.5 -> 9.05 (10.6 -> 10.2 on another machine), 1627 x 17280 6-bit 15.0 -> 14.25.  Requesting the next
        // strip's activations a strip ahead gave nothing at up to eight vectors and spilled at sixteen: the wavefronts of a SIMD fill each other's waits.)
        turn(va, !upper || i < 8);
        if (upper) turn(vb, i >= 8);
        // MFMA B operands: the eight activations of step w.  Q3H's decoder yields weights in the order (4s, 4s+2, 4s+1, 4s+3).
        const uint32_t keep = live ? 0xFFFFFFFFu : 0u;
        const bool ragged = t * 64 + wave * 4 + 4 > nbk64;     // (uniform: some of the wavefront's column groups are dead)
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            uint32_t v[4];
#pragma unroll
            for (int hs = 0; hs < 2; ++hs) {
                const uint32_t a0 = n[4 * w + 2 * hs], a1 = n[4 * w + 2 * hs + 1];
                v[2 * hs] = KIND == KIND_Q3H ? __builtin_amdgcn_perm(a1, a0, 0x05040100u) : a0;        // (x[4s], x[4s+2])
                v[2 * hs + 1] = KIND == KIND_Q3H ? __builtin_amdgcn_perm(a1, a0, 0x07060302u) : a1;    // (x[4s+1], x[4s+3])
            }
            xq[w] = __builtin_bit_cast(half8_t, (u32x4_t){v[0], v[1], v[2], v[3]});
        }
        if (ragged)
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                const u32x4_t v = __builtin_bit_cast(u32x4_t, xq[w]);
                xq[w] = __builtin_bit_cast(half8_t, (u32x4_t){v.x & keep, v.y & keep, v.z & keep, v.w & keep});
            }
    };
    // The sums over the wavefronts, in a fixed order, once per batch of rounds (`slots` of them, from round r0 of strip t on): between two of these the
    // wavefronts run freely.  1024 threads: round tid / 256 of the batch, vector tid / 16 % 16, row tid % 16 of the round's sixteen.
    auto finish = [&](int t, int r0, int slots, bool more) {
        int tid = threadIdx.x;
        if constexpr (TIGHT) asm volatile("" : "+v"(tid));    // (worked out here each time: the registers are needed in the rounds)
        const int rl = tid >> 8, b = (tid >> 4) & 15, row16 = tid & 15;
        const int rr = (first + (r0 + rl) * (int)gridDim.x) * 16 + row16;
        const bool stores = rl < slots && rr < rows && b < batch && t + 1 == nstrips;
        const int64_t at = stores ? (int64_t)b * rows + rr : 0;
        float res = 0.f;
        if constexpr (XOP >= 0) {                             // (requested in front of the barrier)
            if (stores && ops.residual != nullptr) res = (float)as_h(ops.residual[at]);
        }
        __syncthreads();
        if (rl < slots) {
            const float *tile = reinterpret_cast<const float *>(lds + SMALL_XBYTES) + rl * (16 * SMALL_TILE) + (row16 >> 2) * 80 + b * 4 + (row16 & 3);
            float *running = part + (r0 + rl) * 256 + (tid & 255);
            float sum = t > 0 && !carry ? *running : 0.f;
#pragma unroll
            for (int w = 0; w < 16; ++w) sum += tile[w * SMALL_TILE];
            if (t + 1 < nstrips) {
                *running = sum;
            } else {
                if constexpr (XOP == IFLOW_X_RMS_GAIN) {      // the vector's normalization scalar: the wavefronts' shares in a fixed order
                    float tot = 0.f;
#pragma unroll
                    for (int w = 0; w < 16; ++w) tot += ssq_lds[w * 16 + b];
                    sum *= 1.0f / __builtin_sqrtf(tot / (float)cols + ops.eps);
                }
                if constexpr (XOP >= 0) sum += res;
                if (stores) Y[at] = as_u16((half_t)sum);
            }
        }
        if (more) __syncthreads();                            // the next batch overwrites the tiles
    };
    // (t, r) of the step `ahead` (<= S) steps after (t, r)
    auto step_after = [&](int t, int r, int ahead, int &t2, int &r2) {
        t2 = t; r2 = r + ahead;
#pragma unroll
        for (int q = 0; q < S; ++q)
            if (r2 >= rounds) { r2 -= rounds; ++t2; }
    };

    // Steps (strip, round) in order, S per trip through S register sets; a set is refilled for S steps ahead right
    // after its use.  The last trips, where some steps or refills no longer exist, run through a guarded copy of the
    // loop body so that the main loop has no load of weights under a branch (the wait counters stay exact there) and nothing is
    // requested that is not used (a wavefront ends only when its last load has returned).
    SmallRaw<KIND> raw[S];
    int t = 0, r = 0, slot = 0, t2, r2;
#pragma unroll
    for (int j = 0; j < S; ++j) {
        step_after(0, 0, j, t2, r2);
        load_step(raw[j], t2, r2);
    }
    int k = 0;
    for (; k + 2 * S - 1 < total; k += S) {
#pragma unroll
        for (int j = 0; j < S; ++j) {
            if (r == 0) stage(t);
            round_body(raw[j], slot, carry && t > 0);
            step_after(t, r, S, t2, r2);
            load_step(raw[j], t2, r2);
            if (++slot == per_batch || r + 1 == rounds) {
                if (!carry || t + 1 == nstrips) finish(t, r + 1 - slot, slot, true);
                slot = 0;
            }
            step_after(t, r, 1, t, r);
        }
    }
    for (; k < total; k += S) {
#pragma unroll
        for (int j = 0; j < S; ++j) {
            if (k + j < total) {                              // (uniform over the workgroup)
                if (r == 0) stage(t);
                round_body(raw[j], slot, carry && t > 0);
                if (k + j + S < total) {
                    step_after(t, r, S, t2, r2);
                    load_step(raw[j], t2, r2);
                }
                if (++slot == per_batch || r + 1 == rounds) {
                    if (!carry || t + 1 == nstrips) finish(t, r + 1 - slot, slot, k + j + 1 < total);
                    slot = 0;
                }
                step_after(t, r, 1, t, r);
            }
        }
    }
}

template <int F, int S, bool UPPER, bool LINES>
__global__ __launch_bounds__(1024) void gemm_small_kernel(const uint8_t *__restrict__ packed, const uint16_t *__restrict__ X,
                                                          uint16_t *__restrict__ Y, int rows, int cols, int batch, int nbk64, int nstrips,
                                                          int64_t header_offset, int group0, int ngroups)
{
    gemm_small_body<F, S, -1, UPPER, LINES>(packed, X, Y, rows, cols, batch, nbk64, nstrips, header_offset, group0, ngroups, SmallOps{});
}

template <int F, int S, int XOP, bool UPPER, bool LINES>
__global__ __launch_bounds__(1024) void gemm_small_fused_kernel(const uint8_t *__restrict__ packed, const uint16_t *__restrict__ X,
                                                                uint16_t *__restrict__ Y, int rows, int cols, int batch, int nbk64, int nstrips,
                                                                int64_t header_offset, int group0, int ngroups, const SmallOps ops)
{
    gemm_small_body<F, S, XOP, UPPER, LINES>(packed, X, Y, rows, cols, batch, nbk64, nstrips, header_offset, group0, ngroups, ops);
}

template <int F, int XOP, bool UPPER, bool LINES>
static hipError_t small_go(const void *packed, int64_t rows, int64_t cols, const uint16_t *X, int64_t batch, uint16_t *Y, const SmallOps ops,
                               hipStream_t s)
{
    typedef Fmt<F> T;
    constexpr int S = SMALL_SETS;
    constexpr int LDS = XOP < 0 ? SMALL_LDS_BYTES : SMALL_LDS_BYTES_OPS;
    static PerDevice pd;
    int cus = 0;
    hipError_t e0 = once_per_device(pd, &cus, [] {
        if constexpr (XOP < 0)
            return hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_small_kernel<F, S, UPPER, LINES>), hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        else
            return hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_small_fused_kernel<F, S, XOP, UPPER, LINES>), hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    });
    if (e0 != hipSuccess) return e0;
    const int nbk64 = (int)(cols / 64);
    const int nstrips = (nbk64 + 63) / 64;
    const int64_t header_offset = rows * (cols / T::block) * (int64_t)T::code_bytes;
    const int64_t ngroups = (rows + 15) / 16;
    if (ngroups > 0x7FFFFFF || rows > 0x7FFFFFFF) return hipErrorInvalidValue;
    // rows spanning several strips keep a running sum per round in LDS: at most SMALL_MAX_ROUNDS rounds per launch then
    const int64_t per_launch = nstrips > 1 ? (int64_t)cus * SMALL_MAX_ROUNDS : ngroups;
    for (int64_t g0 = 0; g0 < ngroups; g0 += per_launch) {
        const int64_t g1 = g0 + per_launch < ngroups ? g0 + per_launch : ngroups;
        const int64_t grid = g1 - g0 < cus ? g1 - g0 : cus;
        if constexpr (XOP < 0)
            hipLaunchKernelGGL((gemm_small_kernel<F, S, UPPER, LINES>), dim3((unsigned)grid), dim3(1024), LDS, s,
                               static_cast<const uint8_t *>(packed), X, Y, (int)rows, (int)cols, (int)batch, nbk64, nstrips, header_offset,
                               (int)g0, (int)g1);
        else
            hipLaunchKernelGGL((gemm_small_fused_kernel<F, S, XOP, UPPER, LINES>), dim3((unsigned)grid), dim3(1024), LDS, s,
                               static_cast<const uint8_t *>(packed), X, Y, (int)rows, (int)cols, (int)batch, nbk64, nstrips, header_offset,
                               (int)g0, (int)g1, ops);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int F, int XOP, bool UPPER>
static hipError_t small_lines(const void *packed, int64_t rows, int64_t cols, const uint16_t *X, int64_t batch, uint16_t *Y, const SmallOps ops,
                              hipStream_t s)
{
    if constexpr (Fmt<F>::kind == KIND_Q8)
        if (cols > SMALL_LINES_COLS) return small_go<F, XOP, UPPER, true>(packed, rows, cols, X, batch, Y, ops, s);
    return small_go<F, XOP, UPPER, false>(packed, rows, cols, X, batch, Y, ops, s);
}

template <int F, int XOP>
static hipError_t small_launch(const void *packed, int64_t rows, int64_t cols, const uint16_t *X, int64_t batch, uint16_t *Y, const SmallOps ops,
                               hipStream_t s)
{
    if constexpr (XOP == IFLOW_X_SILU_MUL) return small_lines<F, XOP, true>(packed, rows, cols, X, batch, Y, ops, s);
    return batch > 8 ? small_lines<F, XOP, true>(packed, rows, cols, X, batch, Y, ops, s) : small_lines<F, XOP, false>(packed, rows, cols, X, batch, Y, ops, s);
}

hipError_t launch_qgemm_small(int format, const void *packed, int64_t rows, int64_t cols,
                              const uint16_t *X, int64_t batch, uint16_t *Y, hipStream_t s)
{
    if (batch < 1 || batch > 16 || cols % 64 != 0) return hipErrorInvalidValue;
    return for_format(format, [&](auto f) { return small_launch<decltype(f)::value, -1>(packed, rows, cols, X, batch, Y, SmallOps{}, s); });
}

hipError_t launch_qgemm_small_fused(int format, const void *packed, int64_t rows, int64_t cols, const uint16_t *X, int64_t batch, int x_op,
                                    const uint16_t *aux, float eps, const uint16_t *residual, uint16_t *Y, hipStream_t s)
{
    if (batch < 1 || batch > 16 || cols % 64 != 0) return hipErrorInvalidValue;
    const SmallOps ops = {aux, residual, eps};
    return for_format(format, [&](auto f) {
        constexpr int F = decltype(f)::value;
        switch (x_op) {
        case IFLOW_X_PLAIN: return small_launch<F, IFLOW_X_PLAIN>(packed, rows, cols, X, batch, Y, ops, s);
        case IFLOW_X_RMS_GAIN: return small_launch<F, IFLOW_X_RMS_GAIN>(packed, rows, cols, X, batch, Y, ops, s);
        case IFLOW_X_SILU_MUL: return small_launch<F, IFLOW_X_SILU_MUL>(packed, rows, cols, X, batch, Y, ops, s);
        default: return hipErrorInvalidValue;
        }
    });
}

}  // namespace iflow
