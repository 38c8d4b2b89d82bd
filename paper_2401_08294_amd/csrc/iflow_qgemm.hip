// Dequantize-and-multiply on the matrix cores for 17 and more activation vectors: Y[b][n] = sum_k w'[n][k] X[b][k].
//
// A wavefront owns RT x 32 weight rows and MB x 32 vectors and walks along K in chunks of 64 columns (one quantization block per
// weight row, two for the 32-wide formats) with v_mfma_f32_32x32x16_f16.  It decodes its weights - Eq.5 and Eq.2 of the paper with the
// single-rounded fp16 fused multiply-add, exactly the values iflow_dequant produces - from packed bytes straight into operand
// registers: nobody else needs these rows, so decoded weights never go through LDS.  The activations do: WR wavefronts side by side
// along the rows share them.  WK such groups split K among them, where rows x vectors alone give too few wavefronts.
//   - Everything comes from memory by copies straight into LDS, several steps ahead, and is waited for by count: no registers are
//     held by loads in flight, and a step's matrix instructions never wait for memory (before, one 64-column chunk took 530 ns for
//     256 cycles of matrix work).
//   - The operands of a k-step of 16 columns are read and decoded while the matrix instructions of the k-step before run.
//   - Which lane holds which k of a chunk is free as long as both operands agree: lane half h takes columns 32 h .. 32 h + 31,
//     so that a lane's weights are 32 consecutive ones of one row.
// What bounds it, by counters: at 2000 vectors (28672 x 8192, 4-bit) the matrix cores are busy 65 % of the cycles of a launch that runs at 1.4 to 1.6 GHz - the power
// limit, a loop of nothing but these instructions on random data runs at 1.5 to 1.8 - next to a decode that issues 28 % of them, which is why
// the largest tile has 256 vectors per decoded weight; at 512 (11008 x 4096, 3.5-bit, three wavefronts per SIMD, 1.7 GHz) both are busy 43 to 44 % of the time; at 33
// (4096 x 11008, 8-bit) wavefronts wait for their copies.
// Measured, us (before: 128 x 64 tiles with both operands decoded or copied into LDS, passes of sixteen below 32 vectors), one matrix again and again:
// 11008 x 4096 3.5-bit, 512 vectors 84.4 -> 50 to 51 (910 TFLOP/s; over a ring of matrices beyond the caches more); 28672 x 8192 4-bit, 2000 vectors 1491 -> 817 to 831 by machine (1130 to
// 1150 TFLOP/s); 4096 x 11008 8-bit, 33 vectors 49.7 -> 17.4 (ring 23); 4096 x 4096 3.5-bit, 64 vectors 23.8 -> 8.0 (ring 9.6).
#include "iflow_common.h"

namespace iflow {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float16_t __attribute__((ext_vector_type(16)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef u32x4_t u32x4_any_t __attribute__((aligned(2)));        // 16 bytes at any fp16 address

__device__ __forceinline__ uint32_t pack_h2(half2_t v) { return as_u32(v); }

// N (16 or 4) bytes per lane from memory straight into LDS: lane l's to lds + N l.  Written out because the compiler, which cannot
// tell which LDS reads such a copy may overlap, puts a wait for all of them in front of the next read; the waits are placed by hand.
// (m0, the copy's LDS address, is a reserved register: it cannot be named as clobbered, and nothing else in these kernels uses it.)
template <int N>
__device__ __forceinline__ void copy_to_lds(const uint8_t *base /* wavefront-uniform */, uint32_t offset, uint32_t lds)
{
    if constexpr (N == 16)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(offset), "s"(base) : "memory");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds), "v"(offset), "s"(base) : "memory");
}

// ---- packed weights of 32 rows: memory -> LDS -> registers -----------------------------------------------------------------
// A 64-column chunk of a row is, per format, one to three runs of consecutive bytes ("parts": the low or only plane's codes, the high
// plane's, the headers; the 3.5-bit format: its two planes).  Parts of G consecutive chunks of a row are consecutive too, so a
// wavefront fetches 32 rows x G chunks at once, with neighbouring lanes on neighbouring pieces of a row: segments of 64 bytes and
// more where G is 4, 2 or 1 by the format's width and the LDS that the tile leaves.  (One 16-byte piece per row and instruction - 64 cache lines each - cost a fifth of
// the whole kernel.)
template <int F, int G_ = 1> struct Parts {
    typedef Fmt<F> T;
    static constexpr bool q3h = T::kind == KIND_Q3H, planes = kind_has_planes(T::kind);
    static constexpr int WA = T::kind == KIND_Q8 ? 8 : planes ? Planes<T::kind>::WA : 4, WB = planes ? Planes<T::kind>::WB : 0;   // bits
    static constexpr int A = q3h ? 16 : 8 * WA, B = q3h ? 16 : 8 * WB, H = q3h ? 0 : 256 / T::block;   // bytes of a row's chunk per part
    static constexpr int G = G_;
    static constexpr int PB = B == 8 ? 4 : 16;                 // bytes per lane and piece (8 bytes a chunk: rows are only 8-byte aligned)
    static constexpr int NA = 32 * G * A / 1024, NB = 32 * G * B / (64 * PB), NH = (32 * G * H + 255) / 256;   // pieces (instructions) per part
    static constexpr int LA = 0, LB = 32 * G * A, LH = LB + 32 * G * B, BYTES = LH + 256 * NH;         // places in LDS, total
    static constexpr int BUFFERS = G == 1 ? 3 : 2;             // groups of G chunks in LDS: the one in use and those on their way
};

// One lane's 32 weights of a row: half h of a chunk.
template <int F> struct RawHalf { uint32_t a[Parts<F>::WA], b[Parts<F>::WB ? Parts<F>::WB : 1], hdr; };

template <int F, int G> struct WeightRows {
    typedef Fmt<F> T;
    typedef Parts<F, G> P;
    const uint8_t *a, *b, *hdr;                                // row r0's start in each part (wavefront-uniform)
    uint32_t ra, rb, rh;                                       // bytes of a row in each part
    int last;                                                  // rows past the matrix's end: row r0 + last again
    int nchunks, lane;
    __device__ __forceinline__ void open(const uint8_t *packed, int rows, int cols, int64_t header_offset, int r0, int l)
    {
        ra = (uint32_t)cols / 64u * (P::q3h ? 32 : P::A); rb = (uint32_t)cols / 64u * P::B; rh = (uint32_t)cols / 64u * P::H;
        a = packed + (int64_t)r0 * ra;
        b = packed + (int64_t)rows * ra + (int64_t)r0 * rb;
        hdr = packed + header_offset + (int64_t)r0 * rh;
        last = rows - 1 - r0; nchunks = cols / 64; lane = l;
    }
    // piece i of a part with `per` bytes a chunk, `each` bytes a lane: the lane's row and byte in that row's G chunks.  The 16-byte
    // slots of a row are permuted by the row, so that 16-byte reads of neighbouring rows' same chunk fall into different banks.
    template <int PER, int EACH> __device__ __forceinline__ void place(int i, int &row, int &byte) const
    {
        constexpr int LANES = G * PER / EACH;                  // lanes per row
        row = ((i * 64 + lane) / LANES) & 31;                  // (a piece of 32 rows x 4 bytes fills half the lanes: the rest repeat)
        const int slot = lane % LANES;
        byte = (EACH == 16 ? slot ^ spread<LANES>(row) : slot) * EACH;
    }
    template <int LANES> static __device__ __forceinline__ int spread(int row)
    {
        return row / (16 / LANES) & (LANES - 1);               // 256 bytes, one turn of the banks, hold 16 / LANES rows
    }
    // chunks kc .. kc + G - 1 (kc a multiple of G, wavefront-uniform) of rows r0 + 32 t .. + 31 -> LDS; chunks past the end: the
    // row's last bytes again
    __device__ __forceinline__ void request(int t, int kc, uint32_t lds) const
    {
        int row, byte;
        if constexpr (P::q3h) {
            const int strip = kc >> 6, n_t = min(64, nchunks - (strip << 6)), in = (kc & 63) * 16;
#pragma unroll
            for (int pl = 0; pl < 2; ++pl)
#pragma unroll
                for (int i = 0; i < P::NA; ++i) {
                    place<16, 16>(i, row, byte);
                    const int at = min(in + byte, (n_t - 1) * 16);
                    copy_to_lds<16>(a + strip * 2048 + pl * (n_t * 16), (uint32_t)min(32 * t + row, last) * ra + at, lds + (pl ? P::LB : P::LA) + 1024 * i);
                }
        } else {
#pragma unroll
            for (int i = 0; i < P::NA; ++i) {
                place<P::A, 16>(i, row, byte);
                copy_to_lds<16>(a, (uint32_t)min(32 * t + row, last) * ra + min(kc * P::A + byte, (int)ra - 16), lds + P::LA + 1024 * i);
            }
            if constexpr (P::B > 0) {
#pragma unroll
                for (int i = 0; i < P::NB; ++i) {
                    place<P::B, P::PB>(i, row, byte);
                    copy_to_lds<P::PB>(b, (uint32_t)min(32 * t + row, last) * rb + min(kc * P::B + byte, (int)rb - P::PB), lds + P::LB + 64 * P::PB * i);
                }
            }
#pragma unroll
            for (int i = 0; i < P::NH; ++i) {
                place<P::H, 4>(i, row, byte);
                copy_to_lds<4>(hdr, (uint32_t)min(32 * t + row, last) * rh + min(kc * P::H + byte, (int)rh - 4), lds + P::LH + 256 * i);
            }
        }
    }
    template <int PER, int LANE_BYTES> static __device__ __forceinline__ const uint8_t *slot_of(const uint8_t *lds, int row, int byte)
    {
        constexpr int LANES = G * PER / LANE_BYTES;
        if constexpr (LANE_BYTES == 16) return lds + row * (G * PER) + (((byte >> 4) ^ spread<LANES>(row)) << 4) + (byte & 15);
        else return lds + row * (G * PER) + byte;
    }
    // ... and half h of chunk c of the group, row `row` of the 32, from there into registers
    static __device__ __forceinline__ void read(const uint8_t *lds, int row, int c, int h, RawHalf<F> &r)
    {
        if constexpr (P::q3h) {
            const u32x4_t v = *reinterpret_cast<const u32x4_t *>(slot_of<16, 16>(lds + (h ? P::LB : P::LA), row, c * 16));
            r.a[0] = v.x; r.a[1] = v.y; r.a[2] = v.z; r.a[3] = v.w;
        } else if constexpr (P::WA == 2) {
            const u32x2_t v = *reinterpret_cast<const u32x2_t *>(slot_of<P::A, 16>(lds + P::LA, row, c * 16 + h * 8));
            r.a[0] = v.x; r.a[1] = v.y;
        } else {
#pragma unroll
            for (int i = 0; i < P::WA / 4; ++i) {
                const u32x4_t v = *reinterpret_cast<const u32x4_t *>(slot_of<P::A, 16>(lds + P::LA, row, c * P::A + h * (P::A / 2) + i * 16));
                r.a[4 * i] = v.x; r.a[4 * i + 1] = v.y; r.a[4 * i + 2] = v.z; r.a[4 * i + 3] = v.w;
            }
        }
        if constexpr (!P::q3h && P::WB == 2) {
            const u32x2_t v = *reinterpret_cast<const u32x2_t *>(slot_of<P::B, 16>(lds + P::LB, row, c * 16 + h * 8));
            r.b[0] = v.x; r.b[1] = v.y;
        }
        if constexpr (P::WB == 1) r.b[0] = *reinterpret_cast<const uint32_t *>(slot_of<P::B, 4>(lds + P::LB, row, c * 8 + h * 4));
        if constexpr (P::H > 0) r.hdr = *reinterpret_cast<const uint32_t *>(slot_of<P::H, 4>(lds + P::LH, row, c * P::H + (T::block == 32 ? h * 4 : 0)));
    }
};

// Eq.5 and Eq.2 for eight of the 32 weights at a time (k-step ks: weights 8 ks .. 8 ks + 7), as fp16 in natural order, bit-identical
// to iflow_dequant.
template <int F> struct HalfDecoder {
    typedef Fmt<F> T;
    typedef RawHalf<F> R;
    typedef Parts<F> P;
    half2_t s2, o2;
    DecodeConstants k;
    __device__ __forceinline__ void open(const R &r, const DecodeConstants &constants, int h)
    {
        k = constants;
        uint32_t hdr = 0;
        if constexpr (T::kind == KIND_Q3H) {
            // word wi of the block carries scale bits 2wi, 2wi+1 at 14-15 and offset bits at 30-31: the four words of this half
            // shift theirs into bits 8-15 and 24-31, the lower half of the block belongs eight bits further down, and the
            // lane 32 apart holds the other half
            uint32_t g = r.a[0] & 0xC000C000u;
#pragma unroll
            for (int i = 1; i < 4; ++i) g = (g >> 2) | (r.a[i] & 0xC000C000u);
            g >>= h ? 0 : 8;
            const auto sw = __builtin_amdgcn_permlane32_swap(g, g, false, false);
            hdr = sw[0] | sw[1];
        } else {
            hdr = r.hdr;
        }
        const half2_t so = as_h2(hdr);
        s2 = (half2_t){so.x, so.x}; o2 = (half2_t){so.y, so.y};
    }
    __device__ __forceinline__ half8_t step(const R &r, int ks) const
    {
        const half2_t m1024 = {(half_t)-1024.0f, (half_t)-1024.0f};
        half2_t lv[4];
        if constexpr (T::kind == KIND_Q3H) {
            const half2_t m1025 = {(half_t)-1025.0f, (half_t)-1025.0f}, m11 = {(half_t)-11.0f, (half_t)-11.0f};
            uint32_t out[4];
#pragma unroll
            for (int hsel = 0; hsel < 2; ++hsel) {
                // two pair codes in the two halves of a register: (4i, 4i+1) at bits 0/16, (4i+2, 4i+3) at bits 7/23
                const uint32_t hc = and_or(r.a[ks] >> (7 * hsel), 0x007F007Fu, k.at0);
                const half2_t q1 = q3h_high_digit(hc) + m1025;                       // floor(c/11), exact
                const half2_t c = as_h2(hc) + m1024;                                 // c, exact
                const half2_t q2 = __builtin_elementwise_fma(q1, m11, c);            // c - 11 q1 = c mod 11, exact
                const half2_t w1 = __builtin_elementwise_fma(q1, s2, o2);            // (w[4m], w[4m+2])   Eq.2, one rounding
                const half2_t w2 = __builtin_elementwise_fma(q2, s2, o2);            // (w[4m+1], w[4m+3])
                out[2 * hsel] = __builtin_amdgcn_perm(pack_h2(w2), pack_h2(w1), 0x05040100u);      // (w[4m], w[4m+1])
                out[2 * hsel + 1] = __builtin_amdgcn_perm(pack_h2(w2), pack_h2(w1), 0x07060302u);  // (w[4m+2], w[4m+3])
            }
            return __builtin_bit_cast(half8_t, (u32x4_t){out[0], out[1], out[2], out[3]});
        } else if constexpr (P::planes) {
            constexpr int WA = P::WA, WB = P::WB;
            const uint32_t lo = WA == 4 ? r.a[ks] : r.a[ks >> 1] >> (8 * (ks & 1));
            const uint32_t hi = WB == 0 ? 0u : WB == 2 ? r.b[ks >> 1] >> (8 * (ks & 1)) : r.b[0] >> (4 * ks);
#pragma unroll
            for (int p = 0; p < 4; ++p) lv[p] = plane_level<WA, WB>(lo, lo >> 8, hi, p, k);
        } else if constexpr (T::kind == KIND_Q4) {
#pragma unroll
            for (int p = 0; p < 4; ++p) lv[p] = plane_level<4, 0>(r.a[ks], r.a[ks] >> 8, 0u, p, k);
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                lv[2 * i] = as_h2(__builtin_amdgcn_perm(0x64646464u, r.a[2 * ks + i], 0x04010400u)) + m1024;     // (b0, b1)
                lv[2 * i + 1] = as_h2(__builtin_amdgcn_perm(0x64646464u, r.a[2 * ks + i], 0x04030402u)) + m1024; // (b2, b3)
            }
        }
        uint32_t out[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) out[m] = pack_h2(__builtin_elementwise_fma(lv[m], s2, o2));   // Eq.2, one rounding
        return __builtin_bit_cast(half8_t, (u32x4_t){out[0], out[1], out[2], out[3]});
    }
};

template <int N> __device__ __forceinline__ void wait_requests()          // all but the N newest vector-memory requests, and all LDS reads
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}

constexpr int TILE_PITCH = 80, TILE_TURN = 32 * TILE_PITCH;   // a 32 x 32 fp16 tile on its way out: bytes between vectors, in all
// LDS of a workgroup: the activations of STAGES steps, then each wavefront's packed weights
template <int F, int G> constexpr int tile_lds_bytes(int rt, int mb, int wr, int wk, int stages)
{
    return stages * wk * mb * 4096 + wr * wk * rt * Parts<F, G>::BUFFERS * Parts<F, G>::BYTES;
}
// Chunks fetched at once: 64 bytes of a row, or 128 where the 8-bit formats find room (28672 x 8192, 512 vectors 281 -> 259 us, then 244 with eight
// wavefronts instead of four: a 64-byte request fetches half a line from memory), and the formats with four bits in their low plane the same in the tiles whose wavefronts do not
// share K (28672 x 8192, 2000 vectors: 4-bit 848 -> 831 us, 5-bit 904 -> 882, 6-bit 907 -> 888; 4505 x 7104 4-bit, 1706 120.2 -> 117.1; 20000 x 512 4-bit and 30000 x 320 5-bit within
// half a per cent).  Where they share K, twice as long runs leave some without work: 28672 x 8192 6-bit, 20 vectors 44.0 -> 47.8.  2-bit: 2 % slower.
template <int F> constexpr int tile_group(int rt, int mb, int wr, int wk, int stages)
{
    typedef Parts<F> P;
    if (P::WA == 8) return tile_lds_bytes<F, 2>(rt, mb, wr, wk, stages) <= 160 * 1024 && stages <= 3 ? 2 : 1;
    if (P::q3h || P::WA == 2) return 4;
    return wk == 1 && tile_lds_bytes<F, 4>(rt, mb, wr, wk, stages) <= 160 * 1024 ? 4 : 2;
}

// Chunks that wavefront group `group` of WK walks: the runs group, group + WK, ... of G chunks each, and what is left over of the last one.
template <int WK, int G> constexpr __host__ __device__ __forceinline__ int tile_steps(int nchunks, int group)
{
    const int runs = nchunks / G;                              // whole ones
    return (runs + WK - 1 - group) / WK * G + (runs % WK == group ? nchunks % G : 0);
}

// Which tile a workgroup takes.  Workgroups go to the eight dies in turn, and each die has an L2 of its own: a die gets a consecutive part of the tiles, in bands of TILE_BAND
// tiles of vectors (the last one two to TILE_BAND + 1 wide) with those of one row tile next to each other, so that the weights of a row tile are fetched by one die instead of by every
// die that a tile of vectors puts it on, while a die's 32 workgroups at a time still share their activations.  Us, rows outermost -> this: 543 x 25856 4-bit, 1254 vectors 86.9 -> 70.4; 2350 x 21632
// 6-bit, 2035 265 -> 247; 11008 x 4096 3.5-bit, 512 55.9 -> 53.2; 3072 x 11840 4-bit, 31 13.5 -> 12.7.
//   - Rows stay outermost where that puts a row tile on one die by itself (row tiles a multiple of eight) and a die's part would hold the same tiles: two to five tiles of vectors.  With
//     consecutive row tiles on a die such products took 0.4 to 0.7 % more in the mean (five samples of 38 to 93).
//   - No band of one: its tiles read every row tile again, all of them on the last dies.  (With it, five tiles of vectors: 2048 x 19264 4-bit, 278 vectors 48.1, 52.7 with it, now 49.3 in the
//     rows' order; 1280 x 21248 5-bit, 300 43.4, 47.5, 43.4.)
//   - The kernel divides by numbers that the host has turned into factors: 24 instructions fewer in front of the first copies than with divisions.
// 750 random products (17 to 2000 vectors) against rows outermost for all: 2.3 % less in the mean, 32 % at best, 4.6 % more at worst (4221 x 27840 8-bit, 316 vectors 123.5 -> 128); what
// is left of the losses are 36 to 44 row tiles, a multiple of four, with five and seven tiles of vectors.  (Before the three points above: 1.8 % less in the mean, 17 % more at worst.)
constexpr uint32_t TILE_DIES = 8, TILE_BAND = 4;
__host__ __device__ __forceinline__ uint32_t tiles_high(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }
static TileOrder tile_order(uint32_t ntr, uint32_t ntb)
{
    if (ntr % TILE_DIES == 0 && ntb > 1 && ntb <= TILE_BAND + 1) return TileOrder{0, 0};
    const uint32_t bands = ntb <= TILE_BAND + 1 ? 1 : (ntb + 2) / TILE_BAND, wide = ntb - (bands - 1) * TILE_BAND;
    return TileOrder{(0x80000000u + wide - 1) / wide, bands == 1 ? 0u : (uint32_t)((1ULL << 32) / (ntr * (uint64_t)TILE_BAND))};
}
// (x, y): the workgroup's place in a grid of ntr x ntb where rows are outermost, (its number, 0) otherwise.  A division by a width of one to five is exact below 2^29 tiles; the one by a
// band's tiles comes out one too small at most.
__host__ __device__ __forceinline__ TilePlace tile_place(uint32_t x, uint32_t y, uint32_t ntr, uint32_t ntb, const TileOrder order)
{
    const uint32_t total = ntr * ntb, die = x % TILE_DIES, more = total % TILE_DIES;
    uint32_t in = die * (total / TILE_DIES) + (die < more ? die : more) + x / TILE_DIES, first = 0, wide = ntb, per_tile = order.per_tile;
    if (order.per_band) {
        const uint32_t last = (ntb + 2) / TILE_BAND - 1, span = ntr * TILE_BAND;
        uint32_t band = tiles_high(in, order.per_band);
        if (in - band * span >= span) ++band;
        if (band > last) band = last;
        first = band * TILE_BAND;
        in -= band * span;
        wide = band == last ? ntb - first : TILE_BAND;
        per_tile = band == last ? per_tile : 0x80000000u / TILE_BAND;
    }
    const uint32_t tr = tiles_high(2 * in, per_tile);
    return order.per_tile ? TilePlace{tr, first + in - tr * wide} : TilePlace{x, y};
}

void qgemm_tile_places(uint32_t ntr, uint32_t ntb, TilePlace *places)
{
    const TileOrder order = tile_order(ntr, ntb);
    const uint32_t width = order.per_tile ? ntr * ntb : ntr;
    for (uint32_t wg = 0; wg < ntr * ntb; ++wg) places[wg] = tile_place(wg % width, wg / width, ntr, ntb, order);
}

// RT x 32 weight rows and MB x 32 activation vectors per wavefront; WR wavefronts side by side along the rows share a chunk's
// activations, WK such groups take every WK-th run of G chunks each and add their sums at the end.
template <int F, int RT, int MB, int WR, int WK, int STAGES>
__global__ __launch_bounds__(64 * WR * WK, RT * MB <= 8 ? 2 : 1) void qgemm_tile_kernel(const uint8_t *packed, const uint16_t *X, uint16_t *Y,
                                                                                        int rows, int cols, int batch, int64_t header_offset,
                                                                                        uint32_t per_tile, uint32_t per_band)
{
    constexpr int G = tile_group<F>(RT, MB, WR, WK, STAGES), BM = 32 * MB;
    typedef Parts<F, G> P;
    constexpr int SLICE = BM * 128, STEP = WK * SLICE;         // bytes of one chunk's activations; of the WK chunks of a step
    constexpr int NX = (4 * MB + WR - 1) / WR;                 // 1 KB pieces of its group's chunk a wavefront copies per step
    constexpr int NG = RT * (P::q3h ? 2 * P::NA : P::NA + P::NB + P::NH);      // a wavefront's requests per group of G chunks
    // With two stages a step waits for what was requested one step ago.  Where a group lasts two steps its request goes out behind that step's
    // activations, so that the wait for them leaves it one step more: these bytes come from memory, the activations from L2.  It is worth something where a group is whole
    // lines, in the 8-bit formats (28672 x 8192, 1000 vectors 467 -> 453 us, 2000 886 -> 877; 8192 x 8192, 512 77.5 -> 76.9); to the tiles whose wavefronts share K, in the 4-, 5- and 6-bit formats, nothing
    // (11008 x 4096, 512, 192 x 128: 57.0 and 57.0).  Groups of four steps keep the other order: 28672 x 8192, 2000 vectors 4-bit 831 -> 833 with this one, 5-bit 882 -> 891, 6-bit 888 -> 884; 3.5-bit,
    // 11008 x 4096, 2048 201 -> 207.  So do wavefronts without a barrier: 4096 x 11008 8-bit, 33 vectors 17.4 -> 17.7.
    constexpr bool XFIRST = STAGES == 2 && G == 2 && WR > 1;
    // what may still be on its way when a step's activations have to be there: the activations of the STAGES - 2 steps after it and
    // the groups requested among them (XFIRST: behind them)
    constexpr int AHEAD = STAGES - 2, SINCE = AHEAD + XFIRST, SURE = AHEAD * NX + SINCE / G * NG;
    static_assert(SURE + NG < 64 && (P::BUFFERS - 1) * G >= STAGES - 1 + XFIRST, "the wait counter's range; a group is there when its steps come");
    extern __shared__ __align__(16) uint8_t smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave % WR, wk = wave / WR;
    const int li = lane & 31, h = lane >> 5;
    const TilePlace place = tile_place(blockIdx.x, blockIdx.y, ((uint32_t)rows + 32 * RT * WR - 1) / (32 * RT * WR), ((uint32_t)batch + BM - 1) / BM, TileOrder{per_tile, per_band});
    const int tr = (int)place.tr, tb = (int)place.tb;
    const int n0 = (tr * WR + wr) * (32 * RT), m0 = tb * BM;
    // Run q of G chunks (the last one may be shorter) belongs to wavefront group q % WK.  A group stops at its own last chunk: nothing is
    // multiplied that the product does not have (weights of zero against the last activations again would turn an infinity there into a NaN),
    // and groups with a chunk less leave the compute unit to the others (with K rounded up to WK G chunks, us, 3.5-bit: 4096 x 11008, 33
    // vectors 19.2, now 17.2; 4096 x 4160, 17 vectors 10.5, now 8.4).
    const int nchunks = cols / 64;
    auto steps_of = [&](int group) { return tile_steps<WK, G>(nchunks, group); };
    const int steps = steps_of(wk);
    auto chunk_of = [&](int step) { return ((step / G) * WK + wk) * G + step % G; };

    // activations: piece p of a step (1 KB = 8 rows of a chunk) -> LDS as it comes; the 16-byte slots of row r are permuted by
    // r / 2 (on the way in by choosing what each lane fetches), so that neighbouring rows' operand reads fall into different banks.
    // A wavefront copies pieces of its own group's chunk (the last ones the last piece again where they do not come out even).
    const uint8_t *xbase = reinterpret_cast<const uint8_t *>(X + (int64_t)m0 * cols);
    uint32_t xoff[NX];
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        const int r = min(wr * NX + i, 4 * MB - 1) * 8 + (lane >> 3);          // past the batch: the last vector again, its results are not stored
        xoff[i] = (uint32_t)min(r, batch - 1 - m0) * (uint32_t)(cols * 2) + ((lane & 7) ^ ((r >> 1) & 7)) * 16;
    }
    auto request_x = [&](int step, int stage) {
        const int kc = min(chunk_of(step), nchunks - 1);       // past the end: the last chunk again, never multiplied
#pragma unroll
        for (int i = 0; i < NX; ++i) copy_to_lds<16>(xbase + (int64_t)kc * 128, xoff[i], lds0 + stage * STEP + wk * SLICE + min(wr * NX + i, 4 * MB - 1) * 1024);
    };
    WeightRows<F, G> rowsw;
    rowsw.open(packed, rows, cols, header_offset, min(n0, rows - 1), lane);
    const int w0 = STAGES * STEP + wave * (RT * P::BUFFERS * P::BYTES);        // this wavefront's packed weights in LDS
    auto request_w = [&](int group, int buf) {
        const int kc = min((group * WK + wk) * G, (nchunks - 1) / G * G);
#pragma unroll
        for (int t = 0; t < RT; ++t) rowsw.request(t, kc, lds0 + w0 + (buf * RT + t) * P::BYTES);
    };

    float16_t acc[RT][MB];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][m][v] = 0.f;

    // k-step ks of a chunk: lane (i, h) takes columns 32 h + 8 ks .. + 7
    const uint8_t *xrow = smem + wk * SLICE + li * 128;
    auto read_x = [&](int stage, int ks, half8_t (&af)[MB]) {
#pragma unroll
        for (int m = 0; m < MB; ++m) af[m] = *reinterpret_cast<const half8_t *>(xrow + stage * STEP + m * 4096 + (((4 * h + ks) ^ ((li >> 1) & 7)) * 16));
    };
    RawHalf<F> w[RT];
    HalfDecoder<F> dec[RT];
    DecodeConstants constants;
    constants.open();
    half8_t af[2][MB], bf[2][RT];
    auto read_w = [&](int c, int buf) {
#pragma unroll
        for (int t = 0; t < RT; ++t) WeightRows<F, G>::read(smem + w0 + (buf * RT + t) * P::BYTES, li, c, h, w[t]);
    };
#pragma unroll
    for (int i = 0; i < P::BUFFERS - 1; ++i) request_w(i, i);
#pragma unroll
    for (int i = 0; i < STAGES - 1; ++i) request_x(i, i);
    wait_requests<(STAGES - 2) * NX>();
    if constexpr (WR > 1) __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if constexpr (XFIRST) request_x(STAGES - 1, STAGES - 1);
    request_w(P::BUFFERS - 1, P::BUFFERS - 1);
    if constexpr (!XFIRST) request_x(STAGES - 1, STAGES - 1);
    read_w(0, 0);
    read_x(0, 0, af[0]);
#pragma unroll
    for (int t = 0; t < RT; ++t) { dec[t].open(w[t], constants, h); bf[0][t] = dec[t].step(w[t], 0); }
    int stage = 0, c = 0, buf = 0, group = 0;
    for (int step = 0; step < steps; ++step) {
        const int next = stage == STAGES - 1 ? 0 : stage + 1;
        // Each k-step's operands are read (activations) and decoded (weights) during the matrix instructions of the one before,
        // the next step's first ones during this step's last: its requests have arrived by then, and this stage is free again.
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            __builtin_amdgcn_sched_barrier(0);
            if (ks < 3) {
                read_x(stage, ks + 1, af[(ks + 1) & 1]);
            } else {
                if (G > 1 && SINCE % G != 0 && c < SINCE % G) wait_requests<SURE + NG>();   // a group was requested since
                else wait_requests<SURE>();                    // step + 1's are there; and the wavefront's reads of this stage are done
                if constexpr (WR > 1) __builtin_amdgcn_s_barrier();   // ... everybody's (a group of one wavefront copies what it reads)
                asm volatile("" ::: "memory");
                if constexpr (XFIRST) request_x(step + STAGES, stage);
                if (G == 1 || ++c == G) {                      // the group is used up
                    c = 0; ++group;
                    const int used = buf;
                    buf = buf == P::BUFFERS - 1 ? 0 : buf + 1;
                    request_w(group + P::BUFFERS - 1, used);
                }
                if constexpr (!XFIRST) request_x(step + STAGES, stage);
                read_w(c, buf);
                read_x(next, 0, af[0]);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                if (ks == 3) dec[t].open(w[t], constants, h);
                bf[(ks + 1) & 1][t] = dec[t].step(w[t], (ks + 1) & 3);
#pragma unroll
                for (int m = 0; m < MB; ++m) acc[t][m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(bf[ks & 1][t], af[ks & 1][m], acc[t][m], 0, 0, 0);
            }
        }
        stage = next;
    }
    if constexpr (WR > 1 && WK > 1)
        for (int step = steps; step < steps_of(0); ++step) __builtin_amdgcn_s_barrier();      // the other groups' steps (group 0 has the most)

    // the groups' sums: tile q of a wavefront is added up, in the order of the groups, by group q % WK
    wait_requests<0>();                                        // what was requested past the end has landed
    __syncthreads();                                           // ... everybody's, and everybody's last operands have been read
    if constexpr (WK > 1) {
#pragma unroll
        for (int q = 0; q < RT * MB; ++q) {
            if (wk == q % WK) continue;
            float4_t *part = reinterpret_cast<float4_t *>(smem) + ((wr * RT * MB + q) * (WK - 1) + (wk > q % WK ? wk - 1 : wk)) * 256 + lane;
            const float16_t v = acc[q / MB][q % MB];
#pragma unroll
            for (int j = 0; j < 4; ++j) part[j * 64] = (float4_t){v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]};
        }
        __syncthreads();
    }
    // 32x32 accumulator layout: register v of lane (li, h) is weight row (v/4)*8 + h*4 + v%4, vector li.  A tile crosses LDS once more, so that four
    // neighbouring lanes store 64 consecutive bytes of one vector, whatever the number of rows is (stored from the registers, eight bytes
    // per lane where rows are a multiple of four and two where not, odd row counts took 62 -> 73 us at 11007 x 4096 x 512).
    uint8_t *turn = smem + (WK > 1 ? WR * RT * MB * (WK - 1) * 4096 : 0) + wave * TILE_TURN;
#pragma unroll
    for (int q = 0; q < RT * MB; ++q) {
        if (WK > 1 && wk != q % WK) continue;
        const int t = q / MB, m = q % MB;
        float16_t sum = acc[t][m];
        if constexpr (WK > 1) {
            const float4_t *part = reinterpret_cast<const float4_t *>(smem) + (wr * RT * MB + q) * (WK - 1) * 256 + lane;
            const float16_t own = sum;
#pragma unroll
            for (int k = 0; k < WK; ++k) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float4_t p = k == q % WK ? (float4_t){own[4 * j], own[4 * j + 1], own[4 * j + 2], own[4 * j + 3]}
                                                   : part[(k > q % WK ? k - 1 : k) * 256 + j * 64];
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[4 * j + e] = k == 0 ? p[e] : sum[4 * j + e] + p[e];
                }
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const half2_t lo = {(half_t)sum[4 * j], (half_t)sum[4 * j + 1]}, hi = {(half_t)sum[4 * j + 2], (half_t)sum[4 * j + 3]};
            *reinterpret_cast<u32x2_t *>(turn + li * TILE_PITCH + j * 16 + h * 8) = (u32x2_t){as_u32(lo), as_u32(hi)};
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int vec = m0 + m * 32 + i * 16 + (lane >> 2), row = n0 + t * 32 + (lane & 3) * 8;
            const u32x4_t v = *reinterpret_cast<const u32x4_t *>(turn + (i * 16 + (lane >> 2)) * TILE_PITCH + (lane & 3) * 16);
            uint16_t *y = Y + (int64_t)vec * rows + row;
            if (vec < batch && row < rows) {
                if (row + 8 <= rows) {
                    *reinterpret_cast<u32x4_any_t *>(y) = v;
                } else {
                    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (row + e < rows) y[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();                      // the next tile overwrites this one
    }
}

// Byte offsets inside a tile (of its vectors' activations, of a wavefront's rows) are 32-bit: the longest rows a tile can take.  (One limit of
// 2^22 for all of them left longer rows to passes of sixteen vectors: 512 rows of 2^22 + 64 columns, 4-bit, 96 vectors 22.3 ms, now 6.8; passes
// remain faster by up to a fifth for 17 to 32 vectors on 64 4-bit rows of 2^22 columns and more, slower on 16 and on 512 rows.)
constexpr int64_t tile_max_cols(int rt, int mb) { return (1LL << 32) / (32 * (2 * mb > rt ? 2 * mb : rt)); }

template <int F, int RT, int MB, int WR, int WK, int STAGES>
static hipError_t tile_go(const void *packed, int64_t rows, int64_t cols, const uint16_t *X, int64_t batch, uint16_t *Y, hipStream_t s)
{
    typedef Fmt<F> T;
    constexpr int staged = tile_lds_bytes<F, tile_group<F>(RT, MB, WR, WK, STAGES)>(RT, MB, WR, WK, STAGES), merge = WR * RT * MB * (WK - 1) * 4096 + WR * WK * TILE_TURN;
    constexpr int lds = staged > merge ? staged : merge;
    static_assert(lds <= 160 * 1024, "LDS of a compute unit");
    if (cols > tile_max_cols(RT, MB)) return hipErrorInvalidValue;
    static PerDevice pd;
    int cus = 0;
    const hipError_t e = once_per_device(pd, &cus, [] {
        return hipFuncSetAttribute(reinterpret_cast<const void *>(&qgemm_tile_kernel<F, RT, MB, WR, WK, STAGES>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    });
    if (e != hipSuccess) return e;
    const int64_t header_offset = rows * (cols / T::block) * (int64_t)T::code_bytes;
    const int64_t ntr = (rows + 32 * RT * WR - 1) / (32 * RT * WR), ntb = (batch + 32 * MB - 1) / (32 * MB);
    if (ntr * ntb >= 1LL << 29) return hipErrorInvalidValue;   // (Y alone would be a terabyte)
    const TileOrder order = tile_order((uint32_t)ntr, (uint32_t)ntb);
    hipLaunchKernelGGL((qgemm_tile_kernel<F, RT, MB, WR, WK, STAGES>), order.per_tile ? dim3((unsigned)(ntr * ntb)) : dim3((unsigned)ntr, (unsigned)ntb), dim3(64 * WR * WK), lds, s,
                       static_cast<const uint8_t *>(packed), X, Y, (int)rows, (int)cols, (int)batch, header_offset, order.per_tile, order.per_band);
    return hipGetLastError();
}

// The tiles in use and what a launch of each costs in microseconds, for every format: rounds * (round + steps * step), rounds = workgroups per compute unit, steps =
// chunks that one wavefront walks.  `step` was fitted to four formats x eleven shapes (1024^2 to 28672 x 8192 and 11885 x 17792) x 17 .. 2000 vectors,
// `round` (start, first copies, sums and stores) is the median of what rows of 64 to 1024 columns take beyond their steps, both on earlier kernels; the two of 192 x 128 and 128 x 64 are set
// by hand since.  On 200 random products that no constant was fitted to (all formats, 512 to 28672 rows, 1024 to 28672 columns, 17 to 2000 vectors) the chosen tile is
// 0.33 % slower than the best in the mean and 11 % at worst; on 300 of 64 to 1024 columns 2.2 % and 18 %: there 128 x 64 is the best for 109, its price takes it for 38 (before it
// had eight wavefronts 1.3 % and 9.5 %, and the chosen one was slower).  (`round` fitted to the long rows too came out at 0.6 to 4.9 us and took
// 256 x 160 for nearly everything below 256 columns, 13 % slower than the best: 131072 x 64, 3.5-bit, 33 vectors 9.6 us, now 8.8; 33 x 256, 512 vectors 8.6, now 5.1.)
// A workgroup too many for the last round costs up to half of a
// launch, so sizes in between are worth having (with nine tiles 6.5 % slower than the best of 33 in the mean); eight wavefronts of 32 rows beat four of 64 where LDS holds
// their weights (two per SIMD hide each other's waits: 28672 x 8192, 512 vectors 228 -> 220 us, 8-bit 259 -> 244, in addition to the longer requests; 4096 x 4096 x 512 32 -> 25).
// 192 x 128 and 128 x 64 were four wavefronts of 96 and 64 rows: twelve and eight of 32, three and two per SIMD instead of one, read the activations from LDS three times and twice
// as often and are faster all the same (tile against tile, the places with them, on the 200 and the 300 products above: 192 x 128 14 and 24 % in the mean, at worst the same, 128 x 64 9 and 15 %, at worst
// 6 % slower where it is not the one to take; 11008 x 4096, 512 vectors 53.9 -> 50.7 us in 4-bit, 62.2 -> 57.2 in 5-bit, 63 -> 56.5 in 8-bit).  Of 1050 products the choice changed for 27, all
// 6 to 22 % faster.  Not so where a wavefront has its vectors to itself (64 x 64 as eight wavefronts of 32 rows 2 to 8 % slower than four of 64).
// The choice depends on sizes, format and the number of compute units only, so a call always takes the same path on the same device.
#define IFLOW_TILES(V) /* RT MB WR WK STAGES  round  step */ \
    V(1, 8, 8, 1, 2, 5.12, 1.47)    /* 256 rows x 256 vectors: the fewest decodes and reads per product */ \
    V(1, 7, 8, 1, 2, 4.23, 1.38)    /* 256 x 224 (28672 rows x 2000 vectors: 1008 workgroups, four rounds (256 x 256: 3.5)) */ \
    V(1, 6, 4, 2, 2, 4.55, 1.40)    /* 128 x 192 */ \
    V(1, 5, 8, 1, 2, 3.71, 1.12)    /* 256 x 160 */ \
    V(1, 4, 8, 1, 3, 3.59, 0.93)    /* 256 x 128 */ \
    V(1, 4, 4, 2, 2, 3.39, 1.11)    /* 128 x 128 */ \
    V(1, 4, 6, 2, 2, 4.50, 1.55)    /* 192 x 128 (11008 rows x 512 vectors: 232 workgroups) */ \
    V(1, 4, 3, 2, 2, 3.61, 1.00)    /* 96 x 128 */ \
    V(1, 3, 4, 2, 3, 3.54, 0.91)    /* 128 x 96 */ \
    V(1, 4, 2, 2, 3, 3.83, 0.71)    /* 64 x 128 */ \
    V(1, 2, 4, 2, 2, 3.50, 0.78)    /* 128 x 64 */ \
    V(3, 2, 1, 4, 2, 5.47, 1.10)    /* 96 x 64 */ \
    V(2, 3, 1, 4, 2, 5.31, 0.93)    /* 64 x 96 */ \
    V(2, 2, 1, 4, 2, 4.03, 0.79)    /* 64 x 64 */ \
    V(2, 1, 1, 4, 3, 3.18, 0.60)    /* 64 x 32 */ \
    V(1, 2, 1, 4, 3, 2.72, 0.51)    /* 32 x 64 */ \
    V(1, 1, 1, 8, 2, 3.00, 0.66)    /* 32 x 32 */

// The cheapest tile's place in the list (-1: rows too long for every one).
template <int F> static int tile_choice(int64_t rows, int64_t cols, int64_t batch, int cus)
{
    int best = -1, i = 0;
    double best_us = 0;
#define IFLOW_TILE_PRICE(RT, MB, WR, WK, STAGES, ROUND, STEP_US) { \
        constexpr int G = tile_group<F>(RT, MB, WR, WK, STAGES); \
        const int64_t wgs = ((rows + 32 * RT * WR - 1) / (32 * RT * WR)) * ((batch + 32 * MB - 1) / (32 * MB)); \
        const double rounds = (double)((wgs + cus - 1) / cus), steps = (double)tile_steps<WK, G>((int)(cols / 64), 0); \
        const double us = rounds * (ROUND + steps * STEP_US); \
        if (cols <= tile_max_cols(RT, MB) && (best < 0 || us < best_us)) { best = i; best_us = us; } \
        ++i; }
    IFLOW_TILES(IFLOW_TILE_PRICE)
#undef IFLOW_TILE_PRICE
    return best;
}

template <int F>
static hipError_t tile_launch(int tile, const void *packed, int64_t rows, int64_t cols, const uint16_t *X, int64_t batch, uint16_t *Y, hipStream_t s)
{
    int i = 0;
#define IFLOW_TILE_GO(RT, MB, WR, WK, STAGES, ROUND, STEP_US) \
    if (tile == i++) return tile_go<F, RT, MB, WR, WK, STAGES>(packed, rows, cols, X, batch, Y, s);
    IFLOW_TILES(IFLOW_TILE_GO)
#undef IFLOW_TILE_GO
    return hipErrorInvalidValue;
}

template <int F> static bool tile_shape(int tile, TileShape *shape)
{
    int i = 0;
#define IFLOW_TILE_SHAPE(RT, MB, WR, WK, STAGES, ROUND, STEP_US) \
    if (tile == i++) { \
        constexpr int G = tile_group<F>(RT, MB, WR, WK, STAGES); \
        *shape = TileShape{32 * RT * WR, 32 * MB, WK, G, Parts<F, G>::BUFFERS, tile_max_cols(RT, MB)}; \
        return true; \
    }
    IFLOW_TILES(IFLOW_TILE_SHAPE)
#undef IFLOW_TILE_SHAPE
    return false;
}

int qgemm_tile_choice(int format, int64_t rows, int64_t cols, int64_t batch, int cus)
{
    int tile = -1;
    if (cols % 64 == 0)
        (void)for_format(format, [&](auto f) { tile = tile_choice<decltype(f)::value>(rows, cols, batch, cus); return hipSuccess; });
    return tile;
}

bool qgemm_tile_shape(int format, int tile, TileShape *shape)
{
    bool known = false;
    (void)for_format(format, [&](auto f) { known = tile_shape<decltype(f)::value>(tile, shape); return hipSuccess; });
    return known;
}

hipError_t launch_qgemm_tile(int format, int tile, const void *packed, int64_t rows, int64_t cols,
                             const uint16_t *X, int64_t batch, uint16_t *Y, hipStream_t s)
{
    if (cols % 64 != 0) return hipErrorInvalidValue;
    return for_format(format, [&](auto f) { return tile_launch<decltype(f)::value>(tile, packed, rows, cols, X, batch, Y, s); });
}

hipError_t launch_qgemm_mfma(int format, const void *packed, int64_t rows, int64_t cols,
                             const uint16_t *X, int64_t batch, uint16_t *Y, hipStream_t s)
{
    int cus = 0;
    const hipError_t e = device_compute_units(&cus);
    if (e != hipSuccess) return e;
    return launch_qgemm_tile(format, qgemm_tile_choice(format, rows, cols, batch, cus), packed, rows, cols, X, batch, Y, s);
}

}  // namespace iflow
