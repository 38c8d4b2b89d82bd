// One decode step of grouped-query attention over an fp16 key/value cache (arXiv 2401.08294, section "Grouped-query
// attention": head_i = Attention(Q_i, K^j, V^j) with j the group of query head i; Attention = scaled dot-product
// attention; with as many groups as heads it is multi-head attention).
//
// Next to the weight stream this is the other part of a decode step that is bound by memory: every cached key and
// value is read once per step and used for a handful of multiply-adds.  So the kernel is laid out like the GEMV: long
// contiguous 16-byte-per-lane reads, everything else in registers.
//   - The cache is [kv head][position][128] fp16, so the positions of a head are one contiguous stream.  A workgroup
//     (four wavefronts) takes one kv head and one contiguous range of positions (a "split"); the grid is
//     kv heads x splits, about one workgroup per compute unit.
//   - A wavefront walks its range in blocks of sixteen positions.  Sixteen lanes share a position (8 of the 128
//     components each), so one load instruction covers four consecutive positions = 1 KB; the four lane groups of a
//     wavefront keep separate running softmax states (maximum, sum, 128-component weighted value sum) for their
//     positions.  The block after the current one is already requested while a block is processed.
//   - All query heads of a group are served from the same loaded keys and values: one or two heads by the kernel
//     described here, on the vector units; more by attn_decode_mfma_kernel further down, on the matrix cores.
//   - Softmax is computed the streaming way: per block one rescale of the running sums to the new maximum, then
//     exp2 of the (pre-scaled) score differences.  fp32 throughout; the output is rounded to fp16 once.
//   - A workgroup merges its sixteen states through LDS and writes one state per (head, split) to the caller's
//     workspace; a second, small kernel (one workgroup per query head) merges the splits and writes the output.  Two
//     launches rather than "the last workgroup to finish merges": device-wide release/acquire fences write back and
//     invalidate whole L2 caches on this part (several microseconds per workgroup, measured), and one workgroup per
//     kv head merging all its heads' splits one after the other is a long serial tail; the second launch costs about
//     two microseconds and merges all heads at once.  With a single split the first kernel writes the output itself.
#include "iflow_common.h"

namespace iflow {

constexpr int ATT_D = 128;                                    // head dimension
constexpr int ATT_WAVES = 4;
constexpr int ATT_TILES = 4;                                  // tiles of four positions per block: 16 positions per wavefront and block
constexpr int ATT_MAX_SPLITS = 64;
// States are merged relative to 2^-16 of the largest reference, so that one whose reference lags its maximum (the matrix-core kernel's, by up to 2^ATT_LAG) is not lost for
// that: a factor is zero, and an infinite sum times it a NaN, from 2^-142 on.  (Sums are below 2^51 - 2^20 positions, probabilities up to 2^15 - and below 2^99 after three merges.)
constexpr float ATT_SPARE = 16.f;
// workspace: value sums O[head][ATT_MAX_SPLITS][component], then maxima M[head][ATT_MAX_SPLITS], then sums L[head][ATT_MAX_SPLITS]
// (fp32; a state's 128 components are contiguous: written and read by 128 neighbouring threads)

typedef uint32_t att_u32x4 __attribute__((ext_vector_type(4)));

// One head's keys or values of a workgroup's positions, as a buffer that ends with them: blocks are requested ahead without a branch (behind one the compiler waits
// for everything), and what lies past the end arrives as zeros without a request to memory.  (With the last position requested again in
// their place, 32/32 heads, 64 positions took 2.80 us, now 2.67; 64/32 3.74 and 3.49.)  Bytes are counted in 32 bits: a cache has at most 2^20 positions, 2^28 bytes of a head.
struct AttRange {
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ AttRange(const uint16_t *first, int positions, int d)
    {
        rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(first), 0, (int)((uint32_t)positions * (2u * (uint32_t)d)), 0x00027000);
    }
    __device__ __forceinline__ att_u32x4 load(uint32_t byte) const       // (2: nontemporal)
    {
        return __builtin_bit_cast(att_u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)byte, 0, 2));
    }
};

template <int R>
__global__ __launch_bounds__(64 * ATT_WAVES) void attn_decode_kernel(const uint16_t *__restrict__ q, const uint16_t *__restrict__ kc,
                                                                     const uint16_t *__restrict__ vc, uint16_t *__restrict__ out,
                                                                     float *__restrict__ ws, int n_heads, int seq_len, int64_t head_stride /* halves */,
                                                                     int chunk, int nsplit, float scale_log2e)
{
    __shared__ float s_acc[16][ATT_D];
    __shared__ float s_m[16], s_l[16];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int gq = lane >> 4, dseg = lane & 15;               // position inside a tile; which 8 of the 128 components
    const int j = blockIdx.x / nsplit, sp = blockIdx.x - j * nsplit;
    const int t_begin = sp * chunk, t_end = min(seq_len, t_begin + chunk);      // t_begin < seq_len by construction
    const AttRange keys(kc + (int64_t)j * head_stride + (int64_t)t_begin * ATT_D, t_end - t_begin, ATT_D);
    const AttRange values(vc + (int64_t)j * head_stride + (int64_t)t_begin * ATT_D, t_end - t_begin, ATT_D);

    // the group's queries: lane holds components 8 dseg .. 8 dseg + 7 of each
    half2_t qr[R][4];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const att_u32x4 v = *reinterpret_cast<const att_u32x4 *>(q + (int64_t)(j * R + r) * ATT_D + dseg * 8);
        qr[r][0] = as_h2(v.x); qr[r][1] = as_h2(v.y); qr[r][2] = as_h2(v.z); qr[r][3] = as_h2(v.w);
    }
    float m[R], l[R], acc[R][8];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        m[r] = -INFINITY; l[r] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[r][e] = 0.f;
    }

    // positions past the range are zeros and their scores set to -inf
    auto load_block = [&](att_u32x4 (&kt)[ATT_TILES], att_u32x4 (&vt)[ATT_TILES], int p0) {
        const uint32_t byte = (uint32_t)(p0 - t_begin) * (2 * ATT_D) + lane * 16;
#pragma unroll
        for (int t = 0; t < ATT_TILES; ++t) kt[t] = keys.load(byte + t * 1024);
        // (all keys first, which are needed first: with both in turn 32/32 heads, 3001 of 4096 positions 9.66 us, now 9.57, over a ring 12.4 and 12.1; 50 lengths and head counts 0.2 to 0.4 % less
        // in the mean)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < ATT_TILES; ++t) vt[t] = values.load(byte + t * 1024);
    };
    auto process_block = [&](const att_u32x4 (&kt)[ATT_TILES], const att_u32x4 (&vt)[ATT_TILES], int p0) {
        float vf[ATT_TILES][8];
#pragma unroll
        for (int t = 0; t < ATT_TILES; ++t) {
            const half2_t a = as_h2(vt[t].x), b = as_h2(vt[t].y), c = as_h2(vt[t].z), d = as_h2(vt[t].w);
            vf[t][0] = (float)a.x; vf[t][1] = (float)a.y; vf[t][2] = (float)b.x; vf[t][3] = (float)b.y;
            vf[t][4] = (float)c.x; vf[t][5] = (float)c.y; vf[t][6] = (float)d.x; vf[t][7] = (float)d.y;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float s[ATT_TILES];
            float bm = -INFINITY;
#pragma unroll
            for (int t = 0; t < ATT_TILES; ++t) {
                float d = __builtin_amdgcn_fdot2(qr[r][0], as_h2(kt[t].x), 0.f, false);
                d = __builtin_amdgcn_fdot2(qr[r][1], as_h2(kt[t].y), d, false);
                d = __builtin_amdgcn_fdot2(qr[r][2], as_h2(kt[t].z), d, false);
                d = __builtin_amdgcn_fdot2(qr[r][3], as_h2(kt[t].w), d, false);
                d = row16_sum(d) * scale_log2e;               // the score of this lane group's position, in units of log2
                s[t] = (p0 + t * 4 + gq < t_end) ? d : -INFINITY;
                bm = fmaxf(bm, s[t]);
            }
            const float m_new = fmaxf(m[r], bm);
            // (a state that has not seen a valid position yet has maximum -inf: nothing to rescale, and no -inf - -inf)
            const float alpha = (m_new == -INFINITY) ? 1.0f : __builtin_amdgcn_exp2f(m[r] - m_new);
            const float base = (m_new == -INFINITY) ? 0.f : m_new;
            l[r] *= alpha;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[r][e] *= alpha;
#pragma unroll
            for (int t = 0; t < ATT_TILES; ++t) {
                const float p = __builtin_amdgcn_exp2f(s[t] - base);            // exp2(-inf) = 0 for masked positions
                l[r] += p;
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[r][e] = __builtin_fmaf(p, vf[t][e], acc[r][e]);
            }
            m[r] = m_new;
        }
    };

    // blocks of this wavefront: wave, wave + 4, ... of the range, two per trip so that the two register sets alternate
    att_u32x4 ka[ATT_TILES], va[ATT_TILES], kb[ATT_TILES], vb[ATT_TILES];
    constexpr int STEP = 16 * ATT_WAVES;                      // positions between a wavefront's consecutive blocks
    int p0 = t_begin + wave * 16;
    // (The wait in front of a block counts the requests issued after that block's own, so the order in which the two sets are requested has to be the same in front of the loop and in
    // it, or the wait becomes one for everything.  Scheduling barriers pin it, but not against moving requests behind the loop's own test, one by one: they stand behind it.  Us over a ring
    // of caches: 32/32 heads, 16001 positions 42.4 with half of the first block's values requested last, now 41.7; 8000 23.9 and 23.2; 3001 11.8 and 11.6; 16/16, 16001 23.7 and 23.1.)
    if (p0 < t_end) {
        load_block(ka, va, p0);
        __builtin_amdgcn_sched_barrier(0);
        load_block(kb, vb, p0 + STEP);
        __builtin_amdgcn_sched_barrier(0);
        do {
            process_block(ka, va, p0);
            __builtin_amdgcn_sched_barrier(0);
            load_block(ka, va, p0 + 2 * STEP);
            __builtin_amdgcn_sched_barrier(0);
            if (p0 + STEP < t_end) process_block(kb, vb, p0 + STEP);          // (uniform over the wavefront)
            __builtin_amdgcn_sched_barrier(0);
            load_block(kb, vb, p0 + 3 * STEP);
            __builtin_amdgcn_sched_barrier(0);
            p0 += 2 * STEP;
        } while (p0 < t_end);
    }

    // ---- merge the sixteen states (4 wavefronts x 4 lane groups) of each head, store or hand over -----------------------
    const int pid = wave * 4 + gq;
    float *ws_o = ws, *ws_m = ws + (int64_t)n_heads * ATT_D * ATT_MAX_SPLITS, *ws_l = ws_m + (int64_t)n_heads * ATT_MAX_SPLITS;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r > 0) __syncthreads();                           // the previous head's states have been read
#pragma unroll
        for (int e = 0; e < 8; ++e) s_acc[pid][dseg * 8 + e] = acc[r][e];
        if (dseg == 0) { s_m[pid] = m[r]; s_l[pid] = l[r]; }
        __syncthreads();
        if (tid < ATT_D) {
            float M = s_m[0];
#pragma unroll
            for (int i = 1; i < 16; ++i) M = fmaxf(M, s_m[i]);                  // finite: the range is not empty
            float L = 0.f, O = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float f = __builtin_amdgcn_exp2f(s_m[i] - M);
                L = __builtin_fmaf(s_l[i], f, L);
                O = __builtin_fmaf(s_acc[i][tid], f, O);
            }
            const int head = j * R + r;
            if (nsplit == 1) {
                out[(int64_t)head * ATT_D + tid] = as_u16((half_t)(O / L));
            } else {
                ws_o[((int64_t)head * ATT_MAX_SPLITS + sp) * ATT_D + tid] = O;
                if (tid == 0) { ws_m[(int64_t)head * ATT_MAX_SPLITS + sp] = M; ws_l[(int64_t)head * ATT_MAX_SPLITS + sp] = L; }
            }
        }
    }
}

// ---- three or more query heads per kv head, or 64 components: scores and weighted sums on the matrix cores -------------
// With eight heads per loaded key the vector units bind (about 46 instructions per position in the kernel above).  But a
// block of 32 positions against a group of heads is two small dense contractions:
//   S[position][head]  = sum_k K[position][k] Q[head][k]            2 x 16 x 128 x (16 heads, up to RMAX of them real)
//   O[head][component] = sum_position P[position][head] V[position][component]
// and v_mfma_f32_16x16x32_f16 does the first in eight instructions per block and the second in sixteen, with the probabilities as two fp16 numbers each (as one,
// their rounding adds half as much again to the error of the output's own).  Operand layouts of that instruction, lane =
// i + 16 g: A: lane holds A[i][8g..8g+7]; B: lane holds B[8g..8g+7][i]; C/D: lane holds D[4g..4g+3][i].
//   - A load instruction takes 1 KB of consecutive positions (a lane has 16 bytes of one), as in the kernel above; the tile of 32 keys crosses
//     LDS, then the tile of values in the same place.  (Loaded straight into operand layout, an instruction takes 64 bytes of each of
//     sixteen positions.)
//   - Scores: A = keys (row = position), B = queries (column = head).  A lane reads its position's pieces K[position][32u + 8g .. +8]: one
//     operand each.
//   - The results D[position 4g+e][head i] of the block's two halves are, read the other way round, P^T[head i][positions
//     4g..4g+3 of each half]: exactly an A operand of the second contraction (row = head, k = position, in that order).  So the
//     probabilities never move between lanes.
//   - The second contraction wants B = values with k = position, i.e. values of ONE component from 2 x 4 consecutive positions
//     per lane, while the cache holds a position's components together: the tile is read by columns with the transposing read (ds_read_b64_tr_b16: of the 16
//     lanes of a group, lane s asks for four components of row s / 4 and lane l gets component l of all four rows; rows 2 D + 16
//     bytes apart, which spreads a read's sixteen rows evenly over the banks).
//   - Streaming softmax per head in the lanes that hold that head's column of S.  The sums are kept relative to a reference that only
//     follows, to 2^-ATT_BELOW of a block's maximum, when a block exceeds it by more than 2^ATT_LAG: a probability is then at most that
//     large, which fp16 holds as well as one below 1, and the accumulators, which are laid out by (head, component) and need the
//     factors from other lanes, are left alone in nearly every block.
// What bounds it: memory at long contexts (64/8 heads, 16001 positions, 65 MB over a ring of caches beyond the last-level cache: 15.8 us with the merge's launch, 17.6 before; one cache
// again and again stays in that and takes 13.2, before 16.4), and before that the loads of a compute unit.
// Us (64/8 heads, graph replay on one cache) of blocks of sixteen positions, 64-byte pieces and two-byte column reads / 32 positions and the transposing read / and loads of
// 1 KB / and nothing requested past a range's end: 16001 positions 16.9 / 16.9 / 13.9 / 13.0, 8000 11.2 / 11.6 / 10.3 / 9.5, 128 in one range 5.1 / 5.9 / 5.2 / 4.5.  Not faster where a
// wavefront has one block: 4096 positions over a ring 9.2 before, 9.4.
// RMAX (4, 8 or 16) is the number of query heads a workgroup serves from one pass over its keys and values: a group of up
// to RMAX heads takes one pass, a larger group (the paper's multi-query models: every head shares one key/value head) is
// cut into pieces of RMAX heads along the grid's second dimension.  D (64 or 128) is the head dimension: D / 32 pieces of
// 16 bytes per lane and position, D / 16 column groups of the weighted sum.
constexpr int ATT_BLOCK = 32;                                 // positions per wavefront and block
constexpr float ATT_BELOW = 7.f, ATT_LAG = 15.f;              // in units of log2

typedef _Float16 att_half8 __attribute__((ext_vector_type(8)));
typedef float att_float4 __attribute__((ext_vector_type(4)));
typedef short att_short4 __attribute__((ext_vector_type(4)));

// the maximum over the four lanes i, i + 16, i + 32, i + 48
__device__ __forceinline__ float max_of_rows(float x)
{
    const auto a = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
    x = fmaxf(__builtin_bit_cast(float, (uint32_t)a[0]), __builtin_bit_cast(float, (uint32_t)a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
    return fmaxf(__builtin_bit_cast(float, (uint32_t)b[0]), __builtin_bit_cast(float, (uint32_t)b[1]));
}

template <int RMAX, int D>
__global__ __launch_bounds__(64 * ATT_WAVES) void attn_decode_mfma_kernel(const uint16_t *__restrict__ q, const uint16_t *__restrict__ kc,
                                                                          const uint16_t *__restrict__ vc, uint16_t *__restrict__ out,
                                                                          float *__restrict__ ws, int n_heads, int group, int seq_len,
                                                                          int64_t head_stride /* halves */, int chunk, int nsplit,
                                                                          float scale_log2e)
{
    static_assert((RMAX == 4 || RMAX == 8 || RMAX == 16) && (D == 64 || D == 128), "group piece and head dimension");
    constexpr int NU = D / 32, NC = D / 16;
    constexpr int LANES = D / 8, LOADS = ATT_BLOCK * LANES / 64;      // lanes per position in a load; loads per block
    constexpr int VROW = 2 * D + 16;                          // bytes between rows of the staged tile: an odd number of 16-byte slots
    // a wavefront's tile of keys, then values, and, once its last block is done, its weighted sums [RMAX][D] for the merge
    constexpr int WAVE_BYTES = ATT_BLOCK * VROW > RMAX * D * 4 ? ATT_BLOCK * VROW : RMAX * D * 4;
    __shared__ __align__(16) uint8_t s_wave[ATT_WAVES][WAVE_BYTES];
    __shared__ float s_m[ATT_WAVES][16], s_l[ATT_WAVES][16];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, g = lane >> 4;
    const int j = blockIdx.x / nsplit, sp = blockIdx.x - j * nsplit;
    const int r0 = blockIdx.y * RMAX, rr = min(RMAX, group - r0);     // this workgroup's heads of the group: r0 .. r0 + rr - 1
    const int t_begin = sp * chunk, t_end = min(seq_len, t_begin + chunk);
    const AttRange keys(kc + (int64_t)j * head_stride + (int64_t)t_begin * D, t_end - t_begin, D);
    const AttRange values(vc + (int64_t)j * head_stride + (int64_t)t_begin * D, t_end - t_begin, D);

    // queries as B operands: lane (head li, g) holds Q[head][32u + 8g .. +8]; heads past the piece are zero
    att_half8 qb[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const att_u32x4 v = *reinterpret_cast<const att_u32x4 *>(q + (int64_t)(j * group + r0 + min(li, rr - 1)) * D + 32 * u + 8 * g);
        qb[u] = __builtin_bit_cast(att_half8, li < rr ? v : (att_u32x4){0u, 0u, 0u, 0u});
    }
    float m = -INFINITY, l = 0.f;                             // of head li (the reference is the same in the four lanes of a head)
    att_float4 oacc[NC];                                      // oacc[c][e] = O[head 4g+e][16c + li]
#pragma unroll
    for (int c = 0; c < NC; ++c) oacc[c] = (att_float4){0.f, 0.f, 0.f, 0.f};

    auto load_block = [&](att_u32x4 (&kt)[LOADS], att_u32x4 (&vt)[LOADS], int p0) {      // (past the range: zeros, scores masked below)
        const uint32_t byte = (uint32_t)(p0 - t_begin) * (2 * D) + lane * 16;
#pragma unroll
        for (int t = 0; t < LOADS; ++t) kt[t] = keys.load(byte + t * 1024);
#pragma unroll
        for (int t = 0; t < LOADS; ++t) vt[t] = values.load(byte + t * 1024);
    };
    uint8_t *myv = s_wave[wave];
    const uint8_t *column = myv + (4 * g + (li >> 2)) * VROW + 8 * (li & 3);  // what this lane asks for in a transposing read
    uint8_t *placed = myv + lane / LANES * VROW + 16 * (lane % LANES);        // where its part of a load goes
    auto turn = [] {                                          // (the wavefront's own tile: its LDS operations are served in order)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    auto process_block = [&](const att_u32x4 (&kt)[LOADS], const att_u32x4 (&vt)[LOADS], int p0) {
        // keys through the tile into operands: lane (position li of a half, g) takes the pieces 32u + 8g
#pragma unroll
        for (int t = 0; t < LOADS; ++t) *reinterpret_cast<att_u32x4 *>(placed + t * (64 / LANES) * VROW) = kt[t];
        turn();
        att_float4 sacc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const att_half8 a = *reinterpret_cast<const att_half8 *>(myv + (16 * h + li) * VROW + 64 * u + 16 * g);
                sacc[h] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, qb[u], sacc[h], 0, 0, 0);
            }
        turn();
        // values into the same tile
#pragma unroll
        for (int t = 0; t < LOADS; ++t) *reinterpret_cast<att_u32x4 *>(placed + t * (64 / LANES) * VROW) = vt[t];
        float sc[8], bm = -INFINITY;
#pragma unroll
        for (int e = 0; e < 8; ++e) {                         // position p0 + 16 (e / 4) + 4g + e % 4, head li
            sc[e] = (p0 + 16 * (e >> 2) + 4 * g + (e & 3) < t_end) ? sacc[e >> 2][e & 3] * scale_log2e : -INFINITY;
            bm = fmaxf(bm, sc[e]);
        }
        bm = max_of_rows(bm);                                 // the head's maximum over the block
        const bool follow = bm > m + ATT_LAG;                 // (the first block with a score above -inf: always)
        if (__builtin_amdgcn_ballot_w64(follow) != 0) {
            const float alpha = follow ? __builtin_amdgcn_exp2f(fmaxf(m - (bm - ATT_BELOW), -126.f)) : 1.0f;   // (never zero: an infinite sum stays infinite)
            const bool first = __builtin_amdgcn_ballot_w64(m != -INFINITY) == 0;
            l *= alpha;
            m = follow ? bm - ATT_BELOW : m;
            if (!first) {                                     // the accumulators hold heads 4g .. 4g+3: their factors live in lanes 4g .. 4g+3
                float al[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) al[e] = __shfl(alpha, 4 * g + e);
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int e = 0; e < 4; ++e) oacc[c][e] *= al[e];
            }
        }
        const float base = (m == -INFINITY) ? 0.f : m;        // (a head that has seen nothing above -inf: no -inf - -inf)
        // The probabilities as two fp16 numbers, 31/32 and what that leaves: the sum is within 2^-17 of p, and both are positive for every p above 2^-19 (half the smallest
        // fp16 number and the first one's rounding, 2^-25 each, against p / 32), so that an infinite value stays infinite down to 2^-26 of the maximum.  (One rounded number loses it
        // at 2^-25; with 1023/1024 the second one is zero for most p below 2^-15, and zero times infinity is a NaN.)
        att_half8 pa, pr;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float p = __builtin_amdgcn_exp2f(sc[e] - base);                     // exp2(-inf) = 0 for masked positions
            l += p;
            pa[e] = (_Float16)(p * (1.f - 0x1p-5f));
            pr[e] = (_Float16)(p - (float)pa[e]);
        }
        // weighted sums: B = values by columns
        turn();
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            typedef __attribute__((address_space(3))) att_short4 lds_short4;
            const att_short4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4 *)(column + 32 * c));
            const att_short4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4 *)(column + 16 * VROW + 32 * c));
            const att_half8 vb = __builtin_bit_cast(att_half8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            oacc[c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(pa, vb, oacc[c], 0, 0, 0);
            oacc[c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(pr, vb, oacc[c], 0, 0, 0);
        }
        turn();                                               // the next block overwrites the tile
    };

    att_u32x4 ka[LOADS], va[LOADS], kb[LOADS], vb2[LOADS];
    constexpr int STEP = ATT_BLOCK * ATT_WAVES;
    int p0 = t_begin + wave * ATT_BLOCK;
    load_block(ka, va, p0);                                   // (scheduling barriers: see attn_decode_kernel)
    __builtin_amdgcn_sched_barrier(0);
    load_block(kb, vb2, p0 + STEP);
    __builtin_amdgcn_sched_barrier(0);
    for (; p0 < t_end; p0 += 2 * STEP) {
        process_block(ka, va, p0);
        __builtin_amdgcn_sched_barrier(0);
        load_block(ka, va, p0 + 2 * STEP);
        __builtin_amdgcn_sched_barrier(0);
        if (p0 + STEP < t_end) process_block(kb, vb2, p0 + STEP);
        __builtin_amdgcn_sched_barrier(0);
        load_block(kb, vb2, p0 + 3 * STEP);
        __builtin_amdgcn_sched_barrier(0);
    }

    // ---- merge the four wavefronts' states ----------------------------------------------------------------------------------
    l += __shfl_xor(l, 16);                                   // a head's sum over its four lanes
    l += __shfl_xor(l, 32);
    if (g == 0) { s_m[wave][li] = m; s_l[wave][li] = l; }
    if (4 * g < RMAX) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) reinterpret_cast<float *>(myv)[(4 * g + e) * D + 16 * c + li] = oacc[c][e];
    }
    __syncthreads();
    float *ws_o = ws, *ws_m = ws + (int64_t)n_heads * ATT_D * ATT_MAX_SPLITS, *ws_l = ws_m + (int64_t)n_heads * ATT_MAX_SPLITS;
#pragma unroll
    for (int i = 0; i < RMAX * D / (64 * ATT_WAVES); ++i) {
        const int idx = tid + i * 64 * ATT_WAVES, r = idx / D, d = idx & (D - 1);
        float M = s_m[0][r];
#pragma unroll
        for (int w = 1; w < ATT_WAVES; ++w) M = fmaxf(M, s_m[w][r]);            // finite: the range is not empty
        M -= ATT_SPARE;
        float L = 0.f, O = 0.f;
#pragma unroll
        for (int w = 0; w < ATT_WAVES; ++w) {
            const float f = __builtin_amdgcn_exp2f(s_m[w][r] - M);
            L = __builtin_fmaf(s_l[w][r], f, L);
            O = __builtin_fmaf(reinterpret_cast<const float *>(s_wave[w])[idx], f, O);
        }
        if (r >= rr) break;                                   // (heads past the piece)
        const int head = j * group + r0 + r;
        if (nsplit == 1) {
            out[(int64_t)head * D + d] = as_u16((half_t)(O / L));
        } else {
            ws_o[((int64_t)head * ATT_MAX_SPLITS + sp) * ATT_D + d] = O;
            if (d == 0) { ws_m[(int64_t)head * ATT_MAX_SPLITS + sp] = M; ws_l[(int64_t)head * ATT_MAX_SPLITS + sp] = L; }
        }
    }
}

// Merge of the splits: one workgroup per query head, thread (d, u) for component d of splits 8u .. 8u + 7 (a state keeps 128 slots
// whatever the head dimension).  Only entries below nsplit are read (the rest of the workspace is whatever earlier calls left there, possibly
// never touched).  Every split is requested at once: one memory round trip, where one group of threads walking over the splits
// eight at a time takes up to eight (us per call, query / key-value heads, before -> after: 8/1, 8000 positions 10.8 -> 9.1; 128/8 of 64
// components, 4096 8.7 -> 7.8; 64/8, 16001 19.8 -> 19.3); the groups'
// states then meet in LDS and are added in order.
constexpr int ATT_MERGE = 8;                                  // splits per group of threads
__global__ __launch_bounds__(ATT_D * (ATT_MAX_SPLITS / ATT_MERGE)) void attn_merge_kernel(const float *__restrict__ ws, uint16_t *__restrict__ out, int n_heads,
                                                                                         int nsplit)
{
    constexpr int GROUPS = ATT_MAX_SPLITS / ATT_MERGE;
    __shared__ float s_o[GROUPS][ATT_D], s_m[GROUPS], s_l[GROUPS];
    const int head = blockIdx.x, head_dim = blockDim.x, d = threadIdx.x, group = threadIdx.y;
    const int groups = (nsplit + ATT_MERGE - 1) / ATT_MERGE;
    const float *ws_o = ws + (int64_t)head * ATT_MAX_SPLITS * ATT_D + d;
    const float *ws_m = ws + (int64_t)n_heads * ATT_D * ATT_MAX_SPLITS + (int64_t)head * ATT_MAX_SPLITS;
    const float *ws_l = ws_m + (int64_t)n_heads * ATT_MAX_SPLITS;
    float m[ATT_MERGE], l[ATT_MERGE], o[ATT_MERGE];
#pragma unroll
    for (int u = 0; u < ATT_MERGE; ++u) {
        const int i = min(group * ATT_MERGE + u, nsplit - 1); // past the end: the last range again (not added below)
        m[u] = ws_m[i]; l[u] = ws_l[i]; o[u] = ws_o[(int64_t)i * ATT_D];
    }
    float M = m[0], L = 0.f, O = 0.f;
#pragma unroll
    for (int u = 1; u < ATT_MERGE; ++u) M = fmaxf(M, m[u]);   // finite: no range is empty (a repeated range does not change the maximum)
    M -= ATT_SPARE;
#pragma unroll
    for (int u = 0; u < ATT_MERGE; ++u) {
        const bool there = group * ATT_MERGE + u < nsplit;    // (the sums are left out, not multiplied by zero: the last range's may be infinite)
        const float f = __builtin_amdgcn_exp2f(m[u] - M);
        L = __builtin_fmaf(there ? l[u] : 0.f, f, L);
        O = __builtin_fmaf(there ? o[u] : 0.f, f, O);
    }
    if (groups > 1) {                                         // (uniform over the workgroup)
        s_o[group][d] = O;
        if (d == 0) { s_m[group] = M; s_l[group] = L; }
        __syncthreads();
        if (group > 0) return;
        for (int u = 1; u < groups; ++u) M = fmaxf(M, s_m[u]);
        M -= ATT_SPARE;
        L = 0.f; O = 0.f;
        for (int u = 0; u < groups; ++u) {
            const float f = __builtin_amdgcn_exp2f(s_m[u] - M);
            L = __builtin_fmaf(s_l[u], f, L);
            O = __builtin_fmaf(s_o[u][d], f, O);
        }
    }
    out[(int64_t)head * head_dim + d] = as_u16((half_t)(O / L));
}

// Positions per split (a multiple of 64) and number of splits for a sequence length: about one workgroup per compute unit, and one range per key/value head, without
// the second launch, for short sequences.  Time of one range over that of ranges and merge, in graph replay / as separate calls: mean over head counts and caches of 1024, 4096 and 4160 positions a head [worst]:
//                                                        256 positions      288               320               352               384               448
//   matrix cores, 128 components (32/8, 64/8, 128/8, 8/1, 16/4, 64/16, 96/32 heads)
//                                                        .87 / .84 [.98]    .97 / .95 [1.06]  1.00 / .98 [1.12] 1.01 / .99 [1.08] 1.04 / 1.01 [1.13] 1.13 / 1.10 [1.26]
//   vector units, up to 16 key/value heads (16/16, 8/8, 4/4, 16/8)
//                                                        .78 / .66 [.89]    .88 / .73 [1.00]  .94 / .78 [1.04]  .98 / .82 [1.05]  1.01 / .84 [1.15]  1.16 / .97 [1.25]
//   vector units, more (32/32, 64/64, 64/32)             .79 / .71 [.96]    .88 / .80 [1.02]  .93 / .83 [1.08]  .92 / .83 [1.11]  .93 / .83 [1.17]   1.10 / 1.01 [1.33]
//   64 components (32/4, 16/16, 32/32, 128/8, 71/1)      .72 / .63 [.73]    .84 / .73 [.92]   .86 / .75 [.92]   .88 / .78 [.95]   .87 / .78 [.94]    .94 / .85 [1.04]
// The lines lie where graph replay breaks even, and for many heads on the vector units, where it depends on the caches most (32/32: 1.17 and .98 at 384), below.
// (A matrix-core workgroup has a block of 32 positions for two of its wavefronts in a range of 64; ranges of 128 instead: 64/8 at 1001 positions 6.6 -> 7.1.)
static void attn_geometry(int n_kv_heads, int head_dim, bool vector, int64_t seq_len, int cus, int *chunk, int *nsplit)
{
    int64_t want = ((int64_t)cus + n_kv_heads - 1) / n_kv_heads;
    if (seq_len <= (head_dim == 64 ? 384 : !vector ? 320 : n_kv_heads > 16 ? 256 : 352)) want = 1;
    if (want > ATT_MAX_SPLITS) want = ATT_MAX_SPLITS;
    int64_t c = (seq_len + want - 1) / want;
    c = (c + 63) / 64 * 64;
    *chunk = (int)c;
    *nsplit = (int)((seq_len + c - 1) / c);
}

size_t attn_workspace_bytes(int n_heads)
{
    return (size_t)n_heads * (ATT_D + 2) * ATT_MAX_SPLITS * sizeof(float);
}

hipError_t launch_attn_decode(const uint16_t *q, const uint16_t *k_cache, const uint16_t *v_cache, int n_heads, int n_kv_heads,
                              int head_dim, int64_t seq_len, int64_t max_seq, float scale, uint16_t *out, void *workspace, hipStream_t s)
{
    static PerDevice pd;
    int cus = 0;
    hipError_t e = once_per_device(pd, &cus, [] { return hipSuccess; });
    if (e != hipSuccess) return e;
    if (n_kv_heads < 1 || n_kv_heads > 64 || n_heads % n_kv_heads != 0 || seq_len < 1 || seq_len > max_seq) return hipErrorInvalidValue;
    if (head_dim != 64 && head_dim != 128) return hipErrorInvalidValue;
    const int R = n_heads / n_kv_heads;
    int chunk = 0, nsplit = 0;
    attn_geometry(n_kv_heads, head_dim, head_dim == 128 && R <= 2, seq_len, cus, &chunk, &nsplit);
    if (nsplit < 1 || nsplit > ATT_MAX_SPLITS) return hipErrorInvalidValue;
    const dim3 block(64 * ATT_WAVES);
    const float scale_log2e = scale * 1.4426950408889634f;
    const int64_t head_stride = max_seq * head_dim;
#define IFLOW_ATT_GO(RR) hipLaunchKernelGGL((attn_decode_kernel<RR>), dim3((unsigned)(n_kv_heads * nsplit)), block, 0, s, q, k_cache, \
        v_cache, out, static_cast<float *>(workspace), n_heads, (int)seq_len, head_stride, chunk, nsplit, scale_log2e)
#define IFLOW_ATT_GO_MFMA(RMAX, DD) hipLaunchKernelGGL((attn_decode_mfma_kernel<RMAX, DD>), \
        dim3((unsigned)(n_kv_heads * nsplit), (unsigned)((R + RMAX - 1) / RMAX)), block, 0, s, q, k_cache, v_cache, out, \
        static_cast<float *>(workspace), n_heads, R, (int)seq_len, head_stride, chunk, nsplit, scale_log2e)
    // one or two heads per key/value head at 128 components: the vector kernel; everything else on the matrix cores, in
    // pieces of 4, 8 or 16 heads
    if (head_dim == 128 && R == 1) IFLOW_ATT_GO(1);
    else if (head_dim == 128 && R == 2) IFLOW_ATT_GO(2);
    else if (head_dim == 128 && R <= 4) IFLOW_ATT_GO_MFMA(4, 128);
    else if (head_dim == 128 && R <= 8) IFLOW_ATT_GO_MFMA(8, 128);
    else if (head_dim == 128) IFLOW_ATT_GO_MFMA(16, 128);
    else if (R <= 4) IFLOW_ATT_GO_MFMA(4, 64);
    else if (R <= 8) IFLOW_ATT_GO_MFMA(8, 64);
    else IFLOW_ATT_GO_MFMA(16, 64);
#undef IFLOW_ATT_GO
#undef IFLOW_ATT_GO_MFMA
    e = hipGetLastError();
    if (e != hipSuccess || nsplit == 1) return e;
    hipLaunchKernelGGL(attn_merge_kernel, dim3((unsigned)n_heads), dim3((unsigned)head_dim, (unsigned)((nsplit + ATT_MERGE - 1) / ATT_MERGE)), 0, s,
                       static_cast<const float *>(workspace), out, n_heads, nsplit);
    return hipGetLastError();
}

// ---- the same call for callers that cannot allocate ------------------------------------------------------------
// The partial results of the position ranges live in a file-scope device array instead of a caller's workspace.  In
// host code the array's name is only a handle: its device address is asked for once per device (each device holds its
// own copy at its own address) and only that address is ever handed to a kernel.
constexpr int ATT_STATIC_MAX_HEADS = IFLOW_ATTN_STATIC_MAX_HEADS;
static __device__ __align__(256) float scratch[(size_t)ATT_STATIC_MAX_HEADS * (ATT_D + 2) * ATT_MAX_SPLITS];

hipError_t launch_attn_decode_static(const uint16_t *q, const uint16_t *k_cache, const uint16_t *v_cache, int n_heads, int n_kv_heads,
                                     int head_dim, int64_t seq_len, int64_t max_seq, float scale, uint16_t *out, hipStream_t s)
{
    static std::mutex lock;
    static float *address[IFLOW_MAX_DEVICES] = {};
    if (n_heads < 1 || n_heads > ATT_STATIC_MAX_HEADS) return hipErrorInvalidValue;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= IFLOW_MAX_DEVICES) return hipErrorInvalidDevice;
    float *ptr = nullptr;
    {
        std::lock_guard<std::mutex> hold(lock);
        if (!address[dev]) {
            void *sym = nullptr;
            e = hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch));
            if (e != hipSuccess) return e;
            if (!sym) return hipErrorInvalidSymbol;
            address[dev] = static_cast<float *>(sym);
        }
        ptr = address[dev];
    }
    return launch_attn_decode(q, k_cache, v_cache, n_heads, n_kv_heads, head_dim, seq_len, max_seq, scale, out, ptr, s);
}

}  // namespace iflow
