// ssd_prefill_scores: accumulated attention scores of a prompt that is processed at once
// (Algorithm 2: the scores of semantic heads are accumulated whenever attention weights exist, and a
// prefill is followed by a compression at once).  For every (layer, sequence, head) unit
//     a_i      = softmax over keys 0..i of scale * q_i . k_j        (causal)
//     score[j] = sum_{i >= j} a_i(j)
// which is what ssd_compress_kv's dense-source mode takes as score_src.
//
// This is the one step of the path that is a dense contraction (an n x n x d product per unit), so
// it runs on the matrix cores: 32 x 32 output tiles of Q K^T with v_mfma_f32_32x32x16_bf16 (bf16
// inputs, 8 k-values per lane and step) or v_mfma_f32_32x32x2_f32 (fp32 inputs).  Both operands keep their
// row-major [n, d] layout on the way, from memory or through LDS: lane l supplies row (l mod 32) and the k-slice
// selected by (l div 32), the same slice for Q and K, so nothing is transposed.
// A tile's 32 x 32 results sit 16 per lane: column = l mod 32, row = 8*(v/4) + 4*(l/32) + v%4.
//
// One workgroup per unit at a time.
// Prompts of up to 128 tokens (one block per wave; the case the decode path's prompts fall in): the workgroup
// fetches the unit's Q and K once, fully coalesced, and hands the matrix cores their fragments through LDS; the
// tiles are taken as K Q^T so that a query's softmax statistics stay inside a lane pair and only the column
// sums cross lanes; the logits stay in registers; workgroups are persistent and request the next unit's rows
// while working on the current one.  This form is bound by HBM: at n = 64, d = 128 a unit does 1 MFLOP on 32 KB,
// and what used to hold it back was the softmax bookkeeping on the vector ALUs (about 1100 instructions per
// wave with the queries along the registers, about 400 now), not the matrix cores or the memory.
// Longer prompts take two sweeps over the tiles on or below the diagonal -- the rows' maxima and sums, then the
// column sums -- in which one operand stays in registers and the other streams through LDS
// (prefill_scores_long_kernel).  Nothing is added across waves but in a fixed order (bit-reproducible, no atomics).
#include <cmath>
#include <type_traits>

#include "ssd_device.h"

namespace ssd {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

template <typename T> struct Mma;

template <> struct Mma<bf16_t> {
    static constexpr int KSTEP = 16;                 // k-values one MFMA consumes
    typedef uint4 Frag;                              // 8 bf16 per lane
    static __device__ __forceinline__ Frag load(const char *row, int ks, int half) {
        return *reinterpret_cast<const uint4 *>(row + (size_t)(ks * KSTEP + 8 * half) * 2);
    }
    static __device__ __forceinline__ f32x16_t mma(const Frag &a, const Frag &b, const f32x16_t &c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
    }
};

template <> struct Mma<float> {
    static constexpr int KSTEP = 2;
    typedef float Frag;                              // 1 float per lane
    static __device__ __forceinline__ Frag load(const char *row, int ks, int half) {
        return *reinterpret_cast<const float *>(row + (size_t)(ks * KSTEP + half) * 4);
    }
    static __device__ __forceinline__ f32x16_t mma(const Frag &a, const Frag &b, const f32x16_t &c) {
        return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
    }
};

struct PrefillArgs {
    const char *Q;
    const char *K;
    float *score_out;
    int n_units;
    int n;
    int row_bytes;
    float qscale;        // softmax scale * log2(e)
};

static __device__ __forceinline__ void write_scores(const PrefillArgs &a, const float *colsum, int waves, int unit) {
    __syncthreads();
    float *out = a.score_out + (size_t)unit * (size_t)a.n;
    for (int j = threadIdx.x; j < a.n; j += blockDim.x) {
        float t = colsum[j];
        for (int x = 1; x < waves; ++x) t += colsum[x * a.n + j];
        out[j] = t;
    }
}

// Fragment of an operand block that was staged in LDS: what Mma<T>::load takes from memory.
template <typename T> static __device__ __forceinline__ typename Mma<T>::Frag lds_frag(const unsigned char *row, int ks, int half);
template <> __device__ __forceinline__ uint4 lds_frag<bf16_t>(const unsigned char *row, int ks, int half) {
    return *reinterpret_cast<const uint4 *>(row + (ks * Mma<bf16_t>::KSTEP + 8 * half) * 2);
}
template <> __device__ __forceinline__ float lds_frag<float>(const unsigned char *row, int ks, int half) {
    return *reinterpret_cast<const float *>(row + (ks * Mma<float>::KSTEP + half) * 4);
}

// ---- tiles with the keys along the registers (short prompts) --------------------------------------------------
//
// The product is taken as K Q^T: a tile's 32 x 32 results then sit with the query along the lanes (column =
// lane mod 32) and the key along the registers (row = 8*(v/4) + 4*(lane/32) + v%4).  Every lane pair (l, l + 32)
// owns one query, so the softmax statistics of a row are sums and maxima over a lane's own registers plus one
// exchange between the halves -- no reduction over lanes -- and what is left to add up over lanes is the column
// sums, which only one lane per key has to end up with.

// One tile of scaled logits, masked where key > query (causal) or either lies beyond n.  `plain`: the tile lies
// below the diagonal and inside the prompt, nothing to mask.
template <typename T, int D>
static __device__ __forceinline__ void logits_tile_keys_in_regs(const typename Mma<T>::Frag (&kf)[D / Mma<T>::KSTEP],
                                                                const typename Mma<T>::Frag (&qa)[D / Mma<T>::KSTEP], int qb, int kb,
                                                                int n, int l32, int half, float qscale, bool plain, float (&z)[16]) {
    f32x16_t c = {0.f};
#pragma unroll
    for (int ks = 0; ks < D / Mma<T>::KSTEP; ++ks) c = Mma<T>::mma(kf[ks], qa[ks], c);
    if (plain) {                                           // wave-uniform
#pragma unroll
        for (int v = 0; v < 16; ++v) z[v] = c[v] * qscale;
        return;
    }
    const int query = qb * 32 + l32;
    const int key0 = kb * 32 + half * 4;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int key = key0 + (v >> 2) * 8 + (v & 3);
        z[v] = (key <= query && query < n) ? c[v] * qscale : NEG_BIG;      // key <= query < n implies key < n
    }
}

// Column sums of one tile: x[v] of lane l is the probability of key (v, l / 32) for query l mod 32; the sum over
// the 32 queries ends up in the 16 lanes of each half that have bit 1 of the lane index clear, lane l holding
// key row  8*(u/4) + 4*(l/32) + u%4  with  u = 8*bit4(l) + 4*bit3(l) + 2*bit2(l) + bit0(l).
// Five exchange steps (the two 16-lane rows of a half, then lanes 8 apart, mirrored within 8, neighbours,
// lanes 2 apart), each of the first four halving the values a lane still carries: 38 operations for the 512 sums.
static __device__ __forceinline__ float column_sums_over_lanes(const float (&x)[16], int lane) {
    float y[8], wv[4], r[2];
#pragma unroll
    for (int v = 0; v < 8; ++v) {                          // row 0 of the half keeps keys 0..7, row 1 keys 8..15
        const uint2v_t sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[v]), __float_as_uint(x[v + 8]), false, false);
        y[v] = __uint_as_float(sw.x) + __uint_as_float(sw.y);
    }
    const bool b3 = (lane & 8) != 0, b2 = (lane & 4) != 0, b0 = (lane & 1) != 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) wv[u] = (b3 ? y[u + 4] : y[u]) + dpp_f<0x128>(b3 ? y[u] : y[u + 4]);        // row_ror:8
#pragma unroll
    for (int u = 0; u < 2; ++u) r[u] = (b2 ? wv[u + 2] : wv[u]) + dpp_f<0x141>(b2 ? wv[u] : wv[u + 2]);     // row_half_mirror
    const float q = (b0 ? r[1] : r[0]) + dpp_f<0xB1>(b0 ? r[0] : r[1]);                                     // quad_perm [1,0,3,2]
    return q + dpp_f<0x4E>(q);                                                                              // quad_perm [2,3,0,1]
}
static __device__ __forceinline__ int column_sum_key_row(int lane) {       // the key row (0..31) the lane's sum belongs to
    const int u = ((lane >> 4) & 1) * 8 + ((lane >> 3) & 1) * 4 + ((lane >> 2) & 1) * 2 + (lane & 1);
    return (u >> 2) * 8 + (lane >> 5) * 4 + (u & 3);
}

// Prompts of at most KT blocks of 32 tokens: one wave per query block, launched with exactly that many waves.
// The unit's Q and K (two contiguous runs of n rows) are brought in by the whole workgroup with fully coalesced
// loads -- every wave-wide load is 1 KB of consecutive bytes, every byte is requested once per workgroup, all
// requests of a thread are in flight together -- and pass through LDS, from which each wave takes the fragments
// the matrix cores want (lane = row of the block, register = k-slice).  One staging area serves both operands:
// Q goes through it first (every wave leaves with its own query block in registers), then K, which stays for the
// tiles; K's requests are in flight all the while.  Rows are padded by 16 bytes in LDS: with that, the 16 lanes
// of one pass of a 16-byte LDS access hit the 64 banks exactly once, on the way in (16 lanes = 16 consecutive
// fragments of one row) and on the way out (16 lanes = 16 consecutive rows).
// The logits stay in registers between the two sweeps.
// A workgroup takes units blockIdx.x, blockIdx.x + gridDim.x, ... (the grid is sized to what the chip holds at
// once): the next unit's rows are requested as soon as this unit's have left the registers for LDS, so the
// memory pipe stays busy while the matrix cores and the softmax arithmetic work on the current unit.
template <typename T, int D, int KT>
__global__ __launch_bounds__(64 * KT) void prefill_scores_short_kernel(PrefillArgs a) {
    typedef typename Mma<T>::Frag Frag;
    constexpr int NK = D / Mma<T>::KSTEP;
    constexpr int ROW = D * (int)sizeof(T);                // bytes of a row in memory
    constexpr int STRIDE = ROW + 16;                       // ... and in LDS
    constexpr int FPR = ROW / 16;                          // 16-byte fragments per row
    constexpr int NF = FPR / 2;                            // fragments of one operand per thread: 32 rows per wave of 64 threads
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // = this wave's query block
    const int waves = blockDim.x >> 6;
    const int lane = threadIdx.x & 63;
    const int half = lane >> 5;
    const int l32 = lane & 31;
    const int n = a.n;
    const int n_pad = waves * 32;
    unsigned char *stage = lds_raw;                        // [n_pad][STRIDE]: Q, then K
    float *colsum = reinterpret_cast<float *>(lds_raw + (size_t)n_pad * STRIDE);     // [waves][n]
    float *mine = colsum + (size_t)w * n;

    // thread t owns fragments t, t + threads, ... of either operand (NF of them: n_pad * FPR in all)
    const int n_frag = n * FPR;
    const int step = (int)blockDim.x;
    u32x4_nt_t qv[NF], kv[NF];
    auto request = [&](int unit) {                         // clamped, unconditional: every request is out before the first wait
        const size_t unit_off = (size_t)unit * (size_t)n * (size_t)ROW;
        const char *Qu = a.Q + unit_off;
        const char *Ku = a.K + unit_off;
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            int f = (int)threadIdx.x + i * step;
            f = f < n_frag ? f : n_frag - 1;
            qv[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_nt_t *>(Qu + (size_t)f * 16));
        }
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            int f = (int)threadIdx.x + i * step;
            f = f < n_frag ? f : n_frag - 1;
            kv[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_nt_t *>(Ku + (size_t)f * 16));
        }
    };
    const u32x4_nt_t zero = {0u, 0u, 0u, 0u};
    auto to_lds = [&](const u32x4_nt_t (&v)[NF]) {
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            const int f = (int)threadIdx.x + i * step;
            if (f < n_pad * FPR)                           // rows past the prompt's end: zeros (masked later anyway)
                *reinterpret_cast<u32x4_nt_t *>(stage + (f / FPR) * STRIDE + (f % FPR) * 16) = f < n_frag ? v[i] : zero;
        }
    };
    // a wave only ever writes the columns of its own key blocks; the others stay zero for every unit
    for (int j = lane; j < n; j += 64) mine[j] = 0.f;

    int unit = (int)blockIdx.x;                            // < n_units (the grid is never larger)
    request(unit);
    for (;;) {
        to_lds(qv);
        __syncthreads();
        Frag qa[NK], kf[NK];
        {
            const unsigned char *qrow = stage + (size_t)(w * 32 + l32) * STRIDE;
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) qa[ks] = lds_frag<T>(qrow, ks, half);
        }
        __syncthreads();                                   // everybody has its query block: the area is free for K
        to_lds(kv);
        __syncthreads();
        const int next = unit + (int)gridDim.x;
        if (next < a.n_units) request(next);               // wave-uniform

        // logits of this query block against key blocks 0..w, kept in registers; running maximum per lane
        float z[KT][16];
        float m_lane = NEG_BIG;
        const bool whole = n == n_pad;                     // the prompt fills its last block: nothing lies beyond n
#pragma unroll
        for (int kb = 0; kb < KT; ++kb) {
            if (kb <= w) {
                const unsigned char *krow = stage + (size_t)(kb * 32 + l32) * STRIDE;
#pragma unroll
                for (int ks = 0; ks < NK; ++ks) kf[ks] = lds_frag<T>(krow, ks, half);
                logits_tile_keys_in_regs<T, D>(kf, qa, w, kb, n, l32, half, a.qscale, whole && kb < w, z[kb]);
#pragma unroll
                for (int v = 0; v < 16; ++v) m_lane = fmaxf(m_lane, z[kb][v]);
            }
        }
        // the query of lanes l and l + 32: maximum and sum over both halves' keys
        float h0, h1;
        halves_pair(m_lane, h0, h1);
        const float m_row = fmaxf(h0, h1);
        float l_lane = 0.f;
#pragma unroll
        for (int kb = 0; kb < KT; ++kb) {
            if (kb <= w) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {             // a masked logit gives exp2(-3e38 - m) = 0; a query beyond n is zeroed below
                    z[kb][v] = fast_exp2(z[kb][v] - m_row);
                    l_lane += z[kb][v];
                }
            }
        }
        halves_pair(l_lane, h0, h1);
        const float inv_l = (w * 32 + l32 < n) ? __builtin_amdgcn_rcpf(h0 + h1) : 0.f;
        const int key_row = column_sum_key_row(lane);
#pragma unroll
        for (int kb = 0; kb < KT; ++kb) {
            if (kb <= w) {
#pragma unroll
                for (int v = 0; v < 16; ++v) z[kb][v] *= inv_l;
                const float cs = column_sums_over_lanes(z[kb], lane);
                const int key = kb * 32 + key_row;
                if ((lane & 2) == 0 && key < n) mine[key] = cs;
            }
        }
        write_scores(a, colsum, waves, unit);              // starts with a barrier: every wave is done with the staged K
        if (next >= a.n_units) break;
        unit = next;
        // the next round's column sums are written only after three more barriers: write_scores' reads are long over
    }
}

// ---- prompts of more than 128 tokens ----------------------------------------------------------------------------
//
// Two sweeps over the 32 x 32 tiles on or below the diagonal, the same loop with the operands' roles exchanged:
//   sweep 1, K Q^T: queries stay, keys stream.  A lane pair (l, l + 32) owns one query, the tile's keys lie along
//            its registers: running maximum and sum of a query never leave the lane until one exchange at the end.
//   sweep 2, Q K^T: keys stay, queries stream.  A lane pair owns one key, the tile's queries lie along its
//            registers: the key's column sum never leaves the lane until one exchange at the end; the queries'
//            maxima and 1 / sums come from LDS as broadcasts.
// The operand that stays sits in registers (NS tiles per wave, fragment layout); the one that streams passes through
// LDS, STAGE rows at a time, fetched once per workgroup with coalesced loads a stage ahead and read by every wave, so a
// wave reads a streamed fragment once for its NS tiles.  A workgroup holds WAVES * NS tiles at a time and its waves
// pair tile w with tile WAVES * NS - 1 - w, so all of them meet the diagonal after the same amount of work.
// What bounds it: the vector ALUs' share.  Per tile and lane sweep 1 takes 16 exponentials (8 cycles each), 8 three-way
// maxima, 16 multiply-adds and 16 adds, sweep 2 16 exponentials and 32 multiply-adds: 300 cycles of a SIMD each,
// beside 256 of its matrix core (d = 128, bf16).  Keeping a whole row's exponentials instead of taking them twice
// would need 192 KB of registers per 32 queries at 1500 tokens.  Measured at 256 units of 1500 tokens (bf16, d = 128):
// 839 -> 195 us (counters: of the cycles its waves are resident the vector ALUs are busy in 50 %, the matrix cores in 35 %; the
// rest is the waves of a SIMD waiting for each other at the stages' barriers).  One wave per query block with all operands read from memory in fragment layout,
// which is what the 839 us were, touched 32 rows per load.  Tried on this form, no faster: 16 waves of one tile, 12 of
// two, stages of 128 rows, three stages with the next fragments read ahead, held tiles brought in through LDS, and
// one logarithm of the sum per query in place of maximum and 1 / sum (which doubles the error against 64 bits).
static __device__ __forceinline__ void arrived(uint4 &v) { asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w)); }
static __device__ __forceinline__ void arrived(float &v) { asm volatile("" : "+v"(v)); }

template <typename T> struct LongShape;
template <> struct LongShape<bf16_t> { static constexpr int NS = 2, STAGE = 64; };
template <> struct LongShape<float> { static constexpr int NS = 1, STAGE = 32; };      // (fp32 fragments take twice the registers and LDS)

template <typename T, int D, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void prefill_scores_long_kernel(PrefillArgs a) {
    typedef typename Mma<T>::Frag Frag;
    constexpr int NK = D / Mma<T>::KSTEP;
    constexpr int NS = LongShape<T>::NS, STAGE = LongShape<T>::STAGE;
    constexpr int ROW = D * (int)sizeof(T);
    constexpr int STRIDE = ROW + 16;                       // conflict-free both ways, as in the short kernel
    constexpr int FPR = ROW / 16;
    constexpr int THREADS = 64 * WAVES;
    constexpr int NF = STAGE * FPR / THREADS;              // 16-byte fragments per thread and stage
    static_assert(NF * THREADS == STAGE * FPR, "a stage divides evenly over the workgroup");
    constexpr int HELD = WAVES * NS;                       // tiles the workgroup holds at a time
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int half = lane >> 5;
    const int l32 = lane & 31;
    const int n = a.n;
    const int n_tiles = (n + 31) / 32;
    float *row_max = reinterpret_cast<float *>(lds_raw + 2 * STAGE * STRIDE);        // [n_tiles * 32]
    float *row_inv = row_max + n_tiles * 32;                                         // 1 / sum; 0 for queries beyond n
    const size_t unit_off = (size_t)blockIdx.x * (size_t)n * (size_t)ROW;

    auto sweep = [&](auto second, const char *held_base, const char *stream_base) {
        constexpr bool COLS = decltype(second)::value;     // sweep 2
        for (int first = 0; first < n_tiles; first += HELD) {
            int tile[NS];
            Frag keep[NS][NK];
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                tile[s] = first + (s == 0 ? w : HELD - 1 - w);
                int row = tile[s] * 32 + l32;
                row = row < n ? row : n - 1;               // rows past the end repeat the last one
#pragma unroll
                for (int ks = 0; ks < NK; ++ks) keep[s][ks] = Mma<T>::load(held_base + (size_t)row * ROW, ks, half);
            }
            // wait for them here: left pending across the loop below, every use of them would wait for the newest
            // request as well, which is the stage ahead
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int ks = 0; ks < NK; ++ks) arrived(keep[s][ks]);
            // sweep 1: of the lane's query, running maximum (log2 domain) and sum; sweep 2: of the lane's key, the
            // column sum as a compensated pair (one term per tile)
            float st0[NS], st1[NS];
#pragma unroll
            for (int s = 0; s < NS; ++s) { st0[s] = COLS ? 0.f : NEG_BIG; st1[s] = 0.f; }

            const int from = COLS ? first * 32 : 0;                                   // streamed rows [from, to)
            const int to = COLS ? n : (first + HELD) * 32 < n ? (first + HELD) * 32 : n;
            u32x4_nt_t ahead[NF];
            auto fetch = [&](int row0) {
#pragma unroll
                for (int i = 0; i < NF; ++i) {
                    const int f = (int)threadIdx.x + i * THREADS;
                    int r = row0 + f / FPR;
                    r = r < n ? r : n - 1;
                    ahead[i] = *reinterpret_cast<const u32x4_nt_t *>(stream_base + (size_t)r * ROW + (f % FPR) * 16);
                }
            };
            auto stash = [&](int buf) {
#pragma unroll
                for (int i = 0; i < NF; ++i) {
                    const int f = (int)threadIdx.x + i * THREADS;
                    *reinterpret_cast<u32x4_nt_t *>(lds_raw + buf * (STAGE * STRIDE) + (f / FPR) * STRIDE + (f % FPR) * 16) = ahead[i];
                }
            };
            auto fragments = [&](int buf, int sub, Frag (&fr)[NK]) {
                const unsigned char *frow = lds_raw + buf * (STAGE * STRIDE) + (sub * 32 + l32) * STRIDE;
#pragma unroll
                for (int ks = 0; ks < NK; ++ks) fr[ks] = lds_frag<T>(frow, ks, half);
            };
            auto product = [&](const Frag (&fr)[NK], int s) {
                f32x16_t c = {0.f};
#pragma unroll
                for (int ks = 0; ks < NK; ++ks) c = Mma<T>::mma(fr[ks], keep[s][ks], c);
                return c;
            };
            // rm, ri: maxima and 1 / sums of the tile's queries, register by register (sweep 2)
            // A logit that is not a number counts as masked; the tests for it look at one value per lane and tile.
            auto absorb = [&](f32x16_t &c, int s, const float (&rm)[16], const float (&ri)[16]) {
                float p0 = 0.f, p1 = 0.f;
                auto drop_nan = [&]() {
#pragma unroll
                    for (int v = 0; v < 16; ++v) c[v] = c[v] == c[v] ? c[v] : -INFINITY;
                };
                if constexpr (!COLS) {
                    auto tile_max = [&]() {
                        float mx = c[0];
#pragma unroll
                        for (int v = 1; v < 16; ++v) mx = __builtin_elementwise_maximum(mx, c[v]);       // NaN if one of them is
                        return mx;
                    };
                    float mx = tile_max();
                    if (__any(mx != mx)) { drop_nan(); mx = tile_max(); }
                    const float m_new = fmaxf(st0[s], mx * a.qscale);                 // qscale > 0; finite also where all keys are masked
#pragma unroll
                    for (int v = 0; v < 16; v += 2) {
                        p0 += fast_exp2(fmaf(c[v], a.qscale, -m_new));
                        p1 += fast_exp2(fmaf(c[v + 1], a.qscale, -m_new));
                    }
                    st1[s] = fmaf(st1[s], fast_exp2(st0[s] - m_new), p0 + p1);
                    st0[s] = m_new;
                } else {
#pragma unroll
                    for (int v = 0; v < 16; v += 2) {
                        p0 = fmaf(fast_exp2(fmaf(c[v], a.qscale, -rm[v])), ri[v], p0);
                        p1 = fmaf(fast_exp2(fmaf(c[v + 1], a.qscale, -rm[v + 1])), ri[v + 1], p1);
                    }
                    if (__any(p0 + p1 != p0 + p1)) {
                        drop_nan();
                        p0 = p1 = 0.f;
#pragma unroll
                        for (int v = 0; v < 16; ++v) p0 = fmaf(fast_exp2(fmaf(c[v], a.qscale, -rm[v])), ri[v], p0);
                    }
                    // st0 + st1 += p0 + p1 without losing what st0 cannot hold (terms are not negative, so sums over
                    // thousands of queries would otherwise drift by a rounding per tile)
                    const float add = (p0 + p1) + st1[s];
                    const float sum = st0[s] + add;
                    st1[s] = add - (sum - st0[s]);
                    st0[s] = sum;
                }
            };
            auto streamed = [&](int buf, int sub, int t) {          // one streamed tile against the tiles this wave holds
                bool on[NS], any = false;                  // on or below the diagonal (wave-uniform)
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    on[s] = t < n_tiles && tile[s] < n_tiles && (COLS ? t >= tile[s] : t <= tile[s]);
                    any = any || on[s];
                }
                if (!any) return;
                Frag fr[NK];
                fragments(buf, sub, fr);
                float rm[16], ri[16];
                if constexpr (COLS) {
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const float4 x = *reinterpret_cast<const float4 *>(row_max + t * 32 + 8 * g + 4 * half);
                        const float4 y = *reinterpret_cast<const float4 *>(row_inv + t * 32 + 8 * g + 4 * half);
                        ri[4 * g] = y.x; ri[4 * g + 1] = y.y; ri[4 * g + 2] = y.z; ri[4 * g + 3] = y.w;
                        rm[4 * g] = x.x; rm[4 * g + 1] = x.y; rm[4 * g + 2] = x.z; rm[4 * g + 3] = x.w;
                    }
                }
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    if (!on[s]) continue;
                    f32x16_t c = product(fr, s);
                    // register v of the tile is streamed row 8*(v/4) + 4*half + v%4; the diagonal tile is masked where key > query
                    if (t == tile[s]) {
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            const int r = (v >> 2) * 8 + half * 4 + (v & 3);
                            c[v] = (COLS ? l32 <= r : r <= l32) ? c[v] : -INFINITY;
                        }
                    }
                    absorb(c, s, rm, ri);
                }
            };
            fetch(from);
            __syncthreads();                               // everybody is done with the buffers (and, sweep 2, the statistics are written)
            stash(0);
            int cur = 0;
            for (int row0 = from; row0 < to; row0 += STAGE, cur ^= 1) {
                __syncthreads();                           // this stage is in LDS, the other buffer is free
                const bool more = row0 + STAGE < to;
                if (more) fetch(row0 + STAGE);
                for (int sub = 0; sub < STAGE / 32; ++sub) streamed(cur, sub, row0 / 32 + sub);
                if (more) stash(cur ^ 1);
            }
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                if (tile[s] >= n_tiles) continue;
                const int row = tile[s] * 32 + l32;        // this lane's query or key
                float x, y;
                if constexpr (!COLS) {
                    halves_pair(st0[s], x, y);
                    const float m_row = fmaxf(x, y);
                    halves_pair(st1[s] * fast_exp2(st0[s] - m_row), x, y);
                    if (half == 0) {
                        row_max[row] = m_row;
                        row_inv[row] = row < n && x + y > 0.f ? 1.0f / (x + y) : 0.f;      // (0: every logit of the query masked)
                    }
                } else {
                    halves_pair(st0[s], x, y);
                    if (half == 0 && row < n) a.score_out[(size_t)blockIdx.x * (size_t)n + row] = x + y;
                }
            }
        }
    };
    sweep(std::false_type{}, a.Q + unit_off, a.K + unit_off);
    sweep(std::true_type{}, a.K + unit_off, a.Q + unit_off);
}

// LDS of the long kernel: two stages of the streamed operand and the queries' statistics.
template <typename T> static size_t long_lds_bytes(int n, int row_bytes) {
    return 2 * (size_t)LongShape<T>::STAGE * (size_t)(row_bytes + 16) + (size_t)((n + 31) / 32 * 32) * 2 * sizeof(float);
}

// Grid of a kernel whose workgroups walk the units with a stride of the grid size: as many workgroups as are
// resident at once (workgroups per compute unit x compute units of the current device), trimmed so that every
// workgroup gets the same number of units, give or take one at the very end.  0 on failure.
static dim3 resident_grid(int n_units, int per_cu) {
    int dev = 0, cus = 0;
    if (per_cu < 1 || hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        return dim3(0);
    const long long resident = (long long)per_cu * cus;
    const long long rounds = (n_units + resident - 1) / resident;
    return dim3((unsigned)((n_units + rounds - 1) / rounds));
}

// LDS of the short kernel: the staging area of one operand and the waves' column sums.
static size_t short_lds_bytes(int waves, int n, int row_bytes) {
    return (size_t)(waves * 32) * (size_t)(row_bytes + 16) + (size_t)waves * (size_t)n * sizeof(float);
}

}  // namespace ssd

using namespace ssd;

extern "C" int ssd_prefill_scores(const void *Q, const void *K, int n_units, int n_src, int d, int dtype, float softmax_scale,
                                  float *score_out, void *stream) {
    clear_error();
    if (!Q || !K || !score_out) return fail(SSD_ERR_INVALID_ARG, "Q, K or score_out is NULL");
    if (!aligned(Q, 16) || !aligned(K, 16) || !aligned(score_out, 4)) return fail(SSD_ERR_INVALID_ARG, "Q / K must be 16-byte aligned");
    if (n_units < 1) return fail(SSD_ERR_INVALID_ARG, "n_units=%d must be >= 1", n_units);
    if (n_src < 1 || n_src > 4096) return fail(SSD_ERR_INVALID_ARG, "n_src=%d outside 1..4096", n_src);
    if (d != 64 && d != 128) return fail(SSD_ERR_INVALID_ARG, "head_dim=%d, supported: 64, 128", d);
    if (dtype != SSD_F32 && dtype != SSD_BF16) return fail(SSD_ERR_INVALID_ARG, "bad dtype");
    if (!(softmax_scale >= 0.f) || !std::isfinite(softmax_scale)) return fail(SSD_ERR_INVALID_ARG, "softmax_scale must be finite and >= 0");
    PrefillArgs a;
    a.Q = static_cast<const char *>(Q);
    a.K = static_cast<const char *>(K);
    a.score_out = score_out;
    a.n_units = n_units;
    a.n = n_src;
    a.row_bytes = d * (dtype == SSD_F32 ? 4 : 2);
    a.qscale = (softmax_scale > 0.f ? softmax_scale : 1.0f / sqrtf((float)d)) * LOG2E;
    const int n_blocks = (n_src + 31) / 32;
    const int waves = n_blocks < 4 ? n_blocks : 4;
    const size_t lds_short = short_lds_bytes(waves, n_src, a.row_bytes);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const dim3 grid((unsigned)n_units), block(64u * waves);
    hipError_t attr = hipSuccess;
    // more than 64 KB of dynamic LDS has to be asked for (the longest short prompts in fp32: 70 KB of the CU's 160 KB)
#define SSD_PREFILL_SHORT(T_, D_, KT_)                                                                                          \
    do {                                                                                                                        \
        const void *fn = reinterpret_cast<const void *>(&prefill_scores_short_kernel<T_, D_, KT_>);                             \
        if (lds_short > 65536) attr = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_short);      \
        int per_cu = 0;                                                                                                         \
        if (attr == hipSuccess) attr = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, (int)block.x, lds_short);      \
        if (attr == hipSuccess) {                                                                                               \
            const dim3 g = resident_grid(n_units, per_cu);                                                                      \
            if (g.x == 0) attr = hipErrorInvalidValue;                                                                          \
            else hipLaunchKernelGGL((prefill_scores_short_kernel<T_, D_, KT_>), g, block, lds_short, s, a);                     \
        }                                                                                                                       \
    } while (0)
#define SSD_PREFILL_LONG(T_, D_, WAVES_)                                                                                         \
    do {                                                                                                                        \
        const void *fn = reinterpret_cast<const void *>(&prefill_scores_long_kernel<T_, D_, WAVES_>);                           \
        const size_t lds = long_lds_bytes<T_>(n_src, a.row_bytes);                                                              \
        if (lds > 65536) attr = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);                  \
        if (attr == hipSuccess) hipLaunchKernelGGL((prefill_scores_long_kernel<T_, D_, WAVES_>), grid, dim3(64 * WAVES_), lds, s, a); \
    } while (0)
#define SSD_PREFILL(T_, D_)                                                                                          \
    do {                                                                                                             \
        if (n_blocks <= 2) SSD_PREFILL_SHORT(T_, D_, 2);                                                             \
        else if (n_blocks <= 4) SSD_PREFILL_SHORT(T_, D_, 4);                                                        \
        else if (n_blocks <= 8) SSD_PREFILL_LONG(T_, D_, 4);                                                         \
        else SSD_PREFILL_LONG(T_, D_, 8);                                                                            \
    } while (0)
    if (dtype == SSD_BF16) {
        if (d == 128) SSD_PREFILL(bf16_t, 128); else SSD_PREFILL(bf16_t, 64);
    } else {
        if (d == 128) SSD_PREFILL(float, 128); else SSD_PREFILL(float, 64);
    }
#undef SSD_PREFILL
#undef SSD_PREFILL_LONG
#undef SSD_PREFILL_SHORT
    if (attr != hipSuccess) return hip_fail(attr, "prefill score kernel attribute");
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "prefill score launch");
    return SSD_OK;
}
