// ssd_prefill_scores: accumulated attention scores of a prompt that is processed at once
// (Algorithm 2: the scores of semantic heads are accumulated whenever attention weights exist, and a
// prefill is followed by a compression at once).  For every (layer, sequence, head) unit
//     a_i      = softmax over keys 0..i of scale * q_i . k_j        (causal)
//     score[j] = sum_{i >= j} a_i(j)
// which is what ssd_compress_kv's dense-source mode takes as score_src.
//
// This is the one step of the path that is a dense contraction (an n x n x d product per unit), so it runs on the matrix cores,
// in tiles of 32 x 32.  Both operands keep their row-major [n, d] layout on the way, from memory or through LDS: a lane supplies
// one row and the same k-slice of Q and of K, so nothing is transposed.  Short prompts take v_mfma_f32_32x32x16_bf16 (8 k-values
// per lane and step) or v_mfma_f32_32x32x2_f32, whose results sit 16 per lane, column = l mod 32, row = 8*(v/4) + 4*(l/32) + v%4; long
// ones 16 x 16 products (mma_fragment).
//
// Prompts of up to 128 tokens (one block per wave; the case the decode path's prompts fall in): the workgroup
// fetches the unit's Q and K once, fully coalesced, and hands the matrix cores their fragments through LDS; the
// tiles are taken as K Q^T so that a query's softmax statistics stay inside a lane pair and only the column
// sums cross lanes; the logits stay in registers; workgroups are persistent and request the next unit's rows
// while working on the current one.  This form is bound by HBM: at n = 64, d = 128 a unit does 1 MFLOP on 32 KB,
// and what used to hold it back was the softmax bookkeeping on the vector ALUs (about 1100 instructions per
// wave with the queries along the registers, about 400 now), not the matrix cores or the memory.
// Longer prompts take two sweeps over the tiles on or below the diagonal -- the rows' sums, then the column sums -- in
// which one operand stays in registers and the other streams through LDS (prefill_scores_long_kernel).
// Nothing is added across waves but in a fixed order (bit-reproducible, no atomics).
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
    int cut[5];          // long prompts: workgroup y of a unit takes the keys of tiles [cut[y], cut[y + 1])
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
// KEEP: K is read like what will be needed again (when, and why, stands at the launch).
template <typename T, int D, int KT, bool KEEP>
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
            const u32x4_nt_t *p = reinterpret_cast<const u32x4_nt_t *>(Ku + (size_t)f * 16);
            kv[i] = KEEP ? *p : __builtin_nontemporal_load(p);
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
// Two sweeps over the 32 x 32 tiles on or below the diagonal, both taken as K Q^T: a lane has two queries of a tile and eight of
// its keys for each, so a query lies in the four lanes l, l + 16, l + 32, l + 48.
//   sweep 1: queries stay, keys stream.  A query's sum of exponentials never leaves its lanes until one exchange at the end.
//   sweep 2: keys stay, queries stream.  Every lane adds up its own queries' probabilities, key by key; the 16 lanes of a key
//            meet every eight tiles.  A streamed query's maximum and 1 / sum are two registers of its lane.
// The operand that stays sits in registers (NS tiles per wave, fragment layout); the one that streams passes through LDS, a
// stage of up to four tiles (32 KB) at a time in two buffers, requested from memory straight into LDS while the stage before
// it is worked on, across the ends of groups and of sweeps as well.  Fragment f of 16 bytes of row r sits at f ^ r (low bits),
// so that the 16 rows that one pass of a 16-byte LDS access reads hit the 64 banks exactly once.
//
// The reference that a query's exponentials are taken against is the largest logit of its first streamed tile, one for the four lanes
// that share the query, and stays while it can: a maximum per tile, the rescaling and the chain through both are a fifth of the vector
// ALUs' work.  Logits above it cost precision -- an argument x of an exponential is rounded to 2^-24 x, where against a running maximum
// the heavy terms' arguments stay near zero -- so where a stage would bring a lane's sum to 2^20 or makes it no number, the stage's tiles
// are taken again with the reference renewed tile by tile.  Error against 64 bits over a running maximum's (fp32 and bf16, 200 to 1500
// tokens): logits that rise by 2^16 to 2^28 0.98 on average and 1.08 at most, by 2^40 to 2^90 1.00 and 1.08; with that line at 2^100
// 1.01 and 1.13, 1.06 and 1.23.  Tested per stage it costs nothing where nothing rises (256 units of 1500 tokens 168 us, 300 of 640 76.6;
// tested per tile 170 and 77.2) and where all queries' logits rise by 2^24 at once 181 us (170; whole groups of held tiles taken again
// 271).  (The lanes' sums are of one scale: with a reference per lane, a lane whose first keys lie 2^126 below the others' would lose
// what it has added up since.)
//
// What bounds it: a 32 x 32 x 128 product takes a SIMD 256 cycles of its matrix core and 16 exponentials (8 cycles each), 16
// multiply-adds and 16 adds per lane, 260 cycles of its vector ALUs, beside each other where two waves alternate.  The loop by
// itself, with random data, takes 200 ns per product: what a large bf16 matrix product takes on this card, which clocks lower
// under such loads (160 ns with zeros).  256 units of 1500 tokens (bf16, d = 128): 839 us with all operands read from memory in
// fragment layout, 195 with 32 x 32 products and column sums that crossed lanes per tile (whose LDS reads and barriers the
// waves spent half their time on), 165 to 182 now, by the card's clock; of these 113 are the loop, the rest groups' beginnings (a held tile's loads touch a row
// per lane) and diagonals (waves that have less to do wait).  Error against 64 bits 4.3e-8 -> 3.6e-8 (n = 256: 4.7e-8 both).
// Few units: up to 128 leave half of the compute units idle, so two or three workgroups share a unit's keys; each goes through sweep 1
// for the queries that see any of its keys, so the gain is less than their number (32 units of 1500 tokens: 168 -> 141 us in one
// piece, 120 in two, 105 to 112 in three; four as much).
// More than 256 units: four waves per workgroup, two workgroups on a compute unit fill each other's waits and no round is left half empty
// (d = 128, bf16: 300 units of 1500 tokens 354 us before, 307 with eight waves, 293 with four; 512 of 640 103, 87, 80).  Not where
// LDS has room for one (rows of 256 bytes and more, from 2017 tokens on: its statistics grow with the prompt), which would leave a SIMD
// one wave: 300 units of 2049 tokens 663 us before, 814 with four waves, 567 with eight; of 4096 2304, 2960, 2096; fp32, d = 64,
// 300 of 2049 2720, 3101, 2709.  Nor in fp32 with d = 64, whose eight waves need so few registers that two workgroups fit as well: 300 units of 400
// tokens 152 us with four waves, 138 with eight, 1024 of 129 76 and 67.  bf16 with d = 64 holds three workgroups of four waves, 768 units
// at once, or, in 128 registers, two of eight, 512 units, which are better where they need no more rounds and the prompt fills
// them: 300 units of 400 tokens 34.4 -> 31.2 us (30.6 before), of 1000 118 -> 107 (111), 1024 of 400 65.5 -> 61.1 (59), but 600 of 640
// tokens 78.4 and 89.1, 512 of 129 12.9 and 13.8.
// NS = 3 where it takes a group less than NS = 2 (256 units of 640 tokens 51.0 with two and 45.2 us with three, of 1000, where it takes as many, 90.8 and 92.2).
template <int ROW> static constexpr int long_stage_tiles() { return 1024 / ROW < 4 ? 1024 / ROW : 4; }

static __device__ __forceinline__ void arrived(uint4 &v) { asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w)); }

// Products of 16 x 16 with 32 bf16 (16x16x32) or 4 x 4 fp32 (16x16x4) k-values per 16-byte fragment: lane l supplies row l mod 16 of its
// operand and the k-slice of its fragment, l / 16 of four; results: column l mod 16, rows 4 (l / 16) .. + 3.  Not the 32 x 32 forms: a
// chain of those that starts anew (addend zero) with other operands costs 170 to 190 ns per 32 x 32 x 128 where it
// should be 110 (two waves per SIMD; 16 x 16: 110, and 130 for 190 with random data, which the card clocks lower).
typedef float f32x4_t __attribute__((ext_vector_type(4)));
template <typename T> static __device__ __forceinline__ f32x4_t mma_fragment(const uint4 &a, const uint4 &b, f32x4_t c);
template <> __device__ __forceinline__ f32x4_t mma_fragment<bf16_t>(const uint4 &a, const uint4 &b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}
template <> __device__ __forceinline__ f32x4_t mma_fragment<float>(const uint4 &a, const uint4 &b, f32x4_t c) {
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
}

// Sums over the 16 lanes of a row: lane l ends up with the sum of x[u], u = 4 bit3(l) + 2 bit2(l) + bit0(l).  The steps in which a
// rounding is one of a whole sum are taken in double.
template <int CTRL> static __device__ __forceinline__ double dpp_d(double v) {
    return __longlong_as_double((long long)dpp_u64<CTRL>((unsigned long long)__double_as_longlong(v)));
}
static __device__ __forceinline__ double sums_over_16_lanes(const float (&x)[8], int lane) {
    float y[4];
    double r[2];
    const bool b3 = (lane & 8) != 0, b2 = (lane & 4) != 0, b0 = (lane & 1) != 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) y[u] = (b3 ? x[u + 4] : x[u]) + dpp_f<0x128>(b3 ? x[u] : x[u + 4]);         // row_ror:8
#pragma unroll
    for (int u = 0; u < 2; ++u) r[u] = (double)(b2 ? y[u + 2] : y[u]) + (double)dpp_f<0x141>(b2 ? y[u] : y[u + 2]);      // row_half_mirror
    const double q = (b0 ? r[1] : r[0]) + dpp_d<0xB1>(b0 ? r[0] : r[1]);                                    // quad_perm [1,0,3,2]
    return q + dpp_d<0x4E>(q);                                                                              // quad_perm [2,3,0,1]
}

// PER_SIMD: waves that the registers let a SIMD hold at least.
template <typename T, int D, int WAVES, int NS, int PER_SIMD>
__global__ __launch_bounds__(64 * WAVES, PER_SIMD) void prefill_scores_long_kernel(PrefillArgs a) {
    constexpr bool AHEAD = sizeof(T) == 2 && PER_SIMD <= 2;                // fragments a tile ahead (registers: fp32 fragments take twice as many)
    constexpr int ROW = D * (int)sizeof(T);
    constexpr int FPR = ROW / 16;                          // 16-byte fragments per row
    constexpr int NK = FPR / 4;                            // ... per lane and 16 rows of an operand's tile
    constexpr int ST = long_stage_tiles<ROW>();
    constexpr int STAGE_BYTES = ST * 32 * ROW;
    static_assert((ST & (ST - 1)) == 0 && 8 % ST == 0, "eight tiles are whole stages");
    static_assert(STAGE_BYTES % 1024 == 0 && 64 % FPR == 0, "a stage is brought in by wave-wide transfers of whole rows");
    constexpr int HELD = WAVES * NS;                       // tiles the workgroup holds at a time
    constexpr float LARGE = 1048576.f;                     // 2^20, see above
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int l16 = lane & 15, quarter = lane >> 4;
    const int n = a.n;
    const int n_tiles = (n + 31) / 32;
    float2 *stat = reinterpret_cast<float2 *>(lds_raw + 2 * STAGE_BYTES);           // [n_tiles * 32]: maximum (or reference) and 1 / sum; 1 / sum = 0 beyond n
    const size_t unit_off = (size_t)blockIdx.x * (size_t)n * (size_t)ROW;
    const char *Qu = a.Q + unit_off, *Ku = a.K + unit_off;
    auto swizzle = [](int row) { return (FPR == 8 ? row >> 1 : row) & (FPR == 8 ? 7 : 15); };

    // Where a wave's tiles lie in a group: w and HELD - 1 - w, so that all waves meet the diagonal after the same amount of work
    // (NS == 2); counted back and forth so that the waves of a SIMD (w, w + 4, ...) also share it evenly within a stage.
    const int place = (w & ~3) + ((w & 4) ? 3 - (w & 3) : w & 3);

    // Request of one stage, from memory straight into LDS: the wave's share of transfers of 1 KB, lane i's 16 bytes to the i-th
    // place.  Which fragment sits there is the swizzle's choice.  The compiler does not count these transfers: `landed` waits for them.
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds_raw;
    auto request = [&](const char *base, int tile, int buf) {
        for (int i = w; i < STAGE_BYTES / 1024; i += WAVES) {
            const int row = i * (64 / FPR) + lane / FPR;   // of the stage
            int r = tile * 32 + row;
            r = r < n ? r : n - 1;                         // rows past the end repeat the last one
            const uint32_t from = (uint32_t)r * ROW + (uint32_t)((lane % FPR) ^ swizzle(row)) * 16u;
            const uint32_t to = __builtin_amdgcn_readfirstlane(lds_base + buf * STAGE_BYTES + i * 1024);
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"            // m0 is reserved: named all the same, so that its next use sets it anew
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(to), "v"(from), "s"(base) : "memory", "m0");
#pragma clang diagnostic pop
        }
    };
    auto landed = [&]() { asm volatile("s_waitcnt vmcnt(0)" : : : "memory"); };
    const int frag0 = l16 * ROW + (quarter ^ swizzle(l16)) * 16;                     // of a tile's first fragment, and ^ 64 ks; + 16 rows
    auto fragments = [&](int buf, int j, uint4 (&fr)[2][NK]) {
        const int at = buf * STAGE_BYTES + j * (32 * ROW) + frag0;
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) fr[g][ks] = *reinterpret_cast<const uint4 *>(lds_raw + ((at ^ (ks * 64)) + g * (16 * ROW)));
    };

    // Stages in the order they are needed: of sweep 1, held tiles from `begin` on, streamed tiles 0 .. the last held one; of sweep 2,
    // held tiles [begin, stop), streamed tiles from the first held one's stage on (stages lie at multiples of ST, see the fold below).
    // ahead_*: the stage to request next.
    const int begin = a.cut[blockIdx.y], stop = a.cut[blockIdx.y + 1];      // this workgroup's keys, in tiles
    if (begin >= stop) return;
    int ahead_sweep = 0, ahead_first = begin, ahead_tile = 0;
    int cur = 0;                                           // LDS buffer of the stage at hand
    auto request_next = [&](int buf) {
        if (ahead_sweep > 1) return;
        request(ahead_sweep ? Qu : Ku, ahead_tile, buf);
        ahead_tile += ST;
        if (ahead_tile >= (ahead_sweep == 0 && ahead_first + HELD < n_tiles ? ahead_first + HELD : n_tiles)) {
            ahead_first += HELD;
            if (ahead_first >= (ahead_sweep ? stop : n_tiles)) { ++ahead_sweep; ahead_first = begin; }
            ahead_tile = ahead_sweep ? ahead_first & ~(ST - 1) : 0;
        }
    };
    // One group of held tiles; its first stage is requested.  Returns false if a column sum is not a number (CAREFUL: never).
    auto group = [&](auto cols, auto careful, int first, int end) __attribute__((always_inline)) -> bool {
        constexpr bool COLS = decltype(cols)::value, CAREFUL = decltype(careful)::value;
        const char *held_base = COLS ? Ku : Qu;
        int tile[NS];
        uint4 keep[NS][2][NK];
        landed();
        __syncthreads();                                   // the first stage is in LDS (and the statistics are), the other buffer is free
        request_next(cur ^ 1);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            tile[s] = first + s * WAVES + (s & 1 ? WAVES - 1 - place : place);
            if (tile[s] >= end) { tile[s] = n_tiles; continue; }        // none (its loads would all read one row: 8 % of a launch of 256 units of 129 tokens)
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                int row = tile[s] * 32 + g * 16 + l16;
                row = row < n ? row : n - 1;
#pragma unroll
                for (int ks = 0; ks < NK; ++ks) keep[s][g][ks] = *reinterpret_cast<const uint4 *>(held_base + (size_t)row * ROW + (4 * ks + quarter) * 16);
            }
        }
        // wait for them here: left pending across the loop below, every use of them would wait for the newest request as well
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int i = 0; i < 2 * NK; ++i) arrived(keep[s][i / NK][i % NK]);
        float ref[NS][2], sum[NS][2];                      // sweep 1: of the lane's two queries, reference (log2 domain) and sum
        float acc[COLS ? NS : 1][8];                       // sweep 2: per key, the sum over the lane's queries of the last tiles,
        double whole[COLS ? NS : 1];                       //   and of the lane's key over all lanes and tiles
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int g = 0; g < 2; ++g) { ref[s][g] = NEG_BIG; sum[s][g] = 0.f; }
#pragma unroll
        for (int s = 0; s < (COLS ? NS : 1); ++s) {
            whole[s] = 0.;
#pragma unroll
            for (int v = 0; v < 8; ++v) acc[s][v] = 0.f;
        }

        const int from = COLS ? first & ~(ST - 1) : 0;                                // streamed tiles [from, to)
        const int to = COLS ? n_tiles : first + HELD < end ? first + HELD : end;
        // One streamed tile against one held tile.  Value 8 g + 4 k + v of a lane: query 16 g + l mod 16, key 16 k + 4 (l / 16) + v.
        auto product = [&](const uint4 (&fr)[2][NK], int s, float (&c)[16]) {
            f32x4_t x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < NK; ++ks)
#pragma unroll
                for (int i = 0; i < 4; ++i) x[i] = COLS ? mma_fragment<T>(keep[s][i & 1][ks], fr[i >> 1][ks], x[i]) : mma_fragment<T>(fr[i & 1][ks], keep[s][i >> 1][ks], x[i]);
#pragma unroll
            for (int i = 0; i < 16; ++i) c[i] = x[i >> 2][i & 3];
        };
        auto mask = [&](float (&c)[16], int t, int s) {     // the diagonal tile: masked where key > query
            if (t == tile[s]) {
#pragma unroll
                for (int i = 0; i < 16; ++i) c[i] = ((i >> 2) & 1) * 16 + quarter * 4 + (i & 3) <= (i >> 3) * 16 + l16 ? c[i] : -INFINITY;
            }
        };
        auto drop_nan = [&](float (&c)[16]) {               // a logit that is not a number counts as masked
#pragma unroll
            for (int i = 0; i < 16; ++i) c[i] = c[i] == c[i] ? c[i] : -INFINITY;
        };
        // all of one kind before any of the next: an exponential's result is not there for the next instruction
        auto exponentials = [&](float (&c)[16], float m0, float m1) {
#pragma unroll
            for (int i = 0; i < 16; ++i) c[i] = fmaf(c[i], a.qscale, i < 8 ? -m0 : -m1);
#pragma unroll
            for (int i = 0; i < 16; ++i) c[i] = fast_exp2(c[i]);
        };
        auto row_sums = [&](float (&c)[16]) {               // into c[0] and c[8]
#pragma unroll
            for (int h = 4; h >= 1; h >>= 1)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if ((i & 7) < h) c[i] += c[i + h];
        };
        auto renew = [&](float (&c)[16], int s) {           // the references of a tile's queries, as far as its logits lie above them
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                float mx = c[8 * g];
#pragma unroll
                for (int i = 1; i < 8; ++i) mx = fmaxf(mx, c[8 * g + i]);
                const float m_new = fmaxf(ref[s][g], across_groups_max<16>(mx) * a.qscale);      // qscale > 0; finite also where all keys are masked
                sum[s][g] *= fast_exp2(ref[s][g] - m_new);
                ref[s][g] = m_new;
            }
        };
        // One streamed tile against one held tile.
        auto absorb = [&](auto renewed, const uint4 (&fr)[2][NK], int t, int s, const float2 (&qs)[2]) {
            if (!(t < to && tile[s] < n_tiles && (COLS ? t >= tile[s] : t <= tile[s]))) return;         // above the diagonal (wave-uniform)
            float c[16];
            product(fr, s, c);
            mask(c, t, s);
            if constexpr (CAREFUL || decltype(renewed)::value) drop_nan(c);
            if constexpr (COLS) {
                exponentials(c, qs[0].x, qs[1].x);
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[s][i & 7] = fmaf(c[i], qs[i >> 3].y, acc[s][i & 7]);
            } else {
                if (decltype(renewed)::value || t == 0) renew(c, s);
                exponentials(c, ref[s][0], ref[s][1]);
                row_sums(c);
                sum[s][0] += c[0];
                sum[s][1] += c[8];
            }
        };
        auto process = [&](int t, const uint4 (&fr)[2][NK], const float2 (&qs)[2]) {     // ... against the tiles this wave holds
#pragma unroll
            for (int s = 0; s < NS; ++s) absorb(std::false_type{}, fr, t, s, qs);
        };
        auto stats = [&](int t, float2 (&qs)[2]) {
#pragma unroll
            for (int g = 0; g < 2; ++g) qs[g] = COLS ? stat[(t < n_tiles ? t : n_tiles - 1) * 32 + g * 16 + l16] : make_float2(0.f, 0.f);
        };

        uint4 fa[2][NK];
        float2 qa[2];
        for (int t0 = from; t0 < to; t0 += ST) {
            if (t0 != from) {
                landed();
                __syncthreads();                           // this stage is in LDS, the other buffer is free
            }
            if (t0 != from) request_next(cur ^ 1);
            float before[NS][2];
#pragma unroll
            for (int s = 0; s < NS; ++s) { before[s][0] = sum[s][0]; before[s][1] = sum[s][1]; }
            if constexpr (AHEAD) {
                uint4 fb[2][NK];
                float2 qb[2];
                fragments(cur, 0, fa);
                stats(t0, qa);
#pragma unroll
                for (int j = 0; j < ST; j += 2) {
                    fragments(cur, j + 1, fb);
                    stats(t0 + j + 1, qb);
                    process(t0 + j, fa, qa);
                    if (j + 2 < ST) {
                        fragments(cur, j + 2, fa);
                        stats(t0 + j + 2, qa);
                    }
                    process(t0 + j + 1, fb, qb);
                }
            } else {
#pragma unroll 1
                for (int j = 0; j < ST; ++j) {
                    fragments(cur, j, fa);
                    stats(t0 + j, qa);
                    process(t0 + j, fa, qa);
                }
            }
            if constexpr (!COLS) {                         // a sum that the references cannot stand for: the stage's tiles again
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    if (!__any(!(__builtin_elementwise_maximum(sum[s][0], sum[s][1]) < LARGE))) continue;          // (NaN if one of them is)
                    sum[s][0] = before[s][0];
                    sum[s][1] = before[s][1];
#pragma unroll 1
                    for (int j = 0; j < ST; ++j) {
                        fragments(cur, j, fa);
                        absorb(std::true_type{}, fa, t0 + j, s, qa);
                    }
                }
            }
            cur ^= 1;
            // Every eight tiles the lanes meet: a sum over all of a long prompt's tiles in one register would lose a rounding per tile.
            // Counted from the prompt's beginning, so that a unit's scores do not depend on how its tiles are dealt to waves and workgroups.
            if (COLS && (((t0 + ST) & 7) == 0 || t0 + ST >= to)) {
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    if (tile[s] >= t0 + ST) continue;      // nothing added yet (wave-uniform)
                    whole[s] += sums_over_16_lanes(acc[s], lane);
#pragma unroll
                    for (int v = 0; v < 8; ++v) acc[s][v] = 0.f;
                }
            }
        }
        bool good = true;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (tile[s] >= n_tiles) continue;
            if constexpr (!COLS) {
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    const float m_row = across_groups_max<16>(ref[s][g]);
                    const float total = across_groups_sum<16>(sum[s][g] * fast_exp2(ref[s][g] - m_row));
                    const int row = tile[s] * 32 + g * 16 + l16;
                    if (quarter == 0) stat[row] = make_float2(m_row, row < n && total > 0.f ? 1.0f / total : 0.f);       // (0: every logit of the query masked)
                }
            } else {
                const int u = ((lane >> 3) & 1) * 4 + ((lane >> 2) & 1) * 2 + (lane & 1);
                const int key = tile[s] * 32 + (u >> 2) * 16 + quarter * 4 + (u & 3);
                good = good && whole[s] == whole[s];
                if ((lane & 2) == 0 && key < n) a.score_out[(size_t)blockIdx.x * (size_t)n + key] = (float)whole[s];
            }
        }
        return good;
    };
    request_next(cur);
    auto sweep = [&](auto cols, int end) {
        constexpr bool COLS = decltype(cols)::value;
        for (int first = begin; first < end; first += HELD) {
            const bool good = group(cols, std::false_type{}, first, end);
            if constexpr (COLS) {
                if (__syncthreads_or(!good)) {             // again, with a test per logit
                    landed();                              // what the next group's first stage has brought makes way
                    __syncthreads();
                    ahead_sweep = 1;
                    ahead_first = first;
                    ahead_tile = first & ~(ST - 1);
                    request_next(cur);
                    group(cols, std::true_type{}, first, end);
                }
            }
        }
    };
    sweep(std::false_type{}, n_tiles);
    sweep(std::true_type{}, stop);
}

// Where the keys' tiles [0, n_tiles) are cut so that `parts` workgroups of one unit take about equally long: part p does sweep 1
// over the queries from cut[p] on and sweep 2 over its own keys, in tiles n^2 / 2 - cut[p]^2 / 2 and as many as lie below them.
static void cut_long(int n_tiles, int parts, int (&cut)[5]) {
    auto cost = [&](int from, int to) { return (long long)n_tiles * n_tiles - (long long)from * from + (long long)(n_tiles - from) * (n_tiles - from) - (long long)(n_tiles - to) * (n_tiles - to); };
    for (long long limit = (long long)n_tiles * n_tiles;; limit += (limit >> 6) + 1) {       // the smallest limit that all parts keep, within 2 %
        int at = 0;
        for (int p = 0; p < parts; ++p) {
            cut[p] = at;
            while (at < n_tiles && cost(cut[p], at + 1) <= limit) ++at;
        }
        cut[parts] = n_tiles;
        if (at >= n_tiles) return;
    }
}

// LDS of the long kernel: two stages of the streamed operand and the queries' statistics.
template <int ROW> static size_t long_lds_bytes(int n) {
    return 2 * (size_t)long_stage_tiles<ROW>() * 32 * ROW + (size_t)((n + 31) / 32 * 32) * 2 * sizeof(float);
}

// Whether a compute unit's 160 KB of LDS have no room for a second workgroup (256 bytes more each: the vote of a workgroup).
static bool long_alone(size_t lds) { return 2 * (lds + 256) > 163840; }

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
    // Short prompts: a prompt's compression follows and reads K again.  Without the non-temporal hint K stays in the memory-side cache for
    // it, but first has to be let in: where the cache is full of what others wrote, that writes as much back as K has bytes.  A
    // kernel that waits for memory anyway is slower by that and the compression gains less than it loses, so K keeps the hint where
    // rows of 256 bytes or less fill seven eighths of their tiles.  Scores and compression of new, just written and repeated prompts, us
    // per layer with and without the hint (4096 units, bf16, d = 128; "just written" with the writing): 64 tokens 68, 143, 66 and 72, 137,
    // 63; of 48 61, 118, 61 and 61, 112, 56; of 100 98, 211, 94 and 97, 206, 91; fp32 of 64 160, 307, 157 and 150, 291, 143.  Up to 512 MB
    // it gains, or loses nothing (fp32, 16384 units of 64 tokens 583, 1192, 579 and 555, 1170, 547; bf16 of 100 647, 1582, 640 and 643,
    // 1552, 631 for two layers); beyond, where little of K can stay, it gains nothing (fp32, 32768 of 64 1133, 2407, 1120 and 1098, 2386,
    // 1091; 65536 of 64 2197, 4927, 2189 and 2188, 4922, 2185; bf16, 65536 of 40 700, 1466, 685 and 707, 1477, 675, the scores alone 250 and 285).
    // With less than 40 MB, which about fits the L2s, the hint is better (512 units of 64 tokens 13.95 and 14.33).
    const bool full_tiles = n_src * 8 > (n_src + 31) / 32 * 32 * 7;
    const size_t k_bytes = (size_t)n_units * (size_t)n_src * (size_t)a.row_bytes;
    const bool keep_k = k_bytes >= ((size_t)40 << 20) && k_bytes <= ((size_t)512 << 20) && !(full_tiles && a.row_bytes <= 256);
    const int n_blocks = (n_src + 31) / 32;
    const int waves = n_blocks < 4 ? n_blocks : 4;
    const size_t lds_short = short_lds_bytes(waves, n_src, a.row_bytes);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const dim3 block(64u * waves);
    // long prompts (the reasons stand at the kernel): workgroups per unit, and whether a wave holds three tiles rather than two
    const int parts = n_units <= 85 ? 3 : n_units <= 128 ? 2 : 1;
    auto three = [&](int w) { return (n_blocks + 3 * w - 1) / (3 * w) < (n_blocks + 2 * w - 1) / (2 * w); };
    a.cut[0] = 0;
    a.cut[1] = n_blocks;
    if (parts > 1 && n_blocks > 4) cut_long(n_blocks, parts, a.cut);       // (the search takes the host up to 1.6 us)
    hipError_t attr = hipSuccess;
    // more than 64 KB of dynamic LDS has to be asked for (the longest short prompts in fp32: 70 KB of the CU's 160 KB)
#define SSD_PREFILL_SHORT_AS(T_, D_, KT_, KEEP_)                                                                                \
    do {                                                                                                                        \
        const void *fn = reinterpret_cast<const void *>(&prefill_scores_short_kernel<T_, D_, KT_, KEEP_>);                      \
        if (lds_short > 65536) attr = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_short);      \
        int per_cu = 0;                                                                                                         \
        if (attr == hipSuccess) attr = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, (int)block.x, lds_short);      \
        if (attr == hipSuccess) {                                                                                               \
            const dim3 g = resident_grid(n_units, per_cu);                                                                      \
            if (g.x == 0) attr = hipErrorInvalidValue;                                                                          \
            else hipLaunchKernelGGL((prefill_scores_short_kernel<T_, D_, KT_, KEEP_>), g, block, lds_short, s, a);              \
        }                                                                                                                       \
    } while (0)
#define SSD_PREFILL_SHORT(T_, D_, KT_)                                                                                          \
    do {                                                                                                                        \
        if (keep_k) SSD_PREFILL_SHORT_AS(T_, D_, KT_, true); else SSD_PREFILL_SHORT_AS(T_, D_, KT_, false);                     \
    } while (0)
#define SSD_PREFILL_LONG(T_, D_, WAVES_, NS_, PER_SIMD_)                                                                         \
    do {                                                                                                                        \
        const void *fn = reinterpret_cast<const void *>(&prefill_scores_long_kernel<T_, D_, WAVES_, NS_, PER_SIMD_>);           \
        const size_t lds = long_lds_bytes<D_ * (int)sizeof(T_)>(n_src);                                                         \
        if (lds > 65536) attr = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);                  \
        if (attr == hipSuccess)                                                                                                 \
            hipLaunchKernelGGL((prefill_scores_long_kernel<T_, D_, WAVES_, NS_, PER_SIMD_>), dim3((unsigned)n_units, (unsigned)parts), dim3(64 * WAVES_), lds, s, a); \
    } while (0)
#define SSD_PREFILL(T_, D_)                                                                                          \
    do {                                                                                                             \
        constexpr bool wide = sizeof(T_) == 4;             /* fp32 fragments: one tile per wave */                   \
        constexpr bool narrow = !wide && D_ == 64;                                                                   \
        const bool eight = n_units <= 256 || (wide && D_ == 64) || long_alone(long_lds_bytes<D_ * (int)sizeof(T_)>(n_src)); \
        if (n_blocks <= 2) SSD_PREFILL_SHORT(T_, D_, 2);                                                             \
        else if (n_blocks <= 4) SSD_PREFILL_SHORT(T_, D_, 4);                                                        \
        else if (eight && three(8)) SSD_PREFILL_LONG(T_, D_, 8, (wide ? 1 : 3), 2);                                  \
        else if (eight) SSD_PREFILL_LONG(T_, D_, 8, (wide ? 1 : 2), 2);                                              \
        else if (narrow && n_blocks > 8 && (n_units + 511) / 512 <= (n_units + 767) / 768) SSD_PREFILL_LONG(T_, D_, 8, (wide ? 1 : 2), (narrow ? 4 : 2)); \
        else if (three(4)) SSD_PREFILL_LONG(T_, D_, 4, (wide ? 1 : 3), 2);                                           \
        else SSD_PREFILL_LONG(T_, D_, 4, (wide ? 1 : 2), 2);                                                         \
    } while (0)
    if (dtype == SSD_BF16) {
        if (d == 128) SSD_PREFILL(bf16_t, 128); else SSD_PREFILL(bf16_t, 64);
    } else {
        if (d == 128) SSD_PREFILL(float, 128); else SSD_PREFILL(float, 64);
    }
#undef SSD_PREFILL
#undef SSD_PREFILL_LONG
#undef SSD_PREFILL_SHORT
#undef SSD_PREFILL_SHORT_AS
    if (attr != hipSuccess) return hip_fail(attr, "prefill score kernel attribute");
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "prefill score launch");
    return SSD_OK;
}
