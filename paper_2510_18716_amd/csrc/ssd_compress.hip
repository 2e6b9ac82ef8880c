// ssd_compress_kv: top-M selection by accumulated score and the gather into the compact cache
// (Algorithm 1 "IndicesOfTopM" / "SelectAndAppend"; Algorithm 2 "Compress semantic cache
// (heavy-hitter) ... Reset row buffer" and its prefill branch).  The selection itself is in
// ssd_select.h; this file holds the stand-alone in-place kernel and the dense-source kernel.
#include "ssd_select.h"

namespace ssd {

template <int LAYERS, bool HEADS> struct CompressArgs {
    Geom g;
    LayersOf<LAYERS> lm;
    int m;             // heavy slots in use
    int c;             // buffered tokens
    int base;          // ring index of the oldest buffered token
    int R;
    int lpr;           // 16-byte fragments per row
    int seq_off;       // the launch covers sequences [seq_off, seq_off + n_seq)
    int n_seq;
    HeadsOf<HEADS> ht;
};

// One workgroup per (layer, sequence, head); spatial heads return at once.
template <int THREADS, int LAYERS, bool HEADS>
__global__ __launch_bounds__(THREADS) void compress_inplace_kernel(CompressArgs<LAYERS, HEADS> a) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int BH = a.n_seq * a.g.H;
    const int unit = blockIdx.x;
    const int lrel = LAYERS == 1 ? 0 : unit / BH;
    const int rem = LAYERS == 1 ? unit : unit % BH;
    const UnitRef u = unit_ref(a.g, a.lm.layer[lrel], a.seq_off + rem / a.g.H, rem % a.g.H);
    if (!u.sem) return;                       // uniform for the whole workgroup
    int Mh = a.g.M;                           // this head's budget
    if constexpr (HEADS) Mh = a.ht.v[rem % a.g.H];
    const int m = a.m < Mh ? a.m : Mh;        // heavy slots this head has in use
    const int n_old = a.c - a.R;              // buffered tokens that become candidates (> 0, checked on the host)
    const int n_cand = m + n_old;
    unsigned long long *keys = reinterpret_cast<unsigned long long *>(lds);
    for (int i = threadIdx.x; i < n_cand; i += THREADS) {
        const int slot = i < m ? i : a.g.M + (a.base + (i - m)) % a.g.C;
        keys[i] = make_key(u.score[slot], u.pos[slot]);
    }
    __syncthreads();
    select_and_move<THREADS, false>(a.g, u, lds, n_cand, m, n_old, a.base, a.lpr, threadIdx.x, Mh);
}

// ---- dense-source mode -------------------------------------------------------

template <int LAYERS, bool HEADS> struct DenseSrcArgs {
    Geom g;
    LayersOf<LAYERS> lm;
    const char *K_src;      // [L', B, H, n_src, d]
    const char *V_src;
    const float *score_src; // [L', B, H, n_src] or NULL
    int layer_off;
    int n_src;
    int R;
    int lpr;
    int dealt;              // units (a multiple of 512, or none) that go to the XCDs 64 neighbours at a time
    HeadsOf<HEADS> ht;      // budgets per head
};

// The smallest key of the M largest of n distinct keys (n > M >= 1), for a whole workgroup; keys[k] is candidate
// k * THREADS + tid.  Radix descent from the highest bit in which the keys differ, eight bits at a time: a histogram
// of the digit among the keys still in question, the digit at which the count from above reaches what is wanted,
// and on with that digit's keys -- until the wanted ones are all of them, which for scores of any spread is after
// two or three digits.  (Counting every key's rank against all others is n^2 / THREADS LDS reads per thread: at 1500
// candidates 9000, most of a kernel that otherwise moves rows.)
//   hist : LDS [256 + 4], and share : LDS [2 * THREADS / 64] 64-bit
template <int THREADS, int KPT>
static __device__ unsigned long long nth_largest(const unsigned long long (&keys)[KPT], int n, int M, int *hist, unsigned long long *share, int tid) {
    unsigned long long all_or = 0ull, all_and = ~0ull;
#pragma unroll
    for (int k = 0; k < KPT; ++k)
        if (k * THREADS + tid < n) { all_or |= keys[k]; all_and &= keys[k]; }
#pragma unroll
    for (int x = 1; x < 64; x <<= 1) { all_or |= __shfl_xor(all_or, x); all_and &= __shfl_xor(all_and, x); }
    if ((tid & 63) == 0) { share[2 * (tid >> 6)] = all_or; share[2 * (tid >> 6) + 1] = all_and; }
    __syncthreads();
#pragma unroll
    for (int wv = 0; wv < THREADS / 64; ++wv) { all_or |= share[2 * wv]; all_and &= share[2 * wv + 1]; }
    const unsigned long long differ = all_or ^ all_and;       // not 0: the keys are distinct and n > M >= 1
    int top = 64 - __builtin_clzll(differ);                   // the keys agree in bits [top, 64)
    unsigned long long prefix = top < 64 ? all_or >> top << top : 0ull;
    int want = M;                                             // how many of the keys that start with `prefix` are kept
    for (;;) {
        const int low = top > 8 ? top - 8 : 0;
        const int mask = (1 << (top - low)) - 1;
        for (int i = tid; i < 256; i += THREADS) hist[i] = 0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < KPT; ++k)
            if (k * THREADS + tid < n && (top == 64 || keys[k] >> top == prefix >> top)) atomicAdd(&hist[(int)(keys[k] >> low) & mask], 1);
        __syncthreads();
        if (tid < 64) {                                       // lane l: digits 255 - 4l .. 252 - 4l, from the highest down
            int c[4], sum = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) { c[j] = hist[255 - 4 * tid - j]; sum += c[j]; }
            int above = sum;                                  // inclusive prefix over the lanes
#pragma unroll
            for (int x = 1; x < 64; x <<= 1) { const int o = __shfl_up(above, x); if (tid >= x) above += o; }
            above -= sum;
            if (above < want && above + sum >= want) {        // exactly one lane
                int j = 0;
                while (above + c[j] < want) above += c[j++];
                hist[256] = 255 - 4 * tid - j;
                hist[257] = want - above;
                hist[258] = c[j];
            }
        }
        __syncthreads();
        prefix |= (unsigned long long)hist[256] << low;
        want = hist[257];
        const int left = hist[258];
        if (left == want || low == 0) return prefix;          // every key that starts with `prefix` is kept (low == 0: it is the one)
        top = low;
        __syncthreads();                                      // before the histogram is cleared
    }
}

static __device__ __forceinline__ void store_once(char *p, const uint4 &v) {
    const u32x4_nt_t x = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(x, reinterpret_cast<u32x4_nt_t *>(p));
}

// Copy n_frag 16-byte fragments: map(t, src, dst) gives fragment t's addresses.  BATCH loads of a thread are in flight
// together: a fragment at a time, every store waits for its load and the next load for the store, a memory round
// trip per fragment.  Neither side is touched again by this launch, so both carry the non-temporal hint.
// Bound: HBM, rows read and written once.  7B shape, 4096 units, 64 source tokens, 41 kept on average (172 MB): 42.8 us
// with single fragments, 38 with batches of four (two: 42), 35 with the stores non-temporal as well (4.9 TB/s, what a plain copy
// reaches; loads without the hint: 75).  256 units of 1500 tokens, 320 kept by the semantic half: 154 us with
// single fragments and ranks by counting, 19.8 now.
template <int THREADS, int BATCH, typename Map>
static __device__ __forceinline__ void copy_fragments(int n_frag, int tid, Map map) {
    for (int t0 = tid; t0 - tid < n_frag; t0 += THREADS * BATCH) {
        uint4 v[BATCH];
        char *dst[BATCH];
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
            const int t = t0 + j * THREADS;
            const char *src;
            map(t < n_frag ? t : n_frag - 1, src, dst[j]);    // unconditional loads: past the end the last fragment again
            v[j] = load_once(src);
        }
#pragma unroll
        for (int j = 0; j < BATCH; ++j)
            if (t0 + j * THREADS < n_frag) store_once(dst[j], v[j]);
    }
}

// One workgroup per (layer, sequence, head), KPT candidates per thread at most.  With one candidate per thread they are ranked
// by counting (LDS broadcasts: cheaper than the barriers of a radix descent); more go through nth_largest.
template <int THREADS, int KPT, int LAYERS, bool HEADS>
__global__ __launch_bounds__(THREADS, THREADS == 1024 ? 8 : 1) void compress_dense_kernel(DenseSrcArgs<LAYERS, HEADS> a) {
    constexpr int WAVES = THREADS / 64;
    constexpr bool RANK = KPT == 1;
    extern __shared__ int kept[];                             // [M] kept positions, ascending
    __shared__ unsigned long long keys[RANK ? THREADS : 1], share[RANK ? 1 : 2 * WAVES];
    __shared__ int hist[RANK ? 1 : 260], count[KPT * WAVES];
    const int BH = a.g.B * a.g.H;
    int unit = blockIdx.x;                                    // workgroups go round the eight XCDs: dealt, an XCD has 1 MB of neighbouring units
    if (unit < a.dealt) unit = (unit & ~511) + ((unit & 7) << 6) + ((unit >> 3) & 63);
    const int lrel = LAYERS == 1 ? 0 : unit / BH;
    const int rem = LAYERS == 1 ? unit : unit % BH;
    const UnitRef u = unit_ref(a.g, a.lm.layer[lrel], rem / a.g.H, rem % a.g.H);
    int budget = u.sem ? a.g.M : a.g.W;                       // this head's M or W
    if constexpr (HEADS) budget = a.ht.v[rem % a.g.H];
    const size_t src_unit = (size_t)(a.layer_off + lrel) * BH + rem;
    const char *Ks = a.K_src + src_unit * (size_t)a.n_src * a.g.row_bytes;
    const char *Vs = a.V_src + src_unit * (size_t)a.n_src * a.g.row_bytes;
    const int tid = threadIdx.x;
    const int lpr_log2 = __builtin_ctz(a.lpr);                // 8, 16 or 32 fragments per row
    // fragment t of the rows to copy: row t / (2 * lpr), K fragments first, then V's
    auto plane = [&](int t, int p, int slot, const char *&src, char *&dst) {
        const bool v = (t >> lpr_log2) & 1;
        const size_t sub = (size_t)(t & (a.lpr - 1)) * 16u;
        src = (v ? Vs : Ks) + (size_t)p * a.g.row_bytes + sub;
        dst = (v ? u.V : u.K) + (size_t)slot * a.g.row_bytes + sub;
    };

    if (!u.sem) {
        // positions {0..S-1} and the last W: destination slot as in ssd_append_token
        const int S = a.g.S, W = budget, RW = W + (a.g.RW - a.g.W);
        const int n_sink = a.n_src < S ? a.n_src : S;
        const int w_begin = a.n_src - W > S ? a.n_src - W : S;
        const int n_win = a.n_src > w_begin ? a.n_src - w_begin : 0;
        const int n_rows = n_sink + n_win;
        const int ring0 = (w_begin - S) % RW;                 // ring index of the window's first position (w_begin >= S)
        copy_fragments<THREADS, 4>(n_rows << (lpr_log2 + 1), tid, [&](int t, const char *&src, char *&dst) {
            const int k = t >> (lpr_log2 + 1);
            const int r = ring0 + (k - n_sink);               // window rows: at most RW of them, so one wrap at most
            plane(t, k < n_sink ? k : w_begin + (k - n_sink), k < n_sink ? k : S + (r < RW ? r : r - RW), src, dst);
        });
        return;
    }

    const int M = budget;                                 // the row buffer starts at slot g.M
    const int n_rec = a.n_src < a.R ? a.n_src : a.R;      // newest tokens that go to the row buffer
    const int n_cand = a.n_src - n_rec;
    const float *sc = a.score_src ? a.score_src + src_unit * (size_t)a.n_src : nullptr;
    unsigned long long key[KPT];
#pragma unroll
    for (int k = 0; k < KPT; ++k) {
        const int i = k * THREADS + tid;
        key[k] = i < n_cand ? make_key(sc ? sc[i] : 0.f, i) : 0ull;
    }
    unsigned keepbits = ~0u;                              // bit k: candidate k * THREADS + tid stays
    if (n_cand > M) {
        if constexpr (RANK) {
            keys[tid] = key[0];                           // (0 beyond the last candidate: never counted)
            __syncthreads();
            int rank = 0;
            for (int j = 0; j < n_cand; ++j) rank += keys[j] > key[0] ? 1 : 0;
            if (rank >= M) keepbits = 0u;
        } else {
            const unsigned long long least = nth_largest<THREADS, KPT>(key, n_cand, M, hist, share, tid);
#pragma unroll
            for (int k = 0; k < KPT; ++k)
                if (key[k] < least) keepbits &= ~(1u << k);
        }
    }
    // kept positions in ascending order: a count per 64 consecutive candidates, then every kept one finds its place
    const int groups = (n_cand + 63) / 64;                // group g = candidates 64g .. 64g + 63 = (k, wave) with k * WAVES + wave = g
    const int wv = tid >> 6;
    unsigned long long in_group[KPT];
#pragma unroll
    for (int k = 0; k < KPT; ++k) {
        const bool f = k * THREADS + tid < n_cand && ((keepbits >> k) & 1u);
        in_group[k] = __ballot(f);
        if ((tid & 63) == 0 && k * WAVES + wv < groups) count[k * WAVES + wv] = __popcll(in_group[k]);
    }
    __syncthreads();
    if (tid < 64) {                                       // exclusive prefix over the groups (at most 64)
        const int c = tid < groups ? count[tid] : 0;
        int pre = c;
#pragma unroll
        for (int x = 1; x < 64; x <<= 1) { const int o = __shfl_up(pre, x); if (tid >= x) pre += o; }
        if (tid < groups) count[tid] = pre - c;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < KPT; ++k) {
        const unsigned long long below = (1ull << (tid & 63)) - 1ull;
        if (k * THREADS + tid < n_cand && ((keepbits >> k) & 1u))
            kept[count[k * WAVES + wv] + __popcll(in_group[k] & below)] = k * THREADS + tid;
    }
    __syncthreads();
    const int nkeep = n_cand < M ? n_cand : M;
    // heavy slots 0..nkeep-1 in ascending position; row buffer (ring index 0..) gets the newest n_rec
    const int n_rows = nkeep + n_rec;
    copy_fragments<THREADS, 4>(n_rows << (lpr_log2 + 1), tid, [&](int t, const char *&src, char *&dst) {
        const int k = t >> (lpr_log2 + 1);
        plane(t, k < nkeep ? kept[k] : n_cand + (k - nkeep), k < nkeep ? k : a.g.M + (k - nkeep), src, dst);
    });
    for (int k = tid; k < n_rows; k += THREADS) {
        const int p = k < nkeep ? kept[k] : n_cand + (k - nkeep);
        const int slot = k < nkeep ? k : a.g.M + (k - nkeep);
        u.pos[slot] = p;
        u.score[slot] = sc ? sc[p] : 0.f;
    }
}

template <int LAYERS, bool HEADS>
static hipError_t launch_inplace(const ssd_cache *cache, int lb, int le, const LayerState &st, int seq_off, int n_seq, hipStream_t s) {
    const ssd_config &cf = cache->cfg;
    const int n_old = st.c - cf.recent;
    CompressArgs<LAYERS, HEADS> a;
    a.g = make_geom(cache, lb);
    fill_layers(cache, lb, le, &a.lm);
    a.m = st.m;
    a.c = st.c;
    a.base = st.base;
    a.R = cf.recent;
    a.lpr = cf.head_dim * cache->esize / 16;
    a.seq_off = seq_off;
    a.n_seq = n_seq;
    fill_head_table(cache, lb, &a.ht);
    const int n_cand = st.m + n_old;
    const unsigned units = (unsigned)((le - lb) * n_seq * cf.n_heads);
    const size_t lds = select_lds_bytes(cache->Ml[lb], n_cand, n_old);
    if (n_cand <= 192) hipLaunchKernelGGL((compress_inplace_kernel<64, LAYERS, HEADS>), dim3(units), dim3(64), lds, s, a);
    else hipLaunchKernelGGL((compress_inplace_kernel<256, LAYERS, HEADS>), dim3(units), dim3(256), lds, s, a);
    return hipGetLastError();
}

// In-place compression of sequences [seq_off, seq_off + n_seq) of layers [lb, le), which all hold the state `st`
// (st.c - R > 0).
int launch_compress_inplace(const ssd_cache *cache, int lb, int le, const LayerState &st, int seq_off, int n_seq, hipStream_t s) {
    const hipError_t e = heads_differ(cache, lb) ? launch_inplace<1, true>(cache, lb, le, st, seq_off, n_seq, s)
                         : le - lb == 1 ? launch_inplace<1, false>(cache, lb, le, st, seq_off, n_seq, s)
                                        : launch_inplace<LMAX, false>(cache, lb, le, st, seq_off, n_seq, s);
    if (e != hipSuccess) return hip_fail(e, "compression launch");
    return SSD_OK;
}

template <int LAYERS, bool HEADS>
static hipError_t launch_dense_source(const ssd_cache *cache, int lb, int le, int layer_off, const void *K_src, const void *V_src,
                                      const float *score_src, int n_src, hipStream_t s) {
    const ssd_config &cf = cache->cfg;
    DenseSrcArgs<LAYERS, HEADS> a;
    a.g = make_geom(cache, lb);
    fill_layers(cache, lb, le, &a.lm);
    a.K_src = static_cast<const char *>(K_src);
    a.V_src = static_cast<const char *>(V_src);
    a.score_src = score_src;
    a.layer_off = layer_off;
    a.n_src = n_src;
    a.R = cf.recent;
    a.lpr = cf.head_dim * cache->esize / 16;
    fill_head_table(cache, lb, &a.ht);
    const size_t lds = sizeof(int) * (size_t)cache->Ml[lb];
    const int n_cand = n_src - (n_src < cf.recent ? n_src : cf.recent);
    const unsigned units = (unsigned)((le - lb) * cf.n_seqs * cf.n_heads);
    // One candidate per thread as far as it goes (8 units of 64 tokens 5.9 us, with room for 16 per thread 7.4; 4096 units 46.0 and 47.6), but
    // a prompt that just exceeds 256 and is kept whole is a copy, for which few units want sixteen waves (8 units of 257: 7.2 us, 10.4
    // with four).  Few units of many tokens: sixteen waves each, so that the chip has rows enough in flight (256 units of 1500 tokens: 2 % of
    // prompt scoring and compression together), all of them on a compute unit twice (64 registers; 512 units of 600 12.7 us, 16.9
    // with 73 registers).  More units: room for no more candidates than there may be (2048 units of 1024 tokens 51.8 us with 8 per
    // thread, 58.3 with 16).
    const dim3 grid(units);
    // Many units of few rows: with neighbours on one XCD each XCD meets an eighth of the source's pages (us per launch, new prompts and ones
    // just written: 4096 units of 64 tokens 37.4 -> 36.7 and 40.1 -> 37.3, 2560 of 64 26.8 -> 24.8 and 28.3 -> 26.1, 4096 of 120 40.2 -> 39.1
    // and 42.7 -> 40.1).  Longer units have pages to themselves (scores and compression of 2048 of 1024 tokens 742 and 759), and
    // fewer gain nothing (2048 of 96 49.3 both, 768 of 200 47.3 and 48.0).
    a.dealt = units >= 2560 && (size_t)n_src * a.g.row_bytes <= 32768 ? (int)(units & ~511u) : 0;
    if (n_cand <= 256 && (n_src <= 256 || n_cand > cache->Ml[lb])) hipLaunchKernelGGL((compress_dense_kernel<256, 1, LAYERS, HEADS>), grid, dim3(256), lds, s, a);
    else if (units <= 512) hipLaunchKernelGGL((compress_dense_kernel<1024, 4, LAYERS, HEADS>), grid, dim3(1024), lds, s, a);
    else if (n_cand <= 2048) hipLaunchKernelGGL((compress_dense_kernel<256, 8, LAYERS, HEADS>), grid, dim3(256), lds, s, a);
    else hipLaunchKernelGGL((compress_dense_kernel<256, 16, LAYERS, HEADS>), grid, dim3(256), lds, s, a);
    return hipGetLastError();
}

}  // namespace ssd

using namespace ssd;

extern "C" int ssd_compress_kv(ssd_cache *cache, int layer_begin, int layer_end, const void *K_src,
                               const void *V_src, const float *score_src, int n_src, void *stream) {
    clear_error();
    int rc = check_layers(cache, layer_begin, layer_end);
    if (rc != SSD_OK) return rc;
    const ssd_config &cf = cache->cfg;
    hipStream_t s = static_cast<hipStream_t>(stream);

    if (K_src || V_src) {
        if (!K_src || !V_src) return fail(SSD_ERR_INVALID_ARG, "K_src and V_src must both be given");
        if (n_src < 1 || n_src > 4096) return fail(SSD_ERR_INVALID_ARG, "n_src=%d outside 1..4096", n_src);
        if (!aligned(K_src, 16) || !aligned(V_src, 16) || !aligned(score_src, 4))
            return fail(SSD_ERR_INVALID_ARG, "K_src / V_src must be 16-byte aligned, score_src 4-byte aligned");
        const int n_rec = n_src < cf.recent ? n_src : cf.recent;
        const int n_cand = n_src - n_rec;
        if (cache->launch_enabled) {
            for (int lb = layer_begin, le; lb < layer_end; lb = le) {
                le = same_geom_run(cache, lb, layer_end);
                const int off = lb - layer_begin;
                const hipError_t e = heads_differ(cache, lb) ? launch_dense_source<1, true>(cache, lb, le, off, K_src, V_src, score_src, n_src, s)
                                     : le - lb == 1 ? launch_dense_source<1, false>(cache, lb, le, off, K_src, V_src, score_src, n_src, s)
                                                    : launch_dense_source<LMAX, false>(cache, lb, le, off, K_src, V_src, score_src, n_src, s);
                if (e != hipSuccess) return hip_fail(e, "dense-source compression launch");
            }
        }
        for (int l = layer_begin; l < layer_end; ++l) {
            LayerState &st = cache->st[l];
            st.n = n_src;
            st.m = cache->ldesc[l].n_se > 0 ? (n_cand < cache->Ml[l] ? n_cand : cache->Ml[l]) : 0;
            st.c = has_buffer(cache, l) ? n_rec : 0;
            st.base = 0;
            st.nc = n_src;
        }
        return SSD_OK;
    }

    if (score_src) return fail(SSD_ERR_INVALID_ARG, "score_src without K_src / V_src");
    for (int lb = layer_begin; lb < layer_end;) {
        const int le = same_state_run(cache, lb, layer_end);
        const LayerState st = cache->st[lb];
        const int n_old = st.c - cf.recent;
        // kernels run only where semantic heads have candidates; the counters (and the spatial window of
        // Algorithm 2) move in every layer of the range
        if (n_old > 0 && cache->ldesc[lb].n_se > 0 && cache->launch_enabled) {
            rc = launch_compress_inplace(cache, lb, le, st, 0, cf.n_seqs, s);
            if (rc != SSD_OK) return rc;
        }
        for (int l = lb; l < le; ++l) apply_compress_counters(cache, l);
        lb = le;
    }
    return SSD_OK;
}
