// ssd_append_token: write the new token's K and V rows into every head's cache
// (Algorithm 1 "Append"; Algorithm 2 "Append k_t, v_t to row buffer").
//
// Pure data movement: one lane moves one 16-byte fragment, so a row is a run of adjacent lanes
// on both the read side (k_new/v_new, [L',B,H,d]) and the write side (the unit's slot).
#include "ssd_device.h"

namespace ssd {

template <int LAYERS, bool HEADS> struct AppendArgs {
    Geom g;
    const char *k_new;
    const char *v_new;
    int layer_off;       // index of the launch's first layer inside k_new / v_new
    int lpr_log2;        // 16-byte fragments per row: 8, 16 or 32
    int slot_sp;         // destination slot of spatial heads
    int slot_se;         // destination slot of semantic heads
    int pos;             // absolute position of the token
    LayersOf<LAYERS> lm;
    HeadsOf<HEADS> ht;   // budgets per head: a spatial head's slot follows from its own window
};

// grid = (blocks over a sequence's heads and fragments, B, layers): nothing has to be divided.  A launch this small is
// bound by its fixed cost; 512 units of 512 bytes.
template <int LAYERS, bool HEADS>
__global__ __launch_bounds__(256) void append_kernel(AppendArgs<LAYERS, HEADS> a) {
    const int t = (int)(blockIdx.x * 256 + threadIdx.x);
    const int h = t >> (a.lpr_log2 + 1);
    if (h >= a.g.H) return;
    const int b = blockIdx.y, lrel = LAYERS == 1 ? 0 : blockIdx.z;
    const bool v = (t >> a.lpr_log2) & 1;
    const size_t sub = (size_t)(t & ((1 << a.lpr_log2) - 1)) * 16u;
    const size_t src_row = ((size_t)(a.layer_off + lrel) * a.g.B + b) * a.g.H + h;
    const uint4 frag = *reinterpret_cast<const uint4 *>((v ? a.v_new : a.k_new) + src_row * (size_t)a.g.row_bytes + sub);
    const UnitRef u = unit_ref(a.g, a.lm.layer[lrel], b, h);
    int slot = u.sem ? a.slot_se : a.slot_sp;
    if constexpr (HEADS) {
        if (!u.sem) slot = ring_slot(a.g.S, a.ht.v[h] + (a.g.RW - a.g.W), a.pos);
    }
    *reinterpret_cast<uint4 *>((v ? u.V : u.K) + (size_t)slot * (size_t)a.g.row_bytes + sub) = frag;
    if (u.sem && sub == 0 && !v) {
        u.pos[slot] = a.pos;
        u.score[slot] = 0.f;
    }
}

template <int LAYERS, bool HEADS>
static hipError_t launch_append(const ssd_cache *cache, int lb, int le, int layer_off, const void *k_new, const void *v_new, hipStream_t s) {
    const ssd_config &cf = cache->cfg;
    const LayerState &st = cache->st[lb];
    AppendArgs<LAYERS, HEADS> a;
    a.g = make_geom(cache, lb);
    a.k_new = static_cast<const char *>(k_new);
    a.v_new = static_cast<const char *>(v_new);
    fill_layers(cache, lb, le, &a.lm);
    a.layer_off = layer_off;
    a.lpr_log2 = __builtin_ctz((unsigned)(a.g.row_bytes / 16));
    a.pos = st.n;
    a.slot_sp = spatial_slot(cache, lb, st.n);
    a.slot_se = cache->Ml[lb] + (st.base + st.c) % cf.stage_cap;
    fill_head_table(cache, lb, &a.ht);
    const unsigned per_seq = (unsigned)cf.n_heads << (a.lpr_log2 + 1);
    hipLaunchKernelGGL((append_kernel<LAYERS, HEADS>), dim3((per_seq + 255) / 256, (unsigned)cf.n_seqs, (unsigned)(le - lb)), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace ssd

using namespace ssd;

extern "C" int ssd_append_token(ssd_cache *cache, int layer_begin, int layer_end, const void *k_new,
                                const void *v_new, void *stream) {
    clear_error();
    int rc = check_layers(cache, layer_begin, layer_end);
    if (rc != SSD_OK) return rc;
    if (!k_new || !v_new) return fail(SSD_ERR_INVALID_ARG, "k_new or v_new is NULL");
    if (!aligned(k_new, 16) || !aligned(v_new, 16)) return fail(SSD_ERR_INVALID_ARG, "k_new / v_new must be 16-byte aligned");
    const ssd_config &cf = cache->cfg;
    // a full row buffer in any layer refuses the whole call (nothing is appended anywhere)
    for (int l = layer_begin; l < layer_end; ++l)
        if (has_buffer(cache, l) && cache->st[l].c >= cf.stage_cap)
            return fail(SSD_ERR_STAGE_OVERFLOW, "row buffer overflow: layer %d already buffers %d tokens (C=%d); call ssd_compress_kv",
                        l, cache->st[l].c, cf.stage_cap);
    hipStream_t s = static_cast<hipStream_t>(stream);
    for (int lb = layer_begin; lb < layer_end;) {
        const int le = same_state_run(cache, lb, layer_end);
        if (cache->launch_enabled) {
            const hipError_t e = heads_differ(cache, lb) ? launch_append<1, true>(cache, lb, le, lb - layer_begin, k_new, v_new, s)
                                 : le - lb == 1 ? launch_append<1, false>(cache, lb, le, lb - layer_begin, k_new, v_new, s)
                                                : launch_append<LMAX, false>(cache, lb, le, lb - layer_begin, k_new, v_new, s);
            if (e != hipSuccess) return hip_fail(e, "append launch");
        }
        for (int l = lb; l < le; ++l) {
            cache->st[l].n += 1;
            if (has_buffer(cache, l)) cache->st[l].c += 1;       // a layer of Algorithm-1 spatial heads only has no row buffer
        }
        lb = le;
    }
    return SSD_OK;
}
