// ssd_cfg_mix: classifier-free guidance of the two next-token distributions of each prompt (Sec. 3.1,
// Eq. 1):  out[i, v] = p[2i, v] + gamma * (p[2i, v] - p[2i+1, v]),  sequence 2i being the pass conditioned
// on the prompt and 2i+1 the unconditional one.  It is what follows the decode attention of the last layer
// on the way to the next token: after it, one token is sampled per prompt and fed to both sequences.
//
// Elementwise and read-once, so the bound is HBM: 2 * V * e bytes in and 4 * V bytes out per prompt -- at the sizes of an
// image vocabulary the launch itself (64 prompts of 16384: 8.4 MB, 1.6 us at the rate of a large read).  Each lane takes
// 16-byte fragments of the two rows (coalesced) and writes fp32.  Rows of a length that breaks the 16-byte alignment are
// read and written in the same pieces, element-aligned (the hardware takes a 16-byte access at any element boundary);
// the last, shorter piece of a row goes element by element.
// Measured: 256 prompts of 47911 (rows of odd length, bf16): 27.2 us one element per lane with a division each, 20.3 now (4.8
// TB/s); 256 of 65536 27.8 -> 27.3.  64 prompts of 16384 stay at 3.6 us, the launch.
#include <cmath>

#include "ssd_device.h"

namespace ssd {

struct CfgArgs {
    const char *p;
    float *out;
    int V;
    int n_prompts;
    float gamma;
};

static __device__ __forceinline__ float widen(float x) { return x; }
static __device__ __forceinline__ float widen(bf16_t x) { return __uint_as_float((uint32_t)x.bits << 16); }

// 16 bytes at a 16-byte aligned address, and at any element's address
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef u32x4_nt_t u32x4_any_t __attribute__((aligned(2)));
typedef f32x4_t f32x4_any_t __attribute__((aligned(4)));

// grid = (blocks over the pieces of a row, prompts): nothing has to be divided
template <typename T, bool ALIGNED>
__global__ __launch_bounds__(256) void cfg_mix_kernel(CfgArgs a) {
    constexpr int VEC = Elem<T>::VEC;
    const int pieces = a.V / VEC, rest = a.V % VEC;
    for (int i = blockIdx.y; i < a.n_prompts; i += gridDim.y) {
        const T *c = reinterpret_cast<const T *>(a.p) + (size_t)(2 * (long long)i) * a.V;
        const T *u = c + a.V;
        float *o = a.out + (size_t)i * a.V;
        for (int j = (int)(blockIdx.x * 256 + threadIdx.x); j <= pieces; j += (int)(gridDim.x * 256)) {
            const int v0 = j * VEC;
            if (j < pieces) {
                u32x4_nt_t cr, ur;
                if constexpr (ALIGNED) {
                    cr = *reinterpret_cast<const u32x4_nt_t *>(c + v0);
                    ur = *reinterpret_cast<const u32x4_nt_t *>(u + v0);
                } else {
                    cr = *reinterpret_cast<const u32x4_any_t *>(c + v0);
                    ur = *reinterpret_cast<const u32x4_any_t *>(u + v0);
                }
                float cf[VEC], uf[VEC];
                Elem<T>::unpack(make_uint4(cr.x, cr.y, cr.z, cr.w), cf);
                Elem<T>::unpack(make_uint4(ur.x, ur.y, ur.z, ur.w), uf);
#pragma unroll
                for (int e = 0; e < VEC; e += 4) {
                    f32x4_t r;
#pragma unroll
                    for (int k = 0; k < 4; ++k) r[k] = fmaf(a.gamma, cf[e + k] - uf[e + k], cf[e + k]);
                    if constexpr (ALIGNED) *reinterpret_cast<f32x4_t *>(o + v0 + e) = r;
                    else *reinterpret_cast<f32x4_any_t *>(o + v0 + e) = r;
                }
            } else {
                for (int e = v0; e < v0 + rest; ++e) {
                    const float x = widen(c[e]), y = widen(u[e]);
                    o[e] = fmaf(a.gamma, x - y, x);
                }
            }
        }
    }
}

}  // namespace ssd

using namespace ssd;

extern "C" int ssd_cfg_mix(const void *p, int n_seqs, int V, int dtype, float gamma, float *out, void *stream) {
    clear_error();
    if (!p || !out) return fail(SSD_ERR_INVALID_ARG, "p or out is NULL");
    if (!aligned(p, 16) || !aligned(out, 16)) return fail(SSD_ERR_INVALID_ARG, "p and out must be 16-byte aligned");
    if (n_seqs < 2 || n_seqs % 2 != 0) return fail(SSD_ERR_INVALID_ARG, "n_seqs=%d must be even and >= 2 (conditional / unconditional pairs)", n_seqs);
    if (V < 1) return fail(SSD_ERR_INVALID_ARG, "V=%d must be >= 1", V);
    if (dtype != SSD_F32 && dtype != SSD_BF16) return fail(SSD_ERR_INVALID_ARG, "bad dtype");
    if (!std::isfinite(gamma)) return fail(SSD_ERR_INVALID_ARG, "gamma must be finite");
    CfgArgs a;
    a.p = static_cast<const char *>(p);
    a.out = out;
    a.V = V;
    a.n_prompts = n_seqs / 2;
    a.gamma = gamma;
    const int vec = dtype == SSD_F32 ? 4 : 8;
    const bool rows_aligned = V % vec == 0;                    // p is 16-byte aligned; then so is every row of p and of out
    const int want = V / vec + 1;                              // pieces of a row, the shorter last one included
    const unsigned gx = (unsigned)((V % vec ? want : want - 1) + 255) / 256;
    const dim3 grid(gx < 1 ? 1 : gx > 1024 ? 1024 : gx, (unsigned)(a.n_prompts < 65535 ? a.n_prompts : 65535));     // strides cover the rest
    hipStream_t s = static_cast<hipStream_t>(stream);
#define SSD_CFG(T_)                                                                                                  \
    do {                                                                                                             \
        if (rows_aligned) hipLaunchKernelGGL((cfg_mix_kernel<T_, true>), grid, dim3(256), 0, s, a);                  \
        else hipLaunchKernelGGL((cfg_mix_kernel<T_, false>), grid, dim3(256), 0, s, a);                              \
    } while (0)
    if (dtype == SSD_BF16) SSD_CFG(bf16_t); else SSD_CFG(float);
#undef SSD_CFG
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "guidance mix launch");
    return SSD_OK;
}
