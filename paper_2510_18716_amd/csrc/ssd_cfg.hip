// ssd_cfg_mix: classifier-free guidance of the two next-token distributions of each prompt (Sec. 3.1,
// Eq. 1):  out[i, v] = p[2i, v] + gamma * (p[2i, v] - p[2i+1, v]),  sequence 2i being the pass conditioned
// on the prompt and 2i+1 the unconditional one.  It is what follows the decode attention of the last layer
// on the way to the next token: after it, one token is sampled per prompt and fed to both sequences.
//
// Elementwise and read-once, so the bound is HBM: 2 * V * e bytes in and 4 * V bytes out per prompt -- at the sizes of an
// image vocabulary the launch itself (64 prompts of 16384: 8.4 MB, 1.6 us at the rate of a large read).  Each lane takes
// 16-byte fragments of the two rows (coalesced) and writes fp32.  Rows of a length that breaks the 16-byte alignment are
// read and written in the same pieces, element-aligned (the hardware takes a 16-byte access at any element boundary);
// the last, shorter piece of a row goes element by element, all of its loads in flight together.  Short rows share
// a workgroup.
// Measured, against one element per lane with a division each for unaligned rows and flat pieces with a division each for
// aligned ones: 256 prompts of 47911 (bf16) 20.0 -> 17.5 us (4.8 TB/s); 256 of 65536 22.5 -> 22.7; 64 prompts of 16384 stay at 3.5 us,
// the launch.  Short rows: 65536 prompts of 16 3.5 us (30 with a workgroup of its own for each row), 16384 of 257 9.2 -> 7.7.
#include <cmath>

#include "ssd_device.h"

namespace ssd {

struct CfgArgs {
    const char *p;
    float *out;
    int V;
    int n_prompts;
    int lanes_log2;     // threads of a workgroup that share a row: 1, 2, .. 256
    float gamma;
};

static __device__ __forceinline__ float widen(float x) { return x; }
static __device__ __forceinline__ float widen(bf16_t x) { return __uint_as_float((uint32_t)x.bits << 16); }

// 16 bytes at a 16-byte aligned address, and at any element's address
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef u32x4_nt_t u32x4_any_t __attribute__((aligned(2)));
typedef f32x4_t f32x4_any_t __attribute__((aligned(4)));

// Unaligned rows with little work in all: one element per lane.  Such a launch is one round trip to memory and the time to
// get there: 2 prompts of 47911 (bf16) take 2.7 us this way, 3.0 in pieces; 16384 of 7 2.7 and 3.4.
template <typename T>
__global__ __launch_bounds__(256) void cfg_mix_few_kernel(CfgArgs a) {
    const unsigned x = blockIdx.x * 256u + threadIdx.x;
    if (x >= (unsigned)a.V * (unsigned)a.n_prompts) return;
    const unsigned i = x / (unsigned)a.V;
    const T *c = reinterpret_cast<const T *>(a.p) + (size_t)x + (size_t)i * a.V;           // row 2i of p, at the element's place in row i of out
    const float xc = widen(c[0]), xu = widen(c[a.V]);
    a.out[x] = fmaf(a.gamma, xc - xu, xc);
}

// grid = (blocks over the pieces of a row, blocks over the prompts), 256 >> lanes_log2 rows per workgroup: nothing has to be
// divided
template <typename T, bool ALIGNED>
__global__ __launch_bounds__(256) void cfg_mix_kernel(CfgArgs a) {
    constexpr int VEC = Elem<T>::VEC;
    const int pieces = a.V / VEC, rest = a.V % VEC;
    const int lanes = 1 << a.lanes_log2, rows = 256 >> a.lanes_log2;
    const int row = (int)threadIdx.x >> a.lanes_log2, first = (int)threadIdx.x & (lanes - 1);
    for (long long i = (long long)blockIdx.y * rows + row; i < a.n_prompts; i += (long long)gridDim.y * rows) {
        const T *c = reinterpret_cast<const T *>(a.p) + (size_t)(2 * i) * a.V;
        const T *u = c + a.V;
        float *o = a.out + (size_t)i * a.V;
        for (int j = (int)blockIdx.x * lanes + first; j <= pieces; j += (int)gridDim.x * lanes) {
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
            } else if constexpr (!ALIGNED) {
                if (rest == 0) continue;
                float x[VEC], y[VEC];
#pragma unroll
                for (int e = 0; e < VEC; ++e) {            // unconditional loads: past the end the last element again
                    const int v = e < rest ? v0 + e : a.V - 1;
                    x[e] = widen(c[v]);
                    y[e] = widen(u[v]);
                }
#pragma unroll
                for (int e = 0; e < VEC; ++e)
                    if (e < rest) o[v0 + e] = fmaf(a.gamma, x[e] - y[e], x[e]);
            }
        }
    }
}

template <typename T>
static hipError_t launch_mix_few(const CfgArgs &a, hipStream_t s) {
    hipLaunchKernelGGL((cfg_mix_few_kernel<T>), dim3(((unsigned)a.V * (unsigned)a.n_prompts + 255u) / 256u), dim3(256), 0, s, a);
    return hipGetLastError();
}

template <typename T, bool ALIGNED>
static hipError_t launch_mix(CfgArgs a, hipStream_t s) {
    const int want = a.V / Elem<T>::VEC + (ALIGNED ? 0 : 1);   // pieces of a row, the shorter last one included
    // A workgroup of its own for a row of at most 128 pieces leaves half of it idle: 4096 prompts of 512 (fp32) 4.1 us shared, 4.7
    // alone; 16384 of 132 4.8 and 9.7.  Where HBM bounds the launch, bf16 rows (half of whose traffic is stores of two pieces per lane) gain
    // by it: 16384 of 1024 23.2 us shared, 20.9 alone; 4096 of 1000 6.5 and 6.2; 4096 of 640 5.0 and 5.2.
    const bool alone = want > 128 || (sizeof(T) == 2 && want >= 64 && (long long)a.V * a.n_prompts > 4000000);
    a.lanes_log2 = alone ? 8 : 0;
    while (a.lanes_log2 < 8 && 1 << a.lanes_log2 < want) ++a.lanes_log2;
    const int rows = 256 >> a.lanes_log2, gx = want / 256 + (want % 256 ? 1 : 0);
    const int gy = a.n_prompts / rows + (a.n_prompts % rows ? 1 : 0);
    const dim3 grid(gx > 1024 ? 1024 : gx, gy < 65535 ? gy : 65535);                   // strides cover the rest
    hipLaunchKernelGGL((cfg_mix_kernel<T, ALIGNED>), grid, dim3(256), 0, s, a);
    return hipGetLastError();
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
    const bool rows_aligned = V % (dtype == SSD_F32 ? 4 : 8) == 0;     // p is 16-byte aligned; then so is every row of p and of out
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e;
    // The line: 64 prompts of 8191 (bf16) 3.25 us by elements, 3.4 in pieces; 4096 of 1000 6.5 and 6.2 (256 of 47911 20.0 and 17.5).
    const bool few = !rows_aligned && (long long)V * a.n_prompts <= 600000;
    if (dtype == SSD_BF16) e = few ? launch_mix_few<bf16_t>(a, s) : rows_aligned ? launch_mix<bf16_t, true>(a, s) : launch_mix<bf16_t, false>(a, s);
    else e = few ? launch_mix_few<float>(a, s) : rows_aligned ? launch_mix<float, true>(a, s) : launch_mix<float, false>(a, s);
    if (e != hipSuccess) return hip_fail(e, "guidance mix launch");
    return SSD_OK;
}
