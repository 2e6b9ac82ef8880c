// ssd_classify_heads: the sparsity metric s_{l,h} of Sec. 3.3 ("Spatial Sparsity Analysis") and
// the threshold rule of Eq. (3).
//
// One workgroup per (layer, head).  Each thread sums the ratios far/tot of a fixed, strided subset of the P*T terms;
// the partial sums are then added by a fixed binary tree in LDS, so the result does not depend on scheduling and is
// bit-reproducible.  Offline: not on the per-token path.
// Bound: HBM, every term's two floats are read once (2 x 35 MB at the 7B shape with 16 profiled sequences).  A thread
// takes its terms UNROLL pieces at a time, all 2 * UNROLL loads in flight together, the pieces counted through the P
// rows of T terms as one run; a piece is four terms where rows keep 16-byte alignment, one otherwise.
// Measured at L x H = 960, P = 16, T = 576 (71 MB), call to call: 32.4 us with one term per load and one load of each
// array in flight, 13.3 us now (5.3 TB/s; 14.0 with workgroups of 256).
#include "ssd_device.h"

namespace ssd {

static constexpr int UNROLL = 4;

template <int VEC> struct Piece { float v[VEC]; };
template <int VEC> static __device__ __forceinline__ Piece<VEC> load_piece(const float *p) {
    Piece<VEC> r;
    if constexpr (VEC == 4) {
        const uint4 x = load_once(reinterpret_cast<const char *>(p));
        r.v[0] = __uint_as_float(x.x); r.v[1] = __uint_as_float(x.y); r.v[2] = __uint_as_float(x.z); r.v[3] = __uint_as_float(x.w);
    } else {
        r.v[0] = *p;
    }
    return r;
}

template <int VEC, int THREADS>
__global__ __launch_bounds__(THREADS) void classify_kernel(const float *__restrict__ far, const float *__restrict__ tot,
                                                           int P, int H, int T, float tau, float *s_out, uint8_t *type_out) {
    __shared__ float part[THREADS];
    const int l = blockIdx.x / H, h = blockIdx.x % H;
    const int tid = threadIdx.x;
    const size_t row = (size_t)H * (size_t)T;              // floats from one sequence's row of this head to the next one's
    const size_t first = ((size_t)l * P * H + h) * (size_t)T;
    const float *f0 = far + first, *t0 = tot + first;
    // piece j of sequence p; the thread's next piece is THREADS pieces on
    const int per_row = T / VEC;                           // VEC == 4 only if T is a multiple of 4
    const int dp = THREADS / per_row, dj = THREADS % per_row;
    int p = tid / per_row, j = tid % per_row;
    float acc[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
    while (p < P) {
        Piece<VEC> num[UNROLL], den[UNROLL];
        bool in[UNROLL];
#pragma unroll
        for (int k = 0; k < UNROLL; ++k) {                 // unconditional loads: past the end the last row's first piece
            in[k] = p < P;
            const size_t at = in[k] ? (size_t)p * row + (size_t)j * VEC : (size_t)(P - 1) * row;
            num[k] = load_piece<VEC>(f0 + at);
            den[k] = load_piece<VEC>(t0 + at);
            p += dp;
            j += dj;
            if (j >= per_row) { j -= per_row; ++p; }
        }
#pragma unroll
        for (int k = 0; k < UNROLL; ++k)
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[e] += in[k] && den[k].v[e] > 0.f ? num[k].v[e] / den[k].v[e] : 0.f;
    }
    float mine = acc[0];
#pragma unroll
    for (int e = 1; e < VEC; ++e) mine += acc[e];
    part[tid] = mine;
    __syncthreads();
    for (int w = THREADS / 2; w > 0; w >>= 1) {
        if (tid < w) part[tid] += part[tid + w];
        __syncthreads();
    }
    if (tid == 0) {
        const float s = part[0] / ((float)P * (float)T);
        if (s_out) s_out[blockIdx.x] = s;
        if (type_out) type_out[blockIdx.x] = s > tau ? SSD_SEMANTIC : SSD_SPATIAL;
    }
}

}  // namespace ssd

using namespace ssd;

extern "C" int ssd_classify_heads(const float *far, const float *tot, int L, int P, int H, int T, float tau,
                                  float *s_out, uint8_t *type_out, void *stream) {
    clear_error();
    if (!far || !tot) return fail(SSD_ERR_INVALID_ARG, "far or tot is NULL");
    if (!s_out && !type_out) return fail(SSD_ERR_INVALID_ARG, "s_out and type_out are both NULL");
    if (L < 1 || P < 1 || H < 1 || T < 1) return fail(SSD_ERR_INVALID_ARG, "L, P, H, T must be >= 1");
    if ((long long)L * H > 0x7fffffffLL) return fail(SSD_ERR_INVALID_ARG, "L*H too large");
    if (!aligned(far, 4) || !aligned(tot, 4) || !aligned(s_out, 4)) return fail(SSD_ERR_INVALID_ARG, "misaligned pointer");
    if (!(tau == tau)) return fail(SSD_ERR_INVALID_ARG, "tau is NaN");
    const dim3 grid((unsigned)(L * H));
    hipStream_t s = static_cast<hipStream_t>(stream);
#define SSD_CLASSIFY(VEC_, THREADS_) hipLaunchKernelGGL((classify_kernel<VEC_, THREADS_>), grid, dim3(THREADS_), 0, s, far, tot, P, H, T, tau, s_out, type_out)
    if (T % 4 == 0 && aligned(far, 16) && aligned(tot, 16)) SSD_CLASSIFY(4, 512);
    else SSD_CLASSIFY(1, 512);
#undef SSD_CLASSIFY
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "classification launch");
    return SSD_OK;
}
