// ssd_classify_heads: the sparsity metric s_{l,h} of Sec. 3.3 ("Spatial Sparsity Analysis") and
// the threshold rule of Eq. (3).
//
// One workgroup per (layer, head).  Each thread sums the ratios far/tot of a fixed, strided subset of the P*T terms; the
// partial sums are added in 64 bits, over each wave in registers and over the waves in order, so the result does not
// depend on scheduling and is bit-reproducible.  Offline: not on the per-token path.
// Bound: HBM, every term's two floats are read once (2 x 35 MB at the 7B shape with 16 profiled sequences).  A thread
// takes its terms UNROLL pieces at a time, all 2 * UNROLL loads in flight together, the pieces counted through the P
// rows of T terms as one run; a piece is four terms where T is a multiple of four (at any float's address: the same sums in
// the same order whatever the alignment), one otherwise.
// Measured at L x H = 960, P = 16, T = 576 (71 MB): 48 us with one term per load and one load of each array in flight, 13.8
// now (5.1 TB/s).
#include "ssd_device.h"

namespace ssd {

typedef float f32x4_any_t __attribute__((ext_vector_type(4), aligned(4)));      // 16 bytes at any float's address

template <int VEC> struct Piece { float v[VEC]; };
template <int VEC> static __device__ __forceinline__ Piece<VEC> load_piece(const float *p) {
    Piece<VEC> r;
    if constexpr (VEC == 4) {
        const f32x4_any_t x = __builtin_nontemporal_load(reinterpret_cast<const f32x4_any_t *>(p));
        r.v[0] = x.x; r.v[1] = x.y; r.v[2] = x.z; r.v[3] = x.w;
    } else {
        r.v[0] = *p;
    }
    return r;
}

// Sum over the 64 lanes of a wave, in registers; every lane gets it.
static __device__ __forceinline__ double as_f64(unsigned long long v) { return __longlong_as_double((long long)v); }
static __device__ __forceinline__ double wave_sum_f64(double x) {
    auto bits = [](double v) { return (unsigned long long)__double_as_longlong(v); };
    x += as_f64(dpp_u64<0xB1>(bits(x)));       // quad_perm [1,0,3,2]
    x += as_f64(dpp_u64<0x4E>(bits(x)));       // quad_perm [2,3,0,1]
    x += as_f64(dpp_u64<0x141>(bits(x)));      // row_half_mirror
    x += as_f64(dpp_u64<0x140>(bits(x)));      // row_mirror: 16 lanes done
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
}

// first: the head of workgroup 0 (a launch holds at most 2^32 threads); inv: 1 / (P * T)
template <int VEC, int THREADS, int UNROLL>
__global__ __launch_bounds__(THREADS) void classify_kernel(const float *__restrict__ far, const float *__restrict__ tot, int first,
                                                           int P, int H, int T, double inv, float tau, float *s_out, uint8_t *type_out) {
    __shared__ double part[THREADS / 64];
    const int head = first + (int)blockIdx.x;
    const int l = head / H, h = head % H;
    const int tid = threadIdx.x;
    const size_t row = (size_t)H * (size_t)T;              // floats from one sequence's row of this head to the next one's
    const size_t row0 = ((size_t)l * P * H + h) * (size_t)T;
    const float *f0 = far + row0, *t0 = tot + row0;
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
    // a thread's few terms are summed in fp32, everything beyond in 64 bits
    double mine = acc[0];
#pragma unroll
    for (int e = 1; e < VEC; ++e) mine += (double)acc[e];
    mine = wave_sum_f64(mine);
    if ((tid & 63) == 0) part[tid >> 6] = mine;
    __syncthreads();
    if (tid == 0) {
        double sum = part[0];
#pragma unroll
        for (int w = 1; w < THREADS / 64; ++w) sum += part[w];
        const float s = (float)(sum * inv);
        if (s_out) s_out[head] = s;
        if (type_out) type_out[head] = s > tau ? SSD_SEMANTIC : SSD_SPATIAL;
    }
}

// Pieces per head up to which a workgroup is 256 threads with one piece each in flight.  With more, 512 threads with four:
// 64 heads of 2304 pieces 7.0 -> 4.7 us, 960 heads 13.4 and 13.8, 4096 heads 49 -> 45.  With fewer, four pieces are requested
// in vain and half the waves have nothing to do: 960 heads of 16 pieces 3.2 us against 3.9, of 576 5.8 against 7.0; 1280 heads of 16
// 3.5 against 4.7; 32768 heads of 16 23 against 59, of 576 87 against 146.  (All with the waves' sums in fp32; in 64 bits each
// takes 0.1 to 0.2 us more, 32768 heads 2.5, and the error against 64 bits falls from 5e-8 to the result's own rounding, 2.3e-8.)
static constexpr int LITTLE = 1024;

template <int VEC, int THREADS, int UNROLL>
static hipError_t launch_classify(const float *far, const float *tot, int heads, int P, int H, int T, float tau, float *s_out, uint8_t *type_out, hipStream_t s) {
    constexpr int MOST = (int)(0xffffffffu / THREADS);     // workgroups of one launch
    for (int first = 0; first < heads; first += MOST) {
        const int n = heads - first < MOST ? heads - first : MOST;
        hipLaunchKernelGGL((classify_kernel<VEC, THREADS, UNROLL>), dim3((unsigned)n), dim3(THREADS), 0, s, far, tot, first, P, H, T, 1.0 / ((double)P * T), tau, s_out, type_out);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess || heads - first <= MOST) return e;
    }
    return hipSuccess;
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
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int heads = L * H;
    const bool four = T % 4 == 0;
    const bool little = (long long)P * T / (four ? 4 : 1) <= LITTLE;
    const hipError_t e = four ? (little ? launch_classify<4, 256, 1>(far, tot, heads, P, H, T, tau, s_out, type_out, s)
                                        : launch_classify<4, 512, 4>(far, tot, heads, P, H, T, tau, s_out, type_out, s))
                              : (little ? launch_classify<1, 256, 1>(far, tot, heads, P, H, T, tau, s_out, type_out, s)
                                        : launch_classify<1, 512, 4>(far, tot, heads, P, H, T, tau, s_out, type_out, s));
    if (e != hipSuccess) return hip_fail(e, "classification launch");
    return SSD_OK;
}
