// Greedy landmark selection for heads that fit the registers of one workgroup (Warp-Cortex Sec. 3.3).
//
// Between workgroups a step costs two to five thousand cycles of exchange whatever the head's size, and the streaming
// kernel reads D, u and the keys from memory again at every step.  A head of up to 1024 keys (d = 64; 512 at d = 128)
// needs neither: four lanes share a key row, whose elements they hold widened to fp32 in registers for all steps, D and u
// beside them; both maxima of a step (D_max, then the best score) meet in LDS, and the winner's owners leave its row
// there for everybody.  Distances are direct differences in fp32, the score is the streaming kernel's.  One workgroup per
// head, no wait on another one, so any number of heads may be launched.
// Bound by the chain of a step: distances (128 cycles of vector work per row slot and wave, two waves per SIMD), two
// reductions and three barriers.  One fp32 head of 512 keys, 10 steps: 56 us with the streaming kernel, 16
// here.
#include "select_resident_common.h"

namespace ws {

namespace {

using resident::wave_pick_lo;
using resident::wave_umax;

constexpr int kThreads = 512, kWaves = kThreads / 64;
constexpr int kLanes = 4;                       // lanes per key row
constexpr int kRows = kThreads / kLanes;        // key rows per slot

// elements c*16 + part*4 ... +3 of a key row, widened
__device__ __forceinline__ float4 load4(const float *row, int c, int part)
{
    return *reinterpret_cast<const float4 *>(row + c * 16 + part * 4);
}
__device__ __forceinline__ float4 load4(const uint16_t *row, int c, int part)
{
    const uint2 q = *reinterpret_cast<const uint2 *>(row + c * 16 + part * 4);
    return make_float4(__uint_as_float(q.x << 16), __uint_as_float(q.x & 0xFFFF0000u), __uint_as_float(q.y << 16),
                       __uint_as_float(q.y & 0xFFFF0000u));
}

// the largest of the waves' 32-bit entries
__device__ __forceinline__ unsigned waves_umax(const unsigned *e)
{
    unsigned v = e[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) v = max(v, e[w]);
    return v;
}

template <typename T, int D, int R>
__global__ void __launch_bounds__(kThreads)
select_small(const T *__restrict__ K, const float *__restrict__ rho, int32_t *__restrict__ idx, float *__restrict__ score_out,
             int *__restrict__ fail, int L, int k, float alpha)
{
    constexpr int NC = D / 16;
    __shared__ __align__(16) float lrow[D];              // the landmark just chosen
    __shared__ unsigned sd[kWaves], shi[kWaves], slo[kWaves];
    const int h = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int part = tid % kLanes, own = tid / kLanes;   // this lane's rows: own, own + kRows, ...
    const T *Kh = K + (size_t)h * L * D;
    const float *rhoh = rho + (size_t)h * L;
    const float oma = 1.0f - alpha;
    if (h == 0 && tid == 0) *fail = 0;                   // nothing here can give up

    float4 kf[R][NC];
    float Dv[R], u[R];                                   // D = -1: chosen, or past the end
    float rmin = __builtin_inff();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = own + kRows * r;
        const T *row = Kh + (size_t)min(i, L - 1) * D;
#pragma unroll
        for (int c = 0; c < NC; ++c) kf[r][c] = load4(row, c, part);
        u[r] = rhoh[min(i, L - 1)];
        rmin = fminf(rmin, u[r]);
        Dv[r] = i < L ? __builtin_inff() : -1.0f;
    }
    // min over positive floats = max over the complemented bit pattern
    const unsigned wmin = wave_umax(0xFFFFFFFFu - __float_as_uint(rmin));
    if (lane == 0) sd[wave] = wmin;
    __syncthreads();
    rmin = __uint_as_float(0xFFFFFFFFu - waves_umax(sd));
#pragma unroll
    for (int r = 0; r < R; ++r) u[r] = rmin / u[r];
    __syncthreads();

    for (int t = 0; t < k; ++t) {
        float dmax = 0.0f;
        if (t > 0) {
            float acc[R];
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r] = 0.0f;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const float4 m = *reinterpret_cast<const float4 *>(&lrow[c * 16 + part * 4]);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float d0 = kf[r][c].x - m.x, d1 = kf[r][c].y - m.y, d2 = kf[r][c].z - m.z, d3 = kf[r][c].w - m.w;
                    acc[r] = fmaf(d0, d0, acc[r]);
                    acc[r] = fmaf(d1, d1, acc[r]);
                    acc[r] = fmaf(d2, d2, acc[r]);
                    acc[r] = fmaf(d3, d3, acc[r]);
                }
            }
            float lmax = 0.0f;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float dist = __fsqrt_rn(lane_group_sum<kLanes>(acc[r]));
                Dv[r] = dist < Dv[r] ? dist : Dv[r];     // chosen keys stay at -1
                lmax = fmaxf(lmax, Dv[r]);
            }
            const unsigned wm = wave_umax(__float_as_uint(lmax));
            if (lane == 0) sd[wave] = wm;
            __syncthreads();
            dmax = __uint_as_float(waves_umax(sd));
        }
        int s = 0;
        float sc = alpha;
        if (t > 0 || alpha != 1.0f) {
            // score and argmax over the keys not chosen; rows in ascending order per lane
            float best = -1.0f;
            int bi = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float c = t == 0 ? 1.0f : (dmax > 0.0f ? Dv[r] / dmax : 0.0f);
                const float v = alpha * c + oma * u[r];
                if (Dv[r] >= 0.0f && v > best) {
                    best = v;
                    bi = own + kRows * r;
                }
            }
            // one of a row's lanes speaks for it; scores are >= 0, so their bits order like unsigned integers
            const bool has = part == 0 && best >= 0.0f;
            const unsigned hi = has ? __float_as_uint(best) : 0u, lo = has ? 0xFFFFFFu - (unsigned)bi : 0u;
            const unsigned whi = wave_umax(hi), wlo = wave_pick_lo(hi == whi, lo);
            if (lane == 0) {
                shi[wave] = whi;
                slo[wave] = wlo;
            }
            __syncthreads();
            const unsigned mhi = waves_umax(shi);
            unsigned mlo = 0u;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) mlo = max(mlo, shi[w] == mhi ? slo[w] : 0u);
            s = min((int)(0xFFFFFFu - mlo), L - 1);      // in range whatever the inputs held
            sc = __uint_as_float(mhi);
        }
        if (tid == 0) {
            idx[(size_t)h * k + t] = s;
            if (score_out) score_out[(size_t)h * k + t] = sc;
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (own + kRows * r == s) {
                Dv[r] = -1.0f;
#pragma unroll
                for (int c = 0; c < NC; ++c) *reinterpret_cast<float4 *>(&lrow[c * 16 + part * 4]) = kf[r][c];
            }
        __syncthreads();
    }
}

template <typename T, int D, int R>
hipError_t run(const void *K, int H, int L, const float *rho, int k, float alpha, int32_t *idx, float *score_out, int *fail,
               hipStream_t st)
{
    hipLaunchKernelGGL((select_small<T, D, R>), dim3(H), dim3(kThreads), 0, st, reinterpret_cast<const T *>(K), rho, idx,
                       score_out, fail, L, k, alpha);
    return hipGetLastError();
}

// key rows per four lanes of the instance that takes a head of L keys
int row_slots(int L) { return L <= 2 * kRows ? 2 : L <= 4 * kRows ? 4 : 8; }

template <typename T>
hipError_t dispatch(const void *K, int H, int L, int d, const float *rho, int k, float alpha, int32_t *idx, float *score_out,
                    int *fail, hipStream_t st)
{
    const int R = row_slots(L);
    if (d == 64) {
        if (R == 2) return run<T, 64, 2>(K, H, L, rho, k, alpha, idx, score_out, fail, st);
        if (R == 4) return run<T, 64, 4>(K, H, L, rho, k, alpha, idx, score_out, fail, st);
        return run<T, 64, 8>(K, H, L, rho, k, alpha, idx, score_out, fail, st);
    }
    if (R == 2) return run<T, 128, 2>(K, H, L, rho, k, alpha, idx, score_out, fail, st);
    return run<T, 128, 4>(K, H, L, rho, k, alpha, idx, score_out, fail, st);
}

}  // namespace

// bf16 heads up to one per compute unit: there the workgroups run at once and none shares its SIMDs.  Against the resident
// kernel, both dimensions, 16 to 1024 (512) keys, 1 to 256 heads, 2 % and a quarter of the keys picked: 0.42 of its time (200
// heads of 512 keys, 10 picks: 18 us against 43) to 0.98 (8 heads of 1024, 256 picks: 553 against 565), at no size more.  fp32
// heads always: against the streaming kernel 0.05 to 0.8 of its time up to 4000 heads.
int select_small_rows(bool bf16, int H, int L, int d, const Chip &chip)
{
    if (L > (d == 64 ? 8 : 4) * kRows || (bf16 && H > chip.cus)) return 0;
    return row_slots(L);
}

hipError_t launch_select_small(const void *K, bool bf16, int H, int L, int d, const float *rho, int k, float alpha,
                               int32_t *idx, float *score_out, int *fail, hipStream_t st)
{
    return (bf16 ? dispatch<uint16_t> : dispatch<float>)(K, H, L, d, rho, k, alpha, idx, score_out, fail, st);
}

}  // namespace ws
