// Attention-mass density proxy (Warp-Cortex Sec. 3.3, "Attention Score Summation").
//
// Per layer, A_i = sum over the layer's query heads of softmax_i(scale * q . K_i): one dot
// product per (query head, cached token), so the keys are read ONCE -- an HBM-bound sweep, against
// the O(L^2 d) of the kernel density it can stand in for.  Two kernels:
//   mass_logits   one workgroup per (1024-token tile, KV head): the logits of all query heads that share the KV head
//                 from one read of the key rows; writes them (log2 units; staged in LDS, one coalesced pass per tile) and
//                 a (max, sum of exp2) pair per (query head, tile).  The dot products are MFMA tiles of 16 keys by up to
//                 16 query heads, whose operand is fetched from memory as it is, 64 bytes of a row by four lanes
//                 (mass_logits_rows, for fp32 keys, one or two query heads where the chip is full, and workspaces that hold a
//                 pair per 2048 tokens only: 2048 tokens, a lane group per row);
//   mass_combine  folds the pairs of a layer's heads into (max, 1/sum) per head, then per token adds
//                 the normalised exponentials over the heads and writes the result to every KV head
//                 of the layer (as A, or as 1/A when it is to serve as the density).
#include "ws_internal.h"

namespace ws {

namespace {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kMassTile = 1024;    // tokens per workgroup of mass_logits ...
constexpr int kRowTile = 2048;     // ... and of mass_logits_rows
constexpr int kMassFull = 512;     // tiles of mass_logits that fill the chip (a fixed number: the result follows the sizes only)
constexpr int kMassMaxHq = 128;    // query heads per layer
constexpr float kLog2e = 1.4426950408889634f;

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

template <bool BF16>
struct Piece;   // 16 bytes of a row, widened to floats
template <>
struct Piece<true> {
    static constexpr int PER = 8;
    static __device__ __forceinline__ void widen(const uint4 &q, float (&f)[8])
    {
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            f[2 * j] = __uint_as_float(w[j] << 16);
            f[2 * j + 1] = __uint_as_float(w[j] & 0xFFFF0000u);
        }
    }
};
template <>
struct Piece<false> {
    static constexpr int PER = 4;
    static __device__ __forceinline__ void widen(const uint4 &q, float (&f)[4])
    {
        f[0] = __uint_as_float(q.x);
        f[1] = __uint_as_float(q.y);
        f[2] = __uint_as_float(q.z);
        f[3] = __uint_as_float(q.w);
    }
};

// (max, sum of exp2(z - max)) pairs merge associatively; an empty pair is (-inf, 0)
__device__ __forceinline__ void merge(float &m, float &s, float m2, float s2)
{
    const float mn = fmaxf(m, m2);
    const float a = (m > -__builtin_inff()) ? s * __builtin_amdgcn_exp2f(m - mn) : 0.0f;
    const float b = (m2 > -__builtin_inff()) ? s2 * __builtin_amdgcn_exp2f(m2 - mn) : 0.0f;
    m = mn;
    s = a + b;
}

// The form for fp32 keys and, where the chip is full, for one or two query heads per KV head: a lane group per row reads it whole, and the
// arithmetic is little enough (24 x 16 heads of 32768 keys, d = 64, one query head each: 0.30 ms, 0.36 through the MFMA form).
// It also serves more query heads where the caller's workspace has a pair per 2048 tokens.
template <bool BF16, int D, int MAXG>
__global__ void __launch_bounds__(256)
mass_logits_rows(const void *__restrict__ Kv, const void *__restrict__ Qv, float *__restrict__ z,
                 float2 *__restrict__ part, int L, int g, float scale2 /* scale * log2(e) */, int nblk)
{
    typedef Piece<BF16> P;
    constexpr int PER = P::PER;
    constexpr int ES = BF16 ? 2 : 4;
    constexpr int LPR = D / PER;          // lanes per key row
    constexpr int RP = 256 / LPR;         // rows per pass of the workgroup
    constexpr int UN = 4;                 // rows in flight per lane group
    __shared__ float wm[4][MAXG], wsum[4][MAXG];
    // The logits of the tile wait in LDS and leave in one coalesced pass at the end: a 4-byte store per row group
    // inside the streaming loop costs a memory transaction per 32 bytes.  (Eight query heads per KV head would need
    // 64 KB: those keep the direct stores.)
    constexpr bool STAGE = MAXG <= 4;
    __shared__ float zt[STAGE ? MAXG : 1][STAGE ? kRowTile : 1];

    const int kvh = blockIdx.y, blk = blockIdx.x;
    const int tid = threadIdx.x, sub = tid % LPR, rsub = tid / LPR;
    const char *Kh = reinterpret_cast<const char *>(Kv) + (size_t)kvh * L * D * ES;

    float qf[MAXG][PER];
#pragma unroll
    for (int j = 0; j < MAXG; ++j) {
        const int qh = kvh * g + (j < g ? j : 0);
        const uint4 qq = *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(Qv) + ((size_t)qh * D + sub * PER) * ES);
        P::widen(qq, qf[j]);
    }
    float m[MAXG], s[MAXG];
#pragma unroll
    for (int j = 0; j < MAXG; ++j) {
        m[j] = -__builtin_inff();
        s[j] = 0.0f;
    }

    const int lo = blk * kRowTile, hi = min(L, lo + kRowTile);
    for (int r0 = lo; r0 < hi; r0 += UN * RP) {
        uint4 q[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int i = min(r0 + u * RP + rsub, hi - 1);
            // the keys stream through once: loads marked non-temporal keep them from displacing anything cached
            const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(Kh + ((size_t)i * D + sub * PER) * ES));
            q[u] = make_uint4(v.x, v.y, v.z, v.w);
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int i = r0 + u * RP + rsub;
            float f[PER];
            P::widen(q[u], f);
#pragma unroll
            for (int j = 0; j < MAXG; ++j) {
                if (j < g) {
                    float acc = 0.0f;
#pragma unroll
                    for (int e = 0; e < PER; ++e) acc = fmaf(f[e], qf[j][e], acc);
                    acc = lane_group_sum<LPR>(acc);
                    const float zz = acc * scale2;
                    if (i < hi) {
                        if (sub == 0) {
                            if constexpr (STAGE) zt[j][i - lo] = zz;
                            else z[(size_t)(kvh * g + j) * L + i] = zz;
                        }
                        const float mn = fmaxf(m[j], zz);
                        s[j] = s[j] * __builtin_amdgcn_exp2f(m[j] - mn) + __builtin_amdgcn_exp2f(zz - mn);
                        m[j] = mn;
                    }
                }
            }
        }
    }
    // one lane per row group speaks for its rows; fold the lanes of a wave, then the 4 waves
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int j = 0; j < MAXG; ++j) {
        if (j < g) {
            float mm = (sub == 0) ? m[j] : -__builtin_inff();
            float ss = (sub == 0) ? s[j] : 0.0f;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const float m2 = __shfl_xor(mm, o), s2 = __shfl_xor(ss, o);
                merge(mm, ss, m2, s2);
            }
            if (lane == 0) {
                wm[wave][j] = mm;
                wsum[wave][j] = ss;
            }
        }
    }
    __syncthreads();
    if constexpr (STAGE) {
#pragma unroll
        for (int j = 0; j < MAXG; ++j)
            if (j < g)
                for (int i = lo + tid; i < hi; i += 256) z[(size_t)(kvh * g + j) * L + i] = zt[j][i - lo];
    }
    if (tid < g) {
        float mm = wm[0][tid], ss = wsum[0][tid];
        for (int w = 1; w < 4; ++w) merge(mm, ss, wm[w][tid], wsum[w][tid]);
        part[(size_t)(kvh * g + tid) * nblk + blk] = make_float2(mm, ss);
    }
}

// What bounds it: the read of the keys (nothing is left of the arithmetic on the vector pipe but the exponentials of the
// staged logits, one per logit).  With a lane group per row, its dot products, the sums over its lanes and a running
// softmax in every lane of it, the vector pipe took half of the time: 8 heads of 131072 keys, d = 128, four query heads
// each, 94 us for the call; 64 now.
template <int D, int MAXG>
__global__ void __launch_bounds__(256)
mass_logits(const void *__restrict__ Kv, const void *__restrict__ Qv, float *__restrict__ z,
            float2 *__restrict__ part, int L, int g, float scale2 /* scale * log2(e) */, int nblk)
{
    __shared__ float wm[4][MAXG], wsum[4][MAXG];
    // The logits of the tile wait in LDS and leave in one coalesced pass at the end: a 4-byte store per row group
    // inside the streaming loop costs a memory transaction per 32 bytes.
    __shared__ __align__(16) float zt[MAXG][kMassTile];

    const int kvh = blockIdx.y, blk = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lo = blk * kMassTile, hi = min(L, lo + kMassTile);
    {
        // lane l: key l % 16 of a tile (and query head l % 16), elements kk*32 + (l / 16)*8 ... +7 of it
        constexpr int NK = D / 32, UN = 4;     // k-steps; 16-key tiles in flight per wave
        const int n = lane & 15, kg = lane >> 4;
        const uint16_t *Kh = reinterpret_cast<const uint16_t *>(Kv) + (size_t)kvh * L * D;
        bf16x8_t qf[NK];
        const uint16_t *qr = reinterpret_cast<const uint16_t *>(Qv) + (size_t)(kvh * g + min(n, g - 1)) * D;
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) qf[kk] = *reinterpret_cast<const bf16x8_t *>(qr + kk * 32 + kg * 8);
        for (int r0 = lo + wave * 16 * UN; r0 < hi; r0 += 4 * 16 * UN) {
            u32x4_t q[UN][NK];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const uint16_t *kr = Kh + (size_t)min(r0 + u * 16 + n, hi - 1) * D + kg * 8;
                // the keys stream through once: loads marked non-temporal keep them from displacing anything cached
#pragma unroll
                for (int kk = 0; kk < NK; ++kk) q[u][kk] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(kr + kk * 32));
            }
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                // a sum per k-step, added pairwise: a chain through one accumulator rounds the whole sum at every step
                const f32x4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
                f32x4_t p[NK];
#pragma unroll
                for (int kk = 0; kk < NK; ++kk)
                    p[kk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, q[u][kk]), qf[kk], zero, 0, 0, 0);
                f32x4_t acc = p[0] + p[1];
                if constexpr (NK == 4) acc += p[2] + p[3];
                // this lane holds query head n against keys kg*4 ... +3 (keys past the end are staged, not used)
                if (n < g) *reinterpret_cast<f32x4_t *>(&zt[n][r0 - lo + u * 16 + kg * 4]) = acc * scale2;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < MAXG; ++j) {
        if (j < g) {
            constexpr int PT = kMassTile / 256;
            float v[PT], mm = -__builtin_inff(), ss = 0.0f;
#pragma unroll
            for (int e = 0; e < PT; ++e) {
                const int i = lo + tid + 256 * e;
                v[e] = i < hi ? zt[j][i - lo] : -__builtin_inff();
                mm = fmaxf(mm, v[e]);
                if (i < hi) z[(size_t)(kvh * g + j) * L + i] = v[e];
            }
#pragma unroll
            for (int e = 0; e < PT; ++e)
                if (lo + tid + 256 * e < hi) ss += __builtin_amdgcn_exp2f(v[e] - mm);
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const float m2 = __shfl_xor(mm, o), s2 = __shfl_xor(ss, o);
                merge(mm, ss, m2, s2);
            }
            if (lane == 0) {
                wm[wave][j] = mm;
                wsum[wave][j] = ss;
            }
        }
    }
    __syncthreads();
    if (tid < g) {
        float mm = wm[0][tid], ss = wsum[0][tid];
        for (int w = 1; w < 4; ++w) merge(mm, ss, wm[w][tid], wsum[w][tid]);
        part[(size_t)(kvh * g + tid) * nblk + blk] = make_float2(mm, ss);
    }
}

__global__ void __launch_bounds__(256)
mass_combine(const float *__restrict__ z, const float2 *__restrict__ part, float *__restrict__ out, int L, int Hkv,
             int Hq, int nblk, int as_density)
{
    // A = sum over the heads of exp2(z - ref) * rinv, with an integer for ref and 2^(integer part of z - ref) split off: z - max
    // itself rounds at the size of the difference (2^-24 of 20 to 100 for most tokens), z - rint(z) is exact.  8 heads of
    // 131072 heavy-tailed keys, d = 128, four query heads each, mean 2-norm error of 1/A against 64 bits over 160 inputs:
    // 9.0e-7 with z - max, 8.3e-7 this way (with running sums in every lane and z - max: 8.3e-7); d = 64: 8.3e-7, 7.4e-7.
    __shared__ float ref[kMassMaxHq], rinv[kMassMaxHq];
    const int grp = blockIdx.y, tid = threadIdx.x;
    for (int q0 = 0; q0 < Hq; q0 += 32) {       // eight lanes per head
        const int q = q0 + tid / 8;
        float mm = -__builtin_inff(), ss = 0.0f;
        if (q < Hq) {
            const float2 *p = part + (size_t)(grp * Hq + q) * nblk;
            for (int b = tid & 7; b < nblk; b += 8) merge(mm, ss, p[b].x, p[b].y);
        }
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) {
            const float m2 = __shfl_xor(mm, o), s2 = __shfl_xor(ss, o);
            merge(mm, ss, m2, s2);
        }
        if (q < Hq && (tid & 7) == 0) {
            ref[q] = rintf(mm);
            rinv[q] = __builtin_amdgcn_exp2f(ref[q] - mm) / ss;
        }
    }
    __syncthreads();
    const int i = blockIdx.x * 256 + tid;
    if (i >= L) return;
    float A = 0.0f;
#pragma unroll 8
    for (int q = 0; q < Hq; ++q) {
        const float zz = z[(size_t)(grp * Hq + q) * L + i], whole = rintf(zz);
        A = fmaf(__builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f(zz - whole), (int)(whole - ref[q])), rinv[q], A);
    }
    const float v = as_density ? 1.0f / fmaxf(A, 1e-30f) : A;
    for (int hk = 0; hk < Hkv; ++hk) out[(size_t)(grp * Hkv + hk) * L + i] = v;
}

struct MassWs {
    size_t z, part, total;
    int nblk;
};

MassWs mass_layout(int G, int Hq, int L, int tile)
{
    MassWs w;
    w.nblk = (L + tile - 1) / tile;
    w.z = 0;
    w.part = round_up((size_t)G * Hq * L * sizeof(float), 256);
    w.total = w.part + round_up((size_t)G * Hq * w.nblk * sizeof(float2), 256);
    return w;
}

template <bool BF16, int D>
void run_logits(bool rows, const void *K, const void *Q, float *z, float2 *part, int GHkv, int L, int g, float scale2, int nblk,
                hipStream_t st)
{
    auto kern = mass_logits_rows<BF16, D, 8>;
    if (!rows) kern = g <= 4 ? mass_logits<D, 4> : mass_logits<D, 8>;
    else if (g == 1) kern = mass_logits_rows<BF16, D, 1>;
    else if (g == 2) kern = mass_logits_rows<BF16, D, 2>;
    else if (g <= 4) kern = mass_logits_rows<BF16, D, 4>;
    hipLaunchKernelGGL(kern, dim3(nblk, GHkv), dim3(256), 0, st, K, Q, z, part, L, g, scale2, nblk);
}

}  // namespace

bool mass_supported(int Hkv, int Hq) { return Hq % Hkv == 0 && Hq <= kMassMaxHq && Hq / Hkv <= 8; }

size_t mass_workspace_bytes(int G, int Hq, int L) { return mass_layout(G, Hq, L, kMassTile).total; }
size_t mass_workspace_least(int G, int Hq, int L) { return mass_layout(G, Hq, L, kRowTile).total; }

hipError_t launch_attention_mass(const void *K, const void *Q, bool bf16, int G, int Hkv, int Hq, int L, int d,
                                 float scale, int as_density, float *out, void *ws, size_t ws_bytes, hipStream_t st)
{
    const int g = Hq / Hkv;
    // Three and more query heads per KV head: 0.16 to 1.0 of the row form's time (2 heads of 32768 keys, d = 128, eight query
    // heads: 124 -> 20 us; 8 heads of 300 keys: equal).  One or two, where the chip is full (64 heads of 32768 keys, 8 of 131072,
    // 128 of 8192, both dimensions): the row form is 0.80 to 1.02 of the matrix cores' time (24 x 16 heads of 32768 keys, d = 64:
    // 298 us against 360; d = 128, two query heads: 592 against 692).  Below 512 tiles of 1024 keys the row form, with its larger
    // tiles and its longer chain per row, takes 1.0 to 2.6 times as long: one query head, d = 64, 480 tiles 25.4 us against 19.6, 8
    // tiles 17.0 against 15.6; d = 128, 256 tiles 39.4 against 18.7; two, d = 128, 32 tiles 35.6 against 15.7.  Error against 64 bits over 48 of
    // these sizes: 0.96 of the row form's.
    const bool idle = (long long)G * Hkv * ((L + kMassTile - 1) / kMassTile) < kMassFull;
    const bool rows = !bf16 || (g <= 2 && !idle) || ws_bytes < mass_workspace_bytes(G, Hq, L);
    const MassWs w = mass_layout(G, Hq, L, rows ? kRowTile : kMassTile);
    char *base = reinterpret_cast<char *>(ws);
    float *z = reinterpret_cast<float *>(base + w.z);
    float2 *part = reinterpret_cast<float2 *>(base + w.part);
    const float scale2 = scale * kLog2e;
    auto run = bf16 ? (d == 64 ? run_logits<true, 64> : run_logits<true, 128>)
                    : (d == 64 ? run_logits<false, 64> : run_logits<false, 128>);
    run(rows, K, Q, z, part, G * Hkv, L, g, scale2, w.nblk, st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(mass_combine, dim3((L + 255) / 256, G), dim3(256), 0, st, z, part, out, L, Hkv, Hq, w.nblk,
                       as_density);
    return hipGetLastError();
}

}  // namespace ws
