// Density refresh after the context has grown by m rows (Warp-Cortex Sec. 4: the main stream
// re-extracts landmarks inside its decode loop, so the density must follow a cache that grows by a
// row per step).  L*rho is a plain sum of Gaussian kernel values: the m new keys add one kernel
// column each to the old keys' sums, and their own sums are column sums over all L keys.  That is
// one pass over K -- O(L m d), HBM-bound for small m -- instead of the O(L^2 d) sweep.
//   append_sweep   a workgroup per 2048-key tile of one head; the m new rows sit in LDS as fp32;
//                  a lane group per key row (16-byte loads, 4 rows in flight), squared distances by
//                  direct differences in fp32, exp2; what the new rows add to each old key waits in LDS
//                  and the tile's refreshed densities are written in one coalesced pass at the end (a
//                  4-byte load and store per row group inside the loop cost 13 %: each iteration then
//                  waits on memory twice); column sums leave as one partial per (tile, new row);
//   append_finish  adds the partials of each new row in tile order (deterministic) and writes the
//                  m new densities.
// bf16 keys and more than a few new rows: append_gram in place of append_sweep.
#include "ws_internal.h"

namespace ws {

namespace {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kAppTile = 2048;
constexpr int kAppMaxM = 32;
constexpr int kGramRows64 = 8, kGramRows128 = 4;    // new rows from which bf16 keys go through append_gram

constexpr int kAppChunk = 768;               // heads per launch: their scales travel as a kernel argument (3 KB)

struct AppScale {
    float s[kAppChunk];     // 0.5 * log2(e) / sigma^2 per head of the chunk
};

template <bool BF16>
__device__ __forceinline__ void widen16(const uint4 &q, float *f)
{
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
    if constexpr (BF16) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            f[2 * j] = __uint_as_float(w[j] << 16);
            f[2 * j + 1] = __uint_as_float(w[j] & 0xFFFF0000u);
        }
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) f[j] = __uint_as_float(w[j]);
    }
}

// N values of each lane summed over the LPR lanes of its group, the sums dealt out to the lanes: lane i is left with the sum of value
// i / (LPR / N).  While there is more than one value, half of them change hands at every step, so a lane of the group is left with one
// exponential to form instead of N.  The partners (mirror 16, mirror 8, xor 2, xor 1) are reached by DPP; a mirror also turns the lower bits
// of the lane around, which nothing depends on yet when it comes first.
template <int BIT>
__device__ __forceinline__ float partner(float v)
{
    if constexpr (BIT == 16) return __shfl_xor(v, 16);
    else return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), BIT == 8 ? 0x140 : BIT == 4 ? 0x141 : BIT == 2 ? 0x4E : 0xB1,
                                                           0xF, 0xF, false));
}

template <int LPR, int N>
__device__ __forceinline__ float group_scatter(const float (&v)[N], int part)
{
    constexpr int BIT = LPR / 2;
    if constexpr (LPR == 1) return v[0];
    else if constexpr (N == 1) {
        const float t[1] = {v[0] + partner<BIT>(v[0])};
        return group_scatter<BIT, 1>(t, part);
    } else {
        const bool upper = (part & BIT) != 0;
        float t[N / 2];
#pragma unroll
        for (int i = 0; i < N / 2; ++i)
            t[i] = (upper ? v[i + N / 2] : v[i]) + partner<BIT>(upper ? v[i] : v[i + N / 2]);
        return group_scatter<BIT, N / 2>(t, part);
    }
}

template <bool BF16, int D>
__global__ void __launch_bounds__(256)
append_sweep(const void *__restrict__ Kv, const float *__restrict__ rho_old, float *__restrict__ rho_new,
             float *__restrict__ colpart, AppScale sc, int head0, int L, int m, int nblk)
{
    constexpr int ES = BF16 ? 2 : 4;
    constexpr int PER = 16 / ES;
    constexpr int LPR = D / PER;
    constexpr int RP = 256 / LPR;
    constexpr int UN = 4;
    // The sums of a turn's keys are dealt out, one exponential per lane.  With every exponential in all the lanes of a group before: d = 64,
    // 384 heads of 32768 keys, 6 rows 430 -> 358 us, 4 rows 335 -> 323, fewer the same (bound by the read); fp32, 192 heads, 8 rows
    // 445 -> 333, 32 rows 1446 -> 1085; fp32, d = 128, 4 heads of 131072, 1 row 98 -> 91, 32 rows 668 -> 594; bf16, d = 128 the same.
    __shared__ float nr[kAppMaxM][D];        // the new rows, widened
    __shared__ float cs[kAppMaxM][RP];       // column sums, one slot per row group
    __shared__ float added[kAppTile];        // what the new rows add to each old key of the tile

    const int h = head0 + blockIdx.y, blk = blockIdx.x;
    const int tid = threadIdx.x, sub = tid % LPR, rsub = tid / LPR;
    const char *Kh = reinterpret_cast<const char *>(Kv) + (size_t)h * L * D * ES;
    const int Lold = L - m;
    const float s2 = sc.s[blockIdx.y];

    for (int q = tid; q < m * LPR; q += 256) {
        const int r = q / LPR, c = q % LPR;
        const uint4 v = *reinterpret_cast<const uint4 *>(Kh + ((size_t)(Lold + r) * D + c * PER) * ES);
        widen16<BF16>(v, &nr[r][c * PER]);
    }
    for (int q = tid; q < kAppMaxM * RP; q += 256) cs[q / RP][q % RP] = 0.0f;
    __syncthreads();

    const int lo = blk * kAppTile, hi = min(L, lo + kAppTile);
    for (int r0 = lo; r0 < hi; r0 += UN * RP) {
        uint4 q[UN];
        float x[UN][PER], add = 0.0f;
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int i = min(r0 + u * RP + rsub, hi - 1);
            // the keys stream through once: loads marked non-temporal keep them from displacing anything cached
            const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(Kh + ((size_t)i * D + sub * PER) * ES));
            q[u] = make_uint4(v.x, v.y, v.z, v.w);
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) widen16<BF16>(q[u], x[u]);
        const int mine = r0 + sub / (LPR / UN) * RP + rsub;     // the key whose sums this lane is left with
        for (int r = 0; r < m; ++r) {
            float y[PER], acc[UN];
#pragma unroll
            for (int e = 0; e < PER; ++e) y[e] = nr[r][sub * PER + e];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                acc[u] = 0.0f;
#pragma unroll
                for (int e = 0; e < PER; ++e) {
                    const float t = x[u][e] - y[e];
                    acc[u] = fmaf(t, t, acc[u]);
                }
            }
            const float d2 = group_scatter<LPR, UN>(acc, sub);
            const float w = mine < hi ? __builtin_amdgcn_exp2f(-d2 * s2) : 0.0f;
            add += w;
            const float col = lane_group_sum<LPR>(sub % (LPR / UN) == 0 ? w : 0.0f);
            if (sub == 0) cs[r][rsub] += col;          // slot private to this row group
        }
        if (mine < hi && sub % (LPR / UN) == 0) added[mine - lo] = add;
    }
    __syncthreads();
    // the old keys' refreshed densities, a whole tile at a time: consecutive threads, consecutive keys
    for (int i = lo + tid; i < min(hi, Lold); i += 256)
        rho_new[(size_t)h * L + i] = (rho_old[(size_t)h * Lold + i] * (float)Lold + added[i - lo]) / (float)L;
    if (tid < m) {
        float t = 0.0f;
        for (int g = 0; g < RP; ++g) t += cs[tid][g];
        colpart[((size_t)blockIdx.y * nblk + blk) * kAppMaxM + tid] = t;
    }
}

// The form for bf16 keys and more than a few new rows, where the direct differences of every pair are what the sweep is bound by
// (two instructions per element and pair against a read of two bytes per element).
//
// The dot products of 32 keys per turn of a wave with up to 16 (CT = 2: 32) new rows are MFMA tiles, operands fetched as they lie in memory, and
// |k - s|^2 = (|k|^2 - k.s) + (|s|^2 - k.s).  That is as exact as differences where the two rows are far apart, and loses what
// |k|^2 + |s|^2 exceeds the distance by where they are near: a pair nearer than kNear of it is evaluated by direct differences,
// eight lanes (16 at d = 128) to a pair, out of a list of the wave.  A wave that finds a tenth of its pairs near (rows that lie
// near each other as measured from the origin) evaluates the rest of its tile directly: from there the list would cost more.
// Every lane keeps the column sums of its rows, summed over the lanes at the end.
//
// Bound by the read of the keys as one new row is: 384 heads of 32768 keys, d = 64, 8 rows 540 -> 380 us (1 row: 317), 16 rows 990 ->
// 380; 8 heads of 131072, d = 128, 8 rows 148 -> 78 us, 32 rows 410 -> 84.  New rows out of the clusters of the old, so that a few
// per cent of the pairs go through the list: 547 -> 480, 987 -> 560, 147 -> 107.  All pairs near (keys at an offset of 20 per
// coordinate), so in the direct loop: 541 -> 443, 943 -> 775, 146 -> 117; with four keys in flight and an exponential in every lane
// of a group it took 619, 1065 and 160.  Fewer rows than the line stay with append_sweep (far / near /
// all near; 6 rows, d = 64: 355 / 350 / 340 against 376 / 460 / 380; 3 rows, d = 128: 88 / 88 / 88 against 77 / 90 / 77, 4 rows 99
// against 78 / 95 / 86, taken).
// Mean error of the new rows' densities over 36 refreshes: 0.73 of append_sweep's with its sums in fp32 to the end.
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2_t;

constexpr float kNear = 0.25f;      // beyond, rounding the norms and the product costs d^2 at most four roundings more than differences do
constexpr int kPairs = 96;          // pairs in a wave's list
constexpr int kMany = 3;            // near pairs per new row, of 32, from which a wave goes on directly (2 ... 6 are within 2 % at d = 64; at
                                    // d = 128, near pairs, 8 rows: 114, 103, 106, 106 us with 2, 3, 4, 6, and 4 rows 91, 95, 98, -)

// over the four lanes 16 apart, in all of them
__device__ __forceinline__ float quad_sum(float v)
{
    const u32x2_t a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a.x) + __uint_as_float(a.y);
    const u32x2_t b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(b.x) + __uint_as_float(b.y);
}

template <int D, int CT>
__global__ void __launch_bounds__(256)
append_gram(const uint16_t *__restrict__ K, const float *__restrict__ rho_old, float *__restrict__ rho_new,
            float *__restrict__ colpart, AppScale sc, int head0, int L, int m, int nblk)
{
    constexpr int NK = D / 32;              // MFMA k-steps
    constexpr int LPR = D / 8;              // lanes per row in the direct form ...
    constexpr int GRP = 64 / LPR;           // ... and rows a wave takes at a time
    constexpr int KT = 2, KB = 16 * KT;     // 16-key tiles, keys per turn of a wave
    constexpr int MR = 16 * CT;
    __shared__ float nr[MR][D];             // the new rows, widened
    __shared__ float nn[MR];                // their squared norms
    __shared__ float cs[4][MR];             // column sums per wave
    __shared__ float cd[MR][4 * GRP];       // column sums of the direct form, per row group
    __shared__ float added[kAppTile];       // what the new rows add to each old key of the tile
    __shared__ unsigned list[4][kPairs];    // pairs to evaluate directly: key of the turn << 8 | new row ...
    __shared__ float res[4][kPairs];        // ... and their squared distances

    const int h = head0 + blockIdx.y, blk = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, q = lane >> 4;         // key (new row) of a tile of 16; which 16-byte pieces of its row
    const uint16_t *Kh = K + (size_t)h * L * D;
    const int Lold = L - m;
    const float s2 = sc.s[blockIdx.y];
    const int lo = blk * kAppTile, hi = min(L, lo + kAppTile);

    u32x4_t kn[KT][NK];                             // the rows of the wave's next turn
    auto fetch = [&](int b0) {
#pragma unroll
        for (int j = 0; j < KT; ++j)
#pragma unroll
            for (int kk = 0; kk < NK; ++kk)         // the keys stream through once
                kn[j][kk] = __builtin_nontemporal_load(
                    reinterpret_cast<const u32x4_t *>(Kh + (size_t)min(b0 + j * 16 + c, hi - 1) * D + kk * 32 + q * 8));
    };
    fetch(lo + wave * KB);
    for (int i = tid; i < m * LPR; i += 256) {
        const int r = i / LPR, p = i % LPR;
        widen16<true>(*reinterpret_cast<const uint4 *>(Kh + (size_t)(Lold + r) * D + p * 8), &nr[r][p * 8]);
    }
    for (int i = tid; i < MR * 4 * GRP; i += 256) (&cd[0][0])[i] = 0.0f;
    u32x4_t a[CT][NK];                              // new rows 16 ct + c, elements 32 kk + 8 q ...
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int kk = 0; kk < NK; ++kk)
            a[ct][kk] = *reinterpret_cast<const u32x4_t *>(Kh + (size_t)(Lold + min(16 * ct + c, m - 1)) * D + kk * 32 + q * 8);
    __syncthreads();
    {
        // 256 / MR lanes per new row
        constexpr int LN = 256 / MR;
        const int r = tid / LN, p = tid % LN;
        float n = 0.0f;
        if (r < m)
#pragma unroll
            for (int e = 0; e < D / LN; ++e) n = fmaf(nr[r][p + e * LN], nr[r][p + e * LN], n);
        n = lane_group_sum<LN>(n);
        if (p == 0) nn[r] = n;
    }
    __syncthreads();
    float ns[CT][4], col[CT][4];                    // new rows 16 ct + 4 q + e
    bool use[CT][4];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            ns[ct][e] = nn[16 * ct + 4 * q + e];
            use[ct][e] = 16 * ct + 4 * q + e < m;
            col[ct][e] = 0.0f;
        }

    // a tile's products: a sum per k-step, added pairwise (a chain through one accumulator rounds the whole sum at every step)
    auto products = [&](const u32x4_t (&x)[NK], const u32x4_t (&y)[NK]) -> f32x4_t {
        const f32x4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
        f32x4_t t[NK];
#pragma unroll
        for (int kk = 0; kk < NK; ++kk)
            t[kk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, x[kk]), __builtin_bit_cast(bf16x8_t, y[kk]), zero, 0, 0, 0);
        f32x4_t g = t[0] + t[1];
        if constexpr (NK == 4) g += t[2] + t[3];
        return g;
    };

    const int part = lane % LPR, grp = lane / LPR;
    int b0 = lo + wave * KB;
    for (; b0 < hi; b0 += 4 * KB) {
        const bool tail = b0 + KB > Lold;           // new rows among the keys: a row's own 1 joins its sum last, in append_finish (what is
                                                    // left of it here is 0, or the NaN of a row with an infinity)
        bool far = true, last = false;
        u32x4_t k4[KT][NK];
#pragma unroll
        for (int j = 0; j < KT; ++j)
#pragma unroll
            for (int kk = 0; kk < NK; ++kk) k4[j][kk] = kn[j][kk];
        fetch(b0 + 4 * KB);                         // (past the tile: its last row, not used)
        float nk[KT], add[KT];
        bool in[KT];
#pragma unroll
        for (int j = 0; j < KT; ++j) {
            const f32x4_t g = products(k4[j], k4[j]);       // |k|^2: its diagonal
            const float dg = (c & 2) ? ((c & 1) ? g[3] : g[2]) : ((c & 1) ? g[1] : g[0]);
            nk[j] = quad_sum(q == c >> 2 ? dg : 0.0f);
            in[j] = b0 + j * 16 + c < hi;
            add[j] = 0.0f;
        }
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            float d2[KT][4];
            unsigned long long near[KT][4];
            int cnt = 0;
#pragma unroll
            for (int j = 0; j < KT; ++j) {
                const f32x4_t dot = products(a[ct], k4[j]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    d2[j][e] = (nk[j] - dot[e]) + (ns[ct][e] - dot[e]);
                    // (a NaN is near)
                    near[j][e] = __ballot(in[j] && use[ct][e] && !(d2[j][e] >= kNear * (nk[j] + ns[ct][e])));
                    cnt += (int)__popcll(near[j][e]);
                }
            }
            if (ct == 0 && cnt > kMany * min(m, 16)) {
                far = false;
                break;
            }
            // (the sums already hold the first 16 rows' part of this turn: it is finished, the next ones are not begun)
            if (ct > 0 && cnt > kMany * min(m - 16, 16)) last = true;
            for (int first = 0; first < cnt; first += kPairs) {     // the list, as often as it takes (once for 16 rows: kMany * 16 pairs)
                int at = -first;
#pragma unroll
                for (int j = 0; j < KT; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const unsigned long long n = near[j][e];
                        if (n == 0ull) continue;
                        const int w = at + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(n >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)n, 0u));
                        if ((n >> lane & 1) && (CT == 1 || (w >= 0 && w < kPairs)))
                            list[wave][w] = (unsigned)(j * 16 + c) << 8 | (unsigned)(16 * ct + 4 * q + e);
                        at += (int)__popcll(n);
                    }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                const int some = CT == 1 ? cnt : min(cnt - first, kPairs);
                for (int i = 0; i < some; i += GRP) {
                    const int w = min(i + grp, some - 1), r = (int)(list[wave][w] & 0xFFu);
                    float x[8], acc = 0.0f;
                    widen16<true>(*reinterpret_cast<const uint4 *>(
                                      Kh + (size_t)min(b0 + (int)(list[wave][w] >> 8), hi - 1) * D + part * 8), x);
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float t = x[e] - nr[r][part * 8 + e];
                        acc = fmaf(t, t, acc);
                    }
                    acc = lane_group_sum<LPR>(acc);
                    if (part == 0 && i + grp < some) res[wave][w] = acc;
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                at = -first;
#pragma unroll
                for (int j = 0; j < KT; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const unsigned long long n = near[j][e];
                        if (n == 0ull) continue;
                        const int w = at + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(n >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)n, 0u));
                        if ((n >> lane & 1) && (CT == 1 || (w >= 0 && w < kPairs))) d2[j][e] = res[wave][w];
                        at += (int)__popcll(n);
                    }
            }
#pragma unroll
            for (int j = 0; j < KT; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    d2[j][e] = in[j] && use[ct][e] ? __builtin_amdgcn_exp2f(-d2[j][e] * s2) : 0.0f;
                    add[j] += d2[j][e];
                }
            if (tail) {
#pragma unroll
                for (int j = 0; j < KT; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (in[j] && b0 + j * 16 + c - Lold == 16 * ct + 4 * q + e) d2[j][e] -= 1.0f;
            }
#pragma unroll
            for (int j = 0; j < KT; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) col[ct][e] += d2[j][e];
        }
        if (!far) break;
#pragma unroll
        for (int j = 0; j < KT; ++j) {
            const float t = quad_sum(add[j]);
            if (q == 0 && in[j]) added[b0 + j * 16 + c - lo] = t;
        }
        if (last) {
            b0 += 4 * KB;
            break;
        }
    }
    // direct differences, a lane group per key, eight keys in flight (at d = 64 those of two turns)
    constexpr int UN = 8, TURNS = UN * GRP / KB;
    for (; b0 < hi; b0 += TURNS * 4 * KB) {
        const bool tail = b0 + (TURNS - 1) * 4 * KB + KB > Lold;
        float x[UN][8];
        auto key = [&](int u) { return b0 + u * GRP / KB * 4 * KB + u * GRP % KB + grp; };
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(Kh + (size_t)min(key(u), hi - 1) * D + part * 8));
            widen16<true>(make_uint4(v.x, v.y, v.z, v.w), x[u]);
        }
        const int mine = key(part / (LPR / UN));
        float add = 0.0f;
        for (int r = 0; r < m; ++r) {
            float y[8], w[UN];
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] = nr[r][part * 8 + e];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                w[u] = 0.0f;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float df = x[u][e] - y[e];
                    w[u] = fmaf(df, df, w[u]);
                }
            }
            float one = group_scatter<LPR, UN>(w, part);
            one = mine < hi ? __builtin_amdgcn_exp2f(-one * s2) : 0.0f;
            add += one;
            if (tail && mine < hi && mine - Lold == r) one -= 1.0f;
            if (part % (LPR / UN) != 0) one = 0.0f;         // each key once
            one = lane_group_sum<LPR>(one);
            if (part == 0) cd[r][wave * GRP + grp] += one;      // slot private to this row group
        }
        if (mine < hi && part % (LPR / UN) == 0) added[mine - lo] = add;
    }
    // column sums: the 16 keys of a tile share a row of lanes
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float t = lane_group_sum<16>(col[ct][e]);
            if (c == 0) cs[wave][16 * ct + 4 * q + e] = t;
        }
    __syncthreads();
    // the old keys' refreshed densities, a whole tile at a time: consecutive threads, consecutive keys
    for (int i = lo + tid; i < min(hi, Lold); i += 256)
        rho_new[(size_t)h * L + i] = (rho_old[(size_t)h * Lold + i] * (float)Lold + added[i - lo]) / (float)L;
    if (tid < m) {
        float t = (cs[0][tid] + cs[1][tid]) + (cs[2][tid] + cs[3][tid]);
        for (int g = 0; g < 4 * GRP; ++g) t += cd[tid][g];
        colpart[((size_t)blockIdx.y * nblk + blk) * kAppMaxM + tid] = t;
    }
}

__global__ void __launch_bounds__(64)
append_finish(const float *__restrict__ colpart, float *__restrict__ rho_new, int head0, int L, int m, int nblk, float own)
{
    const int r = threadIdx.x;
    if (r >= m) return;
    double t = own;         // up to thousands of partials, in turn
    for (int b = 0; b < nblk; ++b) t += (double)colpart[((size_t)blockIdx.x * nblk + b) * kAppMaxM + r];
    rho_new[(size_t)(head0 + blockIdx.x) * L + (L - m) + r] = (float)(t / (double)L);
}

template <bool BF16, int D>
void run_chunk(const void *K, const float *rho_old, float *rho_new, float *colpart, const AppScale &sc, int head0,
               int nh, int L, int m, int nblk, hipStream_t st)
{
    bool gram = false;
    if constexpr (BF16) {
        gram = m >= (D == 64 ? kGramRows64 : kGramRows128);
        const uint16_t *Kb = reinterpret_cast<const uint16_t *>(K);
        if (gram && m <= 16)
            hipLaunchKernelGGL((append_gram<D, 1>), dim3(nblk, nh), dim3(256), 0, st, Kb, rho_old, rho_new, colpart, sc, head0, L, m, nblk);
        else if (gram)
            hipLaunchKernelGGL((append_gram<D, 2>), dim3(nblk, nh), dim3(256), 0, st, Kb, rho_old, rho_new, colpart, sc, head0, L, m, nblk);
    }
    if (!gram)
        hipLaunchKernelGGL((append_sweep<BF16, D>), dim3(nblk, nh), dim3(256), 0, st, K, rho_old, rho_new, colpart, sc,
                           head0, L, m, nblk);
    hipLaunchKernelGGL(append_finish, dim3(nh), dim3(64), 0, st, colpart, rho_new, head0, L, m, nblk, gram ? 1.0f : 0.0f);
}

}  // namespace

int append_max_rows() { return kAppMaxM; }

size_t append_workspace_bytes(int H, int L)
{
    const int nblk = (L + kAppTile - 1) / kAppTile;
    const int nh = H < kAppChunk ? H : kAppChunk;
    return round_up((size_t)nh * nblk * kAppMaxM * sizeof(float), 256);
}

hipError_t launch_density_append(const void *K, bool bf16, int H, int L, int d, int m, const float *sigma_host,
                                 const float *rho_old, float *rho_new, void *ws, hipStream_t st)
{
    const int nblk = (L + kAppTile - 1) / kAppTile;
    float *colpart = reinterpret_cast<float *>(ws);
    for (int h0 = 0; h0 < H; h0 += kAppChunk) {
        const int nh = (H - h0 < kAppChunk) ? H - h0 : kAppChunk;
        AppScale sc;
        for (int i = 0; i < kAppChunk; ++i) {
            const double sg = (i < nh) ? (double)sigma_host[h0 + i] : 1.0;
            sc.s[i] = (float)(0.5 * 1.4426950408889634 / (sg * sg));
        }
        // the chunks share the partial-sum array: they run in order on the one stream
        if (bf16) {
            if (d == 64) run_chunk<true, 64>(K, rho_old, rho_new, colpart, sc, h0, nh, L, m, nblk, st);
            else run_chunk<true, 128>(K, rho_old, rho_new, colpart, sc, h0, nh, L, m, nblk, st);
        } else {
            if (d == 64) run_chunk<false, 64>(K, rho_old, rho_new, colpart, sc, h0, nh, L, m, nblk, st);
            else run_chunk<false, 128>(K, rho_old, rho_new, colpart, sc, h0, nh, L, m, nblk, st);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace ws
