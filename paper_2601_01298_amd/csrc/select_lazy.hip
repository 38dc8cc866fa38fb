// Greedy landmark selection that evaluates only the keys a step can depend on (Warp-Cortex Sec. 3.3).
//
// A key's distance to the nearest landmark only falls as landmarks are added, and its score rises with that distance, so a
// value computed some steps ago is an upper bound of the value now, in fp32 as well (the same operations on a smaller
// operand).  A step needs two maxima, D_max and then the best score.  Both are found by looking again only at the keys whose
// bound still reaches the best value found so far: the result is the one a sweep over all keys gives, bit for bit.
//
// One workgroup per head, and no wait on another one.  The head's keys are cut into groups of 64 consecutive ones with a record
// each in LDS: the largest D in the group, the largest score, the D_max that score was formed with, and how many landmarks both
// take account of.  D itself and the keys' norms lie in memory.  A round: the groups whose bounds reach what is known (or, when
// a step starts, expected) of the maxima go into a queue, the waves VISIT them, i.e. bring them up to date, and the maxima of
// the records meet in LDS.  A step takes one round where D_max holds, three and more where it falls.
//
// A visit: the group's rows come in MFMA operand layout, the landmarks since its last visit are screened against its 64 keys on
// the matrix cores, 16 at a time (|k|^2 + |s|^2 - 2 k.s with a bound on its error; heads whose norms are out of its range are marked
// and left to the streaming kernel, launched behind this one), and per key the nearest of those that may
// lower its D is evaluated by direct differences in fp32 (others only where the screen cannot tell them apart).  fp32 keys are
// measured from a mean of theirs and rounded to bf16 for the screen (the error bound is wider), never for the evaluation.
//
// What bounds it: the chain of a step (median 9 000 cycles with four groups visited, d = 64; queue, rows, update, score, three
// barriers), and the first steps and those where D_max falls, in which hundreds of groups contend.  A visit is some 800 vector
// instructions.  384 heads of 32768 keys (d = 64, 655 picks): 32.8 ms with the keys on chip, twelve rounds of 32 heads; 16.2 here, all
// heads at once.  Tried: a visit per wave and round to groups of its own (20-25 ms: the slowest wave held the others up), every
// passing pair evaluated (x 1.3), records in registers, the next group's rows asked for ahead (no gain), visits of four tiles.
#include "ws_internal.h"

namespace ws {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2v_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2_t;

constexpr int kGroup = kLazyGroup;      // keys per group
constexpr int kTile = 16;               // landmarks per screening tile
constexpr int kGone = (int)0xBF800000;  // the bits of -1: a chosen key, a key past the end; below every value that counts
constexpr float kGuess = 4.0f;          // mean falls of the best score from step to step that a step's expectation allows for
constexpr int kVisit = 16;              // tiles of landmarks a visit looks at at most: what they lower is often enough
// Rounds of a step after which it is taken to be one in which D_max falls far.  384 heads of 32768 heavy-tailed keys (d = 64) with 1, 2
// and 4: 15.1, 15.3, 15.7 ms, 16.6 with one group per wave and round throughout; 96 of 131072 with far points 42.8, 44.2, 45.1, 48.7;
// clustered clouds the same within 2 %.
constexpr int kPatience = 1;
constexpr float kNever = -3.0e38f;
constexpr float kHuge = 1.0e37f;        // squared norms the screen can do with: products, sums and distances stay in range
constexpr float kTiny = 1.0e-30f;       // the screen's products may lose what lies below 1e-38: rows that small are always evaluated

struct LazyArgs {
    const void *K;
    const float *rho;
    int32_t *idx;
    float *score_out;
    float *slab;          // per workgroup: D^2, the scaled norms, (1 - alpha) u, Lpad floats each
    int *fail;
    int H, L, k, Lpad;
    int ring;             // newest landmark rows kept in LDS, a power of two of at least a tile
    float alpha;
};

// ---- reductions on the bit patterns of floats, ordered as signed integers --------------------------------------------------
template <int CTRL>
__device__ __forceinline__ int dpp_imax(int v)
{
    return max(v, __builtin_amdgcn_update_dpp((int)0x80000000, v, CTRL, 0xF, 0xF, false));
}

__device__ __forceinline__ int row_imax(int v)      // over the 16 lanes of a row, in all of them
{
    v = dpp_imax<0xB1>(v);
    v = dpp_imax<0x4E>(v);
    v = dpp_imax<0x141>(v);
    return dpp_imax<0x140>(v);
}

__device__ __forceinline__ int wave_imax(int v)
{
    v = row_imax(v);
    const int a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 16);
    const int c = __builtin_amdgcn_readlane(v, 32), d = __builtin_amdgcn_readlane(v, 48);
    return max(max(a, b), max(c, d));
}

// the four lanes that share a key (16 apart): sum, and maximum
__device__ __forceinline__ float quad_sum(float v)
{
    const u32x2_t a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a.x) + __uint_as_float(a.y);
    const u32x2_t b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(b.x) + __uint_as_float(b.y);
}

__device__ __forceinline__ float quad_max(float v)
{
    const u32x2_t a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a.x), __uint_as_float(a.y));
    const u32x2_t b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b.x), __uint_as_float(b.y));
}

__device__ __forceinline__ int quad_imax(int v)
{
    const u32x2_t a = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    v = max((int)a.x, (int)a.y);
    const u32x2_t b = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    return max((int)b.x, (int)b.y);
}

// Workgroup barrier that waits for this wave's LDS operations only: nothing is handed from wave to wave through memory, and
// rows asked for ahead of time stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---- eight elements of a row -----------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t pack2(float a, float b)
{
    bf16x2v_t p;
    p.x = (__bf16)a;
    p.y = (__bf16)b;
    return __builtin_bit_cast(uint32_t, p);
}

template <typename T> struct Eight;
template <> struct Eight<uint16_t> {
    // |error| of the screened squared distance <= kSlack * (|k|^2 + |s|^2): products of bf16 numbers are exact, sums of 128 of
    // them in fp32 stay within 2^-16 of |k||s|, the norms within that of theirs
    static constexpr float kSlack = 3.2e-5f;
    uint4 q;
    __device__ __forceinline__ void load(const uint16_t *p) { q = *reinterpret_cast<const uint4 *>(p); }
    __device__ __forceinline__ uint4 screen() const { return q; }
    __device__ __forceinline__ void from(const float *, int) {}      // (the screen is as exact as it has to be)
    __device__ __forceinline__ void widen(float (&f)[8]) const
    {
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            f[2 * j] = __uint_as_float(w[j] << 16);
            f[2 * j + 1] = __uint_as_float(w[j] & 0xFFFF0000u);
        }
    }
};
template <> struct Eight<float> {
    // both rows, as measured from a point c amid the keys, rounded to bf16 (2^-8 of an element each; a difference to c loses 2^-24 of
    // itself): 2 |k-c||s-c| (2^-7 + 2^-16) at most, and the sums
    static constexpr float kSlack = 8.0e-3f;
    float4 a, b;
    __device__ __forceinline__ void load(const float *p)
    {
        a = *reinterpret_cast<const float4 *>(p);
        b = *reinterpret_cast<const float4 *>(p + 4);
    }
    __device__ __forceinline__ uint4 screen() const
    {
        return make_uint4(pack2(a.x, a.y), pack2(a.z, a.w), pack2(b.x, b.y), pack2(b.z, b.w));
    }
    __device__ __forceinline__ void from(const float *centre, int at)
    {
        // (read where it is used, behind the row: kept or fetched ahead it takes registers there are not)
        asm volatile("" : "+v"(at), "+v"(b.w));
        const float *c = centre + at;
        const float4 u = *reinterpret_cast<const float4 *>(c), v = *reinterpret_cast<const float4 *>(c + 4);
        a = make_float4(a.x - u.x, a.y - u.y, a.z - u.z, a.w - u.w);
        b = make_float4(b.x - v.x, b.y - v.y, b.z - v.z, b.w - v.w);
    }
    __device__ __forceinline__ void widen(float (&f)[8]) const
    {
        f[0] = a.x;
        f[1] = a.y;
        f[2] = a.z;
        f[3] = a.w;
        f[4] = b.x;
        f[5] = b.y;
        f[6] = b.z;
        f[7] = b.w;
    }
};

// sum of the squared differences; `held` elements live in registers across the caller's loop: their widening stays inside it
// (the shift passes through an empty statement), or the widened rows would take the registers
__device__ __forceinline__ float diff2_held(const uint4 &held, const Eight<uint16_t> &y)
{
    unsigned sh = 16, hi = 0xFFFF0000u;
    asm volatile("" : "+s"(sh), "+s"(hi));
    const uint32_t w[4] = {held.x, held.y, held.z, held.w};
    float g[8];
    y.widen(g);
    float acc = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float t0 = __uint_as_float(w[j] << sh) - g[2 * j], t1 = __uint_as_float(w[j] & hi) - g[2 * j + 1];
        acc = fmaf(t0, t0, acc);
        acc = fmaf(t1, t1, acc);
    }
    return acc;
}

template <typename T>
__device__ __forceinline__ float diff2(const Eight<T> &x, const Eight<T> &y)
{
    float f[8], g[8];
    x.widen(f);
    y.widen(g);
    float acc = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float t = f[e] - g[e];
        acc = fmaf(t, t, acc);
    }
    return acc;
}

template <typename T>
__device__ __forceinline__ float square(const Eight<T> &x)
{
    float f[8];
    x.widen(f);
    float acc = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc = fmaf(f[e], f[e], acc);
    return acc;
}

// What a wave tells the others after a round (its groups: those whose records its lanes look after; its candidate: the best
// score among the visits it made).
//   a.x  largest D bound of its groups   a.y  the second largest   a.z  largest score bound of those not settled
//   a.w  bit 0: a.x is up to date; bits 1-15: its group; bits 16-: the lowest group that has a.z
//   b.x  candidate's score   b.y  its key   b.z, b.w  largest D and score of the candidate's group without it
struct Post {
    int4 a, b;
};

constexpr int kQueue = 256;         // groups a round visits at most (the others stay for the next)

template <int D, int NW, int SLOTS>
struct LazyShared {
    int4 meta[NW * 64 * SLOTS];     // per group: D bound, score bound, D_max it was scored with, landmarks it has seen
    uint4 cand[NW][D / 8];          // row of each wave's candidate, as the screen sees it
    Post post[2][NW];               // by turns: a round that compares bounds only has no barrier before it posts
    unsigned queue[kQueue];         // groups to visit, and the landmarks they have seen
    int qn[2], qh[2];               // entries, entries taken
    int red[NW], red2[NW];
    float part[NW][64];             // fp32 keys: sums of sampled rows
    float centre[D];                // and their mean, from which the screen measures
};

template <typename T, int D, int NW, int SLOTS, int OCC>
__global__ void __launch_bounds__(NW * 64, OCC)
select_lazy(LazyArgs a)
{
    // Groups a wave asks for in the first round of a step, the foremost of those that reach what is expected of it: where scores tie or
    // fall unevenly that may be all of them, and one round tells which matter.  384 heads of 32768 keys, d = 64, with 2, 4, 8, 256:
    // clustered 16.6, 16.2, 16.1, 16.6 ms, heavy tails 15.5, 15.1, 15.1, 15.1 and at alpha = 0 14.9, 13.2, 19.7, 53.0, 200 points in 164
    // copies each 80.9, 76.9, 87.7, 152; four records per lane (96 heads of 131072) 40.3, 37.0, 34.8, 33.8.
    constexpr int kFirst = SLOTS == 1 ? 4 : 8;
    constexpr int PJ = OCC == 4 ? 1 : 2;            // key tiles evaluated side by side, where the registers allow
    constexpr int KS = D / 32;                      // MFMA k-steps, and 16-byte pieces of the screen per lane and key
    constexpr int NP = D / 8;                       // pieces per row
    extern __shared__ __align__(16) char smem[];
    LazyShared<D, NW, SLOTS> &sh = *reinterpret_cast<LazyShared<D, NW, SLOTS> *>(smem);
    const int kpad = (a.k + kTile - 1) & ~(kTile - 1);
    float *lmC = reinterpret_cast<float *>(smem + sizeof(LazyShared<D, NW, SLOTS>));     // -|s|^2 (1 - slack) / 2 per landmark
    int *lmI = reinterpret_cast<int *>(lmC + kpad);                                  // its index
    uint4 *ring = reinterpret_cast<uint4 *>(lmI + kpad);    // the newest rows as the screen sees them, pieces swizzled by row
    const int rmask = a.ring - 1, rtiles = a.ring / kTile;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, q = lane >> 4;         // key (or landmark) of a tile of 16, and which pieces of its row
    const int L = a.L, k = a.k, nG = (L + kGroup - 1) / kGroup;
    const float alpha = a.alpha, oma = 1.0f - a.alpha;
    const bool flat = alpha == 0.0f;                // distances count for nothing: D and D_max stay what they are at first
    constexpr float kHalf = 0.5f * (1.0f - Eight<T>::kSlack);
    float *Ds = a.slab + (size_t)blockIdx.x * 3 * a.Lpad, *Ns = Ds + a.Lpad, *Us = Ns + a.Lpad;

    for (int h = blockIdx.x; h < a.H; h += gridDim.x) {
        const T *Kh = reinterpret_cast<const T *>(a.K) + (size_t)h * L * D;
        const float *rhoh = a.rho + (size_t)h * L;

        // ---- u_i = rho_min / rho_i; the first landmark
        float rmin = __builtin_inff();
        for (int i = tid; i < L; i += NW * 64) rmin = fminf(rmin, rhoh[i]);
        {
            const int m = wave_imax(~__float_as_int(rmin));     // min over positive floats
            __syncthreads();
            if (lane == 0) sh.red[wave] = m;
            __syncthreads();
            int mm = sh.red[0];
#pragma unroll
            for (int w = 1; w < NW; ++w) mm = max(mm, sh.red[w]);
            rmin = __int_as_float(~mm);
            __syncthreads();
        }
        int pick = 0;
        float pscore = alpha;
        if (alpha != 1.0f) {
            int bs = kGone, bi = 0;
            for (int i = tid; i < L; i += NW * 64) {
                const int v = __float_as_int(alpha * 1.0f + oma * (rmin / rhoh[i]));
                if (v > bs) {
                    bs = v;
                    bi = i;
                }
            }
            const int m = wave_imax(bs);
            const int mi = ~wave_imax(bs == m ? ~bi : (int)0x80000000);
            if (lane == 0) {
                sh.red[wave] = m;
                sh.red2[wave] = mi;
            }
            __syncthreads();
            int best = sh.red[0];
            pick = sh.red2[0];
#pragma unroll
            for (int w = 1; w < NW; ++w) {
                const int s = sh.red[w], i = sh.red2[w];
                if (s > best || (s == best && i < pick)) {
                    best = s;
                    pick = i;
                }
            }
            pick = __builtin_amdgcn_readfirstlane(min(max(pick, 0), L - 1));
            pscore = __int_as_float(best);
            __syncthreads();
        }
        if (tid == 0) {
            a.idx[(size_t)h * k] = pick;
            if (a.score_out) a.score_out[(size_t)h * k] = pscore;
        }
        if (k == 1) continue;

        // ---- landmark 0 into the ring (the rows beside it in its tile take part in the screen, unused), and every key's
        // distance to it
        for (int i = tid; i < a.ring * NP; i += NW * 64) ring[i] = make_uint4(0u, 0u, 0u, 0u);
        if constexpr (sizeof(T) == 4) {
            // 64 rows, evenly spaced: a few far ones among them shift the mean by a small part of their distance
            constexpr int RW = NW * 64 / D;         // rows side by side
            const int e = tid % D, r0 = tid / D;
            float sum = 0.0f;
#pragma unroll
            for (int r = 0; r < 64; r += RW) sum += (float)Kh[(size_t)((long long)(r + r0) * L >> 6) * D + e];
            (&sh.part[0][0])[tid] = sum;
            __syncthreads();
            if (tid < D) {
                sum = 0.0f;
#pragma unroll
                for (int r = 0; r < RW; ++r) sum += (&sh.part[0][0])[r * D + tid];
                sh.centre[tid] = sum * (1.0f / 64.0f);
            }
        }
        __syncthreads();
        if (wave == 0 && lane < NP) {
            Eight<T> x;
            x.load(Kh + (size_t)pick * D + lane * 8);
            x.from(sh.centre, lane * 8);
            ring[lane] = x.screen();
            float n = square(x);
            n = lane_group_sum<NP>(n);
            if (lane == 0) {
                lmC[0] = -n * kHalf;
                lmI[0] = pick;
            }
        }
        // the records of this wave's groups: (r * 64 + lane) * NW + wave
        int4 *mine = sh.meta + wave * 64 * SLOTS;
        auto place = [&](int g) -> int { return (g % NW) * 64 * SLOTS + g / NW; };
#pragma unroll
        for (int r = 0; r < SLOTS; ++r) mine[r * 64 + lane] = make_int4(kGone, kGone, 0x7f800000, 0x7fffffff);
        int dall = kGone;
        bool big = false;
        {
            Eight<T> m0[KS];
#pragma unroll
            for (int s = 0; s < KS; ++s) m0[s].load(Kh + (size_t)pick * D + (s * 4 + q) * 8);
#pragma unroll
            for (int r = 0; r < SLOTS; ++r) {
                for (int l = 0; l < 64; ++l) {
                    const int g = (r * 64 + l) * NW + wave;
                    if (g >= nG) break;
                    float Dl = 0.0f, Nl = 0.0f;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const T *row = Kh + (size_t)min(g * kGroup + j * 16 + c, L - 1) * D;
                        float dd = 0.0f, nn = 0.0f;
                        Eight<T> x[KS];
#pragma unroll
                        for (int s = 0; s < KS; ++s) x[s].load(row + (s * 4 + q) * 8);
#pragma unroll
                        for (int s = 0; s < KS; ++s) {
                            if constexpr (sizeof(T) == 2) dd += diff2_held(m0[s].q, x[s]);
                            else dd += diff2(x[s], m0[s]);
                            x[s].from(sh.centre, (s * 4 + q) * 8);
                            nn += square(x[s]);
                        }
                        dd = quad_sum(dd);
                        nn = quad_sum(nn);
                        big = big || !(nn < kHuge);
                        Dl = q == j ? dd : Dl;
                        Nl = q == j ? nn * kHalf - kTiny : Nl;
                    }
                    const int i = g * kGroup + lane;
                    const float u = rmin / rhoh[min(i, L - 1)];
                    const bool in = i < L && i != pick;
                    Dl = in ? fminf(__builtin_inff(), Dl) : __int_as_float(kGone);
                    Ds[i] = Dl;
                    Ns[i] = Nl;
                    Us[i] = oma * u;
                    const int gd = wave_imax(in ? __float_as_int(__fsqrt_rn(Dl)) : kGone);
                    const int gs = wave_imax(in ? __float_as_int(oma * u) : kGone);
                    if (lane == l) mine[r * 64 + l] = make_int4(gd, gs, 0x7f800000, 1);
                    dall = max(dall, gd);
                }
            }
        }
        for (int i = tid; i < kpad; i += NW * 64)
            if (i > 0) lmC[i] = kNever;             // landmarks to come never pass the screen
        if (tid < 2) sh.qn[tid] = sh.qh[tid] = 0;
        float dm;
        {
            const int any = __ballot(big) != 0ull;
            if (lane == 0) {
                sh.red[wave] = dall;
                sh.red2[wave] = any;
            }
            __syncthreads();
            int mm = sh.red[0], out = sh.red2[0];
#pragma unroll
            for (int w = 1; w < NW; ++w) {
                mm = max(mm, sh.red[w]);
                out |= sh.red2[w];
            }
            dm = __int_as_float(__builtin_amdgcn_readfirstlane(mm));
            if (__builtin_amdgcn_readfirstlane(out) != 0) {     // (or no number at all): left to the kernel behind this one
                if (tid == 0) a.idx[(size_t)h * k] = kSelectLeft;
                continue;
            }
        }

        // the group whose keys this wave holds
        int cg = -1;
        uint4 kv[4][KS];            // rows g*64 + 16j + c, pieces s*4 + q, as the screen sees them
        float Dt[4], hk[4];         // their squared D and scaled norms, the same in the four lanes of a key
        float ul = 0.0f;            // (1 - alpha) u of key g*64 + lane

        // (the D of a group: another wave may have lowered it since; its keys stay)
        auto hold = [&](int g) {
            const unsigned base = (unsigned)g * kGroup;
#pragma unroll
            for (int j = 0; j < 4; ++j) Dt[j] = Ds[base + j * 16 + c];
            if (g == cg) return;
            cg = g;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const unsigned at = (min(base + j * 16 + c, (unsigned)L - 1) * D + q * 8) * (unsigned)sizeof(T);
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    Eight<T> x;
                    x.load(reinterpret_cast<const T *>(reinterpret_cast<const char *>(Kh) + at) + s * 32);
                    x.from(sh.centre, (s * 4 + q) * 8);
                    kv[j][s] = x.screen();
                }
                hk[j] = Ns[base + j * 16 + c];
            }
            ul = Us[base + lane];
        };
        // landmarks 16b + c as the screen's other operand, and what the accumulator starts at: the part that does not depend
        // on the key (a value that never passes for landmarks before t0, which the group has seen)
        auto tile_operand = [&](int b, int bT, int t0, uint4 (&mv)[KS]) -> f32x4_t {
            if (b > bT - rtiles) {
                const int row = (b * kTile + c) & rmask;
#pragma unroll
                for (int s = 0; s < KS; ++s) mv[s] = ring[row * NP + ((s * 4 + q) ^ (row & (NP - 1)))];
            } else {
                const T *row = Kh + (size_t)lmI[b * kTile + c] * D;
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    Eight<T> x;
                    x.load(row + (s * 4 + q) * 8);
                    x.from(sh.centre, (s * 4 + q) * 8);
                    mv[s] = x.screen();
                }
            }
            f32x4_t cc = *reinterpret_cast<const f32x4_t *>(&lmC[b * kTile + q * 4]);
            if (b * kTile < t0) {
#pragma unroll
                for (int r = 0; r < 4; ++r) cc[r] = b * kTile + q * 4 + r >= t0 ? cc[r] : kNever;
            }
            return cc;
        };
        auto dots = [&](const uint4 (&mv)[KS], const uint4 (&kj)[KS], f32x4_t acc) -> f32x4_t {
#pragma unroll
            for (int s = 0; s < KS; ++s)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, mv[s]), __builtin_bit_cast(bf16x8_t, kj[s]),
                                                              acc, 0, 0, 0);
            return acc;
        };
        auto dots4 = [&](const uint4 (&mv)[KS], const f32x4_t &cc, f32x4_t (&acc)[4]) {
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, mv[s]),
                                                                     __builtin_bit_cast(bf16x8_t, kv[j][s]), s ? acc[j] : cc, 0, 0, 0);
        };
        // k.s - |s|^2/2 (1 - slack) above (|k|^2 (1 - slack) - D^2) / 2: the pair may lower D
        auto limit = [&](int j) -> float { return Dt[j] >= 0.0f ? fmaf(-0.5f, Dt[j], hk[j]) : __builtin_inff(); };
        auto passes = [&](const f32x4_t &acc, float thr) -> unsigned long long {
            return __ballot(acc[0] > thr) | __ballot(acc[1] > thr) | __ballot(acc[2] > thr) | __ballot(acc[3] > thr);
        };
        auto landmark = [&](int m, bool inring, Eight<T> (&x)[KS]) {
            if constexpr (sizeof(T) == 2) {
                if (inring) {
                    const int row = m & rmask;
#pragma unroll
                    for (int s = 0; s < KS; ++s) x[s].q = ring[row * NP + ((s * 4 + q) ^ (row & (NP - 1)))];
                    return;
                }
            }
            const T *row = Kh + (size_t)lmI[m] * D;
#pragma unroll
            for (int s = 0; s < KS; ++s) x[s].load(row + (s * 4 + q) * 8);
        };
        auto exact = [&](int j, const Eight<T> (&x)[KS]) -> float {
            float dd = 0.0f;
            if constexpr (sizeof(T) == 2) {
#pragma unroll
                for (int s = 0; s < KS; ++s) dd += diff2_held(kv[j][s], x[s]);
            } else {
                const T *key = Kh + (size_t)min(cg * kGroup + j * 16 + c, L - 1) * D;
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    Eight<T> y;
                    y.load(key + (s * 4 + q) * 8);
                    dd += diff2(y, x[s]);
                }
            }
            return quad_sum(dd);
        };
        // D of the held keys brought up to date with landmarks t0 ... t1-1 (t there are); true if any may have fallen
        auto update = [&](int t0, int t1, int t) -> bool {
            const int bT = (t - 1) / kTile, b0 = t0 / kTile, b1 = (t1 - 1) / kTile;
            float thr[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) thr[j] = limit(j);
            bool moved = false;
            uint4 mv[KS];
            f32x4_t cc = tile_operand(b0, bT, t0, mv), acc[4];
            if (t0 == t - 1) {
                // one landmark: evaluated against all keys of a pair of tiles in which the screen lets one pass
                Eight<T> x[KS];
                landmark(t0, true, x);
                dots4(mv, cc, acc);
#pragma unroll
                for (int j = 0; j < 4; j += PJ) {
                    unsigned long long some = 0ull;
#pragma unroll
                    for (int i = 0; i < PJ; ++i) some |= passes(acc[j + i], thr[j + i]);
                    if (some == 0ull) continue;
                    moved = true;
                    float dd[PJ];
#pragma unroll
                    for (int i = 0; i < PJ; ++i) dd[i] = exact(j + i, x);
#pragma unroll
                    for (int i = 0; i < PJ; ++i) Dt[j + i] = fminf(Dt[j + i], dd[i]);
                }
                return moved;
            }
            // several: per key the best and the second best value of the screen over all of them ...
            float best[4], sec[4];
            int bid[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                best[j] = sec[j] = -__builtin_inff();
                bid[j] = 0;
            }
            for (int b = b0; b <= b1; ++b) {
                dots4(mv, cc, acc);
                if (b < b1) cc = tile_operand(b + 1, bT, t0, mv);
                float old[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) old[j] = best[j];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        // (the row's number in the two lowest bits; med3 of a pair and an infinity: the larger)
                        const float v = __int_as_float((__float_as_int(acc[j][e]) & ~3) | e);
                        sec[j] = __builtin_amdgcn_fmed3f(best[j], sec[j], v);
                        best[j] = __builtin_amdgcn_fmed3f(best[j], v, __builtin_inff());
                    }
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) bid[j] = best[j] > old[j] ? b : bid[j];
            }
            // ... then the best one's landmark exactly, and the others only where the second best might still be nearer
            const int rs = kTile * (bT - rtiles + 1);        // landmarks from here on are in the ring
#pragma unroll
            for (int j = 0; j < 4; j += PJ) {
                unsigned long long some = 0ull;
#pragma unroll
                for (int i = 0; i < PJ; ++i) some |= __ballot(best[j + i] > thr[j + i]);
                if (some == 0ull) continue;
                moved = true;
                int id[PJ], m[PJ], ml = 0x7fffffff;
                Eight<T> x[PJ][KS];
#pragma unroll
                for (int i = 0; i < PJ; ++i) {
                    const float vm = quad_max(best[j + i]);
                    id[i] = bid[j + i] * kTile + q * 4 + (__float_as_int(best[j + i]) & 3);
                    m[i] = min(quad_imax(best[j + i] == vm ? id[i] : 0), t1 - 1);
                    ml = min(ml, m[i]);
                }
                const bool in = __ballot(ml < rs) == 0ull;
                float dd[PJ];
#pragma unroll
                for (int i = 0; i < PJ; ++i) landmark(m[i], in, x[i]);
#pragma unroll
                for (int i = 0; i < PJ; ++i) dd[i] = exact(j + i, x[i]);
#pragma unroll
                for (int i = 0; i < PJ; ++i) Dt[j + i] = fminf(Dt[j + i], dd[i]);
#pragma unroll
                for (int i = 0; i < PJ; ++i) {
                    if (__ballot((id[i] == m[i] ? sec[j + i] : best[j + i]) > limit(j + i)) == 0ull) continue;
                    for (int b = b0; b <= b1; ++b) {
                        cc = tile_operand(b, bT, t0, mv);
                        f32x4_t a1 = dots(mv, kv[j + i], cc);
#pragma unroll
                        for (int e = 0; e < 4; ++e) a1[e] = b * kTile + q * 4 + e == m[i] ? kNever : a1[e];
                        // (a settled pair per key and turn: sixteen turns at most, whatever the inputs hold)
                        for (int turn = 0; turn < kTile; ++turn) {
                            if (passes(a1, limit(j + i)) == 0ull) break;
                            float v = -__builtin_inff();
                            int r = 0;
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (a1[e] > v) {
                                    v = a1[e];
                                    r = e;
                                }
                            const float vn = quad_max(v);
                            const int mr = quad_imax(v == vn ? q * 4 + r : 0), mt = min(b * kTile + mr, t1 - 1);
                            landmark(mt, b * kTile >= rs, x[0]);
                            // (an exact distance may go into any key's minimum; chosen keys stay at -1)
                            Dt[j + i] = fminf(Dt[j + i], exact(j + i, x[0]));
#pragma unroll
                            for (int e = 0; e < 4; ++e) a1[e] = mr == q * 4 + e ? kNever : a1[e];
                        }
                    }
                }
            }
            return moved;
        };

        constexpr unsigned long long kWaves = (1ull << NW) - 1;
        // score bound of a group under the D_max assumed now: scored with a larger one, alpha D / D_max has grown by no more
        // than this (rounding included)
        auto bound = [&](const int4 &m, float rdm) -> int {
            const float v = __int_as_float(m.z);
            if (m.y == kGone || v == dm || !(dm > 0.0f)) return m.y;
            const float add = alpha * __int_as_float(m.x) * fmaxf(0.0f, rdm - __builtin_amdgcn_rcpf(v));
            return __float_as_int((__int_as_float(m.y) + add) * 1.000004f);
        };
        // a step's best score is not known when it starts: groups are visited if their bound reaches what it is expected to
        // be, from the last one and the mean change of late (which decides only what is looked at first)
        float guess = 0.0f, change = 0.02f, lastS = 0.0f;
        int par = 0, pickd = kGone, picks = kGone;      // par: which of the two queue counters; the rest: of the last pick's group
        int gI = 0, gfix = -1;                          // the pick; its group, until the record has been corrected
        int side = 0;                                   // which of the two sets of posts this round's go to

        for (int t = 1; t < k; ++t) {
            // t landmarks so far
            int cs = kGone, ci = 0, cd = kGone, cs2 = kGone;        // this wave's candidate
            int thr = __float_as_int(guess), dcut = flat ? 0x7fffffff : __float_as_int(dm);
            bool wantS = true, look = t > 1;            // look: visit groups in this round, or only compare bounds
            int far = kVisit * kTile;                   // landmarks a visit looks at at most
            int floorS = kGone;
            int tie = 0x7fffffff;               // groups before this one are looked at also where their bound equals thr
            int gS = kGone;
            for (int round = 0; gI >= 0; ++round) {
                const float rdm = __builtin_amdgcn_rcpf(dm);
                if (look) {
                    // ---- what to visit
                    int room = round == 0 ? kFirst : kQueue;
#pragma unroll
                    for (int r = 0; r < SLOTS; ++r) {
                        int4 m = mine[r * 64 + lane];
                        const int g = (r * 64 + lane) * NW + wave;
                        if (g == gfix) {
                            m.x = pickd;
                            m.y = picks;
                            mine[r * 64 + lane] = m;
                        }
                        const int ub = bound(m, rdm);
                        const bool fresh = m.w >= t, open = m.y > kGone && !(fresh && __int_as_float(m.z) == dm);
                        const bool go = (!fresh && m.x >= dcut && m.x > kGone) ||
                                        (wantS && open && (ub > thr || (ub == thr && g < tie)));
                        const unsigned long long bal = __ballot(go);
                        if (bal != 0ull) {
                            const int rank = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(bal >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0u));
                            const int cnt = min((int)__popcll(bal), room);
                            int at = 0;
                            if (lane == 0) at = atomicAdd(&sh.qn[par], cnt);
                            at = __builtin_amdgcn_readfirstlane(at) + rank;
                            if (go && rank < room && at < kQueue) sh.queue[at] = (unsigned)g | (unsigned)m.w << 16;
                            room -= cnt;
                        }
                    }
                    gfix = -1;
                    lds_barrier();
                    const int n = min(__builtin_amdgcn_readfirstlane(sh.qn[par]), kQueue);
                    if (tid < 1) sh.qn[par ^ 1] = sh.qh[par ^ 1] = 0;
                    // ---- the visits
                    int at = wave;
                    while (at < n) {
                        const unsigned ent = (unsigned)__builtin_amdgcn_readfirstlane((int)sh.queue[at]);
                        const int g = (int)(ent & 0xFFFFu), t0 = (int)(ent >> 16), base = g * kGroup;
                        int nx = 0;
                        if (lane == 0) nx = atomicAdd(&sh.qh[par], 1);
                        hold(g);
                        // (alpha = 0: no score depends on D, and D stays as it was at first)
                        const int t1 = flat ? t : min(t, t0 / kTile * kTile + far);
                        const bool moved = t0 < t && !flat && update(t0, t1, t);
                        const float D2 = q < 2 ? (q == 0 ? Dt[0] : Dt[1]) : (q == 2 ? Dt[2] : Dt[3]);
                        if (moved) Ds[base + lane] = D2;
                        const float Dl = __fsqrt_rn(D2), cov = dm > 0.0f ? Dl / dm : 0.0f;
                        const int db = D2 >= 0.0f ? __float_as_int(Dl) : kGone;
                        const int sb = D2 >= 0.0f ? __float_as_int(alpha * cov + ul) : kGone;
                        const int gd = wave_imax(db), gs = wave_imax(sb);
                        if (lane == 0) sh.meta[place(g)] = make_int4(gd, gs, __float_as_int(dm), t1);
                        const int cl = (int)__builtin_ctzll(__ballot(sb == gs));
                        if (t1 == t && (gs > cs || (gs == cs && base + cl < ci))) {
                            cs = gs;
                            ci = base + cl;
                            cd = __builtin_amdgcn_readlane(db, cl) == gd ? wave_imax(lane == cl ? kGone : db) : gd;
                            cs2 = wave_imax(lane == cl ? kGone : sb);
                            if (c == (cl & 15)) {
#pragma unroll
                                for (int j = 0; j < 4; ++j)
                                    if (j == cl >> 4) {
#pragma unroll
                                        for (int s = 0; s < KS; ++s) sh.cand[wave][s * 4 + q] = kv[j][s];
                                    }
                            }
                        }
                        at = NW + __builtin_amdgcn_readfirstlane(nx);
                    }
                    par ^= 1;
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // other waves may visit these groups next
                    lds_barrier();
                }
                // ---- tell the other waves (a wave may still read the last round's posts; it is past those of the round before,
                // or it had not come to the last round's barrier)
                int D1, N1;
                {
                    int d1 = kGone, d2 = kGone, g1 = 0, f1 = 0, n1 = kGone, gn = 0x7fff;
#pragma unroll
                    for (int r = 0; r < SLOTS; ++r) {
                        const int4 m = mine[r * 64 + lane];
                        const int g = (r * 64 + lane) * NW + wave;
                        const int ub = bound(m, rdm);
                        const bool fresh = m.w >= t, open = m.y > kGone && !(fresh && __int_as_float(m.z) == dm);
                        d2 = max(d2, min(d1, m.x));
                        if (m.x > d1) {
                            d1 = m.x;
                            g1 = g;
                            f1 = fresh ? 1 : 0;
                        }
                        if (open && ub > n1) {
                            n1 = ub;
                            gn = g;
                        }
                    }
                    D1 = wave_imax(d1);
                    N1 = wave_imax(n1);
                    const int dl = (int)__builtin_ctzll(__ballot(d1 == D1));
                    const int D2nd = wave_imax(lane == dl ? d2 : d1);
                    const int pk = __builtin_amdgcn_readlane(g1 << 1 | f1, dl);
                    int gl = 0x7fff;
                    if (N1 > kGone) gl = ~wave_imax(n1 == N1 ? ~gn : (int)0x80000000);
                    if (lane == 0) {
                        sh.post[side][wave].a = make_int4(D1, D2nd, N1, pk | gl << 16);
                        sh.post[side][wave].b = make_int4(cs, ci, cd, cs2);
                    }
                }
                lds_barrier();
                const int4 pa = sh.post[side][lane % NW].a, pb = sh.post[side][lane % NW].b;
                side ^= 1;
                const int gD = flat ? __float_as_int(dm) : __builtin_amdgcn_readfirstlane(row_imax(pa.x));
                const int gF = flat ? gD : __builtin_amdgcn_readfirstlane(row_imax((pa.w & 1) ? pa.x : kGone));
                const int gN = __builtin_amdgcn_readfirstlane(row_imax(pa.z));
                gS = __builtin_amdgcn_readfirstlane(row_imax(pb.x));
                const bool same = gD == __float_as_int(dm);
                const int key = ~__builtin_amdgcn_readfirstlane(row_imax(pb.x == gS ? ~pb.y : (int)0x80000000));
                bool done = same && gF >= gD && gS > kGone && gN <= gS;
                if (done && gN == gS)       // a tie: settled only if every key that could share the score comes later
                    done = ~__builtin_amdgcn_readfirstlane(row_imax(pa.z == gN ? ~(pa.w >> 16) : (int)0x80000000)) > key >> 6;
                if (done) {
                    gI = min(max(key, 0), L - 1);
                    const int ww = (int)__builtin_ctzll((__ballot(pb.x == gS && pb.y == gI) & kWaves) | (1ull << (NW - 1)));
                    gfix = gI >> 6;
                    pickd = __builtin_amdgcn_readlane(pb.z, ww);
                    picks = __builtin_amdgcn_readlane(pb.w, ww);
                    // what D_max is at most once the pick is gone
                    if (!flat)
                        dm = __int_as_float(max(pickd, __builtin_amdgcn_readfirstlane(
                                                           row_imax(((pa.w & 0xFFFF) >> 1) == gI >> 6 ? pa.y : pa.x))));
                    if (wave == ww) {
                        // the candidate's row joins the ring, its key leaves the race
                        const int row = t & rmask;
                        if (lane < NP) {
                            const uint4 w = sh.cand[wave][lane];
                            ring[row * NP + (lane ^ (row & (NP - 1)))] = w;
                            Eight<T> x;
                            if constexpr (sizeof(T) == 2) x.q = w;
                            else {
                                x.load(Kh + (size_t)gI * D + lane * 8);
                                x.from(sh.centre, lane * 8);
                            }
                            const float n = lane_group_sum<NP>(square(x));
                            if (lane == 0) {
                                lmC[t] = -n * kHalf;
                                lmI[t] = gI;
                            }
                        }
                        if (lane == 0) Ds[gI] = __int_as_float(kGone);
                        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    }
                    break;
                }
                // ---- not settled: what to visit next.  Every round that visits takes at least one group on by kVisit tiles, or forms its
                // score with the D_max that holds, so a step ends after far fewer rounds than this
                const bool settled = gF >= gD;
                if (round > 2 * nG * (t / (kVisit * kTile) + 4) + 64) {
                    if (tid == 0) *a.fail = 1;
                    gI = -1;        // what the head still owes is marked invalid
                    break;
                }
                if (gS > floorS) floorS = gS;       // (under a lower D_max a score only grows)
                wantS = settled;
                look = true;
                far = round >= kPatience && (settled ? gS : gF) == kGone ? kMaxLazyK : kVisit * kTile;     // nothing known yet: take one group all the way
                if (!settled) {
                    // each wave the group of its own that may have D_max; where that does not do, D_max has fallen far, and every
                    // group that may exceed what is known of it has to be looked at
                    dcut = round >= kPatience && gF > kGone ? gF + 1 : max(gF + 1, D1);
                } else {
                    dcut = 0x7fffffff;
                    // no score known yet: each wave the group of its own with the highest bound, formed with this D_max
                    thr = gS > kGone ? gS : max(floorS, N1);
                    tie = gS > kGone ? key >> 6 : 0x7fffffff;
                    if (!same) look = false;
                }
                if (!same) {
                    // D_max is lower than assumed: what was scored with the old one are bounds now
                    dm = __int_as_float(gD);
                    cs = kGone;
                }
            }
            if (tid == 0) {
                a.idx[(size_t)h * k + t] = gI;
                if (a.score_out) a.score_out[(size_t)h * k + t] = __int_as_float(gS);
            }
            // (a rise comes of a lower D_max and says nothing about the next step; of a sharp fall a part counts)
            const float sc = __int_as_float(gS), fell = lastS - sc;
            if (fell >= 0.0f) change = 0.8f * change + 0.2f * fminf(fell, 4.0f * change + 1.0e-3f);
            lastS = sc;
            guess = fmaxf(0.0f, sc - kGuess * change);
        }
        __syncthreads();
    }
}

template <typename T, int D, int NW, int SLOTS, int OCC>
hipError_t run(LazyArgs a, int groups, hipStream_t st)
{
    const int kpad = (a.k + kTile - 1) & ~(kTile - 1);
    const size_t fixed = sizeof(LazyShared<D, NW, SLOTS>) + (size_t)kpad * 8, room = OCC == 4 ? 80 * 1024 : 160 * 1024;
    a.ring = kTile;
    while (a.ring < kpad && fixed + (size_t)a.ring * 2 * D * 2 <= room) a.ring *= 2;
    const size_t lds = fixed + (size_t)a.ring * D * 2;
    if (lds > 64 * 1024) {      // has to be asked for (the call only sets a limit)
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(select_lazy<T, D, NW, SLOTS, OCC>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((select_lazy<T, D, NW, SLOTS, OCC>), dim3(groups), dim3(NW * 64), lds, st, a);
    return hipGetLastError();
}

template <typename T, int D>
hipError_t dispatch(const LazyArgs &a, const LazyShape &s, hipStream_t st)
{
    // two workgroups per compute unit: 128 registers, which is enough at d = 64 with bf16 keys only
    if constexpr (sizeof(T) == 2 && D == 64)
        if (s.per_cu == 2) return run<T, D, kLazyWaves, 1, 4>(a, s.groups, st);
    if constexpr (sizeof(T) == 2) {     // (fp32 heads of these lengths stay with the streaming kernel)
        if (s.slots == 2) return run<T, D, kLazyWaves, 2, 2>(a, s.groups, st);
        if (s.slots == 4) return run<T, D, kLazyWaves, 4, 2>(a, s.groups, st);
    }
    return run<T, D, kLazyWaves, 1, 2>(a, s.groups, st);
}

}  // namespace

// When it is taken.  `other_us`: what the kernel that would run otherwise takes.  The estimate is a line in k: a start of 0.17 us per
// key (0.24 at d = 128; fp32 0.31, 0.76) until the first landmarks are out, then 8 ... 18 (10 ... 25) us a step.  The lengths are those at which both
// sides were measured, with k from L/50 to the smaller of L and 4096, alpha = 1/2 and 1, and four clouds (drifting clusters, heavy
// tails, Gaussian or clusters, clusters at an offset of 20).  Where the rule takes a call it is 0.13 to 0.95 of the other kernel's time
// (bf16 1.0 to 1.08 on the offset clusters at 40 heads of 131072, d = 128).  Us, lazy / other: bf16, d = 64, k = L/50, 256 heads of
// 16384 keys 3700-6400 / 6400-9900, 384 of 32768 12600-22600 / 32800-56500, 128 of 65536 18700-45500 / 39800-68700, 64 of 131072
// 52600-137500 / 112100-159900; d = 128, 200 of 16384 4700-8900 / 12100-15800, 96 of 32768 9400-23300 / 20600-27500.
// What lies beyond: bf16 heads of 4096 keys and fewer 0.6 to 1.2; at d = 128 above 32768 keys the offset clusters ask for a margin (40 heads of
// 65536, 4096 picks: 92 against 201); fp32 of 65536 keys 0.5 to 2.0, of 131072 0.7 to 3.6, of 1100 0.2 to 0.9 but never taken.
LazyShape select_lazy_shape(bool bf16, int H, int L, int d, int k, float other_us, const Chip &chip, size_t scratch_bytes)
{
    LazyShape s{0, 0, 0};
    if (k > kMaxLazyK || L < (bf16 ? 8192 : 2048) || L > (bf16 ? kMaxLazyL : 16384) || scratch_bytes < kSelectFlagBytes) return s;
    const int per = kLazyWaves * 64 * kGroup;       // keys that a record per lane covers
    s.slots = L <= per ? 1 : L <= 2 * per ? 2 : 4;
    s.per_cu = bf16 && d == 64 && s.slots == 1 && H > chip.cus ? 2 : 1;
    const int most = chip.cus * s.per_cu < kMaxLazyHeads ? chip.cus * s.per_cu : kMaxLazyHeads;
    const int groups = H < most ? H : most;
    // a smaller workspace would mean more passes over the heads
    if ((scratch_bytes - kSelectFlagBytes) / lazy_slab_bytes(L) < (size_t)groups) return s;
    float passes = (float)((H + groups - 1) / groups);
    if (s.per_cu == 2) passes *= 1.7f;              // two heads on a compute unit: 16.4 ms for 320, 9.95 for 256
    const float l = (float)L;
    const float start = bf16 ? (d == 64 ? 0.17f : 0.24f) * l : (d == 64 ? 0.31f : 0.76f) * l;
    const float step = bf16 ? (d == 64 ? 6.7f + 8.5e-5f * l : 8.3f + 1.27e-4f * l) : (d == 64 ? 19.0f : 37.0f) + 1.3e-4f * l;
    if (passes * (start + step * (float)k) < (bf16 && d == 128 && L > 32768 ? 0.85f : 0.95f) * other_us) s.groups = groups;
    return s;
}

hipError_t launch_select_lazy(const LazyShape &shape, const void *K, bool bf16, int H, int L, int d, const float *rho, int k,
                              float alpha, int32_t *idx, float *score_out, void *ws, hipStream_t st)
{
    LazyArgs a;
    a.K = K;
    a.rho = rho;
    a.idx = idx;
    a.score_out = score_out;
    a.slab = reinterpret_cast<float *>(reinterpret_cast<char *>(ws) + kSelectFlagBytes);
    a.fail = reinterpret_cast<int *>(ws);
    a.H = H;
    a.L = L;
    a.k = k;
    a.Lpad = (int)round_up((size_t)L, kGroup);
    a.alpha = alpha;
    if (bf16) return d == 64 ? dispatch<uint16_t, 64>(a, shape, st) : dispatch<uint16_t, 128>(a, shape, st);
    return d == 64 ? dispatch<float, 64>(a, shape, st) : dispatch<float, 128>(a, shape, st);
}

}  // namespace ws
