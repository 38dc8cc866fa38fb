// Gaussian kernel density of the keys of each head (the inverse-kernel-density ingredient of
// the hybrid landmark score; Warp-Cortex Sec. 2 first paragraph and Sec. 3.3):
//     rho_i = (1/L) sum_j exp(-|k_i - k_j|^2 / (2 sigma^2)).
//
// The L x L sweep is a dense contraction and runs on the matrix cores.  With n_i = |k_i|^2,
//     -|k_i - k_j|^2 / 2 = k_i . k_j - n_i/2 - n_j/2,
// and both norm terms are folded INTO the contraction: every key carries a 16-byte side
// record that extends its row by a few extra columns holding -n/2 split into exactly
// representable pieces next to columns of ones, so the MFMA accumulator leaves the matrix
// core already holding -|k_i - k_j|^2/2.  The epilogue per pair is then one multiply by
// log2(e)/sigma^2, one v_exp_f32 and one add into a per-lane row accumulator: the sweep is
// bound by the vector/transcendental pipe, not by the matrix pipe, so every instruction
// removed there counts.  Padded key slots (index >= L) carry -1e30 in their record, which
// drives their kernel value to exactly 0.
//
// Accuracy and translation.  The exponent is formed from fp32 accumulators of magnitude ~|k|^2, so
// a kernel term carries a relative error of about 2^-23 |k|^2 / sigma^2.  The density itself does
// not depend on where the cloud sits, but that error does: a cloud with a common offset (what a
// real key cache looks like) would lose accuracy in proportion to the offset squared.  So the
// prepass moves the cloud: per head and coordinate it takes the mid-range c of the keys (rounded to
// bf16) and, WHERE k - c IS EXACTLY A bf16 NUMBER FOR EVERY KEY of that coordinate (decided from the
// coordinate's minimum, maximum and smallest non-zero magnitude: the keys of a coordinate with an
// offset well above its spread all share a coarse grid, so their differences to c need few bits),
// the sweep runs on a copy of the head holding k - c.  That copy is the same cloud, translated: no
// rounding takes part.  Coordinates where the differences are not exact (a spread comparable to the
// offset: little to gain there) keep c = 0; heads with c = 0 throughout are swept in place.  What is
// left is reported: per head the estimate 2^-23 mean|k - c|^2 / sigma^2 is written to the head of the
// workspace, and a flag is raised when it exceeds kErrBound (bandwidths far below the cloud's spread,
// offsets that cannot be removed exactly).  For sigma -> 0 only the self term survives, and that one
// is exact by construction.
//
// Every unordered pair is evaluated once (the kernel matrix is symmetric) by one of two sweeps: density_sym for bf16
// heads of at least four blocks of 256 keys, density_sym_small for fp32 keys and for shorter heads.
#include "ws_internal.h"

#include <type_traits>

namespace ws {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

typedef __attribute__((ext_vector_type(8))) float f32x8_t;
typedef f32x8_t __attribute__((aligned(16))) f32x8_16_t;     // as rows in memory are aligned

// Lane l of a wave supplies row (l % 32) of a 32-row tile and the k-slice selected by (l / 32).  Both operands of K K^T
// are fetched with the same pattern, so the result does not depend on how the hardware orders the k-slots inside an
// instruction.
__device__ __forceinline__ bf16x8_t load_frag(const uint16_t *row, int kk, int hb)
{
    return *reinterpret_cast<const bf16x8_t *>(row + kk * 16 + hb * 8);
}

// A float is the exact sum of three bf16 numbers (3 x 8 significant bits): p[0] + p[1] + p[2].  A NaN or an infinity
// leaves a NaN in the later pieces.
__device__ __forceinline__ void split3(f32x8_t x, bf16x8_t (&p)[3])
{
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        p[i] = __builtin_convertvector(x, bf16x8_t);
        x -= __builtin_convertvector(p[i], f32x8_t);
    }
}

// ------------------------------------------------------------------------------------------
// Prepass.
//   density_stats  (bf16)  per head, coordinate and chunk of rows: minimum, maximum, smallest non-zero magnitude, first
//                          on a sample, then, only for heads with a coordinate that might be moved, on all rows
//   density_prep           the head's reference point c (zero where k - c would not be exact), which copy of the head the
//                          sweep reads, the exponent scale; per key: k - c written to the copy (heads that move), |k - c|^2
//                          in fp64 and its side record; per block of 256 keys the sum of the squared norms; clears the flag
//   density_finish         rho from the accumulator cells; per head 2^-23 mean|k - c|^2 / sigma^2, and the flag
// The reference point is worked out by every workgroup that needs it (24 KB of L2 reads, only in heads that may move)
// rather than by kernels of their own: between two short kernels the chip idles for longer than that takes.
// ------------------------------------------------------------------------------------------
struct ScaleChunk {
    float s[256];
};

constexpr int kStatChunks = 16;          // row chunks per head in density_stats
constexpr float kErrBound = 2.0e-5f;     // estimated relative error of a kernel term above which a head is flagged

struct PrepWs {
    int *flag;              // [0] = 1 if some head's estimate exceeds kErrBound
    float *est;             // [H] estimated relative error of one kernel term
    float *scale;           // [H] log2(e) / sigma^2
    const void **kbase;     // [H] the rows the sweep reads: the caller's, or the translated copy
    int *cand;              // [H] some coordinate of the head may be moved, going by the sample (bf16 keys only)
    uint16_t *stat;         // [H][kStatChunks][3][D] min, max, smallest non-zero magnitude of the sample (bf16 keys only):
                            // values of the keys, so their 16 bits hold them
    uint16_t *full;         // the same of all rows, for the heads with cand set
    double *nsum;           // [H][Lpad/256] sum of squared norms per block of keys
    void *ext;              // [H][Lpad] side records: 16 bytes, or (density_sym_small) the 8 that are not constant
    void *Kc;               // [H][L][D] translated copy (bf16 keys only)
    unsigned long long *acc;   // [H][Lpad] kernel sums in fixed point: started here at the self term
    int large;              // density_sym reads the records
};

constexpr uint32_t kOnes = 0x3F803F80u;     // two bf16 ones

// 2^(floor(log2 v) - 7): the spacing of bf16 numbers around |v| (v finite, normal, non-zero)
__device__ __forceinline__ float bf16_ulp(float v)
{
    const uint32_t e = (__float_as_uint(v) >> 23) & 0xFFu;
    return e > 7u ? __uint_as_float((e - 7u) << 23) : 0.0f;
}

__device__ __forceinline__ float from_bf16(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ uint16_t bits_of_bf16(float v) { return (uint16_t)(__float_as_uint(v) >> 16); }     // v is one

// the reference point of coordinate j, from the statistics of the head's chunks; 0: the coordinate stays
template <int D>
__device__ __forceinline__ float reference_point(const uint16_t *__restrict__ stat /* the head's */, int j)
{
    float mn = __builtin_inff(), mx = -__builtin_inff(), ma = __builtin_inff();
#pragma unroll
    for (int ch = 0; ch < kStatChunks; ++ch) {
        const uint16_t *st = stat + (size_t)ch * 3 * D;
        mn = fminf(mn, from_bf16(st[j]));
        mx = fmaxf(mx, from_bf16(st[D + j]));
        ma = fminf(ma, from_bf16(st[2 * D + j]));
    }
    float c = 0.0f;
    if (mx >= mn && ma < __builtin_inff()) {          // finite, not all zero
        const float mid = __uint_as_float(bf16_rne(0.5f * mn + 0.5f * mx) << 16);
        if (mid != 0.0f && fabsf(mid) < __builtin_inff()) {
            // every key of the coordinate and c are multiples of g (the finer of their bf16 spacings); k - c is a
            // bf16 number when |k - c| <= 256 g.  g must be a normal number well inside the range.
            const float g = fminf(bf16_ulp(ma), bf16_ulp(mid));
            const float X = fmaxf(mx - mid, mid - mn) * 1.000001f;
            if (g >= 7.0e-31f && X <= 256.0f * g) c = mid;
        }
    }
    return c;
}

// Two passes.  Pass 0 looks at the first eighth of every chunk of rows.  More keys only widen a coordinate's range
// and refine its grid, so a coordinate that fails the exactness test on the sample is taken to fail it on the whole
// head (a rule on the safe side: it decides only whether a head is moved, never a value): heads without a candidate
// coordinate are settled by the sample, and pass 1, which reads the rest and merges, skips them.
template <int D>
__global__ void __launch_bounds__(256)
density_stats(const uint16_t *__restrict__ K, uint16_t *__restrict__ stat, uint16_t *__restrict__ full, int L, int pass,
              int *__restrict__ cand)
{
    constexpr int CH = D / 8;            // 16-byte pieces per row
    constexpr int RPS = 256 / CH;        // rows per sweep of the block
    __shared__ float red[3][RPS][D + 1];
    const int h = blockIdx.y, chunk = blockIdx.x;
    if (pass == 1) {
        float c = 0.0f;
        if (threadIdx.x < D) c = reference_point<D>(stat + (size_t)h * kStatChunks * 3 * D, threadIdx.x);
        const int may = __syncthreads_or(c != 0.0f);
        if (chunk == 0 && threadIdx.x == 0) cand[h] = may;
        if (!may) return;
    }
    const int per = (L + kStatChunks - 1) / kStatChunks;
    const int cut = chunk * per + (per + 7) / 8;
    const int lo = pass == 0 ? chunk * per : min(L, cut);
    const int hi = pass == 0 ? min(L, cut) : min(L, (chunk + 1) * per);
    const int piece = threadIdx.x % CH, r0 = threadIdx.x / CH;
    float mn[8], mx[8], ma[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        mn[i] = __builtin_inff();
        mx[i] = -__builtin_inff();
        ma[i] = __builtin_inff();
    }
    const uint16_t *Kh = K + (size_t)h * L * D;
    for (int r = lo + r0; r < hi; r += RPS) {
        const uint4 q = *reinterpret_cast<const uint4 *>(Kh + (size_t)r * D + piece * 8);
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float v = __uint_as_float((i & 1) ? (w[i >> 1] & 0xFFFF0000u) : (w[i >> 1] << 16));
            mn[i] = fminf(mn[i], v);
            mx[i] = fmaxf(mx[i], v);
            const float av = fabsf(v);
            if (av > 0.0f) ma[i] = fminf(ma[i], av);
        }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        red[0][r0][piece * 8 + i] = mn[i];
        red[1][r0][piece * 8 + i] = mx[i];
        red[2][r0][piece * 8 + i] = ma[i];
    }
    __syncthreads();
    for (int c = threadIdx.x; c < 3 * D; c += 256) {
        const int which = c / D, j = c % D;
        float v = red[which][0][j];
        for (int r = 1; r < RPS; ++r) v = (which == 1) ? fmaxf(v, red[which][r][j]) : fminf(v, red[which][r][j]);
        const size_t at = (((size_t)h * kStatChunks + chunk) * 3 + which) * D + j;
        if (pass == 1) {
            const float o = from_bf16(stat[at]);
            full[at] = bits_of_bf16((which == 1) ? fmaxf(v, o) : fminf(v, o));
        } else {
            stat[at] = bits_of_bf16(v);
        }
    }
}

// sc: the exponent scales of the launch's heads
template <bool kBf16, int D>
__global__ void __launch_bounds__(256)
density_prep(const void *__restrict__ K, PrepWs w, ScaleChunk sc, int head0, int L, int Lpad)
{
    typedef typename std::conditional<kBf16, uint16_t, float>::type Elem;
    __shared__ double part[256];
    __shared__ float cv[kBf16 ? D : 1];
    const int h = head0 + blockIdx.y;
    const int j = blockIdx.x * 256 + threadIdx.x;
    const Elem *Kh = reinterpret_cast<const Elem *>(K) + (size_t)h * L * D;
    Elem *Kch = reinterpret_cast<Elem *>(w.Kc) + (size_t)h * L * D;
    bool moved = false;
    if constexpr (kBf16) {
        if (w.cand[h]) {
            float c = 0.0f;
            if (threadIdx.x < D) cv[threadIdx.x] = c = reference_point<D>(w.full + (size_t)h * kStatChunks * 3 * D, threadIdx.x);
            moved = __syncthreads_or(c != 0.0f);
        }
    }
    if (j == 0) {
        w.kbase[h] = moved ? (const void *)Kch : (const void *)Kh;
        w.scale[h] = sc.s[blockIdx.y];
        if (h == 0) w.flag[0] = 0;
    }
    uint2 rec;
    double n = 0.0;
    if (j < L) {
        // whole row through 16-byte loads (a thread owns a row: 8 or more loads hit the same lines)
        const uint4 *row = reinterpret_cast<const uint4 *>(Kh + (size_t)j * D);
        uint4 *crow = reinterpret_cast<uint4 *>(Kch + (size_t)j * D);
        constexpr int PER = 16 / sizeof(Elem);
        constexpr int NPC = D / PER;             // 16-byte pieces per row
        constexpr int GRP = NPC < 8 ? NPC : 8;   // pieces in flight at a time (all loads of a group before any store)
#pragma unroll
        for (int c0 = 0; c0 < NPC; c0 += GRP) {
            uint4 qs[GRP];
#pragma unroll
            for (int c = 0; c < GRP; ++c) qs[c] = row[c0 + c];
#pragma unroll
            for (int c = 0; c < GRP; ++c) {
                Elem e[PER];
                __builtin_memcpy(e, &qs[c], 16);
                uint32_t xb[PER];
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    if constexpr (kBf16) {
                        // exact: c is non-zero only where every k - c of the coordinate is a bf16 number
                        // (heads that stay in place skip the reference point: it is zero throughout)
                        float xf = __uint_as_float((uint32_t)e[i] << 16);
                        if (moved) xf -= cv[(c0 + c) * PER + i];
                        xb[i] = __float_as_uint(xf) >> 16;
                        n += (double)xf * (double)xf;
                    } else {
                        const double x = (double)e[i];
                        n += x * x;
                    }
                }
                if constexpr (kBf16) {
                    if (moved)
                        crow[c0 + c] = make_uint4(xb[0] | (xb[1] << 16), xb[2] | (xb[3] << 16), xb[4] | (xb[5] << 16),
                                                  xb[6] | (xb[7] << 16));
                }
            }
        }
        double x = -0.5 * n;
        uint32_t p[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            p[q] = bf16_rne((float)x);
            x -= (double)__uint_as_float(p[q] << 16);
        }
        rec = make_uint2(p[0] | (p[1] << 16), p[2] | (p[3] << 16));
    } else {
        // padded slot: -1e30 makes exp2() of the pair exactly 0
        rec = make_uint2(bf16_rne(-1e30f), 0u);
    }
    if (j < Lpad) {
        if (w.large) reinterpret_cast<uint4 *>(w.ext)[(size_t)h * Lpad + j] = make_uint4(rec.x, rec.y, kOnes, kOnes);
        else reinterpret_cast<uint2 *>(w.ext)[(size_t)h * Lpad + j] = rec;
        // the cell of a key starts at its self term, exactly 1 (in 32.32 fixed point): kept out of
        // the fp32 row accumulators, where a 1 would swallow the many kernel values below its half ulp that make
        // up the rest of an isolated key's sum
        w.acc[(size_t)h * Lpad + j] = (j < L) ? (1ull << 32) : 0ull;
    }
    // sum of the block's squared norms, in a fixed order
    part[threadIdx.x] = n;
    __syncthreads();
    for (int o = 128; o >= 1; o >>= 1) {
        if ((int)threadIdx.x < o) part[threadIdx.x] += part[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) w.nsum[(size_t)h * (Lpad / 256) + blockIdx.x] = part[0];
}

// LDS-only barrier: waits for this wave's LDS traffic, not for its global loads
__device__ __forceinline__ void lds_only_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Asynchronous 16-byte-per-lane copy global -> LDS (no registers in between): lane i of the wave reads base +
// byte_offset and lands at lds_base + 16 * i.  Completion is counted by vmcnt like any vector load; the compiler does not see it, so the
// caller waits explicitly before the barrier that publishes the data.
__device__ __forceinline__ void dma16(const void *base /* wave-uniform */, unsigned byte_offset, const void *lds_base)
{
    const unsigned la =
        __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) const void *)lds_base);
    asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(byte_offset), "s"(base), "s"(la) : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// ------------------------------------------------------------------------------------------
// Symmetric sweep (bf16 keys, heads of at least a few row blocks).
//
// The kernel matrix is symmetric, and its cost is the exponential, not the contraction: so every
// unordered pair is evaluated ONCE and its value is added to the row sum of i and to the
// column sum of j.  Keys are cut into blocks of BM rows; workgroup I evaluates block I against
// blocks I (row sums only), I+1 .. I+nBoth (row and column sums) and, when the block count is
// even, I + nB/2 (row sums only; its partner evaluates the transposed copy).  Every workgroup
// does the same amount of work.  Row sums stay in registers for the whole sweep.  Column sums
// of one visited block are reduced over the workgroup's 4 waves in LDS and added to the keys'
// accumulator cells (fixed point, integer atomics: see fixed_add), as are the row sums at the
// end; a last small kernel turns the cells into rho.  Integer addition is associative, so the
// result does not depend on scheduling.
//
// The 4 waves of a workgroup own different rows (RTW tiles of 32 each) and share the stream of
// column tiles: 64 key rows per stage reach the LDS by asynchronous global -> LDS copies (no
// registers in between) issued two stages ahead into three rotating buffers, and are read back in
// MFMA operand layout (16-byte pieces, XOR-swizzled by row so the 8 lanes served per LDS cycle hit
// 8 different bank groups; the swizzle is applied on the global side of the copy).  One LDS-only
// barrier per stage publishes the stage and retires the buffer two stages back.
//
// The contraction runs one tile ahead of the vector work through the whole sweep, across tiles, stages and blocks: at two
// (d = 128) or three (d = 64) waves per SIMD a contraction that stands alone at the head of a column tile is not hidden by
// the other waves.  Against the form that started each column tile with its first contraction exposed: 20.2 -> 18.7 ms for
// 8 heads of 131072 keys at d = 128 (now the matrix cores are busy 54 % of the cycles, the vector pipe 73 %), 39.1 -> 38.2 ms
// for 384 heads of 32768 keys at d = 64 (41 % and 95 %; 39 % and 90 % before).  One body serves the diagonal and the one-sided blocks too (they form column sums that are not used):
// three copies of it do not fit the registers.
// ------------------------------------------------------------------------------------------
// The kernel sums of a key come from many workgroups (its own row block, and every block that visits it as
// a column block).  They are accumulated in 32.32 fixed point with integer atomics: integer addition is
// associative, so the result does not depend on the order in which the workgroups arrive (a floating-point
// atomic would), and one 8-byte cell per key replaces a slot per visiting workgroup.  The 2^-32 resolution is far
// below fp32 rounding of sums that are >= 1 (the self term).
//
// A kernel value is <= 1 in exact arithmetic, but the exponent is rounded, and at norms far above the bandwidth rounding
// can leave it positive: a value of any size up to infinity.  So a contribution enters as a number only up to 32 times
// the pairs it sums (a cell's pairs number less than 2^24 + 2^10, so its sum stays below 2^62); what is larger marks the
// cell as infinite, a NaN marks it as NaN, and the marks outlast whatever is added.
constexpr unsigned long long kNanCell = 1ull << 63, kInfCell = 1ull << 62;

__device__ __forceinline__ bool fits_cell(float v, int pairs) { return v <= 32.0f * (float)pairs; }

__device__ __forceinline__ void fixed_add(unsigned long long *cell, float v)
{
    __hip_atomic_fetch_add(cell, (unsigned long long)__float2ll_rn(v * 4294967296.0f), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void fixed_add_or_mark(unsigned long long *cell, float v, int pairs)
{
    if (fits_cell(v, pairs)) fixed_add(cell, v);
    else __hip_atomic_fetch_or(cell, v == v ? kInfCell : kNanCell, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The row sums of a 32-row tile: summed over the 32 columns held by the lanes of a half-wave, then added to the rows'
// cells by the half-waves' first lanes (n == 0; acc: the cell of this half-wave's first row).  One test for all of them:
// with a branch around every add 16 heads of 4096 keys, d = 64, took 55.2 us against 54.3 without the marks; this way 50.6
// (the sums by DPP steps instead of shuffles are part of that).
__device__ __forceinline__ void add_row_sums(unsigned long long *acc, float (&v)[16], int pairs, int n)
{
    bool fits = true;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        v[r] = lane_group_sum<32>(v[r]);
        fits = fits && fits_cell(v[r], pairs);
    }
    if (__all(fits)) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (n == 0) fixed_add(acc + 8 * (r >> 2) + (r & 3), v[r]);
    } else {
        for (int r = 0; r < 16; ++r)
            if (n == 0) fixed_add_or_mark(acc + 8 * (r >> 2) + (r & 3), v[r], pairs);
    }
}

constexpr int kSymRtw = 2;                        // row tiles per wave of density_sym
constexpr int kSymBm = 128 * kSymRtw;             // keys per block of density_sym ...
constexpr int kSmallBm = 128, kSmallSc = 32;      // ... and of density_sym_small, and keys per stage there

// Piece kk of this lane's row of a column tile: the row's pieces sit XOR-swizzled by the row's low three bits, so with the
// byte of piece 0 in hand the others are an XOR (and an offset) away: one address register for all of them.
__device__ __forceinline__ uint4 operand_piece(const uint4 *lds, unsigned at, int kk)
{
    return *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(lds) + (at ^ (unsigned)((kk & 3) * 32)) + (kk >> 2) * 128);
}

// One step of the pipelined sweep: the contraction of the next tile (row operand an, column operand b) into nxt, one
// MFMA per slice of the vector work of the tile in cur.  diag: cur is a diagonal tile.  RELOAD: this is the last use of
// the column operand; behind each MFMA its piece is fetched anew for the next column tile (piece 0 at byte `next` of lds,
// record at ne), a whole step ahead of use and without a second set of registers.  The last three of the 16 values are
// left behind the last MFMA, whose result the next step begins with.
template <int NS, bool RELOAD>
__device__ __forceinline__ void sym_step(const bf16x8_t (&an)[NS], bf16x8_t (&b)[NS], f32x16_t &nxt, f32x16_t &cur,
                                         float (&racc)[16], float &csum, float s, int n, int hb, bool diag,
                                         const uint4 *lds, unsigned next, const uint4 *ne)
{
    if (diag) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (8 * (r >> 2) + 4 * hb + (r & 3) == n) cur[r] = -1e30f;   // the self term is in the cell already
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) nxt[r] = 0.0f;
#pragma unroll
    for (int kk = 0; kk < NS; ++kk) {
        nxt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(an[kk], b[kk], nxt, 0, 0, 0);
        if (RELOAD) b[kk] = __builtin_bit_cast(bf16x8_t, kk < NS - 1 ? operand_piece(lds, next, kk) : ne[0]);
#pragma unroll
        for (int r = kk * 13 / NS; r < (kk < NS - 1 ? (kk + 1) * 13 / NS : 16); ++r) {
            const float w = __builtin_amdgcn_exp2f(cur[r] * s);
            racc[r] += w;
            csum += w;
            asm volatile("" : "+v"(racc[r]), "+v"(csum));      // or the adds gather behind the step, where no MFMA runs
        }
        // keeps each MFMA between its shares of the vector work
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 64 ? 3 : 2, D == 64 ? 3 : 2)))
density_sym(const void *const *__restrict__ kbase, const uint4 *__restrict__ ext, const float *__restrict__ scale,
            unsigned long long *__restrict__ acc, int L, int Lpad, int nB, int nBoth, int nblk, int parts, int head0, int total)
{
    constexpr int NK = D / 16, NS = NK + 1;
    constexpr int RTW = kSymRtw;           // row tiles per wave
    constexpr int BM = kSymBm;             // rows (and columns) per block
    constexpr int CH = D / 8;              // 16-byte pieces per key row
    constexpr int SC = 64;                 // key rows per LDS stage
    constexpr int SPB = BM / SC;           // stages per block
    constexpr int NLD = SC * CH / 256;     // 16-byte pieces each thread moves per stage
    constexpr int NBUF = 3, PF = NBUF - 1;  // LDS buffers in rotation; stages the copies run ahead
    __shared__ uint4 sB[NBUF][SC * CH];
    __shared__ uint4 sE[NBUF][SC];
    __shared__ float cs[2][4][2][BM];       // column sums of a visited block: per wave and half-wave

    const int logical = xcd_contiguous(blockIdx.x, total);
    // row block I of head h against the visited blocks j0 ... j1-1 of its nblk (see split_parts)
    const int hI = logical / parts, part = logical - hI * parts;
    const int hl = hI / nB, I = hI - hl * nB;
    const int h = head0 + hl;
    const int j0 = (int)((long long)nblk * part / parts), j1 = (int)((long long)nblk * (part + 1) / parts);
    const uint16_t *Kh = reinterpret_cast<const uint16_t *>(kbase[h]);     // the caller's rows or their translated copy
    const uint4 *exth = ext + (size_t)h * Lpad;
    const float s = scale[h];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, hb = lane >> 5;

    bf16x8_t a[RTW][NS];
#pragma unroll
    for (int rt = 0; rt < RTW; ++rt) {
        const int row = I * BM + (wave * RTW + rt) * 32 + n;      // < Lpad
        const uint16_t *rp = Kh + (size_t)min(row, L - 1) * D;
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) a[rt][kk] = load_frag(rp, kk, hb);
        // the record is {m1..m4, 1,1,1,1} with m1+..+m4 = -n/2: the column side uses it as it is, the row side
        // swaps its halves, so the extra k-step adds -n_i/2 - n_j/2.  Only the first 8 k-slots are used: the row
        // side holds zeros in the others, so what the column side holds there does not matter.
        const uint4 rec = exth[row];
        a[rt][NK] = __builtin_bit_cast(bf16x8_t, hb ? make_uint4(0, 0, 0, 0) : make_uint4(rec.z, rec.w, rec.x, rec.y));
    }
    float racc[RTW][16];
#pragma unroll
    for (int rt = 0; rt < RTW; ++rt)
#pragma unroll
        for (int r = 0; r < 16; ++r) racc[rt][r] = 0.0f;

    const int nst = (j1 - j0) * SPB;

    // Key rows reach the LDS by asynchronous copies issued two stages ahead, already in the swizzled order the
    // MFMA operand reads expect (slot c of row r holds piece c ^ (r & 7)); three buffers rotate.
    // per-thread constants of the copy: which row of a stage and which (swizzled) 16-byte piece of it; the
    // thread's further pieces of a stage sit 256 / CH rows below with the same swizzle (256 / CH is a multiple of 8)
    // (byte offsets inside a head are 32-bit: the entry point admits L < 2^24 rows of at most 256 bytes)
    const int crow = tid / CH;
    const unsigned cpiece = (unsigned)(((tid % CH) ^ (crow & 7)) * 16);
    auto issue = [&](int sidx) {
        const int J = (I + j0 + sidx / SPB) % nB;
        const int col0 = J * BM + (sidx % SPB) * SC;
        const int bi = sidx % NBUF;
#pragma unroll
        for (int i = 0; i < NLD; ++i)
            dma16(Kh, (unsigned)min(col0 + crow + i * (256 / CH), L - 1) * (unsigned)(D * 2) + cpiece,
                  &sB[bi][wave * 64 + 256 * i]);
        if (wave == 0) dma16(exth, (unsigned)(col0 + lane) * 16u, &sE[bi][0]);
    };

    // The row operands must be in their registers before the first asynchronous copy is issued: the compiler
    // would otherwise wait for them at their first use inside the loop, with a count that also covers the copies.
    wait_vmcnt<0>();

#pragma unroll
    for (int p = 0; p < PF; ++p)
        if (p < nst) issue(p);
    // the column sums of a visited block go to its keys' cells (cs rotates by block: the next block's sums are written
    // without another barrier)
    auto flush = [&](int j) {
        lds_only_barrier();
        unsigned long long *dst = acc + (size_t)h * Lpad + (size_t)((I + j) % nB) * BM;
        const float (*c2)[2][BM] = cs[j & 1];
        for (int c = tid; c < BM; c += 256)
            fixed_add_or_mark(dst + c, ((c2[0][0][c] + c2[0][1][c]) + (c2[1][0][c] + c2[1][1][c])) +
                                   ((c2[2][0][c] + c2[2][1][c]) + (c2[3][0][c] + c2[3][1][c])), BM);
    };
    // this wave's copies of stage sidx have landed (those of the next stage may still be in flight), and so have
    // everybody's; all waves are through with the stage before
    auto arrive = [&](int sidx) {
        if (sidx + 1 < nst) {
            if (wave == 0) wait_vmcnt<NLD + 1>();
            else wait_vmcnt<NLD>();
        } else {
            wait_vmcnt<0>();
        }
        lds_only_barrier();
        if (sidx + PF < nst) issue(sidx + PF);
    };
    const unsigned at0 = (unsigned)(n * CH + (hb ^ (n & 7))) * 16u;     // this lane's piece 0 in tile 0 of buffer 0
    bf16x8_t b[NS];
    f32x16_t c0, c1;
    arrive(0);
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) b[kk] = __builtin_bit_cast(bf16x8_t, operand_piece(&sB[0][0], at0, kk));
    b[NK] = __builtin_bit_cast(bf16x8_t, sE[0][n]);
#pragma unroll
    for (int r = 0; r < 16; ++r) c0[r] = 0.0f;
#pragma unroll
    for (int kk = 0; kk < NS; ++kk) c0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0][kk], b[kk], c0, 0, 0, 0);
    for (int sidx = 0; sidx < nst; ++sidx) {
        const int buf = sidx % NBUF;
        const int j = j0 + sidx / SPB, sin = sidx % SPB;
        const bool both = j >= 1 && j <= nBoth;
        const bool diag = j == 0 && sin == wave;   // (RTW == SC / 32: the row tiles of a wave meet one stage)
        unsigned next = at0 + (unsigned)(buf * SC + 32) * (CH * 16);
        asm("" : "+v"(next));       // or every piece keeps an address register of its own from stage to stage
        const uint4 *ne = sE[buf] + n + 32;
        float csum = 0.0f;
        sym_step<NS, true>(a[1], b, c1, c0, racc[0], csum, s, n, hb, diag, &sB[0][0], next, ne);
        sym_step<NS, false>(a[0], b, c0, c1, racc[1], csum, s, n, hb, false, &sB[0][0], next, ne);
        if (both) cs[j & 1][wave][hb][n + sin * SC] = csum;
        csum = 0.0f;
        // (behind the last stage the first tile of that stage is contracted once more, and not used)
        if (sidx + 1 < nst) arrive(sidx + 1);
        const int nbuf = sidx + 1 < nst ? (sidx + 1) % NBUF : buf;
        next = at0 + (unsigned)(nbuf * SC) * (CH * 16);
        asm("" : "+v"(next));
        ne = sE[nbuf] + n;
        sym_step<NS, true>(a[1], b, c1, c0, racc[0], csum, s, n, hb, false, &sB[0][0], next, ne);
        sym_step<NS, false>(a[0], b, c0, c1, racc[1], csum, s, n, hb, diag, &sB[0][0], next, ne);
        if (both) cs[j & 1][wave][hb][n + sin * SC + 32] = csum;
        if (both && sin == SPB - 1) flush(j);
    }

    // each wave owns its rows
#pragma unroll
    for (int rt = 0; rt < RTW; ++rt)
        add_row_sums(acc + (size_t)h * Lpad + I * BM + (wave * RTW + rt) * 32 + 4 * hb, racc[rt], nst * SC, n);
}

// ------------------------------------------------------------------------------------------
// The same sweep for fp32 keys and for short heads: blocks of 128 keys, one 32-row tile per wave.
//
// fp32 keys.  Bound by the matrix cores.  The fp32 MFMA forms run at a sixteenth of the bf16 rate, so a key is split into
// its three bf16 pieces (exactly: 24 bits) while a stage is brought to the LDS, and a product of two keys is six of the nine
// piece products, the small ones summed first: 6 x d/16 + 1 MFMAs of 32 cycles per 32 x 32 tile (800 cycles at d = 64)
// against d/2 + 2 of 64 cycles (2176), and half the tiles.  The three left out are at most 2^-24 of |a||b| per coordinate
// (|a1| <= 2^-8, |a2| <= 2^-17 of a's power of two), half the spacing of the product in fp32 and below what the accumulator
// rounds away.  The split costs 50 vector instructions per wave and stage, which run beside the matrix work.
//
// A stage is 32 keys; its rows are loaded one stage ahead into registers and written to the other of two LDS buffers after
// the stage's work, so there is one barrier per stage.  One fp32 head of 512 keys: the sweep 33 -> 7 us against one over all
// ordered pairs with fp32 MFMAs.  Mean 2-norm error against 64 bits over five kinds of clouds of 200 to 6000 keys (ten kinds of
// lattices, duplicates and offsets beside them): d = 64 0.8 to 2.2e-7, with fp32 MFMAs 1.1 to 4.3e-7; d = 128 0.7 to 2.4e-7,
// 1.2 to 6.0e-7; no kind larger than there.
// ------------------------------------------------------------------------------------------
template <bool F32, int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu((F32 && D == 128) ? 2 : 3, (F32 && D == 128) ? 2 : 3)))
density_sym_small(const void *const *__restrict__ kbase, const uint2 *__restrict__ ext, const float *__restrict__ scale,
                  unsigned long long *__restrict__ acc, int L, int Lpad, int nB, int nBoth, int nblk, int parts, int head0,
                  int total)
{
    typedef typename std::conditional<F32, float, uint16_t>::type Elem;
    constexpr int NP = F32 ? 3 : 1;         // bf16 pieces per element
    constexpr int NK = D / 16;
    constexpr int BM = kSmallBm, SC = kSmallSc, SPB = BM / SC;
    constexpr int CR = D / 8;               // groups of eight elements per key row: 16 bytes of each piece
    constexpr int CH = NP * CR;             // 16-byte pieces per LDS row
    constexpr int NLD = SC * CR / 256;      // groups each thread brings in per stage
    __shared__ uint4 sB[2][SC * CH];
    __shared__ uint4 sE[2][SC];
    __shared__ float cs[4][2][BM];          // column sums of a block: per wave and half-wave

    const int logical = xcd_contiguous(blockIdx.x, total);
    const int hI = logical / parts, part = logical - hI * parts;
    const int hl = hI / nB, I = hI - hl * nB;
    const int h = head0 + hl;
    // row block I of head h against the visited stages s0 ... s1-1 of its nblk blocks (see split_parts)
    const int s0 = (int)((long long)nblk * SPB * part / parts), s1 = (int)((long long)nblk * SPB * (part + 1) / parts);
    const Elem *Kh = reinterpret_cast<const Elem *>(kbase[h]);
    const uint2 *exth = ext + (size_t)h * Lpad;
    const float s = scale[h];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, hb = lane >> 5;

    bf16x8_t a[NP][NK], aext;
    {
        const int row = I * BM + wave * 32 + n;         // < Lpad
        const Elem *rp = Kh + (size_t)min(row, L - 1) * D;
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) {
            if constexpr (F32) {
                bf16x8_t p[3];
                split3(*reinterpret_cast<const f32x8_16_t *>(rp + kk * 16 + hb * 8), p);
#pragma unroll
                for (int i = 0; i < 3; ++i) a[i][kk] = p[i];
            } else {
                a[0][kk] = load_frag(rp, kk, hb);
            }
        }
        const uint2 rec = exth[row];
        aext = __builtin_bit_cast(bf16x8_t, hb ? make_uint4(0, 0, 0, 0) : make_uint4(kOnes, kOnes, rec.x, rec.y));
    }
    float racc[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) racc[r] = 0.0f;

    // group c of row r of a stage waits in slot c ^ (r & 7) of the row's pieces (8 lanes served per LDS cycle hit 8
    // different bank groups)
    typedef typename std::conditional<F32, f32x8_16_t, bf16x8_t>::type Group;
    Group g[NLD];
    uint2 grec;
    auto fetch = [&](int sidx) {
        const int col0 = ((I + sidx / SPB) % nB) * BM + (sidx % SPB) * SC;
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const int q = tid + 256 * i, r = q / CR, c = q % CR;
            g[i] = *reinterpret_cast<const Group *>(Kh + (size_t)min(col0 + r, L - 1) * D + c * 8);
        }
        if (tid < SC) grec = exth[col0 + tid];
    };
    auto publish = [&](int buf) {
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const int q = tid + 256 * i, r = q / CR, c = q % CR;
            uint4 *dst = &sB[buf][r * CH + (c ^ (r & 7))];
            if constexpr (F32) {
                bf16x8_t p[3];
                split3(g[i], p);
#pragma unroll
                for (int k = 0; k < 3; ++k) dst[k * CR] = __builtin_bit_cast(uint4, p[k]);
            } else {
                dst[0] = __builtin_bit_cast(uint4, g[i]);
            }
        }
        if (tid < SC) sE[buf][tid] = make_uint4(grec.x, grec.y, kOnes, kOnes);
    };

    fetch(s0);
    publish(s0 & 1);
    for (int sidx = s0; sidx < s1; ++sidx) {
        const int buf = sidx & 1;
        __syncthreads();        // the stage is in; everybody is through with the other buffer
        if (sidx + 1 < s1) fetch(sidx + 1);
        const int j = sidx / SPB, sin = sidx % SPB;
        const bool both = j >= 1 && j <= nBoth;
        const uint4 *row = &sB[buf][n * CH];
        auto piece = [&](int p, int kk) { return __builtin_bit_cast(bf16x8_t, row[p * CR + ((2 * kk + hb) ^ (n & 7))]); };
        f32x16_t t;
#pragma unroll
        for (int r = 0; r < 16; ++r) t[r] = 0.0f;
        if constexpr (F32) {
#pragma unroll
            for (int kk = 0; kk < NK; ++kk) {
                const bf16x8_t b0 = piece(0, kk), b1 = piece(1, kk), b2 = piece(2, kk);
                t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2][kk], b0, t, 0, 0, 0);
                t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0][kk], b2, t, 0, 0, 0);
                t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1][kk], b1, t, 0, 0, 0);
                t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1][kk], b0, t, 0, 0, 0);
                t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0][kk], b1, t, 0, 0, 0);
            }
        }
        // The norms enter half way: of near keys, which make up the sum, the accumulator then holds |k|^2 at no time but half of
        // it at most, and rounds to half of the spacing.
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) {
            if (kk == NK / 2)
                t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aext, __builtin_bit_cast(bf16x8_t, sE[buf][n]), t, 0, 0, 0);
            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0][kk], piece(0, kk), t, 0, 0, 0);
        }
        if (j == 0 && sin == wave) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (8 * (r >> 2) + 4 * hb + (r & 3) == n) t[r] = t[r] == t[r] ? -1e30f : t[r];   // the self term is in the cell already
        }
        float csum = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float w = __builtin_amdgcn_exp2f(t[r] * s);
            racc[r] += w;
            csum += w;
        }
        if (both) cs[wave][hb][sin * SC + n] = csum;
        if (sidx + 1 < s1) publish(buf ^ 1);
        if (both && (sin == SPB - 1 || sidx + 1 == s1)) {
            __syncthreads();
            const int first = max(s0 - j * SPB, 0) * SC;        // the part may have begun, or end, inside the block
            unsigned long long *dst = acc + (size_t)h * Lpad + (size_t)((I + j) % nB) * BM;
            if (tid >= first && tid < (sin + 1) * SC)
                fixed_add_or_mark(dst + tid, ((cs[0][0][tid] + cs[0][1][tid]) + (cs[1][0][tid] + cs[1][1][tid])) +
                                         ((cs[2][0][tid] + cs[2][1][tid]) + (cs[3][0][tid] + cs[3][1][tid])), BM);
        }
    }
    add_row_sums(acc + (size_t)h * Lpad + I * BM + wave * 32 + 4 * hb, racc, (s1 - s0) * SC, n);
}

// rho = accumulated kernel sum / L; the first workgroup of a head also estimates the head's error
__global__ void __launch_bounds__(256)
density_finish(PrepWs w, float *__restrict__ rho, int L, int Lpad, int head0)
{
    const int h = head0 + blockIdx.y;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < L) {
        const unsigned long long cell = w.acc[(size_t)h * Lpad + i];
        const double t = (double)cell * (1.0 / 4294967296.0);
        rho[(size_t)h * L + i] = cell & kNanCell   ? __builtin_nanf("")
                                 : cell & kInfCell ? __builtin_inff()
                                                   : (float)(t / (double)L);
    }
    if (blockIdx.x != 0) return;
    __shared__ double part[256];
    double t = 0.0;
    for (int b = threadIdx.x; b < Lpad / 256; b += 256) t += w.nsum[(size_t)h * (Lpad / 256) + b];
    part[threadIdx.x] = t;
    __syncthreads();
    for (int o = 128; o >= 1; o >>= 1) {
        if ((int)threadIdx.x < o) part[threadIdx.x] += part[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        // scale = log2(e) / sigma^2
        const float est = (float)(1.1920928955078125e-7 * (part[0] / (double)L) * ((double)w.scale[h] / 1.4426950408889634));
        w.est[h] = est;
        if (!(est <= kErrBound)) atomicExch(w.flag, 1);
    }
}

// A launch of the symmetric sweep takes at most this many heads.
constexpr int kSymChunkHeads = 16384;

static inline bool use_large(bool bf16, int L) { return bf16 && (L + kSymBm - 1) / kSymBm >= 4; }

// How many workgroups share a row block's visited blocks.  Few heads of few blocks leave the chip idle with one workgroup
// per row block (16 heads of 4096 keys, d = 64: 256 workgroups where 768 fit), so the visits (blocks in density_sym, stages
// in density_sym_small) are cut into `parts` ranges: the count that makes rounds x visits per workgroup smallest, a
// workgroup's start (row operands, first stage) priced at 0.35 blocks, or at two stages.  Launches of many rounds stay
// whole: cutting them could only add starts.  The call of the example takes 64 us whole and 51 us in three parts; one fp32
// head of 512 keys 25 us whole and 17 in twelve.  The prices are set by what they choose: over ten launches of 1 to 384 heads
// of 512 to 16384 keys the choice was within 2 % of the best of 1 to 12 parts in nine, and 7 % from it for 40 fp32 heads of
// 2048 (88 us whole, 83 in two parts).
// The row sums of a head are grouped as its visits are shared out, so its last bits follow the launch (the header says so;
// sums at fixed visit boundaries instead would add a reduction per boundary to launches that are not cut).
static int split_parts(long long wgs, int visits, long long resident, double start)
{
    int best = 1;
    double cost = 1e300;
    for (int p = 1; p <= visits && p <= 64; ++p) {
        const long long rounds = (wgs * p + resident - 1) / resident;
        const double c = (double)rounds * ((visits + p - 1) / p + start);
        if (c < cost * 0.999) {
            cost = c;
            best = p;
        }
        if (wgs >= 16 * resident) break;
    }
    return best;
}

// ------------------------------------------------------------------------------------------
struct DensityWs {
    size_t est, scale, kbase, cand, stat, full, nsum, ext, kc, acc, total;
    int Lpad;
};

// What callers were told to hold when the statistics were 32-bit, every record 16 bytes and short heads had no cells is
// enough for this layout at all sizes.
static DensityWs density_layout(int H, int L, int d, bool bf16)
{
    DensityWs w;
    w.Lpad = density_lpad(L);
    size_t o = kDensityFlagBytes;                               // the flag block sits in front
    w.est = o;
    o += round_up((size_t)H * sizeof(float), 256);
    w.scale = o;
    o += round_up((size_t)H * sizeof(float), 256);
    w.kbase = o;
    o += round_up((size_t)H * sizeof(void *), 256);
    w.cand = o;
    o += round_up((size_t)H * sizeof(int), 256);
    const size_t stat_bytes = bf16 ? (size_t)H * kStatChunks * 3 * d * sizeof(uint16_t) : 0;     // a multiple of 256
    w.stat = o;
    o += stat_bytes;
    w.full = o;
    o += stat_bytes;
    w.nsum = o;
    o += round_up((size_t)H * (w.Lpad / 256) * sizeof(double), 256);
    w.ext = o;
    o += (size_t)H * w.Lpad * (use_large(bf16, L) ? sizeof(uint4) : sizeof(uint2));
    w.kc = o;
    if (bf16) o += round_up((size_t)H * L * d * 2, 256);
    w.acc = o;
    o += round_up((size_t)H * w.Lpad * sizeof(unsigned long long), 256);
    w.total = o;
    return w;
}

size_t density_workspace_bytes(int H, int L, int d, bool bf16) { return density_layout(H, L, d, bf16).total; }
size_t density_estimate_offset() { return kDensityFlagBytes; }

static PrepWs prep_pointers(const DensityWs &w, char *base, bool large)
{
    PrepWs p;
    p.flag = reinterpret_cast<int *>(base);
    p.est = reinterpret_cast<float *>(base + w.est);
    p.scale = reinterpret_cast<float *>(base + w.scale);
    p.kbase = reinterpret_cast<const void **>(base + w.kbase);
    p.cand = reinterpret_cast<int *>(base + w.cand);
    p.stat = reinterpret_cast<uint16_t *>(base + w.stat);
    p.full = reinterpret_cast<uint16_t *>(base + w.full);
    p.nsum = reinterpret_cast<double *>(base + w.nsum);
    p.ext = base + w.ext;
    p.Kc = base + w.kc;
    p.acc = reinterpret_cast<unsigned long long *>(base + w.acc);
    p.large = large;
    return p;
}

template <bool kBf16, int D>
static void run_prep(const void *K, int H, int L, const float *sigma_host, const DensityWs &w, const PrepWs &p, hipStream_t st)
{
    if constexpr (kBf16) {
        for (int pass = 0; pass < 2; ++pass)
            for (int h0 = 0; h0 < H; h0 += 32768) {      // grid.y is 16 bits wide
                const int nh = (H - h0 < 32768) ? H - h0 : 32768;
                const size_t so = (size_t)h0 * kStatChunks * 3 * D;
                hipLaunchKernelGGL((density_stats<D>), dim3(kStatChunks, nh), dim3(256), 0, st,
                                   reinterpret_cast<const uint16_t *>(K) + (size_t)h0 * L * D, p.stat + so, p.full + so, L,
                                   pass, p.cand + h0);
            }
    }
    for (int h0 = 0; h0 < H; h0 += 256) {
        const int nh = (H - h0 < 256) ? H - h0 : 256;
        ScaleChunk sc;
        for (int i = 0; i < 256; ++i) {
            // exponent scale log2(e)/sigma^2, so the sweep can use the hardware exp2
            const double sg = (i < nh) ? (double)sigma_host[h0 + i] : 1.0;
            sc.s[i] = (float)(1.4426950408889634 / (sg * sg));
        }
        hipLaunchKernelGGL((density_prep<kBf16, D>), dim3(w.Lpad / 256, nh), dim3(256), 0, st, K, p, sc, h0, L, w.Lpad);
    }
}

template <bool kBf16, int D>
static hipError_t run(const void *K, int H, int L, const float *sigma_host, float *rho, void *ws, hipStream_t st)
{
    const DensityWs w = density_layout(H, L, D, kBf16);
    const bool large = use_large(kBf16, L);
    const PrepWs p = prep_pointers(w, reinterpret_cast<char *>(ws), large);
    run_prep<kBf16, D>(K, H, L, sigma_host, w, p, st);
    const int bm = large ? kSymBm : kSmallBm;
    const int nB = large ? w.Lpad / bm : (L + bm - 1) / bm, nBoth = (nB - 1) / 2;
    const int nblk = 1 + nBoth + ((nB > 1 && (nB & 1) == 0) ? 1 : 0);
    const int cus = current_chip().cus;
    for (int h0 = 0; h0 < H; h0 += kSymChunkHeads) {
        const int nh = (H - h0 < kSymChunkHeads) ? H - h0 : kSymChunkHeads;
        const long long wgs = (long long)nh * nB;
        if (wgs > 0x7FFFFFFFLL) return hipErrorInvalidValue;
        const int per_cu = (large ? D == 128 : D == 128 && !kBf16) ? 2 : 3;      // as the kernels' waves_per_eu
        const int parts = large ? split_parts(wgs, nblk, (long long)cus * per_cu, 0.35)
                                : split_parts(wgs, nblk * (kSmallBm / kSmallSc), (long long)cus * per_cu, 2.0);
        const int total = (int)(wgs * parts);
        if (!large)
            hipLaunchKernelGGL((density_sym_small<!kBf16, D>), dim3(total), dim3(256), 0, st, p.kbase,
                               reinterpret_cast<const uint2 *>(p.ext), p.scale, p.acc, L, w.Lpad, nB, nBoth, nblk, parts, h0,
                               total);
        else if constexpr (kBf16)
            hipLaunchKernelGGL(density_sym<D>, dim3(total), dim3(256), 0, st, p.kbase, reinterpret_cast<const uint4 *>(p.ext),
                               p.scale, p.acc, L, w.Lpad, nB, nBoth, nblk, parts, h0, total);
        hipLaunchKernelGGL(density_finish, dim3((L + 255) / 256, nh), dim3(256), 0, st, p, rho, L, w.Lpad, h0);
    }
    return hipGetLastError();
}

hipError_t launch_density(const void *K, bool bf16, int H, int L, int d, const float *sigma_host, float *rho,
                          void *ws, hipStream_t st)
{
    if (d == 64) return (bf16 ? run<true, 64> : run<false, 64>)(K, H, L, sigma_host, rho, ws, st);
    if (d == 128) return (bf16 ? run<true, 128> : run<false, 128>)(K, H, L, sigma_host, rho, ws, st);
    return hipErrorInvalidValue;
}

}  // namespace ws
