// Matrix-core path of the sparse ternary GEMM  Y = X W + b  (Eq. 1 of the paper), from the row sets of the K-blocked
// device form (tcsc_layout_t).
//
// Arithmetic.  A float is cut, without rounding, into three bf16 numbers: the top 8 bits of its significand, the next 8
// and the last 8 (x = hi + mid + lo).  A ternary weight is a bf16 number as it is, so every product of the three
// matrix products hi W, mid W, lo W is exact and the matrix cores add them in fp32; hi W has sums of its own, mid W and
// lo W share a second set, which is 2^8 smaller, so that what is rounded off there does not count.  No bit of X is
// lost.  Measured error against 64 bits (2-norm of the difference over 2-norm of the result): 6e-8 on M = 4096,
// K = N = 8192, where one fp32 sum over a list gives 1.1e-6; 5e-8 .. 8e-8 on every shape from K = 512 to 16384 (lists:
// 9e-8 .. 5e-7).  X goes in times 2^24, so that the pieces of the smallest floats are bf16 numbers too, and a weight is
// 2.0 with its sign (one bit beside the sign bit); sums leave times 2^-25, exactly.  A scaled sum that is not finite --
// X held an infinity, a NaN or something beyond about 2^100 -- is taken again from X by sums_of_any(), which keeps such
// entries apart, so an entry of X under a zero weight never reaches Y here either.
//
// k_matrix is for M > 8, k_waves for those of its calls whose tiles are few or K long for them, k_rows for M <= 10; choose_tile(), with_digits(), rows_plan()
// and matrix_plan() have the rules, with what was measured.  k_matrix also multiplies X cut into 6-bit digits by k_digits beforehand, where a call is large enough.
#include <cmath>
#include <type_traits>

#include "tstgemm_internal.h"

namespace tst {
namespace {

typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef float float32v __attribute__((ext_vector_type(32)));
typedef int int4v __attribute__((ext_vector_type(4)));
typedef int int8v __attribute__((ext_vector_type(8)));
typedef unsigned uint2v __attribute__((ext_vector_type(2)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));
typedef unsigned uint6v __attribute__((ext_vector_type(6)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr float kScaleUp = 16777216.f;            // 2^24
constexpr float kScaleDown = 1.f / 33554432.f;    // 2^-25
constexpr float kLarge = 18446744073709551616.f;  // 2^64
constexpr int kRawBuffer = 0x00020000;            // descriptor word 3: plain bytes; reads beyond num_records give zero

__device__ __forceinline__ bool finite(float v) { return fabsf(v) < __builtin_inff(); }

// The top halves of two floats as a pair of bf16 numbers (cut off, not rounded).
__device__ __forceinline__ unsigned top_halves(float x0, float x1)
{
    return __builtin_amdgcn_perm(__float_as_uint(x1), __float_as_uint(x0), 0x07060302u);
}
// What is left of a float below its top half (exact).
__device__ __forceinline__ float below_top(float x) { return x - __uint_as_float(__float_as_uint(x) & 0xffff0000u); }

// 32 rows of a column (one half of a pair of row sets) as weights for the matrix cores.  A dword of a fragment holds the
// weights of rows j (low half) and j + 16: bit 14 / 30 says non-zero (as bf16: 2.0), bit 15 / 31 is the sign.  `even` and
// `odd` hold these two bits side by side for all even / odd j, so a dword is one shift and one AND.
struct SignedWord {
    unsigned even, odd;
    __device__ __forceinline__ SignedWord(unsigned pos, unsigned neg)
    {
        const unsigned nz = pos | neg;
        even = (nz & 0x55555555u) | ((neg << 1) & 0xAAAAAAAAu);
        odd = ((nz >> 1) & 0x55555555u) | (neg & 0xAAAAAAAAu);
    }
    // rows j0 .. j0 + 3 and j0 + 16 .. j0 + 19 (j0 = 0, 4, 8 or 12)
    __device__ __forceinline__ bf16x8 eight(int j0) const
    {
        uint4v r;
        r[0] = (even << (14 - j0)) & 0xC000C000u;
        r[1] = (odd << (14 - j0)) & 0xC000C000u;
        r[2] = (even << (12 - j0)) & 0xC000C000u;
        r[3] = (odd << (12 - j0)) & 0xC000C000u;
        return __builtin_bit_cast(bf16x8, r);
    }
};

// A byte of two fp4 weights as a dword of two bf16 weights, the low half first.  One conversion, as long as any vector instruction, where
// SignedWord takes a shift and an AND: 27 instructions for 32 rows through FourBitWord in place of 38.
__device__ __forceinline__ unsigned two_weights(unsigned fours, int byte)
{
    switch (byte) {   // (known to the compiler)
    case 0: return __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(fours, 1.f, 0));
    case 1: return __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(fours, 1.f, 1));
    case 2: return __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(fours, 1.f, 2));
    default: return __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(fours, 1.f, 3));
    }
}

// 32 rows of a column as fp4 weights, 2.0 with its sign: bit 2 of four says non-zero, bit 3 is the sign.
struct FourBitWord {
    int4v w;   // dword d: rows 4 n + d
    __device__ __forceinline__ FourBitWord(unsigned pos, unsigned neg)
    {
        const unsigned nz = pos | neg;
        const unsigned even = (nz & 0x55555555u) | ((neg << 1) & 0xAAAAAAAAu);
        const unsigned odd = ((nz >> 1) & 0x55555555u) | (neg & 0xAAAAAAAAu);
        w[0] = (int)((even << 2) & 0xCCCCCCCCu);
        w[1] = (int)((odd << 2) & 0xCCCCCCCCu);
        w[2] = (int)(even & 0xCCCCCCCCu);
        w[3] = (int)(odd & 0xCCCCCCCCu);
    }
    // rows 8 part .. + 7 as bf16 weights: rows d and d + 4 of them in dword d
    __device__ __forceinline__ bf16x8 eight(int part) const
    {
        return __builtin_bit_cast(bf16x8, uint4v{two_weights((unsigned)w[0], part), two_weights((unsigned)w[1], part),
                                                  two_weights((unsigned)w[2], part), two_weights((unsigned)w[3], part)});
    }
};

__device__ __forceinline__ uint4v load16(__amdgpu_buffer_rsrc_t buf, unsigned offset)
{
    return __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(buf, (int)offset, 0, 0));
}

constexpr unsigned kNowhere = 0xffffff00u;   // an offset beyond every buffer: reads as zero, stores nothing
// K and N of a call are at most this (offsets_fit()), so an offset inside a tile of X, Y or partial sums is far below kNowhere.
constexpr int kMaxExtent = 1 << 22;

// A descriptor over `bytes` from p on (at most up to kNowhere; none for a null pointer).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_buffer(const void *p, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0,
                                             p == nullptr ? 0 : (int)(unsigned)min(bytes, (size_t)kNowhere), kRawBuffer);
}
// Cache bits of a buffer store (sc0, sc1): written through the L2.  What a kernel leaves there dirty is written back when it
// ends, before the next one starts; 16 MB of Y written through save 2 us (1024 x 1024 x 4096: 22.9 -> 20.9 us;
// 4096 x 1024 x 8192: 149 -> 142), partial sums 1 to 3 % of a sliced call.
constexpr int kWriteThrough = 17;

// Bias and PReLU of columns, requested before the sums are there; zero for columns >= N and without a bias.
struct Epilogue {
    __amdgpu_buffer_rsrc_t bias, slope;
    int alpha_stride;
    bool prelu;
    __device__ __forceinline__ Epilogue(const float *b, const float *alpha, int stride, int N)
        : bias(raw_buffer(b, (size_t)N * 4)), slope(raw_buffer(alpha, stride ? (size_t)N * 4 : 4)), alpha_stride(stride),
          prelu(alpha != nullptr) {}
    __device__ __forceinline__ float bias_of(int n) const
    {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(bias, n * 4, 0, 0));
    }
    __device__ __forceinline__ float slope_of(int n) const
    {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(slope, n * 4 * alpha_stride, 0, 0));
    }
    __device__ __forceinline__ float operator()(float v, float bias_n, float slope_n) const
    {
        v += bias_n;
        return prelu && !(v > 0.f) ? slope_n * v : v;
    }
};

// X W for 16 x 16 NB outputs over blocks of rows of W whatever X holds: what k_matrix, k_waves and k_rows do again for outputs whose
// scaled sums are not finite.  X is split by size: entries below 2^64 go in times 2^24 as everywhere, larger ones times
// 2^-24 (2^22 of the largest floats do not overflow so), and infinities and NaNs as ones in two planes of their own (a NaN in
// both), multiplied by the +1 rows and by the -1 rows, which counts the members that push a sum up and those that push it
// down.  Bound by cutting X, which every 16 NB columns do anew, and by the latency of its loads.  Single calls with one
// infinity (with one in every row; with all of X near 1e35), 50 % non-zeros, against the list and row-set kernels, whose time
// does not depend on X: 256 x 4096 x 4096 (k_waves, NB = 2) 82 us (124; 207) against 108, 1024 x 2048 x 8192 222 (565; 881) against 359,
// M = 1, 4096 x 4096 12 (12; 20) against 11; finite X 28, 82, 7.  One lane per output that walked the members one by one
// took 1128 (1630), 442 (9361) and 263, and 508 from the base-3 codes (M = 1, 4096 x 4096, one entry of 1e35; 12 now, from the
// row sets, which the codes are built from and uploaded with).  Where K is not a multiple of 64 the first entries of a row also meet the zero
// weights beyond the end of the row before, so an infinity there sends that row here too.
// X: the first of `rows` <= 16 rows; the blocks from kb0 on up to kb1, groups of four of them, every `stride`-th from
// `first` on.  Lane l holds column n[i] = n0 + l % 16 of Y for the i-th 16 columns, element e of v[i] is row 4 (l / 16) + e.
template <int NB>
__device__ __forceinline__ void sums_of_any(float4v (&v)[NB], const float *X, int rows, int K, const uint4v *masks, int n_pad,
                                            const int (&n)[NB], int kb0, int kb1, int first, int stride)
{
    const int r = threadIdx.x & 15, g = (threadIdx.x >> 4) & 3;
    const __amdgpu_buffer_rsrc_t xbuf = raw_buffer(X, (size_t)rows * K * 4);
    float4v top[NB], low[NB], large[NB], up[NB], down[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) top[b] = low[b] = large[b] = up[b] = down[b] = float4v{0.f, 0.f, 0.f, 0.f};
    auto multiply = [](float4v &c, uint4v a, bf16x8 b) {
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), b, c, 0, 0, 0);
    };
    for (int group = first; kb0 + 4 * group < kb1; group += stride) {
        const int kb = kb0 + 4 * group + g;
        uint4v w[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) w[b] = kb < kb1 ? masks[(size_t)kb * n_pad + n[b]] : uint4v{0, 0, 0, 0};
        for (int h = 0; h < 2; ++h) {
            unsigned plus[NB], minus[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                plus[b] = h ? w[b][1] : w[b][0];
                minus[b] = h ? w[b][3] : w[b][2];
            }
            const unsigned off = r < rows ? ((unsigned)r * (unsigned)K + 64u * kb + 32u * h) * 4u : kNowhere;
            float4v x0[4], x1[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                x0[s] = __builtin_bit_cast(float4v, load16(xbuf, r < rows ? off + 16 * s : off));
                x1[s] = __builtin_bit_cast(float4v, load16(xbuf, r < rows ? off + 16 * s + 64 : off));
            }
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                bf16x8 bw[NB];
#pragma unroll
                for (int b = 0; b < NB; ++b) bw[b] = SignedWord(plus[b], minus[b]).eight(4 * s);
                uint4v hi, mid, lo;
                auto cut = [&](int e, float a0, float a1) {
                    hi[e] = top_halves(a0, a1);
                    a0 = below_top(a0);
                    a1 = below_top(a1);
                    mid[e] = top_halves(a0, a1);
                    lo[e] = top_halves(below_top(a0), below_top(a1));
                };
                bool rest = false;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool small0 = fabsf(x0[s][e]) < kLarge, small1 = fabsf(x1[s][e]) < kLarge;
                    rest |= !small0 || !small1;
                    cut(e, small0 ? x0[s][e] * kScaleUp : 0.f, small1 ? x1[s][e] * kScaleUp : 0.f);
                }
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    multiply(top[b], hi, bw[b]);
                    multiply(low[b], mid, bw[b]);
                    multiply(low[b], lo, bw[b]);
                }
                if (!__any(rest)) continue;
                uint4v plus_inf, minus_inf;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float a[2] = {x0[s][e], x1[s][e]};
                    float big[2];
                    plus_inf[e] = minus_inf[e] = 0;
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        big[i] = finite(a[i]) && !(fabsf(a[i]) < kLarge) ? a[i] * (1.f / kScaleUp) : 0.f;
                        plus_inf[e] |= !(a[i] < __builtin_inff()) ? 0x3f80u << (16 * i) : 0u;      // bf16 1.0
                        minus_inf[e] |= !(a[i] > -__builtin_inff()) ? 0x3f80u << (16 * i) : 0u;
                    }
                    cut(e, big[0], big[1]);
                }
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    multiply(large[b], hi, bw[b]);
                    multiply(large[b], mid, bw[b]);
                    multiply(large[b], lo, bw[b]);
                    const bf16x8 pw = SignedWord(plus[b], 0).eight(4 * s), mw = SignedWord(minus[b], 0).eight(4 * s);
                    multiply(up[b], plus_inf, pw);
                    multiply(up[b], minus_inf, mw);
                    multiply(down[b], plus_inf, mw);
                    multiply(down[b], minus_inf, pw);
                }
            }
        }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[b][e] = (top[b][e] + low[b][e]) * kScaleDown + large[b][e] * (0.5f * kScaleUp);
            if (up[b][e] > 0.f || down[b][e] > 0.f)
                v[b][e] = (up[b][e] > 0.f ? __builtin_inff() : 0.f) - (down[b][e] > 0.f ? __builtin_inff() : 0.f);
        }
}

struct MatrixArgs {
    const float *X;
    const uint4v *masks;             // [n_kblocks][n_pad] {+1 rows low, high, -1 rows low, high}; k_rows: or codes
    const uint4v *row_sets;          // the masks also where the call is on the codes, [n_row_blocks][n_pad]
    const float *b, *alpha;
    float *Y, *partials;             // partials[slice][M][n_pad]
    const char *digits;              // k_matrix with X cut beforehand: units of 64 rows x 64 entries, [row tile][K-block] ...
    const unsigned char *counts;     // ... and how many planes of digits each has
    int alpha_stride;
    int M, K, N, n_pad, n_kblocks, n_row_blocks;
    int n_tiles, k_slices, kb_per_slice;
};

// ------------------------------------------------------------------------------------------------------------------
// X in digits.  32 entries of a row share an exponent (that of the largest, E); an entry is a sum of 6-bit floats (e2m3, the
// matrix cores' fp6), each the nearest to what the ones before it leave.  Digit j is a multiple of 2^(E - 4 - 5 j + (j != 0)),
// so three planes of digits hold 14 bits below the largest entry, five 24 and seven 34.  A unit of 64 rows x 64 entries has as
// many of these as leave nothing of any entry, three, five or seven (integers and 16-bit activations mostly three or five,
// uniform X five).  No bit of X is lost: a unit that seven do not hold -- entries with bits below 2^-33 of the largest of their 32, as
// normal X has in nearly every unit, infinities, NaNs, exponents out of range -- is marked
// kNoDigits, and its tile is multiplied in bf16 planes.  The sums of planes 0 to 2 and of the others are kept apart: the
// upper ones are whole numbers of a unit, exact as long as they have 24 bits, so the result is rounded little more than once
// (M = 4096, K = N = 8192: 3.6e-8 of the norm against 64 bits, in bf16 planes 6.1e-8).  fp6 x fp4 runs at 3.3 times the rate of
// bf16 under the power limit (instructions alone, on random operands: 6.4 and 1.93 PFLOP/s): five planes cost 0.5 of the three
// in bf16, seven 0.7.
// In the workspace a unit is [planes 0-2][exponents][planes 3-4][planes 5-6], a plane two fragments (32 rows) as a wavefront
// holds them: lane l has row l % 32 and entries 32 (l / 32) .. + 31, 16 bytes of each lane, then 8.
constexpr int kPlaneBytes = 2 * 64 * 24, kExponents = 3 * kPlaneBytes, kUpperPlanes = 10240, kUnitBytes = 22528;
constexpr int kNoDigits = 8;
constexpr int kMaxDigitBlocks = 1984;   // K-blocks whose counts k_matrix keeps in the LDS
__host__ __device__ constexpr int plane_offset(int j) { return j < 3 ? j * kPlaneBytes : kUpperPlanes + (j - 3) * kPlaneBytes; }
// Exponent of plane j's digits below plane 0's: in steps of 5, but 4 to plane 1 (the top digit of the largest entry, 2 to 4
// units of its plane, is rounded to a quarter)
__host__ __device__ constexpr int plane_shift(int j) { return j == 0 ? 0 : 5 * j - 1; }

// k_digits: one lane cuts 32 entries of a row, a workgroup up to kRun units of a tile one after the other.  Position 8 d + n of a
// lane's digits is entry 4 n + d, the order in which FourBitWord spreads the weights.  Bound by memory where X is held (134 MB of X
// and 130 MB of planes in 44 us, 6 TB/s; 57 us with every lane reading its own 128 bytes and the planes left to the L2).  Where it
// is not, a run ends at the first unit that says so: 4096 x 8192 x 8192 with normal X 1087 us with runs of one unit, 1070 of
// eight (1064 without k_digits); with uniform X no difference there, and 1 to 4 % more on calls of 1024 to 2048 rows.
constexpr int kRun = 8;
__host__ __device__ constexpr int digit_runs(int n_kblocks) { return (n_kblocks + kRun - 1) / kRun; }
__global__ void __launch_bounds__(128)
k_digits(const float *X, int M, int K, int n_kblocks, char *units, unsigned char *counts)
{
    __shared__ uint4v staged[2][32 * 17];   // (17 units a row: other banks)
    __shared__ int need[2][2];
    const int lane = threadIdx.x & 63, frag = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_runs = digit_runs(n_kblocks), tile = blockIdx.x / n_runs;
    const int first = blockIdx.x % n_runs * kRun, last = min(first + kRun, n_kblocks);
    const int rows = min(64, M - 64 * tile);
    const __amdgpu_buffer_rsrc_t xbuf = raw_buffer(X + (size_t)64 * tile * K, (size_t)rows * K * 4);
    uint4v *mine = staged[frag];
    for (int kb = first; kb < last; ++kb) {
        const int k0 = 64 * kb + 32 * (lane >> 5);
        // four rows of 256 bytes at a time, through the LDS to the lane that cuts them
        uint4v v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int row = 32 * frag + 4 * j + (lane >> 4);
            v[j] = load16(xbuf, row < rows ? ((unsigned)row * (unsigned)K + 64 * kb + 4 * (lane & 15)) * 4u : kNowhere);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) mine[(4 * j + (lane >> 4)) * 17 + (lane & 15)] = v[j];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the wavefront's own piece of the LDS
        float x[32];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float4v w = __builtin_bit_cast(float4v, mine[(lane & 31) * 17 + 8 * (lane >> 5) + j]);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[4 * j + e] = w[e];
        }
        if (64 * kb + 64 > K) {   // entries beyond the row belong to the next one
#pragma unroll
            for (int i = 0; i < 32; ++i) x[i] = k0 + i < K ? x[i] : 0.f;
        }
        float largest = 0.f;
#pragma unroll
        for (int i = 0; i < 32; ++i) largest = fmaxf(largest, fabsf(x[i]));
        const unsigned exponent = __float_as_uint(largest) >> 23;   // (a NaN shows in what is left over)
        const bool fits = largest == 0.f || (exponent >= 31 && exponent <= 230);
        const unsigned top = fits && largest != 0.f ? exponent - 1 : 126;   // of the unit of plane 0
        float16v a, b;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            a[i] = x[8 * (i & 3) + (i >> 2)];
            b[i] = x[8 * (i & 3) + 4 + (i >> 2)];
        }
        uint6v digit[7];
        int planes = 3;
#pragma unroll
        for (int j = 0; j < 7; ++j) {
            digit[j] = uint6v{0, 0, 0, 0, 0, 0};
            if (j >= planes) continue;
            const float scale = __uint_as_float((top - plane_shift(j)) << 23);
            digit[j] = __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(a, b, scale);
            const float32v back = __builtin_amdgcn_cvt_scalef32_pk32_f32_fp6(digit[j], scale);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                a[i] -= back[2 * i];
                b[i] -= back[2 * i + 1];
            }
            if (j != 2 && j != 4 && j != 6) continue;
            unsigned rest = 0;   // (a NaN is not zero either)
#pragma unroll
            for (int i = 0; i < 16; ++i) rest |= __float_as_uint(a[i]) | __float_as_uint(b[i]);
            if (__any((rest & 0x7fffffffu) != 0)) planes = j < 6 ? j + 3 : kNoDigits;
        }
        if (__any(!fits)) planes = kNoDigits;
        int *const needed = need[kb & 1];   // (the unit before may still be looking at its own)
        if (lane == 0) needed[frag] = planes;
        __syncthreads();
        planes = __builtin_amdgcn_readfirstlane(max(needed[0], needed[1]));
        const size_t unit = (size_t)tile * n_kblocks + kb;
        if (planes == kNoDigits) {   // the tile goes back to bf16 planes: the rest of the run is not looked at
            if ((int)threadIdx.x < last - kb) counts[unit + threadIdx.x] = kNoDigits;
            return;
        }
        if (threadIdx.x == 0) counts[unit] = (unsigned char)planes;
        const __amdgpu_buffer_rsrc_t out = raw_buffer(units + unit * kUnitBytes, kUnitBytes);
        // scales of planes 0 .. 3, times 2^24 as everywhere
        const unsigned e0 = top + 24;
        __builtin_amdgcn_raw_buffer_store_b32(
            e0 | (e0 - plane_shift(1)) << 8 | (e0 - plane_shift(2)) << 16 | (e0 - plane_shift(3)) << 24, out,
            kExponents + 256 * frag + 4 * lane, 0, kWriteThrough);
#pragma unroll
        for (int j = 0; j < 7; ++j) {
            if (j >= planes) break;
            const int at = plane_offset(j) + frag * (kPlaneBytes / 2);
            __builtin_amdgcn_raw_buffer_store_b128(uint4v{digit[j][0], digit[j][1], digit[j][2], digit[j][3]}, out, at + 16 * lane, 0,
                                                   kWriteThrough);
            __builtin_amdgcn_raw_buffer_store_b64(uint2v{digit[j][4], digit[j][5]}, out, at + 1024 + 8 * lane, 0, kWriteThrough);
        }
    }
}

// 1024 bytes from `buf` straight into the LDS, 16 per lane; counted by vmcnt, which the caller waits for.  (m0 is reserved: it cannot be
// named as clobbered, and the compiler sets it before each use of its own.)
__device__ __forceinline__ void copy_to_lds(uint4v buf, unsigned lds_byte, unsigned offset)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :: "s"(lds_byte), "v"(offset), "s"(buf) : "memory");
}
__device__ __forceinline__ uint4v descriptor(const void *p, size_t bytes)
{
    const unsigned long long a = (unsigned long long)p;
    const unsigned n = p == nullptr ? 0 : (unsigned)min(bytes, (size_t)kNowhere);
    return uint4v{(unsigned)__builtin_amdgcn_readfirstlane((int)a), (unsigned)__builtin_amdgcn_readfirstlane((int)(a >> 32)) & 0xffffu,
                  (unsigned)__builtin_amdgcn_readfirstlane((int)n), kRawBuffer};
}
template <int N> using Int = std::integral_constant<int, N>;

// ------------------------------------------------------------------------------------------------------------------
// k_matrix: a workgroup computes TM x TN of Y over one slice of K, WK groups of WM x WN wavefronts each over their
// share of the slice (their sums meet in the LDS at the end); a wavefront has RF x CF fragments of 32 x 32 (twice: hi,
// and mid + lo).  Per step of 32 rows of W a group cuts its TM x 32 floats of X into the three planes, in registers on
// their way from memory to the LDS (two buffers, one barrier a step); weights come straight from the row sets, 2 bits
// an entry, and are spread into fragments in registers.  Loads run PD steps ahead.  Per step a wavefront
// has 6 RF CF matrix instructions of 32 cycles; the cuts, the spreading and the LDS traffic are dealt over their six
// stages, each ended by a scheduling barrier (without the stages, and with loads whose number the compiler could not
// count, M = 4096, K = N = 8192 took 1.20 ms in place of 1.10).  In the 64 x 512 and 32 x 128 tiles a step has half as many
// pieces of X as the group has lanes: half of the wavefronts stage X, and the compiler puts their whole cut behind the guard
// of their LDS writes, into the last stage.
// Bound: long calls by the power limit (M = 4096, K = N = 8192: 1.04 ms, i.e. 1.59 PFLOP/s of bf16 products, the clock down
// to about 1.85 GHz; 4.4 ms for the lists at 50 % non-zeros, any density here; without any cutting and spreading, which
// gives wrong sums, it would take 0.99 ms), short ones by the start of the first loads, the
// sums at the end and the second launch where K is sliced (777 x 3001 x 2999 in three slices: 39.7 us, 8 of them the second launch).
// Calls with few tiles and K a multiple of 4 are k_waves's.
// DIGITS: X comes from the workspace, straight into the LDS, W too; three steps of 64 rows of W in a ring, copied two steps
// ahead, one barrier a step, placed before the last plane's products so that the next step's first reads are under way behind
// them.  A step has 4 products of 32 cycles per plane and wavefront.  Everything else is dealt between them one by one: all
// copies at once, or the spreading behind the products, cost 3 and 7 % of M = 4096, K = N = 8192 (1010 to 1045 us in bf16; here 580
// to 605 with five planes, 750 with seven, 530 with five at 1/16 non-zeros, where the products draw less power).  Of 587, k_digits takes 44, the four
// rounds' starts and ends about 30; the products by themselves take 430 at the power limit and 273 without it.  64 x 128
// of Y per wavefront, half the LDS reads, is no faster; a ring of four steps neither.
// Rows beyond M and rows of W beyond K: X reads as zero, or as the next row of X where the weights are zero.
template <int WK, int WM, int WN, int RF, int CF, bool DIGITS>
__global__ void __launch_bounds__(64 * WK * WM * WN, CF == 4 ? 1 : 2)
k_matrix(const MatrixArgs a)
{
    constexpr int NG = 64 * WM * WN, TM = 32 * RF * WM, TN = 32 * CF * WN, PD = 2;
    constexpr int kUnits = TM * 4 > NG ? TM * 4 / NG : 1;   // pieces of X (8 floats of a row) per lane and step
    static_assert(TM * 4 % NG == 0 || TM * 4 < NG, "units");
    static_assert(((size_t)TM + NG / 4 + 1) * kMaxExtent * 4 < kNowhere, "offsets inside a tile");
    constexpr int kChunk = TM + 2;                          // 16-byte units per plane and piece; + 2: other banks
    constexpr int kPlane = 4 * kChunk, kBuffer = 3 * kPlane;
    constexpr int kStageUnits = WK * 2 * kBuffer, kSumUnits = (WK / 2) * (TM * TN / 4);
    // digits: three steps of X and W per group, then the counts
    constexpr int kDigitStep = kUnitBytes + 512 * CF * WN, kDigitRing = 3 * kDigitStep, kDigitUnits = WK * (kDigitRing + 2048) / 16;
    constexpr int kBf16Units = kStageUnits > kSumUnits ? kStageUnits : kSumUnits;
    __shared__ uint4v lds_all[DIGITS && kDigitUnits > kBf16Units ? kDigitUnits : kBf16Units];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = wave / (WM * WN), wave_in_group = wave % (WM * WN);
    const int tid = wave_in_group * 64 + lane;
    const int wr = wave_in_group % WM, wc = wave_in_group / WM;
    const int l32 = lane & 31, g = lane >> 5;
    uint4v *lds = lds_all + group * (2 * kBuffer);

    // consecutive tiles of a row of tiles on one XCD: they read the same rows of X through one L2
    int id = blockIdx.x;
    const int per_xcd = gridDim.x / 8;
    if (id < 8 * per_xcd) id = (id & 7) * per_xcd + (id >> 3);
    const int slice = id % a.k_slices;
    id /= a.k_slices;
    const int m0 = id / a.n_tiles * TM, n0 = id % a.n_tiles * TN;
    int kb0 = slice * a.kb_per_slice, kb1 = min(kb0 + a.kb_per_slice, a.n_kblocks);
    const int blocks = (kb1 - kb0 + WK - 1) / WK;           // per group; the last ones may have fewer, or none
    kb0 += group * blocks;
    kb1 = min(kb0 + blocks, kb1);

    // The rows of the tile, and the row sets up to the end of the group's blocks: what lies beyond reads as zero.  No buffer
    // reaches beyond its tile, whatever M is
    const int rows = min(TM, a.M - m0);
    const __amdgpu_buffer_rsrc_t xbuf = raw_buffer(a.X + (size_t)m0 * a.K, (size_t)rows * a.K * 4);
    const __amdgpu_buffer_rsrc_t wbuf = raw_buffer(a.masks, (size_t)kb1 * a.n_pad * 16);
    unsigned xoff[kUnits], woff[CF];
    int unit[kUnits];
#pragma unroll
    for (int p = 0; p < kUnits; ++p) {
        const int q = tid + p * NG, c = q & 3, row = q >> 2;
        xoff[p] = ((unsigned)row * (unsigned)a.K + 4 * c) * 4u;
        unit[p] = c * kChunk + row;
    }
#pragma unroll
    for (int j = 0; j < CF; ++j) woff[j] = (unsigned)min(n0 + (wc * CF + j) * 32 + l32, a.n_pad - 1) * 16u;

    float4v xa[PD][kUnits], xb[PD][kUnits];
    uint4v w[2][CF];
    auto load_x = [&](int set, int step) {
#pragma unroll
        for (int p = 0; p < kUnits; ++p) {
            xa[set][p] = __builtin_bit_cast(float4v, load16(xbuf, xoff[p] + (unsigned)step * 128u));
            xb[set][p] = __builtin_bit_cast(float4v, load16(xbuf, xoff[p] + (unsigned)step * 128u + 64u));
        }
    };
    auto load_w = [&](int set, int kb) {
#pragma unroll
        for (int j = 0; j < CF; ++j) w[set][j] = load16(wbuf, woff[j] + (unsigned)kb * (unsigned)a.n_pad * 16u);
    };
    constexpr int kPairs = kUnits * 4;
    uint4v hi[kUnits], mid[kUnits], lo[kUnits];
    auto cut_pair = [&](int set, int i) {
        const int p = i >> 2, e = i & 3;
        float x0 = xa[set][p][e] * kScaleUp, x1 = xb[set][p][e] * kScaleUp;
        hi[p][e] = top_halves(x0, x1);
        x0 = below_top(x0);
        x1 = below_top(x1);
        mid[p][e] = top_halves(x0, x1);
        lo[p][e] = top_halves(below_top(x0), below_top(x1));
    };
    const bool stages_x = TM * 4 >= NG || tid < TM * 4;
    auto store_planes = [&](int buffer) {
        if (!stages_x) return;
#pragma unroll
        for (int p = 0; p < kUnits; ++p) {
            uint4v *dst = lds + buffer * kBuffer + unit[p];
            dst[0] = hi[p];
            dst[kPlane] = mid[p];
            dst[2 * kPlane] = lo[p];
        }
    };
    auto spread_w = [&](bf16x8 (&bw)[CF], int set, int t, int u) {
#pragma unroll
        for (int j = 0; j < CF; ++j) bw[j] = SignedWord(w[set][j][t] >> (4 * g), w[set][j][2 + t] >> (4 * g)).eight(8 * u);
    };

    int col0 = n0 + wc * CF * 32 + l32, row0 = wr * RF * 32 + 4 * g;
    const Epilogue finish(a.b, a.alpha, a.alpha_stride, a.N);
    float bias[CF], slope[CF];
#pragma unroll
    for (int j = 0; j < CF; ++j) {
        bias[j] = finish.bias_of(col0 + 32 * j);
        slope[j] = finish.slope_of(col0 + 32 * j);
    }

    float16v acc[2][RF][CF];   // [hi | mid + lo]
    auto merge = [&]() {
#pragma unroll
        for (int i = 0; i < RF; ++i)
#pragma unroll
            for (int j = 0; j < CF; ++j) acc[0][i][j] += acc[1][i][j];
    };
    auto clear = [&]() {
#pragma unroll
        for (int d = 0; d < 2; ++d)
#pragma unroll
            for (int i = 0; i < RF; ++i)
#pragma unroll
                for (int j = 0; j < CF; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[d][i][j][e] = 0.f;
    };

    bool in_digits = false;
    if constexpr (DIGITS) {
        static_assert(WM == 1 && RF == 2 && CF % 2 == 0, "a unit is the tile's rows, a wavefront's columns come 64 at a time");
        typedef __attribute__((address_space(3))) const char *Lds;
        constexpr int kChunks = kUnitBytes / 1024, kCopies = (kChunks + WN - 1) / WN, kLoads = kCopies + CF / 2;
        const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) uint4v *)lds_all;
        const unsigned ring = lds0 + group * kDigitRing;
        unsigned char *const counted = reinterpret_cast<unsigned char *>(lds_all) + WK * kDigitRing;   // of the slice's blocks
        int *const flags = reinterpret_cast<int *>(counted + kMaxDigitBlocks);
        const int slice_kb0 = slice * a.kb_per_slice, slice_blocks = min(a.kb_per_slice, a.n_kblocks - slice_kb0);
        const size_t tile_unit = (size_t)(m0 / 64) * a.n_kblocks;
        const uint4v dbuf = descriptor(a.digits + tile_unit * kUnitBytes, (size_t)kb1 * kUnitBytes);
        const uint4v sbuf = descriptor(a.masks, (size_t)kb1 * a.n_pad * 16);
        unsigned scol[CF / 2];
#pragma unroll
        for (int j = 0; j < CF / 2; ++j) scol[j] = (unsigned)min(n0 + wc * 32 * CF + 64 * j + lane, a.n_pad - 1) * 16u;
        auto copy_w = [&](int step, unsigned to) {   // W of the wavefront's columns
#pragma unroll
            for (int j = 0; j < CF / 2; ++j)
                copy_to_lds(sbuf, to + kUnitBytes + (wave_in_group * (CF / 2) + j) * 1024,
                            scol[j] + (unsigned)(kb0 + step) * (unsigned)a.n_pad * 16u);
        };
        // the wavefront's pieces of the group's X: from byte `piece` of a unit, where there are more planes than `above`
        unsigned piece[kCopies], lane_piece[kCopies];
        int above[kCopies];
#pragma unroll
        for (int i = 0; i < kCopies; ++i) {
            const int c = min(wave_in_group + i * WN, kChunks - 1);
            piece[i] = c * 1024;
            lane_piece[i] = c * 1024 + lane * 16;
            above[i] = c < 10 ? 0 : c < 16 ? 3 : 5;
        }
        auto copy_x = [&](int i, int step, unsigned to, int planes) {   // (0xffff0000 and what is added to it: beyond the buffer)
            copy_to_lds(dbuf, to + piece[i], (planes > above[i] ? (unsigned)(kb0 + step) * kUnitBytes : 0xffff0000u) + lane_piece[i]);
        };
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            copy_w(s, ring + s * kDigitStep);
#pragma unroll
            for (int i = 0; i < kCopies; ++i) copy_x(i, s, ring + s * kDigitStep, 7);
        }
        copy_w(2, ring + 2 * kDigitStep);
        bool wide = false;
        for (int i = threadIdx.x; i < WK * blocks + 4; i += 64 * WK * WN) {
            const unsigned char n = i < slice_blocks ? a.counts[tile_unit + slice_kb0 + i] : 3;
            counted[i] = n;
            wide |= n == kNoDigits;
        }
        if (__any(wide)) wide = true;
        if (lane == 0) flags[wave] = wide;
        __syncthreads();
        int any_wide = 0;
#pragma unroll
        for (int i = 0; i < WK * WN; ++i) any_wide |= flags[i];
        in_digits = !__builtin_amdgcn_readfirstlane(any_wide);
        if (in_digits) {
            clear();
            const unsigned char *const count = counted + group * blocks;
            int8v x[2][RF];
            int4v bw[2][CF];
            unsigned scale[2][RF], sets[CF][2];
            const unsigned lane16 = lane * 16, lane8 = 1024 + lane * 8, lane4 = kExponents + lane * 4;
            const unsigned lane_w = kUnitBytes + (wave_in_group * 32 * CF + l32) * 16 + g * 4;
            typedef __attribute__((address_space(3))) const unsigned *Words;
            auto read_scale = [&](unsigned (&to)[RF], unsigned at) {
                const Words p = (Words)(size_t)(at + lane4);
#pragma unroll
                for (int i = 0; i < RF; ++i) to[i] = p[64 * i];
            };
            auto read_x = [&](auto cur, unsigned at16, unsigned at8, int offset) {   // a plane's two fragments
#pragma unroll
                for (int i = 0; i < RF; ++i) {
                    const uint4v u = *(__attribute__((address_space(3))) const uint4v *)((Lds)(size_t)at16 + offset + i * (kPlaneBytes / 2));
                    const uint2v v = *(__attribute__((address_space(3))) const volatile uint2v *)((Lds)(size_t)at8 + offset + i * (kPlaneBytes / 2));
                    x[cur][i] = int8v{(int)u[0], (int)u[1], (int)u[2], (int)u[3], (int)v[0], (int)v[1], 0, 0};
                }
            };
            auto first_plane = [&](int planes) { return planes > 5 ? plane_offset(5) : planes > 3 ? plane_offset(3) : plane_offset(1); };
            auto read_w = [&](unsigned at) {
                const Words p = (Words)(size_t)(at + lane_w);
#pragma unroll
                for (int j = 0; j < CF; ++j) {
                    sets[j][0] = p[128 * j];
                    sets[j][1] = p[128 * j + 2];
                }
            };
            // a plane's products; between them, `between(k)` behind the k-th: a wavefront issues in order, and what it has to do
            // beside the products fits into the cycles they take
            auto multiply = [&](auto plane, auto cur, auto step, auto between) {
                constexpr int P = decltype(plane)::value, kByte = P < 4 ? P : P - 3, S = decltype(step)::value;
#pragma unroll
                for (int i = 0; i < RF; ++i) {
                    const int s = (int)(P < 4 ? scale[S][i] : scale[S][i] - 0x0F0F0F0Fu);
#pragma unroll
                    for (int j = 0; j < CF; ++j) {
                        float16v &c = acc[P < 3 ? 0 : 1][i][j];
                        const int4v b = bw[S][j];
                        const int8v w{b[0], b[1], b[2], b[3], 0, 0, 0, 0};
                        c = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(x[cur][i], w, c, 2, 4, kByte, s, 0, 127);
                        between(i * CF + j);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            };
            auto uniform = [](unsigned char n) { return __builtin_amdgcn_readfirstlane((int)n); };
            int planes = uniform(count[0]), planes1 = uniform(count[1]), planes2 = uniform(count[2]);
            unsigned char count3 = count[3];
            unsigned at = ring, next = ring + kDigitStep, third = ring + 2 * kDigitStep, at16 = at + lane16, at8 = at + lane8;
            asm volatile("s_waitcnt vmcnt(%0)" :: "n"(kLoads + CF / 2) : "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            read_w(at);
            read_scale(scale[0], at);
            {
                const int first = first_plane(planes);
                read_x(Int<0>{}, at16 + first, at8 + first, 0);
            }
#pragma unroll
            for (int j = 0; j < CF; ++j) bw[0][j] = FourBitWord(sets[j][0], sets[j][1]).w;
            constexpr int kProducts = RF * CF;
            // one step: x[A] holds its first plane, x[B] will hold the next step's; weights and exponents are in [A]
            auto step_of = [&](auto parity, int step) {
                constexpr int A = decltype(parity)::value, B = 1 - A;
                auto then_read = [&](auto cur, int offset) {
                    return [&, offset](int k) {
                        if (k == 0) read_x(decltype(cur){}, at16, at8, offset);
                    };
                };
                if (planes > 5) {
                    multiply(Int<5>{}, Int<A>{}, Int<A>{}, then_read(Int<B>{}, plane_offset(6)));
                    multiply(Int<6>{}, Int<B>{}, Int<A>{}, then_read(Int<A>{}, plane_offset(3)));
                }
                if (planes > 3) {
                    multiply(Int<3>{}, Int<A>{}, Int<A>{}, then_read(Int<B>{}, plane_offset(4)));
                    multiply(Int<4>{}, Int<B>{}, Int<A>{}, then_read(Int<A>{}, plane_offset(1)));
                }
                multiply(Int<1>{}, Int<A>{}, Int<A>{}, [&](int k) {
                    if (k == 0) read_x(Int<B>{}, at16, at8, plane_offset(2));
                    if (k == 1) {
                        asm volatile("s_waitcnt vmcnt(%0)" :: "n"(kLoads) : "memory");   // the next step's W, its own copy
                        read_w(next);
                    }
#pragma unroll
                    for (int i = 0; i < kCopies; ++i)
                        if (k >= 2 && k == 2 + i) copy_x(i, step + 2, third, planes2);
                });
                constexpr int kEarly = kCopies < kProducts - 2 ? kCopies : kProducts - 2;   // copies issued above
                multiply(Int<2>{}, Int<B>{}, Int<A>{}, [&](int k) {
                    if (k == 0) read_x(Int<A>{}, at16, at8, plane_offset(0));
#pragma unroll
                    for (int j = 0; j < CF; ++j)
                        if (k == 1 + j * (kProducts - 2) / CF) {
                            bw[B][j] = FourBitWord(sets[j][0], sets[j][1]).w;
                            asm volatile("" : "+v"(bw[B][j]));   // here, not where it is used first
                        }
#pragma unroll
                    for (int i = kEarly; i < kCopies; ++i)
                        if (k == kProducts - 1) copy_x(i, step + 2, third, planes2);
                });
                // the next step's X is there (every wavefront's part of it), and nobody needs this step's any more
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(kLoads) : "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                multiply(Int<0>{}, Int<A>{}, Int<A>{}, [&](int k) {
                    if (k == 0) {
                        const int first = first_plane(planes1);
                        read_x(Int<B>{}, next + lane16 + first, next + lane8 + first, 0);
                    }
                    if (k == 1) read_scale(scale[B], next);
                    if (k == 2) copy_w(step + 3, at);
                });
                planes = planes1;
                planes1 = planes2;
                planes2 = uniform(count3);
                count3 = count[step + 4];
                const unsigned free = at;
                at = next;
                next = third;
                third = free;
                at16 = at + lane16;
                at8 = at + lane8;
            };
            for (int i = 0; i < blocks; i += 2) {
                step_of(Int<0>{}, i);
                if (i + 1 < blocks) step_of(Int<1>{}, i + 1);
            }
            merge();
        }
        // nothing is on its way to the LDS any more
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    }
    if (!in_digits) {
        clear();
#pragma unroll
        for (int s = 0; s < PD; ++s) load_x(s, 2 * kb0 + s);
        load_w(0, kb0);
        load_w(1, kb0 + 1);
#pragma unroll
        for (int i = 0; i < kPairs; ++i) cut_pair(0, i);
        store_planes(0);
        load_x(0, 2 * kb0 + PD);
        bf16x8 bw[2][CF];
        spread_w(bw[0], 0, 0, 0);
        bf16x8 x[2][RF];
        auto read_x = [&](int t, int s) {   // stage s: plane s % 3 of 16 rows
#pragma unroll
            for (int i = 0; i < RF; ++i)
                x[s & 1][i] = __builtin_bit_cast(
                    bf16x8, lds[t * kBuffer + (s % 3) * kPlane + (2 * (s / 3) + g) * kChunk + (wr * RF + i) * 32 + l32]);
        };
        // The next step's planes are written, this step's have been read.  Only LDS traffic is waited for: the loads of the
        // coming steps stay in flight
        auto meet = [&]() {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        };
        // The wavefronts meet in front of a step's last products, which are under way meanwhile, or in front of its first.  Over 195 calls that 32 x 128
        // and 64 x 128 tiles get (K = 65 .. 2400 whole) the former is 2 and 1 % ahead on average, each call timed to 2 % (584 x 91 x 2085 6.05 -> 5.55 us,
        // 135 x 845 x 6476 10.1 -> 9.65, 2104 x 128 x 1621 7.45 -> 7.1; 603 x 579 x 2331 11.6 to 11.9 both ways; 1.3 %, 0.05 us, behind in calls of one step a
        // group that are bound by their start), in slices 1.5 % (20 calls), in 64 x 512 tiles up to 1 %.  The latter is 1 % ahead with four
        // groups of wavefronts, and in 64 x 256 tiles, two of which share a compute unit and fill each other's waits.
        constexpr bool kEarly = WK < 4 && !(CF == 2 && WK * WN == 4);
        constexpr int kCutStages = kEarly ? 4 : 5, kStore = kEarly ? 4 : 5, kSpread = kEarly ? 5 : 4;
        if (kEarly) {
            meet();
            read_x(0, 0);
        }
        for (int i0 = 0; i0 < blocks; i0 += 2) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (i0 + q >= blocks) break;
                const int kb = kb0 + i0 + q;
#pragma unroll
                for (int t = 0; t < 2; ++t) {   // half of the block: 32 rows of W, LDS buffer t
                    const int next = (t + 1) % PD;
                    if (!kEarly) {
                        meet();
                        read_x(t, 0);
                    }
#pragma unroll
                    for (int s = 0; s < 6; ++s) {
                        if (s < 5) {
                            read_x(t, s + 1);
                        } else if (kEarly) {
                            meet();
                            read_x(t ^ 1, 0);
                        }
#pragma unroll
                        for (int i = s * kPairs / kCutStages; i < (s + 1) * kPairs / kCutStages && i < kPairs; ++i) cut_pair(next, i);
                        if (s == 1) spread_w(bw[1], q, t, 1);
                        if (s == 4 && kSpread == 4) {
                            if (t == 1) load_w(q, kb + 2);
                            spread_w(bw[0], t ? q ^ 1 : q, t ^ 1, 0);
                        }
                        if (s == kStore) {
                            // (behind the last block this writes once more what nothing reads)
                            store_planes(t ^ 1);
                            load_x(next, 2 * kb + t + 1 + PD);
                        }
                        if (s == 5 && kSpread == 5) {
                            if (t == 1) load_w(q, kb + 2);
                            spread_w(bw[0], t ? q ^ 1 : q, t ^ 1, 0);
                        }
#pragma unroll
                        for (int i = 0; i < RF; ++i)
#pragma unroll
                            for (int j = 0; j < CF; ++j) {
                                float16v &c = acc[s % 3 ? 1 : 0][i][j];
                                c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[s & 1][i], bw[s / 3][j], c, 0, 0, 0);
                            }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
        }
        merge();
    }

    if constexpr (DIGITS) {   // (the two ways to the sums end here: what follows is not made twice)
#pragma unroll
        for (int i = 0; i < RF; ++i)
#pragma unroll
            for (int j = 0; j < CF; ++j) asm volatile("" : "+v"(acc[0][i][j]));
        asm volatile("" : "+v"(col0), "+v"(row0));
    }

    if constexpr (WK > 1) {   // sums of the groups: the upper half's into the lower half's, until one is left
        float *sums = reinterpret_cast<float *>(lds_all);
#pragma unroll
        for (int half = WK / 2; half >= 1; half /= 2) {
            __syncthreads();
            if (group >= half && group < 2 * half) {
                float *dst = sums + (size_t)(wave - half * WM * WN) * (RF * CF * 1024) + lane;
#pragma unroll
                for (int i = 0; i < RF; ++i)
#pragma unroll
                    for (int j = 0; j < CF; ++j)
#pragma unroll
                        for (int e = 0; e < 16; ++e) dst[((i * CF + j) * 16 + e) * 64] = acc[0][i][j][e];
            }
            __syncthreads();
            if (group < half) {
                const float *src = sums + (size_t)wave * (RF * CF * 1024) + lane;
#pragma unroll
                for (int i = 0; i < RF; ++i)
#pragma unroll
                    for (int j = 0; j < CF; ++j)
#pragma unroll
                        for (int e = 0; e < 16; ++e) acc[0][i][j][e] += src[((i * CF + j) * 16 + e) * 64];
            }
        }
        if (group > 0) return;
    }

    // element e of a fragment is row 8 (e / 4) + 4 g + e % 4, column l32.  The stores are range-checked (rows beyond M,
    // columns beyond the last): guarded by branches they waited for each other, 1.4 us of a short call
    auto row_of = [&](int i, int e) { return row0 + 32 * i + 8 * (e / 4) + e % 4; };
    const bool sliced = a.k_slices > 1;
    float *out = sliced ? a.partials + ((size_t)slice * a.M + m0) * a.n_pad : a.Y + (size_t)m0 * a.N;
    const int width = sliced ? a.n_pad : a.N;
    const __amdgpu_buffer_rsrc_t obuf = raw_buffer(out, (size_t)rows * width * 4);
    float spoilt = 0.f;   // NaN as soon as one sum is not finite
    auto store = [&](auto value) {
#pragma unroll
        for (int j = 0; j < CF; ++j) {
            const int n = col0 + 32 * j;
#pragma unroll
            for (int i = 0; i < RF; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    spoilt = fmaf(acc[0][i][j][e], 0.f, spoilt);
                    __builtin_amdgcn_raw_buffer_store_b32(
                        __float_as_uint(value(i, j, e)), obuf,
                        (int)(n < width ? ((unsigned)row_of(i, e) * (unsigned)width + n) * 4u : kNowhere), 0, kWriteThrough);
                }
        }
    };
    if (sliced) store([&](int i, int j, int e) { return acc[0][i][j][e] * kScaleDown; });
    else store([&](int i, int j, int e) { return finish(acc[0][i][j][e] * kScaleDown, bias[j], slope[j]); });
    if (!__any(spoilt != 0.f)) return;

    // Pieces of 16 x 16 with a value that is not finite: again, from X.  (The wavefront reads what its own lanes stored.)
    __threadfence();
    const int first_block = slice * a.kb_per_slice, end_block = min(first_block + a.kb_per_slice, a.n_kblocks);
    const int r16 = lane & 15, g16 = lane >> 4;
    for (int piece = 0; piece < 4 * RF * CF; ++piece) {
        const int row = wr * RF * 32 + 16 * (piece / (2 * CF)), n = n0 + wc * CF * 32 + 16 * (piece % (2 * CF)) + r16;
        if (row >= rows) break;
        bool bad[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int m = row + 4 * g16 + e;
            bad[e] = m < rows && n < width && !finite(out[(size_t)m * width + n]);
        }
        if (!__any(bad[0] || bad[1] || bad[2] || bad[3])) continue;
        float4v v[1];
        sums_of_any(v, a.X + (size_t)(m0 + row) * a.K, min(rows - row, 16), a.K, a.masks, a.n_pad, {min(n, a.n_pad - 1)}, first_block,
                    end_block, 0, 1);
        const float bias_n = finish.bias_of(n), slope_n = finish.slope_of(n);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (bad[e]) out[(size_t)(row + 4 * g16 + e) * width + n] = sliced ? v[0][e] : finish(v[0][e], bias_n, slope_n);
    }
}

// ------------------------------------------------------------------------------------------------------------------
// k_waves: Y in tiles of 32 x 32 CF, for calls that choose_tile() sends here: from one tile to about a thousand (672 x 1536 x 6528: 1071).  A workgroup is four wavefronts, each with the
// whole tile over a quarter of the workgroup's K: nothing is shared until the sums meet in the LDS at the end, so the loop has
// no barrier, and K is seldom cut into slices.  Per block of 64 rows of W a wavefront copies 32 x 64 floats of X and the row sets of its
// columns straight into a ring of two blocks in the LDS that is its own, the next block's while it is at this one; lane l cuts
// row l % 32, entries 32 (l / 32) .. + 31 of the block, in registers, and spreads that half of each row set.  12 CF matrix
// instructions of 32 cycles per block, the cuts and the spreading of the next 16 rows dealt between them one by one.
// Bound: a SIMD issues a vector instruction in 4.1 cycles beside a matrix instruction, which takes 8 of its own (measured), so a
// block is 48 x 8 + 366 x 4.1 cycles of issue for CF = 4 against 48 x 32 of products; with all compute units at it the power
// limit takes another fifth (2.2 us per block and pair of wavefronts, 1.65 on one compute unit alone, 1.8 for the products by
// themselves).  M = 256, K = N = 4096: 22.2 us, 28.2 as 64 x 256 tiles over four slices of K with a second launch for their sums;
// 64 x 16384 x 4096 24.6 (31.1), 32 x 4096 x 4096 9.2 (10.6), 768 x 1024 x 1024 8.3 (10.5), 512 x 512 x 512 4.9 (5.9).  Eight
// wavefronts a workgroup: 1 to 5 % slower; v_dot2_f32_bf16 for what a plane leaves: 64 instructions a block less, 15 % slower.
// The copies take 16 bytes a lane and want every row of X on such a border; calls whose K is not a multiple of 4 go to k_matrix.  Where X itself lies
// off the border (ON_BORDER false), X goes through registers instead, and the rest is the same, so that the order of a call's sums does not depend on where
// X lies: 7 % more on average over 75 calls, 16 % at most (256 x 4096 x 4096 22.3 -> 26.0 us, 29.4 in k_matrix; 12 x 1664 x 7104 8.3 -> 9.7, 9.3).  Copies of 4 bytes a lane
// in place of the registers: 22 %.
template <int CF, bool ON_BORDER>
__global__ void __launch_bounds__(256, 2)
k_waves(const MatrixArgs a)
{
    constexpr int KW = 4, TN = 32 * CF, kX = 8192, kSlot = kX + 16 * TN;   // a block in the ring: X, then row sets
    constexpr int kCopiesW = TN / 64, kCopies = kCopiesW + (ON_BORDER ? 8 : 0);
    static_assert(CF == 2 || CF == 4, "columns come 64 at a time");
    static_assert((32ull + 4) * kMaxExtent * 4 < kNowhere, "offsets inside a tile, two blocks beyond it");
    __shared__ uint4v lds[KW * 2 * kSlot / 16];
    typedef __attribute__((address_space(3))) const char *Lds;

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    // consecutive tiles of a row of tiles on one XCD, as in k_matrix
    int id = blockIdx.x;
    const int per_xcd = gridDim.x / 8;
    if (id < 8 * per_xcd) id = (id & 7) * per_xcd + (id >> 3);
    const int slice = id % a.k_slices;
    id /= a.k_slices;
    const int m0 = id / a.n_tiles * 32, n0 = id % a.n_tiles * TN, rows = min(32, a.M - m0);
    const int slice0 = slice * a.kb_per_slice, slice1 = min(slice0 + a.kb_per_slice, a.n_kblocks);
    const int blocks = (slice1 - slice0 + KW - 1) / KW, first = slice0 + wave * blocks, end = min(first + blocks, slice1);

    float16v acc[2][CF];   // [hi | mid + lo]
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int j = 0; j < CF; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[d][j][e] = 0.f;

    if (first < end) {   // (the last wavefronts may have no block)
        // Where the next block's copies come from.  A copy of X is four rows of 256 bytes (the last row again in place of those that do not
        // exist); piece c (16 bytes) of row r lies at place c ^ (r % 16) of its row, so that lanes with different rows read different banks.
        const uint4v xbuf = descriptor(a.X + (size_t)m0 * a.K, (size_t)rows * a.K * 4);
        const uint4v wbuf = descriptor(a.masks, (size_t)a.n_kblocks * a.n_pad * 16);
        unsigned from[kCopies];
#pragma unroll
        for (int i = 0; i < kCopiesW; ++i) from[i] = ((unsigned)first * (unsigned)a.n_pad + (unsigned)min(n0 + 64 * i + lane, a.n_pad - 1)) * 16u;
#pragma unroll
        for (int i = 0; kCopiesW + i < kCopies; ++i)
            from[kCopiesW + i] = (unsigned)min(4 * i + (lane >> 4), rows - 1) * (unsigned)a.K * 4u + (unsigned)first * 256u +
                                 16u * (unsigned)((lane & 15) ^ ((4 * i + (lane >> 4)) & 15));
        const unsigned ring = (unsigned)(size_t)(__attribute__((address_space(3))) uint4v *)lds + wave * (2 * kSlot);
        auto copy = [&](int i, unsigned slot) {
            copy_to_lds(i < kCopiesW ? wbuf : xbuf, ring + slot + (i < kCopiesW ? kX + 1024 * i : 1024 * (i - kCopiesW)), from[i]);
            from[i] += i < kCopiesW ? (unsigned)a.n_pad * 16u : 256u;   // (behind the last block: what nobody multiplies, or nothing)
        };
        // Off the border, four of the eight pieces at a time: requested, and two stages later written to where a copy would have put them.  (Rows
        // that do not exist read as zero.)
        const __amdgpu_buffer_rsrc_t xraw = raw_buffer(a.X + (size_t)m0 * a.K, (size_t)rows * a.K * 4);
        uint4v held[4];
        unsigned x_row = (unsigned)(lane >> 4) * (unsigned)a.K * 4u, x_piece = 16u * (unsigned)((lane & 15) ^ (lane >> 4)), x_block = (unsigned)first * 256u;
        auto request = [&](int half) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                unsigned piece = x_piece;
                asm volatile("" : "+v"(piece));   // here: four of them kept do not fit the registers
                held[i] = load16(xraw, (piece ^ 64u * i) + x_row + ((16u * half + 4u * i) * (unsigned)a.K * 4u + x_block));
            }
            if (half == 1) x_block += 256u;
        };
        auto put = [&](int half, unsigned slot) {
#pragma unroll
            for (int i = 0; i < 4; ++i) *(__attribute__((address_space(3))) uint4v *)(size_t)(ring + slot + 1024 * (4 * half + i) + 16 * lane) = held[i];
        };
        // What lies beyond the last row is not to look like a NaN of an earlier kernel, whether or not such a copy writes zeros.  It is in the
        // last block, at the last row and its repeats, and where blocks before used the place, entries of X are there already
        const int last = end - 1 - first;
        if (ON_BORDER && end == a.n_kblocks && a.K % 64 != 0 && last < 2) {
            for (int i = 16 * (rows - 1) + lane; i < kX / 16; i += 64) lds[(2 * wave + last) * (kSlot / 16) + i] = uint4v{0, 0, 0, 0};
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
#pragma unroll
        for (int i = 0; i < kCopies; ++i) copy(i, 0);
#pragma unroll
        for (int i = 0; i < kCopies; ++i) copy(i, kSlot);
        if (!ON_BORDER) {
            request(0);
            put(0, 0);
            request(1);
            put(1, 0);
            request(0);   // of the second block, which the first one's stages 0 and 1 put into the ring
            asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)" ::: "memory");
        }

        // Stage s of a block: rows 4 s .. + 3 and 16 + 4 s .. + 3 of each half.  [.][s % 2]: X as it is, its planes, weights
        float4v raw[2][2];
        uint4v planes[2][3], bw[2][CF];
        unsigned pos[CF], neg[CF], even[CF], odd[CF];
        Lds xat[4][2];
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int h = 0; h < 2; ++h) xat[s][h] = (Lds)(size_t)(ring + l32 * 256 + 16 * ((8 * g + 4 * h + s) ^ (l32 & 15)));
        const Lds wat = (Lds)(size_t)(ring + kX + l32 * 16 + g * 4);
        auto read_x = [&](int set, int s, unsigned slot) {
#pragma unroll
            for (int h = 0; h < 2; ++h) raw[set][h] = *(__attribute__((address_space(3))) const float4v *)(xat[s][h] + slot);
        };
        auto read_w = [&](unsigned slot) {
            const auto p = (__attribute__((address_space(3))) const unsigned *)(wat + slot);
#pragma unroll
            for (int j = 0; j < CF; ++j) {
                pos[j] = p[128 * j];
                neg[j] = p[128 * j + 2];
            }
        };
        auto words = [&](int j) {
            const SignedWord w(pos[j], neg[j]);
            even[j] = w.even;
            odd[j] = w.odd;
        };
        auto spread = [&](int set, int s, int d) {   // dword d % 4 of SignedWord::eight(4 s) for column d / 4
            bw[set][d / 4][d % 4] = ((d & 1 ? odd : even)[d / 4] << ((d & 2 ? 12 : 14) - 4 * s)) & 0xC000C000u;
        };
        float x0 = 0.f, x1 = 0.f;
        auto cut = [&](int set, int part) {   // plane part % 3 of pair part / 3
            if (part % 3 == 0) {
                x0 = raw[set][0][part / 3] * kScaleUp;
                x1 = raw[set][1][part / 3] * kScaleUp;
            } else {
                x0 = below_top(x0);
                x1 = below_top(x1);
            }
            planes[set][part % 3][part / 3] = top_halves(x0, x1);
        };
        auto stage = [&](auto number, unsigned at, unsigned other) __attribute__((always_inline)) {
            constexpr int S = decltype(number)::value, A = S % 2, B = 1 - A, kProducts = 3 * CF;
            if constexpr (!ON_BORDER && S == 0) {
                put(0, other);
                request(1);
            }
            // the next block is there; all of this one has been read, and makes room for the one after the next
            if constexpr (!ON_BORDER && S == 2) put(1, other);
            if constexpr (S == 2) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int q = 0; q < kProducts; ++q) {
                float16v &c = acc[q < CF ? 0 : 1][q % CF];
                c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, planes[A][q / CF]),
                                                            __builtin_bit_cast(bf16x8, bw[A][q % CF]), c, 0, 0, 0);
                if (q == 0) read_x(A, (S + 2) % 4, S < 2 ? at : other);
                if (S == 2 && q == 1) read_w(other);
                if (S == 2 && q >= 2) {
#pragma unroll
                    for (int i = (q - 2) * kCopies / (kProducts - 2); i < (q - 1) * kCopies / (kProducts - 2); ++i) copy(i, at);
                    if (!ON_BORDER && q == kProducts - 1) request(0);
                }
#pragma unroll
                for (int i = q * 12 / kProducts; i < (q + 1) * 12 / kProducts; ++i) cut(B, i);
#pragma unroll
                for (int d = q * (4 * CF) / kProducts; d < (q + 1) * (4 * CF) / kProducts; ++d) {
                    if (S == 3 && d % 4 == 0) words(d / 4);
                    spread(B, (S + 1) % 4, d);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto block = [&](unsigned at, unsigned other) __attribute__((always_inline)) {
            stage(Int<0>{}, at, other);
            stage(Int<1>{}, at, other);
            stage(Int<2>{}, at, other);
            stage(Int<3>{}, at, other);
        };
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"(kCopies) : "memory");
        read_w(0);
        read_x(0, 0, 0);
        read_x(1, 1, 0);
#pragma unroll
        for (int i = 0; i < 12; ++i) cut(0, i);
#pragma unroll
        for (int d = 0; d < 4 * CF; ++d) {
            if (d % 4 == 0) words(d / 4);
            spread(0, 0, d);
        }
        for (int kb = first; kb < end; kb += 2) {
            block(0, kSlot);
            if (kb + 1 < end) block(kSlot, 0);
        }
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // nothing is on its way to the LDS any more
    }

    // Sums of the wavefronts.  Those of hi stay apart from those of mid + lo until the end: they are whole numbers of a unit and mostly exact, so a
    // result is rounded little more than once, as in a kernel where one wavefront has all of K (300 x 832 x 5824 without a bias: 2.8e-8 of the
    // norm; joined in each wavefront first 4.7e-8).  It is 1.5 times the traffic here, 0.1 to 0.4 us a call (87 x 408 x 2435 4.9 -> 5.0 us, 196 x 868 x 3375
    // 8.25 -> 8.5, 256 x 4096 x 4096 23.0 -> 23.4).  Slices in 32 x 64 tiles are joined in each wavefront first: calls that have them had more slices, or as
    // many of tiles that joined as often, before there was this kernel.
    // Quad 4 j + q is elements 4 q .. of column fragment j, rows 8 q + 4 g .. + 3 of column 32 j + l32; a wavefront finishes CF quads from
    // quad0 on, 16 rows or all 32 of 32 columns, and gives the others away through its own ring.
    const bool sliced = a.k_slices > 1;
    const int quad0 = CF * (CF == 2 ? wave : 2 * (wave & 1) + (wave >> 1));
    const int row0 = 8 * (quad0 % 4), col0 = n0 + 32 * (quad0 / 4), n = col0 + l32;
    const Epilogue finish(a.b, a.alpha, a.alpha_stride, a.N);
    const float bias = finish.bias_of(n), slope = finish.slope_of(n);
    float4v *const sums = reinterpret_cast<float4v *>(lds);
    constexpr int kRing = 2 * kSlot / 16;
    const bool joined = CF == 2 && sliced;
    float4v mine[2][CF];   // [hi | mid + lo], or [all | zero]
#pragma unroll
    for (int i = 0; i < CF; ++i) mine[1][i] = float4v{0.f, 0.f, 0.f, 0.f};
    if (joined) {
#pragma unroll
        for (int j = 0; j < CF; ++j) acc[0][j] += acc[1][j];
    }
    auto quad = [&](int d, int i) {
        return float4v{acc[d][i / 4][4 * (i % 4)], acc[d][i / 4][4 * (i % 4) + 1], acc[d][i / 4][4 * (i % 4) + 2], acc[d][i / 4][4 * (i % 4) + 3]};
    };
    if constexpr (CF == 2) {
        static_assert(2 * 8 * 64 <= kRing, "a wavefront's sums in its ring");
        auto place = [&](int w, int d, int i) -> float4v & { return sums[w * kRing + (8 * d + i) * 64 + lane]; };
        auto give = [&](auto own) {
            constexpr int OWN = decltype(own)::value;
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                if (d == 1 && joined) break;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    if (i / 2 == OWN) mine[d][i % 2] = quad(d, i);
                    else place(wave, d, i) = quad(d, i);
                }
            }
        };
        if (wave == 0) give(Int<0>{});
        else if (wave == 1) give(Int<1>{});
        else if (wave == 2) give(Int<2>{});
        else give(Int<3>{});
        __syncthreads();
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            if (d == 1 && joined) break;
#pragma unroll
            for (int i = 0; i < 2; ++i)
                mine[d][i] = (mine[d][i] + place(wave ^ 1, d, quad0 + i)) + (place(wave ^ 2, d, quad0 + i) + place(wave ^ 3, d, quad0 + i));
        }
    } else {
        // three quarters of the sums do not fit the ring: half of the columns to w ^ 1, then half of what is kept to w ^ 2, through the ring
        // that this wavefront alone has read
        static_assert(2 * 8 * 64 <= kRing, "half of a wavefront's sums in its ring");
        float4v half[2][8];
        auto place = [&](int w, int d, int i) -> float4v & { return sums[w * kRing + (8 * d + i) * 64 + lane]; };
        auto give_half = [&](auto keep) {
            constexpr int KEEP = decltype(keep)::value;
#pragma unroll
            for (int d = 0; d < 2; ++d) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    place(wave, d, i) = quad(d, 8 * (1 - KEEP) + i);
                    half[d][i] = quad(d, 8 * KEEP + i);
                }
            }
        };
        auto give_quarter = [&](auto keep) {
            constexpr int KEEP = decltype(keep)::value;
#pragma unroll
            for (int d = 0; d < 2; ++d) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    place(wave ^ 1, d, i) = half[d][4 * (1 - KEEP) + i];
                    mine[d][i] = half[d][4 * KEEP + i];
                }
            }
        };
        if (wave & 1) give_half(Int<1>{});
        else give_half(Int<0>{});
        __syncthreads();
#pragma unroll
        for (int d = 0; d < 2; ++d)
#pragma unroll
            for (int i = 0; i < 8; ++i) half[d][i] += place(wave ^ 1, d, i);
        if (wave & 2) give_quarter(Int<1>{});
        else give_quarter(Int<0>{});
        __syncthreads();
#pragma unroll
        for (int d = 0; d < 2; ++d)
#pragma unroll
            for (int i = 0; i < 4; ++i) mine[d][i] += place(wave ^ 3, d, i);
    }
    float *out = sliced ? a.partials + ((size_t)slice * a.M + m0) * a.n_pad : a.Y + (size_t)m0 * a.N;
    const int width = sliced ? a.n_pad : a.N;
    const __amdgpu_buffer_rsrc_t obuf = raw_buffer(out, (size_t)rows * width * 4);
    float spoilt = 0.f;   // NaN as soon as one sum is not finite
#pragma unroll
    for (int q = 0; q < CF; ++q) {
        const float4v v = mine[0][q] + mine[1][q];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            spoilt = fmaf(v[e], 0.f, spoilt);
            const float y = v[e] * kScaleDown;
            const unsigned row = row0 + 8 * q + 4 * g + e;
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(sliced ? y : finish(y, bias, slope)), obuf,
                                                  (int)(n < width ? (row * (unsigned)width + n) * 4u : kNowhere), 0, kWriteThrough);
        }
    }
    if (!__any(spoilt != 0.f)) return;

    // again, from X, as in k_matrix, but 32 columns from one cut of X: K is whole here, and 16 at a time took longer than k_matrix in slices
    // (one infinity, 256 x 4096 x 4096: 116 us, so 82, there 88).  In k_matrix the registers would cost the tiles of 32 rows a wavefront a SIMD.
    __threadfence();
    const int r16 = lane & 15, g16 = lane >> 4;
    for (int row = row0; row < min(rows, row0 + 8 * CF); row += 16) {
        bool bad[2][4], any_bad = false;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int m = row + 4 * g16 + e, col = col0 + 16 * c + r16;
                bad[c][e] = m < rows && col < width && !finite(out[(size_t)m * width + col]);
                any_bad |= bad[c][e];
            }
        if (!__any(any_bad)) continue;
        float4v v[2];
        sums_of_any(v, a.X + (size_t)(m0 + row) * a.K, min(rows - row, 16), a.K, a.masks, a.n_pad,
                    {min(col0 + r16, a.n_pad - 1), min(col0 + 16 + r16, a.n_pad - 1)}, slice0, slice1, 0, 1);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int col = col0 + 16 * c + r16;
            const float bias_c = finish.bias_of(col), slope_c = finish.slope_of(col);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (bad[c][e]) out[(size_t)(row + 4 * g16 + e) * width + col] = sliced ? v[c][e] : finish(v[c][e], bias_c, slope_c);
        }
    }
}

// k_matrix_sum: Y = slice 0 + slice 1 + ... + b, then the optional PReLU; four columns per thread, all slices
// requested together and added in pairs (error of the norm 5.9e-8 where it was 6.6e-8 one after the other, seven slices).  Bias and slopes are requested
// with them: behind them they were a second trip to memory, 0.33 us (32 x 4096 x 4096 9.45 -> 9.1 us a call).  Bound by its launch and one trip to memory (4 slices of 256 x 4096: about 5 us).  Y is written through the
// L2 (512 x 4096 x 4096 41.0 -> 40.3 us a call, 777 x 3001 x 2999 41.3 -> 40.8; below 1 MB of Y no difference).
template <int S>
__global__ void __launch_bounds__(256)
k_matrix_sum(const MatrixArgs a)
{
    const int n = (blockIdx.x * 256 + threadIdx.x) * 4, m = blockIdx.y;
    if (n >= a.N) return;
    const float *P = a.partials + (size_t)m * a.n_pad + n;
    const size_t stride = (size_t)a.M * a.n_pad;
    float4v part[S];
#pragma unroll
    for (int s = 0; s < S; ++s) part[s] = *reinterpret_cast<const float4v *>(P + s * stride);
    const Epilogue finish(a.b, a.alpha, a.alpha_stride, a.N);   // (nothing beyond column N is read)
    float4v bias = __builtin_bit_cast(float4v, load16(finish.bias, n * 4u)), slope;
    if (a.alpha_stride) slope = __builtin_bit_cast(float4v, load16(finish.slope, n * 4u));
    else slope = float4v{1.f, 1.f, 1.f, 1.f} * finish.slope_of(0);
#pragma unroll
    for (int half = (S + 1) / 2, n_left = S; n_left > 1; n_left = half, half = (half + 1) / 2)
#pragma unroll
        for (int s = 0; s + half < n_left; ++s) part[s] += part[s + half];
    float4v y;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float v = part[0][i];
        if (!finite(v)) {   // on the way, or in all: again where slices of 2^128 do not overflow
            double sum = 0.0;
#pragma unroll 1
            for (int s = 0; s < S; ++s) sum += (double)P[s * stride + i];
            v = (float)sum;
        }
        y[i] = finish(v, bias[i], slope[i]);
    }
    float *dst = a.Y + (size_t)m * a.N + n;
    if (n + 4 <= a.N) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uint4v, y), raw_buffer(a.Y + (size_t)m * a.N, (size_t)a.N * 4), n * 4, 0,
                                               kWriteThrough);
    } else {
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (n + i < a.N) dst[i] = y[i];
    }
}

hipError_t launch_sum(const MatrixArgs &a, hipStream_t stream)
{
    const dim3 grid((a.N + 1023) / 1024, a.M), block(256);
    switch (a.k_slices) {
    case 2: hipLaunchKernelGGL(k_matrix_sum<2>, grid, block, 0, stream, a); break;
    case 3: hipLaunchKernelGGL(k_matrix_sum<3>, grid, block, 0, stream, a); break;
    case 4: hipLaunchKernelGGL(k_matrix_sum<4>, grid, block, 0, stream, a); break;
    case 5: hipLaunchKernelGGL(k_matrix_sum<5>, grid, block, 0, stream, a); break;
    case 6: hipLaunchKernelGGL(k_matrix_sum<6>, grid, block, 0, stream, a); break;
    case 7: hipLaunchKernelGGL(k_matrix_sum<7>, grid, block, 0, stream, a); break;
    case 8: hipLaunchKernelGGL(k_matrix_sum<8>, grid, block, 0, stream, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int CF>
hipError_t launch_waves(const MatrixArgs &a, long long m_tiles, const Call &c)
{
    const dim3 grid((unsigned)(m_tiles * a.n_tiles * a.k_slices)), block(256);
    if (reinterpret_cast<uintptr_t>(a.X) % 16 == 0) hipLaunchKernelGGL((k_waves<CF, true>), grid, block, 0, c.stream, a);
    else hipLaunchKernelGGL((k_waves<CF, false>), grid, block, 0, c.stream, a);
    return hipGetLastError();
}

template <int WK, int WM, int WN, int RF, int CF, bool DIGITS>
hipError_t launch_tiles(const MatrixArgs &a, long long m_tiles, const Call &c)
{
    hipLaunchKernelGGL((k_matrix<WK, WM, WN, RF, CF, DIGITS>), dim3((unsigned)(m_tiles * a.n_tiles * a.k_slices)),
                       dim3(64 * WK * WM * WN), 0, c.stream, a);
    return hipGetLastError();
}

// Tile and K slices of a call: the combination whose estimated time is least.  A workgroup takes `fixed` us and `step`
// us for each of its steps of 32 rows of W while its compute unit has time to spare, `work` us when the unit is full
// (per_cu workgroups at a time); a call takes kCall us more, slices kSlice us and 0.4 us per MB of partial sums; and no
// call is faster than `peak` operations per us, what the tile reaches on long calls under the power limit (64 x 512 against
// 64 x 256: M = 4096, K = N = 8192 1073 -> 1038 us, 2048 x 4096 x 4096 138 -> 132, 1024 x 2048 x 8192 74 -> 70).  Fitted to 13 tiles x 6 slice counts on 77
// shapes (M = 17 .. 2048, K and N = 512 .. 16384): the tile chosen among the last five of k_matrix is 2 % slower than the best of
// all on average, 16 % at worst.  The figures are high by some 5 % on long calls, in slices
// more; those of k_waves, which kLateRounds tells of, likewise.
struct TileShape {
    int rows, cols, groups, waves, per_cu;
    double fixed, step, work, peak;
};
constexpr TileShape kTiles[] = {
    {64, 512, 1, 8, 1, 1.90, 0.900, 0.900, 1.61e9},   // long and wide calls: X is cut half as often as by the next
    {64, 256, 1, 4, 2, 1.27, 0.578, 0.466, 1.55e9},   // two independent workgroups per unit fill each other's barriers
    {64, 256, 2, 8, 1, 2.15, 0.972, 0.972, 1.50e9},   // half the slices of that where rows x columns leave units idle
    {64, 128, 1, 4, 3, 0.31, 0.420, 0.311, 1.45e9},   // short K: little to start with
    {32, 64, 4, 8, 2, 0.65, 0.501, 0.461, 1.30e9},    // small Y
    {32, 128, 2, 8, 2, 0.34, 0.456, 0.383, 1.40e9},   // M <= 32
    {32, 64, 4, 4, 2, -0.45, 0.75, 0.370, 2.30e9},    // k_waves
    {32, 128, 4, 4, 2, 0.05, 1.20, 0.490, 1.28e9},
};
constexpr int kDigitTiles = 2;   // the first two can take X in digits
constexpr int kFirstOfWaves = 6;
// The last two are k_waves, whose copies of X need every row of X as far from a 16-byte border as the first; K of less than a block per
// wavefront leaves wavefronts without work.
bool waves_can(const tcsc_layout_t &l) { return l.K % 4 == 0 && l.n_kblocks >= 4; }
constexpr double kCall = 3.36, kSlice = 2.40, kSliceMb = 0.374;   // us, us, us per MB
// k_waves takes `fixed` us more than its workgroups, and a workgroup `step` us for its sums, which four wavefronts bring to the LDS, beside its steps,
// `work` us each; the workgroups of a compute unit share both.  With K whole and more tiles than two a compute unit nothing covers what is written last
// (kLateRounds, kLateMb, us per MB of Y).  Fitted to 771 timings of 415 shapes with K whole, with 515 others to test, 260 of them where slices are near (M = 11 ..
// 4000, K = 196 .. 16384, N = 64 .. 14000, the estimates of both kernels within 40 %): four of the 930 are more than 1.5 % behind k_matrix (2525 x 15832 x 157 and
// 500 x 7296 x 2705 6 %), and the choice is 0.7 % behind the best of all on average.  With `fixed` for a round of workgroups, as in k_matrix, 40 were, up to 13 %
// (246 x 256 x 6144 7.4 us, k_matrix 7.1 and 6.4; 640 x 256 x 1024 5.7, 5.0; 2943 x 2920 x 348 in three slices 28.4, 27.2), and without the late ones 192 x 4096 x 11008
// (516 tiles on 512 places 53.1 us, 48.6).
constexpr double kLateRounds = 1.04, kLateMb = 0.15;

struct TilePlan {
    int tile, k_slices;
    double us;
    bool digits = false;
};
// A tile of 64 rows in digits, and how many of them a call cuts at a time: as many as fit in `room`, evenly dealt.
size_t digit_tile_bytes(const tcsc_layout_t &l) { return (size_t)l.n_kblocks * (kUnitBytes + 1); }
long long digit_slab(const tcsc_layout_t &l, long long m_tiles, size_t room)
{
    long long fit = (long long)(room / digit_tile_bytes(l));
    const long long launch = 0xffffffffll / 128 / digit_runs(l.n_kblocks);   // threads of k_digits
    if (fit > launch) fit = launch;
    if (fit < 1 || fit >= m_tiles) return fit < 1 ? 0 : m_tiles;
    const long long slabs = (m_tiles + fit - 1) / fit;
    return (m_tiles + slabs - 1) / slabs;
}

// Whole numbers from x up, x >= 0 and below 2^62 (ceil() is a library call here, and the estimates make many).
inline double up(double x)
{
    const double whole = (double)(long long)x;
    return whole < x ? whole + 1.0 : whole;
}

// Digits in place of bf16 planes, on the tile and the slices of K chosen for those.  What X holds is not known here: if digits do
// not hold it, the cut is lost and the products are the same, so a call takes digits where what is lost is at most 2.5 % of it,
// 6 us per slab + 0.08 per million entries of X, and where slabs do not add rounds of workgroups.  Such calls are long and Y is wide,
// and X that digits hold gains far more.  us in bf16 with uniform and normal X, then in digits: M = 4096, K = N = 8192 1024 and 1033,
// 587 and 1034; 4096 x 4096 x 16384 1046 and 1057, 593 and 1068; 2048 x 8192 x 8192 502 and 508, 290 and 516; 1500 x 8192 x 8192 399
// and 404, 234 and 412.  Not taken (same two pairs): 4096 x 4096 x 4096 265 and 270, 171 and 278; 1024 x 4096 x 4096 74 and 75, 58
// and 81; 512 x 4096 x 4096 45 and 46, 46 and 51; up to 64 rows, where calls of that length have 10^9 weights, are not measured.
constexpr double kLost = 6.0, kLostMb = 0.08, kLostPart = 0.025;
// Where W is sparse enough for k_large to be near, the products draw less power and the bf16 planes, too, take 0.92 of the estimate,
// which then is what X that digits do not hold takes: M = 4096, K = N = 8192 at 1/16 non-zeros 955 us, k_large 928, digits 531; M =
// 2048 475, 473, 262.
constexpr double kSparsePart = 0.92;
TilePlan with_digits(const tcsc_layout_t &l, int M, size_t ws_bytes, const TilePlan &p)
{
    const double room = kLostPart * p.us - kLostMb * 1e-6 * M * l.K;
    if (p.tile >= kDigitTiles || M <= 64 || room < kLost) return p;
    const TileShape &s = kTiles[p.tile];
    const long long m_tiles = ((long long)M + 63) / 64, n_tiles = (l.n_pad + s.cols - 1) / s.cols;
    const size_t partial_bytes = p.k_slices > 1 ? (size_t)p.k_slices * M * l.n_pad * 4 : 0;
    if ((l.n_kblocks + p.k_slices - 1) / p.k_slices + 8 > kMaxDigitBlocks || partial_bytes >= ws_bytes) return p;
    const long long slab = digit_slab(l, m_tiles, ws_bytes - partial_bytes);
    if (slab < 1 || (p.k_slices > 1 && slab < m_tiles)) return p;
    const long long slabs = (m_tiles + slab - 1) / slab, slots = (long long)compute_units() * s.per_cu;
    const auto rounds = [&](long long tiles) { return (tiles * n_tiles * p.k_slices + slots - 1) / slots; };
    if (room < kLost * slabs || slabs * rounds(slab) > rounds(m_tiles)) return p;
    return TilePlan{p.tile, p.k_slices, kSparsePart * p.us, true};
}

// The search.  A short call waits for it, and an estimate takes some 20 ns: K whole for every tile first; then slices of the tile that they can
// gain most for, and so on until no tile can gain (`least`: the estimate with what does not depend on the number of slices, and the
// fewest steps).  us of a choice: 14 x 2816 x 2944 0.42 (all 64 estimates one after the other 2.0), 256 x 4096 x 4096 0.38 (1.5), 64 x 512 x 512 0.24 (0.42).
TilePlan choose_tile(const tcsc_layout_t &l, int M, size_t ws_bytes)
{
    constexpr int kCount = (int)(sizeof(kTiles) / sizeof(kTiles[0]));
    TilePlan best{-1, 1, 0.0};
    const int units = compute_units();
    const double y_mb = 4e-6 * (double)M * l.n_pad;
    double tiles[kCount], floor_us[kCount];
    const auto consider = [&](int i, int k) {
        const TileShape &s = kTiles[i];
        const int per = (l.n_kblocks + k - 1) / k;
        const double mb = k * y_mb;
        if (k > 1 && (per * (k - 1) >= l.n_kblocks || (size_t)k * M * l.n_pad * 4 > ws_bytes)) return;
        const double load = up(tiles[i] * k / units), rounds = s.per_cu == 1 ? load : up(load / s.per_cu);
        const double steps = 2.0 * ((per + s.groups - 1) / s.groups);
        const double step_us = s.step * rounds > s.work * load ? s.step * rounds : s.work * load;
        double us = i < kFirstOfWaves ? s.fixed * rounds + steps * step_us : s.fixed + (s.step + steps * s.work) * load;
        if (us < floor_us[i]) us = floor_us[i];
        if (i >= kFirstOfWaves && k == 1 && rounds > 1.0) us = kLateRounds * us + kLateMb * mb;
        us += kCall + (k > 1 ? kSlice + kSliceMb * mb : 0.0);
        if (best.tile < 0 || us < best.us) best = TilePlan{i, k, us};
    };
    const auto whole = [&](int from, int to) {
        for (int i = from; i < to; ++i) {
            const TileShape &s = kTiles[i];
            tiles[i] = (double)(((long long)M + s.rows - 1) / s.rows) * ((l.n_pad + s.cols - 1) / s.cols);
            floor_us[i] = 6.0 * tiles[i] * s.rows * s.cols * l.K / s.peak;
            // a launch has less than 2^32 threads; a call with more tiles than that goes to k_large, which takes X in slabs
            if (tiles[i] * (64 * s.waves) < 4294967296.0) consider(i, 1);
        }
    };
    const auto sliced = [&](int from, int to) {
        if (from >= to || l.n_kblocks < 2 || M > 65535) return;
        double least[kCount];
        for (int i = from; i < to; ++i) {
            const TileShape &s = kTiles[i];
            const int most = kMaxKSlices < l.n_kblocks ? kMaxKSlices : l.n_kblocks;
            const double steps = 2.0 * (((l.n_kblocks + most - 1) / most + s.groups - 1) / s.groups);
            double us = steps * (i < kFirstOfWaves ? s.step : s.work), all = 2.0 * l.n_kblocks * tiles[i] * s.work / (s.groups * (double)units);
            if (us < all) us = all;
            us += i < kFirstOfWaves ? s.fixed : s.fixed + s.step;
            if (us < floor_us[i]) us = floor_us[i];
            // (slices beyond two full rounds only add partial sums)
            least[i] = 2.0 * tiles[i] > 2.0 * units * s.per_cu ? 1e300 : us + kCall + kSlice + kSliceMb * 2.0 * y_mb;
        }
        for (;;) {
            int i = from;
            for (int j = from + 1; j < to; ++j)
                if (least[j] < least[i]) i = j;
            if (least[i] >= (best.tile < 0 ? 1e300 : best.us)) return;
            least[i] = 1e300;
            for (int k = 2; k <= kMaxKSlices && k <= l.n_kblocks && tiles[i] * k <= 2.0 * units * kTiles[i].per_cu; ++k) consider(i, k);
        }
    };
    const bool waves = waves_can(l);
    whole(0, kFirstOfWaves);
    const bool short_call = best.tile >= 0 && kLostPart * best.us < kLost;   // too short for digits, with slices too
    if (!short_call) {
        sliced(0, kFirstOfWaves);
        if (best.tile >= 0) {   // a call that k_matrix takes in digits stays there
            const TilePlan p = with_digits(l, M, ws_bytes, best);
            if (p.digits) return p;
        }
    }
    if (waves) whole(kFirstOfWaves, kCount);
    sliced(short_call ? 0 : kFirstOfWaves, waves ? kCount : short_call ? kFirstOfWaves : 0);
    return best;
}

// ------------------------------------------------------------------------------------------------------------------
// k_rows: M <= MM rows (MM <= 10).  The three planes of X are the rows of A: 3 M of them, in T tiles of 16, so up to five
// rows of X cost one matrix instruction where k_matrix would need three.  A workgroup is KW wavefronts with the same 16 B
// columns, each with every KW-th group of four blocks (256 rows of W): a lane's 16-byte load is one block of one column,
// and serves eight matrix instructions, so the row sets are read once, 2 bits an entry, with no LDS in between.  A group of X
// is cut by its wavefront alone and goes through a piece of the LDS of its own into fragments that all
// B tiles of columns use; the next group's loads are under way meanwhile.  The sums of the KW wavefronts meet in the LDS.
// Bound by the latency of that chain (2.5 us with one group a wavefront, of which launch and first loads are most) and
// then by spreading and cutting on the vector ALU and by the LDS: all three planes are staged before any is read, so that a
// fragment is one read of all lanes; plane by plane, each lane waiting for its own, it was three.  M = 1, 4096 x 11008
// 5.3 -> 4.9 us (a call from Python 5.23, 5.01 since the weights are spread by conversions), M = 8 7.9 -> 7.5, M = 8, 4096 x 4096 5.8 -> 5.3, M = 2, 11008 x 4096 6.4 -> 5.2 (lists, at 50 % non-zeros: 10.0, 23.7, 10.7, 10.7).
// Without the next group's loads 20 % more.  Over 220 shapes (K, N = 700 .. 16384) all planes at once take 2 to 23 % less time
// from the row sets; from the codes 17 % less to 2 % more at M <= 5 (M <= 3: the rule below takes k_rows more often, up to
// 33 %), 8 % less to 3 % more at M = 6, 7, and the same at M = 8 (2 % less to 3 % more: 2500 x 5000 6.1 -> 6.3 us).
//
// PACKED: W from the base-3 codes (a.masks, a.n_kblocks: 16-byte pieces of 80 rows, [piece][n_pad]).  A table in the LDS
// gives the five weights of a code, four bits each; those of codes j and j + 8, put side by side, make bytes that are converted to
// dwords for rows 5 j + i and 40 more (M = 1, 4096 x 11008 7.0 us with a shift and an AND for each, 6.6 so; M = 5 9.05, 8.7).
// A group is 320 rows and ten matrix instructions a tile.
// Against the kernel that multiplies on the vector ALU, 4096 x 11008: M = 2 9.3 -> 8.4 us, M = 8 21.5 -> 10.6 us; 4096 x 4096: M = 1 7.3 -> 5.4 us,
// M = 5 14.8 -> 6.8.  Sixteen copies of the table, so that few lanes meet in a bank, cost more to fill than they saved.
constexpr int kMaxRows = 10;

// The five weights of a code (81 d0 + 27 d1 + 9 d2 + 3 d3 + d4; digit 1: +1, 2: -1) in four bits as in FourBitWord: the first four in the low
// halves of the bytes, the fifth in the high half of the first byte.
__device__ __forceinline__ unsigned weights_of_code(int code)
{
    unsigned bits = 0;
#pragma unroll
    for (int i = 4; i >= 0; --i) {
        const unsigned digit = code % 3;
        code /= 3;
        bits |= (digit == 0 ? 0u : digit == 1 ? 4u : 12u) << (i < 4 ? 8 * i : 4);
    }
    return bits;
}

// (Up to five rows of X and 16 columns: four wavefronts per SIMD, three on the codes, so that as many workgroups of four fit
// side by side.)
template <int MM, int B, int KW, bool PACKED>
__global__ void __launch_bounds__(64 * KW, MM <= 5 && B == 1 ? (PACKED && MM > 2 ? 3 : 4) : 1)
k_rows(const MatrixArgs a)
{
    constexpr int kSteps = PACKED ? 10 : 8;                  // matrix instructions per block of W and tile
    constexpr int kUnits = 4 * kSteps, kRowUnits = kUnits + 1;   // 16-byte units per staged row of a group (+ 1: other banks)
    constexpr int kBlockRows = 8 * kSteps;
    // Weights through FourBitWord, whose pairs are rows j and j + 4 (M = 1, 4096 x 11008 5.53 -> 5.3 us, M = 5 6.76 -> 6.6).  Where the
    // loads of X count, a pair is j and j + 16, so that they bring 64 bytes at a time (M = 8, 4096 x 4096 5.42 us, else 5.51; M = 1 3.52, 3.56).
    constexpr bool kFour = !PACKED && MM <= 5 && (MM > 2 || B > 1);
    constexpr int kPartner = PACKED ? 40 : kFour ? 4 : 16;
    constexpr int T = (3 * MM + 15) / 16, kItems = (MM * kUnits + 63) / 64;
    constexpr int kStage = KW * 3 * MM * kRowUnits, kSums = KW * B * T * 64;
    __shared__ uint4v lds[kStage > kSums ? kStage : kSums];
    __shared__ unsigned table[PACKED ? 256 : 1];
    __shared__ int spoilt;   // a sum was not finite

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int n0 = blockIdx.x * (16 * B), M = a.M, n_groups = (a.n_kblocks + 3) / 4;
    uint4v *stage = lds + wave * (3 * MM * kRowUnits);   // [plane][row]
    const __amdgpu_buffer_rsrc_t wbuf = raw_buffer(a.masks, (size_t)a.n_kblocks * a.n_pad * 16);
    const __amdgpu_buffer_rsrc_t xbuf = raw_buffer(a.X, (size_t)M * a.K * 4);

    uint4v w_next[B];
    float4v x0_next[kItems], x1_next[kItems];   // item: four entries of a row and the four kPartner further on
    auto load = [&](int group) {
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const unsigned n = (unsigned)min(n0 + 16 * b + r, a.n_pad - 1);
            w_next[b] = load16(wbuf, ((unsigned)(4 * group + g) * (unsigned)a.n_pad + n) * 16u);
        }
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
            const int it = lane + 64 * i, m = it / kUnits, unit = it % kUnits, step = unit % kSteps;
            const unsigned k = (unsigned)(kBlockRows * (4 * group + unit / kSteps)) +
                               (PACKED ? 4 * step : kFour ? 8 * step : 32 * (step >> 2) + 4 * (step & 3));
            const unsigned off = m < M ? ((unsigned)m * (unsigned)a.K + k) * 4u : kNowhere;
            x0_next[i] = __builtin_bit_cast(float4v, load16(xbuf, off));
            x1_next[i] = __builtin_bit_cast(float4v, load16(xbuf, off + 4u * kPartner));
        }
    };

    float4v acc[B][T];
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
        for (int t = 0; t < T; ++t) acc[b][t] = float4v{0.f, 0.f, 0.f, 0.f};

    load(wave);
    if constexpr (PACKED) {
        for (int i = threadIdx.x; i < 256; i += 64 * KW) table[i] = weights_of_code(i);
        __syncthreads();
    }
    // of the column this thread finishes first
    const Epilogue finish(a.b, a.alpha, a.alpha_stride, a.N);
    const int n_first = n0 + 16 * ((int)(threadIdx.x >> 4) % B) + (threadIdx.x & 15);
    float bias = finish.bias_of(n_first), slope = finish.slope_of(n_first);
    for (int group = wave; group < n_groups; group += KW) {
        uint4v w[B];
        float4v x0[kItems], x1[kItems];
#pragma unroll
        for (int b = 0; b < B; ++b) w[b] = w_next[b];
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
            x0[i] = x0_next[i] * kScaleUp;
            x1[i] = x1_next[i] * kScaleUp;
        }
        if (group + KW < n_groups) load(group + KW);
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
            const int it = lane + 64 * i, m = it / kUnits, unit = it % kUnits;
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                uint4v d;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    d[e] = top_halves(x0[i][e], x1[i][e]);
                    x0[i][e] = below_top(x0[i][e]);
                    x1[i][e] = below_top(x1[i][e]);
                }
                if (m < M) stage[(p * M + m) * kRowUnits + unit] = d;
            }
        }
        // the wavefront's own piece of the LDS, and its LDS operations stay in order: no barrier
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        bf16x8 x[T][kSteps];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int row = min(16 * t + r, 3 * M - 1);   // (rows of A beyond the planes give rows nobody reads)
#pragma unroll
            for (int s = 0; s < kSteps; ++s) x[t][s] = __builtin_bit_cast(bf16x8, stage[row * kRowUnits + kSteps * g + s]);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int b = 0; b < B; ++b) {
            auto multiply = [&](int step, bf16x8 bw) {
#pragma unroll
                for (int t = 0; t < T; ++t)
                    acc[b][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[t][step], bw, acc[b][t], 0, 0, 0);
            };
            if constexpr (PACKED) {
                unsigned four[8], fifth[8];   // of codes j (low half of a byte) and j + 8
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const unsigned lo = table[w[b][j / 4] >> (8 * (j % 4)) & 255u], hi = table[w[b][2 + j / 4] >> (8 * (j % 4)) & 255u];
                    four[j] = (hi << 4 & 0xF0F0F0F0u) | (lo & 0x0F0F0F0Fu);
                    fifth[j] = (lo >> 4 & 0x0Fu) | (hi & ~0x0Fu);
                }
#pragma unroll
                for (int step = 0; step < kSteps; ++step) {
                    uint4v d;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int j = (4 * step + e) / 5, i = (4 * step + e) % 5;
                        d[e] = i < 4 ? two_weights(four[j], i) : two_weights(fifth[j], 0);
                    }
                    multiply(step, __builtin_bit_cast(bf16x8, d));
                }
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if constexpr (kFour) {
                        const FourBitWord half(w[b][h], w[b][2 + h]);
#pragma unroll
                        for (int s = 0; s < 4; ++s) multiply(4 * h + s, half.eight(s));
                    } else {
                        const SignedWord half(w[b][h], w[b][2 + h]);
#pragma unroll
                        for (int s = 0; s < 4; ++s) multiply(4 * h + s, half.eight(4 * s));
                    }
                }
            }
        }
    }

    // sums of the wavefronts, [wave][b][row of A][column]: element e of a fragment is row 4 g + e, column r
    if (threadIdx.x == 0) spoilt = 0;
    __syncthreads();
    float *sums = reinterpret_cast<float *>(lds);
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) sums[(((wave * B + b) * T + t) * 16 + 4 * g + e) * 16 + r] = acc[b][t][e];
    __syncthreads();
    for (int o = threadIdx.x; o < 16 * B * M; o += 64 * KW) {
        const int c = o & 15, b = (o >> 4) % B, m = (o >> 4) / B, n = n0 + 16 * b + c;
        if (n >= a.N) continue;
        if (o != (int)threadIdx.x) {
            bias = finish.bias_of(n);
            slope = finish.slope_of(n);
        }
        float plane[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            plane[p] = 0.f;
#pragma unroll
            for (int k = 0; k < KW; ++k) plane[p] += sums[((k * B + b) * T * 16 + p * M + m) * 16 + c];
        }
        float v = (plane[0] + (plane[1] + plane[2])) * kScaleDown;
        if (!finite(v)) spoilt = 1;
        a.Y[(size_t)m * a.N + n] = finish(v, bias, slope);
    }
    __syncthreads();
    if (!spoilt) return;
    // again from X and the row sets, groups of them dealt to the wavefronts as before: [wave][b][row][column]
#pragma unroll 1
    for (int b = 0; b < B; ++b) {
        float4v v[1];
        sums_of_any(v, a.X, M, a.K, a.row_sets, a.n_pad, {min(n0 + 16 * b + r, a.n_pad - 1)}, 0, a.n_row_blocks, wave, KW);
#pragma unroll
        for (int e = 0; e < 4; ++e) sums[((wave * B + b) * 16 + 4 * g + e) * 16 + r] = v[0][e];
    }
    __syncthreads();
    for (int o = threadIdx.x; o < 16 * B * M; o += 64 * KW) {
        const int c = o & 15, b = (o >> 4) % B, m = (o >> 4) / B, n = n0 + 16 * b + c;
        if (n >= a.N || finite(a.Y[(size_t)m * a.N + n])) continue;   // the thread's own store
        float v = 0.f;
#pragma unroll
        for (int k = 0; k < KW; ++k) v += sums[((k * B + b) * 16 + m) * 16 + c];
        a.Y[(size_t)m * a.N + n] = finish(v, finish.bias_of(n), finish.slope_of(n));
    }
}

template <int MM, int B, int KW, bool PACKED>
hipError_t launch_rows_kernel(const MatrixArgs &a, const Call &c)
{
    hipError_t e;
    if ((e = c.record_before()) != hipSuccess) return e;
    hipLaunchKernelGGL((k_rows<MM, B, KW, PACKED>), dim3((a.N + 16 * B - 1) / (16 * B)), dim3(64 * KW), 0, c.stream, a);
    e = hipGetLastError();
    if (e == hipSuccess) e = c.record_after();
    return e;
}

// Shape of a call with M <= 10: eight wavefronts from five groups of 256 rows on, else four; as few tiles of 16 columns per
// workgroup as leave one workgroup per compute unit (more of the small ones: they fit side by side), because every
// workgroup cuts X anew.  us: 2.0 .. 2.6 + turns through the groups x (cutting + spreading) (fitted to 119 calls, M = 1 .. 8,
// K and N = 512 .. 16384: 7 % off on average, 24 % at worst).
// These figures, and what matrix_plan() and packed_plan() say of the choices that rest on them, are from before the weights were spread by conversions,
// since when k_rows takes 2 to 6 % less for M <= 5 and from the codes: calls near the line stay with the other kernel.
struct RowsPlan {
    int tiles, waves;
    double us;
};
RowsPlan rows_plan(const tcsc_layout_t &l, int M, bool packed)
{
    const int blocks = packed ? l.n_chunks5 : l.n_kblocks, groups = (blocks + 3) / 4, units = compute_units();
    const double tiles = (double)((l.N + 15) / 16);
    RowsPlan p;
    p.waves = groups > 4 ? 8 : 4;
    const int slots = p.waves == 8 ? units : M <= 5 && !packed ? 4 * units : 2 * units;
    p.tiles = (int)fmin(ceil(tiles / slots), p.waves == 8 ? 4.0 : 2.0);
    const double rounds = fmax(1.0, tiles / ((double)p.tiles * slots));
    double start = p.waves == 4 ? 2.03 : M <= 2 ? 2.25 : M <= 5 ? 2.45 : 2.59;
    double cut = M <= 2 ? 0.10 : M <= 5 ? 0.42 : 0.58, spread = M <= 2 ? 0.46 : M <= 5 ? 0.47 : 0.66;
    if (packed) {
        start = p.waves == 4 ? 2.34 : M <= 2 ? 2.73 : M <= 5 ? 3.02 : 3.33;
        cut = M <= 2 ? 0.20 : M <= 5 ? 0.61 : 1.02;
        spread = M <= 2 ? 0.64 : M <= 5 ? 0.67 : 0.75;
    }
    p.us = start + ((groups + p.waves - 1) / p.waves) * rounds * (cut + spread * p.tiles);
    return p;
}

template <int MM, bool PACKED>
hipError_t pick_rows(const MatrixArgs &a, const MatrixPlan &p, const Call &c)
{
    if (p.split == 4)
        return p.shape == 1 ? launch_rows_kernel<MM, 1, 4, PACKED>(a, c) : launch_rows_kernel<MM, 2, 4, PACKED>(a, c);
    switch (p.shape) {
    case 1: return launch_rows_kernel<MM, 1, 8, PACKED>(a, c);
    case 2: return launch_rows_kernel<MM, 2, 8, PACKED>(a, c);
    case 3: return launch_rows_kernel<MM, 3, 8, PACKED>(a, c);
    default: return launch_rows_kernel<MM, 4, 8, PACKED>(a, c);
    }
}

template <bool PACKED>
hipError_t launch_rows(const MatrixArgs &a, const MatrixPlan &p, const Call &c)
{
    if (a.M <= 2) return pick_rows<2, PACKED>(a, p, c);
    if (a.M <= 5) return pick_rows<5, PACKED>(a, p, c);
    if (a.M <= 8) return pick_rows<8, PACKED>(a, p, c);
    if constexpr (PACKED) return hipErrorInvalidValue;
    else return pick_rows<10, false>(a, p, c);
}

// Offsets inside a tile of X or Y and inside the row sets are 32 bits wide, with some steps to spare.
bool offsets_fit(const tcsc_layout_t &l)
{
    return l.K <= kMaxExtent && l.N <= kMaxExtent && ((long long)l.n_kblocks + 64) * l.n_pad * 16 < (1LL << 32);
}

double density(const tcsc_layout_t &l) { return (double)(l.nnz_pos + l.nnz_neg) / ((double)l.K * (double)l.N); }

}  // namespace

// Partial sums and X in digits of the plan that a call has where the workspace does not bound it.
size_t matrix_workspace_bytes(int M, int K, int N, int n_pad)
{
    tcsc_layout_t l{};
    l.K = K; l.N = N; l.n_pad = n_pad; l.n_kblocks = (K - 1) / kKBlock + 1;
    if (!offsets_fit(l)) return 0;
    const TilePlan p = choose_tile(l, M, (size_t)1 << 62);
    if (p.tile < 0) return 0;
    const size_t partial_bytes = p.k_slices > 1 ? (size_t)p.k_slices * M * n_pad * 4 : 0;
    return partial_bytes + (p.digits ? ((size_t)M + 63) / 64 * digit_tile_bytes(l) : 0);
}

// Whether the matrix cores take a call (the lists or the row-set walk being the other choice).  They do unless W is so
// sparse that those, whose time goes with the number of non-zeros, are ahead.  Measured on 12 shapes (K, N = 512 .. 16384),
// M = 1 .. 4096 and densities from 1/16 to 0: a call taken here is never more than 4 % behind the lists or the row-set walk
// (1024 x 8192 x 8192 at 1/256: 231 against 223 us), but for 0.2 us of 2.9 at M = 2 with an empty W.  Some of the calls that
// are left to those, below 1/64, would be faster here (64 x 4096 x 11008 at 1/256: 39 us; at 1/64, here, 24).
//  * M > 64, tall and wide: k_large with 128 columns per workgroup takes 20 us + 0.0281 + 0.464 density us per row of W
//    and round of its workgroups (measured M = 4096, K = N = 8192: 928 us at 1/16, 2318 us at 1/4; here 1040 us at any
//    density).  Its other shapes are behind this path at every density, by 1.2 to 5 times down to 1/16 and 1.0 to 3 times
//    with an empty W, so where the column count leaves only those this path is always taken, and where K would be sliced
//    there the figure above, too high for that, does no harm.
//  * 8 < M <= 64: k_small, with a tile of 16 rows, takes 6.1 us, or 9.6 us where K is cut into slices (beyond 1024 rows),
//    + 0.1 per 1000 rows of W + 0.12 per million entries + 0.8 per million non-zeros, 1.3 and 1.7 times that for 32 and
//    64 rows (M = 16: 15000 x 600 at 1/16 12.6 against 14.2; from 17 rows on it is behind everywhere, down to an empty W).  The
//    6.1 count as 6.7: k_small has a second launch before it and takes more than that on few columns (1024 x 1024, M = 16, from an
//    empty W to 50 %: 6.2 .. 8.2 against 6.25 in k_waves; 14 shapes x 6 densities: k_small ahead by at most 1 % where this path is taken).
//    With K not a multiple of 4, where k_matrix is the other side, 6.9 .. 10.3 against 6.1 .. 6.6 on 52 shapes that the 6.7 bring here.
//  * M <= 8: k_decode takes 2.55 + 0.5 M + 0.04 us per 1000 rows of W + (0.265 + 0.016 M) us per million non-zeros for one or
//    two rows, 2.03 + 0.58 M + 0.13 + (0.353 + 0.066 M) for more, and 3.5 us for each further time that X fills the LDS (fitted
//    to 17 shapes x 4 densities x M = 1 .. 8; the choice is 0.6 % behind the better of the two on average, 69 % at worst, 3 x 4096
//    x 11008 at 1/16).  It stays ahead for few non-zeros and a long K (M = 1, 16384 x 4096 at 1/8: 4.7 us against 7.2; at 1/4
//    8.6 against 7.3), and k_rows otherwise (M = 1, 4096 x 11008 at 1/2 10.0 against 5.2; M = 3, 2053 x 1531 5.7 against 3.6).
MatrixPlan matrix_plan(const tcsc_layout_t &l, int M, const Call &c)
{
    MatrixPlan none{};
    if (!offsets_fit(l)) return none;
    const double d = density(l), entries = 1e-6 * (double)l.K * (double)l.N;
    RowsPlan r{};
    if (M <= kMaxRows) {
        r = rows_plan(l, M, false);
        if (M <= 8) {
            const double ones = 1e-3 * l.K, hits = entries * d;
            const double lists = M <= 2 ? 2.55 + 0.5 * M + 0.04 * ones + hits * (0.265 + 0.016 * M)
                                        : 2.03 + 0.58 * M + 0.13 * ones + 3.54 * floor(M * (double)l.K / 38400.0) +
                                              hits * (0.353 + 0.066 * M);
            if (r.us >= lists) return none;
            return MatrixPlan{true, r.tiles, r.waves, false};
        }
    }
    const TilePlan p = choose_tile(l, M, c.ws_bytes);
    const bool rows = M <= kMaxRows && (p.tile < 0 || r.us < p.us);
    if (!rows && p.tile < 0) return none;
    const double us = rows ? r.us : p.us;
    double other;
    if (M <= 64) {
        other = (M <= 16 ? 1.0 : M <= 32 ? 1.3 : 1.7) *
                ((l.K <= 1024 ? 6.7 : 9.6) + 0.1e-3 * l.K + entries * (0.12 + 0.8 * d));
    } else {
        if (l.n_pad % 128 != 0) return MatrixPlan{false, p.tile, p.k_slices, p.digits};
        const double groups = ceil(M / 256.0) * (l.n_pad / 128);
        other = 20.0 + ceil(groups / (2.0 * compute_units())) * l.K * (0.0281 + 0.464 * d);
    }
    if (us >= other) return none;
    return rows ? MatrixPlan{true, r.tiles, r.waves, false} : MatrixPlan{false, p.tile, p.k_slices, p.digits};
}

void matrix_tile(const MatrixPlan &p, int M, tstgemm_route_t *out)
{
    out->tile_rows = p.rows ? M : kTiles[p.shape].rows;
    out->tile_cols = p.rows ? 16 * p.shape : kTiles[p.shape].cols;
    out->k_groups = p.rows ? p.split : kTiles[p.shape].groups;
    out->k_slices = p.rows ? 1 : p.split;
}

bool matrix_waves(const MatrixPlan &p) { return p.taken() && !p.rows && p.shape >= kFirstOfWaves; }

hipError_t launch_matrix(const MatrixPlan &p, const float *X, const tcsc *t, const float *b, float *Y, int M, const Call &c)
{
    const tcsc_layout_t &l = t->layout;
    MatrixArgs a{};
    a.X = X; a.masks = reinterpret_cast<const uint4v *>(device_view(t).masks); a.b = b; a.Y = Y;
    a.alpha = c.act.alpha; a.alpha_stride = c.act.alpha_stride;
    a.partials = reinterpret_cast<float *>(c.ws);
    a.M = M; a.K = l.K; a.N = l.N; a.n_pad = l.n_pad; a.n_kblocks = l.n_kblocks;
    a.row_sets = a.masks; a.n_row_blocks = l.n_kblocks;
    if (p.rows) return launch_rows<false>(a, p, c);
    const TileShape &s = kTiles[p.shape];
    a.n_tiles = (l.n_pad + s.cols - 1) / s.cols;
    a.k_slices = p.split;
    a.kb_per_slice = (l.n_kblocks + p.split - 1) / p.split;
    const long long m_tiles = ((long long)M + s.rows - 1) / s.rows;
    const auto launch = [&](long long n) {
        if (p.digits) {
            switch (p.shape) {
            case 0: return launch_tiles<1, 1, 8, 2, 2, true>(a, n, c);
            default: return launch_tiles<1, 1, 4, 2, 2, true>(a, n, c);
            }
        }
        switch (p.shape) {
        case 0: return launch_tiles<1, 1, 8, 2, 2, false>(a, n, c);
        case 1: return launch_tiles<1, 1, 4, 2, 2, false>(a, n, c);
        case 2: return launch_tiles<2, 1, 4, 2, 2, false>(a, n, c);
        case 3: return launch_tiles<1, 1, 4, 2, 1, false>(a, n, c);
        case 4: return launch_tiles<4, 1, 2, 1, 1, false>(a, n, c);
        case 5: return launch_tiles<2, 1, 4, 1, 1, false>(a, n, c);
        case 6: return launch_waves<2>(a, n, c);
        default: return launch_waves<4>(a, n, c);
        }
    };
    const auto tiles = [&](long long n) {   // n tiles of rows, between the call's events
        hipError_t e = c.record_before();
        if (e == hipSuccess) e = launch(n);
        return e == hipSuccess ? c.record_after() : e;
    };
    hipError_t e = hipSuccess;
    if (!p.digits) {
        if ((e = tiles(m_tiles)) != hipSuccess) return e;
    } else {
        // X in slabs of as many tiles as the workspace holds in digits
        const size_t partial_bytes = p.split > 1 ? (size_t)p.split * M * l.n_pad * 4 : 0, tile_bytes = digit_tile_bytes(l);
        const long long slab = digit_slab(l, m_tiles, c.ws_bytes - partial_bytes);
        char *units = c.ws + partial_bytes;
        unsigned char *counts = reinterpret_cast<unsigned char *>(units + slab * (tile_bytes - l.n_kblocks));
        a.digits = units;
        a.counts = counts;
        for (long long t = 0; t < m_tiles; t += slab) {
            const long long n = slab < m_tiles - t ? slab : m_tiles - t;
            a.X = X + (size_t)t * 64 * l.K;
            a.Y = Y + (size_t)t * 64 * l.N;
            a.M = (int)(M - t * 64 < n * 64 ? M - t * 64 : n * 64);
            hipLaunchKernelGGL(k_digits, dim3((unsigned)(n * digit_runs(l.n_kblocks))), dim3(128), 0, c.stream, a.X, a.M, l.K,
                               l.n_kblocks, units, counts);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            if ((e = tiles(n)) != hipSuccess) return e;
        }
    }
    return a.k_slices == 1 ? hipSuccess : launch_sum(a, c.stream);
}

// Whether k_rows takes the base-3 codes, or k_packed, which multiplies on the vector ALU: a workgroup of that takes
// 2.6 us + (0.65 + 0.43 M) us per 1000 rows of W, and 3 us more where it deals K to several workgroups (measured
// M = 1 .. 8, the shapes of rows_plan()).  k_packed stays ahead on short K over many columns (M <= 5, 512 x 16384, M = 5: 4.6 against
// 4.8 us); M = 1, 4096 x 11008 7.1 against 6.3 here.  The choice is 0.3 % behind the better of the two on average.
MatrixPlan packed_plan(const tcsc_layout_t &l, int M)
{
    if (l.K > kMaxExtent || ((long long)l.n_chunks5 + 64) * l.n_pad * 16 >= (1LL << 32)) return MatrixPlan{};
    const int units = compute_units(), groups = l.n_pad / 64;
    int parts = 2 * groups <= units && M * l.n_chunks5 >= 400 ? units / groups : 1;
    if (parts > 4) parts = 4;
    const double rounds = ceil((double)groups * parts / units);
    const double other = 2.6 + rounds * l.K / parts * 1e-3 * (0.65 + 0.43 * M) + (parts > 1 ? 3.0 : 0.0);
    const RowsPlan r = rows_plan(l, M, true);
    return r.us < other ? MatrixPlan{true, r.tiles, r.waves, false} : MatrixPlan{};
}

hipError_t launch_packed_rows(const MatrixPlan &p, const float *X, const tcsc *t, const float *b, float *Y, int M, const Call &c)
{
    const tcsc_layout_t &l = t->layout;
    MatrixArgs a{};
    a.X = X; a.masks = reinterpret_cast<const uint4v *>(device_view(t).packed); a.b = b; a.Y = Y;
    a.row_sets = reinterpret_cast<const uint4v *>(device_view(t).masks);   // (the codes are built from them)
    a.M = M; a.K = l.K; a.N = l.N; a.n_pad = l.n_pad; a.n_kblocks = l.n_chunks5; a.n_row_blocks = l.n_kblocks;
    return launch_rows<true>(a, p, c);
}

}  // namespace tst
