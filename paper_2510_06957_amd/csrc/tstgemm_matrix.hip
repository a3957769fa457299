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
// X held an infinity, a NaN or something beyond about 2^100 -- is taken again from X itself by gather_output(), member by
// member of the lists, so an entry of X under a zero weight never reaches Y here either.
//
// k_matrix is for M > 10, k_rows for M <= 10; choose_tile() and rows_plan() have the rules, with what was measured.
#include <cmath>

#include "tstgemm_internal.h"

namespace tst {
namespace {

typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));   // four floats at any float's address
typedef float float16v __attribute__((ext_vector_type(16)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr float kScaleUp = 16777216.f;            // 2^24
constexpr float kScaleDown = 1.f / 33554432.f;    // 2^-25
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

__device__ __forceinline__ uint4v load16(__amdgpu_buffer_rsrc_t buf, unsigned offset)
{
    return __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(buf, (int)offset, 0, 0));
}

// X W for one output straight from X: adds and subtracts the members of the two sets of every block.  For outputs whose
// sum the matrix cores could not hold; a NaN stays one, so the walk ends there.
__device__ __forceinline__ float gather_output(const float *__restrict__ X, const uint4v *__restrict__ masks, int n_pad,
                                               int n_kblocks, int m, int n, int K)
{
    float s = 0.f;
    const float *x = X + (size_t)m * K;
    for (int kb = 0; kb < n_kblocks; ++kb) {
        const uint4v w = masks[(size_t)kb * n_pad + n];
        unsigned long long pos = w[0] | ((unsigned long long)w[1] << 32), neg = w[2] | ((unsigned long long)w[3] << 32);
        for (; pos; pos &= pos - 1) s += x[kb * kKBlock + __builtin_ctzll(pos)];
        for (; neg; neg &= neg - 1) s -= x[kb * kKBlock + __builtin_ctzll(neg)];
        if (s != s) break;
    }
    return s;
}

struct MatrixArgs {
    const float *X;
    const uint4v *masks;             // [n_kblocks][n_pad] {+1 rows low, high, -1 rows low, high}
    const float *b, *alpha;
    float *Y, *partials;             // partials[slice][M][n_pad], scaled sums
    int alpha_stride;
    int M, K, N, n_pad, n_kblocks;
    int n_tiles, k_slices, kb_per_slice;
};

// ------------------------------------------------------------------------------------------------------------------
// k_matrix: a workgroup computes TM x TN of Y over one slice of K, WK groups of WM x WN wavefronts each over their
// share of the slice (their sums meet in the LDS at the end); a wavefront has RF x CF fragments of 32 x 32 (twice: hi,
// and mid + lo).  Per step of 32 rows of W a group cuts its TM x 32 floats of X into the three planes, in registers on
// their way from memory to the LDS (two buffers, one barrier a step); weights come straight from the row sets, 2 bits
// an entry, and are spread into fragments in registers.  Loads run PD steps ahead.  Per step a wavefront
// has 6 RF CF matrix instructions of 32 cycles; the cuts, the spreading and the LDS traffic are dealt over their six
// stages, each ended by a scheduling barrier (without the stages, and with loads whose number the compiler could not
// count, M = 4096, K = N = 8192 took 1.20 ms in place of 1.10).
// Bound: long calls by the power limit (M = 4096, K = N = 8192: 1.10 ms, i.e. 1.50 PFLOP/s of bf16 products at about
// 1.85 GHz; 4.4 ms for the lists at 50 % non-zeros, any density here), short ones by the start of the first loads, the
// sums at the end and the second launch where K is sliced (M = 256, K = N = 4096: 31 us against 89).
// Rows beyond M and rows of W beyond K: X reads as zero, or as the next row of X where the weights are zero.
template <int WK, int WM, int WN, int RF, int CF>
__global__ void __launch_bounds__(64 * WK * WM * WN, 2)
k_matrix(const MatrixArgs a)
{
    constexpr int NG = 64 * WM * WN, TM = 32 * RF * WM, TN = 32 * CF * WN, PD = 2;
    constexpr int kUnits = TM * 4 > NG ? TM * 4 / NG : 1;   // pieces of X (8 floats of a row) per lane and step
    static_assert(TM * 4 % NG == 0 || TM * 4 < NG, "units");
    constexpr int kChunk = TM + 2;                          // 16-byte units per plane and piece; + 2: other banks
    constexpr int kPlane = 4 * kChunk, kBuffer = 3 * kPlane;
    constexpr int kStageUnits = WK * 2 * kBuffer, kSumUnits = (WK / 2) * (TM * TN / 4);
    __shared__ uint4v lds_all[kStageUnits > kSumUnits ? kStageUnits : kSumUnits];

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

    // X from the first row of the tile on, and the row sets up to the end of the group's blocks: what lies beyond reads
    // as zero
    const size_t x_bytes = (size_t)(a.M - m0) * a.K * sizeof(float);
    const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(a.X + (size_t)m0 * a.K), 0, (int)(unsigned)min(x_bytes, (size_t)0xfffffffcu), kRawBuffer);
    const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint4v *>(a.masks), 0, (int)((unsigned)kb1 * (unsigned)a.n_pad * 16u), kRawBuffer);
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

    float16v acc[2][RF][CF];   // [hi | mid + lo]
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int i = 0; i < RF; ++i)
#pragma unroll
            for (int j = 0; j < CF; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[d][i][j][e] = 0.f;

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
    for (int i0 = 0; i0 < blocks; i0 += 2) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (i0 + q >= blocks) break;
            const int kb = kb0 + i0 + q;
#pragma unroll
            for (int t = 0; t < 2; ++t) {   // half of the block: 32 rows of W, LDS buffer t
                const int next = (t + 1) % PD;
                bf16x8 x[2][RF];
                auto read_x = [&](int s) {   // stage s: plane s % 3 of 16 rows
#pragma unroll
                    for (int i = 0; i < RF; ++i)
                        x[s & 1][i] = __builtin_bit_cast(
                            bf16x8, lds[t * kBuffer + (s % 3) * kPlane + (2 * (s / 3) + g) * kChunk + (wr * RF + i) * 32 + l32]);
                };
                // this step's planes are written, the other buffer's have been read.  Only LDS traffic is waited for:
                // the loads of the coming steps stay in flight
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
                __builtin_amdgcn_s_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
                read_x(0);
#pragma unroll
                for (int s = 0; s < 6; ++s) {
                    if (s < 5) read_x(s + 1);
#pragma unroll
                    for (int i = s * kPairs / 5; i < (s + 1) * kPairs / 5 && i < kPairs; ++i) cut_pair(next, i);
                    if (s == 1) spread_w(bw[1], q, t, 1);
                    if (s == 4) {
                        if (t == 1) load_w(q, kb + 2);
                        spread_w(bw[0], t ? q ^ 1 : q, t ^ 1, 0);
                    }
                    if (s == 5) {
                        // (behind the last block this writes once more what nothing reads)
                        store_planes(t ^ 1);
                        load_x(next, 2 * kb + t + 1 + PD);
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
#pragma unroll
    for (int i = 0; i < RF; ++i)
#pragma unroll
        for (int j = 0; j < CF; ++j) acc[0][i][j] += acc[1][i][j];

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

    // element e of a fragment is row 8 (e / 4) + 4 g + e % 4, column l32
    const int row0 = m0 + wr * RF * 32 + 4 * g, col0 = n0 + wc * CF * 32 + l32;
    auto row_of = [&](int i, int e) { return row0 + 32 * i + 8 * (e / 4) + e % 4; };
    if (a.k_slices > 1) {
        float *P = a.partials + (size_t)slice * a.M * a.n_pad;
#pragma unroll
        for (int j = 0; j < CF; ++j) {
            const int n = col0 + 32 * j;
#pragma unroll
            for (int i = 0; i < RF; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int m = row_of(i, e);
                    if (m < a.M && n < a.n_pad) P[(size_t)m * a.n_pad + n] = acc[0][i][j][e];
                }
        }
        return;
    }
    bool again = false;
#pragma unroll
    for (int j = 0; j < CF; ++j) {
        const int n = col0 + 32 * j;
        const float bias = (a.b != nullptr && n < a.N) ? a.b[n] : 0.f;
        const float slope = (a.alpha != nullptr && n < a.N) ? a.alpha[(size_t)n * a.alpha_stride] : 0.f;
#pragma unroll
        for (int i = 0; i < RF; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int m = row_of(i, e);
                again |= !finite(acc[0][i][j][e]);
                float v = acc[0][i][j][e] * kScaleDown + bias;
                if (a.alpha != nullptr) v = v > 0.f ? v : slope * v;
                if (m < a.M && n < a.N) a.Y[(size_t)m * a.N + n] = v;
            }
    }
    if (!again) return;
    for (int j = 0; j < CF; ++j) {
        const int n = col0 + 32 * j;
        if (n >= a.N) break;
        const float bias = a.b != nullptr ? a.b[n] : 0.f;
        for (int i = 0; i < RF * 16; ++i) {
            const int m = row_of(i / 16, i % 16);
            if (m >= a.M || finite(a.Y[(size_t)m * a.N + n])) continue;   // the lane's own store
            const float v = gather_output(a.X, a.masks, a.n_pad, a.n_kblocks, m, n, a.K) + bias;
            a.Y[(size_t)m * a.N + n] = activate(v, a.alpha, a.alpha_stride, n);
        }
    }
}

// k_matrix_sum: Y = (slice 0 + slice 1 + ...) 2^-25 + b, then the optional PReLU; four columns per thread, all slices
// requested together.  Bound by its launch and one trip to memory (4 slices of 256 x 4096: about 5 us).
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
    float4v y = part[0];
#pragma unroll
    for (int s = 1; s < S; ++s) y += part[s];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (n + i >= a.N) break;
        float v = finite(y[i]) ? y[i] * kScaleDown : gather_output(a.X, a.masks, a.n_pad, a.n_kblocks, m, n + i, a.K);
        if (a.b != nullptr) v += a.b[n + i];
        y[i] = activate(v, a.alpha, a.alpha_stride, n + i);
    }
    float *dst = a.Y + (size_t)m * a.N + n;
    if (n + 4 <= a.N) {
        *reinterpret_cast<float4u *>(dst) = y;
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

template <int WK, int WM, int WN, int RF, int CF>
hipError_t launch_tiles(const MatrixArgs &a, int m_tiles, const Call &c)
{
    hipError_t e;
    if ((e = c.record_before()) != hipSuccess) return e;
    hipLaunchKernelGGL((k_matrix<WK, WM, WN, RF, CF>), dim3((unsigned)((long long)m_tiles * a.n_tiles * a.k_slices)),
                       dim3(64 * WK * WM * WN), 0, c.stream, a);
    e = hipGetLastError();
    if (e == hipSuccess) e = c.record_after();
    if (e != hipSuccess || a.k_slices == 1) return e;
    return launch_sum(a, c.stream);
}

// Tile and K slices of a call: the combination whose estimated time is least.  A workgroup takes `fixed` us and `step`
// us for each of its steps of 32 rows of W while its compute unit has time to spare, `work` us when the unit is full
// (per_cu workgroups at a time); a call takes kCall us more, slices kSlice us and 0.4 us per MB of partial sums; and no
// call is faster than the matrix cores at the power limit (1.5 PFLOP/s).  Fitted to 13 tiles x 6 slice counts on 77
// shapes (M = 17 .. 2048, K and N = 512 .. 16384): the tile chosen among these five is 2 % slower than the best of all on
// average, 15 % at worst.
struct TileShape {
    int rows, cols, groups, per_cu;
    double fixed, step, work;
};
constexpr TileShape kTiles[] = {
    {64, 256, 1, 2, 1.23, 0.574, 0.457},   // long calls: two independent workgroups per unit fill each other's barriers
    {64, 256, 2, 1, 2.08, 0.964, 0.964},   // half the slices of the first where rows x columns leave units idle
    {64, 128, 1, 3, 0.29, 0.417, 0.307},   // short K: little to start with
    {32, 64, 4, 2, 0.52, 0.483, 0.461},    // small Y
    {32, 128, 2, 2, 0.30, 0.449, 0.381},   // M <= 32
};
constexpr double kCall = 4.39, kSlice = 1.30, kSliceMb = 0.40, kPeak = 1.5e9;   // us, us, us per MB, flops per us

struct TilePlan {
    int tile, k_slices;
    double us;
};
TilePlan choose_tile(const tcsc_layout_t &l, int M, size_t ws_bytes)
{
    TilePlan best{-1, 1, 0.0};
    const int units = compute_units();
    for (int i = 0; i < (int)(sizeof(kTiles) / sizeof(kTiles[0])); ++i) {
        const TileShape &s = kTiles[i];
        const double tiles = (double)((M + s.rows - 1) / s.rows) * (double)((l.n_pad + s.cols - 1) / s.cols);
        const double floor_us = 6.0 * tiles * s.rows * s.cols * l.K / kPeak;
        if (tiles * kMaxKSlices > 2e9) continue;
        for (int k = 1; k <= kMaxKSlices && k <= l.n_kblocks; ++k) {
            const int per = (l.n_kblocks + k - 1) / k;
            const double mb = 4e-6 * (double)k * M * l.n_pad;
            if (k > 1 && ((l.n_kblocks + per - 1) / per != k || M > 65535 || mb * 1e6 > (double)ws_bytes)) continue;
            const double load = ceil(tiles * k / units), rounds = ceil(load / s.per_cu);
            const double steps = 2.0 * ((per + s.groups - 1) / s.groups);
            const double step_us = s.step * rounds > s.work * load ? s.step * rounds : s.work * load;
            double us = s.fixed * rounds + steps * step_us;
            if (us < floor_us) us = floor_us;
            us += kCall + (k > 1 ? kSlice + kSliceMb * mb : 0.0);
            if (best.tile < 0 || us < best.us) best = TilePlan{i, k, us};
        }
    }
    return best;
}

// Offsets inside a tile of X and inside the row sets are 32 bits wide, with some steps to spare.
bool offsets_fit(const tcsc_layout_t &l)
{
    return l.K <= (1 << 22) && ((long long)l.n_kblocks + 64) * l.n_pad * 16 < (1LL << 32);
}

double density(const tcsc_layout_t &l) { return (double)(l.nnz_pos + l.nnz_neg) / ((double)l.K * (double)l.N); }

}  // namespace

// Whether the matrix cores take a call with M > 8 (the lists or the row-set walk being the other choice).  They do unless
// W is so sparse that those, whose time goes with the number of non-zeros, are ahead:
//  * M > 64, tall and wide: k_large with 128 columns per workgroup takes 20 us + 0.0281 + 0.464 density us per row of W
//    and round of its workgroups (measured M = 4096, K = N = 8192: 928 us at 1/16, 2318 us at 1/4; here 1100 us at any
//    density).  Its other shapes are 1.3 to 5 times slower than this path down to a density of 1/16.
//  * M <= 64: k_small needs about 4.5 + 0.52 us per 1000 rows of W however few the non-zeros are; it is ahead (up to
//    12 %, measured on M = 16, K = 15000, N = 600 below 1/8) where a few columns meet a long K.
bool matrix_wins(const tcsc_layout_t &l, int M, const Call &c)
{
    if (!offsets_fit(l)) return false;
    const TilePlan p = choose_tile(l, M, c.ws_bytes);
    if (p.tile < 0) return false;
    const double d = density(l);
    if (M > 64) {
        if (l.n_pad % 128 != 0) return true;
        const double groups = ceil(M / 256.0) * (l.n_pad / 128);
        return p.us < 20.0 + ceil(groups / (2.0 * compute_units())) * l.K * (0.0281 + 0.464 * d);
    }
    return d >= 0.13 || l.N >= 2048 || p.us < 4.5 + 0.52e-3 * l.K;
}

hipError_t launch_matrix(const float *X, const tcsc *t, const float *b, float *Y, int M, const Call &c)
{
    const tcsc_layout_t &l = t->layout;
    const TilePlan p = choose_tile(l, M, c.ws_bytes);
    if (p.tile < 0) return hipErrorInvalidValue;
    const TileShape &s = kTiles[p.tile];
    MatrixArgs a{};
    a.X = X; a.masks = reinterpret_cast<const uint4v *>(device_view(t).masks); a.b = b; a.Y = Y;
    a.alpha = c.act.alpha; a.alpha_stride = c.act.alpha_stride;
    a.partials = reinterpret_cast<float *>(c.ws);
    a.M = M; a.K = l.K; a.N = l.N; a.n_pad = l.n_pad; a.n_kblocks = l.n_kblocks;
    a.n_tiles = (l.n_pad + s.cols - 1) / s.cols;
    a.k_slices = p.k_slices;
    a.kb_per_slice = (l.n_kblocks + p.k_slices - 1) / p.k_slices;
    const int m_tiles = (M + s.rows - 1) / s.rows;
    switch (p.tile) {
    case 0: return launch_tiles<1, 1, 4, 2, 2>(a, m_tiles, c);
    case 1: return launch_tiles<2, 1, 4, 2, 2>(a, m_tiles, c);
    case 2: return launch_tiles<1, 1, 4, 2, 1>(a, m_tiles, c);
    case 3: return launch_tiles<4, 1, 2, 1, 1>(a, m_tiles, c);
    default: return launch_tiles<2, 1, 4, 1, 1>(a, m_tiles, c);
    }
}

}  // namespace tst
