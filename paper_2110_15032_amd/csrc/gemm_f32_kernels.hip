// Grouped GEMMs with fp32 operands (sbp_matmul, paper Sec. 3.1, Table 1: device g computes C_g = A_g B_g): fp32 x fp32, and
// an fp32 P(sum) partial next to a bf16 operand where gemm_split_kernel does not take the shape.  Any pitch, any extent.
//
// gemm_f32_kernel: v_mfma_f32_32x32x2_f32.  Operands keep all 32 bits and products enter an fp32 accumulator, as in an FMA
// chain; a bf16 operand is widened, exactly, on its way into LDS.
//
// Bound by the matrix instruction (64 cycles for 4096 flops, 157 TFLOP/s in all): a 64 x 64 wave tile needs 1 KB of
// fragments per 256 cycles and a 128 x 128 workgroup tile 16 KB of operands per 2048, so LDS and L2 have time to spare and
// the loads can take the way that suits any alignment: four elements per lane through registers, one stage ahead, two LDS
// stages, one barrier a stage; three or four workgroups share a compute unit and cover each other's waits.
//
// LDS images, four-element chunks as they lie in memory:
//   KC      [row][BK + 4]: ds_read_b128 gives a lane four consecutive kk of its row (pitch: 16 rows on 16 bank groups)
//   not KC  [kk][R + 8]:   ds_read_b32; the two half-waves read rows kk and kk + 4, which the pitch puts 32 banks apart
// Matrix instruction j of an 8-deep group multiplies kk = j (lanes 0-31) and kk = j + 4 (lanes 32-63) of both operands, so
// either image serves either operand.
//
// [2000, 750] x [750, 1500], 4 devices: 4653 us with one element per lane (gemm_generic_kernel), 177 here (102 TFLOP/s);
// [1024, 512] x [512, 12500], 4 devices: 442 us (119 TFLOP/s).
//
// WK > 1: the waves also split the reduction (8-deep groups in turn), and their partial tiles are added through LDS in
// wave order: few output tiles with a long reduction.
#include "gemm_device.h"

namespace sbp {
namespace {

typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
typedef u16x4 __attribute__((aligned(2))) u16x4_any;

template <typename T>
__device__ inline f32x4 load4(const T* at) {
    if constexpr (sizeof(T) == 4) return *reinterpret_cast<const f32x4_any*>(at);
    else {
        const u16x4 v = *reinterpret_cast<const u16x4_any*>(at);
        return f32x4{bf16_to_f32(v[0]), bf16_to_f32(v[1]), bf16_to_f32(v[2]), bf16_to_f32(v[3])};
    }
}
template <typename T>
__device__ inline float load1(const T* at) {
    if constexpr (sizeof(T) == 4) return *at;
    else return bf16_to_f32(*at);
}

// One operand: R rows (m or n) by BK of the reduction per stage.
template <typename T, int R, bool KC, int BK, int NT>
struct Operand {
    static constexpr int PITCH = KC ? BK + 4 : R + 8;             // floats
    static constexpr int FLOATS = KC ? R * PITCH : BK * PITCH;    // per stage
    static constexpr int CPR = KC ? BK / 4 : R / 4;               // chunks per stored row
    static constexpr int CHUNKS = R * BK / 4, PER_THREAD = CHUNKS / NT;
    static_assert(CHUNKS % NT == 0, "chunks divide over the workgroup");

    const T* at[PER_THREAD];   // this thread's chunks in the current stage (rows past the end: the last row's)
    int64_t step;

    __device__ void open(const void* base, int ld, int first, int limit, int tid) {
#pragma unroll
        for (int i = 0; i < PER_THREAD; ++i) {
            const int p = i * NT + tid, row = p / CPR, c = p % CPR * 4;
            if constexpr (KC) {
                const int g = first + row < limit ? first + row : limit - 1;
                at[i] = static_cast<const T*>(base) + (int64_t)g * ld + c;
            } else {
                const int col = first + c < limit ? first + c : 0;
                at[i] = static_cast<const T*>(base) + (int64_t)row * ld + col;
            }
        }
        step = KC ? BK : (int64_t)BK * ld;
    }
    __device__ void fetch(f32x4 (&r)[PER_THREAD]) {
#pragma unroll
        for (int i = 0; i < PER_THREAD; ++i) r[i] = load4(at[i]);
    }
    __device__ void advance(bool on) {
#pragma unroll
        for (int i = 0; i < PER_THREAD; ++i) at[i] += on ? step : 0;
    }
    // a stage that reaches the end of the reduction or of the memory: zeros behind kk, element by element where a chunk
    // straddles an end; k0: first reduction index of the stage
    __device__ void fetch_tail(f32x4 (&r)[PER_THREAD], const void* base, int ld, int first, int limit, int kk, int k0, int tid) {
#pragma unroll
        for (int i = 0; i < PER_THREAD; ++i) {
            const int p = i * NT + tid, row = p / CPR, c = p % CPR * 4;
            const T* src;
            int valid;
            if constexpr (KC) {
                const int g = first + row < limit ? first + row : limit - 1;
                src = static_cast<const T*>(base) + (int64_t)g * ld + k0 + c;
                valid = kk - (k0 + c);
            } else {
                src = static_cast<const T*>(base) + (int64_t)(k0 + row) * ld + first + c;
                valid = k0 + row < kk ? limit - (first + c) : 0;
            }
            r[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            if (valid >= 4) r[i] = load4(src);
            else {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (e < valid) r[i][e] = load1(src + e);
            }
        }
    }
    __device__ static void stash(float* st, const f32x4 (&r)[PER_THREAD], int tid) {
#pragma unroll
        for (int i = 0; i < PER_THREAD; ++i) {
            const int p = i * NT + tid;
            *reinterpret_cast<f32x4*>(st + p / CPR * PITCH + p % CPR * 4) = r[i];
        }
    }
    // the four instructions' values of 32-row block blk (from row base on) in 8-deep group grp
    __device__ static f32x4 frag(const float* st, int base, int blk, int grp, int lane) {
        const int row = base + blk * 32 + (lane & 31), k = grp * 8 + (lane >> 5) * 4;
        if constexpr (KC) return *reinterpret_cast<const f32x4*>(st + row * PITCH + k);
        else return f32x4{st[k * PITCH + row], st[(k + 1) * PITCH + row], st[(k + 2) * PITCH + row], st[(k + 3) * PITCH + row]};
    }
};

template <int BM, int BN, int BK, int WM, int WN, int WK, typename TA, typename TB, bool A_KC, bool B_KC>
constexpr int f32_tile_floats() {
    constexpr int NT = WM * WN * WK * 64, stages = 2 * (Operand<TA, BM, A_KC, BK, NT>::FLOATS + Operand<TB, BN, B_KC, BK, NT>::FLOATS);
    constexpr int sum = WK > 1 ? WK * BM * BN : 0;
    return stages > sum ? stages : sum;
}
// The tile at (m0, n0) of s; smem: f32_tile_floats of them.  All threads of the workgroup.
template <int BM, int BN, int BK, int WM, int WN, int WK, typename TA, typename TB, bool A_KC, bool B_KC, int EPI>
__device__ inline void f32_tile(const GemmShard& s, int m0, int n0, float* smem) {
    constexpr int NT = WM * WN * WK * 64, TM = BM / WM, TN = BN / WN, FM = TM / 32, FN = TN / 32;
    constexpr int GROUPS = BK / 8 / WK;   // 8-deep groups of a stage per wave
    using OA = Operand<TA, BM, A_KC, BK, NT>;
    using OB = Operand<TB, BN, B_KC, BK, NT>;
    constexpr int STAGE = OA::FLOATS + OB::FLOATS;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave / (WM * WN), wm = wave / WN % WM, wn = wave % WN;

    f32x16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    // Stages whose chunks may be read without a look at the ends: a chunk of a not-KC operand may run past the end of
    // its row into the next one, so the stage with the last row is left to the careful path.
    int plain = (s.kk - (A_KC && B_KC ? 0 : 1)) / BK;
    if ((!A_KC && s.lda < 4) || (!B_KC && s.ldb < 4)) plain = 0;
    if (s.kk == 0) plain = 0;
    const int stages = (s.kk + BK - 1) / BK;

    OA oa;
    OB ob;
    oa.open(s.a, s.lda, m0, s.m, tid);
    ob.open(s.b, s.ldb, n0, s.n, tid);
    f32x4 ra[OA::PER_THREAD], rb[OB::PER_THREAD];
    auto fetch_plain = [&](int t) {
        oa.fetch(ra);
        ob.fetch(rb);
        oa.advance(t + 1 < plain);
        ob.advance(t + 1 < plain);
    };
    auto fetch = [&](int t) {   // t is uniform
        if (t < plain) fetch_plain(t);
        else {
            oa.fetch_tail(ra, s.a, s.lda, m0, s.m, s.kk, t * BK, tid);
            ob.fetch_tail(rb, s.b, s.ldb, n0, s.n, s.kk, t * BK, tid);
        }
    };
    auto stash = [&](float* st) {
        OA::stash(st, ra, tid);
        OB::stash(st + OA::FLOATS, rb, tid);
    };
    auto multiply = [&](const float* st) {
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
            f32x4 fa[FM], fb[FN];
#pragma unroll
            for (int i = 0; i < FM; ++i) fa[i] = OA::frag(st, wm * TM, i, g * WK + wk, lane);
#pragma unroll
            for (int j = 0; j < FN; ++j) fb[j] = OB::frag(st + OA::FLOATS, wn * TN, j, g * WK + wk, lane);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][e], fb[j][e], acc[i][j], 0, 0, 0);
        }
    };
    if (stages > 0) {
        fetch(0);
        stash(smem);
        __syncthreads();
        int t = 0;
        // A loop without the careful path: jumping over it in every stage costs 3 to 12 %, by where the code happens to lie.  (bf16 values
        // are widened where they are loaded, so that they cannot be held back like that.)
        for (; sizeof(TA) == 4 && sizeof(TB) == 4 && t + 1 < plain; ++t) {
            fetch_plain(t + 1);
            __builtin_amdgcn_sched_barrier(0);   // the loads first and what waits for them last
            multiply(smem + (t & 1) * STAGE);
            __builtin_amdgcn_sched_barrier(0);
            stash(smem + ((t + 1) & 1) * STAGE);
            __syncthreads();
        }
        for (; t < stages; ++t) {
            if (t + 1 < stages) fetch(t + 1);
            multiply(smem + (t & 1) * STAGE);
            if (t + 1 < stages) stash(smem + ((t + 1) & 1) * STAGE);
            __syncthreads();
        }
    }

    auto finish = [](float v) {
        if constexpr (EPI == SBP_EPI_GELU) return gelu_erf(v);
        else return v;
    };
    float* const C = static_cast<float*>(s.c);
    // acc[i][j][r] is row 8 (r / 4) + 4 (lane / 32) + r % 4, column lane % 32 of its block: 128 bytes of a row per half-wave
    if constexpr (WK == 1) {
        const int n = n0 + wn * TN + (lane & 31), mb = m0 + wm * TM + 4 * (lane >> 5);
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int m = mb + i * 32 + 8 * (r >> 2) + (r & 3);
                    if (m < s.m && n + j * 32 < s.n) C[(int64_t)m * s.ldc + n + j * 32] = finish(acc[i][j][r]);
                }
    } else {
        // every stage ends with a barrier: the stages are free.  [wk][row of the tile][column]
        constexpr int TILE = BM * BN;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    smem[wk * TILE + (wm * TM + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * BN + wn * TN + j * 32 + (lane & 31)] = acc[i][j][r];
        __syncthreads();
#pragma unroll
        for (int o = 0; o < TILE / NT; ++o) {
            const int e = o * NT + tid, m = m0 + e / BN, n = n0 + e % BN;
            float v = smem[e];
#pragma unroll
            for (int w = 1; w < WK; ++w) v += smem[w * TILE + e];
            if (m < s.m && n < s.n) C[(int64_t)m * s.ldc + n] = finish(v);
        }
    }
}

template <int BM, int BN, int BK, int WM, int WN, int WK, typename TA, typename TB, bool A_KC, bool B_KC, int EPI>
__global__ __launch_bounds__(WM * WN * WK * 64) void gemm_f32_kernel(GemmPlan p, int tm, int tn, int order) {
    __shared__ __attribute__((aligned(16))) float smem[f32_tile_floats<BM, BN, BK, WM, WN, WK, TA, TB, A_KC, B_KC>()];
    const TileCoord tc = map_tile(blockIdx.x, gridDim.x, tm, tn, p.groups, order);
    if (!tc.valid) return;
    const GemmShard s = p.s[tc.g];
    const int m0 = tc.tile_m * BM, n0 = tc.tile_n * BN;
    if (m0 >= s.m || n0 >= s.n) return;
    f32_tile<BM, BN, BK, WM, WN, WK, TA, TB, A_KC, B_KC, EPI>(s, m0, n0, smem);
}

// ---------------------------------------------------------------------------------------------------------------------
// gemm_terms_kernel: the same products on v_mfma_f32_16x16x32_bf16.  An fp32 operand is cut, exactly, into three bf16 terms on its way
// into LDS, and all products of terms that reach 2^-24 of the whole enter the fp32 accumulator, the small ones first: six of nine
// for fp32 x fp32, three for fp32 x bf16.  16 times the fp32 instruction's rate for six times the instructions, and fewer
// roundings of the accumulator: error against float64 on N(0, 1) x N(0, 0.1), relative 2-norm, terms / fp32 128 x 128 and 64 x 64 /
// fp32 32 x 32: length 16 3.4e-8 / 7.4e-8 / 6.0e-8, 128 1.5e-7 / 2.0e-7 / 0.9e-7, 1000 4.8e-7 / 5.7e-7 / 2.1e-7, 16000 2.1e-6 / 2.3e-6 /
// 0.8e-6; on uniform values in [0, 1] at 1000 2.9e-7 / 4.2e-7 / 0.7e-7.
//
// Products as sums of bf16 terms: Henry, Tang, Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For
// Higher-Precision Computations" (2019).
//
// A value is scaled by 2^24 before the cut, which is exact and brings the last bit of the smallest one, 2^-149, into the range of bf16; the
// results are scaled back.  What the cut cannot hold then (infinities, values of 2^104 and more, sums that leave the fp32 range on
// the way) shows as a result that is not finite; such a tile is multiplied again by f32_tile.  NaN stays NaN either way.
// (A look at every value for small ones, and a second multiplication of their tiles, took 106 and 674 us where this takes 105 and 654
// below, and twice as long where there were any.)
//
// Bound by the power limit of the matrix cores: [4096, 4096] x [4096, 4096] 654 us, 1.26 PFLOP/s of bf16 products (1064 us on the
// fp32 instruction).  [2000, 750] x [750, 1500], 4 devices, 152 -> 105.  Four waves; one LDS stage of 48 KB,
// so that three workgroups of 168 registers a wave share a compute unit: one splits while others multiply (two of them with a
// register stage ahead: 110 us).  Six terms for 64 x 64 results a wave read 24 KB of fragments per 96 matrix instructions, half of
// what LDS can deliver meanwhile; splitting a fragment after the read would read two thirds of that and split everything twice.
// ---------------------------------------------------------------------------------------------------------------------
// x 2^24 = hi + mid + lo, each the nearest bf16 of what is left; pairs of values.  Exact below 2^104 in magnitude.
constexpr int CUT_EXP = 24;
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
// x minus one half of a pair of terms.  ONE_ROW: in one instruction where a shift or mask and a subtraction take two; exact as well, the
// difference being an fp32 value.  It multiplies the other half by 0, so that an infinity or NaN there shows in x too: fit for two
// values of one row, not for two columns, one of which may be padding.  It pays next to bf16 with 64 x 64 tiles, where cutting takes as
// long as multiplying: [252, 3016] x [3016, 1013], both reduction-contiguous, 3 devices, 47.2 / 39.8 us, 0.85-1.02 of the time over 378 shapes; with
// 128 x 128 tiles 0.98-1.11, two fp32 operands 0.96-1.12.
template <bool ONE_ROW, int HALF>
__device__ inline float minus_term(float x, uint32_t pair) {
    if constexpr (ONE_ROW) {
        uint32_t minus = HALF ? 0xBF800000u : 0x0000BF80u;   // -1 in that half; in a register: as a constant of the instruction both become the first
        asm("" : "+s"(minus));
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), __builtin_bit_cast(bf16x2, minus), x, false);
    } else return x - __uint_as_float(HALF ? pair & 0xFFFF0000u : pair << 16);
}
struct TermPair { uint32_t hi, mid, lo; };
template <bool ONE_ROW>   // both values of one row along the reduction
__device__ inline TermPair split_pair(float x, float y) {
    TermPair t;
    x *= (float)(1 << CUT_EXP);
    y *= (float)(1 << CUT_EXP);
    t.hi = f32_to_bf16x2(x, y);
    x = minus_term<ONE_ROW, 0>(x, t.hi);
    y = minus_term<ONE_ROW, 1>(y, t.hi);
    t.mid = f32_to_bf16x2(x, y);
    x = minus_term<ONE_ROW, 0>(x, t.mid);
    y = minus_term<ONE_ROW, 1>(y, t.mid);
    t.lo = f32_to_bf16x2(x, y);
    return t;
}

// One operand of gemm_terms_kernel: R rows by 32 of the reduction a stage, as one (bf16) or three (fp32) bf16 tiles.
template <typename T, int R, bool KC, int NT, bool ONE_F32>   // ONE_F32: the other operand is bf16
struct TermOperand {
    using Tl = Tile<R, KC, NT, 32, true>;
    static constexpr bool F32 = sizeof(T) == 4;
    static constexpr int N = F32 ? 3 : 1, PER = Tl::PER_THREAD, BYTES = N * Tl::BYTES, WORDS = F32 ? 8 : 4;
    struct Raw { u32x4 v[PER][WORDS / 4]; };

    const T* at[PER];   // this thread's chunks (eight elements) in the current stage
    int64_t step;

    // where chunk p lies; rows past the end: the last one's, columns past the end: the first ones
    __device__ static const T* origin(const T* base, int ld, int first, int limit, int p, int k0) {
        if constexpr (KC) {
            const int row = p / Tl::CPK, g = first + row < limit ? first + row : limit - 1;
            return base + (int64_t)g * ld + k0 + ((p % Tl::CPK) ^ Tl::ksw(row)) * 8;
        } else {
            const int krow = p / Tl::CPR, col = first + ((p % Tl::CPR) ^ nswz<R>(krow)) * 8;
            return base + (int64_t)(k0 + krow) * ld + (col < limit ? col : 0);
        }
    }
    __device__ void open(const void* base, int ld, int first, int limit, int tid) {
#pragma unroll
        for (int i = 0; i < PER; ++i) at[i] = origin(static_cast<const T*>(base), ld, first, limit, i * NT + tid, 0);
        step = KC ? 32 : (int64_t)32 * ld;
    }
    __device__ void fetch(Raw& r, bool on) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
#pragma unroll
            for (int w = 0; w < WORDS / 4; ++w) r.v[i][w] = *reinterpret_cast<const u32x4_any*>(reinterpret_cast<const char*>(at[i]) + 16 * w);
            at[i] += on ? step : 0;
        }
    }
    // a stage that reaches the end of the reduction or of the memory: zeros behind kk and behind the end of a row
    __device__ static void fetch_tail(Raw& r, const void* base, int ld, int first, int limit, int kk, int k0, int tid) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int p = i * NT + tid;
            const T* src;
            int valid;
            if constexpr (KC) {
                const int row = p / Tl::CPK, g = first + row < limit ? first + row : limit - 1, k = k0 + ((p % Tl::CPK) ^ Tl::ksw(row)) * 8;
                src = static_cast<const T*>(base) + (int64_t)g * ld + k;
                valid = kk - k;
            } else {
                const int krow = p / Tl::CPR, col = first + ((p % Tl::CPR) ^ nswz<R>(krow)) * 8;
                src = static_cast<const T*>(base) + (int64_t)(k0 + krow) * ld + col;
                valid = k0 + krow < kk ? limit - col : 0;
            }
#pragma unroll
            for (int w = 0; w < WORDS / 4; ++w) r.v[i][w] = u32x4{0u, 0u, 0u, 0u};
            if (valid >= 8) {   // element by element [2197, 64] x [64, 445] took 7.0 us, 5.7 on the fp32 instruction
#pragma unroll
                for (int w = 0; w < WORDS / 4; ++w) r.v[i][w] = *reinterpret_cast<const u32x4_any*>(reinterpret_cast<const char*>(src) + 16 * w);
            } else {
#pragma unroll
                for (int e = 0; e < 7; ++e)
                    if (e < valid) {
                        if constexpr (F32) r.v[i][e >> 2][e & 3] = __float_as_uint(src[e]);
                        else r.v[i][0][e >> 1] |= (uint32_t)src[e] << (16 * (e & 1));
                    }
            }
        }
    }
    __device__ static void stash(char* st, Raw& r, int tid) {   // into LDS
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            char* const to = st + (i * NT + tid) * 16;
            if constexpr (F32) {
                asm volatile("" : "+v"(r.v[i][0]), "+v"(r.v[i][1]));   // split here and not where it was loaded: three terms take more registers
                u32x4 h, m, l;
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const TermPair t = split_pair<KC && ONE_F32 && R == 64>(__uint_as_float(r.v[i][d >> 1][2 * (d & 1)]), __uint_as_float(r.v[i][d >> 1][2 * (d & 1) + 1]));
                    h[d] = t.hi;
                    m[d] = t.mid;
                    l[d] = t.lo;
                }
                *reinterpret_cast<u32x4*>(to) = h;
                *reinterpret_cast<u32x4*>(to + Tl::BYTES) = m;
                *reinterpret_cast<u32x4*>(to + 2 * Tl::BYTES) = l;
            } else {
                *reinterpret_cast<u32x4*>(to) = r.v[i][0];
            }
        }
    }
};

template <int BM, int BN, int WPS, typename T1, typename T2, bool A_KC, bool B_KC, int EPI>
__global__ __launch_bounds__(256, WPS) void gemm_terms_kernel(GemmPlan p, int tm, int tn, int order) {
    constexpr int NT = 256, TM = BM / 2, TN = BN / 2, FM = TM / 16, FN = TN / 16, BLOCKS = FM * FN;
    constexpr bool ONE_F32 = sizeof(T1) != sizeof(T2);
    using OA = TermOperand<T1, BM, A_KC, NT, ONE_F32>;
    using OB = TermOperand<T2, BN, B_KC, NT, ONE_F32>;
    // The next stage is loaded ahead of the multiplication where its registers fit beside the fragments; with 128 x 128 tiles of
    // three terms each they do not, and three workgroups a compute unit cover the loads' latency instead.
    constexpr bool AHEAD = BM < 128 || !(OA::F32 && OB::F32);
    constexpr int STAGE = OA::BYTES + OB::BYTES, F32_BYTES = 4 * f32_tile_floats<BM, BN, BM == 128 ? 16 : 32, 2, 2, 1, T1, T2, A_KC, B_KC>();
    __shared__ __attribute__((aligned(1024))) char smem[STAGE > F32_BYTES ? STAGE : F32_BYTES];

    const TileCoord tc = map_tile(blockIdx.x, gridDim.x, tm, tn, p.groups, order);
    if (!tc.valid) return;
    const GemmShard s = p.s[tc.g];
    const int m0 = tc.tile_m * BM, n0 = tc.tile_n * BN;
    if (m0 >= s.m || n0 >= s.n) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int loa = OA::Tl::lane_offset16(wm * TM, lane), lob = OB::Tl::lane_offset16(wn * TN, lane);

    // stages whose chunks may be read without a look at the ends (see f32_tile)
    int plain = (s.kk - (A_KC && B_KC ? 0 : 1)) / 32;
    if (s.kk == 0 || (!A_KC && s.lda < 8) || (!B_KC && s.ldb < 8)) plain = 0;
    const int stages = (s.kk + 31) / 32;
    OA oa;
    OB ob;
    oa.open(s.a, s.lda, m0, s.m, tid);
    ob.open(s.b, s.ldb, n0, s.n, tid);
    typename OA::Raw ra;
    typename OB::Raw rb;
    // LDS traffic of this wave done, then all waves: the loads into registers stay in flight
    auto barrier = []() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    auto stash = [&]() {
        OA::stash(smem, ra, tid);
        OB::stash(smem + OA::BYTES, rb, tid);
    };
    auto multiply = [&]() {
        bf16x8 fa[2][OA::N], fb[OB::N][FN];
        auto read_a = [&](int i) {
#pragma unroll
            for (int u = 0; u < OA::N; ++u) fa[i & 1][u] = OA::Tl::frag16(smem + u * OA::Tl::BYTES, loa, i);
        };
        read_a(0);
#pragma unroll
        for (int u = OB::N - 1; u >= 0; --u)
#pragma unroll
            for (int j = 0; j < FN; ++j) fb[u][j] = OB::Tl::frag16(smem + OA::BYTES + u * OB::Tl::BYTES, lob, j);
        static_for<FM>([&](auto ix) {
            constexpr int i = decltype(ix)::value;
            if constexpr (i + 1 < FM) read_a(i + 1);
            // terms of order 2 (hi lo, mid mid, lo hi), 1 and 0, small ones first; those of order 3 and 4 are below 2^-25 of the product
#pragma unroll
            for (int o = 2; o >= 0; --o)
#pragma unroll
                for (int u = 0; u <= o; ++u)
                    if (u < OA::N && o - u < OB::N)
#pragma unroll
                        for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[o - u][j], fa[i & 1][u], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);   // no further reads ahead: they would not fit the registers
        });
    };
    auto fetch = [&](int next) {   // and on to stage `next`; past the last plain one the source stays: the reload is in bounds and unread
        oa.fetch(ra, next < plain);
        ob.fetch(rb, next < plain);
    };
    if (plain > 0) {
        fetch(1);
        for (int t = 0; t < plain; ++t) {
            stash();
            if constexpr (AHEAD) fetch(t + 2);
            barrier();
            multiply();
            if constexpr (!AHEAD) {
                fetch(t + 2);
                __builtin_amdgcn_sched_barrier(0);
            }
            barrier();
        }
    }
    for (int t = plain; t < stages; ++t) {
        OA::fetch_tail(ra, s.a, s.lda, m0, s.m, s.kk, t * 32, tid);
        OB::fetch_tail(rb, s.b, s.ldb, n0, s.n, s.kk, t * 32, tid);
        stash();
        barrier();
        multiply();
        barrier();
    }

    // Where a result is not finite: the tile again, in fp32.
    const int q = lane >> 4, r = lane & 15;
    bool odd = false;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (m0 + wm * TM + 16 * i + r < s.m && n0 + wn * TN + 16 * j + 4 * q + e < s.n) odd |= !(__builtin_fabsf(acc[i][j][e]) <= 3.4028234663852886e38f);
    uint32_t* const votes = reinterpret_cast<uint32_t*>(smem);
    barrier();
    votes[wave] = __builtin_amdgcn_ballot_w64(odd) != 0;
    barrier();
    uint32_t again = __builtin_amdgcn_readfirstlane(votes[0] | votes[1] | votes[2] | votes[3]);
    barrier();

    // Results through a private part of LDS, as in gemm_reg_kernel: eight consecutive lanes own 128 bytes of a row.
    constexpr int NB = BLOCKS < 8 ? BLOCKS : 8;   // blocks at a time
    constexpr float BACK = 1.0f / (float)((int64_t)1 << CUT_EXP * ((OA::F32 ? 1 : 0) + (OB::F32 ? 1 : 0)));
    static_assert(NB * 4096 <= (int)sizeof(smem) && BLOCKS % NB == 0 && NB % FN == 0 && FN % 2 == 0, "whole rows of blocks");
    char* const win = smem + wave * (NB * 1024);
    if (!again) {
        static_for<BLOCKS / NB>([&](auto rix) {
            constexpr int B0 = decltype(rix)::value * NB;
            static_for<NB>([&](auto bix) {
                constexpr int b = B0 + decltype(bix)::value;
                *reinterpret_cast<f32x4*>(win + decltype(bix)::value * 1024 + (16 * q + (r ^ (4 * q))) * 16) = acc[b / FN][b % FN];
            });
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll EPI == SBP_EPI_GELU ? 1 : 64
            for (int u = 0; u < NB; ++u) {
                const int blk = u / 2 * 2, row = u % 2 * 8 + lane / 8, cg = lane % 8;
                const f32x4 x = *reinterpret_cast<const f32x4*>(win + (blk + cg / 4) * 1024 + (16 * (cg & 3) + (row ^ (4 * (cg & 3)))) * 16);
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = EPI == SBP_EPI_GELU ? gelu_erf(x[e] * BACK) : x[e] * BACK;
                store_columns<float>(s, m0 + wm * TM + (B0 + blk) / FN * 16 + row, n0 + wn * TN + (B0 + blk) % FN * 16 + cg * 4, v);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        });
    }
    asm volatile("" : "+s"(again));   // a branch of its own: as one, both ways would be laid out so that the accumulators outlive the second one's
    if (again) f32_tile<BM, BN, BM == 128 ? 16 : 32, 2, 2, 1, T1, T2, A_KC, B_KC, EPI>(s, m0, n0, reinterpret_cast<float*>(smem));
}

// Tiles of gemm_f32_kernel, or (TERMS: waves per SIMD) of gemm_terms_kernel.
template <int TERMS, int BM, int BN, int BK, int WM, int WN, int WK, typename TA, typename TB, bool A_KC, bool B_KC, int EPI>
constexpr auto pick_kernel() {
    if constexpr (TERMS > 0) return gemm_terms_kernel<BM, BN, TERMS, TA, TB, A_KC, B_KC, EPI>;
    else return gemm_f32_kernel<BM, BN, BK, WM, WN, WK, TA, TB, A_KC, B_KC, EPI>;
}
template <int TERMS, int BM, int BN, int BK, int WM, int WN, int WK, typename TA, typename TB, int EPI>
int32_t launch_layout(const GemmPlan& plan, int max_m, int max_n, int order, hipStream_t st) {
    const int tm = tiles_along(max_m, BM), tn = tiles_along(max_n, BN);
    const int64_t nblk = ((int64_t)tm * tn * plan.groups + 7) / 8 * 8;
    if (!grid_fits(nblk, WM * WN * WK * 64)) return SBP_ERR_UNSUPPORTED;
    void (*kern)(GemmPlan, int, int, int);
    if (plan.a_kc) kern = plan.b_kc ? pick_kernel<TERMS, BM, BN, BK, WM, WN, WK, TA, TB, true, true, EPI>() : pick_kernel<TERMS, BM, BN, BK, WM, WN, WK, TA, TB, true, false, EPI>();
    else kern = plan.b_kc ? pick_kernel<TERMS, BM, BN, BK, WM, WN, WK, TA, TB, false, true, EPI>() : pick_kernel<TERMS, BM, BN, BK, WM, WN, WK, TA, TB, false, false, EPI>();
    hipLaunchKernelGGL(kern, dim3((uint32_t)nblk), dim3(WM * WN * WK * 64), 0, st, plan, tm, tn, order);
    return launch_status(__func__);
}

template <int TERMS, int BM, int BN, int BK, int WM, int WN, int WK>
int32_t launch_types(const GemmPlan& plan, int max_m, int max_n, int order, hipStream_t st) {
    if (plan.f32_operand == 1) return launch_layout<TERMS, BM, BN, BK, WM, WN, WK, float, uint16_t, SBP_EPI_NONE>(plan, max_m, max_n, order, st);
    if (plan.f32_operand == 2) return launch_layout<TERMS, BM, BN, BK, WM, WN, WK, uint16_t, float, SBP_EPI_NONE>(plan, max_m, max_n, order, st);
    if (plan.epilogue == SBP_EPI_GELU) return launch_layout<TERMS, BM, BN, BK, WM, WN, WK, float, float, SBP_EPI_GELU>(plan, max_m, max_n, order, st);
    if (plan.epilogue != SBP_EPI_NONE) return SBP_ERR_UNSUPPORTED;
    return launch_layout<TERMS, BM, BN, BK, WM, WN, WK, float, float, SBP_EPI_NONE>(plan, max_m, max_n, order, st);
}

}  // namespace

int32_t launch_gemm_f32(const GemmPlan& plan, int max_m, int max_n, int tile, int order, hipStream_t stream) {
    switch (tile) {
        case F32_128: return launch_types<0, 128, 128, 16, 2, 2, 1>(plan, max_m, max_n, order, stream);
        case F32_64: return launch_types<0, 64, 64, 32, 2, 2, 1>(plan, max_m, max_n, order, stream);
        case TERMS_128: return launch_types<3, 128, 128, 16, 2, 2, 1>(plan, max_m, max_n, order, stream);
        case TERMS_64: return launch_types<4, 64, 64, 32, 2, 2, 1>(plan, max_m, max_n, order, stream);
        case F32_32: return launch_types<0, 32, 32, 64, 1, 1, 8>(plan, max_m, max_n, order, stream);
        default: return SBP_ERR_UNSUPPORTED;
    }
}

}  // namespace sbp
