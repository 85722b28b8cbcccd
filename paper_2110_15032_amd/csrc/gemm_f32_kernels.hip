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

typedef f32x4 __attribute__((aligned(4))) f32x4_any;
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

template <int BM, int BN, int BK, int WM, int WN, int WK, typename TA, typename TB, bool A_KC, bool B_KC, int EPI>
__global__ __launch_bounds__(WM * WN * WK * 64) void gemm_f32_kernel(GemmPlan p, int tm, int tn, int order) {
    constexpr int NT = WM * WN * WK * 64, TM = BM / WM, TN = BN / WN, FM = TM / 32, FN = TN / 32;
    constexpr int GROUPS = BK / 8 / WK;   // 8-deep groups of a stage per wave
    using OA = Operand<TA, BM, A_KC, BK, NT>;
    using OB = Operand<TB, BN, B_KC, BK, NT>;
    constexpr int STAGE = OA::FLOATS + OB::FLOATS;
    constexpr int SUM = WK > 1 ? WM * WN * WK * TM * TN : 0;
    __shared__ __attribute__((aligned(16))) float smem[2 * STAGE > SUM ? 2 * STAGE : SUM];

    const TileCoord tc = map_tile(blockIdx.x, gridDim.x, tm, tn, p.groups, order);
    if (!tc.valid) return;
    const GemmShard s = p.s[tc.g];
    const int m0 = tc.tile_m * BM, n0 = tc.tile_n * BN;
    if (m0 >= s.m || n0 >= s.n) return;
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
    auto fetch = [&](int t) {   // t is uniform
        if (t < plain) {
            oa.fetch(ra);
            ob.fetch(rb);
            oa.advance(t + 1 < plain);
            ob.advance(t + 1 < plain);
        } else {
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
        for (int t = 0; t < stages; ++t) {
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

template <int BM, int BN, int BK, int WM, int WN, int WK, typename TA, typename TB, int EPI>
int32_t launch_layout(const GemmPlan& plan, int max_m, int max_n, int order, hipStream_t st) {
    const int tm = tiles_along(max_m, BM), tn = tiles_along(max_n, BN);
    const int64_t nblk = ((int64_t)tm * tn * plan.groups + 7) / 8 * 8;
    if (!grid_fits(nblk, WM * WN * WK * 64)) return SBP_ERR_UNSUPPORTED;
    void (*kern)(GemmPlan, int, int, int);
    if (plan.a_kc) kern = plan.b_kc ? gemm_f32_kernel<BM, BN, BK, WM, WN, WK, TA, TB, true, true, EPI> : gemm_f32_kernel<BM, BN, BK, WM, WN, WK, TA, TB, true, false, EPI>;
    else kern = plan.b_kc ? gemm_f32_kernel<BM, BN, BK, WM, WN, WK, TA, TB, false, true, EPI> : gemm_f32_kernel<BM, BN, BK, WM, WN, WK, TA, TB, false, false, EPI>;
    hipLaunchKernelGGL(kern, dim3((uint32_t)nblk), dim3(WM * WN * WK * 64), 0, st, plan, tm, tn, order);
    return launch_status(__func__);
}

template <int BM, int BN, int BK, int WM, int WN, int WK>
int32_t launch_types(const GemmPlan& plan, int max_m, int max_n, int order, hipStream_t st) {
    if (plan.f32_operand == 1) return launch_layout<BM, BN, BK, WM, WN, WK, float, uint16_t, SBP_EPI_NONE>(plan, max_m, max_n, order, st);
    if (plan.f32_operand == 2) return launch_layout<BM, BN, BK, WM, WN, WK, uint16_t, float, SBP_EPI_NONE>(plan, max_m, max_n, order, st);
    if (plan.epilogue == SBP_EPI_GELU) return launch_layout<BM, BN, BK, WM, WN, WK, float, float, SBP_EPI_GELU>(plan, max_m, max_n, order, st);
    if (plan.epilogue != SBP_EPI_NONE) return SBP_ERR_UNSUPPORTED;
    return launch_layout<BM, BN, BK, WM, WN, WK, float, float, SBP_EPI_NONE>(plan, max_m, max_n, order, st);
}

}  // namespace

int32_t launch_gemm_f32(const GemmPlan& plan, int max_m, int max_n, int tile, int order, hipStream_t stream) {
    switch (tile) {
        case F32_128: return launch_types<128, 128, 16, 2, 2, 1>(plan, max_m, max_n, order, stream);
        case F32_64: return launch_types<64, 64, 32, 2, 2, 1>(plan, max_m, max_n, order, stream);
        case F32_32: return launch_types<32, 32, 64, 1, 1, 8>(plan, max_m, max_n, order, stream);
        default: return SBP_ERR_UNSUPPORTED;
    }
}

}  // namespace sbp
