// Grouped bf16 GEMMs (sbp_matmul, paper Sec. 3.1, Table 1: device g computes C_g = A_g B_g) for what the 256 x 256 kernels
// are not made for: few output tiles, and rows that do not start 16-byte aligned.
//
// gemm_wavek_kernel: the waves of a workgroup split the REDUCTION instead of the output tile.  Every wave multiplies the
// whole BM x BN tile, on every NW-th 32-deep stage, and the NW partial tiles are added through LDS at the end.
//
// What that buys (us, 8 devices, [32, 4096] x [4096, 2048] each: 45.8 with the 128 x 128 tile of gemm_mfma_kernel, 35.6
// with that of gemm_mfma_pipe16_kernel, 24.7 here, 5.4 TB/s of weights; feature gradient of a classifier, 4 devices,
// [300, 30000] x [30000, 256]: 340 against 108):
//   * A wave fills a private pair of LDS stages and waits for its own loads only; the reduction loop has no barrier.
//   * Small tiles keep many loads in flight: eight waves bring eight consecutive stages at a time, so a product with
//     few output tiles (a batch of single tokens, the feature gradient of a narrow classifier) streams its operands
//     instead of waiting for one stage after the other.
//   * The fragment reads per matrix instruction are those of the whole tile, not of a wave's quarter of it: 64 x 64
//     per wave reads 8 fragments for 16 instructions, where 32 x 32 reads 4 for 4.
// The price is the final addition (BM BN NW floats through LDS, one or two microseconds).  A 128 x 128 tile per wave does
// not fit the registers (256 accumulators and two sets of 64 fragment registers spill).
//
// gemm_reg_kernel: the waves split the output tile as usual; operands of any pitch through registers.  Bound by the
// unaligned loads and the LDS writes: 540 TFLOP/s on [1500, 1501] x [1501, 2501], 2 devices, where the one-element-per-lane
// kernel reached 4.
//
// Matrix instruction: v_mfma_f32_16x16x32_bf16 fed (B fragment, A fragment), so that a lane's four accumulators are
// four consecutive columns of one row.  DIRECT: rows of both operands start 16-byte aligned, operands go global -> LDS
// directly, fragments are read one stage ahead.  Otherwise (any pitch) the 16-byte chunks pass through registers, two
// stages ahead, with unaligned loads: one cache line more per load instruction at worst, against eight loads of single
// elements.
#include "gemm_device.h"

namespace sbp {
namespace {

constexpr int LGKM0_ONLY = 0xC07F;   // s_waitcnt lgkmcnt(0), vmcnt untouched

// Whole 32-deep stages whose 16-byte chunks may be read without a look at the ends, rows of any pitch: a chunk of a
// not-KC operand may run past the end of its row into the next one, so the stage with the last row is left to the
// careful path, and rows shorter than a chunk leave it everything.
template <bool A_KC, bool B_KC>
__device__ inline int plain_stages(const GemmShard& s) {
    if constexpr (A_KC && B_KC) return s.kk / 32;
    if ((!A_KC && s.lda < 8) || (!B_KC && s.ldb < 8)) return 0;
    return (s.kk - 1) / 32;
}

// Addition of the partial tiles of NW waves (FM x FN blocks of 16 x 16 each), wave order, NB blocks at a time through LDS: 1 KB per
// block and wave.
template <int NW, int FM, int FN>
constexpr int partial_blocks() { return FM * FN * NW <= 128 ? FM * FN : 128 / NW; }
template <int NW, int FM, int FN>
constexpr int partial_bytes() { return partial_blocks<NW, FM, FN>() * NW * 1024; }
template <int NW, int FM, int FN, int EPI, typename OutT>
__device__ __attribute__((always_inline)) inline void add_partial_tiles(const f32x4 (&acc)[FM][FN], char* smem, const GemmShard& s, int m0, int n0, int wave, int lane) {
    constexpr int NB = partial_blocks<NW, FM, FN>(), ROUNDS = FM * FN / NB, SIDE = sizeof(OutT) == 4 ? 2 : 4;
    static_assert(FM * FN % NB == 0 && NB % SIDE == 0 && FN % SIDE == 0, "whole units of blocks side by side");
    // A block is kept as it lies in the registers:
    // row r = lane % 16, four columns from 4 q on, q = lane / 16, at (16 q + (r ^ 4 q)) * 16 (the exclusive-or spreads
    // the reads below over the banks).  Reading, eight consecutive lanes own the 128 (bf16: 64-column) bytes of a row.
    constexpr int EPV = 16 / (int)sizeof(OutT);           // columns per lane
    constexpr int UNIT = sizeof(OutT) == 4 ? 2 : 4;       // blocks side by side that eight lanes cover
    constexpr int UNITS = NB / UNIT * 2;                  // ... by eight rows: half the rows of a block
    const int q = lane >> 4, r = lane & 15;
    char* const dump = smem + wave * (NB * 1024) + (16 * q + (r ^ (4 * q))) * 16;
    static_for<ROUNDS>([&](auto rix) {
        constexpr int B0 = decltype(rix)::value * NB;
        __syncthreads();
        static_for<NB>([&](auto bix) {
            constexpr int b = B0 + decltype(bix)::value;
            *reinterpret_cast<f32x4*>(dump + decltype(bix)::value * 1024) = acc[b / FN][b % FN];
        });
        __syncthreads();
        for (int u = wave; u < UNITS; u += NW) {
            const int blk = u / 2 * UNIT, row = 8 * (u & 1) + (lane >> 3);
            const int m = m0 + (B0 + blk) / FN * 16 + row, n = n0 + (B0 + blk) % FN * 16 + (lane & 7) * EPV;
            float v[EPV];
#pragma unroll
            for (int h = 0; h < EPV / 4; ++h) {
                const int cg = (lane & 7) * (EPV / 4) + h;   // group of four columns: block cg / 4, q = cg % 4
                const char* at = smem + (blk + cg / 4) * 1024 + (16 * (cg & 3) + (row ^ (4 * (cg & 3)))) * 16;
                f32x4 sum = *reinterpret_cast<const f32x4*>(at);
#pragma unroll
                for (int w = 1; w < NW; ++w) sum += *reinterpret_cast<const f32x4*>(at + w * (NB * 1024));
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * h + e] = mfma_epilogue<EPI>(sum[e]);
            }
            store_columns<OutT>(s, m, n, v);
        }
    });
}

template <int BM, int BN, int NW, bool A_KC, bool B_KC, bool DIRECT, int EPI, typename OutT>
__global__ __launch_bounds__(NW * 64) void gemm_wavek_kernel(GemmPlan p, int tm, int tn, int order) {
    constexpr int BKT = 32, FM = BM / 16, FN = BN / 16;
    using TA = Tile<BM, A_KC, 64, BKT, true>;
    using TB = Tile<BN, B_KC, 64, BKT, true>;
    constexpr int NLA = TA::PER_THREAD, NLB = TB::PER_THREAD, NVM = NLA + NLB;   // 16-byte loads per stage
    constexpr int STAGE = TA::BYTES + TB::BYTES;
    constexpr int SMEM = NW * 2 * STAGE > partial_bytes<NW, FM, FN>() ? NW * 2 * STAGE : partial_bytes<NW, FM, FN>();
    static_assert(SMEM <= 160 * 1024 && NVM < 64, "tile does not fit the scheme");
    __shared__ __attribute__((aligned(1024))) char smem[SMEM];

    const TileCoord tc = map_tile(blockIdx.x, gridDim.x, tm, tn, p.groups, order);
    if (!tc.valid) return;
    const GemmShard s = p.s[tc.g];
    const int m0 = tc.tile_m * BM, n0 = tc.tile_n * BN;
    if (m0 >= s.m || n0 >= s.n) return;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    char* const st0 = smem + wave * (2 * STAGE);   // this wave's two stages: A tile, then B tile

    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int loa = TA::lane_offset16(0, lane), lob = TB::lane_offset16(0, lane);

    const int steps = DIRECT ? s.kk / BKT : plain_stages<A_KC, B_KC>(s);
    const int mine = steps > wave ? (steps - wave + NW - 1) / NW : 0;   // stages wave, wave + NW, ...
    gbl_char* A = (gbl_char*)s.a + (uint64_t)TA::step_bytes(s.lda) * (uint32_t)wave;
    gbl_char* B = (gbl_char*)s.b + (uint64_t)TB::step_bytes(s.ldb) * (uint32_t)wave;
    const uint64_t stepa = (uint64_t)TA::step_bytes(s.lda) * NW, stepb = (uint64_t)TB::step_bytes(s.ldb) * NW;
    uint32_t offa[NLA], offb[NLB];
#pragma unroll
    for (int it = 0; it < NLA; ++it) offa[it] = TA::src_offset(s.lda, m0, s.m, it * 64 + lane);
#pragma unroll
    for (int it = 0; it < NLB; ++it) offb[it] = TB::src_offset(s.ldb, n0, s.n, it * 64 + lane);
    int loaded = 0;
    auto advance = [&]() {   // past the last stage the source stays: the reload is in bounds and unread
        ++loaded;
        const bool adv = loaded < mine;
        A += adv ? stepa : 0u;
        B += adv ? stepb : 0u;
    };

    if constexpr (DIRECT) {
        bf16x8 fa[2][FM], fb[2][FN];
        auto issue = [&](char* st) {
            TA::load_direct_untracked(st, A, offa, 0);
            TB::load_direct_untracked(st + TA::BYTES, B, offb, 0);
            advance();
        };
        auto read = [&](const char* st, int set) {
#pragma unroll
            for (int j = 0; j < FN; ++j) fb[set][j] = TB::frag16(st + TA::BYTES, lob, j);
#pragma unroll
            for (int i = 0; i < FM; ++i) fa[set][i] = TA::frag16(st, loa, i);
        };
        // One stage: its fragments are in registers (set CUR), so its LDS stage takes the loads of the stage after the
        // next.  The upper row blocks are multiplied first, which gives the next stage's loads half a step more.
        auto step = [&](auto cur) {
            constexpr int CUR = decltype(cur)::value;
            __builtin_amdgcn_s_waitcnt(LGKM0_ONLY);
            issue(st0 + CUR * STAGE);
#pragma unroll
            for (int i = 0; i < FM / 2; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[CUR][j], fa[CUR][i], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(vmcnt_only(NVM));
            __builtin_amdgcn_sched_barrier(0);
            read(st0 + (1 - CUR) * STAGE, 1 - CUR);
#pragma unroll
            for (int i = FM / 2; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[CUR][j], fa[CUR][i], acc[i][j], 0, 0, 0);
            constexpr int NM = (FM - FM / 2) * FN, NDS = (A_KC ? FM : 2 * FM) + (B_KC ? FN : 2 * FN);
            static_for<NM>([&](auto i) {   // fragment reads spread over the matrix instructions
                constexpr int I = decltype(i)::value, nds = NDS * (I + 1) / NM - NDS * I / NM;
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if constexpr (nds > 0) __builtin_amdgcn_sched_group_barrier(0x100, nds, 0);
            });
        };
        if (mine > 0) {
            issue(st0);
            issue(st0 + STAGE);
            __builtin_amdgcn_s_waitcnt(vmcnt_only(NVM));
            __builtin_amdgcn_sched_barrier(0);
            read(st0, 0);
            int t = 0;
            for (; t + 2 <= mine; t += 2) {
                step(std::integral_constant<int, 0>{});
                step(std::integral_constant<int, 1>{});
            }
            if (mine & 1) step(std::integral_constant<int, 0>{});
            __builtin_amdgcn_s_waitcnt(0x0070);   // the unread trailing loads have landed before their stages are reused
        }
    } else {
        u32x4 ra[2][NLA], rb[2][NLB];
        auto fetch = [&](int set) {
#pragma unroll
            for (int it = 0; it < NLA; ++it) ra[set][it] = *(const __attribute__((address_space(1))) u32x4_any*)(A + offa[it]);
#pragma unroll
            for (int it = 0; it < NLB; ++it) rb[set][it] = *(const __attribute__((address_space(1))) u32x4_any*)(B + offb[it]);
            advance();
        };
        auto stash = [&](char* st, int set) {
#pragma unroll
            for (int it = 0; it < NLA; ++it) *reinterpret_cast<u32x4*>(st + (it * 64 + lane) * 16) = ra[set][it];
#pragma unroll
            for (int it = 0; it < NLB; ++it) *reinterpret_cast<u32x4*>(st + TA::BYTES + (it * 64 + lane) * 16) = rb[set][it];
        };
        auto multiply = [&](const char* st) {
            bf16x8 fb[FN];
#pragma unroll
            for (int j = 0; j < FN; ++j) fb[j] = TB::frag16(st + TA::BYTES, lob, j);
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                const bf16x8 fa = TA::frag16(st, loa, i);
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa, acc[i][j], 0, 0, 0);
            }
        };
        auto step = [&](auto cur) {   // stage t is in LDS (CUR), t + 1 and t + 2 are on their way in registers
            constexpr int CUR = decltype(cur)::value;
            stash(st0 + (1 - CUR) * STAGE, 1 - CUR);
            fetch(1 - CUR);
            multiply(st0 + CUR * STAGE);
            __builtin_amdgcn_wave_barrier();
        };
        if (mine > 0) {
            fetch(0);
            fetch(1);
            stash(st0, 0);
            fetch(0);
            int t = 0;
            for (; t + 2 <= mine; t += 2) {
                step(std::integral_constant<int, 0>{});
                step(std::integral_constant<int, 1>{});
            }
            if (mine & 1) step(std::integral_constant<int, 0>{});
        }
    }
    // what is left behind the whole stages: the next waves in turn, with every chunk checked against the ends
    for (int t = steps + (wave - steps % NW + NW) % NW; t * BKT < s.kk; t += NW) {
#pragma unroll
        for (int it = 0; it < NLA; ++it)
            *reinterpret_cast<u32x4*>(st0 + (it * 64 + lane) * 16) = TA::tail_chunk(static_cast<const uint16_t*>(s.a), s.lda, m0, s.m, s.kk, t * BKT, it * 64 + lane);
#pragma unroll
        for (int it = 0; it < NLB; ++it)
            *reinterpret_cast<u32x4*>(st0 + TA::BYTES + (it * 64 + lane) * 16) = TB::tail_chunk(static_cast<const uint16_t*>(s.b), s.ldb, n0, s.n, s.kk, t * BKT, it * 64 + lane);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        bf16x8 fb[FN];
#pragma unroll
        for (int j = 0; j < FN; ++j) fb[j] = TB::frag16(st0 + TA::BYTES, lob, j);
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const bf16x8 fa = TA::frag16(st0, loa, i);
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa, acc[i][j], 0, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }

    add_partial_tiles<NW, FM, FN, EPI, OutT>(acc, smem, s, m0, n0, wave, lane);
}

// gemm_rows_kernel: both operands reduction-contiguous, rows at any pitch, fp32 results, few output tiles: as gemm_wavek_kernel, every
// wave multiplies the whole tile on its 32 elements of each stage, but the stage is 256 deep and loaded by all waves together, so
// that a load instruction reads 512 consecutive bytes of two rows, not 64 of sixteen.  Bound by a compute unit's load path, which brings
// about 500 cache lines a microsecond from HBM where an instruction touches many rows and 860 where it touches two: [200, 7503] x
// [7503, 256], 4 devices, 40.1 us with gemm_wavek_kernel (32 x 64, 112 workgroups), 26.3 here; [512, 50000] x [50000, 64], 2
// devices, 291 / 120; [500, 62500] x [62500, 512], 8 devices, 1274 / 619 with 64 x 64.
template <int BM, int BN>
__global__ __launch_bounds__(512) void gemm_rows_kernel(GemmPlan p, int tm, int tn, int order) {
    constexpr int NW = 8, NT = 512, BKT = 256, ROWS = BM + BN, STAGE = ROWS * BKT * 2, PER = STAGE / 16 / NT, FM = BM / 16, FN = BN / 16;
    constexpr int SMEM = 2 * STAGE > partial_bytes<NW, FM, FN>() ? 2 * STAGE : partial_bytes<NW, FM, FN>();
    __shared__ __attribute__((aligned(1024))) char smem[SMEM];

    const TileCoord tc = map_tile(blockIdx.x, gridDim.x, tm, tn, p.groups, order);
    if (!tc.valid) return;
    const GemmShard s = p.s[tc.g];
    const int m0 = tc.tile_m * BM, n0 = tc.tile_n * BN;
    if (m0 >= s.m || n0 >= s.n) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // LDS: rows of A, then of B, 32 chunks of 16 bytes each; chunk c of a row lies at c ^ (row % 16), which puts the sixteen rows that
    // a fragment read takes from a chunk column, or from two neighbouring ones, on sixteen different groups of banks
    auto source = [&](int q) {
        const int row = q / 32, c = (q % 32) ^ (row % 16);
        return (row < BM ? static_cast<const uint16_t*>(s.a) + (int64_t)min(m0 + row, s.m - 1) * s.lda
                         : static_cast<const uint16_t*>(s.b) + (int64_t)min(n0 + row - BM, s.n - 1) * s.ldb) + c * 8;
    };
    const uint16_t* at[PER];
#pragma unroll
    for (int it = 0; it < PER; ++it) at[it] = source(it * NT + tid);
    u32x4 r[2][PER];
    const int steps = s.kk / BKT;
    // The rest of the reduction is a stage too, the first one.  Of its chunks (one place c for all of a lane's rows) the one that the
    // row ends in is read so that it ends with the row, and shifted in `trim`; those behind it likewise, and cleared.  With loads of
    // its own behind the last whole stage the rest cost 1 us of 7; trimmed as the last stage it took code that is fetched for
    // one use, and lengths of whole stages 0.7 us.
    static_assert(NT / 32 == 16, "rows of a lane are 16 apart");
    const int rest = s.kk - steps * BKT, left = rest - ((tid % 32) ^ (tid / 32 % 16)) * 8;   // left: from this lane's chunk of the rest on
    int loaded = 0;
    auto fetch = [&](int set) {   // past the last stage the source stays: the reload is in bounds and unread
        ++loaded;
#pragma unroll
        for (int it = 0; it < PER; ++it) {
            r[set][it] = *reinterpret_cast<const u32x4_any*>(at[it]);
            at[it] += loaded < steps ? BKT : 0;
        }
    };
    auto trim = [&](int set) {
        const int e = 8 - left;
#pragma unroll
        for (int it = 0; it < PER; ++it) {
            u32x4 v = r[set][it];
            if (e > 0) {
                if (e & 4) v = u32x4{v[2], v[3], 0u, 0u};
                if (e & 2) v = u32x4{v[1], v[2], v[3], 0u};
                if (e & 1) v = u32x4{v[0] >> 16 | v[1] << 16, v[1] >> 16 | v[2] << 16, v[2] >> 16 | v[3] << 16, v[3] >> 16};
                if (e >= 8) v = u32x4{0u, 0u, 0u, 0u};
            }
            r[set][it] = v;
        }
    };
    auto stash = [&](char* st, int set) {
#pragma unroll
        for (int it = 0; it < PER; ++it) *reinterpret_cast<u32x4*>(st + (it * NT + tid) * 16) = r[set][it];
    };
    const int lo = (lane & 15) * (BKT * 2) + (((4 * wave + (lane >> 4)) ^ (lane & 15)) << 4);
    auto multiply = [&](const char* st) {
        bf16x8 fa[FM], fb[FN];
#pragma unroll
        for (int i = 0; i < FM; ++i) fa[i] = *reinterpret_cast<const bf16x8*>(st + lo + i * 16 * BKT * 2);
#pragma unroll
        for (int j = 0; j < FN; ++j) fb[j] = *reinterpret_cast<const bf16x8*>(st + lo + (BM + j * 16) * BKT * 2);
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    };
    // LDS traffic of this wave done, then all waves: the loads into registers stay in flight
    auto barrier = []() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    auto step = [&](auto cur) {   // stage t is in LDS (CUR), t + 1 and t + 2 are on their way in registers
        constexpr int CUR = decltype(cur)::value;
        stash(smem + (1 - CUR) * STAGE, 1 - CUR);
        fetch(1 - CUR);
        multiply(smem + CUR * STAGE);
        barrier();
    };
    if (steps > 0) {
        if (rest) {
#pragma unroll
            for (int it = 0; it < PER; ++it) r[0][it] = *reinterpret_cast<const u32x4_any*>(at[it] + steps * BKT + min(left - 8, 0));
        } else fetch(0);
        fetch(1);
        if (rest) trim(0);
        stash(smem, 0);
        fetch(0);
        barrier();
        const int stages = steps + (rest ? 1 : 0);
        int t = 0;
        for (; t + 2 <= stages; t += 2) {
            step(std::integral_constant<int, 0>{});
            step(std::integral_constant<int, 1>{});
        }
        if (t < stages) step(std::integral_constant<int, 0>{});
    } else if (s.kk > 0) {   // less than a stage, zeros behind it in both operands
#pragma unroll
        for (int it = 0; it < PER; ++it) {
            const int q = it * NT + tid;
            const uint16_t* src = source(q);
            u32x4 v = {0u, 0u, 0u, 0u};
            if (left >= 8) v = *reinterpret_cast<const u32x4_any*>(src);
            else {
#pragma unroll
                for (int e = 0; e < 7; ++e)
                    if (e < left) v[e >> 1] |= (uint32_t)src[e] << (16 * (e & 1));
            }
            *reinterpret_cast<u32x4*>(smem + q * 16) = v;
        }
        __syncthreads();
        multiply(smem);
    }
    add_partial_tiles<NW, FM, FN, SBP_EPI_NONE, float>(acc, smem, s, m0, n0, wave, lane);
}

// 4 waves of BM/2 x BN/2, two 32-deep LDS stages filled from registers that run two stages ahead, one barrier a
// stage.  Two or three workgroups share a compute unit and cover each other's waits; a register ring of four stages was
// no faster (odd sizes 1500 x 1501 x 2501, 2 devices: 42.0 us with two stages, 43.2 with four).
template <int BM, int BN, bool A_KC, bool B_KC, int EPI, typename OutT>
__global__ __launch_bounds__(256, 2) void gemm_reg_kernel(GemmPlan p, int tm, int tn, int order) {
    constexpr int BKT = 32, NT = 256, TM = BM / 2, TN = BN / 2, FM = TM / 16, FN = TN / 16, BLOCKS = FM * FN;
    using TA = Tile<BM, A_KC, NT, BKT, true>;
    using TB = Tile<BN, B_KC, NT, BKT, true>;
    constexpr int NLA = TA::PER_THREAD, NLB = TB::PER_THREAD, STAGE = TA::BYTES + TB::BYTES;
    constexpr int DEPTH = 2;   // the register ring and the two LDS stages turn together
    __shared__ __attribute__((aligned(1024))) char smem[2 * STAGE];

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
    const int loa = TA::lane_offset16(wm * TM, lane), lob = TB::lane_offset16(wn * TN, lane);
    const int steps = plain_stages<A_KC, B_KC>(s);
    gbl_char* A = (gbl_char*)s.a;
    gbl_char* B = (gbl_char*)s.b;
    const uint32_t stepa = TA::step_bytes(s.lda), stepb = TB::step_bytes(s.ldb);
    uint32_t offa[NLA], offb[NLB];
#pragma unroll
    for (int it = 0; it < NLA; ++it) offa[it] = TA::src_offset(s.lda, m0, s.m, it * NT + tid);
#pragma unroll
    for (int it = 0; it < NLB; ++it) offb[it] = TB::src_offset(s.ldb, n0, s.n, it * NT + tid);
    int loaded = 0;
    u32x4 ra[DEPTH][NLA], rb[DEPTH][NLB];
    auto fetch = [&](int set) {   // past the last stage the source stays: the reload is in bounds and unread
#pragma unroll
        for (int it = 0; it < NLA; ++it) ra[set][it] = *(const __attribute__((address_space(1))) u32x4_any*)(A + offa[it]);
#pragma unroll
        for (int it = 0; it < NLB; ++it) rb[set][it] = *(const __attribute__((address_space(1))) u32x4_any*)(B + offb[it]);
        ++loaded;
        const bool adv = loaded < steps;
        A += adv ? stepa : 0u;
        B += adv ? stepb : 0u;
    };
    auto stash = [&](char* st, int set) {
#pragma unroll
        for (int it = 0; it < NLA; ++it) *reinterpret_cast<u32x4*>(st + (it * NT + tid) * 16) = ra[set][it];
#pragma unroll
        for (int it = 0; it < NLB; ++it) *reinterpret_cast<u32x4*>(st + TA::BYTES + (it * NT + tid) * 16) = rb[set][it];
    };
    auto multiply = [&](const char* st) {
        bf16x8 fb[FN];
#pragma unroll
        for (int j = 0; j < FN; ++j) fb[j] = TB::frag16(st + TA::BYTES, lob, j);
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const bf16x8 fa = TA::frag16(st, loa, i);
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa, acc[i][j], 0, 0, 0);
        }
    };
    // LDS traffic of this wave done, then all waves: the loads into registers stay in flight
    auto barrier = []() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    auto step = [&](auto tix) {   // stage t (= T mod DEPTH) is in LDS stage t & 1, the next DEPTH ones on their way
        constexpr int T = decltype(tix)::value, N = (T + 1) % DEPTH;
        stash(smem + (N & 1) * STAGE, N);
        fetch(N);
        multiply(smem + (T & 1) * STAGE);
        barrier();
    };
    if (steps > 0) {
        static_for<DEPTH>([&](auto d) { fetch(decltype(d)::value); });
        stash(smem, 0);
        fetch(0);
        barrier();
        int t = 0;
        for (; t + DEPTH <= steps; t += DEPTH) static_for<DEPTH>(step);
        static_for<DEPTH - 1>([&](auto d) {
            if (t + decltype(d)::value < steps) step(d);
        });
    }
    for (int t = steps; t * BKT < s.kk; ++t) {   // the rest, every chunk checked against the ends
#pragma unroll
        for (int it = 0; it < NLA; ++it)
            *reinterpret_cast<u32x4*>(smem + (it * NT + tid) * 16) = TA::tail_chunk(static_cast<const uint16_t*>(s.a), s.lda, m0, s.m, s.kk, t * BKT, it * NT + tid);
#pragma unroll
        for (int it = 0; it < NLB; ++it)
            *reinterpret_cast<u32x4*>(smem + TA::BYTES + (it * NT + tid) * 16) = TB::tail_chunk(static_cast<const uint16_t*>(s.b), s.ldb, n0, s.n, s.kk, t * BKT, it * NT + tid);
        __syncthreads();
        multiply(smem);
        __syncthreads();
    }

    // Results through a private part of LDS, layout as in gemm_wavek_kernel: LPR consecutive lanes own a row of UNIT blocks.
    constexpr int NB = 2 * STAGE / 4096 < BLOCKS ? 2 * STAGE / 4096 : BLOCKS;   // blocks at a time
    constexpr int EPV = 16 / (int)sizeof(OutT), UNIT = sizeof(OutT) == 4 || FN < 4 ? 2 : 4;
    constexpr int LPR = UNIT * 16 / EPV, ROWS = 64 / LPR;
    static_assert(BLOCKS % NB == 0 && NB % FN == 0 && FN % UNIT == 0, "whole rows of blocks");
    char* const win = smem + wave * (NB * 1024);
    const int q = lane >> 4, r = lane & 15;
    static_for<BLOCKS / NB>([&](auto rix) {
        constexpr int B0 = decltype(rix)::value * NB;
        static_for<NB>([&](auto bix) {
            constexpr int b = B0 + decltype(bix)::value;
            *reinterpret_cast<f32x4*>(win + decltype(bix)::value * 1024 + (16 * q + (r ^ (4 * q))) * 16) = acc[b / FN][b % FN];
        });
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll EPI == EPI_GELU_ERF ? 1 : 64   // erfcf is long
        for (int u = 0; u < NB / UNIT * (16 / ROWS); ++u) {
            const int blk = u / (16 / ROWS) * UNIT, row = u % (16 / ROWS) * ROWS + lane / LPR;
            float v[EPV];
#pragma unroll
            for (int h = 0; h < EPV / 4; ++h) {
                const int cg = (lane % LPR) * (EPV / 4) + h;
                const f32x4 x = *reinterpret_cast<const f32x4*>(win + (blk + cg / 4) * 1024 + (16 * (cg & 3) + (row ^ (4 * (cg & 3)))) * 16);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * h + e] = mfma_epilogue<EPI>(x[e]);
            }
            store_columns<OutT>(s, m0 + wm * TM + (B0 + blk) / FN * 16 + row, n0 + wn * TN + (B0 + blk) % FN * 16 + (lane % LPR) * EPV, v);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    });
}

// gemm_deep_kernel: 128 x 128 tile, rows 16-byte aligned, for products with about one such tile per compute unit.  Two groups
// of four waves (64 x 64 each) take the two 32-deep halves of every 64-deep stage; four stages, one barrier a stage, the
// two partial tiles added through LDS.
//   * Two waves per SIMD cover each other's waits, which one workgroup of gemm_mfma_pipe16_kernel per compute unit does not.
//   * A stage reads one cache line of a reduction-contiguous row, whole, wherever the row starts (LINES, Tile::line_offset): pieces
//     of 128 bytes that straddle two lines cost the load path twice (all lines in L2, rows 250000 bytes apart: 0.58 us a stage
//     against 0.35 with rows on lines).  A fragment then comes from two neighbouring stages, so that one stage less is in
//     flight; with every row on a line the stages are read as they are (with lines all the same [1500, 2048] x [2048, 1500] took
//     17.3 us, without 16.2).  Over the stages as they are, rows off lines: operands read from HBM 0.67-0.97, from the memory-side
//     cache 160 tiles and more 0.71-1.03, 100 to 128 tiles 1.00-1.07 up to length 1000, 0.71-1.07 up to 3000.
//   * The load path returns in order.  A stage of 32 KB takes 0.21 us when all of it is in L2 and 0.58 us when any of it comes from
//     HBM, whatever the number of stages in flight; operand tiles shared by the workgroups of an XCD are in L2 for all but the
//     first, but all of them wait for that one.  So the lines of four stages are touched at once, three stages ahead of their
//     loads, every workgroup the part that is its share among those that read the same tile: one wait for HBM in four stages (TOUCH).
// us, stages as they are / now: feature gradient of a classifier, 8 devices, [1024, 125000] x [125000, 512], left rows on lines 1475 / 1058, with both
// rows 250000 bytes apart 1915 / 1073, neither operand reduction-contiguous 1250 / 1099; without the touches 1168.  [1024, 16384] x
// [16384, 512] 160 / 148; [777, 1000] x [1000, 1000], 3 devices, 14.7 / 13.1.  Of the 0.54 us a stage that are left the multiplication
// and its LDS reads take 0.36.
// LINES: some row of a reduction-contiguous operand starts inside a cache line.  TOUCH: see touches_pay.
template <bool A_KC, bool B_KC, bool LINES, bool TOUCH, int EPI, typename OutT>
__global__ __launch_bounds__(512) void gemm_deep_kernel(GemmPlan p, int tm, int tn, int order) {
    constexpr int BM = 128, BN = 128, BKT = 64, NT = 512, NST = 4, FM = 4, FN = 4;
    using TA = Tile<BM, A_KC, NT, BKT, true>;
    using TB = Tile<BN, B_KC, NT, BKT, true>;
    constexpr int NVM = TA::PER_THREAD + TB::PER_THREAD, STAGE = TA::BYTES + TB::BYTES;
    constexpr bool LA_ = LINES && A_KC, LB_ = LINES && B_KC;   // operands that are loaded by whole lines
    static_assert(!LINES || A_KC || B_KC, "only rows along the reduction are pieced together");
    // Lines are touched this many stages ahead (5, 6 and 8 measured: within 2 % with a reduction-contiguous operand, 2 to 12 % slower
    // without), as long as a workgroup's share of four stages is not more than TOUCH_MAX.  us, with / without: share of 192 lines
    // 1073 / 1168 and 150.3 / 158.7, 288 182.7 / 178.3; neither operand reduction-contiguous 192 148.5 / 159.9, 288 165.5 / 176.3.
    constexpr int TOUCH_DIST = 7, TOUCH_MAX = A_KC || B_KC ? DEEP_TOUCH_MAX_KC : DEEP_TOUCH_MAX;
    static_assert(NST * STAGE == 8 * FM * FN * 1024, "the partial tiles fill the stages");
    __shared__ __attribute__((aligned(1024))) char smem[NST * STAGE + (TOUCH ? 256 : 0)];   // the last 256 bytes: what the touches bring

    const TileCoord tc = map_tile(blockIdx.x, gridDim.x, tm, tn, p.groups, order);
    if (!tc.valid) return;
    const GemmShard s = p.s[tc.g];
    const int m0 = tc.tile_m * BM, n0 = tc.tile_n * BN;
    if (m0 >= s.m || n0 >= s.n) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sub = wave & 3, half = wave >> 2, wm = sub >> 1, wn = sub & 1;

    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int loa = TA::lane_offset16(wm * 64, lane, half), lob = TB::lane_offset16(wn * 64, lane, half);

    const int steps = s.kk / BKT;
    // whole lines (line_offset): stage `steps` is the last one of a reduction-contiguous operand, steps - 1 of the other kind
    gbl_char* A = (gbl_char*)s.a - (LA_ ? 128 : 0);
    gbl_char* B = (gbl_char*)s.b - (LB_ ? 128 : 0);
    uint32_t offa[TA::PER_THREAD], offb[TB::PER_THREAD], enda[TA::PER_THREAD], endb[TB::PER_THREAD], begina[TA::PER_THREAD], beginb[TB::PER_THREAD];
#pragma unroll
    for (int it = 0; it < TA::PER_THREAD; ++it) {
        if constexpr (LA_) offa[it] = TA::line_offset(s.a, s.lda, m0, s.m, it * NT + tid, begina[it], enda[it]);
        else offa[it] = TA::src_offset(s.lda, m0, s.m, it * NT + tid), begina[it] = enda[it] = 0;
    }
#pragma unroll
    for (int it = 0; it < TB::PER_THREAD; ++it) {
        if constexpr (LB_) offb[it] = TB::line_offset(s.b, s.ldb, n0, s.n, it * NT + tid, beginb[it], endb[it]);
        else offb[it] = TB::src_offset(s.ldb, n0, s.n, it * NT + tid), beginb[it] = endb[it] = 0;
    }
    const uint32_t stepa = TA::step_bytes(s.lda), stepb = TB::step_bytes(s.ldb);
    int loaded = 0;
    enum Issue { FIRST, INNER, ANY };   // INNER: the stages up to the one loaded are whole, and another follows
    auto issue = [&](char* st, auto kind) {   // past the last stage the source stays: the reload is in bounds and unread
        constexpr Issue KIND = decltype(kind)::value;
        if constexpr (KIND == INNER) {
            TA::load_direct_untracked(st, A, offa, wave);
            TB::load_direct_untracked(st + TA::BYTES, B, offb, wave);
            ++loaded;
            A += stepa;
            B += stepb;
            return;
        }
        constexpr bool first = KIND == FIRST;
        const uint32_t last = !first && loaded >= steps ? ~0u : 0u;
        uint32_t oa[TA::PER_THREAD], ob[TB::PER_THREAD];
#pragma unroll
        for (int it = 0; it < TA::PER_THREAD; ++it) oa[it] = !LA_ ? offa[it] : first ? offa[it] + begina[it] : offa[it] - (enda[it] & last);
#pragma unroll
        for (int it = 0; it < TB::PER_THREAD; ++it) ob[it] = !LB_ ? offb[it] : first ? offb[it] + beginb[it] : offb[it] - (endb[it] & last);
        TA::load_direct_untracked(st, A, oa, wave);
        TB::load_direct_untracked(st + TA::BYTES, B, ob, wave);
        ++loaded;
        A += loaded < steps + (LA_ ? 1 : 0) ? stepa : 0u;
        B += loaded < steps + (LB_ ? 1 : 0) ? stepb : 0u;
    };
    // this workgroup's share of the lines of NST stages, one per lane; worked out while the first stages are on their way
    const char* touch = static_cast<const char*>(s.a);
    uint32_t touch_step = 0;
    uint64_t touch_lanes = 0;
    auto share_touches = [&]() {
        const Sharers sh = tile_sharers(blockIdx.x, gridDim.x, tm, tn, p.groups, order);
        constexpr int LA = TA::template touch_lines<NST>(), LB = TB::template touch_lines<NST>();
        const int qa = (LA + sh.na - 1) / sh.na, qb = (LB + sh.nb - 1) / sh.nb;
        const int l = lane * 8 + wave;   // dealt over the waves; l >= qa + qb: no line
        const bool a = l < qa;
        const int la = min(sh.a * qa + l, LA - 1), lb = min(sh.b * qb + l - qa, LB - 1);
        touch = a ? (const char*)s.a + TA::template touch_offset<NST>(s.lda, m0, s.m, la) : (const char*)s.b + TB::template touch_offset<NST>(s.ldb, n0, s.n, max(lb, 0));
        touch_step = a ? TA::step_bytes(s.lda) : TB::step_bytes(s.ldb);
        static_assert(TOUCH_MAX <= NT, "one line per lane");
        if (qa + qb <= TOUCH_MAX) touch_lanes = __ballot(l < qa + qb);
    };
    auto touch_ahead = [&](int t) {   // the lines of stages t .. t + NST - 1
        touch_untracked(touch + (uint64_t)touch_step * (uint32_t)min(t, steps - NST), touch_lanes, smem + NST * STAGE);
    };
    bf16x8 fa[2][FM], fb[2][FN];
    // does this lane's chunk of a step lie in the next stage?  (misalignments repeat every 16 rows)
    const bool nexta = LA_ && 4 * half + (lane >> 4) + TA::misalignment(s.a, s.lda, m0 + (lane & 15)) >= 8;
    const bool nextb = LB_ && 4 * half + (lane >> 4) + TB::misalignment(s.b, s.ldb, n0 + (lane & 15)) >= 8;
    // what that makes of the lane offsets, for each stage that a step may start in (kept: worked out in every step they cost 60 ns)
    int oa[NST], ob[NST];
#pragma unroll
    for (int i = 0; i < NST; ++i) {
        oa[i] = loa + (nexta ? (i + 1) % NST : i) * STAGE;
        ob[i] = lob + (nextb ? (i + 1) % NST : i) * STAGE;
        if constexpr (LA_) asm("" : "+v"(oa[i]));
        if constexpr (LB_) asm("" : "+v"(ob[i]));
    }
    auto read_at = [&](int la, int lb, int set) {
#pragma unroll
        for (int j = 0; j < FN; ++j) fb[set][j] = TB::frag16(smem + TA::BYTES, lb, j);
#pragma unroll
        for (int i = 0; i < FM; ++i) fa[set][i] = TA::frag16(smem, la, i);
    };
    auto mfmas = [&](int set) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[set][j], fa[set][i], acc[i][j], 0, 0, 0);
    };
    // Step t's fragments were read in the step before.  What step t + 1 reads (stage t + 1, with whole lines t + 2 as well) has
    // landed for this wave, and this wave's reads have returned, before the barrier; behind it that holds for all waves: stage t
    // is free for t + NST, and the next fragments may be read, all through the multiplication.
    int t = 0;
    auto wait_keep = [](auto n) { __builtin_amdgcn_s_waitcnt((vmcnt_only(decltype(n)::value) & ~0x0F00)); };   // vmcnt(n) lgkmcnt(0)
    auto step = [&](auto cur, auto kind) {
        constexpr int CUR = decltype(cur)::value;
        // stages t + 2, t + 3 (with whole lines only t + 3) and the touch behind the one waited for stay in flight
        if constexpr (LINES) wait_keep(std::integral_constant<int, (NST - 3) * NVM + (TOUCH && (CUR == 1 || CUR == 2))>{});
        else wait_keep(std::integral_constant<int, (NST - 2) * NVM + (TOUCH && CUR != 0)>{});
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        issue(smem + CUR * STAGE, kind);
        if constexpr (TOUCH && CUR == 0) touch_ahead(t + TOUCH_DIST);
        read_at(oa[(CUR + 1) % NST], ob[(CUR + 1) % NST], (CUR + 1) & 1);
        mfmas(CUR & 1);
        constexpr int NDS = (A_KC ? FM : 2 * FM) + (B_KC ? FN : 2 * FN), NM = FM * FN - 4;
        static_for<NM>([&](auto i) {   // fragment reads spread over all but the last matrix instructions
            constexpr int I = decltype(i)::value, nds = NDS * (I + 1) / NM - NDS * I / NM;
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if constexpr (nds > 0) __builtin_amdgcn_sched_group_barrier(0x100, nds, 0);
        });
        __builtin_amdgcn_sched_group_barrier(0x008, FM * FN - NM, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    if (steps > 0) {
        using Inner = std::integral_constant<Issue, INNER>;
        using Any = std::integral_constant<Issue, ANY>;
        issue(smem, std::integral_constant<Issue, FIRST>{});
        static_for<NST - 1>([&](auto i) { issue(smem + (decltype(i)::value + 1) * STAGE, Any{}); });
        if constexpr (TOUCH) if (steps >= DEEP_TOUCH_STEPS) share_touches();
        wait_keep(std::integral_constant<int, (NST - (LINES ? 2 : 1)) * NVM>{});
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        read_at(oa[0], ob[0], 0);
        for (; t + 2 * NST < steps; t += NST) static_for<NST>([&](auto i) { step(i, Inner{}); });
        for (; t + NST <= steps; t += NST) static_for<NST>([&](auto i) { step(i, Any{}); });
        const int rem = steps - t;
        static_for<NST - 1>([&](auto i) {
            if (decltype(i)::value < rem) step(i, Any{});
        });
        __builtin_amdgcn_s_waitcnt(0x0070);   // the unread trailing loads have landed before their stages are reused
    }
    __syncthreads();
    if (const int k0 = steps * BKT; k0 < s.kk) {   // the last 1 .. 63 elements, zeros behind them
#pragma unroll
        for (int it = 0; it < TA::PER_THREAD; ++it)
            *reinterpret_cast<u32x4*>(smem + (it * NT + tid) * 16) = TA::tail_chunk(static_cast<const uint16_t*>(s.a), s.lda, m0, s.m, s.kk, k0, it * NT + tid);
#pragma unroll
        for (int it = 0; it < TB::PER_THREAD; ++it)
            *reinterpret_cast<u32x4*>(smem + TA::BYTES + (it * NT + tid) * 16) = TB::tail_chunk(static_cast<const uint16_t*>(s.b), s.ldb, n0, s.n, s.kk, k0, it * NT + tid);
        __syncthreads();
        read_at(loa, lob, 0);
        mfmas(0);
        __syncthreads();
    }

    // the partial tiles, blocks as in gemm_wavek_kernel; the two waves of a 64 x 64 part share its sum
    constexpr int EPV = 16 / (int)sizeof(OutT), UNIT = sizeof(OutT) == 4 ? 2 : 4, PART = FM * FN * 1024;
    const int q = lane >> 4, r = lane & 15;
    static_for<FM * FN>([&](auto bix) {
        constexpr int b = decltype(bix)::value;
        *reinterpret_cast<f32x4*>(smem + wave * PART + b * 1024 + (16 * q + (r ^ (4 * q))) * 16) = acc[b / FN][b % FN];
    });
    __syncthreads();
#pragma unroll EPI == EPI_GELU_ERF ? 1 : 64
    for (int u = 0; u < FM * FN / UNIT; ++u) {   // this wave: eight of every 16 rows
        const int blk = u * UNIT, row = 8 * half + (lane >> 3);
        float v[EPV];
#pragma unroll
        for (int h = 0; h < EPV / 4; ++h) {
            const int cg = (lane & 7) * (EPV / 4) + h;
            const char* at = smem + sub * PART + (blk + cg / 4) * 1024 + (16 * (cg & 3) + (row ^ (4 * (cg & 3)))) * 16;
            const f32x4 sum = *reinterpret_cast<const f32x4*>(at) + *reinterpret_cast<const f32x4*>(at + 4 * PART);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * h + e] = mfma_epilogue<EPI>(sum[e]);
        }
        store_columns<OutT>(s, m0 + wm * 64 + blk / FN * 16 + row, n0 + wn * 64 + blk % FN * 16 + (lane & 7) * EPV, v);
    }
}

template <int BM, int BN, int NW, bool DIRECT, bool A_KC, bool B_KC, int EPI, typename OutT>
constexpr auto pick_kernel() {   // NW = 0: gemm_reg_kernel
    if constexpr (NW == 0) return gemm_reg_kernel<BM, BN, A_KC, B_KC, EPI, OutT>;
    else return gemm_wavek_kernel<BM, BN, NW, A_KC, B_KC, DIRECT, EPI, OutT>;
}

template <int BM, int BN, int NW, bool DIRECT, int EPI, typename OutT>
int32_t launch_layout(const GemmPlan& plan, int max_m, int max_n, int order, hipStream_t st) {
    const int tm = tiles_along(max_m, BM), tn = tiles_along(max_n, BN);
    const int64_t nblk = ((int64_t)tm * tn * plan.groups + 7) / 8 * 8;
    if (!grid_fits(nblk, NW > 0 ? NW * 64 : 256)) return SBP_ERR_UNSUPPORTED;
    void (*kern)(GemmPlan, int, int, int) = nullptr;
    if (plan.a_kc) {
        if (plan.b_kc) kern = pick_kernel<BM, BN, NW, DIRECT, true, true, EPI, OutT>();
        else kern = pick_kernel<BM, BN, NW, DIRECT, true, false, EPI, OutT>();
    } else if constexpr (BM >= 64) {
        if (plan.b_kc) kern = pick_kernel<BM, BN, NW, DIRECT, false, true, EPI, OutT>();
        else kern = pick_kernel<BM, BN, NW, DIRECT, false, false, EPI, OutT>();
    }
    if (!kern) return SBP_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(kern, dim3((uint32_t)nblk), dim3(NW > 0 ? NW * 64 : 256), 0, st, plan, tm, tn, order);
    return launch_status(__func__);
}

template <int BM, int BN, int NW, bool DIRECT>
int32_t launch_out(const GemmPlan& plan, int max_m, int max_n, int order, hipStream_t st) {
    if (plan.out_dtype == SBP_F32) {
        if (plan.epilogue != SBP_EPI_NONE) return SBP_ERR_UNSUPPORTED;
        return launch_layout<BM, BN, NW, DIRECT, SBP_EPI_NONE, float>(plan, max_m, max_n, order, st);
    }
    if constexpr (DIRECT)
        if (plan.epilogue == SBP_EPI_GELU) return launch_layout<BM, BN, NW, DIRECT, SBP_EPI_GELU, uint16_t>(plan, max_m, max_n, order, st);
    // rows of any pitch are erfcf's; a forced register kernel on others gets the more accurate form as well
    if (plan.epilogue == EPI_GELU_ERF || plan.epilogue == SBP_EPI_GELU) return launch_layout<BM, BN, NW, DIRECT, EPI_GELU_ERF, uint16_t>(plan, max_m, max_n, order, st);
    if (plan.epilogue != SBP_EPI_NONE) return SBP_ERR_UNSUPPORTED;
    return launch_layout<BM, BN, NW, DIRECT, SBP_EPI_NONE, uint16_t>(plan, max_m, max_n, order, st);
}

template <int BM, int BN>
int32_t launch_rows(const GemmPlan& plan, int max_m, int max_n, int order, hipStream_t st) {
    if (!plan.a_kc || !plan.b_kc || plan.out_dtype != SBP_F32 || plan.epilogue != SBP_EPI_NONE) return SBP_ERR_UNSUPPORTED;
    const int tm = tiles_along(max_m, BM), tn = tiles_along(max_n, BN);
    const int64_t nblk = ((int64_t)tm * tn * plan.groups + 7) / 8 * 8;
    if (!grid_fits(nblk, 512)) return SBP_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((gemm_rows_kernel<BM, BN>), dim3((uint32_t)nblk), dim3(512), 0, st, plan, tm, tn, order);
    return launch_status(__func__);
}

template <int EPI, typename OutT>
int32_t launch_deep_layout(const GemmPlan& plan, int max_m, int max_n, int order, bool touch, hipStream_t st) {
    const int tm = tiles_along(max_m, 128), tn = tiles_along(max_n, 128);
    const int64_t nblk = ((int64_t)tm * tn * plan.groups + 7) / 8 * 8;
    if (!grid_fits(nblk, 512)) return SBP_ERR_UNSUPPORTED;
    const bool lines = !rows_on_lines(plan);
    auto launch = [&](auto a_kc, auto b_kc, auto ln, auto tc) {
        hipLaunchKernelGGL((gemm_deep_kernel<decltype(a_kc)::value, decltype(b_kc)::value, decltype(ln)::value, decltype(tc)::value, EPI, OutT>), dim3((uint32_t)nblk), dim3(512), 0, st, plan, tm, tn, order);
    };
    auto either = [](bool on, auto f) { on ? f(std::true_type{}) : f(std::false_type{}); };
    either(plan.a_kc, [&](auto a) {
        either(plan.b_kc, [&](auto b) {
            either(touch, [&](auto t) {
                if constexpr (decltype(a)::value || decltype(b)::value) either(lines, [&](auto l) { launch(a, b, l, t); });
                else launch(a, b, std::false_type{}, t);
            });
        });
    });
    return launch_status(__func__);
}

}  // namespace

int32_t launch_gemm_deep(const GemmPlan& plan, int max_m, int max_n, int order, bool touch, hipStream_t stream) {
    if (plan.out_dtype == SBP_F32) return plan.epilogue == SBP_EPI_NONE ? launch_deep_layout<SBP_EPI_NONE, float>(plan, max_m, max_n, order, touch, stream) : SBP_ERR_UNSUPPORTED;
    if (plan.epilogue == SBP_EPI_GELU) return launch_deep_layout<SBP_EPI_GELU, uint16_t>(plan, max_m, max_n, order, touch, stream);
    if (plan.epilogue == EPI_GELU_ERF) return launch_deep_layout<EPI_GELU_ERF, uint16_t>(plan, max_m, max_n, order, touch, stream);
    if (plan.epilogue != SBP_EPI_NONE) return SBP_ERR_UNSUPPORTED;
    return launch_deep_layout<SBP_EPI_NONE, uint16_t>(plan, max_m, max_n, order, touch, stream);
}

int32_t launch_gemm_any(const GemmPlan& plan, int max_m, int max_n, int tile, bool direct, int order, hipStream_t stream) {
    switch (tile) {
        case WAVEK_128: return direct ? launch_out<128, 64, 4, true>(plan, max_m, max_n, order, stream) : SBP_ERR_UNSUPPORTED;
        case WAVEK_64: return direct ? launch_out<64, 64, 8, true>(plan, max_m, max_n, order, stream) : launch_out<64, 64, 8, false>(plan, max_m, max_n, order, stream);
        case WAVEK_32: return direct ? launch_out<32, 64, 8, true>(plan, max_m, max_n, order, stream) : launch_out<32, 64, 8, false>(plan, max_m, max_n, order, stream);
        case ROWS_32: return launch_rows<32, 32>(plan, max_m, max_n, order, stream);
        case ROWS_64: return launch_rows<64, 64>(plan, max_m, max_n, order, stream);
        case REG_128: return launch_out<128, 128, 0, false>(plan, max_m, max_n, order, stream);
        case REG_64: return launch_out<64, 64, 0, false>(plan, max_m, max_n, order, stream);
        default: return SBP_ERR_UNSUPPORTED;
    }
}

}  // namespace sbp
