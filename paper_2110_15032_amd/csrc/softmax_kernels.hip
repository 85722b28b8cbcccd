// Local row reductions of the model-parallel softmax (paper Sec. 6.3.1): each device reduces the
// columns of the logits it holds, first to a row max (P(max)), then -- once the max has been boxed
// to B -- to a row sum of exp(l - max) (P(sum)).  One workgroup per (row, shard); 16-byte loads
// where the row pitch allows, wavefront shuffles then one LDS hop across the four waves.
#include <type_traits>

#include "sbp_internal.h"

namespace sbp {
namespace {

constexpr int RS_THREADS = 256;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ inline float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// SUMEXP: m is passed as -max * log2(e), so that exp(v - max) is one FMA and one hardware exp2
// (relative error about |v - max| * 1e-7: the argument is at most 0 and a term below 2^-126 adds
// nothing to a sum that contains exp(0) = 1 somewhere on the row's devices)
constexpr float LOG2E = 1.4426950408889634f;
template <bool SUMEXP>
__device__ inline float fold(float acc, float v, float m) {
    if constexpr (SUMEXP) return acc + __builtin_amdgcn_exp2f(fmaf(v, LOG2E, m));
    else return fmaxf(acc, v);
}

template <bool SUMEXP>
__device__ inline float wave_reduce(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const float o = __shfl_xor(v, off, 64);
        v = SUMEXP ? v + o : fmaxf(v, o);
    }
    return v;
}

// Bound by HBM.  Four vectors a lane are in flight, in cached rows of 256 threads one (8 x 153 of 32237: one 14.2, four 15.0).
// THREADS: 1024 for few long rows, which leave compute units idle.  STREAM:
// non-temporal loads, for logits that the memory-side cache does not hold until the next pass anyway.  us, one vector a lane, 256
// threads, cached / now: 8 devices x 1024 rows of 125000 bf16 logits (2 GB) 338 / 294 (7.0 TB/s; cached 334), 3 x 19 of 114091 14.1 / 7.4
// (256 threads 8.8), 2 x 8 of 250000 26.9 / 11.5 (15.2); cached / streaming 4 x 200 of 7503 5.0 / 6.8, 5 x 100 of 17000 5.0 / 7.8.
template <bool SUMEXP, bool BF16, int THREADS, bool STREAM>
__global__ __launch_bounds__(THREADS) void row_stat_kernel(RowStatPlan p) {
    const int shard = blockIdx.y;
    const int64_t row = blockIdx.x;
    const int32_t cols = p.cols[shard];
    const float ident = SUMEXP ? 0.0f : -INFINITY;
    const float m = SUMEXP ? -p.gmax[shard][row] * LOG2E : 0.0f;
    float acc = ident;
    if (cols > 0) {
        constexpr int EPV = BF16 ? 8 : 4;  // elements per 16-byte vector
        const char* base = static_cast<const char*>(p.logits[shard]) + (int64_t)row * p.ld[shard] * (BF16 ? 2 : 4);
        // rows start 16-byte aligned only when the pitch is a multiple of EPV; otherwise peel
        const int32_t mis = (int32_t)((reinterpret_cast<uintptr_t>(base) & 15u) / (BF16 ? 2 : 4));
        int32_t head = mis ? EPV - mis : 0;
        if (head > cols) head = cols;
        const int32_t nvec = (cols - head) / EPV;
        const int32_t tail0 = head + nvec * EPV;
        auto elem = [&](int32_t c) -> float {
            if constexpr (BF16) return __uint_as_float((uint32_t) reinterpret_cast<const uint16_t*>(base)[c] << 16);
            else return reinterpret_cast<const float*>(base)[c];
        };
        for (int32_t c = threadIdx.x; c < head; c += THREADS) acc = fold<SUMEXP>(acc, elem(c), m);
        for (int32_t c = tail0 + threadIdx.x; c < cols; c += THREADS) acc = fold<SUMEXP>(acc, elem(c), m);
        const char* vbase = base + (int64_t)head * (BF16 ? 2 : 4);
        float a0 = ident, a1 = ident, a2 = ident, a3 = ident;   // four chains per lane
        using Vec = std::conditional_t<BF16, u32x4, f32x4>;
        const Vec* const vec = reinterpret_cast<const Vec*>(vbase);
        auto take = [&](const Vec w) {
            if constexpr (BF16) {
                a0 = fold<SUMEXP>(fold<SUMEXP>(a0, bf16_lo(w.x), m), bf16_hi(w.x), m);
                a1 = fold<SUMEXP>(fold<SUMEXP>(a1, bf16_lo(w.y), m), bf16_hi(w.y), m);
                a2 = fold<SUMEXP>(fold<SUMEXP>(a2, bf16_lo(w.z), m), bf16_hi(w.z), m);
                a3 = fold<SUMEXP>(fold<SUMEXP>(a3, bf16_lo(w.w), m), bf16_hi(w.w), m);
            } else {
                a0 = fold<SUMEXP>(a0, w.x, m);
                a1 = fold<SUMEXP>(a1, w.y, m);
                a2 = fold<SUMEXP>(a2, w.z, m);
                a3 = fold<SUMEXP>(a3, w.w, m);
            }
        };
        int32_t v = threadIdx.x;
        constexpr int DEPTH = THREADS > RS_THREADS || STREAM ? 4 : 1;
        for (; v + (int64_t)(DEPTH - 1) * THREADS < nvec; v += DEPTH * THREADS) {
            Vec w[DEPTH];
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                if constexpr (STREAM) w[d] = __builtin_nontemporal_load(vec + v + d * THREADS);
                else w[d] = vec[v + d * THREADS];
            }
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) take(w[d]);
        }
        if (DEPTH > 1 && v < nvec) {   // up to DEPTH more, loaded together (the last one again where there are fewer)
            Vec w[DEPTH];
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) w[d] = vec[(int32_t)min(v + (int64_t)d * THREADS, (int64_t)nvec - 1)];
#pragma unroll
            for (int d = 0; d < DEPTH; ++d)
                if (v + (int64_t)d * THREADS < nvec) take(w[d]);
        }
        if constexpr (SUMEXP) acc += (a0 + a1) + (a2 + a3);
        else acc = fmaxf(fmaxf(acc, fmaxf(a0, a1)), fmaxf(a2, a3));
    }
    acc = wave_reduce<SUMEXP>(acc);
    __shared__ float part[THREADS / 64];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        float r = part[0];
#pragma unroll
        for (int w = 1; w < THREADS / 64; ++w) r = SUMEXP ? r + part[w] : fmaxf(r, part[w]);
        p.out[shard][row] = r;
    }
}

// ------------------------------------------------------------------------------------------------
// Sparse cross entropy on the same S(1) logits (Sec. 6.3.1): with the global row max m and
// denominator s in hand (B), the loss needs one logit per row, held by exactly one device, so every
// device writes a partial vector (P(sum)); the gradient is elementwise on every shard.
// ------------------------------------------------------------------------------------------------
template <bool BF16>
__global__ __launch_bounds__(RS_THREADS) void xent_loss_kernel(XentPlan p) {
    const int i = blockIdx.y;
    const int64_t r = (int64_t)blockIdx.x * RS_THREADS + threadIdx.x;
    if (r >= p.rows) return;
    const int32_t c = p.labels[i][r] - p.begin[i];
    float out = 0.0f;
    if (c >= 0 && c < p.cols[i]) {
        const int64_t pos = r * p.ld[i] + c;
        float l;
        if constexpr (BF16) l = __uint_as_float((uint32_t) static_cast<const uint16_t*>(p.logits[i])[pos] << 16);
        else l = static_cast<const float*>(p.logits[i])[pos];
        out = logf(p.denom[i][r]) + p.gmax[i][r] - l;
    }
    static_cast<float*>(p.out[i])[r] = out;
}

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ inline uint32_t pack_bf16(float lo, float hi) {
    const f32x2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

typedef u32x4 __attribute__((aligned(2))) u32x4_any;
typedef f32x4 __attribute__((aligned(4))) f32x4_any;
// how the rows of the logits and of their gradient lie
enum RowLayout {
    ROWS_WHOLE,     // every row starts 16-byte aligned and is whole vectors
    ROWS_ALIGNED,   // every row starts 16-byte aligned
    ROWS_ANY
};
// Streaming load and the store of 16 bytes: past the caches where rows are aligned.  (The unaligned types are named here, since a
// template argument drops the attribute.)
template <RowLayout L>
__device__ inline u32x4 load16(const uint16_t* at) {
    if constexpr (L == ROWS_WHOLE) return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(at));
    else return __builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(at));
}
template <RowLayout L>
__device__ inline f32x4 load16(const float* at) {
    if constexpr (L == ROWS_WHOLE) return __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(at));
    else return __builtin_nontemporal_load(reinterpret_cast<const f32x4_any*>(at));
}
template <RowLayout L>
__device__ inline void store16(uint16_t* at, u32x4 v) {
    if constexpr (L == ROWS_WHOLE) __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(at));
    else if constexpr (L == ROWS_ALIGNED) __builtin_nontemporal_store(v, reinterpret_cast<u32x4_any*>(at));
    else *reinterpret_cast<u32x4_any*>(at) = v;
}
template <RowLayout L>
__device__ inline void store16(float* at, f32x4 v) {
    if constexpr (L == ROWS_WHOLE) __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(at));
    else if constexpr (L == ROWS_ALIGNED) __builtin_nontemporal_store(v, reinterpret_cast<f32x4_any*>(at));
    else *reinterpret_cast<f32x4_any*>(at) = v;
}
// VE elements per lane, 16 bytes or one (see launch_xent_grad).  Vectors of rows that are not whole ones are read and written
// unaligned, which costs a second cache line per wave and instruction; the last vector of a row ends with it, and two lanes may
// store the same values; no row is shorter than a vector.  Where rows are not aligned neighbouring waves share a line, which L2
// has to keep for both: the result is stored past the caches otherwise.
template <bool BF16, int VE, RowLayout L>
__global__ __launch_bounds__(RS_THREADS) void xent_grad_kernel(XentPlan p) {
    using Elem = std::conditional_t<BF16, uint16_t, float>;
    const int i = blockIdx.y;
    const uint32_t cols = (uint32_t)p.cols[i], cols_v = (cols + VE - 1) / VE;
    if (cols_v == 0) return;
    // (row, vector) of this lane's first item by one division, then advanced by the grid stride with adds only:
    // a 64-bit division per item costs more vector instructions than the item's arithmetic and made the kernel
    // instruction-bound instead of memory-bound
    const uint64_t stride = (uint64_t)gridDim.x * RS_THREADS;
    const uint32_t dr = (uint32_t)(stride / cols_v), dc = (uint32_t)(stride % cols_v);
    const uint64_t first = (uint64_t)blockIdx.x * RS_THREADS + threadIdx.x;
    uint64_t r64 = first / cols_v;
    uint32_t cv = (uint32_t)(first % cols_v);
    for (; r64 < (uint64_t)p.rows; r64 += dr, cv += dc) {
        if (cv >= cols_v) {
            cv -= cols_v;
            if (++r64 >= (uint64_t)p.rows) break;
        }
        const uint32_t r = (uint32_t)r64;
        uint32_t c = cv * VE;
        if constexpr (L != ROWS_WHOLE && VE > 1) c = c + VE <= cols ? c : cols - VE;
        const int32_t y = p.labels[i][r];
        const bool live = y >= 0 && y < p.total_cols;
        const float g = live ? p.grad[i][r] : 0.0f;
        const float m = p.gmax[i][r], inv = 1.0f / p.denom[i][r];
        const int32_t yc = y - p.begin[i] - (int32_t)c;   // position of the label inside this group, if any
        const Elem* src = static_cast<const Elem*>(p.logits[i]) + (int64_t)r * p.ld[i] + c;
        Elem* dst = static_cast<Elem*>(p.out[i]) + (int64_t)r * p.ld_out[i] + c;
        auto value = [&](float v, int e) { return (__expf(v - m) * inv - (e == yc ? 1.0f : 0.0f)) * g; };
        if constexpr (VE > 1) {
            // streaming load: the gradient pass is the last reader of the logits (measured 2 % faster than a cached load;
            // two items per lane and round, both loaded before either is worked on, 1 % slower than this)
            const auto w = load16<L>(src);
            std::conditional_t<BF16, u32x4, f32x4> o;
            if constexpr (BF16) {
#pragma unroll
                for (int d = 0; d < 4; ++d) o[d] = pack_bf16(value(bf16_lo(w[d]), 2 * d), value(bf16_hi(w[d]), 2 * d + 1));
            } else {
#pragma unroll
                for (int e = 0; e < VE; ++e) o[e] = value(w[e], e);
            }
            store16<L>(dst, o);
        } else if constexpr (BF16) {
            *dst = (uint16_t)(pack_bf16(value(__uint_as_float((uint32_t)*src << 16), 0), 0.0f) & 0xFFFFu);
        } else {
            *dst = value(*src, 0);
        }
    }
}

}  // namespace

int32_t launch_xent_loss(const XentPlan& plan, hipStream_t stream) {
    if (plan.rows == 0) return SBP_OK;
    const int64_t bx = (plan.rows + RS_THREADS - 1) / RS_THREADS;
    if (bx > 0x7FFFFFFF) return SBP_ERR_UNSUPPORTED;
    const dim3 grid((uint32_t)bx, (uint32_t)plan.k);
    if (plan.dtype == SBP_BF16) hipLaunchKernelGGL(xent_loss_kernel<true>, grid, dim3(RS_THREADS), 0, stream, plan);
    else hipLaunchKernelGGL(xent_loss_kernel<false>, grid, dim3(RS_THREADS), 0, stream, plan);
    return launch_status(__func__);
}

int32_t launch_xent_grad(const XentPlan& plan, hipStream_t stream) {
    if (plan.rows == 0 || plan.total_cols == 0) return SBP_OK;
    const bool bf = plan.dtype == SBP_BF16;
    const int epv = bf ? 8 : 4;
    bool aligned = true, whole = true;
    int32_t narrowest = INT32_MAX;
    int64_t widest = 0;
    for (int i = 0; i < plan.k; ++i) {
        if (plan.cols[i] == 0) continue;
        if (plan.ld[i] % epv || plan.ld_out[i] % epv) aligned = false;
        if (plan.cols[i] % epv) whole = false;
        narrowest = plan.cols[i] < narrowest ? plan.cols[i] : narrowest;
        widest = plan.cols[i] > widest ? plan.cols[i] : widest;
    }
    // Vectors where rows hold one and there is enough to do, else one element per lane.  us, element / vectors, columns a device:
    // bf16, 3 devices: 65536 rows of 9 7.6 / 5.1, of 31 20.1 / 10.6; 512 rows of 31 3.6 / 4.0; fp32: 65536 rows of 5 6.0 / 5.3.
    // Vectors known to be whole and aligned: 1024 x 1000000 bf16, 8 devices, 685 against 742.
    whole = whole && aligned;
    const bool vec = whole || (narrowest >= epv && plan.rows * plan.total_cols >= (1 << 19));
    const int64_t max_units = (vec ? (widest + epv - 1) / epv : widest) * plan.rows;
    int64_t bx = (max_units + RS_THREADS - 1) / RS_THREADS;
    // at most 65536 workgroups, grid-stride beyond (2 GB of bf16 logits: 0.68 ms; with one vector per lane and
    // half a million short-lived workgroups 0.74 ms, with 16384 workgroups 0.73 ms)
    const int64_t cap = (1 << 16) / plan.k;
    if (bx > cap) bx = cap;
    if (bx < 1) bx = 1;
    const dim3 grid((uint32_t)bx, (uint32_t)plan.k);
    void (*kern)(XentPlan);
    if (bf) kern = whole ? xent_grad_kernel<true, 8, ROWS_WHOLE> : !vec ? xent_grad_kernel<true, 1, ROWS_ANY> : aligned ? xent_grad_kernel<true, 8, ROWS_ALIGNED> : xent_grad_kernel<true, 8, ROWS_ANY>;
    else kern = whole ? xent_grad_kernel<false, 4, ROWS_WHOLE> : !vec ? xent_grad_kernel<false, 1, ROWS_ANY> : aligned ? xent_grad_kernel<false, 4, ROWS_ALIGNED> : xent_grad_kernel<false, 4, ROWS_ANY>;
    hipLaunchKernelGGL(kern, grid, dim3(RS_THREADS), 0, stream, plan);
    return launch_status(__func__);
}

int32_t launch_row_stat(const RowStatPlan& plan, bool sumexp, hipStream_t stream_) {
    if (plan.rows == 0) return SBP_OK;
    if (plan.rows > 0x7FFFFFFF) return SBP_ERR_UNSUPPORTED;
    const dim3 grid((uint32_t)plan.rows, (uint32_t)plan.k);
    const bool bf = plan.dtype == SBP_BF16;
    int32_t cols = 0;
    int64_t total = 0;
    for (int i = 0; i < plan.k; ++i) {
        cols = plan.cols[i] > cols ? plan.cols[i] : cols;
        total += plan.rows * plan.cols[i] * (bf ? 2 : 4);
    }
    const bool wide = plan.rows * plan.k <= 2 * compute_units() && cols >= 16384;      // two rows a compute unit; 2 KB of bf16 and more for each wave
    const bool stream = !wide && total > (int64_t)256 << 20;           // the memory-side cache's size
    auto pick = [&](auto s, auto b) -> void (*)(RowStatPlan) {
        constexpr bool S = decltype(s)::value, BF = decltype(b)::value;
        return wide ? row_stat_kernel<S, BF, 1024, false> : stream ? row_stat_kernel<S, BF, RS_THREADS, true> : row_stat_kernel<S, BF, RS_THREADS, false>;
    };
    void (*kern)(RowStatPlan) = sumexp ? (bf ? pick(std::true_type{}, std::true_type{}) : pick(std::true_type{}, std::false_type{}))
                                       : (bf ? pick(std::false_type{}, std::true_type{}) : pick(std::false_type{}, std::false_type{}));
    hipLaunchKernelGGL(kern, grid, dim3(wide ? 1024 : RS_THREADS), 0, stream_, plan);
    return launch_status(__func__);
}

}  // namespace sbp
