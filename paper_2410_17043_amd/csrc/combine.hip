// Aggregation of Sec. 2.1: y[t] = sum_j w[t,j] * ret[slot_to_row[t*k+j]] (+ shared_out[t]).
//
// `ret` is in send-buffer row order (the second all-to-all is the reverse of the
// first with the same sizes, Sec. 2.2).  One wave per token: the k source rows are
// gathered with 16-byte lanes (1 KB per wave access), accumulated in fp32 in slot
// order j = 0..k-1 and rounded once on the way out.  Every input row is read exactly
// once (plain loads while the rows fit the memory-side cache, streaming loads beyond,
// see kCombineCacheableBytes); the output goes out with streaming stores.
#include "common.h"

namespace {

template <int DT> struct Pack;
template <> struct Pack<MOE_BF16> {
    static constexpr int V = 8;
    __device__ static void unpack(const u32x4& q, float (&f)[8]) {
        const uint32_t u[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = __uint_as_float(u[i] << 16);
            f[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u);
        }
    }
    __device__ static u32x4 pack(const float (&f)[8]) {
        uint32_t u[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) u[i] = f32_to_bf16_bits(f[2 * i]) | (f32_to_bf16_bits(f[2 * i + 1]) << 16);
        return u32x4{u[0], u[1], u[2], u[3]};
    }
};
template <> struct Pack<MOE_F32> {
    static constexpr int V = 4;
    __device__ static void unpack(const u32x4& q, float (&f)[4]) {
        f[0] = __uint_as_float(q.x); f[1] = __uint_as_float(q.y); f[2] = __uint_as_float(q.z); f[3] = __uint_as_float(q.w);
    }
    __device__ static u32x4 pack(const float (&f)[4]) {
        return u32x4{__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3])};
    }
};

template <int DT, int K, bool STREAM>
__global__ __launch_bounds__(256) void combine_kernel(const u32x4* __restrict__ ret, const int32_t* __restrict__ slot_to_row,
                                                      const float* __restrict__ topk_w, const u32x4* __restrict__ shared_out,
                                                      int T, int row16, u32x4* __restrict__ y) {
    constexpr int V = Pack<DT>::V;
    constexpr int KM = K;
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= T) return;
    int rows[KM];
    float w[KM];
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        rows[j] = slot_to_row[(size_t)t * K + j];
        w[j] = topk_w[(size_t)t * K + j];
    }
    // CPT 16-byte chunks per lane per trip, about eight independent row loads in flight before the first use
    constexpr int CPT = (K < 4) ? 8 / K : 2;
    for (int c0 = lane; c0 < row16; c0 += 64 * CPT) {
        u32x4 q[CPT][KM];
#pragma unroll
        for (int u = 0; u < CPT; ++u) {
            const int c = c0 + 64 * u;
#pragma unroll
            for (int j = 0; j < KM; ++j)
                if (c < row16 && rows[j] >= 0) {
                    const u32x4* p = ret + (size_t)rows[j] * row16 + c;
                    q[u][j] = STREAM ? __builtin_nontemporal_load(p) : *p;
                }
        }
#pragma unroll
        for (int u = 0; u < CPT; ++u) {
            const int c = c0 + 64 * u;
            if (c >= row16) continue;
            float acc[V];
#pragma unroll
            for (int v = 0; v < V; ++v) acc[v] = 0.f;
#pragma unroll
            for (int j = 0; j < KM; ++j) {
                if (rows[j] >= 0) {
                    float f[V];
                    Pack<DT>::unpack(q[u][j], f);
#pragma unroll
                    for (int v = 0; v < V; ++v) acc[v] = fmaf(w[j], f[v], acc[v]);
                }
            }
            if (shared_out) {
                float f[V];
                Pack<DT>::unpack(shared_out[(size_t)t * row16 + c], f);
#pragma unroll
                for (int v = 0; v < V; ++v) acc[v] += f[v];
            }
            __builtin_nontemporal_store(Pack<DT>::pack(acc), y + (size_t)t * row16 + c);
        }
    }
}

// One token and 1 KB of its rows per wave, all source rows of K slots in flight at a time (K = 0: any k, four at a time).  For any
// k, and for the k of the kernel above where its one wave per token leaves the chip to a few waves that walk through their
// rows (see kFewTokens).  The loads
// are issued unconditionally (a slot past k or a dropped one reads a valid row whose value is not used): with the loads of
// a 16-slot array under conditions the compiler kept the whole array in registers (217 of them) and waited
// for each load in turn.  For K = 0 each row goes out as soon as its number is known, and the shared expert's at the end: all numbers
// first and the shared row in front, as for K > 0, was 0.1 to 0.8 us slower in bf16 (64 tokens, k = 16, H = 4096 from cold memory 4.7 -> 5.5).
template <int DT, int K, bool STREAM>
__global__ __launch_bounds__(256) void combine_pieces_kernel(const u32x4* __restrict__ ret, const int32_t* __restrict__ slot_to_row,
                                                             const float* __restrict__ topk_w, const u32x4* __restrict__ shared_out,
                                                             int T, int any_k, int row16, u32x4* __restrict__ y) {
    constexpr int V = Pack<DT>::V, J = K > 0 ? K : 4;
    const int k = K > 0 ? K : any_k;
    const int lane = threadIdx.x & 63;
    const int t = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (t >= T) return;
    const int c0 = blockIdx.y * 64;
    const int c = min(c0 + lane, row16 - 1);
    float acc[V];
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] = 0.f;
    u32x4 sh = {0, 0, 0, 0};
    if (K > 0 && shared_out) sh = shared_out[(size_t)t * row16 + c];
    auto load = [&](int row) {
        const u32x4* p = ret + (size_t)max(row, 0) * row16 + c;
        return STREAM ? __builtin_nontemporal_load(p) : *p;
    };
    for (int j0 = 0; j0 < k; j0 += J) {
        int rows[J];
        float w[J];
        u32x4 d[J];
#pragma unroll
        for (int i = 0; i < J; ++i) {
            const int j = min(j0 + i, k - 1);
            rows[i] = (j0 + i < k) ? slot_to_row[(size_t)t * k + j] : -1;
            w[i] = topk_w[(size_t)t * k + j];
            if constexpr (K == 0) d[i] = load(rows[i]);
        }
        if constexpr (K > 0)
#pragma unroll
            for (int i = 0; i < J; ++i) d[i] = load(rows[i]);
#pragma unroll
        for (int i = 0; i < J; ++i) {
            if (rows[i] >= 0) {
                float f[V];
                Pack<DT>::unpack(d[i], f);
#pragma unroll
                for (int v = 0; v < V; ++v) acc[v] = fmaf(w[i], f[v], acc[v]);
            }
        }
    }
    if (shared_out) {
        float f[V];
        Pack<DT>::unpack(K > 0 ? sh : shared_out[(size_t)t * row16 + c], f);
#pragma unroll
        for (int v = 0; v < V; ++v) acc[v] += f[v];
    }
    if (c0 + lane < row16) __builtin_nontemporal_store(Pack<DT>::pack(acc), y + (size_t)t * row16 + c0 + lane);
}

// Rows that were just written by the return transfer are still in the memory-side cache (256 MB) when they
// are not too many: plain loads then (17 against 19 us at the Mixtral-shape share, 67 MB); beyond half of that
// cache plain loads only evict each other (103 against 86 us at 403 MB) and streaming loads are used.
constexpr size_t kCombineCacheableBytes = (size_t)128 << 20;

// A wave per token and piece of its rows up to this many tokens, or bytes read and written: the walk of one wave through its
// rows is then what takes the time (us, bf16, H = 4096: 16 tokens, k = 2 4.9 -> 2.2; 64, k = 6 7.7 -> 2.5; 1024, k = 2 7.6 ->
// 5.2; H = 1024, k = 1, 4096 tokens 4.1 -> 3.8).  Beyond, the memory system prefers waves that keep reading and writing (8192
// tokens, k = 2, H = 4096: 39 against 44).  Rows of more than 96 KB are many pieces: up to half as many tokens (fp32, 1024
// tokens, rows from cold memory: H = 24576, k = 1, 2 and 6 1.06, 1.04 and 1.03 times faster, H = 32768 0.97, 0.96 and 0.97; 512 tokens of those 1.16,
// 1.16 and 1.10; bf16 up to 64 KB 1.08 to 5.0).
constexpr int kFewTokens = 1024;
constexpr size_t kFewBytes = (size_t)16 << 20;
constexpr int kLongRow16 = 96 * 1024 / 16;
bool few_tokens(int T, int k, int row16) {
    return T <= (row16 > kLongRow16 ? kFewTokens / 2 : kFewTokens) || (size_t)T * (k + 1) * row16 * 16 <= kFewBytes;
}

template <int DT, bool STREAM>
int launch_combine(const moe_ctx* c, const void* ret, const int32_t* s2r, const float* w, const void* shared, void* y,
                   hipStream_t st) {
    const moe_shape& s = c->s;
    const int row16 = (int)((int64_t)s.H * elem_size(s.dtype) / 16);
    const dim3 grid((s.T + 3) / 4);
    const u32x4* r = reinterpret_cast<const u32x4*>(ret);
    const u32x4* sh = reinterpret_cast<const u32x4*>(shared);
    u32x4* yo = reinterpret_cast<u32x4*>(y);
    const dim3 pieces((s.T + 3) / 4, (row16 + 63) / 64);
    const bool few = few_tokens(s.T, s.k, row16);
#define MOE_COMBINE(K)                                                                                                              \
    if (few) hipLaunchKernelGGL((combine_pieces_kernel<DT, K, STREAM>), pieces, dim3(256), 0, st, r, s2r, w, sh, s.T, s.k, row16, yo); \
    else hipLaunchKernelGGL((combine_kernel<DT, K, STREAM>), grid, dim3(256), 0, st, r, s2r, w, sh, s.T, row16, yo)
    if (s.k == 1) { MOE_COMBINE(1); }
    else if (s.k == 2) { MOE_COMBINE(2); }
    else if (s.k == 6) { MOE_COMBINE(6); }
    else hipLaunchKernelGGL((combine_pieces_kernel<DT, 0, STREAM>), pieces, dim3(256), 0, st, r, s2r, w, sh, s.T, s.k, row16, yo);
#undef MOE_COMBINE
    MOE_LAUNCH_CHECK("combine_kernel");
    return MOE_OK;
}

template <int DT>
int launch_combine_dt(const moe_ctx* c, const void* ret, const int32_t* s2r, const float* w, const void* shared, void* y,
                      hipStream_t st) {
    const moe_shape& s = c->s;
    const size_t bytes = (size_t)s.T * s.k * s.H * elem_size(s.dtype);
    if (bytes > kCombineCacheableBytes) return launch_combine<DT, true>(c, ret, s2r, w, shared, y, st);
    return launch_combine<DT, false>(c, ret, s2r, w, shared, y, st);
}

}  // namespace

extern "C" int moe_selfcheck_combine_pieces(int32_t T, int32_t k, int32_t row16) {
    if (T < 1 || k < 1 || k > MOE_MAX_K || row16 < 1) return moe_set_error(MOE_EINVAL, "moe_selfcheck_combine_pieces: bad argument");
    return (k != 1 && k != 2 && k != 6) || few_tokens(T, k, row16) ? 1 : 0;
}

extern "C" int moe_combine(moe_ctx* ctx, const void* ret, const int32_t* slot_to_row, const float* topk_w,
                           const void* shared_out, void* y, void* stream) {
    if (!ctx || !ret || !slot_to_row || !topk_w || !y) return moe_set_error(MOE_EINVAL, "moe_combine: NULL argument");
    if (!aligned16(ret) || !aligned16(y) || !aligned16(shared_out))
        return moe_set_error(MOE_EALIGN, "moe_combine: ret, y and shared_out must be 16-byte aligned");
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (ctx->s.dtype == MOE_BF16) return launch_combine_dt<MOE_BF16>(ctx, ret, slot_to_row, topk_w, shared_out, y, st);
    return launch_combine_dt<MOE_F32>(ctx, ret, slot_to_row, topk_w, shared_out, y, st);
}
