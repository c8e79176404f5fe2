// Grouped per-adapter AdamW on the LoRA matrices (fp32 state, decoupled weight decay).
//
// The paper keeps one optimizer instance per LoRA job (Sec. 5.2) and trains with AdamW, weight decay
// 0.01, constant learning rate (App., training details).  Here up to kBatch adapters are updated by one launch whose
// arguments carry their pointers and hyper-parameters (no table to upload first, nothing for the next call to overwrite).
// The update is a pure stream (28 bytes per bf16 parameter), so it is bound by HBM bandwidth: a work group takes a run of
// kRun consecutive elements of one matrix - every group the same work, whatever the ranks - and a thread has the
// 16-byte pieces of gradient, master, m and v of its four groups of four elements in flight together.  The seven updates of an 8B
// block with 19.7 M bf16 parameters: 156 us with a table upload per launch and the grid sized by the largest rank, 121 now (4.5 TB/s; a
// device copy reaches 5.0).
// The state, 24 of the 28 bytes, goes past the caches (non-temporal): nobody reads it before the next step, and what it pushed out of the Infinity
// Cache were the frozen weights and activations that the next kernels read: the steps of a block of 79 to 3000 tokens take 1 to 5 % less (360 tokens, rank 64:
// 1222 -> 1164 us).  Not where all of a step has room in the 256 MB of that cache, which a plan can only know of a layer that is by itself: state, operands,
// gradients, weight and activations below that, and no other plan over its tables.  us, one layer's step, cached / past, state (all of it): 50 MB (134)
// 120.2 / 124.0 and 114.9 / 118.7, 101 MB (235) 213.8 / 217.4; 113 MB (343) 330 / 324, 142 MB (381) 368 / 349, 201 MB (368) 296 / 290, 453 MB (840) 1062 /
// 1034.  (The update by itself, over and over, is faster cached up to 226 MB, 74.8 / 84.1; no training does that.)
#include <cmath>
#include <cstring>

#include "common.h"

namespace mlora {

struct AdamwEntry {
    void* A; void* B;
    const void* dA; const void* dB;
    float* sA; float* sB;
    float lr, beta1, beta2, eps, wd;
    float c1, c2;          // 1 / (1 - beta1^t), 1 / (1 - beta2^t)
    int32_t rank;
    int32_t endA, endB;    // work groups up to the end of this adapter's A / B
};

constexpr int kBatch = 32;
constexpr int kRun = 4096;                  // elements per work group: 256 threads x 4 groups x 4 elements
struct AdamwBatch {
    AdamwEntry e[kBatch];
};
static_assert(sizeof(AdamwBatch) + 64 <= 4096, "the batch travels in the kernel arguments");

template <typename T> __device__ inline float ldp(const T* p);
template <> __device__ inline float ldp<float>(const float* p) { return *p; }
template <> __device__ inline float ldp<uint16_t>(const uint16_t* p) { return __uint_as_float(((uint32_t)*p) << 16); }
template <typename T> __device__ inline void stp(T* p, float v);
template <> __device__ inline void stp<float>(float* p, float v) { *p = v; }
template <> __device__ inline void stp<uint16_t>(uint16_t* p, float v) {
    uint32_t u = __float_as_uint(v);
    if ((u & 0x7fffffffu) > 0x7f800000u) { *p = (uint16_t)((u >> 16) | 0x40); return; }
    u += 0x7fffu + ((u >> 16) & 1u);
    *p = (uint16_t)(u >> 16);
}

typedef float f32x4a4 __attribute__((ext_vector_type(4), aligned(4)));

// INIT: master <- parameter, m = v = 0.  Otherwise one AdamW step.  (All buffers may start at any element: a piece is loaded and
// stored as bytes, which global memory takes at any alignment.)  PAST: the state goes past the caches.
template <typename T, bool INIT, bool PAST = true>
__global__ __launch_bounds__(256) void adamw_kernel(AdamwBatch batch, int32_t count, int64_t k, int64_t n) {
    const int32_t wg = blockIdx.x;
    int32_t lo = 0, hi = count;              // the first adapter whose matrices end behind this work group
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (batch.e[mid].endB <= wg) lo = mid + 1; else hi = mid;
    }
    const AdamwEntry& e = batch.e[lo];
    const bool isB = wg >= e.endA;
    const int64_t numel = (isB ? n : k) * (int64_t)e.rank;
    const int32_t first = isB ? e.endA : (lo > 0 ? batch.e[lo - 1].endB : 0);
    T* param = (T*)(isB ? e.B : e.A);
    const T* grad = (const T*)(isB ? e.dB : e.dA);
    float* master = isB ? e.sB : e.sA;
    float* mm = master + numel;
    float* vv = mm + numel;
    const float lr = e.lr, beta1 = e.beta1, beta2 = e.beta2, eps = e.eps, wd = e.wd, c1 = e.c1, c2 = e.c2;
    auto update = [&](float g, float& th, float& m, float& v) {
        m = beta1 * m + (1.0f - beta1) * g;
        v = beta2 * v + (1.0f - beta2) * g * g;
        th = th - lr * ((m * c1) / (sqrtf(v * c2) + eps) + wd * th);
    };
    const int64_t base = (int64_t)(wg - first) * kRun + threadIdx.x * 4;
    struct T4 { T t[4]; };
    auto load = [](const float* at) {
        const f32x4a4* const src = reinterpret_cast<const f32x4a4*>(at);
        return PAST ? __builtin_nontemporal_load(src) : *src;
    };
    auto store = [](f32x4a4 x, float* at) {
        f32x4a4* const dst = reinterpret_cast<f32x4a4*>(at);
        if (PAST) __builtin_nontemporal_store(x, dst); else *dst = x;
    };
    if (base + 3 * 1024 + 4 <= numel) {
        T4 g[4];
        f32x4a4 th[4], m[4], v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t idx = base + u * 1024;
            if (INIT) {
                __builtin_memcpy(&g[u], param + idx, sizeof(T4));
            } else {
                __builtin_memcpy(&g[u], grad + idx, sizeof(T4));
                th[u] = load(master + idx);
                m[u] = load(mm + idx);
                v[u] = load(vv + idx);
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t idx = base + u * 1024;
            T4 p;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float x = ldp<T>(&g[u].t[c]);
                if (INIT) { th[u][c] = x; m[u][c] = 0.f; v[u][c] = 0.f; continue; }
                float tc = th[u][c], mc = m[u][c], vc = v[u][c];
                update(x, tc, mc, vc);
                th[u][c] = tc; m[u][c] = mc; v[u][c] = vc;
                stp<T>(&p.t[c], tc);
            }
            store(th[u], master + idx);
            store(m[u], mm + idx);
            store(v[u], vv + idx);
            if (!INIT) __builtin_memcpy(param + idx, &p, sizeof(T4));
        }
    } else {
        for (int u = 0; u < 4; ++u)
            for (int c = 0; c < 4; ++c) {
                const int64_t idx = base + u * 1024 + c;
                if (idx >= numel) continue;
                if (INIT) {
                    master[idx] = ldp<T>(param + idx); mm[idx] = 0.f; vv[idx] = 0.f;
                } else {
                    float th = master[idx], m = mm[idx], v = vv[idx];
                    update(ldp<T>(grad + idx), th, m, v);
                    master[idx] = th; mm[idx] = m; vv[idx] = v;
                    stp<T>(param + idx, th);
                }
            }
    }
}

static bool misaligned4(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 3u) != 0; }

static int run(mlora_plan* p, void* const* A, void* const* B, const void* const* dA, const void* const* dB,
               float* const* sA, float* const* sB, const mlora_adamw_hparams* hp, bool init, hipStream_t st) {
    if (!p) { set_error("plan is NULL"); return MLORA_ERR_NULL; }
    if (p->N == 0) return MLORA_OK;
    if (!A || !B || !sA || !sB || (!init && (!dA || !dB || !hp))) {
        set_error("A / B / dA / dB / stateA / stateB / hp is NULL");
        return MLORA_ERR_NULL;
    }
    for (int32_t i = 0; i < p->N; ++i) {
        if (p->ranks[i] == 0) continue;
        if (!A[i] || !B[i] || !sA[i] || !sB[i] || (!init && (!dA[i] || !dB[i]))) {
            set_error("a pointer of an adapter with rank > 0 is NULL");
            return MLORA_ERR_NULL;
        }
        if (misaligned4(sA[i]) || misaligned4(sB[i])) {
            set_error("optimizer state must be 4-byte aligned");
            return MLORA_ERR_ALIGN;
        }
        if (!init) {
            const mlora_adamw_hparams& h = hp[i];
            if (h.step < 1 || !(h.beta1 >= 0.f && h.beta1 < 1.f) || !(h.beta2 >= 0.f && h.beta2 < 1.f) ||
                !std::isfinite(h.lr) || !std::isfinite(h.eps) || !std::isfinite(h.weight_decay)) {
                set_error("AdamW hyper-parameters out of range (step >= 1, 0 <= beta < 1, finite lr / eps / weight_decay)");
                return MLORA_ERR_SCALE;
            }
        }
    }
    int64_t params = 0;
    for (int32_t i = 0; i < p->N; ++i) params += p->ranks[i] * (p->k + p->n);
    const int64_t element = p->dtype == MLORA_F32 ? 4 : 2, whole_step = params * (12 + 2 * element) + (p->k * p->n + 2 * p->T * (p->k + p->n)) * element;
    const bool cached = !p->shares_tables && p->blocks.front().use_count() == 1 && whole_step < 256000000;
    auto groups = [](int64_t numel) { return (numel + kRun - 1) / kRun; };
    for (int32_t base = 0; base < p->N;) {
        AdamwBatch batch;
        std::memset(&batch, 0, sizeof(batch));
        int32_t cnt = 0;
        int64_t total = 0;
        for (; base < p->N && cnt < kBatch; ++base) {
            const int32_t i = base;
            if (p->ranks[i] == 0) continue;
            const int64_t endA = total + groups(p->k * p->ranks[i]), endB = endA + groups(p->n * p->ranks[i]);
            if (endB > INT32_MAX) {
                if (cnt > 0) break;                        // the next launch takes it
                set_error("AdamW: an adapter's matrices exceed 2^43 elements");
                return MLORA_ERR_SHAPE;
            }
            AdamwEntry& e = batch.e[cnt++];
            e.A = A[i]; e.B = B[i]; e.sA = sA[i]; e.sB = sB[i];
            e.rank = p->ranks[i]; e.endA = (int32_t)endA; e.endB = (int32_t)endB;
            total = endB;
            if (!init) {
                e.dA = dA[i]; e.dB = dB[i];
                const mlora_adamw_hparams& h = hp[i];
                e.lr = h.lr; e.beta1 = h.beta1; e.beta2 = h.beta2; e.eps = h.eps; e.wd = h.weight_decay;
                e.c1 = (float)(1.0 / (1.0 - std::pow((double)h.beta1, (double)h.step)));
                e.c2 = (float)(1.0 / (1.0 - std::pow((double)h.beta2, (double)h.step)));
            }
        }
        if (cnt == 0) break;
        ProfScope prof(p, MLORA_K_ADAMW, st);
        const bool f32 = p->dtype == MLORA_F32;
        const dim3 grid((unsigned)total);
        if (init && f32)       hipLaunchKernelGGL((adamw_kernel<float, true>), grid, dim3(256), 0, st, batch, cnt, p->k, p->n);
        else if (init)         hipLaunchKernelGGL((adamw_kernel<uint16_t, true>), grid, dim3(256), 0, st, batch, cnt, p->k, p->n);
        else if (f32 && cached) hipLaunchKernelGGL((adamw_kernel<float, false, false>), grid, dim3(256), 0, st, batch, cnt, p->k, p->n);
        else if (f32)          hipLaunchKernelGGL((adamw_kernel<float, false>), grid, dim3(256), 0, st, batch, cnt, p->k, p->n);
        else if (cached)       hipLaunchKernelGGL((adamw_kernel<uint16_t, false, false>), grid, dim3(256), 0, st, batch, cnt, p->k, p->n);
        else                   hipLaunchKernelGGL((adamw_kernel<uint16_t, false>), grid, dim3(256), 0, st, batch, cnt, p->k, p->n);
    }
    MLORA_HIP_TRY(hipGetLastError());
    return MLORA_OK;
}

}  // namespace mlora

extern "C" int multi_lora_adamw_init(mlora_plan* plan, const void* const* A, const void* const* B,
                                     float* const* stateA, float* const* stateB, void* stream) {
    return mlora::run(plan, (void* const*)A, (void* const*)B, nullptr, nullptr, stateA, stateB, nullptr, true,
                      (hipStream_t)stream);
}

extern "C" int multi_lora_adamw_step(mlora_plan* plan, void* const* A, void* const* B, const void* const* dA,
                                     const void* const* dB, float* const* stateA, float* const* stateB,
                                     const mlora_adamw_hparams* hp, void* stream) {
    return mlora::run(plan, A, B, dA, dB, stateA, stateB, hp, false, (hipStream_t)stream);
}
