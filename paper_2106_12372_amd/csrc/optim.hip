// Weight-gradient reduction and the Adam update (Sec. 5 "Optimizer").
//
// k_reduce<ADAM>: a workgroup owns 32 consecutive weights; its 8 groups of 32
// lanes each sum every 8th partial (a tile's, or a workgroup's of the 16-bit
// trainer) for one weight (coalesced 128-byte rows), with Neumaier compensation, and
// the 8 group sums are combined in a fixed order, so the reduced gradient does not
// depend on scheduling.
// Without ADAM the gradient is written out (backward of the autograd form).
// With ADAM the workgroup ORs the non-finite flags the training kernel wrote, one per
// partial: if any is set the whole step is skipped (weights, moments and
// step count stay as they are); otherwise each weight's FP32 master copy and
// Adam moments are updated and its FP16/BF16 copies in both matrix-core
// fragment layouts are refreshed.  The step count lives in two device slots
// used in alternation (read one, write the other), so no thread of the launch
// reads a value another thread of the same launch writes.  Workgroup 0 also
// reduces the tiles' loss terms.
#include "nrc_internal.h"

namespace nrc {
namespace {

__device__ inline void neumaier_add(float& s, float& c, float x) {
    const float t = s + x;
    if (fabsf(s) >= fabsf(x)) c += (s - t) + x; else c += (x - t) + s;
    s = t;
}

// Layer holding flat index p (weights and partial slots share the ranges).
__device__ inline int layer_of(const Geo& d, int p) {
    if (p < d.w_off(1)) return 0;
    if (p >= d.w_off(d.H)) return d.H;
    return 1 + (p - d.w_off(1)) / (d.W * d.W);
}

// Weight index held by partial slot s in the matrix-core accumulator layout:
// slot w_off(l) + ((mb * NB + nb) * 64 + lane) * 4 + j holds
// dW_l[16 mb + 4 (lane / 16) + j][16 nb + lane % 16]; the output layer is
// row-major.
__device__ inline int param_of_slot(const Geo& d, int s) {
    const int l = layer_of(d, s);
    if (l == d.H) return s;
    const int r = s - d.w_off(l);
    const int cols = d.cols(l), NB = cols >> 4;
    const int j = r & 3, lane = (r >> 2) & 63, blk = r >> 8;
    const int mb = blk / NB, nb = blk - mb * NB;
    return d.w_off(l) + (16 * mb + 4 * (lane >> 4) + j) * cols + 16 * nb + (lane & 15);
}

// Locate weight p (flat index) as (layer, row, column).
__device__ inline void locate(const Geo& d, int p, int& l, int& o, int& k) {
    l = layer_of(d, p);
    const int r = p - d.w_off(l);
    const int cols = d.cols(l);
    o = r / cols;
    k = r - o * cols;
}

// Forward and backward fragment slots of weight p.
__device__ inline void frag_slots(const Geo& d, int p, int64_t& fi, int64_t& bi) {
    int l, o, k;
    locate(d, p, l, o, k);
    fi = fwd_frag_index(d, l, o, k);
    bi = bwd_frag_index(d, l, o, k);
}

// A weight into its forward and backward fragment slots fi, bi.  split: also
// the lo part w - hi into the second copy that follows each array (the BF16
// form's training fragments).
template <typename T>
__device__ inline void put_frags(const Geo& d, int64_t fi, int64_t bi, float w, T* ffr, T* bfr, bool split) {
    const T v = (T)w;
    if (ffr) ffr[fi] = v;
    if (bfr) bfr[bi] = v;
    if (split) {
        const T lo = (T)(w - (float)v);
        if (ffr) ffr[(int64_t)d.n_fwd_frags() * kFragElems + fi] = lo;
        if (bfr) bfr[(int64_t)d.n_bwd_frags() * kFragElems + bi] = lo;
    }
}

template <typename T>
__device__ inline void write_frags(const Geo& d, int p, float w, T* ffr, T* bfr, bool split = false) {
    int64_t fi, bi;
    frag_slots(d, p, fi, bi);
    put_frags<T>(d, fi, bi, w, ffr, bfr, split);
}

constexpr int kRedParams = 32;   // weights per workgroup
constexpr int kRedGroups = 8;    // tile groups per workgroup

// Threads: the groups and, with ADAM, a fifth wave for what the update needs
// beside the sums.  It ORs the flags and forms the bias corrections (a load and
// three powf, one after the other) while the other four wait for their partials,
// and workgroup 0's also adds up the loss.  In the first wave, ahead of its
// partials' loads, these held every launch up (us: 16 partials 5.5 -> 4.6, 256 6.8
// -> 6.5; 512 partials and 4,096 loss terms 24.0 -> 11.8, 8.1 at the rate of a
// copy).  Twice as many groups of half as many partials: 1.5 us slower; half as
// many: the same.
constexpr int kRedThreads = kRedParams * kRedGroups;
constexpr int red_threads(bool adam) { return kRedThreads + (adam ? 64 : 0); }

template <typename T, bool ADAM, bool NATIVE>
__global__ __launch_bounds__(red_threads(ADAM)) void k_reduce(const float* __restrict__ partials, int n_tiles,
                                                const int32_t* __restrict__ tile_bad,
                                                const float* __restrict__ loss_part, int n_loss,
                                                float inv_count, float* __restrict__ loss_out, float inv_scale,
                                                float* __restrict__ grad_out, float* __restrict__ w,
                                                float* __restrict__ m, float* __restrict__ v,
                                                int32_t* __restrict__ tslots, int parity, AdamHyper hp,
                                                EmaArgs ema, int32_t* __restrict__ skipped_out,
                                                T* __restrict__ ffr, T* __restrict__ bfr, int width,
                                                int n_hidden) {
    __shared__ float s_sum[kRedGroups][kRedParams];
    __shared__ float s_cmp[kRedGroups][kRedParams];
    __shared__ float s_bc[3];
    __shared__ int s_skip;
    const Geo d(width, n_hidden);
    const int P = d.n_params();
    const int tid = threadIdx.x, lane = tid & 63;
    const int pl = tid % kRedParams, grp = tid / kRedParams;
    const int sidx = blockIdx.x * kRedParams + pl;          // partial slot (coalesced across lanes)
    const bool side = ADAM && __builtin_amdgcn_readfirstlane(tid >> 6) == kRedThreads / 64;

    int t_old = 0;
    if (ADAM) t_old = tslots[parity];
    if (side) {
        constexpr int kBad = 8;                             // loads in flight
        int any = 0;
        for (int t = lane; t < n_tiles; t += 64 * kBad) {
            int b[kBad];
            #pragma unroll
            for (int u = 0; u < kBad; ++u) b[u] = t + 64 * u < n_tiles ? tile_bad[t + 64 * u] : 0;
            #pragma unroll
            for (int u = 0; u < kBad; ++u) any |= b[u];
        }
        // bias corrections of the step this update would make (a skipped step
        // updates nothing): lane 0's of m, lane 1's of v, lane 2's of the EMA
        const float base = lane == 0 ? hp.beta1 : lane == 1 ? hp.beta2 : ema.alpha;
        if (lane < (ema.alpha > 0.0f ? 3 : 2)) s_bc[lane] = 1.0f - powf(base, (float)(t_old + 1));
        #pragma unroll
        for (int off = 32; off >= 1; off >>= 1) any |= __shfl_xor(any, off, 64);
        if (lane == 0) s_skip = any;
    }
    // The update's operands for this thread's weight are loaded before the
    // partials, so their latency overlaps the sums.
    const bool owner = grp == 0 && sidx < P;
    const int p = NATIVE ? param_of_slot(d, owner ? sidx : 0) : sidx;
    float w0 = 0.0f, m0 = 0.0f, v0 = 0.0f, e0 = 0.0f;
    int64_t fi = 0, bi = 0;
    if (ADAM && owner) {
        w0 = w[p];
        m0 = m[p];
        v0 = v[p];
        if (ema.alpha > 0.0f) e0 = ema.e[p];
        if (ffr != nullptr || ema.effr != nullptr) frag_slots(d, p, fi, bi);
    }
    // The thread's partials, every kRedGroups-th, summed in order.  Rounds of 32
    // loads in flight, then 16, 8, 4, 2 and 1, the same for every group, and the
    // last, which only some groups have (64 partials, 4,096 records: one round of 8
    // instead of 8 loads one after another, 2.4 us less per step).
    float s = 0.0f, c = 0.0f;
    if (!side && sidx < P) {
        const float* src = partials + (int64_t)grp * P + sidx;
        const int64_t step = (int64_t)kRedGroups * P;
        auto round = [&](auto k_) {
            constexpr int K = decltype(k_)::value;
            float x[K];
            #pragma unroll
            for (int u = 0; u < K; ++u) x[u] = __builtin_nontemporal_load(src + u * step);
            src += K * step;
            #pragma unroll
            for (int u = 0; u < K; ++u) neumaier_add(s, c, x[u]);
        };
        int k = n_tiles / kRedGroups;
        for (; k >= 32; k -= 32) round(IntC<32>{});
        if (k & 16) round(IntC<16>{});
        if (k & 8) round(IntC<8>{});
        if (k & 4) round(IntC<4>{});
        if (k & 2) round(IntC<2>{});
        if (k & 1) round(IntC<1>{});
        if (grp < n_tiles % kRedGroups) round(IntC<1>{});
    }
    if (!side) {
        s_sum[grp][pl] = s;
        s_cmp[grp][pl] = c;
    }
    __syncthreads();

    if (side) {
        if (blockIdx.x != 0 || loss_out == nullptr) return;
        // compensated sum of the per-tile loss terms, then a compensated
        // combine of the 64 lane sums in a fixed order
        constexpr int kLoss = 32;                           // loads in flight
        float ls = 0.0f, lc = 0.0f;
        for (int t = lane; t < n_loss; t += 64 * kLoss) {
            float x[kLoss];
            #pragma unroll
            for (int u = 0; u < kLoss; ++u) x[u] = t + 64 * u < n_loss ? loss_part[t + 64 * u] : 0.0f;
            #pragma unroll
            for (int u = 0; u < kLoss; ++u)
                if (t + 64 * u < n_loss) neumaier_add(ls, lc, x[u]);
        }
        #pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const float os = __shfl_xor(ls, off, 64), oc = __shfl_xor(lc, off, 64);
            // both partners form the same pair sum (the lower lane's operand first)
            const bool lo = (lane & off) == 0;
            float a = lo ? ls : os, ac = lo ? lc : oc;
            neumaier_add(a, ac, lo ? os : ls);
            ac += lo ? oc : lc;
            ls = a;
            lc = ac;
        }
        if (lane == 0) *loss_out = (ls + lc) * inv_count;
        return;
    }
    if (!owner) return;   // workgroup 0's thread 0 has slot 0 and stays
    float gv = 0.0f;
    {
        float S = 0.0f, C = 0.0f;
        #pragma unroll
        for (int k = 0; k < kRedGroups; ++k) {
            neumaier_add(S, C, s_sum[k][pl]);
            C += s_cmp[k][pl];
        }
        gv = (S + C) * inv_scale;
    }
    if (!ADAM) {
        grad_out[p] = gv;
        return;
    }
    const int skip = s_skip;
    const int t_new = skip ? t_old : t_old + 1;
    if (blockIdx.x == 0 && tid == 0) {
        tslots[parity ^ 1] = t_new;
        if (skipped_out) *skipped_out = skip;
    }
    if (skip) return;
    const float bc1 = s_bc[0], bc2 = s_bc[1];
    // explicit fused multiply-adds: the rounding does not depend on which
    // product the compiler would contract
    const float m1 = fmaf(hp.beta1, m0, (1.0f - hp.beta1) * gv);
    const float v1 = fmaf(hp.beta2, v0, ((1.0f - hp.beta2) * gv) * gv);
    const float w1 = w0 - hp.lr * (m1 / bc1) / (sqrtf(v1 / bc2) + hp.eps);
    w[p] = w1;
    m[p] = m1;
    v[p] = v1;
    if (ffr != nullptr) put_frags<T>(d, fi, bi, w1, ffr, bfr, __is_same(T, __bf16));
    if (ema.alpha > 0.0f) {
        // Eq. 2, bias-corrected: E_t = a E_{t-1} + (1 - a) W_t, W_bar_t = E_t / (1 - a^t).
        const float e1 = fmaf(ema.alpha, e0, (1.0f - ema.alpha) * w1);
        const float wb = e1 / s_bc[2];
        ema.e[p] = e1;
        ema.wbar[p] = wb;
        if (ema.effr != nullptr) put_frags<T>(d, fi, bi, wb, (T*)ema.effr, (T*)nullptr, false);
    }
}

template <typename T>
__global__ __launch_bounds__(256) void k_build_frags(const float* __restrict__ w, T* __restrict__ ffr,
                                                     T* __restrict__ bfr, T* __restrict__ ffr2,
                                                     int width, int n_hidden) {
    const Geo d(width, n_hidden);
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= d.n_params()) return;
    write_frags<T>(d, p, w[p], ffr, bfr, __is_same(T, __bf16) && bfr != nullptr);
    if (ffr2) write_frags<T>(d, p, w[p], ffr2, (T*)nullptr);
}

// Weights set from device memory, everything that goes with them in one launch:
// the master copy, the Adam moments and step count cleared, the EMA set at
// W_bar = W, E = 0 (e, wbar NULL: none) and the fragments of each
// reduced-precision copy (ffr NULL: none; the slots no weight maps to stay the
// zeros they were created with).  Bound by latency: a thread per weight, ~28
// bytes each; it replaces two copies, up to seven fills and the fragment build
// (W = 128, 5 layers: 61 -> 5 us of device time per call).
template <typename T>
__global__ __launch_bounds__(256) void k_install(const float* src, float* w, float* __restrict__ m,
                                                 float* __restrict__ v, int32_t* __restrict__ tslots,
                                                 float* __restrict__ e, float* __restrict__ wbar,
                                                 T* __restrict__ ffr, T* __restrict__ bfr, T* __restrict__ effr,
                                                 int width, int n_hidden) {
    const Geo d(width, n_hidden);
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p < 4) tslots[p] = 0;
    if (p >= d.n_params()) return;
    const float x = src[p];
    w[p] = x;
    m[p] = 0.0f;
    v[p] = 0.0f;
    if (wbar) {
        wbar[p] = x;
        e[p] = 0.0f;
    }
    if (ffr) {
        int64_t fi, bi;
        frag_slots(d, p, fi, bi);
        put_frags<T>(d, fi, bi, x, ffr, bfr, __is_same(T, __bf16));
        if (effr) put_frags<T>(d, fi, bi, x, effr, (T*)nullptr, false);
    }
}

}  // namespace

int reduce_blocks(int n_params) { return (n_params + kRedParams - 1) / kRedParams; }

hipError_t launch_reduce(const Geo& d, bool native, const float* partials, int n_parts,
                         float inv_scale, float* grad, hipStream_t s) {
    const dim3 grid(reduce_blocks(d.n_params())), block(red_threads(false));
    auto k = native ? k_reduce<_Float16, false, true> : k_reduce<_Float16, false, false>;
    hipLaunchKernelGGL(k, grid, block, 0, s, partials, n_parts, (const int32_t*)nullptr,
                       (const float*)nullptr, 0, 1.0f, (float*)nullptr, inv_scale, grad, (float*)nullptr, (float*)nullptr,
                       (float*)nullptr, (int32_t*)nullptr, 0, AdamHyper{}, EmaArgs{},
                       (int32_t*)nullptr, (_Float16*)nullptr, (_Float16*)nullptr, d.W, d.H);
    return hipGetLastError();
}

hipError_t launch_reduce_adam(int precision, const Geo& d, bool native, const float* partials,
                              int n_parts, const int32_t* tile_bad, const float* loss_part, int n_loss,
                              float inv_count, float* loss_out, float inv_scale, float* w, float* m,
                              float* v, int32_t* tslots, int parity, AdamHyper hp, EmaArgs ema,
                              int32_t* skipped_out, void* ffr, void* bfr, hipStream_t s) {
    const dim3 grid(reduce_blocks(d.n_params())), block(red_threads(true));
    if (precision == NRC_BF16) {
        auto k = native ? k_reduce<__bf16, true, true> : k_reduce<__bf16, true, false>;
        hipLaunchKernelGGL(k, grid, block, 0, s, partials, n_parts, tile_bad, loss_part, n_loss, inv_count,
                           loss_out, inv_scale, (float*)nullptr, w, m, v, tslots, parity, hp, ema,
                           skipped_out, (__bf16*)ffr, (__bf16*)bfr, d.W, d.H);
    } else {
        // FP32 caches have no reduced-precision copies (ffr, bfr, ema.effr are NULL).
        auto k = native ? k_reduce<_Float16, true, true> : k_reduce<_Float16, true, false>;
        hipLaunchKernelGGL(k, grid, block, 0, s, partials, n_parts, tile_bad, loss_part, n_loss, inv_count,
                           loss_out, inv_scale, (float*)nullptr, w, m, v, tslots, parity, hp, ema,
                           skipped_out, (_Float16*)ffr, (_Float16*)bfr, d.W, d.H);
    }
    return hipGetLastError();
}

hipError_t launch_build_frags(int precision, const Geo& d, const float* w, void* ffr, void* bfr,
                              void* ffr2, hipStream_t s) {
    const dim3 grid((d.n_params() + 255) / 256), block(256);
    if (precision == NRC_FP16)
        hipLaunchKernelGGL(k_build_frags<_Float16>, grid, block, 0, s, w, (_Float16*)ffr,
                           (_Float16*)bfr, (_Float16*)ffr2, d.W, d.H);
    else if (precision == NRC_BF16)
        hipLaunchKernelGGL(k_build_frags<__bf16>, grid, block, 0, s, w, (__bf16*)ffr, (__bf16*)bfr,
                           (__bf16*)ffr2, d.W, d.H);
    return hipGetLastError();
}

hipError_t launch_install(int precision, const Geo& d, const float* src, float* w, float* m, float* v,
                          int32_t* tslots, float* e, float* wbar, void* ffr, void* bfr, void* effr,
                          hipStream_t s) {
    const dim3 grid((d.n_params() + 255) / 256), block(256);
    if (precision == NRC_BF16)
        hipLaunchKernelGGL(k_install<__bf16>, grid, block, 0, s, src, w, m, v, tslots, e, wbar, (__bf16*)ffr,
                           (__bf16*)bfr, (__bf16*)effr, d.W, d.H);
    else
        // FP32 caches have no reduced-precision copies (ffr, bfr, effr are NULL)
        hipLaunchKernelGGL(k_install<_Float16>, grid, block, 0, s, src, w, m, v, tslots, e, wbar, (_Float16*)ffr,
                           (_Float16*)bfr, (_Float16*)effr, d.W, d.H);
    return hipGetLastError();
}

}  // namespace nrc
