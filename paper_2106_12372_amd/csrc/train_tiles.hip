// Training in the FP16/BF16 matrix-core forms: forward pass, loss gradient of Eq.
// 5 (or an upstream gradient), data backward pass and weight gradients, with the
// weight gradients of all a workgroup's tiles summed in registers.
//
// A workgroup of 8 waves takes 64-record tiles one after another.  In every
// layer a wave owns one 16-row block of the output for NC of the tile's four
// 16-record columns, so a weight fragment is read by one wave per tile (two at
// width 64; every wave that holds records in k_train_mfma) and goes from L2 to
// registers while the wave waits for the layer before.  Activations and deltas
// pass between the waves through LDS, record-major, each 32-feature chunk of a
// row in the order of the operand slots ("chained" order, nrc_internal.h): the B
// operand of the next product is one 16-byte read.  Only two layers' deltas are
// held.  While the waves form delta_l they also form dW_l = delta_{l+1} h_l^T over
// the tile's 64 records, the record index along K by LDS transpose reads, into
// accumulators that stay in registers from tile to tile.  Each workgroup writes
// its sums once, in the accumulator layout the reduction expects: one partial per
// up to kHeld tiles.
//
// Every record's forward pass, loss and deltas go through the same products in
// the same order as in k_train_mfma; only the grouping of the records' weight
// gradients differs.
//
// Bound by LDS traffic and the barrier between layers.  Cycle stamps of a tile: width
// 128 (FP16) 28k cycles, 1.9k per forward layer, 3.2k per backward layer with its
// weight gradient; width 64, two workgroups per CU, 15k, 0.9k and 1.4k (a backward
// layer reads 88 KB from LDS, 0.7k cycles at 128 bytes each). The partials' one write
// takes 27k cycles at width 128 (76 MB over the chip, at the rate of a copy).  At width
// 128 the sums alone take 148 of a wave's 256 registers and some of the rest spill:
// BF16 steps 22 (92 bytes of scratch per lane), backward passes 10 from the buffer and
// 19 to 21 without; FP16 steps 8, recomputing backward passes 2 to 5, from the buffer
// none.  Whole training steps, us, k_train_mfma before and now: width 64 FP16 16,384
// records 17.5 / 16.0, 65,536 48 / 29, 262,144 183 / 72, BF16 1,000 records 18.6 /
// 13.9, 262,144 232 / 82; width 128 FP16 1,000 records 53 / 28, 16,384 97 / 41, 65,536
// 306 / 73, BF16 65,536 438 / 94.  At width 128 a wave with two row blocks and two
// columns instead of one and four was slower (83 and 134 us: its fragments spill).
#include "mfma_ops.h"
#include "nrc_internal.h"

namespace nrc {
namespace {

constexpr int kTS = 64;           // records per tile
constexpr int kWaves = 8;
constexpr int kLdT = 72;          // dL/dy, feature-major

// The most tiles of a workgroup; larger batches take several launches, one after the
// other, each with partials of its own.  A tile adds to its workgroup's sums in plain
// FP32, the reduction adds the partials with compensation.  Held without end the sums'
// error grows with the batch: small terms after large ones vanish, and in a model of
// the additions (non-negative terms, 256 workgroups, mean relative error) 512 tiles
// each give 2.8e-8 and 4,096 6.5e-8.  With 8 it is 2.0e-8 for any number, as with one
// partial per tile: that of rounding the result.  Steps at depth 5, us, one launch /
// as here (more partials, 4 us from launch to launch): FP16 width 64 262,208 records
// 73.9 / 81.6, 524,288 132 / 141, 1,048,576 252 / 279; width 128 262,144 208 / 232.
// Starting the sums anew inside the kernel took 75.2, 139, 272 and 223, but spills more
// registers at width 128 (BF16 steps of 65,536 records 93.9 -> 96.4).
constexpr int kHeld = 8;

// Where a wave has 256 registers at width 64 (ROOMY), the LDS rows of h_0 .. h_H and
// the deltas are unpadded and element e of row r lies at e ^ row_key: the row's
// 16-byte chunks change places by bits of r, so that no 16-byte read of a chunk of 16
// rows (a pass takes 8 lanes of one lane group and the other 8 rows' of the next) and
// no transpose read of two chunks of rows 8g .. +3 by two lane groups puts two lanes
// of a pass on one bank.  With 8 elements of padding, as elsewhere, these take twice
// their passes (by the conflict counters, 8 and 4 instead of 4 and 2); the fewer
// 8-byte stores take 16 instead of 8, the 8-byte reads 4 either way.  Swapped rows'
// addresses need registers and vector instructions that the other instances lack.
// Steps, us, padded / swapped: FP16 1,000 records 13.2 / 12.8, 16,384 16.0 / 15.9, a raw
// frame's four 70.5 / 67.8, depth 8 16.8 / 16.3; two workgroups per CU, 262,144 records,
// 72.5 / 75.5; width 128, 65,536, 73 / 78.  A key that spreads the stores as well (bits
// 3 ^ 2 and 2 below bit 1) gives rows r and r + 4 of a transpose read addresses of
// their own: 1,000 records 13.1, 40,001 24.0 instead of 24.7, not kept.
__host__ __device__ constexpr bool roomy(int W, int wgs) { return W == 64 && wgs == 1; }
__host__ __device__ constexpr int row_stride(int W, bool swap) { return swap ? W : W + 8; }
template <bool SWAP>
__device__ inline int row_key(int r) {
    return SWAP ? (r & 2) << 4 | (r & 8) << 1 : 0;
}
// LDS bytes: h_0 [64][72 or 64], h_1 .. h_H and two deltas [64][W + 8 or W], dL/dy
// feature-major [3][72] and record-major [64][4], network outputs [64][4] (FP32).
__host__ __device__ constexpr int tiles_lds_bytes(int W, int H, bool swap) {
    return (kTS * (row_stride(64, swap) + (H + 2) * row_stride(W, swap)) + 3 * kLdT + kTS * 4) * 2 + kTS * 16;
}

// UPSTREAM: tgt holds dL/d(prediction) instead of targets.  GENC: dL/d(input) is
// formed too.  RAWL >= 0: enc points at raw records of that layout, encoded here
// with PRESET; -1: encoded rows.  ACT: kActLoad reads the
// forward pass from the activation buffer ([record][layer][feature], and the
// network outputs [record][4]) instead of computing it; kActStore computes it,
// writes the buffer and the predictions (to out) and stops there.  out: dL/d(input)
// in the GENC forms.  MAXH: the most hidden layers the accumulators hold.  WGS:
// workgroups per CU.
constexpr int kActNone = 0, kActStore = 1, kActLoad = 2;

template <typename T, int W, int MAXH, int WGS, bool UPSTREAM, bool GENC, int ACT, int RAWL, int PRESET>
__global__ __launch_bounds__(64 * kWaves, 2 * WGS) void k_train_tiles(const T* __restrict__ ffr, const T* __restrict__ bfr,
                                                             const T* __restrict__ enc,
                                                             const float* __restrict__ tgt,
                                                             const int32_t* __restrict__ idx, int64_t n, int n_hidden,
                                                             float loss_eps, float grad_scale,
                                                             float* __restrict__ partials,
                                                             float* __restrict__ loss_part,
                                                             int32_t* __restrict__ part_bad,
                                                             float* __restrict__ out, int fcol,
                                                             T* __restrict__ act, float* __restrict__ act_y,
                                                             LcgGather lg) {
    using V = typename Vec8<T>::type;
    typedef T t4 __attribute__((ext_vector_type(4)));
    constexpr bool SPLIT = __is_same(T, __bf16);
    constexpr bool ROOMY = roomy(W, WGS);
    constexpr int MB = W / 16, KC = W / 32, LD0 = row_stride(64, ROOMY), LDR = row_stride(W, ROOMY);
    constexpr int RG = W / 16, NC = W / 32;                  // waves: RG row blocks x (8 / RG) groups of NC columns
    constexpr int NTH = 64 * kWaves;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    __shared__ float wsum[4];
    // every region at a fixed offset, the activations last
    T* h0 = reinterpret_cast<T*>(smem_raw);
    T* dO = h0 + kTS * LD0;                                 // dL/dy [3][kLdT]
    T* dR = dO + 3 * kLdT;                                   // dL/dy [64][4]
    float* fy = reinterpret_cast<float*>(dR + kTS * 4);      // network outputs [64][4]
    T* ds = reinterpret_cast<T*>(fy + kTS * 4);              // delta_l in block l & 1
    T* hs = ds + 2 * kTS * LDR;                              // h_1 .. h_H
    auto hrow = [&](int l) { return hs + (l - 1) * kTS * LDR; };
    auto drow = [&](int l) { return ds + (l & 1) * kTS * LDR; };

    const Geo geo(W, n_hidden);
    const int P = geo.n_params();
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, ln = lane & 15;
    const int rb = wave % RG, col0 = (wave / RG) * NC;
    const int lo_f = geo.n_fwd_frags() * 64, lo_b = geo.n_bwd_frags() * 64;

    // A product's weight operand, hi part and (BF16) lo part.
    struct Frag { V hi, lo; };
    auto ld = [&](const V* f, int lo) {
        Frag r;
        r.hi = *f;
        if (SPLIT) r.lo = f[lo];
        return r;
    };
    auto mm = [&](const Frag& a, const V& b, f32x4 c) {
        c = mfma(a.hi, b, c);
        if (SPLIT) c = mfma(a.lo, b, c);
        return c;
    };
    const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
    // This wave's fragments of a layer, loaded while the layer before finishes.
    Frag fr[KC];
    auto load_frags = [&](const V* base, int kc, int row, int lo) {
        #pragma unroll
        for (int c = 0; c < KC; ++c)
            if (c < kc) fr[c] = ld(base + (row * kc + c) * 64, lo);
    };
    // The four values of this wave's row block a lane holds of column col, into a
    // row store.
    auto put = [&](T* rows, int col, f32x4 v, bool relu_it) {
        T* dst = rows + (16 * col + ln) * LDR + ((32 * (rb >> 1) + 8 * g + 4 * (rb & 1)) ^ row_key<ROOMY>(ln));
        const V p = pack8<T, V>(v, v);
        const V q = relu_it ? relu_packed(p) : p;
        *reinterpret_cast<t4*>(dst) = __builtin_shufflevector(q, q, 0, 1, 2, 3);
    };
    // B operand chunk c of column col from a row store in slot order.
    auto get = [&](const T* rows, int stride, int col, int c) {
        return *reinterpret_cast<const V*>(rows + (16 * col + ln) * stride + ((32 * c + 8 * g) ^ row_key<ROOMY>(ln)));
    };
    // Operand of records 32 kc + 8 g .. +7 for row positions 16 blk + ln of a
    // record-major store (the transpose read of k_train_mfma).
    auto gather = [&](const T* base, int stride, int blk, int kc) {
        typedef short s16x4 __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
        const int r = 8 * g + (ln >> 2);                     // rows r and r + 4 have one key
        const T* p = base + (32 * kc + r) * stride + ((16 * blk + 4 * (ln & 3)) ^ row_key<ROOMY>(r));
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * stride));
        return __builtin_bit_cast(V, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };

    // Weight-gradient accumulators.  Layer l >= 1: row blocks MW (wave >> 2) ..,
    // column blocks NW (wave & 3) ..; layer 0 (64 columns): one column block,
    // wave & 3; output layer: column blocks wave, wave + 8 (waves 0 .. MB - 1).
    constexpr int MW = MB / 2, NW = MB / 4;
    const int mw0 = (wave >> 2) * MW, nw0 = (wave & 3) * NW;
    f32x4 acc0[MW], accw[MAXH > 1 ? MAXH - 1 : 1][MW][NW], acco = zero;
    #pragma unroll
    for (int i = 0; i < MW; ++i) {
        acc0[i] = zero;
        #pragma unroll
        for (int l = 0; l < MAXH - 1; ++l)
            #pragma unroll
            for (int j = 0; j < NW; ++j) accw[l][i][j] = zero;
    }

    // ROOMY (one workgroup per CU, 256 registers per wave): a layer's LDS reads at width
    // 64 go out together, before its first product: left to the compiler, each
    // product waits for operands read just before it, nine LDS latencies one after
    // another in a backward layer (16,384 records, us per step: FP16 16.6 -> 16.2, BF16
    // 17.7 -> 17.0).  128 registers hold neither these nor the weights below beside
    // the sums (they spill).
    // FP16: the weights of the whole backward chain are loaded ahead of it, too, as
    // loads behind the stores of a layer's sums wait for those (1,000 records 13.6 ->
    // 13.3 us per step; BF16, with its hi and lo parts, 17.1 -> 17.4 at 16,384).
    constexpr bool EARLY = ROOMY && MAXH <= 5 && !SPLIT;
    Frag fb[EARLY ? MAXH : 1][KC];
    auto reads_first = [] {
        if (ROOMY) __builtin_amdgcn_sched_barrier(0);
    };
    // The weights are read anew for each tile, and what only a part of the tile
    // needs is computed there: held in registers across the tiles (their loads and
    // addresses are loop-invariant) they would spill the accumulators.
    auto anew = [](int v) {
        asm volatile("" : "+v"(v));
        return v;
    };
    // A block of the workgroup's sums, in the layout of k_train_mfma's partials:
    // slot w_off + ((mb * NB + nb) * 64 + 16 g' + ln') * 4 + j holds
    // dW[16 mb + 4 g' + j][16 nb + ln'].  Rows (and, past layer 0, columns) sit in
    // slot order here: row positions 16 mbp + 4 g + j of a chunk are features
    // 16 (g & 1) + 4 (2 (mbp & 1) + (g >> 1)) + j, column position 16 nbp + ln
    // feature 16 ((ln >> 2) & 1) + 4 (2 (nbp & 1) + (ln >> 3)) + (ln & 3).  A layer's
    // sums leave as soon as the last tile has added to them, beside the layers
    // before it.
    float* part = partials + (int64_t)blockIdx.x * P;
    float bad = 0.0f;                        // NaN once a sum is not finite
    auto flush = [&](int l, int mbp, int nbp, const f32x4& a) {
        const int fl = anew(lane), fg = fl >> 4, fn = fl & 15;
        const int NB = l == 0 ? 4 : MB;
        const int mb = (mbp & ~1) + (fg & 1), gq = 2 * (mbp & 1) + (fg >> 1);
        const int nb = l == 0 ? nbp : (nbp & ~1) + ((fn >> 2) & 1);
        const int lq = l == 0 ? fn : 4 * (2 * (nbp & 1) + (fn >> 3)) + (fn & 3);
        __builtin_nontemporal_store(a, reinterpret_cast<f32x4*>(part + geo.w_off(l) + ((mb * NB + nb) * 64 + 16 * gq + lq) * 4));
        #pragma unroll
        for (int j = 0; j < 4; ++j) bad = fmaf(a[j], 0.0f, bad);
    };
    auto flush_layer = [&](int l) {
        #pragma unroll
        for (int i = 0; i < MW; ++i)
            #pragma unroll
            for (int j = 0; j < NW; ++j) flush(l, mw0 + i, nw0 + j, accw[l - 1][i][j]);
    };
    // Encoded rows: a thread moves 16 bytes of record tid / 8, and the output lanes
    // their record's targets; both are loaded during the tile before.
    const int64_t n_tiles = (n + kTS - 1) / kTS;
    V in_v = zero8<V>();
    float tg[3] = {0.f, 0.f, 0.f};
    int src_e = -1, src_t = -1;              // n <= 2^31
    auto find = [&](int64_t t) {             // the records behind tile t's slots (-1: none)
        const int ft = anew(tid);
        const int re = ft >> 3, rt = 16 * (wave & 3) + (ft & 15);
        const int64_t base = t * kTS;
        src_e = base + re < n ? (int)gather_row(idx, lg, base, re) : -1;
        src_t = wave < 4 && g == 0 && base + rt < n ? (int)gather_row(idx, lg, base, rt) : -1;
    };
    auto fetch = [&] {
        in_v = zero8<V>();
        if (src_e >= 0) in_v = *reinterpret_cast<const V*>(enc + (int64_t)src_e * kEncWidth + 8 * (anew(tid) & 7));
        #pragma unroll
        for (int c = 0; c < 3; ++c) tg[c] = ACT != kActStore && src_t >= 0 ? tgt[(int64_t)src_t * 3 + c] : 0.0f;
    };
    if constexpr (RAWL < 0) {
        find(blockIdx.x);
        fetch();
    }
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const int fresh = anew(lane);
        const bool last = tile + gridDim.x >= n_tiles;       // the sums leave with this tile
        const V* gf = reinterpret_cast<const V*>(ffr) + fresh;
        const V* gb = reinterpret_cast<const V*>(bfr) + fresh;
        // ---- h_0, targets ------------------------------------------------------
        const bool out_wave = wave < 4;                      // holds the outputs of records 16 wave ..
        const int sl = 16 * (wave & 3) + ln;
        const int64_t row = tile * kTS + sl;
        const bool valid = row < n;
        if constexpr (RAWL >= 0) {
            constexpr int RW = RAWL == NRC_RAW14 ? 14 : 16;
            load_frags(gf, 2, rb, lo_f);                     // beside the encoding
            const int64_t src = valid ? gather_row(idx, lg, tile * kTS, sl) : 0;
            if (out_wave && g == 0 && valid) {
                #pragma unroll
                for (int c = 0; c < 3; ++c) tg[c] = tgt[src * 3 + c];
            }
            encode_half<T, PRESET, RAWL>(reinterpret_cast<const float*>(enc) + src * RW, h0 + sl * LD0, row_key<ROOMY>(ln),
                                    wave >> 2, g, valid);
        } else {
            const int ft = anew(tid);
            *reinterpret_cast<V*>(h0 + (ft >> 3) * LD0 + ((8 * (ft & 7)) ^ row_key<ROOMY>(ft >> 3))) = in_v;
            find(tile + gridDim.x);
        }
        f32x4 y = zero;
        if constexpr (ACT == kActLoad) {
            // a thread moves 16 bytes (8 consecutive features: two operand-slot
            // groups of 4) of NR records per layer, a batch of layers' loads in flight
            constexpr int CPR = W / 8, NR = kTS * CPR / NTH;
            const int ft = anew(tid), q = ft % CPR, rec0 = ft / CPR;
            // features 8q .. +3 and +4 .. +7 sit in slots (g', i') and (g' + 1, i')
            const int rq = (8 * q) & 31, gq = (rq & 15) >> 2, iq = rq < 16 ? 0 : 4;
            constexpr int LB = W == 128 ? 2 : MAXH;          // layers per batch of loads
            #pragma unroll
            for (int lb = 0; lb < MAXH; lb += LB) {
                V v[LB][NR];
                #pragma unroll
                for (int u = 0; u < LB; ++u)
                    #pragma unroll
                    for (int k = 0; k < NR; ++k) {
                        const int64_t ar = tile * kTS + rec0 + k * (NTH / CPR);
                        v[u][k] = zero8<V>();
                        if (lb + u < n_hidden && ar < n)
                            v[u][k] = *reinterpret_cast<const V*>(act + (ar * n_hidden + lb + u) * W + 8 * q);
                    }
                #pragma unroll
                for (int u = 0; u < LB; ++u)
                    #pragma unroll
                    for (int k = 0; k < NR; ++k)
                        if (lb + u < n_hidden) {
                            const V x = v[u][k];
                            const int r = rec0 + k * (NTH / CPR), at = 32 * (q >> 2) + 8 * gq + iq;
                            T* dst = hrow(lb + u + 1) + r * LDR;
                            *reinterpret_cast<t4*>(dst + (at ^ row_key<ROOMY>(r))) = __builtin_shufflevector(x, x, 0, 1, 2, 3);
                            *reinterpret_cast<t4*>(dst + ((at + 8) ^ row_key<ROOMY>(r))) =
                                __builtin_shufflevector(x, x, 4, 5, 6, 7);
                        }
            }
            if (out_wave && g == 0 && valid) {
                #pragma unroll
                for (int c = 0; c < 3; ++c) y[c] = act_y[row * 4 + c];
            }
            __syncthreads();
        } else {
            // ---- forward -------------------------------------------------------
            if constexpr (RAWL < 0) load_frags(gf, 2, rb, lo_f);
            __syncthreads();                                 // h_0 is in LDS
            auto layer = [&](const T* in, int stride, auto kc_, int l) {
                constexpr int kc = decltype(kc_)::value;
                f32x4 a[NC];
                V b[KC][NC];
                if (ROOMY) {
                    #pragma unroll
                    for (int c = 0; c < kc; ++c)
                        #pragma unroll
                        for (int col = 0; col < NC; ++col) b[c][col] = get(in, stride, col0 + col, c);
                    reads_first();
                }
                #pragma unroll
                for (int c = 0; c < kc; ++c)
                    #pragma unroll
                    for (int col = 0; col < NC; ++col)
                        a[col] = mm(fr[c], ROOMY ? b[c][col] : get(in, stride, col0 + col, c), c == 0 ? zero : a[col]);
                // the next layer's weights are on their way before the barrier
                if (l + 1 < n_hidden)
                    load_frags(gf + geo.fwd_base(l + 1) * 64, KC, rb, lo_f);
                else if (out_wave)
                    load_frags(gf + geo.fwd_base(n_hidden) * 64, KC, 0, lo_f);
                #pragma unroll
                for (int col = 0; col < NC; ++col) put(hrow(l + 1), col0 + col, a[col], true);
                __syncthreads();                             // h_{l+1} is in LDS
            };
            layer(h0, LD0, IntC<2>{}, 0);
            for (int l = 1; l < n_hidden; ++l) layer(hrow(l), LDR, IntC<KC>{}, l);
            if (out_wave) {
                #pragma unroll
                for (int c = 0; c < KC; ++c) y = mm(fr[c], get(hrow(n_hidden), LDR, wave, c), y);
            }
        }
        if constexpr (ACT == kActStore) {
            fetch();                                         // the next tile's rows
            if (out_wave) {
                float r[3];
                reflectance_operand(get(h0, LD0, wave & 3, 1), fcol, ln, r);
                if (g == 0 && valid) {
                    #pragma unroll
                    for (int c = 0; c < 3; ++c) out[row * 3 + c] = y[c] * r[c];
                    *reinterpret_cast<f32x4*>(act_y + row * 4) = f32x4{y[0], y[1], y[2], 0.0f};
                }
            }
            // 16 bytes (8 consecutive features) of a record's layer per thread
            constexpr int CPR = W / 8;
            const int q = tid % CPR, rq = (8 * q) & 31, gq = (rq & 15) >> 2, iq = rq < 16 ? 0 : 4;
            for (int l = 0; l < n_hidden; ++l)
                #pragma unroll
                for (int rec = tid / CPR; rec < kTS; rec += NTH / CPR) {
                    const int64_t ar = tile * kTS + rec;
                    const T* p = hrow(l + 1) + rec * LDR;
                    const int at = 32 * (q >> 2) + 8 * gq + iq;
                    const t4 a = *reinterpret_cast<const t4*>(p + (at ^ row_key<ROOMY>(rec)));
                    const t4 b = *reinterpret_cast<const t4*>(p + ((at + 8) ^ row_key<ROOMY>(rec)));
                    if (ar < n)
                        *reinterpret_cast<V*>(act + (ar * n_hidden + l) * W + 8 * q) =
                            __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
                }
            __syncthreads();                                 // h_0 .. h_H have been read
            continue;
        }
        // delta_H's weights: K = 32, one fragment per row block
        fr[0] = ld(gb + (geo.bwd_base(n_hidden) + rb) * 64, lo_b);
        if (EARLY) {
            #pragma unroll
            for (int l = MAXH - 1; l >= (GENC ? 0 : 1); --l)
                if (l < n_hidden) {
                    #pragma unroll
                    for (int c = 0; c < KC; ++c)
                        fb[l][c] = ld(gb + (geo.bwd_base(l) + (l ? rb : wave & 3) * KC + c) * 64, lo_b);
                }
        }

        // ---- loss gradient (Eq. 5) in lanes 0 .. 15 of waves 0 .. 3 --------------
        float lterm = 0.0f;
        if (out_wave) {
            float r[3];
            reflectance_operand(get(h0, LD0, wave & 3, 1), fcol, ln, r);
            t4 d = t4{0, 0, 0, 0};
            if (g == 0 && valid) {
                if (UPSTREAM) {
                    d[0] = mul_to<T>(tg[0] * grad_scale, r[0]);
                    d[1] = mul_to<T>(tg[1] * grad_scale, r[1]);
                    d[2] = mul_to<T>(tg[2] * grad_scale, r[2]);
                } else {
                    const float p0 = y[0] * r[0], p1 = y[1] * r[1], p2 = y[2] * r[2];
                    const float lum = (p0 + p1 + p2) * (1.0f / 3.0f);
                    const float inv_den = 1.0f / fmaf(lum, lum, loss_eps);
                    const float e0 = p0 - tg[0];
                    const float e1 = p1 - tg[1];
                    const float e2 = p2 - tg[2];
                    lterm = fmaf(e2, e2, fmaf(e1, e1, e0 * e0)) * inv_den;
                    d[0] = mul_to<T>(2.0f * e0 * inv_den * grad_scale, r[0]);
                    d[1] = mul_to<T>(2.0f * e1 * inv_den * grad_scale, r[1]);
                    d[2] = mul_to<T>(2.0f * e2 * inv_den * grad_scale, r[2]);
                }
            }
            if (g == 0) {
                dO[0 * kLdT + sl] = d[0];
                dO[1 * kLdT + sl] = d[1];
                dO[2 * kLdT + sl] = d[2];
                *reinterpret_cast<t4*>(dR + sl * 4) = d;
                if (GENC) *reinterpret_cast<f32x4*>(fy + sl * 4) = y;
            }
        }
        __syncthreads();                                     // dL/dy is in LDS
        if constexpr (RAWL < 0) fetch();                     // the next tile's rows and targets

        // ---- data backward and weight gradients --------------------------------
        // h_l where this wave's delta_l goes, and delta_l masked by ReLU'(z_l) into its
        // row store
        auto h_at = [&](int l, int col) {
            return *reinterpret_cast<const t4*>(hrow(l) + (16 * (col0 + col) + ln) * LDR +
                                                ((32 * (rb >> 1) + 8 * g + 4 * (rb & 1)) ^ row_key<ROOMY>(ln)));
        };
        auto put_delta = [&](int l, const f32x4 (&a)[NC], const t4 (&h)[NC]) {
            #pragma unroll
            for (int col = 0; col < NC; ++col) {
                const t4 hv = ROOMY ? h[col] : h_at(l, col);
                f32x4 v;
                #pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = (float)hv[j] > 0.0f ? a[col][j] : 0.0f;
                put(drow(l), col0 + col, v, false);
            }
        };
        {
            f32x4 a[NC];
            t4 hv[NC];
            V ho[2], dv[2];
            auto out_operands = [&](int kc) {
                dv[kc] = ln < kNOut ? *reinterpret_cast<const V*>(dO + ln * kLdT + 32 * kc + 8 * g) : zero8<V>();
                ho[kc] = gather(hrow(n_hidden), LDR, wave, kc);
            };
            #pragma unroll
            for (int col = 0; col < NC; ++col) {
                V bd = zero8<V>();
                const t4 d = *reinterpret_cast<const t4*>(dR + (16 * (col0 + col) + ln) * 4);
                if (g == 0) { bd[0] = d[0]; bd[1] = d[1]; bd[2] = d[2]; }
                a[col] = mm(fr[0], bd, zero);
                if (ROOMY) hv[col] = h_at(n_hidden, col);
            }
            if (ROOMY && wave < MB) {
                out_operands(0);
                out_operands(1);
            }
            if (!EARLY) {
                if (n_hidden > 1)
                    load_frags(gb + geo.bwd_base(n_hidden - 1) * 64, KC, rb, lo_b);
                else if (GENC)
                    load_frags(gb, KC, wave & 3, lo_b);
            }
            put_delta(n_hidden, a, hv);
            if (wave < MB) {
                #pragma unroll
                for (int kc = 0; kc < 2; ++kc) {
                    if (!ROOMY) out_operands(kc);
                    acco = mfma(dv[kc], ho[kc], acco);
                }
                if (last && g == 0) {
                    const int f = 32 * (wave >> 1) + 16 * ((ln >> 2) & 1) + 4 * (2 * (wave & 1) + (ln >> 3)) + (ln & 3);
                    #pragma unroll
                    for (int j = 0; j < kNOut; ++j) {
                        part[geo.w_off(n_hidden) + j * W + f] = acco[j];
                        bad = fmaf(acco[j], 0.0f, bad);
                    }
                }
            }
        }
        __syncthreads();                                     // delta_H is in LDS
        #pragma unroll
        for (int l = MAXH - 1; l >= 1; --l) {
            if (l < n_hidden) {
                f32x4 a[NC];
                t4 hv[NC];
                V dv[KC][NC], bw[2][NW], aw[2][MW];
                auto operands = [&](int kc) {
                    #pragma unroll
                    for (int j = 0; j < NW; ++j) bw[kc][j] = gather(hrow(l), LDR, nw0 + j, kc);
                    #pragma unroll
                    for (int i = 0; i < MW; ++i) aw[kc][i] = gather(drow(l + 1), LDR, mw0 + i, kc);
                };
                if (ROOMY) {
                    #pragma unroll
                    for (int c = 0; c < KC; ++c)
                        #pragma unroll
                        for (int col = 0; col < NC; ++col) dv[c][col] = get(drow(l + 1), LDR, col0 + col, c);
                    #pragma unroll
                    for (int col = 0; col < NC; ++col) hv[col] = h_at(l, col);
                    operands(0);
                    operands(1);
                    reads_first();
                }
                #pragma unroll
                for (int c = 0; c < KC; ++c)
                    #pragma unroll
                    for (int col = 0; col < NC; ++col)
                        a[col] = mm(EARLY ? fb[l][c] : fr[c], ROOMY ? dv[c][col] : get(drow(l + 1), LDR, col0 + col, c),
                                    c == 0 ? zero : a[col]);
                if (!EARLY) {
                    if (l > 1)
                        load_frags(gb + geo.bwd_base(l - 1) * 64, KC, rb, lo_b);
                    else if (GENC)
                        load_frags(gb, KC, wave & 3, lo_b);
                }
                put_delta(l, a, hv);
                #pragma unroll
                for (int kc = 0; kc < 2; ++kc) {
                    if (!ROOMY) operands(kc);
                    #pragma unroll
                    for (int i = 0; i < MW; ++i)
                        #pragma unroll
                        for (int j = 0; j < NW; ++j) accw[l - 1][i][j] = mfma(aw[kc][i], bw[kc][j], accw[l - 1][i][j]);
                }
                if (last) flush_layer(l);
                __syncthreads();                             // delta_l is in LDS, delta_{l+1} has been read
            }
        }
        if constexpr (GENC) {
            // dL/dh_0 = W_0^T delta_1, row block wave & 3 of two columns, with the
            // loss scale of the upstream gradient divided out
            const int rg = wave & 3, cg = 2 * (wave >> 2);
            const int fl = anew(lane), fg = fl >> 4, fn = fl & 15;
            const float inv_scale = 1.0f / grad_scale;
            f32x4 a[2];
            #pragma unroll
            for (int c = 0; c < KC; ++c)
                #pragma unroll
                for (int col = 0; col < 2; ++col)
                    a[col] = mm(EARLY ? fb[0][c] : fr[c], get(drow(1), LDR, cg + col, c), c == 0 ? zero : a[col]);
            #pragma unroll
            for (int col = 0; col < 2; ++col) {
                const int rec = 16 * (cg + col) + fn;
                const int64_t gr = tile * kTS + rec;
                #pragma unroll
                for (int j = 0; j < 4; ++j) a[col][j] *= inv_scale;
                if (gr < n) {
                    if (fcol) {
                        // d(f_c R_c)/d(albedo column) = f_c
                        #pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            int c = 16 * rg + 4 * fg + j - fcol;
                            if (c >= 0 && c < 6) {
                                c = c >= 3 ? c - 3 : c;
                                a[col][j] = fmaf(tgt[gr * 3 + c], fy[rec * 4 + c], a[col][j]);
                            }
                        }
                    }
                    *reinterpret_cast<float4*>(out + gr * kEncWidth + 16 * rg + 4 * fg) =
                        make_float4(a[col][0], a[col][1], a[col][2], a[col][3]);
                }
            }
        }
        {
            V bw[2], aw[2][MW];
            auto operands = [&](int kc) {
                bw[kc] = gather(h0, LD0, wave & 3, kc);
                #pragma unroll
                for (int i = 0; i < MW; ++i) aw[kc][i] = gather(drow(1), LDR, mw0 + i, kc);
            };
            if (ROOMY) {
                operands(0);
                operands(1);
                reads_first();
            }
            #pragma unroll
            for (int kc = 0; kc < 2; ++kc) {
                if (!ROOMY) operands(kc);
                #pragma unroll
                for (int i = 0; i < MW; ++i) acc0[i] = mfma(aw[kc][i], bw[kc], acc0[i]);
            }
        }
        if (last) {
            #pragma unroll
            for (int i = 0; i < MW; ++i) flush(0, mw0 + i, wave & 3, acc0[i]);
        }
        if (!UPSTREAM && out_wave) {
            const float wl = wave_sum_compensated<16>(lterm);
            if (lane == 0) wsum[wave] = wl;
        }
        __syncthreads();                                     // h_0 and delta_1 have been read
        if (!UPSTREAM && tid == NTH - 1) {
            // compensated combine of the waves' sums, in wave order
            float t = 0.0f, c = 0.0f;
            for (int w = 0; w < 4; ++w) {
                const float x = wsum[w], u = t + x;
                c += fabsf(t) >= fabsf(x) ? (t - u) + x : (x - u) + t;
                t = u;
            }
            loss_part[tile] = t + c;
        }
    }

    if constexpr (ACT == kActStore) return;
    const int any_bad = __syncthreads_or(bad != 0.0f ? 1 : 0);
    if (tid == 0 && part_bad) part_bad[blockIdx.x] = any_bad ? 1 : 0;
}

// Workgroups of a launch.  Two fit a CU at width 64 up to depth 5 (at width 128 a wave
// takes 256 registers and one fills the CU; with two, a step of 65,536 FP16 records took
// 25.4 instead of 21.9 us at depth 1, 41.4 instead of 33.0 at depth 2), but up to three
// tiles per CU one is better: the second partial per CU costs the reduction more than
// the overlap saves (us per step, one / two per CU: FP16 32,768 records 21.1 / 23.3,
// 49,152 25.8 / 25.2, 65,536 30.9 / 28.8, 98,304 40.9 / 35.6; BF16 32,768 21.9 / 25.1,
// 49,152 27.1 / 28.1, 65,536 32.4 / 31.7).
int64_t train_wgs(const Geo& d, int64_t n) {
    const int64_t tiles = (n + kTS - 1) / kTS, cus = device_cu_count();
    const bool two = d.W == 64 && d.H <= 5 && tiles > 3 * cus;
    const int64_t wgs = two ? 2 * cus : cus;
    return tiles < wgs ? tiles : wgs;
}

template <typename T, int W, int MAXH, int WGS, bool UP, bool GE, int ACT, int RAWL, int PRESET>
hipError_t tiles_launch_as(const Geo& d, int64_t wgs, const void* ffr, const void* bfr, const void* enc,
                           const float* tgt, const int32_t* idx, int64_t n, float loss_eps, float grad_scale,
                           float* partials, float* loss_part, int32_t* part_bad, float* out, hipStream_t s, void* act,
                           float* act_y, LcgGather lg) {
    const size_t lds = (size_t)tiles_lds_bytes(W, d.H, roomy(W, WGS));
    auto k = k_train_tiles<T, W, MAXH, WGS, UP, GE, ACT, RAWL, PRESET>;
    (void)hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    // the forward-only form keeps no sums: one launch
    const int64_t span = ACT == kActStore ? n : wgs * kHeld * kTS;
    const bool gathered = idx || lg.mask;
    for (int64_t at = 0, part = 0; at < n; at += span, part += wgs) {
        const int64_t cnt = n - at < span ? n - at : span, tiles = (cnt + kTS - 1) / kTS;
        const int64_t row = gathered ? 0 : at;               // the launch's first record
        const LcgGather l{lg.step, apply(power(lg.step, (uint64_t)at), lg.x0) & lg.mask, lg.mask};
        const void* e = RAWL >= 0 ? (const void*)((const float*)enc + row * (RAWL == NRC_RAW14 ? 14 : 16))
                                  : (const void*)((const T*)enc + row * kEncWidth);
        hipLaunchKernelGGL(k, dim3((unsigned)(tiles < wgs ? tiles : wgs)), dim3(64 * kWaves), lds, s, (const T*)ffr,
                           (const T*)bfr, (const T*)e, tgt ? tgt + row * 3 : nullptr, idx ? idx + at : nullptr, cnt, d.H,
                           loss_eps, grad_scale, partials ? partials + part * d.n_params() : nullptr,
                           loss_part ? loss_part + at / kTS : nullptr, part_bad ? part_bad + part : nullptr,
                           out ? out + at * (GE ? kEncWidth : kNOut) : nullptr, d.F,
                           act ? (T*)act + at * d.H * d.W : nullptr, act_y ? act_y + at * 4 : nullptr, l);
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

template <typename T, int W, int MAXH, bool UP, bool GE, int ACT, int RAWL, int PRESET>
hipError_t tiles_launch(const Geo& d, const void* ffr, const void* bfr, const void* enc, const float* tgt,
                        const int32_t* idx, int64_t n, float loss_eps, float grad_scale, float* partials,
                        float* loss_part, int32_t* part_bad, float* out, hipStream_t s, void* act, float* act_y,
                        LcgGather lg) {
    const int64_t wgs = train_wgs(d, n);
    if constexpr (W == 64 && MAXH <= 5)
        if (wgs > device_cu_count())
            return tiles_launch_as<T, W, MAXH, 2, UP, GE, ACT, RAWL, PRESET>(d, wgs, ffr, bfr, enc, tgt, idx, n, loss_eps,
                                                                             grad_scale, partials, loss_part,
                                                                             part_bad, out, s, act, act_y, lg);
    return tiles_launch_as<T, W, MAXH, 1, UP, GE, ACT, RAWL, PRESET>(d, wgs, ffr, bfr, enc, tgt, idx, n, loss_eps,
                                                                     grad_scale, partials, loss_part, part_bad, out,
                                                                     s, act, act_y, lg);
}

template <typename T, int W, int MAXH>
hipError_t tiles_dispatch(const Geo& d, const void* ffr, const void* bfr, const void* enc, const float* tgt,
                          const int32_t* idx, int64_t n, bool upstream, float loss_eps, float grad_scale,
                          float* partials, float* loss_part, int32_t* part_bad, float* genc, hipStream_t s,
                          void* act, float* act_y, LcgGather lg) {
#define NRC_TILES(UP, GE, ACT)                                                                                    \
    return tiles_launch<T, W, MAXH, UP, GE, ACT, -1,  NRC_PRESET_CONFIG>(d, ffr, bfr, enc, tgt, idx, n, loss_eps, \
                                                                         grad_scale, partials, loss_part,         \
                                                                         part_bad, genc, s, act, act_y, lg)
    if (!upstream) NRC_TILES(false, false, kActNone);
    if (act) {
        if (genc) NRC_TILES(true, true, kActLoad);
        NRC_TILES(true, false, kActLoad);
    }
    if (genc) NRC_TILES(true, true, kActNone);
    NRC_TILES(true, false, kActNone);
#undef NRC_TILES
}

template <typename T, int MAXH>
hipError_t tiles_raw_dispatch(const Geo& d, int preset, int layout, const void* ffr, const void* bfr,
                              const float* raw, const float* tgt, const int32_t* idx, int64_t n, float loss_eps,
                              float grad_scale, float* partials, float* loss_part, int32_t* part_bad, hipStream_t s,
                              LcgGather lg) {
#define NRC_TILES(PR)                                                                                            \
    return layout == NRC_RAW14                                                                                   \
               ? tiles_launch<T, 64, MAXH, false, false, kActNone, NRC_RAW14, PR>(d, ffr, bfr, raw, tgt, idx, n,    \
                                                                               loss_eps, grad_scale, partials,   \
                                                                               loss_part, part_bad, nullptr, s,  \
                                                                               nullptr, nullptr, lg)             \
               : tiles_launch<T, 64, MAXH, false, false, kActNone, NRC_RAW16, PR>(d, ffr, bfr, raw, tgt, idx, n,    \
                                                                               loss_eps, grad_scale, partials,   \
                                                                               loss_part, part_bad, nullptr, s,  \
                                                                               nullptr, nullptr, lg)
    if (preset == NRC_PRESET_PAPER_GAUSS) NRC_TILES(NRC_PRESET_PAPER_GAUSS);
    if (preset == NRC_PRESET_PAPER_TRI) NRC_TILES(NRC_PRESET_PAPER_TRI);
    if (preset == NRC_PRESET_PAPER) NRC_TILES(NRC_PRESET_PAPER);
    NRC_TILES(NRC_PRESET_CONFIG);
#undef NRC_TILES
}

}  // namespace

// Everything but the FP16 backward passes of up to one tile per CU at width 64,
// where k_train_mfma's chain in registers is shorter.  us, k_train_mfma / here,
// with the reduction: FP16 backward of 300 records 9.7 / 10.4 from the buffer and
// 10.3 / 11.1 without, of 16,384 17.8 / 18.5 and 19.1 / 19.9; FP16 steps 300 records
// 15.1 / 12.6, 16,384 17.5 / 16.0; BF16 steps 17.9 / 13.4 and 20.9 / 17.0, backward
// without the buffer 13.7 / 12.2 and 22.0 / 20.5.
bool train_in_tiles(int precision, const Geo& d, int64_t n, bool upstream) {
    return !(precision == NRC_FP16 && d.W == 64 && upstream && (n + kTS - 1) / kTS <= device_cu_count());
}

// Partials of a step or backward pass: one for each workgroup of its launches.
int64_t train_parts(const Geo& d, int64_t n) {
    const int64_t tiles = (n + kTS - 1) / kTS, wgs = train_wgs(d, n);
    const int64_t full = (tiles - 1) / (wgs * kHeld), left = tiles - full * wgs * kHeld;
    return full * wgs + (left < wgs ? left : wgs);
}

hipError_t launch_train_tiles(int precision, const Geo& d, const void* ffr, const void* bfr, const void* enc,
                              const float* tgt, const int32_t* idx, int64_t n, bool upstream, float loss_eps,
                              float grad_scale, float* partials, float* loss_part, int32_t* part_bad, float* genc,
                              hipStream_t s, const void* act, const float* act_y, LcgGather lg) {
#define NRC_TILES(T, W, MAXH)                                                                                      \
    return tiles_dispatch<T, W, MAXH>(d, ffr, bfr, enc, tgt, idx, n, upstream, loss_eps, grad_scale, partials,    \
                                      loss_part, part_bad, genc, s, (void*)act, (float*)act_y, lg)
    if (precision == NRC_FP16) {
        if (d.W == 128) NRC_TILES(_Float16, 128, 5);
        if (d.H <= 5) NRC_TILES(_Float16, 64, 5);
        NRC_TILES(_Float16, 64, 8);
    }
    if (d.W == 128) NRC_TILES(__bf16, 128, 5);
    if (d.H <= 5) NRC_TILES(__bf16, 64, 5);
    NRC_TILES(__bf16, 64, 8);
#undef NRC_TILES
}

hipError_t launch_train_tiles_raw(int precision, const Geo& d, int preset, int layout, const void* ffr,
                                  const void* bfr, const float* raw, const float* tgt, const int32_t* idx, int64_t n,
                                  float loss_eps, float grad_scale, float* partials, float* loss_part,
                                  int32_t* part_bad, hipStream_t s, LcgGather lg) {
#define NRC_TILES(T, MAXH)                                                                                      \
    return tiles_raw_dispatch<T, MAXH>(d, preset, layout, ffr, bfr, raw, tgt, idx, n, loss_eps, grad_scale,    \
                                       partials, loss_part, part_bad, s, lg)
    if (precision == NRC_FP16) {
        if (d.H <= 5) NRC_TILES(_Float16, 5);
        NRC_TILES(_Float16, 8);
    }
    if (d.H <= 5) NRC_TILES(__bf16, 5);
    NRC_TILES(__bf16, 8);
#undef NRC_TILES
}

hipError_t launch_fwd_train_tiles_bf16(const Geo& d, const void* ffr, const void* enc, int64_t n, void* act,
                                       float* act_y, float* rgb, hipStream_t s) {
    return tiles_launch<__bf16, 128, 5, true, false, kActStore, -1, NRC_PRESET_CONFIG>(
        d, ffr, nullptr, enc, nullptr, nullptr, n, 0.0f, 1.0f, nullptr, nullptr, nullptr, rgb, s, act, act_y,
        LcgGather{});
}

}  // namespace nrc
