// Weight-streaming GEMM  Y[rows, N] = X[rows, K] * W[N, K]^T  for any row count (the general kernel).
//
// Every linear layer of the verify forward has at most a few dozen activation rows (the
// pending token plus the drafts; paper Sec. 3 and Sec. 4.3), so the step is bound by reading
// each weight byte once from HBM.  The weights are the MFMA A operand, streamed from global
// memory straight into registers as 1 KiB-per-wavefront contiguous fragments; the activations
// are the B operand, staged in LDS once per workgroup and re-used by all its wavefronts.
// Products are accumulated in float32 and written as split-K partial sums [ks][rows][N]; the
// consumer kernels add the partials in a fixed order, which keeps results bit-reproducible.
//
// Unless VF_OPT_FAST_PATH is 0, calls take the kernels of gemm_rows.h instead, whatever their row count;
// which of those shapes, and how far K is split, is worked out below.
#include "gemm_rows.h"

namespace {

constexpr int GEMM_WAVES = 4;
constexpr int PREFETCH = 4;   // weight fragments in flight per stream and wavefront

template <int NB> struct Chunk { static constexpr int KC = (NB <= 2) ? 16 : 8; };


// NB: 16-row activation blocks handled per pass; NBW: weight n-blocks per wavefront.
template <int NB, int NBW>
__global__ __launch_bounds__(GEMM_WAVES * 64) VF_MFMA_KERNEL void gemm_bf16_kernel(
    const u32x4 *__restrict__ Wp, const u32x4 *__restrict__ Xp, float *__restrict__ part, int N,
    int KB, int ncb, int row_lo, int row_hi, int ld_rows, int kb_per_split) {
    constexpr int KC = Chunk<NB>::KC;
    __shared__ u32x4 xs[KC * NB * 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int NBt = N >> 4;
    const int cb0 = (row_lo >> 4) + blockIdx.z * NB;
    const int nb0 = (blockIdx.x * GEMM_WAVES + wave) * NBW;
    const int kb_begin = blockIdx.y * kb_per_split;
    const int kb_end = min(KB, kb_begin + kb_per_split);
    const bool active = nb0 < NBt;

    floatx4 acc[NBW][NB];
#pragma unroll
    for (int i = 0; i < NBW; ++i)
#pragma unroll
        for (int c = 0; c < NB; ++c) acc[i][c] = floatx4{0.f, 0.f, 0.f, 0.f};

    const u32x4 *wp[NBW];
#pragma unroll
    for (int i = 0; i < NBW; ++i) {
        int nb = min(nb0 + i, NBt - 1);  // out-of-range streams re-read a valid block, never stored
        wp[i] = Wp + (size_t)nb * KB * 64 + lane;
    }
    u32x4 w[PREFETCH][NBW];
    if (active) {
#pragma unroll
        for (int d = 0; d < PREFETCH; ++d)
            if (kb_begin + d < kb_end)
#pragma unroll
                for (int i = 0; i < NBW; ++i) w[d][i] = load_stream(wp[i] + (size_t)(kb_begin + d) * 64);
    }

    for (int kc = kb_begin; kc < kb_end; kc += KC) {
        const int nk = min(KC, kb_end - kc);
        __syncthreads();
        for (int idx = threadIdx.x; idx < nk * NB * 64; idx += GEMM_WAVES * 64) {
            int l = idx & 63, f = idx >> 6;
            int c = f % NB, kbl = f / NB;
            int cb = cb0 + c;
            u32x4 v = u32x4{0u, 0u, 0u, 0u};
            if (cb < ncb) v = Xp[((size_t)(kc + kbl) * ncb + cb) * 64 + l];
            xs[idx] = v;
        }
        __syncthreads();
        if (!active) continue;
#pragma unroll 1
        for (int k0 = 0; k0 < nk; k0 += PREFETCH) {
#pragma unroll
            for (int d = 0; d < PREFETCH; ++d) {
                const int kbl = k0 + d;
                if (kbl < nk) {
                    bf16x8 a[NBW];
#pragma unroll
                    for (int i = 0; i < NBW; ++i) a[i] = __builtin_bit_cast(bf16x8, w[d][i]);
                    const int nxt = kc + kbl + PREFETCH;
                    if (nxt < kb_end)
#pragma unroll
                        for (int i = 0; i < NBW; ++i) w[d][i] = load_stream(wp[i] + (size_t)nxt * 64);
#pragma unroll
                    for (int c = 0; c < NB; ++c) {
                        bf16x8 b = __builtin_bit_cast(bf16x8, xs[(kbl * NB + c) * 64 + lane]);
#pragma unroll
                        for (int i = 0; i < NBW; ++i)
                            acc[i][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b, acc[i][c], 0, 0, 0);
                    }
                }
            }
        }
    }
    if (!active) return;
    // lane holds Y[row = 16*cb + (lane & 15)][n = 16*nb + 4*(lane >> 4) + 0..3]
    float *out = part + (size_t)blockIdx.y * ld_rows * N;
#pragma unroll
    for (int i = 0; i < NBW; ++i) {
        if (nb0 + i >= NBt) break;
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            int row = (cb0 + c) * 16 + (lane & 15);
            if (row >= row_lo && row < row_hi) {
                float *p = out + (size_t)row * N + (nb0 + i) * 16 + (lane >> 4) * 4;
                *reinterpret_cast<floatx4 *>(p) = acc[i][c];
            }
        }
    }
}

template <int NB>
int launch_bf16(const vf_model *m, const void *W, const void *X, float *part, int N, int K, int ncb,
                int row_lo, int row_hi, int ld_rows, const GemmPlan &plan, hipStream_t st) {
    const int KB = K >> 5, NBt = N >> 4;
    const int kbps = (KB + plan.ks - 1) / plan.ks;
    const int cbs = ((row_hi + 15) >> 4) - (row_lo >> 4);
    dim3 grid((NBt + GEMM_WAVES * plan.nbw - 1) / (GEMM_WAVES * plan.nbw), plan.ks, (cbs + NB - 1) / NB);
    dim3 block(GEMM_WAVES * 64);
    auto args = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, block, 0, st, (const u32x4 *)W, (const u32x4 *)X, part, N, KB, ncb,
                           row_lo, row_hi, ld_rows, kbps);
    };
    switch (plan.nbw) {
        case 1: args(gemm_bf16_kernel<NB, 1>); break;
        case 2: args(gemm_bf16_kernel<NB, 2>); break;
        default: args(gemm_bf16_kernel<NB, 4>); break;
    }
    VF_LAUNCH_CHECK("gemm_bf16");
    return VF_OK;
}


// ---- which kernel, which tile, how many K splits ---------------------------------------
// A call's time on a shape of tile is modelled as
//     start + step * k-blocks per split * rounds of the chip + written * MB + hbm * MB of weights
// (us; rounds: workgroups / 256 rounded up while there are few, fractional beyond) plus the time the
// consumer takes to read the partial sums, and the cheapest (shape, split) is taken.
// Layers: the constants are least-squares fits to the time of a layer of the model with one of its four matrices forced to
// each shape and split (0.5B, 1.5B and 3B shapes, twenty row counts of 16 to 1500), the timings within 15 % of the
// best.  Timed anew (20 row counts of 7 to 1300, and a model 2048 wide), the choice costs a layer 0.4 % on average against the
// best kernel and split, 3.4 % at worst of the three (down of 250 rows at 3B), 5 % of the fourth;
// profiles/layer_gemm_plan_timings.txt.  What decides is visible in them: a
// shape of few weight blocks per tile (stream) wins while its column tiles fill the chip once, the square tiles
// once there are several rounds of them anyway (their step covers more products).  Activations four k-blocks ahead
// serve as well as eight (RK_S16x5, gate/up of 256 rows at 1.5B, a layer 73.3 -> 72.5), twelve and sixteen are no
// better, nor are rings of shorter slots.
// Output heads of WIDE_HEAD columns and more (dozens of rounds of column tiles) have constants of their own: the layers'
// choose badly for them, 104 rows of 0.5B 89 us in RK_S8x5 where RK_T8x8 takes 72.5.  Fitted to the time of the head
// alone (0.5B, 1.5B and 3B and four other widths and vocabularies of 32000 to 262144, up to 60 row counts of 1 to 1500, every
// shape; profiles/output_head_timings.txt); the choice is 0.4 % slower than the best of all shapes on average, 13 % at worst (264
// rows of 0.5B, whose second tile of 256 is nearly empty).  With the top-k epilogue a call's time goes on with the merge of its lists,
// twice as many in RK_T16x8 as in RK_T16x16 (240 rows of 1.5B, top 4: 209 and 221 us the GEMM, 284 and 268 with norm and merge): fitted to
// both, for 1 to 8 candidates; 0.3 % slower than the best on average, 11 % at worst (7 % of the three full-size shapes).
// Heads of 4096 and 16384 columns are like the layers' matrices: 0.8 % with the layers' constants, 55 % at worst with these.
enum RowsKernel { RK_T16x16, RK_T16x8, RK_T8x8, RK_S4x2, RK_S4x4, RK_S4x5, RK_S8x4, RK_S8x5, RK_S16x5, RK_S24x5, RK_S8x3, RK_S16x5W4, RK_COUNT };
constexpr int WIDE_HEAD = 24576;
struct RowsCost { float start, step, written, hbm, again = 0.f; };   // again: a round of the chip, for each candidate after the first
constexpr RowsCost NEVER{0.f, 0.f, 0.f, 0.f};
struct RowsShape {
    int mb, nb;                        // 16-row blocks x weight blocks of a tile
    RowsCost layer;
    bool partial, qkv, swiglu, topk;   // epilogues it is built with: those that rows of the three full-size shapes, or a narrow head's, take
    int lists;                         // top-k candidate lists per tile and row
    RowsCost head, head_topk;          // of wide heads
};
constexpr RowsShape ROWS_SHAPES[RK_COUNT] = {
    // RK_T16x16: square tile, 8 wavefronts of 64 x 128
    {16, 16, {4.99f, 0.4876f, 0.182f, 0.0377f}, true, true, true, true, 2, {5.36f, 0.5984f, 0.211f, 0.0788f}, {10.03f, 0.5180f, 2.491f, 0.0604f, 10.60f}},
    // RK_T16x8: square tile, 8 wavefronts of 64 x 64
    {16, 8, {3.54f, 0.2849f, 0.228f, 0.0505f}, true, true, true, true, 2, {3.99f, 0.3404f, 0.292f, 0.0598f}, {11.13f, 0.3468f, 2.699f, 0.0368f, 4.58f}},
    // RK_T8x8: square tile, 4 wavefronts of 64 x 64
    {8, 8, {3.21f, 0.1769f, 0.183f, 0.0964f}, true, true, true, true, 2, {2.39f, 0.1847f, 0.362f, 0.0873f}, {11.59f, 0.1955f, 1.711f, 0.0521f, 2.34f}},
    // RK_S4x2, RK_S4x4, RK_S4x5: stream, 4 wavefronts of 16 rows
    {4, 2, {2.09f, 0.0571f, 0.325f, 0.0910f}, true, true, false, false, 0, NEVER, NEVER},
    {4, 4, {2.46f, 0.0795f, 0.220f, 0.0868f}, true, true, true, false, 0, {12.95f, 0.0548f, 0.471f, 0.0919f}, NEVER},
    {4, 5, {2.35f, 0.1088f, 0.371f, 0.0626f}, true, false, true, false, 0, NEVER, NEVER},
    // RK_S8x4, RK_S8x5: stream, 8 wavefronts of 16 rows
    {8, 4, {2.47f, 0.1248f, 0.232f, 0.0618f}, true, true, true, false, 0, NEVER, NEVER},
    {8, 5, {2.51f, 0.1477f, 0.277f, 0.0451f}, true, true, true, true, 1, NEVER, {0.f, 0.f, 0.f, 0.f, 2.2f}},
    // RK_S16x5, RK_S24x5: stream, 8 wavefronts of 32 and of 48 rows
    {16, 5, {2.30f, 0.2643f, 0.256f, 0.0094f}, false, false, true, false, 0, NEVER, NEVER},
    {24, 5, {1.20f, 0.3275f, 0.618f, 0.0203f}, false, false, true, false, 0, NEVER, NEVER},
    // RK_S8x3: stream, 8 wavefronts of 16 rows
    {8, 3, {2.59f, 0.1066f, 0.330f, 0.0681f}, false, true, false, false, 0, NEVER, NEVER},
    // RK_S16x5W4: stream, 4 wavefronts of 64 rows
    {16, 5, {2.86f, 0.2717f, 0.214f, 0.0122f}, true, true, false, false, 0, NEVER, NEVER},
};
// ROWS_EPI_*
constexpr bool rows_built(const RowsShape &s, int epi) {
    return epi == ROWS_EPI_PARTIAL ? s.partial : epi == ROWS_EPI_QKV ? s.qkv : epi == ROWS_EPI_SWIGLU ? s.swiglu : s.topk;
}

template <typename Kern> struct Launch { Kern kern; int threads, lds; };
template <typename Kern> Launch(Kern, int, int) -> Launch<Kern>;

// calls fn(Launch) for the kernel of shape `k` with epilogue EPI (only combinations that are built)
template <int EPI, typename F> int with_rows_kernel(int k, F fn) {
#define VF_ROWS_CASE(RK, KERN, THREADS, LDS) \
    case RK:                                 \
        if constexpr (rows_built(ROWS_SHAPES[RK], EPI)) return fn(Launch{KERN, THREADS, LDS}); \
        break;
#define VF_TILE_KERNEL(RK, MB, NB, WM, WN) \
    VF_ROWS_CASE(RK, (gemm_tile_kernel<MB, NB, WM, WN, 4, EPI>), WM * WN * 64, 4 * (MB + NB) * 1024)
#define VF_STREAM_KERNEL(RK, CW, WMB, NB, D, KS, SW) \
    VF_ROWS_CASE(RK, (gemm_stream_kernel<CW, WMB, NB, D, KS, SW, EPI>), (CW + 1) * 64, SW * KS * NB * 1024)
    switch (k) {
        VF_TILE_KERNEL(RK_T16x16, 16, 16, 4, 2)
        VF_TILE_KERNEL(RK_T16x8, 16, 8, 4, 2)
        VF_TILE_KERNEL(RK_T8x8, 8, 8, 2, 2)
        VF_STREAM_KERNEL(RK_S4x2, 4, 1, 2, 8, 4, 9)
        VF_STREAM_KERNEL(RK_S4x4, 4, 1, 4, 8, 4, 5)
        VF_STREAM_KERNEL(RK_S4x5, 4, 1, 5, 8, 4, 5)
        VF_STREAM_KERNEL(RK_S8x4, 8, 1, 4, 8, 4, 5)
        VF_STREAM_KERNEL(RK_S8x5, 8, 1, 5, 4, 4, 5)
        VF_STREAM_KERNEL(RK_S16x5, 8, 2, 5, 4, 4, 5)
        VF_STREAM_KERNEL(RK_S24x5, 8, 3, 5, 4, 4, 5)
        VF_STREAM_KERNEL(RK_S8x3, 8, 1, 3, 8, 4, 5)
        VF_STREAM_KERNEL(RK_S16x5W4, 4, 4, 5, 4, 4, 5)
        default: break;
    }
#undef VF_ROWS_CASE
#undef VF_TILE_KERNEL
#undef VF_STREAM_KERNEL
    return vf_fail(VF_ERR_ARG, "many-row GEMM: shape %d is not built with this epilogue", k);
}

template <int EPI> int allow_lds() {
    for (int k = 0; k < RK_COUNT; ++k) {
        if (!rows_built(ROWS_SHAPES[k], EPI)) continue;
        const int rc = with_rows_kernel<EPI>(k, [&](auto l) -> int {
            VF_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(l.kern), hipFuncAttributeMaxDynamicSharedMemorySize, l.lds));
            return VF_OK;
        });
        if (rc) return rc;
    }
    return VF_OK;
}

template <int EPI> int launch_rows_as(int k, const RowsArgs<EPI> &p, int workgroups, hipStream_t st) {
    return with_rows_kernel<EPI>(k, [&](auto l) -> int {
        hipLaunchKernelGGL(l.kern, dim3(workgroups), dim3(l.threads), l.lds, st, p);
        VF_LAUNCH_CHECK("gemm_rows");
        return VF_OK;
    });
}

int launch_rows(int epi, int k, const RowsGemm &p, int workgroups, hipStream_t st) {
    if (epi == ROWS_EPI_SWIGLU) return launch_rows_as<ROWS_EPI_SWIGLU>(k, p, workgroups, st);
    if (epi == ROWS_EPI_TOPK) return launch_rows_as<ROWS_EPI_TOPK>(k, p, workgroups, st);
    return launch_rows_as<ROWS_EPI_PARTIAL>(k, p, workgroups, st);
}

}  // namespace

int vf_gemm_init() {
    int rc = allow_lds<ROWS_EPI_PARTIAL>();
    if (!rc) rc = allow_lds<ROWS_EPI_SWIGLU>();
    if (!rc) rc = allow_lds<ROWS_EPI_TOPK>();
    if (!rc) rc = allow_lds<ROWS_EPI_QKV>();
    return rc;
}

static int epilogue_of(GemmUse use) {
    return use == GEMM_SWIGLU ? ROWS_EPI_SWIGLU : use == GEMM_TOPK ? ROWS_EPI_TOPK : use == GEMM_QKV ? ROWS_EPI_QKV : ROWS_EPI_PARTIAL;
}

GemmPlan vf_gemm_plan(const vf_model *m, int N, int K, int rows, GemmUse use, int top_k) {
    GemmPlan p{1, 1, -1, GEMM_PARTIAL, 0, nullptr};
    const int NBt = N >> 4, KB = K >> 5;
    if (m->fast_path) {
        const int cbs = (rows + 15) >> 4;
        const bool wide = (use == GEMM_PARTIAL || use == GEMM_TOPK) && N >= WIDE_HEAD;
        float best = 1e30f;
        for (int k = 0; k < RK_COUNT; ++k) {
            const RowsShape &s = ROWS_SHAPES[k];
            const RowsCost &cost = !wide ? s.layer : use == GEMM_TOPK ? s.head_topk : s.head;
            if (cost.step <= 0.f) continue;
            const float mb_w = (float)N * K * 2e-6f;
            // Up to 64 rows the stream kernels read each weight once and past the caches.  A head that the last-level cache (256
            // MB) does not hold, read through it by a square tile, costs the layers of the next pass more than the tile gains:
            // one row of 0.5B, RK_T8x8 44.6 us and RK_S4x4 50.4, a prefill of 51 tokens 840 and 817.
            if (use == GEMM_PARTIAL && cbs <= 4 && mb_w > 256.f && s.lists == 2) continue;
            const int tiles = (NBt + s.nb - 1) / s.nb * ((cbs + s.mb - 1) / s.mb);
            for (int ks : {1, 2, 3, 4, 6, 8, 10, 12, 16}) {
                if (ks > 1 && ((use != GEMM_SPLIT && use != GEMM_QKV) || KB / ks < 4 || (size_t)ks * rows * N > m->part_floats)) break;
                const int nk = (KB + ks - 1) / ks, splits = (KB + nk - 1) / nk, wgs = tiles * splits;
                if (!rows_built(s, splits > 1 ? ROWS_EPI_PARTIAL : epilogue_of(use))) continue;
                const float rounds = wgs <= 768 ? (float)((wgs + 255) / 256) : (float)wgs / 256.f + 0.2f;
                const float mb_out = (use == GEMM_SWIGLU ? 1.f : use == GEMM_TOPK ? 0.5f : 4.f * splits) * rows * N * 1e-6f;
                float t = cost.start + cost.step * nk * rounds + cost.written * mb_out + cost.hbm * mb_w;
                if (use == GEMM_TOPK) {   // the merge reads a row's lists once per candidate
                    const float lists = (NBt + s.nb - 1) / s.nb * s.lists, read = lists * top_k * top_k;
                    t += s.head_topk.again * (top_k - 1) * rounds + 2.38e-3f * read + 1.44e-6f * read * rows;
                }
                if (use == GEMM_SPLIT) t += 0.18f * mb_out;   // the consumer reads the partial sums at about 5 TB/s
                // Unsplit, the QKV epilogue runs in the GEMM, at the end of every wavefront; split, it is a launch of its own, and
                // no call of the full-size shapes gains by that: a layer of 3B, unsplit / the best split, 9 rows 60.6 / 62.5
                // us, 48 65.8 / 68.1, 72 76.9 / 79.2 (a smaller term than this split it there), 128 87.6 / 90.2; of 1.5B 72
                // rows 50.8 / 53.7, of 0.5B 37.3 / 40.0.
                if (use == GEMM_QKV) t += splits == 1 ? 0.f : 5.5f + 0.13f * mb_out;
                if (t < best) {
                    best = t;
                    p.shape = k;
                    p.ks = splits;
                }
            }
        }
        p.epi = use == GEMM_SPLIT || (use == GEMM_QKV && p.ks > 1) ? GEMM_PARTIAL : use;
        return p;
    }
    const int groups1 = (NBt + GEMM_WAVES - 1) / GEMM_WAVES;
    if (groups1 >= 4096) p.nbw = 4;
    else if (groups1 >= 2048) p.nbw = 2;
    if (use != GEMM_SPLIT && use != GEMM_QKV && use != GEMM_SWIGLU) return p;
    const int groups = (NBt + GEMM_WAVES * p.nbw - 1) / (GEMM_WAVES * p.nbw);
    int ks = 1;
    while (groups * ks < 256 && KB / (ks * 2) >= 4) ks *= 2;
    // the partial buffer must hold ks * ld_rows * N floats
    while (ks > 1 && (size_t)ks * m->cfg.max_rows * N > m->part_floats) ks /= 2;
    p.ks = ks;
    return p;
}

bool vf_gemm_built(int shape, GemmUse epi) { return shape >= 0 && shape < RK_COUNT && rows_built(ROWS_SHAPES[shape], epilogue_of(epi)); }

int vf_gemm_topk_lists(const GemmPlan &p, int N) {
    const RowsShape &s = ROWS_SHAPES[p.shape];
    return ((N >> 4) + s.nb - 1) / s.nb * s.lists;
}

static RowsGemm rows_gemm(const RowsShape &s, const void *W, const void *X, float *out, int N, int K, int ncb, int row_lo, int row_hi,
                          int ld_rows, int ks) {
    RowsGemm p;
    memset(&p, 0, sizeof p);
    p.W = (const u32x4 *)W;
    p.X = (const u32x4 *)X;
    p.out = out;
    p.N = N;
    p.KB = K >> 5;
    p.ncb = ncb;
    p.row_lo = row_lo;
    p.row_hi = row_hi;
    p.ld_rows = ld_rows;
    p.kb_per_split = (p.KB + ks - 1) / ks;
    p.nx = ((N >> 4) + s.nb - 1) / s.nb;
    p.ny = (((row_hi + 15) >> 4) - (row_lo >> 4) + s.mb - 1) / s.mb;
    return p;
}

int vf_launch_gemm_qkv(const vf_model *m, const void *W, const void *X, int N, int K, int rows, int layer, const GemmPlan &plan,
                       hipStream_t st) {
    QkvColumns e = vf_qkv_columns(m, layer);
    e.cosv = m->row_cos;
    e.sinv = m->row_sin;
    if (plan.epi != GEMM_QKV || plan.ks != 1 || N != (e.hq + 2 * e.hkv) * e.hd) return vf_fail(VF_ERR_ARG, "QKV GEMM: not its plan");
    RowsGemmQkv p{rows_gemm(ROWS_SHAPES[plan.shape], W, X, nullptr, N, K, (rows + 15) >> 4, 0, rows, rows, 1), e, m->row_place};
    return launch_rows_as<ROWS_EPI_QKV>(plan.shape, p, p.nx * p.ny, st);
}

int vf_launch_gemm(const vf_model *m, const void *W, const void *X, float *out, int N, int K,
                   int rows_total, int row_lo, int row_hi, int ld_rows, const GemmPlan &plan, hipStream_t st) {
    if (row_hi <= row_lo) return VF_OK;
    const int ncb = (rows_total + 15) >> 4;
    const int cbs = ((row_hi + 15) >> 4) - (row_lo >> 4);
    if (plan.shape >= 0) {
        const RowsShape &s = ROWS_SHAPES[plan.shape];
        if (plan.epi == GEMM_TOPK && (plan.topk < 1 || plan.topk > VF_TOPK_MAX || !plan.topk_ids))
            return vf_fail(VF_ERR_ARG, "top-k epilogue: k %d", plan.topk);
        RowsGemm p = rows_gemm(s, W, X, out, N, K, ncb, row_lo, row_hi, ld_rows, plan.ks);
        p.cand_i = plan.topk_ids;
        p.topk = plan.topk;
        const int epi = plan.epi == GEMM_SWIGLU ? ROWS_EPI_SWIGLU : plan.epi == GEMM_TOPK ? ROWS_EPI_TOPK : ROWS_EPI_PARTIAL;
        return launch_rows(epi, plan.shape, p, p.nx * p.ny * plan.ks, st);
    }
    if (plan.epi == GEMM_TOPK) return vf_fail(VF_ERR_ARG, "top-k epilogue: no many-row kernel");
    if (cbs <= 1) return launch_bf16<1>(m, W, X, out, N, K, ncb, row_lo, row_hi, ld_rows, plan, st);
    if (cbs == 2) return launch_bf16<2>(m, W, X, out, N, K, ncb, row_lo, row_hi, ld_rows, plan, st);
    if (cbs == 3) return launch_bf16<3>(m, W, X, out, N, K, ncb, row_lo, row_hi, ld_rows, plan, st);
    return launch_bf16<4>(m, W, X, out, N, K, ncb, row_lo, row_hi, ld_rows, plan, st);
}
