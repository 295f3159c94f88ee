// The decoder layers of a call whose rows do not fit LDS whole, as the staging of fused.hip needs them, as one persistent
// kernel.  Same structure and memory protocol; the phases are
//   embed | per layer: norm, QKV, attention, O, norm, gate/up, down
// The normalised rows go through memory as MFMA fragments, written once by the norm phases, and every GEMM phase
// reads both operands in operand order straight into registers: no staging in LDS, no limit on the rows from it, no
// K split for its sake.  A norm phase costs a barrier and a round trip (3.8 and 5.0 us a layer at 33 rows of 3072
// columns); staging costs every workgroup the loads and conversions of all its rows (there 8 us twice a layer, and K
// splits that meet in memory on top).
// The output head is the many-row path's.
#include "fused_core.h"

namespace {

// A GEMM phase's items: (unit of UB weight blocks) x (K split), all rows of the call, dealt to the workgroups in turn.
struct DirectGemm {
    global_w_ptr W;
    const bf16_t *X;     // [K / 32][NBW] fragments
    int N, KB, m;
    int units, ks, kbps;
    // epilogues
    FastGemm e;          // QKV: bias, angles, q, layer; SwiGLU: a_out; residual: h_in, h
    float *xch;
    unsigned *fail;
};

// NBW: row blocks of the call.
// What bounds a phase of some 30 to 48 rows is the operand fragments through the vector cache (64 bytes a cycle and
// compute unit), then HBM: per k-block a wavefront loads UB + NBW fragments for UB * NBW products, so tiles are as
// square as the accumulators allow.  The eight wavefronts of a workgroup share the K slice and nothing else; weights
// are requested PW k-blocks ahead, the first of them before the grid barrier, activations PX ahead (from the L2).
template <int HD, int NBW, int UB, int PW, int PX, int EPI>
__device__ __forceinline__ XchUsed direct_phase(const DirectGemm &g, GridBar &bar, unsigned char *smem, const FusedShared &sh TRACE_ARG) {
    static_assert(PW % PX == 0 && (EPI != EPI_SWIGLU || UB % 2 == 0), "rings and pairs");
    constexpr int NTILE = UB * NBW;                                   // partial tiles of an item
    constexpr int NOUT = EPI == EPI_SWIGLU ? NTILE / 2 : NTILE;      // tiles with an epilogue
    constexpr int TPW = (NOUT + FW - 1) / FW;                         // of which a wavefront finishes so many
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = gridDim.x, wg = blockIdx.x, KB = g.KB, NBt = g.N >> 4;
    const int items = g.units * g.ks;
    // K splits only where every workgroup has one item at most
    const int split = g.ks > 1 ? wg % g.ks : 0, first = g.ks > 1 ? wg / g.ks : wg;
    const int n_my = wg < items ? (g.ks > 1 ? 1 : (items - wg + G - 1) / G) : 0;
    const int kb0 = split * g.kbps, kb1 = min(KB, kb0 + g.kbps);
    const int cnt = (kb1 - kb0 + FW - 1) / FW, rounds = (cnt + PW - 1) / PW;
    const int wk0 = kb0 + wave * cnt, mine = min(cnt, kb1 - wk0);   // k-blocks wk0 .. wk0 + mine - 1 (none: mine <= 0)
    floatx4 *red = reinterpret_cast<floatx4 *>(smem);
    const XchUsed used{(unsigned)(first * g.ks * NTILE) * 1024, NTILE * 1024, n_my > 0 && g.ks > 1 ? g.ks : 0, split, NTILE};

    u32x4 w[PW][UB], x[PX][NBW];
#pragma unroll
    for (int d = 0; d < PW; ++d)
#pragma unroll
        for (int u = 0; u < UB; ++u) w[d][u] = u32x4{0u, 0u, 0u, 0u};
    // never predicated: a step past the end of the run loads the run's last fragment again and is skipped
    auto load_w = [&](int unit, int d, int kbl) {
        const int kb = min(wk0 + min(kbl, cnt - 1), kb1 - 1);
#pragma unroll
        for (int u = 0; u < UB; ++u)
            w[d][u] = __builtin_nontemporal_load(g.W + ((size_t)min(unit * UB + u, NBt - 1) * KB + kb) * 64 + lane);
    };
    auto load_x = [&](int r0, int d, int kbl) {
        const int kb = min(wk0 + min(kbl, cnt - 1), kb1 - 1);
#pragma unroll
        for (int c = 0; c < NBW; ++c) x[d][c] = ssa_load_16(g.X + ((size_t)(kb * NBW + r0 + c) * 64 + lane) * 8);
    };
    // this wavefront's tiles of an item: t = wave + 8 i; weight block t / NBW of the unit (SwiGLU: pair), row block t % NBW
    EpiPre pre[TPW];
#pragma unroll
    for (int i = 0; i < TPW; ++i) pre[i].v = pre[i].bias = floatx4{0.f, 0.f, 0.f, 0.f};
    auto ask = [&](int unit, int row0) {
        if (EPI == EPI_SWIGLU) return;
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
            const int t = min(wave + i * FW, NOUT - 1), nb = min(unit * UB + t / NBW, NBt - 1);
            const int row = min(row0 + t % NBW * 16 + (lane & 15), g.m - 1);
            if (EPI == EPI_QKV) pre[i] = epi_qkv_ask<HD>(g.e, sh, row, nb, lane);
            else pre[i].v = ssa_load_f4(g.e.h_in + (size_t)row * g.N + nb * 16 + (lane >> 4) * 4);
        }
    };
    if (n_my > 0) {
#pragma unroll
        for (int d = 0; d < PW; ++d) load_w(first, d, d);
        ask(first, 0);
    }
    TRACE(1);
    bar.wait();
    TRACE(2);
    if (n_my <= 0) return used;
#pragma unroll
    for (int d = 0; d < PX; ++d) load_x(0, d, d);
    for (int it = 0; it < n_my; ++it) {
        const bool has_next = it + 1 < n_my;
        const int unit = first + it * G;
        // 0, which the compiler doesn't know: addresses that depend on it are formed anew for every item.  Held in registers
        // from item to item they spill 43 others (33 rows of 3B 2251 -> 2396 us).
        int row0 = 0;
        asm volatile("" : "+s"(row0));
        floatx4 acc[UB][NBW];
#pragma unroll
        for (int u = 0; u < UB; ++u)
#pragma unroll
            for (int c = 0; c < NBW; ++c) acc[u][c] = floatx4{0.f, 0.f, 0.f, 0.f};
        auto round_body = [&](auto refill_tag, int r) {
            constexpr bool REFILL = decltype(refill_tag)::value;   // false: the last round of the last item
            const bool last_round = r + 1 == rounds;
#pragma unroll
            for (int d = 0; d < PW; ++d) {
                if (r * PW + d < mine) {
#pragma unroll
                    for (int c = 0; c < NBW; ++c)
#pragma unroll
                        for (int u = 0; u < UB; ++u)
                            acc[u][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[d][u]),
                                                                                __builtin_bit_cast(bf16x8, x[d % PX][c]), acc[u][c], 0, 0, 0);
                }
                // the slot's next k-block: of this round, the next one, or the next item's first
                if (d + PX < PW) load_x(row0, d % PX, r * PW + d + PX);
                else if (REFILL) load_x(row0, d % PX, last_round ? d + PX - PW : r * PW + d + PX);
                if (REFILL) load_w(last_round ? unit + G : unit, d, last_round ? d : (r + 1) * PW + d);
            }
        };
#pragma unroll 1
        for (int r = 0; r + 1 < rounds; ++r) round_body(std::true_type{}, r);
        if (has_next) round_body(std::true_type{}, rounds - 1);
        else round_body(std::false_type{}, rounds - 1);
        TRACE(4);
        if (it) lds_sync();   // the previous item's sums have been read
#pragma unroll
        for (int u = 0; u < UB; ++u)
#pragma unroll
            for (int c = 0; c < NBW; ++c) red[((u * NBW + c) * FW + wave) * 64 + lane] = acc[u][c];
        lds_sync();
        floatx4 v[TPW], v1[TPW];
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
            const int t = wave + i * FW;
            if (t < NOUT) {
                if (EPI == EPI_SWIGLU) {   // pair t / NBW: weight blocks 2 p and 2 p + 1
                    const int p = t / NBW, c = t % NBW;
                    v[i] = sum_waves(red, 2 * p * NBW + c, lane);
                    v1[i] = sum_waves(red, (2 * p + 1) * NBW + c, lane);
                } else {
                    v[i] = sum_waves(red, t, lane);
                }
            }
        }
        const unsigned at = (unsigned)(first * g.ks * NTILE) * 1024, stride = NTILE * 1024;
        if (EPI == EPI_RESID && g.ks > 1) {
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
                const int t = wave + i * FW;
                if (t < NOUT && t % g.ks != split) xch_send(g.xch + (at + t * 1024 + split * stride) / 4 + lane * 4, v[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
            const int t = wave + i * FW;
            if (t >= NOUT) continue;
            const int row = row0 + t % NBW * 16 + (lane & 15);
            if (EPI == EPI_SWIGLU) {
                const int nb = unit * UB + t / NBW * 2;
                if (row < g.m && nb < NBt) epi_swiglu_frag(g.e, row, nb, lane, v[i], v1[i], NBW);
            } else if (EPI == EPI_QKV) {
                const int nb = unit * UB + t / NBW;
                if (row < g.m && nb < NBt) epi_qkv_store<HD>(g.e, sh, row, nb, lane, v[i], pre[i]);
            } else if (g.ks == 1 || t % g.ks == split) {
                if (g.ks > 5) v[i] = xch_sum<MAX_DOWN_SPLITS>(v[i], g.xch, at + t * 1024, stride, g.ks, split, lane, g.fail);
                else if (g.ks > 1) v[i] = xch_sum<5>(v[i], g.xch, at + t * 1024, stride, g.ks, split, lane, g.fail);
                const int nb = unit * UB + t / NBW;
                if (row < g.m && nb < NBt) st_f32x4<true>(g.e.h + (size_t)row * g.N + nb * 16 + (lane >> 4) * 4, pre[i].v + v[i]);
            }
        }
        TRACE(5);
        if (has_next) ask(unit + G, row0);
    }
    return used;
}

// x = bf16(h / rms * gain) in operand order, one row a workgroup; eight columns a thread.  The first P passes stay in
// registers between the sum and the products; what a wider row has beyond them is read twice.
__device__ __forceinline__ void norm_phase(const float *h, const float *gain, bf16_t *x, int m, int ncb, int d, float inv_d, float eps, GridBar &bar,
                                           FusedShared &sh TRACE_ARG) {
    constexpr int P = 2;   // passes of 4096 columns
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), row = blockIdx.x, n = d >> 3;
    floatx4 g[P][2], v[P][2];
#pragma unroll
    for (int p = 0; p < P; ++p)
        if (p * FT < n) {
            const int c = min(p * FT + tid, n - 1) * 8;
            g[p][0] = load_global_f4(gain + c);
            g[p][1] = load_global_f4(gain + c + 4);
        }
    TRACE(1);
    bar.wait();
    TRACE(2);
    if (row >= m) return;
    float sq = 0.f;
#pragma unroll
    for (int p = 0; p < P; ++p)
        if (p * FT < n) {
            const int c = min(p * FT + tid, n - 1) * 8;
            v[p][0] = ssa_load_f4(h + (size_t)row * d + c);
            v[p][1] = ssa_load_f4(h + (size_t)row * d + c + 4);
            float s = 0.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) s += v[p][0][j] * v[p][0][j] + v[p][1][j] * v[p][1][j];
            if (p * FT + tid < n) sq += s;
        }
    const float *hrow = h + (size_t)row * d;
    for (int i = P * FT + tid; i < n; i += FT) {
        const floatx4 a = ssa_load_f4(hrow + i * 8), b = ssa_load_f4(hrow + i * 8 + 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) sq += a[j] * a[j] + b[j] * b[j];
    }
#pragma unroll
    for (int o = 32; o; o >>= 1) sq += __shfl_xor(sq, o, 64);
    if (lane == 0) sh.rs_tmp[wave][0] = sq;
    lds_sync();
    float tot = 0.f;
#pragma unroll
    for (int i = 0; i < FW; ++i) tot += sh.rs_tmp[i][0];
    const float r = 1.0f / sqrtf(tot * inv_d + eps);
    auto put = [&](int i, floatx4 a, floatx4 b, floatx4 ga, floatx4 gb) {
        const u32x2 lo = pack4_bf16(a[0] * r * ga[0], a[1] * r * ga[1], a[2] * r * ga[2], a[3] * r * ga[3]);
        const u32x2 hi = pack4_bf16(b[0] * r * gb[0], b[1] * r * gb[1], b[2] * r * gb[2], b[3] * r * gb[3]);
        st_f32x4<true>(reinterpret_cast<float *>(x + xfrag_index(row, i * 8, ncb)), __builtin_bit_cast(floatx4, u32x4{lo[0], lo[1], hi[0], hi[1]}));
    };
#pragma unroll
    for (int p = 0; p < P; ++p)
        if (p * FT + tid < n) put(p * FT + tid, v[p][0], v[p][1], g[p][0], g[p][1]);
    for (int i = P * FT + tid; i < n; i += FT)
        put(i, ssa_load_f4(hrow + i * 8), ssa_load_f4(hrow + i * 8 + 4), load_global_f4(gain + i * 8), load_global_f4(gain + i * 8 + 4));
    // rs_tmp is written again two barriers from here at the earliest
}

template <int NBW, int HD>
__global__ __launch_bounds__(FT, 2) void layers_direct_kernel(FusedArgs a, Batch b) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ FusedShared sh;
    const unsigned start = barrier_start(a.bar_start);
#ifdef FUSED_TRACE
    Trace trace{reinterpret_cast<unsigned long long *>(a.bar + 8192), 0};
#endif
    const int d = a.d, F = a.F, nq = a.hq * HD, nkv = a.hkv * HD;
    const size_t hstride = (size_t)a.frows * d;
    const int len0 = launch_tables(a, b, sh);
    embed_phase(a, b);
    GridBar bar = grid_bar(a.bar, a.fail, __builtin_amdgcn_readfirstlane(start));
    bar.arrive();
    FastGemm base;
    base.m = a.m;
    base.F = F;
    base.cosv = a.cosv;
    base.sinv = a.sinv;
    base.hq = a.hq;
    base.hkv = a.hkv;
    base.hd = HD;

#pragma unroll 1
    for (int l = 0; l < a.n_layers; ++l) {
        const FusedLayer lp = layer_params(a, l);
        float *h0 = a.hv + (size_t)(2 * l) * hstride, *h1 = h0 + hstride, *h2 = l + 1 < a.n_layers ? h1 + hstride : a.h_last;
        bf16_t *q = a.qv + (size_t)l * a.frows * nq, *o = a.ov + (size_t)l * a.frows * nq, *act = a.av + (size_t)l * a.frows * F;
        bf16_t *x0 = a.xv + (size_t)(2 * l) * hstride, *x1 = x0 + hstride;
        norm_phase(h0, lp.attn_norm, x0, a.m, NBW, d, a.inv_d, a.eps, bar, sh TRACE_PASS);
        bar.arrive();
        TRACE(17);
        {
            const int units = (nq + 2 * nkv) / 16;
            DirectGemm g{(global_w_ptr)lp.wqkv, x0, nq + 2 * nkv, d / 32, a.m, units, 1, d / 32, base, a.xch, a.fail};
            g.e.bias = a.has_bias ? lp.bqkv : nullptr;
            g.e.q = q;
            g.e.layer = l;
            if (units <= FUSED_G) {
                direct_phase<HD, NBW, 1, 6, 6, EPI_QKV>(g, bar, smem, sh TRACE_PASS);
            } else {
                g.units = (units + 1) / 2;
                direct_phase<HD, NBW, 2, 6, 3, EPI_QKV>(g, bar, smem, sh TRACE_PASS);
            }
        }
        bar.arrive();
        TRACE(10);
        const XchUsed att_used = attn_phase<HD>(a, b, l, q, o, NBW, len0, bar, smem, sh TRACE_PASS);
        bar.arrive();
        TRACE(13);
        xch_clear<2>(a.xch, att_used);
        {
            DirectGemm g{(global_w_ptr)lp.wo, o, d, nq / 32, a.m, d / 16, 1, nq / 32, base, a.xch, a.fail};
            g.e.h_in = h0;
            g.e.h = h1;
            if (g.units <= FUSED_G) {
                direct_phase<HD, NBW, 1, 6, 6, EPI_RESID>(g, bar, smem, sh TRACE_PASS);
            } else {
                g.units = (g.units + 1) / 2;
                direct_phase<HD, NBW, 2, 6, 3, EPI_RESID>(g, bar, smem, sh TRACE_PASS);
            }
        }
        bar.arrive();
        TRACE(14);
        norm_phase(h1, lp.ffn_norm, x1, a.m, NBW, d, a.inv_d, a.eps, bar, sh TRACE_PASS);
        bar.arrive();
        TRACE(18);
        {
            DirectGemm g{(global_w_ptr)lp.wgu, x1, 2 * F, d / 32, a.m, (F / 8 + 3) / 4, 1, d / 32, base, a.xch, a.fail};
            g.e.a_out = act;
            direct_phase<HD, NBW, 4, 4, 2, EPI_SWIGLU>(g, bar, smem, sh TRACE_PASS);
        }
        bar.arrive();
        TRACE(15);
        XchUsed down_used;
        {
            DirectGemm g{(global_w_ptr)lp.wd, act, d, F / 32, a.m, (d / 16 + a.down_ub - 1) / a.down_ub, a.ks_down,
                         (F / 32 + a.ks_down - 1) / a.ks_down, base, a.xch, a.fail};
            g.e.h_in = h1;
            g.e.h = h2;
            if (a.down_ub == 4) down_used = direct_phase<HD, NBW, 4, 4, 2, EPI_RESID>(g, bar, smem, sh TRACE_PASS);
            else down_used = direct_phase<HD, NBW, 2, 6, 3, EPI_RESID>(g, bar, smem, sh TRACE_PASS);
        }
        bar.arrive();
        TRACE(16);
        xch_clear<1>(a.xch, down_used);
    }
    barrier_advance(a.bar_start, bar);
}

}  // namespace

// K split and weight blocks an item of the down projection: operand fragments through the cache at 154 GB/s a compute
// unit, an exchange at about 1.3 us.
static void plan_down(const vf_config &c, int nbw, FusedArgs &a) {
    const int KB = c.d_ffn / 32;
    float best = 0.f;
    for (int ub = 2; ub <= 4; ub += 2) {
        const int items = (c.d_model / 16 + ub - 1) / ub;
        for (int ks = 1; ks <= MAX_DOWN_SPLITS; ++ks) {
            const int kbps = (KB + ks - 1) / ks;
            if (ks > 1 && (items * ks > FUSED_G || kbps < FW || (KB + kbps - 1) / kbps != ks)) continue;
            const int rounds = (items * ks + FUSED_G - 1) / FUSED_G;
            const float us = rounds * (ub + nbw) * kbps * 6.6e-3f + (ks > 1 ? 1.3f : 0.f);
            if (best == 0.f || us < best) { best = us; a.down_ub = ub; a.ks_down = ks; }
        }
    }
}

// Calls of vf_verify with up to 48 rows (FROWS) that the staging does not take.  More rows get a launch per operation, and
// so does a chunk of a prompt whatever its rows: launches share the GPU with what runs on other streams, another model's
// calls among them, and a persistent kernel needs all of it.
bool vf_direct_ok(const vf_config &c, int rows) { return fused_shape_ok(c) && rows <= FROWS; }

int vf_run_direct(vf_model *m, const Batch &b, const int32_t *tokens, bool tree, hipStream_t st) {
    const vf_config &c = m->cfg;
    if (!vf_direct_ok(c, b.total_rows)) return vf_fail(VF_ERR_UNSUPPORTED, "persistent kernel does not apply to this call");
    FusedArgs a;
    memset(&a, 0, sizeof a);
    fused_args(m, b, tokens, tree, a);
    a.h_last = m->h;
    const int nb = (b.total_rows + 15) / 16;
    plan_down(c, std::max(2, nb), a);   // one row block: timed with the plan of two
    ProfScope ps(m, VF_SITE_STEP, st);
    if (c.head_dim == 128) {
        if (nb == 1) return fused_launch<&layers_direct_kernel<1, 128>>(a, b, st);
        if (nb == 2) return fused_launch<&layers_direct_kernel<2, 128>>(a, b, st);
        return fused_launch<&layers_direct_kernel<3, 128>>(a, b, st);
    }
    if (nb == 1) return fused_launch<&layers_direct_kernel<1, 64>>(a, b, st);
    if (nb == 2) return fused_launch<&layers_direct_kernel<2, 64>>(a, b, st);
    return fused_launch<&layers_direct_kernel<3, 64>>(a, b, st);
}
