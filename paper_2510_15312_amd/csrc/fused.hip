// The whole verify forward pass (paper Sec. 3 / Sec. 4.3: rows [T, x_1..x_k] of every sequence of
// the batch through all decoder layers and the output head) as ONE persistent kernel.
//
// The grid is sized so that every workgroup is resident at once (one workgroup of eight
// wavefronts per CU); the phases of the pass
//   embed | per layer: QKV, attention, O, gate/up, down | output head
// are separated by grid-wide barriers instead of kernel boundaries.  What this buys over a chain
// of kernels: no launch gap and no ramp-up per phase, and the weight stream pauses only for the
// hand-over of the activations -- a workgroup issues the first loads of its next phase (weights
// do not depend on the previous phase) between arriving at a barrier and waiting on it, and
// inside a phase it refills its register ring with the next work item's fragments during the
// current item's last round.
//
// Memory protocol between workgroups (different compute dies have separate L2 caches):
//   * everything one workgroup writes and another reads later in the launch is stored through
//     to memory (agent-scope stores), and a workgroup waits until its stores have completed
//     before it arrives at a barrier (partial tiles in the exchange are their own signal);
//   * bulk data is read with ordinary loads from single-assignment buffers -- one version of
//     the residual stream per half layer, one q / attention output / SwiGLU buffer per
//     layer -- so no cache can hold a stale line of it: a line is never read before its only
//     write in a launch, and caches start clean at every launch;
//   * data in reused buffers (the exchange of partial tiles, the barrier's counters) is read with agent-scope loads.
// The KV cache is written (new rows) and read (all rows) once per layer and launch, in that
// order; tiles that hold new rows are read with agent-scope loads.
//
// Results do not depend on timing: every sum has a fixed order.
#include "fused_core.h"

namespace {

#ifndef FUSED_BB_AHEAD
#define FUSED_BB_AHEAD 1          // GEMM phases: activation fragments are read from LDS this many steps ahead of their MFMAs (0: right before)
#endif
#ifndef FUSED_SGB
#define FUSED_SGB 1               // GEMM phases: LDS reads are scheduled this many steps ahead of their MFMAs (0: left to the compiler)
#endif

// Staging of a normalising phase: x = bf16(h * rstd * gain) of all rows, to LDS as [k-block][row][32].
// What bounds it is instruction issue: two wavefronts a SIMD, every instruction of a piece (four columns of a row per
// lane) at four to five cycles.  So a wavefront takes whole rows, w, w + 8, ...: its columns are the same in every row,
// and gain, load and LDS offsets stay in registers, worked out before the grid barrier; what is left of a piece is
// its load, eight products, two conversions, an addition and its write.  Two rows are in flight per wavefront, and
// none is loaded that is not needed: with few rows the loads themselves (16 cycles each in the vector cache) were
// most of it.  Release to staged, 1 row of 0.5B: 3.0 us with pieces dealt to threads in turn and 16 loads a thread,
// 1.7 with pieces dealt to wavefronts and as many loads as a call needs, 1.1 so; 17 rows of 1.5B 3.2, 3.0, 2.2 us.
// 1/rms from the producer's sums of squares per 16 columns: wavefront w adds blocks w, w + 8, ... of row `lane`
// (one contiguous load a block), the eight sums meet in LDS, and every wavefront adds them up for itself.
// pieces of a row in one pass: rows of up to 1024 columns with heads of 64, 1536 with heads of 128
constexpr int JP_OF(int hd) { return hd == 64 ? 4 : 6; }
template <int JP> struct NormStage {
    static constexpr int TS = 12;   // sums of squares requested ahead of the rows
    floatx4 gain[JP];
    unsigned off[JP], out[JP];      // bytes: of the lane's piece j in a row, and in the staged k-blocks (row 0)
    const float *h, *gain_p, *ss;
    int K, n_ss, m, chunks;
    float inv_d, eps;

    // columns of pieces seg * 64 JP ..: a row of more than 64 JP pieces takes several passes over the rows
    __device__ __forceinline__ void columns(int seg, int lane) {
#pragma unroll
        for (int j = 0; j < JP; ++j) {
            const int c = min((seg * JP + j) * 64 + lane, chunks - 1);   // past the end: the last piece, written again
            off[j] = c * 16;
            out[j] = (c >> 3) * m * 64 + (c & 7) * 8;
            gain[j] = load_global_f4(gain_p + c * 4);
        }
    }
    // before the barrier
    __device__ __forceinline__ void init(const FastGemm &g, int lane) {
        h = g.Xh;
        gain_p = g.gain;
        ss = g.ss_in;
        K = g.KB * 32;
        n_ss = g.n_ss;
        m = g.m;
        chunks = g.KB * 8;
        inv_d = g.inv_d;
        eps = g.eps;
        columns(0, lane);
    }
    __device__ __forceinline__ void load(floatx4 (&v)[JP], int row) const {
        const char *src = reinterpret_cast<const char *>(h + (size_t)row * K);   // the same for all lanes
#pragma unroll
        for (int j = 0; j < JP; ++j) v[j] = ssa_load_f4(reinterpret_cast<const float *>(src + off[j]));
        asm volatile("" ::: "memory");
    }
    __device__ __forceinline__ void put(const floatx4 (&v)[JP], int row, float rs, unsigned char *xs) const {
        const float r = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, rs), row));
#pragma unroll
        for (int j = 0; j < JP; ++j) {
            const floatx4 x = v[j], gv = gain[j];
            *reinterpret_cast<u32x2 *>(xs + (out[j] + row * 64)) = pack4_bf16(x[0] * r * gv[0], x[1] * r * gv[1], x[2] * r * gv[2], x[3] * r * gv[3]);
        }
    }
    __device__ __forceinline__ void ask(float (&t)[TS], int lane, int wave) const {
        const float *p = ss + min(lane, m - 1);
#pragma unroll
        for (int i = 0; i < TS; ++i) t[i] = ssa_load_f1(p + min(wave + i * FW, n_ss - 1) * 64);   // the block is the same for all lanes
        asm volatile("" ::: "memory");   // all of them before the first is used
    }
    // 1/rms of row `lane`; a workgroup barrier inside
    __device__ __forceinline__ float rms(const float (&t)[TS], FusedShared &sh, int lane, int wave) const {
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < TS; ++i) sum += t[i] * (wave + i * FW < n_ss ? 1.f : 0.f);
        for (int b = wave + TS * FW; b < n_ss; b += 4 * FW) {
            float r[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) r[i] = ssa_load_f1(ss + min(b + i * FW, n_ss - 1) * 64 + min(lane, m - 1)) * (b + i * FW < n_ss ? 1.f : 0.f);
#pragma unroll
            for (int i = 0; i < 4; ++i) sum += r[i];
        }
        sh.rs_tmp[wave][lane] = sum;
        lds_sync();
        float part[FW], tot = 0.f;
#pragma unroll
        for (int i = 0; i < FW; ++i) part[i] = sh.rs_tmp[i][lane];
        asm volatile("" ::: "memory");  // the eight reads are issued together
#pragma unroll
        for (int i = 0; i < FW; ++i) tot += part[i];
        return 1.0f / sqrtf(tot * inv_d + eps);
    }
    // Rows wave, wave + 8, ... from the k-th on, n of them, rows k and k + 1 in flight in a and b.  The branches are
    // the same for all lanes, and every path waits only for what it uses next.
    __device__ __forceinline__ void rows(floatx4 (&a)[JP], floatx4 (&b)[JP], int n, float rs, unsigned char *xs, int wave) const {
        for (int k = 0;; k += 2) {
            put(a, wave + k * FW, rs, xs);
            if (k + 2 >= n) {
                put(b, wave + (k + 1) * FW, rs, xs);
                return;
            }
            load(a, wave + (k + 2) * FW);
            put(b, wave + (k + 1) * FW, rs, xs);
            if (k + 3 >= n) {
                put(a, wave + (k + 2) * FW, rs, xs);
                return;
            }
            load(b, wave + (k + 3) * FW);
        }
    }
    // behind the barrier
    __device__ __forceinline__ void run(unsigned char *xs, FusedShared &sh, int lane, int wave TRACE_ARG) {
        const int n = m > wave ? (m - wave + FW - 1) / FW : 0;   // this wavefront's rows
        float t[TS], rs;
        ask(t, lane, wave);
        if (n == 0) {
            rs = rms(t, sh, lane, wave);
        } else if (n == 1) {
            floatx4 a[JP];
            load(a, wave);
            rs = rms(t, sh, lane, wave);
            TRACE(7);
            put(a, wave, rs, xs);
        } else {
            floatx4 a[JP], b[JP];
            load(a, wave);
            load(b, wave + FW);
            rs = rms(t, sh, lane, wave);
            TRACE(7);
            rows(a, b, n, rs, xs, wave);
        }
        for (int seg = 1; seg * 64 * JP < chunks; ++seg) {
            columns(seg, lane);
            floatx4 a[JP], b[JP];
            if (n == 1) {
                load(a, wave);
                put(a, wave, rs, xs);
            } else if (n > 1) {
                load(a, wave);
                load(b, wave + FW);
                rows(a, b, n, rs, xs, wave);
            }
        }
    }
};

// A workgroup's items in a GEMM phase: units unit0 + i * ustep, i < n_my, of K split `split`; worked out once per launch.
// Workgroup w takes items w, w + G, ... of (unit, split): the splits divide G, or there is one item per workgroup at most.
struct Items { int unit0, ustep, split, n_my; };
__device__ __forceinline__ Items items_of(int units, int ks) {
    const int w = blockIdx.x, G = gridDim.x, n = units * ks;
    return Items{w / ks, G / ks, w % ks, w < n ? (n - w + G - 1) / G : 0};
}
// ---- QKV phase --------------------------------------------------------------------------------------------
// One 16-row weight block per item; the wavefronts share its K.  Few items a workgroup (one at the 0.5B and
// 1.5B shapes, whose weights are then all requested before the barrier), so what counts is the chain behind the
// barrier: staging, one read of the wavefront's activation fragments, products, the sum over the wavefronts.
template <int NB, int HD, int JP>
__device__ __forceinline__ void qkv_phase(const FastGemm &g, const Items &im, GridBar &bar, unsigned char *smem, int lds_total,
                                          FusedShared &sh TRACE_ARG) {
    constexpr int PD = JP;   // k-blocks of a wavefront: an eighth of a pass's columns
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = g.m, KB = g.KB;
    const int cnt = (KB + FW - 1) / FW, rounds = (cnt + PD - 1) / PD;
    const int wk0 = wave * cnt, mine = min(cnt, KB - wk0);   // k-blocks wk0 .. wk0 + mine - 1 (none: mine <= 0)
    floatx4 *red = reinterpret_cast<floatx4 *>(smem + lds_total - FW * NB * 1024);
    const int row = wave * 16 + (lane & 15);   // wavefront c < NB finishes the tile of row block c
    global_w_ptr W = (global_w_ptr)g.W;

    u32x4 w[PD];
#pragma unroll
    for (int d = 0; d < PD; ++d) w[d] = u32x4{0u, 0u, 0u, 0u};
    auto load_w = [&](int unit, int d, int kbl) {   // never predicated: see resid_phase
        w[d] = __builtin_nontemporal_load(W + ((size_t)unit * KB + min(wk0 + min(kbl, cnt - 1), KB - 1)) * 64 + lane);
    };
    NormStage<JP> ns;
    EpiPre pre;
    pre.v = pre.bias = floatx4{0.f, 0.f, 0.f, 0.f};
    if (im.n_my > 0) {
        ns.init(g, lane);
#pragma unroll
        for (int d = 0; d < PD; ++d) load_w(im.unit0, d, d);
        if (wave < NB) pre = epi_qkv_ask<HD>(g, sh, min(row, m - 1), im.unit0, lane);
    }
    TRACE(1);
    bar.wait();
    TRACE(2);
    if (im.n_my <= 0) return;
    ns.run(smem, sh, lane, wave TRACE_PASS);
    lds_sync();
    TRACE(3);
    // lane's 16 bytes of row block 0 in a k-block; rows past the last read what lies behind (their columns of the
    // product are not stored)
    const unsigned char *xl = smem + (lane & 15) * 64 + (lane >> 4) * 16;
    for (int it = 0; it < im.n_my; ++it) {
        const int unit = im.unit0 + it * im.ustep;
        const bool has_next = it + 1 < im.n_my;
        floatx4 acc[NB];
#pragma unroll
        for (int c = 0; c < NB; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
        auto round_body = [&](auto refill_tag, int r) {
            constexpr bool REFILL = decltype(refill_tag)::value;
            const bool last_round = r + 1 == rounds;
            bf16x8 x[PD][NB];
#pragma unroll
            for (int d = 0; d < PD; ++d) {
                const int kx = min(wk0 + min(r * PD + d, cnt - 1), KB - 1);
#pragma unroll
                for (int c = 0; c < NB; ++c) x[d][c] = *reinterpret_cast<const bf16x8 *>(xl + kx * m * 64 + c * 1024);
            }
#pragma unroll
            for (int d = 0; d < PD; ++d) {
                if (r * PD + d < mine) {
#pragma unroll
                    for (int c = 0; c < NB; ++c)
                        acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[d]), x[d][c], acc[c], 0, 0, 0);
                }
                if (REFILL) load_w(last_round ? unit + im.ustep : unit, d, last_round ? d : (r + 1) * PD + d);
            }
        };
#pragma unroll 1
        for (int r = 0; r + 1 < rounds; ++r) round_body(std::true_type{}, r);
        if (has_next) round_body(std::true_type{}, rounds - 1);
        else round_body(std::false_type{}, rounds - 1);
        TRACE(4);
        if (it) lds_sync();   // the previous item's sums have been read
#pragma unroll
        for (int c = 0; c < NB; ++c) red[(c * FW + wave) * 64 + lane] = acc[c];
        lds_sync();
        if (wave < NB) {
            const floatx4 v = sum_waves(red, wave, lane);
            if (row < m) epi_qkv_store<HD>(g, sh, row, unit, lane, v, pre);
            if (has_next) pre = epi_qkv_ask<HD>(g, sh, min(row, m - 1), unit + im.ustep, lane);
        }
        TRACE(5);
    }
}

// ---- residual phases: O and down projection -----------------------------------------------------------
// h_out = h_in + X W^T with X bfloat16 in MFMA operand order (the attention and SwiGLU epilogues write it that
// way).  Every fragment of X has one reader in a workgroup, the wavefront that owns its k-blocks, so X goes from
// memory into registers: no staging in LDS, no barrier between the loads and the products, no index arithmetic,
// and no limit on the K slice.  Behind the grid barrier a wavefront issues one load per fragment, its products,
// and the sum over the wavefronts; everything else (weights, addresses, the residual tile) comes before it.
// Items: (unit of UB weight blocks) x (K split).  The splits of a unit exchange their sums tile by
// tile, wavefront to wavefront; no workgroup barrier is in that chain.
// Depth: all k-blocks of a wavefront at once where the shape allows (weights requested before the barrier, X in one
// round trip behind it).  Release to last arrival, staged through LDS / so: O of 0.5B, 1 row 2.9 / 1.7 us, of 1.5B,
// 17 rows 3.1 / 2.5; down of 1.5B, 17 rows 8.3 / 7.0 (in two rounds of five k-blocks instead of one of seven 8.4).
struct ResidGemm {
    global_w_ptr W;
    const bf16_t *X;   // [K / 32][NB] fragments
    const float *h_in;
    float *h, *ss_out;
    float *xch;        // partial tiles of the K splits
    unsigned *fail;
    int N, KB, m, ks, kbps;
    Items im;
};
template <int NB, int UB, int PD>
__device__ __forceinline__ XchUsed resid_phase(const ResidGemm &g, GridBar &bar, unsigned char *smem TRACE_ARG) {
    const XchUsed used{(unsigned)(g.im.unit0 * g.ks * UB * NB) * 1024, UB * NB * 1024, g.im.n_my > 0 && g.ks > 1 ? g.ks : 0, g.im.split, UB * NB};
    constexpr int NTILE = UB * NB;
    static_assert(NTILE <= FW, "a tile of the unit per wavefront");
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KB = g.KB, NBt = g.N >> 4;
    const int kb0 = g.im.split * g.kbps, kb1 = min(KB, kb0 + g.kbps);
    const int cnt = (kb1 - kb0 + FW - 1) / FW, rounds = (cnt + PD - 1) / PD;
    const int wk0 = kb0 + wave * cnt, mine = min(cnt, kb1 - wk0);   // k-blocks wk0 .. wk0 + mine - 1 (none: mine <= 0)
    floatx4 *red = reinterpret_cast<floatx4 *>(smem);
    const int tu = wave / NB, tc = wave % NB;   // this wavefront's tile of a unit (wave < NTILE)
    const int owner = wave % g.ks;              // the K split that puts it together
    const int row = tc * 16 + (lane & 15), crow = min(row, g.m - 1);

    u32x4 w[PD][UB], x[PD][NB];
#pragma unroll
    for (int d = 0; d < PD; ++d)
#pragma unroll
        for (int u = 0; u < UB; ++u) w[d][u] = u32x4{0u, 0u, 0u, 0u};
    // never predicated: a step past the end of the run loads the run's last fragment again and is skipped
    auto load_w = [&](int unit, int d, int kbl) {
        const int kb = min(wk0 + min(kbl, cnt - 1), kb1 - 1);
#pragma unroll
        for (int u = 0; u < UB; ++u)
            w[d][u] = __builtin_nontemporal_load(g.W + ((size_t)min(unit * UB + u, NBt - 1) * KB + kb) * 64 + lane);
    };
    auto load_x = [&](int d, int kbl) {
        const int kb = min(wk0 + min(kbl, cnt - 1), kb1 - 1);
#pragma unroll
        for (int c = 0; c < NB; ++c) x[d][c] = ssa_load_16(g.X + ((size_t)(kb * NB + c) * 64 + lane) * 8);
    };
    auto load_h = [&](int unit) {
        const int nb = min(unit * UB + tu, NBt - 1);
        return ssa_load_f4(g.h_in + (size_t)crow * g.N + nb * 16 + (lane >> 4) * 4);
    };
    EpiPre pre;
    pre.v = pre.bias = floatx4{0.f, 0.f, 0.f, 0.f};
    if (g.im.n_my > 0) {
#pragma unroll
        for (int d = 0; d < PD; ++d) load_w(g.im.unit0, d, d);
        pre.v = load_h(g.im.unit0);   // written two or more barriers ago
    }
    TRACE(1);
    bar.wait();
    TRACE(2);
    if (g.im.n_my <= 0) return used;
#pragma unroll
    for (int d = 0; d < PD; ++d) load_x(d, d);
    for (int it = 0; it < g.im.n_my; ++it) {
        const int unit = g.im.unit0 + it * g.im.ustep;
        const bool has_next = it + 1 < g.im.n_my;
        floatx4 acc[UB][NB];
#pragma unroll
        for (int u = 0; u < UB; ++u)
#pragma unroll
            for (int c = 0; c < NB; ++c) acc[u][c] = floatx4{0.f, 0.f, 0.f, 0.f};
        auto round_body = [&](auto refill_tag, int r) {
            constexpr bool REFILL = decltype(refill_tag)::value;
            const bool last_round = r + 1 == rounds;
            const int nunit = last_round ? unit + g.im.ustep : unit, nk = last_round ? 0 : (r + 1) * PD;
#pragma unroll
            for (int d = 0; d < PD; ++d) {
                if (r * PD + d < mine) {
#pragma unroll
                    for (int c = 0; c < NB; ++c)
#pragma unroll
                        for (int u = 0; u < UB; ++u)
                            acc[u][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[d][u]),
                                                                                __builtin_bit_cast(bf16x8, x[d][c]), acc[u][c], 0, 0, 0);
                }
                if (REFILL) {
                    load_w(nunit, d, nk + d);
                    load_x(d, nk + d);
                }
            }
        };
#pragma unroll 1
        for (int r = 0; r + 1 < rounds; ++r) round_body(std::true_type{}, r);
        if (has_next) round_body(std::true_type{}, rounds - 1);
        else round_body(std::false_type{}, rounds - 1);
        TRACE(4);
        // sum over the wavefronts: pairs (w, w + 4), then the four pairs in order
        if (it) lds_sync();   // the previous item's sums have been read
#pragma unroll
        for (int u = 0; u < UB; ++u)
#pragma unroll
            for (int c = 0; c < NB; ++c) red[((u * NB + c) * FW + wave) * 64 + lane] = acc[u][c];
        lds_sync();
        if (wave < NTILE) {
            floatx4 v = sum_waves(red, wave, lane);
            TRACE(8);
            const unsigned at = (unsigned)(unit * g.ks * NTILE + wave) * 1024, stride = NTILE * 1024;
            if (g.ks > 1 && owner != g.im.split) {
                xch_send(g.xch + (at + g.im.split * stride) / 4 + lane * 4, v);
            } else {
                if (g.ks > 5) v = xch_sum<MAX_DOWN_SPLITS>(v, g.xch, at, stride, g.ks, g.im.split, lane, g.fail);
                else if (g.ks > 1) v = xch_sum<5>(v, g.xch, at, stride, g.ks, g.im.split, lane, g.fail);
                TRACE(9);
                const int nb = unit * UB + tu;
                FastGemm e;
                e.N = g.N; e.h = g.h; e.ss_out = g.ss_out;
                epi_resid_pre(e, row, row < g.m && nb < NBt, nb, lane, v, pre);
            }
            if (has_next) pre.v = load_h(unit + g.im.ustep);
        }
        TRACE(5);
    }
    return used;
}

// ---- GEMM phase with whole weight blocks per wavefront ---------------------------------------------------
// For the matrices with many more 16-row blocks than a K split across workgroups could use (gate/up,
// output head) and a K that fits LDS whole.  A wavefront streams its share of a block's fragments
// through a ring of RING registers and keeps the accumulators to itself: no partial sums in LDS
// per work item, no workgroup barrier inside the streaming loop.  Every wavefront of the chip holds
// RING fragments in flight, issued before the barrier wait; what limits a compute unit's share of
// the stream is the bytes it has in flight, so all eight wavefronts of a workgroup carry a ring.
//   gate/up: a pass covers two units of the workgroup (unit = 16 ffn columns: a block of gate rows
//            and a block of up rows); its eight tasks (unit, gate | up, lower | upper half of K) go
//            to the eight wavefronts.  At the end of a pass the four tiles of a unit meet in LDS;
//            wavefront q of the unit adds the halves of row block q and applies SwiGLU.
//   head:    blocks w, w + W, ... (W = wavefronts of the grid) per wavefront, full K, one after
//            the other through the same ring; logits are stored from the accumulators.
constexpr int wave_tail_bytes(int nb) { return FW * nb * 1024; }   // LDS behind the staged activations: the tiles of a pass
template <int NB, int HD, int EPI>
__device__ __forceinline__ void wave_phase(const FastGemm &g, int n_light, GridBar &bar, unsigned char *smem, int lds_total,
                                           FusedShared &sh TRACE_ARG) {
    static_assert(EPI == EPI_SWIGLU || EPI == EPI_LOGITS, "gate/up and output head");
    static_assert(NB <= 4, "one row block per wavefront of a unit");
    constexpr int RING = HD == 64 ? 16 : 24;   // half a row of the narrow models' K, of 1536 columns
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = gridDim.x, wg = blockIdx.x;
    const int m = g.m, KB = g.KB, NBt = g.N >> 4;
    u32x4 *xs = reinterpret_cast<u32x4 *>(smem);
    floatx4 *exch = reinterpret_cast<floatx4 *>(smem + lds_total - wave_tail_bytes(NB));

    // this wavefront's tasks: block of task j = blk0 + j * bstride, all over the K range [kb_lo, kb_hi)
    // (gate/up: pass j, slot s covers units (2j + s) G .. + G; a range that the units fill only in part is
    //  handed out from the top workgroup downwards: the workgroups at the bottom of the grid are the ones
    //  busy in the O projection before, and the last to start here)
    // (With n_light > 0 the first n_light workgroups -- the ones that work in the O projection and so
    //  start here last, their weight ring requested behind everybody else's -- take one unit each, and
    //  the others, which have had their rings in flight since the O projection began, share the rest:
    //  unit n_light + (wg - n_light) + t H for t = 0, 1, 2, ..., H = G - n_light.)
    int blk0, bstride, n_task, kb_lo, kb_hi, passes, blk_last = -1;
    if (EPI == EPI_SWIGLU) {
        const int n_units = NBt >> 1, slot = wave >> 2, KBh = (KB + 1) >> 1;
        const int sub = (wave >> 1) & 1;
        if (n_light > 0) {
            const int H = G - n_light, T = (max(n_units - n_light, 0) + H - 1) / H;
            passes = max(1, (T + 1) / 2);
            if (wg < n_light) {
                blk0 = 2 * wg + sub;
                bstride = 0;
                n_task = (slot == 0 && wg < n_units) ? 1 : 0;
            } else {
                const int u0 = n_light + (wg - n_light) + slot * H;
                blk0 = 2 * u0 + sub;
                bstride = 4 * H;
                n_task = u0 < n_units ? (n_units - u0 + 2 * H - 1) / (2 * H) : 0;
            }
        } else {
            blk0 = 2 * (wg + slot * G) + sub;
            bstride = 4 * G;
            passes = max(1, (n_units + 2 * G - 1) / (2 * G));
            n_task = 0;
            for (int j = 0; j < passes; ++j) {
                const int start = (2 * j + slot) * G, left = n_units - start;
                if (left >= G) ++n_task;
                else if (left > 0) {
                    const int idx = G - 1 - wg;
                    if (idx < left) { blk_last = 2 * (start + idx) + sub; ++n_task; }
                }
            }
        }
        kb_lo = (wave & 1) ? KBh : 0;
        kb_hi = (wave & 1) ? KB : KBh;
    } else {
        const int gw = wave * G + wg, W = FW * G;          // neighbouring blocks on different compute units
        blk0 = gw;
        bstride = W;
        n_task = gw < NBt ? (NBt - gw + W - 1) / W : 0;
        kb_lo = 0;
        kb_hi = KB;
        passes = n_task;
    }
    const int rpt = max(1, (kb_hi - kb_lo + RING - 1) / RING);  // rounds per task
    const int rounds = n_task * rpt;
    global_w_ptr wbase = (global_w_ptr)g.W + lane;
    u32x4 w[RING];
#pragma unroll
    for (int d = 0; d < RING; ++d) w[d] = u32x4{0u, 0u, 0u, 0u};
    // fragment of flat round r, slot d.  Never predicated: a step past the end of the K range (or of
    // the wavefront's tasks) reads a valid fragment again and its product is discarded.
    auto task_block = [&](int j) { return (j == n_task - 1 && blk_last >= 0) ? blk_last : blk0 + j * bstride; };
    auto frag = [&](int r, int d) {
        const int j = min(r / rpt, max(n_task - 1, 0));
        const int kb = min(kb_lo + (r % rpt) * RING + d, kb_hi - 1);
        const size_t blk = (size_t)min(task_block(j), NBt - 1);
        return __builtin_nontemporal_load(wbase + (blk * KB + kb) * 64);
    };
    NormStage<JP_OF(HD)> ns;
    ns.init(g, lane);
    if (n_task > 0) {
#pragma unroll
        for (int d = 0; d < RING; ++d) w[d] = frag(0, d);
    }
    TRACE(1);
    bar.wait();
    TRACE(2);

    ns.run(smem, sh, lane, wave TRACE_PASS);
    lds_sync();
    TRACE(3);

    int xoff[NB];
#pragma unroll
    for (int c = 0; c < NB; ++c) xoff[c] = min(c * 16 + (lane & 15), m - 1) * 4 + (lane >> 4);

    floatx4 acc[NB];
#pragma unroll
    for (int c = 0; c < NB; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};

    // one round = RING steps of straight-line code; REFILL: every slot is loaded again after its
    // use with the fragment of the next round (the same task's next K range or the next task)
    auto round_body = [&](auto refill_tag, int r) {
        constexpr bool REFILL = decltype(refill_tag)::value;
        const int kbase = kb_lo + (r % rpt) * RING;
        constexpr int BA = FUSED_BB_AHEAD < RING ? FUSED_BB_AHEAD : RING - 1;
        bf16x8 bb[BA + 1][NB];
        auto read_bb = [&](int d) {
            const int kx = min(kbase + d, kb_hi - 1);
#pragma unroll
            for (int c = 0; c < NB; ++c) bb[d % (BA + 1)][c] = __builtin_bit_cast(bf16x8, xs[kx * m * 4 + xoff[c]]);
        };
#pragma unroll
        for (int d = 0; d < BA; ++d) read_bb(d);
#pragma unroll
        for (int d = 0; d < RING; ++d) {
            const bool live = kbase + d < kb_hi;
            const bf16x8 a = __builtin_bit_cast(bf16x8, live ? w[d] : u32x4{0u, 0u, 0u, 0u});
            if (REFILL) w[d] = frag(r + 1, d);
            if (d + BA < RING) read_bb(d + BA);
#pragma unroll
            for (int c = 0; c < NB; ++c)
                acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bb[d % (BA + 1)][c], acc[c], 0, 0, 0);
        }
        if (FUSED_SGB > 0) {
            constexpr int SA = FUSED_SGB < RING ? FUSED_SGB : RING;
            __builtin_amdgcn_sched_group_barrier(0x100, SA * NB, 0);
#pragma unroll
            for (int d = 0; d < RING; ++d) {
                __builtin_amdgcn_sched_group_barrier(0x008, NB, 0);
                if (d + SA < RING) __builtin_amdgcn_sched_group_barrier(0x100, NB, 0);
            }
        }
    };

#pragma unroll 1
    for (int j = 0; j < passes; ++j) {
        const bool mine = j < n_task;
        if (mine) {
#pragma unroll 1
            for (int rr = 0; rr < rpt; ++rr) {
                const int r = j * rpt + rr;
                if (r + 1 < rounds) round_body(std::true_type{}, r);
                else round_body(std::false_type{}, r);
            }
        }
        TRACE(4);
        const int nb = task_block(j);
        if (EPI == EPI_LOGITS) {
#pragma unroll
            for (int c = 0; c < NB; ++c) {
                const int row = c * 16 + (lane & 15);
                if (row < m)
                    __builtin_nontemporal_store(acc[c], reinterpret_cast<floatx4 *>(g.logits + (size_t)row * g.N + nb * 16 + (lane >> 4) * 4));
                acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
        } else {
            // tile (wavefront w, row block c) at exch[(w * NB + c) * 64 + lane]; wavefronts 4u .. 4u + 3 hold
            // unit u's gate lower, gate upper, up lower, up upper half
            if (j) lds_sync();   // the previous pass's tiles have been read
            if (mine) {
#pragma unroll
                for (int c = 0; c < NB; ++c) exch[(wave * NB + c) * 64 + lane] = acc[c];
            }
            lds_sync();
            const int q = wave & 3, w0 = wave & ~3;
            if (mine && q < NB) {
                floatx4 t4[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) t4[i] = exch[((w0 + i) * NB + q) * 64 + lane];
                asm volatile("" ::: "memory");
                const int row = q * 16 + (lane & 15);
                if (row < m) epi_swiglu_frag(g, row, nb & ~1, lane, t4[0] + t4[1], t4[2] + t4[3], NB);
            }
#pragma unroll
            for (int c = 0; c < NB; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
        TRACE(5);
    }
}

template <int NB, int HD>
__global__ __launch_bounds__(FT, 2) void verify_fused_kernel(FusedArgs a, Batch b) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ FusedShared sh;
    const unsigned start = barrier_start(a.bar_start);
    const int d = a.d, F = a.F, hd = a.hd, nq = a.hq * hd, nkv = a.hkv * hd;
    const size_t hstride = (size_t)a.frows * d, sstride = (size_t)(d / 16) * 64;

#ifdef FUSED_TRACE
    Trace trace{reinterpret_cast<unsigned long long *>(a.bar + 8192), 0};
#endif
    const int len0 = launch_tables(a, b, sh);
    TRACE(0);
    embed_phase(a, b);
    GridBar bar = grid_bar(a.bar, a.fail, __builtin_amdgcn_readfirstlane(start));
    bar.arrive();   // (a workgroup barrier inside: the row table is visible to every wavefront from here on)

    FastGemm base;
    base.m = a.m;
    base.n_ss = d / 16;
    base.inv_d = a.inv_d;
    base.eps = a.eps;
    base.F = F;
    base.cosv = a.cosv;
    base.sinv = a.sinv;
    base.depth = a.tree_depth;
    base.hq = a.hq;
    base.hkv = a.hkv;
    base.hd = hd;
    base.kch = 0;
    base.X = nullptr; base.Xh = nullptr; base.gain = nullptr; base.ss_in = nullptr; base.h_in = nullptr;
    base.h = nullptr; base.ss_out = nullptr; base.a_out = nullptr; base.logits = nullptr; base.bias = nullptr;
    base.q = nullptr; base.layer = 0;

    const Items it_qkv = items_of((nq + 2 * nkv) / 16, 1), it_o = items_of(d / 16, 1);
    const Items it_down = items_of((d / 16 + a.down_ub - 1) / a.down_ub, a.ks_down);
    const int kbps_down = (F / 32 + a.ks_down - 1) / a.ks_down;

#pragma unroll 1
    for (int l = 0; l < a.n_layers; ++l) {
        const FusedLayer lp = layer_params(a, l);
        float *h0 = a.hv + (size_t)(2 * l) * hstride, *h1 = h0 + hstride, *h2 = h1 + hstride;
        float *ss0 = a.ssv + (size_t)(2 * l) * sstride, *ss1 = ss0 + sstride, *ss2 = ss1 + sstride;
        bf16_t *q = a.qv + (size_t)l * a.frows * nq, *o = a.ov + (size_t)l * a.frows * nq;
        bf16_t *act = a.av + (size_t)l * a.frows * F;
        {
            FastGemm g = base;
            g.W = lp.wqkv; g.N = nq + 2 * nkv; g.KB = d / 32; g.Xh = h0; g.gain = lp.attn_norm; g.ss_in = ss0;
            g.bias = a.has_bias ? lp.bqkv : nullptr; g.layer = l; g.q = q;
            qkv_phase<NB, HD, JP_OF(HD)>(g, it_qkv, bar, smem, a.lds_total, sh TRACE_PASS);
        }
        bar.arrive();
        TRACE(10);
        const XchUsed att_used = attn_phase<HD>(a, b, l, q, o, NB, len0, bar, smem, sh TRACE_PASS);
        bar.arrive();
        xch_clear<2>(a.xch, att_used);
        TRACE(13);
        {
            const ResidGemm g{(global_w_ptr)lp.wo, o, h0, h1, ss1, a.xch, a.fail, d, nq / 32, a.m, 1, nq / 32, it_o};
            if (nq <= 4 * FW * 32) resid_phase<NB, 1, 4>(g, bar, smem TRACE_PASS);   // four k-blocks a wavefront
            else resid_phase<NB, 1, 6>(g, bar, smem TRACE_PASS);
        }
        bar.arrive();
        TRACE(14);
        {
            FastGemm g = base;
            g.W = lp.wgu; g.N = 2 * F; g.KB = d / 32; g.Xh = h1; g.gain = lp.ffn_norm; g.ss_in = ss1; g.a_out = act;
            wave_phase<NB, HD, EPI_SWIGLU>(g, a.gu_light, bar, smem, a.lds_total, sh TRACE_PASS);
        }
        bar.arrive();
        TRACE(15);
        XchUsed down_used;
        {
            const ResidGemm g{(global_w_ptr)lp.wd, act, h1, h2, ss2, a.xch, a.fail, d, F / 32, a.m, a.ks_down, kbps_down, it_down};
            if (a.down_ub == 1) down_used = resid_phase<NB, 1, 5>(g, bar, smem TRACE_PASS);
            else down_used = resid_phase<NB, 2, NB <= 2 ? 7 : 5>(g, bar, smem TRACE_PASS);
        }
        bar.arrive();
        xch_clear<1>(a.xch, down_used);
        TRACE(16);
    }
    {
        FastGemm g = base;
        g.W = a.lm_head; g.N = a.vocab; g.KB = d / 32;
        g.Xh = a.hv + (size_t)(2 * a.n_layers) * hstride; g.gain = a.final_norm;
        g.ss_in = a.ssv + (size_t)(2 * a.n_layers) * sstride; g.logits = a.logits;
        wave_phase<NB, HD, EPI_LOGITS>(g, 0, bar, smem, a.lds_total, sh TRACE_PASS);
    }
    barrier_advance(a.bar_start, bar);
    TRACE(99);
#ifdef FUSED_ARRIVALS
    if (threadIdx.x == 0) bar.stamps[((size_t)bar.n_arr * 2) * gridDim.x + blockIdx.x] = wall_clock64();  // end of the head phase
#endif
}

// ---- host side -------------------------------------------------------------------------------------

// K split of the down projection, whose slices are not staged: as many splits as leave one item per workgroup and a
// k-block per wavefront.
int fill_split(int G, int units, int KB) {
    int best = 1;
    for (int ks = 2; units * ks <= G && ks <= std::min(KB, MAX_DOWN_SPLITS); ++ks) {
        const int kbps = (KB + ks - 1) / ks;
        if ((KB + kbps - 1) / kbps == ks && kbps >= FW) best = ks;
    }
    return best;
}

}  // namespace

// What a work item sends through the exchange at most: 4 x 3 tiles of a down projection (fused_direct.hip), the d-blocks of
// an attention part with their (max, sum) pairs.  One item per workgroup.
static size_t xch_bytes(const vf_config &c) { return (size_t)FUSED_G * std::max(4 * 3, c.head_dim / 16 * 2) * 1024; }

// [barrier][arrival | release][workgroup]
static size_t stamp_bytes(const vf_config &c) {
#ifdef FUSED_ARRIVALS
    return (size_t)(2 + 7 * c.n_layers) * 2 * FUSED_G * 8;
#else
    return 0;
#endif
}

struct FusedBuffers { size_t h, ss, q, o, a, x, xch, bar, total; };
static FusedBuffers fused_buffers(const vf_config &c) {
    const size_t L = c.n_layers, d = c.d_model, nq = (size_t)c.n_q_heads * c.head_dim, F = c.d_ffn, R = fused_rows(c);
    FusedBuffers f;
    size_t n = 0;
    auto add = [&](size_t bytes) { const size_t at = n; n += (bytes + 255) & ~(size_t)255; return at; };
    f.h = add((2 * L + 1) * R * d * 4);
    f.ss = add((2 * L + 1) * (d / 16) * 64 * 4);
    f.q = add(L * R * nq * 2);
    f.o = add(L * R * nq * 2);
    f.a = add(L * R * F * 2);
    f.x = add(2 * L * R * d * 2);
    f.xch = add(xch_bytes(c));
    f.bar = add(BAR_WORDS * 4 + stamp_bytes(c));
    f.total = n;
    return f;
}

size_t vf_fused_workspace_bytes(const vf_config &c) { return c.dtype == VF_BF16 ? fused_buffers(c).total : 0; }

int vf_fused_init(vf_model *m, char *ws, hipStream_t st) {
    const vf_config &c = m->cfg;
    const FusedBuffers f = fused_buffers(c);
    m->fz_h = (float *)(ws + f.h);
    m->fz_ss = (float *)(ws + f.ss);
    m->fz_q = ws + f.q;
    m->fz_o = ws + f.o;
    m->fz_a = ws + f.a;
    m->fz_x = ws + f.x;
    m->fz_xch = (float *)(ws + f.xch);
    VF_HIP(hipMemsetAsync(m->fz_xch, 0xff, xch_bytes(c), st));   // marks everywhere
    m->fz_bar = (unsigned *)(ws + f.bar);
    // the kernel addresses the parameters of layer l as those of layer 0 plus l times one distance
    for (int l = 1; l < c.n_layers; ++l) {
        const LayerPacked &x = m->layers[l - 1], &y = m->layers[l], &z = m->layers[0], &o = m->layers[1];
        auto same = [](const void *a, const void *b, const void *c, const void *d) { return (const char *)b - (const char *)a == (const char *)d - (const char *)c; };
        if (!same(x.wqkv, y.wqkv, z.wqkv, o.wqkv) || !same(x.wo, y.wo, z.wqkv, o.wqkv) || !same(x.wgu, y.wgu, z.wqkv, o.wqkv) ||
            !same(x.wd, y.wd, z.wqkv, o.wqkv) || !same(x.attn_norm, y.attn_norm, z.wqkv, o.wqkv) ||
            !same(x.ffn_norm, y.ffn_norm, z.wqkv, o.wqkv) || !same(x.bqkv, y.bqkv, z.wqkv, o.wqkv))
            return vf_fail(VF_ERR_ARG, "persistent kernel: layers at unequal distances");
    }
    VF_HIP(hipStreamSynchronize(st));   // a model is ready for any stream once it is created
    return VF_OK;
}

// Whether a call's rows fit LDS next to the tiles of a pass.
bool vf_fused_ok(const vf_config &c, int rows) {
    return fused_shape_ok(c) && rows <= FROWS &&
           (size_t)(c.d_model / 32) * rows * 64 + wave_tail_bytes((rows + 15) / 16) <= (size_t)LDS_BYTES;
}

int vf_run_fused(vf_model *m, const Batch &b, const int32_t *tokens, float *logits_out, bool tree, hipStream_t st) {
    const vf_config &c = m->cfg;
    if (!vf_fused_ok(c, b.total_rows)) return vf_fail(VF_ERR_UNSUPPORTED, "persistent kernel does not apply to this call");
    FusedArgs a;
    memset(&a, 0, sizeof a);
    fused_args(m, b, tokens, tree, a);
    a.logits = logits_out;
    // one weight block an item where that still gives three splits or more: a narrow model's items of two blocks need
    // nine splits to fill the chip, and an owner waits for all of them (0.5B, 1 row: 632 us a pass, with four 601)
    a.down_ub = c.d_model / 16 * 3 <= FUSED_G ? 1 : 2;
    a.ks_down = fill_split(FUSED_G, (c.d_model / 16 + a.down_ub - 1) / a.down_ub, c.d_ffn / 32);
    {
        // one unit for each workgroup of the O projection, if the others can take the rest in at most
        // three units each (two passes)
        const int n_o = c.d_model / 16, units = c.d_ffn / 16, H = FUSED_G - n_o;
        a.gu_light = (H > 0 && n_o < units && units - n_o <= 3 * H && units - n_o > H) ? n_o : 0;
    }
    ProfScope ps(m, VF_SITE_STEP, st);
    const int nb = (b.total_rows + 15) / 16;
    if (c.head_dim == 128) {
        if (nb == 1) return fused_launch<&verify_fused_kernel<1, 128>>(a, b, st);
        if (nb == 2) return fused_launch<&verify_fused_kernel<2, 128>>(a, b, st);
        return fused_launch<&verify_fused_kernel<3, 128>>(a, b, st);
    }
    if (nb == 1) return fused_launch<&verify_fused_kernel<1, 64>>(a, b, st);
    if (nb == 2) return fused_launch<&verify_fused_kernel<2, 64>>(a, b, st);
    return fused_launch<&verify_fused_kernel<3, 64>>(a, b, st);
}

// Whether any barrier of an earlier launch gave up (the stream must be idle).
int vf_fused_check(vf_model *m) {
    if (!m->fz_bar) return VF_OK;
    unsigned flag = 0;
    VF_HIP(hipMemcpy(&flag, m->fz_bar + BAR_FAIL, 4, hipMemcpyDeviceToHost));
    if (flag) {
        // counters and their start value are out of step now: start over from zero
        VF_HIP(hipMemset(m->fz_bar, 0, BAR_WORDS * 4));
        VF_HIP(hipMemset(m->fz_xch, 0xff, xch_bytes(m->cfg)));
        return vf_fail(VF_ERR_HIP, "persistent verify kernel: a grid barrier timed out; results of that call are invalid");
    }
    return VF_OK;
}

#ifdef FUSED_ARRIVALS
// Copies the arrival / release stamps of the last launch: [barrier][2][workgroup].
extern "C" int vf_debug_arrivals(vf_model *m, unsigned long long *out_host, int n_barriers) {
    if (!m->fz_bar || n_barriers < 0 || (size_t)n_barriers * 2 * FUSED_G * 8 > stamp_bytes(m->cfg)) return vf_fail(VF_ERR_ARG, "vf_debug_arrivals");
    VF_HIP(hipDeviceSynchronize());
    VF_HIP(hipMemcpy(out_host, m->fz_bar + BAR_WORDS, (size_t)n_barriers * 2 * FUSED_G * 8, hipMemcpyDeviceToHost));
    return VF_OK;
}
#endif

#ifdef FUSED_TRACE
// Copies the phase timeline of the traced workgroup's last launch: pairs (clock, mark id).
extern "C" int vf_debug_trace(vf_model *m, unsigned long long *out_host, int n_pairs) {
    VF_HIP(hipDeviceSynchronize());
    VF_HIP(hipMemcpy(out_host, m->fz_bar + 8192, (size_t)n_pairs * 16, hipMemcpyDeviceToHost));
    return VF_OK;
}
#endif
