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
//     before it signals anything (a barrier arrival, a counter) to other workgroups;
//   * bulk data is read with ordinary loads from single-assignment buffers -- one version of
//     the residual stream per half layer, one q / attention output / SwiGLU buffer and one set
//     of attention records per layer -- so no cache can hold a stale line of it: a line is never
//     read before its only write in a launch, and caches start clean at every launch;
//   * data in reused buffers (split-K partial tiles, counters) is read with agent-scope loads.
// The KV cache is written (new rows) and read (all rows) once per layer and launch, in that
// order; tiles that hold new rows are read with agent-scope loads.
//
// Results do not depend on timing: every sum has a fixed order.
#include "fast_common.h"

#include <type_traits>

namespace {

constexpr int FW = 8;            // wavefronts per workgroup
constexpr int FT = FW * 64;      // threads per workgroup
constexpr int FROWS = 48;        // most rows of a call
constexpr int MAX_DOWN_SPLITS = 9;   // K splits of the down projection
#ifndef BAR_COUNTERS
#define BAR_COUNTERS 64           // counters a barrier's arrivals are spread over
#endif
constexpr int LDS_BYTES = 152 * 1024;  // dynamic LDS of the one workgroup a CU holds (160 KB less the static part)
constexpr long long SPIN_LIMIT = 4000000;  // polls before a barrier gives up (seconds, not microseconds)

#ifndef FUSED_AHEAD
#define FUSED_AHEAD 3          // gate/up, down and head phases: this many steps of the item after next are held in registers too (0: off)
#endif
#ifndef FUSED_MAXP
#define FUSED_MAXP 6              // most key parts per attention block (8 parts: 1280 us per launch, 6 1261, 5 1258, 4 1254, 3 1274, 2 1318;
                                  // every setting gives the same mean logit error at the full 1.5B size, 1.3e-2, but with 4 and 5 parts one row
                                  // of 136 lands at 2.12e-2 and 2.005e-2, past the stated 2e-2: 6 is the fastest setting inside it)
#endif
// One workgroup of 8 wavefronts per CU: two wavefronts per SIMD, so each may use up to 256 vector
// registers (weight ring + staging loads in flight) without spilling.
#ifndef FUSED_G
#define FUSED_G 256
#endif

// Pointers that reach the kernel through memory lose their address space; loads through them would
// be generic (flat) loads, which the compiler orders against every other load in flight.
typedef const floatx4 __attribute__((address_space(1))) *global_f4_ptr;
__device__ inline floatx4 load_global_f4(const float *p) { return *(global_f4_ptr)(p); }
typedef const u32x4 __attribute__((address_space(1))) *global_w_ptr;

// Loads from the single-assignment buffers (one version per phase and layer, written once per launch
// before they are read): no cache can hold an older copy of such a line, so an ordinary load will do.
#ifndef FUSED_SSA_PLAIN
#define FUSED_SSA_PLAIN 1
#endif
__device__ __forceinline__ floatx4 ssa_load_f4(const float *p) {
    return FUSED_SSA_PLAIN ? *reinterpret_cast<const floatx4 *>(p) : load_coherent(p);
}
__device__ __forceinline__ u32x4 ssa_load_16(const void *p) {
    return FUSED_SSA_PLAIN ? *reinterpret_cast<const u32x4 *>(p) : load_coherent16(p);
}
__device__ __forceinline__ float ssa_load_f1(const float *p) { return FUSED_SSA_PLAIN ? *p : load_coherent1(p); }

struct FusedLayer {
    const u32x4 *wqkv, *wo, *wgu, *wd;
    const float *attn_norm, *ffn_norm, *bqkv;
};

struct FusedArgs {
    FusedLayer layer0;              // the first layer's parameters; the others follow at equal distances
    unsigned long long layer_bytes;
    const bf16_t *embed;
    const u32x4 *lm_head;
    const float *final_norm, *cosv, *sinv;
    const int32_t *tree_depth;      // tree-structured drafts (else NULL): depth and ancestor mask of every row
    const tree_mask_t *tree_anc;
    const int32_t *tokens;
    float *hv;        // residual stream, [2L+1][FROWS][d]
    float *ssv;       // sums of squares of its rows per 16 columns, [2L+1][d/16][64]
    bf16_t *qv, *ov, *av;  // per layer: q [FROWS][Hq*hd], attention output, SwiGLU product [FROWS][F]
    float *xch;       // partial tiles of the down projection's K splits, then of the attention's key parts; marks between uses
    float *part;
    int *counters;
    unsigned *bar, *fail;
    float *logits;
    int n_layers, d, F, hq, hkv, hd, vocab, m, has_bias;
    int att_blocks, att_parts;  // (query block, kv head, sequence) blocks of the call; key parts per block
    // First attention work item of every workgroup (-1: none).  Workgroup w runs on compute die w % 8;
    // the map puts the query blocks that read the same keys (same sequence, kv head and key part) on one
    // die, so that its L2 serves all but the first of those reads.
    short att_first[FUSED_G];
    float inv_d, eps, scale_log2e;
    unsigned root0;   // value of the barrier's root counter when this launch starts
    int ks_qkv, ks_gu, ks_down, ks_head;
    int down_ub;              // weight blocks of a down projection item
    int gu_light;            // gate/up: the first gu_light workgroups (busy in the O projection) take one unit each (0: even shares)
    int wave_gu, wave_head;  // gate/up, output head: one weight block per wavefront (K unsplit and the staged rows fit)
    int lds_total;    // dynamic LDS bytes of this launch
};

// Counting barrier, split into arrive and wait.  The workgroups are spread over BAR_COUNTERS counters
// (each in a memory channel of its own, so that the increments of a barrier are not all serialised
// at one address); an arrival is one increment that returns nothing, and a barrier is complete when
// every counter has grown by the number of workgroups mapped to it.  Counters only ever grow:
// barrier number e of a launch waits for the counters' value at launch start + e * (G / BAR_COUNTERS).
// Lanes 0..BAR_COUNTERS-1 of the first wavefront poll one counter each.
struct GridBar {
    unsigned *mem, *fail;
    unsigned target, per;  // per: workgroups per counter
    bool dead;
#ifdef FUSED_ARRIVALS
    unsigned long long *stamps;  // [barrier][2][workgroup]: clock at the arrival and at the end of the wait
    int n_arr, n_wait;
#endif
    __device__ __forceinline__ void arrive() {
        stores_done();  // this wavefront's write-through stores have reached memory
        __syncthreads();
#ifdef FUSED_ARRIVALS
        if (threadIdx.x == 0) stamps[((size_t)n_arr * 2) * gridDim.x + blockIdx.x] = wall_clock64();
        ++n_arr;
#endif
        target += per;
        if (threadIdx.x == 0)
            __hip_atomic_fetch_add(mem + (blockIdx.x % BAR_COUNTERS) * 64, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ void wait() {
        if (threadIdx.x < 64 && !dead) {
            const int lane = threadIdx.x;
            const unsigned *mine = mem + min(lane, BAR_COUNTERS - 1) * 64;
            long long spins = 0;
            for (;;) {
                const bool done = (int)(__hip_atomic_load(mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - target) >= 0;
                if (__all(done)) break;
                __builtin_amdgcn_s_sleep(1);
                ++spins;
                if (spins > SPIN_LIMIT ||
                    ((spins & 1023) == 0 && __hip_atomic_load(fail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
                    __hip_atomic_store(fail, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    dead = true;  // give up for good: the launch drains without waiting again
                    break;
                }
            }
        }
        lds_sync();
#ifdef FUSED_ARRIVALS
        if (threadIdx.x == 0) stamps[((size_t)n_wait * 2 + 1) * gridDim.x + blockIdx.x] = wall_clock64();
        ++n_wait;
#endif
    }
};

// Optional phase timeline of one workgroup (build with -DFUSED_TRACE=<workgroup>): thread 0 stamps the
// constant-rate clock at the marked points into the second half of the barrier block.
#ifdef FUSED_TRACE
struct Trace {
    unsigned long long *buf;
    int n;
    __device__ __forceinline__ void mark(int id) {
        if (blockIdx.x == FUSED_TRACE && threadIdx.x == 0 && n < 2040) {
            buf[2 * n] = wall_clock64();
            buf[2 * n + 1] = ((unsigned long long)clock64() << 8) | (unsigned long long)id;  // shader-clock count
            ++n;
        }
    }
};
#define TRACE(id) trace.mark(id)
#define TRACE_ARG , Trace &trace
#define TRACE_PASS , trace
#else
#define TRACE(id)
#define TRACE_ARG
#define TRACE_PASS
#endif

// Where a row of the call goes in the KV cache and which rotary angle it takes; the same in every
// layer of a launch (sequence lengths do not change while it runs), so it is worked out once.
struct RowMeta {
    bf16_t *kv;      // the sequence's KV pool
    int n_pages;     // pages in that pool
    int page, tin;   // page and row inside the page of the row's cache slot
    int pos;         // position whose rotary angle the row takes
    int live;        // 0: the slot lies outside the sequence's capacity, nothing is written
};
struct FusedShared {
    float rs_s[64];
    float rs_tmp[FW][64];
    int s_last;
    RowMeta rows[FROWS];
};

// ---- embedding: row r by workgroup r ---------------------------------------------------------------
__device__ __forceinline__ void embed_phase(const FusedArgs &a, const Batch &b) {
    const int d = a.d;
    for (int row = blockIdx.x; row < a.m; row += gridDim.x) {
        int tok = a.tokens[row];
        if (tok == VF_PENDING) tok = b.s[find_seq(b, row)].state[1];
        if (tok < 0 || tok >= a.vocab) tok = 0;
        for (int k0 = 0; k0 < d; k0 += FT) {
            const int k = k0 + threadIdx.x;
            float v = 0.f;
            if (k < d) {
                v = (float)a.embed[wfrag_index(tok, k, d)];
                st_f32<true>(a.hv + (size_t)row * d + k, v);
            }
            float sq = v * v;
            sq += __shfl_xor(sq, 8, 64);
            sq += __shfl_xor(sq, 4, 64);
            sq += __shfl_xor(sq, 2, 64);
            sq += __shfl_xor(sq, 1, 64);
            if (k < d && (threadIdx.x & 15) == 0) st_f32<true>(a.ssv + (k >> 4) * 64 + row, sq);
        }
    }
}

#ifndef FUSED_BB_AHEAD
#define FUSED_BB_AHEAD 1          // GEMM phases: activation fragments are read from LDS this many steps ahead of their MFMAs (0: right before)
#endif
#ifndef FUSED_SGB
#define FUSED_SGB 1               // GEMM phases: LDS reads are scheduled this many steps ahead of their MFMAs (0: left to the compiler)
#endif

// Epilogues of the persistent kernel.  What they read from memory is requested ahead of the products, for a phase's
// first item before the grid barrier, so that no round trip is left between the last product and the stores.
//   QKV: bias, rotary embedding, q to its buffer, K and V rows into the cache (row table in LDS)
//   residual: h = h_in + y, and the tile's sums of squares for the next RMSNorm
struct EpiPre { floatx4 v, bias; };
// nb: the same for all lanes
template <int HD>
__device__ __forceinline__ EpiPre epi_qkv_ask(const FastGemm &g, const FusedShared &sh, int row, int nb, int lane) {
    EpiPre p;
    p.bias = floatx4{0.f, 0.f, 0.f, 0.f};
    if (g.bias) p.bias = load_global_f4(g.bias + nb * 16 + (lane >> 4) * 4);
    const unsigned at = sh.rows[row].pos * (HD / 2) + (((nb * 16) % HD + (lane >> 4) * 4) >> 1);   // past the K heads: loaded, not used
    const float2 c = *reinterpret_cast<const float2 *>(g.cosv + at), sn = *reinterpret_cast<const float2 *>(g.sinv + at);
    p.v = floatx4{c.x, sn.x, c.y, sn.y};
    return p;
}
__device__ __forceinline__ void epi_resid_pre(const FastGemm &g, int row, bool live, int nb, int lane, floatx4 v, const EpiPre &pre) {
    const int n0 = nb * 16 + (lane >> 4) * 4;
    floatx4 hv = {0.f, 0.f, 0.f, 0.f};
    if (live) {
        hv = pre.v + v;
        st_f32x4<true>(g.h + (size_t)row * g.N + n0, hv);
    }
    float ssq = hv[0] * hv[0] + hv[1] * hv[1] + hv[2] * hv[2] + hv[3] * hv[3];
    ssq += __shfl_xor(ssq, 16, 64);
    ssq += __shfl_xor(ssq, 32, 64);
    if (live && (lane >> 4) == 0) st_f32<true>(g.ss_out + nb * 64 + row, ssq);
}
template <int HD>
__device__ __forceinline__ void epi_qkv_store(const FastGemm &g, const FusedShared &sh, int row, int nb, int lane, floatx4 v, const EpiPre &pre) {
    const int head = nb * 16 / HD, p0 = nb * 16 % HD + (lane >> 4) * 4;   // the head is the same for all lanes
    v += pre.bias;
    const RowMeta rm = sh.rows[row];
    if (!rm.live) return;
    if (head < g.hq + g.hkv) {
        const int i0 = p0 >> 1;  // packed columns 2i, 2i+1 are elements i and i + HD/2
        const float c0 = pre.v[0], s0 = pre.v[1], c1 = pre.v[2], s1 = pre.v[3];
        const float a0 = v[0] * c0 - v[1] * s0, b0 = v[1] * c0 + v[0] * s0;
        const float a1 = v[2] * c1 - v[3] * s1, b1 = v[3] * c1 + v[2] * s1;
        // i0 is even: elements i0, i0 + 1 are neighbours in either layout, 4-byte aligned
        bf16_t *d0, *d1;
        if (head < g.hq) {
            d0 = g.q + ((size_t)row * g.hq + head) * HD + i0;
            d1 = d0 + HD / 2;
        } else {
            d0 = rm.kv + kv_k_index(g.layer, rm.n_pages, rm.page, g.hkv, head - g.hq, rm.tin, i0, HD);
            d1 = rm.kv + kv_k_index(g.layer, rm.n_pages, rm.page, g.hkv, head - g.hq, rm.tin, i0 + HD / 2, HD);
        }
        st_u32<true>(d0, pack2_bf16(a0, a1));
        st_u32<true>(d1, pack2_bf16(b0, b1));
    } else {
        bf16_t *d = rm.kv + kv_v_index(g.layer, rm.n_pages, rm.page, g.hkv, head - g.hq - g.hkv, rm.tin, p0, HD);
#pragma unroll
        for (int i = 0; i < 4; ++i) {   // four dimensions of a key: 16 bytes apart
            const bf16_t x = (bf16_t)v[i];
            st_u16<true>(d + i * 8, __builtin_bit_cast(unsigned short, x));
        }
    }
}

// SwiGLU product in MFMA operand order (fragment (K block, row block), see xfrag_index).  v0, v1: tiles of the weight
// blocks nb (even) and nb + 1: a lane holds ffn columns f, f + 1 and f + 8, f + 9 of its row.
template <int NB>
__device__ __forceinline__ void epi_swiglu_frag(const FastGemm &g, int row, int nb, int lane, floatx4 v0, floatx4 v1) {
    bf16_t *out = g.a_out + xfrag_index(row, nb * 8, NB) + (lane >> 4) * 2;
    auto act = [](float gt, float up) { return gt / (1.0f + expf(-gt)) * up; };
    st_u32<true>(out, pack2_bf16(act(v0[0], v0[1]), act(v0[2], v0[3])));
    st_u32<true>(out + 128, pack2_bf16(act(v1[0], v1[1]), act(v1[2], v1[3])));
}

// Staging of a normalising phase: x = bf16(h * rstd * gain) of nk k-blocks of all rows, to LDS as [k-block][row][32].
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
    unsigned off[JP], out[JP];      // bytes: of the lane's piece j in a row's slice, and in the staged k-blocks (row 0)
    const float *h, *gain_p, *ss;
    int K, n_ss, m, chunks;
    float inv_d, eps;

    // columns of pieces seg * 64 JP ..: a slice of more than 64 JP pieces takes several passes over the rows
    __device__ __forceinline__ void columns(int seg, int lane) {
#pragma unroll
        for (int j = 0; j < JP; ++j) {
            const int c = min((seg * JP + j) * 64 + lane, chunks - 1);   // past the end: the last piece, written again
            off[j] = c * 16;
            out[j] = (c >> 3) * m * 64 + (c & 7) * 8;
            gain[j] = load_global_f4(gain_p + c * 4);
        }
    }
    // before the barrier.  h, gain: first column of the slice; K: stride of h; nk: k-blocks of the slice
    __device__ __forceinline__ void init(const FastGemm &g, int kb0, int nk, int lane) {
        h = g.Xh + (size_t)kb0 * 32;
        gain_p = g.gain + (size_t)kb0 * 32;
        ss = g.ss_in;
        K = g.KB * 32;
        n_ss = g.n_ss;
        m = g.m;
        chunks = nk * 8;
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
// ---- GEMM phase -------------------------------------------------------------------------------------
// Work items = (unit of UB weight blocks) x (K split); workgroup w takes items w, w + G, ...  G is
// a multiple of ks, so all items of a workgroup share one K slice and its activations are staged
// in LDS once.  The wavefronts split the slice into equal runs of `cnt` k-blocks (the last run may
// reach past the slice: those steps load a valid fragment again and multiply it by zero), and
// each streams its fragments through a ring of PD registers per weight block, refilled with the
// next item's fragments in the last round.  Trip counts are the same for every wavefront, so the
// loop has no divergent branches.  The caller has arrived at the grid barrier; this function
// waits on it after issuing the first loads.
template <int NB, int HD, int UB, int PD, int EPI>
__device__ __forceinline__ void gemm_phase(const FastGemm &g, const Items &im, GridBar &bar, unsigned char *smem,
                                  int lds_total, FusedShared &sh TRACE_ARG) {
    static_assert(EPI == EPI_SWIGLU || EPI == EPI_LOGITS, "gate/up and output head");
    constexpr int RW = FW / 2;               // wavefronts whose partial sums sit in LDS at a time
    constexpr int RED_BYTES = RW * 2 * NB * 1024;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));  // per-thread index math is redone per phase instead of living across all of them
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = g.m, KB = g.KB, NBt = g.N >> 4;
    const int n_my = im.n_my, split = im.split;
    const int kb0 = split * g.kbps, kb1 = min(KB, kb0 + g.kbps), nk = kb1 - kb0;
    const int cnt = (nk + FW - 1) / FW;          // k-blocks per wavefront, the same for all
    const int rounds = (cnt + PD - 1) / PD;
    const int wk0 = kb0 + wave * cnt;            // this wavefront's run: wk0 .. wk0 + cnt - 1, valid below kb1
    u32x4 *xs = reinterpret_cast<u32x4 *>(smem);
    floatx4 *red = reinterpret_cast<floatx4 *>(smem + lds_total - RED_BYTES);

    global_w_ptr wp[UB], wpn[UB];
    u32x4 w[PD][UB];
    // AHEAD: a second set of registers holds the first round of the item after next, so that two
    // items' worth of weights are requested before the barrier and during every item
    // slots of the second set; none with three row blocks, whose accumulators leave no room
    constexpr int A2 = (FUSED_AHEAD > 0 && UB == 2 && NB <= 2) ? (FUSED_AHEAD < PD ? FUSED_AHEAD : PD) : 0;
    constexpr bool AHEAD = A2 > 0;
    global_w_ptr wpa[UB];
    u32x4 w2[AHEAD ? A2 : 1][UB];
#pragma unroll
    for (int d = 0; d < PD; ++d)
#pragma unroll
        for (int u = 0; u < UB; ++u) w[d][u] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int d = 0; d < (AHEAD ? A2 : 1); ++d)
#pragma unroll
        for (int u = 0; u < UB; ++u) w2[d][u] = u32x4{0u, 0u, 0u, 0u};
    auto unit_ptrs = [&](int it, global_w_ptr (&dst)[UB]) {
        const int unit = im.unit0 + it * im.ustep;
#pragma unroll
        for (int u = 0; u < UB; ++u) dst[u] = (global_w_ptr)g.W + (size_t)min(unit * UB + u, NBt - 1) * KB * 64 + lane;
    };
    auto frag = [&](global_w_ptr base, int kbl) {
        return __builtin_nontemporal_load(base + (size_t)min(wk0 + kbl, kb1 - 1) * 64);
    };
    // Loads are never predicated: a step past the end of the run reads the run's last fragment again
    // (a cache hit) and its product is discarded.  Straight-line loads let the compiler wait for
    // exactly the fragment it needs instead of for everything in flight.
    auto first_fragments = [&]() {
        unit_ptrs(0, wp);
#pragma unroll
        for (int d = 0; d < PD; ++d)
#pragma unroll
            for (int u = 0; u < UB; ++u) w[d][u] = frag(wp[u], min(d, cnt - 1));
        if (AHEAD && n_my > 1) {
            unit_ptrs(1, wpa);
#pragma unroll
            for (int d = 0; d < A2; ++d)
#pragma unroll
                for (int u = 0; u < UB; ++u) w2[d][u] = frag(wpa[u], min(d, cnt - 1));
        }
    };
    NormStage<JP_OF(HD)> ns;
    if (n_my > 0) {
        ns.init(g, kb0, nk, lane);
        first_fragments();
    }
    TRACE(1);
    bar.wait();
    TRACE(2);
    if (n_my == 0) return;

    ns.run(smem, sh, lane, wave TRACE_PASS);
    lds_sync();
    TRACE(3);

    int xoff[NB];  // this lane's 16 bytes of row block c inside a k-block of the staged activations
#pragma unroll
    for (int c = 0; c < NB; ++c) {
        const int row = min(c * 16 + (lane & 15), m - 1);
        xoff[c] = row * 4 + (lane >> 4);
    }

    for (int it = 0; it < n_my; ++it) {
        const bool has_next = it + 1 < n_my;
        const bool has_ahead = AHEAD && it + 2 < n_my;
        unit_ptrs(has_next ? it + 1 : it, wpn);
        if (AHEAD) unit_ptrs(has_ahead ? it + 2 : it, wpa);
        const int unit = im.unit0 + it * im.ustep;
        const int nb0 = unit * UB;
        floatx4 acc[UB][NB];
#pragma unroll
        for (int u = 0; u < UB; ++u)
#pragma unroll
            for (int c = 0; c < NB; ++c) acc[u][c] = floatx4{0.f, 0.f, 0.f, 0.f};
        // One round = PD steps of straight-line code.  REFILL: after its use every slot is loaded
        // again, with the same item's next round or, in the last round, the next item's first; the
        // final round of the final item has nothing left to load and runs without.
        auto round_body = [&](auto refill_tag, int r) {
            constexpr bool REFILL = decltype(refill_tag)::value;
            const bool last_round = r + 1 == rounds;
            global_w_ptr rp[UB];
#pragma unroll
            for (int u = 0; u < UB; ++u) rp[u] = last_round ? wpn[u] : wp[u];
            const int rbase = last_round ? 0 : (r + 1) * PD;
            // activation fragments leave LDS FUSED_BB_AHEAD steps before the MFMAs that use them, so
            // that no MFMA waits for a read issued right in front of it
            constexpr int BA = FUSED_BB_AHEAD < PD ? FUSED_BB_AHEAD : PD - 1;
            bf16x8 bb[BA + 1][NB];
            auto read_bb = [&](int d) {
                const int kx = min(wk0 + min(r * PD + d, cnt - 1), kb1 - 1) - kb0;
#pragma unroll
                for (int c = 0; c < NB; ++c) bb[d % (BA + 1)][c] = __builtin_bit_cast(bf16x8, xs[kx * m * 4 + xoff[c]]);
            };
#pragma unroll
            for (int d = 0; d < BA; ++d) read_bb(d);
#pragma unroll
            for (int d = 0; d < PD; ++d) {
                const int kbl = r * PD + d;
                const bool live = kbl < cnt && wk0 + kbl < kb1;
                bf16x8 a[UB];
#pragma unroll
                for (int u = 0; u < UB; ++u) a[u] = __builtin_bit_cast(bf16x8, live ? w[d][u] : u32x4{0u, 0u, 0u, 0u});
                if (REFILL) {
                    if (AHEAD && d < A2 && last_round) {
                        // the next item's first round is already here; its slot takes the one after
#pragma unroll
                        for (int u = 0; u < UB; ++u) w[d][u] = w2[d][u];
                        if (has_ahead) {
#pragma unroll
                            for (int u = 0; u < UB; ++u) w2[d][u] = frag(wpa[u], min(d, cnt - 1));
                        }
                    } else {
#pragma unroll
                        for (int u = 0; u < UB; ++u) w[d][u] = frag(rp[u], min(rbase + d, cnt - 1));
                    }
                }
                if (d + BA < PD) read_bb(d + BA);
#pragma unroll
                for (int c = 0; c < NB; ++c) {
                    const bf16x8 b1 = bb[d % (BA + 1)][c];
#pragma unroll
                    for (int u = 0; u < UB; ++u)
                        acc[u][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], b1, acc[u][c], 0, 0, 0);
                }
            }
            // Order of the round's LDS reads and MFMAs for the instruction scheduler: the reads of
            // the first steps, then per step its MFMAs followed by the reads of a later step, so
            // that an MFMA never waits for a read issued right in front of it.
            if (FUSED_SGB > 0) {
                constexpr int SA = FUSED_SGB < PD ? FUSED_SGB : PD;
                __builtin_amdgcn_sched_group_barrier(0x100, SA * NB, 0);
#pragma unroll
                for (int d = 0; d < PD; ++d) {
                    __builtin_amdgcn_sched_group_barrier(0x008, UB * NB, 0);
                    if (d + SA < PD) __builtin_amdgcn_sched_group_barrier(0x100, NB, 0);
                }
            }
        };
#pragma unroll 1
        for (int r = 0; r + 1 < rounds; ++r) round_body(std::true_type{}, r);
        if (has_next) round_body(std::true_type{}, rounds - 1);
        else round_body(std::false_type{}, rounds - 1);
        TRACE(4);
        // ---- wavefront partial sums: upper half through LDS into the lower half, then all four ----
        // (the LDS reads of a stage are issued together, ahead of the first sum: the empty asm
        // statements keep the compiler from moving each read down to its use)
        if (wave >= RW) {
#pragma unroll
            for (int u = 0; u < UB; ++u)
#pragma unroll
                for (int c = 0; c < NB; ++c) red[(((wave - RW) * UB + u) * NB + c) * 64 + lane] = acc[u][c];
        }
        lds_sync();
        if (wave < RW) {
            floatx4 other[UB][NB];
#pragma unroll
            for (int u = 0; u < UB; ++u)
#pragma unroll
                for (int c = 0; c < NB; ++c) other[u][c] = red[((wave * UB + u) * NB + c) * 64 + lane];
            asm volatile("" ::: "memory");
#pragma unroll
            for (int u = 0; u < UB; ++u)
#pragma unroll
                for (int c = 0; c < NB; ++c) red[((wave * UB + u) * NB + c) * 64 + lane] = acc[u][c] + other[u][c];
        }
        lds_sync();

        constexpr int NT = UB * NB * 64;                       // tiles of 4 outputs per unit
        constexpr int NTH = EPI == EPI_SWIGLU ? NB * 64 : NT;  // tiles with an epilogue of their own
        static_assert(NTH <= FT, "one tile per thread");
        const int t = tid;
        floatx4 v0 = {0.f, 0.f, 0.f, 0.f}, v1 = {0.f, 0.f, 0.f, 0.f};
        if (t < NTH) {
            floatx4 p0[RW], p1[RW];
            if (EPI == EPI_SWIGLU) {
                const int c = t >> 6;
#pragma unroll
                for (int ww = 0; ww < RW; ++ww) {
                    p0[ww] = red[((ww * UB + 0) * NB + c) * 64 + lane];
                    p1[ww] = red[((ww * UB + (UB - 1)) * NB + c) * 64 + lane];
                }
            } else {
                const int u = t / (NB * 64), c = (t >> 6) % NB;
#pragma unroll
                for (int ww = 0; ww < RW; ++ww) {
                    p0[ww] = red[((ww * UB + u) * NB + c) * 64 + lane];
                    p1[ww] = floatx4{0.f, 0.f, 0.f, 0.f};
                }
            }
            asm volatile("" ::: "memory");
#pragma unroll
            for (int ww = 0; ww < RW; ++ww) {
                v0 += p0[ww];
                if (EPI == EPI_SWIGLU) v1 += p1[ww];
            }
        }
        bool do_epi = true;
        if (g.ks > 1) {
            float *mine = g.part + ((size_t)(unit * g.ks + split) * NT) * 4;
            if (t < NTH) {
                store_coherent(mine + (size_t)t * 4, v0);
                if (EPI == EPI_SWIGLU) store_coherent(mine + (size_t)(NTH + t) * 4, v1);
            }
            stores_done();
            __syncthreads();
            if (tid == 0) {
                const int old = __hip_atomic_fetch_add(g.counters + unit, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                sh.s_last = old == g.ks - 1;
                if (old == g.ks - 1) __hip_atomic_store(g.counters + unit, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __syncthreads();
            do_epi = sh.s_last != 0;
            if (do_epi && t < NTH) {
                v0 = floatx4{0.f, 0.f, 0.f, 0.f};
                v1 = floatx4{0.f, 0.f, 0.f, 0.f};
                for (int sp0 = 0; sp0 < g.ks; sp0 += 8) {
                    floatx4 t0[8], t1[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        t0[i] = floatx4{0.f, 0.f, 0.f, 0.f};
                        t1[i] = floatx4{0.f, 0.f, 0.f, 0.f};
                        if (sp0 + i < g.ks) {
                            const float *p = g.part + ((size_t)(unit * g.ks + sp0 + i) * NT) * 4;
                            t0[i] = load_coherent(p + (size_t)t * 4);
                            if (EPI == EPI_SWIGLU) t1[i] = load_coherent(p + (size_t)(NTH + t) * 4);
                        }
                    }
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        v0 += t0[i];
                        v1 += t1[i];
                    }
                }
            }
        }
        if (do_epi && t < NTH) {  // whole wavefronts: NTH is a multiple of 64
            const int u = EPI == EPI_SWIGLU ? 0 : t / (NB * 64), c = (t >> 6) % NB;
            const int nb = nb0 + u;
            const int row = c * 16 + (lane & 15);
            const bool live = row < m && nb < NBt;
            if (live) {
                if (EPI == EPI_SWIGLU) epi_swiglu_frag<NB>(g, row, nb, lane, v0, v1);
                else __builtin_nontemporal_store(v0, reinterpret_cast<floatx4 *>(g.logits + (size_t)row * g.N + nb * 16 + (lane >> 4) * 4));
            }
        }
        TRACE(5);
        if (has_next) {
            lds_sync();  // the partial sums in LDS are consumed before the next item's arrive
#pragma unroll
            for (int u = 0; u < UB; ++u) wp[u] = wpn[u];
        }
    }
}

// ---- sums over wavefronts and K splits -------------------------------------------------------------------
// red: partial tiles [tile][wavefront][lane].  Pairs (w, w + 4), then the four pairs in order.
__device__ __forceinline__ floatx4 sum_waves(const floatx4 *red, int tile, int lane) {
    floatx4 p[FW], v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < FW; ++i) p[i] = red[(tile * FW + i) * 64 + lane];
    asm volatile("" ::: "memory");   // all reads are issued before the first sum
#pragma unroll
    for (int i = 0; i < FW / 2; ++i) v += p[i] + p[i + FW / 2];
    return v;
}
// K splits of a tile meet: this split's sums go to part (of split 0; the next splits' at `stride` floats each), the
// last to count itself in adds all of them in split order.  True: v is the whole sum.
__device__ __forceinline__ bool meet_splits(floatx4 &v, float *part, int *counter, int split, int ks, int stride, int lane) {
    part += lane * 4;
    store_coherent(part + (size_t)split * stride, v);
    stores_done();
    int old = 0;
    if (lane == 0) old = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane(old) != ks - 1) return false;
    if (lane == 0) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    v = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int sp0 = 0; sp0 < ks; sp0 += 8) {
        floatx4 t[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i] = load_coherent(part + (size_t)min(sp0 + i, ks - 1) * stride);
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (sp0 + i < ks) v += t[i];
    }
    return true;
}

// ---- exchange of partial tiles ------------------------------------------------------------------------------
// K splits of a down projection tile, and key parts of an attention block, meet through memory that holds a mark
// (all bits set, which no sent value has) wherever nothing has been sent.  Each tile has an owner among the
// workgroups that share it; the others send theirs and go on, the owner reads until no mark is left, puts the marks
// back and goes on with the sum.  Against a counter that the last to arrive reads (store, wait for the store,
// increment with its round trip, read): the wait and the increment are gone from the chain, and the owners of
// different tiles work at the same time.
// Everyone who sends is resident and sends without waiting for anybody, so the wait ends; it is bounded like the
// grid barrier's all the same.  Attention and down projection together: 1.5B, 17 rows 1252 -> 1154 us a pass, 0.5B, 9
// rows 714 -> 674.
constexpr unsigned XCH_MARK = 0xffffffffu;
__device__ __forceinline__ void xch_send(float *slot, floatx4 v) {
    u32x4 r = __builtin_bit_cast(u32x4, v);
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = r[i] == XCH_MARK ? 0x7fc00000u : r[i];   // a NaN like any other
    st_f32x4<true>(slot, __builtin_bit_cast(floatx4, r));
}
// What parts 0 .. n - 1 (n >= 2) but `self` have sent: NV values a lane and part, value k of part i `at` + i * stride +
// k * 1024 bytes into the exchange.  t[i] of part `self` and of parts past the last is undefined.  A round of the wait
// is one round trip to memory and what its code costs: 16-byte loads past the caches (two of 8 bytes each before),
// and a maximum over the words instead of a comparison of each.
template <int MAXN, int NV>
__device__ __forceinline__ void xch_receive(floatx4 (&t)[MAXN][NV], float *xch, unsigned at, unsigned stride, int n, int self, int lane,
                                            unsigned *fail) {
    constexpr int AGENT = 16;   // cache policy of an agent-scope load
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(xch, 0, 0x7fffffff, 0x00027000);
    const int other = self == 0 ? 1 : 0;
    for (int spins = 0;;) {
        asm volatile("" ::: "memory");   // read again in every round
#pragma unroll
        for (int i = 0; i < MAXN; ++i)
#pragma unroll
            for (int k = 0; k < NV; ++k)
                t[i][k] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(
                                                          rsrc, lane * 16, at + (i < n && i != self ? i : other) * stride + k * 1024, AGENT));
        unsigned most = 0;
#pragma unroll
        for (int i = 0; i < MAXN; ++i)
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                const u32x4 r = __builtin_bit_cast(u32x4, t[i][k]);
                most = max(max(most, r[0]), max(r[1], max(r[2], r[3])));
            }
        if (!__any(most == XCH_MARK)) break;
        ++spins;
        if (spins > SPIN_LIMIT || ((spins & 1023) == 0 && __hip_atomic_load(fail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
            __hip_atomic_store(fail, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            break;
        }
    }
}
// Puts the marks back where this workgroup has received: tiles self, self + n, ... of `tiles`, NV values a lane.  Called
// behind the arrival at the grid barrier, when all wavefronts are done with the values; the next arrival waits for
// these stores, the next use is a phase or more behind that.  Not by the wavefront that polls the barrier: its polls
// would wait for the stores (1.5B, 17 rows: 1178 us a pass; marks put back at the end of the phase 1162; so 1154).
struct XchUsed { unsigned at, stride; int n, self, tiles; };   // at: of tile 0; n = 0: nothing received
template <int NV>
__device__ __forceinline__ void xch_clear(float *xch, const XchUsed &u) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), t = u.self + (FW - 1 - wave) * u.n;
    if (u.n < 2 || wave < 2 || t >= u.tiles) return;
    const floatx4 mark = __builtin_bit_cast(floatx4, u32x4{XCH_MARK, XCH_MARK, XCH_MARK, XCH_MARK});
    float *p = xch + (u.at + t * NV * 1024) / 4 + (threadIdx.x & 63) * 4;
    for (int i = 0; i < u.n; ++i)
        if (i != u.self)
#pragma unroll
            for (int k = 0; k < NV; ++k) st_f32x4<true>(p + (i * u.stride + k * 1024) / 4, mark);
}
// Sum of a tile over its K splits, in split order.
template <int MAXN>
__device__ __forceinline__ floatx4 xch_sum(floatx4 v, float *xch, unsigned at, unsigned stride, int n, int self, int lane, unsigned *fail) {
    floatx4 t[MAXN][1], sum = {0.f, 0.f, 0.f, 0.f};
    xch_receive<MAXN, 1>(t, xch, at, stride, n, self, lane, fail);
#pragma unroll
    for (int i = 0; i < MAXN; ++i)
        if (i < n) sum += i == self ? v : t[i][0];
    return sum;
}

// ---- QKV phase --------------------------------------------------------------------------------------------
// One 16-row weight block per item; the wavefronts share its K slice.  Few items a workgroup (one at the 0.5B and
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
    const int kb0 = im.split * g.kbps, kb1 = min(KB, kb0 + g.kbps), nk = kb1 - kb0;
    const int cnt = (nk + FW - 1) / FW, rounds = (cnt + PD - 1) / PD;
    const int wk0 = kb0 + wave * cnt, mine = min(cnt, kb1 - wk0);   // k-blocks wk0 .. wk0 + mine - 1 (none: mine <= 0)
    floatx4 *red = reinterpret_cast<floatx4 *>(smem + lds_total - FW * NB * 1024);
    const int row = wave * 16 + (lane & 15);   // wavefront c < NB finishes the tile of row block c
    global_w_ptr W = (global_w_ptr)g.W;

    u32x4 w[PD];
#pragma unroll
    for (int d = 0; d < PD; ++d) w[d] = u32x4{0u, 0u, 0u, 0u};
    auto load_w = [&](int unit, int d, int kbl) {   // never predicated: see resid_phase
        w[d] = __builtin_nontemporal_load(W + ((size_t)unit * KB + min(wk0 + min(kbl, cnt - 1), kb1 - 1)) * 64 + lane);
    };
    NormStage<JP> ns;
    EpiPre pre;
    pre.v = pre.bias = floatx4{0.f, 0.f, 0.f, 0.f};
    if (im.n_my > 0) {
        ns.init(g, kb0, nk, lane);
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
                const int kx = min(wk0 + min(r * PD + d, cnt - 1), kb1 - 1) - kb0;
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
            floatx4 v = sum_waves(red, wave, lane);
            bool whole = true;
            if (g.ks > 1) whole = meet_splits(v, g.part + ((size_t)unit * g.ks * NB + wave) * 256, g.counters + unit * NB + wave, im.split, g.ks, NB * 256, lane);
            if (whole && row < m) epi_qkv_store<HD>(g, sh, row, unit, lane, v, pre);
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
// Items: (unit of UB weight blocks) x (K split), as in gemm_phase.  The splits of a unit exchange their sums tile by
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
#ifndef FUSED_ATT_TOP
#define FUSED_ATT_TOP 1         // attention items go to the workgroups at the top of the grid
#endif
#ifndef FUSED_GU_LIGHT
#define FUSED_GU_LIGHT 1        // gate/up: workgroups busy in the O projection take one unit, the others share the rest
#endif
#ifndef FUSED_GU_REV
#define FUSED_GU_REV 1          // gate/up: the units of a partial last range go to the workgroups at the top of the grid
#endif
#ifndef FUSED_WAVE_PHASES
#define FUSED_WAVE_PHASES 1     // 1: gate/up and the output head run this way when K is not split across workgroups
#endif
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
                    const int idx = FUSED_GU_REV ? G - 1 - wg : wg;
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
    ns.init(g, 0, KB, lane);
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
                if (row < m) epi_swiglu_frag<NB>(g, row, nb & ~1, lane, t4[0] + t4[1], t4[2] + t4[3]);
            }
#pragma unroll
            for (int c = 0; c < NB; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
        TRACE(5);
    }
}

// ---- attention phase -----------------------------------------------------------------------------------
// Work item = (block of 16 query items, kv head, sequence, part of the keys); a query item is a
// (row, head of the group) pair.  The eight wavefronts of a workgroup take the 32-key tiles of the
// part in turn; K and V^T fragments go from the cache straight into registers in MFMA operand
// order (no LDS staging: every fragment is used by exactly one wavefront).  Scores
// S^T[key, item] = K Q^T leave the MFMA with eight keys per lane once the K rows are fed in the
// order 8*(rho >> 2) + (rho & 3) (+ 4 for the second 16-key block): that is the B-operand layout
// of O^T[d, item] += V^T[d, key] P[key, item], and the matching V^T fragment is one 16-byte load.
// Wavefront results (running max, sum, O^T) are merged through LDS; with several parts the
// merged partials go to memory and the last workgroup to arrive merges the parts.  No second
// grid-wide phase is needed for the merge.
constexpr int FKT = ATT_TILE;  // keys per tile

// (sequence, kv head, query block, key part) of attention work item i
struct AttItem { int seq, kvh, qb, part, blk; };
__device__ __forceinline__ AttItem att_item(const FusedArgs &a, const Batch &b, int i) {
    const int group = a.hq / a.hkv;
    AttItem it;
    it.part = i / a.att_blocks;
    it.blk = i % a.att_blocks;
    int blk = it.blk, seq = 0;
    while (seq + 1 < b.n_seqs) {
        const int nb_seq = a.hkv * ((b.s[seq].nrows * group + 15) >> 4);
        if (blk < nb_seq) break;
        blk -= nb_seq;
        ++seq;
    }
    const int nqb = (b.s[seq].nrows * group + 15) >> 4;
    it.seq = seq;
    it.kvh = blk / nqb;
    it.qb = blk % nqb;
    return it;
}

// len0: length of the sequence of this workgroup's first item, read once per launch (lengths do
// not change during a launch).
template <int NB, int HD>
__device__ __forceinline__ XchUsed attn_phase(const FusedArgs &a, const Batch &b, int layer, const bf16_t *q, bf16_t *o,
                                  int len0, GridBar &bar, unsigned char *smem, FusedShared &sh TRACE_ARG) {
    XchUsed used{0, 0, 0, 0, 0};
    constexpr int KD = HD / 32, DB = HD / 16, MAXP = FUSED_MAXP;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    // the wavefront's number as a scalar: which tile it takes, and whether that tile holds keys of
    // this launch, are then decided by scalar branches
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g4 = lane >> 4, l15 = lane & 15;
    const int G = gridDim.x, hq = a.hq, hkv = a.hkv, group = hq / hkv, P = a.att_parts;
    floatx4 *o_s = reinterpret_cast<floatx4 *>(smem);                      // [wave][db][lane]
    float *ml_s = reinterpret_cast<float *>(smem + FW * DB * 64 * 16);    // [wave][2][16]
    const int n_work = a.att_blocks * P;
    AttTile<HD> tile;
    auto tile_range = [&](const SeqDesc &s, const AttItem &it, int len, int &t_begin, int &t_end, int &kmax) {
        kmax = min(len + s.nrows, s.capacity);  // keys 0..kmax-1 exist
        const int blk_last = min(kmax - 1, len + min(s.nrows - 1, (it.qb * 16 + 15) / group));
        const int tiles = blk_last / FKT + 1, tpp = (tiles + P - 1) / P;
        t_begin = it.part * tpp;
        t_end = min(tiles, t_begin + tpp);
    };
    // keys below the sequence length were written by earlier calls: a first tile made of them is
    // loaded before the barrier wait
    bool preloaded = false;
    const int i_first = a.att_first[blockIdx.x];
    if (i_first >= 0) {
        const AttItem it = att_item(a, b, i_first);
        int t_begin, t_end, kmax;
        tile_range(b.s[it.seq], it, len0, t_begin, t_end, kmax);
        const int t = t_begin + wave;
        if (t < t_end && (t + 1) * FKT <= len0) {
            tile.load(b.s[it.seq], layer, hkv, it.kvh, t, false, lane);
            preloaded = true;
        }
    }
    TRACE(1);
    bar.wait();
    TRACE(2);
    // further items (more work than workgroups; then there is one part per block) follow in steps of G
    for (int i = i_first; i >= 0 && i < n_work; i += G) {
        const AttItem it = att_item(a, b, i);
        const SeqDesc &s = b.s[it.seq];
        const int kvh = it.kvh, part = it.part;
        const int n_items = s.nrows * group;
        const int len = i == i_first ? len0 : s.state[0];
        int t_begin, t_end, kmax;
        tile_range(s, it, len, t_begin, t_end, kmax);
        const int item = it.qb * 16 + l15;
        const bool valid = item < n_items;
        const int r = valid ? item / group : 0, head = kvh * group + (valid ? item % group : 0);
        const int row = s.row0 + r;
        const int last_key = valid ? len + r : -1;
        // a value every lane shares (kernel argument and the item's sequence length)
        const int own_base = a.tree_anc ? __builtin_amdgcn_readfirstlane(len) : ATT_NO_TREE;
        const tree_mask_t own_mask = a.tree_anc && valid ? a.tree_anc[row] : 0;

        bf16x8 qf[KD];
#pragma unroll
        for (int kd = 0; kd < KD; ++kd)
            qf[kd] = __builtin_bit_cast(bf16x8, ssa_load_16(q + ((size_t)row * hq + head) * HD + kd * 32 + g4 * 8));
        AttState<HD> st;
#pragma unroll
        for (int db = 0; db < DB; ++db) st.o[db] = floatx4{0.f, 0.f, 0.f, 0.f};
        st.m_run = -1e30f;
        st.l_run = 0.f;
#pragma unroll 1
        for (int t = t_begin + wave; t < t_end; t += FW) {
            const int t0 = t * FKT;
            if (!preloaded) tile.load(s, layer, hkv, kvh, t, (t + 1) * FKT > len, lane);
            preloaded = false;
            tile.mask_values(t0, kmax, lane);
            att_tile_update<HD>(st, qf, tile, t0, last_key, own_base, own_mask, a.scale_log2e, lane);
        }
        preloaded = false;
        TRACE(20);
        // ---- merge of the eight wavefronts through LDS ----
        if (i != i_first) lds_sync();  // the previous item's merge has been read
#pragma unroll
        for (int db = 0; db < DB; ++db) o_s[(wave * DB + db) * 64 + lane] = st.o[db];
        if (g4 == 0) {
            ml_s[(wave * 2 + 0) * 16 + l15] = st.m_run;
            ml_s[(wave * 2 + 1) * 16 + l15] = st.l_run;
        }
        lds_sync();
        // thread (db = wave, lane) owns O^T[d = 16*db + 4*g4 + j][item l15]; HD = 64 leaves waves 4..7 idle
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
        float M = -1e30f, L = 0.f;
        if (wave < DB) {
            // all LDS reads of the merge are issued together, ahead of the arithmetic
            float mw[FW], lw[FW];
            floatx4 ow[FW];
#pragma unroll
            for (int w = 0; w < FW; ++w) {
                mw[w] = ml_s[(w * 2) * 16 + l15];
                lw[w] = ml_s[(w * 2 + 1) * 16 + l15];
                ow[w] = o_s[(w * DB + wave) * 64 + lane];
            }
            asm volatile("" ::: "memory");
#pragma unroll
            for (int w = 0; w < FW; ++w) M = fmaxf(M, mw[w]);
#pragma unroll
            for (int w = 0; w < FW; ++w) {
                const float wt = exp2f(mw[w] - M);
                L += lw[w] * wt;
                acc += ow[w] * wt;
            }
        }
        TRACE(21);
        if (P > 1) {
            // The parts of a block exchange their results: d-block db is put together by part db % P, whose wavefront
            // db has the other parts' O tiles and (max, sum) pairs sent to it.
            const unsigned at = (unsigned)(it.blk * P * DB + wave) * 2048, stride = DB * 2048;
            used = XchUsed{at - wave * 2048, stride, P, part, DB};
            if (wave < DB && wave % P != part) {
                float *slot = a.xch + (at + part * stride) / 4 + lane * 4;
                xch_send(slot, acc);
                xch_send(slot + 256, floatx4{M, L, 0.f, 0.f});
            } else if (wave < DB) {
                floatx4 t[MAXP][2];
                xch_receive<MAXP, 2>(t, a.xch, at, stride, P, part, lane, a.fail);
                TRACE(22);
                float Mg = M;
#pragma unroll
                for (int pp = 0; pp < MAXP; ++pp) Mg = pp < P && pp != part ? fmaxf(Mg, t[pp][1][0]) : Mg;
                float Lg = 0.f;
                floatx4 og = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int pp = 0; pp < MAXP; ++pp) {
                    if (pp < P) {
                        const float wt = exp2f((pp == part ? M : t[pp][1][0]) - Mg);
                        Lg += (pp == part ? L : t[pp][1][1]) * wt;
                        og += (pp == part ? acc : t[pp][0]) * wt;
                    }
                }
                if (valid) {
                    const float inv = 1.0f / Lg;
                    st_u32x2<true>(o + xfrag_index(row, head * HD + wave * 16 + g4 * 4, NB),
                                   pack4_bf16(og[0] * inv, og[1] * inv, og[2] * inv, og[3] * inv));
                }
            }
        } else if (wave < DB && valid) {
            const float inv = 1.0f / L;
            st_u32x2<true>(o + xfrag_index(row, head * HD + wave * 16 + g4 * 4, NB),
                           pack4_bf16(acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv));
        }
    }
    return used;
}

#ifndef FUSED_MINW
#define FUSED_MINW 2
#endif
template <int NB, int HD>
__global__ __launch_bounds__(FT, FUSED_MINW) void verify_fused_kernel(FusedArgs a, Batch b) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ FusedShared sh;
#ifdef FUSED_ARRIVALS
    // debug build: stamps go behind the first 64 rows of the logits buffer (the model workspace's, when the caller passes none)
    GridBar bar{a.bar, a.fail, a.root0, gridDim.x / BAR_COUNTERS, false,
                reinterpret_cast<unsigned long long *>(a.logits + (size_t)64 * a.vocab), 0, 0};
#else
    GridBar bar{a.bar, a.fail, a.root0, gridDim.x / BAR_COUNTERS, false};
#endif
    const int d = a.d, F = a.F, hd = a.hd, nq = a.hq * hd, nkv = a.hkv * hd;
    const size_t hstride = (size_t)FROWS * d, sstride = (size_t)(d / 16) * 64;

#ifdef FUSED_TRACE
    Trace trace{reinterpret_cast<unsigned long long *>(a.bar + 8192), 0};
#endif
    // length of the sequence of this workgroup's first attention item (lengths are constant during a launch)
    int len0 = 0;
    if (a.att_first[blockIdx.x] >= 0) len0 = b.s[att_item(a, b, a.att_first[blockIdx.x]).seq].state[0];
    if ((int)threadIdx.x < FROWS) {
        const int row = min((int)threadIdx.x, a.m - 1);
        const SeqDesc &s = b.s[find_seq(b, row)];
        const int len = s.state[0], slot = len + (row - s.row0);
        RowMeta rm;
        rm.kv = reinterpret_cast<bf16_t *>(s.kv);
        rm.n_pages = s.n_pages;
        rm.live = slot >= 0 && slot < s.capacity;
        rm.page = rm.live ? kv_page(s, slot) : 0;
        rm.tin = rm.live ? slot % VF_TILE : 0;
        rm.pos = rm.live ? (a.tree_depth ? len + a.tree_depth[row] : slot) : 0;
        sh.rows[threadIdx.x] = rm;
    }
    TRACE(0);
    embed_phase(a, b);
    bar.arrive();   // (a workgroup barrier inside: the row table is visible to every wavefront from here on)

    FastGemm base;
    base.m = a.m;
    base.part = a.part;
    base.counters = a.counters;
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

    const Items it_qkv = items_of((nq + 2 * nkv) / 16, a.ks_qkv), it_o = items_of(d / 16, 1);
    const Items it_gu = items_of(F / 16, a.ks_gu), it_down = items_of((d / 16 + a.down_ub - 1) / a.down_ub, a.ks_down);
    const int kbps_down = (F / 32 + a.ks_down - 1) / a.ks_down;

#pragma unroll 1
    for (int l = 0; l < a.n_layers; ++l) {
        // kernel arguments and a multiple of the layer's number: addresses that the scalar unit forms, no load
        FusedLayer lp = a.layer0;
        const size_t lo = (size_t)l * a.layer_bytes;
        auto at_layer = [&](auto &p) { p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(reinterpret_cast<uintptr_t>(p) + lo); };
        at_layer(lp.wqkv); at_layer(lp.wo); at_layer(lp.wgu); at_layer(lp.wd);
        at_layer(lp.attn_norm); at_layer(lp.ffn_norm); at_layer(lp.bqkv);
        float *h0 = a.hv + (size_t)(2 * l) * hstride, *h1 = h0 + hstride, *h2 = h1 + hstride;
        float *ss0 = a.ssv + (size_t)(2 * l) * sstride, *ss1 = ss0 + sstride, *ss2 = ss1 + sstride;
        bf16_t *q = a.qv + (size_t)l * FROWS * nq, *o = a.ov + (size_t)l * FROWS * nq;
        bf16_t *act = a.av + (size_t)l * FROWS * F;
        {
            FastGemm g = base;
            g.W = lp.wqkv; g.N = nq + 2 * nkv; g.KB = d / 32; g.Xh = h0; g.gain = lp.attn_norm; g.ss_in = ss0;
            g.bias = a.has_bias ? lp.bqkv : nullptr; g.layer = l; g.q = q;
            g.ks = a.ks_qkv; g.kbps = (g.KB + g.ks - 1) / g.ks;
            qkv_phase<NB, HD, JP_OF(HD)>(g, it_qkv, bar, smem, a.lds_total, sh TRACE_PASS);
        }
        bar.arrive();
        TRACE(10);
        const XchUsed att_used = attn_phase<NB, HD>(a, b, l, q, o, len0, bar, smem, sh TRACE_PASS);
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
            g.ks = a.ks_gu; g.kbps = (g.KB + g.ks - 1) / g.ks;
            if (a.wave_gu) wave_phase<NB, HD, EPI_SWIGLU>(g, a.gu_light, bar, smem, a.lds_total, sh TRACE_PASS);
            else gemm_phase<NB, HD, 2, 6, EPI_SWIGLU>(g, it_gu, bar, smem, a.lds_total, sh TRACE_PASS);
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
        g.ks = a.ks_head; g.kbps = (g.KB + g.ks - 1) / g.ks;
        if (a.wave_head) wave_phase<NB, HD, EPI_LOGITS>(g, 0, bar, smem, a.lds_total, sh TRACE_PASS);
        else gemm_phase<NB, HD, 2, 6, EPI_LOGITS>(g, items_of((a.vocab / 16 + 1) / 2, a.ks_head), bar, smem, a.lds_total, sh TRACE_PASS);
    }
    TRACE(99);
#ifdef FUSED_ARRIVALS
    if (threadIdx.x == 0) bar.stamps[((size_t)bar.n_arr * 2) * gridDim.x + blockIdx.x] = wall_clock64();  // end of the head phase
#endif
}

// ---- host side -------------------------------------------------------------------------------------

// Largest K slice (in 32-wide blocks) whose activations fit LDS next to the partial sums.
int slice_limit(int lds_total, int rows, int nb) {
    const int x_bytes = lds_total - (FW / 2) * 2 * nb * 1024;
    return x_bytes / (rows * 64);
}

// K split of a phase that stages its activations: the smallest divisor of G whose slice fits LDS (workgroup w takes
// items w, w + G, ...: they share a K slice if ks divides G).  0: nothing fits.
int pick_split(int G, int lds_total, int KB, int rows, int nb) {
    const int lim = slice_limit(lds_total, rows, nb);
    for (int ks = 1; ks <= G && ks <= KB; ++ks) {
        const int kbps = (KB + ks - 1) / ks;
        if (G % ks == 0 && (KB + kbps - 1) / kbps == ks && kbps <= lim) return ks;   // every split owns k-blocks
    }
    return 0;
}
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

template <int NB, int HD>
int launch_fused(vf_model *m, FusedArgs &a, const Batch &b, int G, hipStream_t st) {
    auto kern = verify_fused_kernel<NB, HD>;
    static int max_wgs = -1;  // workgroups that can be resident at once
    if (max_wgs < 0) {
        VF_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   LDS_BYTES));
        int per_cu = 0, dev = 0;
        hipDeviceProp_t prop;
        VF_HIP(hipGetDevice(&dev));
        VF_HIP(hipGetDeviceProperties(&prop, dev));
        VF_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(kern), FT, LDS_BYTES));
        max_wgs = per_cu * prop.multiProcessorCount;
    }
    if (G > max_wgs)
        return vf_fail(VF_ERR_UNSUPPORTED, "persistent kernel: %d workgroups wanted, %d can be resident", G, max_wgs);
    hipLaunchKernelGGL(kern, dim3(G), dim3(FT), a.lds_total, st, a, b);
    VF_LAUNCH_CHECK("verify_fused");
    return VF_OK;
}

}  // namespace

// One work item per workgroup sends: the tiles of a down projection item, or the d-blocks of an attention part with
// their (max, sum) pairs.
static size_t xch_bytes(const vf_config &c) { return (size_t)FUSED_G * std::max(2 * (FROWS / 16), c.head_dim / 16 * 2) * 1024; }

size_t vf_fused_workspace_bytes(const vf_config &c) {
    if (c.dtype != VF_BF16) return 0;
    const size_t L = c.n_layers, d = c.d_model, nq = (size_t)c.n_q_heads * c.head_dim, F = c.d_ffn;
    size_t n = 0;
    auto add = [&](size_t bytes) { n += (bytes + 255) & ~(size_t)255; };
    add((2 * L + 1) * FROWS * d * 4);
    add((2 * L + 1) * (d / 16) * 64 * 4);
    add(L * FROWS * nq * 2);
    add(L * FROWS * nq * 2);
    add(L * FROWS * F * 2);
    add(xch_bytes(c));
    add(65536);
    return n;
}

int vf_fused_init(vf_model *m, char *ws, hipStream_t st) {
    const vf_config &c = m->cfg;
    const size_t L = c.n_layers, d = c.d_model, nq = (size_t)c.n_q_heads * c.head_dim, F = c.d_ffn;
    size_t off = 0;
    auto take = [&](size_t bytes) { char *p = ws + off; off += (bytes + 255) & ~(size_t)255; return p; };
    m->fz_h = (float *)take((2 * L + 1) * FROWS * d * 4);
    m->fz_ss = (float *)take((2 * L + 1) * (d / 16) * 64 * 4);
    m->fz_q = take(L * FROWS * nq * 2);
    m->fz_o = take(L * FROWS * nq * 2);
    m->fz_a = take(L * FROWS * F * 2);
    m->fz_xch = (float *)take(xch_bytes(c));
    VF_HIP(hipMemsetAsync(m->fz_xch, 0xff, xch_bytes(c), st));   // marks everywhere
    m->fz_bar = (unsigned *)take(65536);
    // the kernel addresses the parameters of layer l as those of layer 0 plus l times one distance
    for (size_t l = 1; l < L; ++l) {
        const LayerPacked &x = m->layers[l - 1], &y = m->layers[l], &z = m->layers[0], &o = m->layers[1];
        auto same = [](const void *a, const void *b, const void *c, const void *d) { return (const char *)b - (const char *)a == (const char *)d - (const char *)c; };
        if (!same(x.wqkv, y.wqkv, z.wqkv, o.wqkv) || !same(x.wo, y.wo, z.wqkv, o.wqkv) || !same(x.wgu, y.wgu, z.wqkv, o.wqkv) ||
            !same(x.wd, y.wd, z.wqkv, o.wqkv) || !same(x.attn_norm, y.attn_norm, z.wqkv, o.wqkv) ||
            !same(x.ffn_norm, y.ffn_norm, z.wqkv, o.wqkv) || !same(x.bqkv, y.bqkv, z.wqkv, o.wqkv))
            return vf_fail(VF_ERR_ARG, "persistent kernel: layers at unequal distances");
    }
    VF_HIP(hipStreamSynchronize(st));   // a model is ready for any stream once it is created
    m->fz_epoch = 0;
    return VF_OK;
}

// Whether the persistent kernel can run this call; fills the grid size, LDS size and K splits.
// K splits of the six GEMM phases for a call of `rows` rows (nb blocks of 16), and the floats of
// partial-sum workspace they need.  false: some phase does not fit.
struct Splits { int qkv, gu, down, down_ub, head; };
static bool plan_splits(const vf_config &c, int rows, int nb, Splits *sp, size_t *part_floats) {
    const int d = c.d_model, F = c.d_ffn, hd = c.head_dim, nq = c.n_q_heads * hd, nkv = c.n_kv_heads * hd;
    if (c.dtype != VF_BF16 || rows > FROWS || d % 64) return false;
    if (std::max(std::max((nq + 2 * nkv) / 16, F / 16), (c.vocab / 16 + 1) / 2) > VF_N_COUNTERS) return false;
    const int G = FUSED_G, lds = LDS_BYTES;
    if (G % BAR_COUNTERS) return false;
    sp->qkv = pick_split(G, lds, d / 32, rows, nb);
    sp->gu = pick_split(G, lds, d / 32, rows, nb);
    // one weight block an item where that still gives three splits or more: a narrow model's items of two blocks need
    // nine splits to fill the chip, and an owner waits for all of them (0.5B, 1 row: 632 us a pass, with four 601)
    sp->down_ub = d / 16 * 3 <= G ? 1 : 2;
    sp->down = fill_split(G, (d / 16 + sp->down_ub - 1) / sp->down_ub, F / 32);
    sp->head = pick_split(G, lds, d / 32, rows, nb);
    if (!sp->qkv || !sp->gu || !sp->head) return false;
    // a counter per tile of a split unit
    if ((nq + 2 * nkv) / 16 * nb > VF_N_COUNTERS) return false;
    // partial tiles of the split phases: units * ks tiles of UB * NB * 256 floats
    size_t tiles = std::max((nq + 2 * nkv) / 16 * sp->qkv, F / 16 * sp->gu);
    if (sp->head > 1) tiles = std::max(tiles, (size_t)((c.vocab / 16 + 1) / 2) * sp->head);
    *part_floats = tiles * 2 * nb * 256;
    return true;
}

// Partial-sum workspace (floats) the persistent kernel may ask for with this model, over all row counts.
size_t vf_fused_part_floats(const vf_config &c) {
    size_t need = 0;
    for (int nb = 1; nb * 16 <= FROWS; ++nb) {
        if (c.max_rows < (nb - 1) * 16 + 1) break;
        // the most rows a call of nb blocks can have: the smallest K slices, the most splits
        Splits sp;
        size_t pf = 0;
        if (plan_splits(c, std::min(nb * 16, (int)c.max_rows), nb, &sp, &pf)) need = std::max(need, pf);
    }
    return need;
}

static bool plan_fused(const vf_model *m, const Batch &b, FusedArgs &a, int *G_out) {
    if (!m->fz_h) return false;
    const int rows = b.total_rows, nb = (rows + 15) / 16;
    Splits sp;
    size_t pf = 0;
    if (!plan_splits(m->cfg, rows, nb, &sp, &pf) || pf > m->part_floats) return false;
    a.ks_qkv = sp.qkv;
    a.ks_gu = sp.gu;
    a.ks_down = sp.down;
    a.down_ub = sp.down_ub;
    a.ks_head = sp.head;
    a.lds_total = LDS_BYTES;
    *G_out = FUSED_G;
    return true;
}

bool vf_fused_ok(const vf_model *m, const Batch &b) {
    FusedArgs a;
    int G;
    return plan_fused(m, b, a, &G);
}

int vf_run_fused(vf_model *m, const Batch &b, const int32_t *tokens, float *logits_out, bool tree, hipStream_t st) {
    const vf_config &c = m->cfg;
    FusedArgs a;
    memset(&a, 0, sizeof a);
    int G = 0;
    if (!plan_fused(m, b, a, &G)) return vf_fail(VF_ERR_UNSUPPORTED, "persistent kernel does not apply to this call");
    int max_keys = 0;
    for (int i = 0; i < b.n_seqs; ++i) max_keys = std::max(max_keys, b.s[i].len_ub + b.s[i].nrows);
    // attention: blocks of 16 query items per (sequence, kv head); as many key parts per block as
    // fill the grid, but no more than give every wavefront of a part a tile of its own
    const int group = c.n_q_heads / c.n_kv_heads;
    int blocks = 0;
    for (int i = 0; i < b.n_seqs; ++i) blocks += c.n_kv_heads * ((b.s[i].nrows * group + 15) / 16);
    int parts = std::max(1, std::min(G / std::max(1, blocks), ((max_keys + FKT - 1) / FKT + FW - 1) / FW));
    parts = std::min(parts, FUSED_MAXP);
    if (blocks * parts > FUSED_G) parts = 1;  // the exchange has room for one item per workgroup
    const LayerPacked &l0 = m->layers[0];
    a.layer0 = FusedLayer{(const u32x4 *)l0.wqkv, (const u32x4 *)l0.wo, (const u32x4 *)l0.wgu, (const u32x4 *)l0.wd, l0.attn_norm, l0.ffn_norm, l0.bqkv};
    a.layer_bytes = c.n_layers > 1 ? (unsigned long long)((char *)m->layers[1].wqkv - (char *)l0.wqkv) : 0;
    a.embed = (const bf16_t *)m->embed;
    a.lm_head = (const u32x4 *)m->lm_head;
    a.final_norm = m->final_norm;
    a.cosv = m->rope_cos;
    a.sinv = m->rope_sin;
    a.tree_depth = tree ? m->tree_depth : nullptr;
    a.tree_anc = tree ? m->tree_anc : nullptr;
    a.tokens = tokens;
    a.hv = m->fz_h;
    a.ssv = m->fz_ss;
    a.qv = (bf16_t *)m->fz_q;
    a.ov = (bf16_t *)m->fz_o;
    a.av = (bf16_t *)m->fz_a;
    a.xch = m->fz_xch;
    a.part = m->part;
    a.counters = m->counters;
    a.bar = m->fz_bar;
    a.fail = m->fz_bar + 8000;
    a.logits = logits_out;
    a.n_layers = c.n_layers;
    a.d = c.d_model;
    a.F = c.d_ffn;
    a.hq = c.n_q_heads;
    a.hkv = c.n_kv_heads;
    a.hd = c.head_dim;
    a.vocab = c.vocab;
    a.m = b.total_rows;
    a.att_blocks = blocks;
    a.att_parts = parts;
    {
        // item = part * blocks + block, block = (sequence, kv head, query block) in that order
        const int n_work = blocks * parts;
        for (int w = 0; w < FUSED_G; ++w) a.att_first[w] = (short)(w < n_work && n_work > G ? w : -1);
        if (n_work <= G) {
            // from the top of the grid downwards: the QKV phase before it keeps the lowest workgroups busy
            // (one item each), and a workgroup that is idle there has worked out its attention item and
            // requested its first key tile by the time the others arrive
            int next[8], die = 0;
            for (int x = 0; x < 8; ++x) next[x] = FUSED_ATT_TOP ? G - 8 + x : x;
            int blk0 = 0;
            for (int sq = 0; sq < b.n_seqs; ++sq) {
                const int nqb = (b.s[sq].nrows * group + 15) / 16;
                for (int kvh = 0; kvh < c.n_kv_heads; ++kvh)
                    for (int p = 0; p < parts; ++p) {
                        for (int qb = 0; qb < nqb; ++qb) {
                            int x = die;
                            for (int tries = 0; tries < 8 && (next[x] >= G || next[x] < 0); ++tries) x = (x + 1) % 8;  // that die is full
                            a.att_first[next[x]] = (short)(p * blocks + blk0 + kvh * nqb + qb);
                            next[x] += FUSED_ATT_TOP ? -8 : 8;
                        }
                        die = (die + 1) % 8;
                    }
                blk0 += c.n_kv_heads * nqb;
            }
        }
    }
    a.has_bias = c.qkv_bias;
    a.inv_d = 1.0f / (float)c.d_model;
    a.eps = c.rms_eps;
    a.scale_log2e = 1.4426950408889634f / sqrtf((float)c.head_dim);
    a.root0 = m->fz_epoch;
    m->fz_epoch += (1u + 5u * (unsigned)c.n_layers) * (unsigned)(G / BAR_COUNTERS);  // barriers per launch x arrivals per counter
    const int rows = b.total_rows;
    {
        const bool fits = FUSED_WAVE_PHASES && (size_t)(c.d_model / 32) * rows * 64 + wave_tail_bytes((rows + 15) / 16) <= (size_t)LDS_BYTES;
        a.wave_gu = fits && a.ks_gu == 1;
        {
            // one unit for each workgroup of the O projection, if the others can take the rest in at most
            // three units each (two passes)
            const int n_o = c.d_model / 16, units = c.d_ffn / 16, H = G - n_o;
            a.gu_light = (FUSED_GU_LIGHT && n_o > 0 && H > 0 && n_o < units && units - n_o <= 3 * H && units - n_o > H) ? n_o : 0;
        }
        a.wave_head = fits && a.ks_head == 1;
    }
    ProfScope ps(m, VF_SITE_STEP, st);
    if (c.head_dim == 128) {
        if (rows <= 16) return launch_fused<1, 128>(m, a, b, G, st);
        if (rows <= 32) return launch_fused<2, 128>(m, a, b, G, st);
        return launch_fused<3, 128>(m, a, b, G, st);
    }
    if (rows <= 16) return launch_fused<1, 64>(m, a, b, G, st);
    if (rows <= 32) return launch_fused<2, 64>(m, a, b, G, st);
    return launch_fused<3, 64>(m, a, b, G, st);
}

// Whether any barrier of an earlier launch gave up (the stream must be idle).
int vf_fused_check(vf_model *m) {
    if (!m->fz_bar) return VF_OK;
    unsigned flag = 0;
    VF_HIP(hipMemcpy(&flag, m->fz_bar + 8000, 4, hipMemcpyDeviceToHost));
    if (flag) {
        // counters are out of step now: start over from zero
        VF_HIP(hipMemset(m->fz_bar, 0, 65536));
        VF_HIP(hipMemset(m->counters, 0, VF_N_COUNTERS * 4));
        VF_HIP(hipMemset(m->fz_xch, 0xff, xch_bytes(m->cfg)));
        m->fz_epoch = 0;
        return vf_fail(VF_ERR_HIP, "persistent verify kernel: a grid barrier timed out; results of that call are invalid");
    }
    return VF_OK;
}

#ifdef FUSED_ARRIVALS
// Copies the arrival / release stamps of the last launch (logits left in the model workspace): [barrier][2][workgroup].
extern "C" int vf_debug_arrivals(vf_model *m, unsigned long long *out_host, int n_barriers) {
    VF_HIP(hipDeviceSynchronize());
    VF_HIP(hipMemcpy(out_host, m->logits + (size_t)64 * m->cfg.vocab, (size_t)n_barriers * 2 * FUSED_G * 8, hipMemcpyDeviceToHost));
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
