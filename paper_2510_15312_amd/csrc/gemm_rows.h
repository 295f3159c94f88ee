// GEMM kernels for many rows (a prefill chunk, a large verify batch): Y[rows, N] = X[rows, K] * W[N, K]^T,
// both operands in 1 KB MFMA fragments (vf_internal.h).  Two shapes of kernel; gemm.hip picks.
//
// What bounds them (measured with parts taken out, gate/up of the 1.5B shape, 256 x 17920 x 1536): the
// matrix instructions, the weight stream from HBM and the activation fragments from the L2 (every column
// tile reads all of X) take about the same time each, so each has to run under the others; and with few
// workgroups the weight bytes in flight set the stream's rate (140 workgroups of a 256 x 128 tile: 2 TB/s).
//
//   gemm_stream_kernel (wide matrices, up to a few hundred rows): a tile covers 16 * CW * WMB rows and a
//   few weight blocks, so that the column tiles fill the chip once.  A producer wavefront keeps a deep
//   ring of weight fragments filled with direct loads to LDS; the compute wavefronts stack up over the
//   rows, keep their own activation fragments in registers several k-blocks ahead, and all take the
//   weights from the ring.  Gate/up of the 1.5B shape in a prefill (17920 x 1536, SwiGLU): 256 rows 27 -> 21.5
//   us, 128 rows 27 -> 16.7 (before: a 256 x 128 tile, two k-blocks of weights ahead in registers).
//   What is left at 256 rows, with operands made hot in copies: 6 us of weights from HBM, 2 of activations from the L2;
//   the stream alone takes 9.5 us of the 20, products alone 7, and the two overlap little.
//
//   gemm_tile_kernel (square tiles, K splits): both operands go through an LDS ring of S stages of one
//   k-block, filled by direct loads S - 1 k-blocks ahead; fragments leave LDS one k-block ahead of their
//   products, and a step's LDS reads and load requests are spread between its matrix instructions
//   (requests in front of them left the matrix pipes idle for their address arithmetic: 102 -> 90 us on
//   1024 x 16384 x 3072).
#pragma once

#include "fast_common.h"
#include "lds_stream.h"

namespace {

constexpr int ROWS_EPI_PARTIAL = 0, ROWS_EPI_SWIGLU = 1, ROWS_EPI_TOPK = 2, ROWS_EPI_QKV = 3;

struct RowsGemm {
    const u32x4 *W, *X;
    float *out;              // PARTIAL: [ks][ld_rows][N]; SWIGLU: a in activation layout; TOPK: candidate values
    int N, KB, ncb;          // output columns, k-blocks, 16-row blocks of X
    int row_lo, row_hi, ld_rows;
    int kb_per_split, nx, ny;  // k-blocks per split, column tiles, row tiles; workgroups = nx * ny * splits
    int32_t *cand_i;
    int topk;
};
struct RowsGemmQkv : RowsGemm {
    QkvColumns e;             // cosv, sinv: by row of the call
    const RowPlace *place;
};
template <int EPI> using RowsArgs = std::conditional_t<EPI == ROWS_EPI_QKV, RowsGemmQkv, RowsGemm>;
// QKV: where a wavefront's rows go and, of tiles of up to five blocks a wavefront, the rotary angles of its first row block:
// requested behind the first activations, ahead of the products (behind those each is a memory round trip, in front of
// the activations these wait).
template <int EPI, int WNB, int WMB> struct RowsQkv {
    __device__ __forceinline__ void request(const RowsGemm &, int, int, int) {}
};
template <int WNB, int WMB> struct RowsQkv<ROWS_EPI_QKV, WNB, WMB> {
    static constexpr bool EARLY = WNB * WMB <= 5;
    u32x4 place[WMB][2];
    QkvAngles an[2][WNB];
    static __device__ __forceinline__ int row_of(const RowsGemmQkv &p, int cb0, int c, int lane) { return min((cb0 + c) * 16 + (lane & 15), p.row_hi - 1); }
    __device__ __forceinline__ void request_angles(const RowsGemmQkv &p, int nb0, int cb0, int c, int lane) {
#pragma unroll
        for (int n = 0; n < WNB; ++n) an[c & 1][n] = qkv_angles(p.e, row_of(p, cb0, c, lane), min(nb0 + n, (p.N >> 4) - 1), lane >> 4);
    }
    __device__ __forceinline__ void request(const RowsGemmQkv &p, int nb0, int cb0, int lane) {
#pragma unroll
        for (int c = 0; c < WMB; ++c)
#pragma unroll
            for (int i = 0; i < 2; ++i) place[c][i] = reinterpret_cast<const u32x4 *>(p.place + row_of(p, cb0, c, lane))[i];
        if constexpr (EARLY) request_angles(p, nb0, cb0, 0, lane);
    }
    __device__ __forceinline__ QkvPlace at(const RowsGemmQkv &p, int c, int lane) const {
        const u32x4 a = place[c][0], b = place[c][1];
        return qkv_place(p.e, {(unsigned long long)a[1] << 32 | a[0], (unsigned long long)a[3] << 32 | a[2], (int)b[0], (int)b[1], 0, 0}, lane >> 4);
    }
};

// Workgroup -> (row tile, column tile, split).  Neighbours in the order (split, column tile, row tile)
// share a compute die, so that its L2 serves all but the first reader of a weight tile.
__device__ __forceinline__ void rows_tile(const RowsGemm &p, int &ty, int &tx, int &split) {
    const int l = die_order(blockIdx.x, gridDim.x);
    ty = l % p.ny;
    tx = (l / p.ny) % p.nx;
    split = l / (p.ny * p.nx);
}

// silu(g) * u as the other SwiGLUs compute it: expf and the division know what a gate past e^88 gives.  The
// hardware's exp2 and reciprocal by hand instead: 1 % of a prefill's time (16.79 ms for 16.95, 2048 tokens at 1.5B),
// a third more error (mean 0.70 units of 2^-24 for 0.52, gates of -20 to -1), and the overflow to deal with.
__device__ __forceinline__ float silu_mul(float g, float u) { return g / (1.0f + expf(-g)) * u; }

// Epilogue of one wavefront: acc[n][c] is the tile of weight block nb0 + n and row block cb0 + c; a lane
// holds Y[row = 16 cb + (lane & 15)][16 nb + 4 (lane >> 4) + 0..3].
//   PARTIAL: float32 sums of this K split.
//   SWIGLU : gate row f is column 2 f and up row f column 2 f + 1 of the packed matrix, so a lane holds
//            two (gate, up) pairs: a = bf16(silu(gate) * up), columns 8 nb + 2 (lane >> 4) + 0..1.  Written through:
//            workgroups of all dies write four bytes of the same lines, and what is left in a die's L2 has to be
//            written back before the next kernel starts (down behind it, 256 rows of 1.5B, 17.6 -> 17.4 us).  Partial sums,
//            whose lines have one writer, and norms lose by it what the kernel behind them gains.
//   QKV    : bias, rotary embedding, q rows and the cache's keys and values (qkv_store): a lane's four
//            columns are its unit.
//   TOPK   : per row, the topk largest of the wavefront's 16 WNB columns with their ids, in falling order,
//            equal values by rising id, as list `list` of n_lists.  The four lanes that share a row run one
//            round per result: every lane offers its best remaining value, two shuffles pick the row's.
template <int EPI, int WNB, int WMB>
__device__ __forceinline__ void rows_epilogue(const RowsArgs<EPI> &p, RowsQkv<EPI, WNB, WMB> &qkv, const floatx4 (&acc)[WNB][WMB], int nb0,
                                              int cb0, int split, int list, int n_lists, int lane) {
    const int NBt = p.N >> 4, g4 = lane >> 4;
    if constexpr (EPI == ROWS_EPI_SWIGLU) {
        unsigned *a_out = reinterpret_cast<unsigned *>(p.out);
#pragma unroll
        for (int c = 0; c < WMB; ++c) {
            const int cb = cb0 + c, row = cb * 16 + (lane & 15);
            if (row < p.row_lo || row >= p.row_hi) continue;
#pragma unroll
            for (int n = 0; n < WNB; ++n) {
                const int nb = nb0 + n;
                if (nb >= NBt) break;
                const floatx4 v = acc[n][c];
                typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
                const bf16x2 o = {(bf16_t)silu_mul(v[0], v[1]), (bf16_t)silu_mul(v[2], v[3])};
                st_u32<true>(a_out + (((size_t)(nb >> 2) * p.ncb + cb) * 64 + ((nb & 3) << 4) + (lane & 15)) * 4 + g4, __builtin_bit_cast(unsigned, o));
            }
        }
    } else if constexpr (EPI == ROWS_EPI_QKV) {
        // the next row block's angles are on their way while one is stored
        if constexpr (!RowsQkv<EPI, WNB, WMB>::EARLY) qkv.request_angles(p, nb0, cb0, 0, lane);
#pragma unroll
        for (int c = 0; c < WMB; ++c) {
            if (c + 1 < WMB) qkv.request_angles(p, nb0, cb0, c + 1, lane);
            const int row = (cb0 + c) * 16 + (lane & 15);
            if (row < p.row_lo || row >= p.row_hi) continue;
            const QkvPlace at = qkv.at(p, c, lane);
#pragma unroll
            for (int n = 0; n < WNB; ++n) {
                if (nb0 + n >= NBt) break;
                qkv_store(p.e, at, qkv.an[c & 1][n], row, nb0 + n, g4, acc[n][c]);
            }
        }
    } else if constexpr (EPI == ROWS_EPI_TOPK) {
        constexpr int NV = WNB * 4;
        float *cand_v = p.out;
        auto first_of = [](float av, int ai, float bv, int bi) { return av > bv || (av == bv && ai < bi); };
#pragma unroll
        for (int c = 0; c < WMB; ++c) {
            const int row = (cb0 + c) * 16 + (lane & 15);
            const bool store = g4 == 0 && row >= p.row_lo && row < p.row_hi;
            const size_t o = ((size_t)row * n_lists + list) * p.topk;
            float v[NV];   // this lane's values of the row; columns past N cannot win
#pragma unroll
            for (int e = 0; e < NV; ++e) v[e] = nb0 + e / 4 < NBt ? acc[e / 4][c][e % 4] : -INFINITY;
            const int id0 = nb0 * 16 + g4 * 4;  // id of element e: id0 + 16 * (e / 4) + e % 4
#pragma unroll 1
            for (int r = 0; r < p.topk; ++r) {
                float bv = -INFINITY;
                int bi = 0x7fffffff;
#pragma unroll
                for (int e = 0; e < NV; ++e) {
                    const int id = id0 + 16 * (e / 4) + e % 4;
                    if (v[e] != -INFINITY && first_of(v[e], id, bv, bi)) { bv = v[e]; bi = id; }
                }
#pragma unroll
                for (int off = 16; off <= 32; off <<= 1) {
                    const float ov = __shfl_xor(bv, off, 64);
                    const int oi = __shfl_xor(bi, off, 64);
                    if (first_of(ov, oi, bv, bi)) { bv = ov; bi = oi; }
                }
#pragma unroll
                for (int e = 0; e < NV; ++e)   // the lane that owns the winner retires it
                    if (id0 + 16 * (e / 4) + e % 4 == bi) v[e] = -INFINITY;
                if (store) {
                    cand_v[o + r] = bv;
                    p.cand_i[o + r] = bi == 0x7fffffff ? -1 : bi;
                }
            }
        }
    } else {
        float *out = p.out + (size_t)split * p.ld_rows * p.N;
#pragma unroll
        for (int n = 0; n < WNB; ++n) {
            const int nb = nb0 + n;
            if (nb >= NBt) break;
#pragma unroll
            for (int c = 0; c < WMB; ++c) {
                const int row = (cb0 + c) * 16 + (lane & 15);
                if (row >= p.row_lo && row < p.row_hi)
                    *reinterpret_cast<floatx4 *>(out + (size_t)row * p.N + nb * 16 + g4 * 4) = acc[n][c];
            }
        }
    }
}

// CW compute wavefronts of WMB row blocks each and one producer; NB weight blocks per tile; activation
// fragments D k-blocks ahead; weight ring of SW slots of KS k-blocks (one barrier per slot).
template <int CW, int WMB, int NB, int D, int KS, int SW, int EPI>
__global__ __launch_bounds__((CW + 1) * 64) VF_MFMA_KERNEL void gemm_stream_kernel(RowsArgs<EPI> p) {
    static_assert(D % 2 == 0 && D % KS == 0, "register sets and LDS slots line up with the unrolled loop");
    static_assert((SW - 2) * NB * KS < 64, "the wait counter counts to 63");
    extern __shared__ __align__(1024) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int ty, tx, split;
    rows_tile(p, ty, tx, split);
    const int nb0 = tx * NB, cb0 = (p.row_lo >> 4) + ty * (CW * WMB);
    const int kb_begin = split * p.kb_per_split, nk = min(p.KB, kb_begin + p.kb_per_split) - kb_begin;
    if (nk <= 0) return;
    const unsigned lane_off = lane * 16;
    if (wave == CW) {
        // producer: slot t has landed before barrier t; slot t - 1 has been read by every wavefront then
        const unsigned lds0 = lds_address(smem);
        const int NBt = p.N >> 4, ns = (nk + KS - 1) / KS;
        const char *src[NB];
#pragma unroll
        for (int n = 0; n < NB; ++n) src[n] = (const char *)p.W + ((size_t)min(nb0 + n, NBt - 1) * p.KB + kb_begin) * 1024;
        auto issue_as = [&](int s, int slot, auto once) {
            static_for<0, KS>([&](auto h) {
                const unsigned kb = min(s * KS + (int)h, nk - 1);   // past the end: the last k-block again, not used
                static_for<0, NB>([&](auto n) {
                    fragment_to_lds<((int)h * NB + (int)n) * 1024, decltype(once)::value>(src[n] + (size_t)kb * 1024, lane_off,
                                                                                          lds0 + (unsigned)slot * (KS * NB * 1024));
                });
            });
        };
        // weights that no other row tile reads are not kept (a prompt of 777 tokens of 0.5B in chunks of 128 6466 -> 6411 us)
        auto issue = [&](int s, int slot) {
            if (p.ny == 1) issue_as(s, slot, std::true_type{});
            else issue_as(s, slot, std::false_type{});
        };
        const int first = min(SW - 1, ns);
        for (int s = 0; s < first; ++s) issue(s, s);
        int slot = SW - 1;
        for (int t = 0; t < ns; ++t) {
            stage_wait<SW - 2, NB * KS>(ns - 1 - t);
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (t + SW - 1 < ns) issue(t + SW - 1, slot);
            slot = slot + 1 == SW ? 0 : slot + 1;
        }
        return;
    }
    // the wavefront's activation fragments: a uniform base that advances one k-block per fetch, and a
    // fixed offset per row block (rows past the call: a valid block, result dropped)
    const char *xbase = (const char *)p.X + (size_t)kb_begin * p.ncb * 1024;
    unsigned xoff[WMB];
#pragma unroll
    for (int c = 0; c < WMB; ++c) xoff[c] = (unsigned)min(cb0 + wave * WMB + c, p.ncb - 1) * 1024u + lane_off;
    const unsigned xstride = (unsigned)p.ncb * 1024u;
    int xleft = nk - 1;
    floatx4 acc[NB][WMB];
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int c = 0; c < WMB; ++c) acc[n][c] = floatx4{0.f, 0.f, 0.f, 0.f};
    u32x4 x[D][WMB];
    bf16x8 w[2][NB];
    auto fetch = [&](u32x4 (&r)[WMB]) {
#pragma unroll
        for (int c = 0; c < WMB; ++c) r[c] = *reinterpret_cast<const u32x4 *>(xbase + xoff[c]);
        xbase += xleft > 0 ? xstride : 0u;   // past the end: the last k-block again, not used
        --xleft;
    };
    int slot = 0;
    auto read = [&](bf16x8 (&f)[NB], int h) {   // weight fragments of k-block h of the current slot
        if (h == 0) lds_sync();
        const unsigned char *st = smem + slot * (KS * NB * 1024) + lane_off;
#pragma unroll
        for (int n = 0; n < NB; ++n) f[n] = *reinterpret_cast<const bf16x8 *>(st + (h * NB + n) * 1024);
        if (h == KS - 1) slot = slot + 1 == SW ? 0 : slot + 1;
    };
    auto mma = [&](const bf16x8 (&f)[NB], const u32x4 (&r)[WMB]) {
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int c = 0; c < WMB; ++c)
                acc[n][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[n], __builtin_bit_cast(bf16x8, r[c]), acc[n][c], 0, 0, 0);
    };
    // In order: the compiler's wait at the top of the loop is the stricter of what the loop and what these need.  Rearranged,
    // x[0] came last and every D k-blocks waited until one load of all that were in flight was left (777 tokens of 0.5B in
    // chunks of 128 6332 -> 6243 us, 1900 of 3B in chunks of 1024 15315 -> 15059, 2048 of 1.5B in chunks of 256 the same).
#pragma unroll
    for (int d = 0; d < D; ++d) {
        fetch(x[d]);
        __builtin_amdgcn_sched_barrier(0);
    }
    RowsQkv<EPI, NB, WMB> qkv;
    qkv.request(p, nb0, cb0 + wave * WMB, lane);
    read(w[0], 0);
    const int groups = (nk - 1) / D;
    for (int g = 0; g < groups; ++g) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            read(w[(d + 1) & 1], (d + 1) % KS);
            mma(w[d & 1], x[d]);
            fetch(x[d]);
            // the LDS reads go out first, then the products, then the next activation loads
            __builtin_amdgcn_sched_group_barrier(0x100, NB, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, NB * WMB, 0);
            __builtin_amdgcn_sched_group_barrier(0x020, WMB, 0);
        }
    }
    const int t = groups * D;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        if (t + d < nk) {
            if (t + d + 1 < nk) read(w[(d + 1) & 1], (d + 1) % KS);
            mma(w[d & 1], x[d]);
        }
    }
    rows_epilogue<EPI, NB, WMB>(p, qkv, acc, nb0, cb0 + wave * WMB, split, tx, p.nx, lane);
}

// Tile of MB row blocks x NB weight blocks, WM x WN wavefronts, ring of S stages of one k-block.
template <int MB, int NB, int WM, int WN, int S, int EPI>
__global__ __launch_bounds__(WM *WN * 64) VF_MFMA_KERNEL void gemm_tile_kernel(RowsArgs<EPI> p) {
    constexpr int NW = WM * WN, WMB = MB / WM, WNB = NB / WN, FR = MB + NB, LPW = FR / NW, NR = WMB + WNB, NM = WMB * WNB;
    static_assert(FR % NW == 0 && MB % WM == 0 && NB % WN == 0 && (S & (S - 1)) == 0, "tile shape");
    extern __shared__ __align__(1024) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM, NBt = p.N >> 4;
    int ty, tx, split;
    rows_tile(p, ty, tx, split);
    const int nb0 = tx * NB, cb0 = (p.row_lo >> 4) + ty * MB;
    const int kb_begin = split * p.kb_per_split, nk = min(p.KB, kb_begin + p.kb_per_split) - kb_begin;
    if (nk <= 0) return;
    const unsigned lds0 = lds_address(smem) + wave * LPW * 1024;
    const char *src[LPW];   // this wavefront's share of a stage: fragments of X first, then of W
    unsigned stride[LPW];
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
        const int f = wave * LPW + i;
        if (f < MB) {
            src[i] = (const char *)p.X + ((size_t)kb_begin * p.ncb + min(cb0 + f, p.ncb - 1)) * 1024;
            stride[i] = (unsigned)p.ncb * 1024u;
        } else {
            src[i] = (const char *)p.W + ((size_t)min(nb0 + f - MB, NBt - 1) * p.KB + kb_begin) * 1024;
            stride[i] = 1024u;
        }
    }
    const unsigned lane_off = lane * 16;
    struct Frags { bf16x8 a[WNB], b[WMB]; };
    floatx4 acc[WNB][WMB];
#pragma unroll
    for (int n = 0; n < WNB; ++n)
#pragma unroll
        for (int c = 0; c < WMB; ++c) acc[n][c] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto read1 = [&](Frags &f, const unsigned char *st, auto ii) {
        constexpr int i = decltype(ii)::value;
        if constexpr (i < WMB) f.b[i] = *reinterpret_cast<const bf16x8 *>(st + (wm * WMB + i) * 1024);
        else f.a[i - WMB] = *reinterpret_cast<const bf16x8 *>(st + (MB + wn * WNB + i - WMB) * 1024);
    };
    auto mma1 = [&](const Frags &f, auto ii) {
        constexpr int i = decltype(ii)::value, n = i / WMB, c = i % WMB;
        acc[n][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[n], f.b[c], acc[n][c], 0, 0, 0);
    };
    int left = nk - 1;   // k-blocks the sources still advance; past the end the last one is loaded again, not used
    auto issue1 = [&](unsigned buf, auto ii) {
        constexpr int i = decltype(ii)::value;
        fragment_to_lds<i * 1024>(src[i], lane_off, lds0 + buf);
        src[i] += left > 0 ? stride[i] : 0u;
    };
    // Step s: stage s + 1 has landed everywhere behind the barrier and stage s has left LDS, so its
    // buffer takes stage s + S while stage s + 1 is read and stage s multiplied.
    auto step = [&](Frags &cur, Frags &nxt, int s) {
        vm_wait<(S - 2) * LPW>();
        lds_sync();
        const unsigned char *st = smem + ((s + 1) & (S - 1)) * (FR * 1024) + lane_off;
        const unsigned buf = (unsigned)((s & (S - 1)) * FR) * 1024u;
        static_for<0, LPW>([&](auto qq) {
            constexpr int q = decltype(qq)::value;
            __builtin_amdgcn_sched_barrier(0);
            static_for<NR * q / LPW, NR *(q + 1) / LPW>([&](auto i) { read1(nxt, st, i); });
            static_for<NM * q / LPW, NM *(q + 1) / LPW>([&](auto i) { mma1(cur, i); });
            issue1(buf, qq);
        });
        --left;
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int s = 0; s < S; ++s) {
        static_for<0, LPW>([&](auto i) { issue1((unsigned)(s * FR) * 1024u, i); });
        --left;
    }
    RowsQkv<EPI, WNB, WMB> qkv;
    qkv.request(p, nb0 + wn * WNB, cb0 + wm * WMB, lane);
    Frags f0, f1;
    vm_wait<(S - 1) * LPW>();
    lds_sync();
    static_for<0, NR>([&](auto i) { read1(f0, smem + lane_off, i); });
    int s = 0;
    for (; s + 2 <= nk; s += 2) {
        step(f0, f1, s);
        step(f1, f0, s + 1);
    }
    if (s < nk) static_for<0, NM>([&](auto i) { mma1(f0, i); });
    vm_wait<0>();   // nothing is on its way to LDS when the workgroup ends
    rows_epilogue<EPI, WNB, WMB>(p, qkv, acc, nb0 + wn * WNB, cb0 + wm * WMB, split, tx * WN + wn, p.nx * WN, lane);
}

}  // namespace
