// Projections of the verify pass: Y[R][N] = X[R][K] * W[N][K]^T.
//
// With R = B*(k+1) block rows (88 at batch 8, k = 10) every weight is used R times, far
// below the ~312 flop/byte ridge of MI355X, so these GEMMs are bound by streaming W from
// HBM once.  The tuned kernel therefore treats W as the operand that must never be
// re-read: each consumer wave loads its W tiles straight from global memory into MFMA
// A-operand registers (W is pre-tiled so that a wave load is 1 KB contiguous), while the
// small X block (in the same order) is brought into LDS by producer waves and shared by the consumers.
// Operands are float16 (weights converted exactly from bfloat16 when the model is created,
// activations rounded to float16 by their producers); v_mfma_f32_16x16x32_f16 accumulates
// in float32.  Small-N projections are split along K across workgroups; the float32 partial
// tiles are summed by the consumer kernel in a fixed order (deterministic, no atomics).
// With hundreds of block rows (large k, large batches, prompt blocks) the same projections
// become compute-bound and go to a second kernel, k_gemm_dma below, that tiles for operand
// reuse and feeds both operands through LDS with direct-to-LDS loads.
#include "cs_common.h"
#include <type_traits>

// -------------------------------------------------------------------------------------
// float32 kernel (float32 models, and any model on the plain kernels)
//
// Small models: launch and load latency bound it, not the matrix rate (o and down of a 256-wide model, 11 rows:
// 87 us with a wave per W row that walked K 64 scalars at a time, 5 us now).  A workgroup owns 16 W rows
// by 16*NT block rows; its eight waves take the 16-wide pieces of K in turn, two pieces of loads in
// flight each, straight into the operands of v_mfma_f32_16x16x4_f32 (float32 products and sums; lane l
// holds row l % 16, and element j of its four is k = 4 * (l / 16) + j in both operands).  The instruction
// rounds after each of its four products, so an accumulator is one chain of them: a wave keeps eight, for
// chains of K / 64 products, and all partial sums are added in pairs, those of the waves through LDS.
// Error against float64, N(0, 1) operands: 7.7e-8 at K = 256, 1.6e-7 at 4096, as with 64 lanes of K / 64 products
// each (one chain of K / 8 per wave: 1.2e-7, 4.1e-7).  Two row tiles and two pieces ahead leave room for two
// workgroups on a compute unit, four and four for one (4096 x 4096, 300 rows: 214 us, as much with four and
// four; 128256 x 256, 65 rows: 158 against 279).  VEC: K % 4 == 0 and both operands aligned to four elements;
// otherwise the same kernel loads single elements.
// -------------------------------------------------------------------------------------
// X given as the residual stream and what its RMSNorm needs (blocks of few rows, see cs_gemm_few_rows).
struct cs_norm_in {
    const float* x;         // [R][K] residual stream
    const float* gain;      // [K]
    const float* ss;        // [nss][row tiles of 16] pieces of every row's sum of squares
    int nss;
    float eps;
    int32_t* flags;
};

#define GF_WAVES 8
template <bool VEC, typename T>
__device__ __forceinline__ f32x4 gf_load4(const T* __restrict__ row, int k, int K, bool live) {
    f32x4 v = (f32x4){0.f, 0.f, 0.f, 0.f};
    if constexpr (VEC) {
        if (live && k < K) {
            if constexpr (sizeof(T) == 4) {
                v = *reinterpret_cast<const f32x4*>(row + k);
            } else {
                const bf16x4 t = *reinterpret_cast<const bf16x4*>(row + k);
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = (float)t[j];
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (live && k + j < K) v[j] = cs_ld(row, k + j);
    }
    return v;
}

// Few rows (see cs_gemm_few_rows) have modes of their own, so that a layer of a small model is six launches, not nine:
// GF_NORM reads X through the RMSNorm of the residual stream (GF_SWIGLU as well, with a gate and an up tile per
// workgroup and SwiGLU of both as the result), GF_RESIDUAL adds to the residual stream and leaves the sums of squares.
enum { GF_STORE = 0, GF_NORM = 1, GF_SWIGLU = 2, GF_RESIDUAL = 3 };
template <typename WT, int NT, bool VEC, int MODE>
__global__ __launch_bounds__(64 * GF_WAVES) void k_gemm_f32(const float* __restrict__ X,
                                                            const WT* __restrict__ W, float* __restrict__ Y,
                                                            int R, int N, int K, cs_norm_in nrm, float* __restrict__ ss) {
    constexpr int AHEAD = 2;                      // pieces of K in flight per wave
    constexpr bool XN = MODE == GF_NORM || MODE == GF_SWIGLU;
    constexpr int MT = MODE == GF_SWIGLU ? 2 : 1; // 16-row W tiles
    __shared__ __attribute__((aligned(16))) f32x4 red[GF_WAVES][MT][NT][64];
    __shared__ __attribute__((aligned(16))) float sq[XN ? GF_WAVES : 1][16 * NT];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lrow = lane & 15, g = lane >> 4;
    const int n0 = blockIdx.x * 16 * MT, r0 = blockIdx.y * 16 * NT;
    bool w_live[MT];
    const WT* __restrict__ w[MT];
    constexpr int CHAINS = 4 * AHEAD;             // accumulators of a wave per tile pair
    bool x_live[NT];
    const float* x[NT];
    f32x4 acc[CHAINS][MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int n = n0 + mt * 16 + lrow;
        w_live[mt] = n < N;
        w[mt] = W + (int64_t)(w_live[mt] ? n : 0) * K;
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int r = r0 + nt * 16 + lrow;
        x_live[nt] = r < R;
        x[nt] = X + (int64_t)(x_live[nt] ? r : 0) * K;
#pragma unroll
        for (int c = 0; c < CHAINS; ++c)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[c][mt][nt] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    float scale[NT];
    if constexpr (XN) {
        f32x4 q = (f32x4){0.f, 0.f, 0.f, 0.f};
        for (int i = threadIdx.x; i < 4 * NT * nrm.nss; i += 64 * GF_WAVES) q += *reinterpret_cast<const f32x4*>(nrm.ss + 4 * i);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int o = 4 * NT; o < 64; o <<= 1) q[j] += __shfl_xor(q[j], o, 64);
        if (lane < 4 * NT) *reinterpret_cast<f32x4*>(&sq[wave][4 * lane]) = q;
        __syncthreads();
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            float t = 0.f;
#pragma unroll
            for (int u = 0; u < GF_WAVES; ++u) t += sq[u][nt * 16 + lrow];
            scale[nt] = x_live[nt] ? 1.0f / sqrtf(t / (float)K + nrm.eps) : 0.f;
        }
    }
    for (int k0 = 16 * wave; k0 < K; k0 += AHEAD * 16 * GF_WAVES) {
        f32x4 a[AHEAD][MT], b[AHEAD][NT], gn[AHEAD];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const int k = k0 + u * 16 * GF_WAVES + 4 * g;          // (pieces past K are zeros)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) a[u][mt] = gf_load4<VEC>(w[mt], k, K, w_live[mt]);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) b[u][nt] = gf_load4<VEC>(x[nt], k, K, x_live[nt]);
            if constexpr (XN) gn[u] = gf_load4<VEC>(nrm.gain, k, K, true);
        }
        if constexpr (XN) {
#pragma unroll
            for (int u = 0; u < AHEAD; ++u)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) b[u][nt] = b[u][nt] * scale[nt] * gn[u];
        }
#pragma unroll
        for (int u = 0; u < AHEAD; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        f32x4& o = acc[4 * u + j][mt][nt];
                        o = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][mt][j], b[u][nt][j], o, 0, 0, 0);
                    }
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
            for (int h = CHAINS / 2; h > 0; h /= 2)
#pragma unroll
                for (int c = 0; c < h; ++c) acc[c][mt][nt] += acc[c + h][mt][nt];
            red[wave][mt][nt][lane] = acc[0][mt][nt];
        }
    __syncthreads();
    if (wave >= NT) return;
    // wave nt sums row tile nt: y[mt][j] = Y[row r0 + nt*16 + lrow][col n0 + mt*16 + 4g + j]
    f32x4 y[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        f32x4 part[GF_WAVES];
#pragma unroll
        for (int u = 0; u < GF_WAVES; ++u) part[u] = red[u][mt][wave][lane];
#pragma unroll
        for (int h = GF_WAVES / 2; h > 0; h /= 2)
#pragma unroll
            for (int u = 0; u < h; ++u) part[u] += part[u + h];
        y[mt] = part[0];
    }
    const int r = r0 + wave * 16 + lrow;
    if constexpr (MODE == GF_SWIGLU) {
        if (r >= R) return;
        const int F = N / 2, f = n0 / 2 + 4 * g;  // 16 gate rows, then the 16 up rows of the same channels
#pragma unroll
        for (int j = 0; j < 4; ++j) Y[(int64_t)r * F + f + j] = y[0][j] / (1.0f + expf(-y[0][j])) * y[1][j];
    } else if constexpr (MODE == GF_RESIDUAL) {
        float q = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (r < R && n0 + 4 * g + j < N) {
                float* __restrict__ o = Y + (int64_t)r * N + n0 + 4 * g + j;
                const float v = *o + y[0][j];
                *o = v;
                q += v * v;
            }
        q += __shfl_xor(q, 16, 64);
        q += __shfl_xor(q, 32, 64);
        if (g == 0) ss[blockIdx.x * 16 * NT + wave * 16 + lrow] = q;
    } else {
        if (r >= R) return;
        float* __restrict__ out = Y + (int64_t)r * N + n0 + 4 * g;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (n0 + 4 * g + j < N) out[j] = y[0][j];
    }
}

template <typename WT, int MODE>
static int launch_f32(const float* X, const WT* W, float* Y, int R, int N, int K, const cs_norm_in& nrm, float* ss,
                      hipStream_t s) {
    const bool vec = K % 4 == 0 && (uintptr_t)X % 16 == 0 && (uintptr_t)W % (4 * sizeof(WT)) == 0;
    const int nt = R <= 16 ? 1 : 2;
    dim3 grid((unsigned)cs_ceil_div(N, MODE == GF_SWIGLU ? 32 : 16), (unsigned)cs_ceil_div(R, 16 * nt));
    auto start = [&](auto nt_tag) {
        constexpr int NT = decltype(nt_tag)::value;
        if (vec) k_gemm_f32<WT, NT, true, MODE><<<grid, 64 * GF_WAVES, 0, s>>>(X, W, Y, R, N, K, nrm, ss);
        else k_gemm_f32<WT, NT, false, MODE><<<grid, 64 * GF_WAVES, 0, s>>>(X, W, Y, R, N, K, nrm, ss);
    };
    if (nt == 1) start(std::integral_constant<int, 1>{});
    else start(std::integral_constant<int, 2>{});
    return cs_launch_ok("k_gemm_f32");
}

// by the weights' type
template <int MODE>
static int launch_plain(int dtype, const float* X, const void* W, float* Y, int R, int N, int K, const cs_norm_in& nrm,
                        float* ss, hipStream_t s) {
    return dtype == CS_BF16 ? launch_f32<bf16_t, MODE>(X, (const bf16_t*)W, Y, R, N, K, nrm, ss, s)
                            : launch_f32<float, MODE>(X, (const float*)W, Y, R, N, K, nrm, ss, s);
}

// -------------------------------------------------------------------------------------
// tuned kernel (fp16 operands, fp32 accumulation)
// -------------------------------------------------------------------------------------
#define GEMM_KC 128                       // K elements per pipeline stage
#define GEMM_LDS_ROW (GEMM_KC * 2 + 16)   // bytes per X row in LDS (padded)
#define GEMM_STAGES 4                     // X chunks in LDS
#define GEMM_RING_TILES 8                 // W tile-chunks (4 KB each) in flight per consumer wave

// The workgroup is specialised by wave.  Waves 0..CW-1 (consumers; 4, or 2 or 5, see mfma_plan) stream W:
// each owns MT 16-row tiles, keeps 8/MT K-chunks of them (32 KB) in flight in registers and multiplies.
// Two more waves (producers) bring the X block of every chunk into a ring of four LDS stages, direct-to-LDS, three
// chunks ahead.  The hardware counts outstanding loads per wave and retires
// them in order, so a wave that waits for a near X load would also drain its far W loads;
// giving X its own waves keeps the W stream deep.  One barrier per chunk hands the LDS
// stages over.
// What bounds it at 88 rows is the weights from HBM, and in launches of few chunks the time to the first X (6 us while
// 256 workgroups start their W streams; a load waits behind those requested before it).  Against X row-major through
// registers into two buffers, fragments read one multiply ahead and surplus chunks loaded again, cold weights, us:
// 8B q/k/v 15.4 -> 13.5, down 26.6 -> 24.1, gate/up 44.3 -> 41.4 (5.7 TB/s); 1B q/k/v 9.3 -> 7.2, gate/up 18.4 -> 16.0,
// down 13.0 -> 11.9.
// MT: 16-row W tiles per consumer wave.  NT: 16-row X tiles per workgroup.
// grid.x: (W row tile of 16*MT*CW, X row block of 16*NT) pairs, see the mapping below;
// grid.y: K splits.
// X and the SwiGLU output are in fragment order (cs_xt_index); am_tiles: pairs per row of the argmax epilogue.
// XN: X is not given; the producers normalise the float32 residual stream themselves (few rows, see cs_norm_in).

#define GEMM_STORE_STREAM 3   // CS_GEMM_STORE whose partial tiles leave through streaming stores
template <int MT, int NT, int MODE, int CW, bool XN = false>
__global__ __launch_bounds__(64 * (CW + 2)) void k_gemm_mfma(const f16_t* __restrict__ X,
                                                            const f16_t* __restrict__ W,
                                                            float* __restrict__ Y,
                                                            f16_t* __restrict__ act, int R, int N,
                                                            int K, int Ks, int RB, int am_tiles,
                                                            cs_norm_in nrm) {
    // X chunks: 16-row tiles in fragment order, a ring of GEMM_STAGES; XN: padded rows, two buffers
    constexpr int STAGE = XN ? 16 * NT * GEMM_LDS_ROW : NT * 4096;
    __shared__ __attribute__((aligned(16))) unsigned char xs[(XN ? 2 : GEMM_STAGES) * STAGE];
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int k_begin = blockIdx.y * Ks;
    const int k_end = min(K, k_begin + Ks);
    const int nchunks = (k_end - k_begin) / GEMM_KC;
    const int steps = max(nchunks, GEMM_RING_TILES / MT);  // chunks that producers and consumers hand over
    // Workgroup -> (W tile, X row block).  Consecutive workgroup ids go to different XCDs
    // (8 of them, each with its own L2), so the RB row blocks that share one W tile are given
    // ids 8 apart: they run on the same XCD at about the same time and all but the first read
    // W from that L2 instead of HBM.
    const int grp = blockIdx.x / (8 * RB), rem = blockIdx.x % (8 * RB);
    const int w_tile = grp * 8 + (rem & 7);
    if (w_tile * 16 * MT * CW >= N) return;               // whole workgroup, before any barrier
    const int r_base = (rem >> 3) * 16 * NT;

    // XN: the rows' sums of squares come in nss pieces [nss][16], one per column tile of the kernel that wrote the
    // stream.  All waves take a share, requested before anything else (loads return in order).
    constexpr int SQ = XN ? 4 : 1;
    f32x4 sq[SQ];
    auto sq_request = [&]() {
#pragma unroll
        for (int u = 0; u < SQ; ++u) {
            const int i = tid + u * 64 * (CW + 2);
            sq[u] = i < 4 * nrm.nss ? *reinterpret_cast<const f32x4*>(nrm.ss + 4 * i) : (f32x4){0.f, 0.f, 0.f, 0.f};
        }
    };
    __shared__ __attribute__((aligned(16))) float sq_part[XN ? CW + 2 : 1][16];
    auto sq_reduce = [&]() {
        f32x4 a = sq[0];
#pragma unroll
        for (int u = 1; u < SQ; ++u) a += sq[u];
        for (int i = tid + SQ * 64 * (CW + 2); i < 4 * nrm.nss; i += 64 * (CW + 2)) a += *reinterpret_cast<const f32x4*>(nrm.ss + 4 * i);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int o = 4; o < 64; o <<= 1) a[j] += __shfl_xor(a[j], o, 64);
        if (lane < 4) *reinterpret_cast<f32x4*>(&sq_part[wave][4 * lane]) = a;
        __syncthreads();
    };
    if constexpr (XN) sq_request();

    if constexpr (XN) {
        if (wave >= CW) {
            // ---------------- producers, X the residual stream: RMSNorm on the way to LDS ----------------
            static_assert(NT == 1, "few rows only");
            constexpr int ROWS4 = 2;                   // rows of a lane, four apart
            const int seg = lane & 15, row0 = (lane >> 4) + (wave - CW) * 8;
            const int dst0 = row0 * GEMM_LDS_ROW + seg * 16;
            const float* xrow[ROWS4];
#pragma unroll
            for (int i = 0; i < ROWS4; ++i) xrow[i] = nrm.x + (int64_t)min(row0 + 4 * i, R - 1) * K + k_begin + seg * 8;
            const float* grow = nrm.gain + k_begin + seg * 8;
            f32x4 xr[2][ROWS4][2], gr[2][2];
            const int last = nchunks - 1;
            // chunk indices are clamped instead of guarded: a surplus load re-reads the last chunk and a surplus store
            // lands in the buffer nobody reads any more, so the loop body is branch-free and the compiler's load
            // counters stay exact (through buffers of no bytes, as W: 1B gate/up 13.7 -> 14.3 us)
            auto load_x = [&](int slot, int c) {
                c = c < last ? c : last;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    gr[slot][h] = *reinterpret_cast<const f32x4*>(grow + c * GEMM_KC + 4 * h);
#pragma unroll
                    for (int i = 0; i < ROWS4; ++i) xr[slot][i][h] = *reinterpret_cast<const f32x4*>(xrow[i] + c * GEMM_KC + 4 * h);
                }
            };
            load_x(0, 0);
            load_x(1, 1);
            sq_reduce();
            float scale[ROWS4];
#pragma unroll
            for (int i = 0; i < ROWS4; ++i) {
                float q = 0.f;
#pragma unroll
                for (int w = 0; w < CW + 2; ++w) q += sq_part[w][row0 + 4 * i];
                scale[i] = row0 + 4 * i < R ? 1.0f / sqrtf(q / (float)K + nrm.eps) : 0.f;      // rows past R: zeros
            }
            bool hit = false;
            auto store_x = [&](int slot, int buf) {
#pragma unroll
                for (int i = 0; i < ROWS4; ++i) {
                    f16x8 o;
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[e] = cs_f16_sat(xr[slot][i][e >> 2][e & 3] * scale[i] * gr[slot][e >> 2][e & 3], hit);
                    *reinterpret_cast<f16x8*>(&xs[buf * STAGE + dst0 + i * 4 * GEMM_LDS_ROW]) = o;
                }
            };
            store_x(0, 0);
            load_x(0, 2);
            __syncthreads();
            int c = 0;
            for (; c + 1 < steps; c += 2) {            // chunk c+1 lives in slot 1, chunk c+2 in slot 0
                store_x(1, 1);
                load_x(1, c + 3);
                __syncthreads();
                store_x(0, 0);
                load_x(0, c + 4);
                __syncthreads();
            }
            if (c < steps) __syncthreads();
            cs_range_report(nrm.flags, hit, CS_RANGE_NORM);
            return;
        }
    }
    if (!XN && wave >= CW) {
        // ---------------- producers: X chunks -> LDS ----------------
        // Chunk c + 3 is requested while chunk c is multiplied, by direct-to-LDS loads: every request is one 1 KB
        // fragment block, the two waves take every second one.  They issue no other loads, so the counts are exact.
        // (A stage is free again when its chunk's barrier is behind: the fragments read from it have been multiplied.)
        const int p = __builtin_amdgcn_readfirstlane(wave) - CW;
        const int rt_tiles = (R + 15) >> 4;
        const f16_t* xt[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)                      // (tiles past R: the last one again)
            xt[nt] = X + ((int64_t)min((r_base >> 4) + nt, rt_tiles - 1) * (K >> 5) + (k_begin >> 5)) * 512;
        const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)xs;
        const unsigned lane16 = lane * 16;
        auto issue = [&](int c) {
            const unsigned dst = lds0 + (c & (GEMM_STAGES - 1)) * STAGE;
#pragma unroll
            for (int i = 0; i < 2 * NT; ++i) {
                const int s = 2 * (i & 1) + p;
                cs_load_to_lds(lane16, xt[i >> 1] + (c * 4 + s) * 512, dst + ((i >> 1) * 4 + s) * 1024);
            }
        };
        static_assert(GEMM_STAGES == 4 && GEMM_STAGES == GEMM_RING_TILES / MT && 6 * NT <= 63, "three chunks in flight");
        if (nchunks >= GEMM_STAGES) {
            issue(0);
            issue(1);
            issue(2);
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(4 * NT) : "memory");
            for (int c = 0; c + 3 < nchunks; ++c) {          // chunk c is multiplied, chunk c + 1 has to be there next
                issue(c + 3);
                asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(4 * NT) : "memory");
            }
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * NT) : "memory");
            asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
            asm volatile("s_barrier" ::: "memory");
        } else {
            // Less than a ring: the consumers multiply the surplus chunks too, zeros of W by zeros of X (an infinity
            // of X times the zeros of W would be a NaN).
            for (int c = 0; c < nchunks; ++c) issue(c);
            for (int i = nchunks * STAGE + p * 1024 + lane16; i < GEMM_STAGES * STAGE; i += 2048)
                *reinterpret_cast<f16x8*>(xs + i) = (f16x8){0, 0, 0, 0, 0, 0, 0, 0};
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            for (int c = 0; c < GEMM_STAGES; ++c) asm volatile("s_barrier" ::: "memory");
        }
        if (MODE == CS_GEMM_ARGMAX) {                      // the two barriers of the consumers' epilogue
            __syncthreads();
            __syncthreads();
        }
        return;
    }

    // ---------------- consumers: W stream + MFMA ----------------
    const int lrow = lane & 15, g = lane >> 4;
    const int n_wave = (w_tile * CW + wave) * MT * 16;           // first W row of this wave
    // W is stored in MFMA fragment order, K-chunk major: W_t[k/128][n/16][(k%128)/32][lane][8].
    // The 16-byte piece `lane` of a 1 KB block is exactly that lane's A operand, so every wave
    // load reads 8 whole cache lines, and all workgroups working on the same K chunk read one
    // contiguous slab of N*256 bytes, which spreads evenly over the HBM channels (a row-major
    // W with its power-of-two row pitch makes concurrent workgroups hit the same channels).
    // (row tiles past N are clamped; their results are never stored)
    unsigned wtile[MT];                                           // byte offsets within a slab
    const int n_tiles = N >> 4;
    const int64_t chunk_stride = (int64_t)n_tiles * 4 * 512;     // elements per K chunk slab
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        int t = (n_wave >> 4) + mt;
        t = t < n_tiles ? t : n_tiles - 1;
        wtile[mt] = (unsigned)t * 4096 + lane * 16;
    }
    const f16_t* __restrict__ wsplit = W + (k_begin / GEMM_KC) * chunk_stride;
    f32x4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = (f32x4){0.f, 0.f, 0.f, 0.f};

    constexpr int GEMM_DEPTH = GEMM_RING_TILES / MT;            // K chunks in flight
    f16x8 a[GEMM_DEPTH][MT][4];
    auto w_rsrc = [&](int c) { return cs_rsrc(wsplit + c * chunk_stride, c < nchunks ? (unsigned)n_tiles * 4096u : 0u); };
    auto load_w = [&](f16x8 (*dst)[4], auto rsrc, int mt, int s0, int s1) {
        unsigned off = wtile[mt];
        asm volatile("" : "+v"(off));                          // (one register: the additions below stay in the loads)
#pragma unroll
        for (int s = s0; s < s1; ++s) dst[mt][s] = __builtin_bit_cast(f16x8, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off + s * 1024, 0, 0));
    };
    // The X fragments of a chunk are read AHEAD of their multiplies: a consumer has a SIMD to itself (nearly), so a read
    // that is waited for at once costs its whole latency, which is three multiplies.  From three row tiles on the order is
    // pinned and a k-step of the ring is requested anew right after its last multiply (8B down, 88 rows: 24.1 us, 27.5 with
    // all requests behind the chunk); fewer rows leave it to the compiler (one stream's 1B gate/up 13.8, pinned 14.5).
    constexpr int NF = 4 * NT, AHEAD = NF < 6 ? NF : 6;
    auto compute = [&](f16x8 (*src)[4], int buf, int c_next) {
        const unsigned char* xb = xs + (XN ? (buf & 1) * STAGE + lrow * GEMM_LDS_ROW + g * 16 : buf * STAGE + lane * 16);
        auto frag = [&](int f) {
            return *reinterpret_cast<const f16x8*>(xb + (XN ? (f % NT) * 16 * GEMM_LDS_ROW + (f / NT) * 64 : ((f % NT) * 4 + f / NT) * 1024));
        };
        const auto rsrc = w_rsrc(c_next);                      // (past the last chunk: no memory traffic, see cs_rsrc)
        f16x8 b[AHEAD];
#pragma unroll
        for (int f = 0; f < AHEAD; ++f) b[f] = frag(f);
        if constexpr (NT >= 3) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                acc[mt][f % NT] = __builtin_amdgcn_mfma_f32_16x16x32_f16(src[mt][f / NT], b[f % AHEAD], acc[mt][f % NT], 0, 0, 0);
            if (f + AHEAD < NF) b[f % AHEAD] = frag(f + AHEAD);
            if (NT >= 3 && f % NT == NT - 1)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) load_w(src, rsrc, mt, f / NT, f / NT + 1);
            if constexpr (NT >= 3) __builtin_amdgcn_sched_barrier(0);
        }
        if (NT < 3)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) load_w(src, rsrc, mt, 0, 4);
    };
#pragma unroll
    for (int u = 0; u < GEMM_DEPTH; ++u) {
        const auto rsrc = w_rsrc(u);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) load_w(a[u], rsrc, mt, 0, 4);
    }
    if constexpr (XN) sq_reduce();
    __syncthreads();
    // Branch-free rings of DEPTH chunks, at least one (surplus chunks are zeros on both sides; XN: of W, its X is saturated): with a way round the loop the
    // compiler copied the ring from one set of registers into another, which waits for every load in it.
    int c = 0;
    do {
#pragma unroll
        for (int u = 0; u < GEMM_DEPTH; ++u) {
            compute(a[u], u, c + u + GEMM_DEPTH);
            __syncthreads();
        }
        c += GEMM_DEPTH;
    } while (c + GEMM_DEPTH <= nchunks);
#pragma unroll
    for (int u = 0; u < GEMM_DEPTH - 1; ++u) {                // remainder, data already in a[u]
        if (c + u < nchunks) {
            compute(a[u], u, nchunks);
            __syncthreads();
        }
    }

    // epilogue.  acc[mt][nt][j] = Y[row r_base + nt*16 + lrow][col n_wave + mt*16 + 4g + j]
    if (MODE == CS_GEMM_STORE || MODE == GEMM_STORE_STREAM) {
        float* __restrict__ y = Y + (int64_t)blockIdx.y * R * N;
        if constexpr (MT == 2) {
            // The wave's two 16-column tiles are neighbours: lanes 8 rows apart swap one tile each, so
            // that a store instruction covers 8 rows x 128 bytes (whole lines) instead of 16 rows x 64.
            const bool low = lrow < 8;
            const int n = n_wave + (low ? 0 : 16) + 4 * g;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                f32x4 t0, t1;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    t0[j] = __shfl_xor(acc[0][nt][j], 8, 64);
                    t1[j] = __shfl_xor(acc[1][nt][j], 8, 64);
                }
                const int ra = r_base + nt * 16 + (lrow & 7), rb = ra + 8;
                f32x4* pa = reinterpret_cast<f32x4*>(y + (int64_t)ra * N + n);
                f32x4* pb = reinterpret_cast<f32x4*>(y + (int64_t)rb * N + n);
                const f32x4 va = low ? acc[0][nt] : t1, vb = low ? t0 : acc[1][nt];
                if constexpr (MODE == GEMM_STORE_STREAM) {  // see the launcher
                    if (ra < R && n < N) cs_store_stream(pa, va);
                    if (rb < R && n < N) cs_store_stream(pb, vb);
                } else {
                    if (ra < R && n < N) *pa = va;
                    if (rb < R && n < N) *pb = vb;
                }
            }
        } else {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int r = r_base + nt * 16 + lrow;
                if (r >= R) continue;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const int n = n_wave + mt * 16 + 4 * g;
                    if (n < N) *reinterpret_cast<f32x4*>(y + (int64_t)r * N + n) = acc[mt][nt];
                }
            }
        }
    } else if (MODE == CS_GEMM_ARGMAX) {
        // Per row, the largest of this workgroup's 16*MT*CW columns and its column (the lowest on
        // ties): over the lane's own columns in increasing order, over the four lanes that share
        // a row, then over the waves through LDS (the X buffers are free).  Y carries the
        // pair buffer [R][tiles][2], am_tiles the number of tiles per row.
        int32_t* __restrict__ am = reinterpret_cast<int32_t*>(Y);
        const int nch = am_tiles;
        float* rv = reinterpret_cast<float*>(xs);                 // [CW waves][16*NT rows]
        int* ri = reinterpret_cast<int*>(xs) + CW * 16 * NT;
        __syncthreads();                                    // every wave is past its last X fragment
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            float bv = -INFINITY;
            int bi = 0x7fffffff;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                if (n_wave + mt * 16 >= N) continue;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float v = acc[mt][nt][j];
                    if (v > bv) { bv = v; bi = n_wave + mt * 16 + 4 * g + j; }
                }
            }
#pragma unroll
            for (int o = 16; o <= 32; o <<= 1) {
                const float ov = __shfl_xor(bv, o, 64);
                const int oi = __shfl_xor(bi, o, 64);
                cs_am_take(bv, bi, ov, oi);
            }
            if (g == 0) {
                rv[wave * 16 * NT + nt * 16 + lrow] = bv;
                ri[wave * 16 * NT + nt * 16 + lrow] = bi;
            }
        }
        __syncthreads();
        if (tid < 16 * NT && r_base + tid < R) {
            float bv = rv[tid];
            int bi = ri[tid];
#pragma unroll
            for (int w = 1; w < CW; ++w) cs_am_take(bv, bi, rv[w * 16 * NT + tid], ri[w * 16 * NT + tid]);
            const int64_t o = ((int64_t)(r_base + tid) * nch + w_tile) * 2;
            am[o] = __float_as_int(bv);
            am[o + 1] = bi;
        }
    } else {
        // W rows alternate 16 gate rows / 16 up rows of the same 16 FFN channels.  The result is
        // the float16 input of the down projection: saturated at +-65504, and reported through the
        // range flags (Y carries their address in this mode)
        const int F = N / 2;
        bool hit = false;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int r = r_base + nt * 16 + lrow;
            if (r >= R) continue;
#pragma unroll
            for (int mp = 0; mp < MT / 2; ++mp) {
                const int n = n_wave + mp * 32;
                if (n >= N) continue;
                const int f = n / 2 + 4 * g;
                f16x4 o;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float gt = acc[2 * mp][nt][j], up = acc[2 * mp + 1][nt][j];
                    o[j] = cs_f16_sat(gt / (1.0f + __expf(-gt)) * up, hit);
                }
                *reinterpret_cast<f16x4*>(act + cs_xt_index(r, f, F)) = o;        // fragment order
            }
        }
        cs_range_report(reinterpret_cast<int32_t*>(Y), hit, CS_RANGE_FFN);
    }
}

// -------------------------------------------------------------------------------------
// tuned kernel for many rows (e.g. batch 16 x (k = 32) + 1 = 528 rows)
//
// With hundreds of block rows the projections are bound by the matrix cores, and those by power: the loop below runs
// its multiplies at 1.4 to 1.65 GHz where constant operands leave the clock at 2.4 (a loop of nothing but multiplies of random
// registers: 1.9 GHz, 1.88 PFLOP/s; with 32x32x16 instructions 1.63).  So the tile is chosen for operand reuse: a
// workgroup of eight waves (4 x 2, two per SIMD) owns a 256 (W rows) x 32*NT (X rows) output tile, each wave 64 x 16*NT.  Both
// operands go through LDS, every element fetched from L2 once per workgroup.  LDS holds them
// in MFMA fragment order (1 KB blocks of 16 rows x 32 k, lane l's 16 bytes at offset 16*l), so
// fragment reads are conflict-free without padding; the pre-tiled W is already stored that
// way in memory.  The operands never pass through registers on their way in: every wave
// issues 16-byte direct-to-LDS loads (lane l's 16 bytes land at the wave-uniform LDS address
// in M0 plus 16*l, so one load fills one fragment block; X is stored in the same order, see
// cs_xt_index).  K advances 32 at a time through a ring of four LDS stages.
// The two waves of a SIMD, one of each wave row, take turns: while one multiplies a chunk out of its registers, the
// other reads its fragments of the next and requests its share of the chunk three further on; a barrier, and they change
// places.  With both in phase, fragments read a few multiplies ahead and one barrier per chunk, the reads of all eight
// waves met at the chunk's start: 1303 cycles a chunk at 17 X tiles, 841 at ten, now 1170 and 761 (1088 and 640 of them
// multiplies).  Gate/up of the 8B shape at 2048 rows 390 -> 372 us (1.29 PFLOP/s), at 528 100.3 -> 98.3, at 300 68.1 -> 66.2; by
// X tiles 6, 7, 8, 10, 16, 17 over 690 launches 0.93, 0.95, 0.96, 0.96, 0.96, 0.97 of the time.  (One barrier per chunk with the
// wave rows half a chunk apart: 850 us where in phase took 807; four waves of 128 x 128, a third fewer LDS
// reads: the cycles it loses are what the clock gains, 841; two chunks per phase: 78 where one took 72.)
//
// The loads and the waits on them are written as inline assembly: the compiler's own
// bookkeeping would make every LDS read wait for all outstanding direct-to-LDS loads.  This
// kernel issues no other vector memory loads, so the load counter counts exactly the
// requests below and the s_waitcnt immediates are exact.
// -------------------------------------------------------------------------------------
#define TD_KC 32
#define TG_THREADS 512
#define TG_WROWS 256
#define TG_XT_MIN 6        // fewest X tiles of a workgroup (three per wave)
#define TG_PANEL 4          // row blocks a compute die walks per W tile, see the mapping in the kernel


// XT: 16-row X tiles per workgroup (TG_XT_MIN..18).  The two wave rows split them as evenly as whole tiles
// allow: wave row 0 takes the first NT0 = ceil(XT/2), wave row 1 the other NT1 = floor(XT/2); with
// XT odd (528 rows in two blocks: 17 tiles) the two waves of a SIMD, one of each row, then multiply
// 4*17 tile pairs per chunk where an even split rounded up would make it 4*18.
template <int XT, int MODE>
__global__ __launch_bounds__(TG_THREADS) void k_gemm_dma(const f16_t* __restrict__ X,
                                                         const f16_t* __restrict__ W,
                                                         float* __restrict__ Y,
                                                         f16_t* __restrict__ act, int R, int N, int K,
                                                         int Ks, int RB, int am_tiles) {
    constexpr int NT0 = (XT + 1) / 2, NT1 = XT / 2;   // X tiles of a wave in wave row 0 / 1
    constexpr int NBLK = 16 + XT;                     // 1 KB blocks per stage: 16 W tiles, then X tiles
    constexpr int XLD = (XT + 7) / 8;                 // X loads per wave per stage (the last may be partial)
    constexpr int LDMIN = 2 + XT / 8;                 // loads every wave issues per stage
    constexpr int STAGE = NBLK * 1024;
    __shared__ __attribute__((aligned(16))) unsigned char lds[4 * STAGE];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int wn = wave & 3, wm = wave >> 2;
    const int lrow = lane & 15, g = lane >> 4;
    const int k_begin = blockIdx.y * Ks;              // multiple of 128
    const int k_end = min(K, k_begin + Ks);
    const int nchunks = (k_end - k_begin) / TD_KC;    // multiple of 4
    // Workgroup -> (W tile, X row block): XCD x (workgroup ids x, x + 8, ...) owns W tiles x, x + 8, ...
    // and walks them in panels of TG_PANEL row blocks, all row blocks of a panel per W tile before the
    // next tile, so that its 32 compute units share few W tiles and few row blocks at any time.
    // Against one panel of all row blocks: 16384 x 2048 (1B gate/up), 4095 rows in 16 or 20 blocks 227, 246 -> 214,
    // 228 us; the 8B and Qwen2.5-7B projections within 3 % either way, their whole prompts within half a percent.
    const int per_xcd = (int)gridDim.x / (8 * RB), seq = (int)blockIdx.x >> 3;
    const int panel = seq / (TG_PANEL * per_xcd), in_panel = seq - panel * TG_PANEL * per_xcd;
    const int panel_rows = min(TG_PANEL, RB - panel * TG_PANEL);
    const int w_tile = in_panel / panel_rows * 8 + ((int)blockIdx.x & 7);
    if (w_tile * TG_WROWS >= N) return;
    const int r_base = (panel * TG_PANEL + in_panel % panel_rows) * 16 * XT;
    const int n_tiles = N >> 4;
    const int64_t chunk_stride = (int64_t)n_tiles * 4 * 512;

    // wave w requests W tiles w, w+8 and X tiles w, w+8, ... of every chunk.  Both operands are
    // stored in fragment order (W: see k_tile_w; X: cs_xt_index), so every request is one 1 KB
    // block: the lane offset is 16*lane for all of them and the block moves the uniform base.
    const unsigned lane16 = lane * 16;
    const int rt_tiles = (R + 15) >> 4;
    const int64_t x_pitch = (int64_t)(K >> 5) * 512;                   // elements per X row tile
    int tw[2], tx[XLD];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int t = w_tile * 16 + wave + 8 * i;
        tw[i] = t < n_tiles ? t : n_tiles - 1;
    }
#pragma unroll
    for (int i = 0; i < XLD; ++i) {
        int j = wave + 8 * i;
        j = j < XT ? j : XT - 1;
        const int t = (r_base >> 4) + j;
        tx[i] = t < rt_tiles ? t : rt_tiles - 1;
    }
    const f16_t* wbase = W + (int64_t)(k_begin / GEMM_KC) * chunk_stride;
    const f16_t* xbase = X + (int64_t)(k_begin / TD_KC) * 512;
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;

    int extra = __builtin_amdgcn_readfirstlane(wave < XT % 8 ? 1 : 0);   // requests one X block more than the others
    asm volatile("" : "+s"(extra));                  // stays a scalar register
    // request number `idx` (0, 1: W blocks; 2..: X blocks) of chunk c into stage sb
    constexpr int NL = 2 + XLD;                       // requests per wave and chunk (the last may be void)
    auto issue_one = [&](int sb, int c, int idx) {
        const unsigned dst = lds0 + sb * STAGE + wave * 1024;
        if (idx < 2) {
            const f16_t* wc = wbase + (int64_t)(c >> 2) * chunk_stride + (c & 3) * 512;
            cs_load_to_lds(lane16, wc + (int64_t)tw[idx] * 2048, dst + 8 * idx * 1024);
        } else {
            const int i = idx - 2;
            const f16_t* xc = xbase + (int64_t)c * 512 + tx[i] * x_pitch;
            if (8 * i + 7 < XT) cs_load_to_lds(lane16, xc, dst + (16 + 8 * i) * 1024);
            else cs_load_to_lds_if(extra, lane16, xc, dst + (16 + 8 * i) * 1024);
        }
    };
    auto issue = [&](int sb, int c) {
#pragma unroll
        for (int idx = 0; idx < NL; ++idx) issue_one(sb, c, idx);
    };
    const unsigned char* a_base = lds + wn * 4 * 1024 + lane * 16;
    const unsigned char* b_base = lds + (16 + wm * NT0) * 1024 + lane * 16;
    auto a_frag = [&](int sb, int mt) { return *reinterpret_cast<const f16x8*>(a_base + sb * STAGE + mt * 1024); };
    auto b_frag = [&](int sb, int nt) { return *reinterpret_cast<const f16x8*>(b_base + sb * STAGE + nt * 1024); };
    const int n_wave = w_tile * TG_WROWS + wn * 64;

    // TD_WAIT: until at most `n` chunks of this wave's requests are outstanding.  With XT no multiple of 8 the first
    // XT % 8 waves request one block more per chunk and count their own number.  (One asm statement: a branch the compiler
    // sees splits the accumulators' live ranges.)  TD_MEET is a plain s_barrier: the workgroup fence of
    // __syncthreads would drain every load in flight; nothing moves across it.
#define TD_WAIT(n)                                                                                    \
    do {                                                                                              \
        if constexpr (XT % 8 == 0 || (n) == 0)                                                        \
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((n) * LDMIN) : "memory");                        \
        else                                                                                          \
            asm volatile("s_cmp_eq_u32 %0, 0\n\ts_cbranch_scc1 .Lfew%=\n\ts_waitcnt vmcnt(%1)\n"      \
                         "\ts_branch .Lmet%=\n.Lfew%=:\n\ts_waitcnt vmcnt(%2)\n.Lmet%=:"             \
                         ::"s"(extra), "n"((n) * (LDMIN + 1)), "n"((n) * LDMIN) : "memory", "scc");   \
    } while (0)
#define TD_MEET()                                                                                     \
    do {                                                                                              \
        __builtin_amdgcn_sched_barrier(0);                                                            \
        asm volatile("s_barrier" ::: "memory");                                                       \
        __builtin_amdgcn_sched_barrier(0);                                                            \
    } while (0)
    // the next chunk has landed, as far as this wave requested it; of those behind it two may be outstanding
#define TD_LANDED(left)                                                                               \
    do {                                                                                              \
        if constexpr ((left) == 3) TD_WAIT(2);                                                        \
        else if constexpr ((left) == 2) TD_WAIT(1);                                                   \
        else if constexpr ((left) == 1) TD_WAIT(0);                                                   \
    } while (0)

    // Everything a wave does with its NT X tiles: the multiply loop and the epilogue.  Both wave rows
    // run it with their own NT; the requests, the waits and the barriers are the same in both, so
    // the two instantiations stay in step.
    auto body = [&](auto nt_tag, auto row_tag) {
        constexpr int NT = decltype(nt_tag)::value;
        constexpr bool SECOND = decltype(row_tag)::value == 1;
        const int xt0 = wm * NT0;                        // first X tile of this wave within the block
        f32x4 acc[4][NT];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = (f32x4){0.f, 0.f, 0.f, 0.f};
        f16x8 a[4], b[NT];

        issue(0, 0);
        issue(1, 1);
        issue(2, 2);
        TD_WAIT(2);                                                // chunk 0 has landed
        TD_MEET();
        if constexpr (SECOND) TD_MEET();                           // from here on half a chunk behind
        // One chunk, two phases.  LEFT: chunks behind it, 3 for three or more.  The first wave row reads chunk c in phase
        // 2c and multiplies it in 2c + 1, the second a phase later each.  Chunk c + 3 takes the stage of chunk c - 1, last
        // read in phase 2c - 1 (and waited for before its barrier); chunk c + 1 is first read in phase 2c + 2, so
        // both wave rows wait for their requests of it at the end of phase 2c + 1.
        auto chunk = [&](int u, int c, auto left_tag) {
            constexpr int LEFT = decltype(left_tag)::value;
            // read and request; the other wave row multiplies
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) a[mt] = a_frag(u, mt);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) b[nt] = b_frag(u, nt);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (LEFT == 3) issue((u + 3) & 3, c + 3);
            __builtin_amdgcn_s_waitcnt(0xC07F);                    // the fragments are here (lgkmcnt 0, no other count)
            if constexpr (SECOND) TD_LANDED(LEFT);
            TD_MEET();
            // multiply; the other wave row reads
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int mt = 0; mt < 4; ++mt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[mt], b[nt], acc[mt][nt], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (!SECOND) TD_LANDED(LEFT);
            TD_MEET();
        };
        constexpr std::integral_constant<int, 3> more{};
        int c0 = 0;
        for (; c0 + 4 < nchunks; c0 += 4)
#pragma unroll
            for (int u = 0; u < 4; ++u) chunk(u, c0 + u, more);
        chunk(0, c0, more);
        chunk(1, c0 + 1, std::integral_constant<int, 2>{});
        chunk(2, c0 + 2, std::integral_constant<int, 1>{});
        chunk(3, c0 + 3, std::integral_constant<int, 0>{});
        if constexpr (!SECOND) TD_MEET();

        // epilogue: acc[mt][nt][j] = Y[r_base + (xt0 + nt)*16 + lrow][n_wave + mt*16 + 4g + j]
        if (MODE == CS_GEMM_STORE) {
            float* __restrict__ y = Y + (int64_t)blockIdx.y * R * N;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int r = r_base + (xt0 + nt) * 16 + lrow;
                if (r >= R) continue;
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) {
                    const int n = n_wave + mt * 16 + 4 * g;
                    if (n < N) *reinterpret_cast<f32x4*>(y + (int64_t)r * N + n) = acc[mt][nt];
                }
            }
        } else if (MODE == CS_GEMM_ARGMAX) {
            // as in k_gemm_mfma: the largest of the workgroup's 256 columns per row, lowest column on ties
            int32_t* __restrict__ am = reinterpret_cast<int32_t*>(Y);
            const int nch = am_tiles;
            float* rv = reinterpret_cast<float*>(lds);                        // [4 column waves][16*XT rows]
            int* ri = reinterpret_cast<int*>(lds) + 4 * 16 * XT;
            __syncthreads();                                    // every wave is past its last fragment
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                float bv = -INFINITY;
                int bi = 0x7fffffff;
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) {
                    if (n_wave + mt * 16 >= N) continue;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float v = acc[mt][nt][j];
                        if (v > bv) { bv = v; bi = n_wave + mt * 16 + 4 * g + j; }
                    }
                }
#pragma unroll
                for (int o = 16; o <= 32; o <<= 1) {
                    const float ov = __shfl_xor(bv, o, 64);
                    const int oi = __shfl_xor(bi, o, 64);
                    cs_am_take(bv, bi, ov, oi);
                }
                if (g == 0) {
                    rv[wn * 16 * XT + (xt0 + nt) * 16 + lrow] = bv;
                    ri[wn * 16 * XT + (xt0 + nt) * 16 + lrow] = bi;
                }
            }
            __syncthreads();
            if (tid < 16 * XT && r_base + tid < R) {
                float bv = rv[tid];
                int bi = ri[tid];
#pragma unroll
                for (int w = 1; w < 4; ++w) cs_am_take(bv, bi, rv[w * 16 * XT + tid], ri[w * 16 * XT + tid]);
                const int64_t o = ((int64_t)(r_base + tid) * nch + w_tile) * 2;
                am[o] = __float_as_int(bv);
                am[o + 1] = bi;
            }
        } else {
            const int F = N / 2;
            bool hit = false;                                   // as in k_gemm_mfma
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int r = r_base + (xt0 + nt) * 16 + lrow;
                if (r >= R) continue;
#pragma unroll
                for (int mp = 0; mp < 2; ++mp) {
                    const int n = n_wave + mp * 32;
                    if (n >= N) continue;
                    const int f = n / 2 + 4 * g;
                    f16x4 o;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float gt = acc[2 * mp][nt][j], up = acc[2 * mp + 1][nt][j];
                        o[j] = cs_f16_sat(gt / (1.0f + __expf(-gt)) * up, hit);
                    }
                    *reinterpret_cast<f16x4*>(act + cs_xt_index(r, f, F)) = o;
                }
            }
            cs_range_report(reinterpret_cast<int32_t*>(Y), hit, CS_RANGE_FFN);
        }
    };
    if (wm == 0) body(std::integral_constant<int, NT0>{}, std::integral_constant<int, 0>{});
    else body(std::integral_constant<int, NT1>{}, std::integral_constant<int, 1>{});
#undef TD_WAIT
#undef TD_MEET
#undef TD_LANDED
}

template <int XT>
static int launch_tile(const f16_t* X, const f16_t* W, float* Y, f16_t* act, int R, int N, int K, int mode,
                       int ksplit, int am_tiles, hipStream_t s) {
    CS_REQUIRE(((int64_t)R + 15) * K < ((int64_t)1 << 31), CS_E_UNSUPPORTED, "R*K too large for the many-row GEMM");
    const int Ks = (int)cs_round_up(cs_ceil_div(K, ksplit), GEMM_KC);
    const int RB = (int)cs_ceil_div(R, 16 * XT);
    dim3 grid((unsigned)(cs_round_up(cs_ceil_div(N, TG_WROWS), 8) * RB), (unsigned)cs_ceil_div(K, Ks));
    const int pg = cs_prof_begin(CS_PROF_GEMM, s);
    if (mode == CS_GEMM_STORE) k_gemm_dma<XT, CS_GEMM_STORE><<<grid, TG_THREADS, 0, s>>>(X, W, Y, act, R, N, K, Ks, RB, am_tiles);
    else if (mode == CS_GEMM_ARGMAX) k_gemm_dma<XT, CS_GEMM_ARGMAX><<<grid, TG_THREADS, 0, s>>>(X, W, Y, act, R, N, K, Ks, RB, am_tiles);
    else k_gemm_dma<XT, CS_GEMM_SWIGLU><<<grid, TG_THREADS, 0, s>>>(X, W, Y, act, R, N, K, Ks, RB, am_tiles);
    cs_prof_end(pg, s);
    return cs_launch_ok("k_gemm_dma");
}

// Launch shape of the weight-streaming kernel.
struct mfma_shape { int r_blocks, ksplit, waves; };

// Estimated time of a launch, us.  A workgroup fills a compute unit and takes 30 us per 4096 of K while it
// is bound by its weights, 6.1 us per X tile from five tiles on; five consumer waves share four SIMDs, 1.35 of the time for
// 1.25 of the rows; a partial tile is written and read once more at about 4.9 TB/s (an unsplit output is charged nothing here
// and once in tile_plan: with both charged alike, and the rate fitted anew, 21 of 284 whole calls of 97 to 1024
// rows and prompts up to 4096 got faster and 53 slower, 1 to 6 % each).
// The constants of both estimates are of the kernels as they were when X came row-major and the many-row kernel's waves
// worked in phase (224 workgroups at the 8B width, 4, 6, 7, 8 X tiles: 30, 37, 43 to 48, 49 to 55 us; cold weights and the
// present kernel 39, 43, 45, 47).  They stay because they decide the K splits, and those the results (see gemm_plan).
static double mfma_us(int R, int N, int K, const mfma_shape& p) {
    const int nt = (int)cs_ceil_div(cs_ceil_div(R, 16), p.r_blocks);
    const int64_t wgs = cs_ceil_div(N, 32 * p.waves) * p.r_blocks * p.ksplit;
    const double per = (6.1 * nt > 30. ? 6.1 * nt : 30.) * (p.waves == 5 ? 1.35 : 1.);
    return cs_ceil_div(wgs, 256) * per * K / p.ksplit / 4096. + (p.ksplit > 1 ? p.ksplit * 8e-6 * R * N / 4.9 : 0.);
}

// Up to 96 rows: one row block, and K splits until about 3/4 of the compute units have a workgroup (8B shapes, 88 rows: q/k/v
// with 2, 4, 8 splits 19.0, 14.4, 19.1 us, o with 4 and 8 12.8 and 12.0, down with 4, 8, 16 31.0, 24.7, 29.7).  More rows: row
// blocks of up to 128 rows and K splits by estimated time (100 rows: gate/up 60 us in two blocks, 44 in one; 256 rows: q/k/v,
// gate/up, down 33, 94, 54 us in three blocks, 22, 79, 37 in two; the 1B shape keeps two blocks of 64, which fill the chip, 18 us
// against 23).  Five consumer waves where tiles of 128 W rows need a second, nearly empty round of the chip
// (Qwen2.5-7B gate/up, 37888 rows: 296 tiles, 237 of 160 rows; 105 rows 72 -> 50 us), not for the few
// chunks of a K split (1B q/k/v at 200 rows: unsplit with five 22 us against 8).  Two consumer waves where a projection that may
// not split K has tiles of 128 W rows for half of the chip at most (1B gate/up, 16384 rows: 16, 48, 88 rows 13.9, 16.0,
// 19.5 -> 11.9, 13.5, 16.9 us); with twice as many tiles as compute units they lose (8B gate/up, 88 rows: 42 -> 54).
static mfma_shape mfma_plan(int R, int N, int K, bool may_split) {
    const int rt_total = (int)cs_ceil_div(R, 16);
    const int max_split = may_split && K / (4 * GEMM_KC) > 0 ? K / (4 * GEMM_KC) : 1;
    mfma_shape best = {1, 1, 4};
    if (rt_total <= 6) {
        const int n_tiles = (int)cs_ceil_div(N, 128);
        while (n_tiles * best.ksplit < 192 && best.ksplit * 2 <= max_split) best.ksplit *= 2;
        if (best.ksplit > 1) return best;
        mfma_shape five = best;
        five.waves = 5;
        if (mfma_us(R, N, K, five) < mfma_us(R, N, K, best)) return five;
        if (!may_split && cs_ceil_div(N, 64) <= 256) best.waves = 2;
        return best;
    }
    double best_us = -1.;
    for (int rb = (int)cs_ceil_div(rt_total, 8); rb <= (int)cs_ceil_div(rt_total, 4); ++rb)
        for (int ks = 1; ks <= max_split && ks <= 16; ks *= 2)
            for (int waves = 4; waves <= (ks == 1 ? 5 : 4); ++waves) {
                const mfma_shape p = {rb, ks, waves};
                const double us = mfma_us(R, N, K, p);
                if (best_us < 0. || us < best_us) { best_us = us; best = p; }
            }
    return best;
}

template <int MT, int NT, int CW>
static void start_mfma(const f16_t* X, const f16_t* W, float* Y, f16_t* act, int R, int N, int K, int mode, int Ks,
                       int am_tiles, hipStream_t s) {
    const int RB = (int)cs_ceil_div(R, 16 * NT);
    constexpr int threads = 64 * (CW + 2);
    dim3 grid((unsigned)(cs_round_up(cs_ceil_div(N, 16 * MT * CW), 8) * RB), (unsigned)cs_ceil_div(K, Ks));
    // From about 64 rows on the partial tiles are better sent on at once (88 rows: step -1 %,
    // 168: -0.9 %, 264: -0.3 %); with few rows the readers find them in the caches and a plain
    // store wins (48 rows +0.4 %, one stream of 11 rows +2.5 to +3.6 %).
    if (mode == CS_GEMM_STORE && R >= 64)
        k_gemm_mfma<MT, NT, GEMM_STORE_STREAM, CW><<<grid, threads, 0, s>>>(X, W, Y, act, R, N, K, Ks, RB, am_tiles, cs_norm_in{});
    else if (mode == CS_GEMM_STORE)
        k_gemm_mfma<MT, NT, CS_GEMM_STORE, CW><<<grid, threads, 0, s>>>(X, W, Y, act, R, N, K, Ks, RB, am_tiles, cs_norm_in{});
    else if (mode == CS_GEMM_ARGMAX)
        k_gemm_mfma<MT, NT, CS_GEMM_ARGMAX, CW><<<grid, threads, 0, s>>>(X, W, Y, act, R, N, K, Ks, RB, am_tiles, cs_norm_in{});
    else if constexpr (MT % 2 == 0)
        k_gemm_mfma<MT, NT, CS_GEMM_SWIGLU, CW><<<grid, threads, 0, s>>>(X, W, Y, act, R, N, K, Ks, RB, am_tiles, cs_norm_in{});
}

// few rows, normalised by the producers
static void start_norm(const cs_norm_in& nrm, const f16_t* W, float* Y, f16_t* act, int R, int N, int K, int mode, int Ks,
                       int waves, hipStream_t s) {
    dim3 grid((unsigned)cs_round_up(cs_ceil_div(N, 32 * waves), 8), (unsigned)cs_ceil_div(K, Ks));
    auto start = [&](auto cw_tag) {
        constexpr int CW = decltype(cw_tag)::value;
        if (mode == CS_GEMM_STORE)
            k_gemm_mfma<2, 1, CS_GEMM_STORE, CW, true><<<grid, 64 * (CW + 2), 0, s>>>(nullptr, W, Y, act, R, N, K, Ks, 1, 0, nrm);
        else
            k_gemm_mfma<2, 1, CS_GEMM_SWIGLU, CW, true><<<grid, 64 * (CW + 2), 0, s>>>(nullptr, W, Y, act, R, N, K, Ks, 1, 0, nrm);
    };
    if (waves == 5) start(std::integral_constant<int, 5>{});
    else if (waves == 2) start(std::integral_constant<int, 2>{});
    else start(std::integral_constant<int, 4>{});
}

template <int MT, int NT>
static int launch_mfma(const f16_t* X, const f16_t* W, float* Y, f16_t* act, int R, int N, int K,
                       int mode, int ksplit, int waves, int am_tiles, hipStream_t s) {
    const int Ks = (int)cs_round_up(cs_ceil_div(K, ksplit), GEMM_KC);
    const int pg = cs_prof_begin(CS_PROF_GEMM, s);
    if (waves == 5) start_mfma<MT, NT, 5>(X, W, Y, act, R, N, K, mode, Ks, am_tiles, s);
    else if (waves == 4) start_mfma<MT, NT, 4>(X, W, Y, act, R, N, K, mode, Ks, am_tiles, s);
    else if constexpr (NT <= 6) start_mfma<MT, NT, 2>(X, W, Y, act, R, N, K, mode, Ks, am_tiles, s);   // (see mfma_plan)
    else CS_REQUIRE(false, CS_E_STATE, "two consumer waves take at most six row tiles");
    cs_prof_end(pg, s);
    return cs_launch_ok("k_gemm_mfma");
}

static bool mfma_shape_ok(int N, int K) { return K % GEMM_KC == 0 && N % 16 == 0; }

// dst[k/128][n/16][(k%128)/32][lane l][8]: lane l (row n%16 = l%16, k-group l/16) holds the 8
// elements W[n][(k/32)*32 + (l/16)*8 ..].  N_total/n_off place a block of rows inside a taller
// matrix (the fused q,k,v projection).  rowmap 0: source row = n.  rowmap 1: rows alternate
// 16 gate rows (src) / 16 up rows (src2).
__global__ void k_tile_w(const bf16_t* __restrict__ src, const bf16_t* __restrict__ src2, int N, int K,
                         int rowmap, int N_total, int n_off, f16_t* __restrict__ dst, int32_t* flags) {
    const int64_t nvec = (int64_t)N * K / 8;
    const int n_tiles = N >> 4, nt_total = N_total >> 4;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < nvec;
         v += (int64_t)gridDim.x * blockDim.x) {
        const int lane = (int)(v & 63);
        const int s = (int)((v >> 6) & 3);
        const int64_t tile = v >> 8;
        const int nt = (int)(tile % n_tiles);
        const int kc = (int)(tile / n_tiles);
        const int n = nt * 16 + (lane & 15);
        const int k = kc * 128 + s * 32 + (lane >> 4) * 8;
        const bf16_t* sp = src + (int64_t)n * K;
        if (rowmap == 1) {
            const int f = (n >> 5) * 16 + (n & 15);
            sp = (((n >> 4) & 1) ? src2 : src) + (int64_t)f * K;
        }
        const int64_t o = ((((int64_t)kc * nt_total + (n_off >> 4) + nt) * 4 + s) * 64 + lane) * 8;
        // bfloat16 -> float16: exact for 2^-17 <= |w| < 65504 (8 significant bits fit the
        // 11-bit significand, subnormals included); smaller magnitudes round to 2^-24 steps
        const bf16x8 wv = *reinterpret_cast<const bf16x8*>(sp + k);
        f16x8 hv;
        bool bad = false;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            hv[j] = (f16_t)(float)wv[j];
            bad |= !(fabsf((float)wv[j]) <= CS_F16_MAX);      // would become inf (or is a NaN)
        }
        *reinterpret_cast<f16x8*>(dst + o) = hv;
        if (bad && flags) atomicOr(flags, CS_RANGE_WEIGHT);
    }
}

int cs_tile_weights_launch(const void* src, const void* src2, int N, int K, int rowmap, int N_total,
                           int n_off, void* dst, int32_t* flags, hipStream_t s) {
    CS_REQUIRE(mfma_shape_ok(N, K) && N_total % 16 == 0 && n_off % 16 == 0, CS_E_UNSUPPORTED,
               "cannot tile a %d x %d matrix", N, K);
    const int64_t nvec = (int64_t)N * K / 8;
    const int blocks = (int)(cs_ceil_div(nvec, 256) < 8192 ? cs_ceil_div(nvec, 256) : 8192);
    k_tile_w<<<blocks, 256, 0, s>>>((const bf16_t*)src, (const bf16_t*)src2, N, K, rowmap, N_total, n_off,
                                    (f16_t*)dst, flags);
    return cs_launch_ok("k_tile_w");
}

// f16 [R][K] row-major -> fragment order (cs_xt_index); rows of the last tile beyond R are zero
__global__ void k_tile_x(const f16_t* __restrict__ src, f16_t* __restrict__ dst, int R, int K, int rt_tiles) {
    // (one thread per 8 consecutive k of one row)
    const int64_t n = (int64_t)rt_tiles * 16 * (K / 8);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int r = (int)(i / (K / 8)), k = (int)(i % (K / 8)) * 8;
        f16x8 v = (f16x8){0, 0, 0, 0, 0, 0, 0, 0};
        if (r < R) v = *reinterpret_cast<const f16x8*>(src + (int64_t)r * K + k);
        *reinterpret_cast<f16x8*>(dst + cs_xt_index(r, k, K)) = v;
    }
}

int cs_tile_x_launch(const void* src, void* dst, int R, int K, hipStream_t s) {
    const int rt_tiles = (int)cs_ceil_div(R, 16);
    const int64_t n = (int64_t)rt_tiles * 16 * (K / 8);
    k_tile_x<<<(unsigned)(cs_ceil_div(n, 256) < 4096 ? cs_ceil_div(n, 256) : 4096), 256, 0, s>>>(
        (const f16_t*)src, (f16_t*)dst, R, K, rt_tiles);
    return cs_launch_ok("k_tile_x");
}

// Row blocks and K splits of a many-row GEMM: the pair with the least estimated time.  A workgroup
// with rt X tiles takes 4.5 us * (6.7 + rt) per 4096 of K on a full chip (the requests and the barriers of a chunk cost
// what 6.7 tiles cost to multiply, so a tile shorter by a ninth pays only where it does not add a round of the chip; see
// mfma_us on the constants); a round that fills a part f of the chip takes 0.65 + 0.35 f of a full one (less contention);
// every partial tile is written and read once more at about 4.9 TB/s.
// 4095 rows, 8B width, against the fewest row blocks (15 x 288 rows): gate/up 756 -> 686 us,
// q/k/v 200 -> 166, o 111 -> 106, down 355 -> 340 us; 528 rows: o 32 -> 27 us with half the partial tiles.
// (returns the time; a launch of its own costs about 4 us on top)
static double tile_plan(int R, int N, int K, bool may_split, int* r_blocks, int* ksplit) {
    const int rt_total = (int)cs_ceil_div(R, 16);
    const int per_xcd = (int)cs_ceil_div(cs_ceil_div(N, TG_WROWS), 8);   // W tiles of one die
    const int max_split = may_split && K / (4 * GEMM_KC) > 0 ? K / (4 * GEMM_KC) : 1;
    const int rb_min = (int)cs_ceil_div(rt_total, 18), rb_max = (int)cs_ceil_div(rt_total, TG_XT_MIN);
    double best = -1.;
    for (int rb = rb_min; rb <= rb_max; ++rb) {
        const int rt = (int)cs_ceil_div(rt_total, rb) < TG_XT_MIN ? TG_XT_MIN : (int)cs_ceil_div(rt_total, rb);
        for (int ks = 1; ks <= max_split && ks <= 16; ks *= 2) {
            const int wgs = per_xcd * (int)cs_ceil_div(rt_total, rt) * ks;   // on 32 compute units
            const double part = (wgs % 32) / 32., rounds = wgs / 32 + (part > 0. ? 0.65 + 0.35 * part : 0.);
            const double us = rounds * 4.5 * (6.7 + rt) * K / ks / 4096. + (may_split ? ks * 8e-6 * R * N / 4.9 : 0.);
            if (best < 0. || us < best) {
                best = us;
                *r_blocks = rb;
                *ksplit = ks;
            }
        }
    }
    return best + 4.;
}

// Which kernel a projection of R rows takes, and its launch shape (waves 0: the many-row kernel, 256 W rows
// x up to 288 block rows per workgroup): from 97 rows on the many-row kernel where its 256-row W tiles alone fill most of
// the chip (lm_head; 128 rows of the 8B one 196 -> 178 us), from 289 on everywhere, between 129 and 288 rows where the two estimates say so (250 rows: 8B gate/up
// 79 -> 63 us; 1B gate/up stays, 24 us in two row blocks against 28 in three), up to 128 rows nowhere else (128 rows, 8B
// gate/up: 47 against 63 us).
// The K splits are part of the result: each float32 sum is a chain of K / splits products, and fewer, longer chains round
// worse.  Estimates fitted to both kernels as they are now, whatever the splits, took half as many or fewer at 8B o
// (88 rows 12.0 -> 10.8 us, 300 rows 20.3 -> 17.7, 528 rows 27.4 -> 27.5) and q/k/v (300 rows 25.1 -> 26.3) and at the
// 1B shape (eight batched prompts 4 % faster), and doubled the error of some of them against float64 (o at 528 rows
// 1.9e-7 -> 4.0e-7).  Not kept.
static mfma_shape gemm_plan(int R, int N, int K, bool may_split) {
    mfma_shape t = {1, 1, 0};
    if (R <= 96) return mfma_plan(R, N, K, may_split);
    const double tile_us = tile_plan(R, N, K, may_split, &t.r_blocks, &t.ksplit);
    const bool tile_fits = ((int64_t)R + 15) * K < ((int64_t)1 << 31);      // (launch_tile refuses more)
    if (tile_fits && (R > 288 || cs_ceil_div(N, TG_WROWS) >= 192)) return t;
    const mfma_shape p = mfma_plan(R, N, K, may_split);
    return R > 128 && tile_fits && tile_us < mfma_us(R, N, K, p) ? t : p;
}

// 16-row X tiles of a workgroup
static int gemm_row_tiles(int R, const mfma_shape& p) {
    const int rt = (int)cs_ceil_div(cs_ceil_div(R, 16), p.r_blocks);
    return p.waves == 0 && rt < TG_XT_MIN ? TG_XT_MIN : rt;
}

bool cs_gemm_x_tiled(int R, int N, int K, bool may_split) { return gemm_plan(R, N, K, may_split).waves == 0; }
void cs_gemm_shape(int R, int N, int K, bool may_split, int* shape) {
    const mfma_shape p = gemm_plan(R, N, K, may_split);
    shape[0] = p.waves;
    shape[1] = gemm_row_tiles(R, p);
    shape[2] = p.ksplit;
}

int cs_gemm_launch(const cs_model* m, const void* X, const void* W, float* Y, int R, int N, int K,
                   int mode, int allow_split, int* nparts_out, hipStream_t s) {
    if (nparts_out) *nparts_out = 1;
    if (R <= 0) return CS_OK;
    if (!m->fast) return cs_gemm_plain_launch(m->cfg.dtype, (const float*)X, W, Y, R, N, K, s);
    CS_REQUIRE(mfma_shape_ok(N, K) && (mode != CS_GEMM_SWIGLU || N % 32 == 0), CS_E_UNSUPPORTED,
               "bf16 GEMM needs N %% 16 == 0 and K %% 128 == 0 (N=%d K=%d)", N, K);
    // Shape of the launch.
    // Weight-streaming kernel: a workgroup takes up to 128 block rows; more rows are split into
    // equal row blocks whose workgroups share each W tile through one XCD's L2 (see the mapping
    // in the kernel and mfma_plan).
    const bool may_split = allow_split && mode == CS_GEMM_STORE;
    const mfma_shape plan = gemm_plan(R, N, K, may_split);
    const bool tile = plan.waves == 0;
    int am_tiles = 0;                         // pairs per row of the argmax epilogue
    if (mode == CS_GEMM_ARGMAX) {
        // one (value, column) pair per row and workgroup column tile, in place of Y
        CS_REQUIRE(!allow_split && nparts_out, CS_E_STATE, "argmax epilogue: no K split, tile count wanted");
        Y = reinterpret_cast<float*>(m->am_val_idx);
    }
    if (mode == CS_GEMM_SWIGLU) Y = reinterpret_cast<float*>(m->range_flags);   // see the epilogue
    const int waves = plan.waves;
    int ksplit = plan.ksplit;
    // the partial tiles must fit the workspace
    while (ksplit > 1 && (size_t)ksplit * R * N > m->part_floats) ksplit /= 2;
    if (ksplit > 1) CS_REQUIRE(allow_split, CS_E_STATE, "K split without a partial-tile buffer");
    const int Ks = (int)cs_round_up(cs_ceil_div(K, ksplit), GEMM_KC);
    const int nparts = (int)cs_ceil_div(K, Ks);
    if (mode == CS_GEMM_ARGMAX) am_tiles = (int)cs_ceil_div(N, tile ? TG_WROWS : 32 * waves);
    if (nparts_out) *nparts_out = mode == CS_GEMM_ARGMAX ? am_tiles : nparts;
    const int rt = gemm_row_tiles(R, plan);
    const f16_t* x = (const f16_t*)X;
    const f16_t* w = (const f16_t*)W;
    f16_t* act = (f16_t*)m->act;
    if (tile) {
        switch (rt) {                                // 16-row X tiles per workgroup
            case 7: return launch_tile<7>(x, w, Y, act, R, N, K, mode, nparts, am_tiles, s);
            case 8: return launch_tile<8>(x, w, Y, act, R, N, K, mode, nparts, am_tiles, s);
            case 9: return launch_tile<9>(x, w, Y, act, R, N, K, mode, nparts, am_tiles, s);
            case 10: return launch_tile<10>(x, w, Y, act, R, N, K, mode, nparts, am_tiles, s);
            case 11: return launch_tile<11>(x, w, Y, act, R, N, K, mode, nparts, am_tiles, s);
            case 12: return launch_tile<12>(x, w, Y, act, R, N, K, mode, nparts, am_tiles, s);
            case 13: return launch_tile<13>(x, w, Y, act, R, N, K, mode, nparts, am_tiles, s);
            case 14: return launch_tile<14>(x, w, Y, act, R, N, K, mode, nparts, am_tiles, s);
            case 15: return launch_tile<15>(x, w, Y, act, R, N, K, mode, nparts, am_tiles, s);
            case 16: return launch_tile<16>(x, w, Y, act, R, N, K, mode, nparts, am_tiles, s);
            case 17: return launch_tile<17>(x, w, Y, act, R, N, K, mode, nparts, am_tiles, s);
            case 18: return launch_tile<18>(x, w, Y, act, R, N, K, mode, nparts, am_tiles, s);
            default: return launch_tile<TG_XT_MIN>(x, w, Y, act, R, N, K, mode, nparts, am_tiles, s);
        }
    }
    switch (rt) {
        case 1: return launch_mfma<2, 1>(x, w, Y, act, R, N, K, mode, nparts, waves, am_tiles, s);
        case 2: return launch_mfma<2, 2>(x, w, Y, act, R, N, K, mode, nparts, waves, am_tiles, s);
        case 3: return launch_mfma<2, 3>(x, w, Y, act, R, N, K, mode, nparts, waves, am_tiles, s);
        case 4: return launch_mfma<2, 4>(x, w, Y, act, R, N, K, mode, nparts, waves, am_tiles, s);
        case 5: return launch_mfma<2, 5>(x, w, Y, act, R, N, K, mode, nparts, waves, am_tiles, s);
        case 6: return launch_mfma<2, 6>(x, w, Y, act, R, N, K, mode, nparts, waves, am_tiles, s);
        case 7: return launch_mfma<2, 7>(x, w, Y, act, R, N, K, mode, nparts, waves, am_tiles, s);
        default: return launch_mfma<2, 8>(x, w, Y, act, R, N, K, mode, nparts, waves, am_tiles, s);
    }
}

// -------------------------------------------------------------------------------------
// output and down projections of few rows (up to 16): x += X * W^T, all of K in one workgroup
//
// A step of one stream is a chain of short launches, and what the partial tiles of a K split cost there is the kernel
// that adds them to the residual stream and normalises it (4 to 5 us, twice per layer).  Here a workgroup owns 16 W
// rows and all of K: its eight waves take the 128-wide chunks of K in turn, W and X fragments (both stored in that
// order; X row-major, 64 bytes per row and load, 9.4 against 8.6 us) straight into registers, four chunks (16 KB of W
// each wave) in flight, and are summed through LDS.  It then adds its columns to the residual stream and leaves their
// sums of squares per row, from which the next projection's producers normalise the stream (cs_norm_in).
// 11 rows, a layer's norms, q/k/v, o, gate/up, down: 1B shape 45 -> 40 us, 8B 94 -> 84 us.  Tiles of 8 W rows on twice
// the compute units: no faster at 1B, 24 against 15 us at 8B.  17 to 32 rows the same way (two row tiles): no gain,
// the float32 rows that every workgroup reads and its 32 rows of X cost what the norm kernels did.
// -------------------------------------------------------------------------------------
#define GR_WAVES 8
#define GR_DEPTH 4            // chunks in flight per wave
__global__ __launch_bounds__(64 * GR_WAVES) void k_gemm_residual(const f16_t* __restrict__ X, const f16_t* __restrict__ W,
                                                                 float* __restrict__ x, float* __restrict__ ss, int R,
                                                                 int N, int K) {
    __shared__ f32x4 red[GR_WAVES][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lrow = lane & 15, g = lane >> 4;
    const int64_t chunk_stride = (int64_t)(N >> 4) * 2048;
    const f16_t* __restrict__ w = W + (int64_t)blockIdx.x * 2048 + lane * 8;
    const f16_t* __restrict__ xr = X + (min(lrow, R - 1) + 16 * g) * 8;         // (rows past R: the last row again)
    const int nch = K / GEMM_KC, mine = (nch - wave + GR_WAVES - 1) / GR_WAVES;
    // wave 0 adds to the residual stream: row lrow, columns n .. n + 3
    const int n = blockIdx.x * 16 + 4 * g;
    const bool out = wave == 0 && lrow < R;
    float* __restrict__ dst = x + (int64_t)(out ? lrow : 0) * N + n;
    f32x4 res = (f32x4){0.f, 0.f, 0.f, 0.f};
    if (out) res = *reinterpret_cast<const f32x4*>(dst);
    f16x8 a[GR_DEPTH][4], b[GR_DEPTH][4];
    auto load = [&](int u, int i) {                    // (clamped: a surplus load re-reads the last chunk)
        const int c = min(wave + GR_WAVES * i, nch - 1);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            a[u][s] = *reinterpret_cast<const f16x8*>(w + c * chunk_stride + s * 512);
            b[u][s] = *reinterpret_cast<const f16x8*>(xr + c * 2048 + s * 512);
        }
    };
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    auto multiply = [&](int u) {
#pragma unroll
        for (int s = 0; s < 4; ++s) acc[s & 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[u][s], b[u][s], acc[s & 1], 0, 0, 0);
    };
#pragma unroll
    for (int u = 0; u < GR_DEPTH; ++u) load(u, u);
    int i = 0;
    for (; i + GR_DEPTH <= mine; i += GR_DEPTH) {
#pragma unroll
        for (int u = 0; u < GR_DEPTH; ++u) {
            multiply(u);
            load(u, i + u + GR_DEPTH);
        }
    }
#pragma unroll
    for (int u = 0; u < GR_DEPTH - 1; ++u)
        if (i + u < mine) multiply(u);
    red[wave][lane] = acc[0] + acc[1];
    __syncthreads();
    if (wave > 0) return;
    f32x4 part[GR_WAVES];
#pragma unroll
    for (int u = 0; u < GR_WAVES; ++u) part[u] = red[u][lane];
#pragma unroll
    for (int h = GR_WAVES / 2; h > 0; h /= 2)
#pragma unroll
        for (int u = 0; u < h; ++u) part[u] += part[u + h];
    const f32x4 v = res + part[0];
    if (out) *reinterpret_cast<f32x4*>(dst) = v;
    float q = out ? v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3] : 0.f;
    q += __shfl_xor(q, 16, 64);
    q += __shfl_xor(q, 32, 64);
    if (g == 0) ss[blockIdx.x * 16 + lrow] = q;
}

// Blocks that take the normalising projections and the ones that write the residual stream: up to 16 rows (float32 kernel
// 32, one row block), while that is the faster way.  Tuned kernels: a residual workgroup per 16 columns is one round of
// the chip up to d_model 4096; with more they read W at 4.2 TB/s where the K split reads it at 5.1, so that a large down
// projection costs what the norm kernels did, sooner with more than 8 rows of X.  A layer at 1 / 8 / 11 / 16 rows, against the
// same with norm kernels (d_model / d_ff): 4096 / 14336 -8, -9, -6, -7 us, 4096 / 38400 -11, -13, -7, -9, 5120 / 13824 -8, -8, -3,
// -4, 5120 / 27648 -5, -4, +5, +4, 6144 / 16384 -2, -3, +5, +4, 7168 / 20480 -4, -5, +6, +5, 6144 / 24576 +5, +4, +14, +12,
// 8192 / 28672 +11, +9, +14, +14.  Float32 kernel with bfloat16 weights (3 layers, 1 / 16 / 32 rows): 1024 / 4096 216, 239, 331
// against 223, 250, 345 us, 3072 / 8192 478, 516, 774 against 479, 541, 766, 4096 / 11008 779, 830, 1154 against 724, 797, 1103;
// with float32 weights it is ahead or within 5 % at all widths (3072 / 8192 418, 464, 640 against 423, 508, 708).
bool cs_gemm_few_rows(const cs_model* m, int R) {
    const int64_t d = m->cfg.d_model, down = d * m->cfg.d_ff;
    if (!m->fast) {
        if (m->cfg.dtype == CS_BF16 && d > 1024) return d <= 3072 && R <= 16;
        return R <= 32;
    }
    return R <= 16 && (d <= 4096 || (d <= 7168 && down <= (R <= 8 ? 150000000 : 100000000)));
}

int cs_gemm_norm_launch(const cs_model* m, const float* gain, int nss, const void* W, float* Y, int R, int N, int K, int mode,
                        int* nparts_out, hipStream_t s) {
    const cs_norm_in nrm = {m->x, gain, m->ss, nss, m->cfg.rms_eps, m->range_flags};
    if (!m->fast) {
        if (nparts_out) *nparts_out = 1;
        if (mode == CS_GEMM_SWIGLU) return launch_plain<GF_SWIGLU>(m->cfg.dtype, m->x, W, (float*)m->act, R, N, K, nrm, nullptr, s);
        return launch_plain<GF_NORM>(m->cfg.dtype, m->x, W, Y, R, N, K, nrm, nullptr, s);
    }
    CS_REQUIRE(mfma_shape_ok(N, K) && (mode == CS_GEMM_STORE || N % 32 == 0), CS_E_UNSUPPORTED,
               "bf16 GEMM needs N %% 16 == 0 and K %% 128 == 0 (N=%d K=%d)", N, K);
    mfma_shape plan = mfma_plan(R, N, K, mode == CS_GEMM_STORE);
    while (plan.ksplit > 1 && (size_t)plan.ksplit * R * N > m->part_floats) plan.ksplit /= 2;
    const int Ks = (int)cs_round_up(cs_ceil_div(K, plan.ksplit), GEMM_KC);
    if (nparts_out) *nparts_out = (int)cs_ceil_div(K, Ks);
    if (mode == CS_GEMM_SWIGLU) Y = reinterpret_cast<float*>(m->range_flags);   // see the epilogue
    const int pg = cs_prof_begin(CS_PROF_GEMM, s);
    start_norm(nrm, (const f16_t*)W, Y, (f16_t*)m->act, R, N, K, mode, Ks, plan.waves, s);
    cs_prof_end(pg, s);
    return cs_launch_ok("k_gemm_mfma (normalising)");
}

int cs_gemm_residual_launch(const cs_model* m, const void* X, const void* W, int R, int N, int K, int* nss, hipStream_t s) {
    if (!m->fast) {
        *nss = (int)cs_ceil_div(N, 16);
        return launch_plain<GF_RESIDUAL>(m->cfg.dtype, (const float*)X, W, m->x, R, N, K, cs_norm_in{}, m->ss, s);
    }
    CS_REQUIRE(mfma_shape_ok(N, K), CS_E_UNSUPPORTED, "bf16 GEMM needs N %% 16 == 0 and K %% 128 == 0 (N=%d K=%d)", N, K);
    *nss = N / 16;
    const int pg = cs_prof_begin(CS_PROF_GEMM, s);
    k_gemm_residual<<<*nss, 64 * GR_WAVES, 0, s>>>((const f16_t*)X, (const f16_t*)W, m->x, m->ss, R, N, K);
    cs_prof_end(pg, s);
    return cs_launch_ok("k_gemm_residual");
}

int cs_gemm_plain_launch(int dtype, const float* X, const void* W, float* Y, int R, int N, int K,
                         hipStream_t s) {
    if (R <= 0) return CS_OK;
    return launch_plain<GF_STORE>(dtype, X, W, Y, R, N, K, cs_norm_in{}, nullptr, s);
}
