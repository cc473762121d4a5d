// Block attention of the verify pass: the k+1 block rows of every stream attend to the
// stream's KV cache plus the causal part of the block itself (Sec. 3.2: the draft is
// appended to the context and evaluated in one pass; App. B.2: per-layer K, V).
//
// The pass is bound by streaming K and V from HBM once.  All G*(k+1) query rows that share
// a KV head (G = n_heads / n_kv_heads) are processed together, so each K/V byte is used
// G*(k+1) times: 44 flop per byte at k = 10, more than the vector ALUs can deliver at
// 8 TB/s, which is why QK^T and PV run on the matrix cores although the kernel is graded
// against the HBM roofline.
//
// Tuned kernel, per wave (K, V, scores and O stay in registers):
//   S^T[token][qrow] = K[token][:] . Q[qrow][:]        v_mfma_f32_16x16x32_bf16, A = K rows
//   O^T[hd][qrow]   += V^T[hd][token] * P^T[token][qrow]                         A = V^T rows
// K rows are fed in a permuted token order chosen so that the S^T accumulator layout of two
// 16-token tiles is exactly the B-operand layout of the PV product (8 consecutive tokens per
// lane); V is cached transposed in 128-token blocks (token index contiguous) so its A operand is one 16-byte
// load per lane.  Softmax runs online in float32 (base 2), the row maximum is shared by the
// four lanes that hold a query row, and O is only rescaled when some maximum moved.
// The token range of a stream is split over workgroups, whose waves take its 32-token blocks in
// turn; a merge kernel combines the partial (max, sum, O) triples.
#include <algorithm>
#include <type_traits>

#include "cs_common.h"

// -------------------------------------------------------------------------------------
// plain reference kernels: one workgroup per (block row, query head, stream); see the launcher for which of the two
// -------------------------------------------------------------------------------------
#define PA_CHUNK 2048
#define PA_THREADS 256

template <int THREADS>
__device__ __forceinline__ float block_max(float v, float* wred) {
    v = cs_wave_max(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) wred[threadIdx.x >> 6] = v;
    __syncthreads();
    float r = wred[0];
    for (int w = 1; w < THREADS / CS_WAVE; ++w) r = fmaxf(r, wred[w]);
    return r;
}
template <int THREADS>
__device__ __forceinline__ float block_sum(float v, float* wred) {
    v = cs_wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) wred[threadIdx.x >> 6] = v;
    __syncthreads();
    float r = 0.f;
    for (int w = 0; w < THREADS / CS_WAVE; ++w) r += wred[w];
    return r;
}

__device__ __forceinline__ f32x4 pa_ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ f32x4 pa_ld4(const bf16_t* p) {
    const bf16x4 t = *reinterpret_cast<const bf16x4*>(p);
    return (f32x4){(float)t[0], (float)t[1], (float)t[2], (float)t[3]};
}

// A key row per thread, four tokens of one V feature per thread: every wave's loads touch 64 lines, but a thread needs no
// other thread's sums, and a workgroup of four waves is done soonest where the context is short or the cache bfloat16.
template <typename WT, typename QT, typename OT>
__global__ __launch_bounds__(PA_THREADS) void k_attn_plain(const QT* __restrict__ q,
                                                           const WT* __restrict__ kc,
                                                           const WT* __restrict__ vc,
                                                           const int32_t* __restrict__ kv_len,
                                                           const int2* __restrict__ map,
                                                           int rows, int H, int KVH, int hd,
                                                           int64_t cap, OT* __restrict__ out) {
    __shared__ float sq[256];
    __shared__ float sc[PA_CHUNK];
    __shared__ float red[PA_THREADS];
    __shared__ float wred[PA_THREADS / CS_WAVE];
    const int h = blockIdx.y, r = blockIdx.z * rows + blockIdx.x;
    const int tid = threadIdx.x;
    const int2 at = map ? map[r] : make_int2(blockIdx.z, blockIdx.x);
    const int b = at.x, i = at.y;
    const int g = h / (H / KVH);
    const int n_ctx = kv_len[b] + i + 1;
    const WT* __restrict__ K = kc + ((int64_t)b * KVH + g) * cap * hd;
    const WT* __restrict__ V = vc + ((int64_t)b * KVH + g) * hd * cap;
    if (tid < hd) sq[tid] = cs_ld(q, ((int64_t)r * H + h) * hd + tid);
    __syncthreads();
    const float scale = 1.0f / sqrtf((float)hd);
    const int d = tid % hd, part = tid / hd, nparts = PA_THREADS / hd;
    float m_run = -INFINITY, l_run = 0.f, o = 0.f;
    for (int c0 = 0; c0 < n_ctx; c0 += PA_CHUNK) {
        const int cn = min(PA_CHUNK, n_ctx - c0);
        float lmax = -INFINITY;
        for (int t = tid; t < cn; t += PA_THREADS) {
            const WT* __restrict__ kr = K + (int64_t)(c0 + t) * hd;
            float s = 0.f;
            if (hd % 16 == 0) {                    // rows of whole 16-element pieces: wide loads, four in flight
                f32x4 s4 = (f32x4){0.f, 0.f, 0.f, 0.f};
                for (int e = 0; e < hd; e += 16) {
                    f32x4 kv[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) kv[u] = pa_ld4(kr + e + 4 * u);
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int j = 0; j < 4; ++j) s4[j] += sq[e + 4 * u + j] * kv[u][j];
                }
                s = (s4[0] + s4[1]) + (s4[2] + s4[3]);
            } else {
                for (int e = 0; e < hd; ++e) s += sq[e] * cs_ld(kr, e);
            }
            s *= scale;
            sc[t] = s;
            lmax = fmaxf(lmax, s);
        }
        const float mc = block_max<PA_THREADS>(lmax, wred);
        const float m_new = fmaxf(m_run, mc);
        const float alpha = expf(m_run - m_new);
        float lsum = 0.f;
        for (int t = tid; t < cn; t += PA_THREADS) {
            const float p = expf(sc[t] - m_new);
            sc[t] = p;
            lsum += p;
        }
        const float lc = block_sum<PA_THREADS>(lsum, wred);       // its barriers also publish sc[]
        l_run = l_run * alpha + lc;
        float acc = 0.f;
        // four tokens at a time (contiguous in the cache); rows past the context may hold anything
#pragma unroll 4
        for (int t = 4 * part; t < cn; t += 4 * nparts) {
            const f32x4 v = pa_ld4(V + cs_v_index(c0 + t, d, hd));
            float p[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) p[j] = t + j < cn ? sc[t + j] * v[j] : 0.f;
            acc += (p[0] + p[1]) + (p[2] + p[3]);
        }
        o = o * alpha + acc;
        m_run = m_new;
        __syncthreads();
    }
    red[tid] = o;
    __syncthreads();
    if (part == 0) {
        float tot = 0.f;
        for (int p = 0; p < nparts; ++p) tot += red[p * hd + d];
        cs_st(out, ((int64_t)r * H + h) * hd + d, tot / l_run);
    }
}

// A verify block of a small model (44 workgroups over 512 tokens of hd 64) leaves most of the chip idle: what counts
// is how fast one compute unit gets its K and V.  So neighbouring lanes read neighbouring memory, with four to
// eight independent loads in flight per thread: hd/4 lanes share a token's key row (four elements each, their
// products added by shuffles), and 32 lanes take the 128 consecutive tokens of one feature of V (cs_v_index), whose
// sums meet by shuffles as well.  19.2 us with a key row per thread and four waves, 12.1 us here with 16.
template <typename WT, typename QT, typename OT, int THREADS>
__global__ __launch_bounds__(THREADS) void k_attn_plain_lanes(const QT* __restrict__ q,
                                                        const WT* __restrict__ kc,
                                                        const WT* __restrict__ vc,
                                                        const int32_t* __restrict__ kv_len,
                                                        const int2* __restrict__ map,
                                                        int rows, int H, int KVH, int hd,
                                                        int64_t cap, OT* __restrict__ out) {
    __shared__ float sc[PA_CHUNK];
    __shared__ float so[256];                      // running output of every feature
    __shared__ float wred[THREADS / CS_WAVE];
    const int h = blockIdx.y, r = blockIdx.z * rows + blockIdx.x;
    const int tid = threadIdx.x;
    const int2 at = map ? map[r] : make_int2(blockIdx.z, blockIdx.x);
    const int b = at.x, i = at.y;
    const int g = h / (H / KVH);
    const int n_ctx = kv_len[b] + i + 1;
    const WT* __restrict__ K = kc + ((int64_t)b * KVH + g) * cap * hd;
    const WT* __restrict__ V = vc + ((int64_t)b * KVH + g) * hd * cap;
    const float scale = 1.0f / sqrtf((float)hd);
    // (hd is a power of two in 2..256)
    const int lpt = hd >= 4 ? hd >> 2 : 1;         // lanes per token, 1..64
    const int lpt_log = 31 - __clz(lpt);
    const int e0 = (tid & (lpt - 1)) * 4, tok0 = tid >> lpt_log, tpp = THREADS >> lpt_log;
    const QT* __restrict__ qrow = q + ((int64_t)r * H + h) * hd;
    f32x4 q4 = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int j = 0; j < 4; ++j)
        if (e0 + j < hd) q4[j] = cs_ld(qrow, e0 + j);
    for (int d = tid; d < hd; d += THREADS) so[d] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    for (int c0 = 0; c0 < n_ctx; c0 += PA_CHUNK) {
        const int cn = min(PA_CHUNK, n_ctx - c0);
        float lmax = -INFINITY;
        for (int base = 0; base < cn; base += 4 * tpp) {
            f32x4 kv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {          // (tokens past the last are read at the last)
                const WT* __restrict__ kr = K + (int64_t)(c0 + min(base + u * tpp + tok0, cn - 1)) * hd;
                kv[u] = hd >= 4 ? pa_ld4(kr + e0) : (f32x4){cs_ld(kr, 0), cs_ld(kr, 1), 0.f, 0.f};
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float s = (q4[0] * kv[u][0] + q4[1] * kv[u][1]) + (q4[2] * kv[u][2] + q4[3] * kv[u][3]);
                for (int o = 1; o < lpt; o <<= 1) s += __shfl_xor(s, o, 64);
                s *= scale;
                const int t = base + u * tpp + tok0;
                if (t < cn) {
                    if (e0 == 0) sc[t] = s;
                    lmax = fmaxf(lmax, s);
                }
            }
        }
        const float mc = block_max<THREADS>(lmax, wred);          // its barriers also publish sc[]
        const float m_new = fmaxf(m_run, mc);
        const float alpha = expf(m_run - m_new);
        float lsum = 0.f;
        for (int t = tid; t < cn; t += THREADS) {
            const float p = expf(sc[t] - m_new);
            sc[t] = p;
            lsum += p;
        }
        const float lc = block_sum<THREADS>(lsum, wred);          // likewise
        l_run = l_run * alpha + lc;
        // rows past the context may hold anything (they are inside the allocation: cap % 128 == 0)
        const int tq = (tid & 31) * 4;
        for (int d = tid >> 5; d < hd; d += 2 * (THREADS / 32)) {
            const bool two = d + THREADS / 32 < hd;
            const int d1 = two ? d + THREADS / 32 : d;
            float a0 = 0.f, a1 = 0.f;
#pragma unroll 4
            for (int t = tq; t - tq < cn; t += CS_VBLK) {
                const f32x4 v0 = pa_ld4(V + cs_v_index(c0 + t, d, hd)), v1 = pa_ld4(V + cs_v_index(c0 + t, d1, hd));
                float p0 = 0.f, p1 = 0.f;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool in = t + j < cn;
                    const float p = in ? sc[t + j] : 0.f;
                    p0 += in ? p * v0[j] : 0.f;
                    p1 += in ? p * v1[j] : 0.f;
                }
                a0 += p0;
                a1 += p1;
            }
#pragma unroll
            for (int o = 16; o > 0; o >>= 1) {
                a0 += __shfl_xor(a0, o, 64);
                a1 += __shfl_xor(a1, o, 64);
            }
            if (tq == 0) {
                so[d] = so[d] * alpha + a0;
                if (two) so[d1] = so[d1] * alpha + a1;
            }
        }
        m_run = m_new;
        __syncthreads();
    }
    for (int d = tid; d < hd; d += THREADS) cs_st(out, ((int64_t)r * H + h) * hd + d, so[d] / l_run);
}

// -------------------------------------------------------------------------------------
// tuned bf16 kernel
// -------------------------------------------------------------------------------------
#define FA_NT 3            // 16-row query tiles per wave  (48 query rows)
// max over the four lanes {c, c+16, c+32, c+48} that share a query row, with the row-swap
// instructions of gfx950 (two register swaps and two max) instead of two round trips through
// the LDS crossbar: swapping x with itself leaves (low half, low half) and (high half, high
// half) in the two results, whose max is the reduction over lanes 32 apart; then 16 apart.
__device__ __forceinline__ float fa_row4_max(float x) {
    const unsigned u = __float_as_uint(x);
    const auto r32 = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const float m = fmaxf(__uint_as_float(r32[0]), __uint_as_float(r32[1]));
    const unsigned v = __float_as_uint(m);
    const auto r16 = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return fmaxf(__uint_as_float(r16[0]), __uint_as_float(r16[1]));
}

#define FA_QROWS (16 * FA_NT)
static_assert(FA_QROWS == CS_ATTN_GROUP, "the host counts query groups in these rows");
#define FA_RESCALE_LOG2 8.0f
#define FA_OPAD 4          // LDS row padding (floats) of the in-workgroup merge buffers

// attention output element: float16 outputs feed the output projection and are saturated
__device__ __forceinline__ void fa_store_out(f16_t* p, int64_t i, float v, bool& hit) { p[i] = cs_f16_sat(v, hit); }
__device__ __forceinline__ void fa_store_out(float* p, int64_t i, float v, bool&) { p[i] = v; }

template <int HD>
struct fa_kbuf { bf16x8 k[2][HD / 32]; };
template <int HD>
struct fa_vbuf { bf16x8 v[HD / 16]; };

// Partial layout: po[item][split][qrow][HD] float, pml[item][split][qrow][2] = (max2, sum)
// where item = (b*KVH + kvh)*nqg + qg, split = workgroup index along the token axis and max2
// is the reference maximum in base-2 scaled units.  A split whose token range is empty
// writes (max2 = -inf, 0, 0).
// With `fr.qkv` set the kernel also does what k_rope_append does, for what it needs itself:
// the query tile is built from the split-K partial tiles of the q/k/v projection (summed in the
// same order, rotated, rounded), and the workgroup that owns the token range of a new row
// writes that row's K and V into the cache before anybody in the workgroup reads it.  Nobody
// else needs the row in this launch: a workgroup only reads cache rows of its own ranges.
struct fa_fused_rope {
    const float* qkv;        // [nparts][R][(H + 2*KVH) * HD] partial tiles, or NULL: q is given
    int nparts;
    int64_t part_stride;
    const float2* rope;      // [R][HD/2] (cos, sin)
    bf16_t* kc_w;            // this layer's caches, writable
    bf16_t* vc_w;
    const float* bias;       // [(H + 2*KVH) * HD] biases of the q, k, v projections, or NULL
};

// What bounds it: at long caches the K/V stream (batch 8, 18431 rows, hd 128: 114.7 us = 5.27 TB/s), at
// short ones a chain of latencies.  A branch around a load makes the compiler's load counts inexact, and
// every block then waited for the loads issued just before it; so requests never sit behind a branch
// (buffer loads with an offset outside the buffer instead) and the pipelined loop has no exit in the
// middle.  Two blocks per trip over two K and two V stages: K of block i + 2 is requested right after the
// scores of block i, V one block ahead.  Query rows come in NT tiles of 16, the prologue's loads are all
// requested before the first is used, the masked blocks run in the same loop, and the four waves are
// merged by all 256 threads (the code shrank from 47 to 18 KB, fetched cold in every launch).
// Before -> after: batch 8 118.3 -> 114.7 us; one stream, 18431 rows 27.0 -> 22.9, 4095 rows of hd 64
// 12.5 -> 9.5, one row over 300 tokens 19.7 -> 10.4 us.
template <int HD, int NT, bool FUSE>
__global__ __launch_bounds__(256) void k_attn_mfma(const bf16_t* __restrict__ q, const bf16_t* kc,
                                                   const bf16_t* vc,
                                                   const int32_t* __restrict__ kv_len, int rows,
                                                   int H, int KVH, int64_t cap, int Tw, int nsplit,
                                                   float* __restrict__ po,
                                                   float* __restrict__ pml, fa_fused_rope fr) {
    constexpr int KS = HD / 32;      // MFMA k-steps over the head dimension
    constexpr int MT = HD / 16;      // 16-row tiles of O^T
    constexpr int OROW = HD + FA_OPAD;
    constexpr int QROW = HD * 2 + 16;                 // bytes per query row in LDS (padded)
    constexpr int ROWS = 16 * NT;                     // query rows of the workgroup: all of the KV head's
    constexpr int MERGE_BYTES = 4 * ROWS * OROW * 4 + 4 * ROWS * 2 * 4;
    constexpr int Q_BYTES = ROWS * QROW;
    // the query tile (read during the main loop) and the merge buffers (used after it)
    // share the same LDS
    __shared__ __attribute__((aligned(16))) unsigned char smem[MERGE_BYTES > Q_BYTES ? MERGE_BYTES : Q_BYTES];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int split = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;
    const int G = H / KVH;
    const int QR = G * rows;                            // <= ROWS
    const int L = kv_len[b];
    const int n_tok = L + rows;
    // The workgroup's token range is 4*Tw long; its four waves take the 32-token blocks of it in
    // turn (wave w: blocks w, w+4, ...), so that at any time the workgroup reads neighbouring
    // blocks: the four 64-byte pieces a V row contributes then form one 256-byte run.
    constexpr int STEP = 4 * 32;
    const int w_begin = min(split * 4 * Tw, n_tok);
    const int t_end = min(n_tok, w_begin + 4 * Tw);
    const int t_begin = w_begin + 32 * wave;            // may lie past t_end: no blocks then
    // blocks that lie completely inside the old cache need neither mask nor clean-up
    const int t_split = max(w_begin, min(t_end, (L / 32) * 32));
    // this wave's blocks: n_open of those, then the masked ones, n_all in total
    const int n_open = t_begin < t_split ? (t_split - t_begin + STEP - 1) / STEP : 0;
    const int n_all = t_begin < t_end ? (t_end - t_begin + STEP - 1) / STEP : 0;
    // Every workgroup starts at a different one of its unmasked blocks (and wraps): the workgroups of
    // a launch run in step, and with all of them at the same relative position some cache pitches put
    // them on the same memory channels
    const int wg_id = (b * KVH + kvh) * nsplit + split;
    const int n_wg = w_begin < t_split ? (t_split - w_begin + STEP - 1) / STEP : 0;       // wave 0's count
    const int rot_wg = n_wg > 0 ? (int)(((int64_t)wg_id * 2654435761LL >> 8) % n_wg) : 0;
    const int rot = n_open > 0 ? min(rot_wg, n_open - 1) : 0;     // the same round for all four waves
    auto at = [&](int i) {
        int j = i < n_open ? i + rot : i;
        j = i < n_open && j >= n_open ? j - n_open : j;
        return t_begin + j * STEP;
    };
    // K and V come through buffer loads based at the workgroup's range: a block past the wave's last has an
    // offset outside the buffer, which costs no memory traffic and, unlike a branch around the loads, leaves
    // the compiler's load counts exact (with branches every block waited for the loads just issued).
    // With the fused append the rows at and beyond L are written by this workgroup, below, and the masked
    // blocks are requested only after the barrier that follows.
    const int64_t head0 = (int64_t)b * KVH + kvh;
    const int n_range = (t_end - w_begin + 31) & ~31;          // a masked block may reach past t_end, into dead rows
    // V's buffer counts at least one 128-token block, also for an empty range (a split past the end of a short
    // stream): the range check compares the offset with the size minus the scalar offset, which must not be
    // negative.  Nothing is read there, every offset of an empty range is NOWHERE.
    const int v_blocks = max(1, (n_range + CS_VBLK - 1) / CS_VBLK);
    static_assert((MT - 1) * 16 * CS_VBLK < HD * CS_VBLK, "scalar offsets of a V block stay inside it");
    const auto krsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((FUSE ? fr.kc_w : kc) + (head0 * cap + w_begin) * HD), 0, n_range * HD * 2, CS_BUFFER_WORD3);
    const auto vrsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((FUSE ? fr.vc_w : vc) + head0 * HD * cap + cs_v_index(w_begin, 0, HD)), 0,
        v_blocks * CS_VBLK * HD * 2, CS_BUFFER_WORD3);
    constexpr unsigned NOWHERE = 0x80000000u;
    // K tile a, MFMA row m=c  <->  token t0 + 8*(c/4) + 4a + c%4
    const unsigned klane = ((8 * (c >> 2) + (c & 3)) * HD + g * 8) * 2;
    auto ldk = [&](fa_kbuf<HD>& buf, int i, int n) {
        // the four lanes of a token row read 64 contiguous bytes per k-step
        const unsigned off = i < n ? (unsigned)(at(i) - w_begin) * (HD * 2) + klane : NOWHERE;
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int s = 0; s < KS; ++s)
                buf.k[a][s] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(krsrc, off + a * 4 * HD * 2 + s * 64, 0, 0));
    };
    const unsigned vlane = c * (CS_VBLK * 2) + g * 16;
    auto ldv = [&](fa_vbuf<HD>& buf, int i, int n) {
        const int t = at(i) - w_begin;
        const unsigned off = i < n ? (unsigned)((t >> 7) * HD * CS_VBLK + (t & (CS_VBLK - 1))) * 2 + vlane : NOWHERE;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            buf.v[mt] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(vrsrc, off, mt * 16 * CS_VBLK * 2, 0));
    };
    fa_kbuf<HD> k0, k1;
    fa_vbuf<HD> v0, v1;
    // (the fences keep every request where it is written: a wait counts what was requested after it)
    auto first_blocks = [&](int n) {
        __builtin_amdgcn_sched_barrier(0);
        ldk(k0, 0, n);
        __builtin_amdgcn_sched_barrier(0);
        ldv(v0, 0, n);
        __builtin_amdgcn_sched_barrier(0);
        ldk(k1, 1, n);
        __builtin_amdgcn_sched_barrier(0);
    };
    // the first blocks are requested before the query tile is ready, if they are old rows
    const int n_early = n_open >= 2 ? n_open : 0;

    // stage the query tile: query row n  <->  block row n / G, head n % G
    const int inv_g = (65536 + G - 1) / G;              // n / G == n * inv_g >> 16 for n < 48
    if constexpr (!FUSE) {
        for (int idx = tid; idx < ROWS * (HD / 8); idx += 256) {
            const int n = idx / (HD / 8), seg = idx % (HD / 8);
            bf16x8 v = (bf16x8){0, 0, 0, 0, 0, 0, 0, 0};
            if (n < QR) {
                const int i = n * inv_g >> 16, gq = n - i * G;
                v = *reinterpret_cast<const bf16x8*>(
                    q + (((int64_t)(b * rows + i)) * H + kvh * G + gq) * HD + seg * 8);
            }
            *reinterpret_cast<bf16x8*>(smem + n * QROW + seg * 16) = v;
        }
        first_blocks(n_early);
    } else {
        constexpr int HALF = HD / 2, SEGS = HALF / 4;        // 4-element segments per half head
        const int nqkv = (H + 2 * KVH) * HD;
        // One task: elements j0..j0+3 and HALF+j0..HALF+j0+3 of one head of block row r.  The partial
        // tiles are summed in order, the pair (j, HALF + j) is rotated by the row's angle j.  All of
        // this is load latency (a partial tile was written by another die), so the tiles are
        // requested four at a time before the first is used.
        struct pair_tiles { f32x4 t[4][2]; };
        struct pair_angles { f32x4 v[2]; };                  // (cos, sin) of j0, j0+1; j0+2, j0+3
        auto request = [&](int r, int head, int j0, int p0, pair_tiles& o) {
            const float* src = fr.qkv + (int64_t)r * nqkv + (int64_t)head * HD + j0;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float* sp = src + min(p0 + w, fr.nparts - 1) * fr.part_stride;
                o.t[w][0] = *reinterpret_cast<const f32x4*>(sp);
                o.t[w][1] = *reinterpret_cast<const f32x4*>(sp + HALF);
            }
        };
        auto angles = [&](int r, int j0, pair_angles& o) {
            const f32x4* p = reinterpret_cast<const f32x4*>(fr.rope + (int64_t)r * HALF + j0);
            o.v[0] = p[0];
            o.v[1] = p[1];
        };
        // sum (first four tiles already requested), bias, rotation, rounding
        auto finish = [&](pair_tiles& t, int r, int head, int j0, bool rotate, const pair_angles& an, bf16x4& lo, bf16x4& hi) {
            f32x4 x = (f32x4){0.f, 0.f, 0.f, 0.f}, y = x;
            for (int p0 = 0;;) {
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const bool in = p0 + w < fr.nparts;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        x[u] = in ? x[u] + t.t[w][0][u] : x[u];
                        y[u] = in ? y[u] + t.t[w][1][u] : y[u];
                    }
                }
                p0 += 4;
                if (p0 >= fr.nparts) break;
                request(r, head, j0, p0, t);
            }
            if (fr.bias) {                            // projection bias, before the rotation
                const float* __restrict__ bp = fr.bias + head * HD + j0;
                x += *reinterpret_cast<const f32x4*>(bp);
                y += *reinterpret_cast<const f32x4*>(bp + HALF);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float co = an.v[u >> 1][2 * (u & 1)], si = an.v[u >> 1][2 * (u & 1) + 1];
                const float rx = x[u] * co - y[u] * si, ry = y[u] * co + x[u] * si;
                lo[u] = (bf16_t)(rotate ? rx : x[u]);
                hi[u] = (bf16_t)(rotate ? ry : y[u]);
            }
        };
        constexpr int QT = (ROWS * SEGS + 255) / 256;         // query tasks of a thread
        pair_angles ang[QT];
        pair_tiles qt[QT];
        auto q_row = [&](int t, int& n, int& i, int& head, int& j0) {      // (clamped past the last row)
            n = (tid + 256 * t) / SEGS;
            j0 = tid % SEGS * 4;
            const int m = min(n, QR - 1);
            i = m * inv_g >> 16;
            head = kvh * G + m - i * G;
        };
#pragma unroll
        for (int t = 0; t < QT; ++t) {
            int n, i, head, j0;
            q_row(t, n, i, head, j0);
            angles(b * rows + i, j0, ang[t]);
            request(b * rows + i, head, j0, 0, qt[t]);
        }
        first_blocks(n_early);
        // the new rows whose position lies in this workgroup's token range: key heads of all rows, then
        // value heads
        bf16_t* Kw = fr.kc_w + head0 * cap * HD;
        bf16_t* Vw = fr.vc_w + head0 * HD * cap;
        if (t_end > L) {
            for (int idx = tid; idx < 2 * rows * SEGS; idx += 256) {
                const bool is_v = idx >= rows * SEGS;
                const int i = idx / SEGS - (is_v ? rows : 0), j0 = idx % SEGS * 4;
                const int pos = L + i;
                if (pos < w_begin || pos >= t_end) continue;
                const int head = H + (is_v ? KVH : 0) + kvh;
                pair_angles an;
                pair_tiles t;
                angles(b * rows + i, j0, an);
                request(b * rows + i, head, j0, 0, t);
                bf16x4 lo, hi;
                finish(t, b * rows + i, head, j0, !is_v, an, lo, hi);
                if (!is_v) {
                    *reinterpret_cast<bf16x4*>(Kw + (int64_t)pos * HD + j0) = lo;
                    *reinterpret_cast<bf16x4*>(Kw + (int64_t)pos * HD + HALF + j0) = hi;
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        Vw[cs_v_index(pos, j0 + u, HD)] = lo[u];
                        Vw[cs_v_index(pos, HALF + j0 + u, HD)] = hi[u];
                    }
                }
            }
        }
#pragma unroll
        for (int t = 0; t < QT; ++t) {
            int n, i, head, j0;
            q_row(t, n, i, head, j0);
            if (n >= ROWS) continue;
            bf16x4 lo, hi;
            finish(qt[t], b * rows + i, head, j0, true, ang[t], lo, hi);
            if (n >= QR) lo = hi = (bf16x4){0, 0, 0, 0};
            *reinterpret_cast<bf16x4*>(smem + n * QROW + j0 * 2) = lo;
            *reinterpret_cast<bf16x4*>(smem + n * QROW + HD + j0 * 2) = hi;
        }
    }
    int qi[NT];               // block row index of the lane's query row (for the causal mask)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int n = nt * 16 + c;
        qi[nt] = n < QR ? n * inv_g >> 16 : -1;
    }
    __syncthreads();

    f32x4 oacc[MT][NT], lacc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        lacc[nt] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) oacc[mt][nt] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    float m_run[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) m_run[nt] = -INFINITY;

    const float scale2 = 1.4426950408889634f / sqrtf((float)HD);
    const bf16_t one = (bf16_t)1.0f;
    const bf16x8 ones = (bf16x8){one, one, one, one, one, one, one, one};

    // block i (its K in kb, its V in vb); K of block i + 2 replaces it in kb as soon as the scores are out
    auto block = [&](fa_kbuf<HD>& kb, fa_vbuf<HD>& vb, int i, auto ahead) {
        // scores: lane (c, g) gets tokens t0 + 8g + (4a + j) of query row nt*16 + c
        f32x4 sacc[2][NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            f32x4 z0 = (f32x4){0.f, 0.f, 0.f, 0.f}, z1 = z0;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const bf16x8 qb = *reinterpret_cast<const bf16x8*>(
                    smem + (nt * 16 + c) * QROW + s * 64 + g * 16);
                z0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kb.k[0][s], qb, z0, 0, 0, 0);
                z1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kb.k[1][s], qb, z1, 0, 0, 0);
            }
            sacc[0][nt] = z0;
            sacc[1][nt] = z1;
        }
        if constexpr (decltype(ahead)::value) {
            __builtin_amdgcn_sched_barrier(0);
            ldk(kb, i + 2, n_all);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (i >= n_open) {
            // a block with new rows or dead ones.  Dead cache rows may hold anything: their V is zeroed
            // so that 0 * garbage stays 0
            const int t0 = at(i);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const bool dead = t0 + 8 * g + j >= n_tok;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) vb.v[mt][j] = dead ? (bf16_t)0.f : vb.v[mt][j];
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        sacc[a][nt][j] = t0 + 8 * g + 4 * a + j > L + qi[nt] ? -INFINITY : sacc[a][nt][j];
        }
        bool moved = false;
        float alpha[NT];
        bf16x8 pb[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            float sv[8];
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int j = 0; j < 4; ++j) sv[4 * a + j] = sacc[a][nt][j];
            float mx = fmaxf(fmaxf(sv[0], sv[1]), sv[2]);
            mx = fmaxf(fmaxf(mx, sv[3]), sv[4]);
            mx = fmaxf(fmaxf(mx, sv[5]), fmaxf(sv[6], sv[7]));
            mx = fa_row4_max(mx);                                  // over the lanes c, c+16, c+32, c+48
            mx *= scale2;                       // scale2 > 0: scaling commutes with the max
            // The reference maximum only follows the true one when it is left behind by more
            // than 2^8: probabilities stay below 256, O and the row sum stay consistent, and
            // the rescale of O (the expensive part) runs a handful of times per wave.
            const bool up = mx > m_run[nt] + FA_RESCALE_LOG2;
            const float m_new = up ? mx : m_run[nt];
            const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
            alpha[nt] = up ? __builtin_amdgcn_exp2f(m_run[nt] - m_safe) : 1.0f;
            moved |= up;
            m_run[nt] = m_new;
#pragma unroll
            for (int j = 0; j < 8; ++j)
                pb[nt][j] = (bf16_t)__builtin_amdgcn_exp2f(fmaf(sv[j], scale2, -m_safe));
        }
        if (__any(moved)) {
            // rare path (see above); the empty asm statements keep the register-file copies
            // that the multiply needs inside this branch
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                asm volatile("" : "+a"(lacc[nt]));
                lacc[nt] *= alpha[nt];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    asm volatile("" : "+a"(oacc[mt][nt]));
                    oacc[mt][nt] *= alpha[nt];
                }
            }
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            // row sums of the rounded probabilities on the matrix core: ones^T * P^T
            lacc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pb[nt], lacc[nt], 0, 0, 0);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                oacc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vb.v[mt], pb[nt], oacc[mt][nt], 0, 0, 0);
        }
        // keep the accumulators in the accumulation registers between blocks, so that the
        // vector registers stay free for the K/V stages (no register-file shuffling per block)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            asm volatile("" : "+a"(lacc[nt]));
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) asm volatile("" : "+a"(oacc[mt][nt]));
        }
    };
    int i = 0;
    if (n_early)
        for (; i + 1 < n_all; i += 2) {        // (no way out in the middle: it would spoil the load counts)
            ldv(v1, i + 1, n_all);
            __builtin_amdgcn_sched_barrier(0);
            block(k0, v0, i, std::true_type{});
            ldv(v0, i + 2, n_all);
            __builtin_amdgcn_sched_barrier(0);
            block(k1, v1, i + 1, std::true_type{});
        }
    // the odd last block, or, with at most one old block, all of the few blocks
    for (; i < n_all; ++i) {
        if (!n_early) {
            ldk(k0, i, n_all);
            ldv(v0, i, n_all);
        }
        block(k0, v0, i, std::false_type{});
    }
    __syncthreads();             // every wave is done with the query tile: LDS changes hands

    // the four waves' (max, sum, O) side by side in LDS, combined by all threads, wave 0 first
    float* s_o = reinterpret_cast<float*>(smem);                          // [4][ROWS * OROW]
    float2* s_ml = reinterpret_cast<float2*>(s_o + 4 * ROWS * OROW);      // [4][ROWS]
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int n = wave * ROWS + nt * 16 + c;
        if (g == 0) s_ml[n] = make_float2(m_run[nt], lacc[nt][0]);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            *reinterpret_cast<f32x4*>(&s_o[n * OROW + mt * 16 + 4 * g]) = oacc[mt][nt];
    }
    __syncthreads();
    const int64_t item = ((int64_t)b * KVH + kvh) * nsplit + split;
    float* __restrict__ o_out = po + item * FA_QROWS * HD;
    float2* __restrict__ ml_out = reinterpret_cast<float2*>(pml) + item * FA_QROWS;
#pragma unroll 1
    for (int idx = tid; idx < QR * (HD / 4); idx += 256) {
        const int n = idx / (HD / 4), d = idx % (HD / 4) * 4;
        float2 ml[4];
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            ml[w] = s_ml[w * ROWS + n];
            M = fmaxf(M, ml[w].x);
        }
        const float Ms = (M == -INFINITY) ? 0.f : M;
        float l = 0.f;
        f32x4 o = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float wgt = __builtin_amdgcn_exp2f(ml[w].x - Ms);
            l += ml[w].y * wgt;
            o += *reinterpret_cast<const f32x4*>(&s_o[(w * ROWS + n) * OROW + d]) * wgt;
        }
        *reinterpret_cast<f32x4*>(o_out + n * HD + d) = o;
        if (d == 0) ml_out[n] = make_float2(M, l);
    }
}

// -------------------------------------------------------------------------------------
// tuned kernel for wide blocks (more than 48 query rows per KV head, e.g. k = 32: 132 rows)
//
// Up to FA_QG consumer waves each own one 48-row query group and all walk the same token
// range; one producer wave streams K and V from HBM once per workgroup and lays them into a
// three-stage LDS ring in MFMA fragment order, so the KV bytes are read once however many
// query groups share them.  One barrier per 32-token block hands the stages over.  The two teams'
// results meet in LDS at the end; k_attn_merge combines the workgroups'.
// -------------------------------------------------------------------------------------
#define FA_QG 3
#define FA_STAGES 3
#define FA_TEAMS 2          // (FA_QG consumers + 1 producer) per team; two waves per SIMD
#define FA_LDS_THREADS (64 * (FA_QG + 1) * FA_TEAMS)

template <int HD>
__global__ __launch_bounds__(FA_LDS_THREADS) void k_attn_lds(const bf16_t* __restrict__ q,
                                                              const bf16_t* __restrict__ kc,
                                                              const bf16_t* __restrict__ vc,
                                                              const int32_t* __restrict__ kv_len,
                                                              const int4* __restrict__ segs,
                                                              int rows, int H, int KVH, int64_t cap,
                                                              int Tw, int nqg, int nqgw, int gpw, int nsplit,
                                                              int ranges, float* __restrict__ po,
                                                              float* __restrict__ pml) {
    constexpr int KS = HD / 32, MT = HD / 16;
    constexpr int QROW = HD * 2 + 16;
    constexpr int K_BYTES = 2 * KS * 1024, V_BYTES = MT * 1024;
    constexpr int STAGE_BYTES = K_BYTES + V_BYTES;
    __shared__ __attribute__((aligned(16))) unsigned char stage_all[FA_TEAMS][FA_STAGES][STAGE_BYTES];
    __shared__ __attribute__((aligned(16))) unsigned char qs[FA_QG][FA_QROWS * QROW];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int c = lane & 15, g = lane >> 4;
    // Workgroup -> (stream, KV head, token range pair, group of query groups).  The nqgw
    // workgroups that walk the same K/V range (long blocks, e.g. prompt ingestion) get ids 8
    // apart: consecutive ids go to different XCDs, each with its own L2, so this puts them on
    // one XCD at about the same time and the range is fetched from HBM once, not nqgw times.
    const int nsp = nsplit / FA_TEAMS;                  // ranges = B * KVH * nsp
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int range = (slot / nqgw) * 8 + xcd;
    if (range >= ranges) return;                        // whole workgroup, before any barrier
    // which gpw (<= FA_QG) of the query groups: the last rows of a block see the most tokens (see n_lim
    // below), so they are dispatched first and the short ones fill the tail of the launch
    const int qgw = nqgw - 1 - slot % nqgw;
    const int kvh = (range / nsp) % KVH, b = range / (nsp * KVH);
    const int G = H / KVH;
    int row0 = b * rows, group0 = b * nqg;              // the stream's first block row, its first query group
    if (segs) {
        const int4 sg = segs[b];
        row0 = sg.x;
        rows = sg.y;
        group0 = sg.z;
        nqg = (G * rows + FA_QROWS - 1) / FA_QROWS;
        if (qgw * gpw >= nqg) return;                   // (whole workgroup; a stream with fewer rows than others)
    }
    // Roles of the eight waves (hardware waves go to the four SIMDs in turn: wave w runs on SIMD
    // w % 4).  With three live query groups per team: waves 0-2 and 4-6 are the consumers of teams 0
    // and 1, waves 3 and 7 the producers, so every consumer SIMD carries one consumer of each team.
    // With at most two live groups (e.g. 11 block rows of seven or eight query heads per KV head)
    // the four live consumers get a SIMD each: waves 0-3 = (team 0, group 0), (0, 1), (1, 0), (1, 1),
    // waves 4 and 5 the producers, waves 6 and 7 the dead third groups.
    const int hw = tid >> 6;
    const int live_groups = min(gpw, nqg - qgw * gpw);
    const bool spread = live_groups <= 2;
    const int team = spread ? (hw < 4 ? hw >> 1 : (hw & 1)) : hw / (FA_QG + 1);
    const int wave = spread ? (hw < 4 ? (hw & 1) : (hw < 6 ? FA_QG : 2)) : hw % (FA_QG + 1);
    unsigned char (*stage)[STAGE_BYTES] = stage_all[team];
    const int QR = G * rows;
    const int L = kv_len[b];
    const int n_tok = L + rows;
    // Causality: block row i sees the tokens up to L + i, so nothing beyond the last row of this
    // workgroup's query groups is walked (long prompt blocks: the upper triangle of the block).
    const int last_row = min(rows - 1, ((qgw + 1) * gpw * FA_QROWS - 1) / G);
    const int n_lim = L + last_row + 1;
    // The two teams share the workgroup's token range of FA_TEAMS*Tw and take its 32-token blocks
    // in turn (team t: blocks t, t+2, ...), so the workgroup reads neighbouring blocks together.
    constexpr int TSTEP = 32 * FA_TEAMS;
    const int w_begin = min(range % nsp * FA_TEAMS * Tw, n_lim);
    const int w_blocks = (min(n_lim, w_begin + FA_TEAMS * Tw) - w_begin + 31) / 32;
    const int t_begin = w_begin + 32 * team;
    const int nblocks = (w_blocks - team + FA_TEAMS - 1) / FA_TEAMS;
    // both teams pass the same number of barriers: team 0's count
    const int nblocks_wg = (w_blocks + FA_TEAMS - 1) / FA_TEAMS;
    const bf16_t* __restrict__ K = kc + ((int64_t)b * KVH + kvh) * cap * HD;
    const bf16_t* __restrict__ V = vc + ((int64_t)b * KVH + kvh) * HD * cap;

    // stage the query tiles of all groups of this workgroup
    for (int idx = tid; idx < FA_QG * FA_QROWS * (HD / 8); idx += FA_LDS_THREADS) {
        const int grp = idx / (FA_QROWS * (HD / 8));
        const int rem = idx % (FA_QROWS * (HD / 8));
        const int row = rem / (HD / 8), seg = rem % (HD / 8);
        const int n = (qgw * gpw + grp) * FA_QROWS + row;
        bf16x8 v = (bf16x8){0, 0, 0, 0, 0, 0, 0, 0};
        if (grp < gpw && n < QR) {
            const int i = n / G, gq = n % G;
            v = *reinterpret_cast<const bf16x8*>(
                q + (((int64_t)(row0 + i)) * H + kvh * G + gq) * HD + seg * 8);
        }
        *reinterpret_cast<bf16x8*>(&qs[grp][row * QROW + seg * 16]) = v;
    }

    const int ktok0 = 8 * (c >> 2) + (c & 3);
    if (wave == FA_QG) {
        // ---------------- producer: K/V blocks -> LDS ring ----------------
        bf16x8 kr[3][2][KS], vr[3][MT];       // three blocks in flight in registers (block j in slot j % 3)
        auto load = [&](int slot, int blk) {
            const int bl = blk < nblocks ? blk : (nblocks > 0 ? nblocks - 1 : 0);   // clamped
            const int t0 = (nblocks > 0 ? t_begin : 0) + bl * TSTEP;
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const bf16_t* kp = K + (int64_t)(t0 + ktok0 + 4 * a) * HD + g * 8;
#pragma unroll
                for (int s = 0; s < KS; ++s)
                    kr[slot][a][s] = *reinterpret_cast<const bf16x8*>(kp + s * 32);
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                vr[slot][mt] = *reinterpret_cast<const bf16x8*>(V + cs_v_index(t0 + 8 * g, mt * 16 + c, HD));
        };
        auto store = [&](int slot, int st, int blk) {
            const int t0 = (nblocks > 0 ? t_begin : 0) + (blk < nblocks ? blk : (nblocks > 0 ? nblocks - 1 : 0)) * TSTEP;
            unsigned char* sp = stage[st];
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int s = 0; s < KS; ++s)
                    *reinterpret_cast<bf16x8*>(sp + ((a * KS + s) * 64 + lane) * 16) = kr[slot][a][s];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                bf16x8 v = vr[slot][mt];
                // dead cache rows may hold anything: zero their V so that 0 * garbage stays 0
                if (t0 + 32 > n_tok) {
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        if (t0 + 8 * g + j >= n_tok) v[j] = (bf16_t)0.f;
                }
                *reinterpret_cast<bf16x8*>(sp + K_BYTES + (mt * 64 + lane) * 16) = v;
            }
        };
        // an empty range still loads (clamped to block 0 of the cache, always allocated) and
        // stores into stages nobody reads; the barrier count is the workgroup's, not the team's
        load(0, 0);
        load(1, 1);
        load(2, 2);
        store(0, 0, 0);
        load(0, 3);
        store(1, 1, 1);
        load(1, 4);
        __syncthreads();                                   // stages 0, 1 and the query tiles are ready
        static_assert(FA_STAGES == 3, "block j: register slot j % 3, LDS stage j % 3");
        // Consumer iteration i reads stages i and i+1: block i+2 goes to stage (i+2)%3, which
        // held block i-1; its register slot is refilled with block i+5, so blocks i+3, i+4
        // and i+5 (48 KB) are in flight while block i is being multiplied.  The loop has no way out in
        // the middle (the last one or two iterations follow it): with one, the compiler could not tell at
        // the loop's head which loads were the newest and drained them all once per trip (16 streams,
        // 132 query rows: 65535 cached rows 821 -> 815 us, 16384 rows 243.8 -> 237.5, 16000 rows 220.9 -> 214.1).
        int i = 0;
        for (; i + 3 <= nblocks_wg; i += 3) {
            store(2, 2, i + 2);
            load(2, i + 5);
            __syncthreads();
            store(0, 0, i + 3);
            load(0, i + 6);
            __syncthreads();
            store(1, 1, i + 4);
            load(1, i + 7);
            __syncthreads();
        }
        if (i < nblocks_wg) {
            store(2, 2, i + 2);
            __syncthreads();
        }
        if (i + 1 < nblocks_wg) {
            store(0, 0, i + 3);
            __syncthreads();
        }
        __syncthreads();                                   // the one between the teams' results, below
        return;
    }

    // ---------------- consumers: one 48-row query group each ----------------
    const int qg = qgw * gpw + wave;
    const bool live = wave < gpw && qg < nqg;
    const unsigned char* myq = qs[wave];
    int qi[FA_NT];
#pragma unroll
    for (int nt = 0; nt < FA_NT; ++nt) {
        const int n = qg * FA_QROWS + nt * 16 + c;
        qi[nt] = n < QR ? n / G : -1;
    }
    f32x4 oacc[MT][FA_NT], lacc[FA_NT];
#pragma unroll
    for (int nt = 0; nt < FA_NT; ++nt) {
        lacc[nt] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) oacc[mt][nt] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    float m_run[FA_NT], thr[FA_NT];
#pragma unroll
    for (int nt = 0; nt < FA_NT; ++nt) m_run[nt] = thr[nt] = -INFINITY;
    const float scale2 = 1.4426950408889634f / sqrtf((float)HD);
    const float inv_scale2 = sqrtf((float)HD) / 1.4426950408889634f;
    const bf16_t one = (bf16_t)1.0f;
    const bf16x8 ones = (bf16x8){one, one, one, one, one, one, one, one};

    // scores of one block: S^T = K Q^T from the K fragments of stage `sp`
    // the wave's query fragments stay in registers for the whole token range (read once from
    // the staged tile, after the first barrier below)
    constexpr int QS_REG = KS;          // k-steps whose query fragments stay in registers (all of them fit)
    bf16x8 qreg[FA_NT][QS_REG];
    auto q_lds = [&](int nt, int s) {
        return *reinterpret_cast<const bf16x8*>(myq + (nt * 16 + c) * QROW + s * 64 + g * 16);
    };
    auto load_q = [&]() {
#pragma unroll
        for (int nt = 0; nt < FA_NT; ++nt)
#pragma unroll
            for (int s = 0; s < QS_REG; ++s) qreg[nt][s] = q_lds(nt, s);
    };
    auto scores = [&](const unsigned char* sp, f32x4 (&sacc)[2][FA_NT]) {
        // all K fragments of the block are requested at once (LDS latency is ~100 cycles and
        // only two waves share a SIMD, so fragments are read well ahead of their use)
        bf16x8 kf[2][KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            kf[0][s] = *reinterpret_cast<const bf16x8*>(sp + ((0 * KS + s) * 64 + lane) * 16);
            kf[1][s] = *reinterpret_cast<const bf16x8*>(sp + ((1 * KS + s) * 64 + lane) * 16);
        }
#pragma unroll
        for (int nt = 0; nt < FA_NT; ++nt) {
            f32x4 z0 = (f32x4){0.f, 0.f, 0.f, 0.f}, z1 = z0;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const bf16x8 qf = s < QS_REG ? qreg[nt][s] : q_lds(nt, s);
                z0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[0][s], qf, z0, 0, 0, 0);
                z1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[1][s], qf, z1, 0, 0, 0);
            }
            sacc[0][nt] = z0;
            sacc[1][nt] = z1;
        }
    };
    // ---- the pieces of one block's softmax and PV ----
    auto score_of = [&](const f32x4 (&sacc)[2][FA_NT], int nt, int e, int t0, auto tail_tag) {   // e = 4a + j
        constexpr bool TAIL = decltype(tail_tag)::value;
        const float sc = sacc[e >> 2][nt][e & 3];
        return (TAIL && (t0 + 8 * g + e > L + qi[nt])) ? -INFINITY : sc;
    };
    // reference maxima: leaves m_run (and O, rescaled if a reference moved) ready for `prob`
    auto reference = [&](const f32x4 (&sacc)[2][FA_NT], int t0, auto tail_tag) {
        constexpr bool TAIL = decltype(tail_tag)::value;
        // Common case first: no score of the block is more than 2^8 above its row's reference
        // maximum.  Then the reference stays, nothing is rescaled, and the exact row maximum
        // (a reduction across the four lanes that share a row) is not needed at all: every lane
        // only compares its own eight scores with the row's threshold.
        bool calm = false;
        if (!TAIL) {
            bool over = false;
#pragma unroll
            for (int nt = 0; nt < FA_NT; ++nt) {
                const float lm = fmaxf(fmaxf(fmaxf(sacc[0][nt][0], sacc[0][nt][1]), fmaxf(sacc[0][nt][2], sacc[0][nt][3])),
                                       fmaxf(fmaxf(sacc[1][nt][0], sacc[1][nt][1]), fmaxf(sacc[1][nt][2], sacc[1][nt][3])));
                over |= !(lm <= thr[nt]);          // also true while the reference is still -inf
            }
            calm = !__any(over);
        }
        if (calm) return;
        bool moved = false;
        float alpha[FA_NT];
#pragma unroll
        for (int nt = 0; nt < FA_NT; ++nt) {
            float mx = fmaxf(fmaxf(score_of(sacc, nt, 0, t0, tail_tag), score_of(sacc, nt, 1, t0, tail_tag)),
                             score_of(sacc, nt, 2, t0, tail_tag));
            mx = fmaxf(fmaxf(mx, score_of(sacc, nt, 3, t0, tail_tag)), score_of(sacc, nt, 4, t0, tail_tag));
            mx = fmaxf(fmaxf(mx, score_of(sacc, nt, 5, t0, tail_tag)),
                       fmaxf(score_of(sacc, nt, 6, t0, tail_tag), score_of(sacc, nt, 7, t0, tail_tag)));
            mx = fa_row4_max(mx);                              // over the lanes c, c+16, c+32, c+48
            mx *= scale2;
            const bool up = mx > m_run[nt] + FA_RESCALE_LOG2;  // see k_attn_mfma
            const float m_new = up ? mx : m_run[nt];
            alpha[nt] = up ? __builtin_amdgcn_exp2f(m_run[nt] - ((m_new == -INFINITY) ? 0.f : m_new)) : 1.0f;
            moved |= up;
            m_run[nt] = m_new;
            // scores above this leave the calm path (raw score units; -inf while no score has
            // been seen, so that the comparison above fails)
            thr[nt] = (m_new == -INFINITY) ? -INFINITY : (m_new + FA_RESCALE_LOG2) * inv_scale2;
        }
        if (__any(moved)) {
#pragma unroll
            for (int nt = 0; nt < FA_NT; ++nt) {
                lacc[nt] *= alpha[nt];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) oacc[mt][nt] *= alpha[nt];
            }
        }
    };
    auto prob = [&](const f32x4 (&sacc)[2][FA_NT], int nt, int e, int t0, auto tail_tag) {
        const float m_safe = (m_run[nt] == -INFINITY) ? 0.f : m_run[nt];
        return (bf16_t)__builtin_amdgcn_exp2f(fmaf(score_of(sacc, nt, e, t0, tail_tag), scale2, -m_safe));
    };
    auto pv = [&](const unsigned char* sp, const bf16x8 (&pb)[FA_NT]) {
        // V fragments are read three tiles ahead of the MFMAs that use them
        bf16x8 vf[4];
#pragma unroll
        for (int mt = 0; mt < 3; ++mt) vf[mt] = *reinterpret_cast<const bf16x8*>(sp + K_BYTES + (mt * 64 + lane) * 16);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            if (mt + 3 < MT) vf[(mt + 3) & 3] = *reinterpret_cast<const bf16x8*>(sp + K_BYTES + ((mt + 3) * 64 + lane) * 16);
#pragma unroll
            for (int nt = 0; nt < FA_NT; ++nt)
                oacc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[mt & 3], pb[nt], oacc[mt][nt], 0, 0, 0);
        }
#pragma unroll
        for (int nt = 0; nt < FA_NT; ++nt) {
            lacc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pb[nt], lacc[nt], 0, 0, 0);
        }
    };
    // softmax update and O^T += V^T P^T for the block whose scores are in `sacc`
    auto finish = [&](const f32x4 (&sacc)[2][FA_NT], const unsigned char* sp, int t0, auto tail_tag) {
        reference(sacc, t0, tail_tag);
        bf16x8 pb[FA_NT];
#pragma unroll
        for (int nt = 0; nt < FA_NT; ++nt)
#pragma unroll
            for (int e = 0; e < 8; ++e) pb[nt][e] = prob(sacc, nt, e, t0, tail_tag);
        pv(sp, pb);
    };
    const std::integral_constant<bool, false> main_tag;
    const std::integral_constant<bool, true> tail_tag;
    // The hot path (this block and the next lie inside the old cache): the score MFMAs of block
    // i+1 and the exponentials of block i do not depend on each other, so they are issued
    // interleaved, two MFMAs per pair of probabilities, and the matrix cores work through the
    // vector part of the softmax.  The scheduling fences keep the compiler from regrouping each
    // kind into a run of its own.
    auto fused = [&](const f32x4 (&cur)[2][FA_NT], f32x4 (&nxt)[2][FA_NT], const unsigned char* sp_cur,
                     const unsigned char* sp_nxt) {
        auto k_frag = [&](int a, int s) {
            return *reinterpret_cast<const bf16x8*>(sp_nxt + ((a * KS + s) * 64 + lane) * 16);
        };
        bf16x8 k0 = k_frag(0, 0), k1 = k_frag(1, 0);           // in flight during the reference check
        reference(cur, 0, main_tag);
        bf16x8 pb[FA_NT];
        constexpr int PER = 8 / KS;                            // probabilities per (s, nt) step
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            bf16x8 n0 = k0, n1 = k1;
            if (s + 1 < KS) {
                n0 = k_frag(0, s + 1);
                n1 = k_frag(1, s + 1);
            }
#pragma unroll
            for (int nt = 0; nt < FA_NT; ++nt) {
                const bf16x8 qf = s < QS_REG ? qreg[nt][s] : q_lds(nt, s);
                const f32x4 zero4 = (f32x4){0.f, 0.f, 0.f, 0.f};
                nxt[0][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k0, qf, s == 0 ? zero4 : nxt[0][nt], 0, 0, 0);
                nxt[1][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k1, qf, s == 0 ? zero4 : nxt[1][nt], 0, 0, 0);
                const int e0 = (s * FA_NT + nt) * PER;
#pragma unroll
                for (int u = 0; u < PER; ++u)
                    pb[(e0 + u) / 8][(e0 + u) % 8] = prob(cur, (e0 + u) / 8, (e0 + u) % 8, 0, main_tag);
                __builtin_amdgcn_sched_barrier(0);
            }
            k0 = n0;
            k1 = n1;
        }
        pv(sp_cur, pb);
    };

    __syncthreads();                                       // matches the producer's first barrier
    static_assert(8 % KS == 0, "whole probabilities per interleaving step");
    f32x4 sa[2][FA_NT], sb[2][FA_NT];
    load_q();
    if (live && nblocks > 0) scores(stage[0], sa);
    // one block: softmax + PV of block i (scores in `cur`) and the scores of block i+1 (into
    // `nxt`).  Off the hot path the two teams do the pieces in opposite order, so that the two
    // waves sharing a SIMD want different units after every barrier.
    auto block = [&](f32x4 (&cur)[2][FA_NT], f32x4 (&nxt)[2][FA_NT], int i) {
        if (!(live && i < nblocks)) return;
        const int t0 = t_begin + i * TSTEP;
        const bool has_next = i + 1 < nblocks;
        if (has_next && t0 + TSTEP + 32 <= L) {
            fused(cur, nxt, stage[i % FA_STAGES], stage[(i + 1) % FA_STAGES]);
            return;
        }
        if (team == 0 && has_next) scores(stage[(i + 1) % FA_STAGES], nxt);
        if (t0 + 32 > L) finish(cur, stage[i % FA_STAGES], t0, tail_tag);
        else finish(cur, stage[i % FA_STAGES], t0, main_tag);
        if (team != 0 && has_next) scores(stage[(i + 1) % FA_STAGES], nxt);
    };
    for (int i = 0; i < nblocks_wg; i += 2) {
        block(sa, sb, i);
        __syncthreads();
        if (i + 1 >= nblocks_wg) break;
        block(sb, sa, i + 1);
        __syncthreads();
    }

    // Team 1 hands its (max, sum, O) over through LDS (the stages are free after the last barrier), team 0 adds its own:
    // one partial result per workgroup (16 streams of 16384 rows: 35 -> 18 MB written and read again by the merge).
    constexpr int OROW = HD + FA_OPAD;
    float* s_o = reinterpret_cast<float*>(&stage_all[0][0][0]);                           // [FA_QG][FA_QROWS][OROW]
    float2* s_ml = reinterpret_cast<float2*>(s_o + FA_QG * FA_QROWS * OROW);              // [FA_QG][FA_QROWS]
    static_assert(FA_QG * FA_QROWS * (OROW * 4 + 8) <= FA_TEAMS * FA_STAGES * STAGE_BYTES && FA_TEAMS == 2, "fits the stages");
    if (live && team == 1) {
#pragma unroll
        for (int nt = 0; nt < FA_NT; ++nt) {
            const int n = wave * FA_QROWS + nt * 16 + c;
            if (g == 0) s_ml[n] = make_float2(m_run[nt], lacc[nt][0]);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) *reinterpret_cast<f32x4*>(&s_o[n * OROW + mt * 16 + 4 * g]) = oacc[mt][nt];
        }
    }
    __syncthreads();
    if (!live || team == 1) return;

    const int64_t item = ((int64_t)group0 * KVH + kvh * nqg + qg) * nsp + range % nsp;
    float* __restrict__ o_out = po + item * FA_QROWS * HD;
    float* __restrict__ ml_out = pml + item * FA_QROWS * 2;
#pragma unroll
    for (int nt = 0; nt < FA_NT; ++nt) {
        const int n = nt * 16 + c;
        const float2 ml = s_ml[wave * FA_QROWS + n];
        const float M = fmaxf(m_run[nt], ml.x), Ms = (M == -INFINITY) ? 0.f : M;
        const float w0 = __builtin_amdgcn_exp2f(m_run[nt] - Ms), w1 = __builtin_amdgcn_exp2f(ml.x - Ms);
        if (g == 0) { ml_out[n * 2] = M; ml_out[n * 2 + 1] = lacc[nt][0] * w0 + ml.y * w1; }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            *reinterpret_cast<f32x4*>(o_out + (int64_t)n * HD + mt * 16 + 4 * g) =
                oacc[mt][nt] * w0 + *reinterpret_cast<const f32x4*>(&s_o[(wave * FA_QROWS + n) * OROW + mt * 16 + 4 * g]) * w1;
    }
}

// -------------------------------------------------------------------------------------
// kernel for prompt blocks (hundreds of rows per stream and more)
//
// There the pass is bound by the matrix cores and the vector unit, not by HBM: a block of 4096
// rows has 16384 query rows per KV head, and every cached token is used by all of them.  So the
// token axis is not split at all: a workgroup of eight waves owns 256 query rows (32 each: with
// 48, the register tile of the kernels above, a 2048-row block gives 176 workgroups for 256
// compute units and is slower), walks the tokens its rows can see once, and writes the
// normalised result itself (no partial results, no merge).  Short blocks are a serial walk over few
// workgroups instead: there four waves of 16 rows each, with a SIMD for themselves, take a 32-token block in
// 0.6 us where the 256-row tile takes 1.2 (see the launcher).  All waves multiply; nobody
// is set aside to load: each wave requests its share (1 KB fragment blocks) of every 32-token
// block with direct-to-LDS loads into a ring of six (four) stages, so four (two) blocks are in flight while
// one is multiplied, and the loads cost no registers.  The loads and the waits on them are
// inline assembly with exact counts, as in the many-row GEMM: after the query fragments have
// arrived the kernel issues no other vector memory load until its final stores.  Per block a
// wave runs scores -> softmax -> PV in sequence (the other wave of its SIMD fills the gaps);
// interleaving them inside the wave, or across the two waves of a SIMD, was slower or spilled.
// The last rows of a block see the most tokens and are dispatched first, those of all KV heads and streams in
// turn (8 streams of 512 rows: 55.5 -> 45 us against one group of 8 heads after the other); with 8 of them or a
// multiple each stays on one XCD and its L2, with fewer all XCDs work (Qwen2.5-7B's 4 heads, 700 rows: 42 -> 27 us).
// -------------------------------------------------------------------------------------
// NT: 16-row query tiles per wave.  PF_WAVES: 8, or 4.
template <int HD, int NT, int PF_WAVES, typename OT>
__global__ __launch_bounds__(64 * PF_WAVES) void k_attn_prefill(const bf16_t* __restrict__ q,
                                                             const bf16_t* __restrict__ kc,
                                                             const bf16_t* __restrict__ vc,
                                                             const int32_t* __restrict__ kv_len,
                                                             const int4* __restrict__ segs,
                                                             int rows, int H, int KVH, int64_t cap,
                                                             int nqt, int ranges, unsigned inv_g,
                                                             OT* __restrict__ out, int tiled,
                                                             int32_t* __restrict__ flags) {
    constexpr int KS = HD / 32, MT = HD / 16;
    constexpr int WQROWS = 16 * NT;                     // query rows per wave
    constexpr int PF_QROWS = PF_WAVES * WQROWS;         // ... per workgroup
    constexpr int PF_STAGES = PF_WAVES == 4 ? 4 : 6;    // four: two small workgroups share a compute unit's LDS
    constexpr int K_BYTES = 2 * KS * 1024, V_BYTES = MT * 1024;
    constexpr int STAGE_BYTES = K_BYTES + V_BYTES;
    constexpr int NLOAD = 2 * KS + MT;                  // 1 KB requests per 32-token block
    constexpr int LD = NLOAD / PF_WAVES;                // ... per wave
    static_assert(NLOAD % PF_WAVES == 0, "every wave issues the same number of requests");
    __shared__ __attribute__((aligned(16))) unsigned char stage[PF_STAGES][STAGE_BYTES];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wave_s = __builtin_amdgcn_readfirstlane(wave);   // uniform copy for the request addresses
    const int c = lane & 15, g = lane >> 4;
    const int range = (int)(blockIdx.x % ranges);       // (stream, KV head)
    const int qt = nqt - 1 - (int)(blockIdx.x / ranges);          // heaviest first
    const int kvh = range % KVH, b = range / KVH;
    const int G = H / KVH;
    int row0 = b * rows;                                // first of the stream's rows
    if (segs) {
        row0 = segs[b].x;
        rows = segs[b].y;
    }
    const int QR = G * rows;
    if (qt * PF_QROWS >= QR) return;                    // (whole workgroup; a stream with fewer rows than others)
    const int L = kv_len[b];
    const int n_tok = L + rows;
    // causality: nothing beyond the last row of this workgroup is walked
    const int last_row = min(rows - 1, ((qt + 1) * PF_QROWS - 1) / G);
    const int n_lim = L + last_row + 1;
    const int nblocks = (n_lim + 31) / 32;              // >= 1
    const bf16_t* __restrict__ K = kc + ((int64_t)b * KVH + kvh) * cap * HD;
    const bf16_t* __restrict__ V = vc + ((int64_t)b * KVH + kvh) * HD * cap;

    // query fragments: straight from memory into registers, once
    // query row nt*16 + c of this wave is row n0 + nt*16 of the KV head: block row n / G, head n % G of the group
    // (inv_g = 2^32 / G rounded up, exact while n * G < 2^32; 0 for G = 1)
    auto block_row = [&](int n) { return inv_g ? (int)__umulhi((unsigned)n, inv_g) : n; };
    const int n0 = qt * PF_QROWS + wave * WQROWS + c;
    bf16x8 qreg[NT][KS];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int n = n0 + nt * 16;
        const int i = n < QR ? block_row(n) : 0;
        const bf16_t* qp = q + ((int64_t)(row0 + i) * H + kvh * G + (n < QR ? n - i * G : 0)) * HD + g * 8;
#pragma unroll
        for (int s = 0; s < KS; ++s)
            qreg[nt][s] = n < QR ? *reinterpret_cast<const bf16x8*>(qp + s * 32) : (bf16x8){0, 0, 0, 0, 0, 0, 0, 0};
    }
    // they must have arrived before the first counted request below: the compiler waits for a
    // load where its result is first used, which is here
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int s = 0; s < KS; ++s) asm volatile("" : "+v"(qreg[nt][s]));

    // this wave's requests of a block: fragment block id = wave + 8*u; ids below 2*KS are K
    // fragments (a = id / KS, s = id % KS), the others V fragments (mt = id - 2*KS).  Lane
    // (c, g) of a K fragment holds token ktok0 + 4a, elements s*32 + g*8 ..; of a V fragment
    // feature mt*16 + c, tokens 8g ...
    const int ktok0 = 8 * (c >> 2) + (c & 3);
    unsigned voff[LD];
    const bf16_t* sbase[LD];
    int tstep[LD];                                      // elements the uniform base advances per token
#pragma unroll
    for (int u = 0; u < LD; ++u) {
        const int id = wave_s + PF_WAVES * u;
        if (id < 2 * KS) {
            voff[u] = (unsigned)(((ktok0 + 4 * (id / KS)) * HD + g * 8) * 2);
            sbase[u] = K + (id % KS) * 32;
            tstep[u] = HD;
        } else {
            voff[u] = (unsigned)((((id - 2 * KS) * 16 + c) * CS_VBLK + 8 * g) * 2);
            sbase[u] = V;
            tstep[u] = 0;                               // V: the block address is not linear in t0, see issue
        }
    }
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)&stage[0][0];
    // request block blk (clamped: a surplus request re-reads the last block into a stage nobody reads)
    auto issue = [&](int blk, int st) {
        const int t0 = (blk < nblocks ? blk : nblocks - 1) * 32;
#pragma unroll
        for (int u = 0; u < LD; ++u)
            cs_load_to_lds(voff[u],
                           tstep[u] ? sbase[u] + (int64_t)t0 * tstep[u] : sbase[u] + cs_v_index(t0, 0, HD),
                           lds0 + st * STAGE_BYTES + (wave_s + PF_WAVES * u) * 1024);
    };
    // at most `n` of this wave's requests still in flight, then meet the other waves
#define PF_SYNC(n) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(n) : "memory")

    f32x4 oacc[MT][NT], lacc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        lacc[nt] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) oacc[mt][nt] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    float m_run[NT], thr[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) m_run[nt] = thr[nt] = -INFINITY;
    const float scale2 = 1.4426950408889634f / sqrtf((float)HD);
    const float inv_scale2 = sqrtf((float)HD) / 1.4426950408889634f;
    const bf16_t one = (bf16_t)1.0f;
    const bf16x8 ones = (bf16x8){one, one, one, one, one, one, one, one};

    // ---- the pieces of one block (the same arithmetic as in k_attn_lds) ----
    auto scores = [&](const unsigned char* sp, f32x4 (&sacc)[2][NT]) {
        auto k_frag = [&](int a, int s) {
            return *reinterpret_cast<const bf16x8*>(sp + ((a * KS + s) * 64 + lane) * 16);
        };
        bf16x8 k0 = k_frag(0, 0), k1 = k_frag(1, 0);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            bf16x8 n0 = k0, n1 = k1;
            if (s + 1 < KS) {
                n0 = k_frag(0, s + 1);
                n1 = k_frag(1, s + 1);
            }
            const f32x4 zero4 = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                sacc[0][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k0, qreg[nt][s], s == 0 ? zero4 : sacc[0][nt], 0, 0, 0);
                sacc[1][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k1, qreg[nt][s], s == 0 ? zero4 : sacc[1][nt], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            k0 = n0;
            k1 = n1;
        }
    };
    int last_tok[NT];                                   // the last token the lane's query row sees
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) last_tok[nt] = L + block_row(n0 + nt * 16);
    auto score_of = [&](const f32x4 (&sacc)[2][NT], int nt, int e, int t0, auto tail_tag) {   // e = 4a + j
        constexpr bool TAIL = decltype(tail_tag)::value;
        const float sc = sacc[e >> 2][nt][e & 3];
        return (TAIL && (t0 + 8 * g + e > last_tok[nt])) ? -INFINITY : sc;
    };
    auto reference = [&](const f32x4 (&sacc)[2][NT], int t0, auto tail_tag) {
        constexpr bool TAIL = decltype(tail_tag)::value;
        bool calm = false;
        if (!TAIL) {
            bool over = false;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const float lm = fmaxf(fmaxf(fmaxf(sacc[0][nt][0], sacc[0][nt][1]), fmaxf(sacc[0][nt][2], sacc[0][nt][3])),
                                       fmaxf(fmaxf(sacc[1][nt][0], sacc[1][nt][1]), fmaxf(sacc[1][nt][2], sacc[1][nt][3])));
                over |= !(lm <= thr[nt]);
            }
            calm = !__any(over);
        }
        if (calm) return;
        bool moved = false;
        float alpha[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            float mx = fmaxf(fmaxf(score_of(sacc, nt, 0, t0, tail_tag), score_of(sacc, nt, 1, t0, tail_tag)),
                             score_of(sacc, nt, 2, t0, tail_tag));
            mx = fmaxf(fmaxf(mx, score_of(sacc, nt, 3, t0, tail_tag)), score_of(sacc, nt, 4, t0, tail_tag));
            mx = fmaxf(fmaxf(mx, score_of(sacc, nt, 5, t0, tail_tag)),
                       fmaxf(score_of(sacc, nt, 6, t0, tail_tag), score_of(sacc, nt, 7, t0, tail_tag)));
            mx = fa_row4_max(mx);
            mx *= scale2;
            const bool up = mx > m_run[nt] + FA_RESCALE_LOG2;
            const float m_new = up ? mx : m_run[nt];
            alpha[nt] = up ? __builtin_amdgcn_exp2f(m_run[nt] - ((m_new == -INFINITY) ? 0.f : m_new)) : 1.0f;
            moved |= up;
            m_run[nt] = m_new;
            thr[nt] = (m_new == -INFINITY) ? -INFINITY : (m_new + FA_RESCALE_LOG2) * inv_scale2;
        }
        if (__any(moved)) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                lacc[nt] *= alpha[nt];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) oacc[mt][nt] *= alpha[nt];
            }
        }
    };
    auto prob = [&](const f32x4 (&sacc)[2][NT], int nt, int e, int t0, auto tail_tag) {
        const float m_safe = (m_run[nt] == -INFINITY) ? 0.f : m_run[nt];
        return (bf16_t)__builtin_amdgcn_exp2f(fmaf(score_of(sacc, nt, e, t0, tail_tag), scale2, -m_safe));
    };
    // dead: the block reaches past the last appended row; cache rows there may hold anything, and
    // 0 * garbage must stay 0
    auto pv = [&](const unsigned char* sp, const bf16x8 (&pb)[NT], int t0, bool dead) {
        bf16x8 vf[4];
        auto v_frag = [&](int mt) {
            bf16x8 v = *reinterpret_cast<const bf16x8*>(sp + K_BYTES + (mt * 64 + lane) * 16);
            if (dead) {
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (t0 + 8 * g + j >= n_tok) v[j] = (bf16_t)0.f;
            }
            return v;
        };
#pragma unroll
        for (int mt = 0; mt < 3; ++mt) vf[mt] = v_frag(mt);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            if (mt + 3 < MT) vf[(mt + 3) & 3] = v_frag(mt + 3);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                oacc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[mt & 3], pb[nt], oacc[mt][nt], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            lacc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pb[nt], lacc[nt], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto finish = [&](const f32x4 (&sacc)[2][NT], const unsigned char* sp, int t0, auto tail_tag) {
        reference(sacc, t0, tail_tag);
        __builtin_amdgcn_sched_barrier(0);
        bf16x8 pb[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int e = 0; e < 8; ++e) pb[nt][e] = prob(sacc, nt, e, t0, tail_tag);
        __builtin_amdgcn_sched_barrier(0);
        pv(sp, pb, t0, decltype(tail_tag)::value && t0 + 32 > n_tok);
    };
    const std::integral_constant<bool, false> main_tag;
    const std::integral_constant<bool, true> tail_tag;
    // Blocks 0 .. STAGES-2 are requested up front; iteration i requests block i+STAGES-1 into the
    // stage block i-1 has left, works on block i, and ends when block i+1 has landed in every
    // wave's share (its requests are followed by those of the STAGES-2 blocks that may still be
    // in flight then).
    constexpr int INFLIGHT = LD * (PF_STAGES - 2);
#pragma unroll
    for (int j = 0; j < PF_STAGES - 1; ++j) issue(j, j);
    PF_SYNC(INFLIGHT);
    int st_cur = 0, st_req = PF_STAGES - 1;                 // stage of block i; stage of the next request
    // The loop bound and the cache length are taken from a vector register the compiler cannot
    // see through: with provably uniform branches it splits the live ranges of the accumulators
    // at every branch and ends up copying and spilling them (and a spill reload waits on the
    // same counter as the requests); with branches it must treat as divergent, both sides of
    // a branch work in place under the execution mask.
    int vzero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(vzero));
    const int nblocks_v = nblocks + vzero, L_v = L + vzero;
    // this wave's rows see the tokens up to L + row_lo .. L + row_hi: a block entirely below
    // needs no mask (and holds no dead token), a block entirely above is not computed
    const int row_lo = block_row(n0 - c);
    const int row_hi = min(rows - 1, block_row(n0 - c + WQROWS - 1));
    f32x4 sa[2][NT];
    for (int i = 0; i < nblocks_v; ++i) {
        issue(i + PF_STAGES - 1, st_req);
        st_req = st_req + 1 == PF_STAGES ? 0 : st_req + 1;
        const int t0 = i * 32;
        if (t0 <= L_v + row_hi) {
            scores(stage[st_cur], sa);
            if (t0 + 31 > L_v + row_lo) finish(sa, stage[st_cur], t0, tail_tag);
            else finish(sa, stage[st_cur], t0, main_tag);
        }
        st_cur = st_cur + 1 == PF_STAGES ? 0 : st_cur + 1;
        PF_SYNC(INFLIGHT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // surplus requests, before the LDS is given up
#undef PF_SYNC

    // out[r][head*HD + d] = O[d] / l: acc[mt][nt][j] holds O of query row nt*16 + c, feature mt*16 + 4g + j
    // (the float16 input of the output projection: saturated at +-65504, reported if it was)
    bool hit = false;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int n = n0 + nt * 16;
        if (n >= QR) continue;
        const int i = block_row(n), r = row0 + i;
        const int col0 = (kvh * G + n - i * G) * HD + 4 * g;
        const float inv = 1.0f / lacc[nt][0];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int col = col0 + mt * 16;
            const int64_t off = tiled ? cs_xt_index(r, col, H * HD) : (int64_t)r * H * HD + col;
#pragma unroll
            for (int j = 0; j < 4; ++j) fa_store_out(out, off + j, oacc[mt][nt][j] * inv, hit);
        }
    }
    cs_range_report(flags, hit, CS_RANGE_ATTN);
}

// out[r][h*HD + d] = sum_s 2^(m_s - M) O_s[d] / sum_s 2^(m_s - M) l_s  over the splits
#define FA_MAX_SPLIT 64
// Four output columns per lane (16-byte loads of the partials), HD/4 lanes per query row, so a
// 128-thread workgroup merges 512/HD rows.  Every lane derives the split weights of its row
// itself from the (max, sum) pairs (the HD/4 lanes of a row read the same words, which the
// cache broadcasts): no LDS, no barrier, and the same summation order in every lane.
#define FA_MERGE_THREADS 128
template <typename OT>
__global__ __launch_bounds__(FA_MERGE_THREADS) void k_attn_merge(const float* __restrict__ po,
                                                                 const float* __restrict__ pml,
                                                                 const int4* __restrict__ segs,
                                                                 int rows, int H, int KVH, int HD,
                                                                 int nqg, int nsplit,
                                                                 OT* __restrict__ out, int tiled,
                                                                 int32_t* __restrict__ flags) {
    const int lpr = HD >> 2;                  // lanes per query row
    const int n = blockIdx.x * (FA_MERGE_THREADS / lpr) + (int)threadIdx.x / lpr;   // row within the KV head: i*G + gq
    const int d = ((int)threadIdx.x % lpr) * 4;
    const int kvh = blockIdx.y, b = blockIdx.z;
    const int G = H / KVH;
    int row0 = b * rows, group0 = b * nqg;    // the stream's first block row, its first query group
    if (segs) {
        const int4 sg = segs[b];
        row0 = sg.x;
        rows = sg.y;
        group0 = sg.z;
        nqg = (G * rows + FA_QROWS - 1) / FA_QROWS;
    }
    if (n >= G * rows) return;
    const int i = n / G, gq = n % G;
    const int qg = n / FA_QROWS, nl = n % FA_QROWS;
    const int64_t item = (int64_t)group0 * KVH + kvh * nqg + qg;
    const float2* __restrict__ ml = reinterpret_cast<const float2*>(pml) + (item * nsplit * FA_QROWS + nl);
    const float* __restrict__ o = po + (item * nsplit * FA_QROWS + nl) * HD + d;
    // eight splits at a time, all their loads issued before the first is used: with many splits
    // (one stream: 32) and few workgroups this kernel is nothing but load latency
    float M = -INFINITY;
    for (int w0 = 0; w0 < nsplit; w0 += 8) {
        float mx[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) mx[u] = w0 + u < nsplit ? ml[(int64_t)(w0 + u) * FA_QROWS].x : -INFINITY;
#pragma unroll
        for (int u = 0; u < 8; ++u) M = fmaxf(M, mx[u]);
    }
    float den = 0.f;
    f32x4 num = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int w0 = 0; w0 < nsplit; w0 += 8) {                // same order in every lane
        float2 p[8];
        f32x4 ov[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool in = w0 + u < nsplit;
            p[u] = in ? ml[(int64_t)(w0 + u) * FA_QROWS] : make_float2(-INFINITY, 0.f);
            ov[u] = in ? *reinterpret_cast<const f32x4*>(o + (int64_t)(w0 + u) * FA_QROWS * HD)
                       : (f32x4){0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float wgt = (p[u].x == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(p[u].x - M);
            den += wgt * p[u].y;
            num += wgt * ov[u];
        }
    }
    const float inv = 1.0f / den;
    const int r = row0 + i;
    // tiled: the output projection reads fragment order
    const int col = (kvh * G + gq) * HD + d;
    const int64_t off = tiled ? cs_xt_index(r, col, H * HD) : (int64_t)r * H * HD + col;
    bool hit = false;
    if constexpr (std::is_same<OT, f16_t>::value) {       // one 8-byte store
        const f16x4 o = (f16x4){cs_f16_sat(num[0] * inv, hit), cs_f16_sat(num[1] * inv, hit),
                                cs_f16_sat(num[2] * inv, hit), cs_f16_sat(num[3] * inv, hit)};
        *reinterpret_cast<f16x4*>(out + off) = o;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) fa_store_out(out, off + j, num[j] * inv, hit);
    }
    cs_range_report(flags, hit, CS_RANGE_ATTN);
}

// Into how many token ranges the `items` (stream, KV head) pairs are split, `wgs` workgroups per range.  A workgroup
// fills a compute unit and takes its share of the tokens plus the time of about 512 more (wide blocks of 16 streams:
// 26 us per 1000 tokens and 12 us): as many ranges as one round of the chip holds rather than a few workgroups
// more.  Wide, 5 streams of 6001 rows, 147 query rows per KV head: 288 workgroups 38.1 us, 240 29.8 us (with groups of
// 3 + 1 43.1 and 35.6); narrow, 18431 rows, batch 3 / 5 / 6 / 7: 51 / 107 / 130 / 149 -> 41 / 77 / 90 / 105 us, batches that
// divide 256 as before.
static int fit_ranges(int64_t items, int wgs, int64_t n_tok) {
    int best = 1;
    double best_t = 0.;
    for (int n = 1; n <= (int)cs_ceil_div(256, items * wgs); ++n) {
        const double t = (double)cs_ceil_div(cs_round_up(items * n, 8) * wgs, 256) * (512. + (double)n_tok / n);
        if (n == 1 || t < best_t) { best_t = t; best = n; }
    }
    return best;
}

// How the wide kernel would take a block: query groups per workgroup, token ranges, and what that costs, in tokens' worth
// of a workgroup's time (about 17 ns at hd 128, 11 at hd 64).
struct wide_plan {
    int nqgw, gpw, nsplit, Tw;      // workgroups per token range, query groups of each; team ranges, tokens of one
    int64_t groups;                 // query groups of one KV head, over all streams
    double cost;
};
static wide_plan plan_wide(int B, int KVH, int G, int nqg, int64_t n_tok, const cs_ragged* rg) {
    wide_plan p;
    p.nqgw = (int)cs_ceil_div(nqg, FA_QG);
    // query groups evenly over the workgroups of a range (147 rows: 2 + 2, which spread over the SIMDs, not 3 + 1)
    p.gpw = (int)cs_ceil_div(nqg, p.nqgw);
    int64_t wgs = (int64_t)B * p.nqgw;                   // workgroups per token range that have query groups
    p.groups = (int64_t)B * nqg;
    if (rg) {
        p.groups = wgs = 0;
        for (int b = 0; b < B; ++b) {
            const int64_t g = cs_ceil_div((int64_t)G * rg->rows[b], FA_QROWS);
            p.groups += g;
            wgs += cs_ceil_div(g, p.gpw);
        }
    }
    p.nsplit = FA_TEAMS * (rg ? fit_ranges(KVH * wgs, 1, n_tok) : fit_ranges((int64_t)B * KVH, p.nqgw, n_tok));
    const int max_split = (int)cs_ceil_div(n_tok, 256);
    if (p.nsplit > max_split) p.nsplit = max_split;
    if (p.nsplit > FA_MAX_SPLIT) p.nsplit = FA_MAX_SPLIT;
    if (p.nsplit < 1) p.nsplit = 1;
    p.Tw = (int)cs_round_up(cs_ceil_div(n_tok, p.nsplit), 32);
    p.nsplit = (int)cs_round_up(cs_ceil_div(n_tok, p.Tw), FA_TEAMS);
    const int ranges = p.nsplit / FA_TEAMS;
    p.cost = 400. + (double)cs_ceil_div(KVH * wgs * ranges, 256) * (1000. + (double)n_tok / ranges) + 1.2 * (double)(KVH * p.groups * ranges);
    return p;
}

bool cs_attention_fuses_rope(const cs_model* m, int rows) {
    return m->fast && (m->cfg.n_heads / m->cfg.n_kv_heads) * rows <= FA_QROWS;
}

int cs_attention_launch(const cs_model* m, cs_kv* kv, int layer, int rows, int64_t len_ub,
                        int for_o_proj, const float* qkv_part, int qkv_nparts, const cs_ragged* rg, hipStream_t s) {
    const cs_model_cfg& c = m->cfg;
    const int B = kv->B, H = c.n_heads, KVH = c.n_kv_heads, hd = c.head_dim;
    const int64_t per_layer = (int64_t)B * KVH * kv->cap * hd;
    if (!m->fast) {
        dim3 grid(rg ? rg->R : rows, H, rg ? 1 : B);
        // The kernel whose lanes share a key row does more per token and has more to add up at the end: it is for
        // contexts that outweigh this, measured by the elements of a head's K that a row sees on average (rows of 4 or 8
        // elements, which the other kernel reads one by one, count eightfold).  Its workgroups of 16 waves fill a compute
        // unit each (113 to 127 registers), those of four pay where there are many.
        // Times against the kernel with a key row per thread, hd 32 / 64 / 128:
        //   up to 256 workgroups, 16 waves:  200 tokens 1.07 / 0.91 / 0.82, 1000 0.71 / 0.58 / 0.55 (bfloat16 0.90 / 0.71 / 0.72)
        //   384 workgroups, 16 waves:        500 tokens 1.29 / 1.03 / 0.89, 2000 0.86 / 0.65 / 0.68 (1.30 / 0.99 / 1.00)
        //   768 workgroups, four:            100 tokens 1.16 / 1.20 / 1.14, 500 0.96 / 0.93 / 0.87 (1.27 / 1.21 / 1.12)
        //   8192 workgroups, four:           100 tokens 1.33 / 1.21 / 1.01, 500 0.83 / 0.72 / 0.62 (1.29 / 1.15 / 0.84)
        const int64_t wgs = (int64_t)grid.x * grid.y * grid.z;
        const bool bf16 = c.dtype == CS_BF16;
        const bool narrow = hd == 4 || hd == 8;
        const double seen = (narrow ? 8 : 1) * hd * ((double)len_ub + 0.5 * ((rg ? *std::max_element(rg->rows, rg->rows + B) : rows) + 1));
        int lanes;                                       // threads of the kernel whose lanes share a row, 0: the other
        if (wgs <= 256) lanes = seen >= (bf16 ? 12288. : 9216.) ? 1024 : 0;
        else if (wgs <= 512) lanes = (bf16 ? hd == 256 && wgs >= 384 && seen >= 131072. : (hd >= 32 || narrow) && seen >= 30720.) ? 1024 : 0;
        else if (wgs < 1024) lanes = (bf16 ? narrow && seen >= 32768. : seen >= (hd <= 32 ? 16384. : 32768.)) ? 256 : 0;
        else lanes = (bf16 ? (hd >= 64 || narrow) && seen >= (hd == 64 ? 65536. : 32768.) : seen >= 12288.) ? 256 : 0;
        auto start = [&](auto* k, auto threads) {
            typedef std::remove_pointer_t<decltype(k)> WT;
            constexpr int THREADS = decltype(threads)::value;
            const float* q = (const float*)m->q;
            const WT* kc = (const WT*)kv->k + layer * per_layer;
            const WT* vc = (const WT*)kv->v + layer * per_layer;
            const int2* map = rg ? rg->row : nullptr;
            if constexpr (THREADS > 0)
                k_attn_plain_lanes<WT, float, float, THREADS><<<grid, THREADS, 0, s>>>(q, kc, vc, kv->d_len, map, rows, H, KVH, hd,
                                                                                       kv->cap, (float*)m->xn);
            else
                k_attn_plain<WT, float, float><<<grid, PA_THREADS, 0, s>>>(q, kc, vc, kv->d_len, map, rows, H, KVH, hd, kv->cap,
                                                                           (float*)m->xn);
        };
        auto by_type = [&](auto threads) {
            if (bf16) start((bf16_t*)nullptr, threads);
            else start((float*)nullptr, threads);
        };
        if (lanes == 1024) by_type(std::integral_constant<int, 1024>{});
        else if (lanes == 256) by_type(std::integral_constant<int, 256>{});
        else by_type(std::integral_constant<int, 0>{});
        return cs_launch_ok("k_attn_plain");
    }
    const int G = H / KVH;
    int widest = rows;
    if (rg) widest = *std::max_element(rg->rows, rg->rows + B);
    const int QR = G * widest;
    const int nqg = (int)cs_ceil_div(QR, FA_QROWS);
    const int64_t n_tok_ub = len_ub + widest;
    const int tiled = for_o_proj ? 1 : 0;      // the output projection reads fragment order
    const bf16_t* kc = (const bf16_t*)kv->k + layer * per_layer;
    const bf16_t* vc = (const bf16_t*)kv->v + layer * per_layer;
    CS_REQUIRE(!qkv_part || nqg == 1, CS_E_STATE, "fused rotary embedding needs a narrow block");
    int nsplit;
    // The prompt kernel, which walks all tokens of a tile in one workgroup, or the token ranges of the wide kernel and
    // their merge.  Considered for the first: prompt blocks of at least two tiles of 256 query rows per KV head and 40
    // workgroups, and, while the context is short, wide blocks that a round of 64-row tiles covers and blocks with their
    // own number of rows per stream, however narrow.  Those of more than two 64-row tiles per compute unit take it; the
    // others where it is estimated to take less.  (7260 blocks of hd 64 and 128, one to eight query heads per KV head, 1
    // to 32 streams of 0 to 24000 tokens, all three ways: on average 2 % slower than the fastest.  8B widths, one stream,
    // 24, 64, 128, 256 rows: 18.3, 20.7, 24.0, 29.7 us split, 9.4, 9.8, 11.7, 15.4 unsplit; Qwen2.5-7B, 4 streams of 80
    // rows behind 1500, 3000, 24000 tokens: 39, 44, 140 us split, 48, 79, 534 unsplit; a prompt of 8000 tokens in passes of
    // 64 rows, four layers of 8B widths: 72 ms split, 104 unsplit.)
    const int64_t ranges = (int64_t)B * KVH;
    int64_t wgs_many = 0, wgs_few = 0;
    for (int b = 0; b < B; ++b) {
        const int64_t n = (int64_t)G * (rg ? rg->rows[b] : rows);
        wgs_many += KVH * cs_ceil_div(n, 256);
        wgs_few += KVH * cs_ceil_div(n, 64);
    }
    const bool many = QR >= 512 && wgs_many >= 40, brief = n_tok_ub <= 768 && (rg || (nqg > 1 && wgs_few <= 256));
    wide_plan wide = {};
    if (nqg > 1 || rg) wide = plan_wide(B, KVH, G, nqg, n_tok_ub, rg);
    const double reach = (double)len_ub + 0.5 * (widest + 1);        // tokens the rows see on average, at most
    const double unsplit = wgs_few <= 256 ? (hd == 64 ? 650. : 500.) + 2. * reach : 1400. + 1.2 * reach;
    if ((many || brief) && (wgs_few > 512 || unsplit <= wide.cost)) {
        // 64 query rows in four waves while that gives at most two workgroups per compute unit (three, of half the LDS
        // each, at hd 64 up to 2048 tokens), or three of a long prompt's first block, whose early rows see few tokens
        // (300, 512, 700, 1024, 1500 rows of the 8B shape: 21.1, 27.3, 33.4, 42.6, 57.0 us with 256-row tiles, 15.8, 20.0,
        // 27.5, 38.0, 54.0 with 64; 8 streams of 300 rows, 1216 workgroups: 31 against 34 us; 3 streams of 256 rows of
        // eight query heads, 768 workgroups, behind 0 / 200 tokens: 36 / 43 against 38 / 50; hd 64, 5 streams of 200 rows
        // of four, 520 workgroups, behind 300 / 2000 tokens: 26 / 62 against 22 / 62)
        const bool first = len_ub < widest;
        const bool three = first ? hd == 64 || QR >= 4096 : hd == 64 && n_tok_ub <= 2048;
        const bool small = wgs_few <= (three ? 768 : 512);
        const int nqt = (int)cs_ceil_div(QR, small ? 64 : 256);
        const unsigned inv_g = G > 1 ? (unsigned)(((1ull << 32) + G - 1) / G) : 0;
        dim3 grid((unsigned)(ranges * nqt));
        const int pa = cs_prof_begin(CS_PROF_ATTN, s);
        auto start = [&](auto hd_tag, auto nt_tag, auto wave_tag) {
            constexpr int HD = decltype(hd_tag)::value, NT = decltype(nt_tag)::value, WAVES = decltype(wave_tag)::value;
            k_attn_prefill<HD, NT, WAVES, f16_t><<<grid, 64 * WAVES, 0, s>>>(
                (const bf16_t*)m->q, kc, vc, kv->d_len, rg ? rg->seg : nullptr, rows, H, KVH, kv->cap, nqt, (int)ranges, inv_g, (f16_t*)m->xn, tiled,
                m->range_flags);
        };
        auto by_tile = [&](auto hd_tag) {
            if (small) start(hd_tag, std::integral_constant<int, 1>{}, std::integral_constant<int, 4>{});
            else start(hd_tag, std::integral_constant<int, 2>{}, std::integral_constant<int, 8>{});
        };
        if (hd == 128) by_tile(std::integral_constant<int, 128>{});
        else by_tile(std::integral_constant<int, 64>{});
        cs_prof_end(pa, s);
        return cs_launch_ok("k_attn_prefill");
    }
    if (nqg > 1 || rg) {
        // wide block: consumers share the K/V stream of one producer wave through LDS
        const int nqgw = wide.nqgw, gpw = wide.gpw, Tw = wide.Tw;
        nsplit = wide.nsplit;
        const size_t items = (size_t)wide.groups * KVH * (nsplit / FA_TEAMS);
        CS_REQUIRE(items * FA_QROWS * (hd + 2) <= m->attn_part_floats, CS_E_CAPACITY,
                   "attention workspace too small");
        float* po = m->attn_part;
        float* pml = m->attn_part + items * FA_QROWS * hd;
        // one-dimensional grid, decoded in the kernel (XCD-aware order)
        const int ranges = B * KVH * (nsplit / FA_TEAMS);
        const int4* segs = rg ? rg->seg : nullptr;
        dim3 grid((unsigned)(cs_round_up(ranges, 8) * nqgw));
        const int pa = cs_prof_begin(CS_PROF_ATTN, s);
        if (hd == 128)
            k_attn_lds<128><<<grid, FA_LDS_THREADS, 0, s>>>((const bf16_t*)m->q, kc, vc, kv->d_len, segs, rows,
                                                             H, KVH, kv->cap, Tw, nqg, nqgw, gpw, nsplit, ranges, po, pml);
        else
            k_attn_lds<64><<<grid, FA_LDS_THREADS, 0, s>>>((const bf16_t*)m->q, kc, vc, kv->d_len, segs, rows,
                                                            H, KVH, kv->cap, Tw, nqg, nqgw, gpw, nsplit, ranges, po, pml);
        cs_prof_end(pa, s);
        CS_TRY(cs_launch_ok("k_attn_lds"));
        dim3 mgrid((unsigned)cs_ceil_div(QR, FA_MERGE_THREADS / (hd / 4)), KVH, B);
        const int pm = cs_prof_begin(CS_PROF_ATTN_MERGE, s);
        k_attn_merge<f16_t><<<mgrid, FA_MERGE_THREADS, 0, s>>>(po, pml, segs, rows, H, KVH, hd, nqg, nsplit / FA_TEAMS,
                                                              (f16_t*)m->xn, tiled, m->range_flags);
        cs_prof_end(pm, s);
        return cs_launch_ok("k_attn_merge");
    }
    // The kernel keeps one wave per SIMD (register budget), so one workgroup fills a compute
    // unit: aim at one round of the chip, at least 128 tokens per wave; up to eight splits, which
    // the merge reads in one batch, also of 32 tokens per wave (one row, 300 tokens, hd 128: 1, 2, 3 splits
    // 10.4, 7.6, 7.0 us; 4106 tokens of hd 64 in 9, 17 splits: 9.6, 9.1 us, but the merge 4.0, 5.1).
    nsplit = fit_ranges((int64_t)B * KVH, 1, n_tok_ub);
    const int few = (int)cs_ceil_div(n_tok_ub, 4 * 32) < 8 ? (int)cs_ceil_div(n_tok_ub, 4 * 32) : 8;
    const int max_split = (int)cs_ceil_div(n_tok_ub, 4 * 128) > few ? (int)cs_ceil_div(n_tok_ub, 4 * 128) : few;
    if (nsplit > max_split) nsplit = max_split;
    if (nsplit > FA_MAX_SPLIT) nsplit = FA_MAX_SPLIT;
    // a workgroup's range is addressed with 31-bit byte offsets: at most 2^22 tokens of 256 bytes
    if (nsplit < cs_ceil_div(n_tok_ub, (int64_t)1 << 22)) nsplit = (int)cs_ceil_div(n_tok_ub, (int64_t)1 << 22);
    if (nsplit < 1) nsplit = 1;
    const int Tw = (int)cs_round_up(cs_ceil_div(n_tok_ub, (int64_t)nsplit * 4), 32);
    nsplit = (int)cs_ceil_div(n_tok_ub, (int64_t)Tw * 4);
    const size_t items = (size_t)B * KVH * nqg * nsplit;
    const size_t need = items * FA_QROWS * (hd + 2);
    CS_REQUIRE(need <= m->attn_part_floats, CS_E_CAPACITY,
               "attention workspace too small (%zu > %zu floats)", need, m->attn_part_floats);
    float* po = m->attn_part;
    float* pml = m->attn_part + items * FA_QROWS * hd;
    dim3 grid(nsplit * nqg, KVH, B);
    const int pa = cs_prof_begin(CS_PROF_ATTN, s);
    fa_fused_rope fr = {nullptr, 0, 0, nullptr, nullptr, nullptr, nullptr};
    if (qkv_part) {
        fr.qkv = qkv_part;
        fr.nparts = qkv_nparts;
        fr.part_stride = (int64_t)B * rows * (H + 2 * KVH) * hd;
        fr.rope = m->rope;
        fr.kc_w = (bf16_t*)kv->k + layer * per_layer;
        fr.vc_w = (bf16_t*)kv->v + layer * per_layer;
        fr.bias = m->layers[layer].bqkv;
    }
    const int nt = (int)cs_ceil_div(QR, 16);              // 16-row query tiles
    // (without partial tiles: cs_op_attention, whose queries are given; the model's narrow blocks always fuse)
    auto launch = [&](auto hd_tag, auto nt_tag) {
        constexpr int HD = decltype(hd_tag)::value, NT = decltype(nt_tag)::value;
        if (qkv_part)
            k_attn_mfma<HD, NT, true><<<grid, 256, 0, s>>>((const bf16_t*)m->q, kc, vc, kv->d_len, rows, H, KVH,
                                                           kv->cap, Tw, nsplit, po, pml, fr);
        else
            k_attn_mfma<HD, NT, false><<<grid, 256, 0, s>>>((const bf16_t*)m->q, kc, vc, kv->d_len, rows, H, KVH,
                                                            kv->cap, Tw, nsplit, po, pml, fr);
    };
    auto by_rows = [&](auto hd_tag) {
        if (nt == 1) launch(hd_tag, std::integral_constant<int, 1>{});
        else if (nt == 2) launch(hd_tag, std::integral_constant<int, 2>{});
        else launch(hd_tag, std::integral_constant<int, FA_NT>{});
    };
    if (hd == 128) by_rows(std::integral_constant<int, 128>{});
    else by_rows(std::integral_constant<int, 64>{});
    cs_prof_end(pa, s);
    CS_TRY(cs_launch_ok("k_attn_mfma"));
    dim3 mgrid((unsigned)cs_ceil_div(QR, FA_MERGE_THREADS / (hd / 4)), KVH, B);
    const int pm = cs_prof_begin(CS_PROF_ATTN_MERGE, s);
    k_attn_merge<f16_t><<<mgrid, FA_MERGE_THREADS, 0, s>>>(po, pml, nullptr, rows, H, KVH, hd, nqg, nsplit,
                                                          (f16_t*)m->xn, tiled, m->range_flags);
    cs_prof_end(pm, s);
    return cs_launch_ok("k_attn_merge");
}
