"""Per-kernel GPU parity at the benchmark's full shapes (sampled outputs) and edge cases.

The oracle computes sampled outputs one by one (a GEMM column, an attention head, an argmax
row); every stream is independent, so a sampled stream is a complete check of that stream.
"""
import numpy as np
import pytest
import torch

import synth
from synth import ModelShape
from oracle import copyspec_oracle as orc

pytestmark = pytest.mark.gpu
cs = pytest.importorskip("paper_2502_08923_amd.binding")
DEV = "cuda:0"

HOST = ModelShape("host-8b-width", 1, 4096, 32, 8, 128, 14336, 2048, 500000.0, 1e-5, "bf16")


def t32(a):
    return torch.tensor(np.asarray(a), dtype=torch.int32, device=DEV)


def bf16_dev(bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).view(torch.bfloat16).to(DEV)


@pytest.fixture(scope="module")
def host_model():
    """A one-layer model at the 8B width: owns the workspace the op entry points use."""
    w = synth.model_weights(HOST, 99, threads=16)
    m = cs.Model(w, max_batch=16, max_k=32)
    yield m
    m.destroy()


# ----------------------------------------------------------------------------------------
# argmax + accept
# ----------------------------------------------------------------------------------------

@pytest.mark.parametrize("B,k,V", [(8, 10, 128256), (16, 32, 128256), (3, 4, 97), (1, 0, 1024)])
def test_argmax_accept_full_size(host_model, B, k, V):
    rng = np.random.default_rng(B * 1000 + k)
    logits = rng.standard_normal((B, k + 1, V)).astype(np.float32)
    # exact ties: duplicate the maximum at a later index in some rows (lowest index must win)
    for b in range(B):
        for i in range(0, k + 1, 3):
            j = int(np.argmax(logits[b, i]))
            if j + 5 < V:
                logits[b, i, j + 5] = logits[b, i, j]
    am = np.array([[orc.argmax_first(logits[b, i]) for i in range(k + 1)] for b in range(B)])
    draft = np.zeros((B, max(k, 1)), dtype=np.int32)
    dlen = np.zeros(B, dtype=np.int32)
    for b in range(B):
        m = int(rng.integers(0, k + 1))
        dlen[b] = m
        draft[b, :k] = rng.integers(0, V, k) if k else 0
        good = int(rng.integers(0, m + 1))                 # accept exactly `good`, unless luck
        draft[b, :good] = am[b, :good]
    acc, nxt, ram = cs.cs_op_argmax_accept(host_model, torch.from_numpy(logits).to(DEV),
                                           t32(draft[:, :k]) if k else t32(np.zeros((B, 0))),
                                           t32(dlen))
    torch.cuda.synchronize()
    assert np.array_equal(ram.cpu().numpy(), am)
    for b in range(B):
        tau, nx = orc.accept_prefix(am[b], draft[b, :dlen[b]].tolist())
        assert (int(acc[b]), int(nxt[b])) == (tau, nx)


# ----------------------------------------------------------------------------------------
# projections at the 8B shapes, R = 88 (benchmark) and 528 (batch 16, k = 32)
# ----------------------------------------------------------------------------------------

def _gemm_case(host_model, N, K, R):
    seed = N * 7 + K + R
    xb = synth.workloads._draw(seed, (R, K), "n", 1.0, "bf16")
    wb = synth.workloads._draw(seed + 1, (N, K), "u", (3.0 / K) ** 0.5, "bf16")
    Y = cs.cs_op_gemm(host_model, bf16_dev(xb), bf16_dev(wb)).cpu().numpy()
    rng = np.random.default_rng(seed)
    cols = np.unique(np.concatenate([rng.integers(0, N, 192), [0, 15, 16, N - 17, N - 1]]))
    x64 = synth.bf16_bits_to_f32(xb).astype(np.float64)
    w64 = synth.bf16_bits_to_f32(wb[cols]).astype(np.float64)
    ref = x64 @ w64.T
    err = np.abs(Y[:, cols] - ref).max()
    assert err < 2e-4 * max(1.0, np.abs(ref).max()), err      # fp32 accumulation of exact products


@pytest.mark.parametrize("N,K", [(6144, 4096), (4096, 4096), (28672, 4096), (4096, 14336),
                                 (128256, 4096)])
@pytest.mark.parametrize("R", [88, 528, 1])
def test_gemm_bf16_full_shapes(host_model, N, K, R):
    _gemm_case(host_model, N, K, R)


@pytest.mark.parametrize("R", [97, 120, 168, 200, 250, 264, 300, 408, 528])
@pytest.mark.parametrize("N,K", [(49168, 512), (49168, 128), (6144, 4096)])
def test_gemm_row_sweep(host_model, N, K, R):
    """Row counts between the two regimes.  The 193 W tiles of the 49168-row matrix send every
    row count above 96 to the many-row kernel (7 to 17 X tiles, one and two row blocks, ragged last tiles in both dimensions, K of one and of four pipeline trips); the
    q/k/v shape switches kernels by estimated time below 289 rows and is split along K."""
    _gemm_case(host_model, N, K, R)


@pytest.mark.parametrize("N,K,R", [(4112, 512, 1023), (4112, 512, 1300), (6144, 4096, 1300), (4096, 4096, 2064),
                                   (2048, 8192, 4095), (4096, 1024, 4095)])
def test_gemm_prompt_rows(host_model, N, K, R):
    """Prompt-sized row counts: more row blocks than one panel of the workgroup mapping holds, a last
    panel of fewer, a W tile count that is no multiple of the eight dies, with and without K splits."""
    _gemm_case(host_model, N, K, R)


@pytest.mark.parametrize("R", [5, 88, 105, 112, 113, 128, 129, 200, 256, 257])
@pytest.mark.parametrize("N,K", [(37888, 256), (33040, 128), (4096, 1024)])
def test_gemm_wide_blocks_and_five_wave_tiles(host_model, N, K, R):
    """The weight-streaming kernel with five consumer waves (more than 256 tiles of 128 W rows, ragged last tile) and one to
    eight X tiles over the one or two K chunks of its remainder loop, and with four waves and K splits."""
    _gemm_case(host_model, N, K, R)


@pytest.mark.parametrize("R", [190, 215, 235, 280])
def test_gemm_row_tile_counts_between(host_model, R):
    """The row-tile counts of the many-row kernel that the sweep above leaves out (12, 14, 15 and 18), which differ in
    how many requests a wave counts per chunk; four pipeline trips."""
    _gemm_case(host_model, 49168, 512, R)


@pytest.mark.parametrize("R,N,K", [(R, N, K) for N, K in ((37888, 512), (33040, 640), (33040, 1408)) for R in (5, 88, 105, 128, 200, 256)]
                         + [(105, 37888, 3584)])
def test_gemm_five_wave_tiles_over_long_rows(host_model, R, N, K):
    """Five consumer waves with 1, 6, 7 and 8 X tiles through the pipelined loop (four K chunks per trip): one trip, one and a
    remainder of one, two and a remainder of three, and the 28 chunks of a 3584-wide model's gate/up."""
    _gemm_case(host_model, N, K, R)


@pytest.mark.parametrize("chunks", [1, 2, 3, 5, 6, 7, 9])
@pytest.mark.parametrize("R", [1, 16, 33, 81, 96, 112, 128])
def test_gemm_chunk_counts_of_the_ring(host_model, R, chunks):
    """The weight-streaming kernel over 128 * chunks of K: less than its ring of four chunks, whole rings and every
    remainder, for row tiles below and above the count from which the multiply order is pinned (1, 1, 3, 6, 6 and, in two
    row blocks, 4 and 4)."""
    _gemm_case(host_model, 1040, 128 * chunks, R)


@pytest.mark.parametrize("chunks", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("R", [32, 80, 105, 128])
def test_gemm_chunk_counts_in_one_row_block(host_model, R, chunks):
    """The same with 2, 5, 7 and 8 row tiles: 225 tiles of 128 W rows fill the chip in one row block."""
    _gemm_case(host_model, 28688, 128 * chunks, R)


@pytest.mark.parametrize("K", [128, 256, 384, 512, 640])
@pytest.mark.parametrize("R", [1, 33, 88, 128])
def test_gemm_input_beyond_float16(host_model, R, K):
    """An X beyond float16 is an infinity to the multiplies: its row of Y is infinite with the sign of each weight (the
    others stay finite), also where K is shorter than the ring of four chunks."""
    N, at, row = 1040, K - 3, R // 2
    rng = np.random.default_rng(R + K)
    x = rng.standard_normal((R, K)).astype(np.float32)
    x[row, at] = 1e5
    w = (rng.integers(1, 8, (N, K)) * 0.125 * rng.choice([-1.0, 1.0], (N, K))).astype(np.float32)
    Y = cs.cs_op_gemm(host_model, bf16_dev(synth.f32_to_bf16_bits(x)), bf16_dev(synth.f32_to_bf16_bits(w))).cpu().numpy()
    assert np.array_equal(Y[row], np.copysign(np.inf, w[:, at]))
    assert np.isfinite(np.delete(Y, row, axis=0)).all()


def test_gemm_tiny_weights_are_not_flushed(host_model):
    """The tuned projections multiply in float16 (weights converted from bfloat16, exactly for
    |w| >= 2^-17).  Weights in float16's subnormal range must still contribute."""
    N, K, R = 64, 512, 16
    rng = np.random.default_rng(3)
    w = (rng.integers(1, 8, (N, K)) * 2.0 ** -17 * rng.choice([-1.0, 1.0], (N, K))).astype(np.float32)
    x = (rng.integers(1, 4, (R, K)) * 256.0).astype(np.float32)
    wb, xb = synth.f32_to_bf16_bits(w), synth.f32_to_bf16_bits(x)
    assert np.array_equal(synth.bf16_bits_to_f32(wb), w) and np.array_equal(synth.bf16_bits_to_f32(xb), x)
    Y = cs.cs_op_gemm(host_model, bf16_dev(xb), bf16_dev(wb)).cpu().numpy()
    ref = x.astype(np.float64) @ w.astype(np.float64).T
    assert np.abs(ref).max() > 0.05
    assert np.abs(Y - ref).max() <= 1e-5 * np.abs(ref).max() + 1e-7


def test_gemm_f32_plain(host_model):
    rng = np.random.default_rng(5)
    X = rng.standard_normal((11, 256)).astype(np.float32)
    W = rng.standard_normal((777, 256)).astype(np.float32)
    Y = cs.cs_op_gemm(host_model, torch.from_numpy(X).to(DEV), torch.from_numpy(W).to(DEV))
    ref = X.astype(np.float64) @ W.astype(np.float64).T
    assert np.abs(Y.cpu().numpy() - ref).max() < 1e-4


@pytest.mark.parametrize("R,N,K", [(1, 97, 64), (11, 777, 256), (16, 16, 4), (17, 250, 1030), (33, 64, 7), (70, 33, 516),
                                   (511, 256, 1024), (5, 31, 1)])
@pytest.mark.parametrize("shift", [0, 1])
def test_gemm_f32_edges(host_model, R, N, K, shift):
    """The float32 kernel at the edges of its tiles: one row tile, two and more, ragged last rows and
    columns, K below one piece and no multiple of four, operands that are not 16-byte aligned (shift).
    Bound: a sum of K float32 products in any order is within K roundings of sum |x||w|."""
    rng = np.random.default_rng(R * 1000 + N + K)
    X = rng.standard_normal((R, K)).astype(np.float32)
    W = rng.standard_normal((N, K)).astype(np.float32)

    def dev(a):
        buf = torch.empty(a.size + shift, dtype=torch.float32, device=DEV)
        buf[shift:].copy_(torch.from_numpy(a.ravel()))
        return buf[shift:].view(a.shape)

    Y = cs.cs_op_gemm(host_model, dev(X), dev(W)).cpu().numpy()
    ref = X.astype(np.float64) @ W.astype(np.float64).T
    bound = (K + 16) * 2.0 ** -24 * (np.abs(X).astype(np.float64) @ np.abs(W).astype(np.float64).T)
    assert (np.abs(Y - ref) <= bound).all()


@pytest.mark.parametrize("R,N,K", [(5, 300, 64), (11, 256, 256), (40, 512, 1024), (100, 256, 4096), (16, 640, 1030)])
def test_gemm_f32_error_of_short_chains(host_model, R, N, K):
    """The rounding error of the float32 kernel against float64 is no larger than that of a sum over 64 interleaved
    chains of K / 64 fused multiply-adds, added in pairs (root mean square over at least 1500 outputs, so 10 % is
    about four times its sampling error)."""
    rng = np.random.default_rng(R + N + K)
    X = rng.standard_normal((R, K)).astype(np.float32)
    W = rng.standard_normal((N, K)).astype(np.float32)
    Y = cs.cs_op_gemm(host_model, torch.from_numpy(X).to(DEV), torch.from_numpy(W).to(DEV)).cpu().numpy()
    x64, w64 = X.astype(np.float64), W.astype(np.float64)
    ref = x64 @ w64.T
    acc = np.zeros((64, R, N), dtype=np.float32)
    for k0 in range(0, K, 64):              # (a product of two float32 is exact in float64)
        for lane in range(min(64, K - k0)):
            acc[lane] = acc[lane].astype(np.float64) + np.outer(x64[:, k0 + lane], w64[:, k0 + lane])
    half = 32
    while half:
        acc[:half] += acc[half:2 * half]
        half //= 2
    rms = lambda e: float(np.sqrt(np.mean(np.square(e))))
    assert rms(Y - ref) <= 1.1 * rms(acc[0] - ref), (rms(Y - ref), rms(acc[0] - ref))


# ----------------------------------------------------------------------------------------
# block attention
# ----------------------------------------------------------------------------------------

def _attention_case(model, shape, lens, rows, sample, seed, poison=False, k_ramp=None, device_fill=False):
    """device_fill: streams the oracle does not look at get their cache rows from a device-side
    generator (cheap at long lengths); sampled streams always get the seeded host rows."""
    B = len(lens)
    cap = max(lens) + rows + 5
    kv = cs.KV(model, B, cap)
    ks, vs = {}, {}
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    for b, L in enumerate(lens):
        if device_fill and b not in {sb for sb, _ in sample}:
            shp = (shape.n_kv_heads, L + rows, shape.head_dim)
            kv.load(0, b, 0, torch.randn(shp, generator=gen, device=DEV).bfloat16(),
                    torch.randn(shp, generator=gen, device=DEV).bfloat16())
            kv.set_len(b, L)
            continue
        kr, vr = synth.random_kv(shape, L + rows, seed, 0, b)
        if k_ramp is not None:
            # keys scaled along the sequence: the scores, and with them the running maximum of
            # the online softmax, drift by many powers of two over the cache
            t = np.arange(L + rows, dtype=np.float32) / max(L + rows - 1, 1)
            scale = (k_ramp[0] + (k_ramp[1] - k_ramp[0]) * t)[None, :, None]
            kr = synth.f32_to_bf16_bits(synth.bf16_bits_to_f32(kr) * scale)
        kv.load(0, b, 0, kr, vr)
        if poison and L + rows + 3 <= cap:
            # rows past the block are dead: whatever they hold must not matter
            bad = np.full((shape.n_kv_heads, 3, shape.head_dim), 0x7FC0, dtype=np.uint16)  # bf16 NaN
            kv.load(0, b, L + rows, bad, bad)
        kv.set_len(b, L)
        ks[b], vs[b] = kr, vr
    rng = np.random.default_rng(seed)
    q = rng.standard_normal((B, rows, shape.n_heads, shape.head_dim)).astype(np.float32)
    if k_ramp is not None:
        # with scores this large the rounding of the queries to bfloat16 (what the tuned kernels
        # take) moves the softmax weights by percents: give both sides the rounded queries
        q = synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(q))
    out = cs.cs_op_attention(model, kv, 0, torch.from_numpy(q).to(DEV)).cpu().numpy()
    G = shape.n_heads // shape.n_kv_heads
    worst = 0.0
    for b, h in sample:
        L = lens[b]
        kc = synth.bf16_bits_to_f32(ks[b][h // G]).astype(np.float64)
        vc = synth.bf16_bits_to_f32(vs[b][h // G]).astype(np.float64)
        ref = orc.causal_attention(q[b, :, h].astype(np.float64), kc, vc, L + np.arange(rows))
        got = out[b, :, h * shape.head_dim:(h + 1) * shape.head_dim]
        err = np.abs(got - ref).max() / max(np.abs(ref).max(), 1e-6)
        worst = max(worst, err)
    kv.destroy()
    return worst


def test_attention_benchmark_shape(host_model):
    """8 streams x 18431 cached rows, 11 block rows, 32 heads over 8 KV heads, hd 128."""
    worst = _attention_case(host_model, HOST, [18431] * 8, 11,
                            [(0, 0), (0, 31), (3, 13), (7, 5), (5, 22)], seed=11)
    assert worst < 1e-2, worst


def test_attention_ragged_and_degenerate_lengths(host_model):
    lens = [0, 1, 31, 32, 33, 1000, 4097, 129]
    sample = [(b, h) for b in range(8) for h in (0, 17, 31)]
    worst = _attention_case(host_model, HOST, lens, 11, sample, seed=12, poison=True)
    assert worst < 1e-2, worst
    worst = _attention_case(host_model, HOST, [5, 300], 1, [(0, 3), (1, 30)], seed=13, poison=True)
    assert worst < 1e-2, worst


def test_attention_k32_block(host_model):
    """k = 32: 132 query rows per KV head, three query groups per workgroup column."""
    worst = _attention_case(host_model, HOST, [3000, 2999, 64, 7], 33,
                            [(0, 0), (0, 3), (1, 12), (2, 31), (3, 8)], seed=14)
    assert worst < 1e-2, worst


def test_attention_k32_block_65535_rows_batch16(host_model):
    """The long multi-turn configuration's launch: 16 streams x 65535 cached rows, 33 block rows
    (132 query rows per KV head, the wide-block kernel), 128-token V blocks up to index 511.
    Five (stream, head) pairs are checked element by element against the oracle's attention."""
    worst = _attention_case(host_model, HOST, [65535] * 16, 33,
                            [(0, 0), (3, 31), (9, 14), (15, 7), (15, 24)], seed=17, device_fill=True)
    assert worst < 1e-2, worst


def test_attention_k32_block_long_ragged(host_model):
    """Wide-block kernel with ragged long caches (lengths around the 128-token V blocks and the
    32-token K blocks) next to an empty one; rows past the block poisoned."""
    worst = _attention_case(host_model, HOST, [40000, 0, 16383, 16385, 127, 32769], 33,
                            [(0, 5), (1, 0), (2, 31), (3, 16), (4, 9), (5, 20)], seed=18, poison=True)
    assert worst < 1e-2, worst


@pytest.mark.parametrize("rows", [11, 33])
@pytest.mark.parametrize("k_ramp", [(0.05, 6.0), (6.0, 0.05)])
def test_attention_drifting_maximum(host_model, rows, k_ramp):
    """Keys that grow (shrink) 120-fold along the cache: the row maxima rise by far more than
    the 2^8 slack of the lazily updated reference again and again (or sit at the start, with
    everything after it far below), in both tuned kernels."""
    worst = _attention_case(host_model, HOST, [2500, 777, 40], rows,
                            [(0, 0), (0, 21), (1, 6), (1, 31), (2, 15)], seed=16, k_ramp=k_ramp)
    assert worst < 1e-2, worst


@pytest.mark.parametrize("k_ramp", [None, (0.05, 6.0)])
def test_attention_prompt_block(k_ramp):
    """256 block rows per stream (1024 query rows per KV head): the kernel for prompt blocks, which
    walks the tokens unsplit and writes the normalised rows itself.  Empty, short and long caches
    under the block, rows past the block poisoned."""
    w = synth.model_weights(HOST, 99, threads=16)
    m = cs.Model(w, max_batch=3, max_k=255)
    sample = [(0, 0), (0, 31), (1, 13), (2, 5), (2, 22)]
    worst = _attention_case(m, HOST, [0, 700, 2049], 256, sample, seed=21, poison=True, k_ramp=k_ramp)
    m.destroy()
    assert worst < 1e-2, worst


def _attention_kernels(kernels_of, m, shape, lens, rows):
    """The attention kernels of a block behind caches of these lengths."""
    kv = cs.KV(m, len(lens), max(lens) + rows)
    for b, n in enumerate(lens):
        kv.set_len(b, n)
    q = torch.zeros(len(lens), rows, shape.n_heads, shape.head_dim, device=DEV)
    names = kernels_of(lambda: cs.cs_op_attention(m, kv, 0, q))
    kv.destroy()
    return [n for n in names if "k_attn" in n]


def _prompt_tile(hd, rows):
    """What the name of the prompt kernel with tiles of this many query rows has in it."""
    return f"k_attn_prefillILi{hd}ELi{1 if rows == 64 else 2}ELi{4 if rows == 64 else 8}E"


@pytest.mark.parametrize("H,KVH,hd,lens,rows,k_ramp,tile", [
    (28, 4, 128, [0], 7, None, 64), (28, 4, 128, [0, 600], 65, (0.05, 6.0), 64), (28, 4, 128, [300, 0, 17], 257, None, 64),
    (8, 8, 64, [0, 33, 400], 49, None, 64), (8, 8, 64, [31, 500], 257, (6.0, 0.05), 64), (64, 8, 128, [250, 0], 17, None, 64),
    (6, 2, 64, [100, 0, 3, 64], 128, None, 64), (6, 2, 64, [0] * 34, 256, None, 256), (28, 4, 128, [0, 1] * 5, 257, None, 256)])
def test_attention_unsplit_short_contexts(kernels_of, H, KVH, hd, lens, rows, k_ramp, tile):
    """Wide blocks over short contexts, which the prompt kernel takes without splitting the tokens: 64-row tiles (most)
    and 256-row tiles (the last two), one, three, seven and eight query heads per KV head, 4 to 68 (stream, KV head)
    pairs, ragged last tiles, poisoned rows past the block."""
    shape = ModelShape("brief", 1, 256, H, KVH, hd, 256, 512, 10000.0, 1e-5, "bf16")
    m = cs.Model(synth.model_weights(shape, 97, threads=8), max_batch=len(lens), max_k=256)
    sample = [(b, h) for b in sorted({0, len(lens) // 2, len(lens) - 1}) for h in (0, H // 2, H - 1)]
    worst = _attention_case(m, shape, lens, rows, sample, seed=80 + rows, poison=True, k_ramp=k_ramp)
    assert _prompt_tile(hd, tile) in _attention_kernels(kernels_of, m, shape, lens, rows)[0]
    m.destroy()
    assert worst < 1e-2, worst


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("k_ramp", [None, (0.05, 6.0), (6.0, 0.05)])
def test_attention_prompt_block_in_large_tiles(kernels_of, hd, k_ramp):
    """The 256-row tiles of eight waves that large prompts take, over empty, short and long ragged caches, growing and
    shrinking keys, rows past the block poisoned: 640 tiles of 64 rows would be more than two per compute unit."""
    shape = ModelShape("large-tiles", 1, 256, 32, 8, hd, 256, 512, 10000.0, 1e-5, "bf16")
    lens = [0, 700, 2049, 33, 4097]
    m = cs.Model(synth.model_weights(shape, 95, threads=8), max_batch=5, max_k=255)
    sample = [(0, 0), (0, 31), (1, 13), (2, 5), (3, 22), (4, 9), (4, 30)]
    worst = _attention_case(m, shape, lens, 256, sample, seed=22, poison=True, k_ramp=k_ramp)
    assert _prompt_tile(hd, 256) in _attention_kernels(kernels_of, m, shape, lens, 256)[0]
    m.destroy()
    assert worst < 1e-2, worst


@pytest.mark.parametrize("H,KVH,hd,lens,rows,kernel", [
    (28, 4, 128, [6000, 5999, 3000, 1], 80, "k_attn_lds"), (40, 8, 128, [3000, 2999], 128, "k_attn_lds"),
    (32, 8, 64, [700], 16, "k_attn_lds"), (32, 8, 128, [3000, 700], 128, "k_attn_lds"),
    (32, 8, 64, [400], 16, _prompt_tile(64, 64)), (28, 4, 128, [500, 0, 499, 3], 80, _prompt_tile(128, 64))])
def test_attention_long_contexts_are_split_over_the_tokens(kernels_of, H, KVH, hd, lens, rows, kernel):
    """Wide blocks of few tiles behind a long context go to the kernel that splits the tokens, whatever the head group;
    behind a short one they do not."""
    shape = ModelShape("split", 1, 256, H, KVH, hd, 256, 512, 10000.0, 1e-5, "bf16")
    m = cs.Model(synth.model_weights(shape, 96, threads=8), max_batch=len(lens), max_k=rows - 1)
    sample = [(b, h) for b in range(len(lens)) for h in (0, H // 2, H - 1)]
    worst = _attention_case(m, shape, lens, rows, sample, seed=60 + rows, poison=True)
    assert kernel in _attention_kernels(kernels_of, m, shape, lens, rows)[0]
    m.destroy()
    assert worst < 1e-2, worst


@pytest.mark.parametrize("rows", [6, 21, 51, 101])
def test_attention_block_size_sweep(rows):
    """Block sizes of the paper's sweep (Sec. 5.3, Table 4: 5, 10, 50, 100 draft tokens; 20 added):
    6 rows fit one 48-row query group, 21 rows fill two groups of a three-group workgroup column
    partly, 51 and 101 rows need two and three columns with a ragged last one."""
    w = synth.model_weights(HOST, 99, threads=16)
    m = cs.Model(w, max_batch=5, max_k=100)
    sample = [(0, 0), (0, 31), (1, 13), (2, 5), (3, 22), (4, 9)]
    worst = _attention_case(m, HOST, [2500, 777, 40, 0, 4100], rows, sample, seed=30 + rows, poison=True)
    m.destroy()
    assert worst < 1e-2, worst


@pytest.mark.parametrize("H,KVH,B,rows", [(28, 4, 5, 21), (28, 4, 3, 7), (32, 8, 3, 37), (32, 8, 1, 60),
                                          (32, 8, 5, 11), (32, 8, 3, 4)])
def test_attention_even_query_groups_and_one_round(H, KVH, B, rows):
    """Wide blocks whose query groups are shared out evenly over the workgroups of a token range: 4 groups (of 147 rows)
    as 2 + 2, 49 rows in two groups, 4 groups (148 rows) as 2 + 2, 5 (240 rows) as 3 + 2; stream counts for which the
    token ranges stop at one round of the chip, also in narrow blocks (44 and 16 rows)."""
    shape = ModelShape("groups", 1, 256, H, KVH, 128, 256, 512, 10000.0, 1e-5, "bf16")
    m = cs.Model(synth.model_weights(shape, 98, threads=8), max_batch=B, max_k=rows - 1)
    lens = [2500, 777, 40, 0, 4100][-B:]
    sample = [(b, h) for b in range(B) for h in (0, H // 2, H - 1)]
    worst = _attention_case(m, shape, lens, rows, sample, seed=70 + rows, poison=True)
    m.destroy()
    assert worst < 1e-2, worst


def test_attention_hd64():
    shape = ModelShape("w-hd64", 1, 2048, 32, 8, 64, 8192, 1024, 10000.0, 1e-5, "bf16")
    w = synth.model_weights(shape, 5, threads=16)
    m = cs.Model(w, max_batch=4, max_k=10)
    worst = _attention_case(m, shape, [4096, 100, 0, 2500], 11, [(0, 0), (1, 9), (2, 31), (3, 20)],
                            seed=15)
    m.destroy()
    assert worst < 1e-2, worst


# ----------------------------------------------------------------------------------------
# whole verify step at depth
# ----------------------------------------------------------------------------------------

def _deep_verify(shape, B, L, k, check_streams, seed):
    w = synth.model_weights(shape, seed, threads=16)
    model = cs.Model(w, max_batch=B, max_k=k)
    kv = cs.KV(model, B, L + k + 8)
    rng = np.random.default_rng(seed)
    pending = rng.integers(0, shape.vocab, B)
    draft = rng.integers(0, shape.vocab, (B, k))
    dlen = np.full(B, k)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    for b in range(B):
        for layer in range(shape.n_layers):
            if b in check_streams:
                kr, vr = synth.random_kv(shape, L, seed, layer, b)
            else:   # streams the oracle does not look at: cheap device-side fill
                kr = torch.randn((shape.n_kv_heads, L, shape.head_dim), generator=gen, device=DEV).bfloat16()
                vr = torch.randn((shape.n_kv_heads, L, shape.head_dim), generator=gen, device=DEV).bfloat16()
            kv.load(layer, b, 0, kr, vr)
        kv.set_len(b, L)
    acc, nxt, logits = cs.cs_verify(model, kv, t32(pending), t32(draft), t32(dlen), k, want_logits=True)
    torch.cuda.synchronize()
    # the same step without the logits: the lm_head then takes the argmax in its own epilogue and
    # writes no logits; every stream must come out identical (same accumulators, same tie rule)
    for b in range(B):
        kv.set_len(b, L)
    acc2, nxt2, _ = cs.cs_verify(model, kv, t32(pending), t32(draft), t32(dlen), k, want_logits=False)
    torch.cuda.synchronize()
    assert torch.equal(acc, acc2) and torch.equal(nxt, nxt2)
    for b in range(B):
        row = logits[b, int(acc2[b])]
        assert float(row[int(nxt2[b])]) == float(row.max())
    logits = logits.cpu().numpy()
    worst = 0.0
    for b in check_streams:
        okv = orc.KVCache(shape, L + k + 8)
        for layer in range(shape.n_layers):
            kr, vr = synth.random_kv(shape, L, seed, layer, b)
            okv.load(layer, kr, vr)
        okv.truncate(L)
        tau, nx, ol = orc.verify(w, okv, int(pending[b]), draft[b].tolist())
        worst = max(worst, np.abs(logits[b] - ol).max())
        am = [orc.argmax_first(r) for r in ol]
        if all((np.partition(ol[i], -2)[-1] - np.partition(ol[i], -2)[-2]) > 1e-2 for i in range(tau + 1)):
            assert (int(acc[b]), int(nxt[b])) == (tau, nx)
        assert kv.len(b) == L + int(acc[b]) + 1
    kv.destroy()
    model.destroy()
    return worst


def test_verify_llama1b_full_depth():
    """Configuration 3 shape at full depth: 16 layers, 4096 cached rows, k = 10."""
    worst = _deep_verify(synth.LLAMA_1B, 1, 4096, 10, [0], seed=synth.seed_for(3))
    assert worst <= 2e-2, worst


def test_verify_llama8b_width_many_rows():
    """8B width, batch 8, k = 32: 264 block rows go through the many-row projection kernel
    (SwiGLU epilogue, K splits) and the wide-block attention kernel; 2 layers, short cache."""
    shape = synth.LLAMA_8B.with_layers(2)
    worst = _deep_verify(shape, 8, 700, 32, [0, 7], seed=synth.seed_for(5))
    assert worst <= 2e-2, worst


def test_verify_llama8b_width_528_rows():
    """8B width, batch 16, k = 32: with 528 block rows every projection runs the many-row kernel,
    so every GEMM input (both norms, the merged attention output, the SwiGLU output) is written in
    fragment order by its producer; 1 layer, short cache."""
    shape = synth.LLAMA_8B.with_layers(1)
    worst = _deep_verify(shape, 16, 300, 32, [3, 15], seed=synth.seed_for(5) + 1)
    assert worst <= 2e-2, worst


def test_verify_llama8b_width_batch8():
    """8B width, batch 8, 18431 cached rows, k = 10 (the benchmark's launch configuration),
    4 of the 32 layers; the oracle checks two sampled streams."""
    shape = synth.LLAMA_8B.with_layers(4)
    worst = _deep_verify(shape, 8, 18431, 10, [0, 5], seed=synth.seed_for(4))
    assert worst <= 2e-2, worst


@pytest.mark.parametrize("B,k", [(1, 50), (1, 100), (8, 100), (8, 20), (8, 5)])
def test_verify_llama8b_width_block_size_sweep(B, k):
    """Block sizes of the paper's sweep (Sec. 5.3, Table 4) at the 8B width, one layer, short cache:
    51 and 101 rows of a single stream (the paper's batch size) go through the weight-streaming
    projections with one and two row blocks and the wide-block attention; 808 rows (batch 8,
    k = 100) take three row blocks of the many-row projections; 168 and 48 rows sit between."""
    shape = synth.LLAMA_8B.with_layers(1)
    worst = _deep_verify(shape, B, 300, k, [B - 1], seed=synth.seed_for(5) + 10 * k + B)
    assert worst <= 2e-2, worst


@pytest.mark.parametrize("B,k", [(8, 10), (16, 32), (1, 50)])
def test_verify_llama8b_width_with_qkv_bias(B, k):
    """Biases on the q, k, v projections at the 8B width, one layer: 88 rows (added in the attention
    kernel's own rotary stage), 528 rows (the many-row rotary kernel), 51 rows of one stream (the
    small rotary kernel), against the oracle with the same biases."""
    shape = synth.LLAMA_8B.with_layers(1).with_qkv_bias()
    worst = _deep_verify(shape, B, 300, k, [B - 1], seed=synth.seed_for(5) + 100 + k)
    assert worst <= 2e-2, worst


QWEN_7B = ModelShape("qwen2.5-7b-width", 1, 3584, 28, 4, 128, 18944, 152064, 1000000.0, 1e-6, "bf16", True)


@pytest.mark.parametrize("B,k,L", [(8, 10, 300), (1, 10, 4000), (16, 32, 300)])
def test_verify_qwen7b_width(B, k, L):
    """The other model family of Sec. 4.1 at its 7B width, one layer: 28 query heads over 4 KV heads
    (seven per KV head, so 11 block rows already need two 48-row query groups), d_model 3584,
    d_ff 18944, 152064-token vocabulary, q/k/v biases; 88 and 528 block rows and one stream."""
    worst = _deep_verify(QWEN_7B, B, L, k, [B - 1], seed=synth.seed_for(5) + 300 + k + B)
    assert worst <= 2e-2, worst


def test_verify_qwen7b_width_105_rows():
    """105 block rows at the Qwen2.5-7B width: gate/up (with its SwiGLU epilogue) in one block of seven X tiles by five
    consumer waves, lm_head with and without stored logits."""
    worst = _deep_verify(QWEN_7B, 5, 300, 20, [4], seed=synth.seed_for(5) + 325)
    assert worst <= 2e-2, worst


LLAMA_70B_WIDTH = ModelShape("llama-70b-width", 1, 8192, 64, 8, 128, 28672, 128256, 500000.0, 1e-5, "bf16")


@pytest.mark.parametrize("B,k", [(8, 10), (1, 10)])
def test_verify_llama70b_width(B, k):
    """The largest width the paper runs (Sec. 4.1: 70B / 72B models), one layer: d_model 8192 (the
    widest row the norm kernel takes), 64 heads over 8 KV heads, d_ff 28672."""
    worst = _deep_verify(LLAMA_70B_WIDTH, B, 300, k, [B - 1], seed=synth.seed_for(5) + 700 + B)
    assert worst <= 2e-2, worst
