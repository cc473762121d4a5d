"""CPU-only checks of the boundary: the shared library loads and exports every entry point
that include/copyspec.h declares, and the binding's struct layouts match the header."""
import ctypes
import itertools
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "copyspec.h")
LIB = os.path.join(ROOT, "paper_2502_08923_amd", "libcopyspec.so")


def declared_symbols():
    src = open(HEADER).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(cs_[a-z0-9_]+)\s*\(", src)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        from paper_2502_08923_amd.build import build_lib
        build_lib()
    return ctypes.CDLL(LIB)


def test_header_declares_the_named_calls():
    syms = declared_symbols()
    for name in ("cs_find_match", "cs_verify", "cs_decode", "cs_step", "cs_kv_set_len"):
        assert name in syms


def test_library_exports_every_declared_symbol(lib):
    for name in declared_symbols():
        assert hasattr(lib, name), f"{name} declared in copyspec.h but not exported"


def test_binding_lists_every_declared_symbol():
    from paper_2502_08923_amd import binding
    assert sorted(binding.EXPORTS) == declared_symbols()
    binding.load_library()


def test_struct_layouts_match_header():
    from paper_2502_08923_amd import binding
    assert ctypes.sizeof(binding.cs_model_cfg) == 12 * 4
    assert ctypes.sizeof(binding.cs_layer_weights) == 12 * 8
    assert ctypes.sizeof(binding.cs_weights) == 4 * 8
    assert ctypes.sizeof(binding.cs_stats) == 4 * 8
    assert ctypes.sizeof(binding.cs_merged_stats) == 8 * 8


def test_version_and_error_strings_without_gpu(lib):
    lib.cs_version.restype = ctypes.c_char_p
    lib.cs_last_error.restype = ctypes.c_char_p
    assert b"copyspec" in lib.cs_version()
    assert isinstance(lib.cs_last_error(), bytes)


def test_product_path_does_not_import_the_oracle():
    pkg = os.path.join(ROOT, "paper_2502_08923_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".h", ".cpp")):
                text = open(os.path.join(dirpath, f)).read()
                assert "oracle" not in text.lower(), f
    for f in os.listdir(os.path.join(ROOT, "oracle")):
        if f.endswith(".py"):
            text = open(os.path.join(ROOT, "oracle", f)).read()
            assert "paper_2502_08923_amd" not in text and "libcopyspec" not in text


@pytest.mark.parametrize("R,N,K", [(129, 1152, 16_000_000), (200, 2048, 10_000_128), (288, 8192, 8_000_000)])
def test_rows_too_long_for_the_many_row_gemm_go_to_the_other_kernel(lib, R, N, K):
    """Up to 288 rows a projection has two kernels; the one that refuses operands of 2^31 elements is not chosen for
    them, however its estimated time compares."""
    tiled = lib._Z15cs_gemm_x_tilediiib
    tiled.restype = ctypes.c_bool
    assert (R + 15) * K >= 2**31
    assert not tiled(R, N, K, True) and not tiled(R, N, K, False)


@pytest.mark.parametrize("N,K,splits", [
    (6144, 4096, {88: 4, 264: 1, 300: 4, 528: 2, 1000: 2, 4095: 1}), (4096, 4096, {88: 8, 105: 4, 300: 4, 528: 4, 1000: 2, 2048: 2}),
    (4096, 14336, {88: 8, 200: 8, 300: 8, 528: 8, 1000: 4}), (3072, 2048, {88: 4, 300: 4, 528: 2, 1000: 2}),
    (2048, 2048, {88: 4, 300: 4, 528: 4, 2048: 2}), (2048, 8192, {88: 16, 105: 8, 300: 8, 528: 8, 1000: 4, 2048: 4}),
    (4608, 3584, {105: 4, 300: 4, 528: 2, 1000: 2}), (3584, 3584, {88: 4, 300: 4, 528: 4, 1000: 2}), (3584, 18944, {88: 8, 200: 16, 528: 8})])
def test_k_splits_of_the_projections(lib, N, K, splits):
    """Every output of a projection is the sum of K / splits products in a chain, then of the splits: the rounding error
    grows with the chain, so a launch shape with fewer splits is another result and a worse one (8B q/k/v at 300 rows
    unsplit: twice the largest error against float64)."""
    shape = (ctypes.c_int * 3)()
    for R, want in splits.items():
        lib._Z13cs_gemm_shapeiiibPi(R, N, K, True, shape)
        assert shape[2] == want, (R, list(shape))


@pytest.mark.parametrize("R", [289, 528, 2048])
def test_rows_too_long_for_the_many_row_gemm_are_still_taken(lib, R):
    """The other kernel takes them, and the lm_head's as well."""
    K = 16_000_000
    lib._Z15cs_gemm_x_tilediiib.restype = ctypes.c_bool
    assert not lib._Z15cs_gemm_x_tilediiib(R, 1152, K, True) and not lib._Z15cs_gemm_x_tilediiib(R, 128256, K, False)


def test_matrix_instructions_are_the_compilers():
    """A multiply written as inline assembly is no matrix instruction to the compiler: it then places neither the wait
    states that an operand's last writer needs before it nor those that a reader of its sums needs behind it."""
    csrc = os.path.join(ROOT, "paper_2502_08923_amd", "csrc")
    for f in sorted(os.listdir(csrc)):
        for line in open(os.path.join(csrc, f)):
            assert not ("asm" in line and "v_mfma" in line), (f, line)


def test_projection_tests_reach_every_kernel(lib):
    """The launch shapes of the projection tests' matrices, which a change of the launch rules may move: every row-tile count
    of the many-row kernel (6 to 18) and of the weight-streaming one (1 to 8), the latter over less than a ring of
    four K chunks, whole rings and every remainder; its tiles of five consumer waves with 6 to 8."""
    import test_gpu_ops as ops
    reached = {}
    shape = (ctypes.c_int * 3)()
    for test in (ops.test_gemm_bf16_full_shapes, ops.test_gemm_row_sweep, ops.test_gemm_prompt_rows, ops.test_gemm_row_tile_counts_between,
                 ops.test_gemm_wide_blocks_and_five_wave_tiles, ops.test_gemm_five_wave_tiles_over_long_rows,
                 ops.test_gemm_chunk_counts_of_the_ring, ops.test_gemm_chunk_counts_in_one_row_block):
        wide = {ops.test_gemm_chunk_counts_of_the_ring: 1040, ops.test_gemm_chunk_counts_in_one_row_block: 28688}.get(test)
        marks = [(m.args[0].split(","), m.args[1]) for m in test.pytestmark if m.name == "parametrize"]
        for values in itertools.product(*(m[1] for m in marks)):
            case = {} if test is not ops.test_gemm_row_tile_counts_between else {"N": 49168, "K": 512}
            for (names, _), v in zip(marks, values):
                case.update(zip(names, v if len(names) > 1 else [v]))
            if wide:
                case.update(N=wide, K=128 * case["chunks"])
            R, N, K = case["R"], case["N"], case["K"]
            lib._Z13cs_gemm_shapeiiibPi(R, N, K, True, shape)
            per_split = -(-K // shape[2] // 128)
            while K > 0:
                reached.setdefault((shape[0], shape[1]), set()).add(min(per_split, K // 128))
                K -= 128 * per_split
    assert {t for w, t in reached if w == 0} == set(range(6, 19))
    for waves, tiles in [(4, t) for t in range(1, 9)] + [(5, 6), (5, 7), (5, 8)]:
        chunks = reached[waves, tiles]
        assert any(c < 4 for c in chunks) and any(c > 4 for c in chunks), (waves, tiles, chunks)
        if waves == 4:
            assert {1, 2, 3} <= chunks and {c % 4 for c in chunks if c >= 4} == {0, 1, 2, 3}, (tiles, chunks)
