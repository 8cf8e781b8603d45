"""Which kernels the calls of include/bimask.h launch, checked on the host: the library's objects linked against a HIP runtime
that records launches instead of making them (tests/dispatch/hip_stub.cpp).  Pointers are never dereferenced."""
import collections
import ctypes
import math
import os
import random
import re
import shutil
import subprocess

import pytest

import paper_2302_06058_amd as bm
import test_gpu_gemm_exact as exact
import test_gpu_parity_small as small
from paper_2302_06058_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
Launch = collections.namedtuple("Launch", "kernel args grid threads lds")
A, B, C, D, E = (0x10000000000 * k for k in range(1, 6))           # far apart, aligned

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")


@pytest.fixture(scope="module")
def rec(tmp_path_factory):
    from paper_2302_06058_amd import build as b
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    out = tmp_path_factory.mktemp("dispatch")
    objs = []
    for s in b.SOURCES:
        o = os.path.join(b.OBJ, s[:-4] + ".o")
        if not os.path.exists(o):
            if not os.path.exists(hipcc):
                pytest.skip("library objects not built and no hipcc")
            o = str(out / (s[:-4] + ".o"))
            subprocess.run([hipcc] + b.FLAGS + ["-c", os.path.join(b.CSRC, s), "-o", o], check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
        objs.append(o)
    so = str(out / "librecord.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wl,-Bsymbolic", os.path.join(ROOT, "tests", "dispatch", "hip_stub.cpp")] + objs
                   + ["-o", so], check=True)
    lib = ctypes.CDLL(so)
    for name, (res, args) in bm._SIGNATURES.items():
        fn = getattr(lib, name)
        fn.restype, fn.argtypes = res, args
    lib.stub_launches.restype = lib.stub_kernels.restype = ctypes.c_char_p

    def call(name, *args):
        lib.stub_clear()
        status = getattr(lib, name)(*args)
        launches = []
        for line in lib.stub_launches().decode().splitlines():
            k, grid, threads, lds = line.split("|")
            m = re.fullmatch(r"(\w+)(?:<(.*)>)?", k)
            launches.append(Launch(m.group(1), m.group(2) or "", tuple(map(int, grid.split(","))), int(threads), int(lds)))
        for l in launches:                               # a dimension of a launch holds fewer than 2^32 work-items
            assert l.grid[0] * l.threads < 1 << 32 and l.grid[1] < 1 << 16, l
        return status, launches

    call.lib = lib
    return call


def fwd(rec, I, J, T, N=2, M=4, dtype=bm.BF16, ld=0, X=A):
    st, l = rec("bimask_sparse_gemm_fwd", X, T, ld or J, B, C, I, J, dtype, N, M, D, I, None, 0, None)
    assert st == 0
    return l


def bwd(rec, I, J, T, N=2, M=4, dtype=bm.BF16, dY=A, dX=D, ld=0, perm=C, lddx=0):
    need = bm.workspace_bytes(bm.WS_GEMM_BWD, I, J, T, 0, dtype, N, M)
    st, l = rec("bimask_sparse_gemm_bwd", dY, T, ld or I, perm, B, C, I, J, dtype, N, M, dX, lddx or J, E, need, None)
    assert st == 0
    return l


@pytest.mark.parametrize("I,J,T", [(4096, 8, (1 << 20) + 21), (4096, 512, (1 << 20) + 21), (64, 32, 1 << 28), (16, 64, 1 << 30), (65536, 8, 1 << 18)])
def test_fp32_grids_stay_within_a_launch(rec, I, J, T):
    (l,) = fwd(rec, I, J, T, dtype=bm.F32)               # the fixture checks the dimensions
    rows = 16 * int((l.args.split(", ") + ["1"])[3])     # weight rows of a workgroup: 16 per row tile
    assert l.kernel == "k_gemm_f32" and l.grid[0] * l.grid[1] >= -(-T // 16) * -(-I // rows)


@pytest.mark.parametrize("C_,T,N,M,dtype,direct", [(64, 70, 2, 4, bm.F32, "k_gemm_f32"), (64, 200, 4, 8, bm.BF16, "k_unpermute_dense")])
def test_backward_product_on_top_of_its_input_copies_it_first(rec, C_, T, N, M, dtype, direct):
    row = C_ * (4 if dtype == bm.F32 else 2)
    assert bwd(rec, C_, C_, T, N, M, dtype)[0].kernel == direct
    assert bwd(rec, C_, C_, T, N, M, dtype, dX=A + T * row)[0].kernel == direct          # next to each other
    assert bwd(rec, C_, C_, T, N, M, dtype, dX=A - T * row)[0].kernel == direct
    for dX in (A, A + (T - 1) * row, A - (T - 1) * row):
        assert bwd(rec, C_, C_, T, N, M, dtype, dX=dX)[0].kernel.startswith("k_gather_cols"), dX - A


@pytest.mark.parametrize("I,J,T,N,M", [(384, 384, 9001, 2, 4), (384, 384, 9001, 4, 8), (512, 512, 9001, 4, 8), (1032, 456, 5003, 2, 4), (392, 392, 17003, 2, 4)])
def test_fused_gather_in_place_leaves_each_token_row_to_one_workgroup(rec, I, J, T, N, M):
    (l,) = bwd(rec, I, J, T, N, M, dX=A)
    assert l.kernel in ("k_gemm_sp24_coltile", "k_gemm_sp24_resident") and l.grid[1] == 1, l


def pieces_of_weight_rows(l, J):
    """Workgroups that read the same token rows, each for some of the J weight rows."""
    if l.kernel.startswith("k_gemm_sp24_narrow"):        # 32 weight rows per row tile; the pieces follow each other in blockIdx.x
        return -(-J // (32 * int(l.args.split(",")[0])))
    assert l.kernel in ("k_gemm_sp24_coltile", "k_gemm_sp24_resident"), l
    return l.grid[1]


@pytest.mark.parametrize("I,J,T,N,M", exact.IN_PLACE_SHAPES)
def test_dX_on_dY_without_a_workspace_leaves_each_token_row_to_one_workgroup(rec, I, J, T, N, M):
    ld = max(I, J)
    (l,) = bwd(rec, I, J, T, N, M, dX=A, ld=ld, lddx=ld)
    assert pieces_of_weight_rows(l, J) == 1, l


def test_dX_on_dY_without_a_workspace_over_all_forms(rec):
    rng = random.Random(31)
    for _ in range(3000):
        N, M = rng.choice(((2, 4), (1, 4), (2, 8), (4, 8)))
        I, J = (M * round(math.exp(rng.uniform(0, math.log(c / M)))) for c in (2048, 4608))
        T, ld = round(math.exp(rng.uniform(0, 12))), (max(I, J) + rng.choice((0, 0, 2, 8)) + 1) // 2 * 2
        if bm.workspace_bytes(bm.WS_GEMM_BWD, I, J, T, 0, bm.BF16, N, M) or (I > 512 or N > 2) and ld % 8:
            continue
        (l,) = bwd(rec, I, J, T, N, M, dX=A, ld=ld, lddx=ld)
        assert pieces_of_weight_rows(l, J) == 1, (I, J, T, N, M, ld, l)


@pytest.mark.parametrize("I,J,T,N,M", [(384, 384, 25216, 2, 4), (256, 64, 40000, 2, 4), (1152, 384, 25216, 2, 4), (384, 1536, 9000, 4, 8), (128, 256, 3000, 2, 4)])
def test_dX_beside_dY_in_one_buffer_takes_the_way_of_separate_buffers(rec, I, J, T, N, M):
    ld = I + J
    apart = bwd(rec, I, J, T, N, M, ld=ld, lddx=ld)
    assert bwd(rec, I, J, T, N, M, dX=A + 2 * I, ld=ld, lddx=ld) == apart and bwd(rec, I, J, T, N, M, dX=A - 2 * J, ld=ld, lddx=ld) == apart
    assert bwd(rec, I, J, T, N, M, dX=A + 2 * ld * (T // 2) + 2 * I, ld=ld, lddx=ld) == apart


# the tile of the streaming kernel (weight rows, tokens, wavefronts M and N, groups), or another kernel
@pytest.mark.parametrize("I,J,T,N,M,ld,want", [
    (512, 264, 64, 2, 4, 0, "64, 32, 2, 1, 4"), (512, 384, 1024, 2, 4, 0, "64, 32, 2, 1, 4"), (512, 1152, 2000, 2, 4, 0, "64, 64, 2, 2, 2"),
    (512, 256, 64, 2, 4, 0, "128, 64, 4, 1, 1"), (1000, 256, 64, 2, 4, 0, "64, 32, 2, 1, 4"), (1000, 256, 8, 2, 4, 0, "k_gemm_sp24_resident"),
    (512, 192, 64, 2, 4, 0, "64, 32, 2, 1, 4"), (512, 192, 8, 2, 4, 0, "k_gemm_sp24_resident"), (512, 128, 64, 2, 4, 0, "k_gemm_sp24_resident"),
    (512, 132, 64, 2, 4, 0, "k_gemm_sp24_resident"), (512, 260, 64, 2, 4, 0, "128, 64, 4, 1, 1"), (512, 264, 64, 2, 4, 266, "128, 64, 4, 1, 1"),
    (512, 388, 64, 2, 4, 0, "64, 32, 2, 1, 4"), (64, 576, 8000, 2, 4, 0, "64, 32, 2, 1, 4"), (64, 576, 13000, 2, 4, 0, "64, 64, 2, 2, 1"),
    (64, 256, 784, 4, 8, 0, "64, 64, 2, 2, 1"), (64, 264, 784, 4, 8, 0, "64, 32, 2, 1, 4"), (512, 128, 256, 4, 8, 0, "128, 64, 4, 1, 1"),
    (512, 136, 256, 4, 8, 0, "64, 32, 2, 1, 4")])
def test_split_contractions_are_taken_where_they_gain(rec, I, J, T, N, M, ld, want):
    (l,) = fwd(rec, I, J, T, N, M, ld=ld)
    assert (l.args.startswith(want + ", ") if l.kernel == "k_gemm_sp24" else l.kernel == want), l


# forward products (K terms to A columns) on the wavefront-private kernel: whole pieces and row tiles whatever their number
@pytest.mark.parametrize("K", [64, 128])
@pytest.mark.parametrize("A_", [32, 64, 96, 128, 160, 192, 256])
def test_whole_pieces_and_row_tiles_take_the_instance_for_them(rec, K, A_):
    for T in (100, 70000):
        for l in (*fwd(rec, A_, K, T), *bwd(rec, K, A_, T)):
            assert l.kernel == "k_gemm_sp24_narrow_rows" and l.args.endswith("true"), l
    for l in (*fwd(rec, A_, K - 8, 100), *fwd(rec, A_ - 8, K, 100), *bwd(rec, K - 8, A_, 100)):
        assert l.kernel == "k_gemm_sp24_narrow_rows" and l.args.endswith("false"), l


@pytest.mark.parametrize("I,J,T,want", [
    (256, 32, 100, "narrow_rows"), (256, 64, 4000, "narrow_rows"), (256, 64, 40000, "narrow_rows"), (256, 64, 2000, "coltile"), (256, 56, 40000, "coltile"), (248, 64, 40000, "coltile"),
    (144, 32, 70000, "narrow"), (160, 8, 70000, "narrow"), (144, 32, 48000, "coltile"), (168, 32, 200000, "coltile"), (144, 40, 200000, "coltile")])
def test_narrow_gathers_of_two_stages(rec, I, J, T, want):
    assert bwd(rec, I, J, T)[0].kernel == "k_gemm_sp24_" + want


@pytest.mark.parametrize("I,J,T,want", [
    (104, 256, 60000, "k_gemm_sp24"), (104, 256, 100000, "k_gemm_sp24_narrow_rows"), (128, 256, 20000, "k_gemm_sp24_narrow_rows"), (128, 256, 16000, "k_gemm_sp24"),
    (104, 248, 20000, "k_gemm_sp24_narrow_rows"), (64, 256, 100, "k_gemm_sp24_narrow_rows")])
def test_narrow_products_of_two_stages(rec, I, J, T, want):
    assert fwd(rec, I, J, T)[0].kernel == want


# columns that end inside a 128-byte line against the resident kernel with full rounds; four stages and a second round just begun
@pytest.mark.parametrize("d,K,A_,T,want", [
    ("p", 192, 3040, 32475, "resident"), ("p", 160, 3232, 6665, "resident"), ("f", 224, 3680, 16316, "resident"), ("p", 192, 3072, 32475, "wide"),
    ("p", 192, 3040, 34000, "wide"), ("p", 192, 736, 32475, "wide"), ("p", 288, 3040, 32475, "wide"), ("f", 224, 992, 16316, "wide"), ("p", 192, 3040, 18000, "wide"),
    ("f", 448, 384, 16681, ""), ("f", 480, 640, 18165, ""), ("f", 512, 576, 20953, ""), ("f", 448, 480, 18000, "wide"), ("f", 416, 1056, 19755, "wide"),
    ("f", 416, 544, 21834, "wide"), ("f", 384, 384, 18000, "wide"), ("p", 448, 576, 18000, "wide")])
def test_wide_products_and_their_neighbours(rec, d, K, A_, T, want):
    (l,) = fwd(rec, A_, K, T) if d == "f" else bwd(rec, K, A_, T)
    assert l.kernel == "k_gemm_sp24" + ("_" + want if want else ""), l


@pytest.mark.parametrize("I,J,T,N,M,fused", [
    (1792, 1952, 68, 4, 8, False), (1792, 1952, 28, 4, 8, True), (1792, 1952, 250, 4, 8, True), (1376, 1600, 121, 4, 8, True), (1752, 4056, 470, 4, 8, False),
    (1632, 3776, 527, 4, 8, True), (1216, 3776, 300, 4, 8, True), (2048, 3680, 915, 2, 4, False), (1984, 3808, 242, 2, 4, False), (2016, 3752, 515, 2, 4, True),
    (1792, 3808, 242, 2, 4, True)])
def test_few_tokens_on_large_weights_gather_first(rec, I, J, T, N, M, fused):
    kernels = [l.kernel for l in bwd(rec, I, J, T, N, M)]
    assert kernels == ["k_gemm_sp24_coltile"] if fused else kernels[0].startswith("k_gather_cols") and len(kernels) == 2, kernels


def test_dense_backward_puts_the_weights_in_natural_order(rec):
    for (I, J, N, M, T), rows in small.NATURAL_ORDER.items():
        l = bwd(rec, I, J, T, N, M)
        assert (l[0].lds == (I + 8) * 2 * rows and l[0].kernel == "k_unpermute_dense") if rows else l[0].kernel.startswith("k_gather_cols"), (I, J, T)
        if rows:
            assert bwd(rec, I, J, T, N, M, ld=I + 24)[0].kernel == "k_unpermute_dense"
            assert bwd(rec, I, J, T, N, M, ld=I + 2)[0].kernel.startswith("k_gather_cols")
    for I, J, T, natural in ((4096, 2976, 3000, True), (8192, 2240, 3000, False), (8192, 1984, 3000, True), (16384, 1472, 3000, False), (16384, 992, 3000, True)):
        assert (bwd(rec, I, J, T, 4, 8)[0].kernel == "k_unpermute_dense") == natural, (I, J, T)


def label(l):
    """A kernel as the table of test_gpu_gemm_exact.py names it."""
    a = l.args.split(", ")
    if l.kernel == "k_gemm_sp24":
        return f"{'split ' if int(a[4]) > 1 else ''}{a[0]} x {a[1]}"
    if l.kernel == "k_gemm_sp24_resident":
        return f"resident {a[0]} x {a[1]}{' persistent' if a[0] == '256' and a[4] == 'true' else ''}"
    return "gather" if l.kernel.startswith("k_gather_cols") else l.kernel.replace("k_gemm_sp24_", "")


def test_exact_products_run_on_the_kernels_that_their_table_names(rec):
    for (I, J, T), want in exact.SP24_SHAPES.items():
        assert (", ".join(map(label, fwd(rec, I, J, T))), ", ".join(map(label, bwd(rec, I, J, T)))) == want, (I, J, T)


def test_exact_products_reach_every_instance_of_the_gemm_kernels(rec):
    reached = set()
    for I, J, T, N, M, dtype, perms in exact.exact_products():
        code = bm.F32 if dtype == synth.F32 else bm.BF16
        reached.update(fwd(rec, I, J, T, N, M, code))
        for perm in perms:
            reached.update(bwd(rec, I, J, T, N, M, code, perm=C if perm else None))
    for I, J, T, N, M in exact.IN_PLACE_SHAPES:
        ld = max(I, J)
        reached.update(bwd(rec, I, J, T, N, M) + bwd(rec, I, J, T, N, M, dX=A, ld=ld, lddx=ld))
    names = {f"{l.kernel}<{l.args}>" if l.args else l.kernel for l in reached}
    families = ("k_gemm_sp24", "k_gemm_f32", "k_unpermute_dense", "k_gather_cols_rows")
    missing = {k for k in rec.lib.stub_kernels().decode().splitlines() if k.startswith(families)} - names
    assert not missing, sorted(missing)


@pytest.mark.parametrize("I,J,N,M,dtype,want", [
    (3536, 3472, 1, 16, bm.BF16, "16, 128, true"), (3536, 3472, 8, 16, bm.BF16, "16, 128, true"), (3072, 4096, 8, 16, bm.BF16, "16, 128, false"),
    (3536, 3472, 8, 16, bm.F32, "16, 128, false"), (3536, 3472, 4, 8, bm.BF16, "8, 128, false"), (1024, 1024, 1, 16, bm.BF16, "16, 32, false")])
def test_backward_masks_of_16_on_fewer_registers(rec, I, J, N, M, dtype, want):
    st, (l,) = rec("bimask_backward_mask_compress", A, I, J, J, dtype, N, M, B, C, D, E, A, None)
    assert st == 0 and l.kernel == "k_backward" and l.args.endswith(want), l
    for I, J, lean in ((3536, 3472, "true"), (5088, 4016, "false"), (3632, 8384, "true")):           # the mask alone: 784, 1280 and 1914 tiles
        st, (l,) = rec("bimask_backward_mask", A, I, J, J, bm.BF16, 4, 16, B, C, D, None)
        assert st == 0 and l.args.endswith("16, 128, " + lean), l


def search(rec, I, J, N, M, K):
    need = bm.workspace_bytes(bm.WS_PERM_SEARCH, I, J, 0, K, bm.BF16, N, M)
    st, l = rec("bimask_perm_search", A, I, J, N, M, B, K, C, C, D, E, need, None)
    assert st == 0 and l[-1].kernel == "k_perm_final"
    return l[0].kernel


def group(rec, shapes, N, M, K):
    arr = (bm.GroupLayer * len(shapes))()
    for g, (I, J) in zip(arr, shapes):
        g.I, g.J, g.ldw = I, J, J
        g.B_bits, g.perms, g.scores, g.best, g.best_perm, g.workspace = A, B, C, C, D, E
        g.workspace_bytes = bm.workspace_bytes(bm.WS_PERM_SEARCH, I, J, 0, K, bm.BF16, N, M)
    st, l = rec("bimask_perm_search_group", ctypes.cast(arr, ctypes.c_void_p), len(shapes), N, M, K, None)
    assert st == 0 and l[-1].kernel == "k_perm_final_group"
    return [x.kernel for x in l[:-1]]


def test_searches_of_the_parity_tests_reach_the_kernels_they_name(rec):
    for c in small.LDS_SEARCHES:
        assert search(rec, *c) == "k_perm_score_lds", c
    for N, M, K in small.GROUP_SEARCHES_LDS:
        assert group(rec, small.group_search_shapes(M), N, M, K)[0] == "k_perm_score_lds_group", (N, M, K)
    for N, M, K in small.GROUP_SEARCHES_L2:
        assert set(group(rec, small.group_search_shapes(M), N, M, K)) == {"k_perm_score_group"}, (N, M, K)


DEIT = [(1152, 384), (384, 384), (1536, 384), (384, 1536)] * 12


def test_search_scores_from_lds_where_that_is_shorter(rec):
    for I, J, N, M, K in ((4096, 11008, 2, 4, 100), (3072, 1504, 4, 8, 100), (2048, 4608, 4, 8, 100)):
        assert search(rec, I, J, N, M, K) == "k_perm_score_lds", (I, J, N, M, K)
    for I, J, N, M, K in ((4096, 4096, 2, 4, 100), (1024, 11008, 4, 8, 100), (1024, 11008, 1, 16, 100), (4096, 11008, 1, 4, 32), (4096, 11008, 4, 8, 32)):
        assert search(rec, I, J, N, M, K) == "k_perm_score", (I, J, N, M, K)


def test_group_search_scores_from_lds_where_that_is_shorter(rec):
    assert group(rec, DEIT, 2, 4, 100) == ["k_perm_score_lds_group"]
    assert group(rec, DEIT, 4, 8, 100) == ["k_perm_score_lds_group"]
    for shapes, N, M, K in ((DEIT, 2, 4, 16), ([(64, 64)] * 63, 2, 4, 40), ([(64, 64)] * 63, 1, 16, 100), ([(512, 1152)] * 32, 1, 16, 40),
                            ([(1152, 9216)] * 36, 4, 8, 100), ([(1152, 9216)] * 36, 1, 16, 100), (DEIT[:24], 2, 4, 100)):
        assert set(group(rec, shapes, N, M, K)) == {"k_perm_score_group"}, (shapes[0], len(shapes), N, M, K)


def test_search_falls_back_where_the_lds_limit_cannot_be_raised(rec):
    rec.lib.stub_refuse_lds(1)
    try:
        for N, M in ((2, 4), (4, 8), (1, 16)):
            assert search(rec, 3072, 1504, N, M, 100) == "k_perm_score"
            assert set(group(rec, DEIT, N, M, 100)) == {"k_perm_score_group"}
    finally:
        rec.lib.stub_refuse_lds(0)
    assert search(rec, 3072, 1504, 2, 4, 100) == "k_perm_score_lds"


def test_no_kernel_keeps_registers_in_scratch(rec, tmp_path):
    """A spilled register is reloaded through the vector-memory path, in order behind every load and store in flight."""
    from paper_2302_06058_amd import build as b
    llvm = "/opt/rocm/llvm/bin/"
    if not os.path.exists(llvm + "llvm-readelf") or not os.path.isdir(b.OBJ):
        pytest.skip("no LLVM tools or no library objects")
    kernels = 0
    for s in b.SOURCES:
        obj, fat, co = os.path.join(b.OBJ, s[:-4] + ".o"), str(tmp_path / "fat"), str(tmp_path / "co")
        if not os.path.exists(obj) or subprocess.run([llvm + "llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, obj, os.devnull], stderr=subprocess.DEVNULL).returncode:
            continue                                     # (no kernels in this file)
        subprocess.run([llvm + "clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--input=" + fat, "--output=" + co], check=True)
        notes = subprocess.run([llvm + "llvm-readelf", "--notes", co], check=True, capture_output=True, text=True).stdout
        scratch = dict(re.findall(r"\.name: +(_Z\S+)\n +\.private_segment_fixed_size: (\d+)", notes))
        assert not any(map(int, scratch.values())), {k: v for k, v in scratch.items() if v != "0"}
        kernels += len(scratch)
    assert kernels >= len(rec.lib.stub_kernels().decode().splitlines())
