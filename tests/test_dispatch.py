"""The shapes of the GPU tests take the kernels that the tests name: every
table of (shape, kernel) in them against the launchers' own rules.  CPU only,
so that a changed rule is seen before a GPU run."""
import pytest

import paper_2406_13868_amd as sdq
from tests import test_gpu_bf16_out as bf16_out
from tests import test_gpu_dual as dual
from tests import test_gpu_dual_tiled as dual_tiled
from tests import test_gpu_gemm as gemm
from tests import test_gpu_partial_chunk as partial
from tests import test_zz_no_alloc as no_alloc
from tests.gpu_util import kernel_of

INT, MX, DUAL = sdq.Config.int_family(), sdq.Config.mx_family(), sdq.Config.dual_family()


def _cases():
    for M, N, K, kernel in dual.FORMS + dual_tiled.NAN_SHAPES:
        yield DUAL, M, N, K, sdq.PATH_AUTO, kernel
    for M, N, K, form in dual_tiled.SHAPES:
        yield DUAL, M, N, K, sdq.PATH_AUTO, dual_tiled.kernel_name(form)
    for fam, M, N, K, kernel in gemm.KERNELS_ABOVE_64 + partial.KERNELS:
        yield INT if fam == "int" else MX, M, N, K, sdq.PATH_MFMA, kernel
    for M, N, K, fmt_o, kernel in gemm.INT_32_ROWS:
        yield sdq.Config.int_family(fmt_o=fmt_o), M, N, K, sdq.PATH_MFMA, kernel
    for M, N, K, kernel in gemm.MX_SPLITK:
        yield MX, M, N, K, sdq.PATH_SPLITK, kernel
    for fam, fmt_o, M, N, K, path, kernel in bf16_out.WIDE:
        yield sdq.Config.int_family(fmt_o=fmt_o) if fam == "int" else MX, M, N, K, path, kernel
    for fam, *shapes in no_alloc.STATIC_SPLITK:
        for M, N, K, kernel in shapes:
            yield INT if fam == "int" else MX, M, N, K, sdq.PATH_SPLITK, kernel


@pytest.mark.parametrize("cfg,M,N,K,path,kernel", list(_cases()))
def test_the_shape_takes_the_kernel(cfg, M, N, K, path, kernel):
    assert kernel_of(cfg, M, N, K, path) == kernel


def test_every_kernel_of_the_dispatch_is_named_by_a_test():
    seen = {kernel.split(" (")[0] for *_, kernel in _cases()}
    assert seen >= {"dual_splitk", "dual_tiled 32x128", "dual_tiled 64x128", "dual_tiled 64x256", "dual_tiled 128x256",
                    "int_splitk 32", "int_splitk 64", "int_tiled", "int_split 32", "int_split 64", "int_tiled 128",
                    "mx_small", "mx_mfma 32", "mx_mfma 64", "mx_mfma 128"}


DUAL2 = sdq.Config("dual", 2, 8, "int8", 4, 8, "e2m1", "int8")
INT8O, INT8S = sdq.Config.int_family(fmt_o="int8"), sdq.Config("int", 1, 8, "e4m3", 3, 8, "int4", "int8", sfmt_i="e4m3")


@pytest.mark.parametrize("cfg,M,N,K,kernel", [
    # long rows, few of them: the kernel for few tokens walks all of K in each
    # workgroup, and leaves them to the K ranges
    (INT, 16, 512, 11008, "int_split 32 (21 K ranges)"), (INT, 9, 1024, 8704, "int_split 32 (17 K ranges)"),
    (INT, 9, 1024, 8672, "int_small"), (INT, 16, 1056, 13824, "int_small"),
    (INT8S, 16, 1024, 8704, "int_small"), (INT8S, 16, 1024, 10240, "int_split 32 (20 K ranges)"),
    (INT8O, 16, 512, 11008, "int_small"), (INT8O, 16, 512, 12288, "int_split 32 (24 K ranges)"),
    (INT, 17, 1536, 8192, "int_split 32 (16 K ranges)"), (INT, 17, 1568, 8192, "int_small"),
    (INT, 32, 2048, 12288, "int_split 32 (24 K ranges)"), (INT8S, 64, 1024, 10208, "int_small"),
    (INT8S, 64, 1024, 10240, "int_split 64 (20 K ranges)"), (INT8O, 32, 1024, 11008, "int_split 32 (21 K ranges)"),
    (INT, 32, 2080, 13824, "int_small"), (INT, 32, 2048, 8160, "int_small"),
    (INT, 33, 512, 11008, "int_split 64 (21 K ranges)"), (INT8O, 64, 1024, 8192, "int_split 64 (16 K ranges)"),
    (INT, 64, 1056, 11008, "int_small"), (INT, 64, 1024, 8160, "int_small"),
    # (MX: above 32 tokens alike)
    (MX, 32, 1024, 16000, "mx_small"), (MX, 33, 1024, 8160, "mx_small"), (MX, 64, 1024, 8192, "mx_mfma 64 (16 K ranges)"),
    (MX, 64, 1536, 11008, "mx_mfma 64 (18 K ranges)"), (MX, 64, 1568, 12288, "mx_small"),
    (MX, 48, 2048, 12320, "mx_mfma 64 (20 K ranges)"), (MX, 64, 2048, 14336, "mx_small"),
    (MX, 64, 2048, 14368, "mx_mfma 64 (23 K ranges)"), (MX, 64, 8192, 5120, "mx_small"),
    (MX, 64, 8192, 5152, "mx_mfma 64 (7 K ranges)"), (MX, 64, 8224, 3072, "mx_small"),
    (MX, 64, 11008, 4096, "mx_mfma 64 (5 K ranges)"), (MX, 128, 256, 11008, "mx_mfma 128 (18 K ranges)"),
    (MX, 128, 512, 11008, "mx_small"), (MX, 128, 1024, 16000, "mx_mfma 128 (25 K ranges)"),
    (MX, 192, 1024, 16000, "mx_small"), (MX, 128, 256, 8192, "mx_small"),
    # dual: the split-K form for few tokens on wide layers
    (DUAL, 12, 11008, 4096, "dual_splitk"), (DUAL, 13, 11008, 4096, "dual_tiled 32x128"),
    (DUAL2, 16, 11008, 4096, "dual_splitk"), (DUAL2, 17, 11008, 4096, "dual_tiled 32x128"),
    (DUAL, 24, 8224, 768, "dual_splitk"), (DUAL, 24, 8224, 800, "dual_tiled 32x128"),
    (DUAL, 32, 11008, 512, "dual_splitk"), (DUAL, 25, 11008, 544, "dual_tiled 32x128"),
    (INT, 1, 4096, 4096, "int_decode"), (INT, 16, 4096, 4096, "int_small"), (INT, 64, 16384, 4096, "int_split 64 (4 K ranges)"),
    (INT, 201, 4096, 11008, "int_tiled 128 (8 K ranges)"), (INT, 2048, 4096, 4096, "int_tiled"),
    (MX, 1, 4096, 4096, "mx_small"), (MX, 301, 4096, 11008, "mx_mfma 128 (5 K ranges)"),
    (MX, 16, 22016, 4096, "mx_mfma 32"), (MX, 16, 4096, 512, "mx_mfma 32"),
    (MX, 2048, 11008, 4096, "mx_dense (two passes)"),
    (DUAL, 1, 4096, 4096, "dual_decode"), (DUAL, 256, 4096, 4096, "dual_tiled 32x128"),
    (DUAL, 4096, 11008, 4096, "dual_tiled 128x256")])
def test_what_the_entry_points_choose_with_a_workspace(cfg, M, N, K, kernel):
    assert kernel_of(cfg, M, N, K) == kernel
