"""Which tile a GEMM of 129..256 rows takes, at the sizes where both were measured (no GPU needed)."""
import pytest

from tests.helpers import gemm_shape


@pytest.mark.parametrize("N,K,M,kind,mb", [
    # the head (K whole): 64-row tiles while they fit the chip in one round, tall ones beyond; 8-bit weights not with four row blocks
    (8192, 4096, 160, "head", 2), (16384, 4096, 160, "head", 2), (16384, 4096, 256, "head", 2), (24576, 4096, 160, "head", 3), (24576, 4096, 256, "head", 4),
    (32000, 4096, 192, "head", 3), (32000, 4096, 256, "head", 4), (24576, 4096, 160, "head w8", 3), (24576, 4096, 256, "head w8", 2), (32000, 2048, 224, "head w8", 2),
    # hi + lo projections: tall where 64-row tiles are not split and the tall ones do less work each, from K = 2560 on
    (6144, 4096, 256, "", 2), (8192, 4096, 256, "", 2), (9216, 4096, 256, "", 4), (10240, 4096, 224, "", 4), (11264, 4096, 256, "", 2), (14336, 4096, 256, "", 2),
    (10240, 4096, 160, "", 2), (11264, 4096, 160, "", 3), (14336, 4096, 160, "", 3), (16384, 4096, 192, "", 3), (18432, 4096, 192, "", 2),
    (9216, 2560, 256, "w8", 4), (9216, 2048, 256, "", 2), (12288, 2048, 160, "", 2), (12288, 2560, 160, "w8", 3),
    # fp16 inputs, K split: tall with 16-bit weights from an eighth of the chip on
    (1024, 3584, 256, "f16", 2), (2048, 7168, 256, "f16", 2), (3072, 10752, 160, "f16", 3), (4096, 14336, 160, "f16", 3), (4096, 14336, 256, "f16", 4),
    (8192, 28672, 256, "f16", 4), (4096, 14336, 256, "f16 w8", 2), (6144, 21504, 160, "f16 w8", 2),
])
def test_row_blocks_of_plain_outputs(N, K, M, kind, mb):
    g = gemm_shape(N, K, M, w8="w8" in kind, f16="f16" in kind or "head" in kind, whole="head" in kind)
    assert g["wide"] and g["tile_nb"] == 8 and g["mb"] == mb, g
    assert g["m_tiles"] == -(-M // (32 * mb)) and g["n_tiles"] == -(-N // 256)


def test_row_blocks_of_the_fused_gate_up_projection():
    assert [gemm_shape(28672, 4096, M, f16=True, swiglu=True)["mb"] for M in (132, 192, 196, 256)] == [3, 3, 4, 4]
