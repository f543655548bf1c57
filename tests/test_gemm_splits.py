"""Which gradient products of 16 to 23 stages (of 128) are split along K, read from the workspace
that the split's partials take (host logic; both routes' results are compared on the GPU)."""
import pytest

H = pytest.importorskip("paper_2306_11987_amd", reason="libhqlss.so not built")


def is_split(which, N, D, C):
    try:
        rule = H.workspace_bytes(which, N, D, C)
        H.debug_set_gemm_splits(1)
        return rule > H.workspace_bytes(which, N, D, C)
    finally:
        H.debug_set_gemm_splits(0)


@pytest.mark.parametrize("rows,cols,stages,dx,dw", [
    # 128 x 128 tiles: 64, 72 (uneven for both products), 96 and 110 (for dW), 144
    (1024, 1024, 16, False, False), (1024, 1024, 23, False, False), (1024, 1024, 24, True, True),
    (1536, 768, 16, False, False), (1536, 768, 19, False, False), (1536, 768, 20, True, True),
    (1536, 768, 23, True, True),
    (1024, 1536, 19, False, False), (1024, 1536, 20, False, True), (1408, 1280, 23, False, True),
    (1536, 1536, 23, False, False), (1536, 1536, 15, False, False),
])
def test_two_splits_where_they_pay(rows, cols, stages, dx, dw):
    K = 128 * stages
    assert is_split(H.WS_BWD_DX, rows, cols, K) == dx
    assert is_split(H.WS_BWD_DW, K, cols, rows) == dw
