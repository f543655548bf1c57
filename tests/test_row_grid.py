"""How the row kernels share a grid between two tensors and choose their row groups (host logic)."""
import pytest

H = pytest.importorskip("paper_2306_11987_amd", reason="libhqlss.so not built")

WG = 512  # threads of a workgroup


def needed(rows, cols, log2g, flat):
    if flat:
        return -(-rows * (cols // 16) // WG)
    return -(-rows // (WG >> log2g))


@pytest.mark.parametrize("flat", [False, True])
@pytest.mark.parametrize("cap", [512, 768, 1024])
def test_no_job_loses_its_share_of_the_grid(cap, flat):
    """The grid fits the device, and each job gets what it needs or at least 7/8 of its share by
    size, rounded down to 8 workgroups: a short batch beside a wide weight once got a single one."""
    rows = [1, 7, 16, 33, 48, 64, 80, 127, 200, 777, 1024, 5001, 16384, 65536]
    for cols in (64, 832, 1024, 4096, 8192, 11008):
        for r0 in rows:
            for r1 in rows[4:]:
                jobs = H.debug_row_grid(r0, r1, cols, cap=cap, flat=flat)
                wg = [j[0] for j in jobs]
                assert min(wg) >= 1 and sum(wg) <= cap, (cols, r0, r1, wg)
                for r, (w, l) in zip((r0, r1), jobs):
                    share = cap * r // (r0 + r1)
                    want = min(needed(r, cols, l, flat), max(1, 7 * share // 8 // 8 * 8))
                    assert w >= want, (cols, r0, r1, wg, want)
                    # rows taken in several rounds stay on one XCD from kernel to kernel
                    assert w == needed(r, cols, l, flat) or w % 8 == 0, (cols, r0, r1, wg)


def test_one_tensor_takes_the_whole_grid():
    for cols in (64, 832, 4096):
        for r in (1, 100, 16384, 65536):
            (w, l), (w1, _) = H.debug_row_grid(r, 0, cols)
            assert w == min(needed(r, cols, l, False), 1024) and w1 == 0


def default_group(cols):
    """Largest power of two, of 4 to 64, that divides the row's 16-column chunks."""
    l = 2
    while l < 6 and (cols // 16) % (2 << l) == 0:
        l += 1
    return l


@pytest.mark.parametrize("cols", [64, 192, 320, 448, 768, 832, 1088, 1344, 1536, 2304, 2944, 6016, 11008])
def test_row_groups(cols):
    """Rows that keep three waves on each of the 1024 SIMDs leave no lane idle (a wider group then
    only adds work); a few rows spread over enough lanes to finish in a few steps."""
    d, chunks = default_group(cols), cols // 16
    for batch in (1, 160):
        for rows in (3 * 1024 * 64 >> d, 100000, 300000):
            rows = -(-max(rows, 3 * 1024 * 64 >> d) // batch)
            assert H.debug_row_grid(rows, 0, cols, batch=batch)[0][1] == d, (rows, batch)
    for rows in (1, 64, 300):
        l = H.debug_row_grid(rows, 0, cols)[0][1]
        assert l >= d and (chunks - 1 >> l) + 1 <= 3, (rows, l)
