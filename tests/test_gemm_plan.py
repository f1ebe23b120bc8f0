"""The GEMM's choice of tile and K split (host only): what the callers that size buffers from it
rely on, and the choices whose alternatives were measured much slower."""
import pytest

from paper_2505_05286_amd import hxf


@pytest.mark.parametrize("N,K,rows", [(4096, 14336, (176, 192, 208, 240, 251, 255, 513, 600, 704, 768, 900, 1024)),
                                      (5120, 27648, (176, 192, 513, 600, 704, 768, 900))])
def test_down_projections_above_128_rows_take_128_columns(N, K, rows):
    """A few thousand columns and long K: 256-column workgroups leave most of the chip idle
    (513 rows of 4096 x 14336: 141 us against 92)."""
    for M in rows:
        tm, nw, wv = hxf.op_gemm_plan(M, N, K, hxf.EPI_RESID)[:3]
        assert 16 * nw * wv == 128, (M, tm, nw, wv)


@pytest.mark.parametrize("N", [256, 688, 2048, 4096, 5120, 7168, 10240, 16383])
def test_partials_are_largest_at_the_last_rows_of_a_row_tile(N):
    """Buffers for every row count are sized at the multiples of 16 and the rows before them alone;
    above 512 rows K is whole."""
    for K in (512, 2048, 4096, 8192, 11008, 14336, 28672):
        for M16 in range(16, 513, 16):
            full = max(hxf.op_gemm_workspace_bytes(M, N, K) for M in (M16 - 1, M16))
            assert all(hxf.op_gemm_workspace_bytes(M, N, K) <= full for M in range(M16 - 15, M16 - 1))
        assert hxf.op_gemm_workspace_bytes(513, N, K) == hxf.op_gemm_workspace_bytes(2080, N, K) == 0


@pytest.mark.parametrize("N,last", [(65664, 64), (66048, 64), (80000, 64), (98304, 64), (140000, 32), (152064, 32),
                                    (200064, 32), (65536, 0), (98432, 0), (128256, 0), (256000, 0)])
def test_wide_outputs_take_128_columns_where_256_leave_the_cus_uneven(N, last):
    """Up to `last` rows: a quarter less for the fullest CU pays up to 64 rows, an eighth up to 32."""
    for K in (2304, 8192):
        for M in (1, 16, 32, 33, 40, 64, 65, 128):
            assert hxf.op_gemm_plan(M, N, K, hxf.EPI_F32)[1] == (2 if M <= last else 4), M


@pytest.mark.parametrize("N,K,pieces", [(6144, 4096, (4, 4, 4, 4)), (5120, 5120, (5, 5, 5, 5)), (4096, 4096, (8, 8, 4, 4)),
                                        (4096, 14336, (8, 8, 8, 8)), (7168, 5120, (4, 4, 4, 4)),
                                        (2048, 8192, (8, 8, 8, 8)), (256, 688, (1, 1, 1, 1))])
def test_few_rows_cut_k_only_where_a_piece_saves_more_than_its_partials(N, K, pieces):
    for M, want in zip((1, 17, 64, 128), pieces):
        *_, s, k = hxf.op_gemm_plan(M, N, K, hxf.EPI_BF16)
        assert s == want and k % 64 == 0 and (s - 1) * k < K <= s * k, (M, s, k)


def test_the_allocation_free_call_serves_what_it_served():
    """Down projections whose partials the allocation-free entry point took, and one it refuses."""
    limit = hxf.GEMM_NOALLOC_MAX_BYTES
    assert all(hxf.op_gemm_workspace_bytes(M, 4096, 4096) <= limit for M in range(1, 513))
    assert all(hxf.op_gemm_workspace_bytes(M, N, K) <= limit for M in range(1, 129) for N, K in ((4096, 14336), (8192, 28672)))
    assert hxf.op_gemm_workspace_bytes(256, 4096, 14336) > limit


@pytest.mark.parametrize("M,N,K,pieces", [(208, 5120, 27648, 6), (251, 5120, 27648, 6), (256, 4096, 14336, 7),
                                          (144, 8192, 28672, 8), (256, 10240, 8192, 3)])
def test_plans_beyond_the_allocation_free_array_take_the_pieces_that_measured_best(M, N, K, pieces):
    """Within 4% of the best split of the sweep (251 x 5120 x 27648: six pieces 93 us, five 100)."""
    assert hxf.op_gemm_plan(M, N, K, hxf.EPI_RESID)[4] == pieces
    assert hxf.op_gemm_workspace_bytes(M, N, K) > hxf.GEMM_NOALLOC_MAX_BYTES
