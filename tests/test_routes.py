"""The rules that choose kernels and splits, asked on the host (no GPU needed)."""
import pytest


@pytest.fixture(scope="module")
def K():
    import paper_2602_08387_amd as k
    return k


T128X256, T128, T64, PERSISTENT = 0, 1, 2, 3


@pytest.mark.parametrize("cus", [256, 128, 64, 32])
def test_the_choice_of_a_product_goes_by_the_compute_units_there_are(K, cus):
    """One round of 256 x 256 tiles, and one tile more, on a whole device and on partitions of it."""
    one_round = K.gemm_route(0, 0, [256 * cus], [256], [4096], compute_units=cus)
    assert one_round == (PERSISTENT, -1, 256 * cus)
    first, second, rows = K.gemm_route(0, 0, [256 * (cus + 1)], [256], [4096], compute_units=cus)
    assert (first, rows) == (PERSISTENT, 256 * cus) and second in (T128, T64)
    # the same product on a device of another size: not a round
    assert K.gemm_route(0, 0, [256 * cus // 4], [256], [4096], compute_units=cus)[0] != PERSISTENT


def test_key_blocks_are_split_for_the_compute_units_there_are(K):
    shape = (2, 2944, 16, 4, 64)
    assert K.attention_backward_pieces(*shape, compute_units=256) > 1
    assert K.attention_backward_pieces(*shape, compute_units=32) == 1
    assert K.attention_backward_pieces(1, 100, 4, 4, 64) == 0 and K.attention_backward_pieces(1, 128, 4, 3, 64) == 0


def test_route_query_rejects_what_no_call_runs(K):
    for bad in ((3, 0, [64], [64], [64]), (0, 5, [64], [64], [64]), (2, 1, [64], [64], [64]), (1, 3, [64], [64], [64]),
                (0, 3, [64], [64], [64]), (0, 0, [64, 64], [64, 64], [64, 64]), (0, 0, [0], [64], [64]), (0, 0, [64], [64], [65])):
        with pytest.raises(K.DLayerError):
            K.gemm_route(*bad)
