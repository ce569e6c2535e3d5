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


@pytest.mark.parametrize("T,Kd,N", [(128, 3392, 3136), (192, 960, 8896), (192, 11136, 832), (320, 2624, 3392)])
def test_weight_gradients_over_few_tokens_take_a_smaller_tile(K, T, Kd, N):
    """Up to a round of 256 x 256 tiles that are all fill and drain: slower than any other tile (most where dW accumulates)."""
    assert K.gemm_route(2, 0, [N], [Kd], [T], compute_units=256)[0] in (T128, T128X256, T64)


def test_full_tiles_over_few_tokens(K):
    """A workgroup's further tiles cost less than its first, and a product of one K-step less than others: full 256 x 256 tiles from
    a round of them on, and smaller tiles for half a round."""
    for T in (64, 128, 192, 256, 512):
        assert K.gemm_route(2, 0, [14336], [4096], [T], compute_units=256)[0] == PERSISTENT
    assert K.gemm_route(2, 0, [4096], [4096], [64], compute_units=256) == (PERSISTENT, -1, 4096)
    assert K.gemm_route(2, 0, [2048], [4096], [64], compute_units=256)[0] != PERSISTENT


@pytest.mark.parametrize("T,N,Kd", [(64, 4160, 5120), (128, 1344, 9216), (192, 3584, 10304), (256, 4160, 13568), (512, 5440, 1792)])
def test_weight_gradients_over_few_tokens_that_accumulate(K, T, N, Kd):
    """The full tile waits for each part of the old value: another tile, though without accumulation the full one is faster."""
    assert K.gemm_route(2, 0, [N], [Kd], [T], compute_units=256)[0] == PERSISTENT
    assert K.gemm_route(2, 5, [N], [Kd], [T], compute_units=256)[0] != PERSISTENT
    assert K.gemm_route(2, 5, [N], [Kd], [2048], compute_units=256) == K.gemm_route(2, 0, [N], [Kd], [2048], compute_units=256)


def test_key_blocks_are_split_for_the_compute_units_there_are(K):
    shape = (2, 2944, 16, 4, 64)
    assert K.attention_backward_pieces(*shape, compute_units=256) > 1
    assert K.attention_backward_pieces(*shape, compute_units=32) == 1
    assert K.attention_backward_pieces(1, 100, 4, 4, 64) == 0 and K.attention_backward_pieces(1, 128, 4, 3, 64) == 0


def test_route_query_rejects_what_no_call_runs(K):
    for bad in ((3, 0, [64], [64], [64]), (0, 5, [64], [64], [64]), (1, 5, [64], [64], [64]), (2, 6, [64], [64], [64]), (2, 1, [64], [64], [64]), (1, 3, [64], [64], [64]),
                (0, 3, [64], [64], [64]), (0, 0, [64, 64], [64, 64], [64, 64]), (0, 0, [0], [64], [64]), (0, 0, [64], [64], [65])):
        with pytest.raises(K.DLayerError):
            K.gemm_route(*bad)


def test_the_shapes_of_the_gpu_tests_reach_the_paths_they_name(K):
    """The constants of the choice were fitted and may be fitted again: the shapes then have to follow."""
    from tests import test_gpu_shapes as shapes
    for (T, Kd, N), _, route in shapes.LINEAR:
        assert K.gemm_route(0, 0, [T], [N], [Kd], compute_units=256)[:2] == route, ("linear", T, Kd, N)
    for T, products, route in shapes.WEIGHT_GRADIENTS:
        assert K.gemm_route(2, 0, [n for n, _ in products], [k for _, k in products], [T] * len(products),
                            compute_units=256)[:2] == route, ("weight gradients", T, products)
    for T, products, route in shapes.OLD_VALUES:
        assert K.gemm_route(2, 5, [n for n, _ in products], [k for _, k in products], [T] * len(products),
                            compute_units=256)[:2] == route, ("accumulation", T, products)
    for (T, Kd, F), route in shapes.GATED_PAIRS:
        assert K.gemm_route(0, 1, [T], [F], [Kd], compute_units=256)[:2] == route, ("gated pair", T, Kd, F)
    for (T, D, F), stored, route in shapes.ACTIVATION_GRADIENTS:
        assert K.gemm_route(1 if stored else 0, 2, [T], [F], [D], compute_units=256)[:2] == route, ("activation gradient", T, D, F)
    for rows, Kd, N, tiles in shapes.INPUT_GRADIENTS:
        for T, tile in zip(rows, tiles):
            stored = T <= 4096 and T * Kd <= 4096 * 2048
            assert K.gemm_route(1 if stored else 0, 0, [T], [Kd], [N], compute_units=256)[:2] == (tile, -1), ("input gradient", T, Kd, N)
    assert {t for *_, tiles in shapes.INPUT_GRADIENTS for t in tiles} == {T64, T128, T128X256, PERSISTENT}
    for (B, S, D, Hq, Hkv, dh, layout), route in shapes.ROTARY:
        assert K.gemm_route(0, 3 + layout, [B * S] * 3, [Hq * dh, Hkv * dh, Hkv * dh], [D] * 3, head_dim=dh,
                            compute_units=256)[:2] == route, ("rotary", B, S, D, Hq, Hkv, dh, layout)
    for shape, pieces in shapes.SPLIT_ATTENTION + shapes.IN_PLACE_ATTENTION:
        assert K.attention_backward_pieces(*shape, compute_units=256) == pieces, ("attention", shape)
    # between them every epilogue runs on every tile, alone and behind a cut
    for rows, second in ((shapes.LINEAR, {T64, T128, T128X256}), (shapes.WEIGHT_GRADIENTS, {T64, T128}), (shapes.GATED_PAIRS, {T64, T128}),
                         (shapes.ACTIVATION_GRADIENTS, {T64, T128}), (shapes.ROTARY, {T128})):
        routes = [r[-1] for r in rows]
        assert {a for a, b in routes if b == -1} == {T64, T128, T128X256, PERSISTENT}
        assert {b for a, b in routes if b != -1} == second and all(a == PERSISTENT for a, b in routes if b != -1)
