"""GPU parity at the sizes where a rule on sizes changes the kernel or the split of the work: edges of tiles,
remainders, the smallest and largest shapes of a branch.  Everything through the C ABI, against the fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import decoder_layer as odl
from synth import inputs as si
from tests.parity import dev_bf16, dev_from_f64, host_f64
from tests.test_gpu_layer import GpuLayer, _check_layer, _oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def K():
    import paper_2602_08387_amd as k
    return k


def _rand_bits(rng, shape, std=1.0):
    return si.f32_to_bf16_bits((rng.standard_normal(shape) * std).astype(np.float32))


def _norm_err(got, ref):
    d = host_f64(got).ravel() - np.asarray(ref, np.float64).ravel()
    return float(np.linalg.norm(d) / np.linalg.norm(ref))


def _poisoned(nbytes):
    return torch.full((max(int(nbytes), 256),), 0xFF, dtype=torch.uint8, device="cuda")


# ------------------------------------------------------------------ dK/dV pass with several workgroups per key block
# (batch, seq, query heads, KV heads, head width), pieces of a key block
SPLIT_ATTENTION = [
    ((1, 128, 4, 1, 32), 8),      # one key block of sixteen tiles
    ((1, 640, 6, 2, 64), 8),      # a group of three heads
    ((1, 1792, 1, 1, 64), 8),     # one head: the last key block has four tiles for eight pieces
    ((2, 384, 8, 1, 128), 8),     # a group as wide as the number of pieces
    ((2, 1408, 16, 4, 64), 5),    # pieces that neither divide the group nor are a multiple of it
    ((1, 2048, 3, 1, 128), 8),    # with the dS hand-over
]


@pytest.mark.parametrize("shape,pieces", SPLIT_ATTENTION)
def test_attention_backward_with_split_key_blocks(K, shape, pieces):
    B, S, Hq, Hkv, dh = shape
    assert K.attention_backward_pieces(*shape) == pieces
    rng = np.random.default_rng(S + dh + Hq)
    qb, kb = _rand_bits(rng, (B, S, Hq, dh)), _rand_bits(rng, (B, S, Hkv, dh))
    vb, dob = _rand_bits(rng, (B, S, Hkv, dh)), _rand_bits(rng, (B, S, Hq, dh))
    q, k, v, do = map(si.bf16_bits_to_f64, (qb, kb, vb, dob))
    qd, kd, vd, dod = map(dev_bf16, (qb, kb, vb, dob))
    o, lse = torch.full_like(qd, float("nan")), torch.empty(B, Hq, S, dtype=torch.float32, device="cuda")
    K.attention_forward(qd, kd, vd, B, S, Hq, Hkv, dh, o, lse)
    refs = odl.attention_bwd(q, k, v, do)
    od = dev_from_f64(odl.attention_fwd(q, k, v)[0])
    runs = []
    for _ in range(2):
        grads = [torch.full_like(t, float("nan")) for t in (qd, kd, vd)]
        K.attention_backward(qd, kd, vd, od, dod, lse, B, S, Hq, Hkv, dh, *grads,
                             _poisoned(K.attention_backward_workspace_bytes(B, S, Hq, Hkv, dh)))
        runs.append(grads)
    # In the 2-norm: independent bf16 roundings of o (in delta), of P, of dS and of the result, each at most 2^-8 of its
    # operand, add up to 2 x 2^-8 = 7.8e-3.  (Element by element the early rows dominate, whatever the split: dq, which the split
    # does not touch, has elements 7.5e-2 of its rms off at S = 384.)
    for name, got, again, ref in zip(("dq", "dk", "dv"), runs[0], runs[1], refs):
        assert _norm_err(got, ref) <= 7.8e-3, name
        assert torch.equal(got.view(torch.int16), again.view(torch.int16)), f"{name} is not reproducible"


IN_PLACE_ATTENTION = [
    ((8, 512, 12, 12, 64), 1),    # one workgroup per key block; dQ in the same launch where dq is a buffer of its own
    ((1, 640, 6, 2, 64), 8),
    ((1, 256, 4, 2, 32), 8),
    ((1, 640, 3, 1, 128), 8),
    ((1, 2048, 2, 1, 128), 8),    # with the dS hand-over: two launches anyway
]


@pytest.mark.parametrize("shape,pieces", IN_PLACE_ATTENTION)
def test_attention_backward_with_dq_in_place(K, shape, pieces):
    """Every key block reads q and dO, so dq may only replace one of them once the dK/dV pass is over."""
    B, S, Hq, Hkv, dh = shape
    assert K.attention_backward_pieces(*shape) == pieces
    rng = np.random.default_rng(S + dh)
    q, do = (dev_bf16(_rand_bits(rng, (B, S, Hq, dh))) for _ in range(2))
    k, v = (dev_bf16(_rand_bits(rng, (B, S, Hkv, dh))) for _ in range(2))
    o, lse = torch.empty_like(q), torch.empty(B, Hq, S, dtype=torch.float32, device="cuda")
    K.attention_forward(q, k, v, B, S, Hq, Hkv, dh, o, lse)

    def backward(q, do, dq):
        dk, dv = torch.full_like(k, float("nan")), torch.full_like(v, float("nan"))
        K.attention_backward(q, k, v, o, do, lse, B, S, Hq, Hkv, dh, dq, dk, dv,
                             _poisoned(K.attention_backward_workspace_bytes(B, S, Hq, Hkv, dh)))
        return dq, dk, dv

    want = backward(q, do, torch.full_like(q, float("nan")))
    over_q, over_do = q.clone(), do.clone()
    for what, got in (("q", backward(over_q, do, over_q)), ("dO", backward(q, over_do, over_do))):
        for name, g, w in zip(("dq", "dk", "dv"), got, want):
            assert torch.equal(g.view(torch.int16), w.view(torch.int16)), f"{name} with dq over {what}"


@pytest.mark.parametrize("override", [
    {"seq": 640, "d_model": 192, "n_q_heads": 6, "n_kv_heads": 2, "head_dim": 64, "d_ff": 320, "rope_layout": 1},
    {"seq": 512, "d_model": 256, "n_q_heads": 4, "n_kv_heads": 1, "head_dim": 128, "d_ff": 320},
    {"seq": 512, "d_model": 256, "n_q_heads": 4, "n_kv_heads": 1, "head_dim": 128, "d_ff": 320, "rope_layout": 1},
])
def test_layer_with_split_key_blocks(K, override):
    """The rotation of dK moves from the dK/dV pass into the kernel that adds the pieces."""
    cfg = si.CONFIGS["tiny"].with_(**override)
    inp = si.make_layer_inputs(cfg, seed=1)
    f, r = _oracle(cfg, inp)
    g = GpuLayer(K, cfg, inp)
    g.forward()
    g.backward()
    torch.cuda.synchronize()
    _check_layer(g, f, r, "split")


# ------------------------------------------------------------------ products on every tile size and on two launches
# rounding the fp32 sum to bf16 is off by 2^-8 of an element at most (1.7e-3 in the 2-norm of many); 5 % more for the
# order of the fp32 sums
ONE_ROUNDING = 1.05 * 2.0 ** -8
# Tiles as gemm_route names them.  Every shape below states the tile of its launch, or of its two: full rounds of 256 x 256
# tiles and a smaller tile for the rows behind them.
T128X256, T128, T64, PERSISTENT = 0, 1, 2, 3


def _same_bits(a, b, what):
    assert torch.equal(a.contiguous().view(torch.int16), b.contiguous().view(torch.int16)), what


LINEAR = [
    ((1, 64, 8), False, (T64, -1)),                   # one row, one K-step, one vector of columns
    ((65, 192, 136), True, (T64, -1)),                # remainders on every side, fewer K-steps than ring stages
    ((1000, 1024, 1024), True, (T64, -1)),
    ((1920, 576, 1160), True, (T128, -1)),            # ragged columns
    ((8192, 320, 768), False, (T128X256, -1)),
    ((16640, 128, 1096), False, (PERSISTENT, -1)),    # more than one round, in one launch
    ((4160, 448, 4288), True, (PERSISTENT, T64)),     # cut at row 3840: the rows behind it lie in two groups of 2048
    ((16640, 512, 1096), True, (PERSISTENT, T128)),
    ((10560, 576, 1856), False, (PERSISTENT, T128X256)),
]


@pytest.mark.parametrize("shape,res,route", LINEAR)
def test_linear_forward_on_every_tile_size(K, shape, res, route):
    T, Kd, N = shape
    assert K.gemm_route(0, 0, [T], [N], [Kd])[:2] == route
    rng = np.random.default_rng(T + N)
    xb, wb, rb = _rand_bits(rng, (T, Kd)), _rand_bits(rng, (N, Kd), 0.05), _rand_bits(rng, (T, N))
    x, w, r = map(si.bf16_bits_to_f64, (xb, wb, rb))
    xd, wd, rd = map(dev_bf16, (xb, wb, rb))
    y = torch.full((T, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    K.linear_forward(xd, wd, rd if res else None, T, Kd, N, y)
    assert _norm_err(y, x @ w.T + (r if res else 0.0)) <= ONE_ROUNDING

    def part(rows, cols):
        out = torch.full((rows, cols), float("nan"), dtype=torch.bfloat16, device="cuda")
        K.linear_forward(xd[:rows], wd[:cols], rd[:rows, :cols].contiguous() if res else None, rows, Kd, cols, out)
        return out

    # a product has the same bits whatever kernel its size selects: fewer rows, and all of them with fewer columns
    for rows in (max(T // 2, 1), 1):
        _same_bits(part(rows, N), y[:rows], f"{rows} rows")
    for cols in (72, 136, 264):
        if cols < N:
            assert K.gemm_route(0, 0, [T], [cols], [Kd])[1] == -1
            _same_bits(part(T, cols), y[:, :cols], f"{cols} columns")


# rows, contraction, columns, gated pair, tile: one and two K-steps, all of them loaded at the start; ragged rows and columns
FEW_STEPS = [
    ((65, 128, 136), False, T64),
    ((1600, 64, 1160), False, T64),
    ((2000, 128, 1160), False, T128),
    ((2000, 64, 1864), False, T128),
    ((1088, 128, 6792), False, T128X256),
    ((1000, 64, 7000), False, T128X256),
    ((65, 128, 72), True, T64),
    ((900, 64, 1800), True, T128),
    ((600, 128, 3400), True, T128X256),
]


@pytest.mark.parametrize("shape,gated,tile", FEW_STEPS)
def test_one_and_two_k_steps_on_small_tiles(K, shape, gated, tile):
    """The same bits as the contraction with 128 zeros behind it, which runs with waves that only load (and within 2048 rows adds
    the same terms in the same order)."""
    T, Kd, N = shape
    for k in (Kd, Kd + 128):
        assert K.gemm_route(0, int(gated), [T], [N], [k], compute_units=256) == (tile, -1, T)
    rng = np.random.default_rng(T)
    xb, wb, vb, rb = _rand_bits(rng, (T, Kd)), _rand_bits(rng, (N, Kd), 0.1), _rand_bits(rng, (N, Kd), 0.1), _rand_bits(rng, (T, N))
    x, w, v, r = map(si.bf16_bits_to_f32, (xb, wb, vb, rb))
    xd, wd, vd, rd = map(dev_bf16, (xb, wb, vb, rb))

    def run(res, pad):
        a, b, c = (torch.nn.functional.pad(t, (0, pad)) for t in (xd, wd, vd))
        out = [torch.full((T, N), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(3 if gated else 1)]
        if gated:
            K.linear_swiglu_forward(a, b, c, T, Kd + pad, N, *out)
        else:
            K.linear_forward(a, b, rd if res else None, T, Kd + pad, N, *out)
        return out

    for res in (False,) if gated else (False, True):
        got, padded = run(res, 0), run(res, 128)
        g, u = x @ w.T, x @ v.T
        for i, ref in enumerate((g, u, odl.swiglu_fwd(g, u)) if gated else (g + (r if res else 0.0),)):
            assert _norm_err(got[i], ref) <= ONE_ROUNDING, i
            _same_bits(got[i], padded[i], f"output {i}, residual {res}")


def test_layer_with_two_segments_of_one_k_step(K):
    """d_ff 64: the fused input gradient of gate and up is two segments of one K-step each."""
    cfg = si.CONFIGS["tiny"].with_(batch=1, seq=640, d_model=2112, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ff=64)
    assert K.gemm_route(0, 0, [640], [2112], [128], compute_units=256)[0] != PERSISTENT
    inp = si.make_layer_inputs(cfg, seed=4)
    f, r = _oracle(cfg, inp)
    g = GpuLayer(K, cfg, inp)
    g.forward()
    g.backward()
    torch.cuda.synchronize()
    _check_layer(g, f, r, "two segments of one K-step")


@pytest.mark.parametrize("shape,res", [((4096, 4096), False), ((4160, 4288), True), ((20520, 2056), True)])
def test_linear_forward_over_one_k_step_on_full_tiles(K, shape, res):
    """K = 64 on the persistent kernel: one tile to a workgroup, two, and three with ragged rows and columns."""
    T, N = shape
    assert K.gemm_route(0, 0, [T], [N], [64]) == (PERSISTENT, -1, T)
    rng = np.random.default_rng(T)
    xb, wb, rb = _rand_bits(rng, (T, 64)), _rand_bits(rng, (N, 64), 0.1), _rand_bits(rng, (T, N))
    xd, wd, rd = map(dev_bf16, (xb, wb, rb))
    y = torch.full((T, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    K.linear_forward(xd, wd, rd if res else None, T, 64, N, y)
    x, w, r = (si.bf16_bits_to_f32(b) for b in (xb, wb, rb))
    assert _norm_err(y, x @ w.T + (r if res else 0.0)) <= ONE_ROUNDING
    for c0 in (0, N - 136):   # the same bits on another kernel, in the first and the last columns
        assert K.gemm_route(0, 0, [T], [136], [64])[0] != PERSISTENT
        part = torch.full((T, 136), float("nan"), dtype=torch.bfloat16, device="cuda")
        K.linear_forward(xd, wd[c0:c0 + 136].contiguous(), rd[:, c0:c0 + 136].contiguous() if res else None, T, 64, 136, part)
        _same_bits(part, y[:, c0:c0 + 136], f"columns from {c0}")


WEIGHT_GRADIENTS = [
    (64, [(64, 64)], (T64, -1)),                                                  # one tile, one K-step
    (320, [(64, 192), (320, 64), (128, 128)], (T64, -1)),
    (64, [(512, 3072), (960, 576)], (T128, -1)),
    (1024, [(1152, 1152), (384, 1152), (1152, 3136)], (T128X256, -1)),
    (256, [(4160, 832), (4608, 1600), (5120, 192)], (PERSISTENT, -1)),            # less than a round
    (192, [(4032, 4224), (576, 448)], (PERSISTENT, T64)),                         # the cut falls into the first product
    (384, [(1792, 576), (3328, 3136), (4480, 1344)], (PERSISTENT, T128)),         # into the last: two products lie before it
]


@pytest.mark.parametrize("T,shapes,route", WEIGHT_GRADIENTS)
def test_weight_gradients_on_every_tile_size(K, T, shapes, route):
    assert K.gemm_route(2, 0, [n for n, _ in shapes], [k for _, k in shapes], [T] * len(shapes))[:2] == route
    rng = np.random.default_rng(T + len(shapes))
    dyb, xb = [_rand_bits(rng, (T, n)) for n, _ in shapes], [_rand_bits(rng, (T, k)) for _, k in shapes]
    dyd, xd = [dev_bf16(b) for b in dyb], [dev_bf16(b) for b in xb]
    dws = [torch.full((n, k), float("nan"), dtype=torch.bfloat16, device="cuda") for n, k in shapes]
    K.linear_wgrad_group(dyd, xd, [n for n, _ in shapes], [k for _, k in shapes], T, dws, 0)
    for i, (n, k) in enumerate(shapes):
        assert _norm_err(dws[i], si.bf16_bits_to_f64(dyb[i]).T @ si.bf16_bits_to_f64(xb[i])) <= ONE_ROUNDING, i
        one = torch.empty_like(dws[i])
        K.linear_backward(xd[i], xd[i], dyd[i], T, k, n, None, one, 0, None)
        _same_bits(one, dws[i], f"grouped dw[{i}] differs from the single launch")
        narrow = torch.empty(n, 64, dtype=torch.bfloat16, device="cuda")
        assert K.gemm_route(2, 0, [n], [64], [T])[1] == -1
        K.linear_backward(xd[i][:, :64].contiguous(), xd[i], dyd[i], T, 64, n, None, narrow, 0, None)
        _same_bits(narrow, dws[i][:, :64], f"dw[{i}] of 64 columns")


ONE_STEP_GRADIENTS = [
    [(4096, 4096)],                                   # one tile to a workgroup
    [(7232, 4160)],                                   # two, ragged in both directions
    [(8192, 2112), (4160, 1088), (8256, 448)],        # a group of nearly two, its products ragged
]


@pytest.mark.parametrize("accumulate", [0, 1])
@pytest.mark.parametrize("shapes", ONE_STEP_GRADIENTS)
def test_weight_gradients_over_one_k_step_on_full_tiles(K, shapes, accumulate):
    """64 tokens on the persistent kernels, and, accumulating, on the tiles that those take."""
    Ns, Ks = [n for n, _ in shapes], [k for _, k in shapes]
    first, second, _ = K.gemm_route(2, 5 if accumulate else 0, Ns, Ks, [64] * len(shapes))
    assert (first != PERSISTENT if accumulate else first == PERSISTENT) and second == -1
    rng = np.random.default_rng(len(shapes))
    dyb, xb, wb = ([_rand_bits(rng, s) for s in sizes] for sizes in ([(64, n) for n in Ns], [(64, k) for k in Ks], shapes))
    dyd, xd, dws = ([dev_bf16(b) for b in bits] for bits in (dyb, xb, wb))
    first = [w.clone() for w in dws]
    K.linear_wgrad_group(dyd, xd, Ns, Ks, 64, dws, accumulate)
    for i, (n, k) in enumerate(shapes):
        dy, x, w = (si.bf16_bits_to_f32(b[i]) for b in (dyb, xb, wb))
        assert _norm_err(dws[i], dy.T @ x + (w if accumulate else 0.0)) <= ONE_ROUNDING, i
        for c0 in (0, k - 64):   # the same bits on a smaller tile, in the first and the last columns
            assert K.gemm_route(2, 0, [n], [64], [64])[0] != PERSISTENT
            part = first[i][:, c0:c0 + 64].contiguous()
            K.linear_backward(xd[i][:, c0:c0 + 64].contiguous(), xd[i], dyd[i], 64, 64, n, None, part, accumulate, None)
            _same_bits(part, dws[i][:, c0:c0 + 64], f"dw[{i}], columns from {c0}")


# tokens, products that accumulate, route: either side of the line at 512 tokens
OLD_VALUES = [
    (512, [(5440, 1792), (448, 192)], (T128, -1)),
    (576, [(5440, 1792), (448, 192)], (PERSISTENT, -1)),
    (576, [(4160, 4288), (448, 192)], (PERSISTENT, T64)),
]


@pytest.mark.parametrize("T,shapes,route", OLD_VALUES)
def test_weight_gradients_that_accumulate(K, T, shapes, route):
    """One rounding of product and old value, and the same bits whatever kernel."""
    Ns, Ks = [n for n, _ in shapes], [k for _, k in shapes]
    assert K.gemm_route(2, 5, Ns, Ks, [T] * len(shapes))[:2] == route
    rng = np.random.default_rng(T)
    dyb, xb, wb = ([_rand_bits(rng, s) for s in sizes] for sizes in ([(T, n) for n in Ns], [(T, k) for k in Ks], shapes))
    dyd, xd, dws = ([dev_bf16(b) for b in bits] for bits in (dyb, xb, wb))
    first = [w.clone() for w in dws]
    K.linear_wgrad_group(dyd, xd, Ns, Ks, T, dws, 1)
    for i, (n, k) in enumerate(shapes):
        dy, x, w = (si.bf16_bits_to_f32(b[i]) for b in (dyb, xb, wb))
        assert _norm_err(dws[i], dy.T @ x + w) <= ONE_ROUNDING, i
        part = first[i][:, k - 64:].contiguous()
        K.linear_backward(xd[i][:, k - 64:].contiguous(), xd[i], dyd[i], T, 64, n, None, part, 1, None)
        _same_bits(part, dws[i][:, k - 64:], f"last columns of dw[{i}]")


GATED_PAIRS = [
    ((64, 64, 64), (T64, -1)),
    ((200, 192, 104), (T64, -1)),
    ((1920, 1152, 200), (T64, -1)),
    ((1000, 64, 1608), (T128, -1)),
    ((1920, 1152, 1096), (T128X256, -1)),
    ((4160, 192, 2176), (PERSISTENT, -1)),
    ((4160, 64, 4288), (PERSISTENT, -1)),             # one K-step
    ((4160, 1024, 2176), (PERSISTENT, T64)),
    ((2048, 512, 4224), (PERSISTENT, T128)),
]


@pytest.mark.parametrize("shape,route", GATED_PAIRS)
def test_gated_pair_on_every_tile_size(K, shape, route):
    T, Kd, F = shape
    assert K.gemm_route(0, 1, [T], [F], [Kd])[:2] == route
    rng = np.random.default_rng(T + F)
    xb, wgb, wub = _rand_bits(rng, (T, Kd)), _rand_bits(rng, (F, Kd), 0.1), _rand_bits(rng, (F, Kd), 0.1)
    x, wg, wu = map(si.bf16_bits_to_f64, (xb, wgb, wub))
    xd, wgd, wud = map(dev_bf16, (xb, wgb, wub))
    out = [torch.full((T, F), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    K.linear_swiglu_forward(xd, wgd, wud, T, Kd, F, *out)
    g, u = x @ wg.T, x @ wu.T
    for name, got, ref in zip("gua", out, (g, u, odl.swiglu_fwd(g, u))):
        assert _norm_err(got, ref) <= ONE_ROUNDING, name
    narrow = [torch.full((T, 64), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    assert K.gemm_route(0, 1, [T], [64], [Kd])[1] == -1
    K.linear_swiglu_forward(xd, wgd[:64], wud[:64], T, Kd, 64, *narrow)
    for name, got, few in zip("gua", out, narrow):
        _same_bits(few, got[:, :64], f"{name} of 64 columns")


# tokens, width, d_ff; whether the weights are read as stored (up to 4096 tokens and 8M elements of da)
ACTIVATION_GRADIENTS = [
    ((64, 64, 64), True, (T64, -1)),
    ((192, 128, 320), True, (T64, -1)),
    ((1920, 192, 1152), True, (T128, -1)),
    ((3200, 512, 2496), True, (T128X256, -1)),
    ((4160, 512, 1152), False, (T128X256, -1)),
    ((4160, 64, 4288), False, (PERSISTENT, -1)),
    ((4160, 512, 4288), False, (PERSISTENT, T64)),
    ((7360, 256, 2368), False, (PERSISTENT, T128)),
]


@pytest.mark.parametrize("shape,stored,route", ACTIVATION_GRADIENTS)
def test_activation_gradient_on_every_tile_size(K, shape, stored, route):
    T, D, F = shape
    assert K.gemm_route(1 if stored else 0, 2, [T], [F], [D])[:2] == route
    rng = np.random.default_rng(T + F)
    dyb, wb, gb, ub = _rand_bits(rng, (T, D)), _rand_bits(rng, (D, F), 0.1), _rand_bits(rng, (T, F)), _rand_bits(rng, (T, F))
    dy, w, g, u = map(si.bf16_bits_to_f64, (dyb, wb, gb, ub))
    dyd, wd, gd, ud = map(dev_bf16, (dyb, wb, gb, ub))

    def backward(cols):
        dg, du = (torch.full((T, cols), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        K.linear_swiglu_backward(dyd, wd[:, :cols].contiguous(), gd[:, :cols].contiguous(), ud[:, :cols].contiguous(), T, D, cols, dg, du,
                                 _poisoned(K.linear_swiglu_backward_workspace_bytes(T, D, cols)))
        return dg, du

    got = backward(F)
    for name, d, ref in zip(("dg", "du"), got, odl.swiglu_bwd(g, u, dy @ w)):
        assert _norm_err(d, ref) <= ONE_ROUNDING, name
    assert K.gemm_route(1 if T <= 4096 else 0, 2, [T], [64], [D])[1] == -1
    for name, d, few in zip(("dg", "du"), got, backward(64)):
        _same_bits(few, d[:, :64], f"{name} of 64 columns")


INPUT_GRADIENTS = [
    ((64,), 64, 64, (T64,)),                                    # one tile, one K-step
    ((4160, 4096, 64), 320, 192, (T64, T64, T64)),              # the last rows that read the weights as stored, and the first that do not
    ((4032, 1984, 320), 2112, 448, (PERSISTENT, T64, T64)),     # the same for rows x columns
    ((1600, 576), 2624, 448, (T128X256, T64)),
    ((1920, 64), 1152, 3136, (T128, T64)),
]


@pytest.mark.parametrize("rows,Kd,N,tiles", INPUT_GRADIENTS)
def test_input_gradient_with_and_without_the_transposed_weights(K, rows, Kd, N, tiles):
    rng = np.random.default_rng(rows[0] + N)
    dyb, wb = _rand_bits(rng, (rows[0], N)), _rand_bits(rng, (N, Kd), 0.05)
    ref = si.bf16_bits_to_f64(dyb) @ si.bf16_bits_to_f64(wb)
    dyd, wd, first = dev_bf16(dyb), dev_bf16(wb), None
    for T, tile in zip(rows, tiles):
        assert K.gemm_route(1 if T <= 4096 and T * Kd <= 4096 * 2048 else 0, 0, [T], [Kd], [N])[:2] == (tile, -1)
        dx = torch.full((T, Kd), float("nan"), dtype=torch.bfloat16, device="cuda")
        K.linear_backward(dx, wd, dyd[:T], T, Kd, N, dx, None, 0, _poisoned(K.linear_backward_workspace_bytes(T, Kd, N)))
        assert _norm_err(dx, ref[:T]) <= ONE_ROUNDING, T
        first = dx if first is None else first
        assert torch.equal(dx.view(torch.int16), first[:T].view(torch.int16)), T


# batch, seq, width, query heads, KV heads, head width, d_ff; weights as stored; tile of the o projection's input gradient
STATISTICS = [
    ((1, 256, 128, 4, 2, 32, 192), True, T64),        # two heads per tile
    ((1, 256, 128, 2, 1, 64, 192), True, T64),
    ((1, 256, 128, 2, 1, 128, 192), True, T64),       # a head spans two tiles: statistics in a launch of their own
    ((3, 640, 192, 9, 3, 128, 320), False, T128),
    ((3, 640, 192, 18, 6, 64, 320), False, T128),
    ((8, 1024, 320, 6, 2, 128, 320), False, T128X256),
    ((8, 1024, 320, 24, 8, 32, 320), False, T128X256),
]


@pytest.mark.parametrize("shape,stored,tile", STATISTICS)
def test_layer_with_row_statistics_in_the_epilogue(K, shape, stored, tile):
    """The attention backward's row statistics come out of the product that makes dO, the norms' gain sums out of the weight
    gradients' launch."""
    B, S, D, Hq, Hkv, dh, F = shape
    T, QD = B * S, Hq * dh
    assert stored == (D * max(F, QD) <= 65536 and T <= 4096)
    assert K.gemm_route(1 if stored else 0, 0, [T], [QD], [D], compute_units=256)[:2] == (tile, -1)
    cfg = si.CONFIGS["tiny"].with_(batch=B, seq=S, d_model=D, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=dh, d_ff=F)
    inp = si.make_layer_inputs(cfg, seed=5)
    f, r = _oracle(cfg, inp)
    g = GpuLayer(K, cfg, inp)
    g.forward()
    g.backward()
    torch.cuda.synchronize()
    _check_layer(g, f, r, "statistics")


# query heads, KV heads, head width; batches whose o projection's input gradient runs on a tile kernel, and which
STATISTICS_BITS = [(32, 16, 32, ((16, T64), (32, T128), (48, T128X256))), (16, 8, 64, ((16, T64), (32, T128), (48, T128X256))),
                   (8, 4, 128, ((32, T128), (48, T128X256)))]


@pytest.mark.parametrize("Hq,Hkv,dh,fewer", STATISTICS_BITS)
def test_row_statistics_have_the_same_bits_in_the_epilogue_and_in_a_launch_of_their_own(K, Hq, Hkv, dh, fewer):
    """Layers of 128 batches take them from a launch of their own (the o projection's input gradient runs on the persistent kernel), of
    fewer from its epilogue.  Where dy is zero for the batches beyond those, everything else is the same bit for bit.  All
    tokens of a sequence are the same, so that dP - rowsum(dO * O), and with it dq and dk, is nothing but the order of sums."""
    S, D, F, many = 128, 192, 192, 128
    assert K.gemm_route(0, 0, [many * S], [Hq * dh], [D])[0] == PERSISTENT and D * Hq * dh > 65536
    cfg = si.CONFIGS["tiny"].with_(batch=many, seq=S, d_model=D, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=dh, d_ff=F)
    inp = si.make_layer_inputs(cfg, seed=11)
    inp["x"] = np.repeat(inp["x"][:, :1], S, axis=1)
    for batch, tile in fewer:
        assert K.gemm_route(0, 0, [batch * S], [Hq * dh], [D])[:2] == (tile, -1)
        assert K.attention_backward_pieces(batch, S, Hq, Hkv, dh) == K.attention_backward_pieces(many, S, Hq, Hkv, dh)
        dy = inp["dy"].copy()
        dy[batch:] = 0
        layers = [GpuLayer(K, cfg, dict(inp, dy=dy)), GpuLayer(K, cfg.with_(batch=batch), dict(inp, x=inp["x"][:batch], dy=dy[:batch]))]
        for g in layers:
            g.forward()
            g.backward()
        own, epilogue = layers
        rows = batch * S
        _same_bits(epilogue.dx.reshape(rows, D), own.dx.reshape(-1, D)[:rows], f"{batch} batches: dx")
        for n in si.WEIGHT_NAMES:
            if not n.startswith("g_"):   # the gains' partial sums go by the number of rows
                _same_bits(epilogue.dw[n], own.dw[n], f"{batch} batches: d{n}")


# batch, seq, width, query heads, KV heads, head width, d_ff; weights as stored; kernel of the gated gradient
REBUILT = [
    ((1, 128, 192, 2, 1, 64, 320), True, T64),         # a wave per row of the norm
    ((1, 256, 576, 2, 1, 64, 192), False, T64),
    ((5, 384, 1088, 1, 1, 64, 1216), False, T128),     # ragged tiles, two waves share a row's end
    ((8, 1024, 320, 2, 1, 128, 832), False, T128X256),
    ((1, 2176, 2112, 1, 1, 64, 64), False, T64),       # more rows than one per compute unit at a time
    ((1, 256, 2112, 1, 1, 64, 64), False, T64),        # two rows to a workgroup
    ((1, 128, 4160, 1, 1, 64, 64), False, T64),
    ((1, 128, 8256, 1, 1, 64, 64), False, T64),        # two vectors of a row per thread
    ((8, 2048, 128, 2, 1, 64, 1024), False, PERSISTENT),   # a in a launch of its own
]


@pytest.mark.parametrize("shape,stored,kernel", REBUILT)
def test_activations_rebuilt_in_passing(K, shape, stored, kernel):
    """recompute: the norms' backward writes h1 and h2 again (same bits), the gated gradient's epilogue a."""
    B, S, D, Hq, Hkv, dh, F = shape
    T = B * S
    assert stored == (D * max(F, Hq * dh) <= 65536 and T <= 4096)
    assert K.gemm_route(1 if stored else 0, 2, [T], [F], [D], compute_units=256)[0] == kernel
    cfg = si.CONFIGS["tiny"].with_(batch=B, seq=S, d_model=D, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=dh, d_ff=F)
    inp = si.make_layer_inputs(cfg, seed=7)
    f, r = _oracle(cfg, inp)
    a, b = GpuLayer(K, cfg, inp), GpuLayer(K, cfg.with_(recompute=3), inp)
    for g in (a, b):
        g.forward()
        g.backward()
    torch.cuda.synchronize()
    _check_layer(b, f, r, "rebuilt")
    for n, p, q in [("dx", a.dx, b.dx)] + [(n, a.dw[n], b.dw[n]) for n in si.WEIGHT_NAMES if n != "w_down"]:
        assert torch.equal(p.view(torch.int16), q.view(torch.int16)), f"{n} differs between keeping and rebuilding"


def test_layer_with_short_segments_on_full_tiles(K):
    """The fused input gradients on 256 x 256 tiles with segments of one and of three K-steps: walks that start in any segment
    (a row group of 2048 starts its eighth of the way further on), odd and even, over more than one round of tiles."""
    cfg = si.CONFIGS["tiny"].with_(batch=8, seq=2048, d_model=2112, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ff=192)
    for steps in (3 * 64, 2 * 192):
        assert K.gemm_route(0, 0, [16384], [2112], [steps], compute_units=256)[0] == PERSISTENT
    inp = si.make_layer_inputs(cfg, seed=3)
    f, r = _oracle(cfg, inp)
    g = GpuLayer(K, cfg, inp)
    g.forward()
    g.backward()
    torch.cuda.synchronize()
    _check_layer(g, f, r, "short segments")


# batch, seq, width, query heads, KV heads, head width, layout (0 split pairs, 1 adjacent)
ROTARY = [
    ((1, 128, 64, 2, 1, 64, 0), (T64, -1)),           # a head per tile
    ((1, 192, 64, 4, 2, 32, 0), (T64, -1)),           # two heads per tile
    ((3, 320, 128, 3, 1, 128, 1), (T64, -1)),         # adjacent pairs: a 128-wide head spans two 64-column tiles
    ((2, 384, 192, 4, 2, 128, 0), (T128, -1)),        # split pairs of 128-wide heads
    ((1, 1216, 64, 9, 9, 64, 1), (T128, -1)),
    ((5, 384, 192, 9, 9, 128, 0), (T128X256, -1)),
    ((3, 2816, 64, 12, 12, 64, 0), (PERSISTENT, -1)), # more than one round, in one launch
    ((5, 1024, 64, 31, 8, 128, 0), (PERSISTENT, -1)), # one K-step, weight tiles in partner order
    ((5, 1728, 256, 30, 2, 64, 0), (PERSISTENT, T128)),     # cut in q, in the middle of a sequence: positions go on across it
    ((5, 1664, 256, 15, 1, 128, 0), (PERSISTENT, T128)),    # the same, weight tiles of the full rounds in partner order
    ((5, 1664, 256, 15, 1, 128, 1), (PERSISTENT, T128)),
]


@pytest.mark.parametrize("shape,route", ROTARY)
def test_rotary_projections_on_every_tile_size(K, shape, route):
    B, S, D, Hq, Hkv, dh, layout = shape
    T, QD, KD = B * S, Hq * dh, Hkv * dh
    *tiles, first_rows = K.gemm_route(0, 3 + layout, [T] * 3, [QD, KD, KD], [D] * 3, head_dim=dh)
    assert tuple(tiles) == route and (route[1] == -1 or first_rows < T and first_rows % S)
    rng = np.random.default_rng(S + dh)
    hb, wqb, wkb, wvb = (_rand_bits(rng, s, std) for s, std in (((T, D), 1.0), ((QD, D), 0.1), ((KD, D), 0.1), ((KD, D), 0.1)))
    h, wq, wk, wv = map(si.bf16_bits_to_f64, (hb, wqb, wkb, wvb))
    hd, wqd, wkd, wvd = map(dev_bf16, (hb, wqb, wkb, wvb))
    phi = odl.rope_angles(S, dh, 1e4)
    refs = (odl.rope_rotate((h @ wq.T).reshape(B, S, Hq, dh), phi, layout=layout),
            odl.rope_rotate((h @ wk.T).reshape(B, S, Hkv, dh), phi, layout=layout), h @ wv.T)

    def project(heads, kv_heads):
        out = [torch.full((T, n * dh), float("nan"), dtype=torch.bfloat16, device="cuda") for n in (heads, kv_heads, kv_heads)]
        K.qkv_rope_forward(hd, wqd[:heads * dh], wkd[:kv_heads * dh], wvd[:kv_heads * dh], B, S, D, heads, kv_heads, dh, 1e4, layout, *out,
                           _poisoned(K.qkv_rope_workspace_bytes(S, dh)))
        return out

    out = project(Hq, Hkv)
    for name, got, ref in zip("qkv", out, refs):
        assert _norm_err(got, ref) <= ONE_ROUNDING, name
    assert K.gemm_route(0, 3 + layout, [T] * 3, [dh] * 3, [D] * 3, head_dim=dh)[1] == -1
    for name, got, one in zip("qkv", out, project(1, 1)):
        _same_bits(one, got[:, :dh], f"{name} of one head")


# ------------------------------------------------------------------ RMSNorm backward: threads per row, rows per workgroup
@pytest.mark.parametrize("T,D", [(1, 8), (3, 512), (2050, 520), (1025, 1024), (5000, 1032), (77, 2056), (1030, 4096), (9, 8192), (515, 8200), (3, 16384),
                                 (2048, 2056), (2049, 4096)])   # the last and the first of the two workgroup sizes
def test_rmsnorm_backward_on_every_row_split(K, T, D):
    rng = np.random.default_rng(T + D)
    xb, db, rb = (_rand_bits(rng, (T, D)) for _ in range(3))
    gb = si.f32_to_bf16_bits((1 + 0.02 * rng.standard_normal(D)).astype(np.float32))
    x, g, dh, dres = map(si.bf16_bits_to_f64, (xb, gb, db, rb))
    _, rstd = odl.rmsnorm_fwd(x, g, 1e-5)
    dx_ref, dg_ref = odl.rmsnorm_bwd(x, g, rstd, dh)
    xd, gd, dhd, dresd = map(dev_bf16, (xb, gb, db, rb))
    rstdd = torch.from_numpy(rstd.astype(np.float32)).cuda()
    dx, dg = torch.full_like(xd, float("nan")), torch.full_like(gd, float("nan"))
    ws = _poisoned(K.rmsnorm_backward_workspace_bytes(T, D))
    K.rmsnorm_backward(xd, gd, rstdd, dhd, None, T, D, dx, dg, 0, ws)
    # dgamma's fp32 sums of T products: 2^-24 sqrt(T) of their rms, far below the rounding of the result
    assert _norm_err(dx, dx_ref) <= ONE_ROUNDING and _norm_err(dg, dg_ref) <= ONE_ROUNDING
    first = dg.clone()
    K.rmsnorm_backward(xd, gd, rstdd, dhd, dresd, T, D, dresd, dg, 1, ws)     # in place over dres, gain gradient accumulated
    assert _norm_err(dresd, dx_ref + dres) <= ONE_ROUNDING
    assert _norm_err(dg, host_f64(first) + dg_ref) <= ONE_ROUNDING


# ------------------------------------------------------------------ embedding gradient: light, medium and heavy ids, pieces
@pytest.mark.parametrize("V,D,T,counts", [
    (3, 8, 1, [1]),                              # one token
    (70, 72, 1000, [4, 5, 63, 64, 65, 512, 200]),# both sides of every class, ids without tokens
    (9, 1032, 1200, [513, 600]),                 # the bitmap; nine column splits, the last one partly filled
    (4, 16, 6000, [4096, 1800]),                 # a full list
    (4, 16, 9000, [4097, 4800]),                 # more tokens than the list holds: walked in pieces
    (3, 264, 131072, [4096, 20000, 9001]),       # the largest batch that one bitmap spans, three column splits
    (5, 8, 140000, [3000, 65, 4]),               # tokens beyond one bitmap: lists of more than 512 sorted beforehand,
    (6, 136, 140033, [512, 513, 8192, 8193, 40000, 70]),   # up to 8192 in LDS, longer ones from the ids
])
def test_embedding_gradient_by_token_counts(K, V, D, T, counts):
    rng = np.random.default_rng(T + V)
    ids = np.full(T, -1, dtype=np.int64)         # ids outside the table are skipped
    at = rng.permutation(T)[:sum(counts)]
    ids[at] = np.repeat(np.arange(len(counts)) % V, counts)
    db = _rand_bits(rng, (T, D))
    d = si.bf16_bits_to_f64(db)
    ref = np.zeros((V, D))
    np.add.at(ref, ids[at], d[at])
    dd, idd = dev_bf16(db), torch.from_numpy(ids).cuda()
    runs = []
    for _ in range(2):
        got = torch.full((V, D), float("nan"), dtype=torch.bfloat16, device="cuda")
        K.embed_backward(dd, idd, T, V, D, got, _poisoned(K.embed_backward_workspace_bytes(T, V)))
        runs.append(got)
    assert _norm_err(runs[0], ref) <= ONE_ROUNDING
    assert not host_f64(runs[0])[ref.any(axis=1) == False].any()   # noqa: E712
    assert torch.equal(runs[0].view(torch.int16), runs[1].view(torch.int16))


def test_embedding_gradient_time_grows_with_the_tokens(K):
    """Half of the batch is one id (a padding token): four times the tokens may take four times as long, not sixteen."""
    def best_ms(T):
        rng = np.random.default_rng(T)
        ids = rng.integers(0, 1000, T)
        ids[rng.permutation(T)[:T // 2]] = 7
        idd, dd = torch.from_numpy(ids).cuda(), torch.zeros(T, 8, dtype=torch.bfloat16, device="cuda")
        out, ws = torch.empty(1000, 8, dtype=torch.bfloat16, device="cuda"), _poisoned(K.embed_backward_workspace_bytes(T, 1000))
        times = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            K.embed_backward(dd, idd, T, 1000, 8, out, ws)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)
    small, large = best_ms(1 << 18), best_ms(1 << 20)
    print(f"{small:.3f} ms, {large:.3f} ms")
    assert large <= 8 * small
