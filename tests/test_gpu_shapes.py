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
@pytest.mark.parametrize("B,S,Hq,Hkv,dh", [
    (1, 128, 4, 1, 32),      # one key block, two pieces
    (1, 640, 6, 2, 64),      # eight pieces, a group of three heads
    (1, 1792, 1, 1, 64),     # one head: the last key block has four tiles for eight pieces
    (2, 384, 8, 1, 128),     # a group as wide as the number of pieces
    (1, 2048, 3, 1, 128),    # with the dS hand-over
])
def test_attention_backward_with_split_key_blocks(K, B, S, Hq, Hkv, dh):
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
    # In the 2-norm: bf16 roundings of o (in delta), of P, of dS and of the result, each at most 2^-9 of its operand,
    # add up to 7.8e-3 at most.  (Element by element the early rows dominate, whatever the split: dq, which the split
    # does not touch, has elements 7.5e-2 of its rms off at S = 384.)
    for name, got, again, ref in zip(("dq", "dk", "dv"), runs[0], runs[1], refs):
        assert _norm_err(got, ref) <= 7.8e-3, name
        assert torch.equal(got.view(torch.int16), again.view(torch.int16)), f"{name} is not reproducible"


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
