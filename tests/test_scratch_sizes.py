"""Scratch sizes on the host: a buffer that was taken for a larger call serves the smaller ones (no GPU needed)."""
import pytest

from synth import inputs as si


@pytest.fixture(scope="module")
def K():
    import paper_2602_08387_amd as k
    return k


def _never_falls(sizes, what):
    assert all(s > 0 for s in sizes), what
    assert all(a <= b for a, b in zip(sizes, sizes[1:])), f"{what}: {sizes}"


@pytest.mark.parametrize("Hq,Hkv,dh", [(12, 12, 64), (16, 4, 64), (8, 1, 32), (16, 8, 128), (3, 1, 128), (32, 8, 128)])
def test_attention_backward_scratch_serves_smaller_batches_and_sequences(K, Hq, Hkv, dh):
    query = K.attention_backward_workspace_bytes
    for S in (128, 512, 1024, 2944, 4224, 8192):
        _never_falls([query(B, S, Hq, Hkv, dh) for B in range(1, 33)], f"batch at S = {S}")
    for B in (1, 3, 8):
        _never_falls([query(B, S, Hq, Hkv, dh) for S in range(128, 8193, 128)], f"seq at B = {B}")
        for S in (1024, 4096):
            _never_falls([query(B, S, Hq, h, dh) for h in range(1, Hq + 1) if Hq % h == 0], f"KV heads at B = {B}, S = {S}")
            _never_falls([query(B, S, Hq, Hkv, d) for d in (32, 64, 128)], f"head_dim at B = {B}, S = {S}")


@pytest.mark.parametrize("override", [
    {"d_model": 768, "n_q_heads": 12, "n_kv_heads": 6, "head_dim": 64, "d_ff": 2112},
    {"d_model": 1024, "n_q_heads": 8, "n_kv_heads": 2, "head_dim": 128, "d_ff": 2816, "recompute": 3},
    {"d_model": 128, "n_q_heads": 4, "n_kv_heads": 4, "head_dim": 32, "d_ff": 384},
])
def test_layer_scratch_serves_smaller_batches_and_sequences(K, override):
    cfg = si.CONFIGS["tiny"].with_(**override)
    for query in (K.dlayer_workspace_bytes, K.dlayer_saved_bytes):
        for S in (128, 512, 2048):
            _never_falls([query(cfg.with_(batch=B, seq=S)) for B in range(1, 25)], f"batch at S = {S}")
        for B in (1, 4):
            _never_falls([query(cfg.with_(batch=B, seq=S)) for S in range(128, 4097, 128)], f"seq at B = {B}")


@pytest.mark.parametrize("D", [8, 512, 520, 1024, 2048, 2056, 4096, 4104, 8192, 16384])
def test_rmsnorm_backward_scratch_is_a_partial_row_per_eight_rows(K, D):
    for T in (1, 7, 8, 9, 128, 1000, 4088, 4096, 4104, 16384):
        assert K.rmsnorm_backward_workspace_bytes(T, D) == 4 * D * min(-(-T // 8), 512) + (4 * T if D > 4096 else 0)
