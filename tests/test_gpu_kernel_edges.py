"""Kernels and dispatch branches at the sizes where they can go wrong (edges of tiles, remainders,
the smallest and largest of their ranges), against the fp64 oracle."""
import numpy as np
import pytest
import torch

from gkv_traces import CONFIGS
from oracle import gkv_oracle as O
from paper_2512_00504_amd import make_config
from paper_2512_00504_amd.state import DecodeState, k_rows_to_cache

from parity_utils import run_parity

pytestmark = pytest.mark.gpu

# fp32: the stated 1e-5 of the row's largest magnitude.  bf16: the result's own rounding, half a
# unit in the 8th bit (2^-9 relative, doubled for the reference's own value next to a border), and,
# at d = 128, probabilities rounded the same way: at most 2^-9 of the largest value each.
def _bound(dtype, d, ref, V):
    if dtype == "f32":
        return 1e-5 * np.abs(ref).max(axis=-1, keepdims=True)
    p_part = 2.0 ** -9 * np.abs(V).max() if d == 128 else 1e-5 * np.abs(V).max()
    return 2.0 ** -8 * np.abs(ref) + p_part


def _attend_state(dtype, d, g, lens, cap, n_tiled, seed, params=None):
    B = len(lens)
    st = DecodeState(make_config(1, B, 2 * g, 2, d, 16, 4, 8, cap, dtype), params=params)
    gen = torch.Generator().manual_seed(seed)
    rnd = lambda *s: torch.randn(*s, generator=gen).to(st.K.dtype)
    K, V, q = rnd(1, B, 2, cap, d), rnd(1, B, 2, cap, d), rnd(1, B, 2 * g, d)
    kn, vn = rnd(1, B, 2, d), rnd(1, B, 2, d)
    for i, n in enumerate(lens):                # rows past the end hold NaN: they must not be used
        K[0, i, :, n:] = float("nan"); V[0, i, :, n:] = float("nan")
        st.K[0, i] = k_rows_to_cache(K[0, i], min(n_tiled, n // 16 * 16)).cuda()
    st.V.copy_(V)
    rec = [[n, 5, 0, min(n_tiled, n // 16 * 16)] for n in lens]
    st.d_state.copy_(torch.tensor([rec], dtype=torch.int32))
    st.len_host = max(lens)
    return st, K, V, q, kn, vn


def _check_attend(st, K, V, q, kn, vn, lens, dtype, d, append):
    dev = lambda t: t.cuda() if append else None
    out = st.attend_decode(q.cuda(), dev(kn), dev(vn), 5).double().cpu().numpy()
    for i, n in enumerate(lens):
        Ki, Vi = K[0, i].double().numpy().copy(), V[0, i].double().numpy().copy()
        if append:
            Ki[:, n], Vi[:, n] = kn[0, i].double().numpy(), vn[0, i].double().numpy()
        n_tot = n + append
        ref = O.attend(q[0, i].double().numpy(), Ki[:, :n_tot], Vi[:, :n_tot], n_tot)
        err = np.abs(out[0, i] - ref)
        assert (err <= _bound(dtype, d, ref, Vi[:, :n_tot])).all(), (n, err.max())
        if append:
            assert torch.equal(st.K[0, i, :, n].cpu(), kn[0, i]) and torch.equal(st.V[0, i, :, n].cpu(), vn[0, i])
            assert (st.pos[0, i, :, n] == 5).all()
    assert torch.equal(st.qwin[5 % 4].cpu(), q)


@pytest.mark.parametrize("append", [True, False])
@pytest.mark.parametrize("dtype,d,g", [("f32", 64, 1), ("f32", 64, 16), ("f32", 128, 7), ("f32", 128, 16),
                                       ("bf16", 64, 5), ("bf16", 64, 16), ("bf16", 128, 3)])
def test_attend_at_tile_edges(dtype, d, g, append):
    lens = [1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 250, 255]
    for n_tiled in (0, 48, 4096):
        st, *t = _attend_state(dtype, d, g, lens, 256, n_tiled, seed=d + g)
        _check_attend(st, *t, lens, dtype, d, append)


@pytest.mark.parametrize("over", [
    dict(dtype="f32", n_layers=2, batch=2, n_q_heads=14, n_kv_heads=2, budget=96, window=16, interval=32),    # fp32, d = 128, g = 7
    dict(dtype="f32", n_layers=1, batch=2, n_q_heads=6, n_kv_heads=2, budget=70, window=5, interval=24, head_dim=64),
    dict(dtype="bf16", n_layers=2, batch=2, n_q_heads=16, n_kv_heads=1, budget=80, window=8, interval=24, head_dim=64),
])
def test_whole_path_fp32_and_head_dim_64(over):
    wl = CONFIGS["cfg2_single_layer"].with_(n_steps=320, seed=61, **over)
    st = run_parity(wl, wl.n_steps, chunk=64)
    assert st["events"] >= 5
