"""Kernels and dispatch branches at the sizes where they can go wrong (edges of tiles, remainders,
the smallest and largest of their ranges), against the fp64 oracle."""
import numpy as np
import pytest
import torch

from gkv_traces import CONFIGS
from oracle import gkv_oracle as O
from paper_2512_00504_amd import make_config
from paper_2512_00504_amd.state import DecodeState, k_cache_to_rows, k_rows_to_cache

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


def _attend_state(dtype, d, g, lens, cap, n_tiled, seed, params=None, b=16, s=8):
    B = len(lens)
    st = DecodeState(make_config(1, B, 2 * g, 2, d, b, 4, s, cap, dtype), params=params)
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


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("B,hkv,n_tiled", [(85, 3, 16), (87, 3, 48), (52, 5, 0)])   # 255, 261 and 260 units
def test_attend_on_both_sides_of_256_units(dtype, d, B, hkv, n_tiled):
    # 4 and 8 wavefronts, of which those beyond a unit's end ask for its last slice, or in an empty unit for rows that do
    # not count: lengths from nothing to the last row, both K formats, a group of 5 and rows of NaN behind every length;
    # KV heads and workgroups that are no power of two
    g, b, cap = 5, 40, 96
    st = DecodeState(make_config(1, B, hkv * g, hkv, d, b, 4, 8, cap, dtype))
    gen = torch.Generator().manual_seed(B * d)
    rnd = lambda *s: torch.randn(*s, generator=gen).to(st.K.dtype)
    K, V, q, kn, vn = rnd(1, B, hkv, cap, d), rnd(1, B, hkv, cap, d), rnd(1, B, hkv * g, d), rnd(1, B, hkv, d), rnd(1, B, hkv, d)
    lens = [i % cap for i in range(B)]
    for i, n in enumerate(lens):
        K[0, i, :, n:] = float("nan"); V[0, i, :, n:] = float("nan")
        st.K[0, i] = k_rows_to_cache(K[0, i], min(n_tiled, n // 16 * 16)).cuda()
    st.V.copy_(V)
    st.d_state.copy_(torch.tensor([[[n, 5, 0, min(n_tiled, n // 16 * 16)] for n in lens]], dtype=torch.int32))
    st.len_host = max(lens)
    out = st.attend_decode(q.cuda(), kn.cuda(), vn.cuda(), 5).double().cpu().numpy()
    for i, n in enumerate(lens):
        Ki, Vi = K[0, i].double().numpy().copy(), V[0, i].double().numpy().copy()
        Ki[:, n], Vi[:, n] = kn[0, i].double().numpy(), vn[0, i].double().numpy()
        ref = O.attend(q[0, i].double().numpy(), Ki[:, : n + 1], Vi[:, : n + 1], n + 1)
        assert (np.abs(out[0, i] - ref) <= _bound(dtype, d, ref, Vi[:, : n + 1])).all(), n
        assert torch.equal(st.V[0, i, :, n].cpu(), vn[0, i]) and (st.pos[0, i, :, n] == 5).all()
    assert torch.equal(st.qwin[5 % 4].cpu(), q)


@pytest.mark.parametrize("append", [True, False])
@pytest.mark.parametrize("dtype,d,g", [("f32", 64, 1), ("f32", 64, 16), ("f32", 128, 7), ("f32", 128, 16),
                                       ("bf16", 64, 5), ("bf16", 64, 16), ("bf16", 128, 3)])
def test_attend_at_tile_edges(dtype, d, g, append):
    lens = [1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 250, 255]
    for n_tiled in (0, 48, 4096):
        st, *t = _attend_state(dtype, d, g, lens, 256, n_tiled, seed=d + g)
        _check_attend(st, *t, lens, dtype, d, append)


# every instantiation of the decode kernel: wavefronts, keys per slice, whole and cut units; the last number: more units than that, for
# the forms of larger launches (at 256 and 512 workgroups, see launch_by_size)
DECODE_FORMS = [("f32", 64, 3, 256, None, 0), ("f32", 128, 7, 256, None, 0), ("bf16", 64, 5, 256, None, 0), ("bf16", 128, 7, 256, None, 0),
                ("f32", 128, 2, 640, None, 0), ("bf16", 64, 5, 1312, None, 0), ("bf16", 128, 7, 3936, None, 0),      # cut
                ("f32", 64, 2, 256, {"attend_waves": 16}, 0), ("f32", 128, 2, 256, {"attend_waves": 8}, 0),
                ("bf16", 64, 2, 256, {"attend_waves": 16}, 0), ("bf16", 128, 2, 256, {"attend_waves": 16}, 0),
                ("bf16", 64, 2, 256, {"attend_waves": 8}, 0), ("f32", 64, 2, 256, {"attend_waves": 8}, 0),
                ("bf16", 128, 2, 640, {"attend_tile": 32, "attend_splits": 2}, 0), ("f32", 64, 2, 640, {"force_generic": 1}, 0),
                ("f32", 64, 2, 256, {"attend_waves": 4}, 0), ("bf16", 128, 3, 256, {"attend_waves": 4}, 0)]
LARGE_FORMS = [(*t, 2, 256, {"attend_waves": waves}, units) for t in (("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128))
               for waves, units in ((4, 256), (4, 512), (8, 256)) if (*t, waves) != ("f32", 128, 8)]
DECODE_FORMS += LARGE_FORMS


def _repeated(lens, units):
    """The lengths, two units each, as often as it takes for more than that many units."""
    return lens * (units // (2 * len(lens)) + 1)


@pytest.mark.parametrize("dtype,d,g,cap,params,units", DECODE_FORMS)
def test_attend_over_nothing(dtype, d, g, cap, params, units):
    # an empty sequence and no new row: every wavefront is beyond the end, and the rows that are there (NaN) count for nobody
    lens = _repeated([0, 1, 0, 40], units)
    st, K, V, q, kn, vn = _attend_state(dtype, d, g, lens, cap, 48, seed=9, params=params)
    out = st.attend_decode(q.cuda(), None, None, 5).double().cpu().numpy()
    assert (out[0, ::2] == 0).all()
    for i in range(1, len(lens), 2):
        Ki, Vi = K[0, i].double().numpy(), V[0, i].double().numpy()
        ref = O.attend(q[0, i].double().numpy(), Ki[:, : lens[i]], Vi[:, : lens[i]], lens[i])
        assert (np.abs(out[0, i] - ref) <= _bound(dtype, d, ref, Vi[:, : lens[i]])).all()


@pytest.mark.parametrize("dtype,d,g,cap,params,units", DECODE_FORMS)
def test_attend_logits_of_minus_infinity(dtype, d, g, cap, params, units):
    # a key whose logit is -inf has weight 0, wherever it stands: the cache's first half, the newest row,
    # whole slices; a row of nothing else is NaN, as softmax gives; the others keep their accuracy
    lens = _repeated([1, 17, 33, 34, 65, 250, cap - 1], units)
    st, K, V, q, kn, vn = _attend_state(dtype, d, g, lens, cap, 64, seed=7, params=params)
    q = q.abs() + 0.125                                                 # so that no other logit is inf * 0
    for i, n in enumerate(lens):
        K[0, i, :, : n // 2, 3] = -float("inf")
        K[0, i, :, n // 2 + 1: n: 5, 3] = -float("inf")
        st.K[0, i] = k_rows_to_cache(K[0, i], min(64, n // 16 * 16)).cuda()
    kn[0, 1, :, 3] = kn[0, 5, :, 3] = -float("inf")
    K[0, 2, :, :33, 3] = kn[0, 2, :, 3] = -float("inf")                 # sequence 2: nothing else
    st.K[0, 2] = k_rows_to_cache(K[0, 2], 32).cuda()
    out = st.attend_decode(q.cuda(), kn.cuda(), vn.cuda(), 5).double().cpu().numpy()
    for i, n in enumerate(lens):
        Ki, Vi = K[0, i].double().numpy().copy(), V[0, i].double().numpy().copy()
        Ki[:, n], Vi[:, n] = kn[0, i].double().numpy(), vn[0, i].double().numpy()
        if i == 2:
            assert np.isnan(out[0, i]).all()
            continue
        ref = O.attend(q[0, i].double().numpy(), Ki[:, : n + 1], Vi[:, : n + 1], n + 1)
        assert np.isfinite(ref).all()
        err = np.abs(out[0, i] - ref)
        assert (err <= _bound(dtype, d, ref, Vi[:, : n + 1])).all(), (n, err.max())


@pytest.mark.parametrize("size", [1e9, -1e9, 3e33, -3e33])
@pytest.mark.parametrize("dtype,d,g,cap,params,units", DECODE_FORMS)
def test_attend_huge_logits(dtype, d, g, cap, params, units, size):
    # finite logits of any size: keys are multiples of one vector, so every logit is a known share of the
    # largest (whichever its sign) and the softmax is one-hot; the output is that key's V, to the bit
    lens = _repeated([1, 17, 33, 65, 250, cap - 1], units)
    st, K, V, q, kn, vn = _attend_state(dtype, d, g, lens, cap, 64, seed=19, params=params)
    q = q.abs() + 0.125
    u = torch.rand(d, generator=torch.Generator().manual_seed(4)) + 0.5
    best = []
    for i, n in enumerate(lens):
        mult = (torch.randperm(n + 1, generator=torch.Generator().manual_seed(i)) % 32 + 2) * 0.5     # 1 .. 16.5
        top = (7 * i) % (n + 1)                               # one that stands out: 20 if positive, 0.25 if negative
        mult[top] = 20.0 if size > 0 else 0.25
        rows = (mult[:, None] * size * u).to(q.dtype)
        K[0, i, :, :n], kn[0, i] = rows[:n], rows[n]
        st.K[0, i] = k_rows_to_cache(K[0, i], min(64, n // 16 * 16)).cuda()
        best.append(vn[0, i] if top == n else V[0, i, :, top])
    out = st.attend_decode(q.cuda(), kn.cuda(), vn.cuda(), 5).cpu()
    for i, n in enumerate(lens):
        assert torch.equal(out[0, i].view(2, g, d), best[i][:, None].expand(2, g, d)), n


@pytest.mark.parametrize("dtype,d,g,cap,params,units", DECODE_FORMS)
def test_attend_infinite_values(dtype, d, g, cap, params, units):
    # an infinite value with a weight above zero makes its channel infinite, two of opposite sign NaN, and
    # neither touches the other channels
    lens = _repeated([1, 17, 33, 65, 250, cap - 1], units)
    st, K, V, q, kn, vn = _attend_state(dtype, d, g, lens, cap, 64, seed=13, params=params)
    q = (q * 0.125).to(q.dtype)                                         # every weight well above zero
    for i, n in enumerate(lens):
        V[0, i, :, n // 2, 3] = float("inf")
        V[0, i, :, n // 2, d - 2] = -float("inf")
        V[0, i, :, 0, 17] = float("inf")
        if n > 1:
            V[0, i, :, n - 1, 17] = -float("inf")
    vn[0, 2, :, 5] = -float("inf")
    st.V.copy_(V)
    out = st.attend_decode(q.cuda(), kn.cuda(), vn.cuda(), 5).double().cpu().numpy()
    for i, n in enumerate(lens):
        Ki, Vi = K[0, i].double().numpy().copy(), V[0, i].double().numpy().copy()
        Ki[:, n], Vi[:, n] = kn[0, i].double().numpy(), vn[0, i].double().numpy()
        ref = O.attend(q[0, i].double().numpy(), Ki[:, : n + 1], Vi[:, : n + 1], n + 1)
        assert np.isinf(ref).any() and (n == 1 or np.isnan(ref).any())
        bad = ~np.isfinite(ref)
        np.testing.assert_array_equal(out[0, i][bad], ref[bad])
        fin = np.where(bad, 0.0, ref)
        Vf = np.where(np.isfinite(Vi[:, : n + 1]), Vi[:, : n + 1], 0.0)
        assert (np.abs(np.where(bad, 0.0, out[0, i]) - fin) <= _bound(dtype, d, fin, Vf)).all()


@pytest.mark.parametrize("dtype,d,g,cap,params,units", DECODE_FORMS)
def test_attend_infinite_values_of_small_weight(dtype, d, g, cap, params, units):
    # a weight that is a normal fp32 number makes its infinite value's channel infinite, whatever parts it enters in
    lens = _repeated([15, 40], max(units, 118))
    log2_weight = np.linspace(-100, -125, len(lens))
    st, K, V, q, kn, vn = _attend_state(dtype, d, g, lens, cap, 0, seed=17, params=params)
    q.fill_(1.0)
    K.zero_(); kn.zero_()                                               # the others' logits
    K[0, :, :, 4] = torch.from_numpy(log2_weight * np.log(2) / np.sqrt(d)).view(-1, 1, 1).to(q.dtype)
    V[0, :, :, 4, 3], V[0, :, :, 4, d - 2] = float("inf"), -float("inf")
    st.K.copy_(K); st.V.copy_(V)
    out = st.attend_decode(q.cuda(), kn.cuda(), vn.cuda(), 5).double().cpu().numpy()
    for i, n in enumerate(lens):
        Ki, Vi = (torch.cat([x[0, i, :, :n], y[0, i, :, None]], dim=1).double().numpy() for x, y in ((K, kn), (V, vn)))
        ref = O.attend(q[0, i].double().numpy(), Ki, Vi, n + 1)
        bad = ~np.isfinite(ref)
        assert bad.sum() == 2 * 2 * g
        np.testing.assert_array_equal(out[0, i][bad], ref[bad])
        fin = np.where(bad, 0.0, ref)
        Vf = np.where(np.isfinite(Vi), Vi, 0.0)
        assert (np.abs(np.where(bad, 0.0, out[0, i]) - fin) <= _bound(dtype, d, fin, Vf)).all()


def _error_of_cancelling_values(dtype, d, g, cap, params, lens):
    # Values whose weighted sum cancels to about 2^-27 of its terms leave the rounding of the weights in
    # the output: the 2-norm of the error over that of the terms, as a power of two.
    st, K, V, q, kn, vn = _attend_state(dtype, d, g, lens, cap, 64, seed=3, params=params)
    q = (q * 0.0625).to(q.dtype)
    err2 = terms2 = 0.0
    for i, n in enumerate(lens):
        for j in range(2):
            k = np.concatenate([K[0, i, j, :n].double().numpy(), kn[0, i, j : j + 1].double().numpy()])
            z = k @ q[0, i, j * g].double().numpy() / np.sqrt(d)            # head 0 of the group
            p = np.exp(z - z.max()); p /= p.sum()
            v = V[0, i, j, :n].double().numpy()
            v = np.concatenate([v, vn[0, i, j : j + 1].double().numpy()])
            for x in range(n - 3, n):                                       # the last three cached rows take what is left
                v[x] = 0.0
                v[x] = torch.from_numpy(-(p @ v) / p[x]).to(q.dtype).double().numpy()
            V[0, i, j, :n] = torch.from_numpy(v[:n]).to(q.dtype)
    st.V.copy_(V)
    out = st.attend_decode(q.cuda(), kn.cuda(), vn.cuda(), 5).double().cpu().numpy()
    for i, n in enumerate(lens):
        for j in range(2):
            k = np.concatenate([K[0, i, j, :n].double().numpy(), kn[0, i, j : j + 1].double().numpy()])
            v = np.concatenate([V[0, i, j, :n].double().numpy(), vn[0, i, j : j + 1].double().numpy()])
            z = k @ q[0, i, j * g].double().numpy() / np.sqrt(d)
            p = np.exp(z - z.max()); p /= p.sum()
            err2 += ((out[0, i, j * g] - p @ v) ** 2).sum()
            terms2 += ((p[:, None] * v) ** 2).sum()
    return 0.5 * np.log2(err2 / terms2)


@pytest.mark.parametrize("dtype,d,g,cap,params,units", [f for f in DECODE_FORMS if f[:2] != ("bf16", 128)])
def test_attend_probabilities_keep_32_bits(dtype, d, g, cap, params, units):
    # Small logits: their own rounding and the exponential's are about 2^-23.  2^-23 and less for weights
    # in fp32 (bound 2^-21), 2^-18.5 for 16 bits.
    assert _error_of_cancelling_values(dtype, d, g, cap, params, _repeated([60, 61, 63, 120, 200, 250, cap - 1], units)) <= -21


# Cut units, and short ones of launches that could be: weights in two parts of 8 bits, the second rounded to 2^-9 of at most
# 2^-7 of the weight (bound 2^-15), 2^-9.6 for weights of one.
@pytest.mark.parametrize("g,cap,params", [(7, 3936, None), (16, 640, None), (1, 640, {"attend_splits": 3}), (7, 160, None)])
def test_attend_probabilities_of_cut_units_keep_16_bits(g, cap, params):
    assert _error_of_cancelling_values("bf16", 128, g, cap, params, [60, 61, 63, 120, cap // 3, cap // 2, cap - 1]) <= -15


@pytest.mark.parametrize("over", [
    dict(dtype="f32", n_layers=2, batch=2, n_q_heads=14, n_kv_heads=2, budget=96, window=16, interval=32),    # fp32, d = 128, g = 7
    dict(dtype="f32", n_layers=1, batch=2, n_q_heads=6, n_kv_heads=2, budget=70, window=5, interval=24, head_dim=64),
    dict(dtype="bf16", n_layers=2, batch=2, n_q_heads=16, n_kv_heads=1, budget=80, window=8, interval=24, head_dim=64),
])
def test_whole_path_fp32_and_head_dim_64(over):
    wl = CONFIGS["cfg2_single_layer"].with_(n_steps=320, seed=61, **over)
    st = run_parity(wl, wl.n_steps, chunk=64)
    assert st["events"] >= 5


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_attend_tile_changes_nothing_at_head_dim_64(dtype):
    outs = []
    for tile in (16, 32):
        st, _, _, q, kn, vn = _attend_state(dtype, 64, 3, [600, 333], 640, 64, seed=2, params={"attend_tile": tile, "attend_splits": 1})
        outs.append(st.attend_decode(q.cuda(), kn.cuda(), vn.cuda(), 5))
    assert torch.equal(*outs)


# ---- window score -----------------------------------------------------------------------------
def _check_window_score(dtype, d, g, w, params, reuse, scale=0.0, hidden=False, size=None):
    cap, b = 320, 48
    lens = [b + 1, b + 15, b + 17, 100, 127, 160, 161, cap]           # rows the compression sees
    lens = [max(n, w + 1) for n in lens]
    B = len(lens)
    st = DecodeState(make_config(1, B, g, 1, d, b, w, max(w, 8), cap, dtype, softmax_scale=scale), params=params)
    st.ctx.set_param("score_reuse_stats", reuse)
    gen = torch.Generator().manual_seed(100 * g + w)
    rnd = lambda *s: torch.randn(*s, generator=gen).to(st.K.dtype)
    K, q = 2 * rnd(1, B, 1, cap, d), rnd(w, 1, B, g, d)
    if hidden:                                                          # logits of -inf, for some keys of candidates and window
        q = q.abs() + 0.125
        K[..., 1::3, 3] = -float("inf")
    if size:                    # logits that are known shares of the largest one: one-hot window rows, in or out of the candidates
        q = q.abs() + 0.125
        mult = torch.arange(cap, dtype=torch.float32) % 37 * 0.25 + 1.0
        mult[[11, 30]] = torch.tensor([20.0, 0.25])
        K[:] = (mult[:, None] * size * (torch.rand(d, generator=gen) + 0.5)).to(K.dtype)
    n_tiled = [(n - w) // 32 * 16 for n in lens]                        # some of the candidate tiles are row-major
    t0 = 7
    for i, n in enumerate(lens):
        Ki = K[0, i].clone(); Ki[:, n - w:] = float("nan")             # the window's rows come from the decode calls
        st.K[0, i] = k_rows_to_cache(Ki, n_tiled[i]).cuda()
    st.d_state.copy_(torch.tensor([[[n - w, t0, 0, m] for n, m in zip(lens, n_tiled)]], dtype=torch.int32))
    for k in range(w):
        kn = torch.stack([K[0, i, :, n - w + k] for i, n in enumerate(lens)])[None].contiguous()
        st.ctx.attend_decode(q[k].cuda(), kn.cuda(), kn.cuda(), st.K, st.V, st.pos, t0 + k, st.qwin, st.d_state,
                             cap - w + k, st.out, st.workspace)
    t = t0 + w - 1
    st.len_host = cap
    st.S.fill_(-3.0)
    if params:                                                            # through gkv_evict
        st.ctx.evict(st.qwin, st.K, st.V, st.F_hist, st.pos, st.d_state, t, cap, st.S, st.F, st.keep_idx, st.workspace)
    else:
        st.score_window(t)
    S = st.S.double().cpu().numpy()
    for i, n in enumerate(lens):
        A = O.window_probs(q[:, 0, i].permute(1, 0, 2).double().numpy(), K[0, i].double().numpy(), n,
                           float(np.float32(scale)) if scale else None)
        ref = O.local_score(A, 1)[:, : n - w]
        err = np.abs(S[0, i, :, : n - w] - ref)
        assert (err <= 1e-5 * ref + 1e-30).all(), (n, (err / (ref + 1e-300)).max())
        assert (S[0, i, :, n - w:] == -3.0).all()
        if params:
            F = O.global_score(ref, np.zeros_like(ref), 0, 0.8, "max")
            np.testing.assert_allclose(st.F[0, i, :, : n - w].double().cpu().numpy(), F, rtol=1e-5, atol=1e-30)


# Elementwise 1e-5 of the fp64 score (plus 1e-30 absolute), the bound of the whole-path tests: fp32
# sums of up to 128 products and one exponential.
@pytest.mark.parametrize("dtype,d,g,w,params", [
    ("bf16", 128, 7, 16, None),                       # two row pairs of tiles, one block per head
    ("bf16", 128, 16, 32, None),                      # queries beyond one staging pass
    ("bf16", 128, 3, 8, None), ("bf16", 128, 4, 5, None),     # two heads share a block, odd and even groups
    ("bf16", 64, 1, 1, None), ("bf16", 64, 5, 33, None),      # a window row count just past a block
    ("f32", 128, 7, 16, None), ("f32", 128, 16, 24, None),    # two staging passes of 128 KiB
    ("f32", 64, 2, 8, None), ("f32", 64, 16, 40, None),
    ("bf16", 128, 5, 32, {"evict_fuse_global": 1}),
])
@pytest.mark.parametrize("reuse", [1, 0])
def test_window_score_at_tile_edges(dtype, d, g, w, params, reuse):
    _check_window_score(dtype, d, g, w, params, reuse)


# The window rows' own statistics with keys hidden from some rows, at scales whose low part (scale *
# log2 e rounded to fp32) has either sign: a hidden key must add nothing, whatever the residue of its
# masked logit.  Same bound.
@pytest.mark.parametrize("scale", [0.1, 0.05, 0.2, 0.125])
@pytest.mark.parametrize("dtype,d,g,w", [("bf16", 128, 7, 16), ("bf16", 64, 5, 8), ("f32", 128, 3, 16), ("f32", 64, 2, 24),
                                         ("bf16", 128, 5, 32), ("bf16", 64, 5, 30), ("bf16", 128, 8, 9), ("bf16", 128, 15, 4),
                                         ("bf16", 128, 16, 16)])
def test_window_score_own_statistics_other_scales(dtype, d, g, w, scale):
    _check_window_score(dtype, d, g, w, None, 0, scale)


@pytest.mark.parametrize("reuse", [1, 0])
@pytest.mark.parametrize("dtype,d,g,w", [("bf16", 128, 7, 16), ("bf16", 64, 5, 8), ("f32", 128, 3, 16), ("f32", 64, 2, 24)])
def test_window_score_logits_of_minus_infinity(dtype, d, g, w, reuse):
    # probability 0 for those keys, with the statistics recorded by the decode calls and with its own
    _check_window_score(dtype, d, g, w, None, reuse, hidden=True)


@pytest.mark.parametrize("size", [1e9, -1e9, 3e33, -3e33])
@pytest.mark.parametrize("reuse", [1, 0])
@pytest.mark.parametrize("dtype,d,g,w", [("bf16", 128, 7, 16), ("bf16", 64, 5, 8), ("f32", 128, 3, 16), ("f32", 64, 2, 24)])
def test_window_score_huge_logits(dtype, d, g, w, reuse, size):
    # every window row has one key of probability 1 (row 11 for positive logits, row 30 for negative)
    _check_window_score(dtype, d, g, w, None, reuse, size=size)


# 4 wavefronts: two slices in flight (up to 256 workgroups) or one, the next K behind V and paced (up to 512) or before it; 8: one, behind (up to 256), or
# in step or early: no slice, one, two, ... for a wavefront, the unit's last one on both sides of its border
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("waves,many", [(4, 1), (4, 6), (4, 12), (8, 1), (8, 6), (8, 12)])
def test_attend_slices_in_turn(dtype, d, waves, many):
    per_round = waves * (32 if (dtype, d) == ("bf16", 64) else 16)
    lens = [k * per_round + e for k in (1, 2, 3, 4, 5) for e in (-2, -1, 0, 1)] + [0, per_round // 2, 4 * per_round + 17]
    lens = lens * many                                                  # two units each
    cap = -(-(5 * per_round + 2) // 32) * 32
    st, *t = _attend_state(dtype, d, 3, lens, cap, 3 * per_round, seed=waves, params={"attend_waves": waves, "attend_splits": 1})
    _check_attend(st, *t, lens, dtype, d, append=True)


# The same call again gives the same bits, in launches of more than 256 and 512 workgroups too (cut ones: below)
@pytest.mark.parametrize("dtype,d,g,cap,params,units", LARGE_FORMS)
def test_attend_repeats_itself(dtype, d, g, cap, params, units):
    lens = _repeated([1, 17, 33, 34, 65, 250, cap - 1], units)
    st, K, V, q, kn, vn = _attend_state(dtype, d, g, lens, cap, 64, seed=23, params=params)
    q = q.cuda()
    want = st.attend_decode(q, None, None, 5).clone()
    for _ in range(20):
        st.out.zero_()
        assert torch.equal(st.attend_decode(q, None, None, 5), want)


# ---- units cut over several workgroups ----------------------------------------------------------
@pytest.mark.parametrize("dtype,d,g,cap", [("bf16", 128, 7, 3936), ("bf16", 128, 16, 640), ("bf16", 64, 5, 1312), ("f32", 128, 7, 640),
                                           ("f32", 64, 2, 1312)])
def test_attend_cut_over_workgroups(dtype, d, g, cap):
    # lengths around the borders of one, two and all pieces, on the same workspace call after call
    lens = [0, 1, 127, 128, 129, 255, 256, 257, cap // 2, cap - 1]
    st, *t = _attend_state(dtype, d, g, lens, cap, 64, seed=d)
    for _ in range(2):
        _check_attend(st, *t, lens, dtype, d, append=True)
        tickets = st.workspace[: 4 * 8 * 2 * len(lens) * 9].view(torch.int32)   # 8 a unit, 8 sets and that of "attend_splits"
        assert int(tickets.abs().sum()) == 0                                # back at zero for the next call
        st.len_host = max(lens)
    # a context that never asked for the workspace's size does without the partials: same result
    a = st.attend_decode(t[2].cuda(), t[3].cuda(), t[4].cuda(), 5).clone()
    from paper_2512_00504_amd import Context
    st.ctx = Context(st.cfg)
    st.len_host = max(lens)
    b = st.attend_decode(t[2].cuda(), t[3].cuda(), t[4].cuda(), 5)
    tol = 1e-5 if dtype == "f32" else 2.0 ** -7
    np.testing.assert_allclose(a.double().cpu().numpy(), b.double().cpu().numpy(), rtol=tol, atol=tol)


# Budgets long enough for pieces of 8 wavefronts, and the shortest of them: a unit of more than eight slices is cut into
# both whatever the others' lengths, with the running maxima, and so the bits, that asking for this gives.
@pytest.mark.parametrize("dtype,d,b", [("bf16", 128, 1040), ("bf16", 128, 640), ("bf16", 64, 1280), ("f32", 64, 1040), ("f32", 64, 630)])
def test_long_units_have_the_bits_of_two_pieces_of_8_wavefronts(dtype, d, b):
    lens = [b + 31 - 7 * i for i in range(60)]
    outs = []
    for params in (None, {"attend_waves": 8, "attend_splits": 2}):
        st, K, V, q, kn, vn = _attend_state(dtype, d, 3, lens, (b + 63) // 32 * 32, 64, seed=b, params=params, b=b, s=32)
        outs.append(st.attend_decode(q.cuda(), kn.cuda(), vn.cuda(), 5).clone())
    assert torch.equal(*outs)
    for i in (0, 30, 59):
        Ki, Vi = (torch.cat([x[0, i, :, : lens[i]], n[0, i, :, None]], dim=1).double().numpy() for x, n in ((K, kn), (V, vn)))
        ref = O.attend(q[0, i].double().numpy(), Ki, Vi, lens[i] + 1)
        assert (np.abs(outs[0][0, i].double().cpu().numpy() - ref) <= _bound(dtype, d, ref, Vi)).all()


# One context and one workspace, several streams with buffers of their own: decode calls that the library
# cuts by its own choice stay independent.
def _call(st, ctx, ws, q, kn, vn, out, t=5):
    ctx.attend_decode(q, kn, vn, st.K, st.V, st.pos, t, st.qwin, st.d_state, 1000, out, ws)


def _two_users(dtype="bf16", d=128, g=7, cap=1056):
    users = []
    for seed in (21, 22):
        st, K, V, q, kn, vn = _attend_state(dtype, d, g, [1000, 700, 930], cap, 512, seed=seed)
        users.append((st, q.cuda(), kn.cuda(), vn.cuda()))
    torch.cuda.synchronize()
    return users


def test_cut_calls_of_different_streams_have_partial_results_of_their_own():
    # without a new row a call changes nothing in the workspace but partial results: what the first
    # stream's call left there is still there after the other's, and after a recorded one's
    (a, qa, _, _), (b, qb, _, _) = _two_users()
    ctx, ws = a.ctx, a.workspace
    streams = [torch.cuda.Stream() for _ in range(2)]
    before = ws.clone()
    torch.cuda.synchronize()
    with torch.cuda.stream(streams[0]):
        _call(a, ctx, ws, qa, None, None, a.out)
    torch.cuda.synchronize()
    mine = ws != before
    assert int(mine.sum()) > 0                                              # it was cut
    held = ws.clone()
    with torch.cuda.stream(streams[1]):
        _call(b, ctx, ws, qb, None, None, b.out)
    torch.cuda.synchronize()
    assert torch.equal(ws[mine], held[mine]) and not torch.equal(ws, held)
    held = ws.clone()
    graph = torch.cuda.CUDAGraph()
    streams[1].wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=streams[1]):                        # a capture on a stream that has a set
        _call(b, ctx, ws, qb, None, None, b.out)
    want = b.out.clone()
    for _ in range(3):
        b.out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(b.out, want)
    changed = held != before
    assert torch.equal(ws[changed], held[changed]) and not torch.equal(ws, held)


@pytest.mark.parametrize("dtype,d,g", [("bf16", 128, 7), ("f32", 128, 7), ("bf16", 64, 5), ("f32", 64, 2)])
def test_overlapping_decode_calls_share_a_workspace(dtype, d, g):
    users = _two_users(dtype, d, g)
    ctx, ws = users[0][0].ctx, users[0][0].workspace
    want = []
    for st, q, kn, vn in users:                                             # one after the other
        _call(st, ctx, ws, q, kn, vn, st.out)
        torch.cuda.synchronize()
        want.append(st.out.clone())
    streams = [torch.cuda.Stream() for _ in range(2)]
    for _ in range(20):
        outs = [[torch.zeros_like(st.out) for _ in range(10)] for st, *_ in users]
        torch.cuda.synchronize()
        for i in range(10):
            for (st, q, kn, vn), stream, out in zip(users, streams, outs):
                with torch.cuda.stream(stream):
                    _call(st, ctx, ws, q, kn, vn, out[i])
        torch.cuda.synchronize()
        for got, ref in zip(outs, want):
            assert all(torch.equal(x, ref) for x in got)
    # more streams than there are sets: not cut, the same up to the order of the sums
    st, q, kn, vn = users[0]
    for stream in [torch.cuda.Stream() for _ in range(10)]:
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            _call(st, ctx, ws, q, kn, vn, st.out)
        torch.cuda.synchronize()
        tol = 1e-5 if dtype == "f32" else 2.0 ** -7
        np.testing.assert_allclose(st.out.double().cpu().numpy(), want[0].double().cpu().numpy(), rtol=tol, atol=tol)


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 64), ("bf16", 128)])
@pytest.mark.parametrize("other_cache,other_stream", [(True, True), (True, False), (False, True)])
def test_recorded_statistics_of_another_stream_are_not_trusted(dtype, d, other_cache, other_stream):
    # a decode call on another K cache and another stream may write its statistics at any time; here what
    # it would write is put there by hand after the window's calls.  On one stream, or on one cache (with
    # another ring), the record is used.
    w, b, cap = 4, 40, 96
    st = [DecodeState(make_config(1, 2, 4, 2, d, b, w, 8, cap, dtype)) for _ in range(2)]
    ctx, ws = st[0].ctx, st[0].workspace
    gen = torch.Generator().manual_seed(5)
    rnd = lambda *s: torch.randn(*s, generator=gen).to(st[0].K.dtype)
    K, q, kn = rnd(1, 2, 2, cap, d), rnd(w, 1, 2, 4, d), rnd(w, 1, 2, 2, d)
    for x in st:
        x.K.copy_(K)
        x.d_state.copy_(torch.tensor([60, 8, 0, 0], dtype=torch.int32).expand(1, 2, 4))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    if not other_stream:
        streams[0] = streams[1]
    if not other_cache:
        st[0].K = st[1].K
    torch.cuda.synchronize()
    with torch.cuda.stream(streams[0]):
        ctx.attend_decode(q[0].cuda(), None, None, st[0].K, st[0].V, st[0].pos, 8, st[0].qwin, st[0].d_state, 60, st[0].out, ws)
    torch.cuda.synchronize()
    with torch.cuda.stream(streams[1]):
        for i in range(w):
            ctx.attend_decode(q[i].cuda(), kn[i].cuda(), kn[i].cuda(), st[1].K, st[1].V, st[1].pos, 8 + i, st[1].qwin,
                              st[1].d_state, 60 + i, st[1].out, ws)
        torch.cuda.synchronize()
        ws.view(torch.float32).mul_(1.5)                                    # statistics; the counters are zero
        ctx.score_window(st[1].qwin, st[1].K, st[1].d_state, 8 + w - 1, 60 + w, st[1].S, ws)
        torch.cuda.synchronize()
    S = st[1].S.double().cpu().numpy()
    right = True
    for i in range(2):
        Ki = K[0, i].double().numpy().copy()
        Ki[:, 60 : 60 + w] = kn[:, 0, i].permute(1, 0, 2).double().numpy()
        ref = O.local_score(O.window_probs(q[:, 0, i].permute(1, 0, 2).double().numpy(), Ki, 60 + w), 2)[:, :60]
        right &= bool((np.abs(S[0, i, :, :60] - ref) <= 1e-5 * ref + 1e-30).all())
    assert right == (other_cache and other_stream)


def test_window_score_reuses_statistics_of_cut_units():
    # a cut unit's (max, sum) come from the workgroup that merges it: same score as without the record
    st, K, V, q, kn, vn = _attend_state("bf16", 128, 7, [1000, 700], 1056, 512, seed=9)
    st.ctx = type(st.ctx)(make_config(1, 2, 14, 2, 128, 512, 16, 96, 1056, "bf16"))
    st.cfg = st.ctx.cfg
    st.workspace = torch.zeros(st.ctx.workspace_bytes(), dtype=torch.uint8, device="cuda")
    st.ctx.workspace_init(st.workspace)
    st.qwin = torch.zeros(16, 1, 2, 14, 128, dtype=torch.bfloat16, device="cuda")
    st.K.nan_to_num_(); st.V.nan_to_num_()
    for k in range(16):
        st.ctx.attend_decode((q * (1 + k / 16)).cuda(), kn.cuda(), vn.cuda(), st.K, st.V, st.pos, 5 + k, st.qwin, st.d_state,
                             1000 + k, st.out, st.workspace)
    S = []
    for reuse in (1, 0):
        st.ctx.set_param("score_reuse_stats", reuse)
        st.S.zero_()
        st.ctx.score_window(st.qwin, st.K, st.d_state, 20, 1016, st.S, st.workspace)
        S.append(st.S.double().cpu().numpy().copy())
    assert (S[0][..., :700] > 0).all()
    np.testing.assert_allclose(S[0], S[1], rtol=3e-6, atol=1e-30)


@pytest.mark.parametrize("g,w,rows,d", [(7, 16, 1690, 128), (8, 16, 1650, 128), (3, 32, 1681, 128), (5, 32, 1690, 128),
                                        (7, 16, 1690, 64), (5, 32, 1650, 64)])
def test_window_score_of_keys_beyond_the_cache(g, w, rows, d):
    # more than 256 MiB of K: up to 8 blocks of window rows keep three tiles in turn, 10 keep two; a launch of one sequence
    # (two tiles, cut into key shares) gives the same scores up to the statistics' last bits
    cap, B, hkv = 1696, 160 * 128 // d, 4
    gen = torch.Generator(device="cuda").manual_seed(g)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda").to(torch.bfloat16)
    K, q, kn = rnd(1, B, hkv, cap, d), rnd(w, 1, B, g * hkv, d), rnd(w, 1, B, hkv, d)
    assert B * hkv * rows * 2 * d > 256 << 20
    out = []
    for part in (slice(0, B), slice(3, 4), slice(B - 1, B)):
        st = DecodeState(make_config(1, part.stop - part.start, g * hkv, hkv, d, 1600, w, 96, cap, "bf16"))
        st.K.copy_(K[:, part])
        st.d_state.copy_(torch.tensor([rows - w, 5, 0, 1600], dtype=torch.int32).expand(1, part.stop - part.start, 4))
        for k in range(w):
            st.ctx.attend_decode(q[k][:, part].contiguous(), kn[k][:, part].contiguous(), kn[k][:, part].contiguous(), st.K, st.V,
                                 st.pos, 5 + k, st.qwin, st.d_state, rows - w + k, st.out, st.workspace)
        st.ctx.score_window(st.qwin, st.K, st.d_state, 5 + w - 1, rows, st.S, st.workspace)
        out.append(st.S[0, ..., : rows - w].double().cpu().numpy())
    assert (out[0] > 0).all()
    np.testing.assert_allclose(out[0][3], out[1][0], rtol=3e-6, atol=1e-30)
    np.testing.assert_allclose(out[0][B - 1], out[2][0], rtol=3e-6, atol=1e-30)


# ---- redundancy score in 64 bits ----------------------------------------------------------------
# n_recent at least the window, 4: several workgroups share a unit's columns (bf16, d = 128: from a capacity of 448)
@pytest.mark.parametrize("n_recent,cap", [(3, 288), (5, 288), (3, 480), (5, 480)])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
def test_redundancy_at_tile_edges(dtype, d, n_recent, cap):
    # lengths around tile borders and one tile per wavefront, both K formats; keys in clusters so that
    # cosines lie on both sides of the threshold and none near it
    w, b = 4, 20
    lens = [21, 31, 32, 33, 128, 129, 257, cap]
    B = len(lens)
    st = DecodeState(make_config(1, B, 2, 1, d, b, w, 8, cap, dtype))
    rng = np.random.default_rng(d)
    centres = rng.standard_normal((6, d))
    K = torch.full((1, B, 1, cap, d), float("nan")).to(st.K.dtype)
    for i, n in enumerate(lens):
        rows = centres[rng.integers(0, 6, n)] + 0.05 * rng.standard_normal((n, d))
        K[0, i, 0, :n] = torch.from_numpy(rows * rng.uniform(0.5, 20, (n, 1))).to(st.K.dtype)
    n_tiled = [0, 16, 32, 16, 64, 128, 240, 288]
    for i in range(B):
        st.K[0, i] = k_rows_to_cache(K[0, i], n_tiled[i]).cuda()
    st.d_state.copy_(torch.tensor([[[n - w, 100 - w, 0, min(m, (n - w) // 16 * 16)] for n, m in zip(lens, n_tiled)]],
                                  dtype=torch.int32))
    for i in range(B):                                     # the record's tiled prefix, not more
        m = min(n_tiled[i], (lens[i] - w) // 16 * 16)
        st.K[0, i] = k_rows_to_cache(K[0, i], m).cuda()
    st.F.fill_(0.25)
    st.len_host = cap
    st.redundancy_combine(99, lam=0.5, tau=0.5, n_recent=n_recent)
    R, Fs = st.R.double().cpu().numpy(), st.F_sel.double().cpu().numpy()
    for i, n in enumerate(lens):
        Kn = K[0, i, :, :n].double().numpy()
        Rr = O.redundancy_score(Kn, n, tau=0.5, n_recent=n_recent, eps=float(np.float32(1e-8)))
        ref = Rr / Rr.max()
        # R' = exp(col - max): fp64 sums give fp32 rounding, the fp32 products of bf16 d = 128 the stated 1e-5
        rel = 1e-5 if (dtype, d) == ("bf16", 128) else 1e-6
        np.testing.assert_allclose(R[0, i, 0, :n], ref[0], rtol=rel, atol=1e-40)
        # half of R' <= 1 with that error, and two roundings of numbers below 1
        np.testing.assert_allclose(Fs[0, i, 0, : n - w], 0.125 - 0.5 * ref[0, : n - w], rtol=0, atol=0.5 * rel + 1.2e-7)


@pytest.mark.parametrize("n_recent", [3, 4])
@pytest.mark.parametrize("n", [33, 97, 288])
def test_redundancy_of_keys_of_any_norm(n, n_recent):
    # bf16 at d = 128 scales by 2^80 what it compares, and serves units with norms outside 1e-9 .. 1e13 in other ways:
    # unit 0 has neither, 1 a tiny key, 2 a huge one, 3 an infinite one, which counts for nobody else
    w, b, cap, d = 4, 20, 288, 128
    st = DecodeState(make_config(1, 4, 2, 1, d, b, w, 8, cap, "bf16"))
    rng = np.random.default_rng(n)
    centres = rng.standard_normal((6, d))
    K = torch.full((1, 4, 1, cap, d), float("nan")).to(st.K.dtype)
    for i, factor in enumerate([1e3, 1e-13, 1e16, float("inf")]):
        rows = centres[rng.integers(0, 6, n)] + 0.05 * rng.standard_normal((n, d))
        rows[:: 5] *= 1e-8 if i == 0 else 1.0
        rows[n // 2] *= factor
        K[0, i, 0, :n] = torch.from_numpy(rows).to(st.K.dtype)
    st.K.copy_(K)
    st.d_state.copy_(torch.tensor([[[n - w, 100 - w, 0, 0]]], dtype=torch.int32).expand(1, 4, 4))
    st.len_host = cap
    st.redundancy_combine(99, lam=0.5, tau=0.5, n_recent=n_recent, eps=0.0)
    R = st.R.double().cpu().numpy()
    for i in range(4):
        rest = np.delete(np.arange(n), n // 2) if i == 3 else np.arange(n)
        Rr = O.redundancy_score(K[0, i, :, rest].double().numpy(), len(rest), tau=0.5, n_recent=n_recent, eps=0.0)
        np.testing.assert_allclose(R[0, i, 0, rest], (Rr / Rr.max())[0], rtol=1e-5, atol=1e-40)


@pytest.mark.parametrize("n_recent", [3, 4])
@pytest.mark.parametrize("n", [97, 450])
def test_redundancy_scale_of_a_unit(n, n_recent):
    # bf16 at d = 128: units within the common scale's norms (0), with a scale of their own (1 to 5: all keys large or
    # small, one of them, both ends of the span), and beyond it (6, 7: by comparisons)
    w, b, cap, d = 4, 20, 480, 128
    units = [(1.0, 1.0), (1e15, 1.0), (1e-11, 1.0), (1.0, 3e14), (1.0, 1e-11), (1e-9, 3e14), (1e-15, 1.0), (1.0, 1e-16)]
    st = DecodeState(make_config(1, len(units), 2, 1, d, b, w, 8, cap, "bf16"))
    rng = np.random.default_rng(n)
    centres = rng.standard_normal((6, d))
    K = torch.full((1, len(units), 1, cap, d), float("nan")).to(st.K.dtype)
    for i, (every, one) in enumerate(units):
        rows = every * (centres[rng.integers(0, 6, n)] + 0.05 * rng.standard_normal((n, d)))
        rows[n // 2] *= one
        K[0, i, 0, :n] = torch.from_numpy(rows).to(st.K.dtype)
    st.K.copy_(K)
    st.d_state.copy_(torch.tensor([[[n - w, 100 - w, 0, 0]]], dtype=torch.int32).expand(1, len(units), 4))
    st.len_host = cap
    st.redundancy_combine(99, lam=0.5, tau=0.5, n_recent=n_recent, eps=0.0)
    R = st.R.double().cpu().numpy()
    for i in range(len(units)):
        Rr = O.redundancy_score(K[0, i, :, :n].double().numpy(), n, tau=0.5, n_recent=n_recent, eps=0.0)
        np.testing.assert_allclose(R[0, i, 0, :n], (Rr / Rr.max())[0], rtol=1e-5, atol=1e-40)


# 2, 64, 66, 128 and 130 units: fp64 shares columns up to 128; bf16 from 448 rows on up to 64 units, from 704 on up to 128
@pytest.mark.parametrize("B,cap", [(1, 384), (64, 384), (65, 384), (1, 416), (1, 448), (32, 448), (33, 448), (33, 672), (33, 704),
                                   (64, 704), (65, 704)])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 128)])
def test_redundancy_leaves_what_is_not_its_own(dtype, d, B, cap):
    # sums of shared columns travel in the results' places: behind the candidates F_sel, and behind the rows R', stay as they
    # were, sequences that are not compressed keep both, and results in one buffer come out as they always have
    w, b, n = 8, cap - 84, cap - 54
    st = DecodeState(make_config(1, B, 2, 2, d, b, w, 16, cap, dtype))
    gen = torch.Generator().manual_seed(d)
    st.K.copy_(torch.randn(st.K.shape, generator=gen)); st.F.copy_(torch.rand(st.F.shape, generator=gen))
    rec = torch.tensor([n - w, 100 - w, 0, 0], dtype=torch.int32).repeat(1, B, 1)
    if B > 1:
        rec[0, 1, 0] = b - w                               # at the budget
    st.d_state.copy_(rec)
    st.len_host = cap
    out = {}
    for n_recent in (w, w - 1):                            # w - 1: a workgroup per unit
        st.R.fill_(7.0); st.F_sel.fill_(9.0)
        st.redundancy_combine(99, lam=0.5, tau=0.3, n_recent=n_recent)
        assert (st.R[..., n:] == 7).all() and (st.F_sel[..., n - w:] == 9).all()
        if B > 1:
            assert (st.R[0, 1] == 7).all() and (st.F_sel[0, 1] == 9).all()
        out[n_recent] = (st.R.clone(), st.F_sel.clone())
    st.R.fill_(7.0)
    st.ctx.redundancy_combine(st.K, st.d_state, 99, cap, st.F, 0.5, 0.3, 1e-8, w, st.R, st.R, st.workspace)
    assert torch.equal(st.R[..., : n - w][0, 0], out[w][1][..., : n - w][0, 0])
    assert torch.equal(st.R[0, 0, :, n - w:], out[w][0][0, 0, :, n - w:])
    # the columns that both leave in: the same sums, and the same maximum unless the one column more had it
    a, c = out[w][0][0, 0, :, : n - w].double(), out[w - 1][0][0, 0, :, : n - w].double()
    for x, y in zip(a, c):
        r = (x / y)[(x > 1e-30) & (y > 1e-30)]
        assert ((r / r[0] - 1).abs() < 1e-6).all()


@pytest.mark.parametrize("dtype,d,n_recent", [("bf16", 128, 8), ("bf16", 128, 7), ("f32", 64, 8)])    # two launches, one, two
def test_redundancy_timing_counts_calls(dtype, d, n_recent):
    st = DecodeState(make_config(1, 1, 2, 2, d, 400, 8, 16, 480, dtype))
    st.K.normal_()
    st.d_state.copy_(torch.tensor([450, 92, 0, 0], dtype=torch.int32).expand(1, 1, 4))
    st.len_host = 480
    st.ctx.profile_enable(True)
    for _ in range(3):
        st.redundancy_combine(99, lam=0.5, tau=0.3, n_recent=n_recent)
    ms, calls = st.ctx.profile_read("redundancy")
    assert calls == 3 and ms > 0


@pytest.mark.parametrize("dtype,d,n_recent", [("bf16", 128, 8), ("f32", 64, 8), ("bf16", 128, 7)])    # two launches, two, one
def test_redundancy_replays_in_a_graph(dtype, d, n_recent):
    w, b, cap, n = 8, 400, 480, 458
    st = DecodeState(make_config(1, 2, 2, 2, d, b, w, 16, cap, dtype))
    st.d_state.copy_(torch.tensor([n - w, 100 - w, 0, 0], dtype=torch.int32).expand(1, 2, 4))
    call = lambda: st.ctx.redundancy_combine(st.K, st.d_state, 99, cap, st.F, 0.5, 0.3, 1e-8, n_recent, st.R, st.F_sel, st.workspace)
    gen = torch.Generator().manual_seed(d)
    st.K.zero_(); st.F.zero_(); call(); torch.cuda.synchronize()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call()
    for _ in range(3):
        st.K.copy_(torch.randn(st.K.shape, generator=gen)); st.F.copy_(torch.rand(st.F.shape, generator=gen))
        call()
        torch.cuda.synchronize()
        R, F_sel = st.R.clone(), st.F_sel.clone()
        st.R.fill_(7.0); st.F_sel.fill_(9.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(st.R[..., :n], R[..., :n]) and torch.equal(st.F_sel[..., : n - w], F_sel[..., : n - w])


# ---- compaction in column shares ----------------------------------------------------------------
@pytest.mark.parametrize("dtype,d,B,b", [
    ("bf16", 128, 2, 512),        # 4 units: 4 shares, 256 threads
    ("bf16", 128, 2, 2000),       # 4 shares, 1024 threads, b not a multiple of 16 per round
    ("bf16", 128, 16, 1037),      # 32 units: 4 shares, 1024 threads, ragged b
    ("bf16", 128, 4, 560),        # 8 units: 4 shares of 35 KiB, 1024 threads
    ("bf16", 128, 33, 600),       # 66 units: 2 shares of 76 KiB, 1024 threads
    ("bf16", 64, 3, 300),         # 128-byte rows: 2 shares
    ("bf16", 96, 3, 300),         # 12 pieces a row: 2 shares (3 would be too narrow in 4)
    ("bf16", 32, 3, 300),         # 64-byte rows: whole
    ("f32", 128, 4, 700),
    ("bf16", 128, 65, 512),       # 130 units: whole
    ("bf16", 128, 65, 1500),      # more kept rows than a thread's first four
])
def test_compaction_in_shares(dtype, d, B, b):
    w, s_ = 16, 96
    cap = (b + s_ + 31) // 32 * 32
    st = DecodeState(make_config(1, B, 2, 2, d, b, w, s_, cap, dtype))
    gen = torch.Generator().manual_seed(b)
    K, V = torch.randn(st.K.shape, generator=gen).to(st.K.dtype), torch.randn(st.K.shape, generator=gen).to(st.K.dtype)
    pos = torch.randint(0, 1 << 30, (1, B, 2, cap), generator=gen, dtype=torch.int32)
    F = torch.rand(1, B, 2, cap, generator=gen)
    k, nt = b - w, b // 16 * 16
    for turn in range(2):                          # twice on the same workspace: the counters are back at zero
        l = b + 1 + (s_ - 1) * turn                # one row to drop, then s
        c = l - w
        keep = torch.rand(B, 2, c, generator=gen).topk(k, dim=-1).indices.sort(dim=-1).values
        # K's format as it stays (the shares move their own columns) and as it changes (one share moves all);
        # never past the recorded length, so on the first turn only where b is that far from its multiple of 16
        tiled = [nt if i % 2 and nt <= l - w else (l - w) // 16 * 16 if i % 3 == 0 else 32 for i in range(B)]
        assert turn == 0 or {n == nt for n in tiled} == {True, False}
        st.K.copy_(torch.stack([k_rows_to_cache(K[0, i], tiled[i]) for i in range(B)])[None])
        st.V.copy_(V); st.pos.copy_(pos); st.F.copy_(F); st.keep_idx.copy_(keep.int()[None])
        st.d_state.copy_(torch.tensor([[[l - w, 200, 0, n] for n in tiled]], dtype=torch.int32))
        if turn == 0:                              # sequence 0 is at the budget: left alone
            st.d_state[0, 0, 0] = b - w
        K0, pos0 = st.K[0, 0].clone(), st.pos[0, 0].clone()
        st.ctx.compact(st.keep_idx, st.F, st.K, st.V, st.F_hist, st.pos, st.d_state, 200 + w - 1, st.workspace)
        src = torch.cat([keep, torch.arange(c, l).expand(B, 2, w)], dim=-1)
        first = 1 if turn == 0 else 0
        if turn == 0:
            assert torch.equal(st.K[0, 0], K0) and torch.equal(st.pos[0, 0], pos0)
            assert st.d_state[0, 0].tolist() == [b - w, 200, 0, tiled[0]]
        assert (st.d_state[0, first:].cpu() == torch.tensor([b, 200 + w, k, nt], dtype=torch.int32)).all()
        rows = src[..., None].expand(B, 2, b, d)
        Kr = k_cache_to_rows(st.K[0], nt)[:, :, :b].cpu()
        assert torch.equal(Kr[first:], K[0].gather(2, rows)[first:])
        assert torch.equal(st.V[0, :, :, :b].cpu()[first:], V[0].gather(2, rows)[first:])
        assert torch.equal(st.pos[0, :, :, :b].cpu()[first:], pos[0].gather(2, src)[first:])
        assert torch.equal(st.F_hist[0, :, :, :k].cpu()[first:], F[0].gather(2, keep)[first:])


# rows whose pieces are no power of two, whole and in shares with 1024 threads; 514 units, which divide in any case, and 258 and 256
@pytest.mark.parametrize("dtype,d,B,b", [("bf16", 96, 65, 300), ("f32", 96, 4, 700), ("bf16", 48, 65, 300),
                                         ("bf16", 128, 257, 98), ("f32", 64, 257, 130), ("bf16", 128, 129, 98), ("f32", 64, 128, 130)])
def test_compaction_of_rows_that_are_no_power_of_two(dtype, d, B, b):
    test_compaction_in_shares(dtype, d, B, b)


# ---- native calls -------------------------------------------------------------------------------
def test_native_call_leaves_other_gpu_tensors_to_ctypes():
    st = DecodeState(make_config(1, 2, 4, 2, 64, 40, 8, 16, 64, "f32"))
    call = lambda F: st.ctx._call.gkv_select_topk(st.ctx._handle, F, st.d_state, 20, 64, st.keep_idx, st.workspace)
    assert call(st.F) == 0 and call(torch.nn.Parameter(st.F)) == 0
    for other in (st.F.transpose(1, 2), st.F[..., ::2], st.F.cpu(), st.F.as_subclass(type("Sub", (torch.Tensor,), {}))):
        assert call(other) is None
    with pytest.raises(ValueError):
        st.ctx.select_topk(st.F[..., ::2], st.d_state, 20, 64, st.keep_idx, st.workspace)
