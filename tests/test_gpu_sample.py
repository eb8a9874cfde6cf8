"""GPU parity of sampling verification (ptd_verify_sample) against the fp64
CPU oracle, through the C ABI, on the same seeded logits, trees and uniforms.

Accepted lengths, paths and emitted tokens are integers decided by comparing
uniforms with probabilities.  The kernel computes the normalizer and the bonus
CDF from fp32 exponentials taken per block of 2048 entries and rescaled to
the row maximum (each factor within ~1.2e-7 relative: one ulp of the hardware
exp2, argument rounding compensated) summed in fp64, the oracle in fp64
throughout, so a probability or cumulative probability may differ by ~5e-7
at most.  The oracle reports, per sequence, the smallest distance of a
uniform from a boundary it was compared with (its margin).  A sequence whose
margin exceeds DELTA must equal the oracle's result exactly; one with a
smaller margin must equal it for the given uniforms, or for the same
uniforms all shifted by +DELTA or -DELTA (a decision within rounding of its
boundary going either way).
"""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu
DELTA = 6e-7


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_10661_amd as lib
    return lib


def cu(a: np.ndarray) -> torch.Tensor:
    if a.dtype == np.uint16:
        return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda().view(torch.bfloat16)
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def likely_tokens(rng, logits_f32, parent, top=3, p_random=0.2):
    """Child tokens drawn among the top few of the parent's row (so walks go
    deep), sometimes uniformly at random."""
    B, T = parent.shape
    V = logits_f32.shape[-1]
    tok = np.empty((B, T), np.int32)
    for b in range(B):
        order = np.argsort(-logits_f32[b], axis=-1, kind="stable")[:, :top]
        for i in range(T):
            if rng.random() < p_random:
                tok[b, i] = rng.integers(0, V)
            else:
                tok[b, i] = order[parent[b, i] + 1, rng.integers(0, top)]
    return tok


def sample_case(P, lg, tok, par, temp, u1, u2, tree_len=None, ld=None):
    B, T = par.shape
    al_r, an_r, ot_r, mg_r = O.verify_sample(lg, tok, par, temp, u1, u2, tree_len)
    V = lg.shape[-1]
    flat = lg.reshape(B * (T + 1), V)
    if ld is not None and ld > V:
        buf = np.zeros((B * (T + 1), ld), flat.dtype)
        buf[:, :V] = flat
        t = cu(buf)[:, :V]
    else:
        t = cu(flat)
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    al, an, ot = P.verify_sample(t, cu(tok), cu(par), temp, cu(u1), cu(u2),
                                 None if tree_len is None else cu(tree_len), dev_status=st)
    torch.cuda.synchronize()
    assert st.item() == 0
    al, an, ot = al.cpu().numpy(), an.cpu().numpy(), ot.cpu().numpy()
    lgb = lg.reshape(B, T + 1, V)
    for b in range(B):
        if al[b] == al_r[b] and np.array_equal(an[b], an_r[b]) and np.array_equal(ot[b], ot_r[b]):
            continue
        assert mg_r[b] <= DELTA, (b, "differs although every decision is %.3g from its boundary"
                                  % mg_r[b])
        ok = False
        for sgn in (1.0, -1.0):
            sl = slice(b, b + 1)
            r = O.verify_sample(lgb[sl], tok[sl], par[sl], temp,
                                np.clip(u1[sl] + sgn * DELTA, 0.0, 1.0 - 2 ** -53),
                                np.clip(u2[sl] + sgn * DELTA, 0.0, 1.0 - 2 ** -53),
                                None if tree_len is None else tree_len[sl])
            if r[0][0] == al[b] and np.array_equal(r[1][0], an[b]) and np.array_equal(r[2][0], ot[b]):
                ok = True
        assert ok, (b, al[b], al_r[b], ot[b][:al[b] + 2], ot_r[b][:al_r[b] + 2])
    return al_r, ot_r


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("temp", [0.6, 1.0, 1.7])
def test_sample_random_trees(P, dtype, temp):
    rng = np.random.default_rng(int(temp * 10) + (dtype == "bf16"))
    B, T, V = 24, 20, 1000
    par = np.stack([W.tree_uniform(rng, T)[0] for _ in range(B)])
    x = (rng.standard_normal((B, T + 1, V)) * 2.0).astype(np.float32)
    # a dominant token per row (+8 nats) so that accepted chains form
    np.put_along_axis(x, np.argmax(x, axis=-1)[..., None],
                      np.max(x, axis=-1, keepdims=True) + 8.0, axis=-1)
    lg = W.f32_to_bf16_bits(x) if dtype == "bf16" else x
    lf = W.bf16_bits_to_f32(lg) if dtype == "bf16" else lg
    tok = likely_tokens(rng, lf, par)
    al, _ = sample_case(P, lg, tok, par, temp, rng.random((B, T)), rng.random((B, T + 1)))
    assert al.max() >= 2  # the walks do go below the roots


@pytest.mark.parametrize("name", ["llama2-7b", "llama2-13b", "llama3-8b-long", "ragged-16"])
def test_sample_configs(P, name):
    w = W.make_workload(name)
    rng = np.random.default_rng(5)
    B, T = w.B, w.T
    lf = W.bf16_bits_to_f32(w.logits).reshape(B, T + 1, w.V)
    tok = likely_tokens(rng, lf, w.parent, top=2, p_random=0.1)
    for draw in range(4):  # several draws of the uniforms
        sample_case(P, w.logits.reshape(B, T + 1, w.V), tok, w.parent, 1.0, rng.random((B, T)),
                    rng.random((B, T + 1)))


@pytest.mark.parametrize("B,T", [(2, 8), (8, 63)])
def test_sample_wide_rows_f32(P, B, T):
    # fp32 rows of more than 32 statistics blocks (the walk's wave-per-row
    # forms), with few blocks per call and with many (8192 or more: the
    # wave-per-block statistics)
    rng = np.random.default_rng(11 + B)
    V = 70001
    par = np.stack([W.tree_uniform(rng, T)[0] for _ in range(B)])
    x = (rng.standard_normal((B, T + 1, V)) * 2.0).astype(np.float32)
    np.put_along_axis(x, np.argmax(x, axis=-1)[..., None],
                      np.max(x, axis=-1, keepdims=True) + 6.0, axis=-1)
    tok = likely_tokens(rng, x, par, top=2, p_random=0.1)
    sample_case(P, x, tok, par, 1.0, rng.random((B, T)), rng.random((B, T + 1)))


def test_sample_wide_star_with_duplicates(P):
    # one node with 1000 children (many rejections, repeated tokens): the
    # rejected-token bitmap and the residual CDF
    rng = np.random.default_rng(6)
    B, T, V = 4, 1000, 5000
    par = np.full((B, T), -1, np.int32)
    x = rng.standard_normal((B, T + 1, V)).astype(np.float32)
    top = np.argsort(-x[:, 0], axis=-1)[:, :50]
    tok = np.stack([top[b, rng.integers(0, 50, T)] for b in range(B)]).astype(np.int32)
    u1 = rng.uniform(0.3, 1.0, (B, T))   # mostly rejections
    sample_case(P, x, tok, par, 1.0, u1, rng.random((B, T + 1)))


def test_sample_chain_padding_and_strided_rows(P):
    rng = np.random.default_rng(7)
    B, T, V = 6, 40, 3001
    par = np.stack([W.tree_chain(T)[0]] * 3 + [W.tree_uniform(rng, T)[0] for _ in range(3)])
    x = (rng.standard_normal((B, T + 1, V)) * 3.0).astype(np.float32)
    tok = likely_tokens(rng, x, par, top=1, p_random=0.0)
    tl = np.array([T, 7, 0, T, 1, 25], np.int32)
    sample_case(P, x, tok, par, 0.8, rng.random((B, T)) * 0.5, rng.random((B, T + 1)),
                tree_len=tl, ld=V + 5)


def test_sample_single_node_and_low_temperature(P):
    rng = np.random.default_rng(8)
    B, V = 32, 777
    x = rng.standard_normal((B, 2, V)).astype(np.float32)
    par = np.full((B, 1), -1, np.int32)
    tok = np.argmax(x[:, 0], axis=-1).astype(np.int32)[:, None]
    tok[::3] = (tok[::3] + 1) % V
    sample_case(P, x, tok, par, 0.05, rng.uniform(0.01, 0.99, (B, 1)), rng.random((B, 2)))


def test_sample_bad_tree_reports(P):
    rng = np.random.default_rng(9)
    par = np.array([[-1, 0, 2, 1], [-1, -1, 0, 1]], np.int32)
    x = rng.standard_normal((2, 5, 64)).astype(np.float32)
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    al, an, ot = P.verify_sample(cu(x), cu(np.zeros((2, 4), np.int32)), cu(par), 1.0,
                                 cu(rng.random((2, 4))), cu(rng.random((2, 5))), dev_status=st)
    torch.cuda.synchronize()
    assert st.item() == 7
    assert al[0].item() == 0 and (an[0] == -1).all() and (ot[0] == -1).all()


def test_sample_deterministic(P):
    rng = np.random.default_rng(10)
    B, T, V = 8, 64, 32000
    par = np.stack([W.tree_uniform(rng, T)[0] for _ in range(B)])
    x = W.f32_to_bf16_bits(rng.standard_normal((B, T + 1, V)).astype(np.float32))
    tok = likely_tokens(rng, W.bf16_bits_to_f32(x), par)
    args = (cu(x), cu(tok), cu(par), 1.0, cu(rng.random((B, T))), cu(rng.random((B, T + 1))))
    r1 = [t.cpu() for t in P.verify_sample(*args)]
    r2 = [t.cpu() for t in P.verify_sample(*args)]
    assert all(torch.equal(a, b) for a, b in zip(r1, r2))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V", [1, 9, 2047, 2049, 4103])
@pytest.mark.parametrize("kind", ["plain", "masked", "far"])
def test_sample_odd_rows_masks_and_far_logits(P, dtype, V, kind):
    # rows that start at any element address (odd strides; block edges), masked
    # vocabulary entries (-inf and the type's lowest value, a whole block of
    # them too), and logits whose exponents leave the fp32 fast range
    rng = np.random.default_rng(V + len(kind))
    B, T = 4, 12
    par = np.stack([W.tree_uniform(rng, T)[0] for _ in range(B)])
    x = (rng.standard_normal((B, T + 1, V)) * 2.0).astype(np.float32)
    if kind == "masked" and V > 8:
        x[:, :, rng.choice(V, V // 3, replace=False)] = -np.inf
        x[:, :, rng.choice(V, V // 4, replace=False)] = np.float32(-3.3e38)
        if V > 4096:
            x[:, :, 2048:4096] = -np.inf
    if kind == "far":
        x = x * np.float32(40.0) + np.float32(3000.0)
    lg = W.f32_to_bf16_bits(x) if dtype == "bf16" else x
    lf = W.bf16_bits_to_f32(lg) if dtype == "bf16" else lg
    tok = likely_tokens(rng, lf, par, top=min(3, V))
    for ld in (None, V + 3):
        sample_case(P, lg, tok, par, 1.0, rng.random((B, T)), rng.random((B, T + 1)), ld=ld)


def low_level(P, lg, tok, par, temp, u1, u2):
    """The entry point itself on output buffers that hold -7 before the call."""
    B, T = par.shape
    V = lg.shape[-1]
    t = cu(lg.reshape(B * (T + 1), V))
    al, an, ot = (torch.full(s, -7, dtype=torch.int32, device="cuda") for s in ((B,), (B, T), (B, T + 1)))
    ws = torch.empty(P.ptd_verify_sample_workspace_bytes(B, T, V), dtype=torch.uint8, device="cuda")
    code = P.PTD_BF16 if lg.dtype == np.uint16 else P.PTD_F32
    P.ptd_verify_sample(t, code, V, V, cu(tok), cu(par), None, B, T, temp, cu(u1), cu(u2), al, an, ot,
                        ws, ws.numel())
    torch.cuda.synchronize()
    return al.cpu().numpy(), an.cpu().numpy(), ot.cpu().numpy()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T", [3, 31])  # one workgroup per block, one wave per block
@pytest.mark.parametrize("masked,temp", [(-np.inf, 1.0), (-3.3e38, 1.0), (-1.0e4, 1.0), (-np.inf, 0.01)])
def test_sample_bonus_where_a_block_lost_all_its_mass(P, dtype, T, masked, temp):
    # block 1 holds the mass of two neighbours, both drafted and rejected; what
    # rounding leaves of its sum must not draw the bonus (uniforms of 0 and near 1
    # reach it from either side): that is block 0's or block 3's only entry
    rng = np.random.default_rng(T)
    B, V = 64, 8195
    par = np.full((B, T), 0, np.int32)
    par[:, :2] = -1
    y0, y3 = 77, 3 * 2048 + 5
    x = np.full((B, T + 1, V), masked, np.float32)
    a = 2048 + 2 * rng.integers(0, 1000, B)
    base = 3.0 if temp == 1.0 else 20.0  # a reference of 4 or 2885 (outside the fast range)
    for b in range(B):
        x[b, 0, a[b]] = base + temp * rng.random()
        x[b, 0, a[b] + 1] = base + temp * rng.random()
        x[b, 0, (y0, y3)[b % 2]] = base
        x[b, 1:, y0] = 0.0
    lg = W.f32_to_bf16_bits(x) if dtype == "bf16" else x
    tok = np.full((B, T), y0 + 1, np.int32)
    tok[:, 0], tok[:, 1] = a, a + 1
    u1 = np.full((B, T), 0.999)
    for u in (0.0, 1.0 - 2.0 ** -53):
        al, an, ot = low_level(P, lg, tok, par, temp, u1, np.full((B, T + 1), u))
        assert (al == 0).all() and (an == -1).all()
        assert np.array_equal(ot[:, 0], np.where(np.arange(B) % 2, y3, y0))
        assert (ot[:, 1:] == -1).all()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_sample_every_token_rejected(P, dtype):
    # the two drafted tokens hold all the mass; the second one is accepted, or
    # (the uniform within rounding of 1) nothing is left to draw the bonus from
    rng = np.random.default_rng(12)
    B, T, V = 64, 2, 5000
    par = np.full((B, T), -1, np.int32)
    x = np.full((B, T + 1, V), -np.inf, np.float32)
    a = 2 * rng.integers(0, 2000, B)
    x[np.arange(B), 0, a] = 3.0 + rng.random(B)
    x[np.arange(B), 0, a + 1] = 3.0 + rng.random(B)
    x[:, 1:, 9] = 0.0
    lg = W.f32_to_bf16_bits(x) if dtype == "bf16" else x
    tok = np.stack([a, a + 1], 1).astype(np.int32)
    u1 = np.full((B, T), 1.0 - 2.0 ** -53)
    u2 = rng.random((B, T + 1))
    al, an, ot = low_level(P, lg, tok, par, 1.0, u1, u2)
    for b in range(B):
        if al[b] == 0:
            assert (ot[b] == -1).all() and (an[b] == -1).all()
        else:
            assert al[b] == 1 and ot[b, 1] == 9 and ot[b, 0] == tok[b, an[b, 0]]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("kind", ["plain", "masked", "far"])
def test_sample_batch_statistics_odd_rows_masks_and_far_logits(P, dtype, kind):
    # 2560 rows of 5 blocks: one wave per block.  Rows start at any element
    # address; a few entries or whole blocks are masked (-inf, the type's lowest
    # value), or a few blocks lie outside the fp32 fast range
    rng = np.random.default_rng(len(kind))
    B, T, V = 40, 63, 8195
    par = np.stack([W.tree_uniform(rng, T)[0] for _ in range(B)])
    x = (rng.standard_normal((B, T + 1, V), dtype=np.float32) * 2.0).astype(np.float32)
    np.put_along_axis(x, np.argmax(x, axis=-1)[..., None], np.max(x, axis=-1, keepdims=True) + 5.0, axis=-1)
    if kind == "masked":
        x[::2, :, rng.choice(V, 40, replace=False)] = -np.inf
        x[1::2, :, rng.choice(V, 40, replace=False)] = np.float32(-3.3e38)
        x[::3, :, 2048:4096] = -np.inf
        x[1::3, :, 6144:8195] = -np.inf
        x[2::3, :, :2048] = np.float32(-3.3e38)
    if kind == "far":
        x[::2, :, 2048:4096] += np.float32(700.0)
        x[1::2, :, 4096:6144] -= np.float32(900.0)
        x[::5] = x[::5] * np.float32(3.0) - np.float32(1500.0)
    lg = W.f32_to_bf16_bits(x) if dtype == "bf16" else x
    lf = W.bf16_bits_to_f32(lg) if dtype == "bf16" else lg
    tok = likely_tokens(rng, lf, par)
    al, _ = sample_case(P, lg, tok, par, 1.0, rng.random((B, T)), rng.random((B, T + 1)), ld=V + 2)
    assert al.max() >= 2


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,T", [(4, 12), (40, 63)])
@pytest.mark.parametrize("temp", [0.05, 0.02, 0.01, 1e-3, 1e-32])
def test_sample_low_temperatures(P, dtype, B, T, temp):
    # references far from 0; logits a few temperatures apart near the top, so that
    # the probabilities are not all 0 or 1
    rng = np.random.default_rng(B)
    V = 8195
    par = np.stack([W.tree_uniform(rng, T)[0] for _ in range(B)])
    x = (rng.standard_normal((B, T + 1, V), dtype=np.float32) * 2.0 + 10.0).astype(np.float32)
    lg = W.f32_to_bf16_bits(x) if dtype == "bf16" else x
    lf = W.bf16_bits_to_f32(lg) if dtype == "bf16" else lg
    if dtype == "f32" and temp > 1e-6:
        for j in range(4):
            y = rng.integers(0, V, (B, T + 1))
            np.put_along_axis(x, y[..., None], (24.0 - temp * rng.random((B, T + 1)) * 3)[..., None].astype(np.float32),
                              axis=-1)
    tok = likely_tokens(rng, lf, par)
    sample_case(P, lg, tok, par, temp, rng.random((B, T)), rng.random((B, T + 1)))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,T,V", [(1, 96, 128256), (2, 64, 129100), (2, 8, 151936), (1, 5, 262144), (1, 63, 131073)])
def test_sample_statistics_beyond_the_staged_and_above_64_blocks(P, dtype, B, T, V):
    # more block statistics than the walk keeps in LDS; more than 64 blocks a row,
    # the largest entries in the last ones
    rng = np.random.default_rng(V)
    par = np.stack([W.tree_uniform(rng, T)[0] for _ in range(B)])
    x = rng.standard_normal((B, T + 1, V), dtype=np.float32) * np.float32(1.4)
    hot = rng.integers(max(0, V - 2500), V, (B, T + 1, 6))
    np.put_along_axis(x, hot, (rng.random((B, T + 1, 6)) * 3 + 11.0).astype(np.float32), axis=-1)
    x[:, ::3, 100] = 14.5
    lg = W.f32_to_bf16_bits(x) if dtype == "bf16" else x
    lf = W.bf16_bits_to_f32(lg) if dtype == "bf16" else lg
    tok = likely_tokens(rng, lf, par)
    sample_case(P, lg, tok, par, 1.0, rng.random((B, T)), rng.random((B, T + 1)))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,T", [(2, 8), (40, 63)])
def test_sample_whole_rows_masked(P, dtype, B, T):
    # rows of masks alone: of the type's lowest value (every entry as likely as any
    # other), with -inf among them, with one entry above
    rng = np.random.default_rng(T)
    V = 8195
    low = np.float32(-3.3895314e38)  # the lowest bf16 value
    par = np.stack([W.tree_chain(T)[0]] * B)
    x = np.full((B, T + 1, V), low, np.float32)
    x[:, 1::3, : V // 2] = -np.inf
    x[:, 2::3, 4097] = -1.0e30
    lg = W.f32_to_bf16_bits(x) if dtype == "bf16" else x
    lf = W.bf16_bits_to_f32(lg) if dtype == "bf16" else lg
    tok = likely_tokens(rng, lf, par, top=1, p_random=0.5)
    for temp in (1.0, 0.01, 1e25):
        sample_case(P, lg, tok, par, temp, rng.random((B, T)) * 1e-4, rng.random((B, T + 1)))
