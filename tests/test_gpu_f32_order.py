"""The order of the fp32 layer's sums, bit for bit: ascending in the summed
index, one fused multiply-add a term.  The near-zero count is a threshold on the
activations, so sums in another order change a count now and then.  Each
projection is held to a chain of exactly rounded fused multiply-adds over the
inputs that the call left in its workspace, the attention to inputs whose
probabilities are exactly 0 or 1, and the counts to the stored activations."""
import numpy as np
import pytest

from gpu_util import dev, log, view_ws, view_ws_f32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    from paper_2607_14557_amd import seer
    seer.load_library()
    return seer


def _fma(a, b, c):
    """fp32 a * b + c with one rounding: the float64 sum rounded to odd (its error by the two-sum), then to fp32."""
    p = a.astype(np.float64) * b.astype(np.float64)           # exact
    c = np.broadcast_to(c.astype(np.float64), p.shape)
    s = p + c
    t = s - p
    err = (p - (s - t)) + (c - t)
    even = (s.view(np.int64) & 1) == 0
    return np.where((err != 0) & even, np.nextafter(s, np.copysign(np.inf, err)), s).astype(np.float32)


def _chain(a, w):
    """a [M, K] w[N, K]^T in ascending K."""
    acc = np.zeros((a.shape[0], w.shape[0]), np.float32)
    for k in range(a.shape[1]):
        acc = _fma(a[:, k, None], w[None, :, k], acc)
    return acc


def test_the_fused_multiply_add():
    from fractions import Fraction
    rng = np.random.default_rng(0)
    a, b, c = (rng.standard_normal(400).astype(np.float32) for _ in range(3))
    c[200:] = -(a * b)[200:]                                  # cancellation
    c[:100] *= np.float32(2.0) ** rng.integers(-40, 40, 100).astype(np.float32)
    for x, y, z, r in zip(a, b, c, _fma(a, b, c)):
        exact = Fraction(float(x)) * Fraction(float(y)) + Fraction(float(z))
        near = [np.nextafter(r, np.float32(-np.inf)), np.nextafter(r, np.float32(np.inf))]
        d = abs(Fraction(float(r)) - exact)
        assert all(d <= abs(Fraction(float(n)) - exact) for n in near)


# d, heads, d_ff, sequence lengths, floats by which the rows are shifted off 16-byte alignment
FORMS = {
    "small_tiles": (96, 3, 204, [1, 15, 16, 17, 64, 65, 130], 0),
    "odd_widths": (30, 3, 37, [1, 15, 16, 17, 64, 65, 130], 0),
    "misaligned": (96, 3, 203, [300, 8], 1),
    "wide_tiles": (256, 4, 688, [1500, 900, 401], 0),
    "wide_tiles_odd": (128, 2, 687, [1100, 1000, 900], 0),
}


@pytest.mark.parametrize("name", list(FORMS))
def test_projections_and_counts(S, name):
    import torch
    from paper_2607_14557_amd.runner import SeerStack, dims_for
    d, H, I, lens, shift = FORMS[name]
    rng = np.random.default_rng(3)
    T = sum(lens)
    log("fp32 sums in order, %s: d %d, d_ff %d, %d rows" % (name, d, I, T))
    f = lambda *s: rng.standard_normal(s).astype(np.float32) * np.float32(0.1)
    W = dict(wq=f(d, d), wk=f(d, d), wv=f(d, d), wo=f(d, d), wg=f(I, d), wu=f(I, d), wd=f(d, I))
    st = SeerStack(dims_for(d, H, d // H, I, "f32"), 1, T)
    ones = torch.ones(d, device="cuda")
    st.set_layer(0, dict({k: torch.from_numpy(w).cuda() for k, w in W.items()}, g1=ones, g2=ones))
    rows = lambda: torch.zeros(T * d + shift, device="cuda")[shift:].view(T, d)
    x, y = rows(), rows()
    x.copy_(torch.from_numpy(rng.standard_normal((T, d)).astype(np.float32)))
    cu = np.concatenate([[0], np.cumsum(lens)])
    cnt = torch.full((T,), -1, dtype=torch.int32, device="cuda")
    eps = 0.01 * 0.1 * 0.1 * d
    st.layer(0, x, y, dev(cu), None, len(lens), T, act_eps=eps, act_count=cnt)
    torch.cuda.synchronize()
    off = S.seer_layer_workspace_offsets(st.dims, T)
    part = lambda k, cols: view_ws(st.workspace, off[k], T, cols, "f32").cpu().numpy()
    qkv, o, h1, act = part(0, 3 * d), part(1, d), part(2, d), part(3, I)
    inv1, inv2 = (view_ws_f32(st.workspace, off[k], T).cpu().numpy()[:, None] for k in (4, 5))
    x, y = x.cpu().numpy(), y.cpu().numpy()
    r = np.unique(np.r_[0:8, T // 2:T // 2 + 8, T - 24:T])    # rows of the first, a middle and the last tiles
    assert np.array_equal(qkv[r], _chain(x[r], np.concatenate([W["wq"], W["wk"], W["wv"]])) * inv1[r]), "q, k, v"
    assert np.array_equal(h1[r], x[r] + _chain(o[r], W["wo"])), "output projection"
    assert np.array_equal(y[r], h1[r] + _chain(act[r], W["wd"])), "down projection"
    n = (np.abs(act) < np.float32(eps)).sum(axis=1)
    assert n.max() > 0 and np.array_equal(cnt.cpu().numpy(), n), "counts"
    # a gate above 104 has exp(-gate) = 0, so its silu is the gate itself
    W["wg"], W["wo"] = np.abs(W["wg"]) * np.float32(1000), np.zeros((d, d), np.float32)
    st.set_layer(0, dict({k: torch.from_numpy(w).cuda() for k, w in W.items()}, g1=ones, g2=ones))
    xd = rows()
    xd.copy_(torch.from_numpy(np.abs(x)))
    st.layer(0, xd, rows(), dev(cu), None, len(lens), T)
    torch.cuda.synchronize()
    h1, act, inv2 = part(2, d), part(3, I), view_ws_f32(st.workspace, off[5], T).cpu().numpy()[:, None]
    assert np.array_equal(h1, np.abs(x))
    g = _chain(h1[r], W["wg"]) * inv2[r]
    assert g.min() > 104
    assert np.array_equal(act[r], g * (_chain(h1[r], W["wu"]) * inv2[r])), "gate and up projections"


@pytest.mark.parametrize("hd,heads", [(64, 2), (32, 3), (20, 2), (10, 3), (96, 1), (128, 2), (5, 2)])
def test_attention_sums(S, hd, heads):
    """Cached keys r e_0 with r one of a few multiples of 8192 and own keys 0: a score is at the running maximum or
    hundreds below it, so a probability is 1 or 0 and the factor of the sums before a raised maximum 0.  Queries of
    both signs in one tile of 16 raise it at different keys."""
    import torch
    from paper_2607_14557_amd.runner import SeerStack, dims_for
    d, I = hd * heads, 16
    lens, prefix = [5, 33, 18, 40, 16], [300, 0, 17, 513, 256]
    B, T, n_kv = len(lens), sum(lens), sum(prefix)
    log("fp32 attention sums in order: %d heads of %d, prefixes %s" % (heads, hd, prefix))
    rng = np.random.default_rng(hd)
    f = lambda *s: rng.standard_normal(s).astype(np.float32)
    W = {k: np.zeros((d, d), np.float32) for k in ("wq", "wk", "wv", "wo")}
    for h in range(heads):
        W["wq"][h * hd, 0] = 1.0
    W.update(wv=f(d, d), wg=f(I, d), wu=f(I, d), wd=f(d, I))
    st = SeerStack(dims_for(d, heads, hd, I, "f32"), 1, T)
    ones = torch.ones(d, device="cuda")
    st.set_layer(0, dict({k: torch.from_numpy(w).cuda() for k, w in W.items()}, g1=ones, g2=ones))
    x = f(T, d)
    sign = rng.choice([-1.0, 1.0], T)
    x[:, 0] = 2.0 * sign
    r = rng.integers(1, 7, (n_kv, heads)) * 8192.0
    kv = np.zeros((n_kv, 2 * d), np.float32)
    kv[:, d:] = f(n_kv, d)
    for h in range(heads):
        kv[:, h * hd] = r[:, h]
    cu, ckv = (np.concatenate([[0], np.cumsum(v)]) for v in (lens, prefix))
    used = np.array([n - b % 3 for b, n in enumerate(lens)])
    y = torch.zeros(T, d, device="cuda")
    S.seer_layer_forward_cached(st.dims, st.packed[0], torch.from_numpy(x).cuda(), y, T, dev(cu), dev(used), B,
                                torch.from_numpy(kv).cuda(), dev(ckv), n_kv, st.workspace)
    torch.cuda.synchronize()
    off = S.seer_layer_workspace_offsets(st.dims, T)
    qkv = view_ws(st.workspace, off[0], T, 3 * d, "f32").cpu().numpy()
    got = view_ws(st.workspace, off[1], T, d, "f32").cpu().numpy()
    # 8192 of the score's units (|q_0| times the scale) leave exp at 0
    assert 8192 * np.abs(qkv[:, 0]).min() / np.sqrt(hd) > 104
    for b in range(B):
        for h in range(heads):
            c = slice(h * hd, (h + 1) * hd)
            v = np.concatenate([kv[ckv[b]:ckv[b + 1], d:][:, c], qkv[cu[b]:cu[b] + used[b], 2 * d:][:, c]])
            score = np.concatenate([r[ckv[b]:ckv[b + 1], h], np.zeros(used[b])])
            for sg in (-1.0, 1.0):
                top, o, n = -np.inf, None, 0
                for s, row in zip(score * sg, v):
                    if s > top:
                        top, o, n = s, row.copy(), 1
                    elif s == top:
                        o, n = o + row, n + 1
                q = np.nonzero(sign[cu[b]:cu[b] + used[b]] == sg)[0] + cu[b]
                assert np.array_equal(got[q, c], np.broadcast_to(o * (np.float32(1) / np.float32(n)), (q.size, hd))), \
                    "sequence %d, head %d, sign %d" % (b, h, sg)
        assert (got[cu[b] + used[b]:cu[b + 1]] == 0).all()
