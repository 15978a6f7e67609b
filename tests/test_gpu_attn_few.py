"""Attention of few query tiles (32 queries a workgroup, the keys split over its
waves) and the form that larger bounds take, over the same sequences: the output
that a layer call leaves in its workspace against float64 attention of the q, k
and v that it left there.  Lengths around the 32-query tiles and the 32 keys of
a wave, padding rows, sequences without keys, cached prefixes whose end is no
multiple of 4, scores that rise past the fp16 range of the first tile's
reference maximum in keys of every wave, and infinite ones."""
import numpy as np
import pytest

from gpu_util import dev, log, view_ws

pytestmark = pytest.mark.gpu

LENS = [1, 31, 32, 33, 64, 65, 97, 128, 129, 300, 40]
FORMS = {
    # heads, lengths, used (None: all), cached prefixes (None: no cache), factor of the q and k projections
    "own": (2, LENS, None, None, 1.0),
    "padded": (2, LENS, [0, 1, 32, 30, 33, 64, 96, 127, 128, 200, 0], None, 1.0),
    "prefix": (2, LENS, None, [0, 1, 2, 3, 31, 32, 33, 95, 127, 130, 401], 1.0),
    "prefix_padded": (2, LENS, [0, 1, 32, 30, 33, 64, 96, 127, 128, 200, 0], [5, 0, 97, 3, 31, 64, 1, 128, 6, 401, 0], 1.0),
    "rising": (2, [700], None, None, 6.0),
    "one_row": (4, [1], None, [793], 1.0),
}


@pytest.fixture(scope="module")
def S():
    from paper_2607_14557_amd import seer
    seer.load_library()
    return seer


@pytest.mark.parametrize("bound", ["few", "many"])
@pytest.mark.parametrize("name", list(FORMS))
def test_attention_forms(S, name, bound):
    import torch
    from paper_2607_14557_amd.runner import SeerStack, dims_for
    H, lens, used, prefix, factor = FORMS[name]
    d, T, B = 128 * H, sum(lens), len(lens)
    d, I = max(d, 256), 256
    H = d // 128
    # the rule sees the bounds: one round of 32-query tiles and 320 keys a sequence, or several rounds
    ub = max(T + 7, 320 * B) if bound == "few" else 128 * 128 // H + 128 + T
    assert (((ub - B) // 32 + B) * H <= 256) == (bound == "few")
    log("attention %s, %s tiles: %d heads, %d rows, bound %d" % (name, bound, H, T, ub))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    f = lambda *s: (torch.randn(*s, device="cuda", generator=gen) * 0.06).bfloat16()
    W = dict(wq=f(d, d), wk=f(d, d), wv=f(d, d), wo=f(d, d), wg=f(I, d), wu=f(I, d), wd=f(d, I),
             g1=torch.ones(d, device="cuda"), g2=torch.ones(d, device="cuda"))
    for n in ("wq", "wk"):
        W[n] = (W[n].float() * factor).bfloat16()
    st = SeerStack(dims_for(d, H, 128, I, "bf16"), 1, ub)
    st.set_layer(0, W)
    x = torch.randn(ub, d, device="cuda", generator=gen).bfloat16()
    cu = np.concatenate([[0], np.cumsum(lens)])
    un = np.array(used if used else lens)
    y = torch.empty_like(x)
    cu_kv = np.concatenate([[0], np.cumsum(prefix)]) if prefix else None
    if prefix:
        n = int(cu_kv[-1])
        kv = torch.cat([f(n, d) * 16, (f(n, d) * 16).to(torch.float16).view(torch.bfloat16)], dim=1).contiguous()
        S.seer_layer_forward_cached(st.dims, st.packed[0], x, y, ub, dev(cu), dev(un), B, kv, dev(cu_kv), n,
                                    st.workspace)
    else:
        st.layer(0, x, y, dev(cu), dev(un), B, ub)
    torch.cuda.synchronize()
    off = S.seer_layer_workspace_offsets(st.dims, ub)
    qkv = view_ws(st.workspace, off[0], ub, 3 * d, "bf16")[:T].contiguous()
    o = view_ws(st.workspace, off[1], ub, d, "bf16")[:T].double()
    q, k, v = qkv[:, :d].double(), qkv[:, d:2 * d].double(), qkv.view(torch.float16)[:, 2 * d:].double()
    worst = 0.0
    rise = []
    for b in range(B):
        r, u = slice(int(cu[b]), int(cu[b + 1])), slice(int(cu[b]), int(cu[b]) + int(un[b]))
        assert bool((o[u.stop:r.stop] == 0).all()), "padding rows of sequence %d" % b
        if un[b] == 0:
            continue
        kb, vb = k[u], v[u]
        if prefix:
            c = slice(int(cu_kv[b]), int(cu_kv[b + 1]))
            kb = torch.cat([kv[c, :d].double(), kb])
            vb = torch.cat([kv.view(torch.float16)[c, d:].double(), vb])
        for h in range(H):
            s = slice(128 * h, 128 * h + 128)
            z = q[u, s] @ kb[:, s].t().contiguous() / 128 ** 0.5
            if factor != 1.0:
                # log2 units by which the keys of each wave exceed the first reference (the first 64 keys' maximum)
                top = z * 1.4427 - z[:, :64].amax(dim=1, keepdim=True) * 1.4427
                rise.append(torch.stack([top[:, [i for i in range(64, top.shape[1]) if i % 128 // 32 == w]].amax(dim=1)
                                         for w in range(4)], dim=1))
            pr = torch.softmax(z, dim=1)
            ref, mag = pr @ vb[:, s].contiguous(), pr @ vb[:, s].abs().contiguous()
            # half an ulp of the bf16 output; an fp16 rounding of each probability and of their sum (2^-11 each,
            # and 2^-25 a key for those below fp16's normal range); fp32 scores of 128 terms in the exponent
            zmag = (q[u, s].abs() @ kb[:, s].abs().t().contiguous()).amax(dim=1, keepdim=True) / 128 ** 0.5
            tol = 2.0 ** -8 * ref.abs() + mag * (2.0 ** -10 + 8 * zmag * 2.0 ** -24) \
                + kb.shape[0] * 2.0 ** -25 * vb[:, s].abs().amax() + 1e-30
            worst = max(worst, ((o[u, s] - ref).abs() / tol).max().item())
    log("  largest error over its bound: %.2f" % worst)
    assert worst <= 1.0
    if rise:
        share = (torch.cat(rise) > 16).double().mean(dim=0)
        log("  keys more than 16 log2 units above the first reference, by wave: %s" % share.tolist())
        assert bool((share > 0.3).all()), "the case does not move the reference maximum in every wave"


@pytest.mark.parametrize("bound", ["few", "many"])
def test_infinite_scores(S, bound):
    """Cached keys whose first 32 have minus infinity in one dim: where the query is positive there, their scores are
    minus infinity and they weigh nothing beside the other keys, of the same 64-key tile and of later ones; where it is
    negative the scores are plus infinity and the output is NaN, as softmax's is."""
    import torch
    from paper_2607_14557_amd.runner import SeerStack, dims_for
    H, T, n = 2, 40, 420
    d, I = 256, 256
    ub = T + 7 if bound == "few" else 128 * 128 // H + 128 + T
    assert ((ub - 1) // 32 + 1) * H <= 256 or bound == "many"
    log("attention with infinite scores, %s tiles" % bound)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9)
    f = lambda *s: (torch.randn(*s, device="cuda", generator=gen) * 0.06).bfloat16()
    W = dict(wq=f(d, d), wk=f(d, d), wv=f(d, d), wo=f(d, d), wg=f(I, d), wu=f(I, d), wd=f(d, I),
             g1=torch.ones(d, device="cuda"), g2=torch.ones(d, device="cuda"))
    st = SeerStack(dims_for(d, H, 128, I, "bf16"), 1, ub)
    st.set_layer(0, W)
    x = torch.randn(ub, d, device="cuda", generator=gen).bfloat16()
    kv = torch.cat([f(n, d) * 16, (f(n, d) * 16).to(torch.float16).view(torch.bfloat16)], dim=1).contiguous()
    kv[:32, :d] = 0
    kv[:32, 0:d:128] = float("-inf")
    y = torch.empty_like(x)
    S.seer_layer_forward_cached(st.dims, st.packed[0], x, y, ub, dev(np.array([0, T])), None, 1, kv,
                                dev(np.array([0, n])), n, st.workspace)
    torch.cuda.synchronize()
    off = S.seer_layer_workspace_offsets(st.dims, ub)
    qkv = view_ws(st.workspace, off[0], ub, 3 * d, "bf16")[:T].contiguous()
    o = view_ws(st.workspace, off[1], ub, d, "bf16")[:T].double()
    q = qkv[:, :d].double()
    k = torch.cat([kv[32:, :d].double(), qkv[:, d:2 * d].double()])
    v = torch.cat([kv.view(torch.float16)[32:, d:].double(), qkv.view(torch.float16)[:, 2 * d:].double()])
    for h in range(H):
        s = slice(128 * h, 128 * h + 128)
        good = q[:, 128 * h] > 0
        assert 5 < int(good.sum()) < T - 5
        assert bool(torch.isnan(o[~good][:, s]).all()), "head %d: a score of plus infinity" % h
        pr = torch.softmax(q[good][:, s] @ k[:, s].t().contiguous() / 128 ** 0.5, dim=1)
        ref, mag = pr @ v[:, s].contiguous(), pr @ v[:, s].abs().contiguous()
        # half an ulp of the bf16 output, fp16 roundings of the probabilities and their sum, fp32 sums in the exponent
        err = (o[good][:, s] - ref).abs() / (2.0 ** -8 * ref.abs() + 2.0 ** -9 * mag)
        assert bool((err <= 1.0).all()), "head %d: %.2f of the bound" % (h, err.max().item())
