"""The bf16 GEMMs of launches of few tiles, stage by stage: each projection of
one layer call against its float64 product of the inputs that the call itself
left in the workspace, so that a stage's error is its output rounding plus its
fp32 sums.  Row counts at the edges of the 32-row blocks and the 128-row tiles,
widths whose K is split or not, of whole and of odd runs of K tiles, and the
forms of a launch; then the detection layer's row-tile list over the same."""
import math

import numpy as np
import pytest

from gpu_util import dev, log, view_ws, view_ws_f32

pytestmark = pytest.mark.gpu

# half an ulp relative to the value: 8 significant bits (bf16), 11 (fp16); the
# pair's low part rounds a remainder of at most the first to 8 bits again
BF16, FP16 = 2.0 ** -8, 2.0 ** -11
# d_model, d_ff, rows
FORMS = [
    (256, 4096, [1, 31, 33, 128, 129, 300]),     # 128x64 tiles, the down projection's K split eight ways
    (256, 384, [97, 640]),                       # six K tiles: waves with one and with two
    (512, 1408, [338, 1110]),                    # 22 K tiles: an odd number a wave
    (512, 1024, [1024, 1110, 2700]),             # one full round of 128x64 tiles (gate/up), whole tiles beside them
    (1024, 5632, [385]),
    (4096, 12288, [97, 450, 640, 1100]),         # 128x128 tiles, split two ways (450, down); parts of 256x256 tiles
                                                 # added by a second launch (640 and 1100, down)
]


@pytest.fixture(scope="module")
def S():
    from paper_2607_14557_amd import seer
    seer.load_library()
    return seer


def _layer(S, d, I, rows_ub, seed):
    import torch
    from paper_2607_14557_amd.runner import SeerStack, dims_for
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    f = lambda *s: (torch.randn(*s, device="cuda", generator=gen) * 0.02).bfloat16()
    W = dict(wq=f(d, d), wk=f(d, d), wv=f(d, d), wo=f(d, d), wg=f(I, d), wu=f(I, d), wd=f(d, I),
             g1=torch.ones(d, device="cuda"), g2=torch.ones(d, device="cuda"))
    st = SeerStack(dims_for(d, d // 128, 128, I, "bf16"), 1, rows_ub)
    st.set_layer(0, W)
    x = torch.randn(rows_ub, d, device="cuda", generator=gen).bfloat16()
    return st, W, x


def _check(what, got, ref, unit, K):
    """Half an ulp of the stored type, and 8 sqrt(K) roundings of the fp32 sums (of terms about the row's size)."""
    rms = ref.square().mean(dim=1, keepdim=True).sqrt()
    e = ((got.double() - ref).abs() / ref.abs().maximum(rms)).max().item()
    tol = unit + 8 * math.sqrt(K) * 2.0 ** -24
    log("  %s: %.2e (bound %.2e)" % (what, e, tol))
    assert e <= tol, what


@pytest.mark.parametrize("d,I,rows", [(d, I, r) for d, I, rs in FORMS for r in rs])
def test_projections(S, d, I, rows):
    import torch
    ub = rows + 40
    log("few tiles: d %d, d_ff %d, %d rows" % (d, I, rows))
    st, W, x = _layer(S, d, I, ub, rows)
    y = torch.empty_like(x)
    for _ in range(2):                           # a second call finds the first one's arrival counts
        st.layer(0, x, y, dev(np.array([0, rows])), None, 1, ub)
    torch.cuda.synchronize()
    off = S.seer_layer_workspace_offsets(st.dims, ub)
    part = lambda k, cols: view_ws(st.workspace, off[k], ub, cols, "bf16")[:rows]
    inv1, inv2 = (view_ws_f32(st.workspace, off[k], ub)[:rows].double()[:, None] for k in (4, 5))
    W = {k: w.double().t().contiguous() for k, w in W.items() if k[0] == "w"}
    xd = x[:rows].double()
    qkv, o, h1, act, h1lo = part(0, 3 * d), part(1, d).double(), part(2, d), part(3, I).double(), part(6, d)
    a = xd * inv1
    for k, n in enumerate(("wq", "wk")):
        _check(n, qkv[:, k * d:(k + 1) * d], a @ W[n], BF16, d)
    _check("wv", qkv.contiguous().view(torch.float16)[:, 2 * d:], a @ W["wv"], FP16, d)
    pair = h1.double() + h1lo.double()
    _check("wo", pair, xd + o @ W["wo"], BF16 ** 2, d)
    m = h1.double() * inv2
    g = m @ W["wg"]
    _check("gate/up", act, g * torch.sigmoid(g) * (m @ W["wu"]), BF16, 4 * d)
    _check("wd", y[:rows], pair + act @ W["wd"], BF16, I)


@pytest.mark.parametrize("d,I,lens,off,win,spare", [
    (512, 1024, [370, 370, 370], 170, 200, 300),     # nine 128-row tiles, all listed
    (256, 4096, [370, 370, 370], 170, 200, 300),     # the same with the down projection split
    (256, 4096, [700, 300, 650], 10, 20, 300),       # split, tiles dropped
    (512, 1024, [700, 300, 1700], 10, 20, 300),
    (2048, 5632, [270, 300], 30, 20, 300),
    (4096, 12288, [600, 500], 30, 20, 300),          # 128x128 tiles in a full round and a split one
    (4096, 12288, [600, 500], 30, 20, 100),          # parts added by a second launch
])
def test_row_tile_list(S, d, I, lens, off, win, spare):
    """The detection layer with every position of the windows kept (act_eps 0): its listed tiles equal the plain
    layer's bit for bit."""
    import torch
    cu = np.concatenate([[0], np.cumsum(lens)])
    T, B = int(cu[-1]), len(lens)
    log("row-tile list: d %d, d_ff %d, rows %s, %d kept of each" % (d, I, lens, off + win))
    st, _, x = _layer(S, d, I, T + spare, T)
    cud, offd, wind = dev(cu), dev(np.full(B, off)), dev(np.full(B, win))
    ref, y = torch.empty_like(x), torch.empty_like(x)
    cnt = [torch.empty(T + spare, dtype=torch.int32, device="cuda") for _ in range(2)]
    st.layer(0, x, ref, cud, None, B, T + spare, 0.0, cnt[0])
    bnd, keep = (torch.empty(B, dtype=torch.int32, device="cuda") for _ in range(2))
    for _ in range(2):
        y.fill_(77.0)
        S.seer_layer_forward_detect(st.dims, st.packed[0], x, y, T + spare, cud, B, 0.0, cnt[1], offd, wind,
                                    S.seer_snr_params(3, 100, 3, 5, 3), bnd, keep, st.workspace, st.ws_bytes)
        torch.cuda.synchronize()
        assert bool((keep == win).all())
        live = set()
        for s in cu[:-1]:
            live.update(range(int(s) // 256, (int(s) + off + win - 1) // 256 + 1))
        for t in range(-(-T // 256)):
            r = slice(256 * t, min(256 * t + 256, T))
            if t in live:
                assert torch.equal(y[r], ref[r]), "tile %d differs" % t
            else:
                assert bool((y[r] == 77.0).all()), "tile %d was written" % t
