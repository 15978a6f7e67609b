"""The fp32 layer over the forms its kernels branch on, against the fp64
oracle: head dims of every padded size and not a multiple of 4 or 16, widths
that are no multiple of 4, rows that are only 4-byte aligned, sequence lengths
around the 16-row query tiles and the 16-key steps of a quarter of the keys,
padding rows, cached prefixes, and row counts on both sides of the GEMM's tile
choice."""
import numpy as np
import pytest

from gpu_util import dev, host, log, rel_err, upload_weights

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    from paper_2607_14557_amd import seer
    seer.load_library()
    return seer


def _tol(d, I):
    # five chained sums (two projections, scores, the weighted sum, the MLP) of
    # at most max(d, I) fp32 terms, each within 4 sqrt(K) 2^-24 of its value
    return 5 * 4 * np.sqrt(max(d, I)) * 2.0 ** -24


SHORT = [1, 15, 16, 17, 64, 65, 130]
CASES = {
    "tiny": (256, 4, 64, 688, SHORT, 0),
    "dh32_odd_ff": (96, 3, 32, 203, SHORT, 0),
    "dh20": (40, 2, 20, 64, SHORT, 0),
    "dh10_nothing_aligned": (30, 3, 10, 37, SHORT, 0),
    "dh96": (96, 1, 96, 128, SHORT, 0),
    "dh128": (256, 2, 128, 640, [300, 1, 33], 0),
    "misaligned_rows": (256, 4, 64, 688, SHORT, 1),
    "wide_tiles": (512, 8, 64, 1376, [1500, 900, 401], 0),
    "wide_tiles_odd_ff": (256, 2, 128, 687, [1100, 1000, 900], 0),
}


def _weights(rng, d, I):
    f = lambda *s: (rng.standard_normal(s) * 0.05).astype(np.float32)
    return dict(wq=f(d, d), wk=f(d, d), wv=f(d, d), wo=f(d, d), wg=f(I, d), wu=f(I, d), wd=f(d, I),
                g1=np.ones(d, np.float32), g2=np.ones(d, np.float32))


def _setup(S, name, rng):
    import torch
    from paper_2607_14557_amd.runner import dims_for
    d, H, dh, I, lens, shift = CASES[name]
    W = _weights(rng, d, I)
    dims = dims_for(d, H, dh, I, "f32")
    packed = torch.empty(S.seer_prepacked_bytes(dims), dtype=torch.uint8, device="cuda")
    S.seer_prepack_weights(dims, upload_weights(W, "f32"), packed)
    cu = np.concatenate([[0], np.cumsum(lens)])
    T = int(cu[-1])
    x = rng.standard_normal((T, d)).astype(np.float32)
    rows = lambda: torch.zeros(T * d + shift, dtype=torch.float32, device="cuda")[shift:].view(T, d)
    xd = rows()
    xd.copy_(torch.from_numpy(x))
    ws = torch.empty(S.seer_layer_workspace_bytes(dims, T), dtype=torch.uint8, device="cuda")
    used = np.array([max(0, n - (i % 3)) for i, n in enumerate(lens)])
    return d, H, I, lens, W, dims, packed, cu, T, x, xd, rows(), ws, used


@pytest.mark.parametrize("name", list(CASES))
def test_layer_forms(S, name):
    from oracle.layer import layer_forward
    rng = np.random.default_rng(11)
    d, H, I, lens, W, dims, packed, cu, T, x, xd, y, ws, used = _setup(S, name, rng)
    log("fp32 layer %s: d %d, %d heads, d_ff %d, %d rows" % (name, d, H, I, T))
    S.seer_layer_forward_varlen(dims, packed, xd, y, T, dev(cu), dev(used), len(lens), 0.0, None, ws)
    ref, _ = layer_forward(x, cu, W, H, 1e-5, seqused=used)
    e = rel_err(host(y), ref)
    log("  rel err %.2e" % e)
    assert e <= _tol(d, I)


@pytest.mark.parametrize("name,prefix", [("tiny", [0, 1, 16, 37, 5, 200, 64]), ("dh10_nothing_aligned", [3, 0, 40, 1, 17, 9, 2]),
                                         ("dh128", [129, 4, 0])])
def test_cached_forms(S, name, prefix):
    import torch
    from oracle.kvcache import layer_forward_cached
    rng = np.random.default_rng(12)
    d, H, I, lens, W, dims, packed, cu, T, x, xd, y, ws, used = _setup(S, name, rng)
    cu_kv = np.concatenate([[0], np.cumsum(prefix)])
    kv = rng.standard_normal((int(cu_kv[-1]), 2 * d)).astype(np.float32)
    log("fp32 cached layer %s: prefixes %s" % (name, prefix))
    S.seer_layer_forward_cached(dims, packed, xd, y, T, dev(cu), dev(used), len(lens), torch.from_numpy(kv).cuda(),
                                dev(cu_kv), int(cu_kv[-1]), ws)
    pre = [(kv[cu_kv[b]:cu_kv[b + 1], :d], kv[cu_kv[b]:cu_kv[b + 1], d:]) for b in range(len(lens))]
    ref = layer_forward_cached(x, cu, pre, W, H, 1e-5, seqused=used)
    e = rel_err(host(y), ref)
    log("  rel err %.2e" % e)
    assert e <= _tol(d, I)
