"""The causal forward of a few short sequences, which goes by definition in one launch (fwd_direct_kernel in
csrc/la_block.h): edges of its blocks, the most and the fewest workgroups it takes, all element types and layouts.

Tolerances, max-norm relative.  fp32: scores, their sums and the products with V are exact to 2^-23 each and at most
256 terms are added, in 32-token blocks and then over up to 8 blocks: 1e-5 for O (as for the workgroup kernels), and for
den 1e-6 of the sum of its terms' sizes (den itself but for the polynomial map, whose features have signs and cancel:
each is rounded, 2^-24, before its product is).  bf16 tensors: the result rounded to 8 bits, 2^-9, and scores of 16 bits
against V, 2^-17 per term: 3e-3; den is formed from three-part operands as for fp32 tensors, 1e-6."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_util import DEV, maybe_bf16, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu


def forward(la, dev, eps, features, token_major=False, ws_bytes=0):
    q, k, v = (x.transpose(1, 2).contiguous() for x in dev) if token_major else dev
    B, H, N = dev[0].shape[:3]
    O = torch.full_like(v, float("nan"))
    den = torch.full((B, H, N), float("nan"), device=DEV)
    ws = torch.zeros(max(ws_bytes, 16), dtype=torch.uint8, device=DEV)
    (la.la_causal_fwd_bnhd if token_major else la.la_causal_fwd)(q, k, v, O, den, eps, ws=ws, features=features)
    torch.cuda.synchronize()
    return to_host(O.transpose(1, 2) if token_major else O), den.cpu().numpy(), ws.cpu().numpy()


@pytest.mark.parametrize("kind", ["f32", "bf16", "given", "poly2"])
@pytest.mark.parametrize("D,M", [(64, 64), (32, 32), (64, 32), (32, 64)])
@pytest.mark.parametrize("B,H,N", [(1, 1, 33), (1, 3, 64), (1, 1, 65), (2, 3, 97), (1, 3, 160), (1, 5, 255), (1, 1, 256), (4, 8, 256),
                                   (3, 11, 256)])
def test_short_forward(oracle, monkeypatch, B, H, N, D, M, kind):
    import paper_2006_16236_amd as la
    if kind == "poly2" and D != 64:
        pytest.skip("the polynomial map has 64 features")
    bf16, eps = kind == "bf16", 0.5 if kind == "poly2" else 1e-6
    q, k, v, _ = maybe_bf16(wl.random_case(9300 + N + D + 2 * M, B, H, N, D, M), bf16)
    if kind == "given":
        q, k = (np.where(x > 0, x + 1, np.exp(x)).astype(np.float32) for x in (q, k))
        fq, fk = q.astype(np.float64), k.astype(np.float64)
    elif kind == "poly2":
        q, k = q[..., :8].copy(), k[..., :8].copy()
        fq, fk = ((x[..., :, None].astype(np.float64) * x[..., None, :]).reshape(*x.shape[:-1], 64) for x in (q, k))
    if kind in ("given", "poly2"):
        w = np.tril(fq @ fk.swapaxes(-1, -2))
        ref_den = w.sum(-1) + eps
        ref = (w @ v.astype(np.float64)) / ref_den[..., None]
    else:
        ref = oracle.causal_fwd_prefix(q, k, v, eps)
        fq, fk = (np.where(x > 0, x + 1.0, np.exp(np.minimum(x, 0.0))) for x in (q.astype(np.float64), k.astype(np.float64)))
        ref_den = np.tril(fq @ fk.swapaxes(-1, -2)).sum(-1) + eps
    code = {"f32": la.LA_F32, "bf16": la.LA_BF16, "given": la.LA_F32 + 2, "poly2": la.LA_F32_POLY2}[kind]
    features = {"given": True, "poly2": "poly2"}.get(kind, False)
    dev = [to_dev(x, bf16) for x in (q, k, v)]
    need = la.la_causal_fwd_workspace(B, H, N, 8 if kind == "poly2" else D, M, code)
    O, den, ws = forward(la, dev, eps, features, ws_bytes=need)
    assert rel_err(O, ref) <= (3e-3 if bf16 else 1e-5)
    sizes = np.tril(np.abs(fq) @ np.abs(fk).swapaxes(-1, -2)).sum(-1) + eps
    assert (np.abs(den - ref_den) / sizes).max() <= 1e-6
    Ot, dent, wst = forward(la, dev, eps, features, token_major=True, ws_bytes=need)
    assert np.array_equal(O, Ot) and np.array_equal(den, dent) and np.array_equal(ws, wst)
    # the states it leaves for a backward are those of the kernels that go segment by segment
    monkeypatch.setenv("LA_BLOCK_KERNELS", "1")
    la.la_tuning_reload()
    try:
        _, _, wsb = forward(la, dev, eps, features, ws_bytes=need)
    finally:
        monkeypatch.delenv("LA_BLOCK_KERNELS")
        la.la_tuning_reload()
    assert np.array_equal(ws, wsb)


@pytest.mark.parametrize("bf16", [False, True])
def test_later_tokens_do_not_reach_earlier_ones(bf16):
    import paper_2006_16236_amd as la
    q, k, v, _ = maybe_bf16(wl.random_case(9400, 1, 2, 150, 64, 64), bf16)
    O, den, _ = forward(la, [to_dev(x, bf16) for x in (q, k, v)], 1e-6, False, ws_bytes=1 << 20)
    for bad in (1e30, np.inf, np.nan):
        for t in (1, 40, 97, 149):
            x = [a.copy() for a in (q, k, v)]
            for a in x:
                a[:, :, t:] = bad
            Ob, denb, _ = forward(la, [to_dev(a, bf16) for a in x], 1e-6, False, ws_bytes=1 << 20)
            assert np.array_equal(O[:, :, :t], Ob[:, :, :t]) and np.array_equal(den[:, :, :t], denb[:, :, :t])
