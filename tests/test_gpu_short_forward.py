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
from gpu_util import DEV, grad_errs, maybe_bf16, rel_err, schedule, to_dev, to_host, tol_for

pytestmark = pytest.mark.gpu


def forward(la, dev, eps, features, token_major=False, ws_bytes=0):
    """(O, den, workspace, launches by kernel)"""
    q, k, v = (x.transpose(1, 2).contiguous() for x in dev) if token_major else dev
    B, H, N = dev[0].shape[:3]
    O = torch.full_like(v, float("nan"))
    den = torch.full((B, H, N), float("nan"), device=DEV)
    ws = torch.zeros(max(ws_bytes, 16), dtype=torch.uint8, device=DEV)
    la.la_profile_begin()
    (la.la_causal_fwd_bnhd if token_major else la.la_causal_fwd)(q, k, v, O, den, eps, ws=ws, features=features)
    launches = {name: n for name, (_, n) in la.la_profile_end().items()}
    torch.cuda.synchronize()
    return to_host(O.transpose(1, 2) if token_major else O), den.cpu().numpy(), ws.cpu().numpy(), launches


SEG_KV, SCAN, FWD = 0, 1, 2                # la_kernel_id of include/la.h
SIZES = [(1, 1, 33), (1, 3, 64), (1, 1, 65), (2, 3, 97), (1, 3, 160), (1, 5, 255), (1, 1, 256), (4, 8, 256), (3, 11, 256)]
CASES = [(kind, D, M, *size) for kind in ("f32", "bf16", "given", "given_bf16", "poly2")
         for D, M in ((64, 64), (32, 32), (64, 32), (32, 64)) if kind != "poly2" or D == 64 for size in SIZES]


def by_definition(kind, D, B, H, N):
    """whether the plan sends a call there (tests/test_plan.py draws the same lines)"""
    return (N > 64 or (N > 32 and D == 64 and "bf16" not in kind)) and B * H * -(-N // 32) <= 256


@pytest.mark.parametrize("kind,D,M,B,H,N", CASES)
def test_short_forward(oracle, monkeypatch, B, H, N, D, M, kind):
    import paper_2006_16236_amd as la
    bf16, eps = "bf16" in kind, 0.5 if kind == "poly2" else 1e-6
    q, k, v, _ = maybe_bf16(wl.random_case(9300 + N + D + 2 * M, B, H, N, D, M), bf16)
    if kind.startswith("given"):
        q, k = (np.where(x > 0, x + 1, np.exp(x)).astype(np.float32) for x in (q, k))
        if bf16:
            q, k, v = maybe_bf16((q, k, v), True)
        fq, fk = q.astype(np.float64), k.astype(np.float64)
    elif kind == "poly2":
        q, k = q[..., :8].copy(), k[..., :8].copy()
        fq, fk = ((x[..., :, None].astype(np.float64) * x[..., None, :]).reshape(*x.shape[:-1], 64) for x in (q, k))
    if kind.startswith("given") or kind == "poly2":
        w = np.tril(fq @ fk.swapaxes(-1, -2))
        ref_den = w.sum(-1) + eps
        ref = (w @ v.astype(np.float64)) / ref_den[..., None]
    else:
        ref = oracle.causal_fwd_prefix(q, k, v, eps)
        fq, fk = (np.where(x > 0, x + 1.0, np.exp(np.minimum(x, 0.0))) for x in (q.astype(np.float64), k.astype(np.float64)))
        ref_den = np.tril(fq @ fk.swapaxes(-1, -2)).sum(-1) + eps
    code = {"f32": la.LA_F32, "bf16": la.LA_BF16, "given": la.LA_F32 + 2, "given_bf16": la.LA_BF16 + 2, "poly2": la.LA_F32_POLY2}[kind]
    features = {"given": True, "given_bf16": True, "poly2": "poly2"}.get(kind, False)
    dev = [to_dev(x, bf16) for x in (q, k, v)]
    need = la.la_causal_fwd_workspace(B, H, N, 8 if kind == "poly2" else D, M, code)
    O, den, ws, launches = forward(la, dev, eps, features, ws_bytes=need)
    assert rel_err(O, ref) <= (3e-3 if bf16 else 1e-5)
    sizes = np.tril(np.abs(fq) @ np.abs(fk).swapaxes(-1, -2)).sum(-1) + eps
    assert (np.abs(den - ref_den) / sizes).max() <= 1e-6
    Ot, dent, wst, launches_t = forward(la, dev, eps, features, token_major=True, ws_bytes=need)
    assert np.array_equal(O, Ot) and np.array_equal(den, dent) and np.array_equal(ws, wst)
    # the states it leaves for a backward are those of the kernels that go segment by segment
    monkeypatch.setenv("LA_BLOCK_KERNELS", "1")
    la.la_tuning_reload()
    try:
        _, _, wsb, launches_b = forward(la, dev, eps, features, ws_bytes=need)
    finally:
        monkeypatch.delenv("LA_BLOCK_KERNELS")
        la.la_tuning_reload()
    assert np.array_equal(ws, wsb)
    # in one launch, where those take one for the segment totals first unless there is one segment in all
    name = la.la_kernel_name
    assert launches == launches_t and launches[name(FWD)] == 1
    if by_definition(kind, D, B, H, N):
        assert name(SEG_KV) not in launches and launches_b in (launches, {**launches, name(SEG_KV): 1})
        assert name(SEG_KV) in launches_b or N <= 64
    else:
        assert launches == launches_b


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("N", [133, 256])
def test_scanned_totals(oracle, bf16, N):
    """LA_FOLD_MAX_SEGS=1: the totals that the forward leaves are scanned behind it, and a backward starts from them."""
    import paper_2006_16236_amd as la
    B, H, D, M, eps = 1, 2, 64, 64, 1e-6
    q, k, v, g = maybe_bf16(wl.random_case(9500 + N, B, H, N, D, M), bf16)
    ref, gref = oracle.causal_fwd_prefix(q, k, v, eps), oracle.causal_bwd_linear(q, k, v, g, eps)
    dq, dk, dv, dg = (to_dev(x, bf16) for x in (q, k, v, g))
    with schedule(fold_max_segs=1):
        code = la.LA_BF16 if bf16 else la.LA_F32
        O, den, ws = torch.empty_like(dv), torch.empty(B, H, N, device=DEV), torch.empty(la.la_causal_fwd_workspace(B, H, N, D, M, code), dtype=torch.uint8, device=DEV)
        la.la_profile_begin()
        la.la_causal_fwd(dq, dk, dv, O, den, eps, ws=ws)
        launches = {name: n for name, (_, n) in la.la_profile_end().items()}
        assert launches == {la.la_kernel_name(FWD): 1, la.la_kernel_name(SCAN): 1}
        grads = [torch.empty_like(x) for x in (dq, dk, dv)]
        la.la_causal_bwd(dq, dk, dv, None, den, dg, *grads, eps, fwd_ws=ws)
        torch.cuda.synchronize()
    assert rel_err(to_host(O), ref) <= tol_for(N, bf16)
    for e, name in zip(grad_errs([to_host(x) for x in grads], gref), ("dQ", "dK", "dV")):
        assert e <= tol_for(N, bf16), name


@pytest.mark.parametrize("bf16", [False, True])
def test_later_tokens_do_not_reach_earlier_ones(bf16):
    import paper_2006_16236_amd as la
    q, k, v, _ = maybe_bf16(wl.random_case(9400, 1, 2, 150, 64, 64), bf16)
    O, den, *_ = forward(la, [to_dev(x, bf16) for x in (q, k, v)], 1e-6, False, ws_bytes=1 << 20)
    for bad in (1e30, np.inf, np.nan):
        for t in (1, 40, 97, 149):
            x = [a.copy() for a in (q, k, v)]
            for a in x:
                a[:, :, t:] = bad
            Ob, denb, *_ = forward(la, [to_dev(a, bf16) for a in x], 1e-6, False, ws_bytes=1 << 20)
            assert np.array_equal(O[:, :, :t], Ob[:, :, :t]) and np.array_equal(den[:, :, :t], denb[:, :, :t])
