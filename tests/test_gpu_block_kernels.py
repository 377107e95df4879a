"""The workgroup kernels of the causal passes (32-token blocks, csrc/la_block.h): every kind of call
at the edges of their blocks, forced on and off (LA_BLOCK_KERNELS), against the oracle.

Tolerances, max-norm relative: outputs of fp32 tensors 1e-5 (every product is exact to 2^-23 and an
element is the sum of a few dozen of them per block, each rounded at 2^-24; measured 5e-7 at most).
Gradients of fp32 tensors 1e-4: grad_errs floors a tensor's scale at 1e-3 of the largest, and where dQ
and dK vanish by cancellation (N = 1) a rounding of 2^-24 of the terms that cancel counts a
thousandfold, 6e-5.  bf16 tensors: the gate of the oracle comparison everywhere else, 2e-2."""
import contextlib

import numpy as np
import pytest
import torch

import workloads as wl
from gpu_util import DEV, SCHEDULES, grad_errs, maybe_bf16, rel_err, schedule, to_dev, to_host

pytestmark = pytest.mark.gpu


@contextlib.contextmanager
def block_kernels(monkeypatch, on, sched):
    """LA_BLOCK_KERNELS is read with the schedule's own knobs"""
    import paper_2006_16236_amd as la
    monkeypatch.setenv("LA_BLOCK_KERNELS", on)
    try:
        with schedule(**SCHEDULES[sched]):
            yield la
    finally:
        monkeypatch.delenv("LA_BLOCK_KERNELS")
        la.la_tuning_reload()


def run(la, dev, eps, token_major=False, **kw):
    """forward and backward: O, den, dQ, dK, dV as [B, H, N, .] host arrays"""
    q, k, v, g = (x.transpose(1, 2).contiguous() for x in dev) if token_major else dev
    B, H, N = dev[0].shape[:3]
    O = torch.full_like(v, float("nan"))
    den = torch.full((B, H, N), float("nan"), device=DEV)
    fwd = la.la_causal_fwd_bnhd if token_major else la.la_causal_fwd
    bwd = la.la_causal_bwd_bnhd if token_major else la.la_causal_bwd
    ws = fwd(q, k, v, O, den, eps, **kw)
    grads = [torch.full_like(x, float("nan")) for x in (q, k, v)]
    bwd(q, k, v, None, den, g, *grads, eps, fwd_ws=ws, **kw)
    torch.cuda.synchronize()
    return [to_host(x.transpose(1, 2) if token_major else x) for x in (O, *grads)], den.cpu().numpy()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("D,M", [(64, 64), (32, 32), (64, 32), (32, 64)])
@pytest.mark.parametrize("N,sched", [(1, "default"), (16, "default"), (31, "default"), (32, "default"), (33, "default"),
                                     (65, "many_segments"), (255, "many_segments"), (700, "three_chunk_segments"),
                                     (1027, "default")])
def test_block_edges(oracle, monkeypatch, N, sched, D, M, bf16):
    B, H = 1, 3
    host = maybe_bf16(wl.random_case(8100 + N + D + 2 * M, B, H, N, D, M), bf16)
    ref = oracle.causal_fwd_prefix(*host[:3], 1e-6)
    gref = oracle.causal_bwd_linear(*host, 1e-6)
    dev = [to_dev(x, bf16) for x in host]
    tol = 2e-2 if bf16 else 1e-5
    got = {}
    for on in "01":
        with block_kernels(monkeypatch, on, sched) as la:
            (O, *grads), den = got[on] = run(la, dev, 1e-6)
            (Ot, *gt), dent = run(la, dev, 1e-6, token_major=True)
        assert rel_err(O, ref) <= tol
        assert max(grad_errs(grads, gref)) <= (tol if bf16 else 1e-4)
        for a, b in zip((O, *grads, den), (Ot, *gt, dent)):
            assert np.array_equal(a, b)
    # den is an fp32 result whatever the tensors are; for bf16 tensors the wave kernels form the part of it
    # that comes from a token's own chunk from two-part operands, 2^-16
    assert rel_err(got["1"][1], got["0"][1].astype(np.float64)) <= (1.6e-5 if bf16 else 1e-6)


@pytest.mark.parametrize("sched", ["default", "many_segments"])
@pytest.mark.parametrize("kind", ["f32", "bf16", "poly2"])
def test_state_in_and_out(oracle, monkeypatch, kind, sched):
    """forward and backward from a state and into one: both kinds of kernels give the same to
    rounding, and the pieces the caller sees (final state, its gradient) are finite and equal"""
    B, H, N, M, bf16 = 2, 2, 301, 64, kind == "bf16"
    D = 8 if kind == "poly2" else 64
    C, eps, kw = 64, 0.5 if kind == "poly2" else 1e-6, {"features": "poly2"} if kind == "poly2" else {}
    dev = [to_dev(x, bf16) for x in maybe_bf16(wl.random_case(8300 + D, B, H, N, D, M), bf16)]
    S0, z0 = (torch.rand(s, device=DEV, generator=torch.Generator(DEV).manual_seed(3)) * 8 for s in ((B, H, C, M), (B, H, C)))
    dS1, dz1 = torch.randn(B, H, C, M, device=DEV), torch.randn(B, H, C, device=DEV)
    res = []
    for on in "01":
        with block_kernels(monkeypatch, on, sched) as la:
            q, k, v, g = dev
            O, den = torch.full_like(v, float("nan")), torch.full((B, H, N), float("nan"), device=DEV)
            S1, z1, dS0, dz0 = (torch.full_like(x, float("nan")) for x in (S0, z0, S0, z0))
            ws = la.la_causal_fwd_state(q, k, v, O, den, S0, z0, S1, z1, eps, **kw)
            grads = [torch.full_like(x, float("nan")) for x in (q, k, v)]
            la.la_causal_bwd_state(q, k, v, None, den, g, *grads, S0, z0, dS1, dz1, dS0, dz0, eps, fwd_ws=ws, **kw)
            torch.cuda.synchronize()
            res.append([to_host(x) for x in (O, den, S1, z1, *grads, dS0, dz0)])
    for i, (a, b) in enumerate(zip(*res)):
        exact = i in (1, 2, 3)               # den, S1, z1: fp32 results for every element type
        tol = (1e-2 if i == 2 else 1e-5) if exact and bf16 else 2e-2 if bf16 else 2e-5
        assert np.isfinite(b).all() and rel_err(b, a.astype(np.float64)) <= tol, i


def test_poly2_edges(oracle, monkeypatch):
    for N, sched in ((1, "default"), (33, "default"), (130, "many_segments"), (515, "default")):
        host = wl.random_case(8500 + N, 1, 2, N, 8, 64)
        ref = oracle.causal_fwd_poly2(*host[:3], 0.5)
        gref = oracle.causal_bwd_poly2(*host, 0.5)
        with block_kernels(monkeypatch, "1", sched) as la:
            for token_major in (False, True):
                (O, *grads), _ = run(la, [to_dev(x) for x in host], 0.5, token_major, features="poly2")
                assert rel_err(O, ref) <= 1e-5 and max(grad_errs(grads, gref)) <= 1e-4, N


def test_non_temporal_loads_change_no_bit(monkeypatch):
    dev = [to_dev(x) for x in wl.random_case(8600, 2, 2, 333, 64, 64)]
    with block_kernels(monkeypatch, "1", "many_segments") as la:
        a = run(la, dev, 1e-6)
    monkeypatch.setenv("LA_BLOCK_KERNELS", "1")
    with schedule(**SCHEDULES["many_segments"], stream_loads=1):
        b = run(la, dev, 1e-6)
    monkeypatch.delenv("LA_BLOCK_KERNELS")
    la.la_tuning_reload()
    for x, y in zip((*a[0], a[1]), (*b[0], b[1])):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("BH,N,D,M", [(1, 64, 32, 32), (3, 64, 64, 64), (3, 65, 64, 64), (40, 250, 32, 32), (16, 784, 32, 64),
                                      (96, 160, 64, 32), (128, 113, 32, 32), (200, 160, 32, 32), (200, 161, 32, 32)])
def test_short_sequences_and_their_workspaces(oracle, BH, N, D, M, bf16):
    """The default cut of short sequences at both sides of its lines; workspaces of exactly the size the
    queries name, followed by a mark that has to stay."""
    import paper_2006_16236_amd as la
    host = maybe_bf16(wl.random_case(8300 + N + BH, 1, BH, N, D, M), bf16)
    q, k, v, g = (to_dev(x, bf16) for x in host)
    code = la.LA_BF16 if bf16 else la.LA_F32
    sizes = [max(16, f(1, BH, N, D, M, code)) for f in (la.la_causal_fwd_workspace, la.la_causal_bwd_workspace)]
    bufs = [torch.full((n + 4096,), 0xA5, dtype=torch.uint8, device=DEV) for n in sizes]
    fws, bws = (b[:n] for b, n in zip(bufs, sizes))
    O, den = torch.empty_like(v), torch.empty(1, BH, N, device=DEV)
    grads = [torch.empty_like(x) for x in (q, k, v)]
    la.la_causal_fwd(q, k, v, O, den, 1e-6, ws=fws)
    la.la_causal_bwd(q, k, v, None, den, g, *grads, 1e-6, ws=bws, fwd_ws=fws)
    torch.cuda.synchronize()
    assert all(bool((b[n:] == 0xA5).all()) for b, n in zip(bufs, sizes))
    assert rel_err(to_host(O), oracle.causal_fwd_prefix(*host[:3], 1e-6)) <= (2e-2 if bf16 else 1e-5)
    errs = grad_errs([to_host(x) for x in grads], oracle.causal_bwd_linear(*host, 1e-6))
    assert max(errs) <= (2e-2 if bf16 else 1e-4), errs


def test_very_many_token_major_heads(monkeypatch):
    """[B, N, H, .] tensors with so many heads that a block of 32 tokens spans more than 4 GB, beyond what the
    workgroup kernels address: a few heads of the call against the same heads on their own."""
    with block_kernels(monkeypatch, "1", "default") as la:
        very_many_token_major_heads(la)


def very_many_token_major_heads(la):
    H, N, D = 1 << 19, 33, 64
    g = torch.Generator(DEV).manual_seed(8700)
    q, k, v, dO = (torch.randn(1, N, H, D, device=DEV, generator=g) for _ in range(4))
    O, dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(4))
    den = torch.empty(1, H, N, device=DEV)
    ws = la.la_causal_fwd_bnhd(q, k, v, O, den, 1e-6)
    la.la_causal_bwd_bnhd(q, k, v, None, den, dO, dq, dk, dv, 1e-6, fwd_ws=ws)
    some = torch.tensor([0, 1, H // 2 - 1, H // 2, H - 1], device=DEV)
    sq, sk, sv, sg = (x[:, :, some].transpose(1, 2).contiguous() for x in (q, k, v, dO))
    got = [to_host(x[:, :, some].transpose(1, 2)) for x in (O, dq, dk, dv)]
    sO, sden, *sgrads = (torch.empty_like(sv), torch.empty(1, len(some), N, device=DEV), *(torch.empty_like(x) for x in (sq, sk, sv)))
    sws = la.la_causal_fwd(sq, sk, sv, sO, sden, 1e-6)
    la.la_causal_bwd(sq, sk, sv, None, sden, sg, *sgrads, 1e-6, fwd_ws=sws)
    assert rel_err(got[0], to_host(sO).astype(np.float64)) <= 1e-5
    assert max(grad_errs(got[1:], [to_host(x).astype(np.float64) for x in sgrads])) <= 1e-4
    del q, k, v, dO, O, dq, dk, dv, ws
    torch.cuda.empty_cache()


@pytest.mark.parametrize("kind", ["f32", "bf16", "poly2"])
@pytest.mark.parametrize("D,M", [(64, 64), (32, 32), (64, 32), (32, 64)])
def test_nothing_is_touched_past_the_last_token(oracle, monkeypatch, kind, D, M):
    """Last blocks of 1, 2, 15, 17 and 31 tokens, both layouts: every tensor of the call ends where a guard
    begins, NaN behind the inputs (a value read there would show) and a mark that has to stay behind the
    outputs.  One sequence, so that a row past its end is past the tensor's; three token-major heads."""
    if kind == "poly2" and D != 64:
        pytest.skip("the polynomial map has 64 features")
    bf16, W, eps = kind == "bf16", 8 if kind == "poly2" else D, 0.5 if kind == "poly2" else 1e-6
    kw = {"features": "poly2"} if kind == "poly2" else {}
    dt, guard = torch.bfloat16 if bf16 else torch.float32, 64 * 64 * 3

    def guarded(t, fill):
        """a copy of t (or its uninitialised like) at the front of a longer buffer"""
        buf = torch.full((t.numel() + guard,), fill, dtype=t.dtype, device=DEV)
        view = buf[:t.numel()].view(t.shape)
        return buf, view

    with block_kernels(monkeypatch, "1", "default") as la:
        for N in (1, 2, 15, 17, 33, 47, 49, 63, 65, 79):
            for token_major in (False, True):
                B, H = 1, 3 if token_major else 1
                host = maybe_bf16(wl.random_case(8800 + N + D + 2 * M, B, H, N, W, M), bf16)
                ins = []
                for x in host:
                    t = to_dev(x, bf16)
                    t = t.transpose(1, 2).contiguous() if token_major else t
                    _, view = guarded(t, float("nan"))
                    view.copy_(t)
                    ins.append(view)
                q, k, v, g = ins
                outs = [guarded(t, -7.0) for t in (v, q, k, v, torch.empty(B, H, N, device=DEV))]
                (O, dq, dk, dv, den) = (view for _, view in outs)
                fwd, bwd = (la.la_causal_fwd_bnhd, la.la_causal_bwd_bnhd) if token_major else (la.la_causal_fwd, la.la_causal_bwd)
                ws = fwd(q, k, v, O, den, eps, **kw)
                bwd(q, k, v, None, den, g, dq, dk, dv, eps, fwd_ws=ws, **kw)
                torch.cuda.synchronize()
                assert all(bool((buf[view.numel():] == -7.0).all()) for buf, view in outs), (N, token_major)
                ref = (oracle.causal_fwd_poly2 if kw else oracle.causal_fwd_prefix)(*host[:3], eps)
                gref = (oracle.causal_bwd_poly2 if kw else oracle.causal_bwd_linear)(*host, eps)
                got = [to_host(x.transpose(1, 2) if token_major else x) for x in (O, dq, dk, dv)]
                assert rel_err(got[0], ref) <= (2e-2 if bf16 else 1e-5), (N, token_major)
                assert max(grad_errs(got[1:], gref)) <= (2e-2 if bf16 else 1e-4), (N, token_major)


@pytest.mark.parametrize("on", ["0", "1"])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("D,M", [(64, 64), (32, 32), (64, 32), (32, 64)])
def test_gradient_for_z0_is_an_fp32_sum(monkeypatch, D, M, bf16, on):
    """dz0 = dz1 + sum over the tokens of delta phi(Q), in fp32 for every element type: against that sum in
    fp64 from the very deltas the backward has left in its workspace (second array, after 1/den).  Bound:
    every product exact to 2^-23, sums of N terms in runs of at most 32 rounded at 2^-24 of their running
    size; the terms change sign, so the measure is the sum of their sizes: 2^-20 of it is ample, and half
    of what a factor cut to 16 bits (2^-17 of each term, with N = 40 hardly averaged) would do to single terms."""
    B, H, N = 2, 2, 40
    dev = [to_dev(x, bf16) for x in maybe_bf16(wl.random_case(8900 + D + 2 * M, B, H, N, D, M), bf16)]
    q, k, v, g = dev
    gen = torch.Generator(DEV).manual_seed(4)
    S0, z0 = (torch.rand(s, device=DEV, generator=gen) for s in ((B, H, D, M), (B, H, D)))
    dS1, dz1 = torch.zeros_like(S0), torch.zeros_like(z0)
    with block_kernels(monkeypatch, on, "default") as la:
        code = la.LA_BF16 if bf16 else la.LA_F32
        O, den, dS0, dz0 = torch.empty_like(v), torch.empty(B, H, N, device=DEV), torch.empty_like(S0), torch.empty_like(z0)
        ws = la.la_causal_fwd_state(q, k, v, O, den, S0, z0)
        grads = [torch.empty_like(x) for x in (q, k, v)]
        bws = torch.zeros(la.la_causal_bwd_workspace(B, H, N, D, M, code), dtype=torch.uint8, device=DEV)
        la.la_causal_bwd_state(q, k, v, None, den, g, *grads, S0, z0, dS1, dz1, dS0, dz0, ws=bws, fwd_ws=ws)
        torch.cuda.synchronize()
    rows = (B * H * N * 4 + 255) // 256 * 256
    delta = bws[rows:rows + B * H * N * 4].view(torch.float32).view(B, H, N).double()
    x = q.float()
    phi = torch.where(x > 0, x + 1.0, torch.exp(x)).double()
    terms = delta[..., None] * phi
    err = (dz0.double() - terms.sum(2)).abs() / terms.abs().sum(2)
    assert float(err.max()) <= 2.0 ** -20


@pytest.mark.parametrize("group", [None, 1, 2])
@pytest.mark.parametrize("D,M,N", [(64, 64, 5000), (64, 32, 5009), (32, 64, 4991)])
def test_workgroup_backward_on_the_wave_kernels_cut(oracle, D, M, N, group):
    """bf16 sequences in segments of more than 512 tokens: the wave kernels' forward, the workgroup kernels'
    backward on one, two or four of its segments (odd numbers of chunks among them)"""
    import paper_2006_16236_amd as la
    host = maybe_bf16(wl.random_case(9000 + N, 1, 3, N, D, M), True)
    with schedule(target_waves=24, bwd_seg_group=group):
        (O, *grads), _ = run(la, [to_dev(x, True) for x in host], 1e-6)
    assert rel_err(O, oracle.causal_fwd_prefix(*host[:3], 1e-6)) <= 2e-2
    assert max(grad_errs(grads, oracle.causal_bwd_linear(*host, 1e-6))) <= 2e-2


@pytest.mark.parametrize("sched", ["default", "many_segments"])
@pytest.mark.parametrize("kind", ["f32", "bf16"])
@pytest.mark.parametrize("D,M", [(64, 64), (32, 32), (64, 32), (32, 64)])
def test_states_against_fp64(monkeypatch, kind, D, M, sched):
    """The states a call returns and the gradients for the ones it took, from the workgroup kernels, against
    fp64 from the same (rounded) inputs; every error measured against the sum of the sizes of the terms.
    fp32: products exact to 2^-23, sums of 301 terms in runs of 32 and over segments: 2^-20; twice that behind
    delta.  bf16: phi(K) in two parts in S1 (2^-17 per term, V exact): 2^-16; phi(Q) in two parts in dS0, dO exact:
    2^-16; behind delta in dz0 at most three such cuts on a way (phi(K) in S and S; or the scores, phi(K) and
    their smallest product dropped): 2^-15.  A part lost anywhere (2^-9) is far outside."""
    B, H, N, bf16 = 1, 2, 301, kind == "bf16"
    dev = [to_dev(x, bf16) for x in maybe_bf16(wl.random_case(9100 + D + 2 * M, B, H, N, D, M), bf16)]
    q, k, v, g = dev
    gen = torch.Generator(DEV).manual_seed(6)
    S0, z0 = (torch.rand(s, device=DEV, generator=gen) * 8 for s in ((B, H, D, M), (B, H, D)))
    dS1, dz1 = (torch.randn(s, device=DEV, generator=gen) for s in ((B, H, D, M), (B, H, D)))
    with block_kernels(monkeypatch, "1", sched) as la:
        O, den = torch.empty_like(v), torch.empty(B, H, N, device=DEV)
        S1, z1, dS0, dz0 = (torch.full_like(x, float("nan")) for x in (S0, z0, S0, z0))
        ws = la.la_causal_fwd_state(q, k, v, O, den, S0, z0, S1, z1, 1e-6)
        grads = [torch.empty_like(x) for x in (q, k, v)]
        la.la_causal_bwd_state(q, k, v, None, den, g, *grads, S0, z0, dS1, dz1, dS0, dz0, 1e-6, fwd_ws=ws)
        torch.cuda.synchronize()
    x = [t.cpu().double() for t in (*dev, S0, z0, dS1, dz1)]
    q, k, v, g, s0, zz0, ds1, dzz1 = x
    fq, fk = (torch.where(t > 0, t + 1, torch.exp(t)) for t in (q, k))

    def states(a, b, start):                      # running sums of a b^T behind `start`, after every token
        return start[:, :, None] + torch.cumsum(a[..., :, None] * b[..., None, :], 2)

    z = zz0[:, :, None] + torch.cumsum(fk, 2)
    dn = (fq * z).sum(-1, keepdim=True) + 1e-6
    gd = g / dn
    S, Sabs = states(fk, v, s0), states(fk, v.abs(), s0)
    delta = -(fq * (S @ gd[..., None])[..., 0]).sum(-1, keepdim=True) / dn
    dabs = (fq * (Sabs @ gd.abs()[..., None])[..., 0]).sum(-1, keepdim=True) / dn
    want = {"S1": (S1, S[:, :, -1], Sabs[:, :, -1], 20, 16), "z1": (z1, z[:, :, -1], z[:, :, -1], 20, 20),
            "dS0": (dS0, ds1 + fq.transpose(2, 3) @ gd, ds1.abs() + fq.transpose(2, 3) @ gd.abs(), 20, 16),
            "dz0": (dz0, dzz1 + (delta * fq).sum(2), dzz1.abs() + (dabs * fq).sum(2), 19, 15)}
    for name, (got, ref, size, bits, bits16) in want.items():
        err = float(((got.cpu().double() - ref).abs() / size).max())
        assert err <= 2.0 ** -(bits16 if bf16 else bits), (name, err)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("D,M", [(64, 64), (32, 32), (64, 32), (32, 64)])
@pytest.mark.parametrize("N,sched", [(33, "default"), (70, "many_segments")])
def test_gradients_scale_with_the_upstream_gradient(monkeypatch, N, sched, D, M, bf16):
    """dO times a power of two scales every product and sum of the backward exactly, wherever the kernel brings
    1/den in (to dO, to phi(Q) or to the finished row): the gradients scale bit for bit."""
    q, k, v, g = (to_dev(x, bf16) for x in maybe_bf16(wl.random_case(9200 + N + D + 2 * M, 1, 3, N, D, M), bf16))
    with block_kernels(monkeypatch, "1", sched) as la:
        (_, *want), _ = run(la, (q, k, v, g), 1e-6)
        for scale in (2.0 ** 40, 2.0 ** -40):
            (_, *got), _ = run(la, (q, k, v, g * scale), 1e-6)
            for a, b in zip(got, want):
                assert np.array_equal(a / scale, b)


@pytest.mark.parametrize("on", ["0", "1"])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("D,M", [(64, 64), (32, 32), (64, 32), (32, 64)])
@pytest.mark.parametrize("N,sched", [(33, "default"), (300, "many_segments"), (1027, "default")])
def test_range_of_the_backward(monkeypatch, N, sched, D, M, bf16, on):
    """The backward's sums hold dO/den, not dO: gradients are finite wherever |dO| |V| M and dO/den are, however
    large den is.  Features phi(Q) 2^a, phi(K) 2^b and dO 2^c (eps = 0) scale den by 2^(a + b), and dQ, dK, dV by
    2^(c - a), 2^(c - b), 2^c, bit for bit while nothing leaves the range of fp32; sums of dO itself would reach
    2^(c + a + b + 20).  With the elu map den is up to 2^18 here."""
    host = wl.random_case(9300 + N + D + 2 * M, 1, 3, N, D, M)
    q, k, v, g = (to_dev(x, bf16) for x in maybe_bf16(host, bf16))
    fq, fk = (to_dev(x, bf16) for x in maybe_bf16([np.abs(x) + np.float32(0.125) for x in host[:2]], bf16))
    with block_kernels(monkeypatch, on, sched) as la:
        for dev, eps, kw, exponents in (((q, k, v, g), 1e-6, {}, [(0, 0, 110), (0, 0, -60)]),
                                        ((fq, fk, v, g), 0.0, {"features": True},
                                         [(27, 27, 85), (45, 20, 100), (-30, -30, 40), (-70, 70, 0), (60, -60, 40)])):
            (O, *want), den = run(la, dev, eps, **kw)
            for a, b, c in exponents:
                x = [t * 2.0 ** e for t, e in zip(dev, (a, b, 0, c))]
                (Ox, *got), denx = run(la, x, eps, **kw)
                assert np.array_equal(Ox, O) and np.array_equal(denx.astype(np.float64), den * 2.0 ** (a + b)), (a, b, c)
                for name, have, ref, e in zip(("dQ", "dK", "dV"), got, want, (c - a, c - b, c)):
                    assert np.isfinite(have).all() and np.array_equal(have.astype(np.float64), ref * 2.0 ** e), (name, a, b, c)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("D,M", [(64, 64), (32, 32), (64, 32), (32, 64)])
@pytest.mark.parametrize("N,sched", [(33, "default"), (300, "many_segments")])
def test_small_denominators(oracle, monkeypatch, N, sched, D, M, bf16):
    """Keys around -60, phi(K) = e^-60: den is near 1e-23 and eps = 0.  A reciprocal applied twice, left out, or
    taken out of delta again by mistake is 20 decades off.  fp32: of exp(x) comes 2^-24 |x log2 e| <= 2^-17, of
    every key alike in den, S and the gradients' sums: 1e-4 is ample (grad_errs' floor included)."""
    host = wl.random_case(9400 + N + D + 2 * M, 1, 3, N, D, M)
    host = maybe_bf16([host[0], host[1] - np.float32(60.0), *host[2:]], bf16)
    with block_kernels(monkeypatch, "1", sched) as la:
        (O, dq, dk, dv), _ = run(la, [to_dev(x, bf16) for x in host], 0.0)
    assert rel_err(O, oracle.causal_fwd_prefix(*host[:3], 0.0)) <= (2e-2 if bf16 else 1e-4)
    for got, ref in zip((dq, dk, dv), oracle.causal_bwd_linear(*host, 0.0)):
        assert rel_err(got, ref) <= (2e-2 if bf16 else 1e-4)
