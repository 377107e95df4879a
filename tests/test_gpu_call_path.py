"""The native accepting path of the binding (csrc/la_call.cpp) against the Python checks beside it, which
an explicit `stream` selects: the same bits (the same library call is made), nothing taken that the
checks refuse, and the current stream respected."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def tensors(shape_qk, shape_v, rows, dt, seed=5):
    g = torch.Generator(DEV).manual_seed(seed)
    q, k = (torch.randn(shape_qk, device=DEV, generator=g).to(dt) for _ in range(2))
    v, dO = (torch.randn(shape_v, device=DEV, generator=g).to(dt) for _ in range(2))
    return q, k, v, dO, torch.empty_like(v), torch.empty(rows, device=DEV), *(torch.empty_like(x) for x in (q, k, v))


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("layout", ["", "_bnhd"])
@pytest.mark.parametrize("kind", ["causal", "global"])
def test_same_bits_as_the_python_checks(kind, layout, dt):
    import paper_2006_16236_amd as la
    from paper_2006_16236_amd import binding
    B, H, N, D, M = 2, 3, 37, 64, 32
    lead = (B, N, H) if layout else (B, H, N)
    fwd, bwd = getattr(la, f"la_{kind}_fwd{layout}"), getattr(la, f"la_{kind}_bwd{layout}")
    code = ["causal", "causal_bnhd", "global", "global_bnhd"].index(kind + layout)
    for features in (False, True):
        got = []
        side = torch.cuda.Stream()
        for stream in (None, torch.cuda.current_stream(), side):
            q, k, v, dO, O, den, dq, dk, dv = tensors((*lead, D), (*lead, M), (B, H, N), dt)
            if features:
                q, k = q.abs(), k.abs()
            torch.cuda.synchronize()
            if stream is side:                             # the native path on another current stream
                with torch.cuda.stream(side):
                    ws = binding._call.fwd(code, q, k, v, O, den, None, 1e-6, features)
                    assert isinstance(ws, torch.Tensor)
                    assert binding._call.bwd(code, q, k, v, None, den, dO, dq, dk, dv, None, ws, 1e-6, features) is not None
            else:
                ws = fwd(q, k, v, O, den=den, eps=1e-6, stream=stream, features=features)
                bwd(q, k, v, None, den, dO, dq, dk, dv, 1e-6, fwd_ws=ws, stream=stream, features=features)
            torch.cuda.synchronize()
            got.append((O, den, dq, dk, dv))
        for other in got[1:]:
            assert all(torch.equal(a, b) for a, b in zip(got[0], other))


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
def test_step_same_bits(dt):
    import paper_2006_16236_amd as la
    from paper_2006_16236_amd import binding
    B, H, D, M = 2, 3, 32, 64
    q, k, v, _, out, *_ = tensors((B, H, D), (B, H, M), (B, H), dt)
    S, z = torch.rand(B, H, D, M, device=DEV), torch.rand(B, H, D, device=DEV)
    S1, z1, out1 = S.clone(), z.clone(), torch.empty_like(out)
    assert binding._call.step(q, k, v, S, z, out, 1e-6, False) == 0
    la.la_recurrent_step(q, k, v, S1, z1, out1, 1e-6, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert torch.equal(out, out1) and torch.equal(S, S1) and torch.equal(z, z1)


def test_what_is_not_taken():
    """Every tensor of a call replaced in turn by one that the checks refuse: native code answers None
    and the call raises; too small a workspace is refused by the library on both paths."""
    import paper_2006_16236_amd as la
    from paper_2006_16236_amd import binding

    class Sub(torch.Tensor):
        pass

    B, H, N, D, M = 1, 2, 19, 32, 32
    q, k, v, dO, O, den, dq, dk, dv = tensors((B, H, N, D), (B, H, N, M), (B, H, N), torch.float32)
    ws = la.la_causal_fwd(q, k, v, O, den)
    S, z = torch.rand(B, H, D, M, device=DEV), torch.rand(B, H, D, device=DEV)
    step = [q[:, :, 0].contiguous(), k[:, :, 0].contiguous(), v[:, :, 0].contiguous(), S, z, O[:, :, 0].contiguous()]
    fwd, bwd = [q, k, v, O, den], [q, k, v, O, den, dO, dq, dk, dv]
    calls = ((lambda a: binding._call.fwd(0, *a, None, 1e-6, False), lambda a: la.la_causal_fwd(*a), fwd),
             (lambda a: binding._call.bwd(0, *a, None, ws, 1e-6, False), lambda a: la.la_causal_bwd(*a, fwd_ws=ws), bwd),
             (lambda a: binding._call.step(*a, 1e-6, False), lambda a: la.la_recurrent_step(*a), step))
    for native, public, args in calls:
        for i, t in enumerate(args):
            wide = torch.empty(*t.shape[:-1], 2 * t.shape[-1], device=DEV, dtype=t.dtype)
            wrong = [t.cpu(), t.double(), t[..., 1:].contiguous(), t[None].contiguous(), wide[..., ::2], 3.0]
            for w in wrong:
                a = args[:i] + [w] + args[i + 1:]
                assert native(a) is None, (i, type(w))
                with pytest.raises((ValueError, TypeError, la.LaError)):
                    public(a)
            assert native(args[:i] + [t.as_subclass(Sub)] + args[i + 1:]) is None
    assert binding._call.fwd(0, *fwd, None, 1e-6, "poly2") is None
    for stream in (None, torch.cuda.current_stream()):
        with pytest.raises(la.LaError):
            la.la_causal_bwd(*bwd, ws=torch.empty(16, device=DEV, dtype=torch.uint8), fwd_ws=ws, stream=stream)
    torch.cuda.synchronize()
