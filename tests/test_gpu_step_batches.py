"""la_recurrent_steps takes its steps in batches of eight, or one at a time where a launch has few for many
sequences: every remainder of a batch and both sides of the line between the two, for every element type
and head size, must leave the bits that single steps leave (exact: the additions are the same in the same
order)."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("kind", ["f32", "bf16", "given", "poly2"])
@pytest.mark.parametrize("D,M", [(64, 64), (32, 32), (64, 32), (32, 64)])
def test_batches_equal_single_steps(kind, D, M):
    if kind == "poly2" and D != 64:
        pytest.skip("the polynomial map has 64 features")
    check(kind, 2, 3, D, M, (1, 2, 7, 8, 9, 16, 17, 31))


@pytest.mark.parametrize("kind", ["f32", "bf16", "poly2"])
@pytest.mark.parametrize("D,M", [(64, 64), (32, 32), (64, 32), (32, 64)])
def test_few_steps_of_many_sequences(kind, D, M):
    if kind == "poly2" and D != 64:
        pytest.skip("the polynomial map has 64 features")
    for BH, steps in ((1023, (2,)), (1024, (1, 2, 3)), (2047, (3,)), (2048, (2, 3, 4, 5)), (2559, (2,)), (2560, (2,)), (4095, (1, 2)),
                      (4096, (1, 2, 3, 8)), (4097, (2, 3, 4)), (15359, (1,)), (15360, (1,))):
        check(kind, BH, 1, D, M, steps)


def check(kind, B, H, D, M, lengths):
    import paper_2006_16236_amd as la
    W = 8 if kind == "poly2" else D
    kw = {"given": {"features": True}, "poly2": {"features": "poly2"}}.get(kind, {})
    dt = torch.bfloat16 if kind == "bf16" else torch.float32
    g = torch.Generator(DEV).manual_seed(D + 2 * M)
    for T in lengths:
        q, k = (torch.randn(T, B, H, W, device=DEV, generator=g).to(dt) for _ in range(2))
        if kind == "given":
            q, k = q.abs(), k.abs()
        v = torch.randn(T, B, H, M, device=DEV, generator=g).to(dt)
        S = torch.rand(B, H, D, M, device=DEV, generator=g)
        z = torch.rand(B, H, D, device=DEV, generator=g)
        S1, z1, out, out1 = S.clone(), z.clone(), torch.empty_like(v), torch.empty_like(v)
        la.la_recurrent_steps(q, k, v, S, z, out, 0.5, **kw)
        for t in range(T):
            la.la_recurrent_step(q[t], k[t], v[t], S1, z1, out1[t], 0.5, **kw)
        torch.cuda.synchronize()
        assert torch.equal(out, out1) and torch.equal(S, S1) and torch.equal(z, z1), (B * H, T)


@pytest.mark.parametrize("kind", ["f32", "bf16"])
@pytest.mark.parametrize("D,M", [(64, 64), (32, 32), (64, 32)])
@pytest.mark.parametrize("mb", [24, 288])
def test_states_beyond_the_cache(kind, D, M, mb):
    """Above 288 MB of S, fp32 from 24 MB on, the step passes the caches by: the same bits, sequence by sequence, as calls
    of few sequences, which do not."""
    import paper_2006_16236_amd as la
    BH = (mb << 20) // (D * M * 4) + 3
    dt = torch.bfloat16 if kind == "bf16" else torch.float32
    g = torch.Generator(DEV).manual_seed(D + 2 * M)
    q, k = (torch.randn(BH, 1, D, device=DEV, generator=g).to(dt) for _ in range(2))
    v = torch.randn(BH, 1, M, device=DEV, generator=g).to(dt)
    S = torch.rand(BH, 1, D, M, device=DEV, generator=g)
    z = torch.rand(BH, 1, D, device=DEV, generator=g)
    S1, z1, out, out1 = S.clone(), z.clone(), torch.empty_like(v), torch.empty_like(v)
    la.la_recurrent_step(q, k, v, S, z, out, 1e-6)
    for part in (slice(b, b + 1024) for b in range(0, BH, 1024)):
        la.la_recurrent_step(q[part], k[part], v[part], S1[part], z1[part], out1[part], 1e-6)
    torch.cuda.synchronize()
    assert torch.equal(out, out1) and torch.equal(S, S1) and torch.equal(z, z1)


@pytest.mark.parametrize("D,M", [(64, 64), (64, 32), (32, 64)])
@pytest.mark.parametrize("BH,T", [(3, 1), (3, 2), (3, 8), (3, 17), (1100, 2), (4100, 2)])
def test_products_of_the_denominator_are_not_rounded(D, M, BH, T):
    """den = sum q z, the rows a lane sweeps one after the other as fused multiply-adds: 1 * -(1 + 2^-11) and then
    (1 + 2^-12)^2 = 1 + 2^-11 + 2^-24 leave 2^-24, where the rounded products leave nothing."""
    import paper_2006_16236_amd as la
    RPI = 1024 // M                          # rows of S that a workgroup sweeps at a time
    q, k = (torch.zeros(T, BH, 1, D, device=DEV) for _ in range(2))
    v = torch.ones(T, BH, 1, M, device=DEV)
    S, z = torch.zeros(BH, 1, D, M, device=DEV), torch.zeros(BH, 1, D, device=DEV)
    row = torch.arange(BH, device=DEV) % RPI
    i = torch.arange(BH, device=DEV)
    q[:, i, 0, row], q[:, i, 0, row + RPI] = 1.0, 1 + 2.0 ** -12
    z[i, 0, row], z[i, 0, row + RPI] = -(1 + 2.0 ** -11), 1 + 2.0 ** -12
    S[i, 0, row] = 0.5
    out = torch.zeros_like(v)
    la.la_recurrent_steps(q, k, v, S, z, out, 0.0, features=True)
    torch.cuda.synchronize()
    assert (out == 2.0 ** 23).all()
    out.zero_()
    la.la_recurrent_step(q[0], k[0], v[0], S, z, out[0], 0.0, features=True)
    torch.cuda.synchronize()
    assert (out[0] == 2.0 ** 23).all()
