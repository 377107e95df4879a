"""The host side of the schedule (csrc/la_plan.h), without a GPU: plans, and the workspaces that have to
hold what the plans write."""
import os
import random
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2006_16236_amd", "csrc")
FIELDS = ("nchunks", "nseg", "cps", "fold", "fwd_block", "bwd_block", "bwd_group", "writes", "states", "bwd", "step_streams", "one_by_one", "nt_causal", "nt_global", "fwd_direct")
DEFAULT = dict(target=2048, min_chunks=2, fold=8, group=0, block=-1, heads=0)
F32, BF16, GIVEN, POLY2 = 0, 1, 2, 4


@pytest.fixture(scope="session")
def plans(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_probe")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", os.path.join(ROOT, "tests", "plan_probe.cpp"), "-o", exe], check=True)

    def run(calls):
        """calls: (BH, N, C, M, dtype, tuning overrides) -> one dict per call"""
        lines = []
        for BH, N, C, M, t, kw in calls:
            k = {**DEFAULT, **kw}
            lines.append(f"{k['target']} {k['min_chunks']} {k['fold']} {k['group']} {k['block']} {BH} {N} {C} {M} {t} {k['heads']}")
        out = subprocess.run([exe], input="\n".join(lines), capture_output=True, text=True, check=True).stdout.split("\n")
        return [dict(zip(FIELDS, map(int, o.split()))) for o in out if o]

    return run


def test_one_snapshot_of_the_tuning_values_per_call():
    """The plan of a call and the workspace it checks for come from the same values: la_plan.h is given them
    and cannot read them, and no function of the C ABI reads them twice."""
    text = open(os.path.join(CSRC, "la_api.hip")).read()
    assert "tuning()" not in open(os.path.join(CSRC, "la_plan.h")).read()
    bodies = re.findall(r"^(?:static )?(?:int|size_t|void|Plan|Tuning) (\w+)\([^;{]*\) \{\n(.*?)^\}", text, re.S | re.M)
    reads = {name: len(re.findall(r"(?<!read_)\btuning\(\)", body)) for name, body in bodies}
    entries = {"causal_fwd_impl", "la_causal_fwd_noalloc", "causal_fwd_state_impl", "causal_bwd_impl", "global_fwd_impl",
               "global_bwd_impl", "la_causal_fwd_workspace", "la_causal_bwd_workspace", "la_global_fwd_workspace",
               "la_global_bwd_workspace"}
    assert {n for n, c in reads.items() if c} == entries
    assert all(reads[n] == 1 for n in entries)
    # ... nor calls another function that does
    for name, body in bodies:
        others = entries & set(re.findall(r"\b(\w+)\(", body))
        assert not (others and name in entries), (name, others)


def test_a_plan_never_has_more_segments_than_its_workspace_holds(plans):
    rng, calls = random.Random(1), []
    for _ in range(20000):
        C, M = rng.choice(((64, 64), (32, 32), (64, 32), (32, 64)))
        kw = dict(target=rng.choice((1, 3, 24, 256, 2047, 2048, 2048, 2048, 1 << 20)), min_chunks=rng.choice((1, 2, 2, 3, 8)),
                  group=rng.choice((0, 1, 2)), block=rng.choice((-1, 0, 1)))
        calls.append((int(2 ** rng.uniform(0, 13)), int(2 ** rng.uniform(0, 17)), C, M, rng.choice((F32, BF16)), kw))
    for call, p in zip(calls, plans(calls)):
        assert p["writes"] <= p["states"] and 2 * p["states"] < p["bwd"], (call, p)
        assert (p["nseg"] - 1) * p["cps"] < p["nchunks"] <= p["nseg"] * p["cps"], (call, p)      # no segment is empty
        if p["fwd_block"] or p["bwd_block"]:                # whole 32-token blocks
            assert p["cps"] % 2 == 0 or p["nseg"] == 1 or (not p["fwd_block"] and p["cps"] * p["bwd_group"] % 2 == 0), (call, p)


def test_very_many_heads_keep_the_wave_kernels(plans):
    """Token-major tensors whose 32 tokens span more bytes than a 32-bit offset holds are not for the workgroup
    kernels, whatever the tuning values; head-major tensors of the same sizes are."""
    for t, e in ((F32, 4), (BF16, 2), (POLY2, 4)):
        for C, M in ((64, 64), (32, 32), (64, 32), (32, 64)):
            if t == POLY2 and C != 64:
                continue
            last = (2 ** 31 - 1) // (32 * max(C, M) * e)         # the most heads that fit
            for block in (-1, 1):
                for N in (1, 33, 512):
                    calls = [(H, N, C, M, t, dict(block=block, heads=heads)) for H in (last, last + 1, 2 * last + 2, (1 << 20) - 1)
                             if H < 1 << 20 for heads in (H, 0)]
                    for (H, *_, kw), p in zip(calls, plans(calls)):
                        if kw["heads"] > last:
                            assert not (p["fwd_block"] or p["bwd_block"]), (H, kw, p)
                        elif block == 1:
                            assert p["fwd_block"] and p["bwd_block"], (H, kw, p)
    # fp32 64 x 64 beyond one round of sequences is the workgroup kernels' by default: the case that overflowed
    assert plans([(4096, 64, 64, 64, F32, dict(heads=4096))])[0]["bwd_block"] == 1


def test_no_nearly_empty_second_round(plans):
    """Two workgroups per CU have a place, 512 in all: sequences long enough to be cut are not cut into a few
    workgroups more than that."""
    calls = [(BH, N, C, M, t, {}) for BH in range(1, 512) for N in (520, 1100, 2048, 3524, 7942, 20000)
             for C, M, t in ((64, 64, F32), (64, 64, BF16), (32, 64, F32), (64, 32, BF16))]
    for call, p in zip(calls, plans(calls)):
        BH, N, C, M, t, _ = call
        if p["fwd_block"]:
            assert p["nseg"] <= 3 or not 512 < BH * p["nseg"] < 585, (call, p)
        elif p["bwd_block"] and p["bwd_group"] == 4:         # the forward's segments four at a time
            assert BH * -(-p["nseg"] // 4) <= 512, (call, p)


def test_half_empty_blocks_of_many_sequences(plans):
    """One chunk or three fill half of their last 32-token block: the wave kernels' forward takes them."""
    calls = [(BH, N, C, M, t, {}) for BH in (512, 700, 1023, 1024, 2000) for N in (1, 16, 33, 48)
             for C, M in ((64, 64), (32, 32), (64, 32), (32, 64)) for t in (F32, BF16)]
    assert not any(p["fwd_block"] for p in plans(calls))
    assert all(p["fwd_block"] for p in plans([(BH, N, 64, 64, F32, {}) for BH in (1, 8, 255) for N in (1, 16, 33, 48, 64)]))


def test_a_requested_segment_group_is_honoured(plans):
    """LA_BWD_SEG_GROUP = 1 or 2 holds for every plan that cuts its sequences, the wave kernels' forward with the
    workgroup kernels' backward (long bf16 sequences) among them."""
    rng = random.Random(2)
    for group in (1, 2):
        calls = [(int(2 ** rng.uniform(0, 9)), int(2 ** rng.uniform(9, 17)), *rng.choice(((64, 64), (32, 32), (64, 32), (32, 64))),
                  rng.choice((F32, BF16)), dict(group=group, block=rng.choice((-1, 0, 1)))) for _ in range(3000)]
        mixed = 0
        for call, p in zip(calls, plans(calls)):
            if p["nseg"] > 1:
                assert p["bwd_group"] == group, (call, p)
                mixed += p["bwd_block"] and not p["fwd_block"]
                assert not p["bwd_block"] or p["cps"] * group % 2 == 0, (call, p)
        assert mixed > 100


def test_which_decode_steps_pass_the_caches_by(plans):
    """States above 288 MB, and from the size of the L2s on those of fp32 calls: with plain loads and stores a step of
    2048 to 14000 sequences, D = M = 64, took 4 to 9 % longer than with the two in turn."""
    def streams(MB, t, C=64, M=64):
        return plans([((MB << 20) // (C * M * 4), 1, C, M, t, {})])[0]["step_streams"]
    for C, M in ((64, 64), (64, 32), (32, 64), (32, 32)):
        assert [streams(mb, F32, C, M) for mb in (1, 16, 23, 24, 32, 128, 239, 240, 256, 287, 288, 1024)] == [0, 0, 0, 1, 1, 1, 1, 0, 0, 0, 1, 1]
        assert [streams(mb, BF16, C, M) for mb in (1, 24, 128, 240, 287, 288, 1024)] == [0, 0, 0, 0, 0, 1, 1]
    assert streams(32, POLY2) == 1 and streams(16, POLY2) == 0


def test_which_decode_steps_go_one_by_one(plans):
    """One step, and two of many sequences, a token at a time but where the batched kernel is faster; a single step of
    fp32 sequences with more than 240 MB of state had become up to 14 % slower in a batch."""
    def one(T, BH, C, M, t=F32):
        return plans([(BH, T, C, M, t, {})])[0]["one_by_one"]
    assert [one(1, b, 64, 64) for b in (1, 4095, 4096, 15359, 15360, 1 << 20)] == [1, 1, 0, 0, 1, 1]
    assert [one(1, b, 64, 64, POLY2) for b in (1, 4096, 16384)] == [1, 0, 1]
    assert all(one(1, b, C, M, t) for b in (1, 4096, 16384) for C, M, t in ((64, 64, BF16), (32, 32, F32), (64, 32, F32), (32, 64, F32)))
    assert [one(2, b, 64, 64) for b in (1023, 1024, 2559, 2560, 16384)] == [0, 1, 1, 0, 0]
    assert [one(2, b, 64, 64, BF16) for b in (1023, 1024, 16384)] == [0, 1, 1]
    for t in (F32, BF16, POLY2):
        assert [one(2, b, 64, 32, t) for b in (4095, 4096, 16384)] == [0, 1, 1]
    assert not any(one(2, b, C, M) for b in (1, 4096, 16384) for C, M in ((32, 32), (32, 64)))
    assert not any(one(T, b, C, M, t) for T in (3, 4, 8, 9, 784) for b in (1, 1024, 16384)
                   for C, M, t in ((64, 64, F32), (64, 64, BF16), (32, 32, F32), (64, 32, F32)))


def test_which_outputs_leave_non_temporally(plans):
    """Outputs of bf16 calls and the elements of given fp32 features stay in the caches for whoever reads them next, up to 64 to 128
    MB (projection and weight gradients of 4 x 3072 tokens, bf16: 352 -> 404 us behind non-temporal stores)."""
    def nt(mb, t, C=64, M=64, kind="nt_causal"):
        N = 1024
        return plans([((mb << 20) // (N * max(C, M) * (2 if t in (BF16, 3) else 4)), N, C, M, t, {})])[0][kind]
    for t in (BF16, 3):
        for M in (64, 32):
            assert [nt(mb, t, M=M) for mb in (1, 12, 64, 79, 80, 256)] == [0, 0, 0, 0, 1, 1]
            assert not any(nt(mb, t, 32, M, kind) for mb in (1, 64, 128, 1024) for kind in ("nt_causal", "nt_global"))
            assert not nt(1024, t, 64, 32, "nt_global")
        assert [nt(mb, t, kind="nt_global") for mb in (1, 64, 127, 128, 256)] == [0, 0, 0, 1, 1]
    for kind in ("nt_causal", "nt_global"):
        for C, M in ((64, 64), (32, 32), (32, 64), (64, 32)):
            assert [nt(mb, GIVEN, C, M, kind) for mb in (1, 24, 63, 64, 256)] == [0, 0, 0, 1, 1]
            assert all(nt(mb, F32, C, M, kind) for mb in (1, 64, 256))
        assert all(nt(mb, POLY2, kind=kind) for mb in (1, 64, 256))


def test_which_forwards_go_by_definition(plans):
    """fwd_direct_kernel: 33 to 256 tokens, from 65 on where one segment in one launch is as fast (bf16, a 32-wide D), up to 256
    workgroups of 32 queries, in head-major and token-major calls; a forced choice of kernels turns it off."""
    def direct(BH, N, C, M, t=F32, **kw):
        return plans([(BH, N, C, M, t, kw)])[0]["fwd_direct"]
    for M in (64, 32):
        for t, C in ((F32, 64), (GIVEN, 64), (POLY2, 64)):
            assert [direct(1, N, C, M, t) for N in (1, 32, 33, 64, 65, 255, 256, 257)] == [0, 0, 1, 1, 1, 1, 1, 0]
        for t, C in ((BF16, 64), (3, 64), (F32, 32), (BF16, 32), (GIVEN, 32), (3, 32)):
            assert [direct(1, N, C, M, t) for N in (1, 32, 33, 64, 65, 255, 256, 257)] == [0, 0, 0, 0, 1, 1, 1, 0]
    for t in (F32, BF16, GIVEN, POLY2):
        assert [direct(BH, 256, 64, 64, t) for BH in (1, 32, 33, 64)] == [1, 1, 0, 0]               # 8 workgroups each
        assert [direct(BH, 65, 64, 64, t) for BH in (85, 86)] == [1, 0]                               # 3 each
    for N in (33, 65, 256):
        assert direct(8, N, 64, 64, heads=8) == 1 and direct(8, N, 64, 64, block=0) == 0 and direct(8, N, 64, 64, block=1) == 0
    # the schedule's other knobs do not turn it off, and its totals are scanned where they do not fold
    assert all(direct(1, 133, 64, 64, **kw) for kw in (dict(target=1 << 20, min_chunks=1), dict(target=1 << 20, min_chunks=3), dict(target=24, fold=64),
                                                            dict(target=24, fold=1), dict(fold=1), dict(group=2)))
    scanned = plans([(1, 133, 64, 64, F32, dict(fold=1))])[0]
    assert scanned["fwd_direct"] and scanned["nseg"] > 1 and not scanned["fold"]
