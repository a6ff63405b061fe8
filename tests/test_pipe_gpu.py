"""The software-pipelined kernel's forms (wavefronts x queries, key groups), each by name, where they can go wrong."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2604_14825_amd import binding as nb
from paper_2604_14825_amd import synth

import gpu_util as gu
from test_safe_sync_gpu import both_prefill

FORMS = [("w4q32", 64), ("w4q32", 80), ("w4q32", 128), ("w4q32g2", 64), ("w4q32g2", 96), ("w4q32g2", 128), ("w8q32", 96),
         ("w8q32", 128), ("w8q32", 64)]     # w8q32 at D = 64: four wavefronts of 64 queries
EDGES = [1, 31, 32, 33, 64, 65, 96, 97, 127, 128, 129, 160, 191, 223, 256, 257, 288, 333, 511, 545]


def make(B, Hq, Hkv, S, D, idt, seed):
    q = synth.fill(B, Hq, S, D, seed, synth.TAG_Q, idt)
    k = synth.fill(B, Hkv, S, D, seed, synth.TAG_K, idt, S // 50, 8.0)
    return q, k, synth.fill(B, Hkv, S, D, seed, synth.TAG_V, idt)


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("variant,D", FORMS)
def test_key_block_counts(variant, D, causal, monkeypatch):
    """Every residue of the 32-key blocks modulo the four buffers, with and without a ragged last one, down to key groups
    and wavefronts that have none: against the oracle, and bit for bit against the conservatively synchronised build."""
    monkeypatch.setenv("NAUT_ATTN_VARIANT", variant)
    scale = 1.0 / math.sqrt(D)
    for S in EDGES:
        q, k, v = make(1, 2, 1, S, D, synth.BF16, 7100 + S)
        print("pipe", variant, D, causal, S, flush=True)
        qd, kd, vd = (gu.to_device(a, synth.BF16) for a in (q, k, v))
        o = torch.full((1, 2, S, D), float("nan"), device="cuda")
        lse = torch.full((1, 2, S), float("nan"), device="cuda")
        nb.naut_attn_fwd_strided(qd, kd, vd, o, lse, causal, scale)
        torch.cuda.synchronize()
        o_ref, lse_ref = oracle.attn_rows(q, k, v, synth.BF16, causal, scale)
        gu.check(o.double().cpu().numpy(), lse.double().cpu().numpy(), o_ref, lse_ref, "%s S=%d" % (variant, S))
        if D in (64, 128) and S in (1, 33, 129, 288, 545):
            both_prefill(q, k, v, synth.BF16, synth.BF16, causal, scale, "%s S=%d" % (variant, S))


@pytest.mark.gpu
@pytest.mark.parametrize("idt,odt", [(synth.BF16, synth.BF16), (synth.BF16, synth.F32), (synth.F16, synth.F16), (synth.F16, synth.F32)])
@pytest.mark.parametrize("variant", ["w4q32", "w4q32g2", "w8q32"])
def test_against_the_plain_kernel(variant, idt, odt, monkeypatch):
    """Orders and strides, storage types and odd sizes: the same call on kernel 1 with one key group differs by the rounding
    of P to 16 bits on either side and, for 16-bit O, of O."""
    B, Hq, Hkv, S = 2, 6, 2, 301
    dt, ot = gu.TORCH_DT[idt], gu.TORCH_DT[odt]
    eps = 2.0 ** -8 if idt == synth.BF16 else 2.0 ** -11
    g = torch.Generator(device="cuda").manual_seed(5)
    for D in (40, 64, 72, 128):
        def padded(H, pad_b=0, pad_s=0, pad_d=0, seq_major=False):
            x = torch.randn(B, *((S, H) if seq_major else (H, S + pad_s)), D + pad_d, generator=g, device="cuda").to(dt)[..., :D]
            return x.transpose(1, 2) if seq_major else x[:, :, :S]
        for what, q, k, v, sm in (("dense", padded(Hq), padded(Hkv), padded(Hkv), False),
                                  ("sequence-major", padded(Hq, seq_major=True), padded(Hkv, seq_major=True), padded(Hkv, seq_major=True), True),
                                  ("padded rows", padded(Hq, pad_d=8), padded(Hkv, pad_d=24), padded(Hkv, pad_s=3, pad_d=8), False),
                                  ("one cache for the batch", padded(Hq), padded(Hkv)[:1].expand(B, -1, -1, -1), padded(Hkv)[:1].expand(B, -1, -1, -1), False)):
            res = []
            for name in ("bm128g1", variant):
                monkeypatch.setenv("NAUT_ATTN_VARIANT", name)
                for causal in (True, False):
                    print("against plain", variant, name, D, what, causal, idt, odt, flush=True)
                    o = torch.full((B, S, Hq, D) if sm else (B, Hq, S, D), float("nan"), dtype=ot, device="cuda")
                    o = o.transpose(1, 2) if sm else o
                    lse = torch.full((B, Hq, S), float("nan"), device="cuda")
                    nb.naut_attn_fwd_strided(q, k, v, o, lse, causal, 1.0 / math.sqrt(D))
                    torch.cuda.synchronize()
                    res.append((o.double(), lse))
            vmax = v.double().abs().max().item()
            for (o1, l1), (o2, l2) in zip(res[:2], res[2:]):
                # each side: sum of w |v| eps over rounded P, at most eps |v| max; 16-bit O half a unit in the last place
                bound = 2 * (eps / 2 * vmax + (eps / 2 * vmax if odt != synth.F32 else 0)) + 1e-5
                assert (o1 - o2).abs().max().item() <= bound, (what, D, (o1 - o2).abs().max().item(), bound)
                assert torch.allclose(l1, l2, rtol=1e-6, atol=1e-5), (what, D)


@pytest.mark.gpu
@pytest.mark.parametrize("D,S", [(128, 2048), (64, 2048), (128, 640)])
@pytest.mark.parametrize("heads", [12, 24, 32, 36])
def test_every_tile_is_done(D, S, heads, monkeypatch):
    """The order of a causal launch -- the second round of work-groups reversed, heads in groups, or eight that do not divide
    the heads -- is a permutation: with V = 1 every element of O is 1, and lse is that of kernel 1."""
    g = torch.Generator(device="cuda").manual_seed(heads + S + D)
    q, k = (torch.randn(1, heads, S, D, device="cuda", generator=g).to(torch.bfloat16) for _ in range(2))
    v = torch.ones(1, heads, S, D, device="cuda", dtype=torch.bfloat16)
    lses = []
    for name in ("bm128g1", "bm128g2", "w4q32", "w4q32g2", "w8q32"):
        gu.use_form(monkeypatch, name, 1, heads, S, D, True)
        print("order", name, D, S, heads, flush=True)
        o = torch.full((1, heads, S, D), float("nan"), dtype=torch.bfloat16, device="cuda")
        lse = torch.full((1, heads, S), float("nan"), device="cuda")
        nb.naut_attn_fwd_strided(q, k, v, o, lse, True, 1.0 / math.sqrt(D))
        torch.cuda.synchronize()
        assert torch.equal(o, torch.ones_like(o)), name
        lses.append(lse)
    for lse in lses[1:]:
        assert torch.allclose(lse, lses[0], rtol=1e-6, atol=1e-5)


@pytest.mark.gpu
@pytest.mark.parametrize("variant,D", [("w4q32", 128), ("w4q32g2", 64), ("w8q32", 64), ("w8q32", 128)])
def test_scores_below_any_start_value(variant, D, monkeypatch):
    """Finite scores that all lie below -1e30 (see the test of the same kind for kernel 1): O is the mean of V."""
    monkeypatch.setenv("NAUT_ATTN_VARIANT", variant)
    S, high = 600, 2.0 ** (55 if D == 64 else 54)
    q = torch.full((1, 2, S, D), high, dtype=torch.bfloat16, device="cuda")
    k = torch.full((1, 1, S, D), -2.0 * high, dtype=torch.bfloat16, device="cuda")
    k[:, :, ::5] = -high
    v = (torch.arange(S * D, device="cuda") * 7 % 16).to(torch.bfloat16).view(1, 1, S, D)
    o, lse = torch.full((1, 2, S, D), float("nan"), device="cuda"), torch.full((1, 2, S), float("nan"), device="cuda")
    nb.naut_attn_fwd_strided(q, k, v, o, lse, False, 0.125)
    torch.cuda.synchronize()
    assert torch.allclose(o[0].double(), v[0, 0].double()[::5].mean(0).expand(2, S, D), rtol=0, atol=16 * 2.0 ** -22)
    assert torch.allclose(lse.double(), torch.full_like(lse, -D * high * high * 0.125).double(), rtol=2e-7)


def test_kernel_names(monkeypatch):
    """What a launch runs, by shape and by name."""
    monkeypatch.delenv("NAUT_ATTN_VARIANT", raising=False)
    for args, want in (((1, 2, 256, 64, False), "plain_4x32"), ((1, 8, 1024, 128, True), "plain_2x32_g4"),
                       ((1, 32, 1003, 128, True), "pipe_4x32_g2"), ((4, 32, 4096, 128, True), "pipe_4x32"),
                       ((2, 64, 8192, 128, True), "pipe_8x32"), ((1, 32, 4096, 64, False), "pipe_4x64"),
                       ((8, 16, 1024, 64, True), "pipe_4x32"), ((1, 32, 16384, 256, True), "plain_8x32"), ((1, 8, 64, 100, True), None)):
        assert nb.kernel_name(*args) == want, args
    for name, at64, at128 in (("w8q32", "pipe_4x64", "pipe_8x32"), ("w4q64", "pipe_4x64", "plain_4x32"), ("w4q32", "pipe_4x32", "pipe_4x32"),
                              ("w4q32g2", "pipe_4x32_g2", "pipe_4x32_g2"), ("bm128g1", "plain_4x32", "plain_4x32"),
                              ("bm128g2", "plain_4x32_g2", "plain_4x32_g2"), ("bm128g4", "plain_2x32_g4", "plain_2x32_g4"), ("no", None, None)):
        monkeypatch.setenv("NAUT_ATTN_VARIANT", name)
        assert nb.kernel_name(1, 2, 128, 64, False) == at64 and nb.kernel_name(1, 2, 128, 128, False) == at128, name


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("D,variant,S", [(64, "w4q32", 200), (128, "w4q32", 200), (128, "w8q32", 200), (64, "w8q32", 512), (128, "w4q32", 129)])
def test_error_is_that_of_the_plain_kernel(D, variant, S, causal, monkeypatch):
    """Short sequences, where it matters most how many keys the first reference maximum is taken over: the error of O against
    64 bits is no larger than kernel 1's on the same call.  Both round P and nothing else to 16 bits, so over the 4e5 and more
    elements of these calls the ratio of two such errors is steady to a per cent (1e6 independent roundings behind each)."""
    g = torch.Generator(device="cuda").manual_seed(D + S)
    for hot in (1.0, 2.0):
        q, k, v = (torch.randn(1, 64, S, D, device="cuda", generator=g).to(torch.bfloat16) for _ in range(3))
        scale = hot / math.sqrt(D)
        s = torch.matmul(q.double(), k.double().transpose(-1, -2).contiguous()) * scale
        if causal:
            s = s.masked_fill(torch.ones(S, S, device="cuda", dtype=torch.bool).triu(1), -math.inf)
        ref = torch.matmul(torch.softmax(s, -1), v.double())
        err = {}
        for name in ("bm128g1", variant):
            monkeypatch.setenv("NAUT_ATTN_VARIANT", name)
            o, lse = torch.full(q.shape, math.nan, device="cuda"), torch.empty(1, 64, S, device="cuda")
            nb.naut_attn_fwd_strided(q, k, v, o, lse, causal, scale)
            torch.cuda.synchronize()
            err[name] = ((o.double() - ref).norm() / ref.norm()).item()
        print("error", D, S, causal, hot, variant, "%.4e of %.4e: %.4f" % (err[variant], err["bm128g1"], err[variant] / err["bm128g1"]), flush=True)
        assert err[variant] <= 1.01 * err["bm128g1"]


@pytest.mark.gpu
@pytest.mark.parametrize("H,S,D,causal", [(16, 4096, 128, True), (16, 4096, 96, False), (4, 16384, 64, False), (48, 640, 128, True), (24, 1500, 128, False)])
def test_a_named_form_is_the_form_of_the_rule(H, S, D, causal, monkeypatch):
    """Naming the form that the shape runs anyway changes nothing, bit for bit, also on long loops, where the reference
    maximum may lag further: comparisons by name time and test what runs."""
    monkeypatch.delenv("NAUT_ATTN_VARIANT", raising=False)
    form = nb.kernel_name(1, H, S, D, causal)
    name = {"pipe_8x32": "w8q32", "pipe_4x64": "w8q32", "pipe_4x32": "w4q32", "pipe_4x32_g2": "w4q32g2"}[form]
    g = torch.Generator(device="cuda").manual_seed(S)
    q, k, v = (torch.randn(1, H, S, D, device="cuda", generator=g).to(torch.bfloat16) for _ in range(3))
    k[:, :, :: S // 40] *= 4  # the maximum grows along the sequence
    res = []
    for e in ("", name):
        monkeypatch.setenv("NAUT_ATTN_VARIANT", e)
        print("named", H, S, D, causal, form, e, flush=True)
        o, lse = torch.full(q.shape, math.nan, device="cuda"), torch.full((1, H, S), math.nan, device="cuda")
        nb.naut_attn_fwd_strided(q, k, v, o, lse, causal, 1.0 / math.sqrt(D))
        torch.cuda.synchronize()
        res.append((o, lse))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])


def test_launches_have_the_key_groups_of_their_class(monkeypatch):
    """Every key group has a reference maximum of its own: with fewer than key_groups() of them fewer keys' P are exactly 1,
    and O is less accurate (up to 1.4 times the error on keys with outliers)."""
    monkeypatch.delenv("NAUT_ATTN_VARIANT", raising=False)
    for D in (64, 72, 80, 96, 128):
        for causal in (True, False):
            for H in (1, 3, 8, 12, 16, 25, 32, 48, 63, 64, 80, 96, 100, 128, 256):
                for S in (1, 129, 257, 300, 511, 513, 640, 768, 900, 1003, 1280, 1536, 2048, 2560, 4096, 8192, 16384):
                    name = nb.kernel_name(1, H, S, D, causal)
                    groups = int(name.split("_g")[1]) if "_g" in name else 1
                    assert groups >= nb.key_groups(1, H, S, D, causal), (H, S, D, causal, name)


def test_kernel_names_of_grids_that_eight_does_not_divide_and_of_short_ones(monkeypatch):
    """Where 4 x 32 queries of the pipelined kernel would take longer than what ran before it, by 3 to 20 %: XCDs that share
    heads, short sequences of many heads just beyond one round, sequences of two to three tiles."""
    monkeypatch.delenv("NAUT_ATTN_VARIANT", raising=False)
    for args, want in (((1, 63, 2304, 128, False), "pipe_8x32"), ((1, 73, 3000, 128, False), "pipe_8x32"), ((1, 43, 3000, 128, True), "pipe_8x32"),
                       ((1, 150, 2100, 128, False), "pipe_8x32"), ((1, 40, 2048, 128, False), "pipe_4x32"), ((1, 63, 2304, 80, True), "pipe_4x32"),
                       ((1, 63, 2700, 64, True), "plain_4x32"), ((1, 192, 384, 128, True), "plain_4x32"), ((1, 144, 512, 96, True), "plain_4x32"),
                       ((1, 256, 256, 128, False), "plain_4x32"), ((1, 512, 256, 64, True), "plain_4x32"), ((1, 512, 288, 64, True), "pipe_4x32"),
                       ((1, 16, 160, 64, True), "plain_4x32"), ((1, 16, 200, 64, True), "plain_2x32_g4"), ((1, 16, 140, 128, True), "plain_4x32")):
        assert nb.kernel_name(*args) == want, args
