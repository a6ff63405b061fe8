"""Decode split kernels at the edges of their blocks, splits and wavefronts: one split and several, half and all
wavefronts, one query row to more than a tile, and every form of the in-LDS merge.

The reference is attention in float64 on the same 16-bit (FP8: dequantised) inputs.  O may differ by the rounding of P and
of O to the input type: relative to the rows' largest |V| each is at most 2^-9 (bf16); FP8 rounds P to 4 bits (2^-4 per
weight, averaging over the keys; the worst row holds one key).
"""
import math

import pytest
import torch

from paper_2604_14825_amd import binding

pytestmark = pytest.mark.gpu

# D, Hkv, query heads per K/V head, Sq
ROWS = [(128, 8, 1, 1), (128, 2, 4, 4), (128, 3, 16, 1), (72, 2, 8, 5), (64, 4, 2, 1), (64, 2, 8, 4), (256, 2, 4, 1), (200, 2, 8, 4)]
# in blocks of 32 keys: a block, half the wavefronts, all of them, one split and the first with several
BLOCKS = (1, 2, 4, 5, 8, 9, 16, 17, 33)


def reference(q, k, v, scale, dtype=torch.float64):
    B, Hq, Sq, D = q.shape
    Hkv, Sk = k.shape[1:3]
    g = Hq // Hkv
    q, k, v = (x.to(dtype) for x in (q, k, v))
    k, v = k.repeat_interleave(g, 1), v.repeat_interleave(g, 1)
    s = torch.matmul(q, k.transpose(-1, -2).contiguous()) * scale
    lim = Sk - Sq + torch.arange(Sq, device=q.device)
    s = s.masked_fill(torch.arange(Sk, device=q.device)[None, :] > lim[:, None], -math.inf)
    return torch.matmul(torch.softmax(s, -1), v), torch.logsumexp(s, -1)


def run(q, k, v, scale, fp8=None):
    B, Hq, Sq, D = q.shape
    Hkv, Sk = k.shape[1:3]
    L = binding.lib()
    ws = torch.empty(L.naut_attn_decode_workspace_bytes(B, Hq, Hkv, Sq, Sk, D), device="cuda", dtype=torch.uint8)
    o = torch.full((B, Hq, Sq, D), math.nan, device="cuda", dtype=torch.bfloat16)
    lse = torch.full((B, Hq, Sq), math.nan, device="cuda")
    st = binding.NautStrides(*([Hq * Sq * D, Sq * D, D] + [Hkv * Sk * D, Sk * D, D] * 2 + [Hq * Sq * D, Sq * D, D]))
    stream = torch.cuda.current_stream().cuda_stream
    ptr = [x.data_ptr() for x in (q, k, v, o, lse)]
    if fp8 is None:
        rc = L.naut_attn_decode_strided(*ptr, B, Hq, Hkv, Sq, Sk, D, 1, scale, ws.data_ptr(), ws.numel(), stream, 0, 0, st)
    else:
        rc = L.naut_attn_decode_fp8_strided(*ptr, B, Hq, Hkv, Sq, Sk, D, 1, scale, *fp8, ws.data_ptr(), ws.numel(), stream, st)
    assert rc == 0, L.naut_last_error_string()
    return o, lse


@pytest.mark.parametrize("D,Hkv,g,Sq", ROWS)
@pytest.mark.parametrize("B", [1, 140])  # fewer and more work-groups than CUs
def test_block_and_split_edges(D, Hkv, g, Sq, B):
    torch.manual_seed(D + g + B)
    for nb in BLOCKS:
        for Sk in {nb * 32, nb * 32 - 31 if nb > 1 else max(Sq, 9)}:
            if B > 1 and nb > 17:
                continue
            q = torch.randn(B, Hkv * g, Sq, D, device="cuda").bfloat16()
            k, v = (torch.randn(B, Hkv, Sk, D, device="cuda").bfloat16() for _ in range(2))
            scale = 1 / math.sqrt(D)
            o, lse = run(q, k, v, scale)
            ro, rl = reference(q, k, v, scale)
            bound = 2 ** -8 * v.abs().max().item()
            assert (o.double() - ro).abs().max().item() <= bound, (D, Hkv, g, Sq, B, Sk)
            assert (lse.double() - rl).abs().max().item() <= 2e-5, (D, Hkv, g, Sq, B, Sk)
            again = run(q, k, v, scale)
            assert torch.equal(o, again[0]) and torch.equal(lse, again[1]), (D, Hkv, g, Sq, B, Sk)


@pytest.mark.parametrize("D,Hkv,g,Sq", [r for r in ROWS if r[0] in (64, 128)])
@pytest.mark.parametrize("B", [1, 140])
def test_block_and_split_edges_fp8(D, Hkv, g, Sq, B):
    torch.manual_seed(D + g + B)
    for nb in BLOCKS:
        for Sk in {nb * 64, nb * 64 - 63 if nb > 1 else max(Sq, 9)}:
            if B > 1 and nb > 17:
                continue
            q, k, v = (torch.randn(B, h, s, D, device="cuda").to(torch.float8_e4m3fn) for h, s in ((Hkv * g, Sq), (Hkv, Sk), (Hkv, Sk)))
            scale = 1 / math.sqrt(D)
            o, lse = run(*(x.view(torch.uint8) for x in (q, k, v)), scale, (1.0, 1.0, 1.0))
            ro, rl = reference(q.float(), k.float(), v.float(), scale)
            # every weight within 2^-4 of itself, and the store's 2^-9
            bound = (2 ** -4 + 2 ** -8) * v.float().abs().max().item()
            assert (o.double() - ro).abs().max().item() <= bound, (D, Hkv, g, Sq, B, Sk)
            # one matrix instruction adds 64 exact products aligned to the largest of them: at most 64 * 2^-20 of that product
            # (|q| |k| < 25 here), times scale <= 1/8
            assert (lse.double() - rl).abs().max().item() <= 2e-4, (D, Hkv, g, Sq, B, Sk)
            again = run(*(x.view(torch.uint8) for x in (q, k, v)), scale, (1.0, 1.0, 1.0))
            assert torch.equal(o, again[0]) and torch.equal(lse, again[1]), (D, Hkv, g, Sq, B, Sk)


@pytest.mark.parametrize("D,fp8", [(64, False), (64, True), (128, False), (128, True), (256, False)])
def test_one_split_is_two_blocks_a_wavefront(D, fp8):
    """Up to two blocks for each wavefront one split stores O itself and leaves the workspace alone; from there on there are
    several, at every width: fewer partials than that are fewer keys whose P is exactly 1."""
    limit = 2 * (4 if D > 128 else 8) * (64 if fp8 else 32)
    L = binding.lib()
    for Sk in (limit - 1, limit, limit + 1, 2 * limit):
        x = [torch.randn(1, h, s, D, device="cuda") for h, s in ((4, 1), (2, Sk), (2, Sk))]
        q, k, v = (t.to(torch.float8_e4m3fn).view(torch.uint8) if fp8 else t.bfloat16() for t in x)
        o, lse = torch.empty(1, 4, 1, D, device="cuda", dtype=torch.bfloat16), torch.empty(1, 4, 1, device="cuda")
        ws = torch.full((L.naut_attn_decode_workspace_bytes(1, 4, 2, 1, Sk, D),), 0xA5, device="cuda", dtype=torch.uint8)
        if fp8:
            binding.naut_attn_decode_fp8(q, k, v, o, lse, True, 0.1, 1.0, 1.0, 1.0, ws)
        else:
            binding.naut_attn_decode_strided(q, k, v, o, lse, True, 0.1, ws)
        torch.cuda.synchronize()
        assert bool((ws == 0xA5).all()) == (Sk <= limit), (D, fp8, Sk)
