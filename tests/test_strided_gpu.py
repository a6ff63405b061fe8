"""GPU parity of the strided / any-head-dimension entry point (through the C ABI) against the fp64 oracle."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2604_14825_amd import binding as nb
from paper_2604_14825_amd import synth

import gpu_util as gu

pytestmark = pytest.mark.gpu


def make(B, Hq, Hkv, S, D, idt, seed):
    q = synth.fill(B, Hq, S, D, seed, synth.TAG_Q, idt)
    k = synth.fill(B, Hkv, S, D, seed, synth.TAG_K, idt, S // 50, 8.0)
    v = synth.fill(B, Hkv, S, D, seed, synth.TAG_V, idt)
    return q, k, v


def run_strided(qd, kd, vd, od, causal, scale, want_lse=True):
    B, Hq, S, D = qd.shape
    lse = torch.full((B, Hq, S), float("nan"), dtype=torch.float32, device="cuda") if want_lse else None
    nb.naut_attn_fwd_strided(qd, kd, vd, od, lse, causal, scale)
    torch.cuda.synchronize()
    return od.double().cpu().numpy(), (lse.double().cpu().numpy() if want_lse else None)


@pytest.mark.parametrize("variant", ["w8q32", "w4q32", "w4q32g2", "bm128", "bm128g1", "bm128g2"])
@pytest.mark.parametrize("D", [8, 32, 40, 64, 80, 96, 112, 128])
def test_head_dimensions(D, variant, monkeypatch):
    """Every multiple of 8 runs on the next of the 64-, 80-, 96- and 128-wide kernels; contiguous layout."""
    B, Hq, Hkv, S, causal, idt, odt = 1, 4, 2, 333, True, synth.BF16, synth.F32
    gu.use_form(monkeypatch, variant, B, Hq, S, D, causal)
    q, k, v = make(B, Hq, Hkv, S, D, idt, 9000 + D)
    scale = 1.0 / math.sqrt(D)
    print("head dim", D, variant, flush=True)
    qd, kd, vd = (gu.to_device(a, idt) for a in (q, k, v))
    od = torch.full((B, Hq, S, D), float("nan"), dtype=gu.TORCH_DT[odt], device="cuda")
    o, lse = run_strided(qd, kd, vd, od, causal, scale)
    o_ref, lse_ref = oracle.attn_rows(q, k, v, idt, causal, scale)
    gu.check(o, lse, o_ref, lse_ref, "D=%d %s" % (D, variant))


@pytest.mark.parametrize("variant", ["w8q32", "w4q32", "w4q32g2", "bm128", "bm128g1", "bm128g2"])
@pytest.mark.parametrize("D,causal,idt,odt", [(128, True, synth.BF16, synth.BF16), (64, False, synth.F16, synth.F16),
                                             (96, True, synth.BF16, synth.BF16)])
def test_bshd_layout(D, causal, idt, odt, variant, monkeypatch):
    """Tensors stored [B][S][H][D] (sequence-major), passed as transposed views; O written in the same layout."""
    B, Hq, Hkv, S = 2, 6, 2, 300
    gu.use_form(monkeypatch, variant, B, Hq, S, D, causal)
    q, k, v = make(B, Hq, Hkv, S, D, idt, 9100 + D)
    scale = 1.0 / math.sqrt(D)
    bshd = lambda a: gu.to_device(np.ascontiguousarray(a.transpose(0, 2, 1, 3)), idt)   # memory [B][S][H][D]
    qd, kd, vd = bshd(q).transpose(1, 2), bshd(k).transpose(1, 2), bshd(v).transpose(1, 2)  # logical [B,H,S,D]
    assert not qd.is_contiguous()
    o_mem = torch.full((B, S, Hq, D), float("nan"), dtype=gu.TORCH_DT[odt], device="cuda")
    print("bshd", D, variant, flush=True)
    o, lse = run_strided(qd, kd, vd, o_mem.transpose(1, 2), causal, scale)
    o_ref, lse_ref = oracle.attn_rows(q, k, v, idt, causal, scale)
    gu.check(o, lse, o_ref, lse_ref, "bshd D=%d %s" % (D, variant))


def test_padded_rows_and_untouched_gaps():
    """Rows padded to a wider pitch (D = 80 in rows of 128): nothing is read as data from the gaps (they hold
    NaN patterns) and nothing is written into the gaps of O."""
    B, Hq, Hkv, S, D, P = 1, 2, 1, 260, 80, 128
    idt = synth.BF16
    q, k, v = make(B, Hq, Hkv, S, D, idt, 9200)
    scale = 1.0 / math.sqrt(D)

    def padded(a):
        H = a.shape[1]
        buf = np.full((B, H, S, P), 0x7FC0, dtype=np.uint16)  # bf16 NaN in the gaps
        buf[..., :D] = a
        return gu.to_device(buf, idt)[..., :D]
    qd, kd, vd = padded(q), padded(k), padded(v)
    o_buf = torch.full((B, Hq, S, P), 7.0, dtype=torch.float32, device="cuda")
    o, lse = run_strided(qd, kd, vd, o_buf[..., :D], True, scale)
    o_ref, lse_ref = oracle.attn_rows(q, k, v, idt, True, scale)
    gu.check(o, lse, o_ref, lse_ref, "padded rows")
    assert torch.all(o_buf[..., D:] == 7.0).item(), "the gaps between O rows were written"


@pytest.mark.parametrize("variant", ["w8q32", "w4q32", "w4q32g2", "bm128", "bm128g1", "bm128g2"])
@pytest.mark.parametrize("D,odt", [(128, synth.BF16), (64, synth.F16), (80, synth.BF16)])
def test_o_rows_aligned_to_8_bytes_only(D, odt, variant, monkeypatch):
    """16-bit O with a row pitch of D + 4 elements: rows start on 8-byte, not 16-byte, boundaries (the least the
    entry point accepts), the S = 333 rows end in a ragged tile, and the 4-element gaps must stay untouched.
    The pipelined kernels write O in 16-byte pieces of whole rows, so this is their unaligned-store case."""
    B, Hq, Hkv, S = 2, 4, 2, 333
    gu.use_form(monkeypatch, variant, B, Hq, S, D, True)
    idt = odt
    q, k, v = make(B, Hq, Hkv, S, D, idt, 9300 + D)
    scale = 1.0 / math.sqrt(D)
    qd, kd, vd = (gu.to_device(a, idt) for a in (q, k, v))
    o_buf = torch.full((B, Hq, S, D + 4), 7.0, dtype=gu.TORCH_DT[odt], device="cuda")
    print("8-byte O rows", D, variant, flush=True)
    o, lse = run_strided(qd, kd, vd, o_buf[..., :D], True, scale)
    o_ref, lse_ref = oracle.attn_rows(q, k, v, idt, True, scale)
    gu.check(o, lse, o_ref, lse_ref, "8-byte O rows D=%d %s" % (D, variant))
    assert torch.all(o_buf[..., D:] == 7.0).item(), "the gaps between O rows were written"


@pytest.mark.parametrize("D,odt", [(256, synth.BF16), (200, synth.F16), (136, synth.BF16)])
def test_o_rows_aligned_to_8_bytes_only_wide(D, odt):
    """The same on the wide kernels (two O rows per store instruction, 25 or 17 of the 32 chunks of a staged row real
    at D = 200 and 136)."""
    B, Hq, Hkv, S = 1, 4, 2, 333
    idt = odt
    q, k, v = make(B, Hq, Hkv, S, D, idt, 9400 + D)
    scale = 1.0 / math.sqrt(D)
    qd, kd, vd = (gu.to_device(a, idt) for a in (q, k, v))
    o_buf = torch.full((B, Hq, S, D + 4), 7.0, dtype=gu.TORCH_DT[odt], device="cuda")
    print("8-byte O rows, wide kernel", D, flush=True)
    o, lse = run_strided(qd, kd, vd, o_buf[..., :D], True, scale)
    o_ref, lse_ref = oracle.attn_rows(q, k, v, idt, True, scale)
    gu.check(o, lse, o_ref, lse_ref, "8-byte O rows D=%d" % D)
    assert torch.all(o_buf[..., D:] == 7.0).item(), "the gaps between O rows were written"


def test_broadcast_kv_over_batch():
    """Stride 0 on the batch axis of K and V: one cache shared by every batch entry."""
    B, Hq, Hkv, S, D = 3, 4, 4, 200, 64
    idt = synth.BF16
    q, k, v = make(B, Hq, Hkv, S, D, idt, 9300)
    k[1:], v[1:] = k[0], v[0]
    scale = 1.0 / math.sqrt(D)
    qd = gu.to_device(q, idt)
    kd = gu.to_device(k[:1], idt).expand(B, Hkv, S, D)
    vd = gu.to_device(v[:1], idt).expand(B, Hkv, S, D)
    assert kd.stride(0) == 0
    od = torch.full((B, Hq, S, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    o, lse = run_strided(qd, kd, vd, od, False, scale)
    o_ref, lse_ref = oracle.attn_rows(q, k, v, idt, False, scale)
    gu.check(o, lse, o_ref, lse_ref, "broadcast kv")


def test_bshd_prefill_size_sampled_rows():
    """The prefill workload's shape in sequence-major layout, on the default variant, sampled rows."""
    w = synth.WORKLOADS["prefill"]
    q, k, v = synth.make_inputs(w)
    bshd = lambda a: gu.to_device(np.ascontiguousarray(a.transpose(0, 2, 1, 3)), w.in_dtype)
    qd, kd, vd = bshd(q).transpose(1, 2), bshd(k).transpose(1, 2), bshd(v).transpose(1, 2)
    o_mem = torch.full((w.B, w.S, w.Hq, w.D), float("nan"), dtype=torch.bfloat16, device="cuda")
    o, lse = run_strided(qd, kd, vd, o_mem.transpose(1, 2), w.causal, w.scale)
    rows = gu.sample_rows(w, 1500, 77)
    o_ref, lse_ref = oracle.attn_rows(q, k, v, w.in_dtype, w.causal, w.scale, rows=rows)
    gu.check(o.reshape(-1, w.D)[rows], lse.reshape(-1)[rows], o_ref, lse_ref, "bshd prefill")


@pytest.mark.parametrize("D,S,causal,idt,odt", [
    (256, 333, True, synth.BF16, synth.F32),
    (256, 500, False, synth.F16, synth.F16),
    (136, 260, True, synth.BF16, synth.BF16),
    (160, 129, False, synth.BF16, synth.F32),
    (192, 1000, True, synth.F16, synth.F32),
    (248, 97, True, synth.BF16, synth.BF16),
    (256, 1, True, synth.BF16, synth.F32),
])
def test_wide_head_dimensions(D, S, causal, idt, odt):
    """Head dimensions above 128 run on the 192- and 256-wide instantiations of kernel 1 (32 keys per step)."""
    B, Hq, Hkv = 2, 4, 2
    q, k, v = make(B, Hq, Hkv, S, D, idt, 9400 + D + S)
    scale = 1.0 / math.sqrt(D)
    print("wide head dim", D, S, flush=True)
    qd, kd, vd = (gu.to_device(a, idt) for a in (q, k, v))
    od = torch.full((B, Hq, S, D), float("nan"), dtype=gu.TORCH_DT[odt], device="cuda")
    o, lse = run_strided(qd, kd, vd, od, causal, scale)
    o_ref, lse_ref = oracle.attn_rows(q, k, v, idt, causal, scale)
    gu.check(o, lse, o_ref, lse_ref, "D=%d S=%d" % (D, S))


def test_wide_head_bshd_long_sampled_rows():
    """D = 256 at a prefill-sized sequence in sequence-major layout: many key steps, sampled rows."""
    B, Hq, Hkv, S, D, idt = 1, 8, 2, 4096, 256, synth.BF16
    q, k, v = make(B, Hq, Hkv, S, D, idt, 9500)
    scale = 1.0 / math.sqrt(D)
    bshd = lambda a: gu.to_device(np.ascontiguousarray(a.transpose(0, 2, 1, 3)), idt)
    qd, kd, vd = bshd(q).transpose(1, 2), bshd(k).transpose(1, 2), bshd(v).transpose(1, 2)
    o_mem = torch.full((B, S, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    o, lse = run_strided(qd, kd, vd, o_mem.transpose(1, 2), True, scale)
    rng = np.random.default_rng(5)
    rows = np.unique(np.concatenate([rng.integers(0, B * Hq * S, 600), [0, S - 1, B * Hq * S - 1]]))
    o_ref, lse_ref = oracle.attn_rows(q, k, v, idt, True, scale, rows=rows)
    gu.check(o.reshape(-1, D)[rows], lse.reshape(-1)[rows], o_ref, lse_ref, "bshd D=256")


@pytest.mark.parametrize("B,Hq,Hkv,S", [(3, 8, 4, 1024), (9, 8, 2, 300), (1, 80, 8, 513), (13, 8, 1, 300), (1, 136, 8, 257)])
def test_wide_head_groups_of_heads(B, Hq, Hkv, S, monkeypatch):
    """The tile scheduler of the eight-wavefront D = 256 shape with B*Hq a multiple of eight: 24, 72, 80, 104 and 136
    heads are 3, 9, 10, 13 and 17 to an XCD, taken in groups of 3, 9, 10, 7 + 6 and 9 + 8.  Every element of O against
    the four-wavefront shape (the same tiles in the same order: bit-identical), sampled rows against the oracle."""
    D, idt = 256, synth.BF16
    q, k, v = make(B, Hq, Hkv, S, D, idt, 9600)
    scale = 1.0 / math.sqrt(D)
    qd, kd, vd = (gu.to_device(a, idt) for a in (q, k, v))
    for causal in (True, False):
        outs = []
        for variant in ("w8q32", "bm128"):
            monkeypatch.setenv("NAUT_ATTN_VARIANT", variant)
            od = torch.full((B, Hq, S, D), float("nan"), dtype=torch.bfloat16, device="cuda")
            print("wide head groups", B, Hq, S, causal, variant, flush=True)
            outs.append(run_strided(qd, kd, vd, od, causal, scale))
        o, lse = outs[0]
        assert np.isfinite(o).all(), "an output tile was never written"
        assert np.array_equal(o, outs[1][0]) and np.array_equal(lse, outs[1][1])
        rng = np.random.default_rng(6)
        rows = np.unique(np.concatenate([rng.integers(0, B * Hq * S, 2000),
                                         [bh * S + i for bh in range(B * Hq) for i in (0, 255, 256, S - 1)]]))
        o_ref, lse_ref = oracle.attn_rows(q, k, v, idt, causal, scale, rows=rows)
        gu.check(o.reshape(-1, D)[rows], lse.reshape(-1)[rows], o_ref, lse_ref, "D=256, %d heads" % (B * Hq))


@pytest.mark.parametrize("D,variant,mib", [(256, None, 16), (128, "bm128", 16), (128, "w8q32", 16), (64, "w8q32", 16), (64, "bm128", 16),
                                           (256, "w8q32", 16), (128, "bm128g1", 16), (64, "bm128g1", 16), (128, "bm128g2", 16),
                                           (128, "w4q32", 16), (64, "w4q32", 16), (128, "w4q32g2", 8), (64, "w4q32g2", 8),
                                           (128, "w4q32g2", 16), (64, "w4q32g2", 16)])   # more than 8 MiB: kernel 1's two groups
@pytest.mark.parametrize("causal", [True, False])
def test_wide_head_row_stride_beyond_32_bits(D, variant, mib, causal, monkeypatch):
    """K and V rows 16 MiB apart (the largest row stride the entry point admits) or as far as two key groups of the pipelined
    kernel go, on every kernel: S times the stride passes 2^32 bytes, so the tile addresses must be formed in 64 bits (the
    pipelined kernel moves its base past 2^30 several times), and the last row of a tile (the 64th; the 32nd at D = 256, in
    the pipelined kernel and with the four key groups that bm128 runs at D = 128 here) must fit the 32-bit offsets inside
    a tile."""
    B, H, S, idt = 1, 1, 4800 // mib, synth.BF16
    if variant is not None:
        gu.use_form(monkeypatch, variant, B, H, S, D, causal)
    stride = mib << 19  # elements
    q, k, v = make(B, H, H, S, D, idt, 9700)
    scale = 1.0 / math.sqrt(D)
    qd = gu.to_device(q, idt)

    def spread(a):
        buf = torch.empty(S * stride, dtype=torch.bfloat16, device="cuda")  # 4.7 GiB, rows at the start of each pitch
        rows = buf.view(S, stride)[:, :D]
        rows.copy_(gu.to_device(a, idt)[0, 0])
        return rows.unsqueeze(0).unsqueeze(0)  # logical [1,1,S,D]
    kd, vd = spread(k), spread(v)
    assert kd.stride(2) == stride and kd.stride(2) * 2 * S > 1 << 32
    od = torch.full((B, H, S, D), float("nan"), dtype=torch.float32, device="cuda")
    print("row stride of %d MiB" % mib, D, variant, causal, flush=True)
    o, lse = run_strided(qd, kd, vd, od, causal, scale)
    o_ref, lse_ref = oracle.attn_rows(q, k, v, idt, causal, scale)
    gu.check(o, lse, o_ref, lse_ref, "D=%d %s, row stride of %d MiB" % (D, variant, mib))
    if variant == "w4q32g2" and mib > 8:  # still two groups, and their accuracy
        gu.use_form(monkeypatch, "bm128g2", B, H, S, D, causal)
        again = run_strided(qd, kd, vd, torch.full_like(od, float("nan")), causal, scale)
        assert np.array_equal(o, again[0]) and np.array_equal(lse, again[1])


@pytest.mark.parametrize("D,variant", [(72, "w8q32"), (80, "w8q32"), (88, "w8q32"), (96, "w8q32"), (104, "w8q32"),
                                       (72, "bm128"), (88, "bm128"), (96, "bm128"), (104, "bm128"),
                                       (72, "bm128g1"), (88, "bm128g1"), (96, "bm128g2"), (104, "bm128g1"),
                                       (136, ""), (184, ""), (192, ""), (200, "")])
@pytest.mark.parametrize("causal,idt,odt,S", [(True, synth.BF16, synth.BF16, 197), (False, synth.F16, synth.F32, 322)])
def test_compiled_widths(D, variant, causal, idt, odt, S, monkeypatch):
    """Head dimensions on both sides of every width a kernel is compiled for (80, 96, 128, 192, 256), on rows padded
    with NaN patterns: the columns between D and the compiled width must come from the padding of Q, never from
    memory, and nothing may be written there."""
    monkeypatch.setenv("NAUT_ATTN_VARIANT", variant)
    B, Hq, Hkv = 1, 4, 2
    P = D + 24
    q, k, v = make(B, Hq, Hkv, S, D, idt, 9500 + D)
    scale = 1.0 / math.sqrt(D)

    def padded(a):
        buf = np.full(a.shape[:3] + (P,), 0x7FC0 if idt == synth.BF16 else 0x7E00, dtype=np.uint16)
        buf[..., :D] = a
        return gu.to_device(buf, idt)[..., :D]
    o_buf = torch.full((B, Hq, S, P), 7.0, dtype=gu.TORCH_DT[odt], device="cuda")
    print("compiled widths", D, variant, causal, flush=True)
    o, lse = run_strided(padded(q), padded(k), padded(v), o_buf[..., :D], causal, scale)
    o_ref, lse_ref = oracle.attn_rows(q, k, v, idt, causal, scale)
    gu.check(o, lse, o_ref, lse_ref, "D=%d %s" % (D, variant))
    assert torch.all(o_buf[..., D:] == 7.0).item(), "the gaps between O rows were written"
