"""Prefill parity on the GPU: tk_attn_prefill against the fp64 oracle on the same
seeded inputs — every output at sweep sizes and at the GPT-2 fp32 size, and
65 rows of every sequence (all heads) at the Mistral 8192-token size in the launch
configuration the benchmark times — plus causal invariants."""
import pytest
import torch

import paper_2603_04427_amd as tk
from gpu_cases import device, gate, prefill_on_gpu, prefill_oracle, prefill_rows_oracle, say
from synth import FULLKEY, WORKLOADS, PrefillSpec, make_prefill, with_shape

pytestmark = pytest.mark.gpu

BASE = PrefillSpec("sweep", 600, 2, 4, 2, 200, 200, 32, 128, dtype="bf16", amp=1.0)


def run_full(spec, structured=False):
    dev = device()
    p = make_prefill(spec, structured=structured)
    say(f"prefill {spec} structured={structured}")
    out = prefill_on_gpu(p, spec, dev)
    torch.cuda.synchronize()
    return out, prefill_oracle(p, spec)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("r", [16, 32, 64, 128])
@pytest.mark.parametrize("dv", [64, 128])
def test_sweep_widths(dtype, r, dv):
    spec = with_shape(BASE, config_id=600 + r + dv, r=r, d_v=dv, dtype=dtype)
    for structured in (False, True):
        out, ref = run_full(spec, structured)
        gate(out, ref, dtype, f"{spec} structured={structured}")


SHAPES = [  # (B, Hq, Hkv, Sq, Sk, causal)
    (1, 1, 1, 1, 1, True),
    (1, 2, 1, 31, 31, True),
    (2, 4, 4, 33, 33, True),
    (1, 8, 2, 100, 100, False),
    (1, 4, 2, 64, 200, True),     # bottom-right alignment: 64 new rows after 136 cached keys
    (1, 4, 1, 5, 300, True),
    (2, 6, 2, 257, 257, True),    # G = 3
    (1, 16, 2, 130, 130, True),   # G = 8
    (1, 2, 2, 65, 129, False),
]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("shape", SHAPES)
def test_shapes_and_masks(dtype, shape):
    B, Hq, Hkv, Sq, Sk, causal = shape
    spec = with_shape(BASE, config_id=700, batch=B, h_q=Hq, h_kv=Hkv, seq_q=Sq, seq_k=Sk, causal=causal,
                      dtype=dtype, r=32 if dtype == "bf16" else 16, d_v=128 if dtype == "bf16" else 64)
    out, ref = run_full(spec, structured=True)
    gate(out, ref, dtype, str(spec))


WORKGROUP_WIDTHS = [(16, 64), (32, 128), (64, 64), (64, 128), (128, 128)]
WORKGROUP_SHAPES = [  # units of 32 rows of one head; every form of every width (waves per tile x key groups)
    (1, 6, 2, 1050, 1050, True),   # 198 units: one unit per workgroup, G = 3, a ragged 17th tile
    (1, 4, 1, 130, 190, False),    # 3 tiles: split in two at most
    (5, 20, 5, 70, 300, True),     # 300 units over a prefix: two per workgroup, key groups without a fifth tile
    (9, 20, 5, 90, 530, True),     # 540 units, rows of equal walks: two units x 2, four for wide values
    (9, 20, 5, 90, 100, True),     # 540 units, 2 tiles: two units x 2 for narrow values, four units whole for wide
    (4, 12, 12, 700, 1030, True),  # 1056 units on a causal ramp of 17 tiles: two units x 2, four for wide values
]


@pytest.mark.parametrize("r,dv", WORKGROUP_WIDTHS)
@pytest.mark.parametrize("shape", WORKGROUP_SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_workgroup_shapes(shape, r, dv):
    """The bf16 workgroup shapes for few rows (waves per tile x key groups), every output."""
    B, Hq, Hkv, Sq, Sk, causal = shape
    spec = with_shape(BASE, config_id=750 + r, batch=B, h_q=Hq, h_kv=Hkv, seq_q=Sq, seq_k=Sk, causal=causal, r=r, d_v=dv)
    for structured in (False, True):
        out, ref = run_full(spec, structured)
        gate(out, ref, "bf16", f"{spec} structured={structured}")


ORDERS = [  # four units whole, at every width; the order of their workgroups
    ((4, 64, 8, 300, 300, True), "owned"),           # two head groups per KV sequence, 64 pairs: 10 ragged blocks each
    ((12, 28, 4, 50, 60, True), "owned"),            # seven head groups, 336 pairs: an eighth ends inside a sequence
    ((3, 28, 4, 50, 60, True), "by sequence"),       # 84 pairs: their number doesn't divide among the XCDs
    ((25, 33, 33, 140, 140, False), "by sequence"),  # 825 pairs of 2 blocks, equal walks over more than one round
    ((25, 33, 33, 60, 90, True), "longest first"),   # 825 pairs on a ramp
]


@pytest.mark.parametrize("r,dv", [(32, 64), *WORKGROUP_WIDTHS])
@pytest.mark.parametrize("shape,order", ORDERS)
def test_workgroup_orders(shape, order, r, dv):
    """Every output where the workgroups take each of their orders."""
    B, Hq, Hkv, Sq, Sk, causal = shape
    spec = with_shape(BASE, config_id=770 + r, batch=B, h_q=Hq, h_kv=Hkv, seq_q=Sq, seq_k=Sk, causal=causal, r=r, d_v=dv)
    out, ref = run_full(spec, structured=True)
    gate(out, ref, "bf16", f"{spec} {order}")


def test_gpt2_prefill_f32_full():
    """GPT-2 small shape, fp32, every output against the oracle (gate 1e-4)."""
    spec = WORKLOADS["gpt2_prefill_f32"]
    for structured in (False, True):
        out, ref = run_full(spec, structured)
        mx, rel = gate(out, ref, "f32", f"gpt2 structured={structured}")
        say(f"  max-abs {mx:.2e} rel-L2 {rel:.2e}")


# first and last row of 32-row wave blocks (and of 64-key tiles) at causal depths
# from the first tile to the last, plus interior rows: 65 rows per sequence
BLOCKS = [0, 1, 2, 3, 7, 15, 31, 32, 63, 64, 100, 127, 128, 129, 191, 200, 223, 240, 250, 253, 254, 255]
ROWS = sorted({32 * kb + d for kb in BLOCKS for d in (0, 31)} | {5, 17, 47, 48, 95, 1000, 2049, 3071, 4096,
                                                                    4111, 5000, 6143, 7000, 7777, 8000,
                                                                    8100, 8129, 8150, 8160, 8175, 8180,
                                                                    8185, 8189, 8190, 2, 33, 1023, 1024, 4095})


@pytest.mark.parametrize("structured", [False, True])
@pytest.mark.parametrize("name", ["mistral_prefill_s8192", "mistral_prefill_s8192_fullkey"])
def test_mistral_prefill_s8192_full_sampled(name, structured):
    """Batch 4, 32/8 heads, 8192 tokens, d_v 128, bf16, thin keys (r 32) and the
    full-key control (r 128): the whole call on the GPU, 65 rows of every sequence
    (all heads) against the oracle."""
    dev = device()
    spec = {**WORKLOADS, **FULLKEY}[name]
    p = make_prefill(spec, device=dev, structured=structured)
    say(f"prefill full {spec.name} structured={structured}")
    out = prefill_on_gpu(p, spec, dev)
    torch.cuda.synchronize()
    assert len(ROWS) >= 64
    for b in range(spec.batch):
        ref = prefill_rows_oracle(p, spec, b, ROWS)                  # [n, Hq, dv]
        got = out[b, :, ROWS].permute(1, 0, 2)
        mx, rel = gate(got, ref, "bf16", f"b={b}")
        say(f"  b={b} max-abs {mx:.2e} rel-L2 {rel:.2e}")


def test_causal_future_perturbation_bitwise():
    dev = device()
    spec = with_shape(BASE, config_id=800, seq_q=300, seq_k=300)
    p = make_prefill(spec, structured=True)
    a = prefill_on_gpu(p, spec, dev)
    i = 150
    p2 = {k: v.clone() for k, v in p.items()}
    p2["k"][:, :, i + 1:] = 3.0
    p2["v"][:, :, i + 1:] = -7.0
    say("prefill future perturbation")
    b = prefill_on_gpu(p2, spec, dev)
    assert torch.equal(a[:, :, :i + 1], b[:, :, :i + 1])
    assert not torch.equal(a[:, :, i + 1:], b[:, :, i + 1:])
    assert torch.equal(a, prefill_on_gpu(p, spec, dev))   # deterministic


@pytest.mark.parametrize("seq,r", [(6300, 32), (6145, 64)])   # just past the line, ragged query blocks
def test_long_batch_ordered_by_sequence(seq, r):
    """Eight long sequences run one after the other within each XCD; alone, each runs
    longest walk first with the same arithmetic, so the rows agree bit for bit."""
    dev = device()
    g = torch.Generator(device=dev).manual_seed(seq)
    q, k, v = (torch.randn(8, h, seq, w, generator=g, device=dev, dtype=torch.bfloat16)
               for h, w in ((32, r), (8, r), (8, 128)))
    say(f"prefill by sequence {seq} r {r}")
    out = tk.tk_attn_prefill(q, k, v)
    for b in range(8):
        assert torch.equal(out[b:b + 1], tk.tk_attn_prefill(q[b:b + 1], k[b:b + 1], v[b:b + 1])), b
