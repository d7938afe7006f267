"""The channel aggregation loads a patch's chunks (512 / d rows) in groups whose
size follows C. Every group size and its remainders against the oracle. fp32
arithmetic on bf16 inputs: the bound is a hundred fp32 roundoffs of the norm."""
import numpy as np
import pytest

from oracle import aggregation as agg
import workloads
from gpu_util import rel_l2, to_device, torch

pytestmark = pytest.mark.gpu


def np64(t):
    return t.detach().double().cpu().numpy()


@pytest.mark.parametrize("C,d", [(101, 64), (128, 64), (49, 128), (66, 128)])
def test_large_calls_store_the_bits_of_small_ones(C, d):
    # past 440,000 chunks of more than one group the backward stores whole rows of its lanes
    import paper_2405_15780_amd as va

    t = torch()
    H, chunks = 16, -(-C // (512 // d))
    M = 440000 // (H * chunks) + 8
    print(f"case aggregation large call M={M} H={H} C={C} d={d}", flush=True)
    g = t.Generator(device="cuda").manual_seed(7300 + C)
    q, k, v, do = (t.randn(s, generator=g, device="cuda").bfloat16()
                   for s in ((H, d), (M, H, C, d), (M, H, C, d), (M, H, d)))
    o, lse = va.agg_fwd(q, k, v)
    _, dk, dv = va.agg_bwd(q, k, v, o, lse, do)
    for m in (slice(0, M // 2), slice(M // 2, M)):
        o2, lse2 = va.agg_fwd(q, k[m], v[m])
        _, dk2, dv2 = va.agg_bwd(q, k[m], v[m], o2, lse2, do[m])
        for name, a, b in (("o", o, o2), ("lse", lse, lse2), ("dk", dk, dk2), ("dv", dv, dv2)):
            assert t.equal(a[m], b), name


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("chunks", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 20, 24, 25])
def test_group_sizes_against_the_oracle(chunks, d):
    import paper_2405_15780_amd as va

    rows = 512 // d
    for C in sorted({(chunks - 1) * rows + 2, chunks * rows}):  # a chunk of two rows, and a whole last chunk
        M, H = 5, 3
        print(f"case aggregation groups C={C} d={d}", flush=True)
        x = workloads.make_aggregation_inputs(M, H, C, d, seed=7100 + C + d)
        dev = {n: to_device(a) for n, a in x.items()}
        scale = 1.0 / np.sqrt(d)
        o, lse = va.agg_fwd(dev["q"], dev["k"], dev["v"], scale)
        dq, dk, dv = va.agg_bwd(dev["q"], dev["k"], dev["v"], o, lse, dev["dout"], scale)
        ref = agg.backward(x["q"], x["k"], x["v"], x["dout"], scale)
        for name, got in (("o", o), ("lse", lse), ("dq", dq), ("dk", dk), ("dv", dv)):
            assert rel_l2(np64(got), ref[name]) < 6e-6, (name, C, d)
