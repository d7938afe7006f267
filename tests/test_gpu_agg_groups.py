"""The channel aggregation loads a patch's chunks (512 / d rows) in groups whose
size follows C. Every group size and its remainders against the oracle. fp32
arithmetic on bf16 inputs: the bound is a hundred fp32 roundoffs of the norm."""
import numpy as np
import pytest

from oracle import aggregation as agg
import workloads
from gpu_util import rel_l2, to_device

pytestmark = pytest.mark.gpu


def np64(t):
    return t.detach().double().cpu().numpy()


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
