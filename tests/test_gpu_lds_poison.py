"""The LDS-poison debug build (-DVITATTN_DEBUG_LDS_POISON): every kernel first
fills its LDS with all-ones bytes, NaN as bf16 and as fp32, so a read of LDS
that nothing wrote would turn outputs into NaN. Each case runs through the
normal library and then through the poisoned one (swapped in for the
package's library), and every output must be equal bitwise: forward and both
backward modes over ragged tails, Nq != Nk, every tile width and a
sequence-major layout, the merge and the channel aggregation. The short cases
take the kernels' narrow forms; FULL fills 256 CUs and takes the wide ones
(eight waves per workgroup in the forward and dQ, twelve where there are such,
the widest dK/dV with 64-key workgroups behind it, and split key blocks)."""
import os

import numpy as np
import pytest

import workloads
from gpu_util import cus, forms, random_qkvg, to_device, torch

pytestmark = pytest.mark.gpu


# H, Nq, Nk, d and what the recompute mode takes: forward and dQ waves, dK/dV keys, split blocks
FULL = [(64, 1001, 2501, 64, 8, 8, 256, 0), (64, 1001, 2501, 72, 8, 8, 128, 0), (64, 1001, 2501, 88, 8, 8, 128, 0),
        (64, 1001, 2501, 128, 8, 8, 128, 0), (64, 1001, 2501, 160, 8, 8, 128, 0), (64, 1530, 2501, 64, 12, 12, 256, 0),
        (64, 1530, 2501, 72, 4, 12, 128, 0), (9, 200, 11001, 72, 4, 4, 192, 0), (26, 16400, 2500, 64, 4, 8, 256, 4),
        (52, 16400, 1900, 72, 4, 12, 192, 8), (26, 16400, 1250, 96, 4, 4, 128, 4), (26, 16400, 1250, 128, 4, 8, 128, 4),
        (26, 16400, 1250, 160, 4, 8, 128, 4)]


def test_full_grids_take_the_wide_forms():
    if cus() != 256:
        pytest.skip("the shapes are made for 256 CUs")
    for H, Nq, Nk, d, fwd, dq, keys, split in FULL:
        f = forms(1, H, Nq, Nk, d)
        assert (f.fwd_waves, f.dq_waves, f.dkdv_keys, f.dkdv_split) == (fwd, dq, keys, split), (H, Nq, Nk, d)
        assert f.dkdv_whole >= 256


@pytest.mark.parametrize("H,Nq,Nk,d", [c[:4] for c in FULL])
def test_poisoned_lds_changes_no_output_on_full_grids(H, Nq, Nk, d):
    import paper_2405_15780_amd as va
    import paper_2405_15780_amd.binding as b
    from paper_2405_15780_amd._build import LDS_POISON_LIB_PATH

    t = torch()
    print(f"case LDS poison full grid H={H} Nq={Nq} Nk={Nk} d={d}", flush=True)
    q, k, v, g = random_qkvg(1, H, Nq, Nk, d, seed=9300 + d)
    normal = b.library()
    libs = (normal, b.open_library(LDS_POISON_LIB_PATH))
    try:
        for store_ds in (False, True):
            ref = None
            for lib in libs:
                b._lib = lib
                o, lse = va.fwd(q, k, v)
                got = (o, lse) + tuple(va.bwd(q, k, v, o, lse, g, store_ds=store_ds))
                t.cuda.synchronize()
                if ref is None:
                    ref = got
            for name, x, y in zip(("o", "lse", "dq", "dk", "dv"), ref, got):
                assert bool(t.isfinite(y).all()), f"{name}: non-finite values with poisoned LDS"
                assert t.equal(x, y), f"{name} differs when the kernels' LDS starts as NaN (store_ds={store_ds})"
            t.cuda.empty_cache()
    finally:
        b._lib = normal


def _outputs():
    import paper_2405_15780_amd as va

    t = torch()
    res = {}
    cases = [(1, 2, 300, 300, 64), (2, 1, 129, 77, 128), (1, 1, 1, 1, 8), (1, 2, 200, 450, 72), (1, 1, 257, 130, 160),
             (2, 3, 70, 600, 96)]
    for ci, (B, H, Nq, Nk, d) in enumerate(cases):
        xq = workloads.make_small_inputs(B, H, Nq, d, seed=9000 + ci)
        xk = workloads.make_small_inputs(B, H, Nk, d, seed=9100 + ci, with_dout=False)
        scale = 1.0 / np.sqrt(d)
        bnhd = ci % 2 == 1

        def put(bits):
            if bnhd:
                return to_device(np.ascontiguousarray(bits.transpose(0, 2, 1, 3))).transpose(1, 2)
            return to_device(bits)

        q, k, v, g = put(xq["q"]), put(xk["k"]), put(xk["v"]), put(xq["dout"])
        o, lse = va.fwd(q, k, v, scale)
        res[f"case {ci} o"], res[f"case {ci} lse"] = o, lse
        for store_ds in (False, True):
            dq, dk, dv = va.bwd(q, k, v, o, lse, g, scale, store_ds=store_ds)
            for n, x in (("dq", dq), ("dk", dk), ("dv", dv)):
                res[f"case {ci} {n} store_ds={store_ds}"] = x
    rng = np.random.default_rng(5)
    parts = t.from_numpy(rng.standard_normal((3, 1, 2, 77, 72)).astype(np.float32)).cuda()
    lparts = t.from_numpy(rng.standard_normal((3, 1, 2, 77)).astype(np.float32)).cuda()
    res["merge o"], res["merge lse"] = va.merge(parts, lparts)
    for M, H, C, d in ((3, 2, 92, 64), (5, 3, 200, 128), (1, 1, 1, 64)):
        x = workloads.make_aggregation_inputs(M, H, C, d, seed=9200 + C)
        dev = {n: to_device(a) for n, a in x.items()}
        o, lse = va.agg_fwd(dev["q"], dev["k"], dev["v"])
        dq, dk, dv = va.agg_bwd(dev["q"], dev["k"], dev["v"], o, lse, dev["dout"])
        for n, y in (("o", o), ("lse", lse), ("dq", dq), ("dk", dk), ("dv", dv)):
            res[f"agg {M},{H},{C},{d} {n}"] = y
    t.cuda.synchronize()
    return res


def test_poisoned_lds_changes_no_output():
    import paper_2405_15780_amd.binding as b
    from paper_2405_15780_amd._build import LDS_POISON_LIB_PATH

    t = torch()
    print("case LDS poison build", flush=True)
    assert os.path.exists(LDS_POISON_LIB_PATH), "build() compiles the LDS-poison variant beside the library"
    normal = b.library()
    ref = _outputs()
    b._lib = b.open_library(LDS_POISON_LIB_PATH)
    try:
        got = _outputs()
    finally:
        b._lib = normal
    for name, x in ref.items():
        y = got[name]
        assert bool(t.isfinite(y).all()) == bool(t.isfinite(x).all()), f"{name}: non-finite values with poisoned LDS"
        assert t.equal(x, y), f"{name} differs when the kernels' LDS starts as NaN"
