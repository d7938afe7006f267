"""The key blocks that the dK/dV kernel's whole rounds leave over go to 64-key
workgroups, launched behind them (below 256 query tiles, where no block is
split). The shapes put 258 key blocks (or two more than a whole number of
rounds) on 256 CUs; each head of the launch must give the bits of a call of its
own, which takes another form, and the fp64 oracle's values, in both backward
modes. In the stored-dS mode dQ reads every block that the 64-key workgroups
stored, those past the last key included."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import assert_close, cus, forms, to_device, torch

pytestmark = pytest.mark.gpu


def np64(t):
    return t.detach().double().cpu().numpy()


def run(xq, xk, scale, store_ds, heads):
    import paper_2405_15780_amd as va

    t = torch()
    q, g = (to_device(np.ascontiguousarray(xq[n][:, heads])) for n in ("q", "dout"))
    k, v = (to_device(np.ascontiguousarray(xk[n][:, heads])) for n in ("k", "v"))
    o, lse = va.fwd(q, k, v, scale)
    ws = t.full((va.workspace_bytes_kv(*q.shape[:3], k.shape[2], q.shape[3], 2 * store_ds) // 4,), float("nan"),
                device="cuda")  # a dS block that nothing stores would reach dQ as NaN
    dq, dk, dv = va.bwd(q, k, v, o, lse, g, scale, workspace=ws, store_ds=store_ds)
    t.cuda.synchronize()
    return {"dq": dq, "dk": dk, "dv": dv}


@pytest.mark.parametrize("d,H,Nk,store_ds", [
    (64, 6, 11001, False), (72, 9, 11001, False), (96, 3, 11001, False), (128, 3, 11001, False), (160, 3, 11001, False),
    (64, 3, 11001, True), (72, 3, 11001, True), (96, 3, 11001, True), (128, 3, 11001, True), (160, 3, 11001, True),
    (128, 6, 5441, True)])  # one key in the last 128: three of its four dS blocks lie past it
def test_left_over_blocks(d, H, Nk, store_ds):
    t = torch()
    Nq = 200
    print(f"case left-over key blocks H={H} Nk={Nk} d={d} store_ds={store_ds}", flush=True)
    f, one = (forms(1, h, Nq, Nk, d, store_ds=store_ds) for h in (H, 1))
    if cus() == 256:
        assert f.dkdv_whole >= 256 and f.dkdv_rest64 > 0 and f.dkdv_split == 0
        assert one.dkdv_whole < 256
    xq = workloads.make_small_inputs(1, H, Nq, d, seed=8100 + d)
    xk = workloads.make_small_inputs(1, H, Nk, d, seed=8200 + d, with_dout=False)
    scale = 1.0 / np.sqrt(d)
    full = run(xq, xk, scale, store_ds, list(range(H)))
    for h in (0, H - 2, H - 1):
        alone = run(xq, xk, scale, store_ds, [h])
        for name in full:
            assert t.equal(full[name][:, h:h + 1], alone[name]), (name, h)
    h = slice(H - 1, H)
    ref = oracle.forward_backward(xq["q"][:, h], xk["k"][:, h], xk["v"][:, h], xq["dout"][:, h], scale)
    assert_close({n: np64(a[:, h]) for n, a in full.items()}, ref, names=("dq", "dk", "dv"),
                 label=f"left-over key blocks d={d} store_ds={store_ds}")


@pytest.mark.parametrize("store_ds", [False, True], ids=["recompute", "stored-ds"])
def test_few_blocks_left_over_do_not_take_a_whole_round(store_ds):
    # 258 and 300 key blocks on 256 CUs, 172 and 200 query tiles: the remaining
    # blocks took a whole round of 128-key workgroups, or all blocks 64-key ones
    if cus() != 256:
        pytest.skip("the shapes are made for 256 CUs")
    for d in (96, 128, 160):
        for N, blocks in ((11008, 258), (12800, 300)):
            f = forms(1, 3, N, N, d, store_ds=store_ds)
            assert (f.dkdv_keys, f.dkdv_whole, f.dkdv_rest64) == (128, 256, 2 * (blocks - 256)), (d, N)
