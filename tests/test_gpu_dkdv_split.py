"""GPU parity of the dK/dV kernel's grid balance: from 256 query tiles on, when
the last round of key-block workgroups is at most half full, those key blocks
are split into two workgroups over the two halves of the query tiles, which
add dK and dV into zeroed rows, while whole key blocks form the same two
partial sums (the first stored at the midpoint), so the bits do not depend on
the split. SPLIT puts whole and split key blocks in one launch on a 256-CU
part with one dK/dV workgroup per CU (B*H*ceil(Nk/BK) work items, BK = 128
keys, or in the recompute mode 256 at head dims up to 64 and 192 at 65-80:
260 -> 256 whole + 4 split, 520 -> 512 + 8), over 257 query tiles, an odd
number and the last one ragged, and few keys, which keeps them cheap; the last
key block is ragged too. Both backward modes, every tile width, against the
fp64 oracle, the same heads in calls of their own, and a second run. CASES are
shorter sequences on the same grids, whose key blocks take one sum and are
never split, and one of 16,600 tokens; on any other device the same comparisons
hold whatever the split."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import assert_close, bits, cus, forms, random_qkvg, run_device, run_hip, torch

pytestmark = pytest.mark.gpu

SPLIT = [(64, 26, 2500, False), (72, 52, 1900, False), (96, 26, 1250, False), (128, 26, 1250, False),
         (160, 26, 1250, False), (64, 26, 1250, True), (72, 26, 1250, True), (96, 26, 1250, True),
         (128, 26, 1250, True), (160, 26, 1250, True)]
CASES = [(1, 257, 256, 64), (1, 300, 130, 128), (2, 70, 200, 160), (1, 4, 16600, 64), (1, 33, 1000, 96),
         (1, 45, 1000, 72)]


def np64(t):
    return t.detach().double().cpu().numpy()


@pytest.mark.parametrize("d,H,Nk,store_ds", SPLIT)
def test_whole_and_split_blocks_in_one_launch(d, H, Nk, store_ds):
    t = torch()
    Nq = 16400
    print(f"case dkdv split H={H} Nq={Nq} Nk={Nk} d={d} store_ds={store_ds}", flush=True)
    if cus() == 256:
        f, one = (forms(1, h, Nq, Nk, d, store_ds=store_ds) for h in (H, 1))
        assert (f.dkdv_whole, f.dkdv_split, f.dkdv_rest64) == ((512, 8, 0) if H == 52 else (256, 4, 0))
        assert (one.dkdv_whole, one.dkdv_split) != (256, 4)
    x = random_qkvg(1, H, Nq, Nk, d, seed=7800 + d)
    scale = 1.0 / np.sqrt(d)
    full = run_device(*x, scale, store_ds=store_ds)
    again = run_device(*x, scale, store_ds=store_ds)
    for name in full:  # two fp32 adds onto zero commute: the split blocks' atomics give the same bits on every run
        assert t.equal(full[name], again[name]), name
    for h in (0, H // 2, H - 1):
        one = run_device(*(a[:, h:h + 1].contiguous() for a in x), scale, store_ds=store_ds)
        for name in full:
            assert t.equal(full[name][:, h:h + 1], one[name]), (name, h)
    ref = oracle.forward_backward(*(bits(a[:, H - 1:]) for a in x), scale)
    assert_close({n: np64(a[:, H - 1:]) for n, a in full.items()}, ref, label=f"dkdv split d={d} store_ds={store_ds}")


@pytest.mark.parametrize("store_ds", [False, True], ids=["recompute", "stored-ds"])
@pytest.mark.parametrize("B,H,N,d", CASES)
def test_split_key_blocks_match_oracle(B, H, N, d, store_ds):
    print(f"case dkdv split B={B} H={H} N={N} d={d} store_ds={store_ds}", flush=True)
    x = workloads.make_small_inputs(B, H, N, d, seed=7700 + H + N + d)
    scale = 1.0 / np.sqrt(d)
    got = {n: np64(t) for n, t in run_hip(x, scale, store_ds=store_ds).items()}
    ref = oracle.forward_backward(x["q"], x["k"], x["v"], x["dout"], scale)
    assert_close(got, ref, label=f"dkdv split {B},{H},{N},{d} store_ds={store_ds}")


def test_split_key_blocks_are_deterministic():
    # (three query tiles: no block is split; split blocks are run twice above)
    t = torch()
    B, H, N, d = 1, 300, 130, 128
    print(f"case dkdv split determinism B={B} H={H} N={N} d={d}", flush=True)
    x = workloads.make_small_inputs(B, H, N, d, seed=7799)
    runs = [run_hip(x, 1.0 / np.sqrt(d), store_ds=s) for s in (False, False, True, True)]
    for a, b in ((runs[0], runs[1]), (runs[2], runs[3])):
        for name in ("dq", "dk", "dv"):
            assert t.equal(a[name], b[name]), name


@pytest.mark.parametrize("store_ds", [False, True], ids=["recompute", "stored-ds"])
def test_head_alone_and_among_others(store_ds):
    # N = 25,600 at d = 64 gives 100 key blocks of 256 (200 of 128) per head: on
    # a 256-CU part a head alone takes 128 keys per workgroup or, in the
    # stored-dS mode, 200 whole blocks; three heads are 300 (600) work items,
    # the last 44 (88) split, all of head 2. Every key block sums its query tiles as the same two
    # rounded partials whether it is split or whole, so all five outputs of
    # head 2 are bitwise equal (the check of Sec. VI-A that every process
    # computes the same matrices, here across call shapes).
    t = torch()
    B, H, N, d = 1, 3, 25600, 64
    print(f"case head alone vs among others store_ds={store_ds}", flush=True)
    x = workloads.make_small_inputs(B, H, N, d, seed=7801)
    scale = 1.0 / np.sqrt(d)
    full = run_hip(x, scale, store_ds=store_ds)
    alone = run_hip({n: np.ascontiguousarray(a[:, 2:3]) for n, a in x.items()}, scale, store_ds=store_ds)
    for name in ("o", "lse", "dq", "dk", "dv"):
        assert t.equal(full[name][:, 2:3], alone[name]), name


@pytest.mark.parametrize("B,H,N,d", [(1, 300, 130, 128), (1, 4, 16600, 64), (1, 33, 1000, 96), (2, 70, 200, 160),
                                     (1, 45, 1000, 72)])
def test_split_blocks_bitwise_equal_to_single_head_calls(B, H, N, d):
    # heads of the CASES grids against the same heads in calls of their own,
    # where the grid is far from a whole round
    t = torch()
    print(f"case split vs single-head calls B={B} H={H} N={N} d={d}", flush=True)
    x = workloads.make_small_inputs(B, H, N, d, seed=7900 + H + N + d)
    scale = 1.0 / np.sqrt(d)
    full = run_hip(x, scale)
    for h in sorted({0, H // 2, H - 1}):
        for b in range(B):
            one = run_hip({n: np.ascontiguousarray(a[b:b + 1, h:h + 1]) for n, a in x.items()}, scale)
            for name in ("o", "lse", "dq", "dk", "dv"):
                assert t.equal(full[name][b:b + 1, h:h + 1], one[name]), (name, b, h)
