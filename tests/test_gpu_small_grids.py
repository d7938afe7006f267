"""Grids that leave CUs idle take narrower workgroups (the forward and dQ: four
waves, 128 queries). One call over 64 heads of 1,001 queries and 2,501 keys
fills 256 CUs with eight-wave workgroups; a single head of it takes the narrow
ones. Every output must be bitwise equal between the two, and single calls at
the edges of the narrow tiles must match the fp64 oracle."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import assert_close, bits, cus, forms, random_qkvg, run_device, run_hip, torch

pytestmark = pytest.mark.gpu


def np64(t):
    return t.detach().double().cpu().numpy()


@pytest.mark.parametrize("store_ds", [False, True])
@pytest.mark.parametrize("d", [64, 72, 96, 128, 160])
def test_single_heads_equal_the_full_grid(d, store_ds):
    t = torch()
    H, Nq, Nk = 64, 1001, 2501
    print(f"case small grids H={H} Nq={Nq} Nk={Nk} d={d} store_ds={store_ds}", flush=True)
    if cus() == 256:
        f, one = (forms(1, h, Nq, Nk, d, store_ds=store_ds) for h in (H, 1))
        assert (f.fwd_waves, one.fwd_waves) == (8, 4)
        assert (f.dq_waves, one.dq_waves) == (8, 8 if store_ds else 4)  # dQ from stored dS has one form
        assert f.dkdv_whole >= 256 and one.dkdv_whole < 256
    x = random_qkvg(1, H, Nq, Nk, d, seed=6100 + d)
    scale = 1.0 / np.sqrt(d)
    full = run_device(*x, scale, store_ds=store_ds)
    for h in (0, 37, 63):
        one = run_device(*(a[:, h:h + 1].contiguous() for a in x), scale, store_ds=store_ds)
        for name in ("o", "lse", "dq", "dk", "dv"):
            assert t.equal(full[name][:, h:h + 1], one[name]), (name, h)
    ref = oracle.forward_backward(*(bits(a[:, 63:]) for a in x), scale)
    assert_close({n: np64(a[:, 63:]) for n, a in full.items()}, ref, label=f"full grid d={d} store_ds={store_ds}")


@pytest.mark.parametrize("N", [1, 31, 97, 127, 128, 129, 255, 385])
@pytest.mark.parametrize("d", [40, 72, 88, 128, 160])
def test_tile_edges_against_the_oracle(d, N):
    print(f"case small grids, tile edges N={N} d={d}", flush=True)
    x = workloads.make_small_inputs(1, 2, N, d, seed=6200 + N + d)
    scale = 1.0 / np.sqrt(d)
    got = {n: np64(a) for n, a in run_hip(x, scale).items()}
    ref = oracle.forward_backward(x["q"], x["k"], x["v"], x["dout"], scale)
    assert_close(got, ref, label=f"small grids N={N} d={d}")


# From 256 query tiles on, key blocks of a last round that is at most half full
# are split over two workgroups. On 256 CUs these grids split 128 of 640 blocks
# (d = 64, 128, 160) and 90 of 602 (d = 72); a single head takes another form
# (narrower blocks, or in the stored-dS mode all of its blocks split).
@pytest.mark.parametrize("d,H,store_ds", [(64, 10, False), (72, 7, False), (128, 5, False), (128, 5, True), (160, 5, False)])
def test_split_key_blocks_equal_whole_ones(d, H, store_ds):
    t = torch()
    B, N = 1, 16384 - 17
    print(f"case split key blocks H={H} N={N} d={d} store_ds={store_ds}", flush=True)
    if cus() == 256:
        f, one = (forms(B, h, N, N, d, store_ds=store_ds) for h in (H, 1))
        assert (f.dkdv_whole, f.dkdv_split) == ((512, 90) if d == 72 else (512, 128))
        assert one.dkdv_keys < f.dkdv_keys or one.dkdv_whole == 0
    x = workloads.make_small_inputs(B, H, N, d, seed=6300 + d)
    scale = 1.0 / np.sqrt(d)
    full = run_hip(x, scale, store_ds=store_ds)
    for h in (0, H - 1):
        one = run_hip({n: np.ascontiguousarray(a[:, h:h + 1]) for n, a in x.items()}, scale, store_ds=store_ds)
        for name in ("o", "lse", "dq", "dk", "dv"):
            assert t.equal(full[name][:, h:h + 1], one[name]), (name, h)
    if d == 128 and not store_ds:
        h = H - 1
        lse, D = oracle.row_statistics(x["q"], x["k"], x["v"], x["dout"], scale, 0, h)
        keys = np.sort(np.random.default_rng(d).choice(N, 32, replace=False))
        dk, dv = oracle.key_rows(x["q"], x["k"], x["v"], x["dout"], scale, 0, h, keys, lse, D)
        kk = t.from_numpy(keys).cuda()
        assert_close({"dk": np64(full["dk"][0, h][kk]), "dv": np64(full["dv"][0, h][kk])}, {"dk": dk, "dv": dv},
                     names=("dk", "dv"), label="split key blocks, sampled key rows")
