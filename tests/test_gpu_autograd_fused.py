"""attention()'s backward for an fp32 upstream gradient converts inside the
kernels. Every form of gradient (layouts the kernels read in place, and ones
that are converted around the plain backward) must give the bits of the
separate conversions: the gradient rounded to bf16, bwd(), its outputs rounded."""
import numpy as np
import pytest

import workloads
from gpu_util import to_device, torch

pytestmark = pytest.mark.gpu


def grads(t, form, shape):
    """An fp32 gradient of this logical shape in one of several layouts."""
    B, H, N, d = shape
    g = t.Generator(device="cuda").manual_seed(97 + N + d)

    def rand(*s):
        return t.randn(s, generator=g, device="cuda")

    if form == "dense":
        return rand(B, H, N, d)
    if form == "bnhd":
        return rand(B, N, H, d).transpose(1, 2)
    if form == "padded":
        return rand(B, H, N, d + 4)[..., :d]
    if form == "odd pitch":  # rows that are not 16-byte aligned
        return rand(B, H, N, d + 1)[..., :d]
    if form == "offset":  # a start that is not 16-byte aligned
        return rand(B * H * N * d + 1)[1:].view(B, H, N, d)
    if form == "shared heads":
        return rand(B, 1, N, d).expand(B, H, N, d)
    if form == "one row":
        return rand(B, H, 1, d).expand(B, H, N, d)
    if form == "scalar":
        return rand(1).expand(B, H, N, d)
    return rand(B, H, d, N).transpose(2, 3)  # "column major"


FORMS = ["dense", "bnhd", "padded", "odd pitch", "offset", "shared heads", "one row", "scalar", "column major"]


def check(q, k, v, g, scale):
    import paper_2405_15780_amd as va

    t = torch()
    leaves = [x.detach().requires_grad_(True) for x in (q, k, v)]
    o = va.attention(*leaves, scale)
    got = t.autograd.grad(o, leaves, g)
    o_ref, lse = va.fwd(q, k, v, scale)
    ref = va.bwd(q, k, v, o_ref, lse, g.to(t.bfloat16).contiguous(), scale)
    assert t.equal(o, o_ref)
    for name, a, b in zip(("dq", "dk", "dv"), got, ref):
        assert a.dtype == t.bfloat16 and a.shape == b.shape and t.equal(a, b.to(t.bfloat16)), name


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("d", [8, 64, 72, 128, 160])
def test_gradient_layouts(form, d):
    t = torch()
    for N in (1, 97, 333):
        print(f"case fused conversions {form} N={N} d={d}", flush=True)
        x = workloads.make_small_inputs(2, 3, N, d, seed=7400 + N + d)
        q, k, v = (to_device(x[n]) for n in ("q", "k", "v"))
        check(q, k, v, grads(t, form, (2, 3, N, d)), 1.0 / np.sqrt(d))


@pytest.mark.parametrize("Nq,Nk", [(16384 - 17, 300), (16384 - 17, 16384 - 17), (16384 - 64, 300), (300, 16384)])
def test_both_sides_of_the_two_sum_limit(Nq, Nk):
    # from 256 query tiles (16,321 rows) dk and dv are two sums added in fp32
    t = torch()
    B, H, d = 1, 2, 64
    print(f"case fused conversions Nq={Nq} Nk={Nk}", flush=True)
    g = t.Generator(device="cuda").manual_seed(7500)
    q, k, v = (t.randn((B, H, n, d), generator=g, device="cuda").bfloat16() for n in (Nq, Nk, Nk))
    check(q, k, v, grads(t, "bnhd", (B, H, Nq, d)), 0.125)


def test_gradient_row_pitch_past_31_bits():
    # rows 2^31 elements apart (heads between them): more than the library's pitch limit, so converted first
    t = torch()
    B, H, N, d = 1, 2, 2, 64
    print("case fused conversions, row pitch 2^31", flush=True)
    x = workloads.make_small_inputs(B, H, N, d, seed=7600)
    q, k, v = (to_device(x[n]) for n in ("q", "k", "v"))
    pitch = 1 << 31
    g = t.empty(pitch + H * d, dtype=t.float32, device="cuda").as_strided((B, H, N, d), (H * d, d, pitch, 1))
    g.copy_(grads(t, "dense", (B, H, N, d)))
    check(q, k, v, g, 0.125)


@pytest.mark.parametrize("kind", ["negated view", "zeros without memory"])
def test_gradients_whose_memory_is_not_their_values(kind):
    # a lazily negated view holds the opposite signs, a lazy zero tensor no memory at all
    t = torch()
    B, H, N, d = 1, 2, 97, 64
    print(f"case fused conversions {kind}", flush=True)
    x = workloads.make_small_inputs(B, H, N, d, seed=7700)
    q, k, v = (to_device(x[n]) for n in ("q", "k", "v"))
    if kind == "negated view":
        g = t._neg_view(grads(t, "dense", (B, H, N, d)))
        assert g.is_neg() and g.is_contiguous()
    else:
        g = t._efficientzerotensor((B, H, N, d), device="cuda")
        assert g.data_ptr() == 0
    check(q, k, v, g, 0.125)
