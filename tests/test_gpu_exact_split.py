"""Exact fp32 attention on split operands: accuracy over value ranges, and values
that are not finite, which take the fp32 matrix cores."""
import numpy as np
import pytest
import torch

from paper_2506_08520_amd import binding as B

pytestmark = pytest.mark.gpu


def qkv(units, N, d, seed, scale=1.0):
    g = torch.Generator().manual_seed(seed)
    return [torch.randn(units, 1, N, d, generator=g) * scale for _ in range(3)]


def softmax64(q, k, v):
    q, k, v = (t.double() for t in (q, k, v))
    return torch.softmax(q.shape[-1] ** -0.5 * (q @ k.transpose(-1, -2)), -1) @ v


# The fp32 matrix cores (N = 64, 128; one query tile per wave), the split kernel (256 to
# 448 in steps of 64 with four to seven waves, and multiples of 512 with eight, several
# workgroups per unit), and multiples of 64 that neither takes (192, 576); every width
@pytest.mark.parametrize("N,d", [(64, 8), (128, 12), (192, 16), (256, 20), (256, 24), (320, 16),
                                 (384, 8), (448, 30), (512, 28), (576, 30), (1024, 30), (256, 32)])
@pytest.mark.parametrize("scale", [1e-3, 1.0, 4.0])
def test_accuracy(N, d, scale):
    q, k, v = qkv(3, N, d, N + d, scale)
    ref = softmax64(q, k, v)
    out = B.nystra_exact_attn_forward(*(t.cuda() for t in (q, k, v))).cpu().double()
    # Roundings of 2^-24 (u): a row's N terms add up in chains of N / 32 matrix
    # steps of six products, and the result of N near-equal weights is smaller
    # than the terms by sqrt(N): sqrt(6 N / 32) u on the sum, N / 16 u at worst on
    # the row sum of equal terms; scores of size s = scale^2 sqrt(d) carry s u
    # into the exponent.  (The fp32 matrix cores measured 1.4e-6 at N = 1024,
    # scale 1e-3, and 1.1e-6 at scale 4.)
    u = 2.0 ** -24
    bound = u * ((6 * N / 32) ** 0.5 + N / 16 + 2 * scale ** 2 * d ** 0.5 + 4)
    rel = ((out - ref).norm() / ref.norm()).item()
    print(f"exact split N={N} d={d} scale={scale}: rel {rel:.2e} (bound {bound:.2e})")
    assert rel <= bound


@pytest.mark.parametrize("N", [64, 256, 320, 512])
def test_values_that_are_not_finite(N):
    """-inf keys mask (probability 0), inf in V and NaN reach what they touch and
    nothing else: as a plain fp32 evaluation gives it."""
    d = 32
    q, k, v = qkv(6, N, d, 5)
    q = q.abs() + 0.5
    k[0, 0, 3] = float("-inf")             # a masked key: every score -inf
    k[0, 0, N - 1] = float("-inf")
    v[1, 0, 7, 2] = float("inf")
    v[2, 0, N - 2, d - 1] = float("nan")
    q[3, 0, 5, 0] = float("nan")           # one query row
    k[4, 0, 1, 1] = float("nan")           # the whole unit
    ref = softmax64(q, k, v)
    out = B.nystra_exact_attn_forward(*(t.cuda() for t in (q, k, v))).cpu().double()
    assert torch.equal(torch.isnan(out), torch.isnan(ref))
    assert torch.equal(torch.isinf(out), torch.isinf(ref))
    ok = torch.isfinite(ref)
    assert (out[ok] - ref[ok]).abs().max() <= 1e-4
    assert torch.isfinite(out[0]).all() and torch.isfinite(out[5]).all()
    assert np.isfinite(out[3, 0, :5].numpy()).all() and torch.isnan(out[3, 0, 5]).all()
