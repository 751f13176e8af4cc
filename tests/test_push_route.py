"""A push's history update rides in the batch's launch. Where the fused kernel is
slower for it, batches have a kernel without it, and pushes of more than 2^25
samples take that and update the history in a second launch.
"""
import numpy as np
import pytest

from paper_1411_3656_amd import ppf
from tests import launches

# N, taps, the kernel, whether its long pushes keep one launch
SHAPES = [(64, 8, "ppf_fused_kernel", False), (1024, 3, "ppf_fused_kernel", True), (4096, 4, "ppf_fused_kernel", True), (256, 12, "ppf_fused_kernel", False),
          (1024, 8, "ppf_fused_kernel", False), (2048, 4, "ppf_fused_kernel", False),
          (2048, 8, "ppf_long_kernel", True), (4096, 8, "ppf_long_kernel", True), (512, 24, "ppf_long_kernel", True)]


@pytest.mark.parametrize("in_type", [0, 1, 2])
@pytest.mark.parametrize("n,taps,kernel,keeps", SHAPES)
def test_route(n, taps, kernel, keeps, in_type):
    m = (1 << 25) // n
    batch, at, above = launches.run(f"exec {n} {taps} {in_type} 0 {m}", f"push {n} {taps} {in_type} 0 {m}",
                                    f"push {n} {taps} {in_type} 0 {m + 1}")
    assert [launches.kernel(w) for w in batch] == [launches.kernel(w) for w in at] == [kernel]
    assert [launches.kernel(w) for w in above] == [kernel] + ([] if keeps else ["ppf_history_kernel"])
    if kernel == "ppf_fused_kernel":
        hist = [w[0].rstrip(">").split(",")[-1] for w in (batch, at, above)]
        assert hist == (["true"] * 3 if keeps else ["false", "true", "false"])


@pytest.mark.gpu
@pytest.mark.parametrize("n,taps", [(2048, 4), (256, 16)])
def test_long_push(n, taps):
    """Pushes on both sides of the limit: the batch's bits, the history's blocks."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m = (1 << 25) // n
    h = np.random.default_rng(n + taps).standard_normal(taps * n).astype(np.float32)
    gen = torch.Generator("cuda").manual_seed(n)
    x = torch.view_as_complex(torch.randn((2 * m + 4) * n, 2, generator=gen, device="cuda"))
    print(f"case long push N={n} T={taps} M={m}", flush=True)
    plan = ppf.Plan(n, taps, h)
    padded = torch.cat([torch.zeros_like(x[:(taps - 1) * n]), x])
    whole = plan.execute(padded, nspectra=2 * m + 4)
    ppf.ppf_set_stream(plan.handle, torch.cuda.current_stream().cuda_stream)
    stream = ppf.ppf_stream_create(plan.handle)
    hist = np.empty((taps - 1) * n, np.complex64)
    at = 0
    for s in (m, m + 1, 1, 2):                    # one launch, two, one, one
        part = torch.empty((s, n), dtype=torch.complex64, device="cuda")
        ppf.ppf_stream_push(stream, x[at * n:(at + s) * n].clone(), part, s)
        assert torch.equal(part, whole[at:at + s]), (at, s)
        at += s
        ppf.ppf_stream_get_history(stream, hist)
        assert np.array_equal(hist, padded[at * n:(at + taps - 1) * n].cpu().numpy()), s
    ppf.ppf_stream_destroy(stream)
    plan.close()
