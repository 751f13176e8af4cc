"""Batches of several rounds of tiles at N = 512 and 1024 with up to 8 taps: the
last round nearly empty, a little under and over five eighths full, and full,
for each stored type, and as detection. Every row is compared with the same
rows of short batches (one tile's spectra each), whose arithmetic is the same.
"""
import numpy as np
import pytest

import oracle
from paper_1411_3656_amd import ppf, signals

pytestmark = pytest.mark.gpu
TOL = 1e-5          # max |error| over output RMS: the FP32 bar of every path


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("n,taps,in_type,m_total,k_int", [
    (1024, 8, ppf.PPF_C32, 131073, 0), (1024, 8, ppf.PPF_CI8, 163841, 0), (1024, 3, ppf.PPF_C16, 214000, 0),
    (1024, 8, ppf.PPF_CI8, 262144, 0), (512, 8, ppf.PPF_C16, 530001, 0), (1024, 5, ppf.PPF_C32, 131088, 16),
])
def test_rounds(n, taps, in_type, m_total, k_int):
    torch = _torch()
    print(f"case tile rounds N={n} T={taps} in_type={in_type} M={m_total} K={k_int}", flush=True)
    h = np.random.default_rng(taps).standard_normal(n * taps).astype(np.float32)
    gen = torch.Generator("cuda").manual_seed(m_total)
    samples = (m_total + taps - 1) * n
    x = torch.randn(samples, 2, generator=gen, device="cuda")
    x = (torch.view_as_complex(x) if in_type == ppf.PPF_C32 else x.half() if in_type == ppf.PPF_C16
         else (x * 16).round().clamp(-127, 127).to(torch.int8))
    plan = ppf.Plan(n, taps, h, in_type=in_type)
    step = 4096
    if k_int:
        out = plan.execute_power(x, k_int, nspectra=m_total)
    else:
        out = torch.full((m_total + 1, n), 7.0, dtype=torch.complex64, device="cuda")
        plan.execute(x, out=out, nspectra=m_total)
        torch.cuda.synchronize()
        assert bool((out[m_total] == 7.0).all())     # nothing beyond the batch is written
    part = torch.empty((step, n), dtype=torch.complex64, device="cuda")
    worst = 0.0
    for m0 in range(0, m_total, step):
        k = min(step, m_total - m0)
        xs = x[m0 * n:(m0 + k + taps - 1) * n].clone()
        plan.execute(xs, out=part, nspectra=k)
        if k_int:
            ref = part[:k].abs().double().square().reshape(k // k_int, k_int, n).sum(1)
            got = out[m0 // k_int:(m0 + k) // k_int].double()
            # the FP32 sums and squares: at most (K + 4) * 2^-24 of a group's power
            worst = max(worst, float(((got - ref).abs() / ref).max()))
            assert worst <= (k_int + 4) * 2.0 ** -24, m0
        else:
            assert torch.equal(out[m0:m0 + k], part[:k]), m0
        if m0 == 0:      # the short batches themselves, against the oracle
            xr = xs[:(40 + taps - 1) * n].cpu().numpy()
            ref = oracle.ppf(xr, h, n, taps, spectra=list(range(40)))
            rms = float(np.sqrt(np.mean(np.abs(ref) ** 2)))
            assert np.max(np.abs(part[:40].cpu().numpy() - ref)) <= TOL * rms
    torch.cuda.synchronize()
    plan.close()
