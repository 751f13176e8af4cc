"""Two-pass calls larger than the memory-side cache (256 MiB): the four-step form
in equal chunks of at most that size, and the FIR pass with nontemporal loads.
Sizes one spectrum below and above the limits, the spectra on both sides of
each chunk's edge against the oracle, and every row against the same rows
computed in short calls, whose arithmetic is the same.
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


@pytest.mark.parametrize("n,taps,m_total", [
    (16384, 3, 2048), (16384, 8, 2049),                  # one chunk, two
    (16384, 16, 1016), (16384, 16, 1017),                # input and presums of 256 MiB, and more
    (16384, 9, 2041), (2048, 20, 16370),                 # nontemporal loads; in equal chunks
])
def test_calls_around_the_cache_size(n, taps, m_total):
    torch = _torch()
    h = np.random.default_rng(taps).standard_normal(n * taps).astype(np.float32)
    x = signals.complex_gaussian((m_total + taps - 1) * n, 1.0, seed=taps + m_total)
    print(f"case large call N={n} T={taps} M={m_total}", flush=True)
    edges = [0, m_total // 3, m_total // 2, 2 * m_total // 3, m_total]
    idx = sorted({i for e in edges for i in range(max(0, e - 3), min(m_total, e + 3))})
    ref = oracle.ppf(x, h, n, taps, spectra=idx)
    rms = float(np.sqrt(np.mean(np.abs(ref) ** 2)))
    plan = ppf.Plan(n, taps, h)
    xd = torch.from_numpy(x).cuda()
    out = torch.full((m_total + 1, n), 7.0, dtype=torch.complex64, device="cuda")
    plan.execute(xd, out=out, nspectra=m_total)
    torch.cuda.synchronize()
    assert np.max(np.abs(out[idx].cpu().numpy() - ref)) <= TOL * rms
    assert bool((out[m_total] == 7.0).all())     # nothing beyond the batch is written
    step = 63                                    # below the shortest batch of any one-pass form
    part = torch.empty((step, n), dtype=torch.complex64, device="cuda")
    for m0 in range(0, m_total, step):
        k = min(step, m_total - m0)
        plan.execute(xd[m0 * n:(m0 + k + taps - 1) * n].clone(), out=part, nspectra=k)
        assert torch.equal(out[m0:m0 + k], part[:k]), m0
    plan.close()
