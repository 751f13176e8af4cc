"""The main loop of the fused kernels with FIR and FFT layouts of their own, for
every size and stored type: batches in which each workgroup takes more than two
revolutions of its ring of blocks. Spectra spread over the batch against the
oracle, and every row against the same rows in short calls, whose workgroups
take one step (or which take two passes) with the same arithmetic.
"""
import numpy as np
import pytest

import oracle
from paper_1411_3656_amd import ppf, signals

pytestmark = pytest.mark.gpu
TOL = 1e-5          # max |error| over output RMS: the FP32 bar of every path
# N, taps, ring blocks, most tiles at once (256 CUs, workgroups per CU, tiles in each)
SHAPES = [(64, 30, 36, 256 * 3 * 4), (128, 32, 40, 256 * 3 * 2), (256, 17, 40, 256 * 3), (512, 32, 40, 256),
          (1024, 32, 36, 256), (2048, 16, 18, 256), (2048, 7, 10, 256), (4096, 8, 9, 256)]


@pytest.mark.parametrize("in_type", [ppf.PPF_C32, ppf.PPF_C16, ppf.PPF_CI8])
@pytest.mark.parametrize("n,taps,ring,tiles", SHAPES)
def test_many_steps(n, taps, ring, tiles, in_type):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m_total = tiles * (2 * ring + 5) + 3
    h = np.random.default_rng(n + taps).standard_normal(taps * n).astype(np.float32)
    gen = torch.Generator("cuda").manual_seed(n + taps)
    x = torch.randn((m_total + taps - 1) * n, 2, generator=gen, device="cuda")
    if in_type == ppf.PPF_C16:
        x = x.half()
    elif in_type == ppf.PPF_CI8:
        x = (x * 16).round().clamp(-127, 127).to(torch.int8)
    else:
        x = torch.view_as_complex(x)
    print(f"case long steps N={n} T={taps} in_type={in_type} M={m_total}", flush=True)
    plan = ppf.Plan(n, taps, h, in_type=in_type)
    out = torch.full((m_total + 1, n), 7.0, dtype=torch.complex64, device="cuda")
    plan.execute(x, out=out, nspectra=m_total)
    torch.cuda.synchronize()
    idx = sorted(set(range(0, m_total, m_total // (150 if n < 2048 else 40))) | set(range(2 * ring + 9)) | set(range(m_total - 9, m_total)))
    blocks = x.reshape(m_total + taps - 1, n, -1)
    rms = 0.0
    errs = []
    for lo in range(0, len(idx), 50):                  # the oracle on the blocks that it needs only
        for m in idx[lo:lo + 50]:
            ref = oracle.ppf(blocks[m:m + taps].reshape(x[:taps * n].shape).cpu().numpy(), h, n, taps)[0]
            rms += float(np.mean(np.abs(ref) ** 2))
            errs.append(float(np.max(np.abs(out[m].cpu().numpy() - ref))))
    assert max(errs) <= TOL * np.sqrt(rms / len(idx))
    assert bool((out[m_total] == 7.0).all())           # nothing beyond the batch is written
    step = 63 if n >= 512 else 500
    part = torch.empty((step, n), dtype=torch.complex64, device="cuda")
    for m0 in range(0, m_total, step):
        k = min(step, m_total - m0)
        plan.execute(x[m0 * n:(m0 + k + taps - 1) * n].clone(), out=part, nspectra=k)
        assert torch.equal(out[m0:m0 + k], part[:k]), m0
    plan.close()
