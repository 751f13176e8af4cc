"""N = 4096 with 9 to 16 taps and N = 8192 with 2 to 8 in batches of eight and
four spectra per workgroup: batch lengths around those that take these
kernels (two thirds of a round of eight spectra per CU, two fifths of a round
of four, a full round, two), ragged last batches, every stored type, and a
history in front of the batch; two passes take the others.
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


@pytest.mark.parametrize("n,taps,in_type,m_total", [
    (4096, 16, ppf.PPF_C32, 1365), (4096, 16, ppf.PPF_C32, 1366), (4096, 16, ppf.PPF_C32, 1401),
    (4096, 13, ppf.PPF_C32, 2048), (4096, 16, ppf.PPF_C32, 2049), (4096, 9, ppf.PPF_C32, 2735),
    (4096, 16, ppf.PPF_CI8, 1999), (4096, 10, ppf.PPF_C16, 2041),
    (8192, 8, ppf.PPF_C32, 409), (8192, 8, ppf.PPF_C32, 410), (8192, 5, ppf.PPF_C32, 1024),
    (8192, 4, ppf.PPF_C32, 1025), (8192, 3, ppf.PPF_C16, 611), (8192, 2, ppf.PPF_C32, 415),
    (8192, 7, ppf.PPF_CI8, 1001),
])
def test_batched_batches_and_pushes(n, taps, in_type, m_total):
    torch = _torch()
    h = np.random.default_rng(taps).standard_normal(n * taps).astype(np.float32)
    x = signals.complex_gaussian((m_total + taps - 1) * n, 1.0, seed=taps + m_total)
    if in_type == ppf.PPF_C16:
        x = signals.to_complex_fp16(x)
    elif in_type == ppf.PPF_CI8:
        x = signals.quantize_int8(x * 16)
    print(f"case batched N={n} T={taps} in_type={in_type} M={m_total}", flush=True)
    idx = sorted(set(range(0, m_total, 61)) | set(range(min(26, m_total))) | set(range(m_total - 26, m_total)))
    ref = oracle.ppf(x, h, n, taps, spectra=idx)
    rms = float(np.sqrt(np.mean(np.abs(ref) ** 2)))
    plan = ppf.Plan(n, taps, h, in_type=in_type)
    xd = torch.from_numpy(x).cuda()
    out = torch.full((m_total + 1, n), 7.0, dtype=torch.complex64, device="cuda")
    plan.execute(xd, out=out, nspectra=m_total)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.max(np.abs(got[idx] - ref)) <= TOL * rms
    assert np.isfinite(got).all()
    assert (got[m_total] == 7.0).all()          # nothing beyond the batch is written
    stream = ppf.ppf_stream_create(plan.handle)
    ppf.ppf_stream_set_history(stream, x[:(taps - 1) * n])
    pushed = torch.zeros((m_total, n), dtype=torch.complex64, device="cuda")
    ppf.ppf_stream_push(stream, xd[(taps - 1) * n:].clone(), pushed, m_total)
    torch.cuda.synchronize()
    ppf.ppf_stream_destroy(stream)
    plan.close()
    assert np.max(np.abs(pushed.cpu().numpy()[idx] - ref)) <= TOL * rms
