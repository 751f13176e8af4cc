"""N = 4096 with 9 to 16 taps in batches of eight spectra per workgroup: batch
lengths around those that take this kernel (two thirds of a round of eight
spectra per CU, a full round, two), ragged last batches, every stored type,
and a history in front of the batch; two passes take the others.
"""
import numpy as np
import pytest

import oracle
from paper_1411_3656_amd import ppf, signals

pytestmark = pytest.mark.gpu
TOL = 1e-5          # max |error| over output RMS: the FP32 bar of every path
N = 4096


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("taps,in_type,m_total", [
    (16, ppf.PPF_C32, 1365), (16, ppf.PPF_C32, 1366), (16, ppf.PPF_C32, 1401), (13, ppf.PPF_C32, 2048),
    (16, ppf.PPF_C32, 2049), (9, ppf.PPF_C32, 2735), (16, ppf.PPF_CI8, 1999), (10, ppf.PPF_C16, 2041),
])
def test_batched_batches_and_pushes(taps, in_type, m_total):
    torch = _torch()
    h = np.random.default_rng(taps).standard_normal(N * taps).astype(np.float32)
    x = signals.complex_gaussian((m_total + taps - 1) * N, 1.0, seed=taps + m_total)
    if in_type == ppf.PPF_C16:
        x = signals.to_complex_fp16(x)
    elif in_type == ppf.PPF_CI8:
        x = signals.quantize_int8(x * 16)
    print(f"case batched N={N} T={taps} in_type={in_type} M={m_total}", flush=True)
    idx = sorted(set(range(0, m_total, 61)) | set(range(min(26, m_total))) | set(range(m_total - 26, m_total)))
    ref = oracle.ppf(x, h, N, taps, spectra=idx)
    rms = float(np.sqrt(np.mean(np.abs(ref) ** 2)))
    plan = ppf.Plan(N, taps, h, in_type=in_type)
    xd = torch.from_numpy(x).cuda()
    out = torch.full((m_total + 1, N), 7.0, dtype=torch.complex64, device="cuda")
    plan.execute(xd, out=out, nspectra=m_total)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.max(np.abs(got[idx] - ref)) <= TOL * rms
    assert np.isfinite(got).all()
    assert (got[m_total] == 7.0).all()          # nothing beyond the batch is written
    stream = ppf.ppf_stream_create(plan.handle)
    ppf.ppf_stream_set_history(stream, x[:(taps - 1) * N])
    pushed = torch.zeros((m_total, N), dtype=torch.complex64, device="cuda")
    ppf.ppf_stream_push(stream, xd[(taps - 1) * N:].clone(), pushed, m_total)
    torch.cuda.synchronize()
    ppf.ppf_stream_destroy(stream)
    plan.close()
    assert np.max(np.abs(pushed.cpu().numpy()[idx] - ref)) <= TOL * rms
