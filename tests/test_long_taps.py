"""The fused kernels whose FIR and FFT have layouts of their own: 17 to 32
taps at N = 64 to 1024, 5 to 16 at N = 2048, 5 to 8 at N = 4096. The batch
lengths sit at their edges: one spectrum, a step (1 to 8 spectra) less or
more one, several workgroups with a ragged last tile, and either side of the
lengths below which another kernel takes the batch (3 and 64 at N = 2048).
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


def _stored(x, in_type):
    if in_type == ppf.PPF_C16:
        return signals.to_complex_fp16(x)
    if in_type == ppf.PPF_CI8:
        return signals.quantize_int8(x * 16)
    return x


@pytest.mark.parametrize("n,taps,in_type,sizes", [
    (64, 32, ppf.PPF_C32, [1, 5, 17, 1003]),
    (64, 17, ppf.PPF_CI8, [3, 130]),
    (128, 31, ppf.PPF_C32, [1, 7, 33, 500]),
    (256, 32, ppf.PPF_C32, [1, 9, 257]),
    (256, 20, ppf.PPF_C16, [2, 49]),
    (512, 32, ppf.PPF_C32, [1, 8, 17, 203]),
    (512, 25, ppf.PPF_CI8, [41]),
    (1024, 32, ppf.PPF_C32, [1, 3, 5, 150]),
    (1024, 18, ppf.PPF_C16, [35]),
    (2048, 16, ppf.PPF_C32, [1, 63, 64, 65, 530]),
    (2048, 9, ppf.PPF_CI8, [64, 131]),
    (2048, 12, ppf.PPF_C16, [67]),
    (2048, 8, ppf.PPF_C32, [1, 2, 3, 5, 515]),
    (2048, 5, ppf.PPF_CI8, [3, 7]),
    (2048, 7, ppf.PPF_C16, [4, 33]),
    (4096, 8, ppf.PPF_C32, [1, 2, 10, 261]),
    (4096, 5, ppf.PPF_C16, [1, 19]),
    (4096, 6, ppf.PPF_CI8, [23]),
])
def test_long_tap_batches_and_streams(n, taps, in_type, sizes):
    torch = _torch()
    h = np.random.default_rng(n + 31 * taps).standard_normal(n * taps).astype(np.float32)
    plan = ppf.Plan(n, taps, h, in_type=in_type)
    ppf.ppf_set_stream(plan.handle, torch.cuda.current_stream().cuda_stream)
    for m_total in sizes:
        print(f"case long taps N={n} T={taps} in_type={in_type} M={m_total}", flush=True)
        x = _stored(signals.complex_gaussian((m_total + taps - 1) * n, 1.0, seed=n + taps + m_total), in_type)
        ref = oracle.ppf(x, h, n, taps)
        rms = float(np.sqrt(np.mean(np.abs(ref) ** 2)))
        xd = torch.from_numpy(x).cuda()
        out = torch.full((m_total + 1, n), 7.0, dtype=torch.complex64, device="cuda")
        plan.execute(xd, out=out, nspectra=m_total)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        assert np.max(np.abs(got[:m_total] - ref)) <= TOL * rms
        assert (got[m_total] == 7.0).all()          # nothing beyond the batch is written
        # the same samples as a stream: history ++ chunk, the history saved ones
        stream = ppf.ppf_stream_create(plan.handle)
        ppf.ppf_stream_set_history(stream, x[:(taps - 1) * n])
        pushed = torch.zeros((m_total, n), dtype=torch.complex64, device="cuda")
        ppf.ppf_stream_push(stream, xd[(taps - 1) * n:].clone(), pushed, m_total)
        torch.cuda.synchronize()
        ppf.ppf_stream_destroy(stream)
        assert np.max(np.abs(pushed.cpu().numpy() - ref)) <= TOL * rms
    plan.close()
