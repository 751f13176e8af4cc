"""A push's history update, carried out by extra blocks of the batch's own
launch (or by the history kernel where the batch takes several launches):
after every push the history is exactly the last (T-1)*N samples of the
stream, for chunks shorter than, as long as and longer than it, every stored
type and the kernels of each kind; the spectra match the oracle's stream.
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


@pytest.mark.parametrize("n,taps,in_type", [
    (16, 2, ppf.PPF_CI8),       # one 32-byte block of history
    (64, 8, ppf.PPF_C32),
    (256, 16, ppf.PPF_C16),
    (1024, 8, ppf.PPF_C32),
    (1024, 3, ppf.PPF_CI8),
    (2048, 8, ppf.PPF_C32),     # two kernels: below and from 3 spectra
    (4096, 4, ppf.PPF_C32),
    (4096, 8, ppf.PPF_C16),
    (128, 32, ppf.PPF_C32),
    (1024, 17, ppf.PPF_CI8),
    (2048, 12, ppf.PPF_C32),    # two passes below 64 spectra, one launch from there on
    (512, 40, ppf.PPF_C32),     # two passes, the history kernel
    (512, 1, ppf.PPF_C32),      # no history
])
def test_history_after_every_push(n, taps, in_type):
    torch = _torch()
    h = np.random.default_rng(n + 77 * taps).standard_normal(n * taps).astype(np.float32)
    sizes = [s for s in (1, 2, taps - 2, taps - 1, taps, 2 * taps + 3, 70, 1) if s > 0]
    total = sum(sizes)
    x = signals.complex_gaussian(total * n, 1.0, seed=n + taps)
    if in_type == ppf.PPF_C16:
        x = signals.to_complex_fp16(x)
    elif in_type == ppf.PPF_CI8:
        x = signals.quantize_int8(x * 16)
    plan = ppf.Plan(n, taps, h, in_type=in_type)
    ppf.ppf_set_stream(plan.handle, torch.cuda.current_stream().cuda_stream)
    stream = ppf.ppf_stream_create(plan.handle)
    zeros = np.zeros(((taps - 1) * n,) + x.shape[1:], x.dtype)
    padded = np.concatenate([zeros, x])
    got, at = [], 0
    for s in sizes:
        print(f"case push history N={n} T={taps} in_type={in_type} S={s}", flush=True)
        xd = torch.from_numpy(np.ascontiguousarray(x[at * n:(at + s) * n])).cuda()
        out = torch.zeros((s, n), dtype=torch.complex64, device="cuda")
        ppf.ppf_stream_push(stream, xd, out, s)
        at += s
        if taps > 1:
            hist = np.empty_like(zeros)
            ppf.ppf_stream_get_history(stream, hist)
            assert np.array_equal(hist, padded[at * n:(at + taps - 1) * n]), s
        got.append(out.cpu().numpy())
    ppf.ppf_stream_destroy(stream)
    plan.close()
    ref = oracle.ppf(padded, h, n, taps)
    rms = float(np.sqrt(np.mean(np.abs(ref) ** 2)))
    assert np.max(np.abs(np.concatenate(got) - ref)) <= TOL * rms
