"""Short batches of the shapes whose long ones take one launch (17 to 32 taps at
N = 512 and 1024, 9 to 16 at N = 2048): two passes below the length from which
one launch is as fast, with the same bits on both sides of it.
"""
import numpy as np
import pytest

import oracle
from paper_1411_3656_amd import ppf, signals
from tests import launches

TOL = 1e-5          # max |error| over output RMS: the FP32 bar of every path
# N, taps, input type, last length in two passes
EDGES = [
    (512, 17, ppf.PPF_C32, 511), (512, 32, ppf.PPF_C32, 511), (1024, 17, ppf.PPF_C32, 575),
    (1024, 32, ppf.PPF_C32, 575), (1024, 20, ppf.PPF_CI8, 15), (1024, 31, ppf.PPF_C16, 15),
    (2048, 9, ppf.PPF_C32, 399), (2048, 16, ppf.PPF_C16, 127), (2048, 12, ppf.PPF_CI8, 127),
]


@pytest.mark.parametrize("n,taps,in_type,last", EDGES)
def test_route(n, taps, in_type, last):
    below, one, above = launches.run(*(f"exec {n} {taps} {in_type} 0 {m}" for m in (last, 1, last + 1)))
    fft = "ppf_fused_kernel" if n == 2048 else "ppf_long_kernel"
    for words in (below, one):
        assert [launches.kernel(w) for w in words] == ["ppf_fir_kernel", fft]
    assert [launches.kernel(w) for w in above] == ["ppf_long_kernel"]


@pytest.mark.parametrize("n,taps,in_type", [(512, 24, 1), (512, 17, 2), (256, 32, 0), (64, 17, 2), (128, 20, 1)])
def test_one_launch_from_one_spectrum_on(n, taps, in_type):
    words, = launches.run(f"exec {n} {taps} {in_type} 0 1")
    assert [launches.kernel(w) for w in words] == ["ppf_long_kernel"]


@pytest.mark.gpu
@pytest.mark.parametrize("n,taps,in_type,last", EDGES)
def test_same_bits_on_both_sides(n, taps, in_type, last):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m_total = last + 2
    h = np.random.default_rng(n + taps).standard_normal(taps * n).astype(np.float32)
    x = signals.complex_gaussian((m_total + taps - 1) * n, 1.0, seed=n + taps)
    if in_type == ppf.PPF_C16:
        x = signals.to_complex_fp16(x)
    elif in_type == ppf.PPF_CI8:
        x = signals.quantize_int8(x * 16)
    print(f"case short long taps N={n} T={taps} in_type={in_type} M={m_total}", flush=True)
    plan = ppf.Plan(n, taps, h, in_type=in_type)
    xd = torch.from_numpy(x).cuda()
    whole = plan.execute(xd, nspectra=m_total)                     # one launch
    ref = oracle.ppf(x, h, n, taps)
    assert np.max(np.abs(whole.cpu().numpy() - ref)) <= TOL * np.sqrt(np.mean(np.abs(ref) ** 2))
    at = 0
    for k in (1, 2, 5, last - 8):                                  # two passes each
        part = torch.full((k + 1, n), 7.0, dtype=torch.complex64, device="cuda")
        plan.execute(xd[at * n:(at + k + taps - 1) * n].clone(), out=part, nspectra=k)
        assert torch.equal(part[:k], whole[at:at + k]), (at, k)
        assert bool((part[k] == 7.0).all())                        # nothing beyond the batch is written
        at += k
    plan.close()
