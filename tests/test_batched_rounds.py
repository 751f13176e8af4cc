"""N = 8192, 5 to 8 taps, FP16 and int8 input: the second and third rounds of the
one-pass kernel's batches (1024 spectra each on 256 CUs) pay from a quarter full
on; the spectra have the same bits in either form.
"""
import numpy as np
import pytest

import oracle
from paper_1411_3656_amd import ppf, signals
from tests import launches

TOL = 1e-5          # max |error| over output RMS: the FP32 bar of every path


@pytest.mark.parametrize("taps,in_type,two,one", [
    (8, ppf.PPF_CI8, (409, 1025, 1279, 2049, 2303), (410, 1024, 1280, 2048, 2304, 3072, 3073, 4100)),
    (5, ppf.PPF_C16, (409, 1025, 1279, 2049, 2303), (410, 1024, 1280, 2048, 2304, 3072, 3073, 4100)),
    (4, ppf.PPF_CI8, (409,), (410, 1025, 2049)),
    (8, ppf.PPF_C32, (409,), (410, 1025, 2049)),
])
def test_route(taps, in_type, two, one):
    for m in two + one:
        words, = launches.run(f"exec 8192 {taps} {in_type} 0 {m}")
        assert (launches.kernel(words[0]) == "ppf_large_kernel") == (m in one), (m, words)


@pytest.mark.gpu
@pytest.mark.parametrize("taps,in_type", [(8, ppf.PPF_CI8), (5, ppf.PPF_C16)])
def test_same_bits_around_a_round(taps, in_type):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, m_total = 8192, 1281
    h = np.random.default_rng(taps).standard_normal(taps * n).astype(np.float32)
    x = signals.complex_gaussian((m_total + taps - 1) * n, 1.0, seed=taps)
    x = signals.to_complex_fp16(x) if in_type == ppf.PPF_C16 else signals.quantize_int8(x * 16)
    print(f"case batched rounds N={n} T={taps} in_type={in_type} M={m_total}", flush=True)
    plan = ppf.Plan(n, taps, h, in_type=in_type)
    xd = torch.from_numpy(x).cuda()
    whole = plan.execute(xd, nspectra=m_total)                     # one pass, two rounds
    idx = [0, 1, 640, 1023, 1024, 1280]
    ref = oracle.ppf(x, h, n, taps, spectra=idx)
    assert np.max(np.abs(whole[idx].cpu().numpy() - ref)) <= TOL * np.sqrt(np.mean(np.abs(ref) ** 2))
    for k in (1279, 1024, 3):                                      # two passes, one pass, two passes
        assert torch.equal(plan.execute(xd[:(k + taps - 1) * n].clone(), nspectra=k), whole[:k]), k
    plan.close()
