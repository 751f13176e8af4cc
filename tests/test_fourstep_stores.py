"""The four-step form stores Z past L2 where Z is about L2's size (7 MiB up to 28
at N = 8192, 22 at N = 16384) and through it elsewhere; the spectra are the same.
"""
import numpy as np
import pytest

import oracle
from paper_1411_3656_amd import ppf, signals
from tests import launches

TOL = 1e-5          # max |error| over output RMS: the FP32 bar of every path
# N, taps, batches with ordinary stores, with nontemporal ones (first and last of each run)
RUNS = [(8192, 2, (1, 111, 448), (112, 447)), (8192, 7, (111, 448), (112, 300, 447)),
        (16384, 4, (55, 176, 2049), (56, 175)), (16384, 8, (1, 55, 176), (56, 120, 175))]


@pytest.mark.parametrize("n,taps,plain,nt", RUNS)
def test_route(n, taps, plain, nt):
    # N = 8192 takes the form from 410 spectra on only when two passes are asked for
    path = 2 if n == 8192 else 0
    for m in plain + nt:
        words, = launches.run(f"exec {n} {taps} 0 {path} {m}")
        stores = {w.rstrip(">").split(",")[-1] for w in words[::2]}           # pass A's
        assert stores == {"true" if m in nt else "false"}, (m, words)


@pytest.mark.gpu
@pytest.mark.parametrize("n,taps", [(8192, 2), (8192, 7), (16384, 1), (16384, 4), (16384, 8)])
def test_same_spectra(n, taps):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m_total = (22 << 20) // (8 * n) + 3                    # nontemporal at N = 8192; ordinary at 16384
    h = np.random.default_rng(n + taps).standard_normal(taps * n).astype(np.float32)
    x = signals.complex_gaussian((m_total + taps - 1) * n, 1.0, seed=n + taps)
    print(f"case four-step stores N={n} T={taps} M={m_total}", flush=True)
    plan = ppf.Plan(n, taps, h)
    xd = torch.from_numpy(x).cuda()
    whole = plan.execute(xd)
    idx = [0, 1, m_total // 2, m_total - 1]
    ref = oracle.ppf(x, h, n, taps, spectra=idx)
    assert np.max(np.abs(whole[idx].cpu().numpy() - ref)) <= TOL * np.sqrt(np.mean(np.abs(ref) ** 2))
    at = 0
    for k in (2, 9, (8 << 20) // (8 * n)):                 # ordinary, ordinary, nontemporal
        part = plan.execute(xd[at * n:(at + k + taps - 1) * n].clone(), nspectra=k)
        assert torch.equal(part, whole[at:at + k]), (at, k)
        at += k
    plan.close()
