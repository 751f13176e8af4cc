"""ppf_plan_set_path(PPF_PATH_TWO_PASS) means two passes at every batch length,
also where the library's own choice for the shape is one kernel.
"""
import numpy as np
import pytest

import oracle
from paper_1411_3656_amd import ppf, signals
from tests import launches

TOL = 1e-5          # max |error| over output RMS: the FP32 bar of every path
ONE = {"ppf_long_kernel", "ppf_batched_kernel", "ppf_large_kernel"}
SHAPES = [(64, 17, 1000), (256, 32, 300), (1024, 24, 700), (2048, 12, 500), (4096, 16, 2048), (8192, 8, 1024)]


@pytest.mark.parametrize("in_type", [0, 1, 2])
@pytest.mark.parametrize("n,taps,m_total", SHAPES)
def test_forced_two_passes(n, taps, m_total, in_type):
    ops = ("exec", "push")
    auto = launches.run(*(f"{op} {n} {taps} {in_type} 0 {m_total}" for op in ops))
    forced = launches.run(*(f"{op} {n} {taps} {in_type} 2 {m_total}" for op in ops))
    fs = n == 8192 and in_type == 0                       # the four-step form's two passes
    for a, f in zip(auto, forced):
        assert launches.kernel(a[0]) in ONE
        names = [launches.kernel(w) for w in f if launches.kernel(w) != "ppf_history_kernel"]
        assert names and names == ["ppf_fs_kernel" if fs else k
                                   for _ in range(len(names) // 2) for k in ("ppf_fir_kernel", "ppf_fused_kernel")]


@pytest.mark.gpu
@pytest.mark.parametrize("n,taps,m_total", SHAPES)
def test_forced_two_passes_on_the_gpu(n, taps, m_total):
    """Right, and the same bits in one call and in several of other lengths."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    h = np.random.default_rng(n + taps).standard_normal(taps * n).astype(np.float32)
    x = signals.complex_gaussian((m_total + taps - 1) * n, 1.0, seed=n + taps)
    print(f"case forced two passes N={n} T={taps} M={m_total}", flush=True)
    plan = ppf.Plan(n, taps, h, ppf.PPF_PATH_TWO_PASS)
    xd = torch.from_numpy(x).cuda()
    got = plan.execute(xd)
    idx = sorted({0, 1, 77, m_total // 2, m_total - 1})
    ref = oracle.ppf(x, h, n, taps, spectra=idx)
    assert np.max(np.abs(got[idx].cpu().numpy() - ref)) <= TOL * np.sqrt(np.mean(np.abs(ref) ** 2))
    at = 0
    for k in (1, 5, 70, m_total - 76):
        part = plan.execute(xd[at * n:(at + k + taps - 1) * n].clone(), nspectra=k)
        assert torch.equal(part, got[at:at + k]), (at, k)
        at += k
    plan.close()
