"""A stream's two-pass workspace (128 MiB, 512 MiB from N = 8192 on) is allocated by
the first call that presums into it, not by one-kernel calls of the same plan,
and also if that first call is being captured.
"""
import numpy as np
import pytest

import oracle
from paper_1411_3656_amd import ppf, signals
from tests import launches

TOL = 1e-5          # max |error| over output RMS: the FP32 bar of every path


@pytest.mark.parametrize("n,taps,in_type,one,two,mib", [
    (64, 32, 0, 100, None, 128), (1024, 24, 0, 600, 300, 128), (1024, 24, 2, 300, 3, 128),
    (2048, 16, 1, 500, 20, 128), (4096, 16, 0, 2048, 100, 128), (8192, 8, 0, 1024, 100, 512),
])
def test_only_two_passes_allocate(n, taps, in_type, one, two, mib):
    (got,), = launches.run(f"query {n} {taps} {in_type} 0 {one} 0")
    assert int(got) == 0
    if two:
        (got,), = launches.run(f"query {n} {taps} {in_type} 0 {two} 0")
        assert int(got) == mib << 20


@pytest.mark.gpu
@pytest.mark.parametrize("n,taps,warm,m_total", [(4096, 16, 2048, 40), (8192, 8, 1024, 30), (1024, 40, 0, 50)])
def test_first_two_pass_call_under_capture(n, taps, warm, m_total):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    h = np.random.default_rng(n + taps).standard_normal(taps * n).astype(np.float32)
    x = signals.complex_gaussian((max(warm, m_total) + taps - 1) * n, 1.0, seed=n + taps)
    print(f"case capture N={n} T={taps} M={m_total} after M={warm}", flush=True)
    plan = ppf.Plan(n, taps, h)
    xd = torch.from_numpy(x).cuda()
    out = torch.zeros((m_total, n), dtype=torch.complex64, device="cuda")
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    if warm:                                               # one kernel: no workspace yet
        with torch.cuda.stream(st):
            plan.execute(xd, nspectra=warm)
        torch.cuda.synchronize()
        assert ppf.ppf_plan_query(plan.handle, ppf.PPF_Q_WORKSPACE_BYTES) == 0
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        plan.execute(xd, out=out, nspectra=m_total)
    ref = oracle.ppf(x[:(m_total + taps - 1) * n], h, n, taps)
    rms = np.sqrt(np.mean(np.abs(ref) ** 2))
    for _ in range(3):
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.max(np.abs(out.cpu().numpy() - ref)) <= TOL * rms
        with torch.cuda.stream(st):
            eager = plan.execute(xd, nspectra=m_total)
        torch.cuda.synchronize()
        assert torch.equal(eager, out)
    plan.close()
