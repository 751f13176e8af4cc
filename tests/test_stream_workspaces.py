"""One plan on several HIP streams at once, each host thread with its own: calls
that run in two passes, and two-pass detection whose partial sums lie behind
the presums, have a workspace per stream, so no call sees another's.
"""
import threading

import numpy as np
import pytest

import oracle
from paper_1411_3656_amd import ppf, signals
from tests import launches

TOL = 1e-5          # max |error| over output RMS: the FP32 bar of every path
BAR = 1.2e-4        # detection: max |P - P_ref| over mean(P_ref)
# N, taps, input type, spectra, K (0: a batch), MiB per stream
CASES = [
    (4096, 32, ppf.PPF_C32, 300, 0, 128), (16384, 8, ppf.PPF_C32, 120, 0, 512), (1024, 40, ppf.PPF_C32, 300, 0, 128),
    (1024, 40, ppf.PPF_CI8, 300, 0, 128), (8192, 16, ppf.PPF_C16, 60, 0, 512), (1024, 24, ppf.PPF_C32, 300, 0, 128),
    (4096, 16, ppf.PPF_C32, 64, 64, 128), (1024, 24, ppf.PPF_CI8, 90, 30, 128),
]


@pytest.mark.parametrize("n,taps,in_type,m_total,k_int,mib", CASES)
def test_the_cases_take_two_passes(n, taps, in_type, m_total, k_int, mib):
    op = f"power {n} {taps} {in_type} 0 {m_total} {k_int}" if k_int else f"exec {n} {taps} {in_type} 0 {m_total}"
    words, = launches.run(op)
    assert len(words) == (3 if k_int else 2)


@pytest.mark.gpu
@pytest.mark.parametrize("n,taps,in_type,m_total,k_int,mib", CASES)
def test_threads_on_streams_of_their_own(n, taps, in_type, m_total, k_int, mib):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    h = np.random.default_rng(n + taps).standard_normal(taps * n).astype(np.float32)
    plan = ppf.Plan(n, taps, h, in_type=in_type)
    n_threads, reps = 3, 10
    xs = [signals.complex_gaussian((m_total + taps - 1) * n, 1.0 + i, seed=900 + i) for i in range(n_threads)]
    if in_type == ppf.PPF_C16:
        xs = [signals.to_complex_fp16(x) for x in xs]
    elif in_type == ppf.PPF_CI8:
        xs = [signals.quantize_int8(x * 16) for x in xs]
    if k_int:
        refs = [oracle.ppf_power(x, h, n, taps, k_int) for x in xs]
        scale = [BAR * np.mean(r) for r in refs]
        shape, dtype = (m_total // k_int, n), torch.float32
    else:
        refs = [oracle.ppf(x, h, n, taps) for x in xs]
        scale = [TOL * float(np.sqrt(np.mean(np.abs(r) ** 2))) for r in refs]
        shape, dtype = (m_total, n), torch.complex64
    xds = [torch.from_numpy(x).cuda() for x in xs]
    outs = [[torch.zeros(shape, dtype=dtype, device="cuda") for _ in range(reps)] for _ in range(n_threads)]
    streams = [torch.cuda.Stream() for _ in range(n_threads)]
    torch.cuda.synchronize()
    errors = []
    barrier = threading.Barrier(n_threads)
    print(f"case own workspaces N={n} T={taps} in_type={in_type} M={m_total} K={k_int}", flush=True)

    def worker(i):
        try:
            ppf.ppf_set_stream(plan.handle, streams[i].cuda_stream)
            barrier.wait()
            for r in range(reps):
                if k_int:
                    ppf.ppf_execute_power(plan.handle, xds[i], outs[i][r], m_total, k_int)
                else:
                    ppf.ppf_execute(plan.handle, xds[i], outs[i][r], m_total)
            streams[i].synchronize()
        except Exception as e:  # noqa: BLE001 - reported below
            errors.append(e)

    threads = [threading.Thread(target=worker, args=(i,)) for i in range(n_threads)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for i in range(n_threads):
        for r in range(reps):
            assert np.max(np.abs(outs[i][r].cpu().numpy() - refs[i])) <= scale[i], (i, r)
    assert ppf.ppf_plan_query(plan.handle, ppf.PPF_Q_WORKSPACE_BYTES) == n_threads * mib << 20
    plan.close()
