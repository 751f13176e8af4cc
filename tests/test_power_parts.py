"""Detection of few groups, each cut into parts that are summed side by side:
group lengths with many divisors, none, and beyond the longest cut, groups up
to and past the number that is cut, single calls of one group, the two-pass
form in chunks that leave room for the parts, and a call under capture (whole
groups there: a graph may be replayed beside the stream's own calls).

Bar as for every detection: max |P - P_ref| <= 1.2e-4 mean(P_ref), from the
FP32 bar of the spectra; the sums themselves add at most K * 2^-24 of a group's
power, 1e-4 of it at the largest K here and far less in parts.
"""
import numpy as np
import pytest

import oracle
from paper_1411_3656_amd import ppf, signals

pytestmark = pytest.mark.gpu
BAR = 1.2e-4


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _case(torch, n, taps, in_type, m_total, k_int):
    h = np.random.default_rng(taps + k_int).standard_normal(n * taps).astype(np.float32)
    x = signals.complex_gaussian((m_total + taps - 1) * n, 1.0, seed=taps + m_total)
    if in_type == ppf.PPF_C16:
        x = signals.to_complex_fp16(x)
    elif in_type == ppf.PPF_CI8:
        x = signals.quantize_int8(x * 16)
    print(f"case power parts N={n} T={taps} in_type={in_type} M={m_total} K={k_int}", flush=True)
    return x, h, ppf.Plan(n, taps, h, in_type=in_type)


@pytest.mark.parametrize("n,taps,in_type,m_total,k_int", [
    (64, 4, ppf.PPF_C32, 64, 64), (64, 8, ppf.PPF_C32, 1536, 1536), (16, 3, ppf.PPF_C32, 480, 240),
    (256, 8, ppf.PPF_C32, 23, 23), (1024, 8, ppf.PPF_C32, 4096, 4), (1024, 8, ppf.PPF_C32, 48, 6),
    (1024, 16, ppf.PPF_C32, 1600, 16), (2048, 8, ppf.PPF_C32, 15, 15), (2048, 12, ppf.PPF_C32, 128, 32),
    (4096, 8, ppf.PPF_C32, 514, 2), (4096, 5, ppf.PPF_C32, 64, 64), (4096, 16, ppf.PPF_CI8, 36, 9),
    (1024, 24, ppf.PPF_C16, 90, 30), (16384, 8, ppf.PPF_C32, 13, 13), (16384, 3, ppf.PPF_C32, 16, 2),
    (8192, 20, ppf.PPF_C32, 30, 10),
])
def test_power_in_parts(n, taps, in_type, m_total, k_int):
    torch = _torch()
    x, h, plan = _case(torch, n, taps, in_type, m_total, k_int)
    groups = m_total // k_int
    out = torch.full((groups + 1, n), 7.0, dtype=torch.float32, device="cuda")
    xd = torch.from_numpy(x).cuda()
    plan.execute_power(xd, k_int, out=out[:groups], nspectra=m_total)
    plan.execute_power(xd, k_int, out=out[:groups], nspectra=m_total)
    torch.cuda.synchronize()
    plan.close()
    got = out.cpu().numpy().astype(np.float64)
    ref = oracle.ppf_power(x, h, n, taps, k_int)
    assert np.max(np.abs(got[:groups] - ref)) <= BAR * np.mean(ref)
    assert (got[groups] == 7.0).all()            # nothing beyond the groups is written


def test_two_pass_chunks_leave_room():
    """N = 16384, 4096 spectra in groups of 64: a full workspace of presums. Every
    group equals the same group detected in a call of its own, to the rounding
    of its sum (64 terms in FP32: 64 * 2^-24 of it at most, both ways)."""
    torch = _torch()
    n, taps, m_total, k_int = 16384, 4, 4096, 64
    h = np.random.default_rng(1).standard_normal(n * taps).astype(np.float32)
    print(f"case power parts N={n} T={taps} M={m_total} K={k_int}", flush=True)
    gen = torch.Generator("cuda").manual_seed(5)
    x = torch.view_as_complex(torch.randn((m_total + taps - 1) * n, 2, generator=gen, device="cuda"))
    plan = ppf.Plan(n, taps, h)
    out = plan.execute_power(x, k_int, nspectra=m_total)
    for g in (0, 1, 30, 61, 62, 63):
        part = x[g * k_int * n:((g + 1) * k_int + taps - 1) * n].clone()
        one = plan.execute_power(part, k_int, nspectra=k_int)[0]
        assert bool(((out[g] - one).abs() <= 2 * 64 * 2.0 ** -24 * one).all()), g
    torch.cuda.synchronize()
    plan.close()


def test_power_under_capture():
    torch = _torch()
    n, taps, m_total, k_int = 1024, 8, 64, 32
    x, h, plan = _case(torch, n, taps, ppf.PPF_C32, m_total, k_int)
    ref = oracle.ppf_power(x, h, n, taps, k_int)
    xd = torch.from_numpy(x).cuda()
    eager = torch.zeros((2, n), dtype=torch.float32, device="cuda")
    out = torch.zeros((2, n), dtype=torch.float32, device="cuda")
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        plan.execute_power(xd, k_int, out=out, nspectra=m_total)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        with torch.cuda.stream(st):
            plan.execute_power(xd, k_int, out=eager, nspectra=m_total)
        torch.cuda.synchronize()
        for got in (out, eager):
            assert np.max(np.abs(got.cpu().numpy() - ref)) <= BAR * np.mean(ref)
    plan.close()
