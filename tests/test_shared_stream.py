"""One plan, several host threads, one stream handle: calls that hand data from
one kernel to the next through a buffer of the stream (two-pass batches,
detection in parts) must not come between each other's launches.
"""
import threading

import numpy as np
import pytest

import oracle
from paper_1411_3656_amd import ppf, signals
from tests import launches

TOL = 1e-5          # max |error| over output RMS: the FP32 bar of every path
BAR = 1.2e-4        # detection: max |P - P_ref| over mean(P_ref)
PER_THREAD = 2      # hipStreamPerThread: one handle, a stream per thread

# every call of one thread, launch by launch
CALLS = [
    ("power 1024 8 0 0 64 64", ["ppf_fused_kernel", "ppf_power_parts_kernel"]),          # detection in parts
    ("power 4096 8 0 0 64 64", ["ppf_fused_kernel", "ppf_power_parts_kernel"]),
    ("power 4096 16 2 0 36 9", ["ppf_fir_kernel", "ppf_fused_kernel", "ppf_power_parts_kernel"]),
    ("exec 4096 32 0 0 64 1", ["ppf_fir_kernel", "ppf_fused_kernel"]),                   # two-pass batches
    ("exec 1024 40 1 0 64 1", ["ppf_fir_kernel", "ppf_fused_kernel"]),
    ("exec 16384 8 0 0 64 1", ["ppf_fs_kernel", "ppf_fs_kernel"]),
]


@pytest.mark.parametrize("command,call", CALLS)
def test_a_calls_launches_stay_together(command, call):
    words, = launches.run(f"threads {command} 0")
    assert len(words) == 2 * 4 * len(call)
    for i in range(0, len(words), len(call)):
        mine = [w.split(":", 1) for w in words[i:i + len(call)]]
        assert len({t for t, _ in mine}) == 1, words
        assert [launches.kernel(w) for _, w in mine] == call


@pytest.mark.parametrize("command,call", CALLS)
def test_per_thread_streams_take_turns(command, call):
    """The same on hipStreamPerThread, where launch order says nothing: the
    first call leaves an event, every later one waits for it and leaves its
    own. Fused detection needs no buffer there: whole groups, one kernel."""
    words, = launches.run(f"threads {command} {PER_THREAD}")
    if command.startswith("power") and call[0] != "ppf_fir_kernel":
        assert [launches.kernel(w.split(":", 1)[1]) for w in words] == call[:1] * 8
        return
    at = 0
    for i in range(8):
        want = (["wait"] if i else []) + call + ["record"]
        mine = [w.split(":", 1) for w in words[at:at + len(want)]]
        assert len({t for t, _ in mine}) == 1, words
        assert [launches.kernel(w) for _, w in mine] == want, words
        at += len(want)
    assert at == len(words)


@pytest.mark.gpu
@pytest.mark.parametrize("stream", [0, PER_THREAD])
@pytest.mark.parametrize("n,taps,m_total,k_int", [
    (1024, 8, 64, 64), (4096, 8, 64, 64), (4096, 16, 36, 9),      # detection, k_int spectra a group
    (4096, 32, 70, 0), (16384, 8, 40, 0), (1024, 40, 300, 0),     # batches
])
def test_threads_on_one_handle(n, taps, m_total, k_int, stream):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    h = np.random.default_rng(n + taps).standard_normal(taps * n).astype(np.float32)
    plan = ppf.Plan(n, taps, h)
    n_threads, reps = 3, 12
    xs = [signals.complex_gaussian((m_total + taps - 1) * n, 1.0 + i, seed=700 + i) for i in range(n_threads)]
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
    torch.cuda.synchronize()
    errors = []
    barrier = threading.Barrier(n_threads)
    print(f"case shared handle N={n} T={taps} M={m_total} K={k_int} stream={stream}", flush=True)

    def worker(i):
        try:
            ppf.ppf_set_stream(plan.handle, stream)
            barrier.wait()
            for r in range(reps):
                if k_int:
                    ppf.ppf_execute_power(plan.handle, xds[i], outs[i][r], m_total, k_int)
                else:
                    ppf.ppf_execute(plan.handle, xds[i], outs[i][r], m_total)
            # in this thread: no other call waits for a per-thread stream
            torch.cuda.ExternalStream(stream).synchronize()
        except Exception as e:  # noqa: BLE001 - reported below
            errors.append(e)

    threads = [threading.Thread(target=worker, args=(i,)) for i in range(n_threads)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for i in range(n_threads):
        for r in range(reps):
            assert np.max(np.abs(outs[i][r].cpu().numpy() - refs[i])) <= scale[i], (i, r)
    plan.close()
