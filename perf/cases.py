"""Performance cases of the polyphase filter bank: what a program calls, at the sizes it calls it with.

Each case is a dict of plain values. ``prepare`` makes a program's inputs, plan
and buffers on the GPU, ``run`` is one call (or one round of calls) through the
public entry points, ``work`` the bytes and operations that no implementation
can avoid, and ``exact`` the same outputs in 64 bits from plain torch.

Keys: ``op`` (batch, power, stream, serve), ``n`` channels, ``taps``,
``nspectra`` per call, ``dtype`` (c32, c16, ci8: complex float32, float16 and
int8 samples), ``fft`` (f32, or mfma for the matrix-core transform), ``k``
(spectra summed per power spectrum), ``window`` of the prototype filter.
"""

import math

import numpy as np
import torch

from paper_1411_3656_amd import ppf

_IN_TYPE = {"c32": ppf.PPF_C32, "c16": ppf.PPF_C16, "ci8": ppf.PPF_CI8}


def _case(name, op, n, taps, nspectra, dtype="c32", fft="f32", k=1, window="hamming"):
    return {"name": name, "op": op, "n": n, "taps": taps, "nspectra": nspectra, "dtype": dtype, "fft": fft, "k": k,
            "window": window}


def listed():
    m = lambda log2_samples, n, taps: (1 << log2_samples) // n - taps + 1  # noqa: E731 - spectra of so many samples
    return [
        # one chunk of one live stream: the smallest call, all launch latency
        _case("stream_n1024_t8_s16", "stream", 1024, 8, 16),
        # one arrival round of the 64-stream serving mix, until the last chunk is done
        _case("serve_64streams", "serve", 0, 0, 64),
        # a short batch (67 MB in and out): fits the last-level cache
        _case("batch_n256_t8_m16384", "batch", 256, 8, 16384),
        # the single-SKA-LFAA-channel batch, 1 GiB of input: the benchmark's default
        _case("batch_n1024_t8_2p27", "batch", 1024, 8, m(27, 1024, 8)),
        # the same shape detected: power summed over 16 spectra instead of spectra out
        _case("power_n1024_t8_2p27", "power", 1024, 8, (m(27, 1024, 8)) // 16 * 16, k=16),
        # the same shape from half-precision samples, transform in float32
        _case("batch_n1024_t8_2p27_c16", "batch", 1024, 8, m(27, 1024, 8), dtype="c16"),
        # shape sweep: few channels with the longest filter
        _case("batch_n64_t32_2p28", "batch", 64, 32, m(28, 64, 32), window="hann"),
        # a medium batch with a tap count that is no power of two and a ragged spectrum count
        _case("batch_n2048_t12_m20011", "batch", 2048, 12, 20011),
        # shape sweep: many channels, short and long filter
        _case("batch_n4096_t8_2p28", "batch", 4096, 8, m(28, 4096, 8), window="hann"),
        _case("batch_n4096_t16_2p28", "batch", 4096, 16, m(28, 4096, 16), window="hann"),
        # shape sweep: most channels
        _case("batch_n16384_t8_2p28", "batch", 16384, 8, m(28, 16384, 8), window="hann"),
        # precision form: int8 samples, float16 coefficients, matrix-core transform
        _case("mfma_n4096_t16_2p28_ci8", "batch", 4096, 16, m(28, 4096, 16), dtype="ci8", fft="mfma"),
    ]


def draw(rng):
    """One more case: any op but serving, N = 64..16384, 1..32 taps, 2^14..2^27 samples (log-uniform)."""
    op = rng.choice(["batch", "batch", "batch", "batch", "power", "stream"])
    fft = "mfma" if op == "batch" and rng.random() < 0.2 else "f32"
    if fft == "mfma":
        n, taps, dtype = rng.choice([256, 1024, 4096]), rng.randint(1, 16), rng.choice(["ci8", "c16"])
    else:
        n, taps, dtype = 1 << rng.randint(6, 14), rng.randint(1, 32), rng.choice(["c32", "c32", "c32", "c16", "ci8"])
    nspectra = max(1, int(2.0 ** rng.uniform(14, 27) / n))
    k = 1
    if op == "power":
        k = rng.choice([1, 4, 16, 64])
        nspectra = max(1, nspectra // k) * k
    if op == "stream":
        nspectra = rng.randint(1, 64)
    case = _case("", op, n, taps, nspectra, dtype, fft, k, rng.choice(["hamming", "hann"]))
    del case["name"]
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _coeffs(n, taps, window):
    """Windowed sinc of one channel's width over taps*n points, unit sum (float64)."""
    length = n * taps
    j = np.arange(length, dtype=np.float64)
    a = 0.54 if window == "hamming" else 0.5
    w = a - (1.0 - a) * np.cos(2.0 * np.pi * j / (length - 1))
    h = w * np.sinc((j - (length - 1) / 2.0) / n)
    return h / h.sum()


def _stored_coeffs(case):
    """Coefficients as the plan takes them: (array, shift). float16 ones hold h * 2^shift."""
    h = _coeffs(case["n"], case["taps"], case["window"])
    if case["dtype"] == "c32":
        return h.astype(np.float32), 0
    shift = int(max(0, min(24, np.floor(14 - np.log2(np.abs(h).max())))))
    return (h * 2.0 ** shift).astype(np.float16), shift


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _samples(count, dtype, gen):
    """Complex Gaussian voltages in their stored form: complex64, or (count, 2) float16 or int8 pairs."""
    x = torch.randn((count, 2), generator=gen, device="cuda", dtype=torch.float32)
    if dtype == "c16":
        return x.half()
    if dtype == "ci8":
        return x.mul_(16.0).round_().clamp_(-127, 127).to(torch.int8)
    return torch.view_as_complex(x)


# the serving mix: channels and taps per stream, chunks of 16 to 64 spectra
_SERVE_N, _SERVE_T = (256, 1024, 4096), (8, 16)


def _serve_streams(case):
    """(n, taps, spectra of the chunk) of every stream; fixed, so that every seed serves the same load."""
    r = np.random.Generator(np.random.PCG64(14113656))
    return [(int(r.choice(_SERVE_N)), int(r.choice(_SERVE_T)), int(r.integers(16, 65)))
            for _ in range(case["nspectra"])]


def _serve_inputs(case, seed):
    gen = _generator(seed)
    return [_samples(n * s, "c32", gen) for n, _, s in _serve_streams(case)]


def _stream_chunks(case):
    """Pushes of one pass: at least taps-1 spectra in all, so that a pass leaves the history it began with."""
    return max(1, math.ceil((case["taps"] - 1) / case["nspectra"]))


# ---------------------------------------------------------------------------
# the calls
# ---------------------------------------------------------------------------

def _plan(case):
    h, shift = _stored_coeffs(case)
    return ppf.Plan(case["n"], case["taps"], h, in_type=_IN_TYPE[case["dtype"]], coeff_shift=shift,
                    fft_mode=ppf.PPF_FFT_MFMA_F16 if case["fft"] == "mfma" else ppf.PPF_FFT_F32)


class _Stream:
    """A live stream: its plan, handle and chunk buffers."""

    def __init__(self, case, seed):
        n, s, c = case["n"], case["nspectra"], _stream_chunks(case)
        self.s = s
        self.plan = _plan(case)
        self.x = list(_samples(n * s * c, case["dtype"], _generator(seed)).chunk(c))
        # chunks start on 16-byte boundaries whatever their length
        self.x = [t.clone() for t in self.x]
        self.out = torch.empty((c, s, n), dtype=torch.complex64, device="cuda")
        self.handle = ppf.ppf_stream_create(self.plan.handle)
        ppf.ppf_set_stream(self.plan.handle, torch.cuda.current_stream().cuda_stream)
        self.push()                      # from here on the history is the end of the chunks

    def push(self):
        for i, x in enumerate(self.x):
            ppf.ppf_stream_push(self.handle, x, self.out[i], self.s, i)
        return self.out

    def __del__(self):
        if getattr(self, "handle", None):
            ppf.ppf_stream_destroy(self.handle)
            self.handle = None


class _Server:
    """64 streams of six plans on one server; a round is one chunk per stream."""

    def __init__(self, case, seed):
        self.server, self.handles = None, []
        shapes = _serve_streams(case)
        self.x = _serve_inputs(case, seed)
        self.out = torch.empty(sum(n * s for n, _, s in shapes), dtype=torch.complex64, device="cuda")
        self.plans = {}
        self.server = ppf.ppf_server_create(32 * 10**9, 2)
        self.chunks, at = [], 0
        for i, (n, taps, s) in enumerate(shapes):
            if (n, taps) not in self.plans:
                self.plans[n, taps] = ppf.Plan(n, taps, _coeffs(n, taps, "hamming").astype(np.float32))
            h = ppf.ppf_server_open_stream(self.server, self.plans[n, taps].handle)
            self.handles.append(h)
            self.chunks.append((h, self.x[i].data_ptr(), self.out.data_ptr() + 8 * at, s, i))
            at += n * s
        torch.cuda.synchronize()
        self.round()                     # from here on each history is the end of its chunk

    def round(self):
        for h, x, out, s, tag in self.chunks:
            ppf.ppf_server_submit(h, x, out, s, tag)
        ppf.ppf_server_drain(self.server, 60.0)
        ppf.ppf_server_poll(self.server, len(self.chunks))
        return self.out

    def __del__(self):
        for h in self.handles:
            ppf.ppf_stream_destroy(h)
        self.handles = []
        if self.server:
            ppf.ppf_server_destroy(self.server)
            self.server = None


def prepare(case, seed):
    if case["op"] == "stream":
        return {"case": case, "stream": _Stream(case, seed)}
    if case["op"] == "serve":
        return {"case": case, "server": _Server(case, seed)}
    n, m = case["n"], case["nspectra"]
    x = _samples((m + case["taps"] - 1) * n, case["dtype"], _generator(seed))
    if case["op"] == "power":
        out = torch.empty((m // case["k"], n), dtype=torch.float32, device="cuda")
    else:
        out = torch.empty((m, n), dtype=torch.complex64, device="cuda")
    return {"case": case, "x": x, "out": out, "plan": _plan(case)}


def run(state):
    case = state["case"]
    if case["op"] == "stream":
        return state["stream"].push()
    if case["op"] == "serve":
        return state["server"].round()
    if case["op"] == "power":
        return state["plan"].execute_power(state["x"], case["k"], out=state["out"], nspectra=case["nspectra"])
    return state["plan"].execute(state["x"], out=state["out"], nspectra=case["nspectra"])


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _ppf_work(n, taps, m, blocks_in, sample_bytes, coeff_bytes, out_bytes):
    return {"bytes": blocks_in * n * sample_bytes + out_bytes + taps * n * coeff_bytes,
            "flops": m * n * (4.0 * taps + 5.0 * math.log2(n))}


def work(case):
    if case["op"] == "serve":
        each = [_ppf_work(n, t, s, s, 8, 4, s * n * 8) for n, t, s in _serve_streams(case)]
        return {"bytes": sum(w["bytes"] for w in each), "flops": sum(w["flops"] for w in each)}
    n, taps, m = case["n"], case["taps"], case["nspectra"]
    sb = {"c32": 8, "c16": 4, "ci8": 2}[case["dtype"]]
    cb = 4 if case["dtype"] == "c32" else 2
    if case["op"] == "stream":
        m *= _stream_chunks(case)
        return _ppf_work(n, taps, m, m + taps - 1, sb, cb, m * n * 8)
    out = m // case["k"] * n * 4 if case["op"] == "power" else m * n * 8
    return _ppf_work(n, taps, m, m + taps - 1, sb, cb, out)


# ---------------------------------------------------------------------------
# the same outputs in 64 bits
# ---------------------------------------------------------------------------

def _exact_ppf(x, h, n, taps, m, k=0):
    """Spectra (or, with k, power sums over k spectra) of m+taps-1 blocks x, in slices of about 2^24 samples."""
    if not x.is_complex():
        x = torch.view_as_complex(x.float())
    x = x.reshape(-1, n)
    h = torch.from_numpy(h).to(x.device).reshape(taps, n)
    if k:
        out = torch.empty((m // k, n), dtype=torch.float64, device=x.device)
    else:
        out = torch.empty((m, n), dtype=torch.complex128, device=x.device)
    step = max(1, (1 << 24) // n)
    if k:
        step = max(1, step // k) * k
    for m0 in range(0, m, step):
        c = min(step, m - m0)
        u = torch.zeros((c, n), dtype=torch.complex128, device=x.device)
        for t in range(taps):
            u += h[t] * x[m0 + t:m0 + t + c].to(torch.complex128)
        s = torch.fft.fft(u, dim=1)
        if k:
            out[m0 // k:(m0 + c) // k] = (s.real.square() + s.imag.square()).reshape(c // k, k, n).sum(1)
        else:
            out[m0:m0 + c] = s
    return out


def exact(case, seed):
    if case["op"] == "serve":
        outs = []
        for (n, taps, s), x in zip(_serve_streams(case), _serve_inputs(case, seed)):
            h = _coeffs(n, taps, "hamming").astype(np.float32).astype(np.float64)
            outs.append(_exact_ppf(torch.cat([x[(s - taps + 1) * n:], x]), h, n, taps, s).reshape(-1))
        return torch.cat(outs)
    n, taps, m = case["n"], case["taps"], case["nspectra"]
    stored, shift = _stored_coeffs(case)
    h = stored.astype(np.float64) * 2.0 ** -shift
    if case["op"] == "stream":
        c = _stream_chunks(case)
        x = _samples(n * m * c, case["dtype"], _generator(seed))
        x = torch.cat([x[(m * c - taps + 1) * n:], x])
        return _exact_ppf(x, h, n, taps, m * c).reshape(c, m, n)
    x = _samples((m + taps - 1) * n, case["dtype"], _generator(seed))
    return _exact_ppf(x, h, n, taps, m, case["k"] if case["op"] == "power" else 0)
