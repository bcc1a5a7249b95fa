"""Performance cases: the calls that users of the library make, over the sizes they make them with.

A case names one kind of call and its sizes.  `listed()` gives the fixed cases, `draw()` more of the
same ranges, `prepare()` what a program holds before the call, `run()` one pass through the public
entry points, `work()` the bytes and operations such a pass cannot do without, and `exact()` the
computed numbers in plain numpy or torch, without the library's code.

The kinds and their ranges:

* message -- Context.encrypt / Context.decrypt of one message, one byte to 64 MiB, in the canonical
  format and (smaller) in the other two integrator formats.
* batch   -- Batch.encrypt / Batch.decrypt: 16 to 1024 messages of 1 KiB to 1 MiB, each with its own
  password, or the sequential version (one chain per message) on messages of 256 B to 4 KiB.
* stream  -- one message fed chunk by chunk, chunks of 4 KiB to 8 MiB, at once or deferred.
* serve   -- a burst of 50 to 800 requests through the request server, both directions mixed,
  lognormal sizes of median 16 KiB.
* bytes   -- the analyses of a byte sequence: histogram, entropy and autocorrelation, 1 KiB to 64 MiB.
* image   -- the analyses of a byte matrix: power spectrum and autocorrelation matrix, sides 16 to 1500.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1201_3114_amd as lz

KiB, MiB = 1024, 1024 * 1024
TAG = 24
OPS_PER_STEP = {"euler": 14, "euler_fma": 9, "rk4": 68}
N_IT = 3000  # steps per byte of the default format


def listed():
    return [
        # a short note or a record's field: the shortest call there is, one partial block
        {"name": "note_100B_enc", "kind": "message", "n": 100, "decrypt": False, "integrator": "euler"},
        # a page or a small file, the benchmark's small message
        {"name": "message_64KiB_dec", "kind": "message", "n": 64 * KiB, "decrypt": True, "integrator": "euler"},
        # a photograph: an ordinary file with a ragged end
        {"name": "message_3MB_dec", "kind": "message", "n": 3_000_001, "decrypt": True, "integrator": "euler"},
        # an ordinary large file, of no round size
        {"name": "message_24MB_enc", "kind": "message", "n": 24_000_000, "decrypt": False, "integrator": "euler"},
        # the benchmark's headline message, the largest call
        {"name": "message_64MiB_enc", "kind": "message", "n": 64 * MiB, "decrypt": False, "integrator": "euler"},
        # the costliest format, on a small file
        {"name": "message_rk4_256KiB_enc", "kind": "message", "n": 256 * KiB, "decrypt": False, "integrator": "rk4"},
        # a folder of files, each under its own password, in one launch
        {"name": "batch_512_enc", "kind": "batch", "count": 512, "lo": KiB, "hi": MiB, "sequential": False,
         "decrypt": False},
        # the paper's sequential version, many short records at a time
        {"name": "batch_sequential_dec", "kind": "batch", "count": 2048, "lo": 256, "hi": 4 * KiB, "sequential": True,
         "decrypt": True},
        # a file read in pieces as they arrive
        {"name": "stream_8MiB_deferred_enc", "kind": "stream", "n": 8 * MiB + 77, "chunk": 256 * KiB + 1,
         "deferred": True, "decrypt": False},
        # a burst of requests to a service
        {"name": "serve_400", "kind": "serve", "count": 400},
        # the statistical check of a ciphertext file: frequencies, entropy, correlation of neighbours
        {"name": "bytes_16MiB_lag256", "kind": "bytes", "n": 16 * MiB, "max_lag": 256},
        # the statistical check of an image of no convenient size
        {"name": "image_1009x1009", "kind": "image", "h": 1009, "w": 1009},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["message", "message", "message", "batch", "stream", "serve", "bytes", "image"])
    if kind == "message":
        integ = rng.choice(["euler", "euler", "euler", "euler_fma", "rk4"])
        hi = {"euler": 64 * MiB, "euler_fma": 64 * MiB, "rk4": 8 * MiB}[integ]
        return {"kind": kind, "n": _log_uniform(rng, 1, hi), "decrypt": rng.random() < 0.5, "integrator": integ}
    if kind == "batch":
        if rng.random() < 0.3:
            return {"kind": kind, "count": _log_uniform(rng, 64, 2048), "lo": 256, "hi": _log_uniform(rng, 300, 4 * KiB),
                    "sequential": True, "decrypt": rng.random() < 0.5}
        return {"kind": kind, "count": _log_uniform(rng, 16, 1024), "lo": KiB, "hi": _log_uniform(rng, 4 * KiB, MiB),
                "sequential": False, "decrypt": rng.random() < 0.5}
    if kind == "stream":
        deferred = rng.random() < 0.5
        chunk = _log_uniform(rng, 4 * KiB, 8 * MiB)
        # chunks run at once cost a block's serial time each: at most eight of them
        n = _log_uniform(rng, chunk, min(32 * MiB, chunk * (512 if deferred else 8)))
        return {"kind": kind, "n": n, "chunk": chunk, "deferred": deferred, "decrypt": rng.random() < 0.5}
    if kind == "serve":
        return {"kind": kind, "count": _log_uniform(rng, 50, 800)}
    if kind == "bytes":
        n = _log_uniform(rng, KiB, 64 * MiB)
        return {"kind": kind, "n": n, "max_lag": min(_log_uniform(rng, 16, 16384), n)}
    side = lambda: rng.choice([_log_uniform(rng, 16, 1500), _log_uniform(rng, 16, 1500), 1 << rng.randint(4, 10)])
    return {"kind": kind, "h": side(), "w": side()}


# ---- inputs -------------------------------------------------------------------------------------


def _password(rng, lo=8, hi=65):
    return bytes(rng.integers(32, 127, int(rng.integers(lo, hi)), dtype=np.uint8))


def _bytes(n, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 7919 + 11)
    return torch.randint(0, 256, (n,), dtype=torch.uint8, device="cuda", generator=g)


def _offsets(sizes, extra):
    offs = np.zeros(len(sizes), dtype=np.int64)
    offs[1:] = np.cumsum(np.asarray(sizes) + extra)[:-1]
    return offs, int(np.sum(sizes)) + extra * len(sizes)


def _batch_sizes(case, seed):
    # the sizes belong to the case (a seed changes contents and passwords alone), so passes compare
    rng = np.random.default_rng(case["count"] * 31 + case["hi"])
    lo, hi = case["lo"], max(case["lo"] + 1, case["hi"])
    return np.floor(np.exp(rng.uniform(math.log(lo), math.log(hi), case["count"]))).astype(np.int64)


def _serve_sizes(case):
    rng = np.random.default_rng(case["count"] * 17 + 5)
    sizes = np.clip(np.floor(rng.lognormal(math.log(16 * KiB), 1.5, case["count"])), 64, MiB).astype(np.int64)
    return sizes, rng.integers(0, 2, case["count"]).astype(np.uint8)


def _batch_encrypt(ctx, sizes, pws, data, in_off):
    """Ciphertexts of messages laid end to end (a program that decrypts has them in hand)."""
    out_off, total = _offsets(sizes, TAG)
    out = torch.empty(total, dtype=torch.uint8, device="cuda")
    b = lz.Batch(ctx, False, sizes, pws, data, in_off, out, out_off)
    b.encrypt()
    torch.cuda.synchronize()
    b.close()
    return out, out_off


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    state = {"kind": kind, "case": case}
    if kind == "message":
        state["ctx"] = ctx = lz.Context(0, lz.params(integrator=case["integrator"]))
        state["pw"] = _password(rng)
        data = _bytes(case["n"], seed)
        if case["decrypt"]:
            data = ctx.encrypt(data, state["pw"])
            state["status"] = torch.empty(1, dtype=torch.int32, device="cuda")
        state["data"] = data
    elif kind == "batch":
        sizes = _batch_sizes(case, seed)
        prm = lz.params(block_len=4 * KiB) if case["sequential"] else lz.params()
        state["ctx"] = ctx = lz.Context(0, prm)
        pws = [_password(rng) for _ in sizes]
        in_off, total = _offsets(sizes, 0)
        data = _bytes(total, seed)
        if case["decrypt"]:
            data, in_off = _batch_encrypt(ctx, sizes, pws, data, in_off)
            out_off, out_total = _offsets(sizes, 0)
            state["status"] = torch.full((len(sizes),), 99, dtype=torch.int32, device="cuda")
        else:
            out_off, out_total = _offsets(sizes, TAG)
        state["out"] = torch.empty(out_total, dtype=torch.uint8, device="cuda")
        state["batch"] = lz.Batch(ctx, case["decrypt"], sizes, pws, data, in_off, state["out"], out_off)
    elif kind == "stream":
        state["ctx"] = ctx = lz.Context(0)
        state["pw"] = _password(rng)
        data = _bytes(case["n"], seed)
        if case["decrypt"]:
            data = ctx.encrypt(data, state["pw"])
            state["tag"] = data[case["n"]:].clone()
            data = data[:case["n"]].clone()
            state["status"] = torch.empty(1, dtype=torch.int32, device="cuda")
        state["data"] = data
    elif kind == "serve":
        sizes, dec = _serve_sizes(case)
        state["ctx"] = ctx = lz.Context(0)
        pws = [_password(rng, 16) for _ in sizes]
        in_off, total = _offsets(sizes, 0)
        plain = _bytes(total, seed)
        ciph, c_off = _batch_encrypt(ctx, sizes, pws, plain, in_off)
        out_len = sizes + np.where(dec == 1, 0, TAG)
        out_off = np.zeros(len(sizes), dtype=np.int64)
        out_off[1:] = np.cumsum(out_len)[:-1]
        state["out"] = torch.zeros(int(out_len.sum()), dtype=torch.uint8, device="cuda")
        state["keep"] = (plain, ciph)
        state["src"] = np.where(dec == 1, ciph.data_ptr() + c_off, plain.data_ptr() + in_off)
        state["dst"] = state["out"].data_ptr() + out_off
        state["sizes"], state["dec"], state["pws"] = sizes, dec, pws
        state["server"] = lz.Server(ctx, 2 << 30)
    elif kind == "bytes":
        state["ctx"] = lz.Context(0)
        state["data"] = _bytes(case["n"], seed)
    else:
        state["ctx"] = lz.Context(0)
        state["data"] = _bytes(case["h"] * case["w"], seed).view(case["h"], case["w"])
    torch.cuda.synchronize()
    return state


# ---- one pass -----------------------------------------------------------------------------------


def _run_stream(state):
    case, data = state["case"], state["data"]
    n, chunk = case["n"], case["chunk"]
    out = torch.empty(n, dtype=torch.uint8, device="cuda")
    st = lz.Stream(state["ctx"], case["decrypt"], state["pw"])
    feed = st.update_deferred if case["deferred"] else st.update
    for o in range(0, n, chunk):
        e = min(n, o + chunk)
        feed(data[o:e], out=out[o:e])
    if case["decrypt"]:
        st.finish(state["tag"], status=state["status"])
        end = state["status"]
    else:
        end = st.finish()
    st.close()
    return {"out": out, "end": end}


def _run_serve(state):
    srv, count = state["server"], len(state["sizes"])
    now = lz.now_ns()
    srv.submit_many(np.arange(count), state["dec"], state["pws"], state["src"], state["sizes"], state["dst"],
                    np.full(count, now, dtype=np.uint64))
    status = np.full(count, 99, dtype=np.int64)
    left = count
    while left:
        for rid, st, _, _, _ in srv.poll(4096, 1000):
            status[rid] = st
            left -= 1
    return {"out": state["out"], "status": status}


def run(state):
    kind, case = state["kind"], state["case"]
    if kind == "message":
        if case["decrypt"]:
            return {"out": state["ctx"].decrypt(state["data"], state["pw"], status=state["status"]),
                    "status": state["status"]}
        return {"out": state["ctx"].encrypt(state["data"], state["pw"])}
    if kind == "batch":
        if case["decrypt"]:
            state["batch"].decrypt(state["status"])
            return {"out": state["out"], "status": state["status"]}
        state["batch"].encrypt()
        return {"out": state["out"]}
    if kind == "stream":
        return _run_stream(state)
    if kind == "serve":
        return _run_serve(state)
    if kind == "bytes":
        hist = lz.histogram(state["ctx"], state["data"])
        return {"hist": hist, "entropy": lz.entropy(state["ctx"], hist),
                "r": lz.autocorrelation(state["ctx"], state["data"], case["max_lag"])}
    return {"spectrum": lz.power_spectrum_2d(state["ctx"], state["data"]),
            "r": lz.autocorrelation_2d(state["ctx"], state["data"])}


# ---- the work a pass cannot do without ------------------------------------------------------------


def work(case):
    kind = case["kind"]
    if kind == "message":
        n = case["n"]
        return {"bytes": 2 * n + TAG, "flops": (OPS_PER_STEP[case["integrator"]] * N_IT + 11) * n}
    if kind in ("batch", "serve"):
        sizes = _batch_sizes(case, 0) if kind == "batch" else _serve_sizes(case)[0]
        n = int(sizes.sum())
        return {"bytes": 2 * n + TAG * len(sizes), "flops": (OPS_PER_STEP["euler"] * N_IT + 11) * n}
    if kind == "stream":
        n = case["n"]
        return {"bytes": 2 * n + TAG, "flops": (OPS_PER_STEP["euler"] * N_IT + 11) * n}
    if kind == "bytes":
        n, lags = case["n"], case["max_lag"] + 1
        # frequencies and correlation read the bytes once each; a lag sum by FFT of the padded sequence
        # would take 5 m log2 m operations, two of them, and directly two operations a byte and lag
        m = 2 * n
        return {"bytes": 2 * n + 8 * (256 + lags) + 8, "flops": min(2 * n * lags, 10 * m * math.log2(m))}
    h, w = case["h"], case["w"]
    n = h * w
    # the spectrum and the matrix are written once, the image is read once for each; a real transform
    # each way over an n-point image at 2.5 n log2 n operations, three of them in all
    return {"bytes": 2 * n + 16 * n, "flops": 3 * 2.5 * n * math.log2(max(2, n))}


# ---- the computed numbers in plain numpy and torch ---------------------------------------------------


def _exact_bytes(case, x):
    n, L = case["n"], case["max_lag"]
    hist = torch.bincount(x.to(torch.int64), minlength=256).cpu().numpy()
    p = hist[hist > 0].astype(np.longdouble) / n
    ent = float(-(p * np.log2(p)).sum())
    xi = x.to(torch.int64)
    S = [int(v) for v in torch.stack([(xi[: n - k] * xi[k:]).sum() for k in range(min(L, n - 1) + 1)]).cpu()]
    csum = torch.cumsum(xi, 0)
    T = int(csum[-1])
    ends = min(L, n - 1) + 1
    head = [0] + [int(v) for v in csum[: ends].cpu()]               # head[k] = first k bytes
    tail = [0] + [int(v) for v in torch.cumsum(xi.flip(0)[: ends], 0).cpu()]  # tail[k] = last k bytes
    r = np.zeros(L + 1)
    den = n * n * S[0] - n * T * T
    for k in range(ends):
        a, b = T - tail[k], T - head[k]
        r[k] = (n * n * S[k] - n * T * (a + b) + (n - k) * T * T) / den if den else float("nan")
    return {"hist": None, "entropy": ent, "r": r}


def _exact_image(case, x):
    img = x.cpu().numpy().reshape(case["h"], case["w"]).astype(np.int64)
    z = np.fft.fft2(img.astype(np.longdouble))
    spectrum = z.real ** 2 + z.imag ** 2
    n, s1, s2 = img.size, int(img.sum()), int((img * img).sum())
    den = n * s2 - s1 * s1
    # circular lag sums of the mean-removed bytes, as whole numbers: n S(d) - S1^2
    p = spectrum.copy()
    p[0, 0] = 0
    g = np.fft.ifft2(p).real * np.longdouble(n)
    r = g / np.longdouble(den) if den else np.full(img.shape, np.nan)
    return {"spectrum": spectrum.astype(np.float64), "r": r.astype(np.float64)}


def exact(case, seed):
    if case["kind"] == "bytes":
        if case["n"] * case["max_lag"] > 1 << 37:  # longer than a few seconds
            return None
        return _exact_bytes(case, _bytes(case["n"], seed))
    if case["kind"] == "image":
        return _exact_image(case, _bytes(case["h"] * case["w"], seed))
    return None
