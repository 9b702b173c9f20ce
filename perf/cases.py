"""Performance cases of the ACDC / AFDF cascades.

Each case is one pass of a user's program through the public binding
(``paper_1511_05946_amd.acdc``), in one of four modes:

* ``train``      autograd: ``acdc_cascade`` and the gradients of x, A, D (and
                 the bias) for an upstream gradient; cascades without ReLU.
* ``step``       the calls of a training loop that owns its buffers, one
                 forward that stores the layer inputs of the next micro-batch
                 and one backward from the stored layer inputs of the previous
                 one. The stored inputs are part of the state, so the ReLU
                 decisions that the backward follows are given: two correct
                 implementations decide differently where a value lies within
                 rounding of zero, and gradients would then differ by whole
                 elements.
* ``recompute``  forward without stored layer inputs, then a backward that
                 recomputes them (the paper's policy for memory, Sec. 5.3).
* ``serve``      forward alone into caller-owned buffers.

Inputs follow the workload recipe of the package: x ~ N(0, 1), or its positive
part ahead of ReLU layers, diagonals ~ N(1, 0.1^2) (complex ones with an
imaginary part ~ N(0, 0.1^2)), biases ~ N(0, 0.1^2), uniform random
permutations between layers (the first layer keeps the identity).
"""

import math

import torch

from paper_1511_05946_amd import acdc

FUSED_WIDTHS = (8, 16, 32, 64, 128, 256, 512, 1024, 2048, 4096, 8192, 9216, 16384, 32768)
WIDE = (65536, 131072, 262144)
COMPLEX_WIDTHS = (8, 16, 32, 64, 128, 256, 512, 1024, 2048, 4096, 8192, 16384)
COMPLEX_WIDE = (32768, 65536, 131072)


def _case(mode, N, K, batch, perm=False, relu=False, bias=False, cplx=False, **more):
    return dict(more, mode=mode, N=N, K=K, batch=batch, perm=perm, relu=relu, bias=bias, complex=cplx)


def listed():
    return [
        # operator recovery by minibatch gradient descent: 32-wide rows, minibatches of 100, launch-bound
        _case("train", 32, 16, 100, name="fit_n32_k16_b100"),
        # one layer in a small network: the smallest call, host and launches
        _case("train", 256, 1, 64, name="layer_n256_k1_b64"),
        # a structured layer in place of a dense one at the batch of the layer comparison
        _case("step", 2048, 1, 128, name="layer_n2048_k1_b128"),
        # inference on a handful of requests through a whole ReLU cascade with biases: latency
        _case("serve", 4096, 12, 16, perm=True, relu=True, bias=True, name="serve_n4096_k12_b16"),
        # a mid-size permuted cascade under autograd
        _case("train", 1024, 12, 4096, perm=True, name="train_n1024_k12_b4096"),
        # the benchmark cascade
        _case("step", 4096, 12, 8192, perm=True, relu=True, name="step_n4096_k12_b8192"),
        # the same cascade with biases at a ragged, moderate batch (the last one of an epoch, a data-parallel shard)
        _case("step", 4096, 12, 1003, perm=True, relu=True, bias=True, name="step_n4096_k12_b1003_bias"),
        # flattened 6x6x256 convolution features, mixed radix
        _case("step", 9216, 16, 1024, perm=True, relu=True, name="step_n9216_k16_b1024"),
        # wide fused rows without memory for the layer inputs
        _case("recompute", 16384, 8, 500, perm=True, bias=True, name="recompute_n16384_k8_b500_bias"),
        # complex cascade, fused
        _case("train", 4096, 8, 2048, perm=True, cplx=True, name="train_afdf_n4096_k8_b2048"),
        # rows past the fused widths: every layer goes through HBM
        _case("step", 65536, 12, 512, perm=True, relu=True, name="step_n65536_k12_b512"),
        _case("train", 65536, 8, 256, perm=True, cplx=True, name="train_afdf_n65536_k8_b256"),
    ]


def draw(rng):
    """Another case of the same ranges: any supported width, 1 to 16 layers,
    batches from one row up (odd ones as likely as even ones), every option."""
    cplx = rng.random() < 0.25
    wide = rng.random() < 0.2
    N = rng.choice((COMPLEX_WIDE if cplx else WIDE) if wide else (COMPLEX_WIDTHS if cplx else FUSED_WIDTHS))
    K = rng.randint(1, 16)
    mode = rng.choice(("train", "step", "recompute", "serve"))
    relu = not cplx and mode in ("step", "serve") and rng.random() < 0.6
    # elements through all layers: below the largest listed cases', with room for
    # the recomputed forward and for rows whose transform takes a pass more
    most = 1.2e8 if wide else 2.4e8
    cap = max(1.0, min(65536.0, most / (N * K * (2 if cplx else 1))))
    batch = int(round(math.exp(rng.uniform(0.0, math.log(cap)))))
    return _case(mode, N, K, max(1, batch), perm=rng.random() < 0.75, relu=relu,
                 bias=not cplx and rng.random() < 0.35, cplx=cplx)


def _flags(c):
    return (acdc.FLAG_PERM if c["perm"] else 0) | (acdc.FLAG_RELU if c["relu"] else 0)


def _inputs(c, seed):
    """(x, A, D, bias or None, perm or None, grad_y) on the GPU."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(seed)
    N, K, B, cplx = c["N"], c["K"], c["batch"], c["complex"]

    def normal(rows, mean=0.0, std=1.0, im_std=1.0):
        re = torch.randn(rows, N, generator=gen, device=dev).mul_(std).add_(mean)
        if not cplx:
            return re
        return torch.complex(re, torch.randn(rows, N, generator=gen, device=dev).mul_(im_std))

    x = normal(B)
    if c["relu"]:
        x = x.clamp_(min=0.0)
    A, D = normal(K, 1.0, 0.1, 0.1), normal(K, 1.0, 0.1, 0.1)
    gy = normal(B)
    bias = normal(K, 0.0, 0.1) if c["bias"] else None
    perm = None
    if c["perm"]:
        perm = torch.arange(N, device=dev).repeat(K, 1)
        for k in range(1, K):
            perm[k] = torch.argsort(torch.rand(N, generator=gen, device=dev))
        perm = perm.to(torch.int32).contiguous()
    return x, A, D, bias, perm, gy


# ------------------------------------------------- the cascade in plain torch

def _turn(N, device):
    k = torch.arange(N, dtype=torch.float64, device=device)
    return torch.polar(torch.ones_like(k), -math.pi * k / (2 * N)), k


def _dct(u):
    """Orthonormal DCT-II of the rows (one even/odd-reversed FFT), in u's precision."""
    N = u.shape[1]
    w, _ = _turn(N, u.device)
    scale = torch.full((N,), math.sqrt(2.0 / N), dtype=torch.float64, device=u.device)
    scale[0] = math.sqrt(1.0 / N)
    v = torch.cat([u[:, 0::2], u[:, 1::2].flip(1)], dim=1)
    V = torch.fft.fft(v.to(torch.complex128 if u.dtype == torch.float64 else torch.complex64))
    return (V * (w * scale).to(V.dtype)).real


def _idct(X):
    """The inverse (orthonormal DCT-III)."""
    N = X.shape[1]
    w, _ = _turn(N, X.device)
    scale = torch.full((N,), math.sqrt(N / 2.0), dtype=torch.float64, device=X.device)
    scale[0] = math.sqrt(float(N))
    Y = X * scale.to(X.dtype)
    # V[k] = (Y[k] - i Y[N-k]) / w[k], with Y[N] = 0
    back = torch.cat([torch.zeros_like(Y[:, :1]), Y[:, 1:].flip(1)], dim=1)
    V = torch.complex(Y, -back) * w.conj().to(torch.complex128 if X.dtype == torch.float64 else torch.complex64)
    v = torch.fft.ifft(V).real
    out = torch.empty_like(X)
    out[:, 0::2] = v[:, : (N + 1) // 2]
    out[:, 1::2] = v[:, (N + 1) // 2:].flip(1)
    return out


def _forward(c, x, A, D, bias, perm):
    """(y, layer inputs u_0 .. u_{K-1}) in x's precision."""
    f, g = (torch.fft.fft, torch.fft.ifft) if c["complex"] else (_dct, _idct)
    z, inputs = x, []
    for k in range(c["K"]):
        u = z[:, perm[k].long()] if perm is not None else z
        inputs.append(u)
        h = f(u * A[k]) * D[k]
        if bias is not None:
            h = h + bias[k]
        z = g(h)
        if c["relu"] and k < c["K"] - 1:
            z = z.clamp(min=0.0)
    return z, inputs


def _backward(c, inputs, gy, A, D, bias, perm):
    f, b = (torch.fft.fft, torch.fft.ifft) if c["complex"] else (_dct, _idct)
    N, g = c["N"], gy
    gA, gD = torch.empty_like(A), torch.empty_like(D)
    gB = torch.empty_like(bias) if bias is not None else None
    for k in range(c["K"] - 1, -1, -1):
        u = inputs[k].to(g.dtype)
        h2 = f(u * A[k])
        g3 = f(g) / N if c["complex"] else f(g)
        gD[k] = (g3 * h2.conj()).sum(0) if c["complex"] else (g3 * h2).sum(0)
        if gB is not None:
            gB[k] = g3.sum(0)
        if c["complex"]:
            g1 = b(g3 * D[k].conj()) * N
            gA[k] = (g1 * u.conj()).sum(0)
            gu = g1 * A[k].conj()
        else:
            g1 = b(g3 * D[k])
            gA[k] = (g1 * u).sum(0)
            gu = g1 * A[k]
        if c["relu"] and k > 0:
            gu = gu * (u > 0)
        if perm is not None:
            g = torch.empty_like(gu)
            g[:, perm[k].long()] = gu
        else:
            g = gu
    return (g, gA, gD) + ((gB,) if gB is not None else ())


def _stored(c, inputs):
    """The layer inputs in the order of the library's buffer: u_1 .. u_{K-1},
    then u_0 with permutations."""
    order = inputs[1:] + (inputs[:1] if c["perm"] else [])
    return torch.cat([u.reshape(-1) for u in order]) if order else inputs[0].new_empty(0)


def _unstored(c, saved, x):
    B, N, K = c["batch"], c["N"], c["K"]
    view = saved.view(-1, B, N)
    return [view[K - 1] if c["perm"] else x] + [view[k] for k in range(K - 1)]


# ------------------------------------------------------------------ the cases

def prepare(case, seed):
    c = case
    x, A, D, bias, perm, gy = _inputs(c, seed)
    s = {"case": c, "flags": _flags(c), "x": x, "A": A, "D": D, "bias": bias, "perm": perm, "gy": gy}
    acdc.prepare(c["N"], s["flags"] | (acdc.FLAG_COMPLEX if c["complex"] else 0))
    K = c["K"]

    def space(n):
        return torch.empty(max(n, 1), dtype=torch.uint8, device=x.device)

    if c["mode"] == "train":
        for t in (x, A, D, bias):
            if t is not None:
                t.requires_grad_(True)
    else:
        s["y"] = torch.empty_like(x)
        s["fws"] = space(acdc.forward_workspace_bytes(x, K, s["flags"], bias=bias))
    if c["mode"] == "step":
        # the previous micro-batch: its input, and its layer inputs as stored by its forward
        s["x0"] = x.roll(1, 0).contiguous() if c["batch"] > 1 else x.clone()
        s["saved0"] = _stored(c, _forward(c, s["x0"], A, D, bias, perm)[1])
        s["saved"] = acdc.alloc_saved(x, K, s["flags"])
    if c["mode"] in ("step", "recompute"):
        s["gx"] = torch.empty_like(x)
        s["grads"] = tuple(torch.empty_like(t) for t in (A, D, bias) if t is not None)
        s["bws"] = space(acdc.backward_workspace_bytes(x, K, s["flags"], c["mode"] == "step", bias=bias))
    return s


def run(state):
    s = state
    c, x, A, D, bias, perm, flags = s["case"], s["x"], s["A"], s["D"], s["bias"], s["perm"], s["flags"]
    if c["mode"] == "train":
        y = acdc.acdc_cascade(x, A, D, perm, flags, bias)
        wrt = [t for t in (x, A, D, bias) if t is not None]
        return (y.detach(),) + torch.autograd.grad(y, wrt, s["gy"])
    if c["mode"] == "serve":
        return acdc.forward(x, A, D, perm, flags, out=s["y"], bias=bias, workspace=s["fws"])[0]
    if c["mode"] == "recompute":
        y, _ = acdc.forward(x, A, D, perm, flags, out=s["y"], bias=bias, workspace=s["fws"])
        grads = acdc.backward(x, s["gy"], A, D, perm, flags, bias=bias, grads=s["grads"], out=s["gx"],
                              workspace=s["bws"])
        return (y,) + grads
    y, saved = acdc.forward(x, A, D, perm, flags, out=s["y"], saved=s["saved"], bias=bias, workspace=s["fws"])
    grads = acdc.backward(s["x0"], s["gy"], A, D, perm, flags, saved=s["saved0"], bias=bias, grads=s["grads"],
                          out=s["gx"], workspace=s["bws"])
    return (y, saved) + grads


def exact(case, seed):
    c = case
    x, A, D, bias, perm, gy = _inputs(c, seed)
    wide = torch.complex128 if c["complex"] else torch.float64
    up = [t.to(wide) if t is not None else None for t in (A, D, bias)]
    y, inputs = _forward(c, x.to(wide), *up, perm)
    if c["mode"] == "serve":
        return y
    if c["mode"] != "step":
        return (y,) + _backward(c, inputs, gy.to(wide), *up, perm)
    saved = _stored(c, inputs)
    del inputs
    x0 = x.roll(1, 0).contiguous() if c["batch"] > 1 else x.clone()
    given = _unstored(c, _stored(c, _forward(c, x0, A, D, bias, perm)[1]), x0)
    return (y, saved) + _backward(c, given, gy.to(wide), *up, perm)


def work(case):
    c = case
    B, N, K, e = c["batch"], c["N"], c["K"], 8 if c["complex"] else 4
    lg = math.log2(N)
    per = (10 * N * lg + 12 * N) if c["complex"] else (4 * N + 5 * N * lg)  # one row through one layer
    params = K * N * (e * (3 if c["bias"] else 2) + (4 if c["perm"] else 0))
    rows = B * N * e
    if c["mode"] == "serve":
        return {"bytes": 2 * rows + params, "flops": B * K * per}
    grads = K * N * e * (3 if c["bias"] else 2)
    stored = (K - 1 + (1 if c["perm"] else 0)) if c["mode"] == "step" else 0
    # x, y; x, grad_y, grad_x; in a step the stored layer inputs are an output and an input
    return {"bytes": (5 + 2 * stored) * rows + 2 * params + grads, "flops": 2 * B * K * per}


def tolerance(case):
    # single precision throughout: the transforms' rounding grows with the
    # square root of the layers, the batch sums add little to it
    return {"rel": 2e-6 * math.sqrt(case["K"] + 1.0)}
