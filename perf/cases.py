"""Timing cases of the spherical harmonic transforms, and a plain FP64
evaluation of each to hold their outputs against.

A case is a dict: `op` (what is called), `nside`, `lmax`, `batch` and `dtype`
(f64, f32 or bf16 maps).  The operations are the calls a program makes:

  map2alm   analysis of a batch of RING maps
  alm2map   synthesis of a batch of coefficient sets
  round     analysis, then synthesis of the result (filtering, denoising)
  grad      a training step's share: analysis, spectral loss, gradient map
  iter      three-iteration refined analysis (map-making, power spectra)
  nest2ring NESTED maps, as surveys ship them, into the transforms' order
"""
import math

import numpy as np
import torch

import paper_2510_01785_amd as shtx

_REAL = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
_ITERATIONS = 3


def _case(op, nside, lmax, batch, dtype, name=None):
    c = dict(op=op, nside=nside, lmax=lmax, batch=batch, dtype=dtype)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a single small map in double precision, to and back: latency of one
        # call after another (interactive use, a solver's inner loop)
        _case("round", 32, 95, 1, "f64", "round_n32_l95_b1_f64"),
        # a small request of a serving loop: a few low-resolution channels
        _case("alm2map", 64, 191, 3, "f32", "alm2map_n64_l191_b3_f32"),
        # a ragged one: odd band limit, an odd number of channels
        _case("map2alm", 128, 301, 5, "f32", "map2alm_n128_l301_b5_f32"),
        # a wide batch of medium resolution (ensembles, feature channels)
        _case("round", 256, 767, 64, "f32", "round_n256_l767_b64_f32"),
        # the throughput workload of the library, each direction by itself
        _case("map2alm", 1024, 2047, 16, "f32", "map2alm_n1024_l2047_b16_f32"),
        _case("alm2map", 1024, 2047, 16, "f32", "alm2map_n1024_l2047_b16_f32"),
        # the same analysis of bfloat16 maps
        _case("map2alm", 1024, 2047, 16, "bf16", "map2alm_n1024_l2047_b16_bf16"),
        # double precision, a half batch (simulation ensembles)
        _case("round", 512, 1023, 8, "f64", "round_n512_l1023_b8_f64"),
        # forward and backward through the analysis at the full band limit
        _case("grad", 512, 1535, 12, "f32", "grad_n512_l1535_b12_f32"),
        # one high-resolution map, single precision, full band limit
        _case("map2alm", 1024, 3071, 1, "f32", "map2alm_n1024_l3071_b1_f32"),
        # refined analysis of one map at the highest resolution
        _case("iter", 2048, 4095, 1, "f64", "iter_n2048_l4095_b1_f64"),
        # pixel order conversion of the throughput workload's maps
        _case("nest2ring", 1024, 2047, 16, "f32", "nest2ring_n1024_b16_f32"),
    ]


def draw(rng):
    """One more case of the same ranges: nside 32 .. 1024, band limits from
    nside to 3 nside - 1, 1 .. 64 channels within the pixels of 16 maps at
    nside 1024."""
    op = rng.choice(["map2alm", "map2alm", "alm2map", "alm2map", "round", "grad", "iter", "nest2ring"])
    nside = 1 << rng.randint(5, 9 if op in ("grad", "iter") else 10)
    lmax = rng.randint(nside, 3 * nside - 1)
    most = min(4 if op == "iter" else 64, 16 * (1024 // nside) ** 2)
    batch = max(1, min(most, int(2 ** rng.uniform(0, math.log2(most + 1)))))
    kinds = {"map2alm": ["f32", "f32", "bf16", "f64"], "grad": ["f32", "f32", "bf16", "f64"],
             "nest2ring": ["f32", "f64", "bf16"]}.get(op, ["f32", "f32", "f64"])
    return _case(op, nside, lmax, batch, rng.choice(kinds))


# ------------------------------------------------------------------ geometry
def _rings(nside):
    """Per ring, north to south: length, first pixel, z, longitude of the first
    pixel in units of pi / length (0 or 1)."""
    i = np.arange(1, 4 * nside)
    k = np.minimum(np.minimum(i, 4 * nside - i), nside)
    n = 4 * k
    start = np.concatenate([[0], np.cumsum(n)[:-1]])
    cap = 1.0 - k.astype(np.float64) ** 2 / (3.0 * nside * nside)
    z = np.where(i < nside, cap, np.where(i > 3 * nside, -cap, (4 * nside - 2 * i) / (3.0 * nside)))
    half = np.where((i < nside) | (i > 3 * nside), 1, 1 - (i - nside) % 2)
    return n, start, z, half


def _nalm(lmax):
    return (lmax + 1) * (lmax + 2) // 2


def _ls(lmax, device):
    """l of every coefficient idx(l, m) = m (2 lmax + 1 - m) / 2 + l."""
    return torch.cat([torch.arange(m, lmax + 1, device=device) for m in range(lmax + 1)])


# -------------------------------------------------------------------- inputs
def _field(nside, batch, seed, device):
    """Smooth random fields plus pixel noise, [batch, npix] float32: plane
    waves of random direction and wave number on the sphere, their amplitudes
    falling with the wave number."""
    g = torch.Generator(device=device).manual_seed(seed)
    n, _, z, half = _rings(nside)
    nt = torch.tensor(n, device=device)
    zp = torch.repeat_interleave(torch.tensor(z, device=device), nt)
    first = torch.repeat_interleave(torch.tensor(np.pi * half / n, device=device), nt)
    step = torch.repeat_interleave(torch.tensor(2 * np.pi / n, device=device), nt)
    at = torch.arange(12 * nside * nside, device=device) - torch.repeat_interleave(
        torch.tensor(np.concatenate([[0], np.cumsum(n)[:-1]]), device=device), nt)
    phi = first + step * at
    sth = torch.sqrt((1 - zp) * (1 + zp))
    x, y, zp = ((sth * torch.cos(phi)).float(), (sth * torch.sin(phi)).float(), zp.float())
    out = 0.05 * torch.randn(batch, 12 * nside * nside, device=device, generator=g)
    waves = 8
    u = torch.randn(waves, 3, device=device, generator=g)
    u = (u / u.norm(dim=1, keepdim=True)).tolist()
    amp = torch.randn(waves, batch, device=device, generator=g)
    turn = (2 * math.pi * torch.rand(waves, device=device, generator=g)).tolist()
    for w in range(waves):
        k = (2.0 * nside) ** ((w + 0.5) / waves)
        f = torch.cos(k * (u[w][0] * x + u[w][1] * y + u[w][2] * zp) + turn[w])
        out += (amp[w] / (1 + w)).unsqueeze(1) * f
    return out


def _coefficients(lmax, batch, seed, device):
    """Gaussian coefficients with C_l = (l + 10)^-2, [batch, nalm] complex128."""
    g = torch.Generator(device=device).manual_seed(seed)
    a = torch.randn(batch, _nalm(lmax), 2, device=device, generator=g, dtype=torch.float64)
    c = 1.0 / (_ls(lmax, device).double() + 10.0)
    a *= (c / math.sqrt(2.0))[:, None]
    a[:, :lmax + 1, 0] *= math.sqrt(2.0)
    a[:, :lmax + 1, 1] = 0
    return torch.view_as_complex(a)


def _input(case, seed, device):
    real = _REAL[case["dtype"]]
    if case["op"] == "alm2map":
        a = _coefficients(case["lmax"], case["batch"], seed, device)
        return a if real == torch.float64 else a.to(torch.complex64)
    return _field(case["nside"], case["batch"], seed, device).to(real)


def prepare(case, seed):
    device = torch.device("cuda", torch.cuda.current_device())
    s = dict(case, x=_input(case, seed, device))
    if case["op"] != "nest2ring":
        shtx.get_tables(case["nside"], case["lmax"], device)  # the resident plan of (nside, lmax)
    if case["op"] == "grad":
        s["x"].requires_grad_(True)
        s["w"] = 1.0 / (_ls(case["lmax"], device).to(torch.float64 if case["dtype"] == "f64" else torch.float32) + 1.0)
    return s


def run(s):
    op, x = s["op"], s["x"]
    if op == "map2alm":
        return shtx.map2alm(x, s["lmax"])
    if op == "alm2map":
        return shtx.alm2map(x, s["nside"], s["lmax"])
    if op == "round":
        a = shtx.map2alm(x, s["lmax"])
        return a, shtx.alm2map(a, s["nside"], s["lmax"])
    if op == "iter":
        return shtx.map2alm_iter(x, s["lmax"], _ITERATIONS)
    if op == "nest2ring":
        return shtx.nest2ring(x)
    a = shtx.map2alm(x, s["lmax"])
    loss = (s["w"] * (a.real.square() + a.imag.square())).sum()
    (g,) = torch.autograd.grad(loss, x)
    return a.detach(), g


# ---------------------------------------------------------------------- work
def work(case):
    """Bytes: inputs read once, outputs written once.  Operations: the ring
    FFTs and the Legendre sums over the (l, m, ring pair) terms with
    m <= l sin(theta), beyond which lambda_lm vanishes."""
    nside, lmax, B = case["nside"], case["lmax"], case["batch"]
    e = {"f64": 8, "f32": 4, "bf16": 2}[case["dtype"]]
    map_bytes = 12.0 * nside * nside * B * e
    if case["op"] == "nest2ring":
        return {"bytes": 2 * map_bytes, "flops": 0}
    alm_bytes = float(_nalm(lmax)) * B * (16 if case["dtype"] == "f64" else 8)
    n, _, z, _ = _rings(nside)
    fft = 2.5 * float((n * np.log2(n)).sum()) * B
    terms = 0.5 * lmax * lmax * float(np.sqrt(1 - z[:2 * nside] ** 2).sum())
    one = fft + 4.0 * B * terms
    times = {"round": 2, "grad": 2, "iter": 2 * _ITERATIONS + 1}.get(case["op"], 1)
    nbytes = {"round": 2 * map_bytes + alm_bytes, "grad": 2 * map_bytes + alm_bytes}.get(case["op"],
                                                                                       map_bytes + alm_bytes)
    return {"bytes": nbytes, "flops": times * one}


# --------------------------------------------------------------- exact values
class _Exact:
    """The transforms' definition in FP64: numpy's FFT on every ring, and the
    Legendre sums with lambda_lm from its three-term recurrence in l, carried
    with an exponent of its own per (m, ring)."""

    chunk = 16  # l of one parity per product

    def __init__(self, nside, lmax, device):
        self.N, self.L, self.dev = nside, lmax, device
        self.n, self.start, z, self.half = _rings(nside)
        self.z = torch.tensor(z[:2 * nside], device=device)
        m = np.arange(lmax + 1)
        self.col = m * (2 * lmax + 1 - m) // 2  # idx(l, m) - l

    def _lambda(self):
        """lambda_lm of the rings down to the equator, [m <= l, ring], for l = 0 .. lmax."""
        L, P, dev = self.L, 2 * self.N, self.dev
        s = torch.sqrt((1 - self.z) * (1 + self.z))
        cur = torch.zeros(L + 1, P, dtype=torch.float64, device=dev)
        prv = torch.zeros_like(cur)
        ex = torch.zeros_like(cur)
        x = torch.full((P,), 1.0 / math.sqrt(4 * math.pi), dtype=torch.float64, device=dev)
        e = torch.zeros(P, dtype=torch.float64, device=dev)

        def factor(v):
            return torch.exp2(v.clamp(min=-1000.0)) * (v > -900)
        f = torch.zeros_like(cur)
        for l in range(L + 1):
            if l:
                m = torch.arange(l, dtype=torch.float64, device=dev)[:, None]
                al = torch.sqrt((4.0 * l * l - 1) / (l * l - m * m))
                be = torch.sqrt(((l - 1.0) ** 2 - m * m).clamp(min=0) / (4.0 * (l - 1.0) ** 2 - 1)) if l > 1 else 0 * m
                nxt = al * (self.z * cur[:l] - be * prv[:l])
                prv[:l] = cur[:l]
                cur[:l] = nxt
                x = x * (-math.sqrt((2.0 * l + 1) / (2.0 * l))) * s
                x, k = torch.frexp(x)
                e = e + k
            cur[l], ex[l], f[l] = x, e, factor(e)
            if l % 8 == 0:
                big = cur[:l + 1].abs() > 2.0 ** 400
                down = 400.0 * big.double()
                cur[:l + 1] *= torch.exp2(-down)
                prv[:l + 1] *= torch.exp2(-down)
                ex[:l + 1] += down
                f[:l + 1] = factor(ex[:l + 1])
            yield l, cur[:l + 1] * f[:l + 1]

    def _products(self, take):
        """take(parity, l's, lambda [m, l, ring]) for runs of l of one parity."""
        L, P = self.L, 2 * self.N
        buf = [torch.zeros(L + 1, self.chunk, P, dtype=torch.float64, device=self.dev) for _ in range(2)]
        held = [[], []]
        for l, lam in self._lambda():
            q = l & 1
            buf[q][:l + 1, len(held[q])] = lam
            held[q].append(l)
            if len(held[q]) == self.chunk or l >= L - 1:
                take(q, held[q], buf[q][:, :len(held[q])])
                held[q] = []
                buf[q].zero_()

    def _swap(self, a, b):
        """Even-(l - m) and odd-(l - m) parts <-> the parts of even and odd l."""
        odd = (torch.arange(self.L + 1, device=self.dev) % 2 == 1)[:, None, None]
        return torch.where(odd, b, a), torch.where(odd, a, b)

    def analysis(self, maps, weight):
        """maps [B, npix] float64 -> [B, nalm] complex128, every pixel weighted by `weight`."""
        N, L, B = self.N, self.L, maps.shape[0]
        h = maps.cpu().numpy()
        m = np.arange(L + 1)
        F = np.zeros((2, 2 * N, L + 1, B), dtype=np.complex128)
        for r, (n, st, hf) in enumerate(zip(self.n, self.start, self.half)):
            X = np.fft.fft(h[:, st:st + n], axis=1)
            t = X[:, m % n] * np.exp(-1j * np.pi * ((m * hf) % (2 * n)) / n)
            south = r >= 2 * N
            F[int(south), 4 * N - 2 - r if south else r] = t.T
        F = torch.view_as_real(torch.from_numpy(F)).to(self.dev)
        F = F.permute(0, 2, 1, 3, 4).reshape(2, L + 1, 2 * N, 2 * B)
        E, O = self._swap(F[0] + F[1], F[0] - F[1])
        Y = [E.contiguous(), O.contiguous()]
        del F, E, O
        out = torch.zeros(_nalm(L), 2 * B, dtype=torch.float64, device=self.dev)
        col = torch.tensor(self.col, device=self.dev)

        def take(q, ls, lam):
            got = torch.bmm(lam, Y[q])
            for k, l in enumerate(ls):
                out[col[:l + 1] + l] = got[:l + 1, k]
        self._products(take)
        a = torch.view_as_complex(out.reshape(-1, B, 2).contiguous()).T * weight
        a = a.contiguous()
        a.imag[:, :L + 1] = 0
        return a

    def synthesis(self, alm):
        """alm [B, nalm] complex128 -> [B, npix] float64."""
        N, L, B = self.N, self.L, alm.shape[0]
        a = torch.view_as_real(alm.T.contiguous()).reshape(-1, 2 * B).clone()
        a[:L + 1, 1::2] = 0
        Z = [torch.zeros(L + 1, 2 * N, 2 * B, dtype=torch.float64, device=self.dev) for _ in range(2)]
        col = torch.tensor(self.col, device=self.dev)

        def take(q, ls, lam):
            rows = torch.zeros(L + 1, len(ls), 2 * B, dtype=torch.float64, device=self.dev)
            for k, l in enumerate(ls):
                rows[:l + 1, k] = a[col[:l + 1] + l]
            Z[q].baddbmm_(lam.transpose(1, 2), rows)
        self._products(take)
        E, O = self._swap(Z[0], Z[1])
        G = torch.stack([E + O, E - O]).reshape(2, L + 1, 2 * N, B, 2)
        G = torch.view_as_complex(G.permute(0, 2, 1, 3, 4).contiguous()).cpu().numpy()
        out = np.empty((B, 12 * N * N))
        m = np.arange(L + 1)
        for r, (n, st, hf) in enumerate(zip(self.n, self.start, self.half)):
            south = r >= 2 * N
            c = G[int(south), 4 * N - 2 - r if south else r] * np.exp(1j * np.pi * ((m * hf) % (2 * n)) / n)[:, None]
            runs = -(-(L + 1) // n)
            p = np.zeros((runs * n, B), dtype=np.complex128)
            p[:L + 1] = c
            p = p.reshape(runs, n, B)
            up = p.sum(axis=0)
            up[0] -= 0.5 * c[0]  # m = 0 is counted from both sides
            # f_j = 2 Re sum_k up_k exp(2 pi i j k / n)
            out[:, st:st + n] = 2 * n * np.fft.ifft(up, axis=0).real.T
        return torch.from_numpy(out).to(self.dev)


def _nest2ring(nside, maps):
    """RING-ordered copy of NESTED maps (the HEALPix definition)."""
    n, start, _, _ = _rings(nside)
    dev = maps.device
    p = torch.arange(12 * nside * nside, device=dev)
    f, q = p // (nside * nside), p % (nside * nside)
    x, y = torch.zeros_like(q), torch.zeros_like(q)
    for b in range(nside.bit_length()):
        x |= ((q >> (2 * b)) & 1) << b
        y |= ((q >> (2 * b + 1)) & 1) << b
    row = f // 4
    i = (row + 2) * nside - x - y - 1
    k = torch.minimum(torch.minimum(i, 4 * nside - i), torch.full_like(i, nside))
    shift = torch.where((i < nside) | (i > 3 * nside), torch.zeros_like(i), (i - nside) % 2)
    j = ((2 * (f % 4) + (row != 1).long()) * k + x - y + 1 + shift) // 2
    j = torch.where(j > 4 * k, j - 4 * k, torch.where(j < 1, j + 4 * k, j))
    ring = torch.tensor(start, device=dev)[i - 1] + j - 1
    out = torch.empty_like(maps)
    out[:, ring] = maps
    return out


def exact(case, seed):
    op, nside, lmax, B = case["op"], case["nside"], case["lmax"], case["batch"]
    passes = {"round": 2, "grad": 2, "iter": 2 * _ITERATIONS + 1}.get(op, 1)
    if passes * (nside / 1024.0) ** 2 * (B + 8) > 30:  # about half a minute and more
        return None
    device = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    x = _input(case, seed, device)
    if op == "nest2ring":
        return _nest2ring(nside, x)
    x = x.to(torch.complex128 if x.is_complex() else torch.float64)
    t = _Exact(nside, lmax, device)
    weight = 4 * math.pi / (12 * nside * nside)
    if op == "alm2map":
        return t.synthesis(x)
    a = t.analysis(x, weight)
    if op == "map2alm":
        return a
    if op == "round":
        return a, t.synthesis(a)
    if op == "iter":
        for _ in range(_ITERATIONS):
            a = a + t.analysis(x - t.synthesis(a), weight)
        return a
    g = a * (2.0 / (_ls(lmax, device).double() + 1.0))
    g[:, lmax + 1:] *= 0.5  # the adjoint on the m >= 0 storage
    return a, weight * t.synthesis(g)
