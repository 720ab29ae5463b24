"""The work a user of this library has it do, as timed cases.

Each case is one call, or one short chain of calls, through the package's public entry points on
inputs of the shapes and value distributions the search meets: whole dumps (channelize, correlate
and image, detect), uneven sub-bands as one batch, and every later stage on cubes of the imaged
size.  Sizes come from the repository's configurations and benchmark legs: the 16-antenna
configuration is the smallest work (launches and host time count), the 352-antenna ones the
largest.  `draw` spreads the same kinds over their ranges, with odd and ragged sizes.

Left out: FP16 / BF16 gridding (accuracy modes that exist to measure what a reduced-precision
gridder would lose), the plain FP32 correlator and the direct-Fourier imager (reference forms of
the int8 and gridding paths).
"""
import math

import numpy as np
import torch

import paper_2606_04304_amd as nb

C_LIGHT = 299792458.0
F_COARSE = 23.9e3   # coarse channel width, Hz
NU0 = 70e6          # its sky frequency
SIGMA = 8.0         # voltage noise per component, in int8 counts
RHO = (4.0 / 9.0, 1.0 / 36.0)  # channel correlations of the periodic Hann window's cross-products
WIDTHS = (1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 16, 20, 24, 28, 32, 36, 40, 44, 48, 50, 60, 70, 80, 90, 100)
MAD_K = 1.482602218505602


def listed():
    return [
        # The smallest dump: one commissioning array of 16 antennas.  Tens of microseconds of GPU
        # work, so launches, waits and host time are what a user sees.
        dict(name="tiny_dump", kind="dump", n_ant=16, radius=100.0, n_fft=4096, n_spec=16, n_chan=64, n_pix=64),
        # The instrument's dump (352 antennas, 65,536-point transforms, T = 32, 4,096 kept
        # channels, 256 x 256 images): the step that production repeats for every coarse channel.
        dict(name="instrument_dump", kind="dump", n_ant=352, radius=750.0, n_fft=65536, n_spec=32, n_chan=4096,
             n_pix=256),
        # Re-processing with other transform lengths: three uneven sub-bands as one captured batch.
        dict(name="subbands", kind="subbands", n_ant=352, radius=750.0, n_sub=3, first=0, n_chan=512),
        # The correlator alone on a long integration, where the matrix cores carry the work.
        dict(name="correlate_deep", kind="correlate", n_in=704, n_spec=1024, n_chan=1024),
        # The paper's batch of 300 channels over its 30 s dump (298 spectra: a row length that is
        # no multiple of 16), calibrated in the correlator, imaged from float visibilities at
        # 512 x 512 with the shortest baselines cut.
        dict(name="calibrated_batch", kind="calibrated", n_ant=352, radius=750.0, n_spec=298, n_chan=300, n_pix=512,
             uv_min=5.0),
        # Re-imaging kept Stokes-I visibilities of the instrument's dump.
        dict(name="image_allsky", kind="image", n_ant=352, radius=750.0, n_chan=4096, n_pix=256),
        # Standardising an imaged cube: candidates and the SNR cube that every later stage reads.
        dict(name="standardise", kind="detect", n_chan=4096, n_pix=256, mode=0),
        # Full Stage I search (26 boxcar widths, Benjamini-Hochberg) of that SNR cube.
        dict(name="stage1_search", kind="search", n_chan=4096, n_pix=256, cubes=False),
        # Drift-rate search over four sub-integrations of a dump, 33 drifts.
        dict(name="drift_search", kind="drift", n_sub=4, n_chan=4096, n_pix=256, max_drift=16),
        # Stage II centroid fits and cuts of 4,096 candidates on a cube.
        dict(name="stage2_cuts", kind="stage2", n_chan=4096, n_pix=256, n_cand=4096),
        # One training step of the candidate classifier: a mini-batch of 512 out of a stamp set.
        dict(name="classifier_train", kind="train", n_set=20000, batch=512),
        # Screening a dump's candidates: their stamps from the SNR cube, then the network's scores.
        dict(name="classifier_screen", kind="screen", n_chan=1024, n_pix=256, n_cand=4096),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("dump", "subbands", "correlate", "calibrated", "image", "detect", "search", "drift",
                       "stage2", "train", "screen"))
    n_ant = _log(rng, 8, 352)
    # a disk that leaves a sparse array some baselines short enough to image
    radius = rng.choice((100.0, 300.0, 750.0)[:1 + (n_ant >= 24) + (n_ant >= 96)])
    n_pix = rng.choice((64, 128, 256, 512))
    if kind == "dump":
        n_fft = 1 << rng.randint(10, 18)
        n_spec = min(_log(rng, 3, 400), max(3, (1 << 21) // n_fft))
        n_chan = min(_log(rng, 24, 4096), n_fft, (1 << 28) // (n_pix * n_pix))
        return dict(kind=kind, n_ant=n_ant, radius=radius, n_fft=n_fft, n_spec=n_spec, n_chan=n_chan, n_pix=n_pix)
    if kind == "subbands":
        return dict(kind=kind, n_ant=n_ant, radius=radius, n_sub=rng.randint(1, 3), first=rng.randint(0, 14),
                    n_chan=_log(rng, 16, 512))
    if kind == "correlate":
        n_in, n_spec = _log(rng, 6, 704), _log(rng, 2, 2048)
        cap = min((1 << 31) // (2 * n_in * n_spec), (1 << 32) // (4 * n_in * (n_in + 1)))
        return dict(kind=kind, n_in=n_in, n_spec=n_spec, n_chan=max(1, min(_log(rng, 8, 4096), cap)))
    if kind == "calibrated":
        return dict(kind=kind, n_ant=n_ant, radius=radius, n_spec=_log(rng, 4, 400), n_chan=_log(rng, 12, 300),
                    n_pix=n_pix, uv_min=rng.choice((0.0, 5.0, 12.5)))
    if kind == "image":
        return dict(kind=kind, n_ant=n_ant, radius=radius, n_chan=min(_log(rng, 24, 4096), (1 << 28) // (n_pix * n_pix)),
                    n_pix=n_pix)
    n_px = 8 * _log(rng, 4, 48)  # the detector, the searches and Stage II take any multiple of 8
    n_chan = min(_log(rng, 200, 8192), (1 << 28) // (n_px * n_px))
    if kind == "detect":
        return dict(kind=kind, n_chan=n_chan, n_pix=n_px, mode=rng.choice((0, 0, 1)))
    if kind == "search":
        return dict(kind=kind, n_chan=n_chan, n_pix=n_px, cubes=rng.choice((False, True)))
    if kind == "drift":
        n_sub = rng.randint(2, 8)
        return dict(kind=kind, n_sub=n_sub, n_chan=max(64, n_chan * 4 // (4 + n_sub)), n_pix=n_px,
                    max_drift=rng.choice((5, 10, 16, 16)))
    if kind == "stage2":
        return dict(kind=kind, n_chan=n_chan, n_pix=max(64, n_px), n_cand=_log(rng, 12, 4096))
    if kind == "train":
        return dict(kind=kind, n_set=_log(rng, 2000, 20000), batch=_log(rng, 32, 1024))
    return dict(kind=kind, n_chan=min(n_chan, 2048), n_pix=max(64, n_px), n_cand=_log(rng, 20, 4096))


# ---- inputs ----

def _gen(seed, k):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 64 + k)
    return g


def _rng(seed, k):
    return np.random.Generator(np.random.PCG64([int(seed), k]))


def _layout(n_ant, radius):
    """The array stands still: one layout per size, whatever the data's seed."""
    rng = _rng(n_ant, 1)
    r, a = radius * np.sqrt(rng.uniform(size=n_ant)), rng.uniform(0.0, 2.0 * math.pi, n_ant)
    return np.stack([r * np.cos(a), r * np.sin(a), np.zeros(n_ant)], axis=1)


def _freqs(n_fft, chan0, n_chan, nu0=NU0):
    return nu0 + (np.arange(chan0, chan0 + n_chan) - n_fft / 2) * (F_COARSE / n_fft)


def _voltages(xyz, n_fft, n_spec, chan0, n_chan, seed, k, n_tones=4):
    """Gaussian voltages of sigma 8 with a few on-bin tones from the sky, rounded to int8."""
    n_in = 2 * xyz.shape[0]
    out = torch.empty((n_in, n_spec * n_fft, 2), dtype=torch.int8, device="cuda")
    g, rng = _gen(seed, 100 + k), _rng(seed, 100 + k)
    n = torch.arange(n_fft, device="cuda", dtype=torch.float64)
    tones = []
    for _ in range(n_tones):
        bin_ = int(rng.integers(chan0 + n_chan // 8, chan0 + n_chan - n_chan // 8)) - n_fft // 2
        r, a = 0.8 * math.sqrt(rng.uniform()), rng.uniform(0.0, 2.0 * math.pi)
        turns = (NU0 + bin_ * F_COARSE / n_fft) * (xyz[:, 0] * r * math.cos(a) + xyz[:, 1] * r * math.sin(a)) / C_LIGHT
        # an amplitude that stands well above the noise of the image
        amp = SIGMA * math.sqrt(rng.uniform(4.0, 16.0) * 3.0 / (2.0 * n_fft * math.sqrt(n_spec) * xyz.shape[0]))
        w = torch.exp(2j * math.pi * ((bin_ * n) % n_fft) / n_fft) * amp
        tones.append((torch.view_as_real(w).float(), np.exp(2j * math.pi * turns)))
    step = max(1, (1 << 28) // (2 * n_spec * n_fft))
    for i0 in range(0, n_in, step):
        m = min(step, n_in - i0)
        x = torch.randn((m, n_spec, n_fft, 2), generator=g, device="cuda").mul_(SIGMA)
        for w, ph in tones:
            p = torch.from_numpy(ph[np.arange(i0, i0 + m) // 2]).to("cuda", torch.complex64)
            x += torch.view_as_real(torch.view_as_complex(w)[None, :] * p[:, None])[:, None]
        out[i0:i0 + m] = x.round_().clamp_(-127, 127).to(torch.int8).view(m, n_spec * n_fft, 2)
    return out


def _gain(n_fft):
    return 8.0 / (SIGMA * math.sqrt(3.0 * n_fft / 8.0))


def _spectra(n_chan, n_in, n_spec, seed, k):
    """Requantised spectra as the channelizer leaves them: Gaussian of sigma 8 codes."""
    g = _gen(seed, k)
    out = torch.empty((n_chan, n_in, 2, n_spec), dtype=torch.int8, device="cuda")
    step = max(1, (1 << 28) // (2 * n_in * n_spec))
    for c0 in range(0, n_chan, step):
        m = min(step, n_chan - c0)
        out[c0:c0 + m] = torch.randn((m, n_in, 2, n_spec), generator=g, device="cuda").mul_(8.0).round_().clamp_(-127, 127)
    return out


def _pairs(xyz, freq, n_pix, uv_min=0.0):
    """The imaged candidate pairs (a, b) of a gridding plan in Stokes-I row order: by 8 x 8 antenna
    block, then by position in the block."""
    a, b = np.tril_indices(xyz.shape[0], -1)
    d = xyz[a] - xyz[b]
    lim = (n_pix - 5) * 0.25
    lo, hi = freq.min() / C_LIGHT, freq.max() / C_LIGHT
    r = np.hypot(d[:, 0], d[:, 1])
    ok = (np.abs(d[:, 0]) * lo <= lim) & (np.abs(d[:, 1]) * lo <= lim) & (r * hi >= uv_min)
    a, b = a[ok], b[ok]
    tile = (a // 8) * (a // 8 + 1) // 2 + b // 8
    order = np.lexsort(((a % 8) * 8 + b % 8, tile))
    return a[order], b[order]


def _stokes(case, seed):
    """(xyz, freq, Stokes I of the candidate pairs): noise of a 32-spectra correlation and two
    point sources, one of them in all channels."""
    xyz = _layout(case["n_ant"], case["radius"])
    freq = _freqs(65536, 32768 - case["n_chan"] // 2, case["n_chan"])
    a, b = _pairs(xyz, freq, case["n_pix"])
    rng = _rng(seed, 3)
    v = torch.randn((case["n_chan"], max(1, a.size), 2), generator=_gen(seed, 3), device="cuda").mul_(512.0)
    if a.size:
        d = xyz[a] - xyz[b]
        for c0, c1, flux in ((0, case["n_chan"], 40.0), (case["n_chan"] // 3, case["n_chan"] // 3 + 2, 300.0)):
            r, t = 0.8 * math.sqrt(rng.uniform()), rng.uniform(0.0, 2.0 * math.pi)
            turns = np.outer(freq[c0:c1] / C_LIGHT, d[:, 0] * r * math.cos(t) + d[:, 1] * r * math.sin(t))
            ph = torch.from_numpy(2.0 * math.pi * (turns - np.floor(turns))).to("cuda", torch.float32)
            v[c0:c1, :, 0] += flux * torch.cos(ph)
            v[c0:c1, :, 1] += flux * torch.sin(ph)
    return xyz, freq, v.mul_(2.0).round_().mul_(0.5)  # sums of two integers, halved


def _horizon(n_pix):
    h = n_pix // 2
    i = torch.arange(n_pix, device="cuda") - h
    return (i[:, None] ** 2 + i[None, :] ** 2) < h * h


def _lines(cube, seed, k, n, widths):
    """Narrowband lines of the given widths at random pixels inside the horizon."""
    rng = _rng(seed, k)
    n_chan, n_pix = cube.shape[0], cube.shape[1]
    for i in range(n):
        w = min(int(widths[i % len(widths)]), n_chan)
        y, x = (int(q) for q in rng.integers(n_pix // 4, max(n_pix // 4 + 1, 3 * n_pix // 4), 2))
        c0 = int(rng.integers(0, n_chan - w + 1))
        cube[c0:c0 + w, y, x] += float(rng.uniform(8.0, 30.0)) / math.sqrt(w)


def _image_cube(n_chan, n_pix, seed):
    """An imaged cube: noise of one level, a smooth continuum per pixel, some lines."""
    g = _gen(seed, 5)
    x = torch.randn((n_chan, n_pix, n_pix), generator=g, device="cuda")
    _lines(x, seed, 5, 48, (1, 1, 2, 3))
    x.mul_(30.0).add_(torch.randn((n_pix, n_pix), generator=g, device="cuda").mul_(200.0)[None])
    return x


def _snr_cube(n_chan, n_pix, seed, k=6):
    """A standardised residual cube as the detector writes it: unit noise with the window's
    correlation between neighbouring channels, lines, zero outside the horizon."""
    w = torch.randn((n_chan + 2, n_pix, n_pix), generator=_gen(seed, k), device="cuda")
    x = w[2:] * 0.8693899
    x.add_(w[1:-1], alpha=0.4930979).add_(w[:-2], alpha=0.0319510)
    _lines(x, seed, k, 64, (1, 2, 3, 5, 8, 12, 20, 32, 50, 80, 100))
    return x.mul_(_horizon(n_pix)[None])


def _params(seed):
    rng = _rng(seed, 7)
    p = []
    for co, ci in ((32, 33), (64, 32), (32, 64)):
        p += [rng.uniform(-1.0, 1.0, co * ci * 9) * math.sqrt(6.0 / (ci * 9)), rng.uniform(-0.05, 0.05, co)]
    p += [rng.uniform(-1.0, 1.0, 32) * math.sqrt(6.0 / 32), np.zeros(1)]
    return np.concatenate(p).astype(np.float32)


def _train_set(case, seed):
    g = _gen(seed, 8)
    labels = (torch.rand(case["n_set"], generator=g, device="cuda") < 0.4).float()
    stamps = torch.randn((case["n_set"], 33, 9, 9), generator=g, device="cuda")
    stamps[:, 16, 4, 4] += 6.0 * labels  # tones: one bright channel at the centre
    index = torch.randperm(case["n_set"], generator=g, device="cuda")[:case["batch"]].to(torch.int32)
    return stamps.half(), labels, index


def _blobs(case, seed):
    """A unit-noise cube with beam-shaped blobs, a quarter of them three times wider, and their
    candidate records [n][5]."""
    n, n_chan, n_pix = case["n_cand"], case["n_chan"], case["n_pix"]
    cube = torch.randn((n_chan, n_pix, n_pix), generator=_gen(seed, 9), device="cuda")
    rng = _rng(seed, 9)
    xs, ys = rng.integers(8, n_pix - 8, n), rng.integers(8, n_pix - 8, n)
    cs = rng.integers(0, n_chan, n)
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).to("cuda")  # noqa: E731
    k = torch.arange(-5, 6, device="cuda")
    u = k[None, None, :] - dev(rng.uniform(-0.5, 0.5, n))[:, None, None]
    v = k[None, :, None] - dev(rng.uniform(-0.5, 0.5, n))[:, None, None]
    f = dev(np.where(np.arange(n) % 4 == 3, 3.0, 1.0))[:, None, None]
    amp = dev(rng.uniform(8.0, 40.0, n))[:, None, None]
    ct, st = math.cos(0.5), math.sin(0.5)
    patch = amp * torch.exp(-0.5 * (((u * ct + v * st) / (1.6 * f)) ** 2 + ((v * ct - u * st) / (1.2 * f)) ** 2))
    at = ((dev(cs)[:, None, None] * n_pix + dev(ys)[:, None, None] + k[None, :, None]) * n_pix
          + dev(xs)[:, None, None] + k[None, None, :])
    flat, patch = cube.view(-1), patch.float()
    for i0 in range(0, n, 64):  # in order: blobs may overlap, and sums have to repeat
        for i in range(i0, min(n, i0 + 64)):
            flat[at[i].view(-1)] += patch[i].view(-1)
    cands = np.stack([xs, ys, cs, np.ones(n, np.int64), np.zeros(n, np.int64)], axis=1).astype(np.int32)
    return cube, dev(cands)


SUB_NT = ((1 << 14, 128), (1 << 16, 32), (1 << 18, 8), (1 << 15, 64), (1 << 17, 16))
SUB_PIX = (256, 128, 512)


def _subband(case, i):
    n_fft, n_spec = SUB_NT[(case["first"] + i) % 5]
    return n_fft, n_spec, n_fft // 2 - case["n_chan"] // 2, SUB_PIX[(case["first"] + i) % 3]


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "dump":
        n_in, n_fft, T, C, P = 2 * case["n_ant"], case["n_fft"], case["n_spec"], case["n_chan"], case["n_pix"]
        chan0 = n_fft // 2 - C // 2
        xyz = _layout(case["n_ant"], case["radius"])
        s["volt"] = _voltages(xyz, n_fft, T, chan0, C, seed, 0)
        s["gain"] = torch.full((n_in,), _gain(n_fft), dtype=torch.float32, device="cuda")
        s["plan"] = nb.nbsi_image_plan_create(xyz, _freqs(n_fft, chan0, C), P)
        s["chan0"] = chan0
        s["spec"] = torch.empty((C, n_in, 2, T), dtype=torch.int8, device="cuda")
        s["vis"] = torch.empty((C, n_in * (n_in + 1) // 2, 2), dtype=torch.int32, device="cuda")
        s["stokes"] = torch.zeros((C, max(1, s["plan"].n_pairs()), 2), dtype=torch.float32, device="cuda")
        s["img"] = torch.empty((C, P, P), dtype=torch.float32, device="cuda")
    elif kind == "subbands":
        xyz = _layout(case["n_ant"], case["radius"])
        subs = []
        for i in range(case["n_sub"]):
            n_fft, T, chan0, P = _subband(case, i)
            subs.append(dict(volt=_voltages(xyz, n_fft, T, chan0, case["n_chan"], seed, 1 + i),
                             gain=torch.full((2 * case["n_ant"],), _gain(n_fft), dtype=torch.float32, device="cuda"),
                             n_fft=n_fft, n_spec=T, chan0=chan0, n_chan=case["n_chan"],
                             freq_hz=_freqs(n_fft, chan0, case["n_chan"], NU0 + i * F_COARSE), n_pix=P))
        s["batch"] = nb.nbsi_batch_plan(xyz, subs)
    elif kind == "correlate":
        s["spec"] = _spectra(case["n_chan"], case["n_in"], case["n_spec"], seed, 2)
        s["vis"] = torch.empty((case["n_chan"], case["n_in"] * (case["n_in"] + 1) // 2, 2), dtype=torch.int32,
                               device="cuda")
    elif kind == "calibrated":
        n_in, C, P = 2 * case["n_ant"], case["n_chan"], case["n_pix"]
        xyz = _layout(case["n_ant"], case["radius"])
        s["spec"] = _spectra(C, n_in, case["n_spec"], seed, 2)
        s["cal"] = _cal(case, seed)
        s["plan"] = nb.nbsi_image_plan_create(xyz, _freqs(65536, 32768 - C // 2, C), P, uv_min=case["uv_min"])
        s["vis"] = torch.empty((C, n_in * (n_in + 1) // 2, 2), dtype=torch.float32, device="cuda")
        s["img"] = torch.empty((C, P, P), dtype=torch.float32, device="cuda")
    elif kind == "image":
        xyz, freq, s["stokes"] = _stokes(case, seed)
        s["plan"] = nb.nbsi_image_plan_create(xyz, freq, case["n_pix"])
        s["img"] = torch.empty((case["n_chan"], case["n_pix"], case["n_pix"]), dtype=torch.float32, device="cuda")
    elif kind == "detect":
        s["cube"] = _image_cube(case["n_chan"], case["n_pix"], seed)
    elif kind == "search":
        s["cube"] = _snr_cube(case["n_chan"], case["n_pix"], seed)
    elif kind == "drift":
        s["cube"] = torch.stack([_snr_cube(case["n_chan"], case["n_pix"], seed, 10 + i) for i in range(case["n_sub"])])
        s["best"] = torch.empty((case["n_chan"], case["n_pix"], case["n_pix"]), dtype=torch.float32, device="cuda")
        s["drift"] = torch.empty((case["n_chan"], case["n_pix"], case["n_pix"]), dtype=torch.int8, device="cuda")
    elif kind == "stage2":
        s["cube"], s["cands"] = _blobs(case, seed)
        k = 2.0 * math.sqrt(2.0 * math.log(2.0))
        s["beam"] = torch.tensor([[k * 1.6, k * 1.2, 0.5]] * case["n_chan"], dtype=torch.float64, device="cuda")
        s["out"] = torch.empty((case["n_cand"], 160), dtype=torch.uint8, device="cuda")
    elif kind == "train":
        s["stamps"], s["labels"], s["index"] = _train_set(case, seed)
        s["net"] = nb.nbsi_net_create(_params(seed), max_batch=case["batch"])
        s["grad"] = torch.empty(nb.NBSI_NET_NPARAM, dtype=torch.float32, device="cuda")
    else:
        s["cube"] = _snr_cube(case["n_chan"], case["n_pix"], seed)
        s["cands"] = _screen_cands(case, seed)
        s["net"] = nb.nbsi_net_create(_params(seed), max_batch=case["n_cand"])
    return s


def _cal(case, seed):
    """Correction factors of unit order: 20 % amplitude and any phase per input and channel."""
    g = _gen(seed, 4)
    shape = (case["n_chan"], 2 * case["n_ant"])
    amp = 1.0 + 0.2 * torch.randn(shape, generator=g, device="cuda")
    ph = 2.0 * math.pi * torch.rand(shape, generator=g, device="cuda")
    return torch.stack([amp * torch.cos(ph), amp * torch.sin(ph)], dim=-1).contiguous()


def _screen_cands(case, seed):
    rng = _rng(seed, 11)
    n = case["n_cand"]
    c = np.stack([rng.integers(0, case["n_pix"], n), rng.integers(0, case["n_pix"], n),
                  rng.integers(0, case["n_chan"], n), np.ones(n, np.int64), np.zeros(n, np.int64)], axis=1)
    return torch.from_numpy(c.astype(np.int32)).to("cuda")


CAND_ROOM = 2048


def _records(rec):
    """Candidate records in arrays of a fixed length (their number differs from dump to dump)."""
    at, snr = np.zeros((CAND_ROOM, 4), np.int32), np.zeros(CAND_ROOM, np.float32)
    m = min(CAND_ROOM, rec.size)
    at[:m] = rec[:m].view(np.int32).reshape(-1, 5)[:, :4]
    snr[:m] = rec["snr"][:m]
    return {"at": at, "snr": snr}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "dump":
        nb.nbsi_channelize(state["volt"], case["n_fft"], case["n_spec"], state["chan0"], case["n_chan"], state["gain"],
                           spec_q=state["spec"])
        nb.nbsi_correlate_image(state["spec"], state["plan"], vis=state["vis"], stokes_i=state["stokes"],
                                img=state["img"])
        rec, _, n = nb.nbsi_detect(state["img"])
        return {"spec": state["spec"], "vis": state["vis"], "stokes": state["stokes"], "img": state["img"], "n": n,
                **_records(rec)}
    if kind == "subbands":
        state["batch"].run()
        return [{k: d[k] for k in ("spec_q", "vis", "img")} for d in state["batch"].subbands]
    if kind == "correlate":
        return nb.nbsi_correlate(state["spec"], vis=state["vis"])
    if kind == "calibrated":
        nb.nbsi_correlate_cal(state["spec"], state["cal"], vis=state["vis"])
        nb.nbsi_image(state["plan"], state["vis"], img=state["img"])
        return {"vis": state["vis"], "img": state["img"]}
    if kind == "image":
        return nb.nbsi_image_stokes(state["plan"], state["stokes"], img=state["img"])
    if kind == "detect":
        rec, snr, n = nb.nbsi_detect(state["cube"], mode=case["mode"], want_snr=True)
        return {"snr_cube": snr, "n": n, **_records(rec)}
    if kind == "search":
        rec, thr, k, best, width = nb.nbsi_search(state["cube"], rho=RHO, want_cubes=case["cubes"])
        return {"threshold": thr, "k": k, "best": best, "best_width": width, **_records(rec)}
    if kind == "drift":
        nb.nbsi_dedoppler(state["cube"], case["max_drift"], best=state["best"], drift=state["drift"])
        return {"best": state["best"], "drift": state["drift"]}
    if kind == "stage2":
        nb.nbsi_stage2(state["cube"], state["cands"], state["beam"], out=state["out"])
        rec = nb.fits_host(state["out"], case["n_cand"])
        return {k: np.ascontiguousarray(rec[k]) for k in rec.dtype.names}
    if kind == "train":
        loss, grad = state["net"].grad(state["stamps"], state["labels"], index=state["index"], grad=state["grad"])
        state["net"].adam(grad)
        return {"loss": loss, "grad": grad}
    stamps = nb.nbsi_stamps(state["cube"], state["cands"])
    return {"stamps": stamps, "logits": state["net"].forward(stamps)}


# ---- what the paths cannot do without ----

def _chan_work(n_in, n_fft, n_spec, n_chan):
    keep = 1 << max(0, (n_chan - 1).bit_length())
    return (2 * n_in * n_fft * n_spec + 2 * n_in * n_spec * n_chan,
            n_in * n_spec * 5.0 * n_fft * math.log2(min(keep, n_fft)) + 8.0 * n_in * n_spec * n_fft)


def _corr_work(n_in, n_spec, n_chan):
    prod = n_in * (n_in + 1) // 2
    return n_chan * (2 * n_in * n_spec + 8 * prod), 8.0 * prod * n_spec * n_chan


def _image_work(n_base, n_chan, n_pix):
    # an 8 x 8 footprint of complex sums per baseline (half of the grid is free by symmetry) and
    # a real 2D transform of the twice oversampled grid
    return (n_chan * (8 * n_base + 4 * n_pix * n_pix),
            n_chan * (n_base * 256.0 + 2.5 * 4 * n_pix * n_pix * math.log2(4.0 * n_pix * n_pix)))


def _n_base(case, n_pix):
    xyz = _layout(case["n_ant"], case["radius"])
    return _pairs(xyz, np.array([NU0]), n_pix, case.get("uv_min", 0.0))[0].size


def work(case):
    kind = case["kind"]
    if kind == "dump":
        a = _chan_work(2 * case["n_ant"], case["n_fft"], case["n_spec"], case["n_chan"])
        b = _corr_work(2 * case["n_ant"], case["n_spec"], case["n_chan"])
        c = _image_work(_n_base(case, case["n_pix"]), case["n_chan"], case["n_pix"])
        vox = case["n_chan"] * case["n_pix"] ** 2
        # every product is an output of its own: spectra, visibilities, Stokes I, images; the
        # detector reads the cube again
        return {"bytes": a[0] + b[0] + c[0] + 4 * vox, "flops": a[1] + b[1] + c[1] + 4.0 * vox}
    if kind == "subbands":
        by, fl = 0, 0.0
        for i in range(case["n_sub"]):
            n_fft, T, _, P = _subband(case, i)
            for w in (_chan_work(2 * case["n_ant"], n_fft, T, case["n_chan"]),
                      _corr_work(2 * case["n_ant"], T, case["n_chan"]),
                      _image_work(_n_base(case, P), case["n_chan"], P)):
                by, fl = by + w[0], fl + w[1]
        return {"bytes": by, "flops": fl}
    if kind == "correlate":
        by, fl = _corr_work(case["n_in"], case["n_spec"], case["n_chan"])
        return {"bytes": by, "flops": fl}
    if kind == "calibrated":
        b = _corr_work(2 * case["n_ant"], case["n_spec"], case["n_chan"])
        c = _image_work(_n_base(case, case["n_pix"]), case["n_chan"], case["n_pix"])
        return {"bytes": b[0] + c[0] + 16 * case["n_ant"] * case["n_chan"], "flops": b[1] + c[1]}
    if kind == "image":
        by, fl = _image_work(_n_base(case, case["n_pix"]), case["n_chan"], case["n_pix"])
        return {"bytes": by, "flops": fl}
    if kind == "train":
        return {"bytes": case["batch"] * 2 * 33 * 81 + 5 * 4 * nb.NBSI_NET_NPARAM, "flops": 21.0e6 * case["batch"]}
    if kind == "screen":
        return {"bytes": case["n_cand"] * (6 * 33 * 81 + 24) + 4 * nb.NBSI_NET_NPARAM, "flops": 7.52e6 * case["n_cand"]}
    vox = case["n_chan"] * case["n_pix"] ** 2
    if kind == "detect":
        return {"bytes": 8 * vox, "flops": 6.0 * vox}
    if kind == "search":
        return {"bytes": (9 if case["cubes"] else 4) * vox, "flops": 3.0 * len(WIDTHS) * vox}
    if kind == "drift":
        return {"bytes": (4 * case["n_sub"] + 5) * vox,
                "flops": (2.0 * case["max_drift"] + 1) * (case["n_sub"] + 1) * vox}
    return {"bytes": 4 * vox + 180 * case["n_cand"], "flops": 4.0 * vox + 81 * 40.0 * 20 * case["n_cand"]}


# ---- the same in 64 bits ----

def _exact_images(xyz, freq, n_pix, uv_min, vis_of):
    """Direct Fourier sums of the imaged baselines; vis_of(c, a, b) -> complex128 Stokes I."""
    a, b = _pairs(xyz, freq, n_pix, uv_min)
    d = torch.from_numpy(xyz[a] - xyz[b]).to("cuda")
    lm = (torch.arange(n_pix, device="cuda", dtype=torch.float64) - n_pix / 2) * (2.0 / n_pix)
    out = torch.zeros((len(freq), n_pix, n_pix), dtype=torch.float64, device="cuda")
    lim = (n_pix - 5) * 0.25
    ta, tb = torch.from_numpy(a).to("cuda"), torch.from_numpy(b).to("cuda")
    for c, nu in enumerate(freq):
        u, v = d[:, 0] * float(nu) / C_LIGHT, d[:, 1] * float(nu) / C_LIGHT
        ok = (u.abs() <= lim) & (v.abs() <= lim) & (torch.sqrt(u * u + v * v) >= uv_min)
        val = vis_of(c, ta, tb) * ok
        n = int(ok.sum())
        if n == 0:
            continue
        pu, pv = 2.0 * math.pi * torch.outer(u, lm), 2.0 * math.pi * torch.outer(lm, v)
        cv, sv, cu, su = torch.cos(pv), torch.sin(pv), torch.cos(pu), torch.sin(pu)
        # Re[V exp(-i (pu + pv))], summed over baselines as two real products
        re = (cv * val.real + sv * val.imag) @ cu + (cv * val.imag - sv * val.real) @ su
        out[c] = re / n
    return out


def _median(x):
    """Median along the last axis, the mean of the central pair for an even count."""
    s = torch.sort(x, dim=-1).values
    n = x.shape[-1]
    return 0.5 * (s[..., (n - 1) // 2] + s[..., n // 2])


def _exact_net(params, stamps, labels=None):
    """Logits (and loss and gradient of every parameter) of the classifier in float64."""
    p = torch.from_numpy(params.astype(np.float64)).to("cuda").requires_grad_(labels is not None)
    x, at = stamps.double().reshape(-1, 33, 9, 9), 0

    def take(*shape):
        nonlocal at
        n = math.prod(shape)
        at += n
        return p[at - n:at].view(*shape)

    for co, ci in ((32, 33), (64, 32), (32, 64)):
        w, bias = take(co, ci, 3, 3), take(co)
        q = torch.nn.functional.pad(x, (1, 1, 1, 1))
        z = bias.view(1, co, 1).expand(x.shape[0], co, 81)
        for dy in range(3):
            for dx in range(3):
                z = z + torch.matmul(w[:, :, dy, dx], q[:, :, dy:dy + 9, dx:dx + 9].reshape(-1, ci, 81))
        x = torch.relu(z).view(-1, co, 9, 9)
    w4, b4 = take(32), take(1)
    logit = x.mean(dim=(2, 3)) @ w4 + b4
    if labels is None:
        return logit.detach()
    loss = torch.nn.functional.binary_cross_entropy_with_logits(logit, labels.double())
    loss.backward()
    return loss.detach().view(1), p.grad


def _q_tail(s):
    return 0.5 * torch.special.erfc(s / math.sqrt(2.0))


def exact(case, seed):
    kind = case["kind"]
    none = {"at": None, "snr": None}
    if kind == "calibrated":
        C, n_in = case["n_chan"], 2 * case["n_ant"]
        spec, cal = _spectra(C, n_in, case["n_spec"], seed, 2), torch.view_as_complex(_cal(case, seed).double())
        i, j = (torch.from_numpy(k).to("cuda") for k in np.tril_indices(n_in))
        vis = torch.empty((C, i.numel(), 2), dtype=torch.float64, device="cuda")
        for c in range(C):
            re, im = spec[c, :, 0].double(), spec[c, :, 1].double()
            full = torch.complex(re @ re.T + im @ im.T, im @ re.T - re @ im.T)
            vis[c] = torch.view_as_real(full[i, j] * cal[c][i] * cal[c][j].conj())
        t = lambda a, b: a * (a + 1) // 2 + b  # noqa: E731
        v = torch.view_as_complex(vis)
        img = _exact_images(_layout(case["n_ant"], case["radius"]), _freqs(65536, 32768 - C // 2, C),
                            case["n_pix"], case["uv_min"],
                            lambda c, a, b: 0.5 * (v[c, t(2 * a, 2 * b)] + v[c, t(2 * a + 1, 2 * b + 1)]))
        return {"vis": vis, "img": img}
    if kind == "image":
        xyz, freq, st = _stokes(case, seed)
        z = torch.view_as_complex(st)
        return _exact_images(xyz, freq, case["n_pix"], 0.0, lambda c, a, b: z[c, :a.numel()].to(torch.complex128))
    if kind == "detect":
        cube, hor = _image_cube(case["n_chan"], case["n_pix"], seed), _horizon(case["n_pix"])
        snr = torch.zeros(cube.shape, dtype=torch.float64, device="cuda")
        if case["mode"]:
            x = cube[:, hor].double()
            for c0 in range(0, x.shape[0], 256):
                d = x[c0:c0 + 256]
                d -= _median(d)[:, None]
                d /= MAD_K * _median(d.abs())[:, None]
            snr[:, hor] = x - _median(x.T.contiguous())[None]
            return {"snr_cube": snr, "n": None, **none}
        for y in range(case["n_pix"]):
            if bool(hor[y].any()):
                x = cube[:, y, hor[y]].double().T.contiguous()
                x -= _median(x)[:, None]
                x /= MAD_K * _median(x.abs())[:, None]
                snr[:, y, hor[y]] = x.T
        return {"snr_cube": snr, "n": None, **none}
    if kind == "search":
        cube, hor = _snr_cube(case["n_chan"], case["n_pix"], seed), _horizon(case["n_pix"])
        C = case["n_chan"]
        best = torch.full(cube.shape, -math.inf, dtype=torch.float64, device="cuda")
        for y0 in range(0, case["n_pix"], 64):
            x = cube[:, y0:y0 + 64].double()
            s = torch.cat([torch.zeros_like(x[:1]), torch.cumsum(x, dim=0)])
            for w in WIDTHS:
                if w > C:
                    break
                sd = math.sqrt(w + 2.0 * sum((w - l) * RHO[l - 1] for l in range(1, min(w - 1, 2) + 1)))
                b = best[w // 2:w // 2 + C - w + 1, y0:y0 + 64]
                torch.maximum(b, (s[w:] - s[:C - w + 1]) / sd, out=b)
        v = best[:, hor]
        m = v.numel()
        v = torch.sort(v[v > 2.0], descending=True).values
        ok = torch.nonzero(_q_tail(v) <= torch.arange(1, v.numel() + 1, device="cuda") * (0.01 / m)).view(-1)
        thr = float(v[ok[-1]]) if ok.numel() else math.inf
        return {"threshold": thr, "k": None, "best": best if case["cubes"] else None, "best_width": None, **none}
    if kind == "drift":
        S, C, D = case["n_sub"], case["n_chan"], case["max_drift"]
        best = torch.full((C, case["n_pix"], case["n_pix"]), -math.inf, dtype=torch.float64, device="cuda")
        cubes = [_snr_cube(C, case["n_pix"], seed, 10 + i) for i in range(S)]
        for y0 in range(0, case["n_pix"], 64):
            x = [q[:, y0:y0 + 64].double() for q in cubes]
            for d in range(-D, D + 1):
                lo, hi = max(0, -d), C - max(0, d)
                if hi <= lo:
                    continue
                acc = torch.zeros_like(x[0][lo:hi])
                for i in range(S):
                    k = (2 * abs(d) * i + S - 1) // (2 * (S - 1)) if S > 1 else 0
                    k = k if d > 0 else -k
                    acc += x[i][lo + k:hi + k]
                b = best[lo:hi, y0:y0 + 64]
                torch.maximum(b, acc / math.sqrt(S), out=b)
        return {"best": best, "drift": None}
    if kind == "train":
        stamps, labels, index = _train_set(case, seed)
        loss, grad = _exact_net(_params(seed), stamps[index.long()], labels[index.long()])
        return {"loss": loss, "grad": grad}
    if kind == "screen":
        cube, cands = _snr_cube(case["n_chan"], case["n_pix"], seed), _screen_cands(case, seed).long()
        pad = torch.nn.functional.pad(cube, (4, 4, 4, 4, 16, 16))
        dc = torch.arange(33, device="cuda")[None, :, None, None] + cands[:, 2, None, None, None]
        dy = torch.arange(9, device="cuda")[None, None, :, None] + cands[:, 1, None, None, None]
        dx = torch.arange(9, device="cuda")[None, None, None, :] + cands[:, 0, None, None, None]
        stamps = pad[dc, dy, dx].half()
        return {"stamps": stamps.double(), "logits": _exact_net(_params(seed), stamps)}
    # Whole dumps, sub-bands and correlations are integers or follow from them; Stage II's fits
    # are minima found by iteration.
    return None
