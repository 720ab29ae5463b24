"""Edges of the size-dependent dispatches: shapes on both sides of every rule that picks a kernel
or a register / tile count, against the oracle or against the general form."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2606_04304_amd as nb
import synth
from oracle import drift as odr
from oracle import search as osr
from test_gpu_drift import test_dedoppler_matches_oracle as dedoppler_parity
from test_gpu_net import _stamps
from test_gpu_net import test_forward_matches_oracle as forward_parity
from test_gpu_parity import _noise_vis, _rel, detect_parity
from test_gpu_search import _check_bank, _cube, _expected_records

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("mode", [nb.NBSI_DETECT_PER_PIXEL, nb.NBSI_DETECT_PER_IMAGE])
@pytest.mark.parametrize("n_chan,n_pix", [(12, 8), (1024, 8), (1025, 24), (2048, 16), (2049, 8), (4096, 8), (4097, 8)])
def test_detect_register_counts(n_chan, n_pix, mode):
    """Spectra at and just past 16, 32 and 64 registers of 64 channels, SNR cube included."""
    detect_parity(n_chan, n_pix, mode)


@pytest.mark.parametrize("mode", [nb.NBSI_DETECT_PER_PIXEL, nb.NBSI_DETECT_PER_IMAGE])
@pytest.mark.parametrize("n_chan", [3, 10, 100, 1500])
def test_detect_snr_cube_in_place(n_chan, mode):
    """The SNR cube written over the images equals the one written beside them, and a pixel with
    a non-finite value is zero in both."""
    print(f"detect in place n_chan={n_chan} mode={mode}", flush=True)
    rng = np.random.default_rng(n_chan)
    cube = torch.from_numpy(rng.standard_normal((n_chan, 16, 16)).astype(np.float32)).to(DEV)
    cube[n_chan // 2, 8, 9] = 30.0
    cube[n_chan - 1, 7, 7] = float("nan")
    rec, snr, n = nb.nbsi_detect(cube, mode=mode, want_snr=True)
    both = cube.clone()
    rec2, snr2, n2 = nb.nbsi_detect_noalloc(both, mode=mode, snr=both)
    assert n == n2 and np.array_equal(rec, rec2)
    assert torch.equal(snr, snr2)
    assert torch.all(snr[:, 7, 7] == 0) and torch.isfinite(snr).all()


@pytest.mark.parametrize("n_sub,n_chan,n_pix,max_drift", [(1, 3, 8, 16), (2, 33, 8, 16), (4, 35, 16, 16), (4, 67, 24, 16),
                                                          (4, 68, 8, 15), (7, 130, 8, 16), (8, 65, 16, 16), (5, 64, 8, 0)])
def test_dedoppler_segment_ends(n_sub, n_chan, n_pix, max_drift):
    """Bands shorter than a segment, ending inside a step, and just past a segment's end; pixel
    counts below a workgroup's; the full drift range and less."""
    dedoppler_parity(n_sub, n_chan, n_pix, max_drift)


@pytest.mark.parametrize("n_chan,n_pix", [(3, 8), (99, 8), (100, 16), (101, 8), (127, 8), (128, 24), (129, 8), (145, 8),
                                          (256, 16), (257, 8), (383, 8), (640, 40)])
def test_search_default_bank_edges(n_chan, n_pix):
    """The default bank on bands shorter than its widths, at the ends of its 16-channel groups,
    128-channel blocks and 64-channel segments: the cubes against the oracle, and the same records
    with the width cube, from it, and from the widths found voxel by voxel."""
    print(f"search default bank n_chan={n_chan} n_pix={n_pix}", flush=True)
    lines = [(n_pix // 2, n_pix // 2, n_chan // 2, 1, 25.0)]
    r = _cube(n_chan, n_pix, n_chan + n_pix, lines)
    x = torch.from_numpy(r).to(DEV)
    for q in (0.01, 0.4):  # few provisional detections, and nearly all voxels
        rec, thr, k, S, W = nb.nbsi_search(x, fdr_q=q, want_cubes=True)
        rec2, thr2, k2, _, _ = nb.nbsi_search(x, fdr_q=q)
        assert (thr, k) == (thr2, k2) and np.array_equal(rec, rec2)
        _check_bank(r, S, W)


@pytest.mark.parametrize("n_pix,n_ant,radius,freqs", [
    (64, 3, 30.0, (70e6,)),                  # bands of a few entries, or none
    (64, 60, 60.0, (40e6, 70e6, 110e6)),     # one octave and a half: block ranges far wider than a channel's
    (128, 130, 120.0, (55e6, 85e6)),         # several staging rounds per band
    (256, 352, 500.0, (69e6, 71e6)),
    (256, 20, 60.0, (50e6, 100e6)),          # all baselines in the middle bands
    (512, 40, 400.0, (60e6, 75e6)),          # four-row bands: the vector form
])
def test_image_grid_block_ranges(n_pix, n_ant, radius, freqs):
    """Gridding over the plan's list ranges: plans whose frequencies move baselines by many grid
    columns, sparse bands and bands of several rounds, against the direct-Fourier oracle."""
    print(f"image grid ranges n_pix={n_pix} n_ant={n_ant}", flush=True)
    xyz = synth.antenna_layout(n_ant, radius, 5 + n_pix)
    freq = np.array(freqs)
    plan = nb.nbsi_image_plan_create(xyz, freq, n_pix, nb.NBSI_IMAGE_GRID)
    np.testing.assert_array_equal(plan.n_baselines(), oracle.count_baselines(xyz, freq, n_pix))
    vis = _noise_vis(len(freqs), n_ant, n_pix + n_ant)
    img = nb.nbsi_image(plan, torch.from_numpy(vis).to(DEV)).cpu().numpy()
    if n_pix < 256:
        ref = oracle.image_dft(vis, xyz, freq, n_pix, grid_n_pix=n_pix)
    else:  # sampled pixels of the large images
        rng = np.random.default_rng(n_pix)
        pix = rng.integers(0, n_pix, (300, 2)).astype(np.int32)
        ref = oracle.image_dft_pixels(vis, xyz, freq, n_pix, pix, grid_n_pix=n_pix)
        img = img[:, pix[:, 1], pix[:, 0]]
    assert _rel(img, ref)[0] < 1e-5


@pytest.mark.parametrize("n_pix", [8, 64, 128, 136, 256, 264])
def test_image_statistics_register_counts(n_pix):
    """Per-image medians and MADs where a thread holds 1 to 64 values and where it holds none, on
    noise, few distinct values, one value, ramps that mislead the samples, a range wider than the
    largest float, subnormal values, outliers and non-finite pixels."""
    print(f"image statistics n_pix={n_pix}", flush=True)
    rng = np.random.default_rng(n_pix)
    cube = rng.standard_normal((12, n_pix, n_pix)).astype(np.float32)
    cube[1] = rng.integers(-2, 3, (n_pix, n_pix))
    cube[2] = 7.5
    cube[3] = np.arange(n_pix * n_pix, dtype=np.float32).reshape(n_pix, n_pix)
    cube[4] = -cube[3].T
    cube[5] *= 1e38
    cube[6] *= 1e-41
    cube[7, ::3, ::2] = 1e30
    cube[8, rng.random((n_pix, n_pix)) < 0.4] = np.nan
    cube[9, ::2] = np.inf
    cube[10] = np.exp(8.0 * cube[10])
    x = torch.from_numpy(cube).to(DEV)
    beam = torch.full((12, 3), float("nan"), dtype=torch.float64, device=DEV)
    cands = torch.tensor([[n_pix // 2, n_pix // 2, c, 1, 0] for c in range(12)], dtype=torch.int32, device=DEV)
    # Stage II reports the channel's 1.4826 MAD through chi2_red = rss / (sigma^2 (n - 7))
    fit = nb.fits_host(nb.nbsi_stage2(x, cands, beam, half=2), 12)
    h = n_pix // 2
    yy, xx = np.mgrid[:n_pix, :n_pix]
    hor = (xx - h) ** 2 + (yy - h) ** 2 < h * h
    for c in range(12):
        v = cube[c][hor]
        v = v[np.isfinite(v)]
        med = np.float32(0.5) * (np.sort(v)[(v.size - 1) // 2] + np.sort(v)[v.size // 2])
        d = np.sort(np.abs(v - med))
        mad = np.float32(0.5) * (d[(v.size - 1) // 2] + d[v.size // 2])
        sigma = float(np.float32(1.482602218505602) * mad)
        if np.isfinite(fit["chi2_red"][c]) and fit["rss"][c] > 0 and sigma > 0:
            got = np.sqrt(fit["rss"][c] / (fit["chi2_red"][c] * (25 - 7)))
            assert abs(got - sigma) <= 1e-6 * sigma, (c, got, sigma)


@pytest.mark.parametrize("n", [2, 5, 8, 19, 128, 511])
def test_net_row_groups(n):
    """Batches whose 128-row groups start and end at every place of a stamp, a last group of one
    row (n = 19) and of whole groups only (n = 128): against the oracle, and every logit bit for bit
    that of the stamp in another place of a batch (each output is one sum in a fixed order)."""
    forward_parity(n, 50 + n)
    net = nb.Net(synth.net_init(50 + n), max_batch=512)
    x = torch.from_numpy(_stamps(n, 50 + n)).to(DEV)
    z = net.forward(x)
    for shift in (1, n // 2, n - 1):
        order = ((torch.arange(n) + shift) % n).to(torch.int32).to(DEV)
        assert torch.equal(net.forward(x, index=order), z[order.long()])
    assert torch.equal(net.forward(x[n - 1:].clone()), z[n - 1:])
    net.close()


@pytest.mark.parametrize("half", [2, 5])
def test_stage2_fits_beside_the_statistics(half):
    """2^22 voxels take the two-stream form, half of them the single sequence.  The same 512
    channels twice over have the same noise median, so the records are the same, bit for bit."""
    g = torch.Generator(device="cpu").manual_seed(half)
    n_chan, n_pix = 512, 64
    cube = torch.randn((n_chan, n_pix, n_pix), generator=g)
    cube[7] *= 9.0  # a channel of deviant noise
    yy, xx = torch.meshgrid(torch.arange(n_pix), torch.arange(n_pix), indexing="ij")
    cands = []
    for i, (x, y, c, width) in enumerate([(20, 30, 3, 1.2), (33, 31, 7, 1.2), (40, 22, 100, 4.0), (31, 32, 511, 0.6),
                                          (0, 5, 9, 1.0), (63, 63, 10, 1.0), (30, 40, -1, 1.0)]):
        if c >= 0:
            cube[c] += 40.0 * torch.exp(-((xx - x) ** 2 + (yy - y) ** 2) / (2.0 * width ** 2))
        cands.append([x, y, c, 1, 0])
    cands = torch.tensor(cands * 40, dtype=torch.int32, device="cuda:0")
    beam = torch.tensor([[2.8, 2.8, 0.0]], dtype=torch.float64, device="cuda:0").repeat(2 * n_chan, 1)
    one = cube.to("cuda:0")
    two = torch.cat([one, one])
    assert two.numel() == 1 << 22
    want = nb.fits_host(nb.nbsi_stage2(one, cands, beam[:n_chan].contiguous(), half=half), len(cands))
    for _ in range(2):  # the second call finds the first one's statistics in the scratch
        got = nb.fits_host(nb.nbsi_stage2(two, cands, beam, half=half), len(cands))
        assert got.tobytes() == want.tobytes()
    flags = want["flags"][:7]
    assert flags[1] & 4 and not flags[0] & 4 and flags[2] & 2 and all(flags[4:] & 8)
    assert np.isfinite(want["chi2_red"][:4]).all() and np.isnan(want["chi2_red"][4:7]).all()


def test_search_infinite_detections_only():
    """Every provisional detection infinite: the threshold is +inf (not NaN), and the survivor, whose
    re-evaluated sum is infinite too, is kept."""
    n_chan, n_pix = 300, 16
    r = _cube(n_chan, n_pix, 5, sigma=0.1)
    r[150, 8, 9] = np.inf
    x = torch.from_numpy(r).to(DEV)
    for cubes in (False, True):
        rec, thr, k, _, _ = nb.nbsi_search(x, fdr_q=0.01, want_cubes=cubes)
        # the windows of 100 channels that hold channel 150 stand at channels 101 .. 200; of equal
        # SNRs the lowest channel survives
        assert thr == np.inf and k == 100
        assert rec[["x", "y", "c", "width"]].tolist() == [(9, 8, 101, 100)] and rec["snr"][0] == np.inf


@pytest.mark.parametrize("n_chan,n_pix", [(150, 16), (640, 40)])
def test_search_suppression_of_dense_detections(n_chan, n_pix):
    """Nearly every voxel a provisional detection: waves of a few detections and of 64, the last wave
    not full; the records against the oracle's suppression of the same SNRs and widths."""
    print(f"search dense n_chan={n_chan} n_pix={n_pix}", flush=True)
    r = _cube(n_chan, n_pix, n_chan)
    rec, thr, k, S, W = nb.nbsi_search(torch.from_numpy(r).to(DEV), fdr_q=0.6, want_cubes=True)
    assert k > (500000 if n_chan > 600 else 20000)
    Sg, Wg = (v.cpu().numpy().reshape(n_chan, -1).astype(t) for v, t in ((S, np.float64), (W, np.int32)))
    exp = _expected_records(r, Sg, Wg, thr, n_pix)
    got = {(int(a["x"]), int(a["y"]), int(a["c"])): int(a["width"]) for a in rec}
    assert len(got) == len(rec) and set(got) <= set(exp)
    for (x, y, c), snr2 in exp.items():
        if abs(snr2 - thr) < 1e-4 * max(1.0, thr):
            continue  # a float32 re-evaluation may fall on either side of the threshold
        assert ((x, y, c) in got) == (snr2 >= thr)
        assert (x, y, c) not in got or got[(x, y, c)] == Wg[c, y * n_pix + x]


def test_stage2_captured_beside_eager():
    """A captured nbsi_stage2 of 2^22 voxels keeps one sequence: every replay, with eager calls (which
    take the two-stream form) and new inputs in between, equals the eager records."""
    g = torch.Generator(device="cpu").manual_seed(3)
    n_chan, n_pix = 1024, 64
    cubes = [torch.randn((n_chan, n_pix, n_pix), generator=g).to(DEV) for _ in range(2)]
    for q, cube in enumerate(cubes):
        cube[5 + q] *= 9.0
    cands = torch.tensor([[10 + 3 * i, 12 + 2 * i, 5 * i + 5, 1, 0] for i in range(16)] + [[1, 1, 6, 1, 0]],
                         dtype=torch.int32, device=DEV)
    beam = torch.tensor([[2.8, 2.8, 0.0]], dtype=torch.float64, device=DEV).repeat(n_chan, 1)
    want = [nb.fits_host(nb.nbsi_stage2(cube, cands, beam), len(cands)).tobytes() for cube in cubes]
    x, out = cubes[0].clone(), torch.zeros((len(cands), 160), dtype=torch.uint8, device=DEV)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        nb.nbsi_stage2(x, cands, beam, out=out)  # scratch is made before the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        nb.nbsi_stage2(x, cands, beam, out=out)
    for q in (0, 1, 0, 1):
        x.copy_(cubes[q])
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert nb.fits_host(out, len(cands)).tobytes() == want[q]
        assert nb.fits_host(nb.nbsi_stage2(cubes[1 - q], cands, beam), len(cands)).tobytes() == want[1 - q]


@pytest.mark.parametrize("n_pix", [8, 64, 128, 136, 256, 264])
def test_image_statistics_every_image_observed(n_pix):
    """Medians and MADs of images that are hard to select from, through the per-image SNRs of every
    searched pixel: ties, ramps, outliers, a range wider than the largest float, subnormal values,
    NaN and infinite pixels, and no finite pixel where the samples are taken."""
    print(f"image statistics observed n_pix={n_pix}", flush=True)
    rng = np.random.default_rng(100 + n_pix)
    n_chan, h = 13, n_pix // 2
    cube = rng.standard_normal((n_chan, n_pix, n_pix)).astype(np.float32)
    cube[1] = rng.integers(-2, 3, (n_pix, n_pix))
    cube[2] = 7.5
    cube[3] = np.arange(n_pix * n_pix, dtype=np.float32).reshape(n_pix, n_pix)
    cube[4] = -cube[3].T
    with np.errstate(over="ignore"):
        cube[5] *= np.float32(1e38)
    cube[6] *= np.float32(1e-41)
    cube[7, ::3, ::2] = 1e30
    cube[8, rng.random((n_pix, n_pix)) < 0.4] = np.nan
    cube[9, ::4] = np.inf
    cube[10] = np.exp(4.0 * cube[10])
    cube[11, h:h + 2] = np.nan
    _, snr, _ = nb.nbsi_detect(torch.from_numpy(cube).to(DEV), mode=nb.NBSI_DETECT_PER_IMAGE, want_snr=True)
    ref, valid = oracle.detect.snr_cube(cube, "per_image")
    got = snr.cpu().numpy().astype(np.float64)
    assert valid.sum() > n_pix * n_pix // 8 and np.all(got[:, ~valid] == 0.0)
    mask = oracle.detect.horizon_mask(n_pix)
    z = ref[:, valid]
    tol = np.zeros_like(z)
    for c in range(n_chan):
        v = cube[c][mask].astype(np.float64)
        v = v[np.isfinite(v)]
        med = np.median(v)
        sigma = 1.482602218505602 * np.median(np.abs(v - med))
        assert (sigma > 0) == (c != 2)  # only the constant image has none
        # float32 roundings of x - med, of the MAD and of the quotient, each relative to the values
        # they are formed from; subnormal values are rounded to their spacing
        x = np.abs(cube[c][valid].astype(np.float64))
        unit = (2.0 ** -24 * (x + abs(med)) + 2.0 ** -149) / sigma if sigma > 0 else 0.0
        tol[c] = 8.0 * (unit + 2.0 ** -24) * (1.0 + np.abs(z[c]))
    # the pixel's median over the channels moves by no more than the values next to it
    tol += np.where(np.abs(z) < 0.01, tol, 0.0).max(axis=0)
    d = np.abs(got[:, valid] - z)
    assert np.all(d <= tol), np.unravel_index(np.argmax(d - tol), d.shape)


@pytest.mark.parametrize("n_sub,n_chan,max_drift", [(1, 5, 16), (4, 5, 16), (4, 40, 16), (4, 40, 3), (1, 33, 2)])
def test_dedoppler_nonfinite_and_band_ends(n_sub, n_chan, max_drift):
    """Tracks that leave the band never win, also beside infinite and NaN values: results bit for bit
    those of the trials in order (1 / sqrt(n_sub) is exact here)."""
    print(f"dedoppler non-finite S={n_sub} C={n_chan} D={max_drift}", flush=True)
    rng = np.random.default_rng(n_sub * 1000 + n_chan)
    r = rng.standard_normal((n_sub, n_chan, 8, 8)).astype(np.float32)
    for v in (np.inf, -np.inf, np.nan, -3e38, 3e38):
        r[rng.integers(0, n_sub, 12), rng.integers(0, n_chan, 12), rng.integers(0, 8, 12), rng.integers(0, 8, 12)] = v
    r[:, :, 3, 3] = -np.inf
    r[:, :, 3, 4] = np.nan
    best, drift = nb.nbsi_dedoppler(torch.from_numpy(r).to(DEV), max_drift)
    want = np.full(r.shape[1:], -np.inf, np.float32)
    at = np.zeros(want.shape, np.int8)
    with np.errstate(invalid="ignore", over="ignore"):
        for k in range(2 * max_drift + 1):
            d = -((k + 1) // 2) if k & 1 else k // 2
            for c in range(max(0, -d), min(n_chan, n_chan - d)):
                acc = np.zeros((8, 8), np.float32)
                for s in range(n_sub):
                    acc = acc + r[s, c + odr.shift(d, s, n_sub)]
                v = acc * np.float32(1.0 / np.sqrt(n_sub))
                up = v > want[c]
                want[c][up], at[c][up] = v[up], d
    assert np.array_equal(best.cpu().numpy(), want) and np.array_equal(drift.cpu().numpy(), at)


@pytest.mark.parametrize("mode", [nb.NBSI_DETECT_PER_PIXEL, nb.NBSI_DETECT_PER_IMAGE])
@pytest.mark.parametrize("n_chan,n_pix", [(3, 8), (10, 16), (11, 256), (2500, 32), (3, 264), (7, 512)])
def test_detect_snr_cube_with_and_without_scratch(n_chan, n_pix, mode):
    """The SNR cube from medians and scales in scratch (nbsi_detect), in the fixed workspace or, beyond
    256 x 256 pixels, in its own first planes (nbsi_detect_noalloc): the same values, also after more
    candidates than the scratch held."""
    print(f"detect SNR cube n_chan={n_chan} n_pix={n_pix} mode={mode}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(n_chan)
    cube = torch.randn((n_chan, n_pix, n_pix), generator=g, device=DEV)
    cube[n_chan // 2, n_pix // 2, n_pix // 2] += 40.0
    buf = torch.full_like(cube, float("nan"))
    rec, _, n = nb.nbsi_detect_noalloc(cube, mode=mode, snr=buf)
    rec2, snr, n2 = nb.nbsi_detect(cube, mode=mode, want_snr=True)
    assert n == n2 and np.array_equal(rec, rec2) and torch.equal(buf, snr)
    if n_chan == 2500:  # every local maximum above zero: a second pass with a longer list
        rec3, snr3, n3 = nb.nbsi_detect(cube, mode=mode, thresh=0.0, want_snr=True)
        assert n3 > 1 << 18 and len(rec3) == n3 and torch.equal(snr3, snr)
        rec4, snr4, _ = nb.nbsi_detect(cube, mode=mode, want_snr=True)
        assert np.array_equal(rec4, rec) and torch.equal(snr4, snr)


@pytest.mark.parametrize("n_chan", [1500, 2100])
def test_search_default_bank_marches(n_chan):
    """Workgroups that march over three and five 128-channel blocks, the last ones ragged, and passes of
    more than one tile per wave (256 x 256 pixels): sampled spectra against the oracle, and the whole
    cubes bit for bit those of the general kernel, which takes any other list of widths, wherever the
    width added to the list does not win; with the width cube, without it, and without either cube."""
    print(f"search default bank marches n_chan={n_chan}", flush=True)
    n_pix = 256
    g = torch.Generator(device="cuda")
    g.manual_seed(n_chan)
    x = torch.randn((n_chan, n_pix, n_pix), generator=g, device=DEV)
    rng = np.random.default_rng(n_chan)
    for c0, w in ((100, 40), (120, 20), (250, 12), (383, 3), (500, 100), (n_chan - 30, 30), (0, 5), (1279, 2)):
        px, py = rng.integers(70, 180, 2)
        x[c0:c0 + w, py, px] += 20.0 / w ** 0.5
    x[700, 128, 130], x[300, 127, 131], x[n_chan - 1, 126, 132], x[2, 125, 133] = np.inf, np.nan, -np.inf, np.inf
    rec, thr, k, S, W = nb.nbsi_search(x, want_cubes=True)
    rec2, thr2, k2, _, _ = nb.nbsi_search(x)
    assert (thr, k) == (thr2, k2) and np.array_equal(rec, rec2) and len(rec) >= 8
    only = torch.empty_like(S)  # best SNRs without the widths, through the C entry point
    ctx = nb.nbsi_create(0)
    ctx._sync_stream()
    n_out, out = ctypes.c_int(), torch.empty((4096, 5), dtype=torch.int32, device=DEV)
    assert nb.lib().nbsi_search_corr(ctx._h, x.data_ptr(), n_chan, n_pix, None, 0, None, 0, 0.01, only.data_ptr(), None,
                                     out.data_ptr(), 4096, ctypes.byref(n_out), None, None) == 0
    assert n_out.value == len(rec) and torch.equal(only, S)
    _, _, _, Sg, Wg = nb.nbsi_search(x, widths=list(osr.WIDTHS) + [127], want_cubes=True)
    same = Wg != 127
    assert torch.equal(S[same], Sg[same]) and torch.equal(W[same], Wg[same]) and bool((S <= Sg).all())
    assert float(same.float().mean()) > 0.9
    pix = rng.integers(0, n_pix * n_pix, 24)
    pix = torch.from_numpy(pix[(pix // n_pix < 120) | (pix // n_pix > 132)]).to(DEV)  # (finite spectra)
    spectra = x.view(n_chan, -1)[:, pix].cpu().numpy()
    _check_bank(spectra, S.view(n_chan, -1)[:, pix], W.view(n_chan, -1)[:, pix])
