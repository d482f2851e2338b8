"""Edges of the kernels' tiles, remainders and dispatch rules, against numpy or the oracle."""
import ctypes

import numpy as np
import pytest
import torch

import tfsc_inputs as ti
from gpu_common import dev, gridspec, lib, note, small_data, store_from_oracle
from oracle import transform as otf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, n_tiles", [(1, 1), (2047, 64), (2049, 1), (70_001, 4096), (70_001, 4097), (40_000, 12_000)])
@pytest.mark.parametrize("kind", ["mixed", "equal"])
def test_tile_max_at_block_and_table_edges(n, n_tiles, kind):
    """One batch more or less than a block takes, tables of 4096 tiles in LDS and of 4097 in memory, more tiles than
    a block has templates; values with infinities and ties, or all equal (every template attains its maximum)."""
    tfsc = lib()
    rng = np.random.default_rng(n + n_tiles)
    note(f"tile max: {n} values, {n_tiles} tiles, {kind}")
    stat = np.zeros(n) if kind == "equal" else np.round(rng.exponential(30.0, n), 1)
    if kind == "mixed" and n > 8:
        stat[rng.integers(0, n, 4)] = np.inf
        stat[rng.integers(0, n, 4)] = np.nan
    tile = rng.integers(-1, n_tiles, n).astype(np.int32)
    mx, arg = (t.cpu().numpy() for t in tfsc.tile_max(dev(stat), dev(tile), n_tiles))
    ok = (tile >= 0) & (stat >= 0.0)
    rmx = np.zeros(n_tiles)
    np.maximum.at(rmx, tile[ok], stat[ok])
    rarg = np.full(n_tiles, n, np.int64)
    at = np.flatnonzero(ok & (stat == rmx[np.maximum(tile, 0)]))
    np.minimum.at(rarg, tile[at], at)
    rarg[rarg == n] = -1
    assert np.array_equal(mx, rmx) and np.array_equal(arg, rarg)


@pytest.mark.parametrize("n, n_tiles", [(63, 1), (3071, 64), (3072, 64), (52_223, 1024), (52_224, 1024), (131_071, 64),
                                        (131_072, 64), (3_350_527, 8192), (3_350_528, 8192), (500_000, 8193)])
@pytest.mark.parametrize("order", ["any", "tiles", "runs"])
def test_tile_max_where_its_rule_changes(n, n_tiles, order):
    """One template more or less than from which a block keeps its maxima in LDS, or takes more at a time, and the
    largest table; templates in any order, in the tiles' order, and in runs of 64 with some of them left out (a wave
    with a single tile sends one maximum)."""
    tfsc = lib()
    rng = np.random.default_rng(n + n_tiles)
    note(f"tile max rule: {n} values, {n_tiles} tiles, {order}")
    stat = np.round(rng.exponential(30.0, n), 2)
    stat[rng.integers(0, n, n // 50)] = -1.0
    tile = rng.integers(0, n_tiles, n).astype(np.int32)
    if order == "tiles":
        tile.sort()
    if order == "runs":
        tile = np.repeat(tile[: (n + 63) // 64], 64)[:n].copy()
        tile[rng.integers(0, n, n // 3)] = -1
    mx, arg = (t.cpu().numpy() for t in tfsc.tile_max(dev(stat), dev(tile), n_tiles))
    ok = (tile >= 0) & (stat >= 0.0)
    rmx = np.zeros(n_tiles)
    np.maximum.at(rmx, tile[ok], stat[ok])
    rarg = np.full(n_tiles, n, np.int64)
    at = np.flatnonzero(ok & (stat == rmx[np.maximum(tile, 0)]))
    np.minimum.at(rarg, tile[at], at)
    rarg[rarg == n] = -1
    assert np.array_equal(mx, rmx) and np.array_equal(arg, rarg)


def _planes(store):
    """The store's pixels as complex128 [C][K][Nt]."""
    z = torch.view_as_complex(store.pix.to(torch.float64).contiguous())
    z = {"layer": lambda v: v, "tranche": lambda v: v.transpose(1, 2), "layer_ci": lambda v: v.permute(2, 0, 1)}[store.layout](z)
    if store.layer_scale is not None:
        z = z * store.layer_scale.to(torch.float64)[:, :, None]
    return z.cpu().numpy()


@pytest.mark.parametrize("C, M, Nt", [(1, 64, 1), (2, 64, 257), (3, 128, 66), (2, 256, 63), (1, 512, 33), (3, 512, 17),
                                      (2, 1024, 9), (1, 2048, 5), (2, 2048, 4), (2, 2048, 33), (3, 2048, 3), (2, 4096, 5)])
@pytest.mark.parametrize("layout", ["layer", "tranche", "layer_ci"])
def test_transform_at_tile_edges(C, M, Nt, layout):
    """Every transform length (one to four exchanges, a remainder of none, one or two stages), tranche counts of one
    tile more or less, every layout and channel count; white noise and a smooth PSD, so every pixel is of order 1.

    Bounds, relative to the largest pixel: an FFT's error is below log2(M) roundings of each butterfly's operations (6,
    at most 12 * 6 * u), u = 1.1e-16 in FP64 and 6e-8 in FP32 (M = 4096), plus one rounding of the stored value; the
    16-bit grid adds half a step of 1/32767 of its layer's maximum."""
    tfsc = lib()
    g = ti.custom_grid(C, M, Nt, dt=5.0, modulated=False, gapped=False, cfg_id=11)
    rng = np.random.default_rng(M + Nt)
    x = rng.standard_normal((C, M * Nt))
    K = M // 2 + 1
    psd, mu = 1.0 + 0.5 * np.cos(np.arange(K) / K), 1.0 + 0.2 * rng.random(Nt)
    keep = (rng.random(Nt) > 0.2).astype(np.uint8)
    keep[-1] = 1
    note(f"transform edges C={C} M={M} Nt={Nt} {layout}")
    x32 = x.astype(np.float32)
    for dtype, xx in (("f64", x), ("f32", x32), ("f32", x), ("i16", x32)):
        if M == 4096 and dtype == "f64":
            continue
        st = tfsc.transform(gridspec(g), dev(xx), dev(psd), dev(mu), dev(keep), dtype=dtype, layout=layout)
        ref, u, wm = otf.transform(xx.astype(np.float64), g, psd, mu, keep, 0.1, "rfft")
        d = np.abs(_planes(st) - ref)
        unit = 6e-8 if M == 4096 else 1.1e-16
        bound = 72 * unit * np.abs(ref).max() + (0.0 if dtype == "f64" else 1.2e-7 * np.abs(ref).max())
        if dtype == "i16":
            bound = bound + 0.75 * np.maximum(np.abs(ref.real), np.abs(ref.imag)).max(axis=2, keepdims=True) / 32767.0
        assert np.all(d <= bound), (dtype, float((d - bound).max()))
        assert np.all(_planes(st)[:, :, keep == 0] == 0)


def test_transform_into_a_store_off_16_bytes():
    """An FP32 A+E store that starts 8 bytes off a 16-byte boundary holds the same bits as an aligned one."""
    tfsc = lib()
    g = ti.custom_grid(2, 256, 45, dt=5.0, modulated=False, gapped=False, cfg_id=11)
    x = dev(np.random.default_rng(5).standard_normal((2, 256 * 45)).astype(np.float32))
    args = (dev(np.ones(129)), dev(np.ones(45)), dev(np.ones(45, np.uint8)))
    note("transform into an unaligned store")
    a = tfsc.transform(gridspec(g), x, *args, dtype="f32", layout="layer_ci")
    flat = torch.zeros(a.pix.numel() + 2, dtype=torch.float32, device="cuda")
    b = tfsc.PixelStore(flat[2:].view_as(a.pix), torch.empty_like(a.inv_asd), torch.empty_like(a.tranche_w), "f32", "layer_ci")
    tfsc.transform(gridspec(g), x, *args, dtype="f32", layout="layer_ci", out=b)
    assert torch.equal(a.pix, b.pix) and float(flat[:2].abs().max()) == 0.0


@pytest.mark.parametrize("C, M, Nt", [(2, 64, 33_000), (3, 128, 22_001), (1, 512, 66_000)])
@pytest.mark.parametrize("layout", ["tranche", "layer"])
def test_sixteen_bit_store_of_many_tranches(C, M, Nt, layout):
    """More than 65,536 tranche-major rows (shorter and longer than a block of the quantisation): the 16-bit store holds
    the nearest integer to each FP32 pixel over its layer's scale, which is the layer's largest FP32 component over
    32767.  The division by the scale is a multiplication there: at most one step apart where it rounds."""
    tfsc = lib()
    grid = tfsc.GridSpec(C, M, Nt, 5.0, 0.1)
    gen = torch.Generator(device="cuda").manual_seed(C)
    x = torch.randn((C, M * Nt), generator=gen, device="cuda")
    args = (dev(np.ones(M // 2 + 1)), dev(np.ones(Nt)), dev(np.ones(Nt, np.uint8)))
    note(f"16-bit store C={C} M={M} Nt={Nt} {layout}")
    a = tfsc.transform(grid, x, *args, dtype="f32", layout=layout)
    b = tfsc.transform(grid, x, *args, dtype="i16", layout=layout)
    p = (a.pix if layout == "layer" else a.pix.transpose(1, 2)).double()  # [C][K][Nt][2]
    q = (b.pix if layout == "layer" else b.pix.transpose(1, 2)).double()
    top = p.abs().amax(dim=(2, 3))
    assert float((b.layer_scale.double() * 32767.0 / top - 1.0).abs().max()) < 2.0 ** -23
    want = p * (32767.0 / top)[:, :, None, None]
    # half a step, and the float rounding of the factor and of the product (2^-24 each of at most 32767)
    assert float((q - want).abs().max()) <= 0.5 + 2.0 * 32767.0 * 2.0 ** -24


@pytest.mark.parametrize("C, M, Nt", [(1, 64, 1), (2, 128, 3), (2, 2048, 1), (1, 4096, 3)])
@pytest.mark.parametrize("layout", ["layer_ci", "tranche"])
def test_layer_scale_is_the_maximum_of_stored_pixels(C, M, Nt, layout):
    """An odd number of tranches of a sinusoid on a bin: in most layers all pixels are of rounding size, and the scale of
    the 16-bit store is the largest of them, exactly (the FP32 store holds the same FP32 values; the maximum divided by
    32767 is one rounding); where all of them are zero it is 1."""
    tfsc = lib()
    grid = tfsc.GridSpec(C, M, Nt, 5.0, 0.0)
    note(f"layer scale C={C} M={M} Nt={Nt} {layout}")
    x = dev(np.tile(np.cos(2.0 * np.pi * (M // 8) * np.arange(M) / M + 0.3), (C, Nt)).astype(np.float32))
    args = (dev(np.ones(M // 2 + 1)), dev(np.ones(Nt)), dev(np.ones(Nt, np.uint8)))
    p = tfsc.transform(grid, x, *args, dtype="f32", layout=layout).pix
    top = {"layer_ci": lambda v: v.abs().amax(dim=(1, 3)).T, "tranche": lambda v: v.abs().amax(dim=(1, 3))}[layout](p)
    got = tfsc.transform(grid, x, *args, dtype="i16", layout=layout).layer_scale
    top = top.cpu().numpy()  # numpy's division is correctly rounded; torch divides by a number with its reciprocal
    assert np.array_equal(got.cpu().numpy(), np.where(top > 0, top / np.float32(32767.0), np.float32(1.0)))


@pytest.mark.parametrize("C, M, Nt, dtype, layout", [
    (2, 2048, 515, "f32", "layer_ci"), (2, 64, 16_453, "f64", "layer_ci"), (2, 256, 4_117, "i16", "layer_ci"),
    (2, 4096, 259, "f32", "layer_ci"), (3, 2048, 685, "f64", "layer_ci"), (3, 64, 21_895, "i16", "layer_ci"),
    (1, 512, 8_205, "i16", "layer"), (2, 1024, 2_053, "i16", "tranche"), (1, 2048, 2_055, "i16", "layer_ci")])
def test_transform_of_many_tranches_equals_its_pieces(C, M, Nt, dtype, layout):
    """Sets just above the sizes from which a block does several transforms, with a remainder, against the same tranches
    in pieces below them (an even number, so that the same tranches are paired): the same bits.  A 16-bit store's scale is
    the largest component over its grid, its pixels within half a step and two float roundings of at most 32767."""
    tfsc = lib()
    note(f"transform of many tranches C={C} M={M} Nt={Nt} {dtype} {layout}")
    f = "f32" if dtype == "i16" else dtype
    gen = torch.Generator(device="cuda").manual_seed(M)
    x = torch.randn((C, Nt, M), generator=gen, device="cuda", dtype=torch.float64 if dtype == "f64" else torch.float32)

    def run(a, b, d):
        n = b - a
        return tfsc.transform(tfsc.GridSpec(C, M, n, 5.0, 0.1), x[:, a:b].contiguous(), dev(np.ones(M // 2 + 1)),
                              dev(np.ones(n)), dev(np.ones(n, np.uint8)), dtype=d, layout=layout)

    at = {"layer": 2, "tranche": 1, "layer_ci": 1}[layout]
    step = 2 * (2048 // M or 1) * 20
    want = torch.cat([run(a, min(a + step, Nt), f).pix for a in range(0, Nt, step)], dim=at)
    assert torch.equal(run(0, Nt, f).pix, want)
    if dtype == "i16":
        got = run(0, Nt, "i16")
        over = {"layer": (2, 3), "tranche": (1, 3), "layer_ci": (1, 3)}[layout]
        top = want.abs().amax(dim=over)
        scale = (top.T if layout == "layer_ci" else top).cpu().numpy() / np.float32(32767.0)
        assert np.array_equal(got.layer_scale.cpu().numpy(), scale)
        top = {"layer": lambda v: v[:, :, None, None], "tranche": lambda v: v[:, None, :, None],
               "layer_ci": lambda v: v[:, None, :, None]}[layout](top.double())
        assert float((got.pix.double() - want.double() * (32767.0 / top)).abs().max()) <= 0.5 + 2.0 * 32767.0 * 2.0 ** -24


def _bank(tfsc, n, seed):
    b = ti.random_bank(n, seed, mc_range=(5.0, 100.0), f0_range=(0.004, 0.08), eta=None, stream=62)
    if n > 20:
        b.mc[3], b.eta[5], b.f0[7], b.cos_iota[9] = -2.0, 0.3, 0.2, 1.0  # invalid, invalid, empty track, face-on
    return tfsc.BankTensors.from_host(b)


def _all_equal(a, b):
    for k in ("stat", "seg_terms", "seg_zn", "flags", "n_active"):
        x, y = getattr(a, k), getattr(b, k)
        assert torch.equal(x, y), (k, int((x != y).sum()))


@pytest.mark.parametrize("nseg", [0, 1, 7, 8, 1000])
@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_split_templates_equal_whole_ones(precision, nseg):
    """Chunks shared out over the waves (a workspace with room for it) against whole templates (the static scratch
    has none for this bank), bit for bit: segments inside a unit, across units, shorter than a tranche, tracks that
    end in every part of the grid, invalid and empty templates, excluded tranches."""
    tfsc = lib()
    d = small_data()
    g = gridspec(d["grid"])
    store = store_from_oracle(d, precision, "layer_ci")
    for n in (5000, 1):
        bank = _bank(tfsc, n, 13)
        seg = tfsc.segment_layout(g, bank, nseg)
        order = tfsc.processing_order(g, bank)
        note(f"split against whole templates: {precision} nseg={nseg} n={n}")
        for o in (order, None):
            a = tfsc.bank_statistic(g, store, bank, seg, precision=precision, want_zn=True, want_active=True, order=o)
            b = tfsc.bank_statistic_noalloc(g, store, bank, seg, precision=precision, want_zn=True, want_active=True,
                                            order=o)
            _all_equal(a, b)
        if n == 5000:  # fewer than a run per XCD: the first templates of this bank by themselves, their terms in the same places
            few = tfsc.BankTensors(*(getattr(bank, k)[:300].contiguous() for k in tfsc.BankTensors.FIELDS))
            fs = tfsc.segment_layout(g, few, nseg)
            c = tfsc.bank_statistic(g, store, few, fs, precision=precision, want_zn=True, want_active=True)
            for k in ("stat", "flags", "n_active"):
                assert torch.equal(getattr(c, k), getattr(a, k)[:300]), k
            assert torch.equal(c.seg_terms, a.seg_terms[: fs.total]) and torch.equal(c.seg_zn, a.seg_zn[: fs.total])


@pytest.mark.parametrize("block_waves", [1, 3, 4])
def test_runs_of_the_processing_order_equal_the_counter(block_waves):
    """A bank too large to split: one wave per template in runs per XCD (with a processing order) against the work
    counter (without), bit for bit, with an order whose last entries are out of range (those templates are left out)."""
    tfsc = lib()
    g = ti.custom_grid(2, 64, 130, dt=5.0, modulated=False, gapped=False, cfg_id=11)
    rng = np.random.default_rng(3)
    z = rng.standard_normal((2, 33, 130)) + 1j * rng.standard_normal((2, 33, 130))
    store = tfsc.PixelStore.from_complex(dev(z), dev(np.ones(33)), dev(np.ones(130)), "f32", "layer_ci")
    grid = gridspec(g)
    bank = _bank(tfsc, 100_003, 17)
    seg = tfsc.segment_layout(grid, bank)
    order = tfsc.processing_order(grid, bank)
    note(f"runs against the counter: block_waves={block_waves}")
    kw = dict(precision="f32", want_zn=True, want_active=True, block_waves=block_waves)
    a = tfsc.bank_statistic(grid, store, bank, seg, order=order, **kw)
    b = tfsc.bank_statistic(grid, store, bank, seg, **kw)
    _all_equal(a, b)
    left = order[-2:].long()
    short = order.clone()
    short[-2:] = torch.tensor([-1, 100_003], dtype=torch.int32, device="cuda")
    a.stat[left] = -1.0
    tfsc.bank_statistic(grid, store, bank, seg, order=short, out=a, **kw)
    b.stat[left] = -1.0
    assert torch.equal(a.stat, b.stat)


@pytest.mark.parametrize("C, layout, dtype", [(1, "layer", "f32"), (2, "layer_ci", "f32"), (3, "tranche", "f64")])
@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_vjp_units_equal_whole_templates(C, layout, dtype, precision):
    """The VJP with a template's chunks shared out (5003 templates) against whole templates (the same ones in a bank of
    90,000, which is not split): equal but for the order of the FP64 sum over the tranches, at most 130 terms of at most
    1e3 times the largest gradient, so below 130 * 1.1e-16 * 1e3 = 1.5e-11 of it; 1e-9 is asked for."""
    tfsc = lib()
    M, Nt = 64, 130
    g = ti.custom_grid(C, M, Nt, dt=5.0, modulated=False, gapped=False, cfg_id=11)
    grid = gridspec(g)
    rng = np.random.default_rng(5)
    z = rng.standard_normal((C, M // 2 + 1, Nt)) + 1j * rng.standard_normal((C, M // 2 + 1, Nt))
    wm = np.where(rng.random(Nt) > 0.1, 1.0, 0.0)
    store = tfsc.PixelStore.from_complex(dev(z), dev(np.ones(M // 2 + 1)), dev(wm), dtype, layout)
    big = _bank(tfsc, 90_003, 19)
    few = tfsc.BankTensors(*(getattr(big, k)[:5003].contiguous() for k in tfsc.BankTensors.FIELDS))
    note(f"VJP units against whole templates: C={C} {layout} {dtype} {precision}")
    out = []
    for bank in (big, few):
        seg = tfsc.segment_layout(grid, bank, 3)
        zn = torch.as_tensor(np.random.default_rng(6).standard_normal((90_003 * 3, 3)), device="cuda")[: 3 * bank.n].abs()
        out.append(tfsc.statistic_vjp(grid, store, bank, seg, zn.contiguous(),
                                      g_stat=torch.ones(bank.n, dtype=torch.float64, device="cuda"), precision=precision))
    a, b = out[0][:5003], out[1]
    assert torch.isfinite(b).all()
    assert float(((a - b).abs() / a.abs().amax(dim=0)).max()) < 1e-9


def _noise_store(tfsc, grid, C, M, Nt, dtype, layout, rho, gen):
    """Unit-variance noise pixels, a tenth of the tranches excluded; a 16-bit store through the transform."""
    K = M // 2 + 1
    w = (torch.rand(Nt, generator=gen, device="cuda") > 0.1).to(torch.float64)
    if dtype == "i16":
        x = torch.randn((C, M * Nt), generator=gen, device="cuda")
        store = tfsc.transform(grid, x, dev(np.ones(K)), dev(np.ones(Nt)), w.to(torch.uint8), dtype="i16", layout=layout)
    else:
        z = torch.view_as_complex(torch.randn((C, K, Nt, 2), generator=gen, device="cuda"))
        store = tfsc.PixelStore.from_complex(z, dev(np.ones(K)), w, dtype, layout)
    if rho:
        store.rho = 0.5 + torch.rand((K, Nt), generator=gen, device="cuda")
    return store


def _whole(tfsc, grid, n, precision):
    """A workspace without the scratch of split templates."""
    g, opt = grid.c(), tfsc._options(precision)
    nb = tfsc.lib().tfsc_workspace_bytes(ctypes.byref(g), n, ctypes.byref(opt), tfsc._lib.WS_WHOLE)
    return torch.empty(nb, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("C, layout, dtype, precision, rho", [
    (2, "layer_ci", "f32", "f32", False), (2, "layer_ci", "f32", "f32", True), (2, "layer_ci", "i16", "f32", False),
    (1, "layer", "f32", "f32", False), (3, "layer_ci", "f32", "f32", False), (3, "layer", "i16", "f32", False),
    (2, "layer", "f64", "f64", True), (1, "layer_ci", "f32", "f64", False)])
@pytest.mark.parametrize("n, nseg", [(1, 7), (300, 0), (2000, 3), (6000, 40), (20_000, 0)])
def test_units_of_several_chunks_equal_whole_templates(C, layout, dtype, precision, rho, n, nseg):
    """35 chunks of tranches in units of 1, 2, 6 and 16 (on 256 CUs; the last unit is shorter) against whole templates,
    bit for bit: segments inside a unit, over several units and their chunks, tracks that end in any of them."""
    tfsc = lib()
    M, Nt = 64, 2200
    grid = tfsc.GridSpec(C, M, Nt, 5.0, 0.1)
    store = _noise_store(tfsc, grid, C, M, Nt, dtype, layout, rho, torch.Generator(device="cuda").manual_seed(n + C))
    bank = _bank(tfsc, n, 31)
    seg = tfsc.segment_layout(grid, bank, nseg)
    note(f"units of several chunks: C={C} {layout} {dtype}/{precision} rho={rho} n={n} nseg={nseg}")
    kw = dict(precision=precision, want_zn=True, want_active=True)
    a = tfsc.bank_statistic(grid, store, bank, seg, ws=_whole(tfsc, grid, n, precision), **kw)
    for order in (None, tfsc.processing_order(grid, bank)):
        _all_equal(tfsc.bank_statistic(grid, store, bank, seg, order=order, **kw), a)


@pytest.mark.parametrize("C, layout, dtype, rho", [(2, "layer_ci", "f32", False), (3, "tranche", "i16", False),
                                                   (1, "layer", "f64", True)])
@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("n", [1, 30, 1500])
def test_vjp_units_of_several_chunks_equal_whole_templates(C, layout, dtype, rho, precision, n):
    """The VJP in units of 1 and of 3 (FP32) and 6 (FP64) of the 35 chunks against whole templates: equal but for the order of the
    FP64 sum over the tranches, at most 2200 terms of at most 1e3 times the largest gradient, so below
    2200 * 1.1e-16 * 1e3 = 2.4e-10 of it; 1e-9 is asked for."""
    tfsc = lib()
    M, Nt = 64, 2200
    grid = tfsc.GridSpec(C, M, Nt, 5.0, 0.1)
    store = _noise_store(tfsc, grid, C, M, Nt, dtype, layout, rho, torch.Generator(device="cuda").manual_seed(n + C))
    bank = _bank(tfsc, n, 37)
    seg = tfsc.segment_layout(grid, bank, 5)
    zn = torch.rand((5 * n, 3), generator=torch.Generator(device="cuda").manual_seed(3), device="cuda", dtype=torch.float64)
    note(f"VJP units of several chunks: C={C} {layout} {dtype} rho={rho} {precision} n={n}")
    ones = torch.ones(n, dtype=torch.float64, device="cuda")
    b = tfsc.statistic_vjp(grid, store, bank, seg, zn, g_stat=ones, precision=precision)
    a, ws = torch.empty_like(b), _whole(tfsc, grid, n, precision)
    g, opt, pc, bc, sc = grid.c(), tfsc._options(precision), store.c(), bank.c(), seg.c()
    st = tfsc.lib().tfsc_statistic_vjp(ctypes.byref(g), ctypes.byref(pc), ctypes.byref(bc), ctypes.byref(sc),
                                       ctypes.byref(opt), zn.data_ptr(), ones.data_ptr(), None, a.data_ptr(),
                                       ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert st == 0 and torch.isfinite(b).all()
    assert ((a - b).abs() <= 1e-9 * a.abs().amax(dim=0)).all()


@pytest.mark.parametrize("n, n_real, C", [(1, 2, 1), (515, 2, 2), (2049, 4, 1)])
def test_interleaved_runs_equal_the_counter(n, n_real, C):
    """Realisations cell by cell: runs of the processing order per XCD against the work counter, bit for bit."""
    tfsc = lib()
    g = ti.custom_grid(C, 64, 130, dt=5.0, modulated=False, gapped=False, cfg_id=11)
    grid = gridspec(g)
    stores = []
    for r in range(n_real):
        rng = np.random.default_rng(r)
        z = rng.standard_normal((C, 33, 130)) + 1j * rng.standard_normal((C, 33, 130))
        stores.append(tfsc.PixelStore.from_complex(dev(z), dev(np.ones(33)), dev(np.ones(130)), "f32", "layer_ci"))
    ri = tfsc.interleave_stores(grid, stores)
    bank = _bank(tfsc, n, 23)
    seg = tfsc.segment_layout(grid, bank)
    note(f"interleaved runs against the counter: n={n} realisations={n_real} C={C}")
    a = tfsc.bank_statistic_interleaved(grid, ri, n_real, bank, seg, order=tfsc.processing_order(grid, bank), want_active=True)
    b = tfsc.bank_statistic_interleaved(grid, ri, n_real, bank, seg, want_active=True)
    for k in ("stat", "seg_terms", "flags", "n_active"):
        assert torch.equal(getattr(a, k), getattr(b, k)), k


@pytest.mark.parametrize("n", [1 << 25, (1 << 25) + 4096])
def test_largest_bank_in_runs_and_the_first_on_the_counter(n):
    """At the size where an ordered bank goes from one wave per template to the persistent grid (its grid would pass 2^32
    threads at twice that): a bank of repeated templates gives the small bank's values, bit for bit."""
    tfsc = lib()
    g = ti.custom_grid(1, 64, 66, dt=5.0, modulated=False, gapped=False, cfg_id=11)
    grid = gridspec(g)
    rng = np.random.default_rng(4)
    z = rng.standard_normal((1, 33, 66)) + 1j * rng.standard_normal((1, 33, 66))
    store = tfsc.PixelStore.from_complex(dev(z), dev(np.ones(33)), dev(np.ones(66)), "f32", "layer_ci")
    small = _bank(tfsc, 4096, 29)
    seg = tfsc.segment_layout(grid, small, nseg_fixed=1)
    want = tfsc.bank_statistic(grid, store, small, seg).stat
    bank = tfsc.BankTensors(**{f: getattr(small, f).repeat(n // 4096) for f in small.FIELDS})
    seg = tfsc.segment_layout(grid, bank, nseg_fixed=1)
    order = tfsc.processing_order(grid, bank)
    note(f"ordered bank of {n}")
    got = tfsc.bank_statistic(grid, store, bank, seg, order=order)
    assert torch.equal(got.stat.view(-1, 4096), want.expand(n // 4096, 4096))
    del got
    ri = tfsc.interleave_stores(grid, [store, store])
    got = tfsc.bank_statistic_interleaved(grid, ri, 2, bank, seg, order=order)
    want = tfsc.bank_statistic_interleaved(grid, ri, 2, small, tfsc.segment_layout(grid, small, nseg_fixed=1)).stat
    for r in range(2):
        assert torch.equal(got.stat[r].view(-1, 4096), want[r].expand(n // 4096, 4096)), r
