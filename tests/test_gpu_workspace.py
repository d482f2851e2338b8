"""A caller's workspace is the one that is used: with the optional scratch of split templates, or without it."""
import ctypes

import numpy as np
import pytest
import torch

import tfsc_inputs as ti
from gpu_common import dev, gridspec, lib, note

pytestmark = pytest.mark.gpu


def _count():
    torch.cuda.synchronize()
    return torch.cuda.memory_stats()["allocation.all.allocated"]


def _bytes(tfsc, grid, n, opt, which):
    g = grid.c()
    return tfsc.lib().tfsc_workspace_bytes(ctypes.byref(g), n, None if opt is None else ctypes.byref(opt), which)


def _inputs(tfsc, M, Nt, n, seed):
    g = ti.custom_grid(2, M, Nt, dt=5.0, modulated=False, gapped=False, cfg_id=11)
    K = M // 2 + 1
    rng = np.random.default_rng(seed)
    z = rng.standard_normal((2, K, Nt)) + 1j * rng.standard_normal((2, K, Nt))
    store = tfsc.PixelStore.from_complex(dev(z), dev(np.ones(K)), dev(np.ones(Nt)), "f32", "layer_ci")
    bank = tfsc.BankTensors.from_host(ti.random_bank(n, seed, mc_range=(5.0, 100.0), f0_range=(0.004, 0.08), stream=62))
    return gridspec(g), store, bank, tfsc.segment_layout(gridspec(g), bank, 1)


@pytest.mark.parametrize("which", ["WS_WHOLE", "WS_STATISTIC"])
def test_statistic_takes_the_workspace_it_is_given(which):
    tfsc = lib()
    grid, store, bank, seg = _inputs(tfsc, 64, 700, 300, 5)
    want = tfsc.bank_statistic(grid, store, bank, seg, want_zn=True)
    ws = torch.empty(_bytes(tfsc, grid, bank.n, tfsc._options("f32"), getattr(tfsc._lib, which)), dtype=torch.uint8, device="cuda")
    out = tfsc.StatResult(*(torch.zeros_like(t) for t in (want.stat, want.seg_terms, want.flags, want.seg_zn)))
    note(f"workspace of {ws.numel()} bytes ({which})")
    before = _count()
    tfsc.bank_statistic(grid, store, bank, seg, ws=ws, out=out)
    assert _count() == before
    for k in ("stat", "seg_terms", "flags", "seg_zn"):
        assert torch.equal(getattr(out, k), getattr(want, k)), k


@pytest.mark.parametrize("n, kw", [(60_000, {}), (300, {"multi": True}), (300, {"interleave": 2})])
def test_realisation_graph_allocates_its_workspace_once(n, kw):
    """60,000 templates of 6144 tranches: the scratch of split templates passes its 128 MiB in FP64 but not in FP32,
    which is what the calls run in.  The passes over several realisations never split."""
    tfsc = lib()
    from paper_2510_19047_amd import batching
    M, Nt = 64, 6144
    grid, _, bank, seg = _inputs(tfsc, M, Nt, n, 6)
    note(f"realisation graph: n={n} {kw}")
    x = torch.randn((2, 2, M * Nt), generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
    rg = batching.RealisationGraph(grid, x, dev(np.ones(M // 2 + 1)), dev(np.ones(Nt)), dev(np.ones(Nt, np.uint8)), bank,
                                   seg, **kw)
    which = tfsc._lib.WS_WHOLE if kw else tfsc._lib.WS_STATISTIC
    assert rg.ws.numel() == _bytes(tfsc, grid, n, tfsc._options("f32"), which)
    before = _count()
    rg.eager()
    assert _count() == before
