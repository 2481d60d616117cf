"""Row widths, strides and positions at which the kernels change their way of working, against
the CPU oracle: rows that start at any 2-byte position and are no multiple of 8 columns (the
row-band pass loads 8 elements at a time and shifts at the row's end), the first and last
widths of each number of 512-column chunks per wave, and widths outside the row-band pass on
both sides (below 8 columns, above 16384). Every tensor is a view of a wider buffer whose other
elements are NaN in the gradient, so that a value read past a row's end would show in the
results, and must keep their values in the weights."""
import pytest
import torch

import oracle
from paper_2607_19058_amd import workloads as W

from parity_util import ParityRun, bits, log

pytestmark = pytest.mark.gpu

WIDTHS = (7, 8, 9, 15, 511, 513, 1029, 2730, 3077, 4099, 8192, 8193, 12291, 16381, 16390)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    torch.cuda.init()


def _views(specs, pad, shift):
    """Weights and gradients as views at a row stride `pad` above the width, `shift` elements into
    their buffers; weights drawn as the workloads draw them."""
    wl = W.Workload("views", specs, 1)
    ws, gs, bufs = [], [], []
    for s in specs:
        ld = s.shape[-1] + pad
        rows = s.shape[0] * s.shape[1] if len(s.shape) == 3 else s.shape[0]
        strides = (s.shape[1] * ld, ld, 1) if len(s.shape) == 3 else (ld, 1)
        wb = torch.full((rows * ld + shift + 8,), 3.0, dtype=torch.bfloat16, device="cuda")
        gb = torch.full_like(wb, float("nan"))
        w, g = (b.as_strided(s.shape, strides, shift) for b in (wb, gb))
        w.copy_(W.init_weight(s, wl, torch.device("cuda")))
        g.zero_()
        ws.append(w)
        gs.append(g)
        bufs.append((wb, w))
    return ws, gs, bufs


@pytest.mark.parametrize("hp", [oracle.DEFAULTS, dict(oracle.DEFAULTS, weight_decay=0.05, max_grad_norm=1e-2)],
                         ids=["plain", "gnorm+decay"])
@pytest.mark.parametrize("pad,shift", [(0, 0), (3, 1), (16, 8)], ids=["dense", "unaligned", "aligned_views"])
@pytest.mark.parametrize("tier", [W.BACKBONE, W.EXPERT], ids=["momentum", "expert"])
def test_row_widths_and_positions(tier, pad, shift, hp):
    specs = [W.Spec(f"w{m}", tier, (37 if m > 600 else 530, m), k) for k, m in enumerate(WIDTHS)]
    specs.append(W.Spec("stack", tier, (3, 41, 523), len(specs)))
    specs.append(W.Spec("one_row", tier, (1, 2055), len(specs)))
    ws, gs, bufs = _views(specs, pad, shift)
    log(f"[parity] widths {WIDTHS}, tier {tier}, row stride width + {pad}, {hp}; 3 steps")
    pr = ParityRun(W.Workload("widths", specs, 3), weights=ws, grads=gs, hp=hp)
    for t in (1, 2, 3):
        pr.step(t)
    assert pr.stats.ok(), pr.stats
    for s, (wb, w) in zip(specs, bufs):   # nothing outside the views was written
        keep = wb.clone()
        w_now = w.clone()
        w.fill_(3.0)
        assert bool((wb == 3.0).all()), s.name
        wb.copy_(keep)
        assert (bits(w) == bits(w_now)).all()


@pytest.mark.parametrize("tier", [W.BACKBONE, W.EXPERT], ids=["momentum", "expert"])
def test_narrow_chunks_taken_several_rows_at_a_time(tier):
    """The update pass takes 64 / g rows at a time where a chunk of 512 columns holds only g groups of
    8 (up to 32): aligned tables with one to 33 groups in their last chunk, and numbers of rows
    around those of a block of rows."""
    widths = (8, 16, 24, 40, 128, 168, 248, 256, 264, 520, 776, 1032, 2056)
    specs = [W.Spec(f"w{m}x{n}", tier, (n, m), k) for k, (m, n) in
             enumerate((m, n) for m in widths for n in (1, 2, 63, 65, 531) if m <= 776 or n > 63)]
    log(f"[parity] aligned widths {widths}, tier {tier}; 3 steps")
    pr = ParityRun(W.Workload("narrow", specs, 3), device="cuda:0")
    for t in (1, 2, 3):
        pr.step(t)
    assert pr.stats.ok(), pr.stats


@pytest.mark.parametrize("hp", [oracle.DEFAULTS, dict(oracle.DEFAULTS, weight_decay=0.05, max_grad_norm=1e-2)],
                         ids=["plain", "gnorm+decay"])
@pytest.mark.parametrize("pad,shift", [(0, 0), (3, 1)], ids=["dense", "unaligned"])
@pytest.mark.parametrize("tier", [W.BACKBONE, W.EXPERT], ids=["momentum", "expert"])
def test_rows_of_fewer_than_8_columns(tier, pad, shift, hp):
    """Up to 2048 of them take the tiled passes, more the row-band pass, one column per lane: every width,
    with numbers of rows on both sides, and a stack."""
    specs = [W.Spec(f"w{n}x{m}", tier, (n, m), 10 * n + m) for m in range(1, 8) for n in (1, 2, 31, 33, 530, 2048, 2049, 4099)]
    specs.append(W.Spec("stack", tier, (5, 77, 3), 9))
    ws, gs, bufs = _views(specs, pad, shift)
    log(f"[parity] widths 1 to 7, tier {tier}, row stride width + {pad}, {hp}; 3 steps")
    pr = ParityRun(W.Workload("narrow_rows", specs, 3), weights=ws, grads=gs, hp=hp)
    for t in (1, 2, 3):
        pr.step(t)
    assert pr.stats.ok(), pr.stats
    for s, (wb, w) in zip(specs, bufs):   # nothing outside the views was written
        w.fill_(3.0)
        assert bool((wb == 3.0).all()), s.name


@pytest.mark.parametrize("flags", [0, 2], ids=["plain", "exact_ulp"])
@pytest.mark.parametrize("fp32", [False, True], ids=["bf16", "fp32"])
def test_exact_moment_tensors_at_row_ends(fp32, flags):
    """Routers and vectors (the exact second moment, taken 8 elements at a time): contiguous ones of
    one element to several tiles, with and without a whole number of 2048-element rows, and
    router views whose rows start at any position, with momentum (vectors of the backbone) and
    without."""
    sf = oracle.STATE_FP32 if fp32 else 0
    shapes = [(W.ROUTER, (n, m)) for n, m in ((1, 1), (3, 5), (256, 8), (37, 7), (64, 96), (2049, 3), (130, 1031))]
    shapes += [(tier, (n,)) for tier in (W.BACKBONE, W.EXPERT) for n in (1, 7, 8, 9, 2047, 2048, 2049, 10240, 10243)]
    views = [W.Spec(f"rv{m}", W.ROUTER, (33, m), 100 + m, state_flags=sf) for m in (7, 8, 13, 130)]
    specs = [W.Spec(f"x{k}", t, s, k, state_flags=sf) for k, (t, s) in enumerate(shapes)] + views
    wl = W.Workload("exact", specs, 3)
    dt = torch.float32 if fp32 else torch.bfloat16
    ws, gs = [], []
    for s in specs:
        if s in views:
            base = [torch.zeros(33 * (s.shape[1] + 3) + 9, dtype=dt, device="cuda") for _ in range(2)]
            w, g = (b.as_strided(s.shape, (s.shape[1] + 3, 1), 1) for b in base)
        else:
            w, g = (torch.zeros(s.shape, dtype=dt, device="cuda") for _ in range(2))
        w.copy_(W.init_weight(s, wl, torch.device("cuda")))
        ws.append(w)
        gs.append(g)
    log(f"[parity] {len(specs)} exact-moment tensors, fp32={fp32}, flags={flags}; 3 steps")
    pr = ParityRun(wl, weights=ws, grads=gs, hp=dict(oracle.DEFAULTS, weight_decay=0.05), flags=flags)
    for t in (1, 2, 3):
        pr.step(t)
    assert pr.stats.ok(), pr.stats
