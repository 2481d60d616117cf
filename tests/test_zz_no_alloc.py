"""The no-allocation context set-up (skew_state_init_static) against skew_state_init.

skew_state_init_static swaps the caller's workspace for the library's static one; the
kernels are the same, so every weight and state bit must equal the ordinary set-up's on
the same inputs. Two set-ups in a row share the one static array: the second, with a
smaller table, must still match (the set-up clears what its table uses), and the first
context is then refused (SKEW_ESTALE) instead of stepping on the array. A table whose own
plan is larger than the array is planned with larger bands: against the oracle.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_19058_amd import SkewAdam, SkewError
from paper_2607_19058_amd import workloads as W
from paper_2607_19058_amd.skewadam import SKEW_ESTALE, STATIC_WORKSPACE_BYTES

from parity_util import ParityRun, bits, log

pytestmark = pytest.mark.gpu


def _run(wl, specs, static, steps):
    dev = torch.device("cuda")
    Wt = [W.init_weight(s, wl, dev) for s in specs]
    G = [torch.zeros(s.shape, dtype=torch.bfloat16, device=dev) for s in specs]
    opt = SkewAdam([(s.tier, Wt[k], G[k], s.tensor_id) for k, s in enumerate(specs)], static_workspace=static)
    for t in range(1, steps + 1):
        sc = W.expert_scales(wl, t)
        for k, s in enumerate(specs):
            W.fill_grad(s, wl, t, G[k], sc)
        opt.step(t, seed=3, weight_decay=0.05, clip_threshold=0.5)
    torch.cuda.synchronize()
    return Wt, opt


def _same(a_w, a, b_w, b, what):
    for k, (x, y) in enumerate(zip(a_w, b_w)):
        assert np.array_equal(bits(x), bits(y)), (what, "w", k)
    assert torch.equal(a.state, b.state), (what, "state")
    ka, ra = a.clip_info()
    kb, rb = b.clip_info()
    assert ka == kb and ra == rb, (what, "clip factors")


def test_static_workspace_matches_caller_workspace():
    wl = W.get("tiny")
    log("[no-alloc] call 1: tiny (21 tensors), 4 steps, static vs caller workspace")
    wa, a = _run(wl, wl.specs, False, 4)
    wb, b = _run(wl, wl.specs, True, 4)
    _same(wa, a, wb, b, "call 1")
    sub = wl.specs[::3]
    log(f"[no-alloc] call 2: a smaller table ({len(sub)} tensors), 3 steps, on the same static array")
    wc, c = _run(wl, sub, False, 3)
    wd, d = _run(wl, sub, True, 3)
    _same(wc, c, wd, d, "call 2")
    assert d.workspace is None and b.workspace is None
    with pytest.raises(SkewError) as ei:
        b.step(5)
    assert ei.value.status == SKEW_ESTALE
    # the newer context keeps stepping, and still matches
    for opt in (c, d):
        opt.step(4, seed=3, weight_decay=0.05, clip_threshold=0.5)
    torch.cuda.synchronize()
    _same(wc, c, wd, d, "call 2, step 4")
    for o in (a, b, c, d):
        o.close()


@pytest.mark.parametrize("hp", [dict(), dict(weight_decay=0.05, max_grad_norm=1e-2)], ids=["plain", "gnorm+decay"])
def test_static_workspace_plans_of_larger_bands(hp):
    """A table whose own plan needs more than the static workspace (its row bands would fill the chip):
    planned with larger bands, tiles and matrix rows (not flat) for its exact moments, every tensor
    against the oracle."""
    shapes = [(W.BACKBONE, (4096, 16384)), (W.EXPERT, (2048, 16384)), (W.BACKBONE, (1024, 2048)), (W.BACKBONE, (3, 12000)),
              (W.EXPERT, (3000, 5)), (W.BACKBONE, (1024, 20000)), (W.EXPERT, (5, 77, 523)), (W.ROUTER, (2048, 7)),
              (W.ROUTER, (256, 8)), (W.BACKBONE, (2051,)), (W.EXPERT, (1024, 16000))]
    specs = [W.Spec(f"t{k}", t, s, k) for k, (t, s) in enumerate(shapes)]
    pr = ParityRun(W.Workload("static_large", specs, 2), hp=dict(oracle.DEFAULTS, **hp))
    assert pr.opt.workspace_nbytes > STATIC_WORKSPACE_BYTES
    pr.opt.close()
    pr.opt = SkewAdam([(s.tier, pr.W[k], pr.G[k], s.tensor_id) for k, s in enumerate(specs)], static_workspace=True)
    log(f"[no-alloc] {len(specs)} tensors whose plan takes {pr.opt.workspace_nbytes} bytes of workspace, 2 steps, {hp}")
    for t in (1, 2):
        pr.step(t)
    assert pr.stats.ok(), pr.stats
    pr.opt.close()
