"""The benchmark configurations at their own batch sizes, against the oracle.

AlexNet at batch 32 (seed 1), ResNet-18 at batch 128 (seed 2), VGG-16 at
batch 32 (seed 3) and ResNet-50 at batch 64 (seed 4); the tiny network at its
own batch of 4 is in test_gpu_step.py.  One dc_step (Sec. III-A: pull,
forward, backward, push, server SGD at lr 0.01) runs under a random
segmentation, which leaves the numbers unchanged (Sec. V-B), and the oracle
runs the same iteration in float64.

* Loss within 1e-4 relative.
* Every parameter tensor's gradient, post-step weight and update within 1e-3
  max relative error (max |x - r| / max |r|; the update's distance is taken
  less half an ulp of each stored float32 weight, its rounding on the server).  Only a tensor that misses 1e-3
  and whose float32 scatter at this batch exceeds 2e-4 is held to 5x that
  scatter instead.  The scatter is the largest distance from the oracle of
  four float32-grade evaluations of the same iteration: torch's CPU float32,
  the same with every parameter nudged by 2^-24 relative, and torch's float64
  with every conv / FC / BN output scaled by (1 + eps xi), eps = 2^-23 and
  2^-21.  The test reports how many tensors missed 1e-3, how many got the
  wider bar and the worst error / bar.
* For VGG-16 and ResNet-50 every op's kernels, plain and as the model folds
  them, also run on the oracle's own tensors of this iteration at kernel
  bars (tests/layerwise.py).
* The same iteration with the GPU's own discrete decisions given to the
  oracle (every ReLU mask read back as the ReLU output > 0, every max-pool's
  window taps): what float32 rounding leaves once no decision near a tie can
  flip.  The same bar rule, with the scatter of the same float32-grade
  evaluations taken with the GPU's decisions held fixed as well.
"""
import numpy as np
import pytest

from oracle import cnn as OC
from paper_2101_07968_amd import _lib as D
from paper_2101_07968_amd import nets as PN
from tests import layerwise
from tests.gpu_helpers import rel_err, report, update_err
from tests.test_gpu_step import UNPACED, gpu_decisions, plans_for, setup_model

pytestmark = pytest.mark.gpu

FULL = [("alexnet", 32, 1), ("resnet18", 128, 2), ("vgg16", 32, 3), ("resnet50", 64, 4)]
LAYERWISE = {"vgg16", "resnet50"}
BAR = 1e-3
SCATTER_FLOOR = 2e-4


def fp32_scatter(spec, onet, x, y, params, g_ref, decisions=None):
    """Per tensor, the largest distance from the oracle of float32-grade evaluations
    (gradients and post-step weights), with the given decisions held if any; see the
    module docstring."""
    import torch
    from tests import torch_ref
    rng = np.random.default_rng(4321)
    runs = [torch_ref.loss_and_grads(spec, onet, x, y, params, torch.float32, decisions=decisions)[1]]
    pp = params.astype(np.float64) * (1.0 + 2.0 ** -24 * rng.standard_normal(params.size))
    runs.append(torch_ref.loss_and_grads(spec, onet, x, y, pp, torch.float32, decisions=decisions)[1])
    for eps in (2.0 ** -23, 2.0 ** -21):
        def nudge(i, o, eps=eps):
            xi = torch.from_numpy(rng.standard_normal(tuple(o.shape)))
            return o * (1.0 + eps * xi)
        runs.append(torch_ref.loss_and_grads(spec, onet, x, y, params, torch.float64, perturb=nudge,
                                             decisions=decisions)[1])
    w_ref = params.astype(np.float64) - OC.LR * g_ref
    out_g, out_w = {}, {}
    for i, slots in enumerate(onet.pslots):
        for pname, (off, shape) in slots.items():
            sl = slice(off, off + int(np.prod(shape)))
            out_g[(i, pname)] = max(rel_err(r[sl], g_ref[sl]) for r in runs)
            out_w[(i, pname)] = max(rel_err(params[sl].astype(np.float64) - OC.LR * r[sl], w_ref[sl]) for r in runs)
    return out_g, out_w


@pytest.mark.parametrize("name,batch,seed", FULL, ids=[f"{n}-b{b}" for n, b, _ in FULL])
def test_full_batch_matches_oracle(name, batch, seed):
    import torch
    model, onet, xd, yd, x, y, params = setup_model(name, batch, seed)
    print(f"full batch {name} batch {batch} seed {seed}: dc_step", flush=True)
    st = model.step(xd, yd, plans_for(model.L, seed=seed)["random"], UNPACED)
    p_new, g = model.ps_read()
    dec = gpu_decisions(model, onet, name)  # the GPU's ReLU masks and max-pool taps in this iteration
    model.close()
    del model, xd, yd
    torch.cuda.empty_cache()
    print(f"full batch {name}: oracle iteration", flush=True)
    res = onet.loss_and_grads(x, y, params, keep=name in LAYERWISE)
    loss_ref, g_ref = res[0], res[1]
    p_ref = OC.sgd(params, g_ref)
    assert np.isfinite(st["loss"])
    loss_err = abs(st["loss"] - loss_ref) / abs(loss_ref)
    assert loss_err <= 1e-4, (st["loss"], loss_ref)

    rows = []
    for i, slots in enumerate(onet.pslots):
        for pname, (off, shape) in slots.items():
            sl = slice(off, off + int(np.prod(shape)))
            rows.append(((i, pname), rel_err(g[sl], g_ref[sl]), rel_err(p_new[sl], p_ref[sl]),
                         update_err(p_new[sl], params[sl], -OC.LR * g_ref[sl])))
    missed = [r for r in rows if max(r[1], r[2], r[3]) > BAR]
    scatter_g = scatter_w = {}
    if missed:
        print(f"full batch {name}: {len(missed)} tensors above {BAR:g}; float32 scatter", flush=True)
        scatter_g, scatter_w = fp32_scatter(onet.spec, onet, x, y, params, g_ref)

    def bar_for(sc):
        return BAR if sc <= SCATTER_FLOOR else max(BAR, 5.0 * sc)

    widened, worst, fails = 0, 0.0, []
    for key, eg, ew, eu in rows:
        bg = bar_for(scatter_g.get(key, 0.0))
        bw = bar_for(scatter_w.get(key, 0.0))
        widened += bg > BAR or bw > BAR
        worst = max(worst, eg / bg, ew / bw, eu / (1.01 * bg + 1e-6))
        if eg > bg or ew > bw or eu > 1.01 * bg + 1e-6:
            fails.append((key, eg, ew, eu, scatter_g.get(key), bg))
    rows.sort(key=lambda r: -r[1])
    report(f"full batch {name} b{batch} seed {seed}: loss rel err {loss_err:.1e}; {len(rows)} tensors, "
           f"{len(missed)} above {BAR:g}, {widened} on a widened bar, worst err/bar {worst:.3f}; "
           "largest gradient errors (op, tensor, err, fp32 scatter): "
           + ", ".join(f"({k[0]},{k[1]},{eg:.1e},{scatter_g.get(k, float('nan')):.1e})"
                       for k, eg, _, _ in rows[:4]))
    assert not fails, fails[:5]
    print(f"full batch {name}: oracle iteration with the GPU's decisions", flush=True)
    loss_d, g_d = onet.loss_and_grads(x, y, params, decisions=dec)
    p_d = OC.sgd(params, g_d)
    flips = sum(int((dec[i] != res[3][i]).sum()) for i in dec) if name in LAYERWISE else None
    assert abs(st["loss"] - loss_d) <= 1e-4 * abs(loss_d)
    errs = {}
    for i, slots in enumerate(onet.pslots):
        for pname, (off, shape) in slots.items():
            sl = slice(off, off + int(np.prod(shape)))
            errs[(i, pname)] = max(rel_err(g[sl], g_d[sl]), rel_err(p_new[sl], p_d[sl]),
                                   update_err(p_new[sl], params[sl], -OC.LR * g_d[sl]) / 1.01)
    scatter_d = {}
    if max(errs.values()) > BAR:
        print(f"full batch {name}: float32 scatter with the decisions held", flush=True)
        scatter_d, _ = fp32_scatter(onet.spec, onet, x, y, params, g_d, dec)
    worst_d, widened_d, fails_d = (None, 0.0), 0, []
    for key, e in errs.items():
        b = bar_for(scatter_d.get(key, 0.0))
        widened_d += b > BAR
        if e / b > worst_d[1]:
            worst_d = (key, e / b)
        if e > b:
            fails_d.append((key, e, scatter_d.get(key), b))
    report(f"full batch {name} b{batch} with the GPU's decisions: loss rel err "
           f"{abs(st['loss'] - loss_d) / abs(loss_d):.1e}; {len(errs)} tensors, "
           f"{sum(e > BAR for e in errs.values())} above {BAR:g}, {widened_d} on a widened bar, worst err/bar "
           f"{worst_d[1]:.3f} at {worst_d[0]} (err {errs[worst_d[0]]:.1e})"
           + (f"; decisions that differ from the oracle's own: {flips}" if flips is not None else ""))
    assert not fails_d, fails_d[:5]
    if name in LAYERWISE:
        print(f"full batch {name}: each op on the oracle's tensors", flush=True)
        worst_ops = layerwise.check_ops(name, onet, y, params, res)
        report(f"layer-wise {name} b{batch}: worst error / bar per op kind: "
               + ", ".join(f"{k} {v:.3f}" for k, v in sorted(worst_ops.items())))


def test_googlenet_batch_gradients_with_gpu_decisions():
    """GoogLeNet at its own batch, where most of its passes multiply split operands: its gradients move by about
    1e-4 to 1e-3 with any change of rounding, because some of its 1.5e8 ReLU and max-pool decisions lie within
    rounding of a tie.  With the GPU's own decisions given to the oracle every tensor stays within the bar of a
    single pass of 1000 terms (2e-5), so nothing but those decisions differs."""
    name, batch, seed = "googlenet", 32, 5
    ops, hwc, _ = PN.build(name)
    split = [D.conv_plan_split(g, p) for _i, g, first in PN.conv_geoms(ops, hwc, batch) for p in range(3)
             if not (first and p == 1)]
    assert sum(split) > len(split) // 2, split
    model, onet, xd, yd, x, y, params = setup_model(name, batch, seed)
    print(f"full batch {name}: dc_step", flush=True)
    st = model.step(xd, yd, plans_for(model.L, seed=seed)["random"], UNPACED)
    _p, g = model.ps_read()
    dec = gpu_decisions(model, onet, name)
    model.close()
    print(f"full batch {name}: oracle iteration, with its own and with the GPU's decisions", flush=True)
    own = onet.loss_and_grads(x, y, params, keep=True)
    flips = sum(int((dec[i] != own[3][i]).sum()) for i in dec)
    loss_d, g_d = onet.loss_and_grads(x, y, params, decisions=dec)
    errs = {(i, pname): rel_err(g[off:off + int(np.prod(shape))], g_d[off:off + int(np.prod(shape))])
            for i, slots in enumerate(onet.pslots) for pname, (off, shape) in slots.items()}
    worst = max(errs, key=errs.get)
    plain = np.linalg.norm(g - own[1]) / np.linalg.norm(own[1])
    report(f"full batch {name} b{batch}: {sum(split)} of {len(split)} passes on split operands; {flips} decisions of "
           f"{sum(d.size for d in dec.values())} differ from the oracle's own, gradients {plain:.1e} from it; with the "
           f"GPU's decisions worst tensor {errs[worst]:.1e} at {worst}")
    assert abs(st["loss"] - loss_d) <= 1e-6 * abs(loss_d)
    assert errs[worst] <= 2e-5, (worst, errs[worst])
