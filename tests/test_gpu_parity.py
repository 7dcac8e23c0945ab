"""End-to-end parity of libcdp (through the C ABI) with the CPU oracle on the same seeded
inputs: final weights of every stage, every micro-batch loss, and the exact tick trace.

Acceptance criteria (tests/parity_gates.py):
  fp32 runs: max|w_gpu - w_ref| / max|w_ref| <= 1e-4 for every parameter tensor;
  bf16 runs: <= 2e-2 over every stage vector theta^j, and per tensor the error of the applied
  update at most K = 4 times the error of the oracle run again with bf16 rounding wherever a
  bf16 path stores a value (tests/precision_standins.py), both measured against the fp64 oracle.
Every bf16 configuration is ALSO run with fp32 arithmetic (`also_f32`) at the same shapes, in the
same launch grouping, against the same oracle run at the fp32 criterion: that is the run which
would expose a wrong weight version, a dropped micro-batch gradient or a misplaced tile at full
size, below the bf16 noise floor.
"""
import time

import numpy as np
import pytest

import cdp_workloads as wl
from oracle import cdp_oracle as O
from oracle import layers as OL
from paper_2403_08837_amd import binding as b
from precision_standins import Bf16Storage, Fp32Accumulation
import parity_gates as G
import oracle_legs as OLG

pytestmark = pytest.mark.gpu
RULES = [wl.RULE_DP, wl.RULE_V1, wl.RULE_V2]


def run_gpu(cfg, rule, T, p0, xs, ys, lr=None, momentum=0.0, weight_decay=0.0, dp_batched=False, mask=None, bwd_fresh=False,
            dtype=None, dw_group=1):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    tr = b.Trainer(cfg.stages, cfg.in_shape, cfg.N, cfg.B, cfg.lr if lr is None else lr, rule, cfg.dtype if dtype is None else dtype,
                   momentum=momentum, weight_decay=weight_decay, dp_batched=dp_batched, fresh_mask=mask, bwd_fresh=bwd_fresh,
                   dw_group=dw_group)
    tr.set_weights(p0)
    keep = []
    for t in range(T):
        x = torch.from_numpy(xs[t]).cuda()
        y = torch.from_numpy(ys[t]).cuda()
        keep.append((x, y))
        tr.step(x, y)
    tr.drain()
    torch.cuda.synchronize()
    weights = [wl.unflatten_params(tr.weights(j), cfg.stages[j]) for j in range(cfg.S)]
    losses = np.stack([tr.losses(t) for t in range(T)])
    out = dict(weights=weights, losses=losses, trace=tr.trace(), live=tr.live_counts(), stats=tr.stats(),
               live_bytes=tr.live_bytes())
    tr.close()
    del keep
    torch.cuda.empty_cache()
    return out


def say(capfd, line):
    """Result lines of the long tests, written past pytest's capture."""
    import sys
    if capfd is not None:
        with capfd.disabled():
            sys.stdout.write(line + "\n")
            sys.stdout.flush()
    else:
        print(line)


def check(cfg, rule, T, seed=0, lr=None, emulate=True, also_f32=False, capfd=None, momentum=0.0, weight_decay=0.0,
          dp_batched=False, mask=None, bwd_fresh=False, full_size=False, dw_group=1):
    """One oracle run (fp64) against the library in the configuration's arithmetic; for bf16
    configurations the bf16-storage stand-in as yardstick (`emulate`) and optionally the library again
    in fp32 (`also_f32`).  full_size: benchmark-sized runs - the oracle legs run side by side in child
    processes and the fp32 run is judged with the fp32-accumulation stand-in as yardstick
    (parity_gates.yardstick_gate) instead of the strict per-tensor criterion."""
    xs, ys = wl.make_data(cfg, T, seed)
    p0 = wl.init_params(cfg, seed)
    kw = dict(lr=lr, momentum=momentum, weight_decay=weight_decay, mask=mask, bwd_fresh=bwd_fresh)
    f32 = cfg.dtype == wl.F32
    legs = ["fp64"] + (["bf16"] if (emulate and not f32) else []) + (["fp32"] if (full_size and (f32 or also_f32)) else [])
    t0 = time.time()
    if full_size:
        say(capfd, "[oracle %s] %s, %d steps ..." % (cfg.name, " + ".join(legs), T))
        runs = OLG.run_legs(cfg, rule, T, seed, kw, legs,
                            heartbeat=lambda sec: say(capfd, "[oracle %s] %.0f s" % (cfg.name, sec)))
        ref = runs["fp64"]
        emu = {k: v.params for k, v in runs.items() if k != "fp64"}
    else:
        ref = O.train_schedule(cfg, p0, xs, ys, rule, keep_versions=False, **kw)
        emu = {}
        if "bf16" in legs:
            emu["bf16"] = O.train_schedule(cfg, p0, xs, ys, rule, keep_versions=False, stage_impl=Bf16Storage, **kw).params
    t_ref = time.time() - t0
    got = run_gpu(cfg, rule, T, p0, xs, ys, dp_batched=dp_batched, dw_group=dw_group, **kw)
    assert got["trace"] == ref.trace
    assert got["live"] == ref.live_inputs
    assert np.isfinite(got["losses"]).all()
    den = max(1e-6, np.abs(ref.losses).max())
    tag = "%s rule=%d T=%d" % (cfg.name, rule, T)
    failures = []

    def judge(run, what, bf16):
        loss_e = np.abs(run["losses"] - ref.losses).max() / den
        if not bf16 and not full_size:
            ok, rep = G.f32_gate(run["weights"], ref.params)
            say(capfd, "%s %s: tensor max-rel %.3e at %s, loss err %.3e (oracle %.0f s)"
                % (tag, what, rep["tensor_max_rel"], rep["where"], loss_e, t_ref))
            loss_tol = 1e-4
        else:
            ok, rep = G.yardstick_gate(run["weights"], ref.params, emu.get("bf16" if bf16 else "fp32"), p0, T, bf16=bf16)
            say(capfd, "%s %s: stage err %.3e (stand-in %.3e), tensor max-rel %.3e, update err / bound worst %.2f %s "
                "(stand-in median %.3e), loss err %.3e (oracle %.0f s)"
                % (tag, what, rep["stage_err"], rep["emu_stage_err"], rep["tensor_max_rel"], rep["worst_ratio"], rep["worst"],
                   rep["emu_median"], loss_e, t_ref))
            loss_tol = 1e-1 if bf16 else 1e-2    # micro-batch losses of a few samples; weights are the gate
        if not ok:
            failures.append((what, rep["failed"][:8]))
        if not loss_e <= loss_tol:
            failures.append((what, "loss", loss_e))

    judge(got, "fp32" if f32 else "bf16", not f32)
    if also_f32 and not f32:
        g32 = run_gpu(cfg, rule, T, p0, xs, ys, dp_batched=dp_batched, dtype=wl.F32, dw_group=dw_group, **kw)
        assert g32["trace"] == ref.trace and g32["live"] == ref.live_inputs
        judge(g32, "same shapes in fp32", False)
    assert not failures, failures
    return got, ref


@pytest.mark.parametrize("rule", RULES)
@pytest.mark.parametrize("name", ["mlp_mini", "mlp_odd"])
def test_small_mlp_fp32_all_rules(name, rule):
    cfg = wl.get_config(name)
    check(cfg, rule, cfg.steps)


@pytest.mark.parametrize("rule", RULES)
def test_cfg1_tiny_mlp_fp32(rule):
    cfg = wl.get_config("cfg1")
    check(cfg, rule, cfg.steps)


@pytest.mark.parametrize("name", ["cfg2_mini", "cfg5_mini"])
@pytest.mark.parametrize("rule", [wl.RULE_V1, wl.RULE_V2])
def test_small_mlp_bf16(name, rule):
    cfg = wl.get_config(name)
    check(cfg, rule, cfg.steps)


@pytest.mark.parametrize("name", ["mlp_mini", "mlp_odd", "cfg1", "resnet18_mini_f32", "resnet50_mini_f32", "cfg2_mini",
                                  "cfg5_mini", "resnet18_mini"])
def test_lockstep_batched_dp_matches_dp_oracle(name):
    """The lock-step executor (all N micro-batches of a step as one batch per stage pass) against
    the oracle's DP rule: same trace, live counts, per-micro-batch losses and weights."""
    cfg = wl.get_config(name)
    got, _ = check(cfg, wl.RULE_DP, cfg.steps, dp_batched=True)
    assert got["stats"]["peak_live_stage_inputs"] == cfg.N * cfg.S


def test_lockstep_batched_dp_momentum():
    cfg = wl.get_config("mlp_mini")
    check(cfg, wl.RULE_DP, 4, momentum=0.9, weight_decay=5e-4, dp_batched=True)


@pytest.mark.parametrize("name", ["mlp_mini", "mlp_odd", "resnet18_mini_f32", "resnet50_mini_f32", "cfg2_mini", "resnet18_mini"])
def test_rules_between_v1_and_v2(name):
    """A per-(micro-batch, stage) mask of v2 / v1 choices (Sec. 3.2, "Update rules")."""
    cfg = wl.get_config(name)
    m = np.random.default_rng(7).integers(0, 2, (cfg.N, cfg.S))
    check(cfg, wl.RULE_MASK, cfg.steps, mask=m)


@pytest.mark.parametrize("name", ["mlp_mini", "mlp_odd", "resnet18_mini_f32", "resnet50_mini_f32", "cfg5_mini"])
def test_backward_with_freshest_parameters(name):
    """The backward reads the version that is freshest at its tick (the forward's plain weights
    still rebuild the pre-affine activation of folded conv+affine layers)."""
    cfg = wl.get_config(name)
    check(cfg, wl.RULE_V2, cfg.steps, bwd_fresh=True)


def test_single_microbatch_and_zero_lr():
    cfg = wl.get_config("mlp_odd")
    cfg.N = 1
    check(cfg, wl.RULE_V2, 4)
    cfg = wl.get_config("mlp_mini")
    got, ref = check(cfg, wl.RULE_V2, 3, lr=0.0)
    p0 = wl.init_params(cfg, 0)
    for j in range(cfg.S):
        for a, w in zip(got["weights"][j], p0[j]):
            assert np.array_equal(a, w)


@pytest.mark.parametrize("name", ["resnet18_mini_f32", "resnet50_mini_f32", "resnet18_odd_f32"])
@pytest.mark.parametrize("rule", [wl.RULE_DP, wl.RULE_V2])
def test_resnet_mini_fp32(name, rule):
    cfg = wl.get_config(name)
    check(cfg, rule, cfg.steps)


@pytest.mark.parametrize("name", ["resnet18_mini", "resnet50_mini", "resnet18_odd"])
def test_resnet_mini_bf16(name):
    cfg = wl.get_config(name)
    check(cfg, wl.RULE_V2, cfg.steps)


def test_cfg2_cifar_mlp_bf16_few_steps(capfd):
    check(wl.get_config("cfg2"), wl.RULE_V2, 5, also_f32=True, full_size=True, capfd=capfd)


def test_cfg2_cifar_mlp_bf16_full(capfd):
    """All 50 steps.  Rounding differences grow along a 50-step ReLU-net trajectory (the bf16-storage
    yardstick itself is 25-70 % away from the fp64 trajectory in the update of single tensors by
    then, and an fp32 run has left the fp64 trajectory through flipped ReLU masks as well), so the sharp
    check of this configuration is the fp32 run of the 5-step test above."""
    cfg = wl.get_config("cfg2")
    got, _ = check(cfg, wl.RULE_V2, cfg.steps, full_size=True, capfd=capfd)
    st = got["stats"]
    assert st["peak_live_stage_inputs"] == 36
    assert st["peak_activation_bytes"] < 0.7 * st["dp_activation_bytes"] * 1.2


def steady_ticks(cfg, T):
    """Ticks in which all N micro-batches are in flight."""
    return range(cfg.delay * (cfg.N - 1), 2 * cfg.S * T)


def test_cfg5_deep_wide_mlp_bf16_full_size(capfd):
    """24 x Linear(4096->4096), N=16 micro-batches of 64, d=3: full size, 3 steps + drain, in the launch
    configuration bench.py times: versions t-1, t, t+1 of a stage are distinct, and version t+1 overwrites
    the ring slot of t-1 while t is still being read."""
    cfg = wl.get_config("cfg5")
    got, _ = check(cfg, wl.RULE_V2, 3, also_f32=True, full_size=True, capfd=capfd)
    st = got["stats"]
    assert st["peak_live_stage_inputs"] == 200
    assert st["peak_activation_bytes"] < 0.6 * 2 * st["dp_activation_bytes"]
    # homogeneous stages: 200 retained stage inputs in every steady-state tick (plus the head's hidden
    # activation and dlogits while a micro-batch sits between the last stage's forward and backward)
    lb = [got["live_bytes"][k] for k in steady_ticks(cfg, 3)]
    unit = cfg.B * 4096 * 2
    assert min(lb) == 200 * unit and max(lb) == 201 * unit + cfg.B * 1000 * 2, (min(lb), max(lb))


def test_cfg3_resnet18_bf16_full_size(capfd):
    cfg = wl.get_config("cfg3")
    got, _ = check(cfg, wl.RULE_V2, 3, also_f32=True, full_size=True, capfd=capfd)
    assert got["stats"]["peak_live_stage_inputs"] == 18
    # heterogeneous stages: the retained bytes are periodic in the tick with the delay as period
    lb = [got["live_bytes"][k] for k in steady_ticks(cfg, 3)]
    assert len(set(lb)) <= cfg.delay and all(lb[k] == lb[k + cfg.delay] for k in range(len(lb) - cfg.delay))


def test_cfg4_resnet50_reduced_images_all_microbatches(capfd):
    """The ResNet-50 configuration as benchmarked (16 bottleneck stages at their real channel widths,
    N = 8 micro-batches of 32, d = 4, 1000 classes) on 64x64 inputs, 3 steps + drain: the mixing of
    theta_t and theta_{t-1} per Eq. (CDP-v2) and the weight-gradient accumulation over 8 micro-batches
    on these layers, at a twelfth of the oracle's cost."""
    cfg = wl.get_config("cfg4_s64")
    got, _ = check(cfg, wl.RULE_V2, 3, also_f32=True, full_size=True, capfd=capfd)
    assert got["stats"]["peak_live_stage_inputs"] == 68


def test_cfg4_resnet50_bf16_full_config_weights(capfd):
    """N = 8 micro-batches of 32 at 224x224 as benchmarked, 2 steps + drain (the second step mixes theta_0
    and theta_1 per Eq. (CDP-v2)): weights of every stage and all 16 objectives against the oracle, in
    bf16 and in fp32, each with its stand-in as yardstick (the three oracle runs side by side)."""
    cfg = wl.get_config("cfg4")
    got, _ = check(cfg, wl.RULE_V2, 2, also_f32=True, full_size=True, capfd=capfd)
    assert got["stats"]["peak_live_stage_inputs"] == 68
    lb = [got["live_bytes"][k] for k in steady_ticks(cfg, 2)]
    assert len(set(lb)) <= cfg.delay


@pytest.mark.parametrize("name,rule", [("mlp_odd", wl.RULE_V2), ("mlp_odd", wl.RULE_V1), ("resnet18_mini_f32", wl.RULE_V2),
                                       ("cfg2_mini", wl.RULE_V2), ("resnet18_mini", wl.RULE_DP)])
def test_momentum_and_weight_decay(name, rule):
    """SGD with momentum 0.9 and weight decay 5e-4 (the optimiser of Sec. 5 "Hyperparameters")."""
    cfg = wl.get_config(name)
    check(cfg, rule, cfg.steps, momentum=0.9, weight_decay=5e-4)


@pytest.mark.parametrize("momentum", [0.0, 0.9])
@pytest.mark.parametrize("dtype,inputs,width,classes", [(wl.F32, 70, 132, 10), (wl.F32, 64, 130, 12), (wl.BF16, 70, 136, 10),
                                                        (wl.BF16, 72, 132, 16), (wl.BF16, 264, 72, 33)])
def test_layers_with_one_width_that_is_not_whole_pieces(dtype, inputs, width, classes, momentum):
    """The update writes a forward and a transposed copy of the new weights, each in 16-byte pieces where its own rows are whole ones:
    input widths, output widths, both or neither."""
    # bf16: an update is 5.4e-2 off in its worst tensor, the storage stand-in by as much, and the gate is 2e-2 of the largest weight, so the
    # steps together have to stay below 0.37 of it; momentum 0.9 adds up to 2.7 times as much in three steps and takes a fifth of the rate
    cfg = wl.Config("mlp_one_odd", wl._mlp(inputs, width, 2, classes, stem=False), (inputs,), classes, N=2, B=5, dtype=dtype,
                    lr=0.004 if momentum else 0.02, steps=3)
    check(cfg, wl.RULE_V2, cfg.steps, momentum=momentum, weight_decay=5e-4 if momentum else 0.0)


def test_ring_copy_of_previous_version():
    """cdp_get_weights(version = freshest-1) returns the compute copy still in the ring."""
    import torch
    cfg = wl.get_config("mlp_mini")
    xs, ys = wl.make_data(cfg, 2)
    p0 = wl.init_params(cfg)
    ref = O.train_schedule(cfg, p0, xs, ys, wl.RULE_V2)
    tr = b.Trainer(cfg.stages, cfg.in_shape, cfg.N, cfg.B, cfg.lr, wl.RULE_V2, cfg.dtype)
    tr.set_weights(p0)
    for t in range(2):
        tr.step(torch.from_numpy(xs[t]).cuda(), torch.from_numpy(ys[t]).cuda())
    tr.drain()
    for j in range(cfg.S):
        prev = wl.unflatten_params(tr.weights(j, version=1), cfg.stages[j])
        assert O.max_rel_err(prev, ref.versions[(j, 1)]) <= 1e-4
        with pytest.raises(b.CdpError) as e:
            tr.weights(j, version=0)
        assert e.value.code == b.CDP_ESTATE
    tr.close()


@pytest.mark.parametrize("name", ["cfg1", "cfg2_mini"])
def test_tick_by_tick_and_unaligned_inputs_give_the_same_weights(name):
    """Three ways to feed the same three steps: cdp_step; cdp_tick with the mini-batch pointer on
    every tick of its step and NULL during the drain; cdp_step on input rows that are not
    16-byte aligned (the first layer then reads the staged copy instead of the caller's rows).
    Tick by tick gives bit-identical weights (the same launches); the unaligned run groups its
    launches differently and agrees with the oracle and with the first run at the usual tolerance;
    the logged losses are equal
    bit for bit tick by tick (row losses are summed in fixed point) and agree to fp32 rounding otherwise."""
    import torch
    cfg = wl.get_config(name)
    T = 3
    xs, ys = wl.make_data(cfg, T)
    p0 = wl.init_params(cfg)
    ref = O.train_schedule(cfg, p0, xs, ys, wl.RULE_V2, keep_versions=False)

    def run(mode):
        tr = b.Trainer(cfg.stages, cfg.in_shape, cfg.N, cfg.B, cfg.lr, wl.RULE_V2, cfg.dtype)
        tr.set_weights(p0)
        keep = []
        for t in range(T):
            x, y = torch.from_numpy(xs[t]).cuda(), torch.from_numpy(ys[t]).cuda()
            if mode == "unaligned":
                big = torch.empty(x.numel() + 1, dtype=torch.float32, device="cuda")
                big[1:].copy_(x.reshape(-1))
                x = big[1:].view(x.shape)
                assert x.data_ptr() % 16 != 0
            keep.append((x, y))
            if mode == "tick":
                for _ in range(2 * cfg.S):
                    tr.tick(x, y)
            else:
                tr.step(x, y)
        tr.drain()
        torch.cuda.synchronize()
        w = [tr.weights(j) for j in range(cfg.S)]
        losses = np.stack([tr.losses(t) for t in range(T)])
        trace = tr.trace()
        tr.close()
        return w, losses, trace

    base = run("step")
    assert base[2] == ref.trace
    tol = 1e-4 if cfg.dtype == wl.F32 else 2e-2
    for j in range(cfg.S):
        err = G.stage_max_rel(wl.unflatten_params(base[0][j], cfg.stages[j]), ref.params[j])
        assert err <= tol, err
    for mode in ("tick", "unaligned"):
        got = run(mode)
        assert got[2] == base[2]
        if mode == "tick":
            assert np.array_equal(got[1], base[1]), mode     # the same launches; row losses meet in integer (fixed-point) adds
        else:
            assert np.allclose(got[1], base[1], rtol=1e-5, atol=0), mode
        for j in range(cfg.S):
            if mode == "tick":
                assert np.array_equal(got[0][j], base[0][j]), (mode, j)   # the same launches in the same order
            else:
                # other launch grouping, hence another summation order inside the contractions
                w = wl.unflatten_params(got[0][j], cfg.stages[j])
                assert G.stage_max_rel(w, ref.params[j]) <= tol, (mode, j)
                assert G.stage_max_rel(w, wl.unflatten_params(base[0][j], cfg.stages[j])) <= tol, (mode, j)


@pytest.mark.parametrize("rule", RULES)
def test_vit_mini_fp32_all_rules(rule):
    """ViT-shaped stages (LayerNorm, attention, GELU, residuals around token-wise linear maps)."""
    cfg = wl.get_config("vit_mini_f32")
    check(cfg, rule, cfg.steps)


def test_vit_mini_bf16_and_variants():
    cfg = wl.get_config("vit_mini")
    check(cfg, wl.RULE_V2, cfg.steps)
    cfg = wl.get_config("vit_mini_f32")
    check(cfg, wl.RULE_DP, 3, dp_batched=True)
    check(cfg, wl.RULE_V2, 3, momentum=0.9, weight_decay=5e-4)
    check(cfg, wl.RULE_V2, 3, bwd_fresh=True)


@pytest.mark.parametrize("name,rule", [("vit_odd", wl.RULE_V2), ("vit_odd", wl.RULE_V1), ("vit_odd_bf16", wl.RULE_V2),
                                       ("vit_long", wl.RULE_V2)])
def test_vit_odd_shapes(name, rule):
    """9 tokens of width 20 in heads of width 5, micro-batches of 3: no extent is a multiple of
    four, so the attention products take their element-wise staging path, every tile is ragged and
    (in bf16) LayerNorm rows are not whole 16-byte chunks.
    vit_long has 324 tokens (more than one 256-wide pass of the softmax lanes, six ragged 64-row tiles)."""
    cfg = wl.get_config(name)
    check(cfg, rule, cfg.steps)


@pytest.mark.parametrize("dim,heads,B,rule", [(64, 4, 3, wl.RULE_V2),     # 192 rows, hidden width 256: the smallest tiles
                                              (40, 5, 3, wl.RULE_V1),     # channel counts that are not whole slabs
                                              (64, 2, 13, wl.RULE_V2),    # 832 rows, a ragged last tile
                                              (32, 2, 40, wl.RULE_DP)])   # 2560 rows, hidden width 128
def test_vit_gelu_in_the_contractions(dim, heads, B, rule):
    """More than 128 token rows in bf16: the block's GELU is computed by the contractions before and after it (fewer rows, and
    fp32, have kernels of its own)."""
    cfg = wl.Config("vit_gelu", wl._vit(32, 4, dim, heads, 2, 5), (32, 32, 3), 5, N=2, B=B, dtype=wl.BF16, lr=0.02, steps=3,
                    init_gain_last_affine=0.25, init_gain_head=0.2)
    check(cfg, rule, cfg.steps)


def test_vit_b16_full_shapes_single_microbatch(capfd):
    """Every stage of the ViT-B/16-shaped workload at its real shape (B = 32, 196 tokens of width
    768, 12 heads, 12 block stages, 1000 classes) with one micro-batch per step, where CDP-v2 is
    plain SGD: 2 steps against the oracle at the stated weight tolerance."""
    cfg = wl.get_config("vit_b16")
    cfg.N = 1
    check(cfg, wl.RULE_V2, 2, also_f32=True, full_size=True, capfd=capfd)


def test_vit_b16_full_config_sampled():
    """N = 8 micro-batches as benchmarked: exact tick trace / live counts against the oracle's
    bookkeeping, the objective of two sampled micro-batches of the first step against an oracle
    forward pass, and finite weights that moved."""
    cfg = wl.get_config("vit_b16")
    T = 2
    xs, ys = wl.make_data(cfg, T, 0)
    p0 = wl.init_params(cfg, 0)
    got = run_gpu(cfg, wl.RULE_V2, T, p0, xs, ys)
    ref = O.train_schedule(cfg, None, [None] * T, [None] * T, wl.RULE_V2, compute=False)
    assert got["trace"] == ref.trace and got["live"] == ref.live_inputs
    assert got["stats"]["peak_live_stage_inputs"] == 52
    assert got["stats"]["peak_activation_bytes"] < 0.7 * got["stats"]["dp_activation_bytes"]
    p64 = [[np.asarray(a, dtype=np.float64) for a in st] for st in p0]
    for i in (0, cfg.N - 1):
        sl = slice(i * cfg.B, (i + 1) * cfg.B)
        h = np.asarray(xs[0][sl], dtype=np.float64)
        for j, st in enumerate(cfg.stages):
            h, _ = OL.stage_forward(st, p64[j], h, ys[0][sl] if j == cfg.S - 1 else None)
        print("vit_b16 micro-batch %d: loss gpu %.5f oracle %.5f" % (i, got["losses"][0, i], h))
        assert abs(got["losses"][0, i] - h) <= 2e-2 * abs(h)
    assert np.isfinite(got["losses"]).all()
    for j in range(cfg.S):
        for g, w0 in zip(got["weights"][j], p0[j]):
            assert np.isfinite(g).all()
        assert any(np.abs(g - w0).max() > 0 for g, w0 in zip(got["weights"][j], p0[j]))


@pytest.mark.parametrize("name,rule", [("mlp_longk", wl.RULE_V2), ("mlp_longk", wl.RULE_V1), ("mlp_longk", wl.RULE_DP),
                                       ("mlp_longk_bf16", wl.RULE_V2), ("mlp_longk_b40", wl.RULE_V2)])
def test_long_reduction_shared_by_several_workgroups(name, rule):
    """A stem whose reduction is long enough that the thin forward tiles split it over several
    workgroups (partial tiles in the workspace, the last arrival finishes the tile), with a
    ragged last slab and ragged output tiles; with 40 rows the 64-row tiles do the same."""
    cfg = wl.get_config(name)
    check(cfg, rule, cfg.steps)



@pytest.mark.parametrize("name,T", [("resnet18_mini", 3), ("resnet50_mini_f32", 3), ("cfg2_mini", 3), ("mlp_longk", 60),
                                    ("mlp_longk_b40", 60), ("resnet18_mini_f32", 40)])
def test_two_runs_give_identical_bits(name, T):
    """Nothing in a step depends on the order in which workgroups happen to finish: partial sums meet in
    fixed orders, row losses in integer adds.  Two runs of the same steps agree bit for bit in every
    weight and every logged loss.  The long runs are a soak of the reductions shared by several workgroups
    (partial tiles in a workspace, the last arrival adds them): some thousand such launches per run, and a
    partial tile read before it was complete would change the bits."""
    cfg = wl.get_config(name)
    xs, ys = wl.make_data(cfg, T)
    p0 = wl.init_params(cfg)
    a = run_gpu(cfg, wl.RULE_V2, T, p0, xs, ys)
    b2 = run_gpu(cfg, wl.RULE_V2, T, p0, xs, ys)
    assert np.array_equal(a["losses"], b2["losses"])
    for wa, wb in zip(a["weights"], b2["weights"]):
        for x, y in zip(wa, wb):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("name,rule,g", [("cfg1", wl.RULE_V2, 2), ("cfg1", wl.RULE_V2, 4), ("cfg1", wl.RULE_V1, 2), ("mlp_odd", wl.RULE_V2, 2),
                                         ("mlp_odd", wl.RULE_V2, 4), ("mlp_longk_b40", wl.RULE_V2, 4), ("cfg2_mini", wl.RULE_V2, 2),
                                         ("cfg5_mini", wl.RULE_V2, 4), ("resnet18_mini_f32", wl.RULE_V2, 2)])
def test_weight_gradients_of_a_group_of_micro_batches_in_one_pass(name, rule, g):
    """dw_group = g: the Linear layers keep (dY, X) of g consecutive micro-batches of a stage and take one pass
    over the accumulator per group.  The sum of Eq. (CDP) is the same, in the same order of micro-batches:
    same trace, same live counts, weights and losses within the usual criteria; what changes is the memory:
    finished backward passes keep their activations until the group is complete."""
    cfg = wl.get_config(name)
    got, _ = check(cfg, rule, cfg.steps, dw_group=g)
    xs, ys = wl.make_data(cfg, cfg.steps)
    base = run_gpu(cfg, rule, cfg.steps, wl.init_params(cfg), xs, ys)
    linear_only = all(l.kind != wl.CONV2D for st in cfg.stages for l in st)
    if linear_only:
        assert got["stats"]["peak_activation_bytes"] > base["stats"]["peak_activation_bytes"]
        assert max(got["live_bytes"]) > max(base["live_bytes"])


def test_cfg5_grouped_weight_gradients_full_size(capfd):
    """cfg5 with dw_group = 4: a quarter of the accumulator passes, at full size, 3 steps."""
    cfg = wl.get_config("cfg5")
    got, _ = check(cfg, wl.RULE_V2, 3, full_size=True, dw_group=4, capfd=capfd)
    assert got["stats"]["peak_live_stage_inputs"] == 200
