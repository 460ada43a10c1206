"""End-to-end parity of the schedule-executed training step on a real MI355X, through the C ABI.

Loss and parameter gradients are compared with the fp64 store-everything oracle (normwise per
tensor: activations/loss 1e-4, gradients 1e-3); the executor's reported peak must equal the
oracle interpreter's peak for the same schedule and stay within the predicted bound; gradients
must not depend on the schedule (bitwise when the operator variants are the same)."""
import itertools

import numpy as np
import pytest

from oracle import network as onet
from oracle import schedule as osch
from workloads import graphs, schedules, tensors
import paper_2010_14501_amd as M
from paper_2010_14501_amd.runner import StepRunner

pytestmark = pytest.mark.gpu

from parity_util import (ACT_TOL, GRAD_TOL, DEEP_ACT_TOL, DECISION_BAND, check_close, compare_grads,
                         oracle_with_gpu_decisions)


def oracle_step(g, exts, params):
    oe, op = tensors.oracle_inputs(exts, params)
    return onet.store_everything_step(g.text(), oe, op)


def pick_seed(g, min_margin=1e-4):
    """Seed whose ReLU inputs all stay away from zero in the oracle, so that the fp32 path cannot
    flip a sign bit and the end-to-end mask comparison is exact."""
    for seed in range(50):
        exts, params = tensors.make_inputs(g, seed=seed, gamma_beta="random")
        ref = oracle_step(g, exts, params)
        margin = min(np.abs(ref["acts"][n.ins[0]]).min() for n in g.nodes if n.op in ("relu", "relu6"))
        if margin > min_margin:
            return seed, exts, params, ref
    raise RuntimeError("no seed found")


@pytest.fixture(scope="module")
def tiny():
    g = graphs.tiny_chain()
    seed, exts, params, ref = pick_seed(g)
    return g, exts, params, ref


def test_tiny_chain_named_schedule(tiny):
    g, exts, params, ref = tiny
    sch = schedules.tiny_chain_schedule(g, {0, 2})
    want = osch.interpret(g.text(), sch.text())
    run = StepRunner(g.text(), sch.text(), exts, params, poison=True)
    peak = run.step()
    assert peak == want["peak"] == run.plan.exact_peak == 232448
    assert peak <= run.plan.predicted_peak
    assert abs(run.loss_value() - ref["loss"]) < ACT_TOL * abs(ref["loss"])
    compare_grads(run.grads_numpy(), ref)
    # a second step on the same plan gives the same bits
    g1 = run.grads_numpy()
    run.step()
    g2 = run.grads_numpy()
    assert all(np.array_equal(g1[p], g2[p]) for p in g1)


def test_tiny_chain_all_16_subsets(tiny):
    g, exts, params, ref = tiny
    first = {}
    for variants_name, variants in (("lean", schedules.DEFAULT_VARIANTS), ("standard", schedules.STANDARD_VARIANTS)):
        for bits in itertools.product([0, 1], repeat=4):
            C = {b for b in range(4) if bits[b]}
            sch = schedules.tiny_chain_schedule(g, C, variants)
            want = osch.interpret(g.text(), sch.text())
            run = StepRunner(g.text(), sch.text(), exts, params, poison=True)
            peak = run.step()
            assert peak == want["peak"] <= run.plan.predicted_peak, (variants_name, C)
            assert abs(run.loss_value() - ref["loss"]) < ACT_TOL * abs(ref["loss"])
            got = run.grads_numpy()
            compare_grads(got, ref)
            # same operator variants, different checkpoint sets: identical bits
            if variants_name in first:
                assert all(np.array_equal(got[p], first[variants_name][p]) for p in got), (variants_name, C)
            else:
                first[variants_name] = got


def test_tiny_chain_schedules_of_the_integer_program(tiny):
    """Schedules chosen by the 0-1 program of Section 4 (per-tensor bits, per-operator variants, in-place
    recomputation) run like any other: peak as interpreted, within the budget the program was given, loss and
    gradients within tolerance of the oracle."""
    from workloads import ilp
    g, exts, params, ref = tiny
    store = M.Plan(g.text(), schedules.store_everything_schedule(g).text()).predicted_peak
    peaks = []
    for frac in (0.8, 0.6, 0.45):
        budget = int(frac * store)
        sch, obj, status = ilp.solve(g, budget, time_limit=120)
        assert sch is not None, status
        want = osch.interpret(g.text(), sch.text())
        run = StepRunner(g.text(), sch.text(), exts, params, poison=True)
        peak = run.step()
        assert peak == want["peak"] == run.plan.exact_peak <= run.plan.predicted_peak <= budget, frac
        assert abs(run.loss_value() - ref["loss"]) < ACT_TOL * abs(ref["loss"])
        compare_grads(run.grads_numpy(), ref)
        peaks.append(peak)
    assert peaks[0] > peaks[-1]


def test_tiny_chain_intermediates_and_masks(tiny):
    """Stop the step where tensors are still in memory and compare them with the oracle's."""
    g, exts, params, ref = tiny
    gt = g.text()
    sch = schedules.store_everything_schedule(g, schedules.DEFAULT_VARIANTS)
    run = StepRunner(gt, sch.text(), exts, params)
    trace = run.plan.trace()
    # last forward RUN event: every saved forward tensor is resident after it
    fwd_runs = [i for i, e in enumerate(trace) if e["kind"] == M.RUN_FWD]
    last = fwd_runs[-1]
    run.plan.set_stop_after(last)
    run.step()
    import torch
    torch.cuda.synchronize()
    checked = 0
    for n in g.nodes:
        off = run.plan.tensor_offset(last, n.id)
        if off < 0:
            continue
        if n.op == "mask":
            words = n.shape[0]
            got = run.read(off, (words,), torch.int64).view(np.uint64)
            assert np.array_equal(got, ref["aux"][n.id]), n.id          # bit-exact end to end
        elif n.op in ("bn", "relu", "conv"):
            got = run.read(off, n.shape)
            check_close(got, tensors.act_from_oracle(ref["acts"][n.id]), ACT_TOL, what=n.id)
        checked += 1
    assert checked >= 8
    for n in g.nodes:
        if n.op == "bn":
            C = n.shape[-1]
            st = run.read(run.plan.bn_stats_offset(n.id), (2 * C,))
            mean, invstd = ref["stats"][n.id]
            check_close(st[:C], mean, ACT_TOL, what=("mean", n.id))
            check_close(st[C:], invstd, ACT_TOL, what=("invstd", n.id))


def small_resnet():
    return graphs.resnet50(batch=4, hw=64, classes=16, widths=(16, 32, 32, 64), depths=(2, 2, 1, 1), stem=16)


def test_small_resnet_schedules_agree_with_oracle():
    g = small_resnet()
    exts, params = tensors.make_inputs(g, seed=2, gamma_beta="random")
    ref = oracle_step(g, exts, params)
    got_by_name = {}
    for name, sch in (("store_std", schedules.store_everything_schedule(g)),
                      ("store_lean", schedules.store_everything_schedule(g, schedules.DEFAULT_VARIANTS)),
                      ("blocks_lean", schedules.block_output_schedule(g))):
        want = osch.interpret(g.text(), sch.text())
        run = StepRunner(g.text(), sch.text(), exts, params, poison=True)
        peak = run.step()
        assert peak == want["peak"] <= run.plan.predicted_peak, name
        assert abs(run.loss_value() - ref["loss"]) < ACT_TOL * abs(ref["loss"]), name
        got_by_name[name] = run.grads_numpy()
        compare_grads(got_by_name[name], ref)
    # recomputation alone (same variants) must not change a single bit
    a, b = got_by_name["store_lean"], got_by_name["blocks_lean"]
    same = [np.array_equal(a[p], b[p]) for p in a]
    assert all(same), [p for p, s in enumerate(same) if not s]


@pytest.mark.parametrize("batch", [2, 8])
def test_resnet50_reduced_batch_against_oracle(batch):
    """The full ResNet-50 graph (224x224, 1000 classes) at the batches the fp64 oracle does in seconds.

    In a network this deep some ReLU inputs land closer to zero than fp32 can resolve, and one
    different sign bit moves a gradient tensor by about 1/sqrt(numel).  Both signs are valid there.
    The comparison checks that every sign bit of the GPU is the strict predicate of the GPU's own
    pre-activation, records for every bit that differs from the oracle's how far the oracle's value is
    from the kink (in units of the tensor's rms) and requires that distance to stay below DECISION_BAND;
    the oracle then goes on with the GPU's decision at those elements, and loss, BatchNorm outputs and
    gradients are compared at the stated tolerances.  Run with the default variants (F(4x4) Winograd
    on the sixteen 3x3 / stride-1 layers) and with every convolution on the implicit GEMM."""
    g = graphs.resnet50(batch=batch)
    exts, params = tensors.make_inputs(g, seed=0)
    gt = g.text()
    for vname, variants in (("default", schedules.DEFAULT_VARIANTS), ("igemm", schedules.IGEMM_VARIANTS)):
        ref, st, gpu_bn = oracle_with_gpu_decisions(g, exts, params, variants)
        print(f"resnet50 b{batch} {vname}: {st['differ']} of {st['total']} decisions differ, farthest from the kink "
              f"{st['max_dist']:.2e} rms (band {DECISION_BAND:.0e}); worst BatchNorm-output error {st['worst_act']:.2e} "
              f"normwise, {st['worst_act_maxabs']:.2e} rms element-wise")
        assert st["differ"] < 1e-4 * st["total"]
        sch = schedules.block_output_schedule(g, variants)
        run = StepRunner(gt, sch.text(), exts, params)
        peak = run.step()
        assert peak == run.plan.exact_peak <= run.plan.predicted_peak
        assert abs(run.loss_value() - ref["loss"]) < ACT_TOL * abs(ref["loss"])
        worst = compare_grads(run.grads_numpy(), ref)
        print(f"resnet50 b{batch} {vname}: worst gradient error {worst:.2e}")
        assert st["worst_act"] < DEEP_ACT_TOL and st["worst_act_maxabs"] < 50 * DEEP_ACT_TOL


def test_fused_neighbours_give_identical_bits():
    """The executor launches BN-apply/add + ReLU and ReLU-backward + BN-backward/add-backward as one
    kernel each; results must not differ from the one-kernel-per-operator path by a single bit."""
    small_mobilenet = graphs.mobilenet_v2(batch=2, hw=32, classes=10, stem=8, last=64,
                                          stages=((1, 8, 1, 1), (6, 12, 2, 2), (6, 16, 2, 2), (6, 24, 1, 1)))
    wide_resnet = graphs.resnet50(batch=2, hw=32, classes=10, widths=(64, 128), depths=(2, 1), stem=16)   # Winograd layers
    for g, sched in ((graphs.tiny_chain(), lambda g: schedules.tiny_chain_schedule(g, {0, 2})),
                     (small_resnet(), schedules.block_output_schedule),
                     (small_resnet(), schedules.store_everything_schedule),
                     (small_mobilenet, schedules.mobilenet_depthwise_schedule),      # recomputed depthwise conv + BatchNorm
                     (wide_resnet, schedules.block_output_schedule)):
        exts, params = tensors.make_inputs(g, seed=4, gamma_beta="random")
        sch = sched(g)
        run = StepRunner(g.text(), sch.text(), exts, params)
        n_fused = len(run.plan.launches())
        run.step()
        fused, loss_f = run.grads_numpy(), run.loss_value()
        run.plan.set_fusion(False)
        n_plain = len(run.plan.launches())
        assert n_fused < n_plain
        run.step()
        plain, loss_p = run.grads_numpy(), run.loss_value()
        assert loss_f == loss_p
        assert all(np.array_equal(fused[p], plain[p]) for p in fused)
        fused_list = StepRunner(g.text(), sch.text(), exts, params).plan.launches()
        labels = {l[0] for l in fused_list}
        assert labels & {"bn_relu_fwd", "bn_relu_apply", "relu_bn_bwd", "add_relu_fwd", "relu_add_bwd"}
    # the last two graphs recompute convolutions whose in-place BatchNorm goes into the convolution's kernel:
    # fewer BatchNorm apply launches than recomputed BatchNorm operators
    recomputed_bn = sum(1 for e in run.plan.trace_tuples() if e[0] == M.RUN_RECOMPUTE and g.nodes[e[2] - 1].op == "bn")
    apply_launches = sum(1 for l in fused_list if l[0] in ("bn_apply", "bn_relu_apply", "bn_add_relu_apply"))
    assert recomputed_bn > 0 and apply_launches < recomputed_bn


@pytest.mark.parametrize("n, h, w, c", [(1, 32, 32, 72), (1, 25, 41, 72), (1, 32, 32, 48), (1, 28, 28, 36), (1, 29, 28, 36), (2, 32, 32, 128), (1, 45, 46, 64)])
def test_fused_batchnorm_backward_of_few_rows_gives_identical_bits(n, h, w, c):
    """On either side of the lines between the kernels of BatchNorm's backward pass, which a residual block calls with the other branch's gradient to write or without, fused or not."""
    g = graphs.Graph()
    a = g.ext("x", "f32", (n, h, w, c))
    g.begin_block("before")
    a = g.relu(g.bn(g.conv(a, c, 1, name="before"), name="before.bn"))
    g.end_block()
    g.begin_block("block")
    b = g.relu(g.bn(g.conv(a, c, 1, name="first"), name="first.bn"))
    a = g.relu(g.add(g.bn(g.conv(b, c, 1, name="second"), name="second.bn"), a))
    g.end_block()
    g.sumloss(a)
    exts, params = tensors.make_inputs(g, seed=4, gamma_beta="random")
    run = StepRunner(g.text(), schedules.block_output_schedule(g).text(), exts, params)
    labels = {l[0] for l in run.plan.launches()}
    assert {"relu_bn_bwd", "relu_add_bn_bwd"} <= labels, labels
    run.step()
    fused = run.grads_numpy()
    run.plan.set_fusion(False)
    run.step()
    plain = run.grads_numpy()
    assert all(np.array_equal(fused[p], plain[p]) for p in fused)


def test_layers_with_a_workspace_and_one_range_cut_their_reduction_in_a_plan(monkeypatch):
    """Convolutions that declare a workspace with splits = 1 cut a reduction of few tiles by themselves.  Statistics, BatchNorm and ReLU that ride
    in the epilogue otherwise then follow it: the same bits with fused launches as one by one, and the loss and
    gradients of the plan without such workspaces to rounding (block by block the tolerance of all gradients)."""
    sched = lambda g: schedules.block_output_schedule(g, schedules.IGEMM_VARIANTS)
    make = lambda: graphs.resnet50(batch=2, hw=32, classes=10, widths=(64, 128), depths=(2, 1), stem=16)
    results = []
    for plan in (lambda rows, cols, red, classes=1, out=None: (1, 0),
                 lambda rows, cols, red, classes=1, out=None: (1, 16 * 4 * (rows * cols * classes if out is None else out))):
        monkeypatch.setattr(graphs, "conv_split_plan", plan)
        g = make()
        exts, params = tensors.make_inputs(g, seed=4, gamma_beta="random")
        run = StepRunner(g.text(), sched(g).text(), exts, params)
        run.step()
        fused, loss = run.grads_numpy(), run.loss_value()
        run.plan.set_fusion(False)
        run.step()
        plain = run.grads_numpy()
        assert run.loss_value() == loss and all(np.array_equal(fused[p], plain[p]) for p in fused)
        results.append((loss, fused))
    (loss0, grads0), (loss1, grads1) = results
    assert any(not np.array_equal(grads0[p], grads1[p]) for p in grads0), "no reduction was cut"
    assert abs(loss0 - loss1) < ACT_TOL * abs(loss0)
    for p in grads0:
        check_close(grads1[p], grads0[p], GRAD_TOL, what=p, floor=1e-2 * np.linalg.norm(grads0[max(p - 1, 0)]))


def test_steps_of_two_plans_overlap_on_two_streams():
    """Nothing is shared between plans: two of them, each stepped again and again by a thread of its own on a stream of its own, give
    the bits of their steps taken alone.  The convolutions of both run split reductions and Winograd layers at the same time."""
    import threading
    import torch
    cases = [(graphs.resnet50(batch=16, hw=64, classes=10, widths=(64, 128), depths=(2, 2), stem=64), schedules.block_output_schedule),
             (graphs.resnet50(batch=12, hw=64, classes=10, widths=(64, 96), depths=(2, 1), stem=32), schedules.store_everything_schedule)]
    runs, alone = [], []
    for seed, (g, sched) in enumerate(cases):
        exts, params = tensors.make_inputs(g, seed=seed, gamma_beta="random")
        run = StepRunner(g.text(), sched(g).text(), exts, params)
        peak = run.step()
        runs.append(run)
        alone.append((peak, run.grads_numpy(), run.loss_value()))
        for t in run.grads:
            t.fill_(float("nan"))
    torch.cuda.synchronize()
    peaks = [set(), set()]

    def work(i):
        stream = torch.cuda.Stream()
        for _ in range(20):
            peaks[i].add(runs[i].step(stream))
        stream.synchronize()
    threads = [threading.Thread(target=work, args=(i,)) for i in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for run, (peak, grads, loss), seen in zip(runs, alone, peaks):
        assert seen == {peak}
        got = run.grads_numpy()
        assert run.loss_value() == loss
        assert all(np.array_equal(got[p], grads[p]) for p in grads)


def test_recomputed_relu_rides_in_the_convolution_epilogue_when_its_mask_is_kept():
    """A schedule that keeps block outputs and every ReLU's 1-bit sign mask: the recomputed convolution -> BatchNorm -> ReLU
    chains then write no mask, and the executor runs each as one launch (BatchNorm apply and ReLU in the convolution's
    epilogue, the ReLU's result beside the BatchNorm's where that is still needed).  Fewer launches than one by one,
    the same bits with fusion on and off and as the block-output schedule, the oracle's gradients."""
    g = graphs.resnet50(batch=2, hw=64, classes=10, widths=(16, 32, 64, 64), depths=(2, 2, 1, 1), stem=16)
    exts, params = tensors.make_inputs(g, seed=5, gamma_beta="random")
    masks = {n.id for n in g.nodes if g.is_aux(n.id) and g.nodes[n.ins[0] - 1].op in ("relu", "relu6")}
    F = schedules.block_output_set(g)
    grads, alone = {}, {}
    for name, saved in (("blocks", F), ("blocks+masks", F | masks)):
        sch = schedules.schedule_for_saved_set(g, saved)
        for fusion in (True, False):
            run = StepRunner(g.text(), sch.text(), exts, params)
            run.plan.set_fusion(fusion)
            launches = run.plan.launches()
            labels = [l[0] for l in launches]
            # channel counts of the ReLUs that are recomputed as launches of their own
            alone[(name, fusion)] = sorted(g.nodes[l[2] - 1].shape[-1] for l in launches if l[0] == "relu_fwd" and l[1] == 3)
            peak = run.step()
            assert peak == run.plan.exact_peak == osch.interpret(g.text(), sch.text())["peak"]
            grads[(name, fusion)] = (run.grads_numpy(), labels.count("relu_fwd"), len(labels))
            del run
    # with the masks kept, the recomputed ReLUs are gone from the fused program
    assert grads[("blocks+masks", True)][1] < grads[("blocks+masks", False)][1]
    assert grads[("blocks+masks", True)][1] < grads[("blocks", True)][1]
    # without the masks kept, a recomputed ReLU writes its mask again: it rides in the epilogue as well where a word of the
    # mask is 64 channels of one position (the 64-channel layers of this network), and stays a launch elsewhere
    assert any(c % 64 == 0 for c in alone[("blocks", False)]) and alone[("blocks", True)]
    assert all(c % 64 != 0 for c in alone[("blocks", True)])
    ref = grads[("blocks", False)][0]
    for key, (got, _, _) in grads.items():
        assert all(np.array_equal(got[p], ref[p]) for p in ref), key
