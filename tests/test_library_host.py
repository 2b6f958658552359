"""Host-side checks of libdds that need no GPU: the library loads, exports every
symbol the header declares, its integer schedule equals the oracle's closed forms,
and spec validation / arena sizing behave."""
import os
import re

import numpy as np
import pytest

import paper_2509_05679_amd as P
from dds_inputs import workload, WORKLOAD_NAMES
from dds_inputs.configs import tiny_mlp, tiny_resnet
from oracle import fdg

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_declared_symbol_is_exported():
    header = open(os.path.join(ROOT, "include", "dds.h")).read()
    declared = set(re.findall(r"\b(dds_[a-z_]+)\s*\(", header))
    assert declared == set(P.EXPORTS)
    for name in declared:
        assert hasattr(P.lib, name), name


def _sched_row(rec):
    """The oracle's schedule record in the order of dds_schedule's DDS_SCHED_INTS integers."""
    return [rec[k] for k in ("f", "b", "ring_depth", "fwd_slot", "bwd_slot", "err_read", "err_write", "label_slot",
                             "in_fwd_slot", "in_bwd_slot", "label_bwd_slot", "snap_write", "label_write")]


@pytest.mark.parametrize("K", range(1, 9))
def test_schedule_is_bit_exact_against_the_oracle(K):
    for t in range(64):
        got = P.dds_schedule(K, None, t)
        for rec in fdg.schedule(t, K):
            k0 = rec["k0"]
            assert got[k0].tolist() == _sched_row(rec), (K, t, k0)


@pytest.mark.parametrize("K,d", [(3, [4, 2, 0]), (3, [3, 1, 0]), (4, [5, 4, 2, 1]), (2, [3, 1])])
def test_schedule_with_custom_delays(K, d):
    for t in range(40):
        got = P.dds_schedule(K, d, t)
        for rec in fdg.schedule(t, K, d):
            k0 = rec["k0"]
            assert got[k0].tolist() == _sched_row(rec), (K, d, t, k0)


def test_schedule_rejects_acausal_delays():
    with pytest.raises(P.DdsError) as e:
        P.dds_schedule(3, [1, 1, 0], 0)
    assert e.value.code == P.DDS_EINVAL
    with pytest.raises(P.DdsError):
        P.dds_schedule(2, [1, -1], 0)


@pytest.mark.parametrize("name", WORKLOAD_NAMES)
def test_arena_sizing_of_the_benchmark_configs(name):
    wl = workload(name)
    n = P.dds_arena_bytes(P.Spec.from_workload(wl), wl.K, wl.W)
    assert 0 < n < 200 * 2 ** 30
    half = workload(name, B=wl.B // 2)
    assert P.dds_arena_bytes(P.Spec.from_workload(half), wl.K, wl.W) < n


def test_recompute_policy_shrinks_the_arena_of_delayed_modules_only():
    """Recompute keeps one input and one output per ring slot instead of every saved tensor; a net whose only
    module has d = 0 keeps nothing across iterations, so the policy changes nothing there."""
    for name in ("cfg1_cnn", "cfg2_resnet18", "cfg3_resnet56", "cfg4_resnet34w"):
        wl = workload(name)
        store = P.dds_arena_bytes(P.Spec.from_workload(wl), wl.K, wl.W)
        rec = P.dds_arena_bytes(P.Spec.from_workload(wl, activations="recompute"), wl.K, wl.W)
        assert rec < 0.7 * store, (name, store, rec)
    from dds_inputs.configs import tiny_resnet
    one = tiny_resnet(K=1)
    assert P.dds_arena_bytes(P.Spec.from_workload(one), 1, one.W) == \
        P.dds_arena_bytes(P.Spec.from_workload(one, activations="recompute"), 1, one.W)
    bad = P.Spec.from_workload(one)
    bad.c.activations = 7
    with pytest.raises(P.DdsError) as e:
        P.dds_arena_bytes(bad, 1, one.W)
    assert e.value.code == P.DDS_EINVAL


def test_paper_experiment_workloads_are_resnet20():
    from dds_inputs.configs import PAPER_WORKLOAD_NAMES
    assert set(PAPER_WORKLOAD_NAMES) == {"paper_r20_S1K1", "paper_r20_S1K2", "paper_r20_S4K1", "paper_r20_S4K2"}
    for name in PAPER_WORKLOAD_NAMES:
        wl = workload(name)
        convs = [o for o in wl.ops if o["op"] == "conv"]
        shortcuts = [o for o in wl.ops if o["op"] == "res_add" and o["shortcut"]]
        assert len(convs) + 1 == 20 and len(shortcuts) == 2  # 19 convs + 1 linear; two projection blocks
        assert wl.B == 194 and wl.K == len(wl.bounds) - 1 and wl.W in (1, 4)
        assert P.dds_arena_bytes(P.Spec.from_workload(wl), wl.K, wl.W) > 0


def _spec(ops, bounds, in_shape=(3, 8, 8), precision="f32"):
    return P.Spec(ops, bounds, in_shape, 10, 4, precision, 0.1, 0.0)


def test_spec_validation_errors():
    good = tiny_resnet(K=2)
    P.dds_arena_bytes(P.Spec.from_workload(good), 2, 2)
    # channel mismatch
    ops = [dict(op="conv", cin=4, cout=8, k=3, stride=1, pad=1), dict(op="relu"), dict(op="gap"),
           dict(op="linear", cin=8, cout=10), dict(op="softmax_ce")]
    with pytest.raises(P.DdsError) as e:
        P.dds_arena_bytes(_spec(ops, [0, 5]), 1, 1)
    assert e.value.code == P.DDS_EINVAL
    # missing loss
    ops2 = [dict(op="conv", cin=3, cout=8, k=3, stride=1, pad=1), dict(op="relu")]
    with pytest.raises(P.DdsError):
        P.dds_arena_bytes(_spec(ops2, [0, 2]), 1, 1)
    # linear on a spatial tensor is not covered
    ops3 = [dict(op="linear", cin=3, cout=10), dict(op="softmax_ce")]
    with pytest.raises(P.DdsError) as e:
        P.dds_arena_bytes(_spec(ops3, [0, 2]), 1, 1)
    assert e.value.code == P.DDS_EUNSUPPORTED
    # module boundary inside a residual block
    wl = tiny_resnet(K=2)
    with pytest.raises(P.DdsError):
        P.dds_arena_bytes(P.Spec(wl.ops, [0, 4, len(wl.ops)], wl.in_shape, 10, 4, "f32", 0.1, 0.0), 2, 1)
    # W out of range, bad bounds
    with pytest.raises(P.DdsError):
        P.dds_arena_bytes(P.Spec.from_workload(good), 2, 33)
    with pytest.raises(P.DdsError):
        P.dds_arena_bytes(P.Spec(good.ops, [0, 3, 3], good.in_shape, 10, 4, "f32", 0.1, 0.0), 2, 1)


def test_mixing_matrix_validation_and_arena_growth():
    from dds_inputs.configs import complete_mixing, ring_mixing
    wl = tiny_resnet(K=2, W=4)
    shared = P.dds_arena_bytes(P.Spec.from_workload(wl), 2, 4)
    own = P.dds_arena_bytes(P.Spec.from_workload(wl, ring_mixing(4, 0.3)), 2, 4)
    assert own > shared  # W weight copies, momenta and snapshot rings instead of one
    assert P.dds_arena_bytes(P.Spec.from_workload(wl, complete_mixing(4)), 2, 4) == own
    ring = np.array(ring_mixing(4, 0.3))
    assert np.allclose(ring.sum(0), 1) and np.allclose(ring.sum(1), 1) and np.array_equal(ring, ring.T)
    assert np.array_equal(ring, fdg.gossip_matrix(4, [(0, 1), (1, 2), (2, 3), (3, 0)], 0.3).numpy())
    bad_rows = ring.copy(); bad_rows[0, 0] += 0.1
    asym = ring.copy(); asym[0, 1] += 0.1; asym[0, 0] -= 0.1
    neg = np.array(ring_mixing(4, 0.6))  # diagonal 1 - 1.2 < 0
    for bad in (bad_rows, asym, neg):
        with pytest.raises(P.DdsError) as e:
            P.dds_arena_bytes(P.Spec.from_workload(wl, bad), 2, 4)
        assert e.value.code == P.DDS_EINVAL


def test_no_gpu_means_a_loud_failure_not_a_fallback():
    import torch
    if torch.cuda.is_available():
        pytest.skip("GPU present")
    wl = tiny_mlp()
    with pytest.raises(RuntimeError):
        P.Trainer(P.Spec.from_workload(wl), wl.W)


def test_step_size_rules_against_printed_values_and_oracle():
    gold = os.path.join(ROOT, "tests", "golden", "step_size_strategies.txt")
    rules = {"constant": P.DDS_ETA_CONSTANT, "piecewise": P.DDS_ETA_PIECEWISE, "diminishing": P.DDS_ETA_DIMINISHING}
    n = 0
    for line in open(gold):
        if not line.strip() or line.startswith("#"):
            continue
        rule, t, eta = line.split()
        got = P.dds_step_size(rules[rule], int(t), 0.1)
        assert got == pytest.approx(float(eta), rel=1e-6), (rule, t)
        assert got == pytest.approx(fdg.step_size(rule, int(t), 0.1), rel=1e-6)
        n += 1
    assert n >= 14
    assert np.isnan(P.dds_step_size(99, 0, 0.1)) and np.isnan(P.dds_step_size(P.DDS_ETA_CONSTANT, -1, 0.1))


def test_batchnorm_spec_validation_and_arena():
    from dds_inputs.configs import BN_WORKLOAD_NAMES
    for name in BN_WORKLOAD_NAMES:
        wl = workload(name)
        plain = workload(name[:-3])
        with_bn = P.dds_arena_bytes(P.Spec.from_workload(wl), wl.K, wl.W)
        assert with_bn > P.dds_arena_bytes(P.Spec.from_workload(plain), plain.K, plain.W)
    conv = dict(op="conv", cin=3, cout=8, k=3, stride=1, pad=1)
    tail = [dict(op="gap"), dict(op="linear", cin=8, cout=10), dict(op="softmax_ce")]
    ok = [conv, dict(op="bn", c=8, eps=1e-5), dict(op="relu")] + tail
    P.dds_arena_bytes(_spec(ok, [0, len(ok)]), 1, 2)
    # wrong channel count, eps missing, normalisation not behind a convolution
    for bad, code in (([conv, dict(op="bn", c=4, eps=1e-5), dict(op="relu")] + tail, P.DDS_EINVAL),
                      ([conv, dict(op="bn", c=8, eps=0.0), dict(op="relu")] + tail, P.DDS_EINVAL),
                      ([conv, dict(op="relu"), dict(op="bn", c=8, eps=1e-5)] + tail, P.DDS_EUNSUPPORTED)):
        with pytest.raises(P.DdsError) as e:
            P.dds_arena_bytes(_spec(bad, [0, len(bad)]), 1, 2)
        assert e.value.code == code


_DEVICE_ONCE = r"""
#include "device_once.h"
#include <cstdio>
#include <thread>
#include <vector>
int main() {
  dds::DeviceOnce once;
  std::atomic<int> runs[3] = {{0}, {0}, {0}};
  auto act = [&](int d) { return once(d, [&, d] { ++runs[d]; return true; }); };
  if (!act(0) || !act(0) || runs[0] != 1) return 1;             // once on a device
  if (!act(1) || runs[1] != 1 || !act(0) || runs[0] != 1) return 2;  // and once on the next one
  int tries = 0;
  auto fails_first = [&] { return ++tries > 1; };
  if (once(2, fails_first) || !once(2, fails_first) || !once(2, fails_first) || tries != 2) return 3;
  if (!once(64, fails_first) || !once(64, fails_first) || tries != 4) return 4;  // no bit of its own
  dds::DeviceOnce shared;
  std::atomic<int> done{0};
  std::vector<std::thread> threads;
  for (int i = 0; i < 16; ++i)
    threads.emplace_back([&, i] { if (shared(i % 4, [&] { return true; })) ++done; });
  for (auto& t : threads) t.join();
  return done == 16 ? 0 : 5;
}
"""


def test_device_once_runs_on_every_device_and_again_after_a_failure(tmp_path):
    # what raises the LDS limit of a kernel: per device and not per process, and not forgotten when it fails
    import subprocess
    src = tmp_path / "once.cpp"
    src.write_text(_DEVICE_ONCE)
    exe = tmp_path / "once"
    subprocess.run(["g++", "-std=c++17", "-pthread", "-I", os.path.join(ROOT, "paper_2509_05679_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    assert subprocess.run([str(exe)]).returncode == 0


_WGRAD_PLANS = r"""
#include <cstdio>
#include "kernels.h"
using namespace dds;
static const int zeros = 0;
static WgradParams layer(int cin, int cout, int hw, int images, int nrep) {
  WgradParams w{};
  w.zeros = &zeros;
  w.Nimg = images; w.H = w.Ho = w.W = w.Wo = hw; w.Cx = cin; w.Mout = w.ldy = cout;
  w.R = w.S = 3; w.stride = w.pad = 1; w.NK = 9 * cin; w.P = images * hw * hw; w.nrep = nrep; w.alpha = 1.f;
  return w;
}
int main() {
  // splits of the two 16-channel layers of a net of 16 x 16 images: the mean of 63, 64, 255 and 256 (two images a split: 448 workgroups), a mixing step of 7, 8, 31 and 32 a data-group
  const int images[8][2] = {{63, 1}, {64, 1}, {255, 1}, {256, 1}, {14, 2}, {24, 3}, {62, 2}, {160, 5}};
  for (auto& c : images) {
    const WgradParams two[2] = {layer(16, 16, 16, c[0], c[1]), layer(16, 16, 16, c[0], c[1])};
    int q[2];
    wgrad_choose_splits(DT_BF16, two, 2, true, q);
    printf("%d %d ", q[0], q[1]);
  }
  for (int n : {8, 9, 64, 65}) {  // ... and of one layer of 16 or 32 input channels
    int q[2];
    const WgradParams a = layer(16, 16, 16, n, 1), b = layer(32, 32, 16, n, 1);
    wgrad_choose_splits(DT_BF16, &a, 1, true, q);
    wgrad_choose_splits(DT_BF16, &b, 1, true, q + 1);
    printf("%d %d ", q[0], q[1]);
  }
  // a layer that has its launch to itself: workgroups for the whole chip, in 64 x 64 blocks, or for half of it beside other modules; a stride-2 layer of rows so long that one workgroup takes a CU: two rounds
  int alone[3];
  WgradParams stem = layer(8, 256, 32, 62, 1), wide = layer(128, 128, 512, 2, 1);
  wgrad_choose_splits(DT_BF16, &stem, 1, true, alone);
  wgrad_choose_splits(DT_BF16, &stem, 1, false, alone + 2);
  wide.stride = 2; wide.Ho = wide.Wo = 256; wide.P /= 4;
  wgrad_choose_splits(DT_BF16, &wide, 1, true, alone + 1);
  printf("%d %d %d ", 4 * alone[0], 4 * alone[2], 16 * alone[1]);
  // refused before anything is launched: a layer of another kernel, more splits than tiles, splits that are not equal
  WgradParams uneven = layer(64, 64, 16, 8, 1);
  uneven.R = uneven.S = 5; uneven.pad = 2; uneven.NK = 25 * 64; uneven.nsplit = 3; uneven.pix_per_split = uneven.P / 3;
  WgradParams mixed[2] = {layer(64, 64, 16, 8, 1), uneven};
  mixed[0].nsplit = mixed[1].nsplit = 8;
  mixed[0].pix_per_split = mixed[1].pix_per_split = uneven.P / 8;
  WgradParams many = layer(16, 16, 16, 1, 1);
  many.nsplit = 3;
  many.pix_per_split = many.P / 3;
  printf("%d %d %d\n", launch_wgrad(DT_BF16, mixed, 2, nullptr), launch_wgrad(DT_BF16, &many, 1, nullptr), launch_wgrad(DT_BF16, &uneven, 1, nullptr));
}
"""


def test_split_counts_of_narrow_layers_and_refused_weight_gradients(tmp_path):
    # the counts that the GPU tests of the update by split count name, and no launch that drops a layer or some of its pixels
    import subprocess
    pkg = os.path.join(ROOT, "paper_2509_05679_amd")
    src = tmp_path / "plans.cpp"
    src.write_text(_WGRAD_PLANS)
    exe = tmp_path / "plans"
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(pkg, "csrc"), str(src), "-o", str(exe),
                    os.path.join(pkg, "libdds.so"), "-Wl,-rpath," + pkg, "-L/opt/rocm/lib", "-Wl,-rpath,/opt/rocm/lib", "-lamdhip64"], check=True)
    out = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True, timeout=60, check=True).stdout.split()
    splits = [63, 64, 128, 128, 14, 24, 62, 160, 8, 9, 64, 65]
    assert [int(v) for v in out] == [v for q in splits for v in (q, q)] + [248, 124, 512, -1, -1, -1]


def test_no_kernel_attribute_is_remembered_per_process():
    csrc = os.path.join(ROOT, "paper_2509_05679_amd", "csrc")
    for name in os.listdir(csrc):
        text = open(os.path.join(csrc, name)).read()
        assert not re.search(r"static\s+bool", text), name
        assert text.count("hipFuncSetAttribute(") <= (1 if name == "gemm.hip" else 0), name
