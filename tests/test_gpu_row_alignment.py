"""Rows of every length modulo the vector width, against the CPU oracle.

Rows start at any element (row m at m P): the step takes the buffers as flat
arrays and the averaging kernels take vectors at unaligned addresses, so what
can go wrong is the last partial vector of a row or buffer, the clip factor
where a wave's elements cross a row end (rows of 256 elements and more) or
several (shorter rows), and the launch of more than 64 MB, which limits the
workgroups per CU.  Each case runs the separate and the fused calls over a
schedule in which every state is averaged, compares every element with the
oracle at the suite's tolerances and the two with each other bit for bit.
"""

import pytest
import torch

import synth
from gpu_harness import compare, free, log, run_gpu, run_oracle, run_oracle_parallel

pytestmark = pytest.mark.gpu

BASE = {"adam": "adam_n3_k4_p16m", "adopt": "adopt_n2_k8_p124m_bf16", "sgdm": "sgdm_n2_k16_p354m_clip"}


def _workload(form, P, K, x="f32", g="f32", clip=1.0, steps=8):
    b = synth.WORKLOADS[BASE[form]]
    return b.replace(tensors=(synth.TensorSpec("t", P, "matrix"),), replicas=K, steps=steps, param_dtype=x,
                     grad_dtype=g, clip_rho=0.0 if form == "adopt" else clip, period_x=2,
                     period_u=(4,) * b.n_moments, period_v=3)


def _check(w, label, oracle_run=run_oracle):
    log(f"case {label}")
    steps = list(range(1, w.steps + 1))
    sep, fused, ref = run_gpu(w, steps), run_gpu(w, steps, fused=True), oracle_run(w, steps)
    assert sep.masks == fused.masks == ref.masks and any(sep.masks)
    compare(w, sep.opt, ref, label)
    for p, q in zip(sep.opt.states(), fused.opt.states()):
        assert torch.equal(p, q)
    free(sep, fused)


@pytest.mark.parametrize("P", [2, 6, 251, 255, 256, 257, 258, 259, 515, 1027, 2049, 4098])
@pytest.mark.parametrize("form,K,x,g", [("adam", 3, "f32", "f32"), ("sgdm", 16, "f32", "bf16"),
                                        ("adopt", 8, "bf16", "bf16"), ("adam", 5, "bf16", "f32"),
                                        ("sgdm", 24, "f32", "f32")])
def test_row_lengths(form, K, x, g, P):
    _check(_workload(form, P, K, x, g), f"rows-{form}-{K}-{x}-{g}-{P}")


@pytest.mark.parametrize("K", [12, 16])
def test_every_state_staged(K):
    """Five due states of 12 and 16 replicas exchanged at once (s = 12): the
    largest LDS request of the suite's forms, 80 KiB."""
    _check(_workload("adam", 1027, K, steps=12), f"staged-{K}")


@pytest.mark.parametrize("form,K,P,x", [("adam", 3, 1_500_003, "f32"), ("sgdm", 8, 1_000_005, "bf16")])
def test_limited_residency(form, K, P, x):
    """More than 64 MB loaded per launch."""
    _check(_workload(form, P, K, x, x, steps=4), f"resident-{form}-{K}-{P}", run_oracle_parallel)
