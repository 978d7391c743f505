"""GPU parity of the register-resident loss kernels (any number of actions, layout and batch size) where their shape
rules change: lanes per step, elements per lane, trajectories and chunks per workgroup, padding of the scan."""
from dataclasses import replace

import numpy as np
import pytest

import oracle
import workloads
from gpu_common import check_against_oracle, gpu_loss, say, shape_workload, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_1912_00167_amd import binding
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    binding.load()
    return torch, binding


SHAPES = [
    # records: one element, one lane, lanes that share elements, the longest per count of lanes, the longest of all and one more
    ("categorical", 9, 3, 1), ("categorical", 9, 5, 5), ("categorical", 9, 5, 13), ("categorical", 9, 5, 47), ("categorical", 9, 5, 48),
    ("categorical", 9, 5, 49), ("categorical", 5, 3, 257), ("categorical", 5, 3, 512), ("categorical", 5, 3, 513),
    ("gaussian", 9, 3, 1), ("gaussian", 9, 5, 7), ("gaussian", 9, 5, 11), ("gaussian", 9, 5, 49), ("gaussian", 3, 3, 512), ("gaussian", 3, 3, 513),
    # trajectories per workgroup (1, 2, 4, 8) with a ragged last one
    ("categorical", 20, 383, 7), ("categorical", 20, 385, 7), ("gaussian", 20, 771, 5), ("categorical", 11, 1025, 7), ("gaussian", 11, 1027, 2),
    # one chunk just filled, one row more, many chunks, several workgroups per compute unit
    ("categorical", 1024, 2, 3), ("categorical", 1025, 2, 3), ("gaussian", 256, 3, 22), ("gaussian", 257, 3, 22), ("categorical", 700, 5, 300),
    ("categorical", 67, 4101, 5), ("gaussian", 35, 4099, 10), ("categorical", 37, 1030, 100),
]


@pytest.mark.parametrize("dist,T,Bn,A", SHAPES)
def test_shapes(env, dist, T, Bn, A):
    """Time-major; the same batch from a bf16 buffer through slots in no order with every learner tensor batch-major."""
    torch, binding = env
    base = workloads.C2 if dist == "categorical" else workloads.C3
    base = replace(base, hyper=replace(base.hyper, kl_coeff=0.5))
    wl = shape_workload(base, T=T, B=Bn, A=A, num_slots=Bn + 3, storage="f32")
    say(f"case lanes {dist} T={T} B={Bn} A={A}")
    x = workloads.make_trajectories(wl, Bn + 3, stream=T + Bn + A)
    slots = np.random.default_rng(A).permutation(Bn + 3)[:Bn].astype(np.int32)
    xb = workloads.take_trajectories(x, slots)
    d = to_device(xb, torch)
    out = binding.impact_loss_fwd_bwd(dist, d["learner"], d["values"], d["bootstrap"], d, binding.config_from_hyper(wl.hyper, 1))
    torch.cuda.synchronize()
    check_against_oracle(wl, xb, {k: v.cpu().numpy() for k, v in out.items()}, label="time-major")

    wl = replace(wl, storage="bf16")
    buf = binding.Buffer(dist, T, A, Bn + 3, 2, "bf16")
    binding.impact_buffer_insert(buf, to_device(x, torch))
    learner = d["learner"].to(torch.bfloat16)
    xb["learner"] = oracle.quantize_bf16(xb["learner"])[1]
    out = binding.impact_loss_fwd_bwd_from_buffer(buf, torch.from_numpy(slots).cuda(), learner.transpose(0, 1).contiguous(),
                                                  d["values"].t().contiguous(), d["bootstrap"],
                                                  binding.config_from_hyper(wl.hyper, binding.IMPACT_FLAG_BATCH_MAJOR))
    torch.cuda.synchronize()
    got = {k: out[k].transpose(0, 1).contiguous().cpu().numpy() for k in ("grad_dist", "grad_values", "vs", "adv")}
    got.update(loss5=out["loss5"].cpu().numpy(), fractions=out["fractions"].cpu().numpy())
    check_against_oracle(wl, xb, got, label="batch-major from the buffer")
    buf.close()


@pytest.mark.parametrize("mask", [-1e9, float(np.finfo(np.float32).min)], ids=["1e9", "lowest"])
def test_masked_actions(env, mask):
    """Actions that no policy can take, marked by logits far below the others': probability and gradient are zero."""
    torch, binding = env
    wl = shape_workload(workloads.C2, T=12, B=21, A=7, storage="f32")
    say(f"case lanes masked logits {mask}")
    x = workloads.make_batch(wl, stream=3)
    for k in ("worker", "target", "learner"):
        x[k][..., 5:] = mask
    x["actions"] = (x["actions"] % 5).astype(np.int32)
    d = to_device(x, torch)
    out = binding.impact_loss_fwd_bwd(wl.dist, d["learner"], d["values"], d["bootstrap"], d, binding.config_from_hyper(wl.hyper, 1))
    torch.cuda.synchronize()
    check_against_oracle(wl, x, {k: v.cpu().numpy() for k, v in out.items()}, label="masked")
    assert not out["grad_dist"][..., 5:].any()


# on both sides of each line at which a specialised record changes from the pipeline to these kernels: the number of
# trajectories, one chunk of the pipeline and more, short and long trajectories on few compute units
ROUTES = [("categorical", 33, 1024, 18), ("categorical", 33, 1032, 18), ("categorical", 16, 40, 18), ("categorical", 17, 40, 18),
          ("categorical", 32, 24, 6), ("categorical", 33, 24, 6), ("gaussian", 20, 192, 6), ("gaussian", 20, 200, 6), ("gaussian", 188, 12, 17),
          ("gaussian", 189, 12, 17), ("categorical", 355, 40, 18), ("categorical", 356, 40, 18), ("categorical", 600, 192, 18)]


@pytest.mark.parametrize("dist,T,Bn,A", ROUTES)
def test_specialised_records(env, dist, T, Bn, A):
    torch, binding = env
    base = workloads.C2 if dist == "categorical" else workloads.C3
    wl = shape_workload(replace(base, hyper=replace(base.hyper, kl_coeff=0.5)), T=T, B=Bn, A=A, storage="f32")
    say(f"case lanes route {dist} T={T} B={Bn} A={A}")
    x = workloads.make_batch(wl, stream=T + Bn)
    got = gpu_loss(torch, binding, wl, x)
    check_against_oracle(wl, x, got, label=f"{dist} T{T} B{Bn} A{A}")
