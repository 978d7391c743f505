"""Records into the ring and out of it, byte for byte against the oracle's ring, at the edges of the copy kernels' tiles:
trajectories and time steps around a tile, records from one element to too long for a tile, every storage variant."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_common import oracle_inputs, say, shape_workload, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_1912_00167_amd import binding
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    binding.load()
    return torch, binding


# dist, T, trajectories, A, storage
SHAPES = [("categorical", 31, 63, 4, "f32"), ("categorical", 32, 64, 18, "f32"), ("categorical", 33, 65, 7, "bf16"), ("categorical", 1, 1, 2, "bf16"),
          ("categorical", 9, 17, 128, "f32"), ("categorical", 9, 15, 129, "bf16"), ("categorical", 3, 9, 1024, "f32"), ("categorical", 3, 5, 1025, "bf16"),
          ("gaussian", 24, 130, 17, "bf16"), ("gaussian", 25, 8, 17, "f32"), ("gaussian", 47, 7, 1, "bf16"), ("gaussian", 70, 100, 3, "f32"),
          ("gaussian", 100, 1500, 6, "f32"), ("gaussian", 65, 1030, 5, "bf16"), ("categorical", 100, 3000, 18, "f32"), ("categorical", 67, 1300, 9, "bf16")]


@pytest.mark.parametrize("dist,T,n,A,storage", SHAPES)
@pytest.mark.parametrize("variant", ["plain", "cached", "u8"])
def test_round_trip(env, dist, T, n, A, storage, variant):
    torch, binding = env
    u8 = variant == "u8"
    if u8 and (dist == "gaussian" or A > 256):
        pytest.skip("one-byte indices: categorical, at most 256 actions")
    N = n + n // 2 + 3
    wl = shape_workload(workloads.C2 if dist == "categorical" else workloads.C3, T=T, A=A, B=n, num_slots=N, K=1, storage=storage)
    say(f"case ring moves {dist} T={T} n={n} A={A} {storage} {variant}")
    flags = {"plain": 0, "cached": binding.IMPACT_BUFFER_CACHE_LOGP, "u8": binding.IMPACT_BUFFER_ACTIONS_U8}[variant]
    buf = binding.Buffer(dist, T, A, N, 1, storage, flags=flags)
    for rnd in range(2):                                     # the second round wraps around: two runs of slots
        x = workloads.make_trajectories(wl, n, stream=rnd + A)
        d = to_device(x, torch)
        if u8:
            d["actions"] = d["actions"].to(torch.uint8)
        with_target = rnd == 0
        slots = binding.impact_buffer_insert(buf, {k: d[k] for k in ("worker", "actions", "rewards", "dones") + (("target",) if with_target else ())})
        if not with_target:                                  # appended later, in an order of its own
            order = np.random.default_rng(A).permutation(n)[: min(n, 40)]
            rest = np.setdiff1d(np.arange(n), order)
            for part in (order, rest):
                if len(part):
                    binding.impact_buffer_put_target(buf, slots[part], d["target"][:, torch.from_numpy(part).cuda()].contiguous())
        perm = np.random.default_rng(rnd).permutation(n)
        got = binding.impact_buffer_gather(buf, torch.from_numpy(np.ascontiguousarray(slots[perm])).cuda())
        torch.cuda.synchronize()
        xi = workloads.take_trajectories(x, perm)
        want = dict(oracle_inputs(xi, storage))
        for k in ("target", "rewards", "dones") + (("worker",) if variant != "cached" else ()) + ("actions",):
            g = got[k].float().cpu().numpy() if got[k].dtype == torch.bfloat16 else got[k].cpu().numpy()
            assert g.shape == want[k].shape and np.array_equal(g, want[k].astype(g.dtype)), (k, rnd)
        if variant == "cached":
            lp = oracle.behaviour_logp(dist, xi["target"], xi["worker"], want["actions"])
            np.testing.assert_allclose(got["logp"].cpu().numpy(), lp, rtol=1e-12, atol=1e-12)
        binding.impact_buffer_sample(buf, n)
        binding.impact_buffer_release_discarded(buf)
    buf.close()
