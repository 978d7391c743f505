"""Performance cases of the IMPACT learner's hot path: what a training program calls once per SGD step, or once per
batch of trajectories that its workers send.

A case names one of five operations, each a sequence of public calls of ``paper_1912_00167_amd.binding``:

  "step"    sample B trajectories from the ring, loss and gradients read from the ring in place
            (slots "ring": the slots as sampled, in page-locked host memory; "scattered": a device tensor of slots
            in no order, as a learner that shuffles its minibatches passes them)
  "batch"   loss and gradients on a batch that is at hand time-major (on-policy data, or gathered before)
  "insert"  B finished trajectories enter the ring with the target network's output, and are handed out once
  "gather"  B trajectories are copied out of the ring into time-major tensors
  "loop"    the learner loop of Algorithm 1 over one filling of the ring: the workers' fragments arrive (without
            target output), then every minibatch is traversed K = 2 times: at the first traversal the target's output is
            appended, at each the loss and its gradients are computed and a learner step is counted

The listed shapes are the repository's workloads (``workloads/``: C1-C5), the appendix tables' own batches, and shapes of
the same sizes without a favourable divisor.
"""
from __future__ import annotations

import math

import torch

from paper_1912_00167_amd import binding

CATEGORICAL, GAUSSIAN = "categorical", "gaussian"

# dist, T, B, A: the policy's distribution, steps per trajectory, trajectories per batch, actions / action dimensions.
# storage: element type of the ring's float fields (and of a time-major batch's).
DEFAULTS = dict(op="step", dist=CATEGORICAL, T=50, B=512, A=18, storage="f32", slots="ring",
                cached=False,          # the ring keeps log pi(a) of worker and target instead of the worker's distribution
                kl=False,              # KL term (a cached ring then keeps the target's distribution)
                actions_u8=False,      # one-byte action indices
                learner_bf16=False,    # the learner network runs under mixed precision
                batch_major=False,     # learner-side tensors [B][T][..], as a recurrent network produces them
                packed=False,          # per-step outputs as one record per step
                fragment=0)            # "loop": trajectories per insert


def case(name, **kw):
    c = dict(DEFAULTS, name=name)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest calls: a toy discrete task; one training batch of the discrete table (500 steps in fragments of 50)
        case("step_discrete_tiny", T=20, B=32, A=6),
        case("step_discrete_table", T=50, B=10, A=18, actions_u8=True),
        # an ordinary discrete learner, 25600 steps
        case("step_discrete_mid", T=50, B=512, A=18),
        # a large discrete learner, fp32 throughout
        case("step_discrete_large", T=100, B=8192, A=18),
        # an ordinary continuous learner with the continuous table's KL term
        case("step_continuous_mid", dist=GAUSSIAN, T=64, B=1024, A=6, kl=True),
        # the largest: a humanoid-sized action space on a bf16 ring
        case("step_continuous_large", dist=GAUSSIAN, T=128, B=16384, A=17, storage="bf16", kl=True),
        # the continuous table's training batch: 32768 steps in fragments of 1024, on-policy
        case("batch_continuous_long", op="batch", dist=GAUSSIAN, T=1024, B=32, A=6, kl=True),
        # an action set and a batch size without favourable divisors
        case("batch_discrete_odd", op="batch", T=61, B=2047, A=7),
        # a recurrent network under mixed precision: batch-major learner tensors in bf16, shuffled minibatches
        case("step_recurrent", dist=GAUSSIAN, T=100, B=1000, A=8, storage="bf16", kl=True, learner_bf16=True,
             batch_major=True, slots="scattered"),
        # a block of trajectories enters the large continuous learner's ring
        case("insert_continuous_large", op="insert", dist=GAUSSIAN, T=128, B=4096, A=17, storage="bf16"),
        # a learner that wants its minibatch as tensors
        case("gather_discrete_large", op="gather", T=100, B=8192, A=18, slots="scattered"),
        # the whole loop on a ring that keeps log-probabilities
        case("loop_discrete_cached", op="loop", T=50, B=512, A=18, cached=True, fragment=128),
    ]


LARGEST_BYTES = 966.8e6        # of the largest listed case (step_continuous_large)
LOOP_BATCHES, LOOP_K = 2, 2    # "loop": minibatches in the ring, traversals of each


def draw(rng):
    """One more case: sizes spread over the range of the listed ones by their logarithm, options as they occur together."""
    def log_uniform(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["step", "step", "step", "step", "batch", "batch", "insert", "gather", "loop"])
    dist = rng.choice([CATEGORICAL, GAUSSIAN])
    discrete = dist == CATEGORICAL
    if discrete:       # the minimal action sets, any small set, and action spaces of hundreds of entries
        A = rng.choice([4, 6, 9, 18, 18, log_uniform(2, 32), log_uniform(2, 32), log_uniform(32, 512)])
    else:
        A = rng.choice([3, 6, 17, 17, log_uniform(1, 32), log_uniform(1, 32)])
    T = log_uniform(16, 1024)
    steps = math.exp(rng.uniform(math.log(500), math.log(2.1e6)))
    c = dict(DEFAULTS, op=op, dist=dist, A=A, T=T, B=max(1, int(steps / T)))
    if c["B"] >= 64 and rng.random() < 0.5:
        c["B"] -= c["B"] % 8
    c["storage"] = rng.choice(["f32", "f32", "bf16"])
    c["kl"] = not discrete or rng.random() < 0.2
    c["slots"] = rng.choice(["ring", "scattered"])
    if op != "batch":
        c["cached"] = rng.random() < 0.25
    c["actions_u8"] = discrete and A <= 256 and rng.random() < 0.2
    if op in ("step", "batch", "loop"):
        c["learner_bf16"] = c["storage"] == "bf16" and rng.random() < 0.5
        c["batch_major"] = rng.random() < 0.2
        c["packed"] = rng.random() < 0.2
    if op == "loop":
        c["fragment"] = max(1, c["B"] // rng.choice([1, 2, 4, 8]))
    while c["B"] > 1 and work(c)["bytes"] > LARGEST_BYTES:
        c["B"] = max(1, c["B"] // 2)
        c["fragment"] = min(c["fragment"], c["B"])
    return c


# ---------------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------------

def _hyper(c):
    """The appendix tables: discrete eps 0.3, entropy bonus 0.01, gamma 0.99; continuous eps 0.4, KL 1, gamma 0.995."""
    if c["dist"] == CATEGORICAL:
        kw = dict(gamma=0.99, eps=0.3, ent_coeff=0.01, kl_coeff=1.0 if c["kl"] else 0.0)
    else:
        kw = dict(gamma=0.995, eps=0.4, ent_coeff=0.0, kl_coeff=1.0 if c["kl"] else 0.0)
    return binding.make_config(rho_clip=2.0, flags=(binding.IMPACT_FLAG_BATCH_MAJOR if c["batch_major"] else 0)
                               | (binding.IMPACT_FLAG_ACTIONS_U8 if c["actions_u8"] and c["op"] == "batch" else 0), **kw)


def _trajectories(c, n, gen):
    """n trajectories, time-major fp32, as workers, target network and learner produce them: the target's parameters lie
    a little way from the learner's and the worker's a little way from the target's, actions are the worker's draws."""
    T, A = c["T"], c["A"]
    dev = "cuda"

    def normal(shape, std=1.0):
        return torch.randn(shape, generator=gen, device=dev) * std

    x = {}
    if c["dist"] == CATEGORICAL:
        x["learner"] = normal((T, n, A), 2.0)
        x["target"] = x["learner"] + normal((T, n, A), 0.1)
        x["worker"] = x["target"] + normal((T, n, A), 0.5)
        gumbel = -torch.log(torch.empty((T, n, A), device=dev).exponential_(generator=gen))
        actions = (x["worker"] + gumbel).argmax(dim=2)
        x["actions"] = actions.to(torch.uint8 if c["actions_u8"] else torch.int32)
        p = torch.rand((T, n), generator=gen, device=dev)
        x["rewards"] = (p < 0.025).float() - (p > 0.975).float()         # sparse and clipped to +-1
        p_done = 0.002
    else:
        lo, hi = -1.5, 0.0
        mean = normal((T, n, A))
        means = [mean]
        for std in (0.1, 0.1):
            means.append(means[-1] + normal((T, n, A), std))
        for key, m in zip(("learner", "target", "worker"), means):
            ls = torch.rand((T, n, A), generator=gen, device=dev) * (hi - lo) + lo
            x[key] = torch.cat([m, ls], dim=2)
        x["actions"] = x["worker"][..., :A] + torch.exp(x["worker"][..., A:]) * normal((T, n, A))
        x["rewards"] = normal((T, n))
        p_done = 0.001
    x["dones"] = (torch.rand((T, n), generator=gen, device=dev) < p_done).to(torch.uint8)
    x["values"] = normal((T, n))
    x["bootstrap"] = normal((n,))
    return {k: v.contiguous() for k, v in x.items()}


RECORD = ("worker", "target", "actions", "rewards", "dones")


def _learner_side(c, x, which):
    """The learner network's tensors for the trajectories `which` (a slice, or a tensor of numbers), and outputs and
    workspace for one loss call."""
    T, A = c["T"], c["A"]
    W = A if c["dist"] == CATEGORICAL else 2 * A
    learner, values, bootstrap = x["learner"][:, which], x["values"][:, which], x["bootstrap"][which]
    B = bootstrap.numel()
    if c["batch_major"]:
        learner, values = learner.transpose(0, 1), values.transpose(0, 1)
    learner = learner.to(torch.bfloat16) if c["learner_bf16"] else learner
    shape = (B, T, W) if c["batch_major"] else (T, B, W)
    # (the bootstrap values as a tensor of their own: a slice may start off the boundary that the library asks for)
    return dict(learner=learner.contiguous(), values=values.contiguous(), bootstrap=bootstrap.clone(),
                out=binding.alloc_loss_out(*shape, packed=c["packed"]),
                workspace=torch.empty(binding.impact_loss_workspace_bytes(c["dist"], T, B, A), dtype=torch.uint8, device="cuda"))


def _ring(c, slots, K):
    flags = 0
    if c["cached"]:
        flags |= binding.IMPACT_BUFFER_CACHE_LOGP | (0 if c["kl"] else binding.IMPACT_BUFFER_NO_TARGET_DIST)
    if c["actions_u8"]:
        flags |= binding.IMPACT_BUFFER_ACTIONS_U8
    return binding.Buffer(c["dist"], c["T"], c["A"], slots, K, c["storage"], flags=flags)


def _pinned(B):
    t = torch.empty(B, dtype=torch.int32, pin_memory=True)
    return t, t.numpy()


def prepare(case, seed):
    c = dict(DEFAULTS, **case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    B, op = c["B"], c["op"]
    s = dict(c=c, cfg=_hyper(c))
    if op == "batch":
        x = _trajectories(c, B, gen)
        s.update(_learner_side(c, x, slice(0, B)))
        es = torch.bfloat16 if c["storage"] == "bf16" else torch.float32
        s["batch"] = {k: v.to(es) if v.dtype == torch.float32 else v for k, v in x.items() if k in RECORD}
    elif op == "insert":
        x = _trajectories(c, B, gen)
        s["src"] = {k: x[k] for k in RECORD}
        s["ring"] = _ring(c, B, 1)                             # used once, then free again
    elif op == "loop":
        n = LOOP_BATCHES * B
        x = _trajectories(c, n, gen)
        cuts = list(range(0, n, c["fragment"])) + [n]
        s["fragments"] = [{k: x[k][:, i:j].contiguous() for k in RECORD if k != "target"} for i, j in zip(cuts, cuts[1:])]
        s["targets"] = [x["target"][:, b * B:(b + 1) * B].contiguous() for b in range(LOOP_BATCHES)]
        s["steps"] = [_learner_side(c, x, slice(b * B, (b + 1) * B)) for _ in range(LOOP_K) for b in range(LOOP_BATCHES)]
        s["slots"] = [_pinned(B) for _ in s["steps"]]           # a set per step in flight: the kernels read them in place
        s["counts"] = _pinned(B)[1]
        s["ring"] = _ring(c, n, LOOP_K)
        s["period"] = binding.impact_target_period(n, B, LOOP_K)
    else:
        n = B if c["slots"] == "ring" else B + B // 2 + 1
        x = _trajectories(c, n, gen)
        s["ring"] = _ring(c, n, 1 << 30)
        binding.impact_buffer_insert(s["ring"], {k: x[k] for k in RECORD})
        which = torch.arange(B, device="cuda") if c["slots"] == "ring" else torch.randperm(n, generator=gen, device="cuda")[:B]
        s["dev_slots"] = which.to(torch.int32)
        if op == "step":
            s.update(_learner_side(c, x, which))
        else:
            s["dst"] = binding.alloc_batch(s["ring"], B)
        s["slots"], s["counts"] = _pinned(B), _pinned(B)[1]
    return s


# ---------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------

def _results(out):
    if out.get("step_outputs") is not None:
        return {k: out[k] for k in ("grad_dist", "step_outputs", "loss5", "fractions")}
    return {k: out[k] for k in ("grad_dist", "grad_values", "vs", "adv", "loss5", "fractions")}


def _planes(ring):
    """The ring's contents after an insert.  A ring of log-probabilities keeps them as doubles after the target's plane."""
    raw = ring.storage
    if not ring.flags & binding.IMPACT_BUFFER_CACHE_LOGP:
        return {"storage": raw}
    at = 0
    if not ring.flags & binding.IMPACT_BUFFER_NO_TARGET_DIST:
        es = 4 if ring.float_dtype == torch.float32 else 2
        per_slot = -(-ring.T * ring.W * es // 16) * 16
        at = -(-(ring.num_slots * per_slot + 16) // 256) * 256
    end = at + ring.num_slots * ring.T * 16
    return {"before": raw[:at], "logp": raw[at:end].view(torch.float64), "after": raw[end:]}


def run(s):
    c = s["c"]
    op, B = c["op"], c["B"]
    if op == "batch":
        return _results(binding.impact_loss_fwd_bwd(c["dist"], s["learner"], s["values"], s["bootstrap"], s["batch"], s["cfg"],
                                                    out=s["out"], workspace=s["workspace"]))
    ring = s["ring"]
    if op == "insert":
        binding.impact_buffer_insert(ring, s["src"])
        binding.impact_buffer_sample(ring, B)
        binding.impact_buffer_release_discarded(ring)
        return _planes(ring)
    if op == "gather":
        return binding.impact_buffer_gather(ring, s["dev_slots"], s["dst"])
    if op == "step":
        if c["slots"] == "scattered":
            slots = s["dev_slots"]
        else:
            slots, at = s["slots"]
            binding.impact_buffer_sample(ring, B, at, s["counts"])
        return _results(binding.impact_loss_fwd_bwd_from_buffer(ring, slots, s["learner"], s["values"], s["bootstrap"], s["cfg"],
                                                                out=s["out"], workspace=s["workspace"]))
    for f in s["fragments"]:
        binding.impact_buffer_insert(ring, f)
    for i, st in enumerate(s["steps"]):
        slots, at = s["slots"][i]
        binding.impact_buffer_sample(ring, B, at, s["counts"])
        missing = binding.impact_buffer_missing_targets(ring, at)
        if len(missing):
            binding.impact_buffer_put_target(ring, at[missing], s["targets"][i % LOOP_BATCHES])
        binding.impact_loss_fwd_bwd_from_buffer(ring, slots, st["learner"], st["values"], st["bootstrap"], s["cfg"],
                                                out=st["out"], workspace=st["workspace"])
        binding.impact_buffer_learner_step(ring, s["period"])
    binding.impact_buffer_release_discarded(ring)
    return [_results(st["out"]) for st in s["steps"]]


# ---------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------------------------

def work(case):
    """Bytes: every input of the pass read once and every output written once.  Operations: per distribution element
    about 5 for each policy's log-probability (difference, exponential, product, two sums) and 15 for entropy, KL and
    gradient; per step about 40 for weights, scan, ratio and surrogate."""
    c = dict(DEFAULTS, **case)
    T, B, A, op = c["T"], c["B"], c["A"], c["op"]
    discrete = c["dist"] == CATEGORICAL
    W = A if discrete else 2 * A
    es = 4 if c["storage"] == "f32" else 2
    idx = 1 if c["actions_u8"] else 4
    action = idx if discrete else A * es
    keeps_worker, keeps_target = not c["cached"], not c["cached"] or c["kl"]
    kept_dist = (int(keeps_worker) + int(keeps_target)) * W * es
    logp = 16 if c["cached"] else 0
    kept = kept_dist + logp + action + es + 1                                # the ring's bytes per step
    offered = W * 4 + (idx if discrete else A * 4) + 4 + 1                   # a worker's record without the target's output
    loss_bytes = kept + (2 if c["learner_bf16"] else 4) * W + 4 + W * 4 + (16 if c["packed"] else 12)
    loss_flops = W * (5 * (3 - 2 * int(c["cached"])) + 15) + 40
    logp_flops = 2 * (5 * W + 10) if c["cached"] else 0
    n = T * B
    if op in ("step", "batch"):
        return {"bytes": n * loss_bytes + 8 * B, "flops": n * loss_flops}
    if op == "insert":
        return {"bytes": n * (offered + W * 4 + kept), "flops": n * logp_flops}
    if op == "gather":
        return {"bytes": n * 2 * kept + 4 * B, "flops": 0}
    per_ring = n * LOOP_BATCHES
    return {"bytes": per_ring * (offered + W * 4 + kept + LOOP_K * loss_bytes), "flops": per_ring * (logp_flops + LOOP_K * loss_flops)}


def tolerance(case):
    """The loss against the shape-generic kernels, which compute every step in fp64: 2-norms 8e-8 apart at most, which is the
    rounding of the fp32 results.  Log-probabilities are kept in fp64; the other contents of the ring are copies and
    defined roundings."""
    c = dict(DEFAULTS, **case)
    if c["op"] == "gather" or (c["op"] == "insert" and not c["cached"]):
        return "exact"
    if c["op"] == "insert":
        return {"rel": 1e-14}
    return {"rel": 4e-7}


# ---------------------------------------------------------------------------------------------------------------
# the same in 64 bits, by plain torch
# ---------------------------------------------------------------------------------------------------------------

def _stored(c, x):
    """A float tensor as the ring keeps it."""
    return (x.to(torch.bfloat16) if c["storage"] == "bf16" else x).double()


def _logp64(c, dist, actions):
    if c["dist"] == CATEGORICAL:
        return torch.log_softmax(dist, dim=2).gather(2, actions.long().unsqueeze(2)).squeeze(2)
    mean, ls = dist[..., :c["A"]], dist[..., c["A"]:]
    return (-0.5 * (actions - mean) ** 2 * torch.exp(-2 * ls) - ls - 0.5 * math.log(2 * math.pi)).sum(dim=2)


def _loss64(c, x, which):
    """What one loss call on the trajectories `which` returns, from the definition of the loss."""
    h, A = _hyper(c), c["A"]
    learner = x["learner"][:, which]
    z = (learner.to(torch.bfloat16) if c["learner_bf16"] else learner).double()
    V, boot = x["values"][:, which].double(), x["bootstrap"][which].double()
    worker, target, r = x["worker"][:, which], x["target"][:, which], _stored(c, x["rewards"][:, which])
    done = x["dones"][:, which]
    act = x["actions"][:, which]
    act = act.long() if c["dist"] == CATEGORICAL else _stored(c, act)
    zt = _stored(c, target)
    if c["cached"]:                        # computed when the distributions arrive, from fp32
        lw, lt = _logp64(c, worker.double(), act), _logp64(c, target.double(), act)
    else:
        lw, lt = _logp64(c, _stored(c, worker), act), _logp64(c, zt, act)
    T, B = V.shape
    w = torch.exp(lt - lw)
    gamma = h.gamma * (1.0 - done.double())
    delta = w.clamp(max=h.rho_bar) * (r + gamma * torch.cat([V[1:], boot[None]]) - V)
    g = gamma * h.lam * w.clamp(max=h.c_bar)
    adv, acc = torch.empty_like(V), torch.zeros_like(boot)
    for t in range(T - 1, -1, -1):
        acc = delta[t] + g[t] * acc
        adv[t] = acc
    R = torch.exp(_logp64(c, z, act) - torch.maximum(lt, lw - math.log(h.rho_clip)))
    lo, hi = 1.0 - h.eps, 1.0 + h.eps
    surrogate = torch.minimum(R * adv, R.clamp(lo, hi) * adv)
    clipped = ((adv > 0) & (R > hi)) | ((adv < 0) & (R < lo))
    M = T * B
    gp = torch.where(clipped, torch.zeros_like(R), -adv * R / M).unsqueeze(2)      # dL / d log pi_theta(a)
    ce, ck = h.ent_coeff / M, h.kl_coeff / M
    if c["dist"] == CATEGORICAL:
        lp, lq = torch.log_softmax(z, dim=2), torch.log_softmax(zt, dim=2)
        p, q = lp.exp(), lq.exp()
        H, KL = -(p * lp).sum(dim=2), (q * (lq - lp)).sum(dim=2)
        taken = torch.zeros_like(p).scatter_(2, act.unsqueeze(2), 1.0)
        grad = gp * (taken - p) + ce * p * (lp + H.unsqueeze(2)) + ck * (p - q)
    else:
        mu, ls, mt, lst = z[..., :A], z[..., A:], zt[..., :A], zt[..., A:]
        inv = torch.exp(-2 * ls)
        H = (ls + 0.5 * (1 + math.log(2 * math.pi))).sum(dim=2)
        q = (torch.exp(2 * lst) + (mu - mt) ** 2) * inv
        KL = (ls - lst + 0.5 * q - 0.5).sum(dim=2)
        grad = torch.cat([gp * (act - mu) * inv + ck * (mu - mt) * inv,
                          gp * ((act - mu) ** 2 * inv - 1) + ck * (1 - q) - ce], dim=2)
    if c["cached"] and not c["kl"]:
        KL = torch.zeros_like(KL)          # the target's distribution is not kept
    pg, vf = -surrogate.mean(), 0.5 * (adv ** 2).mean()
    total = pg + h.vf_coeff * vf - h.ent_coeff * H.mean() + h.kl_coeff * KL.mean()
    gV = -h.vf_coeff * adv / M
    lay = (lambda t: t.transpose(0, 1).contiguous()) if c["batch_major"] else (lambda t: t)
    out = dict(grad_dist=lay(grad), loss5=torch.stack([total, pg, vf, H.mean(), KL.mean()]),
               fractions=torch.stack([clipped.double().mean(), (w > h.rho_bar).double().mean()]))
    if c["packed"]:
        out["step_outputs"] = lay(torch.stack([gV, V + adv, adv, torch.zeros_like(adv)], dim=2))
        return {k: out[k] for k in ("grad_dist", "step_outputs", "loss5", "fractions")}
    out.update(grad_values=lay(gV), vs=lay(V + adv), adv=lay(adv))
    return {k: out[k] for k in ("grad_dist", "grad_values", "vs", "adv", "loss5", "fractions")}


def exact(case, seed):
    c = dict(DEFAULTS, **case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    B, op = c["B"], c["op"]
    if op == "gather" or (op == "insert" and not c["cached"]):
        return None                        # copies and roundings
    if op == "insert":
        x = _trajectories(c, B, gen)
        act = x["actions"] if c["dist"] == CATEGORICAL else _stored(c, x["actions"])
        pair = torch.stack([_logp64(c, x["worker"].double(), act), _logp64(c, x["target"].double(), act)], dim=2)
        return {"before": None, "logp": pair.transpose(0, 1).contiguous().reshape(-1), "after": None}
    if op == "loop":
        x = _trajectories(c, LOOP_BATCHES * B, gen)
        return [_loss64(c, x, slice(b * B, (b + 1) * B)) for _ in range(LOOP_K) for b in range(LOOP_BATCHES)]
    if op == "batch" or c["slots"] == "ring":
        return _loss64(c, _trajectories(c, B, gen), slice(0, B))
    n = B + B // 2 + 1
    x = _trajectories(c, n, gen)
    return _loss64(c, x, torch.randperm(n, generator=gen, device="cuda")[:B])
