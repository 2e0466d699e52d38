"""The work that users of this library have it do, as cases that can be timed.

Two kinds of program drive the batched physics step.  A *rollout* advances a batch of environments by many
engine steps in one launch (engine-only throughput, evaluation of recorded actions, open-loop planning); a
*control loop* comes back to the host after every step, because a policy or a player chooses the next
action from what it observes.  Every case is one pass through such a program's calls of
`paper_2410_23208_amd`; scenes are drawn by `scenegen`, so that they have its workloads' shapes, masks,
joints and contact densities.

Fields of a case
  flow      "rollout"   new episodes in all environments, `steps` engine steps in one launch, then the state
                        (checkpoint) and the flat observation;
            "restarts"  the same, with a seeded 5 % of the environments starting a new episode after every step
                        inside the launch;
            "agent"     one iteration of a training loop's environment side: decode the policy's multi-discrete
                        actions, one engine step, reward and termination, new episodes where one ended, and the
                        entity observation with its attention masks;
            "play"      one engine step and the flat observation of a few environments
  content   what the scenes hold: "S", "M", "L", "pile" (contact-heavy L), "hetero" (S, M and L content in L
            capacities), "dense" (a pile in a narrow pen), "towers" (stacked boxes)
  envs, steps, substeps, sweeps   sizes; order, batch   schedule of the collision constraints: k2d_params
            sweep_order and batch_size
"""
import numpy as np
import torch

import paper_2410_23208_amd as k2d
import scenegen

# scenegen workload that a content is drawn from, capacity class, substeps and solver sweeps it is run with, and
# its arithmetic (one per add, multiply, division, root, sine, cosine) per environment and substep: a part that
# does not depend on the number of sweeps and one for every sweep, from the contacts that 256 environments have
# on average over 256 steps
CONTENT = {
    "S": dict(config=0, caps="S", substeps=1, sweeps=5, fixed=3789, sweep=578),
    "M": dict(config=1, caps="M", substeps=2, sweeps=8, fixed=4116, sweep=628),
    "L": dict(config=2, caps="L", substeps=3, sweeps=10, fixed=11714, sweep=931),
    "pile": dict(config=3, caps="L", substeps=3, sweeps=10, fixed=15591, sweep=1064),
    "hetero": dict(config=4, caps="L", substeps=3, sweeps=10, fixed=10708, sweep=939),
    "dense": dict(config=3, caps="L", substeps=3, sweeps=10, fixed=15793, sweep=1186),
    "towers": dict(config=3, caps="L", substeps=3, sweeps=10, fixed=18035, sweep=1639),
}
LEVELS = 2048        # distinct scenes a batch draws its levels from (a training run keeps a buffer of levels)
ACTION_SETS = 8      # control loops take their actions from this many rows in turn
RESTART_SHARE = 0.05


def _case(name, flow, content, envs, steps=1, order=0, batch=0, substeps=None, sweeps=None):
    c = CONTENT[content]
    case = dict(flow=flow, content=content, envs=envs, steps=steps, order=order, batch=batch,
                substeps=substeps or c["substeps"], sweeps=sweeps or c["sweeps"])
    return dict(case, name=name) if name else case


def listed():
    return [
        # a person or a script plays one small level: one step, one observation, nothing but latency
        _case("play_s1", "play", "S", 1),
        # the environment side of a training loop, two common sizes: launches and host calls between steps count
        _case("agent_m2048", "agent", "M", 2048),
        _case("agent_l8192", "agent", "L", 8192),
        # engine-only rollouts of the three scene sizes (the small one leaves most of the chip idle, the large one is
        # the benchmark's workload)
        _case("rollout_s64", "rollout", "S", 64, 200),
        _case("rollout_m1024", "rollout", "M", 1024, 256),
        _case("rollout_l8192", "rollout", "L", 8192, 256),
        # small scenes in a batch that fills the chip several times over
        _case("rollout_s65536", "rollout", "S", 65536, 64),
        # contact-heavy scenes, the largest batch and the longest rollout
        _case("rollout_pile32768", "rollout", "pile", 32768, 512),
        # a training batch of mixed content, with episodes restarted inside the launch
        _case("restarts_hetero16384", "restarts", "hetero", 16384, 256),
        # a ragged batch of deep piles (more colliding pairs than lanes in some environments)
        _case("rollout_dense5003", "rollout", "dense", 5003, 100),
        # stacks, swept level after level (the order meant for them)
        _case("rollout_towers8192_levels", "rollout", "towers", 8192, 128, order=1),
        # the batched impulse resolution, with the batch size of the paper's engine
        _case("rollout_l2048_batched", "rollout", "L", 2048, 64, batch=16),
    ]


def _log_uniform(rng, lo, hi):
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    flow = rng.choice(["rollout", "rollout", "rollout", "restarts", "agent", "agent", "play"])
    content = rng.choice(sorted(CONTENT))
    if flow == "play":
        return _case(None, flow, content, _log_uniform(rng, 1, 64), 1, order=rng.choice([0, 0, 1]))
    if flow == "agent":
        return _case(None, flow, content, _log_uniform(rng, 32, 16384), 1, order=rng.choice([0, 0, 1]))
    batch = rng.choice([0, 0, 0, 0, 0, 16, rng.choice([4, 8, 32])])
    envs = _log_uniform(rng, 16, 65536 if content == "S" else 32768)
    # (no drawn case is to cost more than the largest listed one, and the batches of A.8 cost several times a sweep)
    most = min(512, max(4, (1 << 19 if batch else 1 << 22) // envs))
    steps = _log_uniform(rng, 4, most)
    c = CONTENT[content]
    return _case(None, flow, content, envs, steps, order=0 if batch else rng.choice([0, 0, 1]), batch=batch,
                 substeps=rng.choice([c["substeps"], 1, 2, 3]), sweeps=rng.choice([c["sweeps"], 5, 8, 10]))


def _scenes(content, n, episode, seed):
    c = CONTENT[content]
    if content == "dense":
        return scenegen.make_dense_scene(n_envs=n, episode=episode, seed=seed)
    if content == "towers":
        return scenegen.make_stack_scene(n_envs=n, episode=episode, seed=seed)
    return scenegen.make_scene(c["config"], n_envs=n, episode=episode, seed=seed)


def prepare(case, seed):
    n, steps, flow = case["envs"], case["steps"], case["flow"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    caps, _, scene = _scenes(case["content"], min(n, LEVELS), 0, seed)
    params = dict(scenegen.default_params(case["substeps"], case["sweeps"]), sweep_order=case["order"],
                  batch_size=case["batch"])
    levels = torch.from_numpy(k2d.pack_scenes(caps, scene).view(np.int32)).cuda()

    def level_of_each():   # every level at least once, in some order, where the batch is that large
        idx = torch.arange(n, device="cuda") % levels.shape[0]
        return idx[torch.randperm(n, generator=gen, device="cuda")]

    batch = k2d.Batch(caps, n, params)
    width = caps[2] + caps[3]
    s = dict(flow=flow, batch=batch, steps=steps)
    if flow in ("rollout", "restarts"):
        s["words"] = levels[level_of_each()].contiguous()
        s["actions"] = torch.rand((steps, n, width), generator=gen, device="cuda") * 2 - 1
        if flow == "restarts":
            s["levels"] = levels
            new = torch.randint(0, levels.shape[0], (steps, n), generator=gen, device="cuda", dtype=torch.int32)
            restart = torch.rand((steps, n), generator=gen, device="cuda") < RESTART_SHARE
            s["restart"] = torch.where(restart, new, torch.full_like(new, -1)).contiguous()
        return s
    # control loops are met in the middle of their episodes
    batch.reset(levels[level_of_each()].contiguous())
    batch.step(torch.rand((32, n, width), generator=gen, device="cuda") * 2 - 1)
    s["turn"] = 0
    if flow == "agent":
        motors = torch.randint(0, 3, (ACTION_SETS, n, caps[2]), generator=gen, device="cuda", dtype=torch.int32)
        thrusters = torch.randint(0, 2, (ACTION_SETS, n, caps[3]), generator=gen, device="cuda", dtype=torch.int32)
        s["policy"] = torch.cat([motors, thrusters], -1).contiguous()
        s["next_words"] = levels[level_of_each()].contiguous()   # the level that an environment plays next
        s["ids"] = torch.arange(n, dtype=torch.int32, device="cuda")
        s["none"] = torch.full((n,), -1, dtype=torch.int32, device="cuda")
        s["dist"] = torch.full((n,), -1.0, device="cuda")
    else:
        s["actions"] = torch.rand((ACTION_SETS, 1, n, width), generator=gen, device="cuda") * 2 - 1
    torch.cuda.synchronize()
    return s


def run(s):
    batch = s["batch"]
    if s["flow"] == "rollout":
        batch.reset(s["words"])
        batch.step(s["actions"], s["steps"])
        return {"state": batch.read_state(), "obs": batch.read_obs()}
    if s["flow"] == "restarts":
        batch.reset(s["words"])
        batch.step_reset(s["actions"], s["levels"], s["restart"], s["steps"])
        return {"state": batch.read_state(), "obs": batch.read_obs()}
    turn = s["turn"]
    s["turn"] = (turn + 1) % ACTION_SETS
    if s["flow"] == "play":
        batch.step(s["actions"][turn], 1)
        return {"obs": batch.read_obs()}
    actions = batch.decode_actions(s["policy"][turn])
    batch.step(actions, 1)
    reward, done = batch.read_outcome(s["dist"])
    ended = done.bool()
    batch.reset(s["next_words"], torch.where(ended, s["ids"], s["none"]))   # (indices out of range are skipped)
    s["dist"].masked_fill_(ended, -1.0)
    return {"reward": reward, "done": done, "dist": s["dist"], "entities": batch.read_entities()}


def work(case):
    c = CONTENT[case["content"]]
    P, C, J, T = scenegen.CAPS[c["caps"]]
    N = P + C
    n, steps, flow = case["envs"], case["steps"], case["flow"]
    layout = k2d.get_layout((P, C, J, T))
    scene, record, flat = layout["scene_words"], layout["state_words"], layout["obs_dim"]
    dynamic = 6 * N + 3 * J + (layout["n_pairs"] + 3) // 4   # what a step changes (impulses of resting contacts aside)
    flops = float(n) * steps * case["substeps"] * (c["fixed"] + case["sweeps"] * c["sweep"])
    words = float(steps) * (J + T)                           # actions
    if flow in ("rollout", "restarts"):
        words += scene + record + flat                       # scenes in, state and observation out
        if flow == "restarts":
            words += steps * (1 + RESTART_SHARE * scene)
    else:
        words += scene + dynamic + (0 if flow == "agent" else flat)
        if flow == "agent":   # policy's actions, reward, done, distance in and out; entities and masks
            words += (J + T) + 3.25 + 30 * N + 2 * J * 13 + 7 * T + 4 * N
    return {"bytes": 4.0 * n * words, "flops": flops}


def tolerance(case):
    # The sweep visits the constraints in a stated order and every formula's rounding is stated too: fp32 results
    # are the same bits in every correct implementation, and nothing less would do, since a difference in the last
    # bit grows without bound over the contacts of a rollout.
    return "exact"
