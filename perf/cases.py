"""The work that is timed: one call of the roll-out path on a batch of Tag environments.

A case is a batch (discrete or continuous Tag, envs, agents, observation form) in the middle of
training and the call its program makes: ``iterate`` (sample + step + reset of done envs in one
call), ``separate`` (the three services one by one) or ``rollout`` (several iterations in one call,
their outputs recorded for the trainer).  The environments of a batch stand at different points of
their episodes, as they do after the first few: the later in its episode, the fewer runners of an env
are left.  The policy's output is float32 softmax of N(0, 1) logits, one of a ring of steps per pass.
"""
import math

import numpy as np
import torch

import paper_2108_13976_amd as wd

RING = 4  # steps of policy output that the passes take in turn


# ---- the cases -------------------------------------------------------------------------------------
def _tag(name, E, N, taggers, grid, T, K=4, call="iterate", k=1, obs="partial"):
    return {"name": name, "kind": "tag", "num_envs": E, "num_agents": N, "num_taggers": taggers, "grid_size": grid,
            "episode_length": T, "obs": obs, "obs_k": K, "call": call, "k": k}


def _ctag(name, E, N, taggers, world, T, K=4, call="iterate", k=1):
    return {"name": name, "kind": "ctag", "num_envs": E, "num_agents": N, "num_taggers": taggers, "world_size": world,
            "episode_length": T, "obs": "partial", "obs_k": K, "call": call, "k": k}


def listed():
    return [
        # the paper's small shape (2000 envs x 5 agents): latency and the launch itself
        _tag("tag_2000x5_iterate", 2000, 5, 1, 20, 500),
        # the workload tag_100x50 as a trainer collects a batch of it: twenty recorded iterations per call
        _tag("tag_100x50_rollout", 100, 50, 10, 50, 500, call="rollout", k=20),
        # the headline workload: 2000 envs x 1000 agents
        _tag("tag_2000x1000_iterate", 2000, 1000, 100, 100, 500),
        # the workload with the most environments
        _tag("tag_20000x100_iterate", 20000, 100, 10, 40, 200),
        # the workload with the largest environments: ten of them
        _tag("tag_10x8192_iterate", 10, 8192, 512, 512, 200),
        # a middling batch of odd sizes, the three services called one by one (as the paper has them)
        _tag("tag_777x333_separate", 777, 333, 33, 58, 300, call="separate"),
        # larger environments than the headline's, fewer of them, a recorded batch of four iterations
        _tag("tag_300x2000_rollout", 300, 2000, 200, 141, 500, call="rollout", k=4),
        # a wider view: twelve nearest agents
        _tag("tag_500x1000_k12_iterate", 500, 1000, 100, 100, 500, K=12),
        # every agent sees all others (the second observation mode)
        _tag("tag_200x500_full_iterate", 200, 500, 50, 71, 500, K=0, obs="full"),
        # continuous Tag at the paper's throughput shape
        _ctag("ctag_2000x5_iterate", 2000, 5, 1, 20.0, 500),
        # continuous Tag at the paper's snapshot shape (5 taggers, 100 runners)
        _ctag("ctag_2000x105_iterate", 2000, 105, 5, 20.0, 500),
        # continuous Tag at the most agents the paper runs, a recorded batch of four iterations
        _ctag("ctag_250x820_rollout", 250, 820, 40, 56.0, 500, call="rollout", k=4),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(max(lo, hi))))))


def draw(rng):
    call = rng.choice(["iterate", "iterate", "separate", "rollout"])
    k = rng.randint(2, 4) if call == "rollout" else 1
    if rng.random() < 0.3:
        N = _log_uniform(rng, 5, 1000)
        E = _log_uniform(rng, 10, min(4000, 200000 // N))
        world = math.sqrt(N / rng.uniform(0.0125, 0.3))
        c = _ctag("", E, N, max(1, N // rng.choice([5, 10, 20])), round(max(world, 3.0), 2), rng.choice([100, 200, 500]),
                  K=min(N - 1, rng.choice([4, 4, 2, 6, 8])), call=call, k=k)
        del c["name"]
        return c
    full = rng.random() < 0.12
    N = _log_uniform(rng, 5, 500 if full else 8192)
    K = 0 if full else min(N - 1, rng.choice([4, 4, 4, 1, 2, 3, 5, 6, 8, 10, 12, 16]))
    agents = 2000000 if N <= 1000 and K <= 4 else 500000  # in all
    if full:
        agents = min(agents, 200000000 // (5 + 4 * N))
    if call == "rollout":
        agents //= k
    E = _log_uniform(rng, 10, max(10, min(20000, agents // N)))
    grid = max(5, int(round(math.sqrt(N / rng.uniform(0.0125, 0.1)))))
    c = _tag("", E, N, max(1, N // rng.choice([5, 10, 16])), grid, rng.choice([100, 200, 500]), K=K, call=call, k=k,
             obs="full" if full else "partial")
    del c["name"]
    return c


# ---- inputs -------------------------------------------------------------------------------------------
def _continuous(case):
    return case["kind"] == "ctag"


# constants of the continuous variant (those of the repository's continuous workloads)
HEADINGS, ACCEL, VMAX_TAGGER, VMAX_RUNNER, CTAG_R2, TAG_R2 = 16, 0.25, 1.0, 0.75, 1.0, 2


def _inputs(case, seed, device):
    """A batch in the middle of training: state tensors by name, and the ring of policy outputs."""
    gen = torch.Generator(device=device)
    gen.manual_seed(int(seed))
    E, N, Nt, T = case["num_envs"], case["num_agents"], case["num_taggers"], case["episode_length"]

    def uniform(*shape):
        return torch.rand(shape, generator=gen, device=device, dtype=torch.float32)

    def integers(high, *shape):
        return torch.randint(0, high, shape, generator=gen, device=device, dtype=torch.int32)

    s = {}
    s["t"] = integers(T, E)
    side = case["world_size"] if _continuous(case) else case["grid_size"]
    # runners leave at a rate that goes with the density of taggers (fitted to the mean live fractions
    # that the repository's workloads show over two episodes)
    wane = 1.4 * T * Nt / float(side * side)
    s["live"] = (uniform(E, N) < torch.exp(-wane * s["t"].to(torch.float32) / T)[:, None]).to(torch.int32)
    s["live"][:, :Nt] = 1
    s["live"][:, -1] = 1
    s["n_live_runners"] = s["live"][:, Nt:].sum(1).to(torch.int32)
    if _continuous(case):
        for n in ("x", "y", "x0", "y0"):
            s[n] = uniform(E, N) * float(np.float32(side))
        s["h"], s["h0"] = integers(HEADINGS, E, N), integers(HEADINGS, E, N)
        s["v"] = uniform(E, N)
        s["v"][:, Nt:] *= VMAX_RUNNER
    else:
        for n in ("pos_x", "pos_y", "pos_x0", "pos_y0"):
            s[n] = integers(side, E, N)
    shape = (RING, E, N, 2, 5) if _continuous(case) else (RING, E, N, 5)
    ring = torch.softmax(torch.randn(shape, generator=gen, device=device, dtype=torch.float32), dim=-1).contiguous()
    return s, ring


def prepare(case, seed):
    args = dict(num_envs=case["num_envs"], num_agents=case["num_agents"], num_taggers=case["num_taggers"],
                episode_length=case["episode_length"], seed=seed, obs_k=case["obs_k"])
    if _continuous(case):
        envs = wd.CTagEnvs(world_size=case["world_size"], num_headings=HEADINGS, accel=ACCEL,
                           max_speed_tagger=VMAX_TAGGER, max_speed_runner=VMAX_RUNNER, tag_r2=CTAG_R2, **args)
        out = ("x", "y", "v", "h", "live", "action", "reward", "obs", "t", "done", "n_live_runners", "tags_step")
    else:
        envs = wd.TagEnvs(grid_size=case["grid_size"], tag_r2=TAG_R2,
                          obs_mode=wd.WD_OBS_FULL if case["obs"] == "full" else wd.WD_OBS_PARTIAL, **args)
        out = ("pos_x", "pos_y", "live", "action", "reward", "obs", "t", "done", "n_live_runners", "tags_step")
    envs.reset(wd.WD_RESET_ALL)
    state, ring = _inputs(case, seed, envs.device)
    for name, value in state.items():  # a batch restored into the buffers, as from a checkpoint
        envs.tensors[name].copy_(value)
    if not _continuous(case):
        wd.wd_invalidate_obs(envs.handle)
    return {"call": case["call"], "k": case["k"], "envs": envs, "ring": ring, "steps": list(ring), "at": 0,
            "out": {n: envs.tensors[n] for n in out}}


def run(state):
    envs = state["envs"]
    if state["call"] == "rollout":
        return envs.rollout(state["ring"], state["k"]), state["out"]
    probs = state["steps"][state["at"] % RING]
    state["at"] += 1
    if state["call"] == "iterate":
        envs.iterate(probs)
    else:
        envs.sample(probs)
        envs.step()
        envs.reset(wd.WD_RESET_DONE)
    return state["out"]


def work(case):
    """Probabilities and state read once, state, actions, rewards and rows written once; a roll-out also
    writes every iteration's recorded slices."""
    E, N, k = case["num_envs"], case["num_agents"], case["k"]
    if _continuous(case):
        D, probs, state, action = 8 + 6 * case["obs_k"], 40, 20, 8
    else:
        D, probs, state, action = 5 + 4 * (N if case["obs"] == "full" else case["obs_k"]), 20, 12, 4
    outputs = action + 4 + 4 * D
    per_agent = k * probs + 2 * state + outputs
    per_env = 12 + 16
    if case["call"] == "rollout":
        per_agent += k * outputs
        per_env += 4 * k
    return {"bytes": E * (N * per_agent + per_env), "flops": 0}


def tolerance(case):
    # Whole values (positions, actions, flags, counts) and rewards are exact.  Rows hold quotients that
    # an implementation may take as a product with the rounded reciprocal, and continuous positions
    # are sums of a few float32 steps: measured against 64 bits, outputs are up to 3.6e-8 off as a
    # whole, a single element up to 4e-7 of the root mean square.
    return {"rel": 1.5e-7, "max": 2e-6, "differ": 0.0}


# ---- the same pass in plain torch, rows and state in 64 bits ------------------------------------------------
_M32 = 0xFFFFFFFF


def _mul_hi_lo(c, x):
    """High and low words of the 64-bit product of a constant and 32-bit words held in int64."""
    lo, hi = x & 0xFFFF, x >> 16
    p, q = c * lo, c * hi  # below 2^48
    s = p + ((q & 0xFFFF) << 16)
    return ((q >> 16) + (s >> 32)) & _M32, s & _M32


def _philox(c0, c1, c2, c3, k0, k1):
    for _ in range(10):
        hi_a, lo_a = _mul_hi_lo(0xD2511F53, c0)
        hi_b, lo_b = _mul_hi_lo(0xCD9E8D57, c2)
        c0, c1, c2, c3 = hi_b ^ c1 ^ k0, lo_b, hi_a ^ c3 ^ k1, lo_a
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    return torch.stack([c0, c1, c2, c3], -1)


def _words(case, seed, g, device):
    """Random words [E, N] (discrete: one draw per agent) or [E, N, 2] (continuous) of step g."""
    E, N = case["num_envs"], case["num_agents"]
    per_agent = _continuous(case)
    n = N if per_agent else (N + 3) // 4
    e = torch.arange(E, device=device, dtype=torch.int64)[:, None].expand(E, n)
    i = torch.arange(n, device=device, dtype=torch.int64)[None, :].expand(E, n)
    stream = 2 if per_agent else 0
    zero = torch.zeros_like(e)
    w = _philox(e, i, zero + (g & _M32), zero + (stream | ((g >> 32) << 8 & _M32)), seed & _M32, (seed >> 32) & _M32)
    return w[..., :2] if per_agent else w.reshape(E, 4 * n)[:, :N]


def _draw_actions(probs, words):
    """Inverse CDF with a float32 running sum (the rule: strict comparison, last action falls through)."""
    u = (words >> 8).to(torch.float32) * (1.0 / 16777216.0)
    c0 = probs[..., 0]
    c1 = c0 + probs[..., 1]
    c2 = c1 + probs[..., 2]
    c3 = c2 + probs[..., 3]
    return sum((u >= c).to(torch.int64) for c in (c0, c1, c2, c3))


def _squares(a, b, c, d):
    """(a - b)^2 + (c - d)^2 in the type of the operands, each operation rounded by itself."""
    dx, dy = a - b, c - d
    return dx * dx + dy * dy


def _order(d2, n):
    """Keys that order by (squared distance, index of the last dimension)."""
    if d2.dtype == torch.float32:
        d2 = d2.view(torch.int32).to(torch.int64)  # not negative: its bits order like its value
    return (d2 << 16) | torch.arange(n, device=d2.device, dtype=torch.int64)


_FAR = 1 << 62


def _tag_check(x, y, live, Nt, r2):
    """Runners tagged now [E, N] and credits per tagger [E, Nt]; decided on the given coordinates."""
    E, N = x.shape
    tagged = torch.zeros((E, N), dtype=torch.bool, device=x.device)
    credits = torch.zeros((E, Nt), dtype=torch.int64, device=x.device)
    step = max(1, 60000000 // (N * Nt))
    for a in range(0, E, step):
        s = slice(a, a + step)
        d2 = _squares(x[s, Nt:, None], x[s, None, :Nt], y[s, Nt:, None], y[s, None, :Nt])
        best = _order(d2, Nt).min(-1).values
        near = d2.min(-1).values <= r2
        hit = near & (live[s, Nt:] != 0)
        tagged[s, Nt:] = hit
        credits[s].scatter_add_(1, best & 0xFFFF, hit.to(torch.int64))
    return tagged, credits


def _nearest(x, y, live, K):
    """Indices [E, N, K] of the nearest other live agents by (d2, index), -1 where there are fewer."""
    E, N = x.shape
    out = torch.full((E, N, K), -1, dtype=torch.int64, device=x.device)
    if K == 0:
        return out
    step = max(1, 60000000 // (N * N))
    rows = max(1, 60000000 // N) if N * N > 60000000 else N
    own = torch.arange(N, device=x.device)
    for a in range(0, E, step):
        s = slice(a, a + step)
        for b in range(0, N, rows):
            r = slice(b, b + rows)
            key = _order(_squares(x[s, r, None], x[s, None, :], y[s, r, None], y[s, None, :]), N)
            none = (live[s, None, :] == 0) | (live[s, r, None] == 0) | (own[r, None] == own[None, :])[None]
            key = torch.where(none, torch.full_like(key, _FAR), key)
            best = torch.topk(key, K, dim=-1, largest=False, sorted=True).values
            out[s, r] = torch.where(best == _FAR, torch.full_like(best, -1), best & 0xFFFF)
    return out


def _take(a, idx):
    """a[e, idx[e, ...]]"""
    E = a.shape[0]
    return torch.gather(a, 1, idx.reshape(E, -1)).reshape(idx.shape)


def _heading_table(device):
    h = torch.arange(HEADINGS, dtype=torch.float64, device=device) * (2.0 * math.pi / HEADINGS)
    c, s = torch.cos(h), torch.sin(h)
    zero = torch.zeros_like(c)
    return torch.where(c.abs() < 1e-12, zero, c), torch.where(s.abs() < 1e-12, zero, s)


def exact(case, seed):
    E, N, Nt, T, K = (case[n] for n in ("num_envs", "num_agents", "num_taggers", "episode_length", "obs_k"))
    if E * N * N > 2.2e9:
        return None
    device = "cuda" if torch.cuda.is_available() else "cpu"
    cont = _continuous(case)
    s, ring = _inputs(case, seed, device)
    t, live, nlr = (s[n].to(torch.int64) for n in ("t", "live", "n_live_runners"))
    tagger = (torch.arange(N, device=device) < Nt)[None, :].expand(E, N)
    f64 = torch.float64
    if cont:
        side = float(np.float32(case["world_size"]))
        cos64, sin64 = _heading_table(device)
        cos32, sin32 = cos64.to(torch.float32), sin64.to(torch.float32)
        h = s["h"].to(torch.int64)
        low = {n: s[n].clone() for n in ("x", "y", "v")}  # float32, as the rules round: what decides
        hi = {n: s[n].to(f64) for n in ("x", "y", "v")}
        vmax32 = torch.where(tagger, VMAX_TAGGER, VMAX_RUNNER).to(torch.float32)
    else:
        side = case["grid_size"]
        x, y = s["pos_x"].to(torch.int64), s["pos_y"].to(torch.int64)
    recorded = {"action": [], "reward": [], "done": [], "obs": []}
    for it in range(case["k"]):
        g = it  # prepare leaves the step counter at 0
        act = _draw_actions(ring[g % RING], _words(case, seed, g, device))
        alive = live != 0
        if cont:
            h = torch.where(alive, (h + act[..., 1] - 2) % HEADINGS, h)
            for c, cos, sin, kind in ((low, cos32, sin32, torch.float32), (hi, cos64, sin64, f64)):
                v = c["v"] + (act[..., 0] - 2).to(kind) * ACCEL
                v = torch.minimum(torch.clamp(v, min=0.0), vmax32.to(kind))
                nx, ny = c["x"] + v * cos[h], c["y"] + v * sin[h]
                if c is low:  # walls are met where the rounded positions meet them
                    out_lo = (nx < 0, ny < 0)
                    out_hi = (nx > side, ny > side)
                    wall = out_lo[0] | out_lo[1] | out_hi[0] | out_hi[1]
                for n, q in (("x", nx), ("y", ny)):
                    a = 0 if n == "x" else 1
                    q = torch.where(out_lo[a], torch.zeros_like(q), torch.where(out_hi[a], torch.full_like(q, side), q))
                    c[n] = torch.where(alive, q, c[n])
                c["v"] = torch.where(alive, torch.where(wall, torch.zeros_like(v), v), c["v"])
            px, py = low["x"], low["y"]
        else:
            x = torch.where(alive, torch.clamp(x + (act == 4).long() - (act == 3).long(), 0, side - 1), x)
            y = torch.where(alive, torch.clamp(y + (act == 1).long() - (act == 2).long(), 0, side - 1), y)
            px, py = x, y
        tagged, credits = _tag_check(px, py, live, Nt, CTAG_R2 if cont else TAG_R2)
        live = torch.where(tagged, torch.zeros_like(live), live)
        tags = tagged.sum(1)
        reward = -tagged.to(f64)
        reward[:, :Nt] = credits.to(f64)
        t, nlr = t + 1, nlr - tags
        done = (nlr == 0) | (t >= T)
        recorded["action"].append(act)
        recorded["reward"].append(reward)
        recorded["done"].append(done.to(torch.int64))
        d = done[:, None]
        if cont:
            for c in (low, hi):
                for n, n0 in (("x", "x0"), ("y", "y0")):
                    c[n] = torch.where(d, s[n0].to(c[n].dtype), c[n])
                c["v"] = torch.where(d, torch.zeros_like(c["v"]), c["v"])
            h = torch.where(d, s["h0"].to(torch.int64), h)
            px, py, wx, wy = low["x"], low["y"], hi["x"], hi["y"]
        else:
            x = torch.where(d, s["pos_x0"].to(torch.int64), x)
            y = torch.where(d, s["pos_y0"].to(torch.int64), y)
            px, py, wx, wy = x, y, x.to(f64), y.to(f64)
        live = torch.where(d, torch.ones_like(live), live)
        t = torch.where(done, torch.zeros_like(t), t)
        nlr = torch.where(done, torch.full_like(nlr, N - Nt), nlr)
        tags = torch.where(done, torch.zeros_like(tags), tags)
        # rows
        tf = (t.to(f64) / T)[:, None].expand(E, N)
        own = [wx / side, wy / side]
        if cont:
            own += [hi["v"], cos64[h], sin64[h]]
        own += [tagger.to(f64), live.to(f64), tf]
        if case["obs"] == "full":
            both = ((live[:, :, None] != 0) & (live[:, None, :] != 0)).to(f64)
            slots = [both * (wx[:, None, :] - wx[:, :, None]) / side, both * (wy[:, None, :] - wy[:, :, None]) / side,
                     both * tagger[:, None, :].to(f64), both]
        else:
            idx = _nearest(px, py, live, K)
            have = (idx >= 0).to(f64)
            idx = torch.clamp(idx, min=0)
            slots = [have * (_take(wx, idx) - wx[..., None]) / side, have * (_take(wy, idx) - wy[..., None]) / side]
            if cont:
                slots += [have * _take(hi["v"] * cos64[h], idx), have * _take(hi["v"] * sin64[h], idx)]
            slots += [have * (idx < Nt).to(f64), have]
        obs = torch.cat([torch.stack(own, -1), torch.stack(slots, -1).reshape(E, N, -1)], -1)
        recorded["obs"].append(obs)
    out = {"live": live, "action": act, "reward": reward, "obs": obs, "t": t, "done": torch.zeros_like(t),
           "n_live_runners": nlr, "tags_step": tags}
    out.update({"x": hi["x"], "y": hi["y"], "v": hi["v"], "h": h} if cont else {"pos_x": x, "pos_y": y})
    if case["call"] == "rollout":
        return {n: torch.stack(v) for n, v in recorded.items()}, out
    return out
