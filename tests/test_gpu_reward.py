"""Graph reward and dual-group advantage on the GPU (through the C ABI) against the oracle, and
the edge similarities written by the classes kernels.

Scores, step rewards and advantages are fp64 on both sides from the same integer counts and the
same float32 edge similarities, so they agree to rounding (1e-12; NaN where both are undefined).
Edge similarities are fp32 sums of bf16 products on the GPU: within 3e-4 of the float64 cosine
(the kernel's bound is 2.5e-4 at dim 4096).
"""
import json
import os

import numpy as np
import pytest
import torch

from oracle import graphattn_oracle as O
from paper_2606_18954_amd import graphattn as G
from paper_2606_18954_amd import workloads as W

from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu
KEYS = {"S": "score", "r": "step_reward", "A_cor": "a_cor", "A_eff": "a_eff", "A_dual": "a_dual"}


def gpu_adv(parent, labels, reward, sim, w, lam):
    require_gpu()
    with G.Forest(parent) as f:
        out = f.advantages(torch.as_tensor(np.asarray(labels), dtype=torch.int32).cuda(),
                           torch.as_tensor(np.asarray(reward), dtype=torch.int32).cuda(),
                           torch.as_tensor(np.asarray(sim), dtype=torch.float32).cuda(), w, lam)
        torch.cuda.synchronize()
        return {k: v.cpu().numpy() for k, v in out.items()}


def compare(tag, got, ref, tol=1e-12):
    for k, g in KEYS.items():
        a, b = got[g], ref[k]
        assert np.array_equal(np.isnan(a), np.isnan(b)), (tag, k)
        m = ~np.isnan(b)
        err = float(np.abs(a[m] - b[m]).max()) if m.any() else 0.0
        say(f"[reward] {tag} {k}: max|d| = {err:.2e}")
        assert err <= tol, (tag, k, err)


def test_fixture_on_gpu():
    with open(os.path.join(os.path.dirname(__file__), "golden", "graph_reward_small.json")) as f:
        fx = json.load(f)
    got = gpu_adv(fx["parent"], fx["labels"], fx["reward"],
                  np.array(fx["edge_sim"], dtype=np.float32), fx["w"], fx["lambda_eff"])
    ref = {k: np.array([np.nan if x is None else x for x in fx[k]]) for k in KEYS}
    # the fixture's similarities are float32-rounded here: compare with the oracle on those
    ref2 = O.graph_advantages(np.array(fx["parent"]), np.array(fx["labels"]),
                              np.array(fx["reward"]),
                              np.array(fx["edge_sim"], dtype=np.float32).astype(np.float64),
                              fx["w"], fx["lambda_eff"])
    compare("fixture (oracle, float32 sims)", got, ref2)
    compare("fixture (hand values)", got, ref, tol=2e-7)


@pytest.mark.parametrize("case", ["routes", "undefined"])
def test_route_fixture_on_gpu(case):
    """The hand-derived rollouts of graph_reward_routes.json: a class anchored below the root,
    edges on several members' and classes' routes, a shared edge whose own source's group
    differs from its class label's, and a class member with an undefined score."""
    from test_oracle_reward_pins import exact
    with open(os.path.join(os.path.dirname(__file__), "golden", "graph_reward_routes.json")) as f:
        fx = next(c for c in json.load(f)["cases"] if c["name"] == case)
    sim32 = np.array(fx["edge_sim"], dtype=np.float32)
    got = gpu_adv(fx["parent"], fx["labels"], fx["reward"], sim32, fx["w"], fx["lambda_eff"])
    ref = O.graph_advantages(np.array(fx["parent"]), np.array(fx["labels"]),
                             np.array(fx["reward"]), sim32.astype(np.float64), fx["w"],
                             fx["lambda_eff"])
    compare(f"{case} (oracle, float32 sims)", got, ref)
    hand = {k: np.array([exact(x) for x in fx[k]]) for k in KEYS}
    compare(f"{case} (hand values)", got, hand, tol=2e-7)


@pytest.mark.parametrize("prompts,sched,seed", [(3, (3, 3, 2), 1), (2, (4, 5, 3, 2), 2),
                                                (5, (2, 2, 2, 2, 2), 3), (1, (8,), 4),
                                                (2, (6, 6, 15), 5)])
@pytest.mark.parametrize("w,lam", [(0.7, 0.5), (0.0, 1.0), (1.0, 0.0)])
def test_random_rollouts(prompts, sched, seed, w, lam):
    rng = np.random.default_rng(seed)
    parent = W.state_forest(prompts, sched)
    N = len(parent)
    reward = W.state_rewards(parent, seed)
    z = W.draw_state_embeddings(parent, 64, seed, share=1.0)
    labels = O.equivalence_classes(z.view(torch.int16).numpy().view(np.uint16), "bf16", parent,
                                   0.92)
    sim = rng.uniform(-0.5, 1.0, N).astype(np.float32)
    say(f"[case] {prompts}x{sched} N={N} classes={len(set(labels.tolist()))} w={w} lam={lam}")
    got = gpu_adv(parent, labels, reward, sim, w, lam)
    ref = O.graph_advantages(parent, labels, reward, sim.astype(np.float64), w, lam)
    compare(f"{prompts}x{sched}", got, ref, tol=1e-9)


def test_pipeline_classes_similarities_advantages():
    """Classes and edge similarities from the GPU kernels feed the advantages: labels bit-exact,
    similarities within the bound, scores and efficiency advantages (which do not depend on the
    similarities) to rounding, step rewards within the similarity bound."""
    wl = W.equiv_batch(prompts=4, schedule=(4, 5, 3, 2), dim=1024, seed=23)
    N = len(wl.parent)
    reward = W.state_rewards(wl.parent, 23)
    zb = wl.z_bits()
    ref_lab = O.equivalence_classes(zb, "bf16", wl.parent, wl.kappa)
    ref_sim = np.zeros(N)
    for v in range(N):
        if wl.parent[v] >= 0:
            ref_sim[v] = O.cosine(zb, "bf16", int(wl.parent[v]), v)
    with G.Forest(wl.parent) as f:
        es = torch.empty(N, dtype=torch.float32, device="cuda")
        lab = f.classes(wl.z.cuda(), wl.kappa, edge_sim=es)
        out = f.advantages(lab, torch.from_numpy(reward).cuda(), es, 0.7, 0.5)
        torch.cuda.synchronize()
        got = {k: v.cpu().numpy() for k, v in out.items()}
        assert np.array_equal(lab.cpu().numpy(), ref_lab)
        d = float(np.abs(es.cpu().numpy().astype(np.float64) - ref_sim).max())
        say(f"[reward] edge similarity max|d| = {d:.2e}")
        assert d <= 3e-4
    ref = O.graph_advantages(wl.parent, ref_lab, reward, ref_sim, 0.7, 0.5)
    for k, tol in [("S", 1e-12), ("A_eff", 1e-12), ("r", 3e-4)]:
        a, b = got[KEYS[k]], ref[k]
        assert np.array_equal(np.isnan(a), np.isnan(b))
        m = ~np.isnan(b)
        assert float(np.abs(a[m] - b[m]).max()) <= tol, k


def test_one_launch_and_multi_kernel_paths_agree():
    """A batch of prompts of at most 512 states runs in one launch; adding one larger prompt
    sends the whole batch through the multi-kernel path: the small prompts' results must agree
    (to the rounding of the few fp64 sums that the two paths take in different orders)."""
    small = W.state_forest(3, (4, 5, 3, 2))
    big = W.state_forest(1, (6, 6, 15)) + len(small)
    big[0] = -1
    both = np.concatenate([small, big])
    rng = np.random.default_rng(9)
    N, n = len(both), len(small)
    reward = W.state_rewards(both, 9)
    labels = np.arange(N, dtype=np.int32)
    for v in range(5, n, 7):                          # link some same-depth states
        d = O.state_depths(both)
        same = [u for u in range(1, n) if d[u] == d[v] and u < v and (u // 205) == (v // 205)]
        if same:
            u = int(rng.choice(same))
            lo, hi = min(labels[u], labels[v]), max(labels[u], labels[v])
            labels[labels == hi] = lo
    sim = rng.uniform(-0.5, 1.0, N).astype(np.float32)
    one = gpu_adv(small, labels[:n], reward[:n], sim[:n], 0.7, 0.5)
    multi = gpu_adv(both, labels, reward, sim, 0.7, 0.5)
    for k in KEYS.values():
        assert np.allclose(one[k][:n], multi[k][:n], rtol=0, atol=1e-12, equal_nan=True), k


def random_tree(rng, n, kind):
    if kind == "chain":
        return np.arange(-1, n - 1, dtype=np.int32)
    parent = np.zeros(n, dtype=np.int32) if kind == "star" else np.array(
        [0] + [int(rng.integers(max(0, v - 40), v)) for v in range(1, n)], dtype=np.int32)
    parent[0] = -1
    return parent


@pytest.mark.parametrize("kind", ["random", "star", "chain"])
@pytest.mark.parametrize("n", [1, 2, 64, 65, 255, 256, 257, 512, 513, 1024, 1025, 2047, 2048])
def test_one_launch_sizes(n, kind):
    """One prompt at the edges of the workgroup sizes and of the one-launch range, alone and next
    to a prompt beyond that range (2,203 states), which sends both through the multi-kernel path:
    the two agree to the rounding of the few fp64 sums taken in another order (n terms of size at
    most sqrt(n) each).  Small prompts also against the oracle."""
    rng = np.random.default_rng(n)
    small = random_tree(rng, n, kind)
    big = W.state_forest(1, (6, 6, 60)) + n
    big[0] = -1
    both = np.concatenate([small, big])
    N = len(both)
    d = O.state_depths(both)
    labels = np.arange(N, dtype=np.int32)
    last = {}
    for v in range(1, n):                             # classes of states of one depth, some large
        key = (int(d[v]), int(rng.integers(0, 4)))
        if rng.random() < 0.5:
            labels[v] = last.setdefault(key, v)
    reward = W.state_rewards(both, n)
    sim = rng.uniform(-0.5, 1.0, N).astype(np.float32)
    say(f"[case] n={n} {kind} classes={len(set(labels[:n].tolist()))}")
    one = gpu_adv(small, labels[:n], reward[:n], sim[:n], 0.7, 0.5)
    multi = gpu_adv(both, labels, reward, sim, 0.7, 0.5)
    for k in KEYS.values():
        assert np.allclose(one[k], multi[k][:n], rtol=1e-12, atol=1e-10, equal_nan=True), k
    if n <= 257 and kind != "chain":
        compare(f"n={n} {kind}", one, O.graph_advantages(
            small, labels[:n], reward[:n], sim[:n].astype(np.float64), 0.7, 0.5), tol=1e-9)
