"""Equivalence detection and the graph suffix on the GPU (through the C ABI) against the oracle.

Labels and suffix lists are integer results: bit-exact.  The cosine decision is taken in fp32
on the GPU and in float64 by the oracle, so every input here keeps all compared pairs at least
1e-3 from kappa (the kernel's error bound is 2.5e-4 at dim 4096); each test checks that margin
with the oracle before comparing.
"""
import numpy as np
import pytest
import torch

from oracle import graphattn_oracle as O
from paper_2606_18954_amd import graphattn as G
from paper_2606_18954_amd import workloads as W

from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu
MARGIN = 1e-3


def gpu_labels(z, parent, kappa):
    require_gpu()
    lab = G.equivalence_classes(z.cuda(), G.HostForest(parent), kappa)
    torch.cuda.synchronize()
    return lab.cpu().numpy()


def check(wl, kappa=None):
    kappa = wl.kappa if kappa is None else kappa
    say(f"[case] {wl.name} kappa={kappa}")
    m = O.similarity_margin(wl.z_bits(), "bf16", wl.parent, kappa)
    assert m >= MARGIN, f"inputs within {m} of kappa"
    ref = O.equivalence_classes(wl.z_bits(), "bf16", wl.parent, kappa)
    got = gpu_labels(wl.z, wl.parent, kappa)
    merged = int((ref != np.arange(len(ref))).sum())
    say(f"[equiv] {wl.name}: {len(set(ref.tolist()))} classes, {merged} merged states, "
        f"margin {m:.4f}, equal={np.array_equal(got, ref)}")
    assert np.array_equal(got, ref)
    return got


@pytest.mark.parametrize("prompts,sched,dim", [(3, (4, 5, 3, 2), 256), (2, (4, 5, 3, 2), 4096),
                                               (4, (2, 2, 2, 2, 2), 128), (2, (6, 6, 8), 64),
                                               (5, (8, 8), 192)])
def test_classes_match_oracle(prompts, sched, dim):
    check(W.equiv_batch(prompts=prompts, schedule=sched, dim=dim, seed=prompts * 31 + dim))


def test_threshold_extremes_and_ancestor_rule():
    wl = W.equiv_batch(prompts=2, schedule=(3, 4), dim=64, seed=7)
    N = len(wl.parent)
    assert np.array_equal(gpu_labels(wl.z, wl.parent, 2.0), np.arange(N))
    lab = gpu_labels(wl.z, wl.parent, -2.0)
    assert np.array_equal(lab, O.equivalence_classes(wl.z_bits(), "bf16", wl.parent, -2.0))
    chain = np.array([-1, 0, 1, 2, 3, -1, 5, 5, 6, 7], dtype=np.int32)
    z = torch.ones((10, 64), dtype=torch.bfloat16)
    assert gpu_labels(z, chain, 0.9).tolist() == [0, 1, 2, 3, 4, 5, 6, 6, 6, 6]
    z[3] = 0                                          # a zero embedding is never linked
    zero = np.array([-1, 0, 0, 0, 0], dtype=np.int32)
    assert gpu_labels(z[:5], zero, 0.5).tolist() == [0, 1, 1, 3, 1]


def test_graph_suffix_matches_oracle():
    wl = W.equiv_batch(prompts=3, schedule=(4, 5, 3, 2), dim=256, seed=11)
    lab = check(wl)
    fo = G.HostForest(wl.parent)
    offs, states = G.graph_suffix(torch.from_numpy(lab).cuda(), fo)
    torch.cuda.synchronize()
    ro, rs = O.graph_suffix(lab, wl.parent)
    say(f"[suffix] {len(rs)} entries")
    assert np.array_equal(offs.cpu().numpy(), ro) and np.array_equal(states.cpu().numpy(), rs)
    # too small a buffer: GA_ERANGE, total reported, outputs untouched
    with pytest.raises(G.GraphAttnError) as e:
        G.graph_suffix(torch.from_numpy(lab).cuda(), fo, capacity=len(rs) - 1)
    assert e.value.status == G.GA_ERANGE


def test_graph_suffix_fixture_on_gpu():
    import json, os
    with open(os.path.join(os.path.dirname(__file__), "golden", "graph_suffix_small.json")) as f:
        fx = json.load(f)
    offs, states = G.graph_suffix(torch.tensor(fx["labels"], dtype=torch.int32).cuda(),
                                  G.HostForest(fx["parent"]))
    torch.cuda.synchronize()
    assert offs.cpu().tolist() == fx["offsets"] and states.cpu().tolist() == fx["states"]


def test_full_batch_sampled_prompts():
    """The benchmark's batch (512 prompts x 205 states, dim 4096): labels of sampled prompts
    against the oracle run on those prompts alone (classes never cross prompts)."""
    wl = W.equiv_batch()
    got = gpu_labels(wl.z, wl.parent, wl.kappa)
    per = 205
    for p in [0, 1, 137, 300, 511]:
        a, b = p * per, (p + 1) * per
        sub = wl.parent[a:b].copy()
        sub[1:] -= a
        zb = wl.z_bits()[a:b]
        assert O.similarity_margin(zb, "bf16", sub, wl.kappa) >= MARGIN
        ref = O.equivalence_classes(zb, "bf16", sub, wl.kappa) + a
        say(f"[equiv] prompt {p}: {len(set(ref.tolist()))} classes")
        assert np.array_equal(got[a:b], ref), p


def test_forest_plan_serves_several_thresholds():
    """One uploaded forest, classes at two thresholds and the suffix of each, against the
    one-shot calls and the oracle."""
    wl = W.equiv_batch(prompts=3, schedule=(4, 5, 3, 2), dim=512, seed=19)
    z = wl.z.cuda()
    with G.Forest(wl.parent) as f:
        for kappa in (0.92, 0.5):
            assert O.similarity_margin(wl.z_bits(), "bf16", wl.parent, kappa) >= MARGIN
            lab = f.classes(z, kappa)
            torch.cuda.synchronize()
            ref = O.equivalence_classes(wl.z_bits(), "bf16", wl.parent, kappa)
            assert np.array_equal(lab.cpu().numpy(), ref)
            ro, rs = O.graph_suffix(ref, wl.parent)
            offs = torch.empty(len(wl.parent) + 1, dtype=torch.int64, device="cuda")
            st = torch.empty(len(rs) + 5, dtype=torch.int32, device="cuda")
            n = f.suffix(lab, offs, st)
            torch.cuda.synchronize()
            assert n == len(rs)
            assert np.array_equal(offs.cpu().numpy(), ro)
            assert np.array_equal(st[:n].cpu().numpy(), rs)


@pytest.mark.parametrize("sizes", [[1], [255, 1, 300], [1024, 1025, 3], [2203], [256, 256, 1]])
def test_suffix_spans(sizes):
    """Prompts below, at and beyond the staged piece of 1,024 states and the block of 256, with
    many linked states, against the oracle; a buffer one entry short leaves both outputs as they
    were."""
    require_gpu()
    rng = np.random.default_rng(sum(sizes))
    parent = []
    for n in sizes:
        s0 = len(parent)
        parent += [-1] + [s0 + int(rng.integers(max(0, v - 30), v)) for v in range(1, n)]
    parent = np.array(parent, dtype=np.int32)
    N = len(parent)
    root = np.maximum.accumulate(np.where(parent < 0, np.arange(N), 0))
    labels = np.arange(N, dtype=np.int32)
    first = {}
    for v in range(N):
        if rng.random() < 0.6:
            labels[v] = first.setdefault((int(root[v]), int(rng.integers(0, 40))), v)
    ro, rs = O.graph_suffix(labels, parent)
    say(f"[case] {sizes}: {len(rs)} entries")
    with G.Forest(parent) as f:
        lab = torch.from_numpy(labels).cuda()
        offs = torch.full((N + 1,), -7, dtype=torch.int64, device="cuda")
        st = torch.full((len(rs) + 3,), -7, dtype=torch.int32, device="cuda")
        if len(rs):
            with pytest.raises(G.GraphAttnError) as e:
                f.suffix(lab, offs, st[:len(rs) - 1])
            assert e.value.status == G.GA_ERANGE
            torch.cuda.synchronize()
            assert (offs == -7).all() and (st == -7).all()
        assert f.suffix(lab, offs, st) == len(rs)
        torch.cuda.synchronize()
        assert np.array_equal(offs.cpu().numpy(), ro)
        assert np.array_equal(st[:len(rs)].cpu().numpy(), rs) and (st[len(rs):] == -7).all()


def test_suffix_of_many_blocks():
    """More than 4,096 blocks of 256 states (the block totals are then scanned by a kernel of
    their own): without classes a state's list is its children."""
    require_gpu()
    n = 210_000
    parent = np.tile(np.array([-1, 0, 0, 1, 1], dtype=np.int32), n)
    parent = np.where(parent < 0, -1, parent + 5 * np.repeat(np.arange(n, dtype=np.int32), 5))
    N = len(parent)
    with G.Forest(parent.astype(np.int32)) as f:
        lab = torch.arange(N, dtype=torch.int32, device="cuda")
        offs = torch.empty(N + 1, dtype=torch.int64, device="cuda")
        st = torch.empty(4 * n, dtype=torch.int32, device="cuda")
        assert f.suffix(lab, offs, st) == 4 * n
        cnt = np.bincount(parent[parent >= 0], minlength=N)
        assert np.array_equal(offs.cpu().numpy(), np.concatenate([[0], np.cumsum(cnt)]))
        assert np.array_equal(st.cpu().numpy(), np.nonzero(parent >= 0)[0])


def ragged_forest(sizes, seed):
    rng = np.random.default_rng(seed)
    parent = []
    for n in sizes:
        s0 = len(parent)
        parent += [-1] + [s0 + int(rng.integers(max(0, v - 30), v)) for v in range(1, n)]
    return np.array(parent, dtype=np.int32)


SIZES = [([1, 2, 15, 16, 17, 33], 64), ([63, 64, 65], 128), ([127, 128, 129], 64),
         ([191, 192, 193, 205], 192), ([255, 256], 64), ([257, 130], 64), ([320, 321], 128),
         ([383, 385], 64), ([517], 192), ([641], 64), ([257, 300, 5] * 5, 64),
         # 64 x 64 tiles (in stages of 64 components) as long as at most 1,024 of them make the
         # batch, with one stage, an odd number and many; 128 x 128 beyond (1,035 here)
         ([449, 300], 64), ([300, 257], 256), ([385], 576), ([257] * 68, 64), ([257] * 69, 128),
         ([517] * 23, 64)]


@pytest.mark.parametrize("sizes,dim", SIZES)
def test_classes_and_similarities_at_tile_edges(sizes, dim):
    """Prompts at the edges of the 16-state strips, of the 64-state blocks of one workgroup and of
    the 64- and 128-state tiles (whole tiles, narrow ones, empty quadrants), and enough of the larger ones
    that their tiles are dealt to the XCDs.  Labels are exact; edge similarities are two fp32 sums
    of `dim` products and a reciprocal root each: within (dim + 8) 2^-24 of the float64 cosine,
    times two for the two norms."""
    require_gpu()
    parent = ragged_forest(sizes, sum(sizes))
    N = len(parent)
    z = W.draw_state_embeddings(parent, dim, sum(sizes), share=2.0)
    zb = z.view(torch.int16).numpy().view(np.uint16)
    kappa = 0.75
    assert O.similarity_margin(zb, "bf16", parent, kappa) >= MARGIN
    ref = O.equivalence_classes(zb, "bf16", parent, kappa)
    zd = z.double().numpy()
    zd /= np.linalg.norm(zd, axis=1, keepdims=True)
    sim = np.where(parent < 0, 0.0, (zd * zd[np.maximum(parent, 0)]).sum(1))
    say(f"[case] {sizes} x {dim}: {len(set(ref.tolist()))} classes")
    with G.Forest(parent) as f:
        es = torch.full((N,), -7.0, dtype=torch.float32, device="cuda")
        for _ in range(2):                            # (the second call finds the first's scratch)
            lab = f.classes(z.cuda(), kappa, edge_sim=es)
            torch.cuda.synchronize()
            assert np.array_equal(lab.cpu().numpy(), ref)
        err = float(np.abs(es.cpu().numpy().astype(np.float64) - sim).max())
        say(f"[equiv] similarity max|d| = {err:.1e}")
        assert err <= 2 * (dim + 8) * 2.0 ** -24
        assert np.array_equal(f.classes(z.cuda(), kappa).cpu().numpy(), ref)


@pytest.mark.parametrize("n,dim", [(1, 64), (40, 512), (205, 4096), (256, 2048), (300, 1024), (517, 64)])
def test_a_prompt_has_the_same_bits_anywhere(n, dim):
    """One prompt alone, and at many places among other prompts (so many that the larger prompts
    change from 64 x 64 to 128 x 128 tiles): the same bits of its similarities and the same classes
    (also for a threshold at one of its own cosines, where the last bit decides)."""
    require_gpu()
    rng = np.random.default_rng(n)
    fill = 12
    one, other = ragged_forest([n], n), ragged_forest([fill], 3)
    zo = W.draw_state_embeddings(one, dim, n, share=2.0)
    parts, zs, at = [], [], []
    pos = 0
    for k in range(17 if n <= 256 else 69):
        parts.append(np.where(one < 0, -1, one + pos))
        zs.append(zo)
        at.append(pos)
        pos += n
        for _ in range(int(rng.integers(1, 12))):
            parts.append(np.where(other < 0, -1, other + pos))
            zs.append(torch.randn((fill, dim), generator=torch.Generator().manual_seed(pos)).bfloat16())
            pos += fill
    z, parent = torch.cat(zs).cuda(), np.concatenate(parts).astype(np.int32)

    def classes(par, emb, kappa):
        with G.Forest(par) as f:
            es = torch.full((len(par),), -7.0, dtype=torch.float32, device="cuda")
            lab = f.classes(emb, kappa, edge_sim=es)
            torch.cuda.synchronize()
            return lab.cpu().numpy(), es.cpu().numpy()

    lab1, es1 = classes(one, zo.cuda(), 0.75)
    for kappa in {0.75, float(np.sort(es1)[n // 2])}:
        lab1, es1 = classes(one, zo.cuda(), kappa)
        lab, es = classes(parent, z, kappa)
        for a in at:
            assert np.array_equal(es[a:a + n].view(np.int32), es1.view(np.int32)), (kappa, a)
            assert np.array_equal(lab[a:a + n] - a, lab1), (kappa, a)
    say(f"[case] {n} x {dim}: {len(at)} places, {len(parent)} states")
