"""The multi-query attention kernel (bf16 plans with many query rows per page) at the sizes where it
can go wrong, against the fp64 CPU oracle: the last row block's remainder, odd and single pages,
the ring's start and end (1 to 11 pages), chunks of up to 128 pages, causal origins inside a chain
with ragged pages, one to eight query heads per kv-head, rows written by the kernel itself (one
partial each, bf16) and rows folded by the merge (several partials each, or float32 output).

Which kernel a plan takes shows in its chunks: these plans are small, and the kernel for few query rows
per page would cut them below 16 pages, which this one never does.  Who wrote the rows shows in their
bits: the merge rounds its float32 result to bf16, so a merged bf16 output is the float32 one rounded,
while rows written by the kernel have not been through an fp16 partial and differ here and there.

Tolerance: the parity bar of bf16 inputs, max |out - oracle| <= 1e-2 and max |lse - oracle| <= 1e-3.
Probabilities are rounded to bf16 (relative 2^-9) before a convex combination of values below 5, and
the output once more, so 2 x 2^-9 x max|out| < 1e-2 wherever |out| < 2.5; contexts of a few tokens,
where outputs are single values, take float32 output, or more than 40 tokens.
Unused slots and free pages hold NaN in every case.
"""
import os
import re
import subprocess

import numpy as np
import pytest
import torch

from oracle import graphattn_oracle as O
from paper_2606_18954_amd import graphattn as G
from paper_2606_18954_amd import workloads as W

from gpu_util import compare, params_of, require_gpu, say


def _run(lens, paths, counts, Hq, Hkv, D, seed, out_f32, rows=None, one_partial=None, chunk=None):
    require_gpu()
    g = W.assemble_graph(lens, paths, seed, 3)
    wl = W.make_extend_workload(f"mq {Hq}/{Hkv}/{D} lens={lens[:4]} counts={counts[:4]}", g, counts,
                                Hq, Hkv, D, "bf16", seed, poison=True)
    R = int(np.sum(counts))
    q, pool = wl.q.cuda(), wl.pool.cuda()
    out = torch.full((R, Hq, D), float("nan"), dtype=torch.float32 if out_f32 else q.dtype,
                     device="cuda")
    lse = torch.full((R, Hq), float("nan"), dtype=torch.float32, device="cuda")
    say(f"[case] {wl.name} R={R} f32={out_f32}")
    with G.Plan(G.HostGraph.from_graph(g), params_of(wl, out_f32=out_f32),
                query_counts=wl.query_counts) as pl:
        inf = pl.info()
        assert inf.workgroups_per_cu == (3 if D == 64 else 2) and inf.chunk_pages >= 16
        if chunk is not None:
            assert inf.chunk_pages == chunk
        if one_partial is not None:
            assert (inf.num_partial_rows == R) == one_partial
        for _ in range(2):                  # (the second run starts from re-armed work streams)
            pl.schedule()
            pl.run(q, pool, out, lse)
            torch.cuda.synchronize()
            first = (out.clone(), lse.clone())
        pl.run(q, pool, out, lse)           # and a third on the same schedule
        torch.cuda.synchronize()
        assert torch.equal(first[0], out) and torch.equal(first[1], lse)
    if not out_f32:
        o32 = torch.empty((R, Hq, D), dtype=torch.float32, device="cuda")
        with G.Plan(G.HostGraph.from_graph(g), params_of(wl, out_f32=True),
                    query_counts=wl.query_counts) as pl:
            pl.run(q, pool, o32, lse)
        differ = (o32.to(out.dtype) != out).sum().item()
        say(f"[mq] {differ} of {out.numel()} values are not the merge's")
        assert (differ > 0) == (inf.num_partial_rows == R)
        lse = first[1]
    oo, ol = O.extend(wl.q_bits(), wl.pool_bits(), g.seg_len, g.seg_page_offsets, g.seg_pages,
                      g.path_offsets, g.path_segs, wl.query_counts, Hq, Hkv, D, "bf16", rows=rows)
    go, gl = out.double().cpu().numpy(), lse.double().cpu().numpy()
    if rows is not None:
        go, gl = go[rows], gl[rows]
    compare(wl.name, go, gl, oo, ol)


@pytest.mark.gpu
@pytest.mark.parametrize("Hq,Hkv,D", [(28, 4, 128), (8, 1, 64), (5, 5, 128), (6, 3, 64)])
@pytest.mark.parametrize("tokens,queries", [(19, 19), (33, 32), (65, 37), (100, 100), (130, 129),
                                            (161, 40), (176, 176)])
def test_one_prompt(Hq, Hkv, D, tokens, queries):
    """2 to 11 pages, all in one chunk: every remainder of the ring; one partial a row, merged (float32
    output) and, with enough tokens for the tolerance, written directly."""
    if queries * (Hq // Hkv) < 128:
        counts, lens, paths = [queries] * 8, [2000] + [tokens] * 8, [[0, 1 + b] for b in range(8)]
        if 8 * queries * (Hq // Hkv) < 128:
            pytest.skip("too few rows for this kernel")
        _run(lens, paths, counts, Hq, Hkv, D, 50 + tokens, True)
    else:
        _run([tokens], [[0]], [queries], Hq, Hkv, D, 50 + tokens, True, one_partial=True)
        if tokens - queries >= 40:
            _run([tokens], [[0]], [queries], Hq, Hkv, D, 51 + tokens, False, one_partial=True)


@pytest.mark.gpu
@pytest.mark.parametrize("Hq,Hkv,D", [(28, 4, 128), (4, 1, 64)])
def test_rows_written_by_the_kernel(Hq, Hkv, D):
    """bf16 outputs without a merge: ragged prompts of 41 to 700 tokens whose last tokens are
    queries, four row blocks and more each, last blocks of every size."""
    rng = np.random.default_rng(8)
    lens = [int(x) for x in rng.integers(120, 250, size=6)]
    counts = [int(n) - 41 - int(rng.integers(0, 20)) for n in lens]
    _run(lens, [[i] for i in range(6)], counts, Hq, Hkv, D, 61, False, one_partial=True)


@pytest.mark.gpu
@pytest.mark.parametrize("out_f32", [True, False])
def test_several_chunks(out_f32):
    """Prompts of 2048 tokens and a chain that ends mid-page, many row blocks, three chunks of 43 pages
    at most, sampled rows."""
    lens = [2048, 2031, 1500, 517]
    paths = [[0], [1], [2, 3]]
    counts = [2048, 1900, 500]
    rows = sorted(set([0, 1, 2047, 2048, 3947, 3948, 4447] + list(range(5, 4448, 211))))
    _run(lens, paths, counts, 28, 4, 128, 71, out_f32, rows=rows, one_partial=False)


@pytest.mark.gpu
@pytest.mark.parametrize("out_f32", [True, False])
def test_chunks_of_up_to_128_pages(out_f32):
    """Units of 128, 127 and 128 pages (both halves of the page words and of the mask's bits; the
    longest a descriptor takes), one partial a row: prompts whose every token is a query, enough of
    them that the step is not cut finer; a prompt of whose 2,031 tokens the last 700 are queries; and a
    chain whose first segment ends inside page 94, with its causal origin after it.  Rows are sampled
    around the page pairs 31 to 33, the short page and the ends."""
    lens = [2048] * 5 + [2031, 1517, 517]
    paths = [[i] for i in range(6)] + [[6, 7]]
    counts = [2048] * 5 + [700, 500]
    at = np.concatenate([[0], np.cumsum(counts)])
    rows = [0, 1, 40, 700, 1007, 1008, 1023, 1024, 1025, 1040, 1500, 2046, 2047]
    rows += [int(at[3]) + r for r in (63, 991, 1056, 2047)]
    rows += [int(at[5]) + r for r in (0, 1, 350, 684, 699)]
    rows += [int(at[6]) + r for r in (0, 7, 8, 250, 498, 499)]
    if not out_f32:
        rows = [r for r in rows if not r < 40]
    _run(lens, paths, counts, 28, 4, 128, 91, out_f32, rows=rows, one_partial=True, chunk=128)


@pytest.mark.gpu
def test_shared_prefix_and_ragged_chains():
    """Shared and private segments, ragged pages inside chains, counts below the step's length."""
    lens = [400, 17, 3, 33, 16, 21, 50, 40, 64]
    paths = [[0, 1, 2, 3], [0, 4, 5], [0, 1, 6], [0, 7], [0, 8]]
    counts = [30, 21, 47, 40, 64]
    for Hq, Hkv, D in [(28, 4, 128), (16, 2, 64)]:
        _run(lens, paths, counts, Hq, Hkv, D, 81, True)


@pytest.mark.gpu
def test_rows_written_directly_need_no_partial_buffers():
    """A plan whose rows the kernel writes itself allocates no partial rows (here 4000 x 28 x 264
    bytes, 28 MiB); with float32 output, which is merged, it does."""
    require_gpu()
    lens = [250] * 16
    g = W.assemble_graph(lens, [[i] for i in range(16)], 3, 0)
    torch.cuda.synchronize()
    took = {}
    for out_f32 in (False, True):
        p = G.make_params(28, 4, 128, g.num_pages, "bf16", 0.0, out_f32)
        free = torch.cuda.mem_get_info()[0]
        with G.Plan(G.HostGraph.from_graph(g), p, query_counts=lens) as pl:
            assert pl.info().num_partial_rows == 4000
            took[out_f32] = free - torch.cuda.mem_get_info()[0]
    say(f"[case] bytes of a plan: {took}")
    assert took[True] - took[False] >= 4000 * 28 * 264 - (4 << 20)


def test_generated_code(tmp_path):
    """The copies write M0 by inline assembly, so every M0 write must feed one, and no kernel may
    spill (a spill's loads would wait for the copies in flight)."""
    from paper_2606_18954_amd import build_lib
    if not os.path.exists(build_lib.HIPCC):
        pytest.skip("hipcc not available")
    out = tmp_path / "mq.s"
    flags = [f for f in build_lib.CFLAGS if f != "-fPIC"]
    subprocess.run([build_lib.HIPCC, *flags, "-x", "hip", "-S", "--cuda-device-only",
                    os.path.join(build_lib.CSRC, "mq_attn.hip"), "-o", str(out)], check=True,
                   capture_output=True)
    text = out.read_text()
    parts = re.split(r"^(_ZN2ga\w*k_mq_attn\w*):", text, flags=re.M)
    assert len(parts) == 5
    for body in parts[2::2]:
        assert int(re.search(r"ScratchSize:\s+(\d+)", body).group(1)) == 0
        lines = [l.strip() for l in body.split("s_endpgm")[0].splitlines()
                 if l.strip() and not l.strip().startswith((";", "."))]
        for i, l in enumerate(lines):
            if re.search(r"\bm0\b", l):
                assert re.match(r"s_mov_b32 m0, (s\d+|vcc_lo|vcc_hi)$", l), l
                assert lines[i + 1].startswith("global_load_lds_dwordx4"), lines[i + 1]
