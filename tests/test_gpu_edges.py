"""Sizes at the edges of what the kernels' tiles, parts and dispatch rules cover, each against the
oracle (whole outputs exact except on draws it flags; group probabilities within 1e-5).  Run with
``-m gpu`` on an MI355X."""
import numpy as np
import pytest
import torch

import oracle
import paper_2511_13732_amd as pcg
import workloads as W
from parity import (as_oracle_logits, compare_thinning, compare_verify, group_probs_error, oracle_groups,
                    run_both, run_both_thinning)
from test_gpu_asg import as_bf16_tensor, compare_groups
from test_gpu_propose import compare_proposals
from test_oracle_asg import bf16_to_f64, embeddings, stepped_rows

pytestmark = pytest.mark.gpu


def rows_at(x: torch.Tensor, off: int) -> torch.Tensor:
    """The same rows as a view that starts `off` elements into a larger buffer, rows `off` apart."""
    B, n, V = x.shape
    big = torch.full((B, n, V + off), 9.0, dtype=x.dtype, device="cuda")
    big[:, :, off:] = x.cuda()
    return big[:, :, off:]


def with_long_groups(V, rp, mem, longs):
    """The membership with groups of the given sizes put between its own, evenly, the first one ahead."""
    rng = np.random.default_rng([V, *longs])
    sets = np.split(mem, rp[1:-1])
    for i, n in enumerate(longs):
        sets.insert(i * len(sets) // len(longs), np.sort(rng.choice(V, n, replace=False)).astype(np.int32))
    return np.concatenate([[0], np.cumsum([len(s) for s in sets])]).astype(np.int32), np.concatenate(sets)


def check_step(V, G, size, B, K, dtype, off=0, layout="prepared", chunk_groups=0, weighted=False, seed=0,
               thinning=True, sigma=4.0, longs=()):
    print(f"V={V} G={G} size={size} B={B} K={K} {dtype} off={off} {layout} {chunk_groups} w={weighted}", flush=True)
    rp, mem = W.random_groups(V, G, 1, size, seed=seed + V)
    if longs:
        rp, mem = with_long_groups(V, rp, mem, longs)
    og = oracle_groups(V, rp, mem)
    w = W.random_weights(og.V, og.members, seed) if weighted else None
    if weighted:
        og = oracle.with_weights(og, w)
    dg = pcg.Groups.from_csr(V, rp, mem, "cuda", prepare=layout == "prepared", chunk_groups=chunk_groups,
                             reverse=True, weights=w)
    rev = oracle.reverse_index(og)
    rng = np.random.default_rng([V, G, B, K, seed])
    tgt = (sigma * rng.standard_normal((B, K + 1, V))).astype(np.float32)
    dft = (tgt[:, :K] + rng.standard_normal((B, K, V))).astype(np.float32)
    tgt, dft = torch.from_numpy(tgt), torch.from_numpy(dft)
    if dtype == "bf16":
        tgt, dft = tgt.to(torch.bfloat16), dft.to(torch.bfloat16)
    tgt, dft = rows_at(tgt, off), rows_at(dft, off)
    pref = oracle.propose(og, rev, as_oracle_logits(dft), temperature=0.9, seed=3, offset=1, nthreads=8)
    if thinning:
        tok, grp = pcg.propose(dg, dft, temperature=0.9, seed=3, offset=1)
        assert compare_proposals(tok, grp, pref, og).tolerated <= 1
    for step in range(2):
        gpu, ref, _, diag = run_both(V, rp, mem, tgt, dft, pref.tokens, pref.groups, temperature=0.9, seed=3,
                                     offset=step, dg=dg, og=og, nthreads=8)
        assert compare_verify(gpu, ref, og, pref.tokens, pref.groups).tolerated <= 1
        assert diag["sequences"] == B and diag["accepted_total"] == int(gpu.accept_len.sum())
        if thinning:
            g2, trials, r2, _ = run_both_thinning(V, tgt, dft, pref.tokens, pref.groups, dg=dg, og=og, rev=rev,
                                                  temperature=0.9, seed=3, offset=step, nthreads=8)
            assert compare_thinning(g2, trials, r2, og, pref.tokens, pref.groups).tolerated <= 1
    out = pcg.group_probs(dg, tgt[:, 0], 0.9)
    # the terms' own error, and n 2^-24 for the one running sum of a group of n entries (see pcg.h)
    tol = 1e-5 + max(longs, default=0) * 2.0 ** -24
    assert group_probs_error(out, oracle.group_probs(og, as_oracle_logits(tgt[:, 0]), 0.9)) <= tol


# rows of less than one 16-byte piece, of one, around a part of 2048, and around several; every
# start inside 16 bytes
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V,off", [(3, 0), (4, 1), (7, 0), (8, 3), (9, 5), (33, 7), (2040, 1), (2047, 0),
                                   (2049, 2), (2055, 3), (6143, 6), (8193, 1), (20011, 7)])
def test_ragged_rows(V, off, dtype):
    check_step(V, max(1, V // 3), min(V, 9), 3, 2, dtype, off=off)


# the prepared gather: blocks with fewer steps than it keeps in flight, blocks without any in some
# tile (or in all), one to three tiles, one to four blocks per wave, with and without weights
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("V,G,size,chunk", [(900, 4096, 1, 4096), (5000, 700, 40, 4096), (45000, 5000, 3, 4096),
                                            (45001, 300, 400, 8192), (45000, 17000, 9, 16384),
                                            (90002, 9000, 2, 12288), (81400, 40000, 5, 16384)])
def test_prepared_gather_blocks(V, G, size, chunk, weighted):
    check_step(V, G, size, 2, 2, "bf16", chunk_groups=chunk, weighted=weighted, thinning=False)


# the CSR gather: fewer than four entries, every number of lanes per group, groups longer than one trip
# and empty ones, one to four tiles, more chunks than the chunk totals have room for (129 in the last: the last
# kernel takes their totals 64 at a time), few and many rows
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("V,G,size,B", [(3, 1, 3, 1), (5, 1, 5, 3), (700, 900, 6, 1), (700, 900, 14, 300),
                                        (3000, 2500, 29, 5), (9000, 400, 90, 2), (20000, 40000, 8, 2),
                                        (45003, 20001, 17, 1), (81000, 300, 700, 3), (100003, 3000, 60, 12),
                                        (30011, 66000, 40, 1)])
def test_csr_gather(V, G, size, B, weighted):
    check_step(V, G, size, B, 2, "bf16", layout="csr", weighted=weighted, thinning=False)


# the last kernel reads all sums up to 4096 groups and totals beyond; 32 lanes a group up to 4096 groups of more
# than 32 entries and 8 rows, 2048 and 16 rows
@pytest.mark.parametrize("V,G,size,B", [(17000, 4096, 70, 2), (17000, 4097, 70, 2), (17000, 4096, 70, 9), (17000, 2048, 90, 9),
                                        (17000, 4096, 9, 3), (17000, 1, 40, 2), (17000, 511, 66, 2)])
@pytest.mark.parametrize("weighted", [False, True])
def test_csr_few_groups(V, G, size, B, weighted):
    check_step(V, G, size, B, 2, "f32", layout="csr", weighted=weighted, thinning=False)


# groups far above the mean size, which a whole wave of the CSR gather sums: right at the size where that
# begins (64 entries for every lane a group has), past one and several turns of the wave, all tokens; every
# number of lanes, several tiles, the step in one kernel
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("V,G,size,B,longs", [(20000, 9000, 7, 3, (128, 129, 130, 1500, 20000)), (20000, 3000, 20, 2, (256, 257, 1281, 4000)),
                                              (45003, 3000, 40, 2, (512, 513, 2049, 9000)), (81000, 2000, 90, 3, (1024, 1025, 1089, 5000)),
                                              (4000, 3000, 9, 2, (256, 257, 1300, 4000)), (700, 500, 5, 300, (257, 700))])
def test_csr_long_groups(V, G, size, B, longs, weighted):
    check_step(V, G, size, B, 2, "bf16", layout="csr", weighted=weighted, thinning=False, longs=longs)


# the last kernel: groups that end with a lane's first entry, its fourth, with one wave's four turns and beyond,
# and those the whole workgroup sums, in both of its forms (mean size up to 32 and above)
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("layout", ["prepared", "csr"])
@pytest.mark.parametrize("G,size,longs", [(200, 20, (31, 32, 33, 64, 65) * 40 + (255, 256, 257, 700, 5000) * 3),
                                          (200, 90, (127, 128, 129, 33, 32) * 40 + (255, 256, 257, 700, 5000) * 8)])
def test_draws_from_groups_of_every_size(G, size, longs, layout, weighted):
    check_step(20000, G, size, 48, 2, "bf16", layout=layout, weighted=weighted, thinning=False, longs=longs)


# the step in one and in two kernels, and the sizes right beside them: the smallest row, rows of one part
# and more, the most positions, the most tokens and groups the LDS holds, several chunks, batches on
# either side of the rule's lines, the batch beyond it
@pytest.mark.parametrize("layout,weighted", [("prepared", False), ("prepared", True), ("csr", False), ("csr", True)])
@pytest.mark.parametrize("V,G,size,B,K,dtype,off", [
    (8, 5, 4, 2, 1, "bf16", 0), (9, 2, 5, 3, 64, "f32", 1), (1023, 1025, 8, 5, 4, "bf16", 3), (2049, 4101, 3, 2, 8, "f32", 0),
    (4095, 2000, 20, 1, 8, "bf16", 5), (16384, 16384, 3, 208, 1, "bf16", 0), (16383, 16001, 4, 209, 1, "f32", 2),
    (16384, 16385, 3, 208, 1, "bf16", 0), (4097, 4097, 9, 3, 8, "bf16", 1), (8192, 8000, 30, 2, 7, "f32", 0),
    (8193, 9001, 7, 128, 1, "bf16", 3), (12000, 9000, 12, 127, 1, "bf16", 0), (1500, 1500, 9, 2, 33, "f32", 1), (300, 200, 9, 256, 2, "f32", 0), (300, 200, 9, 257, 2, "bf16", 0)])
def test_small_step(V, G, size, B, K, dtype, off, layout, weighted):
    check_step(V, G, size, B, K, dtype, off=off, layout=layout, weighted=weighted, thinning=False, chunk_groups=4096)


# rows of one part in one launch, whose statistics the wave that reduced them finishes, a row per lane: one row
# a wave, two and three, up to the nine of the most positions, few sequences and one per compute unit; the
# longest such row and the first that has two parts
@pytest.mark.parametrize("V,B,K,dtype", [(1024, 3, 7, "bf16"), (1024, 3, 8, "f32"), (2048, 2, 10, "bf16"), (1500, 129, 8, "bf16"),
                                         (2048, 130, 15, "f32"), (2048, 129, 16, "bf16"), (2049, 129, 16, "bf16"),
                                         (700, 131, 24, "bf16"), (300, 256, 64, "f32")])
@pytest.mark.parametrize("layout", ["prepared", "csr"])
def test_small_step_rows_of_one_part(V, B, K, dtype, layout):
    # the draft's rows are the target's up to a position, where every proposal is accepted: the decision falls
    # on rows of every lane
    print(f"V={V} B={B} K={K} {dtype} {layout}", flush=True)
    rp, mem = W.random_groups(V, V, 1, 8, seed=V + K)
    og = oracle_groups(V, rp, mem)
    dg = pcg.Groups.from_csr(V, rp, mem, "cuda", prepare=layout == "prepared", reverse=True)
    rng = np.random.default_rng([V, B, K])
    tgt = torch.from_numpy((3.0 * rng.standard_normal((B, K + 1, V))).astype(np.float32))
    moved = torch.from_numpy(rng.integers(0, K + 1, B))                 # the first position where the rows differ
    noise = torch.from_numpy(rng.standard_normal((B, K, V)).astype(np.float32))
    dft = tgt[:, :K] + torch.where((torch.arange(K)[None] >= moved[:, None])[..., None], noise, torch.zeros(()))
    if dtype == "bf16":
        tgt, dft = tgt.to(torch.bfloat16), dft.to(torch.bfloat16)
    pref = oracle.propose(og, oracle.reverse_index(og), as_oracle_logits(dft), temperature=0.9, seed=3, offset=1, nthreads=8)
    gpu, ref, _, diag = run_both(V, rp, mem, tgt, dft, pref.tokens, pref.groups, temperature=0.9, seed=3, offset=4,
                                 dg=dg, og=og, nthreads=8)
    assert compare_verify(gpu, ref, og, pref.tokens, pref.groups).tolerated <= 1
    assert diag["sequences"] == B and diag["accepted_total"] == int(gpu.accept_len.sum())
    if B > 2 * K:
        assert len(np.unique(gpu.accept_len.cpu().numpy())) > K // 2


def groups_of_one_size(V, size, moved):
    sets = [(g + np.arange(size)) % V for g in range(V)]
    sets = [np.sort(x).astype(np.int32) for x in sets]
    if moved == "one":
        sets[9] = np.sort(np.append(sets[9], np.int32((9 + size) % V)))
        sets[5] = sets[5][:-1] if size > 1 else sets[5][:0]
    if moved == "emptied":
        sets[7] = np.sort(np.concatenate([(7 + np.arange(3 * size)) % V])).astype(np.int32)
        sets[6] = sets[8] = np.zeros(0, np.int32)
    rp = np.concatenate([[0], np.cumsum([len(x) for x in sets])]).astype(np.int32)
    return rp, np.concatenate(sets)


# groups of one size, which are looked up before their bounds are known, around the 64 entries of a wave; and
# of one size on average only: an entry moved from one group to a later one, so that those between start
# elsewhere, or two groups emptied into a third; with the rows of a step streamed or cached, its probes in
# two launches and in four
@pytest.mark.parametrize("V,B,K,dtype,size,moved", [
    (V, B, K, dtype, size, moved) for V, B, K, dtype in [(17003, 3, 6, "bf16"), (4100, 2, 9, "f32")]
    for size in (1, 8, 64, 65, 130) for moved in ("none", "one", "emptied")] +
    [(65536, 16, 17, "bf16", 8, "one"), (65536, 21, 17, "bf16", 8, "one"), (65536, 22, 17, "bf16", 8, "one")])
def test_groups_of_one_size(V, B, K, dtype, size, moved):
    print(f"V={V} B={B} K={K} {dtype} size={size} {moved}", flush=True)
    rp, mem = groups_of_one_size(V, size, moved)
    rng = np.random.default_rng([V, size])
    ptok = rng.integers(0, V, (B, K)).astype(np.int32)
    pgrp = np.where(rng.random((B, K)) < 0.7, rng.integers(0, 14, (B, K)), rng.integers(0, V, (B, K))).astype(np.int32)
    tgt = torch.from_numpy((3 * rng.standard_normal((B, K + 1, V))).astype(np.float32))
    dft = tgt[:, :K] + torch.from_numpy((0.3 * rng.standard_normal((B, K, V))).astype(np.float32))
    if dtype == "bf16":
        tgt, dft = tgt.to(torch.bfloat16), dft.to(torch.bfloat16)
    og = oracle_groups(V, rp, mem)
    for prepare in (True, False):
        dg = pcg.Groups.from_csr(V, rp, mem, "cuda", prepare=prepare)
        gpu, ref, _, diag = run_both(V, rp, mem, tgt, dft, ptok, pgrp, seed=11, offset=2, dg=dg, og=og, nthreads=8)
        assert compare_verify(gpu, ref, og, ptok, pgrp).tolerated <= 1
        assert diag["bad_proposal"] == 0 and diag["sequences"] == B


# the same with weights, which are looked up with the members: proposals of the groups that are not where they
# are looked for (their entries' weights taken from there instead would change 7 to 38 of the sequences)
@pytest.mark.parametrize("V,B,dtype", [(4100, 100, "f32"), (17003, 60, "bf16")])
@pytest.mark.parametrize("size", [8, 64, 65])
@pytest.mark.parametrize("moved", ["none", "one", "emptied"])
def test_weights_of_groups_of_one_size(V, B, dtype, size, moved, K=8):
    print(f"V={V} B={B} {dtype} size={size} {moved}", flush=True)
    rp, mem = groups_of_one_size(V, size, moved)
    og = oracle_groups(V, rp, mem)
    w = W.random_weights(og.V, og.members, 1)
    og = oracle.with_weights(og, w)
    rng = np.random.default_rng([V, size])
    ptok = rng.integers(0, V, (B, K)).astype(np.int32)
    pgrp = rng.choice([5, 7, 7, 9] if moved == "emptied" else [5, 6, 7, 8, 9], (B, K)).astype(np.int32)
    tgt = torch.from_numpy((3 * rng.standard_normal((B, K + 1, V))).astype(np.float32))
    dft = tgt[:, :K] + torch.from_numpy(rng.standard_normal((B, K, V)).astype(np.float32))
    if dtype == "bf16":
        tgt, dft = tgt.to(torch.bfloat16), dft.to(torch.bfloat16)
    for prepare in (True, False):
        dg = pcg.Groups.from_csr(V, rp, mem, "cuda", prepare=prepare, weights=w)
        gpu, ref, _, diag = run_both(V, rp, mem, tgt, dft, ptok, pgrp, seed=11, offset=2, dg=dg, og=og, nthreads=8)
        assert compare_verify(gpu, ref, og, ptok, pgrp).tolerated <= 1
        assert diag["bad_proposal"] == 0 and diag["sequences"] == B


# more entries in the arrays than the groups have, as many as make them divide evenly among the groups: the
# proposed groups are looked up where they are not, among token ids that are none
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("layout", ["prepared", "csr"])
@pytest.mark.parametrize("V,G,size,B,K,dtype", [(17003, 900, 40, 3, 6, "bf16"), (17003, 300, 130, 2, 5, "f32"), (4100, 4090, 9, 2, 9, "f32")])
def test_entries_behind_the_last_group(V, G, size, B, K, dtype, layout, weighted):
    print(f"V={V} G={G} size={size} {layout} w={weighted}", flush=True)
    rp, mem = W.random_groups(V, G, 1, size, seed=V + G)
    og = oracle_groups(V, rp, mem)
    w = W.random_weights(og.V, og.members, 1) if weighted else None
    if weighted:
        og = oracle.with_weights(og, w)
    dg = pcg.Groups.from_csr(V, rp, mem, "cuda", prepare=layout == "prepared", weights=w)
    nnz = (dg.nnz // dg.G + 3) * dg.G
    none = torch.tensor([2 ** 31 - 1, -2 ** 31, V, -1], dtype=torch.int32, device="cuda").repeat(nnz // 4 + 1)
    members = torch.cat([dg.members[:dg.nnz], none[:nnz - dg.nnz]])
    weights = None if w is None else torch.cat([dg.weights, torch.full((nnz - dg.nnz,), 3.0, device="cuda")])
    dg = pcg.Groups(V, dg.row_ptr, members, dg.mult, nnz, dg.prepared, dg.prepared_info, weights=weights)
    rng = np.random.default_rng([V, G])
    ptok = rng.integers(0, V, (B, K)).astype(np.int32)
    pgrp = rng.integers(0, og.G, (B, K)).astype(np.int32)
    pgrp[:, -2:] = og.G - 1 - rng.integers(0, 4, (B, 2))
    tgt = torch.from_numpy((3 * rng.standard_normal((B, K + 1, V))).astype(np.float32))
    dft = tgt[:, :K] + torch.from_numpy((0.05 * rng.standard_normal((B, K, V))).astype(np.float32))
    if dtype == "bf16":
        tgt, dft = tgt.to(torch.bfloat16), dft.to(torch.bfloat16)
    for step in range(3):
        gpu, ref, _, diag = run_both(V, rp, mem, tgt, dft, ptok, pgrp, seed=11, offset=step, dg=dg, og=og, nthreads=8)
        assert compare_verify(gpu, ref, og, ptok, pgrp).tolerated <= 1
        assert diag["bad_proposal"] == 0 and diag["sequences"] == B


# construction of the groups: tokens around the blocks of the scan, rows that fill the registers of the
# pair kernel and rows beyond, sets of 63 to 66 members (ranked in registers or sorted in LDS), more
# duplicates of a set than one look at its members covers
@pytest.mark.parametrize("V,d,theta,centres,sigma", [(1023, 64, 0.2, 0, 0), (1024, 1024, 0.05, 0, 0), (1025, 1088, 0.05, 0, 0),
                                                     (2049, 2112, 0.04, 0, 0), (640, 64, 0.6, 10, 0.3), (650, 128, 0.6, 10, 0.2),
                                                     (660, 192, 0.5, 10, 0.4), (900, 64, 0.9, 6, 0.02)])
def test_group_construction_edges(V, d, theta, centres, sigma):
    E = embeddings(V, d, 7, centres, sigma)[0] if centres else embeddings(V, d, 7)
    got = pcg.asg_build_exact(torch.from_numpy(E).cuda(), theta, cap=64)
    t = compare_groups(got, oracle.asg_build_exact(E, theta, nthreads=8), f"exact V={V} d={d}")
    assert t.flagged_group == 0 and t.tolerated == 0
    bits = oracle.asg_normalize(E)
    ref = oracle.asg_build(bits, theta, nthreads=8)
    assert compare_groups(pcg.asg_build(as_bf16_tensor(bits).cuda(), theta, cap=64), ref, f"V={V} d={d}").tolerated <= 2


# the scan over the tokens in one launch and in two, an unfinished block of it, and lists of more than 64
# entries, undecided pairs among them
@pytest.mark.parametrize("V,d,theta,centres,sigma", [(8192, 64, 0.45, 0, 0), (8193, 64, 0.45, 0, 0), (9217, 64, 0.45, 0, 0),
                                                     (4000, 64, 0.8, 40, 0.3)])
def test_group_construction_scan(V, d, theta, centres, sigma):
    E = embeddings(V, d, 11, centres, sigma)[0] if centres else embeddings(V, d, 11)
    got = pcg.asg_build_exact(torch.from_numpy(E).cuda(), theta, cap=64)
    t = compare_groups(got, oracle.asg_build_exact(E, theta, nthreads=16), f"exact V={V}")
    assert t.flagged_group == 0 and t.tolerated == 0
    assert got.max_size >= int(np.diff(got.row_ptr.cpu().numpy()).max()) and (got.max_size > 64) == (centres > 0)


def test_group_construction_where_rounding_moves_most():
    """Rows whose components all round the same way: similarities off by up to 7e-3, where a band of
    2^-8 + 2^-18 + d 2^-23 around the threshold would leave pairs on the wrong side of it."""
    E, m = stepped_rows(400, 3712, 2900)
    theta = float(np.float32(0.98))
    U = bf16_to_f64(oracle.asg_normalize(E))
    rounded, cos = U @ U.T, np.sqrt(np.minimum.outer(m, m) / np.maximum.outer(m, m))
    outside = np.abs(rounded - theta) > 2.0 ** -8 + 2.0 ** -18 + 3712 * 2.0 ** -23
    assert (outside & ((rounded > theta) != (cos > theta))).sum() > 100
    t = compare_groups(pcg.asg_build_exact(torch.from_numpy(E).cuda(), theta), oracle.asg_build_exact(E, theta, nthreads=8), "stepped")
    assert t.flagged_group == 0 and t.tolerated == 0


def test_group_construction_beside_a_row_that_is_not_finite():
    """A token whose embedding holds an infinity or a NaN is in no other token's group, and the
    others' groups are what they are without it."""
    E = embeddings(700, 128, 9)
    want = pcg.asg_build_exact(torch.from_numpy(E[:698]).cuda(), 0.15)
    E[698, 5], E[699, 7] = np.inf, np.nan
    got = pcg.asg_build_exact(torch.from_numpy(E).cuda(), 0.15)
    assert got.G == want.G + 2 and got.nnz == want.nnz + 2
    assert torch.equal(got.members[:want.nnz], want.members) and torch.equal(got.row_ptr[:want.G + 1], want.row_ptr)


# proposals: a draft row in one workgroup up to 64 parts (V = 131 072), in two launches beyond; one row,
# more rows than compute units; rows of less than one 16-byte piece
@pytest.mark.parametrize("V,B,K,dtype,off", [(2, 3, 2, "f32", 0), (5, 300, 3, "bf16", 1), (2048, 1, 1, "bf16", 0),
                                             (32769, 5, 3, "f32", 3), (131072, 2, 1, "bf16", 0), (131073, 2, 2, "bf16", 5)])
def test_propose_rows(V, B, K, dtype, off):
    rp, mem = W.random_groups(V, max(1, V // 2), 1, min(V, 5), seed=V) if V < 100000 else \
        (np.arange(V + 1, dtype=np.int32), np.arange(V, dtype=np.int32)[::-1].copy())
    og = oracle_groups(V, rp, mem)
    dg = pcg.Groups.from_csr(V, rp, mem, "cuda", prepare=False, reverse=True)
    rng = np.random.default_rng([V, B, K])
    x = torch.from_numpy((3.0 * rng.standard_normal((B, K, V))).astype(np.float32))
    if dtype == "bf16":
        x = x.to(torch.bfloat16)
    if B > 2 and V > 2:
        x[1, 0, : V - 1] = -float("inf")          # all mass on the last token
    x = rows_at(x, off)
    diag = torch.zeros(8, dtype=torch.int32, device="cuda")
    tok, grp = pcg.propose(dg, x, temperature=1.1, seed=4, offset=2, pos0=1, diag=diag)
    ref = oracle.propose(og, oracle.reverse_index(og), as_oracle_logits(x), temperature=1.1, seed=4, offset=2, pos0=1, nthreads=8)
    assert compare_proposals(tok, grp, ref, og).tolerated <= 1
    assert diag[pcg.Diag.NAMES.index("sequences")] == B * K
    if B > 2 and V > 2:
        assert int(tok[1, 0]) == V - 1


# a draw that lands where a run's only mass is the rounding of sums that cancel: the draft rows hold the
# target's logits in another order inside every group, so each T[g] - D[g] is 0 but for rounding, and the
# gather and finalize, which add a group's entries in different orders, need not agree on its sign
@pytest.mark.parametrize("layout", ["prepared", "csr"])
@pytest.mark.parametrize("n", [20, 40, 100])
def test_a_group_without_mass_is_never_drawn(n, layout):
    V, B, K = 20000, 64, 1
    G = 16 * (V // n)                               # in every run of 16 groups the last holds n tokens, the others none
    sizes = np.where(np.arange(G) % 16 == 15, n, 0)
    rp = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    mem = np.random.default_rng(1).permutation(V).reshape(-1, n)
    mem.sort(axis=1)
    dg = pcg.Groups.from_csr(V, rp, mem.ravel().astype(np.int32), "cuda", prepare=layout == "prepared")
    rng = np.random.default_rng(n)
    tgt = (2.0 * rng.standard_normal((B, K + 1, V))).astype(np.float32)
    dft = np.empty((B, K, V), np.float32)
    dft[:, 0, mem] = tgt[:, 0][:, rng.permuted(mem, axis=1)]
    ptok = torch.zeros((B, K), dtype=torch.int32, device="cuda")
    pgrp = torch.full((B, K), dg.G + 5, dtype=torch.int32, device="cuda")        # no group: rejected
    for step in range(4):
        out = pcg.verify(dg, torch.from_numpy(tgt).cuda(), torch.from_numpy(dft).cuda(), ptok, pgrp, seed=2, offset=step)
        g, t = out.out_groups[:, 0].cpu().numpy(), out.out_tokens[:, 0].cpu().numpy()
        assert (out.accept_len == 0).all()
        assert (sizes[g] > 0).all(), f"{int((sizes[g] == 0).sum())} of {B} draws of a group without members"
        assert all(t[b] in mem[g[b] // 16] for b in range(B))


# rows shorter than a piece, of one piece, around a part of 2048, and on both sides of the lines between a
# workgroup per row and two kernels (8 and 16 parts; 64 and 128 rows)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V,n,off,weighted", [
    (3, 2, 0, False), (4, 1, 1, False), (5, 3, 0, True), (7, 9, 2, False), (2047, 2, 3, False), (2050, 5, 1, True),
    (6145, 4, 0, False), (16384, 3, 0, False), (16385, 64, 0, False), (20011, 64, 7, True), (32768, 65, 0, False),
    (32769, 128, 1, False), (36865, 128, 0, False), (65533, 130, 3, False), (65536, 128, 0, True), (65537, 128, 0, False)])
def test_group_probs_table(V, n, off, weighted, dtype):
    """Every row against the oracle, and, where few rows take the two kernels, against the same rows a few at a
    time: masked logits, a row whose second part has no mass, one with a single finite logit."""
    G = min(V, 700)
    rp, mem = W.random_groups(V, G, 1, min(V, 12), seed=V)
    og = oracle_groups(V, rp, mem)
    w = W.random_weights(og.V, og.members, V) if weighted else None
    if weighted:
        og = oracle.with_weights(og, w)
    dg = pcg.Groups.from_csr(V, rp, mem, "cuda", weights=w)
    rng = np.random.default_rng([V, n])
    x = (4.0 * rng.standard_normal((1, n, V))).astype(np.float32)
    x[0, n // 2][rng.random(V) < 0.2] = -np.inf
    if V > 2048:
        x[0, 0, 2048:4096] = -np.inf
    if n > 2:
        x[0, 1] = -np.inf
        x[0, 1, V // 3] = 2.5
    x = torch.from_numpy(x).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    x = rows_at(x, off)[0]
    print(f"V={V} n={n} off={off} w={weighted} {dtype}", flush=True)
    for temperature in (0.9, 0.07):
        out = pcg.group_probs(dg, x, temperature)
        assert group_probs_error(out, oracle.group_probs(og, as_oracle_logits(x), temperature)) <= 1e-5
    few = torch.cat([pcg.group_probs(dg, x[i:i + 20], 0.9) for i in range(0, n, 20)])
    out = pcg.group_probs(dg, x, 0.9)
    # a term's argument is at most some 50 in size: 50 ln 2 2^-24 on either side
    torch.testing.assert_close(out, few, rtol=4.2e-6, atol=1e-30)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_group_probs_table_beside_values_that_are_not_finite(value, dtype):
    """A row with a NaN or an infinity: the same groups are NaN by rows and by two kernels, the rest equal, and
    other rows do not notice."""
    V, n = 20000, 64
    rp, mem = W.random_groups(V, V, 1, 12, seed=5)
    dg = pcg.Groups.from_csr(V, rp, mem, "cuda")
    x = 4.0 * torch.randn((n, V), device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    x[3, 5000] = value
    x = x.to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    out, few = pcg.group_probs(dg, x, 1.0), pcg.group_probs(dg, x[:20], 1.0)
    assert torch.isnan(few[3]).any() and not torch.isnan(out[4:]).any()
    torch.testing.assert_close(out[:20], few, rtol=4.2e-6, atol=1e-30, equal_nan=True)


# rows and chunks in every split over the XCDs, numbers of them that divide by nothing
@pytest.mark.parametrize("V,G,size,B,K,layout,weighted", [
    (50001, 50001, 40, 1, 1, "csr", False), (41000, 41000, 12, 9, 1, "csr", True), (33000, 33000, 70, 12, 1, "csr", False),
    (20000, 20000, 30, 33, 1, "csr", False), (9000, 9000, 100, 24, 1, "csr", True), (50000, 50000, 40, 2, 1, "csr", False),
    (70000, 70000, 20, 9, 1, "prepared", False), (70000, 66000, 20, 17, 1, "prepared", True)])
def test_rows_and_chunks_over_the_chip(V, G, size, B, K, layout, weighted):
    check_step(V, G, size, B, K, "bf16", layout=layout, weighted=weighted, chunk_groups=4096, thinning=False)


# few rows of a prepared membership: from the CSR, one turn and two of its workgroups, one tile and two, and on the
# other side of those lines
@pytest.mark.parametrize("V,G,size,B,K,layout,weighted", [
    (17000, 17000, 8, 1, 2, "prepared", False), (17001, 17003, 30, 3, 2, "prepared", False),
    (20000, 20000, 30, 12, 2, "prepared", False), (20011, 20011, 90, 6, 1, "prepared", False),
    (20011, 20011, 90, 7, 1, "prepared", False), (33000, 33000, 20, 5, 2, "prepared", True),
    (33001, 33001, 50, 20, 1, "prepared", True), (17000, 17000, 10, 17, 1, "prepared", True),
    (50001, 50001, 40, 1, 1, "prepared", False), (50000, 50000, 40, 2, 1, "prepared", False),
    (41000, 41000, 12, 3, 1, "prepared", False), (45000, 45000, 34, 1, 2, "prepared", True),
    (30000, 4096, 9, 2, 2, "prepared", False), (30000, 33, 40, 2, 2, "prepared", False)])
def test_few_rows(V, G, size, B, K, layout, weighted):
    check_step(V, G, size, B, K, "bf16", layout=layout, weighted=weighted, chunk_groups=4096, thinning=False)


@pytest.mark.parametrize("V,size,n", [(17000, 32, 12), (20000, 32, 16), (45000, 20, 2), (45000, 20, 3), (20000, 60, 5)])
def test_few_rows_of_groups_of_one_size(V, size, n):
    """The same lines where all groups are of one size: every sum by the prepared layout's handle and by the CSR's."""
    rp, mem = W.random_groups(V, V, size, size, seed=V)
    dg = pcg.Groups.from_csr(V, rp, mem, "cuda", chunk_groups=4096)
    og = oracle_groups(V, rp, mem)
    x = 4.0 * torch.randn((n, V), device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    print(f"V={V} size={size} n={n}", flush=True)
    ref = oracle.group_probs(og, as_oracle_logits(x.cpu()), 0.9)
    for g in (dg, dg.without_prepared()):
        assert group_probs_error(pcg.group_probs(g, x, 0.9), ref) <= 1e-5


# one row or two more than a batch of the table holds: from the prepared layout by rows and by two kernels, few rows of
# which would be gathered from the CSR, with the CSR alone, with weights
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V,size,n,layout,weighted", [
    (65536, 32, 258, "prepared", False), (65536, 12, 513, "prepared", True), (20000, 32, 839, "prepared", False),
    (12000, 60, 1399, "prepared", False), (20000, 32, 840, "csr", False), (70001, 20, 240, "prepared", False)])
def test_equal_rows_of_a_call(V, size, n, layout, weighted, dtype):
    """Rows of one call that hold the same logits have the same group probabilities, to the bit, wherever they stand."""
    rp, mem = W.random_groups(V, V, size, size, seed=V)
    w = W.random_weights(V, mem, V) if weighted else None
    dg = pcg.Groups.from_csr(V, rp, mem, "cuda", chunk_groups=4096, weights=w, prepare=layout == "prepared")
    x = 4.0 * torch.randn((n, V), device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    x[n // 2] = x[0]
    x[n - 1] = x[0]
    x = x.to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    print(f"V={V} size={size} n={n} {layout} w={weighted} {dtype}", flush=True)
    out = pcg.group_probs(dg, x, 0.9)
    assert torch.equal(out[n // 2], out[0]) and torch.equal(out[n - 1], out[0])


# the table by a workgroup a row for all rows, by two kernels for some of them
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V,n,some,weighted", [
    (65536, 130, 20, False), (65533, 128, 40, True), (32768, 65, 40, False), (30001, 64, 63, False), (36865, 129, 50, False)])
def test_rows_of_calls_of_different_sizes(V, n, some, weighted, dtype):
    """A row's group probabilities by the prepared layout are the same to the bit whatever number of rows comes with it
    (of so many that none is gathered from the CSR)."""
    rp, mem = W.random_groups(V, V, 1, 12, seed=V)
    w = W.random_weights(V, mem, V) if weighted else None
    dg = pcg.Groups.from_csr(V, rp, mem, "cuda", weights=w)
    x = 4.0 * torch.randn((n, V), device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    x[1, :3000] = -float("inf")
    x = x.to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    print(f"V={V} n={n} some={some} w={weighted} {dtype}", flush=True)
    out = pcg.group_probs(dg, x, 0.9)
    assert torch.equal(pcg.group_probs(dg, x[:some], 0.9), out[:some])
    assert torch.equal(pcg.group_probs(dg, x[n - some:], 0.9), out[n - some:])


# few sequences of a prepared membership of one chunk: by four launches from the CSR, and on the other side of that line
@pytest.mark.parametrize("V,G,size,B,K,weighted", [
    (12000, 12000, 64, 1, 2, False), (16384, 16384, 40, 9, 1, False), (9001, 9001, 110, 3, 2, True), (16384, 16000, 200, 2, 8, True),
    (16384, 16384, 12, 1, 2, False), (12001, 12001, 64, 40, 1, False)])
def test_few_sequences_of_one_chunk(V, G, size, B, K, weighted):
    check_step(V, G, size, B, K, "bf16", layout="prepared", weighted=weighted, thinning=False)


@pytest.mark.parametrize("V,n,by_rows", [(4096, 3, True), (20000, 2, False), (65536, 257, True), (65536, 100, False)])
def test_stage_times_of_group_probs(V, n, by_rows):
    """Statistics and table by one kernel are one stage; by two, two.  Of the first batch."""
    rp, mem = W.random_groups(V, 500, 1, 9, seed=1)
    dg = pcg.Groups.from_csr(V, rp, mem, "cuda")
    x = torch.randn((n, V), device="cuda")
    pcg.group_probs(dg, x)
    pcg.profile_begin(3)
    for _ in range(3):
        pcg.group_probs(dg, x)
    ms, calls = pcg.profile_end()
    assert calls == 3 and (ms["row_stats"] == 0.0) == by_rows
    assert ms["weights"] > ms["event_overhead"] > 0.0 and ms["gather"] > ms["event_overhead"] and ms["finalize"] == 0.0


# from the CSR: more chunks of a row than run at once, the last in a second turn, where those spare a tile
@pytest.mark.parametrize("V,G,size,B,weighted", [(28980, 28980, 7, 101, False), (29706, 29000, 4, 127, True), (48852, 48852, 4, 85, False),
                                                 (27001, 27000, 12, 93, False)])
def test_chunks_that_spare_a_tile(V, G, size, B, weighted):
    check_step(V, G, size, B, 1, "bf16", layout="csr", weighted=weighted, thinning=False)


# from the CSR by one workgroup a sequence: the most trips it takes
@pytest.mark.parametrize("V,G,size,B,K,dtype,weighted", [
    (1024, 1024, 120, 5, 8, "f32", False), (2047, 2040, 60, 33, 4, "bf16", True), (5003, 5003, 25, 20, 8, "bf16", False),
    (6100, 6001, 20, 70, 5, "bf16", False), (4096, 4096, 60, 100, 2, "f32", True), (7168, 7168, 12, 97, 4, "bf16", False),
    (700, 640, 260, 100, 2, "bf16", False)])
def test_small_steps_from_the_csr(V, G, size, B, K, dtype, weighted):
    check_step(V, G, size, B, K, dtype, layout="csr", weighted=weighted, thinning=False)
