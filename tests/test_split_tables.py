"""Split key ranges (fc_view_export_split: copies of the uploaded tables),
checked on the CPU against the map-order fused items:

* every (query tile, key tile) of the fused items is taken exactly once by the
  dQ items and exactly once by the forward's chunks, in key order of the slots;
* chunks start at multiples of the chunk length from the source's first key
  and hold keys of one source; each slot is owned once; each combine entry
  names exactly its tile's slots;
* the workspace sizes are those of the slots, and a view whose backward
  workspace without dQ slots fits the static scratch still fits it with them.
"""
import numpy as np
import pytest

from oracle import planner as P
from paper_2606_08476_amd import flashcp as F
from paper_2606_08476_amd import synth

BN = 64


def _tiles(it):
    """(source, first key, end key) of an item's key tiles, received first."""
    q0, q1, r0, r1, l0, l1 = (int(x) for x in it[:6])
    return ([(1, a, min(a + BN, r1)) for a in range(r0, r1, BN)] +
            [(0, a, min(a + BN, l1)) for a in range(l0, l1, BN)])


def _slots_most(i):
    """The most bytes one direction's slots may take: 256 MiB, or four times the
    rank's fp32 output if that is more."""
    return max(256 << 20, 4 * 4 * i["t_q"] * i["hq"] * i["d"])


def check_split(v):
    """Checks v's tables; returns (forward split, dQ split)."""
    i, e, s = v.info, v.export(), v.export_split()
    fused = {(int(it[0]), int(it[1])): it for it in e["fwd_fused"]}
    assert len(fused) == len(e["fwd_fused"])
    hc = i["hq"] // i["hkv"] // (128 // i["bm_fwd"])
    slot_bytes = i["hkv"] * hc * 128 * i["d"] * 4
    f_two, bwd, dkdv = v.workspace_size(F.FC_TWO_PASS)
    f_fused = v.workspace_size(F.FC_FUSED)[0]

    # forward chunks
    u, comb, c = s["fwd_units"], s["fwd_comb"], s["fwd_chunk"]
    if c:
        by_slot = {int(x[7]): x for x in u}
        assert sorted(by_slot) == list(range(len(u)))
        assert f_two == f_fused == -(-len(u) * (slot_bytes + slot_bytes // i["d"]) // 256) * 256
        assert i["meta_bytes"] > f_two   # the tables, then the same slots
        assert i["table_bytes"] == i["meta_bytes"] - f_two
        assert f_two <= _slots_most(i) + 256
        seen = set()
        slots = []
        for q0, q1, first, n_r, n_l, *_ in comb.tolist():
            it = fused[(q0, q1)]
            got = []
            for k in range(n_r + n_l):
                x = by_slot[first + k]
                slots.append(first + k)
                t = _tiles(x)
                src, lo = (1, int(it[2])) if k < n_r else (0, int(it[4]))
                assert x[:2].tolist() == [q0, q1] and {a[0] for a in t} == {src}
                assert len(t) <= c and (t[0][1] - lo) % (c * BN) == 0
                assert src or x[6] == it[6]
                got += t
            assert got == _tiles(it)
            seen.add((q0, q1))
        assert seen == set(fused) and sorted(slots) == list(range(len(u)))
        cost = [len(_tiles(x)) for x in u]
        assert cost == sorted(cost, reverse=True)
    else:
        assert len(u) == len(comb) == 0
        assert f_fused == 0 and i["table_bytes"] == i["meta_bytes"]

    # dQ parts
    d, comb = s["dq_items"], s["dq_comb"]
    n_slots = int(sum(comb[:, 3]))
    assert n_slots * slot_bytes <= _slots_most(i)
    part = 2 * i["n_bwd_slots"] * i["hkv"] * 128 * i["d"] * 4
    delta = -(-i["t_q"] * i["hq"] * 4 // 256) * 256
    assert dkdv == part + n_slots * slot_bytes and bwd == delta + dkdv
    if delta + part <= F.NOALLOC_SCRATCH_BYTES:
        assert bwd <= F.NOALLOC_SCRATCH_BYTES
    if len(d):
        by_slot = {int(x[7]): x for x in d if x[7] >= 0}
        assert sorted(by_slot) == list(range(n_slots))
        done = {(int(x[0]), int(x[1])): _tiles(x) for x in d if x[7] < 0}
        for q0, q1, first, n, *_ in comb.tolist():
            assert n > 1 and (q0, q1) not in done
            parts = [by_slot.pop(first + k) for k in range(n)]
            assert all(x[:2].tolist() == [q0, q1] for x in parts)
            done[(q0, q1)] = [t for x in parts for t in _tiles(x)]
        assert not by_slot and done == {k: _tiles(it) for k, it in fused.items()}
        assert all(x[6] == fused[(int(x[0]), int(x[1]))][6] for x in d)
        cost = [len(_tiles(x)) for x in d]
        assert cost == sorted(cost, reverse=True)
    return bool(c), len(d) > 0


HEADS = [(4, 1, 128), (8, 1, 128), (16, 2, 64), (4, 4, 64), (16, 16, 128), (32, 8, 128)]


def test_split_tables_random():
    rng = np.random.default_rng(17)
    n = np.zeros(2, dtype=int)
    for _ in range(60):
        lens = np.exp(rng.uniform(0, np.log(30000), size=int(rng.integers(1, 9)))).astype(int) + 1
        cp = int(rng.integers(1, 9))
        lens[-1] += (-lens.sum()) % cp
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        plan = [P.plan_per_doc, P.plan_per_seq, lambda a, b: P.plan_hybrid(a, b)[0],
                P.plan_whole_lpt][int(rng.integers(4))](cu, cp)
        for rank in range(cp):
            hq, hkv, d = HEADS[int(rng.integers(len(HEADS)))]
            v = F.View(cu, plan, cp, rank, hq, hkv, d)
            n += check_split(v)
            v.close()
    assert (n > 20).all(), n   # the rule does split, in both directions


def test_slots_of_long_contexts_are_bounded():
    """Long contexts over many ranks, whose best split by time would take more
    than the bound (the first: 287 MiB for 30 MiB of output), or nearly."""
    for lens, cp, (hq, hkv, d) in (([500000] + [10000] * 50, 32, (4, 4, 64)),
                                   ([900000, 148576], 64, (4, 4, 64)),
                                   ([300000, 212144], 64, (4, 1, 128))):
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        v = F.View(cu, F.fc_plan_per_doc(cu, cp), cp, cp - 1, hq, hkv, d)
        check_split(v)
        v.close()


@pytest.mark.parametrize("name", list(synth.WORKLOADS))
def test_workloads_with_enough_workgroups_are_not_split(name):
    """The five workloads fill the chip (or are too short to gain): their
    workspaces and launch lists are the unsplit ones."""
    w = synth.WORKLOADS[name]
    cu = synth.cu_seqlens(synth.doc_lengths(name))
    plan = {"per_doc": P.plan_per_doc, "whole_lpt": P.plan_whole_lpt}.get(
        w.plan, lambda c, n: P.plan_hybrid(c, n)[0])(cu, w.cp)
    work = P.stats(cu, w.cp, plan, 1, 1)["work"]
    rank = {"last": w.cp - 1, "heaviest": int(np.argmax(work))}.get(w.rank)
    v = F.View(cu, plan, w.cp, int(w.rank) if rank is None else rank, w.hq, w.hkv, w.d)
    assert check_split(v) == (False, False)
    v.close()
