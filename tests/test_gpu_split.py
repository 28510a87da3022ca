"""Views whose long key ranges are split over workgroups (few KV heads, one
document much longer than the rest): every entry point against the fp64 oracle
and against the others.

The cases have key ranges that are whole multiples of the chunk length, one key
more, shorter than one chunk and empty, one-token documents, both head dims with
each number of heads per workgroup (1, 2 and 4; ragged ones so that a wave's
rows end inside it); the partial passes run over the view's own
slots and, bound without them or captured into a graph, in one workgroup per
query tile. Tolerances are those of the unsplit paths (test_gpu_parity);
where the same sums are taken in another order in fp32, 2e-5 of the largest
value (a few hundred roundings of 2^-24).
"""
import pytest
import torch

import _cases
from oracle import attention as A
from paper_2606_08476_amd import flashcp as F
from test_gpu_parity import G_TOL, LSE_TOL, O_TOL, Run, _lse_ok, _maxabs, dev, say  # noqa: F401

pytestmark = pytest.mark.gpu

ORDER_TOL = 2e-5

CASES = {
    # local keys only, whole multiples of the chunk length and one key more
    "local_g4": dict(workload="llama8b", lens=[4096, 1, 2049, 512], cp=1, rank=0, hq=4, hkv=1,
                     plan="whole_lpt"),
    # received and local keys
    "long_g8": dict(workload="longdoc", lens=[20001, 1, 70, 600], cp=8, rank=7, hq=8, hkv=1,
                    plan="per_doc"),
    "long_g4": dict(workload="longdoc", lens=[24000, 1, 70, 600], cp=16, rank=14, hq=4, hkv=1,
                    plan="per_doc"),
    # one long document among many of a few tokens
    "skewed_g8": dict(workload="llama8b", lens=[24000] + [40] * 100, cp=8, rank=7, hq=8, hkv=1,
                      plan="per_doc"),
    "aligned_d64_g8": dict(workload="tiny", lens=[16384, 1024, 64], cp=8, rank=7, hq=16, hkv=2,
                           plan="per_doc"),
    "long_d64_g1": dict(workload="tiny", lens=[7001, 1, 1, 300], cp=2, rank=1, hq=4, hkv=4,
                        plan="per_doc"),
    "ragged_d64_g2": dict(workload="tiny", lens=[9001, 1, 77, 300], cp=4, rank=3, hq=4, hkv=2,
                          plan="per_doc"),
    "ragged_g1": dict(workload="llama8b", lens=[6007, 1, 130, 300], cp=4, rank=3, hq=2, hkv=2,
                      plan="per_doc"),
    "ragged_g2": dict(workload="llama8b", lens=[6007, 1, 130, 300], cp=4, rank=3, hq=4, hkv=2,
                      plan="per_doc"),
}


@pytest.mark.parametrize("key", list(CASES))
def test_split_views(key, dev):  # noqa: F811
    kw = dict(CASES[key])
    case = _cases.make_case(key, kw.pop("workload"), **kw)
    r = Run(case, dev)
    i, s = r.v.info, r.v.export_split()
    tq, tr, hq, hkv, d = i["t_q"], i["t_recv"], i["hq"], i["hkv"], i["d"]
    wgs = i["n_fwd_fused"] * hkv * (hq // hkv // (128 // i["bm_fwd"]))
    say(f"[gpu] {key}: t_q {tq} t_recv {tr} workgroups {wgs} chunk {s['fwd_chunk']} "
        f"dQ slots {int(s['dq_comb'][:, 3].sum())}")
    assert s["fwd_chunk"] and (len(s["dq_comb"]) or key == "local_g4")
    # forward and backward against the oracle
    c, o, x = case, case.oview, r.x
    O, L = r.oracle_fwd()
    assert max(_maxabs(r.o, O), _maxabs(r.o32, O)) <= O_TOL and _lse_ok(r.lse, L) <= LSE_TOL
    dq, dk, dv = r.oracle_bwd()
    e = dict(dq=_maxabs(r.dq, dq), dk_loc=_maxabs(r.dk_loc, dk[:tq]), dv_loc=_maxabs(r.dv_loc, dv[:tq]),
             dk_recv=_maxabs(r.dk_recv, dk[tq:]), dv_recv=_maxabs(r.dv_recv, dv[tq:]))
    say(f"[gpu] {key} bwd: " + " ".join(f"{k} {v:.3e}" for k, v in e.items()))
    assert max(e.values()) <= G_TOL, e

    nan = lambda *sh, dt=torch.float32: torch.full(sh, float("nan"), dtype=dt, device=dev)  # noqa: E731
    # the partial passes: each against the oracle, in one launch and in two the
    # same bits, and their merge the two-pass forward's bits
    parts = []
    for src, kg, vg, keys in ((0, r.k_loc, r.v_loc, o.q_gpos), (1, r.k_recv, r.v_recv, o.recv_gpos)):
        op, lp = nan(tq, hq, d), nan(hq, tq)
        F.fc_attn_fwd_partial(r.v, src, r.q, kg, vg, 0.0, op, lp)
        Op, Lp = A.attention_fwd(c.cu, o.q_gpos, x["q"], keys, x["k_recv" if src else "k_loc"],
                                 x["v_recv" if src else "v_loc"])
        assert _maxabs(op, Op) <= O_TOL and _lse_ok(lp, Lp) <= LSE_TOL
        parts.append((op, lp))
    both = [nan(tq, hq, d), nan(hq, tq), nan(tq, hq, d), nan(hq, tq)]
    F.fc_attn_fwd_partials(r.v, r.q, r.k_loc, r.v_loc, r.k_recv, r.v_recv, 0.0, *both)
    torch.cuda.synchronize()
    for a, b in zip((*parts[0], *parts[1]), both):
        assert torch.equal(a, b)
    ob, of, lo = nan(tq, hq, d, dt=torch.bfloat16), nan(tq, hq, d), nan(hq, tq)
    F.fc_lse_merge(*parts[0], *parts[1], ob, of, lo)
    torch.cuda.synchronize()
    assert torch.equal(ob, r.o) and torch.equal(of, r.o32) and torch.equal(lo, r.lse)

    # without slots behind the tables, and replayed from a graph: the same bits
    slots = r.v.workspace_size(F.FC_FUSED)[0]
    again = F.View(case.cu, case.plan, case.cp, case.rank, hq, hkv, d)
    tables = i["meta_bytes"] - slots
    buf = torch.empty(tables + 256, dtype=torch.uint8, device=dev)
    at = buf.data_ptr() + (-buf.data_ptr()) % 256
    assert F.lib().fc_view_bind(again.handle, at, tables - 1, F._stream()) == -5
    assert F.lib().fc_view_bind(again.handle, at, tables, F._stream()) == 0
    seq = [nan(tq, hq, d), nan(hq, tq), nan(tq, hq, d), nan(hq, tq)]
    F.fc_attn_fwd_partials(again, r.q, r.k_loc, r.v_loc, r.k_recv, r.v_recv, 0.0, *seq)
    one = [nan(tq, hq, d), nan(hq, tq), nan(tq, hq, d), nan(hq, tq)]
    F.fc_attn_fwd_partial(again, 0, r.q, r.k_loc, r.v_loc, 0.0, *one[:2])
    F.fc_attn_fwd_partial(again, 1, r.q, r.k_recv, r.v_recv, 0.0, *one[2:])
    graph, cap = torch.cuda.CUDAGraph(), [nan(tq, hq, d), nan(hq, tq), nan(tq, hq, d), nan(hq, tq)]
    with torch.cuda.graph(graph):
        F.fc_attn_fwd_partials(r.v, r.q, r.k_loc, r.v_loc, r.k_recv, r.v_recv, 0.0, *cap)
    for _ in range(3):
        for t in cap:
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for a, b, c1, c2 in zip(both, seq, one, cap):
            assert torch.equal(a, b) and torch.equal(a, c1) and torch.equal(a, c2)
    again.close()

    # the partial passes on two streams at once, twice each: uses of the slots
    # follow one another
    side = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [[nan(tq, hq, d), nan(hq, tq), nan(tq, hq, d), nan(hq, tq)] for _ in range(4)]
    torch.cuda.synchronize()
    for k, o4 in enumerate(outs):
        with torch.cuda.stream(side[k % 2]):
            F.fc_attn_fwd_partials(r.v, r.q, r.k_loc, r.v_loc, r.k_recv, r.v_recv, 0.0, *o4)
    torch.cuda.synchronize()
    for o4 in outs:
        for a, b in zip(both, o4):
            assert torch.equal(a, b)

    # the fused forward, with its workspace and (one pass, unsplit) without
    for ws in (torch.empty(r.v.workspace_size(F.FC_FUSED)[0], dtype=torch.uint8, device=dev), None):
        ob, of, lo = nan(tq, hq, d, dt=torch.bfloat16), nan(tq, hq, d), nan(hq, tq)
        F.fc_attn_fwd(r.v, r.q, r.k_loc, r.v_loc, r.k_recv, r.v_recv, 0.0, F.FC_FUSED, ob, of, lo, ws)
        torch.cuda.synchronize()
        assert max(_maxabs(ob, O), _maxabs(of, O)) <= O_TOL and _lse_ok(lo, L) <= LSE_TOL

    # the backward pass with a workspace for split key tiles alone, and the dQ
    # pass: dK/dV the same bits, dQ the same sums in another order
    delta = torch.empty_like(r.lse)
    F.fc_bwd_preprocess(r.v, None, r.do, delta, o_f32=r.o32)
    part = 2 * i["n_bwd_slots"] * hkv * 128 * d * 4
    out = r.bwd_outputs()
    F.fc_attn_bwd_pass(r.v, r.q, r.k_loc, r.v_loc, r.k_recv, r.v_recv, r.lse, delta, r.do, 0.0, *out,
                       torch.empty(max(part, 1), dtype=torch.uint8, device=dev))
    alone = nan(tq, hq, d)
    F.fc_attn_bwd_dq(r.v, r.q, r.k_loc, r.v_loc, r.k_recv, r.v_recv, r.lse, delta, r.do, 0.0, alone)
    torch.cuda.synchronize()
    for a, b in zip(out[1:], (r.dk_loc, r.dv_loc, r.dk_recv, r.dv_recv)):
        assert torch.equal(a, b)
    assert torch.equal(out[0], alone)
    assert _maxabs(out[0], r.dq.cpu()) <= ORDER_TOL * float(r.dq.abs().max())
    # and the same bits on a second run
    again = Run(case, dev)
    for n in ("o", "o32", "lse", "dq", "dk_loc", "dv_loc"):
        assert torch.equal(getattr(again, n), getattr(r, n)), n
    r.v.close()
    again.v.close()


def _view(key):
    kw = dict(CASES[key])
    case = _cases.make_case(key, kw.pop("workload"), **kw)
    return case, F.View(case.cu, case.plan, case.cp, case.rank, case.hq, case.hkv, case.d)


def test_bind_buffers(dev):  # noqa: F811
    """View.bind takes any buffer with room for the tables, with the slots
    where they fit too, and allocates the tables alone on request; less than
    the tables is refused."""
    _, v = _view("local_g4")
    i = v.info
    tables, slots = i["table_bytes"], i["meta_bytes"] - i["table_bytes"]
    assert slots > 0
    size = lambda n: torch.empty(n, dtype=torch.uint8, device=dev)  # noqa: E731
    big = size(i["meta_bytes"] + 512)
    at = (-big.data_ptr()) % 256
    for n in (tables, i["meta_bytes"] - 1, i["meta_bytes"]):
        assert v.bind(dev, big[at:at + n]).meta.numel() == n
    assert v.bind(dev).meta.numel() >= i["meta_bytes"]
    assert v.bind(dev, slots=False).meta.numel() == tables + 256
    with pytest.raises(ValueError):
        v.bind(dev, big[at:at + tables - 1])
    v.close()


@pytest.mark.parametrize("key", ["long_g8", "aligned_d64_g8", "ragged_g2"])
def test_short_workspaces(key, dev):  # noqa: F811
    """With a workspace that holds no slots every call runs the ranges whole: the
    forward against the oracle and the same bits whatever the size, the backward
    the dQ of fc_attn_bwd_dq and the dK/dV of the split run. NULL holds nothing."""
    kw = dict(CASES[key])
    case = _cases.make_case(key, kw.pop("workload"), **kw)
    r = Run(case, dev)
    i, v = r.v.info, r.v
    tq, hq, d = i["t_q"], i["hq"], i["d"]
    O, L = r.oracle_fwd()
    nan = lambda *sh, dt=torch.float32: torch.full(sh, float("nan"), dtype=dt, device=dev)  # noqa: E731
    ws = lambda n: torch.empty(n, dtype=torch.uint8, device=dev)  # noqa: E731
    kv = (r.k_loc, r.v_loc, r.k_recv, r.v_recv)
    whole = -(-i["n_fwd_fused"] * i["hkv"] * (hq // i["hkv"] // (128 // i["bm_fwd"])) * 128 * d * 4
              // 256) * 256
    for mode, sizes in ((F.FC_FUSED, (0, 1, v.workspace_size(F.FC_FUSED)[0] - 1)),
                        (F.FC_TWO_PASS, (whole, v.workspace_size(F.FC_TWO_PASS)[0] - 1))):
        first = None
        for n in sizes:
            out = nan(tq, hq, d, dt=torch.bfloat16), nan(tq, hq, d), nan(hq, tq)
            F.fc_attn_fwd(v, r.q, *kv, 0.0, mode, *out, ws(n))
            torch.cuda.synchronize()
            assert max(_maxabs(out[0], O), _maxabs(out[1], O)) <= O_TOL
            assert _lse_ok(out[2], L) <= LSE_TOL
            first = first or out
            assert all(torch.equal(a, b) for a, b in zip(out, first))
    delta, alone = torch.empty_like(r.lse), nan(tq, hq, d)
    F.fc_bwd_preprocess(v, None, r.do, delta, o_f32=r.o32)
    F.fc_attn_bwd_dq(v, r.q, *kv, r.lse, delta, r.do, 0.0, alone)
    part = 2 * i["n_bwd_slots"] * i["hkv"] * 128 * d * 4
    base = -(-tq * hq * 4 // 256) * 256 + part
    for n in (base, v.workspace_size()[1] - 1):
        out = r.bwd_outputs()
        F.fc_attn_bwd(v, r.q, *kv, r.o, r.lse, r.do, 0.0, *out, ws(n), o_f32=r.o32)
        torch.cuda.synchronize()
        assert torch.equal(out[0], alone)
        assert all(torch.equal(a, b) for a, b in
                   zip(out[1:], (r.dk_loc, r.dv_loc, r.dk_recv, r.dv_recv)))
    v.close()


def test_sources_on_two_streams(dev):  # noqa: F811
    """The local and the received pass of one view, each on a stream of its own and
    several times over, then the two swapped: the bits of the passes run one
    after the other."""
    kw = dict(CASES["long_g4"])
    case = _cases.make_case("long_g4", kw.pop("workload"), **kw)
    r = Run(case, dev)
    i, v = r.v.info, r.v
    tq, hq, d = i["t_q"], i["hq"], i["d"]
    nan = lambda *sh: torch.full(sh, float("nan"), device=dev)  # noqa: E731
    kv = ((r.k_loc, r.v_loc), (r.k_recv, r.v_recv))
    ref = [(nan(tq, hq, d), nan(hq, tq)) for _ in range(2)]
    for src in (0, 1):
        F.fc_attn_fwd_partial(v, src, r.q, *kv[src], 0.0, *ref[src])
    outs = [[(nan(tq, hq, d), nan(hq, tq)) for _ in range(2)] for _ in range(6)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for k, pair in enumerate(outs):
        for src in (0, 1):
            with torch.cuda.stream(streams[src ^ (k >= 3)]):
                F.fc_attn_fwd_partial(v, src, r.q, *kv[src], 0.0, *pair[src])
    torch.cuda.synchronize()
    for pair in outs:
        for src in (0, 1):
            assert all(torch.equal(a, b) for a, b in zip(pair[src], ref[src]))
    v.close()
