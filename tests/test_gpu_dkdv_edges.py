"""GPU tests of the backward's dK/dV pass at head_dim 128, block 128 where its
tiles end: samples ending inside a 16-row half, a 32-row tile and a wave's 64
keys, lists longer than the 64 entries held in registers, packed samples, and
dS tiles for part of the pairs. Against the float64 oracle (Eq. 8's gradients)
within the tolerances of the other backward tests. Then the dQ pass that forms
the row statistics at head_dim 64, with a gradient buffer that shares memory
with an input."""
import pytest
import torch

import oracle
import paper_2609_23169_amd as ut
import workloads as W
from parity import check_grad

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _run(case, copies=1, **kw):
    """Gradients of `copies` samples that are all the case's one sample; the
    64-key pass takes grids of 2,048 workgroups and more, with stored tiles where
    there is room for three a list and more."""
    q, k, v, do = (case[n].to(DEV).repeat(copies, 1, 1, 1) for n in ("q", "k", "v", "do"))
    idx = ut.build_block_index(torch.from_numpy(case["block_mask"]).to(DEV).repeat(copies, 1, 1, 1))
    o, lse = ut.bsattn_fwd(q, k, v, idx, case["block"], case["scale"])
    lists = idx["kv_colptr"].numel() - 1
    if kw.get("ds_pairs") == "half":
        kw["ds_pairs"] = idx["nnz"] // 2
    elif kw.get("ds_pairs", None) is None:
        kw["ds_pairs"] = max(idx["nnz"], 3 * lists)
    return ut.bsattn_bwd(q, k, v, o, do, lse, idx, case["block"], case["scale"], **kw)


def _copies(case):
    _, h, nb, _ = case["block_mask"].shape
    return -(-2048 // (h * nb))


def _check(case, grads, label):
    ref = oracle.bsattn_bwd(case["q"], case["k"], case["v"], case["do"], case["block_mask"],
                            case["block"], case["scale"])
    for got, want, nm in zip(grads, ref, ("dq", "dk", "dv")):
        check_grad(got[:1], want, f"{label} {nm}")
        if nm != "dq" or "half" not in label:   # (dQ's two passes agree to rounding only)
            assert torch.equal(got, got[:1].expand_as(got)), f"{label} {nm}: copies differ"


# (not n = 1: a single key's dQ and dK are exactly 0, and the tolerance is
# relative to the largest gradient)
@pytest.mark.parametrize("n", [2, 15, 17, 32, 33, 63, 65, 127, 128, 129, 143, 161, 192, 209, 383])
def test_short_blocks(n):
    case = W.random_case(1000 + n, n, 2, 128, 128, 0.6)
    copies = _copies(case)
    _check(case, _run(case, copies), f"stored n {n}")
    _check(case, _run(case, copies, ds_pairs=0), f"recompute n {n}")


@pytest.mark.parametrize("pairs", [None, 0, "half", 40000])
def test_list_longer_than_its_registers(pairs):
    """Key block 1 is selected by all 131 query blocks (three loads of its
    list), the others by one or two. With room for few more tiles than pairs the
    long lists are chains, taken apart by the 32-key pass; with room for 40,000
    (or no tiles) the 64-key pass keeps them."""
    nb = 131
    case = W.random_case(77, nb * 128 - 45, 1, 128, 128, 0.0)
    case["block_mask"][:, :, :, 1] = 1
    copies = _copies(case)
    ut.ut_trace_enable(1)
    try:
        grads = _run(case, copies, ds_pairs=pairs)
        names = [t["name"] for t in ut.trace_read()]
    finally:
        ut.ut_trace_enable(0)
    assert any(n.startswith("bwd_dkdv_long") for n in names) == (pairs is None), names
    _check(case, grads, f"pairs {pairs}")


def test_chains_beside_other_lists():
    """Chains in some of the heads, a packed batch whose samples end before the
    block grid does, and lists of every length below a chain's: every list is
    taken once."""
    lens, reps, h, nb = [90 * 128 - 5, 70 * 128 + 33], 8, 2, 90
    case = W.varlen_case(83, lens, h, 128, 128, 0.0, garbage_past_end=False)
    m = case["block_mask"]
    m[0, 0, :, 17] = m[0, 1, :, 88] = m[1, 1, :70, 3] = 1   # chains
    m[1, 0, :12, 40] = 1                                    # not one
    q, k, v, do = (case[n].to(DEV).repeat(reps, 1, 1) for n in ("q", "k", "v", "do"))
    cu = torch.tensor([0] + lens * reps, device=DEV).cumsum(0).to(torch.int32)
    idx = ut.build_block_index(torch.from_numpy(m).to(DEV).repeat(reps, 1, 1, 1))
    lists = idx["kv_colptr"].numel() - 1
    assert lists >= 2048 and 70 * 256 > idx["nnz"] > 12 * 256
    a = (cu, max(lens), idx, 128, case["scale"])
    o, lse = ut.bsattn_fwd_varlen(q, k, v, *a)
    ut.ut_trace_enable(1)
    try:
        got = ut.bsattn_bwd_varlen(q, k, v, o, do, lse, *a, ds_pairs=3 * lists)
        names = [t["name"] for t in ut.trace_read()]
    finally:
        ut.ut_trace_enable(0)
    assert any(n.startswith("bwd_dkdv_long") for n in names), names
    ref = oracle.bsattn_bwd_varlen(case["q"], case["k"], case["v"], case["do"], case["cu_seqlens"], m,
                                   128, case["scale"])
    for x, y, nm in zip(got, ref, ("dq", "dk", "dv")):
        x = x.reshape(reps, sum(lens), *x.shape[1:])
        check_grad(x[0], y, nm)
        assert torch.equal(x, x[:1].expand_as(x)), f"{nm}: copies differ"


def test_part_of_the_tiles_in_the_64_key_pass():
    """Room for half of the pairs, still three a list, with six lists of 131."""
    nb = 131
    case = W.random_case(81, nb * 128 - 77, 1, 128, 128, 0.0)
    case["block_mask"][:, :, :, 1::25] = 1
    _check(case, _run(case, _copies(case), ds_pairs="half"), "half of the tiles")


@pytest.mark.parametrize("room", [2, 3])
def test_either_side_of_the_list_length(room):
    """2,048 workgroups with lists of one entry: with room for two tiles a list
    they take the 32-key pass, whose bits a small grid gives too, with room for
    three the 64-key pass."""
    case = W.random_case(82, 200, 1, 128, 128, 0.0)
    copies = _copies(case)
    got = _run(case, copies, ds_pairs=room * 2 * copies)
    _check(case, got, f"room for {room} tiles a list")
    small = _run(case)
    same = all(torch.equal(x[:1], y) for x, y in zip(got[1:], small[1:]))
    assert same == (room == 2)


@pytest.mark.parametrize("delta", [-1, 0])
def test_either_side_of_the_grid_size(delta):
    """2,047 and 2,048 workgroups: the 32-key and the 64-key pass."""
    case = W.random_case(80, 100, 1, 128, 128, 1.0)
    _check(case, _run(case, 2048 + delta), f"{2048 + delta} workgroups")


def test_packed_samples():
    lens, reps = [1, 130, 0, 257, 95], 48
    case = W.varlen_case(78, lens, 3, 128, 128, 0.5)
    q, k, v, do = (case[n].to(DEV).repeat(reps, 1, 1) for n in ("q", "k", "v", "do"))
    cu = torch.tensor([0] + lens * reps, device=DEV).cumsum(0).to(torch.int32)
    idx = ut.build_block_index(torch.from_numpy(case["block_mask"]).to(DEV).repeat(reps, 1, 1, 1))
    assert len(lens) * reps * 3 * 3 >= 2048   # workgroups
    a = (cu, case["max_seqlen"], idx, 128, case["scale"])
    o, lse = ut.bsattn_fwd_varlen(q, k, v, *a)
    got = ut.bsattn_bwd_varlen(q, k, v, o, do, lse, *a)
    ref = oracle.bsattn_bwd_varlen(case["q"], case["k"], case["v"], case["do"], case["cu_seqlens"],
                                   case["block_mask"], 128, case["scale"])
    for x, y, nm in zip(got, ref, ("dq", "dk", "dv")):
        x = x.reshape(reps, sum(lens), *x.shape[1:])
        check_grad(x[0], y, nm)
        assert torch.equal(x, x[:1].expand_as(x)), f"{nm}: copies differ"


@pytest.mark.parametrize("shared", ["q", "k", "v", "o", "dout", "lse"])
@pytest.mark.parametrize("block", [64, 128])
def test_dq_written_last_over_an_input(block, shared):
    """At head_dim 64 dQ normally goes first; over an input it goes last, after
    every other read of Q, dO, O and LSE. K and V are also read by the dQ pass
    itself, each workgroup its own rows only under a diagonal mask."""
    n, h = 300, 2
    case = W.random_case(79, n, h, 64, block, 0.0 if shared in "kv" else 0.5)
    want = _run(case, ds_pairs=0)
    x = {name: case[name].to(DEV) for name in ("q", "k", "v")}
    x["dout"] = case["do"].to(DEV)
    idx = ut.build_block_index(torch.from_numpy(case["block_mask"]).to(DEV))
    x["o"], x["lse"] = ut.bsattn_fwd(x["q"], x["k"], x["v"], idx, block, case["scale"])
    ws = torch.empty(ut.ut_bsattn_bwd_workspace_size(1, n, h), dtype=torch.uint8, device=DEV)
    if shared == "lse":   # LSE within the dQ buffer
        dq = torch.empty_like(x["q"])
        within = dq.view(torch.float32).reshape(-1)[n * h * 16:][:n * h].view(1, h, n)
        x["lse"] = within.copy_(x["lse"])
    else:
        dq = x[shared]
    dk, dv = torch.empty_like(x["k"]), torch.empty_like(x["v"])
    assert ut.ut_bsattn_bwd(x["q"], x["k"], x["v"], x["o"], x["dout"], x["lse"], dq, dk, dv, block,
                            idx["q_rowptr"], idx["q_cols"], idx["kv_colptr"], idx["kv_rows"],
                            case["scale"], ws) == ut.UT_OK
    for a, b, nm in zip((dq, dk, dv), want, ("dq", "dk", "dv")):
        assert torch.equal(a, b), nm
