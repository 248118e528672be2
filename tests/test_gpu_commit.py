"""The accepted-path commit (tv_commit_paths) against the oracle's committed
sequence (Def. def2) on the verifier's own outputs, bit-exact (needs an
MI355X)."""

import numpy as np
import pytest
import torch

import paper_2505_12398_amd as tv
import parity
import workloads as W
from oracle import tv_oracle as O

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    tv.load_library()
    yield


def expected(par, tok, out, max_len):
    B = par.shape[0]
    acc, y, st = (out.accepted_node.cpu().numpy(), out.bonus_token.cpu().numpy(),
                  out.status.cpu().numpy())
    pn = np.full((B, max_len), -1, np.int32)
    pt = np.full((B, max_len + 1), -1, np.int32)
    pl = np.zeros(B, np.int32)
    for b in range(B):
        if st[b] != tv.TV_TREE_OK:
            continue
        nodes, toks = O.committed_sequence(par[b], tok[b], int(acc[b]), int(y[b]))
        if len(nodes) > max_len:
            pl[b] = tv.TV_COMMIT_OVERFLOW
            continue
        pn[b, :len(nodes)] = nodes
        pt[b, :len(toks)] = toks
        pl[b] = len(toks)
    return pn, pt, pl


def check(bt, out, max_len):
    pn, pt, pl = tv.commit_paths(bt["parents"], bt["tokens"], out, max_len)
    want = expected(bt["parents"].cpu().numpy(), bt["tokens"].cpu().numpy(), out, max_len)
    for got, w, name in zip((pn, pt, pl), want, ("path_nodes", "path_tokens", "path_len")):
        np.testing.assert_array_equal(got.cpu().numpy(), w, err_msg=name)
    return pl.cpu().numpy()


@pytest.mark.parametrize("tokenlevel", [False, True])
def test_commit_after_verify(tokenlevel):
    """256 benchmark-shaped trees (V reduced to 16381): the commit of the
    verifier's outputs equals the oracle's, and the verifier itself matches the
    oracle; a max_len below some trees' depth reports overflow."""
    bt = W.make_batch(5, step=4, device=DEV, mode=W.WITHOUT_REPLACEMENT, vocab=16381)
    out = tv.verify_batch(bt["parents"], bt["tokens"], bt["target"], bt["draft"],
                          bt["temperature"], bt["uniforms"], bt["mode"], tokenlevel=tokenlevel)
    rep = parity.check(bt, tokenlevel, trees=list(range(0, 256, 16)),
                       gpu=parity.host_outputs(out), label="commit")
    assert not rep.failures, rep.failures[:3]
    pl = check(bt, out, 8)
    assert (pl == out.accept_len.cpu().numpy() + 1).all()
    pl = check(bt, out, 1)
    assert (pl == tv.TV_COMMIT_OVERFLOW).any()
    check(bt, out, 0)


def test_commit_edge_cases():
    """Error trees give length 0; an accepted node out of range or a link that
    does not point back gives TV_COMMIT_INCONSISTENT; the root accepted gives
    Y alone."""
    par = torch.tensor([[-1, 0, 1, 1], [-1, 0, 1, 1], [-1, 0, 2, 1], [-1, 0, 1, 1]],
                       dtype=torch.int32, device=DEV)
    tok = torch.tensor([[0, 5, 6, 7]] * 4, dtype=torch.int32, device=DEV)
    out = tv.VerifyOutputs(
        accept_len=torch.zeros(4, dtype=torch.int32, device=DEV),
        accepted_node=torch.tensor([3, 9, 2, 0], dtype=torch.int32, device=DEV),
        bonus_token=torch.tensor([11, 12, 13, 14], dtype=torch.int32, device=DEV),
        status=torch.tensor([0, 0, 0, tv.TV_TREE_OK], dtype=torch.int32, device=DEV))
    pn, pt, pl = tv.commit_paths(par, tok, out, 3)
    assert pl.cpu().tolist() == [3, tv.TV_COMMIT_INCONSISTENT, tv.TV_COMMIT_INCONSISTENT, 1]
    assert pn.cpu().tolist()[0] == [1, 3, -1] and pt.cpu().tolist()[0] == [5, 7, 11, -1]
    assert pt.cpu().tolist()[3] == [14, -1, -1, -1]
    out.status[0] = tv.TV_TREE_NONFINITE
    pn, pt, pl = tv.commit_paths(par, tok, out, 3)
    assert pl.cpu().tolist()[0] == 0 and pt.cpu().tolist()[0] == [-1] * 4


def walked(par, tok, acc, y, status, max_len):
    """Every tree's chain at once, one step of all trees a time."""
    B, n1 = par.shape
    rows = np.arange(B)
    ok = status == tv.TV_TREE_OK
    bad = ok & ((acc < 0) | (acc >= n1))
    x = np.where(ok & ~bad, acc, 0)
    depth = np.zeros(B, int)
    steps = []
    while (x > 0).any():
        steps.append(x)
        depth += x > 0
        p = par[rows, x]
        broken = (x > 0) & ((p < 0) | (p >= x))
        bad |= broken
        x = np.where((x > 0) & ~broken, p, 0)
    pn = np.full((B, max_len), -1, np.int32)
    pt = np.full((B, max_len + 1), -1, np.int32)
    good = ok & ~bad & (depth <= max_len)
    for k, node in enumerate(steps):
        r = np.nonzero(good & (node > 0))[0]
        pn[r, depth[r] - 1 - k] = node[r]
        pt[r, depth[r] - 1 - k] = tok[r, node[r]]
    r = np.nonzero(good)[0]
    pt[r, depth[r]] = y[r]
    pl = np.where(good, depth + 1, tv.TV_COMMIT_OVERFLOW)
    pl = np.where(bad, tv.TV_COMMIT_INCONSISTENT, np.where(ok, pl, 0))
    return pn, pt, pl


@pytest.mark.parametrize("batch,n1,max_len", [
    (3, 1, 0), (5, 1024, 1024), (8191, 65, 16), (8192, 1, 0), (8193, 3, 2), (8192, 16, 15),
    (8193, 16, 16), (8193, 17, 15), (8193, 128, 63), (8195, 129, 140), (8193, 300, 299),
    (8193, 1024, 1024), (70001, 65, 5)])
def test_commit_many_trees(batch, n1, max_len):
    """Both sides of the number of trees from which a wavefront takes two, or
    sixteen of at most 16 nodes, and reads the links in windows of 128: chains,
    shallow trees and trees in between, with links that do not point back,
    accepted nodes out of range and trees that failed among them; chains of
    several windows."""
    rng = np.random.default_rng(n1)
    i = np.arange(n1)
    reach = rng.choice([1, 2, 30, 127, 128, 129, 1024], (batch, 1))
    par = rng.integers(np.maximum(0, i - reach), np.maximum(i, 1), (batch, n1)).astype(np.int32)
    par[:, 0] = -1
    par[rng.random((batch, n1)) < 0.1 / n1] = n1
    tok = rng.integers(0, 1 << 20, (batch, n1), dtype=np.int32)
    acc = rng.integers(0, n1, batch, dtype=np.int32)
    acc[::97] = n1
    acc[1::97] = -1
    y = rng.integers(0, 1 << 20, batch, dtype=np.int32)
    status = np.where(rng.random(batch) < 0.05, tv.TV_TREE_NONFINITE, 0).astype(np.int32)
    dev = [torch.as_tensor(t, device=DEV) for t in (par, tok, acc, y, status)]
    out = tv.VerifyOutputs(accept_len=None, accepted_node=dev[2], bonus_token=dev[3],
                           status=dev[4])
    got = tv.commit_paths(dev[0], dev[1], out, max_len)
    for g, w, name in zip(got, walked(par, tok, acc, y, status, max_len),
                          ("path_nodes", "path_tokens", "path_len")):
        np.testing.assert_array_equal(g.cpu().numpy(), w, err_msg=name)
