"""Greedy and sampled acceptance where their wide loads, row lists and shortened
exponentials can go wrong: vocabularies smaller than a load, not whole loads, one
past a chunk; rows of equal maxima, of zeros of both signs, of NaN, of -inf and of
the type's lowest value; target logits that are not 16-byte aligned.  Greedy
results are compared bit by bit; sampled ones wherever the oracle's margins are
clear (test_gpu_sampling states them)."""
import numpy as np
import pytest

import oracle
import synth
from oracle import sampling_oracle as so
from test_gpu_parity import _accept_gpu, torch
from test_gpu_sampling import _compare_verify, _t, _verify_gpu
from gpu_helpers import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,dtype,bs,beta", [(9, "f32", 1, 1), (12, "bf16", 3, 2),
                                                     (4097, "bf16", 40, 8), (8200, "bf16", 33, 3),
                                                     (8200, "f32", 5, 4), (4100, "bf16", 2, 1),
                                                     # one value a thread, a chunk of one; 16 waves of single values
                                                     (251, "bf16", 160, 1), (257, "f32", 2, 4), (50257, "bf16", 3, 2)])
def test_greedy_acceptance_edges(V, dtype, bs, beta):
    rng = np.random.default_rng(V + bs)
    cfg = synth.get_config("tiny").with_(batch=bs, branch=beta, vocab=V)
    tree = oracle.build_tree(synth.make_random_topk(cfg, seed=V), np.zeros(bs, np.int32), np.full(bs, 9, np.int32))
    tok, par = tree["node_token"], tree["node_parent"]
    lg = rng.integers(-2, 3, size=(bs, tok.shape[1], V)).astype(np.float32)   # many equal maxima: the smallest id wins
    for b in range(bs):
        cur = 0
        for d in range(cfg.depth):   # a path to accept, mostly to its end
            kids = np.flatnonzero(par[b] == cur)
            if len(kids) == 0 or (b % 4 == 3 and d == b % 15):
                break
            cur = int(rng.choice(kids))
            lg[b, par[b, cur], tok[b, cur]] = 5.0
        lg[b, cur] = [np.nan, -np.inf, -0.0, np.finfo(np.float32).min if dtype == "f32" else -3.3895314e38][b % 4]
        if b % 4 == 2:
            lg[b, cur, V // 2:] = 0.0   # +0 and -0 are equal
        if b % 4 == 0 and V > 8:
            lg[b, cur, V - 1] = -3.0    # the only value of a row of NaN is its last
    t = torch.from_numpy(lg).to("cuda:0").to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    got = _accept_gpu(tok, par, t, cfg.block)
    want = oracle.verify_accept(tok, par, lg, cfg.block)
    log(f"V={V} {dtype} beta={beta}: accept lengths {want['accept_len'].tolist()}")
    for k in want:
        np.testing.assert_array_equal(got[k], want[k], err_msg=k)


@pytest.mark.parametrize("V,dtype,offset,mask", [(50001, "f32", 0, "lowest"), (8200, "f32", 1, "inf"),
                                                 (8196, "bf16", 0, "lowest"), (16384, "bf16", 0, "lowest"),
                                                 (16384, "bf16", 3, "inf"), (16384, "f32", 0, "lowest")])
def test_sampled_acceptance_edges(V, dtype, offset, mask):
    bs, B, T = 6, 16, 1.0
    rng = np.random.default_rng(V + offset)
    keep = V // 3   # the rest of both distributions is masked, whole chunks of it
    draft = (rng.normal(size=(bs, B - 1, V)) * 2.0).astype(np.float32)
    target = np.concatenate([draft, rng.normal(size=(bs, 1, V)).astype(np.float32) * 2.0], axis=1)
    target = (target + rng.normal(size=target.shape) * 0.3).astype(np.float32)
    if dtype == "bf16":
        target = synth.bf16_round(target)
    low = -np.inf if mask == "inf" else np.finfo(np.float32).min
    draft[..., keep:] = low
    target[..., keep:] = low if mask == "inf" or dtype == "f32" else -3.3895314e38
    seed = 99 + V
    tok = np.zeros((bs, B), np.int32)
    for b in range(bs):
        for j in range(1, B):
            tok[b, j], _ = so.sample_draft(draft[b, j - 1], T, seed, b, j)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    flat = torch.zeros(target.size + offset, dtype=dt, device="cuda:0")
    flat[offset:] = torch.from_numpy(target).to("cuda:0").to(dt).reshape(-1)
    got = _verify_gpu(tok, flat[offset:].view(bs, B, V), draft, T, seed)
    ref = so.verify_sample(tok, target.astype(np.float64), draft, T, seed)
    n = _compare_verify(got, ref)
    log(f"V={V} {dtype} offset {offset} {mask}: rows compared {n}/{bs}; accept lengths {ref['accept_len'].tolist()}")
    assert n >= bs // 2
    assert np.all(got["out_tokens"] < keep)


@pytest.mark.parametrize("V", [2**31 - 8192, 2**31 - 8191])
def test_greedy_acceptance_of_the_largest_vocabularies(V):
    """Ids near 2^31, in 16-byte and in single loads: the leaf's scan steps past the last one."""
    if torch.cuda.mem_get_info()[0] < 40 << 30:
        pytest.skip("needs 40 GB of device memory")
    lg = torch.full((1, 2, V), -1.0, device="cuda:0", dtype=torch.bfloat16)
    lg[0, 0, V - 5] = lg[0, 1, V - 3] = lg[0, 1, V - 2] = 2.0
    tok, par = np.array([[7, V - 5]], np.int32), np.array([[-1, 0]], np.int32)
    got = _accept_gpu(tok, par, lg, 2)
    assert got["accept_len"].tolist() == [1] and got["accepted_nodes"].tolist() == [[1]]
    assert got["out_tokens"].tolist() == [[V - 5, V - 3]]
    del lg
    torch.cuda.empty_cache()
