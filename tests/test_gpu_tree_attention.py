"""The one-pass attention under a tree mask (bf16 cache, head width 128) through
the verify forward, against the fp64 oracle: contexts that are empty, end inside
a 64-key block, on one, and leave the tree's own keys split over two runs (where
a node may see none of a run's keys), caches much larger than the contexts (the
runs follow each row's own length), and both workgroup sizes (64 and 128 query rows).

Tolerance: queries, probabilities and the tree's own keys and values are held as
bf16 hi + lo pairs (2^-17 relative), four layers of width 256 then give logits
of unit size to about 4 * 6 * 2^-17 = 2e-4; 5e-4 leaves a factor of two."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_target import Target, _inputs, _t, bd, torch, tg
from gpu_helpers import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("beta,lens,max_ctx", [(1, [0, 60, 64, 113], 160), (2, [0, 50, 64, 47], 120),
                                               (2, [700, 33, 1, 640, 129], 1500), (1, [1000, 5, 48, 52], 3000)])
def test_tree_masked_one_pass(beta, lens, max_ctx):
    cfg = synth.get_config("tiny_target").with_(dtype="bf16", head_dim=128, n_q_heads=8)
    w = synth.make_target_weights(cfg, seed=61, gain_std=0.1)
    inp = _inputs(cfg, lens, max_ctx, seed=61)
    topk = synth.make_random_topk(cfg.with_(batch=len(lens), block=16, branch=beta), seed=61)
    run = Target(cfg, w)
    tok, par, pos, mask = run.tree(topk, inp["anchor"], inp["ctx_lens"])
    ck, cv = _t(inp["ctx_k"], run.kvdt), _t(inp["ctx_v"], run.kvdt)
    lg, ws = run.verify(tok, pos, mask, inp["ctx_lens"], ck, cv, max_ctx)
    assert bd.domino_workspace_error(ws) == 0
    tree = oracle.build_tree(topk, inp["anchor"], inp["ctx_lens"])
    ref = tg.verify_forward(cfg, w, tree["node_token"], tree["node_pos"], tree["ancestor_mask"], inp["ctx_lens"],
                            inp["ctx_k"], inp["ctx_v"])
    err = float(np.abs(lg.cpu().numpy() - ref["logits"]).max())
    log(f"beta={beta} lens={lens}: max |logits - oracle| = {err:.2e}")
    assert err < 5e-4
    run.model.close()
