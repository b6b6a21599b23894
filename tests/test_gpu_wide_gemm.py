"""The wide-activation GEMM at the sizes where its tiling can go wrong, through
the drafting step and against the fp64 oracle: an odd number of k-steps (the
last iteration has one), K ranges of one iteration, row counts just past and at
the edges of 64, 128, 192 and 256 rows, a vocabulary that ends inside a tile and
a column group that ends inside a workgroup's tiles.

Tolerance: a bf16 hi + lo pair holds an activation to 2^-17 relative, so a dot
product over K = 288 unit-size activations and weights of standard deviation
0.02 errs by at most 2^-17 * 288 * 0.016 = 3.5e-5; two layers of four such
projections and the head amplify that to at most about 3e-4."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import GpuRun, check_against_oracle, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("batch,rows", [(3, [0, 2]), (4, [3]), (5, [0, 4]), (8, [0, 7]), (9, [8]), (12, [11]),
                                        (13, [0, 12]), (16, [15]), (17, [0, 16]), (33, [0, 31, 32])])
def test_wide_projection_edges(batch, rows):
    cfg = synth.get_config("tiny").with_(dtype="bf16", hidden=288, ffn=1056, vocab=4100, batch=batch, ctx=48,
                                         ctx_from_hidden=False)
    lens = np.array([(7 * b) % 49 for b in range(batch)], np.int32)
    w = synth.make_weights(cfg, seed=21, gain_std=0.1)
    inp = synth.make_inputs(cfg, seed=21, ctx_lens=lens)
    run = GpuRun(cfg, w, inp["max_ctx"], beta=1)
    gpu = run.step(inp)
    assert gpu["err"] == 0
    run.close()
    rows = np.array(rows)
    ref = oracle.draft_step(cfg, oracle.as_f64_weights(w), inp["anchor"][rows], lens[rows], inp["ctx_k"][:, rows],
                            inp["ctx_v"][:, rows], 1, forced=gpu["topk_ids"][rows, :, 0])
    sub = {k: gpu[k][rows] for k in ("topk_ids", "topk_vals", "hidden", "base_logits", "final_logits", "states")}
    log(f"batch {batch}")
    check_against_oracle(cfg, sub, ref, 3e-4, 1)
