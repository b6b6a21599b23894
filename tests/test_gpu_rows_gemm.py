"""The projections of up to 32 rows at the sizes where their tiling can go wrong,
through the drafting step and against the fp64 oracle: one and two row blocks, row
counts inside, at and past them (36 rows take the wide kernel), an odd number
of k-steps, appended context rows (their K/V projection has its own row count) with
and without the fusion layer.

Tolerance: that of the wide projections, 3e-4, for the same reasons: bf16 hi + lo
pairs hold an activation to 2^-17 relative, two layers of four projections of K = 288
unit-size activations and weights of standard deviation 0.02 and the head."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import GpuRun, check_against_oracle, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("batch,block,fuse,lens", [(1, 4, 0, [48]), (1, 16, 0, [0]), (5, 4, 0, [33, 0, 1, 48, 7]),
                                                   (3, 8, 0, [0, 48, 5]), (2, 16, 0, [1, 48]),
                                                   (9, 4, 0, [48, 2, 0, 9, 17, 16, 15, 1, 33]), (1, 16, 1, [19]),
                                                   (2, 8, 3, [16, 37]), (1, 4, 2, [33])])
def test_few_row_projection_edges(batch, block, fuse, lens):
    cfg = synth.get_config("tiny").with_(dtype="bf16", hidden=288, ffn=1056, vocab=4100, batch=batch, block=block,
                                         n_q_heads=64 // block,
                                         ctx=48, ctx_from_hidden=fuse > 0,
                                         **({"ctx_fuse_layers": fuse} if fuse > 1 else {}))
    lens = np.array(lens, np.int32)
    w = synth.make_weights(cfg, seed=31, gain_std=0.1)
    inp = synth.make_inputs(cfg, seed=31, ctx_lens=lens)
    n_new = inp["ctx_hidden"].shape[1] if fuse else 0
    run = GpuRun(cfg, w, inp["max_ctx"], beta=1, n_new=n_new)
    gpu = run.step(inp)
    assert gpu["err"] == 0
    run.close()
    ref = oracle.draft_step(cfg, oracle.as_f64_weights(w), inp["anchor"], lens, inp["ctx_k"], inp["ctx_v"], 1,
                            forced=gpu["topk_ids"][:, :, 0], ctx_hidden=inp.get("ctx_hidden"))
    log(f"batch {batch} block {block} appended {n_new}")
    check_against_oracle(cfg, gpu, ref, 2e-2 if fuse else 3e-4, 1)   # appended K/V are stored as bf16
