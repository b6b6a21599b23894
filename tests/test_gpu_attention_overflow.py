"""The one-pass attention where products of queries and cached keys overflow to
-inf: whole 64-key blocks at the start of a run, whole runs, and single keys among
others weigh nothing, and the rest of the row is unharmed.  Against the fp64 oracle, in
which those scores are finite and hugely negative.

Queries are made positive in one slowly rotating dimension and zero elsewhere (column 0 of
the embedding is 1, the q rows of that dimension read it alone, the q gain passes it
alone); the keys of weight zero hold -2^127 there.

Tolerance: 3e-4, the projections' (test_gpu_wide_gemm); queries of size 100 and keys of 0.1 give
scores of size one, formed to 2^-17."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import GpuRun, check_against_oracle, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("heads", [8, 16])   # 64 and 128 query rows a workgroup
@pytest.mark.parametrize("batch,ctx,dead", [(4, 200, [(0, 64)]), (32, 1000, [(0, 64), (130, 131)]),
                                            (32, 1000, [(0, 400), (700, 764)]), (5, 64, [(0, 64)])])
def test_scores_of_minus_infinity(heads, batch, ctx, dead):
    dim = 63   # pairs with 127; turns by 1.2e-6 a position
    cfg = synth.get_config("tiny").with_(dtype="bf16", head_dim=128, n_q_heads=heads, n_layers=1, batch=batch, ctx=ctx,
                                         ctx_from_hidden=False)
    w = synth.make_weights(cfg, seed=71)
    lw = w["layers"][0]
    w["embed"][:, 0] = 1.0
    lw["wq"][dim::128] = 0.0
    lw["wq"][dim::128, 0] = 1.0
    lw["q_norm"][:] = 0.0
    lw["q_norm"][dim] = 20.0
    inp = synth.make_inputs(cfg, seed=71)
    inp["ctx_k"] = synth.bf16_round(inp["ctx_k"] * 0.1)
    for a, b in dead:
        inp["ctx_k"][:, :, a:b] = 0.0
        inp["ctx_k"][:, :, a:b, :, dim] = -2.0 ** 127
    run = GpuRun(cfg, w, inp["max_ctx"], beta=1)
    gpu = run.step(inp)
    assert gpu["err"] == 0
    run.close()
    rows = np.unique([0, batch - 1])
    ref = oracle.draft_step(cfg, oracle.as_f64_weights(w), inp["anchor"][rows], inp["ctx_lens"][rows],
                            inp["ctx_k"][:, rows], inp["ctx_v"][:, rows], 1, forced=gpu["topk_ids"][rows, :, 0])
    sub = {k: gpu[k][rows] for k in ("topk_ids", "topk_vals", "hidden", "base_logits", "final_logits", "states")}
    log(f"heads {heads} batch {batch} ctx {ctx} dead {dead}")
    check_against_oracle(cfg, sub, ref, 3e-4, 1)
