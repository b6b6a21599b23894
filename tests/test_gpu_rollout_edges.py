"""The rollout's selection where its row tiles and the bounded top-beta can go
wrong: batches around 16 and 32 rows, vocabularies that end inside a load, a tile
and a 4096-value list, exact ties and NaN logits.  The selected ids and values are
compared bit by bit with the selection from the logits that the step reports, and
those with the fp64 oracle.

Tolerance: 3e-4, as for the projections of this shape (test_gpu_wide_gemm states
why; the rollout adds a rank-256 product of the same kind)."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import GpuRun, check_against_oracle, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("batch,beta,V,dtype", [(1, 8, 130, "bf16"), (2, 2, 4099, "bf16"), (3, 1, 4113, "bf16"),
                                                (16, 3, 8196, "bf16"), (17, 8, 4097, "bf16"), (33, 2, 4099, "bf16"),
                                                (17, 4, 4099, "f32"), (1, 1, 33, "f32")])
def test_rollout_selection_edges(batch, beta, V, dtype):
    cfg = synth.get_config("tiny").with_(dtype=dtype, vocab=V, batch=batch, branch=beta, ctx=16, ctx_from_hidden=False)
    w = synth.make_weights(cfg, seed=41, gain_std=0.1)
    # every third id is a copy of the one before it (exact ties), five ids and the tail past 4096 are NaN
    nan_ids = np.r_[np.arange(5) * (V // 5), np.arange(4096, V)]
    for name in ("lm_head", "w2"):
        w[name][2::3][: len(w[name][1::3])] = w[name][1::3][: len(w[name][2::3])]
    w["lm_head"][nan_ids] = np.nan
    inp = synth.make_inputs(cfg, seed=41)
    run = GpuRun(cfg, w, inp["max_ctx"], beta=beta)
    gpu = run.step(inp)
    assert gpu["err"] == 0
    run.close()
    fin = gpu["final_logits"]
    nan = np.zeros(V, bool)
    nan[nan_ids] = True
    assert np.array_equal(np.isnan(fin), np.broadcast_to(nan, fin.shape))
    for b in range(batch):
        for j in range(cfg.depth):
            ids, vals = oracle.top_beta(fin[b, j], beta)
            np.testing.assert_array_equal(gpu["topk_ids"][b, j], ids, err_msg=f"row {b} depth {j + 1}")
            np.testing.assert_array_equal(gpu["topk_vals"][b, j], vals.astype(np.float32))
    rows = np.unique([0, batch // 2, batch - 1])
    w["lm_head"][nan_ids] = 0.0
    ref = oracle.draft_step(cfg, oracle.as_f64_weights(w), inp["anchor"][rows], inp["ctx_lens"][rows],
                            inp["ctx_k"][:, rows], inp["ctx_v"][:, rows], beta, forced=gpu["topk_ids"][rows, :, 0])
    sub = {k: gpu[k][rows] for k in ("topk_ids", "topk_vals", "hidden", "base_logits", "final_logits", "states")}
    for d in (sub, ref):
        for k in ("base_logits", "final_logits"):
            d[k] = d[k].copy()
            d[k][..., nan] = -1e9
    log(f"batch {batch} beta {beta} V {V} {dtype}")
    check_against_oracle(cfg, sub, ref, 3e-4, beta)


@pytest.mark.parametrize("batch,V,dtype", [(1, 4099, "bf16"), (3, 4097, "bf16"), (17, 10242, "bf16"), (2, 4099, "f32")])
def test_training_cross_entropy_edges(batch, V, dtype):
    """Labels at the edges of waves' and workgroups' vocabulary slices, row counts that are not whole tiles."""
    from oracle import train_oracle as to
    from test_gpu_train import GAMMA, _check, _train
    cfg = synth.get_config("tiny").with_(dtype=dtype, vocab=V, batch=batch, ctx=16, ctx_from_hidden=False)
    w = synth.make_weights(cfg, seed=43, gain_std=0.1)
    inp = synth.make_inputs(cfg, seed=43)
    edges = np.array([0, V - 1, 15, 16, 79, 80, 255, 256, 639, 640, 1279, 1280, 4095, 4096, 31, 32], np.int32)
    labels = np.resize(edges, (batch, cfg.depth)).astype(np.int32)
    run = GpuRun(cfg, w, inp["max_ctx"], beta=1)
    gpu = _train(run, inp, labels, 0.4)
    run.close()
    assert gpu["err"] == 0
    ref = to.train_forward(cfg, oracle.as_f64_weights(w), inp["anchor"], inp["ctx_lens"], inp["ctx_k"], inp["ctx_v"],
                           labels, 0.4, GAMMA)
    _check(gpu, ref, 3e-4)


@pytest.mark.parametrize("batch", [5, 7, 8])
def test_persistent_rollout_of_more_rows(batch, monkeypatch):
    """Up to eight rows share one persistent launch: against the launch-pair rollout and
    the oracle, greedy and sampled (5 and 7 rows leave words of the exchange lines unused)."""
    import test_gpu_parity as tp
    import test_gpu_sampling as ts
    tp.test_persistent_rollout_matches_launch_pair_rollout(batch, monkeypatch)
    monkeypatch.delenv("DOMINO_ROLLOUT", raising=False)
    cfg = tp.persistent_config(batch)
    w = synth.make_weights(cfg, seed=45, gain_std=0.1)
    inp = synth.make_inputs(cfg, seed=45)
    run = GpuRun(cfg, w, inp["max_ctx"], beta=1)
    gpu = ts._sampled_step(run, inp, 1.0, 45)
    from paper_2605_29707_amd import binding as bd
    assert gpu["err"] == 0 and bd.domino_debug_last_paths(run.model) & bd.PATH_PERSISTENT_ROLLOUT
    run.close()
    n, tot = ts._check_sampled(cfg, gpu, inp, oracle.as_f64_weights(w), 1.0, 45, 2e-2)
    assert n >= tot // 2


@pytest.mark.parametrize("batch,beta", [(1, 4), (2, 2), (3, 8), (7, 3)])
def test_persistent_rollout_of_more_candidates(batch, beta):
    """The persistent rollout leaves its corrected logits to the top-beta selection."""
    import test_gpu_parity as tp
    from paper_2605_29707_amd import binding as bd
    cfg = tp.persistent_config(batch).with_(branch=beta, vocab=8196)   # the last tile is a quarter full
    w = synth.make_weights(cfg, seed=47, gain_std=0.1)
    inp = synth.make_inputs(cfg, seed=47)
    run = GpuRun(cfg, w, inp["max_ctx"], beta=beta)
    bare = run.step(inp, debug=False)
    gpu = run.step(inp)
    assert gpu["err"] == 0 and bd.domino_debug_last_paths(run.model) & bd.PATH_PERSISTENT_ROLLOUT
    run.close()
    for k in ("topk_ids", "topk_vals"):
        np.testing.assert_array_equal(bare[k], gpu[k])
    for b in range(batch):
        for j in range(cfg.depth):
            ids, vals = oracle.top_beta(gpu["final_logits"][b, j], beta)
            np.testing.assert_array_equal(gpu["topk_ids"][b, j], ids, err_msg=f"row {b} depth {j + 1}")
            np.testing.assert_array_equal(gpu["topk_vals"][b, j], vals.astype(np.float32))
    ref = oracle.draft_step(cfg, oracle.as_f64_weights(w), inp["anchor"], inp["ctx_lens"], inp["ctx_k"], inp["ctx_v"],
                            beta, forced=gpu["topk_ids"][:, :, 0])
    check_against_oracle(cfg, gpu, ref, 3e-4, beta)


def test_persistent_rollouts_on_two_streams():
    """Steps of two models on two streams, submitted alternately without waiting: their
    persistent launches are ordered, so each ends as it does alone."""
    import test_gpu_parity as tp
    runs = []
    for i, (batch, beta) in enumerate([(2, 3), (5, 1)]):
        cfg = tp.persistent_config(batch).with_(branch=beta)
        run = GpuRun(cfg, synth.make_weights(cfg, seed=51 + i, gain_std=0.1), cfg.ctx, beta=beta)
        inp = synth.make_inputs(cfg, seed=51 + i)
        alone = run.step(inp, debug=False)
        args = (run.t(inp["anchor"], torch.int32), run.t(inp["ctx_lens"], torch.int32),
                run.t(inp["ctx_k"], torch.bfloat16), run.t(inp["ctx_v"], torch.bfloat16))
        runs.append((run, args, alone, torch.cuda.Stream(), beta))
    torch.cuda.synchronize()
    for _ in range(5):
        for run, args, _, st, beta in runs:
            with torch.cuda.stream(st):
                run.bd.domino_draft_step(run.model, *args, run.max_ctx, run.ids, run.vals, run.ws, branch=beta)
    torch.cuda.synchronize()
    for run, _, alone, _, _ in runs:
        assert run.bd.domino_workspace_error(run.ws) == 0
        np.testing.assert_array_equal(run.ids.cpu().numpy(), alone["topk_ids"])
        np.testing.assert_array_equal(run.vals.cpu().numpy(), alone["topk_vals"])
        run.close()


def test_persistent_rollouts_of_two_threads_on_their_own_default_streams():
    """hipStreamPerThread (handle 2) is a stream of its own in each host thread: the launches
    of two threads are ordered although they pass the same handle."""
    import threading
    import test_gpu_parity as tp
    runs = []
    for i, batch in enumerate([1, 6]):
        cfg = tp.persistent_config(batch)
        run = GpuRun(cfg, synth.make_weights(cfg, seed=53 + i, gain_std=0.1), cfg.ctx, beta=1)
        inp = synth.make_inputs(cfg, seed=53 + i)
        alone = run.step(inp, debug=False)
        args = (run.t(inp["anchor"], torch.int32), run.t(inp["ctx_lens"], torch.int32),
                run.t(inp["ctx_k"], torch.bfloat16), run.t(inp["ctx_v"], torch.bfloat16))
        runs.append((run, args, alone))
    torch.cuda.synchronize()

    def steps(run, args):
        for _ in range(5):
            run.bd.domino_draft_step(run.model, *args, run.max_ctx, run.ids, run.vals, run.ws, stream=2)

    threads = [threading.Thread(target=steps, args=r[:2]) for r in runs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for run, _, alone in runs:
        assert run.bd.domino_workspace_error(run.ws) == 0
        np.testing.assert_array_equal(run.ids.cpu().numpy(), alone["topk_ids"])
        np.testing.assert_array_equal(run.vals.cpu().numpy(), alone["topk_vals"])
        run.close()


def test_captured_steps_replayed_at_once(monkeypatch):
    """Graphs of two models' steps (six rows; three candidates), replayed on two streams without
    waiting, with eager steps between: every replay gives, bit for bit, what an eager
    launch-by-launch step gives."""
    import test_gpu_parity as tp
    runs = []
    for i, (batch, beta) in enumerate([(6, 1), (2, 3)]):
        cfg = tp.persistent_config(batch).with_(branch=beta)
        w, inp = synth.make_weights(cfg, seed=55 + i, gain_std=0.1), synth.make_inputs(cfg, seed=55 + i)
        monkeypatch.setenv("DOMINO_ROLLOUT", "loop")
        run = GpuRun(cfg, w, cfg.ctx, beta=beta)
        alone = run.step(inp, debug=False)
        run.close()
        monkeypatch.delenv("DOMINO_ROLLOUT")
        run = GpuRun(cfg, w, cfg.ctx, beta=beta)
        args = (run.t(inp["anchor"], torch.int32), run.t(inp["ctx_lens"], torch.int32),
                run.t(inp["ctx_k"], torch.bfloat16), run.t(inp["ctx_v"], torch.bfloat16))
        st, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            run.bd.domino_draft_step(run.model, *args, run.max_ctx, run.ids, run.vals, run.ws, branch=beta)
        assert run.bd.domino_debug_last_paths(run.model) == 0
        runs.append((run, args, alone, st, graph, beta))
    torch.cuda.synchronize()
    for turn in range(4):
        for run, _, _, _, _, _ in runs:
            run.ids.zero_()
            run.vals.zero_()
        torch.cuda.synchronize()
        for run, _, _, st, graph, _ in runs * 3:
            with torch.cuda.stream(st):
                graph.replay()
        torch.cuda.synchronize()
        for run, args, alone, _, _, beta in runs:
            assert run.bd.domino_workspace_error(run.ws) == 0
            np.testing.assert_array_equal(run.ids.cpu().numpy(), alone["topk_ids"], err_msg=f"turn {turn}")
            np.testing.assert_array_equal(run.vals.cpu().numpy(), alone["topk_vals"])
            run.bd.domino_draft_step(run.model, *args, run.max_ctx, run.ids, run.vals, run.ws, branch=beta)
            torch.cuda.synchronize()
    for run, *_ in runs:
        run.close()
