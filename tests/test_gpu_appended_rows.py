"""Appended context rows in numbers that a 32-bit count of their values does not
hold (64 rows x 8192 tokens x 4096 columns = 2^31; about 35 GB): their K/V in the cache
against steps of one batch row.

Tolerance: both sides are fp32-accurate (a dot product of 4096 unit-size values and
weights of standard deviation 0.02 errs by at most 2^-17 * 4096 * 0.8 * 0.016 = 4e-4) and then
rounded to bf16, where they may fall to neighbouring values (2^-7 of the value)."""
import types

import pytest

from gpu_helpers import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

DEV = "cuda:0"


def _model():
    from paper_2605_29707_amd import binding as bd
    cfg = types.SimpleNamespace(hidden=4096, n_layers=1, n_q_heads=32, n_kv_heads=8, head_dim=128, ffn=1024, vocab=4096,
                                block=16, gru_hidden=1024, rank=256, mask_id=4095, rms_eps=1e-6, rope_theta=1e6,
                                dtype="bf16", ctx_fuse_layers=0)
    g = torch.Generator(device=DEV)
    g.manual_seed(7)

    def mat(*s):
        return torch.randn(s, generator=g, device=DEV, dtype=torch.bfloat16) * 0.02

    def ones(n):
        return torch.ones(n, device=DEV, dtype=torch.bfloat16)

    layer = dict(wq=mat(4096, 4096), wk=mat(1024, 4096), wv=mat(1024, 4096), wo=mat(4096, 4096), w_gate=mat(1024, 4096),
                 w_up=mat(1024, 4096), w_down=mat(4096, 1024), attn_norm=ones(4096), ffn_norm=ones(4096),
                 q_norm=ones(128), k_norm=ones(128))
    w = dict(embed=mat(4096, 4096), lm_head=mat(4096, 4096), final_norm=ones(4096), layers=[layer],
             gru_w_ih=mat(3072, 4096), gru_w_hh=mat(3072, 1024), gru_b_ih=mat(3072), gru_b_hh=mat(3072),
             w1=mat(256, 5120), w2=mat(4096, 256))
    return bd, bd.DominoModel(cfg, w)


def _append(bd, model, new):
    b, n = new.shape[:2]
    ck, cv = (torch.zeros((1, b, n, 8, 128), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    anchor, lens = torch.zeros(b, dtype=torch.int32, device=DEV), torch.full((b,), n, dtype=torch.int32, device=DEV)
    ids = torch.empty((b, 15, 1), dtype=torch.int32, device=DEV)
    vals = torch.empty((b, 15, 1), device=DEV)
    ws = torch.empty(model.workspace_bytes(b, n, n, 1), dtype=torch.uint8, device=DEV)
    bd.domino_draft_step(model, anchor, lens, ck, cv, n, ids, vals, ws, ctx_hidden_new=new, n_new=n)
    torch.cuda.synchronize()
    assert bd.domino_workspace_error(ws) == 0
    return ck[0], cv[0]


def test_two_to_the_31_appended_values():
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("needs 60 GB of device memory")
    bd, model = _model()
    new = torch.empty((64, 8192, 4096), device=DEV)
    g = torch.Generator(device=DEV)
    for b in range(64):
        g.manual_seed(100 + b)
        new[b].normal_(generator=g)
    got = _append(bd, model, new)
    for b in (0, 31, 63):
        want = _append(bd, model, new[b:b + 1].contiguous())
        for name, x, y in zip("kv", got, want):
            x, y = x[b].float(), y[0].float()
            assert y.abs().mean() > 0.1
            worst = ((x - y).abs() - 2.0 ** -7 * torch.maximum(x.abs(), y.abs())).max().item()
            log(f"row {b} {name}: equal {(x == y).float().mean().item():.5f}, beyond one rounding {worst:.1e}")
            assert worst < 5e-4
    model.close()
    del new, got
    torch.cuda.empty_cache()
