"""The prefill GEMMs' tile plans (160- to 256-row tiles, short tiles of 32 to
128 rows, a short-tile tail) against each other: the plan follows the number of
packed rows, and no plan may change a bit of a row's result.  So the first
prompt of a batch has the same hidden states and keys/values whatever is packed
behind it, and the last rows of the batch (a partial tile) those of that prompt
alone.  One batch of each model is also compared with the float64 oracle."""
import dataclasses

import numpy as np
import pytest

import synth
from oracle import rift_oracle as O
from tests.rift_testlib import f64, oracle_layer_weights, rowwise_rel_err, torch_mod, upload, upload_layer

pytestmark = pytest.mark.gpu

FIRST, LAST = 21, 13   # rows of the first and the last prompt

# widths and row counts that reach every plan in one product or another on 256
# CUs (each product of EVERY_PLAN below): one to three prompts of small models run
# as short tiles of 32, 64 and 128 rows; the gate/up product of d = 1,024 with FFN
# 16,512 and 8,192 as 160- to 256-row tiles; FFN 33,024 gives it a tail of 32-row
# tiles, d = 2,048 with 3,000 rows the q, k, v product one of 64 and with 500 rows
# gate/up one of 128
CASES = [
    (256, 128, 256 * 3, (40, 97, 161, 600)),
    (1280, 64, 3456, (129, 914, 1500)),
    (1024, 64, 16512, (150, 200, 256)),
    (1024, 128, 8192, (300, 643)),
    (1024, 128, 33024, (200,)),
    (2048, 128, 5504, (176, 1500, 3000)),
    (2048, 64, 21888, (500,)),
]


@pytest.mark.parametrize("d,hd,ffn,rows", CASES)
def test_rows_do_not_depend_on_the_tile_plan(d, hd, ffn, rows):
    import paper_2609_29029_amd as R
    torch = torch_mod()
    m = synth.ModelShape(d=d, n_heads=d // hd, head_dim=hd, ffn=ffn, n_layers=1)
    W = synth.make_layer(dataclasses.replace(synth.get("one_tile"), model=m, cid=70 + hd), 0)
    Wd = upload_layer(W, "bf16")
    cfg = R.model_cfg(m.d, m.n_heads, m.head_dim, m.ffn, 1, m.rms_eps, m.rope_base, R.RIFT_BF16)
    rng = np.random.default_rng(d + ffn)
    x = synth.store(rng.standard_normal((max(rows), d)).astype(np.float32), "bf16")
    tail = synth.store(rng.standard_normal((LAST, d)).astype(np.float32), "bf16")

    def run(lens, xs):
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        pos = np.concatenate([np.arange(n) for n in lens]).astype(np.int32)
        T, L = int(cu[-1]), max(lens)
        ws = torch.empty(R.rift_prefill_workspace_size(cfg, T, L), dtype=torch.uint8, device="cuda")
        hid = torch.empty(T, d, dtype=torch.float32, device="cuda")
        kv = torch.empty(1, 2, T, d, dtype=torch.bfloat16, device="cuda")
        R.rift_prefill(cfg, [Wd], upload(xs, "bf16"), torch.from_numpy(cu).cuda(), torch.from_numpy(pos).cuda(),
                       len(lens), L, hid, ws, kv_cache=kv)
        torch.cuda.synchronize()
        return hid.cpu().numpy(), kv[0].float().cpu().numpy()

    h_first, kv_first = run([FIRST], x[:FIRST])
    h_last, kv_last = run([LAST], tail)
    for T in rows:
        mid = T - FIRST - LAST
        lens = [FIRST] + [200] * (mid // 200) + ([mid % 200] if mid % 200 else []) + [LAST]
        hid, kv = run(lens, np.concatenate([x[:T - LAST], tail]))
        assert np.array_equal(hid[:FIRST], h_first) and np.array_equal(kv[:, :FIRST], kv_first), T
        assert np.array_equal(hid[-LAST:], h_last) and np.array_equal(kv[:, -LAST:], kv_last), T
        assert np.isfinite(hid).all() and np.isfinite(kv).all(), T
        if T == rows[0]:
            cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
            pos = np.concatenate([np.arange(n) for n in lens]).astype(np.int32)
            ys = O.prefill(f64(np.concatenate([x[:T - LAST], tail]), "bf16"), cu, pos, [oracle_layer_weights(W, "bf16")],
                           m.n_heads, m.head_dim, m.rms_eps, m.rope_base, list(range(len(lens))))
            for i in range(len(lens)):
                # the bf16 prefill's gate, rowwise
                assert rowwise_rel_err(hid[cu[i]:cu[i + 1]].astype(np.float64), ys[i]) <= 2e-2, (T, i)


# (d, head dim, FFN, rows): with CASES, every plan in every product (q, k, v with
# either head dim; the residual products; gate/up) on 256 CUs
EVERY_PLAN = [
    (1024, 128, 1024, (3400, 4060, 4730)),         # q, k, v: tiles of 192, 224 and 256 rows
    (1024, 64, 1024, (330, 3400, 4060, 4730)),     # the same, and short tiles of 64
    (2048, 128, 1024, (2580, 5140)),               # q, k, v: tail of 32; residual: 192 rows
    (2048, 64, 4096, (2070, 2590, 2850)),          # gate/up: tail of 64; q, k, v: of 32 and 64
    (4096, 64, 1024, (1960,)),                     # q, k, v: tail of 128
    (4096, 128, 1024, (1960, 4620)),               # the same; residual: tail of 128
    (3072, 128, 1024, (4070, 4730, 5400, 5660)),   # residual: 224 and 256 rows, tails of 32 and 64
]


@pytest.mark.parametrize("d,hd,ffn,rows", EVERY_PLAN)
def test_every_row_of_every_plan(d, hd, ffn, rows):
    """A batch of copies of one 150-row prompt and a shorter last one: every copy
    has the hidden states, keys and values of the prompt alone, bit for bit."""
    import paper_2609_29029_amd as R
    torch = torch_mod()
    g = torch.Generator(device="cuda")
    g.manual_seed(d + hd)
    mk = lambda *s, std=1.0, mean=0.0: torch.empty(*s, device="cuda", dtype=torch.bfloat16).normal_(mean, std, generator=g)
    shape = dict(wq=(d, d), wk=(d, d), wv=(d, d), wo=(d, d), w_gate=(ffn, d), w_up=(ffn, d), w_down=(d, ffn))
    W = {k: mk(*s, std=0.02) for k, s in shape.items()}
    W["g_attn"], W["g_ffn"] = mk(d, std=0.05, mean=1.0), mk(d, std=0.05, mean=1.0)
    cfg = R.model_cfg(d, d // hd, hd, ffn, 1, 1e-6, 10000.0, R.RIFT_BF16)
    prompt = mk(150, d)

    def run(lens):
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        pos = np.concatenate([np.arange(n) for n in lens]).astype(np.int32)
        T, L = int(cu[-1]), max(lens)
        ws = torch.empty(R.rift_prefill_workspace_size(cfg, T, L), dtype=torch.uint8, device="cuda")
        hid = torch.empty(T, d, dtype=torch.float32, device="cuda")
        kv = torch.empty(1, 2, T, d, dtype=torch.bfloat16, device="cuda")
        R.rift_prefill(cfg, [W], torch.cat([prompt[:n] for n in lens]), torch.from_numpy(cu).cuda(),
                       torch.from_numpy(pos).cuda(), len(lens), L, hid, ws, kv_cache=kv)
        return hid, kv[0]

    hid1, kv1 = run([150])
    assert torch.isfinite(hid1).all() and torch.isfinite(kv1).all()
    for T in rows:
        n, last = T // 150, T % 150
        hid, kv = run([150] * n + ([last] if last else []))
        assert torch.equal(hid[:150 * n].view(n, 150, d), hid1.expand(n, -1, -1)), T
        assert torch.equal(kv[:, :150 * n].view(2, n, 150, d), kv1[:, None].expand(-1, n, -1, -1)), T
        assert torch.equal(hid[150 * n:], hid1[:last]) and torch.equal(kv[:, 150 * n:], kv1[:, :last]), T
