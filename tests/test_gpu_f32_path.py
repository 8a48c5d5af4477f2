"""The float32 prefill's two GEMM kernels (a workgroup per 16 x 32 tile with K split
over its waves, and 64 x 64 tiles) and its 16-query attention blocks, at row
counts around their tiles: against the float64 oracle (rowwise 1e-4), weights
and the key/value cache at 4-byte alignment, and a prompt alone bit for bit
equal to the same prompt in a batch that runs on the other kernel."""
import dataclasses

import numpy as np
import pytest

import synth
from oracle import rift_oracle as O
from tests.rift_testlib import oracle_layer_weights, rowwise_rel_err, torch_mod, upload

pytestmark = pytest.mark.gpu


def unaligned(a):
    """A device tensor of a's values that starts 4 bytes into an allocation."""
    torch = torch_mod()
    flat = torch.empty(a.size + 1, dtype=torch.float32, device="cuda")
    out = flat[1:].view(a.shape)
    out.copy_(torch.from_numpy(a))
    return out


@pytest.mark.parametrize("d,hd,ffn,lens,checked", [
    (64, 64, 16, [1, 15, 16, 17, 33], 5), (128, 128, 80, [31, 2, 48], 3), (256, 64, 688, [88, 88], 2),
    (320, 64, 48, [63, 65], 2), (1024, 128, 2064, [40] + [300] * 4, 1)])
def test_f32_tiles_against_oracle(d, hd, ffn, lens, checked):
    import paper_2609_29029_amd as R
    torch = torch_mod()
    m = synth.ModelShape(d=d, n_heads=d // hd, head_dim=hd, ffn=ffn, n_layers=1)
    W = synth.make_layer(dataclasses.replace(synth.get("tiny"), model=m, cid=90 + hd), 0)
    Wd = {k: (unaligned(v) if v.ndim == 2 else upload(v, "f32")) for k, v in W.items()}
    cfg = R.model_cfg(d, d // hd, hd, ffn, 1, m.rms_eps, m.rope_base, R.RIFT_F32)
    rng = np.random.default_rng(d + len(lens))
    x = rng.standard_normal((sum(lens), d)).astype(np.float32)

    def run(ls, xs, n_prefix=0):
        cu = np.concatenate([[0], np.cumsum(ls)]).astype(np.int32)
        pos = np.concatenate([np.arange(n) + (n_prefix if i else 0) for i, n in enumerate(ls)]).astype(np.int32)
        T, L = int(cu[-1]), max(ls) + n_prefix
        ws = torch.empty(R.rift_prefill_workspace_size(cfg, T, L), dtype=torch.uint8, device="cuda")
        hid = torch.empty(T, d, dtype=torch.float32, device="cuda")
        kv = unaligned(np.zeros((1, 2, T, d), np.float32))
        R.rift_prefill(cfg, [Wd], upload(xs, "f32"), torch.from_numpy(cu).cuda(), torch.from_numpy(pos).cuda(), len(ls),
                       L, hid, ws, kv_cache=kv, n_prefix=n_prefix)
        torch.cuda.synchronize()
        return hid.cpu().numpy(), kv.cpu().numpy(), cu, pos

    hid, kv, cu, pos = run(lens, x)
    ys = O.prefill(x.astype(np.float64), cu, pos, [oracle_layer_weights(W, "f32")], m.n_heads, hd, m.rms_eps, m.rope_base,
                   list(range(checked)))
    for i in range(checked):
        assert rowwise_rel_err(hid[cu[i]:cu[i + 1]].astype(np.float64), ys[i]) <= 1e-4, i
    alone = run(lens[:1], x[:lens[0]])
    assert np.array_equal(alone[0], hid[:lens[0]]) and np.array_equal(alone[1], kv[:, :, :lens[0]])
    # a prompt after a shared prefix of 7 rows against the two packed together
    whole = run([7 + lens[1]], np.concatenate([x[:7], x[cu[1]:cu[2]]]))
    split = run([7, lens[1]], np.concatenate([x[:7], x[cu[1]:cu[2]]]), n_prefix=7)
    assert np.array_equal(whole[0], split[0]) and np.array_equal(whole[1], split[1])


def prefill_f32(lens, xs, W, cfg, n_prefix=0, positions=None, max_seqlen=None):
    import paper_2609_29029_amd as R
    torch = torch_mod()
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    pos = np.concatenate([np.arange(n) + (n_prefix if i else 0) for i, n in enumerate(lens)])
    pos = (pos if positions is None else positions).astype(np.int32)
    T, L = int(cu[-1]), max_seqlen or max(lens) + n_prefix
    ws = torch.empty(R.rift_prefill_workspace_size(cfg, T, L), dtype=torch.uint8, device="cuda")
    ws.fill_(255)
    hid = torch.empty(T, xs.shape[1], dtype=torch.float32, device="cuda")
    R.rift_prefill(cfg, [W], upload(xs, "f32"), torch.from_numpy(cu).cuda(), torch.from_numpy(pos).cuda(), len(lens), L,
                   hid, ws, n_prefix=n_prefix)
    torch.cuda.synchronize()
    return hid.cpu().numpy(), cu


def small_model(d, hd, ffn):
    import paper_2609_29029_amd as R
    m = synth.ModelShape(d=d, n_heads=d // hd, head_dim=hd, ffn=ffn, n_layers=1)
    W = synth.make_layer(dataclasses.replace(synth.get("tiny"), model=m, cid=90 + hd), 0)
    cfg = R.model_cfg(d, d // hd, hd, ffn, 1, m.rms_eps, m.rope_base, R.RIFT_F32)
    return {k: upload(v, "f32") for k, v in W.items()}, cfg


@pytest.mark.parametrize("hd,pre", [(64, 0), (128, 0), (64, 5), (128, 19)])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_f32_rows_before_a_non_finite_one_do_not_see_it(hd, pre, value):
    """Causal attention: a token that is not finite makes itself and the rows
    after it in its sequence not finite, and no other row, wherever in a key
    block it stands."""
    W, cfg = small_model(256, hd, 48)
    rng = np.random.default_rng(hd + pre)
    x = rng.standard_normal((pre + 3 * 37, 256)).astype(np.float32)
    lens = ([pre] if pre else []) + [37, 37, 37]
    good, cu = prefill_f32(lens, x, W, cfg, pre)
    first = 1 if pre else 0
    for j in (0, 1, 14, 15, 16, 17, 33, 36):
        bad = x.copy()
        row = cu[first + 1] + j                    # of the middle prompt
        bad[row, 3] = value
        got, _ = prefill_f32(lens, bad, W, cfg, pre)
        after = np.zeros(len(x), bool)
        after[row:cu[first + 2]] = True
        assert np.array_equal(got[~after], good[~after]), j
        assert np.isnan(got[after]).all(axis=1).all(), j


@pytest.mark.parametrize("hd", [64, 128])
def test_f32_attends_in_sequences_longer_than_declared(hd):
    """max_seqlen bounds the positions (the RoPE table); rows of a sequence past
    it are attended all the same, as in the bfloat16 path."""
    W, cfg = small_model(256, hd, 48)
    rng = np.random.default_rng(hd)
    lens = [20, 75, 33]
    x = rng.standard_normal((sum(lens), 256)).astype(np.float32)
    positions = np.concatenate([np.arange(n) for n in lens]) % 17
    whole, _ = prefill_f32(lens, x, W, cfg, positions=positions)
    short, _ = prefill_f32(lens, x, W, cfg, positions=positions, max_seqlen=17)
    assert np.array_equal(whole, short)


@pytest.mark.parametrize("d,hd,ffn,lens", [
    # more than 4,096 tiles in each product: 64-row tiles, the last one partial (2,117 and
    # 1,497 rows); 65 column tiles of gate/up, so the last pair is a single one
    (1024, 64, 1040, [40] + [300] * 6 + [277]),
    (1536, 128, 1552, [300] * 4 + [297]),
])
def test_f32_rows_of_the_tile_kernel_are_those_of_the_split_kernel(d, hd, ffn, lens):
    W, cfg = small_model(d, hd, ffn)
    x = np.random.default_rng(d).standard_normal((sum(lens), d)).astype(np.float32)
    hid, cu = prefill_f32(lens, x, W, cfg)
    for i in range(len(lens)):
        alone, _ = prefill_f32(lens[i:i + 1], x[cu[i]:cu[i + 1]], W, cfg)
        assert np.isfinite(alone).all() and np.array_equal(hid[cu[i]:cu[i + 1]], alone), i
