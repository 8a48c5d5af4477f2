"""Decode steps at the edges of the key split (one part, several, the most; a
prompt taken whole or in parts; a shared prefix; an empty prompt)
and of the GEMM's row blocks and runs: outputs and the cache slot against
float64, and bit for bit against the prompt decoded alone."""
import numpy as np
import pytest

from tests.rift_testlib import torch_mod

pytestmark = pytest.mark.gpu


def _reference(torch, W, x, keys, values, H, hd, n_pos_of, eps=1e-6, base=10000.0):
    """One layer in float64 for one prompt; keys and values [L][d] as cached."""
    f = lambda t: t.double()
    d = H * hd
    x = f(x)
    h = x / torch.sqrt((x * x).mean() + eps) * f(W["g_attn"])
    q, k, v = (h @ f(W[n]).T for n in ("wq", "wk", "wv"))
    ang = n_pos_of * base ** (-2.0 * torch.arange(hd // 2, device=x.device, dtype=torch.float64) / hd)
    c, s = ang.cos(), ang.sin()

    def rot(t):
        t = t.view(H, hd)
        a, b = t[:, :hd // 2], t[:, hd // 2:]
        return torch.cat([a * c - b * s, b * c + a * s], 1).reshape(d)

    q, k = rot(q), rot(k)
    K = torch.cat([f(keys), k[None]]).view(-1, H, hd).transpose(0, 1)
    V = torch.cat([f(values), v[None]]).view(-1, H, hd).transpose(0, 1)
    p = torch.softmax((K @ q.view(H, hd, 1))[:, :, 0] / hd ** 0.5, dim=1)
    x = x + f(W["wo"]) @ (p[:, :, None] * V).sum(1).reshape(d)
    h = x / torch.sqrt((x * x).mean() + eps) * f(W["g_ffn"])
    g = f(W["w_gate"]) @ h
    return x + f(W["w_down"]) @ (g / (1 + torch.exp(-g)) * (f(W["w_up"]) @ h)), k, v


CASES = [   # heads, head_dim, ffn, prompt rows, prefix rows, step
    (8, 128, 2816, [0, 1, 63, 64, 127, 128, 129, 255, 256, 511, 512, 700, 1030], 0, 0),
    (8, 128, 2176, [5, 300, 900] * 11, 7, 2),            # 33 rows; runs that cross tiles unevenly
    (16, 64, 3456, [0, 127, 254, 255, 256, 700, 1100, 2100], 3, 1),
    (8, 128, 1024, [3 + 11 * i for i in range(66)], 0, 1),      # 66 rows, prompts whole
    (8, 128, 1024, [7 + 19 * i for i in range(63)], 0, 1),      # the most that are taken in parts
    (8, 128, 1024, [2 + 5 * i for i in range(129)], 35, 3),     # 129 rows, prompts whole
    (8, 128, 1024, [1 + i % 40 for i in range(257)], 0, 0),     # three blocks of 128 rows
    (16, 128, 5504, [1 + i % 30 for i in range(190)], 0, 0),    # one block of 192 rows, and two of them
    (16, 128, 5504, [1 + i % 30 for i in range(260)], 0, 0),
    (16, 128, 5504, [1 + i % 30 for i in range(500)], 0, 0),    # two of 256
    (16, 64, 1024, [1 + 17 * i for i in range(64)], 0, 0),      # whole, 64-dimensional heads
    # more than 2,048 workgroups: the two-pass kernel; round, part and stream edges
    (8, 128, 1024, [0, 1, 15, 16, 17, 63, 64, 127, 128, 129, 512, 700, 1030] + [3 + 2 * i for i in range(250)], 0, 2),
    (8, 128, 1024, [1 + i % 70 for i in range(260)], 35, 1),    # prefix rows inside a round
    (16, 64, 1024, [0, 31, 32, 33, 255, 256, 257, 1100] + [2 + 3 * i for i in range(130)], 16, 0),
]


@pytest.mark.parametrize("H,hd,ffn,lens,P,step", CASES)
def test_decode_splits(H, hd, ffn, lens, P, step):
    import paper_2609_29029_amd as R
    torch = torch_mod()
    d, n, max_new = H * hd, len(lens), step + 1
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    mk = lambda *s, std=1.0, mean=0.0: torch.empty(*s, device="cuda", dtype=torch.bfloat16).normal_(mean, std, generator=g)
    shape = dict(wq=(d, d), wk=(d, d), wv=(d, d), wo=(d, d), w_gate=(ffn, d), w_up=(ffn, d), w_down=(d, ffn))
    W = {k: mk(*s, std=0.03) for k, s in shape.items()}
    W["g_attn"], W["g_ffn"] = mk(d, std=0.05, mean=1.0), mk(d, std=0.05, mean=1.0)
    cfg = R.model_cfg(d, H, hd, ffn, 1, 1e-6, 10000.0, R.RIFT_BF16)
    cu = np.concatenate([[0], P + np.cumsum([0] + lens)]) if P else np.concatenate([[0], np.cumsum(lens)])
    T, Lmax = int(cu[-1]), P + max(lens)
    kv = mk(1, 2, max(T, 1), d)
    new = mk(1, 2, n, max_new, d)
    x = mk(n, d)

    def decode(cu, n, kv, new, x, T):
        new = new.clone()
        new[:, :, :, step] = float("nan")   # the slot is written, never read
        ws = torch.empty(R.rift_decode_workspace_size(cfg, n, Lmax, max_new), dtype=torch.uint8, device="cuda")
        ws.fill_(255)
        out = torch.empty(n, d, device="cuda")
        for _ in range(2):                  # a second call on the same workspace gives the same
            R.rift_decode_step(cfg, [W], x, torch.tensor(cu, dtype=torch.int32, device="cuda"), T, Lmax, kv, new, step,
                               out, ws, n_prefix=P)
        return out, new

    out, slots = decode(cu, n, kv, new, x, T)
    torch.cuda.synchronize()
    own = lambda i: int(cu[i + (1 if P else 0)])
    for i in sorted({0, 1, n // 2, n - 2, n - 1} | set(range(min(n, 13)))):
        rows = [kv[0, j, own(i):own(i) + lens[i]] for j in (0, 1)]
        K, V = (torch.cat([kv[0, j, :P], rows[j], new[0, j, i, :step]]) for j in (0, 1))
        ref, k, v = _reference(torch, W, x[i], K, V, H, hd, float(P + lens[i] + step))
        err = lambda a, b: float((a.double() - b).norm() / b.norm())
        # bf16 roundings of h, q, k, v, o and the activation, 2^-9 each relative to its norm
        assert err(out[i], ref) <= 1e-2, (i, lens[i], err(out[i], ref))
        assert err(slots[0, 0, i, step], k) <= 1e-2 and err(slots[0, 1, i, step], v) <= 1e-2
        kv1 = torch.stack([torch.cat([kv[0, j, :P], rows[j]]) for j in (0, 1)])[None].contiguous()
        if kv1.shape[2] == 0:
            kv1 = kv[:, :, :1].contiguous()
        cu1 = [0, P, P + lens[i]] if P else [0, lens[i]]
        alone, slot1 = decode(cu1, 1, kv1, new[:, :, i:i + 1].contiguous(), x[i:i + 1], kv1.shape[2])
        assert torch.equal(alone[0], out[i]), (i, lens[i])
        assert torch.equal(slot1[0, :, 0], slots[0, :, i])


LAYERS = [   # heads, head_dim, ffn, prompt rows, layers: prompts in parts, whole, and many
    (8, 128, 2816, [129, 300, 700, 1100], 3),
    (16, 64, 2816, [129, 257, 700, 1100], 3),
    (16, 128, 4096, [1100, 129, 640], 2),
    (10, 128, 2560, [129, 300, 700, 1100], 3),                  # widths without split K: q, k, v in memory
    (20, 64, 2560, [257, 300, 700, 1100], 3),
    (20, 64, 2560, [257, 300, 700, 1100] * 7, 2),               # whole
    (10, 128, 2560, [129, 300, 700, 1100] * 13, 2),
    (20, 64, 2560, [257, 40, 300, 700, 3] * 21, 2),             # two passes
    (10, 128, 2560, [129, 40, 300, 700, 3] * 42, 2),
    (8, 128, 2816, [129, 40, 300, 700, 3] * 52, 3),
]


@pytest.mark.parametrize("H,hd,ffn,lens,n_layers", LAYERS)
def test_decode_through_layers(H, hd, ffn, lens, n_layers):
    """Several layers with weights and caches of their own: what a layer's attention
    leaves behind (its arrival counters) must not reach the next."""
    import paper_2609_29029_amd as R
    torch = torch_mod()
    d, n = H * hd, len(lens)
    g = torch.Generator(device="cuda")
    g.manual_seed(H + n)
    mk = lambda *s, std=1.0, mean=0.0: torch.empty(*s, device="cuda", dtype=torch.bfloat16).normal_(mean, std, generator=g)
    shape = dict(wq=(d, d), wk=(d, d), wv=(d, d), wo=(d, d), w_gate=(ffn, d), w_up=(ffn, d), w_down=(d, ffn))
    Ws = [{k: mk(*s, std=0.03) for k, s in shape.items()} for _ in range(n_layers)]
    for W in Ws:
        W["g_attn"], W["g_ffn"] = mk(d, std=0.05, mean=1.0), mk(d, std=0.05, mean=1.0)
    cfg = R.model_cfg(d, H, hd, ffn, n_layers, 1e-6, 10000.0, R.RIFT_BF16)
    cu = np.concatenate([[0], np.cumsum(lens)])
    kv, x = mk(n_layers, 2, int(cu[-1]), d), mk(n, d)

    def decode(cu, x, kv):
        m = len(cu) - 1
        slots = torch.full((n_layers, 2, m, 1, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        ws = torch.empty(R.rift_decode_workspace_size(cfg, m, max(lens), 1), dtype=torch.uint8, device="cuda")
        ws.fill_(255)
        out = torch.empty(m, d, device="cuda")
        R.rift_decode_step(cfg, Ws, x, torch.tensor(cu, dtype=torch.int32, device="cuda"), kv.shape[2], max(lens), kv,
                           slots, 0, out, ws)
        return out, slots

    out, slots = decode(cu, x, kv)
    for i in sorted({0, 1, 2, 3, n // 2, n - 1} & set(range(n))):
        rows = kv[:, :, cu[i]:cu[i + 1]]
        ref = x[i].double()
        for l in range(n_layers):
            ref, k, v = _reference(torch, Ws[l], ref, rows[l, 0], rows[l, 1], H, hd, float(lens[i]))
            # as above for one layer; the roundings of the layers before add to it
            for got, want in ((slots[l, 0, i, 0], k), (slots[l, 1, i, 0], v)):
                assert float((got.double() - want).norm() / want.norm()) <= 1e-2 * (l + 1), (i, l)
        assert float((out[i].double() - ref).norm() / ref.norm()) <= 1e-2 * n_layers, i
        alone, slot = decode([0, lens[i]], x[i:i + 1], rows.contiguous())
        assert torch.equal(alone[0], out[i]) and torch.equal(slot[:, :, 0], slots[:, :, i]), i
