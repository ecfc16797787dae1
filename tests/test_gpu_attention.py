"""Decode attention (apex_attention_decode) against the oracle's block.

The output must match to float32 rounding (max error 1e-4 of max |o|); the key and value
written into the caches must equal the oracle's bf16 rounding of the projections, or
differ by one bf16 step where the float32 and float64 projections straddle a rounding
boundary (counted, at most a few per mille).
"""
import types

import numpy as np
import pytest

from oracle import attention as oatt
from paper_2608_11688_amd import configs, inputs, native

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    return t


def dev(torch, a):
    a = np.ascontiguousarray(a)
    if a.dtype == np.uint16:
        a = a.view(np.int16)
    return torch.from_numpy(a).cuda()


def run_case(torch, cfg, B, ctx, layer=0):
    H, G, hd, d = cfg.n_heads, cfg.n_kv_heads, cfg.head_dim, cfg.d
    ctx_max, pos = ctx + 1, ctx
    w_qkv, w_o = inputs.attention_weights(cfg, layer)
    kc, vc = inputs.kv_cache(cfg, layer, B, ctx_max)
    h = inputs.hidden_states(cfg, layer, B, 1)[0][0]
    k_dev, v_dev = dev(torch, kc), dev(torch, vc)
    o = torch.full((B, d), float("nan"), device="cuda")
    ws_bytes = native.apex_attention_workspace_bytes(B, H, G, hd, ctx_max)
    ws = torch.full((ws_bytes,), 0xAB, dtype=torch.uint8, device="cuda")
    native.apex_attention_decode(dev(torch, h), dev(torch, w_qkv), dev(torch, w_o), B, d, H, G, hd,
                                 k_dev, v_dev, ctx_max, pos, o, ws, ws_bytes)
    torch.cuda.synchronize()
    ref = oatt.attention_block(h, w_qkv, w_o, kc, vc, H, G, hd, pos)
    got = o.cpu().numpy().astype(np.float64)
    err = np.abs(got - ref["o"]).max() / np.abs(ref["o"]).max()
    assert err <= 1e-4, err
    # the cache holds the new key and value at pos and is untouched elsewhere
    k_out = k_dev.cpu().numpy().view(np.uint16)
    v_out = v_dev.cpu().numpy().view(np.uint16)
    assert np.array_equal(np.delete(k_out, pos, axis=2), np.delete(kc, pos, axis=2))
    assert np.array_equal(np.delete(v_out, pos, axis=2), np.delete(vc, pos, axis=2))
    off = 0
    for got_bits, want in ((k_out[:, :, pos], ref["k_new"]), (v_out[:, :, pos], ref["v_new"])):
        want_bits = oatt.to_bf16_bits(want)
        steps = np.abs(got_bits.astype(np.int32) - want_bits.astype(np.int32))
        assert steps.max() <= 1
        off += int((steps == 1).sum())
    assert off <= max(2, 0.005 * 2 * B * G * hd), off
    return err, off


@pytest.mark.parametrize("name,B,ctx", [
    ("tiny", 1, 0),                     # nothing cached: attends to the new token only
    ("granite-1b-a400m", 1, 1024),
    ("granite-1b-a400m", 4, 37),        # ragged split boundaries
    ("granite-3b-a800m", 2, 512),       # three query heads per key/value head
    ("olmoe-1b-7b", 1, 2048),           # head size 128, one query head per group
    ("mixtral-8x7b", 1, 1024),          # head size 128, four query heads per group
    ("mixtral-8x7b", 3, 100),
])
def test_attention_matches_oracle(torch, name, B, ctx):
    cfg = configs.CONFIGS[name]
    print(name, B, ctx, run_case(torch, cfg, B, ctx))


def test_attention_eight_heads_per_group(torch):
    cfg = configs.MoEConfig("att_g8", 440, L=1, d=512, E=4, k=1, I=64, C=4, k_max=4, tau=0.9,
                            steps=1, heads=8, kv_heads=1)
    print("g8", run_case(torch, cfg, 2, 300))


# (B, d, heads, key/value heads, head size, positions already cached): every head grouping
# and head size; batches at the edges of the 16-token tiles and past the largest pass of 64;
# widths that are no whole number of 32-value steps or of 16-row tiles, below and above the
# width from which eight wavefronts share a row; contexts at the edges of the 16-position
# tiles, with one split and with many.
SHAPES = [(2, 64, 1, 1, 64, 0), (16, 72, 2, 1, 64, 15), (17, 264, 3, 1, 64, 16), (33, 136, 4, 2, 64, 63),
          (65, 88, 8, 1, 64, 130), (1, 2056, 2, 2, 128, 17), (5, 2072, 4, 2, 128, 333),
          (32, 2048, 3, 1, 128, 47), (48, 520, 4, 1, 128, 64), (7, 1000, 8, 1, 128, 1100),
          (130, 40, 6, 2, 64, 31)]


@pytest.mark.parametrize("B,d,H,G,hd,ctx", SHAPES, ids=["-".join(map(str, c)) for c in SHAPES])
def test_attention_tile_edges(torch, B, d, H, G, hd, ctx):
    cfg = types.SimpleNamespace(cfg_id=441, d=d, n_heads=H, n_kv_heads=G, head_dim=hd)
    # the same 1e-4 as above: fp32 sums of at most 2072 products, 2e-6 in the 2-norm
    print(run_case(torch, cfg, B, ctx))


@pytest.mark.parametrize("B", [1, 3])
def test_attention_infinite_operands_as_in_32_bit_arithmetic(torch, B):
    """An infinite key entry of the sign that scores -inf leaves its position out, and an
    infinite output weight gives infinite outputs, as fp32 multiply-adds do (the matrix
    cores' operands are pieces of a value, some of them zero)."""
    d, H, G, hd, pos = 64, 4, 2, 64, 40
    g = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    h = torch.ones(B, d, device="cuda")
    w_qkv = torch.full(((H + 2 * G) * hd, d), 1.0 / d, device="cuda").to(torch.bfloat16)   # q = k = v = 1
    w_o = rnd(d, H * hd).to(torch.bfloat16)
    kc, vc = (rnd(B, G, pos + 1, hd).to(torch.bfloat16) for _ in range(2))
    kc[:, :, 7, 3] = float("-inf")
    w_o[5, 9] = float("inf")
    ws_bytes = native.apex_attention_workspace_bytes(B, H, G, hd, pos + 1)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    o = torch.empty(B, d, device="cuda")
    native.apex_attention_decode(h, w_qkv, w_o, B, d, H, G, hd, kc, vc, pos + 1, pos, o, ws, ws_bytes)
    keep = [j for j in range(pos + 1) if j != 7]
    p = torch.softmax(kc[:, :, keep].double().sum(-1) / hd ** 0.5, -1)
    a = (p.unsqueeze(-1) * vc[:, :, keep].double()).sum(2).repeat_interleave(H // G, 1).reshape(B, H * hd)
    want = a @ w_o.double().T
    got = o.double()
    assert torch.equal(got[:, 5], want[:, 5])          # +-inf by the sign of a[:, 9]
    rest = [r for r in range(d) if r != 5]
    err = (got[:, rest] - want[:, rest]).abs().max() / want[:, rest].abs().max()
    assert err <= 1e-4, err


def test_attention_replayed_from_a_captured_graph(torch):
    """Replays with other calls (of other sizes, in the same workspace) between them agree with
    the eager call."""
    d, H, G, hd, pos, B = 256, 4, 2, 64, 700, 3
    g = torch.Generator(device="cuda").manual_seed(6)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    w_qkv, w_o = (rnd((H + 2 * G) * hd, d) / 16).to(torch.bfloat16), (rnd(d, H * hd) / 16).to(torch.bfloat16)
    kc, vc = (rnd(B, G, pos + 1, hd).to(torch.bfloat16) for _ in range(2))
    h, o = rnd(B, d), torch.empty(B, d, device="cuda")
    ws_bytes = native.apex_attention_workspace_bytes(B, H, G, hd, pos + 1)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")

    # the call between has caches of its own: it writes its new position into them, which
    # the longer calls would read
    kc2, vc2 = kc.clone(), vc.clone()

    def call(at, n, stream, k=kc, v=vc):
        native.apex_attention_decode(h, w_qkv, w_o, B, d, H, G, hd, k, v, pos + 1, n, at, ws, ws_bytes,
                                     stream.cuda_stream)

    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call(o, pos, side)
    other = torch.empty_like(o)
    for _ in range(4):
        h.copy_(rnd(B, d))
        graph.replay()
        torch.cuda.synchronize()
        got = o.clone()
        call(other, pos // 2, torch.cuda.current_stream(), kc2, vc2)
        call(other, pos, torch.cuda.current_stream())
        torch.cuda.synchronize()
        assert torch.equal(got, other)


def test_attention_rejects_bad_shapes(torch):
    A = 4096
    with pytest.raises(native.ApexError):
        native.apex_attention_decode(A, A, A, 1, 512, 8, 3, 64, A, A, 10, 0, A, A, 1 << 20)
    with pytest.raises(native.ApexError):
        native.apex_attention_decode(A, A, A, 1, 512, 8, 1, 96, A, A, 10, 0, A, A, 1 << 20)
    with pytest.raises(native.ApexError):
        native.apex_attention_decode(A, A, A, 1, 512, 8, 8, 64, A, A, 10, 10, A, A, 1 << 20)
