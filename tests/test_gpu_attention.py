"""Decode attention (apex_attention_decode) against the oracle's block.

The output must match to float32 rounding (max error 1e-4 of max |o|, and 2e-6 in the
2-norm of the attention over the key and value as they were stored); the key and value
written into the caches must equal the oracle's bf16 rounding of the projections, or
differ by one bf16 step where the float32 and float64 projections straddle a rounding
boundary (counted, at most a few per mille).
"""
import types

import numpy as np
import pytest

from oracle import attention as oatt
from oracle.bf16 import bf16_to_f64
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
    # where the products nearly cancel, 32-bit sums may be more than one (tiny) step off: by up
    # to four roundings of the sum of the products' magnitudes
    size = (np.abs(h.astype(np.float64)) @ np.abs(bf16_to_f64(w_qkv)).T)[:, H * hd:].reshape(B, 2, G, hd)
    for i, (got_bits, want) in enumerate(((k_out[:, :, pos], ref["k_new"]), (v_out[:, :, pos], ref["v_new"]))):
        want_bits = oatt.to_bf16_bits(want)
        steps = np.abs(got_bits.astype(np.int32) - want_bits.astype(np.int32))
        assert (np.abs(bf16_to_f64(got_bits) - want)[steps > 1] <= 2.0 ** -22 * size[:, i][steps > 1]).all()
        off += int((steps == 1).sum())
    assert off <= max(2, 0.005 * 2 * B * G * hd), off
    # against float64 over the caches as they are now, so that only 32-bit rounding is left:
    # three stages of 32-bit sums stay below 5e-7; activations short of their last 8 bits (cut
    # toward zero, 2^-17 of a value on average) would be off by 4e-6 and more
    q = (h.astype(np.float64) @ bf16_to_f64(w_qkv[:H * hd]).T).reshape(B, H, hd)
    K, V = bf16_to_f64(k_out[:, :, :pos + 1]), bf16_to_f64(v_out[:, :, :pos + 1])
    a = np.stack([np.stack([oatt.attend(q[b, i], K[b, i // (H // G)], V[b, i // (H // G)], hd ** -0.5)
                            for i in range(H)]) for b in range(B)])
    want = a.reshape(B, H * hd) @ bf16_to_f64(w_o).T
    err2 = np.linalg.norm(got - want) / np.linalg.norm(want)
    assert err2 <= 2e-6, err2
    return err, off, err2


@pytest.mark.parametrize("name,B,ctx", [
    ("tiny", 1, 0),                     # nothing cached: attends to the new token only
    ("granite-1b-a400m", 1, 1024),
    ("granite-1b-a400m", 4, 37),        # ragged split boundaries
    ("granite-3b-a800m", 2, 512),       # three query heads per key/value head
    ("olmoe-1b-7b", 1, 2048),           # head size 128, one query head per group
    ("mixtral-8x7b", 1, 1024),          # head size 128, four query heads per group
    ("granite-3b-a800m", 1, 1024),      # one token, 1536 values of W_o's rows, 8 splits
    ("olmoe-1b-7b", 1, 1024),           # one token, head size 128, 8 splits
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


# One token whose few splits the output projection merges: 2, 3, 5 and 7 splits, rows of W_o
# of one load per lane, of a whole number of loads, and longer than 8 loads per lane; more
# heads than threads and more than 64 KB of merged values.  (B = 1: d, H, G, hd, ctx)
MERGED = [(72, 8, 2, 64, 100), (264, 4, 4, 128, 170), (64, 48, 12, 128, 300), (520, 16, 8, 64, 430),
          (72, 264, 33, 64, 100), (1024, 192, 24, 128, 300)]


@pytest.mark.parametrize("d,H,G,hd,ctx", MERGED, ids=["-".join(map(str, c)) for c in MERGED])
def test_attention_one_token_few_splits(torch, d, H, G, hd, ctx):
    cfg = types.SimpleNamespace(cfg_id=442, d=d, n_heads=H, n_kv_heads=G, head_dim=hd)
    print(run_case(torch, cfg, 1, ctx))


# Batches whose projections go to the matrix cores, W_qkv's, W_o's or both: token counts at
# the edges of the 16-token tiles and past the largest pass of 64, row and K remainders, one
# split and several.  (B, d, H, G, hd, ctx)
MATRIX = [(2, 2056, 132, 33, 64, 20), (5, 2072, 20, 5, 128, 333), (7, 2056, 16, 2, 128, 1100),
          (16, 1640, 8, 4, 64, 15), (17, 1512, 16, 8, 64, 16), (17, 264, 16, 8, 64, 700),
          (33, 776, 3, 1, 64, 63), (33, 776, 12, 4, 64, 300), (48, 520, 4, 1, 128, 64),
          (65, 376, 8, 1, 64, 130), (130, 200, 6, 2, 64, 31)]


@pytest.mark.parametrize("B,d,H,G,hd,ctx", MATRIX, ids=["-".join(map(str, c)) for c in MATRIX])
def test_attention_projections_on_the_matrix_cores(torch, B, d, H, G, hd, ctx):
    cfg = types.SimpleNamespace(cfg_id=443, d=d, n_heads=H, n_kv_heads=G, head_dim=hd)
    print(run_case(torch, cfg, B, ctx))


# Granite-1B's attention: 4 tokens take the projections one at a time, 16 W_qkv on the matrix
# cores, 32 both; with 1024 positions 32 tokens have two splits, 4 more than eight
@pytest.mark.parametrize("B", [1, 4, 16, 32])
@pytest.mark.parametrize("n_pos", [4, 1024])
def test_attention_keeps_all_24_bits_of_activations(torch, B, n_pos):
    """Answers that lie wholly in the last bits of 24-bit activations, behind a cancellation:
    of h in the key and value projections, of the queries in the scores, of the attention
    vector in the output projection."""
    H, G, hd, d = 16, 8, 64, 1024
    wide = [1.0 + 2.0 ** -9 + 2.0 ** -20, -1.0, -2.0 ** -9]   # sum 2^-20
    f32 = dict(dtype=torch.float32, device="cuda")
    bf16 = dict(dtype=torch.bfloat16, device="cuda")
    ws_bytes = native.apex_attention_workspace_bytes(B, H, G, hd, n_pos)
    pos = n_pos - 1

    def call(h, w_qkv, w_o, kc, vc):
        ws, o = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda"), torch.empty(B, d, **f32)
        native.apex_attention_decode(h, w_qkv, w_o, B, d, H, G, hd, kc, vc, n_pos, pos, o, ws, ws_bytes)
        return o.double().cpu()

    zeros = lambda *s: torch.zeros(*s, **bf16)
    # h: every key and value row sums three entries of the token's own
    h, w_qkv = torch.zeros(B, d, **f32), zeros((H + 2 * G) * hd, d)
    w_qkv[H * hd:] = 1.0
    for b in range(B):
        for j, v in zip((7 + 29 * b, 300 + 5 * b, 1023 - b), wide):
            h[b, j % d] = v
    kc, vc = zeros(B, G, n_pos, hd), zeros(B, G, n_pos, hd)
    call(h, w_qkv, zeros(d, H * hd), kc, vc)
    assert (kc[:, :, pos].double() == 2.0 ** -20).all() and (vc[:, :, pos].double() == 2.0 ** -20).all()
    # queries: three dimensions against a key of 2^23 at position 0, so its score is
    # 2^-20 * 2^23 / 8 = 1 and the others' are 0
    h, w_qkv, w_o = torch.zeros(B, d, **f32), zeros((H + 2 * G) * hd, d), zeros(d, H * hd)
    h[:, 0], h[:, 1], h[:, 2] = 1.0, 2.0 ** -9, 2.0 ** -20
    for i in range(H):
        w_qkv[i * hd, :3] = 1.0
        w_qkv[i * hd + 1, 0] = w_qkv[i * hd + 2, 1] = -1.0
        w_o[i, i * hd] = 1.0
    kc, vc = zeros(B, G, n_pos, hd), zeros(B, G, n_pos, hd)
    kc[:, :, 0, :3] = 2.0 ** 23
    vc[:, :, 0, 0] = 1.0
    e = float(np.exp(1.0))
    o = call(h, w_qkv, w_o, kc, vc)
    assert (o[:, :H] * (e + n_pos - 1) / e - 1.0).abs().max() < 2e-6
    # attention vector: equal scores, so the mean over n_pos (a power of two) positions
    h, w_qkv, w_o = torch.zeros(B, d, **f32), zeros((H + 2 * G) * hd, d), zeros(d, H * hd)
    kc, vc = zeros(B, G, n_pos, hd), zeros(B, G, n_pos, hd)
    for p, v in enumerate((1.0, 2.0 ** -9, 2.0 ** -20)):
        vc[:, :, p, 0] = v
    vc[:, :, 0, 1], vc[:, :, 1, 2] = -1.0, -(2.0 ** -9)
    for i in range(H):
        w_o[i, i * hd:i * hd + 3] = 1.0
    o = call(h, w_qkv, w_o, kc, vc)
    assert (o[:, :H] * n_pos == 2.0 ** -20).all()


@pytest.mark.parametrize("B,pos", [(1, 40), (3, 40), (1, 100), (3, 700), (33, 700)])
def test_attention_infinite_operands_as_in_32_bit_arithmetic(torch, B, pos):
    """An infinite key entry of the sign that scores -inf leaves its position out, and an
    infinite output weight gives infinite outputs, as fp32 multiply-adds do (the matrix
    cores' operands are pieces of a value, some of them zero)."""
    d, H, G, hd = (64, 4, 2, 64) if B <= 16 else (1024, 12, 4, 64)   # the latter: matrix cores
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
