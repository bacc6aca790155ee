"""GPU parity of the forward kernel for head dimension 64 against the fp64 CPU oracle, where it can go wrong: the
reference that moves with a slack (late spikes, rows whose first halves are invisible), odd and even numbers of
halves, sinks beside the band, one, two and four heads per workgroup, both formats."""
import math

import numpy as np
import pytest
import torch

from oracle import input_format, swaa_attn_oracle, swaa_decode_oracle
from paper_2512_10411_amd import binding
from paper_2512_10411_amd.inputs import f32_to_bf16_bits, make_qkv
from gpu_util import assert_parity, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hkv,G,Nq,Nk,W,S,P,fmt", [
    (1, 1, 1, 1, 1, 1, 0, None, "bf16"),
    (1, 2, 4, 33, 33, 33, 0, None, "fp16"),          # two halves, the second with one row
    (2, 1, 7, 97, 97, 40, 5, None, "bf16"),          # 4 + 2 + 1 heads, an odd number of halves
    (1, 1, 4, 200, 1000, 64, 70, None, "bf16"),      # three sink halves in front of the band
    (1, 2, 5, 130, 3001, 10**9, 0, None, "fp16"),    # a long chain, ragged last half
    (1, 1, 2, 300, 700, 100, 4, 500, "bf16"),        # prompt rows beside generated ones
])
def test_shapes(B, Hkv, G, Nq, Nk, W, S, P, fmt):
    tag = f"d64 B{B} Hkv{Hkv} G{G} Nq{Nq} Nk{Nk} W{W} S{S} P{P} {fmt}"
    print(f"[case] {tag}", flush=True)
    q, k, v = make_qkv(B, Hkv * G, Hkv, Nk, 64, seed=96000 + Nq + Nk, n_query=Nq, fmt=fmt)
    out, lse = binding.swaa_attn_fwd_ex(to_device(q, fmt), to_device(k, fmt), to_device(v, fmt), W, S, P)
    torch.cuda.synchronize()
    with input_format(fmt):
        ro, rl = swaa_decode_oracle(q, k, v, W, S, 1 / math.sqrt(64), n_prompt=P)
    assert_parity(out, lse, ro, rl, tag=tag)


@pytest.mark.parametrize("key", [0, 40, 95, 700])
@pytest.mark.parametrize("height", [4.0, 40.0, 300.0])  # below the slack of 2^8, above it, far above
def test_a_spike_moves_the_reference(key, height):
    q, k, v = make_qkv(1, 4, 1, 800, 64, seed=97)
    bits = lambda x: f32_to_bf16_bits(np.float32(x))
    q[..., 0], k[..., 0] = bits(2.0), bits(0.0)
    k[:, :, key, 0] = bits(height)
    out, lse = binding.swaa_attn_fwd(to_device(q), to_device(k), to_device(v), 300, 4)
    torch.cuda.synchronize()
    ro, rl = swaa_decode_oracle(q, k, v, 300, 4, 1 / math.sqrt(64))
    assert_parity(out, lse, ro, rl, tag=f"d64 spike {height} at {key}")


@pytest.mark.parametrize("fmt", ["bf16", "fp16"])
def test_non_finite_key_rows_reach_only_the_rows_that_see_them(fmt):
    # NaN and infinities in a few key rows (as at head dimension 128, test_gpu_parity.py): a row that does not see
    # such a key comes out as the oracle has it, although rows 16 above or below it, which share columns of the
    # row sums' products with it, do see the key
    B, Hq, Hkv, N, W, S = 1, 8, 2, 1500, 100, 4
    q, k, v = make_qkv(B, Hq, Hkv, N, 64, seed=4964, fmt=fmt)
    nan, inf = (0x7FC0, 0x7F80) if fmt == "bf16" else (0x7E00, 0x7C00)
    poisoned = {500: nan, 777: inf, 778: 0x8000 | inf, 1290: 0x8000 | nan}
    for j, bits in poisoned.items():
        k[:, :, j, 5::7] = np.uint16(bits)
    out, lse = binding.swaa_attn_fwd_ex(to_device(q, fmt), to_device(k, fmt), to_device(v, fmt), W, S)
    torch.cuda.synchronize()
    touched = sorted({i for j in poisoned for i in range(j, min(N, j + W))})
    rows = np.array([i for i in range(N) if i not in set(touched)], dtype=np.int32)
    with input_format(fmt):
        ro, rl = swaa_attn_oracle(q, k, v, W, S, 1 / math.sqrt(64), rows=rows)
    assert np.isfinite(ro).all() and np.isfinite(rl).all()
    assert_parity(out, lse, ro, rl, rows=rows, tag=f"d64 non-finite invisible keys {fmt}")
    for j in (500, 1290):  # and the rows that see a NaN show it
        assert not torch.isfinite(out[:, :, j:j + W].float()).any() and not torch.isfinite(lse[:, :, j:j + W]).any()


@pytest.mark.parametrize("what", ["spike", "nan"])
@pytest.mark.parametrize("fmt", ["bf16", "fp16"])
def test_packed_prompts_keep_to_the_row_tiles(what, fmt):
    # (prompts of one length run on another kernel up to a size; packed ones never do)
    Hq, Hkv, N, W, S = 8, 2, 900, 100, 4
    q, k, v = make_qkv(1, Hq, Hkv, N, 64, seed=4970, fmt=fmt)
    if what == "spike":  # far above the slack, behind the first halves
        one, high = (0x4000, 0x4396) if fmt == "bf16" else (0x4000, 0x5CB0)  # 2 and 300
        q[..., 0], k[..., 0] = one, 0
        k[:, :, 600, 0] = high
        sees = np.zeros(N, bool)
    else:
        k[:, :, 600, 5::7] = 0x7FC0 if fmt == "bf16" else 0x7E00
        sees = (np.arange(N) >= 600) & (np.arange(N) < 600 + W)
    cu = torch.tensor([0, N], dtype=torch.int32, device="cuda")
    out, lse = binding.swaa_attn_fwd_ex(*(to_device(t[0], fmt) for t in (q, k, v)), W, S, cu_seqlens_q=cu, cu_seqlens_k=cu,
                                        max_seqlen_q=N, max_seqlen_k=N)
    torch.cuda.synchronize()
    k[:, :, 600, 5::7] = k[:, :, 600, 5::7] if what == "spike" else 0
    with input_format(fmt):
        ro, rl = swaa_decode_oracle(q, k, v, W, S, 1 / math.sqrt(64))
    keep = torch.from_numpy(~sees)
    assert_parity(out[None][:, :, keep.cuda()], lse[None][:, :, keep.cuda()], ro[:, :, ~sees], rl[:, :, ~sees], tag=f"packed d64 {what} {fmt}")
    assert what == "spike" or torch.isnan(lse[:, torch.from_numpy(sees).cuda()]).all()


@pytest.mark.parametrize("B,Hkv,G,N,W,S,P,fmt", [
    (1, 1, 1, 32, 32, 0, None, "bf16"),     # one half: rows of four heads together
    (1, 1, 1, 33, 33, 0, None, "bf16"),     # two, a wave each, two waves without any
    (2, 1, 3, 161, 40, 70, 100, "fp16"),    # sinks beside the band, generated rows
    (3, 4, 4, 1000, 260, 4, None, "bf16"),  # 1536 units
    (3, 4, 4, 1030, 260, 4, None, "bf16"),  # 1584: row tiles
    (3, 4, 4, 1030, 40, 4, None, "fp16"),   # ... on a short window
    (4, 4, 4, 1700, 100, 4, 1690, "bf16"),  # 3456, few generated rows are the time
])
def test_both_kernels_at_the_lines_between_them(B, Hkv, G, N, W, S, P, fmt):
    print(f"[case] d64 line B{B} Hkv{Hkv} G{G} N{N} W{W} S{S} P{P} {fmt}", flush=True)
    q, k, v = make_qkv(B, Hkv * G, Hkv, N, 64, seed=96500 + N, fmt=fmt)
    out, lse = binding.swaa_attn_fwd_ex(*(to_device(t, fmt) for t in (q, k, v)), W, S, P)
    torch.cuda.synchronize()
    with input_format(fmt):
        ro, rl = swaa_decode_oracle(q, k, v, W, S, 1 / math.sqrt(64), n_prompt=P)
    assert_parity(out, lse, ro, rl, tag=f"d64 line N{N} W{W}")
