"""GPU parity of the short prompts' forward (head dimension 128, csrc/swaa_fwd_short.hip) against the fp64 CPU oracle,
where it can go wrong: halves that do not divide over four waves, ragged last rows and keys, sinks beside the band,
generated rows, both formats, strided tensors, the two ends of its range.  Packed prompts stay on the pipelined kernel
(row tiles), whose second pass the last test takes, as do the tests of other files that run packed."""
import math

import pytest
import torch

from oracle import input_format, swaa_attn_oracle, swaa_decode_oracle
from paper_2512_10411_amd import binding
from paper_2512_10411_amd.inputs import make_qkv
from gpu_util import assert_parity, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hkv,G,N,W,S,P,fmt", [
    (1, 1, 1, 65, 65, 0, None, "bf16"),       # the shortest: three halves, the last of one row, a wave without any
    (2, 1, 3, 96, 40, 5, None, "fp16"),       # three groups of rows, no power of two of heads
    (1, 2, 4, 161, 1, 0, None, "bf16"),       # every row sees itself only
    (1, 2, 5, 317, 64, 70, None, "fp16"),     # three sink halves in front of the band
    (3, 2, 2, 500, 100, 4, 430, "bf16"),      # prompt rows beside generated ones
    (1, 1, 4, 4096, 10**9, 0, None, "bf16"),  # the most keys, and all 512 workgroups
    (1, 1, 1, 4097, 300, 4, None, "bf16"),    # one key more: the pipelined kernel
])
def test_shapes(B, Hkv, G, N, W, S, P, fmt):
    tag = f"short B{B} Hkv{Hkv} G{G} N{N} W{W} S{S} P{P} {fmt}"
    print(f"[case] {tag}", flush=True)
    q, k, v = make_qkv(B, Hkv * G, Hkv, N, 128, seed=97000 + N, fmt=fmt)
    out, lse = binding.swaa_attn_fwd_ex(to_device(q, fmt), to_device(k, fmt), to_device(v, fmt), W, S, P)
    torch.cuda.synchronize()
    with input_format(fmt):
        ro, rl = swaa_decode_oracle(q, k, v, W, S, 1 / math.sqrt(128), n_prompt=P)
    assert_parity(out, lse, ro, rl, tag=tag)


def test_strided_tensors_give_the_same_bits():
    # rows of k and v 2 Hkv D elements apart, q, out token-major
    B, Hq, Hkv, N, W, S = 2, 4, 2, 300, 90, 4
    q, k, v = (to_device(x) for x in make_qkv(B, Hq, Hkv, N, 128, seed=97500))
    o0, l0 = binding.swaa_attn_fwd(q, k, v, W, S)
    kv = torch.stack([k, v], dim=0).permute(1, 3, 0, 2, 4).contiguous()
    qt = q.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    o1, l1 = binding.swaa_attn_fwd_ex(qt, kv[:, :, 0].permute(0, 2, 1, 3), kv[:, :, 1].permute(0, 2, 1, 3), W, S)
    torch.cuda.synchronize()
    assert torch.equal(o0, o1.contiguous()) and torch.equal(l0, l1)


@pytest.mark.parametrize("fmt", ["bf16", "fp16"])
@pytest.mark.parametrize("Nq,N,W,S,dead", [
    (500, 500, 500, 0, (128, 256)),     # all the keys of one wave
    (1000, 1000, 700, 4, (300, 900)),   # of several, behind the sinks; row 899's own key among them
    (1, 4000, 4000, 4, (0, 1500)),      # few rows on a longer cache: the same routine
    (4, 3000, 1000, 4, (64, 2500)),
])
def test_keys_that_score_minus_infinity_weigh_nothing(Nq, N, W, S, dead, fmt):
    # a mask carried by a component of its own: 1 in every query, 0 or -infinity in the keys.  A wave whose first halves hold
    # such keys alone has no reference yet.
    q, k, v = make_qkv(1, 8, 2, N, 128, seed=97800 + N, n_query=None if Nq == N else Nq, fmt=fmt)
    one, minus_inf = (0x3F80, 0xFF80) if fmt == "bf16" else (0x3C00, 0xFC00)
    q[..., 5], k[..., 5] = one, 0
    k[:, :, dead[0]:dead[1], 5] = minus_inf
    out, lse = binding.swaa_attn_fwd_ex(to_device(q, fmt), to_device(k, fmt), to_device(v, fmt), W, S)
    torch.cuda.synchronize()
    with input_format(fmt):
        ro, rl = swaa_decode_oracle(q, k, v, W, S, 1 / math.sqrt(128))
    assert_parity(out, lse, ro, rl, tag=f"keys {dead} of {N} at -infinity {fmt}")


def test_bits_of_a_prompt_by_the_form_of_the_call():
    # Row tiles give a prompt the same bits packed, paged and in a batch of more than 512 units; alone it runs on the short
    # prompts' kernel.  Each of two results is off by its rounding of P and of O, u / sqrt 3 relative each (u = 2^-9, errors spread
    # evenly over [-u, u]); their distance is 2 u / sqrt 3 of the norm, and the bar twice that.
    Hq, Hkv, N, W, S, page = 8, 2, 500, 200, 4, 16
    B = 512 // (Hq * ((N + 31) // 32)) + 1
    q, k, v = (to_device(x) for x in make_qkv(B, Hq, Hkv, N, 128, seed=97700))
    batch, lse_batch = binding.swaa_attn_fwd(q, k, v, W, S)
    cu = torch.tensor([0, N], dtype=torch.int32).cuda()
    packed, lse_packed = binding.swaa_attn_fwd_ex(q[0], k[0], v[0], W, S, cu_seqlens_q=cu, cu_seqlens_k=cu, max_seqlen_q=N, max_seqlen_k=N)
    pages = (N + page - 1) // page
    cache = [torch.zeros(Hkv, pages * page, 128, dtype=x.dtype, device="cuda") for x in (k, v)]
    for c, x in zip(cache, (k, v)):
        c[:, :N] = x[0]
    cache = [c.view(Hkv, pages, page, 128).transpose(0, 1).contiguous() for c in cache]
    table = torch.arange(pages, dtype=torch.int32, device="cuda")[None]
    paged, lse_paged = binding.swaa_attn_fwd_ex(q[:1], *cache, W, S, block_table=table, max_seqlen_k=N)
    alone, lse_alone = binding.swaa_attn_fwd(q[:1].contiguous(), k[:1].contiguous(), v[:1].contiguous(), W, S)
    torch.cuda.synchronize()
    assert torch.equal(batch[0], packed) and torch.equal(batch[:1], paged)
    assert torch.equal(lse_batch[0], lse_packed) and torch.equal(lse_batch[:1], lse_paged)
    assert (alone.float() - paged.float()).norm() <= 4 * 2.0**-9 / math.sqrt(3) * paged.float().norm()
    assert (lse_alone - lse_paged).abs().max() <= 1e-5


@pytest.mark.parametrize("factor", [1.0, 60.0])  # 60: scores far above the first keys', the second pass
def test_packed_prompts_on_the_pipelined_kernel(factor):
    Hq, Hkv, N, W, S = 4, 1, 700, 300, 4
    q, k, v = make_qkv(1, Hq, Hkv, N, 128, seed=97600)
    kd = to_device(k)
    kd[:, :, 350] *= factor
    k = kd.view(torch.int16).cpu().numpy().view("uint16")
    cu = torch.tensor([0, N], dtype=torch.int32).cuda()
    out, lse = binding.swaa_attn_fwd_ex(to_device(q)[0], kd[0], to_device(v)[0], W, S, cu_seqlens_q=cu, cu_seqlens_k=cu,
                                        max_seqlen_q=N, max_seqlen_k=N)
    torch.cuda.synchronize()
    ro, rl = swaa_attn_oracle(q, k, v, W, S, 1 / math.sqrt(128))
    assert_parity(out[None], lse[None], ro, rl, tag=f"packed, factor {factor}")


@pytest.mark.parametrize("B,Hkv,G,N,W,S,P", [
    (1, 2, 1, 5003, 300, 4, 4800),    # longer than the kernel's own prompts, few generated rows: their chain is the call
    (9, 2, 1, 2500, 100, 70, 2490),   # more than a round of units, sinks, a tile with both kinds of rows
    (1, 1, 4, 6000, 300, 4, 5990),    # four heads to a row tile
])
def test_long_rows_among_short_ones(B, Hkv, G, N, W, S, P):
    q, k, v = make_qkv(B, Hkv * G, Hkv, N, 128, seed=97900 + N)
    print(f"[case] long rows B{B} Hkv{Hkv} G{G} N{N} W{W} S{S} P{P}", flush=True)
    qd, kd, vd = to_device(q), to_device(k), to_device(v)
    out, lse = binding.swaa_attn_fwd_fa_decode(qd, kd, vd, W, S, P)
    ro, rl = swaa_decode_oracle(q, k, v, W, S, 1 / math.sqrt(128), n_prompt=P)
    assert_parity(out, lse, ro, rl, tag=f"long rows of {N}")
