"""GPU parity of the short prompts' forward (head dimension 128, csrc/swaa_fwd_short.hip) against the fp64 CPU oracle,
where it can go wrong: halves that do not divide over four waves, ragged last rows and keys, sinks beside the band,
generated rows, both formats, strided tensors, the two ends of its range.  Packed prompts stay on the pipelined kernel,
whose second pass the last test takes at the sizes that fixed-length calls no longer run there."""
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
