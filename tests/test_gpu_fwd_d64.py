"""GPU parity of the forward kernel for head dimension 64 against the fp64 CPU oracle, where it can go wrong: the
reference that moves with a slack (late spikes, rows whose first halves are invisible), odd and even numbers of
halves, sinks beside the band, one, two and four heads per workgroup, both formats."""
import math

import numpy as np
import pytest
import torch

from oracle import input_format, swaa_decode_oracle
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
