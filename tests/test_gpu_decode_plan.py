"""GPU parity of the decode call at the borders of its split plan (number of (sequence, KV head)
pairs and of visited halves), where the output comes from the split kernel itself (one split), and
where some of the workgroup's four waves have no keys; against the fp64 CPU oracle.
"""
import math

import pytest
import torch

from oracle import swaa_decode_oracle
from paper_2512_10411_amd import binding
from paper_2512_10411_amd.inputs import make_qkv
from gpu_util import assert_parity, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hkv,G,Nq,Nk,W,S", [
    (1, 1, 4, 1, 512, 10**9, 0),      # 16 halves: the longest that one workgroup takes alone
    (1, 1, 4, 1, 513, 10**9, 0),      # 17: several splits
    (1, 2, 4, 1, 97, 10**9, 0),       # four halves and one key: the last wave has none
    (127, 1, 1, 1, 1100, 10**9, 4),   # 127 pairs: two splits
    (1, 1, 4, 1, 6177, 10**9, 4),     # 194 halves: the most splits a pair gets
    (128, 1, 2, 1, 3072, 10**9, 4),   # 128 pairs, 96 halves: one split
    (128, 1, 2, 1, 3073, 10**9, 4),   # ... and 97: four
    (257, 1, 1, 1, 3100, 10**9, 0),   # more than 256 pairs: one
    (513, 1, 1, 1, 3100, 10**9, 0),   # more than the workgroups that run at once: four
    (64, 2, 4, 9, 600, 10**9, 4),     # two column tiles, one split
    (3, 2, 5, 13, 2000, 900, 40),     # three column tiles (one workgroup with a single one), many splits, window + sinks
])
def test_borders_of_the_split_plan(B, Hkv, G, Nq, Nk, W, S):
    tag = f"decode B{B} Hkv{Hkv} G{G} Nq{Nq} Nk{Nk} W{W} S{S}"
    print(f"[case] {tag}", flush=True)
    q, k, v = make_qkv(B, Hkv * G, Hkv, Nk, 128, seed=97000 + B + Nk, n_query=Nq)
    out, lse = binding.swaa_attn_decode(to_device(q), to_device(k), to_device(v), W, S)
    torch.cuda.synchronize()
    ro, rl = swaa_decode_oracle(q, k, v, W, S, 1 / math.sqrt(128))
    assert_parity(out, lse, ro, rl, tag=tag)


def test_sequences_of_one_split_beside_long_ones():
    # per-sequence lengths: short sequences leave the split kernel finished, long ones go through the merge
    lens = [1, 32, 33, 129, 500, 9000, 17, 3000]
    host = [make_qkv(1, 8, 2, n, 128, 97900 + i, n_query=1) for i, n in enumerate(lens)]
    q = torch.cat([to_device(h[0]) for h in host])
    k = torch.zeros((len(lens), 2, max(lens), 128), dtype=torch.bfloat16, device="cuda")
    v = torch.zeros_like(k)
    for b, (h, n) in enumerate(zip(host, lens)):
        k[b, :, :n], v[b, :, :n] = to_device(h[1])[0], to_device(h[2])[0]
    sl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    for W in (10**9, 300):
        out, lse = binding.swaa_attn_decode_ex(q, k, v, W, 4, seq_lens=sl)
        torch.cuda.synchronize()
        for b, h in enumerate(host):
            ro, rl = swaa_decode_oracle(*h, W, 4, 1 / math.sqrt(128))
            assert_parity(out[b:b + 1], lse[b:b + 1], ro, rl, tag=f"seq {b} of {lens[b]} W{W}")
