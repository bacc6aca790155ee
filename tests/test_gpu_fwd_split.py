"""GPU parity of the forward with keys split over several workgroups (swaa_attn_fwd_ex on few query
rows and many keys), against the fp64 CPU oracle: split boundaries inside and outside the window,
ragged last halves, sink halves in the first split only, tiles with fewer halves than the sequence's
split count has (empty splits), rows that see no key of a split, every head grouping, both formats.
"""
import math

import numpy as np
import pytest
import torch

from oracle import input_format, swaa_decode_oracle
from paper_2512_10411_amd import binding
from paper_2512_10411_amd.inputs import make_qkv
from gpu_util import assert_parity, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture
def scratch(monkeypatch):
    """The workspace bytes of every swaa_attn_fwd_ex call (0: its keys stay whole); the workspaces hold 0xFF bytes,
    NaN patterns that show if a partial result is read that was not written."""
    lib, sizes = binding.load_library(), []
    query, launch = lib.swaa_attn_fwd_ex_workspace_bytes, lib.swaa_attn_fwd_ex_ws

    def recording(args):
        sizes.append(int(query(args)))
        return sizes[-1]

    def filled(args, workspace, workspace_bytes):
        full = torch.full((workspace_bytes,), 255, dtype=torch.uint8, device="cuda")
        kept.append(full)
        return launch(args, full.data_ptr(), workspace_bytes)

    kept = []
    monkeypatch.setattr(lib, "swaa_attn_fwd_ex_workspace_bytes", recording)
    monkeypatch.setattr(lib, "swaa_attn_fwd_ex_ws", filled)
    return sizes


@pytest.mark.parametrize("B,Hkv,G,Nq,Nk,W,S,P,fmt", [
    (1, 1, 4, 1, 1025, 10**9, 4, None, "bf16"),     # 33 halves of few rows: a tile of their own kind, whole
    (1, 1, 4, 9, 1025, 10**9, 4, None, "bf16"),     # 33 halves: the shortest split range, odd last split
    (1, 1, 4, 33, 3001, 10**9, 0, None, "fp16"),    # two row tiles, ragged last half
    (1, 2, 5, 130, 4000, 10**9, 4, None, "bf16"),   # groups of four heads and one
    (2, 1, 7, 65, 2500, 1100, 70, None, "bf16"),    # 4 + 2 + 1 heads, sink halves in front of the band
    (1, 1, 1, 300, 5000, 1030, 4, None, "fp16"),    # one head per workgroup: 128 positions, band edges apart
    (1, 1, 4, 700, 2000, 10**9, 4, None, "bf16"),   # causal: tiles with fewer halves than the last
    (1, 1, 4, 40, 3000, 1, 1500, None, "bf16"),     # nearly all keys are sinks
    (1, 1, 4, 64, 2100, 40, 4, 2100 - 64, "bf16"),  # generated rows only
])
def test_fixed_length_chunks(scratch, B, Hkv, G, Nq, Nk, W, S, P, fmt):
    tag = f"split B{B} Hkv{Hkv} G{G} Nq{Nq} Nk{Nk} W{W} S{S} P{P} {fmt}"
    print(f"[case] {tag}", flush=True)
    q, k, v = make_qkv(B, Hkv * G, Hkv, Nk, 128, seed=91000 + Nq + Nk, n_query=Nq, fmt=fmt)
    out, lse = binding.swaa_attn_fwd_ex(to_device(q, fmt), to_device(k, fmt), to_device(v, fmt), W, S, P)
    torch.cuda.synchronize()
    assert scratch[0] > 0
    with input_format(fmt):
        ro, rl = swaa_decode_oracle(q, k, v, W, S, 1 / math.sqrt(128), n_prompt=P)
    assert_parity(out, lse, ro, rl, tag=tag)


def test_a_late_spike_in_one_split_takes_the_second_pass(scratch):
    # scores 80 nats above the first keys of a split: that split's workgroups recompute, the others do not
    q, k, v = make_qkv(1, 4, 1, 3000, 128, seed=92, n_query=40)
    to_bits = lambda x: np.array([x], dtype=np.float32).view(np.uint32)[0] >> 16
    q[..., 0], k[..., 0] = to_bits(3.0), to_bits(0.0)
    k[:, :, 1700, 0] = to_bits(304.0)
    out, lse = binding.swaa_attn_fwd_ex(to_device(q), to_device(k), to_device(v), 10**9, 4)
    torch.cuda.synchronize()
    assert scratch[0] > 0
    ro, rl = swaa_decode_oracle(q, k, v, 10**9, 4, 1 / math.sqrt(128))
    assert_parity(out, lse, ro, rl, tag="split, late spike")


@pytest.mark.parametrize("n_singles,W,fmt,page", [(20, 300, "fp16", 16), (62, 40, "bf16", 48), (3, 2000, "bf16", 0)])
def test_generated_tokens_beside_a_chunk(scratch, n_singles, W, fmt, page):
    # a packed batch: single generated tokens on caches of very different lengths, an empty sequence, a chunk
    # without generated rows, and a sequence of prompt and generated rows (never split)
    rng = np.random.Generator(np.random.Philox(93 + n_singles))
    Hkv, G, S = 2, 4, 4
    nk = [int(40 * 150 ** rng.random()) for _ in range(n_singles)]
    nq = [1] * n_singles
    nk += [500, 3000, 900]
    nq += [0, 150, 200]
    if n_singles > 60:
        nk, nq = nk[2:], nq[2:]  # a batch of 63
    prompts = [n - 1 for n in nk[:-3]] + [500, 3000, 800]
    B = len(nk)
    print(f"[case] {B} sequences, caches {min(nk)}..{max(nk)} W{W} {fmt} page {page}", flush=True)
    dt = torch.float16 if fmt == "fp16" else torch.bfloat16
    host = [make_qkv(1, Hkv * G, Hkv, n, 128, 94000 + i, n_query=max(m, 1), fmt=fmt) for i, (m, n) in enumerate(zip(nq, nk))]
    q = torch.cat([to_device(h[0], fmt)[0, :, :m] for h, m in zip(host, nq)], dim=1).contiguous()
    offs = lambda x: torch.tensor(np.concatenate([[0], np.cumsum(x)]), dtype=torch.int32, device="cuda")
    args = dict(cu_seqlens_q=offs(nq), cu_seqlens_k=offs(nk), max_seqlen_q=max(nq), max_seqlen_k=max(nk),
                n_prompts=torch.tensor(prompts, dtype=torch.int32, device="cuda"))
    dev = [(to_device(h[1], fmt)[0], to_device(h[2], fmt)[0]) for h in host]
    if page:
        pages = [(n + page - 1) // page for n in nk]
        order = rng.permutation(sum(pages))
        kk, vv = (torch.full((sum(pages), Hkv, page, 128), float("nan"), dtype=dt, device="cuda") for _ in range(2))
        table, at = np.zeros((B, max(pages)), np.int32), 0
        for b, n in enumerate(nk):
            table[b, :pages[b]] = order[at:at + pages[b]]
            for j in range(pages[b]):
                rows = slice(j * page, min(n, (j + 1) * page))
                kk[table[b, j], :, :rows.stop - rows.start] = dev[b][0][:, rows]
                vv[table[b, j], :, :rows.stop - rows.start] = dev[b][1][:, rows]
            at += pages[b]
        args["block_table"] = torch.from_numpy(table).cuda()
    else:
        kk, vv = (torch.cat([d[i] for d in dev], dim=1).contiguous() for i in range(2))
    outs = [tuple(t.clone() for t in binding.swaa_attn_fwd_ex(q, kk, vv, W, S, total_rows_q=t, **args)) for t in (None, None, 0)]
    torch.cuda.synchronize()
    assert all(n > 0 for n in scratch)
    assert all(torch.equal(outs[0][0], o) and torch.equal(outs[0][1], l) for o, l in outs[1:])
    r0 = 0
    with input_format(fmt):
        for b, h in enumerate(host):
            if nq[b]:
                ro, rl = swaa_decode_oracle(h[0], h[1], h[2], W, S, 1 / math.sqrt(128), n_prompt=prompts[b])
                assert_parity(outs[0][0][None, :, r0:r0 + nq[b]], outs[0][1][None, :, r0:r0 + nq[b]], ro, rl,
                              tag=f"seq {b}: {nq[b]} rows on {nk[b]} keys")
            r0 += nq[b]


@pytest.mark.parametrize("nq,nk,W,whole", [
    ([333, 400], [1500, 2000], 900, True),    # 72 units on a short window: whole
    ([64, 640], [2000, 1100], 900, True),     # the shortest sequence taken for a chunk
    ([63, 640], [2000, 1100], 900, False),    # one row less: planned on the device
    ([333, 400], [1500, 2000], 1500, False),  # a longer window
])
def test_chunks_give_the_same_bits_whichever_list_they_run_on(scratch, nq, nk, W, whole):
    # whether the caller states the number of rows or not, a batch is split or left whole alike
    Hkv, G, S, B = 3, 4, 4, len(nq)
    print(f"[case] chunks {nq} on {nk} W{W}", flush=True)
    host = [make_qkv(1, Hkv * G, Hkv, n, 128, 95000 + n, n_query=m) for m, n in zip(nq, nk)]
    q, kk, vv = (torch.cat([to_device(h[i])[0] for h in host], dim=1).contiguous() for i in range(3))
    offs = lambda x: torch.tensor(np.concatenate([[0], np.cumsum(x)]), dtype=torch.int32, device="cuda")
    args = dict(cu_seqlens_q=offs(nq), cu_seqlens_k=offs(nk), max_seqlen_q=max(nq), max_seqlen_k=max(nk),
                n_prompts=torch.tensor(nk, dtype=torch.int32, device="cuda"))
    (out, lse), (o0, l0) = (tuple(t.clone() for t in binding.swaa_attn_fwd_ex(q, kk, vv, W, S, total_rows_q=t, **args)) for t in (None, 0))
    torch.cuda.synchronize()
    assert (scratch[0] == 0) == whole and scratch[1] > 0
    assert torch.equal(out, o0) and torch.equal(lse, l0)
    r0 = 0
    for b, h in enumerate(host):
        ro, rl = swaa_decode_oracle(h[0], h[1], h[2], W, S, 1 / math.sqrt(128))
        assert_parity(out[None, :, r0:r0 + nq[b]], lse[None, :, r0:r0 + nq[b]], ro, rl, tag=f"seq {b}: {nq[b]} rows on {nk[b]} keys")
        r0 += nq[b]


@pytest.mark.parametrize("fmt", ["bf16", "fp16"])
@pytest.mark.parametrize("what", ["nan", "inf"])
def test_a_non_finite_key_of_one_split_reaches_the_rows_that_see_it(scratch, what, fmt):
    # the merge must not take a split whose sums are not numbers for one without keys
    q, k, v = make_qkv(1, 4, 1, 5000, 128, seed=9650, n_query=300, fmt=fmt)
    bits = {("nan", "bf16"): 0x7FC0, ("inf", "bf16"): 0x7F80, ("nan", "fp16"): 0x7E00, ("inf", "fp16"): 0x7C00}[what, fmt]
    q[..., 5] = {"bf16": 0x3F80, "fp16": 0x3C00}[fmt]  # 1: the score of an infinite component is +infinity
    W, key = 1030, 3900  # seen by positions 3900 .. 4929, the chunk's first 230 rows
    k[:, :, key, 5] = np.uint16(bits)
    out, lse = binding.swaa_attn_fwd_ex(to_device(q, fmt), to_device(k, fmt), to_device(v, fmt), W, 4)
    torch.cuda.synchronize()
    assert scratch[0] > 0
    assert not torch.isfinite(out[:, :, :230].float()).any() and not torch.isfinite(lse[:, :, :230]).any()
    rows = np.arange(230, 300)
    with input_format(fmt):
        ro, rl = swaa_decode_oracle(q, k, v, W, 4, 1 / math.sqrt(128))
    assert_parity(out[:, :, rows], lse[:, :, rows], ro[:, :, rows], rl[:, :, rows], tag=f"split, {what} key, rows that do not see it")


def test_without_memory_for_scratch_the_keys_stay_whole(scratch, monkeypatch):
    q, k, v = make_qkv(1, 4, 1, 3001, 128, seed=9670, n_query=33)
    qd, kd, vd = to_device(q), to_device(k), to_device(v)
    empty = torch.empty

    def no_scratch(*args, **kwargs):
        if kwargs.get("dtype") == torch.uint8:
            raise torch.cuda.OutOfMemoryError("no memory")
        return empty(*args, **kwargs)

    monkeypatch.setattr(torch, "empty", no_scratch)
    out, lse = binding.swaa_attn_fwd_ex(qd, kd, vd, 10**9, 4)
    torch.cuda.synchronize()
    assert scratch[0] > 0
    monkeypatch.undo()
    ro, rl = swaa_decode_oracle(q, k, v, 10**9, 4, 1 / math.sqrt(128))
    assert_parity(out, lse, ro, rl, tag="no scratch")


@pytest.mark.parametrize("Hkv,G,nq,nk,W,S,P,fmt,page", [
    (2, 4, 8, 3001, 10**9, 4, None, "bf16", 0),       # 32 columns, a full tile
    (1, 4, 9, 3001, 10**9, 4, None, "bf16", 0),       # one row more: a row tile again
    (1, 1, 32, 2500, 900, 70, None, "fp16", 16),      # one head, sinks in front of the band
    (2, 5, 6, 5003, 10**9, 0, None, "fp16", 48),      # 30 columns, pages that are no multiple of a half
    (1, 8, 1, 1040, 10**9, 4, None, "bf16", 16),      # 33 halves, the last of 16 keys: ends inside a page pair
    (1, 8, 4, 1025, 10**9, 4, None, "bf16", 64),      # ... of one key
    (1, 32, 1, 4000, 1500, 1000, None, "bf16", 0),    # 32 heads on one
    (2, 4, 5, 4000, 1100, 40, 3998, "bf16", 32),      # prompt and generated rows in one tile
    (1, 4, 3, 40000, 10**9, 4, None, "fp16", 16),     # many splits
])
def test_few_rows_share_one_column_tile(scratch, Hkv, G, nq, nk, W, S, P, fmt, page):
    # beside a sequence of more rows, so that the batch is planned on the device
    print(f"[case] few rows Hkv{Hkv} G{G} nq{nq} nk{nk} W{W} S{S} P{P} {fmt} page {page}", flush=True)
    lens, rows = [nk, 700, 2000], [nq, 1, 70]
    host = [make_qkv(1, Hkv * G, Hkv, n, 128, 97000 + n + m, n_query=m, fmt=fmt) for m, n in zip(rows, lens)]
    dt = torch.float16 if fmt == "fp16" else torch.bfloat16
    q = torch.cat([to_device(h[0], fmt)[0] for h in host], dim=1).contiguous()
    offs = lambda x: torch.tensor(np.concatenate([[0], np.cumsum(x)]), dtype=torch.int32, device="cuda")
    prompts = [n if P is None else min(n, P) for n in lens]
    args = dict(cu_seqlens_q=offs(rows), cu_seqlens_k=offs(lens), max_seqlen_q=max(rows), max_seqlen_k=max(lens),
                n_prompts=torch.tensor(prompts, dtype=torch.int32, device="cuda"))
    dev = [(to_device(h[1], fmt)[0], to_device(h[2], fmt)[0]) for h in host]
    if page:
        pages = [(n + page - 1) // page for n in lens]
        order = np.random.Generator(np.random.Philox(98)).permutation(sum(pages))
        kk, vv = (torch.full((sum(pages), Hkv, page, 128), float("nan"), dtype=dt, device="cuda") for _ in range(2))
        table, at = np.full((3, max(pages)), 10**9, np.int32), 0
        for b, n in enumerate(lens):
            table[b, :pages[b]] = order[at:at + pages[b]]
            at += pages[b]
            for j in range(pages[b]):
                part = slice(j * page, min(n, (j + 1) * page))
                kk[table[b, j], :, :part.stop - part.start] = dev[b][0][:, part]
                vv[table[b, j], :, :part.stop - part.start] = dev[b][1][:, part]
        args["block_table"] = torch.from_numpy(table).cuda()
    else:
        kk, vv = (torch.cat([d[i] for d in dev], dim=1).contiguous() for i in range(2))
    out, lse = binding.swaa_attn_fwd_ex(q, kk, vv, W, S, **args)
    torch.cuda.synchronize()
    assert scratch[0] > 0
    r0 = 0
    with input_format(fmt):
        for b, h in enumerate(host):
            ro, rl = swaa_decode_oracle(h[0], h[1], h[2], W, S, 1 / math.sqrt(128), n_prompt=prompts[b])
            assert_parity(out[None, :, r0:r0 + rows[b]], lse[None, :, r0:r0 + rows[b]], ro, rl,
                          tag=f"few rows, seq {b}: {rows[b]} rows on {lens[b]} keys")
            r0 += rows[b]


@pytest.mark.parametrize("B,Hkv,Nq,Nk", [(40, 8, 1, 1500), (40, 8, 8, 1500)])
def test_few_rows_of_sequences_of_one_length(scratch, B, Hkv, Nq, Nk):
    # enough of them that no keys are split: 256 bytes of scratch, no merge; without even those the row tiles run
    # (a workspace that is too small is no error where the call needs none)
    q, k, v = make_qkv(B, Hkv * 4, Hkv, Nk, 128, seed=9680 + Nq, n_query=Nq)
    qd, kd, vd = to_device(q), to_device(k), to_device(v)
    print(f"[case] {B} x {Nq} rows on {Nk} keys", flush=True)
    out, lse = (t.clone() for t in binding.swaa_attn_fwd_ex(qd, kd, vd, 10**9, 4))
    assert scratch == [256]
    small = torch.empty(128, dtype=torch.uint8, device="cuda")
    out2, lse2 = binding.swaa_attn_fwd_ex(qd, kd, vd, 10**9, 4, workspace=small)
    torch.cuda.synchronize()
    ro, rl = swaa_decode_oracle(q, k, v, 10**9, 4, 1 / math.sqrt(128))
    assert_parity(out, lse, ro, rl, tag="few rows of one length")
    assert_parity(out2, lse2, ro, rl, tag="few rows of one length, no scratch")
    plain = binding.swaa_attn_fwd_ex(qd, kd, vd, 10**9, 4, workspace=torch.empty(0, dtype=torch.uint8, device="cuda"))
    assert torch.equal(out2, plain[0]) and torch.equal(lse2, plain[1])  # the call without a workspace


@pytest.mark.parametrize("B,Hkv,G,nq,nk,packed,rows", [
    (33, 8, 4, 1, 1500, False, True), (47, 8, 1, 3, 1100, False, True), (19, 16, 2, 2, 1100, False, True),
    (32, 8, 4, 1, 1500, False, False), (48, 8, 4, 1, 1100, False, False),  # 256 and 384 units
    (33, 8, 3, 1, 1100, False, False),                                     # a group of two row tiles
    (33, 8, 4, 1, 1500, True, True), (47, 8, 2, 2, 1100, True, True), (32, 8, 4, 1, 1500, True, False),
])
def test_few_rows_that_fill_more_than_every_compute_unit_once(scratch, B, Hkv, G, nq, nk, packed, rows):
    # 257 to 376 units of whole keys run on row tiles, bit for bit as without a workspace
    q, k, v = make_qkv(B, Hkv * G, Hkv, nk, 128, seed=9695 + B, n_query=nq)
    qd, kd, vd = to_device(q), to_device(k), to_device(v)
    print(f"[case] {B} x {nq} rows on {nk} keys, {Hkv} x {G} heads, packed {packed}", flush=True)
    none = torch.empty(0, dtype=torch.uint8, device="cuda")
    if packed:
        cu = lambda n: torch.arange(0, (B + 1) * n, n, dtype=torch.int32, device="cuda")
        pack = lambda x: x.permute(1, 0, 2, 3).reshape(x.shape[1], -1, 128).contiguous()
        run = lambda ws: binding.swaa_attn_fwd_ex(pack(qd), pack(kd), pack(vd), 10**9, 4, cu_seqlens_q=cu(nq), cu_seqlens_k=cu(nk),
                                                  max_seqlen_q=nq, max_seqlen_k=nk, workspace=ws)
        plain = binding.swaa_attn_fwd_ex(qd, kd, vd, 10**9, 4, workspace=none)
        plain = pack(plain[0]), plain[1].permute(1, 0, 2).reshape(Hkv * G, -1)
    else:
        run = lambda ws: binding.swaa_attn_fwd_ex(qd, kd, vd, 10**9, 4, workspace=ws)
        plain = run(none)
    out, lse = run(None)
    torch.cuda.synchronize()
    assert scratch[-1] > 0
    assert (torch.equal(out, plain[0]) and torch.equal(lse, plain[1])) == rows
    if packed:
        out, lse = (x.view(Hkv * G, B, nq, -1).permute(1, 0, 2, 3) for x in (out, lse))
        lse = lse[..., 0]
    ro, rl = swaa_decode_oracle(q, k, v, 10**9, 4, 1 / math.sqrt(128))
    assert_parity(out, lse, ro, rl, tag=f"few rows, {B * Hkv} units")


@pytest.mark.parametrize("B,Hkv,whole", [(40, 4, False), (41, 4, True), (64, 4, True)])
def test_few_rows_with_a_compute_unit_each_stay_whole(scratch, B, Hkv, whole):
    # 161 to 256 units: 256 bytes of scratch where the sequences are of one length, and the same bits packed
    nk = 14000 if B < 64 else 24000
    q = to_device(make_qkv(B, Hkv, Hkv, 16, 128, seed=9697, n_query=1)[0])
    gen = torch.Generator(device="cuda").manual_seed(B)
    k, v = (torch.randn(B, Hkv, nk, 128, device="cuda", generator=gen).bfloat16() for _ in range(2))
    print(f"[case] {B} x 1 row on {nk} keys, {Hkv} heads", flush=True)
    out, lse = (t.clone() for t in binding.swaa_attn_fwd_ex(q, k, v, 10**9, 4))
    assert (scratch[-1] == 256) == whole
    cu = lambda n: torch.arange(0, (B + 1) * n, n, dtype=torch.int32, device="cuda")
    pack = lambda x: x.permute(1, 0, 2, 3).reshape(Hkv, -1, x.shape[-1]).contiguous()
    out2, lse2 = binding.swaa_attn_fwd_ex(pack(q), pack(k), pack(v), 10**9, 4, cu_seqlens_q=cu(1), cu_seqlens_k=cu(nk),
                                          max_seqlen_q=1, max_seqlen_k=nk)
    torch.cuda.synchronize()
    if whole:
        assert torch.equal(pack(out), out2) and torch.equal(pack(lse[..., None])[..., 0], lse2)
    s = torch.einsum("bhd,bhkd->bhk", q[:, :, 0].float(), k.float()) / math.sqrt(128)
    ro = torch.einsum("bhk,bhkd->bhd", s.softmax(-1), v.float())[:, :, None].cpu().numpy()
    rl = torch.logsumexp(s, -1)[:, :, None].cpu().numpy()
    assert_parity(out, lse, ro, rl, tag=f"few rows, {B * Hkv} units on {nk} keys")


@pytest.mark.parametrize("B,Hkv,G,Nq,Nk", [(1, 2, 5, 6, 3001), (2, 1, 7, 4, 2600), (3, 2, 32, 1, 5000), (1, 1, 31, 1, 40000)])
def test_few_rows_of_large_groups_and_one_length(scratch, B, Hkv, G, Nq, Nk):
    # groups whose row tiles would be two to eight: the workspace, the grid and the merge are those of one tile
    q, k, v = make_qkv(B, Hkv * G, Hkv, Nk, 128, seed=9690 + G, n_query=Nq)
    out, lse = binding.swaa_attn_fwd_ex(to_device(q), to_device(k), to_device(v), 10**9, 4)
    torch.cuda.synchronize()
    assert scratch[0] > 256
    ro, rl = swaa_decode_oracle(q, k, v, 10**9, 4, 1 / math.sqrt(128))
    assert_parity(out, lse, ro, rl, tag=f"few rows, {B} x {Hkv} x {G}, {Nq} on {Nk}")


@pytest.mark.parametrize("nats", [10.0, 13.0, 14.284, 16.0])
@pytest.mark.parametrize("nk", [1100, 5000])  # whole keys (one split), and split
def test_few_rows_in_binary16_keep_the_terms_below_a_sink(scratch, nk, nats):
    # One key `nats` above all the others, and the others alone have values: P of those is p = 2^4 e^-nats beside the
    # reference (2^4 below the largest score), and rounds to a multiple of 2^-24 below 2^-14: off by at most 2^-25 / p
    # of itself there, by 2^-11 above.  2^-11 more for the result's own rounding (values of 32 keep it out of the
    # subnormals), and 2^-11 for the sums of 32-bit terms and the other splits' and waves' weights.
    bits = lambda x: np.array([x], dtype=np.float16).view(np.uint16)[0]
    q, k, v = (np.zeros((1, h, n, 128), dtype=np.uint16) for h, n in ((4, 2), (1, nk), (1, nk)))
    q[..., 0], k[:, :, 0, 0] = bits(1.0), bits(1.0)
    v[:, :, 1:128] = bits(32.0)  # (the keys of the sink's own wave)
    out, lse = binding.swaa_attn_fwd_ex(to_device(q, "fp16"), to_device(k, "fp16"), to_device(v, "fp16"), 10**9, 4, scale=nats)
    torch.cuda.synchronize()
    assert scratch[0] > 0
    with input_format("fp16"):
        ro, rl = swaa_decode_oracle(q, k, v, 10**9, 4, nats)
    p = 16 * math.exp(-nats)
    bound = max(2.0**-25 / p, 2.0**-11) + 2.0**-10
    rel = np.abs(out.float().cpu().numpy() / ro - 1).max()
    print(f"[few rows, sink] {nk} keys, {nats} nats: {rel:.2e} of at most {bound:.2e}", flush=True)
    assert rel <= bound
    assert np.abs(lse.cpu().numpy() - rl).max() <= 1e-3


@pytest.mark.parametrize("fmt", ["bf16", "fp16"])
@pytest.mark.parametrize("nk,at", [(1100, 40), (1100, 300), (1100, 600), (1100, 1060), (5000, 40), (5000, 300), (5000, 2600), (5000, 4990)])
def test_few_rows_with_references_far_apart(scratch, nk, at, fmt):
    # One key 40 nats above the rest, in each of the four waves' quarters of whole keys, in some split and in the last:
    # the others' results have to vanish beside that wave's.
    q, k, v = make_qkv(1, 8, 2, nk, 128, seed=9700 + at, n_query=2, fmt=fmt)
    bits = lambda x: np.array([x], dtype=np.float16).view(np.uint16)[0] if fmt == "fp16" else np.array([x], dtype=np.float32).view(np.uint32)[0] >> 16
    q[..., 0], k[..., 0] = bits(3.0), bits(0.0)
    k[:, :, at, 0] = bits(152.0)
    out, lse = binding.swaa_attn_fwd_ex(to_device(q, fmt), to_device(k, fmt), to_device(v, fmt), 10**9, 4)
    torch.cuda.synchronize()
    assert scratch[0] > 0
    with input_format(fmt):
        ro, rl = swaa_decode_oracle(q, k, v, 10**9, 4, 1 / math.sqrt(128))
    assert_parity(out, lse, ro, rl, tag=f"few rows, {nk} keys, spike at {at} {fmt}")


@pytest.mark.parametrize("fmt", ["bf16", "fp16"])
@pytest.mark.parametrize("what", ["nan", "inf"])
@pytest.mark.parametrize("nk", [1100, 5000])
def test_few_rows_and_what_is_not_a_number(scratch, nk, what, fmt):
    bits = {("nan", "bf16"): 0x7FC0, ("inf", "bf16"): 0x7F80, ("nan", "fp16"): 0x7E00, ("inf", "fp16"): 0x7C00}[what, fmt]
    q, k, v = make_qkv(1, 8, 2, nk, 128, seed=9710, n_query=3, fmt=fmt)
    q[..., 5] = {"bf16": 0x3F80, "fp16": 0x3C00}[fmt]  # 1: the score of an infinite component is +infinity
    run = lambda q, k: tuple(t.clone() for t in binding.swaa_attn_fwd_ex(to_device(q, fmt), to_device(k, fmt), to_device(v, fmt), 10**9, 4))
    want, want_l = run(q, k)
    # a query row that is not a number: it alone, its neighbours in the column tile bit for bit as without it
    bad = q.copy()
    bad[:, 6, 1, 5] = np.uint16(bits)
    out, lse = run(bad, k)
    torch.cuda.synchronize()
    assert scratch[0] > 0
    assert not torch.isfinite(out[0, 6, 1].float()).any() and not torch.isfinite(lse[0, 6, 1])
    out[0, 6, 1], lse[0, 6, 1] = want[0, 6, 1], want_l[0, 6, 1]
    assert torch.equal(out, want) and torch.equal(lse, want_l)
    # a key, in every wave's quarter and in other splits: all rows of its head, and the other head's as before
    for at in [40, 300, 560, 840, 1060, 2600, 4900]:
        if at < nk:
            bad = k.copy()
            bad[:, 1, at, 5] = np.uint16(bits)
            out, lse = run(q, bad)
            torch.cuda.synchronize()
            assert not torch.isfinite(out[0, 4:].float()).any() and not torch.isfinite(lse[0, 4:]).any(), at
            assert torch.equal(out[0, :4], want[0, :4]) and torch.equal(lse[0, :4], want_l[0, :4]), at
    # the newest key: only the row that sees it
    bad = k.copy()
    bad[:, 1, nk - 1, 5] = np.uint16(bits)
    out, lse = run(q, bad)
    torch.cuda.synchronize()
    assert not torch.isfinite(out[0, 4:, 2].float()).any() and not torch.isfinite(lse[0, 4:, 2]).any()
    assert torch.equal(out[0, :, :2], want[0, :, :2]) and torch.equal(lse[0, :, :2], want_l[0, :, :2])


@pytest.mark.parametrize("nq,nk,max_q,max_k,W,prompt", [
    (70, 4000, 70, 4000, 10**9, 3000),    # as long as the host says: its plan; generated rows
    (70, 2100, 128, 6000, 10**9, None),   # shorter: the device's
    (5, 300, 128, 6000, 10**9, None),     # ... few rows, fewer halves than the host's splits
    (40, 4000, 70, 4000, 500, 3980),      # prompt and generated rows behind a window: planned on the device, whole
])
def test_one_packed_sequence(scratch, nq, nk, max_q, max_k, W, prompt):
    Hkv, G, D = 2, 4, 128
    print(f"[case] packed alone nq {nq} nk {nk} of {max_q} {max_k} W {W}", flush=True)
    q, k, v = make_qkv(1, Hkv * G, Hkv, nk, D, seed=9750 + nq, n_query=nq)
    ints = lambda *x: torch.tensor(x, dtype=torch.int32, device="cuda")
    out, lse = binding.swaa_attn_fwd_ex(*(to_device(x[0]) for x in (q, k, v)), W, 4, cu_seqlens_q=ints(0, nq), cu_seqlens_k=ints(0, nk),
                                        max_seqlen_q=max_q, max_seqlen_k=max_k, n_prompts=None if prompt is None else ints(prompt))
    torch.cuda.synchronize()
    assert scratch[0] > 0
    ro, rl = swaa_decode_oracle(q, k, v, min(W, nk), 4, 1 / math.sqrt(D), n_prompt=prompt)
    assert_parity(out[None], lse[None], ro, rl, tag=f"packed alone {nq} of {nk}")


@pytest.mark.parametrize("nq,nk,max_q,max_k,as_bounded", [
    (64, 1000, 64, 32768, False),    # a cache far shorter than its bound
    (3, 600, 3, 32768, False),       # ... few rows
    (64, 20000, 512, 32768, False),  # fewer rows than their bound: more splits, not fewer
    (64, 7648, 64, 8192, False),     # 239 halves of 256
    (64, 7680, 64, 8192, True),      # 240: the host's plan
])
def test_one_packed_sequence_is_split_for_the_length_it_has(monkeypatch, nq, nk, max_q, max_k, as_bounded):
    Hkv, G = 8, 4
    lib, scratch = binding.load_library(), []
    query = lib.swaa_attn_fwd_ex_workspace_bytes
    monkeypatch.setattr(lib, "swaa_attn_fwd_ex_workspace_bytes", lambda a: scratch.append(int(query(a))) or scratch[-1])
    q, k, v = (to_device(x[0]) for x in make_qkv(1, Hkv * G, Hkv, max_k, 128, seed=9800 + nk, n_query=max_q))
    ints = lambda *x: torch.tensor(x, dtype=torch.int32, device="cuda")

    def run(nq, nk, batch):  # the call, and the splits that its plan (the workspace's last 64 ints) gave the sequence
        print(f"[case] nq {nq} of {max_q} nk {nk} of {max_k}, batch of {batch}", flush=True)
        cu = lambda n: ints(0, *[n] * batch)
        ws = torch.zeros(160 << 20, dtype=torch.uint8, device="cuda")
        out, lse = binding.swaa_attn_fwd_ex(q[:, :nq], k[:, :nk], v[:, :nk], 10**9, 4, workspace=ws, cu_seqlens_q=cu(nq),
                                            cu_seqlens_k=cu(nk), max_seqlen_q=max_q, max_seqlen_k=max_k)
        torch.cuda.synchronize()
        end = scratch.pop()
        assert end > 0
        return out, lse, int(ws[end - 256:end - 252].view(torch.int32)[0])

    out, lse, n = run(nq, nk, 1)
    if as_bounded:
        assert n == run(nq, max_k, 1)[2]
        return
    # beside an empty sequence the device always plans for itself
    want, want_l, n2 = run(nq, nk, 2)
    assert n == n2
    assert torch.equal(out, want) and torch.equal(lse, want_l)


@pytest.mark.parametrize("Hkv,G,nq,nk,W,whole", [
    (8, 4, 512, 4000, 1500, True),   # 128 units: whole up to windows of about 2200
    (8, 4, 512, 4000, 2048, True),
    (4, 4, 1000, 4000, 1250, True),
    (8, 4, 512, 4000, 3000, False),  # split, and as many times
    (8, 4, 64, 4000, 2048, False),
])
def test_one_chunk_gives_the_same_bits_whichever_list_it_runs_on(scratch, Hkv, G, nq, nk, W, whole):
    print(f"[case] one chunk {nq} on {nk} W{W}", flush=True)
    q, k, v = make_qkv(1, Hkv * G, Hkv, nk, 128, seed=95500 + nq + W, n_query=nq)
    ints = lambda *x: torch.tensor(x, dtype=torch.int32, device="cuda")
    (out, lse), (o0, l0) = (tuple(t.clone() for t in binding.swaa_attn_fwd_ex(
        *(to_device(x[0]) for x in (q, k, v)), W, 4, total_rows_q=rows, cu_seqlens_q=ints(0, nq), cu_seqlens_k=ints(0, nk),
        max_seqlen_q=nq, max_seqlen_k=nk)) for rows in (None, 0))
    torch.cuda.synchronize()
    assert (scratch[0] == 0) == whole and scratch[1] > 0
    assert torch.equal(out, o0) and torch.equal(lse, l0)
    ro, rl = swaa_decode_oracle(q, k, v, W, 4, 1 / math.sqrt(128))
    assert_parity(out[None], lse[None], ro, rl, tag=f"one chunk {nq} on {nk}")
