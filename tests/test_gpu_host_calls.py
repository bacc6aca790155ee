"""The native way to the library (csrc/host_calls.cpp) against the binding's general one: the same results, bit for bit and
stride for stride, over the forms of call that it takes, and the same refusals."""
import types

import pytest
import torch

from paper_2512_10411_amd import binding
from paper_2512_10411_amd.inputs import make_qkv
from gpu_util import to_device

pytestmark = pytest.mark.gpu


class Counting:
    """The native part, counting the calls that it took."""

    def __init__(self, real):
        self.real, self.taken = real, 0

    def __getattr__(self, name):
        def call(*args):
            r = getattr(self.real, name)(*args)
            self.taken += r is not None
            return r
        return call


NOTHING = types.SimpleNamespace(**{n: lambda *args: None for n in ("fwd", "decode", "decode_ex", "fill_fwd_ex")})


def both(monkeypatch, f):
    binding._torch()
    counting = Counting(binding._host)
    outcome = []
    for host in (counting, NOTHING):
        with monkeypatch.context() as m:
            m.setattr(binding, "_host", host)
            try:
                outcome.append(f())
            except Exception as e:  # noqa: BLE001 (what is refused has to be refused alike)
                outcome.append((type(e), str(e)))
    torch.cuda.synchronize()
    return outcome[0], outcome[1], counting.taken


def calls():
    q, k, v = (to_device(x) for x in make_qkv(2, 4, 2, 300, 128, seed=9900))
    new, one = q[:, :, -2:].contiguous(), q[:, :, -1:]
    cu = torch.tensor([0, 200, 300], dtype=torch.int32, device="cuda")
    lens = torch.tensor([300, 77], dtype=torch.int32, device="cuda")
    pages = torch.randn(40, 2, 16, 128, device="cuda").half()
    table = torch.randperm(40, device="cuda").to(torch.int32)[:38].reshape(2, 19)
    packed = [t[0] for t in (q, k, v)]
    rows = [t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for t in (q, k, v)]  # [B, N, H, D] in memory
    b = binding
    ws = torch.empty(1 << 24, dtype=torch.uint8, device="cuda")
    return {  # name: (call, taken by the native way)
        "fwd": (lambda: b.swaa_attn_fwd(q, k, v, 100, 4), 1),
        "fwd, scale": (lambda: b.swaa_attn_fwd(q, k, v, 100, 4, 0.2), 1),
        "fwd, one row": (lambda: b.swaa_attn_fwd(one.contiguous(), k[:, :, -1:].contiguous(), v[:, :, -1:].contiguous(), 100, 4), 1),
        "fwd, gradients": (lambda: b.swaa_attn_fwd(q.clone().requires_grad_(), k, v, 100, 4), 1),
        "fwd_fa_decode": (lambda: b.swaa_attn_fwd_fa_decode(q, k, v, 100, 4, 250), 1),
        "decode": (lambda: b.swaa_attn_decode(new, k, v, 100, 4), 1),
        "decode, workspace": (lambda: b.swaa_attn_decode(new, k, v, 300, 0, workspace=ws), 1),
        "decode_ex": (lambda: b.swaa_attn_decode_ex(new, rows[1], rows[2], 100, 4, seq_lens=lens), 1),
        "decode_ex, paged": (lambda: b.swaa_attn_decode_ex(new.half(), pages, pages, 100, 4, seq_lens=lens, block_table=table,
                                                           max_seqlen_k=300, workspace=ws), 1),
        "fwd_ex": (lambda: b.swaa_attn_fwd_ex(*rows, 100, 4, n_prompt=250), 1),
        "fwd_ex, chunk": (lambda: b.swaa_attn_fwd_ex(new, k, v, 1000, 4, n_prompts=lens), 1),
        "fwd_ex, packed": (lambda: b.swaa_attn_fwd_ex(*packed, 100, 4, cu_seqlens_q=cu, cu_seqlens_k=cu, max_seqlen_q=200,
                                                      max_seqlen_k=200, total_rows_q=300), 1),
        "fwd_ex, paged": (lambda: b.swaa_attn_fwd_ex(packed[0].half(), pages, pages, 100, 4, cu_seqlens_q=cu, cu_seqlens_k=cu,
                                                     max_seqlen_q=200, max_seqlen_k=200, block_table=table), 1),
        # other forms, and what is refused
        "results given": (lambda: b.swaa_attn_fwd(q, k, v, 100, 4, out=torch.empty_like(q)), 0),
        "a subclass": (lambda: b.swaa_attn_fwd(q.as_subclass(type("T", (torch.Tensor,), {})), k, v, 100, 4)[0].as_subclass(torch.Tensor), 0),
        "a number that is no int": (lambda: b.swaa_attn_fwd(q, k, v, 100.0, 4), 0),
        "not contiguous": (lambda: b.swaa_attn_fwd(rows[0], k, v, 100, 4), 0),
        "binary16": (lambda: b.swaa_attn_fwd(q.half(), k, v, 100, 4), 0),
        "on the CPU": (lambda: b.swaa_attn_decode(new.cpu(), k, v, 100, 4), 0),
        "k of another length": (lambda: b.swaa_attn_fwd(q, k[:, :, 1:].contiguous(), v, 100, 4), 0),
        "no window": (lambda: b.swaa_attn_fwd(q, k, v, 0, 4), 1),
        "scale": (lambda: b.swaa_attn_fwd(q, k, v, 5, 4, -1.0), 1),
        "little workspace": (lambda: b.swaa_attn_decode(new, k, v, 300, 0, workspace=ws[:16]), 1),
        "workspace of floats": (lambda: b.swaa_attn_decode(new, k, v, 300, 0, workspace=ws.view(torch.float32)), 0),
        "paged without a length": (lambda: b.swaa_attn_decode_ex(new, k, v, 100, 4, block_table=table), 0),
        "lengths of int64": (lambda: b.swaa_attn_decode_ex(new, k, v, 100, 4, seq_lens=lens.long()), 0),
        "no sinks below zero": (lambda: b.swaa_attn_fwd_ex(q, k, v, 100, -1), 1),
        "offsets without lengths": (lambda: b.swaa_attn_fwd_ex(*packed, 100, 4, cu_seqlens_q=cu, cu_seqlens_k=cu), 0),
        "prompts of another batch": (lambda: b.swaa_attn_fwd_ex(q, k, v, 100, 4, n_prompts=cu), 0),
    }


@pytest.mark.parametrize("mode", ["plain", "inference", "device context", "autocast"])
def test_native_and_general_calls_agree(monkeypatch, mode):
    for name, (f, taken) in calls().items():
        print(f"[case] {mode}: {name}", flush=True)
        modes = {"plain": torch.enable_grad, "inference": torch.inference_mode, "device context": lambda: torch.device("cuda"),
                 "autocast": lambda: torch.autocast("cuda", torch.float16)}
        with modes[mode]():
            native, general, n = both(monkeypatch, f)
        assert n == (0 if mode == "device context" else taken), name
        if isinstance(general, torch.Tensor):
            native, general = (native,), (general,)
        for x, y in zip(native, general):
            if isinstance(y, torch.Tensor):
                assert x.dtype == y.dtype and x.stride() == y.stride() and x.requires_grad == y.requires_grad, name
                assert torch.equal(x, y), name
            else:
                assert x == y, name
