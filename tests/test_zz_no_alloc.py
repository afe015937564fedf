"""graphkv_compress_static (the entry point for callers that cannot allocate) against
graphkv_compress, through the C ABI: same bytes, on two calls in a row that share the built-in
scratch buffer, the second on a smaller input."""
import numpy as np
import pytest
import torch

from paper_2509_00388_amd import binding as gk
from paper_2509_00388_amd import synth
from tests import util

pytestmark = pytest.mark.gpu


def outputs(p):
    shape = (p.n_kv_heads, p.budget, p.head_dim)
    return (torch.zeros(shape, dtype=p.torch_dtype, device="cuda"), torch.zeros(shape, dtype=p.torch_dtype, device="cuda"),
            torch.zeros((p.n_kv_heads, p.budget), dtype=torch.int32, device="cuda"),
            torch.zeros((p.n_kv_heads, p.n_prefix), dtype=torch.float32, device="cuda"))


def test_static_scratch_entry_equals_workspace_entry():
    c2 = synth.CONFIGS["c2"]
    cases = [(synth.scaled(c2, n_tokens=9100, n_sources=40, n_neighbors=12, budget=700, n_kv_heads=2, n_q_heads=8),
              dict(rounds=3)),                                                    # filter route, lists kept
             (synth.scaled(c2, n_tokens=1500, budget=200, n_sources=16, n_neighbors=8, n_kv_heads=2, n_q_heads=8),
              dict(rounds=2)),                                                    # smaller: dense route
             (synth.scaled(c2, n_tokens=700, budget=90, n_sources=5, n_neighbors=3, n_kv_heads=1, n_q_heads=4),
              dict(rounds=1, scorer=gk.SCORER_KNORM))]
    prepared = []
    for cfg, kw in cases:
        host, dev = util.device_layer(cfg, 1)
        p = util.params_from_cfg(cfg, **kw)
        assert 0 < gk.graphkv_workspace_bytes(p) <= gk.STATIC_SCRATCH_BYTES
        want = outputs(p)
        gk.graphkv_compress(p, *dev, want[0], want[1], want[2], scores_out=want[3])
        prepared.append((p, dev, want, outputs(p)))
    torch.cuda.synchronize()
    # the calls under test, back to back on the one built-in buffer, no allocation in between
    for p, dev, want, got in prepared:
        print(f"static-scratch call N={p.n_tokens}", flush=True)
        gk.graphkv_compress_static(p, *dev, got[0], got[1], got[2], scores_out=got[3])
    torch.cuda.synchronize()
    for p, dev, want, got in prepared:
        assert torch.equal(got[2], want[2]), f"N={p.n_tokens}: indices"
        assert torch.equal(got[0].view(torch.int16), want[0].view(torch.int16)), "gathered keys"
        assert torch.equal(got[1].view(torch.int16), want[1].view(torch.int16)), "gathered values"
        assert np.array_equal(got[3].cpu().numpy(), want[3].cpu().numpy(), equal_nan=True), "refined scores"
        assert int(got[2].max()) == p.n_tokens - 1


def test_static_scratch_entry_rejects_what_does_not_fit():
    cfg = synth.CONFIGS["c5"]
    p = util.params_from_cfg(cfg)
    assert gk.graphkv_workspace_bytes(p) > gk.STATIC_SCRATCH_BYTES
    cfg_s = synth.scaled(synth.CONFIGS["c2"], n_tokens=700, budget=90, n_kv_heads=1, n_q_heads=4)
    host, dev = util.device_layer(cfg_s, 0)
    o = outputs(util.params_from_cfg(cfg_s))
    with pytest.raises(gk.GraphKVError, match="-4"):
        # (buffers of the small problem, params of the large one: the size check comes first)
        lib = gk.load_library()
        import ctypes
        cp = p.c()
        gk._check(lib.graphkv_compress_static(ctypes.byref(cp), dev[0].data_ptr(), dev[1].data_ptr(), dev[2].data_ptr(),
                                              o[0].data_ptr(), o[1].data_ptr(), o[2].data_ptr(), None, None))


def test_static_scratch_entry_falls_back_to_the_dense_block():
    """512 heads of a 2K prompt with 8 sources: the filter route's per-row buffers (with speculative rows)
    would not fit the built-in buffer, the dense edge block does.  Same bytes as the workspace entry, which
    takes the filter route."""
    cfg = synth.scaled(synth.CONFIGS["c2"], n_tokens=2100, window=32, n_sources=8, n_neighbors=32, budget=200,
                       n_kv_heads=8, n_q_heads=8, rounds=2)
    host, dev = util.device_layer(cfg, 1)
    rep = 64
    dev = [t.repeat(rep, 1, 1).contiguous() for t in dev]
    p = util.params_from_cfg(synth.scaled(cfg, n_kv_heads=8 * rep, n_q_heads=8 * rep), scorer=gk.SCORER_KNORM)
    assert gk.graphkv_workspace_bytes(p) > gk.STATIC_SCRATCH_BYTES
    want, got = outputs(p), outputs(p)
    print("static-scratch call with 512 heads", flush=True)
    gk.graphkv_compress(p, *dev, want[0], want[1], want[2], scores_out=want[3])
    gk.graphkv_compress_static(p, *dev, got[0], got[1], got[2], scores_out=got[3])
    torch.cuda.synchronize()
    assert torch.equal(got[2], want[2]) and torch.equal(got[3], want[3])
    assert torch.equal(got[0].view(torch.int16), want[0].view(torch.int16))


@pytest.mark.parametrize("H,G,w,P,pool", [(8, 1, 128, 15892, 7), (2, 4, 128, 16056, 7), (1, 4, 181, 22640, 7), (4, 2, 64, 31500, 131)])
def test_static_scratch_entry_with_logits_that_nearly_fill_it(H, G, w, P, pool):
    """fp32 logits of 61 to 63 MiB: what the row statistics need beside them must not push the call to kernels
    that add up in another order.  Same bytes as the workspace entry."""
    p = gk.Params(n_kv_heads=H, n_q_heads=H * G, head_dim=64, n_tokens=P + w, window=w, pool_kernel=pool, budget=w + 500,
                  n_sources=8, n_neighbors=8, rounds=1, dtype=gk.FP32)
    assert 4 * H * G * w * P > 60 << 20
    g = torch.Generator("cuda").manual_seed(P)
    dev = [torch.randn(h, n, 64, generator=g, device="cuda") for h, n in ((H, P + w), (H, P + w), (H * G, w))]
    print(f"static-scratch call H={H} G={G} w={w} P={P}", flush=True)

    def outs():
        return [torch.empty(H, p.budget, 64, device="cuda"), torch.empty(H, p.budget, 64, device="cuda"),
                torch.empty(H, p.budget, dtype=torch.int32, device="cuda"), torch.empty(H, P, device="cuda")]

    want, got = outs(), outs()
    gk.graphkv_compress(p, *dev, want[0], want[1], want[2], scores_out=want[3])
    gk.graphkv_compress_static(p, *dev, got[0], got[1], got[2], scores_out=got[3])
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a, b)
