"""Decode attention at every span length the batch size selects (64 .. 1024 keys per work item, and the single span whose
output is not merged), with contexts on both sides of the span boundaries: sampled requests of each batch against the
oracle, at the parity bar of the other cases."""
import numpy as np
import pytest
import torch

from paper_2507_06608_amd import synth

from tests.parity_util import assert_close, f32, run_oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nx():
    from paper_2507_06608_amd import binding
    binding.lib()
    return binding


@pytest.fixture(scope="module")
def oracle():
    import oracle
    oracle.lib()
    return oracle


# (requests, contexts that are always there, largest other context): 8 kv heads each
CASES = [
    ("one span of 256, no merge", 5, [0, 15, 16, 254, 255], 255),
    ("spans of 64", 3, [63, 64, 65], 700),
    ("spans of 128", 16, [127, 128, 129, 255, 256, 257], 1000),
    ("spans of 256", 40, [255, 256, 257, 511, 512], 1500),
    ("spans of 512", 300, [511, 512, 513, 1023, 1024, 1025, 2047, 2048], 2060),
    ("spans of 1024", 600, [1022, 1023, 1024, 1025, 0], 1100),
]


@pytest.mark.parametrize("name,n,edges,top", CASES, ids=[c[0] for c in CASES])
def test_every_span_length(nx, oracle, name, n, edges, top):
    print(f"[case] decode attention, {name}", flush=True)
    sh = synth.SHAPES["tiny"]
    rng = np.random.default_rng(n)
    ctx_lens = edges + rng.integers(0, top + 1, n - len(edges)).tolist()
    wl = synth.make_workload(name, sh, 5, chunk_lens=[], prefix_lens=[], decode_ctx=ctx_lens, kv_device="cuda:0")
    w = synth.make_weights(sh, 5)
    ctx = nx.context_for(wl)
    ctx.load_layer(0, w)
    kv = ctx.make_kv(wl.k_pool, wl.v_pool)
    db = nx.DevDecode(wl.decode, ctx.device)
    torch.cuda.synchronize()
    ctx.decode_step(db, kv)
    ctx.sync()
    sampled = list(range(len(edges))) + [n - 1] if n > len(edges) else list(range(n))
    sub = synth.subset_for_oracle(wl, [], sampled)
    ref = run_oracle(oracle, sub, w)
    assert_close(name, f32(db.y[sampled]), ref["y_d"])
    assert torch.isfinite(db.y.float()).all()
    ctx.close()
