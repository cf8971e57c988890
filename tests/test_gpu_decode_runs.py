"""Decode attention dealt to the wavefronts in runs of equal length over all requests and kv heads: run lengths from the
shortest to several requests per run, requests in many runs, more requests than one scan places, more spans in a run
than the wavefront stages, and the batch whose outputs are not merged, for every head ratio and both head dimensions,
with contexts on both sides of the 32-key pairs and of the spans: sampled requests of each batch (those on both sides of
a lane's four and of a scan's 256 among them) against the oracle, at the parity bar of the other cases."""
import numpy as np
import pytest
import torch

from paper_2507_06608_amd import synth

from tests.parity_util import assert_close, f32, run_oracle
from tests.test_gpu_parity import EXTRA_SHAPES

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


SHAPES = dict(EXTRA_SHAPES, tiny=synth.SHAPES["tiny"])  # kv heads: tiny 8, gqa8 1, the others 2
# (requests, contexts that are always there, largest other context, shape)
CASES = [
    ("whole contexts, no merge", 5, [0, 15, 16, 254, 255], 255, "tiny"),
    ("shortest runs", 3, [63, 64, 65], 700, "tiny"),
    ("one long request", 1, [8191], 8191, "tiny"),
    ("runs of two pairs", 16, [31, 32, 33, 127, 128, 129], 1000, "tiny"),
    ("page ids of several fetches", 24, [1022, 1023, 1024, 1055, 1056, 8190], 8191, "tiny"),
    ("several requests a run", 300, [0, 31, 32, 1023, 1024, 2047, 2048], 2060, "tiny"),
    ("more requests than one scan", 600, [1022, 1023, 1024, 1025, 0], 1100, "tiny"),
    ("head dimension 128, G 4", 33, [0, 31, 32, 255, 256, 1023, 1024, 4095, 4096], 4200, "gqa4"),
    ("head dimension 128, G 5", 20, [0, 31, 32, 255, 256, 1023, 1024, 4095, 4096], 4200, "gqa5"),
    ("head dimension 128, G 8", 9, [0, 31, 32, 255, 256, 1023, 1024, 4095, 4096], 4200, "gqa8"),
    ("head dimension 64, G 2", 70, [0, 31, 32, 255, 256, 511, 512, 4095, 4096], 4200, "gqa2"),
    ("more spans a run than staged, G 4", 700, [4090, 0, 255, 256, 511, 512], 4095, "gqa4"),
    ("more spans a run than staged, G 5", 600, [4090, 0, 255, 256, 511, 512], 4095, "gqa5"),
    ("more spans a run than staged, G 8", 700, [4090, 0, 255, 256, 511, 512], 4095, "gqa8"),
]


@pytest.mark.parametrize("name,n,edges,top,shape", CASES, ids=[c[0] for c in CASES])
def test_equal_runs(nx, oracle, name, n, edges, top, shape):
    print(f"[case] decode attention, {name}", flush=True)
    sh = SHAPES[shape]
    rng = np.random.default_rng(n)
    low = 3600 if "staged" in name else 0  # long contexts throughout: runs of more spans of 256 keys than 20 KB hold
    ctx_lens = edges + rng.integers(low, top + 1, n - len(edges)).tolist()
    wl = synth.make_workload(name, sh, 5, chunk_lens=[], prefix_lens=[], decode_ctx=ctx_lens, kv_device="cuda:0")
    w = synth.make_weights(sh, 5)
    ctx = nx.context_for(wl)
    ctx.load_layer(0, w)
    kv = ctx.make_kv(wl.k_pool, wl.v_pool)
    db = nx.DevDecode(wl.decode, ctx.device)
    torch.cuda.synchronize()
    ctx.decode_step(db, kv)
    ctx.sync()
    sampled = sorted(set(range(len(edges))) | {j for j in (3, 4, 255, 256, 511, 512, n // 2, n - 1) if j < n})
    sub = synth.subset_for_oracle(wl, [], sampled)
    ref = run_oracle(oracle, sub, w)
    assert_close(name, f32(db.y[sampled]), ref["y_d"])
    assert torch.isfinite(db.y.float()).all()
    ctx.close()
