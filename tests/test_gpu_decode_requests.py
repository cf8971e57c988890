"""What a decode request's output depends on: its own context, and neither how tight the batch's context hint is nor which
requests share the batch with it.  All comparisons are bit for bit between two decode steps of the library."""
import numpy as np
import pytest
import torch

from paper_2507_06608_amd import synth

from tests.test_gpu_parity import EXTRA_SHAPES

pytestmark = pytest.mark.gpu

SHAPES = dict(EXTRA_SHAPES, tiny=synth.SHAPES["tiny"])


@pytest.fixture(scope="module")
def nx():
    from paper_2507_06608_amd import binding
    binding.lib()
    return binding


class Batch:
    """Decode requests with the given contexts; `run` makes one step of some of them (in the given order) on fresh pools."""

    def __init__(self, nx, shape, ctx_lens, seed=9):
        sh = SHAPES[shape]
        self.nx, self.lens = nx, np.asarray(ctx_lens, np.int32)
        self.wl = synth.make_workload("requests", sh, seed, chunk_lens=[], prefix_lens=[], decode_ctx=ctx_lens, kv_device="cuda:0")
        self.ctx = nx.context_for(self.wl)
        self.ctx.load_layer(0, synth.make_weights(sh, seed))

    def run(self, order=None, lens=None, hint=None):
        d = self.wl.decode
        order = list(range(d.n_reqs)) if order is None else order
        lens = self.lens if lens is None else np.asarray(lens, np.int32)
        db = self.nx.DevDecode(synth.DecodeBatch(d.x[order], lens[order], d.page_table[order]), self.ctx.device)
        if hint is not None:
            db.c.max_ctx = hint
        db.y.fill_(float("nan"))
        kv = self.ctx.make_kv(self.wl.k_pool, self.wl.v_pool)
        torch.cuda.synchronize()
        self.ctx.decode_step(db, kv)
        self.ctx.sync()
        assert torch.isfinite(db.y.float()).all()
        return db.y.view(torch.int16).clone()


@pytest.mark.parametrize("lens", [[300, 40, 299], [254, 200, 31], [767, 511, 700, 32]], ids=["301 keys", "255 keys", "768 keys"])
def test_a_hint_one_short_keeps_the_newest_key(nx, lens):
    """The scheduler's batch states the largest context without the new token, one less than a step's hint.  Up to the next
    multiple of 256 a step has always attended to every key of a context that passes its hint, and still does."""
    print(f"[case] hint one short, {lens}", flush=True)
    b = Batch(nx, "gqa4", lens)
    assert torch.equal(b.run(hint=max(lens)), b.run(hint=max(lens) + 1))
    b.ctx.close()


# contexts around the 32-key pairs and 256 keys, short and long next to one another
LENS = [0, 15, 31, 32, 254, 255, 256, 257, 511, 512, 700, 1023, 1024, 1025, 1500, 2047, 2048, 2100, 3000, 4095, 4096, 4200]


@pytest.mark.parametrize("shape,n", [("tiny", 22), ("gqa2", 33), ("gqa4", 32), ("gqa5", 64), ("gqa8", 65), ("gqa4", 300)],
                         ids=["hd 64 G 1, 22", "G 2, 33", "G 4, 32", "G 5, 64", "G 8, 65", "G 4, 300"])
def test_a_request_does_not_depend_on_its_neighbours(nx, shape, n):
    """The same requests next to others with other contexts, in another order and under a looser hint: the rows of the
    requests that stayed the same keep their bits."""
    print(f"[case] decode neighbours, {shape} {n} requests", flush=True)
    rng = np.random.default_rng(n)
    lens = (LENS + rng.integers(0, 3000, max(0, n - len(LENS))).tolist())[:n]
    b = Batch(nx, shape, lens)
    ref = b.run()
    kept = [j for j in range(n) if j % 3 != 1]
    other = np.asarray(lens, np.int32).copy()
    for j in range(1, n, 3):
        other[j] = rng.integers(0, lens[j] + 1)
    y = b.run(lens=other)
    assert torch.equal(y[kept], ref[kept]), "other contexts next to it"
    order = rng.permutation(n).tolist()
    assert torch.equal(b.run(order=order), ref[order]), "another order"
    short = [j for j in range(n) if lens[j] < 256]
    assert torch.equal(b.run(order=short), b.run(order=short, hint=max(lens) + 1)), "a looser hint"
    b.ctx.close()


def test_a_hint_one_short_in_a_fused_batch(nx):
    """The same for decode requests riding in a chunked-prefill batch."""
    print("[case] hint one short, fused batch", flush=True)
    sh = SHAPES["gqa4"]
    wl = synth.make_workload("fused", sh, 9, chunk_lens=[40], prefix_lens=[5], decode_ctx=[300, 40], kv_device="cuda:0")
    ctx = nx.Nexus(sh, max_prefill_tokens=42, max_prefill_reqs=3, max_decode_reqs=2, max_positions=301)
    ctx.load_layer(0, synth.make_weights(sh, 9))
    ys = []
    for hint in (300, 301):
        pb = nx.DevPrefill(synth.fused_single_batch(wl), ctx.device)
        kv = ctx.make_kv(wl.k_pool, wl.v_pool)
        torch.cuda.synchronize()
        ctx.fused_step(pb, 2, hint, kv)
        ctx.sync()
        assert torch.isfinite(pb.y.float()).all()
        ys.append(pb.y.view(torch.int16).clone())
    assert torch.equal(*ys)
    ctx.close()
