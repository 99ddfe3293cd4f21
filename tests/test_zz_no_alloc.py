"""stand_verify_static (the verification entry point that allocates nothing: its scratch is a fixed
array in the library's device image) against stand_verify, through the C ABI: tokens, nodes and lengths
bit for bit, on calls in a row that share the array -- a larger shape, then a smaller one, then the
larger one again -- so stale contents of the array must not matter."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2506_04708_amd import synth  # noqa: E402


class _Run:
    """A handle driven in a closed loop on a small vocabulary (drafts are accepted often), with a filled table
    and a pending draft after `steps` speculation steps."""

    def __init__(self, binding, lockstep, name, over, steps):
        self.lockstep = lockstep
        self.w = w = synth.Workload(name, run_steps=steps + 16, **over)
        dt = binding.STAND_F32 if w.dtype == "f32" else binding.STAND_BF16
        self.g = binding.Stand(w.V, w.B, w.cfg["order_min"], w.cfg["order_max"], w.K, w.parent, w.T, 1 << 14, 64, 77, dt)
        for b in range(w.B):
            self.g.set_context(b, w.prompt(b))
        self.out = self.g.new_outputs()
        self.g.draft(0, self.out[3])
        self.step = 0
        for _ in range(steps):
            self.advance()

    def logits(self):
        return self.lockstep._logits_to_device(self.w.logits(self.step, self.out[3].cpu().numpy()), self.w.dtype)

    def advance(self):
        # closed loop: what the verification emits is committed
        out_tok, out_node, out_len, d = self.out
        self.g.step(self.step, self.logits(), out_tok, out_node, out_len, d)
        self.step += 1


def _both(g, step, lg):
    ref = g.new_outputs()[:3]
    got = [torch.full_like(t, -7) for t in ref]
    g.verify(step, lg, *ref)
    torch.cuda.synchronize()
    g.verify_static(step, lg, *got)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in ref], [t.cpu().numpy() for t in got]


def test_verify_static_matches_verify_on_calls_that_share_the_scratch():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2506_04708_amd import binding
    from tests import lockstep
    print("no-alloc verify: large shape (cfg3 tree: 64 nodes, K=16, B=8, V=203, bf16, misaligned rows)", flush=True)
    big = _Run(binding, lockstep, "cfg3", dict(V=203, B=8, rho=0.5), 10)
    print("no-alloc verify: small shape (cfg1 tree: 16 nodes, K=10, B=3, V=40, f32)", flush=True)
    small = _Run(binding, lockstep, "cfg1", dict(V=40, B=3, rho=0.5), 10)
    accepted = 0
    for rep in range(8):
        # the larger shape, then the smaller one, in a row on the same array; then both move on one step
        for run in (big, small):
            assert 0 < run.g.static_scratch_need() <= 8 << 20
            ref, got = _both(run.g, run.step, run.logits())
            for r, x, what in zip(ref, got, ("tokens", "nodes", "lengths")):
                assert np.array_equal(r, x), "%s differ: %s vs %s" % (what, x, r)
            assert (ref[2] >= 1).all() and (ref[0][:, 0] >= 0).all()
            accepted += int((ref[2] > 1).sum())
        big.advance()
        small.advance()
    print("no-alloc verify: %d trajectories with accepted drafts among the compared calls" % accepted, flush=True)
    assert accepted >= 8, "too few accepted drafts: the comparison hardly reached the accept tests"
    # a shape whose scratch does not fit the array is refused, and nothing is written
    wide = synth.Workload("cfg5", run_steps=1, V=64)
    g2 = binding.Stand(64, 160, 1, 5, 32, wide.parent, 0.8, 1 << 10, 8, 1, binding.STAND_BF16)
    assert g2.static_scratch_need() > 8 << 20
    outs = [torch.full_like(t, -7) for t in g2.new_outputs()[:3]]
    lg2 = torch.zeros((160, wide.N, 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(binding.StandError):
        g2.verify_static(0, lg2, *outs)
    torch.cuda.synchronize()
    assert all(bool((t == -7).all()) for t in outs)
    g2.verify(0, lg2, *outs)                     # the allocating entry point still takes it
    torch.cuda.synchronize()
    assert bool((outs[2] == 1).all())
    for x in (big.g, small.g, g2):
        x.close()


@pytest.mark.parametrize("name,over", [
    ("cfg1", dict(V=32003, B=3, rho=0.7)),                       # fp32, 48 rows: sixteen waves each
    ("cfg2", dict(V=50257, B=2, rho=0.7)),                       # bf16, rows that start at every alignment
    ("cfg3", dict(V=70003, B=5, rho=0.7)),                       # 320 rows: four waves each
    ("cfg3", dict(V=20011, B=5, rho=0.7)),                       # 320 rows, held whole
])
def test_verify_static_on_long_rows(name, over):
    """Rows of many vectors: the token is located over all segments, and head and tail elements lie outside the vectors."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2506_04708_amd import binding
    from tests import lockstep
    print("no-alloc verify: %s %s" % (name, over), flush=True)
    run = _Run(binding, lockstep, name, over, 4)
    for rep in range(3):
        ref, got = _both(run.g, run.step, run.logits())
        for r, x, what in zip(ref, got, ("tokens", "nodes", "lengths")):
            assert np.array_equal(r, x), "%s differ: %s vs %s" % (what, x, r)
        run.advance()
    assert run.g.stats().filter_mismatch == 0
    run.g.close()
