"""HIP graphs of a partition's calls: captured, replayed, captured again for other buffers and dropped when a setting changes,
each batch against a partition whose calls are launched plainly."""
import numpy as np
import pytest

from paper_1911_05146_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: these tests need a real MI355X")
    from paper_1911_05146_amd import hpf
    return hpf


class Job:
    """A partition, its stream and two sets of buffers."""

    def __init__(self, hpf, spec, params, fusion):
        import torch
        self.torch, self.spec, self.m = torch, spec, spec.num_microbatches
        self.part = hpf.Partition(spec, params)
        self.part.set_fusion(fusion)
        self.stream = torch.cuda.Stream()
        p = self.part

        def tensors(shape):
            return [[torch.empty(shape, dtype=p.tdtype, device="cuda:0") for _ in range(self.m)] for _ in range(2)]
        self.x, self.y, self.dy, self.dx = tensors(p.in_shape), tensors(p.out_shape), tensors(p.out_shape), tensors(p.in_shape)
        self.inf = tensors(p.out_shape)
        torch.cuda.synchronize()

    def fill(self, seed, buf):
        gen = self.torch.Generator("cuda:0").manual_seed(seed)
        for t in self.x[buf]:
            t.copy_(self.torch.randn(t.shape, generator=gen, device="cuda:0"))
        for t in self.dy[buf]:
            t.copy_(0.1 * self.torch.randn(t.shape, generator=gen, device="cuda:0"))

    def calls(self, buf, group):
        p, st, n = self.part, self.stream, self.m
        if group:
            yield p.forward_microbatches(0, self.x[buf], act_out=self.y[buf], stream=st)
            yield p.backward_microbatches(0, n, self.dy[buf], self.dx[buf], stream=st)
            return
        for i in range(n):
            yield p.forward_microbatch(i, self.x[buf][i], act_out=self.y[buf][i], stream=st)
        for i in range(n):
            yield p.backward_microbatch(i, self.dy[buf][i], self.dx[buf][i], stream=st)

    def launches(self, group):
        """Launches of every call of a batch and of the inference behind it."""
        self.fill(1, 0)
        self.torch.cuda.synchronize()
        total, out = 0, []

        def count():
            nonlocal total
            now = sum(r["launches"] for r in self.part.profile_read())
            out.append(now - total)
            total = now
        for _ in self.calls(0, group):
            count()
        self.part.grad_accum_zero(stream=self.stream)
        self.part.forward_inference_group(self.x[0], stream=self.stream, out=self.inf[0])
        count()
        return out

    def batch(self, seed, buf, group, sgd=False):
        """Outputs and gradients of one batch on contents of `seed`, then inference on them."""
        p, st = self.part, self.stream
        with self.torch.cuda.stream(st):
            self.fill(seed, buf)
            for t in self.y[buf] + self.dx[buf] + self.inf[buf]:
                t.fill_(float("nan"))
        for _ in self.calls(buf, group):
            pass
        g = p.grad_accum_read(stream=st)
        p.sgd_step(1e-4, 0.9, stream=st) if sgd else p.grad_accum_zero(stream=st)
        p.forward_inference_group(self.x[buf], stream=st, out=self.inf[buf])
        self.torch.cuda.synchronize()
        return [t.clone() for t in self.y[buf] + self.dx[buf] + self.inf[buf]], g


def _rel(a, b):
    return float(np.linalg.norm(a.astype(np.float64) - b) / np.linalg.norm(b.astype(np.float64)))


def graph_launches(f):
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
        f()
    return sum(e.count for e in prof.key_averages() if e.key == "hipGraphLaunch")


@pytest.mark.parametrize("group", [False, True])
@pytest.mark.parametrize("kind", ["long", "asked", "short"])
def test_replayed_calls_equal_plain_ones(gpu, kind, group):
    """long: calls of 96 launches and more, replayed without being asked for; asked: shorter ones after set_graphs(True); short: without."""
    import torch
    depth, hw = (48, 4) if kind == "long" else (3, 8)
    blocks = (W.Block(W.BASIC, 16, 32, 32, 2),) + (W.Block(W.BASIC, 32, 32, 32, 1),) * depth
    spec = W.PartitionSpec(name="graphs", in_h=2 * hw, in_w=2 * hw, in_c=16, blocks=blocks, microbatch=3, num_microbatches=2, seed=3)
    params = W.make_inputs(spec, randomize_affine=True).params
    fusion = 0 if kind == "long" else 1
    a, b = Job(gpu, spec, params, fusion), Job(gpu, spec, params, fusion)
    try:
        print(f"\n[case] {kind} group={group}", flush=True)
        b.part.set_graphs(False)
        b.part.set_profiling(True)
        calls = b.launches(group)
        b.part.set_profiling(False)
        assert len(calls) == (3 if group else 1 + 2 * spec.num_microbatches) and min(calls) >= (96 if kind == "long" else 8), calls
        assert kind == "long" or max(calls) < 96, calls
        if kind == "asked":
            a.part.set_graphs(True)
        a.batch(99, 0, group)
        seed = 0

        def same(buf, times):
            nonlocal seed
            for _ in range(times):
                seed += 1
                (xa, ga), (xb, gb) = (j.batch(seed, buf, group) for j in (a, b))
                for p, q in zip(xa, xb):
                    assert bool(torch.isfinite(p).all()) and torch.equal(p, q)
                assert _rel(ga, gb) < 1e-5      # fp32 atomics
        same(0, 3)                      # captured, then replayed twice on other contents of the same buffers
        assert graph_launches(lambda: a.batch(seed, 0, group)) == (0 if kind == "short" else len(calls))
        assert graph_launches(lambda: a.batch(seed, 1, group)) == 0
        same(1, 3)                      # other buffers: plain, captured, replayed
        same(0, 1)
        for j in (a, b):
            j.part.set_fusion(2)        # another kernel sequence
        same(0, 2)
        for j in (a, b):
            j.part.set_fusion(fusion)
            j.part.set_bn_momentum(0.5)   # forwards move the running statistics, which the inference reads
        same(0, 4)
        assert np.array_equal(a.part.bn_running_read(), b.part.bn_running_read())
        for j in (a, b):
            j.part.set_bn_momentum(1.0)
        a.part.set_graphs(False)
        same(0, 1)
        a.part.set_graphs(True)
        same(0, 2)
        old, _ = a.batch(seed, 0, group, sgd=True)
        new, _ = a.batch(seed, 0, group)          # replays read the updated weights
        a.part.set_graphs(False)
        plain, _ = a.batch(seed, 0, group)
        assert all(torch.equal(p, q) for p, q in zip(new, plain)) and not any(torch.equal(p, q) for p, q in zip(new[:-a.m], old))   # the inference came behind the update
    finally:
        a.part.close()
        b.part.close()
