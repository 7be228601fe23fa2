"""Calls beside those that the benchmark times, against a call of the same size whose time is known to be near its bound: rules
of the dispatch that are off show as factors here.  Both calls of a pair run in turn on the same GPU, and the smallest of
several means of each counts; the factors lie between what the pairs measure and what they did with the fault they look for."""
import pytest
import torch

from paper_2104_11125_amd import binding

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _normal(numel, seed):
    return torch.randn(numel, generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV)


def _times(calls, rounds=7, least_us=3000.0):
    """Smallest mean time of each call in us; a call takes the number of its turn."""
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    turn, reps, best = [0] * len(calls), [8] * len(calls), [float("inf")] * len(calls)
    for r in range(rounds + 2):                                 # (two to warm up and to find the number of repetitions)
        for c, call in enumerate(calls):
            ev[0].record()
            for _ in range(reps[c]):
                call(turn[c])
                turn[c] += 1
            ev[1].record()
            torch.cuda.synchronize()
            us = ev[0].elapsed_time(ev[1]) * 1e3 / reps[c]
            if r < 2:
                reps[c] = max(8, min(400, int(least_us / us)))
            else:
                best[c] = min(best[c], us)
    return best


@pytest.mark.parametrize("n,numel,chunk,factor", [
    (3, 8_000_000, 255, 1.0), (2, 30_000_000, 255, 0.92), (8, 1_000_000, 255, 1.04), (8, 300_000, 255, 0.79),   # half of the lanes idle in one launch
    (2, 10_000_000, 400, 0.885), (1, 30_000_000, 400, 0.775), (3, 3_000_000, 400, 0.93),                        # one chunk per group of two tiles
    (2, 3_000_000, 340, 0.885), (2, 10_000_000, 509, 0.835),
    (1, 30_000_000, 1000, 0.74), (2, 300_000, 1000, 0.68), (1, 3_000_000, 600, 0.74), (8, 3_000_000, 700, 1.02),   # groups of four tiles
    (2, 10_000_000, 100, 0.82), (1, 30_000_000, 112, 0.68), (4, 3_750_000, 25, 1.0),
])
def test_chunk_sizes_that_leave_lanes_idle(n, numel, chunk, factor):
    """Against chunks of 1030, for which the maxima are always found by atomics (they are too long for a group): the way that the rules choose takes the
    share of that step's time that the faster way was measured to take, and a little more."""
    calls, keep = [], []
    grad = [_normal(numel, i) for i in range(n)]
    for ch in (chunk, 1030):
        k = -(-numel // ch)
        ctx = binding.scalecom_init(numel, n, torch.float32, 1, DEV, k_max=k)
        mem = [torch.zeros(numel, device=DEV) for _ in range(n)]
        idx, red = torch.empty(k, dtype=torch.int32, device=DEV), torch.empty(k, device=DEV)
        keep.append(ctx)
        calls.append(lambda t, ctx=ctx, mem=mem, ch=ch, idx=idx, red=red: ctx.scalecom_step_chunked(mem, grad, ch, 0.1, 0.1, t, idx, red))
    got, base = _times(calls)
    print(f"[speed] {n} x {numel} chunk {chunk}: {got:.1f} us, 1030: {base:.1f} us, {got / base:.3f}", flush=True)
    assert got <= factor * base
    for ctx in keep:
        ctx.close()


@pytest.mark.parametrize("n,tensors,size,factor", [(2, 64, 125_000, 1.25), (8, 98, 60_000, 1.15), (2, 4, 1_250_000, 1.15)])
def test_tensors_of_equal_size_against_one_vector(n, tensors, size, factor):
    """Several million positions in tensors that are all larger than a supertile (8192): no slower than one vector of
    that length beyond the tables and searches per tensor."""
    numel = tensors * size
    offsets, ks = [t * size for t in range(tensors + 1)], [size // 100] * tensors
    grad = [_normal(numel, i) for i in range(n)]
    calls, keep = [], []
    for layered in (True, False):
        k = sum(ks)
        ctx = binding.scalecom_init(numel, n, torch.float32, tensors if layered else 1, DEV, k_max=k)
        mem = [torch.zeros(numel, device=DEV) for _ in range(n)]
        idx, red = torch.empty(k, dtype=torch.int32, device=DEV), torch.empty(k, device=DEV)
        keep.append(ctx)
        if layered:
            calls.append(lambda t, c=ctx, m=mem, i=idx, r=red: c.scalecom_step_layers(m, grad, offsets, ks, 0.1, 0.1, t, i, r))
        else:
            calls.append(lambda t, c=ctx, m=mem, i=idx, r=red: c.scalecom_step(m, grad, k, 0.1, 0.1, t, i, r))
    got, base = _times(calls)
    print(f"[speed] {tensors} x {size}: {got:.1f} us, one vector: {base:.1f} us", flush=True)
    assert got <= factor * base
    for ctx in keep:
        ctx.close()


@pytest.mark.parametrize("select,n,count,size,large,factor", [
    ("exact", 16, 600, 64, [100_000] * 10, 1.12), ("exact", 16, 1000, 50, [50_000] * 10, 1.12),   # short layouts
    ("exact", 3, 20000, 64, [3_000_000] * 10, 1.12), ("chunk", 8, 20000, 64, [3_000_000] * 10, 1.2),   # the all-learner pass
    ("chunk", 3, 600, 64, [300_000] * 10, 1.2),                                                   # the chunk-wise step in one launch
])
def test_small_tensors_side_by_side(select, n, count, size, large, factor):
    """Many small tensors in front of the large ones: no slower than with the same tensors mixed, whose parts, chunks and
    supertiles every one of the chip's XCDs gets a like number of."""
    grad, calls, keep, per = None, [], [], count // len(large)
    for sizes in ([size] * (per * len(large)) + large, [s for l in large for s in [size] * per + [l]]):
        offsets = [0]
        for s in sizes:
            offsets.append(offsets[-1] + s)
        numel, ks = offsets[-1], [-(-s // 100) for s in sizes]
        grad = grad or [_normal(numel, i) for i in range(n)]
        ctx = binding.scalecom_init(numel, n, torch.float32, len(sizes), DEV, k_max=sum(ks))
        mem = [torch.zeros(numel, device=DEV) for _ in range(n)]
        idx, red = torch.empty(sum(ks), dtype=torch.int32, device=DEV), torch.empty(sum(ks), device=DEV)
        keep.append(ctx)
        step = ctx.scalecom_step_layers if select == "exact" else ctx.scalecom_step_layers_chunked
        sel = ks if select == "exact" else [100] * len(sizes)
        calls.append(lambda t, f=step, m=mem, o=offsets, s=sel, i=idx, r=red: f(m, grad, o, s, 0.1, 0.1, t, i, r))
    got, base = _times(calls)
    print(f"[speed] {select} {count} x {size} + {len(large)} x {large[0]}, {n} learners: {got:.1f} us, mixed: {base:.1f} us", flush=True)
    assert got <= factor * base
    for ctx in keep:
        ctx.close()


def test_further_learners_on_short_supertiles():
    """Tensors of 1000, an eighth of a supertile each: seven more learners cost little more than the step of one, whose search takes most of the time."""
    count, size = 10_000, 1000
    numel, offsets, ks = count * size, [t * size for t in range(count + 1)], [size // 100] * count
    grad = [_normal(numel, i) for i in range(8)]
    idx, red = torch.empty(sum(ks), dtype=torch.int32, device=DEV), torch.empty(sum(ks), device=DEV)
    calls, keep = [], []
    for n in (8, 1):
        ctx = binding.scalecom_init(numel, n, torch.float32, count, DEV, k_max=sum(ks))
        mem = [torch.zeros(numel, device=DEV) for _ in range(n)]
        keep.append(ctx)
        calls.append(lambda t, c=ctx, m=mem, n=n: c.scalecom_step_layers(m, grad[:n], offsets, ks, 0.1, 0.1, t, idx, red))
    got, base = _times(calls)
    print(f"[speed] {count} x {size}: 8 learners {got:.1f} us, 1 learner {base:.1f} us", flush=True)
    assert got <= 2.3 * base
    for ctx in keep:
        ctx.close()


@pytest.mark.parametrize("n,large,others,factor", [
    (2, 1_750_000, [262_144] * 21, 1.1), (8, 880_000, [60_000] * 20, 1.38), (2, 880_000, [4_000] * 300, 1.38),
])
def test_diagnostic_with_one_large_tensor(n, large, others, factor):
    """Every block searches its tensor's index set, the longer the more parts that has.  One large tensor beside smaller ones, against as many positions in
    tensors of one size: 1.01, 1.23 and 1.24 times the time with its parts spread over the chip, 1.01, 1.53 and 1.56 with all of them on one or two XCDs."""
    numel = large + sum(others)
    count = len(others) + 1
    grad = [_normal(numel, i) for i in range(n)]
    calls, keep = [], []
    for sizes in ([large] + others, [numel // count] * count):
        offsets = [0]
        for s in sizes:
            offsets.append(offsets[-1] + s)
        ks = [-(-s // 50) for s in sizes]
        ctx = binding.scalecom_init(numel, n, torch.float32, count, DEV, k_max=sum(ks))
        mem = [torch.zeros(numel, device=DEV) for _ in range(n)]
        d = torch.empty(count, dtype=torch.int32, device=DEV)
        for t in range(2 * n):
            ctx.scalecom_step_layers(mem, grad, offsets, ks, 0.1, 0.1, t)
        keep.append(ctx)
        calls.append(lambda t, c=ctx, mem=mem, o=offsets, ks=ks, d=d: c.scalecom_hamming_distance(mem, grad, o, ks, 0.1, t, d))
    got, base = _times(calls)
    print(f"[speed] diagnostic {large} + {len(others)} tensors, {n} learners: {got:.1f} us, equal: {base:.1f} us, {got / base:.3f}", flush=True)
    assert got <= factor * base
    for ctx in keep:
        ctx.close()


@pytest.mark.parametrize("numel,kind", [(200_003, "drop"), (1_048_576, "equal"), (1_048_576, "drop"), (2_097_152, "equal"),
                                        (2_097_152, "sign"), (2_097_152, "two"), (2_097_152, "near"), (2_097_152, "drop")])
def test_ties_and_jumps_on_short_layouts(numel, kind):
    """Magnitudes that are all equal or nearly so, two of them, and gradients whose scale jumps by 64 every third step: the
    search of a short layout takes a few times a step on normal values at most, not a multiple that grows with the length."""
    n, k = 2, numel // 100
    x = _normal(numel, 3)
    other = {"equal": torch.full_like(x, 0.25), "sign": x.sign() * 1e-3, "two": torch.where(x > 2.3, 0.5, 0.25),
             "near": torch.where(x > 0, 1.0, 1.0 + 2.0 ** -23), "drop": x}[kind]
    calls, keep = [], []
    for g, lr, beta in ((x, lambda t: 0.1, 0.1),
                        (other, (lambda t: 1.0 if t % 6 < 3 else 1 / 64) if kind == "drop" else (lambda t: 0.1),
                         1e-3 if kind == "drop" else 1.0)):
        ctx = binding.scalecom_init(numel, n, torch.float32, 1, DEV, k_max=k)
        mem = [torch.zeros(numel, device=DEV) for _ in range(n)]
        grad = [g, g.roll(1)]
        idx, red = torch.empty(k, dtype=torch.int32, device=DEV), torch.empty(k, device=DEV)
        keep.append(ctx)
        calls.append(lambda t, c=ctx, m=mem, g=grad, i=idx, r=red, lr=lr, b=beta: c.scalecom_step(m, g, k, b, lr(t), t, i, r))
    base, got = _times(calls)
    print(f"[speed] {numel} {kind}: {got:.1f} us, normal values: {base:.1f} us", flush=True)
    assert got <= 4.0 * base
    for ctx in keep:
        ctx.close()
