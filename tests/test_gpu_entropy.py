"""GPU parity: edgc_sample_indices / edgc_entropy_estimate against the CPU oracle.

Bar: sample indices, range and histogram counts bit-exact; entropy within 1e-5
absolute (both sides evaluate it in fp64 from identical integer counts)."""
import math
import os

import numpy as np
import pytest
import torch

import edgc_inputs as gen
import paper_2511_10333_amd as edgc
from oracle import edgc_oracle as orc
from gpu_util import ctx, to_dev

pytestmark = pytest.mark.gpu

H_TOL = 1e-5


def _compare(x_host, stride, chunk, seed, step, bins, value_range=None, x_dev=None, c=None):
    ref = orc.entropy(x_host, stride, chunk, seed, step, bins, value_range)
    xd = to_dev(x_host) if x_dev is None else x_dev
    counts = torch.full((bins,), -1, dtype=torch.int64, device="cuda")
    got = (c or ctx()).entropy_estimate(xd, stride, chunk, seed, step, bins, value_range, counts)
    assert got.status == 0
    assert (got.n_sampled, got.n_nonfinite) == (ref.n_sampled, ref.n_nonfinite)
    assert (got.lo, got.hi) == (ref.lo, ref.hi)
    assert np.array_equal(counts.cpu().numpy().astype(np.uint64), ref.counts)
    assert abs(got.H_bits - ref.H_bits) <= H_TOL
    if math.isinf(ref.h_diff_nats):
        assert got.h_diff_nats == ref.h_diff_nats
    else:
        assert abs(got.h_diff_nats - ref.h_diff_nats) <= H_TOL
    return got, ref


@pytest.mark.parametrize("n,stride,chunk", [(1, 1, 1), (1000, 7, 3), (4097, 100, 64), (100_000, 10, 1),
                                             (1_048_576, 100, 64), (300_007, 4, 128), (50, 100, 8),
                                             (70_001, 1, 64), (5000, 3, 4096)])
def test_sample_indices_bit_exact(n, stride, chunk):
    for seed, step in [(0, 0), (123, 7), (2**63 + 5, 2**40)]:
        want = orc.sample_indices(n, stride, chunk, seed, step)
        buf = torch.full((max(want.size, 1) + 8,), -1, dtype=torch.int64, device="cuda")
        cnt = ctx().sample_indices(n, stride, chunk, seed, step, buf)
        torch.cuda.synchronize()
        assert cnt == want.size
        got = buf.cpu().numpy()
        assert np.array_equal(got[:cnt].astype(np.uint64), want)
        assert np.all(got[cnt:] == -1)                      # nothing written past the sample


def test_config1_matrix_sample_one_percent_256_bins():
    w = gen.WORKLOADS["cfg1_1024sq_r4"]
    (_, g), = gen.workload_matrices("cfg1_1024sq_r4")
    for chunk in (64, 1):
        for step in range(3):
            got, ref = _compare(g.reshape(-1), w["stride"], chunk, w["seed"], step, w["bins"])
            assert abs(got.n_sampled - g.size // 100) <= 64


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("stride,chunk,bins", [(1, 64, 256), (10, 64, 4096), (100, 64, 65536),
                                                (1000, 64, 1024), (7, 33, 1000), (10, 1, 256),
                                                (1, 1, 100000), (3, 8, 20000)])
def test_laplace_mixture_buffer(dtype, stride, chunk, bins):
    n = (1 << 22) + 12345                                   # several tiles and a ragged tail
    x = gen.laplace_mixture(n, seed=0, dtype=dtype)
    _compare(x, stride, chunk, 7, 3, bins)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_unaligned_base_pointer_uses_scalar_path(dtype):
    n = 200_003
    x = gen.laplace_mixture(n + 1, seed=3, dtype=dtype)
    xd = to_dev(x)[1:]                                      # 4- or 2-byte aligned only
    _compare(x[1:], 5, 64, 1, 1, 512, x_dev=xd)
    _compare(x[1:], 1, 64, 1, 1, 512, x_dev=xd)


def test_caller_range_and_outliers_clamped():
    x = gen.laplace_mixture(500_000, seed=4)
    _compare(x, 4, 64, 0, 0, 1024, value_range=(-0.01, 0.01))
    _compare(x, 1, 64, 0, 0, 64, value_range=(0.0, 0.0))   # degenerate range: everything in bin 0


def test_nonfinite_values_are_skipped_and_counted():
    x = gen.gaussian(300_000, 1e-3, 1)
    x[::1000] = np.nan
    x[5::3000] = np.inf
    x[7::5000] = -np.inf
    got, ref = _compare(x, 1, 64, 0, 0, 512)
    assert got.n_nonfinite == ref.n_nonfinite > 0


def test_special_cases_constant_uniform_two_values():
    c = np.full(100_000, 0.125, dtype=np.float32)
    got, _ = _compare(c, 1, 64, 0, 0, 256)
    assert got.H_bits == 0.0 and got.h_diff_nats == -math.inf
    bins = 1024
    u = np.repeat(np.arange(bins, dtype=np.float32) + 0.5, 5)
    got, _ = _compare(u, 1, 64, 0, 0, bins, value_range=(0.0, float(bins)))
    assert abs(got.H_bits - 10.0) < 1e-9
    two = np.array([-1.0] * 4096 + [3.0] * 4096, dtype=np.float32)
    got, _ = _compare(two, 1, 64, 0, 0, 64)
    assert abs(got.H_bits - 1.0) < 1e-12


def test_gaussian_lemma2_on_device():
    sigma = 1e-3
    x = gen.gaussian(4_000_000, sigma, 9)
    got = ctx().entropy_estimate(to_dev(x), 1, 64, 0, 0, 4096)
    assert abs(got.h_diff_nats - (math.log(sigma) + 0.5 * math.log(2 * math.pi * math.e))) < 5e-3


def test_all_nonfinite_sample_reports_status_and_empty_sample_is_an_error():
    x = torch.full((4096,), float("nan"), device="cuda")
    got = ctx().entropy_estimate(x, 1, 64, 0, 0, 16)
    assert got.status == edgc.binding.ENONFINITE and got.n_nonfinite == 4096
    ok = ctx().entropy_estimate(torch.ones(4096, device="cuda"), 1, 64, 0, 0, 16)   # context still usable
    assert ok.status == 0 and ok.H_bits == 0.0
    # 10 elements, chunk 8 => two chunks; with stride 100 almost every step selects nothing
    small = torch.ones(10, device="cuda")
    step = next(s for s in range(100) if orc.sample_slot(0, s, 100) >= 2)
    with pytest.raises(edgc.EdgcError) as e:
        ctx().entropy_estimate(small, 100, 8, 0, step, 16)
    assert e.value.code == edgc.binding.ENONFINITE


def test_bad_arguments_rejected_before_launch():
    x = torch.ones(64, device="cuda")
    c = ctx()
    for kw in [dict(stride=0), dict(chunk=0), dict(bins=0), dict(bins=(1 << 20) + 1)]:
        a = dict(stride=1, chunk=1, bins=16); a.update(kw)
        with pytest.raises(edgc.EdgcError) as e:
            c.entropy_estimate(x, a["stride"], a["chunk"], 0, 0, a["bins"])
        assert e.value.code == edgc.binding.EINVAL
    with pytest.raises(edgc.EdgcError):
        c.entropy_estimate(x, 1, 1, 0, 0, 16, value_range=(1.0, 0.0))


def test_repeated_calls_are_deterministic():
    x = to_dev(gen.laplace_mixture(1 << 20, seed=8))
    a = ctx().entropy_estimate(x, 10, 64, 5, 5, 4096)
    for _ in range(3):
        b = ctx().entropy_estimate(x, 10, 64, 5, 5, 4096)
        assert (a.H_bits, a.h_diff_nats, a.lo, a.hi) == (b.H_bits, b.h_diff_nats, b.lo, b.hi)


def test_result_reaches_pageable_and_pinned_host_memory_alike():
    """Pinned host memory takes the result straight from the kernel, pageable memory through a
    copy on the stream: the caller sees the same bytes."""
    x = gen.laplace_mixture(1 << 20, 12)
    d = to_dev(x)
    c = ctx()
    pinned = torch.zeros(edgc.binding.ENTROPY_RESULT_BYTES, dtype=torch.uint8, pin_memory=True)
    pageable = torch.zeros(edgc.binding.ENTROPY_RESULT_BYTES, dtype=torch.uint8)
    odd = torch.zeros(edgc.binding.ENTROPY_RESULT_BYTES + 8, dtype=torch.uint8, pin_memory=True)[4:-4]   # misaligned view
    for out in (pinned, pageable, odd):
        c.entropy_estimate_async(d, 100, 64, 3, 7, 1024, out)
    torch.cuda.synchronize()
    a = edgc.EntropyResult.from_buffer(pinned.numpy().tobytes())
    assert a == edgc.EntropyResult.from_buffer(pageable.numpy().tobytes())
    assert a == edgc.EntropyResult.from_buffer(odd.numpy().tobytes())
    want = orc.entropy(x, 100, 64, 3, 7, 1024)
    assert a.n_sampled == want.n_sampled and abs(a.H_bits - want.H_bits) <= 1e-5


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_seeded_sweep_of_sizes_offsets_strides_chunks_and_bins(dtype):
    """Sixty seeded draws of (size, start offset, stride, chunk, bins, step, seed) on slices of one
    buffer, some with NaN and -Inf planted: sizes around the chunk and item boundaries up to samples
    that take the launch shapes of large samples, aligned and unaligned starts.  Counts, range and
    non-finite count bit-exact, entropy to 1e-5; a draw whose sample is empty must fail on both sides."""
    rng = np.random.default_rng(2024 if dtype == "f32" else 2025)
    big = gen.laplace_mixture(72_000_000, 99, dtype=dtype)
    c = edgc.Context(0, max_bins=65536, max_rank=4, max_rows=64, max_cols=64)
    sizes = [1, 7, 63, 64, 65, 4095, 4096, 4097, 100_003, 1 << 20, 3_000_001, 20_000_000, 33_554_433,
             39_999_999, 67_108_871]
    for it in range(60):
        n = int(rng.choice(sizes))
        off = int(rng.choice([0, 0, 0, 1, 3, 4, 8]))
        stride = int(rng.choice([1, 1, 2, 3, 7, 10, 100, 1000]))
        chunk = int(rng.choice([1, 8, 16, 48, 64, 64, 256, 4096]))
        bins = int(rng.choice([16, 256, 1024, 4096, 16384, 32768, 65536]))
        step, seed = int(rng.integers(0, 1000)), int(rng.integers(0, 1 << 30))
        host = big[off:off + n].copy()
        if n > 100 and it % 4 == 0:
            host[rng.integers(0, n, 3)] = 0x7fc0 if dtype == "bf16" else np.float32(np.nan)
            host[rng.integers(0, n)] = 0xff80 if dtype == "bf16" else np.float32(-np.inf)
        dev = to_dev(np.concatenate([np.zeros(off, dtype=host.dtype), host]))[off:]
        case = (it, n, off, stride, chunk, bins, step, seed)
        try:
            ref = orc.entropy(host, stride, chunk, seed, step, bins)
        except orc.OracleError:
            with pytest.raises(edgc.EdgcError):
                c.entropy_estimate(dev, stride, chunk, seed, step, bins)
            continue
        counts = torch.zeros(bins, dtype=torch.int64, device="cuda")
        got = c.entropy_estimate(dev, stride, chunk, seed, step, bins, None, counts)
        assert (got.n_sampled, got.n_nonfinite) == (ref.n_sampled, ref.n_nonfinite), case
        assert (got.lo, got.hi) == (ref.lo, ref.hi), case
        assert np.array_equal(counts.cpu().numpy().astype(np.uint64), ref.counts), case
        assert abs(got.H_bits - ref.H_bits) <= 1e-5, case
        # (a sample of one value has no width: -inf on both sides)
        assert got.h_diff_nats == ref.h_diff_nats or abs(got.h_diff_nats - ref.h_diff_nats) <= 1e-5, case
    c.close()



def _context_with(**env):
    """A context created under the library's tuning variables (read once, at edgc_create)."""
    old = {k: os.environ.get(k) for k in env}
    os.environ.update({k: str(v) for k, v in env.items()})
    try:
        return edgc.Context(0, max_bins=1 << 17, max_rank=4, max_rows=64, max_cols=64)
    finally:
        for k, v in old.items():
            if v is None:
                del os.environ[k]
            else:
                os.environ[k] = v


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("mode", ["one_read", "plain"])
def test_sixteen_bit_counter_kernels_on_small_and_ragged_samples(mode, dtype):
    """The one-read kernels (16-bit counters per block; bf16 samples counted by bit pattern, fp32
    samples on more than 16384 bins) are chosen for large samples by default; here they take every
    sample.  `plain`: the two-pass kernels alone.  Both must give the oracle's counts, range and
    entropy."""
    c = _context_with(EDGC_TUNE_PATTERN={"one_read": 1, "plain": 0}[mode], EDGC_TUNE_PATTERN_MIN=0)
    bins_list = [16, 256, 4096, 20000, 65536] + ([100000] if dtype == "bf16" else [])
    rng = np.random.default_rng(77)
    big = gen.laplace_mixture(3_000_000, 5, dtype=dtype)
    for n in (1, 9, 64, 4097, 262_147, 2_999_999):
        for off in (0, 1):
            host = big[off:off + n].copy()
            if n > 1000:
                host[rng.integers(0, n, 4)] = 0x7fc0 if dtype == "bf16" else np.float32(np.nan)
                host[rng.integers(0, n)] = 0x7f80 if dtype == "bf16" else np.float32(np.inf)
                host[n // 2: n // 2 + 700] = 0                    # a run of equal values
            dev = to_dev(big[:off + n].copy())
            dev[off:] = to_dev(host)
            for bins in bins_list:
                stride, chunk = int(rng.choice([1, 3, 10])), int(rng.choice([1, 8, 64, 256]))
                try:
                    _compare(host, stride, chunk, 11, int(rng.integers(0, 50)), bins, x_dev=dev[off:], c=c)
                except orc.OracleError:
                    continue
    x = big[:500_000]
    _compare(x, 2, 64, 0, 0, 1024, value_range=(-0.01, 0.01), c=c)
    _compare(x, 1, 64, 0, 0, 40000, value_range=(-0.02, 0.05), c=c)
    _compare(x, 1, 64, 0, 0, 64, value_range=(0.0, 0.0), c=c)
    const = np.full(70_000, big[17], dtype=big.dtype)             # one value 70000 times: 16-bit fields wrap twice
    for bins in (256, 40000):
        got, _ = _compare(const, 1, 64, 0, 0, bins, c=c)
        assert got.H_bits == 0.0
    nan = torch.full((4096,), float("nan"), device="cuda", dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)
    assert c.entropy_estimate(nan, 1, 64, 0, 0, 40000).status == edgc.binding.ENONFINITE
    # a group of buffers is one sample
    parts = [big[:100_001], big[200_000:200_064], big[1_000_000:1_700_003]]
    out = torch.zeros(edgc.binding.ENTROPY_RESULT_BYTES, dtype=torch.uint8, pin_memory=True)
    counts = torch.zeros(65536, dtype=torch.int64, device="cuda")
    c.entropy_estimate_async([to_dev(p) for p in parts], 1, 64, 3, 2, 65536, out, None, counts)
    torch.cuda.synchronize()
    got = edgc.EntropyResult.from_buffer(out.numpy().tobytes())
    ref = orc.entropy(np.concatenate(parts), 1, 64, 3, 2, 65536)           # stride 1: every element, however chunked
    assert (got.n_sampled, got.lo, got.hi) == (ref.n_sampled, ref.lo, ref.hi)
    assert np.array_equal(counts.cpu().numpy().astype(np.uint64), ref.counts)
    c.close()


@pytest.mark.parametrize("a,b", [(0.375, 0.375), (-2.5, 2.0 ** -20), (-3.0, -0.5), (0.0, 1.0), (2.0 ** 100, -2.0 ** -100)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_sixteen_bit_counters_that_end_at_zero(dtype, a, b):
    """Every block counts a whole multiple of 32768 of one value, so that all of it has been moved off and the field is
    zero at the end: range, counts and entropy still hold the value.  Few values: most runs of fields are not stored."""
    n, bins = 1 << 26, 65536 if dtype == "f32" else 4096
    x = torch.full((n,), a, device="cuda", dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)
    x[n // 2:] = b
    counts = torch.empty(bins, dtype=torch.int64, device="cuda")
    got = ctx().entropy_estimate(x, 1, 64, 0, 0, bins, None, counts)
    assert got.status == 0 and (got.lo, got.hi, got.n_sampled) == (min(a, b), max(a, b), n)
    if a == b:
        assert got.H_bits == 0.0 and int(counts[0]) == n
    else:
        assert got.H_bits == 1.0 and int(counts[0]) == n // 2 and int(counts[bins - 1]) == n // 2


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_sixteen_bit_counters_under_the_heaviest_contention(dtype):
    """Every thread of every block hits the same one or two 16-bit fields: a constant buffer and a
    two-valued one of 2^26 + 5 elements (large enough for the one-read kernels by default; fp32 takes
    them on 65536 bins).  The fields wrap thousands of times per block; the counts must still be exact."""
    n = (1 << 26) + 5
    bins = 65536 if dtype == "f32" else 4096
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    c = ctx()
    x = torch.full((n,), 0.375, device="cuda", dtype=tdt)
    counts = torch.empty(bins, dtype=torch.int64, device="cuda")
    got = c.entropy_estimate(x, 1, 64, 0, 0, bins, None, counts)
    assert got.status == 0 and got.n_sampled == n and got.H_bits == 0.0 and (got.lo, got.hi) == (0.375, 0.375)
    assert int(counts[0]) == n and int(counts.sum()) == n
    x[1::3] = -2.5                                         # two values, one third / two thirds
    ref = orc.entropy(to_host_any(x), 1, 64, 0, 0, bins)
    got = c.entropy_estimate(x, 1, 64, 0, 0, bins, None, counts)
    assert (got.lo, got.hi, got.n_sampled) == (ref.lo, ref.hi, n)
    assert np.array_equal(counts.cpu().numpy().astype(np.uint64), ref.counts)
    assert abs(got.H_bits - ref.H_bits) <= H_TOL
    x[7::1000] = float("nan")
    ref = orc.entropy(to_host_any(x), 1, 64, 0, 0, bins)
    got = c.entropy_estimate(x, 1, 64, 0, 0, bins, None, counts)
    assert got.n_nonfinite == ref.n_nonfinite > 0
    assert np.array_equal(counts.cpu().numpy().astype(np.uint64), ref.counts)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rounds", [1, 2, 3, 4, 5, 6])
def test_every_element_of_every_round_is_seen(dtype, rounds):
    """Blocks whose whole range is exactly `rounds` rounds of unconditional loads, and one item more: the range pass (256 and
    1024 threads) finds an extreme value wherever it stands in a round, and the counts of the histogram kernels (512 and 1024
    threads, 16-bit counters) are those of all elements."""
    tdt, vec = (torch.bfloat16, 8) if dtype == "bf16" else (torch.float32, 4)
    gen_ = torch.Generator(device="cuda").manual_seed(rounds)
    plain, one_read = _context_with(EDGC_TUNE_PATTERN=0), _context_with(EDGC_TUNE_PATTERN_MIN=0)
    counts = torch.empty(65536, dtype=torch.int64, device="cuda")
    for blocks, threads, extra in [(1024, 256, 0), (1024, 256, 1), (256, 1024, 0), (256, 1024, 4096)]:
        items = blocks * threads * 4 * rounds + 4096 + extra            # the last chunk is read with checks
        x = (torch.rand(items * vec, generator=gen_, device="cuda") - 0.5).to(tdt)
        for c, bins in [(plain, 4096), (plain, 40000), (one_read, 4096), (one_read, 65536)]:
            got = c.entropy_estimate(x, 1, 64, 0, 0, bins, None, counts[:bins])
            xf = x.float()
            lo, hi = xf.min(), xf.max()
            assert (got.lo, got.hi, got.n_sampled) == (float(lo), float(hi), x.numel())
            scale = torch.tensor(float(bins), dtype=torch.float32) / (hi - lo).cpu()
            want = torch.bincount(((xf - lo) * scale.cuda()).long().clamp_(0, bins - 1), minlength=bins)
            assert torch.equal(counts[:bins], want), (blocks, threads, extra, bins)
        if blocks == 1024:
            for at in range(4 * rounds):                                # every load of a block's rounds, every element of it
                for e in range(vec):
                    k = ((3 * 4 * rounds + at) * threads + (37 * at + 11 * e) % threads) * vec + e
                    old = x[k].clone()
                    x[k] = -2.0 if e % 2 else 2.0
                    got = plain.entropy_estimate(x, 1, 64, 0, 0, 256)
                    assert (got.lo == -2.0) if e % 2 else (got.hi == 2.0), (at, e)
                    x[k] = old
    plain.close()
    one_read.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("off", [0, 1])
def test_sixteen_bit_counters_swept_across_short_and_large_buffers(dtype, off):
    """31 short buffers of one value with ragged ends, then a large one of two values: every round of a block, over one
    buffer or over many, adds as much to one field as a round can, and the fields are swept several times per block.  With
    `off` items are single elements, of which eight rounds go between two sweeps."""
    c = _context_with(EDGC_TUNE_PATTERN_MIN=0)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    sizes = [4000 + 67 * i for i in range(31)] + [20_000_003]
    dev = []
    for n in sizes:
        x = torch.full((n + 8,), 0.375, device="cuda", dtype=tdt)[off:off + n]
        if n > 1 << 20:
            x[1::3] = -2.5
        dev.append(x)
    host = [to_host_any(x) for x in dev]
    for stride, chunk, bins in [(1, 64, 65536), (2, 64, 65536), (1, 64, 20000)]:
        counts = torch.empty(bins, dtype=torch.int64, device="cuda")
        got = c.entropy_estimate(dev, stride, chunk, 5, 1, bins, None, counts)
        cat = np.concatenate([h[orc.sample_indices(h.size, stride, chunk, 5, 1)] for h in host])
        ref = orc.entropy(cat, 1, 1, 0, 0, bins)
        assert (got.lo, got.hi, got.n_sampled) == (ref.lo, ref.hi, cat.size)
        assert np.array_equal(counts.cpu().numpy().astype(np.uint64), ref.counts), (stride, bins)
        assert abs(got.H_bits - ref.H_bits) <= H_TOL
    c.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("items", [1, 4095, 4096, 4097, 16 * 1024, 16 * 1024 + 1, 64 * 1024, 64 * 1024 + 1, 1024 * 1024,
                                   1024 * 1024 + 1])
def test_one_round_kernels_at_the_edges_of_their_blocks(dtype, items):
    """Samples at the line between one block and several, one and two sets of counters, two and four items per thread, one round
    and several; in one buffer and in many, of which a block reads whole ones, parts and ragged ends; non-finite
    values, bin counts on both sides of the line and a caller's range.  Counts and range as plain fp32 arithmetic gives them."""
    tdt, vec = (torch.bfloat16, 8) if dtype == "bf16" else (torch.float32, 4)
    gen_ = torch.Generator(device="cuda").manual_seed(items)
    c, n = ctx(), items * vec
    cuts = [[n], [n - n // 3, n // 3], [64 * vec * (1 + k % 3) - k % vec for k in range(20)]]
    cuts[2].append(max(1, n - sum(-(-k // vec) for k in cuts[2]) * vec))     # (as many items, whole or not)
    for sizes in cuts:
        if min(sizes) < 1 or (len(sizes) > 2 and items < 4095):
            continue
        # every buffer begins on a 16-byte boundary, as torch allocates it
        bufs = [((torch.rand(k, generator=gen_, device="cuda") - 0.25) ** 3).to(tdt) for k in sizes]
        flat = torch.cat(bufs).float()
        if flat.numel() > 100:
            bufs[0][7], bufs[-1][-1] = float("nan"), float("inf")
            flat[7], flat[-1] = float("nan"), float("inf")
        fin = flat[torch.isfinite(flat)]
        for bins, rng in [(1, None), (255, None), (4096, None), (4097, None), (1024, (-0.01, 0.2))]:
            counts = torch.full((bins,), -1, dtype=torch.int64, device="cuda")
            got = c.entropy_estimate(bufs if len(bufs) > 1 else bufs[0], 1, 64, 0, 0, bins, rng, counts)
            lo, hi = (fin.min(), fin.max()) if rng is None else (torch.tensor(v, device="cuda") for v in rng)
            scale = torch.tensor(float(bins), dtype=torch.float32) / (hi - lo).cpu()
            at = (fin - lo) * scale.cuda() if float(hi) > float(lo) else torch.zeros_like(fin)
            want = torch.bincount(at.clamp(0, bins).long().clamp_(0, bins - 1), minlength=bins)
            assert (got.lo, got.hi) == (float(lo), float(hi))
            assert (got.n_sampled, got.n_nonfinite) == (flat.numel(), flat.numel() - fin.numel())
            assert torch.equal(counts, want), (sizes[:3], bins, rng)
            p = want[want > 0].double() / fin.numel()
            assert abs(got.H_bits - float(-(p * torch.log2(p)).sum())) <= H_TOL


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("stride,chunk", [(3, 64), (10, 64), (100, 64), (7, 200)])
def test_one_round_kernels_on_strided_samples_of_many_buffers(dtype, stride, chunk):
    """Strided samples of 1 to 32 buffers of ragged lengths, against the oracle's samples of the same buffers."""
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rng = np.random.default_rng(stride)
    for count in (1, 2, 3, 24, 32):
        sizes = [int(rng.integers(1, 60_000)) for _ in range(count - 1)] + [1_000_003]
        dev = [torch.from_numpy(rng.laplace(0, 1e-3, k).astype(np.float32)).cuda().to(tdt) for k in sizes]
        for step in range(3):
            parts = [x.float().cpu().numpy()[orc.sample_indices(x.numel(), stride, chunk, 7, step).astype(np.int64)] for x in dev]
            ref = orc.entropy(np.concatenate(parts), 1, 64, 0, 0, 1024)
            counts = torch.full((1024,), -1, dtype=torch.int64, device="cuda")
            got = ctx().entropy_estimate(dev if count > 1 else dev[0], stride, chunk, 7, step, 1024, None, counts)
            assert (got.n_sampled, got.lo, got.hi) == (ref.n_sampled, ref.lo, ref.hi)
            assert np.array_equal(counts.cpu().numpy().astype(np.uint64), ref.counts)
            assert abs(got.H_bits - ref.H_bits) <= H_TOL


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [40_001, 600_011, 3_000_007])
def test_last_block_sums_many_bins(dtype, n):
    """Bin counts at the lines between few and many bins per thread, between sets of 32-bit counters and none, and no multiple of
    the bins of an iteration; samples with one set of counters, with eight, of blocks of 512 and 1024 threads."""
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen_ = torch.Generator(device="cuda").manual_seed(n)
    x = ((torch.rand(n, generator=gen_, device="cuda") - 0.25) ** 3).to(tdt)
    x[5] = float("nan")
    fin = x.float()[torch.isfinite(x)]
    c = edgc.Context(0, max_bins=200_000, max_rank=4, max_rows=64, max_cols=64)
    lo, hi = fin.min(), fin.max()
    for bins in (2048, 2049, 4096, 4097, 8195, 16383, 16384, 16385, 32769, 65535, 65536, 100_001):
        counts = torch.full((bins,), -1, dtype=torch.int64, device="cuda")
        got = c.entropy_estimate(x, 1, 64, 0, 0, bins, None, counts)
        scale = torch.tensor(float(bins), dtype=torch.float32) / (hi - lo).cpu()
        want = torch.bincount(((fin - lo) * scale.cuda()).long().clamp_(0, bins - 1), minlength=bins)
        assert torch.equal(counts, want), bins
        p = want[want > 0].double() / fin.numel()
        assert got.n_nonfinite == 1 and abs(got.H_bits - float(-(p * torch.log2(p)).sum())) <= H_TOL, bins
    c.close()


def _kernels_of(c, x, bins):
    c.profile_begin(64)
    c.entropy_estimate(x, 1, 64, 0, 0, bins)
    return c.profile_end()


@pytest.mark.parametrize("bins,line", [(256, 8 << 20), (4096, 8 << 20), (16384, 8 << 20), (16385, 4 << 20), (65536, 4 << 20)])
def test_bf16_samples_are_counted_by_pattern_from_the_line_on(bins, line):
    """The kernels on both sides of the line between two passes and one read."""
    x = (torch.randn(line, device="cuda") * 1e-3).bfloat16()
    c = _context_with()
    assert "k_hist" in _kernels_of(c, x[:-8], bins)
    stats = _kernels_of(c, x, bins)
    assert set(stats) == {"k_wide_hist", "k_wide_reduce"}
    # the blocks' fields (128 KiB each) are mostly not read: not credited.  Marks of up to 1024 blocks, credits, bins are
    assert 8 * (65536 + bins) < stats["k_wide_reduce"]["bytes"] <= 8 * (65536 + bins) + 32 * 1024
    c.close()


def to_host_any(x):
    if x.dtype == torch.bfloat16:
        return x.view(torch.int16).cpu().numpy().view(np.uint16)
    return x.cpu().numpy()


@pytest.mark.parametrize("dtype,bins,n", [("f32", 1, 3000), ("f32", 2, 40000), ("f32", 255, 3000), ("f32", 1000, 60001), ("f32", 1023, 300000),
                                          ("f32", 4096, 2000000), ("f32", 4095, 9000000), ("f32", 5003, 200000), ("f32", 16384, 3000),
                                          ("f32", 16384, 5000000), ("f32", 20001, 700000), ("f32", 65536, 3000000), ("f32", 100000, 400000),
                                          ("bf16", 128, 3000), ("bf16", 100, 50000), ("bf16", 128, 12000000), ("bf16", 40000, 60000)])
def test_entropy_of_given_counts(dtype, bins, n):
    """Every kernel that ends in the sum over the bins, on a histogram that is known: single, odd and empty bins, a bin with half
    of the sample.  The logarithms are taken less the exponent of n, so that a term c/n (log2 c - e0) is at most
    c/n (log2(n/c) + 1) and the terms' magnitudes add up to H + 1 at most; a few roundings of 2^-53 of each: 1e-15 (H + 1)."""
    rng = np.random.default_rng(bins + n)
    top = min(bins, 128) if dtype == "bf16" else bins                       # i + 1/2 is a bf16 value below 128
    c = np.floor(rng.exponential(1.0, top) * rng.integers(0, 2, top) * (n / (2.0 * top))).astype(np.int64)
    c[rng.integers(0, top, 1 + top // 8)] = 1
    c[top // 2] += max(0, n - int(c.sum()))
    c = np.minimum(c, n)
    n = int(c.sum())
    x = torch.from_numpy(np.repeat(np.arange(top, dtype=np.float32) + 0.5, c)).cuda()
    x = x[torch.randperm(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))]
    x = x.to(torch.bfloat16) if dtype == "bf16" else x
    counts = torch.empty(bins, dtype=torch.int64, device="cuda")
    e = edgc.Context(0, max_bins=bins, max_rank=32, max_rows=64, max_cols=64)
    got = e.entropy_estimate(x, 1, 64, 0, 0, bins, value_range=(0.0, float(bins)), counts_out=counts)
    e.close()
    assert np.array_equal(counts.cpu().numpy()[:top], c) and int(counts.sum()) == n and got.n_sampled == n
    want = math.fsum(k / n * math.log2(n / k) for k in c.tolist() if k)
    assert abs(got.H_bits - want) <= 1e-15 * (want + 1.0)
    assert want != 0.0 or got.H_bits == 0.0
