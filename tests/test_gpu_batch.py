"""Batched compress / decompress (every tensor of a stage in one launch sequence) against the
oracle, tensor by tensor, and against the single-tensor entry points."""
import numpy as np
import pytest
import torch

import edgc_inputs as gen
import paper_2511_10333_amd as edgc
from oracle import edgc_oracle as orc
from gpu_util import ELEMENTWISE_TOL, elementwise_ratio, rel_fro, to_dev, to_host

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-3, "bf16": 1e-2}


def _widen(a):
    return gen.bf16_bits_to_f32(a) if a.dtype == np.uint16 else a


class Stage:
    """Host and device state of a list of gradient tensors that share one rank."""

    def __init__(self, shapes, r, dtype, seed=0, ragged_ld=False, mats=None, deferred=False, power_iters=1,
                 signal_rank=48, decay=0.9):
        """``mats``: ready-made 2-D gradients (host arrays) instead of generated ones.
        ``deferred``: the residual buffers keep D between steps (edgc_tensor.deferred)."""
        if mats is not None:
            shapes = [g.shape for g in mats]
        self.shapes, self.r, self.dtype = shapes, r, dtype
        self.deferred, self.power_iters, self.steps = deferred, power_iters, 0
        self.ctx = edgc.Context(0, max_rank=128, max_rows=64, max_cols=64)    # own scratch unused here
        self.ctx.reserve_batch([s if len(s) == 2 else (1, s[0]) for s in shapes])
        tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
        self.G, self.Q, self.E = [], [], []
        self.t = []
        for i, s in enumerate(shapes):
            if len(s) == 1:                                   # 1-D tensor: never compressed
                g = gen.gaussian(s[0], 1e-3, seed + i).astype(np.float32)
                g = gen.to_bf16_bits(g) if dtype == "bf16" else g
                self.G.append(g); self.Q.append(None); self.E.append(None)
                self.t.append(edgc.Tensor(to_dev(g), torch.zeros(s[0], dtype=tdt, device="cuda")))
                continue
            m, n = s
            g = mats[i] if mats is not None else \
                gen.lowrank_plus_noise(m, n, min(m, n, signal_rank), decay, 1e-4, seed + i, dtype=dtype)
            self.G.append(g)
            if edgc.tensor_bypassed(m, n, r):
                self.Q.append(None); self.E.append(None)
                self.t.append(edgc.Tensor(to_dev(g), torch.zeros((m, n), dtype=tdt, device="cuda")))
                continue
            ldq = (r + 3) // 4 * 4
            q = np.zeros((n, ldq), dtype=np.float32)
            orc.init_q(q, 0, r, 100 + i)
            self.Q.append(q)
            self.E.append(None)
            gd = to_dev(g)
            if ragged_ld:                                     # rows embedded in a wider buffer
                wide = torch.zeros((m, n + 8), dtype=tdt, device="cuda")
                wide[:, :n] = gd
                gd = wide[:, :n]
            self.t.append(edgc.Tensor(gd, torch.zeros((m, n), dtype=tdt, device="cuda"),
                                      torch.full((m, n), float("nan"), device="cuda"), to_dev(q),
                                      torch.full((m, ldq), 7.0, device="cuda"), True))

    def compressed(self, i):
        return self.Q[i] is not None

    def step_device(self):
        # a deferred compress expects D and the factors of the step before: not on the first step
        self.ctx.compress_batch(self.t, self.r, power_iters=self.power_iters,
                                deferred=self.deferred and self.steps > 0)
        self.ctx.decompress_batch(self.t, self.r, deferred=self.deferred)
        torch.cuda.synchronize()
        self.steps += 1
        for t in self.t:
            t.residual_is_zero = False

    def step_oracle_and_compare(self):
        r, tol = self.r, TOL[self.dtype]
        code = orc.BF16 if self.dtype == "bf16" else orc.F32
        for i, g in enumerate(self.G):
            t = self.t[i]
            if not self.compressed(i):
                assert np.array_equal(to_host(t.grad_out).reshape(g.shape), g), f"tensor {i} must pass through"
                continue
            first = self.E[i] is None
            Po, Qo, Do = orc.compress(g, self.E[i], np.ascontiguousarray(self.Q[i][:, :r]), r)
            out_o, E_o = orc.decompress(Po, Qo, Do, code)
            self.Q[i][:, :r] = Qo
            self.E[i] = E_o
            nD = np.linalg.norm(Do.astype(np.float64))
            assert rel_fro(to_host(t.P)[:, :r], Po) <= tol, i
            assert rel_fro(to_host(t.Q)[:, :r], Qo) <= tol, i
            assert rel_fro(_widen(to_host(t.grad_out)), _widen(out_o)) <= tol, i
            # ... and element by element, |M^_ij - oracle| against ||p_i|| ||q_j|| (a few wrong elements of one
            # tile would not show in a Frobenius norm over the whole matrix)
            assert elementwise_ratio(_widen(to_host(t.grad_out)), _widen(out_o), Po, Qo) <= ELEMENTWISE_TOL[self.dtype], i
            if self.deferred:                                 # the buffer keeps D; E stays in factored form
                assert np.linalg.norm(to_host(t.residual).astype(np.float64) - Do) <= tol * nD, i
                if first:
                    assert np.array_equal(to_host(t.residual), Do.astype(np.float32)), i
                continue
            assert np.linalg.norm(to_host(t.residual).astype(np.float64) - E_o) <= tol * nD, i
            # D = M^ + E_new on the device (first step: its D is the oracle's D bit for bit)
            if first:
                assert rel_fro(to_host(t.residual) + _widen(to_host(t.grad_out)), Do) <= 1e-6


MIXED = [(384, 640), (100,), (130, 70), (6, 200), (257, 129), (512, 256), (64,)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("r", [4, 16])
def test_mixed_stage_matches_oracle_over_three_steps(dtype, r):
    st = Stage(MIXED, r, dtype, seed=3)
    assert not st.compressed(1) and not st.compressed(6)          # 1-D
    assert st.compressed(3) == (not edgc.tensor_bypassed(6, 200, r))
    for _ in range(3):                                            # residual carried from step to step
        st.step_device()
        st.step_oracle_and_compare()


@pytest.mark.parametrize("name,rank,steps,deferred", [("cfg2_gpt_h2048_r16", 16, 2, False),
                                                      ("cfg4_gpt_h5120_bf16", 64, 1, False),
                                                      ("cfg4_gpt_h5120_bf16", 32, 2, True),
                                                      ("cfg4_gpt_h5120_bf16", 128, 2, True)])
def test_benchmark_workload_full_size_in_the_bench_layout(name, rank, steps, deferred):
    """The benchmark's matrices at full size against the oracle's whole steps, grouped as bench.py groups
    them (two groups balanced by size, largest first into the lighter one): two steps of the hidden-2048
    block so that the second carries a residual; the hidden-5120 bf16 block (20480 x 5120 included) for one
    step at rank 64 and, in the layout bench.py times (residual deferred: the second step runs the
    streaming P-pass that subtracts P^ Q^T on the way), for two steps at ranks 32 and 128."""
    w = gen.WORKLOADS[name]
    mats = [g for _, g in gen.workload_matrices(name)]
    order = sorted(range(len(mats)), key=lambda i: -mats[i].size)
    members, load = [[], []], [0, 0]
    for i in order:
        k = load.index(min(load))
        members[k].append(i)
        load[k] += mats[i].size
    assert sorted(members[0] + members[1]) == list(range(len(mats)))
    for idx in members:
        st = Stage(None, rank, w["dtype"], seed=w["seed"], mats=[mats[i] for i in sorted(idx)], deferred=deferred)
        for _ in range(steps):
            st.step_device()
            st.step_oracle_and_compare()
        del st
        torch.cuda.empty_cache()


def test_ragged_leading_dimension_and_rank_48():
    st = Stage([(200, 328), (192, 192), (333, 100)], 48, "f32", seed=9, ragged_ld=True)
    st.step_device()
    st.step_oracle_and_compare()


def test_more_tensors_than_one_group_holds():
    shapes = [(64 + 8 * i, 96 + 4 * i) for i in range(21)]        # 21 > 16 tensors per launch
    st = Stage(shapes, 8, "f32", seed=11)
    st.step_device()
    st.step_oracle_and_compare()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_batch_equals_single_tensor_calls(dtype):
    shapes, r = [(512, 768), (256, 1024), (1024, 256)], 16
    st = Stage(shapes, r, dtype, seed=21)
    single = edgc.Context(0, max_rank=128, max_rows=1024, max_cols=1024)
    ref = []
    for t in st.t:                                                 # same inputs through the single calls
        Q, P = t.Q.clone(), torch.empty_like(t.P)
        E, out = torch.empty_like(t.residual), torch.empty_like(t.grad_out)
        single.compress(t.grad, E, True, Q, P, r)
        single.decompress(P, Q, r, E, out)
        ref.append((P, Q, E, out))
    st.step_device()
    for t, (P, Q, E, out) in zip(st.t, ref):
        # the launch shapes differ (a batch shares the GPU among its tensors), so sums are taken
        # in another order: equal to rounding, not bit for bit
        assert rel_fro(to_host(t.P)[:, :r], to_host(P)[:, :r]) <= 2e-5
        assert rel_fro(to_host(t.Q)[:, :r], to_host(Q)[:, :r]) <= 2e-5
        assert rel_fro(_widen(to_host(t.grad_out)), _widen(to_host(out))) <= (1e-2 if dtype == "bf16" else 2e-5)
    # a batch of one has the single call's launch shape: bit for bit
    one = Stage([shapes[0]], r, dtype, seed=21)
    one.step_device()
    P, Q, E, out = ref[0]
    assert torch.equal(one.t[0].P[:, :r], P[:, :r]) and torch.equal(one.t[0].Q[:, :r], Q[:, :r])
    assert torch.equal(one.t[0].residual, E) and torch.equal(one.t[0].grad_out, out)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("r,m,n", [(40, 20000, 640), (64, 8200, 520), (40, 1000, 600), (100, 16384, 400), (33, 2048, 1023)])
def test_sums_of_partials_do_not_depend_on_how_many_blocks_share_them(dtype, r, m, n, monkeypatch):
    """One tensor, whose sums of Q's partials (and, up to rank 64, of Gram sets) are spread over narrow blocks, and the same
    tensor twice in a batch that aims at twice the blocks: the same splits, summed by whole blocks.  The order is the same."""
    gen_ = torch.Generator(device="cuda").manual_seed(r + m + n)
    G = torch.randn(m, n, device="cuda", generator=gen_).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    Q0 = torch.randn(n, r, device="cuda", generator=gen_)
    got = []
    for copies in (1, 2):
        for knob in ("EDGC_TUNE_P", "EDGC_TUNE_Q"):
            monkeypatch.setenv(knob, str(copies))
        c = edgc.Context(0, max_bins=16, max_rank=r, max_rows=64, max_cols=64)
        c.reserve_batch([(m, n)] * copies)
        ts = []
        for _ in range(copies):
            Q = torch.zeros(n, (r + 3) // 4 * 4, device="cuda")
            Q[:, :r] = Q0
            ts.append(edgc.Tensor(G, torch.empty_like(G), torch.empty(m, n, device="cuda"), Q,
                                  torch.zeros(m, (r + 3) // 4 * 4, device="cuda"), True))
        c.compress_batch(ts, r)
        torch.cuda.synchronize()
        got += [(t.P, t.Q) for t in ts]
        c.close()
    for P, Q in got[1:]:
        assert torch.equal(P, got[0][0]) and torch.equal(Q, got[0][1])


@pytest.mark.parametrize("r,m,n,most", [(40, 2048, 1023, 2), (100, 2000, 640, 2), (100, 300, 3000, 9), (64, 8192, 512, 2), (48, 1000, 600, 3),
                                        (40, 1024, 1600, 9)])
def test_sums_of_gram_matrices_do_not_depend_on_the_neighbours(r, m, n, most, monkeypatch):
    """A matrix of few rows alone and beside copies of itself, on the same splits (the last one alone with its P summed by a launch of its
    own, the nine not).  Three quarters of P's directions are of small
    length, so that the last bits of a Gram matrix reach P^ (a condition number of some 1e4, squared, of 2^-53 is more than 2^-30)."""
    gen_ = torch.Generator(device="cuda").manual_seed(r + m + n)
    k = r // 4
    G = torch.randn(m, k, device="cuda", generator=gen_) @ torch.randn(k, n, device="cuda", generator=gen_)
    G += 1e-3 * torch.randn(m, n, device="cuda", generator=gen_)
    Q0 = torch.randn(n, r, device="cuda", generator=gen_)
    got = []
    for copies in (1, most):
        for knob in ("EDGC_TUNE_P", "EDGC_TUNE_Q"):
            monkeypatch.setenv(knob, str(copies))
        c = edgc.Context(0, max_bins=16, max_rank=r, max_rows=64, max_cols=64)
        c.reserve_batch([(m, n)] * copies)
        ts = []
        for _ in range(copies):
            Q = torch.zeros(n, (r + 3) // 4 * 4, device="cuda")
            Q[:, :r] = Q0
            ts.append(edgc.Tensor(G, torch.empty_like(G), torch.empty(m, n, device="cuda"), Q,
                                  torch.zeros(m, (r + 3) // 4 * 4, device="cuda"), True))
        c.compress_batch(ts, r)
        torch.cuda.synchronize()
        got += [(t.P, t.Q) for t in ts]
        c.close()
    for P, Q in got[1:]:
        assert torch.equal(P, got[0][0]) and torch.equal(Q, got[0][1])


@pytest.mark.parametrize("deferred", [False, True])
def test_prepared_descriptors_give_the_same_bits_as_a_list(deferred):
    """binding.PreparedBatch builds the descriptor array once and rewrites only the two per-call
    flags: three steps through it equal three steps through the plain list bit for bit."""
    shapes, r = [(512, 768), (256, 1024), (1024, 256)], 16
    a = Stage(shapes, r, "bf16", seed=5, deferred=deferred)
    b = Stage(shapes, r, "bf16", seed=5, deferred=deferred)
    prep = edgc.PreparedBatch(b.t)
    for step in range(3):
        a.step_device()
        b.ctx.compress_batch(prep, r, deferred=deferred and step > 0)
        b.ctx.decompress_batch(prep, r, deferred=deferred)
        torch.cuda.synchronize()
        for t in b.t:
            t.residual_is_zero = False
        for ta, tb in zip(a.t, b.t):
            assert torch.equal(ta.P, tb.P) and torch.equal(ta.Q, tb.Q)
            assert torch.equal(ta.residual, tb.residual) and torch.equal(ta.grad_out, tb.grad_out)


def test_batch_rejects_bad_descriptors_before_launching():
    st = Stage([(256, 256), (128, 384)], 8, "f32", seed=5)
    before = [t.P.clone() for t in st.t]
    big = edgc.Tensor(torch.zeros((300, 256), device="cuda"), torch.zeros((300, 256), device="cuda"),
                      torch.zeros((300, 256), device="cuda"), torch.zeros((256, 8), device="cuda"),
                      torch.zeros((300, 8), device="cuda"), True)
    with pytest.raises(edgc.EdgcError):                            # larger than its slot
        st.ctx.compress_batch([big, st.t[1]], 8)
    with pytest.raises(edgc.EdgcError):                            # more tensors than slots
        st.ctx.compress_batch(st.t + [st.t[0]], 8)
    with pytest.raises(edgc.EdgcError):                            # rank above the context's
        st.ctx.compress_batch(st.t, 129)
    bad = edgc.Tensor(st.t[1].grad, st.t[1].grad_out, None, st.t[1].Q, st.t[1].P, True)
    with pytest.raises(edgc.EdgcError):                            # second descriptor is bad:
        st.ctx.compress_batch([st.t[0], bad], 8)                   # nothing of the first may run
    torch.cuda.synchronize()
    for t, p in zip(st.t, before):
        assert torch.equal(t.P, p)
    with pytest.raises(TypeError):
        st.ctx.compress_batch([st.t[0], edgc.Tensor(st.t[1].grad.bfloat16(), st.t[1].grad_out.bfloat16())], 8)
    st.ctx.compress_batch([], 8)                                   # empty batch: nothing to do
    st.ctx.decompress_batch([], 8)


# ---------------------------------------------------------------------------
# stage-level entropy over separate buffers: the union of the buffers' own samples
# ---------------------------------------------------------------------------
def _oracle_union_entropy(bufs, stride, chunk, seed, step, bins, value_range=None):
    """Each buffer's sample by the oracle's sampler, gathered and concatenated; the oracle's
    estimator then runs over that vector with every element sampled."""
    parts = []
    for b in bufs:
        idx = orc.sample_indices(b.size, stride, chunk, seed, step)
        parts.append(b.reshape(-1)[idx])
    cat = np.concatenate(parts)
    return orc.entropy(cat, 1, 1, 0, 0, bins, value_range), cat.size


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("stride,chunk,bins", [(100, 64, 1024), (10, 1, 256), (1, 64, 4096), (7, 48, 65536)])
def test_stage_entropy_over_separate_buffers(dtype, stride, chunk, bins):
    sizes = [1 << 20, 300_007, 64, 1, 2_000_003, 4096]
    bufs = [gen.laplace_mixture(n, 40 + i, dtype=dtype, scale=1e-3 * (1 + i)) for i, n in enumerate(sizes)]
    dev = [to_dev(b) for b in bufs]
    c = edgc.Context(0, max_bins=65536, max_rank=4, max_rows=64, max_cols=64)
    counts = torch.zeros(bins, dtype=torch.int64, device="cuda")
    for step in (0, 5):
        got = c.entropy_estimate(dev, stride, chunk, 9, step, bins, counts_out=counts)
        want, n_s = _oracle_union_entropy(bufs, stride, chunk, 9, step, bins)
        assert got.n_sampled == n_s == want.n_sampled
        assert (got.lo, got.hi) == (want.lo, want.hi)
        assert np.array_equal(counts.cpu().numpy().astype(np.uint64), want.counts), "bin counts are bit-exact"
        assert abs(got.H_bits - want.H_bits) <= 1e-5 and abs(got.h_diff_nats - want.h_diff_nats) <= 1e-5
    # a caller's range, and one buffer that is not 16-byte aligned (the group falls back to scalar loads)
    odd = [dev[0][1:], dev[1]]
    odd_host = [bufs[0][1:], bufs[1]]
    got = c.entropy_estimate(odd, stride, chunk, 9, 3, bins, value_range=(-2e-3, 2e-3))
    want, n_s = _oracle_union_entropy(odd_host, stride, chunk, 9, 3, bins, (-2e-3, 2e-3))
    assert got.n_sampled == n_s and abs(got.H_bits - want.H_bits) <= 1e-5
    # one buffer through the batch call is the single call
    a = c.entropy_estimate([dev[0]], stride, chunk, 9, 1, bins)
    b = c.entropy_estimate(dev[0], stride, chunk, 9, 1, bins)
    assert a == b
    with pytest.raises(edgc.EdgcError):
        c.entropy_estimate([dev[0]] * 33, stride, chunk, 9, 1, bins)
    with pytest.raises(edgc.EdgcError):
        c.entropy_estimate([], stride, chunk, 9, 1, bins)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("stride,chunk,bins,given", [(1, 64, 257, False), (3, 64, 4096, False), (1, 64, 1024, True),
                                                     (2, 8, 16384, False), (1, 24, 20000, False)])
def test_stage_entropy_over_many_short_and_ragged_buffers(dtype, stride, chunk, bins, given):
    """Blocks take ranges of the union of the buffers: ranges that span many buffers, ends inside an item, samples of
    exactly one block's round (4096 items of 16 bytes) and one item more, and both sides of the bins that fit in LDS."""
    vec = 4 if dtype == "f32" else 8
    tail = vec - 1
    lens = [1, 7, 64, 65, 127, 128, 129, 768, 2304, 3072, 100, 4095, 333, 64 * 9 + 3, 5, 5000]
    groups = [lens, 2 * lens, [4096 * vec], [4096 * vec + tail], [4096 * vec - 64, 64, 1], 3 * [4096 * vec] + lens]
    c = edgc.Context(0, max_bins=65536, max_rank=4, max_rows=64, max_cols=64)
    counts = torch.zeros(bins, dtype=torch.int64, device="cuda")
    value_range = (-2e-3, 3e-3) if given else None
    for k, sizes in enumerate(groups):
        bufs = [gen.laplace_mixture(n, 90 + i, dtype=dtype) for i, n in enumerate(sizes)]
        bufs[0][-1] = 0x7fc0 if dtype == "bf16" else np.float32(np.nan)
        if bufs[-1].size > 1:
            bufs[-1][0] = 0xff80 if dtype == "bf16" else np.float32(-np.inf)
        got = c.entropy_estimate([to_dev(b) for b in bufs], stride, chunk, 9, k, bins, value_range, counts_out=counts)
        want, n_s = _oracle_union_entropy(bufs, stride, chunk, 9, k, bins, value_range)
        assert (got.n_sampled, got.n_nonfinite) == (n_s, want.n_nonfinite), k
        assert (got.lo, got.hi) == (want.lo, want.hi), k
        assert np.array_equal(counts.cpu().numpy().astype(np.uint64), want.counts), k
        # fp64 sums over the same integer counts in another order
        assert abs(got.H_bits - want.H_bits) <= 1e-5, k


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("off", [0, 1])
def test_stage_entropy_short_buffers_beside_a_large_one(dtype, off):
    """A block's range of several rounds that holds many short buffers and a part of a large one, at its front, in its
    middle and at its end; with `off` no buffer is aligned and items are single elements."""
    short = [768, 1, 2304, 65, 3072, 127, 4095, 64, 5, 333]
    big = 9_000_003
    c = edgc.Context(0, max_bins=65536, max_rank=4, max_rows=64, max_cols=64)
    for k, sizes in enumerate([short + [big], [big] + short, short + [big // 2] + 2 * short + [big // 2 + 64]]):
        bufs = [gen.laplace_mixture(n, 60 + i, dtype=dtype, scale=1e-3 * (1 + i % 3)) for i, n in enumerate(sizes)]
        dev = []
        for b in bufs:
            room = torch.zeros(b.size + 8, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
            room[off:off + b.size] = to_dev(b)
            dev.append(room[off:off + b.size])
        for stride, chunk, bins in [(1, 64, 4096), (3, 64, 65536)]:
            counts = torch.zeros(bins, dtype=torch.int64, device="cuda")
            got = c.entropy_estimate(dev, stride, chunk, 9, k, bins, counts_out=counts)
            want, n_s = _oracle_union_entropy(bufs, stride, chunk, 9, k, bins)
            assert got.n_sampled == n_s == want.n_sampled, (k, bins)
            assert (got.lo, got.hi) == (want.lo, want.hi), (k, bins)
            assert np.array_equal(counts.cpu().numpy().astype(np.uint64), want.counts), (k, bins)
            # fp64 sums over the same integer counts in another order
            assert abs(got.H_bits - want.H_bits) <= 1e-5, (k, bins)
    c.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("count", [1, 32, 33])
def test_tensors_sent_as_they_stand_are_copied_whole_and_nothing_else(dtype, count):
    """Vectors and matrices too small to compress, at every alignment and row stride the copy distinguishes, up to one
    more than one launch takes: each reconstruction is the gradient, and nothing around it is written."""
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    shapes = [(768,), (1,), (3071,), (16384 + 3,), (5, 7), (6, 200), (40000, 1), (3, 24), (9, 16)]
    g = torch.Generator(device="cuda").manual_seed(count)
    ts, outs, pads = [], [], []
    for i in range(count):
        s = shapes[i % len(shapes)]
        off, extra = [0, 1, 2, 3, 4, 8][i % 6], [0, 0, 1, 8][i % 4] if len(s) == 2 else 0
        rows, cols = s if len(s) == 2 else (1, s[0])
        def view(fill):
            buf = torch.full((off + rows * (cols + extra) + 8,), fill, device="cuda", dtype=tdt)
            v = buf[off:off + rows * (cols + extra)].view(rows, cols + extra)[:, :cols]
            return buf, (v if len(s) == 2 else v[0])
        _, grad = view(0.0)
        grad.copy_(torch.randn(grad.shape, generator=g, device="cuda"))
        buf, out = view(7.0)
        ts.append(edgc.Tensor(grad, out)); outs.append(out); pads.append(buf)
    c = edgc.Context(0, max_bins=16, max_rank=128, max_rows=64, max_cols=64)
    c.reserve_batch([tuple(t.grad.shape) if t.grad.dim() == 2 else (1, t.grad.numel()) for t in ts])
    c.decompress_batch(ts, 128)
    for t, out, buf in zip(ts, outs, pads):
        assert torch.equal(out, t.grad)
        written = int((buf != 7.0).sum())
        assert written == int((t.grad != 7.0).sum())


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("r", [65, 100, 128])
def test_blocks_of_every_height_of_the_multiply_by_the_inverse_factor(dtype, r, monkeypatch):
    """Above rank 64 that multiply takes 64, 128, 144 or 160 rows per block, by the rows of the launch.  A row's result does
    not depend on the block it is in, so all four give the same bits: rows that end inside a block, inside the 64 rows that
    a tensor is padded to, and at their edges."""
    shapes = [(145, 2600), (161, 2500), (320, 1000), (333, 900), (576, 700), (641, 650)]
    assert not any(edgc.tensor_bypassed(m, n, r) for m, n in shapes)
    mats = [gen.lowrank_plus_noise(m, n, 140, 0.97, 1e-4, seed=m + r, dtype=dtype) for m, n in shapes]
    q0 = []
    for i, (m, n) in enumerate(shapes):
        q = np.zeros((n, (r + 3) // 4 * 4), dtype=np.float32)
        orc.init_q(q, 0, r, 50 + i)
        q0.append(q)
    first = None
    for waves in (4, 8, 9, 10):
        monkeypatch.setenv("EDGC_TUNE_APPLY", str(waves))
        c = edgc.Context(0, max_bins=16, max_rank=128, max_rows=64, max_cols=64)
        c.reserve_batch(shapes)
        ts = []
        for g, q in zip(mats, q0):
            gd = to_dev(g)
            P = torch.full((g.shape[0], q.shape[1]), 7.0, device="cuda")
            ts.append(edgc.Tensor(gd, torch.empty_like(gd), torch.empty(g.shape, device="cuda"), to_dev(q), P, True))
        c.compress_batch(ts, r)
        torch.cuda.synchronize()
        got = [(t.P[:, :r].clone(), t.Q[:, :r].clone()) for t in ts]
        c.close()
        if first is None:
            first = got
            for g, q, (P, Q) in zip(mats, q0, got):
                Po, Qo, _ = orc.compress(g, None, q[:, :r].copy(), r)
                P64 = to_host(P).astype(np.float64)
                assert np.abs(P64.T @ P64 - np.eye(r)).max() < 1e-5
                assert rel_fro(to_host(P) @ to_host(Q).T, Po @ Qo.T) <= TOL[dtype]
        for a, b in zip(first, got):
            assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]), waves


def test_a_tensor_of_more_runs_than_blocks_is_copied_whole():
    """2^28 + 5 elements at 2-byte alignment: a run more than the 2^18 blocks a tensor gets, so one block copies two."""
    n = (1 << 28) + 5
    src, dst = (torch.empty(n + 8, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    src.view(torch.int16).random_(-30000, 30000)
    dst.fill_(7.0)
    t = edgc.Tensor(src[1:n + 1], dst[1:n + 1])
    c = edgc.Context(0, max_bins=16, max_rank=4, max_rows=64, max_cols=64)
    c.reserve_batch([(1, n)])
    c.decompress_batch([t], 4)
    torch.cuda.synchronize()
    assert torch.equal(dst[1:n + 1].view(torch.int16), src[1:n + 1].view(torch.int16))
    assert float(dst[0]) == 7.0 and bool((dst[n + 1:] == 7.0).all())
    c.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_stage_entropy_large_union_sample(dtype):
    """A union sample large enough for the launch shapes of large samples (one block of 1024 threads
    per compute unit, whole-item rounds with the next loads in flight) over several buffers of
    different sizes, with a ragged tail and a few non-finite values."""
    sizes = [(1 << 25) + 5, 1 << 24, (1 << 23) + 64, 12_345_679]
    bufs = [gen.laplace_mixture(n, 70 + i, dtype=dtype, scale=1e-3 * (1 + i)) for i, n in enumerate(sizes)]
    nan, inf = (0x7fc0, 0x7f80) if dtype == "bf16" else (np.float32(np.nan), np.float32(np.inf))
    bufs[0][12345] = nan
    bufs[1][-1] = inf
    bufs[3][7] = nan
    dev = [to_dev(b) for b in bufs]
    c = edgc.Context(0, max_bins=65536, max_rank=4, max_rows=64, max_cols=64)
    for stride, chunk, bins in [(1, 64, 4096), (1, 64, 65536), (3, 64, 1024)]:
        counts = torch.zeros(bins, dtype=torch.int64, device="cuda")
        got = c.entropy_estimate(dev, stride, chunk, 9, 2, bins, counts_out=counts)
        want, n_s = _oracle_union_entropy(bufs, stride, chunk, 9, 2, bins)
        assert got.n_sampled == n_s == want.n_sampled
        assert got.n_nonfinite == want.n_nonfinite and (stride != 1 or got.n_nonfinite == 3)
        assert (got.lo, got.hi) == (want.lo, want.hi)
        assert np.array_equal(counts.cpu().numpy().astype(np.uint64), want.counts), (stride, bins)
        assert int(counts.sum()) == n_s - got.n_nonfinite
        assert abs(got.H_bits - want.H_bits) <= 1e-5 and abs(got.h_diff_nats - want.h_diff_nats) <= 1e-5
    c.close()


# ---------------------------------------------------------------------------
# the batched calls under HIP graph capture: no allocation, no synchronisation, no memset
# node inside them, so a captured step replays like the eager one
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("deferred", [False, True])
def test_batched_step_replays_from_a_hip_graph(deferred):
    shapes, r = [(384, 512), (256, 640), (100,)], 8
    eager = Stage(shapes, r, "f32", seed=31, deferred=deferred)
    graphed = Stage(shapes, r, "f32", seed=31, deferred=deferred)
    for st in (eager, graphed):                       # first step eagerly: it starts from a zero residual
        st.step_device()
    side = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    keep = [(t.residual.clone(), t.Q.clone(), t.P.clone()) if t.residual is not None else None for t in graphed.t]
    ent_out = torch.zeros(edgc.binding.ENTROPY_RESULT_BYTES, dtype=torch.uint8, pin_memory=True)
    flats = [t.grad.view(-1) for t in graphed.t]
    with torch.cuda.graph(g, stream=side, capture_error_mode="thread_local"):
        graphed.ctx.entropy_estimate_async(flats, 10, 64, 3, 0, 256, ent_out, stream=side)
        graphed.ctx.compress_batch(graphed.t, r, stream=side, deferred=deferred)
        graphed.ctx.decompress_batch(graphed.t, r, stream=side, deferred=deferred)
    torch.cuda.synchronize()
    ent_want = graphed.ctx.entropy_estimate(flats, 10, 64, 3, 0, 256)
    for t, k in zip(graphed.t, keep):                 # capture runs nothing, but make the state explicit
        if k is not None:
            t.residual.copy_(k[0]); t.Q.copy_(k[1]); t.P.copy_(k[2])
    for step in range(3):
        eager.step_device()
        g.replay()
        # eager work and a synchronisation between replays
        torch.cuda.synchronize()
        _ = (eager.t[0].grad_out * 2).sum().item()
        assert edgc.EntropyResult.from_buffer(ent_out.numpy().tobytes()) == ent_want, step
        ent_out.zero_()
        for a, b in zip(eager.t, graphed.t):
            assert torch.equal(a.grad_out, b.grad_out), step
            if a.residual is not None:
                assert torch.equal(a.residual, b.residual) and torch.equal(a.Q, b.Q) and torch.equal(a.P, b.P), step


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("r,count,deferred", [(8, 1, False), (8, 16, True), (40, 17, False), (100, 5, True), (100, 33, False), (8, 0, True)])
def test_copies_at_the_head_of_the_decompress(dtype, r, count, deferred):
    """Tensors sent as they stand between compressed ones, fewer and more than one launch takes, before the general kernel and
    (rank 100, deferred) the whole-tile one: every copy is the gradient, and the compressed ones get what they get without copies."""
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(count + r)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda")
    ld = (r + 3) // 4 * 4

    def matrix(m, n):
        D, P, Q = rand(m, n), torch.zeros(m, ld, device="cuda"), torch.zeros(n, ld, device="cuda")
        P[:, :r], Q[:, :r] = rand(m, r), rand(n, r)
        return edgc.Tensor(None, torch.empty(m, n, device="cuda", dtype=tdt), D, Q, P)

    def vector(i):
        n, off = [1, 768, 3071, 16387][i % 4], [0, 1, 2, 8][i // 4 % 4]
        src, dst = rand(n + off).to(tdt)[off:], torch.empty(n + off + 8, device="cuda", dtype=tdt)[off:off + n]
        return edgc.Tensor(src, dst)

    mats = [matrix(512, 640), matrix(768, 512)]
    alone = [edgc.Tensor(None, torch.empty_like(t.grad_out), t.residual.clone(), t.Q, t.P) for t in mats]
    vecs = [vector(i) for i in range(count)]
    ts = vecs[:count // 2] + mats[:1] + vecs[count // 2:] + mats[1:]
    c = edgc.Context(0, max_bins=16, max_rank=128, max_rows=64, max_cols=64)
    for batch in (ts, alone):
        c.reserve_batch([tuple(t.grad_out.shape) if t.grad_out.dim() == 2 else (1, t.grad_out.numel()) for t in batch])
        c.decompress_batch(batch, r, deferred=deferred)
    for t in vecs:
        assert torch.equal(t.grad_out, t.grad)
    for t, u in zip(mats, alone):
        assert torch.equal(t.grad_out, u.grad_out) and torch.equal(t.residual, u.residual)
    c.close()


def _launches(call):
    """Nodes of the graph that `call(stream)` is captured into."""
    import ctypes
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    hip, side, graph, nodes = ctypes.CDLL(path), torch.cuda.Stream(), ctypes.c_void_p(), ctypes.c_size_t()
    torch.cuda.synchronize()
    assert hip.hipStreamBeginCapture(ctypes.c_void_p(side.cuda_stream), 2) == 0
    try:
        call(side)
    finally:
        assert hip.hipStreamEndCapture(ctypes.c_void_p(side.cuda_stream), ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(nodes)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return nodes.value


@pytest.mark.parametrize("kind,count,matrices,launches", [
    ("runs", 16, None, 1), ("runs", 17, None, 1), ("runs", 32, None, 1), ("runs", 33, None, 2),
    ("rows", 16, None, 1), ("rows", 17, None, 1), ("rows", 32, None, 1), ("rows", 33, None, 2), ("both", 64, None, 2), ("both", 66, None, 4),
    ("runs", 16, (512, 640), 1), ("runs", 17, (512, 640), 2), ("runs", 32, (512, 640), 2), ("runs", 33, (512, 640), 2), ("runs", 49, (512, 640), 3),
    ("both", 10, (512, 640), 2), ("both", 40, (512, 640), 3), ("rows", 33, (512, 640), 3), ("both", 10, (511, 641), 3), ("runs", 20, (511, 641), 2)])
def test_launches_of_the_copies(kind, count, matrices, launches):
    """Contiguous tensors sent as they stand and ones whose rows are apart: up to 32 of each in a launch, up to 16 contiguous ones in the
    decompress's own where its rows are whole cache lines.  Every copy is the gradient and nothing around it is written."""
    g = torch.Generator(device="cuda").manual_seed(count)
    ts, pads = [], []
    for i in range(count):
        rows, cols, extra, off = (7, 3 + i % 5, 1 + i % 8, i % 4) if kind == "rows" or (kind == "both" and i % 2) else (1, 100 + i, 0, i % 4)
        def view(fill):
            buf = torch.full((off + rows * (cols + extra) + 8,), fill, device="cuda")
            return buf, buf[off:off + rows * (cols + extra)].view(rows, cols + extra)[:, :cols]
        grad, (buf, out) = view(0.0)[1], view(7.0)
        grad.copy_(torch.randn(rows, cols, generator=g, device="cuda"))
        ts.append(edgc.Tensor(grad, out)); pads.append(buf)
    r, mats = 64, []
    if matrices:
        m, n = matrices
        for _ in range(2):
            D, P, Q = (torch.randn(*s, generator=g, device="cuda") for s in ((m, n), (m, r), (n, r)))
            mats.append(edgc.Tensor(None, torch.empty(m, n, device="cuda"), D, Q, P))
    ts = ts[:count // 2] + mats + ts[count // 2:]
    want = [t.residual - t.P @ t.Q.t() for t in mats]
    c = edgc.Context(0, max_bins=16, max_rank=r, max_rows=64, max_cols=64)
    c.reserve_batch([tuple(t.grad_out.shape) for t in ts])
    assert _launches(lambda s: c.decompress_batch(ts, r, stream=s)) == launches
    c.decompress_batch(ts, r)
    copied = [t for t in ts if t.grad is not None]
    for t, buf in zip(copied, pads):
        assert torch.equal(t.grad_out, t.grad)
        assert int((buf != 7.0).sum()) == int((t.grad != 7.0).sum())
    for t, e in zip(mats, want):
        assert float((t.residual - e).norm() / e.norm()) < 1e-4        # operands of 17 bits: 2^-16 of |P| |Q|, which |E| exceeds
    c.close()


@pytest.mark.parametrize("count", [0, 16, 17])
def test_profile_credits_the_copies_that_ride_in_the_decompress(count):
    """Their time is in the decompress's, so their bytes are: read and written; a launch of their own is not profiled."""
    m, n, r, k = 512, 640, 8, 100_000
    D, P, Q = torch.zeros(m, n, device="cuda"), torch.zeros(m, r, device="cuda"), torch.zeros(n, r, device="cuda")
    ts = [edgc.Tensor(torch.zeros(k, device="cuda"), torch.empty(k, device="cuda")) for _ in range(count)]
    ts.append(edgc.Tensor(None, torch.empty(m, n, device="cuda"), D, Q, P))
    c = edgc.Context(0, max_bins=16, max_rank=r, max_rows=64, max_cols=64)
    c.reserve_batch([(1, k)] * count + [(m, n)])
    c.profile_begin(16)
    c.decompress_batch(ts, r)
    assert c.profile_end()["k_decompress"]["bytes"] == 12 * m * n + (8 * k * count if count <= 16 else 0)
    c.close()


def test_calls_without_a_stream_use_torchs_current_one():
    from paper_2511_10333_amd.binding import _stream_handle
    assert _stream_handle(None) == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert _stream_handle(None) == side.cuda_stream
    assert _stream_handle(side) == side.cuda_stream and _stream_handle(None) == torch.cuda.current_stream().cuda_stream
