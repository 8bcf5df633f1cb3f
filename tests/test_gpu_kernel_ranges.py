"""Kernels at the edges of the size ranges their dispatch rules cut, against the float64 oracle."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle.objectives import LeastSquares, MixtureMLP
from helpers import ALGORITHM1_RUNS, TOL_GEMM, assert_close, make_both

pytestmark = pytest.mark.gpu


def lsq_swarm(gpu, n, d, m, batch, H, geometric, seed, inplace=False):
    A, b, _ = wl.least_squares_data(n, d, m, seed)
    edges = wl.complete_graph(n) if n < 16 else wl.random_regular_graph(n, 4, 0)
    g, c = make_both(gpu, n, d, edges, 8, 2.0 ** -6, H, 0.05, 0, seed=seed, geometric=geometric, inplace=inplace)
    c.objective = LeastSquares(A, b, batch)
    g.set_objective_lsq(torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda(), m, batch)
    gen = np.random.Generator(np.random.PCG64(seed))
    c.X[:] = gen.standard_normal((n, d)).astype(np.float32)
    g.write_models(gpu.COMM, c.X)
    return g, c


# n x ceil(d / 512) > 256: one workgroup takes a node alone, from 256 nodes on, from 128 up to 16384 columns, from 65 up to 2048 and
# from 3080 to 4096 columns (256, 512 or 1024 threads, or a wave per row), or teams of workgroups take one node after the other: all
# others, and of these 64 rows from 2048 columns on, 32 from 4096 and 16 from 16384
@pytest.mark.parametrize("n,d,m,batch,H,geometric", [
    (129, 1024, 8, 4, 2, False), (129, 1032, 8, 20, 3, False), (40, 4096, 40, 64, 1, False), (9, 8 * 2051, 33, 16, 2, True),
    (2, 8 * 33001, 17, 12, 2, False), (255, 8 * 1300, 6, 32, 2, False),
    (257, 512, 9, 4, 3, True), (256, 1032, 8, 36, 2, False), (260, 16384 + 8, 5, 16, 2, False),
    (65, 2048, 8, 12, 2, False), (65, 2056, 8, 16, 2, True), (65, 3080, 7, 20, 2, False), (127, 4104, 5, 16, 2, False),
    (128, 16384, 4, 8, 2, False), (128, 16392, 4, 8, 2, False), (500, 1536, 4, 16, 2, False), (500, 3072, 4, 60, 2, True),
    (257, 3080, 5, 64, 2, False), (384, 4096, 4, 16, 3, True), (300, 6152, 4, 32, 2, False), (260, 12288, 4, 12, 2, False),
    (225, 4096, 5, 48, 2, False)])
def test_wide_least_squares_steps(gpu, n, d, m, batch, H, geometric):
    g, c = lsq_swarm(gpu, n, d, m, batch, H, geometric, seed=n)
    nodes = sorted({n - 1, 0, n // 2}, reverse=True)
    for node in nodes:
        c.local_steps([node])
    g.local_steps(nodes)
    some = g.read_models(gpu.LIVE)[nodes]
    assert_close(some, c.W[nodes], TOL_GEMM, "steps of a few nodes")
    g.write_models(gpu.COMM, c.X)                          # clears the pending marks, same round: same draws
    g.local_steps()
    assert np.array_equal(g.read_models(gpu.LIVE)[nodes], some)        # the same sums whatever the launch carries


# The wide form with several workgroups per node (blocks of 1024 columns, one or more per slice, ragged or a whole number) and a launch
# per step: where not one team fits the chip, where teams would need a second round for a few rows, and where the steps update the
# models themselves; so also the forms of one workgroup per node that teams take otherwise.  One workgroup beyond 16384 columns
@pytest.mark.parametrize("n,d,m,batch,H,geometric", [
    (2, 8 * 41001, 5, 64, 2, False), (2, 8 * 131080, 4, 4, 3, True), (64, 16384, 4, 8, 1, False), (70, 14000, 4, 4, 3, False),
    (260, 16392, 4, 12, 2, False)])
def test_wide_least_squares_steps_beside_teams(gpu, n, d, m, batch, H, geometric):
    test_wide_least_squares_steps(gpu, n, d, m, batch, H, geometric)


@pytest.mark.parametrize("n,d,m,batch,H,geometric", [
    (9, 8 * 2051, 33, 16, 2, True), (64, 8200, 5, 64, 3, False), (2, 8 * 33001, 17, 12, 2, False), (255, 8 * 1300, 6, 32, 2, False),
    (300, 4096, 5, 64, 2, False), (80, 4096, 5, 60, 2, True), (260, 16392, 5, 16, 2, False)])
def test_least_squares_steps_that_update_the_models_themselves(gpu, n, d, m, batch, H, geometric):
    g, c = lsq_swarm(gpu, n, d, m, batch, H, geometric, seed=n, inplace=True)
    nodes = sorted({n - 1, 0, n // 2}, reverse=True)
    start = c.X.copy()
    for node in nodes:
        c.local_steps([node])
    g.local_steps(nodes)
    some = g.read_models(gpu.COMM)
    assert_close(some[nodes], c.X[nodes], TOL_GEMM, "steps of a few nodes")
    others = np.setdiff1d(np.arange(n), nodes)
    assert np.array_equal(some[others], start[others])
    g.write_models(gpu.COMM, start)
    g.local_steps()
    assert np.array_equal(g.read_models(gpu.COMM)[nodes], some[nodes])         # the same sums whatever the launch carries


# n x ceil(d / 512) <= 256: a workgroup per slice of 512 columns.  One, four or sixteen rows per wave and one, two or more requests
# for the words of 1, 5, 9, 33 and 128 slices; a request takes 16, 8 or 4 of them by the batch
@pytest.mark.parametrize("n,d,m,batch,H,geometric", [
    (3, 8, 5, 4, 3, False), (256, 512, 5, 12, 1, False), (4, 2568, 9, 20, 3, True), (28, 4104, 8, 16, 2, False),
    (7, 16408, 9, 36, 2, False), (7, 16408, 9, 16, 2, False), (2, 65536, 6, 64, 2, False), (2, 65512, 6, 28, 3, False)])
def test_split_least_squares_steps(gpu, n, d, m, batch, H, geometric):
    test_wide_least_squares_steps(gpu, n, d, m, batch, H, geometric)


# Teams: two, four, eight or sixteen rows per wave of full and other batches, one, two and four blocks of columns, ragged slices; one node
# after the other (64 nodes of 33 slices) and all at once; one and several reducing workgroups
TEAM_STEPS = [(64, 8200, 5, 64, 2, False), (64, 8200, 5, 60, 2, True), (40, 16392, 6, 32, 2, False), (40, 16392, 6, 20, 2, False),
              (64, 12296, 5, 16, 3, False), (33, 4104, 5, 12, 1, False), (64, 8200, 5, 8, 2, False), (35, 4104, 5, 4, 2, True), (2, 8 * 9001, 6, 64, 3, False), (9, 131072, 5, 32, 2, False), (66, 4096, 5, 32, 2, False),
              (300, 2056, 5, 64, 2, True), (257, 16392, 4, 16, 2, False)]


@pytest.mark.parametrize("n,d,m,batch,H,geometric", TEAM_STEPS)
def test_least_squares_steps_by_teams(gpu, n, d, m, batch, H, geometric):
    test_wide_least_squares_steps(gpu, n, d, m, batch, H, geometric)


# Workgroups that do not wait: one takes what is left of a team's nodes by itself, the sums are the same bits, and the next launch
# starts from the numbers this one has left.  One, two and sixteen workgroups that add rows
@pytest.mark.parametrize("n,d,m,batch,H,geometric", [
    (34, 8200, 5, 64, 3, False), (40, 8200, 6, 20, 2, True), (33, 4104, 5, 12, 2, False), (2, 8 * 9001, 6, 64, 3, False)])
def test_least_squares_steps_by_teams_whose_workgroups_do_not_wait(gpu, n, d, m, batch, H, geometric):
    g, _ = lsq_swarm(gpu, n, d, m, batch, H, geometric, seed=n)
    h, _ = lsq_swarm(gpu, n, d, m, batch, H, geometric, seed=n)
    X = g.read_models(gpu.COMM)
    for ticks in (2000000, 0, 200, 2000, 2000000):
        g.lsq_patience(ticks)
        for s in (g, h):
            s.write_models(gpu.COMM, X)
            s.write_models(gpu.LIVE, np.full_like(X, np.nan))
            s.local_steps()
        assert np.array_equal(g.read_models(gpu.LIVE), h.read_models(gpu.LIVE)), ticks
    g.counters()


# Two swarms on streams of their own take turns, from two threads
def test_least_squares_steps_by_teams_of_two_swarms_at_once(gpu):
    import threading
    swarms = [lsq_swarm(gpu, 16, 16392, 5, 64, 2, False, seed=s)[0] for s in (1, 2)]
    want = []
    for s in swarms:
        s.local_steps()
        want.append(s.read_models(gpu.LIVE))
    X = [s.read_models(gpu.COMM) for s in swarms]
    got = [None, None]

    def work(k):
        for _ in range(20):
            swarms[k].write_models(gpu.COMM, X[k])
            swarms[k].local_steps()
        got[k] = swarms[k].read_models(gpu.LIVE)
    threads = [threading.Thread(target=work, args=(k,)) for k in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k in (0, 1):
        assert np.array_equal(got[k], want[k])
        swarms[k].counters()


def test_wide_least_squares_batched_algorithm1_equals_single_steps(gpu):
    n, d = 9, 8 * 2051
    pair = [lsq_swarm(gpu, n, d, 33, 16, 2, True, seed=4)[0] for _ in range(2)]
    pairs, _ = pair[0].run_sequential(24)
    for i, j in pairs:
        assert pair[1].sample_pair() == (i, j)
        pair[1].interact(i, j)
    for which in (gpu.COMM, gpu.SNAP):
        assert np.array_equal(pair[0].read_models(which), pair[1].read_models(which))


def diag_swarm(gpu, n, d, bits, H, sigma, seed, geometric=False, objective=True):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    a = torch.rand(n, d, generator=gen, device="cuda") + 0.5
    c = torch.randn(n, d, generator=gen, device="cuda")
    s = gpu.Swarm(n, d, wl.complete_graph(n), bits, {0: 1.0, 4: 0.5}.get(bits, 2.0 ** -4), H, 0.1, 0, seed,
                  steps_law=gpu.GEOMETRIC if geometric else gpu.CONSTANT)
    if objective:
        s.set_objective_diag(a, c, sigma)
    X = torch.randn(n, d, generator=gen, device="cuda")
    s.models_view(gpu.COMM).copy_(X)
    s.models_view(gpu.SNAP).copy_(X + 0.01 * c)
    if not objective:
        s.models_view(gpu.LIVE).copy_(X - 0.02 * c)
        s.mark_pending()
    return s


# runs of Algorithm 1 in one launch and by levels (which of them takes which: tests/test_host_calls.py) equal one call per
# interaction, bit for bit
@pytest.mark.parametrize("n,d,bits,H,sigma,geometric,objective", [run[:-1] for run in ALGORITHM1_RUNS])
def test_run_of_algorithm1_in_one_launch(gpu, n, d, bits, H, sigma, geometric, objective):
    one, run = (diag_swarm(gpu, n, d, bits, H, sigma, 3, geometric, objective) for _ in range(2))
    count = 3 * n + 1
    pairs, levels = run.run_sequential(count)
    assert 1 < levels <= count
    for i, j in pairs:
        assert one.sample_pair() == (i, j)
        one.interact(i, j)
    for which in (gpu.COMM, gpu.SNAP):
        assert np.array_equal(run.read_models(which), one.read_models(which))
    if bits:
        for node in range(n):
            assert np.array_equal(run.read_codes(node), one.read_codes(node))
    assert run.counters(raise_on_range=False) == one.counters(raise_on_range=False)


def test_run_of_algorithm1_longer_than_one_upload(gpu):
    """32768 interactions are described per upload: a longer run goes on from where the upload before it ended."""
    whole, parts = (diag_swarm(gpu, 2, 16, 8, 1, 0.1, 6) for _ in range(2))
    whole.run_sequential(33000)
    for _ in range(11):
        parts.run_sequential(3000)
    for which in (gpu.COMM, gpu.SNAP):
        assert np.array_equal(whole.read_models(which), parts.read_models(which))
    assert np.array_equal(whole.read_codes(1), parts.read_codes(1)) and whole.counters() == parts.counters()


# Products in float32 by tiles of 64 x 64 (batch up to 64, and over 128), 128 x 64 and, from 512 tiles on, 128 x 128, each with
# whole and ragged edges; updates down the rows, over 128 samples by tiles of 64 x 64 (of 128 x 128: below).  The hidden bias rides
# in the backward product only when one tile holds the batch.
@pytest.mark.parametrize("arithmetic", ["fp32", "bf16x3"])
@pytest.mark.parametrize("n,n_in,n_hid,n_out,batch", [
    (3, 32, 32, 32, 32), (3, 64, 96, 160, 64), (2, 96, 352, 64, 96), (2, 160, 128, 32, 128), (2, 64, 224, 96, 160),
    (2, 32, 160, 32, 192), (130, 32, 512, 32, 128), (65, 32, 544, 544, 32)])
def test_mlp_tiles(gpu, n, n_in, n_hid, n_out, batch, arithmetic):
    d = n_hid * n_in + n_hid + n_out * n_hid + n_out
    means, cdf = wl.mixture_data(n, n_in, n_out, 1)
    edges = wl.complete_graph(n) if n < 16 else wl.random_regular_graph(n, 4, 0)
    g, c = make_both(gpu, n, d, edges, 8, 2.0 ** -10, 2, 0.05, 0, seed=n)
    c.objective = MixtureMLP(n_in, n_hid, n_out, means, cdf, 0.5, batch)
    g.set_objective_mlp(n_in, n_hid, n_out, torch.from_numpy(means).cuda(), torch.from_numpy(cdf).cuda(), 0.5, batch)
    g.set_mlp_arithmetic(gpu.MLP_BF16X3 if arithmetic == "bf16x3" else gpu.MLP_FP32)
    gen = np.random.Generator(np.random.PCG64(n))
    c.X[:] = (0.1 * gen.standard_normal((n, d))).astype(np.float32)
    g.write_models(gpu.COMM, c.X)
    nodes = sorted({0, n // 2, n - 1})
    c.local_steps(nodes)
    g.local_steps()
    W, want = g.read_models(gpu.LIVE)[nodes].astype(np.float64), c.W[nodes]
    # A hidden unit whose pre-activation is within rounding of zero for some sample may be on for one side and off for the
    # other: within TOL_GEMM, the bar of any product here (the terms that bf16x3 drops, 2^-16 |x w| each with random signs,
    # add up to 2e-5 over 544 of them at |x| = 2, |w| = 0.1).  That moves an entry of its row of W1 (or b1) by
    # eta / batch |sum_o dlogits_o W2_o| |x|, at most eta / batch * 2 max|W2| * max(1, max|x|), features are within
    # 4.9 sigma of a mean; everything else, biases and whole rows, is compared as is.
    near_zero = np.zeros((len(nodes), n_hid), dtype=bool)
    for k, node in enumerate(nodes):
        w = c.X[node].astype(np.float64)
        for q in range(2):
            x, _ = c.objective.batch_data(node, n, 0, q)
            W1, b1, _, _ = c.objective.split(w)
            near_zero[k] |= (np.abs(x @ W1.T + b1) < TOL_GEMM).any(axis=0)
            w = w - 0.05 * c.objective.gradient(node, w, n, 0, q)
    w2 = np.abs(c.X[:, n_hid * n_in + n_hid:-n_out]).max()
    kink = 2 * 0.05 / batch * 2 * w2 * (np.abs(means).max() + 4.9 * 0.5)
    off = np.abs(W - want) > TOL_GEMM * np.maximum(1.0, np.abs(want))
    assert not off[:, n_hid * n_in + n_hid:].any() and off.mean() < 1e-3
    units = off[:, :n_hid * n_in].reshape(len(nodes), n_hid, n_in).any(axis=2) | off[:, n_hid * n_in:n_hid * n_in + n_hid]
    strays = int((units & ~near_zero).sum())
    assert strays == 0 and near_zero.mean() < 0.1
    assert np.abs(W - want)[off].max(initial=0.0) <= kink


# Updates in float32 over 128 samples by tiles of 128 x 128, from 256 of them on: ragged, and whole beside ragged ones
@pytest.mark.parametrize("n,n_in,n_hid,n_out,batch", [(130, 32, 512, 32, 160), (65, 128, 512, 160, 160)])
def test_mlp_float_updates_in_large_tiles(gpu, n, n_in, n_hid, n_out, batch):
    test_mlp_tiles(gpu, n, n_in, n_hid, n_out, batch, "fp32")


# The bf16x3 steps in their forms: updates inside the products for 32 to 128 samples (eight waves per workgroup at 128) with whole
# and ragged groups of columns and odd numbers of slabs, apart at 160, batches in chunks of one block (several: below); logits split
# 8 ways and not at all; rows of the softmax beyond what its lanes hold.
@pytest.mark.parametrize("n,n_in,n_hid,n_out,batch", [
    (100, 96, 224, 64, 32), (50, 160, 512, 96, 64), (70, 64, 384, 32, 96), (26, 32, 1024, 160, 128), (40, 128, 640, 96, 160),
    (2, 64, 96, 64, 352), (3, 96, 1056, 544, 96), (2, 64, 96, 2144, 64)])
def test_mlp_forms_from_bf16_operands(gpu, n, n_in, n_hid, n_out, batch):
    test_mlp_tiles(gpu, n, n_in, n_hid, n_out, batch, "bf16x3")
    d = n_hid * n_in + n_hid + n_out * n_hid + n_out
    means, cdf = wl.mixture_data(n, n_in, n_out, 1)
    s = gpu.Swarm(n, d, wl.complete_graph(n) if n < 16 else wl.random_regular_graph(n, 4, 0), 8, 2.0 ** -10, 2, 0.05, 0, n)
    s.set_objective_mlp(n_in, n_hid, n_out, torch.from_numpy(means).cuda(), torch.from_numpy(cdf).cuda(), 0.5, batch)
    s.set_mlp_arithmetic(gpu.MLP_BF16X3)
    X = torch.randn(n, d, generator=torch.Generator(device="cuda").manual_seed(n), device="cuda").mul_(0.1)
    s.models_view(gpu.COMM).copy_(X)
    s.local_steps()
    whole = s.models_view(gpu.LIVE).clone()
    some = [n - 1, 0]
    s.models_view(gpu.LIVE).zero_()
    s.local_steps(some)                     # the same bits whoever steps along
    assert torch.equal(s.models_view(gpu.LIVE)[some], whole[some])


# Batches in chunks (tests/test_host_calls.py: which): five blocks of 32 samples per workgroup, 4 + 3, 5 + 4, 4 + 4 + 3, the
# backward product apart from the update; the few nodes of the second call take other chunks, and the same bits.  Updates of long
# batches by tiles of 128 x 128, whole and ragged, and of 64 x 64 for few nodes.  Softmax of more than 256 blocks of rows, up to 1024
# classes and beyond.
@pytest.mark.parametrize("n,n_in,n_hid,n_out,batch", [
    (64, 32, 512, 32, 160), (64, 32, 512, 32, 224), (64, 32, 512, 32, 288), (64, 32, 512, 32, 352), (65, 128, 512, 160, 224),
    (33, 32, 32, 1120, 256)])
def test_mlp_products_in_chunks(gpu, n, n_in, n_hid, n_out, batch):
    test_mlp_forms_from_bf16_operands(gpu, n, n_in, n_hid, n_out, batch)


def test_bf16x3_steps_where_memory_is_short(gpu):
    """With too little memory for the workspace of all nodes they step in groups: the same bits."""
    n, n_in, n_hid, n_out, batch = 45, 256, 1024, 256, 1024         # 360 MiB of workspace
    d = n_hid * n_in + n_hid + n_out * n_hid + n_out
    means, cdf = wl.mixture_data(n, n_in, n_out, 1)
    means, cdf = torch.from_numpy(means).cuda(), torch.from_numpy(cdf).cuda()

    def steps(leave):
        s = gpu.Swarm(n, d, wl.random_regular_graph(n, 4, 0), 8, 2.0 ** -10, 2, 0.05, 0, n)
        s.set_objective_mlp(n_in, n_hid, n_out, means, cdf, 0.5, batch)
        X, W = s.models_view(gpu.COMM), s.models_view(gpu.LIVE)
        X.copy_(torch.randn(n, d, generator=torch.Generator(device="cuda").manual_seed(n), device="cuda").mul_(0.1))
        torch.cuda.empty_cache()
        taken, free = [], torch.cuda.mem_get_info()[0]
        while leave and free - leave > 4 << 20:
            taken.append(torch.empty(min(free - leave, 16 << 30), dtype=torch.uint8, device="cuda"))
            free = torch.cuda.mem_get_info()[0]
        s.set_mlp_arithmetic(gpu.MLP_BF16X3)
        used = free - torch.cuda.mem_get_info()[0]
        s.local_steps()
        torch.cuda.synchronize()
        del taken
        torch.cuda.empty_cache()
        return W.clone(), used, s

    whole, used, s = steps(None)
    short, used_short, s_short = steps(160 << 20)
    assert used > 300 << 20 and used_short <= 160 << 20
    assert torch.equal(short, whole)
    some = [44, 3]                                                   # fewer than a group, by a list
    s.local_steps(some)
    s_short.local_steps(some)
    assert torch.equal(s.models_view(gpu.LIVE)[some], s_short.models_view(gpu.LIVE)[some])
    s.close()
    s_short.close()


def test_mlp_contraction_of_more_than_4_gib_of_packed_features(gpu):
    """2^20 + 1 slabs of 32 features and 4 KiB each, the weights of all but the last slab zero: a 32-bit byte offset would come
    round to the first slab's features.  The update of W2 shows the hidden activations; against the float32 arithmetic, whose
    addresses are others, at the bar of the products."""
    n, n_in, n_hid, n_out, batch = 2, 32 * (2 ** 20 + 1), 32, 32, 32
    d = n_hid * n_in + n_hid + n_out * n_hid + n_out
    gen = torch.Generator(device="cuda").manual_seed(3)
    means = torch.randn(n_out, n_in, generator=gen, device="cuda")
    cdf = (torch.arange(1, n_out + 1, device="cuda") / n_out).float().repeat(n, 1).contiguous()
    s = gpu.Swarm(n, d, [[0, 1]], 8, 2.0 ** -10, 1, 0.05, 0, 1)
    s.set_objective_mlp(n_in, n_hid, n_out, means, cdf, 0.1, batch)
    X, W = s.models_view(gpu.COMM), s.models_view(gpu.LIVE)
    W2 = slice(n_hid * n_in + n_hid, d - n_out)
    for i in range(n):
        X[i].zero_()
        X[i, :n_hid * n_in].view(n_hid, n_in)[:, -32:].normal_(0.0, 0.2, generator=gen)
        X[i, W2].normal_(0.0, 0.2, generator=gen)
    step = []
    for arithmetic in (gpu.MLP_FP32, gpu.MLP_BF16X3):
        s.set_mlp_arithmetic(arithmetic)
        s.local_steps()
        step.append((W[:, W2] - X[:, W2]).double())
    assert step[0].norm() > 1e-3 and (step[1] - step[0]).norm() < TOL_GEMM * step[0].norm()
    s.close()


# small least-squares swarms: a run of Algorithm 1 in one launch (graphs that let at most seven interactions run side by
# side, up to 64 groups of 128 columns, batch 32 and 2048 words exchanged per step: tests/test_host_calls.py); beyond each
# of these limits (64 and 65 nodes of a 4-regular graph among them) the form with a launch per level
@pytest.mark.parametrize("n,d,m,batch,H,bits,geometric", [
    (2, 8, 5, 4, 1, 8, False), (3, 136, 20, 12, 3, 2, True), (8, 1032, 30, 16, 2, 4, False), (5, 2600, 40, 20, 2, 16, True),
    (4, 8192, 16, 32, 1, 8, False), (24, 512, 9, 32, 2, 8, False), (64, 512, 9, 32, 2, 0, False), (65, 512, 9, 32, 2, 8, False), (5, 1024, 70, 36, 2, 8, False),
    (4, 8200, 16, 16, 1, 8, False)])
def test_least_squares_run_in_one_launch(gpu, n, d, m, batch, H, bits, geometric):
    A, b, _ = wl.least_squares_data(n, d, m, 2)
    edges = wl.complete_graph(n) if n < 16 else wl.random_regular_graph(n, 4, 0)
    eps = 2.0 ** -6 if bits > 2 else 0.5
    gen = np.random.Generator(np.random.PCG64(n))
    X = (gen.standard_normal((1, d)) + 0.05 * gen.standard_normal((n, d))).astype(np.float32)
    pair = []
    for _ in range(2):
        g, c = make_both(gpu, n, d, edges, bits, eps, H, 0.05, 0, seed=9, geometric=geometric)
        g.set_objective_lsq(torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda(), m, batch)
        g.write_models(gpu.COMM, X)
        g.write_models(gpu.SNAP, X + np.float32(0.01))
        pair.append(g)
    run, one = pair
    c.objective = LeastSquares(A, b, batch)
    c.X[:], c.Xhat[:] = X, X + np.float32(0.01)
    # the first interaction against the oracle: same state, so codes are the same bits
    i, j = c.step_sequential()
    pairs, _ = run.run_sequential(1)
    assert tuple(pairs[0]) == (i, j)
    assert_close(run.read_models(gpu.COMM), c.X, TOL_GEMM, "X after one interaction")
    assert_close(run.read_models(gpu.SNAP), c.Xhat, TOL_GEMM, "snapshots after one interaction")
    assert_close(run.read_models(gpu.LIVE)[i], c.W[i], TOL_GEMM, "W_i after one interaction")
    if bits:
        for node in (i, j):
            assert np.array_equal(run.read_codes(node), c.ring[0][node])
    # the rest of the run against one call per interaction
    one.interact(i, j)
    for t in (3 * n, 2):
        pairs, _ = run.run_sequential(t)
        for i, j in pairs:
            assert one.sample_pair() == (i, j)
            one.interact(i, j)
    for which in (gpu.COMM, gpu.SNAP, gpu.LIVE):
        assert np.array_equal(run.read_models(which), one.read_models(which))
    if bits:
        for node in range(n):
            assert np.array_equal(run.read_codes(node), one.read_codes(node))
    assert run.counters(raise_on_range=False) == one.counters(raise_on_range=False)


# several initiators, both parities of the exchanged words and all four waves of a workgroup, against the oracle.  Exchanged
# unrounded (bits = 0): a rounding decision that differs in the last bit would move the models by a whole lattice step.
# The bar of one GEMM-based step holds for the run: the steps contract (eta m / batch |A_B|^2 < 2), and averaging halves errors.
@pytest.mark.parametrize("n,d,m,batch,H,count", [(5, 1032, 20, 16, 3, 16), (8, 4096, 64, 32, 2, 16), (3, 136, 12, 4, 1, 12)])
def test_short_least_squares_run_against_the_oracle(gpu, n, d, m, batch, H, count):
    A, b, _ = wl.least_squares_data(n, d, m, 5)
    g, c = make_both(gpu, n, d, wl.complete_graph(n), 0, 1.0, H, 0.05, 0, seed=11)
    g.set_objective_lsq(torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda(), m, batch)
    c.objective = LeastSquares(A, b, batch)
    gen = np.random.Generator(np.random.PCG64(n))
    X = gen.standard_normal((n, d)).astype(np.float32)
    c.X[:], c.Xhat[:] = X, X
    g.write_models(gpu.COMM, X)
    g.write_models(gpu.SNAP, X)
    want = [c.step_sequential() for _ in range(count)]
    pairs, _ = g.run_sequential(count)
    assert [tuple(p) for p in pairs] == want and len({i for i, _ in want}) > 2
    assert_close(g.read_models(gpu.COMM), c.X, TOL_GEMM, "X after the run")
    assert_close(g.read_models(gpu.SNAP), c.Xhat, TOL_GEMM, "snapshots after the run")
    led = sorted({i for i, _ in want})
    assert_close(g.read_models(gpu.LIVE)[led], c.W[led], TOL_GEMM, "live copies of the initiators")


# more steps than a call of the generator draws the rows of (8 at up to 16 rows, 4 above); one workgroup, some of a
# request's workgroups, a second turn of requests (64 workgroups, 28 rows), words of rows past the batch
@pytest.mark.parametrize("n,d,m,batch,H,count", [
    (3, 128, 9, 16, 11, 6), (4, 1160, 20, 20, 9, 8), (3, 8184, 12, 28, 5, 5), (3, 8072, 9, 8, 9, 4)])
def test_longer_least_squares_interactions_against_the_oracle(gpu, n, d, m, batch, H, count):
    test_short_least_squares_run_against_the_oracle(gpu, n, d, m, batch, H, count)


@pytest.mark.parametrize("n_edges", [1, 127, 128, 129])
def test_matching_on_the_host_and_on_the_device(gpu, n_edges):
    """Up to 128 edges are matched on the host, more on the device."""
    edges = np.random.Generator(np.random.PCG64(n_edges)).permutation(wl.complete_graph(20))[:n_edges]
    g, c = make_both(gpu, 20, 64, edges, 8, 1.0, 0, 0.0, 0, seed=5)
    for _ in range(6):
        want = c.sample_matching()
        assert np.array_equal(g.sample_matching(), want.astype(np.uint32))
        g.gossip_round()
        c.gossip_round(want)
        assert g.counters()["interactions"] == c.interactions


@pytest.mark.parametrize("d", [504, 512 * 60, 512 * 140])
def test_rounds_enqueued_without_waiting(gpu, d):
    """Small rounds read their descriptors from the staging slots, larger ones from a copy: many rounds in flight give what
    the same rounds give one at a time."""
    n = 64
    gen = torch.Generator(device="cuda").manual_seed(2)
    a, c = torch.rand(n, d, generator=gen, device="cuda") + 0.5, torch.randn(n, d, generator=gen, device="cuda")
    swarms = [gpu.Swarm(n, d, wl.random_regular_graph(n, 4, 0), 8, 2.0 ** -4, 2, 0.1, 1, 3) for _ in range(2)]
    for s in swarms:
        s.set_objective_diag(a, c, 0.1)
        s.models_view(gpu.COMM).copy_(c)
    for _ in range(40):
        swarms[0].round_fused(stale=swarms[0].sample_stale())
    for _ in range(40):
        swarms[1].round_fused(stale=swarms[1].sample_stale())
        torch.cuda.synchronize()
    assert torch.equal(swarms[0].models_view(gpu.COMM), swarms[1].models_view(gpu.COMM))
    assert swarms[0].counters() == swarms[1].counters()


# both reads stale, codes of 2 and 4 bits: one kernel up to three steps from 2^15 tiles on (8 nodes of 2^21 coordinates
# are exactly as many), another below and for more steps
@pytest.mark.parametrize("bits,H,d,inplace", [
    (4, 3, 1 << 21, False), (4, 3, (1 << 21) - 2048, False), (4, 4, 1 << 21, False), (2, 3, (1 << 21) + 8, False),
    (2, 4, 4104, False), (4, 3, 1 << 21, True), (2, 1, 1 << 21, True)])
def test_one_pass_round_with_stale_reads_equals_steps_then_gossip(gpu, bits, H, d, inplace):
    n, pairs = 8, [(0, 5), (1, 2), (3, 6), (4, 7)]
    gen = torch.Generator(device="cuda").manual_seed(bits + H)
    a, c = torch.rand(n, d, generator=gen, device="cuda") + 0.5, torch.randn(n, d, generator=gen, device="cuda")
    X = [torch.randn(n, d, generator=gen, device="cuda") for _ in range(2)]
    swarms = [gpu.Swarm(n, d, wl.complete_graph(n), bits, 0.5, H, 0.1, 1, 7,
                        apply_mode=gpu.INPLACE if inplace else gpu.DEFERRED) for _ in range(2)]
    for s in swarms:
        s.set_objective_diag(a, c, 0.1)
        s.models_view(gpu.COMM).copy_(X[0])
        s.gossip_round(pairs)
        s.models_view(gpu.COMM).copy_(X[1])
    ones = np.ones(n, dtype=np.uint8)
    swarms[0].round_fused(pairs, ones)
    swarms[1].local_steps()
    swarms[1].gossip_round(pairs, ones)
    assert torch.equal(swarms[0].models_view(gpu.COMM), swarms[1].models_view(gpu.COMM))
    for node in (0, 7):
        assert np.array_equal(swarms[0].read_codes(node), swarms[1].read_codes(node))
    assert swarms[0].counters(raise_on_range=False) == swarms[1].counters(raise_on_range=False)


# the same with codes of 8 bits, whose line between the two kernels is the same
@pytest.mark.parametrize("H,d,inplace", [(3, 1 << 21, False), (3, (1 << 21) - 2048, False), (1, (1 << 21) + 8, True)])
def test_one_pass_round_with_stale_reads_of_8_bit_codes(gpu, H, d, inplace):
    test_one_pass_round_with_stale_reads_equals_steps_then_gossip(gpu, 8, H, d, inplace)


# As many interactions as the run has teams for their steps, one more or less, and several turns of them; one node leads half of them
# (star), two take turns (a single edge): run and single interactions are the same bits
@pytest.mark.parametrize("count", [6, 7, 8, 15, 23])
@pytest.mark.parametrize("n,d,batch,H,geometric,graph", [
    (2, 136, 16, 1, False, "edge"), (6, 1032, 32, 1, False, "star"), (9, 648, 20, 3, True, "star"), (12, 2056, 28, 2, False, "complete")])
def test_least_squares_run_of_few_interactions(gpu, n, d, batch, H, geometric, graph, count):
    A, b, _ = wl.least_squares_data(n, d, 24, 3)
    edges = [(0, v) for v in range(1, n)] if graph != "complete" else wl.complete_graph(n)
    gen = np.random.Generator(np.random.PCG64(d))
    X = (gen.standard_normal((1, d)) + 0.05 * gen.standard_normal((n, d))).astype(np.float32)
    pair = []
    for _ in range(2):
        g, _ = make_both(gpu, n, d, np.array(edges, dtype=np.uint32), 8, 2.0 ** -6, H, 0.05, 0, seed=count, geometric=geometric)
        g.set_objective_lsq(torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda(), 24, batch)
        g.write_models(gpu.COMM, X)
        g.write_models(gpu.SNAP, X + np.float32(0.01))
        pair.append(g)
    run, one = pair
    for _ in range(2):                                      # the second run starts from the words the first one left
        pairs, _ = run.run_sequential(count)
        for i, j in pairs:
            one.interact(i, j)
    for which in (gpu.COMM, gpu.SNAP, gpu.LIVE):
        assert np.array_equal(run.read_models(which), one.read_models(which))
    for node in range(n):
        assert np.array_equal(run.read_codes(node), one.read_codes(node))
    assert run.counters(raise_on_range=False) == one.counters(raise_on_range=False)


# The forms of a run of Algorithm 1 that the sizes above leave out: four waves with noise and snapshots held ahead, their largest
# tiles, and from 5 x 2^19 coordinates on 512-coordinate tiles of two and four waves; up to four steps' noise is drawn ahead
@pytest.mark.parametrize("n,d,bits,H,sigma,geometric", [
    (9, 1 << 17, 8, 4, 0.1, False), (4, (1 << 17) + 8, 8, 3, 0.1, True), (8, (1 << 19) - 8, 4, 6, 0.05, False), (12, 3 << 16, 16, 5, 0.1, True),
    (3, 5 << 19, 8, 3, 0.1, False), (10, (5 << 19) + 8, 4, 2, 0.1, True), (39, 1 << 16, 8, 2, 0.0, False), (20, (1 << 16) + 8, 2, 5, 0.1, False),
    (2, 8, 8, 9, 0.1, False), (6, 264, 0, 255, 0.1, False)])
def test_run_of_algorithm1_by_its_forms(gpu, n, d, bits, H, sigma, geometric):
    test_run_of_algorithm1_in_one_launch(gpu, n, d, bits, H, sigma, geometric, True)


# Logits in float32 cut along the hidden units: 14 parts and a shorter one, parts as wide as the row of classes allows (two), the most
# classes that are cut and more; tiles of 32 rows (batch 32 and 96), biases beside the updates.  The same bits whoever steps along.
@pytest.mark.parametrize("n,n_in,n_hid,n_out,batch", [
    (3, 64, 1056, 32, 32), (2, 96, 1120, 96, 96), (5, 32, 2080, 64, 128), (2, 32, 4096, 2048, 32), (2, 64, 2144, 2080, 64),
    (4, 64, 672, 160, 160), (130, 64, 128, 32, 96), (2, 544, 64, 32, 64)])
def test_mlp_logits_in_parts(gpu, n, n_in, n_hid, n_out, batch):
    test_mlp_tiles(gpu, n, n_in, n_hid, n_out, batch, "fp32")
    d = n_hid * n_in + n_hid + n_out * n_hid + n_out
    means, cdf = wl.mixture_data(n, n_in, n_out, 1)
    s = gpu.Swarm(n, d, wl.complete_graph(n) if n < 16 else wl.random_regular_graph(n, 4, 0), 8, 2.0 ** -10, 2, 0.05, 0, n)
    s.set_objective_mlp(n_in, n_hid, n_out, torch.from_numpy(means).cuda(), torch.from_numpy(cdf).cuda(), 0.5, batch)
    X, W = s.models_view(gpu.COMM), s.models_view(gpu.LIVE)
    X.copy_(torch.randn(n, d, generator=torch.Generator(device="cuda").manual_seed(n), device="cuda").mul_(0.1))
    s.local_steps()
    whole = W.clone()
    for some in ([n - 1], [n - 1, 0]):
        W.zero_()
        s.local_steps(some)
        assert torch.equal(W[some], whole[some])
    s.close()
