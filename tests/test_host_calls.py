"""Which kernels the library launches, and how it guards its staging memory: its host code on the CPU, with host_calls.cpp in
place of the HIP runtime."""
import os
import re
import subprocess

import pytest

import paper_1910_12308_amd as swarm
from helpers import ALGORITHM1_RUNS

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def host_calls(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host_calls") / "host_calls")
    package = os.path.dirname(swarm.LIB_PATH)
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-I", os.path.join(ROOT, "include"),
                    os.path.join(HERE, "host_calls.cpp"), "-o", exe, "-L", package, "-l:libswarm.so", "-Wl,-rpath," + package,
                    "-Wl,--allow-shlib-undefined"], check=True)

    def call(*args, **settings):
        out = subprocess.run([exe] + [str(a) for a in args], capture_output=True, text=True,
                             env={**os.environ, **{k: str(v) for k, v in settings.items()}})
        assert out.returncode == 0, out.stdout + out.stderr
        return out.stdout.splitlines()
    return call


def kernels(lines):
    return [re.match(r"launch (\w+)", ln).group(1) for ln in lines if ln.startswith("launch")]


# Least squares, runs of Algorithm 1: one launch on graphs where at most seven interactions run side by side, a launch per level
# otherwise and beyond 64 nodes, a batch of 32, 2048 words and 64 groups of 128 columns
@pytest.mark.parametrize("n,d,batch,graph,merged", [
    (8, 4096, 32, "complete", True), (16, 8192, 32, "complete", True), (32, 4096, 32, "complete", True),
    (48, 2048, 32, "complete", False), (64, 2048, 16, "complete", False), (64, 512, 32, "ring", False),
    (64, 512, 32, "star", True), (65, 512, 16, "star", False), (5, 1024, 36, "complete", False), (5, 8200, 16, "complete", False),
    (2, 4104, 32, "complete", True), (2, 8192, 32, "complete", True), (2, 8200, 12, "complete", False)])
def test_least_squares_runs(host_calls, n, d, batch, graph, merged):
    run = host_calls("run", n, d, 8, 2, batch, graph, 40)
    levels = int(next(ln for ln in run if ln.startswith("reported")).split()[1])
    assert kernels(run) == (["lsq_run_kernel"] if merged else ["lsq_split_kernel"] * levels) and levels > 1
    # a single interaction takes the same form, so that it gives the same sums
    one = host_calls("interact", n, d, 8, 2, batch, graph)
    assert kernels(one) == ["lsq_run_kernel" if merged else "lsq_split_kernel"] and run[-1] == one[-1] == "status 0"


@pytest.mark.parametrize("n,d,bits,H,merged", [(r[0], r[1], r[2], r[3], r[7]) for r in ALGORITHM1_RUNS])
def test_runs_of_the_gpu_tests_take_the_form_they_are_there_for(host_calls, n, d, bits, H, merged):
    run = host_calls("run", n, d, bits, H, 0, "complete", 3 * n + 1)
    assert set(kernels(run)) == {"interact_run_kernel" if merged else "interact_kernel"} and (len(kernels(run)) == 1) == merged


# Diagonal objective, runs of Algorithm 1: one launch where the run has enough interactions, or rows short enough, and, on
# long rows, where enough of them run side by side for their local steps
@pytest.mark.parametrize("n,d,H,graph,count,merged", [
    (8, 8888, 3, "complete", 16, True), (64, 1 << 20, 3, "complete", 256, True), (64, 1 << 20, 3, "complete", 23, False),
    (64, 1 << 20, 3, "ring", 32, True), (78, 1544, 3, "star", 60, True), (79, 1544, 3, "complete", 60, False),
    (64, (3 << 17) - 8, 20, "star", 64, True), (64, 3 << 17, 3, "star", 64, False), (40, 1 << 20, 3, "hubs4", 200, True),
    (40, 1 << 20, 3, "hubs2", 200, False), (24, 4_000_000, 10, "star", 24, False), (24, 4_000_000, 3, "complete", 64, True),
    (31, 1 << 20, 5, "hubs3", 64, True), (20, 1 << 20, 3, "star", 40, False), (19, 1 << 20, 5, "star", 40, True),
    (19, 4_000_000, 20, "star", 40, False), (9, 4_000_000, 5, "star", 16, True), (2, 1 << 20, 3, "path", 4, True),
    (48, 4_000_000, 20, "hubs4", 200, False)])
def test_diagonal_runs(host_calls, n, d, H, graph, count, merged):
    run = host_calls("run", n, d, 8, H, 0, graph, count)
    levels = int(next(ln for ln in run if ln.startswith("reported")).split()[1])
    assert kernels(run) == (["interact_run_kernel"] if merged else ["interact_kernel"] * levels)
    assert levels > 1 and run[-1] == "status 0"


# Least-squares local steps of swarms too wide for the exchanging form, in the wide form: several workgroups per node and a launch
# more than steps, or one workgroup per node and one launch.  All of them take it where the runtime cannot tell how many workgroups
# of a team fit the chip, and where the steps update the models themselves; else the next test says which are taken by teams.
@pytest.mark.parametrize("n,d,batch,kernel,threads,grid", [
    (64, 4104, 32, "lsq_wide_kernel<256, false>", 256, "5 64"), (65, 2048, 16, "lsq_wide_kernel<512, true>", 512, "1 65"),
    (65, 2056, 16, "lsq_wide_kernel<256, false>", 256, "3 65"), (100, 3080, 64, "lsq_wide_kernel<512, true>", 512, "1 100"),
    (100, 4104, 64, "lsq_wide_kernel<256, false>", 256, "5 100"), (128, 16384, 16, "lsq_wide_kernel<512, true>", 512, "1 128"),
    (128, 16392, 16, "lsq_wide_kernel<256, false>", 256, "9 128"), (255, 1032, 16, "lsq_wide_kernel<512, true>", 512, "1 255"),
    (260, 1024, 16, "lsq_wide_kernel<256, true>", 256, "1 260"), (300, 16392, 16, "lsq_wide_kernel<1024, true>", 1024, "1 300"),
    (499, 2048, 16, "lsq_wide_kernel<512, true>", 512, "1 499"), (500, 2048, 16, "lsq_wide_kernel<1024, true>", 1024, "1 500"),
    (500, 3080, 16, "lsq_wide_kernel<512, true>", 512, "1 500"), (512, 4096, 16, "lsq_rows_kernel", 1024, "512 1"),
    (513, 4096, 16, "lsq_wide_kernel<512, true>", 512, "1 513"), (300, 4096, 64, "lsq_rows_kernel", 1024, "300 1"),
    (300, 8192, 32, "lsq_rows_kernel", 1024, "300 1"), (300, 8192, 36, "lsq_wide_kernel<512, true>", 512, "1 300"),
    (256, 8192, 16, "lsq_wide_kernel<512, true>", 512, "1 256")])
def test_wide_least_squares_steps(host_calls, n, d, batch, kernel, threads, grid):
    H = 3
    slices = H + 1 if kernel.endswith("false>") else 1
    for settings in ({}, dict(GROUPS_PER_UNIT=5, INPLACE=1)):
        out = host_calls("steps", n, d, 8, H, batch, "ring", **settings)
        assert [ln for ln in out if ln.startswith("launch")] == [f"launch {kernel} grid {grid} block {threads} shared 0"] * slices
        assert out[-1] == "status 0"


# The same by teams, with five workgroups per compute unit, four at batches up to 8 and six at batches of 12 and 16: teams at
# once (all nodes, or as many as fit, evenly over the rounds), workgroups of a team that hold columns and that add rows
@pytest.mark.parametrize("n,d,batch,kernel,teams,columns,adding", [
    (64, 4104, 32, "8, 2, true", 64, 9, 1), (64, 4104, 28, "8, 2, false", 64, 9, 1), (16, 65544, 64, "16, 1, true", 4, 257, 16),
    (16, 65544, 60, "16, 1, false", 4, 257, 15), (9, 131072, 32, "8, 2, true", 3, 256, 4), (80, 4096, 64, "16, 1, true", 40, 16, 1),
    (255, 2048, 64, "16, 1, true", 128, 8, 1), (255, 2040, 64, None, 0, 0, 0), (100, 4096, 32, "8, 2, true", 100, 8, 1),
    (100, 4088, 32, None, 0, 0, 0), (128, 16384, 16, "4, 2, true", 43, 32, 1), (128, 16376, 16, None, 0, 0, 0),
    (300, 16384, 20, "8, 2, false", 38, 32, 1), (300, 16384, 12, None, 0, 0, 0), (300, 4096, 64, "16, 1, true", 75, 16, 1),
    (65, 2056, 16, "4, 2, true", 65, 5, 1), (33, 4104, 12, "4, 2, false", 33, 9, 1), (64, 8200, 8, "2, 4, true", 64, 9, 1),
    (35, 4104, 4, "2, 4, false", 35, 5, 1), (2, 264008, 64, "16, 1, true", 1, 1032, 16), (2, 330000, 64, None, 0, 0, 0),
    (8, 66000, 16, "4, 2, true", 8, 129, 2)])
def test_least_squares_steps_by_teams(host_calls, n, d, batch, kernel, teams, columns, adding):
    groups = 4 if batch <= 8 else 6 if batch <= 16 else 5
    out = [ln for ln in host_calls("steps", n, d, 8, 3, batch, "ring", GROUPS_PER_UNIT=groups) if ln.startswith("launch")]
    if kernel:
        assert out == [f"launch lsq_team_kernel<{kernel}> grid {teams * (columns + adding)} 1 block 256 shared 0"]
    else:
        assert not any("team" in ln for ln in out)
    # the steps of one node: one team
    one = [ln for ln in host_calls("interact", n, d, 8, 3, batch, "ring", GROUPS_PER_UNIT=groups) if ln.startswith("launch")]
    assert kernel is None or one[0] == f"launch lsq_team_kernel<{kernel}> grid {columns + adding} 1 block 256 shared 0"


# The wide form's exchange takes 2 x 64 x 5 x 64 floats, that of one team with its model 4104 floats and more
@pytest.mark.parametrize("room,teams", [(163840 + 10_000_000, True), (163840 + 4 * 4104, False), (163840, False)])
def test_least_squares_where_memory_is_short_for_teams(host_calls, room, teams):
    out = host_calls("steps", 64, 4104, 8, 3, 32, "ring", GROUPS_PER_UNIT=5, ROOM=room)
    assert kernels(out) == (["lsq_team_kernel"] if teams else ["lsq_wide_kernel"] * 4) and out[-1] == "status 0"


# Whatever the runtime counts, no more workgroups than run at once: six on each of 256 compute units
@pytest.mark.parametrize("counted,grid", [(5, 1161), (6, 1290), (7, 1290), (8, 1290)])
def test_workgroups_of_teams_run_at_once(host_calls, counted, grid):
    out = host_calls("steps", 100, 65536, 8, 1, 16, "ring", GROUPS_PER_UNIT=counted)
    assert [ln for ln in out if ln.startswith("launch")] == [f"launch lsq_team_kernel<4, 2, true> grid {grid} 1 block 256 shared 0"]


# Few rows in all, and a swarm whose workgroups run at once in the wide form but not with reducing workgroups beside them
@pytest.mark.parametrize("n,d,batch,H,teams", [
    (64, 16384, 8, 1, 0), (64, 16384, 4, 3, 0), (64, 16384, 8, 2, 32), (64, 16384, 12, 1, 32), (60, 16384, 4, 1, 60), (65, 16384, 4, 1, 33),
    (124, 8192, 4, 1, 0), (32, 32768, 8, 1, 0), (31, 33000, 4, 1, 16)])
def test_teams_of_few_rows_take_all_nodes_at_once(host_calls, n, d, batch, H, teams):
    out = [ln for ln in host_calls("steps", n, d, 8, H, batch, "ring", GROUPS_PER_UNIT=4 if batch <= 8 else 6) if ln.startswith("launch")]
    if teams:
        groups = -(-d // (1024 if batch <= 8 else 512)) + 1
        assert len(out) == 1 and out[0].startswith("launch lsq_team_kernel") and f" grid {teams * groups} " in out[0]
    else:
        assert out == [f"launch lsq_wide_kernel<256, false> grid {-(-d // 1024)} {n} block 256 shared 0"] * (H + 1)


def test_teams_of_several_swarms_take_turns(host_calls):
    """One swarm alone is not held up; when a second joins, what the first has launched is waited for; from then on a launch waits
    for the one before, whoever made that."""
    out = host_calls("two", 64, 4104, 8, 3, 32, "ring", GROUPS_PER_UNIT=5)
    team, event = "launch lsq_team_kernel<8, 2, true>", next(ln.split()[2] for ln in out if ln.startswith("stream waits"))
    calls = [ln.split(" grid")[0] for ln in out
             if ln.startswith(("launch", "stream waits")) or ln in (f"record {event}", "wait for all")]
    assert calls == [team, "wait for all", team, f"record {event}", f"stream waits {event}", team, f"record {event}", team]
    assert out[-1] == "status 0"


@pytest.mark.parametrize("fail", [0, 1, 2, 3, 4])
def test_staging_slot_is_guarded_until_its_readers_are_done(host_calls, fail):
    """Small rounds are described in a staging slot that their kernels read: the event that frees the slot is recorded behind
    every launch, also where a launch of the round fails."""
    out = host_calls("rounds", 8, 8888, 8, 2, fail, 3)
    ends = [k for k, ln in enumerate(out) if ln.startswith("status")][:3]
    assert [out[k] for k in ends] == ["status 3" if fail and (fail - 1) // 2 == r else "status 0" for r in range(3)]
    for first, end in zip([0] + [k + 1 for k in ends], ends):
        call = out[first:end]
        slot = next(ln.split()[1] for ln in call if ln.startswith("wait"))
        launches = [k for k, ln in enumerate(call) if ln.startswith("launch")]
        assert launches and f"record {slot}" in call[launches[-1]:]
        assert "copy" not in call


# tiles of 512 coordinates x (pair + unmatched nodes) = waves of the round; the graphs are complete: 120 edges at 16 nodes,
# 136 at 17
@pytest.mark.parametrize("n,d,copied", [
    (16, 512 * 273, False), (16, 512 * 274, True), (17, 512 * 80, False), (17, 512 * 81, True), (8, 8888, False)])
def test_descriptors_are_copied_ahead_of_larger_rounds(host_calls, n, d, copied):
    out = host_calls("rounds", n, d, 8, 2, 0, 1)
    assert ("copy" in out) == copied and out[-1] == "status 0"


# Perceptrons, bf16x3 products, one step of `count` of the n nodes: blocks of 32 samples per workgroup and workgroups (dies in
# turn) of the hidden, logits and backward products, the latter with the update of W2 inside or apart.  What a workgroup takes
# follows from the nodes that step: one node of a swarm that fills the chip would leave it idle in the whole swarm's form.
@pytest.mark.parametrize("n,n_in,n_hid,n_out,batch,count,hidden,logits,back,inside", [
    (256, 1024, 4096, 1024, 128, 256, (4, 8192), (4, 2048), (4, 4096), True),
    (256, 1024, 4096, 1024, 128, 8, (4, 256), (1, 256), (4, 128), True),
    (256, 1024, 4096, 1024, 128, 7, (4, 224), (1, 224), (4, 224), False),
    (256, 1024, 4096, 1024, 128, 1, (1, 128), (1, 32), (1, 128), False),
    (32, 800, 1504, 480, 64, 32, (2, 384), (2, 256), (2, 384), True),
    (32, 800, 1504, 480, 64, 5, (1, 120), (1, 80), (1, 120), False),
    (64, 736, 1376, 896, 160, 12, (5, 136), (3, 168), (5, 136), False),
    (64, 736, 1376, 896, 160, 1, (1, 56), (1, 40), (1, 56), False),
    (100, 96, 224, 64, 32, 1, (1, 8), (1, 8), (1, 8), True),
    (100, 96, 224, 64, 96, 1, (1, 8), (1, 8), (3, 8), True), (100, 96, 224, 64, 128, 1, (1, 8), (1, 8), (1, 8), False),
    (64, 32, 512, 32, 160, 64, (5, 256), (5, 256), (5, 256), False),
    (64, 32, 512, 32, 224, 64, (4, 512), (4, 512), (4, 512), False),
    (64, 32, 512, 32, 288, 64, (5, 512), (5, 512), (5, 512), False),
    (64, 32, 512, 32, 352, 64, (4, 768), (4, 768), (4, 768), False),
    (64, 32, 512, 32, 352, 9, (2, 216), (2, 216), (2, 216), False)])
def test_perceptron_products(host_calls, n, n_in, n_hid, n_out, batch, count, hidden, logits, back, inside):
    out = host_calls("mlp", n, n_in, n_hid, n_out, batch, 1, count)
    products = [ln for ln in out if "mlp_product_kernel" in ln]
    threads = 512 if inside and batch == 128 else 256
    assert products == [
        f"launch mlp_product_kernel<{hidden[0]}, true, 0, false> grid {hidden[1]} 1 block 256 shared 0",
        f"launch mlp_product_kernel<{logits[0]}, true, 1, false> grid {logits[1]} 1 block 256 shared 0",
        f"launch mlp_product_kernel<{back[0]}, false, 2, {str(inside).lower()}> grid {back[1]} 1 block {threads} shared 0"]
    assert sum("update" in k for k in kernels(out)) == (1 if inside else 2)
    # the classes' bias goes with the softmax, the hidden one with the backward product, each where it holds the whole batch
    width = 0 if batch == 32 else n_out + (n_hid if back[0] < batch // 32 else 0)
    assert [ln for ln in out if "bias" in ln] == [
        f"launch mlp_bias_of_blocks_kernel grid {-(-width // 256)} {count} block 256 shared 0"] * (width > 0) and out[-1] == "status 0"


# Updates of the weights, bf16x3: up to 160 samples down the rows of the matrix, more by tiles of 128 x 128 weights or, where these
# are fewer than 256, of 64 x 64
@pytest.mark.parametrize("n,n_in,n_hid,n_out,batch,count,w2,w1", [
    (40, 128, 640, 96, 160, 40, ("mlp_update_kernel<5>", 200), ("mlp_update_kernel<5>", 400)),
    (64, 32, 512, 32, 192, 64, ("mlp_update_long_kernel<2>", 256), ("mlp_update_long_kernel<2>", 256)),
    (64, 32, 512, 32, 192, 63, ("mlp_update_long_kernel<1>", 504), ("mlp_update_long_kernel<1>", 504)),
    (65, 128, 512, 160, 224, 65, ("mlp_update_long_kernel<2>", 520), ("mlp_update_long_kernel<2>", 264)),
    (8, 64, 128, 32, 1024, 8, ("mlp_update_long_kernel<1>", 16), ("mlp_update_long_kernel<1>", 16))])
def test_perceptron_updates(host_calls, n, n_in, n_hid, n_out, batch, count, w2, w1):
    out = host_calls("mlp", n, n_in, n_hid, n_out, batch, 1, count)
    assert [ln for ln in out if "update" in ln] == [f"launch {k} grid {g} 1 block 256 shared 0" for k, g in (w2, w1)]


@pytest.mark.parametrize("n,batch,count,waves", [(32, 256, 32, 4), (33, 256, 33, 8), (33, 256, 32, 4), (64, 160, 64, 8), (2, 32, 2, 4)])
def test_perceptron_softmax(host_calls, n, batch, count, waves):
    """bf16x3: eight waves per SIMD from more than 256 blocks of 32 rows on."""
    out = host_calls("mlp", n, 32, 32, 1120, batch, 1, count)
    assert sum(f"softmax_grad_kernel<{waves}> grid {batch // 32} {count} " in ln for ln in out) == 1


# Updates of the weights in float32, up to 128 samples: a block of 32 rows per workgroup while there are at most 1024, two or more
# otherwise
@pytest.mark.parametrize("n,n_in,n_hid,n_out,batch,count,w2,w1", [
    (36, 608, 1280, 64, 128, 1, 24, 200), (36, 608, 1280, 64, 128, 5, 104, 1000), (36, 608, 1280, 64, 128, 6, 120, 600),
    (2, 32, 32, 32, 32, 2, 8, 8), (256, 1024, 4096, 1024, 128, 256, 8192, 2048)])
def test_perceptron_updates_in_float32(host_calls, n, n_in, n_hid, n_out, batch, count, w2, w1):
    out = host_calls("mlp_fp32", n, n_in, n_hid, n_out, batch, 1, count)
    assert [ln for ln in out if "update" in ln] == [
        f"launch mlp_float_update_kernel<{batch // 32}> grid {g} 1 block 256 shared 0" for g in (w2, w1)]


def room_calls(host_calls, *args):
    out = host_calls("mlp_room", *args)
    assert out[-1] == "status 0" and out[-3] == "status 0", out[-3:]
    return kernels(out), [int(v) for v in out[-2].split()[1:]]


# The memory that bf16x3 takes besides the float32 steps' activations: per node the hidden activations and twice the features once
# more (updates inside the products; once, apart), the logits' gradient once more and the logits as often as they are split, all of
# the size of float32 activations, signs, and column sums of blocks of 32 samples.  Going back to float32 frees it.
@pytest.mark.parametrize("n,n_in,n_hid,n_out,batch,features,splits", [
    (256, 1024, 4096, 1024, 128, 2, 1), (32, 800, 1504, 480, 64, 2, 2), (64, 736, 1376, 896, 160, 1, 1), (100, 96, 224, 64, 32, 2, 1)])
def test_memory_of_the_bf16x3_arithmetic(host_calls, n, n_in, n_hid, n_out, batch, features, splits):
    _, (objective, chosen, back) = room_calls(host_calls, n, n_in, n_hid, n_out, batch, 1, n, 1 << 50)
    rest = n * batch * (4 * (n_hid + features * n_in + (1 + splits) * n_out) + n_hid // 8 + ((n_hid + n_out) // 8 if batch > 32 else 0))
    assert chosen - objective == rest and back == objective


# With no room at all a few nodes step at a time, in the float32 steps' activations; nodes follow one another in every kernel
@pytest.mark.parametrize("n,n_in,n_hid,n_out,batch,count,groups", [
    (256, 1024, 4096, 1024, 128, 256, 2), (256, 1024, 4096, 1024, 128, 100, 1), (32, 800, 1504, 480, 64, 32, 4),
    (33, 800, 1504, 480, 64, 33, 5), (64, 96, 96, 1024, 32, 64, 4), (64, 736, 1376, 896, 160, 64, 2)])
def test_bf16x3_steps_where_memory_is_short(host_calls, n, n_in, n_hid, n_out, batch, count, groups):
    whole, _ = room_calls(host_calls, n, n_in, n_hid, n_out, batch, 2, count, 1 << 50)
    short, (objective, chosen, back) = room_calls(host_calls, n, n_in, n_hid, n_out, batch, 2, count, 0)
    assert chosen == back == objective
    assert whole.count("mlp_packed_batch_kernel") == 2 and short.count("mlp_packed_batch_kernel") == 2 * groups


@pytest.mark.parametrize("n,n_in,n_hid,n_out,count,w2,w1", [
    (130, 32, 512, 32, 130, "128, 128> grid 520", "128, 128> grid 520"), (65, 128, 512, 160, 65, "128, 128> grid 520", "128, 128> grid 264"),
    (65, 128, 512, 160, 63, "128, 128> grid 504", "64, 64> grid 1008"), (2, 64, 224, 96, 2, "64, 64> grid 16", "64, 64> grid 8")])
def test_perceptron_updates_in_float32_tiles(host_calls, n, n_in, n_hid, n_out, count, w2, w1):
    """Over 128 samples: tiles of 128 x 128 from 256 of them on."""
    out = host_calls("mlp_fp32", n, n_in, n_hid, n_out, 160, 1, count)
    assert [ln for ln in out if "mlp_gemm_kernel<false, false, 3" in ln] == [
        f"launch mlp_gemm_kernel<false, false, 3, {g} 1 block 256 shared 0" for g in (w2, w1)]
