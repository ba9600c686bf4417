"""Which kernel serves which configuration (host side only, no GPU)."""
import pytest

import test_gpu_parity as gpu_tests
from routes import route


def full_views(E, N, G):
    return dict(num_envs=E, num_agents=N, num_taggers=max(1, N // 10), grid_size=G, obs_mode=1, obs_k=0)


@pytest.mark.parametrize("E,N,G", [
    (8000, 64, 512), (8000, 64, 513), (8000, 64, 1159), (1100, 64, 600), (1000, 96, 600), (3000, 80, 800), (500, 48, 700),
    (6000, 20, 1600), (100, 43, 800), (300, 65, 800)])
def test_full_views_rows_apart_wherever_the_keys_have_32_bits(E, N, G):
    r = route(full_views(E, N, G))
    assert r.wide == 0 and r.apart == 1 and r.kernel == "crew_env_kernel", r


@pytest.mark.parametrize("E,N,G,apart", [
    (8000, 64, 1160, 1), (8000, 64, 5000, 1), (1100, 64, 5000, 1), (900, 64, 5000, 0), (1000, 96, 4500, 1), (300, 96, 4500, 0), (8193, 64, 5000, 0),
    (300, 65, 5000, 0), (256, 101, 5000, 1), (257, 101, 5000, 0), (512, 131, 5000, 1), (513, 131, 5000, 0)])
def test_full_views_with_keys_of_64_bits(E, N, G, apart):
    """env_kernel does the step; agent counts that are multiples of four have their rows apart from 64 MB on."""
    r = route(full_views(E, N, G))
    assert r.wide != 0 and r.apart == apart and r.kernel == "env_kernel", r


@pytest.mark.parametrize("E,N,apart", [(700, 41, 1), (701, 41, 0), (700, 63, 1), (1500, 43, 0), (500, 65, 1), (501, 65, 0), (700, 129, 1), (701, 129, 0),
                                       (9000, 203, 1), (8192, 16, 1), (8193, 16, 0), (8192, 12, 0), (100, 39, 0)])
def test_full_views_rows_apart_by_the_size_of_the_batch(E, N, apart):
    """Agent counts that are no multiple of four gain only in batches that do not fill the chip."""
    assert route(full_views(E, N, 110)).apart == apart


def partial(E, N, taggers, G, K=4, tag_r2=2):
    return dict(num_envs=E, num_agents=N, num_taggers=taggers, grid_size=G, obs_k=K, tag_r2=tag_r2)


@pytest.mark.parametrize("taggers,G,tag_r2,reach", [
    (15, 100, 0, 0), (16, 100, 0, 5), (31, 100, 2, 0), (32, 100, 2, 5), (63, 100, 9, 0), (64, 100, 9, 5), (143, 100, 64, 0), (144, 100, 64, 5),
    (144, 341, 80, 12), (144, 342, 80, 0), (144, 341, 81, 0), (160, 32, 64, 2), (160, 33, 64, 3)])
def test_map_of_the_cells_that_taggers_reach(taggers, G, tag_r2, reach):
    r = route(partial(3, 700, taggers, G, tag_r2=tag_r2))
    assert r.kernel == "crew_env_kernel" and r.reach == reach, r


@pytest.mark.parametrize("E,N,taggers,G,K,tag_r2,kernel", [
    # few agents in reach: by the number of comparisons
    (3, 1000, 170, 342, 4, 64, "crew_env_kernel"), (3, 1000, 171, 342, 4, 64, "env_kernel"), (3, 1000, 171, 342, 8, 64, "env_kernel"),
    (20, 512, 256, 342, 4, 9, "crew_env_kernel"), (10, 700, 600, 342, 4, 100, "env_kernel"), (60, 1000, 500, 400, 4, 400, "env_kernel"),
    (60, 1000, 200, 342, 12, 9, "crew_env_kernel"), (60, 1000, 201, 342, 12, 9, "big_obs_kernel"), (60, 1000, 200, 342, 16, 9, "crew_env_kernel"),
    # the map
    (3, 1000, 500, 341, 4, 64, "crew_env_kernel"),
    # many in reach
    (60, 1000, 500, 100, 4, 100, "crew_env_kernel"), (10, 700, 600, 400, 4, 400, "crew_env_kernel"), (60, 1000, 500, 100, 16, 100, "crew_env_kernel"),
    # no tag check
    (60, 1000, 500, 342, 4, -1, "crew_env_kernel"),
    # the large-env pair for few envs with K > 8, as before crew_env_kernel
    (60, 1000, 500, 342, 16, 9, "big_obs_kernel"), (110, 1000, 500, 342, 16, 9, "big_obs_kernel"), (111, 1000, 500, 342, 16, 9, "env_kernel"),
    (125, 1000, 500, 342, 12, 9, "env_kernel"), (60, 1000, 500, 342, 16, 100, "big_obs_kernel"), (100, 700, 600, 342, 16, 9, "big_obs_kernel"),
    (101, 700, 600, 342, 16, 9, "env_kernel")])
def test_many_taggers_without_a_map(E, N, taggers, G, K, tag_r2, kernel):
    assert route(partial(E, N, taggers, G, K=K, tag_r2=tag_r2)).kernel == kernel


# ---- what the tables of the GPU tests say of the kernels they run ------------------------------------------------
def kernels(kw):
    kw = dict(kw)
    kw.setdefault("num_taggers", kw["num_agents"] // 12)
    return route(kw).kernel, route(kw, recording=True).kernel


ENTERED_DONE = {  # (single calls and wd_rollout, where one name stands for both)
    "quad_env_kernel": "quad_env_kernel", "wave_env_kernel": "wave_env_kernel", "small_env_kernel": "small_env_kernel",
    "crew_env_kernel_two_waves": "crew_env_kernel", "crew_env_kernel": "crew_env_kernel", "crew_env_kernel_k_five": "crew_env_kernel",
    "crew_env_kernel_k_twelve": "crew_env_kernel", "one_workgroup": "env_kernel rollout_kernel", "packed_envs": "env_kernel rollout_kernel",
    "packed_envs_k_run_time": "env_kernel rollout_kernel", "k_twelve_strips": "env_kernel rollout_kernel", "k_twelve_64_bit_keys": "env_kernel",
    "any_k": "env_kernel", "full_views": "crew_env_kernel", "full_views_rows_apart": "crew_env_kernel", "large_env_pair": "big_obs_kernel",
    "large_env_spread": "spread_obs_kernel"}


@pytest.mark.parametrize("name", list(gpu_tests.ENTERED_DONE))
def test_ways_a_roll_out_can_run(name):
    served = ENTERED_DONE[name].split()
    assert kernels(gpu_tests.ENTERED_DONE[name]) == (served[0], served[-1])


@pytest.mark.parametrize("name", list(gpu_tests.CROWDS))
def test_crowds_in_every_form(name):
    kw = gpu_tests.CROWDS[name]
    strips = name.startswith("strips") or name in ("wide_ids", "k_two_wide_workgroup")
    assert kernels(kw) == (("env_kernel", "rollout_kernel") if strips else 2 * ("crew_env_kernel",))
    r = route(dict(kw, num_taggers=kw["num_agents"] // 12))
    assert r.strips and r.teams == {"strips_of_four_envs": 4, "strips_of_two_envs_k_twelve": 2}.get(name, 1), r


@pytest.mark.parametrize("n", range(len(gpu_tests.SMALL_IN_LARGE_BATCHES)))
def test_fewest_envs_of_small_env_kernel(n):
    kw = gpu_tests.SMALL_IN_LARGE_BATCHES[n]
    assert kernels(kw) == 2 * ("small_env_kernel",)
    assert kernels(dict(kw, num_envs=kw["num_envs"] - 1)) == 2 * ("crew_env_kernel",)


@pytest.mark.parametrize("n", range(len(gpu_tests.LARGE_BATCHES)))
def test_fewest_envs_beyond_crew_env_kernel(n):
    kw = gpu_tests.LARGE_BATCHES[n]
    r = route(kw)
    assert kernels(kw) == ("env_kernel", "rollout_kernel") and r.strips and r.teams == (4 if n < 6 else 2 if n < 11 else 1), r
    assert kernels(dict(kw, num_envs=kw["num_envs"] - 2)) == 2 * ("crew_env_kernel",)


def test_slices_in_the_kernels_of_whole_workloads():
    for name, fewest in (("tag_2000x1000", 1025), ("tag_20000x100", 3001)):
        kw = gpu_tests.CONFIGS[name].kwargs()
        assert route(dict(kw, num_envs=fewest))[:5] == route(kw)[:5] != route(dict(kw, num_envs=fewest - 1))[:5]
