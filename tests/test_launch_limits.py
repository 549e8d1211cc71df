"""Launches of the per-tile kernels on the CPU: a launch takes fewer than 2^32 threads.

The library's host code (launch_order, launch_ring_choice and the planner in
radio_kernels.hip, host pass only) is linked with a driver that has its own
hipLaunchKernel, which notes the grid and the first work item of each launch
instead of launching.  Chunks whose particle orders or tiles need more threads than
one launch takes have to arrive in several that together cover every one once.
"""
import pytest

import host_driver

DRIVER = r"""
static long long g_threads, g_most, g_next, g_bad, g_launches;
static int g_item_arg;
extern "C" hipError_t hipLaunchKernel(const void*, dim3 grid, dim3 block, void** args, size_t, hipStream_t)
{
    const long long threads = (long long)grid.x * block.x;
    g_threads += threads;
    g_most = threads > g_most ? threads : g_most;
    if (g_item_arg >= 0 && *(long long*)args[g_item_arg] != g_next)
        ++g_bad;  // not where the last launch ended
    g_next += grid.x;
    ++g_launches;
    return hipSuccess;
}
static void show(const char* what, long long items)
{
    printf("%s items=%lld covered=%lld bad=%lld most=%lld launches=%lld\n", what, items, g_next,
           g_bad, g_most, g_launches);
    g_threads = g_most = g_next = g_bad = g_launches = 0;
}
int main()
{
    using namespace radio;
    const long long cases[][3] = {  // particles, steps, cells
        {256, 1200000, 4096}, {300, 4000000, 16384}, {32, 1100000, 4096}, {40, 2000000, 4096},
        {255, 1300000, 8192}, {1, 1, 1}, {1000, 2048, 16384}, {7, 100, 300000000}};
    for (auto& c : cases)
        for (int mode = 0; mode < 2; ++mode)
            for (int shape = 0; shape < kShapes; ++shape) {
                DepositJob J{};
                J.n_p = c[0]; J.n_s = c[1]; J.n_c = c[2]; J.n_t = 64;
                set_shape(J, shape);
                plan_job(J, 0, 1024);
                set_groups(J, max_order_groups(J, rec_bytes(mode), 0));
                g_item_arg = ORDER_ITEM;
                if (launch_order(J, nullptr) != hipSuccess) return 1;
                show("order", J.n_tiles * J.n_groups);
                g_item_arg = -1;  // a workgroup looks at several tiles
                if (launch_ring_choice(J, mode, nullptr) != hipSuccess) return 1;
                show("choice", J.n_tiles);
                printf("plan batches=%lld groups=%lld runs=%lld\n",
                       (long long)((J.n_p + J.groups - 1) / J.groups), (long long)J.n_groups,
                       (long long)J.n_runs);
            }
    return 0;
}
"""

# place of the first work item among the order kernel's arguments (the last)
ORDER_ITEM = 12


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    if not host_driver.available():
        pytest.skip("needs hipcc")
    out = host_driver.run(tmp_path_factory.mktemp("limits"), DRIVER,
                          (f"-DORDER_ITEM={ORDER_ITEM}",))
    return [(ln.split()[0], {k: int(v) for k, v in (f.split("=") for f in ln.split()[1:])})
            for ln in out.splitlines()]


def test_launches_stay_under_the_thread_limit(lines):
    launches = [d for what, d in lines if what != "plan"]
    assert len(launches) >= 2 * 8 * 2
    assert any(d["items"] * 256 >= 2**32 for d in launches)  # the limit is met
    for d in launches:
        assert d["most"] < 2**32, d
    for what, d in lines:
        if what == "order":
            assert d["covered"] == d["items"] and d["bad"] == 0, d
        elif what == "choice":
            assert d["launches"] == 1 and 0 < d["covered"] <= d["items"], d


def test_few_batches_keep_one_order(lines):
    """A chunk of fewer than 16 batches of particles keeps one order a tile, a
    workspace that does not grow with its steps; a longer one is sorted again."""
    plans = [d for what, d in lines if what == "plan"]
    few = [d for d in plans if d["batches"] < 16]
    assert max(d["runs"] for d in few) > 60000
    assert all(d["groups"] == 1 for d in few), few
    assert any(d["groups"] > 1 for d in plans)
