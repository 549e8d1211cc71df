"""Which chunks take the kernel of a few particles, on the CPU (the rule itself).

Every chunk of up to three particles with the default options does; of four to six
those of little work, or of slots narrower than two steps and fewer than eight steps
to a slot; none beyond that, and none with another geometry, hold rule or quantity.
"""
import pytest

import host_driver

DRIVER = r"""
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t)
{
    return hipSuccess;
}
int main()
{
    using namespace radio;
    // particles, steps, cells, slot width in steps, hold, potentials, far, slots
    const double cases[][8] = {
        {1, 25000, 256, 50, 0, 0, 0, 64},
        {3, 1000000, 16384, 50, 0, 0, 0, 64},
        {3, 1, 1, 0.1, 0, 0, 0, 1},
        {6, 800, 1024, 12, 0, 0, 0, 64},
        {6, 2000, 16384, 0.1, 0, 0, 0, 1000},
        {6, 1, 262144, 12, 0, 0, 0, 64},
        {4, 3000, 4096, 12, 0, 0, 0, 128}, {5, 800, 4096, 12, 0, 0, 0, 64},
        {4, 800, 16384, 12, 0, 0, 0, 64},
        {6, 800, 16384, 12, 0, 0, 0, 4096},
        {5, 200, 65536, 2, 0, 0, 0, 128},
        {6, 500, 16384, 0.1, 0, 0, 0, 32},
        {7, 1, 1, 0.1, 0, 0, 0, 64},
        {1, 10, 10, 1, 1, 0, 0, 64},
        {1, 10, 10, 1, 2, 0, 0, 64},
        {1, 10, 10, 1, 0, 1, 0, 64},
        {1, 10, 10, 1, 0, 0, 1, 64}};
    for (auto& c : cases) {
        DepositJob J{};
        J.n_p = (int64_t)c[0]; J.n_s = (int64_t)c[1]; J.n_c = (int64_t)c[2];
        J.dt = 0.01; J.dt_det = c[3] * 0.01;
        J.n_t = (int64_t)c[7]; J.hold = (int64_t)c[4]; J.potentials = (int64_t)c[5];
        J.far = c[6] != 0 ? &J.dt : nullptr;
        printf("%d", few_particles(J) ? 1 : 0);
    }
    printf("\n");
    return 0;
}
"""


@pytest.mark.skipif(not host_driver.available(), reason="needs hipcc")
def test_few_rule(tmp_path):
    assert host_driver.run(tmp_path, 'extern "C"' + DRIVER).strip() == "11111111" + "0" * 9
