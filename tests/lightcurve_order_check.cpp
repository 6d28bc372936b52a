// The light-curve filter with its threads in several orders: the same results in
// each, and every candidate of the grid filtered.
#include "workgroup_on_cpu.h"

#include "kbmi_filter.hip"

#include <random>

namespace kbmi {
namespace {
alignas(16) unsigned char lc_lds[160 * 1024];
}
}  // namespace kbmi

int main() {
    using namespace kbmi;
    const int h = 2, w = 64, n_img = 5, n_vel = 40, k = 8, pt = 64;
    std::mt19937 rng(1901);
    std::normal_distribution<float> noise;
    std::vector<float2> planes((size_t)n_img * h * w);
    for (float2 &p : planes) p = make_float2(noise(rng), 1.0f);
    std::vector<double> tau(n_img);
    for (int i = 0; i < n_img; ++i) tau[i] = 0.25 * i;
    std::vector<double2> vels(n_vel);
    for (int j = 0; j < n_vel; ++j) vels[j] = make_double2(j - 20.0, 0.1 * (j % 7));
    // Every ninth candidate's velocity is outside the grid.
    std::vector<int32_t> cand((size_t)h * w * k);
    for (size_t c = 0; c < cand.size(); ++c)
        cand[c] = c % 9 == 4 ? -1 : (int32_t)((c / k * 11 + c % k * 5) % n_vel);

    std::vector<std::vector<int>> orders(3, std::vector<int>(LC_THREADS));
    for (int t = 0; t < LC_THREADS; ++t) {
        orders[0][t] = t;
        orders[1][t] = LC_THREADS - 1 - t;
        orders[2][t] = (t + 2 * 64) % LC_THREADS;
    }
    // sigma_cut 1.5: some candidates drop observations, in one round or more.
    std::vector<float> first;
    std::vector<uint64_t> first_rejected;
    for (const auto &order : orders) {
        const size_t n = cand.size();
        std::vector<float> nu(n, 77.f), al(n, 77.f);
        std::vector<int16_t> nobs(n, 77);
        std::vector<uint64_t> rejected(n, 77);
        for (unsigned b = 0; b < 8u * h; ++b)
            cpu_group::run(b, order, [&]() {
                lightcurve_grouped_kernel<16>(k, pt, h, w, 0, h, n_img, planes.data(), tau.data(),
                                              vels.data(), n_vel, 2.25, 0.5, 64.f, cand.data(),
                                              nu.data(), al.data(), nobs.data(), rejected.data());
            });
        for (size_t c = 0; c < n; ++c)
            if ((cand[c] >= 0) != (nobs[c] > 0 && std::isfinite(nu[c]))) {
                std::printf("candidate %zu of velocity %d: nu %g, n_obs %d\n", c, cand[c], nu[c],
                            nobs[c]);
                return 1;
            }
        if (first.empty()) first = nu, first_rejected = rejected;
        if (std::memcmp(first.data(), nu.data(), n * sizeof(float)) != 0 ||
            first_rejected != rejected) {
            std::puts("the order of the threads changes the results");
            return 1;
        }
    }
    std::puts("light curves ok");
    return 0;
}
