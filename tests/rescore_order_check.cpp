// The re-score of kb_topk with its threads in several orders: the same lists in
// each, and every candidate of the grid scored.
#include "workgroup_on_cpu.h"

#include "kbmi_kernels.hip"

#include <random>

namespace kbmi {
namespace {
alignas(16) unsigned char rs_lds[160 * 1024];
}
}  // namespace kbmi

int main() {
    using namespace kbmi;
    const int h = 2, w = 64, n_img = 5, n_vel = 40, kc = 8, k = 8;
    std::mt19937 rng(1901);
    std::normal_distribution<float> noise;
    std::vector<float2> planes((size_t)n_img * h * w);
    for (float2 &p : planes) p = make_float2(noise(rng), 1.0f);
    std::vector<double> tau(n_img);
    for (int i = 0; i < n_img; ++i) tau[i] = 0.25 * i;
    std::vector<double2> vels(n_vel);
    for (int j = 0; j < n_vel; ++j) vels[j] = make_double2(j - 20.0, 0.1 * (j % 7));
    // Distinct velocities a pixel, every ninth outside the grid.
    std::vector<int32_t> cand((size_t)h * w * kc);
    for (size_t c = 0; c < cand.size(); ++c)
        cand[c] = c % 9 == 4 ? -1 : (int32_t)((c / kc * 11 + c % kc * 5) % n_vel);

    std::vector<std::vector<int>> orders(3, std::vector<int>(TK_THREADS));
    for (int t = 0; t < TK_THREADS; ++t) {
        orders[0][t] = t;
        orders[1][t] = TK_THREADS - 1 - t;
        orders[2][t] = (t + 2 * 64) % TK_THREADS;
    }
    std::vector<float> first;
    for (const auto &order : orders) {
        const size_t n = (size_t)h * w * k;
        std::vector<float> nu(n, 77.f), al(n, 77.f);
        std::vector<int32_t> vel(n, 77);
        std::vector<int16_t> nobs(n, 77);
        for (unsigned b = 0; b < 8u * h; ++b)
            cpu_group::run(b, order, [&]() {
                topk_rescore_kernel(h, w, 0, h, n_img, planes.data(), tau.data(), vels.data(),
                                    n_vel, kc, k, cand.data(), nu.data(), al.data(), vel.data(),
                                    nobs.data());
            });
        for (size_t p = 0; p < n / k; ++p) {
            int want = 0, got = 0;
            for (int s = 0; s < k; ++s) {
                want += cand[p * kc + s] >= 0;
                got += nobs[p * k + s] > 0 && std::isfinite(nu[p * k + s]);
                if (s > 0 && nu[p * k + s] > nu[p * k + s - 1]) {
                    std::printf("pixel %zu slot %d out of order\n", p, s);
                    return 1;
                }
            }
            if (got != want) {
                std::printf("pixel %zu: %d of %d candidates scored\n", p, got, want);
                return 1;
            }
        }
        if (first.empty()) first = nu;
        if (std::memcmp(first.data(), nu.data(), n * sizeof(float)) != 0) {
            std::puts("the order of the threads changes nu");
            return 1;
        }
    }
    std::puts("re-score ok");
    return 0;
}
