"""The rule that ends the Newton-Schulz steps of the direct decomposition, run
with the same steps in fp32 on the host: sets of vectors that are not
independent are turned away, also where no two of them are close, and what is
accepted is orthonormal."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_23843_amd", "csrc")

DRIVER = r"""
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>
#include "newton_schulz.h"
using namespace pkv;
typedef std::vector<std::vector<float>> Mat;   // vectors

static bool orthonormalize(Mat &z, float tol, int &steps) {
    const int r = (int)z.size(), n = (int)z[0].size();
    for (int it = 0;; ++it) {
        Mat S(r, std::vector<float>(r));
        bool bounded = true;
        float e = 0.f, f2 = 0.f;
        for (int i = 0; i < r; ++i)
            for (int j = 0; j < r; ++j) {
                float s = 0.f;
                for (int k = 0; k < n; ++k) s = fmaf(z[i][k], z[j][k], s);
                S[i][j] = s;
                const float ei = fabsf(s - (i == j ? 1.f : 0.f));
                bounded = bounded && ei <= kOrthMax;
                e = fmaxf(e, ei);
                f2 = fmaf(ei, ei, f2);
            }
        const Orth next = orth_next(bounded, e <= tol, 0.75f * f2 <= tol, it);
        steps = it;
        if (next == Orth::fail || next == Orth::done) return next == Orth::done;
        Mat y(r, std::vector<float>(n, 0.f));
        for (int i = 0; i < r; ++i)
            for (int j = 0; j < r; ++j) {
                const float c = fmaf(-0.5f, S[j][i], i == j ? 1.5f : 0.f);
                for (int k = 0; k < n; ++k) y[i][k] = fmaf(z[j][k], c, y[i][k]);
            }
        z = y;
        if (next == Orth::last_step) return true;
    }
}

static float error(const Mat &z) {
    double e = 0;
    for (size_t i = 0; i < z.size(); ++i)
        for (size_t j = 0; j < z.size(); ++j) {
            double s = 0;
            for (size_t k = 0; k < z[0].size(); ++k) s += (double)z[i][k] * z[j][k];
            e = std::max(e, fabs(s - (i == j)));
        }
    return (float)e;
}

int main() {
    std::mt19937 rng(1);
    std::normal_distribution<float> g;
    for (float tol : {1e-4f, 1.9e-5f, 3e-7f})
        for (int n : {16, 32, 64})
            for (int trial = 0; trial < 200; ++trial) {
                auto unit = [&] {
                    std::vector<float> v(n);
                    float s = 0;
                    for (float &x : v) s += (x = g(rng)) * x;
                    for (float &x : v) x /= sqrtf(s);
                    return v;
                };
                // three vectors 60 and 120 degrees apart in a plane, a little off it
                const std::vector<float> a = unit(), b0 = unit(), off = unit();
                float ab = 0;
                for (int k = 0; k < n; ++k) ab += a[k] * b0[k];
                std::vector<float> b(n);
                float bb = 0;
                for (int k = 0; k < n; ++k) bb += (b[k] = b0[k] - ab * a[k]) * b[k];
                for (float &x : b) x /= sqrtf(bb);
                Mat z(3, std::vector<float>(n));
                const float tilt = trial % 4 == 0 ? 0.f : powf(10.f, -3.f - trial % 4);
                for (int i = 0; i < 3; ++i) {
                    float s = 0;
                    for (int k = 0; k < n; ++k) {
                        z[i][k] = cosf(1.0471976f * i) * a[k] + sinf(1.0471976f * i) * b[k] + tilt * (i - 1) * off[k];
                        s += z[i][k] * z[i][k];
                    }
                    for (float &x : z[i]) x /= sqrtf(s);
                }
                int steps = 0;
                if (orthonormalize(z, tol, steps) && error(z) > 2 * tol + 1e-6f)
                    return std::printf("coplanar vectors accepted: error %g (n=%d tol=%g tilt=%g)\n", error(z), n, tol, tilt), 1;
                // vectors near an orthonormal set converge, to the tolerance
                const int r = 2 + trial % (n / 2 - 1);
                Mat y(r);
                for (int i = 0; i < r; ++i) {
                    y[i] = std::vector<float>(n, 0.f);
                    y[i][i] = 1.f;
                    const std::vector<float> u = unit();
                    const float w = powf(10.f, -1.f - trial % 6);
                    for (int k = 0; k < n; ++k) y[i][k] += w * u[k] / sqrtf((float)r);
                }
                if (!orthonormalize(y, tol, steps)) return std::printf("near-orthonormal vectors refused (n=%d r=%d tol=%g)\n", n, r, tol), 1;
                if (error(y) > 1.02f * tol + 1e-6f) return std::printf("error %g left (n=%d r=%d tol=%g)\n", error(y), n, r, tol), 1;
            }
    return 0;
}
"""


def test_dependent_vectors_are_turned_away(tmp_path):
    src = tmp_path / "ns.cpp"
    src.write_text(DRIVER)
    exe = str(tmp_path / "ns")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
