// The solver's kernels when `done` is stored while a workgroup starts, as the first workgroup of
// the launch may do: the workgroup goes one way as a whole, so what it writes is all of what it
// writes without a stop, or nothing.
#include "k_solver.hip"

#include <cstdio>
#include <random>

using namespace pafem;

namespace {

constexpr int kN = 2048;  // two workgroups of 1024

struct Vectors {
  std::vector<double> partials, x, r, d, q, dnew, diag, e, hist, z, zold;
  std::vector<float> df, qf, dnewf, dinvf;
  std::vector<uint8_t> mask;
  CGState st{};

  explicit Vectors(unsigned seed, double scale) {
    std::mt19937 g(seed);
    std::uniform_real_distribution<double> u(0.5, 1.5);
    auto fill = [&](std::vector<double>& v, size_t n) {
      v.resize(n);
      for (double& a : v) a = scale * u(g);
    };
    fill(partials, kPartials * kCGBlocks);
    for (auto* v : {&x, &r, &d, &q, &dnew, &diag, &z, &zold}) fill(*v, kN);
    fill(e, 1500);
    hist.assign(64, 0.0);
    for (auto* v : {&df, &qf, &dnewf, &dinvf}) {
      v->resize(kN);
      for (float& a : *v) a = float(u(g));
    }
    mask.assign(kN, 0);
    for (int i = 0; i < kN; i += 7) mask[size_t(i)] = 1;
    st.rz = st.rz_old = st.bb = 1.0;
    st.max_hist = 64;
  }
  // everything that a workgroup writes besides the state
  std::vector<double> outputs() const {
    std::vector<double> o;
    for (auto* v : {&x, &r, &d, &q, &dnew, &z, &zold}) o.insert(o.end(), v->begin(), v->end());
    for (auto* v : {&df, &qf, &dnewf}) o.insert(o.end(), v->begin(), v->end());
    return o;
  }
};

__global__ void direction_kernel(Direction dir, double* out) {
  __shared__ double scratch[2 * kCGThreads / kWave];
  double beta = 0.0;
  if (!direction_beta(dir, scratch, beta)) return;
  out[blockIdx.x * kCGThreads + threadIdx.x] = beta;
}

struct Case {
  const char* name;
  void (*launch)(Vectors&);
};

const Case kCases[] = {
    {"cg_update", [](Vectors& v) {
       launch_cg_update(&v.st, v.partials.data(), v.e.data(), int(v.e.size()), true, v.x.data(),
                        v.r.data(), v.d.data(), v.q.data(), v.diag.data(), nullptr, kN, nullptr);
     }},
    {"cg_direction", [](Vectors& v) {
       launch_cg_direction(&v.st, v.partials.data(), v.r.data(), v.diag.data(), v.d.data(),
                           v.dnew.data(), v.q.data(), v.mask.data(), v.hist.data(), kN, nullptr);
     }},
    {"fcg_update", [](Vectors& v) {
       launch_fcg_update(&v.st, v.partials.data(), v.e.data(), int(v.e.size()), v.x.data(),
                         v.r.data(), v.d.data(), v.q.data(), v.diag.data(), v.mask.data(),
                         v.z.data(), kN, nullptr);
     }},
    {"fcg_direction", [](Vectors& v) {
       launch_fcg_direction(&v.st, v.partials.data(), v.z.data(), v.d.data(), v.q.data(),
                            v.mask.data(), kN, nullptr);
     }},
    {"ir_update", [](Vectors& v) {
       launch_ir_update(&v.st, v.partials.data(), v.e.data(), int(v.e.size()), true, v.x.data(),
                        2.0, v.r.data(), v.df.data(), v.qf.data(), v.dinvf.data(), nullptr, kN,
                        nullptr);
     }},
    {"ir_direction", [](Vectors& v) {
       launch_ir_direction(&v.st, v.partials.data(), false, v.r.data(), v.dinvf.data(),
                           v.df.data(), v.dnewf.data(), v.qf.data(), v.mask.data(), kN, nullptr);
     }},
    {"direction of a fused apply", [](Vectors& v) {
       const Direction dir = make_direction(&v.st, v.partials.data(), v.hist.data(), v.r.data(),
                                            v.diag.data(), v.d.data(), v.dnew.data(), kN);
       hipLaunchKernelGGL(direction_kernel, dim3(2), dim3(kCGThreads), 0, nullptr, dir,
                          v.dnew.data());
     }},
};

// the second workgroup's part of the outputs
std::vector<double> second(const std::vector<double>& o) {
  std::vector<double> s;
  for (size_t i = 0; i < o.size(); ++i)
    if (i % kN >= kCGThreads) s.push_back(o[i]);
  return s;
}

}  // namespace

int main() {
  int bad = 0;
  for (const Case& c : kCases) {
    const Vectors start(1, 1.0);
    Vectors ref = start;
    c.launch(ref);
    const auto none = second(start.outputs()), all = second(ref.outputs());
    if (ref.st.done || all == none) {
      std::printf("%s: the launch without a stop does nothing\n", c.name);
      ++bad;
    }
    for (int first = 0; first < 2; ++first) {  // wave 0 before or after the others
      Vectors other(2, -7.0);                  // leaves its own sums in the LDS slots
      c.launch(other);
      Vectors v = start;
      emulate::gate.block = 1;
      emulate::gate.held = [first](int wave) { return (wave == 0) != (first == 0); };
      emulate::gate.between = [&v] { v.st.done = 1; };
      c.launch(v);
      emulate::gate = {};
      const auto got = second(v.outputs());
      const bool ok = got == none || got == all;
      std::printf("%s, wave 0 %s: %s\n", c.name, first == 0 ? "first" : "last",
                  got == all ? "all" : got == none ? "nothing" : "PART or from unwritten sums");
      if (!ok) ++bad;
    }
  }
  return bad ? 1 : 0;
}
