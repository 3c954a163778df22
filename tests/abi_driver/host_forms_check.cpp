// What the C ABI's host logic (csrc/lb_api.hip) enqueues, and the storage form it
// names for the buffer that each launch reads: every launcher is replaced by one
// that writes a line.  Run without a GPU.  The stream can be made to report that
// it is being captured.  Exit status 0 if every expectation holds.
#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>

#include "d2q37_launch.h"
#include "lb.h"

namespace {
std::vector<std::string> lines;
bool capturing = false;
hipError_t line(const std::string& what) {
  lines.push_back(what);
  return hipSuccess;
}
std::string read(const char* what, const d2q37::Geom& g) {
  const char* form = g.form == d2q37::kFormFull        ? "full"
                     : g.form == d2q37::kFormCoeff     ? "coeff"
                     : g.form == d2q37::kFormUnknown   ? "unknown"
                                                       : "probably coeff";
  return std::string(what) + " " + form;
}
}  // namespace

extern "C" hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* status) {
  *status = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}

namespace d2q37 {
hipError_t current_device(int* dev) {
  *dev = 0;
  return hipSuccess;
}
hipError_t launch_zero(void*, size_t, hipStream_t) { return line("zero"); }
hipError_t launch_halo(void*, const Geom& g, int, hipStream_t) { return line(read("halo", g)); }
hipError_t launch_fused(const void*, void*, const Geom& g, const Phys&, int, int, double*,
                        hipStream_t) {
  return line(read(g.steps == 2 ? "two steps" : "step", g));
}
hipError_t launch_propagate(const void*, void*, const Geom& g, int, hipStream_t) {
  return line(read("propagate", g));
}
hipError_t launch_bc(void*, const Geom& g, const Phys&, int, hipStream_t) {
  return line(read("bc", g));
}
hipError_t launch_propagate_variant(const void*, void*, const Geom& g, int, int, hipStream_t) {
  return line(read("propagate", g));
}
hipError_t launch_collide_mfma(const void*, void*, const Geom& g, const Phys&, int, hipStream_t) {
  return line(read("collide", g));
}
hipError_t launch_collide(const void*, void*, const Geom& g, const Phys&, int, int, hipStream_t) {
  return line(read("collide", g));
}
hipError_t launch_init_feq(void*, const double*, const double*, const double*, const double*,
                           const Geom&, const Phys&, int, hipStream_t) {
  return line("init");
}
hipError_t launch_moments(const void*, double*, double*, double*, double*, const Geom& g,
                          const Phys&, int, hipStream_t) {
  return line(read("moments", g));
}
hipError_t launch_pack(const void*, void*, const Geom& g, int, hipStream_t) {
  return line(read("pack", g));
}
hipError_t launch_unpack(const void*, void*, const Geom&, int, hipStream_t) {
  return line("unpack");
}
hipError_t launch_populations_f64(const void*, double*, const Geom& g, const Phys&, int,
                                  hipStream_t) {
  return line(read("populations", g));
}
hipError_t launch_check(const void*, unsigned int*, const Geom& g, const Phys&, int, hipStream_t) {
  return line(read("check", g));
}
int observable_chunks(const Geom&) { return 4; }
hipError_t launch_observables(const void*, double*, double*, double*, const Geom& g, const Phys&,
                              int, double, double, hipStream_t) {
  return line(read("observables", g));
}
int loss_ke_blocks(const Geom&) { return 4; }
hipError_t launch_loss_ke(const void*, double*, double*, double*, const Geom& g, hipStream_t) {
  return line(read("loss", g));
}
hipError_t launch_adjoint_step(const double*, const double*, double*, const Geom&, const Phys&,
                               int, hipStream_t) {
  return line("adjoint step");
}
hipError_t launch_adjoint_mu(const double*, const double*, bool, double*, const Geom&, const Phys&,
                             int, hipStream_t) {
  return line("adjoint mu");
}
hipError_t launch_adjoint_gather(const double*, double*, const Geom&, hipStream_t) {
  return line("adjoint gather");
}
hipError_t launch_zero_pad_rows(void*, const Geom&, int, hipStream_t) { return line("pads"); }
hipError_t launch_init_adjoint(const double*, const double*, const double*, const double*,
                               const double*, double*, double*, double*, double*, const Geom&,
                               hipStream_t) {
  return line("init adjoint");
}
hipError_t static_scratch(void**) { return hipErrorNoDevice; }
}  // namespace d2q37

namespace {

int failures = 0;

struct Lattice {
  lb_ctx* ctx = nullptr;
  lb_params par;
  void* ws = nullptr;
  size_t bytes = 0;
  std::vector<double> v;
  lb_lattice lat;

  explicit Lattice(int regularize, int lx = 400, int ly = 300, int precision = LB_FP64,
                   int ybc = LB_Y_WALLS)
      : par{0.7, 0.0, -1e-4, 1.5, 0.5, 1.0, regularize, LB_KERNEL_FUSED, 0, 0},
        v(1),
        lat{lx, ly, precision, ybc, LB_LAYOUT_COLUMN, 0} {
    lb_workspace_bytes(&lat, &par, &bytes);
    ws = std::aligned_alloc(256, 256);  // nothing reads it
    init();
  }
  void init() {
    lb_free(ctx);
    if (lb_init(&lat, &par, ws, bytes, nullptr, v.data(), v.data(), v.data(), v.data(), &ctx))
      ++failures;
  }
  void set(int regularize, int kernel = LB_KERNEL_FUSED) {
    par.regularize = regularize;
    par.kernel = kernel;
    if (lb_set_params(ctx, &par)) ++failures;
  }
  ~Lattice() {
    lb_free(ctx);
    std::free(ws);
  }
};

void plain_bgk_after_a_recording() {
  // as many launches as steps, inside the recording and after it
  Lattice l(0);  // 400 x 300: single steps
  lb_step(l.ctx, 2);
  for (int n : {4, 3}) {
    capturing = n == 4;
    lines.clear();
    lb_step(l.ctx, n);
    capturing = false;
    int others = 0;
    for (const std::string& s : lines) others += s.compare(0, 5, "step ") != 0;
    if (int(lines.size()) != n || others) {
      ++failures;
      std::printf("%d plain BGK steps take %d launches, %d of them other than steps\n", n,
                  int(lines.size()), others);
    }
  }
}

// The first launch of every call that reads an FP64 buffer has to look at its
// word: a graph may have run since the last call, whatever context recorded it.
void no_form_is_kept_between_calls() {
  using Strings = std::vector<std::string>;
  const auto enqueues = [](const char* what, int rc, const Strings& want) {
    if (rc != LB_OK || lines != want) {
      ++failures;
      std::printf("%s (status %d) enqueues", what, rc);
      for (const std::string& s : lines) std::printf(", %s", s.c_str());
      std::printf(" instead of");
      for (const std::string& s : want) std::printf(", %s", s.c_str());
      std::printf("\n");
    }
    lines.clear();
  };
  double d[8] = {};
  for (int state : {0, 1, 2, 3}) {  // what the calls before left: start, steps, set_state, collide
    for (int reg : {1, 0}) {
      Lattice l(reg);
      const std::string guess = reg && state < 2 ? " probably coeff" : " unknown";
      if (state == 1) lb_step(l.ctx, 2);
      if (state == 2) lb_set_state(l.ctx, d);
      if (state == 3) lb_collide(l.ctx);
      lines.clear();
      enqueues("get_state", lb_get_state(l.ctx, d), {"pack" + guess});
      enqueues("populations", lb_get_populations(l.ctx, d), {"populations" + guess});
      enqueues("moments", lb_moments(l.ctx, d, d, d, d), {"moments" + guess});
      enqueues("observables", lb_observables(l.ctx, nullptr, d), {"observables" + guess});
      enqueues("loss_ke", lb_loss_ke(l.ctx, d, nullptr), {"loss" + guess});
      enqueues("halo", lb_halo(l.ctx), {"halo" + guess});
      enqueues("propagate", lb_propagate(l.ctx), {"propagate" + guess});
      enqueues("bc", lb_bc(l.ctx), {"bc unknown"});
      enqueues("get_scratch", lb_get_scratch(l.ctx, d), {"pack unknown"});
      const std::string then = reg ? " coeff" : " full";
      enqueues("step", lb_step(l.ctx, 2), {"step" + guess, "step" + then});
      enqueues("step_record", lb_step_record(l.ctx, 2, d),
               {reg ? "step probably coeff" : "step unknown", "step" + then});
      enqueues("run_observed", lb_run_observed(l.ctx, 2, 1, d),
               {reg ? "step probably coeff" : "step unknown", "observables" + then,
                "step" + then, "observables" + then});
      enqueues("collide", lb_collide(l.ctx), {"collide unknown"});
      l.set(reg, LB_KERNEL_SPLIT);
      enqueues("split step", lb_step(l.ctx, 1),
               {"halo unknown", "propagate unknown", "bc full", "collide full"});
      l.init();  // restarted on its workspace
      lines.clear();
      enqueues("get_state", lb_get_state(l.ctx, d), {"pack unknown"});
    }
  }
  {
    Lattice l(1, 1000, 1000);  // two steps per launch
    lines.clear();
    enqueues("five steps", lb_step(l.ctx, 5),
             {"two steps probably coeff", "two steps coeff", "step coeff"});
    lb_set_state(l.ctx, d);
    lines.clear();
    enqueues("six steps", lb_step(l.ctx, 6),
             {"step unknown", "two steps coeff", "two steps coeff", "step coeff"});
    Lattice p(0, 1000, 1000);
    lines.clear();
    enqueues("five plain BGK steps", lb_step(p.ctx, 5),
             {"two steps unknown", "two steps full", "step full"});
    Lattice f(1, 40, 30, LB_FP32_SHIFTED);  // always populations
    lines.clear();
    enqueues("FP32", lb_step(f.ctx, 1) | lb_get_state(f.ctx, d), {"step full", "pack full"});
  }
}

// lb_step_launches counts what lb_step enqueues.
void launches_are_counted() {
  for (int reg : {1, 0})
    for (int lx : {64, 256, 1000})
      for (int n : {0, 1, 4, 5, 6, 9, 20}) {
        Lattice l(reg, lx, lx == 64 ? 48 : 700);
        lines.clear();
        lb_step(l.ctx, n);
        int count = -1;
        if (lb_step_launches(&l.lat, &l.par, n, &count) || count != int(lines.size())) {
          ++failures;
          std::printf("%d steps of %d columns: %d launches, %d counted\n", n, lx,
                      int(lines.size()), count);
        }
      }
}

}  // namespace

int main() {
  launches_are_counted();
  no_form_is_kept_between_calls();
  plain_bgk_after_a_recording();
  std::printf("%d failure(s)\n", failures);
  return failures != 0;
}
