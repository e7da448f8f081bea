"""The driver that runs a graph and the layout of its plan belong together: a
plan laid out for the resident driver stores its short z-lists LANE_MAX apart
for LDS, one for launches stores them transposed.  graph.hip is linked here
against an engine without a device that refuses the resident driver, and the
plan that it is handed afterwards has to be one for launches."""
import os
import subprocess

import pytest

from paper_1603_02526_amd import build as B

SRC = r'''
#include <cstdarg>
#include <cstdio>
#include "graph_plan.h"

static int checks = 0, uploads = 0, bad = 0;

struct Refuser : admmg::EngineBase {
  admm_status resident_check(const admmg::Plan& p, int64_t, bool) override {
    ++checks;
    bad += !(p.no_tiles && p.resident);
    return ADMM_E_UNSUPPORTED;
  }
  admm_status upload(const admmg::Plan& p, const std::vector<double>&, double, double) override {
    ++uploads;
    bad += p.no_tiles || p.resident;
    // two lists of two contributions: in a plan for launches the second
    // list starts right behind the first
    const int64_t n_l = (int64_t)p.var_l.size();
    std::vector<int64_t> dst;
    for (const admmg::BucketDesc& b : p.bt)
      for (int64_t s = 0; s < b.n; ++s) dst.push_back(p.idx[b.dst_off + s] - p.l_base);
    bad += n_l != 2 || dst != std::vector<int64_t>{0, 1, n_l, n_l + 1};
    return ADMM_OK;
  }
  admm_status set_state(const double*, const double*, hipStream_t) override { return ADMM_OK; }
  admm_status run(int32_t, hipStream_t) override { return ADMM_OK; }
  admm_status run_profiled(int32_t, hipStream_t, double*, double*) override { return ADMM_OK; }
  admm_status get_z(double*, hipStream_t) override { return ADMM_OK; }
  admm_status get_slots(double*, int, hipStream_t) override { return ADMM_OK; }
  admm_status residuals(double*, double*, hipStream_t) override { return ADMM_OK; }
  void* z_ptr() override { return nullptr; }
};

namespace admmg {
EngineBase* make_engine_f32(int) { return new Refuser(); }
EngineBase* make_engine_f64(int) { return new Refuser(); }
}
namespace admmi {
admm_status set_err(admm_status s, const char* f, ...) {
  va_list ap;
  va_start(ap, f);
  std::vprintf(f, ap);
  va_end(ap);
  std::puts("");
  return s;
}
void clear_err() {}
admm_status probe_device(int) { return ADMM_OK; }
}
extern "C" hipError_t hipSetDevice(int) { return hipSuccess; }
extern "C" const char* hipGetErrorString(hipError_t) { return ""; }

int main() {
  for (int prec : {ADMM_FP32, ADMM_FP64}) {
    admm_graph* g = nullptr;
    const int32_t dims[2] = {1, 1}, ids[2] = {0, 1};
    const double lam[1] = {0.5};
    if (admm_graph_create(2, dims, prec, &g)) return 1;
    for (int k = 0; k < 2; ++k)
      if (admm_graph_add_factors(g, ADMM_F_L2, 2, 1, ids, lam, 1, 1)) return 2;
    if (admm_graph_finalize(g, 0)) return 3;
    admm_graph_info info;
    if (admm_graph_info_get(g, &info)) return 4;
    bad += info.driver != ADMM_DRIVER_GRAPH || info.resident_lds_bytes != 0;
    if (admm_graph_destroy(g)) return 5;
  }
  std::printf("checks %d uploads %d bad %d\n", checks, uploads, bad);
  return checks == 2 && uploads == 2 && bad == 0 ? 0 : 6;
}
'''


def test_refused_resident_driver_runs_a_plan_for_launches(tmp_path):
    if not os.path.exists(B.HIPCC):
        pytest.skip("hipcc not installed")
    src = tmp_path / "fallback.hip"
    src.write_text(SRC)
    objs = []
    for f in (str(src), os.path.join(B.CSRC, "graph.hip")):
        objs.append(str(tmp_path / (os.path.basename(f) + ".o")))
        subprocess.run([B.HIPCC, *B.FLAGS, "-O1", "--offload-host-only", "-c", f, "-o", objs[-1]], check=True)
    exe = str(tmp_path / "fallback")
    subprocess.run(["g++", *objs, "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
