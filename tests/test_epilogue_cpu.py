"""The GEMM epilogue's element-wise form (gemm_epilogue.h), compiled for the host and run over
every alignment of its output and residual, with each vector access checked against the
alignment its type needs: a base offset by elements, which a caller may pass, takes
element accesses."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = next((c for c in ("/opt/rocm/bin/hipcc", shutil.which("hipcc")) if c and os.path.exists(c)), None)

SOURCE = r"""
#include "gemm_epilogue.h"
#include <cstdio>
#include <vector>
using namespace dn;

// [M][ld] outputs and residuals, both offset by `off` elements from a 16-byte boundary
template <typename R, typename O> int check(int off, int ld, int n_store, const char* what) {
  const int M = 3, N = 8;
  std::vector<float4> rs(M * ld), os(M * ld);  // 16-byte aligned storage, larger than needed
  R* r = reinterpret_cast<R*>(rs.data()) + off;
  O* o = reinterpret_cast<O*>(os.data()) + off;
  for (int i = 0; i < M * ld; ++i) r[i] = static_cast<R>(0.25f * i), o[i] = static_cast<O>(-1.f);
  float bias[N];
  for (int n = 0; n < N; ++n) bias[n] = n;
  GemmParams p;
  p.M = M;
  p.N = N;
  p.n_store = n_store;
  p.bias = bias;
  p.resid = r;
  p.resid_f32 = sizeof(R) == 4;
  p.ldr = ld;
  p.out = o;
  p.out_f32 = sizeof(O) == 4;
  p.ldo = ld;
  for (int m = 0; m < M; ++m)
    for (int n = 0; n < N; n += 4) {
      float v[4] = {1.f, 2.f, 3.f, 4.f};
      epilogue_group<bf16>(p, m, n, v);
    }
  for (int m = 0; m < M; ++m)
    for (int n = 0; n < ld; ++n) {
      const float want = n < n_store ? static_cast<float>(static_cast<O>((n % 4 + 1) + bias[n % N] + static_cast<float>(r[m * ld + n])))
                                     : -1.f;
      if (static_cast<float>(o[m * ld + n]) != want) {
        std::printf("%s off %d ld %d n_store %d: [%d][%d] %f, not %f\n", what, off, ld, n_store, m, n,
                    static_cast<float>(o[m * ld + n]), want);
        return 1;
      }
    }
  return 0;
}

int main() {
  int bad = 0;
  for (int off = 0; off < 8; ++off)
    for (int ld : {8, 9, 12})
      for (int n_store : {5, 8}) {
        bad |= check<float, float>(off, ld, n_store, "fp32 + fp32");
        bad |= check<bf16, bf16>(off, ld, n_store, "bf16 + bf16");
        bad |= check<float, bf16>(off, ld, n_store, "fp32 -> bf16");
        bad |= check<bf16, float>(off, ld, n_store, "bf16 -> fp32");
      }
  return bad;
}
"""


@pytest.mark.skipif(HIPCC is None, reason="no hipcc")
def test_element_wise_epilogue_takes_any_alignment(tmp_path):
    src = tmp_path / "epilogue.hip"
    src.write_text(SOURCE)
    exe = tmp_path / "epilogue"
    # host code only; a misaligned access traps
    cmd = [HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
           os.path.join(ROOT, "paper_2511_06724_amd", "csrc"), "-Xarch_host", "-fsanitize=alignment", "-Xarch_host",
           "-fsanitize-trap=alignment", str(src), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, f"exit {r.returncode}: {r.stdout}"
