"""The C-ABI library loads without a GPU and exports every function that
include/rnnt_greedy.h declares.  No compute calls."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "rnnt_greedy.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    names = re.findall(r"^\s*(?:const\s+char\s*\*|int)\s*\**\s*(\w+)\s*\(", text, flags=re.M)
    return sorted(set(names))


def test_header_declares_the_expected_entry_points():
    names = declared_functions()
    for must in ["rnnt_engine_create", "rnnt_engine_destroy", "rnnt_greedy_decode",
                 "rnnt_label_looping_decode", "tdt_label_looping_decode",
                 "rnnt_encoder_projection", "rnnt_engine_status", "rnnt_engine_stats",
                 "rnnt_status_string"]:
        assert must in names


def test_library_exports_every_declared_symbol():
    import paper_2406_03791_amd as pkg
    path = pkg.lib_path()
    if not os.path.exists(path):
        pytest.fail(f"{path} is not built: run `python -c 'import __graft_entry__ as g; g.build()'`")
    lib = ctypes.CDLL(path)
    for name in declared_functions():
        assert hasattr(lib, name), name
    assert set(pkg.binding.EXPORTS) == set(declared_functions())


def test_status_strings_and_null_checks_need_no_gpu():
    import paper_2406_03791_amd as pkg
    assert pkg.rnnt_status_string(0) == "ok"
    assert "NULL" in pkg.rnnt_status_string(-1)
    lib = pkg.load_library()
    assert lib.rnnt_engine_destroy(None) == -1
    assert lib.rnnt_engine_create(None, 1, 1, 0, None) == -1
    st = ctypes.c_int32(0)
    assert lib.rnnt_engine_status(None, ctypes.byref(st)) == -1
    assert lib.rnnt_engine_set_wait_limit(None, 0) == -1


def test_create_refuses_unsupported_shapes_before_touching_the_device():
    """The limits the header documents for rnnt_engine_create are checked on the host before any
    HIP call: F not a multiple of 16 and V1 above 65 535 are RNNT_ERR_UNSUPPORTED, a layer count
    or a blank index out of range and unknown flag bits are RNNT_ERR_SHAPE.  The weight pointers
    are never dereferenced on these paths, so dummies do."""
    import paper_2406_03791_amd as pkg
    from paper_2406_03791_amd.binding import _ModelDesc
    lib = pkg.load_library()

    def create(flags=0, **dims):
        d = _ModelDesc()
        base = dict(F=64, E=8, H=8, L=1, J=8, V1=5, blank=4, D=0)
        base.update(dims)
        for k, v in base.items():
            setattr(d, k, v)
        L = max(1, min(int(base["L"]), 8))
        fake = (ctypes.c_void_p * L)(*([0x1000] * L))
        for key in ("w_ih", "w_hh", "b_ih", "b_hh"):
            setattr(d, key, ctypes.cast(fake, ctypes.POINTER(ctypes.c_void_p)))
        for key in ("emb", "w_enc", "b_enc", "w_pred", "b_pred", "w_out", "b_out"):
            setattr(d, key, 0x1000)
        dur = (ctypes.c_int32 * 8)(0, 1, 2, 3, 4, 5, 6, 7)
        d.durations = ctypes.cast(dur, ctypes.POINTER(ctypes.c_int32))
        out = ctypes.c_void_p()
        return lib.rnnt_engine_create(ctypes.byref(d), 1, 1, flags, ctypes.byref(out))

    assert create(F=17) == -5
    assert create(F=24) == -5
    assert create(H=10) == -5 and create(J=6) == -5                  # widths are multiples of 4
    assert create(V1=65536, blank=0) == -5
    assert create(L=0) == -2 and create(L=5) == -2
    assert create(blank=5) == -2 and create(blank=-1) == -2
    assert create(D=9) == -2
    assert create(flags=64) == -2                                    # unknown flag bit
    assert create(flags=32) == -2                                    # 4-bit weights without the bfloat16 mode
    assert create(flags=pkg.RNNT_FLAG_BF16_ARITHMETIC | pkg.RNNT_FLAG_BF16_WEIGHTS) == -2
    assert create(flags=pkg.RNNT_FLAG_BF16_WEIGHTS | pkg.RNNT_FLAG_FP8_WEIGHTS) == -2
    assert create(flags=pkg.RNNT_FLAG_PLAIN_LAUNCH | pkg.RNNT_FLAG_COOPERATIVE_LAUNCH) == -2
    # multi-blank: needs big blanks, each spanning at least one frame
    assert create(flags=pkg.RNNT_FLAG_MULTI_BLANK) == -2
    assert create(flags=pkg.RNNT_FLAG_MULTI_BLANK, D=2) == -2         # the test's spans start at 0
    assert create(flags=pkg.RNNT_FLAG_BF16_WEIGHTS | pkg.RNNT_FLAG_FP8_WEIGHTS) == -2
    assert "not supported" in pkg.rnnt_status_string(-5)
    assert "scratch" in pkg.rnnt_status_string(-6)


def test_stage_planner_covers_k_and_fits_the_blocks():
    """Host logic of the weight packer, re-stated: every (groups, K) choice must
    cover K with nks slices of nsteps 16-byte loads (4 fp32, 8 bf16 or 16 e4m3 weights each),
    fill its passes over the blocks without an empty one, keep the zero padding small, and
    never cost more passes-times-steps than the unsliced fallback."""
    import subprocess
    import tempfile
    src = r'''
#include "plan.h"
#include <cstdio>
int main() {
  int bad = 0;
  for (int wt = 0; wt < 3; ++wt)
  for (int K = 4; K <= 2048; K += 4)
    for (int g = 1; g <= 300; g += (g < 40 ? 1 : 13)) {
      rnnt::StagePlan p = rnnt::make_stage_plan(K, g, wt);
      if (p.kper != (4 << wt)) bad++;
      if (p.kpad < K || p.kpad != p.nks * p.nsteps * p.kper || p.nsteps % rnnt::kStepUnroll) bad++;
      if (g * p.nks > rnnt::kBlocksPerWg * p.slots) bad++;
      if (g * p.nks <= rnnt::kBlocksPerWg * (p.slots - 1)) bad++;          // no empty pass
      if (p.nks > 1 && (p.kpad - K) * 8 > K + 8 * p.kper * rnnt::kStepUnroll) bad++;   // padding stays small
      // the fallback for a short LDS: more groups than blocks means unsliced tasks
      rnnt::StagePlan q = rnnt::make_stage_plan(K, g, wt, true);
      if (q.kpad < K || g * q.nks > rnnt::kBlocksPerWg * q.slots) bad++;
      if (q.slots > 1 && q.nks != 1) bad++;
      if (q.slots * (q.nsteps + rnnt::kPassOverheadSteps) < p.slots * (p.nsteps + rnnt::kPassOverheadSteps)) bad++;
    }
  std::printf("%d\n", bad);
  return bad != 0;
}'''
    with tempfile.TemporaryDirectory() as td:
        cpp = os.path.join(td, "t.cpp")
        open(cpp, "w").write(src)
        exe = os.path.join(td, "t")
        subprocess.run(["hipcc", "-std=c++17", "-I", os.path.join(ROOT, "paper_2406_03791_amd", "csrc"),
                        "-x", "hip", "--offload-arch=gfx950", cpp, "-o", exe], check=True,
                       capture_output=True)
        r = subprocess.run([exe], capture_output=True, text=True)
        assert r.returncode == 0 and r.stdout.strip() == "0", r.stdout
