"""The library's rules of a step's forms (csrc/avs_forms.h), compiled for the
host: leaf shares of the 64-lane target and interface stage, waves per cell in
pass C."""
import ctypes as C
import functools
import os
import subprocess
import tempfile
from pathlib import Path

CSRC = Path(__file__).resolve().parents[1] / "paper_2212_05645_amd" / "csrc"

SRC = """
#include "avs_forms.h"
using namespace avs;
#define BY_TYPE(expr2d, expr2f, expr3d, expr3f) \
  (dim == 2 ? (fp32 ? expr2f : expr2d) : (fp32 ? expr3f : expr3d))
static const StageCost& stage(int dim, int fp32, int face) {
  return face ? (fp32 ? face_cost<float>() : face_cost<double>()) : dim == 2 ? target_cost<2>() : target_cost<3>();
}
extern "C" int shares(int dim, int fp32, int count, int nleaf, int numax, int face, int64_t most) {
  const StageCost& c = stage(dim, fp32, face);
  return BY_TYPE((lane_shares<2, double>(c, count, nleaf, numax, most)), (lane_shares<2, float>(c, count, nleaf, numax, most)),
                 (lane_shares<3, double>(c, count, nleaf, numax, most)), (lane_shares<3, float>(c, count, nleaf, numax, most)));
}
extern "C" double cost(int dim, int fp32, int count, int nleaf, int numax, int face, int shares) {
  return stage_cost(stage(dim, fp32, face), dim, count, nleaf, numax, shares);
}
extern "C" int wave(int dim, int fp32, int nc, int nleaf, int numax) {
  return BY_TYPE((passC_wave_form<2, double>(nc, nleaf, numax)), (passC_wave_form<2, float>(nc, nleaf, numax)),
                 (passC_wave_form<3, double>(nc, nleaf, numax)), (passC_wave_form<3, float>(nc, nleaf, numax)));
}
extern "C" int form(int dim, int fp32, int numax) {
  return BY_TYPE((lane_form<2, double>(numax)), (lane_form<2, float>(numax)), (lane_form<3, double>(numax)),
                 (lane_form<3, float>(numax)));
}
"""


@functools.lru_cache(maxsize=1)
def lib():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "forms.cpp"), os.path.join(d, "forms.so")
        Path(src).write_text(SRC)
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fPIC", "-shared", f"-I{CSRC}", src, "-o", so], check=True)
        h = C.CDLL(so)
    h.shares.argtypes = [C.c_int] * 6 + [C.c_int64]
    h.cost.argtypes, h.cost.restype = [C.c_int] * 7, C.c_double
    return h


def shares(dim, fp32, count, nleaf, numax, face, most=1 << 40):
    """Leaf shares of the target (face = 0) or the interface stage (1), 0 for
    the workgroup form."""
    return lib().shares(dim, fp32, count, nleaf, numax, face, most)


def cost(dim, fp32, count, nleaf, numax, face, nshares):
    """The rule's cost of the lane form, of the workgroup form for 0 shares."""
    return lib().cost(dim, fp32, count, nleaf, numax, face, nshares)


def form(dim, fp32, numax):
    return bool(lib().form(dim, fp32, numax))



def wave(dim, fp32, nc, nleaf, numax):
    """One wave per cell in pass C."""
    return bool(lib().wave(dim, fp32, nc, nleaf, numax))
