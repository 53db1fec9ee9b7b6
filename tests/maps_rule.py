"""The rule by which psi of a prompt's keys rides in the row pass's launch, run on the host: the text of csrc's own functions."""
import ctypes
import functools
import re
import subprocess
import tempfile
from pathlib import Path

CSRC = Path(__file__).resolve().parents[1] / "paper_2402_09398_amd" / "csrc"


def _function(name, file):
    src = (CSRC / file).read_text()
    at = src.rindex("\n", 0, src.index(f" {name}(const MlpArgs")) + 1
    return src[at:src.index("\n}\n", at) + 3]


def _constant(name):
    for path in sorted(CSRC.iterdir()):
        if path.suffix in (".h", ".hip") and (m := re.search(rf"^constexpr int {name} = \d+;", path.read_text(), re.M)):
            return m.group(0) + "\n"
    raise KeyError(name)


@functools.cache
def _library():
    text = "struct MlpArgs { int B, Hh, rpu, D, Rp, R; };\n" + _constant("kPsiTiles") + _constant("kPrefillWaves")
    text += _function("mlp_psi_blocks", "lessdec_mlp.h") + _function("mlp_weights_in_registers", "lessdec_mlp.hip")
    text += _function("rows_f16_take_maps", "lessdec_rows.hip")
    text += ('extern "C" int rides(int B, int Hh, int P, int D, int Rp, int R) '
             "{ return rows_f16_take_maps(MlpArgs{B, Hh, P, D, Rp, R}); }\n")
    with tempfile.TemporaryDirectory() as tmp:
        (Path(tmp) / "f.cpp").write_text(text)
        subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-o", f"{tmp}/f.so", f"{tmp}/f.cpp"], check=True)
        return ctypes.CDLL(f"{tmp}/f.so")


def rides(batch, heads, prompt, head_dim, hidden, rank):
    return bool(_library().rides(batch, heads, prompt, head_dim, hidden, rank))
