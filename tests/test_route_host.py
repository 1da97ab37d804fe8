"""lbm_launch_route and lbm_launch_steps on the host: argument errors and the structure's layout (CPU only)."""
import ctypes
import os
import subprocess

from paper_2312_10316_amd import lbm as L

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_null_arguments():
    route, steps = L.lbm_route(), ctypes.c_int32()
    assert L.lib().lbm_launch_route(None, ctypes.byref(route)) == L.LBM_E_STATE
    assert L.lib().lbm_launch_steps(None, ctypes.byref(steps)) == L.LBM_E_STATE


def test_struct_layout_matches_header(tmp_path):
    prog = tmp_path / "layout.c"
    prog.write_text('#include <stdio.h>\n#include <stddef.h>\n#include "lbm.h"\n'
                    'int main(void){printf("%zu %zu %zu %d\\n", sizeof(lbm_route), offsetof(lbm_route, waves), '
                    'offsetof(lbm_route, stores), (int)LBM_ROUTE_GAPLESS); return 0;}\n')
    exe = tmp_path / "layout"
    subprocess.run(["gcc", "-std=c11", f"-I{os.path.join(ROOT, 'include')}", str(prog), "-o", str(exe)], check=True)
    vals = [int(v) for v in subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()]
    assert vals == [ctypes.sizeof(L.lbm_route), L.lbm_route.waves.offset, L.lbm_route.stores.offset, L.LBM_ROUTE_GAPLESS]
