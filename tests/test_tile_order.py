"""The conv input gradients' rows in position order, on the host: tile_order.hip says what is checked."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_every_position_has_one_row(tmp_path):
    exe = str(tmp_path / "tile_order")
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O2", "-std=c++17", os.path.join(HERE, "tile_order.hip"), "-o", exe], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout == "528 problems\n", r.stdout
