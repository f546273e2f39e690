"""The tiled operand layout's index functions, on the host."""
import subprocess

from tests.host.build import build_host


def test_tile_offsets(tmp_path):
    exe = str(tmp_path / "tile_layout")
    build_host("tile_layout.hip", exe)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
