"""The any-alignment loader's reads stay inside its operands (CPU only): tests/piece_bounds.cpp
compiles the kernel's own offset arithmetic (csrc/pieces.h) and walks every 16-byte read of small
products: rows of 16 bytes and more, edges of tiles and stages, row pitches, every K split."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def _walk(tmp_path, *args):
    exe = str(tmp_path / "piece_bounds")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(os.path.dirname(HERE), "include"),
                    os.path.join(HERE, "piece_bounds.cpp"), "-o", exe], check=True)
    return subprocess.run([exe, *args], capture_output=True, text=True)


def test_every_read_is_inside_its_operand(tmp_path):
    r = _walk(tmp_path)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[0]) > 10_000_000


def test_the_walk_sees_a_read_outside(tmp_path):
    """The same walk with the last stage read in place instead of ending at the row's end."""
    r = _walk(tmp_path, "in place")
    assert r.returncode == 1 and "reads [" in r.stdout
