"""The rule that picks the register-resident engine's form against the forms that are built, over all sizes (no GPU needed)."""
import subprocess
from pathlib import Path

ROOT = Path(__file__).resolve().parent.parent


def test_every_size_has_its_form_and_every_form_a_size(tmp_path):
    exe = tmp_path / "resident_shape"
    build = subprocess.run(["g++", "-O2", "-std=c++17", f"-I{ROOT / 'include'}", f"-I{ROOT / 'paper_2410_01799_amd' / 'csrc'}",
                            str(ROOT / "tests" / "resident_shape_driver.cpp"), "-o", str(exe)], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout[-2000:]
    # f32: every matrix of 4 and more columns up to 4096 x 4096
    sizes, forms = run.stdout.split()[0], run.stdout.split()[2]
    assert int(sizes) > 4096 * 4093 and int(forms) > 0
