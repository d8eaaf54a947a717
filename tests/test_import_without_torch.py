"""Building and importing the package need no torch: it is imported by the first call, which brings tensors anyway."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run(code):
    p = subprocess.run([sys.executable, "-c", "import sys; sys.modules['torch'] = None\n" + code], cwd=ROOT, text=True,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    assert p.returncode == 0, p.stdout[-2000:]


def test_package_imports():
    run("import paper_2605_23163_amd as F; assert F.library_path().endswith('.so'); F.fdd_block_attn; F.FddError")


def test_build_module_imports():
    run("import paper_2605_23163_amd.build as b; assert len(b.sources()) >= 5")
