"""The build entry point compiles the libraries without the test modules.

build() is run in a fresh interpreter in which no module of tests/ can be imported
and no file of tests/ is seen, with the compilers replaced by a record of their
commands: it ends normally, having asked for both HIP libraries and the oracle.
"""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SCRIPT = r"""
import importlib.abc, os, subprocess, sys

class NoTests(importlib.abc.MetaPathFinder):
    def find_spec(self, name, path=None, target=None):
        if name == "tests" or name.startswith("tests."):
            raise ImportError("build() imports " + name)

sys.meta_path.insert(0, NoTests())
sys.path.insert(0, ROOT)
exists = os.path.exists
os.path.exists = lambda p: exists(p) and os.path.join(ROOT, "tests") not in os.path.abspath(p)
commands = []

class Done:
    returncode, stdout, stderr = 0, "", ""

subprocess.run = subprocess.check_call = lambda cmd, **kw: commands.append(" ".join(map(str, cmd))) or Done()
os.replace = lambda a, b: None
import __graft_entry__
__graft_entry__.build()
for part in ("lbm_axi.hip", "lbm_axi_s16.hip", "lbm_no.hip", "lbm_oracle.c"):
    assert any(part in c for c in commands), (part, commands)
assert not any(os.path.join(ROOT, "tests") in c for c in commands), commands
print("built")
"""


def test_build_needs_no_test_module():
    r = subprocess.run([sys.executable, "-c", f"ROOT = {ROOT!r}\n" + SCRIPT], capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0 and "built" in r.stdout, r.stderr
