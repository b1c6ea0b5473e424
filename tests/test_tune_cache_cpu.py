"""The autotuner's cache, compiled from the library's own source with the host compiler: a choice is found
again under its key, also through the file, and an entry of a file written before the key named the
kernels' generation, or of another generation, is not used."""
import pathlib
import shutil
import subprocess

import pytest

ROOT = pathlib.Path(__file__).resolve().parents[1]
CSRC = ROOT / "paper_1802_03773_amd" / "csrc"

DRIVER = r"""
#include <cstdio>
#include "tune_cache.hpp"
int main(int argc, char** argv) {
  using namespace qrk;
  const std::string key = tune_key("gfx950", 0, 1, 512, 3, 48000000, 91, 3);
  TuneChoice c;
  if (argc > 2) {  // store a choice in the file
    tune_set_file(argv[1]);
    c.leaf_scale = 4.0;
    if (!tune_store(key, c)) return 3;
    printf("%s\n", key.c_str());
    return 0;
  }
  if (!tune_set_file(argv[1])) return 2;
  const bool found = tune_lookup(key, &c);
  printf("%d %g\n", found ? 1 : 0, c.leaf_scale);
  return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("tune")
    (d / "drv.cpp").write_text(DRIVER)
    subprocess.run([cxx, "-std=c++17", "-O1", f"-I{CSRC}", str(d / "drv.cpp"), str(CSRC / "tune_cache.cpp"), "-o",
                    str(d / "drv")], check=True)
    return lambda *a: subprocess.run([str(d / "drv"), *map(str, a)], check=True, capture_output=True, text=True,
                                     env={}).stdout.split()


def _entry(key):
    return ('{"version": 1, "entries": {\n  "%s": {"leaf_scale": 2, "leaf_queue": 0, "refine_scale": 0.5, "ms": 25.1}\n}}\n'
            % key)


def test_entries_of_other_kernels_are_not_used(driver, tmp_path):
    f = tmp_path / "t.json"
    (key,) = driver(f, "store")
    assert driver(f) == ["1", "4"]
    old = "gfx950/f32/bf16x3/P512/n3/rows67108864/L91/w3"  # the key before it named a generation
    assert key.startswith(old + "/")
    for k in (old, key + "9"):
        f.write_text(_entry(k))
        assert driver(f) == ["0", "1"], k
    f.write_text(_entry(key))
    assert driver(f) == ["1", "2"]
