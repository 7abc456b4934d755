"""The measured traffic that bench.py reports holds for the sources of the kernel it was
counted on: the hash covers every file that kernel is compiled from, so that a change to
any of them takes the figure back."""
import importlib.util
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = "paper_2308_13476_amd/csrc/"


def included(name, seen):
    seen.add(name)
    with open(os.path.join(ROOT, CSRC, name)) as fh:
        for inc in re.findall(r'^#include "(hm_[^"]+)"', fh.read(), re.M):
            if inc not in seen:
                included(inc, seen)
    return seen


def test_traffic_hash_covers_the_kernel_and_its_headers():
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    files = included("hm_gmres_f32.hip", set()) | included("hm_gmres_f64.hip", set())
    assert any("void k_gm_march(" in open(os.path.join(ROOT, CSRC, f)).read() for f in files)
    assert files <= {os.path.basename(p) for p in bench.TRAFFIC_SOURCES}
    for w in ("mp2a", "beyond_cache", "batch64"):
        assert os.path.exists(os.path.join(ROOT, bench.MEASURED_TRAFFIC[w]["profile"]))
