import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

GOLDEN = os.path.join(ROOT, "tests", "golden")


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")


def read_golden(name):
    """Rows of a whitespace-separated golden file (comments dropped)."""
    rows = []
    with open(os.path.join(GOLDEN, name)) as f:
        for line in f:
            line = line.split("#", 1)[0].strip()
            if line:
                rows.append(line.split())
    return rows


def sweep_strips(wl):
    """The automatic strip counts of the sweeps as explicit parameters, with
    which calls of any iteration count run the sweeps."""
    from bench import chain_strips

    q, k = chain_strips(wl, 0, 0)
    return dict(q_strips=q, k_strips=k)
