import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)
# the library prints each product's plan to stderr (captured): the tests that aim at
# one kernel read there whether it ran (gpu_util.plans)
os.environ.setdefault("ESPACE_PLAN_LOG", "1")


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")
    config.addinivalue_line("markers", "slow: large CPU work (full-size input generation)")
