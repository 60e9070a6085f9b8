"""The host payloads begin on cache lines. The binomial payload's inner loop is
short, and where the linker put the function at 48 past a line it took 1.57 times
as long (5,000 groups of 254 steps on one core 72.8 ms against 46.3)."""
import re
import shutil
import subprocess

import pytest

import paper_1805_02755_amd as ce


def test_host_functions_are_aligned():
    if shutil.which("nm") is None:
        pytest.skip("nm not available")
    text = subprocess.run(["nm", "-C", ce.LIB_PATH], check=True, capture_output=True, text=True).stdout
    at = {m.group(2): int(m.group(1), 16) for m in re.finditer(r"^([0-9a-f]+) [tT] ce::(binomial_groups|host_payloads)\(", text, flags=re.M)}
    assert set(at) == {"binomial_groups", "host_payloads"}
    assert all(a % 64 == 0 for a in at.values()), at
