"""Host check of the rule that gives a 32-row block of queries to two waves."""
from test_abi_host import build_and_run_host_check


def test_rule_of_shared_blocks(tmp_path):
    res = build_and_run_host_check(tmp_path, "shared_blocks_check")
    assert res.returncode == 0 and "shared blocks ok" in res.stdout, res.stdout + res.stderr
