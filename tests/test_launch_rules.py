"""Host checks of the rules that choose a launch by its sizes."""
import pytest

from test_abi_host import build_and_run_host_check


@pytest.mark.parametrize("name,said", [("shared_blocks_check", "shared blocks ok"), ("compression_rules_check", "compression rules ok")])
def test_rule(tmp_path, name, said):
    res = build_and_run_host_check(tmp_path, name)
    assert res.returncode == 0 and said in res.stdout, res.stdout + res.stderr
