"""The launches of a level of gates and native MUXes on a fake device (CPU only; tests/host_checks/launches_check.cpp)."""
from test_host_client import run_on_fake_device


def test_gates_and_muxes_share_a_launch_where_it_is_shorter(tmp_path):
    run_on_fake_device("launches_check.cpp", tmp_path)
