"""Host-only checks of library internals compiled from the same sources
(no GPU is used): the per-template prologue's analytic sky derivatives."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run_host(tmp_path, name):
    exe = tmp_path / name
    subprocess.run(["/opt/rocm/bin/hipcc", "-std=c++17", "-O1",
                    "-I", os.path.join(ROOT, "paper_2201_00451_amd", "csrc"),
                    "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "host", name + ".cpp"), "-o", str(exe)],
                   check=True, capture_output=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip().endswith("OK"), out.stdout


def test_prologue_sky_derivatives(tmp_path):
    exe = tmp_path / "prologue_derivatives"
    subprocess.run(["/opt/rocm/bin/hipcc", "-std=c++17", "-O1",
                    "-I", os.path.join(ROOT, "paper_2201_00451_amd", "csrc"),
                    "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "host", "prologue_derivatives.cpp"),
                    "-o", str(exe)], check=True, capture_output=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip().endswith("OK"), out.stdout


def test_span_rule_bounds_the_quintics(tmp_path):
    run_host(tmp_path, "span_rule")


def test_launch_rules(tmp_path):
    run_host(tmp_path, "launch_rules")


def test_parameter_block_lanes(tmp_path):
    run_host(tmp_path, "parameter_lanes")
