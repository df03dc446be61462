"""The host side of the launches without a GPU: which buffers and launches a
call takes, on the CPU, through a C program that stands in for the HIP runtime
(tests/c_fake_device.c)."""

from __future__ import annotations

import os
import shutil
import subprocess

import pytest

from paper_2501_10653_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.skipif(not shutil.which("gcc"), reason="needs gcc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    _lib.load()
    exe = str(tmp_path_factory.mktemp("fake") / "c_fake_device")
    pkg = os.path.dirname(_lib.LIB_PATH)
    subprocess.run(["gcc", "-O1", "-Wall", "-Werror", "-rdynamic", "-pthread", "-I",
                    os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "c_fake_device.c"),
                    "-o", exe, "-L", pkg, "-liqa_hip", f"-Wl,-rpath,{pkg}",
                    "-Wl,--allow-shlib-undefined"], check=True)
    return exe


def scenario(program, name):
    res = subprocess.run([program, name], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout + res.stderr


def test_per_thread_streams_share_no_workspace(program):
    """hipStreamPerThread is one handle for a stream of every host thread."""
    scenario(program, "per_thread")


def test_buffers_that_no_caller_asked_for_are_bounded(program):
    """Merges and default splits without a prepare rule, on ever new streams."""
    scenario(program, "many_streams")


def test_prepare_covers_images_at_any_address(program):
    """iqa_prepare(N, NT), then the capture of images off a 16-byte boundary."""
    scenario(program, "prepared")


def test_the_largest_images_can_be_launched(program):
    """HIP launches fewer than 2^32 work items; 2^17 pixels a side with tiles of
    4 pixels are 2^30 tiles."""
    scenario(program, "sizes")


def test_batches_of_any_number_of_units_can_be_launched(program):
    """The batch kernels are persistent: their grid is capped, not refused."""
    scenario(program, "many_units")


def test_default_configuration_passed_back_is_the_default_launch(program):
    """iqa_tiles_cfg with what iqa_default_cfg returned is captured as iqa_tiles is."""
    scenario(program, "passed_back")


def test_pyramid_refuses_what_the_chain_of_merges_refuses(program):
    """More than 2^31 - 1 tiles in a level: IQA_ERR_SHAPE."""
    scenario(program, "pyramid_sizes")
