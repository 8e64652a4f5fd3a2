"""The traffic figures that bench.py reports belong to the sources they were counted with."""
import glob
import os
import re

import pytest

import bench

CSRC = os.path.join(bench.ROOT, "paper_2511_01282_amd", "csrc")
STAGES = {"attention": ("attention.hip", "attn_stream.hip"), "lm_head": ("lmhead.hip", "lmhead_pair.hip"),
          "vocab_pass": ("vocab.hip",)}
NO_STAGE = {"api.hip", "probe.hip", "stochastic.hip"}


def test_every_kernel_file_belongs_to_a_stage():
    named = {f for files in STAGES.values() for f in files}
    assert named | NO_STAGE == {os.path.basename(f) for f in glob.glob(os.path.join(CSRC, "*.hip"))}


@pytest.mark.parametrize("stage", sorted(STAGES))
def test_stage_hash_covers_the_stage_and_its_headers(stage):
    sources = set(bench.STAGE_SOURCES[stage][0])
    assert sources >= set(STAGES[stage])
    for f in STAGES[stage]:
        headers = re.findall(r'#include "([^/"]+)"', open(os.path.join(CSRC, f)).read())
        assert set(headers) - {"common.hpp", "kernels.hpp"} <= sources
