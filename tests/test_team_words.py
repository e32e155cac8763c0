"""The numbering of a verification team's exchange words, explored on the host
over every order in which a small team's blocks can run."""

import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2609_21827_amd", "csrc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("team") / "team_words_model")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, "-o", exe,
                    os.path.join(HERE, "team_words_model.cpp")], check=True)
    return lambda which: subprocess.run([exe, which], check=True, capture_output=True,
                                        text=True, timeout=60).stdout.strip()


def test_no_block_waits_for_good(model):
    assert model("library") == "ok"


def test_the_model_tells_them_apart(model):
    """One set of words: a fast block overwrites the sum that a slower one has
    yet to see.  Sets by the layer alone: a word of the second set lasts until
    its 16-bit tag comes round again."""
    assert "waits for good" in model("one")
    assert "old word" in model("level")
