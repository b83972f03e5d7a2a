"""The cache of captured steps on the CPU, over a stand-in for the HIP runtime: calls of one kind capture nothing after
the first two, no executable graph is destroyed before its last launch has ended, and graphs over two streams are
not captured during replays."""
import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_graph_cache(tmp_path):
    exe = str(tmp_path / "graph_cache")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(HERE, "stub"), os.path.join(HERE, "graph_cache_driver.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    print(out)
    four, two = re.findall(r"slots (\d): captures (\d+), then (\d+)", out)
    assert four == ("4", "4", "0")
    assert int(two[2]) > 0  # two slots do not hold the four graphs
    assert out.count("storm: captures 200, destroyed while running 0, waited 1, captured during replays 0") == 2
    assert re.findall(r"destroyed while running (\d+)", out) == ["0"] * 8
    assert re.findall(r"live (\d+)", out) == ["0"] * 4
