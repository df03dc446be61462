"""Cells of the tuned table that the tuner did not choose: marked as such, kept by
another run of the tuner, and without a trace in its logs."""

from __future__ import annotations

import json

from paper_2501_10653_amd import build, tune


def committed():
    with open(build.TUNED_JSON) as fh:
        return json.load(fh)


def cells(doc):
    out = {("single", k): v["cfg"] for k, v in doc["single"].items()}
    out.update({(s, k): v for s in ("batch", "serve") for k, v in doc[s].items()})
    return out


def test_another_run_of_the_tuner_keeps_them():
    doc = committed()
    want, waves = cells(doc), doc["batch_waves"]
    other = dict(vec=4, waves=4, unroll=8, seg=4, rp=1, ksplit=1)
    for section in ("single", "batch", "serve"):
        for key, cell in doc["chosen"][section].items():
            assert cell["why"] and want[section, key] == cell["cfg"]
            doc[section][key] = {"cfg": other, "us": 1.0} if section == "single" else other
    doc["batch_waves"] = 1024
    tune.keep_chosen(doc)
    assert cells(doc) == want and doc["batch_waves"] == waves
    assert all("us" not in doc["single"][k] for k in doc["chosen"]["single"])


def test_the_logs_are_the_tuners():
    """A row's choice is among its first pass and within a few percent of its best;
    every served cell that is not the log's choice is a chosen one."""
    doc = committed()
    for row in doc["serve_log"]:
        key = f"{row['N']}x{row['NT']}"
        first = {json.dumps(f["cfg"], sort_keys=True): f["us"] for f in row["first_pass"]}
        us = first[json.dumps(row["cfg"], sort_keys=True)]
        assert us <= 1.1 * min(first.values()) and 0.93 * us <= row["us"] <= 1.1 * us, key
        assert doc["serve"][key] == row["cfg"] or key in doc["chosen"]["serve"], key
