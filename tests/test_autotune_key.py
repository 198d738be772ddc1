"""The autotuner's cache: a choice is served as long as its options mean what they
meant when it was timed."""
import json

import numpy as np

from paper_2509_06924_amd import autotune


def _key():
    return autotune.structure_key(np.array([0, 400]), np.array([0, 12]), np.array([0]), 0, "dev")


def test_choices_of_other_schedules_are_not_served(monkeypatch):
    now = _key()
    # (the key before schedules had a revision)
    old = {k: v for k, v in json.loads(now).items() if k != "schedules"}
    assert json.dumps(old, sort_keys=True) != now
    monkeypatch.setattr(autotune, "SCHEDULES", autotune.SCHEDULES + 1, raising=False)
    assert _key() != now
