"""The autotuner's choices at known costs of every launch (no GPU needed)."""

from test_noise_shape import _run


def test_autotune_keeps_several_steps_per_launch(tmp_path):
    assert _run(tmp_path, "autotune_check").count(": 6 launches of several steps\n") == 2
