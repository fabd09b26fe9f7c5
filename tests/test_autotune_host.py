"""The autotuner's choices at known costs of every launch (no GPU needed)."""

from test_noise_shape import _run


def test_autotune_choices_at_known_costs(tmp_path):
    out = _run(tmp_path, "autotune_check")
    # several D2Q9 steps per launch, without and with statistics
    assert out.count(": 6 launches of several steps\n") == 2
    # trial steps follow one another as steps of a run do
    assert "\n0 trials under noise drawn before\n" in out
    # in-place pairs of row tiles on a small box that leaves them mostly empty
    assert out.endswith("pairs of row tiles\n")
