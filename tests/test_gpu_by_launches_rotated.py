"""The rotated crystal, solving by launches (by_launches.py)."""
from by_launches import by_launches  # noqa: F401
from test_gpu_rotated import (case, pytestmark, test_rotated_mixed_form_matches_fp64,  # noqa: F401
                              test_rotated_steps_match_oracle)
