"""Parity with the oracle, solving by launches (by_launches.py)."""
from by_launches import by_launches  # noqa: F401
from test_gpu_parity import (case, pytestmark,  # noqa: F401
                             test_cube47_sphere_steps_match_oracle,
                             test_gs_row_blocks_of_the_mixed_form_match_oracle, test_operators_match_oracle,
                             test_solves_match_oracle, test_step_cube10_twenty_steps,
                             test_step_on_the_five_tet_split, test_step_with_inclusion_field_and_stress)
