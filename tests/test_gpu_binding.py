"""What Caches.render returns does not depend on the poses' Python type."""
import pytest

from paper_2204_02585_amd import scenes

pytestmark = pytest.mark.gpu


def test_outputs_are_plain_tensors():
    import torch
    from paper_2204_02585_amd import binding

    class Poses(torch.Tensor):
        pass

    sc = scenes.make_scene("tiny")
    caches = binding.caches_from_scene(sc)
    try:
        plain = torch.from_numpy(sc.poses).cuda()
        want = caches.render(plain, sc.intrinsics, sc.near, sc.far, sc.config.n_samples)
        for poses in (plain.as_subclass(Poses), torch.nn.Parameter(plain)):
            got = caches.render(poses, sc.intrinsics, sc.near, sc.far, sc.config.n_samples)
            for a, b in zip(got, want):
                assert type(a) is torch.Tensor and not a.requires_grad and torch.equal(a, b)
    finally:
        caches.close()
