// How many workgroups an object gets, and the pace they keep, where one launch of k_tile_fused fuses several objects and only rows
// leave it (aura_fuse_features, aura_fuse_selected).  Host only.
#pragma once

namespace aura {

constexpr int kXcd = 8;
constexpr int kFusedGroupsMax = 512;   // two workgroups per compute unit

// Many more workgroups per object than are resident at a time: those of an object share its tiles through the per-XCD tickets and
// are dispatched object after object, so the machine works on a few objects at a time - their depth and feature maps stay in
// L2, where with eight workgroups per object all 64 objects of a launch were in progress at once - and no workgroup is left
// with a fixed share of one object while others have run out.  128 where that makes four rounds of resident workgroups, six of
// those with four producers (one per compute unit), 256 where it makes fewer: the launch ends when the last, partly filled round
// has shared out its object.  256 channels take 128 always (their tiles are short, and every workgroup begins with one that
// nothing overlaps).
// us with 128 / 256:
//   one producer    512 channels, 5 objects of 200 000 points, 4 views 458 / 404, 8 views 512 / 434; 8 of 200 000, 3 views 671 / 621;
//     12 of 200 000, 3 views 946 / 912; 24 of 50 000, 8 views 477 / 491; 256 channels, 5 of 200 000, 8 views 223 / 299; 16 of
//     100 000, 8 views 346 / 389
//   four producers (product waves of 128 channels), many views    512 channels, 5 of 200 000, 16 views 469 / 420; 12 of 100 000 500 /
//     556; 24 of 40 000 500 / 514; 768 channels, 16 of 100 000, 16 views 841 / 864; 12 of 50 000 353 / 364; 1024 channels, 12 of
//     50 000, 20 views 476 / 499; 8 of 100 000 583 / 593 (takes 256); 24 of 30 000 636 / 635
//   four producers, few views    512 channels, 3 of 200 000, 6 views 277 / 247; 4 of 150 000, 4 views 248 / 256 (takes 256); 768
//     channels, 5 of 200 000, 8 views 584 / 526; 10 of 100 000, 4 views 552 / 532; 24 of 50 000, 4 views 645 / 634, 16 of 100 000, 3
//     views 854 / 836 and 50 of 40 000, 8 views 1040 / 1032 (take 128); 1024 channels, 5 of 200 000, 4 views 781 / 717; 8 of 100 000
//     604 / 588; 20 of 60 000 906 / 894 (takes 128); 24 of 30 000 552 / 549
// At least eight tiles per workgroup beyond the resident ones (22 objects of 153 tiles, 2 views: 249 us with a workgroup per
// tile, 214 with 24 per object).
// units: channels / 256.
inline int fused_groups_per_object(int units, int producers, int n_obj, int resident, int max_tiles) {
  const bool few = units == 1 || 128 * n_obj >= (producers == 1 ? 4 : 6) * resident;
  const int want = few ? 128 : 256, most = max_tiles / 8 / kXcd * kXcd;
  return want < most ? want : most;
}

}  // namespace aura
