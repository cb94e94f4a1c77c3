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
// us with 128 / 256, in brackets before the producers became faster (with 256):
//   512 channels, 5 objects of 200 000 points, 4 views 458 / 404 (429), 8 views 512 / 434 (471), 16 views 481 / 412 (438);
//     8 of 200 000, 3 views 671 / 621 (635); 12 of 200 000, 3 views 946 / 912 (909); 24 of 50 000, 8 views 477 / 491 (562);
//     12 of 100 000, 16 views 489 / 545 (588)
//   256 channels, 5 of 200 000, 8 views 223 / 299 (327); 16 of 100 000, 8 views 346 / 389 (415)
//   768 channels, 5 of 200 000, 8 views 660 / 596 (601); 16 of 100 000, 3 views 937 / 909 (917), 16 views 843 / 843 (883)
//   1024 channels, 8 of 100 000, 20 views 620 / 580 (580); with 128 12 of 50 000, 20 views 450 (475), 24 of 30 000 570 (605)
// At least eight tiles per workgroup beyond the resident ones (22 objects of 153 tiles, 2 views: 249 us with a workgroup per
// tile, 214 with 24 per object).
// units: channels / 256.
inline int fused_groups_per_object(int units, int producers, int n_obj, int resident, int max_tiles) {
  const bool few = units == 1 || 128 * n_obj >= (producers == 1 ? 4 : 6) * resident;
  const int want = few ? 128 : 256, most = max_tiles / 8 / kXcd * kXcd;
  return want < most ? want : most;
}

}  // namespace aura
