#include "columns_plane.hpp"

namespace apw {
template int columns_plane_n1<80>(const ColumnsCall &);
template int columns_plane_n1<81>(const ColumnsCall &);
template int columns_plane_n1<90>(const ColumnsCall &);
}  // namespace apw
